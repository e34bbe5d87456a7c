"""GPU parity: the HIP library, called through its C ABI, against the float64 CPU
checker on the same seeded inputs.  Bars: f32 |g-r| <= 1e-5|r| + 1e-5 max|r|;
bf16 |g-r| <= 2e-2; every count bit-exact."""
import math

import numpy as np
import pytest

from oracle import attn_oracle as orc
from paper_2012_01114_amd import attnring as ar
from paper_2012_01114_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu

FULL, SYM, CAUSAL = inputs.SCHEME_FULL, inputs.SCHEME_SYMMETRIC, inputs.SCHEME_CAUSAL


def _matrix_core_path(w, scheme):
    """Shapes the library runs on its matrix-core kernels (32 x 32 score blocks per wavefront)."""
    return w.dtype == "bf16" and w.d_k in (64, 128) and w.d_model % 8 == 0 and scheme != SYM


def _run_and_compare(w, scheme, scale=0.0, lens=None, zero_wq=False, sym_no_proj=False, flags=0):
    print(f"[case] {w.name} B{w.batch} N{w.n} D{w.d_model} H{w.n_heads} d{w.d_k} P{w.p} {w.dtype} "
          f"scheme={scheme} scale={scale} lens={'yes' if lens is not None else 'no'}", flush=True)
    stored, f64 = inputs.make_inputs(w, zero_wq=zero_wq)
    stored["lens"] = lens
    if sym_no_proj:
        stored["Wq"] = f64["Wq"] = None
    if scheme == SYM:
        stored["Wk"] = stored["Wv"] = None
    run = hp.GpuRun(w, stored, scale=scale, flags=flags)
    try:
        got, stats = run.forward(scheme)
    finally:
        run.close()
    ref = hp.oracle_forward(w, f64, scheme, scale, lens=lens)
    err = hp.tol_check(got, ref, w.dtype)
    hp.report_max_err(f"{w.name} B{w.batch} N{w.n} D{w.d_model} H{w.n_heads} d{w.d_k} scheme={scheme} "
                      f"scale={scale} lens={'yes' if lens is not None else 'no'} flags={flags}", err, w.dtype)
    hp.check_counts(stats, hp.oracle_counts(w, scheme, lens))
    if _matrix_core_path(w, scheme) and not (flags & ar.ATTN_FLAG_NO_SKIP):
        # what the matrix-core kernel issued, against the blocks the pair predicate makes necessary
        assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, lens)
    return err, stats


# ---- workload 1: Tiny, f32, all three schemes, both scales ---------------------------------
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
@pytest.mark.parametrize("scale", [0.0, 1.0])
def test_tiny(scheme, scale):
    w = inputs.with_scheme(inputs.WORKLOADS["tiny"], scheme)
    _, stats = _run_and_compare(w, scheme, scale)
    expect = {FULL: (16, 256), SYM: (12, 192), CAUSAL: (10, 160)}[scheme]
    assert (stats["tiles_executed"], stats["pairs_executed"]) == expect
    assert stats["proj_gemms"] == (1 if scheme == SYM else 3)


# ---- float path on ragged shapes (several partitions, odd sizes, padding) --------------------
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (2, 50, 24, 3, 20, 10),
    (1, 63, 17, 2, 33, 9),
    (3, 96, 40, 1, 130, 3),     # d_k > 128, rows per partition > one wavefront pass
    (1, 7, 5, 1, 3, 7),
])
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_float_path_ragged(shape, scheme, dtype):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("ragged", B, n, D, H, d, p, dtype, scheme, 4242 + n)
    _run_and_compare(w, scheme, 0.0)
    if scheme != SYM:
        lens = np.random.default_rng(n).integers(0, n + 1, B).astype(np.int32)
        lens[0] = max(1, n // 3)
        _run_and_compare(w, scheme, 0.3, lens=lens)


# ---- float path at the edges of its tiles: 64 x 64 GEMM tiles, 64-key tiles, 16-row and 16-column blocks,
# and both ways of sharing a row tile's keys (512 row tiles of 64 rows is where they change)
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (1, 65, 33, 1, 17, 13),       # one row, one k and one column past a tile
    (2, 64, 64, 2, 48, 8),        # whole tiles, a single key tile
    (2, 192, 96, 2, 64, 24),      # keys shared by the wavefronts, whole tiles
    (1, 129, 100, 3, 100, 43),    # rows of d in whole 16-byte pieces, last block partly used
    (1, 80, 16, 1, 256, 5),       # the largest head
    (3, 70, 72, 4, 48, 7),        # bf16: pieces straight into LDS, last slice of d_model cut, vectors as one run
    (2, 130, 64, 2, 32, 13),      # the same with whole slices
    (32, 72, 20, 16, 12, 9),      # 1024 row tiles: a wavefront for every 16 rows
    (64, 66, 16, 8, 33, 33),      # the same with unaligned rows
])
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_float_path_tile_edges(shape, scheme, dtype):
    B, n, D, H, d, p = shape
    if dtype == "bf16" and d == 64:
        D += 1                    # not a multiple of 8: off the 16-bit matrix-core path
    w = hp.custom_workload("float_edges", B, n, D, H, d, p, dtype, scheme, 6100 + n)
    _, stats = _run_and_compare(w, scheme, 0.0)
    assert (stats["phys_br"], stats["phys_bc"]) == (16, 16)
    if scheme == SYM:
        assert stats["phys_tiles_executed"] == hp.expected_sym_blocks(w, tile=64, block=16)
        return
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, block=16)
    lens = np.random.default_rng(n).integers(0, n + 1, B).astype(np.int32)
    lens[0] = 63 if n > 63 else n
    _run_and_compare(w, scheme, 0.0, lens=lens)


# ---- float path, a vector that is not finite: rows that have no pair with it stay what they are -----------
NOT_FINITE_SHAPES = [
    # B, n, D, H, d, p
    (2, 100, 24, 2, 20, 25),      # keys shared by the wavefronts of a row tile
    (2, 48, 32, 3, 80, 12),       # a single key tile: a wavefront for every 16 rows
    (64, 66, 16, 8, 33, 33),      # the same, two key tiles, unaligned rows
]


def _run_with_a_bad_vector(w, scheme, bad_row, lens=None, flags=0):
    """The output with vector `bad_row` of every item infinite, and the checker's for the finite inputs."""
    stored, f64 = inputs.make_inputs(w)
    stored["X"][:, bad_row] = float("inf")
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=flags)
    try:
        got, _ = run.forward(scheme)
    finally:
        run.close()
    skip = bool(flags & ar.ATTN_FLAG_SKIP_PADDED_ROWS)
    return got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=skip)


@pytest.mark.parametrize("shape", NOT_FINITE_SHAPES)
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("noskip", [0, ar.ATTN_FLAG_NO_SKIP])
def test_left_out_rows_are_zeros_beside_infinite_keys(shape, scheme, dtype, noskip):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("left_out", B, n, D, H, d, p, dtype, scheme, 5200 + n)
    lens = np.full(B, 41, dtype=np.int32)     # rows 41 .. 47 share a 16-row group with rows that are there
    lens[-1] = 0
    got, _ = _run_with_a_bad_vector(w, scheme, 35, lens, ar.ATTN_FLAG_SKIP_PADDED_ROWS | noskip)
    for b, L in enumerate(lens):
        assert np.all(got[b, L:] == 0.0)
    assert not np.isfinite(got[:-1, 35:41]).any()   # rows that do attend the infinite key


@pytest.mark.parametrize("shape", NOT_FINITE_SHAPES + [
    (1, 100, 16, 1, 17, 100),     # one vector per partition, one column past a block
    (1, 90, 40, 2, 100, 90),      # the lane's columns in a group of 64 and one of 32 and 16
    (1, 64, 24, 2, 192, 64),      # the larger heads, both kernels
    (1, 70, 24, 1, 256, 70),
])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bad_row", [21, 32, 47])
def test_masked_infinite_vectors_reach_no_earlier_row(shape, dtype, bad_row):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("later_inf", B, n, D, H, d, p, dtype, CAUSAL, 5300 + n)
    outs = []
    for noskip in (0, ar.ATTN_FLAG_NO_SKIP):
        got, ref = _run_with_a_bad_vector(w, CAUSAL, bad_row, None, noskip)
        hp.tol_check(got[:, :bad_row], ref[:, :bad_row], dtype)
        assert not np.isfinite(got[:, bad_row:]).any()      # every later row has a pair with it
        outs.append(got)
    # the block that is cut by the diagonal with a value that is not finite, and yet allowed for some rows:
    # the same bits without skipping
    assert np.array_equal(outs[0], outs[1], equal_nan=True)


@pytest.mark.parametrize("shape", NOT_FINITE_SHAPES + [(1, 100, 16, 1, 17, 100)])
def test_an_infinite_value_of_one_column_stays_in_it(shape):
    """x with one component of its own, which only Wv takes, into column 0 of every head: v_j[0] infinite for one j,
    all else finite.  Rows from j on have that infinity in column 0, everything else is the checker's."""
    B, n, D, H, d, p = shape
    j = 21
    w = hp.custom_workload("one_inf", B, n, D, H, d, p, "f32", CAUSAL, 5400 + n)
    stored, f64 = inputs.make_inputs(w)
    for k in ("Wq", "Wk", "Wv"):
        stored[k][0] = 0.0
        stored[k][0, 0::d] = 1e30 if k == "Wv" else 0.0
        f64[k][0] = 0.0
    stored["X"][:, :, 0] = 0.0
    stored["X"][:, j, 0] = 1e30               # 1e30 * 1e30 is an infinity in float, 1e30 * 0 is 0
    stored["lens"] = None
    run = hp.GpuRun(w, stored)
    try:
        got, _ = run.forward(CAUSAL)
    finally:
        run.close()
    first = np.arange(H) * d
    assert np.all(got[:, j:, first] == np.inf)
    got[:, j:, first] = 0.0
    ref = hp.oracle_forward(w, f64, CAUSAL, 0.0)
    ref[:, j:, first] = 0.0
    hp.tol_check(got, ref, "f32")


# ---- float projection on products of bfloat16 planes: every kernel that a size selects, for what it stores (floats in
# 16-byte pieces, heads in no whole ones, planes), slices of d_model cut and whole, odd and even in number; then a value
# without planes in one of the rows.  The kernel is part of the table: a rule that moves a shape elsewhere fails here
FLOATS, ODD, PLANES = 0, 1, 2
PROJECTIONS = [
    # kernel, tile and k shared by the wavefronts; what it stores, even number of columns; B, n, D, H, d, p
    ("strands 2, 1, true", FLOATS, True, (1, 40, 100, 2, 20, 8)),
    ("strands 2, 1, true", ODD, True, (1, 40, 33, 2, 30, 8)),
    ("strands 2, 1, true", ODD, False, (3, 50, 295, 1, 31, 10)),
    ("strands 2, 1, true", ODD, False, (2, 30, 3, 3, 5, 10)),      # d_model below a piece
    ("strands 4, 2, true", FLOATS, True, (2, 300, 296, 8, 64, 50)),
    ("strands 4, 2, true", ODD, True, (2, 299, 288, 6, 85, 23)),
    ("strands 4, 2, true", ODD, False, (2, 300, 261, 7, 73, 50)),
    ("strands 2, 1, false", FLOATS, True, (5, 600, 31, 8, 64, 60)),
    ("strands 2, 1, false", FLOATS, True, (5, 600, 32, 8, 60, 60)),
    ("strands 2, 1, false", FLOATS, True, (8, 70, 63, 8, 60, 14)),
    ("strands 2, 1, false", FLOATS, True, (5, 600, 64, 8, 60, 60)),
    ("strands 2, 1, false", FLOATS, True, (8, 63, 64, 8, 60, 21)),
    ("strands 2, 1, false", ODD, True, (5, 600, 32, 6, 85, 60)),
    ("strands 2, 1, false", ODD, False, (5, 600, 50, 7, 73, 60)),
    ("strands 2, 1, false", PLANES, True, (16, 250, 32, 8, 64, 25)),
    ("strands 2, 1, false", PLANES, True, (16, 250, 23, 8, 40, 25)),
    ("split 1, 4", FLOATS, True, (8, 128, 72, 8, 64, 16)),
    ("split 1, 4", FLOATS, True, (10, 128, 39, 8, 64, 16)),       # one whole slice and a cut one
    ("split 1, 4", FLOATS, True, (8, 126, 192, 8, 60, 18)),
    ("split 1, 4", ODD, True, (8, 126, 96, 8, 62, 18)),
    ("split 1, 4", ODD, False, (8, 126, 193, 7, 73, 18)),
    ("split 1, 4", PLANES, True, (16, 250, 168, 8, 64, 25)),
    ("split 1, 4", PLANES, True, (16, 250, 40, 8, 64, 25)),
    ("strands 2, 1, false", PLANES, True, (8, 250, 60, 16, 48, 25)),
    ("split 2, 3", FLOATS, True, (16, 125, 164, 12, 64, 25)),
    ("split 2, 3", FLOATS, True, (10, 100, 40, 12, 64, 25)),
    ("split 2, 3", FLOATS, True, (10, 100, 64, 12, 64, 25)),
    ("split 2, 3", ODD, True, (16, 125, 190, 10, 75, 25)),
    ("split 2, 3", ODD, False, (16, 125, 170, 11, 67, 25)),
    ("split 2, 3", PLANES, True, (8, 250, 168, 16, 48, 25)),
    ("split 2, 3", PLANES, True, (16, 250, 60, 12, 64, 25)),
    ("split 2, 4", FLOATS, True, (4, 300, 192, 16, 64, 30)),
    ("split 2, 4", FLOATS, True, (16, 128, 104, 8, 64, 16)),
    ("split 2, 4", FLOATS, True, (16, 128, 96, 8, 64, 16)),
    ("split 2, 4", FLOATS, True, (32, 100, 33, 12, 64, 25)),
    ("split 2, 4", ODD, True, (4, 300, 200, 14, 73, 30)),
    ("split 2, 4", ODD, False, (4, 300, 161, 15, 67, 30)),
    ("split 2, 4", PLANES, True, (8, 250, 200, 16, 32, 25)),
    ("split 2, 4", PLANES, True, (10, 250, 56, 16, 32, 25)),
]


@pytest.mark.parametrize("kernel,stored_as,even,shape", PROJECTIONS)
def test_float_projection_tiles(kernel, stored_as, even, shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("proj_tiles", B, n, D, H, d, p, "f32", FULL, 7100 + n + D)
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored)
    try:
        names = run.kernels(FULL)
    finally:
        run.close()
    kind, tile = kernel.split(" ", 1)
    want = f"proj_split_{'strands_' if kind == 'strands' else ''}kernel<(attnring::Form){stored_as}, {str(even).lower()}, {tile}>"
    assert want in names[0] and len(names) == 2, names
    assert ("attn_planes_kernel" in names[1]) == (stored_as == PLANES), names
    _run_and_compare(w, FULL)
    if n > 21 and D > 3:
        test_an_infinite_value_of_one_column_stays_in_it(shape)


# ---- float attention on products of bfloat16 planes: head sizes that fill their 32-column steps and not, both tile
# shapes, last tiles whole and cut, then lengths, a negative scale, and vectors without planes
PLANE_SHAPES = [
    # B, n, D, H, d, p
    (4, 1024, 16, 8, 8, 32),
    (16, 256, 24, 8, 32, 64),
    (30, 186, 24, 6, 40, 31),
    (16, 250, 40, 8, 64, 25),
    (16, 244, 32, 8, 72, 61),
    (16, 256, 32, 8, 96, 32),
    (16, 250, 24, 8, 104, 25),    # 128 rows to a workgroup, 32 keys to a tile
    (16, 256, 32, 8, 128, 32),
]


@pytest.mark.parametrize("shape", PLANE_SHAPES)
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_float_attention_on_planes(shape, scheme):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("planes", B, n, D, H, d, p, "f32", scheme, 7300 + n + d)
    run = hp.GpuRun(w, inputs.make_inputs(w)[0])
    try:
        assert "attn_planes_kernel" in run.kernels(scheme)[1]
    finally:
        run.close()
    _, stats = _run_and_compare(w, scheme)
    assert (stats["phys_br"], stats["phys_bc"]) == (16, 16)
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, block=16)
    lens = np.asarray([(37 * b + 1) % (n + 1) for b in range(B)], dtype=np.int32)
    lens[:4] = 1, n, 65, 16
    _run_and_compare(w, scheme, lens=lens, scale=-0.3)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    outs = []
    for flags in (ar.ATTN_FLAG_SKIP_PADDED_ROWS, ar.ATTN_FLAG_SKIP_PADDED_ROWS | ar.ATTN_FLAG_NO_SKIP):
        run = hp.GpuRun(w, stored, flags=flags)
        try:
            outs.append(run.forward(scheme)[0])
        finally:
            run.close()
    ref = hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True)
    hp.tol_check(outs[0], ref, "f32")
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("shape", PLANE_SHAPES)
def test_float_attention_on_planes_beside_values_not_finite(shape):
    for bad_row in (21, 47, 100):
        test_masked_infinite_vectors_reach_no_earlier_row(shape, "f32", bad_row)
    for scheme in (FULL, CAUSAL):
        for noskip in (0, ar.ATTN_FLAG_NO_SKIP):
            test_left_out_rows_are_zeros_beside_infinite_keys(shape, scheme, "f32", noskip)
    test_an_infinite_value_of_one_column_stays_in_it(shape)


@pytest.mark.parametrize("shape", [PLANE_SHAPES[1], PLANE_SHAPES[6]])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("top,scale", [(2e8, 1.0), (2e9, 1.0), (2e9, -0.1), (2e10, 1.0), (1e12, 0.3), (1e30, 1.0), (3e38, 1.0), (3e38, 1e6)])
def test_float_attention_on_planes_of_large_scores(shape, scheme, top, scale):
    """score_ij = +-top x_i x_j, x growing from 1/n to 1: finite, and so far apart that a row's output is the value
    vector of its largest score."""
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("large_scores", B, n, D, H, d, p, "f32", scheme, 7350 + n)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = None
    for k, size in (("Wq", 2.0), ("Wk", top / 2.0 / abs(scale))):
        stored[k].zero_()
        stored[k][0, 0::d] = size
    stored["Wv"][0] = 0.0
    stored["X"][:, :, 0] = torch.arange(1, n + 1) / n
    for k in stored:
        f64[k] = None if stored[k] is None else stored[k].double().numpy()
    run = hp.GpuRun(w, stored, scale=scale)
    try:
        got, _ = run.forward(scheme)
    finally:
        run.close()
    hp.tol_check(got, hp.oracle_forward(w, f64, scheme, scale), "f32")


@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_float_attention_on_planes_of_products_that_cancel(scheme, sign):
    """Every third key has products of -3 * 2^95 in the first columns and 3 * 2^95 in later ones: its score is zero, which
    a sum of planes, 2^32 times as large, leaves float's range before it gets to."""
    B, n, D, H, d, p = 16, 250, 40, 8, 128, 25
    w = hp.custom_workload("cancel", B, n, D, H, d, p, "f32", scheme, 7370)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = None
    X, Wq, Wk, Wv = (stored[k] for k in ("X", "Wq", "Wk", "Wv"))
    X[:, :, 0], X[:, :, 1] = 1.0, 0.0
    X[:, 1::3, 1], X[:, 1::3, 2] = 1.0, 0.0
    Wq.zero_()
    Wk.zero_()
    Wv[:2] = 0.0
    for col, size in ((0, -1.5), (1, -1.5), (32, 1.0), (64, 1.0), (96, 1.0)):
        Wq[0, col::d] = 2.0 ** 48
        Wk[1, col::d] = sign * size * 2.0 ** 47
    Wq[0, 2::d] = 1.0
    Wk[2, 2::d] = 1.0
    for k in stored:
        f64[k] = None if stored[k] is None else stored[k].double().numpy()
    run = hp.GpuRun(w, stored, scale=1.0)
    try:
        assert "attn_planes_kernel" in run.kernels(scheme)[1]
        got, _ = run.forward(scheme)
    finally:
        run.close()
    hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 1.0), "f32")


# ---- float storage near the ends of float's range: X, Wq, Wk, Wv times powers of two.  Below 2^-109 a bfloat16 no longer
# holds the last bits of a float, from 2^111 on its planes no longer hold the value
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (2, 24, 36, 3, 20, 8),        # one kernel
    (2, 500, 296, 8, 64, 50),     # projection into floats
    (32, 100, 24, 7, 73, 25),
    (16, 250, 40, 8, 64, 25),     # and into planes
    (16, 250, 136, 8, 128, 25),
])
@pytest.mark.parametrize("powers", [
    (-122, 100, 100, 100),        # x
    (0, -122, 100, 0),            # q
    (0, 100, -122, 0),            # k
    (0, 0, 0, -122),              # v and the output
    (100, -100, -100, -100),
    (125, -125, -125, -125),      # no planes of x
    (0, 124, -124, 0),            # of q
    (0, -124, 124, 0),            # of k
    (0, 0, 0, 113),               # of v; sums of 500 of them before they are divided
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_float_values_near_the_ends_of_the_range(shape, powers, scheme):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("range_ends", B, n, D, H, d, p, "f32", scheme, 7800 + n + D)
    stored, f64 = inputs.make_inputs(w)
    for k, e in zip(("X", "Wq", "Wk", "Wv"), powers):
        stored[k] *= 2.0 ** e
        f64[k] = stored[k].double().numpy()
        assert np.isfinite(f64[k]).all()
    stored["lens"] = None
    scale = 2.0 ** -(2 * powers[0] + powers[1] + powers[2]) / np.sqrt(d)
    if powers[0] == -122:
        scale = 1.0               # a score is 2^-44: no larger scale than float has is needed
    run = hp.GpuRun(w, stored, scale=scale)
    try:
        got, _ = run.forward(scheme)
    finally:
        run.close()
    hp.tol_check(got, hp.oracle_forward(w, f64, scheme, scale), "f32")


# ---- float storage, key lengths: what the padding holds changes neither the other rows nor the time
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (32, 32, 128, 8, 32, 8),      # one kernel
    (8, 200, 200, 7, 73, 25),     # projection into floats
    (8, 512, 264, 12, 64, 64),    # and into planes
    (8, 500, 264, 8, 128, 50),
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("flags", [0, ar.ATTN_FLAG_SKIP_PADDED_ROWS])
def test_float_padding_of_any_value(shape, scheme, flags):
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("padding", B, n, D, H, d, p, "f32", scheme, 7900 + n + D)
    stored, f64 = inputs.make_inputs(w)
    lens = np.asarray([n // 2 + 5 * b % (n // 2) for b in range(B)], dtype=np.int32)
    lens[0] = n
    stored["lens"] = lens
    ref = hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=flags != 0)
    run = hp.GpuRun(w, stored, flags=flags)
    clean = run.X.clone()
    first, times = None, {}
    try:
        for fill in (0.0, float("nan"), float("inf"), -3e38):
            run.X.copy_(clean)
            for b, L in enumerate(lens):
                run.X[b, int(L):] = fill
            got, _ = run.forward(scheme)
            for b, L in enumerate(lens):
                if flags:
                    assert np.all(got[b, L:] == 0.0)
                hp.tol_check(got[b, :L], ref[b, :L], "f32")
            kept = [got[b, :L] for b, L in enumerate(lens)]
            first = first or kept
            # query rows of padding that are produced and not all NaN take their tile to float arithmetic: same values,
            # other roundings, other times
            alike = flags != 0 or fill == 0.0 or fill != fill
            if alike:
                assert all(np.array_equal(x, y) for x, y in zip(first, kept))
            best = float("inf")
            for _ in range(5):
                ar.attn_profile(run.ctx, True)
                for _ in range(10):
                    ar.attn_forward(run.ctx, run.X, *run.W, scheme, run.out)
                t = ar.attn_profile_read(run.ctx)
                ar.attn_profile(run.ctx, False)
                best = min(best, t["ms_projection"] + t["ms_attention"])
            times[fill] = best
            print(f"[padding] of {fill}: {best:.4f} ms", flush=True)
            if alike:
                assert best < 2.0 * times[0.0]      # 1.0 to 1.25 measured
        torch.cuda.synchronize()
    finally:
        run.close()


@pytest.mark.parametrize("shape", [(64, 256, 32, 8, 64, 32), (16, 500, 64, 8, 72, 25)])
def test_planes_and_symmetric_calls_in_turn(shape):
    """One context whose q, k, v are planes: FULL and CAUSAL calls around q = k = v ones, which take z as floats, give the
    same bits before and after, and all that the first of those allocates is z and the score matrices."""
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("in_turn", B, n, D, H, d, p, "f32", FULL, 8100 + n)
    stored, f64 = inputs.make_inputs(w)
    warm = hp.GpuRun(w, stored)     # what the runtime allocates with a kernel's first launch
    run = hp.GpuRun(w, stored)
    try:
        for scheme in (FULL, CAUSAL, SYM):
            warm.forward(scheme)
        seen = {}
        for scheme in (FULL, CAUSAL, SYM, CAUSAL, FULL, SYM):
            torch.cuda.synchronize()
            before = torch.cuda.mem_get_info()[0]
            got, _ = run.forward(scheme)
            taken = before - torch.cuda.mem_get_info()[0]
            first = scheme == SYM and scheme not in seen
            assert taken <= (4 * (B * n * H * d + B * H * n * (n + 3)) if first else 0) + (8 << 20)   # rounded up to pages
            if scheme in seen:
                assert np.array_equal(got, seen[scheme])
            seen[scheme] = got
            hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0), "f32")
    finally:
        run.close()
        warm.close()


# ---- small float calls in one kernel: every number of row and column blocks, slices of d_model whole and cut
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (3, 1, 4, 2, 4, 1),
    (1, 16, 64, 1, 64, 4),
    (2, 24, 36, 3, 20, 8),
    (5, 32, 64, 7, 48, 8),
    (32, 30, 188, 4, 64, 10),
    (64, 16, 252, 8, 64, 4),      # the longest d_model
    (128, 33, 100, 1, 36, 11),
    (16, 64, 128, 8, 64, 16),
    (33, 50, 8, 31, 16, 25),      # nearly a counter slot for every workgroup
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_small_float_calls_in_one_kernel(shape, scheme):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("one_kernel", B, n, D, H, d, p, "f32", scheme, 7500 + n + D)
    run = hp.GpuRun(w, inputs.make_inputs(w)[0])
    try:
        names = run.kernels(scheme)
        assert len(names) == 1 and "proj_attn_small_kernel" in names[0], names
    finally:
        run.close()
    _, stats = _run_and_compare(w, scheme)
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, block=16)
    lens = np.asarray([(5 * b) % (n + 1) for b in range(B)], dtype=np.int32)
    _run_and_compare(w, scheme, lens=lens, scale=0.4)
    if n > 21:
        test_an_infinite_value_of_one_column_stays_in_it(shape)
        test_masked_infinite_vectors_reach_no_earlier_row(shape, "f32", 21)
    if n > 41:
        test_left_out_rows_are_zeros_beside_infinite_keys(shape, scheme, "f32", 0)


@pytest.mark.parametrize("over", ["X", "X shifted", "Wv"])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_small_float_call_over_its_own_inputs(over, scheme):
    """`out` in the memory of X or of a weight matrix: every input is read before it is written over."""
    import torch
    B, n, D, H, d, p = 64, 16, 128, 8, 16, 8
    if over == "Wv":
        B, n = 16, 8              # as many floats as d_model * n_heads * d_k
    w = hp.custom_workload("in_place", B, n, D, H, d, p, "f32", scheme, 7700 + n)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = None
    run = hp.GpuRun(w, stored)
    try:
        if over == "X":
            run.out = run.X
        elif over == "X shifted":
            room = torch.empty(run.X.numel() + 40 * D, dtype=run.X.dtype, device=run.X.device)
            run.X = room[:run.X.numel()].view(run.X.shape).copy_(run.X)
            run.out = room[40 * D:].view(run.X.shape)
        else:
            run.out = run.W[2].view(B, n, D)
        got, _ = run.forward(scheme)
    finally:
        run.close()
    hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0), "f32")


# ---- float path, steady states: many slices of d_model, many key tiles ----------------------------------------
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (8, 256, 200, 8, 80, 32),     # 64 x 64 GEMM tiles, seven slices of which the last is cut; walk: keys shared
    (16, 200, 261, 8, 64, 25),    # the same on unaligned rows of x; 512 row tiles: K and V through LDS, four key tiles
    (2, 200, 450, 2, 48, 25),     # 32 x 32 GEMM tiles that share k, eight slices (four in 16 bits)
    (2, 200, 453, 2, 47, 25),     # the same, unaligned
    (2, 200, 456, 4, 48, 25),     # 16 bits: pieces straight into LDS, eight slices, the last cut
    (16, 200, 72, 8, 80, 25),     # K and V through LDS at the other head sizes
    (16, 200, 24, 8, 96, 25),
    (16, 200, 24, 8, 128, 25),
    (16, 200, 24, 8, 90, 25),
    (3, 64, 40, 2, 160, 8),       # a single key tile of the large heads
    (3, 60, 40, 2, 192, 6),
    (3, 33, 40, 2, 256, 11),
    (3, 61, 40, 1, 250, 61),
    (2, 300, 40, 2, 192, 30),     # their keys shared
    (2, 300, 40, 2, 250, 30),
    (16, 200, 24, 8, 160, 25),    # and through LDS
])
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_float_path_steady_states(shape, scheme, dtype):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("float_steady", B, n, D, H, d, p, dtype, scheme, 6500 + n + d)
    _run_and_compare(w, scheme, 0.0)
    if scheme != SYM:
        lens = np.random.default_rng(d).integers(0, n + 1, B).astype(np.int32)
        lens[-1] = n - 1
        _run_and_compare(w, scheme, 0.0, lens=lens)


# ---- matrix-core projection, steady states and row subsets, by the GEMM that the size selects ---------------
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (1, 200, 768, 2, 64, 25),     # 64 x 64 tiles, twelve slices: the ring turns four times
    (2, 200, 776, 3, 64, 25),     # the same with a cut slice and an odd number of heads
    (6, 400, 456, 5, 64, 50),     # 630 of them: the shorter ring, eight slices
    (6, 384, 136, 6, 64, 48),     # 128 x 128 tiles, two workgroups per CU, cut slice
    (6, 400, 448, 6, 64, 50),     # the same, seven slices, ragged rows
    (30, 200, 136, 6, 64, 25),    # 540 of them: three workgroups per CU (two with key lengths)
    (30, 200, 448, 6, 64, 25),
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_projection_steady_states_and_lengths(shape, scheme):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("proj_steady", B, n, D, H, d, p, "bf16", scheme, 7300 + D)
    _run_and_compare(w, scheme, 0.0)
    lens = np.random.default_rng(D).integers(0, n + 1, B).astype(np.int32)
    lens[0] = n // 2 + 1
    _run_and_compare(w, scheme, 0.0, lens=lens)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS)
    try:
        padded, _ = run.forward(scheme)
        packed, _ = run.forward_packed(scheme, lens)
    finally:
        run.close()
    hp.tol_check(padded, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True), w.dtype)
    assert np.array_equal(padded, packed)


# ---- weights that are not 16-byte aligned: laid out anew and read by the GEMM for transposed weights ----------
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (2, 320, 136, 2, 64, 40),     # 128 x 128 tiles, cut slice
    (2, 200, 192, 3, 64, 25),     # 64 x 64 tiles (an odd number of 64-wide heads)
    (1, 600, 64, 1, 128, 75),     # one slice, d_k = 128
])
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
def test_unaligned_weights(shape, scheme):
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("unaligned", B, n, D, H, d, p, "bf16", scheme, 7900 + n)
    stored, f64 = inputs.make_inputs(w)
    lens = None
    if scheme == SYM:
        stored["Wk"] = stored["Wv"] = None
    else:
        lens = np.random.default_rng(n).integers(1, n + 1, B).astype(np.int32)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS)
    try:
        for m in range(3):
            if run.W[m] is not None:
                room = torch.empty(run.W[m].numel() + 1, dtype=run.W[m].dtype, device=run.X.device)
                run.W[m] = room[1:].view(run.W[m].shape).copy_(run.W[m])
        got, stats = run.forward(scheme)
        hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=lens is not None))
        packed = run.forward_packed(scheme, lens)[0] if lens is not None else got
    finally:
        run.close()
    ref = hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=lens is not None)
    hp.tol_check(got, ref, w.dtype)
    assert np.array_equal(got, packed)


def test_symmetric_without_projection():
    w = hp.custom_workload("symx", 2, 20, 24, 2, 12, 5, "f32", SYM, 77)
    _, stats = _run_and_compare(w, SYM, 0.2, sym_no_proj=True)
    assert stats["proj_gemms"] == 0


@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (3, 1000, 40, 12, 96, 125),   # K and V through LDS; own tile first in the walk: 8.4e-7
    (2, 900, 64, 24, 64, 90),
])
def test_symmetric_float_sums_keep_their_precision(shape):
    """q = k = v: a row's own weight outweighs the others together, and what is added to a float sum behind it is
    rounded at that size.  2-norm of the error over 2-norm of the output; 2.5e-7 to 3.1e-7 measured, of which the
    scores' own rounding (size |z|^2 / sqrt(d), some 10) is most."""
    B, n, D, H, d, p = shape
    w = hp.custom_workload("sym_precision", B, n, D, H, d, p, "f32", SYM, 2600 + n)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = stored["Wk"] = stored["Wv"] = None
    run = hp.GpuRun(w, stored)
    try:
        got, _ = run.forward(SYM)
    finally:
        run.close()
    ref = hp.oracle_forward(w, f64, SYM, 0.0)
    assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)


# ---- q = k = v on the float path, n no multiple of 4, close to the bound on the score matrices: rows in whole
# 16-byte pieces would take more than the 1 GiB
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (12000, 13, 16, 128, 1, 13),  # a single key tile
    (27391, 70, 8, 2, 4, 10),     # two tiles
    (1, 9459, 16, 3, 16, 3),      # keys shared by the wavefronts
])
def test_symmetric_score_matrices_stay_within_their_bound(shape):
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("score_bound", B, n, D, H, d, p, "f32", SYM, 2700 + n)
    assert B * H * n * n * 4 <= 1 << 30 < B * H * n * ((n + 3) & ~3) * 4
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = stored["Wk"] = stored["Wv"] = None
    _run_and_compare(hp.custom_workload("loaded", 1, n, 16, 2, 16, 1, "f32", SYM, 5), SYM)   # the kernels are on the device
    run = hp.GpuRun(w, stored)
    try:
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        got, stats = run.forward(SYM)
        taken = before - torch.cuda.mem_get_info()[0]
    finally:
        run.close()
    assert taken <= (1 << 30) + (4 << 20)      # the device gives memory in pieces of 2 MiB
    hp.check_counts(stats, hp.oracle_counts(w, SYM))
    rows = sorted({r for r in (0, 1, n // 2, 63, 64, n - 65, n - 2, n - 1) if 0 <= r < n})
    for (b, h) in {(0, 0), (B // 2, H // 2), (B - 1, H - 1)}:
        ref = orc.head_rows(f64["X"], f64["Wq"], f64["Wk"], f64["Wv"], n_heads=H, d_k=d, p=p, scheme=SYM,
                            scale=hp.default_scale(w, 0.0), b=b, h=h, rows=rows)
        hp.tol_check(got[b, rows, h * d:(h + 1) * d], ref, "f32")


# ---- bf16 MFMA path on small shapes: several tiles and a ragged tail -----------------------------
@pytest.mark.parametrize("shape", [
    (2, 320, 64, 2, 64, 40),      # 2.5 row tiles
    (1, 200, 96, 3, 64, 25),      # n not a multiple of 8
    (2, 384, 128, 2, 128, 12),    # d_k = 128, partitions of 32 rows
    (1, 136, 72, 1, 128, 17),     # d_model not a multiple of 64 (k tail)
    (1, 520, 64, 2, 64, 5),       # partitions larger than a score block (104 rows)
    (1, 1096, 64, 1, 128, 137),   # several 256-row tiles and a ragged tail
    (1, 264, 192, 2, 64, 33),     # three 64-deep slices of d_model: the slice ring starts and ends at once
    (2, 256, 320, 2, 128, 32),    # five slices: one steady turn of the slice ring, then its tail
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("tiles", [ar.ATTN_FLAG_NARROW_TILES, ar.ATTN_FLAG_WIDE_TILES])
@pytest.mark.parametrize("seed0", [999, 1000])
def test_mfma_path_small(shape, scheme, tiles, seed0):
    # seed0 = 999 holds the draw (n = 320, unmasked, key lengths) on which q, k, v kept in bfloat16
    # between the kernels put one output of size 2.03 at 2.19e-2: 7.5e-3 from rounding k, 5.7e-3
    # from v, 1.5e-3 from q, 7e-3 from rounding the output itself.  They are kept in half precision
    # since, which leaves the output rounding and about 2e-3.
    B, n, D, H, d, p = shape
    w = hp.custom_workload("mfma_small", B, n, D, H, d, p, "bf16", scheme, seed0 + n)
    _, stats = _run_and_compare(w, scheme, 0.0, flags=tiles)
    assert (stats["phys_br"], stats["phys_bc"]) == (32, 32)
    lens = np.random.default_rng(n + 1).integers(1, n + 1, B).astype(np.int32)
    lens[-1] = n // 2 + 3
    _run_and_compare(w, scheme, 0.0, lens=lens, flags=tiles)
    _run_and_compare(w, scheme, 0.0, lens=np.zeros(B, dtype=np.int32), flags=tiles)


# ---- small launches: 32 rows per workgroup, its wavefronts share the keys (no tile flag) -------------------
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (1, 1, 64, 2, 64, 1),         # a single row and key
    (1, 33, 64, 2, 64, 11),       # one row and one key past a block: three wavefronts without a block
    (3, 96, 72, 2, 64, 12),       # whole blocks
    (2, 200, 128, 3, 64, 25),     # more blocks than wavefronts, ragged
    (2, 129, 64, 2, 128, 43),     # d_k = 128, one row in the last block
    (1, 520, 64, 1, 128, 5),      # partitions larger than a row tile
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_small_launches_share_the_keys(shape, scheme):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("split", B, n, D, H, d, p, "bf16", scheme, 8800 + n)
    _run_and_compare(w, scheme, 0.0)
    lens = np.random.default_rng(n + 3).integers(0, n + 1, B).astype(np.int32)
    lens[-1] = n // 2 + 1
    _run_and_compare(w, scheme, 0.0, lens=lens)
    # padded rows left out: against the checker, and the same bits without skipping and in the packed layout
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    outs = []
    for noskip in (0, ar.ATTN_FLAG_NO_SKIP):
        run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS | noskip)
        try:
            got, stats = run.forward(scheme)
            hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=True), noskip=bool(noskip))
            outs.append(got)
            if not noskip:
                assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, lens, skip_padded_rows=True)
                outs.append(run.forward_packed(scheme, lens)[0])
        finally:
            run.close()
    hp.tol_check(outs[0], hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True), w.dtype)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


# ---- launches that leave the chip idle otherwise: strands of wavefronts share the keys (no tile flag) ------
@pytest.mark.parametrize("strands,shape", [
    # B, n, D, H, d, p
    (4, (1, 1030, 64, 3, 64, 103)),    # five tiles for the first strand, four for the others; six rows in the last
    (4, (9, 140, 64, 9, 64, 35)),      # three tiles: a strand has none
    (3, (2, 516, 64, 19, 64, 129)),    # nine tiles; partitions larger than a row tile
    (2, (1, 1100, 64, 8, 128, 275)),   # d_k = 128
    (2, (3, 150, 64, 20, 128, 30)),    # three tiles, two strands
    (2, (3, 1030, 64, 11, 128, 103)),  # masked: 297 row tiles, a second round; heads that do not divide by eight
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_strands_share_the_keys(strands, shape, scheme):
    B, n, D, H, d, p = shape
    if scheme == FULL and B * H * ((n + 127) // 128) > 256:
        H = 8
    w = hp.custom_workload("strands", B, n, D, H, d, p, "bf16", scheme, 8900 + n)
    _run_and_compare(w, scheme, 0.0)
    lens = np.random.default_rng(n + 3).integers(0, n + 1, B).astype(np.int32)
    lens[-1] = n // 2 + 1
    _run_and_compare(w, scheme, 0.0, lens=lens)
    # padded rows left out: against the checker, and the same bits without skipping and in the packed layout
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    outs = []
    for noskip in (0, ar.ATTN_FLAG_NO_SKIP):
        run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS | noskip)
        try:
            got, stats = run.forward(scheme)
            hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=True), noskip=bool(noskip))
            outs.append(got)
            if not noskip:
                assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, lens, skip_padded_rows=True)
                outs.append(run.forward_packed(scheme, lens)[0])
                assert any(f"attn_strands_kernel<{d}, {strands}," in k for k in run.kernels(scheme))
        finally:
            run.close()
    hp.tol_check(outs[0], hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True), w.dtype)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


# ---- masked scheme, one row tile per workgroup with the heads in turn ------------------------------------
@pytest.mark.parametrize("shape", [
    (3, 700, 64, 13, 64, 100),    # d_k = 64, heads that do not divide by eight
    (5, 500, 64, 70, 64, 125),    # 700 pairs nearly fill a round: paired
    (9, 500, 64, 45, 64, 125),    # 810 pairs: a second round nearly empty
    (3, 1100, 64, 5, 128, 275),   # d_k = 128
    (3, 500, 64, 100, 128, 125),  # d_k = 128, 300 pairs: two rounds of the chip, half empty
    (3, 700, 64, 70, 128, 100),   # 420 pairs of three row tiles per head
    (3, 1000, 64, 40, 128, 125),  # 240 pairs fill one round: paired
])
def test_row_tiles_with_the_heads_in_turn(shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("in_turn", B, n, D, H, d, p, "bf16", CAUSAL, 9100 + n)
    _run_and_compare(w, CAUSAL, 0.0)
    _run_and_compare(w, CAUSAL, 0.0, lens=np.resize(np.array([n, 1, n // 3], dtype=np.int32), B))


# ---- the projection's last slice of d_model when it is not 64 deep (vectors in whole 16-byte pieces) ----
@pytest.mark.parametrize("d_model", [8, 56, 72, 136, 200])   # one slice, cut; then two to four with 8 .. 8 left
@pytest.mark.parametrize("shape", [
    # B, n, H, d, p
    (2, 200, 2, 64, 25),          # 64 x 64 tiles
    (2, 200, 3, 64, 25),          # the same with an odd number of 64-wide heads
    (8, 256, 6, 64, 32),          # 128 x 128 tiles, two workgroups per CU
    (30, 256, 6, 64, 32),         # 540 of them: three workgroups per CU
    (8, 2048, 16, 128, 256),      # 128 x 256 tiles
    (1, 4096, 32, 128, 512),      # with 2048 added to d_model: 256 x 256 tiles
])
def test_projection_with_a_cut_slice(shape, d_model):
    B, n, H, d, p = shape
    if B == 1:
        d_model += 2048
    w = hp.custom_workload("cut_slice", B, n, d_model, H, d, p, "bf16", CAUSAL, 7700 + d_model)
    if n <= 256:
        _run_and_compare(w, CAUSAL, 0.0)
    # values that follow a vector's end belong to the next one and must not reach it: a vector of infinities, and
    # the rows up to the one directly before it
    stored, f64 = inputs.make_inputs(w)
    firsts = {b: 96 if b % 2 else n - 32 for b in range(B)}
    for b, i in firsts.items():
        stored["X"][b, i] = float("inf")
    stored["lens"] = None
    run = hp.GpuRun(w, stored)
    try:
        got, _ = run.forward(CAUSAL)
    finally:
        run.close()
    for (b, h) in {(0, 0), (min(1, B - 1), min(5, H - 1)), (min(3, B - 1), H - 1), (B - 1, H // 2)}:
        rows = [r for r in range(firsts[b]) if r < 140 or r > n - 70]
        ref = orc.head_rows(f64["X"], f64["Wq"], f64["Wk"], f64["Wv"], n_heads=H, d_k=d, p=p, scheme=CAUSAL,
                            scale=hp.default_scale(w, 0.0), b=b, h=h, rows=rows)
        hp.tol_check(got[b, rows, h * d:(h + 1) * d], ref, w.dtype)


# ---- products of one round of large tiles, and of large tiles that fill their rounds badly ------------------------
@pytest.mark.parametrize("tile,shape", [
    # B, n, D, H, d, p
    ("128, 256", (11, 500, 64, 12, 64, 125)),     # 792 tiles of 128 x 128, ragged
    ("128, 256", (18, 250, 72, 8, 128, 125)),     # d_k = 128; a cut slice
    ("256, 256", (6, 1020, 2056, 12, 64, 255)),    # d_model from 2048 on, 216 of 256 x 256
    ("128, 256", (24, 500, 2048, 16, 64, 125)),   # 576 of 256 x 256 in three rounds
    ("128, 128", (8, 512, 64, 24, 64, 64)),       # 1152 of 128 x 128: as before
])
def test_projection_rounds_of_large_tiles(tile, shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("rounds", B, n, D, H, d, p, "bf16", CAUSAL, 7750 + n)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = None
    run = hp.GpuRun(w, stored)
    try:
        assert any(f"proj_dma_kernel<{tile}," in k for k in run.kernels(CAUSAL))
        got, _ = run.forward(CAUSAL)
    finally:
        run.close()
    rows = sorted({0, 1, 127, 128, n // 2, n - 2, n - 1})
    for (b, h) in {(0, 0), (B // 2, H // 2), (B - 1, H - 1)}:
        ref = orc.head_rows(f64["X"], f64["Wq"], f64["Wk"], f64["Wv"], n_heads=H, d_k=d, p=p, scheme=CAUSAL,
                            scale=hp.default_scale(w, 0.0), b=b, h=h, rows=rows)
        hp.tol_check(got[b, rows, h * d:(h + 1) * d], ref, w.dtype)


# ---- 64 x 64 tiles that are more than the CUs: groups of three column tiles --------------------------------------
@pytest.mark.parametrize("scheme,lens,shape", [
    # B, n, D, H, d, p
    (CAUSAL, False, (2, 150, 1288, 16, 64, 25)),   # 288 tiles, 24 in the last row tile; a cut slice
    (FULL, True, (3, 150, 1344, 12, 64, 25)),      # 324, with key lengths (dealt over the matrices)
    (FULL, False, (1, 340, 64, 14, 128, 85)),      # 504
    (SYM, False, (1, 900, 64, 10, 64, 225)),       # 300; 20 column tiles, two in the last group
    (FULL, False, (1, 600, 640, 8, 80, 75)),       # 300, left as floats
])
def test_projection_of_small_tiles_that_share_cus(scheme, lens, shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("shared", B, n, D, H, d, p, "bf16", scheme, 7790 + n)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = np.resize(np.array([n, 70, 1], dtype=np.int32), B) if lens else None
    if scheme == SYM:
        f64["Wk"] = f64["Wv"] = f64["Wq"]
    run = hp.GpuRun(w, stored)
    try:
        assert any("proj_small_kernel<5," in k for k in run.kernels(scheme))
        got, _ = run.forward(scheme)
    finally:
        run.close()
    hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=stored["lens"]), w.dtype)


# ---- queries projected inside the attention kernel (ATTN_FLAG_FUSE_Q_PROJECTION) ----------------------
@pytest.mark.parametrize("shape", [
    (2, 320, 64, 2, 64, 40),      # two 32-row slices of Wq
    (2, 384, 128, 2, 128, 12),    # d_k = 128
    (1, 1096, 64, 1, 128, 137),   # several 256-row tiles and a ragged tail
    (1, 264, 192, 2, 64, 33),     # six slices
    (2, 256, 320, 2, 128, 32),    # ten slices
    (1, 200, 96, 3, 64, 25),      # d_model not a multiple of 64: the flag has no effect
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("tiles", [ar.ATTN_FLAG_NARROW_TILES, ar.ATTN_FLAG_WIDE_TILES])
def test_queries_projected_in_the_attention_kernel(shape, scheme, tiles):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("fuse_q", B, n, D, H, d, p, "bf16", scheme, 3100 + n)
    flags = tiles | ar.ATTN_FLAG_FUSE_Q_PROJECTION
    _run_and_compare(w, scheme, 0.0, flags=flags)
    lens = np.random.default_rng(n + 2).integers(1, n + 1, B).astype(np.int32)
    lens[-1] = n // 2 + 3
    _run_and_compare(w, scheme, 0.0, lens=lens, flags=flags)
    _run_and_compare(w, scheme, 0.0, lens=np.zeros(B, dtype=np.int32), flags=flags)


def test_causal_workload_with_queries_projected_in_the_attention_kernel():
    w = inputs.WORKLOADS["causal"]
    err, stats = _run_and_compare(w, w.scheme, 0.0, flags=ar.ATTN_FLAG_FUSE_Q_PROJECTION)
    assert stats["tiles_executed"] == 96 * 8256


# ---- q = k = v scheme on the matrix cores: each score tile computed once, used for both row blocks ----
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (2, 1100, 64, 2, 64, 275),     # 9 tiles, the last one ragged; odd number of ring partitions
    (1, 1024, 128, 2, 128, 128),   # whole tiles, even partitions (middle diagonal scheduled twice)
    (3, 200, 64, 2, 64, 25),       # two tiles, second nearly empty
    (1, 96, 64, 2, 128, 12),       # a single tile: nothing to reuse
])
def test_symmetric_on_matrix_cores(shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload("sym_mfma", B, n, D, H, d, p, "bf16", SYM, 2300 + n)
    err, stats = _run_and_compare(w, SYM, 0.0)
    assert (stats["phys_br"], stats["phys_bc"]) == (32, 32) and stats["proj_gemms"] == 2
    assert stats["phys_tiles_executed"] == hp.expected_sym_blocks(w)
    half = p * (p + 1) // 2 if p % 2 else p * (p + 2) // 2      # Sec. 4.2, on the tile matrix
    assert stats["tiles_executed"] == B * H * half
    _run_and_compare(w, SYM, 1.0 / 32)


def _sym_both_ways(w, stored, scale):
    """q = k = v with reuse and with every tile computed in its own orientation: the same bits."""
    outs = []
    for flags in (0, ar.ATTN_FLAG_NO_SKIP):
        run = hp.GpuRun(w, stored, scale=scale, flags=flags)
        try:
            got, stats = run.forward(SYM)
        finally:
            run.close()
        hp.check_counts(stats, hp.oracle_counts(w, SYM), noskip=bool(flags))
        if not flags:
            assert stats["phys_tiles_executed"] == hp.expected_sym_blocks(w)
        outs.append(got)
    assert np.array_equal(outs[0], outs[1])
    return outs[0]


# ---- the same: a row tile's partners in runs of several lengths, and references that its own score does not give
@pytest.mark.parametrize("shape", [
    # B, n, D, H, d, p
    (2, 90, 64, 2, 64, 10),       # one tile: no states to merge
    (1, 600, 64, 3, 64, 75),      # five tiles, runs of one partner
    (8, 500, 64, 16, 64, 125),    # four tiles, one run of three or two partners; ragged
    (8, 300, 64, 16, 128, 75),    # three tiles of d_k = 128, one run of two partners
    (1, 1500, 64, 8, 128, 150),   # twelve tiles, runs of three
])
@pytest.mark.parametrize("rows", ["normal", "other rows heavier", "huge", "huger", "hugest"])
def test_symmetric_references(shape, rows):
    """`other rows heavier`: all vectors point one way, with lengths 0.3 to 1.6, so that short rows have scores up to 15
    nats (d_k = 64; 22 at 128) above their own, across tiles, where 11 raise the reference.  z is rounded to half precision, 2^-12
    of a score of up to 90 spread over d products: 3e-3 of a weight, on top of the output's own rounding (below 8).  `huge`: scores of 1e8, where the sum of squares and the
    product differ by more than half precision holds; every row attends to itself.  `huger`, `hugest`: of 1e9 and 1e10, where
    they would differ by more than a float's exponent holds, and so would a score and its reference, rounded apart."""
    import torch
    B, n, D, H, d, p = shape
    w = hp.custom_workload("sym_refs", B, n, D, H, d, p, "bf16", SYM, 2900 + n)
    scale = {"other rows heavier": 3.0 / math.sqrt(d), "hugest": 1.0}.get(rows, 0.0)
    length = {"huge": 3000.0, "huger": 10000.0, "hugest": 10000.0}.get(rows)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = stored["Wk"] = stored["Wv"] = None
    if rows != "normal":
        X = stored["X"].float()
        if length:
            X = length * X
        else:
            g = np.random.default_rng(n)
            way = X[:, :1] * (8.0 / X[:, :1].norm(dim=-1, keepdim=True))
            X = way * torch.from_numpy(g.uniform(0.3, 1.6, (B, n, 1))).float() + 0.02 * X
        stored["X"] = X.to(torch.bfloat16)
        f64["X"] = stored["X"].double().numpy()
    got = _sym_both_ways(w, stored, scale)
    if B * H > 32:  # a few heads
        heads = [(0, 0), (B // 2, H - 1), (B - 1, H // 2)]
        ref = np.stack([orc.head_rows(f64["X"], f64["Wq"], f64["Wq"], f64["Wq"], n_heads=H, d_k=d, p=p, scheme=SYM,
                                      scale=hp.default_scale(w, scale), b=b, h=h, rows=range(n)) for b, h in heads])
        got = np.stack([got[b, :, h * d:(h + 1) * d] for b, h in heads])
    else:
        ref = hp.oracle_forward(w, f64, SYM, scale)
    if length:
        # half an ulp of the output, at most 2^-8 of it, and of z in half precision, 2^-11; where z's 64 products of some 300
        # (a tenth of the length) cancel, the roundings of their sums: 2^-24 of 2e4 each
        assert np.all(np.abs(got - ref) <= (2.0 ** -8 + 2.0 ** -11) * np.abs(ref) + 2e-2 * (length / 3000.0))
    else:
        hp.tol_check(got, ref, w.dtype)


@pytest.mark.parametrize("n,d", [(90, 64), (256, 64), (250, 128), (1500, 64)])   # one tile; two, both uses; runs of several
def test_symmetric_small_weights_keep_their_bits(n, d):
    """z = X.  Some fifty long vectors each along an axis of their own, whose own scores are 16 to 24 (base 2), among others
    that have one in the last column and score 0 against them.  A long row's last column is the sum of weights of 2^-16 to
    2^-24 of its own one.  Bound: the output's rounding, 2^-8 of it, and that of a weight in half precision, 2^-11, and of
    their sum and the row's, 2^-11."""
    import torch
    c2 = math.log2(math.e) / math.sqrt(d)
    w = hp.custom_workload("sym_small", 1, n, d, 1, d, 1, "bf16", SYM, 2950 + n)
    X = torch.zeros(1, n, d)
    X[:, :, d - 1] = 1.0
    long_rows = range(0, n, -(-n // 50))
    for axis, i in enumerate(long_rows):
        X[0, i] = 0.0
        X[0, i, axis] = math.sqrt((16.0 + 8.0 * (axis % 17) / 16.0) / c2)
    stored = {"X": X.to(torch.bfloat16), "Wq": torch.eye(d).to(torch.bfloat16), "Wk": None, "Wv": None, "lens": None}
    X, eye = stored["X"].double().numpy(), np.eye(d)
    ref = hp.oracle_forward(w, {"X": X, "Wq": eye, "Wk": eye, "Wv": eye}, SYM, 0.0)
    got = _sym_both_ways(w, stored, 0.0)
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-3)
    got, ref = got[0, list(long_rows), d - 1], ref[0, list(long_rows), d - 1]
    assert np.all(ref > 0.0) and np.all(np.abs(got - ref) <= (2.0 ** -8 + 2.0 ** -10) * ref), f"{np.abs(got / ref - 1.0).max():.2e}"


# ---- `out` need not start at a multiple of 16 bytes: 8 are enough on the matrix-core path ------------------
@pytest.mark.parametrize("kernel,scheme,tiles,shape", [
    # kernel, scheme, tile flag, (B, n, D, H, d, p)
    ("attn_split_kernel<64,", FULL, 0, (2, 200, 64, 2, 64, 25)),
    ("attn_split_kernel<128,", CAUSAL, 0, (2, 130, 64, 2, 128, 13)),
    ("attn_strands_kernel<64, 4,", CAUSAL, 0, (1, 1030, 64, 3, 64, 103)),
    ("attn_strands_kernel<64, 3,", FULL, 0, (2, 516, 64, 19, 64, 129)),
    ("attn_strands_kernel<128, 2,", CAUSAL, 0, (1, 1100, 64, 8, 128, 275)),
    ("attn_pipe_kernel<64, 4,", CAUSAL, ar.ATTN_FLAG_NARROW_TILES, (2, 300, 64, 2, 64, 75)),
    ("attn_pipe_kernel<64, 8,", FULL, ar.ATTN_FLAG_WIDE_TILES, (2, 300, 64, 2, 64, 75)),
    ("attn_pipe_kernel<128, 8,", FULL, ar.ATTN_FLAG_WIDE_TILES, (2, 300, 64, 1, 128, 75)),
    ("sym_pair_kernel<64>", SYM, 0, (2, 90, 64, 2, 64, 10)),      # one tile: stored by the pair kernel
    ("sym_pair_kernel<128>", SYM, 0, (2, 90, 64, 1, 128, 10)),
    ("sym_merge_kernel<64>", SYM, 0, (2, 300, 64, 2, 64, 75)),
])
def test_out_at_a_multiple_of_8_bytes(kernel, scheme, tiles, shape):
    import torch
    w = hp.custom_workload("out_8", *shape, "bf16", scheme, 3300)
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored, flags=tiles)
    try:
        aligned, _ = run.forward(scheme)
        room = torch.full((run.out.numel() + 16,), 7.0, dtype=run.out.dtype, device=run.out.device)
        for first in (4, 12):
            run.out = room[first:first + aligned.size].view(aligned.shape)
            assert run.out.data_ptr() % 16 == 8
            run.out.fill_(float("nan"))
            assert any(kernel in k for k in run.kernels(scheme))
            assert np.array_equal(run.forward(scheme)[0], aligned)
            assert torch.all(room[:first] == 7.0) and torch.all(room[first + aligned.size:] == 7.0)
            room.fill_(7.0)
    finally:
        run.close()


# ---- row maxima that move along the walk: the running reference of Eq. (2)'s online form ----------
@pytest.mark.parametrize("profile", ["ramp", "steps"])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("d_k,tiles", [(64, ar.ATTN_FLAG_NARROW_TILES), (64, ar.ATTN_FLAG_WIDE_TILES), (64, 0), (128, 0),
                                       (128, ar.ATTN_FLAG_WIDE_TILES)])
def test_reference_moves_along_the_walk(profile, scheme, d_k, tiles):
    """Scores with a designed level per key (inputs.make_level_inputs): `ramp` adds 60 nats at key 0
    falling to 0 at the last key, so along a walk towards key 0 the row maximum outgrows any fixed
    slack a dozen times; `steps` puts 8 and 32 keys 18 and 9 nats above the other thousand, whose
    share of the row sum (a few per cent down to 1e-4) is multiplied by hundreds if a rescaling of
    what has been accumulated is missed or misplaced.  The random part of the inputs makes the
    level's slope differ from row to row, falling along the walk for some."""
    B, n, D, H, p = 2, 1100, 64, 2, 275
    w = hp.custom_workload(f"levels_{profile}", B, n, D, H, d_k, p, "bf16", scheme, 900 + d_k)
    scale = hp.default_scale(w, 0.0)
    stored, f64 = inputs.make_level_inputs(w, profile, scale)
    print(f"[case] {w.name} d_k={d_k} scheme={scheme} tiles={tiles}", flush=True)
    for lens in (None, np.array([n, 700], dtype=np.int32)):
        stored["lens"] = lens
        run = hp.GpuRun(w, stored, flags=tiles)
        try:
            got, stats = run.forward(scheme)
        finally:
            run.close()
        ref = hp.oracle_forward(w, f64, scheme, 0.0, lens=lens)
        err = hp.tol_check(got, ref, w.dtype)
        hp.report_max_err(f"{w.name} d{d_k} scheme={scheme} tiles={tiles} lens={'yes' if lens is not None else 'no'}",
                          err, w.dtype)
        hp.check_counts(stats, hp.oracle_counts(w, scheme, lens))


# ---- the same in the kernels whose wavefronts share the keys: every strand has references of its own ----------
@pytest.mark.parametrize("profile", ["ramp", "steps"])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("kernel,shape", [
    # kernel, B, n, D, H, d, p
    ("attn_split_kernel<64,", (2, 900, 64, 2, 64, 225)),
    ("attn_split_kernel<128,", (2, 900, 64, 2, 128, 225)),
    ("attn_strands_kernel<64, 4,", (2, 1100, 64, 2, 64, 275)),
    ("attn_strands_kernel<64, 3,", (2, 900, 64, 10, 64, 225)),
    ("attn_strands_kernel<128, 2,", (2, 1100, 64, 4, 128, 275)),
])
def test_reference_moves_along_shared_walks(profile, scheme, kernel, shape):
    B, n, D, H, d, p = shape
    w = hp.custom_workload(f"shared_levels_{profile}", B, n, D, H, d, p, "bf16", scheme, 950 + d)
    stored, f64 = inputs.make_level_inputs(w, profile, hp.default_scale(w, 0.0))
    for lens in (None, np.array([n, 700], dtype=np.int32)):
        stored["lens"] = lens
        run = hp.GpuRun(w, stored)
        try:
            assert any(kernel in k for k in run.kernels(scheme))
            got, stats = run.forward(scheme)
        finally:
            run.close()
        hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens), w.dtype)
        hp.check_counts(stats, hp.oracle_counts(w, scheme, lens))


# ---- the -inf practice (Sec. 5.1) against skipping: identical bits ------------------------------
@pytest.mark.parametrize("case", [
    ("f32", 1, 48, 32, 2, 16, 6, 0),
    ("bf16", 2, 320, 64, 2, 64, 40, ar.ATTN_FLAG_NARROW_TILES),
    ("bf16", 1, 264, 64, 1, 128, 33, ar.ATTN_FLAG_NARROW_TILES),
    ("bf16", 2, 704, 64, 2, 64, 88, ar.ATTN_FLAG_WIDE_TILES),
    ("bf16", 1, 520, 64, 1, 128, 65, ar.ATTN_FLAG_WIDE_TILES),
])
@pytest.mark.parametrize("scheme", [FULL, SYM, CAUSAL])
def test_skip_equals_noskip_bits(case, scheme):
    dtype, B, n, D, H, d, p, tiles = case
    w = hp.custom_workload("bits", B, n, D, H, d, p, dtype, scheme, 31 + n)
    stored, _ = inputs.make_inputs(w)
    lens = None
    if scheme != SYM:
        lens = np.random.default_rng(5).integers(1, n + 1, B).astype(np.int32)
    stored["lens"] = lens
    outs = []
    for flags in (0, ar.ATTN_FLAG_NO_SKIP):
        run = hp.GpuRun(w, stored, flags=flags | tiles)
        try:
            got, stats = run.forward(scheme)
        finally:
            run.close()
        outs.append(got)
        hp.check_counts(stats, hp.oracle_counts(w, scheme, lens), noskip=bool(flags))
    assert np.array_equal(outs[0], outs[1])


# ---- workloads 2 and 3 in full -------------------------------------------------------------------
@pytest.mark.parametrize("name", ["encoder", "causal"])
def test_encoder_and_causal_full(name):
    w = inputs.WORKLOADS[name]
    err, stats = _run_and_compare(w, w.scheme, 0.0)
    print(f"{name}: max abs err {err:.3e}; tiles {stats['tiles_executed']}/{stats['tiles_full']}")
    if name == "causal":
        assert stats["pairs_needed"][0] == 50380800
        assert stats["tiles_executed"] == 96 * 8256


@pytest.mark.parametrize("dtype,scheme,unaligned", [("f32", FULL, False), ("f32", SYM, False), ("bf16", CAUSAL, False),
                                                    ("bf16", CAUSAL, True)])
def test_profile_reports_a_prepare_kernel_only_where_there_is_one(dtype, scheme, unaligned):
    """Kernels ahead of the projection: the weight re-layout for unaligned weights, none elsewhere."""
    import torch
    w = hp.custom_workload("profile", 2, 96, 64, 1, 64 if dtype == "bf16" else 48, 12, dtype, scheme, 61)
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored)
    try:
        if unaligned:
            for m in range(3):
                room = torch.empty(run.W[m].numel() + 1, dtype=run.W[m].dtype, device=run.X.device)
                run.W[m] = room[1:].view(run.W[m].shape).copy_(run.W[m])
        ar.attn_profile(run.ctx, True)
        for _ in range(3):
            run.forward(scheme)
        prof = ar.attn_profile_read(run.ctx)
    finally:
        run.close()
    assert prof["calls"] == 3 and prof["ms_projection"] > 0.0 and prof["ms_attention"] > 0.0
    assert (prof["ms_prepare"] > 0.0) == unaligned


def test_repeat_calls_are_stable():
    """Back-to-back calls on one context give identical bits and identical counts."""
    w = inputs.WORKLOADS["causal"]
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored)
    try:
        a, sa = run.forward(w.scheme)
        b, sb = run.forward(w.scheme)
    finally:
        run.close()
    assert np.array_equal(a, b) and sa == sb


@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_key_lengths_change_between_calls(scheme):
    """k and v rows past the key length are not projected; the workspace keeps whatever an earlier
    call with longer keys left there, and none of it may reach a result."""
    import torch
    w = hp.custom_workload("lens_change", 3, 600, 128, 2, 64, 75, "bf16", scheme, 77)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = np.array([600, 600, 517], dtype=np.int32)
    run = hp.GpuRun(w, stored)
    try:
        for lens in (stored["lens"], np.array([100, 300, 0], dtype=np.int32),
                     np.array([257, 64, 600], dtype=np.int32)):
            print(f"[lens] {lens.tolist()}", flush=True)
            dev_lens = torch.from_numpy(lens).to(run.X.device)
            ar.attn_set_key_lengths(run.ctx, dev_lens)
            got, stats = run.forward(scheme)
            hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens), w.dtype)
            hp.check_counts(stats, hp.oracle_counts(w, scheme, lens))
    finally:
        run.close()


# ---- padded vectors left out as queries too (ATTN_FLAG_SKIP_PADDED_ROWS) -------------------------
@pytest.mark.parametrize("case", [
    ("f32", 3, 48, 32, 2, 16, 6, 0),                                   # float path
    ("bf16", 3, 320, 64, 2, 64, 40, ar.ATTN_FLAG_NARROW_TILES),        # 128-row workgroups
    ("bf16", 3, 704, 128, 2, 64, 88, ar.ATTN_FLAG_WIDE_TILES),         # 256-row workgroups, d_k = 64
    ("bf16", 3, 600, 192, 1, 128, 75, 0),                              # d_k = 128, small launch
    ("bf16", 3, 600, 192, 1, 128, 75, ar.ATTN_FLAG_WIDE_TILES),        # 256-row workgroups, d_k = 128
    ("bf16", 3, 320, 64, 2, 64, 40, 0),                                # d_k = 64, small launch
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_padded_rows_left_out(case, scheme):
    dtype, B, n, D, H, d, p, tiles = case
    w = hp.custom_workload("skip_rows", B, n, D, H, d, p, dtype, scheme, 500 + n)
    stored, f64 = inputs.make_inputs(w)
    for lens in (np.array([n // 3 + 1, n, 0], dtype=np.int32), np.array([33, 1, n - 1], dtype=np.int32)):
        print(f"[lens] {lens.tolist()}", flush=True)
        stored["lens"] = lens
        outs = []
        for noskip in (0, ar.ATTN_FLAG_NO_SKIP):
            run = hp.GpuRun(w, stored, flags=tiles | ar.ATTN_FLAG_SKIP_PADDED_ROWS | noskip)
            try:
                got, stats = run.forward(scheme)
            finally:
                run.close()
            hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True), w.dtype)
            hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=True), noskip=bool(noskip))
            if _matrix_core_path(w, scheme) and not noskip:
                assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, lens, skip_padded_rows=True)
            for b, L in enumerate(lens):
                assert np.all(got[b, L:] == 0.0)
            outs.append(got)
        assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
@pytest.mark.parametrize("flags", [0, ar.ATTN_FLAG_SKIP_PADDED_ROWS])
def test_key_lengths_with_heads_dealt_over_the_xcds(scheme, flags):
    """A multiple of eight heads in all and key lengths: every XCD takes every eighth head."""
    w = hp.custom_workload("dealt", 4, 384, 64, 4, 64, 48, "bf16", scheme, 8181)
    stored, f64 = inputs.make_inputs(w)
    lens = np.array([384, 65, 200, 1], dtype=np.int32)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=flags)
    try:
        got, stats = run.forward(scheme)
    finally:
        run.close()
    rows_too = bool(flags)
    worst = hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=rows_too), w.dtype)
    hp.report_max_err(f"dealt scheme={scheme} flags={flags}", worst, w.dtype)
    hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=rows_too))
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, scheme, lens, skip_padded_rows=rows_too)


@pytest.mark.parametrize("case", [
    ("bf16", 3, 320, 64, 2, 64, 40, 0),
    ("bf16", 3, 320, 64, 2, 64, 40, ar.ATTN_FLAG_NARROW_TILES),
    ("bf16", 3, 704, 128, 2, 64, 88, ar.ATTN_FLAG_WIDE_TILES),
    ("bf16", 3, 600, 192, 1, 128, 75, 0),
    ("bf16", 3, 600, 192, 1, 128, 75, ar.ATTN_FLAG_WIDE_TILES),
    ("bf16", 3, 320, 72, 2, 64, 40, 0),      # d_model not in whole 64-deep slices: the other projection kernel
])
@pytest.mark.parametrize("scheme", [FULL, CAUSAL])
def test_packed_layout(case, scheme):
    """Items stored back to back: the checker's answer for the cut items, and bit for bit what the
    padded layout gives with the same lengths and the padded rows left out."""
    dtype, B, n, D, H, d, p, tiles = case
    w = hp.custom_workload("packed", B, n, D, H, d, p, dtype, scheme, 700 + n)
    stored, f64 = inputs.make_inputs(w)
    for lens in (np.array([n // 3 + 1, n, 0], dtype=np.int32), np.array([33, 1, n - 1], dtype=np.int32),
                 np.array([0, 0, 0], dtype=np.int32)):
        print(f"[lens] {lens.tolist()}", flush=True)
        stored["lens"] = lens
        run = hp.GpuRun(w, stored, flags=tiles | ar.ATTN_FLAG_SKIP_PADDED_ROWS)
        try:
            padded, stats_padded = run.forward(scheme)
            got, stats = run.forward_packed(scheme, lens)
            again, _ = run.forward_packed(scheme, lens)   # the workspace keeps nothing that matters
        finally:
            run.close()
        worst = hp.tol_check(got, hp.oracle_forward(w, f64, scheme, 0.0, lens=lens, skip_padded_rows=True), w.dtype)
        hp.report_max_err(f"packed {case[:7]} scheme {scheme} lens {lens.tolist()}", worst, w.dtype)
        hp.check_counts(stats, hp.oracle_counts(w, scheme, lens, skip_padded_rows=True))
        assert stats["phys_tiles_executed"] == stats_padded["phys_tiles_executed"]
        assert np.array_equal(got, padded)
        assert np.array_equal(got, again)


def test_packed_item_longer_than_n_is_cut():
    """An item with more rows than the context's n: its first n rows are the item, the rest take no part and
    their rows of out stay as they were."""
    import torch
    B, n, D, H, d, p = 2, 128, 64, 2, 64, 16
    w = hp.custom_workload("packed_cut", B, n, D, H, d, p, "bf16", CAUSAL, 911)
    stored, f64 = inputs.make_inputs(w)
    extra = 72                                   # item 0 has n + extra rows, item 1 has 64
    run = hp.GpuRun(w, stored)
    try:
        tail = (torch.randn(extra, D, device=run.X.device) * 3.0).to(run.X.dtype)
        Xp = torch.cat([run.X[0], tail, run.X[1, :64]], 0).contiguous()
        offs = torch.tensor([0, n + extra, n + extra + 64], dtype=torch.int32, device=run.X.device)
        outp = torch.full((Xp.shape[0] + 4, w.hd), float("nan"), dtype=run.X.dtype, device=run.X.device)
        ar.attn_forward_packed(run.ctx, offs, Xp, run.W[0], run.W[1], run.W[2], CAUSAL, outp)
        stats = ar.attn_stats(run.ctx)
        host = outp.to("cpu").to(torch.float64).numpy()
    finally:
        run.close()
    lens = np.array([n, 64], dtype=np.int32)
    ref = hp.oracle_forward(w, f64, CAUSAL, 0.0, lens=lens, skip_padded_rows=True)
    hp.tol_check(host[:n], ref[0], w.dtype)
    hp.tol_check(host[n + extra:n + extra + 64], ref[1, :64], w.dtype)
    assert np.all(np.isnan(host[n:n + extra])) and np.all(np.isnan(host[n + extra + 64:]))
    hp.check_counts(stats, hp.oracle_counts(w, CAUSAL, lens, skip_padded_rows=True))


def test_packed_layout_is_refused_off_the_matrix_core_path():
    w = hp.custom_workload("packed_f32", 2, 64, 64, 1, 64, 4, "f32", CAUSAL, 3)
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored)
    try:
        with pytest.raises(ar.AttnError) as e:
            run.forward_packed(CAUSAL, [10, 20])
        assert e.value.status == ar.ATTN_ERR_UNSUPPORTED
    finally:
        run.close()
    w = hp.custom_workload("packed_sym", 2, 128, 64, 1, 64, 4, "bf16", SYM, 3)
    stored, _ = inputs.make_inputs(w)
    run = hp.GpuRun(w, stored)
    try:
        with pytest.raises(ar.AttnError) as e:
            run.forward_packed(SYM, [10, 20])
        assert e.value.status == ar.ATTN_ERR_UNSUPPORTED
    finally:
        run.close()


def test_padded_workload_packed():
    """The padded workload stored back to back: bit for bit the padded layout's rows below the lengths."""
    w = inputs.WORKLOADS["padded"]
    lens = inputs.draw_lengths(w)
    stored, _ = inputs.make_inputs(w)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS)
    try:
        padded, stats_padded = run.forward(w.scheme)
        got, stats = run.forward_packed(w.scheme, lens)
    finally:
        run.close()
    assert np.array_equal(got, padded)
    for key in ("pairs_needed", "tiles_executed", "pairs_executed", "phys_tiles_executed"):
        assert stats[key] == stats_padded[key]


def test_padded_workload_with_padded_rows_left_out():
    w = inputs.WORKLOADS["padded"]
    lens = inputs.draw_lengths(w)
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored, flags=ar.ATTN_FLAG_SKIP_PADDED_ROWS)
    try:
        got, stats = run.forward(w.scheme)
    finally:
        run.close()
    assert np.all(np.isfinite(got))
    for b, L in enumerate(lens):
        assert np.all(got[b, L:] == 0.0)
    worst = 0.0
    for (b, h) in _sample_heads(w, 16, 11):
        rows = _sample_rows(w, 256, 100 * b + h, edges=_length_edges(w, int(lens[b])))
        print(f"[rows] b={b} h={h} len={int(lens[b])} {len(rows)} rows", flush=True)
        ref = orc.head_rows(f64["X"], f64["Wq"], f64["Wk"], f64["Wv"], n_heads=w.n_heads, d_k=w.d_k, p=w.p,
                            scheme=w.scheme, scale=hp.default_scale(w, 0.0), b=b, h=h, rows=rows, lens=lens,
                            skip_padded_rows=True)
        worst = max(worst, hp.tol_check(got[b, rows, h * w.d_k:(h + 1) * w.d_k], ref, w.dtype))
    hp.report_max_err("padded, padded rows left out, 16 heads x 256 rows", worst, w.dtype)
    hp.check_counts(stats, hp.oracle_counts(w, w.scheme, lens, skip_padded_rows=True))
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, w.scheme, lens, skip_padded_rows=True)
    assert stats["pairs_needed"][0] == 16 * 31887155


# ---- workloads 4 and 5: sampled rows + counts + a property that holds at any size --------------
TILE_EDGES = (32, 64, 128, 256)


def _tile_edges(w):
    """Rows on both sides of the first and last boundaries of every tile size the kernels use."""
    rows = {0, 1, w.n - 2, w.n - 1}
    for t in TILE_EDGES:
        for m in (t, 2 * t, w.n // 2, w.n - t):
            rows.update({m - 1, m, m + 1})
    return {r for r in rows if 0 <= r < w.n}


def _length_edges(w, L):
    """The rows around a key length, and around the tile boundaries next to it."""
    rows = _tile_edges(w) | {L - 1, L, L + 1}
    for t in TILE_EDGES:
        lo = (L // t) * t
        rows.update({lo - 1, lo, lo + t - 1, lo + t})
    return {r for r in rows if 0 <= r < w.n}


def _sample_rows(w, count, seed, edges):
    """`count` rows: the edge rows first, the rest drawn without replacement."""
    rng = np.random.default_rng(seed)
    rows = set(sorted(edges)[:count])
    pool = rng.permutation(w.n)
    for r in pool:
        if len(rows) >= min(count, w.n):
            break
        rows.add(int(r))
    return sorted(rows)


def _sample_heads(w, count, seed):
    """`count` distinct (batch, head) pairs, the first and the last among them."""
    rng = np.random.default_rng(seed)
    total = w.batch * w.n_heads
    ids = {0, total - 1}
    for x in rng.permutation(total):
        if len(ids) >= min(count, total):
            break
        ids.add(int(x))
    return [(i // w.n_heads, i % w.n_heads) for i in sorted(ids)]


def _sampled_rows(w, lens, picks):
    stored, f64 = inputs.make_inputs(w)
    stored["lens"] = lens
    run = hp.GpuRun(w, stored)
    try:
        got, stats = run.forward(w.scheme)
    finally:
        run.close()
    assert np.all(np.isfinite(got))
    worst = 0.0
    for (b, h, rows) in picks:
        print(f"[rows] b={b} h={h} {len(rows)} rows", flush=True)
        ref = orc.head_rows(f64["X"], f64["Wq"], f64["Wk"], f64["Wv"], n_heads=w.n_heads, d_k=w.d_k, p=w.p,
                            scheme=w.scheme, scale=hp.default_scale(w, 0.0), b=b, h=h, rows=rows, lens=lens)
        worst = max(worst, hp.tol_check(got[b, rows, h * w.d_k:(h + 1) * w.d_k], ref, w.dtype))
    hp.check_counts(stats, hp.oracle_counts(w, w.scheme, lens))
    assert stats["phys_tiles_executed"] == hp.expected_phys_blocks(w, w.scheme, lens)
    return worst, stats


def test_long_causal_sampled():
    """16 heads x 256 rows of the long workload (rows at the 32/64/128/256 tile edges among them)
    against the checker, element by element."""
    w = inputs.WORKLOADS["long"]
    picks = [(b, h, _sample_rows(w, 256, 7 + h, _tile_edges(w))) for (b, h) in _sample_heads(w, 16, 3)]
    worst, stats = _sampled_rows(w, None, picks)
    hp.report_max_err("long, 16 heads x 256 rows", worst, w.dtype)
    assert stats["pairs_needed"][0] == 1073872896
    assert stats["tiles_executed"] == 32 * 32896


def test_padded_batch_sampled():
    w = inputs.WORKLOADS["padded"]
    lens = inputs.draw_lengths(w)
    b_short, b_long = int(np.argmin(lens)), int(np.argmax(lens))
    heads = _sample_heads(w, 14, 5) + [(b_short, 0), (b_long, w.n_heads - 1)]
    picks = [(b, h, _sample_rows(w, 256, 100 * b + h, _length_edges(w, int(lens[b])))) for (b, h) in heads]
    worst, stats = _sampled_rows(w, lens, picks)
    hp.report_max_err("padded, 16 heads x 256 rows", worst, w.dtype)
    closed = sum(int(L) * (int(L) + 1) // 2 + (w.n - int(L)) * int(L) for L in lens) * w.n_heads
    assert stats["pairs_needed"][0] == closed


def test_zero_query_weights_give_prefix_means_at_full_size():
    """Wq = 0 makes all allowed weights equal, so y_i is the mean of v_0..v_i: checked for
    every row of sampled heads of the long workload against numpy's float64 matmul."""
    w = inputs.WORKLOADS["long"]
    stored, f64 = inputs.make_inputs(w, zero_wq=True)
    run = hp.GpuRun(w, stored)
    try:
        got, _ = run.forward(w.scheme)
    finally:
        run.close()
    for h in (0, 13, 31):
        V = f64["X"][0] @ f64["Wv"][:, h * w.d_k:(h + 1) * w.d_k]
        ref = np.cumsum(V, 0) / np.arange(1, w.n + 1)[:, None]
        hp.tol_check(got[0, :, h * w.d_k:(h + 1) * w.d_k], ref, w.dtype)
