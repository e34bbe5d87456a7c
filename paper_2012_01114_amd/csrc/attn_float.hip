// Phases 1-3 (Sec. 3.1, Eq. (1)-(3)) in float arithmetic, for every shape the 16-bit matrix-core
// kernels do not take: f32 storage, head sizes other than 64 and 128, unaligned pointers, and the
// q = k = v scheme on them.  q, k, v: float [B][H][N][d], d <= 256.
//
// Bound by the float matrix cores (v_mfma_f32_16x16x4_f32: one fp32 fma per product; 157 TFLOP/s on
// the chip).  An MFMA takes 32 cycles, so one operand read from LDS and the vector work of the
// softmax fit beside it, and plain staging through registers is enough: a workgroup walks 64-key
// tiles of K and V, the next tile is fetched while the current one is contracted.
//
// Scores are computed transposed, S^T = K.Q^T: a lane holds four keys of ONE query per 16 x 16
// block, and accumulator register r of the block is, as it stands, the B operand of the MFMA that
// adds keys {r, 4 + r, 8 + r, 12 + r} to O^T += V^T.P^T: the weights never leave their registers
// and a row needs two cross-lane steps per tile (its maximum).  The four products of a score MFMA
// are chosen so that an operand is a quarter of a 16-byte LDS read (lane group g4 holds columns
// 16t + 4 g4 + j in MFMA j); both orders only order the fp32 sums.
//
// The columns of O that the MFMAs of a key hold are dealt so that an operand of four MFMAs is one
// 16-byte read of a row of V (column 4i + e of a 64-column group in MFMA e), which makes the lane's
// outputs runs of four columns as well.
//
// A wavefront owns 16 query rows.  Two kernels:
//   rows  64 rows per workgroup, every wavefront walks all keys; K and V tiles of 64 keys pass
//         through LDS, the next one fetched into registers meanwhile;
//   keys  16 rows per workgroup, its four wavefronts take the 16-key blocks in turn, straight from
//         memory (L2) into operand registers, and their partial states (m, l, O) are merged at the
//         end: four times the wavefronts, no barrier in the walk, four times the reads of K and V.
// The paper's ring: the walk of the rows kernel starts at the rows' own tile and runs downwards,
// wrapping (the order in which PE l meets block (l - j) mod m in Algorithm 1; the q = k = v scheme's
// walk over stored scores enters the ring one tile further and ends at the own one); in both, blocks
// of 16 keys with no needed pair are left out (Sec. 5.1).
//
// q = k = v scheme (Sec. 4): a first kernel computes every score tile once and stores it at both
// of its places of an n x n matrix per head, the same walk then reads its scores from there.
#include <type_traits>

#include "attn_common.h"

namespace attnring {
namespace {

constexpr int KT = 64;  // keys per tile

// Workgroups are numbered through a grid of rows of at most 2^22 (a grid dimension of more than
// 2^32 threads does not exist); the numbers past the last do nothing.
inline dim3 flat_grid(size_t count)
{
    const size_t row = (size_t)1 << 22;
    return dim3((unsigned)(count < row ? count : row), (unsigned)((count + row - 1) / row));
}
__device__ __forceinline__ unsigned flat_block() { return blockIdx.y * gridDim.x + blockIdx.x; }

// Row pitch of the stored score matrices: whole 16-byte pieces, unless only rows without a gap stay
// within the bound.  Pieces then lie at any multiple of 4 bytes and a row's last one reaches into the row
// behind it (the buffer has room for the last row's): what is read there is masked, nothing is written.
__host__ __device__ __forceinline__ int score_pitch(const Problem& pb)
{
    const int whole = (pb.N + 3) & ~3;
    return (size_t)pb.B * pb.H * pb.N * whole * sizeof(float) <= MAX_SCORE_BYTES ? whole : pb.N;
}
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 mfma16f(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Four floats at column `col` of a row of d, zeros past its end (and if not `there`).  No branch: a
// load behind one would wait for all loads in flight.  WHOLE: pieces lie inside or outside the row,
// and what is to be dropped is dropped by clip4 when the piece is used, since that waits for the load.
template <bool WHOLE>
__device__ __forceinline__ f32x4 load4(const float* __restrict__ row, int col, int d, bool there)
{
    f32x4 v;
    if constexpr (WHOLE) {
        v = *(const f32x4*)(row + (col < d ? col : 0));
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = col + j < d;
            const float w = row[in ? col + j : 0];
            v[j] = there && in ? w : 0.f;
        }
    }
    return v;
}

template <bool WHOLE>
__device__ __forceinline__ f32x4 clip4(f32x4 v, bool in)
{
    if constexpr (WHOLE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = in ? v[j] : 0.f;
    }
    return v;
}

// exp(x), x <= 0, as a power of two: x * log2(e) is rounded once, which moves the result by |x| / 2 ulp
// at most, where it is small against the row's largest weight of 1.
__device__ __forceinline__ float exp_neg(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// Four outputs of a row at column `col`.
__device__ __forceinline__ void store4(void* out, size_t row_base, int col, int d, f32x4 y, bool bf16, bool whole)
{
    if (whole) {
        if (col >= d) return;
        if (bf16) *(u32x2*)((bf16_t*)out + row_base + col) = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
        else *(f32x4*)((float*)out + row_base + col) = y;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (col + j >= d) break;
            if (bf16) ((bf16_t*)out)[row_base + col + j] = (bf16_t)(pack_bf16(y[j], 0.f) & 0xffffu);
            else ((float*)out)[row_base + col + j] = y[j];
        }
    }
}

// A 64-row tile of K or V as float4 pieces in registers, then LDS rows of 16 NDB + 4 floats (the
// pitch puts 16 rows, and rows 4 apart, on different banks); rows at or past `limit` and columns
// at or past d are zeros.
template <int NDB, bool WHOLE>
struct Tile {
    static constexpr int DP = 16 * NDB, PITCH = DP + 4, PPR = DP / 4, PER = KT * PPR / 256;
    f32x4 reg[PER];
    __device__ __forceinline__ void fetch(const float* __restrict__ src, int j0, int limit, int d, int tid)
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int c = tid + 256 * u, r = c / PPR, col = (c % PPR) * 4;
            const int j = j0 + r < limit ? j0 + r : (limit > 0 ? limit - 1 : 0);
            reg[u] = load4<WHOLE>(src + (size_t)j * d, col, d, j0 + r < limit);
        }
    }
    __device__ __forceinline__ void stage(float* dst, int j0, int limit, int d, int tid) const
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int c = tid + 256 * u;
            const int r = c / PPR, col = (c % PPR) * 4;
            *(f32x4*)(dst + r * PITCH + col) = clip4<WHOLE>(reg[u], j0 + r < limit && col < d);
        }
    }
};

// The lane's row as the B operand of the score MFMAs.
template <int NDB, bool WHOLE>
__device__ __forceinline__ void load_row(f32x4 (&qf)[NDB], const float* __restrict__ row, int g4, int d)
{
#pragma unroll
    for (int t = 0; t < NDB; ++t) qf[t] = clip4<WHOLE>(load4<WHOLE>(row, 16 * t + 4 * g4, d, true), 16 * t + 4 * g4 < d);
}

// The columns of a row of d in MFMA order: groups of 64, then one of 32, then one of 16.
template <int NDB>
struct Cols {
    static constexpr int N4 = NDB / 4, N2 = (NDB % 4) / 2, N1 = NDB % 2;
    static constexpr int C2 = 64 * N4, C1 = C2 + 32 * N2;
    // lane ln's V operands of one key: column 64m + 4 ln + e in MFMA 4m + e, and so on
    template <class L4, class L2, class L1>
    static __device__ __forceinline__ void read(float (&v)[NDB], int ln, L4&& l4, L2&& l2, L1&& l1)
    {
#pragma unroll
        for (int m = 0; m < N4; ++m) {
            const f32x4 w = l4(64 * m + 4 * ln);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * m + e] = w[e];
        }
        if constexpr (N2 != 0) {
            const f32x2 w = l2(C2 + 2 * ln);
            v[4 * N4] = w[0];
            v[4 * N4 + 1] = w[1];
        }
        if constexpr (N1 != 0) v[NDB - 1] = l1(C1 + ln);
    }
    // column of register r of O[db]
    static __device__ __forceinline__ int column(int db, int r, int g4)
    {
        if (db < 4 * N4) return 64 * (db / 4) + 16 * g4 + 4 * r + db % 4;
        if (db < 4 * N4 + 2 * N2) return C2 + 8 * g4 + 2 * r + (db - 4 * N4);
        return C1 + 4 * g4 + r;
    }
    // f(column, four outputs) for the lane's pieces of its row
    template <class F>
    static __device__ __forceinline__ void pieces(const f32x4 (&O)[NDB], int g4, F&& f)
    {
#pragma unroll
        for (int m = 0; m < N4; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(64 * m + 16 * g4 + 4 * r, f32x4{O[4 * m][r], O[4 * m + 1][r], O[4 * m + 2][r], O[4 * m + 3][r]});
        if constexpr (N2 != 0) {
            constexpr int b = 4 * N4;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                f(C2 + 8 * g4 + 4 * u, f32x4{O[b][2 * u], O[b + 1][2 * u], O[b][2 * u + 1], O[b + 1][2 * u + 1]});
        }
        if constexpr (N1 != 0) f(C1 + 4 * g4, O[NDB - 1]);
    }
};

// Running state of the lane's row (m shared by the row's four lanes, l this lane's part).
template <int NDB>
struct Row {
    f32x4 O[NDB];
    float m, l;
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int db = 0; db < NDB; ++db) O[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        m = -INFINITY;
        l = 0.f;
    }
    // Phase 2 (Eq. (2)) of NB blocks of scores: they become weights.  rel: the last allowed key,
    // counted from the lane's first key.  A row that has met no allowed key keeps m = -inf.
    template <int NB>
    __device__ __forceinline__ void weights(f32x4 (&S)[NB], int rel)
    {
        float mx = m;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[b][r] = 16 * b + r <= rel ? S[b][r] : -INFINITY;
                mx = fmaxf(mx, S[b][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float ref = mx > -INFINITY ? mx : 0.f;
        const float alpha = exp_neg(m - ref);
        m = mx;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[b][r] = exp_neg(S[b][r] - ref);
        f32x4 sum = S[0];  // added up in a tree: fewer roundings behind a large weight
        if constexpr (NB == 4) sum = (S[0] + S[1]) + (S[2] + S[3]);
        l = l * alpha + ((sum[0] + sum[1]) + (sum[2] + sum[3]));
#pragma unroll
        for (int db = 0; db < NDB; ++db) O[db] *= alpha;
    }
    __device__ __forceinline__ float row_sum() const
    {
        float t = l + __shfl_xor(l, 16, 64);
        return t + __shfl_xor(t, 32, 64);
    }
};

// A weight of zero is no protection from a value that is not finite (0 * inf), so the 16-key block that
// the diagonal cuts, if it holds such a value, stays out of the MFMAs: its weights are put aside and, behind
// the walk, each row adds its allowed keys only, one by one.
template <int NDB>
struct CutBlock {
    f32x4 w;
    float m;   // the reference of the weights
    int key0;  // first key of the block; -1: nothing was put aside
    __device__ __forceinline__ void clear() { key0 = -1; }
    // `poison` turns into NaN if a value is an infinity or NaN
    static __device__ __forceinline__ float test(float poison, const float (&v)[NDB])
    {
#pragma unroll
        for (int db = 0; db < NDB; ++db) poison = fmaf(v[db], 0.f, poison);
        return poison;
    }
    // i0: the wavefront's first row; a block above the diagonal (debug mode) has nothing to add
    __device__ __forceinline__ void put_aside(const f32x4& weights, float ref, int key, int i0)
    {
        if (key > i0) return;
        w = weights;
        m = ref;
        key0 = key;
    }
    __device__ __forceinline__ void add(Row<NDB>& row, const float* __restrict__ vh, int d, int last_allowed, int ln, int g4) const
    {
        if (key0 < 0) return;
        const float scale = exp_neg(m - (row.m > -INFINITY ? row.m : 0.f));
#pragma nounroll
        for (int key = 0; key < 16; ++key) {
            const int r = key & 3;
            const float p = scale * __shfl(r == 0 ? w[0] : r == 1 ? w[1] : r == 2 ? w[2] : w[3], 16 * (key >> 2) + ln, 64);
            if (key0 + key > last_allowed) continue;
            const float* vrow = vh + (size_t)(key0 + key) * d;
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int c = Cols<NDB>::column(db, e, g4);
                    row.O[db][e] = fmaf(p, vrow[c < d ? c : 0], row.O[db][e]);
                }
                __builtin_amdgcn_sched_barrier(0);  // rare: registers count, not time
            }
        }
    }
};

// What both kernels need to know about a row tile.
struct RowTile {
    int bh, bb, h, i0, row_end, len, rlen;
    bool there;
    __device__ __forceinline__ RowTile(const Problem& pb, int rows, int n_rowtiles)
    {
        // Consecutive workgroups take the heads in turn, the last row tiles (the most keys under the
        // mask) first, so that the long walks do not start last.
        const unsigned heads = (unsigned)(pb.B * pb.H), item = flat_block();
        there = item < heads * (unsigned)n_rowtiles;
        bh = (int)(item % heads);
        bb = bh / pb.H;
        h = bh - bb * pb.H;
        i0 = (n_rowtiles - 1 - (int)(item / heads)) * rows;
        len = pb.N;
        if (there && pb.lens) { len = pb.lens[bb]; len = len < 0 ? 0 : (len > pb.N ? pb.N : len); }
        rlen = pb.skip_rows ? len : pb.N;                   // query rows at or past it take part in no pair
        row_end = min(pb.noskip ? pb.N : rlen, i0 + rows);  // rows of the tile that take part
    }
    // Logical tiles: row block I is counted by the workgroup that holds its first row; called by one wavefront.
    __device__ __forceinline__ void count(const Problem& pb, const CountCfg& cc, int lane) const
    {
        unsigned cnt = 0;
        const int I = (int)cdiv_b((unsigned)i0, cc) + lane;  // at most 64 row blocks start here
        if (I * cc.b < row_end) {
            cnt = (unsigned)pb.P;
            if (!pb.noskip) {
                if (pb.scheme == SCHEME_CAUSAL) cnt = min(cnt, (unsigned)I + 1u);
                cnt = min(cnt, cdiv_b((unsigned)len, cc));
            }
        }
        unsigned long long total = cnt;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
        if (lane == 0) count_add(pb.counters, flat_block(), total, 0);
    }
    // The row's last allowed key; -1: it has none, and its output is zero whatever its weights of zero met (0 * inf).
    __device__ __forceinline__ int last_key(const Problem& pb, int i) const
    {
        if (i >= rlen) return -1;
        return pb.scheme == SCHEME_CAUSAL ? min(len - 1, i) : len - 1;
    }
};

// Phase 1 (Eq. (1), before the scale) of NB 16-key blocks from key row `kt` of an LDS tile.
template <int NDB, int NB>
__device__ __forceinline__ void score_blocks(f32x4* S, const float* kt, const f32x4 (&qf)[NDB], int ln, int g4)
{
    constexpr int PITCH = Tile<NDB, true>::PITCH;
#pragma unroll
    for (int b = 0; b < NB; ++b) S[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NDB; ++t) {
        f32x4 kf[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) kf[b] = *(const f32x4*)(kt + (16 * b + ln) * PITCH + 16 * t + 4 * g4);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b) S[b] = mfma16f(kf[b][j], qf[t][j], S[b]);
    }
}

// CAUSAL, in both kernels: the masked scheme, or, of the large heads whose rows are no whole pieces, either
// scheme (d = 190, FULL: 112 us, 140 with a kernel of its own, at the same registers).
template <int NDB, bool WHOLE>
constexpr bool EITHER = !WHOLE && NDB >= 12;

// STORED (q = k = v scheme), in both kernels: the scores come from `scores`, which
// sym_scores_float_kernel has filled, instead of q and k, and have been counted there.
template <int NDB, bool WHOLE, bool STORED, bool CAUSAL>
__global__ __launch_bounds__(256, NDB <= 4 ? 3 : NDB <= 8 ? 2 : 1)
void attn_rows_kernel(Problem pb, CountCfg cc, const float* __restrict__ q, const float* __restrict__ k,
                      const float* __restrict__ v, const float* __restrict__ scores, void* __restrict__ out,
                      int n_rowtiles, bool out_whole)
{
    typedef Tile<NDB, WHOLE> TL;
    typedef Cols<NDB> CL;
    constexpr int PITCH = TL::PITCH, NB = 4;
    __shared__ __attribute__((aligned(16))) float ks[STORED ? 4 : KT * PITCH];
    __shared__ __attribute__((aligned(16))) float vs[KT * PITCH];

    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RowTile rt(pb, KT, n_rowtiles);
    if (!rt.there) return;
    const int N = pb.N, d = pb.d, len = rt.len;
    const bool causal = CAUSAL && (!EITHER<NDB, WHOLE> || pb.scheme == SCHEME_CAUSAL);
    const size_t head = (size_t)rt.bh * N * d;
    const int i0w = rt.i0 + 16 * wave, i = i0w + ln;  // rows of the wavefront, the lane's row
    const int wave_end = min(rt.row_end, i0w + 16);

    // needed tiles are 0 .. nJ-1, met from the own one downwards, wrapping; in debug mode the
    // others follow and change nothing
    int nJ = 0, nT = 0;
    if (rt.row_end > rt.i0) {
        nJ = (len + KT - 1) / KT;
        if (causal) nJ = min(nJ, (rt.row_end - 1) / KT + 1);
        nT = pb.noskip ? (N + KT - 1) / KT : nJ;
    }
    // q = k = v: the own tile holds the row's largest weight by far (its own vector's), and everything added
    // behind it would be rounded at that size, so it comes last: error against 64 bits at 2 x 2048, 8 heads of
    // 128, 2.9e-7 (own tile first 1.3e-6, keys in their order 9.0e-7).
    const int own = min(rt.i0 / KT, nJ - 1);
    const int Js = !STORED ? own : own > 0 ? own - 1 : nJ - 1;
    auto tile_of_step = [&](int t) -> int {
        if (t >= nJ) return t;
        const int J = Js - t;
        return J < 0 ? J + nJ : J;
    };
    if (!STORED && wave == 0) rt.count(pb, cc, lane);
    unsigned cnt_phys = 0;  // 16 x 16 score blocks; wave-uniform

    f32x4 qf[NDB];
    if constexpr (!STORED) load_row<NDB, WHOLE>(qf, q + head + (size_t)min(i, N - 1) * d, g4, d);  // rows past the last: not stored
    Row<NDB> row;
    row.clear();
    CutBlock<NDB> cut;
    cut.clear();
    const int last_allowed = rt.last_key(pb, i), lim = last_allowed - 4 * g4;
    // the lane's stored scores of a tile: whole 16-byte pieces of its row (pitch SP)
    const int SP = score_pitch(pb);
    const float* srow = STORED ? scores + ((size_t)rt.bh * N + min(i, N - 1)) * SP : nullptr;
    TL tk, tv;
    f32x4 sreg[NB];
    auto fetch = [&](int t) {
        const int J = tile_of_step(t);
        if constexpr (STORED) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int col = J * KT + 16 * b + 4 * g4;
                sreg[b] = *(const f32x4_any*)(srow + (col < SP ? col : 0));
            }
        } else {
            tk.fetch(k + head, J * KT, len, d, tid);
        }
        tv.fetch(v + head, J * KT, len, d, tid);
    };
    // The own tile, the only one with blocks that the diagonal cuts (values past the row tile's last row are
    // staged as zeros), is met first; the other tiles then go without a look at their values, which keeps
    // branches out of the loop (8 x 1024, 12 heads of 64: 142 -> 138 us).  At the large head sizes two
    // copies of the body are not worth it.
    constexpr bool FIRST_ALONE = CAUSAL && NDB <= 8;
    const int v_end = causal ? min(len, rt.row_end) : len;
    auto walk_tile = [&](int t, auto cut_) __attribute__((always_inline)) {
        constexpr bool CUT = decltype(cut_)::value;
        const int J = tile_of_step(t);
        f32x4 S[NB];
        __syncthreads();  // everyone is done with the tile before
        if constexpr (STORED) {
#pragma unroll
            for (int b = 0; b < NB; ++b) S[b] = sreg[b];
        } else {
            tk.stage(ks, J * KT, len, d, tid);
        }
        tv.stage(vs, J * KT, v_end, d, tid);
        __syncthreads();
        if (t + 1 < nT) fetch(t + 1);
        // 16-key blocks of the tile that hold a pair this wavefront needs: the first nk
        int nk = 0;
        if (wave_end > i0w) {
            int keys = len - J * KT;
            if (causal) keys = min(keys, wave_end - J * KT);
            nk = pb.noskip ? NB : max(0, min(NB, (keys + 15) >> 4));
        }
        if (nk == 0) return;
        if constexpr (!STORED) {
            cnt_phys += (unsigned)nk;
            if (nk == NB) {
                score_blocks<NDB, NB>(S, ks, qf, ln, g4);
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    S[b] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (b < nk) score_blocks<NDB, 1>(&S[b], ks + 16 * b * PITCH, qf, ln, g4);
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) S[b] *= pb.scale;
        }
        row.weights(S, lim - J * KT);
        // phase 3 (Eq. (3))
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= nk) break;
            auto read = [&](float (&vf)[NDB], int r) {
                const float* vrow = vs + (16 * b + 4 * g4 + r) * PITCH;
                CL::read(vf, ln, [&](int c) { return *(const f32x4*)(vrow + c); },
                         [&](int c) { return *(const f32x2*)(vrow + c); }, [&](int c) { return vrow[c]; });
            };
            if (CUT && causal && J * KT + 16 * b + 15 > i0w) {
                float poison = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float vf[NDB];
                    read(vf, r);
                    poison = CutBlock<NDB>::test(poison, vf);
                }
                if (__builtin_amdgcn_ballot_w64(poison != poison) != 0ull) {
                    cut.put_aside(S[b], row.m, J * KT + 16 * b, i0w);
                    continue;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float vf[NDB];
                read(vf, r);
#pragma unroll
                for (int db = 0; db < NDB; ++db) row.O[db] = mfma16f(vf[db], S[b][r], row.O[db]);
            }
        }
    };
    if (nT > 0) {
        fetch(0);
        if constexpr (FIRST_ALONE) walk_tile(0, std::true_type{});
        for (int t = FIRST_ALONE ? 1 : 0; t < nT; ++t) walk_tile(t, std::integral_constant<bool, CAUSAL && !FIRST_ALONE>{});
    }
    if constexpr (!STORED) cut.add(row, v + head, d, last_allowed, ln, g4);
    const float L = row.row_sum();
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const size_t base = ((size_t)rt.bb * N + i) * ((size_t)pb.H * d) + (size_t)rt.h * d;
    if (i < N)
        CL::pieces(row.O, g4, [&](int c, f32x4 y) {
            store4(out, base, c, d, last_allowed < 0 ? zero : y * inv, pb.is_bf16, out_whole);
        });
    if (!STORED && lane == 0) count_add(pb.counters, flat_block(), 0, cnt_phys);
}

// EXACT: d is 16 NDB, no column is dropped.
template <int NDB, bool WHOLE, bool EXACT, bool STORED, bool CAUSAL>
__global__ __launch_bounds__(256, NDB <= 4 ? 3 : NDB <= 6 ? 2 : 1)  // three wavefronts per SIMD at d = 64 rather than two
void attn_keys_kernel(Problem pb, CountCfg cc, const float* __restrict__ q, const float* __restrict__ k,
                      const float* __restrict__ v, const float* __restrict__ scores, void* __restrict__ out,
                      int n_rowtiles, bool out_whole)
{
    typedef Cols<NDB> CL;
    constexpr int DP = 16 * NDB, PITCH = DP + 4;
    __shared__ __attribute__((aligned(16))) float st_o[64 * PITCH];  // [4][16] rows
    __shared__ float st_ml[2 * 64];

    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RowTile rt(pb, 16, n_rowtiles);
    if (!rt.there) return;
    const int N = pb.N, d = pb.d, len = rt.len, last = len > 0 ? len - 1 : 0;
    const size_t head = (size_t)rt.bh * N * d;
    const float *kh = k + head, *vh = v + head;
    const int i = rt.i0 + ln;  // the lane's row
    const bool causal = CAUSAL && (!EITHER<NDB, WHOLE> || pb.scheme == SCHEME_CAUSAL);
    // blocks 0 .. nb-1 hold a needed pair; in debug mode the others follow and change nothing
    int nb = 0;
    if (rt.row_end > rt.i0) {
        nb = (len + 15) / 16;
        if (causal) nb = min(nb, (rt.row_end - 1) / 16 + 1);
        if (pb.noskip) nb = (N + 15) / 16;
    }
    f32x4 qf[NDB];
    if constexpr (!STORED) load_row<NDB, WHOLE>(qf, q + head + (size_t)min(i, N - 1) * d, g4, d);
    const int SP = score_pitch(pb);
    const float* srow = STORED ? scores + ((size_t)rt.bh * N + min(i, N - 1)) * SP : nullptr;

    // Operands of a block: the lane's pieces of key row ln, and of V rows 4 g4 .. 4 g4 + 3; what lies
    // past the length or past d is read from a row that exists and dropped.
    struct Block {
        f32x4 k[STORED ? 1 : NDB];
        float v[4][NDB];
    };
    auto load = [&](Block& x, int b) {
        if constexpr (STORED) {
            const int col = 16 * b + 4 * g4;
            x.k[0] = *(const f32x4_any*)(srow + (col < SP ? col : 0));
        } else {
            const float* krow = kh + (size_t)min(16 * b + ln, last) * d;
#pragma unroll
            for (int t = 0; t < NDB; ++t) x.k[t] = load4<WHOLE>(krow, 16 * t + 4 * g4, d, true);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* vrow = vh + (size_t)min(16 * b + 4 * g4 + r, last) * d;
            CL::read(x.v[r], ln, [&](int c) { return load4<WHOLE>(vrow, c, d, true); },
                     [&](int c) {
                         if constexpr (WHOLE) return *(const f32x2*)(vrow + (c < d ? c : 0));
                         else return f32x2{vrow[c < d ? c : 0], vrow[c + 1 < d ? c + 1 : 0]};
                     },
                     [&](int c) { return vrow[c < d ? c : 0]; });
        }
    };
    Row<NDB> row;
    row.clear();
    CutBlock<NDB> cut;
    cut.clear();
    unsigned cnt_phys = 0;
    const int last_allowed = rt.last_key(pb, i), lim = last_allowed - 4 * g4;
    // Blocks below plain_end hold allowed keys only; the others, cut by the diagonal or the length, follow:
    // one at most, the last of the walk, but for the debug mode.  They have code of their own, which keeps
    // branches out of the loop (4 x 600, 8 heads of 80, masked: 38.4 -> 36 us).
    const int plain_end = (causal ? min(len, rt.i0) : len) >> 4;
    // below_: the block ends below the tile's first row; inside_: below the length.
    auto step = [&](Block& x, int b, auto below_, auto inside_) {
        f32x4 S[1] = {{0.f, 0.f, 0.f, 0.f}};
        if constexpr (STORED) {
            S[0] = x.k[0];
        } else {
            ++cnt_phys;
            // two chains: a product waits for the one before it in its own
            f32x4 s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < NDB; ++t) {
                const f32x4 kf = EXACT ? x.k[t] : clip4<WHOLE>(x.k[t], 16 * t + 4 * g4 < d);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j & 1) s2 = mfma16f(kf[j], qf[t][j], s2);
                    else S[0] = mfma16f(kf[j], qf[t][j], S[0]);
                }
            }
            S[0] = (S[0] + s2) * pb.scale;
        }
        row.weights(S, lim - 16 * b);
        if (CAUSAL && causal && !below_) {
            float poison = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) poison = CutBlock<NDB>::test(poison, x.v[r]);
            if (__builtin_amdgcn_ballot_w64(poison != poison) != 0ull) {
                cut.put_aside(S[0], row.m, 16 * b, rt.i0);
                return;
            }
        }
        if (inside_) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int db = 0; db < NDB; ++db) row.O[db] = mfma16f(x.v[r][db], S[0][r], row.O[db]);
        } else {  // keys past the length: nothing of them reaches O
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = 16 * b + 4 * g4 + r < len;
#pragma unroll
                for (int db = 0; db < NDB; ++db) row.O[db] = mfma16f(in ? x.v[r][db] : 0.f, S[0][r], row.O[db]);
            }
        }
    };
    auto plain = [&](Block& x, int b) __attribute__((always_inline)) { step(x, b, std::true_type{}, std::true_type{}); };
    auto edge = [&](Block& x, int b) __attribute__((always_inline)) { step(x, b, std::false_type{}, std::false_type{}); };
    if (wave < nb) {
        int b = wave;
        if constexpr (NDB <= 8) {
            Block x0, x1;
            load(x0, b);
            if constexpr (WHOLE || NDB <= 5) {
                while (true) {
                    if (b >= plain_end) {
                        if (b < nb) edge(x0, b);
                        break;
                    }
                    // the requests stay in front: left alone, the compiler sinks each to where its wait stands
                    load(x1, b + 4);
                    __builtin_amdgcn_sched_barrier(0);
                    plain(x0, b);
                    __builtin_amdgcn_sched_barrier(0);
                    b += 4;
                    if (b >= plain_end) {
                        if (b < nb) edge(x1, b);
                        break;
                    }
                    load(x0, b + 4);
                    __builtin_amdgcn_sched_barrier(0);
                    plain(x1, b);
                    __builtin_amdgcn_sched_barrier(0);
                    b += 4;
                }
                for (b += 4; b < nb; b += 4) {
                    load(x0, b);
                    edge(x0, b);
                }
            } else {  // rows in no whole pieces: one body with branches is the smaller one (d = 113: 57 us, 81 with two)
                while (true) {
                    load(x1, b + 4);
                    __builtin_amdgcn_sched_barrier(0);
                    step(x0, b, 16 * b + 16 <= rt.i0, 16 * b + 16 <= len);
                    __builtin_amdgcn_sched_barrier(0);
                    b += 4;
                    if (b >= nb) break;
                    load(x0, b + 4);
                    __builtin_amdgcn_sched_barrier(0);
                    step(x1, b, 16 * b + 16 <= rt.i0, 16 * b + 16 <= len);
                    __builtin_amdgcn_sched_barrier(0);
                    b += 4;
                    if (b >= nb) break;
                }
            }
        } else {  // two blocks would not fit the registers
            for (; b < nb; b += 4) {
                Block x;
                load(x, b);
                if constexpr (!WHOLE) step(x, b, 16 * b + 16 <= rt.i0, 16 * b + 16 <= len);
                else if (b < plain_end) plain(x, b);
                else edge(x, b);
            }
        }
    }
    if (!STORED && wave == 0) rt.count(pb, cc, lane);
    if (!STORED && lane == 0) count_add(pb.counters, flat_block(), 0, cnt_phys);

    if constexpr (!STORED) cut.add(row, vh, d, last_allowed, ln, g4);

    // partial state of wavefront w, row r: m, l, then O
    const float L0 = row.row_sum();
    CL::pieces(row.O, g4, [&](int c, f32x4 y) { *(f32x4*)(st_o + (16 * wave + ln) * PITCH + c) = y; });
    if (g4 == 0) {
        st_ml[2 * (16 * wave + ln)] = row.m;
        st_ml[2 * (16 * wave + ln) + 1] = L0;
    }
    __syncthreads();
    const int r = tid >> 4;
    float mw[4], M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        mw[w] = st_ml[2 * (16 * w + r)];
        M = fmaxf(M, mw[w]);
    }
    const float ref = M > -INFINITY ? M : 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        mw[w] = exp_neg(mw[w] - ref);
        L += mw[w] * st_ml[2 * (16 * w + r) + 1];
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const bool none = rt.last_key(pb, rt.i0 + r) < 0;
    const size_t base = ((size_t)rt.bb * N + rt.i0 + r) * ((size_t)pb.H * d) + (size_t)rt.h * d;
    if (rt.i0 + r < N)
        for (int c = tid & 15; c < DP / 4; c += 16) {
            f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) y += mw[w] * *(const f32x4*)(st_o + (16 * w + r) * PITCH + 4 * c);
            y *= inv;
            if (none) y = f32x4{0.f, 0.f, 0.f, 0.f};
            store4(out, base, 4 * c, d, y, pb.is_bf16, out_whole);
        }
}

// Phase 1 of the q = k = v scheme (Sec. 4.1, Eq. (4)): one workgroup per unordered pair of 64-row
// tiles of z computes S_AB = scale * z_A . z_B^T once and stores it at both places, w'_ji = w'_ij.
// The paper's rule (Sec. 4.2: circulant diagonals 0 .. floor(P/2) of the P x P matrix of n/P-row
// tiles, the middle one by both owners when P is even) fixes which of the two a ring of P
// processing elements computes; the logical tiles it selects are counted over the regions the
// workgroup covers (each position of the P x P matrix lies in exactly one use).  Products and their
// order are the same in both orientations, so S is symmetric to the bit, and the debug mode, which
// computes every ordered pair in its own orientation, gives the same bits.
template <int NDB, bool WHOLE>
__global__ __launch_bounds__(256)
void sym_scores_float_kernel(Problem pb, CountCfg cc, const float* __restrict__ z, float* __restrict__ scores, int T)
{
    typedef Tile<NDB, WHOLE> TL;
    __shared__ __attribute__((aligned(16))) float ks[KT * TL::PITCH];
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = pb.N, d = pb.d, P = pb.P;
    const unsigned pairs = pb.noskip ? (unsigned)(T * T) : (unsigned)(T * (T + 1) / 2), item = flat_block();
    if (item >= pairs * (unsigned)(pb.B * pb.H)) return;
    const int bh = (int)(item / pairs), pair = (int)(item - (unsigned)bh * pairs);
    int A, B;
    if (pb.noskip) {
        A = pair / T;
        B = pair - A * T;
    } else {  // pair number A (A + 1) / 2 + B, A >= B
        A = (int)((sqrtf(8.f * (float)pair + 1.f) - 1.f) * 0.5f);
        while (A * (A + 1) / 2 > pair) --A;
        while ((A + 1) * (A + 2) / 2 <= pair) ++A;
        B = pair - A * (A + 1) / 2;
    }
    const bool twice = !pb.noskip && A != B;
    const float* zh = z + (size_t)bh * N * d;
    TL tk;
    tk.fetch(zh, B * KT, N, d, tid);
    const int i = A * KT + 16 * wave + ln;
    f32x4 qf[NDB];
    load_row<NDB, WHOLE>(qf, zh + (size_t)min(i, N - 1) * d, g4, d);

    unsigned long long cnt = 0;
    {
        const int ia0 = (int)cdiv_b(A * KT, cc), ia1 = (int)cdiv_b(min((A + 1) * KT, N), cc);
        const int ib0 = (int)cdiv_b(B * KT, cc), ib1 = (int)cdiv_b(min((B + 1) * KT, N), cc);
        const int na = ia1 - ia0, nb = ib1 - ib0;
        for (int e = tid; e < na * nb; e += 256) {
            const int I = ia0 + e / nb, J = ib0 + e % nb;
            const int gd = I >= J ? I - J : I - J + P;              // (I - J) mod P
            cnt += (pb.noskip || 2 * gd <= P) ? 1u : 0u;            // region (A, B)
            const int gt = gd ? P - gd : 0;
            if (twice) cnt += (2 * gt <= P) ? 1u : 0u;              // region (B, A), filled by the mirrored store
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    const int nk = min(4, (N - B * KT + 15) >> 4);  // 16-key blocks that hold a key
    const bool rows = A * KT + 16 * wave < N;
    if (lane == 0)
        count_add(pb.counters, item * 4u + wave, cnt, rows ? (unsigned)nk : 0u);

    tk.stage(ks, B * KT, N, d, tid);
    __syncthreads();
    if (!rows) return;
    f32x4 S[4];
    score_blocks<NDB, 4>(S, ks, qf, ln, g4);  // key rows past the last are zeros and not stored
    const int SP = score_pitch(pb);
    float* Sh = scores + (size_t)bh * N * SP;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        S[b] *= pb.scale;
        const int j = B * KT + 16 * b + 4 * g4;  // the lane's four keys
        if (i < N && j + 4 <= SP) {
            *(f32x4_any*)(Sh + (size_t)i * SP + j) = S[b];
        } else if (i < N) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (j + r < SP) Sh[(size_t)i * SP + j + r] = S[b][r];
        }
        if (twice && i < N) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (j + r < N) Sh[(size_t)(j + r) * SP + i] = S[b][r];
        }
    }
}

}  // namespace

namespace {

// Rows or keys kernel.  Measured (us, rows / keys; f32, d = 64, by the number of 64-row tiles): 32 99 / 31,
// 96 30 / 21, 192 31 / 28, 320 (d = 80, masked) 49 / 41, 384 48 / 47 (masked 35 / 31), 768 77 / 93 (masked
// 48 / 53); a single key tile has no keys to share (256 row tiles 11 / 14).
template <int NDB, bool WHOLE, bool STORED>
void launch_rows(const Problem& pb, const float* q, const float* k, const float* v, const float* scores, void* out,
                 hipStream_t s)
{
    const CountCfg cc = count_cfg(pb.b);
    const bool out_whole = pb.d % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & (pb.is_bf16 ? 7 : 15)) == 0;
    const long heads = (long)pb.B * pb.H;
    const bool keys = pb.N > KT && heads * ((pb.N + 63) / 64) < 2L * 256;
    const int n_rowtiles = keys ? (pb.N + 15) / 16 : (pb.N + 63) / 64;
    const dim3 grid = flat_grid((size_t)heads * n_rowtiles);
    auto kernel = [&](auto causal) {
        constexpr bool C = decltype(causal)::value;
        if (!keys) return attn_rows_kernel<NDB, WHOLE, STORED, C>;
        return pb.d == 16 * NDB ? attn_keys_kernel<NDB, WHOLE, WHOLE, STORED, C> : attn_keys_kernel<NDB, WHOLE, false, STORED, C>;
    };
    auto* const f = !STORED && (EITHER<NDB, WHOLE> || pb.scheme == SCHEME_CAUSAL) ? kernel(std::integral_constant<bool, !STORED>{}) : kernel(std::false_type{});
    hipLaunchKernelGGL(f, grid, dim3(256), 0, s, pb, cc, q, k, v, scores, out, n_rowtiles, out_whole);
}

template <int NDB, bool WHOLE>
hipError_t launch_sym(const Problem& pb, const float* z, float* scores, void* out, hipStream_t s)
{
    const int T = (pb.N + KT - 1) / KT;
    const dim3 grid = flat_grid((size_t)(pb.noskip ? T * T : T * (T + 1) / 2) * pb.B * pb.H);
    hipLaunchKernelGGL((sym_scores_float_kernel<NDB, WHOLE>), grid, dim3(256), 0, s, pb, count_cfg(pb.b), z, scores, T);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_rows<NDB, WHOLE, true>(pb, nullptr, nullptr, z, scores, out, s);
    return hipGetLastError();
}

// f(NDB, WHOLE) for the number of 16-column blocks of d and whether rows are whole 16-byte pieces
// (the workspace is aligned).
template <class F>
hipError_t with_size(int d, F&& f)
{
    auto pick = [&](auto ndb) { return d % 4 == 0 ? f(ndb, std::true_type{}) : f(ndb, std::false_type{}); };
    const int need = (d + 15) / 16;
    if (need <= 1) return pick(std::integral_constant<int, 1>{});
    if (need <= 2) return pick(std::integral_constant<int, 2>{});
    if (need <= 3) return pick(std::integral_constant<int, 3>{});
    if (need <= 4) return pick(std::integral_constant<int, 4>{});
    if (need <= 5) return pick(std::integral_constant<int, 5>{});
    if (need <= 6) return pick(std::integral_constant<int, 6>{});
    if (need <= 8) return pick(std::integral_constant<int, 8>{});
    if (need <= 10) return pick(std::integral_constant<int, 10>{});
    if (need <= 12) return pick(std::integral_constant<int, 12>{});
    return pick(std::integral_constant<int, 16>{});
}

}  // namespace

hipError_t launch_attn_float(const Problem& pb, const float* q, const float* k, const float* v, void* out, hipStream_t s)
{
    return with_size(pb.d, [&](auto ndb, auto whole) {
        launch_rows<decltype(ndb)::value, decltype(whole)::value, false>(pb, q, k, v, nullptr, out, s);
        return hipGetLastError();
    });
}

size_t sym_float_score_floats(const Problem& pb)
{
    const int pitch = score_pitch(pb);
    return (size_t)pb.B * pb.H * pb.N * pitch + (pitch % 4 ? 3 : 0);
}

hipError_t launch_sym_float(const Problem& pb, const float* z, float* scores, void* out, hipStream_t s)
{
    return with_size(pb.d, [&](auto ndb, auto whole) {
        return launch_sym<decltype(ndb)::value, decltype(whole)::value>(pb, z, scores, out, s);
    });
}

}  // namespace attnring
