// Phases 1-3 (Sec. 3.1, Eq. (1)-(3)) in float arithmetic, for every shape the 16-bit matrix-core
// kernels do not take (f32 storage, head sizes other than 64 and 128, unaligned pointers, and the q = k = v scheme
// on them) and that neither attn_planes.hip (larger f32 calls) nor proj_attn_small.hip (small ones, which walk their
// one tile by attn_rows.h as well) takes.  q, k, v: float [B][H][N][d], d <= 256.
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
#include "attn_rows.h"

namespace attnring {
namespace {

template <int NDB, bool WHOLE, bool STORED, bool CAUSAL>
__global__ __launch_bounds__(256, NDB <= 4 ? 3 : NDB <= 8 ? 2 : 1)
void attn_rows_kernel(Problem pb, CountCfg cc, const float* __restrict__ q, const float* __restrict__ k,
                      const float* __restrict__ v, const float* __restrict__ scores, void* __restrict__ out,
                      int n_rowtiles, bool out_whole)
{
    typedef Tile<NDB, WHOLE> TL;
    __shared__ __attribute__((aligned(16))) float ks[STORED ? 4 : KT * TL::PITCH];
    __shared__ __attribute__((aligned(16))) float vs[KT * TL::PITCH];
    const RowTile rt(pb, KT, n_rowtiles);
    if (!rt.there) return;
    const int lane = threadIdx.x & 63;
    if (!STORED && threadIdx.x < 64) rt.count(pb, cc, lane);
    const unsigned cnt_phys = rows_walk<NDB, WHOLE, STORED, CAUSAL>(
        pb, rt, FloatRows::head(pb, q, rt.bh), FloatRows::head(pb, k, rt.bh), FloatRows::head(pb, v, rt.bh), scores, out, out_whole, ks, vs);
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
    if constexpr (!STORED) load_row<NDB, WHOLE>(qf, FloatRows{q + head, d}, min(i, N - 1), g4);
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

    if constexpr (!STORED) cut.add(row, FloatRows{vh, d}, last_allowed, ln, g4);

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
    tk.fetch(FloatRows{zh, d}, B * KT, N, tid);
    const int i = A * KT + 16 * wave + ln;
    f32x4 qf[NDB];
    load_row<NDB, WHOLE>(qf, FloatRows{zh, d}, min(i, N - 1), g4);

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
