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
// A wavefront owns 16 query rows.  Two ways to share the work of a workgroup's four wavefronts:
//   rows  64 rows per workgroup, every wavefront walks all keys of the tile;
//   keys  16 rows per workgroup, wavefront w takes the 16-key block w of every tile and the four
//         partial states (m, l, O) are merged at the end: four times the workgroups, for launches
//         that would leave CUs idle, for four times the reads of K and V (from L2).
// The paper's ring: the walk starts at the rows' own tile and runs downwards, wrapping (the order
// in which PE l meets block (l - j) mod m in Algorithm 1); tiles and, inside a tile, 16-key blocks
// with no needed pair are left out (Sec. 5.1).
#include "attn_common.h"

namespace attnring {
namespace {

constexpr int KT = 64;  // keys per tile

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

template <int NDB, bool KEYS, bool WHOLE>
__global__ __launch_bounds__(256)
void attn_float_kernel(Problem pb, CountCfg cc, const float* __restrict__ q, const float* __restrict__ k,
                       const float* __restrict__ v, void* __restrict__ out, int n_rowtiles, bool out_whole)
{
    typedef Tile<NDB, WHOLE> TL;
    constexpr int PITCH = TL::PITCH, DP = TL::DP;
    constexpr int ROWS = KEYS ? 16 : 64;  // query rows per workgroup
    constexpr int NB = KEYS ? 1 : 4;      // 16-key blocks of a tile that a wavefront takes
    __shared__ __attribute__((aligned(16))) float ks[KT * PITCH];
    __shared__ __attribute__((aligned(16))) float vs[KT * PITCH];

    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Consecutive workgroups take the heads in turn, the last row tiles (the most keys under the
    // mask) first, so that the long walks do not start last.
    const int heads = pb.B * pb.H;
    const int bh = blockIdx.x % heads;
    const int x = n_rowtiles - 1 - blockIdx.x / heads;
    const int bb = bh / pb.H, h = bh - bb * pb.H;
    const int N = pb.N, d = pb.d;
    const bool causal = pb.scheme == SCHEME_CAUSAL;
    int len = N;
    if (pb.lens) { len = pb.lens[bb]; len = len < 0 ? 0 : (len > N ? N : len); }
    const int rlen = pb.skip_rows ? len : N;  // query rows at or past it take part in no pair
    const size_t head = (size_t)bh * N * d;
    const int i0 = x * ROWS;                       // rows of the workgroup
    const int i0w = KEYS ? i0 : i0 + 16 * wave;    // rows of the wavefront
    const int i = i0w + ln;                        // the lane's query row
    const int row_end = min(pb.noskip ? N : rlen, i0 + ROWS);       // rows that take part
    const int wave_end = min(pb.noskip ? N : rlen, i0w + 16);

    // needed tiles are 0 .. nJ-1, met from the own one downwards, wrapping; in debug mode the
    // others follow and change nothing
    const int n_all = (N + KT - 1) / KT;
    int nJ = 0;
    if (row_end > i0) {
        nJ = (len + KT - 1) / KT;
        if (causal) nJ = min(nJ, (row_end - 1) / KT + 1);
    }
    const int nT = pb.noskip && row_end > i0 ? n_all : nJ;
    const int Js = min((i0 + ROWS - 1) / KT, nJ - 1);
    auto tile_of_step = [&](int t) -> int {
        if (t >= nJ) return t;
        const int J = Js - t;
        return J < 0 ? J + nJ : J;
    };

    // logical tiles: row block I is counted by the workgroup that holds its first row
    if (wave == 0) {
        unsigned cnt = 0;
        const int I = (int)cdiv_b((unsigned)i0, cc) + lane;  // at most 64 row blocks start here
        if (I * cc.b < row_end) {
            cnt = (unsigned)pb.P;
            if (!pb.noskip) {
                if (causal) cnt = min(cnt, (unsigned)I + 1u);
                cnt = min(cnt, cdiv_b((unsigned)len, cc));
            }
        }
        unsigned long long total = cnt;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
        if (lane == 0) count_add(pb.counters, blockIdx.x, total, 0);
    }
    unsigned cnt_phys = 0;  // 16 x 16 score blocks; wave-uniform

    f32x4 qf[NDB], O[NDB];
    load_row<NDB, WHOLE>(qf, q + head + (size_t)min(i, N - 1) * d, g4, d);  // rows past the last: not stored
#pragma unroll
    for (int db = 0; db < NDB; ++db) O[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;  // running maximum of the row; this lane's part of the row sum
    int lim = len - 1;             // the row's last allowed key
    if (causal) lim = min(lim, i);
    if (i >= rlen) lim = -1;

    TL tk, tv;
    if (nT > 0) {
        const int J = tile_of_step(0);
        tk.fetch(k + head, J * KT, len, d, tid);
        tv.fetch(v + head, J * KT, len, d, tid);
    }
    for (int t = 0; t < nT; ++t) {
        const int J = tile_of_step(t);
        __syncthreads();  // everyone is done with the tile before
        tk.stage(ks, J * KT, len, d, tid);
        tv.stage(vs, J * KT, len, d, tid);
        __syncthreads();
        if (t + 1 < nT) {
            const int Jn = tile_of_step(t + 1);
            tk.fetch(k + head, Jn * KT, len, d, tid);
            tv.fetch(v + head, Jn * KT, len, d, tid);
        }
        // 16-key blocks of the tile that hold a pair this wavefront needs: the first nk
        const int key0 = J * KT + (KEYS ? 16 * wave : 0);
        int nk = 0;
        if (wave_end > i0w) {
            int keys = len - key0;
            if (causal) keys = min(keys, wave_end - key0);
            nk = pb.noskip ? NB : max(0, min(NB, (keys + 15) >> 4));
        }
        if (nk == 0) continue;
        cnt_phys += (unsigned)nk;
        f32x4 S[NB];
        const float* kt = ks + (KEYS ? 16 * wave * PITCH : 0);
        if (nk == NB) {
            score_blocks<NDB, NB>(S, kt, qf, ln, g4);
        } else {
            for (int b = 0; b < NB; ++b) {
                f32x4 s1[1] = {{0.f, 0.f, 0.f, 0.f}};
                if (b < nk) score_blocks<NDB, 1>(s1, kt + 16 * b * PITCH, qf, ln, g4);
                // written out: S stays in registers
                if (b == 0) S[0] = s1[0];
                if constexpr (NB == 4) {
                    if (b == 1) S[1] = s1[0];
                    if (b == 2) S[2] = s1[0];
                    if (b == 3) S[3] = s1[0];
                }
            }
        }
        // phase 2 (Eq. (2)), running maximum; a row that has met no allowed key keeps m = -inf
        float mx = m;
        const int rel = lim - key0 - 4 * g4;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[b][r] = 16 * b + r <= rel ? S[b][r] * pb.scale : -INFINITY;
                mx = fmaxf(mx, S[b][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float ref = mx > -INFINITY ? mx : 0.f;
        const float alpha = exp_neg(m - ref);
        m = mx;
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                S[b][r] = exp_neg(S[b][r] - ref);
                sum += S[b][r];
            }
        l = l * alpha + sum;
#pragma unroll
        for (int db = 0; db < NDB; ++db) O[db] *= alpha;
        // phase 3 (Eq. (3))
        const float* vt = vs + ((KEYS ? 16 * wave : 0) + 4 * g4) * PITCH + ln;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= nk) break;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int db = 0; db < NDB; ++db) O[db] = mfma16f(vt[(16 * b + r) * PITCH + 16 * db], S[b][r], O[db]);
        }
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);

    const size_t pitch = (size_t)pb.H * d;
    const size_t base = ((size_t)bb * N + i0) * pitch + (size_t)h * d;
    if constexpr (KEYS) {
        // partial state of wavefront w, row r: m, l, then O
        __syncthreads();
        float* st_o = ks;  // [4][16] rows of PITCH
        float* st_ml = vs;
#pragma unroll
        for (int db = 0; db < NDB; ++db) *(f32x4*)(st_o + (16 * wave + ln) * PITCH + 16 * db + 4 * g4) = O[db];
        if (g4 == 0) {
            st_ml[2 * (16 * wave + ln)] = m;
            st_ml[2 * (16 * wave + ln) + 1] = l;
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
        const float inv = L > 0.f ? 1.f / L : 0.f;  // a row with no allowed pair is zero
        if (i0 + r < N)
            for (int c = tid & 15; c < DP / 4; c += 16) {
                f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) y += mw[w] * *(const f32x4*)(st_o + (16 * w + r) * PITCH + 4 * c);
                store4(out, base + (size_t)r * pitch, 4 * c, d, y * inv, pb.is_bf16, out_whole);
            }
    } else {
        const float inv = l > 0.f ? 1.f / l : 0.f;
        if (i < N)
#pragma unroll
            for (int db = 0; db < NDB; ++db)
                store4(out, base + (size_t)(i - i0) * pitch, 16 * db + 4 * g4, d, O[db] * inv, pb.is_bf16, out_whole);
    }
    if (lane == 0) count_add(pb.counters, blockIdx.x, 0, cnt_phys);
}

}  // namespace

hipError_t launch_attn_float(const Problem& pb, const float* q, const float* k, const float* v, void* out, hipStream_t s)
{
    const CountCfg cc = count_cfg(pb.b);
    const bool whole = pb.d % 4 == 0;  // the workspace is aligned
    const bool out_whole = whole && (reinterpret_cast<uintptr_t>(out) & (pb.is_bf16 ? 7 : 15)) == 0;
    const long heads = (long)pb.B * pb.H;
    // Measured (us, rows / keys): 320 workgroups of 64 rows 55 / 46, 384 56 / 54 (masked 41 / 35), 768 85 / 105
    // (masked 54 / 61); a single tile has no keys to share (256 workgroups 11 / 15).
    const bool keys = pb.N > KT && heads * ((pb.N + 63) / 64) < 2L * 256;
    const int n_rowtiles = keys ? (pb.N + 15) / 16 : (pb.N + 63) / 64;
    const dim3 grid((unsigned)(heads * n_rowtiles));
#define ATTN_FLOAT_LAUNCH(NDB_, K_, W_)                                                                                  \
    hipLaunchKernelGGL((attn_float_kernel<NDB_, K_, W_>), grid, dim3(256), 0, s, pb, cc, q, k, v, out, n_rowtiles, out_whole)
#define ATTN_FLOAT(NDB_)                                                                                               \
    if (whole) { if (keys) ATTN_FLOAT_LAUNCH(NDB_, true, true); else ATTN_FLOAT_LAUNCH(NDB_, false, true); }            \
    else { if (keys) ATTN_FLOAT_LAUNCH(NDB_, true, false); else ATTN_FLOAT_LAUNCH(NDB_, false, false); }
    const int need = (pb.d + 15) / 16;
    if (need <= 1) { ATTN_FLOAT(1); }
    else if (need <= 2) { ATTN_FLOAT(2); }
    else if (need <= 3) { ATTN_FLOAT(3); }
    else if (need <= 4) { ATTN_FLOAT(4); }
    else if (need <= 5) { ATTN_FLOAT(5); }
    else if (need <= 6) { ATTN_FLOAT(6); }
    else if (need <= 8) { ATTN_FLOAT(8); }
    else if (need <= 10) { ATTN_FLOAT(10); }
    else if (need <= 12) { ATTN_FLOAT(12); }
    else { ATTN_FLOAT(16); }
#undef ATTN_FLOAT
#undef ATTN_FLOAT_LAUNCH
    return hipGetLastError();
}

}  // namespace attnring
