// Float path, for every shape the 16-bit matrix-core kernels do not take (f32 storage, head sizes
// other than 64 and 128, unaligned pointers): the projections, and the q = k = v scheme.  The
// attention kernel of the FULL and masked schemes is in attn_float.hip.
#include <type_traits>

#include "mfma_common.h"

namespace attnring {
namespace {

__device__ __forceinline__ float load_as_float(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_as_float(const bf16_t* p, size_t i)
{
    return __uint_as_float(((unsigned)p[i]) << 16);
}
__device__ __forceinline__ void store_from_float(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_from_float(bf16_t* p, size_t i, float v)
{
    unsigned u = __float_as_uint(v);
    u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (inputs are finite)
    p[i] = (bf16_t)(u >> 16);
}

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
    return x;
}
__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// ---------------------------------------------------------------------------
// Projections (Sec. 3.1): out_m[b][h][i][l] = sum_c X[b][i][c] * W_m[c][h*d + l], for up to three
// weight matrices in one launch, any d_model, any number of columns, any alignment.
//
// Bound by the matrix cores: float operands are contracted by v_mfma_f32_32x32x2_f32 (one fp32
// fma per product, as an fmaf loop; 157 TFLOP/s on the chip, a large torch product reaches 153),
// bfloat16 operands by v_mfma_f32_32x32x16_bf16 (products exact in float).  An MFMA of 64 (32)
// cycles leaves room for its operand reads, so tiles are small, 64 x 64, a 32 x 32 block for each
// of 2 x 2 wavefronts: several workgroups share a CU and fill each other's waits, and small
// products leave fewer CUs idle (4096 x 768 -> 2304 in f32: 136 us, 128 x 128 tiles 171; 1024 x 768
// -> 768: 23 against 65).  Slices of k are fetched into registers three ahead, past the end of
// d_model too, so that the wait for one leaves the others in flight, and pass through two LDS
// buffers with one barrier each.
//
// X rows lie k-contiguous in LDS and are read 16 bytes at a time; the k a lane half contracts in
// one float MFMA are chosen to suit that read (half g takes 8t + 4g + j in MFMA j), which only
// orders the sum.  W stays k-major: float columns are read one by one, bfloat16 ones by the
// transposing read.  Row pitches put the rows that one read touches on different banks.
// ---------------------------------------------------------------------------
template <typename T>
struct Slice;
template <>
struct Slice<float> {
    static constexpr int KS = 32;              // k per slice
    static constexpr int VEC = 4;              // elements of a 16-byte piece
    static constexpr int APITCH = KS + 4;      // elements of an X row in LDS
    static constexpr int bpitch(int bn) { return bn + 8; }
};
template <>
struct Slice<bf16_t> {
    static constexpr int KS = 64;
    static constexpr int VEC = 8;
    static constexpr int APITCH = KS + 8;
    static constexpr int bpitch(int bn) { return bn + 32; }
};

struct ProjArgs {
    const void* W[3];
    float* out[3];
};

// 16 bytes at element `col` of a row of `count` elements, zeros past its end (and if not `there`).
// No branch: what must not be read is read at the row's start instead; a load behind a branch would
// wait for all loads in flight.  WHOLE: pieces are aligned and lie inside or outside, and what is to
// be dropped is dropped by clip_piece when the piece is used, since that waits for the load.
template <typename T, bool WHOLE>
__device__ __forceinline__ u32x4 load_piece(const T* __restrict__ row, int col, int count, bool there)
{
    constexpr int VEC = Slice<T>::VEC;
    u32x4 v = {0u, 0u, 0u, 0u};
    if constexpr (WHOLE) {
        v = *(const u32x4*)(row + (col < count ? col : 0));
    } else {
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const bool in = col + j < count;
            const T w = row[in ? col + j : 0];
            if constexpr (sizeof(T) == 4) v[j] = there && in ? __float_as_uint(w) : 0u;
            else v[j >> 1] |= there && in ? (unsigned)w << (16 * (j & 1)) : 0u;
        }
    }
    return v;
}

template <bool WHOLE>
__device__ __forceinline__ u32x4 clip_piece(u32x4 v, bool in)
{
    if constexpr (WHOLE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = in ? v[j] : 0u;
    }
    return v;
}

template <typename T, bool WHOLE>
__global__ __launch_bounds__(256) void proj_float_kernel(int M, int N, int D, int H, int d, const T* __restrict__ X,
                                                         ProjArgs pa, int tiles_n)
{
    typedef Slice<T> SL;
    constexpr int BM = 64, BN = 64, KS = SL::KS, VEC = SL::VEC;
    constexpr int AP = SL::APITCH, BP = SL::bpitch(BN);
    constexpr int ACH = KS / VEC, BCH = BN / VEC;             // 16-byte pieces per row
    constexpr int NAL = BM * ACH / 256, NBL = KS * BCH / 256;  // pieces per thread
    constexpr int PF = 3;  // slices fetched ahead, a set of registers each
    __shared__ __attribute__((aligned(16))) T As2[2][BM * AP];
    __shared__ __attribute__((aligned(16))) T Bs2[2][KS * BP];
    const int HD = H * d;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int which = blockIdx.x / tiles_n;
    const int col0 = (blockIdx.x - which * tiles_n) * BN, row0 = blockIdx.y * BM;
    const T* __restrict__ W = (const T*)pa.W[which];

    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;

    u32x4 areg[PF][NAL], breg[PF][NBL];
    auto fetch = [&](int k0, auto set_) {
        constexpr int SET = decltype(set_)::value;
#pragma unroll
        for (int u = 0; u < NAL; ++u) {
            const int c = tid + 256 * u, r = c / ACH, kk = k0 + (c % ACH) * VEC;
            // rows past the last are the last again: they are not stored
            areg[SET][u] = load_piece<T, WHOLE>(X + (size_t)min(row0 + r, M - 1) * D, kk, D, true);
        }
#pragma unroll
        for (int u = 0; u < NBL; ++u) {
            const int c = tid + 256 * u, kk = k0 + c / BCH, cc = col0 + (c % BCH) * VEC;
            breg[SET][u] = load_piece<T, WHOLE>(W + (size_t)min(kk, D - 1) * HD, cc, HD, kk < D);
        }
    };
    // Slice k0 goes from its register set to LDS buffer `buf`, which was last read two slices ago,
    // on the other side of the barrier of the slice in between.
    auto slice = [&](int k0, int buf, auto set_) {
        constexpr int SET = decltype(set_)::value;
        T* As = As2[buf];
        T* Bs = Bs2[buf];
#pragma unroll
        for (int u = 0; u < NAL; ++u) {
            const int c = tid + 256 * u;
            *(u32x4*)(As + (c / ACH) * AP + (c % ACH) * VEC) = clip_piece<WHOLE>(areg[SET][u], k0 + (c % ACH) * VEC < D);
        }
#pragma unroll
        for (int u = 0; u < NBL; ++u) {
            const int c = tid + 256 * u;
            *(u32x4*)(Bs + (c / BCH) * BP + (c % BCH) * VEC) = clip_piece<WHOLE>(breg[SET][u], k0 + c / BCH < D);
        }
        fetch(k0 + PF * KS, set_);  // unconditional (past d_model: dropped), so that waits can count the loads in flight
        __syncthreads();
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int t = 0; t < KS / 8; ++t) {
                const f32x4 af = *(const f32x4*)(As + (wm + ln) * AP + 8 * t + 4 * g);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[j], Bs[(8 * t + 4 * g + j) * BP + wn + ln], acc, 0, 0, 0);
            }
        } else {
            // transposing read: 16 lanes hand in a 4 (k) x 16 (columns) patch, lane i gets column i
            const int i16 = lane & 15;
            const int kr = 8 * g + (i16 >> 2), cb = wn + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
#pragma unroll
            for (int ks = 0; ks < KS / 16; ++ks) {
                const u32x4 af = *(const u32x4*)(As + (wm + ln) * AP + 16 * ks + 8 * g);
                const u32x2 lo = lds_read_tr16(Bs + (16 * ks + kr) * BP + cb);
                const u32x2 hi = lds_read_tr16(Bs + (16 * ks + kr + 4) * BP + cb);
                acc = mfma32(af, u32x4{lo[0], lo[1], hi[0], hi[1]}, acc);
            }
        }
    };
    fetch(0, std::integral_constant<int, 0>{});
    fetch(KS, std::integral_constant<int, 1>{});
    fetch(2 * KS, std::integral_constant<int, 2>{});
    for (int k0 = 0, buf = 0;; k0 += PF * KS, buf ^= 1) {
        slice(k0, buf, std::integral_constant<int, 0>{});
        if (k0 + KS >= D) break;
        slice(k0 + KS, buf ^ 1, std::integral_constant<int, 1>{});
        if (k0 + 2 * KS >= D) break;
        slice(k0 + 2 * KS, buf, std::integral_constant<int, 2>{});
        if (k0 + 3 * KS >= D) break;
    }
    // register r: vector acc_row(r, g), column ln; 32 lanes write 128 consecutive bytes
    float* __restrict__ out = pa.out[which];
    const int gc = col0 + wn + ln;
    if (gc >= HD) return;
    const int h = gc / d, l = gc - h * d;
    const int first = row0 + wm;
    const int b0 = first / N, edge = (b0 + 1) * N;  // most blocks lie in one batch item
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int gr = first + acc_row(e, g);
        if (gr >= M) continue;
        const int bb = gr < edge ? b0 : gr / N;
        out[(((size_t)bb * H + h) * N + (gr - bb * N)) * d + l] = acc[e];
    }
}

// z = x split into heads, for the q = k = v scheme without a projection matrix.
template <typename T>
__global__ void copy_heads_kernel(int total, int N, int H, int d, const T* __restrict__ X, float* __restrict__ out)
{
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    int l = e % d, t = e / d;
    int h = t % H, bi = t / H;  // bi = b*N + i
    int bb = bi / N, i = bi - bb * N;
    out[(((size_t)bb * H + h) * N + i) * d + l] = load_as_float(X, (size_t)e);
}

// ---------------------------------------------------------------------------
// Online row state of phases 2 and 3 (Eq. (2), Eq. (3)) for one query row held
// by one wavefront: running maximum m, running sum l of exp(s - m), and the
// un-normalised output o (lane L holds columns L, L+64, ...).
// ---------------------------------------------------------------------------
enum { MAX_ACC = 4 };  // d_k <= 256

struct RowState {
    float m, l;
    float o[MAX_ACC];
};

// Fold up to 64 keys (one per lane) into the row state.  `s` is the lane's score,
// `ok` whether its pair takes part; keys jbase .. jbase+cnt-1 of head `vh`.
__device__ __forceinline__ void fold_chunk(RowState& st, float s, bool ok, int jbase, int cnt,
                                           const float* __restrict__ vh, int d, int lane)
{
    s = ok ? s : -INFINITY;
    const float m_new = fmaxf(st.m, wave_max(s));
    if (m_new == -INFINITY) return;  // nothing allowed so far (uniform over the wave)
    const float alpha = expf(st.m - m_new);
    const float p = ok ? expf(s - m_new) : 0.f;
    st.l = st.l * alpha + wave_sum(p);
    st.m = m_new;
#pragma unroll
    for (int a = 0; a < MAX_ACC; ++a) st.o[a] *= alpha;
    for (int jj = 0; jj < cnt; ++jj) {
        const float pj = __shfl(p, jj, 64);
        const float* vr = vh + (size_t)(jbase + jj) * d;
#pragma unroll
        for (int a = 0; a < MAX_ACC; ++a) {
            int col = lane + 64 * a;
            if (col < d) st.o[a] = fmaf(pj, vr[col], st.o[a]);
        }
    }
}

template <typename T>
__device__ __forceinline__ void store_row(const RowState& st, T* out, size_t base, int d, int lane)
{
    const float inv = st.l > 0.f ? 1.f / st.l : 0.f;  // a row with no allowed pair is zero
#pragma unroll
    for (int a = 0; a < MAX_ACC; ++a) {
        int col = lane + 64 * a;
        if (col < d) store_from_float(out, base + col, st.o[a] * inv);
    }
}

// ---------------------------------------------------------------------------
// q = k = v scheme (Sec. 4).  Phase 1 on tiles: PE I computes the tiles on the
// circulant tile diagonals (I - J) mod P = 0 .. floor(P/2) (Sec. 4.2 applied to
// the P x P tile matrix; for even P the middle diagonal is computed by both of
// its owners, the paper's balance trade-off) and stores each score also at its
// mirrored position, which is the reuse of w'_ij as w'_ji (Eq. (4)).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void sym_scores_kernel(Problem pb, const float* __restrict__ z,
                                                         float* __restrict__ scores)
{
    const int I = blockIdx.x, h = blockIdx.y, bb = blockIdx.z;
    const int N = pb.N, d = pb.d, b = pb.b, P = pb.P;
    const size_t bh = (size_t)bb * pb.H + h;
    const float* zh = z + bh * (size_t)N * d;
    float* S = scores + bh * (size_t)N * N;
    const int gmax = pb.noskip ? P - 1 : P / 2;
    for (int g = 0; g <= gmax; ++g) {
        int J = I - g; if (J < 0) J += P;
        const bool mirror = !pb.noskip && g != 0 && !(P % 2 == 0 && g == P / 2);
        for (int e = threadIdx.x; e < b * b; e += 256) {
            const int i = I * b + e / b, j = J * b + e % b;
            const float* zi = zh + (size_t)i * d;
            const float* zj = zh + (size_t)j * d;
            float s = 0.f;
            for (int l = 0; l < d; ++l) s = fmaf(zi[l], zj[l], s);
            s *= pb.scale;
            S[(size_t)i * N + j] = s;
            if (mirror) S[(size_t)j * N + i] = s;
        }
    }
    if (threadIdx.x == 0) {
        count_add(pb.counters, (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x,
                  (unsigned long long)(gmax + 1), (unsigned long long)(gmax + 1));
    }
}

// Phases 2 and 3 of the q = k = v scheme: unchanged from the original definition
// (Sec. 4.1), reading the stored scores.  One wavefront per row.
template <typename T>
__global__ __launch_bounds__(256) void sym_softmax_pv_kernel(Problem pb, const float* __restrict__ z,
                                                             const float* __restrict__ scores, T* __restrict__ out)
{
    const int h = blockIdx.y, bb = blockIdx.z;
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int N = pb.N, d = pb.d;
    if (i >= N) return;
    const size_t bh = (size_t)bb * pb.H + h;
    const float* vh = z + bh * (size_t)N * d;
    const float* Srow = scores + bh * (size_t)N * N + (size_t)i * N;
    RowState st;
    st.m = -INFINITY; st.l = 0.f;
#pragma unroll
    for (int a = 0; a < MAX_ACC; ++a) st.o[a] = 0.f;
    for (int j0 = 0; j0 < N; j0 += 64) {
        const int cnt = (N - j0) < 64 ? (N - j0) : 64;
        const bool valid = lane < cnt;
        const float s = valid ? Srow[j0 + lane] : 0.f;
        fold_chunk(st, s, valid, j0, cnt, vh, d, lane);
    }
    store_row(st, out, ((size_t)bb * N + i) * ((size_t)pb.H * d) + (size_t)h * d, d, lane);
}

}  // namespace

namespace {

template <typename T>
void launch_proj_type(const Problem& pb, const T* X, const ProjArgs& pa, int count, hipStream_t s)
{
    const int M = pb.B * pb.N, HD = pb.H * pb.d;
    const int tiles_n = (HD + 63) / 64;
    uintptr_t bits = reinterpret_cast<uintptr_t>(X);
    for (int m = 0; m < count; ++m) bits |= reinterpret_cast<uintptr_t>(pa.W[m]);
    const bool whole = pb.D % Slice<T>::VEC == 0 && HD % Slice<T>::VEC == 0 && (bits & 15) == 0;
    const dim3 grid(tiles_n * count, (M + 63) / 64);
    if (whole) hipLaunchKernelGGL((proj_float_kernel<T, true>), grid, dim3(256), 0, s, M, pb.N, pb.D, pb.H, pb.d, X, pa, tiles_n);
    else hipLaunchKernelGGL((proj_float_kernel<T, false>), grid, dim3(256), 0, s, M, pb.N, pb.D, pb.H, pb.d, X, pa, tiles_n);
}

}  // namespace

hipError_t launch_proj_generic(const Problem& pb, const void* X, const void* const* W, float* const* out, int count,
                               hipStream_t s)
{
    ProjArgs pa = {};
    for (int m = 0; m < count; ++m) {
        pa.W[m] = W[m];
        pa.out[m] = out[m];
    }
    if (pb.is_bf16) launch_proj_type(pb, (const bf16_t*)X, pa, count, s);
    else launch_proj_type(pb, (const float*)X, pa, count, s);
    return hipGetLastError();
}

hipError_t launch_copy_heads_generic(const Problem& pb, const void* X, float* out, hipStream_t s)
{
    const int total = pb.B * pb.N * pb.H * pb.d;
    dim3 grid((total + 255) / 256);
    if (pb.is_bf16)
        hipLaunchKernelGGL(copy_heads_kernel<bf16_t>, grid, dim3(256), 0, s, total, pb.N, pb.H, pb.d,
                           (const bf16_t*)X, out);
    else
        hipLaunchKernelGGL(copy_heads_kernel<float>, grid, dim3(256), 0, s, total, pb.N, pb.H, pb.d,
                           (const float*)X, out);
    return hipGetLastError();
}

hipError_t launch_sym_generic(const Problem& pb, const float* z, float* scores, void* out, hipStream_t s)
{
    hipLaunchKernelGGL(sym_scores_kernel, dim3(pb.P, pb.H, pb.B), dim3(256), 0, s, pb, z, scores);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 grid((pb.N + 3) / 4, pb.H, pb.B);
    if (pb.is_bf16)
        hipLaunchKernelGGL(sym_softmax_pv_kernel<bf16_t>, grid, dim3(256), 0, s, pb, z, scores, (bf16_t*)out);
    else
        hipLaunchKernelGGL(sym_softmax_pv_kernel<float>, grid, dim3(256), 0, s, pb, z, scores, (float*)out);
    return hipGetLastError();
}

}  // namespace attnring
