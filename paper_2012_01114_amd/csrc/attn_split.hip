// Fused phases 1-3 (Sec. 3.1, Eq. (1)-(3)) on the 16-bit matrix cores for launches that are too
// small to fill the chip with attn_pipe.hip's workgroups, FULL and masked scheme, the same operands
// and layouts.
//
// What bounds such a launch is the length of one wavefront's walk: 128 rows of a 512-vector item are
// 16 blocks of 32 keys, 0.4 us each (d_k = 64) whatever else the chip does, on as many CUs as there
// are row tiles.  Here a workgroup owns 32 query rows and its wavefronts share the keys: wavefront w
// takes the 32-key blocks w, w + 4, ... (the ring is met in four strands), straight from memory (L2)
// into operand registers, the next block's operands on their way while one is worked on, no barrier;
// the four partial states (m, l, O) are merged through LDS at the end.  Four times the row tiles, a
// quarter of the walk, for four times the reads of K and V per row: the larger kernels, which pass them
// through LDS, stay ahead where their workgroups fill the CUs (launch_attn in this file draws the line).
//
// Blocks with no needed pair are left out (Sec. 5.1); pair by pair masking only in blocks cut by the
// diagonal or the key length.  Scores are computed transposed (S^T = K.Q^T), so that a lane holds 16
// keys of ONE query and its exponentials are in B-operand layout for O^T += V^T.P^T.  The softmax
// reference is the running maximum of the wavefront's strand; q arrives pre-multiplied by
// scale*log2(e), so exponentials are v_exp_f32 of a difference.
#include "attn_common.h"

namespace attnring {
namespace {

template <int DK, bool CAUSAL>
__global__ __launch_bounds__(256, 2)
void attn_split_kernel(Problem pb, CountCfg cc, FastDiv heads_all, FastDiv heads_d, const h16_t* __restrict__ q,
                       const h16_t* __restrict__ k, const h16_t* __restrict__ vt, bf16_t* __restrict__ out, int n_rowtiles)
{
    constexpr int NKS = DK / 16, NDB = DK / 32, PITCH = DK + 4;
    __shared__ __attribute__((aligned(16))) float st_o[4 * 32 * PITCH];
    __shared__ float st_ml[2 * 4 * 32];

    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the heads in turn, the last row tiles (the most keys under the mask) first
    const int t = (int)divide(blockIdx.x, heads_all);
    const int bh = (int)blockIdx.x - t * (int)heads_all.d;
    const int bb = (int)divide((unsigned)bh, heads_d), h = bh - bb * pb.H;
    const int N = pb.N, Npad = pb.Npad;
    int len = N;
    if (pb.lens) { len = pb.lens[bb]; len = len < 0 ? 0 : (len > N ? N : len); }
    const int rlen = pb.skip_rows ? len : N;  // query rows at or past it take part in no pair
    const size_t out_row0 = pb.row0 ? (size_t)pb.row0[bb] : (size_t)bb * N;
    const int n_out = pb.row0 ? rlen : N;     // packed layout: rows past the item belong to the next one
    const int i0 = (n_rowtiles - 1 - t) * 32, i = i0 + ln;
    if (i0 >= n_out) return;

    // blocks 0 .. nb-1 hold a needed pair; in debug mode the others follow and change nothing
    const int row_end = min(pb.noskip ? N : rlen, i0 + 32);
    int nb = 0;
    if (row_end > i0) {
        nb = (len + 31) >> 5;
        if (CAUSAL) nb = min(nb, (row_end + 31) >> 5);
        if (pb.noskip) nb = (N + 31) >> 5;
    }
    const size_t head = (size_t)bh * Npad * DK;
    const h16_t* kh = k + head;
    const h16_t* vh = vt + head;

    // Operands of 32-key block b: K rows 32b + ln, and rows of V^T (columns of v) over its keys.
    struct Block {
        u32x4 k[NKS], v[2][NDB];
    };
    auto load = [&](Block& x, int b) {
        const h16_t* kr = kh + (size_t)(32 * b + ln) * DK + 8 * g;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) x.k[ks] = *(const u32x4*)(kr + 16 * ks);
        const h16_t* vr = vh + ((size_t)(b >> 1) * DK + ln) * 64 + 32 * (b & 1) + 8 * g;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int db = 0; db < NDB; ++db) x.v[hf][db] = *(const u32x4*)(vr + db * 32 * 64 + 16 * hf);
    };
    u32x4 qf[NKS];
    f32x16 O[NDB];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[db][e] = 0.f;
    int lim = CAUSAL ? min(len - 1, i) : len - 1;  // the row's last allowed key, less the lane's first of a block
    if (i >= rlen) lim = -1;
    lim -= 4 * g;

    auto step = [&](const Block& x, int b) {
        f32x16 S;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) S = mfma32h(x.k[ks], qf[ks], S);
        if (pb.noskip || 32 * b + 32 > len || rlen < i0 + 32 || (CAUSAL && 32 * b + 31 > i0)) {
            const int rel = lim - 32 * b;
#pragma unroll
            for (int e = 0; e < 16; ++e) S[e] = 8 * (e >> 2) + (e & 3) <= rel ? S[e] : -INFINITY;
        }
        float mx = fmaxf(m, S[0]);
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float ref = mx > -INFINITY ? mx : 0.f;  // a row that has met no allowed key keeps m = -inf
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        m = mx;
        u32x4 P[2];
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float p0 = __builtin_amdgcn_exp2f(S[8 * hf + 2 * w] - ref);
                const float p1 = __builtin_amdgcn_exp2f(S[8 * hf + 2 * w + 1] - ref);
                P[hf][w] = pack_f16(p0, p1);
                s0 += p0;
                s1 += p1;
            }
        l = l * alpha + (s0 + s1);
#pragma unroll
        for (int db = 0; db < NDB; ++db) O[db] *= alpha;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int db = 0; db < NDB; ++db) O[db] = mfma32h(x.v[hf][db], P[hf], O[db]);
    };
    unsigned cnt_phys = 0;
    if (wave < nb) {
        Block x0, x1;
        int b = wave;
        const h16_t* qr = q + head + (size_t)i * DK + 8 * g;  // rows past n: padding of the workspace
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const u32x4*)(qr + 16 * ks);
        load(x0, b);
        cnt_phys = (unsigned)((nb - b + 3) >> 2);
        while (true) {
            // past the last block its operands once more, which nobody uses; the requests stay in front
            load(x1, b + 4 < nb ? b + 4 : b);
            __builtin_amdgcn_sched_barrier(0);
            step(x0, b);
            __builtin_amdgcn_sched_barrier(0);
            b += 4;
            if (b >= nb) break;
            load(x0, b + 4 < nb ? b + 4 : b);
            __builtin_amdgcn_sched_barrier(0);
            step(x1, b);
            __builtin_amdgcn_sched_barrier(0);
            b += 4;
            if (b >= nb) break;
        }
    }
    // counts: a row block is counted by the workgroup that holds its first row
    if (wave == 0 && nb > 0) {
        unsigned cnt = 0;
        if (g == 0 && i < row_end && is_multiple(i, cc))
            cnt = cdiv_b((unsigned)(pb.noskip ? N : CAUSAL ? min(len, i + 1) : len), cc);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
        if (lane == 0) count_add(pb.counters, blockIdx.x * 4u, cnt, 0);
    }
    if (lane == 0) count_add(pb.counters, blockIdx.x * 4u + wave, 0, cnt_phys);

    // merge: sum over the strands of 2^(m_w - M) (l_w, O_w)
    l += __shfl_xor(l, 32, 64);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *(f32x4*)(st_o + (32 * wave + ln) * PITCH + 32 * db + 8 * r4 + 4 * g) =
                f32x4{O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
    if (g == 0) {
        st_ml[2 * (32 * wave + ln)] = m;
        st_ml[2 * (32 * wave + ln) + 1] = l;
    }
    __syncthreads();
    const int r = tid >> 3, c0 = (tid & 7) * 8;  // eight threads per row, eight columns each per turn
    float mw[4], M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        mw[w] = st_ml[2 * (32 * w + r)];
        M = fmaxf(M, mw[w]);
    }
    const float ref = M > -INFINITY ? M : 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        mw[w] = __builtin_amdgcn_exp2f(mw[w] - ref);
        L += mw[w] * st_ml[2 * (32 * w + r) + 1];
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;  // a row with no allowed pair is zero
    if (i0 + r < n_out) {
        bf16_t* o = out + (out_row0 + i0 + r) * ((size_t)pb.H * DK) + (size_t)h * DK;
#pragma unroll
        for (int u = 0; u < DK / 64; ++u) {
            const int c = c0 + 64 * u;
            f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                y0 += mw[w] * *(const f32x4*)(st_o + (32 * w + r) * PITCH + c);
                y1 += mw[w] * *(const f32x4*)(st_o + (32 * w + r) * PITCH + c + 4);
            }
            y0 *= inv;
            y1 *= inv;
            *(u32x2*)(o + c) = u32x2{pack_bf16(y0[0], y0[1]), pack_bf16(y0[2], y0[3])};
            *(u32x2*)(o + c + 4) = u32x2{pack_bf16(y1[0], y1[1]), pack_bf16(y1[2], y1[3])};
        }
    }
}

hipError_t launch_attn_split(const Problem& pb, const h16_t* q, const h16_t* k, const h16_t* vt, bf16_t* out, hipStream_t s)
{
    const int heads = pb.B * pb.H, n_rowtiles = (pb.N + 31) / 32;
    const CountCfg cc = count_cfg(pb.b);
    const dim3 grid(heads * n_rowtiles);
    const FastDiv ha = fast_div((unsigned)heads), hd = fast_div((unsigned)pb.H);
    const bool causal = pb.scheme == SCHEME_CAUSAL;
#define ATTN_SPLIT(DK_, C_) \
    hipLaunchKernelGGL((attn_split_kernel<DK_, C_>), grid, dim3(256), 0, s, pb, cc, ha, hd, q, k, vt, out, n_rowtiles)
    if (pb.d == 64) { if (causal) ATTN_SPLIT(64, true); else ATTN_SPLIT(64, false); }
    else if (pb.d == 128) { if (causal) ATTN_SPLIT(128, true); else ATTN_SPLIT(128, false); }
    else return hipErrorInvalidValue;
#undef ATTN_SPLIT
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn(const Problem& pb, const h16_t* q, const h16_t* k, const h16_t* vt, bf16_t* out, int asked_waves,
                       hipStream_t s, const bf16_t* X, const bf16_t* Wq)
{
    const bool fuse = X != nullptr && Wq != nullptr;
    // Measured (us, one kernel; W: 128-row tiles of all heads; split: attn_split, 2 3 4: attn_strands with so many strands).
    //   d_k = 64, FULL           n 32 W 272 pipe 7.7 split 6.6    n 256 W 64 pipe 10.5 split 8.3 4: 9.4    W 128 10.7 / 11.6 / 9.8
    //     n 512 W 64 13.4 / 10.1 / 10.7    W 256 pipe 14.9 3: 14.7    n 1024 W 64 20.1 / 13.6 / 13.3    W 128 19.6 / 22.2 / 13.8
    //     W 256 pipe 21.0 3: 19.3    n 4096 W 64 54.6 / 34.9 / 28.8    W 128 55 / 64 / 30    W 256 pipe 56 3: 46    n 1024 W 288
    //     pipe 24.7 3: 31.8 (a second round of one workgroup per CU; pipe has three)
    //   d_k = 64, masked         n 128 W 128 pipe 10.1 split 9.1 4: 9.0    n 256 W 128 11.7 / 10.6 / 9.8    n 512 W 160 pipe 14.9 3: 13.9
    //     n 1024 W 288 pipe 21.9 3: 19.9    W 384 22.2 / 24.2    n 2048 W 256 pipe 32.2 3: 26.1 4: 24.3    W 512 35.2 / 33.5    W 640
    //     37.8 / 45.3    n 8192 W 384 103 / 76
    //   d_k = 128, FULL          n 192 W 64 pipe 14.0 split 11.8 2: 13.2    W 128 14.4 / 18.0 / 13.5    n 512 W 256 pipe 22.1 2: 20.2
    //     n 1024 W 128 30.4 / 39.3 / 24.6    n 4096 W 256 pipe 89 2: 78    W 288 n 1024 32 / 47
    //   d_k = 128, masked        n 100 W 128 pipe 13.4 2: 12.2    n 512 W 320 24.7 / 24.0    n 1024 W 512 40.6 / 35.8    W 640 47.8 / 48.9
    //     n 4096 W 512 99.7 / 84.3    W 768 117 / 129
    if (asked_waves == 0 && !fuse) {
        const int n = pb.N;
        const bool masked = pb.scheme == SCHEME_CAUSAL;
        const long heads = (long)pb.B * pb.H;
        const long w32 = heads * ((n + 31) / 32), w64 = heads * ((n + 63) / 64), w128 = heads * ((n + 127) / 128);
        bool split = w32 <= (n <= 32 ? 640 : 256);
        int strands = 0;
        if (pb.d == 64) {
            split = split && n < 1024;
            // masked, beyond 256 tiles of 32 rows: up to 128 vectors, or, where items differ in length and padded rows are left
            // out, some more (lengths uniform in n / 32 .. n, split / 4: 48 items of 232 9.1 / 9.3, 32 of 300 9.4 / 10.0, of 500
            // 12.8 / 11.0).  Key lengths with every query row produced: the walks that the split shortens are short already.
            split = split || (masked && (pb.lens && pb.skip_rows ? n <= 320 && w32 <= (n <= 128 ? 512 : 400)
                                                                  : n <= 128 && w32 <= (pb.lens ? 384 : 512)));
            if ((w64 <= 256 && n > 64) || (masked && n >= 2048 && w128 <= 256)) strands = 4;
            else if (w128 <= 256 && n > (masked ? 256 : 512)) strands = 3;
            else if (masked && w128 <= (n >= 2048 ? 512 : n >= 1024 ? 288 : 0)) strands = 3;
        } else {
            if (w128 <= 256 && n > (masked ? 64 : 128)) strands = 2;
            else if (masked && w128 <= (n >= 1024 ? 512 : n >= 512 ? 320 : 0)) strands = 2;
        }
        if (split) return launch_attn_split(pb, q, k, vt, out, s);
        if (strands) return launch_attn_strands(pb, q, k, vt, out, strands, s);
    }
    // d_k = 64: 128-row workgroups of 4 wavefronts, three of them per CU; d_k = 128: 256 rows, 8 wavefronts
    const int waves = pb.d == 128 ? 8 : asked_waves == 8 ? 8 : 4;
    return launch_attn_pipe(pb, q, k, vt, out, waves, s, X, Wq);
}

}  // namespace attnring
