// Fused phases 1-3 (Sec. 3.1, Eq. (1)-(3)) on the 16-bit matrix cores, FULL and masked scheme, for launches
// between the small ones of attn_split.hip and those that fill the chip with attn_pipe.hip's workgroups.
//
// What bounds such a launch is the length of one wavefront's walk on a chip that is partly idle: attn_pipe.hip
// gives a CU 256 rows (d_k = 128) or 128 (d_k = 64) and every wavefront all keys of its rows.  Here the eight or twelve
// wavefronts of a workgroup are KS strands of RW: a wavefront owns 32 query rows, the wavefronts of a strand
// the RW * 32 rows of the workgroup, and strand s takes tiles s, s + KS, ... of the walk (the ring is met in KS
// strands).  Half (a quarter) of the rows per workgroup, half (a quarter) of the walk, for the same operand
// reads from LDS per pair and KS times the copies into it; the partial states (m, l, O) are merged through
// LDS at the end.  The walk itself, block by block, is that of attn_pipe.hip (attn_walk.h).
//
// Order of phases.  Wavefronts w and w + 4 share a SIMD; step t is tile t of every strand:
//     wavefronts 0..3 (and 8..11):  | E(2t)     M(2t)  E(2t+1)  M(2t+1)  | ...
//     wavefronts 4..7:              | M(2t-1)   E(2t)  M(2t)    E(2t+1)  | M(2t+1) ...
// with the workgroup barrier of step t at the bar: one side is in a vector phase while the other is in a matrix
// phase.  LDS is read in vector phases only (K of the next block, V^T of this one), so that behind barrier t every
// wavefront reads V^T of step t, K of steps t and t + 1: three ring stages of K and two of V^T, 160 KiB in all with two
// strands at d_k = 128 and four at 64, 120 with three.  Every barrier waits for all copies sent behind the one before.
//
// d_k = 128: two strands of four wavefronts (two per SIMD, 234 registers); d_k = 64: three of four (three per SIMD) or,
// where 64-row workgroups still find a CU each, four of two.  Measured against attn_pipe.hip: 3 x 1100 rows, 8 heads of 128,
// FULL 37.7 -> 31.5 us; one item of 8192 rows, 4 heads of 64, FULL 113 -> 87, of 128, masked, 165 -> 126; 4096 rows, 4 heads of
// 64 57 -> 33 (the lines: launch_attn).  With the chip full a step of d_k = 128 takes 2.0 us without its copies (as
// attn_pipe.hip's do at 256 workgroups, 1.4 at 128: the clock) and 2.4 with them: with one stage ahead their latency is
// not hidden in full.  Requests spread over the matrix phases instead of sent behind the barrier: 3.6 us.
#include <type_traits>

#include "attn_walk.h"

namespace attnring {
namespace {

template <int DK, int KS, int RW>
struct Strands : Walk<DK> {
    using Walk<DK>::K_BYTES;
    using Walk<DK>::V_BYTES;
    static constexpr int WAVES = KS * RW;                  // KS strands of RW wavefronts
    static constexpr int BR = 32 * RW;                     // rows per workgroup
    static constexpr int KPIECES = K_BYTES / 1024 / RW;    // 1 KiB copy pieces per wavefront and tile
    static constexpr int VPIECES = V_BYTES / 1024 / RW;
    static constexpr int K_STAGE = KS * K_BYTES, V_STAGE = KS * V_BYTES;
    static constexpr int NK = 3, NV = 2;
    static constexpr int V_BASE = NK * K_STAGE;
    static constexpr int PITCH = DK + 4;                   // floats per row of a partial state in LDS
    static constexpr int MERGE = KS * BR * (PITCH + 2) * 4;
    static constexpr int LDS = V_BASE + NV * V_STAGE;
    static_assert(LDS <= 160 * 1024 && MERGE <= LDS, "what a CU holds");
    static_assert(RW * 1024 / (DK * 2) % 16 == 0 && RW * 1024 / (BC * 2) % 16 == 0, "dma_lane_offset: whole periods of the swizzle");
};

template <int DK, int KS, int RW, bool CAUSAL>
__global__ __launch_bounds__(64 * KS * RW) __attribute__((amdgpu_waves_per_eu(KS * RW / 4, KS * RW / 4)))
void attn_strands_kernel(Problem pb, CountCfg cc, const h16_t* __restrict__ q, const h16_t* __restrict__ k,
                         const h16_t* __restrict__ vt, bf16_t* __restrict__ out, int row_tiles, int heads,
                         FastDiv split_d, FastDiv heads_d)
{
    typedef Strands<DK, KS, RW> T;
    constexpr int NKS = T::NKS, NDB = T::NDB, BR = T::BR;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[T::LDS];

    const int tid = threadIdx.x;
    const int lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strand = wave / RW, rw = wave % RW;
    const bool late = (wave >> 2) & 1;  // the side that starts a step with a matrix phase

    // FULL: every XCD takes a run of heads, so that the workgroups of one head share an L2.  Masked: the same where the
    // heads divide over the XCDs, its heads in turn and the heaviest row tiles first; elsewhere all heads in turn.
    int bh, I;
    if (!CAUSAL) {
        const int work = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        bh = (int)divide((unsigned)work, split_d);
        I = work - bh * (int)split_d.d;
        if (bh >= heads) return;
    } else {
        const int nh = (int)split_d.d;  // heads taken in turn: those of an XCD, or all
        const bool by_xcd = nh < heads;
        const int p = by_xcd ? blockIdx.x >> 3 : blockIdx.x;
        const int t = (int)divide((unsigned)p, split_d);
        bh = (by_xcd ? (blockIdx.x & 7) * nh : 0) + p - t * nh;
        I = row_tiles - 1 - t;
        if (I < 0) return;
    }
    const int bb = (int)divide((unsigned)bh, heads_d), h = bh - bb * pb.H;

    const int N = pb.N, Npad = pb.Npad;
    int len = N;
    if (pb.lens) { len = pb.lens[bb]; len = len < 0 ? 0 : (len > N ? N : len); }
    const int rlen = pb.skip_rows ? len : N;  // query rows at or past it take part in no pair
    const size_t out_row0 = pb.row0 ? (size_t)pb.row0[bb] : (size_t)bb * N;
    const int n_out = pb.row0 ? rlen : N;     // packed layout: rows past the item belong to the next one
    if (I * BR >= n_out) return;
    const int i0w = I * BR + rw * 32;  // first row of this wavefront
    const int i = i0w + ln;            // this lane's query row
    const bool cut_rows = rlen < i0w + 32;

    // The walk over the 64-key tiles of the head, as in attn_pipe.hip: needed tiles are 0 .. nJ-1, masked from
    // the diagonal tile down, FULL the tile cut by the key length first, then in ring order from the own tile.
    // Debug mode walks the others first, in whole steps, so that a needed tile belongs to the same strand in either
    // mode: the first strands may have no tile in step 0.
    const int nkt_all = Npad / BC;
    int nJ = (len + BC - 1) / BC;
    if (CAUSAL) nJ = min(nJ, ((I + 1) * BR + BC - 1) / BC);
    if (I * BR >= rlen && !pb.noskip) nJ = 0;
    const int n_dead = pb.noskip ? nkt_all - nJ : 0;
    const int dead_steps = (n_dead + KS - 1) / KS;
    const int has_cut = (!CAUSAL && (len % BC) != 0) ? 1 : 0;
    const int n_ring = nJ - has_cut;
    const int Jown = ((I + 1) * BR - 1) / BC;
    const int Js = CAUSAL ? nJ - 1 : (Jown < n_ring ? Jown : n_ring - 1);
    const int n_steps = dead_steps + (nJ + KS - 1) / KS;
    const int n_own = dead_steps + (nJ - strand + KS - 1) / KS;
    auto tile_of_step = [&](int t) -> int {
        const int w = KS * (t - dead_steps) + strand;
        int J = nJ - 1 - w;  // masked; FULL: the cut tile, and, w < 0, the tiles behind the needed ones, the last one first
        if (!CAUSAL && w >= has_cut) {
            J = Js - (w - has_cut);
            J += J < 0 ? n_ring : 0;
        }
        return J;  // nkt_all and more: no tile
    };
    const int NB = 2 * n_own;  // 32-key blocks of this wavefront's walk, the upper half of a tile first
    auto key_of_block = [&](int n) -> int { return tile_of_step(n >> 1) * BC + 32 * (1 - (n & 1)); };
    auto block_needed = [&](int kb) -> bool { return pb.noskip ? kb < Npad : kb < len && (!CAUSAL || kb <= i0w); };
    auto block_is_edge = [&](int kb) -> bool {
        return pb.noskip || cut_rows || kb + 32 > len || (CAUSAL && kb + 31 > i0w);
    };
    int n_first = 0;
    if (i0w >= (pb.noskip ? N : rlen)) n_first = NB;
    while (n_first < NB && !block_needed(key_of_block(n_first))) ++n_first;
    int n_edge_end = n_first;
    while (n_edge_end < NB && block_is_edge(key_of_block(n_edge_end))) ++n_edge_end;

    typename T::Row r;
#pragma unroll
    for (int db = 0; db < NDB; ++db) r.O[db] = T::zero16();
    r.S = T::zero16();
    r.Cneg = T::zero16();
    r.P[0] = r.P[1] = u32x4{0u, 0u, 0u, 0u};
    r.thr = -INFINITY;
    r.mref = 0.f;
    r.l = 0.f;

    if (n_steps > 0) {
        const size_t head = (size_t)bh * Npad * DK;
        u32x4 qf[NKS];  // rows past n: padding of the workspace
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const u32x4*)(q + head + (size_t)i * DK + ks * 16 + g * 8);

        const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(k + head), 0, -1, 0x00020000);
        const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(vt + head), 0, -1, 0x00020000);
        // A strand's wavefronts copy its tiles, RW pieces apart (attn_common.h).
        const unsigned k_lane_off = dma_lane_offset<T::KROWB>(rw, lane);
        const unsigned v_lane_off = dma_lane_offset<BC * 2>(rw, lane);
        unsigned char* const k_ring = lds + strand * T::K_BYTES;
        unsigned char* const v_ring = lds + T::V_BASE + strand * T::V_BYTES;
        int k_next = 0, v_next = 0, k_slot = 0, v_slot = 0;  // steps to be requested next, and their places in the rings
        auto request_k = [&]() {
            if (k_next < n_own) {
                const int src = min(tile_of_step(k_next), nkt_all - 1) * T::K_BYTES;
#pragma unroll
                for (int c = 0; c < T::KPIECES; ++c) {
                    unsigned char* const dst = k_ring + k_slot + (rw + c * RW) * 1024;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (__attribute__((address_space(3))) void*)dst, 16,
                                                             (int)k_lane_off, src + (rw + c * RW) * 1024, 0, 0);
                }
            }
            ++k_next;
            k_slot = k_slot + T::K_STAGE == T::V_BASE ? 0 : k_slot + T::K_STAGE;
        };
        auto request_v = [&]() {
            if (v_next < n_own) {
                const int src = min(tile_of_step(v_next), nkt_all - 1) * T::V_BYTES;
#pragma unroll
                for (int c = 0; c < T::VPIECES; ++c) {
                    unsigned char* const dst = v_ring + v_slot + (rw + c * RW) * 1024;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (__attribute__((address_space(3))) void*)dst, 16,
                                                             (int)v_lane_off, src + (rw + c * RW) * 1024, 0, 0);
                }
            }
            ++v_next;
            v_slot = v_slot + T::V_STAGE == T::NV * T::V_STAGE ? 0 : v_slot + T::V_STAGE;
        };
        // Barrier of step t: behind it K of steps t and t + 1 and V^T of step t are in LDS, and the stages of K of
        // step t - 1 and of V^T of step t - 1, which nobody reads any more, take the next requests.
        auto step_sync = [&]() {
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront's LDS reads are done
            __builtin_amdgcn_s_barrier();
            request_k();  // of step t + 2
            request_v();  // of step t + 1
        };
#pragma unroll
        for (int t = 0; t < T::NV; ++t) {
            request_k();
            if (t < T::NV - 1) request_v();
        }
        step_sync();
        int next_sync = 1;
        const int t_first = n_first >> 1;
        for (; next_sync <= t_first && next_sync < n_steps; ++next_sync) step_sync();

        if (n_first < NB) {
            typename T::Frags fr;
            int t = t_first;
            int kst = (t % T::NK) * T::K_STAGE, vst = (t % T::NV) * T::V_STAGE;
            const int koff0 = ln * T::KROWB + swz<T::KROWB>(g, ln) * 16;
            int voff[2];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) voff[hf] = ln * (BC * 2) + swz<BC * 2>(2 * hf + g, ln) * 16;
            T::read_k(fr, k_ring, kst + (1 - (n_first & 1)) * 32 * T::KROWB + koff0);
            r.S = T::scores(r, fr, qf, [](int) {});
            int lim_base = len - 1;  // the lane's last allowed key
            if (CAUSAL) lim_base = lim_base < i ? lim_base : i;
            if (i >= rlen) lim_base = -1;  // a row that is left out has no allowed key
            const bool live = lim_base >= 0;
            bool fresh = true;  // a live row may still be without a reference
            lim_base -= 4 * g;

            // E(n) of the upper or lower 32 keys of tile J, the tile of step t (see attn_pipe.hip)
            auto phase_e = [&](auto upper, bool masked, int J) {
                constexpr int UPPER = decltype(upper)::value;
                if (masked) T::mask_block(r.S, lim_base - (J * BC + 32 * UPPER));
                if (fresh) {
                    const float mxl = T::max16(r.S);
                    if (__builtin_amdgcn_ballot_w64(mxl > r.thr) != 0ull) T::raise_reference(r, mxl);
                    fresh = __builtin_amdgcn_ballot_w64(live && !(r.thr > -INFINITY)) != 0ull;
                }
                const int kst_n = kst + T::K_STAGE == T::V_BASE ? 0 : kst + T::K_STAGE;
                const unsigned ka0 = (UPPER ? kst : kst_n + 32 * T::KROWB) + koff0;
                const unsigned char* vstage = v_ring + vst;
                const int voff0 = voff[0] ^ (64 * UPPER), voff1 = voff[1] ^ (64 * UPPER);
                auto reads = [&](int p) {
                    if ((p & 1) == 0) return;
                    const int u4 = p >> 1;
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < NKS / 4; ++u) fr.kf[u4 * (NKS / 4) + u] = T::read_k1(k_ring, ka0, u4 * (NKS / 4) + u);
#pragma unroll
                    for (int u = 0; u < (2 * NDB) / 4; ++u) {
                        const int e = u4 * ((2 * NDB) / 4) + u, hf = e / NDB, db = e % NDB;
                        fr.vf[hf][db] = *(const u32x4*)(vstage + (hf ? voff1 : voff0) + db * 32 * (BC * 2));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                float bsum = T::template exponentials<false>(r, 0.f, reads);
                if (__builtin_amdgcn_ballot_w64(bsum > PIPE_SUM_LIMIT) != 0ull) {
                    const float mxl = T::max16(r.S);
                    T::raise_reference(r, mxl);
                    bsum = T::template exponentials<false>(r, 0.f, [](int) {});
                }
                r.l += bsum;
                asm volatile("" : "+v"(r.P[0]), "+v"(r.P[1]), "+v"(r.l));
            };
            auto phase_m = [&]() {
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
                r.S = T::scores(r, fr, qf, [](int) {});
                T::weighted_sum(r, fr, [](int) {});
                __builtin_amdgcn_s_setprio(0);
            };
            const std::integral_constant<int, 1> upper{};
            const std::integral_constant<int, 0> lower{};
            auto end_of_step = [&]() {  // between the two phases of a tile's lower block
                if (late && next_sync == t + 1 && next_sync < n_steps) { step_sync(); ++next_sync; }
                phase_m();
                ++t;
                kst = kst + T::K_STAGE == T::V_BASE ? 0 : kst + T::K_STAGE;
                vst = vst + T::V_STAGE == T::NV * T::V_STAGE ? 0 : vst + T::V_STAGE;
            };
            auto run_steps = [&](int t_end, bool masked) {
#pragma nounroll
                while (t < t_end) {
                    const int J = masked ? tile_of_step(t) : 0;
                    if (!late && next_sync == t) { step_sync(); ++next_sync; }
                    phase_e(upper, masked, J);
                    phase_m();
                    phase_e(lower, masked, J);
                    end_of_step();
                }
            };
            if (n_first & 1) {  // a walk that starts with the lower block of a tile
                const bool masked = n_first < n_edge_end;
                phase_e(lower, masked, masked ? tile_of_step(t) : 0);
                end_of_step();
            }
            const int t_edge_end = (n_edge_end + 1) >> 1;
            run_steps(t_edge_end < n_own ? t_edge_end : n_own, true);
            run_steps(n_own, false);
        }
        for (; next_sync < n_steps; ++next_sync) step_sync();
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();  // the partial states go where the rings were
    }

    // counts: blocks by the wavefronts that walked them, logical tiles by the first strand's
    unsigned cnt_logical = 0;
    if (strand == 0 && g == 0 && i < (pb.noskip ? N : rlen) && is_multiple(i, cc))
        cnt_logical = cdiv_b((unsigned)(pb.noskip ? N : CAUSAL ? min(len, i + 1) : len), cc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt_logical += __shfl_xor(cnt_logical, o, 64);
    if (lane == 0) count_add(pb.counters, blockIdx.x * (unsigned)T::WAVES + wave, cnt_logical, (unsigned)(NB - n_first));

    // merge: sum over the strands of 2^(m_s - M) (l_s, O_s)
    float* const st_o = (float*)lds;
    float* const st_ml = st_o + KS * BR * T::PITCH;
    {
        const float l_tot = r.l + __shfl_xor(r.l, 32, 64);
        const int row = strand * BR + rw * 32 + ln;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *(f32x4*)(st_o + row * T::PITCH + 32 * db + 8 * r4 + 4 * g) =
                    f32x4{r.O[db][4 * r4], r.O[db][4 * r4 + 1], r.O[db][4 * r4 + 2], r.O[db][4 * r4 + 3]};
        if (g == 0) {
            st_ml[2 * row] = r.thr > -INFINITY ? r.mref : -INFINITY;
            st_ml[2 * row + 1] = l_tot;
        }
    }
    __syncthreads();
    constexpr int TPR = DK / 8;  // threads per row, eight columns each
    const int c0 = (tid % TPR) * 8;
    for (int row = tid / TPR; row < BR; row += 64 * T::WAVES / TPR) {
        float ms[KS], M = -INFINITY, L = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            ms[s] = st_ml[2 * (s * BR + row)];
            M = fmaxf(M, ms[s]);
        }
        const float ref = M > -INFINITY ? M : 0.f;
        f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const float w = __builtin_amdgcn_exp2f(ms[s] - ref);
            L += w * st_ml[2 * (s * BR + row) + 1];
            y0 += w * *(const f32x4*)(st_o + (s * BR + row) * T::PITCH + c0);
            y1 += w * *(const f32x4*)(st_o + (s * BR + row) * T::PITCH + c0 + 4);
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;  // a row with no allowed pair is zero
        y0 *= inv;
        y1 *= inv;
        if (I * BR + row < n_out)
            *(u32x4_out*)(out + (out_row0 + I * BR + row) * ((size_t)pb.H * DK) + (size_t)h * DK + c0) =
                u32x4{pack_bf16(y0[0], y0[1]), pack_bf16(y0[2], y0[3]), pack_bf16(y1[0], y1[1]), pack_bf16(y1[2], y1[3])};
    }
}

}  // namespace

hipError_t launch_attn_strands(const Problem& pb, const h16_t* q, const h16_t* k, const h16_t* vt, bf16_t* out, int strands,
                               hipStream_t s)
{
    const int br = strands == 4 ? 64 : 128, row_tiles = (pb.N + br - 1) / br;
    const int heads = pb.B * pb.H;
    const dim3 grid((heads * row_tiles + 7) / 8 * 8);
    const CountCfg cc = count_cfg(pb.b);
    const bool causal = pb.scheme == SCHEME_CAUSAL;
    const FastDiv split_d = fast_div((unsigned)(!causal ? row_tiles : heads % 8 == 0 ? heads / 8 : heads));
#define ATTN_STRANDS(DK_, KS_, RW_)                                                                                      \
    do {                                                                                                                 \
        if (causal)                                                                                                      \
            hipLaunchKernelGGL((attn_strands_kernel<DK_, KS_, RW_, true>), grid, dim3(64 * KS_ * RW_), 0, s, pb, cc, q,  \
                               k, vt, out, row_tiles, heads, split_d, fast_div((unsigned)pb.H));             \
        else                                                                                                             \
            hipLaunchKernelGGL((attn_strands_kernel<DK_, KS_, RW_, false>), grid, dim3(64 * KS_ * RW_), 0, s, pb, cc, q, \
                               k, vt, out, row_tiles, heads, split_d, fast_div((unsigned)pb.H));             \
    } while (0)
    if (pb.d == 128 && strands == 2) ATTN_STRANDS(128, 2, 4);
    else if (pb.d == 64 && strands == 3) ATTN_STRANDS(64, 3, 4);
    else if (pb.d == 64 && strands == 4) ATTN_STRANDS(64, 4, 2);
    else return hipErrorInvalidValue;
#undef ATTN_STRANDS
    return hipGetLastError();
}

}  // namespace attnring
