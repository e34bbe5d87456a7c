// What a wavefront does with one 32-key block in the matrix-core attention kernels whose K and V^T
// tiles stand in LDS (attn_pipe.hip, attn_strands.hip): scores, exponentials against a lazily raised
// reference, weighted sum, and the registers they work on.
#pragma once

#include "attn_common.h"

namespace attnring {
namespace {

constexpr float PIPE_RAISE = 8.f;  // slack of the lazy reference, in base-2 exponent units
// A lane's 16 exponentials of a block add up to more than this only if one of them is above
// 2^PIPE_RAISE, and as long as they do not, none is above 2^12, far inside half precision.
constexpr float PIPE_SUM_LIMIT = 4096.f;

template <int DK>
struct Walk {
    static constexpr int NKS = DK / 16;         // k-steps of the score product
    static constexpr int NDB = DK / 32;         // 32-row blocks of O^T
    static constexpr int KROWB = DK * 2;        // bytes per key row in LDS
    static constexpr int K_BYTES = BC * KROWB;  // 8 or 16 KiB
    static constexpr int V_BYTES = DK * BC * 2;
    // Fold the reference into the score accumulator: saves a subtraction per pair, costs 16 registers
    // (168 in all for the 4-wavefront d_k = 64 kernel, just what three wavefronts per SIMD allow).
    static constexpr bool USE_CNEG = true;

    struct Row {
        f32x16 O[NDB];  // O^T, un-normalised
        f32x16 S;       // base-2 scores, minus the reference, of the block whose phase 2 comes next
        f32x16 Cneg;    // minus the reference: the C operand the score MFMAs start from
        u32x4 P[2];     // exponentials of the current block, half precision, B-operand layout
        float thr;      // RAISE once the row has a reference, -inf before
        float mref;     // the reference (0 before the row has one)
        float l;        // this lane's part of the row sum
    };
    struct Frags {
        u32x4 kf[NKS];     // K of block n+1
        u32x4 vf[2][NDB];  // V^T of block n: keys 0..15 and 16..31 of the block
    };

    static __device__ __forceinline__ f32x16 zero16()
    {
        f32x16 z;
#pragma unroll
        for (int e = 0; e < 16; ++e) z[e] = 0.f;
        return z;
    }
    static __device__ __forceinline__ float max16(const f32x16& S)
    {
        float m0 = fmaxf(fmaxf(S[0], S[1]), S[2]), m1 = fmaxf(fmaxf(S[3], S[4]), S[5]);
        float m2 = fmaxf(fmaxf(S[6], S[7]), S[8]), m3 = fmaxf(fmaxf(S[9], S[10]), S[11]);
        float m4 = fmaxf(fmaxf(S[12], S[13]), S[14]);
        m0 = fmaxf(fmaxf(m0, m1), m2);
        m3 = fmaxf(fmaxf(m3, m4), S[15]);
        return fmaxf(m0, m3);
    }
    // Pair test of an edge block: key kb + acc_row(e, g) against the lane's last allowed key.
    static __device__ __forceinline__ void mask_block(f32x16& S, int lim)
    {
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = (8 * (e >> 2) + (e & 3)) <= lim ? S[e] : -INFINITY;
    }
    // The chunk of k-step ks is chunk 2*ks + g XOR-ed with row bits, and 2*ks has no bit in
    // common with g: the lane's byte address for k-step ks is its address for k-step 0 XOR 32*ks
    // (32-key blocks start at multiples of 256 bytes).  ka0: LDS byte offset for k-step 0.
    static __device__ __forceinline__ u32x4 read_k1(const unsigned char* lds, unsigned ka0, int ks)
    {
        return *(const u32x4*)(lds + (ka0 ^ (unsigned)(32 * ks)));
    }
    static __device__ __forceinline__ void read_k(Frags& fr, const unsigned char* lds, unsigned ka0)
    {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) fr.kf[ks] = read_k1(lds, ka0, ks);
    }
    // Phase 1 (Eq. (1)) of one block from the K fragments in fr; the accumulator starts at minus
    // the row's reference, so the result is the exponent phase 2 needs.
    // `between(m)` runs behind MFMA m of the phase (a copy request, or nothing).
    template <class F>
    static __device__ __forceinline__ f32x16 scores(const Row& r, const Frags& fr, const u32x4 (&qf)[NKS], F&& between)
    {
        f32x16 S;
        if constexpr (USE_CNEG) {
            // D and C in different registers: written with the builtin, the compiler copies the 16
            // registers of C first and accumulates in place.
            asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %3" : "=&v"(S) : "v"(fr.kf[0]), "v"(qf[0]), "v"(r.Cneg));
        } else {
            S = mfma32h(fr.kf[0], qf[0], zero16());
        }
        between(0);
#pragma unroll
        for (int ks = 1; ks < NKS; ++ks) {
            S = mfma32h(fr.kf[ks], qf[ks], S);
            between(ks);
        }
        return S;
    }
    // Phase 3 (Eq. (3)) of one block from the V^T fragments in fr and the row's exponentials.
    template <class F>
    static __device__ __forceinline__ void weighted_sum(Row& r, const Frags& fr, F&& between)
    {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                r.O[db] = mfma32h(fr.vf[hf][db], r.P[hf], r.O[db]);
                between(NKS + hf * NDB + db);
            }
    }

    // A score beyond the slack (or the first finite score of a row): move the reference to the
    // row's largest score and rescale what the row has accumulated.  Returns what the reference
    // went up by; the scores at hand were computed against the old reference.
    static __device__ __forceinline__ float raise_reference(Row& r, float mxl)
    {
        asm volatile("" ::: "memory");  // keeps this rare path a branch of its own
        const float mx = fmaxf(mxl, __shfl_xor(mxl, 32, 64));  // both halves of a row agree
        const bool raise = mx > r.thr;
        const bool started = r.thr > -INFINITY;
        const float delta = raise ? mx : 0.f;
        const float alpha = (raise && started) ? __builtin_amdgcn_exp2f(-delta) : 1.f;
        r.mref = raise ? r.mref + delta : r.mref;
        r.thr = raise ? PIPE_RAISE : r.thr;
        r.l *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) r.O[db][e] *= alpha;
        if (USE_CNEG) {
            // the scores at hand were taken against the old reference
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                r.Cneg[e] = -r.mref;
                r.S[e] -= delta;
            }
        }
        return delta;
    }

    // Phase 2 (Eq. (2)) of the block in r.S; the row sum is normalised at the very end.
    // SHIFT: the scores still refer to a reference that was `delta` lower.
    // `between(p)` runs behind score pair p (0..7): the LDS requests for the matrix phase.
    // Returns the sum of the lane's 16 exponentials, which the caller adds to r.l.
    template <bool SHIFT, class F>
    static __device__ __forceinline__ float exponentials(Row& r, float delta, F&& between)
    {
        // The row sum is taken with plain additions of the unrounded exponentials.  A v_dot2c on
        // the rounded pairs would be half the instructions, but dot instructions do not run beside
        // the matrix pipe: each one waits until the MFMAs in flight on its SIMD have drained, from
        // whichever wavefront they are, which serialises the vector phase with the matrix phase
        // of the wavefront it shares the SIMD with (measured: an MFMA followed by one v_dot2c
        // takes 51 cycles instead of 32; exponentials, conversions, max and fma add 1-3).
        float psum0 = 0.f, psum1 = 0.f;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float s0 = r.S[8 * hf + 2 * w], s1 = r.S[8 * hf + 2 * w + 1];
                const float p0 = __builtin_amdgcn_exp2f(SHIFT ? s0 - delta : s0);
                const float p1 = __builtin_amdgcn_exp2f(SHIFT ? s1 - delta : s1);
                r.P[hf][w] = pack_f16(p0, p1);
                psum0 += p0;
                psum1 += p1;
                between(4 * hf + w);
            }
        return psum0 + psum1;
    }
};

}  // namespace
}  // namespace attnring
