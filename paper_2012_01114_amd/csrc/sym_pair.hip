// The q = k = v scheme (Sec. 4) on the matrix cores, with the reuse kept on chip.
//
// Eq. (4): with one set of vectors z in all three roles, w'_ij = w'_ji, so phase 1 needs one
// element of every symmetric pair; phases 2 and 3 do not share it (Sec. 4.1).  Here the unit of
// reuse is a 128 x 128 score tile.  S_AB = z_A . z_B^T is computed once with MFMAs and used twice:
//     as it stands      for the rows of A against the keys of B   (phases 2 and 3 of row block A)
//     transposed        for the rows of B against the keys of A   (phases 2 and 3 of row block B)
// A workgroup owns row tile A and meets a run of its partners A, A + 1, .. (mod T = n/128; every
// unordered pair of tiles has one owner, a circulant choice).  The first use adds to sums it keeps in
// registers over the whole run, the second yields a partial row state (m, l, O) of B over the 128 keys
// of A; a second kernel merges the states of a row block.  The scores never leave the chip; what does
// is 128 (d + 2) floats per second use and per run.  Tiles on the diagonal (A == B) are used once.
//
// Both uses take their exponentials from the accumulators: the reference of a row is 8 (base 2) below its own
// score |z_i|^2 (among the row's largest: s_ij <= |z_i| |z_j|), so no maximum is searched for, and a row has one
// reference in every workgroup.  The own score comes from the MFMAs that form the scores, in their order of sums,
// and is rounded as they are, so that a row's own weight is the same exactly in all of them, whatever its size (a
// sum of squares of another order misses a score of 1e9 by hundreds).  A score that exceeds the reference by 15.5
// makes a weight near the end of half precision, and then the reference is set 8 below the largest score of the
// tile (first use: before the exponentials are taken; second: they are taken again).
//
// The 8 keep weights down to 2^-22 of the own one at all bits of half precision and to 2^-33 off zero: the others
// of vectors from N(0, 1) lie around 2^-12 of it at d_k = 64 and 2^-16 at 128.  A model in 64 bits of the roundings
// between z and out (n 200 .. 16384, z of rms 0.3 .. 1.4) has errors of 1.0 to 1.4 times those of a maximum per tile
// with sums of unrounded weights where either is above 1e-6 (out rounds by 1.7e-3); 5 to 380 times without the 8 at
// rms 1.2 to 1.4 and n 8192 and more.
// The exponentials of the second use are stored to LDS in half precision, [row of A][row of B], and
// read back as operands by the transposing read.  Row sums are MFMAs with ones: float sums of the weights
// as rounded (what multiplies V is what is summed), the same for either use.
//
// What bounds it: exponentials (16 cycles per 64 pairs and use) and the partial states.  96 heads of
// 512 at d_k = 64, us (pairs, merge): 30.9, 10.3 with a workgroup per pair of tiles, scores staged in fp32,
// maxima and a state per use, 22.2, 7.3 so; 32 heads of 2048 159 -> 93 together, 8 heads of 2048 at d_k = 128
// 97 -> 62.  Of that the barriers that leave memory alone gave 4, addresses recomputed per tile (no spills) 4.
// One vector in 50 four times as long as the others, so that many tiles raise a reference: 8 heads of 2048,
// whole calls, 43 -> 48 us.
//
// The paper's selection rule (Sec. 4.2: circulant diagonals 0 .. floor(P/2) of the P x P matrix of
// (n/P)-row tiles, the middle one computed by both owners when P is even) fixes WHICH element of a
// pair a ring of P processing elements computes.  On 128-row tiles every unordered pair of tiles
// is simply computed once; the count of logical tiles the rule selects is taken on the device over
// the regions the kernel covers (each position of the P x P matrix lies in exactly one use).
//
// Both operands of the score MFMAs are the same half-precision z (the scale is applied to the
// fp32 scores), so S_AB and S_BA^T are equal bit for bit, as Eq. (4) has it; with every tile
// computed in its own orientation instead (the debug mode) the outputs are the same bits.
#include <type_traits>

#include "attn_common.h"

namespace attnring {
namespace {

constexpr int ST = 128;           // rows and keys of a score tile

// Byte offset of the weight of (row of A, row of B) in LDS: rows of 256 bytes, their 16-byte chunks XOR-ed with four bits
// of the row: 16 rows of one 8-byte store meet all banks, and the four rows of a transposing read four pairs of chunks.
__device__ __forceinline__ int weight_at(int row, int col)
{
    const int f = ((row & 7) << 1) | ((row >> 3) & 1);
    return row * 256 + (((col >> 3) ^ f) << 4) + ((col & 7) << 1);
}

template <int DK>
struct Sym {
    static constexpr int NKS = DK / 16, NDB = DK / 32;
    static constexpr int KROWB = DK * 2;             // bytes of a key row in LDS
    static constexpr int K_BYTES = ST * KROWB;       // K tile: 128 keys
    static constexpr int V_BYTES = 2 * DK * 64 * 2;  // V^T of 128 keys, two 64-key blocks
    static constexpr int W_BYTES = ST * ST * 2;      // the weights of the second use, in the place of the K tile
    // d_k = 64: V^T of A stays, and the next tiles wait in registers.  d_k = 128: V^T of A takes the place of that of B, and
    // nothing waits (256 registers).  Two workgroups per CU either way.
    static constexpr bool RESIDENT = DK == 64;
    static constexpr int KW_BYTES = K_BYTES > W_BYTES ? K_BYTES : W_BYTES;
    static constexpr int LDS_BYTES = KW_BYTES + (RESIDENT ? 2 : 1) * V_BYTES;
};

// z rows [row0, row0 + 128) of one head as a K tile: rows of KROWB bytes, 16-byte chunks swizzled.
template <int DK>
struct KTile {
    static constexpr int CPR = DK / 8, PER = ST * CPR / 256;
    u32x4 reg[PER];
    __device__ __forceinline__ void fetch(const h16_t* kh, int row0, int tid)
    {
        const u32x4* src = (const u32x4*)(kh + (size_t)row0 * DK);
#pragma unroll
        for (int u = 0; u < PER; ++u) reg[u] = src[tid + 256 * u];
    }
    __device__ __forceinline__ void stage(unsigned char* dst, int tid) const
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int c = tid + 256 * u, row = c / CPR, p = c % CPR;
            *(u32x4*)(dst + row * (DK * 2) + swz<DK * 2>(p, row) * 16) = reg[u];
        }
    }
};
// V^T of the same rows: two 64-key blocks of [DK][64], rows of 128 bytes, chunks swizzled; through
// registers, so that the request can go out long before the tile in LDS is free.
template <int DK>
struct VtTile {
    static constexpr int PER = 2 * DK * 8 / 256;
    u32x4 reg[PER];
    __device__ __forceinline__ void fetch(const h16_t* vth, int row0, int tid)
    {
        const u32x4* src = (const u32x4*)(vth + (size_t)(row0 >> 6) * DK * 64);
#pragma unroll
        for (int u = 0; u < PER; ++u) reg[u] = src[tid + 256 * u];
    }
    __device__ __forceinline__ void stage(unsigned char* dst, int tid) const
    {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int c = tid + 256 * u, row = c >> 3, p = c & 7;  // row: block * DK + column of v
            *(u32x4*)(dst + row * 128 + swz<128>(p, row % DK) * 16) = reg[u];
        }
    }
};

// A workgroup barrier that orders LDS only: __syncthreads would also wait for the tiles on their way from memory and for
// the stores of states, 1 to 2 us each.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Score of row ln with itself out of the product of 32 rows with themselves, in the lanes whose half holds it: register
// 4 (ln / 8) + ln % 4 of half (ln / 4) % 2 (acc_row).
__device__ __forceinline__ bool holds_diagonal(int ln, int g) { return ((ln >> 2) & 1) == g; }
__device__ __forceinline__ float diagonal(const f32x16& D, int ln)
{
    // by masks: written as conditions, each choice becomes an element with a number known at run time, 16 comparisons
    auto pick = [](float a, float b, int bit) {  // b where the bit is set
        const unsigned m = 0u - (unsigned)bit;
        return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, b) & m) | (__builtin_bit_cast(unsigned, a) & ~m));
    };
    const int b0 = ln & 1, b1 = (ln >> 1) & 1, b3 = (ln >> 3) & 1, b4 = (ln >> 4) & 1;
    float x[4];
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) x[r4] = pick(pick(D[4 * r4], D[4 * r4 + 1], b0), pick(D[4 * r4 + 2], D[4 * r4 + 3], b0), b1);
    return pick(pick(x[0], x[1], b3), pick(x[2], x[3], b3), b4);
}

// V^T of one 16-key group, group 2 kb + hf of the 128 keys in LDS at vt, as operands.
template <int DK>
__device__ __forceinline__ void read_group(u32x4 (&vf)[DK / 32], const unsigned char* vt, int kb, int hf, int ln, int g)
{
#pragma unroll
    for (int db = 0; db < DK / 32; ++db) {
        const int row = db * 32 + ln;
        const int chunk = swz<128>(2 * hf + g, row) ^ (4 * (kb & 1));
        vf[db] = *(const u32x4*)(vt + (kb >> 1) * (DK * 128) + row * 128 + chunk * 16);
    }
}
// Ones for the keys of such a group that are there, `keys` of the 128, zeros for the others (whose rows of V^T are zeros, and
// whose weights are finite).
__device__ __forceinline__ u32x4 ones_of_group(int keys, int kb, int hf, int g)
{
    constexpr unsigned ONES = 0x3C003C00u;
    u32x4 ones = {ONES, ONES, ONES, ONES};
    if (keys < ST)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int left = keys - (kb * 32 + acc_row(8 * hf + 2 * w, g));
            ones[w] = left > 1 ? ONES : left == 1 ? ONES & 0xFFFFu : 0u;
        }
    return ones;
}
// O += V^T.P^T and l += 1.P^T (Eq. (3), (2)) of such a group.
template <int DK>
__device__ __forceinline__ void add_group(f32x16 (&O)[DK / 32], f32x16& l, u32x4 P, const u32x4 (&vf)[DK / 32], u32x4 ones)
{
    l = mfma32h(ones, P, l);
#pragma unroll
    for (int db = 0; db < DK / 32; ++db) O[db] = mfma32h(vf[db], P, O[db]);
}

__device__ __forceinline__ unsigned max_f16(unsigned a, unsigned b)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b)));
}
// A score further above its row's reference raises it: no weight is above 2^15.5 then, and half precision holds them all.
constexpr float RAISE = 15.5f;
constexpr float BELOW = 8.f;
// A row's reference by the score at hand.  From 2^26 on scores are 8 and more apart, and a step of 8 could become one of 16.
__device__ __forceinline__ float reference(float score) { return score < 0x1p26f ? score - BELOW : score; }
// Whether one of two weights (not negative) is 2^15 or more: only then scores are compared with RAISE.
__device__ __forceinline__ bool near_the_end(unsigned m) { return (m & 0xFFFFu) >= 0x7800u || m >= 0x78000000u; }

template <int DK>
__device__ __forceinline__ void store_state(const f32x16 (&O)[DK / 32], float m, float l, int g, float* __restrict__ pm,
                                            float* __restrict__ pl, float* __restrict__ po)
{
    if (g == 0) { *pm = m; *pl = l; }
#pragma unroll
    for (int db = 0; db < DK / 32; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *(f32x4*)(po + db * 32 + 8 * r4 + 4 * g) = f32x4{O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
}

// Partners of row tile A that it owns: A .. A + owned(A, T) - 1 (mod T).
__device__ __forceinline__ int owned(int A, int T) { return (T + 1) / 2 + (T % 2 == 0 && A < T / 2 ? 1 : 0); }

// Work items: (head, row tile, run of `run` partners), runs in turn.  all_ordered: every ordered pair of tiles computed in
// its own orientation, nothing reused (the debug mode): the runs are followed by the tiles of other owners, one by one.
template <int DK>
__global__ __launch_bounds__(256, 2) void sym_pair_kernel(Problem pb, CountCfg cc, const h16_t* __restrict__ z,
                                                          const h16_t* __restrict__ zt, float* __restrict__ part_m,
                                                          float* __restrict__ part_l, float* __restrict__ part_o,
                                                          bf16_t* __restrict__ out, int T, int runs, int run, bool all_ordered, float c2, int heads)
{
#pragma clang fp contract(off)  // scores are rounded before references are taken from them
    typedef Sym<DK> Y;
    constexpr int NKS = Y::NKS, NDB = Y::NDB;
    __shared__ __attribute__((aligned(16))) unsigned char lds[Y::LDS_BYTES];
    __shared__ __attribute__((aligned(16))) float ref_b[ST];
    __shared__ float high_b[ST];
    __shared__ unsigned raised, raised_rows[ST / 32];
    unsigned char* const kt = lds;  // K tile of B, then the weights
    unsigned char* const vt = lds + Y::KW_BYTES;
    unsigned char* const vt_a = Y::RESIDENT ? vt + Y::V_BYTES : vt;

    const int tid0 = threadIdx.x, tid = tid0, lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Where the heads divide over the XCDs an XCD has whole heads; the row tiles with the most partners first.
    const int nh = heads % 8 == 0 ? heads / 8 : heads, p = heads % 8 == 0 ? blockIdx.x >> 3 : blockIdx.x;
    const int item = p / nh, bh = (heads % 8 == 0 ? (blockIdx.x & 7) * nh : 0) + p - item * nh;
    const int A = item / runs, turn = item - A * runs;
    if (A >= T) return;
    const int mine = owned(A, T), own_runs = all_ordered ? runs - T : runs;
    int j0 = turn * run, j1 = min(j0 + run, mine);
    if (all_ordered && turn >= own_runs) {
        j0 = mine + turn - own_runs;
        j1 = min(j0 + 1, T);
    }
    if (j0 >= j1) return;

    const int N = pb.N, Npad = pb.Npad;
    const h16_t* zh = z + (size_t)bh * Npad * DK;
    const h16_t* zth = zt + (size_t)bh * Npad * DK;
    auto partner = [&](int j) { return A + j < T ? A + j : A + j - T; };

    KTile<DK> kr;
    VtTile<DK> vr;
    const int ia = A * ST + wave * 32 + ln;  // this lane's row of A
    u32x4 qf[NKS];
    auto fetch_q = [&](int at) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const u32x4*)(zh + at + ks * 16);
    };
    fetch_q(ia * DK + g * 8);
    kr.fetch(zh, partner(j0) * ST, tid);
    vr.fetch(zth, partner(j0) * ST, tid);
    f32x16 O[NDB], l;
#pragma unroll
    for (int e = 0; e < 16; ++e) l[e] = 0.f;
    auto own_scores = [&]() __attribute__((always_inline)) {  // behind the requests of the tiles
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) l = mfma32h(qf[ks], qf[ks], l);
    };
    if constexpr (Y::RESIDENT) {
        VtTile<DK> va;
        va.fetch(zth, A * ST, tid);
        own_scores();
        va.stage(vt_a, tid);
    } else {
        own_scores();
    }
    kr.stage(kt, tid);
    vr.stage(vt, tid);
    if (tid == 0) raised = 0u;
    float ref = reference(diagonal(l, ln) * c2);
    const float other = __shfl_xor(ref, 32, 64);
    if (!holds_diagonal(ln, g)) ref = other;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        l[e] = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db) O[db][e] = 0.f;
    }
    unsigned long long cnt = 0;
    unsigned phys = 0;

#pragma nounroll
    for (int j = j0; j < j1; ++j) {
        // Addresses that depend on the thread only, from an opaque copy of its number: else they are kept over the loop, more
        // of them than there are registers.
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, ln = lane & 31, g = lane >> 5;
        const int B = partner(j);
        const bool twice = !all_ordered && j > 0;
        const int keys_left = N - B * ST;
        if constexpr (!Y::RESIDENT) {  // not kept over a tile: the registers are wanted
            int at = ia * DK + g * 8;
            asm volatile("" : "+v"(at));
            fetch_q(at);
        }
        lds_barrier();  // the tiles of B are there
        if (twice) {      // references of the rows of B, as a wavefront takes those of its own rows
            const int row = wave * 32 + ln;
            f32x16 own;
#pragma unroll
            for (int e = 0; e < 16; ++e) own[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const u32x4 f = *(const u32x4*)(kt + row * Y::KROWB + swz<Y::KROWB>(2 * ks + g, row) * 16);
                own = mfma32h(f, f, own);
            }
            const float x = reference(diagonal(own, ln) * c2);
            if (holds_diagonal(ln, g)) ref_b[row] = high_b[row] = x;
        }
        // ---- phase 1 (Eq. (1)), once: S^T = z_B . z_A^T, the wavefront's 32 rows of A against 128 keys of B ----
        f32x16 S[4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) S[kb][e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                if (kb == 0) __builtin_amdgcn_sched_barrier(0);
                const int row = kb * 32 + ln;
                S[kb] = mfma32h(*(const u32x4*)(kt + row * Y::KROWB + swz<Y::KROWB>(2 * ks + g, row) * 16), qf[ks], S[kb]);
            }
        // scale and base-2 exponent, rounded here once: a product and difference in one step would leave as much of a score as
        // the rounding of its reference has taken away, 2^64 and more at 1e9
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) S[kb][e] *= c2;
        // ---- counts: logical tiles the selection rule picks, over the regions of this tile, and 32 x 32 score blocks
        // issued: the key blocks that hold a key, for a wavefront that holds a row ----
        {
            const int ia0 = (int)cdiv_b(A * ST, cc), ia1 = (int)cdiv_b(min((A + 1) * ST, N), cc);
            const int ib0 = (int)cdiv_b(B * ST, cc), ib1 = (int)cdiv_b(min((B + 1) * ST, N), cc);
            const int na = ia1 - ia0, nb = ib1 - ib0, P = pb.P;
            for (int e = tid; e < na * nb; e += 256) {
                const int I = ia0 + e / nb, J = ib0 + e % nb;
                const int gd = I >= J ? I - J : I - J + P, gt = I > J ? J - I + P : J - I;
                cnt += (all_ordered || 2 * gd <= P) ? 1u : 0u;          // region (A, B)
                if (twice) cnt += (2 * gt <= P) ? 1u : 0u;              // region (B, A), met transposed
            }
            if (A * ST + wave * 32 < N) phys += (unsigned)min(4, (keys_left + 31) / 32);
        }
        lds_barrier();  // nobody reads the K tile any more; the references are there
        if (j + 1 < j1 && Y::RESIDENT) {
            kr.fetch(zh, partner(j + 1) * ST, tid);
            vr.fetch(zth, partner(j + 1) * ST, tid);
        } else if (!Y::RESIDENT && twice) {
            vr.fetch(zth, A * ST, tid);
        }
        // ---- weights of the second use: rows of B against keys of A ----
        auto store_group = [&](int kb, int r4) __attribute__((always_inline)) -> unsigned {  // the largest, in either half
            const f32x4 rb = *(const f32x4*)(ref_b + kb * 32 + 8 * r4 + 4 * g);
            float p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(S[kb][4 * r4 + e] - rb[e]);
            const u32x2 w = {pack_f16(p[0], p[1]), pack_f16(p[2], p[3])};
            *(u32x2*)(kt + weight_at(wave * 32 + ln, kb * 32 + 8 * r4 + 4 * g)) = w;
            return max_f16(w[0], w[1]);
        };
        if (twice) {
            unsigned most = 0u;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    if ((r4 & 1) == 0) __builtin_amdgcn_sched_barrier(0);
                    most = max_f16(most, store_group(kb, r4));
                }
            if (__builtin_amdgcn_ballot_w64(near_the_end(most)) != 0ull && lane == 0) raised = 1u;
        }
        // ---- first use: phases 2 and 3 of the rows of A over the keys of B ----
        {
            float most = S[0][0];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int e = 0; e < 16; ++e) most = fmaxf(most, S[kb][e]);
            most = fmaxf(most, __shfl_xor(most, 32, 64));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(most - ref > RAISE) != 0ull, 0)) {
                const bool raise = most - ref > RAISE;
                const float higher = raise ? reference(most) : ref;
                const float alpha = __builtin_amdgcn_exp2f(ref - higher);
                ref = higher;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    l[e] *= alpha;
#pragma unroll
                    for (int db = 0; db < NDB; ++db) O[db][e] *= alpha;
                }
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    __builtin_amdgcn_sched_barrier(0);
                    u32x4 P, vf[NDB];
                    read_group<DK>(vf, vt, kb, hf, ln, g);
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float p0 = __builtin_amdgcn_exp2f(S[kb][8 * hf + 2 * w] - ref);
                        const float p1 = __builtin_amdgcn_exp2f(S[kb][8 * hf + 2 * w + 1] - ref);
                        P[w] = pack_f16(p0, p1);
                    }
                    add_group<DK>(O, l, P, vf, ones_of_group(keys_left, kb, hf, g));
                }
        }
        lds_barrier();  // the weights of the second use are complete, V^T of B no longer needed
        if (twice && __builtin_expect(raised != 0u, 0)) {
            // some rows of B have scores too large for their references: 8 below the largest of the tile take the places
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int row = kb * 32 + 8 * r4 + 4 * g;
                    const f32x4 rb = *(const f32x4*)(ref_b + row);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (S[kb][4 * r4 + e] - rb[e] > RAISE) atomicMax(high_b + row + e, S[kb][4 * r4 + e]);
                }
            lds_barrier();
            if (tid == 0) raised = 0u;
            if (tid < ST) {
                const float mx = high_b[tid];
                const bool raise = mx - ref_b[tid] > RAISE;
                if (raise) ref_b[tid] = reference(mx);
                const unsigned long long rows = __builtin_amdgcn_ballot_w64(raise);
                if (ln == 0) raised_rows[tid >> 5] = (unsigned)(rows >> (32 * g));
            }
            lds_barrier();
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                const unsigned rows = __builtin_amdgcn_readfirstlane(raised_rows[kb]);
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    if ((rows >> (8 * r4)) & 0xFFu) store_group(kb, r4);
            }
            lds_barrier();
        }
        if constexpr (Y::RESIDENT) {
            if (j + 1 < j1) vr.stage(vt, tid);
        } else if (twice) {
            vr.stage(vt, tid);
            lds_barrier();
        }
        if (twice) {
            // ---- second use: the wavefront's 32 rows of B over the 128 keys of A ----
            f32x16 Ob[NDB], lb;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                lb[e] = 0.f;
#pragma unroll
                for (int db = 0; db < NDB; ++db) Ob[db][e] = 0.f;
            }
            const int i16 = lane & 15, col = wave * 32 + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
            u32x2 lo[2], hi[2];
            u32x4 vf[2][NDB];
            auto read = [&](int n) {  // group n of the keys of A, which V^T has in the order 0..3, 8..11 (lower half of the lanes),
                                      // 4..7, 12..15 (upper half)
                const int row = n * 16 + 4 * g + (i16 >> 2);
                lo[n & 1] = lds_read_tr16(kt + weight_at(row, col));
                hi[n & 1] = lds_read_tr16(kt + weight_at(row + 8, col));
                read_group<DK>(vf[n & 1], vt_a, n >> 1, n & 1, ln, g);
            };
            read(0);
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                __builtin_amdgcn_sched_barrier(0);
                if (n < 7) read(n + 1);
                add_group<DK>(Ob, lb, u32x4{lo[n & 1][0], lo[n & 1][1], hi[n & 1][0], hi[n & 1][1]}, vf[n & 1],
                              ones_of_group(N - A * ST, n >> 1, n & 1, g));
            }
            __builtin_amdgcn_sched_barrier(0);
            const int jb = wave * 32 + ln;  // this lane's row of B within the tile
            if (B * ST + jb < N) {
                const size_t slot = (((size_t)bh * T + B) * T + A) * ST + jb;
                store_state<DK>(Ob, ref_b[jb], lb[0], g, part_m + slot, part_l + slot, part_o + slot * DK);
            }
        }
        if (j + 1 < j1) {
            if constexpr (!Y::RESIDENT) {
                kr.fetch(zh, partner(j + 1) * ST, tid);
                vr.fetch(zth, partner(j + 1) * ST, tid);
            }
            lds_barrier();  // nobody reads the weights (or V^T of A in the place of that of B) any more
            kr.stage(kt, tid);
            if constexpr (!Y::RESIDENT) vr.stage(vt, tid);
        }
    }
    if (T == 1) {
        // the only state of its rows: y_i = O_i / l_i, through LDS (nobody reads the K tile any more), so that whole rows leave
        constexpr int CPR = DK / 8;
        const float inv = 1.f / l[0];
        unsigned char* const stage = kt + wave * (32 * DK * 2);
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *(u32x2*)(stage + ln * (DK * 2) + (((4 * db + r4) ^ (ln & (CPR - 1))) << 4) + 8 * g) =
                    u32x2{pack_bf16(O[db][4 * r4] * inv, O[db][4 * r4 + 1] * inv), pack_bf16(O[db][4 * r4 + 2] * inv, O[db][4 * r4 + 3] * inv)};
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): only this wavefront reads what it wrote
        const int bb = bh / pb.H, h = bh - bb * pb.H;
#pragma unroll
        for (int it = 0; it < 32 * CPR / 64; ++it) {
            const int row = it * (64 / CPR) + lane / CPR, c = lane % CPR;
            const u32x4 v = *(const u32x4*)(stage + row * (DK * 2) + ((c ^ (row & (CPR - 1))) << 4));
            if (wave * 32 + row < N) *(u32x4_out*)(out + ((size_t)bb * N + wave * 32 + row) * ((size_t)pb.H * DK) + (size_t)h * DK + c * 8) = v;
        }
    } else if (ia < N) {
        const size_t slot = (((size_t)bh * T + A) * T + partner(j0)) * ST + wave * 32 + ln;
        store_state<DK>(O, ref, l[0], g, part_m + slot, part_l + slot, part_o + slot * DK);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
    if (lane == 0) count_add(pb.counters, blockIdx.x * 4u + wave, cnt, phys);
}

// y_i = sum over the key tiles of a row of 2^(m_t - M) O_t / sum 2^(m_t - M) l_t, M the largest m_t.
// Bound by the reads of the partial states, T (d + 2) floats per row: a thread owns four output
// columns of one row and the rows of a wavefront are neighbours, so that every request is a run of
// whole KiB and four of them are in flight per thread (96 heads of 512: 71 -> 10 us against a wavefront per row, 52 MB).
template <int DK>
__global__ __launch_bounds__(256) void sym_merge_kernel(Problem pb, const float* __restrict__ part_m,
                                                        const float* __restrict__ part_l,
                                                        const float* __restrict__ part_o, bf16_t* __restrict__ out, int T, int run)
{
    constexpr int CPR = DK / 4, RPW = 256 / CPR;  // pieces of a row; rows per workgroup, a divisor of 128
    const int bh = blockIdx.y;
    const int bb = bh / pb.H, h = bh - bb * pb.H;
    const int i = blockIdx.x * RPW + threadIdx.x / CPR, c = (threadIdx.x % CPR) * 4;
    if (i >= pb.N) return;
    const int A = i / ST, row = i - A * ST;
    const size_t base = ((size_t)bh * T + A) * T * ST + row;
    const float* pm = part_m + base;
    const float* pl = part_l + base;
    const float* po = part_o + base * DK + c;
    // the states there are: one for every run of own partners, in the place of its first, and one for every other tile
    const int mine = owned(A, T), own_states = (mine + run - 1) / run, states = own_states + T - mine;
    auto place = [&](int s) -> size_t {
        const int t = A + (s < own_states ? s * run : mine + s - own_states);
        return (size_t)(t < T ? t : t - T) * ST;
    };
    float M = -INFINITY, L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < states; s0 += 4) {
        float m[4], lt[4];
        f32x4 o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // past the last: its state once more, with weight zero
            const size_t t = place(min(s0 + u, states - 1));
            m[u] = pm[t];
            lt[u] = pl[t];
            o[u] = *(const f32x4*)(po + t * DK);
        }
        const float before = M;
#pragma unroll
        for (int u = 0; u < 4; ++u) M = fmaxf(M, m[u]);
        const float alpha = __builtin_amdgcn_exp2f(before - M);
        L *= alpha;
        acc *= alpha;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float w = s0 + u < states ? __builtin_amdgcn_exp2f(m[u] - M) : 0.f;
            L += w * lt[u];
            acc += w * o[u];
        }
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    *(u32x2*)(out + ((size_t)bb * pb.N + i) * ((size_t)pb.H * DK) + (size_t)h * DK + c) =
        u32x2{pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
}

}  // namespace

size_t sym_pair_workspace_floats(const Problem& pb)
{
    const size_t T = (size_t)(pb.N + ST - 1) / ST;
    return (size_t)pb.B * pb.H * T * T * ST * (size_t)(pb.d + 2);
}

// z: [B][H][Npad][d] half precision, rows past N zeros; zt: the same vectors in the transposed layout of the
// attention kernels; work: sym_pair_workspace_floats(pb) floats.  The scale has to be above zero (as it is wherever the
// matrix-core kernels are taken): a row's own score is then not below the zeros of the keys past N, whose weights stay finite.
hipError_t launch_sym_pair(const Problem& pb, const h16_t* z, const h16_t* zt, float* work, bf16_t* out, hipStream_t s)
{
    const int T = (pb.N + ST - 1) / ST;
    const size_t rows = (size_t)pb.B * pb.H * T * T * ST;
    float* part_m = work;
    float* part_l = work + rows;
    float* part_o = work + 2 * rows;
    const CountCfg cc = count_cfg(pb.b);
    const float c2 = pb.scale * 1.4426950408889634f;
    const int rows_merge = 1024 / pb.d;
    const dim3 merge_grid((pb.N + rows_merge - 1) / rows_merge, pb.B * pb.H);
    // Runs of a row tile's partners: as short as one workgroup per CU allows, two with six row tiles and more per head, for
    // every run writes a state of its own.  Measured (us, both kernels; runs per row tile one, two, three): 384 row tiles of
    // d_k = 64, T 4 32.6 / 37.1 / -; 192, T 3 24.7 / 26.4; 128, T 16 63 / 43.5 / 43.2; d_k = 128 128, T 4 36.7 / 29.9 / 31.5, T 16 90 / 62 /
    // 63.  Runs of one against two partners: 96 row tiles, T 4 (240 runs) 21.3 / 22.0; 72, T 12 (468 runs) 27.3 / 32.8.
    const long tiles = (long)pb.B * pb.H * T, more = T % 2 == 0 ? tiles / 2 : 0;  // `more` of them have one partner more
    const int least = (T + 1) / 2, most = T / 2 + 1;
    int run = 1;
    while (run < most && more * ((most + run - 1) / run) + (tiles - more) * ((least + run - 1) / run) > (T >= 6 ? 512 : 256)) ++run;
    const int runs = (most + run - 1) / run + (pb.noskip ? T : 0);
    const dim3 grid((unsigned)((tiles * runs + 7) / 8 * 8));
    if (pb.d == 64) {
        hipLaunchKernelGGL(sym_pair_kernel<64>, grid, dim3(256), 0, s, pb, cc, z, zt, part_m, part_l, part_o, out, T, runs, run, pb.noskip, c2, pb.B * pb.H);
        if (T > 1) hipLaunchKernelGGL(sym_merge_kernel<64>, merge_grid, dim3(256), 0, s, pb, part_m, part_l, part_o, out, T, run);
    } else if (pb.d == 128) {
        hipLaunchKernelGGL(sym_pair_kernel<128>, grid, dim3(256), 0, s, pb, cc, z, zt, part_m, part_l, part_o, out, T, runs, run, pb.noskip, c2, pb.B * pb.H);
        if (T > 1) hipLaunchKernelGGL(sym_merge_kernel<128>, merge_grid, dim3(256), 0, s, pb, part_m, part_l, part_o, out, T, run);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace attnring
