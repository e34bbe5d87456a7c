// q/k/v projections (Sec. 3.1: q, k, v are linear maps of the inputs x by three
// learned matrices; one set per head) as ONE bf16 MFMA GEMM over the stacked
// output columns [q | k | v], fp32 accumulation, rounded once to half precision and
// written straight into the layouts the attention kernel streams:
//   q, k : [B][H][Npad][d]            (row = vector, d contiguous)
//   v^T  : [B][H][Npad/64][d][64]     (per 64-key block, key contiguous, and the
//                                      keys of each 16-group in MFMA operand order)
// The weights arrive as [D][H*d] (q = x.W), i.e. contiguous along the output
// columns, while an MFMA operand register wants 8 consecutive values of the
// contraction index.  The main kernel leaves them where they are and turns them
// while reading LDS (ds_read_b64_tr_b16); for weights that are not 16-byte aligned
// a small kernel lays them out as W^T [3*H*d][D] first and the fallback GEMM reads that.
#include "mfma_common.h"

namespace attnring {
namespace {

// ---------------------------------------------------------------------------
// W^T: 64 x 64 tiles through LDS; grid (HD/64, ceil(D/64), 3).  Where it runs it is
// the call's first kernel, so workgroup (0,0,0) clears the counter slots.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void transpose_w_kernel(int D, int HD, const bf16_t* __restrict__ Wq,
                                                          const bf16_t* __restrict__ Wk,
                                                          const bf16_t* __restrict__ Wv, bf16_t* __restrict__ Wt,
                                                          unsigned long long* counters)
{
    __shared__ bf16_t tile[64][64 + 2];
    clear_counters(counters);
    const bf16_t* W = blockIdx.z == 0 ? Wq : (blockIdx.z == 1 ? Wk : Wv);
    bf16_t* dst = Wt + (size_t)blockIdx.z * HD * D;
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int r = ty; r < 64; r += 4) {
        const int gr = r0 + r;
        tile[r][tx] = gr < D ? W[(size_t)gr * HD + c0 + tx] : (bf16_t)0;
    }
    __syncthreads();
    for (int c = ty; c < 64; c += 4) {
        const int gk = r0 + tx;
        if (gk < D) dst[(size_t)(c0 + c) * D + gk] = tile[tx][c];
    }
}

// ---------------------------------------------------------------------------
// Fallback GEMM (unaligned weights), on transposed weights:
// C = A . B^T with both operands k-contiguous.  Square BT x BT tile per
// workgroup, 2 x 2 wavefronts, 32x32x16 MFMA blocks, 64-deep k slices double
// buffered in LDS.  The "x side" rows are vectors (with the per-batch row pitch
// Npad; rows past n read the last real row and are not stored), the "w side"
// rows are output columns of [q | k | v].
// For q and k tiles the w side is the A operand, so a lane ends up with four
// consecutive output columns of one vector (8-byte store into [..][d]); for v
// tiles the x side is the A operand, so a lane holds four consecutive vectors of
// one column (8-byte store into the transposed layout).
// ---------------------------------------------------------------------------
constexpr int BK = 64;
constexpr int ROWB = BK * 2 + 16;  // LDS bytes per tile row (padded)

// Tile order.  Workgroup ids are dealt round-robin to the 8 XCDs, so each XCD is
// given a contiguous run of tile numbers; within the run, tiles are walked in
// groups of GROUP_W weight tiles by all x tiles, weight tile fastest, so that the
// ~32 tiles in flight on one XCD form a 4 x 8 patch that shares its operand
// slices in that XCD's L2 instead of fetching 32 different x slices.
constexpr int GROUP_W = 4;
// What a kernel needs for its tile's place, with the divisions prepared on the host.
struct TileMap {
    int tiles_x, tiles_w, n_tiles;
    int group_w;       // weight tiles walked together
    FastDiv width;     // group_w * tiles_x
    FastDiv per_item;  // x tiles per batch item that hold a vector
    int spread;        // matrices over which the column tiles are dealt (below), 0: not
    int per_matrix;    // column tiles of one matrix
    int mult;          // coprime to tiles_x
    FastDiv by_x;      // tiles_x
};
__device__ __forceinline__ int small_div(int n, int d)  // d in 1..4
{
    return d == 4 ? n >> 2 : d == 2 ? n >> 1 : d == 1 ? n : (int)(__umulhi((unsigned)n, 0xAAAAAAABu) >> 1);
}
// With key lengths some k and v tiles return at once, and an XCD keeps the run of tiles it was
// given: the order above would hand some XCDs q tiles only and others the short batch items.
// Both tile indices are therefore permuted, so that every run holds q, k and v tiles in equal
// parts (groups of three column tiles, dealt round-robin over the three matrices) and x tiles
// from all over the batch (a multiplier that is coprime to their number).
__device__ __forceinline__ void tile_of(const TileMap& tm, int id, int& tw, int& tx)
{
    const int grp = (int)divide((unsigned)id, tm.width);
    const int first_w = grp * tm.group_w;
    const int gsz = min(tm.tiles_w - first_w, tm.group_w);
    const int local = id - grp * (int)tm.width.d;
    tx = small_div(local, gsz);
    tw = first_w + (local - tx * gsz);
    if (tm.spread) {
        const int q = small_div(tw, tm.spread);
        tw = (tw - q * tm.spread) * tm.per_matrix + q;
        const long long t = (long long)tx * tm.mult;
        tx = t <= 0x7fffffffLL ? (int)t - (int)divide((unsigned)t, tm.by_x) * tm.tiles_x : (int)(t % tm.tiles_x);
    }
}
inline TileMap tile_map(const Problem& pb, int bx, int bw, int matrices, bool spread)
{
    TileMap tm;
    // Only tiles that hold a vector are launched: of a short item's 256 padded rows a grid of 64-row tiles was three quarters
    // empty, and the workgroups that had a tile came to lie two to a CU (64 x 2048 -> 6144 29.5 -> 18 us).
    const int per_item = (pb.N + bx - 1) / bx;
    tm.tiles_x = pb.B * per_item;
    tm.tiles_w = matrices * pb.H * pb.d / bw;
    tm.n_tiles = tm.tiles_x * tm.tiles_w;
    // 64 x 64 tiles that are more than the CUs, two workgroups to some of them: groups of three.  What tiles come to share a CU
    // (32 apart in an XCD's run) decides, in groups of four often tiles of the same x rows; measured, whole calls, four / three
    // (rows, d_model -> columns): 256 x 4096 -> 4608 40.2 / 31.8, 512 x 4096 -> 2304 34.7 / 30.3, 360 x 4096 -> 4608 40.5 / 35.1, 128 x
    // 4096 -> 12288 54.3 / 49.7, 384 x 768 -> 4608 17.1 / 16.4, 400 x 1024 -> 3072 18.1 / 18.0; the other way 320 x 4096 -> 6144 38.3 /
    // 41.2, 4096 x 1024 -> 384 22.0 / 22.2.  Up to 256 tiles within 1 %.
    const bool shared = bx == 64 && tm.n_tiles > 256 && tm.n_tiles <= 512;
    tm.group_w = spread ? matrices : shared ? 3 : GROUP_W;
    tm.width = fast_div((unsigned)(tm.group_w * tm.tiles_x));
    tm.per_item = fast_div((unsigned)per_item);
    tm.spread = spread ? matrices : 0;
    tm.per_matrix = tm.tiles_w / matrices;
    tm.mult = tm.tiles_x / 8 + 1;
    for (;; ++tm.mult) {
        int a = tm.mult, b = tm.tiles_x;
        while (b) { const int r = a % b; a = b; b = r; }
        if (a == 1) break;
    }
    tm.by_x = fast_div((unsigned)tm.tiles_x);
    return tm;
}

// Whether every row of an x tile that starts at vector i0 of batch item bb lies at or past the
// item's key length.
__device__ __forceinline__ bool past_key_length(const int* __restrict__ lens, int bb, int i0, int N)
{
    int len = lens[bb];
    len = len < 0 ? 0 : (len > N ? N : len);
    return i0 >= len;
}

template <int BT>
__global__ __launch_bounds__(256) void proj_mfma_kernel(int Bsz, int N, int Npad, int D, int H, int d,
                                                        const bf16_t* __restrict__ X,
                                                        const bf16_t* __restrict__ Wt, h16_t* __restrict__ qo,
                                                        h16_t* __restrict__ ko, h16_t* __restrict__ vto,
                                                        TileMap tm, float qscale, const int* __restrict__ lens, bool skip_q_rows, bool no_q,
                                                        const int* __restrict__ row0)
{
    constexpr int WT = BT / 2;          // wavefront tile edge
    constexpr int NB = WT / 32;         // MFMA blocks per edge
    constexpr int NCH = BT * 8 / 256;   // 16-byte chunks per thread and side
    constexpr int SIDE = BT * ROWB;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * 2 * SIDE];

    const int tid = threadIdx.x;
    const int lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int HD = H * d;

    const int per_xcd = gridDim.x >> 3;
    const int tile_id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile_id >= tm.n_tiles) return;
    int tw, tx_;
    tile_of(tm, tile_id, tw, tx_);
    const int w0 = tw * BT;    // first stacked output column
    const int bb = (int)divide((unsigned)tx_, tm.per_item);  // one batch item per tile
    const int i0 = (tx_ - bb * (int)tm.per_item.d) * BT;
    const bool is_v = w0 >= 2 * HD;
    // Keys past the key length of their batch item are in no allowed pair (Sec. 5.1 applied to
    // padding): their k and v rows are not computed.  (q rows are: every query row has an output.)
    // With padded rows left out as queries too, the same holds for their q rows.
    if (lens != nullptr && (w0 >= HD || skip_q_rows) && past_key_length(lens, bb, i0, N)) return;
    if (no_q && w0 < HD) return;  // q = k = v scheme: the shared vectors are wanted as k and v^T only

    // per-thread source rows: chunk ch = tid + 256*u -> row ch/8, k-chunk ch%8
    const int kc = tid & 7;
    unsigned xoff[NCH], woff[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
        const int row = (tid >> 3) + 32 * u;
        xoff[u] = source_row(row0, Bsz, N, bb, i0 + row) * (unsigned)D;
        woff[u] = (unsigned)(w0 + row) * (unsigned)D;
    }

    f32x16 acc[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

    u32x4 xreg[NCH], wreg[NCH];
    auto issue_loads = [&](int k0) {
        const int kk = k0 + kc * 8;
        const bool in = kk < D;  // D is a multiple of 8
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
            u32x4 z = {0u, 0u, 0u, 0u};
            xreg[u] = in ? *(const u32x4*)(X + (size_t)xoff[u] + kk) : z;
            wreg[u] = in ? *(const u32x4*)(Wt + (size_t)woff[u] + kk) : z;
        }
    };
    // A operand side first, then B operand side
    auto stage_store = [&](int buf) {
        unsigned char* base = lds + buf * 2 * SIDE;
        unsigned char* xs = base + (is_v ? 0 : SIDE);
        unsigned char* ws = base + (is_v ? SIDE : 0);
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
            const int row = (tid >> 3) + 32 * u;
            *(u32x4*)(xs + row * ROWB + kc * 16) = xreg[u];
            *(u32x4*)(ws + row * ROWB + kc * 16) = wreg[u];
        }
    };

    const int nk = (D + BK - 1) / BK;
    issue_loads(0);
    stage_store(0);
    __syncthreads();
    for (int it = 0; it < nk; ++it) {
        if (it + 1 < nk) issue_loads((it + 1) * BK);
        const unsigned char* as = lds + (it & 1) * 2 * SIDE + (wr * WT + ln) * ROWB + g * 16;
        const unsigned char* bs = lds + (it & 1) * 2 * SIDE + SIDE + (wc * WT + ln) * ROWB + g * 16;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            u32x4 af[NB], bf[NB];
#pragma unroll
            for (int a = 0; a < NB; ++a) af[a] = *(const u32x4*)(as + a * 32 * ROWB + ks * 32);
#pragma unroll
            for (int b = 0; b < NB; ++b) bf[b] = *(const u32x4*)(bs + b * 32 * ROWB + ks * 32);
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = mfma32(af[a], bf[b], acc[a][b]);
        }
        if (it + 1 < nk) stage_store((it + 1) & 1);
        __syncthreads();
    }

    // Epilogue.  acc[a][b][r]: A-side row wr*WT + 32a + acc_row(r,g), B-side row wc*WT + 32b + ln.
    if (!is_v) {
        // A side = output columns (4 consecutive per register quad), B side = vectors.
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int i = i0 + wc * WT + 32 * b + ln;
            if (i >= N) continue;
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int col = w0 + wr * WT + 32 * a + 8 * r4 + 4 * g;  // stacked column of register 4*r4
                    const int which = col >= HD ? 1 : 0;
                    const int cc = col - which * HD;
                    const int h = cc / d, l = cc - h * d;
                    h16_t* dst = (which ? ko : qo) + (((size_t)bb * H + h) * Npad + i) * d + l;
                    const float qs = which ? 1.f : qscale;  // q is stored pre-multiplied (see launch_proj_mfma)
                    u32x2 w;
                    w[0] = pack_f16_sat(acc[a][b][4 * r4 + 0] * qs, acc[a][b][4 * r4 + 1] * qs);
                    w[1] = pack_f16_sat(acc[a][b][4 * r4 + 2] * qs, acc[a][b][4 * r4 + 3] * qs);
                    *(u32x2*)dst = w;
                }
        }
    } else {
        // A side = vectors (4 consecutive per register quad), B side = output columns of v.
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int cc = w0 - 2 * HD + wc * WT + 32 * b + ln;
            const int h = cc / d, l = cc - h * d;
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int i = i0 + wr * WT + 32 * a + 8 * r4 + 4 * g;  // vector of register 4*r4
                    if (i >= N) continue;
                    const int blk = i >> 6, r64 = i & 63;
                    const int slot = (r64 & 48) | vt_slot16(r64 & 15);
                    h16_t* dst = vto + ((((size_t)bb * H + h) * (Npad >> 6) + blk) * d + l) * 64 + slot;
                    u32x2 w;
                    w[0] = pack_f16_sat(acc[a][b][4 * r4 + 0], acc[a][b][4 * r4 + 1]);
                    w[1] = pack_f16_sat(acc[a][b][4 * r4 + 2], acc[a][b][4 * r4 + 3]);
                    *(u32x2*)dst = w;
                }
        }
    }
}

// ---------------------------------------------------------------------------
// The GEMM for 16-byte aligned weights, with the operands
// copied from global memory straight into LDS (buffer_load ... lds, 16 bytes per lane) and
// the weights taken in the caller's layout.
//
// A request for 64 KiB of operands takes longer to come back than the MFMAs of one
// 64-deep slice take to run, so two slices have to be in flight, and LDS cannot hold
// three 64-deep stages of a 256 x 256 tile.  The two sides are kept in rings of their own:
//   x side   three units of BX rows x 128 bytes (64 k of a vector: a whole slice).  The vector
//            cache works by 128-byte lines, and a request that takes 64 bytes from each of 16
//            rows costs it twice the lines of one that takes 8 whole ones.  A unit is free when
//            its slice is done; its 16-byte chunks are XOR-swizzled with bits 1..3 of the row
//            index (128-bit operand reads of 16 consecutive rows fall on distinct banks).
//   weights  four slots of 32 k-rows x BW columns (half a slice) as they lie in memory, read
//            with the transposing LDS read (see the offset table in the kernel).  A slot is
//            free half a slice after its first read.
// Every request has at least one slice period to land.  WR x WC wavefronts share a BX x BW tile.
// The 128 x 256 tile has smaller rings (two x units, three weight slots: 80 KiB), so that two
// workgroups share a CU (slice_pair); TRI are 128 x 128 tiles on rings of 48 KiB, three to a CU
// (slice_tri).
// TAIL: d_model is a multiple of 8 only.  In the last slice the 16-byte pieces of a vector past its
// end, and the k-rows past the last, are fetched from a piece of zeros, through per-lane addresses.
// ---------------------------------------------------------------------------
__device__ const u32x4 zero_piece = {0u, 0u, 0u, 0u};

template <int BX, int BW, int WR, int WC, bool TRI, bool TAIL>
__global__ __launch_bounds__(64 * WR * WC, TRI ? 3 : 2)
void proj_dma_kernel(int Bsz, int N, int Npad, int D, int H, int d, const bf16_t* __restrict__ X,
                     const bf16_t* __restrict__ Wq, const bf16_t* __restrict__ Wk, const bf16_t* __restrict__ Wv,
                     h16_t* __restrict__ qo, h16_t* __restrict__ ko, h16_t* __restrict__ vto, TileMap tm,
                     float qscale, const int* __restrict__ lens, bool skip_q_rows, bool no_q,
                     const int* __restrict__ row0, unsigned long long* __restrict__ counters)
{
    constexpr int NW = WR * WC;
    constexpr bool PAIR = BX != BW;              // 128 x 256 tile, two workgroups per CU
    // A side: output columns for q and k tiles, vectors for v tiles.  MFMA blocks of a wavefront:
    constexpr int NBLK = BX * BW / (1024 * NW);
    constexpr int NX = PAIR ? BX / WC / 32 : 0, NWC = PAIR ? BW / WR / 32 : 0;  // PAIR: the same for both kinds
    constexpr int XU = BX * 128;                 // bytes of one x unit: BX rows x 64 k
    constexpr int NXU = PAIR || TRI ? 2 : 3;
    constexpr int WROWB = BW * 2;                // bytes of one k-row of the weight side in a slot
    constexpr int WS = 32 * WROWB;               // bytes of one weight slot: 32 k-rows
    constexpr int NWS = TRI ? 2 : PAIR ? 3 : 4;
    constexpr int W_BASE = NXU * XU;
    constexpr int XPW = (BX / 8) / NW;           // x pieces (1 KiB: 8 rows x 128 bytes) per wavefront and slice
    constexpr int WPW = (WS / 1024) / NW;        // weight pieces (1 KiB) per wavefront and half slice
    static_assert(XPW == 4 && WPW == (PAIR ? 4 : 2), "what the request schedules below deal out");
    constexpr int WCPR = WROWB / 16;             // 16-byte chunks of a weight k-row
    constexpr int WRPP = 64 / WCPR;              // k-rows per 1 KiB piece
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NXU * XU + NWS * WS];
    clear_counters(counters);  // this is the first kernel of a forward pass on this path

    const int tid = threadIdx.x;
    const int lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int HD = H * d;

    const int per_xcd = gridDim.x >> 3;
    const int tile_id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile_id >= tm.n_tiles) return;
    int tw, tx_;
    // no_q (the queries are not wanted: q = k = v scheme, or projected by the attention kernel): the
    // grid holds the k and v column tiles only
    tile_of(tm, tile_id, tw, tx_);
    const int bb = (int)divide((unsigned)tx_, tm.per_item);  // one batch item per tile
    const int i0 = (tx_ - bb * (int)tm.per_item.d) * BX;
    const int w0 = tw * BW + (no_q ? HD : 0);
    const bool is_v = w0 >= 2 * HD;
    // Keys past the key length of their batch item are in no allowed pair (Sec. 5.1 applied to
    // padding): their k and v rows are not computed.  (q rows are: every query row has an output.)
    // With padded rows left out as queries too, the same holds for their q rows.
    if (lens != nullptr && (w0 >= HD || skip_q_rows) && past_key_length(lens, bb, i0, N)) return;

    // The weights stay in the caller's layout, W[k][column]: this tile's columns of the one matrix
    // it lies in.
    const int which = w0 >= 2 * HD ? 2 : w0 >= HD ? 1 : 0;
    const bf16_t* Wm = (which == 0 ? Wq : (which == 1 ? Wk : Wv)) + (w0 - which * HD);

    // Source byte offsets of this lane for its pieces.  32 bits hold them (attn_init bounds the
    // element counts), which lets a request take a uniform 64-bit base and this offset.
    //   x side: rows are vectors, 128 bytes (64 k) each; piece m = wave + NW*u holds rows
    //           8m..8m+7; the lane lands at row 8m + lane/8, chunk position lane%8;
    //   w side: rows are k, BW columns each; piece m holds k-rows m*WRPP..; the lane lands at
    //           k-row m*WRPP + lane/WCPR, chunk position lane%WCPR.
    // Either way it fetches the chunk that the swizzle of its row puts at that position.
    unsigned xoff[XPW], woff[WPW];
#pragma unroll
    for (int u = 0; u < XPW; ++u) {
        const int row = (wave + NW * u) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        xoff[u] = 2u * (source_row(row0, Bsz, N, bb, i0 + row) * (unsigned)D + c * 8);
    }
#pragma unroll
    for (int u = 0; u < WPW; ++u) {
        const int kr = (wave + NW * u) * WRPP + lane / WCPR;
        const int wc16 = (lane % WCPR) ^ (4 * (kr & 3));
        woff[u] = 2u * ((unsigned)kr * (unsigned)HD + wc16 * 8);
    }
    // Buffer addressing: descriptor base + the lane's 32-bit offset + a scalar offset for the
    // slice, so that a request costs no vector instruction for its address.
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, -1, 0x00020000);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Wm, 0, -1, 0x00020000);
    // piece u of the x side of the slice that starts at k0, into unit `unit`
    typedef const __attribute__((address_space(1))) void* global_ptr;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    auto req_x = [&](int u, int k0, int unit) {
        unsigned char* dst = lds + unit * XU + (wave + NW * u) * 1024;
        if (TAIL && k0 + 64 > D) {
            const int c = (lane & 7) ^ ((((wave + NW * u) * 8 + (lane >> 3)) >> 1) & 7);
            const void* src = k0 + 8 * c < D ? (const void*)((const unsigned char*)X + xoff[u] + 2u * (unsigned)k0)
                                             : (const void*)&zero_piece;
            __builtin_amdgcn_global_load_lds((global_ptr)src, (lds_ptr)dst, 16, 0, 0);
            return;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (__attribute__((address_space(3))) void*)dst, 16,
                                                 (int)xoff[u], (int)(2u * (unsigned)k0), 0, 0);
    };
    // piece u of half h of the weight side of the slice that starts at k0, into slot `slot`
    auto req_w = [&](int u, int k0, int h, int slot) {
        unsigned char* dst = lds + W_BASE + slot * WS + (wave + NW * u) * 1024;
        if (TAIL && k0 + 64 > D) {
            const int kr = k0 + 32 * h + (wave + NW * u) * WRPP + lane / WCPR;
            const void* src = kr < D ? (const void*)((const unsigned char*)Wm + woff[u] +
                                                     2u * ((unsigned)(k0 + 32 * h) * (unsigned)HD))
                                     : (const void*)&zero_piece;
            __builtin_amdgcn_global_load_lds((global_ptr)src, (lds_ptr)dst, 16, 0, 0);
            return;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (__attribute__((address_space(3))) void*)dst, 16,
                                                 (int)woff[u], (int)(2u * (unsigned)(k0 + 32 * h) * (unsigned)HD), 0, 0);
    };

    // LDS byte offsets of this lane's operand reads, from the unit / slot base, for the first
    // 32-row block of the wavefront's share of each side.
    //   x side: 128 bits = 8 k of row ln, chunk 2*ks + g of the four k-steps of a slice; 2*ks has no
    //           bit in common with g, so the offset for k-step ks is the one for k-step 0 XOR 32*ks.
    //   w side: stored k-major, read with the transposing 64-bit LDS read: 16 lanes hand in the
    //           addresses of a 4 (k) x 16 (columns) patch, four columns each, and lane i gets
    //           column i of the patch, its four k values.  Lanes 16..31 take the next 16 columns,
    //           the upper half of the wavefront the upper 8 k of the k-step; two reads (4 k each)
    //           make one operand.  k-rows are BW*2 bytes apart, a multiple of the 256 bytes the
    //           banks span, and LDS serves 32 lanes (two patches, 4 k x 32 columns) at a time, so
    //           the chunks of k-row k are XOR-ed with 4*(k%4): the four 64-byte runs then fall on
    //           different banks.  That XOR reaches bits 2 and 3 of the chunk index, which is also
    //           where the 32-column block number sits: one table per block.
    // Square tiles: the A side is split WR ways and the B side WC ways, whichever is which; the 128 x 256
    // tile splits the columns WR ways and the vectors WC ways.
    const int x_row0 = PAIR || !is_v ? wc * (BX / WC) : wr * (BX / WR);  // first x row / w column of this wavefront
    const int w_col0 = PAIR || !is_v ? wr * (BW / WR) : wc * (BW / WC);
    constexpr int NWB = BW / 32 / (WR < WC ? WR : WC);  // 32-column blocks of the weight side of a wavefront, at most
    int wfo[NWB];  // w side: k-step 0, first read; the others lie whole k-rows further (same k % 4)
    const int xfo0 = (x_row0 + ln) * 128 + ((g ^ ((ln >> 1) & 7)) << 4);  // x_row0 is a multiple of 32
#pragma unroll
    for (int blk = 0; blk < NWB; ++blk) {
        const int i16 = lane & 15;
        const int k = 8 * g + (i16 >> 2);
        const int col = w_col0 + 32 * blk + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
        wfo[blk] = k * WROWB + (((col >> 3) ^ (4 * (k & 3))) << 4) + ((col & 7) << 1);
    }

    f32x16 acc[NBLK];  // [A block][B block]
#pragma unroll
    for (int e = 0; e < NBLK; ++e)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[e][r] = 0.f;

    // One k-step = the MFMAs of 16 k values on fragments that are already in registers.  Behind
    // the first MFMAs go, two at a time, the reads of the fragments of the following k-step (order
    // a0, b0.., a1..: what its first MFMAs need comes first); nd requests (numbers q0 .. q0+nd-1 of
    // a slice) are spread over the MFMAs: a wavefront that sends all requests of a slice in one run
    // issues no MFMA meanwhile, and since all wavefronts do so at the same point the matrix pipe
    // would drain.  The order is pinned with scheduling fences; the group-barrier solver drops its
    // pattern as soon as memory requests are part of it.
    // MFMA blocks of a wavefront on the A and on the B side
    constexpr int NA_V = PAIR ? NX : BX / WR / 32, NB_V = NBLK / NA_V;
    constexpr int NA_QK = PAIR ? NWC : BW / WR / 32, NB_QK = NBLK / NA_QK;
    constexpr int NA_MAX = NA_V > NA_QK ? NA_V : NA_QK, NB_MAX = NB_V > NB_QK ? NB_V : NB_QK;
    u32x4 af[2][NA_MAX], bf[2][NB_MAX];
    // ks4: k-step of the slice, 0..3
    auto x_frag = [&](const unsigned char* unit_base, int ks4, int blk) -> u32x4 {
        return *(const u32x4*)(unit_base + (xfo0 ^ (32 * ks4)) + blk * 4096);
    };
    // The transposing reads are written out by hand: as a builtin, the compiler takes them to
    // alias the copies into LDS that are still in flight and makes each of them wait for all of
    // those (vmcnt(0)), which is the prefetch gone.  It does not count hand-written requests, so
    // every k-step starts with its own wait for the LDS reads of the one before.
    const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
    auto w_frag = [&](const unsigned char* slot_base, int ks, int blk) -> u32x4 {
        const unsigned addr = lds_addr + (unsigned)(slot_base - lds) + (unsigned)wfo[blk];
        u32x2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(16 * ks * WROWB));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"((16 * ks + 4) * WROWB));
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };
    // fragment number r of a k-step, in the order a0, b0.., a1..; the weights are the A side of q and
    // k tiles and the B side of v tiles
    // hs: half slice 0 / 1 of x unit `unit` and weight slot `slot`; ks: k-step 0 / 1 of the half slice
    auto read_frag = [&](auto is_v_, u32x4 (&fa)[NA_MAX], u32x4 (&fb)[NB_MAX], int r, const unsigned char* unit_base,
                         const unsigned char* slot_base, int hs, int ks) {
        constexpr bool IS_V = decltype(is_v_)::value;
        constexpr int NBK = IS_V ? NB_V : NB_QK;
        if (r == 0 || r > NBK) {
            const int a = r == 0 ? 0 : r - NBK;
            fa[a] = IS_V ? x_frag(unit_base, 2 * hs + ks, a) : w_frag(slot_base, ks, a);
        } else {
            fb[r - 1] = IS_V ? w_frag(slot_base, ks, r - 1) : x_frag(unit_base, 2 * hs + ks, r - 1);
        }
    };
    auto load_frags = [&](auto is_v_, u32x4 (&fa)[NA_MAX], u32x4 (&fb)[NB_MAX], int unit, int slot, int hs, int ks) {
        constexpr bool IS_V = decltype(is_v_)::value;
#pragma unroll
        for (int r = 0; r < (IS_V ? NA_V + NB_V : NA_QK + NB_QK); ++r)
            read_frag(is_v_, fa, fb, r, lds + unit * XU, lds + W_BASE + slot * WS, hs, ks);
    };
    // `reqs(i)`, i = 0 .. ND-1: the requests that go out behind the MFMAs of this k-step
    auto kstep = [&](auto is_v_, const u32x4 (&fa)[NA_MAX], const u32x4 (&fb)[NB_MAX], u32x4 (&na)[NA_MAX],
                     u32x4 (&nb)[NB_MAX], int unit, int slot, int hs, int ks, auto nd_, auto&& reqs) {
        constexpr int ND = decltype(nd_)::value;
        constexpr bool IS_V = decltype(is_v_)::value;
        constexpr int NA = IS_V ? NA_V : NA_QK, NBK = IS_V ? NB_V : NB_QK;
        constexpr int NRD = NA + NBK, NMF = NA * NBK;
        static_assert(NRD % 2 == 0 && NRD / 2 <= NMF, "read pairs fit behind the MFMAs of a k-step");
        static_assert(ND <= NMF, "at most one request per MFMA");
        const unsigned char* unit_base = lds + unit * XU;
        const unsigned char* slot_base = lds + W_BASE + slot * WS;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the fragments of this k-step are in
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int b = 0; b < NBK; ++b) {
                acc[a * NBK + b] = mfma32(fa[a], fb[b], acc[a * NBK + b]);
                const int m = a * NBK + b + 1;  // MFMAs issued so far
                if (m <= NRD / 2) {
                    read_frag(is_v_, na, nb, 2 * m - 2, unit_base, slot_base, hs, ks);
                    read_frag(is_v_, na, nb, 2 * m - 1, unit_base, slot_base, hs, ks);
                }
                if (ND > 0 && (m * ND) % NMF == 0) reqs(m * ND / NMF - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr std::integral_constant<int, 0> no_req{};
    constexpr std::integral_constant<int, 1> one_req{};
    constexpr std::integral_constant<int, 2> two_req{};

    // Slice j: x in unit ux, its two weight half slices in slots wa and wa+1.  A k-step runs the
    // MFMAs of fragments that are in registers and reads those of the next k-step.  The barrier
    // of a half slice sits before its second k-step, whose fragments are in registers by then:
    // behind the first barrier (A) slot wa is free, behind the second (B) slot wa+1 and unit ux,
    // and the matrix pipe has work on both sides of either.  Each k-step sends two requests for
    // what has just become free, the weight piece first:
    //     step 1   weights (j+1, half 1) piece 1  -> slot wa+3      x (j+2) piece 0 -> unit ux+2
    //     step 2   weights (j+2, half 0) piece 0  -> slot wa        x (j+2) piece 1
    //     step 3   weights (j+2, half 0) piece 1  -> slot wa        x (j+2) piece 2
    //     step 4   weights (j+2, half 1) piece 0  -> slot wa+1      x (j+2) piece 3
    // Loads return in order.  Barrier B wants x (j+1) and the first weight half of slice j+1 in,
    // whose last piece went out in step 4 of slice j-1: the six requests of steps 1-3 may be in
    // flight.  Barrier A wants the second weight half of slice j in, whose last piece went out
    // first in step 1 of slice j-1: nine requests may be in flight.  VAR: 2 if slice j+2 exists,
    // 1 if slice j+1 is the last, 0 if slice j is.
    auto slice = [&](auto is_v_, auto var_, int j, int& ux, int& wa) {
        constexpr int VAR = decltype(var_)::value;
        constexpr bool E1 = VAR >= 1, E2 = VAR == 2;
        const int ux1 = ux == NXU - 1 ? 0 : ux + 1, ux2 = ux1 == NXU - 1 ? 0 : ux1 + 1;
        const int wb = (wa + 1) & 3, wc = (wa + 2) & 3, wd = (wa + 3) & 3;
        const int k1 = (j + 1) * 64, k2 = (j + 2) * 64;
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, wa, 0, 1, std::integral_constant<int, (E1 ? 1 : 0) + (E2 ? 1 : 0)>{},
              [&](int i) {
                  if (E1 && i == 0) req_w(1, k1, 1, wd);
                  else req_x(0, k2, ux2);
              });
        __builtin_amdgcn_s_waitcnt(0x0070 | (8 * (E1 ? 1 : 0) + (E2 ? 1 : 0)));  // lgkmcnt(0), see above
        __builtin_amdgcn_s_barrier();
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux, wb, 1, 0, std::integral_constant<int, E2 ? 2 : 0>{}, [&](int i) {
            if (i == 0) req_w(0, k2, 0, wa);
            else req_x(1, k2, ux2);
        });
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, wb, 1, 1, std::integral_constant<int, E2 ? 2 : 0>{}, [&](int i) {
            if (i == 0) req_w(1, k2, 0, wa);
            else req_x(2, k2, ux2);
        });
        __builtin_amdgcn_s_waitcnt(0x0070 | ((E1 ? 1 : 0) + 5 * (E2 ? 1 : 0)));
        __builtin_amdgcn_s_barrier();
        // reads ahead into slice j+1
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux1, wc, 0, 0, std::integral_constant<int, E2 ? 2 : 0>{}, [&](int i) {
            if (i == 0) req_w(0, k2, 1, wb);
            else req_x(3, k2, ux2);
        });
        ux = ux1;
        wa = wc;
    };

    // The 128 x 256 tile: two x units, three weight half slices (h = 2j, 2j + 1 of slice j, slot h mod 3), the
    // same two barriers per slice.  Behind the first barrier (half slice 2j read) its slot takes half slice
    // 2j + 3, two pieces in each of steps 2 and 3; behind the second, half slice 2j + 1's slot takes 2j + 4 and
    // slice j's x unit takes x of slice j + 2, two pieces of either in step 4 and in step 1 of the next slice.
    // Loads return in order: the first barrier of slice j wants half slice 2j + 1, sent in steps 2 and 3 of
    // slice j - 1, and the eight requests sent since may be in flight; the second wants all that was sent
    // up to step 1, four may be.  The other workgroup of the CU fills what these short distances leave.
    auto slice_pair = [&](auto is_v_, auto var_, int j, int& ux, int& sa) {
        constexpr int VAR = decltype(var_)::value;
        constexpr bool E1 = VAR >= 1, E2 = VAR == 2;
        const int sb = sa == 2 ? 0 : sa + 1, sc = sb == 2 ? 0 : sb + 1;  // slots of half slices 2j + 1 and 2j + 2
        const int k1 = (j + 1) * 64, k2 = (j + 2) * 64;
        const std::integral_constant<int, E1 ? 4 : 0> four{};
        const std::integral_constant<int, E1 ? 2 : 0> two{};
        const std::integral_constant<int, E2 ? 4 : 0> next_four{};
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, sa, 0, 1, four, [&](int i) {
            if (i < 2) req_w(2 + i, k1, 0, sc);
            else req_x(i, k1, ux ^ 1);
        });
        __builtin_amdgcn_s_waitcnt(0x0070 | (E1 ? 8 : 0));
        __builtin_amdgcn_s_barrier();
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux, sb, 1, 0, two, [&](int i) { req_w(i, k1, 1, sa); });
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, sb, 1, 1, two, [&](int i) { req_w(2 + i, k1, 1, sa); });
        __builtin_amdgcn_s_waitcnt(0x0070 | (E1 ? 4 : 0));
        __builtin_amdgcn_s_barrier();
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux ^ 1, sc, 0, 0, next_four, [&](int i) {
            if (i < 2) req_w(i, k2, 0, sb);
            else req_x(i - 2, k2, ux);
        });
        ux ^= 1;
        sa = sc;
    };

    // TRI, 128 x 128 tiles with three workgroups per CU: two x units and two weight half slices (48 KiB).  Behind
    // the first barrier half slice 2j's slot takes 2j + 2 (step 2), behind the second that of 2j + 1 takes
    // 2j + 3 and slice j's unit takes x of slice j + 2 (steps 4 and 1).  The second barrier wants everything in,
    // the first all but x of the next slice; the other two workgroups fill the waits.
    auto slice_tri = [&](auto is_v_, auto var_, int j, int& ux, int&) {
        constexpr int VAR = decltype(var_)::value;
        constexpr bool E1 = VAR >= 1, E2 = VAR == 2;
        const int k1 = (j + 1) * 64, k2 = (j + 2) * 64;
        const std::integral_constant<int, E1 ? 2 : 0> two{};
        const std::integral_constant<int, E2 ? 4 : E1 ? 2 : 0> last{};
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, 0, 0, 1, two, [&](int i) { req_x(2 + i, k1, ux ^ 1); });
        __builtin_amdgcn_s_waitcnt(0x0070 | (E1 ? 4 : 0));
        __builtin_amdgcn_s_barrier();
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux, 1, 1, 0, two, [&](int i) { req_w(i, k1, 0, 0); });
        kstep(is_v_, af[0], bf[0], af[1], bf[1], ux, 1, 1, 1, no_req, [&](int) {});
        __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();
        kstep(is_v_, af[1], bf[1], af[0], bf[0], ux ^ 1, 0, 0, 0, last, [&](int i) {
            if (i < 2) req_w(i, k1, 1, 1);
            else req_x(i - 2, k2, ux);
        });
        ux ^= 1;
    };

    // Prologue: slice 0 whole, and of slice 1 what steps 2-4 of a slice before slice 0 would
    // have sent (its last weight piece follows in step 1 of slice 0).
    const int ns = TAIL ? (D + 63) / 64 : D / 64;
#pragma unroll
    for (int u = 0; u < WPW; ++u) req_w(u, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < XPW; ++u) req_x(u, 0, 0);
#pragma unroll
    for (int u = 0; u < WPW; ++u) req_w(u, 0, 1, 1);
    if constexpr (TRI) {
        if (ns > 1) {
            req_x(0, 64, 1);
            req_x(1, 64, 1);
            __builtin_amdgcn_s_waitcnt(0x0F70 | 4);
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70);
        }
    } else if constexpr (PAIR) {  // and what step 4 of a slice before slice 0 would have sent
        if (ns > 1) {
            req_w(0, 64, 0, 2);
            req_w(1, 64, 0, 2);
            req_x(0, 64, 1);
            req_x(1, 64, 1);
            __builtin_amdgcn_s_waitcnt(0x0F70 | 8);  // x and the first half of the weights of slice 0 have landed
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70);
        }
    } else if (ns > 1) {
        req_x(0, 64, 1);
        req_w(0, 64, 0, 2);
        req_x(1, 64, 1);
        req_w(1, 64, 0, 2);
        req_x(2, 64, 1);
        req_w(0, 64, 1, 3);
        req_x(3, 64, 1);
        __builtin_amdgcn_s_waitcnt(0x0F70 | 7);  // loads return in order: slice 0 has landed
    } else {
        __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    __builtin_amdgcn_s_barrier();
    auto all_slices = [&](auto is_v_) {
        load_frags(is_v_, af[0], bf[0], 0, 0, 0, 0);
        int ux = 0, wa = 0;
        int j = 0;
        auto one = [&](auto var_) {
            if constexpr (TRI) slice_tri(is_v_, var_, j, ux, wa);
            else if constexpr (PAIR) slice_pair(is_v_, var_, j, ux, wa);
            else slice(is_v_, var_, j, ux, wa);
        };
#pragma nounroll
        for (; j + 2 < ns; ++j) one(two_req);
#pragma nounroll
        for (; j + 1 < ns; ++j) one(one_req);
#pragma nounroll
        for (; j < ns; ++j) one(no_req);
    };
    if (is_v) all_slices(std::true_type{});
    else all_slices(std::false_type{});
    __builtin_amdgcn_s_waitcnt(0x0070);  // the fragments read ahead for a slice that does not exist are dropped
    __builtin_amdgcn_s_barrier();

    // Epilogue.  Register r of block (a, b): A-side row 32a + acc_row(r,g), B-side row 32b + ln of the
    // wavefront's share.  A lane owns 8-byte runs whose neighbours in memory sit in other lanes' later registers, so
    // storing them directly would touch 64 cache lines per instruction.  The tile is staged in LDS
    // (free by now) in the order of the output arrays and leaves in 16-byte pieces, a full KiB of
    // consecutive addresses per wavefront and instruction.  Staged rows are XOR-swizzled by 16-byte
    // chunk like the operand tiles, which keeps both the 8-byte writes and the 16-byte reads spread
    // over the banks.
    constexpr int NT = 64 * NW;
    constexpr int UNITS = BX * BW / 8;  // 16-byte pieces of the tile
    const int dsh = d == 128 ? 7 : 6;   // d is 64 or 128 on this path
    if (!is_v) {
        // q and k: [head][vector][d], a staged row is one vector's d values of one head.
        const int which = w0 >= HD ? 1 : 0;
        const float qs = which ? 1.f : qscale;  // q is stored pre-multiplied (see launch_proj_mfma)
        const int cmask = (d >> 3) - 1, rowb = 2 * d;
#pragma unroll
        for (int b = 0; b < NB_QK; ++b) {
            const int v = x_row0 + 32 * b + ln;
#pragma unroll
            for (int a = 0; a < NA_QK; ++a)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int ct = w_col0 + 32 * a + 8 * r4;  // tile column of register 4*r4 in half 0
                    const int hc = ct >> dsh, c = (ct & (d - 1)) >> 3;
                    u32x2 w;
                    w[0] = pack_f16_sat(acc[a * NB_QK + b][4 * r4 + 0] * qs, acc[a * NB_QK + b][4 * r4 + 1] * qs);
                    w[1] = pack_f16_sat(acc[a * NB_QK + b][4 * r4 + 2] * qs, acc[a * NB_QK + b][4 * r4 + 3] * qs);
                    *(u32x2*)(lds + (hc * BX + v) * rowb + ((c ^ (v & cmask)) << 4) + 8 * g) = w;
                }
        }
        __syncthreads();
        h16_t* base = (which ? ko : qo) + ((size_t)bb * H + ((w0 - which * HD) >> dsh)) * Npad * d;
#pragma unroll 4
        for (int e0 = tid; e0 < UNITS; e0 += NT) {
            const int hv = e0 >> (dsh - 3);  // head-in-tile * BX + vector
            const int c = e0 & cmask;
            const int hc = hv / BX, v = hv - hc * BX;
            if (i0 + v >= N) continue;  // rows past n are left as they are
            const u32x4 val = *(const u32x4*)(lds + hv * rowb + ((c ^ (v & cmask)) << 4));
            *(u32x4*)(base + ((size_t)hc * Npad + i0 + v) * d + c * 8) = val;
        }
    } else {
        // v transposed: [head][64-key block][d][64 key slots], a staged row is the 64 slots of one
        // column; vectors past n are staged as zeros.
#pragma unroll
        for (int b = 0; b < NB_V; ++b) {
            const int cl = w_col0 + 32 * b + ln;
            const int hc = cl >> dsh, l = cl & (d - 1);
#pragma unroll
            for (int a = 0; a < NA_V; ++a)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const int vl = x_row0 + 32 * a + 8 * r4 + 4 * g;  // vector of register 4*r4
                    const int vb = vl >> 6, r64 = vl & 63;
                    const int slot = (r64 & 48) | vt_slot16(r64 & 15);
                    const int left = N - (i0 + vl);
                    u32x2 w;
                    w[0] = pack_f16_sat(left > 0 ? acc[a * NB_V + b][4 * r4 + 0] : 0.f, left > 1 ? acc[a * NB_V + b][4 * r4 + 1] : 0.f);
                    w[1] = pack_f16_sat(left > 2 ? acc[a * NB_V + b][4 * r4 + 2] : 0.f, left > 3 ? acc[a * NB_V + b][4 * r4 + 3] : 0.f);
                    *(u32x2*)(lds + ((hc * (BX / 64) + vb) * d + l) * 128 + (((slot >> 3) ^ (l & 7)) << 4) +
                              2 * (slot & 7)) = w;
                }
        }
        __syncthreads();
        const int h0 = (w0 - 2 * HD) >> dsh;
#pragma unroll 4
        for (int e0 = tid; e0 < UNITS; e0 += NT) {
            const int ul = e0 >> 3;  // (head-in-tile * blocks + block) * d + column
            const int c = e0 & 7;
            const int u = ul >> dsh, l = ul & (d - 1);
            const int hc = u / (BX / 64), vb = u - hc * (BX / 64);
            const int blk = (i0 >> 6) + vb;
            if (blk * 64 >= N) continue;  // so are blocks past n
            const u32x4 val = *(const u32x4*)(lds + ul * 128 + ((c ^ (l & 7)) << 4));
            *(u32x4*)(vto + ((((size_t)bb * H + h0 + hc) * (Npad >> 6) + blk) * d + l) * 64 + c * 8) = val;
        }
    }
}

// ---------------------------------------------------------------------------
// The GEMM for products of few tiles, and for columns that do not come in 128s (an odd number of
// 64-wide heads): 64 x 64 tiles, four wavefronts of 32 x 32, operands copied straight into LDS.
// Both sides are rows of 128 bytes: x rows with their chunks XOR-ed with bits 1..3 of the row, k-rows of W
// with 4 * bit 1 of k (transposing reads).  A slice is one barrier, eight LDS reads and four MFMAs per
// wavefront.  Stores go out from the accumulators, eight bytes per lane: four instructions per wavefront.
//
// STAGES, the slices of x and W that the ring holds.  A product that leaves CUs idle is bound by its own
// chain of slices and by what the first read of an input takes, so five (80 KiB, two workgroups share a CU):
// 15 packed items of up to 536 vectors, 576 -> 192, on inputs new to every call 16.5 us the call, 17.4 with
// three.  A product of more tiles than those 512 workgroups is bound by how many workgroups a CU holds
// against the barriers and the stores, so three (48 KiB, three to a CU): 576 tiles and more 5 to 25 % less
// time (8192 x 136 -> 2880 40 -> 31 us, 8192 x 960 -> 2880 85 -> 75, 2400 x 640 -> 1920 22 -> 18).
// ---------------------------------------------------------------------------
inline bool ring_of_three(long tiles) { return tiles > 512; }
// FLOAT_OUT (the float path's bfloat16 storage): the product is written as floats, all three matrices
// as [vector][d] rows of their heads, d a multiple of 4; the vectors of all batch items are one run of
// rows (Bsz 1, N of them), `items` divides by an item's.
template <int STAGES, bool TAIL, bool FLOAT_OUT>
__global__ __launch_bounds__(256, STAGES == 3 ? 3 : 2)
void proj_small_kernel(int Bsz, int N, int Npad, int D, int H, int d, const bf16_t* __restrict__ X,
                       const bf16_t* __restrict__ Wq, const bf16_t* __restrict__ Wk, const bf16_t* __restrict__ Wv,
                       void* __restrict__ qo, void* __restrict__ ko, void* __restrict__ vto, TileMap tm,
                       float qscale, const int* __restrict__ lens, bool skip_q_rows, bool no_q,
                       const int* __restrict__ row0, unsigned long long* __restrict__ counters, FastDiv items,
                       FastDiv columns)
{
    constexpr int XB = 64 * 128, STAGE = 2 * XB;  // x: 64 rows x 64 k; W: 64 k-rows x 64 columns
    __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES * STAGE];
    clear_counters(counters);  // this is the first kernel of a forward pass on this path

    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HD = H * d;
    const int per_xcd = gridDim.x >> 3;
    const int tile_id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (tile_id >= tm.n_tiles) return;
    int tw, tx_;
    tile_of(tm, tile_id, tw, tx_);
    const int bb = (int)divide((unsigned)tx_, tm.per_item);
    const int i0 = (tx_ - bb * (int)tm.per_item.d) * 64;
    const int w0 = tw * 64 + (no_q ? HD : 0);
    if (lens != nullptr && (w0 >= HD || skip_q_rows) && past_key_length(lens, bb, i0, N)) return;  // see proj_dma_kernel
    const int which = w0 >= 2 * HD ? 2 : w0 >= HD ? 1 : 0;
    const int c0 = w0 - which * HD;  // first column in its matrix
    const bf16_t* Wm = (which == 0 ? Wq : (which == 1 ? Wk : Wv)) + c0;

    // pieces wave and wave + 4 of either side: rows 8 * piece + lane / 8, chunk position lane % 8
    unsigned xoff[2], woff[2];
    const int rl = lane >> 3, xc = (lane & 7) ^ ((rl >> 1) & 3);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row = 8 * (wave + 4 * u) + rl;
        const int cx = xc ^ (((row >> 3) & 1) << 2);  // chunk XOR (row >> 1) & 7
        const int cw = (lane & 7) ^ (4 * ((row >> 1) & 1));
        xoff[u] = 2u * (source_row(row0, Bsz, N, bb, i0 + row) * (unsigned)D + cx * 8);
        woff[u] = 2u * ((unsigned)row * (unsigned)HD + cw * 8);
    }
    const __amdgpu_buffer_rsrc_t x_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, -1, 0x00020000);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Wm, 0, -1, 0x00020000);
    typedef const __attribute__((address_space(1))) void* global_ptr;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    auto request = [&](int j, int stage) {  // slice j: two x and two W pieces of this wavefront
        const int k0 = 64 * j;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            unsigned char* xd = lds + stage * STAGE + (wave + 4 * u) * 1024;
            unsigned char* wd = xd + XB;
            if (TAIL && k0 + 64 > D) {
                const int row = 8 * (wave + 4 * u) + rl, cx = xc ^ (((row >> 3) & 1) << 2);
                const void* xs = k0 + 8 * cx < D ? (const void*)((const unsigned char*)X + xoff[u] + 2u * (unsigned)k0)
                                                 : (const void*)&zero_piece;
                const void* ws = k0 + row < D ? (const void*)((const unsigned char*)Wm + woff[u] +
                                                              2u * ((unsigned)k0 * (unsigned)HD))
                                              : (const void*)&zero_piece;
                __builtin_amdgcn_global_load_lds((global_ptr)xs, (lds_ptr)xd, 16, 0, 0);
                __builtin_amdgcn_global_load_lds((global_ptr)ws, (lds_ptr)wd, 16, 0, 0);
            } else {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_ptr)xd, 16, (int)xoff[u], (int)(2u * (unsigned)k0), 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_ptr)wd, 16, (int)woff[u],
                                                         (int)(2u * (unsigned)k0 * (unsigned)HD), 0, 0);
            }
        }
    };
    // operand offsets within a stage: x row (wave >> 1) * 32 + ln, columns (wave & 1) * 32 ...
    const int xr = (wave >> 1) * 32, wcol = (wave & 1) * 32;
    const int xfo = (xr + ln) * 128 + ((g ^ ((ln >> 1) & 7)) << 4);
    const int i16 = lane & 15, kr = 8 * g + (i16 >> 2);
    const int col = wcol + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
    const int wfo = XB + kr * 128 + (((col >> 3) ^ (4 * ((kr >> 1) & 1))) << 4) + ((col & 7) << 1);
    const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;

    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const int ns = TAIL ? (D + 63) / 64 : D / 64;
    const int ahead = ns < STAGES - 1 ? ns : STAGES - 1;
    for (int j = 0; j < ahead; ++j) request(j, j);
    auto all_slices = [&](auto is_v_) {
        constexpr bool IS_V = decltype(is_v_)::value;
        int stage = 0;
#pragma nounroll
        for (int j = 0; j < ns; ++j) {
            // slices j + 1 .. j + STAGES - 2 may be in flight, four requests each; loads return in order
            const int more = min(ns - 1 - j, STAGES - 2);
            if (more >= 3) __builtin_amdgcn_s_waitcnt(0x0070 | 12);
            else if (more == 2) __builtin_amdgcn_s_waitcnt(0x0070 | 8);
            else if (more == 1) __builtin_amdgcn_s_waitcnt(0x0070 | 4);
            else __builtin_amdgcn_s_waitcnt(0x0070);
            // behind the barrier the slice is in LDS for everyone, and everyone has read the one before
            // (its reads were waited for ahead of its MFMAs), whose stage takes slice j + STAGES - 1
            __builtin_amdgcn_s_barrier();
            const int free_stage = stage == 0 ? STAGES - 1 : stage - 1;
            if (j + STAGES - 1 < ns) request(j + STAGES - 1, free_stage);
            const unsigned char* base = lds + stage * STAGE;
            const unsigned waddr = lds_addr + (unsigned)(stage * STAGE + wfo);
            u32x4 xf[4];
            u32x2 lo[4], hi[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                xf[ks] = *(const u32x4*)(base + (xfo ^ (32 * ks)));
                asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo[ks]) : "v"(waddr), "n"(16 * ks * 128));
                asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi[ks]) : "v"(waddr), "n"((16 * ks + 4) * 128));
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): hand-written reads are not counted by the compiler
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const u32x4 wf = {lo[ks][0], lo[ks][1], hi[ks][0], hi[ks][1]};
                acc = IS_V ? mfma32(xf[ks], wf, acc) : mfma32(wf, xf[ks], acc);
            }
            stage = stage == STAGES - 1 ? 0 : stage + 1;
        }
    };
    if (!FLOAT_OUT && which == 2) all_slices(std::true_type{});
    else all_slices(std::false_type{});

    if constexpr (FLOAT_OUT) {
        // through LDS, so that 16 lanes store a row's 64 columns: from the accumulators it would be 32 bytes of a line at a time
        constexpr int PITCH = 64 + 4;
        float* const stage = (float*)lds;
        __builtin_amdgcn_s_barrier();  // everyone has read the last slice (and waited for that)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
            *(f32x4*)(stage + (xr + ln) * PITCH + wcol + 8 * r4 + 4 * g) = f32x4{acc[4 * r4], acc[4 * r4 + 1], acc[4 * r4 + 2], acc[4 * r4 + 3]};
        __syncthreads();
        float* o = (float*)(which == 0 ? qo : (which == 1 ? ko : vto));
        const int cl = (tid & 15) * 4, cc = c0 + cl, h = (int)divide((unsigned)cc, columns), l = cc - h * d;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = 16 * it + (tid >> 4), gr = i0 + row;
            if (gr >= N) break;
            const int item = (int)divide((unsigned)gr, items), i = gr - item * (int)items.d;
            *(f32x4*)(o + (((size_t)item * H + h) * items.d + i) * d + l) = *(const f32x4*)(stage + row * PITCH + cl);
        }
        return;
    }

    const int dsh = d == 128 ? 7 : 6;  // d is 64 or 128 on this path
    if (which != 2) {
        // A side = columns (four consecutive per register quad), B side = vectors
        const int i = i0 + xr + ln;
        const float qs = which ? 1.f : qscale;  // q is stored pre-multiplied (see launch_proj_mfma)
        if (i < N) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int cc = c0 + wcol + 8 * r4 + 4 * g, h = cc >> dsh, l = cc & (d - 1);
                *(u32x2*)((h16_t*)(which ? ko : qo) + (((size_t)bb * H + h) * Npad + i) * d + l) =
                    u32x2{pack_f16_sat(acc[4 * r4] * qs, acc[4 * r4 + 1] * qs),
                          pack_f16_sat(acc[4 * r4 + 2] * qs, acc[4 * r4 + 3] * qs)};
            }
        }
    } else {
        // A side = vectors (four consecutive key slots per register quad), B side = columns; the tile
        // is one 64-key block, in which vectors past n are stored as zeros
        const int cc = c0 + wcol + ln, h = cc >> dsh, l = cc & (d - 1);
        h16_t* blk = (h16_t*)vto + ((((size_t)bb * H + h) * (Npad >> 6) + (i0 >> 6)) * d + l) * 64;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int r64 = xr + 8 * r4 + 4 * g, left = N - (i0 + r64);
            *(u32x2*)(blk + ((r64 & 48) | vt_slot16(r64 & 15))) =
                u32x2{pack_f16_sat(left > 0 ? acc[4 * r4] : 0.f, left > 1 ? acc[4 * r4 + 1] : 0.f),
                      pack_f16_sat(left > 2 ? acc[4 * r4 + 2] : 0.f, left > 3 ? acc[4 * r4 + 3] : 0.f)};
        }
    }
}

// The stored q carries the score scale and the change to base-2 exponentials:
// q' = q * scale * log2(e), applied to the fp32 accumulator before the one rounding to
// half precision, so that the attention kernels get base-2 scores straight out of the MFMA.
inline float q_prescale(const Problem& pb) { return pb.scale * 1.4426950408889634f; }

template <int BX, int BW, int WR, int WC, bool TRI = false>
hipError_t launch_dma(const Problem& pb, const bf16_t* X, const bf16_t* Wq, const bf16_t* Wk, const bf16_t* Wv,
                      h16_t* q, h16_t* k, h16_t* vt, hipStream_t s)
{
    const float qscale = q_prescale(pb);
    const int* lens = pb.noskip ? nullptr : pb.lens;
    const TileMap tm = tile_map(pb, BX, BW, pb.no_q ? 2 : 3, lens != nullptr);
    const int grid = ((tm.n_tiles + 7) / 8) * 8;
    if (pb.D % 64 == 0)
        hipLaunchKernelGGL((proj_dma_kernel<BX, BW, WR, WC, TRI, false>), dim3(grid), dim3(64 * WR * WC), 0, s, pb.B, pb.N, pb.Npad,
                           pb.D, pb.H, pb.d, X, Wq, Wk, Wv, q, k, vt, tm, qscale, lens, pb.skip_rows, pb.no_q, pb.row0, pb.counters);
    else
        hipLaunchKernelGGL((proj_dma_kernel<BX, BW, WR, WC, TRI, true>), dim3(grid), dim3(64 * WR * WC), 0, s, pb.B, pb.N, pb.Npad,
                           pb.D, pb.H, pb.d, X, Wq, Wk, Wv, q, k, vt, tm, qscale, lens, pb.skip_rows, pb.no_q, pb.row0, pb.counters);
    return hipGetLastError();
}

hipError_t launch_small(const Problem& pb, const bf16_t* X, const bf16_t* Wq, const bf16_t* Wk, const bf16_t* Wv,
                        h16_t* q, h16_t* k, h16_t* vt, hipStream_t s)
{
    const float qscale = q_prescale(pb);
    const int* lens = pb.noskip ? nullptr : pb.lens;
    const TileMap tm = tile_map(pb, 64, 64, pb.no_q ? 2 : 3, lens != nullptr);
    const int grid = ((tm.n_tiles + 7) / 8) * 8;
    const FastDiv none = {1u, 0u, 0u};
    const bool tail = pb.D % 64 != 0;
    auto* const kernel = ring_of_three((long)pb.B * ((pb.N + 63) / 64) * tm.tiles_w)
                             ? (tail ? proj_small_kernel<3, true, false> : proj_small_kernel<3, false, false>)
                             : (tail ? proj_small_kernel<5, true, false> : proj_small_kernel<5, false, false>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, pb.B, pb.N, pb.Npad, pb.D, pb.H, pb.d, X, Wq, Wk, Wv, q, k, vt, tm,
                       qscale, lens, pb.skip_rows, pb.no_q, pb.row0, pb.counters, none, none);
    return hipGetLastError();
}

template <int BT>
hipError_t launch_bt(const Problem& pb, const bf16_t* X, const bf16_t* Wt, h16_t* q, h16_t* k, h16_t* vt,
                     hipStream_t s)
{
    const float qscale = q_prescale(pb);
    const TileMap tm = tile_map(pb, BT, BT, 3, false);
    const int grid = ((tm.n_tiles + 7) / 8) * 8;
    hipLaunchKernelGGL(proj_mfma_kernel<BT>, dim3(grid), dim3(256), 0, s, pb.B, pb.N, pb.Npad, pb.D, pb.H, pb.d, X, Wt,
                       q, k, vt, tm, qscale, pb.noskip ? nullptr : pb.lens, pb.skip_rows, pb.no_q, pb.row0);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose_w(const Problem& pb, const bf16_t* Wq, const bf16_t* Wk, const bf16_t* Wv, bf16_t* Wt,
                              hipStream_t s)
{
    const int HD = pb.H * pb.d;
    const dim3 grid(HD / 64, (pb.D + 63) / 64, 3);
    hipLaunchKernelGGL(transpose_w_kernel, grid, dim3(256), 0, s, pb.D, HD, Wq, Wk, Wv, Wt, pb.counters);
    return hipGetLastError();
}

// Whether the projection reads the weights where the caller has them (no W^T, no re-layout kernel):
// 16-byte aligned weights for the 16-byte copies.
bool proj_reads_weights_in_place(const Problem& pb, const bf16_t* Wq, const bf16_t* Wk, const bf16_t* Wv)
{
    const bool aligned16 = ((reinterpret_cast<uintptr_t>(Wq) | reinterpret_cast<uintptr_t>(Wk) |
                             reinterpret_cast<uintptr_t>(Wv)) & 15) == 0;
    return pb.D % 8 == 0 && aligned16;
}

// The float path's products of bfloat16 storage, where X and the weights come in whole 16-byte pieces and
// the columns in whole 64s; false: not such a product.  W[0 .. count-1] -> out.
bool launch_proj_small_float(const Problem& pb, const bf16_t* X, const bf16_t* const* W, float* const* out, int count,
                             hipStream_t s)
{
    const int HD = pb.H * pb.d;
    const long M = (long)pb.B * pb.N;
    uintptr_t bits = reinterpret_cast<uintptr_t>(X);
    for (int m = 0; m < count; ++m) bits |= reinterpret_cast<uintptr_t>(W[m]);
    if (pb.D % 8 != 0 || HD % 64 != 0 || pb.d % 4 != 0 || (bits & 15) != 0 || M > 0x7fffffffL - 64) return false;
    Problem rows = pb;  // all vectors as one item
    rows.B = 1;
    rows.N = (int)M;
    rows.Npad = (int)((M + 63) / 64 * 64);
    const TileMap tm = tile_map(rows, 64, 64, count, false);
    const int grid = ((tm.n_tiles + 7) / 8) * 8;
    const bf16_t* w[3] = {W[0], W[count > 1 ? 1 : 0], W[count > 2 ? 2 : 0]};
    float* o[3] = {out[0], out[count > 1 ? 1 : 0], out[count > 2 ? 2 : 0]};
    const FastDiv items = fast_div((unsigned)pb.N), columns = fast_div((unsigned)pb.d);
    const bool tail = pb.D % 64 != 0;
    auto* const kernel = ring_of_three(tm.n_tiles)
                             ? (tail ? proj_small_kernel<3, true, true> : proj_small_kernel<3, false, true>)
                             : (tail ? proj_small_kernel<5, true, true> : proj_small_kernel<5, false, true>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, 1, rows.N, rows.Npad, pb.D, pb.H, pb.d, X, w[0], w[1], w[2], o[0], o[1],
                       o[2], tm, 1.f, nullptr, false, false, nullptr, pb.counters, items, columns);
    return true;
}

hipError_t launch_proj_mfma(const Problem& pb, const bf16_t* X, const bf16_t* Wq, const bf16_t* Wk,
                            const bf16_t* Wv, const bf16_t* Wt, h16_t* q, h16_t* k, h16_t* vt, hipStream_t s)
{
    // Tile by the number of tiles that hold a vector and by d_model.  Measured (us; 128 x 128,
    // 256 x 256, 128 x 256 with two workgroups per CU; rows x d_model -> columns):
    //   8192 x 768 -> 2304 (288)   36.4 / 45.2 / 36.1     16384 x 768 -> 2304 (576)    61 / 70 / 57
    //   8192 x 1024 -> 3072 (384)  52 / 55 / 48           65536 x 1024 -> 3072 (3072)  435 / 374 / 377, with key
    //   4096 x 4096 -> 12288 (768) 344 / 301 / 310        lengths 338 / 309 / 282, packed 266 / 249 / 224
    //   4096 x 4096 -> 6144 (384)  182 / - / 165          7168 x 1536 -> 6144 (672)    - / 126 / 124
    //                                                     7168 x 1984 -> 6144 (672)    - / 155 / 155
    // A workgroup's prologue and epilogue take as long as five slices and are hidden by the CU's other one, if
    // there is one; 256 x 256 reads the least per product, which decides when d_model is long.  No tile mixes
    // columns of two matrices.
    const int HD = pb.H * pb.d;
    const long t256 = HD % 256 == 0 ? (long)pb.B * ((pb.N + 255) / 256) * ((pb.no_q ? 2L : 3L) * HD / 256) : 0;
    if (proj_reads_weights_in_place(pb, Wq, Wk, Wv)) {  // operands go straight to LDS
        // Few tiles: 64 x 64 ones, up to two to a CU.  Measured (us, 128 x 128 / 64 x 64, by the number of 64 x 64 tiles), the kernel
        // at d_model 768: 144 11.3 / 9.3, 288 11.8 / 11.2, 576 12.9 / 13.7, 900 15.8 / 17.4; whole calls of 128 to 640 rows at d_model
        // 4096: -> 3072 columns 288 37.8 / 30.9, 384 38.9 / 36.1, 432 37.9 / 31.8; -> 4608 288 38.9 / 31.8, 360 40.2 / 38.9, 432 38.5 / 35.1; ->
        // 6144 288 34.6 / 28.0, 384 37.7 / 33.5, 480 40.3 / 41.2; -> 9216 288 38.9 / 35.8, 432 39.6 / 36.9; -> 2304 360 43.8 / 40.0.
        // Columns not in 128s have no other tiles: 8192 x 960 -> 2880 78 us, 32768 x 1024 -> 2880 322, 32768 x 4096 -> 2880 1408.
        const long cols = (pb.no_q ? 2L : 3L) * HD;
        const long t64 = (long)pb.B * ((pb.N + 63) / 64) * (cols / 64);
        if (HD % 128 != 0 || t64 <= 512) return launch_small(pb, X, Wq, Wk, Wv, q, k, vt, s);
        const long t128x256 = HD % 256 == 0 ? (long)pb.B * ((pb.N + 127) / 128) * (cols / 256) : 0;
        // At long d_model 256 x 256 where its tiles, one to a CU, fill four fifths of their rounds of the chip (256 x 256 /
        // 128 x 256: 432 tiles 110 / 112, 576 157 / 140, d_model 2048).
        if (t256 >= 512 && pb.D >= 2048 && 5 * t256 >= 4 * 256 * ((t256 + 255) / 256))
            return launch_dma<256, 256, 2, 4>(pb, X, Wq, Wk, Wv, q, k, vt, s);
        if (t128x256 >= 640) return launch_dma<128, 256, 2, 2>(pb, X, Wq, Wk, Wv, q, k, vt, s);
        // One round of either: more 128 x 128 tiles than the chip holds at three per CU, and no more than 256 of 256 x 256 (two
        // of 128 x 256 to a CU).  Measured (128 x 128 two, three per CU / 128 x 256 / 256 x 256): d_model 768, 864 tiles 34.0 /
        // 35.6 / 29.2 / 29.5, 1024 40.2 / 43.1 / 33.7 / 33.2, 768 (still three per CU) 27.4 / 26.4 / 28.5 / 28.2; d_model 2048, 864 64.8
        // / 75.1 / 59.4 / 56.8.  With key lengths the tiles that are left are not known here.
        if (!pb.lens && t128x256 > 384 && t128x256 <= 512) {
            if (pb.D >= 2048 && t256 <= 256) return launch_dma<256, 256, 2, 4>(pb, X, Wq, Wk, Wv, q, k, vt, s);
            return launch_dma<128, 256, 2, 2>(pb, X, Wq, Wk, Wv, q, k, vt, s);
        }
        // 128 x 128 tiles, two or three workgroups to a CU: whichever needs the less in whole rounds of the chip, a
        // round of 768 taking 1.5 times one of 512.  Measured (three per CU over two, by tiles, at d_model 768 / 4096):
        // 540 0.90 / 0.92, 756 0.90 / 0.97, 798 1.05 / 1.22, 1008 1.01 / 1.15, 1080 0.92 / 1.01, 1296 0.93 / 0.98,
        // 1548 1.01 / 1.09, 1806 1.03 / 1.01, 2052 0.97 / 0.98, 2520 1.07 / 1.05, 3024 0.99 / 1.00, 3800 1.01 / 0.98 (at
        // d_model 256 1.05); from 5400 on rounds no longer count: 5700 0.96, 7300 0.95.  With key lengths the number of
        // tiles that are left decides, 0.85 to 0.9 where it lies between 512 and 768 and 1.1 to 1.2 elsewhere, and is not
        // known here: three for the counts whose tiles, some of them left out, mostly end up there.  Means over lengths
        // uniform in n / 32 .. n, n 128 to 2000, d_model 512 and 2048: 600 tiles 1.09, 672 1.02, 714 0.88, 768 0.97, 798 0.93,
        // 840 0.98, 864 0.97, 912 1.01, 960 1.04, 1008 1.07, 1104 1.06.
        const long live = (long)pb.B * ((pb.N + 127) / 128) * (cols / 128);
        const bool fewer_rounds = 3 * ((live + 767) / 768) <= 2 * ((live + 511) / 512);
        if (live > 5376 || (pb.lens ? live >= 680 && live <= 920 : fewer_rounds && live <= 3072))
            return launch_dma<128, 128, 2, 2, true>(pb, X, Wq, Wk, Wv, q, k, vt, s);
        return launch_dma<128, 128, 2, 2>(pb, X, Wq, Wk, Wv, q, k, vt, s);
    }
    if (HD % 128 == 0) return launch_bt<128>(pb, X, Wt, q, k, vt, s);
    return launch_bt<64>(pb, X, Wt, q, k, vt, s);
}

}  // namespace attnring
