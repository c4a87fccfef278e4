// Fused base projection + grouped expand (Eq. "pertok"):
//
//     h[perm[p]][:] = x[perm[p]] W  +  t_p B_{c(p)}           for every sorted position p
//
// One bf16 MFMA GEMM over the rows in bucket order.  The grouped expand is not a second
// kernel: after the d_in-long K loop over (x, W) the same accumulators take the products of the
// low-rank intermediate t (as [hi | lo] bf16 halves) with the B_c of every bucket c that owns rows
// of the tile (the expand phase below).  h is then written once, in fp32, to the rows' original
// positions (the "scatter to original positions" of the paper's pipeline).  Rows past offsets[C]
// (tokens without adapter) take part in no such product.
//
// Tiling: BM x BN output tile per workgroup, WM x WN wavefronts, each owning a grid of
// 16x16 MFMA tiles (v_mfma_f32_16x16x32_bf16, fp32 accumulate).
//   x tile  [BM][BK]  16-byte chunks XOR-swizzled inside a row so that the operand read (one
//                     row per lane, ds_read_b128) is bank-conflict free;
//   W tile  [BK][BN]  exactly as it lies in HBM (K-major), 32-byte chunks swizzled by (k & 3);
//                     the LDS transpose read turns it into the k-contiguous operand, so W needs
//                     no packing pass and no transposed copy.
// Every K tile goes HBM -> LDS directly (global_load_lds_dwordx4: no staging registers; the
// gathered row address and the swizzle are applied on the global side, the LDS side is
// linear).  Whatever has to read as zero -- k past d_in, padding of the rank -- is fetched from a
// small all-zero page instead, so the K tail travels the same path as the full tiles.
// One main loop for two to four LDS stages, with the operand fragments of the next k-step
// prefetched into registers behind the MFMAs.  (Small batches, which are bound by streaming W
// once, have a kernel of their own in small_batch.hip; launch_fused_gemm chooses.)
// Workgroups are numbered so that the 8 XCDs (blockIdx % 8) each walk a compact group of
// tiles and share x rows / W columns in their own L2.
#include <math.h>
#include <type_traits>
#include <utility>

#include "common.h"
#include "lds_dma.h"

namespace molora {

namespace {

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

constexpr int kGroupM = 8;  // row tiles per scheduling group
// Consecutive tiles that an XCD takes at a time (two rounds of its 32 compute units): the eight XCDs then work
// on neighbouring groups of row tiles, and the x rows of a group come from HBM once for all of its column
// tiles.  With an eighth of all tiles, one after the other, to each XCD, the chip goes over all of x in every
// round, which the 256 MB behind the L2s do not hold when x is larger (launch of 16384 x 12288 -> 4096 1308 ->
// 1256 us; x 4096 -> 4096 464 -> 453 us; runs of 32: 1257 and 463, of 16: 1268 and 466 us).
constexpr int kXcdRun = 64;

// BM x BN output tile, WM x WN wavefronts, BK deep K tiles, STAGES LDS buffers.
template <int BM_, int BN_, int WM_, int WN_, int BK_, int STAGES_>
struct GemmCfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, BK = BK_, STAGES = STAGES_;
    static constexpr int NW = WM * WN, NT = 64 * NW;
    static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
    // A tile = x rows, B tile = W rows; a load instruction fills 1 KB = one "piece"
    static constexpr int A_RB = BK * 2, A_CPR = A_RB / 16, A_RPI = 64 / A_CPR;
    static constexpr int B_RB = BN * 2, B_CPR = B_RB / 16, B_RPI = 64 / B_CPR;
    static constexpr int A_PIECES = BM / A_RPI, B_PIECES = BK / B_RPI;
    static constexpr int LPW = (A_PIECES + B_PIECES) / NW;  // pieces (loads) per wavefront and tile
    static constexpr int A_BYTES = BM * A_RB, B_BYTES = BK * B_RB, STAGE = A_BYTES + B_BYTES;
    static constexpr int SLAB_PIECES = 16 / B_RPI;          // pieces of a slab, 16 rows of B
    static constexpr int BATCH_LPW = 4 * SLAB_PIECES / NW;  // loads per wavefront and batch of four slabs
    static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE + 9 * BM * sizeof(int32_t) + 16;
    static_assert(BK == 64, "the expand phase lays 32 columns of hi and of lo side by side in an x tile");
    static_assert(A_PIECES % NW == 0, "every wavefront loads as many x pieces");
    static_assert(BATCH_LPW * NW == 4 * SLAB_PIECES, "a batch's pieces split evenly over wavefronts");
    static_assert(LPW * NW == A_PIECES + B_PIECES && LPW >= 1, "pieces split evenly over wavefronts");
    static_assert(STAGES >= 2 && STAGES <= 4, "stages");
    static_assert(TM % 2 == 0 && TM >= 4 && (TN == 2 || TN == 4), "four x fragments in flight, bands of 32 rows in the epilogue");

    // Where the 32-byte chunk `chunk` (16 columns) of k-row `row` of the W tile lies in its LDS row.
    // All rows start at bank 0.  Lanes 0-31 of a transpose read, which the hardware serves together, take
    // one chunk of the k-rows 0-3 and 8-11 (or 4-7 and 12-15, ...): row & 3 sends the first four to the
    // four chunks of a 128-byte window, bit 3 of the row the others to the other window, and a cache
    // line's eight lanes of an LDS-direct load stay together.
    __device__ static __forceinline__ int swz_b(int chunk, int row) { return chunk ^ (row & 3) ^ ((row >> 1) & 4); }
    __device__ static __forceinline__ int swz_b_inv(int pos, int row) { return swz_b(pos, row); }
    // XOR applied to the 16-byte chunk index of an x-tile row
    // (ds_read_b128 serves 16 lanes at a time, rows 0-3 and 12-15 of one chunk and 4-11 of the next;
    // two rows share the 256 bytes of all banks)
    __device__ static __forceinline__ int swz_a(int row) { return (row >> 1) & 7; }
};

template <class Cfg>
// (two wavefronts per SIMD at least: with 512 registers to a wavefront the compiler keeps the accumulators in
// the second half of them and moves some there and back in every tile)
__global__ __launch_bounds__(Cfg::NT, 2) void fused_gemm_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ W, const uint16_t *__restrict__ B,
    const uint16_t *__restrict__ t2, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ perm, float *__restrict__ h, int N, int d_in, int d_out, int C,
    int rank, int tiles_m, int tiles_n, Mix mix) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK, NT = Cfg::NT, TM = Cfg::TM,
                  TN = Cfg::TN, STAGES = Cfg::STAGES;
    // (1 KB alignment: the operand reads XOR k-step bits into addresses relative to this base)
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int32_t *tile_perm = (int32_t *)(smem + STAGES * Cfg::STAGE);  // [BM] token per row, -1 = none
    int32_t *seg_lo = tile_perm + BM;  // buckets that own rows of the tile: their sorted-position ranges
    int32_t *seg_hi = seg_lo + BM;
    int32_t *nseg_p = seg_hi + BM;
    int32_t *seg_ad = nseg_p + 4;  // [BM][4] pool positions of the adapters of a bucket's tuple
    int32_t *seg_c = seg_ad + 4 * BM;  // [BM] the buckets' indices (the token-order intermediate is addressed by them)
    int32_t *row_c = seg_c + BM;       // [BM] bucket per row (token-order form only; 0 where there is none)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;

    // ---- tile of this workgroup: groups of kGroupM row tiles, all column tiles of one after the other ----
    const int total = tiles_m * tiles_n;
    // runs of kXcdRun tiles go to the XCDs in turn; what is left after the last whole round of them is
    // shared out evenly
    const int xcd = (int)(blockIdx.x % 8), in_xcd = (int)(blockIdx.x / 8);
    const int whole = total / (8 * kXcdRun) * kXcdRun;  // tiles per XCD in whole rounds
    const int share = (total - whole * 8 + 7) / 8;
    const int logical = in_xcd < whole ? (in_xcd / kXcdRun * 8 + xcd) * kXcdRun + in_xcd % kXcdRun
                                       : whole * 8 + xcd * share + in_xcd - whole;
    if (logical >= total) return;
    // Group g holds the row tiles g, g + ng, g + 2 ng, ... (at most kGroupM of them), not
    // kGroupM consecutive ones: the rows are gathered through perm, so consecutive row tiles
    // share nothing, but under a skewed routing the LAST row tiles are the ones crossed by many
    // small buckets (many slabs of B each), and consecutive grouping put them all on one XCD.
    const int ng = (tiles_m + kGroupM - 1) / kGroupM;
    const int q = tiles_m / ng, rem = tiles_m % ng;  // the first rem groups have q + 1 row tiles
    const int big = rem * (q + 1) * tiles_n;         // output tiles in those groups
    const int gm = logical < big ? q + 1 : q;
    const int rest = logical < big ? logical : logical - big;
    const int g = (logical < big ? 0 : rem) + rest / (gm * tiles_n);
    const int in_group = rest % (gm * tiles_n);
    const int tile_m = g + ng * (in_group % gm);
    const int tile_n = in_group / gm;
    const int n0 = tile_n * BN;
    // Sorted position of tile row r: blk_pos(r / 32) + r % 32.  The tile is BM consecutive rows, or,
    // when it crosses a bucket per 32-row block or more anyway (C against the row tiles), every
    // tiles_m-th 32-row block: the rows are gathered either way, and under a skewed routing the
    // long tail of small buckets (the end of the sorted order) is then spread over all row tiles
    // instead of making the last ones wait for a hundred B_c, a megabyte from HBM (zipf(1.1), 256
    // buckets of rank 16: 4096 x 4096 -> 4096 158 -> 124 us, 16384 rows 519 -> 473 us; level routing
    // 128 -> 123 us).
    const bool strided = (int64_t)C * 32 >= (int64_t)tiles_m * BM;
    const int blk0 = strided ? tile_m * 32 : tile_m * BM, blk_step = strided ? tiles_m * 32 : 32;
    auto blk_pos = [&](int k) __attribute__((always_inline)) { return blk0 + k * blk_step; };
    auto row_pos = [&](int r) __attribute__((always_inline)) { return blk_pos(r >> 5) + (r & 31); };

    const int R = mix.k * rank;  // width of a bucket's intermediate (k adapters side by side)
    const int two_r = 2 * R;
    const int nkf = d_in / BK;              // full K tiles
    const int nkb = (d_in + BK - 1) / BK;   // K tiles of x.W, the last one possibly partial

    // ---- per-lane sources of this wavefront's load instructions ----
    // A stage is A_PIECES + B_PIECES pieces of 1 KB, x pieces (A_RPI rows each) first, then W
    // pieces (B_RPI k-rows each); load i of wavefront w is piece i*NW + w, so every wavefront
    // carries its share of the gathered x rows and of the W rows.
    // Rows past N and columns past d_out are clamped to valid memory: what they produce is
    // never stored.
    auto piece_of = [&](int i) __attribute__((always_inline)) { return i * Cfg::NW + wave; };
    auto slot_is_a = [&](int i) __attribute__((always_inline)) { return i < Cfg::A_PIECES / Cfg::NW; };  // a compile-time fact
    // geometry of load i of this wavefront: x piece -> (tile row, 8-k chunk index after the
    // swizzle); W piece -> (k-row, global column).  Recomputed where needed instead of kept in
    // registers: only the special tiles and the set-up use it.
    auto slot_geom = [&](int i, int &row, int &col) __attribute__((always_inline)) {
        if (slot_is_a(i)) {
            row = piece_of(i) * Cfg::A_RPI + lane / Cfg::A_CPR;
            col = (lane % Cfg::A_CPR) ^ Cfg::swz_a(row);
        } else {
            row = (piece_of(i) - Cfg::A_PIECES) * Cfg::B_RPI + lane / Cfg::B_CPR;
            const int pos = lane % Cfg::B_CPR;
            // this lane fills 16-byte position pos of the LDS row, i.e. half pos & 1 of physical
            // 32-byte chunk pos >> 1, which holds the logical chunk given by swz_b's inverse
            const int u16 = (Cfg::swz_b_inv(pos >> 1, row) << 1) | (pos & 1);
            col = min(n0 + u16 * 8, d_out - 8);
        }
    };
    uint32_t off_g[Cfg::LPW];  // full tiles: byte offset from the scalar base
#pragma unroll
    for (int i = 0; i < Cfg::LPW; ++i) {  // W pieces (the x pieces need the row table, below)
        int row, col;
        slot_geom(i, row, col);
        off_g[i] = slot_is_a(i) ? 0u : (uint32_t)(((int64_t)row * d_out + col) * 2);
    }
    // scalar bases of the full tiles, advanced per tile (x and W are < 4 GiB each)
    const unsigned char *a_base = (const unsigned char *)x;
    const unsigned char *b_base = (const unsigned char *)W;
    const int64_t b_step = (int64_t)BK * d_out * 2;

    auto issue_one = [&](unsigned char *stage, int i) __attribute__((always_inline)) {  // i-th load of a full tile
        load_to_lds16(slot_is_a(i) ? a_base : b_base, off_g[i], stage + piece_of(i) * 1024);
    };
    // The x part (want_a) and / or the W part (want_b) of base tile T < nkb; a partial last
    // tile computes a source per lane, k past d_in reads from the zero page.  Each part must
    // be issued in ascending tile order (the fast form advances its base).
    auto issue_base_parts = [&](unsigned char *stage, int T, bool want_a, bool want_b) __attribute__((always_inline)) {
        if (T < nkf) {
#pragma unroll
            for (int i = 0; i < Cfg::LPW; ++i)
                if (slot_is_a(i) ? want_a : want_b) issue_one(stage, i);
            if (want_a) a_base += BK * 2;
            if (want_b) b_base += b_step;
            return;
        }
        const uint16_t *zero = (const uint16_t *)g_zero_page;
#pragma unroll
        for (int i = 0; i < Cfg::LPW; ++i) {
            if (!(slot_is_a(i) ? want_a : want_b)) continue;
            const uint16_t *src;
            int row, col;
            slot_geom(i, row, col);
            if (slot_is_a(i)) {
                const int k = T * BK + col * 8;
                const int tok = tile_perm[row];
                src = (k < d_in) ? x + (int64_t)(tok >= 0 ? tok : 0) * d_in + k : zero;
            } else {
                const int k = T * BK + row;
                src = (k < d_in) ? W + (int64_t)k * d_out + col : zero;
            }
            load_to_lds16_ptr(src, stage + piece_of(i) * 1024);
        }
    };
    // With two stages every wait of the main loop is for all outstanding loads, so the order in
    // which the first tiles' pieces are issued is free: their W pieces, which depend on nothing
    // the dispatch step produced, go out before the tables are even read.
    const bool early_w = STAGES == 2 && nkb >= STAGES;
    if (early_w) {
#pragma unroll
        for (int T = 0; T < STAGES; ++T) issue_base_parts(smem + T * Cfg::STAGE, T, false, true);
    }

    // ---- per-tile tables: the rows' tokens and the buckets that own rows, both global reads
    // in flight together ----
    if (tid == 0) *nseg_p = 0;
    int32_t my_tok = -1, o_lo = 0, o_hi = 0;
    if (tid < BM && row_pos(tid) < N) my_tok = perm[row_pos(tid)];
    if (tid < C) {
        o_lo = offsets[tid];
        o_hi = offsets[tid + 1];
    }
    __syncthreads();  // the segment counter is zero
    if (tid < BM) tile_perm[tid] = my_tok;
    for (int i = tid + NT; i < BM; i += NT) tile_perm[i] = row_pos(i) < N ? perm[row_pos(i)] : -1;
    for (int c = tid; c < C; c += NT) {
        if (c != tid) {
            o_lo = offsets[c];
            o_hi = offsets[c + 1];
        }
        // does one of the tile's blocks hold rows of the bucket?  (blocks are counted in steps from
        // blk0; the first one that ends after the bucket's first row)
        const int k = max(0, (o_lo - blk0 - 31 + blk_step - 1) / blk_step);
        if (o_lo < o_hi && k < BM / 32 && blk_pos(k) < o_hi) {
            const int idx = atomicAdd(nseg_p, 1);
            seg_lo[idx] = o_lo;
            seg_hi[idx] = o_hi;
            seg_c[idx] = c;
            // slot table and tuple decoded once here, not inside the K loop
            for (int j = 0; j < mix.k; ++j) seg_ad[idx * 4 + j] = mix_adapter(mix, c, j);
        }
    }
    __syncthreads();
    const int nseg = __builtin_amdgcn_readfirstlane(*nseg_p);
    if (mix.t_dense) {
        for (int i = tid; i < BM; i += NT) {
            int c = 0;
            for (int sg = 0; sg < nseg && mix.C > 1; ++sg)  // (a few narrow adapters)
                if (row_pos(i) >= seg_lo[sg] && row_pos(i) < seg_hi[sg]) c = seg_c[sg];
            row_c[i] = c;
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < Cfg::LPW; ++i) {  // x pieces: the gathered row of every lane
        if (!slot_is_a(i)) continue;
        int row, col;
        slot_geom(i, row, col);
        const int tok = tile_perm[row];
        off_g[i] = (uint32_t)(((int64_t)(tok >= 0 ? tok : 0) * d_in + col * 8) * 2);
    }

    // `opaque` keeps the compiler from precomputing addresses (one per stage, k-step and fragment of
    // the main loop; those of the expand phase's loads) long before they are used, which costs
    // far more registers than it saves.
    auto opaque = [](uint32_t v) __attribute__((always_inline)) {
        asm volatile("" : "+v"(v));
        return v;
    };
    // ---- expand phase: what it loads ----
    // The rank is taken in chunks of 32.  For chunk q the x-side operand is one K tile of the rows'
    // own t, columns [hi of the chunk | lo of the chunk], whatever bucket a row belongs to, and the
    // W-side operand comes in slabs of 16 rows of a B_c (one slab serves hi and lo), four slabs to a
    // batch, in the place of a stage's W tile.  A 32-row block of the tile multiplies only the slabs
    // of the buckets that own rows of it.  (The form this replaces spent one K tile of 64 k on
    // every bucket of the tile, or on 2-4 buckets of rank 8 or 16, nearly all of it zeros when the
    // buckets are small.  Launch timer, before and now: 1333 x 2048 -> 6144, 40 buckets of rank 24
    // 66.7 / 62 us; 8192 x 2048 -> 6144, 64 tuples of rank 32 196 / 191 us, 512 tuples of rank 48
    // 382 / 291 us; 16384 x 12288 -> 4096, 32 buckets of rank 32 1325 / 1312-1322 us.)
    const int nq = nseg > 0 ? (R + 31) / 32 : 0;
    auto slabs_per_seg = [&](int q) __attribute__((always_inline)) { return R - q * 32 > 16 ? 2 : 1; };
    auto batches = [&](int q) __attribute__((always_inline)) { return (nseg * slabs_per_seg(q) + 3) / 4; };
    auto issue_t = [&](unsigned char *stage, int q) __attribute__((always_inline)) {  // x-side operand of chunk q
        const uint16_t *zero = (const uint16_t *)g_zero_page;
        const int ln = (int)opaque((uint32_t)lane);
#pragma unroll
        for (int i = 0; i < Cfg::LPW; ++i) {
            if (!slot_is_a(i)) continue;
            const int row = piece_of(i) * Cfg::A_RPI + ln / Cfg::A_CPR;
            const int col = (ln % Cfg::A_CPR) ^ Cfg::swz_a(row);
            const int j = q * 32 + (col & 3) * 8, lo_half = col >> 2, p = row_pos(row);
            const uint16_t *src = zero;
            if (p < N && j < R) {
                // token-order intermediate: the row of this token, the columns of its bucket's adapter
                if (mix.t_dense)
                    src = t2 + (int64_t)tile_perm[row] * (2 * mix.C * rank) + (lo_half * mix.C + row_c[row]) * rank + j;
                else
                    src = t2 + (int64_t)p * two_r + lo_half * R + j;
            }
            load_to_lds16_ptr(src, stage + piece_of(i) * 1024);
        }
    };
    // b-th batch of chunk q: all of its loads, whether its four places are used or not
    auto issue_slabs = [&](unsigned char *area, int q, int b) __attribute__((always_inline)) {
        const uint16_t *zero = (const uint16_t *)g_zero_page;
        const int sps = slabs_per_seg(q), ln = (int)opaque((uint32_t)lane);
        // the batch's buckets are among one group of 64: their adapters, one to a lane
        const int grp = (4 * b / sps) & ~63;
        const int ad_lane = seg_ad[min(grp + ln, nseg - 1) * 4];
        // a slab of 16 rows of one adapter, all there: one scalar base, the same lane offsets for all
        const bool whole = mix.k == 1 && (rank & 15) == 0 && d_out < (1 << 26);
#pragma unroll
        for (int u = 0; u < Cfg::BATCH_LPW; ++u) {
            const int v = u * Cfg::NW + wave;
            const int j = v / Cfg::SLAB_PIECES, piece = v % Cfg::SLAB_PIECES;  // place in the batch, piece of it
            const int row = piece * Cfg::B_RPI + ln / Cfg::B_CPR, pos = ln % Cfg::B_CPR;
            const int u16 = (Cfg::swz_b_inv(pos >> 1, row) << 1) | (pos & 1);
            const int col = min(n0 + u16 * 8, d_out - 8);
            const int i = min(4 * b + j, nseg * sps - 1);
            const int sg = sps == 2 ? i >> 1 : i, part = sps == 2 ? i & 1 : 0;
            unsigned char *dst = area + v * 1024;
            if (whole) {
                const int ad = __builtin_amdgcn_readlane(ad_lane, sg - grp);
                load_to_lds16(B + ((int64_t)ad * rank + q * 32 + part * 16) * d_out, (uint32_t)(row * d_out + col) * 2, dst);
                continue;
            }
            const int rr = q * 32 + part * 16 + row;     // row of the tuple's stacked B
            const int jj = mix.k > 1 ? min(rr / rank, mix.k - 1) : 0;   // which adapter of the tuple
            const int64_t brow = (int64_t)seg_ad[sg * 4 + jj] * rank + (rr - jj * rank);
            load_to_lds16_ptr(rr < R ? B + brow * d_out + col : zero, dst);
        }
    };
    // K tile T < nkb, or, as tile nkb, the first loads of the expand phase.  In ascending order.
    auto issue_tile = [&](unsigned char *stage, int T) __attribute__((always_inline)) {
        if (T < nkb) {
            issue_base_parts(stage, T, true, true);
        } else if (T == nkb && nq > 0) {
            issue_t(stage, 0);
            issue_slabs(stage + Cfg::A_BYTES, 0, 0);
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Operand fragments of v_mfma_f32_16x16x32_bf16: lane -> row (x) or column (W) lane % 16 of a block of
    // 16, k-group lane / 16 of 8 inside a k-step of 32.  Per-lane LDS addresses in stage 0:
    //   x fragment tm of k-step ks: row l16 + tm*16 of the wavefront's rows, 16-byte chunk (4*ks + kg) ^
    //     swizzle(row).  The swizzle looks at bits 1-3 of the row, the same for every tm: pa[ks] plus the
    //     read's immediate offset tm * 16 rows;
    //   W fragment tn: k-rows kg*8 + {0..3 | 4..7}, through the transpose read, of the swizzled 32-byte chunk
    //     of columns tn*16; the swizzle looks at bits 0, 1 and 3 of the row, the same for every k-step, which
    //     is again an immediate offset.
    // A tile's addresses are these plus its stage's offset.
    constexpr int KS = BK / 32;
    static_assert(Cfg::A_RB == 128 && KS == 2, "the XOR form of the x fragment address");
    const int kg = lane >> 4, l16 = lane & 15;
    const uint32_t smem0 = (uint32_t)(uintptr_t)(MOLORA_LDS unsigned char *)smem;
    const int a_row = wm * (BM / Cfg::WM) + l16, b_row = kg * 8 + (l16 >> 2);
    const uint32_t pa_row = smem0 + a_row * Cfg::A_RB;
    struct Addr {
        uint32_t a[KS], b[TN];
    };
    Addr p0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) p0.a[ks] = pa_row + (((4 * ks + kg) ^ Cfg::swz_a(a_row)) << 4);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
        p0.b[tn] = smem0 + Cfg::A_BYTES + b_row * Cfg::B_RB + (Cfg::swz_b(wn * TN + tn, b_row) << 5) + (l16 & 3) * 8;
    // Addresses of the tile being multiplied (cur) and of the next one (nxt).  With two or three stages the hot
    // loop is unrolled by their number, so each copy knows its stage and reads through the constants in
    // `at`; elsewhere the stage offset is added once per tile.  (Three stages, formed per tile and unrolled: 655 x
    // 8888 -> 10624 146 -> 133 us, 2464 x 11720 -> 2304 176 -> 171, 635 x 8192 -> 2048 42.7 -> 42.1.)
    constexpr bool kUnrolled = STAGES <= 3;
    Addr at[kUnrolled ? STAGES : 1], cur_rt, nxt_rt;
#pragma unroll
    for (int st = 0; st < (kUnrolled ? STAGES : 1); ++st) {  // (opaque: as a sum it is formed again for every read)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) at[st].a[ks] = st == 0 ? p0.a[ks] : opaque(p0.a[ks] + st * Cfg::STAGE);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) at[st].b[tn] = st == 0 ? p0.b[tn] : opaque(p0.b[tn] + st * Cfg::STAGE);
    }
    auto stage_addresses = [&](Addr &ad, int T) {
        const uint32_t so = (uint32_t)(T % STAGES) * Cfg::STAGE;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ad.a[ks] = opaque(p0.a[ks] + so);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) ad.b[tn] = opaque(p0.b[tn] + so);
    };
    auto read_x = [](uint32_t p) __attribute__((always_inline)) -> bf16x8 {
        return *(const MOLORA_LDS bf16x8 *)(uintptr_t)p;
    };
    auto read_w = [](uint32_t p) __attribute__((always_inline)) -> bf16x8 {
        const i16x4 lo = lds_read_tr16((const MOLORA_LDS void *)(uintptr_t)p);
        const i16x4 hi = lds_read_tr16((const MOLORA_LDS void *)(uintptr_t)(p + 4 * Cfg::B_RB));
        const i16x8 b8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, b8);
    };

    // ---- main loop ----
    // STAGES LDS stages (tile kt lives in stage kt % STAGES, tiles kt+1 .. kt+STAGES-1 are in flight).  A
    // tile is KS * TM places, one x fragment times the TN fragments of W each, k-step after k-step.  Behind
    // the MFMAs of a place the x fragment four places ahead is fetched from LDS, and in the last four
    // places of a k-step the W fragments of the next one, into the other of two sets, so the matrix pipe
    // never waits for LDS.  The workgroup barrier sits in front of the LAST four places of a tile: at that
    // point every wavefront holds the tile's last fragments in registers, so the stage can be refilled
    // (tile kt+STAGES) and the first fragments of tile kt+1 can be fetched while the last MFMAs of tile kt
    // still run.  Two stages are enough when a tile's MFMAs outlast the load latency (256 x 256 tiles);
    // smaller tiles need the next tiles further ahead.
    // The chip's power limit sets the clock under these products (16384 x 4096 -> 4096: 319 us on zeros, 427 on
    // normal data), so what an instruction costs in power counts.  On random operands in registers alone 16x16x32
    // sustains 2.10 PFLOP/s, 32x32x16, which this kernel took before, 1.86 (zeros 2.45 both): its accumulators are
    // read and written half as often per product.  16384 x 12288 -> 4096 1256 -> 1190 us, x 4096 453 -> 432, 8192 x
    // 2048 -> 6144 183 -> 174 us; 80 random shapes 4 % less.  W goes in as the first operand: a lane
    // then holds four consecutive columns of one row of h.
    constexpr int NA = 4, NP = KS * TM;
    static_assert(NP % NA == 0, "a place's x fragment is in register set place % NA in every tile");
    // Places that a refill's loads are spread over: behind the last loads of a short two-stage tile there is little time.
    // One, two, three and four places over 44 shapes of this configuration (600 .. 11300 rows, K 192 .. 4424), of the time
    // of the 32x32x16 form: inputs from HBM 0.996, 0.991, 0.993, 0.994 (geometric mean; at worst 1.019, 1.015, 1.026,
    // 1.045), from the Infinity Cache 0.986, 0.979, 0.977, 0.975 (4096 x 2048 -> 2048 42.1 -> 41.3, 41.1, 42.0, 43.0 and
    // 37.2 -> 35.6, 35.5, 35.6, 35.2 us).
    constexpr int kRefill = STAGES == 2 && TM == 4 ? 2 : NA;
    bf16x8 fa[NA], fb[2][TN];
    auto fetch_a = [&](const Addr &ad, int p) __attribute__((always_inline)) {
        fa[p % NA] = read_x(ad.a[p / TM] + (uint32_t)(p % TM) * (16 * Cfg::A_RB));
    };
    auto fetch_b = [&](const Addr &ad, int ks, int tn) __attribute__((always_inline)) {
        fb[ks & 1][tn] = read_w(ad.b[tn] + (uint32_t)(ks * 32 * Cfg::B_RB));
    };
    // loads return in order: tile T has landed once at most the loads of the `younger` tiles
    // issued after it are outstanding
    auto wait_tiles = [&](int younger) __attribute__((always_inline)) {
        if constexpr (STAGES >= 4) {
            if (younger >= 3) return wait_vmcnt<3 * Cfg::LPW>();
            if (younger >= 2) return wait_vmcnt<2 * Cfg::LPW>();
        }
        if constexpr (STAGES >= 3)
            if (younger >= 1) return wait_vmcnt<Cfg::LPW>();
        wait_vmcnt<0>();
    };
    auto stage_of = [&](int T) __attribute__((always_inline)) { return smem + (T % STAGES) * Cfg::STAGE; };
#pragma unroll
    for (int T = 0; T < STAGES; ++T) {
        if (early_w)
            issue_base_parts(smem + T * Cfg::STAGE, T, true, false);  // the W part is on its way
        else
            issue_tile(smem + T * Cfg::STAGE, T);
    }
    // (the expand phase's loads are not a tile's number: wait for everything when they are among these)
    wait_tiles(nkb >= STAGES ? STAGES - 1 : 0);
    wg_barrier();
#pragma unroll
    for (int p = 0; p < NA; ++p) fetch_a(p0, p);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) fetch_b(p0, 0, tn);

    // one K tile.  MORE: another tile follows.
    // REFILL: 0 = nothing to load, 1 = tile kt+STAGES is a full tile and its loads are
    // interleaved with the MFMAs, 2 = tile kt+STAGES is of any kind (or none), loaded in one go.
    // SP: the tile's stage when the caller knows it (unrolled hot loop), -1 otherwise.
    auto k_tile = [&](int kt, auto more_c, auto refill_c, auto sp_c) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more_c)::value;
        constexpr int REFILL = decltype(refill_c)::value;
        constexpr int SP = decltype(sp_c)::value;
        unsigned char *as = SP >= 0 ? smem + SP * Cfg::STAGE : stage_of(kt);
        const Addr &cur = SP < 0 ? cur_rt : at[SP < 0 ? 0 : SP];
        const Addr &nxt = SP < 0 ? nxt_rt : at[SP < 0 ? 0 : (SP + 1) % STAGES];
        if constexpr (MORE && SP < 0) stage_addresses(nxt_rt, kt + 1);
        static_for<NP * TN>([&](auto step) __attribute__((always_inline)) {
            constexpr int p = step / TN, j = step % TN, ks = p / TM, tm = p % TM;
            constexpr int late = p - (NP - NA);  // >= 0: behind the barrier
            if constexpr (MORE && late == 0 && j == 0) {
                wait_lds();  // this wavefront's reads of stage kt are complete
                // its part of tile kt+1 has landed; the tiles after it may still be in flight
                wait_tiles(REFILL == 1 || kt + STAGES <= nkb ? STAGES - 2 : 0);
                wg_barrier();  // ... and so has everyone else's; stage kt is free
                if constexpr (REFILL == 2) issue_tile(as, kt + STAGES);
            }
            constexpr int tn = tm & 1 ? TN - 1 - j : j;  // neighbouring products share an operand
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks & 1][tn], fa[p % NA], acc[tm][tn], 0, 0, 0);
            // W fragments of the next k-step, two to a place
            if constexpr (constexpr int q = (tm - (TM - NA)) * 2; q >= 0 && q < TN && j < 2) {
                if constexpr (ks + 1 < KS)
                    fetch_b(cur, ks + 1, q + j);
                else if constexpr (MORE)
                    fetch_b(nxt, 0, q + j);
            }
            // the refill's loads, in the places behind the barrier
            if constexpr (REFILL == 1 && late >= 0) {
                constexpr int per = (Cfg::LPW + kRefill - 1) / kRefill;  // loads per place
                static_for<per>([&](auto u) __attribute__((always_inline)) {
                    if constexpr ((TN > 2 ? 1 : 0) + u * (TN - 1) / per == j && late * per + u < Cfg::LPW) issue_one(as, late * per + u);
                });
            }
            if constexpr (j == TN - 1) {  // the place's x fragment is used up
                if constexpr (p + NA < NP)
                    fetch_a(cur, p + NA);
                else if constexpr (MORE)
                    fetch_a(nxt, p + NA - NP);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (REFILL == 1) {
            a_base += BK * 2;
            b_base += b_step;
        }
        if constexpr (MORE && SP < 0) cur_rt = nxt_rt;  // the next tile becomes the current one
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using RT = std::integral_constant<int, -1>;
    int kt = 0;
    if constexpr (kUnrolled) {  // the hot loop, as many tiles per round as there are stages
        for (; kt + STAGES - 1 + STAGES < nkf; kt += STAGES)
            static_for<STAGES>([&](auto st) __attribute__((always_inline)) { k_tile(kt + st, std::true_type{}, I1{}, st); });
    }
    stage_addresses(cur_rt, kt);
    for (; kt + STAGES < nkf; ++kt) k_tile(kt, std::true_type{}, I1{}, RT{});  // the hot loop
    for (; kt + 1 < nkb; ++kt) k_tile(kt, std::true_type{}, I2{}, RT{});       // last tiles, first loads of the expand
    k_tile(kt, std::false_type{}, I0{}, RT{});

    // ---- expand phase ----
    // Chunk q has its t in the x part of stage (nkb + q) % STAGES.  The batches, counted over all
    // chunks, go round the W parts of the stages; with two stages and one chunk also the x part
    // that holds no t.  While a batch is multiplied the next ones (two, with three places) travel:
    // B_c is on its first way from HBM, and a row tile crossed by a hundred small buckets waits
    // for nothing else.
    constexpr bool kInX = STAGES == 2 && Cfg::A_BYTES >= Cfg::B_BYTES;  // the x part of a stage holds a batch
    const int places = STAGES >= 3 || (kInX && nq == 1) ? 3 : 2;
    auto slab_area = [&](int e) __attribute__((always_inline)) {
        if constexpr (kInX)
            if (nq == 1) return (e % 3 == 0 ? stage_of(nkb) : stage_of(nkb + 1)) + (e % 3 == 2 ? 0 : Cfg::A_BYTES);
        return stage_of(nkb + e) + Cfg::A_BYTES;
    };
    struct Pos { int q, b, e; };  // chunk, batch of it, batch counted over all
    auto next_pos = [&](Pos p) __attribute__((always_inline)) {
        return p.b + 1 < batches(p.q) ? Pos{p.q, p.b + 1, p.e + 1} : Pos{p.q + 1, 0, p.e + 1};
    };
    // A fragment is [hi | lo] of 16 columns of t and its partner the slab's 16 rows of B twice: the
    // k-groups 0, 1 of a lane are hi columns, 2, 3 the lo ones, both against rows 0 .. 15.
    const uint32_t ea0 = pa_row + ((((kg >> 1) * 4 + (kg & 1)) ^ Cfg::swz_a(a_row)) << 4);
    const int kw = wm * (TM / 2);  // this wavefront's first 32-row block
    // Leave out the products of 16 rows of which the bucket has none.  Launches of random shapes in graphs, level and skewed
    // routing, rank 24 and more: 128 x 128 two-stage tiles 0.986 of the time (0.995 of the 32x32x16 form of this loop, 1.009
    // without), 192 x 256 0.994, 128 x 256 0.997 (one bucket for all tokens 1.004 at 128 x 128, at worst 1.03).  The other
    // tiles lose with one bucket what they gain with many (64 x 128 with rank 64 and more 1.02 / 0.99).
    constexpr bool kSkipHalf = TN == 4 && TM <= 6;
    // ranges of a group of 64 buckets, one to a lane, and which of them own rows of this wavefront
    int grp = -1, lo_lane = 0, hi_lane = 0;
    uint64_t mine = 0;
    Pos nx = nq > 0 ? next_pos(Pos{0, 0, 0}) : Pos{0, 0, 0};  // the next batch to load (0 is on its way)
    for (Pos at{0, 0, 0}; at.q < nq; at = next_pos(at)) {
        const int q = at.q, b = at.b, e = at.e;
        wait_lds();  // this wavefront's reads of the batch before are complete
        // its part of this batch has landed; the one after it, if loaded before, may be in flight
        constexpr int kBatch = Cfg::BATCH_LPW, kT = Cfg::A_PIECES / Cfg::NW;
        if (nx.e == e + 2) {
            if (b + 1 == batches(q)) wait_vmcnt<kBatch + kT>();
            else wait_vmcnt<kBatch>();
        } else {
            wait_vmcnt<0>();
        }
        wg_barrier();
        for (; nx.q < nq && nx.e < e + places; nx = next_pos(nx)) {
            if (nx.b == 0) issue_t(stage_of(nkb + nx.q), nx.q);
            issue_slabs(slab_area(nx.e), nx.q, nx.b);
        }
        const uint32_t ea = ea0 + (uint32_t)((nkb + q) % STAGES) * Cfg::STAGE;
        const uint32_t so_b = (uint32_t)(slab_area(e) - smem) - Cfg::A_BYTES - (kg >> 1) * (16 * Cfg::B_RB);  // (p0.b holds A_BYTES)
        uint32_t eb[TN];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) eb[tn] = p0.b[tn] + so_b;
        const int sps = slabs_per_seg(q);
        if (grp != ((4 * b / sps) & ~63)) {
            grp = (4 * b / sps) & ~63;
            const int i = min(grp + lane, nseg - 1);
            lo_lane = seg_lo[i];
            hi_lane = seg_hi[i];
            bool any = false;
#pragma unroll
            for (int k = 0; k < TM / 2; ++k) any |= hi_lane > blk_pos(kw + k) && lo_lane < blk_pos(kw + k) + 32;
            mine = __ballot(grp + lane < nseg && any);
        }
        for (int j = 0; j < 4; ++j) {
            const int i = 4 * b + j;
            const int sg = (sps == 2 ? i >> 1 : i) - grp, part = sps == 2 ? i & 1 : 0;
            if (i >= nseg * sps || !(mine >> sg & 1)) continue;
            const int lo = __builtin_amdgcn_readlane(lo_lane, sg), hi = __builtin_amdgcn_readlane(hi_lane, sg);
            bf16x8 bb[TN];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) bb[tn] = read_w(eb[tn] + (uint32_t)(j * 16 * Cfg::B_RB));
#pragma unroll
            for (int k = 0; k < TM / 2; ++k) {  // (both fragments of a 32-row block are read before either is waited for)
                const int pr = blk_pos(kw + k);
                if (hi <= pr || lo >= pr + 32) continue;
                i16x8 t[2];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    t[u] = __builtin_bit_cast(i16x8, read_x((ea ^ (uint32_t)(part * 32)) + (uint32_t)(2 * k + u) * (16 * Cfg::A_RB)));
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if constexpr (kSkipHalf)
                        if (hi <= pr + u * 16 || lo >= pr + u * 16 + 16) continue;
                    // rows of other buckets (and of none) count as zero
                    const int p = pr + u * 16 + l16;
                    const i16x8 own = p >= lo && p < hi ? t[u] : i16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
                        acc[2 * k + u][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb[tn], __builtin_bit_cast(bf16x8, own), acc[2 * k + u][tn], 0, 0, 0);
                }
            }
        }
    }

    // ---- epilogue: every row to its original position ----
    // acc[tm][tn][v]: row tm*16 + lane%16, column tn*16 + lane/16*4 + v.
    // The accumulators go through LDS one 32-row band per wavefront row at a time, so that
    // the global stores are 16 bytes per lane and a whole BN-wide row segment (1 KB) per
    // instruction: the rows are scattered over all of h by the permutation, and narrow
    // stores to scattered rows are what the memory system handles worst.
    constexpr int EP_STRIDE = BN * 4 + 32;           // bytes per staged row (+32: bank shift)
    constexpr int EP_CPR = BN / 4;                   // 16-byte chunks per row
    {
        constexpr int EP_ROWS = Cfg::WM * 32;
        static_assert(EP_ROWS * EP_STRIDE <= STAGES * Cfg::STAGE, "epilogue staging fits the stages");
        static_assert(EP_ROWS * EP_CPR % NT == 0, "every thread stores the same number of chunks of a band");
        constexpr int EP_IT = EP_ROWS * EP_CPR / NT;
#pragma unroll
        for (int band = 0; band < TM / 2; ++band) {
            __syncthreads();  // operand stages (or the previous band) are no longer read
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    *(f32x4 *)(smem + (wm * 32 + i * 16 + l16) * EP_STRIDE + (wn * (BN / Cfg::WN) + tn * 16 + kg * 4) * 4) = acc[band * 2 + i][tn];
            __syncthreads();
            // All of a thread's staged chunks and their rows' tokens are read before the first
            // store is issued: as a loop that reads one token, waits, reads one chunk, waits and
            // stores, the band took two LDS round trips per chunk, eight chunks in a row.
            int tok[EP_IT];
            f32x4 val[EP_IT];
#pragma unroll
            for (int j = 0; j < EP_IT; ++j) {
                const int it = tid + j * NT;
                const int r = it / EP_CPR, ch = it % EP_CPR;
                const int row = (r >> 5) * (BM / Cfg::WM) + band * 32 + (r & 31);
                tok[j] = tile_perm[row];
                val[j] = *(const f32x4 *)(smem + r * EP_STRIDE + ch * 16);
            }
#pragma unroll
            for (int j = 0; j < EP_IT; ++j) {
                const int col = n0 + ((tid + j * NT) % EP_CPR) * 4;
                if (tok[j] >= 0 && col < d_out)
                    // h is written once and not read again here: a streaming store keeps it
                    // from displacing x and W tiles in L2 (measured: -11 % at config 1)
                    __builtin_nontemporal_store(val[j], (f32x4 *)(h + (int64_t)tok[j] * d_out + col));
            }
        }
    }
}

// more than 64 KB of dynamic LDS has to be asked for, once per device (see common.h)
template <class Cfg>
struct GemmKernel {
    static inline LdsRegistrar lds{(const void *)fused_gemm_kernel<Cfg>, Cfg::LDS_BYTES};
};

template <class Cfg>
hipError_t launch_cfg(const uint16_t *x, const uint16_t *W, const uint16_t *B, const uint16_t *t2,
                           const int32_t *offsets, const int32_t *perm, float *h, int64_t N, int d_in,
                           int d_out, int C, int rank, Mix mix, hipStream_t s) {
    auto kern = fused_gemm_kernel<Cfg>;
    (void)&GemmKernel<Cfg>::lds;  // instantiates the registration
    const int tiles_m = (int)((N + Cfg::BM - 1) / Cfg::BM);
    const int tiles_n = (d_out + Cfg::BN - 1) / Cfg::BN;
    const int total = tiles_m * tiles_n;
    const unsigned blocks = (unsigned)(((total + 7) / 8) * 8);
    launch_base_kernel(kern, dim3(blocks), dim3(Cfg::NT), Cfg::LDS_BYTES, s, x, W, B, t2, offsets, perm, h,
                       (int)N, d_in, d_out, C, rank, tiles_m, tiles_n, mix);
    return hipGetLastError();
}

}  // namespace

// The row-tile configurations.  Tall tiles move the fewest operand bytes per product (a compute unit
// takes 64 bytes per cycle from its caches: at the full matrix rate 128 x 128 tiles need all of
// that, 256 x 256 tiles half), low ones fit the output closely and keep more units busy.
using Gemm64 = GemmCfg<64, 128, 1, 4, 64, 3>;     // two workgroups per compute unit
using GemmSmall = GemmCfg<128, 128, 2, 2, 64, 2>;  // two workgroups per compute unit
using GemmMid = GemmCfg<128, 128, 2, 4, 64, 4>;    // one: four stages and eight wavefronts in its place
using GemmWide = GemmCfg<128, 256, 2, 4, 64, 3>;
using Gemm192 = GemmCfg<192, 256, 2, 4, 64, 2>;
using GemmBig = GemmCfg<256, 256, 2, 4, 64, 2>;
using Gemm320 = GemmCfg<320, 256, 2, 4, 64, 2>;    // (8 registers spilled, 36 bytes a lane)
constexpr int kSmallBatchMax = 512;  // up to here the small-batch kernel takes operands of any size

bool fused_gemm_sizes_ok(int64_t N, int d_in, int d_out, int force_tile) {
    const bool tiled = force_tile == 128 || force_tile == 256 || (force_tile == 0 && N > kSmallBatchMax);
    if (!tiled) return true;  // the small-batch kernel checks its own offsets
    const uint64_t lim = uint64_t(1) << 32;
    return (uint64_t)N * (uint64_t)d_in * 2 < lim && (uint64_t)d_in * (uint64_t)d_out * 2 < lim;
}

namespace {
// Kernel and tile choice from static shapes only (no host read of the histogram): the smallest of
// the costs below.  Every configuration runs in rounds of (256 compute units x workgroups per
// unit) tiles; a round costs a start and an end, a time per K tile of 64 that grows from `k_few`
// to `k_few + k_full` with the share of the places in use, and the expand phase's batches and chunks.
// The coefficients are fitted (non-negative least squares of the relative error) to 270 shapes of
// 65 .. 16384 rows, 256 .. 12288 wide, 2 .. 64 adapters of rank 8 .. 64, every configuration forced on
// each (events around back-to-back launches, rotating inputs, us); the expand's were then lowered, the tiles' by
// a fifth, the streaming kernel's from 0.1 to 0.06, on 1600 random shapes of 1 .. 300 adapters up to rank 128,
// half of them with skewed routing.  Over those the choice is 1.25 % behind the best configuration (geometric
// mean; 4 % of them are more than 10 % behind, where the skew, which the rule cannot see, or a wide rank against a
// short K decides).  With the fitted ones it was 1.43 %, and up to 1.6x where 40 .. 200 adapters
// of rank 96 and more outweigh the product (311 x 256 -> 7168, 62 of rank 128: streaming 41, 64-row
// tiles 64 us; 528 x 1664 -> 5120, 180 of rank 128 88 / 121 us).  Fixed thresholds between 64, 128, 128 x 256
// and 256 rows are 8 % behind (5003 x 2728 -> 3176 in 256-row tiles, 260 of them for 256 units: 154 us,
// in 320-row tiles 109 us; 1333 x 2048 -> 6144 67 -> 55 us).
// These are fits of the kernels before their loop took 16x16x32 products, but for the row of 128 x 256: unrolled by three
// its loop gained more than the others, and of 8700 random shapes, every configuration forced with inputs from HBM and
// from the Infinity Cache, those that took 128 x 128 two-stage tiles were 3.3 and 3.5 % behind the best one, in half of
// them 128 x 256.  That row is lowered by 6 %: 4.6 % of the shapes go there, which take 0.954 (HBM) and 0.948 of the time
// (4096 x 2048 -> 2048 behind a shrink, W from HBM: 41 -> 35.5 us); 0.4 and 0.25 % of all are more than 3 % slower, one
// by 11 %, 2.9 % more than 3 % faster.  The choice is then 1.0 and 1.3 % behind the best configuration (1.2 and 1.6
// before; on 2300 other shapes the same).  A refit of all rows gains 0.7 % more on average and loses more than 3 % on
// more shapes: wide ranks and skewed routing against a short K.
struct GemmCost {
    int bm, bn, per_cu;
    double once, per_round, partial, k_round, k_few, k_full, expand;
};
constexpr GemmCost kGemmCosts[] = {
    {64, 128, 2, 4.7, 1.6, 0.0, 0.62, 0.28, 0.38, 1.11},
    {128, 128, 1, 1.9, 3.9, 3.6, 0.52, 0.37, 0.16, 0.91},
    {128, 128, 2, 0.0, 5.3, 5.2, 0.86, 0.55, 0.36, 1.02},
    {128, 256, 1, 0.0, 6.6, 6.5, 0.79, 0.545, 0.254, 1.06},
    {192, 256, 1, 2.1, 9.1, 4.5, 1.13, 0.85, 0.36, 1.29},
    {256, 256, 1, 3.7, 12.5, 4.2, 1.42, 0.98, 0.51, 1.54},
    {320, 256, 1, 4.9, 15.8, 5.8, 1.78, 1.18, 0.59, 1.58},
};
constexpr int kGemmConfigs = sizeof(kGemmCosts) / sizeof(kGemmCosts[0]);

double tiled_cost(const GemmCost &g, int64_t N, int d_in, int d_out, int C, int R) {
    const int64_t tiles = ((N + g.bm - 1) / g.bm) * ((d_out + g.bn - 1) / g.bn);
    const int64_t slots = (int64_t)256 * g.per_cu, full = tiles / slots;
    const double last = (double)(tiles % slots) / (double)slots, part = last > 0 ? 1 : 0;
    const double kt = (d_in + 63) / 64;
    const double segs = fmin((double)C, 1.0 + (double)g.bm * C / (double)N);  // buckets that own rows of a tile
    const double expand = segs * ((R + 15) / 16) / 4 + (R + 31) / 32;
    return g.once + g.per_round * (double)full + g.partial * part + kt * (g.k_round * (double)full + g.k_few * part + g.k_full * last) +
           g.expand * ((double)full + part) * expand;
}
// the streaming kernel: rounds of 256 workgroups, column groups of 64 (of 32 when that leaves at most
// 128) x row tiles of 64
double streaming_cost(int64_t N, int d_in, int d_out, int C, int R) {
    int64_t wgs = (int64_t)((d_out + 63) / 64) * ((N + 63) / 64);
    if (wgs <= 128) wgs *= 2;
    const double rounds = (double)((wgs + 255) / 256);
    const double segs = fmin((double)C, 1.0 + 64.0 * C / (double)N);
    return 0.6 + rounds * (5.6 + 3.26 * d_in / 1024.0 + 0.06 * segs * R / 16.0);
}
// -1: the streaming kernel, else the place in kGemmCosts
int gemm_choice(int64_t N, int d_in, int d_out, int C, int R) {
    const uint64_t lim = uint64_t(1) << 32;
    // one row tile always streams; so do operands beyond the tiled kernel's 32-bit offsets
    // (fused_gemm_sizes_ok refuses them above kSmallBatchMax)
    if ((N <= 64 || (N <= kSmallBatchMax && ((uint64_t)N * d_in * 2 >= lim || (uint64_t)d_in * d_out * 2 >= lim))))
        return -1;
    double best = N <= 4096 ? streaming_cost(N, d_in, d_out, C, R) : 1e30;
    int pick = -1;
    for (int i = 0; i < kGemmConfigs; ++i) {
        const double cost = tiled_cost(kGemmCosts[i], N, d_in, d_out, C, R);
        if (cost < best) {
            best = cost;
            pick = i;
        }
    }
    return pick;
}
}  // namespace

void fused_gemm_tile(int64_t N, int d_in, int d_out, int C, int R, int32_t *tile) {
    static constexpr int stages[kGemmConfigs] = {Gemm64::STAGES,   GemmMid::STAGES, GemmSmall::STAGES, GemmWide::STAGES,
                                                 Gemm192::STAGES, GemmBig::STAGES, Gemm320::STAGES};  // the order of kGemmCosts
    const int pick = gemm_choice(N, d_in, d_out, C, R);
    tile[0] = pick < 0 ? 64 : kGemmCosts[pick].bm;
    tile[1] = pick < 0 ? small_batch_cols(N, d_out) : kGemmCosts[pick].bn;
    tile[2] = pick < 0 ? 0 : stages[pick];
}

// force_tile: 0 = the choice below; 64 / 128 / 256 = that row-tile height whatever the shape
// (the tiling ablation compares the choice with fixed tiles).
hipError_t launch_fused_gemm(const uint16_t *x, const uint16_t *W, const uint16_t *B,
                             const uint16_t *t2, const int32_t *offsets, const int32_t *perm,
                             float *h, int64_t N, int d_in, int d_out, int C, int rank, Mix mix,
                             hipStream_t s, int force_tile) {
    if (N == 0) return hipSuccess;
    // the token-order intermediate is read by the kernels chosen below, for a batch of several row tiles
    if (mix.t_dense && (force_tile == 64 || N <= 64 || mix.k != 1)) return hipErrorInvalidValue;
#define MOLORA_GEMM_ARGS x, W, B, t2, offsets, perm, h, N, d_in, d_out, C, rank, mix, s
    if (force_tile == 64) return launch_small_batch_gemm(MOLORA_GEMM_ARGS);
    if (force_tile == 128) return launch_cfg<GemmSmall>(MOLORA_GEMM_ARGS);
    if (force_tile == 256) return launch_cfg<GemmBig>(MOLORA_GEMM_ARGS);
    switch (gemm_choice(N, d_in, d_out, C, mix.k * rank)) {  // the order of kGemmCosts
        case 0: return launch_cfg<Gemm64>(MOLORA_GEMM_ARGS);
        case 1: return launch_cfg<GemmMid>(MOLORA_GEMM_ARGS);
        case 2: return launch_cfg<GemmSmall>(MOLORA_GEMM_ARGS);
        case 3: return launch_cfg<GemmWide>(MOLORA_GEMM_ARGS);
        case 4: return launch_cfg<Gemm192>(MOLORA_GEMM_ARGS);
        case 5: return launch_cfg<GemmBig>(MOLORA_GEMM_ARGS);
        case 6: return launch_cfg<Gemm320>(MOLORA_GEMM_ARGS);
        default: return launch_small_batch_gemm(MOLORA_GEMM_ARGS);
    }
#undef MOLORA_GEMM_ARGS
}

}  // namespace molora
