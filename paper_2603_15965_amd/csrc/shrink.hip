// Grouped shrink:  t_p = x_{perm[p]} A_{c(p)}  for every routed sorted position p (the
// "x A_{r(i)}" factor of Eq. "pertok", evaluated group by group as in the paper's grouped
// GEMM over buckets).
//
// The step is HBM bound (2*rank flops per 2 bytes of x), so the kernel is organised around
// keeping many bytes of x in flight.  A work item is 32 consecutive sorted rows of one
// bucket.  Its 4 wavefronts split the K range four ways (a workgroup per 32 rows gives N/32
// workgroups, enough to cover the chip even at 4096 tokens) and each wavefront streams on
// its own, with no workgroup barrier inside the loop:
//   x    straight from HBM into the bf16 MFMA operand layout (row lane%16, 8 consecutive k
//        per lane: 4 lanes = 64 contiguous bytes per row and instruction), two 16-row blocks;
//   A_c  its k-slice, 32 k at a time, into a wavefront-private LDS buffer and back through
//        the LDS transpose read, which turns the row-major [k][rank] slab into the
//        "8 consecutive k per lane" operand;
//   a ring of kDepth such steps is in flight per wavefront (v_mfma_f32_16x16x32_bf16, fp32
//   accumulate).  The four partial sums are added in a fixed order through LDS.
//
// The result is written as two bf16 halves, t = hi + lo with hi = bf16(t) and
// lo = bf16(t - hi), laid out [N][2*rank] = [hi | lo], so the expand step can feed it to a
// bf16 MFMA as a K = 2*rank contraction against [B_c; B_c] without losing t's fp32 precision.
#include "shrink_body.h"

namespace molora {

namespace {

template <int NJ, int RB, int KW, int kDepth, bool SORT = false>
__global__ __launch_bounds__(64 * KW) void shrink_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ A,
    const int32_t *__restrict__ offsets, const int32_t *__restrict__ perm,
    uint16_t *__restrict__ t2, int d_in, int C, int rank, Mix mix, int N, SortArgs sort) {
    shrink_body<NJ, RB, KW, kDepth, false, SORT>(x, A, offsets, perm, t2, d_in, C, rank, mix, (int)blockIdx.x, N,
                                                 nullptr, sort);
}

template <int NJ, int RB, int KW>
void launch_row_items(const uint16_t *x, const uint16_t *A, const int32_t *offsets, const int32_t *perm, uint16_t *t2, int N,
                      int d_in, int C, int rank, Mix mix, hipStream_t s, unsigned blocks, SortArgs sort) {
    if (sort.r != nullptr)
        hipLaunchKernelGGL((shrink_kernel<NJ, RB, KW, 4, true>), dim3(blocks), dim3(64 * KW), 0, s, x, A, offsets, perm, t2,
                           d_in, C, rank, mix, N, sort);
    else
        hipLaunchKernelGGL((shrink_kernel<NJ, RB, KW, 4>), dim3(blocks), dim3(64 * KW), 0, s, x, A, offsets, perm, t2, d_in, C,
                           rank, mix, N, sort);
}

}  // namespace

namespace {
// Which kernel a shrink takes: 0 = the row-item kernel below (16 or 32 rows, every column), 1 = the
// streaming kernel (a workgroup per 64 rows of a bucket and 32 columns, K split over its 8 wavefronts, x
// staged as whole 128-byte lines), 2 or 4 = that kernel with K cut into so many slices over workgroups.
// Timed side by side on 2000 random shapes (65 .. 24576 rows, K 256 .. 14336 off the powers of two too, R 8 ..
// 128, 1 .. 400 buckets, level, skewed and single-bucket routing; launch sums, K slices with their reduction):
// the rule is 2.9 % behind the best of the four (geometric mean).
//   * Buckets far smaller than the 64-row tiles leave them empty, and with many buckets the workgroups of
//     those tiles are most of the launch (1638 x 11224, R 96, 203 buckets: items 89 us, streaming 169 us);
//     up to 128 buckets a long and wide A_c still pays (130 x 7680, R 128, 111 buckets: 40 / 22 us).
//   * A long chain of K against few workgroups, up to 2048 rows: K slices while the workgroups are few,
//     down to narrow intermediates (611 x 12032, R 16, 37 buckets: streaming 22.5, four slices 13.0 us; 761 x
//     5248, R 40 15.9 / 10.8 us).  Two slices only from K = 4096 on (more
//     rows: 6144), the second launch costs as much as they save below (1065 x 1248, R 128: 7.5 us in
//     one launch, 9.5 in two).
//   * Large batches whose buckets fill the tiles stream (16384 x 4096, R 32, 32 buckets: items 48, 37 us),
//     in slices where K is long (2350 x 12544, R 64, 2 buckets: 34.7 / 23.9 us in two).
//   * So do wide intermediates of other batches -- a row item reads its A_c, all columns of it, in one
//     wavefront chain (3200 x 2048, R 128, 16 buckets 18.4 / 11.4 us) -- and narrow ones with enough work
//     per compute unit, (64-row tiles) x (16-column blocks) x K, in at least 80 workgroups (3594 x 2560, R 32
//     in one bucket: 56 of them, items 8.5, streaming 11.3 us; 12800 x 1024, R 32, 16 buckets 13.1 / 9.4 us).
//     Short rows with half-used second column groups stay with the items (17652 x 288, R 48 9.1 / 12.8 us).
bool shrink_tiny(int64_t N, int64_t R) { return N <= kShrinkTinyMax && (R + 15) / 16 <= 2; }

int shrink_form(int64_t N, int d_in, int C, int64_t R) {
    int ks = small_batch_shrink_ksplit(N, d_in, C, (int)R);
    if (N <= 64) return ks;
    const int64_t a_c = d_in * R;
    if (C > 64 && N < 16 * (int64_t)C && (C > 128 || a_c < 550000)) return 0;
    if (ks == 2 && d_in < (N <= 2048 ? 4096 : 6144)) ks = 1;
    if (N <= 2048 && a_c >= (1 << 17)) return ks;
    if (N * (int64_t)d_in >= (1 << 24) && N >= 128 * (int64_t)C && (N + 63) / 64 * C <= 32768) return ks;
    const bool wide = R > 64;
    const bool filled = C <= 64 ? wide || N >= 16 * (int64_t)C : C <= 256 && N >= (R <= 32 ? 64 : 128) * (int64_t)C;
    if (!filled || wide) return filled;
    const int64_t tiles = N / 64 + (N < C ? N : C) / 2, groups = (R + 31) / 32;
    return tiles * groups >= 80 && (groups == 1 || R > 48 || d_in > 512) && tiles * ((R + 15) / 16) * d_in >= 250000;
}
}  // namespace

size_t shrink_scratch_bytes(int64_t N, int d_in, int C, int R) {
    if (N == 0) return 0;
    const int ks = shrink_tiny(N, R) ? 1 : shrink_form(N, d_in, C, R);
    return ks > 1 ? (size_t)ks * (size_t)N * (size_t)R * sizeof(float) : 0;
}

int shrink_scratch_peaks(int64_t N, int d_in, int C, int R, int64_t *peaks) {
    // where shrink_form changes its slices as a batch grows; the scratch grows with it in between
    const int64_t groups = (R + 31) / 32, four = 64 / groups, two = 128 / groups;
    const int64_t ends[kShrinkPeaks] = {four < 64 ? four : 64, two < 64 ? two : 64, 63, 64, 127, 64 * (four - C) + 63,
                                        64 * (two - C) + 63, 2048, 64 * (512 - (int64_t)C / 2), 64 * (32768 / (int64_t)C)};
    int n = 0;
    for (const int64_t e : ends) {
        const int64_t b = e < N ? e : N;
        if (b >= 1 && shrink_scratch_bytes(b, d_in, C, R) > 0) peaks[n++] = b;
    }
    return n;
}

bool sort_in_shrink_ok(int64_t N, int d_in, int C, int rank) {
    (void)d_in, (void)C;
    return N > 0 && N <= 64 && !shrink_tiny(N, rank);
}

// Sixteen targets per lane of a workgroup at most.  molora_apply of 250 random shapes, 65 .. 8192 tokens, 1 .. 1024
// buckets, level, skewed, single-target and run-structured, in front of a narrow layer: dispatch launch, then
// shrink 1, in one launch 0.896 (geometric mean), none slower by more than 2 %, also where every one of a
// thousand workgroups sorts (launch of 8192 x 2048, 8 buckets of rank 16: 6.9 + 10.6 -> 13.3 us; 4096 x 4096, 256 of rank
// 16 8.1 + 18.5 -> 21.4; 256 x 4096, 8 of rank 64 4.2 + 7.8 -> 8.2).  With twice the targets per lane it would be
// level: at 16384 tokens the dispatch launch takes 8.7 us.
// Every round of workgroups sorts, so there are two of them at most: 11600 random shapes in graphs, up to 4096 tokens
// 0.85 whatever the workgroups, above 0.95 .. 0.98 up to 480 of them, 0.99 at 490, 1.005 at 525, 1.016 beyond 540 (7531
// x 8, 61 buckets of rank 128 33 / 39 us).
bool sort_large_in_shrink(int64_t N, int d_in, int C, int R) {
    if (N <= 64 || N > sort_max(8)) return false;
    if (N <= sort_max(4)) return true;
    return shrink_form(N, d_in, C, R) > 0 && !shrink_four_waves(N, C) && (N / 64 + C / 2) * ((R + 31) / 32) <= 500;
}

hipError_t launch_shrink(const uint16_t *x, const uint16_t *A, const int32_t *offsets,
                         const int32_t *perm, uint16_t *t2, int64_t N, int d_in, int C, int rank,
                         Mix mix, hipStream_t s, float *scratch, SortArgs sort) {
    if (N == 0) return hipSuccess;
    if (sort.r != nullptr) {
        if (N <= 64 && (mix.k != 1 || !sort_in_shrink_ok(N, d_in, C, rank))) return hipErrorInvalidValue;
        if (!sort.offsets || !sort.perm) return hipErrorInvalidValue;
        if (N > 64 && (sort.err_flag != nullptr || !sort_large_in_shrink(N, d_in, C, (int)(mix.k * rank)))) return hipErrorInvalidValue;
        offsets = sort.offsets;  // what the reduction pass of a K-split shrink reads afterwards
        perm = sort.perm;
    }
    const int64_t R = (int64_t)mix.k * rank;
    const int nj = (mix.k * rank + 15) / 16;
    // a few work items only, narrow intermediate: 16 (8) wavefronts per 16-row item
    if (shrink_tiny(N, R)) {
        const unsigned blocks = (unsigned)((N + 15) / 16 + C);
        if (nj == 1)
            hipLaunchKernelGGL((shrink_kernel<1, 1, 16, 8>), dim3(blocks), dim3(1024), 0, s, x, A,
                               offsets, perm, t2, d_in, C, rank, mix, (int)N, SortArgs{});
        else
            hipLaunchKernelGGL((shrink_kernel<2, 1, 8, 8>), dim3(blocks), dim3(512), 0, s, x, A,
                               offsets, perm, t2, d_in, C, rank, mix, (int)N, SortArgs{});
        return hipGetLastError();
    }
    const int form = shrink_form(N, d_in, C, R);
    if (form > 0)  // (K slices only when scratch is there)
        return launch_small_batch_shrink(x, A, offsets, perm, t2, N, d_in, C, rank, mix, s, scratch, form, sort);
    // 32-row items when they still cover the chip twice, 16-row items otherwise
    const bool small_items = (N + 31) / 32 + C < 512;
    const int rows = small_items ? 16 : 32;
    const unsigned blocks = (unsigned)most_tiles(N, C + (sort.r != nullptr ? 1 : 0), rows);  // (and the tokens without adapter)
    // fewer items than compute units and a long K: 8 wavefronts split it (measured 11.3 us
    // against 14.9 us at 2048 tokens x 4096, 64 adapters; no gain once every unit has an item)
    const bool wide = (N + rows - 1) / rows + C <= 256 && d_in >= 4096;
#define MOLORA_SHRINK_ARGS x, A, offsets, perm, t2, (int)N, d_in, C, rank, mix, s, blocks, sort
#define MOLORA_SHRINK_CASE(NJ)                                 \
    case NJ:                                                   \
        if (small_items && wide)                               \
            launch_row_items<NJ, 1, (NJ <= 2 ? 8 : 4)>(MOLORA_SHRINK_ARGS); \
        else if (small_items)                                  \
            launch_row_items<NJ, 1, 4>(MOLORA_SHRINK_ARGS);    \
        else                                                   \
            launch_row_items<NJ, 2, 4>(MOLORA_SHRINK_ARGS);    \
        break;
    switch (nj) {
        MOLORA_SHRINK_CASE(1)
        MOLORA_SHRINK_CASE(2)
        MOLORA_SHRINK_CASE(3)
        MOLORA_SHRINK_CASE(4)
        MOLORA_SHRINK_CASE(5)
        MOLORA_SHRINK_CASE(6)
        MOLORA_SHRINK_CASE(7)
        MOLORA_SHRINK_CASE(8)
        default:
            return hipErrorInvalidValue;
    }
#undef MOLORA_SHRINK_CASE
#undef MOLORA_SHRINK_ARGS
    return hipGetLastError();
}

}  // namespace molora
