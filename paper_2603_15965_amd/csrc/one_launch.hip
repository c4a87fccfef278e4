// A small batch with a few narrow adapters in ONE launch (targets given, C * rank <= 32):
//
//     h_i = x_i W + (x_i A_{r(i)}) B_{r(i)}
//
// Such a call is bound by launches and by trips to memory, not by work: 256 x 256 -> 256 with four adapters of rank
// 8 took 5.5 us for dispatch and shrink and 6.4 for the GEMM, and takes 4.8 here.  Here every workgroup, RB * 16 tokens x 32 columns
// of W, carries the C * rank <= 32 columns of all adapters A through the same K loop, in token order (nothing has
// to be sorted), zeroes what is not the token's own adapter's, and multiplies the rest by the stacked B
// (C * rank rows of d_out) of its columns.  Every column group repeats the shrink of its tokens, which the rule
// below (one_launch_ok) keeps small.
//
// Eight wavefronts split K into contiguous ranges of steps of 32; x goes from memory straight into the
// operand layout, W and A through a private LDS slab and the transpose read.  The partial sums are added in
// wavefront order; the low-rank intermediate is carried as two bf16 halves, as everywhere.
#include "common.h"

namespace molora {

namespace {

constexpr int kOneWaves = 8, kOneThreads = 64 * kOneWaves;
constexpr int kOneCols = 32;   // columns of W per workgroup, and of all adapters (padded)

// RB: 16-row blocks of a workgroup; DEPTH: steps in flight per wavefront, one, two or, where it has more, four (a load
// for nothing costs its time in the address unit: 256 x 256 -> 256, one step per wavefront, 11.4 us with four in flight)
template <int RB, int DEPTH>
__global__ __launch_bounds__(kOneThreads) void one_launch_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ W, const uint16_t *__restrict__ A,
    const uint16_t *__restrict__ B, const int32_t *__restrict__ r, float *__restrict__ h, int N, int d_in, int d_out,
    int C, int rank) {
    constexpr int ROWS = 16 * RB;
    constexpr int SLAB_ROW = 2 * kOneCols * 2;           // bytes: 32 columns of A, then 32 of W
    constexpr int SLAB = 32 * SLAB_ROW;                  // a step's slab
    constexpr int PART = ROWS * kOneCols * 4;            // a wavefront's partial sums of either half
    constexpr int REGION = 2 * (SLAB > PART ? SLAB : PART);
    constexpr int T_ROW = 2 * kOneCols * 2 + 16;         // bytes: hi, lo of 32 columns (+16: bank shift)
    constexpr int B_ROW = kOneCols * 2;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kOneWaves * REGION + ROWS * T_ROW + 32 * B_ROW];
    __shared__ int32_t own_lds[ROWS];  // adapter of a row, -1: none
    unsigned char *t_lds = lds + kOneWaves * REGION, *b_lds = t_lds + ROWS * T_ROW;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int n0 = blockIdx.x * kOneCols, row0 = blockIdx.y * ROWS;
    const int R = C * rank;
    unsigned char *region = lds + wave * REGION;

    // the 32-byte chunk of column block `cb` (16 columns) of slab row `row`: rows 0-3 and 8-11 of a chunk, which a
    // transpose read takes together, lie in different banks
    auto slab_chunk = [](int cb, int row) { return (cb ^ (row & 3)) << 5; };

    // adapter of column `col` of the C * rank <= 32 (at most four of them, and no division)
    auto adapter_of = [&](int col) { return (col >= rank) + (col >= 2 * rank) + (col >= 3 * rank); };

    // ---- operands of a step ----
    const int steps = (d_in + 31) / 32, per = (steps + kOneWaves - 1) / kOneWaves;
    const int s_begin = min(wave * per, steps), s_end = min(s_begin + per, steps);
    // x through a buffer descriptor (at most 2 MB, one_launch_ok): a load past its end brings zeros
    const auto x_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x), 0, N * d_in * 2, 0x00020000);
    uint32_t xrow[RB];  // byte offsets
#pragma unroll
    for (int i = 0; i < RB; ++i) xrow[i] = (uint32_t)(min(row0 + i * 16 + l16, N - 1) * d_in) * 2;
    // a slab is 4 pieces of 64 x 16 bytes: piece m, lane -> slab row m * 8 + lane / 8, 8 columns lane % 8 of it
    const int s_row = lane >> 3, s_u = lane & 7;
    const bool is_a = s_u < 4;
    const int a_col = min(s_u * 8, R - 8), w_col = min(n0 + (s_u - 4) * 8, d_out - 8);
    const int a_c = adapter_of(a_col);
    const uint16_t *src = is_a ? A + (int64_t)a_c * d_in * rank + (a_col - a_c * rank) : W + w_col;
    const int pitch = is_a ? rank : d_out;
    const bool dead = is_a && s_u * 8 >= R;  // columns that no adapter has: zero
    u32x4 xg[DEPTH][RB], sg[DEPTH][4];
    // Loads are never predicated.  Addresses of W and A are clamped and their slab is masked; x past K and past the
    // wavefront's range comes from past the buffer, as zero (its own values there, against the zeros of the slab,
    // would make NaN of an infinity).  Against clamped addresses for x too, 40 shapes, launches in a graph: 0.989 of
    // the time (geometric mean; 256 x 256 -> 256 4.2 us both, 512 x 1160 -> 1024 14.5 / 14.0, 500 x 712 -> 1000 9.8 /
    // 10.0, at worst).  Zeroed in registers in every step instead: 20 % more with 64 rows and four steps, where
    // all registers are in use (6 are spilled); from a zero page: 3 % more in the shortest launches.
    auto load_step = [&](int slot, int s) {
        const int k0 = s * 32, kx = k0 + kg * 8;
        const uint32_t k_off = s < s_end && kx < d_in ? (uint32_t)kx * 2 : 0x80000000u;
#pragma unroll
        for (int i = 0; i < RB; ++i) xg[slot][i] = __builtin_amdgcn_raw_buffer_load_b128(x_buf, xrow[i] + k_off, 0, 0);
#pragma unroll
        for (int m = 0; m < 4; ++m) sg[slot][m] = *(const u32x4 *)(src + (int64_t)min(k0 + m * 8 + s_row, d_in - 1) * pitch);
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load_step(d, s_begin + d);  // (past the range: harmless)
    // the stacked B of this workgroup's columns, and the targets, on their way beside the first steps
    u32x4 bg{0, 0, 0, 0};
    if (tid < 128 && (tid >> 2) < R) bg = *(const u32x4 *)(B + (int64_t)(tid >> 2) * d_out + min(n0 + (tid & 3) * 8, d_out - 8));
    constexpr int IT = ROWS * kOneCols / 2 / kOneThreads;  // pairs of columns per thread of either half
    int own[IT];
#pragma unroll
    for (int j = 0; j < IT; ++j) own[j] = r[min(row0 + (tid + j * kOneThreads) / (kOneCols / 2), N - 1)];

    f32x4 acc[RB][4];  // column blocks: 0, 1 the adapters, 2, 3 W
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = s_begin; s0 < s_end; s0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int s = s0 + d;  // steps past the range meet an all-zero slab
            unsigned char *slab = region + (d & 1) * SLAB;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int row = m * 8 + s_row;
                const uint32_t ok = s < s_end && s * 32 + row < d_in && !dead ? 0xFFFFFFFFu : 0u;
                const u32x4 v = sg[d][m];
                *(u32x4 *)(slab + row * SLAB_ROW + slab_chunk(s_u >> 1, row) + (s_u & 1) * 16) =
                    u32x4{v[0] & ok, v[1] & ok, v[2] & ok, v[3] & ok};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = kg * 8 + (l16 >> 2);
                const unsigned char *p = slab + row * SLAB_ROW + slab_chunk(j, row) + (l16 & 3) * 8;
                const i16x4 lo = lds_read_tr16((const MOLORA_LDS void *)p);
                const i16x4 hi = lds_read_tr16((const MOLORA_LDS void *)(p + 4 * SLAB_ROW));
                const i16x8 b8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
                for (int i = 0; i < RB; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xg[d][i]), __builtin_bit_cast(bf16x8, b8),
                                                                        acc[i][j], 0, 0, 0);
            }
            if (s0 + DEPTH < s_end) load_step(d, s + DEPTH);  // (wave-uniform)
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- t of the tokens' own adapters: partial sums in wavefront order, other adapters' columns zero ----
    // acc[i][j][v] = [row i*16 + kg*4 + v][column j*16 + l16]; a wavefront's partial sums lie in its own region
    float *pa = (float *)region, *pw = (float *)(region + PART);
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) pa[(i * 16 + kg * 4 + v) * kOneCols + j * 16 + l16] = acc[i][j][v];
    if (tid < 128) *(u32x4 *)(b_lds + (tid >> 2) * B_ROW + (((tid >> 1) & 1) ^ ((tid >> 5) & 1)) * 32 + (tid & 1) * 16) = bg;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = tid + q * kOneThreads, row = e / (kOneCols / 2), col = e % (kOneCols / 2) * 2;
        const int c = own[q] >= 0 && own[q] < C ? own[q] : -1;
        const bool mine = col < R && adapter_of(col) == c;
        if (col == 0) own_lds[row] = c;
        uint32_t hi2 = 0, lo2 = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float t = 0.f;
#pragma unroll
            for (int w = 0; w < kOneWaves; ++w) t += ((const float *)(lds + w * REGION))[row * kOneCols + col + i];
            t = mine ? t : 0.f;
            const uint32_t hi = f32_to_bf16_bits(t);
            hi2 |= hi << (16 * i);
            lo2 |= f32_to_bf16_bits(t - bf16_bits_to_f32(hi)) << (16 * i);
        }
        *(uint32_t *)(t_lds + row * T_ROW + col * 2) = hi2;
        *(uint32_t *)(t_lds + row * T_ROW + kOneCols * 2 + col * 2) = lo2;
    }
    __syncthreads();

    // ---- the expand, a 16 x 16 block per wavefront, joins that wavefront's partial sums of x W ----
    // Adapter by adapter (at most four): the rows of B of the others count as zero, and a row takes the product of its
    // own adapter only, so that no value of another one reaches it, be it an infinity.
    f32x4 ex{0.f, 0.f, 0.f, 0.f};
    if (wave < 2 * RB) {
        const int i = wave >> 1, j = wave & 1, row = kg * 8 + (l16 >> 2);
        const unsigned char *p = b_lds + row * B_ROW + ((j ^ ((row >> 3) & 1)) << 5) + (l16 & 3) * 8;
        const i16x4 lo = lds_read_tr16((const MOLORA_LDS void *)p);
        const i16x4 hi = lds_read_tr16((const MOLORA_LDS void *)(p + 4 * B_ROW));
        const i16x8 b8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        bf16x8 t[2];
        int own_row[4];
#pragma unroll
        for (int half = 0; half < 2; ++half) t[half] = *(const bf16x8 *)(t_lds + (i * 16 + l16) * T_ROW + half * kOneCols * 2 + kg * 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) own_row[v] = own_lds[i * 16 + kg * 4 + v];
        for (int c = 0; c < C; ++c) {
            // (a lane's eight rows of B lie inside one adapter: the rank is a multiple of 8)
            const bf16x8 bc = __builtin_bit_cast(bf16x8, adapter_of(kg * 8) == c ? b8 : i16x8{0, 0, 0, 0, 0, 0, 0, 0});
            f32x4 e{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int half = 0; half < 2; ++half) e = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[half], bc, e, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) ex[v] = own_row[v] == c ? e[v] : ex[v];
        }
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bool here = wave == 2 * i + j;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                pw[(i * 16 + kg * 4 + v) * kOneCols + j * 16 + l16] = acc[i][2 + j][v] + (here ? ex[v] : 0.f);
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int e = tid + q * kOneThreads, row = e / (kOneCols / 2), col = e % (kOneCols / 2) * 2;
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kOneWaves; ++w)
#pragma unroll
            for (int i = 0; i < 2; ++i) sum[i] += ((const float *)(lds + w * REGION + PART))[row * kOneCols + col + i];
        if (row0 + row < N && n0 + col < d_out) {
            u32x2 v = {__float_as_uint(sum[0]), __float_as_uint(sum[1])};
            *(u32x2 *)(h + (int64_t)(row0 + row) * d_out + n0 + col) = v;
        }
    }
}

// rows per workgroup: 32 while that is one round of workgroups, else 64
inline int one_launch_rows(int64_t N, int d_out) {
    return (N + 31) / 32 * ((d_out + kOneCols - 1) / kOneCols) <= 256 ? 32 : 64;
}

}  // namespace

// One round of workgroups whose streams of A beside W are small.  molora_apply of 500 random shapes, 1 .. 512 tokens,
// 64 .. 4096 -> 64 .. 8192, C * rank <= 32, against the two launches these took before (through Python, whose
// call takes 9 us): 375 inside the line 0.753 (geometric mean), at worst 0.97; past it up to 1.3 with a K of 3000 and
// more, where the two launches cut K over workgroups, and 4 with several rounds of workgroups.  The launches alone, in a
// graph, 1368 shapes inside the line: 0.54.  Up to 32 tokens with a K past 1024 the two, which cut K there, come close: 4400
// shapes 0.94 with three or four adapters or more than 100000 of (workgroups x K), 0.82 with less, at worst 1.13 (one
// token, 1280 -> 8, four of rank 8 7.5 / 9.0 us); called one after the other these take 0.83 and 0.77 all the same.
bool one_launch_ok(int64_t N, int d_in, int d_out, int C, int rank) {
    if (N < 1 || N > 512 || (int64_t)C * rank > kOneCols || d_in > 2048) return false;
    const int rows = one_launch_rows(N, d_out);
    const int64_t wgs = (N + rows - 1) / rows * ((d_out + kOneCols - 1) / kOneCols);
    return wgs <= 256 && wgs * d_in <= 300000;
}

hipError_t launch_one(const uint16_t *x, const uint16_t *W, const uint16_t *A, const uint16_t *B, const int32_t *r,
                      float *h, int64_t N, int d_in, int d_out, int C, int rank, hipStream_t s) {
    if (N < 1 || (int64_t)C * rank > kOneCols || N * d_in >= (1 << 30)) return hipErrorInvalidValue;  // (x: 31-bit offsets)
    const int rows = one_launch_rows(N, d_out);
    const dim3 grid((unsigned)((d_out + kOneCols - 1) / kOneCols), (unsigned)((N + rows - 1) / rows));
    const int per = ((d_in + 31) / 32 + kOneWaves - 1) / kOneWaves;  // steps of a wavefront
#define MOLORA_ONE(RB, DEPTH) \
    launch_base_kernel(one_launch_kernel<RB, DEPTH>, grid, dim3(kOneThreads), 0, s, x, W, A, B, r, h, (int)N, d_in, d_out, C, rank)
    if (rows == 32) {
        if (per == 1) MOLORA_ONE(2, 1);
        else if (per == 2) MOLORA_ONE(2, 2);
        else MOLORA_ONE(2, 4);
    } else {
        if (per == 1) MOLORA_ONE(4, 1);
        else if (per == 2) MOLORA_ONE(4, 2);
        else MOLORA_ONE(4, 4);
    }
#undef MOLORA_ONE
    return hipGetLastError();
}

}  // namespace molora
