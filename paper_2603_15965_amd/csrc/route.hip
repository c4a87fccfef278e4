// Learned top-1 routing (Sec. "Router Architecture", k = 1; linear gate of Table
// "tab:moe_adapter"):  r[i] = argmax_c sum_k x[i][k] G[k][c], lowest index on ties.
//
// The result has to be a deterministic function of the input bits, so every logit is the
// strict fp32 chain  acc <- fl(acc + x_k * g_k),  k ascending (the bf16 x bf16 product is
// exact in fp32, so fused and unfused steps round identically).  That chain is exactly what
// the fp32 matrix instruction v_mfma_f32_16x16x4_f32 computes: it walks its 4 k in order
// with one fp32 rounding per step, so a sequence of them is the scalar chain for 16 tokens
// x 16 targets at the full fp32 MFMA rate.  A chain cannot be split over k, so parallelism
// comes only from (token, target) blocks: one wavefront owns 16 tokens and NB blocks of 16
// targets; the TB wavefronts that share a token group take different target blocks and merge
// their winners at the end.
//
// What bounds it: a SIMD finishes one chain instruction (4 k of 16 x 16 logits) per 32 cycles,
// whether its chains belong to one wavefront or to two -- 13.7 us per 4096 k and chain -- and the
// fp32 matrix instructions leave no slot for vector instructions: each of those adds ~3 cycles,
// and one that stands BETWEEN two chain instructions ~10 more (measured, cycles per chain
// instruction: 32 bare, 53 with two vector instructions after each, 44 with sixteen after every
// eighth, 39 with two bf16 matrix instructions after every eighth; memory reads cost nothing).
// So the loop has hardly any vector instructions.  x goes straight from memory into registers, 16
// bytes per lane, a ring of kRing chunks of 32 k deep; G likewise, once per workgroup and slab of
// KS k, one slab ahead.  bf16 matrix instructions by constant 0/1 matrices bring both, four steps
// at a time, into the layout of the chain instruction (x[t][4s + kq] in lane (t, kq), G[4s + kq][c]
// in lane (c, kq)) and widen them to fp32 on the way: one product by 1 and zeros, exact for every
// finite value, denormals included.  The operands of G are shared through LDS, in the order the
// wavefronts read them back.  (A NaN or an infinity would spread over its 16 k and 32 targets: a
// wavefront that ends up with a NaN logit computes its chains again.  A call with one such value, in x or
// in G, takes 2 to 3 times as long: 16384 x 12288 x 32 targets 131 -> 355 us, 8192 x 2048 x 8 15.6 -> 45
// us.  One multiply-add after another, as it was, it took 8.8 ms and 0.55 ms.)
// Measured (events around back-to-back calls, rotating x; us, before: x regrouped through LDS with
// byte permutes and widened with shifts between the chain instructions, C not a multiple of 8
// fetched element by element): 16384 x 4096 x 32 targets 57 -> 44.5 (the chains alone: 27),
// 16384 x 12288 x 32 157 -> 119, 8192 x 2048 x 64 38 -> 28, 8192 x 2048 x 8 20 -> 17,
// 5003 x 2728 x 13 77 -> 21.
#include <type_traits>

#include "common.h"

namespace molora {

namespace {

constexpr int kRing = 8;        // chunks of x in flight per wavefront
constexpr int kXK = 32;         // k per chunk: one x load of 16 tokens x 64 bytes
constexpr int kSCK = kRing * kXK;  // k per unrolled super-chunk

// 16 bytes at any element's address
struct __attribute__((packed, aligned(2))) G8 {
    u32x4 v;
};

// NB target blocks per wavefront, TB wavefronts per token group, TGW token groups per workgroup
template <int NB, int TB, int TGW>
struct RouteCfg {
    static constexpr int NWV = TB * TGW, TOK_WG = TGW * 16;
    static constexpr int NBLK = NB * TB;   // 16-target blocks of a pass
    static constexpr int CW = NBLK * 16;   // targets per pass
    static constexpr int KS = NBLK <= 2 ? 256 : 512 / NBLK;  // k per G slab: at most 32 KB of operands
    static constexpr int FRAG = 1024;      // operands of four steps of one block: 64 lanes x 16 bytes
    static constexpr int SLAB = KS / 16 * NBLK * FRAG;  // [k / 16][block][lane]
    // A staging unit is one load and two products: 16 k x 32 targets, or 32 k x 16 targets (one
    // block).  A wavefront takes units of one pair of blocks, so that its constants are fixed.
    static constexpr int PAIRS = NBLK >= 2 ? NBLK / 2 : 1;
    static constexpr int UNITS = NBLK >= 2 ? KS / 16 : KS / 32;  // per pair
    static constexpr int UPW = UNITS * PAIRS / NWV;              // per wavefront
    static_assert(NWV % PAIRS == 0 && UPW * NWV == UNITS * PAIRS, "staging split");
    static_assert(kSCK % KS == 0, "slab boundaries fall on static positions of the super-chunk");
};

__device__ __forceinline__ void route_barrier() {
    // LDS-only workgroup barrier: the loads stay in flight across it
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The chains of 16 tokens and NB blocks of 16 targets with operands that are widened value by value: a chain instruction
// takes each of them into its own token or target only.  32 k at a time, GROUPS such groups in flight, all
// vector instructions of a group in front of its chain instructions.  Not inlined: the code costs
// the kernel's main loop registers otherwise (16384 x 4096 x 32 targets 43.1 -> 43.7 us).
//   xt: this lane's token; c: its target in the first block
template <int NB>
struct Chains {
    f32x4 acc[NB];
};
template <int NB>
__device__ __attribute__((noinline)) Chains<NB> route_chains_again(const uint16_t *xt, const uint16_t *G, int d_in, int C, int kq, int c) {
    constexpr int GROUPS = NB == 1 ? 4 : 3;
    const uint16_t *gt[NB];
    Chains<NB> r;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        gt[b] = G + kq * C + min(c + b * 16, C - 1);
        r.acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    u32x4 xr[GROUPS][4];
    uint16_t gr[GROUPS][8][NB];
    auto fetch = [&](int set, int k0) __attribute__((always_inline)) {  // (past the end: the last eight, or four rows, again)
#pragma unroll
        for (int i = 0; i < 4; ++i) xr[set][i] = *(const u32x4 *)(xt + min(k0 + 8 * i, d_in - 8));
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int b = 0; b < NB; ++b) gr[set][s][b] = gt[b][(int64_t)min(k0 + 4 * s, d_in - 4) * C];
    };
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) fetch(g, 32 * g);
    for (int k0 = 0; k0 < d_in; k0 += 32 * GROUPS) {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int kg = k0 + 32 * g;
            if (kg >= d_in) break;  // (uniform)
            float xv[8], gv[8][NB];
#pragma unroll
            for (int s = 0; s < 8; ++s) {  // x[t][kg + 4 s + kq]; k past the end adds +0
                const uint32_t ok = kg + 4 * s < d_in ? 0xFFFFFFFFu : 0u;
                const uint32_t two = ((kq & 2) ? xr[g][s >> 1][2 * (s & 1) + 1] : xr[g][s >> 1][2 * (s & 1)]) & ok;
                xv[s] = __uint_as_float((kq & 1) ? two & 0xFFFF0000u : two << 16);
#pragma unroll
                for (int b = 0; b < NB; ++b) gv[s][b] = bf16_bits_to_f32(gr[g][s][b] & ok);
            }
            fetch(g, kg + 32 * GROUPS);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    r.acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s], gv[s][b], r.acc[b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return r;
}

// ROWS8: C is a multiple of 8 (16-byte pieces of G's rows are aligned and end with the row).
// (At most 256 registers: where the chains are many, two wavefronts per SIMD take 87 us against 98
// with one, 16384 x 4096 x 64 targets.)
template <int NB, int TB, int TGW, bool ROWS8>
__global__ __launch_bounds__(TB * TGW * 64, 2) void route_gate_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ G, int32_t *__restrict__ r,
    float *__restrict__ logits_out, int64_t N, int d_in, int C) {
    using K = RouteCfg<NB, TB, TGW>;
    constexpr int CW = K::CW, TOK_WG = K::TOK_WG;
    extern __shared__ __attribute__((aligned(16))) unsigned char route_lds[];  // two slabs

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int tb = wave % TB, tgw = wave / TB;  // target-block group, token group
    const int64_t tok_wave = (int64_t)blockIdx.x * TOK_WG + tgw * 16;

    // load side: lane (t = l16, cq = kq) fetches x[t][k0 + 8*cq .. +8)
    const int64_t tok = tok_wave + l16;
    const bool tok_ok = tok < N;
    const uint16_t *xrow = x + (tok_ok ? tok : 0) * (int64_t)d_in + kq * 8;  // + k0

    // one bf16 1.0 at inner index j of this lane's eight (none if j is outside)
    auto unit8 = [](int j) -> bf16x8 {
        u32x4 w = {0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i == j) w[i >> 1] = (i & 1) ? 0x3F800000u : 0x3F80u;
        return __builtin_bit_cast(bf16x8, w);
    };
    // x: D = P_h X^T, the raw chunk as the B operand (lane: token l16, k = 8 kq + j).  Row 4 q + v
    // of P_h picks k = 16 h + 4 v + q, so register v of lane (t, q) is the operand of step 4 h + v.
    const int ksel = 4 * (l16 & 3) + (l16 >> 2);
    bf16x8 sel_x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) sel_x[h] = unit8(h * 16 + ksel - kq * 8);

    float best[4];
    int bidx[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        best[v] = -__builtin_huge_valf();
        bidx[v] = 0x7FFFFFFF;
    }

    for (int c0 = 0; c0 < C; c0 += CW) {  // passes of up to CW targets
        f32x4 acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int cw = c0 + tb * NB * 16;  // first target of this wavefront

        // G: D = G_rows S, the raw rows as the A operand: lane l16 loads row ksel of 16 (so that
        // register v of lane (c, q) is the operand of step v, as above) at eight targets.  A pair of
        // blocks: the four kq take 32 targets; S picks 16 of them.  One block: kq 0, 1 take its 16
        // targets in the first 16 k, kq 2, 3 in the next; S picks the half.  An eight that would
        // pass the end of G's row starts earlier instead.
        constexpr bool PAIR = K::NBLK >= 2;
        const int pair = PAIR ? wave % K::PAIRS : 0, unit0 = wave / K::PAIRS;
        constexpr int UNIT_STEP = K::NWV / K::PAIRS, UNIT_K = PAIR ? 16 : 32;
        const int g_c8 = max(0, min(c0 + 32 * pair + 8 * (PAIR ? kq : kq & 1), C - 8));
        const int g_row = ksel + (PAIR ? 0 : 16 * (kq >> 1));
        const uint32_t g_off = (uint32_t)(g_row * C + g_c8) * 2;  // bytes from the unit's first row
        bf16x8 sel_g[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = c0 + 32 * pair + (PAIR ? 16 * i : 0) + l16;
            sel_g[i] = unit8(kq == 2 * i + (l16 >> 3) && c < C ? c - g_c8 : -1);
        }
        u32x4 greg[K::UPW];
        // the slab that starts at k0: this wavefront's units into registers
        auto g_load = [&](int k0) __attribute__((always_inline)) {
            // (a row to spare: with C < 8 an eight of G's last rows passes its end)
            if (k0 + K::KS + 8 <= d_in) {
                const unsigned char *p = (const unsigned char *)(G + (int64_t)(k0 + unit0 * UNIT_K) * C);
#pragma unroll
                for (int m = 0; m < K::UPW; ++m) {
                    if constexpr (ROWS8)
                        greg[m] = *(const u32x4 *)(p + g_off);
                    else
                        greg[m] = ((const G8 *)(p + g_off))->v;
                    p += (int64_t)(UNIT_STEP * UNIT_K) * C * 2;
                }
                return;
            }
#pragma unroll
            for (int m = 0; m < K::UPW; ++m) {  // k past d_in repeats the last row (it meets x = 0)
                const int64_t e = (int64_t)min(k0 + (unit0 + m * UNIT_STEP) * UNIT_K + g_row, d_in - 1) * C + g_c8;
                if constexpr (ROWS8) {
                    greg[m] = *(const u32x4 *)(G + e);
                } else {
                    const int64_t last = (int64_t)d_in * C - 1;
                    uint32_t v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = G[min(e + i, last)];
                    greg[m] = u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
                }
            }
        };
        // ... and, one slab later, as operands into LDS
        auto g_store = [&](unsigned char *slab) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < K::UPW; ++m) {
                const int u = unit0 + m * UNIT_STEP;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, greg[m]), sel_g[i],
                                                                            f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    const int frag = PAIR ? u * K::NBLK + 2 * pair + i : 2 * u + i;
                    *(f32x4 *)(slab + frag * K::FRAG + lane * 16) = d;
                }
            }
        };

        u32x4 xg[kRing];
        // Chunk starting at k0 into ring slot j.  x past d_in re-reads the row's last 16 bytes (the
        // values are zeroed before use), a token past N reads token 0 (never stored).
        auto x_load = [&](int j, int k0) __attribute__((always_inline)) {
            xg[j] = *(const u32x4 *)(xrow + max(min(k0, d_in - 8 - kq * 8), -kq * 8));
        };

#pragma unroll
        for (int j = 0; j < kRing; ++j) x_load(j, j * kXK);
        if (c0 > 0) route_barrier();  // the previous pass has finished reading the slabs
        g_load(0);
        g_store(route_lds);
        g_load(K::KS);
        route_barrier();

        // The loop is software-pipelined by one chunk: in front of the chain instructions of chunk j
        // the operands of chunk j+1 are made (x) or read (G) and its ring slot is refilled.
        int slab_idx = 0;  // slab of the chunk whose operands are being read
        f32x4 xf[2][2], gf[2][NB][2];  // operands of steps 0-3, 4-7
        auto operands = [&](int j, int set, int k0, bool fast) __attribute__((always_inline)) {
            const unsigned char *slab = route_lds + (slab_idx & 1) * K::SLAB;
            const int h0 = ((j * kXK) % K::KS) / 16;  // first 16 k of the chunk inside the slab
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    gf[set][b][h] = *(const f32x4 *)(slab + ((h0 + h) * K::NBLK + tb * NB + b) * K::FRAG + lane * 16);
            if (!fast && k0 + kXK > d_in) {  // (uniform) k past d_in adds +0
                const uint32_t ok = k0 + kq * 8 < d_in ? 0xFFFFFFFFu : 0u;
                xg[j] = u32x4{xg[j][0] & ok, xg[j][1] & ok, xg[j][2] & ok, xg[j][3] & ok};
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                xf[set][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel_x[h], __builtin_bit_cast(bf16x8, xg[j]),
                                                                     f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        };
        operands(0, 0, 0, false);
        x_load(0, kSCK);
        const uint16_t *xp = xrow + kSCK;  // the super-chunk being fetched
        // One super-chunk from k_sc on.  FAST: everything it fetches of x (up to chunk 0 of the super-
        // chunk after the next) lies inside d_in, at fixed distances from one pointer.
        auto super_chunk = [&](int k_sc, auto fast_c) __attribute__((always_inline)) {
            constexpr bool FAST = decltype(fast_c)::value;
#pragma unroll
            for (int j = 0; j < kRing; ++j) {
                const int jn = (j + 1) % kRing;            // ring position of the next chunk
                const int k_next = k_sc + (j + 1) * kXK;   // its first k (may be past d_in)
                const int cur = j & 1, nxt = cur ^ 1;
                if (!FAST && k_next - kXK >= d_in) break;  // (uniform) nothing left
                if (((j + 2) * kXK) % K::KS == 0) {
                    // the chunk after the next starts a G slab, which was loaded into registers one slab
                    // ago; the other buffer is free since this slab's barrier
                    g_store(route_lds + ((slab_idx + 1) & 1) * K::SLAB);
                    g_load((slab_idx + 2) * K::KS);
                }
                if (((j + 1) * kXK) % K::KS == 0) {  // the next chunk starts it
                    ++slab_idx;
                    route_barrier();
                }
                operands(jn, nxt, k_next, FAST);
                // refill the ring slot
                if constexpr (FAST)
                    xg[jn] = *(const u32x4 *)(xp + (j + 1) * kXK);
                else
                    x_load(jn, k_next + kSCK);
                // nothing else stands among the chain instructions, and nothing moves across a chunk
                // boundary (left alone, the scheduler sinks all loads of a round to its end and
                // the next round starts by waiting for them)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[cur][s >> 2][s & 3], gf[cur][b][s >> 2][s & 3],
                                                                      acc[b], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            xp += kSCK;
        };
        int k_sc = 0;
        for (; k_sc + 2 * kSCK + kXK <= d_in; k_sc += kSCK) super_chunk(k_sc, std::true_type{});
        for (; k_sc < d_in; k_sc += kSCK) super_chunk(k_sc, std::false_type{});

        bool nan = false;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) nan |= acc[b][v] != acc[b][v];
        if (__any(nan)) {
            const Chains<NB> again = route_chains_again<NB>(x + (tok_ok ? tok : 0) * (int64_t)d_in, G, d_in, C, kq, cw + l16);
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = again.acc[b];
        }

        // acc[b][v] is the logit of token kq*4 + v and target cw + b*16 + l16.
        if (logits_out != nullptr) {  // the chains themselves are wanted (first layer of a router MLP)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t t = tok_wave + kq * 4 + v;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int tgt = cw + b * 16 + l16;
                    if (t < N && tgt < C) logits_out[t * C + tgt] = acc[b][v];
                }
            }
        }
        // ---- running argmax: lexicographic (largest logit, then lowest index) ----
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int tgt = cw + b * 16 + l16;
                float val = acc[b][v];
                // a NaN logit never wins, except that target 0 is the scan's starting point
                if (val != val) val = (tgt == 0) ? __builtin_huge_valf() : -__builtin_huge_valf();
                if (tgt < C && (val > best[v] || (val == best[v] && tgt < bidx[v]))) {
                    best[v] = val;
                    bidx[v] = tgt;
                }
            }
        }
    }

    // winners of this wavefront's targets: reduce over the 16 lanes that hold a token's row
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            const float ov = __shfl_xor(best[v], d, 64);
            const int oi = __shfl_xor(bidx[v], d, 64);
            if (ov > best[v] || (ov == best[v] && oi < bidx[v])) {
                best[v] = ov;
                bidx[v] = oi;
            }
        }
    }
    if constexpr (TB > 1) {
        // merge the TB wavefronts of a token group through LDS
        __syncthreads();  // the slabs are done with
        float *red_v = (float *)route_lds;                 // [TB][TOK_WG]
        int32_t *red_i = (int32_t *)(red_v + TB * TOK_WG);
        if (l16 == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                red_v[tb * TOK_WG + tgw * 16 + kq * 4 + v] = best[v];
                red_i[tb * TOK_WG + tgw * 16 + kq * 4 + v] = bidx[v];
            }
        }
        __syncthreads();
        if (tb == 0 && l16 == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
#pragma unroll
                for (int o = 1; o < TB; ++o) {
                    const float ov = red_v[o * TOK_WG + tgw * 16 + kq * 4 + v];
                    const int oi = red_i[o * TOK_WG + tgw * 16 + kq * 4 + v];
                    if (ov > best[v] || (ov == best[v] && oi < bidx[v])) {
                        best[v] = ov;
                        bidx[v] = oi;
                    }
                }
            }
        }
    }
    if (tb == 0 && l16 == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t t = tok_wave + kq * 4 + v;
            if (t < N && r != nullptr) r[t] = bidx[v];
        }
    }
}

// more than 64 KB of dynamic LDS would have to be asked for
template <int NB, int TB, int TGW>
hipError_t launch_cfg(const uint16_t *x, const uint16_t *G, int32_t *r, float *lo, int64_t N,
                      int d_in, int C, hipStream_t s) {
    using K = RouteCfg<NB, TB, TGW>;
    static_assert(2 * K::SLAB <= 64 * 1024, "LDS");
    const dim3 blocks((unsigned)((N + K::TOK_WG - 1) / K::TOK_WG)), threads(K::NWV * 64);
    if (C % 8 == 0)
        hipLaunchKernelGGL((route_gate_kernel<NB, TB, TGW, true>), blocks, threads, 2 * K::SLAB, s, x, G, r, lo, N, d_in, C);
    else
        hipLaunchKernelGGL((route_gate_kernel<NB, TB, TGW, false>), blocks, threads, 2 * K::SLAB, s, x, G, r, lo, N, d_in, C);
    return hipGetLastError();
}

}  // namespace

// One chain per wavefront while the chains number at most one per SIMD (1024): they then run
// beside each other.  Beyond that two chains per wavefront, which share the operands of x (16384
// tokens x 32 targets: 44 us, one chain each 52 us).  Up to 16 targets a workgroup holds four token groups
// at any batch size: what its compute unit draws of x does not bound a chain, and the slab of G is staged by
// four wavefronts, not by one that runs a chain (groups per workgroup 1 / 2 / 4: 1024 x 4096 x 8 30 / 26 / 25
// us, 8192 x 2048 x 8 21 / 16 / 16, 5003 x 2048 x 13 27 / 18 / 17, 16384 x 12288 x 16 107 / 113 / 81).
hipError_t launch_route_gate(const uint16_t *x, const uint16_t *G, int32_t *r, float *logits_out,
                             int64_t N, int d_in, int C, hipStream_t s) {
    if (N == 0) return hipSuccess;
    const int64_t groups = (N + 15) / 16, blocks = (C + 15) / 16;
    const bool one = groups * blocks <= 1024;
#define MOLORA_ROUTE(NB, TB, TGW) launch_cfg<NB, TB, TGW>(x, G, r, logits_out, N, d_in, C, s)
    if (C <= 16) return MOLORA_ROUTE(1, 1, 4);
    if (C <= 32) return one ? MOLORA_ROUTE(1, 2, 2) : MOLORA_ROUTE(2, 1, 4);
    if (C <= 64) return one ? MOLORA_ROUTE(1, 4, 1) : MOLORA_ROUTE(2, 2, 2);
    return one ? MOLORA_ROUTE(1, 8, 1) : MOLORA_ROUTE(2, 4, 1);  // 128 targets per pass
#undef MOLORA_ROUTE
}

}  // namespace molora
