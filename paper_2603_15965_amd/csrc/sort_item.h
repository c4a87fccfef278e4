// The dispatch step inside a shrink launch, for batches beyond one wavefront: every workgroup finds its own
// work item (a tile of sorted rows of one bucket) and the item's tokens from the targets r, and writes its
// part of the permutation for the launch that follows.  No workgroup waits for another.
//
// The dispatch kernel is a launch of its own of 4 to 8 us that the shrink waits for, all of it latency; here
// a workgroup reads the targets once (at most 32 KB, from the L2), counts them per bucket, and picks its
// item's tokens out of the same registers.  Against a shrink that is given offsets and perm, which spends two dependent
// trips to memory on them, the launch takes 1.4 us more at 512 targets, 2.2 at 4096 and 3 at 8192 (5.9 where the
// workgroups make a second round: 8192 x 2048, 8 buckets of rank 64, 272 of them; the dispatch launch takes 6.4
// there).  The order is the dispatch step's: buckets
// ascending, tokens ascending inside a bucket, tokens without adapter behind the last bucket.
#pragma once
#include "common.h"

namespace molora {
namespace {

// the most tiles of `rows` rows that N tokens in at most `buckets` buckets can make: all buckets but one hold a row
// more than whole tiles do
inline int64_t most_tiles(int64_t N, int64_t buckets, int rows) {
    const int64_t m = buckets < N ? buckets : N;
    return (N + (rows - 1) * m) / rows;
}

struct SortedItem {
    int bucket;    // -1: no such item; C: tokens without adapter
    int row_base;  // first sorted position
    int nrows;
};

constexpr int kSortUnroll = 16;  // targets per lane, all in registers
constexpr int sort_max(int waves) { return waves * 64 * kSortUnroll; }  // tokens of a batch

// LDS words a workgroup needs beside rows[ROWS]: a row of counts per wavefront, one for each of the C + 1 keys
// (target C: no adapter) and one for the lanes past the batch
__host__ __device__ constexpr int sort_lds_words(int C, int waves) { return (C + 2) * waves; }

// inclusive prefix sum over the lanes of a wavefront, in the vector ALU (a shuffle is a trip through the LDS)
__device__ __forceinline__ int wave_prefix(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1, inside rows of 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);  // row_bcast:15, into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);  // row_bcast:31, into rows 2 and 3
    return v;
}

// For all threads of a workgroup of NWV wavefronts (barriers inside), N <= sort_max(NWV).  item_of(real, total) ->
// this workgroup's item, or -1, the same for all threads: the first `real` items are tiles of the buckets, the others
// list tokens without adapter.  lds: sort_lds_words(C, NWV) words, free again after the
// call; rows[ROWS + 1]: the item's tokens.  write_offsets: this workgroup writes offsets[0 .. C].
//
// 8192 targets, 8 wavefronts, cycles: targets from memory 1800, counts 3000 (an LDS add of a wavefront takes 17
// to 28 of the compute unit), their prefixes 1100, the item's tokens 2000, barriers 700.
template <int NWV, int ROWS, class ItemOf>
__device__ __forceinline__ SortedItem sort_item(const int32_t *__restrict__ r, int N, int C, int32_t *lds,
                                                int32_t *rows, int32_t *__restrict__ offsets, bool write_offsets,
                                                ItemOf item_of) {
    static_assert(ROWS >= 16 && sort_max(NWV) < 32768, "a count and a number of tiles share a word");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int keys = C + 1, pitch = C + 2;
    // this wavefront's tokens: a contiguous range, a multiple of 64 long
    const int per = (N + NWV * 64 - 1) / (NWV * 64) * 64;
    const int start = min(wave * per, N), end = min(start + per, N);
    int32_t key[kSortUnroll];
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) key[u] = r[min(start + u * 64 + lane, N - 1)];  // never predicated
    for (int i = tid; i < pitch * NWV; i += NWV * 64) lds[i] = 0;
    __syncthreads();
    int32_t *mine = lds + wave * pitch;
#pragma unroll
    for (int u = 0; u < kSortUnroll; ++u) {
        const int32_t c = key[u];
        key[u] = start + u * 64 + lane < end ? ((unsigned)c < (unsigned)C ? c : C) : keys;
    }
    if (C <= 3) {  // every group would add to two or three words: ballots
        int n[4] = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < kSortUnroll; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) n[k] += (int)__popcll(__ballot(key[u] == k));
        if (lane < keys) mine[lane] = lane == 0 ? n[0] : lane == 1 ? n[1] : lane == 2 ? n[2] : n[3];
    } else {
#pragma unroll
        for (int u = 0; u < kSortUnroll; ++u) {
            if (start + u * 64 >= end) continue;  // wave-uniform
            // one target for the whole group (runs of tokens of a sequence): one add of its size, where 64 adds
            // to one word would be served one after the other
            const int32_t k0 = __builtin_amdgcn_readfirstlane(key[u]);
            if (__ballot(key[u] != k0) == 0) {
                if (lane == 0) __hip_atomic_fetch_add(&mine[k0], 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                __hip_atomic_fetch_add(&mine[key[u]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    __syncthreads();

    // of a group of 64 keys, one to a lane: count | tiles << 16, and its inclusive prefix; of the count, what
    // the wavefronts before this one and this one hold
    int one = 0, incl = 0, below = 0, own = 0;
    auto scan_group = [&](int c0) {
        int n = 0;
        below = 0;
        const int c = min(c0 + lane, keys);
#pragma unroll
        for (int w = 0; w < NWV; ++w) {
            const int v = lds[w * pitch + c];
            n += v;
            below += w < wave ? v : 0;
            own = w == wave ? v : own;
        }
        if (c0 + lane >= keys) n = 0;
        one = n | ((n + ROWS - 1) / ROWS) << 16;
        incl = wave_prefix(one);
    };
    int run = 0;  // of the groups before
    for (int c0 = 0; c0 < keys; c0 += 64) {
        scan_group(c0);
        if (write_offsets && wave == 0 && c0 + lane < keys) offsets[c0 + lane] = (run + incl - one) & 0xffff;
        run += __builtin_amdgcn_readlane(incl, 63);
    }
    // (the last group scanned holds key C)
    const int item = item_of((run >> 16) - (__builtin_amdgcn_readlane(one, C & 63) >> 16), run >> 16);
    SortedItem it{-1, 0, 0};
    int at = 0, held = 0;  // place in the item of this wavefront's next token of the bucket, tokens it holds
    if (item >= 0) {
        run = 0;
        for (int c0 = 0; c0 < keys && it.bucket < 0; c0 += 64) {
            if (keys > 64) scan_group(c0);  // (one group: still in registers)
            const int before = run + incl - one;
            const int rel = item - (before >> 16);
            const uint64_t m = __ballot(rel >= 0 && rel < (one >> 16));
            if (m) {
                const int src = __builtin_ctzll(m);
                const int first = __builtin_amdgcn_readlane(rel, src) * ROWS;  // among the bucket's tokens
                it.bucket = c0 + src;
                it.row_base = (__builtin_amdgcn_readlane(before, src) & 0xffff) + first;
                it.nrows = min(ROWS, (__builtin_amdgcn_readlane(one, src) & 0xffff) - first);
                at = __builtin_amdgcn_readlane(below, src) - first;
                held = __builtin_amdgcn_readlane(own, src);
            }
            run += __builtin_amdgcn_readlane(incl, 63);
        }
    }
    if (it.bucket < 0) return it;  // (the whole workgroup)

    // the item's tokens, picked out by the wavefronts that hold some; rows[ROWS] takes what is not the item's
    if (at < it.nrows && at + held > 0) {
#pragma unroll
        for (int u = 0; u < kSortUnroll; ++u) {
            if (start + u * 64 >= end) continue;  // wave-uniform
            const bool in = key[u] == it.bucket;
            const uint64_t m = __ballot(in);
            const int place = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at));
            rows[in && (unsigned)place < (unsigned)it.nrows ? place : ROWS] = start + u * 64 + lane;
            at += (int)__popcll(m);
        }
    }
    __syncthreads();
    return it;
}

}  // namespace
}  // namespace molora
