// Tile geometry of the radix sort, shared with the kernels that produce the
// keys: a producer whose workgroup b writes keys [b * kSortTile,
// (b + 1) * kSortTile) can count the first pass's digits of its tile as it
// goes (Pass0Hist), which saves the sort one read of the keys.
#pragma once

#include "expand.h"
#include "internal.h"

namespace gs {

// Build-time tunables: keys per thread of a sort tile (the emit's tile
// follows) and the widest digit of a pass.
#ifndef GS_SORT_ITEMS
#define GS_SORT_ITEMS 8
#endif
#ifndef GS_RADIX_BITS
#define GS_RADIX_BITS 10
#endif
constexpr int kSortItems = GS_SORT_ITEMS;
constexpr int kSortTile = kBlock * kSortItems;  // 2048
constexpr int kMaxDigitBits = GS_RADIX_BITS;
constexpr int kMaxDigits = 1 << kMaxDigitBits;
static_assert(kSortTile == kExpandTile, "emit tiles are sort tiles");
// Sorts of at least kBigSort pairs take tiles of kBigItems keys a thread
// (measured on a 22 M-pair index sort: 0.11 ms faster a sort; on 4 M pairs
// the longer tiles leave the chip under-filled).
constexpr int kBigItems = 2 * kSortItems;
constexpr int64_t kBigSort = (int64_t)1 << 23;

struct Pass0Hist {
    uint32_t *h;  // LDS, kMaxDigits words
    RadixPass0 p;
    __device__ __forceinline__ Pass0Hist(uint32_t *lds, const RadixPass0 &pass0) : h(lds), p(pass0) {
        if (p.table)
            for (uint32_t d = threadIdx.x; d <= p.mask; d += kBlock) h[d] = 0;
        __syncthreads();
    }
    __device__ __forceinline__ void add(uint32_t key) {
        if (p.table) atomicAdd(&h[key & p.mask], 1u);
    }
    // tile: the index of the tile this workgroup produced
    __device__ __forceinline__ void finish_tile(uint32_t tile) {
        __syncthreads();
        if (p.table)
            for (uint32_t d = threadIdx.x; d <= p.mask; d += kBlock) p.table[(size_t)d * p.nb + tile] = h[d];
    }
};

// Sorts of at most kSmallSort pairs take one workgroup that forms the keys,
// sorts them in LDS and writes them out: a sort's five to seven launches of 3
// to 9 us each cost more than the work (5,003 queries on 32^3 cells: keys and
// sort 33 -> 21 us; 4,096 Gaussians 20 -> 15).
constexpr int kSmallBlock = 1024;
constexpr int kSmallItems = 8;
constexpr int64_t kSmallSort = (int64_t)kSmallBlock * kSmallItems;
constexpr int kSmallWaves = kSmallBlock / kWave;
constexpr int kSmallBits = 6;  // bits of a pass: a counter per (digit, wave) for every thread
struct SmallSortLds {
    uint32_t k[kSmallSort], v[kSmallSort];
    uint32_t cnt[kSmallWaves << kSmallBits];
    uint32_t scan[kSmallWaves];
};

// Stable LSD sort of the pairs (key(i), i), i < n <= kSmallSort, by the low
// `bits` bits of the keys, into keys and vals, by a workgroup of kSmallBlock
// threads. The elements stay in (wave, item, lane) order in registers; a wave
// ranks its rows of 64 with one ballot per digit bit and a running count per
// digit, as the large sort does.
template <class Key>
__device__ __forceinline__ void small_sort(SmallSortLds &L, uint32_t n, int bits, Key key,
                                           uint32_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    if (n == 1) {
        if (tid == 0) {
            keys[0] = key(0u);
            vals[0] = 0;
        }
        return;
    }
    const uint32_t items = (n + kSmallBlock - 1) / kSmallBlock;
    const uint32_t e0 = wave * kWave * items + lane;  // item i is element e0 + 64 i
    uint32_t k[kSmallItems], v[kSmallItems];
#pragma unroll
    for (int i = 0; i < kSmallItems; ++i) {
        const uint32_t e = e0 + kWave * (uint32_t)i;
        v[i] = e;
        k[i] = (uint32_t)i < items && e < n ? key(e) : 0xFFFFFFFFu;  // past the end: last
    }
    const int passes = bits > 0 ? (bits + kSmallBits - 1) / kSmallBits : 1;
    const int db = bits > 0 ? (bits + passes - 1) / passes : 1;
    const uint32_t nd = 1u << db;
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
    uint32_t *mine = L.cnt + wave * nd;
    for (int p = 0; p < passes; ++p) {
        if (tid < kSmallWaves * nd) L.cnt[tid] = 0;
        __syncthreads();
        uint32_t slot[kSmallItems];
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if ((uint32_t)i >= items) continue;
            const uint32_t d = (k[i] >> (p * db)) & (nd - 1u);
            uint64_t m = ~0ull;
            for (int b = 0; b < db; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bm = __ballot(bit);
                m &= bit ? bm : ~bm;
            }
            const uint32_t before = (uint32_t)__popcll(m & lt), base = mine[d];
            // every lane of the wave has read the counter before its leader writes
            __builtin_amdgcn_wave_barrier();
            if (before == 0) mine[d] = base + (uint32_t)__popcll(m);
            __builtin_amdgcn_wave_barrier();
            slot[i] = base + before;
        }
        __syncthreads();
        // exclusive scan over (digit, wave), one counter a thread
        const uint32_t at = (tid % kSmallWaves) * nd + tid / kSmallWaves;
        const uint32_t c = tid < kSmallWaves * nd ? L.cnt[at] : 0u;
        const uint32_t incl = wave_incl_sum(c);
        if (lane == kWave - 1) L.scan[wave] = incl;
        __syncthreads();
        uint32_t pre = 0;
        for (uint32_t w = 0; w < wave; ++w) pre += L.scan[w];
        if (tid < kSmallWaves * nd) L.cnt[at] = pre + incl - c;
        __syncthreads();
        const bool last = p == passes - 1;
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if ((uint32_t)i >= items) continue;
            const uint32_t to = slot[i] + mine[(k[i] >> (p * db)) & (nd - 1u)];
            if (last) {
                if (to < n) {
                    keys[to] = k[i];
                    vals[to] = v[i];
                }
            } else {
                L.k[to] = k[i];
                L.v[to] = v[i];
            }
        }
        if (last) return;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallItems; ++i) {
            if ((uint32_t)i >= items) continue;
            k[i] = L.k[e0 + kWave * (uint32_t)i];
            v[i] = L.v[e0 + kWave * (uint32_t)i];
        }
        __syncthreads();
    }
}

}  // namespace gs
