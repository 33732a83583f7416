// node2vec's adjacency test (Tempest, Sec. "Temporal Bias Sampling"): the
// return and in-out weights need to know whether the window holds an edge
// prev -> w at any timestamp. The window's (source, destination) pairs live
// in an open-addressing hash table with a record count per pair, built on
// the first node2vec walk and then kept current by every ingest and
// eviction: the evicted window records count their pairs down, the kept
// batch records count theirs up, so an update costs O(batch), not
// O(window). A lookup is one 16-byte slot read for most pairs.
#include <algorithm>
#include <type_traits>

#include "tw_internal.h"

namespace tw {

namespace {

constexpr int AT = 256;  // threads per workgroup

__global__ void __launch_bounds__(AT) k_adj_clear(AdjSlot* __restrict__ tab, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * AT + threadIdx.x;
    if (i < n) tab[i] = AdjSlot{ADJ_EMPTY, 0u, 0u};
}

// d for pair k: claim the first empty slot of the probe sequence or count on
// the pair's slot. The table never fills (the host keeps it at most three
// quarters full), so the probe ends; a pair counted down was counted up before
// (it is a window record), so its slot comes before any empty one.
// probe starts at the pair's `at`-th slot.
__device__ __forceinline__ void adj_count(AdjSlot* __restrict__ tab, uint64_t mask, uint64_t k,
                                          int32_t d, uint64_t at = 0) {
    uint64_t j = (adj_hash(k) + at) & mask;
    for (uint64_t probe = at; probe <= mask; ++probe, j = (j + 1) & mask) {
        const uint64_t cur = tab[j].key;
        bool mine = cur == k;
        if (cur == ADJ_EMPTY) {
            if (d < 0) return;
            // a stale read only costs a failed claim: the exchange decides
            const unsigned long long prev =
                atomicCAS(reinterpret_cast<unsigned long long*>(&tab[j].key),
                          (unsigned long long)ADJ_EMPTY, (unsigned long long)k);
            mine = prev == ADJ_EMPTY || prev == k;
        }
        if (mine) {
            atomicAdd(&tab[j].cnt, (uint32_t)d);
            return;
        }
    }
}

// The pairs (src[i], dst[i]) of two record ranges, the first n0 counted down
// and the others up, a tile of AT * ITEMS records of one range per workgroup.
// Hub-to-hub pairs repeat (a few percent of a skewed batch are one pair), and
// atomics on one slot run one after the other, so a tile first counts its
// pairs in LDS: a pair takes the entry its hash names if that is free or its
// own, and otherwise goes to the table at once; then every entry goes to the
// table with its count. One atomic per record before: the table of a 50M-record
// window 29 -> 4.6 ms, 500,000 records down and as many up 338 -> 110 us.
constexpr int ADJ_ENTRIES = 2048;
// Records from which a tile takes 16 a thread instead of 4: a larger tile meets
// more of its repeats, a smaller one leaves fewer compute units idle (skewed
// sources and destinations, an ingest of b records that evicts as many: b =
// 100,000 319 us, at 16 a thread 337; 250,000 343 and 342; 500,000 433 and 406;
// 4M 1.43 and 1.19 ms; evenly spread pairs 200,000 318 and 337, 500,000 363 and
// 365).
constexpr int64_t ADJ_LARGE = 3 << 18;
template <int ITEMS>
__global__ void __launch_bounds__(AT) k_adj_count(AdjSlot* __restrict__ tab, uint64_t mask,
                                                   const int32_t* __restrict__ src0,
                                                   const int32_t* __restrict__ dst0, int64_t n0,
                                                   int64_t tiles0,
                                                   const int32_t* __restrict__ src1,
                                                   const int32_t* __restrict__ dst1, int64_t n1) {
    __shared__ unsigned long long key[ADJ_ENTRIES];
    __shared__ int32_t cnt[ADJ_ENTRIES];
    for (int e = threadIdx.x; e < ADJ_ENTRIES; e += AT) {
        key[e] = ADJ_EMPTY;
        cnt[e] = 0;
    }
    __syncthreads();
    const bool down = (int64_t)blockIdx.x < tiles0;
    const int32_t* src = down ? src0 : src1;
    const int32_t* dst = down ? dst0 : dst1;
    const int64_t n = down ? n0 : n1;
    const int64_t base = ((int64_t)blockIdx.x - (down ? 0 : tiles0)) * (AT * ITEMS);
    const int32_t one = down ? -1 : 1;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t i = base + r * AT + threadIdx.x;
        if (i >= n) break;
        const uint64_t k = adj_key(src[i], dst[i]);
        const int e = (int)(adj_hash(k) >> 32) & (ADJ_ENTRIES - 1);
        unsigned long long held = key[e];
        if (held == ADJ_EMPTY) {
            held = atomicCAS(&key[e], (unsigned long long)ADJ_EMPTY, (unsigned long long)k);
            if (held == ADJ_EMPTY) held = k;
        }
        if (held == k) atomicAdd(&cnt[e], one);
        else adj_count(tab, mask, k, one);
    }
    __syncthreads();
    // The entries' first probes together: all slots read, then all claims, so
    // a thread waits for two random accesses instead of two an entry.
    constexpr int E = ADJ_ENTRIES / AT;
    uint64_t cur[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * AT + threadIdx.x;
        cur[e] = cnt[i] != 0 ? tab[adj_hash(key[i]) & mask].key : 0;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * AT + threadIdx.x;
        if (cnt[i] > 0 && cur[e] == ADJ_EMPTY) {
            cur[e] = atomicCAS(
                reinterpret_cast<unsigned long long*>(&tab[adj_hash(key[i]) & mask].key),
                (unsigned long long)ADJ_EMPTY, key[i]);
            if (cur[e] == ADJ_EMPTY) cur[e] = key[i];
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * AT + threadIdx.x;
        const int32_t d = cnt[i];
        if (d == 0) continue;
        const uint64_t k = key[i];
        if (cur[e] == k) atomicAdd(&tab[adj_hash(k) & mask].cnt, (uint32_t)d);
        else if (cur[e] != ADJ_EMPTY) adj_count(tab, mask, k, d, 1);
    }
}

// counts the first range's pairs down and the second's up
hipError_t count_pairs(AdjSlot* tab, uint64_t mask, const int32_t* src0, const int32_t* dst0,
                       int64_t n0, const int32_t* src1, const int32_t* dst1, int64_t n1,
                       hipStream_t s) {
    auto run = [&](auto items) {
        constexpr int I = decltype(items)::value;
        const int64_t t0 = ceil_div(n0, AT * I), t1 = ceil_div(n1, AT * I);
        if (t0 + t1 > 0)
            hipLaunchKernelGGL(k_adj_count<I>, dim3((unsigned)(t0 + t1)), dim3(AT), 0, s, tab, mask,
                               src0, dst0, n0, t0, src1, dst1, n1);
    };
    if (n0 + n1 > ADJ_LARGE) run(std::integral_constant<int, 16>{});
    else run(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

dim3 grid_of(int64_t n) { return dim3((unsigned)std::max<int64_t>((n + AT - 1) / AT, 1)); }

// slots for a table holding m pairs at most half full (a power of two)
uint64_t adj_capacity(int64_t m) {
    uint64_t cap = 1024;
    while (cap < 2 * (uint64_t)std::max<int64_t>(m, 1)) cap <<= 1;
    return cap;
}

constexpr uint64_t ADJ_MAX_SLOTS = 1ull << 31;

}  // namespace

tw_status build_adjacency(tw_graph* g, Error& err) {
    if (g->adj_ready) return TW_OK;
    hipStream_t s = g->stream;
    const int64_t m = g->m;
    const uint64_t cap = adj_capacity(m);
    if (cap > ADJ_MAX_SLOTS) {
        err = Error{TW_ENOMEM, "node2vec adjacency: the window has too many records"};
        return err.code;
    }
    TW_HIP(ensure(g->adj_tab, sizeof(AdjSlot) * cap, s));
    hipLaunchKernelGGL(k_adj_clear, grid_of((int64_t)cap), dim3(AT), 0, s,
                       g->adj_tab.as<AdjSlot>(), cap);
    TW_HIP(count_pairs(g->adj_tab.as<AdjSlot>(), cap - 1, nullptr, nullptr, 0,
                       g->e_src.as<int32_t>() + g->e_base, g->e_dst.as<int32_t>() + g->e_base, m,
                       s));
    g->adj_mask = cap - 1;
    g->adj_used = m;
    g->adj_ready = true;
    return TW_OK;
}

tw_status adj_update(tw_graph* g, const int32_t* ev_src, const int32_t* ev_dst, int64_t ev_n,
                     const int32_t* add_src, const int32_t* add_dst, int64_t add_n, Error& err) {
    if (!g->adj_ready) return TW_OK;
    const uint64_t cap = g->adj_mask + 1;
    if ((uint64_t)(g->adj_used + add_n) > cap / 4 * 3) {
        // too full (counting every insert since the build): rebuild when needed
        g->adj_ready = false;
        return TW_OK;
    }
    hipStream_t s = g->stream;
    TW_HIP(count_pairs(g->adj_tab.as<AdjSlot>(), g->adj_mask, ev_src, ev_dst, ev_n, add_src, add_dst,
                       add_n, s));
    g->adj_used += add_n;
    return TW_OK;
}

}  // namespace tw
