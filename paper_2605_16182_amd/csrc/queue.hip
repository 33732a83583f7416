// Walk dispatches beside the walk blocks of walk.hip: the work queue and the
// cooperative per-step regrouping (Tempest, Sec. "Hierarchical Cooperative
// Scheduling").
#include <algorithm>

#include "walk_kernels.h"

namespace tw {
namespace {

// The last four output slots of a walk in registers (a shift register, so
// no slot is ever indexed at run time): when a walk has filled slots
// 4k..4k+3 they leave as one 16-byte store of nodes and two of timestamps.
struct RowChunk {
    int32_t n0 = -1, n1 = -1, n2 = -1, n3 = -1;
    int64_t t0 = TS_NONE, t1 = TS_NONE, t2 = TS_NONE, t3 = TS_NONE;
    __device__ __forceinline__ void push(int32_t v, int64_t t) {
        n0 = n1;
        n1 = n2;
        n2 = n3;
        n3 = v;
        t0 = t1;
        t1 = t2;
        t2 = t3;
        t3 = t;
    }
    // slots [at, at + 4) of a row; both pointers 16-byte aligned there
    __device__ __forceinline__ void store(int32_t* __restrict__ on, int64_t* __restrict__ ot,
                                          int32_t at) const {
        *reinterpret_cast<int4*>(on + at) = make_int4(n0, n1, n2, n3);
        *reinterpret_cast<longlong2*>(ot + at) = make_longlong2(t0, t1);
        *reinterpret_cast<longlong2*>(ot + at + 2) = make_longlong2(t2, t3);
    }
};

// Ends a row whose first len slots were pushed through c (and stored up to
// the last multiple of 4): the partial chunk is completed with padding, then
// every slot up to L (a multiple of 4) is padded with 16-byte stores.
__device__ __forceinline__ void finish_row(RowChunk& c, int32_t* __restrict__ on,
                                           int64_t* __restrict__ ot, int32_t len, int32_t L) {
    int32_t at = len & ~3;
    if (len & 3) {
        for (int32_t k = len & 3; k < 4; ++k) c.push(-1, TS_NONE);
        c.store(on, ot, at);
        at += 4;
    }
    const RowChunk pad;
    for (; at < L; at += 4) pad.store(on, ot, at);
}

// A lane's current four output slots in LDS, slot p in row p & 3 of the
// lane's column (registers the FP64 pickers need instead): when slots
// 4k..4k+3 are complete they leave as one 16-byte store of nodes and two of
// timestamps. Each lane touches its own column only.
struct RowRing {
    int32_t (*n)[WALK_THREADS];
    int64_t (*t)[WALK_THREADS];
    int tid;
    __device__ __forceinline__ void put(int32_t p, int32_t v, int64_t x) const {
        n[p & 3][tid] = v;
        t[p & 3][tid] = x;
    }
    // slots [at, at + 4) of a row; both pointers 16-byte aligned there
    __device__ __forceinline__ void flush(int32_t* __restrict__ on, int64_t* __restrict__ ot,
                                          int32_t at) const {
        *reinterpret_cast<int4*>(on + at) = make_int4(n[0][tid], n[1][tid], n[2][tid], n[3][tid]);
        *reinterpret_cast<longlong2*>(ot + at) = make_longlong2(t[0][tid], t[1][tid]);
        *reinterpret_cast<longlong2*>(ot + at + 2) = make_longlong2(t[2][tid], t[3][tid]);
    }
    // ends a row of len slots (stored up to the last multiple of 4): the
    // partial chunk is completed with padding, then every slot up to L (a
    // multiple of 4) is padded with 16-byte stores
    __device__ __forceinline__ void finish(int32_t* __restrict__ on, int64_t* __restrict__ ot,
                                           int32_t len, int32_t L) const {
        int32_t at = len & ~3;
        if (len & 3) {
            for (int32_t k = len & 3; k < 4; ++k) put(k, -1, TS_NONE);
            flush(on, ot, at);
            at += 4;
        }
        const RowChunk pad;
        for (; at < L; at += 4) pad.store(on, ot, at);
    }
};

// Backward walks (Gamma-_t(v): in-edges of v with t' < t, the backward case
// of Sec. "Design Constraints") on the in-view: the candidates of a hop at
// node v and time t are the groups [gb, hi) of v before the first group at
// or after t, listed from the latest, so every pick index is mirrored.
__device__ __forceinline__ bool back_pick(const WalkArgs& a, const HopBias& hb, uint64_t seed,
                                          const NodeRec& r, uint32_t hi, uint64_t id,
                                          uint64_t hop, int32_t prev, Pick& p, int32_t& nx) {
    const uint32_t end = hi < r.ge ? a.ng[hi].first : r.ee;  // the candidates' edges end
    const bool rate = reads_first_ts(hb.kind);
    const int64_t t_lo = rate ? group_ts(a.ng, a.fence, r, r.gb) : 0;
    const int64_t t_hi = rate ? group_ts(a.ng, a.fence, r, hi - 1) : 0;
    if (hb.kind != TW_NODE2VEC) {
        const Draw d = philox(id, hop, 0, seed);
        p = pick_node(a.ng, a.n_dst, a.n_ts, r.gb, hi, end, hb.kind, hb.tau, t_lo, t_hi, d,
                      true);
        nx = p.dst;
        return true;
    }
    // the edge candidate -> prev of the graph is prev -> candidate here
    for (uint32_t trial = 0; trial < N2V_MAX_TRIALS; ++trial) {
        const Draw d = philox(id, hop, trial, seed);
        p = pick_node(a.ng, a.n_dst, a.n_ts, r.gb, hi, end, TW_EXPONENTIAL, hb.tau, t_lo, t_hi,
                      d, true);
        nx = p.dst;
        if (n2v_accept(a, hb, d.x2, prev, nx)) return true;
    }
    atomicAdd(&a.err[2], 1u);
    return false;
}

// ----------------------------------------------------------------- queue
//
// Persistent dispatch with a device work queue. Every lane of a wavefront
// carries one walk at a time; when walks end, the wavefront takes as many
// new walk ids as it has idle lanes with one atomic add on a counter. The
// ids are split in QUEUE_SLICES contiguous slices, each with its own counter,
// and a wavefront starts on slice blockIdx % QUEUE_SLICES (consecutive
// workgroups go to different XCDs), moving to the next slice when one runs
// out, so the counters see little contention. Per walk: its length limit,
// its hop bias (one of up to TW_MAX_BIASES) and its output row.

__global__ void k_queue_reset(unsigned long long* counters) {
    if (threadIdx.x < QUEUE_SLICES) counters[threadIdx.x] = 0;
}

// REFILL = false is the same per-walk work without the queue: thread i runs
// walk i only (the full-walk form of a batch). REV: backward walks on the
// in-view.
template <bool REFILL, int HK, int SK, bool REV = false>
// The instantiation for mixed hop kinds (HK < 0) carries every picker's
// registers (about 160 VGPRs, 3 waves per SIMD); it is held to 4 waves, which
// spills a few registers and measured 11 % faster on mixed batches.
__global__ void __launch_bounds__(WALK_THREADS)
__attribute__((amdgpu_waves_per_eu(HK < 0 ? 4 : 1)))
k_walk_queue(const WalkArgs a, const QueueArgs q) {
    const int lane = threadIdx.x & 63;
    const int64_t W = a.num_walks;
    const int64_t slice_len = REFILL ? (W + QUEUE_SLICES - 1) / QUEUE_SLICES : W;
    int slice = REFILL ? (int)(blockIdx.x % QUEUE_SLICES) : 0;
    int exhausted = 0;  // slices this wavefront found empty (wave-uniform)
    int64_t w = -1;
    uint64_t id = 0, hop = 0;
    int32_t len = 0, lim = 0, cur = 0, prev = 0;
    int64_t tcur = 0;
    int32_t* out_n = nullptr;
    int64_t* out_t = nullptr;
    HopBias hb{};
    while (true) {
        const uint64_t idle = __ballot(w < 0);
        if (idle && exhausted < QUEUE_SLICES) {
            const int n = __popcll(idle);
            const int leader = __ffsll((unsigned long long)idle) - 1;
            unsigned long long got = 0;
            if (REFILL) {
                if (lane == leader) got = atomicAdd(&q.counters[slice], (unsigned long long)n);
                got = __shfl(got, leader, 64);
            } else {
                // each lane its own walk, once: the wave's first walk id
                got = (unsigned long long)blockIdx.x * WALK_THREADS + (threadIdx.x & ~63);
            }
            const int64_t lo = (int64_t)slice * slice_len;
            const int64_t hi = lo + slice_len < W ? lo + slice_len : W;
            if (w < 0) {
                const int rank = __popcll(idle & ((1ull << lane) - 1));
                const int64_t cand = lo + (int64_t)got + rank;
                if (cand < hi) {
                    w = cand;
                    id = a.base + (uint64_t)w;
                    lim = q.max_len ? q.max_len[w] : a.L;
                    const uint32_t b = q.bias_idx ? q.bias_idx[w] : (uint32_t)(id % (uint64_t)q.n_bias);
                    const int64_t row = q.row ? q.row[w] : w * (int64_t)a.L;
                    if (lim < 1 || lim > a.L || b >= (uint32_t)q.n_bias || row < 0 ||
                        row > q.out_slots - lim) {  // a sum could wrap
                        atomicOr(&a.err[3], 1u);
                        a.len[w] = 0;
                        w = -1;
                    } else {
                        hb = fixed_hop<HK>(q.bias[b]);
                        out_n = a.nodes + row;
                        out_t = a.ts + row;
                        const StartState st = walk_start(a, fixed_start<SK>(start_of(a)), w, id,
                                                         lim, out_n, out_t, REV);
                        len = st.len;
                        cur = st.cur;
                        prev = st.prev;
                        tcur = st.t;
                        hop = 1;
                        if (len < 2 || len >= lim) {
                            a.len[w] = len;
                            w = -1;
                        }
                    }
                }
            }
            if (!REFILL) {
                exhausted = QUEUE_SLICES;  // no more walks for this wavefront
            } else if (lo + (int64_t)got + n >= hi) {
                slice = (slice + 1) % QUEUE_SLICES;
                ++exhausted;
            }
        }
        if (__ballot(w >= 0) == 0) {
            if (exhausted >= QUEUE_SLICES) break;
            continue;
        }
        if (w >= 0) {
            bool done = true;
            const NodeRec r = a.rec[cur];
            // forward: Gamma_t(cur) is empty when t >= the last timestamp;
            // backward: when cur has no in-edge or none before t
            bool live = REV ? r.gb != r.ge : tcur < r.t_last;
            uint32_t g = 0;
            if (live) {
                if (REV) {
                    g = tcur - 1 >= r.t_last
                            ? r.ge
                            : fence_search(a.ng, a.fence, r, tcur - 1, nullptr, 0, 0);
                    live = g != r.gb;
                } else {
                    g = fence_search(a.ng, a.fence, r, tcur, nullptr, 0, 0);
                }
            }
            if (live) {
                Pick p;
                int32_t nx;
                if (REV ? back_pick(a, hb, a.seed, r, g, id, hop, prev, p, nx)
                        : hop_pick(a, hb, a.seed, r, g, id, hop, prev, p, nx)) {
                    out_n[len] = nx;
                    out_t[len] = p.t;
                    ++len;
                    ++hop;
                    prev = cur;
                    cur = nx;
                    tcur = p.t;
                    done = len >= lim;
                }
            }
            if (done) {
                a.len[w] = len;
                w = -1;
            }
        }
    }
}

// Live walks between steps: current node, walk index, current timestamp.
struct Live {
    uint32_t* node;
    uint32_t* walk;
    uint64_t* t;
};

// Hops of the live walks after their start (k_coop_start and
// k_compact_live leave them in `live`, n_live of them): the work queue
// without the start pick, so a lane that takes a walk only loads its state.
// ROWS: each lane writes its walk's whole output row, four slots per store,
// padding included; otherwise the rows were pre-filled. node2vec and mixed kinds
// keep a walk's current four slots in an LDS ring and are held to 4 waves per
// SIMD: 4.47 ms against 5.00 with the slots in
// registers at 3 waves (2M walks of length 40, 100M-edge graph). The other
// kinds keep the slots in registers at the occupancy their registers give:
// there the ring and more waves measured slower (exponential 5.33 against
// 4.98 ms at 5 waves, linear 2.45 against 2.30 at 8).
template <int HK, bool ROWS>
__global__ void __launch_bounds__(WALK_THREADS)
__attribute__((amdgpu_waves_per_eu(HK == TW_NODE2VEC || HK < 0 ? 4 : 1)))
k_walk_hops(const WalkArgs a, Live live, const int32_t* __restrict__ prev_of,
            const uint32_t* __restrict__ n_live_p, unsigned long long* counters) {
    constexpr bool RING = HK == TW_NODE2VEC || HK < 0;
    const int lane = threadIdx.x & 63;
    const int64_t W = *n_live_p;
    const int64_t slice_len = (W + QUEUE_SLICES - 1) / QUEUE_SLICES;
    int slice = (int)(blockIdx.x % QUEUE_SLICES);
    int exhausted = 0;
    int64_t w = -1;
    uint64_t id = 0, hop = 0;
    int32_t len = 0, cur = 0, prev = 0;
    int64_t tcur = 0;
    __shared__ int32_t ring_n[RING ? 4 : 1][WALK_THREADS];
    __shared__ int64_t ring_t[RING ? 4 : 1][WALK_THREADS];
    const RowRing ring{ring_n, ring_t, (int)threadIdx.x};
    RowChunk c;
    // the walk's output row: kept as pointers (fewer instructions), or
    // recomputed from w where registers are short (RING)
    int32_t* out_n = nullptr;
    int64_t* out_t = nullptr;
    auto row_n = [&]() { return RING ? a.nodes + w * (int64_t)a.L : out_n; };
    auto row_t = [&]() { return RING ? a.ts + w * (int64_t)a.L : out_t; };
    const HopBias hb = fixed_hop<HK>(a.hop);
    while (true) {
        const uint64_t idle = __ballot(w < 0);
        // refill once half the lanes are idle: a refill is an atomic round
        // trip and three dependent loads on the wavefront's critical path,
        // and plain walks end after a few hops
        if (exhausted < QUEUE_SLICES &&
            (idle == ~0ull || (idle && __popcll(idle) >= QUEUE_REFILL_MIN))) {
            const int n = __popcll(idle);
            const int leader = __ffsll((unsigned long long)idle) - 1;
            unsigned long long got = 0;
            if (lane == leader) got = atomicAdd(&counters[slice], (unsigned long long)n);
            got = __shfl(got, leader, 64);
            const int64_t lo = (int64_t)slice * slice_len;
            const int64_t hi = lo + slice_len < W ? lo + slice_len : W;
            if (w < 0) {
                const int rank = __popcll(idle & ((1ull << lane) - 1));
                const int64_t j = lo + (int64_t)got + rank;
                if (j < hi) {
                    w = live.walk[j];
                    cur = (int32_t)live.node[j];
                    tcur = (int64_t)live.t[j];
                    prev = prev_of[w];
                    id = a.base + (uint64_t)w;
                    if (!RING) {
                        out_n = a.nodes + w * (int64_t)a.L;
                        out_t = a.ts + w * (int64_t)a.L;
                    }
                    len = 2;
                    hop = 1;
                    // positions 0 and 1: the start edge's source and target
                    if (ROWS && RING) {
                        ring.put(0, prev, TS_NONE);
                        ring.put(1, cur, tcur);
                    } else if (ROWS) {
                        c = RowChunk();
                        c.push(prev, TS_NONE);
                        c.push(cur, tcur);
                    }
                }
            }
            if (lo + (int64_t)got + n >= hi) {
                slice = (slice + 1) % QUEUE_SLICES;
                ++exhausted;
            }
        }
        if (__ballot(w >= 0) == 0) {
            if (exhausted >= QUEUE_SLICES) break;
            continue;
        }
        if (w >= 0) {
            bool done = true;
            const NodeRec r = a.rec[cur];
            if (tcur < r.t_last) {
                const uint32_t gc = fence_search(a.ng, a.fence, r, tcur, nullptr, 0, 0);
                Pick p;
                int32_t nx;
                if (hop_pick(a, hb, a.seed, r, gc, id, hop, prev, p, nx)) {
                    if (ROWS && RING) {
                        ring.put(len, nx, p.t);
                        if ((len & 3) == 3) ring.flush(row_n(), row_t(), len - 3);
                    } else if (ROWS) {
                        c.push(nx, p.t);
                        if ((len & 3) == 3) c.store(row_n(), row_t(), len - 3);
                    } else {
                        row_n()[len] = nx;
                        row_t()[len] = p.t;
                    }
                    ++len;
                    ++hop;
                    prev = cur;
                    cur = nx;
                    tcur = p.t;
                    done = len >= a.L;
                }
            }
            if (done) {
                if (ROWS && RING) ring.finish(row_n(), row_t(), len, a.L);
                else if (ROWS) finish_row(c, row_n(), row_t(), len, a.L);
                a.len[w] = len;
                w = -1;
            }
        }
    }
}

// ------------------------------------------------------------------ coop
//
// Cooperative dispatch (Sec. "Hierarchical Cooperative Scheduling"): each
// step sorts the live walks by current node, and k_hop_coop advances them
// in that order. A wavefront whose 64 walks share one node, or a workgroup
// whose 256 walks do, reads the node record once and stages the top levels
// of the node's fence in LDS (the panel); mixed chunks run one walk per
// thread. Walks at a node with W walks thus get the workgroup tier for each
// full 256-walk chunk, the wavefront tier for each remaining full 64-walk
// chunk, and the thread tier otherwise; a node's walks beyond one
// workgroup are split over several workgroups.

// Live walks of one step, structure of arrays in one order: current node,
// walk index, time of arrival.
// ROWS: the rows are not pre-filled; a walk that ends at its start writes
// its whole padded row here, and the hop kernel writes the rows of the others.
template <int SK, bool ROWS = false>
__global__ void __launch_bounds__(WALK_THREADS) k_coop_start(const WalkArgs a, Live nx,
                                                              int32_t* __restrict__ prev,
                                                              uint32_t* __restrict__ alive) {
    const int64_t w = (int64_t)blockIdx.x * WALK_THREADS + threadIdx.x;
    if (w >= a.num_walks) return;
    const uint64_t id = a.base + (uint64_t)w;
    int32_t* out_n = a.nodes + w * a.L;
    int64_t* out_t = a.ts + w * a.L;
    StartState st = walk_start(a, fixed_start<SK>(start_of(a)), w, id, a.L,
                               ROWS ? nullptr : out_n, out_t);
    bool live = st.len >= 2 && st.len < a.L;
    if (live) {
        nx.node[w] = (uint32_t)st.cur;
        nx.walk[w] = (uint32_t)w;
        nx.t[w] = (uint64_t)st.t;
        prev[w] = st.prev;
    } else {
        if (ROWS) {
            RowChunk c;
            if (st.len >= 1) c.push(st.first, TS_NONE);
            if (st.len >= 2) c.push(st.cur, st.t);
            finish_row(c, out_n, out_t, st.len, a.L);
        }
        finish_walk(a, w, st.len);
    }
    alive[w] = live ? 1u : 0u;
}

// in-order compaction of the walks flagged alive
__global__ void k_compact_live(const uint32_t* __restrict__ flags, const uint32_t* __restrict__ pos,
                               int64_t n, Live in, Live out) {
    int64_t i = (int64_t)blockIdx.x * WALK_THREADS + threadIdx.x;
    if (i < n && flags[i]) {
        uint32_t o = pos[i];
        out.node[o] = in.node[i];
        out.walk[o] = in.walk[i];
        out.t[o] = in.t[i];
    }
}

// One hop for the live walks of `cur` (*n_live of the n_ub entries; the
// rest are idle), in node order when the step sorted them. Results go to
// `nx` at the same positions, with alive[i] set for walks that continue (0
// for idle entries). A wavefront engages the wavefront tier for the node of
// its first lane when at least wave_min of its lanes are at that node: the
// record is read once and the top levels of the node's fence are staged in
// LDS for those lanes; a workgroup whose four wavefronts engage it for one
// node stages a panel four times larger.
template <int HK>
__global__ void __launch_bounds__(WALK_THREADS)
k_hop_coop(const WalkArgs a, Live cur, Live nxt, int32_t* __restrict__ prev_of,
           const uint32_t* __restrict__ n_live, int64_t n_ub, uint64_t hop, uint32_t panel_cap,
           int wave_min, uint32_t* __restrict__ alive) {
    extern __shared__ __align__(16) uint32_t panel[];
    __shared__ int32_t wave_node[WALK_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * WALK_THREADS + threadIdx.x;
    const bool valid = i < (int64_t)*n_live;
    const int32_t v = valid ? (int32_t)cur.node[i] : -1;
    const int32_t v0 = __shfl(v, 0, 64);
    const int at_v0 = __popcll(__ballot(valid && v == v0));
    const bool wave_tier = v0 >= 0 && at_v0 >= wave_min;
    if (lane == 0) wave_node[wave] = wave_tier ? v0 : -1;
    __syncthreads();
    bool wg_tier = wave_node[0] >= 0;
#pragma unroll
    for (int k = 1; k < WALK_THREADS / 64; ++k) wg_tier &= wave_node[k] == wave_node[0];

    // stage the top levels of the node's fence: the whole panel for a
    // workgroup of one node, a quarter of it per wavefront otherwise.
    // Levels are stored bottom-up, so levels K down to some m are one
    // contiguous range.
    const uint32_t* my_panel = nullptr;
    uint64_t my_base = 0;
    uint32_t my_cap = 0;
    int32_t panel_node = -1;
    if (wg_tier || wave_tier) {
        panel_node = wg_tier ? wave_node[0] : v0;
        const NodeRec r = a.rec[panel_node];
        const uint32_t slice = wg_tier ? panel_cap : panel_cap / (WALK_THREADS / 64);
        uint32_t* dst = wg_tier ? panel : panel + wave * slice;
        const int K = (int)rec_levels(r.lv);
        if (K > 0) {
            const uint64_t cap = seg_groups(rec_code(r.lv));
            const uint64_t top = (uint64_t)r.fence_off +
                                 fence_level_off(seg_lg(rec_code(r.lv)), K) +
                                 fence_level_len(cap, K);  // end of level K
            uint64_t from = top;
            for (int k = K; k >= 0; --k) {
                const uint32_t len = fence_level_len(cap, k);
                if (top - (from - len) > slice) break;
                from -= len;
            }
            my_base = from;
            my_cap = (uint32_t)(top - from);
        }
        const int first = wg_tier ? threadIdx.x : lane;
        const int stride = wg_tier ? WALK_THREADS : 64;
        for (uint32_t j = first; j < my_cap; j += stride) dst[j] = a.fence[my_base + j];
        my_panel = dst;
    }
    __syncthreads();
    if (!valid) {
        if (i < n_ub) alive[i] = 0u;
        return;
    }
    if (v != panel_node) {
        my_panel = nullptr;
        my_base = 0;
        my_cap = 0;
    }

    const uint32_t w = cur.walk[i];
    const uint64_t id = a.base + (uint64_t)w;
    const NodeRec r = a.rec[v];
    const int64_t tcur = (int64_t)cur.t[i];
    const int32_t len = (int32_t)hop + 1;  // nodes written before this hop
    bool live = false;
    if (tcur < r.t_last) {
        const uint32_t gc = fence_search(a.ng, a.fence, r, tcur, my_panel, my_base, my_cap);
        Pick p;
        int32_t nx;
        const int32_t prev = a.hop.kind == TW_NODE2VEC ? prev_of[w] : 0;
        if (hop_pick(a, fixed_hop<HK>(a.hop), a.seed, r, gc, id, hop, prev, p, nx)) {
            a.nodes[(int64_t)w * a.L + len] = nx;
            a.ts[(int64_t)w * a.L + len] = p.t;
            if (len + 1 < a.L) {
                nxt.node[i] = (uint32_t)nx;
                nxt.walk[i] = w;
                nxt.t[i] = (uint64_t)p.t;
                if (a.hop.kind == TW_NODE2VEC) prev_of[w] = v;
                live = true;
            } else {
                a.len[w] = len + 1;
            }
        } else {
            finish_walk(a, w, len);
        }
    } else {
        finish_walk(a, w, len);
    }
    alive[i] = live ? 1u : 0u;
}

// entries [*n_live, n_ub) of a live list get a node id above every real
// one, so a sort by node leaves them last
__global__ void k_live_tail(Live live, const uint32_t* __restrict__ n_live, int64_t n_ub,
                            uint32_t sentinel) {
    const int64_t i = (int64_t)blockIdx.x * WALK_THREADS + threadIdx.x;
    if (i < n_ub && i >= (int64_t)*n_live) live.node[i] = sentinel;
}

}  // namespace

// Host loop of the cooperative dispatch: per step, regroup the live walks
// by node (a stable sort, or none), one hop, in-order compaction. The live
// count is read back every coop_sync steps; in between, launches cover the
// last count read (an upper bound) and their threads past the device count
// idle.
tw_status coop_walks(tw_graph* g, const WalkArgs& a, Error& err) {
    hipStream_t s = g->stream;
    const int64_t W = a.num_walks;
    DevBuf* bufs32[] = {&g->c_node0, &g->c_walk0, &g->c_node1, &g->c_walk1, &g->c_node2,
                        &g->c_walk2, &g->c_flags, &g->c_pos, &g->c_prev};
    for (DevBuf* b : bufs32) TW_HIP(ensure(*b, sizeof(uint32_t) * W, g->stream));
    TW_HIP(ensure(g->c_t0, sizeof(uint64_t) * W, g->stream));
    TW_HIP(ensure(g->c_t1, sizeof(uint64_t) * W, g->stream));
    TW_HIP(ensure(g->c_t2, sizeof(uint64_t) * W, g->stream));
    // live (compacted) -> sorted (by node) -> next (after the hop) -> live
    Live live{g->c_node0.as<uint32_t>(), g->c_walk0.as<uint32_t>(), g->c_t0.as<uint64_t>()};
    Live sorted{g->c_node1.as<uint32_t>(), g->c_walk1.as<uint32_t>(), g->c_t1.as<uint64_t>()};
    Live next{g->c_node2.as<uint32_t>(), g->c_walk2.as<uint32_t>(), g->c_t2.as<uint64_t>()};
    int32_t* prev = g->c_prev.as<int32_t>();
    uint32_t* flags = g->c_flags.as<uint32_t>();
    uint32_t* pos = g->c_pos.as<uint32_t>();
    uint32_t* n_live_d = g->scal.as<uint32_t>() + SLOT_U32_N_LIVE;
    // node ids and the sentinel V sort in bits_for(V) bits
    const int vbits = bits_for((uint64_t)g->V);
    const uint32_t panel_cap = g->coop_panel;
    const int sync_every = std::max(g->coop_sync, 1);
    const dim3 wgrid((unsigned)ceil_div(W, WALK_THREADS));

    with_kinds(-1, a.start_kind, [&](auto, auto sk) {
        hipLaunchKernelGGL((k_coop_start<decltype(sk)::value>), wgrid, dim3(WALK_THREADS), 0, s, a,
                           next, prev, flags);
    });
    TW_HIP(scan_exclusive_u32(flags, pos, W, n_live_d, g->ws, s));
    hipLaunchKernelGGL(k_compact_live, wgrid, dim3(WALK_THREADS), 0, s, flags, pos, W, next, live);
    TW_HIP(hipGetLastError());
    int64_t n_ub = W;
    for (uint64_t hop = 1; hop + 1 < (uint64_t)a.L; ++hop) {
        if ((hop - 1) % (uint64_t)sync_every == 0) {
            if (pull_scalars(g, false, err) != TW_OK) return err.code;
            n_ub = host_u32(g, SLOT_U32_N_LIVE);
            if (n_ub == 0) break;
        }
        const dim3 grid((unsigned)ceil_div(n_ub, WALK_THREADS));
        Live in = live;
        if (g->coop_regroup == 0) {
            if (sync_every > 1)
                hipLaunchKernelGGL(k_live_tail, grid, dim3(WALK_THREADS), 0, s, live, n_live_d,
                                   n_ub, (uint32_t)g->V);
            TW_HIP(radix_sort_u32_kv(live.node, live.walk, live.t, sorted.node, sorted.walk,
                                     sorted.t, n_ub, 0, vbits, g->ws, s));
            in = sorted;
        }
        with_kinds(a.hop.kind, TW_UNIFORM, [&](auto hk, auto) {
            hipLaunchKernelGGL((k_hop_coop<decltype(hk)::value>), grid, dim3(WALK_THREADS),
                               sizeof(uint32_t) * panel_cap, s, a, in, next, prev, n_live_d,
                               n_ub, hop, panel_cap, g->coop_wave_min, flags);
        });
        TW_HIP(scan_exclusive_u32(flags, pos, n_ub, n_live_d, g->ws, s));
        hipLaunchKernelGGL(k_compact_live, grid, dim3(WALK_THREADS), 0, s, flags, pos, n_ub, next,
                           live);
        TW_HIP(hipGetLastError());
    }
    return TW_OK;
}

// compute units, queried once per graph (a host-side query only, so a walk
// launch can be captured in a graph afterwards)
tw_status queue_shape(tw_graph* g, Error& err) {
    if (g->cu_count) return TW_OK;
    int n = 0;
    TW_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, g->device));
    g->cu_count = std::max(n, 1);
    return TW_OK;
}

// resident workgroups per compute unit of one queue kernel instantiation
template <typename K>
int resident_bpc(K kernel) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, WALK_THREADS, 0) != hipSuccess)
        nb = 1;
    return std::max(nb, 1);
}

// rev: backward walks (a is the in-view's)
tw_status queue_walks(tw_graph* g, const WalkArgs& a, const QueueArgs& q0, int bpc, Error& err,
                      bool rev) {
    if (queue_shape(g, err) != TW_OK) return err.code;
    TW_HIP(ensure(g->wq, sizeof(unsigned long long) * QUEUE_SLICES, g->stream));
    QueueArgs q = q0;
    q.counters = g->wq.as<unsigned long long>();
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, g->stream, q.counters);
    const int hk = q.n_bias == 1 ? q.bias[0].kind : -1;
    with_kinds(hk, a.start_kind, [&](auto h, auto st) {
        with_direction<decltype(h)::value>(rev, [&](auto r) {
            auto kernel =
                k_walk_queue<true, decltype(h)::value, decltype(st)::value, decltype(r)::value>;
            static const int maxb = resident_bpc(kernel);  // per instantiation
            const int b = (bpc <= 0 || bpc > maxb) ? maxb : bpc;
            const int64_t blocks =
                std::min<int64_t>(ceil_div(a.num_walks, WALK_THREADS), (int64_t)g->cu_count * b);
            hipLaunchKernelGGL(kernel, dim3((unsigned)std::max<int64_t>(blocks, 1)),
                               dim3(WALK_THREADS), 0, g->stream, a, q);
        });
    });
    TW_HIP(hipGetLastError());
    return TW_OK;
}

// the batch with one thread per walk and no queue
tw_status batch_full_walk(tw_graph* g, const WalkArgs& a, const QueueArgs& q, Error& err,
                          bool rev) {
    const int hk = q.n_bias == 1 ? q.bias[0].kind : -1;
    with_kinds(hk, a.start_kind, [&](auto h, auto st) {
        with_direction<decltype(h)::value>(rev, [&](auto r) {
            hipLaunchKernelGGL((k_walk_queue<false, decltype(h)::value, decltype(st)::value,
                                             decltype(r)::value>),
                               dim3((unsigned)ceil_div(a.num_walks, WALK_THREADS)),
                               dim3(WALK_THREADS), 0, g->stream, a, q);
        });
    });
    TW_HIP(hipGetLastError());
    return TW_OK;
}

// The queue dispatch of plain walks: every start in one pass (as the
// cooperative dispatch starts), the live walks compacted, then one
// persistent launch of k_walk_hops over them. The lists (the walks alive
// after their start before and after compaction, each walk's previous node,
// the alive flags and their scan) are graph buffers, grown as needed.
tw_status queue_hops(tw_graph* g, const WalkArgs& a, int bpc, Error& err) {
    hipStream_t s = g->stream;
    const int64_t W = a.num_walks;
    if (queue_shape(g, err) != TW_OK) return err.code;
    DevBuf* bufs32[] = {&g->c_node0, &g->c_walk0, &g->c_node2, &g->c_walk2, &g->c_flags,
                        &g->c_pos, &g->c_prev};
    for (DevBuf* b : bufs32) TW_HIP(ensure(*b, sizeof(uint32_t) * W, s));
    TW_HIP(ensure(g->c_t0, sizeof(uint64_t) * W, s));
    TW_HIP(ensure(g->c_t2, sizeof(uint64_t) * W, s));
    TW_HIP(ensure(g->wq, sizeof(unsigned long long) * QUEUE_SLICES, s));
    const Live live{g->c_node0.as<uint32_t>(), g->c_walk0.as<uint32_t>(), g->c_t0.as<uint64_t>()};
    const Live next{g->c_node2.as<uint32_t>(), g->c_walk2.as<uint32_t>(), g->c_t2.as<uint64_t>()};
    int32_t* prev = g->c_prev.as<int32_t>();
    uint32_t* flags = g->c_flags.as<uint32_t>();
    uint32_t* pos = g->c_pos.as<uint32_t>();
    uint32_t* n_live = g->scal.as<uint32_t>() + SLOT_U32_N_LIVE;
    unsigned long long* counters = g->wq.as<unsigned long long>();
    const dim3 wgrid((unsigned)ceil_div(W, WALK_THREADS));
    const bool rows = own_rows(a);
    with_kinds(-1, a.start_kind, [&](auto, auto sk) {
        if (rows)
            hipLaunchKernelGGL((k_coop_start<decltype(sk)::value, true>), wgrid,
                               dim3(WALK_THREADS), 0, s, a, next, prev, flags);
        else
            hipLaunchKernelGGL((k_coop_start<decltype(sk)::value, false>), wgrid,
                               dim3(WALK_THREADS), 0, s, a, next, prev, flags);
    });
    TW_HIP(scan_exclusive_u32(flags, pos, W, n_live, g->ws, s));
    hipLaunchKernelGGL(k_compact_live, wgrid, dim3(WALK_THREADS), 0, s, flags, pos, W, next, live);
    hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, s, counters);
    with_kinds(a.hop.kind, TW_UNIFORM, [&](auto hk, auto) {
        auto launch = [&](auto kernel) {
            static const int maxb = resident_bpc(kernel);  // per instantiation
            const int b = (bpc <= 0 || bpc > maxb) ? maxb : bpc;
            const int64_t blocks =
                std::min<int64_t>(ceil_div(W, WALK_THREADS), (int64_t)g->cu_count * b);
            hipLaunchKernelGGL(kernel, dim3((unsigned)std::max<int64_t>(blocks, 1)),
                               dim3(WALK_THREADS), 0, s, a, live, prev, n_live, counters);
        };
        if (rows)
            launch(k_walk_hops<decltype(hk)::value, true>);
        else
            launch(k_walk_hops<decltype(hk)::value, false>);
    });
    TW_HIP(hipGetLastError());
    return TW_OK;
}

}  // namespace tw
