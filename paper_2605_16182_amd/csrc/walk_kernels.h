// What the walk kernels share (walk.hip: walk blocks, the entry points;
// queue.hip: the work queue and the cooperative dispatch): a launch's
// arguments, the start of a walk, a hop's pick, padding.
#pragma once

#include <algorithm>
#include <type_traits>

#include "walk_device.h"

namespace tw {

// A hop bias with node2vec's constants precomputed.
struct HopBias {
    int32_t kind;
    double tau, inv_p, inv_q, beta_max;
};

inline HopBias make_hop_bias(const tw_bias& b) {
    HopBias h;
    h.kind = b.kind;
    h.tau = b.tau;
    h.inv_p = b.kind == TW_NODE2VEC ? 1.0 / b.p : 1.0;
    h.inv_q = b.kind == TW_NODE2VEC ? 1.0 / b.q : 1.0;
    h.beta_max = std::max(std::max(h.inv_p, 1.0), h.inv_q);
    return h;
}

struct WalkArgs {
    // timestamp view and its groups
    const int32_t* e_src;
    const int32_t* e_dst;
    const int64_t* e_ts;
    const uint32_t* gg_off;  // first record of each timestamp group (from gg_base), then the end
    // read from the graph's scalar slots, where the last update wrote them: the
    // window's first and last timestamps, its global group count, and
    // win = (e_base, m, gg_base): the window is e_*[e_base, e_base + m), its
    // groups start at gg_off[gg_base]
    const int64_t* wsum;
    const int64_t* wgg;
    const int64_t* win;
    // node view
    const int32_t* n_dst;
    const int64_t* n_ts;
    const GroupRec* ng;
    const NodeRec* rec;
    const uint32_t* fence;
    const AdjSlot* adj_tab;  // node2vec pair table (adj_mask + 1 slots)
    uint64_t adj_mask;
    const double* cw;  // cumulative group weights (weight-based picker)
    int32_t V;
    // parameters
    int64_t num_walks;
    int32_t L;
    HopBias hop;
    int32_t start_kind, start_mode;
    double start_tau;
    const int32_t* start_nodes;
    uint64_t seed, base;
    // outputs
    int32_t* nodes;
    int64_t* ts;
    int32_t* len;
    uint32_t* err;  // [0] start node out of range, [2] node2vec trial cap hits
    bool pre_filled;  // the outputs hold padding already (walk blocks leave theirs out)
};

// The start of a walk: RNG seed, start bias and mode, start nodes.
struct StartParams {
    uint64_t seed;
    int32_t kind, mode;
    double tau;
    const int32_t* nodes;
};

__device__ __forceinline__ StartParams start_of(const WalkArgs& a) {
    return StartParams{a.seed, a.start_kind, a.start_mode, a.start_tau, a.start_nodes};
}

constexpr int WALK_THREADS = 256;

// Kernels are instantiated per hop kind HK and start kind SK (-1: read at
// run time). A fixed kind leaves only that picker's arithmetic in the
// kernel: the full-walk kernel takes 62 VGPRs for uniform and linear hops and
// 68 for exponential ones, against 97 for the serving kernel, which carries every
// picker.
template <int HK>
__device__ __forceinline__ HopBias fixed_hop(HopBias h) {
    if (HK >= 0) h.kind = HK;
    return h;
}
template <int SK>
__device__ __forceinline__ StartParams fixed_start(StartParams sp) {
    if (SK >= 0) sp.kind = SK;
    return sp;
}
constexpr uint32_t N2V_MAX_TRIALS = 4096;

// Walk state after the first pick (RNG hop 0).
struct StartState {
    int32_t len;   // nodes written so far
    int32_t cur, prev;
    int64_t t;
    int32_t first; // the node at position 0 (when len >= 1)
};

// First pick of walk w: EDGE mode draws from the whole window, NODE mode from
// the start node's run; writes output positions 0 and 1 (out_n null: writes
// nothing, the caller takes them from the state). rev: a backward walk
// (candidates listed in reverse). A start node out of range sets
// *range_flag (the graph's flag word when null).
__device__ __forceinline__ StartState walk_start(const WalkArgs& a, const StartParams& sp, int64_t w,
                                                 uint64_t id, int32_t L, int32_t* out_n,
                                                 int64_t* out_t, bool rev = false,
                                                 uint32_t* range_flag = nullptr) {
    StartState st{0, 0, 0, 0, -1};
    const Draw d0 = philox(id, 0, 0, sp.seed);
    if (sp.mode == TW_START_EDGE) {
        const uint32_t m = (uint32_t)a.win[1];
        if (m == 0) return st;
        uint32_t e;
        if (sp.kind == TW_UNIFORM) {
            const uint32_t i = (uint32_t)scale_u64(d0.x0, m);
            e = (uint32_t)a.win[0] + (rev ? m - 1 - i : i);
        } else {
            e = pick_global(a.gg_off + a.win[2], (uint32_t)*a.wgg, a.wsum[0], a.wsum[1], sp.kind,
                            sp.tau, d0, rev);
        }
        const int32_t s = a.e_src[e], t_dst = a.e_dst[e];
        const int64_t t = a.e_ts[e];
        if (out_n) out_n[0] = s;
        st.first = s;
        st.len = 1;
        if (L == 1) return st;
        if (out_n) {
            out_n[1] = t_dst;
            out_t[1] = t;
        }
        st.len = 2;
        st.prev = s;
        st.cur = t_dst;
        st.t = t;
        return st;
    }
    const int32_t v0 = sp.nodes[w];
    if (v0 < 0 || v0 >= a.V) {
        atomicOr(range_flag ? range_flag : &a.err[0], 1u);
        return st;
    }
    if (out_n) out_n[0] = v0;
    st.first = v0;
    st.len = 1;
    if (L == 1) return st;
    const NodeRec r = a.rec[v0];
    if (r.gb == r.ge) return st;
    const int64_t t_first = reads_first_ts(sp.kind) ? a.ng[r.gb].ts : 0;
    Pick p = pick_node(a.ng, a.n_dst, a.n_ts, r.gb, r.ge, r.ee, sp.kind, sp.tau, t_first,
                       r.t_last, d0, rev);
    const int32_t nx = p.dst;
    if (out_n) {
        out_n[1] = nx;
        out_t[1] = p.t;
    }
    st.len = 2;
    st.prev = v0;
    st.cur = nx;
    st.t = p.t;
    return st;
}

// node2vec's acceptance of candidate dst: u beta_max < beta with beta = 1/p
// for the previous node, 1 where the window holds the edge prev -> dst, else
// 1/q. The edge is looked up (a random read of the pair table) only where the
// answer depends on it: u beta_max between 1 and 1/q (a quarter of the trials
// for p = 1/2, q = 2, none for q = 1).
__device__ __forceinline__ bool n2v_accept(const WalkArgs& a, const HopBias& hb, uint64_t x2,
                                           int32_t prev, int32_t dst) {
    const double u = unit_closed_open(x2) * hb.beta_max;
    if (dst == prev) return u < hb.inv_p;
    const bool adjacent = u < 1.0, apart = u < hb.inv_q;
    if (adjacent == apart) return adjacent;
    return adj_has(a.adj_tab, a.adj_mask, prev, dst) ? adjacent : apart;
}

// The pick of hop `hop` among groups [gc, r.ge) of node cur (previous node
// prev): the hop bias, or node2vec's rejection loop. Returns false when
// node2vec exhausts its trials (the walk ends and is counted).
__device__ __forceinline__ bool hop_pick(const WalkArgs& a, const HopBias& hb, uint64_t seed,
                                         const NodeRec& r, uint32_t gc, uint64_t id, uint64_t hop,
                                         int32_t prev, Pick& p, int32_t& nx) {
    if (hb.kind == TW_WEIGHT) {
        const Draw d = philox(id, hop, 0, seed);
        p = pick_weight(a.ng, a.n_dst, a.cw, r.gb, gc, r.ge, r.ee, hb.tau > 0.0 ? hb.tau : 1.0,
                        group_ts(a.ng, a.fence, r, gc), r.t_last, d);
        nx = p.dst;
        return true;
    }
    if (hb.kind != TW_NODE2VEC) {
        const Draw d = philox(id, hop, 0, seed);
        const int64_t t_first = reads_first_ts(hb.kind) ? group_ts(a.ng, a.fence, r, gc) : 0;
        p = pick_node(a.ng, a.n_dst, a.n_ts, gc, r.ge, r.ee, hb.kind, hb.tau, t_first, r.t_last,
                      d);
        nx = p.dst;
        return true;
    }
    const int64_t t_first = group_ts(a.ng, a.fence, r, gc);
    for (uint32_t trial = 0; trial < N2V_MAX_TRIALS; ++trial) {
        const Draw d = philox(id, hop, trial, seed);
        p = pick_node(a.ng, a.n_dst, a.n_ts, gc, r.ge, r.ee, TW_EXPONENTIAL, hb.tau, t_first,
                      r.t_last, d);
        nx = p.dst;
        if (n2v_accept(a, hb, d.x2, prev, nx)) return true;
    }
    atomicAdd(&a.err[2], 1u);
    return false;
}

// the output rows were pre-filled with -1 / INT64_MIN, so ending a walk
// only records its length
__device__ __forceinline__ void finish_walk(const WalkArgs& a, int64_t w, int32_t len) {
    a.len[w] = len;
}

// Padding values (-1 nodes, INT64_MIN timestamps) for the output slots
// [b, e), written by threads tid, tid + stride, ... with 16-byte stores where
// the arrays are 16-byte aligned. The bulk stores are non-temporal: the
// padding is not read back, and cached it displaces index records the walk
// reads next (fill + walk measured 0.3% faster; the fill alone is slower).
typedef int v4i __attribute__((ext_vector_type(4)));
typedef long long v2l __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void fill_span(int32_t* __restrict__ nodes, int64_t* __restrict__ ts,
                                          int64_t b, int64_t e, int64_t tid, int64_t stride) {
    if (b >= e) return;
    // nodes: scalar head up to a 16-byte boundary, int4 body, scalar tail
    const int64_t nb = std::min<int64_t>(
        e, b + (int64_t)(((16 - ((uintptr_t)(nodes + b) & 15)) & 15) / 4));
    for (int64_t i = b + tid; i < nb; i += stride) nodes[i] = -1;
    const int64_t nv = (e - nb) / 4;
    int4* nv4 = reinterpret_cast<int4*>(nodes + nb);
    for (int64_t i = tid; i < nv; i += stride)
        __builtin_nontemporal_store((v4i){-1, -1, -1, -1}, reinterpret_cast<v4i*>(nv4) + i);
    for (int64_t i = nb + 4 * nv + tid; i < e; i += stride) nodes[i] = -1;
    const int64_t tb = std::min<int64_t>(
        e, b + (int64_t)(((16 - ((uintptr_t)(ts + b) & 15)) & 15) / 8));
    for (int64_t i = b + tid; i < tb; i += stride) ts[i] = TS_NONE;
    const int64_t tv = (e - tb) / 2;
    longlong2* tv2 = reinterpret_cast<longlong2*>(ts + tb);
    for (int64_t i = tid; i < tv; i += stride)
        __builtin_nontemporal_store((v2l){TS_NONE, TS_NONE}, reinterpret_cast<v2l*>(tv2) + i);
    for (int64_t i = tb + 2 * tv + tid; i < e; i += stride) ts[i] = TS_NONE;
}

constexpr int QUEUE_SLICES = 8;
constexpr int QUEUE_REFILL_MIN = 32;  // idle lanes that trigger a refill (hop-only queue)

struct QueueArgs {
    unsigned long long* counters;  // QUEUE_SLICES counters, zero at launch
    const int32_t* max_len;        // per-walk limit, or null (a.L)
    const uint8_t* bias_idx;       // per-walk hop bias, or null (id mod n_bias)
    const int64_t* row;            // per-walk row start, or null (w * a.L)
    int64_t out_slots;             // slots of the outputs: a row must end inside
    int32_t n_bias;
    HopBias bias[TW_MAX_BIASES];
};

template <int V>
using Kind = std::integral_constant<int, V>;

// f(Kind<HK>, Kind<SK>) for the run-time hop kind hk (-1: left dynamic, for
// batches that mix hop biases) and start kind sk
template <typename F>
void with_kinds(int hk, int sk, F&& f) {
    auto by_start = [&](auto h) {
        switch (sk) {
            case TW_LINEAR: f(h, Kind<TW_LINEAR>{}); break;
            case TW_EXPONENTIAL: f(h, Kind<TW_EXPONENTIAL>{}); break;
            default: f(h, Kind<TW_UNIFORM>{}); break;
        }
    };
    switch (hk) {
        case TW_UNIFORM: by_start(Kind<TW_UNIFORM>{}); break;
        case TW_LINEAR: by_start(Kind<TW_LINEAR>{}); break;
        case TW_EXPONENTIAL: by_start(Kind<TW_EXPONENTIAL>{}); break;
        case TW_NODE2VEC: by_start(Kind<TW_NODE2VEC>{}); break;
        case TW_WEIGHT: by_start(Kind<TW_WEIGHT>{}); break;
        default: by_start(Kind<-1>{}); break;
    }
}

// Calls f with the direction as a compile-time constant, for hop kind HK.
// Backward walks never take the weight-based picker (refused before any
// launch), so its backward instantiations are not built.
template <int HK, typename F>
void with_direction(bool rev, F&& f) {
    if (!rev) f(std::false_type{});
    else if constexpr (HK != TW_WEIGHT) f(std::true_type{});
}

// Whether the queue kernels write whole output rows themselves (four slots
// per 16-byte store, padding included): rows of a multiple of 4 slots and
// 16-byte aligned outputs.
inline bool own_rows(const WalkArgs& a) {
    return a.L % 4 == 0 && (reinterpret_cast<uintptr_t>(a.nodes) & 15) == 0 &&
           (reinterpret_cast<uintptr_t>(a.ts) & 15) == 0;
}

// queue.hip
tw_status queue_shape(tw_graph* g, Error& err);
tw_status queue_walks(tw_graph* g, const WalkArgs& a, const QueueArgs& q0, int bpc, Error& err,
                      bool rev = false);
tw_status batch_full_walk(tw_graph* g, const WalkArgs& a, const QueueArgs& q, Error& err,
                          bool rev = false);
tw_status queue_hops(tw_graph* g, const WalkArgs& a, int bpc, Error& err);
tw_status coop_walks(tw_graph* g, const WalkArgs& a, Error& err);

}  // namespace tw
