// Walk sampling (Tempest, Sec. "Temporal Bias Sampling" and "The Full-Walk
// Baseline"). A walk is keyed by (seed, walk id); hop h, trial r draws
// Philox4x64-10 at counter (id, h, r, 0), so every dispatch produces the
// same walks.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "walk_kernels.h"

namespace tw {
namespace {

// Fill every output slot with the padding values, fully coalesced, for the
// dispatches whose walks write only the slots they reach, and for walk blocks
// where their own padding takes longer (blocks_pad).
__global__ void k_fill_outputs(int32_t* __restrict__ nodes, int64_t* __restrict__ ts,
                               int64_t n) {
    fill_span(nodes, ts, 0, n, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
              (int64_t)gridDim.x * blockDim.x);
}

// ------------------------------------------------------------- walk blocks
//
// A wavefront runs a block of 64 walks, a lane each, and writes their rows
// whole: slots leave in chunks of eight through LDS, and when every walk of
// the block has ended the wavefront pads all its rows together. A rejected
// node2vec trial is an attempt of its own, so a lane whose trial was accepted
// goes on to its next hop while others try again.
//
// Large launches are bound by the random lines they read and the lines they
// write (4M exponential walks of length 80 on 100M edges: 5.6 TB/s of them, a
// copy reaches 4.7), small ones by the chain of dependent loads; what helps is
// wavefronts in flight (68 VGPRs for exponential hops, 76 to 78 for node2vec, 6.4
// KB of LDS: 6 a SIMD) and whole sectors in the writes. Against one walk per
// lane that padded its own row in chunks of four, with FP64 constants hoisted
// into 128 VGPRs (4 a SIMD): that launch 3.75 -> 2.96 ms; 1M uniform walks of 25
// slots on an undirected graph 817 -> 605 us (rows of any width are no longer
// pre-filled); 2M node2vec walks 3.71 -> 2.24 ms; 1M weight-based 1.01 -> 0.83
// ms; 1M backward exponential 1.02 -> 0.68 ms; 10,000 walks 22.1 -> 18.2 us.
// Also tried: blocks of 128 or 256 walks whose idle lanes take the next start
// from LDS (busy lanes 48 % instead of 34 % of an instruction's, but fewer
// wavefronts in flight: equal, node2vec 4 % faster, mixed batches 15 %
// slower); chunks of 4 (5 % slower) and 16 (10-40 % slower); workgroups of
// four wavefronts (10,000 walks 25.7 us against 20.3).

// The walks of a block (uniform over the wavefront): walk j of the block is
// walk w0 + j stride of its request, with RNG id id0 + j stride.
struct WalkBlock {
    int n;
    int64_t w0, stride;
    uint64_t id0;
    int32_t L;  // row width and length limit
    StartParams sp;
    HopBias hop;
    int32_t* nodes;
    int64_t* ts;
    int32_t* len;
    uint32_t* range_flag;  // a start node out of range
    uint32_t* cap_count;   // walks node2vec's trial cap ended
    // ragged blocks: per-walk length limits (null: L) and row starts (null:
    // rows of L slots) inside out_slots slots; a walk whose limit or row is
    // out of range sets *bad_flag and writes nothing
    const int32_t* limits;
    const int64_t* rows;
    int64_t out_slots;
    uint32_t* bad_flag;
    bool pad;  // the block pads its rows, of L slots (else the outputs were pre-filled)

    // nodes and ts 16-byte aligned: four slots leave as vectors
    __device__ __forceinline__ bool vec() const {
        return (((uintptr_t)nodes | (uintptr_t)ts) & 15) == 0;
    }
};

// LDS of a block: each lane's ring of its walk's current chunk (its own
// column), and the rows' first slots left to pad.
constexpr int CHUNK = 8;
struct BlockLds {
    int64_t ring_t[CHUNK][64];
    int32_t ring_n[CHUNK][64];
    int32_t at[64];
};

// LDS written by one lane of a wavefront and read by another: in program
// order for the hardware, so only the compiler has to keep it
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane's output row, from slot row0 of the outputs. Its slots are grouped
// in aligned chunks (ph: the row's first slot inside its first chunk), which
// leave for memory once their last slot is known, as 16-byte stores where four
// slots belong to the row: 32 bytes of nodes and a whole 64-byte sector of
// timestamps at once.
struct RowOut {
    const WalkBlock& b;
    BlockLds& m;
    int lane;
    int64_t row0;
    int32_t width;
    int ph;
    __device__ RowOut(const WalkBlock& b_, BlockLds& m_, int lane_, int64_t row, int32_t w)
        : b(b_), m(m_), lane(lane_), row0(row), width(w), ph((int)(row & (CHUNK - 1))) {}
    // The row's slots [from, to) of the chunk at slot q (a multiple of CHUNK);
    // the slots from `known` on are padding.
    __device__ __forceinline__ void store(int64_t q, int from, int to, int known) const {
        const int64_t at = row0 - ph + q;
#pragma unroll
        for (int k0 = 0; k0 < CHUNK; k0 += 4) {
            int32_t v[4];
            int64_t x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = k0 + i < known ? m.ring_n[k0 + i][lane] : -1;
                x[i] = k0 + i < known ? m.ring_t[k0 + i][lane] : TS_NONE;
            }
            int32_t* n = b.nodes + at + k0;
            int64_t* t = b.ts + at + k0;
            if (b.vec() && from <= k0 && k0 + 4 <= to) {
                *reinterpret_cast<int4*>(n) = make_int4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<longlong2*>(t) = make_longlong2(x[0], x[1]);
                *reinterpret_cast<longlong2*>(t + 2) = make_longlong2(x[2], x[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k0 + i >= from && k0 + i < to) {
                        n[i] = v[i];
                        t[i] = x[i];
                    }
            }
        }
    }
    __device__ __forceinline__ void push(int32_t p, int32_t v, int64_t t) const {
        const int64_t q = (int64_t)ph + p;
        const int r = (int)(q & (CHUNK - 1));
        m.ring_n[r][lane] = v;
        m.ring_t[r][lane] = t;
        if (r == CHUNK - 1) store(q - r, q - r < ph ? ph : 0, CHUNK, CHUNK);
    }
    // Ends a row of len slots: the chunk of the last slot is completed with
    // padding up to the row's end. Returns the first slot left to the padding
    // passes.
    __device__ __forceinline__ int32_t finish(int32_t len) const {
        const int64_t q = (int64_t)ph + len;
        const int r = (int)(q & (CHUNK - 1));
        if (len == 0 || r == 0) return len;
        const int64_t c = q - r, end = (int64_t)ph + width - c;
        store(c, c < ph ? ph : 0, end < CHUNK ? (int)end : CHUNK, r);
        const int64_t at = c + CHUNK - ph;
        return at < width ? (int32_t)at : width;
    }
};

// Padding of one row from slot `at` to its end by `lanes` lanes (this one
// is lane `sub`): consecutive lanes write consecutive 16 bytes.
__device__ __forceinline__ void pad_row(int32_t* __restrict__ nodes, int64_t* __restrict__ ts,
                                        int64_t row0, int64_t at, int32_t width, bool vec, int sub,
                                        int lanes) {
    const int64_t b = row0 + at, e = row0 + width;
    if (!vec) {
        for (int64_t s = b + sub; s < e; s += lanes) {
            nodes[s] = -1;
            ts[s] = TS_NONE;
        }
        return;
    }
    const int64_t vb = (b + 3) & ~3ll, ve = e & ~3ll;  // whole chunks
    const int64_t head = vb < e ? vb : e;
    if (b + sub < head) {
        nodes[b + sub] = -1;
        ts[b + sub] = TS_NONE;
    }
    for (int64_t s = vb + 4 * sub; s < ve; s += 4 * lanes)
        *reinterpret_cast<int4*>(nodes + s) = make_int4(-1, -1, -1, -1);
    for (int64_t s = vb + 2 * sub; s < ve; s += 2 * lanes)
        *reinterpret_cast<longlong2*>(ts + s) = make_longlong2(TS_NONE, TS_NONE);
    if (ve >= vb && ve + sub < e) {
        nodes[ve + sub] = -1;
        ts[ve + sub] = TS_NONE;
    }
}

// Padding of a block of n rows of L slots each from slot s0 of the outputs,
// row r from its slot at[r] on: groups of four slots of the whole block over
// consecutive lanes, so a store instruction covers 1 KB without a gap. The
// row of a slot comes from a multiplication, exact for L < 4096.
constexpr int PAD_FLAT_MIN_L = 4, PAD_FLAT_MAX_L = 4096;
__device__ __forceinline__ void pad_rows_flat(int32_t* __restrict__ nodes, int64_t* __restrict__ ts,
                                              int64_t s0, int n, int32_t L, const int32_t* at,
                                              int lane) {
    const uint32_t inv = 0xFFFFFFFFu / (uint32_t)L + 1u;  // ceil(2^32 / L)
    const int ph = (int)(s0 & 3);
    int32_t* on = nodes + (s0 - ph);
    int64_t* ot = ts + (s0 - ph);
    const int quads = (ph + n * L + 3) >> 2;
    // whether quad c lies in one row; its first own slot's row and place there
    auto place = [&](int c, int& r, int& p) {
        const int x = 4 * c - ph, y = x < 0 ? 0 : x;
        r = (int)__umulhi((uint32_t)y, inv);
        p = y - r * L;
        return x >= 0 && p + 4 <= L;
    };
    // (a row's `at` is a multiple of four from the aligned start, or its end)
#pragma unroll 2
    for (int c = lane; c < quads; c += 64) {
        int r, p;
        if (place(c, r, p)) {
            if (p >= at[r]) *reinterpret_cast<int4*>(on + 4 * c) = make_int4(-1, -1, -1, -1);
        } else {  // a quad that ends one row and begins the next (or an end of the block)
            for (int q = 4 * c < ph ? ph : 4 * c; q < 4 * c + 4 && r < n; ++q) {
                if (p >= at[r]) {
                    on[q] = -1;
                    ot[q] = TS_NONE;
                }
                if (++p == L) {
                    ++r;
                    p = 0;
                }
            }
        }
    }
#pragma unroll 4
    for (int h = lane; h < 2 * quads; h += 64) {
        int r, p;
        if (place(h >> 1, r, p) && p >= at[r])
            *reinterpret_cast<longlong2*>(ot + 2 * h) = make_longlong2(TS_NONE, TS_NONE);
    }
}

// The candidates of a hop: groups [c0, c1) of a node with edges ending at
// end, their first and last timestamps, the node's first live group.
struct Candidates {
    uint32_t c0, c1, end, gb;
    int64_t t_lo, t_hi;
};

// Gamma_t of the node of record r: forward the groups after t, backward (on
// the in-view) those before t; false when there is none. rate: the pick reads
// the first candidate's timestamp. (node2vec, which reads the group's record in
// every trial, searches as ever: its kernels take 76 to 80 VGPRs, backward batches
// with linear or exponential starts 82, and from 81 on five wavefronts a SIMD fit
// instead of six.)
template <bool REV>
__device__ __forceinline__ bool candidates(const WalkArgs& a, const NodeRec& r, int64_t t,
                                           bool rate, bool n2v, Candidates& c) {
    c.gb = r.gb;
    if (!REV) {
        if (t >= r.t_last) return false;
        c.c1 = r.ge;
        c.end = r.ee;
        c.t_hi = r.t_last;
        if (!n2v && t >= r.t_prev) {  // the last group only
            c.c0 = r.ge - 1;
            c.t_lo = r.t_last;
            return true;
        }
        c.c0 = fence_search(a.ng, a.fence, r, t, nullptr, 0, 0);
        c.t_lo = rate ? group_ts(a.ng, a.fence, r, c.c0) : 0;
        return true;
    }
    if (r.gb == r.ge) return false;
    // the first group at or after t (first with a timestamp > t - 1)
    const uint32_t hi = t - 1 >= r.t_last
                            ? r.ge
                            : fence_search(a.ng, a.fence, r, t - 1, nullptr, 0, 0);
    if (hi == r.gb) return false;
    c.c0 = r.gb;
    c.c1 = hi;
    c.end = hi < r.ge ? a.ng[hi].first : r.ee;
    c.t_lo = rate ? group_ts(a.ng, a.fence, r, r.gb) : 0;
    c.t_hi = rate ? group_ts(a.ng, a.fence, r, hi - 1) : 0;
    return true;
}

// The pick when a node's last group is the one candidate (weight-based: a
// one-edge group only, its edges are picked by weight): from the node record
// alone, but for a group of several edges.
__device__ __forceinline__ Pick pick_last(const int32_t* __restrict__ n_dst, const NodeRec& r,
                                          int kind, const Draw& d) {
    if (r.last_dst < 0) return Pick{r.last_dst & 0x7fffffff, r.t_last};
    const uint32_t j =
        (uint32_t)scale_u64(kind == TW_UNIFORM ? d.x0 : d.x1, r.ee - r.last_first);
    return Pick{n_dst[r.last_first + j], r.t_last};
}

// keeps a value's computation above this point (a draw made while a load
// it does not need is in flight)
__device__ __forceinline__ void computed_here(uint64_t& x) { asm volatile("" : "+v"(x)); }

// The walks of block b, by one wavefront (b.n <= 64). RAGGED: per-walk limits
// and rows. NEST (node2vec): a lane whose trial was rejected tries again at once,
// and the others wait for it. Returns the length of the lane's walk.
template <int HK, int SK, bool REV, bool RAGGED, bool NEST = false>
__device__ __forceinline__ int32_t walk_block(const WalkArgs& a, const WalkBlock& b, BlockLds& m) {
    const int lane = threadIdx.x & 63;
    const HopBias hb = fixed_hop<HK>(b.hop);
    const StartParams sp = fixed_start<SK>(b.sp);
    const bool n2v = hb.kind == TW_NODE2VEC;
    const int64_t w = b.w0 + lane * b.stride;
    const uint64_t id = b.id0 + (uint64_t)(lane * b.stride);
    const bool mine = lane < b.n;
    int32_t limit = b.L, width = b.L;
    int64_t row0 = w * (int64_t)b.L;
    if (RAGGED && mine) {
        if (b.limits) limit = b.limits[w];
        if (b.rows) {
            row0 = b.rows[w];
            width = limit;
        }
        // (no sum: a row start near INT64_MAX would wrap past the check)
        if (limit < 1 || limit > b.L || row0 < 0 || row0 > b.out_slots - limit) {
            atomicOr(b.bad_flag, 1u);
            limit = 0;
        } else if (row0 + width > b.out_slots) {
            width = (int32_t)(b.out_slots - row0);  // the last row of outputs cut short
        }
    }
    StartState st{0, 0, 0, 0, -1};
    if (mine && limit > 0) st = walk_start(a, sp, w, id, limit, nullptr, nullptr, REV, b.range_flag);
    const RowOut row(b, m, lane, row0, width);
    int32_t len = st.len, cur = st.cur, prev = st.prev;
    int64_t t = st.t;
    if (len >= 1) row.push(0, st.first, TS_NONE);
    if (len >= 2) row.push(1, cur, t);
    bool active = len >= 2 && len < limit;
    uint32_t trial = 0;
    Candidates c{};
    ExpLaw law{};
    while (active) {
        const bool fresh = !n2v || trial == 0;
        NodeRec r;
        if (fresh) r = a.rec[cur];
        // hop len - 1 of the walk; drawn while the record is on its way, except
        // for node2vec, which needs the registers
        Draw d;
        if (!n2v) {
            d = philox(id, (uint64_t)(len - 1), 0, sp.seed);
            computed_here(d.x0);
        }
        bool live = true;
        if (fresh) {
            live = candidates<REV>(a, r, t, reads_first_ts(hb.kind), n2v, c);
            if (n2v && live)
                law = exp_law(c.c1 - c.c0, exp_lambda(c.t_lo, c.t_hi, c.c1 - c.c0, hb.tau));
        }
        if (n2v) d = philox(id, (uint64_t)(len - 1), trial, sp.seed);
        if (!live) {
            active = false;
            continue;
        }
        Pick p;
        bool take = true;
        if (!REV && !n2v && c.c0 + 1 == c.c1 && (hb.kind != TW_WEIGHT || r.last_dst < 0)) {
            p = pick_last(a.n_dst, r, hb.kind, d);
        } else if (!REV && hb.kind == TW_WEIGHT) {
            p = pick_weight(a.ng, a.n_dst, a.cw, c.gb, c.c0, c.c1, c.end,
                            hb.tau > 0.0 ? hb.tau : 1.0, group_ts(a.ng, a.fence, r, c.c0), c.t_hi,
                            d);
        } else if (n2v) {
            while (true) {
                const uint32_t i = exp_draw(law, d.x0);
                p = edge_of_group(a.ng, a.n_dst, c.c1, c.end, REV ? c.c1 - 1 - i : c.c0 + i, d,
                                  REV);
                // the edge prev -> candidate (backward: candidate -> prev of the
                // graph, which is prev -> candidate of the in-view)
                take = n2v_accept(a, hb, d.x2, prev, p.dst);
                if (!NEST || take || trial + 1 == N2V_MAX_TRIALS) break;
                d = philox(id, (uint64_t)(len - 1), ++trial, sp.seed);
            }
        } else {
            p = pick_node(a.ng, a.n_dst, a.n_ts, c.c0, c.c1, c.end, hb.kind, hb.tau, c.t_lo,
                          c.t_hi, d, REV);
        }
        if (take) {
            row.push(len, p.dst, p.t);
            ++len;
            trial = 0;
            prev = cur;
            cur = p.dst;
            t = p.t;
            active = len < limit;
        } else if (++trial == N2V_MAX_TRIALS) {
            atomicAdd(b.cap_count, 1u);
            active = false;
        }
    }
    if (mine) {
        b.len[w] = len;
        const int32_t at = row.finish(len);
        m.at[lane] = at;
    }
    if (!b.pad) return len;
    wave_lds_fence();
    if (!RAGGED && b.vec() && b.L >= PAD_FLAT_MIN_L && b.L < PAD_FLAT_MAX_L) {
        pad_rows_flat(b.nodes, b.ts, b.w0 * (int64_t)b.L, b.n, b.L, m.at, lane);
        return len;
    }
    // 16 lanes a row
    for (int k = lane >> 4; k < b.n; k += 4)
        pad_row(b.nodes, b.ts, (b.w0 + k * b.stride) * (int64_t)b.L, m.at[k], b.L, b.vec(), lane & 15,
                16);
    return len;
}

// The full-walk dispatch (Sec. "The Full-Walk Baseline"), forward and (REV, on
// the in-view) backward: contiguous blocks, a workgroup of one wavefront each.
template <int HK, int SK, bool REV, bool NEST = false>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
k_walk_full(const WalkArgs a) {
    __shared__ BlockLds lds;
    WalkBlock b;
    b.w0 = (int64_t)blockIdx.x * 64;
    b.n = (int)std::min<int64_t>(64, a.num_walks - b.w0);
    b.stride = 1;
    b.id0 = a.base + (uint64_t)b.w0;
    b.L = a.L;
    b.sp = start_of(a);
    b.hop = a.hop;
    b.nodes = a.nodes;
    b.ts = a.ts;
    b.len = a.len;
    b.range_flag = &a.err[0];
    b.cap_count = &a.err[2];
    b.pad = !a.pre_filled;
    walk_block<HK, SK, REV, false, NEST>(a, b, lds);
}

// A batch in walk blocks. With several biases assigned by walk id (id mod
// n_bias), a block takes the walks of one bias of a stretch of n_bias x 64
// walks, so its wavefront runs one picker: lanes of six different biases ran
// all six pickers one after the other. only >= 0: the launch runs the biases'
// `only`-th walks of every stretch, with that bias's kernel (8M walks of
// lengths 5-120 and six biases on a 40M-record graph: 12.7 ms with per-lane
// biases on a work queue and a fill pass before it, 10.0 with one launch of
// this kernel at 128 VGPRs, 6.95 with one launch a bias); else the blocks of a
// stretch go to one XCD (every eighth workgroup), where the lines that
// their rows share meet in its L2. The blocks pad their rows unless the outputs
// are pre_filled.
template <int HK, int SK, bool REV>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
k_walk_batch(const WalkArgs a, const QueueArgs q, int only) {
    __shared__ BlockLds lds;
    const int nb = q.n_bias;
    WalkBlock b;
    b.stride = nb;
    if (only >= 0) {
        b.w0 = (int64_t)blockIdx.x * nb * 64 + only;
    } else {
        const uint32_t xcd = blockIdx.x % NUM_XCD, i = blockIdx.x / NUM_XCD;
        b.w0 = ((int64_t)(i / nb) * NUM_XCD + xcd) * nb * 64 + i % nb;
    }
    if (b.w0 >= a.num_walks) return;
    b.n = (int)std::min<int64_t>(64, (a.num_walks - b.w0 + nb - 1) / nb);
    b.id0 = a.base + (uint64_t)b.w0;
    b.L = a.L;
    b.sp = start_of(a);
    b.hop = q.bias[b.id0 % (uint64_t)nb];
    b.nodes = a.nodes;
    b.ts = a.ts;
    b.len = a.len;
    b.range_flag = &a.err[0];
    b.cap_count = &a.err[2];
    b.limits = q.max_len;
    b.rows = q.row;
    b.out_slots = q.out_slots;
    b.bad_flag = &a.err[3];
    b.pad = !a.pre_filled;
    walk_block<HK, SK, REV, true>(a, b, lds);
}

// ----------------------------------------------------------------- serve
//
// A serving launch: the walks of several requests, each with its own seed,
// id base, length limit, hop and start bias, start nodes and output rows, in
// walk blocks: a block's walks are all of one request (the last one of a
// request may be partial), so its parameters are uniform over the wavefront, it
// runs one picker, and it writes its rows whole. A request's result does not
// depend on what else shares the launch.

constexpr int SERVE_MAX_REQ = 1024;

struct ServeReqDev {
    int64_t block0, count;  // first block of the launch, walks
    uint64_t seed, base;
    int32_t L, start_kind, start_mode, pre_filled;
    double start_tau;
    HopBias hop;
    const int32_t* start_nodes;
    int32_t* nodes;
    int64_t* ts;
    int32_t* len;
    uint32_t* err;  // the request's own words: [0] start node out of range, [1] trial-cap hits
};

// the outputs of the requests whose blocks do not pad their rows, request
// blockIdx.y each
__global__ void k_fill_requests(const ServeReqDev* __restrict__ reqs) {
    const ServeReqDev& R = reqs[blockIdx.y];
    if (R.pre_filled)
        fill_span(R.nodes, R.ts, 0, R.count * (int64_t)R.L,
                  (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// REV: backward requests on the in-view. Before, lanes took walks of any
// request from a work queue (per-lane parameters, about 180 VGPRs held to 3
// waves a SIMD) into rows that one fill launch per request had padded: 16
// requests of 100 to 10,000 mixed walks 397 + 36 us of fills -> 316 us.
template <bool REV>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4)))
k_walk_serve(const WalkArgs a, const ServeReqDev* __restrict__ reqs, int nreq, int64_t block0,
             unsigned long long* hops_out) {
    __shared__ BlockLds lds;
    const int lane = threadIdx.x;
    const int64_t block = block0 + blockIdx.x;
    // the block's request: the last one that starts at or before it (requests
    // without walks start where the next one does)
    int k = -1;
    for (int i = 0; i < nreq; i += 64)
        k += __popcll(__ballot(i + lane < nreq && reqs[i + lane].block0 <= block));
    const ServeReqDev& R = reqs[__builtin_amdgcn_readfirstlane(k)];
    WalkBlock b;
    b.w0 = (block - R.block0) * 64;
    b.n = (int)std::min<int64_t>(64, R.count - b.w0);
    b.stride = 1;
    b.id0 = R.base + (uint64_t)b.w0;
    b.L = R.L;
    b.sp = StartParams{R.seed, R.start_kind, R.start_mode, R.start_tau, R.start_nodes};
    b.hop = R.hop;
    b.nodes = R.nodes;
    b.ts = R.ts;
    b.len = R.len;
    b.range_flag = R.err;
    b.cap_count = R.err + 1;
    b.pad = R.pre_filled == 0;
    const int32_t len = walk_block<-1, -1, REV, false>(a, b, lds);
    // hops of the launch: one atomic a block
    int32_t hops = len > 1 ? len - 1 : 0;
    for (int off = 32; off > 0; off >>= 1) hops += __shfl_down(hops, off, 64);
    if (lane == 0 && hops) atomicAdd(hops_out, (unsigned long long)hops);
}

bool valid_tau(double t) { return std::isfinite(t); }

tw_status check_bias(const tw_bias& b, bool hop, Error& err) {
    if (b.kind < TW_UNIFORM || b.kind > (hop ? TW_WEIGHT : TW_EXPONENTIAL) || !valid_tau(b.tau)) {
        err = Error{TW_EINVAL, "sample_walks: bad bias kind or tau (start bias cannot be node2vec)"};
        return err.code;
    }
    if (b.kind == TW_NODE2VEC &&
        !(b.p > 0.0 && b.q > 0.0 && std::isfinite(b.p) && std::isfinite(b.q))) {
        err = Error{TW_EINVAL, "sample_walks: node2vec needs p > 0 and q > 0"};
        return err.code;
    }
    return TW_OK;
}

tw_status check_start(int mode, const int32_t* starts, int64_t num_walks, Error& err) {
    if (mode != TW_START_EDGE && mode != TW_START_NODE) {
        err = Error{TW_EINVAL, "sample_walks: bad start mode"};
        return err.code;
    }
    if (mode == TW_START_NODE && !starts && num_walks > 0) {
        err = Error{TW_EINVAL, "sample_walks: start mode NODE needs d_start_nodes"};
        return err.code;
    }
    return TW_OK;
}

// The index part of the walk arguments and the common parameters.
// Walk arguments over the graph's current views. node2vec: the adjacency
// is needed; weight_tau (NaN: none) the cumulative weights at that scale.
tw_status fill_args(tw_graph* g, int64_t num_walks, int32_t L, const tw_bias& sb, int start_mode,
                    const int32_t* starts, uint64_t seed, uint64_t base, bool node2vec,
                    double weight_tau, int32_t* nodes, int64_t* ts, int32_t* len, WalkArgs& a,
                    Error& err) {
    if (!g->rec.p && init_empty(g, err) != TW_OK) return err.code;
    if (node2vec && g->m > 0 && build_adjacency(g, err) != TW_OK) return err.code;
    if (!std::isnan(weight_tau) && build_weights(g, weight_tau, err) != TW_OK) return err.code;
    a = WalkArgs{};
    a.e_src = g->e_src.as<int32_t>();
    a.e_dst = g->e_dst.as<int32_t>();
    a.e_ts = g->e_ts.as<int64_t>();
    a.wsum = g->scal.as<int64_t>() + SLOT_I64_SUMMARY;
    a.wgg = g->scal.as<int64_t>() + SLOT_I64_GG;
    a.gg_off = g->gg_off.as<uint32_t>();
    a.win = g->scal.as<int64_t>() + SLOT_I64_WIN;
    a.n_dst = g->n_dst.as<int32_t>();
    a.n_ts = g->n_ts.as<int64_t>();
    a.ng = g->ng.as<GroupRec>();

    a.rec = g->rec.as<NodeRec>();
    a.fence = g->fence.as<uint32_t>();
    a.adj_tab = g->adj_tab.as<AdjSlot>();
    a.adj_mask = g->adj_mask;
    a.cw = g->cw.as<double>();
    a.V = g->V;
    a.num_walks = num_walks;
    a.L = L;
    a.start_kind = sb.kind;
    a.start_mode = start_mode;
    a.start_tau = sb.tau;
    a.start_nodes = starts;
    a.seed = seed;
    a.base = base;
    a.nodes = nodes;
    a.ts = ts;
    a.len = len;
    a.err = g->err.as<uint32_t>();
    return TW_OK;
}

// workgroups of a fill of `slots` slots, at most `most`
constexpr int64_t FILL_BLOCKS = 8192;
unsigned fill_grid(int64_t slots, int64_t most) {
    return (unsigned)std::max<int64_t>(
        std::min<int64_t>(ceil_div(slots, 4 * WALK_THREADS), most), 1);
}

void launch_fill(tw_graph* g, int32_t* nodes, int64_t* ts, int64_t slots) {
    hipLaunchKernelGGL(k_fill_outputs, dim3(fill_grid(slots, FILL_BLOCKS)), dim3(WALK_THREADS), 0,
                       g->stream, nodes, ts, slots);
}

// Most walks one launch of walk blocks takes: a launch holds fewer than 2^32
// threads (a batch's grid is rounded up to eight stretches of 64 walks a bias).
constexpr int64_t BLOCK_MAX_WALKS = (1ll << 32) - 8 * 64 * (TW_MAX_BIASES + 1);

// Whether `blocks` walk blocks pad their own rows (of L slots), or the outputs
// are filled in a launch of their own first. A block's padding is one
// wavefront's work after its longest walk (about 10 GB/s of it), the fill is the
// whole chip's: in few blocks the padding of wide rows is a serial tail (64 linear
// walks of 10,001 slots 341 us, filled first 58; 1,000 of 1,000 128 and 61; of
// 80 slots 63 and 60). With a wavefront on most SIMDs it hides under other
// blocks' walks while the outputs fit the 256 MB last-level cache (64,000 of
// 160 89 and 99; 256,000 of 500 513 and 404), and with rows so long that a launch
// is their bandwidth alone: there the fill's slots and the walks' are written one
// launch after the other (128,000 of 4,000 1.27 and 1.32 ms). From 4,096 slots on
// a block pads row by row, at about 27 GB/s, and fewer blocks do, fewest where
// every row begins on 16 bytes (16,000 of 4,096 203 and 211 us; of 5,001 264 and
// 242; 32,000 of 5,001 452 and 460). Walks end after a few hops, so the slots that
// a fill writes in vain are few.
constexpr int64_t PAD_MAX_L = 96, PAD_MIN_BLOCKS = 600, PAD_MAX_SLOTS = 320 << 10;
constexpr int64_t PAD_LONG_L = 3072;
bool blocks_pad(int64_t blocks, int64_t L) {
    if (L <= PAD_MAX_L) return true;
    if (L >= PAD_FLAT_MAX_L) return blocks > (L % 4 == 0 ? 192 : 400);
    return blocks > PAD_MIN_BLOCKS && (L >= PAD_LONG_L || blocks <= PAD_MAX_SLOTS / L);
}

// Whether node2vec walks of at most L nodes retry rejected trials at once
// (NEST). Interleaved with other lanes' next hops a retry costs a whole
// iteration, the search of a hop included, as long as some lane begins one: over
// many hops a lane's trials even out and the block ends sooner, over two to six
// hops its unluckiest lane sets the pace (50,000 walks of 4 nodes, p = 2, q = 1/2:
// 84 us, nested 71; of 8 139 and 134; of 12 166 and 180). Once the launch fills the
// chip, wavefronts in flight decide (76 VGPRs, nested 82; 1.5M walks of 8 nodes
// 0.74 and 0.87 ms, 400,000 of 4 0.18 and 0.16), and with few blocks seven nodes
// are many already (1,000 walks of 8 94 and 98 us).
bool n2v_nested(int64_t blocks, int64_t L) {
    if (L <= 6) return blocks <= (L == 4 ? 8192 : 2048);
    return L <= 8 && blocks > 256 && blocks <= 1600;
}

// the full-walk kernel, after a fill of the outputs where its blocks do not
// pad their rows
tw_status full_walks(tw_graph* g, WalkArgs a, bool rev, Error& err) {
    a.pre_filled = !blocks_pad(ceil_div(a.num_walks, 64), a.L);
    if (a.pre_filled) launch_fill(g, a.nodes, a.ts, a.num_walks * (int64_t)a.L);
    const dim3 grid((unsigned)ceil_div(a.num_walks, 64));
    const bool nest = n2v_nested(grid.x, a.L);
    with_kinds(a.hop.kind, a.start_kind, [&](auto h, auto st) {
        constexpr int HK = decltype(h)::value, SK = decltype(st)::value;
        // (these walks share one hop kind)
        if constexpr (HK >= 0)
            with_direction<HK>(rev, [&](auto r) {
                constexpr bool REV = decltype(r)::value;
                if (HK == TW_NODE2VEC && nest)
                    hipLaunchKernelGGL((k_walk_full<HK, SK, REV, HK == TW_NODE2VEC>), grid, dim3(64),
                                       0, g->stream, a);
                else
                    hipLaunchKernelGGL((k_walk_full<HK, SK, REV>), grid, dim3(64), 0, g->stream, a);
            });
    });
    TW_HIP(hipGetLastError());
    return TW_OK;
}

// A batch whose biases go by walk id, in walk blocks.
tw_status batch_blocks(tw_graph* g, WalkArgs a, const QueueArgs& q, Error& err, bool rev) {
    if (queue_shape(g, err) != TW_OK) return err.code;
    hipStream_t s = g->stream;
    // whichever batch comes first: a later one may run on the queue under graph
    // capture, which must not allocate
    TW_HIP(ensure(g->wq, sizeof(unsigned long long) * QUEUE_SLICES, s));
    // Rows of L slots that cover the outputs are padded by their blocks, as plain
    // walks' are. Given rows are filled first: whether they cover every slot
    // would have to be checked on the device, and checked and padded by the blocks
    // they took longer at every size (1M linear walks of 5-120 slots 732 us, filled
    // first 665; 8M exponential ones 5.80 and 5.35 ms; 250,000 of 1-60 slots with
    // gaps between the rows 151 and 101 us).
    const int64_t W = a.num_walks, slots = q.out_slots, used = W * (int64_t)a.L;
    a.pre_filled = q.row || slots < used || !blocks_pad(ceil_div(W, 64), a.L);
    if (a.pre_filled)
        launch_fill(g, a.nodes, a.ts, slots);
    else if (slots > used)
        launch_fill(g, a.nodes + used, a.ts + used, slots - used);
    const int nb = q.n_bias;
    const int64_t stretches = ceil_div(W, (int64_t)64 * nb);
    auto launch = [&](int hk, int only) {
        const dim3 grid((unsigned)(only >= 0 ? stretches
                                             : ceil_div(stretches, NUM_XCD) * NUM_XCD * nb));
        with_kinds(hk, a.start_kind, [&](auto h, auto st) {
            with_direction<decltype(h)::value>(rev, [&](auto r) {
                hipLaunchKernelGGL((k_walk_batch<decltype(h)::value, decltype(st)::value,
                                                 decltype(r)::value>),
                                   grid, dim3(64), 0, s, a, q, only);
            });
        });
    };
    // Several biases: one launch a bias, with the kernel that carries that
    // picker only, where each fills the chip; else one launch of the kernel
    // that carries all of them.
    if (nb == 1) {
        launch(q.bias[0].kind, -1);
    } else if (W / nb < (int64_t)g->cu_count * 16 * 64) {
        launch(-1, -1);
    } else {
        for (int o = 0; o < nb; ++o)
            launch(q.bias[(a.base + (uint64_t)o) % (uint64_t)nb].kind, o);
    }
    TW_HIP(hipGetLastError());
    return TW_OK;
}

// run the walks of `a` under a dispatch; the output rows are padded first
// unless the walk kernel writes them whole
tw_status run_dispatch(tw_graph* g, const WalkArgs& a, int dispatch, int bpc, Error& err) {
    if (dispatch == TW_DISPATCH_FULL_WALK) return full_walks(g, a, false, err);
    if (dispatch != TW_DISPATCH_QUEUE || !own_rows(a))
        launch_fill(g, a.nodes, a.ts, a.num_walks * (int64_t)a.L);
    if (dispatch == TW_DISPATCH_COOP) return coop_walks(g, a, err);
    return queue_hops(g, a, bpc, err);
}

tw_status prepare_plain(tw_graph* g, const tw_walk_params* p, int32_t* nodes, int64_t* ts,
                        int32_t* len, WalkArgs& a, Error& err) {
    if (!p || p->num_walks < 0 || p->max_len < 1) {
        err = Error{TW_EINVAL, "sample_walks: need num_walks >= 0 and max_len >= 1"};
        return err.code;
    }
    if (check_bias(p->hop_bias, true, err) != TW_OK) return err.code;
    if (check_bias(p->start_bias, false, err) != TW_OK) return err.code;
    if (check_start(p->start_mode, p->d_start_nodes, p->num_walks, err) != TW_OK) return err.code;
    if (p->dispatch < TW_DISPATCH_AUTO || p->dispatch > TW_DISPATCH_QUEUE) {
        err = Error{TW_EINVAL, "sample_walks: bad dispatch"};
        return err.code;
    }
    if (p->num_walks > 0 && (!nodes || !ts || !len)) {
        err = Error{TW_EINVAL, "sample_walks: null output"};
        return err.code;
    }
    if (fill_args(g, p->num_walks, p->max_len, p->start_bias, p->start_mode, p->d_start_nodes,
                  p->seed, p->walk_id_base, p->hop_bias.kind == TW_NODE2VEC,
                  p->hop_bias.kind == TW_WEIGHT ? p->hop_bias.tau : NAN, nodes, ts, len, a,
                  err) != TW_OK)
        return err.code;
    a.hop = make_hop_bias(p->hop_bias);
    return TW_OK;
}

}  // namespace

// Backward walks on the in-view: the full-walk kernel (AUTO,
// FULL_WALK) or the work queue (QUEUE).
tw_status sample_backward(tw_graph* g, const tw_walk_params* p, int32_t* nodes, int64_t* ts,
                          int32_t* len, Error& err) {
    if (p->hop_bias.kind == TW_WEIGHT) {
        err = Error{TW_EINVAL, "sample_walks: the weight-based picker walks forward only"};
        return err.code;
    }
    if (p->dispatch == TW_DISPATCH_COOP) {
        err = Error{TW_EINVAL,
                    "sample_walks: backward walks run on the full-walk or the queue dispatch"};
        return err.code;
    }
    tw_graph* b = nullptr;
    if (backward_view(g, &b, err) != TW_OK) return err.code;
    WalkArgs a;
    if (prepare_plain(b, p, nodes, ts, len, a, err) != TW_OK) return err.code;
    if (p->num_walks == 0) return TW_OK;
    if (p->dispatch == TW_DISPATCH_QUEUE) {
        // the work queue with the one hop bias
        launch_fill(b, nodes, ts, p->num_walks * (int64_t)p->max_len);
        QueueArgs q{};
        q.n_bias = 1;
        q.bias[0] = a.hop;
        q.out_slots = p->num_walks * (int64_t)p->max_len;
        return queue_walks(b, a, q, g->auto_bpc, err, true);
    }
    return full_walks(b, a, true, err);
}

tw_status sample_walks(tw_graph* g, const tw_walk_params* p, int32_t* nodes, int64_t* ts,
                       int32_t* len, Error& err) {
    if (p && p->direction == TW_BACKWARD) return sample_backward(g, p, nodes, ts, len, err);
    if (p && p->direction != TW_FORWARD) {
        err = Error{TW_EINVAL, "sample_walks: bad direction"};
        return err.code;
    }
    WalkArgs a;
    if (prepare_plain(g, p, nodes, ts, len, a, err) != TW_OK) return err.code;
    if (p->num_walks == 0) return TW_OK;
    int dispatch = p->dispatch;
    // AUTO: the autotuned choice, else the full-walk kernel
    if (dispatch == TW_DISPATCH_AUTO)
        dispatch = g->auto_dispatch ? g->auto_dispatch : TW_DISPATCH_FULL_WALK;
    return run_dispatch(g, a, dispatch, g->auto_bpc, err);
}

tw_status sample_walks_batch(tw_graph* g, const tw_batch_params* p, int32_t* nodes, int64_t* ts,
                             int32_t* len, Error& err) {
    if (!p || p->num_walks < 0 || p->max_len < 1 || p->num_biases < 1 ||
        p->num_biases > TW_MAX_BIASES) {
        err = Error{TW_EINVAL,
                    "sample_walks_batch: need num_walks >= 0, max_len >= 1, 1..8 hop biases"};
        return err.code;
    }
    bool n2v = false;
    double wtau = NAN;  // the weight-based biases' time scale: one per launch
    for (int b = 0; b < p->num_biases; ++b) {
        const tw_bias& hb = p->hop_biases[b];
        if (check_bias(hb, true, err) != TW_OK) return err.code;
        n2v |= hb.kind == TW_NODE2VEC;
        if (hb.kind == TW_WEIGHT) {
            const double sc = hb.tau > 0.0 ? hb.tau : 1.0;
            if (!std::isnan(wtau) && wtau != sc) {
                err = Error{TW_EINVAL,
                            "sample_walks_batch: weight-based biases of one launch need one tau"};
                return err.code;
            }
            wtau = sc;
        }
    }
    if (check_bias(p->start_bias, false, err) != TW_OK) return err.code;
    if (check_start(p->start_mode, p->d_start_nodes, p->num_walks, err) != TW_OK) return err.code;
    if (p->dispatch != TW_DISPATCH_AUTO && p->dispatch != TW_DISPATCH_QUEUE &&
        p->dispatch != TW_DISPATCH_FULL_WALK) {
        err = Error{TW_EINVAL, "sample_walks_batch: dispatch must be AUTO, QUEUE or FULL_WALK"};
        return err.code;
    }
    if (p->direction != TW_FORWARD && p->direction != TW_BACKWARD) {
        err = Error{TW_EINVAL, "sample_walks_batch: bad direction"};
        return err.code;
    }
    const bool rev = p->direction == TW_BACKWARD;
    if (rev && !std::isnan(wtau)) {
        err = Error{TW_EINVAL, "sample_walks_batch: the weight-based picker walks forward only"};
        return err.code;
    }
    if (p->num_walks == 0) return TW_OK;
    if (!nodes || !ts || !len) {
        err = Error{TW_EINVAL, "sample_walks_batch: null output"};
        return err.code;
    }
    // backward walks run on the in-view, on the same stream
    tw_graph* vg = g;
    if (rev && backward_view(g, &vg, err) != TW_OK) return err.code;
    WalkArgs a;
    if (fill_args(vg, p->num_walks, p->max_len, p->start_bias, p->start_mode, p->d_start_nodes,
                  p->seed, p->walk_id_base, n2v, wtau, nodes, ts, len, a, err) != TW_OK)
        return err.code;
    a.hop = make_hop_bias(p->hop_biases[0]);
    QueueArgs q{};
    q.max_len = p->d_max_len;
    q.bias_idx = p->d_bias;
    q.row = p->d_row;
    q.n_bias = p->num_biases;
    for (int b = 0; b < p->num_biases; ++b) q.bias[b] = make_hop_bias(p->hop_biases[b]);
    if (p->d_row && p->out_slots < 1) {
        err = Error{TW_EINVAL, "sample_walks_batch: ragged rows need out_slots"};
        return err.code;
    }
    const int64_t slots = p->out_slots > 0 ? p->out_slots : p->num_walks * (int64_t)p->max_len;
    q.out_slots = slots;
    // biases by walk id: walk blocks, a wavefront's walks all of one bias; given
    // per walk: the work queue
    // (the queue also where ids wrap past 2^64, which changes the order of the
    // biases, and for more walks than a launch of blocks holds)
    if (p->dispatch != TW_DISPATCH_FULL_WALK && !p->d_bias && p->num_walks <= BLOCK_MAX_WALKS &&
        p->walk_id_base <= UINT64_MAX - (uint64_t)p->num_walks)
        return batch_blocks(vg, a, q, err, rev);
    launch_fill(vg, nodes, ts, slots);
    if (p->dispatch == TW_DISPATCH_FULL_WALK) return batch_full_walk(vg, a, q, err, rev);
    return queue_walks(vg, a, q, g->auto_bpc, err, rev);
}

// Allocation-free walks, for callers that cannot allocate device memory: one
// launch of the full-walk kernel, which keeps a walk's state in registers and
// LDS. (The queue dispatch, with its lists in a device array, took five more
// launches around it: 1,000 linear walks 85 -> 50 us.)
tw_status sample_walks_noalloc(tw_graph* g, const tw_walk_params* p, int32_t* nodes, int64_t* ts,
                               int32_t* len, Error& err) {
    if (!p) {
        err = Error{TW_EINVAL, "sample_walks_noalloc: null params"};
        return err.code;
    }
    if (p->num_walks > (int64_t)TW_NOALLOC_MAX_WALKS) {
        err = Error{TW_EINVAL, "sample_walks_noalloc: num_walks exceeds TW_NOALLOC_MAX_WALKS (" +
                                   std::to_string(TW_NOALLOC_MAX_WALKS) + ")"};
        return err.code;
    }
    if (p->direction != TW_FORWARD) {
        err = Error{TW_EINVAL, "sample_walks_noalloc: forward walks only"};
        return err.code;
    }
    if (p->hop_bias.kind == TW_WEIGHT) {
        err = Error{TW_EINVAL, "sample_walks_noalloc: TW_WEIGHT needs its weights built (allocates)"};
        return err.code;
    }
    // nothing may be built lazily: an index must exist, and node2vec needs
    // the adjacency of the current window
    if (!g->rec.p) {
        err = Error{TW_EINVAL, "sample_walks_noalloc: the graph holds no index yet (ingest first)"};
        return err.code;
    }
    if (p->hop_bias.kind == TW_NODE2VEC && g->m > 0 && !g->adj_ready) {
        err = Error{TW_EINVAL,
                    "sample_walks_noalloc: the node2vec adjacency of the current window is not "
                    "built (one tw_sample_walks call with a node2vec bias builds it)"};
        return err.code;
    }
    WalkArgs a;
    if (prepare_plain(g, p, nodes, ts, len, a, err) != TW_OK) return err.code;
    if (p->num_walks == 0) return TW_OK;
    return full_walks(g, a, false, err);
}

tw_status check_walk_params(const tw_walk_params* p, Error& err) {
    if (!p || p->num_walks < 0 || p->max_len < 1) {
        err = Error{TW_EINVAL, "walk request: need num_walks >= 0 and max_len >= 1"};
        return err.code;
    }
    if (check_bias(p->hop_bias, true, err) != TW_OK) return err.code;
    if (check_bias(p->start_bias, false, err) != TW_OK) return err.code;
    return check_start(p->start_mode, p->d_start_nodes, p->num_walks, err);
}

size_t serve_table_bytes(int n) { return sizeof(ServeReqDev) * (size_t)std::max(n, 1); }

// hops of n walks from their lengths, added to *out
__global__ void k_sum_hops(const int32_t* __restrict__ len, int64_t n,
                           unsigned long long* out) {
    uint64_t h = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        h += len[i] > 1 ? (uint64_t)(len[i] - 1) : 0;
    for (int off = 32; off > 0; off >>= 1) h += __shfl_down(h, off, 64);
    if ((threadIdx.x & 63) == 0 && h) atomicAdd(out, (unsigned long long)h);
}

// error words of a one-request launch run by the full-walk kernel: it
// counts trial-cap hits in word 2, the request's layout has them in word 1
__global__ void k_err_words(uint32_t* e, int finish) {
    if (threadIdx.x == 0) {
        if (finish) {
            e[1] = e[2];
            e[2] = 0u;
        } else {
            e[2] = 0u;
        }
    }
}

// Requests of at least this many walks launched alone run the full-walk
// kernel on their own rows (the fastest dispatch for one rectangular batch).
constexpr int64_t SERVE_FULL_MIN = 1 << 16;

tw_status serve_launch(tw_graph* g, const ServeReq* reqs, int n, void* d_table, void* h_table,
                       unsigned long long* d_hops, uint32_t* d_err, bool rev, Error& err) {
    if (n < 1 || n > SERVE_MAX_REQ) {
        err = Error{TW_EINVAL, "serve: 1..1024 requests per launch"};
        return err.code;
    }
    if (!rev && n == 1 && reqs[0].count >= SERVE_FULL_MIN && reqs[0].count <= BLOCK_MAX_WALKS &&
        reqs[0].hop.kind != TW_WEIGHT) {
        const ServeReq& q = reqs[0];
        WalkArgs a;
        if (fill_args(g, q.count, q.max_len, q.start, q.start_mode, q.start_nodes, q.seed, q.base,
                      q.hop.kind == TW_NODE2VEC, NAN, q.nodes, q.ts, q.len, a, err) != TW_OK)
            return err.code;
        a.hop = make_hop_bias(q.hop);
        a.err = d_err;  // [0] start node out of range, [2] trial-cap hits
        hipLaunchKernelGGL(k_err_words, dim3(1), dim3(64), 0, g->stream, d_err, 0);
        if (full_walks(g, a, false, err) != TW_OK) return err.code;
        hipLaunchKernelGGL(k_err_words, dim3(1), dim3(64), 0, g->stream, d_err, 1);
        hipLaunchKernelGGL(k_sum_hops, dim3(1024), dim3(256), 0, g->stream, q.len, q.count, d_hops);
        TW_HIP(hipGetLastError());
        return TW_OK;
    }
    bool n2v = false;
    double wtau = NAN;  // the weight-based requests' time scale: one per launch
    int64_t total = 0, blocks = 0;
    ServeReqDev* tab = static_cast<ServeReqDev*>(h_table);
    for (int r = 0; r < n; ++r) {
        const ServeReq& q = reqs[r];
        if (q.hop.kind == TW_WEIGHT) {
            const double sc = q.hop.tau > 0.0 ? q.hop.tau : 1.0;
            if (rev || (!std::isnan(wtau) && wtau != sc)) {
                err = Error{TW_EINVAL, "serve: weight-based requests of one launch need one "
                                       "tau and walk forward"};
                return err.code;
            }
            wtau = sc;
        }
        n2v |= q.hop.kind == TW_NODE2VEC;
        ServeReqDev d{};
        d.block0 = blocks;
        blocks += ceil_div(q.count, 64);
        d.count = q.count;
        d.seed = q.seed;
        d.base = q.base;
        d.L = q.max_len;
        d.start_kind = q.start.kind;
        d.start_mode = q.start_mode;
        d.start_tau = q.start.tau;
        d.hop = make_hop_bias(q.hop);
        d.start_nodes = q.start_nodes;
        d.nodes = q.nodes;
        d.ts = q.ts;
        d.len = q.len;
        d.err = d_err + 2 * r;
        tab[r] = d;
        total += q.count;
    }
    int64_t fill_slots = 0;  // of the largest request to fill first
    for (int r = 0; r < n; ++r) {
        if (blocks_pad(blocks, tab[r].L)) continue;
        tab[r].pre_filled = 1;
        fill_slots = std::max(fill_slots, tab[r].count * (int64_t)tab[r].L);
    }
    WalkArgs a;
    tw_bias none{TW_UNIFORM, 0.0, 1.0, 1.0};
    if (fill_args(g, total, 1, none, TW_START_EDGE, nullptr, 0, 0, n2v, wtau, nullptr, nullptr,
                  nullptr, a, err) != TW_OK)
        return err.code;
    TW_HIP(hipMemcpyAsync(d_table, h_table, sizeof(ServeReqDev) * n, hipMemcpyHostToDevice,
                          g->stream));
    const ServeReqDev* tab_d = static_cast<const ServeReqDev*>(d_table);
    if (fill_slots > 0) {
        const int64_t most = std::min<int64_t>(std::max(16384 / n, 64), FILL_BLOCKS);
        hipLaunchKernelGGL(k_fill_requests, dim3(fill_grid(fill_slots, most), (unsigned)n),
                           dim3(WALK_THREADS), 0, g->stream, tab_d);
    }
    for (int64_t b0 = 0; b0 < blocks; b0 += BLOCK_MAX_WALKS / 64) {
        const dim3 grid((unsigned)std::min<int64_t>(blocks - b0, BLOCK_MAX_WALKS / 64));
        if (rev)
            hipLaunchKernelGGL(k_walk_serve<true>, grid, dim3(64), 0, g->stream, a, tab_d, n, b0,
                               d_hops);
        else
            hipLaunchKernelGGL(k_walk_serve<false>, grid, dim3(64), 0, g->stream, a, tab_d, n, b0,
                               d_hops);
    }
    TW_HIP(hipGetLastError());
    return TW_OK;
}

tw_status row_offsets(tw_graph* g, const int32_t* max_len, int64_t n, int64_t* row,
                      int64_t* total, Error& err) {
    if (!row || n < 0 || (n > 0 && !max_len)) {
        err = Error{TW_EINVAL, "row_offsets: null argument or negative count"};
        return err.code;
    }
    uint64_t* out = reinterpret_cast<uint64_t*>(row);
    TW_HIP(scan_exclusive_i32_to_u64(max_len, out, n, out + n, g->ws, g->stream));
    int64_t t = 0;
    TW_HIP(hipMemcpyAsync(&t, row + n, sizeof(t), hipMemcpyDeviceToHost, g->stream));
    TW_HIP(hipStreamSynchronize(g->stream));
    if (total) *total = t;
    return TW_OK;
}

tw_status autotune(tw_graph* g, const tw_walk_params* p, int64_t sample, int32_t* nodes,
                   int64_t* ts, int32_t* len, int32_t best[2], Error& err) {
    if (!p || sample < 1 || p->direction != TW_FORWARD) {
        err = Error{TW_EINVAL, "autotune: need forward parameters and sample_walks >= 1"};
        return err.code;
    }
    tw_walk_params q = *p;
    q.num_walks = std::min<int64_t>(p->num_walks, sample);
    WalkArgs a;
    if (prepare_plain(g, &q, nodes, ts, len, a, err) != TW_OK) return err.code;
    if (q.num_walks == 0) return TW_OK;
    if (queue_shape(g, err) != TW_OK) return err.code;
    // full-walk; the queue at three launch shapes (as many workgroups as
    // fit, 4 or 2 per CU); the cooperative dispatch over its regroup, the
    // lanes that engage the wavefront tier, the LDS panel and the read-back
    // cadence of the live count
    std::vector<tw_tuning> cands;
    const tw_tuning base{TW_DISPATCH_FULL_WALK, 0, 0, 64, 4096, 1};
    cands.push_back(base);
    for (int bpc : {0, 4, 2}) {
        tw_tuning c = base;
        c.dispatch = TW_DISPATCH_QUEUE;
        c.queue_bpc = bpc;
        cands.push_back(c);
    }
    for (int regroup : {0, 1})
        for (int wave_min : {64, 16})
            for (int panel : {2048, 8192})
                for (int sync : {1, 4}) {
                    if (regroup == 1 && (wave_min != 64 || panel != 2048)) continue;
                    cands.push_back(tw_tuning{TW_DISPATCH_COOP, 0, regroup, wave_min, panel, sync});
                }
    const tw_tuning saved = get_tuning(g);
    hipEvent_t e0, e1;
    TW_HIP(hipEventCreate(&e0));
    TW_HIP(hipEventCreate(&e1));
    float best_ms = 0.0f;
    tw_tuning pick = base;
    bool first = true;
    for (const tw_tuning& c : cands) {
        set_tuning_fields(g, c);
        float ms_min = 0.0f;
        for (int rep = 0; rep < 3; ++rep) {  // the first run warms up
            hipEventRecord(e0, g->stream);
            if (run_dispatch(g, a, c.dispatch, c.queue_bpc, err) != TW_OK) {
                hipEventDestroy(e0);
                hipEventDestroy(e1);
                set_tuning_fields(g, saved);
                return err.code;
            }
            hipEventRecord(e1, g->stream);
            TW_HIP(hipEventSynchronize(e1));
            float ms = 0.0f;
            TW_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (rep == 1 || (rep > 1 && ms < ms_min)) ms_min = ms;
        }
        if (first || ms_min < best_ms) {
            best_ms = ms_min;
            pick = c;
            first = false;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    set_tuning_fields(g, pick);
    if (best) {
        best[0] = pick.dispatch;
        best[1] = pick.queue_bpc;
    }
    return TW_OK;
}

tw_tuning get_tuning(const tw_graph* g) {
    return tw_tuning{g->auto_dispatch ? g->auto_dispatch : TW_DISPATCH_FULL_WALK, g->auto_bpc,
                     g->coop_regroup, g->coop_wave_min, (int32_t)g->coop_panel, g->coop_sync};
}

void set_tuning_fields(tw_graph* g, const tw_tuning& t) {
    g->auto_dispatch = t.dispatch;
    g->auto_bpc = t.queue_bpc;
    g->coop_regroup = t.coop_regroup;
    g->coop_wave_min = t.coop_wave_min;
    g->coop_panel = (uint32_t)t.coop_panel;
    g->coop_sync = t.coop_sync;
}

tw_status set_tuning(tw_graph* g, const tw_tuning* t, Error& err) {
    if (!t || t->dispatch < TW_DISPATCH_FULL_WALK || t->dispatch > TW_DISPATCH_QUEUE ||
        t->queue_bpc < 0 || t->coop_regroup < 0 || t->coop_regroup > 1 || t->coop_wave_min < 1 ||
        t->coop_wave_min > 64 || t->coop_panel < 64 || t->coop_panel > 8192 ||
        t->coop_panel % 64 != 0 || t->coop_sync < 1 || t->coop_sync > 64) {
        err = Error{TW_EINVAL, "set_tuning: dispatch FULL_WALK..QUEUE, queue_bpc >= 0, regroup 0 or "
                               "1, wave_min 1..64, panel 64..8192 in steps of 64, sync 1..64"};
        return err.code;
    }
    set_tuning_fields(g, *t);
    return TW_OK;
}

}  // namespace tw
