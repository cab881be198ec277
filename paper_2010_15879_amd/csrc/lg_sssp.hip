// lg_sssp: single-source shortest paths over a weighted graph (SSSP of
// section "Considered Algorithms", a delta-stepping traversal), reading the
// weight stored right after each ID (subsection "Accessing an Edge Weight").
//
// Distances are uint64 (UINT64_MAX: not reached).  A bitmap marks vertices
// whose distance dropped since their edges were last relaxed.  Each step of
// bucket k (distances below hi = (k+1) delta):
//   collect  marked vertices with a distance below hi leave the bitmap and
//            join the frontier queue with their list start, ID width,
//            degree and distance (a count pass per 64-vertex word, a scan,
//            a write pass); the smallest distance among the marked vertices
//            left behind is kept for choosing the next bucket
//   relax    the frontier's edges, flattened by an exclusive scan of the
//            degrees, 64 consecutive edges per wave step: nd = dist(u) + w;
//            an atomic minimum on dist(v), and v is marked when it lowered it
// An empty frontier moves to the bucket of the smallest marked distance;
// none marked ends the search.  The device takes these decisions itself
// (SsspState), so that the host queues several steps before it looks.  Every vertex relaxed from a distance d
// reaches the final distances of the paths through it, so the result is the
// exact distances whatever delta and the order of the atomics.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "lg_device.hpp"

namespace lg {

// ---------------------------------------------------------------------------
// Weighted entries (subsections "Logarithmization of Edge Weights" and
// "Accessing an Edge Weight"): packed, each entry is the ID at its width w
// followed by the weight at omega bits; plain, the CSR plus a weight array.
// ---------------------------------------------------------------------------

// start: first bit (packed) or first index (plain); w: ID width
struct WInfo {
    uint64_t start;
    uint32_t deg;
    uint32_t w;
};

template <int IDM, int OFM>
struct WPackedAcc {
    PackedAcc<IDM, OFM> base;
    uint32_t omega;

    __device__ __forceinline__ WInfo info(uint32_t v) const {
        uint64_t o0, o1;
        base.offsets(v, o0, o1);
        WInfo r;
        if constexpr (IDM == kIdsGlobal) {
            r.w = base.pv.s;
            r.start = o0 * (uint64_t)(r.w + omega);
            r.deg = (uint32_t)(o1 - o0);
        } else {
            r.w = base.width(v);
            r.start = o0;
            r.deg = o1 > o0 ? (uint32_t)((o1 - o0) / (uint64_t)(r.w + omega)) : 0u;
        }
        return r;
    }
    __device__ __forceinline__ void entry(uint64_t start, uint32_t w, uint64_t i, uint32_t &id, uint32_t &wt) const {
        const uint64_t b = start + i * (uint64_t)(w + omega);
        id = base.get(b, width_mask(w));
        wt = base.get(b + w, width_mask(omega));
    }
};

template <bool OFF64>
struct WPlainAcc {
    PlainAcc<OFF64> base;
    const uint32_t *wt;

    __device__ __forceinline__ WInfo info(uint32_t v) const {
        const VInfo vi = base.info(v);
        return WInfo{vi.start, vi.deg, 32u};
    }
    __device__ __forceinline__ void entry(uint64_t start, uint32_t, uint64_t i, uint32_t &id, uint32_t &w) const {
        id = base.pv.col[start + i];
        w = wt[start + i];
    }
};

template <class Fn>
lg_status dispatch_wacc(const lg_graph *g, Fn &&fn) {
    if (!g->weighted) {
        set_error("the graph has no edge weights (build it with lg_encode_weighted)");
        return LG_ERR_UNSUPPORTED;
    }
    if (g->layout == LG_LAYOUT_PLAIN) {
        const uint32_t *wt = g->pwt.as<uint32_t>();
        if (g->poff64) return fn(WPlainAcc<true>{PlainAcc<true>{g->plain_view()}, wt});
        return fn(WPlainAcc<false>{PlainAcc<false>{g->plain_view()}, wt});
    }
    const PackedView pv = g->packed_view();
    const uint32_t om = g->omega;
    if (g->id_mode == LG_IDS_GLOBAL) {
        if (g->offset_mode == LG_OFFS_PACKED) return fn(WPackedAcc<kIdsGlobal, kOffsPacked>{{pv}, om});
        return fn(WPackedAcc<kIdsGlobal, kOffsEF>{{pv}, om});
    }
    if (g->offset_mode == LG_OFFS_PACKED) return fn(WPackedAcc<kIdsLocal, kOffsPacked>{{pv}, om});
    return fn(WPackedAcc<kIdsLocal, kOffsEF>{{pv}, om});
}

constexpr uint64_t kInfDist = ~0ull;

// Where the search stands (device memory, read back by the host).
struct SsspState {
    unsigned long long hi;     // distances below it are collected
    unsigned long long count;  // frontier vertices of this step
    unsigned long long steps;
    unsigned long long done;   // 1: no vertex is marked any more, 2: the step bound was hit
};
// What a collecting workgroup found in its words.
struct SsspPart {
    unsigned long long edges;  // entries of the vertices taken
    unsigned long long left;   // the smallest distance staying marked
    unsigned long long count;  // vertices taken
};

struct SsspWork {
    DevBuf upd;                         // bitmap, one bit per vertex
    DevBuf qv;                          // frontier: vertex
    DevBuf qstart, qdist, qoff;         // list start (as in vstart), distance, entries of the vertices before
    DevBuf state;                       // SsspState
    DevBuf tmask, wdeg;                 // per bitmap word: vertices taken, their degrees' sum
    DevBuf parts;                       // SsspPart of every collecting workgroup
    DevBuf vstart, vdeg;                // per vertex, of the first call on: list start | ID width << 56, degree
    bool lists = false;
    DevBuf dl;                          // label-space distances (relabeled graphs)
    uint64_t *host = nullptr;           // pinned readback slots
    SsspWork() = default;
    SsspWork(const SsspWork &) = delete;
    SsspWork &operator=(const SsspWork &) = delete;
    ~SsspWork() {
        if (host) (void)hipHostFree(host);
    }
    uint64_t bytes() const {
        return upd.bytes + qv.bytes + qstart.bytes + qdist.bytes + qoff.bytes +
               state.bytes + tmask.bytes + wdeg.bytes + parts.bytes + vstart.bytes + vdeg.bytes + dl.bytes;
    }
};

uint64_t sssp_bytes(const lg_graph *g) { return g->sssp ? g->sssp->bytes() : 0; }

lg_status sssp_free(lg_graph *g) {
    delete g->sssp;
    g->sssp = nullptr;
    return LG_OK;
}

// The root arrives as its original ID and is mapped to its label (inv,
// when relabeled) here.
__global__ void sssp_init_kernel(uint32_t n, uint64_t words, uint32_t root_id, const uint32_t *__restrict__ inv,
                                 uint64_t first_hi, uint64_t *__restrict__ dist, uint64_t *__restrict__ upd,
                                 SsspState *__restrict__ state) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t total = n > words ? n : words;
    const uint32_t root = inv ? inv[root_id] : root_id;
    if (blockIdx.x == 0 && threadIdx.x == 0) *state = SsspState{first_hi, 0, 0, 0};
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        if (i < n) dist[i] = i == root ? 0ull : kInfDist;
        if (i < words) upd[i] = i == (root >> 6) ? 1ull << (root & 63) : 0ull;
    }
}

// Every vertex's list, decoded once per graph: a search collects a vertex
// about one and a half times, each time for its degree and again for its
// start (Elias-Fano selects in every step: 4.3 of 11 ms on a relabeled
// Kronecker graph of 2^23 vertices).
template <class Acc>
__global__ void sssp_lists_kernel(Acc acc, uint32_t n, uint64_t *__restrict__ vstart, uint32_t *__restrict__ vdeg) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const WInfo vi = acc.info((uint32_t)v);
        vstart[v] = vi.start | (uint64_t)vi.w << 56;  // streams stay far below 2^56 bits
        vdeg[v] = vi.deg;
    }
}

// The frontier is compacted without a shared counter (single-address atomics
// from thousands of workgroups took 20 us a step).  Every workgroup has its
// fixed tiles of bitmap words, dealt in turn (a relabeled graph's marks crowd
// in the first words).  The count pass takes each word's marked vertices
// below the bound out of the bitmap and leaves the workgroup's vertices,
// entries and smallest distance left marked; the write pass sums the
// workgroups before its own (at most kCollectParts) and places its vertices
// with the running entry count the relax pass walks by.  Two launches for
// what were seven (a reset, the count, two scans of up to three launches),
// and no read-back between them: Kronecker 2^20 vertices, 20 steps, 2.65 ->
// 1.62 ms.  Every marked vertex has edges (it was reached over one) but the
// root, which may have none: it is then alone in the first frontier, which
// holds no edges.
constexpr int kCollectThreads = 256;
constexpr uint32_t kCollectWaves = kCollectThreads / kWave;
constexpr uint64_t kCollectParts = 2048;
constexpr uint64_t kCollectTile = 64;  // words of a tile, at most

__global__ __launch_bounds__(kCollectThreads) void sssp_count_kernel(
    uint32_t n, uint64_t words, uint32_t tile, const SsspState *__restrict__ state,
    const uint32_t *__restrict__ vdeg, const uint64_t *__restrict__ dist, uint64_t *__restrict__ upd,
    uint64_t *__restrict__ tmask, uint64_t *__restrict__ wdeg, SsspPart *__restrict__ parts) {
    if (state->done) return;
    __shared__ unsigned long long s_left[kCollectWaves], s_edges[kCollectWaves], s_count[kCollectWaves];
    const uint64_t hi = state->hi;
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    uint64_t left = kInfDist;  // the smallest distance staying marked
    unsigned long long edges = 0, count = 0;
    // a wave holds every fourth word of a tile (so that its marked words
    // spread over the waves), then takes the marked ones two at a time, their
    // vertices' distances and list lengths in flight together
    constexpr int kWords = 2;
    for (uint64_t b = (uint64_t)blockIdx.x * tile; b < words; b += (uint64_t)gridDim.x * tile) {
        const uint64_t q = b + lane * kCollectWaves + wv;
        const bool in = lane * kCollectWaves + wv < tile && q < words;
        const uint64_t mine = in ? upd[q] : 0ull;
        uint64_t my_take = 0, my_deg = 0;
        for (uint64_t todo = __ballot(mine != 0ull); todo;) {
            uint32_t t[kWords];
            uint64_t d[kWords];
            uint32_t deg[kWords];
            bool set[kWords], take[kWords];
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                const bool any = todo != 0;
                t[k] = any ? (uint32_t)__ffsll((long long)todo) - 1 : 0u;
                todo &= todo - 1;
                const uint64_t bits = __shfl(mine, t[k], kWave);
                const uint64_t v = (b + t[k] * kCollectWaves + wv) * 64 + lane;
                set[k] = any && ((bits >> lane) & 1ull) && v < n;
                d[k] = set[k] ? dist[v] : kInfDist;
                deg[k] = set[k] ? vdeg[v] : 0u;
            }
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                take[k] = set[k] && d[k] < hi;
                if (set[k] && !take[k] && d[k] < left) left = d[k];
            }
#pragma unroll
            for (int k = 0; k < kWords; ++k) {
                const uint64_t take_m = __ballot(take[k]);
                const uint64_t sum = wave_sum((unsigned long long)(take[k] ? deg[k] : 0u));
                if (take_m && lane == t[k]) {
                    my_take = take_m;
                    my_deg = sum;
                }
            }
        }
        if (in) {
            tmask[q] = my_take;
            if (my_take) {
                wdeg[q] = my_deg;
                upd[q] = mine & ~my_take;
            }
        }
        edges += my_deg;
        count += (unsigned long long)__popcll(my_take);
    }
#pragma unroll
    for (int s = kWave / 2; s > 0; s >>= 1) {
        const uint64_t o = __shfl_xor(left, s, kWave);
        left = o < left ? o : left;
    }
    edges = wave_sum(edges);
    count = wave_sum(count);
    if (lane == 0) {
        s_left[wv] = left;
        s_edges[wv] = edges;
        s_count[wv] = count;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        SsspPart p{0, kInfDist, 0};
        for (uint32_t w = 0; w < kCollectWaves; ++w) {
            p.edges += s_edges[w];
            p.count += s_count[w];
            p.left = s_left[w] < p.left ? s_left[w] : p.left;
        }
        parts[blockIdx.x] = p;
    }
}

// exclusive prefix over a workgroup's threads, and the total
__device__ __forceinline__ uint64_t collect_scan(uint64_t x, uint64_t *s_wave, uint64_t &total) {
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint64_t incl = wave_incl_scan(x);
    __syncthreads();  // the last use of s_wave is over
    if (lane == kWave - 1) s_wave[wv] = incl;
    __syncthreads();
    uint64_t base = 0;
    total = 0;
    for (uint32_t w = 0; w < kCollectWaves; ++w) {
        if (w < wv) base += s_wave[w];
        total += s_wave[w];
    }
    return base + incl - x;
}

__global__ __launch_bounds__(kCollectThreads) void sssp_write_kernel(
    const uint64_t *__restrict__ vstart, const uint32_t *__restrict__ vdeg, uint64_t words, uint32_t tile,
    uint64_t delta, uint64_t max_steps, const uint64_t *__restrict__ dist, const uint64_t *__restrict__ tmask,
    const uint64_t *__restrict__ wdeg, const SsspPart *__restrict__ parts,
    uint32_t *__restrict__ qv, uint64_t *__restrict__ qstart, uint64_t *__restrict__ qdist,
    uint64_t *__restrict__ qoff, SsspState *__restrict__ state) {
    __shared__ uint64_t s_wave[kCollectWaves];
    __shared__ uint64_t s_pos[kCollectTile], s_off[kCollectTile], s_take[kCollectTile];
    __shared__ unsigned long long s_left;
    __shared__ bool s_done;
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    // the workgroups before this one
    uint64_t cnt = 0, edges = 0, all_cnt = 0, all_edges = 0, left = kInfDist;
    for (uint32_t i = threadIdx.x; i < gridDim.x; i += kCollectThreads) {
        const SsspPart p = parts[i];
        if (i < blockIdx.x) {
            cnt += p.count;
            edges += p.edges;
        }
        all_cnt += p.count;
        all_edges += p.edges;
        left = p.left < left ? p.left : left;
    }
    // Block 0 sets `done` below while others start: one thread looks, so that a
    // workgroup goes on or ends as a whole.  (One that sees it set in this
    // launch had nothing to write, or the step bound was hit and nothing is
    // relaxed.)
    if (threadIdx.x == 0) {
        s_left = kInfDist;
        s_done = state->done != 0;
    }
    uint64_t pos0, off0, total_cnt, total_edges;
    (void)collect_scan(cnt, s_wave, pos0);
    if (s_done) return;
    (void)collect_scan(edges, s_wave, off0);
    if (blockIdx.x == 0) {
        (void)collect_scan(all_cnt, s_wave, total_cnt);
        (void)collect_scan(all_edges, s_wave, total_edges);
        if (left != kInfDist) atomicMin(&s_left, (unsigned long long)left);
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long steps = state->steps + 1;
            state->steps = steps;
            qoff[total_cnt] = total_edges;
            if (steps > max_steps) {  // the queue may be left unwritten: nothing is relaxed
                state->count = 0;
                state->done = 2;
            } else {
                state->count = total_cnt;
                if (!total_cnt) {  // the next bucket with a marked vertex
                    const uint64_t k = s_left / delta;
                    if (s_left == kInfDist) state->done = 1;
                    else state->hi = k + 1 > kInfDist / delta ? kInfDist : (k + 1) * delta;
                }
            }
        }
    }
    for (uint64_t b = (uint64_t)blockIdx.x * tile; b < words; b += (uint64_t)gridDim.x * tile) {
        const uint64_t q = b + threadIdx.x;
        const uint64_t take = threadIdx.x < tile && q < words ? tmask[q] : 0ull;
        const uint64_t deg = take ? wdeg[q] : 0ull;
        uint64_t tile_cnt, tile_edges;
        const uint64_t at = collect_scan((uint64_t)__popcll(take), s_wave, tile_cnt);
        const uint64_t off = collect_scan(deg, s_wave, tile_edges);
        if (threadIdx.x < tile) {
            s_take[threadIdx.x] = take;
            s_pos[threadIdx.x] = pos0 + at;
            s_off[threadIdx.x] = off0 + off;
        }
        __syncthreads();
        for (uint32_t t = wv; t < tile; t += kCollectWaves) {
            const uint64_t m = s_take[t];
            if (!m) continue;  // same for every lane
            const bool in = (m >> lane) & 1ull;
            const uint64_t v = (b + t) * 64 + lane;
            const uint32_t deg = in ? vdeg[v] : 0u;
            const uint64_t start = in ? vstart[v] : 0ull;
            const uint64_t incl = wave_incl_scan((uint64_t)deg);
            if (in) {
                const uint64_t pos = s_pos[t] + popc_below(m);
                qv[pos] = (uint32_t)v;
                qstart[pos] = start;
                qdist[pos] = dist[v];
                qoff[pos] = s_off[t] + incl - deg;
            }
        }
        pos0 += tile_cnt;
        off0 += tile_edges;
        __syncthreads();  // the next tile rewrites the words' places
    }
}

// Edge t of the frontier belongs to slot s with qoff[s] <= t < qoff[s + 1];
// every slot holds at least one edge.  Each wave takes a contiguous range
// of edges, 64 per step, and finds its first slot by one search.  In
// a step starting at edge t0 in slot s0, lane j loads the boundary
// qoff[s0 + 1 + j]; the boundaries inside (t0, t0 + 64) form a bit mask
// (a wave sum of distinct bits), so the slot of edge t0 + i is s0 plus the
// number of mask bits at or below i, and the next step's slot is s0 plus
// the number of boundaries at or below t0 + 64.  No lane runs a search per
// edge.
template <class Acc>
__global__ void sssp_relax_kernel(Acc acc, uint32_t n, const SsspState *__restrict__ state,
                                  const uint64_t *__restrict__ qoff, const uint32_t *__restrict__ qv,
                                  const uint64_t *__restrict__ qstart, const uint64_t *__restrict__ qdist,
                                  unsigned long long *__restrict__ dist, unsigned long long *__restrict__ upd) {
    const uint32_t lane = lane_id();
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
    const uint64_t count = state->count;
    if (!count) return;
    const uint64_t E = qoff[count];
    const uint64_t per = ((E + nwaves - 1) / nwaves + kWave - 1) / kWave * kWave;
    const uint64_t tb = wave * per;
    if (tb >= E) return;  // same for every lane
    const uint64_t te = tb + per < E ? tb + per : E;
    uint64_t s0 = 0, hi = count;  // qoff[s0] <= tb < qoff[hi], 64 probes a step
    while (hi - s0 > 1) {
        const uint64_t step = (hi - s0 + kWave - 1) / kWave;
        const uint64_t at = s0 + lane * step;
        const uint64_t le = __ballot(at < hi && qoff[at < hi ? at : s0] <= tb);
        s0 += (uint64_t)(__popcll(le) - 1) * step;
        hi = hi - s0 > step ? s0 + step : hi;
    }
    const uint64_t below = lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1ull);  // bits 0..lane
    for (uint64_t t0 = tb; t0 < te; t0 += kWave) {
        const uint64_t j = s0 + 1 + lane;
        const uint64_t b = j <= count ? qoff[j] : ~0ull;  // > t0
        const uint64_t o = b - t0;
        const uint64_t M = wave_sum(o < kWave ? 1ull << o : 0ull);
        const uint64_t adv = (uint64_t)__popcll(__ballot(o <= kWave));
        const uint64_t t = t0 + lane;
        // a frontier vertex whose distance dropped again since it was
        // collected is marked again and relaxes next step from the lower
        // distance: its edges are skipped now
        const uint64_t a = s0 + (uint64_t)__popcll(M & below);
        if (t < te && dist[qv[a]] >= qdist[a]) {
            uint32_t id, w;
            const uint64_t st = qstart[a];
            acc.entry(st & ((1ull << 56) - 1ull), (uint32_t)(st >> 56), t - qoff[a], id, w);
            if (id < n) {  // only a corrupt stream fails this
                const unsigned long long nd = qdist[a] + (unsigned long long)w;
                if (nd < dist[id]) {
                    const unsigned long long old = atomicMin(&dist[id], nd);
                    if (nd < old) atomicOr(&upd[id >> 6], 1ull << (id & 63));
                }
            }
        }
        s0 += adv;
    }
}

// distances in original IDs: dist[o] = dist of label inv[o]
__global__ void sssp_unpermute_kernel(uint32_t n, const uint32_t *__restrict__ inv, const uint64_t *__restrict__ dl,
                                      uint64_t *__restrict__ dist) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t o = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; o < n; o += stride) dist[o] = dl[inv[o]];
}

}  // namespace lg

static lg_status lg_sssp_impl(const lg_graph *gc, uint32_t root, uint32_t delta, uint64_t *dist, hipStream_t stream) {
    using namespace lg;
    lg_graph *g = const_cast<lg_graph *>(gc);
    if (!g || !dist) { set_error("lg_sssp: NULL argument"); return LG_ERR_INVALID; }
    if (root >= g->n) { set_error("lg_sssp: root %u >= n", root); return LG_ERR_INVALID; }
    if (!g->weighted) {
        set_error("lg_sssp: the graph has no edge weights (build it with lg_encode_weighted)");
        return LG_ERR_UNSUPPORTED;
    }
    // default bucket width: the weight range 2^omega (one edge of the
    // heaviest weight spans about one bucket; 256 for 8-bit weights, the
    // best of a sweep on weights in [1, 255])
    const uint64_t D = delta ? delta : (1ull << g->omega);
    const uint32_t n = g->n;
    const uint64_t words = ((uint64_t)n + 63) / 64;
    // one workspace per graph: calls on the same graph run one at a time, and
    // each waits for its own last kernel before letting the next one in
    std::lock_guard<std::mutex> hold(g->sssp_mu);
    if (!g->sssp) {
        g->sssp = new (std::nothrow) SsspWork();
        if (!g->sssp) { set_error("lg_sssp: host allocation failed"); return LG_ERR_OOM; }
    }
    SsspWork &W = *g->sssp;
    if (!W.host) {
        if (hipHostMalloc((void **)&W.host, 4 * sizeof(uint64_t)) != hipSuccess) {
            W.host = nullptr;
            set_error("lg_sssp: pinned host allocation failed");
            return LG_ERR_OOM;
        }
    }
    LG_TRY(W.upd.ensure(words * 8));
    LG_TRY(W.tmask.ensure(words * 8));
    LG_TRY(W.wdeg.ensure(words * 8));
    LG_TRY(W.parts.ensure(kCollectParts * sizeof(SsspPart)));
    LG_TRY(W.qv.ensure((uint64_t)n * 4));
    LG_TRY(W.vstart.ensure((uint64_t)n * 8));
    LG_TRY(W.vdeg.ensure((uint64_t)n * 4));
    LG_TRY(W.qstart.ensure((uint64_t)n * 8));
    LG_TRY(W.qdist.ensure((uint64_t)n * 8));
    LG_TRY(W.qoff.ensure(((uint64_t)n + 1) * 8));
    LG_TRY(W.state.ensure(sizeof(SsspState)));
    // a relabeled graph runs in label space, then maps back
    const bool rel = g->relabel != LG_RELABEL_NONE;
    uint64_t *const dist_out = dist;
    if (rel) {
        LG_TRY(W.dl.ensure((uint64_t)n * 8));
        dist = W.dl.as<uint64_t>();
    }
    SsspState *state = W.state.as<SsspState>();
    LG_LAUNCH(sssp_init_kernel, grid_for(std::max<uint64_t>(n, words), 256, 1u << 16), 256, 0, stream, n, words, root,
              rel ? (const uint32_t *)g->inv.as<uint32_t>() : (const uint32_t *)nullptr, D, dist,
              W.upd.as<uint64_t>(), state);
    LG_CHECK_LAUNCH();
    return dispatch_wacc(g, [&](auto acc) -> lg_status {
        using Acc = decltype(acc);
        int cus = 0;
        LG_CHECK_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, g->device));
        // tiles of one word per wave on small graphs, up to kCollectTile words
        uint32_t tile = kCollectWaves;
        while (tile < kCollectTile && words > tile * kCollectParts) tile *= 2;
        const uint32_t collect_grid = (uint32_t)std::min<uint64_t>(kCollectParts, (words + tile - 1) / tile);
        const uint32_t relax_grid = (uint32_t)std::max(1, cus) * 8;
        if (!W.lists) {
            LG_LAUNCH(sssp_lists_kernel<Acc>, grid_for(n, 256, 1u << 16), 256, 0, stream, acc, n,
                      W.vstart.as<uint64_t>(), W.vdeg.as<uint32_t>());
            LG_CHECK_LAUNCH();
            W.lists = true;
        }
        // every step either relaxes a non-empty frontier (each entry of it
        // lowered a distance) or moves to a later bucket: bounded for
        // non-negative weights; the cap only guards against a corrupt graph
        const uint64_t cap = 64ull * n + 1024;
        // steps queued between two looks at the state: the ones past the end
        // find it done and return at once
        constexpr int kAhead = 4;
        SsspState now{};
        while (!now.done) {
            for (int i = 0; i < kAhead; ++i) {
                LG_LAUNCH(sssp_count_kernel, collect_grid, kCollectThreads, 0, stream, n, words, tile,
                          (const SsspState *)state, (const uint32_t *)W.vdeg.as<uint32_t>(), (const uint64_t *)dist,
                          W.upd.as<uint64_t>(), W.tmask.as<uint64_t>(), W.wdeg.as<uint64_t>(), W.parts.as<SsspPart>());
                LG_CHECK_LAUNCH();
                LG_LAUNCH(sssp_write_kernel, collect_grid, kCollectThreads, 0, stream,
                          (const uint64_t *)W.vstart.as<uint64_t>(), (const uint32_t *)W.vdeg.as<uint32_t>(), words,
                          tile, D, cap, (const uint64_t *)dist, (const uint64_t *)W.tmask.as<uint64_t>(),
                          (const uint64_t *)W.wdeg.as<uint64_t>(), (const SsspPart *)W.parts.as<SsspPart>(),
                          W.qv.as<uint32_t>(), W.qstart.as<uint64_t>(), W.qdist.as<uint64_t>(),
                          W.qoff.as<uint64_t>(), state);
                LG_CHECK_LAUNCH();
                LG_LAUNCH(sssp_relax_kernel<Acc>, relax_grid, 256, 0, stream, acc, n, (const SsspState *)state,
                          (const uint64_t *)W.qoff.as<uint64_t>(), (const uint32_t *)W.qv.as<uint32_t>(),
                          (const uint64_t *)W.qstart.as<uint64_t>(), (const uint64_t *)W.qdist.as<uint64_t>(),
                          (unsigned long long *)dist, W.upd.as<unsigned long long>());
                LG_CHECK_LAUNCH();
            }
            LG_CHECK_HIP(hipMemcpyAsync(W.host, state, sizeof(SsspState), hipMemcpyDeviceToHost, stream));
            LG_CHECK_HIP(hipStreamSynchronize(stream));
            std::memcpy(&now, W.host, sizeof(now));
        }
        if (now.done == 2) {
            set_error("lg_sssp: no convergence after %llu steps", now.steps);
            return LG_ERR_DEVICE;
        }
        if (rel) {
            LG_LAUNCH(sssp_unpermute_kernel, grid_for(n, 256, 1u << 16), 256, 0, stream, n, g->inv.as<uint32_t>(),
                      (const uint64_t *)dist, dist_out);
            LG_CHECK_LAUNCH();
            LG_CHECK_HIP(hipStreamSynchronize(stream));
        }
        return LG_OK;
    });
}

extern "C" lg_status lg_sssp(const lg_graph *gc, uint32_t root, uint32_t delta, uint64_t *dist, hipStream_t stream) {
    LG_TRY(lg_sssp_impl(gc, root, delta, dist, stream));
    return lg::mark_use(const_cast<lg_graph *>(gc), stream);
}
