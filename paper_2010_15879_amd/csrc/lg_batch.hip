// lg_bfs_batch_*: many BFS queries over many (small) graphs in one
// persistent launch.
//
// Every workgroup is a worker: it takes the next job (graph, root) from a
// device counter, runs that BFS to the end itself (level-synchronous, with
// workgroup barriers between levels), and takes the next job until none is
// left -- so the exit condition is reached by every workgroup.  A vertex of
// degree below `wave_threshold` is handled by one thread, a larger one by a
// whole wave (lanes over its list, coalesced); top-down levels stage `chunk`
// frontier vertices at a time.  The knobs are picked per plan by timing
// candidate settings on the actual batch.  The rule is that of the
// single-query path (the parent is the smallest label one level up), so
// every result equals the per-query result bit for bit.
//
// Two kernels: bfs_batch_kernel keeps a search's bitmaps in LDS and changes
// direction like the single-query path; bfs_batch_large_kernel, for plans
// with a graph whose bitmaps do not fit, goes top-down over depths in memory.
//
// A plan captures "reset the job counter + the persistent launch" in a HIP
// graph, replayed by lg_bfs_batch_run.
#include <algorithm>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <vector>

#include "lg_device.hpp"
#include "lg_varint.hpp"

struct lg_batch_plan;

namespace lg {

constexpr uint32_t kMaxChunk = 1024;

template <class Acc>
struct BatchGraph {
    Acc acc;
    uint32_t n;
    uint64_t m;        // entries (Varint: bytes)
    uint64_t longest;  // no list is longer (Varint: in bytes, five a value)
};

struct BatchJob {
    uint32_t graph;
    uint32_t root;
    uint64_t out_offset;
};

template <class Acc>
__device__ __forceinline__ void batch_visit(uint32_t u, uint32_t v, int32_t nd, int32_t *__restrict__ D,
                                            uint32_t *__restrict__ P, uint32_t *__restrict__ qnext,
                                            uint32_t *s_tail) {
    // a plain read first: most edges of later levels reach vertices settled
    // at earlier levels, which the CAS would only confirm
    const int32_t seen = __builtin_nontemporal_load(&D[u]);
    if (seen != -1 && seen != nd) return;
    const int32_t old = atomicCAS(&D[u], -1, nd);
    if (P && (old == -1 || old == nd)) atomicMin(&P[u], v);
    if (old == -1) qnext[atomicAdd(s_tail, 1u)] = u;
}

template <class Acc, int kThreads>
__global__ __launch_bounds__(kThreads) void bfs_batch_large_kernel(
    const BatchGraph<Acc> *__restrict__ graphs, const BatchJob *__restrict__ jobs, uint32_t num_jobs,
    uint32_t *__restrict__ job_counter, int32_t *__restrict__ depth, int32_t *__restrict__ parent,
    int32_t max_depth, uint32_t *__restrict__ queues, uint64_t qcap, uint32_t chunk, uint32_t wave_threshold) {
    __shared__ uint32_t s_job, s_fsize, s_tail, s_nheavy;
    __shared__ uint32_t s_heavy[kMaxChunk];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = lane_id();
    const uint32_t wv = tid / kWave;
    constexpr uint32_t kWaves = kThreads / kWave;
    uint32_t *qa = queues + (uint64_t)blockIdx.x * 2 * qcap;
    uint32_t *qb = qa + qcap;
    for (;;) {
        if (tid == 0) s_job = atomicAdd(job_counter, 1u);
        __syncthreads();
        const uint32_t job = s_job;
        if (job >= num_jobs) break;
        const BatchJob jb = jobs[job];
        const BatchGraph<Acc> G = graphs[jb.graph];
        const uint32_t n = G.n;
        int32_t *D = depth + jb.out_offset;
        uint32_t *P = parent ? reinterpret_cast<uint32_t *>(parent + jb.out_offset) : nullptr;
        for (uint32_t v = tid; v < n; v += kThreads) {
            D[v] = v == jb.root ? 0 : -1;
            if (P) P[v] = v == jb.root ? jb.root : 0xFFFFFFFFu;
        }
        if (tid == 0) {
            qa[0] = jb.root;
            s_fsize = 1;
        }
        __syncthreads();
        int32_t level = 0;
        uint32_t *qin = qa, *qout = qb;
        for (;;) {
            const uint32_t F = s_fsize;
            if (F == 0 || (max_depth >= 0 && level >= max_depth)) break;
            __syncthreads();  // everyone has read s_fsize
            if (tid == 0) s_tail = 0;
            const int32_t nd = level + 1;
            for (uint32_t c0 = 0; c0 < F; c0 += chunk) {
                const uint32_t c1 = c0 + chunk < F ? c0 + chunk : F;
                if (tid == 0) s_nheavy = 0;
                __syncthreads();
                for (uint32_t i = c0 + tid; i < c1; i += kThreads) {
                    const uint32_t v = qin[i];
                    if constexpr (IsGapAcc<Acc>::value) {
                        // gap lists: a running sum of the differences
                        const GapInfo gi = G.acc.info(v);
                        if (gi.deg >= wave_threshold) {
                            s_heavy[atomicAdd(&s_nheavy, 1u)] = v;
                        } else {
                            uint32_t val = 0;
                            for (uint32_t e = 0; e < gi.deg; ++e) {
                                val += G.acc.get(Acc::entry_bit(gi, e), e ? gi.g : gi.w);
                                batch_visit<Acc>(val < n ? val : n - 1, v, nd, D, P, qout, &s_tail);
                            }
                        }
                    } else if constexpr (IsVarintAcc<Acc>::value) {
                        // Varint lists: bytes from 8-byte windows (the list's
                        // byte count stands in for its degree)
                        uint64_t b0, b1;
                        G.acc.offsets(v, b0, b1);
                        if (b1 - b0 >= wave_threshold) {
                            s_heavy[atomicAdd(&s_nheavy, 1u)] = v;
                        } else {
                            uint32_t label = 0, accv = 0, shift = 0, count = 0;
                            for (uint64_t pos = b0; pos < b1;) {
                                const uint64_t k = pos >> 3;
                                const uint32_t sh = (uint32_t)(pos & 7) * 8;
                                const uint64_t w0 = G.acc.word(k * 8), w1 = G.acc.word(k * 8 + 8);
                                const uint64_t win = sh ? (w0 >> sh) | (w1 << (64 - sh)) : w0;
                                const uint32_t avail = b1 - pos < 8 ? (uint32_t)(b1 - pos) : 8u;
                                for (uint32_t j = 0; j < avail; ++j) {
                                    const uint32_t b = (uint32_t)(win >> (8 * j)) & 255u;
                                    accv |= (b & 127u) << shift;
                                    shift += 7;
                                    if (!(b & 128u)) {
                                        label = Acc::kDifferences && count ? label + accv : accv;
                                        ++count;
                                        accv = 0;
                                        shift = 0;
                                        batch_visit<Acc>(label < n ? label : n - 1, v, nd, D, P, qout, &s_tail);
                                    }
                                }
                                pos += avail;
                            }
                        }
                    } else {
                        const VInfo vi = G.acc.info(v);
                        if (vi.deg >= wave_threshold) {
                            s_heavy[atomicAdd(&s_nheavy, 1u)] = v;
                        } else {
                            const uint32_t st = Acc::step(vi.w), mk = Acc::mask(vi.w);
                            uint64_t pos = vi.start;
                            for (uint32_t e = 0; e < vi.deg; ++e, pos += st)
                                batch_visit<Acc>(G.acc.get(pos, mk), v, nd, D, P, qout, &s_tail);
                        }
                    }
                }
                __syncthreads();
                const uint32_t nh = s_nheavy;
                for (uint32_t h = wv; h < nh; h += kWaves) {
                    const uint32_t v = s_heavy[h];
                    if constexpr (IsGapAcc<Acc>::value) {
                        // 64 entries per step, a wave prefix sum
                        const GapInfo gi = G.acc.info(v);
                        uint32_t carry = 0;
                        for (uint64_t e0 = 0; e0 < gi.deg; e0 += kWave) {
                            const uint64_t e = e0 + lane;
                            const bool valid = e < gi.deg;
                            const uint32_t x = valid ? G.acc.get(Acc::entry_bit(gi, e), e ? gi.g : gi.w) : 0u;
                            const uint32_t val = wave_incl_scan(x) + carry;
                            carry = __shfl(val, kWave - 1, kWave);
                            if (valid) batch_visit<Acc>(val < n ? val : n - 1, v, nd, D, P, qout, &s_tail);
                        }
                    } else if constexpr (IsVarintAcc<Acc>::value) {
                        // 64 bytes per step (value assembly of varint_step)
                        uint64_t b0, b1;
                        G.acc.offsets(v, b0, b1);
                        uint32_t prevb = 0, carry = 0;
                        for (uint64_t p0 = b0; p0 < b1; p0 += kWave) {
                            uint32_t x;
                            const bool end = varint_step(G.acc, p0, b1, prevb, x);
                            uint32_t label = x;
                            if constexpr (Acc::kDifferences) {
                                const uint32_t sc = wave_incl_scan(end ? x : 0u);
                                label = carry + sc;
                                carry += __shfl(sc, kWave - 1, kWave);
                            }
                            if (end) batch_visit<Acc>(label < n ? label : n - 1, v, nd, D, P, qout, &s_tail);
                        }
                    } else {
                        const VInfo vi = G.acc.info(v);
                        const uint32_t st = Acc::step(vi.w), mk = Acc::mask(vi.w);
                        for (uint32_t e = lane; e < vi.deg; e += kWave)
                            batch_visit<Acc>(G.acc.get(vi.start + (uint64_t)e * st, mk), v, nd, D, P, qout,
                                             &s_tail);
                    }
                }
                __syncthreads();
            }
            if (tid == 0) s_fsize = s_tail;
            uint32_t *t = qin; qin = qout; qout = t;
            ++level;
            __syncthreads();
        }
        __syncthreads();  // s_job is rewritten next
    }
}

// ---------------------------------------------------------------------------
// searches with their bitmaps in LDS, direction-optimizing
// ---------------------------------------------------------------------------

// A graph's three bitmaps (visited, frontier, next) in LDS, at most: one
// workgroup per compute unit, which is still 14 times faster at 2^18 vertices
// (96 KB).  Above it (349,504 vertices) the large kernel.
constexpr uint64_t kBatchLdsBytes = 128u << 10;
inline uint64_t batch_bitmap_bytes(uint64_t n) { return (n + 63) / 64 * 8 * 3; }

// Direction of a level: bottom-up when the frontier's entries exceed the
// unexplored ones / 14, back when the frontier falls below n / 24 (the
// customary constants of direction-optimizing BFS).
constexpr uint64_t kBatchAlpha = 14, kBatchBeta = 24;

struct BatchBits {
    uint32_t *vis, *fr, *nx;
    __device__ __forceinline__ bool in(const uint32_t *b, uint32_t u) const { return b[u >> 5] >> (u & 31) & 1u; }
    __device__ __forceinline__ bool mark(uint32_t u) const {  // first to mark it?
        const uint32_t bit = 1u << (u & 31);
        return !(atomicOr(&nx[u >> 5], bit) & bit);
    }
};

// top-down: an edge v -> u; every claimant of the level lowers the parent
__device__ __forceinline__ void batch_claim(const BatchBits &B, uint32_t u, uint32_t v, int32_t nd,
                                            int32_t *__restrict__ D, uint32_t *__restrict__ P,
                                            uint32_t *__restrict__ qnext, uint32_t *s_tail) {
    if (B.in(B.vis, u)) return;
    if (P) atomicMin(&P[u], v);
    if (B.mark(u)) {
        D[u] = nd;
        qnext[atomicAdd(s_tail, 1u)] = u;
    }
}

// fn(label) over the list of one vertex by one lane, in order, until it
// returns false
template <class Acc, class Fn>
__device__ __forceinline__ void batch_lane_list(const Acc &acc, uint32_t n, const GapInfo &gi, Fn &&fn) {
    uint32_t val = 0;
    for (uint32_t e = 0; e < gi.deg; ++e) {
        val += acc.get(Acc::entry_bit(gi, e), e ? gi.g : gi.w);
        if (!fn(val < n ? val : n - 1)) return;
    }
}
template <class Acc, class Fn>
__device__ __forceinline__ void batch_lane_list(const Acc &acc, uint32_t n, const ulonglong2 &range, Fn &&fn) {
    // bytes from 8-byte windows
    uint32_t label = 0, accv = 0, shift = 0, count = 0;
    for (uint64_t pos = range.x; pos < range.y;) {
        const uint64_t k = pos >> 3;
        const uint32_t sh = (uint32_t)(pos & 7) * 8;
        const uint64_t w0 = acc.word(k * 8), w1 = acc.word(k * 8 + 8);
        const uint64_t win = sh ? (w0 >> sh) | (w1 << (64 - sh)) : w0;
        const uint32_t avail = range.y - pos < 8 ? (uint32_t)(range.y - pos) : 8u;
        for (uint32_t j = 0; j < avail; ++j) {
            const uint32_t b = (uint32_t)(win >> (8 * j)) & 255u;
            accv |= (b & 127u) << shift;
            shift += 7;
            if (!(b & 128u)) {
                label = Acc::kDifferences && count ? label + accv : accv;
                ++count;
                accv = 0;
                shift = 0;
                if (!fn(label < n ? label : n - 1)) return;
            }
        }
        pos += avail;
    }
}
template <class Acc, class Fn>
__device__ __forceinline__ void batch_lane_list(const Acc &acc, uint32_t, const VInfo &vi, Fn &&fn) {
    const uint32_t st = Acc::step(vi.w), mk = Acc::mask(vi.w);
    // four independent loads at a time (clamped), then in order
    for (uint32_t e = 0; e < vi.deg; e += 4) {
        uint32_t x[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            x[j] = acc.get(vi.start + (uint64_t)(e + j < vi.deg ? e + j : vi.deg - 1) * st, mk);
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
            if (e + j < vi.deg && !fn(x[j])) return;
    }
}

// fn(valid, label) over the list of one vertex by a wave, 64 entries (or
// bytes) per step, until it returns false (fn must return the same in every
// lane)
template <class Acc, class Fn>
__device__ __forceinline__ void batch_wave_list(const Acc &acc, uint32_t n, const GapInfo &gi, Fn &&fn) {
    const uint32_t lane = lane_id();
    uint32_t carry = 0;
    for (uint64_t e0 = 0; e0 < gi.deg; e0 += kWave) {
        const uint64_t e = e0 + lane;
        const bool valid = e < gi.deg;
        const uint32_t x = valid ? acc.get(Acc::entry_bit(gi, e), e ? gi.g : gi.w) : 0u;
        const uint32_t val = wave_incl_scan(x) + carry;
        carry = __shfl(val, kWave - 1, kWave);
        if (!fn(valid, val < n ? val : n - 1)) return;
    }
}
template <class Acc, class Fn>
__device__ __forceinline__ void batch_wave_list(const Acc &acc, uint32_t n, const ulonglong2 &range, Fn &&fn) {
    uint32_t prevb = 0, carry = 0;
    for (uint64_t p0 = range.x; p0 < range.y; p0 += kWave) {
        uint32_t x;
        const bool end = varint_step(acc, p0, range.y, prevb, x);
        uint32_t label = x;
        if constexpr (Acc::kDifferences) {
            const uint32_t sc = wave_incl_scan(end ? x : 0u);
            label = carry + sc;
            carry += __shfl(sc, kWave - 1, kWave);
        }
        if (!fn(end, label < n ? label : n - 1)) return;
    }
}
template <class Acc, class Fn>
__device__ __forceinline__ void batch_wave_list(const Acc &acc, uint32_t, const VInfo &vi, Fn &&fn) {
    const uint32_t lane = lane_id();
    const uint32_t st = Acc::step(vi.w), mk = Acc::mask(vi.w);
    for (uint32_t e0 = 0; e0 < vi.deg; e0 += kWave) {
        const uint32_t e = e0 + lane;
        const bool valid = e < vi.deg;
        const uint32_t x = acc.get(vi.start + (uint64_t)(valid ? e : 0u) * st, mk);
        if (!fn(valid, x)) return;
    }
}

// a list's place and its length (Varint: its bytes)
template <class Acc>
__device__ __forceinline__ auto batch_list(const Acc &acc, uint32_t v) {
    if constexpr (IsVarintAcc<Acc>::value) {
        uint64_t b0, b1;
        acc.offsets(v, b0, b1);
        return make_ulonglong2(b0, b1);
    } else {
        return acc.info(v);
    }
}
__device__ __forceinline__ uint32_t batch_len(const GapInfo &i) { return i.deg; }
__device__ __forceinline__ uint32_t batch_len(const VInfo &i) { return i.deg; }
__device__ __forceinline__ uint32_t batch_len(const ulonglong2 &i) { return (uint32_t)(i.y - i.x); }

// One search per workgroup at a time.  What bounds it is latency: a search
// reads its lists level by level, each vertex a chain offset -> list -> LDS
// bit, so the bitmaps sit in LDS (a random probe there costs no memory
// access), four list loads are in flight per lane, and bottom-up levels read
// a list only to its first frontier neighbour, with no atomics.  1,024
// searches over 64 Kronecker graphs of 2^12 to 2^16 vertices: 24.1 ms
// top-down over depths in memory, 1.2 ms; 256 over 16 graphs of 2^14 to 2^18:
// 50.0 and 3.5 ms.
//
// Long chains are levels of a few vertices, each the chain of loads once and
// its barriers.  A level therefore sums its frontier's entries ahead only
// where that many could turn it bottom-up, settles the bitmaps by the queue
// while that is the shorter, and has its counters doubled instead of cleared
// between two barriers: two barriers a level, where no list is long (path of
// 2^16 vertices: 155 ms with five and a pass over the bitmaps, 114 ms so; over
// depths in memory 117).
struct BatchCounters {
    uint32_t tail;              // vertices found
    unsigned long long edges;   // entries of the frontier (top-down) or of the vertices found (bottom-up)
    unsigned long long ahead;   // entries of the frontier summed ahead, or the places taken of a queue
};

template <class Acc, int kThreads>
__device__ __forceinline__ void batch_search(const BatchGraph<Acc> &G, uint32_t root, int32_t *__restrict__ D,
                                             uint32_t *__restrict__ P, int32_t max_depth, uint32_t *qa, uint32_t *qb,
                                             uint32_t chunk, uint32_t wave_threshold) {
    extern __shared__ uint32_t s_bits[];
    __shared__ BatchCounters s_ctr[2];  // of odd and even levels
    __shared__ uint32_t s_nheavy;
    __shared__ uint32_t s_heavy[kMaxChunk];
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = lane_id();
    const uint32_t wv = tid / kWave;
    constexpr uint32_t kWaves = kThreads / kWave;
    const uint32_t n = G.n, words = (n + 63) / 64 * 2;
    const BatchBits B{s_bits, s_bits + words, s_bits + 2 * words};
    for (uint32_t i = tid; i < 3 * words; i += kThreads) s_bits[i] = 0;
    if (P)
        for (uint32_t v = tid; v < n; v += kThreads) P[v] = v == root ? root : 0xFFFFFFFFu;
    __syncthreads();
    if (tid == 0) {
        qa[0] = root;
        D[root] = 0;
        B.vis[root >> 5] = 1u << (root & 31);
        s_ctr[0] = s_ctr[1] = BatchCounters{0, 0, 0};
        s_nheavy = 0;
    }
    __syncthreads();
    const bool long_lists = G.longest >= wave_threshold;
    uint32_t *qin = qa, *qout = qb;
    uint32_t F = 1;                  // frontier vertices (the same in every thread, as all below)
    uint64_t unexplored = G.m;       // entries of the lists not on a frontier yet (Varint: bytes count for entries)
    uint64_t edges = 0;              // entries of the frontier, where known
    bool bottom = false;             // the frontier is the bitmap fr, else the queue qin
    bool marked = false;             // fr holds an earlier frontier
    for (int32_t level = 0; F && !(max_depth >= 0 && level >= max_depth); ++level) {
        const int32_t nd = level + 1;
        BatchCounters &ctr = s_ctr[level & 1];
        // the other level's were last read before the barrier that ended it
        if (tid == 0) s_ctr[(level & 1) ^ 1] = BatchCounters{0, 0, 0};
        bool counted = true;
        if (bottom) {
            if (F < n / kBatchBeta) {
                bottom = false;
                for (uint32_t w = tid; w < words; w += kThreads) {
                    uint32_t x = B.fr[w];
                    uint32_t at = x ? (uint32_t)atomicAdd(&ctr.ahead, (unsigned long long)__popc(x)) : 0u;
                    for (; x; x &= x - 1) qin[at++] = w * 32 + (uint32_t)__ffs((int)x) - 1;
                }
                __syncthreads();
            }
        } else if (F * G.longest > unexplored / kBatchAlpha) {
            unsigned long long mine = 0;
            for (uint32_t i = tid; i < F; i += kThreads) mine += batch_len(batch_list(G.acc, qin[i]));
            mine = wave_sum(mine);
            if (lane == 0 && mine) atomicAdd(&ctr.ahead, mine);
            __syncthreads();
            edges = ctr.ahead;
            bottom = edges > unexplored / kBatchAlpha;
            if (bottom) {
                if (marked) {
                    for (uint32_t w = tid; w < words; w += kThreads) B.fr[w] = 0;
                    __syncthreads();
                }
                marked = true;
                for (uint32_t i = tid; i < F; i += kThreads) {
                    const uint32_t u = qin[i];
                    atomicOr(&B.fr[u >> 5], 1u << (u & 31));
                }
                __syncthreads();
            }
        } else {
            counted = false;  // by the level itself
            edges = 0;
        }
        unexplored = unexplored > edges ? unexplored - edges : 0;
        if (bottom) {
            // a lane per unvisited vertex; the first frontier neighbour in its
            // list is the smallest.  Long lists wait for a wave.
            uint32_t found = 0;
            unsigned long long sum = 0;
            for (uint32_t v0 = wv * kWave; v0 < n; v0 += kWaves * kWave) {
                const uint32_t v = v0 + lane;
                const bool open = v < n && !B.in(B.vis, v);
                if (!__ballot(open)) continue;
                auto li = [&]() {
                    if constexpr (IsGapAcc<Acc>::value || IsVarintAcc<Acc>::value)
                        return batch_list(G.acc, v < n ? v : n - 1);
                    else
                        return wave_info(G.acc, v0, n);
                }();
                if (!open) continue;
                const uint32_t len = batch_len(li);
                if (len >= wave_threshold) {
                    qout[atomicAdd(&s_nheavy, 1u)] = v;
                    continue;
                }
                batch_lane_list(G.acc, n, li, [&](uint32_t u) {
                    if (!B.in(B.fr, u)) return true;
                    B.mark(v);
                    D[v] = nd;
                    if (P) P[v] = u;
                    ++found;
                    sum += len;
                    return false;
                });
            }
            __syncthreads();
            const uint32_t nh = s_nheavy;
            for (uint32_t h = wv; h < nh; h += kWaves) {
                const uint32_t v = __builtin_amdgcn_readfirstlane(qout[h]);
                const auto li = batch_list(G.acc, v);
                batch_wave_list(G.acc, n, li, [&](bool valid, uint32_t u) {
                    const uint64_t hit = __ballot(valid && B.in(B.fr, u));
                    if (!hit) return true;
                    if (lane == (uint32_t)__ffsll((long long)hit) - 1) {
                        B.mark(v);
                        D[v] = nd;
                        if (P) P[v] = u;
                        ++found;
                        sum += batch_len(li);
                    }
                    return false;
                });
            }
            found = wave_sum(found);
            sum = wave_sum(sum);
            if (lane == 0 && found) {
                atomicAdd(&ctr.tail, found);
                atomicAdd(&ctr.edges, sum);
            }
        } else {
            unsigned long long mine = 0;
            for (uint32_t c0 = 0; c0 < F; c0 += chunk) {
                const uint32_t c1 = c0 + chunk < F ? c0 + chunk : F;
                for (uint32_t i = c0 + tid; i < c1; i += kThreads) {
                    const uint32_t v = qin[i];
                    const auto li = batch_list(G.acc, v);
                    const uint32_t len = batch_len(li);
                    mine += len;
                    if (len >= wave_threshold) {
                        s_heavy[atomicAdd(&s_nheavy, 1u)] = v;
                    } else {
                        batch_lane_list(G.acc, n, li, [&](uint32_t u) {
                            batch_claim(B, u, v, nd, D, P, qout, &ctr.tail);
                            return true;
                        });
                    }
                }
                if (!long_lists) continue;  // nothing is left for the waves
                __syncthreads();
                const uint32_t nh = s_nheavy;
                for (uint32_t h = wv; h < nh; h += kWaves) {
                    const uint32_t v = __builtin_amdgcn_readfirstlane(s_heavy[h]);
                    batch_wave_list(G.acc, n, batch_list(G.acc, v), [&](bool valid, uint32_t u) {
                        if (valid) batch_claim(B, u, v, nd, D, P, qout, &ctr.tail);
                        return true;
                    });
                }
                if (c1 == F) break;
                __syncthreads();
                if (tid == 0) s_nheavy = 0;
                __syncthreads();
            }
            if (!counted) {
                mine = wave_sum(mine);
                if (lane == 0 && mine) atomicAdd(&ctr.edges, mine);
            }
            uint32_t *t = qin; qin = qout; qout = t;
        }
        __syncthreads();
        F = ctr.tail;
        if (tid == 0) s_nheavy = 0;
        if (bottom) {
            edges = ctr.edges;
            for (uint32_t w = tid; w < words; w += kThreads) {
                const uint32_t x = B.nx[w];
                B.vis[w] |= x;
                B.fr[w] = x;
                B.nx[w] = 0;
            }
        } else {
            if (!counted) unexplored = unexplored > ctr.edges ? unexplored - ctr.edges : 0;
            if (F < words) {
                for (uint32_t i = tid; i < F; i += kThreads) {
                    const uint32_t u = qin[i];
                    atomicOr(&B.vis[u >> 5], 1u << (u & 31));
                    B.nx[u >> 5] = 0;  // (all its bits are in the queue)
                }
            } else {
                for (uint32_t w = tid; w < words; w += kThreads) {
                    B.vis[w] |= B.nx[w];
                    B.nx[w] = 0;
                }
            }
        }
        __syncthreads();
    }
    for (uint32_t v = tid; v < n; v += kThreads)
        if (!B.in(B.vis, v)) D[v] = -1;
}

template <class Acc, int kThreads>
__global__ __launch_bounds__(kThreads) void bfs_batch_kernel(
    const BatchGraph<Acc> *__restrict__ graphs, const BatchJob *__restrict__ jobs, uint32_t num_jobs,
    uint32_t *__restrict__ job_counter, int32_t *__restrict__ depth, int32_t *__restrict__ parent,
    int32_t max_depth, uint32_t *__restrict__ queues, uint64_t qcap, uint32_t chunk, uint32_t wave_threshold) {
    __shared__ uint32_t s_job;
    uint32_t *qa = queues + (uint64_t)blockIdx.x * 2 * qcap;
    for (;;) {
        if (threadIdx.x == 0) s_job = atomicAdd(job_counter, 1u);
        __syncthreads();
        const uint32_t job = s_job;
        if (job >= num_jobs) break;
        const BatchJob jb = jobs[job];
        const BatchGraph<Acc> G = graphs[jb.graph];
        batch_search<Acc, kThreads>(G, jb.root, depth + jb.out_offset,
                                    parent ? reinterpret_cast<uint32_t *>(parent + jb.out_offset) : nullptr, max_depth,
                                    qa, qa + qcap, chunk, wave_threshold);
        __syncthreads();  // s_job and the bitmaps are rewritten next
    }
}

// The searches of one call on a small graph: a workgroup per root, one launch
// and no read-back, where a wide search's levels cost three launches and a
// read-back or two each.  Bound by the chain of levels within a workgroup
// (Kronecker 2^12: 181 -> 61 us for one root, 960 -> 86 for 15; uniform 2^13:
// 175 -> 114 and 801 -> 118).  Lists from 128 entries go to a wave (from 32:
// uniform 2^13 282 us).
constexpr uint32_t kSmallThreads = 1024, kSmallWaveList = 128;
struct SmallRoots {
    uint32_t v[kBfsSmallRoots];
};

template <class Acc>
__global__ __launch_bounds__(kSmallThreads) void bfs_small_kernel(BatchGraph<Acc> G, SmallRoots roots,
                                                                  const uint32_t *__restrict__ inv,
                                                                  int32_t *__restrict__ depth,
                                                                  uint32_t *__restrict__ parent, int32_t max_depth,
                                                                  uint32_t *__restrict__ queues) {
    const uint64_t row = (uint64_t)blockIdx.x * G.n;
    const uint32_t root = roots.v[blockIdx.x];
    uint32_t *qa = queues + 2 * row;
    batch_search<Acc, kSmallThreads>(G, inv ? inv[root] : root, depth + row, parent ? parent + row : nullptr,
                                     max_depth, qa, qa + G.n, kMaxChunk, kSmallWaveList);
}

__global__ void batch_reset_kernel(uint32_t *__restrict__ counter) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *counter = 0;
}

// Workspaces of these searches.  A call returns with its kernels still queued,
// so what it used may only be written again after them, also when the next
// call comes on another stream (a handle can be a new stream's, once the one
// it named is destroyed).  A workspace therefore carries an event, and whoever
// takes it waits for that on the device.  The lock is held while a call queues
// its work.
constexpr uint64_t kSmallBytes = (uint64_t)kBfsSmallRoots * kBfsSmallVertices * 16;
constexpr size_t kSmallSlots = 8;  // per device: calls that can be in flight side by side
struct SmallSlot {
    DevBuf mem;  // two queues a root; relabeled: rows in label space behind them
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
    ~SmallSlot() {
        if (done) {
            (void)hipEventSynchronize(done);
            (void)hipEventDestroy(done);
        }
    }
};
struct SmallSlots {
    std::mutex mu;
    std::map<int, std::vector<std::unique_ptr<SmallSlot>>> of;  // by device, least recently used first
};
static SmallSlots &small_slots() {
    static SmallSlots *s = new SmallSlots();  // never destroyed: no frees during static teardown
    return *s;
}

void bfs_small_trim() {
    SmallSlots &all = small_slots();
    std::lock_guard<std::mutex> hold(all.mu);
    all.of.clear();
}

// the workspace that this stream used last, else an idle or a new one, else
// the least recently used; moved to the end of `slots`
static lg_status small_take(std::vector<std::unique_ptr<SmallSlot>> &slots, hipStream_t s) {
    size_t at = 0;
    while (at < slots.size() && slots[at]->last != s) ++at;
    if (at == slots.size()) {
        at = 0;
        while (at < slots.size() && hipEventQuery(slots[at]->done) != hipSuccess) ++at;
        (void)hipGetLastError();  // "not ready" is no failure
    }
    if (at == slots.size() && at == kSmallSlots) at = 0;
    if (at == slots.size()) {
        auto slot = std::make_unique<SmallSlot>();
        LG_TRY(slot->mem.alloc(kSmallBytes));
        LG_CHECK_HIP(hipEventCreateWithFlags(&slot->done, hipEventDisableTiming));
        slots.push_back(std::move(slot));
    } else {
        LG_CHECK_HIP(hipStreamWaitEvent(s, slots[at]->done, 0));
        std::rotate(slots.begin() + at, slots.begin() + at + 1, slots.end());
    }
    slots.back()->last = s;
    return LG_OK;
}

static lg_status small_launch(lg_graph *g, SmallSlot &slot, const uint32_t *roots, uint32_t r, int32_t *depth,
                              int32_t *parent, int32_t max_depth, hipStream_t s) {
    const uint32_t n = g->n;
    const bool rel = g->relabel != LG_RELABEL_NONE;
    const uint64_t rows = (uint64_t)r * n;
    uint32_t *queues = slot.mem.as<uint32_t>();
    int32_t *d = rel ? (int32_t *)(queues + 2 * rows) : depth;
    uint32_t *p = !parent ? nullptr : rel ? queues + 3 * rows : reinterpret_cast<uint32_t *>(parent);
    SmallRoots ids{};
    for (uint32_t i = 0; i < r; ++i) ids.v[i] = roots[i];
    LG_TRY(dispatch_acc_dec(g, [&](auto acc) -> lg_status {
        using Acc = decltype(acc);
        const BatchGraph<Acc> G{acc, n, IsVarintAcc<Acc>::value ? g->U / 8 : g->m,
                                (uint64_t)g->max_degree * (IsVarintAcc<Acc>::value ? 5 : 1)};
        LG_LAUNCH(bfs_small_kernel<Acc>, r, kSmallThreads, (uint32_t)batch_bitmap_bytes(n), s, G, ids,
                  rel ? g->inv.as<const uint32_t>() : nullptr, d, p, max_depth, queues);
        LG_CHECK_LAUNCH();
        return LG_OK;
    }));
    if (!rel) return LG_OK;
    return bfs_unpermute(g, d, p, r, depth, parent, s);
}

lg_status bfs_small(lg_graph *g, const uint32_t *roots, uint32_t r, int32_t *depth, int32_t *parent,
                    int32_t max_depth, hipStream_t s) {
    SmallSlots &all = small_slots();
    std::lock_guard<std::mutex> hold(all.mu);
    try {
        auto &slots = all.of[g->device];
        LG_TRY(small_take(slots, s));
        const lg_status st = small_launch(g, *slots.back(), roots, r, depth, parent, max_depth, s);
        LG_CHECK_HIP(hipEventRecord(slots.back()->done, s));
        return st;
    } catch (const std::bad_alloc &) {
        set_error("lg_bfs: host allocation failed");
        return LG_ERR_OOM;
    }
}

}  // namespace lg

// ---------------------------------------------------------------------------
// the plan
// ---------------------------------------------------------------------------

struct lg_batch_plan {
    int device = 0;
    uint32_t layout = 0, id_mode = 0, offset_mode = 0;
    uint32_t num_graphs = 0, num_jobs = 0;
    uint64_t qcap = 0;
    int32_t *depth = nullptr, *parent = nullptr;
    int32_t max_depth = -1;
    uint32_t threads = 256, chunk = 256, wave_threshold = 32, workgroups = 0;
    uint64_t lds = 0;  // bytes of the largest graph's bitmaps; 0: the large kernel
    double tuned_ms = 0.0;
    uint32_t candidates = 0;
    lg::DevBuf graphs, jobs, counter, queues;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    std::vector<lg_graph *> handles;  // the plan's graphs (each run is one use of each)
    hipEvent_t last_run = nullptr;    // recorded after every replay
};

namespace lg {

// fn(kernel) with the kernel of the plan's settings
template <class Acc, class Fn>
static lg_status batch_kernel(const lg_batch_plan *p, Fn &&fn) {
    if (!p->lds) return p->threads == 256 ? fn(bfs_batch_large_kernel<Acc, 256>) : fn(bfs_batch_large_kernel<Acc, 512>);
    if (p->threads == 256) return fn(bfs_batch_kernel<Acc, 256>);
    if (p->threads == 512) return fn(bfs_batch_kernel<Acc, 512>);
    return fn(bfs_batch_kernel<Acc, 1024>);
}

template <class Acc>
static lg_status batch_launch(lg_batch_plan *p, hipStream_t s) {
    LG_LAUNCH(batch_reset_kernel, 1, 64, 0, s, p->counter.as<uint32_t>());
    LG_CHECK_LAUNCH();
    const auto *G = p->graphs.as<const BatchGraph<Acc>>();
    const auto *J = p->jobs.as<const BatchJob>();
    return batch_kernel<Acc>(p, [&](auto kernel) -> lg_status {
        // (the launch's name in the profile is the variable's)
        auto launch = [&](auto &&go) -> lg_status {
            go(p->workgroups, p->threads, (uint32_t)p->lds, s, G, J, p->num_jobs, p->counter.as<uint32_t>(), p->depth,
               p->parent, p->max_depth, p->queues.as<uint32_t>(), p->qcap, p->chunk, p->wave_threshold);
            LG_CHECK_LAUNCH();
            return LG_OK;
        };
        if (p->lds) {
            const auto bfs_batch_kernel = kernel;
            return launch([&](uint32_t grid, uint32_t block, uint32_t lds, hipStream_t st, auto... args) {
                LG_LAUNCH(bfs_batch_kernel, grid, block, lds, st, args...);
            });
        }
        const auto bfs_batch_large_kernel = kernel;
        return launch([&](uint32_t grid, uint32_t block, uint32_t lds, hipStream_t st, auto... args) {
            LG_LAUNCH(bfs_batch_large_kernel, grid, block, lds, st, args...);
        });
    });
}

template <class Acc>
static lg_status batch_workgroups(lg_batch_plan *p, uint32_t &wg) {
    int cus = 0, per = 0;
    LG_CHECK_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device));
    LG_TRY(batch_kernel<Acc>(p, [&](auto kernel) -> lg_status {
        LG_CHECK_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, (int)p->threads, (size_t)p->lds));
        return LG_OK;
    }));
    if (per < 1) per = 1;
    wg = (uint32_t)std::min<uint64_t>((uint64_t)cus * per, p->num_jobs ? p->num_jobs : 1);
    return LG_OK;
}

// (Re)allocate the per-workgroup queues for p->workgroups workers.
static lg_status batch_queues(lg_batch_plan *p) {
    return p->queues.ensure((uint64_t)p->workgroups * 2 * p->qcap * 4);
}

template <class Acc>
static lg_status batch_build(lg_batch_plan *p, const lg_graph *const *gs, bool autotune, hipStream_t s) {
    std::vector<BatchGraph<Acc>> hg(p->num_graphs);
    for (uint32_t i = 0; i < p->num_graphs; ++i) {
        const lg_graph *g = gs[i];
        if constexpr (IsGapAcc<Acc>::value || IsVarintAcc<Acc>::value) hg[i].acc = Acc{{g->packed_view()}};
        else if constexpr (Acc::kPacked) hg[i].acc = Acc{g->packed_view()};
        else hg[i].acc = Acc{g->plain_view()};
        hg[i].n = g->n;
        hg[i].m = IsVarintAcc<Acc>::value ? g->U / 8 : g->m;
        hg[i].longest = (uint64_t)g->max_degree * (IsVarintAcc<Acc>::value ? 5 : 1);
    }
    LG_TRY(p->graphs.alloc(sizeof(BatchGraph<Acc>) * hg.size()));
    LG_CHECK_HIP(hipMemcpy(p->graphs.p, hg.data(), sizeof(BatchGraph<Acc>) * hg.size(), hipMemcpyHostToDevice));

    struct Cfg { uint32_t threads, chunk, wt; };
    std::vector<Cfg> cands;
    if (autotune) {
        if (p->lds) {
            for (uint32_t th : {256u, 512u, 1024u})
                for (uint32_t wt : {16u, 32u, 64u, 128u}) cands.push_back({th, kMaxChunk, wt});
        } else {
            for (uint32_t th : {256u, 512u})
                for (uint32_t ch : {256u, 1024u})
                    for (uint32_t wt : {8u, 32u, 128u}) cands.push_back({th, ch, wt});
        }
    } else {
        cands.push_back({p->threads, p->chunk, p->wave_threshold});
    }
    p->candidates = (uint32_t)cands.size();
    hipEvent_t e0, e1;
    LG_CHECK_HIP(hipEventCreate(&e0));
    LG_CHECK_HIP(hipEventCreate(&e1));
    float best = -1.f;
    Cfg bestc = cands[0];
    lg_status st = LG_OK;
    for (const Cfg &c : cands) {
        p->threads = c.threads;
        p->chunk = c.chunk;
        p->wave_threshold = c.wt;
        if ((st = batch_workgroups<Acc>(p, p->workgroups)) != LG_OK) break;
        if ((st = batch_queues(p)) != LG_OK) break;
        if (cands.size() > 1) {
            if ((st = batch_launch<Acc>(p, s)) != LG_OK) break;  // warm-up
        }
        (void)hipEventRecord(e0, s);
        if ((st = batch_launch<Acc>(p, s)) != LG_OK) break;
        (void)hipEventRecord(e1, s);
        if (hipEventSynchronize(e1) != hipSuccess) { st = LG_ERR_DEVICE; set_error("batch: sync failed"); break; }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        if (best < 0.f || ms < best) { best = ms; bestc = c; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    LG_TRY(st);
    p->threads = bestc.threads;
    p->chunk = bestc.chunk;
    p->wave_threshold = bestc.wt;
    p->tuned_ms = best;
    LG_TRY(batch_workgroups<Acc>(p, p->workgroups));
    LG_TRY(batch_queues(p));
    // capture reset + launch into a graph, on a private stream (the legacy
    // default stream cannot be captured; capturing executes nothing, and the
    // graph is launched later on the caller's stream)
    LG_CHECK_HIP(hipStreamSynchronize(s));
    hipStream_t cs = nullptr;
    LG_CHECK_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipError_t ce = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    hipGraph_t gr = nullptr;
    if (ce == hipSuccess) {
        st = batch_launch<Acc>(p, cs);
        ce = hipStreamEndCapture(cs, &gr);
    }
    (void)hipStreamDestroy(cs);
    LG_TRY(st);
    if (ce != hipSuccess) { set_error("batch: graph capture failed: %s", hipGetErrorString(ce)); return LG_ERR_DEVICE; }
    p->graph = gr;
    LG_CHECK_HIP(hipGraphInstantiate(&p->exec, gr, nullptr, nullptr, 0));
    return LG_OK;
}

}  // namespace lg

extern "C" lg_status lg_bfs_batch_plan(const lg_graph *const *graphs, uint32_t num_graphs, const lg_bfs_job *jobs,
                                       uint32_t num_jobs, int32_t *depth, int32_t *parent, int32_t max_depth,
                                       uint32_t flags, hipStream_t stream, lg_batch_plan **out) {
    using namespace lg;
    if (!out) { set_error("lg_bfs_batch_plan: out is NULL"); return LG_ERR_INVALID; }
    *out = nullptr;
    if (!graphs || !num_graphs || (num_jobs && (!jobs || !depth))) {
        set_error("lg_bfs_batch_plan: NULL argument");
        return LG_ERR_INVALID;
    }
    if (flags & ~(uint32_t)LG_BATCH_AUTOTUNE) { set_error("lg_bfs_batch_plan: unknown flags"); return LG_ERR_INVALID; }
    const lg_graph *g0 = graphs[0];
    uint64_t qcap = 1;
    for (uint32_t i = 0; i < num_graphs; ++i) {
        const lg_graph *g = graphs[i];
        if (!g) { set_error("lg_bfs_batch_plan: NULL graph"); return LG_ERR_INVALID; }
        if (g->layout != g0->layout || g->id_mode != g0->id_mode || g->offset_mode != g0->offset_mode ||
            (g->layout == LG_LAYOUT_PLAIN && g->poff64 != g0->poff64)) {
            set_error("lg_bfs_batch_plan: all graphs must share one layout and encoding");
            return LG_ERR_UNSUPPORTED;
        }
        if (g->relabel != LG_RELABEL_NONE) {
            set_error("lg_bfs_batch_plan: relabeled graphs are not supported in batches");
            return LG_ERR_UNSUPPORTED;
        }
        if (g->layout == LG_LAYOUT_PACKED && g->weighted) {
            set_error("lg_bfs_batch_plan: packed weighted graphs are read by lg_sssp only");
            return LG_ERR_UNSUPPORTED;
        }
        qcap = std::max<uint64_t>(qcap, g->n);
    }
    std::vector<BatchJob> hj(num_jobs);
    for (uint32_t j = 0; j < num_jobs; ++j) {
        if (jobs[j].graph >= num_graphs || jobs[j].root >= graphs[jobs[j].graph]->n) {
            set_error("lg_bfs_batch_plan: job %u has a bad graph index or root", j);
            return LG_ERR_INVALID;
        }
        hj[j] = BatchJob{jobs[j].graph, jobs[j].root, jobs[j].out_offset};
    }
    // largest graphs first: long jobs start early, short ones fill the tail
    std::stable_sort(hj.begin(), hj.end(), [&](const BatchJob &a, const BatchJob &b) {
        return graphs[a.graph]->m > graphs[b.graph]->m;
    });
    lg_batch_plan *p = new (std::nothrow) lg_batch_plan();
    if (!p) { set_error("lg_bfs_batch_plan: host allocation failed"); return LG_ERR_OOM; }
    lg_status st = LG_OK;
    do {
        if (hipGetDevice(&p->device) != hipSuccess) { st = LG_ERR_DEVICE; set_error("hipGetDevice failed"); break; }
        p->layout = g0->layout;
        p->id_mode = g0->id_mode;
        p->offset_mode = g0->offset_mode;
        p->num_graphs = num_graphs;
        p->num_jobs = num_jobs;
        p->qcap = qcap;
        p->lds = batch_bitmap_bytes(qcap) <= kBatchLdsBytes ? batch_bitmap_bytes(qcap) : 0;
        p->depth = depth;
        p->parent = parent;
        p->max_depth = max_depth;
        for (uint32_t i = 0; i < num_graphs; ++i) p->handles.push_back(const_cast<lg_graph *>(graphs[i]));
        if (hipEventCreateWithFlags(&p->last_run, hipEventDisableTiming) != hipSuccess) {
            p->last_run = nullptr;
            st = LG_ERR_DEVICE;
            set_error("lg_bfs_batch_plan: hipEventCreateWithFlags failed");
            break;
        }
        if ((st = p->jobs.alloc(sizeof(BatchJob) * (num_jobs ? num_jobs : 1))) != LG_OK) break;
        if (num_jobs && hipMemcpy(p->jobs.p, hj.data(), sizeof(BatchJob) * num_jobs, hipMemcpyHostToDevice) != hipSuccess) {
            st = LG_ERR_DEVICE;
            set_error("lg_bfs_batch_plan: job upload failed");
            break;
        }
        if ((st = p->counter.alloc(8)) != LG_OK) break;
        st = dispatch_acc_dec(g0, [&](auto acc) -> lg_status {
            return batch_build<decltype(acc)>(p, graphs, (flags & LG_BATCH_AUTOTUNE) != 0, stream);
        });
    } while (0);
    if (st != LG_OK) {
        (void)hipStreamSynchronize(stream);
        lg_bfs_batch_free(p);
        return st;
    }
    *out = p;
    return LG_OK;
}

extern "C" lg_status lg_bfs_batch_run(lg_batch_plan *p, hipStream_t stream) {
    if (!p || !p->exec) { lg::set_error("lg_bfs_batch_run: bad plan"); return LG_ERR_INVALID; }
    LG_CHECK_HIP(hipGraphLaunch(p->exec, stream));
    // the plan's scratch and graphs are in use until this point of `stream`
    if (p->last_run) LG_CHECK_HIP(hipEventRecord(p->last_run, stream));
    for (lg_graph *g : p->handles) LG_TRY(lg::mark_use(g, stream));
    return LG_OK;
}

extern "C" lg_status lg_bfs_batch_info(const lg_batch_plan *p, lg_batch_info *out) {
    if (!p || !out) { lg::set_error("lg_bfs_batch_info: NULL argument"); return LG_ERR_INVALID; }
    std::memset(out, 0, sizeof(*out));
    out->num_jobs = p->num_jobs;
    out->workgroups = p->workgroups;
    out->threads = p->threads;
    out->chunk = p->chunk;
    out->wave_threshold = p->wave_threshold;
    out->candidates = p->candidates;
    out->tuned_ms = p->tuned_ms;
    out->scratch_bytes = p->queues.bytes;
    return LG_OK;
}

extern "C" void lg_bfs_batch_free(lg_batch_plan *p) {
    if (!p) return;
    // wait for the plan's own last replay, not for the whole device
    if (p->last_run) {
        (void)hipEventSynchronize(p->last_run);
        (void)hipEventDestroy(p->last_run);
    }
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    delete p;
}
