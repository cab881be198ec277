// lg_decode_neighbors: N_v for a batch of vertices (getNeighbors of the
// library listing in section "High-Performance Library"): the offset lookup,
// d_v = O[v+1] - O[v] (subsection "Accessing a Degree") and the element
// extraction of subsection "Accessing An Edge", a wave per piece of the
// output so that consecutive lanes decode consecutive elements; gap and
// Varint lists are decoded in order by a wave per list, 64 entries or bytes
// per wave step.
#include <algorithm>
#include <mutex>

#include "lg_device.hpp"
#include "lg_varint.hpp"

namespace lg {

// What a decode keeps in its head buffer behind the labels and degrees.
struct DecodeMarks {
    uint32_t bad;            // a requested vertex >= n
    uint32_t n_mid, n_long;  // lists left for the block sorts
    uint32_t n_chunked;      // Varint lists decoded by chunks, gap lists by segments
};
uint64_t decode_head_bytes(uint64_t k) { return k * 8 + sizeof(DecodeMarks); }

// the label of request i (0 where the vertex does not exist)
__device__ __forceinline__ uint32_t dec_label(uint32_t n, const uint32_t *__restrict__ vin, uint64_t i,
                                              const uint32_t *__restrict__ inv, bool &bad) {
    const uint32_t v = vin[i];
    bad = v >= n;
    return bad ? 0u : (inv ? inv[v] : v);
}

template <class Acc>
__global__ void dec_map_kernel(Acc acc, uint32_t n, const uint32_t *__restrict__ vin, uint32_t k,
                               const uint32_t *__restrict__ inv, uint32_t *__restrict__ labels,
                               uint32_t *__restrict__ deg, DecodeMarks *__restrict__ marks) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < k; i += stride) {
        bool bad;
        const uint32_t x = dec_label(n, vin, i, inv, bad);
        if (bad) atomicOr(&marks->bad, 1u);
        labels[i] = x;
        if constexpr (!IsVarintAcc<Acc>::value) deg[i] = acc.info(x).deg;
    }
}

// Varint lists: d_v is the number of bytes with the top bit clear in the
// list's byte range; one wave per vertex counts them 8 bytes per lane.
template <class Acc>
__device__ __forceinline__ uint32_t dec_varint_count(const Acc &acc, uint64_t b0, uint64_t b1) {
    uint32_t cnt = 0;
#pragma unroll 4
    for (uint64_t q = (b0 >> 3) + lane_id(); q * 8 < b1; q += kWave) {
        const uint64_t p = q * 8;
        const uint64_t lo = p < b0 ? b0 - p : 0;         // bytes below the list
        const uint64_t hi = p + 8 > b1 ? p + 8 - b1 : 0;  // bytes above it
        uint64_t keep = ~0ull << (8 * lo);
        if (hi) keep &= ~0ull >> (8 * hi);
        cnt += (uint32_t)__popcll(~acc.word(p) & 0x8080808080808080ull & keep);
    }
    return wave_sum(cnt);
}
template <class Acc>
__device__ __forceinline__ uint32_t dec_varint_degree(const Acc &acc, uint32_t label) {
    uint64_t b0, b1;
    acc.offsets(label, b0, b1);
    return dec_varint_count(acc, b0, b1);
}

template <class Acc>
__global__ void dec_varint_degree_kernel(Acc acc, const uint32_t *__restrict__ labels, uint32_t k,
                                         uint32_t *__restrict__ deg) {
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
    for (uint64_t i = wave; i < k; i += nwaves) {
        const uint32_t cnt = dec_varint_degree(acc, labels[i]);
        if (lane_id() == 0) deg[i] = cnt;
    }
}

// A small request in one launch: labels, degrees, their prefix, and the two
// values the host waits for straight into its pinned memory.  (Clearing the
// mark, labels, degrees, scan and two copies were six launches, each longer
// than its work: 64 lists 138 us in two calls, 77 so.)  Up to kDecSmall
// requests, a thread each; of Varint lists, which a wave counts, up to a
// sixteenth of that.
constexpr uint32_t kDecSmall = 1024;

template <class Acc>
__global__ __launch_bounds__(kDecSmall) void dec_small_kernel(Acc acc, uint32_t n, const uint32_t *__restrict__ vin,
                                                              uint32_t k, const uint32_t *__restrict__ inv,
                                                              uint32_t *__restrict__ labels,
                                                              uint64_t *__restrict__ out_off,
                                                              DecodeMarks *__restrict__ marks,
                                                              uint64_t *__restrict__ host) {
    __shared__ uint32_t s_deg[kDecSmall];
    __shared__ uint64_t s_wave[kDecSmall / kWave];
    __shared__ uint32_t s_bad;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    if (tid == 0) s_bad = 0;
    s_deg[tid] = 0;
    __syncthreads();
    uint32_t x = 0;
    if (tid < k) {
        bool bad;
        x = dec_label(n, vin, tid, inv, bad);
        if (bad) atomicOr(&s_bad, 1u);
        labels[tid] = x;
        if constexpr (!IsVarintAcc<Acc>::value) s_deg[tid] = acc.info(x).deg;
    }
    if constexpr (IsVarintAcc<Acc>::value) {
        __syncthreads();
        for (uint32_t i = wv; i < k; i += kDecSmall / kWave) {
            bool bad;
            const uint32_t cnt = dec_varint_degree(acc, dec_label(n, vin, i, inv, bad));
            if (lane == 0) s_deg[i] = cnt;
        }
    }
    __syncthreads();
    const uint64_t d = s_deg[tid];
    const uint64_t incl = wave_incl_scan(d);
    if (lane == kWave - 1) s_wave[wv] = incl;
    __syncthreads();
    uint64_t base = 0;
    for (uint32_t w = 0; w < wv; ++w) base += s_wave[w];
    if (tid < k) out_off[tid] = base + incl - d;
    if (tid == kDecSmall - 1) {
        out_off[k] = base + incl;
        host[0] = base + incl;
        host[1] = s_bad;
        *marks = DecodeMarks{s_bad, 0, 0, 0};
    }
}

// The values of bytes [p0, p1) of a Varint list to the output from entry o:
// 64 bytes per step, one per lane; a lane holding a value's last byte
// assembles the value (varint_step), whose index is the number of last bytes
// before it; DMd adds a wave prefix sum of the differences to the running
// label.  prevb: the bytes before p0 that belong to the list, carry: the
// label before it.
template <class Acc, bool kSorted>
__device__ __forceinline__ void dec_varint_range(const Acc &acc, uint32_t n, uint64_t p0, uint64_t p1,
                                                 uint32_t prevb, uint32_t carry, uint64_t i, uint64_t o,
                                                 const uint32_t *__restrict__ perm, uint32_t *__restrict__ out_ids,
                                                 uint64_t *__restrict__ keys) {
    for (; p0 < p1; p0 += kWave) {
        uint32_t val;
        const bool end = varint_step(acc, p0, p1, prevb, val);
        const uint64_t ends = __ballot(end);
        uint32_t label = val;
        if constexpr (Acc::kDifferences) {
            const uint32_t sc = wave_incl_scan(end ? val : 0u);
            label = carry + sc;
            carry += __shfl(sc, kWave - 1, kWave);
        }
        if (end) {
            // a stored label is < n; the clamp keeps the lookup in
            // bounds whatever the stream holds
            const uint32_t u = perm ? perm[label < n ? label : n - 1] : label;
            const uint64_t j = o + popc_below(ends);
            if (kSorted) keys[j] = (i << 32) | u;
            else out_ids[j] = u;
        }
        o += (uint64_t)__popcll(ends);
    }
}

// Varint lists in byte chunks (the traversals' chunk tables: a value belongs
// to the chunk holding its last byte, and the label before every chunk is
// stored): a workgroup per list takes a chunk per wave at a time, counts
// their values, and every wave decodes its chunk from its place.  (One wave
// walked a hub's list alone: 0.52 ms for 256,000 lists of a relabeled 2^22
// Kronecker graph, now 0.27 for the others and 0.07 for the hubs'.)
template <class Acc, bool kSorted>
__global__ __launch_bounds__(1024) void dec_varint_chunks_kernel(
    Acc acc, uint32_t n, const uint32_t *__restrict__ labels, const uint64_t *__restrict__ out_off,
    const uint32_t *__restrict__ perm, uint32_t *__restrict__ out_ids, uint64_t *__restrict__ keys,
    const uint32_t *__restrict__ more, const DecodeMarks *__restrict__ marks, const uint32_t *__restrict__ heavy,
    uint32_t n_heavy, const uint64_t *__restrict__ hb0, const uint64_t *__restrict__ hb1,
    const uint64_t *__restrict__ seg_off, const uint32_t *__restrict__ seg_base, uint32_t chunk) {
    constexpr uint32_t kWaves = 1024 / kWave;
    __shared__ uint32_t s_cnt[kWaves];
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint32_t lists = marks->n_chunked;
    for (uint32_t l = blockIdx.x; l < lists; l += gridDim.x) {
        const uint32_t i = more[l];
        const uint32_t h = heavy_index(heavy, n_heavy, labels[i]);
        const uint64_t b0 = hb0[h], b1 = hb1[h], s0 = seg_off[h], chunks = seg_off[h + 1] - s0;
        uint64_t o = out_off[i];
        for (uint64_t c0 = 0; c0 < chunks; c0 += kWaves) {
            const uint64_t c = c0 + wv;
            const uint64_t pa = c < chunks ? b0 + c * chunk : b1;
            const uint64_t pz = pa + chunk < b1 ? pa + chunk : b1;
            const uint32_t cnt = dec_varint_count(acc, pa, pz);
            if (lane == 0) s_cnt[wv] = cnt;
            __syncthreads();
            uint64_t before = 0, all = 0;
            for (uint32_t w = 0; w < kWaves; ++w) {
                if (w < wv) before += s_cnt[w];
                all += s_cnt[w];
            }
            if (c < chunks)
                dec_varint_range<Acc, kSorted>(acc, n, pa, pz, varint_chunk_prevb(acc, b0, pa),
                                               Acc::kDifferences ? seg_base[s0 + c] : 0u, i, o + before, perm,
                                               out_ids, keys);
            o += all;
            __syncthreads();  // the counts are rewritten
        }
    }
}

// Entries [j0, j1) of a gap list to the output from entry o + j0: an element is
// the first element plus the differences up to it; 64 at a time, a wave prefix
// sum plus the running total of the steps before (lanes past the end read the
// first element and drop it).  carry: the entry before j0.
template <class Acc, bool kSorted>
__device__ __forceinline__ void dec_gap_range(const Acc &acc, uint32_t n, const GapInfo &gi, uint64_t j0, uint64_t j1,
                                              uint32_t carry, uint64_t i, uint64_t o,
                                              const uint32_t *__restrict__ perm, uint32_t *__restrict__ out_ids,
                                              uint64_t *__restrict__ keys) {
    const uint32_t lane = lane_id();
    for (; j0 < j1; j0 += kWave) {
        const uint64_t j = j0 + lane;
        const bool valid = j < j1;
        const uint64_t jj = valid ? j : 0;
        const uint32_t x = acc.get(Acc::entry_bit(gi, jj), jj ? gi.g : gi.w);
        const uint32_t val = wave_incl_scan(valid ? x : 0u) + carry;
        carry = __shfl(val, kWave - 1, kWave);
        if (valid) {
            // a stored label is < n; the clamp keeps the lookup in bounds
            // whatever the stream holds
            const uint32_t u = perm ? perm[val < n ? val : n - 1] : val;
            if (kSorted) keys[o + j] = (i << 32) | u;
            else out_ids[o + j] = u;
        }
    }
}

// Gap lists above the split of the segment tables (built with the encoding; the
// entry before every segment is stored): the workgroups share the lists, several
// a list when there are fewer, a wave a segment.  (One wave walked a hub's list:
// 1.5 M entries took 8 ms of a PageRank build.)
constexpr uint32_t kDecGapThreads = 256;
// ... and above m / 2^8: a wave takes 5.3 ns an entry, the chip 0.06 ns, so a list
// is the kernel's tail from m / 90 on (and was left to the waves to m / 2^8, since
// the test and the hand-over cost 5 to 8 % of kron21-d4 where every list over the
// tables' split was taken out)
constexpr uint32_t kDecGapShare = 8;
template <class Acc, bool kSorted>
__global__ __launch_bounds__(kDecGapThreads) void dec_gap_segs_kernel(
    Acc acc, uint32_t n, const uint32_t *__restrict__ labels, const uint64_t *__restrict__ out_off,
    const uint32_t *__restrict__ perm, uint32_t *__restrict__ out_ids, uint64_t *__restrict__ keys,
    const uint32_t *__restrict__ more, const DecodeMarks *__restrict__ marks, const uint32_t *__restrict__ heavy,
    uint32_t n_heavy, const uint64_t *__restrict__ hstart, const uint32_t *__restrict__ hdeg,
    const uint32_t *__restrict__ hw, const uint32_t *__restrict__ hg, const uint64_t *__restrict__ seg_off,
    const uint32_t *__restrict__ seg_base, uint32_t seg_size) {
    constexpr uint32_t kWaves = kDecGapThreads / kWave;
    const uint32_t lists = marks->n_chunked, wv = threadIdx.x / kWave;
    if (!lists) return;
    const uint32_t per = lists < gridDim.x ? gridDim.x / lists : 1, groups = gridDim.x / per;
    if (blockIdx.x >= groups * per) return;
    for (uint32_t l = blockIdx.x / per; l < lists; l += groups) {
        const uint32_t i = more[l], h = heavy_index(heavy, n_heavy, labels[i]);
        const GapInfo gi{hstart[h], hdeg[h], hw[h], hg[h]};
        const uint64_t s0 = seg_off[h], segs = seg_off[h + 1] - s0;
        for (uint64_t k = (uint64_t)(blockIdx.x % per) * kWaves + wv; k < segs; k += (uint64_t)per * kWaves) {
            const uint64_t j0 = k * seg_size, j1 = j0 + seg_size < gi.deg ? j0 + seg_size : gi.deg;
            dec_gap_range<Acc, kSorted>(acc, n, gi, j0, j1, seg_base[s0 + k], i, out_off[i], perm, out_ids, keys);
        }
    }
}

// kSorted: emit ((i << 32) | original ID) keys for the segmented sort
// kSplit: lists longer than `split` are left in `more` (gap lists test it only
// where the graph has such a list: 5 to 8 % of the kernel on lists of 8)
template <class Acc, bool kSorted, bool kSplit>
__global__ void dec_lists_kernel(Acc acc, uint32_t n, const uint32_t *__restrict__ labels, uint32_t k,
                                 const uint64_t *__restrict__ out_off, const uint32_t *__restrict__ perm,
                                 uint32_t *__restrict__ out_ids, uint64_t *__restrict__ keys, uint64_t split,
                                 uint32_t *__restrict__ more, DecodeMarks *__restrict__ marks) {
    const uint32_t lane = lane_id();
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
    if constexpr (IsGapAcc<Acc>::value) {
        // gap lists of up to `split` entries; longer ones are left in `more`
        for (uint64_t i = wave; i < k; i += nwaves) {
            const GapInfo gi = acc.info(labels[i]);
            const uint64_t o = out_off[i];
            if (kSplit && gi.deg > split) {
                if (lane == 0) more[atomicAdd(&marks->n_chunked, 1u)] = (uint32_t)i;
                continue;
            }
            dec_gap_range<Acc, kSorted>(acc, n, gi, 0, gi.deg, 0u, i, o, perm, out_ids, keys);
        }
    } else if constexpr (IsVarintAcc<Acc>::value) {
        // Varint lists of up to `split` bytes; longer ones are left in `more`
        for (uint64_t i = wave; i < k; i += nwaves) {
            uint64_t b0, b1;
            acc.offsets(labels[i], b0, b1);
            if (b1 - b0 > split) {
                if (lane == 0) more[atomicAdd(&marks->n_chunked, 1u)] = (uint32_t)i;
                continue;
            }
            dec_varint_range<Acc, kSorted>(acc, n, b0, b1, 0u, 0u, i, out_off[i], perm, out_ids, keys);
        }
    }
}

// Fixed-width and plain lists: the output is one range of entries (out_off is
// the prefix of the list lengths), cut into equal pieces, a wave each, whatever
// the list lengths.  A piece is `per` units, a list counting for one beside its
// entries, so that empty lists are shared out too (pieces of entries alone
// left a wave millions of empty lists to step over: 1,000 entries in 2^24
// lists 68.7 ms, now 0.33).  (A wave per list left half its lanes idle at
// degree 32 and put a dependent chain label -> offset -> list in front of
// every list: 537 M entries in 16.7 M lists took 5.26 ms, a sixth of the copy
// rate; a hub's list was one wave's.)  The wave finds the lists of its ends
// with 64 probes per step, then takes 64 lists at a time: a lane each decodes
// its list's offsets, and the lists' first entries, held
// across the lanes, tell every entry its list by a search with cross-lane
// reads.  kDecSteps steps of 64 entries have their loads in flight together.
// Same decode: 5.26 -> 1.25 ms (26-bit IDs, 4.0 GB read and written, 3.2
// TB/s; the cross-lane reads, about ten a step, take the rest); 130 M entries
// of a relabeled Kronecker graph, 2.90 -> 0.84 ms, there bound by the random
// reads of perm.
constexpr uint32_t kDecSteps = 4;
constexpr uint64_t kDecWaves = 8192;  // waves resident on 256 CUs

template <class Acc, bool kSorted>
__global__ __launch_bounds__(256) void dec_walk_kernel(Acc acc, const uint32_t *__restrict__ labels, uint32_t k,
                                                       uint64_t total, uint32_t per,
                                                       const uint64_t *__restrict__ out_off,
                                                       const uint32_t *__restrict__ perm,
                                                       uint32_t *__restrict__ out_ids, uint64_t *__restrict__ keys) {
    const uint32_t lane = lane_id();
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    // the piece's units and, for its two ends, the last list whose own unit is
    // not after them (both searches' loads in flight together)
    const uint64_t units = total + k;
    const uint64_t d[2] = {wave * per, wave * per + per < units ? wave * per + per : units};
    if (d[0] >= units) return;
    uint32_t lo[2] = {0, 0}, hi[2] = {k, k};
    while (hi[0] - lo[0] > 1 || hi[1] - lo[1] > 1) {
        uint32_t step[2];
        bool le[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            step[q] = (hi[q] - lo[q] + kWave - 1) / kWave;
            const uint64_t at = (uint64_t)lo[q] + (uint64_t)lane * step[q];
            const uint64_t i = at < hi[q] ? at : lo[q];
            le[q] = at < hi[q] && out_off[i] + i <= d[q];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            lo[q] += (uint32_t)(__popcll(__ballot(le[q])) - 1) * step[q];
            hi[q] = hi[q] - lo[q] > step[q] ? lo[q] + step[q] : hi[q];
        }
    }
    // the entries before a unit: it less the lists begun by then
    auto before = [&](int q) {
        const uint64_t o = out_off[lo[q]];
        return o + lo[q] == d[q] ? o : d[q] - lo[q] - 1;
    };
    uint64_t e = before(0);
    const uint64_t e_end = before(1);
    for (uint64_t r = lo[0]; e < e_end; r += kWave) {
        // lane's list: its first entry relative to e, and where its entry
        // number x of the whole output would lie, less x elements
        const uint64_t i = r + lane;
        const uint64_t beg = out_off[i < k ? i : k];
        const uint64_t next = out_off[r + kWave < k ? r + kWave : k];
        const uint32_t rel = beg <= e ? 0u : (beg - e < 0xFFFFFFFFull ? (uint32_t)(beg - e) : 0xFFFFFFFFu);
        const VInfo vi = i < k ? acc.info(labels[i]) : VInfo{0, 0, 0};
        const uint64_t origin = vi.start - beg * Acc::step(vi.w);
        const uint32_t len = (uint32_t)((next < e_end ? next : e_end) - e);
        for (uint32_t t0 = 0; t0 < len; t0 += kWave * kDecSteps) {
            uint32_t x[kDecSteps], p[kDecSteps];
#pragma unroll
            for (uint32_t q = 0; q < kDecSteps; ++q) {
                const uint32_t t = t0 + q * kWave + lane;
                const uint32_t tt = t < len ? t : len - 1;
                p[q] = 0;  // the last list that begins at or before entry tt
#pragma unroll
                for (uint32_t d = kWave / 2; d; d >>= 1) {
                    const uint32_t b = __shfl(rel, p[q] + d, kWave);
                    if (b <= tt) p[q] += d;
                }
                const uint32_t w = __shfl(vi.w, p[q], kWave);
                const uint64_t pos = __shfl(origin, p[q], kWave) + (e + tt) * Acc::step(w);
                x[q] = acc.get(pos, Acc::mask(w));
            }
            if (perm) {
#pragma unroll
                for (uint32_t q = 0; q < kDecSteps; ++q) x[q] = perm[x[q]];
            }
#pragma unroll
            for (uint32_t q = 0; q < kDecSteps; ++q) {
                const uint32_t t = t0 + q * kWave + lane;
                if (t < len) {
                    if (kSorted) keys[e + t] = ((r + p[q]) << 32) | x[q];
                    else out_ids[e + t] = x[q];
                }
            }
        }
        e += len;
    }
}

// ---------------------------------------------------------------------------
// sorting every list of a decoded batch (relabeled graphs: the lists come in
// label order), in place
// ---------------------------------------------------------------------------
//
// A list's IDs are distinct.  Up to kSortWave of them sort in a wave's
// registers; up to kSortMid in a workgroup's LDS; a longer list by marking
// its IDs in a bitmap of one range of 2^20 IDs at a time and reading the
// marks back.  (One radix sort of all (list, ID) pairs took seven passes over
// 8-byte keys: 1.1 of 1.6 ms for 256,000 lists of a 2^22-vertex graph; now
// 0.32 ms.)
constexpr uint32_t kSortWave = 1024;
constexpr uint32_t kSortMid = 8192;
constexpr uint32_t kSortRangeBits = 20;  // a range's bitmap: 128 KB
// every range of a long list reads the whole list, a workgroup each: up to
// here it is far ahead of the radix sort (one list of 2^23 IDs in 16 ranges 4.3
// ms, by the radix sort 101; 2^20 IDs in 2 ranges 1.5 against 8); beyond it the
// radix sort stays, unmeasured
constexpr uint32_t kSortMaxRanges = 16;

// Bitonic sort of up to 64 kR values in a wave: element e of lane e mod 64,
// register e / 64.
template <int kR>
__device__ __forceinline__ void wave_sort(uint32_t *__restrict__ ids, uint32_t d) {
    const uint32_t lane = lane_id();
    uint32_t x[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) x[r] = r * kWave + lane < d ? ids[r * kWave + lane] : 0xFFFFFFFFu;
#pragma unroll
    for (uint32_t size = 2; size <= 64u * kR; size <<= 1) {
#pragma unroll
        for (uint32_t j = size / 2; j; j >>= 1) {
            if (j >= (uint32_t)kWave) {
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    const int q = r ^ (int)(j / kWave);
                    if (q < r) continue;
                    const bool up = (r * kWave & size) == 0 || size == 64u * kR;
                    const uint32_t lo = x[r] < x[q] ? x[r] : x[q], hi = x[r] < x[q] ? x[q] : x[r];
                    x[r] = up ? lo : hi;
                    x[q] = up ? hi : lo;
                }
            } else {
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    const uint32_t y = __shfl_xor(x[r], j, kWave);
                    const bool low = (lane & j) == 0, up = ((r * kWave + lane) & size) == 0 || size == 64u * kR;
                    x[r] = (low == up) ? (x[r] < y ? x[r] : y) : (x[r] < y ? y : x[r]);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kR; ++r)
        if (r * kWave + lane < d) ids[r * kWave + lane] = x[r];
}

// lists of up to kSortWave entries, 64 lists a workgroup; longer ones go to
// `more`: the middle ones from its front, the long ones from its end
__global__ __launch_bounds__(256) void dec_sort_wave_kernel(uint32_t k, const uint64_t *__restrict__ out_off,
                                                            uint32_t *__restrict__ ids, uint32_t *__restrict__ more,
                                                            DecodeMarks *__restrict__ marks) {
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kWave; i0 < k; i0 += (uint64_t)gridDim.x * kWave) {
        const uint64_t i = i0 + lane;
        const uint64_t o = out_off[i < k ? i : k], d = out_off[i < k ? i + 1 : k] - o;
        if (wv == 0) {
            const bool mid = d > kSortWave && d <= kSortMid, large = d > kSortMid;
            const uint64_t ms = __ballot(mid), ls = __ballot(large);
            uint32_t m0 = 0, l0 = 0;
            if (lane == 0 && ms) m0 = atomicAdd(&marks->n_mid, (uint32_t)__popcll(ms));
            if (lane == 0 && ls) l0 = atomicAdd(&marks->n_long, (uint32_t)__popcll(ls));
            m0 = __shfl(m0, 0, kWave) + popc_below(ms);
            l0 = __shfl(l0, 0, kWave) + popc_below(ls);
            if (mid) more[m0] = (uint32_t)i;
            if (large) more[k - 1 - l0] = (uint32_t)i;
        }
        // the waves take turns over the lists to sort
        uint64_t todo = __ballot(d > 1 && d <= kSortWave);
        for (uint32_t turn = 0; todo; ++turn, todo &= todo - 1) {
            if ((turn & 3u) != wv) continue;
            const uint32_t t = (uint32_t)__ffsll((long long)todo) - 1;
            uint32_t *list = ids + __shfl(o, t, kWave);
            const uint32_t len = __builtin_amdgcn_readfirstlane((uint32_t)__shfl(d, t, kWave));
            if (len <= 64) wave_sort<1>(list, len);
            else if (len <= 128) wave_sort<2>(list, len);
            else if (len <= 256) wave_sort<4>(list, len);
            else if (len <= 512) wave_sort<8>(list, len);
            else wave_sort<16>(list, len);
        }
    }
}

__global__ __launch_bounds__(1024) void dec_sort_mid_kernel(const uint64_t *__restrict__ out_off,
                                                            uint32_t *__restrict__ ids,
                                                            const uint32_t *__restrict__ more,
                                                            const DecodeMarks *__restrict__ marks) {
    __shared__ uint32_t s_x[kSortMid];
    const uint32_t lists = marks->n_mid;
    for (uint32_t l = blockIdx.x; l < lists; l += gridDim.x) {
        const uint32_t i = more[l];
        const uint64_t o = out_off[i];
        const uint32_t d = (uint32_t)(out_off[i + 1] - o);
        uint32_t top = 2 * kSortWave;
        while (top < d) top <<= 1;
        for (uint32_t e = threadIdx.x; e < top; e += 1024) s_x[e] = e < d ? ids[o + e] : 0xFFFFFFFFu;
        for (uint32_t size = 2; size <= top; size <<= 1) {
            for (uint32_t j = size / 2; j; j >>= 1) {
                __syncthreads();
                for (uint32_t t = threadIdx.x; t < top / 2; t += 1024) {
                    const uint32_t a = 2 * t - (t & (j - 1)), b = a + j;
                    const uint32_t x = s_x[a], y = s_x[b];
                    if ((x > y) == ((a & size) == 0 || size == top)) {
                        s_x[a] = y;
                        s_x[b] = x;
                    }
                }
            }
        }
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < d; e += 1024) ids[o + e] = s_x[e];
        __syncthreads();  // the next list takes the buffer
    }
}

// one range of one long list per workgroup step: its IDs in order to `sorted`
__global__ __launch_bounds__(1024) void dec_sort_long_kernel(uint32_t k, uint32_t ranges,
                                                             const uint64_t *__restrict__ out_off,
                                                             const uint32_t *__restrict__ ids,
                                                             const uint32_t *__restrict__ more,
                                                             const DecodeMarks *__restrict__ marks,
                                                             uint32_t *__restrict__ sorted) {
    constexpr uint32_t kWords = 1u << (kSortRangeBits - 5), kPer = kWords / 1024;
    // word w sits at w + w / 32: a thread's 32 words then start on its own bank
    __shared__ uint32_t s_bits[kWords + kWords / 32];
    __shared__ uint32_t s_wave[16], s_below;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const uint64_t items = (uint64_t)marks->n_long * ranges;
    for (uint64_t l = blockIdx.x; l < items; l += gridDim.x) {
        const uint32_t i = more[k - 1 - (uint32_t)(l / ranges)], range = (uint32_t)(l % ranges);
        const uint64_t o = out_off[i];
        const uint32_t d = (uint32_t)(out_off[i + 1] - o);
        for (uint32_t w = tid; w < kWords + kWords / 32; w += 1024) s_bits[w] = 0;
        if (tid == 0) s_below = 0;
        __syncthreads();
        uint32_t below = 0;
#pragma unroll 4
        for (uint32_t e = tid; e < d; e += 1024) {
            const uint32_t u = ids[o + e], r = u >> kSortRangeBits;
            const uint32_t w = (u & ((1u << kSortRangeBits) - 1u)) >> 5;
            if (r == range) atomicOr(&s_bits[w + w / 32], 1u << (u & 31));
            below += r < range;
        }
        below = wave_sum(below);
        if (lane == 0 && below) atomicAdd(&s_below, below);
        __syncthreads();
        uint32_t mine = 0;
        for (uint32_t j = 0; j < kPer; ++j) mine += (uint32_t)__popc(s_bits[tid * (kPer + 1) + j]);
        const uint32_t incl = wave_incl_scan(mine);
        if (lane == kWave - 1) s_wave[wv] = incl;
        __syncthreads();
        uint64_t at = o + s_below + incl - mine;
        for (uint32_t w = 0; w < wv; ++w) at += s_wave[w];
        for (uint32_t j = 0; j < kPer; ++j) {
            const uint32_t id0 = (range << kSortRangeBits) + (tid * kPer + j) * 32;
            for (uint32_t x = s_bits[tid * (kPer + 1) + j]; x; x &= x - 1)
                sorted[at++] = id0 + (uint32_t)__ffs((int)x) - 1;
        }
        __syncthreads();  // the next item clears the bitmap
    }
}

// the long lists back into place, kSortBack workgroups a list
constexpr uint32_t kSortBack = 16;
__global__ void dec_sort_back_kernel(uint32_t k, const uint64_t *__restrict__ out_off,
                                     const uint32_t *__restrict__ sorted, const uint32_t *__restrict__ more,
                                     const DecodeMarks *__restrict__ marks, uint32_t *__restrict__ ids) {
    const uint32_t lists = marks->n_long;
    for (uint32_t l = blockIdx.x / kSortBack; l < lists; l += gridDim.x / kSortBack) {
        const uint32_t i = more[k - 1 - l];
        const uint64_t z = out_off[i + 1];
        for (uint64_t e = out_off[i] + (blockIdx.x % kSortBack) * blockDim.x + threadIdx.x; e < z;
             e += (uint64_t)kSortBack * blockDim.x)
            ids[e] = sorted[e];
    }
}

__global__ void dec_unkey_kernel(uint64_t total, const uint64_t *__restrict__ keys, uint32_t *__restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < total; j += stride)
        out[j] = (uint32_t)keys[j];
}

// How the lists of a sorted request on a relabeled graph are sorted, and the
// temporaries of `total` IDs.
enum class DecodeSort { kLists, kLong, kRadix };  // one by one; with bitmaps for the long ones; all pairs at once
static DecodeSort decode_sort(const lg_graph *g) {
    if (g->max_degree <= kSortMid) return DecodeSort::kLists;
    const uint64_t ranges = ((uint64_t)g->n + (1u << kSortRangeBits) - 1) >> kSortRangeBits;
    return ranges <= kSortMaxRanges ? DecodeSort::kLong : DecodeSort::kRadix;
}
DecodeSortBytes decode_sort_bytes(const lg_graph *g, uint64_t total) {
    switch (decode_sort(g)) {
        case DecodeSort::kLists: return {0, 0, 0, 0, 0};
        case DecodeSort::kLong: return {total * 4, 0, 0, 0, 0};
        default: return {total * 8, total * 8, total * 4, total * 4, radix_sort_tmp_bytes(total)};
    }
}

DecodeWork::~DecodeWork() {
    if (host && host_owned) (void)hipHostFree(host);
}

uint64_t DecodeWork::bytes() const {
    return head.bytes + scan_tmp.bytes + keys.bytes + keys2.bytes + vals.bytes + vals2.bytes + sort_tmp.bytes;
}

// the lists of `labels` to out_ids (kSorted: as sort keys), total > 0
template <class Acc, bool kSorted>
static lg_status dec_lists(const lg_graph *g, Acc acc, const uint32_t *labels, uint32_t k, uint64_t total,
                           const uint64_t *out_off, const uint32_t *perm, uint32_t *out_ids, uint64_t *keys,
                           uint32_t *more, DecodeMarks *marks, hipStream_t stream) {
    if constexpr (IsGapAcc<Acc>::value || IsVarintAcc<Acc>::value) {
        const uint32_t grid = grid_for((uint64_t)k * kWave, 256, 1u << 16);
        if constexpr (IsGapAcc<Acc>::value) {
            // a list that one wave walks longer than the chip takes for the rest
            const uint64_t split = std::max<uint64_t>(g->pr_split, g->m >> kDecGapShare);
            if (g->segs_built && g->n_seg && g->max_degree > split) {
                LG_LAUNCH((dec_lists_kernel<Acc, kSorted, true>), grid, 256, 0, stream, acc, g->n, labels, k,
                          out_off, perm, out_ids, keys, split, more, marks);
                LG_CHECK_LAUNCH();
                LG_LAUNCH((dec_gap_segs_kernel<Acc, kSorted>), 2048, kDecGapThreads, 0, stream, acc, g->n, labels,
                          out_off, perm, out_ids, keys, (const uint32_t *)more, (const DecodeMarks *)marks,
                          g->heavy.as<uint32_t>(), g->n_heavy, g->hstart.as<uint64_t>(), g->hdeg.as<uint32_t>(),
                          g->hw.as<uint32_t>(), g->hg.as<uint32_t>(), g->seg_off.as<uint64_t>(),
                          g->seg_base.as<uint32_t>(), g->seg_size);
            } else
                LG_LAUNCH((dec_lists_kernel<Acc, kSorted, false>), grid, 256, 0, stream, acc, g->n, labels, k,
                          out_off, perm, out_ids, keys, ~0ull, more, marks);
        } else
            LG_LAUNCH((dec_lists_kernel<Acc, kSorted, true>), grid, 256, 0, stream, acc, g->n, labels, k, out_off,
                      perm, out_ids, keys, g->n_vseg ? (uint64_t)g->vseg_split : ~0ull, more, marks);
        if constexpr (IsVarintAcc<Acc>::value) {
            LG_CHECK_LAUNCH();
            if (g->n_vseg)
                LG_LAUNCH((dec_varint_chunks_kernel<Acc, kSorted>), std::min(k, 512u), 1024, 0, stream, acc, g->n,
                          labels, out_off, perm, out_ids, keys, (const uint32_t *)more, (const DecodeMarks *)marks,
                          g->heavy.as<uint32_t>(), g->n_heavy, g->vhb0.as<uint64_t>(), g->vhb1.as<uint64_t>(),
                          g->vseg_off.as<uint64_t>(), g->vseg_base.as<uint32_t>(), g->vseg_bytes);
        }
    } else {
        // pieces of 256 units (one step of the walk) up to 4,096; in
        // between, as many as fill the device twice
        const uint64_t units = total + k;
        uint64_t per = (units / (2 * kDecWaves) + 255) & ~255ull;
        per = per < 256 ? 256 : (per > 4096 ? 4096 : per);
        LG_LAUNCH((dec_walk_kernel<Acc, kSorted>), grid_for((units + per - 1) / per * kWave, 256), 256, 0, stream,
                  acc, labels, k, total, (uint32_t)per, out_off, perm, out_ids, keys);
    }
    LG_CHECK_LAUNCH();
    return LG_OK;
}

lg_status decode_run(lg_graph *g, DecodeWork &w, const uint32_t *vertices, uint32_t k, uint64_t *out_off,
                     uint32_t *out_ids, uint64_t cap, uint32_t flags, hipStream_t stream, uint64_t *total_out) {
    if (total_out) *total_out = 0;
    if (k == 0) return fill_u64(out_off, 0, 1, stream);
    if (!w.host) {
        if (hipHostMalloc((void **)&w.host, 4 * sizeof(uint64_t)) != hipSuccess) {
            w.host = nullptr;
            set_error("lg_decode_neighbors: pinned host allocation failed");
            return LG_ERR_OOM;
        }
    }
    const bool rel = g->relabel != LG_RELABEL_NONE;
    const uint32_t *inv = (rel && flags != LG_DECODE_RAW) ? g->inv.as<uint32_t>() : nullptr;
    const uint32_t *perm = (rel && flags != LG_DECODE_RAW) ? g->perm.as<uint32_t>() : nullptr;
    const bool sorted = rel && flags == LG_DECODE_SORTED;

    // head: labels (k) | degrees (k), later the lists left for other kernels | marks
    LG_TRY(w.head.ensure(decode_head_bytes(k)));
    uint32_t *labels = w.head.as<uint32_t>();
    uint32_t *deg = labels + k;
    DecodeMarks *marks = reinterpret_cast<DecodeMarks *>(deg + k);
    return dispatch_acc_decode(g, [&](auto acc) -> lg_status {
        using Acc = decltype(acc);
        // (a borrowed host slot is ordinary memory, which a kernel cannot write)
        if (w.host_owned && k <= (IsVarintAcc<Acc>::value ? kDecSmall / 16 : kDecSmall)) {
            LG_LAUNCH(dec_small_kernel<Acc>, 1, kDecSmall, 0, stream, acc, g->n, vertices, k, inv, labels, out_off,
                      marks, w.host);
            LG_CHECK_LAUNCH();
        } else {
            LG_TRY(fill_u32(&marks->bad, 0, sizeof(DecodeMarks) / 4, stream));
            LG_LAUNCH(dec_map_kernel<Acc>, grid_for(k, 256, 1u << 16), 256, 0, stream, acc, g->n, vertices, k, inv,
                      labels, deg, marks);
            LG_CHECK_LAUNCH();
            if constexpr (IsVarintAcc<Acc>::value) {
                LG_LAUNCH(dec_varint_degree_kernel<Acc>, grid_for((uint64_t)k * kWave, 256, 1u << 16), 256, 0,
                          stream, acc, labels, k, deg);
                LG_CHECK_LAUNCH();
            }
            LG_TRY(exclusive_scan_u32(deg, out_off, k, w.scan_tmp, stream));
            LG_CHECK_HIP(hipMemcpyAsync(w.host, out_off + k, 8, hipMemcpyDeviceToHost, stream));
            LG_CHECK_HIP(hipMemcpyAsync(w.host + 1, &marks->bad, 4, hipMemcpyDeviceToHost, stream));
        }
        LG_CHECK_HIP(hipStreamSynchronize(stream));
        if (*reinterpret_cast<uint32_t *>(w.host + 1)) {
            set_error("lg_decode_neighbors: vertex id >= n");
            return LG_ERR_INVALID;
        }
        const uint64_t total = w.host[0];
        if (total_out) *total_out = total;
        if (!out_ids || total > cap) {
            set_error("lg_decode_neighbors: %llu ids do not fit in capacity %llu", (unsigned long long)total,
                      (unsigned long long)cap);
            return LG_ERR_CAPACITY;
        }
        if (total == 0) return LG_OK;
        const DecodeSortBytes tmp = sorted ? decode_sort_bytes(g, total) : DecodeSortBytes{};
        if (!sorted || decode_sort(g) != DecodeSort::kRadix) {
            const uint32_t ranges = (uint32_t)(((uint64_t)g->n + (1u << kSortRangeBits) - 1) >> kSortRangeBits);
            const bool has_long = tmp.keys > 0;
            // the fixed scratch of the allocation-free entry point bounds what
            // it sorts, whichever sort that is
            if (sorted && w.keys.borrowed) LG_TRY(w.keys.ensure(total * 8));
            else if (has_long) LG_TRY(w.keys.ensure(tmp.keys));
            LG_TRY((dec_lists<Acc, false>(g, acc, labels, k, total, out_off, perm, out_ids, nullptr, deg, marks,
                                          stream)));
            if (!sorted) return LG_OK;
            LG_LAUNCH(dec_sort_wave_kernel, grid_for(k, kWave, 1u << 14), 256, 0, stream, k,
                      (const uint64_t *)out_off, out_ids, deg, marks);
            LG_CHECK_LAUNCH();
            if (g->max_degree > kSortWave) {
                LG_LAUNCH(dec_sort_mid_kernel, grid_for(k, 1, 1024), 1024, 0, stream, (const uint64_t *)out_off,
                          out_ids, (const uint32_t *)deg, (const DecodeMarks *)marks);
                LG_CHECK_LAUNCH();
            }
            if (has_long) {
                LG_LAUNCH(dec_sort_long_kernel, grid_for((uint64_t)k * ranges, 1, 512), 1024, 0, stream, k, ranges,
                          (const uint64_t *)out_off, (const uint32_t *)out_ids, (const uint32_t *)deg,
                          (const DecodeMarks *)marks, w.keys.as<uint32_t>());
                LG_CHECK_LAUNCH();
                LG_LAUNCH(dec_sort_back_kernel, 1024, 256, 0, stream, k, (const uint64_t *)out_off,
                          (const uint32_t *)w.keys.p, (const uint32_t *)deg, (const DecodeMarks *)marks, out_ids);
                LG_CHECK_LAUNCH();
            }
            return LG_OK;
        }
        LG_TRY(w.keys.ensure(tmp.keys));
        LG_TRY(w.keys2.ensure(tmp.keys2));
        LG_TRY(w.vals.ensure(tmp.vals));
        LG_TRY(w.vals2.ensure(tmp.vals2));
        LG_TRY((dec_lists<Acc, true>(g, acc, labels, k, total, out_off, perm, out_ids, w.keys.as<uint64_t>(), deg,
                                     marks, stream)));
        const uint32_t bits = 32 + bitlen_u64(k - 1);
        LG_TRY(radix_sort_pairs64(w.keys.as<uint64_t>(), w.vals.as<uint32_t>(), w.keys2.as<uint64_t>(),
                                  w.vals2.as<uint32_t>(), total, bits, w.sort_tmp, stream));
        LG_LAUNCH(dec_unkey_kernel, grid_for(total, 256, 1u << 16), 256, 0, stream, total, w.keys.as<uint64_t>(),
                  out_ids);
        LG_CHECK_LAUNCH();
        return LG_OK;
    });
}

}  // namespace lg

static lg_status lg_decode_neighbors_impl(const lg_graph *gc, const uint32_t *vertices, uint32_t k,
                                         uint64_t *out_off, uint32_t *out_ids, uint64_t cap, uint32_t flags,
                                         hipStream_t stream) {
    using namespace lg;
    lg_graph *g = const_cast<lg_graph *>(gc);
    if (!g || !out_off || (k && !vertices)) { set_error("lg_decode_neighbors: NULL argument"); return LG_ERR_INVALID; }
    if (flags > LG_DECODE_RAW) { set_error("lg_decode_neighbors: unknown flags"); return LG_ERR_INVALID; }
    if (!g->dec) {
        g->dec = new (std::nothrow) DecodeWork();
        if (!g->dec) { set_error("lg_decode_neighbors: host allocation failed"); return LG_ERR_OOM; }
    }
    const lg_status st = decode_run(g, *g->dec, vertices, k, out_off, out_ids, cap, flags, stream, nullptr);
    if (st == LG_OK) LG_CHECK_HIP(hipStreamSynchronize(stream));
    return st;
}

extern "C" lg_status lg_decode_neighbors(const lg_graph *gc, const uint32_t *vertices, uint32_t k,
                                         uint64_t *out_off, uint32_t *out_ids, uint64_t cap, uint32_t flags,
                                         hipStream_t stream) {
    const lg_status st = lg_decode_neighbors_impl(gc, vertices, k, out_off, out_ids, cap, flags, stream);
    if (gc && (st == LG_OK || st == LG_ERR_CAPACITY)) LG_TRY(lg::mark_use(const_cast<lg_graph *>(gc), stream));
    return st;
}

// ---------------------------------------------------------------------------
// lg_decode_neighbors_noalloc: the same decode, its temporaries in a fixed
// device array instead of buffers allocated for the graph
// ---------------------------------------------------------------------------

// One copy per GPU, loaded with the library's code object.  In host code this
// name is a stand-in, not a device address: the address on each device comes
// from hipGetSymbolAddress and is the only one passed to kernels.
static __device__ __align__(256) unsigned char scratch[LG_NOALLOC_SCRATCH_BYTES];

namespace lg {
namespace {

constexpr int kNoallocDevices = 64;

struct NoallocDevice {
    std::mutex mu;        // calls on one GPU share its array: one at a time
    void *ptr = nullptr;  // device address of `scratch` on this GPU (set once)
};
NoallocDevice g_noalloc[kNoallocDevices];

inline uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

// byte offsets of the temporaries inside the array, for the largest request
struct NoallocLayout {
    uint64_t head, scan, keys, keys2, vals, vals2, sort, end;
};
NoallocLayout noalloc_layout() {
    NoallocLayout L{};
    uint64_t o = 0;
    L.head = o;  o += align256(decode_head_bytes(LG_NOALLOC_MAX_VERTICES));
    L.scan = o;  o += align256(scan_tmp_bytes(LG_NOALLOC_MAX_VERTICES));
    L.keys = o;  o += align256((uint64_t)LG_NOALLOC_MAX_SORTED_IDS * 8);
    L.keys2 = o; o += align256((uint64_t)LG_NOALLOC_MAX_SORTED_IDS * 8);
    L.vals = o;  o += align256((uint64_t)LG_NOALLOC_MAX_SORTED_IDS * 4);
    L.vals2 = o; o += align256((uint64_t)LG_NOALLOC_MAX_SORTED_IDS * 4);
    L.sort = o;  o += align256(radix_sort_tmp_bytes(LG_NOALLOC_MAX_SORTED_IDS));
    L.end = o;
    return L;
}

}  // namespace
}  // namespace lg

extern "C" lg_status lg_decode_neighbors_noalloc(const lg_graph *gc, const uint32_t *vertices, uint32_t k,
                                                 uint64_t *out_off, uint32_t *out_ids, uint64_t cap,
                                                 uint32_t flags, hipStream_t stream) {
    using namespace lg;
    lg_graph *g = const_cast<lg_graph *>(gc);
    if (!g || !out_off || (k && !vertices)) {
        set_error("lg_decode_neighbors_noalloc: NULL argument");
        return LG_ERR_INVALID;
    }
    if (flags > LG_DECODE_RAW) { set_error("lg_decode_neighbors_noalloc: unknown flags"); return LG_ERR_INVALID; }
    if (k > LG_NOALLOC_MAX_VERTICES) {
        set_error("lg_decode_neighbors_noalloc: %u vertices exceed the limit of %u (LG_NOALLOC_MAX_VERTICES)", k,
                  (unsigned)LG_NOALLOC_MAX_VERTICES);
        return LG_ERR_UNSUPPORTED;
    }
    int dev = 0;
    LG_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNoallocDevices) {
        set_error("lg_decode_neighbors_noalloc: device %d beyond the %d supported", dev, kNoallocDevices);
        return LG_ERR_UNSUPPORTED;
    }
    const NoallocLayout L = noalloc_layout();
    if (L.end > sizeof(scratch)) {
        set_error("lg_decode_neighbors_noalloc: temporaries need %llu bytes, the array holds %llu",
                  (unsigned long long)L.end, (unsigned long long)sizeof(scratch));
        return LG_ERR_UNSUPPORTED;
    }
    NoallocDevice &D = g_noalloc[dev];
    std::lock_guard<std::mutex> hold(D.mu);
    if (!D.ptr) {
        // once per GPU, with that GPU current: this GPU's copy of the array
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error("lg_decode_neighbors_noalloc: hipGetSymbolAddress failed: %s", hipGetErrorString(e));
            return LG_ERR_DEVICE;
        }
        D.ptr = p;
    }
    char *base = static_cast<char *>(D.ptr);
    DecodeWork w;
    w.head.borrow(base + L.head, L.scan - L.head);
    w.scan_tmp.borrow(base + L.scan, L.keys - L.scan);
    w.keys.borrow(base + L.keys, L.keys2 - L.keys);
    w.keys2.borrow(base + L.keys2, L.vals - L.keys2);
    w.vals.borrow(base + L.vals, L.vals2 - L.vals);
    w.vals2.borrow(base + L.vals2, L.sort - L.vals2);
    w.sort_tmp.borrow(base + L.sort, L.end - L.sort);
    uint64_t slots[4] = {0, 0, 0, 0};  // readback into host memory the caller's thread owns
    w.host = slots;
    w.host_owned = false;
    uint64_t total = 0;
    const lg_status st = decode_run(g, w, vertices, k, out_off, out_ids, cap, flags, stream, &total);
    w.host = nullptr;
    // the next call may reuse the array only after this one's kernels ran
    const hipError_t se = hipStreamSynchronize(stream);
    if (st == LG_ERR_UNSUPPORTED && total > LG_NOALLOC_MAX_SORTED_IDS) {
        // the only temporaries whose size depends on the result: the sort keys
        set_error("lg_decode_neighbors_noalloc: sorting %llu ids exceeds the limit of %u "
                  "(LG_NOALLOC_MAX_SORTED_IDS)", (unsigned long long)total, (unsigned)LG_NOALLOC_MAX_SORTED_IDS);
        return st;
    }
    if (st != LG_OK && st != LG_ERR_CAPACITY) return st;
    if (se != hipSuccess) {
        set_error("lg_decode_neighbors_noalloc: hipStreamSynchronize failed: %s", hipGetErrorString(se));
        return LG_ERR_DEVICE;
    }
    LG_TRY(mark_use(g, stream));
    return st;
}
