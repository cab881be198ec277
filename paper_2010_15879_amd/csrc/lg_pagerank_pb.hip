// PageRank by propagation blocking with fixed places (the PR of section
// "Considered Algorithms", same iteration as lg_pagerank.hip).
//
// The pull reads contrib[u] for every stored entry at a random place of a
// 4n-byte array: a 128-byte line per 4-byte gather.  Propagation blocking
// turns the gathers into streams.  A symmetric graph's list of u is also the
// set of vertices whose lists hold u, so sending contrib[u] to every
// neighbour v computes the same sums.  Here every entry's place on the way is
// fixed once per graph, so that an iteration moves nothing but contributions:
//
//   The vertices are cut into source blocks of 2^13 to 2^15 (their
//   contributions fit LDS) and destination bins of 2^8 to 2^14 (their 64-bit
//   sums fit LDS).
//   The entries of (source block, bin) are one tile, in an order fixed by the
//   build, padded to a multiple of four entries (a quad).  Three arrays:
//     src   u16 an entry: the source within its block, block by block
//     val   f32 an entry: its contribution, in the same order
//     dst   u16 an entry: the destination within its bin, bin by bin
//   pb_send_kernel  a workgroup holds a block's contributions in LDS, reads
//                   src and writes val: both streams
//   pb_sum_kernel   a workgroup per bin reads dst as one stream and val as
//                   one run per source block (about 1 KB each), adds in LDS
//                   and finalizes its vertices
//
// 12 bytes an entry and iteration (2 + 4 written, 4 + 2 read back) against
// the 28 of binning (vertex, contribution) pairs twice in every iteration.
//
// The sums are taken in 64-bit fixed point (units of 2^-60) with LDS integer
// atomics: exact whatever the order of the entries, so the scores repeat bit
// for bit and carry no summation error beyond the FP32 rounding of each
// contribution.
#include <algorithm>
#include <new>
#include <type_traits>

#include "lg_device.hpp"

namespace lg {

constexpr uint32_t kMaxSrcShift = 15;   // source block: at most 128 KB of contributions
constexpr uint32_t kMaxFineShift = 14;  // bin: at most 128 KB of sums
constexpr double kFixScale = 1152921504606846976.0;  // 2^60
constexpr double kFixUnit = 1.0 / 1152921504606846976.0;
constexpr double kFixMinBase = 1.0 / 34359738368.0;  // 2^-35
constexpr uint32_t kXcdCount = 8;

// below this many vertices one workgroup does most of either
constexpr uint32_t kPbMinVertices = 1u << 10;
// a build workgroup counts every bin in LDS
constexpr uint32_t kPbMaxVertices = 1u << 28;
// unrelabeled graphs from this size are served whatever the iterations
constexpr uint32_t kPbAlwaysVertices = 1u << 22;
// quads are numbered in 32 bits (entries / 4, and at most one quad of padding
// a tile, of which there are at most 2^27)
constexpr uint64_t kPbMaxEntries = 15ull << 30;

struct PbWork {
    uint32_t ss = 0;        // source block shift
    uint32_t fs = 0;        // bin shift
    uint32_t ns = 0;        // source blocks
    uint32_t nf = 0;        // bins
    uint64_t quads = 0;     // padded entries / 4
    uint32_t n_send = 0, n_sum = 0, n_multi = 0;
    DevBuf deg;             // u32[n]
    DevBuf runs;            // u32[nf * ns + 1] first quad of (bin, block) in dst; u32[nf * ns] the same tile's in src
    DevBuf items;           // uint4[n_send] then uint4[n_sum] then u32[n_multi]
    DevBuf gsum;            // u64[n_multi << fs]: sums of bins shared by several workgroups
    DevBuf buf1;            // val: f32[4 quads]
    DevBuf buf2;            // src, then dst: u16[4 quads] each
    DevBuf ca, cb;          // contribution ping-pong
    bool built = false;
};

uint64_t pb_bytes(const lg_graph *g) {
    if (!g->pb) return 0;
    const PbWork &w = *g->pb;
    return w.deg.bytes + w.runs.bytes + w.items.bytes + w.gsum.bytes + w.buf1.bytes + w.buf2.bytes + w.ca.bytes +
           w.cb.bytes;
}

// The two entry buffers (4 B per stored entry each) outlive their graph in
// one slot per device: the next graph of about the same size takes them
// without an allocation, which at this size can stall for hundreds of
// milliseconds.  lg_free parks them only after the graph's last use, so
// whoever takes them finds them idle; lg_trim frees them.
namespace {
constexpr int kPbSlots = 64;  // devices
struct PbSlot {
    DevBuf buf1, buf2;
};
std::mutex g_pb_slot_mu;
PbSlot *pb_slots() {
    static PbSlot *p = new PbSlot[kPbSlots];  // never destroyed: no frees during static teardown
    return p;
}
}  // namespace

void pb_free(lg_graph *g) {
    if (g->pb && g->pb->built && g->device >= 0 && g->device < kPbSlots) {
        std::lock_guard<std::mutex> lk(g_pb_slot_mu);
        PbSlot &sl = pb_slots()[g->device];
        if (!sl.buf1.p || sl.buf1.bytes < g->pb->buf1.bytes) {  // keep the larger pair
            sl.buf1 = std::move(g->pb->buf1);
            sl.buf2 = std::move(g->pb->buf2);
        }
    }
    delete g->pb;
    g->pb = nullptr;
}

void pb_trim() {
    std::lock_guard<std::mutex> lk(g_pb_slot_mu);
    for (int d = 0; d < kPbSlots; ++d) {
        pb_slots()[d].buf1.release();
        pb_slots()[d].buf2.release();
    }
}

// entry buffers of `bytes` each: the parked pair when it fits (at most a
// quarter larger), else new ones (a parked pair that does not fit is freed
// first, so that its memory is available)
static lg_status pb_take_buffers(lg_graph *g, uint64_t bytes) {
    PbWork &W = *g->pb;
    auto fits = [&](const DevBuf &b) { return b.p && b.bytes >= bytes && b.bytes <= bytes + bytes / 4; };
    if (g->device >= 0 && g->device < kPbSlots) {
        std::lock_guard<std::mutex> lk(g_pb_slot_mu);
        PbSlot &sl = pb_slots()[g->device];
        if (fits(sl.buf1) && fits(sl.buf2)) {
            W.buf1 = std::move(sl.buf1);
            W.buf2 = std::move(sl.buf2);
            return LG_OK;
        }
        sl.buf1.release();
        sl.buf2.release();
    }
    // 1/32 more, so that graphs of the same kind, whose padding differs a
    // little, take each other's
    LG_TRY(W.buf1.alloc(bytes + bytes / 32));
    LG_TRY(W.buf2.alloc(bytes + bytes / 32));
    return LG_OK;
}

// Is propagation blocking the PageRank of this call?  A rule of the graph, the
// damping and the iterations alone (never of timing or of earlier calls), so
// that results do not depend on the run.  Its sums are exact, and it beats the
// pull per iteration 1.5 to 8 times (2^10 to 2^25 vertices, 1 to 24 edges a
// vertex, uniform and Kronecker; uniform Varint lists of a few bytes, which a
// lane reads fast, 0.7 to 1.5 times).
//
// A graph's first call also pays for the build.  Where it meets the pull's,
// in iterations, uniform graphs at means of 2, 8 and 32 entries and Kronecker
// ones, largest over the sizes:
//   one stream of entries   25  9  4,  5     local  29 12  7,  7
//   gap                     38 16  7, 13 (the build decodes the lists first)
//   Varint                  never (2^20 vertices and more: 57 33 7), 16
// (one iteration, uniform, 2^17 vertices, 8 entries: 0.13 ms by the pull, 0.24
// with the build).  Fewer iterations of decoded encodings are left to the pull;
// a line at the crossings would take calls of up to 30 iterations from the
// exact sums and slow down every call but the first up to three times.
static bool pb_always(const lg_graph *g) {
    // Large unrelabeled local IDs among them: the pull's FP32 sums are less
    // accurate (uniform graph, 2^22 vertices, one iteration: largest error
    // 5.5 against 1.7 units of 2^-24; a star of 12 M vertices 441 against 1)
    // and its gathers slower (2^24 vertices: 9.5 ms an iteration against 1.3).
    if (g->relabel != LG_RELABEL_NONE || g->weighted || g->n < kPbAlwaysVertices) return false;
    return g->layout == LG_LAYOUT_PLAIN || g->id_mode == LG_IDS_GLOBAL || g->id_mode == LG_IDS_LOCAL;
}

bool pb_applies(const lg_graph *g, float damping, uint32_t iters) {
    // (a graph that its tables did not fit once keeps to the pull, so that its
    // calls agree whatever else comes and goes in memory)
    if (g->pb_short || g->n < kPbMinVertices || g->n > kPbMaxVertices || g->m >= kPbMaxEntries) return false;
    const bool plain = g->layout == LG_LAYOUT_PLAIN;
    if (!plain && (g->weighted || g->offset_mode == LG_OFFS_INTERLEAVED_BV)) return false;
    if (pb_always(g)) return true;
    // A score is at least the base term (1 - damping) / n, or, where that
    // vanishes, about a first rank's share of the largest list, 1 / (n d).
    // With both below 2^-35 the fixed-point unit, 2^-60, is no longer small
    // beside an FP32 rounding of it (relabeled star of 12 M vertices, damping
    // 1, one iteration: mean error 791 units of 2^-24, by the pull 0.3).
    if (1.0 - (double)damping < (double)g->n * kFixMinBase &&
        (double)g->n * (double)g->max_degree * kFixMinBase > 1.0)
        return false;
    if (plain || g->id_mode == LG_IDS_GLOBAL) return true;
    return iters >= (g->id_mode == LG_IDS_LOCAL || g->id_mode == LG_IDS_LOCAL_GAP ? 6u : 10u);
}

// ---------------------------------------------------------------------------
// the build: once per graph
// ---------------------------------------------------------------------------

// d_v of every vertex (a wave per 64 vertices)
template <class Acc>
__global__ void pb_degree_kernel(Acc acc, uint32_t n, uint32_t *__restrict__ deg) {
    const uint64_t words = ((uint64_t)n + 63) / 64;
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) / kWave;
    for (uint64_t q = wave; q < words; q += nwaves) {
        const VInfo vi = wave_info(acc, q * 64, n);
        const uint64_t v = q * 64 + lane_id();
        if (v < n) deg[v] = vi.deg;
    }
}

__global__ void pb_degree_diff_kernel(uint32_t n, const uint64_t *__restrict__ eoff, uint32_t *__restrict__ deg) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride)
        deg[v] = (uint32_t)(eoff[v + 1] - eoff[v]);
}

__global__ void pb_iota_kernel(uint32_t n, uint32_t *__restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) out[v] = (uint32_t)v;
}

// Entry e of the lists back to back: a fixed-width stream (global IDs) or
// plain 32-bit IDs.
template <bool kPacked>
struct PbEntries {
    const uint32_t *p;
    uint32_t w;
    struct Raw { uint32_t lo, hi, sh; };
    __device__ __forceinline__ Raw load(uint64_t e) const {
        if constexpr (kPacked) {
            const uint64_t bit = e * w, k = bit >> 5;  // the pad word keeps k + 1 in bounds
            return Raw{p[k], p[k + 1], (uint32_t)bit & 31u};
        } else {
            return Raw{p[e], 0u, 0u};
        }
    }
    __device__ __forceinline__ uint32_t value(const Raw &r) const {
        if constexpr (kPacked) return __builtin_amdgcn_alignbit(r.hi, r.lo, r.sh) & width_mask(w);
        else return r.lo;
    }
};

// A part is up to kPbPart consecutive entries of one source block; a
// workgroup takes one: 16 waves of kPbSteps steps of 64 entries.
constexpr uint32_t kPbThreads = 1024;
constexpr uint32_t kPbWaves = kPbThreads / kWave;  // 16
constexpr uint32_t kPbSteps = 16;
constexpr uint32_t kPbPart = kPbThreads * kPbSteps;

// parts of every source block
__global__ void pb_parts_kernel(uint32_t n, uint32_t ns, uint32_t ss, const uint64_t *__restrict__ eoff,
                                uint32_t *__restrict__ parts) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ns) return;
    const uint64_t r0 = (uint64_t)s << ss, r1 = r0 + (1u << ss) < n ? r0 + (1u << ss) : n;
    parts[s] = (uint32_t)((eoff[r1] - eoff[r0] + kPbPart - 1) / kPbPart);
}

__global__ void pb_part_map_kernel(uint32_t ns, const uint64_t *__restrict__ part_off, uint32_t *__restrict__ map) {
    for (uint32_t s = blockIdx.x; s < ns; s += gridDim.x)
        for (uint64_t p = part_off[s] + threadIdx.x; p < part_off[s + 1]; p += blockDim.x) map[p] = s;
}

// Part of block b: the dies take blocks in turn (block b on die b mod 8), and
// the parts of one source block write into the same lines, so every die gets
// one contiguous range of parts.
__device__ __forceinline__ uint32_t pb_part_of(uint32_t b, uint32_t np) {
    const uint32_t q = np / kXcdCount, r = np % kXcdCount, x = b % kXcdCount;
    return x * q + (x < r ? x : r) + b / kXcdCount;
}

// lanes of a wave with equal bins in a row count once: `head` is the first
// lane of this lane's run, `len` the run's lanes
__device__ __forceinline__ void wave_runs(uint32_t bin, uint32_t lane, uint32_t &head, uint32_t &len) {
    const uint32_t prev = __shfl_up(bin, 1, kWave);
    const uint64_t heads = __ballot(lane == 0 || bin != prev);
    head = 63u - (uint32_t)__builtin_clzll(heads & (~0ull >> (63u - lane)));
    const uint64_t after = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    len = (after ? (uint32_t)__builtin_ctzll(after) : 64u) - head;
}

// entries of every part per bin
template <bool kPacked>
__global__ __launch_bounds__(kPbThreads) void pb_count_kernel(PbEntries<kPacked> ent, uint32_t n, uint32_t np,
                                                              const uint64_t *__restrict__ eoff,
                                                              const uint32_t *__restrict__ part_map,
                                                              const uint64_t *__restrict__ part_off, uint32_t ss,
                                                              uint32_t nf, uint32_t fs, uint32_t *__restrict__ pcnt) {
    extern __shared__ uint32_t s_hist[];
    const uint32_t p = pb_part_of(blockIdx.x, np);
    const uint32_t s = part_map[p];
    const uint64_t r0 = (uint64_t)s << ss, r1 = r0 + (1u << ss) < n ? r0 + (1u << ss) : n;
    const uint64_t ea = eoff[r0] + (p - part_off[s]) * kPbPart;
    const uint64_t eb = ea + kPbPart < eoff[r1] ? ea + kPbPart : eoff[r1];
    const uint32_t len = (uint32_t)(eb - ea);
    for (uint32_t b = threadIdx.x; b < nf; b += kPbThreads) s_hist[b] = 0;
    __syncthreads();
    const uint32_t lane = lane_id();
    typename PbEntries<kPacked>::Raw raw[kPbSteps];
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q) {
        const uint32_t x = q * kPbThreads + threadIdx.x;
        raw[q] = ent.load(ea + (x < len ? x : len - 1));
    }
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q) {
        const uint32_t x = q * kPbThreads + threadIdx.x;
        uint32_t v = ent.value(raw[q]);
        v = v < n ? v : n - 1;  // a stored ID is < n; keeps a corrupt stream in bounds
        const uint32_t bin = x < len ? v >> fs : 0xFFFFFFFFu;
        uint32_t head, cnt;
        wave_runs(bin, lane, head, cnt);
        if (head == lane && x < len) atomicAdd(&s_hist[bin], cnt);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < nf; b += kPbThreads) pcnt[(uint64_t)p * nf + b] = s_hist[b];
}

// per tile: the parts' counts become starts within the tile, the total its
// quads (block-major and bin-major).  A workgroup takes 64 bins of a source
// block, its waves a range of the block's parts each: a block of hubs has
// thousands of parts (a thread per tile walking them took 1.4 ms on a
// relabeled Kronecker graph of 2^22 vertices).
constexpr uint32_t kTileWaves = 16;
__global__ __launch_bounds__(kTileWaves *kWave) void pb_tiles_kernel(
    uint32_t ns, uint32_t nf, const uint64_t *__restrict__ part_off, uint32_t *__restrict__ pcnt,
    uint32_t *__restrict__ cnt, uint32_t *__restrict__ tq, uint32_t *__restrict__ tq_bin) {
    __shared__ uint32_t s_sum[kTileWaves][kWave];
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint32_t groups = (nf + kWave - 1) / kWave;
    const uint32_t s = blockIdx.x / groups, b = blockIdx.x % groups * kWave + lane;
    const uint64_t p0 = part_off[s], np = part_off[s + 1] - p0;
    const uint64_t pa = p0 + np * wv / kTileWaves, pz = p0 + np * (wv + 1) / kTileWaves;
    const uint32_t bb = b < nf ? b : nf - 1;
    uint32_t sum = 0;
#pragma unroll 8
    for (uint64_t p = pa; p < pz; ++p) sum += pcnt[p * nf + bb];
    s_sum[wv][lane] = sum;
    __syncthreads();
    uint32_t run = 0, all = 0;
    for (uint32_t w = 0; w < kTileWaves; ++w) {
        if (w < wv) run += s_sum[w][lane];
        all += s_sum[w][lane];
    }
    if (b >= nf) return;
#pragma unroll 8
    for (uint64_t p = pa; p < pz; ++p) {
        const uint32_t c = pcnt[p * nf + b];
        pcnt[p * nf + b] = run;
        run += c;
    }
    if (wv == 0) {
        cnt[(uint64_t)s * nf + b] = all;
        tq[(uint64_t)s * nf + b] = (all + 3) / 4;
        tq_bin[(uint64_t)b * ns + s] = (all + 3) / 4;
    }
}

// first quads of every tile: block-major pairs (in src, in dst) for the
// placement, bin-major runs for the iterations, and the padding entries
// (destination 1 << fs: the sums' spare slot)
__global__ void pb_place_tiles_kernel(uint32_t ns, uint32_t nf, uint32_t fs, const uint64_t *__restrict__ sq,
                                      const uint64_t *__restrict__ dq, const uint32_t *__restrict__ cnt,
                                      uint2 *__restrict__ place, uint32_t *__restrict__ run_dst,
                                      uint32_t *__restrict__ run_src, uint16_t *__restrict__ src,
                                      uint16_t *__restrict__ dst) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t cells = (uint64_t)ns * nf;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cells; i += stride) {
        const uint32_t s = (uint32_t)(i / nf), b = (uint32_t)(i % nf);
        const uint64_t j = (uint64_t)b * ns + s;
        const uint32_t a = (uint32_t)sq[i], d = (uint32_t)dq[j];
        place[i] = make_uint2(a, d);
        run_dst[j] = d;
        run_src[j] = a;
        const uint32_t c = cnt[i];
        for (uint32_t k = c; k < (c + 3) / 4 * 4; ++k) {
            src[(uint64_t)a * 4 + k] = 0;
            dst[(uint64_t)d * 4 + k] = (uint16_t)(1u << fs);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) run_dst[cells] = (uint32_t)dq[cells];
}

// the first quad of every source block (in src) and bin (in dst), and the ends
__global__ void pb_firsts_kernel(uint32_t ns, uint32_t nf, const uint64_t *__restrict__ sq,
                                 const uint64_t *__restrict__ dq, uint64_t *__restrict__ out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= ns) out[i] = sq[(uint64_t)i * nf];
    else if (i - ns - 1 <= nf) out[i] = dq[(uint64_t)(i - ns - 1) * ns];
}

// Places a part's entries: the rows of its entries come from marks at the
// rows' first entries (a running maximum over the entries gives each entry
// its row, whatever the list lengths), the entries are counting-sorted by bin
// in LDS, and every bin's run goes to its place in src and dst.  Once per
// graph; bound by the short runs (8 entries, 16 B each, into two arrays):
// uniform graph, 2^25 vertices, 1.07 G entries: 7.5 ms, and 1.7 ms to count.
template <bool kPacked>
__global__ __launch_bounds__(kPbThreads) void pb_place_kernel(PbEntries<kPacked> ent, uint32_t n, uint32_t np,
                                                              const uint64_t *__restrict__ eoff,
                                                              const uint32_t *__restrict__ part_map,
                                                              const uint64_t *__restrict__ part_off, uint32_t ss,
                                                              uint32_t nf, uint32_t fs, const uint32_t *__restrict__ pcnt,
                                                              const uint2 *__restrict__ place, uint32_t group,
                                                              uint16_t *__restrict__ src,
                                                              uint16_t *__restrict__ dst) {
    extern __shared__ uint32_t s_hist[];  // u32[nf + 1]: counts, then starts
    __shared__ uint32_t s_buf[kPbPart];   // row marks (u16), then the entries sorted by bin
    __shared__ uint32_t s_wave[kPbWaves];
    __shared__ uint32_t s_lo;
    uint16_t *s_mark = reinterpret_cast<uint16_t *>(s_buf);
    const uint32_t tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const uint32_t p = pb_part_of(blockIdx.x, np);
    const uint32_t s = part_map[p];
    const uint64_t r0 = (uint64_t)s << ss, r1 = r0 + (1u << ss) < n ? r0 + (1u << ss) : n;
    const uint32_t rows = (uint32_t)(r1 - r0);
    const uint64_t ea = eoff[r0] + (p - part_off[s]) * kPbPart;
    const uint64_t eb = ea + kPbPart < eoff[r1] ? ea + kPbPart : eoff[r1];
    const uint32_t len = (uint32_t)(eb - ea);
    // the entries' loads go out first; slot q of a lane: entry wv * 64 * kPbSteps + q * 64 + lane
    typename PbEntries<kPacked>::Raw raw[kPbSteps];
    const uint32_t x0 = wv * (kWave * kPbSteps) + lane;
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q) {
        const uint32_t x = x0 + q * kWave;
        raw[q] = ent.load(ea + (x < len ? x : len - 1));
    }
    for (uint32_t i = tid; i < kPbPart / 2; i += kPbThreads) s_buf[i] = 0;
    for (uint32_t b = tid; b < nf; b += kPbThreads) s_hist[b] = 0;
    if (tid == 0) s_lo = 0;
    __syncthreads();
    // the row of the first entry: the last one that begins at or before it,
    // from 1,024 probes, then from the rows between two of them
    {
        const uint32_t step = (rows + kPbThreads - 1) / kPbThreads;
        const uint32_t k = tid * step;
        if (k < rows && eoff[r0 + k] <= ea) atomicMax(&s_lo, k);
        __syncthreads();
        const uint32_t lo = s_lo;
        __syncthreads();
        if (tid < step && lo + tid < rows && eoff[r0 + lo + tid] <= ea) atomicMax(&s_lo, lo + tid);
        __syncthreads();
    }
    for (uint32_t k = s_lo + tid; k < rows; k += kPbThreads) {
        const uint64_t a = eoff[r0 + k], z = eoff[r0 + k + 1];
        if (a >= eb) break;
        // rows with entries in the part mark their first one there, with 1 + the row
        if (z > a && z > ea) s_mark[a > ea ? (uint32_t)(a - ea) : 0u] = (uint16_t)(k + 1);
    }
    __syncthreads();
    uint32_t mark[kPbSteps];
    uint32_t top = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q) {
        mark[q] = s_mark[x0 + q * kWave];
        top = mark[q] > top ? mark[q] : top;
    }
    top = wave_max_scan_dpp(top);
    if (lane == kWave - 1) s_wave[wv] = top;
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t w = 0; w < wv; ++w) carry = s_wave[w] > carry ? s_wave[w] : carry;
    carry = __builtin_amdgcn_readfirstlane(carry);
    uint32_t load[kPbSteps], rank[kPbSteps];  // row << 15 | destination; rank << 16 | bin
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q) {
        const uint32_t sc = wave_max_scan_dpp(mark[q]);
        const uint32_t row = (sc > carry ? sc : carry) - 1;
        const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)sc, kWave - 1);
        carry = last > carry ? last : carry;
        uint32_t v = ent.value(raw[q]);
        v = v < n ? v : n - 1;  // a stored ID is < n; keeps a corrupt stream in bounds
        const bool valid = x0 + q * kWave < len;
        const uint32_t bin = valid ? v >> fs : 0xFFFFu;
        load[q] = ((row & ((1u << ss) - 1u)) << 15) | (v & ((1u << fs) - 1u));
        uint32_t head, cnt;
        wave_runs(bin, lane, head, cnt);
        uint32_t at = 0;
        if (head == lane && valid) at = atomicAdd(&s_hist[bin], cnt);
        at = __shfl(at, head, kWave) + lane - head;
        rank[q] = (at << 16) | bin;
    }
    __syncthreads();
    // counts -> starts
    {
        const uint32_t per = (nf + kPbThreads - 1) / kPbThreads;
        const uint32_t b0 = tid * per;
        uint32_t sum = 0;
        for (uint32_t b = b0; b < b0 + per && b < nf; ++b) sum += s_hist[b];
        const uint32_t incl = wave_scan_dpp(sum);
        if (lane == kWave - 1) s_wave[wv] = incl;
        __syncthreads();
        uint32_t base = incl - sum;
        for (uint32_t w = 0; w < wv; ++w) base += s_wave[w];
        for (uint32_t b = b0; b < b0 + per && b < nf; ++b) {
            const uint32_t c = s_hist[b];
            s_hist[b] = base;
            base += c;
        }
        if (tid == 0) s_hist[nf] = len;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kPbSteps; ++q)
        if (x0 + q * kWave < len) s_buf[s_hist[rank[q] & 0xFFFFu] + (rank[q] >> 16)] = load[q];
    __syncthreads();
    // `group` lanes per bin (a power of two near the expected run length)
    const uint32_t gl = tid & (group - 1);
    for (uint32_t b = tid / group; b < nf; b += kPbThreads / group) {
        const uint32_t a = s_hist[b], c = s_hist[b + 1] - a;
        if (!c) continue;
        const uint2 pl = place[(uint64_t)s * nf + b];
        const uint32_t off = pcnt[(uint64_t)p * nf + b];
        const uint64_t sa = (uint64_t)pl.x * 4 + off, da = (uint64_t)pl.y * 4 + off;
        for (uint32_t i = gl; i < c; i += group) {
            const uint32_t e = s_buf[a + i];
            src[sa + i] = (uint16_t)(e >> 15);
            dst[da + i] = (uint16_t)(e & 0x7FFFu);
        }
    }
}

// ---------------------------------------------------------------------------
// one iteration
// ---------------------------------------------------------------------------

// val of quads [item.y, item.z) of source block item.x.  Bound by memory: 2 B
// read and 4 B written an entry, the gathers from LDS (uniform graph, 2^25
// vertices, 1.07 G entries: 6.4 GB in 1.33 ms, 4.8 TB/s, where a large copy
// reaches 5.1).
template <uint32_t kShift, uint32_t kThreads>
__global__ __launch_bounds__(kThreads) void pb_send_kernel(uint32_t n, const uint4 *__restrict__ items,
                                                           const float *__restrict__ cin,
                                                           const uint16_t *__restrict__ src,
                                                           float *__restrict__ val) {
    constexpr uint32_t kSrc = 1u << kShift;
    constexpr uint32_t kCopy = kSrc / 4 / kThreads;
    __shared__ float4 s_x4[kSrc / 4];
    float *s_x = reinterpret_cast<float *>(s_x4);
    const uint4 it = items[blockIdx.x];
    const uint64_t r0 = (uint64_t)it.x << kShift;
    if (r0 + kSrc <= n) {
        const float4 *c4 = reinterpret_cast<const float4 *>(cin + r0);
        float4 t[kCopy];
#pragma unroll
        for (uint32_t k = 0; k < kCopy; ++k) t[k] = c4[k * kThreads + threadIdx.x];
#pragma unroll
        for (uint32_t k = 0; k < kCopy; ++k) s_x4[k * kThreads + threadIdx.x] = t[k];
    } else {
        for (uint32_t i = threadIdx.x; i < kSrc; i += kThreads) s_x[i] = r0 + i < n ? cin[r0 + i] : 0.0f;
    }
    lds_barrier();
    const ushort4 *s4 = reinterpret_cast<const ushort4 *>(src);
    float4 *v4 = reinterpret_cast<float4 *>(val);
    constexpr uint32_t kIn = 4;  // quads in flight per thread
    const uint32_t last = it.z - 1;
    for (uint64_t q = it.y + threadIdx.x; q < it.z; q += kThreads * kIn) {
        ushort4 u[kIn];
#pragma unroll
        for (uint32_t k = 0; k < kIn; ++k) {
            const uint64_t at = q + k * kThreads;
            u[k] = s4[at < it.z ? at : last];
        }
#pragma unroll
        for (uint32_t k = 0; k < kIn; ++k) {
            const uint64_t at = q + k * kThreads;
            const float4 x = make_float4(s_x[u[k].x & (kSrc - 1)], s_x[u[k].y & (kSrc - 1)], s_x[u[k].z & (kSrc - 1)],
                                         s_x[u[k].w & (kSrc - 1)]);
            if (at < it.z) v4[at] = x;
        }
    }
}

// the score and next contribution of a vertex from its sum
__device__ __forceinline__ void pb_finish(uint64_t v, unsigned long long acc, float base, float alpha,
                                          const uint32_t *__restrict__ deg, float *__restrict__ cout,
                                          float *__restrict__ scores, const uint32_t *__restrict__ perm) {
    const double sum = (double)(long long)acc * kFixUnit;
    const float pr = (float)((double)base + (double)alpha * sum);
    const uint32_t d = deg[v];
    if (d) cout[v] = pr / (float)d;  // vertices without edges hold 0 from the start
    if (scores) scores[perm ? perm[v] : v] = pr;
}

// Quads [item.y, item.z) of bin item.x, split over the waves by quads whatever
// the runs' lengths; each quad finds its run among 64 held across the lanes.
// Bound by memory like pb_send_kernel: 6 B read an entry (the same graph: 6.4
// GB in 1.29 ms, 5.0 TB/s; the two kernels 2.6 ms an iteration, binning pairs
// in two levels 7.7 ms).  item.w: the bin's place in gsum when
// several workgroups share it (its vertices are finished by pb_finish_kernel),
// ~0 when this one has all of it.
template <uint32_t kShift, uint32_t kThreads>
__global__ __launch_bounds__(kThreads) void pb_sum_kernel(uint32_t n, uint32_t ns, const uint4 *__restrict__ items,
                                                          const uint32_t *__restrict__ run_dst,
                                                          const uint32_t *__restrict__ run_src,
                                                          const uint16_t *__restrict__ dst,
                                                          const float *__restrict__ val, float base, float alpha,
                                                          const uint32_t *__restrict__ deg, float *__restrict__ cout,
                                                          float *__restrict__ scores,
                                                          const uint32_t *__restrict__ perm,
                                                          unsigned long long *__restrict__ gsum) {
    constexpr uint32_t kFine = 1u << kShift;
    __shared__ unsigned long long s_acc[kFine + 1];  // and a slot for the padding
    const uint4 it = items[blockIdx.x];
    for (uint32_t i = threadIdx.x; i <= kFine; i += kThreads) s_acc[i] = 0ull;
    lds_barrier();
    const uint32_t lane = lane_id(), wv = threadIdx.x / kWave;
    const uint32_t nw = kThreads / kWave;
    const uint32_t all = it.z - it.y;
    // this wave's quads [j, j_end)
    uint32_t j = it.y + (uint32_t)((uint64_t)all * wv / nw);
    const uint32_t j_end = it.y + (uint32_t)((uint64_t)all * (wv + 1) / nw);
    const uint32_t *rd = run_dst + (uint64_t)it.x * ns, *rs = run_src + (uint64_t)it.x * ns;
    if (j < j_end) {
        // the run holding quad j: rd[lo] <= j < rd[hi] (rd[ns] is the next bin's first run)
        uint32_t lo = 0, hi = ns;
        while (hi - lo > 1) {
            const uint32_t step = (hi - lo + kWave - 1) / kWave;
            const uint32_t at = lo + lane * step;
            const uint64_t le = __ballot(at < hi && rd[at < hi ? at : lo] <= j);
            lo += (uint32_t)(__popcll(le) - 1) * step;
            hi = hi - lo > step ? lo + step : hi;
        }
        const ushort4 *d4 = reinterpret_cast<const ushort4 *>(dst);
        const float4 *v4 = reinterpret_cast<const float4 *>(val);
        constexpr uint32_t kIn = 4;  // steps of 64 quads in flight
        for (uint32_t r = lo; j < j_end; r += kWave) {
            // 64 runs at a time, a lane each: their first quads relative to j,
            // and how far val lies from dst
            const uint32_t i = r + lane < ns ? r + lane : ns;
            const uint32_t beg = rd[i];
            const uint32_t next = rd[r + kWave < ns ? r + kWave : ns];
            const uint32_t shift = (i < ns ? rs[i] : 0u) - beg;
            const uint32_t rel = beg <= j ? 0u : beg - j;
            const uint32_t len = (next < j_end ? next : j_end) - j;
            for (uint32_t t0 = 0; t0 < len; t0 += kWave * kIn) {
                float4 x[kIn];
                ushort4 d[kIn];
#pragma unroll
                for (uint32_t k = 0; k < kIn; ++k) {
                    const uint32_t t = t0 + k * kWave + lane;
                    const uint32_t tt = t < len ? t : len - 1;
                    uint32_t p = 0;  // the last run that begins at or before quad tt
#pragma unroll
                    for (uint32_t b = kWave / 2; b; b >>= 1) {
                        const uint32_t f = __shfl(rel, p + b, kWave);
                        if (f <= tt) p += b;
                    }
                    x[k] = v4[(uint32_t)(__shfl(shift, p, kWave) + j + tt)];
                    d[k] = d4[j + tt];
                }
#pragma unroll
                for (uint32_t k = 0; k < kIn; ++k) {
                    if (t0 + k * kWave + lane >= len) continue;
                    // a contribution is in [0, 1]: its fixed-point value fits
                    auto add = [&](uint32_t at, float y) {
                        atomicAdd(&s_acc[at <= kFine ? at : kFine],
                                  (unsigned long long)__double2ll_rn((double)y * kFixScale));
                    };
                    add(d[k].x, x[k].x);
                    add(d[k].y, x[k].y);
                    add(d[k].z, x[k].z);
                    add(d[k].w, x[k].w);
                }
            }
            j += len;
        }
    }
    lds_barrier();
    const uint64_t v0 = (uint64_t)it.x << kShift;
    if (it.w != 0xFFFFFFFFu) {
        unsigned long long *out = gsum + ((uint64_t)it.w << kShift);
        for (uint32_t i = threadIdx.x; i < kFine; i += kThreads)
            if (s_acc[i]) atomicAdd(&out[i], s_acc[i]);
        return;
    }
    for (uint32_t i = threadIdx.x; i < kFine && v0 + i < n; i += kThreads)
        pb_finish(v0 + i, s_acc[i], base, alpha, deg, cout, scores, perm);
}

// vertices of the bins shared by several workgroups; their sums start the
// next iteration at zero
__global__ void pb_finish_kernel(uint32_t n, uint32_t fs, uint32_t n_multi, const uint32_t *__restrict__ multi,
                                 unsigned long long *__restrict__ gsum, float base, float alpha,
                                 const uint32_t *__restrict__ deg, float *__restrict__ cout,
                                 float *__restrict__ scores, const uint32_t *__restrict__ perm) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (uint64_t)n_multi << fs; i += stride) {
        const uint64_t v = ((uint64_t)multi[i >> fs] << fs) + (i & ((1u << fs) - 1u));
        if (v >= n) continue;
        pb_finish(v, gsum[i], base, alpha, deg, cout, scores, perm);
        gsum[i] = 0ull;
    }
}

// contrib_0 = PR_0 / d (0 for vertices without edges)
__global__ void pb_init_kernel(uint32_t n, double inv_n, const uint32_t *__restrict__ deg, float *__restrict__ ca,
                               float *__restrict__ cb) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const uint32_t d = deg[v];
        const float c = d ? (float)(inv_n / (double)d) : 0.0f;
        ca[v] = c;
        cb[v] = c;
    }
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------

template <bool kPacked>
static lg_status pb_build_tiles(lg_graph *g, PbEntries<kPacked> ent, const uint64_t *eoff, hipStream_t s) {
    PbWork &W = *g->pb;
    const uint32_t n = g->n;
    // Blocks and bins as large as LDS allows on large graphs (a tile's run in
    // val is then 256 entries, 1 KB, at 32 entries a vertex); on smaller ones
    // enough bins and send items to give every compute unit several.  20
    // iterations at (ss, fs), ms: relabeled Kronecker 2^16 (13, 8) 0.34, (15,
    // 8) 0.52; 2^20 (14, 9) 1.5, (15, 11) 1.8; 2^22 (14, 12) 7.1, (15, 11) 7.7;
    // uniform 2^22 (14, 12) 7.4, (15, 13) 8.4; 2^24 (14, 13) 26.3, (14, 14)
    // 27.1; 2^25 (15, 14) 50.9, (15, 13) 54.4
    const uint32_t logn = bitlen_u64((uint64_t)n - 1);
    W.ss = logn < 20 ? 13 : (logn < 25 ? 14 : kMaxSrcShift);
    W.fs = logn <= 16 ? 8 : (logn <= 20 ? 9 : (logn < 25 ? std::min(13u, logn - 10) : kMaxFineShift));
    W.ns = (uint32_t)(((uint64_t)n + (1u << W.ss) - 1) >> W.ss);
    W.nf = (uint32_t)(((uint64_t)n + (1u << W.fs) - 1) >> W.fs);
    const uint32_t ns = W.ns, nf = W.nf;
    const uint64_t cells = (uint64_t)ns * nf;
    DevBuf parts, part_off, map, pcnt, cnt, tq, tqb, sq, dq, place, tmp;
    LG_TRY(parts.scratch((uint64_t)ns * 4, s));
    LG_TRY(part_off.scratch(((uint64_t)ns + 1) * 8, s));
    LG_LAUNCH(pb_parts_kernel, grid_for(ns, 256), 256, 0, s, n, ns, W.ss, eoff,
              parts.as<uint32_t>());
    LG_CHECK_LAUNCH();
    LG_TRY(exclusive_scan_u32(parts.as<uint32_t>(), part_off.as<uint64_t>(), ns, tmp, s));
    uint64_t np64 = 0;
    LG_CHECK_HIP(hipMemcpyAsync(&np64, part_off.as<uint64_t>() + ns, 8, hipMemcpyDeviceToHost, s));
    LG_CHECK_HIP(hipStreamSynchronize(s));
    const uint32_t np = (uint32_t)np64;
    LG_TRY(map.scratch(std::max<uint64_t>(np, 1) * 4, s));
    LG_TRY(pcnt.scratch(std::max<uint64_t>(np64 * nf, 1) * 4, s));
    LG_TRY(cnt.scratch(cells * 4, s));
    LG_TRY(tq.scratch(cells * 4, s));
    LG_TRY(tqb.scratch(cells * 4, s));
    LG_TRY(sq.scratch((cells + 1) * 8, s));
    LG_TRY(dq.scratch((cells + 1) * 8, s));
    LG_TRY(place.scratch(cells * 8, s));
    if (np) {
        LG_LAUNCH(pb_part_map_kernel, std::min(ns, 4096u), 256, 0, s, ns, (const uint64_t *)part_off.p,
                  map.as<uint32_t>());
        LG_CHECK_LAUNCH();
        LG_LAUNCH((pb_count_kernel<kPacked>), np, kPbThreads, nf * 4, s, ent, n, np, eoff, (const uint32_t *)map.p,
                  (const uint64_t *)part_off.p, W.ss, nf, W.fs, pcnt.as<uint32_t>());
        LG_CHECK_LAUNCH();
    }
    const uint32_t cgrid = grid_for(cells, 256, 1u << 15);
    LG_LAUNCH(pb_tiles_kernel, ns * ((nf + kWave - 1) / kWave), kTileWaves * kWave, 0, s, ns, nf,
              (const uint64_t *)part_off.p, pcnt.as<uint32_t>(), cnt.as<uint32_t>(), tq.as<uint32_t>(),
              tqb.as<uint32_t>());
    LG_CHECK_LAUNCH();
    LG_TRY(exclusive_scan_u32(tq.as<uint32_t>(), sq.as<uint64_t>(), cells, tmp, s));
    LG_TRY(exclusive_scan_u32(tqb.as<uint32_t>(), dq.as<uint64_t>(), cells, tmp, s));
    // the blocks' and bins' first quads come to the host, which cuts them into
    // work items
    DevBuf firsts;
    LG_TRY(firsts.scratch(((uint64_t)ns + nf + 2) * 8, s));
    LG_LAUNCH(pb_firsts_kernel, grid_for(ns + nf + 2, 256), 256, 0, s, ns, nf, (const uint64_t *)sq.p,
              (const uint64_t *)dq.p, firsts.as<uint64_t>());
    LG_CHECK_LAUNCH();
    std::vector<uint64_t> host((uint64_t)ns + nf + 2);
    LG_CHECK_HIP(hipMemcpyAsync(host.data(), firsts.p, host.size() * 8, hipMemcpyDeviceToHost, s));
    LG_CHECK_HIP(hipStreamSynchronize(s));
    const uint64_t *hs = host.data(), *hb = hs + ns + 1;
    W.quads = hs[ns];
    if (hs[ns] != hb[nf] || W.quads * 4 < g->m || W.quads >= 1ull << 32) {
        set_error("lg_pagerank: propagation-blocking counts %llu, %llu do not fit %llu entries",
                  (unsigned long long)hs[ns], (unsigned long long)hb[nf], (unsigned long long)g->m);
        return LG_ERR_DEVICE;
    }
    LG_TRY(pb_take_buffers(g, std::max<uint64_t>(W.quads, 1) * 16));
    LG_TRY(W.runs.scratch((2 * cells + 1) * 4, s));
    uint16_t *src = W.buf2.as<uint16_t>(), *dst = src + W.quads * 4;
    LG_LAUNCH(pb_place_tiles_kernel, cgrid, 256, 0, s, ns, nf, W.fs, (const uint64_t *)sq.p, (const uint64_t *)dq.p,
              (const uint32_t *)cnt.p, place.as<uint2>(), W.runs.as<uint32_t>(), W.runs.as<uint32_t>() + cells + 1, src,
              dst);
    LG_CHECK_LAUNCH();
    if (np) {
        uint32_t group = 64;
        while (group > 4 && (uint64_t)group * nf > kPbPart) group /= 2;
        LG_LAUNCH((pb_place_kernel<kPacked>), np, kPbThreads, (nf + 1) * 4, s, ent, n, np, eoff,
                  (const uint32_t *)map.p, (const uint64_t *)part_off.p, W.ss, nf, W.fs, (const uint32_t *)pcnt.p,
                  (const uint2 *)place.p, group, src, dst);
        LG_CHECK_LAUNCH();
    }
    // work items
    int cus = 0;
    LG_CHECK_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, g->device));
    cus = std::max(cus, 1);
    std::vector<uint4> items;
    std::vector<uint32_t> multi;
    const uint64_t x1 = std::max<uint64_t>(1u << (W.ss - 1), std::min<uint64_t>(65536, W.quads / ((uint64_t)cus * 8)));
    for (uint32_t k = 0; k < ns; ++k) {
        const uint64_t a = hs[k], len = hs[k + 1] - a, c = (len + x1 - 1) / x1;
        for (uint64_t i = 0; i < c; ++i)
            items.push_back(make_uint4(k, (uint32_t)(a + len * i / c), (uint32_t)(a + len * (i + 1) / c), 0u));
    }
    W.n_send = (uint32_t)items.size();
    // A bin above the others (a hub's) is shared by several workgroups, which
    // add their sums in memory: too many of them wait on each other's atomics
    // there, too few leave the bin running alone.  An eighth of a compute
    // unit's part each, 1,024 quads at least; bins about as long as the mean
    // are not cut, however long (20 iterations: Kronecker 2^18 cut this way
    // 0.60 ms, bins to 1.5 means whole 0.74; uniform 2^22 7.3 ms, all cut 7.9).
    const uint64_t x2 = std::max<uint64_t>(std::max(1024u, 1u << W.fs), W.quads / ((uint64_t)cus * 8));
    const uint64_t mean = W.quads / nf, whole = std::max<uint64_t>(x2 + x2 / 2, mean + mean / 8);
    for (uint32_t k = 0; k < nf; ++k) {
        const uint64_t a = hb[k], len = hb[k + 1] - a, c = len <= whole ? 1 : (len + x2 - 1) / x2;
        for (uint64_t i = 0; i < c; ++i)
            items.push_back(make_uint4(k, (uint32_t)(a + len * i / c), (uint32_t)(a + len * (i + 1) / c),
                                       c > 1 ? (uint32_t)multi.size() : 0xFFFFFFFFu));
        if (c > 1) multi.push_back(k);
    }
    W.n_sum = (uint32_t)items.size() - W.n_send;
    W.n_multi = (uint32_t)multi.size();
    LG_TRY(W.items.scratch(items.size() * sizeof(uint4) + multi.size() * 4 + 4, s));
    if (W.n_multi) LG_TRY(W.gsum.scratch(((uint64_t)W.n_multi << W.fs) * 8, s));
    LG_TRY(W.ca.alloc((uint64_t)n * 4));
    LG_TRY(W.cb.alloc((uint64_t)n * 4));
    LG_CHECK_HIP(hipMemcpyAsync(W.items.p, items.data(), items.size() * sizeof(uint4), hipMemcpyHostToDevice, s));
    if (W.n_multi)
        LG_CHECK_HIP(hipMemcpyAsync(W.items.as<uint4>() + items.size(), multi.data(), multi.size() * 4,
                                    hipMemcpyHostToDevice, s));
    LG_CHECK_HIP(hipStreamSynchronize(s));  // the host's items are copied
    W.built = true;
    return LG_OK;
}

static lg_status pb_build(lg_graph *g, hipStream_t s) {
    PbWork &W = *g->pb;
    const uint32_t n = g->n;
    LG_TRY(W.deg.scratch((uint64_t)n * 4, s));
    DevBuf eoff;
    LG_TRY(eoff.scratch(((uint64_t)n + 1) * 8, s));
    const bool plain = g->layout == LG_LAYOUT_PLAIN;
    if (plain || g->id_mode == LG_IDS_GLOBAL) {
        // the lists back to back are one stream of fixed-width entries
        DevBuf tmp;
        LG_TRY(dispatch_acc(g, [&](auto acc) -> lg_status {
            using Acc = decltype(acc);
            LG_LAUNCH(pb_degree_kernel<Acc>, grid_for(((uint64_t)n + 63) / 64 * kWave, 256, 1u << 16), 256, 0, s, acc,
                      n, W.deg.as<uint32_t>());
            LG_CHECK_LAUNCH();
            return LG_OK;
        }));
        LG_TRY(exclusive_scan_u32(W.deg.as<uint32_t>(), eoff.as<uint64_t>(), n, tmp, s));
        if (plain)
            return pb_build_tiles(g, PbEntries<false>{g->plain_view().col, 32u}, eoff.as<uint64_t>(), s);
        return pb_build_tiles(g, PbEntries<true>{g->packed_view().A32, g->s}, eoff.as<uint64_t>(), s);
    }
    // every other encoding is decoded into plain lists first (dropped after
    // the build)
    DevBuf col, all;
    LG_TRY(col.scratch(std::max<uint64_t>(g->m, 1) * 4, s));
    LG_TRY(all.scratch((uint64_t)n * 4, s));
    LG_LAUNCH(pb_iota_kernel, grid_for(n, 256, 1u << 16), 256, 0, s, n, all.as<uint32_t>());
    LG_CHECK_LAUNCH();
    DecodeWork dec;
    uint64_t slots[4] = {0, 0, 0, 0};
    dec.host = slots;
    dec.host_owned = false;
    LG_TRY(dec.head.scratch(decode_head_bytes(n), s));
    LG_TRY(dec.scan_tmp.scratch(std::max<uint64_t>(scan_tmp_bytes(n), 8), s));
    LG_TRY(decode_run(g, dec, all.as<uint32_t>(), n, eoff.as<uint64_t>(), col.as<uint32_t>(), g->m, LG_DECODE_RAW, s,
                      nullptr));
    LG_LAUNCH(pb_degree_diff_kernel, grid_for(n, 256, 1u << 16), 256, 0, s, n, (const uint64_t *)eoff.p,
              W.deg.as<uint32_t>());
    LG_CHECK_LAUNCH();
    return pb_build_tiles(g, PbEntries<false>{col.as<uint32_t>(), 32u}, eoff.as<uint64_t>(), s);
}

// fn(std::integral_constant<uint32_t, shift>) for the shifts that a build picks
template <uint32_t... kShifts, class Fn>
static lg_status pb_by_shift(uint32_t shift, Fn &&fn) {
    lg_status st = LG_ERR_UNSUPPORTED;
    (void)((shift == kShifts && (st = fn(std::integral_constant<uint32_t, kShifts>{}), true)) || ...);
    return st;
}

lg_status pagerank_pb(lg_graph *g, float damping, uint32_t iters, float *scores, hipStream_t s) {
    if (!g->pb) {
        g->pb = new (std::nothrow) PbWork();
        if (!g->pb) { set_error("lg_pagerank: host allocation failed"); return LG_ERR_OOM; }
    }
    if (!g->pb->built) {
        lg_status st;
        try {
            st = pb_build(g, s);
        } catch (const std::bad_alloc &) {
            set_error("lg_pagerank: host allocation failed");
            st = LG_ERR_OOM;
        }
        if (st != LG_OK) {  // nothing is kept of a build that did not end
            (void)hipStreamSynchronize(s);
            g->pb_short = st == LG_ERR_OOM;
            delete g->pb;
            g->pb = nullptr;
            return st;
        }
    }
    PbWork &W = *g->pb;
    const uint32_t n = g->n;
    const uint32_t *perm = g->relabel != LG_RELABEL_NONE ? g->perm.as<uint32_t>() : nullptr;
    const double nd = (double)n, a = damping, z = g->isolated;
    const uint64_t cells = (uint64_t)W.ns * W.nf;
    const uint32_t *run_dst = W.runs.as<uint32_t>(), *run_src = run_dst + cells + 1;
    const uint16_t *src = W.buf2.as<uint16_t>(), *dst = src + W.quads * 4;
    const uint4 *send = W.items.as<uint4>(), *sum = send + W.n_send;
    const uint32_t *multi = reinterpret_cast<const uint32_t *>(sum + W.n_sum);
    const uint32_t *deg = W.deg.as<uint32_t>();
    float *val = W.buf1.as<float>();
    float *cin = W.ca.as<float>(), *cout = W.cb.as<float>();
    unsigned long long *gsum = W.gsum.as<unsigned long long>();
    LG_LAUNCH(pb_init_kernel, grid_for(n, 256, 1u << 16), 256, 0, s, n, 1.0 / nd, deg, cin, cout);
    LG_CHECK_LAUNCH();
    if (W.n_multi) LG_TRY(fill_u64((uint64_t *)gsum, 0, (uint64_t)W.n_multi << W.fs, s));
    double D = z / nd;
    for (uint32_t t = 0; t < iters; ++t) {
        const double b = (1.0 - a) / nd + a * D / nd;
        const bool last = t + 1 == iters;
        float *sc = last ? scores : (float *)nullptr;
        const uint32_t *pm = last ? perm : (const uint32_t *)nullptr;
        if (W.n_send) {
            LG_TRY((pb_by_shift<13, 14, 15>(W.ss, [&](auto shift) -> lg_status {
                constexpr uint32_t S = decltype(shift)::value, T = S >= 15 ? 1024 : 512;
                LG_LAUNCH((pb_send_kernel<S, T>), W.n_send, T, 0, s, n, send, (const float *)cin, src, val);
                LG_CHECK_LAUNCH();
                return LG_OK;
            })));
        }
        LG_TRY((pb_by_shift<8, 9, 11, 12, 13, 14>(W.fs, [&](auto shift) -> lg_status {
            constexpr uint32_t S = decltype(shift)::value, T = S >= 14 ? 1024 : (S >= 12 ? 512 : 256);
            LG_LAUNCH((pb_sum_kernel<S, T>), W.n_sum, T, 0, s, n, W.ns, sum, run_dst, run_src, dst, (const float *)val,
                      (float)b, (float)a, deg, cout, sc, pm, gsum);
            LG_CHECK_LAUNCH();
            return LG_OK;
        })));
        if (W.n_multi) {
            LG_LAUNCH(pb_finish_kernel, grid_for((uint64_t)W.n_multi << W.fs, 256, 1u << 14), 256, 0, s, n, W.fs,
                      W.n_multi, multi, gsum, (float)b, (float)a, deg, cout, sc, pm);
            LG_CHECK_LAUNCH();
        }
        D = z * b;
        std::swap(cin, cout);
    }
    return LG_OK;
}

}  // namespace lg
