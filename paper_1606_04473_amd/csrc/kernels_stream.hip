// Streaming trial pass over a 16-bit, part-major copy of the YET.
//
// Algorithm 3 reduces, after the per-request fold (o(E) for every catalogue
// event: the per-ELT terms, the combination over ELTs and the occurrence
// terms, which depend on the event alone), to S_t = sum of o(E) over the
// events of trial t, then the aggregate terms.  Most o(E) are zero, so the
// work per streamed event is one question -- is o(E) nonzero, and what is it
// -- answered here entirely from LDS:
//
//  * the catalogue is cut into parts of 2^16 events.  At table creation the
//    YET is copied part-major: for each part one contiguous stream holding,
//    group of G consecutive trials after group, each trial's events of that
//    part in time order, as 16-bit part-relative IDs.  Each group starts on
//    a 16-byte boundary (the gap holds 0xFFFF), and the end of every trial
//    inside its group is kept as a 16-bit offset.  The stream is half the
//    bytes of the 32-bit IDs.
//  * a workgroup (16 waves, one per CU) takes a contiguous run of (part,
//    group) work items.  For its part it builds in LDS a byte per catalogue
//    event -- 0 for o(E) = 0, else 1 + the event's rank among the nonzero
//    events of its 128-event block -- plus the rank of each block's first
//    nonzero event, and copies the part's first nonzero o(E) (in rank order)
//    into the rest of its LDS.  One ID costs one address operation and one
//    LDS byte read.
//  * each wave streams one group (up to 63 trials) in batches of two 16-byte
//    loads per lane, the next batch in flight while this one is tested, and
//    appends the hits in stream order to its LDS queue.  Lane i holds where
//    trial i starts; the queue index of its first hit comes from the
//    per-chunk hit masks.  At the end of the group lane t sums trial t's
//    queued losses in double-double, in queue order, so the result does not
//    depend on timing.
//  * each (part, trial) partial sum is written once (high part FP64, low part
//    FP32); the combine adds a trial's partials in part order, rounds once and
//    applies the aggregate terms.
//  * the backward's histogram (how often each event with o(E) != 0 occurs in
//    the trials inside the aggregate band, and the TVaR weights of the tail
//    trials) is the same kernel instantiated with kAdj: the same test and
//    queue, a drain that counts occurrences in LDS instead of summing losses.
#include <algorithm>
#include <cmath>
#include <vector>

#include "ara_internal.hpp"
#include "scatter.hpp"

namespace ara {

namespace {

constexpr int kQSize = 1 << kStreamShift;       // catalogue events per stream part
constexpr int kChunkIds = 8;                    // 16-bit IDs per 16-byte load
constexpr int64_t kStreamPad = 512;             // readable 0xFFFF IDs after the stream
constexpr int kSuperEvents = 4096;              // events per superblock of the part images
constexpr int kPartSuper = kQSize / kSuperEvents;

__device__ __forceinline__ uint64_t stream_lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// ---------------------------------------------------------------------------
// create-time layout
// ---------------------------------------------------------------------------

// Per (part, group) k = q * NG + g: the end of each of the group's trials
// relative to the group start (slots past the group's trials repeat the
// group's end), and the group's size padded to whole 16-byte chunks (to its
// place in gstart, scanned there next).  Flags a group with more than 65535 IDs
// of one part.  A workgroup per group: its trials' counts, one contiguous piece
// of cnt, go through LDS; a wave then scans a part over its lanes, one trial
// each, and stores the 64 ends at once (a thread per group and part, walking the
// trials, took 72 us for 150000 trials over 31 parts).
__global__ __launch_bounds__(256) void stream_group_kernel(const int32_t* __restrict__ cnt, int64_t N, int P, int G,
                                                           int64_t NG, int64_t first, uint16_t* __restrict__ gend,
                                                           uint32_t* __restrict__ gstart, CreateResult* __restrict__ res) {
    __shared__ int32_t c[kStreamGroupMax * (kMaxStreamParts + 1)];
    const int lane = threadIdx.x & 63;
    const int64_t g = first + blockIdx.x;
    const int n = static_cast<int>(min(static_cast<int64_t>(G), N - g * G));
    const int row = P | 1;                          // odd: a part's counts lie in different banks
    for (int i = threadIdx.x; i < n * P; i += blockDim.x) c[i / P * row + i % P] = cnt[g * G * P + i];
    __syncthreads();
    for (int q = threadIdx.x >> 6; q < P; q += 4) {
        uint32_t run = lane < n ? static_cast<uint32_t>(c[lane * row + q]) : 0u;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = __shfl_up(run, off, 64);
            if (lane >= off) run = run + v < run ? 0xFFFFFF00u : run + v;      // sums past 32 bits stay above 65535
        }
        const int64_t k = static_cast<int64_t>(q) * NG + g;
        gend[k * kStreamGroupSlots + lane] = static_cast<uint16_t>(run < 65535u ? run : 65535u);
        if (lane == 63) {
            if (run > 65535u) atomicOr(&res->flags, kCreateWideGroup);
            gstart[k + q] = (run + kChunkIds - 1) & ~static_cast<uint32_t>(kChunkIds - 1);
        }
    }
}

// per part (one workgroup each): exclusive scan of the padded group sizes, in
// place; flags a part whose stream reaches 2^32 IDs
__global__ __launch_bounds__(1024) void stream_scan_kernel(int64_t NG, uint32_t* __restrict__ gstart,
                                                           CreateResult* __restrict__ res) {
    __shared__ uint64_t tsum[1024];
    const int q = blockIdx.x;
    uint32_t* dst = gstart + static_cast<int64_t>(q) * (NG + 1);
    const int64_t per = (NG + 1023) / 1024;
    const int64_t j0 = static_cast<int64_t>(threadIdx.x) * per;
    uint64_t local = 0;
    for (int64_t j = j0; j < j0 + per && j < NG; ++j) local += dst[j];
    tsum[threadIdx.x] = local;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t add = static_cast<int>(threadIdx.x) >= off ? tsum[threadIdx.x - off] : 0ull;
        __syncthreads();
        tsum[threadIdx.x] += add;
        __syncthreads();
    }
    uint64_t run = tsum[threadIdx.x] - local;
    for (int64_t j = j0; j < j0 + per && j < NG; ++j) {
        const uint32_t size = dst[j];
        dst[j] = static_cast<uint32_t>(run);
        run += size;
    }
    if (threadIdx.x == 1023) {
        const uint64_t total = tsum[1023];
        dst[NG] = static_cast<uint32_t>(total);
        res->stream_ids[q] = static_cast<int64_t>(total);
        if (total >= (uint64_t(1) << 32) - 4096) atomicOr(&res->flags, kCreateWidePart);
    }
}

// Stable scatter of each trial's events into its segments of the part streams, one
// workgroup per `per` consecutive trials of a group.  Their run of every part is
// staged in LDS with the run's place in a 16-byte chunk kept, so the run leaves
// in 16-byte stores but for its first and last chunk, which other units may share
// and which go ID by ID.  A group's last unit ends its segments with 0xFFFF.
// Several workgroups per CU overlap one's loads with another's stores.  A unit past
// the stage is scattered straight to the stream.  The parts' streams follow each
// other: every workgroup sums their lengths, the first one stores the bases and
// the readable 0xFFFF after the last part.
constexpr int kScatterStage16 = 16 * 1024;          // IDs: 32 KB
struct ScatterEnds16 {                              // dynamic LDS: [P][per + 1] IDs of the group's earlier trials
    uint32_t base[kMaxStreamParts];                 // stage index of the group's first ID of a part (mod 2^32)
    uint32_t seg[kMaxStreamParts + 1];              // staged start of each part's run (whole chunks)
    int64_t out[kMaxStreamParts];                   // where a group's part begins in the stream
    int64_t part_base[kMaxStreamParts + 1];
};
template <int kBits>
__global__ __launch_bounds__(kScatterThreads) void stream_scatter_kernel(
    const int64_t* __restrict__ offsets, const uint32_t* __restrict__ ids, int64_t N, int P, int G, int64_t NG, int per,
    int64_t first_unit, int64_t n_units, const CreateResult* __restrict__ res, int64_t* __restrict__ bases,
    const uint32_t* __restrict__ gstart, const uint16_t* __restrict__ gend, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint16_t stage[kScatterStage16];
    __shared__ __attribute__((aligned(16))) int64_t cursors[kScatterWaves][kMaxStreamParts / 2];
    __shared__ ScatterEnds16 sh;
    extern __shared__ uint32_t ends[];
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int units = (G + per - 1) / per;
    const int64_t of_launch = scatter_unit_index(n_units);
    if (of_launch >= n_units || (res->flags & (kCreateWideGroup | kCreateWidePart))) return;   // no ends to go by
    const int64_t unit = first_unit + of_launch;
    const int64_t g = unit / units;
    const int i0 = static_cast<int>(unit - g * units) * per;
    const int n_group = static_cast<int>(min(static_cast<int64_t>(G), N - g * G));
    const int n = min(per, n_group - i0);
    const int row = per + 1;
    if (unit == 0 || n > 0) {
        for (int j = threadIdx.x; n > 0 && j < P * row; j += kScatterThreads) {
            const int q = j / row, i = i0 + min(j - q * row, n);
            ends[j] = i ? gend[(static_cast<int64_t>(q) * NG + g) * kStreamGroupSlots + i - 1] : 0u;
        }
        if (w == 0) {
            int64_t inc = lane < P ? res->stream_ids[lane] : 0;
            for (int off = 1; off < 64; off <<= 1) {
                const int64_t v = __shfl_up(inc, off, 64);
                if (lane >= off) inc += v;
            }
            sh.part_base[lane + 1] = inc;
            if (lane == 0) sh.part_base[0] = 0;
            if (unit == 0 && lane < P) bases[lane + 1] = inc;
            if (unit == 0 && lane == 0) bases[0] = 0;
        }
    }
    __syncthreads();
    if (unit == 0)
        for (int64_t u = threadIdx.x; u < kStreamPad; u += blockDim.x) out[sh.part_base[P] + u] = 0xFFFFu;
    if (n <= 0) return;
    const bool last = i0 + n == n_group;
    if (w == 0) {
        uint32_t len = 0, phase = 0, rel = 0;
        if (lane < P) {
            const int64_t k = static_cast<int64_t>(lane) * (NG + 1) + g;
            const uint32_t start = gstart[k];
            rel = ends[lane * row];
            phase = rel % kChunkIds;
            len = (last ? gstart[k + 1] - start : ends[lane * row + n]) - rel;
            sh.out[lane] = sh.part_base[lane] + start;
        }
        uint32_t inc = len ? (phase + len + kChunkIds - 1) / kChunkIds * kChunkIds : 0u;
        const uint32_t size = inc;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        if (lane < P) {
            sh.seg[lane] = inc - size;
            sh.base[lane] = inc - size + phase - rel;
        }
        if (lane == P - 1) sh.seg[P] = inc;
    }
    __syncthreads();
    const int64_t t0 = g * G + i0;
    if (sh.seg[P] > static_cast<uint32_t>(kScatterStage16)) {
        int64_t* big = reinterpret_cast<int64_t*>(stage) + w * kMaxStreamParts;    // the stage holds the cursors
        const int n_bits = P > 1 ? 32 - __builtin_clz(static_cast<uint32_t>(P - 1)) : 0;
        for (int i = w; i < n; i += kScatterWaves) {
            if (lane < P) big[lane] = sh.out[lane] + ends[lane * row + i];
            __builtin_amdgcn_wave_barrier();
            scatter_trial_direct(ids, offsets[t0 + i], offsets[t0 + i + 1], kStreamShift, n_bits, big, out);
            __builtin_amdgcn_wave_barrier();
        }
        if (last && w == 0 && lane < P) {
            const int64_t k = static_cast<int64_t>(lane) * (NG + 1) + g;
            for (uint32_t u = ends[lane * row + n]; u < gstart[k + 1] - gstart[k]; ++u) out[sh.out[lane] + u] = 0xFFFFu;
        }
        return;
    }
    if (last && w == kScatterWaves - 1 && lane < P) {
        const uint32_t to = sh.base[lane] + ends[lane * row + n];
        for (uint32_t u = to; u % kChunkIds; ++u) stage[u] = 0xFFFFu;
    }
    uint32_t* cur = reinterpret_cast<uint32_t*>(cursors[w]);
    scatter_unit<kBits>(
        offsets, ids, t0, n, kStreamShift, cur, stage,
        [&](int i) {
            if (lane < P) cur[lane] = sh.base[lane] + ends[lane * row + i];
        },
        [](int) {});
    __syncthreads();
    // a run per group of 16, 32 or 64 lanes
    const int lanes = P > 16 ? 16 : (P > 8 ? 32 : 64);
    for (int q = threadIdx.x / lanes; q < P; q += kScatterThreads / lanes) {
        const uint32_t s0 = sh.seg[q], s1 = sh.seg[q + 1];
        const uint32_t from = sh.base[q] + ends[q * row];
        const uint32_t to = last ? s1 : sh.base[q] + ends[q * row + n];
        uint16_t* dst = out + sh.out[q] - static_cast<int32_t>(sh.base[q]);     // of stage index 0
        for (uint32_t u = s0 + (threadIdx.x % lanes) * kChunkIds; u < s1; u += lanes * kChunkIds) {
            if (u >= from && u + kChunkIds <= to) {
                *reinterpret_cast<u32x4*>(dst + u) = *reinterpret_cast<const u32x4*>(stage + u);
            } else {
                for (uint32_t v = max(u, from); v < min(u + kChunkIds, to); ++v) dst[v] = stage[v];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// the pass
// ---------------------------------------------------------------------------

struct StreamPassArgs {
    const uint16_t* ids;
    const int64_t* part_base;
    const uint32_t* gstart;
    const uint16_t* gend;
    const uint8_t* img;             // [layer] part images of the 2^18-event parts
    const uint32_t* sb_count;       // [layer] nonzero o(E) of each 4096-event superblock
    const double* stage;            // [layer][superblock][4096]: its nonzero o(E), packed in event order
    int64_t img_stride, sb_stride;  // from layer to layer, bytes and superblocks
    int P;
    int G;
    int K;                          // kSplit: units per group
    int n_seg;
    int64_t NG;
    int64_t work;                   // of all segments (Seg::w0 and weight)
    double* part_hi;                // per segment [P][trials]
    float* part_lo;
    const uint16_t* pad;            // 16 readable bytes of 0xFFFF
    int n_xcd;
};

// How a wave takes its work: whole groups with one lane per trial in the
// drain, the same with several lanes per trial where that fills the wave, or
// (with those) single units of a group's trials
enum class PassMode { plain, spread, split };

// One layer over one range of trials: its (part, group) items follow the earlier
// segments' in the work list, each counting `weight`.
struct Seg {
    int64_t t_lo, t_hi;
    int64_t g_lo;                   // first group that holds its trials
    int64_t units;                  // groups (kSplit: units) per part
    int64_t w0;                     // work before it
    int64_t part_at;                // its partial sums' place
    int32_t weight;
    int32_t layer;
};
constexpr int kMaxSegs = 32;
struct SegList {
    Seg seg[kMaxSegs];
};

// bit if the lane's condition holds, else 0: one select on the compare's lane
// mask, so the compare that also guards the lane's queue append is not redone
// in inverted form
template <uint32_t kBit>
__device__ __forceinline__ uint32_t lane_select(bool cond) {
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(cond);
    uint32_t r;
    if constexpr (kBit <= 64)                   // an inline constant
        __asm__("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "i"(kBit), "s"(lanes));
    else
        __asm__("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(kBit), "s"(lanes));
    return r;
}

// Inclusive prefix sum over the 64 lanes of a wave: four DPP row shifts, then
// two row broadcasts carry the row totals.
__device__ __forceinline__ uint32_t stream_wave_scan(uint32_t x) {
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x111, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x112, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x114, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x118, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x142, 0xA, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x143, 0xC, 0xF, false));
    return x;
}

// Extra arguments of the backward histogram over the stream.  Lane i of group
// g holds trial g*G + i's class: 0 outside the layer's trials or outside the
// aggregate band, else bit 0, plus bit 1 when its year loss lies above the
// m-th largest (TVaR weight c_eq) or bit 2 when it equals it (weight m - c_gt)
struct StreamAdjArgs {
    const uint8_t* cls;             // [g_hi - g_lo][64]
    uint64_t* w_mean;               // [C] occurrences in trials inside the band
    uint64_t* w_tvar;               // [C] TVaR weights
    const TailStats* tail;
};

// The pass over the stream.  The forward (kAdj false) sums each trial's
// nonzero o(E), part by part.  The backward histogram (kAdj true) runs the
// same test and queue; its drain counts each queued occurrence of a trial
// inside the aggregate band per event, in 32-bit LDS counters indexed by rank
// that go to W_mean when the workgroup leaves the part (ranks past the
// counters, and the TVaR weights of the few tail trials, use global atomics).
// All weights are integers, so the order of the additions does not matter.
//
// The work list covers one or more segments (layers over trial ranges): many
// layers share a launch, so its start and its end and the images are paid once
// per workgroup's share and not once per layer.
//
// gstart_all is a.gstart again, as a restrict-qualified parameter: its loads at
// wave-uniform addresses then go through the scalar unit, so a group's range
// never waits on the vector loads in flight
template <bool kAdj, PassMode kMode>
__global__ __launch_bounds__(1024) void stream_pass_kernel(StreamPassArgs a, SegList segs, StreamAdjArgs adj,
                                                           const uint32_t* __restrict__ gstart_all) {
    constexpr bool kSplit = kMode == PassMode::split, kSpread = kMode != PassMode::plain;
    constexpr int kU = 2;                                     // 16-byte loads per lane per batch
    constexpr uint32_t kBatch = 64 * kChunkIds * kU;          // IDs per batch
    constexpr int kQ = 64 * kChunkIds;                        // 16-bit queue entries per wave: one load's IDs
    constexpr int kInf = 0x3FFFFFFF;
    constexpr int kHeld = 4;                                  // groups' sums held before a store
    // s_waitcnt operand: vector memory count 0, the other counters at their maximum
    constexpr int kWaitVm0 = (0xF << 8) | (0x7 << 4);
    static_assert(kU == 2, "a batch is two loads per lane, each fitting an empty queue");
    // LDS, one block: the rank of each 128-event block's first nonzero event
    // minus one, then the byte map (a byte's offset from the map's start is its
    // event's part-relative ID; that offset fits the LDS instructions' constant
    // field, so a lookup costs no address arithmetic), the 16 hit queues, and
    // then the forward's copy of the part's nonzero o(E), followed by one 0.0
    // that the drain's idle slots read, or the backward's counters.  A part
    // with more nonzero events than LDS holds keeps those of each superblock's
    // first ones (kSbCap); its ranks are positions in the superblocks' 4096-value
    // slots of the stage, so the others are read there directly.  The backward
    // counts such a part in 16-bit halves, the ranks past those in memory
    constexpr uint32_t kMapOff = (kQSize / 128) * 4;
    constexpr uint32_t kQueueOff = kMapOff + kQSize;
    constexpr uint32_t kValOff = kQueueOff + 16 * kQ * 2;
    constexpr int kCap = static_cast<int>((160 * 1024 - kValOff) / 8) - 1;
    constexpr int kCnt = static_cast<int>((160 * 1024 - kValOff) / 4);
    constexpr uint32_t kSbCap = kCap / kPartSuper, kCnt16 = 2 * kCnt;
    static_assert(kValOff % 16 == 0 && kCap > 0 && kMapOff < 65536, "LDS layout");
    constexpr uint32_t kLdsBytes = kAdj ? kValOff + kCnt * 4 : kValOff + (kCap + 1) * 8;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLdsBytes];
    uint32_t* bases = reinterpret_cast<uint32_t*>(lds);
    uint8_t* map = lds + kMapOff;
    double* vals = reinterpret_cast<double*>(lds + kValOff);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + kValOff);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    uint16_t* q = reinterpret_cast<uint16_t*>(lds + kQueueOff) + wv * kQ;
    const int G = a.G;
    TailStats ts{};
    if constexpr (kAdj) ts = *adj.tail;

    // the work list, segment after segment, in a segment the (part, group) items
    // part-major; workgroup b runs on XCD b % n_xcd, and each XCD takes a
    // contiguous share of the work
    const int64_t n_wg = gridDim.x;
    const int64_t per_x = n_wg / a.n_xcd;
    const int64_t l = static_cast<int64_t>(blockIdx.x % a.n_xcd) * per_x + blockIdx.x / a.n_xcd;
    const int64_t w_begin = l * a.work / n_wg, w_end = (l + 1) * a.work / n_wg;

    // the backward's counters to W_mean once every wave is done with the part,
    // in the byte map's event order; the part before the first has none
    int prev_pq = -1;
    bool prev_fits = true;
    auto flush_counts = [&]() {
        __syncthreads();
        const int64_t ebase = static_cast<int64_t>(prev_pq) << kStreamShift;
        for (int e = threadIdx.x; e < kQSize; e += blockDim.x) {
            const uint32_t b = map[e];
            if (!b) continue;
            const uint32_t r = bases[e >> 7] + b;
            if (!prev_fits && r >= kCnt16) continue;
            const uint32_t cv = prev_fits ? cnt[r] : (cnt[r >> 1] >> (16 * (r & 1u))) & 0xFFFFu;
            if (cv) atomicAdd(reinterpret_cast<unsigned long long*>(&adj.w_mean[ebase + e]),
                              static_cast<unsigned long long>(cv));
        }
    };

    for (int sg = 0; sg < (kAdj ? 1 : a.n_seg); ++sg) {       // the backward takes one segment
        const Seg sgm = segs.seg[sg];
        const int64_t NGr = sgm.units;
        // a work position's item in this segment (shared ends of neighbouring shares agree)
        auto item_at = [&](int64_t w) -> int64_t {
            const int64_t d = w - sgm.w0, n = static_cast<int64_t>(a.P) * NGr;
            return d <= 0 ? 0 : (d >= n * sgm.weight ? n : d / sgm.weight);
        };
        int64_t it = item_at(w_begin);
        const int64_t it_end = item_at(w_end);
        const int64_t t_lo = sgm.t_lo, t_hi = sgm.t_hi, g_lo = sgm.g_lo, count = t_hi - t_lo;
        while (it < it_end) {
            if constexpr (kAdj) {
                if (prev_pq >= 0) flush_counts();
            }
            const int pq = static_cast<int>(it / NGr);
            const int64_t seg_end = min(it_end, static_cast<int64_t>(pq + 1) * NGr);
            // groups of the part, or with kSplit units: K per group from g_lo's first
            const int64_t ga = (kSplit ? 0 : g_lo) + (it - static_cast<int64_t>(pq) * NGr);
            const int64_t gb = (kSplit ? 0 : g_lo) + (seg_end - static_cast<int64_t>(pq) * NGr);
            it = seg_end;
            // ---- the LDS image of stream part pq, from its quarter of the part
            // image of a 2^18-event part: bitmap, ranks of 128-event blocks inside
            // their superblock, and the counts and packed losses of its 16
            // superblocks.  Every global load of the bitmap, the ranks and the
            // counts, and then eight losses per lane, are in flight together.
            const uint8_t* gimg = a.img + sgm.layer * a.img_stride + static_cast<int64_t>(pq >> 2) * kImgPartBytes;
            const u64x2* gbm = reinterpret_cast<const u64x2*>(gimg) + (pq & 3) * (kImgWords / 8);
            const uint16_t* gr16 =
                reinterpret_cast<const uint16_t*>(gimg + int64_t(kImgWords) * 8) + (pq & 3) * (kImgRank16 / 4);
            const double* gstage = a.stage + sgm.layer * a.sb_stride * kSuperEvents + static_cast<int64_t>(pq) * kQSize;
            const uint32_t sb_n =
                a.sb_count[sgm.layer * a.sb_stride + static_cast<int64_t>(pq) * kPartSuper + (lane & (kPartSuper - 1))];
            u64x2 words[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) words[k] = gbm[(k * 1024 + static_cast<int>(threadIdx.x)) >> 3];
            const uint32_t r16 = threadIdx.x < kQSize / 128 ? gr16[threadIdx.x] : 0u;
            // ranks of the superblocks' first nonzero events (lane i: superblock i % 16)
            uint32_t sb_end = sb_n;
#pragma unroll
            for (int off = 1; off < kPartSuper; off <<= 1) {
                const uint32_t v = static_cast<uint32_t>(__shfl_up(static_cast<int>(sb_end), off, kPartSuper));
                if ((lane & (kPartSuper - 1)) >= off) sb_end += v;
            }
            const uint32_t sb_start = sb_end - sb_n;
            const uint32_t n_vals = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sb_end), kPartSuper - 1));
            // when every rank fits the LDS copy of the losses (the counters) the
            // drain skips the L2 fallback (the global atomics)
            const bool fits = n_vals <= static_cast<uint32_t>(kAdj ? kCnt : kCap);
            __syncthreads();
            // byte map, 16 events per thread and round, one 16-byte store each: per
            // four events the bits spread to bytes, their inclusive prefix sum, plus
            // the count of the block's earlier events in every byte
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = k * 1024 + static_cast<int>(threadIdx.x);
                const uint32_t sh = (i & 3) * 16;
                const uint64_t w = (i & 4) ? words[k].y : words[k].x;
                uint32_t before = static_cast<uint32_t>(__popcll(w & ((1ull << sh) - 1ull)));
                if (i & 4) before += static_cast<uint32_t>(__popcll(words[k].x));
                const uint32_t bits = static_cast<uint32_t>(w >> sh) & 0xFFFFu;
                uint32_t run = before * 0x01010101u;
                u32x4 out;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const uint32_t one = (((bits >> (4 * b)) & 15u) * 0x00204081u) & 0x01010101u;
                    const uint32_t two = one + (one << 8);
                    const uint32_t sum = two + (two << 16) + run;
                    out[b] = sum & ((one << 8) - one);
                    run = __builtin_amdgcn_perm(sum, sum, 0x03030303u);
                }
                reinterpret_cast<u32x4*>(map)[i] = out;
            }
            if (threadIdx.x < kQSize / 128) {           // two superblocks of 32 blocks per wave
                const int sb = 2 * wv + (lane >> 5);
                const uint32_t s0 = static_cast<uint32_t>(__shfl(static_cast<int>(sb_start), sb));
                bases[threadIdx.x] = (kAdj || fits ? s0 : static_cast<uint32_t>(sb) * kSuperEvents) + r16 - 1u;
            }
            if constexpr (kAdj) {
                for (int k = threadIdx.x; k < kCnt; k += blockDim.x) cnt[k] = 0u;
            } else {
                // wave w copies superblock w's losses
                const uint32_t n0 =
                    fits ? static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sb_start), wv)) : wv * kSbCap;
                const uint32_t nw = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sb_n), wv));
                const uint32_t take = fits || nw < kSbCap ? nw : kSbCap;
                const double* src = gstage + wv * kSuperEvents;
                for (uint32_t j0 = 0; j0 < take; j0 += 64 * 8) {
                    double v[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t j = j0 + k * 64 + lane;
                        v[k] = src[j < take ? j : 0u];
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t j = j0 + k * 64 + lane;
                        if (j < take) vals[n0 + j] = v[k];
                    }
                }
                if (threadIdx.x == 0) vals[kCap] = 0.0;
            }
            __syncthreads();

            // ---- this wave's groups [wa, wb) of the part
            const int64_t n = gb - ga;
            const int64_t wa = ga + wv * n / 16, wb = ga + (wv + 1) * n / 16;
            if constexpr (kAdj) {
                prev_pq = pq;
                prev_fits = fits;
            }
            if (wa >= wb) continue;
            const uint16_t* ids = a.ids + a.part_base[pq];
            const uint32_t* gs = gstart_all + static_cast<int64_t>(pq) * (a.NG + 1);
            const uint16_t* ge = a.gend + static_cast<int64_t>(pq) * a.NG * kStreamGroupSlots;
            double* out_hi = a.part_hi + sgm.part_at + static_cast<int64_t>(pq) * count;
            float* out_lo = a.part_lo + sgm.part_at + static_cast<int64_t>(pq) * count;
            const int64_t ebase = static_cast<int64_t>(pq) << kStreamShift;   // catalogue ID of the part's event 0
            // B, lane i: where trial i of group g starts; lanes >= G: the group's
            // end.  The next group's trial ends are loaded with every batch (every
            // lane loads, lane 0 then drops its value; no value is carried over, so
            // no copy waits on the load) and added to its start when it begins.
            // The backward loads the next group's trial classes alongside.
            auto group_ends = [&](int64_t gg) -> uint32_t {
                return ge[gg * kStreamGroupSlots + (lane == 0 ? 0 : lane - 1)];
            };
            auto starts = [&](uint32_t s0, uint32_t ends) -> uint32_t { return lane == 0 ? s0 : s0 + ends; };
            auto group_class = [&](int64_t gg) -> uint32_t { return adj.cls[(gg - g_lo) * 64 + lane]; };
            // a group's IDs run from its start to the next group's start (its end
            // rounded up to the 8-ID chunk: the same chunks)
            int64_t g = kSplit ? g_lo + wa / a.K : wa;
            uint32_t rs = gs[g];
            uint32_t re = gs[g + 1];
            uint32_t B = starts(rs, group_ends(g));
            uint32_t next_ends = 0;
            uint32_t cls = 0, next_cls = 0;
            if constexpr (kAdj) cls = group_class(g);
            uint32_t c = rs;                            // first ID of the batch (a multiple of 8)
            int tl = 0, th = G;                         // the trials of the group (of the unit) that this wave sums
            int qs = kInf;                              // lane i: queue index of trial i's first hit
            int qn = 0;                                 // queue entries
            double acc_hi = 0.0, acc_lo = 0.0;
            double held_hi[kHeld];
            float held_lo[kHeld];
            int n_held = 0;

            auto load_batch = [&](uint32_t cb, uint32_t end, u32x4* v) {
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint32_t cu = cb + u * 64 * kChunkIds + lane * kChunkIds;
                    const uint16_t* src = cu < end ? ids + cu : a.pad;
                    v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
                }
            };
            // the batch after the one at c: the rest of this group, else the next group's first
            auto load_next = [&](u32x4* v) {
                next_ends = group_ends(g + 1 < wb ? g + 1 : g);
                if constexpr (kAdj) next_cls = group_class(g + 1 < wb ? g + 1 : g);
                if (c + kBatch < re) {
                    load_batch(c + kBatch, re, v);
                } else {
                    const bool more = g + 1 < wb;
                    const uint32_t n_rs = more ? gs[g + 1] : 0u;
                    const uint32_t n_re = more ? gs[g + 2] : 0u;
                    load_batch(n_rs, n_re, v);
                }
            };
            // the queued hits: lane t takes trial t's entries, four at a time.
            // The loads of a step are issued together.
            auto rank = [&](uint32_t e) -> uint32_t {
                // rank among the part's nonzero events: the block's base (minus one)
                // plus the byte, which is 1 + the rank inside the block
                return bases[e >> 7] + map[e];
            };
            // !fits: an entry's index inside its superblock, and the LDS slot of index i < kSbCap
            auto sb_index = [&](uint32_t rk) -> uint32_t { return rk & (kSuperEvents - 1); };
            auto sb_slot = [&](uint32_t rk, uint32_t i) -> uint32_t { return rk / kSuperEvents * kSbCap + i; };
            // The backward with !fits: one occurrence of each event e with `on`, in
            // the 16-bit counter of its rank, past those in memory.  The lane that
            // brings a counter to 2^15 moves that many to memory; a lane that finds
            // it there or above takes its own back and adds it in memory, so a
            // counter never holds more than 2^15 and one for each of the four
            // entries of 1024 lanes.  The pass with losses for 0.97, 0.85 and
            // 0.6 of the events, against 32-bit counters of half as many events and
            // memory for the others: 650 -> 158 us (5.5e7 events, one part), 545 ->
            // 200 us (5e7, eight parts), 270 -> 183 us (4e7, two parts).
            auto count16 = [&](const uint32_t* e, const uint32_t* rk, const bool* on) {
                constexpr int kN = 4;
                uint32_t old[kN];
                bool rare = false;
#pragma unroll
                for (int r2 = 0; r2 < kN; ++r2) {
                    old[r2] = 0;
                    const uint32_t sh = 16 * (rk[r2] & 1u);
                    if (on[r2] && rk[r2] < kCnt16)
                        old[r2] = (atomicAdd(&cnt[rk[r2] >> 1], 1u << sh) >> sh) & 0xFFFFu;
                    else if (on[r2])
                        atomicAdd(reinterpret_cast<unsigned long long*>(&adj.w_mean[ebase + e[r2]]), 1ull);
                    rare |= old[r2] >= 0x7FFFu;
                }
                if (!__ballot(rare)) return;
#pragma unroll
                for (int r2 = 0; r2 < kN; ++r2) {
                    if (old[r2] < 0x7FFFu) continue;
                    const uint32_t moved = old[r2] == 0x7FFFu ? 0x8000u : 1u;
                    atomicSub(&cnt[rk[r2] >> 1], moved << (16 * (rk[r2] & 1u)));
                    atomicAdd(reinterpret_cast<unsigned long long*>(&adj.w_mean[ebase + e[r2]]),
                              static_cast<unsigned long long>(moved));
                }
            };
            // With many hits of few trials in the queue (long trials over few
            // parts, dense layers) one lane per trial leaves most lanes idle: then
            // 2^s lanes take a trial's entries in turn and their sums are merged,
            // s as large as the 64 lanes allow with at least four entries a lane on
            // average.  s depends on the data alone.
            auto drain = [&]() {
                constexpr int kR = 4;
                int lo = __shfl(qs, lane), hi = __shfl(qs, (lane + 1) & 63);
                lo = lo < 0 ? 0 : (lo > qn ? qn : lo);
                hi = hi < 0 ? 0 : (hi > qn ? qn : hi);
                if (lane >= th || (kSplit && lane < tl)) hi = lo;   // lanes without a trial here
                if constexpr (kAdj) {
                    if (!(cls & 1u)) hi = lo;           // outside the aggregate band: no weight
                }
                bool spread_done = false;
                if constexpr (kSpread) {
                const uint64_t act = __ballot(hi > lo);
                const int i0 = act ? __builtin_ctzll(act) : 0;
                const int n_act = act ? 64 - __builtin_clzll(act) - i0 : 1;
                const int lg_act = n_act > 1 ? 32 - __builtin_clz(static_cast<uint32_t>(n_act - 1)) : 0;
                const int lg_qn = qn > 0 ? 31 - __builtin_clz(static_cast<uint32_t>(qn)) : 0;
                const int s = (lg_qn - 2 < 6 ? lg_qn - 2 : 6) - lg_act;
                if (s > 0) {
                    const int per = 1 << s, slot = lane >> s, sub = lane & (per - 1);
                    const int from = (i0 + slot) & 63;
                    const int mlo = __shfl(lo, from), mhi = __shfl(hi, from);
                    const int jend = slot < n_act ? mhi : mlo;
                    if constexpr (kAdj) {
                        const uint32_t mcls = static_cast<uint32_t>(__shfl(static_cast<int>(cls), from));
                        const unsigned long long wt = (mcls & 6u)
                            ? static_cast<unsigned long long>((mcls & 2u) ? ts.c_eq : ts.m - ts.c_gt) : 0ull;
                        for (int j = mlo + sub; j < jend; j += kR * per) {
                            uint32_t e[kR], rk[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) e[r2] = q[j + r2 * per];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) rk[r2] = rank(e[r2]);
                            bool on[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) on[r2] = j + r2 * per < jend;
                            if (fits) {
#pragma unroll
                                for (int r2 = 0; r2 < kR; ++r2)
                                    if (on[r2]) atomicAdd(&cnt[rk[r2]], 1u);
                            } else {
                                count16(e, rk, on);
                            }
                            if (wt) {
#pragma unroll
                                for (int r2 = 0; r2 < kR; ++r2)
                                    if (on[r2])
                                        atomicAdd(reinterpret_cast<unsigned long long*>(&adj.w_tvar[ebase + e[r2]]), wt);
                            }
                        }
                    } else {
                        double h = 0.0, l = 0.0;
                        for (int j = mlo + sub; j < jend; j += kR * per) {
                            // entries past the trial's last read whatever LDS follows
                            // (inside the allocation), then the 0.0 slot
                            uint32_t e[kR], rk[kR];
                            bool valid[kR];
                            double v[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) {
                                valid[r2] = j + r2 * per < jend;
                                e[r2] = q[j + r2 * per];
                            }
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) rk[r2] = rank(e[r2]);
                            if (fits) {
#pragma unroll
                                for (int r2 = 0; r2 < kR; ++r2) v[r2] = vals[valid[r2] ? rk[r2] : kCap];
                            } else {
                                bool spill = false;
#pragma unroll
                                for (int r2 = 0; r2 < kR; ++r2) {
                                    const uint32_t i = sb_index(rk[r2]);
                                    v[r2] = vals[valid[r2] ? sb_slot(rk[r2], min(i, kSbCap - 1)) : kCap];
                                    spill |= valid[r2] && i >= kSbCap;
                                }
                                if (__ballot(spill)) {
#pragma unroll
                                    for (int r2 = 0; r2 < kR; ++r2)
                                        if (valid[r2] && sb_index(rk[r2]) >= kSbCap) v[r2] = gstage[rk[r2]];
                                }
                            }
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) dd_add(h, l, v[r2]);
                        }
                        for (int off = per >> 1; off >= 1; off >>= 1) dd_merge(h, l, shfl_xor_f64(h, off), shfl_xor_f64(l, off));
                        const int back = ((lane - i0) << s) & 63;
                        const double th_hi = shfl_f64(h, back), th_lo = shfl_f64(l, back);
                        if (lane >= i0 && lane < i0 + n_act) dd_merge(acc_hi, acc_lo, th_hi, th_lo);
                    }
                    spread_done = true;
                }
                }
                if (spread_done) {
                } else if constexpr (kAdj) {
                    if (fits) {
                        // every rank has its LDS counter: whole steps unchecked,
                        // then the last one to three entries (their queue reads,
                        // at most two entries past a full queue, stay inside the
                        // allocation)
                        int j = lo;
                        for (; j + kR <= hi; j += kR) {
                            uint32_t e[kR], rk[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) e[r2] = q[j + r2];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) rk[r2] = rank(e[r2]);
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) atomicAdd(&cnt[rk[r2]], 1u);
                        }
                        if (j < hi) {
                            uint32_t e[kR - 1], rk[kR - 1];
#pragma unroll
                            for (int r2 = 0; r2 < kR - 1; ++r2) e[r2] = q[j + r2];
#pragma unroll
                            for (int r2 = 0; r2 < kR - 1; ++r2) rk[r2] = rank(e[r2]);
#pragma unroll
                            for (int r2 = 0; r2 < kR - 1; ++r2)
                                if (j + r2 < hi) atomicAdd(&cnt[rk[r2]], 1u);
                        }
                    } else {
                        for (int j = lo; j < hi; j += kR) {
                            uint32_t e[kR], rk[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) e[r2] = q[j + r2];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) rk[r2] = rank(e[r2]);
                            bool on[kR];
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2) on[r2] = j + r2 < hi;
                            count16(e, rk, on);
                        }
                    }
                    if (cls & 6u) {
                        // a tail trial: its TVaR weight on each of its occurrences
                        const unsigned long long wt = static_cast<unsigned long long>((cls & 2u) ? ts.c_eq : ts.m - ts.c_gt);
                        for (int j = lo; j < hi; ++j)
                            atomicAdd(reinterpret_cast<unsigned long long*>(&adj.w_tvar[ebase + q[j]]), wt);
                    }
                } else if (fits) {
                    // every rank has its value in LDS: whole steps unchecked, then
                    // the last one to three entries, whose idle slots read the 0.0
                    // after the copied losses (their queue reads, at most two entries
                    // past a full queue, stay inside the allocation)
                    int j = lo;
                    for (; j + kR <= hi; j += kR) {
                        uint32_t e[kR];
                        double v[kR];
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) e[r2] = q[j + r2];
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) v[r2] = vals[rank(e[r2])];
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) dd_add(acc_hi, acc_lo, v[r2]);
                    }
                    if (j < hi) {
                        uint32_t e[kR - 1];
                        double v[kR - 1];
#pragma unroll
                        for (int r2 = 0; r2 < kR - 1; ++r2) e[r2] = q[j + r2];
#pragma unroll
                        for (int r2 = 0; r2 < kR - 1; ++r2) v[r2] = vals[j + r2 < hi ? rank(e[r2]) : kCap];
#pragma unroll
                        for (int r2 = 0; r2 < kR - 1; ++r2) dd_add(acc_hi, acc_lo, v[r2]);
                    }
                } else {
                    for (int j = lo; j < hi; j += kR) {
                        // slots past the trial's last entry read whatever LDS follows
                        // (still inside the allocation), then the 0.0 after the copied
                        // losses, whose sum is exact
                        uint32_t e[kR], rk[kR];
                        bool valid[kR];
                        double v[kR];
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) {
                            valid[r2] = j + r2 < hi;
                            e[r2] = q[j + r2];
                        }
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) rk[r2] = rank(e[r2]);
                        // the LDS copy; entries past it then read the value from L2
                        bool spill = false;
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) {
                            const uint32_t i = sb_index(rk[r2]);
                            v[r2] = vals[valid[r2] ? sb_slot(rk[r2], min(i, kSbCap - 1)) : kCap];
                            spill |= valid[r2] && i >= kSbCap;
                        }
                        if (__ballot(spill)) {
#pragma unroll
                            for (int r2 = 0; r2 < kR; ++r2)
                                if (valid[r2] && sb_index(rk[r2]) >= kSbCap) v[r2] = gstage[rk[r2]];
                        }
#pragma unroll
                        for (int r2 = 0; r2 < kR; ++r2) dd_add(acc_hi, acc_lo, v[r2]);
                    }
                }
                qs = qs == kInf ? kInf : qs - qn;
                qn = 0;
                __builtin_amdgcn_wave_barrier();
            };
            // test a batch against the byte map, append its hits to the queue in
            // stream order, and note where each trial's hits start
            auto process = [&](const u32x4* v) {
                // Chunks past the group's end read padding or the next group's IDs;
                // their hits are queued after the group's end boundary (lanes >= G
                // note where it falls), so no trial takes them.
                uint32_t m[kU];                         // bit w: ID w of the lane's chunk is a hit
                bool hit[kU][8];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    uint32_t b[8];
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        b[2 * d] = map[v[u][d] & 0xFFFFu];
                        b[2 * d + 1] = map[v[u][d] >> 16];
                    }
#pragma unroll
                    for (int w = 0; w < 8; ++w) hit[u][w] = b[w] != 0;
                    m[u] = lane_select<1>(hit[u][0]) | lane_select<2>(hit[u][1]) | lane_select<4>(hit[u][2]) |
                           lane_select<8>(hit[u][3]) | lane_select<16>(hit[u][4]) | lane_select<32>(hit[u][5]) |
                           lane_select<64>(hit[u][6]) | lane_select<128>(hit[u][7]);
                }
                // hit counts per chunk, prefix-summed over the wave two chunks at a time
                // (16-bit halves: at most 8 x 64 hits per load)
                uint32_t pre[kU], tot = 0, tot0 = 0;
                {
                    const uint32_t ca = static_cast<uint32_t>(__popc(m[0]));
                    const uint32_t cb = static_cast<uint32_t>(__popc(m[1]));
                    const uint32_t sc = stream_wave_scan(ca | (cb << 16));
                    const uint32_t tt = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sc), 63));
                    pre[0] = (sc & 0xFFFFu) - ca;
                    pre[1] = (tt & 0xFFFFu) + (sc >> 16) - cb;
                    tot0 = tt & 0xFFFFu;
                    tot = tot0 + (tt >> 16);
                }
                // append the hits of load u; `skip` hits of the batch precede the queue's end
                auto append = [&](int u, uint32_t skip) {
                    uint8_t* at = reinterpret_cast<uint8_t*>(q + qn + (pre[u] - skip));   // LDS byte address
#pragma unroll
                    for (int w = 0; w < 8; ++w) {
                        if (hit[u][w]) *reinterpret_cast<uint16_t*>(at) = static_cast<uint16_t>(v[u][w >> 1] >> (16 * (w & 1)));
                        at += hit[u][w] ? 2 : 0;
                    }
                };
                // trial starts at batch positions [from, to): the hits of the chunk
                // before the start's position, plus the chunk's queue offset
                const uint32_t rel = B - c;
                const uint32_t k = rel >> 3;
                const int src = static_cast<int>(k & 63u);
                const uint32_t p0 = static_cast<uint32_t>(__shfl(static_cast<int>((pre[0] << 8) | m[0]), src));
                const uint32_t p1 = static_cast<uint32_t>(__shfl(static_cast<int>((pre[1] << 8) | m[1]), src));
                const uint32_t pk = (k >> 6) == 0 ? p0 : p1;
                const int before = static_cast<int>(pk >> 8) + __popc((pk & 0xFFu) & ((1u << (rel & 7u)) - 1u));
                auto record = [&](uint32_t from, uint32_t to, int skip) {
                    if (B >= c && rel >= from && rel < to) qs = qn + before - skip;
                };
                if (qn + static_cast<int>(tot) > kQ) drain();
                if (tot <= static_cast<uint32_t>(kQ)) {
                    append(0, 0u);
                    append(1, 0u);
                    record(0u, kBatch, 0);
                    qn += static_cast<int>(tot);
                } else {
                    // more hits than the queue holds (dense layers): the first load's
                    // hits, a drain, then the second load's (each fits an empty queue)
                    const uint32_t t0 = tot0;
                    append(0, 0u);
                    record(0u, kBatch / 2, 0);
                    qn += static_cast<int>(t0);
                    drain();
                    append(1, t0);
                    record(kBatch / 2, kBatch, static_cast<int>(t0));
                    qn += static_cast<int>(tot - t0);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            };
            // Partial sums of the last kHeld groups wait in registers and are stored
            // together, then waited for at once: a store pending at the next wait
            // for a batch would make that wait cover every load in flight (stores
            // and loads share one counter and complete in either order), which at
            // every group's end would stall the stream
            auto flush = [&]() {
#pragma unroll
                for (int k = 0; k < kHeld; ++k) {
                    const int64_t t = (g - k) * G + lane;
                    if (k < n_held && lane < G && t >= t_lo && t < t_hi) {
                        out_hi[t - t_lo] = held_hi[k];
                        out_lo[t - t_lo] = held_lo[k];
                    }
                }
                n_held = 0;
                __builtin_amdgcn_s_waitcnt(kWaitVm0);
            };
            // after a batch: advance; at the end of the group drain the queue, hold
            // the partial sums (the forward) and move to the next group (its first
            // batch is in flight).  Returns false after the wave's last group.
            auto step = [&]() -> bool {
                c += kBatch;
                if (c < re) return true;
                drain();
                if constexpr (!kAdj) {
                    // the group's sums join the held results (newest first)
#pragma unroll
                    for (int k = kHeld - 1; k > 0; --k) {
                        held_hi[k] = held_hi[k - 1];
                        held_lo[k] = held_lo[k - 1];
                    }
                    held_hi[0] = acc_hi + acc_lo;          // renormalised: |lo| <= ulp(hi) / 2
                    held_lo[0] = static_cast<float>(acc_lo - (held_hi[0] - acc_hi));
                    ++n_held;
                    if (n_held == kHeld || g + 1 >= wb) flush();
                    acc_hi = 0.0;
                    acc_lo = 0.0;
                }
                qs = kInf;
                if (g + 1 >= wb) return false;
                ++g;
                rs = gs[g];
                re = gs[g + 1];
                B = starts(rs, next_ends);
                if constexpr (kAdj) cls = next_cls;
                c = rs;
                return true;
            };

            // two register buffers in turn, so the next batch's loads stay in
            // flight while this one is tested
            u32x4 bufA[kU], bufB[kU];
            if constexpr (kSplit) {
                // one unit after the other: trials [tl, th) of a group, from the
                // 16-byte chunk that holds the first one's first ID
                for (int64_t u = wa; u < wb; ++u) {
                    g = g_lo + u / a.K;
                    const int k = static_cast<int>(u % a.K);
                    tl = G * k / a.K;
                    th = G * (k + 1) / a.K;
                    if (u > wa && k == 0) {
                        B = starts(gs[g], group_ends(g));
                        if constexpr (kAdj) cls = group_class(g);
                    }
                    c = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B), tl)) & ~7u;
                    re = (static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B), th)) + 7u) & ~7u;
                    qs = kInf;
                    load_batch(c, re, bufA);
                    while (c < re) {
                        load_batch(c + kBatch, re, bufB);
                        process(bufA);
                        c += kBatch;
                        if (c >= re) break;
                        load_batch(c + kBatch, re, bufA);
                        process(bufB);
                        c += kBatch;
                    }
                    drain();
                    if constexpr (!kAdj) {
                        const int64_t t = g * G + lane;
                        if (lane >= tl && lane < th && t >= t_lo && t < t_hi) {
                            const double hi = acc_hi + acc_lo;      // renormalised: |lo| <= ulp(hi) / 2
                            out_hi[t - t_lo] = hi;
                            out_lo[t - t_lo] = static_cast<float>(acc_lo - (hi - acc_hi));
                        }
                        acc_hi = 0.0;
                        acc_lo = 0.0;
                    }
                }
                continue;
            }
            load_batch(c, re, bufA);
            for (;;) {
                load_next(bufB);
                process(bufA);
                if (!step()) break;
                load_next(bufA);
                process(bufB);
                if (!step()) break;
            }
        }
    }
    if constexpr (kAdj) {
        if (prev_pq >= 0) flush_counts();
    }
}

// The trial classes of StreamAdjArgs, one byte per (group, lane) slot, and the
// partials of the aggregate terms: the trials inside the aggregate band (-1 each
// for the retention) and above it (+1 for the limit), counted for the mean and
// with their TVaR weights.  Four slots per thread in flight; one set of device
// atomics per workgroup.
__global__ __launch_bounds__(256) void stream_class_kernel(const double* __restrict__ S, const double* __restrict__ ylt,
                                                           const TailStats* __restrict__ tail, double aggR, double aggL,
                                                           int64_t t_lo, int64_t t_hi, int G, int64_t g_lo,
                                                           int64_t n_slots, uint8_t* __restrict__ cls,
                                                           long long* __restrict__ agg_mean,
                                                           long long* __restrict__ agg_tvar, int copies, int stride_of,
                                                           uint64_t* __restrict__ to_clear, int64_t n_clear) {
    constexpr int kU = 4;
    const TailStats ts = *tail;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n_clear; i += stride) to_clear[i] = 0;
    long long sums[4] = {0, 0, 0, 0};               // mean: retention, limit; TVaR: the same
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i0 < n_slots; i0 += kU * stride) {
        double sv[kU], yv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t i = i0 + u * stride;
            const int lane = static_cast<int>(i & 63);
            const int64_t t = (g_lo + (i >> 6)) * G + lane;
            const bool in = i < n_slots && lane < G && t >= t_lo && t < t_hi;
            sv[u] = in ? S[t - t_lo] : aggR;        // no trial: neither inside nor above
            yv[u] = in ? ylt[t - t_lo] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t i = i0 + u * stride;
            const int lane = static_cast<int>(i & 63);
            const double ta = sv[u] - aggR;
            // year losses are >= 0, so their bit patterns order like their values
            const uint64_t key = __double_as_longlong(yv[u] + 0.0);
            const uint32_t tail_bits = key > ts.v_bits ? 2u : (key == ts.v_bits ? 4u : 0u);
            const long long wt = (tail_bits & 2u) ? ts.c_eq : ((tail_bits & 4u) ? ts.m - ts.c_gt : 0);
            const bool in_band = (ta > 0.0) && (ta < aggL);
            if (in_band) {
                sums[0] -= 1;
                sums[2] -= wt;
            }
            if (ta > aggL) {
                sums[1] += 1;
                sums[3] += wt;
            }
            if (to_clear) {                         // a wave holds a group's 64 trials
                const uint64_t band = __ballot(in_band), above = __ballot(in_band && (tail_bits & 2u)),
                               at = __ballot(in_band && (tail_bits & 4u));
                if (lane < 3 && i < n_slots)
                    reinterpret_cast<uint64_t*>(cls)[(i >> 6) * 4 + lane] = lane == 0 ? band : (lane == 1 ? above : at);
            } else if (i < n_slots) {
                cls[i] = static_cast<uint8_t>(in_band ? 1u | tail_bits : 0u);
            }
        }
    }
    __shared__ long long red[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int off = 32; off >= 1; off >>= 1) sums[q] += __shfl_xor(sums[q], off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = sums[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        long long v = 0;
        for (int w = 0; w < 4; ++w) v += red[w][threadIdx.x];
        long long* to = (threadIdx.x < 2 ? agg_mean : agg_tvar) + (threadIdx.x & 1) +
                        static_cast<int64_t>(blockIdx.x % copies) * stride_of;
        if (v) atomicAdd(reinterpret_cast<unsigned long long*>(to), static_cast<unsigned long long>(v));
    }
}

__global__ __launch_bounds__(256) void stream_combine_kernel(const double* __restrict__ part_hi,
                                                             const float* __restrict__ part_lo, int P, int64_t count,
                                                             double aggR, double aggL,
                                                             const LayerArgs* __restrict__ L_dev,
                                                             double* __restrict__ ylt, double* __restrict__ ylt_too,
                                                             double* __restrict__ S_out) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= count) return;
    if (L_dev) {                                    // terms from device memory (graph replays)
        aggR = L_dev->aggR;
        aggL = L_dev->aggL;
    }
    double hi = 0.0, lo = 0.0;
    for (int p = 0; p < P; ++p)
        dd_merge(hi, lo, part_hi[p * count + k], static_cast<double>(part_lo[p * count + k]));
    const double S = hi + lo;
    const double y = apply_terms(S, aggR, aggL);
    ylt[k] = y;
    if (ylt_too) ylt_too[k] = y;
    if (S_out) S_out[k] = S;
}

// trials per group: enough that the group's IDs fill whole batches of
// 512-ID loads with little left over, given the mean IDs per (trial, part),
// and few enough that a group of long trials over few parts stays within the
// 16-bit trial ends (six standard deviations of Poisson trials): without this
// line such tables had no copy, and 2e6 events over one part took the 32-bit
// pass 1.5 ms instead of 0.02
int choose_group_trials(double lam) {
    int best_g = kStreamGroupMax;
    double best = 1e300;
    for (int g = kStreamGroupMax; g >= 16; --g) {
        const double mean = g * lam, sd = std::sqrt(mean > 0.0 ? mean : 0.0);
        if (g > 16 && mean + 6.0 * sd > 65535.0) continue;
        const double chunks = (mean + 2.5 * sd) / kChunkIds + 1.0;
        const double loads = std::ceil(chunks / 64.0);
        const double cost = (loads * 512.0 * 5.0 + 200.0) / g;
        if (cost < best - 1e-9) {
            best = cost;
            best_g = g;
        }
    }
    return best_g;
}

}  // namespace

int stream_layout_parts(int64_t N, int64_t C) {
    const int64_t P = (C + kQSize - 1) / kQSize;
    return N < 1 || P < 1 || P > kMaxStreamParts ? 0 : static_cast<int>(P);
}

hipError_t plan_stream_layout(const int32_t* cnt, int64_t N, int64_t n_events, int64_t C, CreateResult* res,
                              hipStream_t s, StreamLayout* out) {
    *out = StreamLayout{};
    const int P = stream_layout_parts(N, C);
    if (P == 0) return hipSuccess;                                     // layout not used
    const int G = choose_group_trials(static_cast<double>(n_events) / (static_cast<double>(N) * P));
    const int64_t NG = (N + G - 1) / G;
    const int64_t n_grp = static_cast<int64_t>(P) * NG;
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&out->gend), sizeof(uint16_t) * n_grp * kStreamGroupSlots, s);
    if (e == hipSuccess) e = dev_alloc(reinterpret_cast<void**>(&out->gstart), sizeof(uint32_t) * P * (NG + 1), s);
    if (e == hipSuccess) e = dev_alloc(reinterpret_cast<void**>(&out->part_base), sizeof(int64_t) * (P + 1), s);
    if (e == hipSuccess) {
        e = in_launches(NG, [&](int64_t first, int64_t n) {
            hipLaunchKernelGGL(stream_group_kernel, dim3(static_cast<uint32_t>(n)), dim3(256), 0, s, cnt, N, P, G, NG,
                               first, out->gend, out->gstart, res);
        });
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(stream_scan_kernel, dim3(static_cast<uint32_t>(P)), dim3(1024), 0, s, NG, out->gstart, res);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        free_stream_layout(out, s);
        return e;
    }
    out->P = P;
    out->G = G;
    out->NG = NG;
    return hipSuccess;
}

namespace {
// the scatter into a copy of `length` IDs (or of room for as many)
hipError_t scatter_stream(const int64_t* offsets, const uint32_t* ids, int64_t N, int64_t n_events, int64_t length,
                          const CreateResult* d_res, hipStream_t s, StreamLayout* out) {
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&out->ids), sizeof(uint16_t) * (length + kStreamPad), s);
    if (e == hipSuccess) {
        // units of even size within a group, each part's run up to 14 IDs from whole chunks
        const double lam = static_cast<double>(n_events) / static_cast<double>(N);
        const int fit = scatter_trials(lam, 14.0 * out->P, kScatterStage16, out->G);
        const int units = (out->G + fit - 1) / fit, per = (out->G + units - 1) / units;
        const int64_t n_units = out->NG * ((out->G + per - 1) / per);
        const size_t lds = sizeof(uint32_t) * static_cast<size_t>(out->P) * (per + 1);
        const auto kernel = out->P <= 8 ? stream_scatter_kernel<3>
                                        : (out->P <= 32 ? stream_scatter_kernel<5> : stream_scatter_kernel<6>);
        e = in_launches(n_units, [&](int64_t first, int64_t n) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>((n + kXcds - 1) / kXcds * kXcds)),
                               dim3(kScatterThreads), lds, s, offsets, ids, N, out->P, out->G, out->NG, per, first, n,
                               d_res, out->part_base, out->gstart, out->gend, out->ids);
        });
    }
    if (e != hipSuccess) free_stream_layout(out, s);
    return e;
}
}  // namespace

hipError_t fill_stream_layout(const int64_t* offsets, const uint32_t* ids, int64_t N, int64_t n_events,
                              const CreateResult& res, const CreateResult* d_res, hipStream_t s, StreamLayout* out) {
    if (out->P == 0) return hipSuccess;
    if (res.flags & (kCreateWideGroup | kCreateWidePart)) {     // too large for 16/32-bit offsets: not used
        free_stream_layout(out, s);
        return hipSuccess;
    }
    int64_t length = 0;
    for (int q = 0; q < out->P; ++q) length += res.stream_ids[q];
    const hipError_t e = scatter_stream(offsets, ids, N, n_events, length, d_res, s, out);
    if (e != hipSuccess) return e;
    out->length = length;
    out->bytes = static_cast<int64_t>(sizeof(uint16_t)) * (length + kStreamPad) +
                 static_cast<int64_t>(sizeof(uint16_t)) * out->P * out->NG * kStreamGroupSlots +
                 static_cast<int64_t>(sizeof(uint32_t)) * out->P * (out->NG + 1) +
                 static_cast<int64_t>(sizeof(int64_t)) * (out->P + 1);
    return hipSuccess;
}

hipError_t fill_stream_layout_unread(const int64_t* offsets, const uint32_t* ids, int64_t N, int64_t n_events,
                                     const CreateResult* d_res, hipStream_t s, StreamLayout* out) {
    if (out->P == 0) return hipSuccess;
    // every group of a part starts on a whole chunk
    return scatter_stream(offsets, ids, N, n_events, n_events + (kChunkIds - 1) * out->P * out->NG, d_res, s, out);
}

void free_stream_layout(StreamLayout* L, hipStream_t s) {
    if (L->ids) dev_free(L->ids, s);
    if (L->part_base) dev_free(L->part_base, s);
    if (L->gstart) dev_free(L->gstart, s);
    if (L->gend) dev_free(L->gend, s);
    *L = StreamLayout{};
}

int64_t stream_partials_bytes(const StreamLayout& lay, int64_t trials) {
    const int64_t n = static_cast<int64_t>(lay.P) * (trials > 0 ? trials : 1);
    return static_cast<int64_t>(sizeof(double) + sizeof(float)) * n + 256;
}

const float* stream_partials_lo(const StreamLayout& lay, const void* partials, int64_t trials) {
    return reinterpret_cast<const float*>(static_cast<const double*>(partials) + static_cast<int64_t>(lay.P) * trials);
}

namespace {

// arguments common to a launch; the fold's outputs of the layers lie at `fold`
StreamPassArgs pass_args(const StreamLayout& lay, const FoldViews& fold) {
    StreamPassArgs a{};
    a.ids = lay.ids;
    a.part_base = lay.part_base;
    a.gstart = lay.gstart;
    a.gend = lay.gend;
    a.img = fold.img;
    a.sb_count = fold.sb_count;
    a.stage = fold.stage;
    a.img_stride = fold.img_stride;
    a.sb_stride = fold.sb_stride;
    a.P = lay.P;
    a.G = lay.G;
    a.NG = lay.NG;
    a.pad = lay.ids + lay.length;
    a.n_xcd = kXcds;
    return a;
}

// groups that hold the trials [t_lo, t_hi)
int64_t first_group(const StreamLayout& lay, int64_t t_lo) { return t_lo / lay.G; }
int64_t group_end(const StreamLayout& lay, int64_t t_hi) { return (t_hi + lay.G - 1) / lay.G; }

// one 1024-thread workgroup per CU (its LDS holds the part's byte map and
// values or counters), a multiple of the XCD count
uint32_t pass_grid(int n_cu) {
    int64_t grid = int64_t(n_cu);
    grid -= grid % kXcds;
    if (grid < kXcds) grid = kXcds;
    return static_cast<uint32_t>(grid);
}

// Units per group.  One wave streams a whole group unless the request has so
// few groups that most waves would have none: then each group's trials are
// split into K units.  K minimises the batches that the busiest wave
// processes, a unit of a split group counting half a batch more (it starts
// with its own load of the trial ends and has no batch in flight before).
// 1e6 events in 320 groups: the pass 17 -> 10 us with K = 6.
int units_per_group(const StreamLayout& lay, int64_t groups, int64_t waves) {
    const double ids = static_cast<double>(lay.length) / (static_cast<double>(lay.P) * lay.NG);
    int best_k = 1;
    double best = 1e300;
    for (int k = 1; k <= lay.G && (k == 1 || ids >= 128.0 * k); ++k) {
        const double units = std::ceil(static_cast<double>(groups) * lay.P * k / static_cast<double>(waves));
        const double cost = units * (std::ceil(ids / (1024.0 * k) + 0.25) + (k > 1 ? 0.5 : 0.0));
        if (cost < best - 1e-9) {
            best = cost;
            best_k = k;
        }
        if (units > 8.0) break;                     // enough groups for every wave
    }
    return best_k;
}

// Where a trial has many hits in a part the queue fills before its group's
// end and holds few trials; the drain then spreads them over the lanes.  The
// code for it costs the pass 2-3% where it finds nothing to do (its size: 0.594
// against 0.58 ms per 1e9 events at 4.4 hits per trial and part), and at 17 and
// 52 hits it takes the pass from 23 to 17 us (1e6 events) and from 357 to 150 us
// (5e7), so the line lies at 12.
constexpr double kSpreadHits = 12.0;

// `units` in order, with the partial sums of each after the earlier ones'
template <bool kAdj>
hipError_t launch_pass(const StreamLayout& lay, StreamPassArgs& a, const StreamUnit* units, int n,
                       const StreamAdjArgs& adj, int n_cu, hipStream_t s) {
    if (n < 1 || n > kMaxSegs) return hipErrorInvalidValue;
    const uint32_t grid = pass_grid(n_cu);
    SegList segs{};
    int64_t groups = 0;
    double hits = 0.0;
    for (int i = 0; i < n; ++i) {
        groups += group_end(lay, units[i].t_lo + units[i].count) - first_group(lay, units[i].t_lo);
        hits = std::max(hits, units[i].density);
    }
    hits *= static_cast<double>(lay.length) / (static_cast<double>(lay.P) * lay.NG * lay.G);
    a.K = units_per_group(lay, groups, int64_t(grid) * 16);
    a.n_seg = n;
    int64_t at = 0;
    for (int i = 0; i < n; ++i) {
        Seg& g = segs.seg[i];
        g.t_lo = units[i].t_lo;
        g.t_hi = units[i].t_lo + units[i].count;
        g.g_lo = first_group(lay, g.t_lo);
        g.units = (group_end(lay, g.t_hi) - g.g_lo) * a.K;
        g.w0 = a.work;
        g.part_at = at;
        // a group of a layer with losses for a share d of the events takes about
        // 1 + 2.2 d times a group without (0.50, 0.60 and 0.85 ms per 1e9 events at
        // d = 0.01, 0.15 and 0.27)
        g.weight = static_cast<int32_t>(16.0 * (1.0 + 2.2 * units[i].density) + 0.5);
        g.layer = units[i].layer;
        a.work += static_cast<int64_t>(lay.P) * g.units * g.weight;
        at += static_cast<int64_t>(lay.P) * units[i].count;
    }
    const dim3 g(grid), t(1024);
    if (a.K > 1)
        hipLaunchKernelGGL((stream_pass_kernel<kAdj, PassMode::split>), g, t, 0, s, a, segs, adj, a.gstart);
    else if (hits > kSpreadHits)
        hipLaunchKernelGGL((stream_pass_kernel<kAdj, PassMode::spread>), g, t, 0, s, a, segs, adj, a.gstart);
    else
        hipLaunchKernelGGL((stream_pass_kernel<kAdj, PassMode::plain>), g, t, 0, s, a, segs, adj, a.gstart);
    return hipGetLastError();
}

// partial sums of `trials` trials over all units: the high parts, then the low parts
void place_partials(const StreamLayout& lay, StreamPassArgs& a, void* partials, int64_t trials) {
    a.part_hi = static_cast<double*>(partials);
    a.part_lo = reinterpret_cast<float*>(a.part_hi + static_cast<int64_t>(lay.P) * trials);
}

// the units' partial sums merged, one range of workgroups per unit
struct CombineUnit {
    int64_t first_block, count, part_at, out_at;
    int32_t layer, pad_;
};
struct CombineArgs {
    CombineUnit unit[kMaxSegs];
    int n;
};
__global__ __launch_bounds__(256) void stream_combine_units_kernel(const double* __restrict__ part_hi,
                                                                   const float* __restrict__ part_lo, int P,
                                                                   CombineArgs c, const LayerArgs* __restrict__ L_dev,
                                                                   double* __restrict__ ylt) {
    int i = 0;
    while (i + 1 < c.n && static_cast<int64_t>(blockIdx.x) >= c.unit[i + 1].first_block) ++i;
    const CombineUnit u = c.unit[i];
    const int64_t k = (static_cast<int64_t>(blockIdx.x) - u.first_block) * blockDim.x + threadIdx.x;
    if (k >= u.count) return;
    part_hi += u.part_at;
    part_lo += u.part_at;
    double hi = 0.0, lo = 0.0;
    for (int p = 0; p < P; ++p)
        dd_merge(hi, lo, part_hi[p * u.count + k], static_cast<double>(part_lo[p * u.count + k]));
    ylt[u.out_at + k] = apply_terms(hi + lo, L_dev[u.layer].aggR, L_dev[u.layer].aggL);
}

}  // namespace

hipError_t launch_stream_pass(const StreamLayout& lay, double density, const LayerArgs& L, void* part_scratch,
                              int n_img_parts, void* partials, int n_cu, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    if (lay.P <= 0 || (lay.P - 1) / 4 >= n_img_parts) return hipErrorInvalidValue;
    StreamPassArgs a = pass_args(lay, fold_views(part_scratch, n_img_parts));
    place_partials(lay, a, partials, L.trial_count);
    const StreamUnit u{0, L.trial_begin, L.trial_count, 0, density};
    return launch_pass<false>(lay, a, &u, 1, StreamAdjArgs{}, n_cu, s);
}

int stream_batch_max() { return kMaxSegs; }

hipError_t launch_stream_pass_units(const StreamLayout& lay, const StreamUnit* units, int n, const FoldViews& fold,
                                    int n_img_parts, void* partials, int n_cu, hipStream_t s) {
    if (lay.P <= 0 || (lay.P - 1) / 4 >= n_img_parts) return hipErrorInvalidValue;
    int64_t trials = 0;
    for (int i = 0; i < n; ++i) trials += units[i].count;
    StreamPassArgs a = pass_args(lay, fold);
    place_partials(lay, a, partials, trials);
    return launch_pass<false>(lay, a, units, n, StreamAdjArgs{}, n_cu, s);
}

hipError_t launch_stream_combine_units(const StreamLayout& lay, const StreamUnit* units, int n, const LayerArgs* L_dev,
                                       const void* partials, double* ylt, hipStream_t s) {
    if (n < 1 || n > kMaxSegs) return hipErrorInvalidValue;
    CombineArgs c{};
    c.n = n;
    int64_t blocks = 0, trials = 0;
    for (int i = 0; i < n; ++i) {
        c.unit[i] = CombineUnit{blocks, units[i].count, trials * lay.P, units[i].out_at, units[i].layer, 0};
        blocks += (units[i].count + 255) / 256;
        trials += units[i].count;
    }
    hipLaunchKernelGGL(stream_combine_units_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s,
                       static_cast<const double*>(partials), stream_partials_lo(lay, partials, trials), lay.P, c, L_dev,
                       ylt);
    return hipGetLastError();
}

int64_t stream_adjoint_scratch_bytes(int64_t trials) {
    // (group, lane) class slots: at most trials / 16 + 2 groups of 64
    return 4 * (trials > 0 ? trials : 0) + 256;
}

hipError_t launch_stream_classes(const StreamLayout& lay, const LayerArgs& L, const double* S, const double* ylt,
                                 const TailStats* tail, void* scratch, int64_t scratch_bytes, long long* agg_mean,
                                 long long* agg_tvar, int copies, int stride, uint64_t* to_clear, int64_t n_clear,
                                 int n_cu, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    // (the masks are of 64 trials, whatever the copy's groups)
    const int G = to_clear ? 64 : lay.G;
    const int64_t t_lo = L.trial_begin, t_hi = t_lo + L.trial_count, g_lo = t_lo / G;
    const int64_t n_slots = ((t_hi + G - 1) / G - g_lo) * 64;
    if (n_slots > scratch_bytes) return hipErrorInvalidValue;
    // the workgroups of a copy add to the same four sums
    const int64_t cb = std::min((n_slots + 255) / 256, int64_t(n_cu));
    hipLaunchKernelGGL(stream_class_kernel, dim3(static_cast<uint32_t>(cb)), dim3(256), 0, s, S, ylt, tail, L.aggR,
                       L.aggL, t_lo, t_hi, G, g_lo, n_slots, static_cast<uint8_t*>(scratch), agg_mean, agg_tvar,
                       copies, stride, to_clear, n_clear);
    return hipGetLastError();
}

hipError_t launch_stream_adjoint(const StreamLayout& lay, double density, const LayerArgs& L, void* part_scratch,
                                 int n_img_parts, const uint8_t* cls, const TailStats* tail, uint64_t* w_mean,
                                 uint64_t* w_tvar, int n_cu, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    if (lay.P <= 0 || (lay.P - 1) / 4 >= n_img_parts) return hipErrorInvalidValue;
    StreamPassArgs a = pass_args(lay, fold_views(part_scratch, n_img_parts));
    const StreamAdjArgs adj{cls, w_mean, w_tvar, tail};
    const StreamUnit u{0, L.trial_begin, L.trial_count, 0, density};
    return launch_pass<true>(lay, a, &u, 1, adj, n_cu, s);
}

hipError_t launch_stream_combine(const StreamLayout& lay, const LayerArgs& L, const LayerArgs* L_dev,
                                 const void* partials, double* ylt, double* ylt_too, double* S, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    const double* hi = static_cast<const double*>(partials);
    const float* lo = stream_partials_lo(lay, partials, L.trial_count);
    const int64_t blocks = (L.trial_count + 255) / 256;
    hipLaunchKernelGGL(stream_combine_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s, hi, lo, lay.P,
                       L.trial_count, L.aggR, L.aggL, L_dev, ylt, ylt_too, S);
    return hipGetLastError();
}

}  // namespace ara
