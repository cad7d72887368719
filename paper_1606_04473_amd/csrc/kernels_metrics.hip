// Risk metrics from a Year Loss Table: mean, PML_p, TVaR_p.
//
// Year losses are >= 0, so their IEEE-754 bit patterns (keys) order like their
// values when read as uint64.  PML_p is the m-th largest.  It is found in one
// histogram over all values and a selection among the few that share its bin:
//  * the largest finite key gives the top bin; the 32 octaves below it are cut
//    into 64 bins each (six mantissa bits), every octave further down is a bin of
//    its own, 4096 bins in all (infinities share the top one, zeros the lowest).
//    The map is monotone, so the histogram's counts from the top give each
//    probability's bin, the rank left to find inside it and the count above it.
//    Values spread over many bins: a histogram of plain top bits (sign and
//    exponent) crowds them into a few, where LDS and device atomics queue up on
//    each other; one bin for all below 64 octaves leaves a million losses over
//    2000 octaves, or below one infinity, to one workgroup: 1340 and 1720 us, now 37 and 39;
//  * values above the bin are summed, the keys inside it collected;
//  * one workgroup narrows those by further 4096-bin steps between their smallest
//    and largest key (one step as a rule; none when all are equal, as at a
//    limit or at zero), ranks the last 256 or fewer against each other, and
//    forms TVaR_p = (sum of the values above v + (m - c_gt) v) / m, with v =
//    PML_p and c_gt the count above it.
// All probabilities advance together.  Up to kSmallMax values one workgroup
// holds them in registers and does everything in one launch; beyond, four
// launches: sums and the largest key, the histogram, the collection, and a
// finishing workgroup per probability (the first launch is the partial sums'
// merge itself where the year losses are formed in the same call).  What bounds
// all of them is latency -- a launch and its dependent loads are 4 us here, the
// data of 1M losses 8 MB -- so launches, barriers and queues on one address were
// taken out: 1M losses and three probabilities 42 us where two 12-bit radix
// passes took 57, 10,000 losses and one probability 14 us (26).
// Sums are double-double.  The order of the values above a bin is fixed by the
// launch, that of the few collected candidates by timing; the rounded results do
// not depend on either beyond the sums' 2^-100 error.  The product (m - c_gt) v
// is added exactly via fma.
#include "ara_internal.hpp"

namespace ara {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kPer = 8;                // values per thread of the multi-workgroup launches
constexpr int kSumBlocks = 512;
constexpr int kBins = 4096;
constexpr int kFinePerOctave = 6;      // log2 of the bins per octave below the largest key
constexpr int kBinShift = 52 - kFinePerOctave;
constexpr int kFineBins = 2048;        // of them; the other 2048 are one per exponent
constexpr int kMaxProbs = 4;
constexpr int kDirect = 256;           // candidates ranked directly (all pairs)
// One workgroup up to here: 16 values per thread in registers.
constexpr int kSmallPer = 16;
constexpr int64_t kSmallMax = int64_t(kThreads) * kSmallPer;
constexpr uint64_t kInfKey = uint64_t(0x7FF) << 52;
constexpr uint64_t kBadKey = ~uint64_t(0);

// one probability's state after the histogram
struct Pick {
    uint32_t bin;     // its m-th largest value's bin
    uint32_t count;   // values in the bin
    int64_t k;        // rank to find inside the bin (1-based, from the largest)
    int64_t above;    // values in higher bins
};

struct Scratch {
    double* part_hi;      // [kMaxProbs + 1][kSumBlocks]: mean partials, then the tails'
    double* part_lo;
    uint64_t* part_max;   // [kSumBlocks] largest finite key; kBadKey when a value is NaN or < 0
    uint32_t* hist;       // [kBins]
    Pick* pick;           // [kMaxProbs] each probability's bin
    uint32_t* ccount;     // [kMaxProbs] candidates collected per probability
    uint64_t* cand;       // [n_probs][n]
};

constexpr int64_t kCandAlign = 256;

constexpr int64_t base_bytes() {
    return static_cast<int64_t>(kMaxProbs + 1) * kSumBlocks * 2 * sizeof(double) + kSumBlocks * sizeof(uint64_t) +
           kBins * sizeof(uint32_t) + kMaxProbs * sizeof(Pick) + 64;
}

// Scratch of the allocation-free entry point: the fixed block plus candidate
// keys for up to kMaxProbs x kStaticTrials year losses (32.1 MiB).  A static
// device array, so each device the library runs on holds its own copy until
// the process ends; host code reaches it only through the address that
// hipGetSymbolAddress returns on that device (metrics_noalloc_scratch).
constexpr int64_t kStaticTrials = int64_t(1) << 20;
constexpr int64_t kStaticBytes =
    (base_bytes() + kCandAlign - 1) / kCandAlign * kCandAlign + kMaxProbs * kStaticTrials * int64_t(sizeof(uint64_t));
static __device__ __align__(256) uint8_t scratch[kStaticBytes];

Scratch carve(void* base) {
    char* p = static_cast<char*>(base);
    char* const start = p;
    Scratch s;
    const int64_t np = static_cast<int64_t>(kMaxProbs + 1) * kSumBlocks;
    s.part_hi = reinterpret_cast<double*>(p);
    p += np * sizeof(double);
    s.part_lo = reinterpret_cast<double*>(p);
    p += np * sizeof(double);
    s.part_max = reinterpret_cast<uint64_t*>(p);
    p += kSumBlocks * sizeof(uint64_t);
    s.hist = reinterpret_cast<uint32_t*>(p);
    p += kBins * sizeof(uint32_t);
    s.pick = reinterpret_cast<Pick*>(p);
    p += kMaxProbs * sizeof(Pick);
    s.ccount = reinterpret_cast<uint32_t*>(p);
    s.cand = reinterpret_cast<uint64_t*>(start + (base_bytes() + kCandAlign - 1) / kCandAlign * kCandAlign);
    return s;
}

__device__ __forceinline__ uint64_t key_of(double x) {
    // +0.0 for -0.0 so that zero losses of either sign rank lowest
    return __double_as_longlong(x + 0.0);
}

// a key's bin; `top`: the largest finite key's top bits (a key above it is infinite)
__device__ __forceinline__ uint32_t top_bits(uint64_t key) { return static_cast<uint32_t>(key >> kBinShift); }
__device__ __forceinline__ uint32_t bin_of(uint64_t key, uint32_t top) {
    const uint32_t bits = top_bits(key);
    const int below = static_cast<int>(top) - static_cast<int>(bits);
    return below < kFineBins ? kBins - 1 - max(below, 0) : bits >> kFinePerOctave;     // below: the exponent
}

// the top bits of a bin's keys: lo .. lo + span
struct BinBits {
    uint32_t lo, span;
};
__device__ __forceinline__ BinBits bits_of(uint32_t bin, uint32_t top) {
    if (bin >= kFineBins) return BinBits{top - (kBins - 1 - bin), bin == kBins - 1 ? ~0u - top : 0u};
    const uint32_t lo = bin << kFinePerOctave, hi = min(lo + (1u << kFinePerOctave) - 1, top - kFineBins);
    return BinBits{lo, hi - lo};
}

// the largest finite key so far
__device__ __forceinline__ uint64_t max_finite(uint64_t mx, uint64_t key) {
    return key > mx && key < kInfKey ? key : mx;
}

__device__ __forceinline__ uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }

__device__ __forceinline__ double read_lane(double v, int lane) { return __shfl(v, lane, kWave); }

// totals over the wave (and over its first 16 lanes), in every lane
__device__ __forceinline__ void wave_sum_dd(double& hi, double& lo) {
#define ARA_STEP(ctrl, mask)                                    \
    {                                                           \
        const double h = dpp_f64<ctrl, mask>(hi), l = dpp_f64<ctrl, mask>(lo); \
        dd_merge(hi, lo, h, l);                                 \
    }
    ARA_WAVE_SCAN(ARA_STEP);
#undef ARA_STEP
    hi = read_lane(hi, 63);
    lo = read_lane(lo, 63);
}
__device__ __forceinline__ void row_sum_dd(double& hi, double& lo) {
#define ARA_STEP(ctrl)                                          \
    {                                                           \
        const double h = dpp_f64<ctrl, 0xF>(hi), l = dpp_f64<ctrl, 0xF>(lo); \
        dd_merge(hi, lo, h, l);                                 \
    }
    ARA_STEP(0x111);
    ARA_STEP(0x112);
    ARA_STEP(0x114);
    ARA_STEP(0x118);
#undef ARA_STEP
    hi = read_lane(hi, 15);
    lo = read_lane(lo, 15);
}
__device__ __forceinline__ uint64_t wave_max(uint64_t v) {
#define ARA_STEP(ctrl, mask) v = max_u64(v, dpp_u64<ctrl, mask>(v))
    ARA_WAVE_SCAN(ARA_STEP);
#undef ARA_STEP
    return __shfl(v, 63, kWave);
}
__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
#define ARA_STEP(ctrl, mask) v += dpp_u64<ctrl, mask>(v)
    ARA_WAVE_SCAN(ARA_STEP);
#undef ARA_STEP
    return __shfl(v, 63, kWave);
}
// inclusive prefix sum over the wave
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
#define ARA_STEP(ctrl, mask) v += dpp_u32<ctrl, mask>(v)
    ARA_WAVE_SCAN(ARA_STEP);
#undef ARA_STEP
    return v;
}

// Workgroup reductions over kThreads threads, valid in every thread: kN sums (n
// of them used), or two largest keys, for two barriers.  `sh` is reused by the
// next call, whose first barrier covers this one's reads.
struct ReduceLds {
    double hi[kMaxProbs + 1][kWaves], lo[kMaxProbs + 1][kWaves];
    uint64_t u[2][kWaves];
};
template <int kN>
__device__ __forceinline__ void block_sums(ReduceLds& sh, double (&hi)[kN], double (&lo)[kN], int n) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < kN; ++q)
        if (q < n) wave_sum_dd(hi[q], lo[q]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kN; ++q)
        if (q < n && lane == 0) {
            sh.hi[q][w] = hi[q];
            sh.lo[q][w] = lo[q];
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kN; ++q)
        if (q < n) {
            hi[q] = sh.hi[q][lane & (kWaves - 1)];
            lo[q] = sh.lo[q][lane & (kWaves - 1)];
            row_sum_dd(hi[q], lo[q]);
        }
}
__device__ __forceinline__ void block_max2(ReduceLds& sh, uint64_t& a, uint64_t& b) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    a = wave_max(a);
    b = wave_max(b);
    __syncthreads();
    if (lane == 0) {
        sh.u[0][w] = a;
        sh.u[1][w] = b;
    }
    __syncthreads();
    a = wave_max(sh.u[0][lane & (kWaves - 1)]);
    b = wave_max(sh.u[1][lane & (kWaves - 1)]);
}
__device__ __forceinline__ uint64_t block_max(ReduceLds& sh, uint64_t v) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) sh.u[0][w] = v;
    __syncthreads();
    return wave_max(sh.u[0][lane & (kWaves - 1)]);
}
__device__ __forceinline__ uint64_t block_count(ReduceLds& sh, uint64_t v) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) sh.u[1][w] = v;
    __syncthreads();
    return wave_sum(lane < kWaves ? sh.u[1][lane] : 0ull);
}

struct MArgs {
    int64_t m[kMaxProbs];
};

// The bins that hold the k[q]-th largest counted values of a histogram, from the
// highest bin down; picks in LDS, valid after the call's last barrier.  Called
// by the whole workgroup of kThreads; thread t brings its four bins' counts,
// thread 0 the highest (own_bins).
struct PickLds {
    uint32_t wave_sum[kWaves];
    Pick pick[kMaxProbs];
};
__device__ __forceinline__ u32x4 own_bins(const uint32_t* h) {
    return reinterpret_cast<const u32x4*>(h)[kThreads - 1 - threadIdx.x];
}
__device__ __forceinline__ void pick_bins(PickLds& sh, u32x4 c, const int64_t* k, int n) {
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int lo_bin = kBins - 4 * (t + 1);
    const uint32_t local = c.x + c.y + c.z + c.w;
    const uint32_t incl = wave_scan(local);
    if (lane == 63) sh.wave_sum[w] = incl;
    __syncthreads();
    const uint32_t before = wave_scan(lane < w ? sh.wave_sum[lane & (kWaves - 1)] : 0u);   // w < 16
    const int64_t excl = static_cast<int64_t>(__builtin_amdgcn_readlane(static_cast<int>(before), 63)) + incl - local;
    for (int q = 0; q < n; ++q) {
        if (excl < k[q] && k[q] <= excl + local) {
            int64_t cum = excl;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                if (cum < k[q] && k[q] <= cum + c[i])
                    sh.pick[q] = Pick{static_cast<uint32_t>(lo_bin + i), c[i], k[q] - cum, cum};
                cum += c[i];
            }
        }
    }
    __syncthreads();
}

// LDS of a workgroup that finishes a probability
struct FinishLds {
    __attribute__((aligned(16))) uint32_t hist[kBins];
    PickLds sel;
    ReduceLds red;
    uint64_t keys[kDirect];
    uint64_t found;
    uint32_t n_keys;
};

// what the selection among a probability's candidates gives
struct Chosen {
    uint64_t v;             // the key of rank k
    double hi, lo;          // sum of the values above it
    int64_t above, equal;   // how many are above it, and equal to it
};

// The k-th largest of c candidates (1 <= k <= c): steps of 4096 bins between the
// smallest and the largest key still possible until at most kDirect are left,
// which are ranked against each other, four threads a key.  `each(f)` calls f for
// every candidate the thread holds, `all(f)` for every value to be summed and
// counted (the candidates, or all values).  Whole workgroup.
template <typename Each, typename All>
__device__ __forceinline__ Chosen select_candidate(FinishLds& sh, Each each, All all, uint32_t c, int64_t k) {
    uint64_t lo = 0, hi = ~uint64_t(0);                    // the range that holds the k-th largest
    uint32_t inside = c;
    int64_t kk = k;
    if (threadIdx.x == 0) sh.n_keys = 0;
    if (c > kDirect) {
        uint64_t mx = 0, mn = 0;                           // mn: the largest complement
        each([&](uint64_t key) {
            mx = max_u64(mx, key);
            mn = max_u64(mn, ~key);
        });
        block_max2(sh.red, mx, mn);
        hi = mx;
        lo = ~mn;
        while (inside > kDirect && lo != hi) {
            const int bits = 64 - __builtin_clzll(hi - lo);        // hi - lo < 2^bits
            const int shift = bits > 12 ? bits - 12 : 0;
            reinterpret_cast<u32x4*>(sh.hist)[threadIdx.x] = u32x4{0, 0, 0, 0};
            __syncthreads();
            each([&](uint64_t key) {
                if (key >= lo && key <= hi) atomicAdd(&sh.hist[(key - lo) >> shift], 1u);
            });
            __syncthreads();
            pick_bins(sh.sel, own_bins(sh.hist), &kk, 1);
            const Pick p = sh.sel.pick[0];
            lo += static_cast<uint64_t>(p.bin) << shift;
            const uint64_t last = lo + ((uint64_t(1) << shift) - 1);
            hi = last < hi ? last : hi;
            inside = p.count;
            kk = p.k;
            __syncthreads();
        }
    }
    Chosen r;
    if (lo == hi) {                                        // every candidate left is the same
        r.v = lo;
    } else {
        // at most kDirect keys in [lo, hi]: the k-th largest has fewer than k
        // keys above it and at least k at or above it
        __syncthreads();
        each([&](uint64_t key) {
            if (key >= lo && key <= hi) sh.keys[atomicAdd(&sh.n_keys, 1u)] = key;
        });
        __syncthreads();
        const int n = static_cast<int>(inside);
        if (static_cast<int>(threadIdx.x) < 4 * n) {
            const uint64_t kj = sh.keys[threadIdx.x >> 2];
            int gt = 0, ge = 0;
            for (int i = threadIdx.x & 3; i < n; i += 4) {
                gt += sh.keys[i] > kj;
                ge += sh.keys[i] >= kj;
            }
            gt += __shfl_xor(gt, 1);
            ge += __shfl_xor(ge, 1);
            gt += __shfl_xor(gt, 2);
            ge += __shfl_xor(ge, 2);
            if (gt < kk && kk <= ge) sh.found = kj;                // every such thread writes the same key
        }
        __syncthreads();
        r.v = sh.found;
    }
    // The sum above it: collected candidates' places depend on timing, the
    // double-double sum's rounded value does not, beyond its 2^-100 error
    double h[1] = {0.0}, l[1] = {0.0};
    uint64_t counts = 0;                                   // above in the high half, equal in the low
    all([&](uint64_t key) {
        if (key > r.v) {
            dd_add(h[0], l[0], __longlong_as_double(static_cast<long long>(key)));
            counts += uint64_t(1) << 32;
        }
        counts += key == r.v;
    });
    block_sums(sh.red, h, l, 1);
    counts = block_count(sh.red, counts);
    r.hi = h[0];
    r.lo = l[0];
    r.above = static_cast<int64_t>(counts >> 32);
    r.equal = static_cast<int64_t>(counts & 0xFFFFFFFFu);
    return r;
}

// A probability's candidates in memory: up to kPer per thread are loaded once, more
// are read again for each step, kPer in flight (one in flight: a million losses within
// 0.1 % of each other 1720 us, now 690).
__device__ __forceinline__ Chosen select_in_memory(FinishLds& sh, const uint64_t* cand, uint32_t c, int64_t k) {
    if (c <= kThreads * kPer) {
        uint64_t key[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t i = u * kThreads + threadIdx.x;
            key[u] = i < c ? cand[i] : 0ull;
        }
        auto each = [&](auto f) {
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (u * kThreads + threadIdx.x < c) f(key[u]);
        };
        return select_candidate(sh, each, each, c, k);
    }
    auto each = [&](auto f) {
        for (int64_t i0 = threadIdx.x; i0 < c; i0 += kThreads * kPer) {
            uint64_t key[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) key[u] = cand[i0 + u * kThreads < c ? i0 + u * kThreads : i0];
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (i0 + u * kThreads < c) f(key[u]);
        }
    };
    return select_candidate(sh, each, each, c, k);
}

// PML and TVaR of probability q, or the tail statistics, from what was chosen and
// the `above` values, of sum (hi, lo), above the candidates
__device__ __forceinline__ void write_one(const Chosen& r, int64_t above, int64_t m, double hi, double lo, int q,
                                          const MetricsOut& out, TailStats* tail) {
    const int64_t gt = above + r.above;
    if (tail) {
        *tail = TailStats{r.v, gt, r.equal, m};
        return;
    }
    dd_merge(hi, lo, r.hi, r.lo);
    const double v = __longlong_as_double(static_cast<long long>(r.v));
    const double copies = static_cast<double>(m - gt);     // copies of v in the top m
    const double pr = copies * v;
    const double pe = fma(copies, v, -pr);                 // exact product pr + pe
    dd_merge(hi, lo, pr, pe);
    out.pml[q * out.stride] = v;
    out.tvar[q * out.stride] = (hi + lo) / static_cast<double>(m);
}

// results of a YLT with a NaN or a negative value
__device__ __forceinline__ void write_bad(int n_probs, const MetricsOut& out, TailStats* tail, const MArgs& ma) {
    if (threadIdx.x != 0) return;
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    if (tail) {
        *tail = TailStats{0, 0, 1, ma.m[0]};
        return;
    }
    *out.mean = nan;
    for (int q = 0; q < n_probs; ++q) {
        out.pml[q * out.stride] = nan;
        out.tvar[q * out.stride] = nan;
    }
}

// A workgroup's part of the first launch: its sum and largest key, and its share
// of the histogram and the counts cleared for the next ones, so the scratch may
// hold anything before a call (a launch of its own for the counts took 4.5 us).  A
// workgroup with an infinite value reads its values (x, strided by the grid) again for
// the largest finite one.
__device__ __forceinline__ void store_partials(ReduceLds& sh, const Scratch& s, double hi, double lo, uint64_t mx,
                                               const double* x, int64_t n) {
    double h[1] = {hi}, l[1] = {lo};
    block_sums(sh, h, l, 1);
    mx = block_max(sh, mx);
    if (mx == kInfKey) {
        mx = 0;
        const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
        for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride)
            mx = max_finite(mx, key_of(x[i]));
        mx = block_max(sh, mx);
    }
    if (threadIdx.x == 0) {
        s.part_hi[blockIdx.x] = h[0];
        s.part_lo[blockIdx.x] = l[0];
        s.part_max[blockIdx.x] = mx;
    }
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < kBins; i += gridDim.x * kThreads) s.hist[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x < kMaxProbs) s.ccount[threadIdx.x] = 0;
}

// launch 1 where the year losses are formed: the merge of the streaming pass's
// per-(part, trial) partial sums (part by part in double-double, rounded once, the
// aggregate terms applied) with the sums and largest keys on the way
__global__ __launch_bounds__(kThreads) void combine_sum_max_kernel(const double* __restrict__ part_hi,
                                                                   const float* __restrict__ part_lo, int P, int64_t n,
                                                                   const LayerArgs* __restrict__ L,
                                                                   double* __restrict__ ylt, Scratch s) {
    __shared__ ReduceLds sh;
    const double aggR = L->aggR, aggL = L->aggL;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    double sum_hi = 0.0, sum_lo = 0.0;
    uint64_t mx = 0;
    bool bad = false;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; k < n; k += stride) {
        double hi = 0.0, lo = 0.0;
        for (int p = 0; p < P; ++p) dd_merge(hi, lo, part_hi[p * n + k], static_cast<double>(part_lo[p * n + k]));
        const double y = apply_terms(hi + lo, aggR, aggL);
        ylt[k] = y;
        bad |= !(y >= 0.0);
        dd_add(sum_hi, sum_lo, y);
        mx = max_u64(mx, key_of(y));
    }
    store_partials(sh, s, sum_hi, sum_lo, bad ? kBadKey : mx, ylt, n);
}

// launch 1: sums and largest keys
__global__ __launch_bounds__(kThreads) void sum_max_kernel(const double* __restrict__ x, int64_t n, Scratch s) {
    __shared__ ReduceLds sh;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    double hi = 0.0, lo = 0.0;
    uint64_t mx = 0;
    bool bad = false;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += kPer * stride) {
        double v[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) v[u] = i + u * stride < n ? x[i + u * stride] : 0.0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            bad |= !(v[u] >= 0.0);
            dd_add(hi, lo, v[u]);
            mx = max_u64(mx, key_of(v[u]));
        }
    }
    store_partials(sh, s, hi, lo, bad ? kBadKey : mx, x, n);
}

// the largest key over the first launch's workgroups
__device__ __forceinline__ uint64_t top_key(ReduceLds& sh, const Scratch& s, int n_part) {
    return block_max(sh, static_cast<int>(threadIdx.x) < n_part ? s.part_max[threadIdx.x] : 0ull);
}

// launch 2: the histogram
__global__ __launch_bounds__(kThreads) void bin_kernel(const double* __restrict__ x, int64_t n, Scratch s, int n_part) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins];
    __shared__ ReduceLds sh;
    reinterpret_cast<u32x4*>(hist)[threadIdx.x] = u32x4{0, 0, 0, 0};
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    double v[kPer];                                        // in flight while the largest key is found
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[u] = first + u * stride < n ? x[first + u * stride] : 0.0;
    const uint64_t mk = top_key(sh, s, n_part);
    if (mk == kBadKey) return;
    const uint32_t top = top_bits(mk);
    for (int64_t i = first; i < n; i += kPer * stride) {
        if (i != first) {
#pragma unroll
            for (int u = 0; u < kPer; ++u) v[u] = i + u * stride < n ? x[i + u * stride] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (i + u * stride < n) atomicAdd(&hist[bin_of(key_of(v[u]), top)], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kBins; k += kThreads) {
        const uint32_t c = hist[k];
        if (c) atomicAdd(&s.hist[k], c);
    }
}

// launch 3: tail sums above each probability's bin, the keys inside it
__global__ __launch_bounds__(kThreads) void collect_kernel(const double* __restrict__ x, int64_t n, Scratch s, MArgs ma,
                                                           int n_probs, int n_part) {
    __shared__ PickLds sel;
    __shared__ ReduceLds red;
    __shared__ uint32_t wave_n[kMaxProbs][kWaves], wave_at[kMaxProbs][kWaves];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    const int64_t begin = static_cast<int64_t>(blockIdx.x) * kThreads;
    double v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t i = begin + u * stride + threadIdx.x;
        v[u] = i < n ? x[i] : 0.0;
    }
    const u32x4 counts = own_bins(s.hist);
    const uint64_t mk = top_key(red, s, n_part);
    if (mk == kBadKey) return;
    const uint32_t top = top_bits(mk);
    pick_bins(sel, counts, ma.m, n_probs);
    if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < n_probs) s.pick[threadIdx.x] = sel.pick[threadIdx.x];
    uint32_t bins[kMaxProbs];
    double hi[kMaxProbs] = {}, lo[kMaxProbs] = {};
#pragma unroll
    for (int q = 0; q < kMaxProbs; ++q) bins[q] = q < n_probs ? sel.pick[q].bin : 0u;
    for (int64_t b = begin; b < n; b += kPer * stride) {
        uint32_t in[kMaxProbs] = {};                       // bit u: value u is a candidate
        if (b != begin) {
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int64_t i = b + u * stride + threadIdx.x;
                v[u] = i < n ? x[i] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const bool ok = b + u * stride + threadIdx.x < n;
            const uint32_t bin = bin_of(key_of(v[u]), top);
#pragma unroll
            for (int q = 0; q < kMaxProbs; ++q) {
                if (q >= n_probs) break;
                if (ok && bin > bins[q]) dd_add(hi[q], lo[q], v[u]);
                in[q] |= ok && bin == bins[q] ? 1u << u : 0u;
            }
        }
        // one device atomic per workgroup and probability: every workgroup adds
        // to the same counters
        uint32_t pre[kMaxProbs];
#pragma unroll
        for (int q = 0; q < kMaxProbs; ++q) {
            if (q >= n_probs) break;
            const uint32_t c = static_cast<uint32_t>(__popc(in[q]));
            const uint32_t incl = wave_scan(c);
            pre[q] = incl - c;
            if (lane == 63) wave_n[q][w] = incl;
        }
        __syncthreads();
        if (w < n_probs && lane < kWaves) {
            const uint32_t c = wave_n[w][lane];
            const uint32_t incl = wave_scan(c);
            uint32_t at = 0;
            if (lane == kWaves - 1 && incl) at = atomicAdd(&s.ccount[w], incl);
            wave_at[w][lane] = __shfl(at, kWaves - 1, kWave) + incl - c;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kMaxProbs; ++q) {
            if (q >= n_probs) break;
            uint64_t* dst = s.cand + static_cast<int64_t>(q) * n + wave_at[q][w] + pre[q];
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if ((in[q] >> u) & 1u) *dst++ = key_of(v[u]);
        }
    }
    block_sums(red, hi, lo, n_probs);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < kMaxProbs; ++q)
            if (q < n_probs) {
                s.part_hi[(1 + q) * kSumBlocks + blockIdx.x] = hi[q];
                s.part_lo[(1 + q) * kSumBlocks + blockIdx.x] = lo[q];
            }
    }
}

// launch 4: one workgroup per probability finishes it; another forms the mean
__global__ __launch_bounds__(kThreads) void finish_kernel(int64_t n, Scratch s, MArgs ma, int n_probs, int n_part,
                                                          int n_tail_part, MetricsOut out, TailStats* tail) {
    __shared__ FinishLds sh;
    const int q = static_cast<int>(blockIdx.x);            // n_probs: the mean
    const bool mean = q == n_probs;
    const int row = mean ? 0 : 1 + q;
    const bool in = static_cast<int>(threadIdx.x) < (mean ? n_part : n_tail_part);
    // everything the workgroup needs from memory but the candidates, in flight together
    double h[1] = {in ? s.part_hi[row * kSumBlocks + threadIdx.x] : 0.0};
    double l[1] = {in ? s.part_lo[row * kSumBlocks + threadIdx.x] : 0.0};
    const Pick p = mean ? Pick{0, 0, 1, 0} : s.pick[q];
    const bool bad = top_key(sh.red, s, n_part) == kBadKey;
    if (bad) {
        if (q == 0) write_bad(n_probs, out, tail, ma);
        return;
    }
    block_sums(sh.red, h, l, 1);
    if (mean) {
        if (!tail && threadIdx.x == 0) *out.mean = (h[0] + l[0]) / static_cast<double>(n);
        return;
    }
    const Chosen r = select_in_memory(sh, s.cand + static_cast<int64_t>(q) * n, p.count, p.k);
    if (threadIdx.x == 0) write_one(r, p.above, ma.m[q], h[0], l[0], q, out, tail);
}

// the mean alone (no probabilities), from the first launch's partials
__global__ __launch_bounds__(kThreads) void mean_kernel(int64_t n, Scratch s, int n_part, MetricsOut out) {
    __shared__ ReduceLds sh;
    const bool in = static_cast<int>(threadIdx.x) < n_part;
    double h[1] = {in ? s.part_hi[threadIdx.x] : 0.0}, l[1] = {in ? s.part_lo[threadIdx.x] : 0.0};
    const bool bad = top_key(sh, s, n_part) == kBadKey;
    block_sums(sh, h, l, 1);
    if (threadIdx.x == 0)
        *out.mean = bad ? __longlong_as_double(0x7ff8000000000000LL) : (h[0] + l[0]) / static_cast<double>(n);
}

// Everything in one workgroup, the values in registers (kV per thread).  The
// selection runs over the registers too: a candidate is a value in the bin.
template <int kV>
__global__ __launch_bounds__(kThreads) void small_metrics_kernel(const double* __restrict__ x, int n, MArgs ma,
                                                                 int n_probs, MetricsOut out, TailStats* tail) {
    __shared__ FinishLds sh;
    __shared__ Pick picks[kMaxProbs];
    double v[kV];
#pragma unroll
    for (int u = 0; u < kV; ++u) {
        const int i = u * kThreads + static_cast<int>(threadIdx.x);
        v[u] = i < n ? x[i] : 0.0;
    }
    reinterpret_cast<u32x4*>(sh.hist)[threadIdx.x] = u32x4{0, 0, 0, 0};
    double mh[1] = {0.0}, ml[1] = {0.0};
    uint64_t mx = 0;
    bool bad = false;
#pragma unroll
    for (int u = 0; u < kV; ++u) {
        bad |= !(v[u] >= 0.0);
        dd_add(mh[0], ml[0], v[u]);
        mx = max_u64(mx, key_of(v[u]));
    }
    mx = block_max(sh.red, bad ? kBadKey : mx);
    if (mx == kBadKey) {
        write_bad(n_probs, out, tail, ma);
        return;
    }
    if (mx == kInfKey) {
        mx = 0;
#pragma unroll
        for (int u = 0; u < kV; ++u) mx = max_finite(mx, key_of(v[u]));
        mx = block_max(sh.red, mx);
    }
    const uint32_t top = top_bits(mx);
#pragma unroll
    for (int u = 0; u < kV; ++u)
        if (u * kThreads + static_cast<int>(threadIdx.x) < n) atomicAdd(&sh.hist[bin_of(key_of(v[u]), top)], 1u);
    if (!tail) {
        block_sums(sh.red, mh, ml, 1);
        if (threadIdx.x == 0) *out.mean = (mh[0] + ml[0]) / static_cast<double>(n);
    }
    if (n_probs == 0) return;
    __syncthreads();
    pick_bins(sh.sel, own_bins(sh.hist), ma.m, n_probs);
    if (threadIdx.x < kMaxProbs) picks[threadIdx.x] = sh.sel.pick[threadIdx.x];
    __syncthreads();
    auto all = [&](auto f) {
#pragma unroll
        for (int u = 0; u < kV; ++u)
            if (u * kThreads + static_cast<int>(threadIdx.x) < n) f(key_of(v[u]));
    };
#pragma unroll 1
    for (int q = 0; q < n_probs; ++q) {
        const Pick p = picks[q];
        const BinBits in = bits_of(p.bin, top);
        auto each = [&](auto f) {
            all([&](uint64_t key) {
                if (top_bits(key) - in.lo <= in.span) f(key);
            });
        };
        const Chosen r = select_candidate(sh, each, all, p.count, p.k);
        if (threadIdx.x == 0) write_one(r, 0, ma.m[q], 0.0, 0.0, q, out, tail);
    }
}

// workgroups of the multi-workgroup launches: kPer values per thread, at most kSumBlocks
int sum_blocks(int64_t n) {
    const int64_t b = (n + kThreads * kPer - 1) / (kThreads * kPer);
    return static_cast<int>(b > kSumBlocks ? kSumBlocks : (b < 1 ? 1 : b));
}

// the launches after the sums and largest keys (n_part workgroups)
hipError_t launch_selection(const double* ylt, int64_t n, const MArgs& ma, int n_probs, const Scratch& s, int n_part,
                            MetricsOut out, TailStats* tail, hipStream_t st) {
    const dim3 g(sum_blocks(n)), t(kThreads);
    if (n_probs == 0) {
        hipLaunchKernelGGL(mean_kernel, dim3(1), t, 0, st, n, s, n_part, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(bin_kernel, g, t, 0, st, ylt, n, s, n_part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(collect_kernel, g, t, 0, st, ylt, n, s, ma, n_probs, n_part);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(finish_kernel, dim3(n_probs + (tail ? 0 : 1)), t, 0, st, n, s, ma, n_probs, n_part,
                       static_cast<int>(g.x), out, tail);
    return hipGetLastError();
}

hipError_t launch_all(const double* ylt, int64_t n, const int64_t* m_host, int n_probs, void* scratch, MetricsOut out,
                      TailStats* tail, hipStream_t st) {
    if (n_probs > kMaxProbs || n < 1) return hipErrorInvalidValue;
    const Scratch s = carve(scratch);
    MArgs ma{};
    for (int q = 0; q < n_probs; ++q) ma.m[q] = m_host[q];
    if (n <= kSmallMax) {
        const int small_n = static_cast<int>(n);
        if (n <= 4 * kThreads)
            hipLaunchKernelGGL(small_metrics_kernel<4>, dim3(1), dim3(kThreads), 0, st, ylt, small_n, ma, n_probs, out,
                               tail);
        else
            hipLaunchKernelGGL(small_metrics_kernel<kSmallPer>, dim3(1), dim3(kThreads), 0, st, ylt, small_n, ma, n_probs,
                               out, tail);
        return hipGetLastError();
    }
    hipError_t err;
    const int b = sum_blocks(n);
    hipLaunchKernelGGL(sum_max_kernel, dim3(b), dim3(kThreads), 0, st, ylt, n, s);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    return launch_selection(ylt, n, ma, n_probs, s, b, out, tail, st);
}

}  // namespace

int64_t metrics_scratch_bytes(int n_probs, int64_t n) {
    const int64_t base = (base_bytes() + kCandAlign - 1) / kCandAlign * kCandAlign;
    return base + static_cast<int64_t>(n_probs) * n * static_cast<int64_t>(sizeof(uint64_t));
}

hipError_t launch_metrics(const double* ylt, int64_t n, const int64_t* m_host, int n_probs, void* scratch,
                          MetricsOut out, hipStream_t st) {
    return launch_all(ylt, n, m_host, n_probs, scratch, out, nullptr, st);
}

hipError_t launch_combine_metrics(const double* part_hi, const float* part_lo, int P, int64_t n, const LayerArgs* L_dev,
                                  double* ylt, const int64_t* m_host, int n_probs, void* scratch, MetricsOut out,
                                  hipStream_t st) {
    if (n_probs > kMaxProbs || n <= kSmallMax) return hipErrorInvalidValue;
    const Scratch s = carve(scratch);
    MArgs ma{};
    for (int q = 0; q < n_probs; ++q) ma.m[q] = m_host[q];
    // a workgroup per 1024 trials, up to kSumBlocks (two per CU)
    const int64_t want = (n + kThreads - 1) / kThreads;
    const int b = static_cast<int>(want < kSumBlocks ? want : kSumBlocks);
    hipLaunchKernelGGL(combine_sum_max_kernel, dim3(b), dim3(kThreads), 0, st, part_hi, part_lo, P, n, L_dev, ylt, s);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    return launch_selection(ylt, n, ma, n_probs, s, b, out, nullptr, st);
}

bool combine_metrics_apply(int64_t n) { return n > kSmallMax; }

int64_t tail_stats_scratch_bytes(int64_t n) { return metrics_scratch_bytes(1, n); }

// the m-th largest year loss with the counts above and at it: the metrics'
// launches, whose last workgroup writes the statistics instead
hipError_t launch_tail_stats(const double* ylt, int64_t n, int64_t m, void* scratch, TailStats* out, hipStream_t st) {
    return launch_all(ylt, n, &m, 1, scratch, MetricsOut{}, out, st);
}

// The device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept; later calls reuse it.  No
// allocation of any kind.
hipError_t metrics_noalloc_scratch(void** ptr, int64_t* capacity) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *capacity = kStaticBytes;
    return hipSuccess;
}

}  // namespace ara
