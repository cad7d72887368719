// Catalogue-partitioned trial pass.
//
// Random 8-byte gathers from a table larger than L2 run an order of magnitude
// below the HBM stream rate on gfx950, and most occurrences of a layer carry
// zero loss (an event absent from every ELT of the layer, or below the
// occurrence retention).  So the per-event question "is o(E) nonzero, and
// where is its value" is answered from LDS:
//
//  * the catalogue is cut into parts of 2^18 events; for each part the fold
//    builds a 37,120-byte image: a 32 KB bitmap of nonzero o(E), a 16-bit rank
//    per 128 events relative to its 4096-event superblock, and the global rank
//    of each superblock; the nonzero values themselves go, in catalogue order,
//    to a compact array small enough to stay in L2;
//  * at table creation the YET is laid out part-major inside tiles of
//    consecutive trials (tile -> part -> trial -> that trial's events of that
//    part in time order, each segment padded to 16 bytes with an ID no event
//    has), so a workgroup can hold one part image in LDS and stream exactly
//    the events that need it;
//  * a workgroup takes a tile, walks the parts in order, and for each trial
//    adds the part's partial sum (double-double) into the trial's LDS
//    accumulator; the trial's owner and the part order are fixed, so the
//    result does not depend on scheduling.
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <vector>

#include "ara_internal.hpp"
#include "scatter.hpp"

namespace ara {

namespace {

constexpr int kPartShift = 18;
constexpr int64_t kPartSize = int64_t(1) << kPartShift;       // catalogue events per part
constexpr int kWords = kPartSize / 64;                        // 4096 u64 bitmap words
constexpr int kRank16 = kPartSize / 128;                      // 2048 u16
constexpr int kSuperShift = 12;
constexpr int kSuper = 1 << kSuperShift;                      // 4096 events per superblock
constexpr int kBase32 = kPartSize / kSuper;                   // 64 u32
constexpr int64_t kImgBytes = int64_t(kWords) * 8 + int64_t(kRank16) * 2 + int64_t(kBase32) * 4;
static_assert(kImgBytes == 37120 && kImgBytes == kImgPartBytes && kPartShift == kImgShift, "part image layout");
static_assert(kImgBytes % 16 == 0, "16-byte copies");
constexpr int kTileMax = 256;                                 // trials per tile (LDS accumulators)
constexpr int kTileAlign = 32;                                // tiles start on 128-byte boundaries
constexpr uint32_t kSentinel = 0xFFFFFFFFu;

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v)), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v >> 32)), lane);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
    return __longlong_as_double(static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(__double_as_longlong(v)), lane)));
}

// ---------------------------------------------------------------------------
// create-time layout
// ---------------------------------------------------------------------------

// what creating tables starts from zero: the IDs' padding, the results and the counts,
// in one launch
__global__ __launch_bounds__(256) void create_clear_kernel(uint32_t* __restrict__ pad, CreateResult* __restrict__ res,
                                                           u32x4* __restrict__ cnt, int64_t n16) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    for (int64_t i = first; i < n16; i += stride) cnt[i] = u32x4{0, 0, 0, 0};
    for (int64_t i = first; i < kIdPad; i += stride) pad[i] = 0;
    for (int64_t i = first; i < static_cast<int64_t>(sizeof(CreateResult) / 4); i += stride)
        reinterpret_cast<uint32_t*>(res)[i] = 0;
}

// smallest t in [lo, hi] with offsets[t] >= target, given offsets[hi] >=
// target; a 64-way search, all arguments uniform over the wave
__device__ int64_t first_trial_at(const int64_t* __restrict__ offsets, int64_t lo, int64_t hi, int64_t target,
                                  int lane) {
    while (hi - lo >= 64) {
        const int64_t step = (hi - lo) / 64;
        const uint64_t m = __ballot(offsets[lo + lane * step] >= target);   // index <= hi - step
        if (m == 0) {
            lo = lo + 63 * step + 1;
        } else {
            const int f = __builtin_ctzll(m);
            const int64_t nlo = f > 0 ? lo + (f - 1) * step + 1 : lo;
            hi = lo + f * step;
            lo = nlo;
        }
    }
    const int64_t idx = lo + lane;
    const uint64_t m = __ballot(idx <= hi && offsets[idx] >= target);
    return lo + __builtin_ctzll(m);
}

// Create's one pass over the IDs, bound by memory: it checks them, counts each trial's events in every part of 2^shift catalogue events (bins parts) and,
// with kCopy, stores them in the tables (16-byte aligned sources).  Each wave
// takes an equal run of the IDs in rows of 256, four rows of 16-byte loads in
// flight while the four before are counted; the counters lie in LDS, repeated for
// groups of lanes where there are few parts, and go to cnt at each trial's end
// (added there for the trials that two waves share; cnt is zero before).  One
// launch instead of a copy, a check and a count for each of the two layouts, 150 M
// IDs over 31 and 8 parts: 260 + 93 + 187 + 198 us -> 230 us.
template <bool kCopy>
__global__ __launch_bounds__(256) void yet_count_kernel(const int64_t* __restrict__ offsets, int64_t N,
                                                        const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                                                        int64_t n, uint32_t c32, int shift, int bins,
                                                        int32_t* __restrict__ cnt, uint32_t* __restrict__ flags) {
    constexpr int kRow = 256, kRows = 4;            // IDs per row, rows in flight
    __shared__ int32_t counters[4][64];
    if (*flags & kCreateBadOffsets) bins = 0;       // the trials' ranges can't be trusted
    int32_t* c = counters[threadIdx.x >> 6];
    const int lane = threadIdx.x & 63;
    const int64_t w = uniform_i64((static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6);
    const int64_t n_w = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    const int64_t rows = (n + kRow - 1) / kRow;
    const int64_t x0 = rows * w / n_w * kRow;
    const int64_t x1 = min(rows * (w + 1) / n_w * kRow, n);
    if (x0 >= x1) return;
    // counter of a part: [part][copy], the copies for lanes apart (64 in all)
    const int rep_bits = bins > 0 ? 31 - __builtin_clz(64u / static_cast<uint32_t>(bins)) : 0;
    const uint32_t rep = static_cast<uint32_t>(lane) & ((1u << rep_bits) - 1u);
    const uint32_t last_bin = static_cast<uint32_t>(bins > 0 ? bins - 1 : 0);
    c[lane] = 0;
    int64_t k = 0, kb = 0, bnd = 0, end = INT64_MAX;
    bool shared = false;                            // the trial began in an earlier wave's run
    if (bins > 0) {
        k = first_trial_at(offsets, 0, N, x0 + 1, lane) - 1;
        kb = k;
        bnd = offsets[min(kb + 1 + lane, N)];
        end = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(bnd), 0));
        shared = uniform_i64(offsets[k]) < x0;
    }
    auto flush = [&](bool add) {
        __builtin_amdgcn_wave_barrier();
        int32_t v = c[lane];
        c[lane] = 0;
        for (int off = 1; off < (1 << rep_bits); off <<= 1) v += __shfl_xor(v, off, 64);
        if (rep == 0 && (lane >> rep_bits) < bins) {
            int32_t* to = cnt + k * bins + (lane >> rep_bits);
            if (!add) *to = v;
            else if (v) atomicAdd(to, v);
        }
        __builtin_amdgcn_wave_barrier();
    };
    uint32_t bad = 0;
    u32x4 nxt[kRows];
    auto load = [&](int64_t x) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t at = x + r * kRow + lane * 4;
            nxt[r] = u32x4{0, 0, 0, 0};
            if (at + 4 <= n) {
                if (x + r * kRow < x1) nxt[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + at));
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (at + q < n) nxt[r][q] = src[at + q];
            }
        }
    };
    load(x0);
    for (int64_t x = x0; x < x1; x += kRow * kRows) {
        u32x4 cur[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) cur[r] = nxt[r];
        if (x + kRow * kRows < x1) load(x + kRow * kRows);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int64_t xr = x + r * kRow;
            if (xr >= x1) continue;
            const int64_t xe = min(xr + kRow, x1);
            const int64_t at = xr + lane * 4;
            if (kCopy) {
                if (at + 4 <= n) {
                    *reinterpret_cast<u32x4*>(dst + at) = cur[r];
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (at + q < n) dst[at + q] = cur[r][q];
                }
            }
            uint32_t most = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) most = max(most, cur[r][q]);
            bad |= most >= c32 ? 1u : 0u;
            if (bins == 0) continue;
            int32_t* slot[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                slot[q] = c + ((min(cur[r][q] >> shift, last_bin) << rep_bits) | rep);
            int64_t from = xr;
            for (;;) {
                const int64_t to = min(end, xe);
                if (from == xr && to == xr + kRow) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) atomicAdd(slot[q], 1);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (at + q >= from && at + q < to) atomicAdd(slot[q], 1);
                }
                from = to;
                if (end > xe) break;
                flush(shared);
                shared = false;
                if (++k - kb == 64) {
                    kb = k;
                    bnd = offsets[min(kb + 1 + lane, N)];
                }
                end = k < N ? static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(bnd), static_cast<int>(k - kb)))
                            : INT64_MAX;
                if (from >= xe) break;
            }
        }
    }
    if (bins > 0 && k < N) flush(true);
    if (bad) atomicOr(flags, kCreateBadId);
}

// The counts of tables whose trials are short (fewer than 16 events on average), a
// thread per trial, after a pass above has copied and checked the IDs: there the flush
// at each trial's end is what takes the time (200000 trials of 2 events: 102 us there,
// 8 in both).  A workgroup's counters lie in LDS (dynamic, [256][bins | 1]); a wave
// counts a trial past 64 events together.
constexpr int kShortTrial = 16;
__global__ __launch_bounds__(256) void short_count_kernel(const int64_t* __restrict__ offsets, int64_t N,
                                                          const uint32_t* __restrict__ ids, int shift, int bins,
                                                          int32_t* __restrict__ cnt, const uint32_t* __restrict__ flags) {
    extern __shared__ int32_t own[];
    if (*flags & kCreateBadOffsets) return;         // the trials' ranges can't be trusted
    const int row = bins | 1;                       // odd: the threads' rows in different banks
    for (int i = threadIdx.x; i < 256 * row; i += 256) own[i] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint32_t last_bin = static_cast<uint32_t>(bins - 1);
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * 256, t = t0 + threadIdx.x;
    const int64_t b = t < N ? offsets[t] : 0, e = t < N ? offsets[t + 1] : 0;
    if (e - b <= 64)
        for (int64_t i = b; i < e; ++i) own[threadIdx.x * row + min(ids[i] >> shift, last_bin)] += 1;
    for (uint64_t many = __ballot(e - b > 64); many; many &= many - 1) {
        const int l = __builtin_ctzll(many);
        const int64_t lb = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(b), l));
        const int64_t le = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(e), l));
        int32_t* of = own + ((threadIdx.x & ~63u) + l) * row;
        for (int64_t i = lb + lane; i < le; i += 64) atomicAdd(of + min(ids[i] >> shift, last_bin), 1);
    }
    __syncthreads();
    const int n = static_cast<int>(N - t0 < 256 ? N - t0 : 256) * bins;
    for (int i = threadIdx.x; i < n; i += 256) cnt[t0 * bins + i] = own[i / bins * row + i % bins];
}

// Per tile: layout-order exclusive scan of the padded segment sizes, from counts
// in `bins` parts, 2^fine of them to a part here.  The tile's counts, one
// contiguous piece of cnt, are summed per (part, trial) in LDS (dynamic, [P][Tk])
// and scanned there.
__global__ __launch_bounds__(256) void tile_scan_kernel(const int32_t* __restrict__ cnt, int bins, int fine, int64_t N,
                                                        int P, int T, uint32_t* __restrict__ seg_rel,
                                                        int64_t* __restrict__ tile_size) {
    __shared__ int64_t part_sum[256];
    extern __shared__ int32_t sizes[];
    const int64_t tile = blockIdx.x;
    const int64_t t0 = tile * T;
    const int Tk = static_cast<int>(N - t0 < T ? N - t0 : T);
    const int n = P * Tk;
    const int64_t base = tile * (static_cast<int64_t>(T) * P + 1);
    for (int j = threadIdx.x; j < n; j += 256) sizes[j] = 0;
    __syncthreads();
    constexpr int kAhead = 8;                       // counts loaded together
    for (int j0 = threadIdx.x; j0 < Tk * bins; j0 += 256 * kAhead) {
        int32_t v[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) v[k] = j0 + k * 256 < Tk * bins ? cnt[t0 * bins + j0 + k * 256] : 0;
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int j = j0 + k * 256, i = j / bins;
            if (j < Tk * bins) atomicAdd(&sizes[((j - i * bins) >> fine) * Tk + i], v[k]);
        }
    }
    __syncthreads();
    const int per = (n + 255) / 256;
    const int j0 = threadIdx.x * per;
    int64_t local = 0;
    for (int j = j0; j < j0 + per && j < n; ++j) local += (static_cast<int64_t>(sizes[j]) + 3) & ~int64_t(3);
    part_sum[threadIdx.x] = local;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        int64_t add = threadIdx.x >= off ? part_sum[threadIdx.x - off] : 0;
        __syncthreads();
        part_sum[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = part_sum[threadIdx.x] - local;
    for (int j = j0; j < j0 + per && j < n; ++j) {
        const int64_t size = (static_cast<int64_t>(sizes[j]) + 3) & ~int64_t(3);
        sizes[j] = static_cast<int32_t>(static_cast<uint32_t>(run));
        run += size;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += 256) seg_rel[base + j] = static_cast<uint32_t>(sizes[j]);
    if (threadIdx.x == 255) {
        seg_rel[base + n] = static_cast<uint32_t>(part_sum[255]);
        tile_size[tile] = part_sum[255];
    }
}

// tile sizes -> tile starts in place (each padded to kTileAlign IDs), one workgroup
__global__ __launch_bounds__(1024) void tile_starts_kernel(int64_t* __restrict__ v, int64_t n_tiles,
                                                           CreateResult* __restrict__ res) {
    __shared__ int64_t tsum[1024];
    const int64_t per = (n_tiles + 1023) / 1024;
    const int64_t j0 = static_cast<int64_t>(threadIdx.x) * per;
    int64_t local = 0;
    bool wide = false;
    for (int64_t j = j0; j < j0 + per && j < n_tiles; ++j) {
        wide |= v[j] >= (int64_t(1) << 31);
        local += (v[j] + kTileAlign - 1) & ~int64_t(kTileAlign - 1);
    }
    if (wide) atomicOr(&res->flags, kCreateWideTile);
    tsum[threadIdx.x] = local;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t add = static_cast<int>(threadIdx.x) >= off ? tsum[threadIdx.x - off] : 0;
        __syncthreads();
        tsum[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = tsum[threadIdx.x] - local;
    for (int64_t j = j0; j < j0 + per && j < n_tiles; ++j) {
        const int64_t size = (v[j] + kTileAlign - 1) & ~int64_t(kTileAlign - 1);
        v[j] = run;
        run += size;
    }
    if (threadIdx.x == 1023) {
        v[n_tiles] = tsum[1023];
        res->part_ids = tsum[1023];
    }
}

__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Scatter of each trial's IDs into its per-part segments of the tiled copy, one
// workgroup per `per` consecutive trials of a tile.  Inside a tile each part's
// segments of consecutive trials are consecutive, so the unit's segments of every
// part form one run per part, whole 16-byte chunks: the runs are staged in LDS and
// leave in 16-byte stores.  A trial's segment ends in sentinels up to four IDs.
// The unit that ends a tile fills the tile's padding, the last one the readable
// IDs after the copy.  A unit past the stage is scattered straight to the copy.
constexpr int kScatterStage32 = 9 * 1024;           // IDs: 36 KB
template <int kBits>
__global__ __launch_bounds__(kScatterThreads) void part_scatter_kernel(
    const int64_t* __restrict__ offsets, const uint32_t* __restrict__ ids, int64_t N, int P, int T, int per,
    int64_t first_unit, int64_t n_units, const uint32_t* __restrict__ seg_rel, const int64_t* __restrict__ tile_start,
    uint32_t* __restrict__ pids) {
    __shared__ __attribute__((aligned(16))) uint32_t stage[kScatterStage32];
    __shared__ uint32_t cursors[kScatterWaves][kMaxParts];
    __shared__ uint32_t seg[kMaxParts + 1];         // staged start of each part's run
    extern __shared__ uint32_t starts[];            // [P][per + 1] segment starts in the tile
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t n_tiles = (N + T - 1) / T;
    const int units = (T + per - 1) / per;
    const int64_t of_launch = scatter_unit_index(n_units);
    if (of_launch >= n_units) return;
    const int64_t unit = first_unit + of_launch;
    const int64_t tile = unit / units;
    const int64_t t0 = tile * T;
    const int Tk = static_cast<int>(N - t0 < T ? N - t0 : T);
    const int i0 = static_cast<int>(unit - tile * units) * per;
    const int n = min(per, Tk - i0);
    if (n <= 0) return;
    const int row = per + 1;
    const uint32_t* rel = seg_rel + tile * (static_cast<int64_t>(T) * P + 1);
    uint32_t* copy = pids + tile_start[tile];
    for (int j = threadIdx.x; j < P * row; j += kScatterThreads) {
        const int p = j / row, i = i0 + min(j - p * row, n);
        starts[j] = rel[static_cast<int64_t>(p) * Tk + i];          // i = Tk: the next part's first
    }
    if (i0 + n == Tk) {
        const int64_t tile_end = tile_start[tile + 1] + (tile + 1 == n_tiles ? kIdPad : 0);
        for (int64_t u = tile_start[tile] + rel[static_cast<int64_t>(P) * Tk] + threadIdx.x; u < tile_end;
             u += blockDim.x)
            pids[u] = kSentinel;
    }
    __syncthreads();
    if (w == 0) {
        const uint32_t size = lane < P ? starts[lane * row + n] - starts[lane * row] : 0u;
        uint64_t inc = size;
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        const uint32_t at = static_cast<uint32_t>(min<uint64_t>(inc, kSentinel));
        if (lane < P) seg[lane] = at - size;
        if (lane == P - 1) seg[P] = at;
    }
    __syncthreads();
    if (seg[P] > static_cast<uint32_t>(kScatterStage32)) {
        int64_t* big = reinterpret_cast<int64_t*>(stage) + w * kMaxParts;      // the stage holds the cursors
        const int n_bits = P > 1 ? 32 - __builtin_clz(static_cast<uint32_t>(P - 1)) : 0;
        for (int i = w; i < n; i += kScatterWaves) {
            if (lane < P) big[lane] = starts[lane * row + i];
            __builtin_amdgcn_wave_barrier();
            scatter_trial_direct(ids, offsets[t0 + i0 + i], offsets[t0 + i0 + i + 1], kPartShift, n_bits, big, copy);
            __builtin_amdgcn_wave_barrier();
            if (lane < P)
                for (int64_t u = big[lane]; u < starts[lane * row + i + 1]; ++u) copy[u] = kSentinel;
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
    uint32_t* cur = cursors[w];
    scatter_unit<kBits>(
        offsets, ids, t0 + i0, n, kPartShift, cur, stage,
        [&](int i) {
            if (lane < P) cur[lane] = seg[lane] + (starts[lane * row + i] - starts[lane * row]);
        },
        [&](int i) {
            if (lane < P)
                for (uint32_t u = cur[lane]; u < seg[lane] + (starts[lane * row + i + 1] - starts[lane * row]); ++u)
                    stage[u] = kSentinel;
        });
    __syncthreads();
    // a run per group of 16, 32 or 64 lanes
    const int lanes = P > 16 ? 16 : (P > 8 ? 32 : 64);
    for (int p = threadIdx.x / lanes; p < P; p += kScatterThreads / lanes) {
        uint32_t* dst = copy + starts[p * row];
        const uint32_t s0 = seg[p], n_ids = seg[p + 1] - s0;
        for (uint32_t u = (threadIdx.x % lanes) * 4; u < n_ids; u += lanes * 4)
            *reinterpret_cast<u32x4*>(dst + u) = *reinterpret_cast<const u32x4*>(stage + s0 + u);
    }
}

// ---------------------------------------------------------------------------
// per-request part images
// ---------------------------------------------------------------------------

// one workgroup (256 threads) per superblock of 4096 catalogue events:
// bitmap words, per-128 ranks inside the superblock, superblock count
__global__ __launch_bounds__(256) void part_image_kernel(const double* __restrict__ o, int64_t C,
                                                         uint8_t* __restrict__ img, uint32_t* __restrict__ sb_count,
                                                         int64_t o_stride, int64_t img_stride, int64_t sb_stride) {
    __shared__ uint32_t wc[64];
    o += blockIdx.y * o_stride;
    img += blockIdx.y * img_stride;
    sb_count += blockIdx.y * sb_stride;
    const int64_t sb = blockIdx.x;
    const int64_t e0 = sb * kSuper;
    const int64_t part = e0 >> kPartShift;
    const int ls = static_cast<int>((e0 & (kPartSize - 1)) >> kSuperShift);
    uint64_t* bm = reinterpret_cast<uint64_t*>(img + part * kImgBytes);
    uint16_t* r16 = reinterpret_cast<uint16_t*>(img + part * kImgBytes + int64_t(kWords) * 8);
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    for (int k = 0; k < 16; ++k) {
        const int word = w * 16 + k;                       // 0..63 inside the superblock
        const int64_t E = e0 + word * 64 + lane;
        const bool nz = E < C && o[E] != 0.0;
        const uint64_t bits = __ballot(nz);
        if (lane == 0) {
            bm[ls * 64 + word] = bits;
            wc[word] = __popcll(bits);
        }
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        uint32_t before = 0;
        for (int b = 0; b < static_cast<int>(threadIdx.x); ++b) before += wc[2 * b] + wc[2 * b + 1];
        r16[ls * 32 + threadIdx.x] = static_cast<uint16_t>(before);
    }
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int k = 0; k < 64; ++k) total += wc[k];
        sb_count[sb] = total;
    }
}

// The fold and the part images in one pass: one workgroup (eight waves) per
// superblock of 4096 catalogue events.  The superblock's ELT-combined losses
// y are summed in LDS from the sparse pool: for each ELT of the layer, in
// layer order, the chunk's nonzero entries (distinct events) each add their
// per-ELT net loss.  An absent loss adds +0.0 (retentions are >= 0), which
// leaves y unchanged, so y is bit-identical to summing every ELT's dense row in
// layer order.  The kernel is a chain of memory and LDS latencies: pieces of an
// ELT's entries, one per thread, are read kFoldAhead ahead, also over the ELTs'
// ends, and a barrier separates the ELTs.  Then o, the bitmap words, the per-128
// ranks and the superblock count are written, and the superblock's nonzero o,
// packed in event order, go to its 4096-value slot of `stage`.  Against staging a
// round of the ELTs' joined entries in LDS, from which each wave sums its own
// 512 events: 16 ELTs over 2e6 events, 41 entries per ELT and superblock, 13.9 us
// both; 12 layers of up to 32 such ELTs 108 -> 71 us; 9 layers of 24 with 82
// entries 44 -> 29 us; 30 ELTs of 246 entries 23 -> 14.5 us; 27 of 834 79 -> 20 us.
// 256 threads take 18 and 29 us for the last two, 34 us instead of 36 per batch of
// the 12 layers.
constexpr int kFoldThreads = 512;
constexpr int kFoldWaves = kFoldThreads / 64;
constexpr int kFoldAhead = 4;                       // pieces of entries in flight
struct FoldOut {
    double* o;                      // dense o, or null
    uint8_t* img;
    uint32_t* sb_count;
    double* stage;
    // the time-ordered passes' lookup tables, or null: a probe word per 32
    // events (bits of o != 0 in the low half, the stage index of the word's
    // first nonzero event in the high half) and a coarse map of one bit per
    // 2^cshift events (null also where one of its words spans superblocks)
    uint64_t* probe;
    uint32_t* coarse;
    int cshift;
    FoldBack back;                  // back
    const uint64_t* slots;          // losses: the pool's events (LossIndex::probe) and the table by slot
    double* tab;
};

// OR of each pair of adjacent bits, packed into the low half
__device__ __forceinline__ uint32_t or_pairs(uint32_t x) {
    x = (x | (x >> 1)) & 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0x0000FFFFu;
}

enum class FoldKind { images, back, losses };
template <FoldKind kKind>
__device__ __forceinline__ void fold_image_body(const SparsePool& sp, int64_t C, const LayerArgs& L,
                                                const FoldOut& out) {
    constexpr bool kBack = kKind == FoldKind::back, kLosses = kKind == FoldKind::losses;
    double* __restrict__ o = out.o;
    uint8_t* __restrict__ img = out.img;
    uint32_t* __restrict__ sb_count = out.sb_count;
    double* __restrict__ stage = out.stage;
    constexpr int kOwn = kSuper / kFoldWaves;       // events a wave sums
    constexpr int kWordsOwn = kOwn / 64;
    __shared__ __attribute__((aligned(16))) double ys[kSuper];
    __shared__ uint64_t wb[64];
    const int64_t sb = blockIdx.x;
    const int64_t e0 = sb * kSuper;
    const int64_t part = e0 >> kPartShift;
    const int ls = static_cast<int>((e0 & (kPartSize - 1)) >> kSuperShift);
    uint64_t* bm = reinterpret_cast<uint64_t*>(img + part * kImgBytes);
    uint16_t* r16 = reinterpret_cast<uint16_t*>(img + part * kImgBytes + int64_t(kWords) * 8);
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    // lane j: ELT j's entries of this chunk in the pool and its terms (J <= kMaxJ <= 64)
    const int J = sb < sp.n_chunks ? L.J : 0;
    int64_t pool_at = 0;
    int cnt = 0;
    double R = 0.0, Lim = 0.0;
    if (lane < J) {
        const int64_t key = static_cast<int64_t>(L.idx[lane]) * sp.n_chunks + sb;
        R = L.R[lane];
        Lim = L.Lim[lane];
        pool_at = sp.chunk_off[key];
        cnt = static_cast<int>(sp.chunk_off[key + 1] - pool_at);      // <= 4096
    }
    {
        u64x2* own = reinterpret_cast<u64x2*>(ys + w * kOwn);
        for (int i = lane; i < kOwn / 2; i += 64) own[i] = u64x2{0, 0};
    }
    uint64_t slots = 0;                             // lane i < 16: the wave's i-th 32 events
    if constexpr (kLosses) {
        const int64_t i = (e0 >> 5) + w * (kOwn / 32) + lane;
        if (lane < kOwn / 32 && i < (C + 31) / 32) slots = out.slots[i];
    }
    uint64_t left = __ballot(cnt > 0);              // ELTs with entries that are not begun
    int pj = -1, pi = 0, pn = 0;                    // the last piece fetched: ELT, first entry, the ELT's entries
    int64_t pat = 0;
    int qj[kFoldAhead], qi[kFoldAhead], qn[kFoldAhead];
    int qe[kFoldAhead];
    double qv[kFoldAhead];
    auto fetch = [&](int u) {
        pi += kFoldThreads;
        if (pi >= pn) {
            pi = 0;
            pj = left ? __builtin_ctzll(left) : -1;
            pn = left ? __builtin_amdgcn_readlane(cnt, pj & 63) : 0;
            pat = static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(pool_at), pj & 63));
            left &= left - 1;
        }
        qj[u] = pj;
        qi[u] = pi;
        qn[u] = pn;
        const int i = pi + static_cast<int>(threadIdx.x);
        qe[u] = 0;
        qv[u] = 0.0;
        if (i < pn) {
            qe[u] = sp.ev[pat + i];
            qv[u] = sp.val[pat + i];
        }
    };
#pragma unroll
    for (int u = 0; u < kFoldAhead; ++u) fetch(u);
    for (bool more = true; more;) {
#pragma unroll
        for (int u = 0; u < kFoldAhead; ++u) {
            const int j = qj[u], i = qi[u] + static_cast<int>(threadIdx.x), n = qn[u];
            const int e = qe[u];
            const double v = qv[u];
            const bool first = qi[u] == 0;
            if (j < 0) {
                more = false;
                break;
            }
            fetch(u);
            if (first) __syncthreads();             // the ELT before is added (the first: the zeros are set)
            if (i < n) ys[e] = ys[e] + apply_terms(v, readlane_f64(R, j), readlane_f64(Lim, j));
        }
    }
    __syncthreads();
    const int64_t eb = e0 + static_cast<int64_t>(w) * kOwn + lane;      // event of word 0 of this wave
    double vk[kWordsOwn];
    uint64_t bk[kWordsOwn];
#pragma unroll
    for (int k = 0; k < kWordsOwn; ++k) {
        const int64_t E = eb + k * 64;
        const double y = ys[w * kOwn + k * 64 + lane];
        const double v = apply_terms(y, L.occR, L.occL);
        if (o && E < C) o[E] = v;
        if (kBack && E < C) {
            const double to = y - L.occR;
            out.back.band[E] = to > L.occL ? 2 : (to > 0.0 && to < L.occL ? 1 : 0);
            out.back.w_mean[E] = 0;
            out.back.w_tvar[E] = 0;
        }
        if constexpr (kLosses) {
            // an event's slot in its part's table, also where the layer has no loss
            const uint64_t a = readlane_u64(slots, 2 * k), b = readlane_u64(slots, 2 * k + 1);
            const uint64_t bits = (b << 32) | (a & 0xFFFFFFFFull);
            const uint32_t first = static_cast<uint32_t>(a >> 32);
            if ((bits >> lane) & 1ull)
                out.tab[static_cast<int64_t>(first >> 16) * kLossSlots + (first & 0xFFFFu) +
                        __popcll(bits & lanemask_lt())] = v;
            continue;
        }
        vk[k] = v;
        bk[k] = __ballot(E < C && v != 0.0);
        if (lane == 0) wb[w * kWordsOwn + k] = bk[k];
    }
    if constexpr (kLosses) return;
    __syncthreads();
    // lane i: bitmap word i and the nonzero events before it, in every wave
    const uint64_t word = wb[lane];
    int before = __popcll(word);
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(before, off, kWave);
        if (lane >= off) before += v;
    }
    const int total = __builtin_amdgcn_readlane(before, 63);
    before -= __popcll(word);
    if (kBack && !img) return;                      // no passes over the images
    if (w == 0) {
        bm[ls * 64 + lane] = word;
        if ((lane & 1) == 0) r16[ls * 32 + (lane >> 1)] = static_cast<uint16_t>(before);
        if (lane == 0) sb_count[sb] = static_cast<uint32_t>(total);
    }
    if (out.probe && w == 1) {
        const uint32_t first = static_cast<uint32_t>(e0) + static_cast<uint32_t>(before);
        const int64_t i = (e0 >> 5) + 2 * lane;
        const int64_t n_words = (C + 31) >> 5;
        const uint32_t low = static_cast<uint32_t>(word);
        if (i < n_words) out.probe[i] = (static_cast<uint64_t>(first) << 32) | low;
        if (i + 1 < n_words)
            out.probe[i + 1] = (static_cast<uint64_t>(first + __popc(low)) << 32) | static_cast<uint32_t>(word >> 32);
    }
    if (out.coarse && static_cast<int>(threadIdx.x) < (128 >> out.cshift)) {
        // coarse word i of the superblock covers 2^cshift of its 32-event pieces
        const int s = out.cshift;
        const uint32_t* piece = reinterpret_cast<const uint32_t*>(wb) + (threadIdx.x << s);
        uint32_t m = 0;
        for (int j = 0; j < (1 << s); ++j) {
            uint32_t x = piece[j];
            if (s <= 5) {
                for (int k = 0; k < s; ++k) x = or_pairs(x);
                m |= x << (j * (32 >> s));
            } else {
                m |= (x ? 1u : 0u) << (j >> (s - 5));
            }
        }
        const int64_t i = (e0 >> (5 + s)) + threadIdx.x;
        if ((i << (5 + s)) < C) out.coarse[i] = m;
    }
    // the nonzero o packed in event order
    double* dst = stage + sb * kSuper;
#pragma unroll
    for (int k = 0; k < kWordsOwn; ++k) {
        const int at = __builtin_amdgcn_readlane(before, w * kWordsOwn + k);
        if ((bk[k] >> lane) & 1ull) dst[at + __popcll(bk[k] & lanemask_lt())] = vk[k];
    }
}

// terms as kernel arguments (eager runs) or read from device memory (graph
// replays, whose terms may change between replays)
__global__ __launch_bounds__(kFoldThreads) void fold_image_kernel(SparsePool sp, int64_t C, LayerArgs L, FoldOut out) {
    fold_image_body<FoldKind::images>(sp, C, L, out);
}
__global__ __launch_bounds__(kFoldThreads) void fold_back_kernel(SparsePool sp, int64_t C, LayerArgs L, FoldOut out) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < out.back.n_acc; i += blockDim.x) out.back.acc[i] = 0;
    fold_image_body<FoldKind::back>(sp, C, L, out);
}
// layer blockIdx.y of several
__global__ __launch_bounds__(kFoldThreads) void fold_image_dev_kernel(SparsePool sp, int64_t C,
                                                                      const LayerArgs* __restrict__ L, FoldOut out,
                                                                      int64_t img_stride, int64_t sb_stride) {
    out.img += blockIdx.y * img_stride;
    out.sb_count += blockIdx.y * sb_stride;
    out.stage += blockIdx.y * sb_stride * kSuper;
    fold_image_body<FoldKind::images>(sp, C, L[blockIdx.y], out);
}
// the tables by slot of one layer, or of layer blockIdx.y
__global__ __launch_bounds__(kFoldThreads) void fold_losses_kernel(SparsePool sp, int64_t C, LayerArgs L, FoldOut out) {
    fold_image_body<FoldKind::losses>(sp, C, L, out);
}
__global__ __launch_bounds__(kFoldThreads) void fold_losses_dev_kernel(SparsePool sp, int64_t C,
                                                                       const LayerArgs* __restrict__ L, FoldOut out,
                                                                       int64_t tab_stride) {
    out.tab += blockIdx.y * tab_stride;
    fold_image_body<FoldKind::losses>(sp, C, L[blockIdx.y], out);
}

// Layer arguments packed into kernel arguments (which take 4 KB): per layer the
// fixed fields, then its J indices (padded to whole doubles), retentions and limits
constexpr int kTermsHead = static_cast<int>(offsetof(LayerArgs, idx) / 4);
constexpr int kTermsLayers = 16;
struct TermsPack {
    uint32_t words[864];
    int32_t start[kTermsLayers];
};
static_assert(sizeof(TermsPack) <= 3600 && kTermsHead + 5 * kMaxJ <= 864, "layer arguments as kernel arguments");
__host__ __device__ constexpr int terms_words(int J) { return kTermsHead + ((J + 1) & ~1) + 4 * J; }

// one workgroup per layer of the pack
__global__ __launch_bounds__(256) void store_terms_kernel(TermsPack p, LayerArgs* __restrict__ dst) {
    const uint32_t* src = p.words + p.start[blockIdx.x];
    uint32_t* d = reinterpret_cast<uint32_t*>(dst + blockIdx.x);
    const int J = static_cast<int>(src[0]), Je = (J + 1) & ~1;
    for (int i = threadIdx.x; i < terms_words(J); i += blockDim.x) {
        int at = i;                                     // head and indices lie as in LayerArgs
        if (i >= kTermsHead + Je) {
            const int k = i - kTermsHead - Je;
            at = k < 2 * J ? static_cast<int>(offsetof(LayerArgs, R) / 4) + k
                           : static_cast<int>(offsetof(LayerArgs, Lim) / 4) + k - 2 * J;
        }
        d[at] = src[i];
    }
}

// After the fold: each superblock's global rank (the nonzero count of the
// superblocks before it, summed by its own workgroup) goes to its part's base
// table, and its packed nonzero o to compact[rank], one workgroup per superblock
__global__ __launch_bounds__(256) void compact_stage_kernel(const double* __restrict__ stage,
                                                            const uint32_t* __restrict__ sb_count,
                                                            uint8_t* __restrict__ img, double* __restrict__ compact) {
    __shared__ uint32_t wsum[4];
    const int64_t sb = blockIdx.x;
    uint32_t before = 0;
    for (int64_t i = threadIdx.x; i < sb; i += blockDim.x) before += sb_count[i];
    for (int off = 32; off >= 1; off >>= 1) before += __shfl_xor(before, off, kWave);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = before;
    __syncthreads();
    const uint32_t base = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    if (threadIdx.x == 0) {
        const int64_t part = sb / kBase32;
        uint32_t* b32 = reinterpret_cast<uint32_t*>(img + part * kImgBytes + int64_t(kWords) * 8 +
                                                    int64_t(kRank16) * 2);
        b32[sb % kBase32] = base;
    }
    const uint32_t n = sb_count[sb];
    const double* src = stage + sb * kSuper;
    for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) compact[static_cast<int64_t>(base) + k] = src[k];
}

// ---------------------------------------------------------------------------
// the sparse pool (built once, when the tables are created)
// ---------------------------------------------------------------------------

// nonzero count of every (row, 4096-event chunk); grid (n_chunks, n_rows)
__global__ __launch_bounds__(256) void sparse_count_kernel(const double* __restrict__ elts, int64_t C,
                                                           int64_t n_chunks, int64_t* __restrict__ counts) {
    __shared__ uint32_t wsum[4];
    const int64_t row = blockIdx.y, chunk = blockIdx.x;
    const double* r = elts + row * C;
    const int64_t e0 = chunk * kSuper;
    uint32_t cnt = 0;
    for (int k = 0; k < kSuper / 256; ++k) {
        const int64_t E = e0 + k * 256 + threadIdx.x;
        cnt += (E < C && __builtin_nontemporal_load(r + E) != 0.0) ? 1u : 0u;
    }
    for (int off = 32; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) counts[row * n_chunks + chunk] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

constexpr int kScanChunk = 16384;

// the sums of chunks of kScanChunk entries
__global__ __launch_bounds__(1024) void chunk_sum_kernel(const int64_t* __restrict__ v, int64_t n,
                                                         int64_t* __restrict__ sums) {
    __shared__ int64_t wsum[16];
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kScanChunk;
    int64_t own = 0;
    for (int k = threadIdx.x; k < kScanChunk; k += 1024)
        if (c0 + k < n) own += v[c0 + k];
    for (int off = 32; off >= 1; off >>= 1) own += __shfl_xor(own, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = own;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t total = 0;
        for (int w = 0; w < 16; ++w) total += wsum[w];
        sums[blockIdx.x] = total;
    }
}

// exclusive scan of n counts in place, the total at [n]: each workgroup takes `per`
// entries in rounds, from[blockIdx.x] before them (0 where `from` is null)
__global__ __launch_bounds__(1024) void sparse_scan_kernel(int64_t* __restrict__ v, int64_t n,
                                                           const int64_t* __restrict__ from, int64_t per) {
    constexpr int kPer = kScanChunk / 1024;         // entries of a thread and round
    __shared__ int64_t wsum[16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t carry = from ? from[blockIdx.x] : 0;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * per, last = min(n, first + per);
    for (int64_t c0 = first; c0 < last; c0 += kScanChunk) {
        const int64_t i0 = c0 + static_cast<int64_t>(threadIdx.x) * kPer;
        int64_t x[kPer], own = 0;
        // two entries a load, as the arrays start on 16 bytes (10000 entries 13 -> 7.6 us)
        const bool whole = i0 + kPer <= n;
        if (whole) {
#pragma unroll
            for (int k = 0; k < kPer / 2; ++k) {
                const u64x2 two = reinterpret_cast<const u64x2*>(v + i0)[k];
                x[2 * k] = static_cast<int64_t>(two.x);
                x[2 * k + 1] = static_cast<int64_t>(two.y);
            }
        } else {
#pragma unroll
            for (int k = 0; k < kPer; ++k) x[k] = i0 + k < n ? v[i0 + k] : 0;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) own += x[k];
        int64_t inc = own;                          // inclusive over the wave
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t add = __shfl_up(inc, off, 64);
            if (lane >= off) inc += add;
        }
        if (lane == 63) wsum[wv] = inc;
        __syncthreads();
        int64_t at = carry + inc - own;
        for (int w = 0; w < 16; ++w) {
            if (w < wv) at += wsum[w];
            carry += wsum[w];
        }
#pragma unroll
        for (int k = 0; k < kPer; k += 2) {
            const u64x2 two{static_cast<uint64_t>(at), static_cast<uint64_t>(at + x[k])};
            if (whole) {
                *reinterpret_cast<u64x2*>(v + i0 + k) = two;
            } else {
                if (i0 + k < n) v[i0 + k] = static_cast<int64_t>(two.x);
                if (i0 + k + 1 < n) v[i0 + k + 1] = static_cast<int64_t>(two.y);
            }
            at += x[k] + x[k + 1];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0 && last == n) v[n] = carry;
}

// each chunk's nonzero entries, in event order, at its offset; grid (n_chunks, n_rows)
__global__ __launch_bounds__(256) void sparse_fill_kernel(const double* __restrict__ elts, int64_t C,
                                                          int64_t n_chunks, const int64_t* __restrict__ off,
                                                          uint16_t* __restrict__ ev, double* __restrict__ val) {
    __shared__ uint32_t wsum[4];
    const int64_t row = blockIdx.y, chunk = blockIdx.x;
    const double* r = elts + row * C;
    const int64_t e0 = chunk * kSuper;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t at = off[row * n_chunks + chunk];
    for (int k = 0; k < kSuper / 256; ++k) {
        const int local = k * 256 + static_cast<int>(threadIdx.x);
        const int64_t E = e0 + local;
        const double x = E < C ? r[E] : 0.0;
        const uint64_t bal = __ballot(x != 0.0);
        if (lane == 0) wsum[w] = __popcll(bal);
        __syncthreads();
        uint32_t before = 0;
        for (int i = 0; i < w; ++i) before += wsum[i];
        const uint32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        if (x != 0.0) {
            const int64_t pos = at + before + __popcll(bal & lanemask_lt());
            ev[pos] = static_cast<uint16_t>(local);
            val[pos] = x;
        }
        at += total;
        __syncthreads();
    }
}

// exclusive scan of the superblock counts (one workgroup) into each part's
// base32 table
__global__ __launch_bounds__(1024) void superblock_scan_kernel(const uint32_t* __restrict__ sb_count, int64_t n_sb,
                                                               uint8_t* __restrict__ img, int64_t img_stride) {
    __shared__ uint64_t s[1024];
    sb_count += blockIdx.y * n_sb;
    img += blockIdx.y * img_stride;
    uint64_t carry = 0;
    for (int64_t c0 = 0; c0 < n_sb; c0 += 1024) {
        const int64_t i = c0 + threadIdx.x;
        const uint64_t v = i < n_sb ? sb_count[i] : 0;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {
            uint64_t add = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < n_sb) {
            const int64_t part = i / kBase32;
            const int ls = static_cast<int>(i % kBase32);
            uint32_t* b32 = reinterpret_cast<uint32_t*>(img + part * kImgBytes + int64_t(kWords) * 8 +
                                                        int64_t(kRank16) * 2);
            b32[ls] = static_cast<uint32_t>(carry + s[threadIdx.x] - v);
        }
        const uint64_t total = s[1023];
        __syncthreads();
        carry += total;
    }
}

// nonzero o(E) to compact[rank(E)], one workgroup per superblock
__global__ __launch_bounds__(256) void compact_kernel(const double* __restrict__ o, int64_t C,
                                                      const uint8_t* __restrict__ img, double* __restrict__ compact,
                                                      int64_t o_stride, int64_t img_stride) {
    __shared__ uint32_t pre[64];
    o += blockIdx.y * o_stride;
    img += blockIdx.y * img_stride;
    compact += blockIdx.y * o_stride;
    const int64_t sb = blockIdx.x;
    const int64_t e0 = sb * kSuper;
    const int64_t part = e0 >> kPartShift;
    const int ls = static_cast<int>((e0 & (kPartSize - 1)) >> kSuperShift);
    const uint64_t* bm = reinterpret_cast<const uint64_t*>(img + part * kImgBytes);
    const uint32_t* b32 = reinterpret_cast<const uint32_t*>(img + part * kImgBytes + int64_t(kWords) * 8 +
                                                            int64_t(kRank16) * 2);
    if (threadIdx.x == 0) {
        uint32_t run = b32[ls];
        for (int k = 0; k < 64; ++k) {
            pre[k] = run;
            run += __popcll(bm[ls * 64 + k]);
        }
    }
    __syncthreads();
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    for (int k = 0; k < 16; ++k) {
        const int word = w * 16 + k;
        const int64_t E = e0 + word * 64 + lane;
        const uint64_t bits = bm[ls * 64 + word];
        if ((bits >> lane) & 1ull) compact[pre[word] + __popcll(bits & lanemask_lt())] = o[E];
    }
}

// ---------------------------------------------------------------------------
// the partitioned trial pass
// ---------------------------------------------------------------------------

// LDS state of one workgroup of the partitioned pass
struct PassLds {
    uint64_t bm[kWords];
    uint16_t r16[kRank16];
    uint32_t b32[kBase32];
    double acc_hi[kTileMax];
    double acc_lo[kTileMax];
    int64_t tile;
    int32_t item;
};

// One (layer, tile): every part image in turn, every trial of the tile inside
// [t_lo, t_hi); writes YLT (and S) for those trials.  All threads of the
// workgroup call it; it starts and ends with a barrier.
template <int LPT>
__device__ __forceinline__ void pass_tile(PassLds& sh, const uint32_t* __restrict__ pids,
                                          const uint32_t* __restrict__ seg_rel,
                                          const int64_t* __restrict__ tile_start, const uint8_t* __restrict__ img,
                                          const double* __restrict__ compact, int64_t N, int P, int T, int64_t tile,
                                          int64_t t_lo, int64_t t_hi, double aggR, double aggL,
                                          double* __restrict__ ylt, double* __restrict__ S_out) {
    static_assert(LPT == 8 || LPT == 16 || LPT == 32 || LPT == 64, "lanes per trial");
    const int lig = threadIdx.x & (LPT - 1);                   // lane in its group
    const int slot = threadIdx.x / LPT;                        // group index in the workgroup
    const int n_slots = blockDim.x / LPT;
    const int64_t t0 = tile * T;
    const int Tk = static_cast<int>(N - t0 < T ? N - t0 : T);
    const int64_t sbase = tile * (static_cast<int64_t>(T) * P + 1);
    const uint32_t* tids = pids + tile_start[tile];
    for (int i = threadIdx.x; i < Tk; i += blockDim.x) {
        sh.acc_hi[i] = 0.0;
        sh.acc_lo[i] = 0.0;
    }
    for (int p = 0; p < P; ++p) {
        __syncthreads();
        {
            const u32x4* src = reinterpret_cast<const u32x4*>(img + p * kImgBytes);
            u32x4* dst_bm = reinterpret_cast<u32x4*>(sh.bm);
            for (int k = threadIdx.x; k < kWords / 2; k += blockDim.x) dst_bm[k] = src[k];
            const u32x4* src_r = src + kWords / 2;
            u32x4* dst_r = reinterpret_cast<u32x4*>(sh.r16);
            for (int k = threadIdx.x; k < kRank16 / 8; k += blockDim.x) dst_r[k] = src_r[k];
            const u32x4* src_b = src_r + kRank16 / 8;
            u32x4* dst_b = reinterpret_cast<u32x4*>(sh.b32);
            for (int k = threadIdx.x; k < kBase32 / 4; k += blockDim.x) dst_b[k] = src_b[k];
        }
        __syncthreads();
        const uint32_t pbase = static_cast<uint32_t>(static_cast<int64_t>(p) << kPartShift);
        // A group walks its trials' segments of this part in batches of
        // LPT*4*kU IDs; the loads of the next batch are issued before the
        // current batch is looked up, so HBM latency overlaps the LDS tests,
        // the gathers and the sums.  Trials outside [t_lo, t_hi) have empty
        // segments.
        constexpr int kU = 4;
        constexpr uint32_t kBatch = LPT * 4 * kU;
        auto seg = [&](int i, uint32_t& sb, uint32_t& se) {
            const int64_t t = t0 + i;
            sb = seg_rel[sbase + static_cast<int64_t>(p) * Tk + i];
            se = (t < t_lo || t >= t_hi) ? sb : seg_rel[sbase + static_cast<int64_t>(p) * Tk + i + 1];
        };
        auto load_batch = [&](uint32_t c, uint32_t e, u32x4* v) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t cu = c + lig * 4 + u * LPT * 4;
                v[u] = cu < e ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tids + cu))
                              : u32x4{kSentinel, kSentinel, kSentinel, kSentinel};
            }
        };
        int i = slot;
        uint32_t cs = 0, ce = 0, c = 0;
        u32x4 cur[kU], nxt[kU];
        if (i < Tk) {
            seg(i, cs, ce);
            c = cs;
            load_batch(c, ce, cur);
        }
        double hi = 0.0, lo = 0.0;
        while (i < Tk) {
            // coordinates of the next batch: the rest of this segment, or the
            // group's next trial
            int ni = i;
            uint32_t ns = cs, ne = ce, nc = c + kBatch;
            if (nc >= ce) {
                ni = i + n_slots;
                if (ni < Tk) {
                    seg(ni, ns, ne);
                    nc = ns;
                }
            }
            if (ni < Tk) load_batch(nc, ne, nxt);
            uint32_t r[kU * 4];
#pragma unroll
            for (int k = 0; k < kU * 4; ++k) {
                const uint32_t el = cur[k >> 2][k & 3] - pbase;   // sentinel and foreign IDs fail the test
                r[k] = 0xFFFFFFFFu;
                if (el < static_cast<uint32_t>(kPartSize)) {
                    const uint64_t word = sh.bm[el >> 6];
                    if ((word >> (el & 63)) & 1ull) {
                        uint32_t rk = sh.b32[el >> kSuperShift] + sh.r16[el >> 7];
                        if ((el >> 6) & 1) rk += __popcll(sh.bm[(el >> 6) - 1]);
                        r[k] = rk + __popcll(word & ((1ull << (el & 63)) - 1ull));
                    }
                }
            }
            double val[kU * 4];
#pragma unroll
            for (int k = 0; k < kU * 4; ++k) val[k] = compact[r[k] == 0xFFFFFFFFu ? 0u : r[k]];
#pragma unroll
            for (int k = 0; k < kU * 4; ++k) dd_add(hi, lo, r[k] == 0xFFFFFFFFu ? 0.0 : val[k]);
            if (ni != i) {
                // the trial's segment is done: group total into its accumulator
                group_reduce_dd(hi, lo, LPT);
                if (lig == 0) {
                    double h = sh.acc_hi[i], l = sh.acc_lo[i];
                    dd_merge(h, l, hi, lo);
                    sh.acc_hi[i] = h;
                    sh.acc_lo[i] = l;
                }
                hi = 0.0;
                lo = 0.0;
            }
            i = ni;
            cs = ns;
            ce = ne;
            c = nc;
#pragma unroll
            for (int u = 0; u < kU; ++u) cur[u] = nxt[u];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < Tk; i += blockDim.x) {
        const int64_t t = t0 + i;
        if (t < t_lo || t >= t_hi) continue;
        const double S = sh.acc_hi[i] + sh.acc_lo[i];
        ylt[t - t_lo] = apply_terms(S, aggR, aggL);
        if (S_out) S_out[t - t_lo] = S;
    }
    __syncthreads();
}

template <int LPT>
__global__ __launch_bounds__(512) void part_pass_kernel(PartPassArgs a) {
    __shared__ __attribute__((aligned(16))) PassLds sh;
    for (;;) {
        if (threadIdx.x == 0) sh.tile = a.first_tile + atomicAdd(a.tile_counter, 1u);
        __syncthreads();
        const int64_t tile = sh.tile;
        if (tile >= a.last_tile) break;
        pass_tile<LPT>(sh, a.pids, a.seg_rel, a.tile_start, a.img, a.compact, a.N, a.P, a.T, tile, a.t_lo,
                       a.t_hi, a.aggR, a.aggL, a.ylt, a.S);
    }
}

// The persistent multi-layer pass: one grid drains a work list of
// (layer, tile) items, ordered by decreasing cost, through an atomic counter.
template <int LPT>
__global__ __launch_bounds__(512) void batched_pass_kernel(BatchedPassArgs a) {
    __shared__ __attribute__((aligned(16))) PassLds sh;
    for (;;) {
        if (threadIdx.x == 0) sh.item = static_cast<int32_t>(atomicAdd(a.item_counter, 1u));
        __syncthreads();
        const int32_t it = sh.item;
        if (it >= a.n_items) break;
        const int2 w = a.items[it];
        const BatchLayerDesc d = a.layers[w.x];
        pass_tile<LPT>(sh, a.pids, a.seg_rel, a.tile_start, a.img + w.x * a.img_stride, a.compact + w.x * a.C,
                       a.N, a.P, a.T, w.y, d.t_lo, d.t_hi, d.aggR, d.aggL, a.ylt + d.out_off, nullptr);
    }
}

// per-layer fold for a batch: o[l][E], ELT terms from device tables
__global__ __launch_bounds__(256) void batched_fold_kernel(const double* __restrict__ elts, int64_t C,
                                                           const BatchFoldDesc* __restrict__ fd,
                                                           const int32_t* __restrict__ idx,
                                                           const double* __restrict__ R,
                                                           const double* __restrict__ Lim, double* __restrict__ o) {
    const int l = blockIdx.y;
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= C) return;
    const BatchFoldDesc d = fd[l];
    double y = 0.0;
    for (int j = 0; j < d.J; ++j) {
        const int k = d.off + j;
        y = y + apply_terms(elts[static_cast<int64_t>(idx[k]) * C + e], R[k], Lim[k]);
    }
    o[static_cast<int64_t>(l) * C + e] = apply_terms(y, d.occR, d.occL);
}

// Backward histogram over the partitioned layout: for every trial inside the
// aggregate band, every occurrence whose event has a movable occurrence loss
// (bit set in the part bitmap) adds 1 to W_mean[E] and the trial's TVaR weight
// to W_tvar[E].  Integer atomics: the histogram does not depend on order.
__global__ __launch_bounds__(512) void part_adjoint_kernel(PartAdjArgs a) {
    __shared__ __attribute__((aligned(16))) uint64_t bm[kWords];
    __shared__ int64_t s_tile;
    const int lane = threadIdx.x & 63;
    const int lig = lane & 15;
    const int slot = (threadIdx.x >> 6) * 4 + (lane >> 4);
    const int P = a.P;
    const TailStats ts = *a.tail;
    for (;;) {
        if (threadIdx.x == 0) s_tile = a.first_tile + atomicAdd(a.tile_counter, 1u);
        __syncthreads();
        const int64_t tile = s_tile;
        if (tile >= a.last_tile) break;
        const int64_t t0 = tile * a.T;
        const int Tk = static_cast<int>(a.N - t0 < a.T ? a.N - t0 : a.T);
        const int64_t sbase = tile * (static_cast<int64_t>(a.T) * P + 1);
        const uint32_t* tids = a.pids + a.tile_start[tile];
        for (int p = 0; p < P; ++p) {
            __syncthreads();
            {
                const u32x4* src = reinterpret_cast<const u32x4*>(a.img + p * kImgBytes);
                u32x4* dst = reinterpret_cast<u32x4*>(bm);
                for (int k = threadIdx.x; k < kWords / 2; k += blockDim.x) dst[k] = src[k];
            }
            __syncthreads();
            const uint32_t pbase = static_cast<uint32_t>(static_cast<int64_t>(p) << kPartShift);
            for (int i = slot; i < Tk; i += 32) {
                const int64_t t = t0 + i;
                if (t < a.t_lo || t >= a.t_hi) continue;
                const int64_t k = t - a.t_lo;
                const double ta = a.S[k] - a.aggR;
                if (!((ta > 0.0) && (ta < a.aggL))) continue;
                const uint64_t key = __double_as_longlong(a.ylt[k] + 0.0);
                const unsigned long long wt =
                    key > ts.v_bits ? ts.c_eq : (key == ts.v_bits ? ts.m - ts.c_gt : 0);
                const uint32_t s = a.seg_rel[sbase + static_cast<int64_t>(p) * Tk + i];
                const uint32_t e = a.seg_rel[sbase + static_cast<int64_t>(p) * Tk + i + 1];
                constexpr int kU = 4;
                for (uint32_t c = s + lig * 4; c < e; c += 64 * kU) {
                    u32x4 v[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const uint32_t cu = c + u * 64;
                        v[u] = cu < e ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tids + cu))
                                      : u32x4{kSentinel, kSentinel, kSentinel, kSentinel};
                    }
#pragma unroll
                    for (int k = 0; k < kU * 4; ++k) {
                        const uint32_t id = v[k >> 2][k & 3];
                        const uint32_t el = id - pbase;
                        if (el < static_cast<uint32_t>(kPartSize) && ((bm[el >> 6] >> (el & 63)) & 1ull)) {
                            atomicAdd(reinterpret_cast<unsigned long long*>(&a.w_mean[id]), 1ull);
                            if (wt) atomicAdd(reinterpret_cast<unsigned long long*>(&a.w_tvar[id]), wt);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
}

// Backward histogram, XCD-affine, for the same result as part_adjoint_kernel.
// Workgroups on XCD x serve the parts p = x (mod 8) as in the forward pass,
// each over a fixed share of the tiles, so a part's probe words (bitmap bits
// and part-relative ranks, built from the part image and its superblock
// counts) are loaded into LDS once.  An occurrence of a movable event in a
// trial inside the aggregate band counts 1 for W_mean: in an LDS counter
// when the event is among the part's first kCounts nonzero events (by rank),
// else with a global atomic; the LDS counters are added to W_mean once per
// part.  TVaR weights (tail trials only) use global atomics.  Each group of
// 16 lanes takes four trials of a tile at once, so their segments' loads are
// in flight together.  All counts are integers, so the order of the additions
// does not matter.  The LDS counters
// are 32-bit: the launcher uses this kernel only for layouts of fewer than
// 2^32 IDs, which bounds every count.
__global__ __launch_bounds__(1024) void xcd_adjoint_kernel(PartAdjArgs a, int n_xcd) {
    constexpr uint32_t kProbeWords = static_cast<uint32_t>(kPartSize >> 5);
    constexpr uint32_t kCounts = 24000;
    __shared__ uint64_t pw[kProbeWords];
    __shared__ uint32_t cnt[kCounts];
    __shared__ uint32_t sbb[kBase32];               // part-relative rank of each superblock's first event
    const int lane = threadIdx.x & 63;
    const int lig = lane & 15;
    const int slot = (threadIdx.x >> 6) * 4 + (lane >> 4);     // 64 groups of 16 lanes, one trial each
    const int n_slots = static_cast<int>(blockDim.x >> 4);
    const int P = a.P;
    const TailStats ts = *a.tail;
    const int x = static_cast<int>(blockIdx.x % n_xcd);
    const int r = static_cast<int>(blockIdx.x / n_xcd);
    const int nr = static_cast<int>(gridDim.x / n_xcd);
    int p0, pstep, srank, nserv;
    if (P >= n_xcd) {
        p0 = x;
        pstep = n_xcd;
        srank = r;
        nserv = nr;
    } else {
        p0 = x % P;
        pstep = P;
        srank = (x / P) * nr + r;
        nserv = ((n_xcd - 1 - p0) / P + 1) * nr;
    }
    const int64_t n_tiles = a.last_tile - a.first_tile;
    for (int p = p0; p < P; p += pstep) {
        const uint8_t* gimg = a.img + static_cast<int64_t>(p) * kImgBytes;
        const uint32_t* gbm = reinterpret_cast<const uint32_t*>(gimg);
        const uint16_t* gr16 = reinterpret_cast<const uint16_t*>(gimg + int64_t(kWords) * 8);
        __syncthreads();                            // the previous part's counters are flushed
        if (threadIdx.x == 0) {
            uint32_t run = 0;
            for (int k = 0; k < kBase32; ++k) {
                sbb[k] = run;
                run += a.sb_count[static_cast<int64_t>(p) * kBase32 + k];
            }
        }
        for (uint32_t k = threadIdx.x; k < kCounts; k += blockDim.x) cnt[k] = 0;
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < kProbeWords; j += blockDim.x) {
            uint32_t rank = sbb[j >> 7] + gr16[j >> 2];
            for (uint32_t k = j & ~3u; k < j; ++k) rank += __builtin_popcount(gbm[k]);
            pw[j] = (static_cast<uint64_t>(rank) << 32) | gbm[j];
        }
        __syncthreads();
        const uint32_t pbase = static_cast<uint32_t>(static_cast<int64_t>(p) << kPartShift);
        for (int64_t m = srank; m < n_tiles; m += nserv) {
            const int64_t tile = a.first_tile + m;
            const int64_t t0 = tile * a.T;
            const int Tk = static_cast<int>(a.N - t0 < a.T ? a.N - t0 : a.T);
            const int64_t sbase = tile * (static_cast<int64_t>(a.T) * P + 1);
            const uint32_t* tids = a.pids + a.tile_start[tile];
            // kTr trials per group of 16 lanes, whose segments' loads are in flight together
            constexpr int kTr = 4;
            for (int i0 = slot; i0 < Tk; i0 += kTr * n_slots) {
                uint32_t sb2[kTr], len2[kTr];
                unsigned long long wt2[kTr];
#pragma unroll
                for (int h = 0; h < kTr; ++h) {
                    const int i = i0 + h * n_slots;
                    sb2[h] = 0;
                    len2[h] = 0;
                    wt2[h] = 0;
                    const int64_t t = t0 + i;
                    if (i >= Tk || t < a.t_lo || t >= a.t_hi) continue;
                    const int64_t k = t - a.t_lo;
                    const double ta = a.S[k] - a.aggR;
                    if (!((ta > 0.0) && (ta < a.aggL))) continue;        // outside the aggregate band
                    const uint64_t key = __double_as_longlong(a.ylt[k] + 0.0);
                    wt2[h] = key > ts.v_bits ? ts.c_eq : (key == ts.v_bits ? ts.m - ts.c_gt : 0);
                    sb2[h] = a.seg_rel[sbase + static_cast<int64_t>(p) * Tk + i];
                    len2[h] = a.seg_rel[sbase + static_cast<int64_t>(p) * Tk + i + 1] - sb2[h];
                }
                constexpr int kU = 4;
                uint32_t lmax = 0;
#pragma unroll
                for (int h = 0; h < kTr; ++h) lmax = len2[h] > lmax ? len2[h] : lmax;
                for (uint32_t off = lig * 4; off < lmax; off += 64 * kU) {
                    u32x4 v[kTr][kU];
#pragma unroll
                    for (int h = 0; h < kTr; ++h)
#pragma unroll
                        for (int u = 0; u < kU; ++u) {
                            const uint32_t o = off + u * 64;
                            v[h][u] = o < len2[h]
                                          ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tids + sb2[h] + o))
                                          : u32x4{kSentinel, kSentinel, kSentinel, kSentinel};
                        }
#pragma unroll
                    for (int h = 0; h < kTr; ++h)
#pragma unroll
                        for (int q = 0; q < kU * 4; ++q) {
                            const uint32_t id = v[h][q >> 2][q & 3];
                            const uint32_t el = id - pbase;
                            if (el >= static_cast<uint32_t>(kPartSize)) continue;     // padding
                            const uint64_t w = pw[el >> 5];
                            const uint32_t bi = el & 31u;
                            if (!((w >> bi) & 1ull)) continue;
                            const uint32_t rank = static_cast<uint32_t>(w >> 32) +
                                                  __builtin_popcount(static_cast<uint32_t>(w) & ((1u << bi) - 1u));
                            if (rank < kCounts)
                                atomicAdd(&cnt[rank], 1u);
                            else
                                atomicAdd(reinterpret_cast<unsigned long long*>(&a.w_mean[id]), 1ull);
                            if (wt2[h]) atomicAdd(reinterpret_cast<unsigned long long*>(&a.w_tvar[id]), wt2[h]);
                        }
                }
            }
        }
        __syncthreads();
        // the LDS counters to W_mean: the events of each probe word, in rank order
        for (uint32_t j = threadIdx.x; j < kProbeWords; j += blockDim.x) {
            const uint64_t w = pw[j];
            uint32_t bits = static_cast<uint32_t>(w);
            uint32_t rank = static_cast<uint32_t>(w >> 32);
            while (bits && rank < kCounts) {
                const uint32_t b = static_cast<uint32_t>(__builtin_ctz(bits));
                const uint32_t c = cnt[rank];
                if (c) atomicAdd(reinterpret_cast<unsigned long long*>(&a.w_mean[pbase + j * 32 + b]),
                                 static_cast<unsigned long long>(c));
                bits &= bits - 1u;
                ++rank;
            }
        }
    }
}

// XCD-affine pass.  Workgroups are dispatched to the 8 XCDs round-robin, so
// workgroup b runs on XCD b % 8; each XCD serves its own catalogue parts
// (part p on XCD p % 8).  A part's dense occurrence losses are 2 MB, so they
// stay in that XCD's 4 MB L2 and a hit gathers o[E] directly, with no rank
// arithmetic; the part's 32 KB bitmap is loaded into LDS once per part.  Each
// (part, trial) double-double partial goes to HBM; xcd_combine_kernel adds
// the parts of a trial in part order.
// Inclusive prefix sum over the 64 lanes of a wave with DPP lane moves: four
// shifts build each 16-lane row's scan, two row broadcasts carry row totals.
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t x) {
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x111, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x112, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x114, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x118, 0xF, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x142, 0xA, 0xF, false));
    x += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x143, 0xC, 0xF, false));
    return x;
}

// the value held by the partner lane (lane ^ 1)
__device__ __forceinline__ double swap_pair_f64(double v) {
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<uint32_t>(b)), 0xB1,
                                                                        0xF, 0xF, false));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(static_cast<uint32_t>(b >> 32)),
                                                                        0xB1, 0xF, 0xF, false));
    return __longlong_as_double(static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo));
}

// XCD-affine trial pass.  Workgroups on XCD x serve the catalogue parts
// p = x (mod 8), whose 2 MB of occurrence losses stay in that XCD's L2.  Each
// wave owns 32 consecutive trials of a tile and streams their IDs of part p
// as one contiguous range, 1024 IDs per batch: every ID is tested against the
// part's bitmap in LDS and the hits are appended, in position order, to the
// wave's LDS queue.  The queue is drained at the end of the tile (or when it
// may overflow): two lanes per trial gather the losses of that trial's hits
// and sum them in double-double, in queue order, so the result does not
// depend on timing.  Tiles are assigned to workgroups statically, so the
// next tile's boundaries are read a tile ahead and its first batch is loaded
// while the current tile's last one is tested.
__global__ __launch_bounds__(1024) void xcd_pass_kernel(XcdPassArgs a) {
    constexpr int kU = 2;                           // 16-byte loads per lane per batch
    constexpr int kTrialsPW = kTileMax / 8;         // 32 trials per wave
    constexpr uint32_t kBatch = 64 * 4 * kU;        // IDs per batch
    constexpr int kQ = 512;                         // queue entries per wave (one batch)
    constexpr int kInf = 0x3FFFFFFF;
    static_assert(kQ >= static_cast<int>(kBatch), "a batch must fit the queue");
    // LDS, one block: the part's probe words (one per 32 events: the bitmap
    // bits in the low half, the part-relative rank of the word's first event
    // among the nonzero ones in the high half) -- first, so a probe word's
    // byte offset is its LDS address -- then the hit queues, then as many of
    // the part's first nonzero losses as fit
    constexpr uint32_t kProbeWords = static_cast<uint32_t>(kPartSize >> 5);
    constexpr uint32_t kProbeMask = (kProbeWords - 1) * 8;              // byte offset bits of a probe word
    constexpr uint32_t kQueueOff = kProbeWords * 8;                     // 16 per-wave hit queues (event IDs)
    constexpr uint32_t kCacheOff = kQueueOff + 16 * kQ * 4;             // the loss cache (8-byte aligned)
    constexpr int kCache = static_cast<int>((160 * 1024 - kCacheOff) / 8);
    static_assert(kCacheOff % 16 == 0 && kCache > 0, "LDS layout");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kCacheOff + kCache * 8];
    uint64_t* pwords = reinterpret_cast<uint64_t*>(lds);
    double* cache = reinterpret_cast<double*>(lds + kCacheOff);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    uint32_t* q = reinterpret_cast<uint32_t*>(lds + kQueueOff) + wv * kQ;
    // parts served by this workgroup (its XCD's), and its rank among the servers
    // of each; the two halves of the workgroup (8 waves each) serve separately
    const int n_xcd = a.n_xcd;
    const int x = static_cast<int>(blockIdx.x % n_xcd);
    const int r = static_cast<int>(blockIdx.x / n_xcd);
    const int nr = static_cast<int>(gridDim.x / n_xcd);
    const int P = a.P;
    int p0, pstep, srank, nserv;
    if (P >= n_xcd) {
        p0 = x;
        pstep = n_xcd;
        srank = r;
        nserv = nr;
    } else {
        p0 = x % P;
        pstep = P;
        srank = (x / P) * nr + r;
        nserv = ((n_xcd - 1 - p0) / P + 1) * nr;
    }
    srank = 2 * srank + (wv >> 3);
    nserv = 2 * nserv;
    const int64_t n_tiles = a.last_tile - a.first_tile;
    const int64_t count = a.t_hi - a.t_lo;
    const int j0w = (wv & 7) * kTrialsPW;           // the wave's first trial in a tile
    const int pt = lane >> 1;                       // the trial this lane sums (with its partner)
    const int half = lane & 1;

    for (int p = p0; p < P; p += pstep) {
        // the part image (bitmap, 128-event ranks within superblocks, global
        // superblock ranks) becomes the probe words
        const uint8_t* gimg = a.img + static_cast<int64_t>(p) * kImgBytes;
        const uint32_t* gbm = reinterpret_cast<const uint32_t*>(gimg);
        const uint16_t* gr16 = reinterpret_cast<const uint16_t*>(gimg + int64_t(kWords) * 8);
        const uint32_t* gb32 = reinterpret_cast<const uint32_t*>(gimg + int64_t(kWords) * 8 + int64_t(kRank16) * 2);
        const uint32_t rank0 = gb32[0];             // global rank of the part's first nonzero loss
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < kProbeWords; j += blockDim.x) {
            uint32_t rank = gb32[j >> 7] - rank0 + gr16[j >> 2];
            for (uint32_t k = j & ~3u; k < j; ++k) rank += __builtin_popcount(gbm[k]);
            pwords[j] = (static_cast<uint64_t>(rank) << 32) | gbm[j];
        }
        __syncthreads();
        // the part's first nonzero losses, in rank order
        for (int k = threadIdx.x; k < kCache; k += blockDim.x) {
            const int64_t g = static_cast<int64_t>(rank0) + k;
            cache[k] = g < a.C ? a.compact[g] : 0.0;
        }
        __syncthreads();
        if (srank >= n_tiles) continue;

        // this server's m-th tile, clamped to a real tile past the end (never used there)
        auto tile_of = [&](int64_t m) -> int64_t {
            const int64_t tile = a.first_tile + srank + m * nserv;
            return tile < a.last_tile ? tile : a.last_tile - 1;
        };
        auto trials_in = [&](int64_t tile) -> int {
            const int64_t t0 = tile * a.T;
            return static_cast<int>(a.N - t0 < a.T ? a.N - t0 : a.T);
        };
        // the wave's 33 segment boundaries in a tile, lane i holding boundary i
        // (lanes past 32 repeat the last), clamped to the tile's trial count
        auto load_bounds = [&](int64_t tile) -> uint32_t {
            const int Tk = trials_in(tile);
            const int64_t sb = tile * (static_cast<int64_t>(a.T) * P + 1) + static_cast<int64_t>(p) * Tk;
            const int i = j0w + (lane < kTrialsPW ? lane : kTrialsPW);
            return a.seg_rel[sb + (i < Tk ? i : Tk)];
        };
        // the wave's trials [jlo, jhi) of a tile (relative to j0w), clipped to
        // the tile and to the layer's trials
        auto clip = [&](int64_t tile, int& jlo, int& jhi) {
            const int64_t t0 = tile * a.T + j0w;
            const int Tk = trials_in(tile) - j0w;
            jlo = 0;
            jhi = kTrialsPW < Tk ? kTrialsPW : (Tk > 0 ? Tk : 0);
            if (t0 + jlo < a.t_lo) jlo = static_cast<int>(a.t_lo - t0 < jhi ? a.t_lo - t0 : jhi);
            if (t0 + jhi > a.t_hi) jhi = static_cast<int>(a.t_hi - t0 > jlo ? a.t_hi - t0 : jlo);
            if (jhi < jlo) jhi = jlo;
        };

        // current tile
        int64_t m = 0;
        int64_t tile = tile_of(0);
        uint32_t B = load_bounds(tile);
        int jlo, jhi;
        uint32_t rs, re;
        const uint32_t* tids;
        // next tile: its range and ID base (its first batch is loaded during
        // this tile's last); boundaries of the next two tiles are read ahead
        uint32_t B1 = load_bounds(tile_of(1));
        uint32_t B2 = load_bounds(tile_of(2));
        uint32_t n_rs, n_re;
        const uint32_t* n_tids;
        bool has_next = srank + nserv < n_tiles;
        int qs;                                     // lane i: queue index of trial i's first hit
        int qn = 0;                                 // entries in the queue
        double acc_hi = 0.0, acc_lo = 0.0;

        auto enter = [&]() {                        // make `tile` (boundaries B) current
            clip(tile, jlo, jhi);
            rs = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B), jlo));
            re = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B), jhi));
            tids = a.pids + a.tile_start[tile];
            qs = B <= rs ? 0 : kInf;
        };
        auto aim = [&](int64_t ntile) {             // the range of `ntile` (boundaries B1)
            int nlo, nhi;
            clip(ntile, nlo, nhi);
            n_rs = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B1), nlo));
            n_re = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(B1), nhi));
            n_tids = a.pids + a.tile_start[ntile];
        };
        enter();
        aim(tile_of(1));
        // batches start on 128-byte lines (tiles are aligned); positions before
        // rs are masked off
        uint32_t c = rs & ~uint32_t(kTileAlign - 1);

        // one batch of 16-byte ID chunks; chunks at or past `end` read the
        // padding instead (cached), so no HBM line past the range is fetched
        auto load_batch = [&](const uint32_t* ids, uint32_t cb, uint32_t end, u32x4* v) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t cu = cb + u * 256 + lane * 4;
                const uint32_t* src = cu < end ? ids + cu : a.pad;
                v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
            }
        };
        // the batch after the one at c: the rest of this tile, else the next tile's first
        auto load_next = [&](u32x4* v) {
            if (c + kBatch < re)
                load_batch(tids, c + kBatch, re, v);
            else
                load_batch(n_tids, n_rs & ~uint32_t(kTileAlign - 1), has_next ? n_re : 0u, v);
        };
        // gather and sum the queued hits: lanes 2t and 2t+1 take trial t's
        // entries alternately, four gathers in flight per lane
        auto drain = [&]() {
            int lo = __shfl(qs, pt), hi = __shfl(qs, pt + 1);
            lo = lo < 0 ? 0 : (lo > qn ? qn : lo);
            hi = hi < 0 ? 0 : (hi > qn ? qn : hi);
            for (int j = lo + half; j < hi; j += 8) {
                double v[4];
#pragma unroll
                for (int r2 = 0; r2 < 4; ++r2) {
                    const int jj = j + 2 * r2;
                    v[r2] = 0.0;
                    if (jj < hi) {
                        // rank of the event among the part's nonzero ones: its probe
                        // word's, plus the set bits below it in the word.  Parts are
                        // aligned, so the low bits of an ID are its part-relative
                        // index; a queued padding ID reads as the part's last event.
                        const uint32_t id = q[jj];
                        const uint32_t e = id & static_cast<uint32_t>(kPartSize - 1);
                        const uint64_t pwd = *reinterpret_cast<const uint64_t*>(lds + (e >> 5) * 8u);
                        const uint32_t below = (1u << (e & 31u)) - 1u;
                        const uint32_t lr = static_cast<uint32_t>(pwd >> 32) +
                                            __builtin_popcount(static_cast<uint32_t>(pwd) & below);
                        // the LDS copy, read at a clamped rank, else the value from L2
                        // (two loads of one address space each, no pointer select)
                        v[r2] = cache[min(lr, static_cast<uint32_t>(kCache - 1))];
                        if (lr >= static_cast<uint32_t>(kCache)) v[r2] = a.compact[rank0 + lr];
                        if (id == kSentinel) v[r2] = 0.0;   // segment padding adds nothing
                    }
                }
                // entries past the trial's last are 0.0, whose sum is exact
#pragma unroll
                for (int r2 = 0; r2 < 4; ++r2) dd_add(acc_hi, acc_lo, v[r2]);
            }
            qs = qs == kInf ? kInf : qs - qn;
            qn = 0;
            __builtin_amdgcn_wave_barrier();
        };
        // test a batch against the bitmap and append its hits to the queue in
        // position order (chunk u, lane, word); note where each trial's hits start
        auto process = [&](const u32x4* ids) {
            // every ID in [rs, re) belongs to part p, and parts are aligned to
            // their size, so an ID's bits 5..17 are its probe word and its low 5
            // bits the bit in it.  The only other IDs are the segment padding,
            // which reads the part's last event: if that event is nonzero the
            // padding is queued like a hit, and the drain gives it 0.0.
            uint32_t hit[kU][4];                    // word w of chunk u is a hit (0 or 1)
            uint32_t cnt[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                // a chunk lies wholly inside or outside [rs, re): both are multiples of 4
                const uint32_t ok = c + u * 256 + lane * 4 - rs < re - rs ? 1u : 0u;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t id = ids[u][w];
                    const uint32_t wa = (id >> 2) & kProbeMask;   // byte address of its probe word
                    const uint32_t word = *reinterpret_cast<const uint32_t*>(lds + wa);
                    hit[u][w] = __builtin_amdgcn_ubfe(word, id, 1u) & ok;
                }
                cnt[u] = hit[u][0] + hit[u][1] + hit[u][2] + hit[u][3];
            }
            // per-chunk hit counts, prefix-summed over the wave two chunks at a time
            // (16-bit halves: at most 4 x 64 hits per chunk)
            uint32_t ex[kU], tot[kU];
#pragma unroll
            for (int u = 0; u < kU; u += 2) {
                const uint32_t ha = cnt[u];
                const uint32_t hb = u + 1 < kU ? cnt[u + 1] : 0u;
                const uint32_t sc = wave_scan_u32(ha | (hb << 16));
                const uint32_t tt = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(sc), 63));
                ex[u] = (sc & 0xFFFFu) - ha;
                tot[u] = tt & 0xFFFFu;
                if (u + 1 < kU) {
                    ex[u + 1] = (sc >> 16) - hb;
                    tot[u + 1] = tt >> 16;
                }
            }
            int total = 0;
#pragma unroll
            for (int u = 0; u < kU; ++u) total += static_cast<int>(tot[u]);
            if (qn + total > kQ) drain();            // exact: the batch always fits an empty queue
            int pre[kU];
            {
                int base = qn;
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    pre[u] = base + static_cast<int>(ex[u]);
                    base += static_cast<int>(tot[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                int at = pre[u];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if (hit[u][w]) q[at] = ids[u][w];
                    at += static_cast<int>(hit[u][w]);
                }
            }
            // trial boundaries inside this batch: the first hit at or after the
            // boundary's chunk is where that trial's hits start
            const uint32_t k = (B - c) >> 2;        // chunk of this lane's boundary (if in the batch)
            const int src = static_cast<int>(k & 63u);
            int vq = 0;
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int v = __shfl(pre[u], src);
                vq = (k >> 6) == static_cast<uint32_t>(u) ? v : vq;
            }
            if (B > rs && B < re && B >= c && B - c < kBatch) qs = vq;
            qn += total;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        // after a batch: advance; at the end of the wave's range drain the queue,
        // write the trial sums and move to the next tile (its first batch is in
        // flight).  Returns false when the server's tiles are done.
        auto step = [&]() -> bool {
            c += kBatch;
            if (c < re) return true;
            drain();
            dd_merge(acc_hi, acc_lo, swap_pair_f64(acc_hi), swap_pair_f64(acc_lo));
            if (half == 0 && pt >= jlo && pt < jhi) {
                const int64_t t = tile * a.T + j0w + pt;
                a.part_hi[static_cast<int64_t>(p) * count + (t - a.t_lo)] = acc_hi;
                a.part_lo[static_cast<int64_t>(p) * count + (t - a.t_lo)] = acc_lo;
            }
            acc_hi = 0.0;
            acc_lo = 0.0;
            if (!has_next) return false;
            ++m;
            tile = tile_of(m);
            B = B1;
            enter();
            c = rs & ~uint32_t(kTileAlign - 1);
            has_next = srank + (m + 1) * nserv < n_tiles;
            B1 = B2;
            aim(tile_of(m + 1));
            B2 = load_bounds(tile_of(m + 2));
            return true;
        };

        // two register buffers in turn, so the loads of the next batch stay in
        // flight while this one is tested, with no copy that waits for them
        u32x4 bufA[kU], bufB[kU];
        load_batch(tids, c, re, bufA);
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

__global__ __launch_bounds__(256) void xcd_combine_kernel(const double* __restrict__ part_hi,
                                                          const double* __restrict__ part_lo, int P, int64_t count,
                                                          double aggR, double aggL, const LayerArgs* __restrict__ L_dev,
                                                          double* __restrict__ ylt, double* __restrict__ S_out) {
    const int64_t k = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= count) return;
    if (L_dev) {                                    // terms from device memory (graph replays)
        aggR = L_dev->aggR;
        aggL = L_dev->aggL;
    }
    double hi = 0.0, lo = 0.0;
    for (int p = 0; p < P; ++p) dd_merge(hi, lo, part_hi[p * count + k], part_lo[p * count + k]);
    const double S = hi + lo;
    ylt[k] = apply_terms(S, aggR, aggL);
    if (S_out) S_out[k] = S;
}


hipError_t launch_part_pass_lpt(int lpt, int grid, const PartPassArgs& a, hipStream_t s) {
    switch (lpt) {
        case 8: hipLaunchKernelGGL(part_pass_kernel<8>, dim3(grid), dim3(512), 0, s, a); break;
        case 32: hipLaunchKernelGGL(part_pass_kernel<32>, dim3(grid), dim3(512), 0, s, a); break;
        case 64: hipLaunchKernelGGL(part_pass_kernel<64>, dim3(grid), dim3(512), 0, s, a); break;
        default: hipLaunchKernelGGL(part_pass_kernel<16>, dim3(grid), dim3(512), 0, s, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_batched_pass_lpt(int lpt, int grid, const BatchedPassArgs& a, hipStream_t s) {
    switch (lpt) {
        case 8: hipLaunchKernelGGL(batched_pass_kernel<8>, dim3(grid), dim3(512), 0, s, a); break;
        case 32: hipLaunchKernelGGL(batched_pass_kernel<32>, dim3(grid), dim3(512), 0, s, a); break;
        case 64: hipLaunchKernelGGL(batched_pass_kernel<64>, dim3(grid), dim3(512), 0, s, a); break;
        default: hipLaunchKernelGGL(batched_pass_kernel<16>, dim3(grid), dim3(512), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace

int64_t part_image_bytes(int P) { return static_cast<int64_t>(P) * kImgBytes; }

hipError_t build_sparse_pool(const double* elts, int32_t n_rows, int64_t C, hipStream_t s, SparsePool* out) {
    *out = SparsePool{};
    if (n_rows > 65535) return hipErrorInvalidValue;            // rows are the grid's second dimension
    const int64_t n_chunks = (C + kSuper - 1) / kSuper;
    const int64_t n = static_cast<int64_t>(n_rows) * n_chunks;
    out->n_chunks = n_chunks;
    hipError_t e;
    if ((e = hipMalloc(&out->chunk_off, sizeof(int64_t) * (n + 1))) != hipSuccess) return e;
    out->bytes = static_cast<int64_t>(sizeof(int64_t)) * (n + 1);
    if (n == 0) return hipMemsetAsync(out->chunk_off, 0, sizeof(int64_t), s);
    const dim3 grid(static_cast<uint32_t>(n_chunks), static_cast<uint32_t>(n_rows));
    hipLaunchKernelGGL(sparse_count_kernel, grid, dim3(256), 0, s, elts, C, n_chunks, out->chunk_off);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_scan_i64(out->chunk_off, n, s)) != hipSuccess) return e;
    int64_t nnz = 0;
    if ((e = hipMemcpyAsync(&nnz, out->chunk_off + n, sizeof(int64_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return e;
    out->nnz = nnz;
    const int64_t cap = nnz > 0 ? nnz : 1;
    // one block where it stays below the 2 MB from which the runtime's free takes 300 us
    const size_t both = (sizeof(double) + sizeof(uint16_t)) * cap;
    out->joint = both < (size_t(2) << 20);
    if ((e = hipMalloc(&out->val, out->joint ? both : sizeof(double) * cap)) != hipSuccess) return e;
    if (out->joint) out->ev = reinterpret_cast<uint16_t*>(out->val + cap);
    else if ((e = hipMalloc(&out->ev, sizeof(uint16_t) * cap)) != hipSuccess) return e;
    out->bytes += static_cast<int64_t>(sizeof(uint16_t) + sizeof(double)) * cap;
    hipLaunchKernelGGL(sparse_fill_kernel, grid, dim3(256), 0, s, elts, C, n_chunks, out->chunk_off, out->ev,
                       out->val);
    return hipGetLastError();
}

void free_sparse_pool(SparsePool* sp) {
    if (sp->ev && !sp->joint) (void)hipFree(sp->ev);
    if (sp->val) (void)hipFree(sp->val);
    if (sp->chunk_off) (void)hipFree(sp->chunk_off);
    *sp = SparsePool{};
}

hipError_t launch_create_clear(uint32_t* pad, CreateResult* res, int32_t* cnt, int64_t n_cnt, int n_cu, hipStream_t s) {
    const int64_t n16 = (n_cnt + 3) / 4;            // the cache's blocks are whole multiples of 16 bytes
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n16 + 1023) / 1024, int64_t(n_cu) * 8));
    hipLaunchKernelGGL(create_clear_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s, pad, res,
                       reinterpret_cast<u32x4*>(cnt), n16);
    return hipGetLastError();
}

hipError_t launch_yet_count(const int64_t* offsets, int64_t N, const uint32_t* src, uint32_t* ids, int64_t n_events,
                            int64_t C, int shift, int bins, int32_t* cnt, CreateResult* res, int n_cu, hipStream_t s) {
    if (n_events <= 0) return hipSuccess;
    if (bins < 0 || bins > 64) return hipErrorInvalidValue;
    const bool copy = src != ids;
    if (reinterpret_cast<uintptr_t>(src) % 16 || reinterpret_cast<uintptr_t>(ids) % 16) return hipErrorInvalidValue;
    const bool apart = bins > 0 && n_events / kShortTrial < N;         // short trials: counted afterwards
    // 32 waves per CU, at least a row of 256 IDs each (16 rows: 10000 trials of 30 events
    // 107 -> 14 us, of 100 40 -> 11: a wave's time goes by its trials)
    int64_t waves = (n_events + 255) / 256;
    waves = std::min(waves, int64_t(n_cu) * 32);
    const dim3 g(static_cast<uint32_t>((waves + 3) / 4)), b(256);
    const uint32_t c32 = static_cast<uint32_t>(std::min<int64_t>(C, 0xFFFFFFFFll));
    hipLaunchKernelGGL((copy ? yet_count_kernel<true> : yet_count_kernel<false>), g, b, 0, s, offsets, N, src, ids,
                       n_events, c32, shift, apart ? 0 : bins, cnt, &res->flags);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !apart) return e;
    hipLaunchKernelGGL(short_count_kernel, dim3(static_cast<uint32_t>((N + 255) / 256)), dim3(256),
                       sizeof(int32_t) * 256 * (bins | 1), s, offsets, N, ids, shift, bins, cnt, &res->flags);
    return hipGetLastError();
}

int part_layout_parts(int64_t N, int64_t C) {
    const int64_t P = (C + kPartSize - 1) / kPartSize;
    return N < 1 || P < 1 || P > kMaxParts ? 0 : static_cast<int>(P);
}

hipError_t begin_part_layout(int64_t N, int64_t C, hipStream_t s, PartLayout* out) {
    *out = PartLayout{};
    const int P = part_layout_parts(N, C);
    if (P == 0) return hipSuccess;                                     // layout not used
    const int T = kTileMax;
    const int64_t n_tiles = (N + T - 1) / T;
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&out->seg_rel),
                             sizeof(uint32_t) * (n_tiles * (static_cast<int64_t>(T) * P + 1)), s);
    if (e == hipSuccess)
        e = dev_alloc(reinterpret_cast<void**>(&out->tile_start), sizeof(int64_t) * (n_tiles + 1), s);
    if (e != hipSuccess) {
        free_part_layout(out, s);
        return e;
    }
    out->P = P;
    out->T = T;
    out->n_tiles = n_tiles;
    return hipSuccess;
}

hipError_t plan_part_layout(const int32_t* cnt, int shift, int bins, int64_t N, CreateResult* res, hipStream_t s,
                            const PartLayout& lay) {
    if (lay.P == 0) return hipSuccess;
    hipLaunchKernelGGL(tile_scan_kernel, dim3(static_cast<uint32_t>(lay.n_tiles)), dim3(256),
                       sizeof(int32_t) * static_cast<size_t>(lay.T) * lay.P, s, cnt, bins, kPartShift - shift, N, lay.P,
                       lay.T, lay.seg_rel, lay.tile_start);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tile_starts_kernel, dim3(1), dim3(1024), 0, s, lay.tile_start, lay.n_tiles, res);
    return hipGetLastError();
}

hipError_t fill_part_layout(const int64_t* offsets, const uint32_t* ids, int64_t N, int64_t n_events,
                            const CreateResult& res, hipStream_t s, PartLayout* out) {
    if (out->P == 0) return hipSuccess;
    if (res.flags & kCreateWideTile) {      // too large for 32-bit positions: keep the plain layout
        free_part_layout(out, s);
        return hipSuccess;
    }
    const int64_t total = res.part_ids;
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&out->pids), sizeof(uint32_t) * (total + kIdPad), s);
    if (e == hipSuccess) {
        const double lam = static_cast<double>(n_events) / static_cast<double>(N);
        const int fit = scatter_trials(lam + 1.5 * out->P, 0.0, kScatterStage32, 64);
        const int units = (out->T + fit - 1) / fit, per = (out->T + units - 1) / units;
        const int64_t n_units = out->n_tiles * ((out->T + per - 1) / per);
        const size_t lds = sizeof(uint32_t) * static_cast<size_t>(out->P) * (per + 1);
        const auto kernel = out->P <= 8 ? part_scatter_kernel<3> : part_scatter_kernel<6>;
        e = in_launches(n_units, [&](int64_t first, int64_t n) {
            hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>((n + kXcds - 1) / kXcds * kXcds)),
                               dim3(kScatterThreads), lds, s, offsets, ids, N, out->P, out->T, per, first, n,
                               out->seg_rel, out->tile_start, out->pids);
        });
    }
    if (e != hipSuccess) return e;
    out->length = total;
    out->bytes = static_cast<int64_t>(sizeof(uint32_t)) * (total + kIdPad) +
                 static_cast<int64_t>(sizeof(uint32_t)) * (out->n_tiles * (int64_t(out->T) * out->P + 1)) +
                 static_cast<int64_t>(sizeof(int64_t)) * (out->n_tiles + 1);
    return hipSuccess;
}

void free_part_layout(PartLayout* L, hipStream_t s) {
    if (L->pids) dev_free(L->pids, s);
    if (L->seg_rel) dev_free(L->seg_rel, s);
    if (L->tile_start) dev_free(L->tile_start, s);
    *L = PartLayout{};
}

int64_t part_scratch_bytes(int64_t C, int P, bool compact) {
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    return part_image_bytes(P) + sizeof(uint32_t) * n_sb + (compact ? sizeof(double) * C : 0) +
           sizeof(double) * n_sb * kSuper + 256;
}

namespace {
struct PartScratch {
    uint8_t* img;
    uint32_t* sb_count;
    uint32_t* counter;
    double* stage;        // [n_sb][kSuper]: each superblock's nonzero o, packed, before compaction
    double* compact;      // [C]: the nonzero o at their global ranks (last: sized by C)
};
PartScratch carve_parts(void* scratch, int P) {
    char* p = static_cast<char*>(scratch);
    PartScratch r;
    r.img = reinterpret_cast<uint8_t*>(p);
    p += part_image_bytes(P);
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    r.sb_count = reinterpret_cast<uint32_t*>(p);
    p += sizeof(uint32_t) * n_sb;
    r.counter = reinterpret_cast<uint32_t*>(p);
    p += 256;
    r.stage = reinterpret_cast<double*>(p);
    p += sizeof(double) * n_sb * kSuper;
    r.compact = reinterpret_cast<double*>(p);
    return r;
}
}  // namespace

double* part_compact_values(void* part_scratch, int P) { return carve_parts(part_scratch, P).compact; }
FoldViews fold_views(void* part_scratch, int P) {
    const PartScratch ps = carve_parts(part_scratch, P);
    return FoldViews{ps.img, ps.sb_count, ps.stage, 0, 0};
}
// [layer] images, [layer] superblock counts, [layer] packed values
FoldViews fold_batch_views(void* scratch, int n_layers, int P) {
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    char* p = static_cast<char*>(scratch);
    FoldViews v;
    v.img = reinterpret_cast<uint8_t*>(p);
    v.img_stride = part_image_bytes(P);
    p += (v.img_stride * n_layers + 255) & ~int64_t(255);
    v.sb_count = reinterpret_cast<uint32_t*>(p);
    v.sb_stride = n_sb;
    p += (static_cast<int64_t>(sizeof(uint32_t)) * n_sb * n_layers + 255) & ~int64_t(255);
    v.stage = reinterpret_cast<double*>(p);
    return v;
}
int64_t fold_batch_bytes(int n_layers, int P) {
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    return n_layers * (part_image_bytes(P) + static_cast<int64_t>(sizeof(uint32_t)) * n_sb +
                       static_cast<int64_t>(sizeof(double)) * n_sb * kSuper) + 512;
}
uint32_t* part_superblock_counts(void* part_scratch, int P) { return carve_parts(part_scratch, P).sb_count; }

// ---------------------------------------------------------------------------
// per-event net losses (the cumulative form of the aggregate terms)
// ---------------------------------------------------------------------------

namespace {

constexpr int kProbeShift = 5;                  // 32 catalogue events per probe word
constexpr int kNetsThreads = 1024;              // one workgroup per CU: its waves share the coarse map
constexpr int kNetsStageBytes = 37 * 1024;     // the waves' queues and flag rows
constexpr int kCoarseBytes = 160 * 1024 - kNetsStageBytes;   // LDS left for the coarse map

// One stage of a segmented double-double scan: (f, h, l) becomes
// left (+) self, where a lane that starts a segment (f set) keeps its sum.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ void seg_stage(uint32_t& f, double& h, double& l) {
    const uint32_t uf = dpp_u32<kCtrl, kRowMask>(f);
    const double uh = dpp_f64<kCtrl, kRowMask>(h), ul = dpp_f64<kCtrl, kRowMask>(l);
    double mh = h, ml = l;
    dd_merge(mh, ml, uh, ul);
    if (!f) {
        h = mh;
        l = ml;
        f = uf;
    }
}
// inclusive over the wave: row shifts 1, 2, 4, 8, then row broadcasts 15, 31
__device__ __forceinline__ void wave_seg_scan_dd(uint32_t& f, double& h, double& l) {
    seg_stage<0x111, 0xF>(f, h, l);
    seg_stage<0x112, 0xF>(f, h, l);
    seg_stage<0x114, 0xF>(f, h, l);
    seg_stage<0x118, 0xF>(f, h, l);
    seg_stage<0x142, 0xA>(f, h, l);
    seg_stage<0x143, 0xC>(f, h, l);
}

// coarse map: bit i is set when any of events [i << cshift, (i + 1) << cshift)
// has a nonzero loss; one thread per 32-bit word, from the probe words' bits
// (for catalogues whose coarse words span superblocks; the fold writes the others)
__global__ __launch_bounds__(256) void coarse_map_kernel(const uint64_t* __restrict__ probe, int64_t n_words,
                                                         int cshift, int64_t n_cw, uint32_t* __restrict__ coarse) {
    const int64_t cw = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (cw >= n_cw) return;
    uint32_t out = 0;
    for (int k = 0; k < 32; ++k) {
        const int64_t s0 = (cw * 32 + k) << cshift;                   // first event of the group
        uint32_t any = 0;
        if (cshift >= kProbeShift) {
            const int64_t w0 = s0 >> kProbeShift, nw = int64_t(1) << (cshift - kProbeShift);
            for (int64_t w = w0; w < w0 + nw && w < n_words; ++w) any |= static_cast<uint32_t>(probe[w]);
        } else if ((s0 >> kProbeShift) < n_words) {
            const uint32_t bits = static_cast<uint32_t>(probe[s0 >> kProbeShift]);
            const uint32_t width = 1u << cshift;
            const uint32_t mask = (width >= 32u ? ~0u : ((1u << width) - 1u)) << (s0 & 31);
            any = bits & mask;
        }
        out |= (any != 0u ? 1u : 0u) << k;
    }
    coarse[cw] = out;
}

// Both time-ordered passes split the layer's trials into one contiguous run
// per wave (event shares rounded to trial starts).  o(E) is 0 unless E's bit is
// set in its probe word, else stage[index + bits below] -- an 8-byte probe and
// one more load per nonzero loss, both from tables that stay in L2.  L2 serves
// these random requests at a bounded rate, so the workgroup's 16 waves first
// test a coarse map in LDS (one bit per 2^cshift events, set when any of them
// has a loss) and probe L2 only for events whose bit is set.  Trial starts are
// held one per lane and marked in a per-wave LDS bit row.

// the coarse map to LDS (n_cw words, both sides 16-byte aligned and padded)
__device__ __forceinline__ void load_coarse(const uint32_t* __restrict__ gcoarse, int64_t n_cw, uint32_t* coarse) {
    const u32x4* src = reinterpret_cast<const u32x4*>(gcoarse);
    u32x4* dst = reinterpret_cast<u32x4*>(coarse);
    const int n = static_cast<int>((n_cw + 3) / 4);
    for (int i0 = threadIdx.x; i0 < n; i0 += 4 * kNetsThreads) {
        u32x4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = src[i0 + k * kNetsThreads < n ? i0 + k * kNetsThreads : i0];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k * kNetsThreads < n) dst[i0 + k * kNetsThreads] = v[k];
    }
}

// The per-event nets.  With S_d a trial's running total and A_d = clamp(S_d;
// AggR, AggL), the net A_d - A_{d-1} is 0 wherever o is 0, so the sums run over
// the events that pass the coarse map alone (the candidates, about a quarter
// of the 1M-trial workload's events) and every other event's net is a stored
// zero.  A wave takes steps of six chunks of 128 positions, two per lane:
//  * each event tests the coarse map; ballots rank the candidates in time order
//    and place (ID, number of trial starts so far in the step) in a per-wave
//    LDS queue of 256;
//  * each lane takes up to four consecutive candidates: probe words together,
//    then losses together, the lane's own double-double prefix, a segmented
//    scan over the lanes (a candidate whose count of trial starts differs from
//    its predecessor's starts a segment), S_d rounded once, A_d and the net,
//    which replaces the queue entry;
//  * the event's lane reads its net back and stores its two positions as 16
//    bytes, 64 lanes to 1 KB.
// Steps with more candidates than the queue holds go through it in balanced
// runs of chunks.
//
// The vector L1 returns data in the order of the requests of the whole CU, so
// an ID load that goes to HBM holds back every probe behind it.  The 16 waves
// therefore step together (one barrier) and issue their next IDs at the start
// of a step, where none has a probe in flight: one wait per step for the CU
// instead of one per wave (2.5e8 events: 0.94 -> 0.83 ms, the L1's address unit
// 88 -> 64% busy).  What is left is L1 request rate (310 random requests per
// wave and step at 0.44 per clock, the rate that independent gathers from a 2 MB
// table reach) and the arithmetic (840 vector instructions), about half each,
// which the barrier keeps from overlapping fully.  A segmented scan over every
// event, eight per lane, took 1.12 ms.
constexpr int kNetsQueue = 256;
typedef double f64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kNetsChunks = 6;

__global__ __launch_bounds__(kNetsThreads) void event_nets_kernel(const int64_t* __restrict__ offsets,
                                                                  const uint32_t* __restrict__ ids,
                                                                  const uint64_t* __restrict__ probe,
                                                                  const uint32_t* __restrict__ gcoarse, int cshift,
                                                                  int64_t n_cw, const double* __restrict__ losses,
                                                                  LayerArgs L, double* __restrict__ nets) {
    constexpr int kCh = kNetsChunks;
    constexpr int kW = 128 * kCh;                                      // positions per step
    constexpr int kN = kNetsQueue / 64;
    static_assert(kW <= kIdPad, "a step may read up to kW - 1 IDs past the table's end");
    static_assert(kNetsStageBytes >= (kNetsThreads / 64) * (kNetsQueue * 8 + kW / 8), "rows fit their LDS share");
    __shared__ uint64_t queues[kNetsThreads / 64][kNetsQueue];
    __shared__ uint32_t flag_rows[kNetsThreads / 64][kW / 32];          // bit i: a trial starts at c + i
    __shared__ int most_steps;
    extern __shared__ __attribute__((aligned(16))) uint32_t coarse[];  // [n_cw]
    if (threadIdx.x == 0) most_steps = 0;
    load_coarse(gcoarse, n_cw, coarse);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    uint64_t* qu = queues[threadIdx.x >> 6];
    uint32_t* fl = flag_rows[threadIdx.x >> 6];
    const int64_t w = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_w = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    const int64_t t0 = L.trial_begin, t1 = L.trial_begin + L.trial_count;
    const int64_t ev0 = offsets[t0];
    const int64_t tot = offsets[t1] - ev0;
    const int64_t k0 = first_trial_at(offsets, t0, t1, ev0 + tot * w / n_w, lane);
    const int64_t k1 = first_trial_at(offsets, t0, t1, ev0 + tot * (w + 1) / n_w, lane);
    const int64_t P0 = uniform_i64(offsets[k0]), P1 = k0 < k1 ? uniform_i64(offsets[k1]) : P0;
    const double A0 = apply_terms(0.0, L.aggR, L.aggL);
    if (lane < kW / 32) fl[lane] = 0;
    int64_t kb = k0;                                                   // trial starts held: kb .. kb + 63
    int64_t bnd = kb + lane < k1 ? offsets[kb + lane] : INT64_MAX;
    const int64_t c0 = P0 & ~int64_t(1);                               // 8-byte aligned ID loads
    u32x2 nxt[kCh];
    auto load_ids = [&](int64_t at) {
#pragma unroll
        for (int u = 0; u < kCh; ++u)
            nxt[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(ids + at + u * 128 + lane * 2));
    };
    // the workgroup's waves step together (see the loop's barrier): as many
    // steps for each as its longest run takes
    if (P0 < P1) load_ids(c0);
    if (lane == 0 && P0 < P1) atomicMax(&most_steps, static_cast<int>((P1 - c0 + kW - 1) / kW));
    __syncthreads();
    const int n_steps = most_steps;
    double ch = 0.0, cl = 0.0;            // running total at the last candidate
    double a_prev = A0;                   // its A
    uint32_t prev_seg = ~0u;              // its trial starts in this step; ~0: a trial started after it
    int64_t c = c0;
    for (int step = 0; step < n_steps; ++step, c += kW) {
        __syncthreads();
        if (c >= P1) continue;
        u32x2 cur[kCh];
#pragma unroll
        for (int u = 0; u < kCh; ++u) cur[u] = nxt[u];
        load_ids(c + kW < P1 ? c + kW : c);
        // mark the trial starts inside [c, c + kW)
        bool any_start = false;
        for (;;) {
            const bool in = bnd >= c && bnd < c + kW;
            if (in) {
                const uint32_t i = static_cast<uint32_t>(bnd - c);
                atomicOr(&fl[i >> 5], 1u << (i & 31u));
            }
            any_start |= __ballot(in) != 0;
            if (static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(bnd), 63)) >= c + kW) break;
            kb += 64;
            bnd = kb + lane < k1 ? offsets[kb + lane] : INT64_MAX;
        }
        __builtin_amdgcn_wave_barrier();
        // positions of the run in this step, relative to c
        const int lo = P0 > c ? static_cast<int>(P0 - c) : 0;
        const int hi = P1 - c < kW ? static_cast<int>(P1 - c) : kW;
        const bool inside = lo == 0 && hi == kW;
        // candidates: bits 2u and 2u + 1 of cm for the lane's positions of chunk u
        uint32_t cm = 0;
        uint32_t bits[kCh][2];
#pragma unroll
        for (int u = 0; u < kCh; ++u)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                // IDs past the run are other trials' or the table's zero padding
                const uint32_t cb = cur[u][k] >> cshift;
                bits[u][k] = coarse[cb >> 5] >> (cb & 31u);
            }
#pragma unroll
        for (int u = 0; u < kCh; ++u)
#pragma unroll
            for (int k = 0; k < 2; ++k) cm |= (bits[u][k] & 1u) << (2 * u + k);
        if (!inside) {
#pragma unroll
            for (int u = 0; u < kCh; ++u)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int i = u * 128 + lane * 2 + k;
                    if (i < lo || i >= hi) cm &= ~(1u << (2 * u + k));
                }
        }
        int n_of[kCh];
        int total = 0;
#pragma unroll
        for (int u = 0; u < kCh; ++u) {
            n_of[u] = static_cast<int>(__popcll(__ballot((cm >> (2 * u)) & 1u)) +
                                       __popcll(__ballot((cm >> (2 * u + 1)) & 1u)));
            total += n_of[u];
        }
        uint32_t starts = 0;                                           // trial starts of the chunks before
        uint32_t at[kCh];                                              // queue index of the lane's first candidate
        // queue the candidates of chunk u from queue index `base` on
        auto append = [&](int u, uint32_t base) {
            const bool h0 = (cm >> (2 * u)) & 1u, h1 = (cm >> (2 * u + 1)) & 1u;
            const uint64_t b0 = __ballot(h0), b1 = __ballot(h1);
            uint32_t s0 = starts, s1 = starts;
            if (any_start) {
                const uint32_t fb = (fl[u * 4 + (lane >> 4)] >> ((lane & 15) * 2)) & 3u;
                const uint64_t g0 = __ballot(fb & 1u), g1 = __ballot(fb & 2u);
                uint32_t seg = starts;
                seg = __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(g0), seg);
                seg = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(g0 >> 32), seg);
                seg = __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(g1), seg);
                seg = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(g1 >> 32), seg);
                starts += static_cast<uint32_t>(__popcll(g0) + __popcll(g1));
                s0 = seg + (fb & 1u);
                s1 = s0 + (fb >> 1);
            }
            uint32_t i = base;
            i = __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b0), i);
            i = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b0 >> 32), i);
            i = __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b1), i);
            i = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b1 >> 32), i);
            at[u] = i;
            if (h0) qu[i] = (static_cast<uint64_t>(s0) << 32) | cur[u][0];
            if (h1) qu[i + (h0 ? 1u : 0u)] = (static_cast<uint64_t>(s1) << 32) | cur[u][1];
        };
        // the queue's n_c candidates: their nets replace them
        auto nets_of = [&](int n_c) {
            const int n = (n_c + 63) >> 6;                             // consecutive candidates per lane
            const uint32_t last_seg = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(qu[n_c - 1] >> 32));
            uint32_t E[kN], sg[kN];
            bool in[kN];
            uint32_t before_seg = prev_seg;
            if (lane > 0 && lane * n - 1 < n_c) before_seg = static_cast<uint32_t>(qu[lane * n - 1] >> 32);
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                in[k] = false;
                E[k] = 0;
                sg[k] = 0;
                if (k >= n) continue;
                const int i = lane * n + k;
                in[k] = i < n_c;
                const uint64_t e = qu[in[k] ? i : 0];
                E[k] = static_cast<uint32_t>(e);
                sg[k] = static_cast<uint32_t>(e >> 32);
            }
            uint64_t pw[kN];
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                pw[k] = 0;
                if (k < n && in[k]) pw[k] = probe[E[k] >> kProbeShift];
            }
            double oq[kN];
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                const uint32_t word = static_cast<uint32_t>(pw[k]), bi = E[k] & 31u;
                oq[k] = 0.0;
                if (k < n && ((word >> bi) & 1u))
                    oq[k] = losses[static_cast<uint32_t>(pw[k] >> 32) + __popc(word & ((1u << bi) - 1u))];
            }
            // the lane's total since its last trial start (all of it if none)
            bool f[kN];
            uint32_t sf = 0;
            double h = 0.0, l = 0.0;
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                f[k] = in[k] && sg[k] != (k == 0 ? before_seg : sg[k - 1]);
                if (k >= n) continue;
                if (f[k]) {
                    h = 0.0;
                    l = 0.0;
                    sf = 1u;
                }
                dd_add(h, l, oq[k]);
            }
            if (lane == 0 && !sf) dd_merge(h, l, ch, cl);              // the open trial's total so far
            double sh = h, sl = l;
            wave_seg_scan_dd(sf, sh, sl);
            // the open trial's total before this lane, then candidate by candidate
            double rh = __shfl_up(sh, 1, 64), rl = __shfl_up(sl, 1, 64);
            if (lane == 0) {
                rh = ch;
                rl = cl;
            }
            double A[kN];
            double a_last = 0.0;
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                A[k] = a_last;
                if (k >= n) continue;
                if (f[k]) {
                    rh = 0.0;
                    rl = 0.0;
                }
                dd_add(rh, rl, oq[k]);
                A[k] = apply_terms(rh + rl, L.aggR, L.aggL);
                a_last = A[k];
            }
            double before = __shfl_up(a_last, 1, 64);
            if (lane == 0) before = a_prev;
#pragma unroll
            for (int k = 0; k < kN; ++k) {
                if (k >= n) continue;
                const double net = A[k] - (f[k] ? A0 : (k == 0 ? before : A[k - 1]));
                if (in[k]) qu[lane * n + k] = static_cast<uint64_t>(__double_as_longlong(net));
            }
            // lanes past the last candidate add zeros: lane 63 holds its totals
            a_prev = readlane_f64(a_last, 63);
            ch = readlane_f64(sh, 63);
            cl = readlane_f64(sl, 63);
            prev_seg = last_seg;
        };
        // the lane's two nets of chunk u (queue entries past a lane's own are read and dropped)
        auto net_pair = [&](int u) -> f64x2_a8 {
            const bool h0 = (cm >> (2 * u)) & 1u, h1 = (cm >> (2 * u + 1)) & 1u;
            const uint32_t i0 = at[u] & (kNetsQueue - 1), i1 = (at[u] + (h0 ? 1u : 0u)) & (kNetsQueue - 1);
            const uint64_t q0 = qu[i0], q1 = qu[i1];
            f64x2_a8 v;
            v.x = __longlong_as_double(static_cast<int64_t>(h0 ? q0 : 0ull));
            v.y = __longlong_as_double(static_cast<int64_t>(h1 ? q1 : 0ull));
            return v;
        };
        double* dst0 = nets + (c + lane * 2 - ev0);
        {
            // in runs of chunks [u0, u1) of at most `limit` candidates (one chunk at least)
            const int runs = (total + kNetsQueue - 1) / kNetsQueue;
            const int limit =
                runs <= 1 ? kNetsQueue : (total / runs + 32 < kNetsQueue ? total / runs + 32 : kNetsQueue);
            int u0 = 0;
            while (u0 < kCh) {
                int u1 = u0, n_c = 0;
#pragma unroll
                for (int u = 0; u < kCh; ++u)
                    if (u == u1 && u >= u0 && (u == u0 || n_c + n_of[u] <= limit)) {
                        append(u, static_cast<uint32_t>(n_c));
                        n_c += n_of[u];
                        u1 = u + 1;
                    }
                __builtin_amdgcn_wave_barrier();
                if (n_c > 0) nets_of(n_c);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int u = 0; u < kCh; ++u) {
                    if (u < u0 || u >= u1) continue;
                    const f64x2_a8 v = net_pair(u);
                    const int i = u * 128 + lane * 2;
                    double* dst = dst0 + u * 128;
                    if (inside || (i >= lo && i + 1 < hi)) {
                        __builtin_nontemporal_store(v, reinterpret_cast<f64x2_a8*>(dst));
                    } else {
                        if (i >= lo && i < hi) dst[0] = v.x;
                        if (i + 1 >= lo && i + 1 < hi) dst[1] = v.y;
                    }
                }
                __builtin_amdgcn_wave_barrier();
                u0 = u1;
            }
        }
        prev_seg = prev_seg == starts ? 0u : ~0u;
        __builtin_amdgcn_wave_barrier();
        if (any_start && lane < kW / 32) fl[lane] = 0;
    }
}

// Every event scanned: nets where most events are candidates (then queues only
// add work), and the stride checkpoints.  Steps of 64 kE positions in time order,
// kE consecutive positions per lane (16-byte loads, the next step's issued
// before this step's work); a segmented double-double scan over the wave gives
// each lane's last running total, the lane below's gives the total before its
// first event, and its own events are added again for their A.  Nets go through
// a per-wave LDS stage, half a step at a time, and out in stores of 64
// consecutive values.  With kStride the kernel writes instead the running total
// S_d of every position d = 64b + 63 to slot b of `nets`.  Eight events per lane
// spread the scan over twice the events of four.
template <int kE, bool kStride>
__global__ __launch_bounds__(kNetsThreads) void event_scan_kernel(const int64_t* __restrict__ offsets,
                                                                  const uint32_t* __restrict__ ids,
                                                                  const uint64_t* __restrict__ probe,
                                                                  const uint32_t* __restrict__ gcoarse, int cshift,
                                                                  int64_t n_cw, const double* __restrict__ losses,
                                                                  LayerArgs L, double* __restrict__ nets) {
    static_assert(kE == 4 || kE == 8, "four or eight events per lane");
    static_assert(64 % kE == 0, "stride slots are lanes' last events when kE divides 64");
    constexpr int kW = 64 * kE;                                        // positions per step
    static_assert(kW <= kIdPad, "a step may read up to kW - 1 IDs past the table's end");
    constexpr int kRow = 32 * (kE + 1);        // half a step's nets, one pad slot per lane
    static_assert(kNetsStageBytes >= (kNetsThreads / 64) * (kRow * 8 + kW / 8), "stage rows fit their LDS share");
    __shared__ double stage[kNetsThreads / 64][kStride ? 1 : kRow];
    __shared__ uint32_t flag_rows[kNetsThreads / 64][kW / 32];          // bit i: a trial starts at c + i
    extern __shared__ __attribute__((aligned(16))) uint32_t coarse[];  // [n_cw]
    // the coarse map, before any wave can leave (the only workgroup barrier)
    load_coarse(gcoarse, n_cw, coarse);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    double* st = stage[threadIdx.x >> 6];
    uint32_t* fl = flag_rows[threadIdx.x >> 6];
    const int64_t w = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_w = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    const int64_t t0 = L.trial_begin, t1 = L.trial_begin + L.trial_count;
    const int64_t ev0 = offsets[t0];
    const int64_t tot = offsets[t1] - ev0;
    const int64_t k0 = first_trial_at(offsets, t0, t1, ev0 + tot * w / n_w, lane);
    const int64_t k1 = first_trial_at(offsets, t0, t1, ev0 + tot * (w + 1) / n_w, lane);
    if (k0 >= k1) return;
    const int64_t P0 = offsets[k0], P1 = offsets[k1];
    if (P0 >= P1) return;
    const double A0 = apply_terms(0.0, L.aggR, L.aggL);
    if (lane < kW / 32) fl[lane] = 0;
    int64_t kb = k0;                                                   // trial starts held: kb .. kb + 63
    int64_t bnd = kb + lane < k1 ? offsets[kb + lane] : INT64_MAX;
    const int64_t c0 = P0 & ~int64_t(kE - 1);                          // 16-byte and lane aligned
    u32x4 nxt[kE / 4];
#pragma unroll
    for (int u = 0; u < kE / 4; ++u)
        nxt[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ids + c0 + lane * kE + 4 * u));
    double ch = 0.0, cl = 0.0;       // running total of the segment open at the step's start
    double a_prev = A0;              // A of the position before the step
    for (int64_t c = c0; c < P1; c += kW) {
        u32x4 cur[kE / 4];
#pragma unroll
        for (int u = 0; u < kE / 4; ++u) cur[u] = nxt[u];
        if (c + kW < P1) {
#pragma unroll
            for (int u = 0; u < kE / 4; ++u)
                nxt[u] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4*>(ids + c + kW + lane * kE + 4 * u));
        }
        // mark the trial starts inside [c, c + kW)
        for (;;) {
            if (bnd >= c && bnd < c + kW) {
                const uint32_t i = static_cast<uint32_t>(bnd - c);
                atomicOr(&fl[i >> 5], 1u << (i & 31u));
            }
            if (static_cast<int64_t>(readlane_u64(static_cast<uint64_t>(bnd), 63)) >= c + kW) break;
            kb += 64;
            bnd = kb + lane < k1 ? offsets[kb + lane] : INT64_MAX;
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t fq[kE];
        {
            const uint32_t fb = fl[(lane * kE) >> 5] >> ((lane * kE) & 31);
#pragma unroll
            for (int q = 0; q < kE; ++q) fq[q] = (fb >> q) & 1u;
        }
        const int64_t pos = c + lane * kE;
        uint32_t E[kE];
        bool ok[kE];
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            ok[q] = pos + q >= P0 && pos + q < P1;
            E[q] = ok[q] ? cur[q >> 2][q & 3] : 0u;
        }
        // the L2 probe only where the coarse map says the event's group has a loss
        uint64_t pw[kE];
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            const uint32_t cb = E[q] >> cshift;
            pw[q] = 0;
            if (ok[q] && ((coarse[cb >> 5] >> (cb & 31u)) & 1u)) pw[q] = probe[E[q] >> kProbeShift];
        }
        double oq[kE];
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            const uint32_t bits = static_cast<uint32_t>(pw[q]);
            const uint32_t bi = E[q] & 31u;
            oq[q] = 0.0;
            if (ok[q] && ((bits >> bi) & 1u)) {
                const uint32_t below = bi ? (~0u >> (32u - bi)) : 0u;
                oq[q] = losses[static_cast<uint32_t>(pw[q] >> 32) + __builtin_popcount(bits & below)];
            }
        }
        // the lane's total since its last trial start (all of it if none)
        uint32_t sf = 0;
        double h = 0.0, l = 0.0;
#pragma unroll
        for (int q = 0; q < kE; ++q) {
            if (fq[q]) {
                h = 0.0;
                l = 0.0;
            }
            dd_add(h, l, oq[q]);
            sf |= fq[q];
        }
        if (lane == 0 && !sf) dd_merge(h, l, ch, cl);              // the open segment's carry
        double sh = h, sl = l;
        wave_seg_scan_dd(sf, sh, sl);
        if constexpr (kStride) {
            // a lane's first position is a multiple of kE, and kE divides 64, so
            // each 64b + 63 is some lane's last event, where the running total is
            // that lane's inclusive scan
            if (ok[kE - 1] && ((pos + kE - 1) & 63) == 63) nets[(pos + kE - 1) >> 6] = sh + sl;
        } else {
            // the open segment's total before this lane's first event, then the
            // running totals again, event by event, and A of each position
            double rh = __shfl_up(sh, 1, 64), rl = __shfl_up(sl, 1, 64);
            if (lane == 0) {
                rh = ch;
                rl = cl;
            }
            double A[kE];
#pragma unroll
            for (int q = 0; q < kE; ++q) {
                if (fq[q]) {
                    rh = 0.0;
                    rl = 0.0;
                }
                dd_add(rh, rl, oq[q]);
                A[q] = apply_terms(rh + rl, L.aggR, L.aggL);
            }
            // A of the position before each: A_0 before a trial's first event,
            // the lane below's last A before this lane's first, a_prev before the step's
            double before = __shfl_up(A[kE - 1], 1, 64);
            if (lane == 0) before = a_prev;
            double net[kE];
#pragma unroll
            for (int q = 0; q < kE; ++q) net[q] = A[q] - (fq[q] ? A0 : (q == 0 ? before : A[q - 1]));
            a_prev = readlane_f64(A[kE - 1], 63);
            // half a step at a time: lanes [32 hf, 32 hf + 32) hold positions
            // [kW/2 hf, kW/2 (hf + 1)); position i of the half sits at i + i / kE
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if ((lane >> 5) == hf) {
#pragma unroll
                    for (int q = 0; q < kE; ++q) st[(lane & 31) * (kE + 1) + q] = net[q];
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int r = 0; r < kE / 2; ++r) {
                    const int i = r * 64 + lane;
                    const int64_t p = c + hf * (kW / 2) + i;
                    const double v = st[i + i / kE];
                    if (p >= P0 && p < P1) __builtin_nontemporal_store(v, nets + (p - ev0));
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        ch = readlane_f64(sh, 63);
        cl = readlane_f64(sl, 63);
        __builtin_amdgcn_wave_barrier();
        if (lane < kW / 32) fl[lane] = 0;
    }
}

}  // namespace

int part_count(int64_t C) { return static_cast<int>((C + kPartSize - 1) / kPartSize); }

namespace {

// where the time-ordered passes' tables lie in their scratch: probe words, then
// the coarse map, the finest (2^cshift events per bit) that fits its LDS share
struct ProbeTables {
    uint64_t* probe;
    uint32_t* coarse;
    int cshift;
    int64_t n_words, n_cw;
    int64_t bytes;
};
ProbeTables probe_tables(void* scratch, int64_t C) {
    ProbeTables t;
    t.n_words = (C + (1 << kProbeShift) - 1) >> kProbeShift;
    t.cshift = 0;
    while ((((C + (int64_t(1) << t.cshift) - 1) >> t.cshift) + 31) / 32 * 4 > kCoarseBytes) ++t.cshift;
    t.n_cw = (((C + (int64_t(1) << t.cshift) - 1) >> t.cshift) + 31) / 32;
    const int64_t words = (static_cast<int64_t>(sizeof(uint64_t)) * t.n_words + 255) & ~int64_t(255);
    t.bytes = words + kCoarseBytes + 256;
    t.probe = static_cast<uint64_t*>(scratch);
    t.coarse = reinterpret_cast<uint32_t*>(static_cast<char*>(scratch) + words);
    return t;
}
// the fold writes coarse words that lie inside one superblock
bool coarse_in_fold(const ProbeTables& t) { return (int64_t(32) << t.cshift) <= kSuper; }

}  // namespace

int64_t probe_table_bytes(int64_t C) { return probe_tables(nullptr, C).bytes; }

namespace {

// workgroups of the time-ordered passes: a wave per trial at most, all resident
template <typename K>
uint32_t nets_grid(K kernel, size_t lds, int64_t trials, int n_cu) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kNetsThreads, lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    int64_t blocks = (trials + kNetsThreads / 64 - 1) / (kNetsThreads / 64);
    const int64_t cap = static_cast<int64_t>(n_cu) * per_cu;
    return static_cast<uint32_t>(blocks > cap ? cap : blocks);
}

hipError_t finish_tables(const ProbeTables& t, hipStream_t s) {
    if (coarse_in_fold(t)) return hipSuccess;
    hipLaunchKernelGGL(coarse_map_kernel, dim3(static_cast<uint32_t>((t.n_cw + 255) / 256)), dim3(256), 0, s, t.probe,
                       t.n_words, t.cshift, t.n_cw, t.coarse);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_event_nets(const int64_t* offsets, const uint32_t* ids, const void* part_scratch, int P, int64_t C,
                             uint64_t* probe, double density, double events, const LayerArgs& L, double* nets, int n_cu,
                             hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    const PartScratch ps = carve_parts(const_cast<void*>(part_scratch), P);
    const ProbeTables t = probe_tables(probe, C);
    hipError_t e = finish_tables(t, s);
    if (e != hipSuccess) return e;
    const size_t lds = (sizeof(uint32_t) * static_cast<size_t>(t.n_cw) + 15) & ~size_t(15);
    // Scan every event where most pass the coarse map (a queue of almost all
    // events only adds work) and the waves have too few steps each to share the
    // gathers' latency.  Scan against candidates, us per call: 447 trials of 1377
    // events at 0.3 / 0.6 / 1.0 of the catalogue with a loss 93 / 105 / 124 against
    // 94 / 111 / 138, 7001 of 137 73 / 80 / 91 against 75 / 83 / 95; with more events
    // the candidates are as fast or faster at every share: 20000 of 800
    // 146 / 166 / 196 against 132 / 153 / 187, 60000 of 1000 468 / 665 / 1002 against
    // 403 / 643 / 1006.
    const double share =
        -std::expm1(std::log1p(-std::min(density, 1.0 - 1e-12)) * static_cast<double>(int64_t(1) << t.cshift));
    if (share > 0.5 && events < 2048.0 * (kNetsThreads / 64) * n_cu) {
        hipLaunchKernelGGL((event_scan_kernel<8, false>),
                           dim3(nets_grid(event_scan_kernel<8, false>, lds, L.trial_count, n_cu)), dim3(kNetsThreads),
                           lds, s, offsets, ids, t.probe, t.coarse, t.cshift, t.n_cw, ps.stage, L, nets);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(event_nets_kernel, dim3(nets_grid(event_nets_kernel, lds, L.trial_count, n_cu)),
                       dim3(kNetsThreads), lds, s, offsets, ids, t.probe, t.coarse, t.cshift, t.n_cw, ps.stage, L, nets);
    return hipGetLastError();
}

hipError_t launch_stride_checkpoints(const int64_t* offsets, const uint32_t* ids, const void* part_scratch, int P,
                                     int64_t C, uint64_t* probe, const LayerArgs& L, double* stride, int n_cu,
                                     hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    const PartScratch ps = carve_parts(const_cast<void*>(part_scratch), P);
    const ProbeTables t = probe_tables(probe, C);
    hipError_t e = finish_tables(t, s);
    if (e != hipSuccess) return e;
    const size_t lds = (sizeof(uint32_t) * static_cast<size_t>(t.n_cw) + 15) & ~size_t(15);
    hipLaunchKernelGGL((event_scan_kernel<8, true>),
                       dim3(nets_grid(event_scan_kernel<8, true>, lds, L.trial_count, n_cu)), dim3(kNetsThreads), lds,
                       s, offsets, ids, t.probe, t.coarse, t.cshift, t.n_cw, ps.stage, L, stride);
    return hipGetLastError();
}

hipError_t launch_part_fold(const double* o, int64_t C, int P, void* scratch, hipStream_t s, bool with_ranks) {
    PartScratch ps = carve_parts(scratch, P);
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    hipError_t e;
    hipLaunchKernelGGL(part_image_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(256), 0, s, o, C, ps.img,
                       ps.sb_count, int64_t(0), int64_t(0), int64_t(0));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (!with_ranks) return hipSuccess;
    hipLaunchKernelGGL(superblock_scan_kernel, dim3(1), dim3(1024), 0, s, ps.sb_count, n_sb, ps.img, int64_t(0));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(compact_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(256), 0, s, o, C, ps.img, ps.compact,
                       int64_t(0), int64_t(0));
    return hipGetLastError();
}

hipError_t launch_fold_parts(const SparsePool& sp, int64_t C, const LayerArgs& L, const LayerArgs* L_dev, double* o,
                             int P, void* scratch, bool compact, uint64_t* probe, hipStream_t s) {
    PartScratch ps = carve_parts(scratch, P);
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    FoldOut out{o, ps.img, ps.sb_count, ps.stage, nullptr, nullptr, 0, {}, nullptr, nullptr};
    if (probe) {
        const ProbeTables t = probe_tables(probe, C);
        out.probe = t.probe;
        out.coarse = coarse_in_fold(t) ? t.coarse : nullptr;
        out.cshift = t.cshift;
    }
    hipError_t e;
    if (L_dev)
        hipLaunchKernelGGL(fold_image_dev_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(kFoldThreads), 0, s, sp, C, L_dev,
                           out, int64_t(0), int64_t(0));
    else
        hipLaunchKernelGGL(fold_image_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(kFoldThreads), 0, s, sp, C, L, out);
    if ((e = hipGetLastError()) != hipSuccess || !compact) return e;
    hipLaunchKernelGGL(compact_stage_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(256), 0, s, ps.stage,
                       ps.sb_count, ps.img, ps.compact);
    return hipGetLastError();
}

hipError_t launch_fold_back(const SparsePool& sp, int64_t C, const LayerArgs& L, int P, void* scratch,
                            const FoldBack& back, hipStream_t s) {
    FoldOut out{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, back, nullptr, nullptr};
    if (scratch) {
        const PartScratch ps = carve_parts(scratch, P);
        out.img = ps.img;
        out.sb_count = ps.sb_count;
        out.stage = ps.stage;
    }
    hipLaunchKernelGGL(fold_back_kernel, dim3(static_cast<uint32_t>(P) * kBase32), dim3(kFoldThreads), 0, s, sp, C, L,
                       out);
    return hipGetLastError();
}

hipError_t launch_fold_losses(const SparsePool& sp, const LossIndex& ix, int64_t C, const LayerArgs* L,
                              const LayerArgs* L_dev, int n_layers, double* tab, hipStream_t s) {
    if (n_layers < 1 || (!L_dev && n_layers != 1)) return hipErrorInvalidValue;
    const FoldOut out{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, {}, ix.probe, tab};
    const dim3 g(static_cast<uint32_t>(sp.n_chunks), static_cast<uint32_t>(n_layers)), b(kFoldThreads);
    if (L_dev)
        hipLaunchKernelGGL(fold_losses_dev_kernel, g, b, 0, s, sp, C, L_dev, out,
                           static_cast<int64_t>(ix.P) * kLossSlots);
    else
        hipLaunchKernelGGL(fold_losses_kernel, g, b, 0, s, sp, C, *L, out);
    return hipGetLastError();
}

// One workgroup takes a round of kScanChunk entries at a time, 18 us each: past one
// round the chunks are summed side by side, their sums scanned, the chunks scanned
// (1e6 entries: 1100 us in rounds).
hipError_t launch_scan_i64(int64_t* v, int64_t n, hipStream_t s) {
    const int64_t chunks = (n + kScanChunk - 1) / kScanChunk;
    if (chunks <= 1) {
        hipLaunchKernelGGL(sparse_scan_kernel, dim3(1), dim3(1024), 0, s, v, n, nullptr, n);
        return hipGetLastError();
    }
    int64_t* sums = nullptr;
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&sums), sizeof(int64_t) * (chunks + 1), s);
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<uint32_t>(chunks));
    hipLaunchKernelGGL(chunk_sum_kernel, grid, dim3(1024), 0, s, v, n, sums);
    hipLaunchKernelGGL(sparse_scan_kernel, dim3(1), dim3(1024), 0, s, sums, chunks, nullptr, chunks);
    hipLaunchKernelGGL(sparse_scan_kernel, grid, dim3(1024), 0, s, v, n, sums, int64_t(kScanChunk));
    e = hipGetLastError();
    dev_free(sums, s);
    return e;
}

hipError_t launch_fold_batch(const SparsePool& sp, int64_t C, const LayerArgs* L_dev, int n_layers, int P, void* scratch,
                             hipStream_t s) {
    const FoldViews v = fold_batch_views(scratch, n_layers, P);
    const FoldOut out{nullptr, v.img, v.sb_count, v.stage, nullptr, nullptr, 0, {}, nullptr, nullptr};
    hipLaunchKernelGGL(fold_image_dev_kernel, dim3(static_cast<uint32_t>(v.sb_stride), static_cast<uint32_t>(n_layers)),
                       dim3(kFoldThreads), 0, s, sp, C, L_dev, out, v.img_stride, v.sb_stride);
    return hipGetLastError();
}

hipError_t launch_store_terms(const LayerArgs* L, int n, LayerArgs* dst, hipStream_t s) {
    static_assert(offsetof(LayerArgs, J) == 0 && offsetof(LayerArgs, idx) % 8 == 0, "packed layer arguments");
    for (int i = 0; i < n;) {
        TermsPack p{};
        int k = 0, at = 0;
        for (; i + k < n && k < kTermsLayers && at + terms_words(L[i + k].J) <= 864; ++k) {
            const LayerArgs& a = L[i + k];
            const int Je = (a.J + 1) & ~1;
            uint32_t* w = p.words + at;
            p.start[k] = at;
            std::memcpy(w, &a, 4 * kTermsHead);
            std::memcpy(w + kTermsHead, a.idx, 4 * static_cast<size_t>(a.J));
            std::memcpy(w + kTermsHead + Je, a.R, 8 * static_cast<size_t>(a.J));
            std::memcpy(w + kTermsHead + Je + 2 * a.J, a.Lim, 8 * static_cast<size_t>(a.J));
            at += terms_words(a.J);
        }
        hipLaunchKernelGGL(store_terms_kernel, dim3(static_cast<uint32_t>(k)), dim3(256), 0, s, p, dst + i);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        i += k;
    }
    return hipSuccess;
}

hipError_t launch_part_pass(const PartLayout& lay, int64_t N, const LayerArgs& L, void* scratch, double* ylt,
                            double* S, int n_cu, hipStream_t s, int lpt) {
    if (L.trial_count <= 0) return hipSuccess;
    const int P = lay.P;
    PartScratch ps = carve_parts(scratch, P);
    hipError_t e;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, ps.counter, int64_t(1), 0u);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    PartPassArgs a{};
    a.pids = lay.pids;
    a.seg_rel = lay.seg_rel;
    a.tile_start = lay.tile_start;
    a.img = ps.img;
    a.compact = ps.compact;
    a.N = N;
    a.P = P;
    a.T = lay.T;
    a.t_lo = L.trial_begin;
    a.t_hi = L.trial_begin + L.trial_count;
    a.first_tile = L.trial_begin / lay.T;
    a.last_tile = (a.t_hi + lay.T - 1) / lay.T;
    a.aggR = L.aggR;
    a.aggL = L.aggL;
    a.ylt = ylt;
    a.S = S;
    a.tile_counter = ps.counter;
    int64_t grid = a.last_tile - a.first_tile;
    if (grid > int64_t(n_cu) * 2) grid = int64_t(n_cu) * 2;
    return launch_part_pass_lpt(lpt, static_cast<int>(grid), a, s);
}

}  // namespace ara

namespace ara {

hipError_t launch_part_adjoint(const PartLayout& lay, int64_t N, const LayerArgs& L, void* part_scratch,
                               const double* S, const double* ylt, const TailStats* tail, uint64_t* w_mean,
                               uint64_t* w_tvar, int n_cu, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    PartScratch ps = carve_parts(part_scratch, lay.P);
    hipError_t e;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, ps.counter, int64_t(1), 0u);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    PartAdjArgs a{};
    a.pids = lay.pids;
    a.seg_rel = lay.seg_rel;
    a.tile_start = lay.tile_start;
    a.img = ps.img;
    a.N = N;
    a.P = lay.P;
    a.T = lay.T;
    a.t_lo = L.trial_begin;
    a.t_hi = L.trial_begin + L.trial_count;
    a.first_tile = L.trial_begin / lay.T;
    a.last_tile = (a.t_hi + lay.T - 1) / lay.T;
    a.aggR = L.aggR;
    a.aggL = L.aggL;
    a.S = S;
    a.ylt = ylt;
    a.tail = tail;
    a.w_mean = w_mean;
    a.w_tvar = w_tvar;
    a.tile_counter = ps.counter;
    a.sb_count = ps.sb_count;
    if (lay.length < (int64_t(1) << 32)) {
        // one workgroup per CU, a multiple of the XCD count (see xcd_adjoint_kernel)
        int64_t grid = int64_t(n_cu);
        grid -= grid % kXcds;
        if (grid < kXcds) grid = kXcds;
        hipLaunchKernelGGL(xcd_adjoint_kernel, dim3(static_cast<uint32_t>(grid)), dim3(1024), 0, s, a, kXcds);
        return hipGetLastError();
    }
    int64_t grid = a.last_tile - a.first_tile;
    if (grid > int64_t(n_cu) * 2) grid = int64_t(n_cu) * 2;
    hipLaunchKernelGGL(part_adjoint_kernel, dim3(static_cast<uint32_t>(grid)), dim3(512), 0, s, a);
    return hipGetLastError();
}

}  // namespace ara

namespace ara {

int64_t batched_scratch_bytes(int64_t C, int P, int n_layers, int64_t n_items, int64_t n_elts_total) {
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    int64_t b = 0;
    b += sizeof(double) * C * n_layers;                  // o
    b += sizeof(double) * C * n_layers;                  // compact
    b += part_image_bytes(P) * n_layers;                 // images
    b += sizeof(uint32_t) * n_sb * n_layers;             // superblock counts
    b += 256;                                            // counter
    b += sizeof(int2) * n_items + 256;
    b += sizeof(BatchLayerDesc) * n_layers + sizeof(BatchFoldDesc) * n_layers + 512;
    b += (sizeof(int32_t) + 2 * sizeof(double)) * n_elts_total + 512;
    return b;
}

BatchedScratch carve_batched(void* scratch, int64_t C, int P, int n_layers, int64_t n_items, int64_t n_elts_total) {
    char* p = static_cast<char*>(scratch);
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    BatchedScratch r;
    r.o = reinterpret_cast<double*>(p);
    p += sizeof(double) * C * n_layers;
    r.compact = reinterpret_cast<double*>(p);
    p += sizeof(double) * C * n_layers;
    r.img = reinterpret_cast<uint8_t*>(p);
    p += part_image_bytes(P) * n_layers;
    r.sb_count = reinterpret_cast<uint32_t*>(p);
    p += sizeof(uint32_t) * n_sb * n_layers;
    r.counter = reinterpret_cast<uint32_t*>(p);
    p += 256;
    r.items = reinterpret_cast<int2*>(p);
    p += sizeof(int2) * n_items + 256;
    r.layers = reinterpret_cast<BatchLayerDesc*>(p);
    p += sizeof(BatchLayerDesc) * n_layers;
    r.fold = reinterpret_cast<BatchFoldDesc*>(p);
    p += sizeof(BatchFoldDesc) * n_layers + 512;
    r.R = reinterpret_cast<double*>(p);
    p += sizeof(double) * n_elts_total;
    r.Lim = reinterpret_cast<double*>(p);
    p += sizeof(double) * n_elts_total;
    r.idx = reinterpret_cast<int32_t*>(p);
    return r;
}

hipError_t launch_batched(const PartLayout& lay, int64_t N, int64_t C, const double* elts, int n_layers,
                          const BatchedScratch& b, int64_t n_items, double* ylt, int n_cu, hipStream_t s,
                          hipEvent_t pass_start, hipEvent_t pass_stop, int lpt) {
    hipError_t e;
    const int P = lay.P;
    const int64_t n_sb = static_cast<int64_t>(P) * kBase32;
    const int64_t img_stride = part_image_bytes(P);
    hipLaunchKernelGGL(batched_fold_kernel, dim3(static_cast<uint32_t>((C + 255) / 256), n_layers), dim3(256), 0, s,
                       elts, C, b.fold, b.idx, b.R, b.Lim, b.o);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(part_image_kernel, dim3(static_cast<uint32_t>(n_sb), n_layers), dim3(256), 0, s, b.o, C, b.img,
                       b.sb_count, C, img_stride, n_sb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(superblock_scan_kernel, dim3(1, n_layers), dim3(1024), 0, s, b.sb_count, n_sb, b.img,
                       img_stride);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(compact_kernel, dim3(static_cast<uint32_t>(n_sb), n_layers), dim3(256), 0, s, b.o, C, b.img,
                       b.compact, C, img_stride);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, b.counter, int64_t(1), 0u);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    BatchedPassArgs a{};
    a.pids = lay.pids;
    a.seg_rel = lay.seg_rel;
    a.tile_start = lay.tile_start;
    a.img = b.img;
    a.img_stride = img_stride;
    a.compact = b.compact;
    a.C = C;
    a.N = N;
    a.P = P;
    a.T = lay.T;
    a.items = b.items;
    a.n_items = static_cast<int32_t>(n_items);
    a.layers = b.layers;
    a.ylt = ylt;
    a.item_counter = b.counter;
    int64_t grid = n_items < int64_t(n_cu) * 2 ? n_items : int64_t(n_cu) * 2;
    if (grid < 1) grid = 1;
    if (pass_start && (e = hipEventRecord(pass_start, s)) != hipSuccess) return e;
    if ((e = launch_batched_pass_lpt(lpt, static_cast<int>(grid), a, s)) != hipSuccess) return e;
    if (pass_stop && (e = hipEventRecord(pass_stop, s)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace ara

namespace ara {

hipError_t launch_xcd_pass(const PartLayout& lay, int64_t N, int64_t C, const LayerArgs& L, void* part_scratch,
                           double* partials, int n_cu, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    const int P = lay.P;
    PartScratch ps = carve_parts(part_scratch, P);
    XcdPassArgs a{};
    a.pids = lay.pids;
    a.seg_rel = lay.seg_rel;
    a.tile_start = lay.tile_start;
    a.img = ps.img;
    a.compact = ps.compact;
    a.C = C;
    a.N = N;
    a.P = P;
    a.T = lay.T;
    a.t_lo = L.trial_begin;
    a.t_hi = L.trial_begin + L.trial_count;
    a.first_tile = L.trial_begin / lay.T;
    a.last_tile = (a.t_hi + lay.T - 1) / lay.T;
    a.part_hi = partials;
    a.part_lo = partials + static_cast<int64_t>(P) * L.trial_count;
    a.pad = lay.pids + lay.length;
    a.n_xcd = kXcds;
    // one 1024-thread workgroup per CU (its LDS holds the part image and the
    // loss cache), a multiple of the XCD count so every XCD gets the same share
    int64_t grid = int64_t(n_cu);
    grid -= grid % kXcds;
    if (grid < kXcds) grid = kXcds;
    hipLaunchKernelGGL(xcd_pass_kernel, dim3(static_cast<uint32_t>(grid)), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_xcd_combine(const PartLayout& lay, const LayerArgs& L, const LayerArgs* L_dev,
                              const double* partials, double* ylt, double* S, hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    const int P = lay.P;
    const int64_t blocks = (L.trial_count + 255) / 256;
    hipLaunchKernelGGL(xcd_combine_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s, partials,
                       partials + static_cast<int64_t>(P) * L.trial_count, P, L.trial_count, L.aggR, L.aggL, L_dev, ylt,
                       S);
    return hipGetLastError();
}

}  // namespace ara
