// Streaming pass over the events that can lose: a second 16-bit copy of the YET
// that holds only the events with a loss in some table of the ELT pool.
//
// An event without a loss in any table of the pool adds zero to every layer, so
// the passes over layers need not read it.  At table creation the pool's events
// are numbered in catalogue order and cut into parts of at most kSlots - 1, whole
// superblocks of 4096 catalogue events each; per request the fold writes o(E) to
// the event's slot of a table per part, zero where the layer has no loss, and a
// workgroup copies its part's table to LDS: an event costs one LDS read and a
// double-double addition, no test, queue or rank.  Zeros leave a double-double sum
// unchanged, so the sums are those of the full copy.
//
// A lane sums one trial: the copy holds the slots of 64 consecutive trials row by
// row, four slots of each lane's trial, short trials padded with the slot that is
// always zero.  A row is one 8-byte load per lane at consecutive addresses, nothing
// goes through LDS, no lane asks where its trial ends, and the sums leave in
// consecutive stores.  (Sorting windows of 1024 trials by their counts saves four
// rows in ten, but then each lane's sum goes to a line of its own: 290 us where this
// order took 190.)  In larger copies a lane holds two trials, one of each half of a
// group of 128, the shorter ones with the longer ones: a third less padding, and the
// sums still leave in the group's own lines.  Bit 15 of a row's first slot ends the
// lane's first trial, those of the others give the trials' places in the group, three
// bits a row.  Parts whose trials are long and few are cut into columns (splits of each
// trial's events) to fill the chip.  Partial sums per (column, trial) merge as those of
// the full copy do.
//
// Bound: the rows' bytes and, next to it, 28 fp64 additions and four LDS reads a row.
// 10^6 trials of 1000 events, 16 tables of 20000 events in 2 * 10^6 (15 % of the
// events): 155 us with a trial per lane (600 MB of rows), 128 with two (400 MB); the
// full copy's pass 590 us.
// Compiled as a part of kernels_portfolio.hip.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>
#include <vector>

#include "ara_internal.hpp"

namespace ara {

namespace {

constexpr int kSlots = kLossSlots;
constexpr int kSuperEvents = 4096;
constexpr uint32_t kPadSlot = kSlots - 1;       // always zero, never an event's
constexpr int kRowIds = 4;                      // slots per lane and row
constexpr int kSlotBits = 0x7FFF;               // of a slot's 16 bits; the last is free for marks
constexpr int kMetaRows = 4;                    // least rows of a group whose lanes hold two trials

// ---------------------------------------------------------------------------
// the pool's events
// ---------------------------------------------------------------------------

// per superblock: the bits of its events with a loss in some table (low halves of
// the probe words) and their number.  A wave takes a table; a lane joins the bits of four
// consecutive events, as the entries are in order and dense tables queue up on a word
// (16 tables of 3700 events per superblock: an event per lane and load 41 us, and 69 in
// four waves, now 12)
__global__ __launch_bounds__(1024) void loss_bits_kernel(SparsePool sp, int n_rows, int64_t C,
                                                        uint64_t* __restrict__ probe, uint32_t* __restrict__ count) {
    __shared__ uint32_t bits[kSuperEvents / 32];
    __shared__ uint32_t total;
    const int64_t sb = blockIdx.x;
    for (int i = threadIdx.x; i < kSuperEvents / 32; i += blockDim.x) bits[i] = 0;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    for (int r = threadIdx.x >> 6; r < n_rows; r += static_cast<int>(blockDim.x >> 6)) {
        const int64_t key = static_cast<int64_t>(r) * sp.n_chunks + sb, end = sp.chunk_off[key + 1];
        for (int64_t k = sp.chunk_off[key] + 4 * (threadIdx.x & 63); k < end; k += 256) {
            uint32_t ev[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) ev[u] = sp.ev[min(k + u, end - 1)];
            uint32_t own = 0;                       // of ev[u]'s word
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                own |= 1u << (ev[u] & 31u);
                if (u < 3 && ev[u + 1] >> 5 == ev[u] >> 5) continue;
                atomicOr(&bits[ev[u] >> 5], own);
                own = 0;
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kSuperEvents / 32; i += blockDim.x) {
        const int64_t w = sb * (kSuperEvents / 32) + i;
        if (w < (C + 31) / 32) probe[w] = bits[i];
        if (bits[i]) atomicAdd(&total, static_cast<uint32_t>(__popc(bits[i])));
    }
    __syncthreads();
    if (threadIdx.x == 0) count[sb] = total;
}

// what the host asks of the plan
struct LossPlan {
    int64_t kept;                   // occurrences in the YET of events with a loss (the scan's total)
    int64_t events;                 // with a loss in some table
    int32_t parts;                  // past `most_parts`: more than there may be
    int32_t pad_;
};
// and of the intermediate copy and the rows: findings, the rows of each column
struct LossRows {
    CreateResult res;
    int64_t rows[kMaxStreamParts * 64];
};

// the superblocks' counts in place[] to the places of their first events, part << 16 |
// slot: whole superblocks to a part, its last slot kept free (one wave)
__global__ __launch_bounds__(64) void loss_plan_kernel(int64_t n_sb, int most_parts, uint32_t* __restrict__ place,
                                                       uint32_t* __restrict__ part_n, LossPlan* __restrict__ plan,
                                                       CreateResult* __restrict__ res) {
    const int lane = threadIdx.x;
    if (lane == 0) res->flags = 0;
    int part = 0;
    uint32_t at = 0;
    int64_t events = 0;
    for (int64_t k0 = 0; k0 < n_sb; k0 += 64) {
        const uint32_t own = k0 + lane < n_sb ? place[k0 + lane] : 0u;
        uint32_t mine = 0;
        for (int i = 0; i < 64; ++i) {
            const uint32_t n = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(own), i));
            if (at + n > kPadSlot) {
                if (part < most_parts && lane == 0) part_n[part] = at;
                if (part < most_parts) ++part;
                at = 0;
            }
            if (i == lane) mine = static_cast<uint32_t>(part) << 16 | at;
            at += n;
            events += n;
        }
        if (k0 + lane < n_sb) place[k0 + lane] = mine;
    }
    if (lane == 0) {
        if (part < most_parts) part_n[part] = at;
        plan->events = events;
        plan->parts = part + 1;
    }
}

// per superblock (one wave): the slots of its events, the first one's at place[sb],
// to the high halves of the probe words, and the events of the slots
__global__ __launch_bounds__(64) void loss_place_kernel(int64_t C, int most_parts, const uint32_t* __restrict__ place,
                                                        uint64_t* __restrict__ probe, uint32_t* __restrict__ events) {
    const int64_t sb = blockIdx.x;
    const int lane = threadIdx.x;
    uint32_t at = place[sb];
    if (static_cast<int>(at >> 16) >= most_parts) return;              // not used
    for (int h = 0; h < kSuperEvents / 32 / 64; ++h) {
        const int64_t w = sb * (kSuperEvents / 32) + h * 64 + lane;
        const uint32_t bits = w < (C + 31) / 32 ? static_cast<uint32_t>(probe[w]) : 0u;
        uint32_t inc = static_cast<uint32_t>(__popc(bits));
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        uint32_t first = at + inc - static_cast<uint32_t>(__popc(bits));
        if (w < (C + 31) / 32) probe[w] = (static_cast<uint64_t>(first) << 32) | bits;
        for (uint32_t b = bits; b; b &= b - 1, ++first)
            events[static_cast<int64_t>(first >> 16) * kSlots + (first & 0xFFFFu)] =
                static_cast<uint32_t>(w * 32 + __builtin_ctz(b));
        at += static_cast<uint32_t>(__shfl(static_cast<int>(inc), 63, 64));
    }
}

// Per trial (one wave): its events with a loss, counted (kFill false) or their
// part << 16 | slot stored in order from start[t] on and counted per part
// (cnt[t][part]).  A probe word is a gather from
// L2, 64 lines an instruction: 5.2 ms per 1e9 events with a gather each.  So a
// workgroup holds a map with a bit per 2^shift events in LDS and gathers the words of
// the events whose bit is set (the other lanes share the first word's line): 2.1 ms
// at 15 % of the events.  kExact, a bit per event: the map is the words' low halves,
// and the count gathers nothing; the high halves lie in LDS too where they fit
// (5e7 events, 84 % of them with a loss: count 183 -> 68 us, fill 208 -> 110).
constexpr int kMapWords = 39936;                // 156 KB
constexpr int kMapShift = 2;
static_assert(int64_t(kMaxStreamParts) << kStreamShift <= int64_t(kMapWords) * 32 << kMapShift,
              "a map for every catalogue with a 16-bit copy");
inline int64_t filter_words(bool fill, bool exact, int64_t n_words) {
    return !exact ? kMapWords : (fill && 2 * n_words <= kMapWords ? 2 * n_words : n_words);
}
template <bool kFill, int kAhead, bool kExact>
__global__ __launch_bounds__(1024) void loss_filter_kernel(const int64_t* __restrict__ offsets,
                                                           const uint32_t* __restrict__ ids, int64_t N,
                                                           const uint64_t* __restrict__ probe, int64_t n_words,
                                                           int shift, int64_t* __restrict__ start,
                                                           uint32_t* __restrict__ out, int P,
                                                           int32_t* __restrict__ cnt) {
    extern __shared__ uint32_t map[];               // filter_words
    __shared__ uint32_t counts[16][kMaxStreamParts];
    const bool whole = kExact && kFill && 2 * n_words <= kMapWords;
    if constexpr (kExact) {
        for (int64_t w = threadIdx.x; w < n_words; w += blockDim.x) {
            const uint64_t v = probe[w];
            map[w] = static_cast<uint32_t>(v);
            if (whole) map[n_words + w] = static_cast<uint32_t>(v >> 32);
        }
    } else {
        for (int i = threadIdx.x; i < kMapWords; i += blockDim.x) map[i] = 0;
        __syncthreads();
        for (int64_t w = threadIdx.x; w < n_words; w += blockDim.x) {
            uint32_t b = static_cast<uint32_t>(probe[w]);
            if (shift >= 1) {                       // pairs, then fours, to the low bits
                b = (b | b >> 1) & 0x55555555u;
                b = (b | b >> 1) & 0x33333333u;
                b = (b | b >> 2) & 0x0F0F0F0Fu;
                b = (b | b >> 4) & 0x00FF00FFu;
                b = (b | b >> 8) & 0x0000FFFFu;
            }
            if (shift >= 2) {
                b = (b | b >> 1) & 0x55555555u;
                b = (b | b >> 1) & 0x33333333u;
                b = (b | b >> 2) & 0x0F0F0F0Fu;
                b = (b | b >> 4) & 0x00FF00FFu;
            }
            const int per = 32 >> shift;            // bits of the map a word gives
            if (b) atomicOr(&map[w * per >> 5], b << (static_cast<int>(w * per) & 31));
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    uint32_t* count = counts[threadIdx.x >> 6];     // this wave's
    if (kFill && lane < P) count[lane] = 0;
    const int64_t n_waves = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    for (int64_t t = uniform_i64((static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6); t < N;
         t += n_waves) {
        const int64_t b = uniform_i64(offsets[t]), e = uniform_i64(offsets[t + 1]);
        int64_t to = kFill ? uniform_i64(start[t]) : 0;
        for (int64_t c = b; c < e; c += 64 * kAhead) {
            uint32_t id[kAhead], bits[kAhead], first[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) id[k] = ids[min(c + k * 64 + lane, e - 1)];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const uint32_t at = id[k] >> 5;
                if constexpr (kExact) {
                    bits[k] = map[at];
                    if constexpr (kFill) {
                        if (whole) first[k] = map[n_words + at];
                        else first[k] = static_cast<uint32_t>(probe[bits[k] >> (id[k] & 31u) & 1u ? at : 0u] >> 32);
                    }
                } else {
                    const uint32_t m = id[k] >> shift;
                    const bool may = map[m >> 5] >> (m & 31u) & 1u;
                    const uint64_t w = probe[may ? at : 0u];
                    bits[k] = may ? static_cast<uint32_t>(w) : 0u;
                    first[k] = static_cast<uint32_t>(w >> 32);
                }
            }
#pragma unroll
            for (int k = 0; k < kAhead; ++k) {
                const bool keep = c + k * 64 + lane < e && (bits[k] >> (id[k] & 31u) & 1u);
                const uint64_t kept = __ballot(keep);
                if (kFill && keep) {
                    const uint32_t slot = first[k] + __popc(bits[k] & ((1u << (id[k] & 31u)) - 1u));
                    out[to + __popcll(kept & ((1ull << lane) - 1))] = slot;
                    if (P > 1) atomicAdd(&count[slot >> 16], 1u);
                }
                to += __popcll(kept);
            }
        }
        if (!kFill && lane == 0) start[t] = to;
        if (kFill && P == 1 && lane == 0) cnt[t] = static_cast<int32_t>(to - start[t]);
        if (kFill && P > 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < P) {
                cnt[t * P + lane] = static_cast<int32_t>(count[lane]);
                count[lane] = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
}

// ---------------------------------------------------------------------------
// the copy, from the kept events part by part (a StreamLayout of their slots)
// ---------------------------------------------------------------------------

// IDs of trial t in part p of the intermediate copy: [from, to) in the part's stream
__device__ __forceinline__ void stream_segment(const StreamLayout& in, int p, int64_t t, uint32_t& from, uint32_t& to) {
    const int64_t g = t / in.G;
    const int i = static_cast<int>(t - g * in.G);
    const uint32_t start = in.gstart[static_cast<int64_t>(p) * (in.NG + 1) + g];
    const uint16_t* ends = in.gend + (static_cast<int64_t>(p) * in.NG + g) * kStreamGroupSlots;
    from = start + (i ? ends[i - 1] : 0u);
    to = start + ends[i];
}

// A lane of a paired group holds one trial of its first 64 and one of its last 64, the
// i-th shortest of the ones with the i-th longest of the others, so that the lanes'
// rows differ little.  Both trials' slots, and where they are in the group:
struct Pair {
    uint32_t from_a, to_a, from_b, to_b;
    int rows_a, rows_b;                         // the first trial has a row even when empty
    int pos_a, pos_b;
};
__device__ __forceinline__ int rank_of(int v, int lane) {
    int rank = 0;
    for (int i = 0; i < 64; ++i) {
        const int o = __builtin_amdgcn_readlane(v, i);
        rank += (o < v || (o == v && i < lane)) ? 1 : 0;
    }
    return rank;
}
__device__ __forceinline__ Pair pair_of(const StreamLayout& in, int p, int64_t t0, int64_t N, int s, int S, int lane) {
    uint32_t from[2] = {0, 0}, to[2] = {0, 0};
    int rows[2], rank[2];
    for (int h = 0; h < 2; ++h) {
        const int64_t t = t0 + h * 64 + lane;
        if (t < N) stream_segment(in, p, t, from[h], to[h]);
        const uint64_t n = to[h] - from[h];
        to[h] = from[h] + static_cast<uint32_t>(n * (s + 1) / S);
        from[h] += static_cast<uint32_t>(n * s / S);
        rows[h] = static_cast<int>(to[h] - from[h] + kRowIds - 1) / kRowIds;
        if (h == 0 && rows[h] == 0) rows[h] = 1;
        rank[h] = rank_of(rows[h], lane);
    }
    rank[1] = 63 - rank[1];
    Pair q;
    auto push = [](int to_lane, int v) { return __builtin_amdgcn_ds_permute(to_lane * 4, v); };
    q.from_a = static_cast<uint32_t>(push(rank[0], static_cast<int>(from[0])));
    q.to_a = static_cast<uint32_t>(push(rank[0], static_cast<int>(to[0])));
    q.rows_a = push(rank[0], rows[0]);
    q.pos_a = push(rank[0], lane);
    q.from_b = static_cast<uint32_t>(push(rank[1], static_cast<int>(from[1])));
    q.to_b = static_cast<uint32_t>(push(rank[1], static_cast<int>(to[1])));
    q.rows_b = push(rank[1], rows[1]);
    q.pos_b = push(rank[1], lane);
    return q;
}

// one wave per (part, group): the rows of its splits to their places in gstart
template <bool kPair>
__global__ __launch_bounds__(256) void loss_group_kernel(StreamLayout in, int64_t N, int S, int64_t NG,
                                                         uint32_t* __restrict__ gstart) {
    const int lane = threadIdx.x & 63;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (g >= NG) return;
    const int p = static_cast<int>(blockIdx.y);
    uint32_t from = 0, to = 0;
    if (!kPair && g * 64 + lane < N) stream_segment(in, p, g * 64 + lane, from, to);
    const uint64_t n = to - from;
    for (int s = 0; s < S; ++s) {
        uint32_t rows = static_cast<uint32_t>(n * (s + 1) / S - n * s / S + kRowIds - 1) / kRowIds;
        if constexpr (kPair) {
            const Pair q = pair_of(in, p, g * 128, N, s, S, lane);
            rows = static_cast<uint32_t>(q.rows_a + q.rows_b);
        }
        for (int off = 32; off >= 1; off >>= 1)
            rows = max(rows, static_cast<uint32_t>(__shfl_xor(static_cast<int>(rows), off, 64)));
        // at least one, so that every group ends with a row
        if (lane == 0)
            gstart[(static_cast<int64_t>(p) * S + s) * (NG + 1) + g] = max(rows, static_cast<uint32_t>(kPair ? kMetaRows : 1));
    }
}

// per column: exclusive sums of its groups' rows in place, the total to rows[q]
__global__ __launch_bounds__(1024) void loss_scan_kernel(int64_t NG, uint32_t* __restrict__ gstart,
                                                         int64_t* __restrict__ rows) {
    __shared__ int64_t tsum[1024];
    uint32_t* v = gstart + static_cast<int64_t>(blockIdx.x) * (NG + 1);
    const int64_t per = (NG + 1023) / 1024, j0 = static_cast<int64_t>(threadIdx.x) * per;
    int64_t local = 0;
    for (int64_t j = j0; j < j0 + per && j < NG; ++j) local += v[j];
    tsum[threadIdx.x] = local;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t add = static_cast<int>(threadIdx.x) >= off ? tsum[threadIdx.x - off] : 0;
        __syncthreads();
        tsum[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = tsum[threadIdx.x] - local;
    for (int64_t j = j0; j < j0 + per && j < NG; ++j) {
        const uint32_t size = v[j];
        v[j] = static_cast<uint32_t>(run);
        run += size;
    }
    if (threadIdx.x == 1023) {
        v[NG] = static_cast<uint32_t>(tsum[1023]);
        rows[blockIdx.x] = tsum[1023];
    }
}

// the columns' first slots from their rows (one wave)
__global__ __launch_bounds__(64) void loss_bases_kernel(int Q, const int64_t* __restrict__ rows,
                                                        int64_t* __restrict__ base) {
    const int lane = threadIdx.x;
    int64_t carry = 0;
    for (int q0 = 0; q0 < Q; q0 += 64) {
        int64_t inc = q0 + lane < Q ? rows[q0 + lane] * 64 * kRowIds : 0;
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        if (q0 + lane < Q) base[q0 + lane + 1] = carry + inc;
        carry += __shfl(inc, 63, 64);
    }
    if (lane == 0) base[0] = 0;
}

// One wave per (column, group): the rows.  A lane's 16 slots of four rows are two
// 16-byte loads at the slot's own alignment; what they read past the lane's last slot
// (inside the copy's padding) is masked.  One load per slot asked the L2 for a line
// each, as 32 waves' lines do not stay in the first-level cache: 2500 us for 288M
// slots, this 480.
struct __attribute__((packed, aligned(2))) FourRows {
    uint64_t row[4];
};
__device__ __forceinline__ uint64_t padded(uint64_t row, uint32_t at, uint32_t to) {
    constexpr uint64_t kPadRow = kPadSlot * 0x0001000100010001ull;
    const uint32_t n = at < to ? to - at : 0u;
    const uint64_t valid = n >= kRowIds ? ~0ull : (1ull << (16 * n)) - 1;
    return (row & valid) | (kPadRow & ~valid);
}
template <bool kPair>
__global__ __launch_bounds__(256) void loss_rows_kernel(StreamLayout in, int64_t N, int S, int64_t NG,
                                                        const uint32_t* __restrict__ gstart,
                                                        const int64_t* __restrict__ base, uint64_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t g = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (g >= NG) return;
    const int q = static_cast<int>(blockIdx.y), p = q / S, s = q - p * S;
    const uint16_t* ids = in.ids + in.part_base[p];
    const uint32_t r0 = gstart[static_cast<int64_t>(q) * (NG + 1) + g], r1 = gstart[static_cast<int64_t>(q) * (NG + 1) + g + 1];
    uint64_t* dst = out + (base[q] / (64 * kRowIds) + r0) * 64 + lane;
    FourRows v;
    if constexpr (kPair) {
        const Pair c = pair_of(in, p, g * 128, N, s, S, lane);
        const int meta = c.pos_a | c.pos_b << 6;
        // each lane copies its two trials by itself: the second starts where the first ends
        const int rows = static_cast<int>(r1 - r0);
        auto put = [&](int r, uint64_t row) {
            if (r == c.rows_a - 1) row |= 0x8000ull;            // the first trial's last row
            if (r < kMetaRows) {                                // the trials' places, three bits a row
                const uint64_t m = static_cast<uint64_t>(meta >> (3 * r) & 7);
                row |= (m & 1) << 31 | (m & 2) << 46 | (m & 4) << 61;
            }
            if (r < rows) dst[static_cast<int64_t>(r) * 64] = row;
        };
        for (int r = 0; r < c.rows_a; r += 4) {
            const uint32_t at = c.from_a + static_cast<uint32_t>(r) * kRowIds;
            __builtin_memcpy(&v, ids + min(at, c.to_a), sizeof(v));
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r + k < c.rows_a) put(r + k, padded(v.row[k], at + k * kRowIds, c.to_a));
        }
        for (int r = 0; r < rows - c.rows_a; r += 4) {
            const uint32_t at = c.from_b + static_cast<uint32_t>(r) * kRowIds;
            __builtin_memcpy(&v, ids + min(at, c.to_b), sizeof(v));
#pragma unroll
            for (int k = 0; k < 4; ++k) put(c.rows_a + r + k, padded(v.row[k], at + k * kRowIds, c.to_b));
        }
        return;
    }
    const int64_t t = g * 64 + lane;
    uint32_t from = 0, to = 0;
    if (t < N) stream_segment(in, p, t, from, to);
    const uint64_t n = to - from;
    to = from + static_cast<uint32_t>(n * (s + 1) / S);
    from += static_cast<uint32_t>(n * s / S);
    for (uint32_t r = r0; r < r1; r += 4, from += 4 * kRowIds, dst += 4 * 64) {
        __builtin_memcpy(&v, ids + min(from, to), sizeof(v));
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (r + k < r1) dst[64 * k] = padded(v.row[k], from + k * kRowIds, to);
    }
}

// ---------------------------------------------------------------------------
// the pass
// ---------------------------------------------------------------------------

// one layer over one range of trials: its (column, group) items follow the
// earlier segments' in the work list
struct LossSeg {
    int64_t t_lo, t_hi;
    int64_t g_lo;                   // first group that holds its trials
    int64_t groups;                 // groups per column
    int64_t w0;                     // items before it
    int64_t part_at;                // its partial sums' place
    int64_t layer;
};
constexpr int kMaxSegs = 32;
struct LossSegs {
    LossSeg seg[kMaxSegs];
};
struct LossPassArgs {
    const uint64_t* rows;           // [row][64]: four slots of each lane's trial (or trials)
    const int64_t* col_base;        // a column's first slot in the copy (64 x 4 to a row)
    const double* tab;              // [layer][part][kSlots]
    const uint32_t* part_n;         // slots in use of each part
    int Q, S, P, n_seg;             // columns, columns per part, parts
    int whole;                      // a workgroup's share lies in one part (whole_share)
    int64_t NG;
    int64_t work;
    double* part_hi;
    float* part_lo;
};
struct LossAdjArgs {
    uint32_t* counts;               // [workgroup + part][kSlots]: what a workgroup counted in a part
    uint64_t* w_tvar;               // [part][kSlots], zeroed by the caller
    int64_t masks_lo, masks_n;      // the 64-trial groups that have class masks
    const TailStats* tail;
};

// Workgroups [p n_wg / P, (p + 1) n_wg / P) share part p's items evenly: each loads (or
// clears and stores) one table, and its waves' shares are not cut at a part's end.
// Passes in us, cut where the part ends and whole: 100003 trials of 500 events in 21
// parts 45.3 / 39.1, 10^6 in 15 parts 129.7 / 124.5, 500000 71.8 / 67.8, their backward
// 62.8 / 59.7; with a group or two per wave the divisions cost more (7.9 / 8.9).
__device__ __host__ __forceinline__ int64_t first_wg(int64_t p, int64_t n_wg, int P) { return (p * n_wg + P - 1) / P; }
__device__ __forceinline__ void whole_share(int64_t l, int64_t n_wg, int P, int64_t items, int64_t& begin, int64_t& end) {
    const int64_t p = l * P / n_wg, f = first_wg(p, n_wg, P), c = first_wg(p + 1, n_wg, P) - f;
    begin = p * items + (l - f) * items / c;
    end = p * items + (l - f + 1) * items / c;
}

// The forward (kAdj false) sums; the backward counts the occurrences of each slot
// in the trials inside the aggregate band in LDS.  A wave takes consecutive groups
// of a column, whose rows lie one after the other: eight rows are in flight (twelve in
// paired groups, which read the places from a group's first four when it starts),
// whatever group they belong to, as nothing but their loads and the groups' stores
// uses the vector memory counter (group ends and class masks are scalar loads) and
// the loop leaves in whole rounds only.  With a group's first rows read ahead and
// its others on their own, the forward above took 260 us and its backward at half
// the trials 160, with the ring of rows 155 and 75, in paired groups 128 and 66.
template <bool kAdj, bool kPair>
__global__ __launch_bounds__(1024) void loss_pass_kernel(LossPassArgs a, LossSegs segs, LossAdjArgs adj,
                                                         const uint32_t* __restrict__ gstart,
                                                         const uint64_t* __restrict__ cls_masks) {
    constexpr int kAhead = kPair ? 12 : 8;          // rows read ahead
    constexpr int kTrials = kPair ? 128 : 64;       // of a group
    __shared__ __attribute__((aligned(16))) uint8_t lds[(kAdj ? 4 : 8) * kSlots];
    double* vals = reinterpret_cast<double*>(lds);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    TailStats ts{};
    if constexpr (kAdj) ts = *adj.tail;
    // each XCD takes a contiguous share of the items
    const int64_t n_wg = gridDim.x;
    const int64_t l = n_wg % kXcds ? static_cast<int64_t>(blockIdx.x)
                                   : static_cast<int64_t>(blockIdx.x % kXcds) * (n_wg / kXcds) + blockIdx.x / kXcds;
    int64_t w_begin = l * a.work / n_wg, w_end = (l + 1) * a.work / n_wg;
    if (a.whole) whole_share(l, n_wg, a.P, a.work / a.P, w_begin, w_end);
    int held = -1;                                  // the part whose table (counters) LDS holds
    int64_t held_layer = -1;
    auto flush_counts = [&] {
        __syncthreads();
        u32x4* to = reinterpret_cast<u32x4*>(adj.counts + (l + held) * kSlots);
        for (int i = threadIdx.x; i < kSlots / 4; i += blockDim.x) to[i] = reinterpret_cast<const u32x4*>(cnt)[i];
    };
    for (int sg = 0; sg < (kAdj ? 1 : a.n_seg); ++sg) {
        const LossSeg sgm = segs.seg[sg];
        const int64_t n_items = static_cast<int64_t>(a.Q) * sgm.groups;
        int64_t it = w_begin - sgm.w0 < 0 ? 0 : (w_begin - sgm.w0 < n_items ? w_begin - sgm.w0 : n_items);
        const int64_t it_end = w_end - sgm.w0 < 0 ? 0 : (w_end - sgm.w0 < n_items ? w_end - sgm.w0 : n_items);
        const int64_t t_lo = sgm.t_lo, t_hi = sgm.t_hi, count = t_hi - t_lo;
        while (it < it_end) {
            const int col = static_cast<int>(it / sgm.groups);
            const int part = col / a.S;
            const int64_t seg_end = min(it_end, static_cast<int64_t>(col + 1) * sgm.groups);
            const int64_t ga = sgm.g_lo + it - static_cast<int64_t>(col) * sgm.groups;
            const int64_t gb = sgm.g_lo + seg_end - static_cast<int64_t>(col) * sgm.groups;
            it = seg_end;
            if (part != held || sgm.layer != held_layer) {
                if constexpr (kAdj) {
                    if (held >= 0) flush_counts();
                }
                __syncthreads();                    // the part before is done
                held = part;
                held_layer = sgm.layer;
                if constexpr (kAdj) {
                    for (int i = threadIdx.x; i < kSlots / 4; i += blockDim.x)
                        reinterpret_cast<u32x4*>(cnt)[i] = u32x4{0, 0, 0, 0};
                } else {
                    const int n2 = static_cast<int>((a.part_n[part] + 1) / 2);
                    const u64x2* src = reinterpret_cast<const u64x2*>(a.tab + (sgm.layer * a.P + part) * kSlots);
                    u64x2 v[kSlots / 2048];
#pragma unroll
                    for (int k = 0; k < kSlots / 2048; ++k)
                        if (k * 1024 + static_cast<int>(threadIdx.x) < n2) v[k] = src[k * 1024 + threadIdx.x];
#pragma unroll
                    for (int k = 0; k < kSlots / 2048; ++k)
                        if (k * 1024 + static_cast<int>(threadIdx.x) < n2)
                            reinterpret_cast<u64x2*>(vals)[k * 1024 + threadIdx.x] = v[k];
                    __syncthreads();
                    if (threadIdx.x == 0) vals[kPadSlot] = 0.0;
                }
                __syncthreads();
            }
            // this wave's groups [g, g_end) of the column, rows [r, r_end)
            const int64_t n = gb - ga;
            int64_t g = ga + wv * n / 16;
            const int64_t g_end = ga + (wv + 1) * n / 16;
            if (g >= g_end) continue;
            const uint32_t* gs = gstart + static_cast<int64_t>(col) * (a.NG + 1);
            const uint64_t* rows = a.rows + a.col_base[col] / kRowIds + lane;
            double* out_hi = a.part_hi + sgm.part_at + static_cast<int64_t>(col) * count;
            float* out_lo = a.part_lo + sgm.part_at + static_cast<int64_t>(col) * count;
            unsigned long long* tvar = reinterpret_cast<unsigned long long*>(adj.w_tvar) + static_cast<int64_t>(part) * kSlots;
            const uint32_t r_last = max(gs[g_end], 1u) - 1u;
            auto row = [&](uint32_t at) -> uint64_t {
                return __builtin_nontemporal_load(rows + static_cast<int64_t>(at < r_last ? at : r_last) * 64);
            };
            double acc_hi = 0.0, acc_lo = 0.0;
            auto add_row = [&](uint64_t x, uint32_t cls) {
                uint32_t e[kRowIds];
#pragma unroll
                for (int i = 0; i < kRowIds; ++i) e[i] = static_cast<uint32_t>(x >> (16 * i)) & (kPair ? kSlotBits : 0xFFFF);
                if constexpr (kAdj) {
                    if (!(cls & 1u)) return;        // outside the aggregate band: no weight
#pragma unroll
                    for (int i = 0; i < kRowIds; ++i)
                        if (e[i] != kPadSlot) atomicAdd(&cnt[e[i]], 1u);
                    if (cls & 6u) {                 // a tail trial: its TVaR weight on each of its events
                        const unsigned long long wt =
                            static_cast<unsigned long long>((cls & 2u) ? ts.c_eq : ts.m - ts.c_gt);
#pragma unroll
                        for (int i = 0; i < kRowIds; ++i)
                            if (e[i] != kPadSlot)
                                atomicAdd(tvar + e[i], wt);
                    }
                } else {
                    double v[kRowIds];
#pragma unroll
                    for (int i = 0; i < kRowIds; ++i) v[i] = vals[e[i]];
#pragma unroll
                    for (int i = 0; i < kRowIds; ++i) dd_add(acc_hi, acc_lo, v[i]);
                }
            };
            // the backward's trial classes, a mask per class and 64 trials: scalar loads too,
            // so that no load but the rows' is waited for
            struct Masks {
                uint64_t band, above, at;
            } masks[2]{}, masks_next[2]{};
            auto masks_of = [&](int64_t grp, Masks(&to)[2]) {
                for (int h = 0; h < (kPair ? 2 : 1); ++h) {
                    const int64_t k = grp * (kTrials / 64) + h - adj.masks_lo;
                    const bool in = k >= 0 && k < adj.masks_n;
                    const uint64_t* m = cls_masks + (in ? k : 0) * 4;
                    to[h] = Masks{in ? m[0] : 0, in ? m[1] : 0, in ? m[2] : 0};
                }
            };
            auto class_of = [&](const Masks& m, int pos) -> uint32_t {
                return static_cast<uint32_t>(m.band >> pos & 1u) | static_cast<uint32_t>(m.above >> pos & 1u) << 1 |
                       static_cast<uint32_t>(m.at >> pos & 1u) << 2;
            };
            if constexpr (kAdj) {
                masks_of(g, masks);
                masks_of(g + 1, masks_next);
            }
            // where a lane's trials are in the group, and their classes
            int pos_a = lane, pos_b = 0;
            uint32_t cls = 0, cls_b = 0;
            auto start_group = [&](uint64_t y0, uint64_t y1, uint64_t y2, uint64_t y3) {
                if constexpr (kPair) {
                    auto m = [](uint64_t y) {
                        return static_cast<int>((y >> 31 & 1) | (y >> 46 & 2) | (y >> 61 & 4));
                    };
                    pos_a = m(y0) | m(y1) << 3;
                    pos_b = m(y2) | m(y3) << 3;
                }
                if constexpr (kAdj) {
                    cls = class_of(masks[0], pos_a);
                    if constexpr (kPair) cls_b = class_of(masks[1], pos_b);
                }
            };
            // where the group ends and the next one does (scalar loads, one group ahead)
            uint32_t r = gs[g], end = gs[g + 1], next = gs[min(g + 2, g_end)];
            uint64_t x[kAhead];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) x[k] = row(r + k);
            start_group(x[0], x[1], x[2], x[3]);
            double first_hi = 0.0, first_lo = 0.0;  // a pair's first trial
            auto store = [&](int64_t t, double sum_hi, double sum_lo) {
                const double hi = sum_hi + sum_lo;                      // renormalised: |lo| <= ulp(hi) / 2
                if (t >= t_lo && t < t_hi) {
                    out_hi[t - t_lo] = hi;
                    out_lo[t - t_lo] = static_cast<float>(sum_lo - (hi - sum_hi));
                }
            };
            // whole rounds of kAhead rows, the last one's past the last group left out
            for (uint32_t left = gs[g_end] - r + kAhead - 1; left >= kAhead; left -= kAhead) {
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const uint64_t y = x[k];
                    x[k] = row(r + kAhead);
                    if (r > r_last) continue;           // past the wave's groups
                    add_row(y, cls);
                    if constexpr (kPair) {
                        const bool ends = y & 0x8000u;                  // the lane's first trial
                        if constexpr (kAdj) {
                            cls = ends ? cls_b : cls;
                        } else {
                            first_hi = ends ? acc_hi : first_hi;
                            first_lo = ends ? acc_lo : first_lo;
                            acc_hi = ends ? 0.0 : acc_hi;
                            acc_lo = ends ? 0.0 : acc_lo;
                        }
                    }
                    ++r;
                    if (r != end) continue;
                    if constexpr (!kAdj) {
                        if constexpr (kPair) {
                            store(g * kTrials + pos_a, first_hi, first_lo);
                            store(g * kTrials + 64 + pos_b, acc_hi, acc_lo);
                        } else {
                            store(g * kTrials + lane, acc_hi, acc_lo);
                        }
                        acc_hi = 0.0;
                        acc_lo = 0.0;
                    }
                    ++g;
                    end = g < g_end ? next : ~0u;
                    next = gs[min(g + 2, g_end)];
                    if constexpr (kAdj) {
                        for (int h = 0; h < 2; ++h) masks[h] = g < g_end ? masks_next[h] : Masks{0, 0, 0};
                        masks_of(g + 1, masks_next);
                    }
                    start_group(x[(k + 1) % kAhead], x[(k + 2) % kAhead], x[(k + 3) % kAhead], x[(k + 4) % kAhead]);
                }
            }
        }
    }
    if constexpr (kAdj) {
        if (held >= 0) flush_counts();
    }
}

// The workgroups' counts of a part summed to its events.  A workgroup's share of the
// items is contiguous, so it holds few parts, and (workgroup + part) tells all of
// them apart; 256 workgroups' counts added by device atomics took about 100 us for
// 300000 events, stored and summed here 10 (12 with eight counts in flight; 37 workgroups' counts
// of three parts 11.6 -> 4.2).
__global__ __launch_bounds__(256) void loss_counts_kernel(LossPassArgs a, int64_t groups, int64_t n_wg,
                                                          const uint32_t* __restrict__ events,
                                                          const uint32_t* __restrict__ counts,
                                                          const uint64_t* __restrict__ tvar,
                                                          uint64_t* __restrict__ w_mean,
                                                          uint64_t* __restrict__ w_tvar) {
    const int part = static_cast<int>(blockIdx.y);
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.part_n[part]) return;
    // workgroup l's items are [l work / n_wg, (l + 1) work / n_wg), not empty
    const int64_t first = static_cast<int64_t>(part) * a.S * groups, last = first + static_cast<int64_t>(a.S) * groups - 1;
    const int64_t l0 = a.whole ? first_wg(part, n_wg, a.P) : ((first + 1) * n_wg - 1) / a.work;
    const int64_t l1 = a.whole ? first_wg(part + 1, n_wg, a.P) - 1 : ((last + 1) * n_wg - 1) / a.work;
    const uint32_t E = events[static_cast<int64_t>(part) * kSlots + i];
    const uint64_t tv = tvar[static_cast<int64_t>(part) * kSlots + i];
    uint64_t sum = 0;
    const uint32_t* c = counts + (l0 + part) * kSlots + i;
    const int more = static_cast<int>(l1 - l0);
    for (int k0 = 0; k0 <= more; k0 += 16) {        // 16 workgroups' counts in flight
        uint32_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = c[static_cast<int64_t>(min(k0 + k, more)) * kSlots];
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += k0 + k <= more ? v[k] : 0u;
    }
    w_mean[E] = sum;
    w_tvar[E] = tv;
}

// one 1024-thread workgroup per CU (its LDS holds the part's table or counters)
int64_t pass_grid(int n_cu) {
    const int64_t grid = int64_t(n_cu) - n_cu % kXcds;
    return grid < kXcds ? kXcds : grid;
}

template <bool kAdj>
hipError_t launch_pass(const StreamLayout& lay, const LossIndex& ix, const StreamUnit* units, int n, const double* tab,
                       void* partials, const LossAdjArgs& adj, const uint64_t* masks, uint64_t* w_mean,
                       uint64_t* w_tvar, int n_cu, hipStream_t s) {
    if (n < 1 || n > kMaxSegs || lay.P <= 0 || ix.P <= 0 || lay.P % ix.P || (lay.G != 64 && lay.G != 128))
        return hipErrorInvalidValue;
    LossPassArgs a{};
    a.rows = reinterpret_cast<const uint64_t*>(lay.ids);
    a.col_base = lay.part_base;
    a.tab = tab;
    a.part_n = ix.part_n;
    a.Q = lay.P;
    a.P = ix.P;
    a.S = lay.P / ix.P;
    a.NG = lay.NG;
    a.n_seg = n;
    int64_t trials = 0;
    for (int i = 0; i < n; ++i) trials += units[i].count;
    a.part_hi = static_cast<double*>(partials);
    a.part_lo = reinterpret_cast<float*>(a.part_hi + static_cast<int64_t>(lay.P) * trials);
    LossSegs segs{};
    int64_t at = 0;
    for (int i = 0; i < n; ++i) {
        LossSeg& g = segs.seg[i];
        g.t_lo = units[i].t_lo;
        g.t_hi = units[i].t_lo + units[i].count;
        g.g_lo = g.t_lo / lay.G;
        g.groups = (g.t_hi + lay.G - 1) / lay.G - g.g_lo;
        g.w0 = a.work;
        g.part_at = at;
        g.layer = units[i].layer;
        a.work += static_cast<int64_t>(lay.P) * g.groups;
        at += static_cast<int64_t>(lay.P) * units[i].count;
    }
    int64_t grid = pass_grid(n_cu);
    if (kAdj) {                                     // a group per wave: fewer counters to store and sum
        grid = std::min(grid, std::max<int64_t>(a.work / 16, 1));
        if (grid > kXcds) grid -= grid % kXcds;
    }
    // where there are three groups per wave and the shares stay within 6 % of even
    const int64_t each = grid / a.P;
    a.whole = n == 1 && a.P > 1 && a.work >= 48 * grid && grid <= 1.06 * static_cast<double>(each * a.P);
    hipLaunchKernelGGL((lay.G == 128 ? loss_pass_kernel<kAdj, true> : loss_pass_kernel<kAdj, false>),
                       dim3(static_cast<uint32_t>(grid)), dim3(1024), 0, s, a, segs, adj, lay.gstart, masks);
    hipError_t e = hipGetLastError();
    if (!kAdj || e != hipSuccess) return e;
    hipLaunchKernelGGL(loss_counts_kernel, dim3(kSlots / 256, static_cast<uint32_t>(a.P)), dim3(256), 0, s, a,
                       segs.seg[0].groups, grid, ix.events, adj.counts, adj.w_tvar, w_mean, w_tvar);
    return hipGetLastError();
}

// columns per part: enough that the whole table's groups fill the waves four
// times, unless that leaves a trial fewer than 32 events, or costs more in the merge
// (0.25 us a column) than the shorter columns save (about 0.1 us a row of a group)
int splits_of(int P, int64_t N, int64_t kept, int n_cu) {
    const double lam = static_cast<double>(kept) / (static_cast<double>(N) * P);
    const double items = static_cast<double>(P) * ((N + 63) / 64);
    const double want = std::min({std::ceil(lam / 32.0), std::ceil(64.0 * n_cu / items), std::sqrt(0.1 * lam / P)});
    return static_cast<int>(std::max(1.0, std::min(want, 64.0)));
}

// Two trials per lane (calls in us, one and two): from 3 slots per trial and column on,
// below which a group's least rows are longer than it, while padding is much of a row
// (up to 64 slots), and where the copy has two groups of 128 for each of the chip's
// waves: 10^6 trials 249 / 215, 12 layers of a library 1030 / 872, 16 layers over 16778
// trials 160 / 183 (a wave's last group is a larger part of its share).
constexpr double kPairLeast = 3.0, kPairMost = 64.0;

// the copy from the intermediate one, unless that is not to be used or the copy takes
// more than `most` bytes
hipError_t build_rows(const StreamLayout& in, int64_t N, int64_t kept, int64_t most, int n_cu, LossRows* d_rows,
                      hipStream_t s, StreamLayout* out) {
    const int S = splits_of(in.P, N, kept, n_cu), Q = in.P * S;
    const double lam = static_cast<double>(kept) / (static_cast<double>(N) * Q);
    const bool pair = lam >= kPairLeast && lam <= kPairMost && Q * (N / 128) >= 32 * int64_t(n_cu);
    const int G = pair ? 128 : 64;
    const int64_t NG = (N + G - 1) / G;
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&out->gstart), sizeof(uint32_t) * Q * (NG + 1), s);
    if (e == hipSuccess) e = dev_alloc(reinterpret_cast<void**>(&out->part_base), sizeof(int64_t) * (Q + 1), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((pair ? loss_group_kernel<true> : loss_group_kernel<false>), dim3(static_cast<uint32_t>((NG + 3) / 4), static_cast<uint32_t>(in.P)),
                       dim3(256), 0, s, in, N, S, NG, out->gstart);
    hipLaunchKernelGGL(loss_scan_kernel, dim3(static_cast<uint32_t>(Q)), dim3(1024), 0, s, NG, out->gstart, d_rows->rows);
    hipLaunchKernelGGL(loss_bases_kernel, dim3(1), dim3(64), 0, s, Q, d_rows->rows, out->part_base);
    std::vector<char> host(offsetof(LossRows, rows) + sizeof(int64_t) * Q);
    LossRows* rows = reinterpret_cast<LossRows*>(host.data());
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(host.data(), d_rows, host.size(), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    bool used = !(rows->res.flags & (kCreateWideGroup | kCreateWidePart));
    for (int q = 0; used && q < Q; ++q) {
        if (rows->rows[q] >= (int64_t(1) << 32) - 4096) return hipErrorOutOfMemory;    // past 32-bit rows
        out->length += rows->rows[q] * 64 * kRowIds;
    }
    if (!used || static_cast<int64_t>(sizeof(uint16_t)) * out->length > most) {
        free_stream_layout(out, s);
        return hipSuccess;
    }
    e = dev_alloc(reinterpret_cast<void**>(&out->ids), sizeof(uint16_t) * (out->length + 64 * kRowIds), s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL((pair ? loss_rows_kernel<true> : loss_rows_kernel<false>), dim3(static_cast<uint32_t>((NG + 3) / 4), static_cast<uint32_t>(Q)),
                           dim3(256), 0, s, in, N, S, NG, out->gstart, out->part_base,
                           reinterpret_cast<uint64_t*>(out->ids));
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    out->P = Q;
    out->G = G;
    out->NG = NG;
    out->bytes = static_cast<int64_t>(sizeof(uint16_t)) * (out->length + 64 * kRowIds) +
                 static_cast<int64_t>(sizeof(uint32_t)) * Q * (NG + 1) + static_cast<int64_t>(sizeof(int64_t)) * (Q + 1);
    return hipSuccess;
}

}  // namespace

int64_t loss_table_bytes(const LossIndex& ix) { return static_cast<int64_t>(sizeof(double)) * kSlots * ix.P; }

hipError_t launch_loss_pass_units(const StreamLayout& lay, const LossIndex& ix, const StreamUnit* units, int n,
                                  const double* tab, void* partials, int n_cu, hipStream_t s) {
    return launch_pass<false>(lay, ix, units, n, tab, partials, LossAdjArgs{}, nullptr, nullptr, nullptr, n_cu, s);
}

int64_t loss_tvar_words(const LossIndex& ix) { return static_cast<int64_t>(kSlots) * ix.P; }

int64_t loss_adjoint_bytes(const LossIndex& ix, int n_cu) {
    return loss_tvar_words(ix) * static_cast<int64_t>(sizeof(uint64_t)) +
           static_cast<int64_t>(sizeof(uint32_t)) * kSlots * (pass_grid(n_cu) + ix.P);
}

hipError_t launch_loss_adjoint(const StreamLayout& lay, const LossIndex& ix, const LayerArgs& L, const uint64_t* masks,
                               const TailStats* tail, void* scratch, uint64_t* w_mean, uint64_t* w_tvar, int n_cu,
                               hipStream_t s) {
    if (L.trial_count <= 0) return hipSuccess;
    uint64_t* tvar = static_cast<uint64_t*>(scratch);
    const int64_t m_lo = L.trial_begin / 64, m_hi = (L.trial_begin + L.trial_count + 63) / 64;
    const LossAdjArgs adj{reinterpret_cast<uint32_t*>(tvar + loss_tvar_words(ix)), tvar, m_lo, m_hi - m_lo, tail};
    const StreamUnit u{0, L.trial_begin, L.trial_count, 0, 0.0};
    return launch_pass<true>(lay, ix, &u, 1, nullptr, nullptr, adj, masks, w_mean, w_tvar, n_cu, s);
}

void free_loss_index(LossIndex* ix, hipStream_t s) {
    dev_free(ix->probe, s);
    *ix = LossIndex{};
}

hipError_t build_losses(const SparsePool& sp, int n_rows, int64_t C, const int64_t* offsets, const uint32_t* ids,
                        int64_t N, int64_t n_events, int n_cu, hipStream_t s, LossIndex* ix, StreamLayout* out) {
    *ix = LossIndex{};
    *out = StreamLayout{};
    if (n_rows < 1 || sp.n_chunks < 1 || N < 1 || C > int64_t(kMaxStreamParts) << kStreamShift) return hipSuccess;
    const int64_t n_sb = sp.n_chunks, n_words = (C + 31) / 32;
    // two neighbouring parts hold more than kSlots - 1 events
    const int most_parts = static_cast<int>(std::min<int64_t>(kMaxStreamParts, 2 * (C / (kSlots - 1)) + 1));
    LossRows* d_rows = nullptr;                 // the temporaries' block: the results,
    int64_t* start = nullptr;                   // [N], then the plan,
    uint32_t* place = nullptr;                  // [n_sb]
    uint32_t* kept_ids = nullptr;
    int32_t* cnt = nullptr;
    StreamLayout by_part{};
    LossPlan plan{};
    int shift = 0;
    while (C > (int64_t(kMapWords) * 32 << shift)) ++shift;
    const bool long_trials = n_events / N > 256;
    auto filter = [&](auto fill, int P) {
        constexpr bool kFill = decltype(fill)::value;
        const auto kernel = shift == 0 ? (long_trials ? loss_filter_kernel<kFill, 16, true> : loss_filter_kernel<kFill, 4, true>)
                                       : (long_trials ? loss_filter_kernel<kFill, 16, false> : loss_filter_kernel<kFill, 4, false>);
        // a workgroup per CU, two where their maps fit beside each other (200000 trials of 2
        // events 44 -> 33 us and 54 -> 41)
        const size_t lds = sizeof(uint32_t) * filter_words(kFill, shift == 0, n_words);
        const int64_t grid = std::min((N + 15) / 16, int64_t(n_cu) * (lds <= 72 * 1024 ? 2 : 1));
        hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(grid)), dim3(1024), lds, s, offsets, ids, N, ix->probe,
                           n_words, shift, start, kept_ids, P, cnt);
    };

    // the events' slots, and how many events the trials keep
    ix->bytes = static_cast<int64_t>(sizeof(uint64_t)) * n_words +
                static_cast<int64_t>(sizeof(uint32_t)) * (static_cast<int64_t>(kSlots) * most_parts + kMaxStreamParts);
    hipError_t e = dev_alloc(reinterpret_cast<void**>(&ix->probe), static_cast<size_t>(ix->bytes), s);
    if (e == hipSuccess)
        e = dev_alloc(reinterpret_cast<void**>(&d_rows),
                      sizeof(LossRows) + sizeof(int64_t) * N + sizeof(LossPlan) + sizeof(uint32_t) * n_sb, s);
    if (e == hipSuccess) {
        static_assert(offsetof(LossPlan, kept) == 0, "the scan's total after the starts");
        ix->events = reinterpret_cast<uint32_t*>(ix->probe + n_words);
        ix->part_n = ix->events + static_cast<int64_t>(kSlots) * most_parts;
        start = reinterpret_cast<int64_t*>(d_rows + 1);
        LossPlan* d_plan = reinterpret_cast<LossPlan*>(start + N);
        place = reinterpret_cast<uint32_t*>(d_plan + 1);
        hipLaunchKernelGGL(loss_bits_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(1024), 0, s, sp, n_rows, C,
                           ix->probe, place);
        hipLaunchKernelGGL(loss_plan_kernel, dim3(1), dim3(64), 0, s, n_sb, most_parts, place, ix->part_n, d_plan,
                           &d_rows->res);
        hipLaunchKernelGGL(loss_place_kernel, dim3(static_cast<uint32_t>(n_sb)), dim3(64), 0, s, C, most_parts, place,
                           ix->probe, ix->events);
        filter(std::false_type{}, 0);
        e = hipGetLastError();
        if (e == hipSuccess) e = launch_scan_i64(start, N, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&plan, d_plan, sizeof(plan), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }

    // Not used without a kept event, past the parts a copy can have, where trials are so
    // short that most of the copy would be padding (a row takes 8 bytes of each trial),
    // or where the copy and its temporaries take more than a quarter of the free memory.
    const int P = plan.parts;
    const int64_t kept = plan.kept, most = 4 * n_events + (int64_t(128) << 20);
    size_t mem_free = 0, mem_all = 0;
    if (e == hipSuccess && kept > 0 && P <= most_parts && 16 * N * P <= most &&
        hipMemGetInfo(&mem_free, &mem_all) == hipSuccess &&
        12 * kept + 16 * N * P + most <= static_cast<int64_t>(mem_free / 4)) {
        e = dev_alloc(reinterpret_cast<void**>(&kept_ids), sizeof(uint32_t) * (kept + kIdPad), s);
        if (e == hipSuccess) e = dev_alloc(reinterpret_cast<void**>(&cnt), sizeof(int32_t) * N * P, s);
        if (e == hipSuccess) {
            filter(std::true_type{}, P);
            e = hipGetLastError();
        }
        // a part's slots as 2^16 catalogue events
        if (e == hipSuccess)
            e = plan_stream_layout(cnt, N, kept, static_cast<int64_t>(P) << kStreamShift, &d_rows->res, s, &by_part);
        if (e == hipSuccess) e = fill_stream_layout_unread(start, kept_ids, N, kept, &d_rows->res, s, &by_part);
        if (e == hipSuccess && by_part.P > 0) e = build_rows(by_part, N, kept, most, n_cu, d_rows, s, out);
    }
    dev_drop(by_part.ids, s);
    by_part.ids = nullptr;
    free_stream_layout(&by_part, s);
    dev_drop(kept_ids, s);
    dev_free(cnt, s);
    dev_free(d_rows, s);
    ix->P = P;
    ix->n_events = plan.events;
    if (e != hipSuccess || out->P == 0) {
        free_stream_layout(out, s);
        free_loss_index(ix, s);
    }
    return e;
}

}  // namespace ara
