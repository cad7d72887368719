// The stable split of trials' events by catalogue part, shared by the builds of
// the YET's 16-bit and 32-bit copies: a workgroup stages a few trials' events in
// LDS, part after part, and each part's run leaves in whole lines.
#pragma once

#include "ara_internal.hpp"

namespace ara {

constexpr int kScatterThreads = 512;                // four workgroups per CU: LDS below 40 KB each
constexpr int kScatterWaves = kScatterThreads / 64;

// n events of a trial from ids[b] on, one wave: event E goes to
// stage[cur[E >> shift]++], in order.  Per 64 events the lanes that hold an event
// of this lane's part are the AND, over kBits bits of the part number, of that
// bit's ballot or its complement (3 instructions per bit and half); a lane's rank
// among the earlier of them places it, and all of them store the same moved
// cursor.  `first` holds the trial's first 512 events and `load_next` starts the
// load of what follows it (reads up to 512 IDs past the trial, which the table's
// padding allows).  Vector instructions are the bound (about 32 per 64 events over
// 32 parts; testing which lane is a part's last, 64-bit positions and a validity
// test per lane took 67).
constexpr int kScatterAhead = 8;                    // chunks of 64 IDs in flight
template <int kBits, typename T, typename LoadNext>
__device__ __forceinline__ void scatter_trial(const uint32_t* __restrict__ ids, int64_t b, int64_t n, int shift,
                                              uint32_t* cur, T* stage, uint32_t (&nxt)[kScatterAhead],
                                              LoadNext load_next) {
    const int lane = threadIdx.x & 63;
    auto chunk = [&](uint32_t id, bool full, bool valid) {
        const uint32_t pid = id >> shift;
        uint32_t lo, hi;
        if (full) {
            lo = hi = ~0u;
        } else {
            const uint64_t v = __builtin_amdgcn_ballot_w64(valid);
            lo = static_cast<uint32_t>(v);
            hi = static_cast<uint32_t>(v >> 32);
        }
#pragma unroll
        for (int bit = 0; bit < kBits; ++bit) {
            const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(pid << (31 - bit)) >> 31);
            const uint64_t lanes = __builtin_amdgcn_ballot_w64(m != 0);
            lo &= ~(static_cast<uint32_t>(lanes) ^ m);
            hi &= ~(static_cast<uint32_t>(lanes >> 32) ^ m);
        }
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        if (full || valid) {
            const uint32_t at = cur[pid];
            stage[at + rank] = static_cast<T>(id);
            cur[pid] = at + __popc(lo) + __popc(hi);
        }
        __builtin_amdgcn_wave_barrier();
    };
    for (int64_t c0 = 0; c0 < n; c0 += 64 * kScatterAhead) {
        uint32_t idk[kScatterAhead];
#pragma unroll
        for (int k = 0; k < kScatterAhead; ++k) idk[k] = nxt[k];
        if (c0 + 64 * kScatterAhead < n) {
#pragma unroll
            for (int k = 0; k < kScatterAhead; ++k) nxt[k] = ids[b + c0 + 64 * kScatterAhead + k * 64 + lane];
        } else {
            load_next();
        }
        const int left = static_cast<int>(n - c0 < 64 * kScatterAhead ? n - c0 : 64 * kScatterAhead);
#pragma unroll
        for (int k = 0; k < kScatterAhead; ++k) {
            if (k * 64 + 64 <= left) chunk(idk[k], true, true);
            else if (k * 64 < left) chunk(idk[k], false, k * 64 + lane < left);
        }
    }
    if (n <= 0) load_next();
}

// Trials [first, first + n) of a unit, dealt to the waves, each one's next trial
// loaded ahead; begin(i) sets the wave's cursors for trial i, end(i) follows it.
template <int kBits, typename T, typename Begin, typename End>
__device__ __forceinline__ void scatter_unit(const int64_t* __restrict__ offsets, const uint32_t* __restrict__ ids,
                                             int64_t first, int n, int shift, uint32_t* cur, T* stage, Begin begin,
                                             End end) {
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    uint32_t nxt[kScatterAhead] = {};
    int64_t b = 0, e = 0, bn = 0, en = 0;
    auto load = [&](int64_t at) {
#pragma unroll
        for (int k = 0; k < kScatterAhead; ++k) nxt[k] = ids[at + k * 64 + lane];
    };
    if (w < n) {
        b = offsets[first + w];
        e = offsets[first + w + 1];
        load(b);
    }
    for (int i = w; i < n; i += kScatterWaves) {
        const bool more = i + kScatterWaves < n;
        if (more) {
            bn = offsets[first + i + kScatterWaves];
            en = offsets[first + i + kScatterWaves + 1];
        }
        begin(i);
        __builtin_amdgcn_wave_barrier();
        scatter_trial<kBits>(ids, b, e - b, shift, cur, stage, nxt, [&] {
            if (more) load(bn);
        });
        end(i);
        __builtin_amdgcn_wave_barrier();
        b = bn;
        e = en;
    }
}

// the same, straight to memory: 64-bit cursors, for units past the stage
template <typename T>
__device__ __forceinline__ void scatter_trial_direct(const uint32_t* __restrict__ ids, int64_t b, int64_t e, int shift,
                                                     int n_bits, int64_t* cur, T* out) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int64_t c = b; c < e; c += 64) {
        const bool valid = c + lane < e;
        const uint32_t id = ids[c + lane];
        const uint32_t pid = id >> shift;
        uint64_t same = __ballot(valid);
        for (int bit = 0; bit < n_bits; ++bit) {
            const bool set = ((pid >> bit) & 1u) != 0;
            const uint64_t lanes = __ballot(set);
            same &= set ? lanes : ~lanes;
        }
        if (valid) {
            const int64_t at = cur[pid];
            out[at + __popcll(same & below)] = static_cast<T>(id);
            cur[pid] = at + __popcll(same);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// consecutive units of a launch to one XCD, whose L2 then merges the lines they share
__device__ __forceinline__ int64_t scatter_unit_index(int64_t n_units) {
    const int64_t per = (n_units + kXcds - 1) / kXcds;
    return static_cast<int64_t>(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

// f(first, count) over `n` workgroups in launches of at most 2^22: a launch may have
// no 2^32 threads, which a workgroup per few trials reaches at 5e8 trials
template <typename F>
inline hipError_t in_launches(int64_t n, F f) {
    constexpr int64_t kMost = int64_t(1) << 22;
    hipError_t e = hipSuccess;
    for (int64_t at = 0; at < n && e == hipSuccess; at += kMost) {
        f(at, n - at < kMost ? n - at : kMost);
        e = hipGetLastError();
    }
    return e;
}

// most trials of mean `lam` events that fit a stage of `cap` (six standard
// deviations of Poisson trials; `slack` more for the parts' ends), at most `most`
inline int scatter_trials(double lam, double slack, int cap, int most) {
    int n = 1;
    for (int k = 2; k <= most; ++k) {
        const double mean = k * lam;
        if (mean + 6.0 * __builtin_sqrt(mean) + slack <= cap) n = k;
        else break;
    }
    return n;
}

}  // namespace ara
