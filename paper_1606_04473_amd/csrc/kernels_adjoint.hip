// Adjoint of the year loss with respect to a layer's terms.
//
// With the strict convention at kinks every partial of YLT_t is an integer:
//   d YLT_t / d theta_k = a_t * sum over the trial's occurrences of g_k(E)
// for the per-ELT and occurrence terms, where a_t = [0 < S_t - AggR < AggL]
// and g_k(E) in {-1, 0, 1} depends on the event only; dYLT_t/dAggR = -a_t and
// dYLT_t/dAggL = [S_t - AggR > AggL].  Summing over trials with weights w_t
// (1 for the mean; for TVaR c_eq above the m-th largest value v and m - c_gt
// at v) regroups by event:
//   sum_t w_t a_t sum_d g_k(E_td) = sum_E g_k(E) * W(E),
//   W(E) = sum over active trials of w_t * (multiplicity of E in trial t).
// So the backward is one pass over the events of active trials that builds
// the integer histogram W (only for events whose occurrence loss can move:
// y(E) - OccR > 0), then one pass over the catalogue that evaluates g(E)
// with the forward's FP64 operations and accumulates g_k(E) W(E) in int64.
// Integer atomics make the result independent of scheduling.
#include "ara_internal.hpp"

namespace ara {

namespace {

constexpr int kMaxP = 2 * kMaxJ + 4;
// copies of the numerators, one per XCD for the workgroups that finish at once
constexpr int kAccCopies = 8;

// signed 64-bit add through the unsigned atomic (two's complement wraps)
__device__ __forceinline__ void add_i64(long long* p, long long v) {
    atomicAdd(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(v));
}

struct AdjScratch {
    uint8_t* mark;         // [C]
    uint64_t* w_mean;      // [C]
    uint64_t* w_tvar;      // [C]
    long long* acc;        // [kAccCopies][2][kMaxP] integer numerators, summed at the end
    TailStats* tail;
    void* cls;             // trial classes of the stream histogram
    int64_t cls_bytes;
    void* tail_scratch;
};

// The same numerators from the sparse ELT pool, after a fold that left each
// event's place against the occurrence terms: one workgroup per chunk of
// kSparseChunk events.  Each event with a weight adds its occurrence-term slopes;
// the weights of those inside the band go to LDS, where each nonzero loss (E, l)
// of ELT j finds them for its per-ELT slopes (an absent loss has l - R_j <= 0 and
// no slope, so the sparse entries give the dense kernel's integer sums).  A wave
// takes whole ELTs, so it sums in registers; its first entries load before the
// weights are in place.  Refolding the chunk's losses here, with their entries
// staged in LDS, one workgroup per CU, took 38 us where this takes 16 (16 ELTs over
// 2e6 events); it takes 90 with the device atomics ELT by ELT and 22 with one copy
// of the sums for all workgroups.
constexpr int kSparseChunk = 4096;                  // events per chunk of the sparse pool
constexpr int kSparseThreads = 512;

// sum over the wave's lanes
__device__ __forceinline__ long long wave_sum_i64(long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__global__ __launch_bounds__(kSparseThreads) void catalogue_sparse_kernel(SparsePool sp, int64_t C, LayerArgs L,
                                                                          const uint8_t* __restrict__ band,
                                                                          const uint64_t* __restrict__ w_mean,
                                                                          const uint64_t* __restrict__ w_tvar,
                                                                          long long* __restrict__ acc) {
    constexpr int kPer = kSparseChunk / kSparseThreads, kWaves = kSparseThreads / 64;
    __shared__ long long wms[kSparseChunk], wvs[kSparseChunk];
    __shared__ long long red[kWaves][4];
    __shared__ long long lacc[2 * kMaxP];           // the workgroup's sums: one pass of device atomics at the end
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t chunk = blockIdx.x;
    const int64_t e0 = chunk * kSparseChunk;
    const int J = L.J;
    for (int i = t; i < 2 * kMaxP; i += kSparseThreads) lacc[i] = 0;
    // lane j: ELT j's entries of the chunk
    int64_t at = 0;
    int cnt = 0;
    if (lane < J) {
        const int64_t key = static_cast<int64_t>(L.idx[lane]) * sp.n_chunks + chunk;
        at = sp.chunk_off[key];
        cnt = static_cast<int>(sp.chunk_off[key + 1] - at);
    }
    uint8_t b[kPer];
    long long wm[kPer], wv[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t e = e0 + k * kSparseThreads + t;
        b[k] = e < C ? band[e] : 0;
        wm[k] = e < C ? static_cast<long long>(w_mean[e]) : 0;
        wv[k] = e < C ? static_cast<long long>(w_tvar[e]) : 0;
    }
    // the next 64 entries of ELT j from f on
    int ev = 0;
    double v = 0.0;
    auto fetch = [&](int j, int f) {
        const int64_t from = __shfl(at, j, 64);
        const int n = __builtin_amdgcn_readlane(cnt, j);
        ev = -1;
        if (f + lane < n) {
            ev = sp.ev[from + f + lane];
            v = sp.val[from + f + lane];
        }
    };
    if (w < J) fetch(w, 0);
    long long sums[4] = {0, 0, 0, 0};               // above, inside; each of the mean and of the TVaR
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (b[k] == 2) {
            sums[0] += wm[k];
            sums[1] += wv[k];
        } else if (b[k] == 1) {
            sums[2] += wm[k];
            sums[3] += wv[k];
        }
        wms[k * kSparseThreads + t] = b[k] == 1 ? wm[k] : 0;
        wvs[k * kSparseThreads + t] = b[k] == 1 ? wv[k] : 0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        sums[q] = wave_sum_i64(sums[q]);
        if (lane == 0) red[w][q] = sums[q];
    }
    __syncthreads();
    if (t < 4) {
        long long s = 0;
        for (int k = 0; k < kWaves; ++k) s += red[k][t];
        lacc[(t & 1) * kMaxP + 2 * J + (t < 2 ? 1 : 0)] = t < 2 ? s : -s;
    }
    for (int j = w; j < J; j += kWaves) {
        const double R = L.R[j], Lim = L.Lim[j];
        const int n = __builtin_amdgcn_readlane(cnt, j);
        long long in_m = 0, in_v = 0, over_m = 0, over_v = 0;
        for (int f = 0; f < n; f += 64) {
            const int e = ev;
            const double tj = v - R;
            if (f + 64 < n) fetch(j, f + 64);
            else if (j + kWaves < J) fetch(j + kWaves, 0);
            if (e < 0) continue;
            if (tj > 0.0 && tj < Lim) {
                in_m += wms[e];
                in_v += wvs[e];
            }
            if (tj > Lim) {
                over_m += wms[e];
                over_v += wvs[e];
            }
        }
        if (n == 0 && j + kWaves < J) fetch(j + kWaves, 0);
        in_m = wave_sum_i64(in_m);
        over_m = wave_sum_i64(over_m);
        in_v = wave_sum_i64(in_v);
        over_v = wave_sum_i64(over_v);
        if (lane == 0) {
            lacc[j] = -in_m;
            lacc[kMaxP + j] = -in_v;
            lacc[J + j] = over_m;
            lacc[kMaxP + J + j] = over_v;
        }
    }
    __syncthreads();
    for (int i = t; i < 2 * kMaxP; i += kSparseThreads)
        if (lacc[i] != 0) add_i64(&acc[blockIdx.x % kAccCopies * (2 * kMaxP) + i], lacc[i]);
}

__global__ __launch_bounds__(256) void mark_kernel(const double* __restrict__ elts, int64_t C, LayerArgs L,
                                                   uint8_t* __restrict__ mark, uint64_t* __restrict__ w_mean,
                                                   uint64_t* __restrict__ w_tvar, int with_mark) {
    const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= C) return;
    w_mean[e] = 0;
    w_tvar[e] = 0;
    if (!with_mark) return;
    double y = 0.0;
    for (int j = 0; j < L.J; ++j)
        y = y + apply_terms(elts[static_cast<int64_t>(L.idx[j]) * C + e], L.R[j], L.Lim[j]);
    mark[e] = (y - L.occR > 0.0) ? 1 : 0;
}

__global__ void clear_acc_kernel(long long* acc) {
    for (int i = threadIdx.x; i < kAccCopies * 2 * kMaxP; i += blockDim.x) acc[i] = 0;
}

// one wavefront per trial; only trials inside the aggregate band read events
__global__ __launch_bounds__(256) void active_trials_kernel(const int64_t* __restrict__ offsets,
                                                            const uint32_t* __restrict__ ids, LayerArgs L,
                                                            const double* __restrict__ S,
                                                            const double* __restrict__ ylt,
                                                            const TailStats* __restrict__ tail,
                                                            const uint8_t* __restrict__ mark,
                                                            uint64_t* __restrict__ w_mean,
                                                            uint64_t* __restrict__ w_tvar,
                                                            long long* __restrict__ acc) {
    const int lane = threadIdx.x & 63;
    const int64_t wave = uniform_i64((static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6);
    const int64_t n_waves = (static_cast<int64_t>(gridDim.x) * blockDim.x) >> 6;
    const TailStats ts = *tail;
    const int P = 2 * L.J + 4;
    long long agg_r_mean = 0, agg_l_mean = 0, agg_r_tvar = 0, agg_l_tvar = 0;
    for (int64_t k = wave; k < L.trial_count; k += n_waves) {
        const double ta = S[k] - L.aggR;
        const bool in_band = (ta > 0.0) && (ta < L.aggL);
        const bool above = ta > L.aggL;
        const uint64_t key = __double_as_longlong(ylt[k] + 0.0);
        const long long wt = key > ts.v_bits ? ts.c_eq : (key == ts.v_bits ? ts.m - ts.c_gt : 0);
        if (in_band) {
            agg_r_mean -= 1;
            agg_r_tvar -= wt;
        }
        if (above) {
            agg_l_mean += 1;
            agg_l_tvar += wt;
        }
        if (!in_band) continue;
        const int64_t t = L.trial_begin + k;
        const int64_t b = offsets[t];
        const int64_t e = offsets[t + 1];
        for (int64_t i = b + lane; i < e; i += kWave) {
            const uint32_t id = ids[i];
            if (mark[id]) {
                atomicAdd(reinterpret_cast<unsigned long long*>(&w_mean[id]), 1ull);
                if (wt) atomicAdd(reinterpret_cast<unsigned long long*>(&w_tvar[id]),
                                  static_cast<unsigned long long>(wt));
            }
        }
    }
    if (lane == 0) {
        if (agg_r_mean) add_i64(&acc[P - 2], agg_r_mean);
        if (agg_l_mean) add_i64(&acc[P - 1], agg_l_mean);
        if (agg_r_tvar) add_i64(&acc[kMaxP + P - 2], agg_r_tvar);
        if (agg_l_tvar) add_i64(&acc[kMaxP + P - 1], agg_l_tvar);
    }
}

// aggregate-term partials alone (the partitioned histogram pass leaves them out)
__global__ __launch_bounds__(256) void agg_counts_kernel(LayerArgs L, const double* __restrict__ S,
                                                         const double* __restrict__ ylt,
                                                         const TailStats* __restrict__ tail,
                                                         long long* __restrict__ acc) {
    const TailStats ts = *tail;
    const int P = 2 * L.J + 4;
    long long r_mean = 0, l_mean = 0, r_tvar = 0, l_tvar = 0;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t n = L.trial_count;
    // four trials per thread per round, their loads in flight together
    constexpr int kU = 4;
    for (int64_t k0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; k0 < n; k0 += kU * stride) {
        double sv[kU], yv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t k = k0 + u * stride;
            sv[u] = k < n ? S[k] : L.aggR;          // a trial past the end: ta = 0, no count
            yv[u] = k < n ? ylt[k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const double ta = sv[u] - L.aggR;
            const uint64_t key = __double_as_longlong(yv[u] + 0.0);
            const long long wt = key > ts.v_bits ? ts.c_eq : (key == ts.v_bits ? ts.m - ts.c_gt : 0);
            if ((ta > 0.0) && (ta < L.aggL)) {
                r_mean -= 1;
                r_tvar -= wt;
            }
            if (ta > L.aggL) {
                l_mean += 1;
                l_tvar += wt;
            }
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        r_mean += __shfl_xor(r_mean, off, kWave);
        l_mean += __shfl_xor(l_mean, off, kWave);
        r_tvar += __shfl_xor(r_tvar, off, kWave);
        l_tvar += __shfl_xor(l_tvar, off, kWave);
    }
    // one set of device atomics per workgroup: every workgroup adds to the
    // same four counters, so per-wave atomics would queue on them
    __shared__ long long red[4][4];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[w][0] = r_mean;
        red[w][1] = l_mean;
        red[w][2] = r_tvar;
        red[w][3] = l_tvar;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        long long v[4] = {0, 0, 0, 0};
        for (int i = 0; i < static_cast<int>(blockDim.x >> 6); ++i)
            for (int q = 0; q < 4; ++q) v[q] += red[i][q];
        if (v[0]) add_i64(&acc[P - 2], v[0]);
        if (v[1]) add_i64(&acc[P - 1], v[1]);
        if (v[2]) add_i64(&acc[kMaxP + P - 2], v[2]);
        if (v[3]) add_i64(&acc[kMaxP + P - 1], v[3]);
    }
}

// g(E) W(E) over the catalogue; per-workgroup int64 accumulators in LDS
__global__ __launch_bounds__(256) void catalogue_kernel(const double* __restrict__ elts, int64_t C, LayerArgs L,
                                                        const uint64_t* __restrict__ w_mean,
                                                        const uint64_t* __restrict__ w_tvar,
                                                        long long* __restrict__ acc) {
    __shared__ long long lacc[2 * kMaxP];
    const int P = 2 * L.J + 4;
    for (int i = threadIdx.x; i < 2 * kMaxP; i += blockDim.x) lacc[i] = 0;
    __syncthreads();
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < C; e += stride) {
        const long long wm = static_cast<long long>(w_mean[e]);
        const long long wv = static_cast<long long>(w_tvar[e]);
        if (wm == 0 && wv == 0) continue;
        double y = 0.0;
        for (int j = 0; j < L.J; ++j)
            y = y + apply_terms(elts[static_cast<int64_t>(L.idx[j]) * C + e], L.R[j], L.Lim[j]);
        const double to = y - L.occR;
        const bool in_occ = (to > 0.0) && (to < L.occL);
        const bool above_occ = to > L.occL;
        if (above_occ) {
            add_i64(&lacc[2 * L.J + 1], wm);
            if (wv) add_i64(&lacc[kMaxP + 2 * L.J + 1], wv);
        }
        if (!in_occ) continue;
        add_i64(&lacc[2 * L.J], -wm);
        if (wv) add_i64(&lacc[kMaxP + 2 * L.J], -wv);
        for (int j = 0; j < L.J; ++j) {
            const double tj = elts[static_cast<int64_t>(L.idx[j]) * C + e] - L.R[j];
            if (tj > 0.0 && tj < L.Lim[j]) {
                add_i64(&lacc[j], -wm);
                if (wv) add_i64(&lacc[kMaxP + j], -wv);
            }
            if (tj > L.Lim[j]) {
                add_i64(&lacc[L.J + j], wm);
                if (wv) add_i64(&lacc[kMaxP + L.J + j], wv);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * kMaxP; i += blockDim.x) {
        const int q = i % kMaxP;
        if (q < P - 2 && lacc[i] != 0) add_i64(&acc[i], lacc[i]);
    }
}

__global__ void finalize_kernel(const long long* acc, const TailStats* tail, int P, int64_t n,
                                double* grad_mean, double* grad_tvar) {
    const int i = threadIdx.x;
    if (i >= P) return;
    const TailStats ts = *tail;
    long long mean = 0, tvar = 0;
#pragma unroll
    for (int c = 0; c < kAccCopies; ++c) {
        mean += acc[c * 2 * kMaxP + i];
        tvar += acc[c * 2 * kMaxP + kMaxP + i];
    }
    if (grad_mean) grad_mean[i] = static_cast<double>(mean) / static_cast<double>(n);
    if (grad_tvar) grad_tvar[i] = static_cast<double>(tvar) / static_cast<double>(ts.m * ts.c_eq);
}

AdjScratch carve(void* base, int64_t C, int64_t n) {
    char* p = static_cast<char*>(base);
    AdjScratch s;
    const int64_t Ca = (C + 255) & ~int64_t(255);
    s.w_mean = reinterpret_cast<uint64_t*>(p);
    p += Ca * sizeof(uint64_t);
    s.w_tvar = reinterpret_cast<uint64_t*>(p);
    p += Ca * sizeof(uint64_t);
    s.acc = reinterpret_cast<long long*>(p);
    p += kAccCopies * 2 * kMaxP * sizeof(long long);
    s.tail = reinterpret_cast<TailStats*>(p);
    p += 256;
    s.mark = reinterpret_cast<uint8_t*>(p);
    p += Ca;
    s.cls = p;
    s.cls_bytes = (stream_adjoint_scratch_bytes(n) + 255) & ~int64_t(255);
    p += s.cls_bytes;
    s.tail_scratch = p;
    return s;
}

}  // namespace

int64_t adjoint_scratch_bytes(int64_t C, int J, int64_t n) {
    (void)J;
    const int64_t Ca = (C + 255) & ~int64_t(255);
    return Ca * (2 * sizeof(uint64_t) + 1) + kAccCopies * 2 * kMaxP * sizeof(long long) + 256 +
           ((stream_adjoint_scratch_bytes(n) + 255) & ~int64_t(255)) + tail_stats_scratch_bytes(n);
}

hipError_t launch_adjoint_fold(const SparsePool& sp, int64_t C, const LayerArgs& L, int P, void* part_scratch,
                               void* scratch, hipStream_t s) {
    const AdjScratch a = carve(scratch, C, L.trial_count);
    return launch_fold_back(sp, C, L, P, part_scratch, FoldBack{a.mark, a.w_mean, a.w_tvar, a.acc, kAccCopies * 2 * kMaxP}, s);
}

hipError_t launch_adjoint(const int64_t* offsets, const uint32_t* ids, const double* elts, int64_t C,
                          const LayerArgs& L, const double* S, const double* ylt, int64_t m, void* scratch,
                          double* d_grad_mean, double* d_grad_tvar, int n_cu, hipStream_t s,
                          const PartLayout* parts, void* part_scratch, int64_t n_trials_total,
                          const SparsePool* sp, const StreamLayout* stream, double density, const LossIndex* losses,
                          void* counts) {
    AdjScratch a = carve(scratch, C, L.trial_count);
    hipError_t err;
    const int64_t n = L.trial_count;
    const int P = 2 * L.J + 4;
    const bool use_parts = parts && parts->P > 0 && part_scratch;
    if ((err = launch_tail_stats(ylt, n, m, a.tail_scratch, a.tail, s)) != hipSuccess) return err;
    if (!sp) {                                      // else launch_adjoint_fold cleared the sums
        hipLaunchKernelGGL(clear_acc_kernel, dim3(1), dim3(256), 0, s, a.acc);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        const uint32_t cblocks = static_cast<uint32_t>((C + 255) / 256);
        hipLaunchKernelGGL(mark_kernel, dim3(cblocks), dim3(256), 0, s, elts, C, L, a.mark, a.w_mean, a.w_tvar,
                           use_parts ? 0 : 1);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (stream && stream->P > 0 && (losses || (use_parts && (stream->P - 1) / 4 < parts->P))) {
        if ((err = launch_stream_classes(*stream, L, S, ylt, a.tail, a.cls, a.cls_bytes, a.acc + P - 2,
                                         a.acc + kMaxP + P - 2, kAccCopies, 2 * kMaxP,
                                         losses ? static_cast<uint64_t*>(counts) : nullptr,
                                         losses ? loss_tvar_words(*losses) : 0, n_cu, s)) != hipSuccess)
            return err;
        err = losses ? launch_loss_adjoint(*stream, *losses, L, static_cast<const uint64_t*>(a.cls), a.tail, counts,
                                           a.w_mean, a.w_tvar, n_cu, s)
                     : launch_stream_adjoint(*stream, density, L, part_scratch, parts->P,
                                             static_cast<const uint8_t*>(a.cls), a.tail, a.w_mean, a.w_tvar, n_cu, s);
        if (err != hipSuccess) return err;
    } else if (use_parts) {
        int64_t ab = (n + 255) / 256;
        if (ab > int64_t(n_cu)) ab = int64_t(n_cu);
        if (ab < 1) ab = 1;
        hipLaunchKernelGGL(agg_counts_kernel, dim3(static_cast<uint32_t>(ab)), dim3(256), 0, s, L, S, ylt, a.tail,
                           a.acc);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        if ((err = launch_part_adjoint(*parts, n_trials_total, L, part_scratch, S, ylt, a.tail, a.w_mean, a.w_tvar,
                                       n_cu, s)) != hipSuccess)
            return err;
    } else {
        int64_t tblocks = (n + 3) / 4;
        if (tblocks > int64_t(n_cu) * 8) tblocks = int64_t(n_cu) * 8;
        if (tblocks < 1) tblocks = 1;
        hipLaunchKernelGGL(active_trials_kernel, dim3(static_cast<uint32_t>(tblocks)), dim3(256), 0, s, offsets,
                           ids, L, S, ylt, a.tail, a.mark, a.w_mean, a.w_tvar, a.acc);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (sp) {
        hipLaunchKernelGGL(catalogue_sparse_kernel, dim3(static_cast<uint32_t>(sp->n_chunks)), dim3(kSparseThreads), 0,
                           s, *sp, C, L, a.mark, a.w_mean, a.w_tvar, a.acc);
    } else {
        int64_t gblocks = (C + 255) / 256;
        if (gblocks > int64_t(n_cu) * 4) gblocks = int64_t(n_cu) * 4;
        hipLaunchKernelGGL(catalogue_kernel, dim3(static_cast<uint32_t>(gblocks)), dim3(256), 0, s, elts, C, L,
                           a.w_mean, a.w_tvar, a.acc);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(256), 0, s, a.acc, a.tail, P, n, d_grad_mean, d_grad_tvar);
    return hipGetLastError();
}

}  // namespace ara
