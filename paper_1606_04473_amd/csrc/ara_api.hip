// C ABI of libara: argument checks, table residency, the library's device
// memory cache, kernel dispatch.  No exception crosses the ABI.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <charconv>
#include <cstdlib>
#include <list>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "ara_internal.hpp"

// ---------------------------------------------------------------------------
// Device memory of the library.  Blocks come from hipMalloc in size classes
// (four per octave, so a block exceeds its request by under 25%) and are kept
// when freed: a freed block is handed out again at once for work on the
// stream that freed it (stream order covers the earlier use), and for work on
// any other stream once an event recorded at the free has completed, which
// is checked without waiting.  In steady state no call allocates from or
// returns memory to the runtime, so independent streams never wait on each
// other inside an allocation.  Idle blocks are released (hipFree) only when
// hipMalloc runs out of memory.
namespace ara {
namespace {

struct CacheBlock {
    size_t size = 0;
    hipStream_t stream = nullptr;   // stream of the last free
    hipEvent_t ready = nullptr;     // recorded on it at that free
    bool in_use = true;
};

struct DeviceCache {
    std::mutex mu;
    std::unordered_map<void*, CacheBlock> blocks;
};

DeviceCache& device_cache(int device) {
    static std::mutex mu;
    static std::vector<std::pair<int, DeviceCache*>> caches;     // kept until the process ends
    std::lock_guard<std::mutex> g(mu);
    for (auto& c : caches)
        if (c.first == device) return *c.second;
    caches.emplace_back(device, new DeviceCache());
    return *caches.back().second;
}

size_t size_class(size_t bytes) {
    if (bytes <= 512) return 512;
    const int k = 63 - __builtin_clzll(static_cast<unsigned long long>(bytes));
    const size_t base = size_t(1) << k;             // base <= bytes < 2 base
    const size_t step = base >> 2;
    return base + (bytes - base + step - 1) / step * step;
}

// hipFree of the idle blocks whose last free has completed, or that have no
// event (hipFree waits for the device); returns the bytes released
int64_t release_idle(DeviceCache& c) {
    std::lock_guard<std::mutex> g(c.mu);
    int64_t freed = 0;
    for (auto it = c.blocks.begin(); it != c.blocks.end();) {
        CacheBlock& b = it->second;
        if (!b.in_use && (!b.ready || hipEventQuery(b.ready) == hipSuccess)) {
            if (b.ready) (void)hipEventDestroy(b.ready);
            (void)hipFree(it->first);
            freed += static_cast<int64_t>(b.size);
            it = c.blocks.erase(it);
        } else {
            ++it;
        }
    }
    return freed;
}

}  // namespace

void cache_stats(int device, int64_t* held, int64_t* idle) {
    DeviceCache& c = device_cache(device);
    std::lock_guard<std::mutex> g(c.mu);
    int64_t h = 0, i = 0;
    for (auto& kv : c.blocks) {
        h += static_cast<int64_t>(kv.second.size);
        if (!kv.second.in_use) i += static_cast<int64_t>(kv.second.size);
    }
    *held = h;
    *idle = i;
}

int64_t cache_release(int device) { return release_idle(device_cache(device)); }

// Events that order work on one device only: nothing on the host reads what came
// before them, so they carry no system-scope fence (a record costs the stream
// 3.4 us instead of 4.5).
constexpr unsigned kOrderEvent = hipEventDisableTiming | hipEventDisableSystemFence;

hipError_t dev_alloc(void** p, size_t bytes, hipStream_t s) {
    *p = nullptr;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    DeviceCache& c = device_cache(device);
    const size_t cls = size_class(bytes);
    {
        std::lock_guard<std::mutex> g(c.mu);
        for (auto& kv : c.blocks) {
            CacheBlock& b = kv.second;
            if (b.in_use || b.size != cls) continue;
            // another stream only once the free is known to be complete (a
            // block without an event serves its own stream only)
            if (b.stream != s && (!b.ready || hipEventQuery(b.ready) != hipSuccess)) continue;
            b.in_use = true;
            *p = kv.first;
            return hipSuccess;
        }
    }
    void* q = nullptr;
    e = hipMalloc(&q, cls);
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);              // what this stream freed is then idle
        release_idle(c);
        e = hipMalloc(&q, cls);
    }
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> g(c.mu);
    CacheBlock b;
    b.size = cls;
    b.stream = s;
    c.blocks.emplace(q, b);
    *p = q;
    return hipSuccess;
}

void dev_free(void* p, hipStream_t s) {
    if (!p) return;
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return;
    DeviceCache& c = device_cache(device);
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.blocks.find(p);
    if (it == c.blocks.end()) return;
    CacheBlock& b = it->second;
    if (!b.ready && hipEventCreateWithFlags(&b.ready, kOrderEvent) != hipSuccess) b.ready = nullptr;
    if (b.ready && hipEventRecord(b.ready, s) != hipSuccess) {
        // without an event the block can only go back to work on s
        (void)hipEventDestroy(b.ready);
        b.ready = nullptr;
    }
    b.stream = s;
    b.in_use = false;
}

void dev_drop(void* p, hipStream_t s) {
    constexpr size_t kKept = size_t(1) << 30;
    int device = 0;
    if (!p || hipGetDevice(&device) != hipSuccess) return;
    DeviceCache& c = device_cache(device);
    bool large = false;
    {
        std::lock_guard<std::mutex> g(c.mu);
        auto it = c.blocks.find(p);
        large = it != c.blocks.end() && it->second.size > kKept;
    }
    if (!large || hipStreamSynchronize(s) != hipSuccess) {
        dev_free(p, s);
        return;
    }
    std::lock_guard<std::mutex> g(c.mu);
    auto it = c.blocks.find(p);
    if (it->second.ready) (void)hipEventDestroy(it->second.ready);
    c.blocks.erase(it);
    (void)hipFree(p);
}

}  // namespace ara

namespace {

thread_local std::string g_error;

ara_status fail(ara_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_error = buf;
    return st;
}

ara_status hip_fail(hipError_t e, const char* what) {
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
        return fail(ARA_ERR_NO_MEMORY, "%s: %s", what, hipGetErrorString(e));
    return fail(ARA_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr, what)                       \
    do {                                          \
        hipError_t e_ = (expr);                   \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

// Make the tables' device current for the scope of a call.
struct DeviceScope {
    int prev = -1;
    bool ok = true;
    explicit DeviceScope(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceScope() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// Stream-ordered scratch that is returned to the pool when the scope ends.
struct PoolBuffer {
    void* p = nullptr;
    hipStream_t s = nullptr;
    ~PoolBuffer() {
        if (p) ara::dev_free(p, s);
    }
    hipError_t alloc(size_t bytes, hipStream_t stream) {
        s = stream;
        if (bytes == 0) bytes = 256;
        return ara::dev_alloc(&p, bytes, stream);
    }
    void free() {
        ara::dev_free(p, s);
        p = nullptr;
    }
};

// Take a kept scratch buffer of at least `bytes` for work on stream s (see
// ScratchBuffer); give it back with scratch_release after enqueueing.
hipError_t scratch_acquire(std::mutex& mu, std::vector<ara::ScratchBuffer*>& sets, size_t bytes, hipStream_t s,
                           ara::ScratchBuffer** out) {
    *out = nullptr;
    ara::ScratchBuffer* pick = nullptr;
    {
        std::lock_guard<std::mutex> g(mu);
        for (auto* b : sets) {
            if (b->busy) continue;
            if (b->stream != s && b->done && hipEventQuery(b->done) != hipSuccess) continue;
            if (!pick || (b->cap >= bytes && (pick->cap < bytes || b->stream == s))) pick = b;
        }
        if (!pick) {
            pick = new (std::nothrow) ara::ScratchBuffer();
            if (!pick) return hipErrorOutOfMemory;
            sets.push_back(pick);
        }
        pick->busy = true;
    }
    hipError_t e = hipSuccess;
    if (!pick->done) e = hipEventCreateWithFlags(&pick->done, ara::kOrderEvent);
    if (e == hipSuccess && pick->cap < bytes) {
        // growing: the old memory may still be read by work on its last
        // stream, so it goes back to the cache in that stream's order; the new
        // memory is taken in this call's stream order
        if (pick->p) ara::dev_free(pick->p, pick->stream);
        pick->p = nullptr;
        pick->cap = 0;
        if (e == hipSuccess) e = ara::dev_alloc(&pick->p, bytes, s);
        if (e == hipSuccess) pick->cap = bytes;
    }
    if (e != hipSuccess) {
        std::lock_guard<std::mutex> g(mu);
        pick->busy = false;
        return e;
    }
    *out = pick;
    return hipSuccess;
}

void scratch_release(std::mutex& mu, ara::ScratchBuffer* b, hipStream_t s) {
    if (!b) return;
    (void)hipEventRecord(b->done, s);
    std::lock_guard<std::mutex> g(mu);
    b->stream = s;
    b->busy = false;
}

// frees on stream fs after each buffer's last use (its event)
void scratch_free_all(std::vector<ara::ScratchBuffer*>& sets, hipStream_t fs) {
    for (auto* b : sets) {
        if (b->done) (void)hipStreamWaitEvent(fs, b->done, 0);
        if (b->p) ara::dev_free(b->p, fs);
        if (b->done) (void)hipEventDestroy(b->done);
        delete b;
    }
    sets.clear();
}

// the stream on which destroyed tables return their memory to the pool (one
// per device, default priority, never destroyed)
hipStream_t free_stream(int device) {
    static std::mutex mu;
    static std::vector<std::pair<int, hipStream_t>> streams;
    std::lock_guard<std::mutex> g(mu);
    for (auto& d : streams)
        if (d.first == device) return d.second;
    hipStream_t st = nullptr;
    if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) st = nullptr;
    streams.emplace_back(device, st);
    return st;
}

// Records, on stream s, an event after the work enqueued there so far on t's
// behalf (one event per stream, re-recorded by later calls).
void note_use(ara_tables* t, hipStream_t s) {
    std::lock_guard<std::mutex> g(t->fence_mu);
    for (auto& f : t->fences)
        if (f.first == s) {
            (void)hipEventRecord(f.second, s);
            return;
        }
    hipEvent_t ev = nullptr;
    if (hipEventCreateWithFlags(&ev, ara::kOrderEvent) != hipSuccess) return;
    if (hipEventRecord(ev, s) != hipSuccess) {
        (void)hipEventDestroy(ev);
        return;
    }
    t->fences.emplace_back(s, ev);
}

// note_use on scope exit, so a call's error returns are covered too; a call that
// holds scratch of the tables hands over to the event its release records anyway
// (destroying the tables waits for those first)
struct UseFence {
    ara_tables* t;
    hipStream_t s;
    void hand_over() { t = nullptr; }
    UseFence(ara_tables* tt, hipStream_t ss) : t(tt), s(ss) {}
    ~UseFence() {
        if (t) note_use(t, s);
    }
};

// releases on scope exit, so early error returns give the buffer back
struct ScratchLease {
    std::mutex& mu;
    ara::ScratchBuffer* b = nullptr;
    hipStream_t s = nullptr;
    ScratchLease(std::mutex& m) : mu(m) {}
    ~ScratchLease() { scratch_release(mu, b, s); }
};

// memory that kernels on `device` read as their own: another device's needs peer
// access, which only the runtime's copies do without
bool memory_of_device(const void* p, int device) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type == hipMemoryTypeDevice && a.device == device;
    (void)hipGetLastError();
    return false;
}

bool bad_term(double v) { return std::isnan(v) || v < 0.0; }

ara_status build_layer_args(const ara_tables* t, const ara_layer& in, ara::LayerArgs& L) {
    std::memset(&L, 0, sizeof(L));
    if (in.n_elts < 0) return fail(ARA_ERR_INVALID_ARG, "layer n_elts < 0");
    if (in.n_elts > ara::kMaxJ)
        return fail(ARA_ERR_UNSUPPORTED, "layer covers %d ELTs; at most %d supported", in.n_elts, ara::kMaxJ);
    if (in.n_elts > 0 && (!in.elt_index || !in.elt_retention || !in.elt_limit))
        return fail(ARA_ERR_INVALID_ARG, "layer ELT arrays are NULL");
    L.J = in.n_elts;
    for (int j = 0; j < in.n_elts; ++j) {
        if (in.elt_index[j] < 0 || in.elt_index[j] >= t->n_pool)
            return fail(ARA_ERR_OUT_OF_RANGE, "ELT index %d outside the pool of %d", in.elt_index[j], t->n_pool);
        if (bad_term(in.elt_retention[j]) || bad_term(in.elt_limit[j]) || std::isinf(in.elt_retention[j]))
            return fail(ARA_ERR_INVALID_ARG, "ELT %d terms must be >= 0, finite retention, not NaN", j);
        L.idx[j] = in.elt_index[j];
        L.R[j] = in.elt_retention[j];
        L.Lim[j] = in.elt_limit[j];
    }
    if (bad_term(in.occ_retention) || bad_term(in.occ_limit) || bad_term(in.agg_retention) ||
        bad_term(in.agg_limit) || std::isinf(in.occ_retention) || std::isinf(in.agg_retention))
        return fail(ARA_ERR_INVALID_ARG, "layer terms must be >= 0, finite retentions, not NaN");
    L.occR = in.occ_retention;
    L.occL = in.occ_limit;
    L.aggR = in.agg_retention;
    L.aggL = in.agg_limit;
    if (in.trial_begin < 0 || in.trial_count < 0 || in.trial_begin > t->n_trials ||
        in.trial_count > t->n_trials - in.trial_begin)
        return fail(ARA_ERR_INVALID_ARG, "trial range [%lld, +%lld) outside [0, %lld)",
                    (long long)in.trial_begin, (long long)in.trial_count, (long long)t->n_trials);
    L.trial_begin = in.trial_begin;
    L.trial_count = in.trial_count;
    return ARA_OK;
}

bool same_layer(const ara::LayerArgs& a, const ara::LayerArgs& b) {
    if (a.J != b.J || a.trial_begin != b.trial_begin || a.trial_count != b.trial_count) return false;
    if (a.occR != b.occR || a.occL != b.occL || a.aggR != b.aggR || a.aggL != b.aggL) return false;
    for (int j = 0; j < a.J; ++j)
        if (a.idx[j] != b.idx[j] || a.R[j] != b.R[j] || a.Lim[j] != b.Lim[j]) return false;
    return true;
}

// m = ceil(n (1 - p)) with p read as the decimal it was written as: the
// shortest decimal string that converts back to the same double (what
// std::to_chars produces), taken exactly.  With that string's digits D and
// k decimal places, p = D / 10^k and m = n - floor(n D / 10^k), clamped to
// [1, n].  n D < 2^63 * 10^17 < 2^120 fits in 128 bits; for k > 38 the
// quotient is 0.  Requires 1 <= n and 0 < p < 1.
int64_t tail_count(int64_t n, double p) {
    char buf[64];
    const auto r = std::to_chars(buf, buf + sizeof(buf), p, std::chars_format::scientific);
    *r.ptr = '\0';
    // "d.ddde-XX" or "de-XX": mantissa digits, then the exponent
    unsigned __int128 D = 0;
    int nd = 0;
    const char* c = buf;
    for (; *c && *c != 'e'; ++c) {
        if (*c == '.') continue;
        D = D * 10u + static_cast<unsigned>(*c - '0');
        ++nd;
    }
    const int e10 = (*c == 'e') ? std::atoi(c + 1) : 0;
    const int k = (nd - 1) - e10;                   // p = D * 10^-k, k >= 1 since p < 1
    unsigned __int128 q = 0;
    if (k <= 38) {
        unsigned __int128 pow10 = 1;
        for (int i = 0; i < k; ++i) pow10 *= 10u;
        q = (static_cast<unsigned __int128>(static_cast<uint64_t>(n)) * D) / pow10;
    }
    int64_t m = n - static_cast<int64_t>(q);
    if (m < 1) m = 1;
    if (m > n) m = n;
    return m;
}

void free_checkpoints(ara::CheckpointState& ck) {
    if (ck.S) (void)hipFree(ck.S);
    if (ck.ylt) (void)hipFree(ck.ylt);
    if (ck.stride) (void)hipFree(ck.stride);
    ck = ara::CheckpointState{};
}

hipError_t take_event(ara::ProfileState& ps, hipEvent_t* ev) {
    if (!ps.free_events.empty()) {
        *ev = ps.free_events.back();
        ps.free_events.pop_back();
        return hipSuccess;
    }
    // timing only: no system-scope fence on record, which would write back and
    // invalidate the caches between the kernels being timed
    return hipEventCreateWithFlags(ev, hipEventDisableSystemFence);
}

// Records an event pair around a launch when profiling is on.
struct KernelTimer {
    ara_tables* t;
    hipStream_t s;
    bool on;
    int kind;
    hipEvent_t a = nullptr, b = nullptr;
    KernelTimer(ara_tables* t_, hipStream_t s_, bool on_, int kind_) : t(t_), s(s_), on(on_), kind(kind_) {
        if (!on) return;
        std::lock_guard<std::mutex> g(t->prof_mu);
        if (take_event(t->prof, &a) != hipSuccess || take_event(t->prof, &b) != hipSuccess) {
            on = false;
            return;
        }
        if (hipEventRecord(a, s) != hipSuccess) on = false;
    }
    void done() {
        if (!on) return;
        if (hipEventRecord(b, s) != hipSuccess) return;
        std::lock_guard<std::mutex> g(t->prof_mu);
        t->prof.pending.push_back({a, b, kind});
        on = false;
    }
};

// Make the staging buffer at least `bytes` and wait for earlier copies out of it.
hipError_t stage_acquire(ara::HostStage& st, size_t bytes) {
    hipError_t e;
    if (!st.done && (e = hipEventCreateWithFlags(&st.done, hipEventDisableTiming)) != hipSuccess) return e;
    if ((e = hipEventSynchronize(st.done)) != hipSuccess) return e;
    if (st.cap < bytes) {
        if (st.p) (void)hipHostFree(st.p);
        st.p = nullptr;
        st.cap = 0;
        size_t want = bytes < (1u << 20) ? (1u << 20) : bytes;
        if ((e = hipHostMalloc(&st.p, want, hipHostMallocDefault)) != hipSuccess) return e;
        st.cap = want;
    }
    return hipSuccess;
}

// Copy a graph's layer arguments to the head of its scratch through its pinned
// stage.  Arguments equal to the last ones copied are already there -- in
// stream order on the stream that copied them, on any stream once that copy
// has completed -- so nothing is copied and the host does not wait for the
// stage: a caller that replays a graph with the same terms can queue many
// replays ahead of the device.
hipError_t upload_layer_args(ara::GraphEntry* e, const void* args, size_t bytes, hipStream_t s) {
    if (e->last.size() == bytes && std::memcmp(e->last.data(), args, bytes) == 0 &&
        (e->last_stream == s || hipEventQuery(e->stage.done) == hipSuccess))
        return hipSuccess;
    e->last.clear();
    hipError_t r = stage_acquire(e->stage, bytes);
    if (r != hipSuccess) return r;
    std::memcpy(e->stage.p, args, bytes);
    if ((r = hipMemcpyAsync(e->scratch, e->stage.p, bytes, hipMemcpyHostToDevice, s)) != hipSuccess) return r;
    if ((r = hipEventRecord(e->stage.done, s)) != hipSuccess) return r;
    const uint8_t* a = static_cast<const uint8_t*>(args);
    e->last.assign(a, a + bytes);
    e->last_stream = s;
    return hipSuccess;
}

void stage_free(ara::HostStage& st) {
    if (st.done) {
        (void)hipEventSynchronize(st.done);
        (void)hipEventDestroy(st.done);
    }
    if (st.p) (void)hipHostFree(st.p);
    st = ara::HostStage{};
}

void free_graph(ara::GraphEntry* g) {
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    stage_free(g->stage);
    if (g->scratch) (void)hipFree(g->scratch);
    delete g;
}

// Host-side description of a batched run.
struct BatchPlan {
    std::vector<ara::BatchLayerDesc> layers;
    std::vector<ara::BatchFoldDesc> fold;
    std::vector<int32_t> idx;
    std::vector<double> R, Lim;
    std::vector<int2> items;
    std::vector<int64_t> key;
};

BatchPlan make_plan(const ara_tables* t, const std::vector<ara::LayerArgs>& L, const double* ylt_ptr,
                    int schedule) {
    BatchPlan b;
    const int T = t->parts.T;
    struct Cost {
        int64_t c;
        int l;
        int64_t tile;
    };
    std::vector<Cost> costs;
    b.key.push_back(static_cast<int64_t>(L.size()));
    b.key.push_back(reinterpret_cast<int64_t>(ylt_ptr));
    for (size_t l = 0; l < L.size(); ++l) {
        const auto& a = L[l];
        b.layers.push_back({a.trial_begin, a.trial_begin + a.trial_count, a.aggR, a.aggL, a.out_offset});
        b.fold.push_back({a.J, static_cast<int32_t>(b.idx.size()), a.occR, a.occL});
        for (int j = 0; j < a.J; ++j) {
            b.idx.push_back(a.idx[j]);
            b.R.push_back(a.R[j]);
            b.Lim.push_back(a.Lim[j]);
        }
        b.key.push_back(a.J);
        b.key.push_back(a.trial_begin);
        b.key.push_back(a.trial_count);
        if (a.trial_count <= 0) continue;
        const int64_t lo = a.trial_begin, hi = a.trial_begin + a.trial_count;
        for (int64_t tile = lo / T; tile * T < hi; ++tile) {
            const int64_t a0 = std::max(lo, tile * T), a1 = std::min(hi, (tile + 1) * T);
            costs.push_back({a1 - a0, static_cast<int>(l), tile});
        }
    }
    // schedule 0: decreasing cost (longest items first); 1: layer-major order
    if (schedule == 0)
        std::stable_sort(costs.begin(), costs.end(), [](const Cost& x, const Cost& y) { return x.c > y.c; });
    b.key.push_back(schedule);
    b.items.reserve(costs.size());
    for (const auto& c : costs) b.items.push_back(make_int2(c.l, static_cast<int>(c.tile)));
    return b;
}

// Copy the plan's descriptors (and, with_items, the work list) into the
// device scratch through pinned staging, on stream s.
hipError_t upload_plan(ara::HostStage& st, const BatchPlan& b, const ara::BatchedScratch& bs, bool with_items,
                       hipStream_t s) {
    const size_t n1 = sizeof(ara::BatchLayerDesc) * b.layers.size();
    const size_t n2 = sizeof(ara::BatchFoldDesc) * b.fold.size();
    const size_t n3 = sizeof(double) * b.R.size();
    const size_t n4 = sizeof(int32_t) * b.idx.size();
    const size_t n5 = with_items ? sizeof(int2) * b.items.size() : 0;
    hipError_t e;
    if ((e = stage_acquire(st, n1 + n2 + 2 * n3 + n4 + n5 + 64)) != hipSuccess) return e;
    char* h = static_cast<char*>(st.p);
    size_t off = 0;
    auto put = [&](void* dst, const void* src, size_t n) -> hipError_t {
        if (n == 0) return hipSuccess;
        std::memcpy(h + off, src, n);
        hipError_t r = hipMemcpyAsync(dst, h + off, n, hipMemcpyHostToDevice, s);
        off += (n + 15) & ~size_t(15);
        return r;
    };
    if ((e = put(bs.layers, b.layers.data(), n1)) != hipSuccess) return e;
    if ((e = put(bs.fold, b.fold.data(), n2)) != hipSuccess) return e;
    if ((e = put(bs.R, b.R.data(), n3)) != hipSuccess) return e;
    if ((e = put(bs.Lim, b.Lim.data(), n3)) != hipSuccess) return e;
    if ((e = put(bs.idx, b.idx.data(), n4)) != hipSuccess) return e;
    if ((e = put(bs.items, b.items.data(), n5)) != hipSuccess) return e;
    return hipEventRecord(st.done, s);
}

// estimated share of the catalogue with a loss in the layer, from its table
// count and the pool's mean nonzero losses per table
double layer_density(const ara_tables* t, const ara::LayerArgs& L) {
    const double cells = static_cast<double>(t->n_pool) * static_cast<double>(t->C);
    return cells > 0.0 ? -std::expm1(-L.J * static_cast<double>(t->sparse.nnz) / cells) : 0.0;
}

// Whether the copy of the pool's events alone is the faster one to stream, for layers
// over `trials` trials in all whose densities add up to `dense` (each times its
// trials).  An estimate of both passes and merges in us, fitted to measured ones.
// That copy costs by its rows (64 trials' slots, padded to the longest) and groups,
// whatever the layer, and by the tables a workgroup takes from part to part; the full
// one by its events, its (part, trial) pairs and its hits, and a start-up that its
// waves share.  Passes, that copy against the full one: 200000 trials of 1000 events
// over 64 tables, a layer of 1: 103 / 115 us where 47 % of the events are in the pool
// (47 parts / 31), 124 / 107 where 73 % are (36 / 16); 16 tables of 16, 15 % of the
// events, 10^6 trials: 155 / 590; whole calls: 554 trials of 38 events 44 / 52 us,
// 20000 of 300 over a pool of 92 %, with the backward: 119 / 104, the 73 % above, with
// two trials per lane: 167 / 159.
bool losses_faster(const ara_tables* t, double trials, double dense) {
    if (t->losses.P <= 0 || trials <= 0.0) return t->losses.P > 0;
    const double per_trial = static_cast<double>(t->n_events) / static_cast<double>(t->n_trials);
    const double rows = static_cast<double>(t->losses.length) / 256.0 * (trials / static_cast<double>(t->n_trials));
    const double groups = t->losses.P * std::ceil(trials / 64.0);
    const double row = t->losses.G == 128 ? 0.127e-3 : 0.104e-3;        // two trials per lane: fewer rows
    auto merge = [&](int parts) { return std::max(1.75e-6 * parts * trials, 0.31 * parts); };
    const double here = (t->loss_index.P > 1 && groups > t->n_cu ? 4.0 : 0.0) + row * rows + 0.078e-3 * groups +
                        merge(t->losses.P);
    const double full = 5.0 + 19.0 * std::min(1.0, trials / 2e5) + 0.3e-6 * per_trial * trials +
                        2.7e-6 * t->stream.P * trials + 1.6e-6 * per_trial * dense + merge(t->stream.P);
    return here <= full;
}
bool losses_faster(const ara_tables* t, const ara::LayerArgs* L, int64_t n) {
    double trials = 0.0, dense = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        const double k = static_cast<double>(std::max<int64_t>(L[i].trial_count, 0));
        trials += k;
        dense += k * layer_density(t, L[i]);
    }
    return losses_faster(t, trials, dense);
}

// A call that finds no memory for its scratch over that copy, which may have more parts,
// runs over the whole one: f(whether that copy may be used).
template <class F>
ara_status on_either_copy(const ara_tables* t, F f) {
    const ara_status st = f(true);
    if (st != ARA_ERR_NO_MEMORY || !t || t->losses.P == 0) return st;
    (void)hipGetLastError();
    return f(false);
}

// The passes that write per-(part, trial) partial sums for a merge: the
// streaming pass over a 16-bit part-major copy (default; the whole one, or the
// pool's events alone), or the XCD-affine pass over the 32-bit partitioned copy
// (pass_variant 2, or tables without the 16-bit copy).
struct SplitPass {
    const ara_tables* t;
    bool stream;
    bool losses;                    // over the copy of the pool's events alone
    SplitPass(const ara_tables* tt, const ara_tuning& tu, bool by_losses)
        : t(tt), stream(tu.pass_variant == 0 && tt->stream.P > 0), losses(stream && tt->losses.P > 0 && by_losses) {}
    const ara::StreamLayout& lay() const { return losses ? t->losses : t->stream; }
    // which pass and copy, as a part of a graph's key
    int64_t kind() const { return losses ? 2 : (stream ? 1 : 0); }
    // the fold, its outputs in part_scratch (terms from L_dev where given)
    hipError_t fold(const ara::LayerArgs& L, const ara::LayerArgs* L_dev, void* part_scratch, uint64_t* probe,
                    hipStream_t s) const {
        if (losses)
            return ara::launch_fold_losses(t->sparse, t->loss_index, t->C, &L, L_dev, 1,
                                           static_cast<double*>(part_scratch), s);
        return ara::launch_fold_parts(t->sparse, t->C, L, L_dev, nullptr, t->parts.P, part_scratch, !stream, probe, s);
    }
    // fold's outputs
    int64_t fold_bytes() const {
        return losses ? ara::loss_table_bytes(t->loss_index) : ara::part_scratch_bytes(t->C, t->parts.P, !stream);
    }
    size_t partial_bytes(int64_t trials) const {
        const int64_t n = trials > 0 ? trials : 1;
        return stream ? static_cast<size_t>(ara::stream_partials_bytes(lay(), n))
                      : sizeof(double) * 2 * static_cast<size_t>(t->parts.P) * n;
    }
    hipError_t pass(const ara::LayerArgs& L, void* part_scratch, void* partials, hipStream_t s) const {
        if (losses) {
            if (L.trial_count <= 0) return hipSuccess;
            const ara::StreamUnit u{0, L.trial_begin, L.trial_count, 0, 0.0};
            return ara::launch_loss_pass_units(t->losses, t->loss_index, &u, 1, static_cast<double*>(part_scratch),
                                               partials, t->n_cu, s);
        }
        if (stream)
            return ara::launch_stream_pass(t->stream, layer_density(t, L), L, part_scratch, t->parts.P, partials,
                                           t->n_cu, s);
        return ara::launch_xcd_pass(t->parts, t->n_trials, t->C, L, part_scratch, static_cast<double*>(partials),
                                    t->n_cu, s);
    }
    // with S the checkpoint of the year losses is written too
    hipError_t combine(const ara::LayerArgs& L, const ara::LayerArgs* L_dev, const void* partials, double* ylt,
                       double* ylt_too, double* S, hipStream_t s) const {
        if (stream) return ara::launch_stream_combine(lay(), L, L_dev, partials, ylt, ylt_too, S, s);
        const hipError_t e =
            ara::launch_xcd_combine(t->parts, L, L_dev, static_cast<const double*>(partials), ylt, S, s);
        if (e != hipSuccess || !ylt_too || L.trial_count <= 0) return e;
        return hipMemcpyAsync(ylt_too, ylt, sizeof(double) * L.trial_count, hipMemcpyDeviceToDevice, s);
    }
};

// Several layers (or trial ranges of layers) through the streaming pass: batches
// of consecutive units share a fold, a pass and a combine launch, as long as
// their scratch (the layers' fold outputs and the units' partial sums) stays
// within kBatchBytes or what the largest unit needs by itself.  A batch saves per
// unit the three launches, the pass's start and end and its LDS images; the
// partial sums of a batch can stay in the 256 MB last-level cache.  Measured, a
// sequence per layer or split against batches: 12 layers of up to 250000 trials of an
// event-loss library 1385 -> 1290 us, a portfolio of 9 layers in 2 splits
// (50000 trials) 720 -> 500 us.
struct StreamBatches {
    static constexpr int64_t kBatchBytes = int64_t(384) << 20;
    struct Batch {
        int first_unit, n_units;
        int first_layer, n_layers;
    };
    SplitPass split;
    std::vector<ara::StreamUnit> units;     // `layer` relative to its batch's first
    std::vector<Batch> batches;
    int64_t scratch_bytes = 0;              // fold outputs and partial sums of the largest batch

    static int64_t up(int64_t n) { return (n + 255) & ~int64_t(255); }
    int64_t fold_bytes(int n_layers) const {
        return up(split.losses ? n_layers * ara::loss_table_bytes(split.t->loss_index)
                               : ara::fold_batch_bytes(n_layers, split.t->parts.P));
    }
    int64_t bytes_of(int n_layers, int64_t trials) const {
        return fold_bytes(n_layers) + up(ara::stream_partials_bytes(split.lay(), trials));
    }
    // How many splits of at most `trials` trials a unit may cover without taking more
    // scratch than a batch: a caller's splits are joined so before they are listed, as a
    // call may name more of them than there is host memory for
    static int64_t splits_per_unit(const SplitPass& sp, int64_t trials, int64_t splits) {
        const StreamBatches b(sp, {});
        int64_t lo = 1, hi = splits;
        while (lo < hi) {
            const int64_t mid = hi - (hi - lo) / 2;
            if (b.bytes_of(1, mid * trials) <= kBatchBytes) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    }
    // units in order of their layers; those of no trials are dropped, and
    // neighbours that continue one layer's range and output are joined
    StreamBatches(const SplitPass& sp, const std::vector<ara::StreamUnit>& in) : split(sp) {
        int64_t most = kBatchBytes;
        for (const auto& u : in) most = std::max(most, bytes_of(1, u.count));
        int64_t trials = 0;
        for (const auto& u : in) {
            if (u.count <= 0) continue;
            Batch* b = batches.empty() ? nullptr : &batches.back();
            if (b) {
                const int n_layers = u.layer - b->first_layer + 1;
                ara::StreamUnit& last = units.back();
                const bool joins = last.layer + b->first_layer == u.layer && last.t_lo + last.count == u.t_lo &&
                                   last.out_at + last.count == u.out_at;
                if (bytes_of(n_layers, trials + u.count) > most ||
                    (!joins && b->n_units >= ara::stream_batch_max()))
                    b = nullptr;
                else if (joins) {
                    last.count += u.count;
                    trials += u.count;
                } else {
                    units.push_back(u);
                    units.back().layer = u.layer - b->first_layer;
                    b->n_units += 1;
                    b->n_layers = n_layers;
                    trials += u.count;
                }
            }
            if (!b) {
                batches.push_back({static_cast<int>(units.size()), 1, u.layer, 1});
                units.push_back(u);
                units.back().layer = 0;
                trials = u.count;
                b = &batches.back();
            }
            scratch_bytes = std::max(scratch_bytes, bytes_of(b->n_layers, trials));
        }
    }

    // every batch's launches; dL holds the layers' arguments, ylt takes out_at
    ara_status run(ara_tables* t, const ara::LayerArgs* dL, void* scratch, double* ylt, bool prof, hipStream_t s) const {
        for (const Batch& b : batches) {
            const ara::StreamUnit* u = units.data() + b.first_unit;
            void* partials = static_cast<char*>(scratch) + fold_bytes(b.n_layers);
            KernelTimer kf(t, s, prof, ARA_KERNEL_FOLD);
            HIP_TRY(split.losses
                        ? ara::launch_fold_losses(t->sparse, t->loss_index, t->C, nullptr, dL + b.first_layer,
                                                  b.n_layers, static_cast<double*>(scratch), s)
                        : ara::launch_fold_batch(t->sparse, t->C, dL + b.first_layer, b.n_layers, t->parts.P, scratch, s),
                    "folds and part images");
            kf.done();
            KernelTimer kp(t, s, prof, ARA_KERNEL_TRIAL_PASS);
            HIP_TRY(split.losses
                        ? ara::launch_loss_pass_units(t->losses, t->loss_index, u, b.n_units,
                                                      static_cast<double*>(scratch), partials, t->n_cu, s)
                        : ara::launch_stream_pass_units(t->stream, u, b.n_units,
                                                        ara::fold_batch_views(scratch, b.n_layers, t->parts.P),
                                                        t->parts.P, partials, t->n_cu, s),
                    "trial pass");
            kp.done();
            KernelTimer kc(t, s, prof, ARA_KERNEL_COMBINE);
            HIP_TRY(ara::launch_stream_combine_units(split.lay(), u, b.n_units, dL + b.first_layer, partials, ylt, s),
                    "partial sums merge");
            kc.done();
        }
        return ARA_OK;
    }
};

int query_cu_count(int device) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess || prop.multiProcessorCount <= 0) return 256;
    return prop.multiProcessorCount;
}

}  // namespace

extern "C" {

const char* ara_last_error(void) { return g_error.c_str(); }

const char* ara_status_string(ara_status s) {
    switch (s) {
        case ARA_OK: return "ARA_OK";
        case ARA_ERR_INVALID_ARG: return "ARA_ERR_INVALID_ARG";
        case ARA_ERR_OUT_OF_RANGE: return "ARA_ERR_OUT_OF_RANGE";
        case ARA_ERR_BUFFER_TOO_SMALL: return "ARA_ERR_BUFFER_TOO_SMALL";
        case ARA_ERR_NO_MEMORY: return "ARA_ERR_NO_MEMORY";
        case ARA_ERR_DEVICE: return "ARA_ERR_DEVICE";
        case ARA_ERR_NOT_READY: return "ARA_ERR_NOT_READY";
        case ARA_ERR_UNSUPPORTED: return "ARA_ERR_UNSUPPORTED";
        default: return "ARA_ERR_UNKNOWN";
    }
}

ara_status ara_tail_count(int64_t n_trials, double p, int64_t* m) {
    if (!m) return fail(ARA_ERR_INVALID_ARG, "m is NULL");
    if (n_trials < 1) return fail(ARA_ERR_INVALID_ARG, "n_trials < 1");
    if (!(p > 0.0 && p < 1.0)) return fail(ARA_ERR_INVALID_ARG, "p must lie in (0, 1)");
    *m = tail_count(n_trials, p);
    return ARA_OK;
}

ara_status ara_device_info(int32_t* n_cu, int32_t* device) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (n_cu) *n_cu = query_cu_count(dev);
    if (device) *device = dev;
    return ARA_OK;
}

static ara_status create_impl(const int64_t* trial_offsets, int64_t n_trials, const uint32_t* event_ids,
                              int64_t n_events, const double* elt_losses, int32_t n_elts, int64_t catalogue_size,
                              uint32_t flags, void* stream, const ara_tables* base, ara_tables** out);

ara_status ara_create_tables(const int64_t* trial_offsets, int64_t n_trials, const uint32_t* event_ids,
                             int64_t n_events, const double* elt_losses, int32_t n_elts,
                             int64_t catalogue_size, uint32_t flags, void* stream, ara_tables** out) {
    return create_impl(trial_offsets, n_trials, event_ids, n_events, elt_losses, n_elts, catalogue_size, flags,
                       stream, nullptr, out);
}

ara_status ara_create_yet(const ara_tables* base, const int64_t* trial_offsets, int64_t n_trials,
                          const uint32_t* event_ids, int64_t n_events, uint32_t flags, void* stream,
                          ara_tables** out) {
    if (!base) return fail(ARA_ERR_INVALID_ARG, "base tables are NULL");
    return create_impl(trial_offsets, n_trials, event_ids, n_events, base->elts, base->n_pool, base->C, flags,
                       stream, base, out);
}

static ara_status create_impl(const int64_t* trial_offsets, int64_t n_trials, const uint32_t* event_ids,
                              int64_t n_events, const double* elt_losses, int32_t n_elts, int64_t catalogue_size,
                              uint32_t flags, void* stream, const ara_tables* base, ara_tables** out) {
    if (!out) return fail(ARA_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n_trials < 0 || n_events < 0 || n_elts < 0 || catalogue_size < 1)
        return fail(ARA_ERR_INVALID_ARG, "negative size or empty catalogue");
    if (catalogue_size >= (int64_t(1) << 32))
        return fail(ARA_ERR_INVALID_ARG, "catalogue of 2^32 events or more (IDs are uint32, 0xFFFFFFFF is reserved)");
    if (!trial_offsets || (n_events > 0 && !event_ids) || (n_elts > 0 && !elt_losses))
        return fail(ARA_ERR_INVALID_ARG, "NULL input array");
    const bool dev_in = (flags & ARA_DEVICE_PTR) != 0;
    if (!dev_in) {
        if (trial_offsets[0] != 0 || trial_offsets[n_trials] != n_events)
            return fail(ARA_ERR_INVALID_ARG, "offsets must start at 0 and end at n_events");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    int device = 0;
    if (base) {
        device = base->device;
        if (hipSetDevice(device) != hipSuccess) return fail(ARA_ERR_DEVICE, "cannot select the base tables' device");
    } else {
        HIP_TRY(hipGetDevice(&device), "hipGetDevice");
    }
    ara_tables* t = new (std::nothrow) ara_tables();
    if (!t) return fail(ARA_ERR_NO_MEMORY, "host allocation failed");
    t->device = device;
    t->n_cu = query_cu_count(device);
    t->n_trials = n_trials;
    t->n_events = n_events;
    t->C = catalogue_size;
    t->n_pool = n_elts;
    auto cleanup = [&](ara_status st) {
        note_use(t, s);                 // the memory goes back after the create's own work
        ara_destroy_tables(t);
        return st;
    };
    const size_t off_bytes = sizeof(int64_t) * (n_trials + 1);
    const size_t id_bytes = sizeof(uint32_t) * (n_events + ara::kIdPad);
    const size_t elt_bytes = base ? 0 : sizeof(double) * static_cast<size_t>(n_elts) * catalogue_size;
    if (base) {
        t->elts = const_cast<double*>(elt_losses);
        t->owns_elts = false;
        t->sparse = base->sparse;
        std::lock_guard<std::mutex> g(const_cast<ara_tables*>(base)->mu);
        t->tuning = base->tuning;
    }
    hipError_t e;
    if ((e = ara::dev_alloc(reinterpret_cast<void**>(&t->offsets), off_bytes, s)) != hipSuccess)
        return cleanup(hip_fail(e, "allocate offsets"));
    if ((e = ara::dev_alloc(reinterpret_cast<void**>(&t->ids), id_bytes, s)) != hipSuccess)
        return cleanup(hip_fail(e, "allocate event ids"));
    if (elt_bytes && (e = hipMalloc(&t->elts, elt_bytes)) != hipSuccess)
        return cleanup(hip_fail(e, "hipMalloc ELT pool"));
    t->bytes = static_cast<int64_t>(off_bytes + id_bytes + elt_bytes);
    const hipMemcpyKind kind = dev_in ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    if ((e = hipMemcpyAsync(t->offsets, trial_offsets, off_bytes, kind, s)) != hipSuccess)
        return cleanup(hip_fail(e, "copy offsets"));
    if (elt_bytes && (e = hipMemcpyAsync(t->elts, elt_losses, elt_bytes, kind, s)) != hipSuccess)
        return cleanup(hip_fail(e, "copy ELT pool"));
    // IDs in this device's memory that lie on 16 bytes are copied by the pass that
    // checks and counts them
    const uint32_t* ids_in = t->ids;
    if (dev_in && reinterpret_cast<uintptr_t>(event_ids) % 16 == 0 && memory_of_device(event_ids, device))
        ids_in = event_ids;
    else if (n_events && (e = hipMemcpyAsync(t->ids, event_ids, sizeof(uint32_t) * n_events, kind, s)) != hipSuccess)
        return cleanup(hip_fail(e, "copy event ids"));
    // The checks and the sizes of the YET's copies, read back at once: the
    // offsets first (the counts walk the trials), then one pass over the IDs,
    // then the copies' starts from the counts.
    PoolBuffer result, counts;
    if ((e = result.alloc(sizeof(ara::CreateResult), s)) != hipSuccess) return cleanup(hip_fail(e, "scratch"));
    ara::CreateResult* d_res = static_cast<ara::CreateResult*>(result.p);
    // counted in the finer parts where the 16-bit copy can be built
    int shift = ara::kImgShift, bins = 0;
    if (!(flags & ARA_PLAIN_LAYOUT) && n_trials > 0) {
        bins = ara::stream_layout_parts(n_trials, catalogue_size);
        if (bins > 0) shift = ara::kStreamShift;
        else bins = ara::part_layout_parts(n_trials, catalogue_size);
    }
    // a copy that does not fit in memory is left out: the passes over the others remain
    auto left_out = [](hipError_t err) {
        if (err != hipErrorOutOfMemory && err != hipErrorMemoryAllocation) return false;
        (void)hipGetLastError();
        return true;
    };
    if (bins > 0) {                 // before the counts, which can be fewer
        e = ara::begin_part_layout(n_trials, catalogue_size, s, &t->parts);
        if (e != hipSuccess && !left_out(e)) return cleanup(hip_fail(e, "partitioned layout"));
    }
    while (bins > 0) {
        e = counts.alloc(sizeof(int32_t) * static_cast<size_t>(n_trials) * bins, s);
        if (e == hipSuccess) break;
        if (!left_out(e)) return cleanup(hip_fail(e, "scratch"));
        // no memory for the finer counts: the 32-bit copy alone, whose parts are a
        // quarter as many; none for those either: the plain layout
        bins = shift == ara::kStreamShift ? t->parts.P : 0;
        shift = ara::kImgShift;
    }
    if (bins == 0) ara::free_part_layout(&t->parts, s);
    int32_t* cnt = static_cast<int32_t*>(counts.p);
    if ((e = ara::launch_create_clear(t->ids + n_events, d_res, cnt, n_trials * bins, t->n_cu, s)) != hipSuccess ||
        (e = ara::launch_validate(t->offsets, n_trials, n_events, t->elts,
                                  base ? 0 : static_cast<int64_t>(n_elts) * catalogue_size, d_res, t->n_cu, s)) !=
            hipSuccess)
        return cleanup(hip_fail(e, "validate kernel"));
    if ((e = ara::launch_yet_count(t->offsets, n_trials, ids_in, t->ids, n_events, catalogue_size, shift, bins, cnt,
                                   d_res, t->n_cu, s)) != hipSuccess)
        return cleanup(hip_fail(e, "pass over the event ids"));
    if (bins > 0) {
        if ((e = ara::plan_part_layout(cnt, shift, bins, n_trials, d_res, s, t->parts)) != hipSuccess)
            return cleanup(hip_fail(e, "partitioned layout"));
        if (shift == ara::kStreamShift) {
            e = ara::plan_stream_layout(cnt, n_trials, n_events, catalogue_size, d_res, s, &t->stream);
            if (e != hipSuccess && !left_out(e)) return cleanup(hip_fail(e, "16-bit stream layout"));
        }
    }
    ara::CreateResult res;
    if ((e = hipMemcpyAsync(&res, d_res, sizeof(res), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (e = hipStreamSynchronize(s)) != hipSuccess)
        return cleanup(hip_fail(e, "read checks and sizes"));
    counts.free();                  // the copies take memory next
    if (res.flags & ara::kCreateBadId)
        return cleanup(fail(ARA_ERR_OUT_OF_RANGE, "an event ID is >= catalogue size %lld", (long long)catalogue_size));
    if (res.flags & ara::kCreateBadOffsets)
        return cleanup(fail(ARA_ERR_INVALID_ARG, "trial offsets must start at 0, not decrease, end at n_events"));
    if (res.flags & ara::kCreateBadLoss) return cleanup(fail(ARA_ERR_INVALID_ARG, "ELT losses must be finite and >= 0"));
    if (!base) {
        // the pool's nonzero entries, which the per-request fold reads
        if ((e = ara::build_sparse_pool(t->elts, n_elts, catalogue_size, s, &t->sparse)) != hipSuccess)
            return cleanup(hip_fail(e, "sparse ELT pool"));
        t->bytes += t->sparse.bytes;
    }
    if (bins > 0) {
        e = ara::fill_part_layout(t->offsets, t->ids, n_trials, n_events, res, s, &t->parts);
        if (e != hipSuccess && t->stream.P > 0 && left_out(e)) {       // rather the 32-bit copy alone than neither
            ara::free_stream_layout(&t->stream, s);
            e = ara::fill_part_layout(t->offsets, t->ids, n_trials, n_events, res, s, &t->parts);
        }
        if (e != hipSuccess) {
            ara::free_part_layout(&t->parts, s);
            if (!left_out(e)) return cleanup(hip_fail(e, "partitioned layout"));
        }
        t->bytes += t->parts.bytes;
        e = ara::fill_stream_layout(t->offsets, t->ids, n_trials, n_events, res, d_res, s, &t->stream);
        if (e != hipSuccess && !left_out(e)) return cleanup(hip_fail(e, "16-bit stream layout"));
        t->bytes += t->stream.bytes;
    }
    // Also the copy of the pool's events alone, for tables that hold both, where the
    // memory is there: the passes then read that where it is faster.
    if (!base && t->stream.P > 0) {
        e = ara::build_losses(t->sparse, n_elts, catalogue_size, t->offsets, t->ids, n_trials, n_events, t->n_cu, s,
                              &t->loss_index, &t->losses);
        if (e != hipSuccess && !left_out(e)) return cleanup(hip_fail(e, "16-bit copy of the events with a loss"));
        t->bytes += t->losses.bytes + t->loss_index.bytes;
    }
    // calls on other streams may follow at once
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return cleanup(hip_fail(e, "synchronize"));
    note_use(t, s);
    *out = t;
    return ARA_OK;
}

void ara_destroy_tables(ara_tables* t) {
    if (!t) return;
    DeviceScope ds(t->device);
    // The YET, its layouts and the kept scratch come from the library's
    // device memory cache: they go back to it on an internal stream once every
    // stream the tables were used on has reached the end of its last call's
    // work, and the host does not wait (a hipFree would wait for the whole
    // device)
    hipStream_t fs = free_stream(t->device);
    {
        std::lock_guard<std::mutex> g(t->fence_mu);
        for (auto& f : t->fences) {
            (void)hipStreamWaitEvent(fs, f.second, 0);
            (void)hipEventDestroy(f.second);
        }
        t->fences.clear();
    }
    for (auto* b : t->scratch)
        if (b->done) (void)hipStreamWaitEvent(fs, b->done, 0);
    if (t->offsets) ara::dev_free(t->offsets, fs);
    if (t->ids) ara::dev_free(t->ids, fs);
    scratch_free_all(t->scratch, fs);
    ara::free_part_layout(&t->parts, fs);
    ara::free_stream_layout(&t->stream, fs);
    ara::free_stream_layout(&t->losses, fs);
    ara::free_loss_index(&t->loss_index, fs);
    if (t->elts && t->owns_elts) (void)hipFree(t->elts);
    if (t->owns_elts) ara::free_sparse_pool(&t->sparse);
    free_checkpoints(t->ck);
    for (auto* g : t->graphs) free_graph(g);
    t->graphs.clear();
    stage_free(t->stage);
    for (auto& p : t->prof.pending) {
        (void)hipEventDestroy(p.start);
        (void)hipEventDestroy(p.stop);
    }
    for (auto e : t->prof.free_events) (void)hipEventDestroy(e);
    delete t;
}

ara_status ara_table_bytes(const ara_tables* t, int64_t* bytes) {
    if (!t || !bytes) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    *bytes = t->bytes;
    return ARA_OK;
}

ara_status ara_cached_memory(int64_t* held_bytes, int64_t* idle_bytes) {
    int device = 0;
    HIP_TRY(hipGetDevice(&device), "hipGetDevice");
    int64_t held = 0, idle = 0;
    ara::cache_stats(device, &held, &idle);
    if (held_bytes) *held_bytes = held;
    if (idle_bytes) *idle_bytes = idle;
    return ARA_OK;
}

ara_status ara_release_cached_memory(int64_t* bytes_released) {
    int device = 0;
    HIP_TRY(hipGetDevice(&device), "hipGetDevice");
    const int64_t freed = ara::cache_release(device);
    if (bytes_released) *bytes_released = freed;
    return ARA_OK;
}

ara_status ara_layout_info_get(const ara_tables* t, ara_layout_info* info) {
    if (!t || !info) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    ara_layout_info v{};
    v.image_parts = t->parts.P;
    v.partitioned_ids = t->parts.length;
    v.partitioned_bytes = t->parts.bytes;
    v.stream_parts = t->stream.P;
    v.stream_group_trials = t->stream.G;
    v.stream_groups = t->stream.NG;
    v.stream_ids = t->stream.length;
    v.stream_bytes = t->stream.bytes;
    *info = v;
    return ARA_OK;
}

ara_status ara_loss_copy_get(const ara_tables* t, const ara_layer* layers, int32_t n_layers, uint32_t flags,
                             ara_loss_copy_info* info) {
    if (!t || !info || n_layers < 0 || (n_layers > 0 && !layers))
        return fail(ARA_ERR_INVALID_ARG, "NULL argument or negative layer count");
    std::vector<ara::LayerArgs> L(n_layers);
    for (int i = 0; i < n_layers; ++i) {
        const ara_status st = build_layer_args(t, layers[i], L[i]);
        if (st != ARA_OK) return st;
    }
    ara_tuning tu;
    {
        std::lock_guard<std::mutex> g(const_cast<ara_tables*>(t)->mu);
        tu = t->tuning;
    }
    const bool other_pass = t->parts.P == 0 || (flags & (ARA_LITERAL | ARA_CHECKPOINT_STRIDE)) != 0;
    ara_loss_copy_info v{};
    v.streamed = n_layers > 0 && !other_pass && SplitPass(t, tu, losses_faster(t, L.data(), n_layers)).losses;
    v.parts = t->loss_index.P;
    v.columns = t->losses.P;
    v.group_trials = t->losses.G;
    v.events = t->loss_index.n_events;
    v.groups = t->losses.NG;
    v.ids = t->losses.length;
    v.bytes = t->losses.bytes + t->loss_index.bytes;
    *info = v;
    return ARA_OK;
}

ara_status ara_kernel_stats(ara_tables* t, int32_t kernel, int64_t* launches, double* total_ms, int32_t reset) {
    if (!t || kernel < 0 || kernel > ARA_KERNEL_AGGREGATE) return fail(ARA_ERR_INVALID_ARG, "bad argument");
    DeviceScope ds(t->device);
    std::lock_guard<std::mutex> g(t->prof_mu);
    auto& ps = t->prof;
    for (auto& p : ps.pending) {
        HIP_TRY(hipEventSynchronize(p.stop), "event synchronize");
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, p.start, p.stop), "event elapsed");
        ps.launches[p.kind] += 1;
        ps.total_ms[p.kind] += ms;
        ps.free_events.push_back(p.start);
        ps.free_events.push_back(p.stop);
    }
    ps.pending.clear();
    if (launches) *launches = ps.launches[kernel];
    if (total_ms) *total_ms = ps.total_ms[kernel];
    if (reset) {
        ps.launches[kernel] = 0;
        ps.total_ms[kernel] = 0.0;
    }
    return ARA_OK;
}

ara_status ara_set_tuning(ara_tables* t, const ara_tuning* tu) {
    if (!t) return fail(ARA_ERR_INVALID_ARG, "NULL tables");
    ara_tuning v{};
    if (tu) v = *tu;
    if (v.lanes_per_trial != 0 && v.lanes_per_trial != 8 && v.lanes_per_trial != 16 &&
        v.lanes_per_trial != 32 && v.lanes_per_trial != 64)
        return fail(ARA_ERR_INVALID_ARG, "lanes_per_trial must be 8, 16, 32 or 64");
    if (v.blocks_per_cu < 0 || v.blocks_per_cu > 64) return fail(ARA_ERR_INVALID_ARG, "blocks_per_cu in [0, 64]");
    if (v.part_lanes_per_trial != 0 && v.part_lanes_per_trial != 8 && v.part_lanes_per_trial != 16 &&
        v.part_lanes_per_trial != 32 && v.part_lanes_per_trial != 64)
        return fail(ARA_ERR_INVALID_ARG, "part_lanes_per_trial must be 8, 16, 32 or 64");
    if (v.schedule < 0 || v.schedule > 1) return fail(ARA_ERR_INVALID_ARG, "schedule must be 0 or 1");
    if (v.pass_variant < 0 || v.pass_variant > 2) return fail(ARA_ERR_INVALID_ARG, "pass_variant must be 0, 1 or 2");
    std::lock_guard<std::mutex> g(t->mu);
    t->tuning = v;
    return ARA_OK;
}

ara_status ara_get_tuning(const ara_tables* t, ara_tuning* tu) {
    if (!t || !tu) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    std::lock_guard<std::mutex> g(const_cast<ara_tables*>(t)->mu);
    *tu = t->tuning;
    return ARA_OK;
}

ara_status ara_footprint(const ara_tables* t, const ara_layer* layers, int32_t n_layers, uint32_t flags,
                         int64_t* bytes) {
    if (!t || !bytes || (n_layers > 0 && !layers) || n_layers < 0)
        return fail(ARA_ERR_INVALID_ARG, "NULL argument or negative layer count");
    int64_t total = 0;
    for (int i = 0; i < n_layers; ++i) total += layers[i].trial_count;
    int64_t b = 0;
    if (!(flags & ARA_LITERAL)) b += sizeof(double) * t->C;            // occurrence losses
    if (!(flags & ARA_LITERAL) && t->parts.P > 0) {
        int64_t most = 0;
        for (int i = 0; i < n_layers; ++i) most = std::max(most, layers[i].trial_count);
        ara_tuning tu;
        {
            std::lock_guard<std::mutex> g(const_cast<ara_tables*>(t)->mu);
            tu = t->tuning;
        }
        int64_t need = 0;
        for (const bool by_losses : {false, true}) {                   // whichever copy the call streams
            const SplitPass split(t, tu, by_losses);
            need = std::max(need, ara::part_scratch_bytes(t->C, t->parts.P, true) +
                                      static_cast<int64_t>(split.partial_bytes(most)));
            if (split.stream && n_layers > 1 && !(flags & (ARA_CHECKPOINT_S | ARA_CHECKPOINT_STRIDE))) {
                std::vector<ara::StreamUnit> units;
                for (int i = 0; i < n_layers; ++i) units.push_back({i, 0, layers[i].trial_count, total, 0.0});
                need = std::max(need, StreamBatches(split, units).scratch_bytes +
                                          static_cast<int64_t>(sizeof(ara::LayerArgs)) * n_layers + 512);
            }
        }
        b += need;
    }
    if (!(flags & ARA_DEVICE_PTR)) b += sizeof(double) * total;       // staged output
    if (flags & (ARA_CHECKPOINT_S | ARA_CHECKPOINT_STRIDE)) b += 2 * sizeof(double) * total;
    if (flags & ARA_CHECKPOINT_STRIDE) b += sizeof(double) * (t->n_events / ara::kStride + 1);
    *bytes = b;
    return ARA_OK;
}

ara_status ara_yet_footprint(int64_t n_trials, int64_t n_events, int64_t catalogue_size, uint32_t flags,
                             int64_t* bytes) {
    if (!bytes || n_trials < 0 || n_events < 0 || catalogue_size < 1)
        return fail(ARA_ERR_INVALID_ARG, "NULL output or negative size");
    const int64_t N = n_trials, E = n_events;
    int64_t b = 8 * (N + 1) + 4 * (E + ara::kIdPad) + 1024;        // offsets, IDs, checks and sizes
    int64_t temp = 0;
    if (!(flags & ARA_PLAIN_LAYOUT) && N > 0) {
        // 32-bit partitioned copy: IDs, segment padding (< 4 per segment,
        // < 32 per tile), segment starts, tile starts; counts while building
        const int64_t P = (catalogue_size + (int64_t(1) << ara::kImgShift) - 1) >> ara::kImgShift;
        if (P <= ara::kMaxParts) {
            const int64_t T = 256, tiles = (N + T - 1) / T;
            b += 4 * (E + 3 * N * P + 32 * tiles + ara::kIdPad) + 4 * tiles * (T * P + 1) + 8 * (tiles + 1);
            temp = 4 * N * P;
        }
        // 16-bit copy: IDs (groups of at least 16 trials padded to 8 IDs per
        // part), trial ends and group starts, part bases; counts while building
        const int64_t Q = (catalogue_size + (int64_t(1) << ara::kStreamShift) - 1) >> ara::kStreamShift;
        if (Q <= ara::kMaxStreamParts) {
            const int64_t NG = (N + 15) / 16;
            b += 2 * (E + 7 * Q * NG + 512) + 2 * ara::kStreamGroupSlots * Q * NG + 4 * Q * (NG + 1) + 8 * (Q + 1);
            temp = 4 * N * Q;
        }
    }
    *bytes = b + temp;
    return ARA_OK;
}

ara_status ara_metrics_footprint(int64_t n_trials, int32_t n_probs, uint32_t flags, int64_t* bytes) {
    if (!bytes || n_trials < 0 || n_probs < 0 || n_probs > 4) return fail(ARA_ERR_INVALID_ARG, "bad argument");
    int64_t b = ara::metrics_scratch_bytes(n_probs, n_trials);
    if (!(flags & ARA_DEVICE_PTR)) b += 8 * n_trials + 8 * (1 + 2 * static_cast<int64_t>(n_probs));
    *bytes = b;
    return ARA_OK;
}

static ara_status run_layers(ara_tables* t, const ara_layer* layers, int32_t n_layers, double* ylt,
                             int64_t ylt_capacity, uint32_t flags, void* stream, bool by_losses) {
    if (!t || !layers || n_layers < 1) return fail(ARA_ERR_INVALID_ARG, "NULL argument or no layer");
    if (flags & ARA_CHECKPOINT_STRIDE) flags |= ARA_CHECKPOINT_S;
    const bool ckpt = (flags & ARA_CHECKPOINT_S) != 0;
    if (ckpt && n_layers != 1) return fail(ARA_ERR_UNSUPPORTED, "ARA_CHECKPOINT_S takes exactly one layer");
    std::vector<ara::LayerArgs> L(n_layers);
    int64_t total = 0;
    for (int i = 0; i < n_layers; ++i) {
        ara_status st = build_layer_args(t, layers[i], L[i]);
        if (st != ARA_OK) return st;
        L[i].out_offset = total;
        total += L[i].trial_count;
    }
    if (total == 0) return ARA_OK;
    if (!ylt) return fail(ARA_ERR_INVALID_ARG, "ylt is NULL");
    if (ylt_capacity < total)
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "ylt holds %lld values, %lld needed", (long long)ylt_capacity,
                    (long long)total);
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    const bool dev_out = (flags & ARA_DEVICE_PTR) != 0;
    const bool literal = (flags & ARA_LITERAL) != 0;
    ara_tuning tu;
    {
        std::lock_guard<std::mutex> g(t->mu);
        tu = t->tuning;
    }
    PoolBuffer staged;
    double* out = ylt;
    if (!dev_out) {
        HIP_TRY(staged.alloc(sizeof(double) * (total > 0 ? total : 1), s), "scratch for YLT");
        out = static_cast<double*>(staged.p);
    }
    // the partitioned passes serve plain runs.  Stride checkpoints need time
    // order: after the streaming or XCD-affine pass a time-ordered pass of their
    // own writes them; with pass_variant 1 the time-ordered trial pass does all
    const bool stride = (flags & ARA_CHECKPOINT_STRIDE) != 0;
    const bool use_parts = !literal && t->parts.P > 0 && !(stride && tu.pass_variant == 1);
    // the streaming pass (default) and the XCD-affine pass (pass_variant 2)
    // write per-part partial sums; pass_variant 1 selects the rank-based pass
    // with the compact value array
    const bool use_xcd = use_parts && tu.pass_variant != 1;
    // (the stride checkpoints read the part images of the whole copy's fold)
    const SplitPass split(t, tu, by_losses && !(flags & ARA_CHECKPOINT_STRIDE) && losses_faster(t, L.data(), n_layers));
    const bool use_stream = use_xcd && split.stream;
    // several layers run as one persistent rank-based launch with pass_variant
    // 1; with the streaming (default) or XCD-affine pass they run one launch
    // sequence per layer, which ARA_GRAPH captures and replays as a whole
    const bool batched = n_layers > 1 && !(flags & ARA_PER_LAYER) && !literal && !ckpt && t->parts.P > 0 &&
                         tu.pass_variant == 1;
    const bool xgraph = (flags & ARA_GRAPH) && use_xcd && !ckpt;
    // several layers over the streaming pass share launches
    bool joined = n_layers > 1 && use_stream && !ckpt;
    std::vector<ara::StreamUnit> units;
    if (joined)
        for (int i = 0; i < n_layers; ++i)
            units.push_back({i, L[i].trial_begin, L[i].trial_count, L[i].out_offset, layer_density(t, L[i])});
    const StreamBatches joint(split, units);
    // one kept scratch buffer for the per-layer path: what the fold leaves for the
    // pass, partial sums (the batched path and graphs keep their own)
    auto up = [](size_t n) { return (n + 255) & ~size_t(255); };
    const size_t o_bytes = literal || use_parts ? 0 : up(sizeof(double) * t->C);
    const size_t p_bytes = !use_parts ? 0 : up(static_cast<size_t>(
        use_xcd ? split.fold_bytes() : ara::part_scratch_bytes(t->C, t->parts.P, true)));
    size_t x_bytes = 0;
    if (use_xcd) {
        int64_t most = 0;
        for (int i = 0; i < n_layers; ++i) most = std::max(most, L[i].trial_count);
        x_bytes = up(split.partial_bytes(most));
    }
    const size_t la_bytes = up(sizeof(ara::LayerArgs) * n_layers);
    ScratchLease lease(t->scratch_mu);
    lease.s = s;
    char* base = nullptr;
    if (!batched && !xgraph) {
        hipError_t e = hipErrorOutOfMemory;
        if (joined) e = scratch_acquire(t->scratch_mu, t->scratch, la_bytes + joint.scratch_bytes + 256, s, &lease.b);
        joined = joined && e == hipSuccess;         // no memory for batches: layer by layer
        if (!joined) {
            if (n_layers > 1) (void)hipGetLastError();
            e = scratch_acquire(t->scratch_mu, t->scratch, o_bytes + p_bytes + x_bytes + 256, s, &lease.b);
        }
        HIP_TRY(e, "scratch for occurrence losses, part images and partial sums");
        use_fence.hand_over();
        base = static_cast<char*>(lease.b->p);
    }
    struct {
        void* p;
    } obuf{base}, pbuf{base ? base + o_bytes : nullptr}, xbuf{base ? base + o_bytes + p_bytes : nullptr};
    double* S_buf = nullptr;
    double* stride_buf = nullptr;
    PoolBuffer probe;                   // the stride checkpoints' lookup tables
    std::unique_lock<std::mutex> ck_lock(t->mu, std::defer_lock);
    if (ckpt) {
        ck_lock.lock();
        auto& ck = t->ck;
        ck.valid = false;
        if (ck.count < L[0].trial_count || !ck.S) {
            if (ck.S) (void)hipFree(ck.S);
            if (ck.ylt) (void)hipFree(ck.ylt);
            ck.S = ck.ylt = nullptr;
            const size_t nb = sizeof(double) * (L[0].trial_count > 0 ? L[0].trial_count : 1);
            HIP_TRY(hipMalloc(&ck.S, nb), "checkpoint S");
            HIP_TRY(hipMalloc(&ck.ylt, nb), "checkpoint YLT");
            ck.count = L[0].trial_count;
        }
        ck.has_stride = false;
        if (flags & ARA_CHECKPOINT_STRIDE) {
            if (!ck.stride) HIP_TRY(hipMalloc(&ck.stride, sizeof(double) * (t->n_events / ara::kStride + 1)),
                                    "stride checkpoints");
            HIP_TRY(ara::launch_fill(ck.stride, t->n_events / ara::kStride + 1, std::nan(""), s), "fill");
            stride_buf = ck.stride;
            ck.has_stride = true;
            if (use_xcd) HIP_TRY(probe.alloc(static_cast<size_t>(ara::probe_table_bytes(t->C)), s), "scratch for probe words");
        }
        S_buf = ck.S;
    }
    if ((flags & ARA_GRAPH) && (batched || xgraph) && (!dev_out || s == nullptr))
        return fail(ARA_ERR_INVALID_ARG, "ARA_GRAPH needs a device output and a non-null stream");
    if (xgraph) {
        // key: the pass captured and the copy it streams (the ELT choices tell which is
        // the faster), layer count, output, trial ranges (terms and ELT choices may
        // change); -1: not a batched plan
        std::vector<int64_t> key{-1, split.kind(), static_cast<int64_t>(n_layers),
                                 reinterpret_cast<int64_t>(out)};
        int64_t most = 0;
        for (int i = 0; i < n_layers; ++i) {
            key.push_back(L[i].trial_begin);
            key.push_back(L[i].trial_count);
            most = std::max(most, L[i].trial_count);
        }
        const size_t xg_bytes = up(split.partial_bytes(most));
        const bool prof = (flags & ARA_PROFILE) != 0;
        std::lock_guard<std::mutex> g(t->stage_mu);
        ara::GraphEntry* ge = nullptr;
        for (auto* c : t->graphs)
            if (c->key == key) ge = c;
        auto upload = [&](ara::GraphEntry* e) -> hipError_t {
            return upload_layer_args(e, L.data(), sizeof(ara::LayerArgs) * n_layers, s);
        };
        if (!ge) {
            ge = new ara::GraphEntry();
            ge->key = key;
            hipError_t e = hipErrorOutOfMemory;
            if (joined) e = hipMalloc(&ge->scratch, la_bytes + joint.scratch_bytes + 256);
            joined = joined && e == hipSuccess;     // no memory for batches: layer by layer
            if (!joined) {
                if (n_layers > 1) (void)hipGetLastError();
                e = hipMalloc(&ge->scratch, la_bytes + p_bytes + xg_bytes);
            }
            if (e != hipSuccess) {
                free_graph(ge);
                return hip_fail(e, "graph scratch");
            }
            char* gb = static_cast<char*>(ge->scratch);
            const ara::LayerArgs* dL = reinterpret_cast<const ara::LayerArgs*>(gb);
            void* gp = gb + la_bytes;
            void* gx = gb + la_bytes + p_bytes;
            if ((e = upload(ge)) != hipSuccess || (e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal)) !=
                                                      hipSuccess) {
                free_graph(ge);
                return hip_fail(e, "graph capture");
            }
            hipError_t le = hipSuccess;
            ara_status js = joined ? joint.run(t, dL, gb + la_bytes, out, false, s) : ARA_OK;
            for (int i = 0; i < n_layers && le == hipSuccess && !joined; ++i) {
                le = split.fold(L[i], dL + i, gp, nullptr, s);
                if (le == hipSuccess) le = split.pass(L[i], gp, gx, s);
                if (le == hipSuccess) le = split.combine(L[i], dL + i, gx, out + L[i].out_offset, nullptr, nullptr, s);
            }
            e = hipStreamEndCapture(s, &ge->graph);
            if (js != ARA_OK) {
                free_graph(ge);
                return js;
            }
            if (le != hipSuccess || e != hipSuccess ||
                (e = hipGraphInstantiate(&ge->exec, ge->graph, nullptr, nullptr, 0)) != hipSuccess) {
                free_graph(ge);
                return hip_fail(le != hipSuccess ? le : e, "graph instantiate");
            }
            if (t->graphs.size() >= 8) {
                free_graph(t->graphs.front());
                t->graphs.erase(t->graphs.begin());
            }
            t->graphs.push_back(ge);
        } else {
            HIP_TRY(upload(ge), "upload layer terms");
        }
        KernelTimer kt(t, s, prof, ARA_KERNEL_BATCHED);
        HIP_TRY(hipGraphLaunch(ge->exec, s), "graph launch");
        kt.done();
        return ARA_OK;
    }
    if (batched) {
        BatchPlan plan = make_plan(t, L, out, tu.schedule);
        const int64_t n_items = static_cast<int64_t>(plan.items.size());
        const int64_t n_elts_total = static_cast<int64_t>(plan.idx.size());
        const int64_t sbytes = ara::batched_scratch_bytes(t->C, t->parts.P, n_layers, n_items, n_elts_total);
        const bool prof = (flags & ARA_PROFILE) != 0;
        if (flags & ARA_GRAPH) {
            std::lock_guard<std::mutex> g(t->stage_mu);
            ara::GraphEntry* ge = nullptr;
            for (auto* c : t->graphs)
                if (c->key == plan.key) ge = c;
            if (!ge) {
                ge = new ara::GraphEntry();
                ge->key = plan.key;
                hipError_t e = hipMalloc(&ge->scratch, sbytes);
                if (e != hipSuccess) {
                    free_graph(ge);
                    return hip_fail(e, "graph scratch");
                }
                ara::BatchedScratch bs =
                    ara::carve_batched(ge->scratch, t->C, t->parts.P, n_layers, n_items, n_elts_total);
                if ((e = upload_plan(ge->stage, plan, bs, true, s)) != hipSuccess ||
                    (e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal)) != hipSuccess) {
                    free_graph(ge);
                    return hip_fail(e, "graph capture");
                }
                hipError_t le = ara::launch_batched(t->parts, t->n_trials, t->C, t->elts, n_layers, bs, n_items, out,
                                                    t->n_cu, s, nullptr, nullptr, tu.part_lanes_per_trial);
                e = hipStreamEndCapture(s, &ge->graph);
                if (le != hipSuccess || e != hipSuccess ||
                    (e = hipGraphInstantiate(&ge->exec, ge->graph, nullptr, nullptr, 0)) != hipSuccess) {
                    free_graph(ge);
                    return hip_fail(le != hipSuccess ? le : e, "graph instantiate");
                }
                if (t->graphs.size() >= 8) {
                    free_graph(t->graphs.front());
                    t->graphs.erase(t->graphs.begin());
                }
                t->graphs.push_back(ge);
            } else {
                ara::BatchedScratch bs =
                    ara::carve_batched(ge->scratch, t->C, t->parts.P, n_layers, n_items, n_elts_total);
                HIP_TRY(upload_plan(ge->stage, plan, bs, false, s), "upload layer terms");
            }
            KernelTimer kt(t, s, prof, ARA_KERNEL_BATCHED);
            HIP_TRY(hipGraphLaunch(ge->exec, s), "graph launch");
            kt.done();
        } else {
            PoolBuffer bbuf;
            HIP_TRY(bbuf.alloc(sbytes, s), "batched scratch");
            ara::BatchedScratch bs = ara::carve_batched(bbuf.p, t->C, t->parts.P, n_layers, n_items, n_elts_total);
            {
                std::lock_guard<std::mutex> g(t->stage_mu);
                HIP_TRY(upload_plan(t->stage, plan, bs, true, s), "upload work list");
            }
            KernelTimer kt(t, s, prof, ARA_KERNEL_BATCHED);
            HIP_TRY(ara::launch_batched(t->parts, t->n_trials, t->C, t->elts, n_layers, bs, n_items, out, t->n_cu, s,
                                        nullptr, nullptr, tu.part_lanes_per_trial),
                    "batched pass");
            kt.done();
        }
    }
    if (joined) {
        ara::LayerArgs* dL = reinterpret_cast<ara::LayerArgs*>(base);
        HIP_TRY(ara::launch_store_terms(L.data(), n_layers, dL, s), "layer terms");
        const ara_status js = joint.run(t, dL, base + la_bytes, out, (flags & ARA_PROFILE) != 0, s);
        if (js != ARA_OK) return js;
    }
    for (int i = 0; i < n_layers && !batched && !joined; ++i) {
        ara::TrialPassArgs a{};
        a.offsets = t->offsets;
        a.ids = t->ids;
        a.elts = t->elts;
        a.C = t->C;
        a.o = static_cast<const double*>(obuf.p);
        a.ylt = out + L[i].out_offset;
        a.S = S_buf;
        a.stride = stride_buf;
        const bool prof = (flags & ARA_PROFILE) != 0;
        if (!literal) {
            KernelTimer kt(t, s, prof, ARA_KERNEL_FOLD);
            if (use_parts)
                HIP_TRY(use_xcd ? split.fold(L[i], nullptr, pbuf.p, static_cast<uint64_t*>(probe.p), s)
                                : ara::launch_fold_parts(t->sparse, t->C, L[i], nullptr, nullptr, t->parts.P, pbuf.p,
                                                         true, static_cast<uint64_t*>(probe.p), s),
                        "fold and part images");
            else
                HIP_TRY(ara::launch_fold(t->elts, t->C, L[i], static_cast<double*>(obuf.p), tu, s), "fold");
            kt.done();
        }
        if (use_xcd) {
            KernelTimer kp(t, s, prof, ARA_KERNEL_TRIAL_PASS);
            HIP_TRY(split.pass(L[i], pbuf.p, xbuf.p, s), "trial pass");
            kp.done();
            KernelTimer kc(t, s, prof, ARA_KERNEL_COMBINE);
            HIP_TRY(split.combine(L[i], nullptr, xbuf.p, a.ylt, ckpt ? t->ck.ylt : nullptr, a.S, s), "partial sums merge");
            kc.done();
            if (stride_buf) {
                HIP_TRY(ara::launch_stride_checkpoints(t->offsets, t->ids, pbuf.p, t->parts.P, t->C,
                                                       static_cast<uint64_t*>(probe.p), L[i], stride_buf, t->n_cu, s),
                        "stride checkpoints");
            }
            continue;
        }
        KernelTimer kt(t, s, prof, ARA_KERNEL_TRIAL_PASS);
        if (use_parts)
            HIP_TRY(ara::launch_part_pass(t->parts, t->n_trials, L[i], pbuf.p, a.ylt, a.S, t->n_cu, s,
                                          tu.part_lanes_per_trial),
                    "partitioned trial pass");
        else
            HIP_TRY(ara::launch_trial_pass(a, L[i], literal, tu, t->n_cu, s), "trial pass");
        kt.done();
    }
    if (ckpt) {
        if (!use_xcd)
            HIP_TRY(hipMemcpyAsync(t->ck.ylt, out, sizeof(double) * L[0].trial_count, hipMemcpyDeviceToDevice, s),
                    "keep YLT");
        t->ck.key = L[0];
        t->ck.valid = true;
    }
    if (!dev_out) {
        HIP_TRY(hipMemcpyAsync(ylt, out, sizeof(double) * total, hipMemcpyDeviceToHost, s), "copy YLT");
        HIP_TRY(hipStreamSynchronize(s), "synchronize");
    }
    return ARA_OK;
}

ara_status ara_run_layers(ara_tables* t, const ara_layer* layers, int32_t n_layers, double* ylt,
                          int64_t ylt_capacity, uint32_t flags, void* stream) {
    return on_either_copy(t, [&](bool by_losses) {
        return run_layers(t, layers, n_layers, ylt, ylt_capacity, flags, stream, by_losses);
    });
}

static ara_status run_portfolio(ara_tables* t, const ara_program* programs, int32_t n_programs, int32_t n_splits,
                                const ara_portfolio_out* out, uint32_t flags, void* stream, bool by_losses) {
    if (!t || !programs || !out) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (n_programs < 1) return fail(ARA_ERR_INVALID_ARG, "a portfolio needs at least one program");
    if (n_programs > ARA_MAX_PROGRAMS)
        return fail(ARA_ERR_UNSUPPORTED, "%d programs, at most %d", n_programs, ARA_MAX_PROGRAMS);
    if (n_splits < 1) return fail(ARA_ERR_INVALID_ARG, "n_splits must be >= 1");
    if (!out->layer_ylt && !out->program_ylt && !out->portfolio_ylt) return fail(ARA_ERR_INVALID_ARG, "no output");
    if (flags & (ARA_CHECKPOINT_S | ARA_CHECKPOINT_STRIDE | ARA_GRAPH))
        return fail(ARA_ERR_INVALID_ARG, "ara_run_portfolio takes ARA_DEVICE_PTR, ARA_LITERAL and ARA_PROFILE");
    std::vector<ara::LayerArgs> L;
    ara::PortfolioSumArgs agg{};
    agg.n_programs = n_programs;
    agg.first[0] = 0;
    for (int p = 0; p < n_programs; ++p) {
        if (programs[p].n_layers < 1 || !programs[p].layers)
            return fail(ARA_ERR_INVALID_ARG, "program %d has no layers", p);
        for (int i = 0; i < programs[p].n_layers; ++i) {
            ara::LayerArgs a;
            ara_status st = build_layer_args(t, programs[p].layers[i], a);
            if (st != ARA_OK) return st;
            if (!L.empty() && (a.trial_begin != L[0].trial_begin || a.trial_count != L[0].trial_count))
                return fail(ARA_ERR_INVALID_ARG, "program %d layer %d covers other trials than the first layer", p, i);
            L.push_back(a);
        }
        agg.first[p + 1] = static_cast<int32_t>(L.size());
    }
    const int64_t n_layers = static_cast<int64_t>(L.size());
    const int64_t begin = L[0].trial_begin, n = L[0].trial_count;
    if (out->layer_ylt && out->layer_capacity < n_layers * n)
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "layer_ylt holds %lld values, %lld needed",
                    (long long)out->layer_capacity, (long long)(n_layers * n));
    if (out->program_ylt && out->program_capacity < n_programs * n)
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "program_ylt holds %lld values, %lld needed",
                    (long long)out->program_capacity, (long long)(n_programs * n));
    if (out->portfolio_ylt && out->portfolio_capacity < n)
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "portfolio_ylt holds %lld values, %lld needed",
                    (long long)out->portfolio_capacity, (long long)n);
    if (n == 0) return ARA_OK;
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    const bool dev_out = (flags & ARA_DEVICE_PTR) != 0;
    const bool literal = (flags & ARA_LITERAL) != 0;
    const bool prof = (flags & ARA_PROFILE) != 0;
    ara_tuning tu;
    {
        std::lock_guard<std::mutex> g(t->mu);
        tu = t->tuning;
    }
    const bool use_parts = !literal && t->parts.P > 0;
    const bool use_xcd = use_parts && tu.pass_variant != 1;
    const SplitPass split(t, tu, by_losses && losses_faster(t, L.data(), n_layers));
    // split i covers [b(i), b(i + 1)): Algorithm 1's YET_i.  More splits than trials are
    // one of each trial and empty ones.
    const int64_t splits = std::min<int64_t>(n_splits, n);
    auto split_at = [&](int64_t i) { return begin + (n * i) / splits; };
    int64_t most = 0;
    for (int64_t i = 0; i < splits; ++i) most = std::max(most, split_at(i + 1) - split_at(i));
    // one kept scratch buffer: what the fold leaves for the passes, partial sums of
    // the largest split, and whatever output the caller keeps on the host
    auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
    const size_t o_bytes = literal || use_parts ? 0 : up(sizeof(double) * t->C);
    const size_t p_bytes = !use_parts ? 0 : up(static_cast<size_t>(
        use_xcd ? split.fold_bytes() : ara::part_scratch_bytes(t->C, t->parts.P, true)));
    // over the streaming pass the layers and splits share launches
    bool joined = use_xcd && split.stream;
    std::vector<ara::StreamUnit> units;
    if (joined) {
        const int64_t per = StreamBatches::splits_per_unit(split, most, splits);
        for (int64_t l = 0; l < n_layers; ++l)
            for (int64_t i = 0; i < splits; i += per)
                units.push_back({static_cast<int32_t>(l), split_at(i), split_at(std::min(i + per, splits)) - split_at(i),
                                 l * n + (split_at(i) - begin), layer_density(t, L[l])});
    }
    const StreamBatches joint(split, units);
    const size_t la_bytes = up(sizeof(ara::LayerArgs) * n_layers);
    const size_t x_bytes = use_xcd ? up(split.partial_bytes(most)) : 0;
    size_t w_bytes = joined ? la_bytes + up(joint.scratch_bytes) : o_bytes + p_bytes + x_bytes;
    const bool stage_layers = !dev_out || !out->layer_ylt;
    const size_t l_bytes = stage_layers ? up(sizeof(double) * n_layers * n) : 0;
    const size_t g_bytes = !dev_out && out->program_ylt ? up(sizeof(double) * n_programs * n) : 0;
    const size_t f_bytes = !dev_out && out->portfolio_ylt ? up(sizeof(double) * n) : 0;
    ScratchLease lease(t->scratch_mu);
    lease.s = s;
    hipError_t me = scratch_acquire(t->scratch_mu, t->scratch, w_bytes + l_bytes + g_bytes + f_bytes + 256, s, &lease.b);
    if (me != hipSuccess && joined) {               // no memory for batches: layer by layer
        (void)hipGetLastError();
        joined = false;
        w_bytes = o_bytes + p_bytes + x_bytes;
        me = scratch_acquire(t->scratch_mu, t->scratch, w_bytes + l_bytes + g_bytes + f_bytes + 256, s, &lease.b);
    }
    HIP_TRY(me, "portfolio scratch");
    use_fence.hand_over();
    char* base = static_cast<char*>(lease.b->p);
    double* o_buf = reinterpret_cast<double*>(base);
    void* p_buf = base + o_bytes;
    void* x_buf = base + o_bytes + p_bytes;
    double* layer_rows = stage_layers ? reinterpret_cast<double*>(base + w_bytes) : out->layer_ylt;
    double* program_rows = nullptr;
    double* portfolio_row = nullptr;
    if (out->program_ylt)
        program_rows = dev_out ? out->program_ylt
                               : reinterpret_cast<double*>(base + w_bytes + l_bytes);
    if (out->portfolio_ylt)
        portfolio_row = dev_out ? out->portfolio_ylt
                                : reinterpret_cast<double*>(base + w_bytes + l_bytes + g_bytes);
    if (joined) {
        ara::LayerArgs* dL = reinterpret_cast<ara::LayerArgs*>(base);
        HIP_TRY(ara::launch_store_terms(L.data(), static_cast<int>(n_layers), dL, s), "layer terms");
        const ara_status js = joint.run(t, dL, base + la_bytes, layer_rows, prof, s);
        if (js != ARA_OK) return js;
    }
    for (int64_t l = 0; l < n_layers && !joined; ++l) {
        if (!literal) {
            KernelTimer kt(t, s, prof, ARA_KERNEL_FOLD);
            if (use_parts)
                HIP_TRY(use_xcd ? split.fold(L[l], nullptr, p_buf, nullptr, s)
                                : ara::launch_fold_parts(t->sparse, t->C, L[l], nullptr, nullptr, t->parts.P, p_buf,
                                                         true, nullptr, s),
                        "fold and part images");
            else
                HIP_TRY(ara::launch_fold(t->elts, t->C, L[l], o_buf, tu, s), "fold");
            kt.done();
        }
        for (int64_t i = 0; i < splits; ++i) {
            ara::LayerArgs Li = L[l];
            Li.trial_begin = split_at(i);
            Li.trial_count = split_at(i + 1) - Li.trial_begin;
            double* ylt_i = layer_rows + l * n + (Li.trial_begin - begin);
            if (use_xcd) {
                KernelTimer kp(t, s, prof, ARA_KERNEL_TRIAL_PASS);
                HIP_TRY(split.pass(Li, p_buf, x_buf, s), "trial pass");
                kp.done();
                KernelTimer kc(t, s, prof, ARA_KERNEL_COMBINE);
                HIP_TRY(split.combine(Li, nullptr, x_buf, ylt_i, nullptr, nullptr, s), "partial sums merge");
                kc.done();
            } else if (use_parts) {
                KernelTimer kp(t, s, prof, ARA_KERNEL_TRIAL_PASS);
                HIP_TRY(ara::launch_part_pass(t->parts, t->n_trials, Li, p_buf, ylt_i, nullptr, t->n_cu, s,
                                              tu.part_lanes_per_trial),
                        "partitioned trial pass");
                kp.done();
            } else {
                ara::TrialPassArgs a{};
                a.offsets = t->offsets;
                a.ids = t->ids;
                a.elts = t->elts;
                a.C = t->C;
                a.o = o_buf;
                a.ylt = ylt_i;
                KernelTimer kp(t, s, prof, ARA_KERNEL_TRIAL_PASS);
                HIP_TRY(ara::launch_trial_pass(a, Li, literal, tu, t->n_cu, s), "trial pass");
                kp.done();
            }
        }
    }
    if (program_rows || portfolio_row) {
        agg.layer_ylt = layer_rows;
        agg.count = n;
        agg.program_ylt = program_rows;
        agg.portfolio_ylt = portfolio_row;
        KernelTimer ka(t, s, prof, ARA_KERNEL_AGGREGATE);
        HIP_TRY(ara::launch_portfolio_sum(agg, t->n_cu, s), "program and portfolio sums");
        ka.done();
    }
    if (!dev_out) {
        if (out->layer_ylt)
            HIP_TRY(hipMemcpyAsync(out->layer_ylt, layer_rows, sizeof(double) * n_layers * n, hipMemcpyDeviceToHost, s),
                    "copy layer YLTs");
        if (out->program_ylt)
            HIP_TRY(hipMemcpyAsync(out->program_ylt, program_rows, sizeof(double) * n_programs * n,
                                   hipMemcpyDeviceToHost, s),
                    "copy program YLTs");
        if (out->portfolio_ylt)
            HIP_TRY(hipMemcpyAsync(out->portfolio_ylt, portfolio_row, sizeof(double) * n, hipMemcpyDeviceToHost, s),
                    "copy portfolio YLT");
        HIP_TRY(hipStreamSynchronize(s), "synchronize");
    }
    return ARA_OK;
}

ara_status ara_run_portfolio(ara_tables* t, const ara_program* programs, int32_t n_programs, int32_t n_splits,
                             const ara_portfolio_out* out, uint32_t flags, void* stream) {
    return on_either_copy(t, [&](bool by_losses) {
        return run_portfolio(t, programs, n_programs, n_splits, out, flags, stream, by_losses);
    });
}

ara_status ara_risk_metrics(const double* ylt, int64_t n_trials, const double* probs, int32_t n_probs,
                            double* mean_out, double* pml_out, double* tvar_out, uint32_t flags, void* stream) {
    if (!ylt || !mean_out || n_probs < 0 || (n_probs > 0 && (!probs || !pml_out || !tvar_out)))
        return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (n_trials < 1) return fail(ARA_ERR_INVALID_ARG, "need at least one trial");
    if (n_probs > 4) return fail(ARA_ERR_UNSUPPORTED, "at most 4 probabilities per call");
    std::vector<int64_t> m(n_probs);
    for (int q = 0; q < n_probs; ++q) {
        if (!(probs[q] > 0.0 && probs[q] < 1.0)) return fail(ARA_ERR_INVALID_ARG, "p must lie in (0, 1)");
        m[q] = tail_count(n_trials, probs[q]);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    int device = 0;
    HIP_TRY(hipGetDevice(&device), "hipGetDevice");
    const bool dev = (flags & ARA_DEVICE_PTR) != 0;
    PoolBuffer staged_in, results;
    // kept per device, like the tables' scratch (see ScratchBuffer)
    static std::mutex metrics_mu;
    static std::list<std::pair<int, std::vector<ara::ScratchBuffer*>>> metrics_sets;   // stable addresses
    std::vector<ara::ScratchBuffer*>* sets = nullptr;
    {
        std::lock_guard<std::mutex> g(metrics_mu);
        for (auto& d : metrics_sets)
            if (d.first == device) sets = &d.second;
        if (!sets) {
            metrics_sets.emplace_back(device, std::vector<ara::ScratchBuffer*>());
            sets = &metrics_sets.back().second;
        }
    }
    ScratchLease scratch(metrics_mu);
    scratch.s = s;
    HIP_TRY(scratch_acquire(metrics_mu, *sets, static_cast<size_t>(ara::metrics_scratch_bytes(n_probs, n_trials)), s,
                            &scratch.b),
            "metrics scratch");
    if (!dev) HIP_TRY(results.alloc(sizeof(double) * (1 + 2 * n_probs), s), "metrics results");
    const double* x = ylt;
    if (!dev) {
        HIP_TRY(staged_in.alloc(sizeof(double) * n_trials, s), "metrics input");
        HIP_TRY(hipMemcpyAsync(staged_in.p, ylt, sizeof(double) * n_trials, hipMemcpyHostToDevice, s), "copy YLT");
        x = static_cast<const double*>(staged_in.p);
    }
    double* r = static_cast<double*>(results.p);
    // device outputs are written by the kernels themselves; host outputs go
    // through the results buffer [mean, PML_0, TVaR_0, PML_1, ...]
    const ara::MetricsOut out = dev ? ara::MetricsOut{mean_out, pml_out, tvar_out, 1}
                                    : ara::MetricsOut{r, r + 1, r + 2, 2};
    HIP_TRY(ara::launch_metrics(x, n_trials, m.data(), n_probs, scratch.b->p, out, s),
            "metrics kernels");
    if (dev) return ARA_OK;
    std::vector<double> h(1 + 2 * n_probs);
    HIP_TRY(hipMemcpyAsync(h.data(), r, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s), "copy metrics");
    HIP_TRY(hipStreamSynchronize(s), "synchronize");
    if (std::isnan(h[0])) return fail(ARA_ERR_INVALID_ARG, "year losses must be >= 0 and not NaN");
    *mean_out = h[0];
    for (int q = 0; q < n_probs; ++q) {
        pml_out[q] = h[1 + 2 * q];
        tvar_out[q] = h[2 + 2 * q];
    }
    return ARA_OK;
}

static ara_status analyze(ara_tables* t, const ara_layer* layer, const double* probs, int32_t n_probs, double* ylt,
                          int64_t ylt_capacity, double* metrics, uint32_t flags, void* stream, bool by_losses) {
    if (!t || !layer || !ylt || !metrics || n_probs < 0 || (n_probs > 0 && !probs))
        return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (n_probs > 4) return fail(ARA_ERR_UNSUPPORTED, "at most 4 probabilities per call");
    if (flags & ~static_cast<uint32_t>(ARA_DEVICE_PTR | ARA_GRAPH | ARA_PROFILE))
        return fail(ARA_ERR_INVALID_ARG, "flags: ARA_DEVICE_PTR, ARA_GRAPH and ARA_PROFILE only");
    ara::LayerArgs L;
    ara_status st = build_layer_args(t, *layer, L);
    if (st != ARA_OK) return st;
    if (L.trial_count < 1) return fail(ARA_ERR_INVALID_ARG, "layer has no trials");
    if (ylt_capacity < L.trial_count)
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "ylt holds %lld values, %lld needed", (long long)ylt_capacity,
                    (long long)L.trial_count);
    std::vector<int64_t> m(n_probs);
    for (int q = 0; q < n_probs; ++q) {
        if (!(probs[q] > 0.0 && probs[q] < 1.0)) return fail(ARA_ERR_INVALID_ARG, "p must lie in (0, 1)");
        m[q] = tail_count(L.trial_count, probs[q]);
    }
    const bool dev = (flags & ARA_DEVICE_PTR) != 0;
    if ((flags & ARA_GRAPH) && (!dev || !stream))
        return fail(ARA_ERR_INVALID_ARG, "ARA_GRAPH needs device outputs and a non-null stream");
    ara_tuning tu;
    {
        std::lock_guard<std::mutex> g(t->mu);
        tu = t->tuning;
    }
    if (!(flags & ARA_GRAPH) || t->parts.P <= 0 || tu.pass_variant == 1) {
        // the two calls one after the other (as ara_run_layers, no graph for
        // the plain layout or the rank-based pass of pass_variant 1)
        st = ara_run_layers(t, layer, 1, ylt, ylt_capacity, flags & (ARA_DEVICE_PTR | ARA_PROFILE), stream);
        if (st != ARA_OK) return st;
        return ara_risk_metrics(ylt, L.trial_count, probs, n_probs, metrics, metrics + 1, metrics + 1 + n_probs,
                                flags & ARA_DEVICE_PTR, stream);
    }
    // one graph: fold, pass, combine and the metrics kernels, on scratch the
    // graph owns.  Terms and ELT choices are read from device memory, so new
    // terms reuse the graph.
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    const SplitPass split(t, tu, by_losses && losses_faster(t, &L, 1));
    auto up = [](size_t n) { return (n + 255) & ~size_t(255); };
    const size_t la_bytes = up(sizeof(ara::LayerArgs));
    const size_t p_bytes = up(static_cast<size_t>(split.fold_bytes()));
    const size_t xg_bytes = up(split.partial_bytes(L.trial_count));
    const size_t m_bytes = up(static_cast<size_t>(ara::metrics_scratch_bytes(n_probs, L.trial_count)));
    // what the graph bakes in: the outputs, the trial range, the pass with its copy and the tail counts
    std::vector<int64_t> key{-2, reinterpret_cast<int64_t>(ylt), reinterpret_cast<int64_t>(metrics), L.trial_begin,
                             L.trial_count, split.kind(), n_probs};
    for (int q = 0; q < n_probs; ++q) key.push_back(m[q]);
    const bool prof = (flags & ARA_PROFILE) != 0;
    std::lock_guard<std::mutex> g(t->stage_mu);
    ara::GraphEntry* ge = nullptr;
    for (auto* c : t->graphs)
        if (c->key == key) ge = c;
    auto upload = [&](ara::GraphEntry* e) -> hipError_t { return upload_layer_args(e, &L, sizeof(L), s); };
    if (!ge) {
        ge = new ara::GraphEntry();
        ge->key = key;
        hipError_t e = hipMalloc(&ge->scratch, la_bytes + p_bytes + xg_bytes + m_bytes);
        if (e != hipSuccess) {
            free_graph(ge);
            return hip_fail(e, "graph scratch");
        }
        char* gb = static_cast<char*>(ge->scratch);
        const ara::LayerArgs* dL = reinterpret_cast<const ara::LayerArgs*>(gb);
        void* gp = gb + la_bytes;
        void* gx = gb + la_bytes + p_bytes;
        void* gm = gb + la_bytes + p_bytes + xg_bytes;
        if ((e = upload(ge)) != hipSuccess ||
            (e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal)) != hipSuccess) {
            free_graph(ge);
            return hip_fail(e, "graph capture");
        }
        hipError_t le = split.fold(L, dL, gp, nullptr, s);
        if (le == hipSuccess) le = split.pass(L, gp, gx, s);
        const ara::MetricsOut mo{metrics, metrics + 1, metrics + 1 + n_probs, 1};
        if (le == hipSuccess && split.stream && ara::combine_metrics_apply(L.trial_count)) {
            le = ara::launch_combine_metrics(static_cast<const double*>(gx),
                                             ara::stream_partials_lo(split.lay(), gx, L.trial_count), split.lay().P,
                                             L.trial_count, dL, ylt, m.data(), n_probs, gm, mo, s);
        } else {
            if (le == hipSuccess) le = split.combine(L, dL, gx, ylt, nullptr, nullptr, s);
            if (le == hipSuccess) le = ara::launch_metrics(ylt, L.trial_count, m.data(), n_probs, gm, mo, s);
        }
        e = hipStreamEndCapture(s, &ge->graph);
        if (le != hipSuccess || e != hipSuccess ||
            (e = hipGraphInstantiate(&ge->exec, ge->graph, nullptr, nullptr, 0)) != hipSuccess) {
            free_graph(ge);
            return hip_fail(le != hipSuccess ? le : e, "graph instantiate");
        }
        if (t->graphs.size() >= 8) {
            free_graph(t->graphs.front());
            t->graphs.erase(t->graphs.begin());
        }
        t->graphs.push_back(ge);
    } else {
        HIP_TRY(upload(ge), "upload layer terms");
    }
    KernelTimer kt(t, s, prof, ARA_KERNEL_BATCHED);
    HIP_TRY(hipGraphLaunch(ge->exec, s), "graph launch");
    kt.done();
    return ARA_OK;
}

ara_status ara_analyze(ara_tables* t, const ara_layer* layer, const double* probs, int32_t n_probs, double* ylt,
                       int64_t ylt_capacity, double* metrics, uint32_t flags, void* stream) {
    return on_either_copy(t, [&](bool by_losses) {
        return analyze(t, layer, probs, n_probs, ylt, ylt_capacity, metrics, flags, stream, by_losses);
    });
}

ara_status ara_risk_metrics_noalloc(const double* ylt, int64_t n_trials, const double* probs, int32_t n_probs,
                                    double* mean_out, double* pml_out, double* tvar_out, void* stream) {
    if (!ylt || !mean_out || n_probs < 0 || (n_probs > 0 && (!probs || !pml_out || !tvar_out)))
        return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (n_trials < 1) return fail(ARA_ERR_INVALID_ARG, "need at least one trial");
    if (n_probs > 4) return fail(ARA_ERR_UNSUPPORTED, "at most 4 probabilities per call");
    int64_t m[4] = {0, 0, 0, 0};
    for (int q = 0; q < n_probs; ++q) {
        if (!(probs[q] > 0.0 && probs[q] < 1.0)) return fail(ARA_ERR_INVALID_ARG, "p must lie in (0, 1)");
        m[q] = tail_count(n_trials, probs[q]);
    }
    void* scratch = nullptr;
    int64_t capacity = 0;
    HIP_TRY(ara::metrics_noalloc_scratch(&scratch, &capacity), "static metrics scratch");
    const int64_t need = ara::metrics_scratch_bytes(n_probs, n_trials);
    if (need > capacity)
        return fail(ARA_ERR_UNSUPPORTED,
                    "%lld trials x %d probabilities need %lld bytes of scratch; the static scratch holds %lld "
                    "(n_probs * n_trials <= %lld); use ara_risk_metrics",
                    (long long)n_trials, n_probs, (long long)need, (long long)capacity,
                    (long long)ARA_METRICS_NOALLOC_KEYS);
    HIP_TRY(ara::launch_metrics(ylt, n_trials, m, n_probs, scratch,
                                ara::MetricsOut{mean_out, pml_out, tvar_out, 1}, static_cast<hipStream_t>(stream)),
            "metrics kernels");
    return ARA_OK;
}

static ara_status backward(ara_tables* t, const ara_layer* layer, double tvar_p, double* grad_mean,
                           double* grad_tvar, uint32_t flags, void* stream, bool by_losses) {
    if (!t || !layer) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (!(tvar_p > 0.0 && tvar_p < 1.0)) return fail(ARA_ERR_INVALID_ARG, "tvar_p must lie in (0, 1)");
    ara::LayerArgs L;
    ara_status st = build_layer_args(t, *layer, L);
    if (st != ARA_OK) return st;
    if (L.trial_count < 1) return fail(ARA_ERR_INVALID_ARG, "layer has no trials");
    std::lock_guard<std::mutex> g(t->mu);
    if (!t->ck.valid || !same_layer(t->ck.key, L))
        return fail(ARA_ERR_NOT_READY, "no checkpointed forward for this layer (run with ARA_CHECKPOINT_S)");
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    const int P = 2 * L.J + 4;
    const bool dev = (flags & ARA_DEVICE_PTR) != 0;
    PoolBuffer scratch, staged;
    HIP_TRY(scratch.alloc(ara::adjoint_scratch_bytes(t->C, L.J, L.trial_count), s), "adjoint scratch");
    double* gm = grad_mean;
    double* gt = grad_tvar;
    if (!dev) {
        HIP_TRY(staged.alloc(sizeof(double) * 2 * P, s), "adjoint output");
        gm = grad_mean ? static_cast<double*>(staged.p) : nullptr;
        gt = grad_tvar ? static_cast<double*>(staged.p) + P : nullptr;
    }
    const int64_t m = tail_count(L.trial_count, tvar_p);
    // with the partitioned layout the histogram pass reads the nonzero bitmap
    // of the part images, rebuilt here from a fold of the layer
    PoolBuffer obuf, pbuf;
    const bool use_parts = t->parts.P > 0;
    // pass_variant 0: the histogram streams the 16-bit copy when the tables
    // hold one; else the XCD-affine pass over the 32-bit partitioned copy
    const bool use_stream = use_parts && t->tuning.pass_variant == 0 && t->stream.P > 0;
    const bool use_losses = by_losses && use_stream && t->sparse.chunk_off && losses_faster(t, &L, 1);
    if (use_parts) {
        const ara_tuning tu = t->tuning;   // t->mu is held
        if (use_losses)                 // that copy's histogram needs no images
            HIP_TRY(pbuf.alloc(ara::loss_adjoint_bytes(t->loss_index, t->n_cu), s), "scratch for counts");
        else
            HIP_TRY(pbuf.alloc(ara::part_scratch_bytes(t->C, t->parts.P, !use_stream), s), "scratch for part images");
        if (!t->sparse.chunk_off) {
            HIP_TRY(obuf.alloc(sizeof(double) * t->C, s), "scratch for occurrence losses");
            HIP_TRY(ara::launch_fold(t->elts, t->C, L, static_cast<double*>(obuf.p), tu, s), "fold");
            HIP_TRY(ara::launch_part_fold(static_cast<const double*>(obuf.p), t->C, t->parts.P, pbuf.p, s, false),
                    "images");
        }
    }
    if (t->sparse.chunk_off)
        HIP_TRY(ara::launch_adjoint_fold(t->sparse, t->C, L, use_parts ? t->parts.P : ara::part_count(t->C),
                                         use_losses ? nullptr : pbuf.p, scratch.p, s),
                "fold");
    HIP_TRY(ara::launch_adjoint(t->offsets, t->ids, t->elts, t->C, L, t->ck.S, t->ck.ylt, m, scratch.p, gm, gt,
                                t->n_cu, s, use_parts ? &t->parts : nullptr, use_losses ? nullptr : pbuf.p, t->n_trials,
                                t->sparse.chunk_off ? &t->sparse : nullptr,
                                use_losses ? &t->losses : (use_stream ? &t->stream : nullptr), layer_density(t, L),
                                use_losses ? &t->loss_index : nullptr, pbuf.p),
            "adjoint kernels");
    if (!dev) {
        std::vector<double> h(2 * P);
        HIP_TRY(hipMemcpyAsync(h.data(), staged.p, sizeof(double) * 2 * P, hipMemcpyDeviceToHost, s), "copy");
        HIP_TRY(hipStreamSynchronize(s), "synchronize");
        if (grad_mean) std::memcpy(grad_mean, h.data(), sizeof(double) * P);
        if (grad_tvar) std::memcpy(grad_tvar, h.data() + P, sizeof(double) * P);
    }
    return ARA_OK;
}

ara_status ara_backward(ara_tables* t, const ara_layer* layer, double tvar_p, double* grad_mean,
                        double* grad_tvar, uint32_t flags, void* stream) {
    return on_either_copy(t, [&](bool by_losses) {
        return backward(t, layer, tvar_p, grad_mean, grad_tvar, flags, stream, by_losses);
    });
}

ara_status ara_debug_lookups(ara_tables* t, const ara_layer* layer, int64_t trial, uint32_t* ids_out,
                             double* losses_out, int64_t capacity, int64_t* n_out, void* stream) {
    if (!t || !layer || !n_out || capacity < 0) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (trial < 0 || trial >= t->n_trials) return fail(ARA_ERR_INVALID_ARG, "trial outside the YET");
    ara_layer probe = *layer;
    probe.trial_begin = 0;
    probe.trial_count = 0;
    ara::LayerArgs L;
    ara_status st = build_layer_args(t, probe, L);
    if (st != ARA_OK) return st;
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    int64_t be[2];
    HIP_TRY(hipMemcpyAsync(be, t->offsets + trial, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s), "offsets");
    HIP_TRY(hipStreamSynchronize(s), "synchronize");
    const int64_t K = be[1] - be[0];
    *n_out = K;
    if (K > capacity) return fail(ARA_ERR_BUFFER_TOO_SMALL, "trial has %lld events, capacity %lld",
                                  (long long)K, (long long)capacity);
    if (K == 0) return ARA_OK;
    if (!ids_out || (L.J > 0 && !losses_out)) return fail(ARA_ERR_INVALID_ARG, "NULL output");
    PoolBuffer dids, dloss;
    HIP_TRY(dids.alloc(sizeof(uint32_t) * K, s), "scratch");
    HIP_TRY(dloss.alloc(sizeof(double) * K * (L.J > 0 ? L.J : 1), s), "scratch");
    HIP_TRY(ara::launch_debug_lookups(t->offsets, t->ids, t->elts, t->C, L, trial, static_cast<uint32_t*>(dids.p),
                                      static_cast<double*>(dloss.p), s),
            "lookup kernel");
    HIP_TRY(hipMemcpyAsync(ids_out, dids.p, sizeof(uint32_t) * K, hipMemcpyDeviceToHost, s), "copy ids");
    if (L.J > 0)
        HIP_TRY(hipMemcpyAsync(losses_out, dloss.p, sizeof(double) * K * L.J, hipMemcpyDeviceToHost, s), "copy");
    HIP_TRY(hipStreamSynchronize(s), "synchronize");
    return ARA_OK;
}

ara_status ara_debug_read(ara_tables* t, const ara_layer* layer, int32_t what, void* out, int64_t capacity,
                          int64_t* n_out, void* stream) {
    if (!t || !n_out || capacity < 0) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    if (what < ARA_DEBUG_OCCURRENCE || what > ARA_DEBUG_STREAM_GEND) return fail(ARA_ERR_INVALID_ARG, "bad `what`");
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    const void* src = nullptr;
    int64_t bytes = 0;
    PoolBuffer buf;
    if (what >= ARA_DEBUG_STREAM_IDS) {
        const ara::StreamLayout& st = t->stream;
        if (st.P == 0) return fail(ARA_ERR_UNSUPPORTED, "the tables hold no 16-bit stream copy");
        switch (what) {
            case ARA_DEBUG_STREAM_IDS: src = st.ids; bytes = sizeof(uint16_t) * st.length; break;
            case ARA_DEBUG_STREAM_BASE: src = st.part_base; bytes = sizeof(int64_t) * (st.P + 1); break;
            case ARA_DEBUG_STREAM_GSTART: src = st.gstart; bytes = sizeof(uint32_t) * st.P * (st.NG + 1); break;
            default: src = st.gend; bytes = sizeof(uint16_t) * st.P * st.NG * ara::kStreamGroupSlots; break;
        }
    } else {
        if (!layer) return fail(ARA_ERR_INVALID_ARG, "the fold's outputs need a layer");
        if (t->parts.P == 0) return fail(ARA_ERR_UNSUPPORTED, "the tables hold no partitioned copy (plain layout)");
        ara_layer probe = *layer;
        probe.trial_begin = 0;
        probe.trial_count = 0;
        ara::LayerArgs L;
        ara_status st = build_layer_args(t, probe, L);
        if (st != ARA_OK) return st;
        const size_t o_bytes = (sizeof(double) * t->C + 255) & ~size_t(255);
        const size_t p_bytes = static_cast<size_t>(ara::part_scratch_bytes(t->C, t->parts.P, true));
        HIP_TRY(buf.alloc(o_bytes + p_bytes, s), "scratch for the fold");
        double* o = static_cast<double*>(buf.p);
        void* pbuf = static_cast<char*>(buf.p) + o_bytes;
        HIP_TRY(ara::launch_fold_parts(t->sparse, t->C, L, nullptr, o, t->parts.P, pbuf, true, nullptr, s),
                "fold and part images");
        if (what == ARA_DEBUG_OCCURRENCE) {
            src = o;
            bytes = sizeof(double) * t->C;
        } else if (what == ARA_DEBUG_IMAGES) {
            src = pbuf;
            bytes = ara::kImgPartBytes * t->parts.P;
        } else {
            const int64_t n_sb = static_cast<int64_t>(t->parts.P) * ara::kImgBase32;
            std::vector<uint32_t> cnt(n_sb);
            HIP_TRY(hipMemcpyAsync(cnt.data(), ara::part_superblock_counts(pbuf, t->parts.P), sizeof(uint32_t) * n_sb,
                                   hipMemcpyDeviceToHost, s),
                    "copy superblock counts");
            HIP_TRY(hipStreamSynchronize(s), "synchronize");
            int64_t nnz = 0;
            for (uint32_t c : cnt) nnz += c;
            src = ara::part_compact_values(pbuf, t->parts.P);
            bytes = sizeof(double) * nnz;
        }
    }
    *n_out = bytes;
    if (bytes > capacity) {
        HIP_TRY(hipStreamSynchronize(s), "synchronize");
        return fail(ARA_ERR_BUFFER_TOO_SMALL, "%lld bytes, capacity %lld", (long long)bytes, (long long)capacity);
    }
    if (bytes > 0) {
        if (!out) return fail(ARA_ERR_INVALID_ARG, "out is NULL");
        HIP_TRY(hipMemcpyAsync(out, src, bytes, hipMemcpyDeviceToHost, s), "copy");
    }
    HIP_TRY(hipStreamSynchronize(s), "synchronize");
    return ARA_OK;
}

ara_status ara_event_nets(ara_tables* t, const ara_layer* layer, double* nets, int64_t capacity, int64_t* n_out,
                          uint32_t flags, void* stream) {
    if (!t || !layer || !n_out || capacity < 0) return fail(ARA_ERR_INVALID_ARG, "NULL argument");
    ara::LayerArgs L;
    ara_status st = build_layer_args(t, *layer, L);
    if (st != ARA_OK) return st;
    DeviceScope ds(t->device);
    if (!ds.ok) return fail(ARA_ERR_DEVICE, "cannot select the tables' device");
    hipStream_t s = static_cast<hipStream_t>(stream);
    UseFence use_fence(t, s);           // the tables' memory outlives this call's work
    // the events of the range; those of the whole table are known
    int64_t be[2] = {0, t->n_events};
    const int64_t t_end = L.trial_begin + L.trial_count;
    if (L.trial_begin > 0)
        HIP_TRY(hipMemcpyAsync(&be[0], t->offsets + L.trial_begin, sizeof(int64_t), hipMemcpyDeviceToHost, s),
                "offsets");
    if (t_end < t->n_trials)
        HIP_TRY(hipMemcpyAsync(&be[1], t->offsets + t_end, sizeof(int64_t), hipMemcpyDeviceToHost, s), "offsets");
    if (L.trial_begin > 0 || t_end < t->n_trials) HIP_TRY(hipStreamSynchronize(s), "synchronize");
    const int64_t n = be[1] - be[0];
    *n_out = n;
    if (n > capacity) return fail(ARA_ERR_BUFFER_TOO_SMALL, "the layer's trials hold %lld events, capacity %lld",
                                  (long long)n, (long long)capacity);
    if (n == 0) return ARA_OK;
    if (!nets) return fail(ARA_ERR_INVALID_ARG, "NULL output");
    const bool dev = (flags & ARA_DEVICE_PTR) != 0;
    // kept scratch: o, the part images with the compact values, the probe
    // words, staged output
    auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
    const int P = ara::part_count(t->C);
    const size_t p_bytes = up(static_cast<size_t>(ara::part_scratch_bytes(t->C, P, false)));
    const size_t w_bytes = up(static_cast<size_t>(ara::probe_table_bytes(t->C)));
    const size_t n_bytes = dev ? 0 : up(sizeof(double) * n);
    ScratchLease lease(t->scratch_mu);
    lease.s = s;
    HIP_TRY(scratch_acquire(t->scratch_mu, t->scratch, p_bytes + w_bytes + n_bytes + 256, s, &lease.b),
            "scratch for part images, probe words and net losses");
    use_fence.hand_over();
    char* base = static_cast<char*>(lease.b->p);
    uint64_t* probe = reinterpret_cast<uint64_t*>(base + p_bytes);
    double* out = dev ? nets : reinterpret_cast<double*>(base + p_bytes + w_bytes);
    HIP_TRY(ara::launch_fold_parts(t->sparse, t->C, L, nullptr, nullptr, P, base, false, probe, s),
            "fold and part images");
    HIP_TRY(ara::launch_event_nets(t->offsets, t->ids, base, P, t->C, probe, layer_density(t, L),
                                   static_cast<double>(n), L, out, t->n_cu, s),
            "net-loss kernel");
    if (!dev) {
        HIP_TRY(hipMemcpyAsync(nets, out, sizeof(double) * n, hipMemcpyDeviceToHost, s), "copy nets");
        HIP_TRY(hipStreamSynchronize(s), "synchronize");
    }
    return ARA_OK;
}

ara_status ara_read_checkpoints(ara_tables* t, int32_t what, double* out, int64_t capacity, int64_t* n_out) {
    if (!t || !n_out || (what != 0 && what != 1)) return fail(ARA_ERR_INVALID_ARG, "bad argument");
    std::lock_guard<std::mutex> g(t->mu);
    if (!t->ck.valid) return fail(ARA_ERR_NOT_READY, "no checkpointed forward");
    if (what == 1 && !t->ck.has_stride)
        return fail(ARA_ERR_NOT_READY, "no stride checkpoints (run with ARA_CHECKPOINT_STRIDE)");
    DeviceScope ds(t->device);
    const int64_t n = what == 0 ? t->ck.key.trial_count : t->n_events / ara::kStride;
    *n_out = n;
    if (capacity < n) return fail(ARA_ERR_BUFFER_TOO_SMALL, "need %lld values", (long long)n);
    if (n == 0) return ARA_OK;
    if (!out) return fail(ARA_ERR_INVALID_ARG, "NULL output");
    HIP_TRY(hipDeviceSynchronize(), "synchronize");
    HIP_TRY(hipMemcpy(out, what == 0 ? t->ck.S : t->ck.stride, sizeof(double) * n, hipMemcpyDeviceToHost), "copy");
    return ARA_OK;
}

}  // extern "C"
