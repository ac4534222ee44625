// Host side of the C ABI: argument validation, the FP64 threshold table,
// launch geometry and the step loop.  Declarations and the contract of every
// entry point are in include/shaken.h.
#include "shaken.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "sd_ahead.hpp"
#include "sd_autotune.hpp"
#include "sd_batch.hpp"
#include "sd_host.hpp"
#include "sd_kernels.hpp"
#include "sd_small.hpp"

namespace sd {

thread_local std::string g_last_error;
static thread_local sd_route g_last_route = SD_ROUTE_NONE;

sd_status fail(sd_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

sd_status hip_fail(hipError_t e, const char* what) {
    return fail(SD_EHIP, "%s: HIP error %d (%s)", what, (int)e, hipGetErrorString(e));
}

bool layout_supported(int32_t L, int32_t layout) {
    if (L < 2 || L > 65535)
        return false;
    switch (layout) {
        case SD_I8:
            return true;
        case SD_P32:
            return L % 32 == 0;
        case SD_P64:
            return L % 8 == 0;
        default:
            return false;
    }
}

size_t lattice_bytes(int32_t L, int32_t layout) {
    if (!layout_supported(L, layout))
        return 0;
    const size_t n = (size_t)L * (size_t)L;
    return layout == SD_I8 ? n : n / 8;
}

int kernel_layout(int32_t L, int32_t layout, const void* p) {
    if (layout == SD_P64)
        return L % 64 == 0 ? kLayP64 : kLayBits;
    if (layout == SD_P32)
        return kLayP32;
    const bool aligned = (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
    return (L % 64 == 0 && aligned) ? kLayI8Row : kLayI8Any;
}

// Kernel layout for the row-oriented reductions (observables, correlations)
// of a packed lattice: 32-bit rows when L % 32 == 0, else the bit string.
int packed_rows_layout(int32_t L) { return L % 32 == 0 ? kLayP32 : kLayBits; }

Geom make_geom(int32_t L, int klay) {
    Geom G;
    G.L = (uint32_t)L;
    G.n_sites = (uint32_t)L * (uint32_t)L;
    G.n_groups = (uint32_t)(((uint64_t)G.n_sites + 63u) / 64u);
    switch (klay) {
        case kLayP64:
        case kLayI8Row:
            G.words_row = (uint32_t)L / 64u;
            break;
        case kLayP32:
            G.words_row = (uint32_t)L / 32u;
            break;
        case kLayBits:
            G.words_row = 1;   // rows need not start on a word: neighbours are string windows
            break;
        default:
            G.words_row = 1;
            break;
    }
    G.div_row = make_fastdiv(G.words_row);
    G.div_L = make_fastdiv((uint32_t)L);
    G.step_rows = 64u / G.words_row;
    G.step_cols = 64u % G.words_row;
    return G;
}

uint32_t threshold(double h) {
    if (h == 0.0)
        return 0x80000000u;
    const double a = std::fabs(h);
    const double u = 4294967296.0 / (1.0 + std::exp(2.0 * a));
    const double r = std::nearbyint(u);
    const uint64_t U = (r < 1.0) ? 1u : (uint64_t)r;
    return h > 0.0 ? (uint32_t)(4294967296ull - U) : (uint32_t)U;
}

void threshold_table(double J, double q, uint32_t T[6]) {
    for (int k = 0; k <= 2; ++k)
        for (int cp = 0; cp <= 1; ++cp)
            T[2 * k + cp] = threshold(J * (double)(2 * k - 2) + q * (double)(2 * cp - 1));
}

DrawParams dynamics_params(double J, double q, uint64_t seed, uint32_t stream, uint32_t t, uint32_t flags) {
    DrawParams dp;
    threshold_table(J, q, dp.T);
    dp.key0 = (uint32_t)(seed & 0xFFFFFFFFu);
    dp.key1 = (uint32_t)(seed >> 32);
    dp.stream = stream;
    dp.t = t;
    dp.tag2 = 2u * kTagDynamics;
    dp.rng_xor = (flags & SD_FLAG_COMPLEMENT_RNG) ? 0xFFFFFFFFu : 0u;
    return dp;
}

sd_status init_params(const char* name, int32_t kind, double p_up, uint64_t seed, uint32_t stream, DrawParams* dp,
                      bool* random, bool* up) {
    if (kind != SD_INIT_UP && kind != SD_INIT_DOWN && kind != SD_INIT_RANDOM)
        return fail(SD_EINVAL, "%s: unknown kind %d", name, kind);
    if (kind == SD_INIT_RANDOM && !(p_up >= 0.0 && p_up <= 1.0))
        return fail(SD_EINVAL, "%s: p_up must lie in [0, 1]", name);
    *dp = DrawParams{};
    const double P = kind == SD_INIT_RANDOM ? std::nearbyint(p_up * 4294967296.0) : 0.0;
    *up = kind == SD_INIT_UP || P >= 4294967296.0;
    *random = kind == SD_INIT_RANDOM && !*up;
    if (*random) {
        for (int i = 0; i < 6; ++i)
            dp->T[i] = (uint32_t)P;
        dp->key0 = (uint32_t)(seed & 0xFFFFFFFFu);
        dp->key1 = (uint32_t)(seed >> 32);
        dp->stream = stream;
        dp->tag2 = 2u * kTagInit;
    }
    return SD_OK;
}

bool overlap(const void* a, const void* b, size_t n) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + n && y < x + n;
}

sd_status check_lattice(const void* p, int32_t L, int32_t layout, const char* name) {
    if (!layout_supported(L, layout))
        return fail(SD_EINVAL, "%s: unsupported (L=%d, layout=%d)", name, L, layout);
    if (!p)
        return fail(SD_EINVAL, "%s: null lattice pointer", name);
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    if ((layout == SD_P64 && (a & 7u)) || (layout == SD_P32 && (a & 3u)))
        return fail(SD_EINVAL, "%s: lattice pointer not aligned to its word size", name);
    return SD_OK;
}

// Launch choice of sd_run for one (device, L, layout), set by sd_tune.
struct RunChoice {
    int mode = 0;           // 0: built-in rule (run_chain), 1: its kernels of several half-steps a launch,
                            // 2: grid kernels
    int width = 64;         // packed layouts with L % 64 == 0: 64- or 32-bit word kernels
    uint32_t blocks = 0;    // grid kernels: workgroups (0 = default)
    // runs that cannot draw ahead by the whole device (sd_run_noalloc, captured
    // runs, the six-class compare) of sizes that otherwise do:
    int mode_free = 0;      // as mode, 1 being the kernels that need no scratch
    uint32_t threads = 256; // LDS kernel: workgroup size
};

std::mutex g_tune_mutex;
std::map<std::tuple<int, int32_t, int32_t>, RunChoice> g_run_choice;

RunChoice run_choice(int32_t L, int32_t layout) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return RunChoice{};
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    auto it = g_run_choice.find(std::make_tuple(dev, L, layout));
    return it == g_run_choice.end() ? RunChoice{} : it->second;
}

hipError_t device_limits(uint32_t* n_cu, size_t* max_lds) {
    int dev = 0, cu = 0, lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    *n_cu = (uint32_t)cu;
    *max_lds = (size_t)lds;
    return e;
}

SmallArgs small_args(int32_t L, double J, double q, uint64_t seed, uint32_t stream, uint64_t step0, uint32_t k_steps,
                     uint32_t flags) {
    SmallArgs a;
    std::memset(&a, 0, sizeof a);
    threshold_table(J, q, a.T);
    a.key0 = (uint32_t)(seed & 0xFFFFFFFFu);
    a.key1 = (uint32_t)(seed >> 32);
    a.stream = stream;
    a.t0 = (uint32_t)(2 * step0);
    a.n_half = 2u * k_steps;
    a.rng_xor = (flags & SD_FLAG_COMPLEMENT_RNG) ? 0xFFFFFFFFu : 0u;
    a.L = (uint32_t)L;
    a.n = lattice_words((uint32_t)L);
    a.div_n = make_fastdiv(a.n);
    a.div_L = make_fastdiv((uint32_t)L);
    return a;
}

static hipError_t launch_small_chain(void* sigma, void* tau, int32_t L, bool int8, double J, double q, uint64_t seed,
                                     uint32_t stream, uint64_t step0, uint32_t k_steps, int64_t* obs,
                                     uint32_t obs_every, uint32_t flags, hipStream_t st) {
    uint32_t n_cu = 0;
    size_t max_lds = 0;
    const hipError_t e = device_limits(&n_cu, &max_lds);
    if (e != hipSuccess)
        return e;
    SmallArgs a = small_args(L, J, q, seed, stream, step0, k_steps, flags);
    a.sigma = sigma;
    a.tau = tau;
    a.int8_io = int8 ? 1u : 0u;
    a.obs = obs;
    a.obs_every = obs ? obs_every : 1u;
    return launch_small(a, 1, false, n_cu, max_lds, st);
}

bool capturing(hipStream_t st) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return cs != hipStreamCaptureStatusNone;
}

// hipMalloc for buffers that are made by the first call that wants them.  In the
// default mode an allocation invalidates what any thread is capturing on any
// stream; this thread's own stream is not being captured here.
static hipError_t malloc_beside_captures(void** p, size_t bytes) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    hipError_t e = hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess)
        return e;
    e = hipMalloc(p, bytes);
    const hipError_t back = hipThreadExchangeStreamCaptureMode(&mode);
    return e == hipSuccess ? back : e;
}

// The stream's workspace; make: one that does not exist yet is made.
static Workspace* stream_workspace(hipStream_t st, bool make) {
    static std::mutex mu;
    static std::map<std::pair<int, hipStream_t>, Workspace*> spaces;   // kept until the process ends
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess)
        return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_pair(dev, st);
    const auto it = spaces.find(key);
    if (it != spaces.end())
        return it->second;
    if (!make)
        return nullptr;
    int64_t* p = nullptr;
    if (malloc_beside_captures(reinterpret_cast<void**>(&p), kPartialsWords * sizeof(int64_t)) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    Workspace* w = new Workspace;
    w->p = p;
    if (st == hipStreamPerThread && hipEventCreateWithFlags(&w->last_use, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        w->lost = true;
    }
    spaces[key] = w;
    return w;
}

// A graph may be replayed on any stream, beside the one it was captured on:
// what it would share with that stream's calls, it must not hold.
WorkspaceUse::WorkspaceUse(hipStream_t st) : st_(st) {
    ws_ = capturing(st) ? nullptr : stream_workspace(st, true);
    if (!ws_)
        return;
    ws_->mu.lock();
    if (st == hipStreamPerThread && (ws_->lost || hipStreamWaitEvent(st, ws_->last_use, 0) != hipSuccess)) {
        (void)hipGetLastError();
        ws_->mu.unlock();
        ws_ = nullptr;
    }
}

void WorkspaceUse::release() {
    if (!ws_)
        return;
    if (st_ == hipStreamPerThread && hipEventRecord(ws_->last_use, st_) != hipSuccess) {
        (void)hipGetLastError();
        ws_->lost = true;
    }
    ws_->mu.unlock();
    ws_ = nullptr;
}

// A scratch buffer that calls on several streams borrow in turn.
struct AheadShared {
    std::mutex mu;   // held while a borrower enqueues
    void* p = nullptr;
    hipEvent_t last_use = nullptr;
};

AheadScratch::AheadScratch(Workspace& ws, hipStream_t st) : st_(st) {
    struct Pool {
        std::mutex mu;
        uint32_t own = 0, next = 0;   // streams with a buffer of their own; the shared one to borrow next
        AheadShared shared[kAheadShared];
    };
    static std::mutex mu;
    static std::map<int, Pool*> pools;   // kept until the process ends
    p_ = ws.ahead;
    int dev = 0;
    if (p_ || hipGetDevice(&dev) != hipSuccess)
        return;
    Pool* pool = nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        Pool*& at = pools[dev];
        if (!at)
            at = new Pool;
        pool = at;
    }
    {
        std::lock_guard<std::mutex> lock(pool->mu);
        if (pool->own < kAheadBuffers) {
            if (malloc_beside_captures(&ws.ahead, kAheadBytes) == hipSuccess) {
                ++pool->own;
                p_ = ws.ahead;
            } else {
                (void)hipGetLastError();
                ws.ahead = nullptr;
            }
            return;
        }
        shared_ = &pool->shared[pool->next++ % kAheadShared];
    }
    shared_->mu.lock();
    AheadShared& s = *shared_;
    hipError_t e = s.last_use ? hipSuccess : hipEventCreateWithFlags(&s.last_use, hipEventDisableTiming);
    if (e == hipSuccess && !s.p)
        e = malloc_beside_captures(&s.p, kAheadBytes);
    if (e == hipSuccess)
        e = hipStreamWaitEvent(st, s.last_use, 0);
    if (e == hipSuccess) {
        p_ = s.p;
        return;
    }
    (void)hipGetLastError();
    s.mu.unlock();
    shared_ = nullptr;
}

AheadScratch::~AheadScratch() {
    if (!shared_)
        return;
    // without the event nothing tells the next borrower when this one is done:
    // the buffer is left behind
    if (hipEventRecord(shared_->last_use, st_) != hipSuccess) {
        (void)hipGetLastError();
        shared_->p = nullptr;
    }
    shared_->mu.unlock();
}

// 64-bit words at their alignment, which 32-bit-word lattices may lack.
static bool words_aligned(const void* sigma, const void* tau) {
    return ((reinterpret_cast<uintptr_t>(sigma) | reinterpret_cast<uintptr_t>(tau)) & 7u) == 0;
}

// True for lattices the draw-ahead kernels take: int8 at any address, packed
// words at 8-byte alignment.
static bool ahead_lattice(int32_t L, int32_t layout, const void* sigma, const void* tau) {
    return ahead_size(L) && (layout == SD_I8 || words_aligned(sigma, tau));
}

// Runs chains through the draw-ahead kernel if the stream's scratch is there;
// *done tells whether it did.  obs: n_chains x n_rec records, chain-major.
static hipError_t run_chains_ahead(void* const* sigma, void* const* tau, uint32_t n_chains, int32_t L, int32_t layout,
                                   const uint32_t (*T)[6], uint64_t seed, const uint32_t* streams, uint64_t step0,
                                   uint32_t k_steps, int64_t* obs, uint32_t obs_every, uint32_t flags, hipStream_t st,
                                   bool* done) {
    *done = false;
    const WorkspaceUse use(st);
    if (!use.get())
        return hipSuccess;
    const AheadScratch scratch(*use.get(), st);
    if (!scratch.get())
        return hipSuccess;
    const uint32_t n_rec = obs ? k_steps / obs_every : 0u;
    AheadArgs a;
    std::memset(&a, 0, sizeof a);
    for (uint32_t c = 0; c < n_chains; ++c) {
        a.sigma[c] = sigma[c];
        a.tau[c] = tau[c];
        std::memcpy(a.T[c], T[c], sizeof a.T[c]);
        a.stream[c] = streams[c];
    }
    a.n_chains = n_chains;
    a.key0 = (uint32_t)(seed & 0xFFFFFFFFu);
    a.key1 = (uint32_t)(seed >> 32);
    a.rng_xor = (flags & SD_FLAG_COMPLEMENT_RNG) ? 0xFFFFFFFFu : 0u;
    a.L = (uint32_t)L;
    a.int8_io = layout == SD_I8 ? 1u : 0u;
    a.obs = n_rec ? obs : nullptr;
    a.obs_chain = 3ull * n_rec;
    a.obs_every = n_rec ? obs_every : 1u;
    g_last_route = SD_ROUTE_AHEAD;
    *done = true;
    static_assert(kAheadBytes >= kAheadMinBytes, "scratch of a run");
    return run_ahead(a, step0, k_steps, scratch.get(), kAheadBytes, st);
}

// Scratch memory of sd_run_noalloc: a file-scope device array (each device
// holds its own copy until the process ends), so that the call allocates
// nothing.  Host code never uses the array's name as an address: its device
// address is looked up once per device with hipGetSymbolAddress and kept.
static __device__ __align__(256) int64_t scratch[kPartialsWords];

sd_status scratch_ptr(const char* name, int64_t** out) {
    static std::mutex mu;
    static std::map<int, int64_t*> ptrs;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e, name);
    std::lock_guard<std::mutex> lock(mu);
    const auto it = ptrs.find(dev);
    if (it != ptrs.end()) {
        *out = it->second;
        return SD_OK;
    }
    int64_t* p = nullptr;
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
        return e != hipSuccess ? hip_fail(e, name) : fail(SD_EHIP, "%s: no device address for the scratch array", name);
    ptrs[dev] = p;
    *out = p;
    return SD_OK;
}

// The step loop of several chains in the grid kernels (or of one): whole steps,
// several per launch, where rows are whole words, else half-steps; records
// through partials (kPartialsWords int64, which a record's sums of either kernel
// must fit), or by atomics without (partials null).
static hipError_t run_many_grid(const ManyChains& mc, const Geom& G, int klay, bool whole_words, bool paired, int32_t L,
                                uint64_t seed, uint64_t step0, uint32_t k_steps, int64_t* obs, uint32_t n_rec,
                                uint32_t obs_every, uint32_t flags, int64_t* partials, hipStream_t st) {
    const uint32_t stride = 4u * mc.blocks_per_chain * mc.n_chains;   // partial sums of one record
    DrawParams base = dynamics_params(0.0, 0.0, seed, 0u, 0u, flags & SD_FLAG_COMPLEMENT_RNG);
    const uint32_t chunk = n_rec ? (uint32_t)(kPartialsWords / stride) : 1u;
    const uint64_t obs_chain = 3ull * n_rec;
    uint32_t pending = 0;
    hipError_t e = hipSuccess;
    if (n_rec && !partials)
        e = launch_fill_i64(obs, (size_t)mc.n_chains * obs_chain, 0, st);
    // Rows of at most 64 words: whole steps, several per launch (bands with
    // halo rows, sigma alternating between the two lattices of each chain),
    // for all but the last step, in an even number of launches so that sigma
    // ends where it started; the last step takes the half-step kernels, which
    // leave tau in place.
    uint32_t n_cu = 0;
    size_t max_lds = 0;
    if (const hipError_t ed = device_limits(&n_cu, &max_lds); ed != hipSuccess)
        return ed;
    const BandPlan plan = band_plan(L, mc.n_chains, n_cu);
    uint32_t depth = plan.depth;
    if (depth && n_rec && partials) {   // the records of one launch must fit the partial-sum buffer
        const uint64_t per_rec = 4ull * plan.bands * mc.n_chains;
        depth = (uint32_t)std::min<uint64_t>(depth, kPartialsWords / per_rec);
    }
    const bool band_ok = depth != 0 && whole_words && k_steps >= 3;
    uint32_t n_fused = band_ok ? k_steps - 1u : 0u;
    // an even number of launches of at most `depth` steps, none empty
    uint32_t n_launch = n_fused ? (n_fused + depth - 1) / depth : 0u;
    n_launch += n_launch % 2;
    if (n_launch > n_fused)   // one step per launch and an odd count: leave one more step to the half-steps
        n_launch = --n_fused;
    g_last_route = n_fused ? SD_ROUTE_BANDS : SD_ROUTE_HALF_STEPS;
    if (n_fused) {
        BandArgs ba;
        std::memset(&ba, 0, sizeof ba);
        for (uint32_t a = 0; a < mc.n_chains; ++a) {
            std::memcpy(ba.T[a], mc.T[a], sizeof ba.T[a]);
            ba.stream[a] = mc.stream[a];
        }
        ba.n_chains = mc.n_chains;
        ba.L = (uint32_t)L;
        ba.W = (uint32_t)L / 64u;
        ba.bands = plan.bands;
        ba.divW = make_fastdiv(ba.W);
        const uint32_t R = ((uint32_t)L + ba.bands - 1u) / ba.bands;   // of the widest band
        ba.key0 = base.key0;
        ba.key1 = base.key1;
        const uint32_t stride_b = 4u * ba.bands * ba.n_chains;
        const uint32_t chunk_b = (uint32_t)(kPartialsWords / stride_b);
        ba.rec_stride = stride_b;
        ba.obs = obs;
        ba.obs_chain = obs_chain;
        const bool complement = (flags & SD_FLAG_COMPLEMENT_RNG) != 0;
        uint32_t m = 0;   // steps done
        for (uint32_t j = 0; j < n_launch && e == hipSuccess; ++j) {
            const uint32_t steps = n_fused / n_launch + (j < n_fused % n_launch ? 1u : 0u);
            for (uint32_t a = 0; a < mc.n_chains; ++a) {
                ba.src[a] = j % 2 ? mc.tau[a] : mc.sigma[a];
                ba.dst[a] = j % 2 ? mc.sigma[a] : mc.tau[a];
            }
            ba.t0 = (uint32_t)(2 * (step0 + m));
            ba.steps = steps;
            ba.threads = band_threads(R, ba.W, steps);
            ba.rec_mask = 0;
            uint32_t n_here = 0;
            if (n_rec)
                for (uint32_t s = 0; s < steps; ++s)
                    if ((m + s + 1) % obs_every == 0) {
                        ba.rec_mask |= 1u << s;
                        ++n_here;
                    }
            ba.rec0 = n_here ? (m + obs_every) / obs_every - 1 : 0u;   // first record of this launch
            if (partials && n_here && pending + n_here > chunk_b) {
                e = launch_obs_finish_many(partials, ba.bands, mc.n_chains, pending, stride_b, obs, obs_chain,
                                           ba.rec0 - pending, st);
                pending = 0;
                if (e != hipSuccess)
                    break;
            }
            e = launch_band_step(ba, klay == kLayI8Row, paired, complement,
                                 partials ? partials + (size_t)pending * stride_b : nullptr, st);
            m += steps;
            pending += partials ? n_here : 0u;
            if (e == hipSuccess && pending && j + 1 == n_launch) {
                e = launch_obs_finish_many(partials, ba.bands, mc.n_chains, pending, stride_b, obs, obs_chain,
                                           m / obs_every - pending, st);
                pending = 0;
            }
        }
    }
    for (uint32_t m = n_fused; m < k_steps && e == hipSuccess; ++m) {
        const uint64_t n = step0 + m;
        base.t = (uint32_t)(2 * n);
        e = launch_half_step_many(klay, 0, mc, G, base, paired, nullptr, nullptr, st);
        if (e != hipSuccess)
            break;
        base.t = (uint32_t)(2 * n + 1);
        const bool rec = n_rec && (m + 1) % obs_every == 0 && (m + 1) / obs_every <= n_rec;
        const uint32_t r = rec ? (m + 1) / obs_every - 1 : 0u;
        e = launch_half_step_many(klay, 1, mc, G, base, paired, rec ? obs + 3u * (size_t)r : nullptr,
                                  rec && partials ? partials + (size_t)pending * stride : nullptr, st);
        if (rec && partials && e == hipSuccess) {
            ++pending;
            if (pending == chunk || r + 1 == n_rec) {
                e = launch_obs_finish_many(partials, mc.blocks_per_chain, mc.n_chains, pending, stride, obs,
                                           obs_chain, r + 1 - pending, st);
                pending = 0;
            }
        }
    }
    return e;
}

// Word draws (words x half-steps) from which a lattice of at most 64 words is
// drawn ahead by the whole device rather than by its own workgroup, which
// saves a launch (us a call, own workgroup against device: 64^2, 10 steps 11.4
// against 12.8, 20 steps 17.6 against 12.9; 32^2, 40 steps 12.3 against 13.4,
// 100 steps 25 against 20).
constexpr uint64_t kAheadDraws = 2048;

// The shortest runs past 64 words pay more for drawing ahead, a launch each to
// draw, to walk and to take records, with one workgroup walking, than they save.
// One step goes to the LDS kernel where that takes the lattice (us a call, drawn
// ahead against it: 128^2 9.6 7.5, recorded 13.8 8.7; 200^2 15.5 10.5, 18.8 11.0),
// and past 512 words to half-steps where it does not (333^2 int8 23.1 13.3,
// recorded 27.2 19.6; 200^2 int8 18.1 10.5; up to there drawn ahead, 180^2 int8
// 16.2 18.4, 127^2 13.9 19.1).  Two recorded steps go to the LDS kernel where it
// has four tiles or fewer (128^2 13.6 10.6; 136^2 and up drawn ahead).
static bool ahead_steps(uint32_t n_words, uint32_t k_steps, bool records, bool lds) {
    if (n_words <= 64u || k_steps > 2u)
        return true;
    if (k_steps == 1u)
        return !lds && n_words <= 512u;
    return !(records && lds && n_words <= 256u);
}

// The step loop behind sd_run and sd_run_noalloc.  The grid kernels of a
// recorded half-step B leave per-workgroup partial sums in a device buffer of
// kPartialsWords int64: the per-(device, stream) workspace for sd_run (null
// under stream capture: atomics into the records instead), the static scratch
// array for sd_run_noalloc.
sd_status run_chain(const char* name, void* sigma, void* tau, int32_t L, int32_t layout, double J, double q,
                    uint64_t seed, uint32_t stream, uint64_t step0, uint32_t k_steps, int64_t* obs,
                    uint32_t obs_every, uint32_t flags, void* hip_stream, bool no_alloc) {
    g_last_route = SD_ROUTE_NONE;
    sd_status s = check_lattice(sigma, L, layout, name);
    if (s == SD_OK)
        s = check_lattice(tau, L, layout, name);
    if (s != SD_OK)
        return s;
    if (!std::isfinite(J) || !std::isfinite(q))
        return fail(SD_EINVAL, "%s: J and q must be finite", name);
    if (step0 + (uint64_t)k_steps > (1ull << 29))
        return fail(SD_EINVAL, "%s: step indices must stay below 2^29", name);
    if (obs && obs_every == 0)
        return fail(SD_EINVAL, "%s: obs given without obs_every", name);
    if (flags & ~(SD_FLAG_COMPLEMENT_RNG | SD_FLAG_GLOBAL_KERNELS | SD_FLAG_GENERAL_COMPARE))
        return fail(SD_EINVAL, "%s: unknown flags", name);
    if (overlap(sigma, tau, lattice_bytes(L, layout)))
        return fail(SD_EINVAL, "%s: sigma and tau overlap", name);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int klay = (layout == SD_I8) ? ((kernel_layout(L, layout, sigma) == kLayI8Row &&
                                     kernel_layout(L, layout, tau) == kLayI8Row)
                                        ? kLayI8Row
                                        : kLayI8Any)
                                 : kernel_layout(L, layout, sigma);
    const RunChoice ch = run_choice(L, layout);
    const uint32_t n_rec = obs ? k_steps / obs_every : 0u;
    const uint32_t n_words = (uint32_t)(((uint64_t)L * (uint64_t)L) / 64u);
    const bool lds_size = n_words <= kSingleLdsMaxWords &&
                          (klay == kLayP64 || klay == kLayI8Row || (klay == kLayP32 && L % 64 == 0) || klay == kLayBits);
    // Small lattices draw ahead of the chain: runs of kAheadDraws word draws and
    // more, and lattices past 64 words, with the whole device drawing (k_ahead,
    // needs scratch, see ahead_steps), the others and those without scratch in one workgroup if
    // they have at most 64 words (k_small).  The six-class cross-check keeps the general kernels.
    const bool ahead_ok = ahead_lattice(L, layout, sigma, tau) &&
                          !(flags & (SD_FLAG_GLOBAL_KERNELS | SD_FLAG_GENERAL_COMPARE));
    if (ahead_ok && k_steps == 0)
        return SD_OK;
    if (ahead_ok && !no_alloc && ch.mode != 2 && ahead_steps(n_words, k_steps, n_rec != 0, lds_size) &&
        (!small_supported(L) || 2ull * k_steps * lattice_words((uint32_t)L) >= kAheadDraws)) {
        uint32_t T[1][6];
        threshold_table(J, q, T[0]);
        bool done = false;
        const hipError_t e = run_chains_ahead(&sigma, &tau, 1, L, layout, T, seed, &stream, step0, k_steps, obs,
                                              obs_every, flags, st, &done);
        if (e != hipSuccess)
            return hip_fail(e, name);
        if (done)
            return SD_OK;
    }
    const int mode = !ahead_size(L) || (ahead_ok && !no_alloc && ch.mode == 2 && !capturing(st)) ? ch.mode : ch.mode_free;
    if (ahead_ok && mode != 2 && small_supported(L)) {
        g_last_route = SD_ROUTE_SMALL;
        const hipError_t e = launch_small_chain(sigma, tau, L, layout == SD_I8, J, q, seed, stream, step0, k_steps,
                                                k_steps >= obs_every ? obs : nullptr, obs_every, flags, st);
        return e == hipSuccess ? SD_OK : hip_fail(e, name);
    }
    // word width and grid of the choice are those of its half-step launches
    if (layout != SD_I8 && L % 64 == 0)
        klay = mode == 2 && ch.width == 32 ? kLayP32 : kLayP64;
    const uint32_t max_blocks = mode == 2 ? ch.blocks : 0u;
    if (lds_size && mode != 2 && !(flags & SD_FLAG_GLOBAL_KERNELS)) {
        if (k_steps == 0)
            return SD_OK;
        g_last_route = SD_ROUTE_LDS;
        hipError_t e = launch_single_chain_lds(sigma, tau, L, klay == kLayI8Row, J, q, seed, stream, step0, k_steps,
                                               n_rec ? obs : nullptr, obs_every, flags, ch.threads, st);
        return e == hipSuccess ? SD_OK : hip_fail(e, name);
    }
    const Geom G = make_geom(L, klay);
    hipError_t e = hipSuccess;
    int64_t* partials = nullptr;
    WorkspaceUse use;
    if (n_rec && no_alloc) {
        const sd_status ss = scratch_ptr(name, &partials);
        if (ss != SD_OK)
            return ss;
    } else if (n_rec) {
        use = WorkspaceUse(st);
        partials = use.get() ? use.get()->p : nullptr;
    }
    // Rows of whole words up to 4096^2: whole steps in bands of rows, several
    // per launch, as sd_run_many runs them (us per half-step, a launch each
    // against this: 512^2 3.8 -> 1.6, 1024^2 3.9 -> 1.7, 2048^2 4.0 -> 2.2,
    // 4096^2 5.9 -> 3.9).
    const bool whole_words = klay == kLayI8Row || (klay == kLayP64 && words_aligned(sigma, tau));
    if (mode != 2 && whole_words && k_steps >= 3 &&
        !(flags & (SD_FLAG_GLOBAL_KERNELS | SD_FLAG_GENERAL_COMPARE))) {
        uint32_t n_cu = 0;
        size_t max_lds = 0;
        e = device_limits(&n_cu, &max_lds);
        if (e == hipSuccess && band_plan(L, 1u, n_cu).bands) {
            ManyChains mc;
            std::memset(&mc, 0, sizeof mc);
            mc.sigma[0] = sigma;
            mc.tau[0] = tau;
            threshold_table(J, q, mc.T[0]);
            mc.stream[0] = stream;
            mc.n_chains = 1;
            mc.blocks_per_chain = many_blocks_per_chain(G);
            mc.obs_chain = 3ull * n_rec;
            e = run_many_grid(mc, G, klay, true, thresholds_paired(mc.T[0]), L, seed, step0, k_steps, obs, n_rec,
                              obs_every, flags, partials, st);
            return e == hipSuccess ? SD_OK : hip_fail(e, name);
        }
        if (e != hipSuccess)
            return hip_fail(e, name);
    }
    g_last_route = k_steps ? SD_ROUTE_HALF_STEPS : SD_ROUTE_NONE;
    // the table and keys once; only the time index changes from step to step
    const DrawParams base = dynamics_params(J, q, seed, stream, 0u, flags & SD_FLAG_COMPLEMENT_RNG);
    const bool general = (flags & SD_FLAG_GENERAL_COMPARE) != 0;
    // Each record's workgroup sums go to a slot of their own in the partials
    // workspace; one finishing launch adds a whole chunk of records, so that
    // frequent records cost no third launch per step.
    const uint32_t blocks = half_step_blocks(klay, G, !general && thresholds_paired(base.T), max_blocks);
    const uint32_t stride = 4u * blocks;
    if (n_rec && stride > kPartialsWords)
        return fail(SD_EINVAL, "%s: %u workgroups need %u partial sums per record, more than the %zu of the "
                    "scratch buffer", name, blocks, stride, kPartialsWords);
    const uint32_t chunk = (uint32_t)(kPartialsWords / stride);
    if (n_rec)
        e = launch_fill_i64(obs, (size_t)n_rec * 3u, 0, st);
    uint32_t pending = 0;   // records whose sums wait in the workspace
    for (uint32_t m = 0; m < k_steps && e == hipSuccess; ++m) {
        const uint64_t n = step0 + m;
        DrawParams dp = base;
        dp.t = (uint32_t)(2 * n);
        e = launch_half_step(klay, 0, sigma, tau, G, dp, nullptr, st, max_blocks, nullptr, general);
        if (e != hipSuccess)
            break;
        dp.t = (uint32_t)(2 * n + 1);
        if (n_rec && (m + 1) % obs_every == 0 && !partials) {
            // no workspace (stream capture): atomics into the record
            e = launch_half_step(klay, 1, tau, sigma, G, dp, obs + 3u * (size_t)((m + 1) / obs_every - 1), st,
                                 max_blocks, nullptr, general);
        } else if (n_rec && (m + 1) % obs_every == 0) {
            const uint32_t r = (m + 1) / obs_every - 1;
            e = launch_half_step(klay, 1, tau, sigma, G, dp, obs + 3u * (size_t)r, st, max_blocks,
                                 partials + (size_t)pending * stride, general, false);
            ++pending;
            if (e == hipSuccess && (pending == chunk || r + 1 == n_rec)) {
                e = launch_obs_finish(partials, blocks, pending, stride, obs + 3u * (size_t)(r + 1 - pending), st);
                pending = 0;
            }
        } else {
            e = launch_half_step(klay, 1, tau, sigma, G, dp, nullptr, st, max_blocks, nullptr, general);
        }
    }
    return e == hipSuccess ? SD_OK : hip_fail(e, name);
}

}  // namespace sd

using namespace sd;

extern "C" {

int32_t sd_abi_version(void) { return SD_ABI_VERSION; }

const char* sd_last_error(void) { return g_last_error.c_str(); }

size_t sd_lattice_bytes(int32_t L, int32_t layout) { return lattice_bytes(L, layout); }

sd_status sd_threshold_table(double J, double q, uint32_t out_host[6]) {
    if (!out_host)
        return fail(SD_EINVAL, "sd_threshold_table: null output");
    if (!std::isfinite(J) || !std::isfinite(q))
        return fail(SD_EINVAL, "sd_threshold_table: J and q must be finite");
    threshold_table(J, q, out_host);
    return SD_OK;
}

sd_status sd_init(void* lattice, int32_t L, int32_t layout, int32_t kind, double p_up, uint64_t seed,
                  uint32_t stream, void* hip_stream) {
    sd_status s = check_lattice(lattice, L, layout, "sd_init");
    if (s != SD_OK)
        return s;
    DrawParams dp;
    bool random = false, up = false;
    s = init_params("sd_init", kind, p_up, seed, stream, &dp, &random, &up);
    if (s != SD_OK)
        return s;
    const int klay = kernel_layout(L, layout, lattice);
    const hipError_t e = launch_init(klay, lattice, make_geom(L, klay), up ? 1 : 0, random, dp,
                                     static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SD_OK : hip_fail(e, "sd_init");
}

sd_status sd_half_step(const void* src, void* dst, int32_t L, int32_t layout, int32_t which, double J, double q,
                       uint64_t seed, uint32_t stream, uint32_t t, uint32_t flags, void* hip_stream) {
    sd_status s = check_lattice(src, L, layout, "sd_half_step(src)");
    if (s == SD_OK)
        s = check_lattice(dst, L, layout, "sd_half_step(dst)");
    if (s != SD_OK)
        return s;
    if (which != 0 && which != 1)
        return fail(SD_EINVAL, "sd_half_step: which must be 0 (A) or 1 (B)");
    if (!std::isfinite(J) || !std::isfinite(q))
        return fail(SD_EINVAL, "sd_half_step: J and q must be finite");
    if (t >= (1u << 30))
        return fail(SD_EINVAL, "sd_half_step: half-step index must be < 2^30");
    if (flags & ~(SD_FLAG_COMPLEMENT_RNG | SD_FLAG_GENERAL_COMPARE))
        return fail(SD_EINVAL, "sd_half_step: unknown flags");
    if (overlap(src, dst, lattice_bytes(L, layout)))
        return fail(SD_EINVAL, "sd_half_step: src and dst overlap");
    const int klay = (layout == SD_I8) ? ((kernel_layout(L, layout, src) == kLayI8Row &&
                                           kernel_layout(L, layout, dst) == kLayI8Row)
                                              ? kLayI8Row
                                              : kLayI8Any)
                                       : kernel_layout(L, layout, src);
    const Geom G = make_geom(L, klay);
    const DrawParams dp = dynamics_params(J, q, seed, stream, t, flags);
    hipError_t e = launch_half_step(klay, which, src, dst, G, dp, nullptr, static_cast<hipStream_t>(hip_stream), 0,
                                    nullptr, (flags & SD_FLAG_GENERAL_COMPARE) != 0);
    return e == hipSuccess ? SD_OK : hip_fail(e, "sd_half_step");
}

sd_status sd_run(void* sigma, void* tau, int32_t L, int32_t layout, double J, double q, uint64_t seed,
                 uint32_t stream, uint64_t step0, uint32_t k_steps, int64_t* obs, uint32_t obs_every,
                 uint32_t flags, void* hip_stream) {
    return run_chain("sd_run", sigma, tau, L, layout, J, q, seed, stream, step0, k_steps, obs, obs_every, flags,
                     hip_stream, false);
}

sd_status sd_run_noalloc(void* sigma, void* tau, int32_t L, int32_t layout, double J, double q, uint64_t seed,
                         uint32_t stream, uint64_t step0, uint32_t k_steps, int64_t* obs, uint32_t obs_every,
                         uint32_t flags, void* hip_stream) {
    return run_chain("sd_run_noalloc", sigma, tau, L, layout, J, q, seed, stream, step0, k_steps, obs, obs_every,
                     flags, hip_stream, true);
}

sd_status sd_run_many(void* const* sigma, void* const* tau, int32_t n_chains, int32_t L, int32_t layout,
                      const double* J, const double* q, uint64_t seed, const uint32_t* streams, uint64_t step0,
                      uint32_t k_steps, int64_t* obs, uint32_t obs_every, uint32_t flags, void* hip_stream) {
    const char* name = "sd_run_many";
    g_last_route = SD_ROUTE_NONE;
    if (n_chains < 1 || n_chains > (int32_t)kManyMax)
        return fail(SD_EINVAL, "%s: n_chains must lie in [1, %u]", name, kManyMax);
    if (!sigma || !tau || !J || !q || !streams)
        return fail(SD_EINVAL, "%s: null host array", name);
    const size_t bytes = lattice_bytes(L, layout);
    for (int32_t a = 0; a < n_chains; ++a) {
        sd_status s = check_lattice(sigma[a], L, layout, name);
        if (s == SD_OK)
            s = check_lattice(tau[a], L, layout, name);
        if (s != SD_OK)
            return s;
        if (!std::isfinite(J[a]) || !std::isfinite(q[a]))
            return fail(SD_EINVAL, "%s: J and q of chain %d must be finite", name, a);
    }
    // no two of the 2 n lattices may overlap
    for (int32_t a = 0; a < 2 * n_chains; ++a)
        for (int32_t b = a + 1; b < 2 * n_chains; ++b) {
            const void* x = a < n_chains ? sigma[a] : tau[a - n_chains];
            const void* y = b < n_chains ? sigma[b] : tau[b - n_chains];
            if (overlap(x, y, bytes))
                return fail(SD_EINVAL, "%s: lattices %d and %d overlap", name, a, b);
        }
    if (step0 + (uint64_t)k_steps > (1ull << 29))
        return fail(SD_EINVAL, "%s: step indices must stay below 2^29", name);
    if (obs && obs_every == 0)
        return fail(SD_EINVAL, "%s: obs given without obs_every", name);
    if (flags & ~(SD_FLAG_COMPLEMENT_RNG | SD_FLAG_GENERAL_COMPARE))
        return fail(SD_EINVAL, "%s: unknown flags", name);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int klay;
    if (layout == SD_I8) {
        bool row = L % 64 == 0;
        for (int32_t a = 0; a < n_chains; ++a)
            row = row && kernel_layout(L, layout, sigma[a]) == kLayI8Row && kernel_layout(L, layout, tau[a]) == kLayI8Row;
        klay = row ? kLayI8Row : kLayI8Any;
    } else {
        klay = kernel_layout(L, layout, sigma[0]);
    }
    const Geom G = make_geom(L, klay);
    ManyChains mc;
    std::memset(&mc, 0, sizeof mc);
    bool paired = (flags & SD_FLAG_GENERAL_COMPARE) == 0;
    for (int32_t a = 0; a < n_chains; ++a) {
        mc.sigma[a] = sigma[a];
        mc.tau[a] = tau[a];
        threshold_table(J[a], q[a], mc.T[a]);
        mc.stream[a] = streams[a];
        paired = paired && thresholds_paired(mc.T[a]);
    }
    mc.n_chains = (uint32_t)n_chains;
    mc.blocks_per_chain = many_blocks_per_chain(G);
    const uint32_t n_rec = obs ? k_steps / obs_every : 0u;
    mc.obs_chain = 3ull * n_rec;
    const uint32_t stride = 4u * mc.blocks_per_chain * mc.n_chains;   // partial sums of one record
    if (n_rec && stride > kPartialsWords)
        return fail(SD_EINVAL, "%s: %u chains of %u workgroups need more partial sums per record than the %zu of "
                    "the scratch buffer", name, mc.n_chains, mc.blocks_per_chain, kPartialsWords);
    if (k_steps == 0)
        return SD_OK;
    const bool whole_words = (layout == SD_P64 && L % 64 == 0) || klay == kLayI8Row;
    const uint32_t n_words = (uint32_t)(((uint64_t)L * (uint64_t)L) / 64u);
    bool ahead = !(flags & SD_FLAG_GENERAL_COMPARE) && ahead_steps(n_words, k_steps, n_rec != 0, false);
    // Past one word a thread of the walker, nine chains and more leave the scratch
    // to rounds of ten half-steps and fewer; whole steps in bands, where rows are
    // whole words (320^2), are quicker in runs of ten steps and more (100 steps,
    // recorded, drawn ahead against bands: 8 chains 354 and 354 us, 9 364 and 356,
    // 16 523 and 375; 5 steps of 16 44 and 47).  Rows of other lengths have no
    // bands, and one word a thread walks faster (256^2: ahead at every count).
    if (whole_words && n_words > 1024u && n_chains > 8 && k_steps >= 10u)
        ahead = false;
    for (int32_t c = 0; c < n_chains; ++c)
        ahead = ahead && ahead_lattice(L, layout, sigma[c], tau[c]);
    if (ahead) {
        bool done = false;
        const hipError_t ea = run_chains_ahead(sigma, tau, mc.n_chains, L, layout, mc.T, seed, streams, step0, k_steps,
                                               obs, obs_every, flags, st, &done);
        if (ea != hipSuccess)
            return hip_fail(ea, name);
        if (done)
            return SD_OK;
    }
    int64_t* partials = nullptr;
    WorkspaceUse use;
    if (n_rec) {
        use = WorkspaceUse(st);
        if (!use.get() && !(capturing(st) && stream_workspace(st, false)))
            return fail(SD_EHIP, "%s: no partial-sum buffer for this stream (stream capture before the first "
                        "eager call on it, or out of device memory)", name);
        partials = use.get() ? use.get()->p : nullptr;   // null: a captured run takes atomics
    }
    const hipError_t e = run_many_grid(mc, G, klay, whole_words, paired, L, seed, step0, k_steps, obs, n_rec, obs_every,
                                       flags, partials, st);
    return e == hipSuccess ? SD_OK : hip_fail(e, name);
}

sd_status sd_observe(const void* sigma, const void* tau, int32_t L, int32_t layout, int64_t* out3,
                     void* hip_stream) {
    sd_status s = check_lattice(sigma, L, layout, "sd_observe(sigma)");
    if (s == SD_OK)
        s = check_lattice(tau, L, layout, "sd_observe(tau)");
    if (s != SD_OK)
        return s;
    if (!out3)
        return fail(SD_EINVAL, "sd_observe: null output");
    const int klay = layout == SD_I8 ? kLayI8Any : packed_rows_layout(L);
    hipError_t e = launch_observe(klay, sigma, tau, make_geom(L, klay), out3, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SD_OK : hip_fail(e, "sd_observe");
}

sd_status sd_corr_row(const void* sigma, int32_t L, int32_t layout, int32_t rmax, int64_t* out,
                      void* hip_stream) {
    sd_status s = check_lattice(sigma, L, layout, "sd_corr_row");
    if (s != SD_OK)
        return s;
    if (!out)
        return fail(SD_EINVAL, "sd_corr_row: null output");
    if (rmax < 0 || rmax >= L)
        return fail(SD_EINVAL, "sd_corr_row: rmax must satisfy 0 <= rmax < L");
    // rows of whole 64-bit words where the layout has them
    int klay = kernel_layout(L, layout, sigma);
    if (klay != kLayP64 && klay != kLayI8Row)
        klay = layout == SD_I8 ? kLayI8Any : packed_rows_layout(L);
    hipError_t e = launch_corr_row(klay, sigma, make_geom(L, klay), rmax, out, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SD_OK : hip_fail(e, "sd_corr_row");
}

sd_status sd_corr_row_many(const void* const* sigma, int32_t n, int32_t L, int32_t layout, int32_t rmax,
                           int64_t* out, void* hip_stream) {
    const char* name = "sd_corr_row_many";
    if (n < 1 || n > (int32_t)kManyMax)
        return fail(SD_EINVAL, "%s: n must lie in [1, %u]", name, kManyMax);
    if (!sigma)
        return fail(SD_EINVAL, "%s: null host array", name);
    for (int32_t a = 0; a < n; ++a) {
        sd_status s = check_lattice(sigma[a], L, layout, name);
        if (s != SD_OK)
            return s;
    }
    if (!out)
        return fail(SD_EINVAL, "%s: null output", name);
    if (rmax < 0 || rmax >= L)
        return fail(SD_EINVAL, "%s: rmax must satisfy 0 <= rmax < L", name);
    // rows of whole 64-bit words when every lattice has them (int8 rows need
    // 16-byte aligned lattices)
    int klay = kernel_layout(L, layout, sigma[0]);
    for (int32_t a = 1; a < n; ++a)
        if (kernel_layout(L, layout, sigma[a]) != klay)
            klay = -1;
    if (klay != kLayP64 && klay != kLayI8Row)
        klay = layout == SD_I8 ? kLayI8Any : packed_rows_layout(L);
    hipError_t e = launch_corr_row_many(klay, sigma, (uint32_t)n, make_geom(L, klay), rmax, out,
                                        static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SD_OK : hip_fail(e, name);
}

sd_status sd_corr_diag(const void* sigma, int32_t L, int32_t layout, int32_t lmax, int64_t* out,
                       void* hip_stream) {
    sd_status s = check_lattice(sigma, L, layout, "sd_corr_diag");
    if (s != SD_OK)
        return s;
    if (!out)
        return fail(SD_EINVAL, "sd_corr_diag: null output");
    if (lmax < 0 || lmax >= L)
        return fail(SD_EINVAL, "sd_corr_diag: lmax must satisfy 0 <= lmax < L");
    const int klay = layout == SD_I8 ? kLayI8Any : packed_rows_layout(L);
    hipError_t e = launch_corr_diag(klay, sigma, make_geom(L, klay), lmax, out, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? SD_OK : hip_fail(e, "sd_corr_diag");
}

sd_status sd_tune(int32_t L, int32_t layout, const char* tune_cache_path, void* hip_stream) {
    if (!layout_supported(L, layout))
        return fail(SD_EINVAL, "sd_tune: unsupported (L=%d, layout=%d)", L, layout);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_fail(e, "sd_tune");
    // run2: the second set of kernels.  A choice made among others is no choice
    // among these: a mode 2 entry from before the runs of several half-steps a
    // launch would keep them off, with workgroups counted for wider tiles (2048^2: 64
    // where the rule wants 256).  Raised whenever candidates or tiles change.
    const std::string key = "run2:" + device_arch() + ":L=" + std::to_string(L) + ":layout=" + std::to_string(layout);
    auto encode = [](const RunChoice& c) -> long {
        return (long)c.mode | ((long)(c.width == 32) << 2) | ((long)c.blocks << 3) | ((long)(c.threads / 64) << 24) |
               ((long)c.mode_free << 32);
    };
    auto decode = [](long v) {
        RunChoice c;
        c.mode = (int)(v & 3);
        c.width = (v >> 2) & 1 ? 32 : 64;
        c.blocks = (uint32_t)((v >> 3) & 0x1FFFFF);
        c.threads = (uint32_t)(((v >> 24) & 0xFF) * 64);
        if (c.threads == 0)
            c.threads = 256;
        c.mode_free = (int)((v >> 32) & 3);
        return c;
    };
    const long cached = tune_cache_get(tune_cache_path, key);
    if (cached > 0) {
        std::lock_guard<std::mutex> lock(g_tune_mutex);
        g_run_choice[std::make_tuple(dev, L, layout)] = decode(cached);
        return SD_OK;
    }
    // candidates
    std::vector<RunChoice> cands;
    const uint32_t n_words = (uint32_t)(((uint64_t)L * (uint64_t)L) / 64u);
    uint32_t n_cu = 0;
    size_t max_lds = 0;
    e = device_limits(&n_cu, &max_lds);
    if (e != hipSuccess)
        return hip_fail(e, "sd_tune");
    if (ahead_size(L) || band_plan(L, 1u, n_cu).bands) {   // several half-steps a launch, as the built-in rule runs them
        RunChoice c;
        c.mode = 1;
        cands.push_back(c);
    }
    // the same without scratch, where that is another route: workgroups of the
    // LDS kernel, or k_small and the bands, which have no choice
    const size_t first_free = cands.size();
    if (ahead_size(L)) {
        const bool lds = !small_supported(L) && n_words <= kSingleLdsMaxWords && L % 8 == 0 &&
                         (layout == SD_I8 ? L % 64 == 0 : layout == SD_P64 || L % 64 == 0);
        for (uint32_t t : {128u, 256u, 512u}) {
            if (!lds && (t != 256u || !(small_supported(L) || band_plan(L, 1u, n_cu).bands)))
                continue;
            RunChoice c;
            c.mode_free = 1;
            c.threads = t;
            cands.push_back(c);
        }
    }
    const size_t first_grid = cands.size();
    for (int width : {64, 32}) {
        if (width == 32 && (layout == SD_I8 || L % 64 != 0))
            continue;
        // only grids that differ: a cap above one workgroup per four tiles
        // launches the same grid as the uncapped one
        int klay = kernel_layout(L, layout, nullptr);
        if (layout != SD_I8 && L % 64 == 0)
            klay = width == 32 ? kLayP32 : kLayP64;
        if (layout == SD_I8)
            klay = L % 64 == 0 ? kLayI8Row : kLayI8Any;
        const Geom G = make_geom(L, klay);
        uint32_t last = 0;
        for (uint32_t b : {256u, 512u, 1024u, 2048u, 4096u, 8192u}) {
            const uint32_t launched = half_step_blocks(klay, G, true, b);
            if (launched == last)
                continue;
            last = launched;
            RunChoice c;
            c.mode = c.mode_free = 2;
            c.width = width;
            c.blocks = launched;
            cands.push_back(c);
        }
    }
    // scratch lattices, a short run per candidate
    const size_t bytes = lattice_bytes(L, layout);
    void* sig = nullptr;
    void* tau = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    e = hipMalloc(&sig, bytes);
    if (e == hipSuccess) e = hipMalloc(&tau, bytes);
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    sd_status s = SD_OK;
    if (e == hipSuccess)
        s = sd_init(sig, L, layout, SD_INIT_RANDOM, 0.5, 1, 0, hip_stream);
    // Every candidate is timed in each of kPasses round-robin passes and keeps
    // its fastest time, so that clock ramp-up at the start of the tuning and
    // one-off stalls do not decide the choice; each timing covers at least a
    // millisecond of work on large lattices.
    const uint32_t k = n_words >= (1u << 20) ? 16u : (n_words >= 4096u ? 16u : 64u);
    constexpr int kPasses = 3;
    std::vector<float> fastest(cands.size(), -1.0f);
    for (int pass = 0; pass < kPasses; ++pass) {
        for (size_t ci = 0; ci < cands.size(); ++ci) {
            if (e != hipSuccess || s != SD_OK)
                break;
            {
                std::lock_guard<std::mutex> lock(g_tune_mutex);
                g_run_choice[std::make_tuple(dev, L, layout)] = cands[ci];
            }
            float ms = -1.0f;
            e = hipEventRecord(e0, st);
            if (e != hipSuccess) break;
            s = run_chain("sd_tune", sig, tau, L, layout, 0.5, 0.5, 1, 0, 0, k, nullptr, 0, 0, hip_stream,
                          ci >= first_free && ci < first_grid);
            if (s != SD_OK) break;
            e = hipEventRecord(e1, st);
            if (e == hipSuccess) e = hipEventSynchronize(e1);
            if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
            if (e != hipSuccess) break;
            if (pass > 0 && ms > 0.0f && (fastest[ci] < 0.0f || ms < fastest[ci]))   // pass 0 warms up
                fastest[ci] = ms;
        }
    }
    // the fastest of cands[from .. to) and the fastest grid; -1: none was timed
    auto fastest_of = [&](size_t from, size_t to) {
        int at = -1;
        for (size_t ci = 0; ci < cands.size(); ++ci)
            if (((ci >= from && ci < to) || ci >= first_grid) && fastest[ci] > 0.0f &&
                (at < 0 || fastest[ci] < fastest[(size_t)at]))
                at = (int)ci;
        return at;
    };
    RunChoice best;
    const int with = fastest_of(0, first_free), without = fastest_of(first_free, first_grid);
    const double best_t = with < 0 ? -1.0 : (double)fastest[(size_t)with];
    if (with >= 0) {
        best = cands[(size_t)with];
        const RunChoice& f = cands[(size_t)(without < 0 ? with : without)];
        best.mode_free = f.mode_free;
        best.threads = f.threads;
        if (f.mode_free == 2) {   // the fastest grid, which mode 2 of either kind takes
            best.width = f.width;
            best.blocks = f.blocks;
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (sig) (void)hipFree(sig);
    if (tau) (void)hipFree(tau);
    {
        std::lock_guard<std::mutex> lock(g_tune_mutex);
        if (best_t > 0.0)
            g_run_choice[std::make_tuple(dev, L, layout)] = best;
        else
            g_run_choice.erase(std::make_tuple(dev, L, layout));
    }
    if (e != hipSuccess)
        return hip_fail(e, "sd_tune");
    if (s != SD_OK)
        return s;
    if (best_t > 0.0)
        tune_cache_put(tune_cache_path, key, encode(best));
    return SD_OK;
}

sd_status sd_tuned_choice(int32_t L, int32_t layout, int32_t* mode, int32_t* width, int32_t* blocks,
                          int32_t* threads) {
    if (!layout_supported(L, layout))
        return fail(SD_EINVAL, "sd_tuned_choice: unsupported (L=%d, layout=%d)", L, layout);
    RunChoice c = run_choice(L, layout);
    if (c.mode != 2) {   // the built-in grid
        c.width = 64;
        c.blocks = 0;
    }
    if (mode) *mode = c.mode;
    if (width) *width = c.width;
    if (blocks) {
        // the grid sd_run launches per half-step when it takes the grid kernels
        // (paired compare, the form every threshold table takes)
        int klay = layout == SD_I8 ? (L % 64 == 0 ? kLayI8Row : kLayI8Any) : kernel_layout(L, layout, nullptr);
        if (layout != SD_I8 && L % 64 == 0)
            klay = c.width == 32 ? kLayP32 : kLayP64;
        *blocks = (int32_t)half_step_blocks(klay, make_geom(L, klay), true, c.blocks);
    }
    if (threads) *threads = (int32_t)c.threads;
    return SD_OK;
}

int32_t sd_debug_last_route(void) { return g_last_route; }

uint32_t sd_debug_fastdiv(uint32_t n, uint32_t d) {
    if (d == 0)
        return 0;
    return fdiv_host(n, make_fastdiv(d));
}

}  // extern "C"
