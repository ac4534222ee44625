// Chains of lattices of up to 2048 words, drawn ahead by the whole device.
//
// A half-step (eqs. (15)-(16)) compares every site's uniform with one of six
// thresholds, and the uniform depends only on (seed, stream, half-step, site).
// So whether r_s < T[k] can be computed for every class k before the lattice
// is known: six bits per site, a class mask.  One chain of a small lattice
// leaves the device idle and waits, half-step after half-step, for the draw of
// the last one (and, in the grid kernels, for a launch); here the other CUs
// draw the masks of the next round of half-steps into global memory while one
// workgroup per chain ("walker") takes the lattice through the current round:
// per half-step it fetches the neighbour words from LDS, picks each site's bit
// among the six masks, which it has loaded several half-steps ahead, writes
// the new word to LDS and meets at one barrier.  Records are taken from the
// new words by other workgroups of the next launch.  What bounds a half-step
// is that chain of LDS reads, about 40 instructions and the barrier, and from
// 1000 words on the 48 bytes of masks per word that one CU must read (256^2:
// 49 KB a half-step, 0.32 us at 64 bytes a clock).  us per half-step, the
// best other kernel against this one: 64^2 0.37 -> 0.07, 128^2 3.4 -> 0.18,
// 200^2 4.2 -> 0.53, 256^2 3.7 -> 0.46, 333^2 int8 6.9 -> 1.25 (recorded 0.69,
// 0.62 and 1.40); five chains of 256^2 in whole steps 1.5 -> 0.8.
//
// No workgroup of a launch waits for another: rounds are separate launches on
// the stream, and each slot of masks or words is written in one launch and
// read in the next.
#include <cstring>

#include "sd_ahead.hpp"
#include "sd_class.hpp"

namespace sd {

namespace {

// ---------------------------------------------------------------------------
// Drawing
// ---------------------------------------------------------------------------
struct DrawScratch {
    ClassList list;
    uint64_t mask[6][64];
};

// The class masks of the launch's round: tiles of 64 (half-step, word) pairs
// of one chain, one per wavefront.
__device__ __forceinline__ void ahead_draw(const AheadArgs& a, DrawScratch& w, uint32_t wave_id, uint32_t n_waves) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t per_chain = (a.draw_count * a.n + 63u) / 64u;
    for (uint32_t task = wave_id; task < per_chain * a.n_chains; task += n_waves) {
        const uint32_t chain = task / per_chain;
        const uint32_t x = 64u * (task - chain * per_chain) + lane;
        const bool active = x < a.draw_count * a.n;
        const uint32_t hs = active ? fdiv(x, a.div_n) : 0u;
        const uint32_t g = active ? x - hs * a.n : 0u;
        const uint32_t t = a.draw_t + hs;
        const uint32_t* T = a.T[chain];
        class_masks<false>(a.key0, a.key1, a.stream[chain], t, g, a.rng_xor, T, active, w.list, &w.mask[0][lane], 64u,
                           [&](uint32_t l, uint32_t& tt, uint32_t& gg, uint64_t*& m) __attribute__((always_inline)) {
                               const uint32_t y = x - lane + l;
                               const uint32_t h = fdiv(y, a.div_n);
                               tt = a.draw_t + h;
                               gg = y - h * a.n;
                               m = &w.mask[0][l];
                           });
        class_sync();
        if (active) {
            ulonglong2* out = reinterpret_cast<ulonglong2*>(
                a.masks + ((size_t)(a.draw_slot * a.n_chains + chain) * a.H + hs) * 6u * a.n) + g;
#pragma unroll
            for (uint32_t k = 0; k < 3; ++k)
                out[(size_t)k * a.n] = make_ulonglong2(w.mask[2 * k][lane], w.mask[2 * k + 1][lane]);
        }
        class_sync();
    }
}

// ---------------------------------------------------------------------------
// Walking
// ---------------------------------------------------------------------------
// How a word's neighbours are found: from other lanes' registers (rows of 64
// or 32 sites), as whole words of the lattice in LDS (rows of whole words), or
// as windows of its bit string (any L).
constexpr int kFormRow64 = 64, kFormRow32 = 32, kFormWords = 1, kFormString = 0;

// 64 sites from position pos of the lattice's bit string (indices mod N), the
// string in LDS with a zero word after its last one and zeros past site N - 1:
// two funnel shifts of three 32-bit words, and where the window passes the
// end, the string's first sites from bit `room` on.
struct Span {
    uint32_t q, sh, room;
};

__device__ __forceinline__ Span make_span(uint32_t pos, uint32_t N) {
    const uint32_t room = N - pos;
    return {pos >> 5, pos & 31u, room < 64u ? room : 64u};
}

__device__ __forceinline__ uint64_t pack64(uint32_t lo, uint32_t hi) { return (uint64_t)lo | ((uint64_t)hi << 32); }

__device__ __forceinline__ uint64_t span_bits(const uint64_t* lat, const Span& s) {
    const lds_dword* d = reinterpret_cast<const lds_dword*>(lat) + s.q;
    const uint32_t d0 = d[0], d1 = d[1], d2 = d[2];
    uint64_t v = pack64(__builtin_amdgcn_alignbit(d1, d0, s.sh), __builtin_amdgcn_alignbit(d2, d1, s.sh));
    if (s.room < 64u)
        v |= lat[0] << s.room;
    return v;
}

// Neighbour fetches of one word for one direction.
struct Fetch {
    Span row;         // the row below (above); row.q is the word's index for rows of whole words
    uint32_t side;    // 32-bit word before (after) the word's own two
    Span across;      // the row's other end, for the sites of `wrap`
    uint64_t wrap;
};

template <int FORM, int WHICH>
__device__ __forceinline__ Fetch make_fetch(const AheadArgs& a, uint32_t g) {
    const uint32_t s0 = 64u * g, L = a.L, N = a.N;
    Fetch f;
    if constexpr (FORM == kFormWords) {
        const uint32_t W = L / 64u, n = a.n;
        const uint32_t w = g - fdiv(s0, a.div_L) * W;
        f.row.q = WHICH == 0 ? (g >= W ? g - W : g + n - W) : (g + W < n ? g + W : g + W - n);
        f.side = WHICH == 0 ? 2u * (w == 0 ? g + W - 1u : g - 1u) + 1u : 2u * (w == W - 1u ? g + 1u - W : g + 1u);
        return f;
    }
    f.wrap = column_mask(g, L, a.div_L, WHICH == 0 ? 0u : L - 1u);
    if constexpr (WHICH == 0) {
        f.row = make_span(s0 >= L ? s0 - L : s0 + N - L, N);
        f.side = g == 0 ? 0u : 2u * g - 1u;
        f.across = make_span(s0 + L - 1u < N ? s0 + L - 1u : s0 + L - 1u - N, N);
    } else {
        f.row = make_span(s0 + L < N ? s0 + L : s0 + L - N, N);
        f.side = 2u * g + 2u;
        f.across = make_span(s0 + 1u >= L ? s0 + 1u - L : s0 + N + 1u - L, N);
    }
    return f;
}

template <int FORM, int WHICH>
__device__ __forceinline__ void fetch_neighbours(uint64_t c, const uint64_t* lat, const Fetch& f, uint64_t& n1,
                                                 uint64_t& n2) {
    if constexpr (FORM == kFormRow64 || FORM == kFormRow32) {
        row_neighbours<FORM, WHICH>(c, n1, n2);
    } else {
        const uint32_t side = reinterpret_cast<const lds_dword*>(lat)[f.side];
        n1 = FORM == kFormWords ? lat[f.row.q] : span_bits(lat, f.row);
        const uint32_t lo = (uint32_t)c, hi = (uint32_t)(c >> 32);
        n2 = WHICH == 0 ? pack64(__builtin_amdgcn_alignbit(lo, side, 31), __builtin_amdgcn_alignbit(hi, lo, 31))
                        : pack64(__builtin_amdgcn_alignbit(hi, lo, 1), __builtin_amdgcn_alignbit(side, hi, 1));
        if (FORM == kFormString && f.wrap)
            n2 = (n2 & ~f.wrap) | (span_bits(lat, f.across) & f.wrap);
    }
}

// Meets the walker's wavefronts (one wavefront needs no barrier).
__device__ __forceinline__ void walk_sync(bool one_wave) {
    if (one_wave)
        class_sync();
    else
        __syncthreads();
}

// One chain through the round's walk_count half-steps (even, A first).  Thread
// t holds words t and (WPL 2) t + blockDim.x; the masks of the next DEPTH
// half-steps are in registers.
template <int FORM, int WPL, int DEPTH>
__device__ __forceinline__ void ahead_walk(const AheadArgs& a, uint32_t chain, uint64_t* smem) {
    static_assert(DEPTH % 2 == 0, "the parity of a half-step is that of its ring slot");
    constexpr bool kRegs = FORM == kFormRow64 || FORM == kFormRow32;   // no lattice in LDS
    const uint32_t n = FORM == kFormRow64 ? 64u : FORM == kFormRow32 ? 16u : a.n;
    const bool one_wave = kRegs || n <= 64u;
    if (one_wave && threadIdx.x >= 64u)
        return;
    uint64_t* lat_s = smem;              // sigma, n words and a zero
    uint64_t* lat_t = smem + n + 1u;     // tau
    const uint32_t stride = one_wave ? 64u : blockDim.x;
    uint64_t sig[WPL], tau[WPL], valid[WPL];
    uint32_t word[WPL];
    Fetch fA[WPL], fB[WPL];
    uint64_t* st_s = a.state + (size_t)chain * 2u * n;
#pragma unroll
    for (int w = 0; w < WPL; ++w) {
        const uint32_t g0 = threadIdx.x + stride * w;
        // threads without a word repeat word 0 (the row form of 32^2: its 16
        // words four times over, so that its row shifts stay within them);
        // they write the same values
        const uint32_t g = FORM == kFormRow32 ? g0 & 15u : g0 < n ? g0 : 0u;
        word[w] = g;
        const uint32_t nv = a.N - 64u * g < 64u ? a.N - 64u * g : 64u;
        valid[w] = nv == 64u ? ~0ull : (1ull << nv) - 1ull;
        if (!kRegs) {
            fA[w] = make_fetch<FORM, 0>(a, g);
            fB[w] = make_fetch<FORM, 1>(a, g);
        }
        if (!a.walk_first)
            sig[w] = st_s[g];
        else if (!a.int8_io)
            sig[w] = static_cast<const uint64_t*>(a.sigma[chain])[g];
        else if (nv == 64u)
            sig[w] = load_bits64_i8<false>(static_cast<const int8_t*>(a.sigma[chain]) + 64u * (size_t)g);
        else
            sig[w] = load_bits64_i8<false>(static_cast<const int8_t*>(a.sigma[chain]) + (a.N - 64u)) >> (64u - nv);
        tau[w] = 0;
        if (!kRegs)
            lat_s[g] = sig[w];
    }
    if (!kRegs && threadIdx.x == 0)
        lat_s[n] = lat_t[n] = 0;
    const uint64_t* masks = a.masks + (size_t)(a.walk_slot * a.n_chains + chain) * a.H * 6u * n;
    uint64_t* hist = a.hist ? a.hist + (size_t)(a.walk_slot * a.n_chains + chain) * a.H * n : nullptr;
    const uint32_t count = a.walk_count;
    ClassMasks ring[DEPTH][WPL];
    auto load = [&](uint32_t i, ClassMasks (&r)[WPL]) __attribute__((always_inline)) {
        // half-steps past the round's last one load that one again
        const uint64_t* p = masks + (size_t)(i < count ? i : count - 1u) * 6u * n;
#pragma unroll
        for (int w = 0; w < WPL; ++w) {
#pragma unroll
            for (uint32_t k = 0; k < 3; ++k) {   // two classes a load, consecutive lanes on consecutive 16 bytes
                const ulonglong2 v = reinterpret_cast<const ulonglong2*>(p + (size_t)2u * k * n)[word[w]];
                r[w].m[2 * k] = v.x;
                r[w].m[2 * k + 1] = v.y;
            }
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        load((uint32_t)d, ring[d]);
    if (!kRegs)
        walk_sync(one_wave);
    auto step = [&](uint32_t i, int d) __attribute__((always_inline)) {
        uint64_t n1, n2;
        if ((d & 1) == 0) {
#pragma unroll
            for (int w = 0; w < WPL; ++w) {
                fetch_neighbours<FORM, 0>(sig[w], lat_s, fA[w], n1, n2);
                tau[w] = pick_class(ring[d][w], sig[w], n1, n2) & (FORM == kFormString ? valid[w] : ~0ull);
                if (!kRegs)
                    lat_t[word[w]] = tau[w];
                if (hist)
                    hist[(size_t)i * n + word[w]] = tau[w];
            }
        } else {
#pragma unroll
            for (int w = 0; w < WPL; ++w) {
                fetch_neighbours<FORM, 1>(tau[w], lat_t, fB[w], n1, n2);
                sig[w] = pick_class(ring[d][w], tau[w], n1, n2) & (FORM == kFormString ? valid[w] : ~0ull);
                if (!kRegs)
                    lat_s[word[w]] = sig[w];
                if (hist)
                    hist[(size_t)i * n + word[w]] = sig[w];
            }
        }
        load(i + DEPTH, ring[d]);
        if (!kRegs)
            walk_sync(one_wave);
    };
    uint32_t i = 0;
    for (; i + DEPTH <= count; i += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            step(i + (uint32_t)d, d);
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (i + (uint32_t)d < count)
            step(i + (uint32_t)d, d);
#pragma unroll
    for (int w = 0; w < WPL; ++w) {
        const uint32_t g = threadIdx.x + stride * w;
        if (g >= n)
            continue;
        if (!a.walk_last) {
            st_s[g] = sig[w];
        } else if (!a.int8_io) {
            static_cast<uint64_t*>(a.sigma[chain])[g] = sig[w];
            static_cast<uint64_t*>(a.tau[chain])[g] = tau[w];
        } else {
            int8_t* ps = static_cast<int8_t*>(a.sigma[chain]) + 64u * (size_t)g;
            int8_t* pt = static_cast<int8_t*>(a.tau[chain]) + 64u * (size_t)g;
            if (valid[w] == ~0ull) {
                store_bits64_i8<false>(ps, sig[w]);
                store_bits64_i8<false>(pt, tau[w]);
            } else {
                for (uint32_t b = 0; 64u * g + b < a.N; ++b) {
                    ps[b] = ((sig[w] >> b) & 1u) ? 1 : -1;
                    pt[b] = ((tau[w] >> b) & 1u) ? 1 : -1;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Records
// ---------------------------------------------------------------------------
// Sites pos .. pos + 63 (mod N) of a packed lattice in memory.
__device__ __forceinline__ uint64_t memory_span(const uint64_t* lat, uint32_t n, uint32_t N, uint32_t pos) {
    const uint32_t q = pos >> 6, sh = pos & 63u, room = N - pos;
    uint64_t v = lat[q] >> sh;
    if (q + 1u < n)
        v |= (lat[q + 1u] << 1) << (63u - sh);
    if (room < 64u)
        v |= lat[0] << room;
    return v;
}

// M, A, B of the recorded steps of the round in hist, one step of one chain
// per wavefront (lattices of one word per lane) or per workgroup, so that the
// latency of a task's loads, which nothing hides, is paid about once.
__device__ __forceinline__ void ahead_records(const AheadArgs& a, uint32_t block, uint32_t n_blocks, uint32_t* sums) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const bool by_wave = a.n <= 64u;
    const uint32_t first = by_wave ? block * waves + wave : block, stride = by_wave ? n_blocks * waves : n_blocks;
    const uint32_t g0 = by_wave ? threadIdx.x & 63u : threadIdx.x, g_step = by_wave ? 64u : blockDim.x;
    const uint32_t steps = a.rec_count / 2u;
    for (uint32_t task = first; task < steps * a.n_chains; task += stride) {
        const uint32_t chain = task / steps;
        const uint32_t s = task - chain * steps;
        const uint32_t done = a.rec_step + s + 1u;
        if (done % a.obs_every != 0)
            continue;
        const uint64_t* tau = a.hist + ((size_t)(a.rec_slot * a.n_chains + chain) * a.H + 2u * s) * a.n;
        const uint64_t* sig = tau + a.n;
        uint32_t v[3] = {0, 0, 0};   // #+1, #differences to up and right, to the partner
        for (uint32_t g = g0; g < a.n; g += g_step) {
            const uint32_t s0 = 64u * g;
            const uint32_t nv = a.N - s0 < 64u ? a.N - s0 : 64u;
            const uint64_t valid = nv == 64u ? ~0ull : (1ull << nv) - 1ull;
            const uint64_t x = sig[g], t = tau[g];
            const uint64_t up = memory_span(tau, a.n, a.N, s0 + a.L < a.N ? s0 + a.L : s0 + a.L - a.N);
            uint64_t right = (t >> 1) | (g + 1u < a.n ? tau[g + 1u] << 63 : 0ull);
            const uint64_t last = column_mask(g, a.L, a.div_L, a.L - 1u);
            if (last)
                right = (right & ~last) |
                        (memory_span(tau, a.n, a.N, s0 + 1u >= a.L ? s0 + 1u - a.L : s0 + a.N + 1u - a.L) & last);
            v[0] += (uint32_t)__popcll(x);
            v[1] += (uint32_t)(__popcll((x ^ up) & valid) + __popcll((x ^ right) & valid));
            v[2] += (uint32_t)__popcll((x ^ t) & valid);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
            v[i] = wave_sum_dpp(v[i]);
        if (!by_wave) {
            if (threadIdx.x < 3u)
                sums[threadIdx.x] = 0u;
            __syncthreads();
            if ((threadIdx.x & 63u) == 0)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    atomicAdd(&sums[i], v[i]);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 3; ++i)
                v[i] = sums[i];
        }
        if (g0 == 0) {
            const int64_t sites = a.N;
            int64_t* o = a.obs + chain * a.obs_chain + 3u * (size_t)(done / a.obs_every - 1u);
            o[0] = 2 * (int64_t)v[0] - sites;
            o[1] = 2 * sites - 2 * (int64_t)v[1];
            o[2] = sites - 2 * (int64_t)v[2];
        }
        if (!by_wave)
            __syncthreads();
    }
}

// Workgroups 0 .. n_chains - 1 walk (when the launch walks), the next
// draw_blocks draw, the last rec_blocks take records.
template <int FORM, int WPL, int DEPTH, int THREADS>
__global__ __launch_bounds__(THREADS) void k_ahead(AheadArgs a) {
    extern __shared__ uint64_t smem[];
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t walkers = a.walk_count ? a.n_chains : 0u;
    if (blockIdx.x < walkers) {
        ahead_walk<FORM, WPL, DEPTH>(a, blockIdx.x, smem);
    } else if (blockIdx.x < walkers + a.draw_blocks) {
        ahead_draw(a, reinterpret_cast<DrawScratch*>(smem)[wave], (blockIdx.x - walkers) * waves + wave,
                   a.draw_blocks * waves);
    } else {
        ahead_records(a, blockIdx.x - walkers - a.draw_blocks, a.rec_blocks, reinterpret_cast<uint32_t*>(smem));
    }
}

template <int FORM, int WPL, int DEPTH, int THREADS>
hipError_t launch_ahead_t(const AheadArgs& a, hipStream_t st) {
    const uint32_t blocks = (a.walk_count ? a.n_chains : 0u) + a.draw_blocks + a.rec_blocks;
    const size_t lat = sizeof(uint64_t) * 2u * (a.n + 1u);   // also holds the records' sums
    const size_t draw = sizeof(DrawScratch) * (THREADS / 64);
    const size_t lds = lat > draw ? lat : draw;
    if (lds > 65536u) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ahead<FORM, WPL, DEPTH, THREADS>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL((k_ahead<FORM, WPL, DEPTH, THREADS>), dim3(blocks), dim3(THREADS), lds, st, a);
    return hipGetLastError();
}

// The walker's form: the half-steps whose masks are in flight cover the
// latency of global memory (about 1 us) at the form's own pace, within the
// registers of its workgroup.
hipError_t launch_ahead(const AheadArgs& a, hipStream_t st) {
    if (a.L == 64u)
        return launch_ahead_t<kFormRow64, 1, 16, 256>(a, st);
    if (a.L == 32u)
        return launch_ahead_t<kFormRow32, 1, 16, 256>(a, st);
    const bool words = a.L % 64u == 0;
    if (a.n <= 256u)
        return words ? launch_ahead_t<kFormWords, 1, 8, 256>(a, st) : launch_ahead_t<kFormString, 1, 8, 256>(a, st);
    if (a.n <= 512u)   // no side has rows of whole words here: 128^2 is 256 words, 192^2 576
        return launch_ahead_t<kFormString, 1, 8, 512>(a, st);
    if (a.n <= 1024u)
        return words ? launch_ahead_t<kFormWords, 1, 4, 1024>(a, st) : launch_ahead_t<kFormString, 1, 4, 1024>(a, st);
    return words ? launch_ahead_t<kFormWords, 2, 2, 1024>(a, st) : launch_ahead_t<kFormString, 2, 2, 1024>(a, st);
}

}  // namespace

hipError_t run_ahead(AheadArgs a, uint64_t step0, uint32_t k_steps, void* scratch, size_t bytes, hipStream_t st) {
    constexpr uint32_t kMaxRound = 512, kMaxDrawBlocks = 1024, kMaxRecBlocks = 512;
    a.N = a.L * a.L;
    a.n = (a.N + 63u) / 64u;
    a.div_n = make_fastdiv(a.n);
    a.div_L = make_fastdiv(a.L);
    const bool records = a.obs != nullptr;
    const uint32_t total = 2u * k_steps;
    // equal rounds, as long as the scratch allows
    const size_t per = sizeof(uint64_t) * a.n_chains * a.n;
    uint64_t most = (bytes / per - 2u) / (2u * (records ? 7u : 6u));
    most = most < kMaxRound ? most & ~1ull : kMaxRound;
    const uint32_t rounds = (uint32_t)((total + most - 1u) / most);
    uint32_t H = (total + rounds - 1u) / rounds;
    H += H & 1u;
    a.H = H;
    a.masks = static_cast<uint64_t*>(scratch);
    a.hist = records ? a.masks + (size_t)2 * a.n_chains * H * 6u * a.n : nullptr;
    a.state = a.masks + (size_t)2 * a.n_chains * H * (records ? 7u : 6u) * a.n;
    const uint32_t waves = a.n <= 256u ? 4u : a.n <= 512u ? 8u : 16u;
    const uint32_t launched = (total + H - 1u) / H;   // rounds that hold half-steps
    hipError_t e = hipSuccess;
    for (uint32_t r = 0; r < launched + (records ? 2u : 1u) && e == hipSuccess; ++r) {
        auto count_of = [&](uint32_t round) { return total - round * H < H ? total - round * H : H; };
        a.draw_count = r < launched ? count_of(r) : 0u;
        a.draw_t = (uint32_t)(2 * step0) + r * H;
        a.draw_slot = r & 1u;
        const uint32_t tiles = (a.draw_count * a.n + 63u) / 64u * a.n_chains;
        a.draw_blocks = (tiles + waves - 1u) / waves;
        a.draw_blocks = a.draw_blocks < kMaxDrawBlocks ? a.draw_blocks : kMaxDrawBlocks;
        const bool walk = r >= 1u && r <= launched;
        a.walk_count = walk ? count_of(r - 1u) : 0u;
        a.walk_slot = (r - 1u) & 1u;
        a.walk_first = r == 1u ? 1u : 0u;
        a.walk_last = r == launched ? 1u : 0u;
        const bool rec = records && r >= 2u;
        a.rec_count = rec ? count_of(r - 2u) : 0u;
        a.rec_step = rec ? (r - 2u) * (H / 2u) : 0u;
        a.rec_slot = r & 1u;
        const uint32_t rec_tasks = a.rec_count / 2u * a.n_chains;
        a.rec_blocks = a.n <= 64u ? (rec_tasks + waves - 1u) / waves : rec_tasks;
        a.rec_blocks = a.rec_blocks < kMaxRecBlocks ? a.rec_blocks : kMaxRecBlocks;
        e = launch_ahead(a, st);
    }
    return e;
}

}  // namespace sd
