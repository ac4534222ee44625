// Chains of small lattices (at most 64 words of 64 sites: L % 8 == 0, L <= 64),
// one workgroup per chain or per coupled pair of chains.
//
// A half-step (eqs. (15)-(16)) draws every site from one of six thresholds,
// picked by the site's class, and its uniform depends only on (seed, stream,
// half-step, site).  So the draws of all six classes can be made before the
// lattice is known: the class mask k of a half-step holds, per site, whether
// r_s < T[k].  Most wavefronts of the workgroup ("workers") compute the masks
// of the next H half-steps into LDS while one wavefront ("walker", one word
// per lane) takes the lattice through the current H: per half-step it only
// fetches the neighbours, picks each site's bit among six masks and writes the
// new word.  What such a chain waits for is the dependence of a half-step on
// the last one; drawing ahead leaves about 30 instructions in that chain
// instead of a whole draw (four plane calls, the scan, the tails, a workgroup
// barrier).  The walker takes 0.053 us a half-step at 32^2 and 0.062 at 64^2,
// whose rows are halves and wholes of a register; on other sides the neighbours
// are windows of the lattice in LDS, and it takes 0.155.  The workers bound 32^2
// and 64^2, 0.092 us and 0.37 (a whole draw per half-step took 1.2-1.5 us).  Long runs of one chain leave the drawing to the whole device
// (k_ahead.hip).
//
// Coupled pairs (coupling from the past, section 3.2) share their uniforms, so
// one set of masks serves two walkers.
#include "sd_class.hpp"
#include "sd_small.hpp"

namespace sd {

namespace {

// Words of a lattice: known at compile time for the row forms, so that mask and
// history addresses are immediates.
template <int ROWS>
__device__ __forceinline__ uint32_t small_words(const SmallArgs& a) {
    return ROWS == 64 ? 64u : ROWS == 32 ? 16u : a.n;
}

// Half-step of index x = (half-step, word) of an epoch.
template <int ROWS>
__device__ __forceinline__ uint32_t small_half(const SmallArgs& a, uint32_t x) {
    return ROWS == 64 ? x >> 6 : ROWS == 32 ? x >> 4 : fdiv(x, a.div_n);
}

// The class masks of half-steps t_first .. t_first + count - 1 into masks
// ([half-step][class][word]), by worker `me` of `workers`.
template <int ROWS>
__device__ __forceinline__ void small_draw(const SmallArgs& a, uint32_t stream, ClassList& w, uint32_t me,
                                           uint32_t workers, uint32_t t_first, uint32_t count, uint64_t* masks) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t nw = small_words<ROWS>(a);
    const uint32_t total = count * nw;
    for (uint32_t x0 = 64u * me; x0 < total; x0 += 64u * workers) {
        const uint32_t x = x0 + lane;
        const bool active = x < total;
        const uint32_t hs = active ? small_half<ROWS>(a, x) : 0u;
        const uint32_t g = active ? x - hs * nw : 0u;
        // a 64-word tile is one half-step of a 64^2 lattice: its index is uniform
        const uint32_t t = ROWS == 64 ? t_first + (x0 >> 6) : t_first + hs;
        class_masks<ROWS == 64>(a.key0, a.key1, stream, t, g, a.rng_xor, a.T, active, w, masks + (hs * 6u * nw + g),
                                nw, [&](uint32_t l, uint32_t& tt, uint32_t& gg, uint64_t*& m)
                                        __attribute__((always_inline)) {
                                            const uint32_t h = small_half<ROWS>(a, x0 + l);
                                            tt = t_first + h;
                                            gg = x0 + l - h * nw;
                                            m = masks + (h * 6u * nw + gg);
                                        });
    }
}

// A lane's neighbour fetches for one direction on lattices whose rows need not
// be 32 or 64 sites: windows of the lattice's bit string, all indices fixed.
struct Window {
    uint32_t q0, q1, sh;        // neighbour row: bits sh .. of word q0, then q1
    uint32_t w0, w1, wsh;       // row wrap of the shifted word
    uint32_t side;              // the word before (after) this one
    uint64_t wrap;              // sites whose neighbour is across the row's end
};

template <int WHICH>
__device__ __forceinline__ Window make_window(const SmallArgs& a, uint32_t g) {
    const uint32_t n = a.n, N = 64u * n, L = a.L;
    auto at = [&](uint32_t off, uint32_t& q0, uint32_t& q1, uint32_t& sh) {
        q0 = g + (off >> 6);
        q0 = q0 >= n ? q0 - n : q0;
        q1 = q0 + 1u == n ? 0u : q0 + 1u;
        sh = off & 63u;
    };
    Window w;
    if constexpr (WHICH == 0) {
        at(N - L, w.q0, w.q1, w.sh);
        at(L - 1u, w.w0, w.w1, w.wsh);
        w.side = g == 0 ? n - 1u : g - 1u;
        w.wrap = column_mask(g, L, a.div_L, 0u);
    } else {
        at(L, w.q0, w.q1, w.sh);
        at(N + 1u - L, w.w0, w.w1, w.wsh);
        w.side = g + 1u == n ? 0u : g + 1u;
        w.wrap = column_mask(g, L, a.div_L, L - 1u);
    }
    return w;
}

__device__ __forceinline__ uint64_t window_bits(uint64_t lo, uint64_t hi, uint32_t sh) {
    return (lo >> sh) | ((hi << 1) << (63u - sh));
}

// Neighbour words n1 (down / up) and n2 (left / right) of the word c of every
// lane, lane l holding word l.  ROWS 64: a row per lane; 32: two rows per
// lane, 16 lanes; 0: any, from the lattice in LDS (lat).
template <int ROWS, int WHICH>
__device__ __forceinline__ void small_neighbours(uint64_t c, const uint64_t* lat, const Window& w, uint64_t& n1,
                                                 uint64_t& n2) {
    if constexpr (ROWS != 0) {
        row_neighbours<ROWS, WHICH>(c, n1, n2);
    } else {
        const uint64_t side = lat[w.side];
        n1 = window_bits(lat[w.q0], lat[w.q1], w.sh);
        const uint64_t across = window_bits(lat[w.w0], lat[w.w1], w.wsh);
        const uint64_t base = WHICH == 0 ? (c << 1) | (side >> 63) : (c >> 1) | (side << 63);
        n2 = (base & ~w.wrap) | (across & w.wrap);
    }
}

template <int ROWS>
__device__ __forceinline__ ClassMasks load_masks(const uint64_t* p, const SmallArgs& a) {
    const uint32_t nw = small_words<ROWS>(a);
    ClassMasks r;
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k)
        r.m[k] = p[k * nw];
    return r;
}

// Half-steps 0 .. count - 1 of an epoch (A first, count even) on the walker's
// words, which update sig and tau.  KEEP: every new word goes to
// hist[half-step][word], from which the records are taken, and the lattice
// before the epoch lies in front of hist; otherwise hist is a two-slot buffer
// (tau, sigma) that only the window form reads.  The masks of a half-step are
// loaded one half-step ahead (the loads past the epoch's last one read other
// parts of the workgroup's LDS and are not used).
template <int ROWS, bool KEEP>
__device__ __forceinline__ void small_walk(const SmallArgs& a, uint32_t count, const uint64_t* masks, uint64_t* hist,
                                           uint32_t slot, const Window& wA, const Window& wB, uint64_t& sig,
                                           uint64_t& tau) {
    const uint32_t nw = small_words<ROWS>(a);
    const uint64_t* p = masks + slot;
    uint64_t* h = hist + slot;
    const uint64_t* before = KEEP ? hist - nw : hist + 64;   // sigma for the window form
    ClassMasks ma = load_masks<ROWS>(p, a);
    for (uint32_t i = 0; i < count; i += 2) {
        uint64_t n1, n2;
        const ClassMasks mb = load_masks<ROWS>(p + 6u * nw, a);
        small_neighbours<ROWS, 0>(sig, before, wA, n1, n2);
        tau = pick_class(ma, sig, n1, n2);
        if (KEEP || ROWS == 0)
            h[0] = tau;
        if (ROWS == 0)
            class_sync();
        p += 12u * nw;
        ma = load_masks<ROWS>(p, a);
        small_neighbours<ROWS, 1>(tau, KEEP ? h - slot : hist, wB, n1, n2);
        sig = pick_class(mb, tau, n1, n2);
        if (KEEP)
            h[nw] = sig;
        else if (ROWS == 0)
            h[64] = sig;
        if (ROWS == 0)
            class_sync();
        if (KEEP) {
            before = h - slot + nw;
            h += 2u * nw;
        }
    }
}

// M, A, B of the steps of an epoch (first step index m0 of the run, `count`
// half-steps in hist) that are recorded, by worker `me` of `workers`.
__device__ __forceinline__ void small_records(const SmallArgs& a, uint32_t me, uint32_t workers, uint32_t m0,
                                              uint32_t count, const uint64_t* hist) {
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t s = me; 2u * s < count; s += workers) {
        const uint32_t m = m0 + s + 1u;   // steps done after it
        if (m % a.obs_every != 0)
            continue;
        uint32_t pc = 0, dpair = 0, dself = 0;
        if (lane < a.n) {
            const uint64_t* tau = hist + (size_t)(2u * s) * a.n;
            const uint64_t x = tau[a.n + lane];
            uint64_t t, up, right;
            gather_bits<1>(tau, a.L, a.n, a.div_L, lane, t, up, right);
            pc = (uint32_t)__popcll(x);
            dpair = (uint32_t)(__popcll(x ^ up) + __popcll(x ^ right));
            dself = (uint32_t)__popcll(x ^ t);
        }
        const uint32_t v0 = wave_sum_dpp(pc), v1 = wave_sum_dpp(dpair), v2 = wave_sum_dpp(dself);
        if (lane == 0) {
            const int64_t sites = 64 * (int64_t)a.n;
            int64_t* o = a.obs + 3u * (size_t)(m / a.obs_every - 1u);
            o[0] = 2 * (int64_t)v0 - sites;
            o[1] = 2 * sites - 2 * (int64_t)v1;
            o[2] = sites - 2 * (int64_t)v2;
        }
    }
}

// PAIR: workgroup b is coupled pair a.pairs[b] (top chain from all +1 on
// wavefront 0, bottom chain from all -1 on wavefront 1); else the one chain
// (a.sigma, a.tau) on wavefront 0.  Every other wavefront is a worker.
template <int ROWS, bool PAIR>
__global__ __launch_bounds__(1024) void k_small(SmallArgs a) {
    extern __shared__ uint64_t smem[];
    constexpr uint32_t kWalkers = PAIR ? 2u : 1u;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t n = small_words<ROWS>(a), H = a.H;
    const uint32_t workers = (blockDim.x >> 6) - kWalkers;
    uint64_t* masks = smem;                                   // [2][H][6][n]
    // one chain with records: [n start][2][H][n] new words; otherwise a two-slot
    // buffer per walker
    const bool record = !PAIR && a.obs != nullptr;
    uint64_t* hist = masks + (size_t)2 * H * 6u * n;
    uint64_t* after = hist + (record ? (2u * H + 1u) * n : kWalkers * 128u);
    ClassList* work = reinterpret_cast<ClassList*>(after);
    const uint32_t pair = PAIR ? a.pairs[blockIdx.x] : 0u;
    const uint32_t stream = a.stream + pair;
    const bool walker = wave < kWalkers;
    ClassList& w = work[walker ? 0u : wave - kWalkers];
    const uint32_t me = wave - kWalkers;
    // the walker's word; lanes past the lattice's words repeat others (the row
    // form of 32^2 four times over, so that its row shifts stay within them)
    const uint32_t slot = ROWS == 32 ? lane & 15u : lane < n ? lane : 0u;

    uint64_t sig = 0, tau = 0;
    Window wA, wB;
    if (walker) {
        if constexpr (ROWS == 0) {
            wA = make_window<0>(a, slot);
            wB = make_window<1>(a, slot);
        }
        if constexpr (PAIR)
            sig = wave == 0 ? ~0ull : 0ull;
        else
            sig = a.int8_io ? load_bits64_i8<false>(static_cast<const int8_t*>(a.sigma) + 64u * slot)
                            : static_cast<const uint64_t*>(a.sigma)[slot];
        hist[record ? slot : 128u * wave + 64u + slot] = sig;
    }
    // epoch e: half-steps e H .. (its masks in slot e & 1, its words in slot e & 1)
    const uint32_t total = a.n_half;
    const uint32_t epochs = (total + H - 1u) / H;
    for (uint32_t e = 0; e <= epochs + (record ? 1u : 0u); ++e) {
        // workers: masks of epoch e, records of epoch e - 2; walkers: epoch e - 1
        if (walker) {
            if (e >= 1u && e <= epochs) {
                const uint32_t x0 = (e - 1u) * H;
                const uint32_t count = total - x0 < H ? total - x0 : H;
                const uint64_t* from = masks + (size_t)((e - 1u) & 1u) * H * 6u * n;
                if (!record) {
                    small_walk<ROWS, false>(a, count, from, hist + 128u * wave, slot, wA, wB, sig, tau);
                } else {
                    // the word before a slot is the last one of the other slot,
                    // or for slot 0 its copy in front
                    uint64_t* to = hist + n + (size_t)((e - 1u) & 1u) * H * n;
                    if (ROWS == 0 && e > 1u && ((e - 1u) & 1u) == 0) {
                        hist[slot] = sig;
                        class_sync();
                    }
                    small_walk<ROWS, true>(a, count, from, to, slot, wA, wB, sig, tau);
                }
            }
        } else {
            if (e < epochs) {
                const uint32_t x0 = e * H;
                small_draw<ROWS>(a, stream, w, me, workers, a.t0 + x0, total - x0 < H ? total - x0 : H,
                           masks + (size_t)(e & 1u) * H * 6u * n);
            }
            if (record && e >= 2u) {
                const uint32_t x0 = (e - 2u) * H;
                const uint32_t done = workers - 1u - me;   // the last worker has the fewest tiles
                small_records(a, done, workers, x0 / 2u, total - x0 < H ? total - x0 : H,
                              hist + n + (size_t)((e - 2u) & 1u) * H * n);
            }
        }
        __syncthreads();
    }
    if constexpr (PAIR) {
        if (walker)
            hist[128u * wave + lane] = sig;
        __syncthreads();
        if (wave == 0) {
            const bool differs = lane < n && hist[lane] != hist[128u + lane];
            if (lane < n)
                reinterpret_cast<uint64_t*>(a.samples)[(size_t)pair * n + lane] = sig;
            const uint64_t any = __ballot(differs);
            if (lane == 0)
                a.equal[blockIdx.x] = any ? 0u : 1u;
        }
    } else if (wave == 0 && lane < n) {
        if (a.int8_io) {
            store_bits64_i8<false>(static_cast<int8_t*>(a.sigma) + 64u * lane, sig);
            store_bits64_i8<false>(static_cast<int8_t*>(a.tau) + 64u * lane, tau);
        } else {
            static_cast<uint64_t*>(a.sigma)[lane] = sig;
            static_cast<uint64_t*>(a.tau)[lane] = tau;
        }
    }
}

template <int ROWS, bool PAIR>
hipError_t launch_small_t(const SmallArgs& a, uint32_t blocks, uint32_t threads, size_t lds, hipStream_t st) {
    if (lds > 65536u) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_small<ROWS, PAIR>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL((k_small<ROWS, PAIR>), dim3(blocks), dim3(threads), lds, st, a);
    return hipGetLastError();
}

}  // namespace

bool small_supported(int32_t L) { return L >= 8 && L <= 64 && L % 8 == 0; }

// Wavefronts and half-steps per epoch.  A tile of 64 (half-step, word) pairs
// is one worker's unit of work, so an epoch holds one per worker: 14 half-steps
// of a 64^2 lattice, 60 of a 32^2 one on 16 wavefronts; when there are more
// workgroups than CUs two share a CU (10 wavefronts and half the LDS each: with
// two walkers the most workers whose scratch leaves a tile for every one; 512
// samples of 32^2 with 7, 8, 9 and 10 wavefronts 9.9, 9.3, 9.2 and 8.8 ms).
// Lattices of few words stop at kMaxEpoch, where the walker is the slower side.
hipError_t launch_small(SmallArgs a, uint32_t blocks, bool pair, uint32_t n_cu, size_t max_lds, hipStream_t st) {
    constexpr uint32_t kMaxEpoch = 64;
    const bool share = blocks > n_cu;
    const uint32_t waves = share ? 10u : 16u;
    const uint32_t walkers = pair ? 2u : 1u;
    const size_t budget = share ? max_lds / 2 : max_lds;
    const size_t scratch = sizeof(ClassList) * (waves - walkers);
    auto lds_of = [&](uint32_t H) {
        const size_t hist = a.obs ? (size_t)(2u * H + 1u) * a.n : walkers * 128u;
        return sizeof(uint64_t) * ((size_t)2 * H * 6u * a.n + hist) + scratch;
    };
    uint32_t H = 64u * (waves - walkers) / a.n;
    H = H > kMaxEpoch ? kMaxEpoch : H;
    H = H > a.n_half ? a.n_half : H;
    H = H < 2u ? 2u : H & ~1u;
    while (H > 2u && lds_of(H) > budget)
        H -= 2u;
    a.H = H;
    const size_t lds = lds_of(H);
    if (lds > max_lds)
        return hipErrorInvalidValue;
    const uint32_t threads = 64u * waves;
#define SD_SMALL(ROWS)                                                          \
    return pair ? launch_small_t<ROWS, true>(a, blocks, threads, lds, st)      \
                : launch_small_t<ROWS, false>(a, blocks, threads, lds, st)
    if (a.L == 64u)
        SD_SMALL(64);
    if (a.L == 32u)
        SD_SMALL(32);
    SD_SMALL(0);
#undef SD_SMALL
}

}  // namespace sd
