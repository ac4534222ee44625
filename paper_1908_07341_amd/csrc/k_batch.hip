// Batched shaken dynamics: many independent chains, each with its own (J, q),
// lattice size L and stream id, in one persistent launch.
//
// The paper's parameter scan runs one chain per CPU thread (section 4, the
// Julia implementation with 80 threads over (q, J) pairs).  Here one workgroup
// owns one chain at a time with both packed lattices resident in LDS: it pops a
// chain index from a global work queue (chains are ordered longest first on the
// host), loads sigma, runs all steps with barriers between half-steps, records
// (M, A, B) of every obs_every-th step into the chain's trace, writes sigma and
// tau back and pops the next chain.  HBM is touched only for the initial and
// final lattices and the traces.
//
// Within a half-step each wavefront takes 64-word tiles of the lattice in
// turn (one word per lane).  Decided bits go straight to the LDS lattice; the
// undecided sites (top byte of the uniform equal to the threshold's, about
// one site in 256) are listed in the wavefront's LDS list, one per lane and
// round of ballots.  Whenever 64 or more sites are listed, and once at the
// end of the half-step, the wavefront resolves its list (one site per lane:
// one tail draw each) and ors the decided bits into the lattice words with
// LDS atomics (several sites may share a word; no other wavefront touches
// it).  So a half-step needs a single workgroup barrier, before the next one
// reads the lattice.  On recorded steps half-step B also accumulates M, A, B:
// the owner counts the decided sites of its word, the resolver the rest.
#include "sd_batch.hpp"

namespace sd {

namespace {

// BITS: rows need not start on a word (L % 64 != 0, L % 8 == 0); neighbours
// are windows of the lattice's bit string, and the word behind the lattice
// repeats its first, so that no window wraps inside.
template <bool BITS>
struct HalfCtx {
    const uint64_t* src;
    uint64_t* dst;
    uint32_t L, W, n_words;
    FastDiv divW;   // division by W = L / 64 (rows of whole words)
    FastDiv divL;   // division by L
    // bit strings: where the first row starts in the lane's first word (it
    // does not if >= 64), and the rows that start in a word whose first does
    // at bit 0
    uint32_t pos0;
    uint64_t starts;
};

// Rows of whole words: word g = j * W + w (row j, column word w) and its
// neighbours; every index is g plus or minus W or 1.
template <int WHICH, bool BITS>
__device__ __forceinline__ void gather_lds_g(const HalfCtx<BITS>& h, uint32_t g, uint32_t j, uint32_t w,
                                             uint64_t& c, uint64_t& n1, uint64_t& n2) {
    c = h.src[g];
    const uint32_t c_lo = (uint32_t)c, c_hi = (uint32_t)(c >> 32);
    if constexpr (WHICH == 0) {
        n1 = h.src[j == 0 ? g + h.n_words - h.W : g - h.W];
        const uint32_t prev_hi = (uint32_t)(h.src[w == 0 ? g + h.W - 1u : g - 1u] >> 32);
        n2 = (uint64_t)__builtin_amdgcn_alignbit(c_lo, prev_hi, 31) |
             ((uint64_t)__builtin_amdgcn_alignbit(c_hi, c_lo, 31) << 32);
    } else {
        n1 = h.src[j == h.L - 1 ? g + h.W - h.n_words : g + h.W];
        const uint32_t next_lo = (uint32_t)h.src[w == h.W - 1 ? g + 1u - h.W : g + 1u];
        n2 = (uint64_t)__builtin_amdgcn_alignbit(c_hi, c_lo, 1) |
             ((uint64_t)__builtin_amdgcn_alignbit(next_lo, c_hi, 1) << 32);
    }
}

// Bit strings: word g, whose first row starts at bit pos.  Every window is
// three dwords and two funnel shifts: its offset from the word is the same for
// all words.  (64-bit words, a division per word for the row start and wrapped
// indices took 50 operations more: 200^2, 1600 chains, 200 recorded steps:
// 4.96 -> 4.44 ms.)
template <int WHICH>
__device__ __forceinline__ void gather_lds_bits(const HalfCtx<true>& h, uint32_t g, uint32_t pos, uint64_t& c,
                                                uint64_t& n1, uint64_t& n2) {
    const lds_dword* d = reinterpret_cast<const lds_dword*>(h.src);
    const uint32_t n = 2u * h.n_words, N = 64u * h.n_words;
    c = h.src[g];
    const uint32_t c_lo = (uint32_t)c, c_hi = (uint32_t)(c >> 32);
    auto window = [&](uint32_t off, uint32_t& lo, uint32_t& hi) __attribute__((always_inline)) {
        uint32_t at = 2u * g + (off >> 5);
        at = at < at - n ? at : at - n;   // at mod n: at - n wraps to a large value while at < n
        const uint32_t w0 = d[at], w1 = d[at + 1u], w2 = d[at + 2u];
        lo = __builtin_amdgcn_alignbit(w1, w0, off & 31u);
        hi = __builtin_amdgcn_alignbit(w2, w1, off & 31u);
    };
    uint32_t n1_lo, n1_hi, lo, hi, wrap_lo, wrap_hi;
    if constexpr (WHICH == 0) {
        window(N - h.L, n1_lo, n1_hi);
        window(h.L - 1u, wrap_lo, wrap_hi);
        const uint32_t before = 2u * g - 1u;
        const uint32_t prev = d[before < n - 1u ? before : n - 1u];
        lo = __builtin_amdgcn_alignbit(c_lo, prev, 31);
        hi = __builtin_amdgcn_alignbit(c_hi, c_lo, 31);
    } else {
        window(h.L, n1_lo, n1_hi);
        window(N + 1u - h.L, wrap_lo, wrap_hi);
        const uint32_t next = d[2u * g + 2u];
        lo = __builtin_amdgcn_alignbit(c_hi, c_lo, 1);
        hi = __builtin_amdgcn_alignbit(next, c_hi, 1);
        pos = pos - 1u < h.L - 1u ? pos - 1u : h.L - 1u;   // the rows' last columns
    }
    const uint64_t edge = pos < 64u ? h.starts << pos : 0ull;
    const uint32_t e_lo = (uint32_t)edge, e_hi = (uint32_t)(edge >> 32);
    n1 = (uint64_t)n1_lo | ((uint64_t)n1_hi << 32);
    n2 = (uint64_t)((lo & ~e_lo) | (wrap_lo & e_lo)) | ((uint64_t)((hi & ~e_hi) | (wrap_hi & e_hi)) << 32);
}

// The partner and neighbour bits of site s.
template <int WHICH, bool BITS>
__device__ __forceinline__ void site_bits(const HalfCtx<BITS>& h, uint32_t s, uint32_t& c, uint32_t& n1, uint32_t& n2) {
    const lds_dword* d = reinterpret_cast<const lds_dword*>(h.src);
    const uint32_t N = 64u * h.n_words;
    const uint32_t i = s - fdiv(s, h.divL) * h.L;
    uint32_t s1, s2;
    if constexpr (WHICH == 0) {
        s1 = s - h.L < s - h.L + N ? s - h.L : s - h.L + N;   // s - L, + N where that is negative
        s2 = s - 1u + (i == 0 ? h.L : 0u);
    } else {
        s1 = s + h.L < s + h.L - N ? s + h.L : s + h.L - N;
        s2 = s + 1u - (i == h.L - 1u ? h.L : 0u);
    }
    c = (d[s >> 5] >> (s & 31u)) & 1u;
    n1 = (d[s1 >> 5] >> (s1 & 31u)) & 1u;
    n2 = (d[s2 >> 5] >> (s2 & 31u)) & 1u;
}

// Per-wavefront list of undecided sites (64 * word + bit).  A round of
// ballots adds at most 64 entries and the list is resolved as soon as it
// holds 64, so it never holds more than 127.
constexpr uint32_t kWListCap = 128;

struct WaveWordList {
    uint32_t site[kWListCap];
};

// The chain's per-launch constants in LDS.
struct ChainShared {
    uint32_t T24[6];   // tail thresholds of the classes (paired_tail in the paired form)
};

// A thread's counts of one half-step: at most 2 per site of the lattice
// (10240 words of 64 sites at most in LDS), so 32 bits hold them and every
// popcount adds in one instruction.
struct ObsSums {
    uint32_t pc = 0, dpair = 0, dself = 0;   // #+1, #differences to up+right, to the partner
};

// Resolves n <= 64 sites of the wavefront's list, from `first` on, into the
// lattice.
template <int WHICH, bool OBS, bool BITS>
__device__ __forceinline__ void resolve_list(const HalfCtx<BITS>& h, const DrawParams& dp, const uint32_t* T24,
                                             WaveWordList& wl, uint32_t first, uint32_t n, ObsSums& acc) {
    const uint32_t lane = threadIdx.x & 63u;
    if (lane < n) {
        const uint32_t v = wl.site[first + lane];
        uint32_t c, n1, n2;
        site_bits<WHICH>(h, v, c, n1, n2);
        const uint32_t bit = draw_tail24(dp, v) < T24[2u * (n1 + n2) + c] ? 1u : 0u;
        if (bit) {
            lds_dword* to = reinterpret_cast<lds_dword*>(h.dst) + (v >> 5);
            atomicOr(to, 1u << (v & 31u));
            if constexpr (BITS) {
                if (v < 64u)   // the copy of the first word
                    atomicOr(to + 2u * h.n_words, 1u << (v & 31u));
            }
        }
        if constexpr (OBS) {
            acc.pc += bit;
            acc.dpair += (bit ^ n1) + (bit ^ n2);
            acc.dself += bit ^ c;
        }
    }
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adds the wavefront's observable sums to obs_sum[0 .. 2] (LDS), one atomic
// per quantity.  A wavefront's counts of one half-step stay far below 2^32
// (at most 2 per site of the lattice).
__device__ __forceinline__ void add_wave_obs(const ObsSums& acc, unsigned long long* obs_sum) {
    const uint32_t v0 = wave_sum_dpp(acc.pc);
    const uint32_t v1 = wave_sum_dpp(acc.dpair);
    const uint32_t v2 = wave_sum_dpp(acc.dself);
    if ((threadIdx.x & 63u) == 0) {
        atomicAdd(&obs_sum[0], (unsigned long long)v0);
        atomicAdd(&obs_sum[1], (unsigned long long)v1);
        atomicAdd(&obs_sum[2], (unsigned long long)v2);
    }
}

// One half-step of the workgroup's chain, src -> dst in LDS, ending with a
// workgroup barrier.  OBS (half-step B of a recorded step): accumulate the
// observables of the new pair (dst, src) in acc and add the wavefront's sums
// to obs_sum[0 .. 2] (LDS) before the closing barrier.
template <int WHICH, bool PAIRED, bool COMPLEMENT, bool OBS, bool BITS>
__device__ __forceinline__ void lds_half_step(const HalfCtx<BITS>& h, const DrawParams& dp, const PlaneMasks& pm,
                                              const uint32_t* T24, WaveWordList& wl, ObsSums& acc,
                                              unsigned long long* obs_sum) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t n_waves = blockDim.x >> 6;
    const uint32_t n_tiles = (h.n_words + 63u) / 64u;
    uint32_t listed = 0;   // wavefront-uniform
    // rows of whole words: (row, column word) of the lane's word, stepped by
    // the 64 * n_waves words between a wavefront's tiles
    uint32_t j = 0, w = 0, step_rows = 0, step_cols = 0;
    // bit strings: where the first row starts in the lane's word
    uint32_t pos = 0, pos_step = 0;
    if constexpr (BITS) {
        pos = h.pos0;
        pos_step = (64u * 64u * n_waves) % h.L;
    } else {
        const uint32_t g0 = 64u * (threadIdx.x >> 6) + lane;
        j = fdiv(g0, h.divW);
        w = g0 - j * h.W;
        const uint32_t step = 64u * n_waves;
        step_rows = step / h.W;
        step_cols = step - step_rows * h.W;
    }
    for (uint32_t tile = threadIdx.x >> 6; tile < n_tiles; tile += n_waves) {
        const uint32_t g = 64u * tile + lane;
        // lattices whose rows are whole words hold L * L / 64 = 64 (L / 64)^2
        // words: every tile is full
        const bool active = !BITS || g < h.n_words;
        const uint32_t ga = active ? g : h.n_words - 1u;   // a word to read and draw in any case
        uint64_t c, n1, n2;
        if constexpr (BITS) {
            gather_lds_bits<WHICH>(h, ga, pos, c, n1, n2);
            // later by pos_step, mod L
            pos = pos - pos_step < pos - pos_step + h.L ? pos - pos_step : pos - pos_step + h.L;
        } else {
            gather_lds_g<WHICH>(h, ga, j, w, c, n1, n2);
            w += step_cols;
            j += step_rows;
            if (w >= h.W) {
                w -= h.W;
                ++j;
            }
        }
        uint64_t P[8];
        draw_planes(dp, ga, P);
        const WordDraw wd = compare_planes<PAIRED, COMPLEMENT>(P, c, n1, n2, pm);
        uint64_t und = active ? wd.und : 0ull;
        if (active) {
            h.dst[g] = wd.lt;
            if constexpr (BITS) {
                if (tile == 0 && lane == 0)   // the copy of the first word
                    h.dst[h.n_words] = wd.lt;
            }
            if constexpr (OBS) {
                acc.pc += __popcll(wd.lt);
                acc.dpair += __popcll((wd.lt ^ n1) & ~und) + __popcll((wd.lt ^ n2) & ~und);
                acc.dself += __popcll((wd.lt ^ c) & ~und);
            }
        }
        for (;;) {
            const uint64_t m = __ballot(und != 0);
            if (m == 0)
                break;
            if (und != 0) {
                const uint32_t e = listed + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                wl.site[e] = 64u * g + (uint32_t)__builtin_ctzll(und);
                und &= und - 1;
            }
            listed += (uint32_t)__popcll(m);
            if (listed >= 64u) {
                listed -= 64u;
                wave_sync_lds();
                resolve_list<WHICH, OBS>(h, dp, T24, wl, listed, 64u, acc);
                wave_sync_lds();
            }
        }
    }
    if (listed) {
        wave_sync_lds();
        resolve_list<WHICH, OBS>(h, dp, T24, wl, 0u, listed, acc);
    }
    if constexpr (OBS)
        add_wave_obs(acc, obs_sum);
    __syncthreads();
}

// Observables of the pair (sig, tau) as sums over the workgroup's threads
// (a separate pass, used for chains with the general compare).
template <bool BITS>
__device__ __forceinline__ ObsSums lds_observe(const uint64_t* sig, const uint64_t* tau, const HalfCtx<BITS>& h) {
    ObsSums acc;
    if constexpr (BITS) {
        for (uint32_t g = threadIdx.x; g < h.n_words; g += blockDim.x) {
            uint64_t t, up, right;
            gather_bits<1>(tau, h.L, h.n_words, h.divL, g, t, up, right);
            const uint64_t sg = sig[g];
            acc.pc += __popcll(sg);
            acc.dpair += __popcll(sg ^ up) + __popcll(sg ^ right);
            acc.dself += __popcll(sg ^ t);
        }
        return acc;
    }
    for (uint32_t g = threadIdx.x; g < h.n_words; g += blockDim.x) {
        const uint32_t j = fdiv(g, h.divW);
        const uint32_t w = g - j * h.W;
        const uint64_t s = sig[g], t = tau[g];
        const uint64_t up = tau[(j == h.L - 1 ? 0 : j + 1) * h.W + w];
        const uint64_t next = tau[j * h.W + (w == h.W - 1 ? 0 : w + 1)];
        const uint64_t right = (t >> 1) | (next << 63);
        acc.pc += __popcll(s);
        acc.dpair += __popcll(s ^ up) + __popcll(s ^ right);
        acc.dself += __popcll(s ^ t);
    }
    return acc;
}

// Copy of an LDS lattice to global memory (the workgroup's threads).
__device__ __forceinline__ void store_lattice(uint64_t* out, const uint64_t* lat, uint32_t n_words) {
    for (uint32_t g = threadIdx.x; g < n_words; g += blockDim.x)
        out[g] = lat[g];
}

// Steps of one chain.  Paired chains fold the observables into half-step B;
// the general compare (only under its flag) leaves them to a separate pass so
// that its register count stays low.  mom (used by thread 0 only): the chain's
// running sums in moments mode.
template <bool PAIRED, bool COMPLEMENT, bool BITS>
__device__ __forceinline__ void run_steps(const BatchArgs& a, const HalfCtx<BITS>& hA, const HalfCtx<BITS>& hB,
                                          DrawParams dp,
                                          const uint32_t* T24, WaveWordList& wl, int64_t* trace,
                                          unsigned long long* obs_sum, uint64_t* traj,
                                          int64_t (&mom)[kMomentWords]) {
    const PlaneMasks pm = make_plane_masks<PAIRED>(dp);
    for (uint32_t m = 0; m < a.k_steps; ++m) {
        const uint32_t n = a.step0 + m;
        ObsSums acc;
        dp.t = 2u * n;
        lds_half_step<0, PAIRED, COMPLEMENT, false>(hA, dp, pm, T24, wl, acc, obs_sum);
        // (each half-step ends with a barrier, so a copy made here is complete
        // before the lattice is next overwritten, two half-steps later)
        if (traj)
            store_lattice(traj + (size_t)(2u * m + 1u) * hA.n_words, hA.dst, hA.n_words);
        dp.t = 2u * n + 1u;
        if (trace && (m + 1) % a.obs_every == 0) {
            if constexpr (PAIRED) {
                lds_half_step<1, PAIRED, COMPLEMENT, true>(hB, dp, pm, T24, wl, acc, obs_sum);
            } else {
                lds_half_step<1, PAIRED, COMPLEMENT, false>(hB, dp, pm, T24, wl, acc, obs_sum);
                acc = lds_observe(hB.dst, hA.dst, hA);
                add_wave_obs(acc, obs_sum);
                __syncthreads();
            }
            // every wavefront added its sums before the last barrier; the
            // next recorded step adds again only after half-step A's barrier
            if (threadIdx.x == 0) {
                const int64_t v[3] = {(int64_t)obs_sum[0], (int64_t)obs_sum[1], (int64_t)obs_sum[2]};
                obs_sum[0] = obs_sum[1] = obs_sum[2] = 0;
                const int64_t sites = (int64_t)hA.n_words * 64;
                const int64_t M = 2 * v[0] - sites, A = 2 * sites - 2 * v[1], B = sites - 2 * v[2];
                if (a.moments) {
                    mom[0] += M;
                    mom[1] += M * M;
                    mom[2] += M < 0 ? -M : M;
                    mom[3] += A;
                    mom[4] += B;
                } else {
                    int64_t* out3 = trace + 3u * (size_t)((m + 1) / a.obs_every - 1);
                    out3[0] = M;
                    out3[1] = A;
                    out3[2] = B;
                }
            }
        } else {
            lds_half_step<1, PAIRED, COMPLEMENT, false>(hB, dp, pm, T24, wl, acc, obs_sum);
        }
        if (traj)
            store_lattice(traj + (size_t)(2u * m + 2u) * hB.n_words, hB.dst, hB.n_words);
    }
}

// PAIRED: every chain of the launch has a paired threshold table.  BITS: the
// chains' L are multiples of 8 but not of 64 (bit-string neighbours).
template <bool COMPLEMENT, bool PAIRED, bool BITS>
__device__ __forceinline__ void batch_chains_body(const BatchArgs& a) {
    extern __shared__ uint64_t smem[];
    __shared__ uint32_t s_chain;
    __shared__ uint32_t s_queue;   // the queue this workgroup takes chains from (0: its own)
    __shared__ ChainShared s_ch;
    __shared__ unsigned long long s_obs[3];   // a recorded step's sums, added by every wavefront
    uint64_t* sig = smem;
    uint64_t* tau = smem + a.max_words + 1u;
    WaveWordList& wl = reinterpret_cast<WaveWordList*>(tau + a.max_words + 1u)[threadIdx.x >> 6];

    if (threadIdx.x == 0) {
        s_queue = 0;
        s_obs[0] = s_obs[1] = s_obs[2] = 0;
        if (a.t_start)
            atomicMin(a.t_start, (unsigned long long)wall_clock64());
    }
    for (uint32_t iter = 0;; ++iter) {
        ChainDesc cd;
        if (a.counter) {
            // the next chain of this launch's queue, then of the later queues
            // in turn once it is empty (every queue is exhausted at most once
            // per workgroup: s_queue only moves forward)
            if (threadIdx.x == 0) {
                uint32_t chain = ~0u;
                while (s_queue <= a.n_steal) {
                    const uint32_t q = s_queue;
                    uint32_t* ctr = q == 0 ? a.counter : a.steal_counter[q - 1];
                    const uint32_t cnt = q == 0 ? a.n_chains : a.steal_count[q - 1];
                    const uint32_t i = atomicAdd(ctr, 1u);
                    if (i < cnt) {
                        chain = q == 0 ? a.order[i] : a.steal_order[q - 1][i];
                        break;
                    }
                    s_queue = q + 1;
                }
                s_chain = chain;
            }
            __syncthreads();
            // a workgroup-uniform index, so that the descriptor is read with
            // scalar loads into scalar registers
            const uint32_t ci = __builtin_amdgcn_readfirstlane(s_chain);
            if (ci == ~0u)
                break;
            cd = a.chains[ci];
        } else if (a.n_uniform) {
            if (iter > 0 || blockIdx.x >= a.n_uniform)
                break;
            cd = a.single;
            cd.stream += blockIdx.x;
        } else {
            if (iter > 0 || blockIdx.x != 0)
                break;
            cd = a.single;
        }
        // the chain's geometry is the same for the whole workgroup: keep it in
        // scalar registers
        auto uni = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane(v); };
        auto uni_div = [&](const FastDiv& f) {
            FastDiv u;
            u.d = uni(f.d);
            u.mul = uni(f.mul);
            u.shift = uni(f.shift);
            u.add = uni(f.add);
            return u;
        };
        cd.L = uni(cd.L);
        cd.stream = uni(cd.stream);
        HalfCtx<BITS> hA, hB;
        hA.L = hB.L = cd.L;
        hA.W = hB.W = cd.L / 64u;
        hA.n_words = hB.n_words = (uint32_t)(((uint64_t)cd.L * cd.L) / 64u);
        hA.divW = hB.divW = uni_div(cd.divW);
        hA.divL = hB.divL = uni_div(cd.divL);
        hA.src = sig; hA.dst = tau;
        hB.src = tau; hB.dst = sig;
        const uint32_t n_words = hA.n_words;
        if constexpr (BITS) {
            const uint32_t s = 64u * threadIdx.x;   // the lane's first word starts at column s mod L
            const uint32_t m = s - fdiv(s, hA.divL) * cd.L;
            hA.pos0 = hB.pos0 = m ? cd.L - m : 0u;
            uint64_t starts = 1u;
            for (uint32_t b = cd.L; b < 64u; b += cd.L)
                starts |= 1ull << b;
            hA.starts = hB.starts = starts;
        }

        // load sigma (packed words, or int8 bytes converted to bits)
        if (a.int8_io) {
            const int8_t* src8 = reinterpret_cast<const int8_t*>(a.counter ? a.lattices + cd.sig_offset : a.single_sig);
            for (uint32_t g = threadIdx.x; g < n_words; g += blockDim.x)
                sig[g] = load_bits64_i8(src8 + (size_t)64u * g);
        } else {
            const uint64_t* src =
                a.counter ? reinterpret_cast<const uint64_t*>(a.lattices + cd.sig_offset)
                          : reinterpret_cast<const uint64_t*>(a.single_sig) + (size_t)(a.n_uniform ? blockIdx.x : 0u) * n_words;
            for (uint32_t g = threadIdx.x; g < n_words; g += blockDim.x)
                sig[g] = src[g];
        }
        if (threadIdx.x == 0) {
#pragma unroll
            for (int i = 0; i < 6; ++i)
                s_ch.T24[i] = PAIRED ? paired_tail(cd.T, i) : cd.T[i] & 0xFFFFFFu;
            if constexpr (BITS)
                sig[n_words] = sig[0];   // word 0 is this thread's
        }
        __syncthreads();

        DrawParams dp;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            dp.T[i] = cd.T[i];
        dp.key0 = a.key0;
        dp.key1 = a.key1;
        dp.stream = cd.stream;
        dp.tag2 = 0;
        dp.rng_xor = COMPLEMENT ? 0xFFFFFFFFu : 0u;
        int64_t* trace = a.traces ? a.traces + cd.trace_offset : nullptr;
        uint64_t* traj = a.traj ? reinterpret_cast<uint64_t*>(a.traj + (size_t)blockIdx.x * a.traj_chain_bytes) : nullptr;
        if (traj)
            store_lattice(traj, sig, n_words);

        int64_t mom[kMomentWords] = {0, 0, 0, 0, 0};
        run_steps<PAIRED, COMPLEMENT, BITS>(a, hA, hB, dp, s_ch.T24, wl, trace, s_obs, traj, mom);
        if (a.moments && trace && threadIdx.x == 0) {
#pragma unroll
            for (uint32_t i = 0; i < kMomentWords; ++i)
                trace[i] = mom[i];
        }
        if (traj) {
            __syncthreads();
            continue;
        }

        // write sigma and tau back
        if (a.int8_io) {
            int8_t* dst8 = reinterpret_cast<int8_t*>(a.counter ? a.lattices + cd.sig_offset : a.single_sig);
            int8_t* dst8t = reinterpret_cast<int8_t*>(a.counter ? a.lattices + cd.tau_offset : a.single_tau);
            for (uint32_t g = threadIdx.x; g < (a.k_steps ? 2u : 1u) * n_words; g += blockDim.x) {
                const bool is_tau = g >= n_words;
                const uint32_t gg = is_tau ? g - n_words : g;
                store_bits64_i8((is_tau ? dst8t : dst8) + (size_t)64u * gg, is_tau ? tau[gg] : sig[gg]);
            }
        } else {
            uint64_t* dsig = reinterpret_cast<uint64_t*>(a.counter ? a.lattices + cd.sig_offset : a.single_sig);
            uint64_t* dtau = reinterpret_cast<uint64_t*>(a.counter ? a.lattices + cd.tau_offset : a.single_tau);
            for (uint32_t g = threadIdx.x; g < n_words; g += blockDim.x) {
                dsig[g] = sig[g];
                if (a.k_steps)
                    dtau[g] = tau[g];
            }
        }
        __syncthreads();
    }
    if (a.t_end && threadIdx.x == 0)
        atomicMax(a.t_end, (unsigned long long)wall_clock64());
}

// The paired compare (every threshold table by default) in workgroups of up
// to 640 threads held to 96 VGPRs, so that two workgroups of ten wavefronts
// share a CU with the largest (512^2) chains in LDS; the six-class compare
// keeps the compiler's register count and at most 512 threads.
template <bool COMPLEMENT, bool BITS>
__global__ __launch_bounds__(kBatchMaxThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_batch_chains(
    BatchArgs a) {
    batch_chains_body<COMPLEMENT, true, BITS>(a);
}

template <bool COMPLEMENT, bool BITS>
__global__ __launch_bounds__(512) void k_batch_chains_general(BatchArgs a) {
    batch_chains_body<COMPLEMENT, false, BITS>(a);
}

// Recorded trajectories of lattices with at most one word per lane of a
// workgroup: chain blockIdx.x of the n_uniform chains, every half-step's
// lattice written to a.traj.
//
// A half-step has two phases.  In the first every lane compares its word with
// the planes it holds and lists its undecided sites in one list for the
// workgroup; in the second the first lanes resolve the list, one site each,
// and every lane draws the planes of the next half-step, which do not depend
// on the lattice.  So a tail's chain of reads and its Philox call hide behind
// the draws, and the resolvers' lanes are all busy: with a list per wavefront
// only a quarter of them is, as about 16 of a tile's 4096 sites are undecided.
// The finished word is written out by the lane that reads it as its partner
// word a half-step later.  Lattices that leave most of a CU's wavefronts idle
// draw with SPLIT lanes per word, 4 / SPLIT Philox calls each, and pass the
// planes through LDS.
// Bound by the vector unit (82% of its issue slots).  256 chains, one
// workgroup per CU, per half-step: 256^2 2.95 us with a list per wavefront and
// two tiles per wavefront (2.9 with one), 2.67 here; 200^2 4.1 -> 2.3; 128^2
// 1.60 -> 1.32; 32^2 2.0 -> 1.2.
__host__ __device__ inline uint32_t recorded_list_cap(uint32_t n_words) {
    // a quarter of a site per word is listed on average; what does not fit is
    // resolved by the lane that found it
    return n_words / 4u + 32u;
}

template <int WHICH, bool BITS>
__device__ __forceinline__ void resolve_site(const HalfCtx<BITS>& h, const DrawParams& dp, const uint32_t* T24,
                                             uint32_t v) {
    uint32_t c, n1, n2;
    site_bits<WHICH>(h, v, c, n1, n2);
    if (draw_tail24(dp, v) < T24[2u * (n1 + n2) + c]) {
        lds_dword* to = reinterpret_cast<lds_dword*>(h.dst) + (v >> 5);
        atomicOr(to, 1u << (v & 31u));
        if constexpr (BITS) {
            if (v < 64u)   // the copy of the first word
                atomicOr(to + 2u * h.n_words, 1u << (v & 31u));
        }
    }
}

// What a workgroup keeps in LDS besides its lattices.
struct RecordedShared {
    uint32_t* list;    // undecided sites of the half-step, up to cap
    uint4* planes;     // SPLIT > 1: the words of call p for word g at p * lanes + g
    uint32_t cap, lanes;
    uint32_t* counts;   // by WHICH: sites listed
    const uint32_t* T24;
};

// The planes of word g: SPLIT == 1 in P, else this lane's share of the calls
// to LDS.
template <int SPLIT>
__device__ __forceinline__ void recorded_draw(const DrawParams& dp, uint32_t g, uint32_t lane_g, uint32_t part,
                                              uint64_t (&P)[8], const RecordedShared& sh) {
    if constexpr (SPLIT == 1) {
        draw_planes(dp, g, P);
    } else {
#pragma unroll
        for (uint32_t k = 0; k < 4u / SPLIT; ++k) {
            const uint32_t p = part * (4u / SPLIT) + k;
            const U4 x = philox10_uuuv(dp.stream, dp.t | (p << 30), dp.tag2, g, dp.key0, dp.key1);
            sh.planes[p * sh.lanes + lane_g] = make_uint4(x.x0, x.x1, x.x2, x.x3);
        }
    }
}

// One half-step from the planes of dp.t, after which those of dp.t + 1 are
// drawn.  Wavefronts with part > 0 only draw and resolve.
template <int WHICH, bool BITS, int SPLIT>
__device__ __forceinline__ void recorded_half_step(const HalfCtx<BITS>& h, DrawParams& dp, uint32_t code, uint32_t g,
                                                   uint32_t part, uint32_t j, uint32_t w, uint64_t (&P)[8],
                                                   uint64_t* record, const RecordedShared& sh) {
    const bool active = g < h.n_words;
    const uint32_t ga = active ? g : h.n_words - 1u;
    if (threadIdx.x == 0)
        sh.counts[1 - WHICH] = 0;   // last read before the barrier that ended the previous half-step
    if (SPLIT == 1 || part == 0) {
        if constexpr (SPLIT > 1) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint4 x = sh.planes[p * sh.lanes + g];
                P[2 * p] = (uint64_t)x.x | ((uint64_t)x.y << 32);
                P[2 * p + 1] = (uint64_t)x.z | ((uint64_t)x.w << 32);
            }
        }
        uint64_t c, n1, n2;
        if constexpr (BITS)
            gather_lds_bits<WHICH>(h, ga, h.pos0, c, n1, n2);
        else
            gather_lds_g<WHICH>(h, ga, j, w, c, n1, n2);
        const WordDraw wd = compare_planes_paired<false>(P, c, n1, n2, code);
        uint64_t und = active ? wd.und : 0ull;
        if (active) {
            h.dst[g] = wd.lt;
            if constexpr (BITS) {
                if (g == 0)   // the copy of the first word
                    h.dst[h.n_words] = wd.lt;
            }
            record[g] = c;
        }
        const uint32_t mine = (uint32_t)__popcll(und);
        const uint32_t upto = wave_prefix_dpp(mine);
        uint32_t base = 0;
        if ((threadIdx.x & 63u) == 63u)
            base = atomicAdd(&sh.counts[WHICH], upto);
        uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)base, 63) + upto - mine;
        for (; und; und &= und - 1, ++e) {
            const uint32_t v = 64u * g + (uint32_t)__builtin_ctzll(und);
            if (e < sh.cap)
                sh.list[e] = v;
            else
                resolve_site<WHICH>(h, dp, sh.T24, v);
        }
    }
    __syncthreads();
    const uint32_t n = sh.counts[WHICH] < sh.cap ? sh.counts[WHICH] : sh.cap;
    if (threadIdx.x < n)
        resolve_site<WHICH>(h, dp, sh.T24, sh.list[threadIdx.x]);
    ++dp.t;
    recorded_draw<SPLIT>(dp, ga, g, part, P, sh);
    __syncthreads();
}

template <bool BITS, int SPLIT>
__global__ __launch_bounds__(kRecordedMaxWords) void k_batch_recorded(BatchArgs a) {
    extern __shared__ uint64_t smem[];
    __shared__ uint32_t T24[6];
    __shared__ uint32_t counts[2];
    const ChainDesc& cd = a.single;
    HalfCtx<BITS> hA, hB;
    hA.L = hB.L = cd.L;
    hA.W = hB.W = cd.L / 64u;
    hA.n_words = hB.n_words = a.max_words;
    hA.divW = hB.divW = cd.divW;
    hA.divL = hB.divL = cd.divL;
    uint64_t* sig = smem;
    uint64_t* tau = smem + a.max_words + 1u;
    RecordedShared sh;
    sh.lanes = 64u * ((a.max_words + 63u) / 64u);
    sh.planes = reinterpret_cast<uint4*>(tau + a.max_words + 1u);   // 16-byte aligned: behind 2 n + 2 words
    sh.cap = recorded_list_cap(a.max_words);
    sh.list = reinterpret_cast<uint32_t*>(sh.planes + (SPLIT > 1 ? 4u * sh.lanes : 0u));
    sh.counts = counts;
    sh.T24 = T24;
    hA.src = sig; hA.dst = tau;
    hB.src = tau; hB.dst = sig;
    const uint32_t part = SPLIT == 1 ? 0u : __builtin_amdgcn_readfirstlane(threadIdx.x / sh.lanes);
    const uint32_t g = threadIdx.x - part * sh.lanes;
    const bool active = part == 0 && g < a.max_words;
    uint32_t j = 0, w = 0;
    if constexpr (BITS) {
        const uint32_t m = 64u * g - fdiv(64u * g, cd.divL) * cd.L;
        hA.pos0 = hB.pos0 = m ? cd.L - m : 0u;
        uint64_t starts = 1u;
        for (uint32_t b = cd.L; b < 64u; b += cd.L)
            starts |= 1ull << b;
        hA.starts = hB.starts = starts;
    } else {
        j = fdiv(g, cd.divW);
        w = g - j * hA.W;
    }
    DrawParams dp;
#pragma unroll
    for (int i = 0; i < 6; ++i)
        dp.T[i] = cd.T[i];
    dp.key0 = a.key0;
    dp.key1 = a.key1;
    dp.stream = cd.stream + blockIdx.x;
    dp.t = 2u * a.step0;
    dp.tag2 = 0;
    dp.rng_xor = 0;
    const uint32_t code = make_plane_masks<true>(dp).code;
    if (active)
        sig[g] = (reinterpret_cast<const uint64_t*>(a.single_sig) + (size_t)blockIdx.x * a.max_words)[g];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < 6; ++i)
            T24[i] = paired_tail(cd.T, i);
        counts[0] = 0;
        if constexpr (BITS)
            sig[a.max_words] = sig[0];
    }
    uint64_t* record = reinterpret_cast<uint64_t*>(a.traj + (size_t)blockIdx.x * a.traj_chain_bytes);
    uint64_t P[8];
    recorded_draw<SPLIT>(dp, g < a.max_words ? g : a.max_words - 1u, g, part, P, sh);
    __syncthreads();
    for (uint32_t m = 0; m < a.k_steps; ++m) {
        recorded_half_step<0, BITS, SPLIT>(hA, dp, code, g, part, j, w, P, record, sh);
        record += a.max_words;
        recorded_half_step<1, BITS, SPLIT>(hB, dp, code, g, part, j, w, P, record, sh);
        record += a.max_words;
    }
    if (active)
        record[g] = sig[g];
}

__global__ void k_zero_u32(uint32_t* p, uint32_t n) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        p[i] = 0;
}

}  // namespace

size_t batch_lds_bytes(uint32_t max_words, uint32_t threads) {
    return (size_t)2 * (max_words + 1u) * sizeof(uint64_t) + (size_t)((threads + 63u) / 64u) * sizeof(WaveWordList);
}

template <bool BITS>
void launch_batch_chains_t(const BatchArgs& a, uint32_t blocks, uint32_t threads, size_t lds, hipStream_t st) {
    if (a.rng_xor && a.paired)
        hipLaunchKernelGGL((k_batch_chains<true, BITS>), dim3(blocks), dim3(threads), lds, st, a);
    else if (a.rng_xor)
        hipLaunchKernelGGL((k_batch_chains_general<true, BITS>), dim3(blocks), dim3(threads), lds, st, a);
    else if (a.paired)
        hipLaunchKernelGGL((k_batch_chains<false, BITS>), dim3(blocks), dim3(threads), lds, st, a);
    else
        hipLaunchKernelGGL((k_batch_chains_general<false, BITS>), dim3(blocks), dim3(threads), lds, st, a);
}

template <int SPLIT>
void launch_batch_recorded_t(const BatchArgs& a, uint32_t lanes, hipStream_t st) {
    const size_t lds = (size_t)2 * (a.max_words + 1u) * sizeof(uint64_t) +
                       (SPLIT > 1 ? (size_t)4 * lanes * sizeof(uint4) : 0) +
                       (size_t)recorded_list_cap(a.max_words) * sizeof(uint32_t);
    if (a.bits)
        hipLaunchKernelGGL((k_batch_recorded<true, SPLIT>), dim3(a.n_uniform), dim3(SPLIT * lanes), lds, st, a);
    else
        hipLaunchKernelGGL((k_batch_recorded<false, SPLIT>), dim3(a.n_uniform), dim3(SPLIT * lanes), lds, st, a);
}

hipError_t launch_batch_recorded(const BatchArgs& a, uint32_t n_cu, hipStream_t st) {
    // As many lanes per word as a workgroup has room for, unless CUs have more
    // than one chain, whose wavefronts then fill each other's waits: 128^2, four
    // and one lane per word, 256 chains 1.32 and 1.68 us per half-step, 600
    // chains 3.8 and 2.3.
    const uint32_t lanes = 64u * ((a.max_words + 63u) / 64u);
    const bool alone = a.n_uniform <= n_cu;
    if (alone && 4u * lanes <= kRecordedMaxWords)
        launch_batch_recorded_t<4>(a, lanes, st);
    else if (alone && 2u * lanes <= kRecordedMaxWords)
        launch_batch_recorded_t<2>(a, lanes, st);
    else
        launch_batch_recorded_t<1>(a, lanes, st);
    return hipGetLastError();
}

hipError_t launch_batch_chains(const BatchArgs& a, uint32_t blocks, uint32_t threads, hipStream_t st) {
    const size_t lds = batch_lds_bytes(a.max_words, threads);
    if (a.bits)
        launch_batch_chains_t<true>(a, blocks, threads, lds, st);
    else
        launch_batch_chains_t<false>(a, blocks, threads, lds, st);
    return hipGetLastError();
}

__global__ void k_times_reset(unsigned long long* starts, unsigned long long* ends, uint32_t n) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        starts[i] = ~0ull;
        ends[i] = 0ull;
    }
}

hipError_t launch_times_reset(unsigned long long* starts, unsigned long long* ends, uint32_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_times_reset, dim3(1), dim3(64), 0, st, starts, ends, n);
    return hipGetLastError();
}

hipError_t launch_zero_u32(uint32_t* p, uint32_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, st, p, n);
    return hipGetLastError();
}

hipError_t batch_kernel_attributes(size_t max_dynamic_lds) {
    const void* kernels[8] = {reinterpret_cast<const void*>(&k_batch_chains_general<false, false>),
                              reinterpret_cast<const void*>(&k_batch_chains<false, false>),
                              reinterpret_cast<const void*>(&k_batch_chains_general<true, false>),
                              reinterpret_cast<const void*>(&k_batch_chains<true, false>),
                              reinterpret_cast<const void*>(&k_batch_chains_general<false, true>),
                              reinterpret_cast<const void*>(&k_batch_chains<false, true>),
                              reinterpret_cast<const void*>(&k_batch_chains_general<true, true>),
                              reinterpret_cast<const void*>(&k_batch_chains<true, true>)};
    for (const void* k : kernels) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)max_dynamic_lds);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t batch_occupancy(uint32_t threads, size_t lds, bool paired, bool bits, int* blocks_per_cu) {
    const void* k = bits ? (paired ? reinterpret_cast<const void*>(&k_batch_chains<false, true>)
                                   : reinterpret_cast<const void*>(&k_batch_chains_general<false, true>))
                         : (paired ? reinterpret_cast<const void*>(&k_batch_chains<false, false>)
                                   : reinterpret_cast<const void*>(&k_batch_chains_general<false, false>));
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, (int)threads, lds);
}

}  // namespace sd
