// Replica-coded shaken dynamics: multi-spin coding across chains.  Word s of a
// replica lattice holds site s (row-major, s = j L + i) of 64 replicas, bit r
// for replica r (1 = spin +1).  The replicas share the seed and the stream, so
// each site's uniform r_s -- the eight bit-planes of its 64-site group and its
// 24-bit tail, exactly as a single chain draws them -- serves all 64, and
// replica r compares it with its own thresholds T_r (its own J_r, q_r).
// Replica r therefore follows, bit for bit, the single chain at (J_r, q_r) with
// that seed and stream, while the uniforms are drawn once per site instead of
// once per site and chain.
//
// The compare of all replicas with one r_s is a table look-up.  For a leader
// class k and a byte b, LT[k][b] marks the replicas with b < B and EQ[k][b]
// those with b = B, where B is the top byte of T_r[k]; with r_s's top byte b
// the first are decided, the second wait for the tail.  The classes 5 - k have
// the complementary thresholds and are read at 255 - b: r < T is LT's and EQ's
// complement there, equality the same EQ.  Six 16-byte reads and a select by
// class per half word take the place of a scan over eight planes.
//
// A wavefront takes batches of 16 groups (1024 sites).  Its 64 lanes evaluate
// the batch's 64 plane calls (lane 4 g + p: call p of group g), transpose them
// through LDS into the 1024 top bytes, and walk the groups one lane per site.
// Sites with undecided replicas are listed and resolved up to 64 at a time:
// about a quarter of the sites has any, so that a pass over the list keeps most
// lanes busy where a pass over the group would keep a quarter, and the tails
// are drawn for the listed sites alone.  A pass decides all undecided replicas
// of a class together, by r_s's position among the class's ordered thresholds:
// replicas whose thresholds share a top byte (strongly ordered classes: 0x00 or
// 0xFF) are undecided together at every site whose top byte matches.
//
// The LDS reads of the tables (random rows: half of their cycles are bank
// conflicts), the vector unit and the memory traffic (three reads, one write)
// each take 50 to 70% of the time.  64 chains of 2048^2: 34 -> 22.4 us per
// half-step (the scan with its tails in the site's own lane: 34; tables with
// the same tails: 26.2), of which 14 us is the traffic at the rate of a copy;
// 512^2, where a batch is two groups: 15.6 -> 6.8 us (14.2 in full batches).
// 8^2 is one group, whose tables cost more than the scan did (4.7 us against
// 3.9), in calls that their launches bound (4 steps 37.3 and 38.2 us).
#include "sd_replica.hpp"

namespace sd {

namespace {

constexpr uint32_t kBatch = 16;   // groups per batch: 16 groups x 4 plane calls = one call per lane
constexpr uint32_t kWaves = 8;    // wavefronts per workgroup of the half-step: one table serves all
constexpr uint32_t kMinWaves = 2048;   // wavefronts below which a batch is halved: two per SIMD
constexpr uint32_t kList = 64;    // listed sites of a wavefront: one pass resolves a full list

// Immediates of V_BITOP3: the function applied bitwise to the operand patterns
// 0xF0, 0xCC, 0xAA.
constexpr uint32_t kTA = 0xF0u, kTB = 0xCCu, kTC = 0xAAu;
constexpr uint32_t tt3(uint32_t f) { return f & 0xFFu; }
constexpr uint32_t kAllEqual = tt3(~((kTA ^ kTB) | (kTA ^ kTC)));
constexpr uint32_t kMajority = tt3((kTA & kTB) | (kTA & kTC) | (kTB & kTC));
constexpr uint32_t kSelect = tt3((kTA & kTB) | (~kTA & kTC));   // a ? b : c
constexpr uint32_t kNorAnd = tt3(~(kTA | kTB) & kTC);           // ~(a | b) & c
constexpr uint32_t kXorAnd = tt3((kTA ^ kTB) & kTC);            // (a ^ b) & c
constexpr uint32_t kXorOr = tt3((kTA ^ kTB) | kTC);             // (a ^ b) | c
constexpr uint32_t kXorAndNot = tt3((kTA ^ kTB) & ~kTC);        // (a ^ b) & ~c
constexpr uint32_t kAndOr = tt3((kTA & kTB) | kTC);             // a & b | c
constexpr uint32_t kAndNotOr = tt3((kTA & ~kTB) | kTC);         // a & ~b | c

template <uint32_t TT>
__device__ __forceinline__ uint32_t op3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}

__device__ __forceinline__ void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint64_t word64(uint32_t lo, uint32_t hi) { return (uint64_t)lo | ((uint64_t)hi << 32); }

// Transposes the 8 x 8 bit matrix whose row k is byte k of (hi:lo).
__device__ __forceinline__ void transpose8(uint32_t& lo, uint32_t& hi) {
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        uint32_t& x = w ? hi : lo;
        uint32_t t = op3<kXorAnd>(x, x >> 7, 0x00AA00AAu);
        x = xor3(x, t, t << 7);
        t = op3<kXorAnd>(x, x >> 14, 0x0000CCCCu);
        x = xor3(x, t, t << 14);
    }
    const uint32_t m = 0x0F0F0F0Fu;
    const uint32_t a = op3<kSelect>(m, lo, hi << 4);
    hi = op3<kSelect>(m, lo >> 4, hi);
    lo = a;
}

struct Listed {   // the listed sites of one wavefront
    uint4 u_n1[kList], n2_c[kList];
    uint2 lt[kList], site_top[kList];
};

// Per leader class: the replicas' thresholds in ascending order, and the
// replicas from each position on.
struct Order {
    uint32_t T[3][kReplicas];
    uint64_t from[3][kReplicas + 1];
};

// Decides the undecided replicas of the `count` listed sites, one site per
// lane, and stores the sites' words.  All undecided replicas of one class are
// decided together: the thresholds above x (r_s, or its complement for the
// classes 5 - k) are the replicas from x's position in the class's order on.
__device__ __forceinline__ void resolve_listed(const Listed& list, uint32_t count, uint32_t lane,
                                               uint64_t* __restrict__ dst, const DrawParams& dp, const Order& order) {
    lds_wave_sync();
    const uint32_t at = lane < count ? lane : 0u;
    const uint4 a = list.u_n1[at], b = list.n2_c[at];
    const uint2 l = list.lt[at], st = list.site_top[at];
    const uint32_t n1[2] = {a.z, a.w}, n2[2] = {b.x, b.y}, c[2] = {b.z, b.w};
    uint32_t u[2] = {a.x, a.y}, lt[2] = {l.x, l.y};
    const U4 y = philox10_uuuv(dp.stream, dp.t, dp.tag2 + 1u, st.x >> 2, dp.key0, dp.key1);
    const uint32_t yl = (st.x & 1u) ? y.x1 : y.x0, yh = (st.x & 1u) ? y.x3 : y.x2;
    const uint32_t r = ((((st.x & 2u) ? yh : yl)) >> 8) | (st.y << 24);
    while (__any((u[0] | u[1]) != 0u)) {
        // the class of the first undecided replica; a lane with none decides none
        const bool low = u[0] != 0u;
        const uint32_t bit = (uint32_t)__builtin_ctz(low ? u[0] : u[1] | 0x80000000u);
        const uint32_t b1 = (uint32_t)__builtin_amdgcn_sbfe(low ? n1[0] : n1[1], bit, 1u);
        const uint32_t b2 = (uint32_t)__builtin_amdgcn_sbfe(low ? n2[0] : n2[1], bit, 1u);
        const uint32_t bc = (uint32_t)__builtin_amdgcn_sbfe(low ? c[0] : c[1], bit, 1u);
        const uint32_t d = b1 ^ b2;
        const uint32_t nl = op3<kMajority>(b1, b2, bc);
        const uint32_t k = d ? 2u : (b1 == bc ? 0u : 1u);
        // x's position: the number of thresholds <= x
        const uint32_t x = r ^ nl;
        const uint32_t* T = order.T[k];
        uint32_t pos = 0;
#pragma unroll
        for (uint32_t step = kReplicas / 2; step; step >>= 1)
            pos += T[pos + step - 1u] <= x ? step : 0u;
        pos += T[pos] <= x ? 1u : 0u;
        const uint64_t above = order.from[k][pos];
        const uint32_t plus[2] = {lo32(above) ^ nl, hi32(above) ^ nl};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // the undecided replicas of that class: n1 + n2 and c alike
            const uint32_t other = op3<kXorOr>(c[h], bc, xor3(n1[h], n2[h], d)) | op3<kXorAndNot>(n1[h], b1, d);
            const uint32_t same = u[h] & ~other;
            lt[h] = op3<kAndOr>(same, plus[h], lt[h]);
            u[h] &= other;
        }
    }
    if (lane < count)
        dst[st.x] = word64(lt[0], lt[1]);
    lds_wave_sync();
}

template <int WHICH>
__global__ __launch_bounds__(64 * kWaves) void k_replica_half(const uint64_t* __restrict__ src,
                                                             uint64_t* __restrict__ dst, uint32_t L, FastDiv divL,
                                                             uint32_t n_groups, uint32_t batch, DrawParams dp,
                                                             ReplicaParams rp) {
    __shared__ uint4 table[3][256];                   // LT (x, y) and EQ (z, w)
    __shared__ Order order;
    __shared__ uint4 tops[kWaves][64];                // the batch's plane words, then its top bytes
    __shared__ Listed lists[kWaves];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: loop bounds stay scalar

    const char* tab = reinterpret_cast<const char*>(&table[0][0]);
    uint8_t* top = reinterpret_cast<uint8_t*>(&tops[wave][0]);
    Listed& list = lists[wave];
    uint32_t listed = 0;   // wavefront-uniform
    const uint32_t i_step = 64u % L;
    const uint64_t n_sites = (uint64_t)n_groups * 64u;

    // The words of a group are loaded one group ahead of their use.  The
    // addresses are a uniform base and the lane; a row's first or last column
    // and the first or last row wrap.  i: this lane's column.
    uint32_t i = 0;
    uint64_t nc = 0, nn1 = 0, nn2 = 0;
    auto load = [&](uint32_t g) __attribute__((always_inline)) {
        const uint64_t s0 = (uint64_t)g * 64u;
        const uint64_t* at = src + s0;
        nc = at[lane];
        if (WHICH == 0) {
            if (s0 >= L) {
                nn1 = (at - L)[lane];
            } else {
                asm volatile("");   // a branch of its own: not selected lane by lane
                nn1 = at[(int64_t)lane - (int64_t)L + (s0 + lane < L ? (int64_t)n_sites : 0)];
            }
            nn2 = (at - 1)[lane + (i == 0 ? L : 0u)];
        } else {
            if (s0 + 64u + L <= n_sites) {
                nn1 = (at + L)[lane];
            } else {
                asm volatile("");
                nn1 = at[(int64_t)lane + (int64_t)L - (s0 + lane + L >= n_sites ? (int64_t)n_sites : 0)];
            }
            nn2 = (at + 1 - L)[lane + (i == L - 1u ? 0u : L)];
        }
        i += i_step;
        i = i < i - L ? i : i - L;   // i mod L: i - L wraps to a large value while i < L
    };
    // the top bytes of a batch, and its first group's words
    auto begin = [&](uint32_t b0) __attribute__((always_inline)) {
        const uint32_t s = 64u * b0 + lane;
        i = s - fdiv(s, divL) * L;
        load(b0);
        // plane call (lane & 3) of group b0 + (lane >> 2): planes 2 p and 2 p + 1, words of sites 0..31, 32..63
        const U4 x = philox10_uuuv(dp.stream, dp.t | ((lane & 3u) << 30), dp.tag2, b0 + (lane >> 2), dp.key0, dp.key1);
        // component t: the sites 16 t .. 16 t + 15 of both planes, for lane t of the four that share the group
        tops[wave][lane] = make_uint4(
            __builtin_amdgcn_perm(x.x2, x.x0, 0x05040100u), __builtin_amdgcn_perm(x.x2, x.x0, 0x07060302u),
            __builtin_amdgcn_perm(x.x3, x.x1, 0x05040100u), __builtin_amdgcn_perm(x.x3, x.x1, 0x07060302u));
        lds_wave_sync();
        uint32_t e[4];
        const uint32_t* d = reinterpret_cast<const uint32_t*>(&tops[wave][lane & 60u]) + (lane & 3u);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            e[p] = d[4 * p];
        lds_wave_sync();
        // row k of a matrix is plane 7 - k of eight sites: bit k of a site's byte
        uint4 y = make_uint4(
            __builtin_amdgcn_perm(e[2], e[3], 0x04060002u), __builtin_amdgcn_perm(e[0], e[1], 0x04060002u),
            __builtin_amdgcn_perm(e[2], e[3], 0x05070103u), __builtin_amdgcn_perm(e[0], e[1], 0x05070103u));
        transpose8(y.x, y.y);
        transpose8(y.z, y.w);
        tops[wave][lane] = y;
        lds_wave_sync();
    };

    // The tables: EQ by one atomic per replica and class, LT as the union of
    // the EQ above, four bytes per lane of one wavefront per class.  The first
    // batch begins between its steps.
    for (uint32_t e = threadIdx.x; e < 3u * 256u; e += 64u * kWaves)
        table[e >> 8][e & 255u] = make_uint4(0u, 0u, 0u, 0u);
    for (uint32_t e = threadIdx.x; e < 3u * kReplicas; e += 64u * kWaves)
        order.T[e / kReplicas][e % kReplicas] = rp.T[e / kReplicas][e % kReplicas];
    for (uint32_t e = threadIdx.x; e < 3u * (kReplicas + 1u); e += 64u * kWaves)
        order.from[e / (kReplicas + 1u)][e % (kReplicas + 1u)] = rp.from[e / (kReplicas + 1u)][e % (kReplicas + 1u)];
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < 3u * kReplicas; e += 64u * kWaves) {
        const uint32_t r = e % kReplicas;
        uint4& at = table[e / kReplicas][rp.top[e / kReplicas][r]];
        atomicOr(r < 32u ? &at.z : &at.w, 1u << (r & 31u));
    }
    const uint32_t n_blocks = gridDim.x;
    // consecutive batches to one XCD (workgroups go to the XCDs in turn): they share rows in its L2
    const uint32_t block = n_blocks % 8u == 0 ? (blockIdx.x % 8u) * (n_blocks / 8u) + blockIdx.x / 8u : blockIdx.x;
    uint32_t b0 = (block * kWaves + wave) * batch;
    if (b0 < n_groups)
        begin(b0);
    __syncthreads();
    if (wave < 3u) {
        uint4* row = &table[wave][4u * lane];
        uint32_t lo = 0, hi = 0;   // the EQ of this lane's four bytes, then of the lanes above
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            lo |= row[b].z;
            hi |= row[b].w;
        }
#pragma unroll
        for (uint32_t d = 1; d < 64u; d <<= 1) {
            const uint32_t l = __shfl_down(lo, d), h = __shfl_down(hi, d);
            lo |= lane + d < 64u ? l : 0u;
            hi |= lane + d < 64u ? h : 0u;
        }
        const uint32_t la = __shfl_down(lo, 1u), ha = __shfl_down(hi, 1u);
        lo = lane < 63u ? la : 0u;
        hi = lane < 63u ? ha : 0u;
#pragma unroll
        for (int b = 3; b >= 0; --b) {
            row[b].x = lo;
            row[b].y = hi;
            lo |= row[b].z;
            hi |= row[b].w;
        }
    }
    __syncthreads();

    while (b0 < n_groups) {
        const uint32_t nb = n_groups - b0 < batch ? n_groups - b0 : batch;
        for (uint32_t gi = 0; gi < nb; ++gi) {
            const uint64_t c = nc, n1 = nn1, n2 = nn2;
            const uint32_t at = (uint32_t)top[64u * gi + lane] << 4;
            if (gi + 1 < nb)
                load(b0 + gi + 1);
            uint4 ta[3], tc[3];   // by class: at the byte and at its complement
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ta[k] = *reinterpret_cast<const uint4*>(tab + 4096 * k + at);
                tc[k] = *reinterpret_cast<const uint4*>(tab + 4096 * k + (at ^ 0xFF0u));
            }
            uint32_t lt2[2], u2[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t a = (uint32_t)(n1 >> (32 * h)), b = (uint32_t)(n2 >> (32 * h)),
                               cc = (uint32_t)(c >> (32 * h));
                const uint32_t q0 = op3<kAllEqual>(a, b, cc);
                const uint32_t q2 = a ^ b;
                const uint32_t nl = op3<kMajority>(a, b, cc);
                auto pick = [&](uint32_t x0, uint32_t x1, uint32_t x2) __attribute__((always_inline)) {
                    return op3<kSelect>(q0, x0, op3<kSelect>(q2, x2, x1));
                };
                const uint32_t lta = h ? pick(ta[0].y, ta[1].y, ta[2].y) : pick(ta[0].x, ta[1].x, ta[2].x);
                const uint32_t eqa = h ? pick(ta[0].w, ta[1].w, ta[2].w) : pick(ta[0].z, ta[1].z, ta[2].z);
                const uint32_t ltc = h ? pick(tc[0].y, tc[1].y, tc[2].y) : pick(tc[0].x, tc[1].x, tc[2].x);
                const uint32_t eqc = h ? pick(tc[0].w, tc[1].w, tc[2].w) : pick(tc[0].z, tc[1].z, tc[2].z);
                u2[h] = op3<kSelect>(nl, eqc, eqa);
                lt2[h] = op3<kAndNotOr>(lta, nl, op3<kNorAnd>(ltc, eqc, nl));
            }
            const uint32_t s = 64u * (b0 + gi) + lane;
            const bool open = (u2[0] | u2[1]) != 0u;
            const uint64_t mask = __ballot(open);
            const uint32_t more = (uint32_t)__popcll(mask);
            if (listed + more > kList) {
                resolve_listed(list, listed, lane, dst, dp, order);
                listed = 0;
            }
            if (open) {
                const uint32_t e = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, listed));
                list.u_n1[e] = make_uint4(u2[0], u2[1], lo32(n1), hi32(n1));
                list.n2_c[e] = make_uint4(lo32(n2), hi32(n2), lo32(c), hi32(c));
                list.lt[e] = make_uint2(lt2[0], lt2[1]);
                list.site_top[e] = make_uint2(s, at >> 4);
            } else {
                dst[s] = word64(lt2[0], lt2[1]);
            }
            listed += more;
        }
        b0 += n_blocks * kWaves * batch;
        if (b0 < n_groups)
            begin(b0);
    }
    if (listed)
        resolve_listed(list, listed, lane, dst, dp, order);
}

// Sites per lane of k_replica_observe, taken four at a time.  The bit-sliced
// counters have kObsPlanes planes: a lane's count fits.
constexpr uint32_t kObsSites = 32;
constexpr uint32_t kObsPlanes = 6;
constexpr uint32_t kObsThreads = 512;
// words between the numbers of two quantities: the sixteen lanes of each read other banks
constexpr uint32_t kObsStride = 64u * kObsPlanes + 16u;
static_assert(kObsSites < (1u << kObsPlanes) && kObsSites % 4u == 0, "lane counts");

__device__ __forceinline__ void full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t& sum, uint32_t& carry) {
    sum = xor3(a, b, c);
    carry = op3<kMajority>(a, b, c);
}

// All 64 replicas' (M, A, B) in one pass over the sites.  Four quantities are
// counted per replica: +1 spins, sigma != tau_up, sigma != tau_right, sigma !=
// tau.  A lane adds its sites' words four at a time into bit-sliced counters
// (carry-save: one count per replica bit, three operations per word).  The 64
// lanes' counters are added bit-sliced too: every lane leaves its numbers in
// LDS, one half word after the other; lane 16 q + j sums those of lanes j, j +
// 16, ... for quantity q, the sixteen lanes j exchange the rest, and lane j
// reads off two replicas' counts, which the workgroup's wavefronts add up in
// LDS.  The workgroup's contributions are added to out[3 r ...] (zeroed before
// the launch).
// Bound by memory (both lattices are read once; 11 us at 2048^2) and by the
// atomics that all workgroups send to the same counts: with as many sites per
// lane as leave one workgroup per CU, and consecutive lanes on consecutive
// counts, 2048^2 takes 20.5 us (84 with a ripple counter per site; 46 with
// workgroups of 256 lanes and one lane per replica at the end).
__global__ __launch_bounds__(kObsThreads) void k_replica_observe(const uint64_t* __restrict__ sig,
                                                                 const uint64_t* __restrict__ tau, uint32_t L,
                                                                 FastDiv divL, int64_t* __restrict__ out) {
    __shared__ uint32_t nums[kObsThreads / 64][4 * kObsStride];
    __shared__ uint32_t blk[4][kReplicas];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    if (threadIdx.x < 4u * kReplicas)
        blk[threadIdx.x >> 6][threadIdx.x & 63u] = 0u;
    __syncthreads();
    const uint32_t n = L * L;
    const uint32_t s0 = blockIdx.x * (kObsThreads * kObsSites);
    uint32_t P[8][kObsPlanes];   // by 2 q + h
#pragma unroll
    for (int x = 0; x < 8; ++x)
#pragma unroll
        for (uint32_t b = 0; b < kObsPlanes; ++b)
            P[x][b] = 0u;
    // a workgroup with few sites has no more rounds than those take
    const uint32_t rounds = (n - s0 + kObsThreads - 1u) / kObsThreads;
    for (uint32_t k = 0; k < kObsSites && k < rounds; k += 4) {
        uint64_t w[4][4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t s = s0 + kObsThreads * (k + m) + threadIdx.x;
            const bool in = s < n;
            const uint32_t at = in ? s : 0u;
            const uint32_t j = fdiv(at, divL);
            const uint32_t i = at - j * L;
            const uint64_t x = sig[at];
            const uint64_t up = tau[(j == L - 1 ? 0 : j + 1) * L + i];
            const uint64_t right = tau[j * L + (i == L - 1 ? 0 : i + 1)];
            const uint64_t own = tau[at];
            w[m][0] = in ? x : 0ull;
            w[m][1] = in ? x ^ up : 0ull;
            w[m][2] = in ? x ^ right : 0ull;
            w[m][3] = in ? x ^ own : 0ull;
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            uint32_t v[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                v[m] = (uint32_t)(w[m][x >> 1] >> (32 * (x & 1)));
            uint32_t t0, t1, carry;
            full_add(P[x][0], v[0], v[1], P[x][0], t0);
            full_add(P[x][0], v[2], v[3], P[x][0], t1);
            full_add(P[x][1], t0, t1, P[x][1], carry);
#pragma unroll
            for (uint32_t b = 2; b < kObsPlanes; ++b) {
                const uint32_t t = P[x][b] & carry;
                P[x][b] ^= carry;
                carry = t;
            }
        }
    }
    // sums of four lanes here, then over the sixteen lanes j: 6 more planes
    constexpr uint32_t kSumPlanes = kObsPlanes + 6;
    const uint32_t x = lane >> 4, j = lane & 15u;
    uint32_t* my = nums[wave];
#pragma unroll
    for (uint32_t half = 0; half < 2; ++half) {
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
#pragma unroll
            for (uint32_t b = 0; b < kObsPlanes; ++b)
                my[e * kObsStride + 64u * b + lane] = P[2 * e + half][b];
        lds_wave_sync();
        uint32_t S[kSumPlanes];
#pragma unroll
        for (uint32_t b = 0; b < kSumPlanes; ++b)
            S[b] = b < kObsPlanes ? my[x * kObsStride + 64u * b + j] : 0u;
#pragma unroll
        for (uint32_t m = 1; m < 4; ++m) {
            uint32_t carry = 0;
#pragma unroll
            for (uint32_t b = 0; b < kObsPlanes + 2; ++b)
                full_add(S[b], b < kObsPlanes ? my[x * kObsStride + 64u * b + 16u * m + j] : 0u, carry, S[b], carry);
        }
        lds_wave_sync();
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d) {
            uint32_t carry = 0;
#pragma unroll
            for (uint32_t b = 0; b < kObsPlanes + 3 + d; ++b)
                full_add(S[b], (uint32_t)__shfl_xor((int)S[b], 1 << d), carry, S[b], carry);
        }
#pragma unroll
        for (uint32_t e = 0; e < 2; ++e) {
            const uint32_t r = 2u * j + e;
            uint32_t count = 0;
#pragma unroll
            for (uint32_t b = 0; b < kSumPlanes; ++b)
                count |= ((S[b] >> r) & 1u) << b;
            atomicAdd(&blk[x][32u * half + r], count);
        }
    }
    __syncthreads();
    // consecutive lanes add to consecutive counts: a wavefront's atomics share their cache lines
    for (uint32_t e = threadIdx.x; e < 3u * kReplicas; e += kObsThreads) {
        const uint32_t r = e / 3u, k = e % 3u;
        const uint32_t end = s0 + kObsThreads * kObsSites < n ? s0 + kObsThreads * kObsSites : n;
        const int64_t N = end > s0 ? (int64_t)(end - s0) : 0;
        const int64_t add = k == 0 ? 2 * (int64_t)blk[0][r] - N
                            : k == 1 ? 2 * N - 2 * ((int64_t)blk[1][r] + (int64_t)blk[2][r])
                                     : N - 2 * (int64_t)blk[3][r];
        atomicAdd(reinterpret_cast<unsigned long long*>(out + e), (unsigned long long)add);
    }
}

}  // namespace

hipError_t launch_replica_half(int which, const uint64_t* src, uint64_t* dst, uint32_t L, const DrawParams& dp,
                               const ReplicaParams& rp, hipStream_t st) {
    const uint32_t n_groups = (uint32_t)(((uint64_t)L * L) / 64u);
    // Full batches leave a small lattice with few wavefronts, each with its
    // groups one after the other: the batch shrinks until there are two per
    // SIMD (half-steps at 512^2 and 1024^2: 6.8 and 10.3 us; 7.5 and 15.1 with
    // one per SIMD, 7.6 and 10.4 with four).
    uint32_t batch = kBatch;
    while (batch > 1u && n_groups / batch < kMinWaves)
        batch /= 2u;
    const uint32_t batches = (n_groups + batch - 1) / batch;
    uint32_t blocks = (batches + kWaves - 1) / kWaves;
    if (blocks > 4096u)
        blocks = 4096u;
    const FastDiv divL = make_fastdiv(L);
    if (which == 0)
        hipLaunchKernelGGL(k_replica_half<0>, dim3(blocks), dim3(64 * kWaves), 0, st, src, dst, L, divL, n_groups,
                           batch, dp, rp);
    else
        hipLaunchKernelGGL(k_replica_half<1>, dim3(blocks), dim3(64 * kWaves), 0, st, src, dst, L, divL, n_groups,
                           batch, dp, rp);
    return hipGetLastError();
}

hipError_t launch_replica_observe(const uint64_t* sigma, const uint64_t* tau, uint32_t L, int64_t* out,
                                  hipStream_t st) {
    hipError_t e = launch_fill_i64(out, 3 * kReplicas, 0, st);
    if (e != hipSuccess)
        return e;
    const uint32_t n = L * L;
    const uint32_t per_block = kObsThreads * kObsSites;
    hipLaunchKernelGGL(k_replica_observe, dim3((n + per_block - 1) / per_block), dim3(kObsThreads), 0, st, sigma, tau, L,
                       make_fastdiv(L), out);
    return hipGetLastError();
}

}  // namespace sd
