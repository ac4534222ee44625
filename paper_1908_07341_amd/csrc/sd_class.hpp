// Class masks: the bits r_s < T[k] of a word's sites for every class k, drawn
// before the lattice is known (k_small.hip, k_ahead.hip).
#pragma once

#include "sd_device.hpp"

namespace sd {

__device__ __forceinline__ void class_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Philox4x32-10 with lane-varying second and fourth counter words (a tile of
// words covers several half-steps).  Rounds 1-3 in plain products, so that
// the four plane calls of a word share what does not depend on the plane.
__device__ __forceinline__ U4 philox10_uvuv(uint32_t u0, uint32_t v1, uint32_t u2, uint32_t v3, uint32_t k0,
                                            uint32_t k1) {
    const uint64_t a0 = (uint64_t)kPhiloxM0 * u0;
    const uint64_t a1 = (uint64_t)kPhiloxM1 * u2;
    U4 c;
    c.x0 = (hi32(a1) ^ k0) ^ v1;
    c.x1 = lo32(a1);
    c.x2 = (hi32(a0) ^ k1) ^ v3;
    c.x3 = lo32(a0);
#pragma unroll
    for (int r = 1; r < 10; ++r) {
        k0 += kPhiloxW0;
        k1 += kPhiloxW1;
        if (r < 3) {
            const uint64_t p0 = (uint64_t)kPhiloxM0 * c.x0;
            const uint64_t p1 = (uint64_t)kPhiloxM1 * c.x2;
            c = U4{hi32(p1) ^ (c.x1 ^ k0), lo32(p1), hi32(p0) ^ (c.x3 ^ k1), lo32(p0)};
        } else {
            c = philox_round(c, k0, k1);
        }
    }
    return c;
}

// Truth tables (operand patterns 0xF0, 0xCC, 0xAA): less-than from the least
// significant bit up, lt' = r bit 0 and threshold bit 1, or bits equal and lt;
// equality so far; select b where a else c.
constexpr uint32_t kLess = ((~kBopA & kBopB) | (~(kBopA ^ kBopB) & kBopC)) & 0xFFu;   // (r, threshold, lt)
constexpr uint32_t kEqual = (~(kBopA ^ kBopB) & kBopC) & 0xFFu;                      // (r, threshold, eq)
constexpr uint32_t kPick = ((kBopA & kBopB) | (~kBopA & kBopC)) & 0xFFu;             // (select, b, c)

template <uint32_t TT>
__device__ __forceinline__ uint32_t class_op3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}

// A wavefront's scratch of one tile: the sites of each lane's word whose top
// byte equals class k's, and the list of sites whose tails are to be drawn.
constexpr uint32_t kClassListCap = 128;
struct ClassList {
    uint64_t eq[6][64];
    uint32_t entry[kClassListCap];   // lane | bit << 6
};

// Draws the tails of the n listed sites of a tile and adds the decided sites
// to the class masks.  at(l, t, g, m): half-step index, stream group and mask
// word (class 0; class k is k * stride further) of the tile's lane l.
template <class At>
__device__ __forceinline__ void class_tails(uint32_t key0, uint32_t key1, uint32_t stream, uint32_t rng_xor,
                                            const uint32_t (&T24)[6], ClassList& w, uint32_t n, uint32_t stride,
                                            const At& at) {
    class_sync();
    for (uint32_t e = threadIdx.x & 63u; e < n; e += 64u) {
        const uint32_t v = w.entry[e];
        const uint32_t l = v & 63u, b = v >> 6;
        uint32_t t, g;
        uint64_t* m64;
        at(l, t, g, m64);
        const U4 y = philox10_uvuv(stream, t, 2u * kTagDynamics + 1u, 16u * g + (b >> 2), key0, key1);
        const uint32_t lo = (b & 1u) ? y.x1 : y.x0, hi = (b & 1u) ? y.x3 : y.x2;
        const uint32_t tail = (((b & 2u) ? hi : lo) ^ rng_xor) >> 8;
        const uint32_t bit = 1u << (b & 31u);
        lds_dword* m = reinterpret_cast<lds_dword*>(m64) + (b >> 5);
        const lds_dword* q = reinterpret_cast<const lds_dword*>(&w.eq[0][l]) + (b >> 5);
        uint32_t open[6];
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k)
            open[k] = q[128u * k] & bit;
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k)   // or-ing nothing costs less than a branch per class
            atomicOr(m + 2u * k * stride, tail < T24[k] ? open[k] : 0u);
    }
    class_sync();
}

// The class masks of the tile's words: this lane's is group g at half-step
// index t, its masks go to out[k * stride] (LDS).  Sites whose top byte equals
// a threshold's are listed and their tails drawn one per lane.  UNIFORM_T: t is the same for the whole wavefront.
template <bool UNIFORM_T, class At>
__device__ __forceinline__ void class_masks(uint32_t key0, uint32_t key1, uint32_t stream, uint32_t t, uint32_t g,
                                            uint32_t rng_xor, const uint32_t* Tk, bool active, ClassList& w,
                                            uint64_t* out, uint32_t stride, const At& at) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t P[8][2];
#pragma unroll
    for (uint32_t p = 0; p < 4; ++p) {
        const U4 y = UNIFORM_T ? philox10_uuuv(stream, t | (p << 30), 2u * kTagDynamics, g, key0, key1)
                               : philox10_uvuv(stream, t | (p << 30), 2u * kTagDynamics, g, key0, key1);
        P[2 * p][0] = y.x0;
        P[2 * p][1] = y.x1;
        P[2 * p + 1][0] = y.x2;
        P[2 * p + 1][1] = y.x3;
    }
    if (rng_xor) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            P[m][0] = ~P[m][0];
            P[m][1] = ~P[m][1];
        }
    }
    uint64_t open = 0;   // sites some class leaves to its tail
    uint32_t T24[6];
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k) {
        uint32_t lt[2] = {0u, 0u}, eq[2] = {~0u, ~0u};
        // the 48 threshold bits are formed where they are used, on the
        // scalar unit: kept across the tile they would not fit its registers
        uint32_t T = Tk[k];
        asm volatile("" : "+s"(T));
#pragma unroll
        for (int m = 7; m >= 0; --m) {
            const uint32_t S = 0u - ((T >> (31 - m)) & 1u);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                lt[h] = class_op3<kLess>(P[m][h], S, lt[h]);
                eq[h] = class_op3<kEqual>(P[m][h], S, eq[h]);
            }
        }
        const uint64_t e = (uint64_t)eq[0] | ((uint64_t)eq[1] << 32);
        w.eq[k][lane] = e;
        T24[k] = T & 0xFFFFFFu;
        if (T24[k])   // uniform; no tail is below a zero threshold tail
            open |= e;
        if (active)
            out[k * stride] = (uint64_t)lt[0] | ((uint64_t)lt[1] << 32);
    }
    if (!active)
        open = 0;
    // Each lane writes its sites behind those of the lanes before it: five or
    // six rounds of 7 operations, where a round of ballots takes 14 and two
    // trips to the scalar unit (512 samples of 32^2: 10.9 -> 9.4 ms).
    uint32_t half[2] = {lo32(open), hi32(open)};
    const uint32_t mine = (uint32_t)__popcll(open);
    const uint32_t upto = wave_prefix_dpp(mine);
    const uint32_t sites = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    if (sites <= kClassListCap) {
        uint32_t e = upto - mine;
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h)
            for (; half[h]; half[h] &= half[h] - 1u)
                w.entry[e++] = lane | ((uint32_t)__builtin_ctz(half[h]) << 6) | (h << 11);
        if (sites)
            class_tails(key0, key1, stream, rng_xor, T24, w, sites, stride, at);
        return;
    }
    // more than the list holds: one site per lane and round, emptied in between
    uint32_t listed = 0;   // wavefront-uniform
    for (;;) {
        const uint64_t m = __ballot(open != 0);
        if (m == 0)
            break;
        if (open != 0) {
            const uint32_t e = listed + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            w.entry[e] = lane | ((uint32_t)__builtin_ctzll(open) << 6);
            open &= open - 1;
        }
        listed += (uint32_t)__popcll(m);
        if (listed >= 64u) {
            class_tails(key0, key1, stream, rng_xor, T24, w, listed, stride, at);
            listed = 0;
        }
    }
    if (listed)
        class_tails(key0, key1, stream, rng_xor, T24, w, listed, stride, at);
}

// A word's class masks, and its new word given its spins c and neighbours.
struct ClassMasks {
    uint64_t m[6];
};

__device__ __forceinline__ uint64_t pick_class(const ClassMasks& r, uint64_t c, uint64_t n1, uint64_t n2) {
    uint32_t out[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t cc = (uint32_t)(c >> (32 * h)), a = (uint32_t)(n1 >> (32 * h)), b = (uint32_t)(n2 >> (32 * h));
        const uint32_t one = a ^ b;   // exactly one J-neighbour is +1 (k = 1); else a tells k = 0 from k = 2
        uint32_t m[6];
#pragma unroll
        for (int k = 0; k < 6; ++k)
            m[k] = (uint32_t)(r.m[k] >> (32 * h));
        const uint32_t down = class_op3<kPick>(one, m[2], class_op3<kPick>(a, m[4], m[0]));
        const uint32_t up = class_op3<kPick>(one, m[3], class_op3<kPick>(a, m[5], m[1]));
        out[h] = class_op3<kPick>(cc, up, down);
    }
    return (uint64_t)out[0] | ((uint64_t)out[1] << 32);
}

// Neighbour words n1 (down / up) and n2 (left / right) of lattices whose rows
// are whole (ROWS 64, lane l holding row l) or half words (ROWS 32, lane l
// holding rows 2 (l % 16) and 2 (l % 16) + 1), from the other lanes' registers.
template <int ROWS, int WHICH>
__device__ __forceinline__ void row_neighbours(uint64_t c, uint64_t& n1, uint64_t& n2) {
    static_assert(ROWS == 64 || ROWS == 32, "rows of one word or half a word");
    const uint32_t lo = (uint32_t)c, hi = (uint32_t)(c >> 32);
    auto pack = [](uint32_t l, uint32_t h) { return (uint64_t)l | ((uint64_t)h << 32); };
    if constexpr (ROWS == 64) {
        if constexpr (WHICH == 0) {   // wave_ror:1, lane l takes lane l - 1 mod 64
            n1 = pack((uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x13C, 0xF, 0xF, true),
                      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x13C, 0xF, 0xF, true));
            n2 = pack(__builtin_amdgcn_alignbit(lo, hi, 31), __builtin_amdgcn_alignbit(hi, lo, 31));
        } else {                      // wave_rol:1
            n1 = pack((uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x134, 0xF, 0xF, true),
                      (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x134, 0xF, 0xF, true));
            n2 = pack(__builtin_amdgcn_alignbit(hi, lo, 1), __builtin_amdgcn_alignbit(lo, hi, 1));
        }
    } else {
        if constexpr (WHICH == 0) {   // row_ror:1, lane l takes lane l - 1 mod 16
            n1 = pack((uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x121, 0xF, 0xF, true), lo);
            n2 = pack(__builtin_amdgcn_alignbit(lo, lo, 31), __builtin_amdgcn_alignbit(hi, hi, 31));
        } else {                      // row_ror:15, lane l takes lane l + 1 mod 16
            n1 = pack(hi, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x12F, 0xF, 0xF, true));
            n2 = pack(__builtin_amdgcn_alignbit(lo, lo, 1), __builtin_amdgcn_alignbit(hi, hi, 1));
        }
    }
}

}  // namespace sd
