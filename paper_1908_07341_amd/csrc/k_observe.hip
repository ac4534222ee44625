// Reductions over lattices: the pair observables M, A, B and the row-wise
// spin-spin correlation sums D(r).
//
// M = sum_x sigma_x (magnetisation times L^2, section 3.1), and from the pair
// Hamiltonian of eq. (5): A = sum_x sigma_x (tau_up + tau_right),
// B = sum_x sigma_x tau_x, so that H(sigma, tau) = -(J A + q B).  With bit
// 1 = +1, a product of two spins is +1 exactly when their bits agree, so every
// sum is n - 2 * popcount(xor) over the n sites involved: exact integers.
//
// D(r) = sum_x sigma_(i,j) sigma_(i+r,j): the row-wise analogue of the
// correlations of Table 1.  Each row is staged in LDS as a bit string followed
// by a second copy of itself, so that the row rotated by r is a plain funnel
// shift of two LDS words for every r.
#include "sd_kernels.hpp"

namespace sd {

namespace {

__device__ __forceinline__ void add_obs(int64_t* out3, int64_t pc, int64_t dpair, int64_t dself, int64_t n,
                                        int64_t* red) {
    int64_t v[4] = {pc, dpair, dself, n};
    block_sum_i64<4>(v, red);
    if (threadIdx.x == 0) {
        atomicAdd(reinterpret_cast<unsigned long long*>(out3 + 0), (unsigned long long)(2 * v[0] - v[3]));
        atomicAdd(reinterpret_cast<unsigned long long*>(out3 + 1), (unsigned long long)(2 * v[3] - 2 * v[1]));
        atomicAdd(reinterpret_cast<unsigned long long*>(out3 + 2), (unsigned long long)(v[3] - 2 * v[2]));
    }
}

// Packed layouts (L % 32 == 0): one lane per 32-bit word.
__global__ __launch_bounds__(256) void k_observe_packed(const uint32_t* __restrict__ sigma,
                                                         const uint32_t* __restrict__ tau, Geom G,
                                                         int64_t* __restrict__ out3) {
    __shared__ int64_t red[4 * 4];
    const uint32_t W = G.L / 32u;
    const uint32_t n_words = G.n_sites / 32u;
    int64_t pc = 0, dpair = 0, dself = 0, n = 0;
    for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < n_words; u += gridDim.x * blockDim.x) {
        const uint32_t j = fdiv(u, G.div_row);
        const uint32_t w = u - j * W;
        const uint32_t s = sigma[u];
        const uint32_t t = tau[u];
        const uint32_t up = tau[(j == G.L - 1 ? 0 : j + 1) * W + w];
        const uint32_t next = tau[j * W + (w == W - 1 ? 0 : w + 1)];
        const uint32_t right = (t >> 1) | (next << 31);
        pc += __popc(s);
        dpair += __popc(s ^ up) + __popc(s ^ right);
        dself += __popc(s ^ t);
        n += 32;
    }
    add_obs(out3, pc, dpair, dself, n, red);
}

// Bit-string layout (any L % 8 == 0): one lane per 64-bit word, the up and
// right neighbour words as windows of tau.
__global__ __launch_bounds__(256) void k_observe_bits(const uint64_t* __restrict__ sigma,
                                                       const uint64_t* __restrict__ tau, Geom G,
                                                       int64_t* __restrict__ out3) {
    __shared__ int64_t red[4 * 4];
    int64_t pc = 0, dpair = 0, dself = 0, n = 0;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < G.n_groups; g += gridDim.x * blockDim.x) {
        uint64_t t, up, right;
        gather_bits<1>(tau, G.L, G.n_groups, G.div_L, g, t, up, right);
        const uint64_t sg = sigma[g];
        pc += __popcll(sg);
        dpair += __popcll(sg ^ up) + __popcll(sg ^ right);
        dself += __popcll(sg ^ t);
        n += 64;
    }
    add_obs(out3, pc, dpair, dself, n, red);
}

__device__ __forceinline__ uint32_t string_bit(const uint64_t* lat, size_t s) {
    return (uint32_t)(lat[s >> 6] >> (s & 63u)) & 1u;
}

// int8 layout, any L: one lane per site.
__global__ __launch_bounds__(256) void k_observe_i8(const int8_t* __restrict__ sigma, const int8_t* __restrict__ tau,
                                                     Geom G, int64_t* __restrict__ out3) {
    __shared__ int64_t red[4 * 4];
    int64_t pc = 0, dpair = 0, dself = 0, n = 0;
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < G.n_sites; s += gridDim.x * blockDim.x) {
        const uint32_t j = fdiv(s, G.div_L);
        const uint32_t i = s - j * G.L;
        const int sx = sigma[s] > 0;
        const int tx = tau[s] > 0;
        const int up = tau[(size_t)(j == G.L - 1 ? 0 : j + 1) * G.L + i] > 0;
        const int right = tau[(size_t)j * G.L + (i == G.L - 1 ? 0 : i + 1)] > 0;
        pc += sx;
        dpair += (sx ^ up) + (sx ^ right);
        dself += sx ^ tx;
        n += 1;
    }
    add_obs(out3, pc, dpair, dself, n, red);
}

// Bits of one row, followed by a second copy, in LDS words (bit p of the
// string is bit p % 32 of word p / 32).
constexpr uint32_t kCorrMaxL = 65535;
constexpr uint32_t kCorrWords = (2 * kCorrMaxL + 64) / 32 + 2;

template <int PACKED>
__device__ __forceinline__ void stage_row(const void* sigma, const Geom& G, uint32_t j, uint32_t* row, uint32_t nw2) {
    if constexpr (PACKED == 2) {
        const uint64_t* s = static_cast<const uint64_t*>(sigma);
        const size_t row0 = (size_t)j * G.L;
        for (uint32_t k = threadIdx.x; k < nw2; k += blockDim.x) {
            uint32_t word = 0;
            uint32_t col = (uint32_t)(((uint64_t)32u * k) % G.L);
            for (int b = 0; b < 32; ++b) {
                word |= string_bit(s, row0 + col) << b;
                if (++col == G.L)
                    col = 0;
            }
            row[k] = word;
        }
    } else if constexpr (PACKED) {
        const uint32_t* s = static_cast<const uint32_t*>(sigma);
        const uint32_t W = G.L / 32u;
        for (uint32_t k = threadIdx.x; k < nw2; k += blockDim.x)
            row[k] = s[(size_t)j * W + (k % W)];
    } else {
        const int8_t* s = static_cast<const int8_t*>(sigma) + (size_t)j * G.L;
        for (uint32_t k = threadIdx.x; k < nw2; k += blockDim.x) {
            uint32_t word = 0;
            uint32_t col = (uint32_t)(((uint64_t)32u * k) % G.L);
            for (int b = 0; b < 32; ++b) {
                word |= (uint32_t)(s[col] > 0) << b;
                if (++col == G.L)
                    col = 0;
            }
            row[k] = word;
        }
    }
}

// out[r] += sum over the block's rows of D_row(r), r = blockIdx.x * blockDim.x + tid.
template <int PACKED>
__global__ __launch_bounds__(256) void k_corr_row(const void* __restrict__ sigma, Geom G, int32_t rmax,
                                                   int64_t* __restrict__ out) {
    __shared__ uint32_t row[kCorrWords];
    const uint32_t L = G.L;
    const uint32_t nwr = (L + 31u) / 32u;                 // words covering one row
    const uint32_t nw2 = (2u * L + 63u) / 32u + 1u;       // words of the doubled string
    const uint32_t last_bits = L - 32u * (nwr - 1u);      // valid bits of the last word
    const uint32_t last_mask = last_bits == 32u ? ~0u : ((1u << last_bits) - 1u);
    const int32_t r = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    int64_t acc = 0;
    for (uint32_t j = blockIdx.y; j < L; j += gridDim.y) {
        __syncthreads();
        stage_row<PACKED>(sigma, G, j, row, nw2);
        __syncthreads();
        if (r <= rmax) {
            uint32_t diff = 0;
            for (uint32_t k = 0; k < nwr; ++k) {
                const uint32_t off = 32u * k + (uint32_t)r;
                const uint32_t q = off >> 5, sh = off & 31u;
                const uint32_t rot = sh ? ((row[q] >> sh) | (row[q + 1] << (32u - sh))) : row[q];
                const uint32_t mask = (k == nwr - 1u) ? last_mask : ~0u;
                diff += __popc((row[k] ^ rot) & mask);
            }
            acc += (int64_t)L - 2 * (int64_t)diff;
        }
    }
    if (r <= rmax)
        atomicAdd(reinterpret_cast<unsigned long long*>(out + r), (unsigned long long)acc);
}

// Rows of whole 64-bit words (the packed string with L % 64 == 0, or int8
// rows whose 64-site groups are 16-byte aligned): workgroup (x, y) takes the
// R <= 16 rows from y R on, one per wavefront, and the `chunks` 64-shift chunks
// r = 64 s + lane from s = x chunks on.  A wavefront stages its row in LDS with
// its first words repeated behind it, so that no shift wraps, and for each s
// sums popcount(row ^ row rotated by r) over the W words, the rotation two
// funnel shifts of consecutive dwords (lanes past 31 start one dword later).
// s is uniform, so the LDS reads are broadcasts of at most two dwords.  The
// wavefronts' sums are added in LDS and each r gets one atomic add into out[r]
// (zeroed first) per workgroup.  Several lattices of one size in one launch:
// lattice z = blockIdx.z, its sums at out + z (rmax + 1).
// Bound by the vector unit (6 operations per word, shift and row).  With one
// chunk per workgroup every chunk's workgroups staged the rows again, and 64-bit
// shifts with wrapped indices took 10 operations; us a call before and now: five
// 1024^2 int8 lattices, r <= 512, 32.1 -> 21.5; two of 2048^2, r <= 1024, 68 ->
// 47; 16384^2, r <= 512, 905 -> 529.
constexpr uint32_t kCorr64Words = 6144;   // staged words (48 KB)
constexpr uint32_t kCorrWaves = 16;
constexpr uint32_t kCorrChunks = 16;
constexpr uint32_t kCorrTarget = 1024;   // workgroups aimed at: four per CU

// Rows are staged as 64-bit words and read as dwords.
typedef uint32_t __attribute__((may_alias)) row_dword;

template <bool INT8>
__global__ __launch_bounds__(1024) void k_corr_row64(CorrLattices cl, uint32_t L, uint32_t R, uint32_t chunks,
                                                     int32_t rmax, int64_t* __restrict__ out) {
    __shared__ uint64_t rows[kCorr64Words];
    __shared__ uint32_t tot[kCorrChunks][64];   // differing pairs by shift
    const void* __restrict__ sigma = cl.p[blockIdx.z];
    out += (size_t)blockIdx.z * ((uint32_t)rmax + 1u);
    const uint32_t W = L / 64u;
    const uint32_t over = (uint32_t)rmax / 64u + 1u;   // words repeated behind a row
    const uint32_t pitch = W + over;
    const uint32_t j0 = blockIdx.y * R;
    const uint32_t n = j0 + R < L ? R : L - j0;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t s0 = blockIdx.x * chunks;   // r >> 6 of the first chunk
    const uint32_t s1 = s0 + chunks < over ? s0 + chunks : over;
    if (threadIdx.x < 64u * chunks)
        tot[threadIdx.x >> 6][lane] = 0u;
    __syncthreads();
    for (uint32_t i = wave; i < n; i += kCorrWaves) {
        uint64_t* row = rows + i * pitch;
        for (uint32_t w = lane; w < W; w += 64u) {
            const size_t q = (size_t)(j0 + i) * W + w;
            const uint64_t x = INT8 ? load_bits64_i8(static_cast<const int8_t*>(sigma) + 64u * q)
                                    : static_cast<const uint64_t*>(sigma)[q];
            row[w] = x;
            if (w < over)
                row[W + w] = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const row_dword* own = reinterpret_cast<const row_dword*>(row);
        for (uint32_t s = s0; s < s1; ++s) {
            const row_dword* d = own + 2u * s + (lane >> 5);
            uint32_t diff = 0, before = d[0];
#pragma unroll 8
            for (uint32_t w = 0; w < W; ++w) {
                const uint32_t mid = d[2u * w + 1u], after = d[2u * w + 2u];
                diff += (uint32_t)__popc(own[2u * w] ^ __builtin_amdgcn_alignbit(mid, before, lane & 31u));
                diff += (uint32_t)__popc(own[2u * w + 1u] ^ __builtin_amdgcn_alignbit(after, mid, lane & 31u));
                before = after;
            }
            atomicAdd(&tot[s - s0][lane], diff);
        }
    }
    __syncthreads();
    const uint32_t r = 64u * s0 + threadIdx.x;
    if (threadIdx.x < 64u * (s1 - s0) && r <= (uint32_t)rmax)
        atomicAdd(reinterpret_cast<unsigned long long*>(out + r),
                  (unsigned long long)((int64_t)n * L - 2 * (int64_t)tot[threadIdx.x >> 6][lane]));
}

// Diagonal correlation sums (section 3.3, Table 1).  Block (x, y): direction
// d = x / (lmax + 1) (0: partner (i+l, j+l), SW-NE; 1: partner (i+l, j-l),
// NW-SE) and l = x % (lmax + 1), rows j = y, y + gridDim.y, ..., a row's words
// (or sites) on 2^row_shift neighbouring threads, so that short rows share the
// workgroup; the block's count of unequal pairs goes to out[x] as
// (pairs - 2 * unequal): stored when the block has all the rows (gridDim.y
// == 1: out need not be zeroed first), else added by one atomic.
// Packed: rows are L / 32 words (L % 32 == 0); the partner row's bits from
// column l on are a funnel shift of two of its words.
// Sites are bound by the vector unit: row and column wrap by a compare, as the
// rows of a workgroup's threads differ and a remainder of each took much
// of the time (512^2 int8, l <= 256: 157 -> 94 us).
template <int PACKED>
__global__ __launch_bounds__(256) void k_corr_diag(const void* __restrict__ sigma, Geom G, int32_t lmax,
                                                    uint32_t row_shift, int64_t* __restrict__ out) {
    __shared__ int64_t red[2 * 4];
    const uint32_t L = G.L;
    const uint32_t n_l = (uint32_t)lmax + 1u;
    const uint32_t dir = blockIdx.x / n_l, l = blockIdx.x % n_l;
    int64_t diff = 0, pairs = 0;
    const uint32_t rows = blockDim.x >> row_shift;                 // rows the block takes at once
    const uint32_t cols = 1u << row_shift, col = threadIdx.x & (cols - 1u);
    const uint32_t row0 = blockIdx.y * rows + (threadIdx.x >> row_shift), row_step = gridDim.y * rows;
    auto wrap = [L](uint32_t x) { return x < L ? x : x - L; };   // x mod L for x < 2 L
    if constexpr (PACKED == 1) {
        const uint32_t* s = static_cast<const uint32_t*>(sigma);
        const uint32_t W = L / 32u;
        const uint32_t sh = l & 31u;
        for (uint32_t j = row0; j < L; j += row_step) {
            const uint32_t jp = wrap(dir == 0 ? j + l : j + L - l);
            const uint32_t* row = s + (size_t)j * W;
            const uint32_t* prow = s + (size_t)jp * W;
            for (uint32_t k = col; k < W; k += cols) {
                uint32_t q0 = k + (l >> 5);
                q0 = q0 >= W ? q0 - W : q0;
                const uint32_t q1 = q0 + 1u == W ? 0u : q0 + 1u;
                const uint32_t rot = sh ? ((prow[q0] >> sh) | (prow[q1] << (32u - sh))) : prow[q0];
                diff += __popc(row[k] ^ rot);
                pairs += 32;
            }
        }
    } else {
        for (uint32_t j = row0; j < L; j += row_step) {
            const uint32_t jp = wrap(dir == 0 ? j + l : j + L - l);
            for (uint32_t i = col; i < L; i += cols) {
                const uint32_t ip = wrap(i + l);
                const size_t a = (size_t)j * L + i, b = (size_t)jp * L + ip;
                if constexpr (PACKED == 2) {
                    const uint64_t* s = static_cast<const uint64_t*>(sigma);
                    diff += string_bit(s, a) != string_bit(s, b);
                } else {
                    const int8_t* s = static_cast<const int8_t*>(sigma);
                    diff += (s[a] > 0) != (s[b] > 0);
                }
                pairs += 1;
            }
        }
    }
    int64_t v[2] = {diff, pairs};
    block_sum_i64<2>(v, red);
    if (threadIdx.x == 0 && gridDim.y == 1u)
        out[blockIdx.x] = v[1] - 2 * v[0];
    else if (threadIdx.x == 0)
        atomicAdd(reinterpret_cast<unsigned long long*>(out + blockIdx.x), (unsigned long long)(v[1] - 2 * v[0]));
}

}  // namespace

hipError_t launch_observe(int layout, const void* sigma, const void* tau, const Geom& G, int64_t* out3,
                          hipStream_t st) {
    hipError_t e = launch_fill_i64(out3, 3, 0, st);
    if (e != hipSuccess)
        return e;
    if (layout == kLayBits) {
        uint32_t blocks = (G.n_groups + 255u) / 256u;
        blocks = blocks < kMaxBlocks ? blocks : kMaxBlocks;
        hipLaunchKernelGGL(k_observe_bits, dim3(blocks ? blocks : 1), dim3(256), 0, st,
                           static_cast<const uint64_t*>(sigma), static_cast<const uint64_t*>(tau), G, out3);
    } else if (layout == kLayP64 || layout == kLayP32) {
        uint32_t n_words = G.n_sites / 32u;
        uint32_t blocks = (n_words + 255u) / 256u;
        blocks = blocks < kMaxBlocks ? blocks : kMaxBlocks;
        hipLaunchKernelGGL(k_observe_packed, dim3(blocks ? blocks : 1), dim3(256), 0, st,
                           static_cast<const uint32_t*>(sigma), static_cast<const uint32_t*>(tau), G, out3);
    } else {
        uint32_t blocks = (G.n_sites + 255u) / 256u;
        blocks = blocks < kMaxBlocks ? blocks : kMaxBlocks;
        hipLaunchKernelGGL(k_observe_i8, dim3(blocks ? blocks : 1), dim3(256), 0, st,
                           static_cast<const int8_t*>(sigma), static_cast<const int8_t*>(tau), G, out3);
    }
    return hipGetLastError();
}

hipError_t launch_corr_diag(int layout, const void* sigma, const Geom& G, int32_t lmax, int64_t* out,
                            hipStream_t st) {
    const uint32_t n = 2u * ((uint32_t)lmax + 1u);
    const uint32_t width = layout == kLayP64 || layout == kLayP32 ? G.L / 32u : G.L;   // items of a row
    uint32_t row_shift = 0;
    while (row_shift < 8u && (1u << row_shift) < width)
        ++row_shift;
    // One workgroup per sum up to 8192 words or 6144 sites a lattice: one launch
    // instead of two, no atomics (32^2 packed, l <= 16: 8.8 us with the zeroing
    // and a workgroup per row, 3.4 so); larger lattices split their rows over
    // about kMaxBlocks workgroups (one workgroup against several, l <= 0 and 64:
    // 80^2 int8 10.4 and 10.7 us, 91^2 split 8.5 and 7.8).
    const uint64_t most = layout == kLayP64 || layout == kLayP32 ? 8192u : 6144u;
    uint32_t row_blocks = 1u;
    if ((uint64_t)width * G.L > most) {
        const uint32_t groups = (G.L + (256u >> row_shift) - 1u) / (256u >> row_shift);
        row_blocks = kMaxBlocks / n;
        row_blocks = row_blocks < groups ? row_blocks : groups;
        row_blocks = row_blocks ? row_blocks : 1u;
    }
    if (row_blocks > 1u) {
        const hipError_t e = launch_fill_i64(out, n, 0, st);
        if (e != hipSuccess)
            return e;
    }
    const dim3 grid(n, row_blocks);
    if (layout == kLayBits)
        hipLaunchKernelGGL((k_corr_diag<2>), grid, dim3(256), 0, st, sigma, G, lmax, row_shift, out);
    else if (layout == kLayP64 || layout == kLayP32)
        hipLaunchKernelGGL((k_corr_diag<1>), grid, dim3(256), 0, st, sigma, G, lmax, row_shift, out);
    else
        hipLaunchKernelGGL((k_corr_diag<0>), grid, dim3(256), 0, st, sigma, G, lmax, row_shift, out);
    return hipGetLastError();
}

// Any layout: one lattice, k_corr_row's workgroups over rows and shifts (out
// zeroed by the caller).
static hipError_t launch_corr_row_generic(int layout, const void* sigma, const Geom& G, int32_t rmax, int64_t* out,
                                          hipStream_t st) {
    const uint32_t r_chunks = ((uint32_t)rmax + 256u) / 256u;
    uint32_t row_blocks = kMaxBlocks / r_chunks;
    row_blocks = row_blocks < G.L ? row_blocks : G.L;
    row_blocks = row_blocks ? row_blocks : 1u;
    const dim3 grid(r_chunks, row_blocks);
    if (layout == kLayBits)
        hipLaunchKernelGGL((k_corr_row<2>), grid, dim3(256), 0, st, sigma, G, rmax, out);
    else if (layout == kLayP64 || layout == kLayP32)
        hipLaunchKernelGGL((k_corr_row<1>), grid, dim3(256), 0, st, sigma, G, rmax, out);
    else
        hipLaunchKernelGGL((k_corr_row<0>), grid, dim3(256), 0, st, sigma, G, rmax, out);
    return hipGetLastError();
}

hipError_t launch_corr_row_many(int layout, const void* const* sigma, uint32_t n, const Geom& G, int32_t rmax,
                                int64_t* out, hipStream_t st) {
    if (n < 1 || n > kManyMax)
        return hipErrorInvalidValue;
    hipError_t e = launch_fill_i64(out, (size_t)n * ((size_t)rmax + 1), 0, st);
    if (e != hipSuccess)
        return e;
    if (layout == kLayP64 || layout == kLayI8Row) {
        // A row per wavefront (fewer when 16 rows exceed the staging buffer),
        // one lattice per grid layer, and as many 64-shift chunks per workgroup
        // as leave kCorrTarget workgroups (five 1024^2 lattices with 256, 512, 1024
        // and 2048 workgroups: 25.1, 22.5, 21.5 and 25.3 us)
        CorrLattices cl{};
        for (uint32_t a = 0; a < n; ++a)
            cl.p[a] = sigma[a];
        const uint32_t over = (uint32_t)rmax / 64u + 1u, pitch = G.L / 64u + over;
        const uint32_t R = kCorrWaves * pitch <= kCorr64Words ? kCorrWaves : kCorr64Words / pitch;
        const uint32_t groups = (G.L + R - 1u) / R;
        uint32_t chunks = (uint32_t)((uint64_t)over * groups * n / kCorrTarget);
        chunks = chunks < 1u ? 1u : chunks > kCorrChunks ? kCorrChunks : chunks;
        chunks = chunks > over ? over : chunks;
        const dim3 grid((over + chunks - 1u) / chunks, groups, n);
        const dim3 block(64u * kCorrWaves);
        if (layout == kLayI8Row)
            hipLaunchKernelGGL((k_corr_row64<true>), grid, block, 0, st, cl, G.L, R, chunks, rmax, out);
        else
            hipLaunchKernelGGL((k_corr_row64<false>), grid, block, 0, st, cl, G.L, R, chunks, rmax, out);
        return hipGetLastError();
    }
    for (uint32_t a = 0; a < n && e == hipSuccess; ++a)
        e = launch_corr_row_generic(layout, sigma[a], G, rmax, out + (size_t)a * ((size_t)rmax + 1), st);
    return e;
}

hipError_t launch_corr_row(int layout, const void* sigma, const Geom& G, int32_t rmax, int64_t* out,
                           hipStream_t st) {
    return launch_corr_row_many(layout, &sigma, 1u, G, rmax, out, st);
}


}  // namespace sd
