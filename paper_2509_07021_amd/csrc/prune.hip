// prune.hip -- the GPU steps of the memory-constrained optimisation (Sec. 3.3, Alg. 1) that act on
// the renderer's outputs: the lobe dynamic range D = |a| (1 - exp(-2 z)) (Sec. 3.3.2), a top-kappa
// selection for the factorised proximal operator, and the proximal, dual and penalty updates.
//
// Top-kappa is an MSB-first radix select on order-preserving 32-bit keys: four histogram passes
// over the candidates that still share the selected prefix, each finding the digit bucket that holds
// the kappa-th largest key. Elements equal to the threshold key are then taken in ascending index
// order, so the selected set is exactly "the kappa largest, ties to the lower index", independent of
// scheduling.
//
// What bounds it is what a score passes through: one read per pass (3M scores: 12 MB, from the cache
// after the first), the histogram's atomics, and the launches. At most 256 workgroups of 1,024 threads
// own one contiguous chunk each and add to one of eight device histograms, so that a bucket receives at
// most 32 adds (scores share few exponents: with one workgroup per 1,024 scores and one histogram the first
// two passes' adds to a handful of addresses took 97 and 155 us at 3M scores; with 256 workgroups and one
// histogram 6 and 10 us, with eight 4.5 us each), and a workgroup counts in 16 tables, one per lane group,
// which holds the adds of a wave to one address to four. Each pass finds the digit of the pass before it
// in its own prologue (256 counts, one scan) instead of a one-thread launch between them, and the last pass
// leaves every workgroup's table, from which the selection knows how many equal keys lie before its chunk:
// no flags, no scan, and with distinct scores no second look at all. Measured at 1M and 3M scores with kappa
// = 3 n / 5 and n / 3: 195 and 360 us in 13 launches, now some 20 and 28 us in six.
#include "megs_internal.hpp"

namespace megs {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelBlocks = 256;
constexpr int kSelCopies = 16;               // histograms of a workgroup, one per lane & 15
constexpr int kSelStride = 257;              // words between them: equal digits fall into different LDS banks
constexpr int kSelHists = 8;                 // histograms of a pass in memory: an eighth of the adds to one address
constexpr int kSelChunk = 2048;              // scores of a workgroup before there are kSelBlocks of them
constexpr int kSelSmall = 16 * kSelThreads;  // scores that one workgroup holds in registers

struct SelectState {
    uint32_t prefix;  // selected high digits of the threshold key
    uint32_t need;    // how many of the remaining candidates (keys matching prefix) to take
};

// Scratch: the state before each pass, the four passes' histograms, and the last pass's histogram of
// every workgroup.
struct SelectScratch {
    SelectState st[4];
    uint32_t hist[4][kSelHists][256];  // a pass's histogram is the sum of kSelHists, a workgroup adds to one
    uint32_t last[kSelBlocks][256];
};

// Order-preserving map from float to uint32 (larger float -> larger key); -0 maps like +0.
__device__ __forceinline__ uint32_t ordered_key(float f) {
    const uint32_t b = __float_as_uint(f + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// From the largest digit down, the bucket that holds the need-th largest candidate, of counts h(digit)
// that sum to need or more. All threads of the workgroup call it and receive the digit, its count and
// what of it is needed.
template <typename H>
__device__ __forceinline__ void pick_digit(H h, uint32_t need, uint32_t& digit, uint32_t& count, uint32_t& take) {
    __shared__ uint32_t wave_total[4], found[3];
    const int t = threadIdx.x, lane = __lane_id();
    uint32_t c = 0, inc = 0;
    if (t < 256) {
        c = inc = h(255 - t);
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += y;
        }
        if (lane == kWave - 1) wave_total[t / kWave] = inc;
    }
    __syncthreads();
    if (t < 256) {
        for (int w = 0; w < t / kWave; ++w) inc += wave_total[w];
        if (inc >= need && inc - c < need) {  // one thread: the counts reach need at one digit
            found[0] = 255 - t;
            found[1] = c;
            found[2] = need - (inc - c);
        }
    }
    __syncthreads();
    digit = found[0]; count = found[1]; take = found[2];
}

__device__ __forceinline__ void clear_tables(uint32_t* h) {
    for (int i = threadIdx.x; i < kSelCopies * kSelStride; i += kSelThreads) h[i] = 0;
    __syncthreads();
}

__device__ __forceinline__ void count_digit(uint32_t* h, uint32_t digit) {
    atomicAdd(&h[(threadIdx.x & (kSelCopies - 1)) * kSelStride + digit], 1u);
}

__device__ __forceinline__ uint32_t sum_tables(const uint32_t* h, int digit) {
    uint32_t s = 0;
#pragma unroll
    for (int c = 0; c < kSelCopies; ++c) s += h[c * kSelStride + digit];
    return s;
}

__global__ __launch_bounds__(kSelThreads) void k_select_init(SelectScratch* sc, uint32_t kappa) {
    uint32_t* const h = &sc->hist[0][0][0];
#pragma unroll
    for (int i = 0; i < kSelHists; ++i) h[i * kSelThreads + threadIdx.x] = 0;  // 4 passes of 256 digits each
    if (threadIdx.x == 0) sc->st[0] = {0u, kappa};
}

// The state before pass PASS: the digit of the pass before it, found by every workgroup and left for
// the next launch by the first.
template <int PASS>
__device__ __forceinline__ SelectState select_state(SelectScratch* sc, uint32_t* equal) {
    SelectState st = sc->st[PASS ? PASS - 1 : 0];
    if (PASS) {
        uint32_t digit, take;
        pick_digit(
            [&](int d) {
                uint32_t s = 0;
#pragma unroll
                for (int i = 0; i < kSelHists; ++i) s += sc->hist[PASS - 1][i][d];
                return s;
            },
            st.need, digit, *equal, take);
        st.prefix |= digit << (32 - 8 * PASS);
        st.need = take;
        if (PASS < 4 && blockIdx.x == 0 && threadIdx.x == 0) sc->st[PASS] = st;
    }
    return st;
}

// f(index, key) over scores lo .. hi - 1, four rows of loads in flight (indexes past the end read the
// first score instead of branching around the load).
template <typename F>
__device__ __forceinline__ void for_rows(const float* __restrict__ score, int64_t lo, int64_t hi, F f) {
    for (int64_t r = lo; r < hi; r += 4 * kSelThreads) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = r + j * kSelThreads + threadIdx.x;
            v[j] = score[i < hi ? i : lo];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = r + j * kSelThreads + threadIdx.x;
            if (i < hi) f(i, ordered_key(v[j]));
        }
    }
}

// Histogram of digit PASS (from the top) over the keys that share the prefix selected so far.
template <int PASS>
__global__ __launch_bounds__(kSelThreads) void k_select_hist(const float* __restrict__ score, int64_t n,
                                                             int64_t chunk, SelectScratch* sc) {
    __shared__ uint32_t h[kSelCopies * kSelStride];
    clear_tables(h);
    uint32_t equal;
    const SelectState st = select_state<PASS>(sc, &equal);
    constexpr int shift = 24 - 8 * PASS;
    const int64_t lo = blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    for_rows(score, lo, hi, [&](int64_t, uint32_t key) {
        if (PASS == 0 || ((key ^ st.prefix) >> (PASS ? shift + 8 : 0)) == 0) count_digit(h, (key >> shift) & 255u);
    });
    __syncthreads();
    if (threadIdx.x < 256) {
        const uint32_t s = sum_tables(h, threadIdx.x);
        if (s) atomicAdd(&sc->hist[PASS][blockIdx.x % kSelHists][threadIdx.x], s);
        if (PASS == 3) sc->last[blockIdx.x][threadIdx.x] = s;
    }
}

// Among the workgroup's keys equal to the threshold, in index order: the rank of this thread's (rows of
// kSelThreads keys; `before` is the rank of the row's first, and then of the next row's).
__device__ __forceinline__ uint32_t row_rank(bool eq, uint32_t& before) {
    __shared__ uint32_t wave_count[kSelThreads / kWave];
    const uint64_t m = __ballot(eq);
    const int lane = __lane_id(), w = threadIdx.x / kWave;
    if (lane == 0) wave_count[w] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t rank = before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    for (int j = 0; j < kSelThreads / kWave; ++j) {
        const uint32_t c = wave_count[j];
        if (j < w) rank += c;
        before += c;
    }
    __syncthreads();
    return rank;
}

__global__ __launch_bounds__(kSelThreads) void k_select_keep(const float* __restrict__ score, int64_t n,
                                                             int64_t chunk, SelectScratch* sc,
                                                             uint8_t* __restrict__ keep) {
    __shared__ uint32_t part[4];
    uint32_t equal;
    const SelectState st = select_state<4>(sc, &equal);
    const int64_t lo = blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    if (equal == st.need) {  // uniform over the grid: all keys equal to the threshold are taken
        for_rows(score, lo, hi, [&](int64_t i, uint32_t key) { keep[i] = key >= st.prefix; });
        return;
    }
    // equal keys before the chunk
    uint32_t before = 0;
    if (threadIdx.x < 256) {
        before = threadIdx.x < blockIdx.x ? sc->last[threadIdx.x][st.prefix & 255u] : 0u;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d);
        if (__lane_id() == 0) part[threadIdx.x / kWave] = before;
    }
    __syncthreads();
    before = part[0] + part[1] + part[2] + part[3];
    for (int64_t r = lo; r < hi; r += kSelThreads) {
        const int64_t i = r + threadIdx.x;
        const uint32_t key = i < hi ? ordered_key(score[i]) : 0u;
        const uint32_t rank = row_rank(i < hi && key == st.prefix, before);
        if (i < hi) keep[i] = key > st.prefix || (key == st.prefix && rank < st.need);
    }
}

// All of it in one workgroup, for scores that fit into its registers: at a few thousand scores the six
// launches are the time.
__global__ __launch_bounds__(kSelThreads) void k_select_small(const float* __restrict__ score, int n, uint32_t kappa,
                                                              uint8_t* __restrict__ keep) {
    __shared__ uint32_t h[kSelCopies * kSelStride];
    constexpr int kRows = kSelSmall / kSelThreads;
    uint32_t key[kRows];
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int i = j * kSelThreads + threadIdx.x;
        key[j] = ordered_key(i < n ? score[i] : 0.0f);
    }
    SelectState st = {0u, kappa};
    uint32_t equal = 0;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        clear_tables(h);
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const bool in = j * kSelThreads + (int)threadIdx.x < n;
            if (in && (pass == 0 || ((key[j] ^ st.prefix) >> (pass ? shift + 8 : 0)) == 0))
                count_digit(h, (key[j] >> shift) & 255u);
        }
        __syncthreads();
        uint32_t digit, take;
        pick_digit([&](int d) { return sum_tables(h, d); }, st.need, digit, equal, take);
        st.prefix |= digit << shift;
        st.need = take;
    }
    uint32_t before = 0;
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        const int i = j * kSelThreads + threadIdx.x;
        bool k = key[j] >= st.prefix;
        if (equal != st.need && j * kSelThreads < n) {  // uniform over the workgroup
            const uint32_t rank = row_rank(i < n && key[j] == st.prefix, before);
            k = key[j] > st.prefix || (k && rank < st.need);
        }
        if (i < n) keep[i] = k;
    }
}

__global__ void k_fill_u8(uint8_t* p, uint8_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// D[l][i] = |a_l,i| (1 - exp(-2 (s + lambda)[l][i])) with |.| the Euclidean norm of the RGB amplitude.
__global__ void k_lobe_range(int64_t n, int32_t k, const float* __restrict__ s, const float* __restrict__ lam,
                             const float* __restrict__ amp, float* __restrict__ D) {
    const int64_t total = n * k;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < total; j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t l = j / n, i = j - l * n;
        const float z = s[j] + (lam ? lam[j] : 0.0f);
        const float a0 = amp[(l * 3 + 0) * n + i], a1 = amp[(l * 3 + 1) * n + i], a2 = amp[(l * 3 + 2) * n + i];
        D[j] = sqrtf(a0 * a0 + a1 * a1 + a2 * a2) * (1.0f - expf(-2.0f * z));
    }
}

__global__ void k_prox_apply(int64_t count, const float* __restrict__ x, const float* __restrict__ lam,
                             const uint8_t* __restrict__ keep, float* __restrict__ xt) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        xt[i] = keep[i] ? x[i] + lam[i] : 0.0f;
}

__global__ void k_dual(int64_t count, float* __restrict__ lam, const float* __restrict__ x,
                       const float* __restrict__ xt) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        lam[i] = lam[i] + (x[i] - xt[i]);
}

__global__ void k_penalty(int64_t count, float delta, const float* __restrict__ x, const float* __restrict__ xt,
                          const float* __restrict__ lam, float* __restrict__ grad) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        grad[i] = __fmaf_rn(delta, (x[i] - xt[i]) + lam[i], grad[i]);
}

inline unsigned grid_of(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return (unsigned)b;
}

}  // namespace

// Scores of a workgroup, a multiple of its threads, and the workgroups.
inline int64_t select_chunk(int64_t n) {
    int64_t chunk = (n + kSelBlocks - 1) / kSelBlocks;
    if (chunk < kSelChunk) chunk = kSelChunk;
    return (chunk + kSelThreads - 1) / kSelThreads * kSelThreads;
}
inline unsigned select_blocks(int64_t n) { return (unsigned)((n + select_chunk(n) - 1) / select_chunk(n)); }

size_t select_scratch_bytes(int64_t n) {  // (the last pass's tables of the workgroups there are)
    return n <= kSelSmall ? 256 : offsetof(SelectScratch, last) + select_blocks(n) * sizeof(SelectScratch::last[0]);
}

hipError_t launch_select_topk(const float* score, int64_t n, int64_t kappa, void* scratch, uint8_t* keep,
                              hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    if (kappa <= 0 || kappa >= n) {
        hipLaunchKernelGGL(k_fill_u8, dim3(grid_of(n)), dim3(256), 0, stream, keep, (uint8_t)(kappa > 0), n);
        return hipGetLastError();
    }
    if (n <= kSelSmall) {
        hipLaunchKernelGGL(k_select_small, dim3(1), dim3(kSelThreads), 0, stream, score, (int)n, (uint32_t)kappa, keep);
        return hipGetLastError();
    }
    SelectScratch* sc = static_cast<SelectScratch*>(scratch);
    const int64_t chunk = select_chunk(n);
    const dim3 grid(select_blocks(n)), block(kSelThreads);
    hipLaunchKernelGGL(k_select_init, dim3(1), block, 0, stream, sc, (uint32_t)kappa);
    hipLaunchKernelGGL(k_select_hist<0>, grid, block, 0, stream, score, n, chunk, sc);
    hipLaunchKernelGGL(k_select_hist<1>, grid, block, 0, stream, score, n, chunk, sc);
    hipLaunchKernelGGL(k_select_hist<2>, grid, block, 0, stream, score, n, chunk, sc);
    hipLaunchKernelGGL(k_select_hist<3>, grid, block, 0, stream, score, n, chunk, sc);
    hipLaunchKernelGGL(k_select_keep, grid, block, 0, stream, score, n, chunk, sc, keep);
    return hipGetLastError();
}

hipError_t launch_lobe_range(int64_t n, int32_t k, const float* s, const float* lam, const float* amp, float* D,
                             hipStream_t stream) {
    if (n * k <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_lobe_range, dim3(grid_of(n * k)), dim3(256), 0, stream, n, k, s, lam, amp, D);
    return hipGetLastError();
}

hipError_t launch_prox_apply(int64_t count, const float* x, const float* lam, const uint8_t* keep, float* xt,
                             hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prox_apply, dim3(grid_of(count)), dim3(256), 0, stream, count, x, lam, keep, xt);
    return hipGetLastError();
}

hipError_t launch_dual(int64_t count, float* lam, const float* x, const float* xt, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dual, dim3(grid_of(count)), dim3(256), 0, stream, count, lam, x, xt);
    return hipGetLastError();
}

hipError_t launch_penalty(int64_t count, float delta, const float* x, const float* xt, const float* lam, float* grad,
                          hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_penalty, dim3(grid_of(count)), dim3(256), 0, stream, count, delta, x, xt, lam, grad);
    return hipGetLastError();
}

}  // namespace megs
