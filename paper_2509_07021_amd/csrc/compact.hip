// compact.hip -- the post-processing of Sec. 3.3 (post-processing procedure), gfx950: Gaussians whose
// opacity is below a threshold are dropped, lobes whose sharpness is below a threshold are dropped
// and their sphere mean is folded into the base colour (the compensation equation; Appendix,
// derivation of the colour compensation: delta c0 = m a (1 - e^{-2s}) / (2s), the average of the
// lobe over all directions), and what remains is written as a compressed-row scene whose Gaussians
// own 0..k lobes each.
//
// Two streaming passes over the parameter planes (HBM-bound, one thread per Gaussian, coalesced SoA
// reads): a mark pass that takes the keep decisions, leaves one byte per Gaussian and the kept
// Gaussians and lobes of each workgroup, one workgroup that turns those into output positions and hands
// the totals to the host, and a write pass that ranks the bytes of its 512 Gaussians again and
// gathers each kept Gaussian into its slot. Kept Gaussians and kept lobes are a subsequence of the
// input, so the writes of a wave land in a narrow window and coalesce too. Decisions and the
// compensation sum are taken in FP64 from the stored values; each output value is rounded once to FP32
// and then to its storage dtype. Planes that need no arithmetic (position, scale, rotation, axis,
// sharpness) are copied bit for bit.
//
// The write pass is bound by HBM and the latency in front of it (1M masked Gaussians of three lobes, 60%
// kept: 220 MB, 43 us at the rate of a copy): 103 us with each element loaded and stored under its own
// branch on the storage type, some forty round trips one after the other; 61 us with the raw words of a
// Gaussian and of kLobeGroup lobes loaded together, the kept Gaussians of a workgroup gathered into its
// first waves (the FP64 work on masks and means then runs on full waves, and the stores are contiguous),
// and one quotient per lobe. Measured beside it: groups of one and two lobes 62 and 68 us, workgroups of
// 256 and 1,024 Gaussians 67 and 63 us.
#include "megs_internal.hpp"

namespace megs {
namespace {

__device__ __forceinline__ double sigmoid_d(double x) { return 1.0 / (1.0 + exp(-x)); }

// logit(sigmoid(a) sigmoid(b)) = -log(e^-a + e^-b + e^-(a+b)), evaluated around the largest term: with
// p <= q the exponents -a and -b in order, that is p + q for p > 0 and q otherwise.
__device__ __forceinline__ double folded_logit(double a, double b) {
    const double p = fmin(-a, -b), q = fmax(-a, -b);
    const bool both = p > 0.0;
    const double m = both ? p + q : q;
    return -(m + log(1.0 + exp(both ? -p : p - q) + exp(both ? -q : p)));
}

constexpr int kThreads = 512;     // Gaussians of a workgroup, and of one entry of CompactArgs::sums
constexpr int kLobeGroup = 4;     // lobes loaded together
constexpr uint32_t kKept = 0x80;  // in CompactArgs::code; below it the number of kept lobes
static_assert(MEGS_MAX_LOBES < kKept, "a byte holds the kept flag and the number of kept lobes");

// f with an object of the unsigned type as wide as the storage type: one uniform branch for all the rows
// that f reads or writes. (With the branch at each element, a Gaussian's loads wait for one another.)
template <typename F>
__device__ __forceinline__ void by_width(int dt, F f) {
    if (dt == MEGS_F32)
        f(uint32_t{});
    else
        f(uint16_t{});
}

// Element `at` of N rows of a plane, as raw words: rows of `stride` elements from element `row` on, all
// three the same for the whole workgroup except `at`, which is small. A row's address stays in scalar
// registers: with a 64-bit index per element and thread the write pass took 250 registers, two waves a
// SIMD, and with an address per row kept over both branches it spent 559 instructions on scalar
// registers that did not fit.
template <typename T, int N>
__device__ __forceinline__ void load_rows(const void* p, int64_t row, int64_t stride, uint32_t at, uint32_t* out) {
    const T* q = static_cast<const T*>(p) + row;
#pragma unroll
    for (int j = 0; j < N; ++j, q += stride)
        out[j] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(q) + at * (uint32_t)sizeof(T));
}

template <typename T, int N>
__device__ __forceinline__ void store_rows(void* p, int64_t row, int64_t stride, uint32_t at, const uint32_t* w) {
    T* q = static_cast<T*>(p) + row;
#pragma unroll
    for (int j = 0; j < N; ++j, q += stride)
        *reinterpret_cast<T*>(reinterpret_cast<char*>(q) + at * (uint32_t)sizeof(T)) = (T)w[j];
}

__device__ __forceinline__ float widen(int dt, uint32_t w) {
    if (dt == MEGS_F32) return __uint_as_float(w);
    return dt == MEGS_F16 ? __half2float(__ushort_as_half((unsigned short)w)) : __uint_as_float(w << 16);
}

// The raw word of a value (round_elem is what store_elem rounds to).
__device__ __forceinline__ uint32_t narrow(int dt, float v) {
    return dt == MEGS_F32 ? __float_as_uint(v) : round_elem(dt, v);
}

// Exclusive scan of the workgroup's values and their sum.
__device__ __forceinline__ uint32_t block_rank(uint32_t x, uint32_t& total) {
    __shared__ uint32_t w[kThreads / kWave];
    const int lane = __lane_id(), me = threadIdx.x / kWave;
    uint32_t inc = x;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += y;
    }
    if (lane == kWave - 1) w[me] = inc;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int j = 0; j < kThreads / kWave; ++j) {
        if (j < me) before += w[j];
        total += w[j];
    }
    return before + inc - x;
}

// Kept Gaussians in the low half, kept lobes in the high half: up to 512 and 4,096 of a workgroup.
__device__ __forceinline__ uint32_t packed_count(uint32_t code) {
    return code & kKept ? 1u | (code & (kKept - 1)) << 16 : 0u;
}

template <bool RAGGED>
__global__ __launch_bounds__(kThreads) void k_compact_mark(CompactArgs a) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const SceneDev& sc = a.in;
    uint32_t code = 0;
    if (i < sc.n) {
        LobeRef<RAGGED> lr;
        const bool ok = lobe_ref<RAGGED>(sc, i, sc.k, lr);
        const void* const p[2] = {sc.op_logit, sc.pmask_logit};
        const int64_t idx[2] = {i, i};
        const bool live[2] = {true, sc.pmask_logit != nullptr};
        float logit[2];
        load_n<2>(sc.dt_geom, p, idx, live, logit);
        uint32_t cnt = 0;
        for (int l0 = 0; l0 < sc.k; l0 += kLobeGroup) {
            const void* sp[kLobeGroup];
            int64_t sidx[kLobeGroup];
            bool slive[kLobeGroup];
            float s[kLobeGroup];
#pragma unroll
            for (int l = 0; l < kLobeGroup; ++l) {
                sp[l] = sc.sharp;
                sidx[l] = lr.at1(l0 + l);
                slive[l] = l0 + l < lr.cnt;
            }
            load_n<kLobeGroup>(sc.dt_color, sp, sidx, slive, s);
#pragma unroll
            for (int l = 0; l < kLobeGroup; ++l) cnt += slive[l] && (double)s[l] >= a.sharp_min;
        }
        const double o = sigmoid_d(logit[0]) * (sc.pmask_logit ? sigmoid_d(logit[1]) : 1.0);
        if (ok && o >= a.opacity_min) code = kKept | cnt;
        a.code[i] = (uint8_t)code;
    }
    uint32_t total;
    block_rank(packed_count(code), total);
    if (threadIdx.x == 0) a.sums[blockIdx.x] = total;
}

// One workgroup: the position of each workgroup's first kept Gaussian and lobe, and the totals, to device
// memory and to the host that waits for them (HostCount). A total that 32 bits cannot hold reads as 2^32 - 1.
constexpr int kTopThreads = 1024;
__global__ __launch_bounds__(kTopThreads) void k_compact_top(CompactArgs a, int64_t m) {
    constexpr int kEach = 4, kWaves = kTopThreads / kWave;
    __shared__ uint64_t wave_sum[2][kWaves];
    const int lane = __lane_id(), me = threadIdx.x / kWave;
    uint64_t carry[2] = {0, 0};
    for (int64_t base = 0; base < m; base += kTopThreads * kEach) {
        const int64_t i0 = base + (int64_t)threadIdx.x * kEach;
        uint32_t v[kEach];
        uint64_t inc[2] = {0, 0};
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            v[j] = i0 + j < m ? a.sums[i0 + j] : 0u;
            inc[0] += v[j] & 0xffffu;
            inc[1] += v[j] >> 16;
        }
        const uint64_t own[2] = {inc[0], inc[1]};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const uint64_t y = __shfl_up(inc[q], d, kWave);
                if (lane >= d) inc[q] += y;
            }
            if (lane == kWave - 1) wave_sum[q][me] = inc[q];
        }
        __syncthreads();
        uint64_t at[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            at[q] = carry[q] + inc[q] - own[q];
            for (int w = 0; w < kWaves; ++w) {
                if (w < me) at[q] += wave_sum[q][w];
                carry[q] += wave_sum[q][w];
            }
        }
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            if (i0 + j < m) a.first[i0 + j] = make_uint2((uint32_t)at[0], (uint32_t)at[1]);
            at[0] += v[j] & 0xffffu;
            at[1] += v[j] >> 16;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const uint32_t no = (uint32_t)carry[0], lo = carry[1] > 0xffffffffull ? 0xffffffffu : (uint32_t)carry[1];
        a.totals[0] = no;
        a.totals[1] = lo;
        if (a.host) {
            a.host->total = no;
            a.host->total2 = lo;
            a.host->bad_lobes = a.in.status[kStatusBadLobes];
            __hip_atomic_store(&a.host->seq, a.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

template <bool RAGGED>
__global__ __launch_bounds__(kThreads) void k_compact_write(CompactArgs a) {
    __shared__ uint32_t source[kThreads];  // of the j-th kept Gaussian: its index and first kept lobe here
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const SceneDev& sc = a.in;
    const uint32_t code = i < sc.n ? a.code[i] : 0u;
    const uint2 first = a.first[blockIdx.x];
    const int64_t x0 = __builtin_amdgcn_readfirstlane(first.x), y0 = __builtin_amdgcn_readfirstlane(first.y);
    uint32_t total;
    const uint32_t rank = block_rank(packed_count(code), total);
    if (code & kKept) source[rank & 0xffffu] = threadIdx.x | (rank >> 16) << 16;
    __syncthreads();
    const int64_t n = sc.n, no = a.n_out, lo = a.l_out, i0 = (int64_t)blockIdx.x * kThreads;
    if (i == 0) a.lobe_off[no] = (int32_t)lo;
    const int64_t off0 = RAGGED ? __builtin_amdgcn_readfirstlane(sc.lobe_off[i0]) : 0;  // lobes of the workgroup begin there
    const uint32_t j = threadIdx.x;  // in the rows that begin at x0
    if (j >= (total & 0xffffu)) return;
    const uint32_t from = source[j];
    const uint32_t t = from & 0xffffu;  // in the rows that begin at i0
    uint32_t d = from >> 16;            // and at y0
    i = i0 + t;
    // All offsets were validated by the mark pass (a malformed one ends the call before this launch), so
    // they do not decrease and a workgroup's lobes are consecutive.
    const uint32_t off = RAGGED ? (uint32_t)(sc.lobe_off[i] - off0) : t;
    const int cnt = RAGGED ? sc.lobe_off[i + 1] - sc.lobe_off[i] : sc.k;

    uint32_t g[12], bw[3];  // position, scale, rotation, opacity, mask; base colour
    by_width(sc.dt_geom, [&](auto e) {
        using T = decltype(e);
        load_rows<T, 3>(sc.pos, i0, n, t, g);
        load_rows<T, 3>(sc.logscale, i0, n, t, g + 3);
        load_rows<T, 4>(sc.quat, i0, n, t, g + 6);
        load_rows<T, 1>(sc.op_logit, i0, n, t, g + 10);
        if (sc.pmask_logit) load_rows<T, 1>(sc.pmask_logit, i0, n, t, g + 11);
    });
    by_width(sc.dt_color, [&](auto e) { load_rows<decltype(e), 3>(sc.base, i0, n, t, bw); });
    double base[3];
    for (int l0 = 0; l0 < sc.k; l0 += kLobeGroup) {
        uint32_t w[kLobeGroup][5], aw[kLobeGroup][3];  // axis, sharpness, mask; amplitude
        by_width(sc.dt_color, [&](auto e) {
            using T = decltype(e);
#pragma unroll
            for (int l = 0; l < kLobeGroup; ++l)
                if (l0 + l < cnt) {
                    const int64_t row = RAGGED ? off0 : (l0 + l) * n + i0, row3 = RAGGED ? off0 : (l0 + l) * 3 * n + i0;
                    const uint32_t at = RAGGED ? off + (uint32_t)(l0 + l) : t;
                    load_rows<T, 1>(sc.sharp, row, 0, at, w[l] + 3);
                    if (sc.lmask_logit) load_rows<T, 1>(sc.lmask_logit, row, 0, at, w[l] + 4);
                    load_rows<T, 3>(sc.axis, row3, RAGGED ? sc.n_lobes : n, at, w[l]);
                }
        });
        by_width(sc.dt_amp, [&](auto e) {
#pragma unroll
            for (int l = 0; l < kLobeGroup; ++l)
                if (l0 + l < cnt)
                    load_rows<decltype(e), 3>(sc.amp, RAGGED ? off0 : (l0 + l) * 3 * n + i0, RAGGED ? sc.n_lobes : n,
                                              RAGGED ? off + (uint32_t)(l0 + l) : t, aw[l]);
        });
        if (l0 == 0)
            for (int c = 0; c < 3; ++c) base[c] = widen(sc.dt_color, bw[c]);
#pragma unroll
        for (int l = 0; l < kLobeGroup; ++l) {
            if (l0 + l >= cnt) continue;
            const double s = widen(sc.dt_color, w[l][3]);
            const bool kept = s >= a.sharp_min;
            // the lobe's mask, and for a dropped lobe times its mean over the sphere, (1 - e^{-2s}) / (2s)
            // (1 at s = 0): one quotient
            double num = 1.0, den = 1.0;
            if (!kept && s != 0.0) {
                num = -expm1(-2.0 * s);
                den = 2.0 * s;
            }
            if (sc.lmask_logit) den *= 1.0 + exp(-(double)widen(sc.dt_color, w[l][4]));
            const double f = num / den;
            if (kept) {
                by_width(sc.dt_color, [&](auto e) {
                    using T = decltype(e);
                    store_rows<T, 3>(a.axis, y0, lo, d, w[l]);
                    store_rows<T, 1>(a.sharp, y0, lo, d, w[l] + 3);
                });
                if (sc.lmask_logit)
                    for (int c = 0; c < 3; ++c) aw[l][c] = narrow(sc.dt_amp, (float)(f * widen(sc.dt_amp, aw[l][c])));
                by_width(sc.dt_amp, [&](auto e) { store_rows<decltype(e), 3>(a.amp, y0, lo, d, aw[l]); });
                const uint32_t src = (uint32_t)(RAGGED ? off0 + off + l0 + l : (int64_t)(l0 + l) * n + i);
                store_rows<uint32_t, 1>(a.lobe_src, y0, lo, d, &src);
                ++d;
            } else {
                for (int c = 0; c < 3; ++c) base[c] += f * widen(sc.dt_amp, aw[l][c]);
            }
        }
    }
    if (sc.k == 0)
        for (int c = 0; c < 3; ++c) base[c] = widen(sc.dt_color, bw[c]);
    for (int c = 0; c < 3; ++c) bw[c] = narrow(sc.dt_color, (float)base[c]);
    by_width(sc.dt_color, [&](auto e) { store_rows<decltype(e), 3>(a.base, x0, no, j, bw); });
    if (sc.pmask_logit)
        g[10] = narrow(sc.dt_geom, (float)folded_logit(widen(sc.dt_geom, g[10]), widen(sc.dt_geom, g[11])));
    by_width(sc.dt_geom, [&](auto e) {
        using T = decltype(e);
        store_rows<T, 3>(a.pos, x0, no, j, g);
        store_rows<T, 3>(a.logscale, x0, no, j, g + 3);
        store_rows<T, 4>(a.quat, x0, no, j, g + 6);
        store_rows<T, 1>(a.op_logit, x0, no, j, g + 10);
    });
    const uint32_t src = (uint32_t)i, at_lobe = (uint32_t)y0 + (from >> 16);
    store_rows<uint32_t, 1>(a.kept, x0, no, j, &src);
    store_rows<uint32_t, 1>(a.lobe_off, x0, no, j, &at_lobe);
}

inline unsigned blocks_of(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

int64_t compact_blocks(int64_t n) { return (n + kThreads - 1) / kThreads; }

hipError_t launch_compact_mark(const CompactArgs& a, hipStream_t stream) {
    if (a.in.n == 0) return hipSuccess;
    if (a.in.lobe_off)
        hipLaunchKernelGGL(k_compact_mark<true>, dim3(blocks_of(a.in.n)), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL(k_compact_mark<false>, dim3(blocks_of(a.in.n)), dim3(kThreads), 0, stream, a);
    hipLaunchKernelGGL(k_compact_top, dim3(1), dim3(kTopThreads), 0, stream, a, compact_blocks(a.in.n));
    return hipGetLastError();
}

hipError_t launch_compact_write(const CompactArgs& a, hipStream_t stream) {
    if (a.in.n == 0 || a.n_out == 0) return hipSuccess;
    if (a.in.lobe_off)
        hipLaunchKernelGGL(k_compact_write<true>, dim3(blocks_of(a.in.n)), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL(k_compact_write<false>, dim3(blocks_of(a.in.n)), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace megs
