// loss.hip -- the training-step pieces around the renderer, gfx950: the 3DGS photometric loss
// L = (1 - lambda) L1 + lambda (1 - SSIM) with its gradient, and an Adam step on parameter planes
// stored in FP32, FP16 or BF16 (the paper trains with 3DGS's loss, hyperparameters and optimiser;
// Appendix, experimental details).
//
// SSIM uses an 11x11 Gaussian window (sigma 1.5, separable, zero padding) and C1 = 0.01^2,
// C2 = 0.03^2. Writing S = a1 a2 / (b1 b2) with a1 = 2 mx my + C1, a2 = 2 sxy + C2,
// b1 = mx^2 + my^2 + C1, b2 = sxx + syy + C2, and the windowed raw moments (mx, Exx, Exy) as the
// variables, the derivative of S at pixel q with respect to x at pixel p is
//   G(p - q) (dS/dmx(q) + 2 x_p dS/dExx(q) + y_p dS/dExy(q)),
//   dS/dmx = (2 my (a2 - a1) - 2 mx S (b2 - b1)) / (b1 b2), dS/dExx = -S / b2, dS/dExy = 2 a1 / (b1 b2),
// so the gradient is a second windowed pass over those three maps. The moments cancel (Exx - mx^2 against
// C2 = 9e-4), so all SSIM arithmetic is FP64; the planes are FP32. The loss sums go through per-wave
// partials reduced in a fixed order, so the loss is deterministic.
//
// Both passes stream: one wave owns 64 columns of a strip of rows and walks them downwards. A row and its
// 5-pixel halo pass through the wave's LDS for the horizontal window, and the vertical window is a shift
// register of partial sums per moment (each new row's sum enters all 11, one FMA each, and the oldest leaves
// complete), so nothing is staged twice and no wave waits for another. Per pixel and channel that is about
// 160 FP64 instructions forward and 80 backward (they run at the FP32 rate here), and 24 bytes of maps
// written and read. One 1080p image takes 74 + 62 us, where 16 x 16 tiles of FP64 patches in LDS took
// 138 + 116 us; four take 248 + 254 us (the maps then exceed the last-level cache). Both passes in one, with
// the maps kept in LDS, saves their traffic but needs 236 registers for one wave and measured 157 us (183 us
// as two waves handing rows over). Small and narrow images, whose strips are few or leave lanes idle, go by such
// tiles (loss_rows).
#include "megs_internal.hpp"

namespace megs {
namespace {

constexpr int kR = 5;               // window radius
constexpr double kC1 = 0.01 * 0.01, kC2 = 0.03 * 0.03;
constexpr int kPatch = kWave + 2 * kR;
// Strips whose loss sums one wave reduces, beside the gradient's strips where there are any: a launch saved,
// and even a wave alone takes less than a pass over that many strips (a launch of its own took 4.7 us of the
// 24 us of a 128 x 128 image).
constexpr int64_t kWaveSums = 8192;

// The strip of work item `item`: view, channel, first column, rows [y0, y1).
struct Strip {
    LossView v;
    int c, x0, y0, y1;
    int64_t plane, off;  // pixels of a channel; the channel's first element in the image layout
};

__device__ __forceinline__ Strip strip_of(const LossViews& vs, int nv, int64_t item) {
    int i = 0;
    while (i + 1 < nv && vs.v[i + 1].part_off <= item) ++i;
    Strip s;
    s.v = vs.v[i];
    const int64_t k = item - s.v.part_off;
    const int sx = (s.v.width + kWave - 1) / kWave, per_c = sx * ((s.v.height + s.v.rows - 1) / s.v.rows);
    s.c = (int)(k / per_c);
    const int q = (int)(k - (int64_t)s.c * per_c);
    s.x0 = (q % sx) * kWave;
    s.y0 = (q / sx) * s.v.rows;
    s.y1 = min(s.y0 + s.v.rows, s.v.height);
    s.plane = (int64_t)s.v.width * s.v.height;
    s.off = s.v.pix_off * 3 + s.c * s.plane;
    return s;
}

// LDS written by some lanes of the wave and read by others.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A row's values for the wave's patch: column x0 - 5 + lane, and for lanes below 10 also column x0 + 59 + lane.
// The loads go to clamped positions and nothing depends on them here, so they stay in flight until put_row,
// which makes what lies outside the image zero.
template <typename T>
struct RowPair {
    T a, b;
};
template <typename T>
__device__ __forceinline__ void load_row(RowPair<T>& v, const T* __restrict__ p, const Strip& s, int r, int lane) {
    const int xa = s.x0 - kR + lane, xb = xa + kWave, last = s.v.width - 1;
    const T* q = p + (int64_t)min(max(r, 0), s.v.height - 1) * s.v.width;
    v.a = q[min(max(xa, 0), last)];
    if (lane < 2 * kR) v.b = q[min(xb, last)];
}
template <typename T>
__device__ __forceinline__ void put_row(double* lds, const RowPair<T>& v, const Strip& s, int r, int lane) {
    const int xa = s.x0 - kR + lane, xb = xa + kWave;
    const bool row = r >= 0 && r < s.v.height;
    lds[lane] = row && xa >= 0 && xa < s.v.width ? v.a : T(0);
    if (lane < 2 * kR) lds[kWave + lane] = row && xb < s.v.width ? v.b : T(0);
}

// The horizontal window's moments at the patch column lane + 5: of x, y, x^2 + y^2 (the variances enter SSIM
// only as their sum) and x y.
__device__ __forceinline__ void row_moments(const double* sx, const double* sy, int lane, const Window11& g, double (&h)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) h[m] = 0.0;
#pragma unroll
    for (int k = 0; k < 11; ++k) {
        const double a = sx[lane + k], b = sy[lane + k];
        const double wa = g.w[k] * a, wb = g.w[k] * b;
        h[0] += wa;
        h[1] += wb;
        h[2] = fma(wb, b, fma(wa, a, h[2]));
        h[3] = fma(wa, b, h[3]);
    }
}

// SSIM from the windowed moments, and its derivatives in mx, Exx and Exy.
struct Ssim {
    double S, d[3];
};
__device__ __forceinline__ Ssim ssim_of(const double (&mo)[4]) {
    const double mx = mo[0], my = mo[1];
    const double a1 = fma(2.0 * mx, my, kC1), a2 = fma(2.0, mo[3] - mx * my, kC2);
    const double mm = fma(mx, mx, my * my), b1 = mm + kC1, b2 = (mo[2] - mm) + kC2;
    const double rd = 1.0 / (b1 * b2);
    Ssim r;
    r.S = a1 * a2 * rd;
    r.d[0] = 2.0 * (my * (a2 - a1) - mx * r.S * (b2 - b1)) * rd;
    r.d[1] = -r.S * b1 * rd;
    r.d[2] = 2.0 * a1 * rd;
    return r;
}

// w h + c into a register of its own. Written out, because the compiler forms the shift register's steps
// with the two-address v_fmac_f64 and copies most of its registers once a row (105 moves beside 160 arithmetic
// instructions in the forward: 71 us for a 1080p image without its gradient instead of 56).
__device__ __forceinline__ double fma_to(double w, double h, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "s"(w), "v"(h), "v"(c));
    return r;
}

// Enters a row's sum into the shift register of the vertical window; returns the row 5 above, complete.
__device__ __forceinline__ double shift_in(double (&acc)[10], double h, const Window11& g) {
    const double out = fma_to(g.w[10], h, acc[0]);
#pragma unroll
    for (int i = 0; i < 9; ++i) acc[i] = fma_to(g.w[9 - i], h, acc[i + 1]);
    acc[9] = g.w[0] * h;
    return out;
}

__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
    return x;
}

// The loss sums, and with MAPS (a gradient follows) the derivative maps.
template <bool MAPS>
__global__ __launch_bounds__(64) void k_ssim_fwd(LossViews vs, int nv, const float* __restrict__ x,
                                                 const float* __restrict__ y, double* __restrict__ maps,
                                                 double* __restrict__ partial, Window11 g) {
    __shared__ double sx[kPatch], sy[kPatch];
    const int lane = threadIdx.x;
    const int64_t item = xcd_item(blockIdx.x, gridDim.x);  // neighbouring strips share an L2 and halos
    const Strip s = strip_of(vs, nv, item);
    const float* xc = x + s.off;
    const float* yc = y + s.off;
    double* mc = maps + s.off * 3;
    const bool col = s.x0 + lane < s.v.width;
    double acc[4][10] = {};
    double ssim = 0.0, l1 = 0.0;
    RowPair<float> xe, ye, xo, yo;
    // row r, in v and w, which then take row r + 2
    auto step = [&](RowPair<float>& v, RowPair<float>& w, int r) {
        put_row(sx, v, s, r, lane);
        put_row(sy, w, s, r, lane);
        wave_sync();
        load_row(v, xc, s, r + 2, lane);
        load_row(w, yc, s, r + 2, lane);
        double h[4], mo[4];
        row_moments(sx, sy, lane, g, h);
        if (r >= s.y0 && r < s.y1 && col) l1 += fabs(sx[lane + kR] - sy[lane + kR]);
        wave_sync();
#pragma unroll
        for (int m = 0; m < 4; ++m) mo[m] = shift_in(acc[m], h[m], g);
        const int q = r - kR;
        if (q >= s.y0 && col) {
            const Ssim t = ssim_of(mo);
            ssim += t.S;
            if (MAPS) {
                const int64_t p = (int64_t)q * s.v.width + s.x0 + lane;
#pragma unroll
                for (int m = 0; m < 3; ++m) mc[m * s.plane + p] = t.d[m];
            }
        }
    };
    const int r1 = s.y1 + kR;
    load_row(xe, xc, s, s.y0 - kR, lane);
    load_row(ye, yc, s, s.y0 - kR, lane);
    load_row(xo, xc, s, s.y0 - kR + 1, lane);
    load_row(yo, yc, s, s.y0 - kR + 1, lane);
    for (int r = s.y0 - kR; r < r1; r += 2) {
        step(xe, ye, r);
        if (r + 1 < r1) step(xo, yo, r + 1);
    }
    ssim = wave_sum_f64(ssim);
    l1 = wave_sum_f64(l1);
    if (lane == 0) {
        partial[2 * item] = ssim;
        partial[2 * item + 1] = l1;
    }
}

// A view's term of the loss, and the loss from the partial sums by one wave, in a fixed order.
__device__ __forceinline__ double view_loss(const LossView& v, double ssim, double l1, double lam) {
    const double n = 3.0 * (double)v.width * v.height;
    return (1.0 - lam) * l1 / n + lam * (1.0 - ssim / n);
}
__device__ __forceinline__ void loss_by_wave(const double* __restrict__ partial, const LossViews& vs, int nv, double lam,
                                             double* __restrict__ loss, int lane) {
    double sum = 0.0;
    for (int i = 0; i < nv; ++i) {
        const LossView v = vs.v[i];
        double s[4] = {}, l[4] = {};
        for (int64_t b = lane; b < v.n_part; b += 4 * kWave)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (b + u * kWave < v.n_part) {
                    const double2 p = reinterpret_cast<const double2*>(partial)[v.part_off + b + u * kWave];
                    s[u] += p.x;
                    l[u] += p.y;
                }
        const double ss = wave_sum_f64((s[0] + s[1]) + (s[2] + s[3])), ll = wave_sum_f64((l[0] + l[1]) + (l[2] + l[3]));
        sum += view_loss(v, ss, ll, lam);
    }
    if (lane == 0) loss[0] = sum;
}

// A pixel's gradient from the windowed derivative maps; n: values of the view (3 per pixel).
__device__ __forceinline__ float gradient_of(float x, float y, const double (&b)[3], double n, double lam) {
    const double cl = (1.0 - lam) / n, cs = lam / n, xv = x, yv = y;
    const double sgn = x > y ? cl : (x < y ? -cl : 0.0);
    const double dssim = fma(yv, b[2], fma(2.0 * xv, b[1], b[0]));
    return (float)fma(-cs, dssim, sgn);
}

// The gradient. With `loss` given, one more workgroup than strips reduces the loss beside them.
__global__ __launch_bounds__(64) void k_ssim_bwd(LossViews vs, int nv, const float* __restrict__ x,
                                                 const float* __restrict__ y, const double* __restrict__ maps,
                                                 float* __restrict__ dl, Window11 g, double lam,
                                                 const double* __restrict__ partial, double* __restrict__ loss) {
    __shared__ double sm[3][kPatch];
    const int lane = threadIdx.x;
    if (loss && blockIdx.x == 0) {
        loss_by_wave(partial, vs, nv, lam, loss, lane);
        return;
    }
    const unsigned first = loss ? 1 : 0;
    const int64_t item = xcd_item(blockIdx.x - first, gridDim.x - first);  // neighbouring strips share an L2 and halos
    const Strip s = strip_of(vs, nv, item);
    const double* mc = maps + s.off * 3;
    const bool col = s.x0 + lane < s.v.width;
    const double n = 3.0 * (double)s.plane;
    double acc[3][10] = {};
    RowPair<double> even[3], odd[3];
    auto load = [&](RowPair<double> (&v)[3], int r) {
#pragma unroll
        for (int m = 0; m < 3; ++m) load_row(v[m], mc + m * s.plane, s, r, lane);
    };
    // row r, in v, which then takes row r + 2 (two rows of maps in flight per wave: with one the waves wait for
    // memory 60% of the time)
    auto step = [&](RowPair<double> (&v)[3], int r) {
#pragma unroll
        for (int m = 0; m < 3; ++m) put_row(sm[m], v[m], s, r, lane);
        wave_sync();
        const int q = r - kR;
        const int64_t p = s.off + (int64_t)max(q, 0) * s.v.width + min(s.x0 + lane, s.v.width - 1);
        const float xf = x[p], yf = y[p];
        load(v, r + 2);
        double b[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            double h = 0.0;
#pragma unroll
            for (int k = 0; k < 11; ++k) h = fma(g.w[k], sm[m][lane + k], h);
            b[m] = shift_in(acc[m], h, g);
        }
        wave_sync();
        if (q >= s.y0 && col) {
            dl[p] = gradient_of(xf, yf, b, n, lam);
        }
    };
    const int r1 = s.y1 + kR;
    load(even, s.y0 - kR);
    load(odd, s.y0 - kR + 1);
    for (int r = s.y0 - kR; r < r1; r += 2) {
        step(even, r);
        if (r + 1 < r1) step(odd, r + 1);
    }
}

// The same two passes by 16 x 16 tiles, one workgroup each, for images so small or narrow that strips leave the
// chip idle or their waves' lanes (loss_rows): a tile and its 5-pixel halo in LDS, the window as a row pass and
// a column pass over all of it at once, where a strip's wave takes its rows one after the other.
constexpr int kT = 16, kP = kT + 2 * kR;

struct Tile {
    LossView v;
    int x0, y0;
    int64_t plane, off;  // as in Strip
};

__device__ __forceinline__ Tile tile_of(const LossViews& vs, int nv, int64_t item) {
    int i = 0;
    while (i + 1 < nv && vs.v[i + 1].part_off <= item) ++i;
    Tile t;
    t.v = vs.v[i];
    const int k = (int)(item - t.v.part_off), tx = (t.v.width + kT - 1) / kT, per_c = tx * ((t.v.height + kT - 1) / kT);
    const int c = k / per_c, q = k - c * per_c;
    t.x0 = q % tx * kT;
    t.y0 = q / tx * kT;
    t.plane = (int64_t)t.v.width * t.v.height;
    t.off = t.v.pix_off * 3 + c * t.plane;
    return t;
}

// Element i of the patch: is it in the image, and where.
__device__ __forceinline__ bool patch_pixel(const Tile& t, int i, int64_t& p) {
    const int y = t.y0 - kR + i / kP, x = t.x0 - kR + i % kP;
    p = (int64_t)y * t.v.width + x;
    return x >= 0 && y >= 0 && x < t.v.width && y < t.v.height;
}

template <bool MAPS>
__global__ __launch_bounds__(kT * kT) void k_ssim_fwd_tile(LossViews vs, int nv, const float* __restrict__ x,
                                                           const float* __restrict__ y, double* __restrict__ maps,
                                                           double* __restrict__ partial, Window11 g) {
    __shared__ double sx[kP * kP], sy[kP * kP], row[4][kP * kT], red[2][kT * kT / kWave];
    const int tid = threadIdx.x, tx = tid % kT, ty = tid / kT;
    const Tile t = tile_of(vs, nv, blockIdx.x);
    for (int i = tid; i < kP * kP; i += kT * kT) {
        int64_t p;
        const bool in = patch_pixel(t, i, p);
        sx[i] = in ? x[t.off + p] : 0.0f;
        sy[i] = in ? y[t.off + p] : 0.0f;
    }
    __syncthreads();
    for (int i = tid; i < kP * kT; i += kT * kT) {
        double h[4];
        row_moments(sx + i / kT * kP, sy + i / kT * kP, i % kT, g, h);
#pragma unroll
        for (int m = 0; m < 4; ++m) row[m][i] = h[m];
    }
    __syncthreads();
    double mo[4] = {};
#pragma unroll
    for (int k = 0; k < 11; ++k)
#pragma unroll
        for (int m = 0; m < 4; ++m) mo[m] = fma(g.w[k], row[m][(ty + k) * kT + tx], mo[m]);
    double ssim = 0.0, l1 = 0.0;
    if (t.x0 + tx < t.v.width && t.y0 + ty < t.v.height) {
        const Ssim s = ssim_of(mo);
        const int c = (ty + kR) * kP + tx + kR;
        ssim = s.S;
        l1 = fabs(sx[c] - sy[c]);
        if (MAPS) {
            double* const mc = maps + t.off * 3 + (int64_t)(t.y0 + ty) * t.v.width + t.x0 + tx;
#pragma unroll
            for (int m = 0; m < 3; ++m) mc[m * t.plane] = s.d[m];
        }
    }
    ssim = wave_sum_f64(ssim);
    l1 = wave_sum_f64(l1);
    if (tid % kWave == 0) {
        red[0][tid / kWave] = ssim;
        red[1][tid / kWave] = l1;
    }
    __syncthreads();
    if (tid < 2) partial[2 * (int64_t)blockIdx.x + tid] = (red[tid][0] + red[tid][1]) + (red[tid][2] + red[tid][3]);
}

__global__ __launch_bounds__(kT * kT) void k_ssim_bwd_tile(LossViews vs, int nv, const float* __restrict__ x,
                                                           const float* __restrict__ y, const double* __restrict__ maps,
                                                           float* __restrict__ dl, Window11 g, double lam,
                                                           const double* __restrict__ partial, double* __restrict__ loss) {
    __shared__ double sm[3][kP * kP], row[3][kP * kT];
    const int tid = threadIdx.x, tx = tid % kT, ty = tid / kT;
    if (loss && blockIdx.x == 0) {
        if (tid < kWave) loss_by_wave(partial, vs, nv, lam, loss, tid);
        return;
    }
    const Tile t = tile_of(vs, nv, blockIdx.x - (loss ? 1 : 0));
    const double* const mc = maps + t.off * 3;
    for (int i = tid; i < kP * kP; i += kT * kT) {
        int64_t p;
        const bool in = patch_pixel(t, i, p);
#pragma unroll
        for (int m = 0; m < 3; ++m) sm[m][i] = in ? mc[m * t.plane + p] : 0.0;
    }
    const bool inside = t.x0 + tx < t.v.width && t.y0 + ty < t.v.height;
    const int64_t p = t.off + (int64_t)(t.y0 + ty) * t.v.width + t.x0 + tx;
    const float xf = inside ? x[p] : 0.0f, yf = inside ? y[p] : 0.0f;
    __syncthreads();
    for (int i = tid; i < kP * kT; i += kT * kT)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            double h = 0.0;
#pragma unroll
            for (int k = 0; k < 11; ++k) h = fma(g.w[k], sm[m][i / kT * kP + i % kT + k], h);
            row[m][i] = h;
        }
    __syncthreads();
    if (!inside) return;
    double b[3] = {};
#pragma unroll
    for (int k = 0; k < 11; ++k)
#pragma unroll
        for (int m = 0; m < 3; ++m) b[m] = fma(g.w[k], row[m][(ty + k) * kT + tx], b[m]);
    dl[p] = gradient_of(xf, yf, b, 3.0 * (double)t.plane, lam);
}

// The loss by a workgroup of its own, in the same order (the same bits): 256 threads per view, thread
// 64 u + lane with the sums that lane adds up in its u-th place above; four views at a time.
__global__ __launch_bounds__(1024) void k_loss_total(const double* __restrict__ partial, LossViews vs, int nv, double lam,
                                                     double* __restrict__ loss) {
    __shared__ double term[MEGS_MAX_VIEWS];
    __shared__ double2 part[1024];
    const int t = threadIdx.x % 256, group = threadIdx.x / 256;
    for (int i0 = 0; i0 < nv; i0 += 4) {
        const int i = i0 + group;
        if (i < nv) {
            double s = 0.0, l = 0.0;
            for (int64_t b = t; b < vs.v[i].n_part; b += 256) {
                const double2 p = reinterpret_cast<const double2*>(partial)[vs.v[i].part_off + b];
                s += p.x;
                l += p.y;
            }
            part[threadIdx.x] = make_double2(s, l);
        }
        __syncthreads();
        if (i < nv && t < kWave) {
            const double2* q = part + group * 256 + t;
            const double s = wave_sum_f64((q[0].x + q[64].x) + (q[128].x + q[192].x));
            const double l = wave_sum_f64((q[0].y + q[64].y) + (q[128].y + q[192].y));
            if (t == 0) term[i] = view_loss(vs.v[i], s, l, lam);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int i = 0; i < nv; ++i) s += term[i];
        loss[0] = s;
    }
}

// Adam (Kingma and Ba) with bias correction, FP32 arithmetic; the parameter is read from and
// written back to its storage dtype (round to nearest even).
__global__ __launch_bounds__(256) void k_adam(int64_t count, void* __restrict__ param, int dt,
                                              const float* __restrict__ grad, float* __restrict__ m,
                                              float* __restrict__ v, float lr, float b1, float b2, float eps,
                                              float bc1, float bc2) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = grad[i];
        const float mi = __fmaf_rn(b1, m[i], (1.0f - b1) * gi);
        const float vi = __fmaf_rn(b2, v[i], (1.0f - b2) * gi * gi);
        m[i] = mi;
        v[i] = vi;
        const float upd = lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
        store_elem(param, dt, i, load_elem(param, dt, i) - upd);
    }
}

}  // namespace

hipError_t launch_loss(const LossViews& vs, int nv, const float* x, const float* y, double* maps, double* partial,
                       double* loss, float* dl, const Window11& g, double lam, hipStream_t stream) {
    const int64_t items = vs.v[nv - 1].part_off + vs.v[nv - 1].n_part;  // strips, or tiles
    const bool tiles = vs.v[0].rows == 0, few = items <= kWaveSums;
    const dim3 grid((unsigned)items), block(tiles ? kT * kT : kWave);
    const auto fwd = tiles ? (dl ? k_ssim_fwd_tile<true> : k_ssim_fwd_tile<false>) : (dl ? k_ssim_fwd<true> : k_ssim_fwd<false>);
    hipLaunchKernelGGL(fwd, grid, block, 0, stream, vs, nv, x, y, maps, partial, g);
    if (!few || !dl)
        hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(nv > 1 ? 1024 : 256), 0, stream, partial, vs, nv, lam, loss);
    if (dl)
        hipLaunchKernelGGL(tiles ? k_ssim_bwd_tile : k_ssim_bwd, dim3((unsigned)items + (few ? 1 : 0)), block, 0, stream, vs,
                           nv, x, y, maps, dl, g, lam, partial, few ? loss : static_cast<double*>(nullptr));
    return hipGetLastError();
}

// Rows of a strip, or 0 for tiles. The strips above and below sum a strip's 10 rows of halo again, so tall strips
// cost least, but a strip is one wave's serial walk, and the chip's 1,024 SIMDs want waves: the rows that make
// (rows + 10) times (1 + strips per SIMD) least. Measured (forward + backward) in strips of 64 / 32 / 16 rows for a 1080p
// image 84 + 68, 74 + 62 and 74 + 63 us, in strips of 16 / 8 / 4 rows for one of 979 x 546 29 + 24, 35 + 28
// and 43 + 38 us, the whole loss with its gradient in strips of 4 / 2 / 1 rows for one of 240 x 180 23, 25
// and 30 us. That measure is some 1.2 times the strips' time in us where images are wide; tiles take 8 us and 0.0108 us
// each. The loss with its gradient in strips and in tiles: 64 x 64 16.9 and 10.0 us, 240 x 180 21.9 and 14.2, 480 x 270 29.6
// and 24.8, 640 x 360 38.8 and 37.0, 800 x 600 54 and 70, 16384 x 1 17.6 and 27.1; narrow images leave lanes of a
// strip's wave without a column: 1 x 16384 66 and 32 us, 16 x 16384 67 and 36, 48 x 16384 78 and 106.
int loss_rows(const LossViews& vs, int nv) {
    int best = 64;
    double least = 1e300, tiles = 0.0;
    for (int i = 0; i < nv; ++i) tiles += (double)loss_partials(vs.v[i].width, vs.v[i].height, 0);
    for (int rows = 64; rows >= 2; rows /= 2) {
        double strips = 0.0;
        for (int i = 0; i < nv; ++i) strips += (double)loss_partials(vs.v[i].width, vs.v[i].height, rows);
        const double t = (rows + 2 * kR) * (1.0 + strips / 1024.0);
        if (t < least) {
            least = t;
            best = rows;
        }
    }
    return 8.0 + 0.0108 * tiles < 0.85 * least ? 0 : best;
}

int64_t loss_partials(int width, int height, int rows) {
    if (rows == 0) return 3ll * ((width + kT - 1) / kT) * ((height + kT - 1) / kT);
    return 3ll * ((width + kWave - 1) / kWave) * ((height + rows - 1) / rows);
}

hipError_t launch_adam(int64_t count, void* param, int dt, const float* grad, float* m, float* v, float lr, float b1,
                       float b2, float eps, int step, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    const float bc1 = (float)(1.0 - pow((double)b1, step)), bc2 = (float)(1.0 - pow((double)b2, step));
    int64_t blocks = (count + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(256), 0, stream, count, param, dt, grad, m, v, lr, b1, b2,
                       eps, bc1, bc2);
    return hipGetLastError();
}

}  // namespace megs
