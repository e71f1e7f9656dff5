// blend.hip -- front-to-back alpha blending (forward) and its back-to-front replay (backward),
// gfx950: per-tile workgroup kernels, and the sub-tile kernels further down (one wave64 per 8 x 8
// sub-tile walking its tile's list; the configuration the benchmark runs).
//
// Compositing follows Sec. 3.1: C = sum_i c_i alpha_i prod_{j<i}(1 - alpha_j), alpha_i = o_i times
// the 2D Gaussian at the pixel, with the 3DGS conventions (alpha clamped to 0.99, fragments below
// 1/255 skipped, stop before the transmittance would fall under 1e-4).
//
// Mapping to CDNA4: a workgroup of 1, 2 or 4 wave64s per (view, tile), TILE^2 / (64 waves) pixels
// per lane, each wave owning a compact block of the tile (the whole tile, a half or a quadrant);
// every LDS read of a staged Gaussian is reused by all of a lane's pixels, and a wave skips a
// Gaussian whose footprint box misses its block or that reaches none of its pixels. More waves
// per tile shorten the serial walk of long tile lists (the latency of the densest tiles bounds a
// launch); one wave needs no workgroup barrier at all. Gaussians of the tile's list are staged into LDS in batches
// (one record per lane per load, gathered through the sorted record indices); their means are
// made tile-relative in FP64 while staging, so the per-fragment arithmetic works on small FP32
// offsets. The wave stops as soon as all its pixels have terminated.
//
// The backward walks each tile's list from the largest per-pixel last index down to 0, recovers
// the transmittance in front of each fragment by division, carries the colour seen behind the
// fragment (as its dot product with the pixel's colour gradient, the only form the gradient
// uses), and accumulates nine per-record sums: e = dL/do_eff of each unclamped fragment,
// its moments e w1, e w2, e w1^2, e w1 w2, e w2^2 in the exponent's factors (Staged; the exponent's
// gradient is o_eff e, so the projection backward turns them into the mean and conic gradients once
// per record), and the colour gradient. They are summed over the wave's pixels (the per-tile kernels with a
// transposed butterfly of permlane swaps and DPP adds, the sub-tile kernel through LDS rows) and added to the
// record's slot with nine lanes of one hardware float atomic, only when some lane of the wave contributed.
#include "megs_internal.hpp"

#include <utility>

namespace megs {
namespace {

// A record as the blends use it, its shape folded into the exponent's affine factors over the
// pixel centres of one frame (a tile or a sub-tile, origin (X0, Y0), pixel centre (px, py) relative
// to it): the exponent in log2 units is -(w1^2 + w2^2) with
//   w1 = ax px + ay py + c1,  w2 = by py + c2,
// ax = kQ2 l11, ay = kQ2 l11 r, by = kQ2 l22 (Shape), c1 = kQ2 l11 ((X0 - u) + r (Y0 - v)) and
// c2 = kQ2 l22 (Y0 - v). c1 and c2 are formed in FP64 from the FP64 mean and ratio, so the
// cancellation along a thin footprint happens there, once per staged record; per pixel the FP32
// terms stay within a frame's width of the footprint. The backward needs the conic itself only per
// record, in the projection backward.
struct Staged {
    float4 box; // frame-relative bounding box of the cutoff ellipse: x - rx, x + rx, y - ry, y + ry
    float4 p0;  // ax, ay, c1, o
    float4 p1;  // by, c2, r, g
    float b;    // blue
};

// An entry kept for an 8x8 sub-tile, as the sub-tile backward reads it back from LDS: the staged
// record without its box (the box only decides whether the entry is kept), plus the entry's list
// position and a record index, so that one LDS address serves every read of the entry (48 bytes).
struct Kept {
    float4 p0, p1;   // as in Staged
    float b;         // as in Staged
    uint32_t pos1;   // one past the entry's list position (relative to the tile's range start)
    uint64_t slot;   // the record's first element in the per-record sums (grad2d_index)
};
static_assert(sizeof(Kept) == 48 && offsetof(Kept, slot) % 8 == 0, "kept entries are 48 bytes, slot 8-aligned");

// &lds[k] through a VGPR copy of its byte offset. The compiler cannot rebuild the result of an asm
// statement, so every read of the entry (and, with immediate offsets, of the entries after it)
// shares this one address register, where it would otherwise re-derive the address from the
// scalar index with a VALU move before each group of reads.
__device__ __forceinline__ const Kept* kept_at(const Kept* lds, int k) {
    uint32_t off;
    asm("v_mov_b32 %0, %1" : "=v"(off) : "s"(k * (int)sizeof(Kept)));
    return reinterpret_cast<const Kept*>(reinterpret_cast<const char*>(lds) + off);
}

// Pixel layout of a (TILE, WAVES) workgroup: wave w owns a WW x WH block of the tile (the whole
// tile, its upper/lower half, or one quadrant), its lanes cover LW x LH pixels per slot, and
// pixel slot j of a lane lies LH j rows below slot 0. Compact blocks let a wave skip every staged
// Gaussian whose footprint box misses its block, which is most of them for small footprints.
template <int TILE, int WAVES>
struct Layout {
    static constexpr int WW = WAVES == 4 ? TILE / 2 : TILE;
    static constexpr int WH = WAVES == 1 ? TILE : TILE / 2;
    static constexpr int LW = WW;
    static constexpr int LH = 64 / LW;
    static constexpr int PPT = WW * WH / 64;
    static_assert(LW * LH == 64 && PPT * 64 == WW * WH, "tile and wave count mismatch");
    __device__ static int wx0(int wave) { return WAVES == 4 ? (wave & 1) * WW : 0; }
    __device__ static int wy0(int wave) { return WAVES == 4 ? (wave >> 1) * WH : (WAVES == 2 ? wave * WH : 0); }
};

// Stages record g for the frame with origin (x0, y0) (pixel coordinates of its top-left corner). Only
// t = (X0 - u) + r (Y0 - v), which cancels along a thin footprint, needs FP64; it is rounded once, and
// c1 = ax t and c2 = by (Y0 - v) then err by about one FP32 rounding of their own size. With box set,
// also the frame-relative box of the cutoff ellipse {d' Q d <= k}: its half-extents are sqrt(k A) and
// sqrt(k C) for the covariance Q^-1 = [[A, B], [B, C]], which the factors give without cancellation as
// A = (r / l22)^2 + 1 / l11^2 and C = 1 / l22^2; widened by 1e-3 relative and 1e-2 px, far more than
// FP32 rounding moves them, so every pixel with alpha >= 1/255 lies inside.
struct RecVecs {  // a record's three vectors
    float4 q0, q1, q2;
};
__device__ __forceinline__ RecVecs gather(const BlendArgs& a, uint32_t g) {
    const float4* q = reinterpret_cast<const float4*>(a.rec + g);
    return RecVecs{q[0], q[1], q[2]};
}

__device__ __forceinline__ Staged staged_of(const RecVecs& v, double x0, double y0, bool box) {
    const float4 &q0 = v.q0, &q1 = v.q1, &q2 = v.q2;
    const double mx = __hiloint2double(__float_as_int(q0.y), __float_as_int(q0.x));
    const double my = __hiloint2double(__float_as_int(q0.w), __float_as_int(q0.z));
    const double r = __hiloint2double(__float_as_int(q1.y), __float_as_int(q1.x));
    const double dx0 = x0 - mx, dy0 = y0 - my;
    const float t = (float)fma(r, dy0, dx0), dxf = (float)dx0, dyf = (float)dy0;
    const float ax = kQ2 * q1.z, by = kQ2 * q1.w;
    Staged s;
    s.p0 = make_float4(ax, ax * (float)r, ax * t, q2.x);
    s.p1 = make_float4(by, by * dyf, q2.y, q2.z);
    s.b = q2.w;
    s.box = make_float4(0.f, -1.f, 0.f, -1.f);
    if (box) {
        const float cut = cutoff_of(q2.x);
        const float il22 = __builtin_amdgcn_rcpf(q1.w), ra = (float)r * il22, il11 = __builtin_amdgcn_rcpf(q1.z);
        const float rx = __builtin_amdgcn_sqrtf(cut * __fmaf_rn(ra, ra, il11 * il11)) * 1.001f + 0.01f;
        const float ry = __builtin_amdgcn_sqrtf(cut) * il22 * 1.001f + 0.01f;
        s.box = make_float4(-dxf - rx, -dxf + rx, -dyf - ry, -dyf + ry);
    }
    return s;
}

__device__ __forceinline__ void stage(const BlendArgs& a, uint32_t g, double x0, double y0, Staged* dst,
                                      bool box = true) {
    *dst = staged_of(gather(a, g), x0, y0, box);
}

// Does the pixel block [x0, x1] x [y0, y1] (tile-relative, centres at +0.5) meet the staged
// footprint's box? Wave-uniform when the block is.
__device__ __forceinline__ bool box_meets(const float4& b, int x0, int x1, int y0, int y1) {
    return (x0 + 0.5f <= b.y) && (x1 + 0.5f >= b.x) && (y0 + 0.5f <= b.w) && (y1 + 0.5f >= b.z);
}

// Alpha test of one fragment (no branches): pass = alpha >= 1/255 with alpha = min(o G, 0.99) and
// G = 2^(-(w1^2 + w2^2)) (Staged). The compositing rule also skips fragments with a positive
// exponent, which a sum of squares never is. The threshold is tested on the unclamped value (the
// same decision for any number, and a NaN fails it). The forward and the backward call this same
// function, so both take identical decisions; w1 and w2 are returned for the backward's moments.
__device__ __forceinline__ bool alpha_of(float w1, float w2, float o, float& G, float& alpha, bool& clamped) {
    const float q2 = __fmaf_rn(-w1, w1, -(w2 * w2));
    G = __builtin_amdgcn_exp2f(q2);
    const float raw = o * G;
    clamped = raw > kAlphaMax;
    alpha = fminf(raw, kAlphaMax);
    // keeps the clamp next to the product: moved into the callers' blend branches, it would need a
    // separate NaN-quieting step there
    asm volatile("" : "+v"(alpha));
    return raw >= kAlphaMin;
}

template <class E>  // Staged or Kept
__device__ __forceinline__ bool frag(const E& s, float px, float py, float& w1, float& w2, float& G,
                                     float& alpha, bool& clamped) {
    w1 = __fmaf_rn(s.p0.x, px, __fmaf_rn(s.p0.y, py, s.p0.z));
    w2 = __fmaf_rn(s.p1.x, py, s.p1.y);
    return alpha_of(w1, w2, s.p0.w, G, alpha, clamped);
}

struct TileCtx {
    int view;
    int64_t tile;
    int x0, y0, width, height;
    int64_t pix_off;
    float bg[3];
};

__device__ __forceinline__ TileCtx tile_ctx(const BlendArgs& a, int view, int64_t t, int TILE) {
    TileCtx c;
    c.tile = t;
    c.view = view;
    const ViewInfo& vw = a.views[c.view];
    const int64_t lt = t - vw.tile_off;
    c.x0 = (int)(lt % vw.tiles_x) * TILE;
    c.y0 = (int)(lt / vw.tiles_x) * TILE;
    c.width = vw.width;
    c.height = vw.height;
    c.pix_off = vw.pix_off;
    c.bg[0] = vw.bg[0]; c.bg[1] = vw.bg[1]; c.bg[2] = vw.bg[2];
    return c;
}

// Next work item: blockIdx.x when not persistent, else pulled from the queue counter (thread 0
// takes the item, the workgroup reads it back through LDS).
__device__ __forceinline__ int64_t next_tile(const BlendArgs& a, int64_t prev, bool persistent, uint32_t* slot) {
    if (!persistent) return prev < 0 ? (int64_t)blockIdx.x : a.n_tiles;
    __syncthreads();
    if (threadIdx.x == 0) *slot = atomicAdd(a.queue, 1u);
    __syncthreads();
    return (int64_t)*slot;
}

// Workgroup of WAVES wave64s per tile, PPT = TILE^2 / (64 WAVES) pixels per lane, each wave owning
// one compact block of the tile (Layout).
template <int TILE, int WAVES, bool STATS, bool IMP>
__global__ __launch_bounds__(64 * WAVES) void k_blend_fwd(BlendArgs a, int batch, int persistent) {
    using Ly = Layout<TILE, WAVES>;
    constexpr int NT = 64 * WAVES, PPT = Ly::PPT, LH = Ly::LH;
    extern __shared__ Staged lds[];
    uint32_t* lds_id = reinterpret_cast<uint32_t*>(lds + batch);  // record ids (importance only)
    __shared__ uint32_t work_slot;
    const int tid = threadIdx.x, lane = __lane_id(), wv = tid / 64;
    const int bx0 = Ly::wx0(wv), by0 = Ly::wy0(wv);   // this wave's block
    const int lx = bx0 + lane % Ly::LW, ly = by0 + lane / Ly::LW;
    uint32_t n_blended = 0, n_evaluated = 0;
    for (int64_t t = next_tile(a, -1, persistent, &work_slot); t < a.n_tiles;
         t = next_tile(a, t, persistent, &work_slot)) {
        const TileCtx c = tile_ctx(a, view_of_tile(a.views, a.nv, t), t, TILE);
        const uint2 rg = a.ranges[t];
        // T < 0 marks a pixel that has terminated (|T| is its final transmittance) or lies outside
        // the image; this keeps the per-pixel state in float registers.
        float T[PPT], C[PPT][3];
        uint32_t last[PPT];
        bool mine = false;
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            T[j] = (c.x0 + lx < c.width && c.y0 + ly + LH * j < c.height) ? 1.0f : -1.0f;
            C[j][0] = C[j][1] = C[j][2] = 0.0f;
            last[j] = 0;
            mine |= T[j] > 0.0f;
        }
        const float px = lx + 0.5f;
        for (uint32_t base = rg.x; base < rg.y; base += batch) {
            // the workgroup stops once every pixel of the tile has terminated
            if (WAVES > 1 ? !__syncthreads_or(mine) : !__any(mine)) break;
            const int cnt = (int)min((uint32_t)batch, rg.y - base);
            for (int q = tid; q < cnt; q += NT) {
                const uint32_t g = a.vals[base + q];
                stage(a, g, (double)c.x0, (double)c.y0, &lds[q]);
                if (IMP) lds_id[q] = g;
            }
            __syncthreads();
            for (int jj = 0; jj < cnt; ++jj) {
                // the wave stops once all its pixels have terminated; checked every 4 Gaussians
                // (a terminated pixel has T < 0 and takes no further fragment in between)
                if ((jj & 3) == 0 && !__any(mine)) break;
                const float4 box = lds[jj].box;
                // wave-uniform: skip a Gaussian whose footprint box misses this wave's block
                if (!box_meets(box, bx0, bx0 + Ly::WW - 1, by0, by0 + Ly::WH - 1)) continue;
                const Staged s = lds[jj];
                const uint32_t pos = base + jj - rg.x;
                float alpha[PPT];
                bool pass[PPT];
                bool any_pass = false;
#pragma unroll
                for (int j = 0; j < PPT; ++j) {
                    pass[j] = false;
                    alpha[j] = 0.0f;
                    // this wave's pixel rows of slot j; skip the slot when the footprint misses them
                    if (PPT > 1 && !box_meets(box, bx0, bx0 + Ly::WW - 1, by0 + LH * j, by0 + LH * j + LH - 1))
                        continue;
                    float w1, w2, G;
                    bool clamped;
                    pass[j] = frag(s, px, ly + LH * j + 0.5f, w1, w2, G, alpha[j], clamped) & (T[j] > 0.0f);
                    any_pass |= pass[j];
                    if (STATS) n_evaluated += T[j] > 0.0f;
                }
                if (!__any(any_pass)) continue;  // wave-uniform: none of this wave's pixels is hit
                float wsum = 0.0f;
                mine = false;
#pragma unroll
                for (int j = 0; j < PPT; ++j) {
                    const float Tn = T[j] * (1.0f - alpha[j]);
                    const bool term = pass[j] & (Tn < kTMin);
                    const bool incl = pass[j] & !term;
                    const float w = incl ? alpha[j] * T[j] : 0.0f;
                    if (IMP) wsum += w;
                    C[j][0] = __fmaf_rn(w, s.p1.z, C[j][0]);
                    C[j][1] = __fmaf_rn(w, s.p1.w, C[j][1]);
                    C[j][2] = __fmaf_rn(w, s.b, C[j][2]);
                    T[j] = incl ? Tn : (term ? -T[j] : T[j]);
                    last[j] = incl ? pos + 1 : last[j];
                    mine |= T[j] > 0.0f;
                    if (STATS) n_blended += incl;
                }
                if (IMP) {
                    // importance score: blending weights of this record summed over the wave's pixels
#pragma unroll
                    for (int d = 32; d >= 1; d >>= 1) wsum += __shfl_xor(wsum, d);
                    if (lane == 0 && wsum != 0.0f)
                        unsafeAtomicAdd(a.importance + (lds_id[jj] - (int64_t)c.view * a.n), wsum);
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const int x = c.x0 + lx, y = c.y0 + ly + LH * j;
            if (x >= c.width || y >= c.height) continue;
            const int64_t p = (int64_t)y * c.width + x;
            const int64_t plane = (int64_t)c.width * c.height;
            float* img = a.image + 3 * c.pix_off;
            const float Tf = fabsf(T[j]);
            img[p] = __fmaf_rn(Tf, c.bg[0], C[j][0]);
            img[plane + p] = __fmaf_rn(Tf, c.bg[1], C[j][1]);
            img[2 * plane + p] = __fmaf_rn(Tf, c.bg[2], C[j][2]);
            a.T_final[c.pix_off + p] = Tf;
            a.last[c.pix_off + p] = last[j];
        }
    }
    if (STATS) {
        unsigned long long nb = n_blended, ne = n_evaluated;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            nb += __shfl_xor(nb, d);
            ne += __shfl_xor(ne, d);
        }
        if (lane == 0) {
            atomicAdd(a.stats, nb);
            atomicAdd(a.stats + 1, ne);
        }
    }
}

// Cross-lane helpers on gfx950 VALU data paths (no LDS traffic). swap32(a, b): lanes 32-63 of a
// trade places with lanes 0-31 of b; swap16 does the same between odd and even 16-lane rows of each
// half. mirror16 / mirror8: the value of lane 15 - i (i - 8 ... ) within each 16- / 8-lane group.
__device__ __forceinline__ void swap32(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {  // lanes whose source lane is invalid read 0
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kQuadXor1 = 0xb1, kQuadXor2 = 0x4e, kRowMirror = 0x140, kRowHalfMirror = 0x141;
constexpr int kRowBcast15 = 0x142;  // lane 15 of the previous 16-lane row (rows 1-3)
constexpr int kRowBcast31 = 0x143;  // lane 31 (rows 2-3)
constexpr int kLaneSum8 = 63;       // the lane that ends with the wave total of v[8] in wave_sum9

// Sum over one 8-lane group (every lane of the group ends with the total).
__device__ __forceinline__ float sum8(float y) {
    y += dpp<kQuadXor1>(y);
    y += dpp<kQuadXor2>(y);
    y += dpp<kRowHalfMirror>(y);
    return y;
}

// Sum over the wave, in lane 63: within each 16-lane row, then across rows with the two row broadcasts.
__device__ __forceinline__ float wave_sum(float y) {
    y = sum8(y);
    y += dpp<kRowMirror>(y);
    y += dpp<kRowBcast15>(y);
    y += dpp<kRowBcast31>(y);
    return y;
}

// Sum of v[0..8] over the wave: a transposed butterfly. After the swaps, lane group (b5 b4 b3) of
// the lane index holds partial sums of v[4 b5 + 2 b4 + b3] only; the last three steps finish
// them within each 8-lane group, so every lane of group m (lanes 8m..8m+7) holds the total of v[m].
// v[8] is summed within each 16-lane row, then across rows with the two row broadcasts, the last of
// which writes only lanes 60-63: on return lanes 8m (m < 8) hold the total of v[m] and lane
// kLaneSum8 (63) the total of v[8].
__device__ __forceinline__ float wave_sum9(const float v[9]) {
    const int lane = __lane_id();
    float w4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // lanes < 32 gather v[i] pairs, lanes >= 32 v[i + 4] pairs
        float a = v[i], b = v[i + 4];
        swap32(a, b);
        w4[i] = a + b;
    }
    float w2[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // even rows keep w4[i], odd rows w4[i + 2]
        float a = w4[i], b = w4[i + 2];
        swap16(a, b);
        w2[i] = a + b;
    }
    const bool b3 = lane & 8;      // lanes 0-7 of a row pair with lanes 15..8 through the mirror
    const float y = (b3 ? w2[1] : w2[0]) + dpp<kRowMirror>(b3 ? w2[0] : w2[1]);
    float out = sum8(y);
    // (all rows take part in the first broadcast so it folds into one DPP add; only row 3's result,
    // which reads a valid lane, is used)
    float z = sum8(v[8]);
    z += dpp<kRowMirror>(z);   // row sums R0..R3 in every lane of their row
    z += dpp<kRowBcast15>(z);  // row 1: R0 + R1, row 3: R2 + R3
    // Lanes 60-63 (row mask 8: row 3; bank mask 8: its lanes 12-15) take R2 + R3 + lane 31's
    // R0 + R1 in place of the total of v[7], which lane 56 also holds; every other lane keeps out.
    // This masked DPP add has no builtin form (a masked DPP move keeps the old value in the move,
    // not in the sum), so it is written out, after the two wait states a DPP read of a VGPR that
    // the previous VALU instruction wrote needs.
    asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_bcast:31 row_mask:0x8 bank_mask:0x8"
                 : "+v"(out)
                 : "v"(z));
    return out;
}

// DET: instead of float atomics into the record's gradient, the tile's 9 sums for each list
// position go to that position's own slot a.grad_pair[pos] (written by exactly one workgroup), and
// a separate pass adds each record's slots in a fixed order: bit-reproducible gradients.
template <int TILE, int WAVES, bool DET>
__global__ __launch_bounds__(64 * WAVES) void k_blend_bwd(BlendArgs a, int batch, int persistent) {
    using Ly = Layout<TILE, WAVES>;
    constexpr int NT = 64 * WAVES, PPT = Ly::PPT, LH = Ly::LH;
    extern __shared__ Staged lds[];
    uint32_t* lds_id = reinterpret_cast<uint32_t*>(lds + batch);
    float* lds_part = reinterpret_cast<float*>(lds_id + batch);  // [batch][WAVES][9] (WAVES > 1)
    __shared__ uint32_t work_slot;
    __shared__ uint32_t red_slot[WAVES];
    const int tid = threadIdx.x, lane = __lane_id(), wv = tid / 64;
    const int bx0 = Ly::wx0(wv), by0 = Ly::wy0(wv);   // this wave's block
    const int lx = bx0 + lane % Ly::LW, ly = by0 + lane / Ly::LW;
    const float px = lx + 0.5f;
    for (int64_t t = next_tile(a, -1, persistent, &work_slot); t < a.n_tiles;
         t = next_tile(a, t, persistent, &work_slot)) {
        const TileCtx c = tile_ctx(a, view_of_tile(a.views, a.nv, t), t, TILE);
        const uint2 rg = a.ranges[t];
        const int64_t plane = (int64_t)c.width * c.height;
        float T[PPT], P[PPT], dl[PPT][3];  // P = S . dL/dC, as in the sub-tile backward
        uint32_t lst[PPT];
        uint32_t maxlast = 0;
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const int x = c.x0 + lx, y = c.y0 + ly + LH * j;
            const bool inside = x < c.width && y < c.height;
            const int64_t p = (int64_t)y * c.width + x;
            T[j] = inside ? a.T_final[c.pix_off + p] : 1.0f;
            lst[j] = inside ? a.last[c.pix_off + p] : 0u;
            const float* dimg = a.dl + 3 * c.pix_off;
            dl[j][0] = inside ? dimg[p] : 0.f;
            dl[j][1] = inside ? dimg[plane + p] : 0.f;
            dl[j][2] = inside ? dimg[2 * plane + p] : 0.f;
            P[j] = __fmaf_rn(c.bg[0], dl[j][0], __fmaf_rn(c.bg[1], dl[j][1], c.bg[2] * dl[j][2]));
            maxlast = max(maxlast, lst[j]);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) maxlast = max(maxlast, (uint32_t)__shfl_xor((int)maxlast, d));
        const uint32_t wave_last = maxlast;
        if (WAVES > 1) {
            if (lane == 0) red_slot[wv] = maxlast;
            __syncthreads();
            for (int w = 0; w < WAVES; ++w) maxlast = max(maxlast, red_slot[w]);
            __syncthreads();
        }
        for (uint32_t end = rg.x + maxlast; end > rg.x;) {
            const uint32_t beg = end - rg.x > (uint32_t)batch ? end - batch : rg.x;
            const int cnt = (int)(end - beg);
            for (int q = tid; q < cnt; q += NT) {
                const uint32_t g = a.vals[end - 1 - q];
                stage(a, g, (double)c.x0, (double)c.y0, &lds[q]);
                lds_id[q] = g;
            }
            __syncthreads();
            for (int jj = 0; jj < cnt; ++jj) {
                const uint32_t pos = end - 1 - jj - rg.x;
                bool any_incl = false;
                float acc[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) acc[i] = 0.f;
                // wave-uniform: positions past every pixel's last, and Gaussians whose footprint
                // box misses this wave's block, are skipped
                if (pos < wave_last && box_meets(lds[jj].box, bx0, bx0 + Ly::WW - 1, by0, by0 + Ly::WH - 1)) {
                    const Staged s = lds[jj];
                    float alpha[PPT], G[PPT], w1s[PPT], w2s[PPT];
                    bool incl[PPT], clamped[PPT];
#pragma unroll
                    for (int j = 0; j < PPT; ++j) {
                        incl[j] = false;
                        alpha[j] = 0.0f; G[j] = 0.0f; w1s[j] = 0.0f; w2s[j] = 0.0f; clamped[j] = false;
                        if (PPT > 1 &&
                            !box_meets(s.box, bx0, bx0 + Ly::WW - 1, by0 + LH * j, by0 + LH * j + LH - 1))
                            continue;
                        incl[j] = frag(s, px, ly + LH * j + 0.5f, w1s[j], w2s[j], G[j], alpha[j], clamped[j]) &
                                  (pos < lst[j]);
                        any_incl |= incl[j];
                    }
                    any_incl = __any(any_incl);
                    if (any_incl) {
#pragma unroll
                        for (int j = 0; j < PPT; ++j) {
                            const float al = incl[j] ? alpha[j] : 0.0f;
                            const float Ti = T[j] * __builtin_amdgcn_rcpf(1.0f - al);
                            const float w = al * Ti;
                            const float dcs =
                                __fmaf_rn(s.p1.z, dl[j][0], __fmaf_rn(s.p1.w, dl[j][1], s.b * dl[j][2])) - P[j];
                            acc[6] = __fmaf_rn(w, dl[j][0], acc[6]);
                            acc[7] = __fmaf_rn(w, dl[j][1], acc[7]);
                            acc[8] = __fmaf_rn(w, dl[j][2], acc[8]);
                            const float dal = Ti * dcs;
                            P[j] = __fmaf_rn(al, dcs, P[j]);
                            T[j] = incl[j] ? Ti : T[j];
                            const bool live = incl[j] & !clamped[j];
                            // dL/do_eff of the fragment; its exponent gradient is o_eff times this
                            const float e = live ? G[j] * dal : 0.0f;
                            const float w1 = w1s[j], w2 = w2s[j];
                            acc[5] += e;
                            const float m1 = e * w1, m2 = e * w2;
                            acc[0] += m1;
                            acc[1] += m2;
                            acc[2] = __fmaf_rn(m1, w1, acc[2]);
                            acc[3] = __fmaf_rn(m1, w2, acc[3]);
                            acc[4] = __fmaf_rn(m2, w2, acc[4]);
                        }
                    }
                }
                if (WAVES == 1) {
                    if (!any_incl) continue;
                    const float tot = wave_sum9(acc);
                    if (DET) {
                        float* slot = a.grad_pair + 9 * (int64_t)(end - 1 - jj);
                        if ((lane & 7) == 0) slot[lane >> 3] = tot;
                        if (lane == kLaneSum8) slot[8] = tot;
                        continue;
                    }
                    // one 9-lane atomic: lanes 0, 8, .., 56 add sums 0..7, lane 63 adds sum 8
                    if ((lane & 7) == 0 || lane == kLaneSum8)
                        unsafeAtomicAdd(a.grad2d + grad2d_index(lds_id[jj], lane == kLaneSum8 ? 8 : lane >> 3), tot);
                } else {
                    // per-wave partial sums to LDS; summed across waves after the batch
                    float tot = 0.f;
                    if (any_incl) tot = wave_sum9(acc);
                    float* part = lds_part + ((int64_t)jj * WAVES + wv) * 9;
                    if ((lane & 7) == 0) part[lane >> 3] = tot;
                    if (lane == kLaneSum8) part[8] = tot;
                }
            }
            __syncthreads();
            if (WAVES > 1) {
                for (int i = tid; i < cnt * 9; i += NT) {
                    const int jj = i / 9, comp = i - jj * 9;
                    float sum = 0.f;
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) sum += lds_part[((int64_t)jj * WAVES + w) * 9 + comp];
                    if (DET)
                        a.grad_pair[9 * (int64_t)(end - 1 - jj) + comp] = sum;
                    else if (sum != 0.f)
                        unsafeAtomicAdd(a.grad2d + grad2d_index(lds_id[jj], comp), sum);
                }
                __syncthreads();
            }
            end = beg;
        }
    }
}

// ------------------------------------------------------------- sub-tile kernels ----
// One wave64 per 8 x 8 sub-tile of a 16 x 16 or 32 x 32 tile: the tile's sorted list (and so the
// key table and its sort) stays at the tile's size, while blending runs at sub-tile size. The wave
// takes 64 entries at a time, one per lane: those of the list that the tile keys flag for the sub-tile
// (FlagQueue; the emission tested the entry's ellipse against it), or, without flags, the list's next 64,
// of which those whose footprint reaches the sub-tile are kept. The kept entries are packed in list order
// into the wave's own LDS (ballot prefix) and blended. Entries are staged relative to the sub-tile's corner,
// so each pixel's exponent factors stay within eight pixels of it. Sub-tiles of a tile never wait for each
// other: there is no workgroup barrier anywhere.

// LDS written by some lanes of a wave and read by others: order the wave's accesses.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Without the work queue a workgroup runs one item. Workgroups are handed out in order, each to the next
// XCD in turn, and one whose XCD is full holds up all behind it; so the XCDs have to be equally busy at
// every moment, and the longest items must not come last. Where with_order says so, the tiles are run by falling
// length of their lists (k_tile_order), each XCD taking all sub-tiles of a tile (forward) or of four tiles
// (backward) in turn, which share the list and the records in its L2; elsewhere each XCD runs one contiguous
// eighth (forward) or the sub-tiles run as numbered (backward).
//
// With the work queue (persistent launch) the items are split into kSlices contiguous slices, one per
// XCD (the same eighths as above), with one counter each (queue[s * kQueueStride], one per 256 bytes).
// A wave pulls one item at a time from the slice of the XCD it runs on (the XCC_ID hardware register),
// so a tile's sub-tiles and its list stay in one L2. Once its slice is drained it reads all the
// counters at once (one lane each) and moves to the first slice with items left, its own XCD's first. Every
// pull advances a counter, so every item is handed out exactly once, and a wave ends when every counter has
// passed its slice's end. The register only steers locality: any value in it gives the same result. Measured on the 8-view 1080p workload (forward / backward blend): with the
// eight counters in one cache line, pulls serialised on it and the blends took 3.7 / 4.3 ms instead of
// 0.99 / 2.24 ms for one workgroup per item; a line per counter brings them to 1.35 / 2.48 ms. More
// slices per XCD (32, 64) lost L2 locality, and several items per pull lost balance (both slower).
// What remains is not the queue: issuing each next pull ahead of its item (its round trip overlapping
// the item's work) changed nothing, and a static assignment without atomics took as long (1.32 ms).
constexpr int kSlices = kXcds;
static_assert(kSlices % kXcds == 0 && kSlices <= 64 && kSlices * kQueueStride <= kQueueWords, "slice counters");

// The tiles by falling list length (to an eighth of an octave), for next_item. One workgroup counts and
// places up to kOrderSlice of them; more tiles are ordered in slices of equal size, which run one after the
// other. Each of the 256 lengths has eight counters, one per lane & 7, so that a wave of equally short lists
// does not queue up at one (14.6 us for 16,320 tiles, 5.3 us for 2,040: two passes of latency; in one slice
// a million tiles would take some 0.7 ms).
constexpr int kOrderSlice = 16384;
constexpr uint32_t kEmptyTile = 1u << 31;  // set in the order beside a tile whose list is empty
constexpr int kOrderThreads = 1024;
__global__ __launch_bounds__(kOrderThreads) void k_tile_order(const uint2* __restrict__ ranges, uint32_t n_tiles,
                                                              uint32_t slice, uint32_t* __restrict__ order) {
    constexpr int kCounters = 256 * 8, kEach = 8;  // 32 octaves of 8 lengths of 8 counters
    static_assert(kCounters == 2 * kOrderThreads, "two counters a thread");
    __shared__ uint32_t count[kCounters];
    __shared__ uint32_t wave_total[kOrderThreads / kWave];
    const int t = threadIdx.x;
    const uint32_t first = blockIdx.x * slice, n = min(slice, n_tiles - first);
    auto for_tiles = [&](auto f) {
        for (uint32_t i0 = 0; i0 < n; i0 += kOrderThreads * kEach) {
            uint2 r[kEach];
#pragma unroll
            for (int j = 0; j < kEach; ++j) r[j] = ranges[first + min(i0 + j * kOrderThreads + t, n - 1u)];
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                const uint32_t i = i0 + j * kOrderThreads + t;
                // the float of length + 1 >= 1: exponent and three bits of the fraction, falling
                const uint32_t b = 255u - ((__float_as_uint((float)(r[j].y - r[j].x + 1u)) >> 20) - (127u << 3));
                if (i < n) f(i, b * 8u + (t & 7));
            }
        }
    };
    count[t] = count[t + kOrderThreads] = 0;
    __syncthreads();
    for_tiles([&](uint32_t, uint32_t b) { atomicAdd(&count[b], 1u); });
    __syncthreads();
    const uint32_t c0 = count[2 * t], c1 = count[2 * t + 1];
    uint32_t inc = c0 + c1;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, kWave);
        if (__lane_id() >= d) inc += y;
    }
    if (__lane_id() == kWave - 1) wave_total[t / kWave] = inc;
    __syncthreads();
    for (int w = 0; w < t / kWave; ++w) inc += wave_total[w];
    count[2 * t] = inc - c0 - c1;
    count[2 * t + 1] = inc - c1;
    __syncthreads();
    for_tiles([&](uint32_t i, uint32_t b) {
        order[first + atomicAdd(&count[b], 1u)] = first + i | (b >> 3 == 255u ? kEmptyTile : 0u);
    });
}

struct Pull {
    int slice = -1;  // the slice the wave pulls from (-1 before its first pull)
};

__device__ __forceinline__ void slice_of(int64_t n_items, int s, int64_t& base, int64_t& cnt) {
    const int64_t per = n_items / kSlices, rem = n_items % kSlices;
    base = s * per + (s < rem ? s : rem);
    cnt = per + (s < rem ? 1 : 0);
}

__device__ __forceinline__ int64_t next_item(const BlendArgs& a, int64_t prev, bool persistent, int64_t n_items,
                                             Pull& q, bool by_xcd, int sub_log2, bool& empty) {
    empty = false;  // (true: the item's tile has an empty list; false: it may have)
    if (!persistent) {
        if (prev >= 0) return n_items;
        if (!a.tile_order) return by_xcd ? xcd_item((int64_t)blockIdx.x, n_items) : (int64_t)blockIdx.x;
        const uint32_t b = blockIdx.x, run = sub_log2 + (by_xcd ? 0 : 2), rest = (uint32_t)n_items >> (run + 3) << (run + 3);
        uint32_t i = b;  // (past the last whole run of every XCD: as they come)
        if (b < rest) i = ((b >> 3 >> run) * kXcds + (b & 7u)) << run | (b >> 3 & ((1u << run) - 1u));
        const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.tile_order[i >> sub_log2]), t = e & ~kEmptyTile;
        empty = e != t;
        return ((int64_t)t << sub_log2) + (i & ((1u << sub_log2) - 1u));
    }
    const int lane = __lane_id();
    constexpr int kPer = kSlices / kXcds;
    const int xcc = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & (kXcds - 1));  // XCC_ID
    if (q.slice < 0) q.slice = xcc * kPer + (int)((blockIdx.x / kXcds) % kPer);
    for (;;) {
        int64_t base, cnt;
        slice_of(n_items, q.slice, base, cnt);
        uint32_t j = 0;
        if (lane == 0) j = atomicAdd(a.queue + q.slice * kQueueStride, 1u);
        j = (uint32_t)__builtin_amdgcn_readfirstlane((int)j);
        if ((int64_t)j < cnt) return base + j;
        // this slice is drained: the slices with items left, one lane each, this XCD's first
        bool left = false;
        if (lane < kSlices) {
            int64_t b2, c2;
            slice_of(n_items, lane, b2, c2);
            left = (int64_t)__hip_atomic_load(a.queue + lane * kQueueStride, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT) < c2;
        }
        uint64_t m = __ballot(left);
        if (!m) return n_items;
        const int r = xcc * kPer;  // rotate so that this XCD's slices come first
        m = (m >> r) | (r ? m << (kSlices - r) : 0ull);
        m &= (kSlices == 64 ? ~0ull : ((1ull << kSlices) - 1ull));
        q.slice = (__builtin_ctzll(m) + r) % kSlices;
    }
}

// Rank of this lane among the lanes set in mask (lanes below it).
__device__ __forceinline__ int lane_rank(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

struct SubCtx {
    TileCtx c;
    int sx, sy;       // sub-tile origin inside the tile
    int sidx;         // sub-tile index r S + c (the bit of its flag in the tile keys)
};

__device__ __forceinline__ SubCtx sub_ctx(const BlendArgs& a, int64_t t, int s, int tile) {
    constexpr int SUB = 8;
    const int per_row = tile / SUB;
    SubCtx q;
    q.sidx = s;
    q.sx = (s % per_row) * SUB;
    q.sy = (s / per_row) * SUB;
    // the last view whose first tile is not behind t: one load, by as many lanes as there are views
    static_assert(MEGS_MAX_VIEWS <= kWave, "a lane for each view");
    const int lane = __lane_id();
    const int view = __popcll(__ballot(lane < a.nv && a.views[min(lane, a.nv - 1)].tile_off <= t)) - 1;
    q.c = tile_ctx(a, view, t, tile);
    return q;
}

// The tile's list, in scalar registers, so that branches on it are branches of the wave.
__device__ __forceinline__ uint2 range_of(const BlendArgs& a, int64_t t) {
    const uint2 r = a.ranges[t];
    return make_uint2((uint32_t)__builtin_amdgcn_readfirstlane((int)r.x), (uint32_t)__builtin_amdgcn_readfirstlane((int)r.y));
}

// How a sub-tile kernel frames its entries and chooses the ones it keeps; a template argument, so each
// form carries only its own tests.
enum SubMode {
    kSubFlags,   // the tile keys carry sub-tile flags (a.tkeys non-null), which decide; staged relative to
                 // the sub-tile's corner
    kSubReach,   // no flags: `reaches` decides; staged relative to the sub-tile's corner
    kSubInTile,  // no flags: `reaches` decides; staged relative to the tile's corner, the frame of the
                 // per-tile kernels, so that every alpha and every decision is bit for bit theirs (the
                 // default launch of 16 x 16 and 32 x 32 tiles)
};

// May the staged entry reach a pixel centre of the 8 x 8 block whose corner is (bx, by) in its frame? No
// when the cutoff ellipse's box misses the block, or when w1^2 + w2^2 exceeds log2(255 o) over the whole
// block taking each factor's least size over it (exact for an upright ellipse). The limit is widened by
// 0.2% and 0.01, far more than FP32 rounding moves w1 and w2 near it, so no entry with a pixel of alpha
// >= 1/255 is dropped.
__device__ __forceinline__ bool reaches(const Staged& s, int bx, int by) {
    const float cx = bx + 4.0f, cy = by + 4.0f;
    const float w1 = __fmaf_rn(s.p0.x, cx, __fmaf_rn(s.p0.y, cy, s.p0.z)), w2 = __fmaf_rn(s.p1.x, cy, s.p1.y);
    const float m1 = fmaxf(fabsf(w1) - 3.5f * (fabsf(s.p0.x) + fabsf(s.p0.y)), 0.0f);
    const float m2 = fmaxf(fabsf(w2) - 3.5f * fabsf(s.p1.x), 0.0f);
    const float lim = __fmaf_rn(cutoff_of(s.p0.w), 0.5f * kLog2e, 0.01f);
    return box_meets(s.box, bx, bx + 7, by, by + 7) & !(__fmaf_rn(m1, m1, m2 * m2) > lim);
}

// The entries of a sub-tile's list whose flag is set, in list order (DOWN: in reverse order from a given
// position), for the sub-tile kernels when the tile keys carry flags. A 32 x 32 tile's list holds some
// eight entries for each one that reaches a given sub-tile of it, so the wave first runs through the keys
// alone, BLOCKS x 64 at a time, and queues the flagged entries' record ids and positions in LDS; records
// are gathered, staged and blended 64 at a time. (Taking each 64 candidates through all of that, a wave
// spent its time on one gather's latency after the other: forward 0.295 -> 0.249 ms for one 1080p view of 1 M
// Gaussians, 1.07 -> 0.93 ms for sixteen views of 0.5 M; backward 0.335 -> 0.288 ms for one 1080p view of 0.96 M.)
// The next keys are loaded while the queue is worked off.
constexpr int kRing = 256;
template <int BLOCKS, bool DOWN>
struct FlagQueue {
    static_assert(kRing >= 63 + 64 * BLOCKS, "a refill fits behind the 63 entries that ask for it");
    uint32_t key[BLOCKS], id[BLOCKS];  // of the candidates from `cursor` on
    uint32_t first, count;             // list index of candidate 0, and the number of candidates
    uint32_t begin;                    // list index of the tile's range
    uint32_t cursor, head, tail;       // queued: ring positions head .. tail - 1
    uint32_t flag;

    __device__ __forceinline__ uint32_t index(uint32_t j) const { return DOWN ? first - j : first + j; }
    __device__ __forceinline__ void load(const BlendArgs& a) {
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b) {
            const uint32_t j = cursor + 64u * b + __lane_id();
            key[b] = 0u;
            if (j < count) {
                key[b] = a.tkeys[index(j)];
                id[b] = a.vals[index(j)];
            }
        }
    }
    __device__ __forceinline__ void start(const BlendArgs& a, uint32_t range, uint32_t at, uint32_t n, int sidx) {
        begin = range; first = at; count = n;
        cursor = head = tail = 0;
        flag = 1u << (16 + sidx);
        load(a);
    }
    // queues entries until there are 64 or the list ends
    __device__ __forceinline__ void fill(const BlendArgs& a, uint2* ring) {
        while (tail - head < 64u && cursor < count) {
#pragma unroll
            for (int b = 0; b < BLOCKS; ++b) {
                const bool hit = key[b] & flag;
                const uint64_t m = __ballot(hit);
                if (hit) {
                    const uint32_t j = cursor + 64u * b + __lane_id();
                    ring[(tail + (uint32_t)lane_rank(m)) % kRing] = make_uint2(id[b], index(j) - begin + 1u);
                }
                tail += (uint32_t)__popcll(m);
            }
            cursor += 64u * BLOCKS;
            load(a);
        }
        wave_sync();
    }
    // takes up to 64 entries: their number, and this lane's (record id, one past the list position)
    __device__ __forceinline__ int take(const uint2* ring, uint2& entry) {
        const int n = (int)min(tail - head, 64u);
        entry = ring[(head + __lane_id()) % kRing];
        head += (uint32_t)n;
        return n;
    }
};

constexpr int kRow = 16;  // lanes of a DPP row

// Lane L of each row of sixteen lanes, as an operand of the instruction that uses it (all lanes active).
template <int L>
__device__ __forceinline__ float bcast16(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + L, 0xf, 0xf, true));  // row_newbcast
}

// acc += (lane L of v's row of sixteen) * x, in one instruction (the compiler folds the broadcast into a
// product but not into a multiply-add). A register must be written two wait states before a row broadcast
// reads it; the compiler does not look into the statement, so it waits by itself.
template <int L>
__device__ __forceinline__ void fmac_bcast16(float& acc, float v, float x) {
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "+v"(acc)
        : "v"(v), "v"(x), "n"(L));
}
template <int L>
__device__ __forceinline__ void fmac3_bcast16(float& a0, float& a1, float& a2, float v0, float v1, float v2, float x) {
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %3, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %1, %4, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f32_dpp %2, %5, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "+v"(a0), "+v"(a1), "+v"(a2)
        : "v"(v0), "v"(v1), "v"(v2), "v"(x), "n"(L));
}

template <typename F, int... I>
__device__ __forceinline__ void for_each_of_row(F& f, std::integer_sequence<int, I...>) {
    (void)(f(std::integral_constant<int, I>{}) && ...);
}

// &p[k] through a VGPR copy of its byte offset (see kept_at).
__device__ __forceinline__ const float4* uniform_at(const float4* p, int k) {
    uint32_t off;
    asm("v_mov_b32 %0, %1" : "=v"(off) : "s"(k * (int)sizeof(float4)));
    return reinterpret_cast<const float4*>(reinterpret_cast<const char*>(p) + off);
}

// The kept entries of a chunk, as the forward sub-tile blend reads them back: every entry's 40 bytes taken
// by every lane is 20 cycles of the CU's LDS for 18 VALU instructions, so a lane reads only what enters two
// multiply-adds with an addend of the entry (four entries ahead); the other factors it reads once per
// sixteen entries, for the entry of its place in a row of sixteen lanes, and the instructions that use them
// take them from there by row broadcast. The transmittance of a stopped pixel needs no mark and no test (the
// lane mask `alive` is in scalar registers). With the list queue: sixteen
// views of 0.5 M Gaussians 0.96 -> 0.83 ms, one 1080p view of 1 M 0.217 -> 0.182 ms, one 979 x 546 view of 0.3 M
// 0.355 -> 0.292 ms. Seven waves per SIMD (72 registers); at eight, five spilled registers cost as much.
template <bool IMP>
struct KeptRow {
    float4 each[64];       // ay, c1, by, c2 of Staged
    float4 lane_vals[64];  // ax, o, r, g
    float blue[64];
    uint32_t pos1[64];     // one past the entry's list position
    uint32_t id[IMP ? 64 : 1];
};

template <bool STATS, bool IMP, SubMode MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MODE == kSubFlags ? 7 : 6))) void k_blend_fwd_sub(BlendArgs a, int tile, int persistent) {
    constexpr bool FLAGS = MODE == kSubFlags;
    __shared__ KeptRow<IMP> lds;
    __shared__ uint2 ring[FLAGS ? kRing : 1];
    const int lane = __lane_id();
    const int sub_log2 = tile == 32 ? 4 : 2;  // (sub-tiles of a 32 x 32 or a 16 x 16 tile)
    const int64_t n_items = a.n_tiles << sub_log2;
    uint64_t n_blended = 0, n_evaluated = 0;  // of the wave
    const int n_sub = 1 << sub_log2;
    Pull pull;
    bool empty;
    for (int64_t w = next_item(a, -1, persistent, n_items, pull, true, sub_log2, empty); w < n_items;
         w = next_item(a, w, persistent, n_items, pull, true, sub_log2, empty)) {
        const int64_t t = w >> sub_log2;
        int sub = (int)w & (n_sub - 1);
        // A tile with an empty list is one wave's (in turn one of the tile's, so that the waves with work are spread
        // over the CUs): it writes all of the tile's pixels, and the others end before they look for their view. (Each writing its own 8 x 8 pixels, a forward of a few records on a 16384 x 16384 image
        // in 32 x 32 tiles took 2.6 ms, per tile 1.2 ms.)
        const bool writer = sub == ((int)t & (n_sub - 1));
        if (empty && !writer) continue;
        const uint2 rg = range_of(a, t);
        if (rg.x == rg.y) {
            if (!writer) continue;
            sub = 0;
        }
        const SubCtx q = sub_ctx(a, t, sub, tile);
        const TileCtx& c = q.c;
        const int lx = q.sx + (lane & 7), ly = q.sy + (lane >> 3);
        const bool inside = c.x0 + lx < c.width && c.y0 + ly < c.height;
        // the lanes whose pixel is in the image and has not terminated: a lane mask in scalar registers,
        // so that its updates and tests cost the vector unit nothing
        uint64_t alive = __ballot(inside);
        if (!alive) continue;  // a sub-tile past the image edge has no pixel
        float T = 1.0f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
        uint32_t last = 0;
        // the frame the entries are staged in (the tile or the sub-tile): its corner, the sub-tile's corner
        // in it, and the pixel centre in it
        const int bx = MODE == kSubInTile ? q.sx : 0, by = MODE == kSubInTile ? q.sy : 0;
        const double fx0 = (double)(c.x0 + q.sx - bx), fy0 = (double)(c.y0 + q.sy - by);
        const float px = bx + (lane & 7) + 0.5f, py = by + (lane >> 3) + 0.5f;
        auto keep = [&](int slot, const Staged& st, uint32_t pos1, uint32_t g) {
            lds.each[slot] = make_float4(st.p0.y, st.p0.z, st.p1.x, st.p1.y);
            lds.lane_vals[slot] = make_float4(st.p0.x, st.p0.w, st.p1.z, st.p1.w);
            lds.blue[slot] = st.b;
            lds.pos1[slot] = pos1;
            if (IMP) lds.id[slot] = g;
        };
        auto blend_kept = [&](int nhit) {
            for (int k0 = 0; k0 < nhit; k0 += kRow) {
                // sixteen entries, one per lane of each row of sixteen lanes
                const float4 per_lane = lds.lane_vals[k0 + (lane & (kRow - 1))];
                const float blue = lds.blue[k0 + (lane & (kRow - 1))];
                const float4* const each = uniform_at(lds.each, k0);
                float4 ahead[4];
                int taken = -1;     // the last of the sixteen that the pixel includes
                float sums = 0.0f;  // lane k: the weights of the k-th, summed over the wave (IMP)
                auto blend = [&](auto index) {
                    constexpr int kk = decltype(index)::value;
                    if (k0 + kk >= nhit) return false;  // wave-uniform
                    // the wave stops once all its pixels have terminated; checked every 4 entries
                    if (kk % 4 == 0 && !alive) return false;
                    if constexpr (kk % 4 == 0) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) ahead[i] = each[kk + i];
                    }
                    const float4 s = ahead[kk % 4];
                    float w1 = __fmaf_rn(s.x, py, s.y);
                    fmac_bcast16<kk>(w1, per_lane.x, px);
                    const float w2 = __fmaf_rn(s.z, py, s.w);
                    float G, alpha;
                    bool clamped;
                    const bool over = alpha_of(w1, w2, bcast16<kk>(per_lane.y), G, alpha, clamped);
                    if (STATS) n_evaluated += (uint32_t)__popcll(alive);
                    const uint64_t pass = __ballot(over) & alive;
                    if (!pass) return true;  // wave-uniform
                    const float Tn = T * (1.0f - alpha);
                    const uint64_t incl = pass & ~__ballot(Tn < kTMin);
                    alive &= incl | ~pass;
                    if (STATS) n_blended += (uint32_t)__popcll(incl);
                    const bool in = __builtin_amdgcn_inverse_ballot_w64(incl);
                    const float wgt = in ? alpha * T : 0.0f;
                    fmac3_bcast16<kk>(C0, C1, C2, per_lane.z, per_lane.w, blue, wgt);
                    T = in ? Tn : T;
                    taken = in ? kk : taken;
                    if (IMP) {
                        const int wsum = __builtin_amdgcn_readlane(__float_as_int(wave_sum(wgt)), kWave - 1);
                        asm("s_nop 3\n\tv_writelane_b32 %0, %1, %2" : "+v"(sums) : "s"(wsum), "n"(kk));
                    }
                    return true;
                };
                for_each_of_row(blend, std::make_integer_sequence<int, kRow>{});
                if (taken >= 0) last = lds.pos1[k0 + taken];
                if (IMP && lane < kRow && sums != 0.0f)
                    unsafeAtomicAdd(a.importance + ((int64_t)lds.id[k0 + lane] - (int64_t)c.view * a.n), sums);
                if (!alive) break;
            }
        };
        if (FLAGS) {
            FlagQueue<3, false> queue;
            queue.start(a, rg.x, rg.x, rg.y - rg.x, q.sidx);
            queue.fill(a, ring);
            while (alive) {
                uint2 entry;
                const int n = queue.take(ring, entry);
                if (n == 0) break;
                RecVecs raw;
                if (lane < n) raw = gather(a, entry.x);
                queue.fill(a, ring);
                if (lane < n) keep(lane, staged_of(raw, fx0, fy0, false), entry.y, entry.x);
                wave_sync();
                blend_kept(n);
                wave_sync();
            }
        } else {
            // each chunk's records are gathered while the chunk before it is blended, and its record ids are
            // loaded one chunk before that (six waves per SIMD for the 12 registers; importance of four 720p
            // views 0.289 -> 0.261 ms, one 720p view of 0.2 M Gaussians 0.148 -> 0.142 ms, at seven with spills
            // 0.285 and 0.141 ms). The queued form above gathers for eight times as many candidates at once and
            // does better at seven waves (eight 1080p views 0.88 ms, gathering ahead 0.94 ms).
            uint32_t g = 0, id_n = 0;
            RecVecs raw;
            if (rg.x + lane < rg.y) raw = gather(a, g = a.vals[rg.x + lane]);
            if (rg.x + 64u + lane < rg.y) id_n = a.vals[rg.x + 64u + lane];
            for (uint32_t base = rg.x; base < rg.y && alive; base += 64) {
                const uint32_t idx = base + lane;
                bool hit = false;
                Staged st;
                if (idx < rg.y) {
                    st = staged_of(raw, fx0, fy0, true);
                    // (the fragment statistics count the entries whose box meets the sub-tile as tested)
                    hit = STATS ? box_meets(st.box, bx, bx + 7, by, by + 7) : reaches(st, bx, by);
                }
                const uint64_t m = __ballot(hit);
                if (hit) keep(lane_rank(m), st, idx - rg.x + 1u, g);
                if (idx + 64u < rg.y) raw = gather(a, g = id_n);
                if (idx + 128u < rg.y) id_n = a.vals[idx + 128u];
                wave_sync();
                blend_kept(__popcll(m));
                wave_sync();
            }
        }
        int x = c.x0 + lx, y = c.y0 + ly;
        for (int s = sub;;) {  // (of an empty list: every sub-tile of the tile)
            if (x < c.width && y < c.height) {
                const int64_t p = (int64_t)y * c.width + x;
                const int64_t plane = (int64_t)c.width * c.height;
                float* img = a.image + 3 * c.pix_off;
                img[p] = __fmaf_rn(T, c.bg[0], C0);
                img[plane + p] = __fmaf_rn(T, c.bg[1], C1);
                img[2 * plane + p] = __fmaf_rn(T, c.bg[2], C2);
                a.T_final[c.pix_off + p] = T;
                a.last[c.pix_off + p] = last;
            }
            if (rg.x != rg.y || ++s == n_sub) break;
            const bool row_end = (s & ((tile >> 3) - 1)) == 0;
            x += row_end ? 8 - tile : 8;
            y += row_end ? 8 : 0;
        }
    }
    if (STATS) {
        if (lane == 0) {
            atomicAdd(a.stats, (unsigned long long)n_blended);
            atomicAdd(a.stats + 1, (unsigned long long)n_evaluated);
        }
    }
}

// The sub-tile backward. Reducing an entry's nine sums over the wave as soon as it is replayed takes a
// butterfly per entry (24 VALU instructions, beside the eight products that form the summands: together
// more than half of the kernel). Instead the replay, one pixel per lane, leaves only the two scalars that
// everything is linear in, e and the blending weight, in a row of LDS per entry (one 8-byte store). After
// kGroup entries the wave turns round: lane (entry, pixel row) takes its entry's eight pixels of one row,
// forms the moments in registers (an entry's second factor w2 is constant along a row), and the eight rows'
// partial sums go through LDS to the lane that adds them: lane 9 k + c ends with sum c of entry k, so the
// kGroup records leave through one atomic instruction, nine consecutive lanes per record (kGroup = 7: 63
// lanes). That is about 12 VALU instructions an entry. Where it replaced the butterfly, eight 1080p views of 1 M
// Gaussians went from 1,369 M VALU instructions per launch and 2.42 ms to 937 M and 2.17 ms, one 1080p view of 0.96 M from
// 0.42 to 0.35 ms. With the list queue and the tile order the launch has 835 M and takes 1.62 ms: VALU issue is 84% of
// it, the rest is the float atomics' completion and latency at four waves per SIMD. (The same sums
// as FP32 matrix products, the entries as rows and 1, x, y, x^2, x y, y^2 and the colour gradients as columns,
// took 2.30 ms where this took 1.93: seven entries keep the matrix pipe busy for 512 cycles.) The kernel is
// compiled for four: at five (96 registers) it spills, and since memory operations complete in order, each
// reload from scratch memory waits for the atomics before it (2.69 ms).
constexpr int kGroup = 7;

template <SubMode MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_blend_bwd_sub(BlendArgs a, int tile,
                                                                                              int persistent) {
    constexpr bool FLAGS = MODE == kSubFlags;
    // the kept entries of a chunk behind up to kGroup - 1 carried over from the chunk before
    __shared__ Kept lds[64 + kGroup - 1];
    // rows[entry][pixel row][pixel]: a row's 64 bytes are four 16-byte pieces, stored in an order that
    // depends on the row and the entry, so that the 16 lanes of a 16-byte read (two entries' eight rows)
    // touch every LDS bank once
    __shared__ __align__(16) float2 rows[kGroup * 64];
    __shared__ uint2 ring[FLAGS ? kRing : 1];
    __shared__ __align__(16) float dlr[3][64];  // the pixels' colour gradients
    const int lane = __lane_id();
    // as replaying lane: pixel (lane & 7, lane >> 3); as summing lane: entry lane >> 3, pixel row lane & 7
    const int sum_entry = min(lane >> 3, kGroup - 1), sum_row = lane & 7;
    const int turn = (sum_row >> 2) | ((lane >> 3 & 1) << 1);  // piece h of the summing lane's row is h ^ turn
    // the replaying lane's place in an even entry's row; an odd entry's is the same with piece bit 1 flipped
    const int piece = ((lane & 7) >> 1) ^ (lane >> 5);
    float2* const put0 = rows + (lane >> 3) * 8 + piece * 2 + (lane & 1);
    float2* const put1 = rows + (lane >> 3) * 8 + (piece ^ 2) * 2 + (lane & 1);
    const float4* const get = reinterpret_cast<const float4*>(rows + sum_entry * 64 + sum_row * 8);
    float* const sums = reinterpret_cast<float*>(rows);  // [kGroup * 9][8] by row, once the rows are read
    // as adding lane: sum lane % 9 of entry lane / 9 (lane 63 adds nothing)
    const int add_entry = min(lane / 9, kGroup - 1), add_comp = lane % 9;
    const float4* const fin = reinterpret_cast<const float4*>(sums + min(lane, 9 * kGroup - 1) * 8);
    const int sub_log2 = tile == 32 ? 4 : 2;
    const int64_t n_items = a.n_tiles << sub_log2;
    Pull pull;
    bool empty;
    for (int64_t w = next_item(a, -1, persistent, n_items, pull, false, sub_log2, empty); w < n_items;
         w = next_item(a, w, persistent, n_items, pull, false, sub_log2, empty)) {
        if (empty) continue;
        const int64_t t = w >> sub_log2;
        const uint2 rg = range_of(a, t);
        if (rg.x == rg.y) continue;  // (before any pixel is read)
        const SubCtx q = sub_ctx(a, t, (int)(w & ((1 << sub_log2) - 1)), tile);
        const TileCtx& c = q.c;
        const int lx = q.sx + (lane & 7), ly = q.sy + (lane >> 3);
        const int x = c.x0 + lx, y = c.y0 + ly;
        const bool inside = x < c.width && y < c.height;
        const int64_t plane = (int64_t)c.width * c.height;
        const int64_t p = (int64_t)y * c.width + x;
        float T = 1.0f, dl0 = 0.f, dl1 = 0.f, dl2 = 0.f;
        uint32_t lst = 0;
        if (inside) {
            const float* dimg = a.dl + 3 * c.pix_off;
            T = a.T_final[c.pix_off + p];
            lst = a.last[c.pix_off + p];
            dl0 = dimg[p];
            dl1 = dimg[plane + p];
            dl2 = dimg[2 * plane + p];
        }
        // the colour accumulated behind the current fragment (background included) enters the
        // gradient only through its dot product with the pixel's colour gradient, so the replay
        // carries that one scalar: P = S . dL/dC, updated as S is (S += alpha (c - S))
        float P = __fmaf_rn(c.bg[0], dl0, __fmaf_rn(c.bg[1], dl1, c.bg[2] * dl2));
        uint32_t wave_last = lst;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) wave_last = max(wave_last, (uint32_t)__shfl_xor((int)wave_last, d));
        wave_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_last);  // into a scalar register
        if (wave_last == 0) continue;  // wave-uniform: no pixel of the sub-tile blended anything
        wave_sync();
        dlr[0][lane] = dl0;
        dlr[1][lane] = dl1;
        dlr[2][lane] = dl2;
        // the frame, as in the forward; the summing lane's pixel row in it
        const int bx = MODE == kSubInTile ? q.sx : 0, by = MODE == kSubInTile ? q.sy : 0;
        const double fx0 = (double)(c.x0 + q.sx - bx), fy0 = (double)(c.y0 + q.sy - by);
        const float px = bx + (lane & 7) + 0.5f, py = by + (lane >> 3) + 0.5f;
        const float row_y = by + sum_row + 0.5f;
        // The list is walked in chunks of 64 (of its flagged entries, FlagQueue) from position wave_last - 1
        // downwards, pipelined: a chunk's record ids are loaded two chunks ahead, and its records are
        // gathered while the chunk before it is replayed, and taken over before that chunk's first atomics
        // leave (memory operations complete in order, so a load waited for behind them would wait for them
        // too).
        uint32_t cur = wave_last;  // without flags: positions not yet taken, from 0 up
        uint32_t id_n = 0, g = 0, pos1 = 0;
        bool flagged = false, hit = false;
        RecVecs raw;
        Staged st;
        FlagQueue<2, true> queue;
        // the next entries' records: true when there are any
        auto issue = [&]() {
            uint32_t n;
            if constexpr (FLAGS) {
                queue.fill(a, ring);
                uint2 entry;
                n = (uint32_t)queue.take(ring, entry);
                g = entry.x;
                pos1 = entry.y;
            } else {
                n = min(cur, 64u);
                g = id_n;
                pos1 = cur - (uint32_t)lane;
                cur -= n;
                if ((uint32_t)lane < cur) id_n = a.vals[rg.x + cur - 1u - (uint32_t)lane];
            }
            flagged = (uint32_t)lane < n;
            if (flagged) raw = gather(a, g);
            return n != 0;
        };
        auto take = [&]() {
            hit = false;
            if (flagged) {
                st = staged_of(raw, fx0, fy0, !FLAGS);
                hit = FLAGS || reaches(st, bx, by);  // the flags already tested the ellipse
            }
        };
        if constexpr (FLAGS)
            queue.start(a, rg.x, rg.x + wave_last - 1u, wave_last, q.sidx);
        else if ((uint32_t)lane < cur)
            id_n = a.vals[rg.x + cur - 1u - (uint32_t)lane];
        issue();
        take();
        int carried = 0;
        for (;;) {
            const uint64_t m = __ballot(hit);
            const int n = carried + __popcll(m);
            if (hit) {
                const int slot = carried + lane_rank(m);
                lds[slot] = Kept{st.p0, st.p1, st.b, pos1, (uint64_t)grad2d_index(g, 0)};
            }
            const bool last = !issue();
            wave_sync();
            // whole groups; what is left waits for the next chunk, and after the last chunk it is a group too
            const int todo = last ? n : n - n % kGroup;
            for (int k0 = 0; k0 < todo; k0 += kGroup) {
                const Kept* kp = kept_at(lds, k0);
                uint32_t included = 0;  // entries that some pixel includes
                Kept ahead = kp[0];
#pragma unroll
                for (int kk = 0; kk < kGroup; ++kk) {
                    if (k0 + kk >= todo) break;  // wave-uniform: the last group's end
                    const Kept s = ahead;        // (each entry is read from LDS one entry ahead)
                    if (kk + 1 < kGroup) ahead = kp[kk + 1];
                    float alpha, G, w1, w2;
                    bool clamped;
                    const bool incl = frag(s, px, py, w1, w2, G, alpha, clamped) & (s.pos1 <= lst);
                    if (!__any(incl)) continue;
                    included |= 1u << kk;
                    // a lane the entry does not include takes alpha = 0: its T is then multiplied by the
                    // reciprocal of 1.0, which is exactly 1.0, and its P by nothing, so it needs no select
                    const float al = incl ? alpha : 0.0f;
                    const float Ti = T * __builtin_amdgcn_rcpf(1.0f - al);
                    // (c - S) . dL/dC, from c . dL/dC and the carried P
                    const float dcs = __fmaf_rn(s.p1.z, dl0, __fmaf_rn(s.p1.w, dl1, __fmaf_rn(s.b, dl2, -P)));
                    const float dal = Ti * dcs;
                    P = __fmaf_rn(al, dcs, P);
                    T = Ti;
                    const bool live = incl & !clamped;
                    // dL/do_eff (the exponent gradient is o_eff times this) and the blending weight
                    (kk & 1 ? put1 : put0)[kk * 64] = make_float2(live ? G * dal : 0.0f, al * Ti);
                }
                if (k0 == 0) take();
                if (!included) continue;  // wave-uniform
                wave_sync();
                float acc[9];
                {
                    int tn = turn;  // (formed again for each group: the addresses would hold four registers)
                    asm volatile("" : "+v"(tn));
                    // rows of entries past the group's end or that no pixel includes hold older values:
                    // they are summed like the others and not added
                    const Kept& s = lds[min(k0 + sum_entry, todo - 1)];
                    const float ax = s.p0.x;
                    float wr = __fmaf_rn(s.p0.y, row_y, s.p0.z);
                    if (MODE == kSubInTile) wr = __fmaf_rn(ax, (float)bx, wr);
                    const float w2 = __fmaf_rn(s.p1.x, row_y, s.p1.y);
                    float r0 = 0.f, r1 = 0.f;
                    acc[2] = 0.f; acc[6] = 0.f; acc[7] = 0.f; acc[8] = 0.f;
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        if (h == 2) __builtin_amdgcn_sched_barrier(0);
                        const float4 v = get[h ^ tn];  // e, weight of pixels 2 h and 2 h + 1
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int j = 2 * h + u;
                            const float e = u ? v.z : v.x, wg = u ? v.w : v.y;
                            const float w1 = __fmaf_rn(ax, j + 0.5f, wr);
                            const float m1 = e * w1;
                            r0 += e;
                            r1 += m1;
                            acc[2] = __fmaf_rn(m1, w1, acc[2]);
                            acc[6] = __fmaf_rn(wg, dlr[0][sum_row * 8 + j], acc[6]);
                            acc[7] = __fmaf_rn(wg, dlr[1][sum_row * 8 + j], acc[7]);
                            acc[8] = __fmaf_rn(wg, dlr[2][sum_row * 8 + j], acc[8]);
                        }
                    }
                    acc[0] = r1;
                    acc[1] = r0 * w2;
                    acc[3] = r1 * w2;
                    acc[4] = acc[1] * w2;
                    acc[5] = r0;
                }
                wave_sync();
                if (lane < 8 * kGroup) {
                    float* o = sums + sum_entry * 72 + sum_row;
#pragma unroll
                    for (int i = 0; i < 9; ++i) o[8 * i] = acc[i];
                }
                wave_sync();
                const float4 f0 = fin[(lane >> 3) & 1], f1 = fin[((lane >> 3) & 1) ^ 1];
                const float val = ((f0.x + f0.y) + (f0.z + f0.w)) + ((f1.x + f1.y) + (f1.z + f1.w));
                if (lane < 9 * kGroup && ((included >> add_entry) & 1u))
                    unsafeAtomicAdd(a.grad2d + (lds[k0 + add_entry].slot + add_comp), val);
                wave_sync();
            }
            if (todo == 0) take();
            if (last) break;
            // carry the rest to the front (at most kGroup - 1 entries, and only past whole groups)
            carried = n - todo;
            if (todo && lane < 3 * carried) {
                const float4 v = reinterpret_cast<const float4*>(lds + todo)[lane];
                reinterpret_cast<float4*>(lds)[lane] = v;
            }
            wave_sync();
        }
    }
}

constexpr int64_t kPersistentGroups = 256 * 24;  // resident workgroups pulling tiles in persistent mode

template <int TILE, int WAVES>
hipError_t launch_fwd_t(const BlendArgs& a, int batch, bool persistent, hipStream_t stream) {
    const size_t lds = (size_t)batch * (sizeof(Staged) + (a.importance ? sizeof(uint32_t) : 0));
    const int64_t groups = persistent ? kPersistentGroups / WAVES : a.n_tiles;
    const unsigned grid = (unsigned)(groups < a.n_tiles ? groups : a.n_tiles);
    const dim3 block(64 * WAVES);
    if (a.importance)
        hipLaunchKernelGGL((k_blend_fwd<TILE, WAVES, false, true>), dim3(grid), block, lds, stream, a, batch,
                           (int)persistent);
    else if (a.stats)
        hipLaunchKernelGGL((k_blend_fwd<TILE, WAVES, true, false>), dim3(grid), block, lds, stream, a, batch,
                           (int)persistent);
    else
        hipLaunchKernelGGL((k_blend_fwd<TILE, WAVES, false, false>), dim3(grid), block, lds, stream, a, batch,
                           (int)persistent);
    return hipGetLastError();
}

template <int TILE, int WAVES>
hipError_t launch_bwd_t(const BlendArgs& a, int batch, bool persistent, hipStream_t stream) {
    size_t lds = (size_t)batch * (sizeof(Staged) + sizeof(uint32_t));
    if (WAVES > 1) lds += (size_t)batch * WAVES * 9 * sizeof(float);
    const int64_t groups = persistent ? kPersistentGroups / WAVES : a.n_tiles;
    const unsigned grid = (unsigned)(groups < a.n_tiles ? groups : a.n_tiles);
    if (a.grad_pair)
        hipLaunchKernelGGL((k_blend_bwd<TILE, WAVES, true>), dim3(grid), dim3(64 * WAVES), lds, stream, a, batch,
                           (int)persistent);
    else
        hipLaunchKernelGGL((k_blend_bwd<TILE, WAVES, false>), dim3(grid), dim3(64 * WAVES), lds, stream, a, batch,
                           (int)persistent);
    return hipGetLastError();
}

template <bool STATS, bool IMP>
hipError_t launch_fwd_sub_t(const BlendArgs& a, unsigned grid, int tile, SubMode mode, bool persistent, hipStream_t stream) {
    if (mode == kSubFlags)
        hipLaunchKernelGGL((k_blend_fwd_sub<STATS, IMP, kSubFlags>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    else if (mode == kSubReach)
        hipLaunchKernelGGL((k_blend_fwd_sub<STATS, IMP, kSubReach>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    else if constexpr (!STATS)
        hipLaunchKernelGGL((k_blend_fwd_sub<false, IMP, kSubInTile>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    else
        return hipErrorInvalidValue;  // (the statistics count the per-tile kernels' fragments there: sub_in_tile)
    return hipGetLastError();
}

// The arguments with the tile order made, or without it. It is made from kOrderItemsFwd (forward) or
// kOrderItemsBwd (backward) sub-tiles on (orders_tiles_fwd, orders_tiles_bwd). Measured without and with it, its launch included:
// at those sizes it gains about what its launch takes when lists are short (20,000 Gaussians over the image,
// 640 x 480: forward 29 and 30 us, backward 38 and 41 us; 1024 x 768: 39 and 33 us, 69 and 64 us; gathered in
// clusters, 960 x 640: 46 and 50 us, 71 and 69 us; 1280 x 1024: 49 and 44 us, 78 and 69 us). Long lists gain
// below the limits too where they are even (1 M over 979 x 546: 95 and 76 us, 124 and 108 us) and forward lose a
// little where they are clustered (445 and 449 us, 634 and 593 us). One 1080p view of 1 M 115 and 83 us, 165 and
// 157 us, clustered 208 and 202 us, 392 and 335 us.
// Upwards: with 16 x 16 tiles a forward of more than kOrderTilesFwd16 tiles mostly loses (8 x 1080p, 65,280 tiles: 1 M 575 and 616 us,
// clustered 777 and 770 us, 0.2 M 376 and 437 us; 8 x 4K: 1.30 and 1.47 ms), with 32 x 32 tiles it gains or is even
// (8 x 1080p 537 and 544 us, 740 and 672 us; 8 x 4K 1.23 and 1.23 ms, 1.47 and 1.42 ms; 16384 x 16384 7.3 and 6.2 ms). A
// backward of more than kOrderTilesBwd tiles loses (65,536 tiles: 8 x 1080p 1653 and 1518 us, 1190 and 1209 us, 8 x 4K
// 3.05 and 2.94 ms; 262,144 tiles of a 16384 x 16384 image 17.9 and 19.3 ms).
BlendArgs with_order(const BlendArgs& a, bool use, hipStream_t stream) {
    BlendArgs r = a;
    if (!use) r.tile_order = nullptr;
    if (r.tile_order) {
        const uint32_t n = (uint32_t)a.n_tiles, slices = (n + kOrderSlice - 1) / kOrderSlice;
        const uint32_t slice = (n + slices - 1) / slices;  // (no slice is empty: n > slice * (slices - 1))
        hipLaunchKernelGGL(k_tile_order, dim3(slices), dim3(kOrderThreads), 0, stream, a.ranges, n, slice, a.tile_order);
    }
    return r;
}

hipError_t launch_fwd_sub(const BlendArgs& args, int tile, SubMode mode, bool persistent, hipStream_t stream) {
    const int64_t items = args.n_tiles * (int64_t)(tile / 8) * (tile / 8);
    const BlendArgs a = with_order(args, !persistent && orders_tiles_fwd(tile, args.n_tiles, args.pairs), stream);
    const int64_t groups = persistent ? kPersistentGroups : items;
    const unsigned grid = (unsigned)(groups < items ? groups : items);
    if (a.importance) return launch_fwd_sub_t<false, true>(a, grid, tile, mode, persistent, stream);
    if (a.stats) return launch_fwd_sub_t<true, false>(a, grid, tile, mode, persistent, stream);
    return launch_fwd_sub_t<false, false>(a, grid, tile, mode, persistent, stream);
}

hipError_t launch_bwd_sub(const BlendArgs& args, int tile, SubMode mode, bool persistent, hipStream_t stream) {
    const int64_t items = args.n_tiles * (int64_t)(tile / 8) * (tile / 8);
    const BlendArgs a = with_order(args, !persistent && orders_tiles_bwd(tile, args.n_tiles), stream);
    const int64_t groups = persistent ? kPersistentGroups : items;
    const unsigned grid = (unsigned)(groups < items ? groups : items);
    if (mode == kSubFlags)
        hipLaunchKernelGGL((k_blend_bwd_sub<kSubFlags>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    else if (mode == kSubReach)
        hipLaunchKernelGGL((k_blend_bwd_sub<kSubReach>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    else
        hipLaunchKernelGGL((k_blend_bwd_sub<kSubInTile>), dim3(grid), dim3(64), 0, stream, a, tile, (int)persistent);
    return hipGetLastError();
}

// 16 x 16 and 32 x 32 tiles launched with waves = 0 (the library's choice) blend per sub-tile, in the
// tile's frame, so that their results are those of the per-tile kernels (the forward's bit for bit): a wave
// then walks only the entries that reach its 8 x 8 pixels, and no wave waits for another. The per-tile
// kernels serve the wave counts a caller names, 8 x 8 tiles, the fragment statistics (they count tested
// fragments), the deterministic backward (one slot of sums per tile and entry), and the sizes at which they
// are faster (blends_by_sub_tile).
bool sub_in_tile(const BlendArgs& a, BlendKind kind, int tile, int waves) {
    return waves == 0 && tile > 8 && !a.stats && !a.grad_pair &&
           blends_by_sub_tile(kind, tile, a.n_tiles, a.records, a.pairs);
}

int waves_or_default(int waves, int tile) { return waves ? waves : (tile == 8 ? 1 : 4); }

}  // namespace

hipError_t launch_blend_fwd(const BlendArgs& a, int tile, int waves, int batch, bool persistent, hipStream_t stream,
                            int subtile) {
    if (a.n_tiles <= 0) return hipSuccess;
    if (subtile == 8 && tile > 8)
        return launch_fwd_sub(a, tile, a.tkeys ? kSubFlags : kSubReach, persistent, stream);
    if (sub_in_tile(a, a.importance ? kBlendImportance : kBlendForward, tile, waves))
        return launch_fwd_sub(a, tile, kSubInTile, persistent, stream);
    waves = waves_or_default(waves, tile);
    if (tile == 8 && waves == 1) return launch_fwd_t<8, 1>(a, batch, persistent, stream);
    if (tile == 16 && waves == 1) return launch_fwd_t<16, 1>(a, batch, persistent, stream);
    if (tile == 16 && waves == 2) return launch_fwd_t<16, 2>(a, batch, persistent, stream);
    if (tile == 16 && waves == 4) return launch_fwd_t<16, 4>(a, batch, persistent, stream);
    if (tile == 32 && waves == 1) return launch_fwd_t<32, 1>(a, batch, persistent, stream);
    if (tile == 32 && waves == 2) return launch_fwd_t<32, 2>(a, batch, persistent, stream);
    if (tile == 32 && waves == 4) return launch_fwd_t<32, 4>(a, batch, persistent, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_blend_bwd(const BlendArgs& a, int tile, int waves, int batch, bool persistent, hipStream_t stream,
                            int subtile) {
    if (a.n_tiles <= 0) return hipSuccess;
    if (subtile == 8 && tile > 8 && !a.grad_pair)
        return launch_bwd_sub(a, tile, a.tkeys ? kSubFlags : kSubReach, persistent, stream);
    if (sub_in_tile(a, kBlendBackward, tile, waves)) return launch_bwd_sub(a, tile, kSubInTile, persistent, stream);
    waves = waves_or_default(waves, tile);
    if (tile == 8 && waves == 1) return launch_bwd_t<8, 1>(a, batch, persistent, stream);
    if (tile == 16 && waves == 1) return launch_bwd_t<16, 1>(a, batch, persistent, stream);
    if (tile == 16 && waves == 2) return launch_bwd_t<16, 2>(a, batch, persistent, stream);
    if (tile == 16 && waves == 4) return launch_bwd_t<16, 4>(a, batch, persistent, stream);
    if (tile == 32 && waves == 1) return launch_bwd_t<32, 1>(a, batch, persistent, stream);
    if (tile == 32 && waves == 2) return launch_bwd_t<32, 2>(a, batch, persistent, stream);
    if (tile == 32 && waves == 4) return launch_bwd_t<32, 4>(a, batch, persistent, stream);
    return hipErrorInvalidValue;
}

}  // namespace megs
