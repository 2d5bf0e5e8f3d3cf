// Internal declarations shared by the HIP translation units of libfastgs_hip (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastgs.h"
#include "small_words.hpp"

namespace fs {

constexpr int TILE = 16;           // pixels per tile edge (the binning unit of the ABI)
constexpr int TILE_PIX = TILE * TILE;

// Camera and conventions as passed by value to kernels.
struct CamDev {
    int width, height;
    float fx, fy, cx, cy;
    float R[9];
    float t[3];
    int tiles_x, tiles_y;
};

struct CfgDev {
    float z_near, lowpass, alpha_min, alpha_max, T_min;
    float bg[3];
    float jclamp;
    int score_mode;
    int compact_box;  // pairs from the ellipse-tile test instead of the 3-sigma square
    float cb_beta;
};

// ---- Compact Box (FastGS Sec. 4.4 and its supplement) ------------------------------------------
// Support of a Gaussian: (p - mu_2D)^T Sigma_2D^-1 (p - mu_2D) <= Q, Q = beta * 2 ln(sigma / tau_alpha)
// with tau_alpha = alpha_min.  These three functions decide integers (pair counts, which keys exist),
// so their fp32 operation order is fixed: plain IEEE operations as written, fused multiply-adds only
// where spelled out.

// ln(x) for x > 0: x = m 2^e, m in [sqrt(1/2), sqrt(2)); s = (m-1)/(m+1); z = s^2;
// ln m = 2 s (1 + z/3 + z^2/5 + z^3/7 + z^4/9) by Horner with fmaf; ln x = fmaf(e, ln 2, ln m).
__device__ __forceinline__ float log_c(float x)
{
    int e;
    float m = frexpf(x, &e);
    if (m < 0x1.6a09e6p-1f) { m = m + m; e = e - 1; }
    const float s = (m - 1.0f) / (m + 1.0f);
    const float z = s * s;
    float p = 0x1.c71c72p-4f;
    p = __builtin_fmaf(p, z, 0x1.24924ap-3f);
    p = __builtin_fmaf(p, z, 0x1.99999ap-3f);
    p = __builtin_fmaf(p, z, 0x1.555556p-2f);
    p = __builtin_fmaf(p, z, 1.0f);
    const float lnm = (s + s) * p;
    return __builtin_fmaf((float)e, 0x1.62e43p-1f, lnm);
}

// Q of a Gaussian of opacity sigma; 0 when it can never reach alpha_min.
__device__ __forceinline__ float cb_threshold(float sigma, const CfgDev& cfg)
{
    const float ratio = sigma / cfg.alpha_min;
    if (!(ratio > 1.0f)) return 0.0f;
    return cfg.cb_beta * (2.0f * log_c(ratio));
}

// Does the closed rectangle of tile (tx, ty) meet the ellipse?  The quadratic form is convex with its
// minimum at mu_2D: the minimum over the rectangle is 0 when mu_2D is inside, and otherwise lies on the
// vertical and/or horizontal edge that faces mu_2D, where it is a 1-D quadratic with a clamped minimiser.
__device__ __forceinline__ bool cb_tile_hit(float mx, float my, float A, float B, float C, float Q, int tx, int ty)
{
    const float X0 = (float)(tx * TILE), X1 = (float)(tx * TILE + TILE);
    const float Y0 = (float)(ty * TILE), Y1 = (float)(ty * TILE + TILE);
    const float dxl = X0 - mx, dxr = X1 - mx, dyt = Y0 - my, dyb = Y1 - my;
    const bool in_x = dxl <= 0.0f && dxr >= 0.0f;
    const bool in_y = dyt <= 0.0f && dyb >= 0.0f;
    if (in_x && in_y) return true;
    const float B2 = B + B;
    bool have = false;
    float qmin = 0.0f;
    if (!in_x) {
        const float ex = dxl > 0.0f ? dxl : dxr;
        float dys = -(B * ex) / C;
        dys = fminf(fmaxf(dys, dyt), dyb);
        qmin = __builtin_fmaf(ex, __builtin_fmaf(B2, dys, A * ex), (C * dys) * dys);
        have = true;
    }
    if (!in_y) {
        const float ey = dyt > 0.0f ? dyt : dyb;
        float dxs = -(B * ey) / A;
        dxs = fminf(fmaxf(dxs, dxl), dxr);
        const float q = __builtin_fmaf(dxs, __builtin_fmaf(B2, ey, A * dxs), (C * ey) * ey);
        if (!have || q < qmin) qmin = q;
    }
    return qmin <= Q;
}

// ---- the render kernels' bound of a Gaussian's support ----------------------------------------------
// A Gaussian can only be blended where sigma*G >= alpha_min, i.e. where q <= qg = 2 ln(sigma/alpha_min).  With the conic (a, b, c)
// and y = dy, {q <= Q} is |dx + (b/a) dy| <= sqrt(Q/a - (det/a^2) dy^2): an interval of x for every line, whose upper end is concave
// in y and largest at y = Y = -(b/c) sqrt(Q c/det), and whose lower end is least at -Y.  Over the four lines of a row of sub-tiles
// the interval's ends are therefore those at Y and -Y, moved into the row's range of y (strip_mask): a sub-tile is met by the
// ellipse or not, with nothing lost to a bounding polygon.
// Q is taken as 1.004 (qg + 0.1 + e), where e bounds the rounding error of the fp32 q for any pixel of a tile the Gaussian is paired
// with (|dx|,|dy| <= 3 sqrt(lambda_max) + 17), and the ends get 0.01 px (they are computed with the fast reciprocal, square root and
// logarithm; what det loses to cancellation, some 1e-7 times the ratio of the eigenvalues, stays below e / Q, which is 1e-6 times
// that ratio).  Y is drawn in by half a thousandth, a quarter of what Q's factor adds, so that it lies inside the ellipse:
// the upper end there is still above that of {q <= qg + 0.1 + e} anywhere.  Outside, the render kernels' arithmetic yields alpha <
// 0.96 alpha_min, so dropping the pair cannot change any result.
// Returned: {Q/a / 16, det/a^2 / 16, -b/a / 4, Y}, x in units of four pixels; no line is met ({-1, 0, 0, 0}) where the Gaussian is blended nowhere, all are where
// the conic is degenerate or its ellipse longer than 16384 px (the exact test decides).
// (An octagon, the box and two diagonals, took 81 instructions for a Gaussian's 16 sub-tiles where strip_mask takes 95, and let through sub-tiles at
// the corners of slanted ellipses.  A whole pass with it and without, us: 3 M Gaussians at 1920x1080 1577 and 1521, with a tail of
// large splats 2333 and 2040, 500k at 1600x1064 507 and 494, a render of 300k at 1332x876 137 and 133, 100k at 980x545 168 and 165.)
__device__ __forceinline__ float4 support_strips(const float4& co /* a, b, c, sigma */, const CfgDev& cfg)
{
    const float ratio = co.w * __builtin_amdgcn_rcpf(cfg.alpha_min);
    // (a little below 1 for the reciprocal's rounding: an opacity of alpha_min itself is blended at the centre; the 0.1 in Q covers it)
    if (!(ratio >= 0.9999f)) return make_float4(-1.f, 0.f, 0.f, 0.f);
    const float det = co.x * co.z - co.y * co.y;
    const float inv = __builtin_amdgcn_rcpf(det), ra = __builtin_amdgcn_rcpf(co.x);
    const float sxx = co.z * inv, syy = co.x * inv;
    const float D = 3.0f * __builtin_amdgcn_sqrtf(sxx + syy) + 17.0f;
    const float e = 1e-6f * (fabsf(co.x) + 2.0f * fabsf(co.y) + fabsf(co.z)) * D * D;
    const float Q = 1.004f * (2.0f * __logf(ratio) + 0.1f + e);
    const float hx = __builtin_amdgcn_sqrtf(Q * sxx), hy = __builtin_amdgcn_sqrtf(Q * syy);
    const float p = Q * ra, r = det * ra * ra, m = -co.y * ra, Y = -0.9995f * hx * co.y * __builtin_amdgcn_rcpf(co.z);
    // (comparisons that NaNs fail as well)
    const bool plain = det > 0.f && co.x > 0.f && co.z > 0.f && hx < 16384.f && hy < 16384.f && p < 1.0e30f && r < 1.0e30f && fabsf(m) < 1.0e30f && fabsf(Y) < 1.0e30f;
    return plain ? make_float4(0.0625f * p, 0.0625f * r, 0.25f * m, Y) : make_float4(3.0e38f, 0.f, 0.f, 0.f);
}

// The sub-tiles (4 x 4 pixels, bit 4 ky + kx of column kx, line ky) of the tile at whose origin the Gaussian sits at (ox, oy) that
// hold a pixel centre's square met by the ellipse of support_strips.
__device__ __forceinline__ uint32_t strip_mask(const float4& ell, float ox, float oy)
{
    // column j's centres are 4j + 0.5 ... 4j + 3.5: met are those up to the upper end, without those that end before the lower one
    const float x_up = 0.25f * (ox + 3.51f), x_low = 0.25f * (ox + 0.49f);
    uint32_t mask = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const float y0 = (float)(4 * k) + 0.5f - oy, y1 = y0 + 3.0f;   // the strip's first and last line of centres
        const float yh = fminf(fmaxf(ell.w, y0), y1), yl = fminf(fmaxf(-ell.w, y0), y1);
        // (a strip that the ellipse does not reach leaves NaNs here, which the maxima with zero below make an empty interval)
        const float sh = __builtin_amdgcn_sqrtf(__builtin_fmaf(-ell.y * yh, yh, ell.x)), sl = __builtin_amdgcn_sqrtf(__builtin_fmaf(-ell.y * yl, yl, ell.x));
        const uint32_t upto = (uint32_t)fminf(fmaxf(__builtin_fmaf(ell.z, yh, x_up) + sh, 0.f), 4.f);
        const uint32_t before = (uint32_t)fminf(fmaxf(__builtin_fmaf(ell.z, yl, x_low) - sl, 0.f), 4.f);
        mask |= ((15u << before) & ((1u << upto) - 1u)) << (4 * k);
    }
    return mask;
}

// A needle: a splat at least some thirty times as long as wide (the ratio of the eigenvalues of Sigma_2D, which is about
// (a + c)^2 / det, above 1000).  What its scales and rotation receive is the small difference of large second moments, down to
// a millionth of them, so any other order of the additions in k_render_bwd shows in their first digits, an equally accurate
// one too: for needles the order is fixed, pixel by pixel, whatever it is for the others.  (3 M Gaussians, scales from
// N(-5, 1.2): from one equally accurate order to another the gradients move by 1e-4 to 3e-4 of their norm where no needles are told
// apart, by 2e-5 where those from 10 000 on are, by 1e-5 with those from 1000 on.)
constexpr uint32_t NEEDLE = 0x80000000u;   // (in a splat record: a bit of its first gradient record's number, which is below 2^31)
__device__ __forceinline__ bool is_needle(const float4& co /* a, b, c, sigma */)
{
    const float tr = co.x + co.z;
    return !(tr * tr <= 1000.0f * (co.x * co.z - co.y * co.y));
}

// ---- wavefront helpers ----------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

// Inclusive scan across the 64 lanes of a wavefront with data-parallel-primitive moves instead of shuffles through
// LDS: four shifts within the rows of 16 lanes (zeros move in at a row's start), then lane 15 of rows 0 and 2 is
// added to every lane of the row after it, then lane 31 to every lane of rows 2 and 3.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v);   // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);   // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);   // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);   // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}
// The same with max (on unsigned values, for which zero is the neutral element).
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t v)
{
    v = max(v, dpp_or_zero<0x111, 0xF>(v));
    v = max(v, dpp_or_zero<0x112, 0xF>(v));
    v = max(v, dpp_or_zero<0x114, 0xF>(v));
    v = max(v, dpp_or_zero<0x118, 0xF>(v));
    v = max(v, dpp_or_zero<0x142, 0xA>(v));
    v = max(v, dpp_or_zero<0x143, 0xC>(v));
    return v;
}

// Which of a wavefront's 64 runs holds element j0 + lane of their concatenation?  Lane l's run is [excl, excl + cnt).
// Every non-empty run leaves 1 + its lane at the slot of its first element (if that falls into this window of 64; the
// slots are distinct), and a running maximum over the slots spreads it over the rest of the run; the window's first slots
// belong to `carry` (zero before the first window; the windows have to be walked in order).  One trip through LDS (a
// wavefront's LDS operations complete in the order they were issued) instead of the six dependent shuffles of a binary
// search over the prefix sums.  `mark`: 64 words of LDS of this wavefront's own.
__device__ __forceinline__ uint32_t wave_run_owner(uint32_t* mark, uint32_t cnt, uint32_t excl, uint32_t j0, uint32_t& carry)
{
    const uint32_t lane = lane_id();
    mark[lane] = 0u;
    const uint32_t rel = excl - j0;
    if (cnt != 0u && rel < 64u) mark[rel] = lane + 1u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint32_t own = mark[lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    own = wave_inclusive_max(lane == 0u ? max(own, carry) : own);
    carry = (uint32_t)__builtin_amdgcn_readlane((int)own, 63);
    return (own - 1u) & 63u;   // (own >= 1 wherever an element is: element 0 is some run's first)
}

// The same for the elements j0 + lane and j0 + 64 + lane at once: the two trips through LDS overlap.  `mark`: 128 words.
__device__ __forceinline__ void wave_run_owner2(uint32_t* mark, uint32_t cnt, uint32_t excl, uint32_t j0, uint32_t& carry, uint32_t (&owner)[2])
{
    const uint32_t lane = lane_id();
    mark[lane] = 0u;
    mark[64 + lane] = 0u;
    const uint32_t rel = excl - j0;
    if (cnt != 0u && rel < 128u) mark[rel] = lane + 1u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    uint32_t a = mark[lane], b = mark[64 + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    a = wave_inclusive_max(lane == 0u ? max(a, carry) : a);
    carry = (uint32_t)__builtin_amdgcn_readlane((int)a, 63);
    b = wave_inclusive_max(b);
    b = max(b, carry);   // (lanes in front of the window's first mark belong to the run before)
    carry = (uint32_t)__builtin_amdgcn_readlane((int)b, 63);
    owner[0] = (a - 1u) & 63u;
    owner[1] = (b - 1u) & 63u;
}

// k / w for the place of a candidate in a rectangle w wide: estimated with the fast reciprocal, off by at most one
// (k < 2^32 and w < 2^16 make the quotient's error < 0.02): corrected by one step either way, never by a loop that bad
// operands could keep a wavefront in.
__device__ __forceinline__ uint32_t rect_row(uint32_t k, uint32_t w)
{
    uint32_t row = (uint32_t)((float)k * __builtin_amdgcn_rcpf((float)w));
    row -= row * w > k ? 1u : 0u;
    row += (row + 1) * w <= k ? 1u : 0u;
    return row;
}

// ---- optimiser ------------------------------------------------------------------------------------
struct AdamArgs {
    float lr, beta1, beta2, omb1, omb2, eps, grad_scale;
    float inv_bc1, inv_bc2;   // 1 / (1 - beta1^t), 1 / (1 - beta2^t), computed on the host in double
};
AdamArgs adam_args(float lr, float beta1, float beta2, float eps, int step, float grad_scale);

__device__ __forceinline__ void adam_one(float& p, float g, float& m, float& v, const AdamArgs& a, float lr)
{
    g = g * a.grad_scale;
    m = a.beta1 * m + a.omb1 * g;
    v = a.beta2 * v + a.omb2 * (g * g);
    const float mhat = m * a.inv_bc1;
    const float vhat = v * a.inv_bc2;
    p = p - lr * mhat / (sqrtf(vhat) + a.eps);
}

// Used from stored parameters (fs_activate) and the chain rule through it.
__device__ __forceinline__ float4 unit_quat(const float4& r, float& inv)
{
    inv = 1.0f / sqrtf(r.x * r.x + r.y * r.y + r.z * r.z + r.w * r.w);
    return make_float4(r.x * inv, r.y * inv, r.z * inv, r.w * inv);
}
__device__ __forceinline__ float logistic(float raw) { return 1.0f / (1.0f + expf(-raw)); }
__device__ __forceinline__ float4 unit_quat_bwd(const float4& r, const float4& g)
{
    float inv;
    const float4 u = unit_quat(r, inv);
    const float dot = u.x * g.x + u.y * g.y + u.z * g.z + u.w * g.w;
    return make_float4((g.x - u.x * dot) * inv, (g.y - u.y * dot) * inv, (g.z - u.z * dot) * inv, (g.w - u.w * dot) * inv);
}

// ---- workgroup reductions in double precision (fixed tree: results do not depend on scheduling) ----------
constexpr int RED_BLOCKS = 1024;  // partial sums per reduction (a multiple of RED_THREADS)
constexpr int RED_THREADS = 256;

__device__ __forceinline__ double shfl_down_f64(double v, int d)
{
    const long long b = __double_as_longlong(v);
    const int lo = __shfl_down((int)(b & 0xffffffffll), d, 64);
    const int hi = __shfl_down((int)(b >> 32), d, 64);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

enum RedOp { RED_SUM, RED_MIN, RED_MAX };

template <RedOp OP>
__device__ __forceinline__ double red_combine(double a, double b)
{
    if (OP == RED_SUM) return a + b;
    if (OP == RED_MIN) return a < b ? a : b;
    return a > b ? a : b;
}

// Reduces one value per thread over the workgroup; the result is valid in thread 0.
template <RedOp OP>
__device__ __forceinline__ double block_reduce(double v, double* smem /*[4]*/)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = red_combine<OP>(v, shfl_down_f64(v, d));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) v = red_combine<OP>(red_combine<OP>(smem[0], smem[1]), red_combine<OP>(smem[2], smem[3]));
    return v;
}

template <RedOp OP>
__device__ __forceinline__ double red_identity()
{
    if (OP == RED_SUM) return 0.0;
    if (OP == RED_MIN) return 1.0e300;
    return -1.0e300;
}

// ---- launchers (each enqueues on `st` and returns hipGetLastError()) ------------------------
// raw: g's scales, quaternions and opacities are the stored parameters (fs_activate is applied on the way)
hipError_t launch_preprocess(hipStream_t st, int64_t n, int deg, const fs_gaussians& g, bool raw, const CamDev& cam,
                             const CfgDev& cfg, const fs_projected& out);
// pair_grad: records of PAIR_REC floats (see render.hip); Gaussian i owns records
// [rec_offsets[i], rec_offsets[i] + rec_counts[i]); touched as in fs_projected (0 = not visible)
constexpr int PAIR_REC = 12;
hipError_t launch_preprocess_bwd(hipStream_t st, int64_t n, int deg, const fs_gaussians& g, const CamDev& cam,
                                 const CfgDev& cfg, const uint8_t* clamped, const uint32_t* touched,
                                 const uint32_t* rec_counts, const uint32_t* rec_offsets, const float* pair_grad, uint8_t* rec_valid,
                                 const fs_grads& out);

// What a training iteration does with a Gaussian's gradients instead of storing them (g of launch_preprocess_bwd_train
// holds stored parameters then): the five groups are means, sh, raw scales, raw quaternions, raw opacities.
struct TrainDev {
    float* p[5];        // the parameters themselves (the arrays g names), updated in place ...
    float* m[5];        // ... with their moments (UPDATE), or null
    float* v[5];
    float* acc[5];      // gradient sums (SUM), or null
    AdamArgs adam;      // (its lr is not used)
    float lr[5];
    float* grad_accum;  // densification statistics (fs_densify_accumulate)
    float* abs_accum;
    uint32_t* denom;
};
enum BwdOut { BWD_GRADS, BWD_UPDATE, BWD_SUM };
hipError_t launch_preprocess_bwd_train(hipStream_t st, int64_t n, int deg, const fs_gaussians& g, const CamDev& cam,
                                       const CfgDev& cfg, const uint8_t* clamped, const uint32_t* touched,
                                       const uint32_t* rec_counts, const uint32_t* rec_offsets, const float* pair_grad,
                                       uint8_t* rec_valid, BwdOut out, const TrainDev& train);

// exclusive scan of n uint32 values; total (uint64) written to *total_dev. tmp: >= scan_tmp_bytes(n).
size_t scan_tmp_bytes(int64_t n);
hipError_t launch_exclusive_scan(hipStream_t st, const uint32_t* in, uint32_t* out, int64_t n, void* tmp,
                                 uint64_t* total_dev);

// Splat record (SPLAT_REC floats = 64 bytes, one per Gaussian): mx my a b | c sigma r g | b offset(+NEEDLE) rect01 rect23 |
// support_strips (formed here once: the render kernels would form them for every pair)
constexpr int SPLAT_REC = 16;
hipError_t launch_emit_pairs(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, const uint32_t* offsets,
                             int tiles_x, uint64_t* keys, uint32_t* vals, float* splats);
// Compact Box: rec_counts[i] = tiles in Gaussian i's box (the candidates of the ellipse test)
hipError_t launch_rect_area(hipStream_t st, int64_t n, const uint16_t* rect, uint32_t* rec_counts);
// Compact Box emission: one key per candidate tile that meets the ellipse, at offsets[i] + its rank among
// the Gaussian's hits.  (No render workgroup writes the gradient record of a candidate that misses, rec_offsets[i] + its row-major
// place in the box: a dense backward pass clears all records first.)
hipError_t launch_emit_pairs_cb(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg,
                                const uint32_t* offsets, const uint32_t* rec_offsets, int tiles_x, int64_t P,
                                uint64_t* keys, uint32_t* vals, float* splats);

// Tile-bucketed ordering (used when no tile's list is longer than TILE_SORT_HUGE; otherwise the global
// radix sort below): per-tile counts and ranges, then placement into the tiles' segments and an LDS sort
// of every segment.  ranges/tile_order/tile_total: [num_tiles]; tile_count: [TILE_COPIES, num_tiles], turned by
// launch_tile_count into each copy's start within its tile, or, with `bands`, into each copy's start within a band in the place of the
// band's first tile (the `cursor` of launch_tile_scatter).
// launch_tile_count also gives every Gaussian the place of its backward records (rec_offsets [n]: disjoint,
// contiguous per Gaussian, not ordered by index; rec_counts [n], may be null: the area of its rectangle), packs the splat
// records, and, with `counters` (TILE_COUNTERS uint64, the first of which is zero at the start and left zero), writes
// totals [4] = {sum of proj.tiles_touched, records handed out, pairs counted per tile, longest list}.
constexpr int TILE_COPIES = 256;        // workgroups of the counting / placement kernels, each with its own counters (a multiple of 64)
constexpr int TILE_COUNTERS = 1 + 2 * TILE_COPIES;   // the arrivals of k_tile_layout's workgroups; the records and pairs of the counting ones
constexpr int TILE_PAIR_THREADS = 1024;
constexpr int TILE_LDS_MAX_TILES = 15360;  // their per-tile counters live in LDS (60 KB)
constexpr int TILE_SORT_SMALL = 2048;  // longest list one workgroup sorts with 22 KB of LDS (256 threads)
constexpr int TILE_SORT_MID = 4096;    // ... with 40.1 KB (512 threads: three such workgroups fit a compute unit, two of the next)
constexpr int TILE_SORT_MAX = 8192;    // ... with 74 KB (1024 threads)
constexpr int TILE_SORT_HUGE = 16384;  // ... with 146 KB (a compute unit of this chip has 160 KB): the longest list of the
                                       // per-tile ordering; anything longer takes the radix path
hipError_t launch_tile_count(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, int tiles_x,
                             int num_tiles, uint32_t* tile_count, uint32_t* tile_total, uint2* ranges,
                             uint32_t* tile_order, uint64_t* totals, uint32_t* rec_offsets, uint32_t* rec_counts,
                             uint64_t* counters, float* splats, bool bands);
// With many pairs the placement goes in two steps, into bands of BAND_TILES consecutive tiles first (see k_band_split): launch_tile_count is told so, `bucket` of
// launch_tile_scatter is what launch_tile_sorts knows as keys_out, launch_tile_scatter is given `places` and launch_tile_sorts TS_SPLIT.
// The words of the first step hold the tile within the band above the Gaussian's index.
constexpr int BAND_TILES = 64;                 // the tiles of one of k_tile_layout's workgroups
constexpr int BAND_SHIFT = 26;                 // bits of a word that the index has
// The two steps write a word twice for lines that fill: they pay where the tiles' open lines do not fit the L2 and there are enough
// words to bind the kernel.  The host does not know these when it chooses, so it goes by the candidate tiles of the context's ordering
// before, and by the number of Gaussians alone in the first one.  (The order does not depend on the choice.)
// Both launches and the sorts, in one step and in two, us: 1920x1080, 2.5 M pairs 109 and 111 (3 M Gaussians of which a fifth is seen),
// 92.6 and 100 (1.5 M, two fifths), 3.1 M 125 and 122, 105 and 108, 4.2 M 122 and 112, 12.5 M 378 and 295; Compact Box, 2.8 M candidates
// 117 and 123, 3.3 M 138 and 132, 168 and 152, 8.3 M 384 and 321; 1332x876, 2.5 M 80.6 and 81.7, 3.0 M 95.6 and 92.0, Compact Box 2.9 M
// 124 and 118; 640x480, 2.2 M 99.7 and 106, 3.0 M 146 and 131; few seen (0.1 to 1.3 M pairs of 1 to 3 M Gaussians) 54.6 to 87 and 62 to 100.
// Where the Compact Box drops two of five candidates, the tests hide the writes, and two steps are within 2 % of one up to 12 M candidates
// (112 and 113 us at 6 M, 671 and 653 at 18 M).  Fewer Gaussians with more pairs each make runs of one band's words, whose adds in LDS
// wait for one another: 700k 102 and 105 at 2.9 M, wide 300k 131 and 145 at 3.4 M, 400k 159 and 161 at 4.5 M, 700k 222 and 204 at 8.0 M.
constexpr int64_t BAND_MIN_N = 1000000;
constexpr int64_t BAND_MIN_CANDIDATES = 2850000;
// candidates_before: -1 where there was no ordering yet
inline bool placed_by_bands(int64_t n, int num_tiles, int64_t candidates_before)
{
    return n >= BAND_MIN_N && n <= (int64_t)1 << BAND_SHIFT && num_tiles > BAND_TILES &&
           (candidates_before < 0 || candidates_before >= BAND_MIN_CANDIDATES);
}
// Placement and the per-tile sorts.  pair_limit: how many words the buffers hold; the
// kernels write nothing at or beyond it and leave alone a segment that reaches beyond pair_limit, so they may be
// enqueued before the host knows the totals.  places: written by a placement into bands, read by the split (null: no bands).
struct BandPlaces {
    uint32_t* tile;   // [num_tiles] where a tile's next words go (the tiles' totals of launch_tile_count, which are done with by then)
    uint2* band;      // [ceil(num_tiles / BAND_TILES)] first and last + 1 place of its pairs ({~0, 0}: none)
};
hipError_t launch_tile_scatter(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg,
                               int tiles_x, int num_tiles, uint32_t pair_limit, const uint2* ranges, uint32_t* cursor, uint64_t* bucket,
                               const BandPlaces& places);
// The sort launches, by the list lengths they take: (0, SMALL], (SMALL, MID], (MID, MAX], (MAX, HUGE], and
// (SMALL, MAX] in one launch (TS_MIDMAX, instead of TS_MID and TS_MAX).  The lists between SMALL and MID get a launch of
// their own (three of its workgroups fit a compute unit, two of the MAX kind) when the lists are long throughout
// (`long_lists`: there are then enough of them to fill the chip); when only a few tiles are that long, every launch is
// a chain of steps that nothing overlaps with, and one launch fewer is the better deal.
// With MID and without: 3 M Gaussians with lists of 3350 on average 2557 and 2565 us per step, of 1228 1726 and 1730, 30k at
// 189x106 207.2 and 208.0; ten views at 300k, whose lists are 400 long and a few 7000, 2254 and 2167.
// tile_sort_variants: the launches still needed for lists of up to max_len entries when those in `have` are enqueued.
enum { TS_SMALL = 1, TS_MID = 2, TS_MAX = 4, TS_HUGE = 8, TS_MIDMAX = 16, TS_SPLIT = 32 };
int tile_sort_variants(int64_t max_len, bool long_lists, int have);
hipError_t launch_tile_sorts(hipStream_t st, int num_tiles, int variants, uint32_t pair_limit, const uint2* ranges,
                             const uint32_t* tile_order, uint64_t* bucket, uint64_t* keys_out, uint32_t* vals_out,
                             const BandPlaces& places);

// The whole ordering of a small frame in one launch (k_small_frame): what launch_tile_count, launch_tile_scatter and the sort of lists up
// to TILE_SORT_SMALL leave, except that the record places are in index order.  said: [SMALL_WORDS] words, zeroed before the first launch and
// whenever call, a number of 16 bits, starts again from 1.  Once buffers that were too small have grown, a second launch with totals null
// writes the pairs to the ranges that the first one left.  A launch whose workgroups have waited too long for each other ends with totals
// 2 and 3 as they were: nothing that it has written counts then.
constexpr int SMALL_MAX_N = 16384;
constexpr int SMALL_WORDS = SMALL_MAX_TILES + 1;   // the tiles' words and the state
// Every tile looks at every Gaussian, so the launch grows with the product and the four that it replaces do not.  In a training step the
// host has waited for the loss before and the GPU has nothing to do while it launches, so three launches fewer count in full; behind
// a render's or a step's longer queue only the GPU's own time does.  Whole passes, the four launches -> this one, us:
//   fs_train_step, Compact Box:  3k at 256x192 (0.6 M tests) 114 -> 95, 6k at 509x337 (4.2 M) 137 -> 124, 12k at 509x337 (8.7 M) 152 -> 142,
//     16k at 509x337 (11.5 M) 162.5 -> 152.5
//   render, squares and Compact Box:  3k at 256x192 36 -> 30 and 36.5 -> 32, 6k at 400x300 (2.9 M) 38 -> 34 and 41 -> 37, 9k at 400x300
//     (4.3 M) 43 -> 41 and 45 -> 44, 9k at 580x400 (8.3 M) 41 -> 43 and 43.5 -> 47, 16k at 256x192 (3.1 M) 57 -> 58 and 56.5 -> 57.5
//   forward and backward by separate calls:  3k at 256x192 71 -> 66 and 70 -> 67, 9k at 400x300 92 -> 89 and 91 -> 91, 16k at 256x192 131 -> 133
inline bool small_frame(int64_t n, int num_tiles, bool training)
{
    return n > 0 && n <= (training ? SMALL_MAX_N : 10000) && num_tiles <= SMALL_MAX_TILES && n * num_tiles <= (training ? 12000000 : 4000000);
}
hipError_t launch_small_frame(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, int tiles_x, int num_tiles,
                              uint32_t pair_limit, uint32_t* said, uint32_t call, uint2* ranges, uint32_t* tile_order, uint64_t* totals,
                              uint32_t* rec_offsets, uint32_t* rec_counts, float* splats, uint64_t* bucket, uint64_t* keys_out, uint32_t* vals_out);

constexpr int RADIX_BLOCK_KEYS = 2048;  // keys ranked by one workgroup per pass
constexpr int RADIX_BITS = 9;            // widest digit
constexpr int RADIX_DIGITS = 1 << RADIX_BITS;
inline int64_t radix_num_blocks(int64_t P) { return (P + RADIX_BLOCK_KEYS - 1) / RADIX_BLOCK_KEYS; }
// Stable LSD sort of P (key,val) pairs on key bits [0,total_bits). Result ends in *keys_out/*vals_out,
// which point into one of the two ping-pong buffers. hist: RADIX_DIGITS*radix_num_blocks(P) uint32.
hipError_t launch_radix_sort(hipStream_t st, int64_t P, int total_bits, uint64_t* keys[2], uint32_t* vals[2],
                             uint32_t* hist, void* scan_tmp, uint64_t* scan_total_dev, int* result_index);

// ranges [num_tiles,2] and tile_order [num_tiles] (tiles by decreasing list length)
hipError_t launch_tile_ranges(hipStream_t st, int64_t P, const uint64_t* keys_sorted, int num_tiles,
                              uint32_t* ranges, uint32_t* tile_order);

// The threshold of the mask from the error map's statistics (Sec. 4.2, second and third equations): mean + k * std
// with the population variance taken as mean(e^2) - mean(e)^2 in double precision (e lies in [0, 1] and the sums
// are exact to about 1e-13, far below what the single-precision threshold resolves), or min + k * (max - min).
__device__ __forceinline__ float threshold_from_stats(double sum, double lo, double hi, double sumsq, int64_t pixels,
                                                      int rule, float k)
{
    if (rule == FS_MASK_MEAN_STD) {
        const double mean = sum / (double)pixels;
        double var = sumsq / (double)pixels - mean * mean;
        var = var > 0.0 ? var : 0.0;
        return (float)(mean + (double)k * sqrt(var));
    }
    const float l = (float)lo, h = (float)hi;
    return l + k * (h - l);
}

// The record a forward pass leaves for the count pass (see k_score_bits).  For every pair that the multi-view score
// counts at one or more pixels of its tile: a row of PAIR_BITS_BYTES (which pixels) and the pair's Gaussian.  The rows of
// a tile sit together at the start of the tile's segment of the pair arrays, [ranges[tile].x, + tile_rows[tile]), in no
// particular order; pairs that are counted nowhere leave nothing.  rows == null: no record.
constexpr int PAIR_BITS_BYTES = 32;
struct ScoreRecord {
    uint4* rows;           // [P, 2]
    uint32_t* row_gauss;   // [P]
    int32_t* tile_rows;    // [tiles]
};
inline size_t score_record_bytes(int64_t num_pairs, int tiles)
{
    return (size_t)num_pairs * (PAIR_BITS_BYTES + sizeof(uint32_t)) + (size_t)tiles * sizeof(int32_t);
}
inline ScoreRecord score_record_at(void* base, int64_t num_pairs)
{
    unsigned char* b = static_cast<unsigned char*>(base);
    ScoreRecord r;
    r.rows = reinterpret_cast<uint4*>(b);
    r.row_gauss = reinterpret_cast<uint32_t*>(b + (size_t)num_pairs * PAIR_BITS_BYTES);
    r.tile_rows = reinterpret_cast<int32_t*>(b + (size_t)num_pairs * (PAIR_BITS_BYTES + sizeof(uint32_t)));
    return r;
}
// The record a forward pass leaves for k_render_bwd: the pairs it blended at some pixel of their tile, in list order, at the start of
// the tile's segment of the pair arrays, [ranges[tile].x, + tile_count[tile]): the Gaussian, and the pair's position in the tile's list
// (from 0, 16 bits) with the sub-tiles that blended it above (bit st: see SubTiles in render.hip).  Lists beyond the
// per-tile sorts' have none.  entries == null: no record.
struct BlendRecord {
    uint2* entries;        // [P]
    int32_t* tile_count;   // [tiles]
};
hipError_t launch_render_fwd(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                             const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, float* image, float* final_T,
                             uint32_t* n_contrib, const ScoreRecord& record, const BlendRecord& blends);

// forward pass with the L1 term and the error map fused into its epilogue (see k_render_fwd);
// tile_partial: 5 * tiles doubles, err: H*W floats, dL may be null; record as for launch_render_fwd
hipError_t launch_render_fwd_fused(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                                   const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats,
                                   float* image, float* final_T, uint32_t* n_contrib, const float* target, float* dL,
                                   float* err, double* tile_partial, const ScoreRecord& record, const BlendRecord& blends);
// the count pass from that record: counts[g] += |bits(row) & mask(tile)| over the rows of every tile
// (longest_list: an upper bound of the rows of any tile, 0 if not known)
hipError_t launch_score_bits(hipStream_t st, const CamDev& cam, const uint32_t* ranges, const ScoreRecord& record,
                             const uint8_t* mask, int32_t* counts, int64_t longest_list);
// the same with the mask made on the way: mask[p] <- err[p] > threshold(stats, rule, k) for every pixel (stats: the four
// doubles {sum, min, max, sum of squares} of the error map), *thr_out <- the threshold, then the count as above
hipError_t launch_mask_score_bits(hipStream_t st, const CamDev& cam, const uint32_t* ranges, const ScoreRecord& record,
                                  const float* err, const double* stats, int rule, float k, uint8_t* mask, float* thr_out,
                                  int32_t* counts, int64_t longest_list);
// rows[tile] <- the record's number of rows of the tile
hipError_t launch_record_rows(hipStream_t st, int tiles, const ScoreRecord& record, int32_t* rows);
// stats: >= fused_partials() doubles: {sum, min, max, sum of squares} of the error map
int fused_partials();
hipError_t launch_fold_tile_partials(hipStream_t st, const double* tile_partial, int tiles, int64_t count,
                                     double* stats, double* loss_out);
hipError_t launch_error_mask_from_map(hipStream_t st, int64_t pixels, int rule, float k, const float* err,
                                      const double* stats, uint8_t* mask, float* thr);

hipError_t launch_render_bwd(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                             const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, const float* final_T,
                             const uint32_t* n_contrib, const float* dL_dimage, float* pair_grad, uint8_t* rec_valid,
                             bool abs_grad, bool per_splat, const BlendRecord& blends);

hipError_t launch_score(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                        const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, const uint32_t* n_contrib,
                        const uint8_t* mask, int32_t* counts);

hipError_t launch_l1_grad(hipStream_t st, const float* image, const float* target, int64_t count,
                          float* dL, double* partial /* >= l1_partials() doubles */, double* loss_out);
int l1_partials();

// err: [H*W] floats, partial: >= 4*mask_partials() doubles
hipError_t launch_error_mask(hipStream_t st, const float* image, const float* target, int64_t pixels, int rule,
                             float k, float* err, double* partial, uint8_t* mask, float* thr_out);
int mask_partials();

// Photometric loss (1-lambda) L1 + lambda (1 - SSIM).  dmaps: 3 * 3*H*W floats (only touched when dL != null);
// partial: >= 2 * photo_blocks(H, W) doubles; dL (may be null): dE/d image; out3 (may be null): {L1, SSIM, E}.
int photo_blocks(int H, int W);
hipError_t launch_photo_loss(hipStream_t st, const float* image, const float* target, int H, int W, float lambda,
                             float* dmaps, double* partial, float* dL, double* out3);
// acc[i] += counts[i] * *E;  then out = min-max normalised acc (partial: >= 2*mask_partials() + 2 doubles)
hipError_t launch_prune_accumulate(hipStream_t st, const int32_t* counts, int64_t n, const double* E, double* acc);
hipError_t launch_score_view_end(hipStream_t st, int32_t* counts, int64_t n, const double* E, double* acc, int32_t* total);
hipError_t launch_prune_normalize(hipStream_t st, const double* acc, int64_t n, double* partial, float* out);

// densification / pruning decisions and index plumbing (densify.hip)
hipError_t launch_densify_accumulate(hipStream_t st, int64_t n, const float* dmean2d, const float* dabs,
                                     const uint32_t* touched, float* grad_accum, float* abs_accum, uint32_t* denom);
hipError_t launch_select(hipStream_t st, int64_t n, const float* grad_accum, const float* abs_accum,
                         const uint32_t* denom, const int32_t* counts, const float* scales, const float* opac,
                         const float* s_p, const fs_select_params& prm, uint8_t* clone, uint8_t* split, uint8_t* prune);
// positions: uint32 [n] scratch; total_dev receives the number of selected elements
hipError_t launch_compact(hipStream_t st, int64_t n, const uint8_t* mask, uint32_t* positions, void* scan_tmp,
                          uint64_t* total_dev, uint32_t* indices);
hipError_t launch_gather_rows(hipStream_t st, const float* src, int row_floats, const uint32_t* indices,
                              int64_t count, float* dst);

hipError_t launch_combine_masks(hipStream_t st, int64_t n, const uint8_t* clone, const uint8_t* split,
                                const uint8_t* prune, uint8_t* keep, uint8_t* clone_eff, uint8_t* split_eff);
hipError_t launch_counts_add(hipStream_t st, int64_t n, int32_t* total, const int32_t* view);
// children of m split parents: rows c*m + r of child_means / child_scales [2m,3]; normals [m,2,3]
hipError_t launch_split_children(hipStream_t st, int64_t m, const float* means, const float* scales, const float* quats,
                                 const uint32_t* parents, const float* normals, float phi, float* child_means,
                                 float* child_scales);
// keys[j] = bits(exponentials[i] / scores[i]) << 32 | i, vals[j] = i for the m listed candidates i = cand_idx[j]
hipError_t launch_sample_keys(hipStream_t st, int64_t m, const uint32_t* cand_idx, const float* scores,
                              const float* exponentials, uint64_t* keys, uint32_t* vals);
// mask[0..n) = 0, then mask[idx[j]] = 1 for j < k
hipError_t launch_mark_indices(hipStream_t st, int64_t n, int64_t k, const uint32_t* idx, uint8_t* mask);

// optimiser and activations (optimizer.hip)
hipError_t launch_adam(hipStream_t st, float* p, float* g, float* m, float* v, int64_t count, float lr, float beta1,
                       float beta2, float eps, int step, float grad_scale, bool zero_grad);
hipError_t launch_grad_accumulate(hipStream_t st, float* acc, const float* g, int64_t count);
hipError_t launch_activate(hipStream_t st, int64_t n, const float* raw_s, const float* raw_q, const float* raw_o,
                           float* s, float* q, float* o);
hipError_t launch_activate_bwd(hipStream_t st, int64_t n, const float* raw_s, const float* raw_q, const float* raw_o,
                               const float* d_s, const float* d_q, const float* d_o, float* d_raw_s, float* d_raw_q,
                               float* d_raw_o);
hipError_t launch_activate_inv(hipStream_t st, int64_t n, const float* s, const float* o, float lo, float hi,
                               float* raw_s, float* raw_o);

// reference measurements: streaming copy of `bytes` (multiple of 16), and 8 fma chains x iters per lane on
// blocks x 256 lanes (out: blocks * 256 floats)
hipError_t launch_copy(hipStream_t st, const void* src, void* dst, int64_t bytes);
hipError_t launch_fma_chain(hipStream_t st, float* out, int blocks, int iters);

hipError_t launch_fill_u32(hipStream_t st, uint32_t* p, uint32_t v, int64_t count);

}  // namespace fs
