// Image-space helpers of the hot path (gfx950): L1 term with its gradient, the per-pixel
// error map / threshold / high-error mask of FastGS Sec. 4.2 (first three equations), the
// photometric loss E = (1 - lambda) L1 + lambda (1 - SSIM) of Sec. 4.3 / Sec. 4.5 with its
// gradient, and the pruning score of Sec. 4.3.
//
// Reductions over the image run in double precision in a fixed tree (per-thread strided sums,
// wavefront shuffle tree, per-workgroup partials, one final workgroup), so results do not depend
// on scheduling.
#include "common.hpp"

namespace fs {

namespace {

// final reduction of RED_BLOCKS partials by one workgroup (thread i takes partials i, i+256, ... in order)
template <RedOp OP>
__device__ __forceinline__ double final_reduce(const double* partial, double* smem)
{
    double v = partial[threadIdx.x];
#pragma unroll
    for (int k = 1; k < RED_BLOCKS / RED_THREADS; k++) v = red_combine<OP>(v, partial[k * RED_THREADS + threadIdx.x]);
    return block_reduce<OP>(v, smem);
}

// VEC = 4: 16-byte accesses (count a multiple of 4, arrays 16-byte aligned); VEC = 1 otherwise.  The sum is
// accumulated per thread in element order either way.
template <int VEC>
__global__ __launch_bounds__(RED_THREADS) void k_l1_grad(const float* __restrict__ image,
                                                        const float* __restrict__ target, int64_t count,
                                                        float scale, float* __restrict__ dL,
                                                        double* __restrict__ partial)
{
    __shared__ double smem[4];
    double s = 0.0;
    const int64_t stride = (int64_t)RED_BLOCKS * RED_THREADS;
    if (VEC == 4) {
        const float4* a4 = reinterpret_cast<const float4*>(image);
        const float4* b4 = reinterpret_cast<const float4*>(target);
        float4* d4 = reinterpret_cast<float4*>(dL);
        for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < (count >> 2); i += stride) {
            const float4 a = a4[i], b = b4[i];
            const float d0 = a.x - b.x, d1 = a.y - b.y, d2 = a.z - b.z, d3 = a.w - b.w;
            s += (double)fabsf(d0); s += (double)fabsf(d1); s += (double)fabsf(d2); s += (double)fabsf(d3);
            d4[i] = make_float4(d0 > 0.f ? scale : (d0 < 0.f ? -scale : 0.f), d1 > 0.f ? scale : (d1 < 0.f ? -scale : 0.f),
                                d2 > 0.f ? scale : (d2 < 0.f ? -scale : 0.f), d3 > 0.f ? scale : (d3 < 0.f ? -scale : 0.f));
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < count; i += stride) {
            const float d = image[i] - target[i];
            s += (double)fabsf(d);
            dL[i] = d > 0.f ? scale : (d < 0.f ? -scale : 0.f);
        }
    }
    s = block_reduce<RED_SUM>(s, smem);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ __launch_bounds__(RED_THREADS) void k_l1_final(const double* __restrict__ partial, int64_t count,
                                                         double* __restrict__ loss_out)
{
    __shared__ double smem[4];
    const double s = final_reduce<RED_SUM>(partial, smem);
    if (threadIdx.x == 0) *loss_out = s / (double)count;
}

// e = ((|d0| + |d1|) + |d2|) / 3 per pixel; partial sums / minima / maxima / sums of squares per workgroup.
// VEC = 4: four neighbouring pixels per thread with 16-byte accesses (pixels a multiple of 4, arrays aligned).
template <int VEC>
__global__ __launch_bounds__(RED_THREADS) void k_err_map(const float* __restrict__ image,
                                                        const float* __restrict__ target, int64_t pixels,
                                                        float* __restrict__ err, double* __restrict__ partial)
{
    __shared__ double smem[4];
    double s = 0.0, sq = 0.0, lo = 1.0e300, hi = -1.0e300;
    const int64_t stride = (int64_t)RED_BLOCKS * RED_THREADS;
    auto one = [&](float i0, float i1, float i2, float t0, float t1, float t2) {
        const float e = ((fabsf(i0 - t0) + fabsf(i1 - t1)) + fabsf(i2 - t2)) / 3.0f;
        s += (double)e;
        sq += (double)e * (double)e;
        lo = (double)e < lo ? (double)e : lo;
        hi = (double)e > hi ? (double)e : hi;
        return e;
    };
    if (VEC == 4) {
        const int64_t q = pixels >> 2;
        const float4* a4 = reinterpret_cast<const float4*>(image);
        const float4* b4 = reinterpret_cast<const float4*>(target);
        float4* e4 = reinterpret_cast<float4*>(err);
        for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < q; i += stride) {
            const float4 a0 = a4[i], a1 = a4[q + i], a2 = a4[2 * q + i];
            const float4 b0 = b4[i], b1 = b4[q + i], b2 = b4[2 * q + i];
            float4 e;
            e.x = one(a0.x, a1.x, a2.x, b0.x, b1.x, b2.x);
            e.y = one(a0.y, a1.y, a2.y, b0.y, b1.y, b2.y);
            e.z = one(a0.z, a1.z, a2.z, b0.z, b1.z, b2.z);
            e.w = one(a0.w, a1.w, a2.w, b0.w, b1.w, b2.w);
            e4[i] = e;
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < pixels; i += stride)
            err[i] = one(image[i], image[pixels + i], image[2 * pixels + i], target[i], target[pixels + i],
                         target[2 * pixels + i]);
    }
    s = block_reduce<RED_SUM>(s, smem);
    lo = block_reduce<RED_MIN>(lo, smem);
    hi = block_reduce<RED_MAX>(hi, smem);
    sq = block_reduce<RED_SUM>(sq, smem);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = s;
        partial[RED_BLOCKS + blockIdx.x] = lo;
        partial[2 * RED_BLOCKS + blockIdx.x] = hi;
        partial[3 * RED_BLOCKS + blockIdx.x] = sq;
    }
}

// After the fused forward kernel: workgroup q folds number q of its per-tile partials ([5][tiles]: sum |d|; sum, min,
// max, sum of squares of e) in a fixed order (thread b takes tiles b, b + 1024, ...; then a shuffle tree), which leaves
// stats[0..3] = {sum e, min e, max e, sum e^2} and the L1 loss.  A chain of latencies (loads, six steps of the tree, sixteen
// wavefronts' results one after the other): one workgroup for all five went through them with five times the work in each.
// 7.1 and 4.2 us at 1600x1064; ten views of the score pass at 300k Gaussians 2016 and 1984 us, at 100k 1468 and 1432.
constexpr int FOLD_THREADS = 1024;
constexpr int FOLD_QUANTITIES = 5;
__global__ __launch_bounds__(FOLD_THREADS) void k_fold_tile_stats(const double* __restrict__ tile_partial, int tiles,
                                                                  int64_t count, double* __restrict__ stats,
                                                                  double* __restrict__ loss_out)
{
    __shared__ double sm[FOLD_THREADS / 64];
    const int q = blockIdx.x;
    if (q == 0 && !loss_out) return;
    const double* const part = tile_partial + (size_t)q * tiles;
    auto fold = [&](double none, auto join) {   // (the result is thread 0's)
        double a = none;
        for (int t0 = threadIdx.x; t0 < tiles; t0 += 8 * FOLD_THREADS) {   // 8 loads in flight per round
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) v[u] = t0 + u * FOLD_THREADS < tiles ? part[t0 + u * FOLD_THREADS] : none;
#pragma unroll
            for (int u = 0; u < 8; u++) a = join(a, v[u]);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) a = join(a, shfl_down_f64(a, d));
        if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = a;
        __syncthreads();
        a = none;
        if (threadIdx.x == 0)
#pragma unroll
            for (int w = 0; w < FOLD_THREADS / 64; w++) a = join(a, sm[w]);
        return a;
    };
    double r;
    if (q == 2) r = fold(1.0e300, [](double a, double v) { return v < a ? v : a; });
    else if (q == 3) r = fold(-1.0e300, [](double a, double v) { return v > a ? v : a; });
    else r = fold(0.0, [](double a, double v) { return a + v; });
    if (threadIdx.x == 0) {
        if (q == 0) *loss_out = r / (double)count;
        else stats[q - 1] = r;
    }
}

// threshold from the RED_BLOCKS-wide partials of k_err_map (one workgroup), written as one float
__global__ __launch_bounds__(RED_THREADS) void k_err_threshold(const double* __restrict__ partial, int64_t pixels,
                                                              int rule, float k, float* __restrict__ thr)
{
    __shared__ double smem[4];
    const double tot = final_reduce<RED_SUM>(partial, smem);
    const double lo = final_reduce<RED_MIN>(partial + RED_BLOCKS, smem);
    const double hi = final_reduce<RED_MAX>(partial + 2 * RED_BLOCKS, smem);
    const double sq = final_reduce<RED_SUM>(partial + 3 * RED_BLOCKS, smem);
    if (threadIdx.x == 0) *thr = threshold_from_stats(tot, lo, hi, sq, pixels, rule, k);
}

__global__ __launch_bounds__(256) void k_err_mask(const float* __restrict__ err, int64_t pixels,
                                                  const float* __restrict__ thr, uint8_t* __restrict__ mask)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < pixels) mask[i] = err[i] > *thr;
}

// the mask straight from the four statistics that k_fold_tile_stats left (every thread forms the threshold itself;
// the first one also stores it)
__global__ __launch_bounds__(256) void k_err_mask_stats(const float* __restrict__ err, int64_t pixels,
                                                        const double* __restrict__ stats, int rule, float k,
                                                        uint8_t* __restrict__ mask, float* __restrict__ thr_out)
{
    const float thr = threshold_from_stats(stats[0], stats[1], stats[2], stats[3], pixels, rule, k);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *thr_out = thr;
    if (i < pixels) mask[i] = err[i] > thr;
}

// ---- photometric loss: (1 - lambda) L1 + lambda (1 - SSIM) ---------------------------------------
// SSIM per channel under an 11x11 Gaussian window (sigma 1.5, sum 1, separable), image continued by
// zeros, C1 = 0.01^2, C2 = 0.03^2; its mean over channels and pixels.  With the window sums
// mu1 = <x>, mu2 = <y>, e11 = <x^2>, e22 = <y^2>, e12 = <x y>:
//   ssim = (2 mu1 mu2 + C1)(2 (e12 - mu1 mu2) + C2) / ((mu1^2 + mu2^2 + C1)(e11 - mu1^2 + e22 - mu2^2 + C2)).
// Gradient with respect to x: the three maps d ssim/d mu1, d ssim/d e11, d ssim/d e12 are window-summed
// again (the window is symmetric) and combined as  g = <d_mu1> + 2 x <d_e11> + y <d_e12>.
//
// One workgroup produces a 32-wide block of one channel: the block's input region goes to LDS, a horizontal 11-tap pass
// (one lane: 4 neighbouring columns of one row, sliding over 14 inputs) leaves the row-filtered planes in registers and then
// in the same LDS, and a vertical pass (one lane: SS_VO neighbouring rows of one column) finishes.
// Vector instructions weigh most in both kernels: 102 multiply-adds per value forward (44 of them 48/38 times for the rows of the
// halo), about 210 instructions in all.  What went, against a 32x32 block with separate LDS for the row-filtered planes, which
// took 260: the inputs' addresses and edge tests (a wavefront loads whole rows), 3 of 12 memory instructions per value (the
// three derivative maps lie side by side), and the serial epilogue (all of a lane's outputs are formed at once and only the
// stores are masked); the row-filtered planes take the inputs' place, so that six workgroups fit a compute unit instead of
// four.  38 rows: 48 rows of eight 4-column units are 384 = 1.5 trips of the 256 lanes.  Forward and backward, before and after:
// 51 and 46 us -> 42 and 34 at 1600x1064, 10.7 and 8.1 -> 8.8 and 7.1 at 509x337; forward alone at 1332x876 27.5 -> 23.7.
// (Blocks 32 rows high: 45 and 34 us at 1600x1064; 54 rows: 42 and 34, but 9.8 and 7.9 at 509x337.)
constexpr int SS_R = 5, SS_TAPS = 2 * SS_R + 1;
constexpr int SS_TW = 32, SS_TH = 38;
constexpr int SS_VO = (SS_TH + 7) / 8;                               // outputs (neighbouring rows of one column) per lane
constexpr int SS_IW = SS_TW + 2 * SS_R, SS_IH = SS_TH + 2 * SS_R;
constexpr int SS_IP = SS_IW + 2;                                     // padded LDS row
constexpr int SS_HR = 8 * SS_VO + 2 * SS_R;                          // rows the vertical pass reads (those from SS_IH on: for outputs nobody wants)
constexpr int SS_UNITS = SS_IH * (SS_TW / 4), SS_TRIPS = (SS_UNITS + 255) / 256;   // of the horizontal pass
constexpr int ss_floats(int planes_in, int planes_h)
{
    return planes_in * SS_IH * SS_IP > planes_h * SS_HR * SS_TW ? planes_in * SS_IH * SS_IP : planes_h * SS_HR * SS_TW;
}

// The window, rounded once from double: exp(-(k - 5)^2 / (2 1.5^2)) over their sum.  Literals: with the weight in a scalar register
// a run of multiply-adds takes 4.4 cycles of a SIMD each, with a literal or three vector registers 2.6.  Both kernels, in us, before and after:
// 73.7 and 71.1 at 1600x1064, 57.5 and 54.4 at 1332x876, 18.6 and 17.5 at 509x337; the forward one and the loss at 1332x876 29.5 and 26.7.
__device__ constexpr float SS_W[SS_TAPS] = {0x1.0d956c0000000p-10f, 0x1.f1fe020000000p-8f, 0x1.26eb180000000p-5f, 0x1.bff0fe0000000p-4f, 0x1.b43c400000000p-3f, 0x1.1065600000000p-2f,
                                            0x1.b43c400000000p-3f, 0x1.bff0fe0000000p-4f, 0x1.26eb180000000p-5f, 0x1.f1fe020000000p-8f, 0x1.0d956c0000000p-10f};
struct Floats3 { float v[3]; };

// The block's input region of one channel, continued by zeros, into NP planes in LDS: a wavefront takes whole rows (their
// addresses are scalar), and every load is issued before the first LDS write, so that their latencies overlap.
// fetch(row's first pixel, column) reads the NP values of one pixel.
template <int NP, typename Fetch>
__device__ __forceinline__ void ss_load(Fetch fetch, int H, int W, int x0, int y0, float (*dst)[SS_IH][SS_IP])
{
    constexpr int IT = (SS_IH + 3) / 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int gx = x0 + lane - SS_R;
    const bool in_col = lane < SS_IW && gx >= 0 && gx < W;
    const uint32_t col = in_col ? (uint32_t)gx : 0u;
    float v[IT][NP];
#pragma unroll
    for (int it = 0; it < IT; it++) {
        const int gy = y0 + wave + 4 * it - SS_R;
        const bool in_row = gy >= 0 && gy < H;
        fetch((size_t)(in_row ? gy : 0) * W, col, v[it]);   // (always a valid address)
#pragma unroll
        for (int p = 0; p < NP; p++) v[it][p] = in_row && in_col ? v[it][p] : 0.0f;
    }
#pragma unroll
    for (int it = 0; it < IT; it++) {
        const int r = wave + 4 * it;
        if (r < SS_IH && lane < SS_IW) {
#pragma unroll
            for (int p = 0; p < NP; p++) dst[p][r][lane] = v[it][p];
        }
    }
}

// vertical pass for the SS_VO outputs of this lane: rows r0 .. r0+SS_VO-1 of column c of one row-filtered plane
__device__ __forceinline__ void ss_vertical(const float (*h)[SS_TW], int r0, int c, float out[SS_VO])
{
    float col[SS_TAPS + SS_VO - 1];
#pragma unroll
    for (int i = 0; i < SS_TAPS + SS_VO - 1; i++) col[i] = h[r0 + i][c];
#pragma unroll
    for (int o = 0; o < SS_VO; o++) {
        float a = 0.f;
#pragma unroll
        for (int k = 0; k < SS_TAPS; k++) a = __builtin_fmaf(SS_W[k], col[k + o], a);
        out[o] = a;
    }
}

// dmaps: the three derivatives of a pixel side by side (12 bytes; null: not wanted)
__global__ __launch_bounds__(256, 6) void k_ssim_fwd(const float* __restrict__ image, const float* __restrict__ target,
                                                  int H, int W, float* __restrict__ dmaps,
                                                  double* __restrict__ partial, int nblocks)
{
    __shared__ __attribute__((aligned(16))) float s_buf[ss_floats(2, 4)];
    __shared__ double s_sum[2][4];
    float (*const s_in)[SS_IH][SS_IP] = reinterpret_cast<float (*)[SS_IH][SS_IP]>(s_buf);
    float (*const s_h)[SS_HR][SS_TW] = reinterpret_cast<float (*)[SS_HR][SS_TW]>(s_buf);
    const int x0 = blockIdx.x * SS_TW, y0 = blockIdx.y * SS_TH;
    const size_t plane = (size_t)blockIdx.z * H * W;
    const float *const img = image + plane, *const tgt = target + plane;
    ss_load<2>([=](size_t row, uint32_t col, float (&v)[2]) { v[0] = (img + row)[col]; v[1] = (tgt + row)[col]; }, H, W, x0, y0, s_in);
    __syncthreads();
    double ssum = 0.0, lsum = 0.0;
    float4 hor[SS_TRIPS][4];
#pragma unroll
    for (int t = 0; t < SS_TRIPS; t++) {
        const int u = threadIdx.x + 256 * t;
        if (u >= SS_UNITS) continue;
        const int r = u / (SS_TW / 4), c0 = (u % (SS_TW / 4)) * 4;
        // 16-byte LDS accesses: a lane's 16 inputs are four aligned float4s, and 8 neighbouring lanes cover
        // all banks (a 4-byte access pattern with stride 4 would hit every fourth bank only)
        // (only the sum e11 + e22 enters the index, so x^2 + y^2 is filtered as one plane)
        float xv[16], yv[16], sq[SS_TAPS + 3], xy[SS_TAPS + 3];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float4 a = *reinterpret_cast<const float4*>(&s_in[0][r][c0 + 4 * i]);
            const float4 b = *reinterpret_cast<const float4*>(&s_in[1][r][c0 + 4 * i]);
            xv[4 * i] = a.x; xv[4 * i + 1] = a.y; xv[4 * i + 2] = a.z; xv[4 * i + 3] = a.w;
            yv[4 * i] = b.x; yv[4 * i + 1] = b.y; yv[4 * i + 2] = b.z; yv[4 * i + 3] = b.w;
        }
#pragma unroll
        for (int i = 0; i < SS_TAPS + 3; i++) {
            sq[i] = __builtin_fmaf(xv[i], xv[i], yv[i] * yv[i]);
            xy[i] = xv[i] * yv[i];
        }
        if (r >= SS_R && r < SS_R + SS_TH) {   // the block's own pixels (both images are zero beyond the edge)
#pragma unroll
            for (int j = 0; j < 4; j++) lsum += (double)fabsf(xv[SS_R + j] - yv[SS_R + j]);
        }
        float o[4][4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float m1 = 0.f, m2 = 0.f, esq = 0.f, e12 = 0.f;
#pragma unroll
            for (int k = 0; k < SS_TAPS; k++) {
                const float wk = SS_W[k];
                m1 = __builtin_fmaf(wk, xv[j + k], m1);
                m2 = __builtin_fmaf(wk, yv[j + k], m2);
                esq = __builtin_fmaf(wk, sq[j + k], esq);
                e12 = __builtin_fmaf(wk, xy[j + k], e12);
            }
            o[0][j] = m1; o[1][j] = m2; o[2][j] = esq; o[3][j] = e12;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) hor[t][k] = make_float4(o[k][0], o[k][1], o[k][2], o[k][3]);
    }
    __syncthreads();   // (the inputs have been read: their place is taken)
#pragma unroll
    for (int t = 0; t < SS_TRIPS; t++) {
        const int u = threadIdx.x + 256 * t;
        if (u >= SS_UNITS) continue;
#pragma unroll
        for (int k = 0; k < 4; k++) *reinterpret_cast<float4*>(&s_h[k][u / (SS_TW / 4)][(u % (SS_TW / 4)) * 4]) = hor[t][k];
    }
    __syncthreads();
    const int c = threadIdx.x % SS_TW, r0 = (threadIdx.x / SS_TW) * SS_VO;
    float q[4][SS_VO];
#pragma unroll
    for (int k = 0; k < 4; k++) ss_vertical(s_h[k], r0, c, q[k]);
    const float C1 = 0.01f * 0.01f, C2 = 0.03f * 0.03f;
    const int gx = x0 + c, gy0 = y0 + r0, rows = gx < W ? min(min(SS_VO, SS_TH - r0), H - gy0) : 0;   // (may be negative)
    float* const d0 = dmaps + 3 * (plane + (size_t)gy0 * W + gx);
#pragma unroll
    for (int o = 0; o < SS_VO; o++) {
        const float m1 = q[0][o], m2 = q[1][o];
        const float mm = m1 * m1 + m2 * m2, s12 = q[3][o] - m1 * m2;
        const float A = 2.f * m1 * m2 + C1, B = 2.f * s12 + C2, Cq = mm + C1, D = (q[2][o] - mm) + C2;
        const float inv = 1.0f / (Cq * D);
        const float sv = A * B * inv;
        ssum += o < rows ? (double)sv : 0.0;
        if (dmaps) {
            Floats3 d;
            d.v[0] = (2.f * m2 * (B - A) - sv * 2.f * m1 * (D - Cq)) * inv;
            d.v[1] = -sv / D;
            d.v[2] = 2.f * A * inv;
            if (o < rows) *reinterpret_cast<Floats3*>(d0 + (size_t)o * 3 * W) = d;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        ssum += shfl_down_f64(ssum, d);
        lsum += shfl_down_f64(lsum, d);
    }
    if ((threadIdx.x & 63) == 0) { s_sum[0][threadIdx.x >> 6] = ssum; s_sum[1][threadIdx.x >> 6] = lsum; }
    __syncthreads();
    if (threadIdx.x < 2) {
        const int b = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        const double* const w = s_sum[threadIdx.x];
        partial[threadIdx.x * nblocks + b] = (w[0] + w[1]) + (w[2] + w[3]);
    }
}

// out3 = {L1, SSIM, (1 - lambda) L1 + lambda (1 - SSIM)}: one workgroup adds the partials in a fixed order
__device__ __forceinline__ void photo_final(const double* __restrict__ partial, int nblocks, double count, double lambda,
                                            double* __restrict__ out3, double* smem /*[4]*/)
{
    // 2 x 8 loads in flight per lane and round; the order of the additions is fixed
    double s = 0.0, l = 0.0;
    for (int i0 = threadIdx.x; i0 < nblocks; i0 += 8 * RED_THREADS) {
        double a[8], b[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int i = i0 + k * RED_THREADS;
            a[k] = i < nblocks ? partial[i] : 0.0;
            b[k] = i < nblocks ? partial[nblocks + i] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 8; k++) { s += a[k]; l += b[k]; }
    }
    s = block_reduce<RED_SUM>(s, smem);
    l = block_reduce<RED_SUM>(l, smem);
    if (threadIdx.x == 0) {
        const double ssim = s / count, l1 = l / count;
        // (a training iteration's host looks at these while the kernel runs: past every cache)
        __hip_atomic_store(&out3[0], l1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&out3[1], ssim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&out3[2], (1.0 - lambda) * l1 + lambda * (1.0 - ssim), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ __launch_bounds__(RED_THREADS) void k_photo_final(const double* __restrict__ partial, int nblocks,
                                                            double count, double lambda, double* __restrict__ out3)
{
    __shared__ double smem[4];
    photo_final(partial, nblocks, count, lambda, out3, smem);
}

// dE/dx = c_l1 sign(x - y) - c_ss (<d_mu1> + 2 x <d_e11> + y <d_e12>),  c_l1 = (1-lambda)/N, c_ss = lambda/N
__global__ __launch_bounds__(256) void k_ssim_bwd(const float* __restrict__ image, const float* __restrict__ target,
                                                  int H, int W, const float* __restrict__ dmaps,
                                                  float c_l1, float c_ss, float* __restrict__ dL,
                                                  const double* __restrict__ partial, int nblocks, double count, double lambda,
                                                  double* __restrict__ out3)
{
    static_assert(RED_THREADS == 256, "the loss is finished by a workgroup of this kernel");
    __shared__ __attribute__((aligned(16))) float s_buf[ss_floats(3, 3)];
    // with out3, the first row of the grid is no block of the image: one of its workgroups finishes the loss
    const int row0 = out3 ? 1 : 0;
    if ((int)blockIdx.y < row0) {
        if (blockIdx.x == 0 && blockIdx.z == 0) photo_final(partial, nblocks, count, lambda, out3, reinterpret_cast<double*>(s_buf));
        return;
    }
    float (*const s_in)[SS_IH][SS_IP] = reinterpret_cast<float (*)[SS_IH][SS_IP]>(s_buf);
    float (*const s_h)[SS_HR][SS_TW] = reinterpret_cast<float (*)[SS_HR][SS_TW]>(s_buf);
    const int x0 = blockIdx.x * SS_TW, y0 = ((int)blockIdx.y - row0) * SS_TH;
    const size_t plane = (size_t)blockIdx.z * H * W;
    const float* const maps = dmaps + 3 * plane;
    ss_load<3>([=](size_t row, uint32_t col, float (&v)[3]) {
        const Floats3 d = reinterpret_cast<const Floats3*>(maps + 3 * row)[col];
        v[0] = d.v[0]; v[1] = d.v[1]; v[2] = d.v[2];
    }, H, W, x0, y0, s_in);
    __syncthreads();
    float4 hor[SS_TRIPS][3];
#pragma unroll
    for (int t = 0; t < SS_TRIPS; t++) {
        const int u = threadIdx.x + 256 * t;
        if (u >= SS_UNITS) continue;
        const int r = u / (SS_TW / 4), c0 = (u % (SS_TW / 4)) * 4;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            float v[16], o[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float4 a = *reinterpret_cast<const float4*>(&s_in[k][r][c0 + 4 * i]);
                v[4 * i] = a.x; v[4 * i + 1] = a.y; v[4 * i + 2] = a.z; v[4 * i + 3] = a.w;
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                float a = 0.f;
#pragma unroll
                for (int i = 0; i < SS_TAPS; i++) a = __builtin_fmaf(SS_W[i], v[j + i], a);
                o[j] = a;
            }
            hor[t][k] = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
    __syncthreads();
    // this lane's pixels (requested here, needed at the end)
    const int c = threadIdx.x % SS_TW, r0 = (threadIdx.x / SS_TW) * SS_VO;
    const int gx = x0 + c, gy0 = y0 + r0, rows = gx < W ? min(min(SS_VO, SS_TH - r0), H - gy0) : 0;   // (may be negative)
    const size_t p0 = plane + (size_t)gy0 * W + gx;
    float x[SS_VO], y[SS_VO];
#pragma unroll
    for (int o = 0; o < SS_VO; o++) {
        x[o] = o < rows ? image[p0 + (size_t)o * W] : 0.f;
        y[o] = o < rows ? target[p0 + (size_t)o * W] : 0.f;
    }
#pragma unroll
    for (int t = 0; t < SS_TRIPS; t++) {
        const int u = threadIdx.x + 256 * t;
        if (u >= SS_UNITS) continue;
#pragma unroll
        for (int k = 0; k < 3; k++) *reinterpret_cast<float4*>(&s_h[k][u / (SS_TW / 4)][(u % (SS_TW / 4)) * 4]) = hor[t][k];
    }
    __syncthreads();
    float q[3][SS_VO];
#pragma unroll
    for (int k = 0; k < 3; k++) ss_vertical(s_h[k], r0, c, q[k]);
#pragma unroll
    for (int o = 0; o < SS_VO; o++) {
        const float g = q[0][o] + 2.f * x[o] * q[1][o] + y[o] * q[2][o];
        const float d = x[o] - y[o];
        const float sg = d > 0.f ? c_l1 : (d < 0.f ? -c_l1 : 0.f);
        if (o < rows) dL[p0 + (size_t)o * W] = sg - c_ss * g;
    }
}

// ---- pruning score (Sec. 4.3): s_p = N(sum_j count_i^j E^j) -------------------------------------
__global__ __launch_bounds__(256) void k_prune_accumulate(const int32_t* __restrict__ counts, int64_t n,
                                                          const double* __restrict__ E, double* __restrict__ acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) acc[i] = acc[i] + (double)counts[i] * *E;
}

// The end of one view of a score pass in one launch: its counts weighed into the score and added to the total, and cleared for
// the next view.  (12 bytes read and 16 written per Gaussian: a launch's own few microseconds.  As a weighing, an addition and
// a fill: 4.6 + 3.3 + 4.4 us at 300k Gaussians, 5.2 this way.)
__global__ __launch_bounds__(256) void k_score_view_end(int32_t* __restrict__ counts, int64_t n, const double* __restrict__ E,
                                                        double* __restrict__ acc, int32_t* __restrict__ total)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t c = counts[i];
    acc[i] = acc[i] + (double)c * *E;
    total[i] = total[i] + c;
    counts[i] = 0;
}

__global__ __launch_bounds__(RED_THREADS) void k_minmax_f64(const double* __restrict__ v, int64_t n,
                                                           double* __restrict__ partial)
{
    __shared__ double smem[4];
    double lo = 1.0e300, hi = -1.0e300;
    for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < n; i += (int64_t)RED_BLOCKS * RED_THREADS) {
        lo = v[i] < lo ? v[i] : lo;
        hi = v[i] > hi ? v[i] : hi;
    }
    lo = block_reduce<RED_MIN>(lo, smem);
    hi = block_reduce<RED_MAX>(hi, smem);
    if (threadIdx.x == 0) { partial[blockIdx.x] = lo; partial[RED_BLOCKS + blockIdx.x] = hi; }
}

__global__ __launch_bounds__(RED_THREADS) void k_minmax_final(double* __restrict__ partial)
{
    __shared__ double smem[4];
    const double lo = final_reduce<RED_MIN>(partial, smem);
    const double hi = final_reduce<RED_MAX>(partial + RED_BLOCKS, smem);
    if (threadIdx.x == 0) { partial[2 * RED_BLOCKS] = lo; partial[2 * RED_BLOCKS + 1] = hi; }
}

__global__ __launch_bounds__(256) void k_prune_normalize(const double* __restrict__ acc, int64_t n,
                                                         const double* __restrict__ lohi, float* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double lo = lohi[0], hi = lohi[1];
    out[i] = hi > lo ? (float)((acc[i] - lo) / (hi - lo)) : 0.0f;
}

}  // namespace

int l1_partials() { return RED_BLOCKS; }
int mask_partials() { return RED_BLOCKS; }
int fused_partials() { return 4; }

hipError_t launch_l1_grad(hipStream_t st, const float* image, const float* target, int64_t count, float* dL,
                          double* partial, double* loss_out)
{
    if (count <= 0) return hipSuccess;
    const float scale = 1.0f / (float)count;
    const bool vec = count % 4 == 0 && ((reinterpret_cast<uintptr_t>(image) | reinterpret_cast<uintptr_t>(target) |
                                         reinterpret_cast<uintptr_t>(dL)) & 15u) == 0;
    if (vec)
        hipLaunchKernelGGL(k_l1_grad<4>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, st, image, target, count, scale, dL, partial);
    else
        hipLaunchKernelGGL(k_l1_grad<1>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, st, image, target, count, scale, dL, partial);
    if (loss_out) hipLaunchKernelGGL(k_l1_final, dim3(1), dim3(RED_THREADS), 0, st, partial, count, loss_out);
    return hipGetLastError();
}

hipError_t launch_error_mask(hipStream_t st, const float* image, const float* target, int64_t pixels, int rule,
                             float k, float* err, double* partial, uint8_t* mask, float* thr)
{
    if (pixels <= 0) return hipSuccess;
    const bool vec = pixels % 4 == 0 && ((reinterpret_cast<uintptr_t>(image) | reinterpret_cast<uintptr_t>(target) |
                                          reinterpret_cast<uintptr_t>(err)) & 15u) == 0;
    if (vec)
        hipLaunchKernelGGL(k_err_map<4>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, st, image, target, pixels, err, partial);
    else
        hipLaunchKernelGGL(k_err_map<1>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, st, image, target, pixels, err, partial);
    hipLaunchKernelGGL(k_err_threshold, dim3(1), dim3(RED_THREADS), 0, st, partial, pixels, rule, k, thr);
    hipLaunchKernelGGL(k_err_mask, dim3((unsigned)((pixels + 255) / 256)), dim3(256), 0, st, err, pixels, thr, mask);
    return hipGetLastError();
}

int photo_blocks(int H, int W) { return ((W + SS_TW - 1) / SS_TW) * ((H + SS_TH - 1) / SS_TH) * 3; }

hipError_t launch_photo_loss(hipStream_t st, const float* image, const float* target, int H, int W, float lambda,
                             float* dmaps, double* partial, float* dL, double* out3)
{
    const dim3 grid((unsigned)((W + SS_TW - 1) / SS_TW), (unsigned)((H + SS_TH - 1) / SS_TH), 3);
    const int nb = photo_blocks(H, W);
    const double count = 3.0 * (double)H * (double)W;
    hipLaunchKernelGGL(k_ssim_fwd, grid, dim3(256), 0, st, image, target, H, W, dL ? dmaps : nullptr, partial, nb);
    // the loss is a few thousand partials, most of whose own launch is waiting: with a gradient it is finished beside it
    // (a training iteration at 12k Gaussians / 509x337 106.3 -> 103.1 us, 300k / 1332x876 428.0 -> 424.4, 500k / 1600x1064 704.8 -> 700.2)
    if (dL)
        hipLaunchKernelGGL(k_ssim_bwd, dim3(grid.x, grid.y + (out3 ? 1 : 0), 3), dim3(256), 0, st, image, target, H, W, dmaps,
                           (float)((1.0 - (double)lambda) / count), (float)((double)lambda / count), dL, partial, nb, count,
                           (double)lambda, out3);
    else if (out3)
        hipLaunchKernelGGL(k_photo_final, dim3(1), dim3(RED_THREADS), 0, st, partial, nb, count, (double)lambda, out3);
    return hipGetLastError();
}

hipError_t launch_prune_accumulate(hipStream_t st, const int32_t* counts, int64_t n, const double* E, double* acc)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prune_accumulate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, counts, n, E, acc);
    return hipGetLastError();
}

hipError_t launch_score_view_end(hipStream_t st, int32_t* counts, int64_t n, const double* E, double* acc, int32_t* total)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_score_view_end, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, counts, n, E, acc, total);
    return hipGetLastError();
}

hipError_t launch_prune_normalize(hipStream_t st, const double* acc, int64_t n, double* partial, float* out)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_minmax_f64, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, st, acc, n, partial);
    hipLaunchKernelGGL(k_minmax_final, dim3(1), dim3(RED_THREADS), 0, st, partial);
    hipLaunchKernelGGL(k_prune_normalize, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, acc, n,
                       partial + 2 * RED_BLOCKS, out);
    return hipGetLastError();
}

// After the fused forward kernel: its per-tile partials -> stats[0..3] and, optionally, the L1 loss.
hipError_t launch_fold_tile_partials(hipStream_t st, const double* tile_partial, int tiles, int64_t count,
                                     double* stats, double* loss_out)
{
    hipLaunchKernelGGL(k_fold_tile_stats, dim3(FOLD_QUANTITIES), dim3(FOLD_THREADS), 0, st, tile_partial, tiles, count, stats, loss_out);
    return hipGetLastError();
}

// fs_error_mask without its first pass: the error map and its statistics are already in place
hipError_t launch_error_mask_from_map(hipStream_t st, int64_t pixels, int rule, float k, const float* err,
                                      const double* stats, uint8_t* mask, float* thr)
{
    if (pixels <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_err_mask_stats, dim3((unsigned)((pixels + 255) / 256)), dim3(256), 0, st, err, pixels, stats, rule, k,
                       mask, thr);
    return hipGetLastError();
}

}  // namespace fs
