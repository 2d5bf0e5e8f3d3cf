// Optimiser side of the training iteration (gfx950): fused Adam update (FastGS Sec. 5.1 trains with Adam;
// supplement "Implementation Details": updates every 32 / 64 iterations late in training, the gradients
// of the iterations in between being summed), and the stored -> used parameter activations of vanilla 3DGS
// with their chain rule.  All HBM-bound streaming kernels.
#include "common.hpp"

namespace fs {

namespace {

// 28 bytes of traffic per parameter (p, g, m, v read; p, m, v written); 16-byte accesses on the aligned body.
// When zero_grad is set the gradient is cleared in the same pass (+4 bytes), which saves the separate fill
// that an accumulate-then-step schedule needs.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, int64_t count, AdamArgs a, int zero_grad)
{
    const int64_t nvec = count >> 2;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    float4* p4 = reinterpret_cast<float4*>(p);
    float4* g4 = reinterpret_cast<float4*>(g);
    float4* m4 = reinterpret_cast<float4*>(m);
    float4* v4 = reinterpret_cast<float4*>(v);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += stride) {
        float4 pp = p4[i], mm = m4[i], vv = v4[i];
        const float4 gg = g4[i];
        adam_one(pp.x, gg.x, mm.x, vv.x, a, a.lr);
        adam_one(pp.y, gg.y, mm.y, vv.y, a, a.lr);
        adam_one(pp.z, gg.z, mm.z, vv.z, a, a.lr);
        adam_one(pp.w, gg.w, mm.w, vv.w, a, a.lr);
        p4[i] = pp; m4[i] = mm; v4[i] = vv;
        if (zero_grad) g4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // tail (count not a multiple of 4)
    const int64_t t = (nvec << 2) + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) {
        float pp = p[t], mm = m[t], vv = v[t];
        adam_one(pp, g[t], mm, vv, a, a.lr);
        p[t] = pp; m[t] = mm; v[t] = vv;
        if (zero_grad) g[t] = 0.f;
    }
}

__global__ __launch_bounds__(256) void k_grad_accumulate(float* __restrict__ acc, const float* __restrict__ g,
                                                         int64_t count)
{
    const int64_t nvec = count >> 2;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    float4* a4 = reinterpret_cast<float4*>(acc);
    const float4* g4 = reinterpret_cast<const float4*>(g);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += stride) {
        float4 a = a4[i];
        const float4 b = g4[i];
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
        a4[i] = a;
    }
    const int64_t t = (nvec << 2) + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) acc[t] = acc[t] + g[t];
}

// s = exp(raw), q = raw / |raw|, sigma = 1 / (1 + exp(-raw))
__global__ __launch_bounds__(256) void k_activate(int64_t n, const float* __restrict__ raw_s,
                                                  const float4* __restrict__ raw_q, const float* __restrict__ raw_o,
                                                  float* __restrict__ s, float4* __restrict__ q, float* __restrict__ o)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int k = 0; k < 3; k++) s[3 * i + k] = expf(raw_s[3 * i + k]);
    float inv;
    q[i] = unit_quat(raw_q[i], inv);
    o[i] = logistic(raw_o[i]);
}

// chain rule through k_activate; gradients may be written over the incoming ones
__global__ __launch_bounds__(256) void k_activate_bwd(int64_t n, const float* __restrict__ raw_s,
                                                      const float4* __restrict__ raw_q,
                                                      const float* __restrict__ raw_o, const float* d_s,
                                                      const float4* d_q, const float* d_o, float* d_raw_s,
                                                      float4* d_raw_q, float* d_raw_o)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int k = 0; k < 3; k++) d_raw_s[3 * i + k] = d_s[3 * i + k] * expf(raw_s[3 * i + k]);
    d_raw_q[i] = unit_quat_bwd(raw_q[i], d_q[i]);
    const float sg = logistic(raw_o[i]);
    d_raw_o[i] = d_o[i] * sg * (1.0f - sg);
}

// the inverse of k_activate for scale and opacity: raw scale = ln s, raw opacity = ln(o' / (1 - o')) with the
// opacity limited to [lo, hi]
__global__ __launch_bounds__(256) void k_activate_inv(int64_t n, const float* __restrict__ s,
                                                      const float* __restrict__ o, float lo, float hi,
                                                      float* __restrict__ raw_s, float* __restrict__ raw_o)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int k = 0; k < 3; k++) raw_s[3 * i + k] = logf(s[3 * i + k]);
    const float v = fminf(fmaxf(o[i], lo), hi);
    raw_o[i] = logf(v / (1.0f - v));
}

// ---- reference measurements ------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy(const float4* __restrict__ src, float4* __restrict__ dst, int64_t nvec)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += stride) dst[i] = src[i];
}

// 8 independent chains of fused multiply-adds per lane; the result is stored so that nothing is optimised away.  Factor and
// addend are in vector registers and the sum replaces its third operand, the form that issues fastest: with the factor in a scalar
// register, where a kernel's argument stays, an instruction takes 4.6 cycles of a SIMD instead of 2.6 (71 and 128 TFLOP/s).
__global__ __launch_bounds__(256) void k_fma_chain(float* __restrict__ out, int iters, float a, float b)
{
    asm volatile("" : "+v"(a), "+v"(b));
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; k++) x[k] = (float)threadIdx.x + (float)k;
#pragma unroll 8
    for (int i = 0; i < iters; i++)
#pragma unroll
        for (int k = 0; k < 8; k++) x[k] = __builtin_fmaf(a, b, x[k]);
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
}

int stream_blocks(int64_t work_items)
{
    const int64_t b = (work_items + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));   // grid-stride beyond 32 waves per CU
}

}  // namespace

AdamArgs adam_args(float lr, float beta1, float beta2, float eps, int step, float grad_scale)
{
    AdamArgs a;
    a.lr = lr; a.beta1 = beta1; a.beta2 = beta2; a.omb1 = (float)(1.0 - (double)beta1);
    a.omb2 = (float)(1.0 - (double)beta2); a.eps = eps; a.grad_scale = grad_scale;
    a.inv_bc1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    a.inv_bc2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    return a;
}

hipError_t launch_adam(hipStream_t st, float* p, float* g, float* m, float* v, int64_t count, float lr, float beta1,
                       float beta2, float eps, int step, float grad_scale, bool zero_grad)
{
    if (count <= 0) return hipSuccess;
    const AdamArgs a = adam_args(lr, beta1, beta2, eps, step, grad_scale);
    hipLaunchKernelGGL(k_adam, dim3(stream_blocks(count >> 2)), dim3(256), 0, st, p, g, m, v, count, a, zero_grad ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_grad_accumulate(hipStream_t st, float* acc, const float* g, int64_t count)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_grad_accumulate, dim3(stream_blocks(count >> 2)), dim3(256), 0, st, acc, g, count);
    return hipGetLastError();
}

hipError_t launch_activate(hipStream_t st, int64_t n, const float* raw_s, const float* raw_q, const float* raw_o,
                           float* s, float* q, float* o)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_activate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, raw_s,
                       reinterpret_cast<const float4*>(raw_q), raw_o, s, reinterpret_cast<float4*>(q), o);
    return hipGetLastError();
}

hipError_t launch_activate_bwd(hipStream_t st, int64_t n, const float* raw_s, const float* raw_q, const float* raw_o,
                               const float* d_s, const float* d_q, const float* d_o, float* d_raw_s, float* d_raw_q,
                               float* d_raw_o)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_activate_bwd, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, raw_s,
                       reinterpret_cast<const float4*>(raw_q), raw_o, d_s, reinterpret_cast<const float4*>(d_q), d_o,
                       d_raw_s, reinterpret_cast<float4*>(d_raw_q), d_raw_o);
    return hipGetLastError();
}

hipError_t launch_activate_inv(hipStream_t st, int64_t n, const float* s, const float* o, float lo, float hi,
                               float* raw_s, float* raw_o)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_activate_inv, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, s, o, lo, hi, raw_s, raw_o);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t st, const void* src, void* dst, int64_t bytes)
{
    const int64_t nvec = bytes / 16;
    if (nvec <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy, dim3(stream_blocks(nvec)), dim3(256), 0, st, static_cast<const float4*>(src),
                       static_cast<float4*>(dst), nvec);
    return hipGetLastError();
}

hipError_t launch_fma_chain(hipStream_t st, float* out, int blocks, int iters)
{
    hipLaunchKernelGGL(k_fma_chain, dim3(blocks), dim3(256), 0, st, out, iters, 0.999f, 0.001f);
    return hipGetLastError();
}

}  // namespace fs
