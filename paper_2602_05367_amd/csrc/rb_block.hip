// The decoder block around the residual-binary layers (the end-to-end decoding setting of
// Section 5.4 and the inference table: a Llama-2 block): entry points of the fused form, which
// runs on the persistent decode kernel, and the three operations as kernels of their own for
// callers that run a block op by op.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include "rabit.h"
#include "rb_internal.h"

namespace rb {
namespace {

// All three move 8 values (16 bytes) per thread and load; at the sizes of a prompt they are chains of one or two trips to memory, launch included
// (333 x 4096: normalisation, two bytes at a time and a tree of eight barriers 10.9 us, now 5.4; addition 5.1 and 5.3; 333 x 11008:
// silu(a) b 7.2 and 6.2).  Buffers need be aligned to 2 bytes only, and n is any number: the last piece of a vector goes element by element.
union Eight {
    uint4 q;
    __half h[8];
};
__device__ __forceinline__ Eight load_eight(const __half *p, size_t left)
{
    Eight v;
    if (left >= 8) {
        __builtin_memcpy(&v.q, p, 16);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v.h[e] = (size_t)e < left ? p[e] : __ushort_as_half(0);
    }
    return v;
}
__device__ __forceinline__ void store_eight(__half *p, size_t left, const Eight &v)
{
    if (left >= 8) {
        __builtin_memcpy(p, &v.q, 16);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if ((size_t)e < left) p[e] = v.h[e];
    }
}

// y = x / sqrt(mean_j x_j^2 + eps) (.) w, one workgroup per token, which keeps its row (up to 8192 values; the rest is read again); fp32
// arithmetic, fp16 in and out
constexpr int NORM_KEPT = 4;
__global__ __launch_bounds__(256) void rmsnorm_kernel(const __half *x, const __half *w, __half *y, int n, float eps)
{
    const __half *xr = x + (size_t)blockIdx.x * n;
    __half *yr = y + (size_t)blockIdx.x * n;
    const int first = 8 * (int)threadIdx.x;
    Eight kept[NORM_KEPT], weights[NORM_KEPT];
#pragma unroll
    for (int i = 0; i < NORM_KEPT; ++i)
        if (first + 2048 * i < n) kept[i] = load_eight(xr + first + 2048 * i, (size_t)(n - first - 2048 * i));
#pragma unroll
    for (int i = 0; i < NORM_KEPT; ++i)
        if (first + 2048 * i < n) weights[i] = load_eight(w + first + 2048 * i, (size_t)(n - first - 2048 * i));
    float sum = 0.f;
    auto add = [&](const Eight &v) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += __half2float(v.h[e]) * __half2float(v.h[e]);
    };
#pragma unroll
    for (int i = 0; i < NORM_KEPT; ++i)
        if (first + 2048 * i < n) add(kept[i]);
    for (long long j = first + 2048ll * NORM_KEPT; j < n; j += 2048) add(load_eight(xr + j, (size_t)(n - j)));
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    __shared__ float red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    const float rinv = rsqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)n + eps);
    auto write = [&](long long j, const Eight &v, const Eight &wv) {
        Eight o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o.h[e] = __float2half_rn(__half2float(v.h[e]) * rinv * __half2float(wv.h[e]));
        store_eight(yr + j, (size_t)(n - j), o);
    };
#pragma unroll
    for (int i = 0; i < NORM_KEPT; ++i)
        if (first + 2048 * i < n) write(first + 2048 * i, kept[i], weights[i]);
    for (long long j = first + 2048ll * NORM_KEPT; j < n; j += 2048) write(j, load_eight(xr + j, (size_t)(n - j)), load_eight(w + j, (size_t)(n - j)));
}

// y = silu(a) * b, elementwise
__global__ __launch_bounds__(256) void silu_mul_kernel(const __half *a, const __half *b, __half *y, size_t n)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    const Eight av = load_eight(a + i, n - i), bv = load_eight(b + i, n - i);
    Eight o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float g = __half2float(av.h[e]);
        o.h[e] = __float2half_rn(g / (1.f + __expf(-g)) * __half2float(bv.h[e]));
    }
    store_eight(y + i, n - i, o);
}

__global__ __launch_bounds__(256) void add_kernel(const __half *a, const __half *b, __half *y, size_t n)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= n) return;
    const Eight av = load_eight(a + i, n - i), bv = load_eight(b + i, n - i);
    Eight o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o.h[e] = __float2half_rn(__half2float(av.h[e]) + __half2float(bv.h[e]));
    store_eight(y + i, n - i, o);
}

int check_block(const rb_layer *layers, int n_layers, const uint16_t *const *norm_weights, int n_norms, float eps,
                const rb_block_op *ops, int n_ops, uint16_t *const *bufs, int n_bufs, int T, void *workspace,
                size_t workspace_bytes)
{
    if (!layers || !ops || !bufs || (n_norms > 0 && !norm_weights)) return RB_ERR_NULL;
    if (n_layers < 1 || n_ops < 1 || n_bufs < 1 || n_norms < 0 || T < 1 || !(eps >= 0.f)) return RB_ERR_SHAPE;
    for (int l = 0; l < n_layers; ++l) {
        const int rc = check_layer(&layers[l]);
        if (rc != RB_OK) return rc;
    }
    for (int i = 0; i < n_norms; ++i) {
        if (!norm_weights[i]) return RB_ERR_NULL;
        if ((uintptr_t)norm_weights[i] & 1) return RB_ERR_ALIGN;
    }
    for (int n = 0; n < n_ops; ++n) {
        const rb_block_op &op = ops[n];
        if (op.layer < 0 || op.layer >= n_layers || op.src < 0 || op.src >= n_bufs || op.dst < 0 || op.dst >= n_bufs ||
            op.src == op.dst || op.norm < -1 || op.norm >= n_norms)
            return RB_ERR_SHAPE;
        if (!bufs[op.src] || !bufs[op.dst]) return RB_ERR_NULL;
        if (((uintptr_t)bufs[op.src] | (uintptr_t)bufs[op.dst]) & 15) return RB_ERR_ALIGN;
        if (op.epilogue == RB_EPI_ADD) {
            if (op.aux < 0 || op.aux >= n_bufs || op.aux == op.src) return RB_ERR_SHAPE;
            if (!bufs[op.aux]) return RB_ERR_NULL;
            if ((uintptr_t)bufs[op.aux] & 15) return RB_ERR_ALIGN;
        } else if (op.epilogue == RB_EPI_SILU_MUL) {
            if (op.aux < 0 || op.aux >= n_layers) return RB_ERR_SHAPE;
            const rb_layer &a = layers[op.layer], &b = layers[op.aux];
            if (a.out != b.out || a.in != b.in || a.K != b.K) return RB_ERR_SHAPE;
        } else if (op.epilogue != RB_EPI_NONE) {
            return RB_ERR_SHAPE;
        }
    }
    if (workspace_bytes < mx::block_workspace_bytes(layers, n_layers, n_ops, T) || !workspace) return RB_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15) return RB_ERR_ALIGN;
    return RB_OK;
}

}  // namespace
}  // namespace rb

extern "C" size_t rb_block_workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int T)
{
    if (!layers || n_layers < 1 || n_ops < 1 || T < 1) return 0;
    return rb::mx::block_workspace_bytes(layers, n_layers, n_ops, T);
}

extern "C" int rb_block_prepare(const rb_layer *layers, int n_layers, const uint16_t *const *norm_weights, int n_norms,
                                float eps, const rb_block_op *ops, int n_ops, uint16_t *const *bufs, int n_bufs, int T,
                                void *workspace, size_t workspace_bytes, void *stream)
{
    const int rc = rb::check_block(layers, n_layers, norm_weights, n_norms, eps, ops, n_ops, bufs, n_bufs, T, workspace,
                                   workspace_bytes);
    if (rc != RB_OK) return rc;
    rb_stack_forget(workspace);
    return rb::mx::prepare_block(layers, norm_weights, eps, ops, n_ops, bufs, T, workspace, workspace_bytes,
                                 static_cast<hipStream_t>(stream));
}

extern "C" int rb_rmsnorm(const uint16_t *x, const uint16_t *w, uint16_t *y, int T, int n, float eps, void *stream)
{
    if (!x || !w || !y) return RB_ERR_NULL;
    if (T < 1 || T > 65535 || n < 1 || !(eps >= 0.f)) return RB_ERR_SHAPE;
    hipLaunchKernelGGL(rb::rmsnorm_kernel, dim3(T), dim3(256), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<const __half *>(x), reinterpret_cast<const __half *>(w),
                       reinterpret_cast<__half *>(y), n, eps);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

extern "C" int rb_silu_mul(const uint16_t *gate, const uint16_t *up, uint16_t *y, size_t n, void *stream)
{
    if (!gate || !up || !y) return RB_ERR_NULL;
    if (n < 1 || n > ((size_t)1 << 38)) return RB_ERR_SHAPE;
    hipLaunchKernelGGL(rb::silu_mul_kernel, dim3((unsigned)((n + 2047) / 2048)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<const __half *>(gate), reinterpret_cast<const __half *>(up),
                       reinterpret_cast<__half *>(y), n);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}

extern "C" int rb_add(const uint16_t *a, const uint16_t *b, uint16_t *y, size_t n, void *stream)
{
    if (!a || !b || !y) return RB_ERR_NULL;
    if (n < 1 || n > ((size_t)1 << 38)) return RB_ERR_SHAPE;
    hipLaunchKernelGGL(rb::add_kernel, dim3((unsigned)((n + 2047) / 2048)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       reinterpret_cast<const __half *>(a), reinterpret_cast<const __half *>(b),
                       reinterpret_cast<__half *>(y), n);
    return hipGetLastError() == hipSuccess ? RB_OK : RB_ERR_HIP;
}
