// Kernel selection for one layer and for a stack of layers.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rabit.h"
#include "rb_internal.h"

namespace rb {

thread_local int g_last_path = RB_PATH_NONE;
void set_last_path(int path) { g_last_path = path; }

constexpr int FUSED_MAX_T = 4;         // tokens of the fused decode kernel

// Which stacks take the few-token kernel: every stack with a three-path layer, and two-path stacks
// of more tokens than the fused decode kernels take.  (7B-shaped dependent chain at three and four tokens: one launch of the persistent
// kernel 0.90 to 0.94 ms, 128 of the few-token kernel 1.09 to 1.11.  At five tokens two passes of the former would take 1.6 ms, the latter 1.11.)
bool batch_applies(const rb_layer *layers, int n_layers, int T)
{
    bool any_three = false, all_three = true;
    for (int l = 0; l < n_layers; ++l) {
        if (!batch::layer_supported(&layers[l], T)) return false;
        any_three = any_three || layers[l].K == 3;
        all_three = all_three && layers[l].K == 3;
    }
    if (all_three && T == 1) return false;       // one token, three paths throughout: the fused decode kernel
    return any_three || T > FUSED_MAX_T;
}

// Which single calls take the few-token kernel (one launch): three paths, and two paths beyond two tokens and whatever
// element types the decode kernels do not take (one and two fp16 tokens with fp16 results stay there: the bits are those of
// a stack).  Three paths at up to five tokens took the generic kernel once, which reads the weights for every token (us in a graph, there
// and here: 4096 x 4096 at one token 10.9 and 5.2, at three 17.0 and 5.2, 4096 x 11008 at one 32.1 and 9.2, 28672 x 8192 at three 168 and 31).
// They still ask for no scratch memory (so their output must not overlap their input) and report what they have always reported.
constexpr int K3_ROOM_MIN_T = 6, K3_BATCH_MAX_T = 12;
bool single_few_applies(const rb_layer *L, int T, int act_dtype, int out_dtype)
{
    if (!batch::call_sized(L, T)) return false;
    return L->K == 3 || T > 2 || act_dtype != RB_F16 || out_dtype != RB_F16;
}
// an output over its input is provided for
bool single_few_has_room(const rb_layer *L, int T) { return T >= (L->K == 3 ? K3_ROOM_MIN_T : 3); }
// the kernel family a few-token call is reported as (rb_last_path): the families these calls have always been
// reported as; the kernel is the same
int single_few_path(const rb_layer *L, int T, int act_dtype, int out_dtype)
{
    if (L->K == 3 && T < K3_ROOM_MIN_T) return RB_PATH_SIGNADD;
    return L->K == 3 && T <= K3_BATCH_MAX_T && act_dtype == RB_F16 && out_dtype == RB_F16 ? RB_PATH_BATCH : RB_PATH_GEMM;
}
bool single_gemm_applies(const rb_layer *L, int T)
{
    return T > batch::CALL_MAX_T && gemm::supported(L, T);
}

// Few rows and tokens leave most compute units without a tile of the many-token kernel: there 64 tokens per workgroup on the few-token
// kernel are faster (us, many-token and few-token kernel: 2048 x 2048 at 128 tokens 11.5 and 7.7, 4096 x 11008 at 128 41 and 33, 512 x 8192 at 512 31 and
// 20; on the other side of the line 300 x 2048 at 2000 12.4 and 16.5, 300 x 28672 at 2000 101 and 123).  The estimates are those of earlier forms of
// both kernels, which have become faster alike: of 40 layers near the line 38 went to the faster one within 1.2 %, two to one that took a quarter more (1020 x 352 at 573
// tokens 7.2 and 8.8, 5465 x 288 at 125 7.1 and 9.0); with 1.7 us less for the many-token kernel three of sixty were 4 to 10 % slower, one 2 % faster
int launch_many(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (batch::blocks_cost(L, T, act_dtype) < gemm::cost(L, T)) return batch::launch_call(L, X, Y, T, act_dtype, out_dtype, workspace, workspace_bytes, stream);
    return gemm::launch(L, X, Y, T, act_dtype, out_dtype, workspace, stream);
}

__global__ __launch_bounds__(256) static void copy_kernel(const uint4 *__restrict__ from, uint4 *__restrict__ to, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) to[i] = from[i];
}
void copy_aside(const void *X, void *to, size_t bytes, hipStream_t stream)
{
    const size_t n = bytes / 16;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)std::min<size_t>(1024, (n + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const uint4 *>(X), static_cast<uint4 *>(to), n);
}

// scratch memory of one call on this layer, whatever its element types
static size_t call_bytes(const rb_layer *L, int T)
{
    if (single_gemm_applies(L, T)) return gemm::workspace_bytes(L, T);
    return single_few_has_room(L, T) && single_few_applies(L, T, RB_F16, RB_F16) ? aside_bytes(L, T) : 0;
}

size_t workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int T)
{
    // one layer, one token: the single-call kernel keeps everything in LDS
    if (n_layers == 1 && n_ops == 1 && T == 1 && gemv1::supported(&layers[0], 1)) return 0;
    if (batch_applies(layers, n_layers, T) && n_ops > 1) return batch::plan_workspace_bytes(layers, n_layers, T);
    // a single call, or ops that run one after the other on the caller's stream and share its scratch
    size_t need = T > FUSED_MAX_T ? 0 : mx::plan_workspace_bytes(layers, n_layers, n_ops, T);
    for (int l = 0; l < n_layers; ++l) need = std::max(need, call_bytes(&layers[l], T));
    return need;
}

int dispatch_linear(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype,
                    void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (act_dtype == RB_F16 && out_dtype == RB_F16 && gemv1::supported(L, T)) {
        g_last_path = RB_PATH_MX;
        return gemv1::launch(L, X, Y, stream);
    }
    if (act_dtype == RB_F16 && out_dtype == RB_F16 && L->K == 2 && T <= 2 && mx::layer_supported(L, T) && workspace &&
        workspace_bytes >= mx::plan_workspace_bytes(L, 1, 1, T)) {
        const rb_stack_op op{0, 0, 1};
        uint16_t *bufs[2] = {static_cast<uint16_t *>(const_cast<void *>(X)), static_cast<uint16_t *>(Y)};
        batch::forget_plan(workspace);
        const int rc = mx::run_plan(L, &op, 1, bufs, T, workspace, workspace_bytes, stream);
        if (rc != RB_ERR_UNSUPPORTED) { g_last_path = RB_PATH_MX; return rc; }
    }
    if (single_few_applies(L, T, act_dtype, out_dtype)) {
        g_last_path = single_few_path(L, T, act_dtype, out_dtype);
        return batch::launch_call(L, X, Y, T, act_dtype, out_dtype, workspace, workspace_bytes, stream);
    }
    if (single_gemm_applies(L, T) && workspace && workspace_bytes >= gemm::workspace_bytes(L, T)) {
        g_last_path = RB_PATH_GEMM;
        return launch_many(L, X, Y, T, act_dtype, out_dtype, workspace, workspace_bytes, stream);
    }
    g_last_path = RB_PATH_SIGNADD;
    return launch_signadd(L, X, Y, T, act_dtype, out_dtype, stream);
}

int dispatch_stack(const rb_layer *layers, int n_layers, const rb_stack_op *ops, int n_ops,
                   uint16_t *const *bufs, int n_bufs, int T, void *workspace, size_t workspace_bytes, hipStream_t stream)
{
    if (n_ops > 1 && batch_applies(layers, n_layers, T)) {
        int rc = batch::prepare_plan(layers, ops, n_ops, bufs, T, workspace, workspace_bytes);
        if (rc == RB_OK) rc = batch::launch_plan(workspace, workspace_bytes, stream);
        if (rc == RB_OK) g_last_path = RB_PATH_BATCH;
        if (rc != RB_ERR_UNSUPPORTED && rc != RB_ERR_WORKSPACE) return rc;
    }
    bool fused = workspace && workspace_bytes >= mx::plan_workspace_bytes(layers, n_layers, n_ops, T);
    for (int n = 0; n < n_ops && fused; ++n) fused = mx::layer_supported(&layers[ops[n].layer], T);
    if (fused) {
        batch::forget_plan(workspace);
        const int rc = mx::run_plan(layers, ops, n_ops, bufs, T, workspace, workspace_bytes, stream);
        if (rc != RB_ERR_UNSUPPORTED) { g_last_path = RB_PATH_MX; return rc; }
    }
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer *L = &layers[ops[n].layer];
        const int rc = dispatch_linear(L, bufs[ops[n].src], bufs[ops[n].dst], T, RB_F16, RB_F16, workspace,
                                       workspace_bytes, stream);
        if (rc != RB_OK) return rc;
    }
    return RB_OK;
}

}  // namespace rb

extern "C" int rb_last_path(void) { return rb::g_last_path; }
