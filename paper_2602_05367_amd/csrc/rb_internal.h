// Declarations shared between the entry points and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>

#include "rabit.h"

namespace rb {

int check_layer(const rb_layer *L);
void set_last_path(int path);

// generic sign-XOR + add kernel, any supported shape, T via grid.y
int launch_signadd(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype,
                   hipStream_t stream);

size_t workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int T);
// stacks that run on the few-token kernel (see rb_dispatch.hip)
bool batch_applies(const rb_layer *layers, int n_layers, int T);
// a single call takes the few-token kernel; of T tokens on this layer, the many-token kernel (given
// the scratch memory it needs)
bool single_few_applies(const rb_layer *L, int T, int act_dtype, int out_dtype);
bool single_few_has_room(const rb_layer *L, int T);      // a call that asks for scratch memory, where the output overlaps the input
int single_few_path(const rb_layer *L, int T, int act_dtype, int out_dtype);
bool single_gemm_applies(const rb_layer *L, int T);

// a call of more than 64 tokens, given gemm::workspace_bytes: the many-token kernel, or the few-token kernel 64 tokens at a time
int launch_many(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace, size_t workspace_bytes, hipStream_t stream);

int dispatch_linear(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype,
                    void *workspace, size_t workspace_bytes, hipStream_t stream);

int dispatch_stack(const rb_layer *layers, int n_layers, const rb_stack_op *ops, int n_ops,
                   uint16_t *const *bufs, int n_bufs, int T, void *workspace, size_t workspace_bytes,
                   hipStream_t stream);

// An output that overlaps its input: workgroups of the matrix-core kernels store rows of Y while others
// still read X, so the input is moved to scratch memory first (in % 32 == 0: whole 16-byte pieces)
inline bool overlap(const void *a, size_t na, const void *b, size_t nb)
{
    return (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}
inline size_t input_bytes(const rb_layer *L, int T) { return (size_t)T * L->in * 2; }
inline size_t output_bytes(const rb_layer *L, int T, int out_dtype) { return (size_t)T * L->out * (out_dtype == RB_F32 ? 4 : 2); }
inline size_t aside_bytes(const rb_layer *L, int T) { return (input_bytes(L, T) + 255) / 256 * 256; }
void copy_aside(const void *X, void *to, size_t bytes, hipStream_t stream);

namespace gemm {
// many-token matrix-core GEMM (K = 2 or 3): workspace holds the input when the output overlaps it
bool supported(const rb_layer *L, int T);
size_t workspace_bytes(const rb_layer *L, int T);
float cost(const rb_layer *L, int T);      // microseconds a call takes, by the rule that picks the workgroup's shape
int launch(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace,
           hipStream_t stream);
}  // namespace gemm

namespace gemv1 {
// one layer, one token, one launch, nothing prepared (K = 2; the expanded input must fit in LDS);
// same bits as the op would give inside a stack
bool supported(const rb_layer *L, int T);
int launch(const rb_layer *L, const void *x, void *y, hipStream_t stream);
}  // namespace gemv1

namespace batch {
// few-token path (K = 2 or 3): the weights are read once for all tokens; independent ops of a
// stack share a launch, dependent ones are ordered by the stream.  Single calls of any element type
// take up to CALL_MAX_T tokens, stacks up to 16.
constexpr int CALL_MAX_T = 64;
bool call_sized(const rb_layer *L, int T);
float blocks_cost(const rb_layer *L, int T, int act_dtype);      // of more tokens, 64 per workgroup; infinite where that is never the faster way
// workspace: aside_bytes(L, T) where single_few_has_room, used when Y overlaps X
int launch_call(const rb_layer *L, const void *X, void *Y, int T, int act_dtype, int out_dtype, void *workspace,
                size_t workspace_bytes, hipStream_t stream);
bool layer_supported(const rb_layer *L, int T);
size_t plan_workspace_bytes(const rb_layer *layers, int n_layers, int T);
int prepare_plan(const rb_layer *layers, const rb_stack_op *ops, int n_ops, uint16_t *const *bufs, int T,
                 void *workspace, size_t workspace_bytes);
int launch_plan(void *workspace, size_t workspace_bytes, hipStream_t stream);      // RB_ERR_UNSUPPORTED: no plan of this kind
bool has_plan(const void *workspace);
void forget_plan(const void *workspace);
}  // namespace batch

namespace mx {
struct PlanOp;
struct OpLinks;
}  // namespace mx

namespace flow {
// the persistent kernel for three and four tokens of two-path layers; its plans are prepared, run, checked and forgotten through namespace mx
size_t plan_workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int tokens, bool block);
int prepare(const rb_layer *layers, const mx::PlanOp *sops, const mx::OpLinks *links, int n_ops, uint16_t *const *bufs, const uint16_t *const *norm_w, float eps, bool block,
            int tokens, void *workspace, size_t workspace_bytes, hipStream_t stream);
int launch(void *workspace, size_t workspace_bytes, int pause, hipStream_t stream);      // RB_ERR_UNSUPPORTED: no plan of this kind
const void *marks(const void *workspace);
void forget(const void *workspace);
}  // namespace flow

namespace mx {
// workgroups of the decode kernels: one per compute unit of the current device (0: no device)
int device_groups();
// matrix-core path (K = 2 and T <= 4, or K = 3 and T = 1): whole op lists run as one persistent kernel
bool layer_supported(const rb_layer *L, int T);
size_t plan_workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int T);
int run_plan(const rb_layer *layers, const rb_stack_op *ops, int n_ops, uint16_t *const *bufs, int T,
             void *workspace, size_t workspace_bytes, hipStream_t stream);
// the two halves of run_plan: set-up that depends only on the frozen layers and the buffer
// addresses, and the per-token launch
int prepare_plan(const rb_layer *layers, const rb_stack_op *ops, int n_ops, uint16_t *const *bufs, int T,
                 void *workspace, size_t workspace_bytes, hipStream_t stream);
int launch_plan(void *workspace, size_t workspace_bytes, hipStream_t stream);
void forget_plan(const void *workspace);
// decoder blocks (norms, gate times up, residual additions in the kernel's finishing step); run,
// checked and forgotten like any other plan of this kernel
size_t block_workspace_bytes(const rb_layer *layers, int n_layers, int n_ops, int T);
int prepare_block(const rb_layer *layers, const uint16_t *const *norm_w, float eps, const rb_block_op *ops, int n_ops,
                  uint16_t *const *bufs, int T, void *workspace, size_t workspace_bytes, hipStream_t stream);
// waits for the stream; RB_ERR_HANDOVER if a run of this plan gave up a wait, RB_ERR_WORKSPACE: no plan
// waited (optional): += input tiles that compute wavefronts found not yet written and waited for, since the plan was made
int plan_status(const void *workspace, hipStream_t stream, unsigned long long *waited = nullptr, int *reason = nullptr);
// pause between a workgroup's last stores of a stage and the moment its compute wavefronts ask for
// that stage's outputs, in clocks (< 0: the built-in timing); launches made afterwards use it
void set_pause(int clks);
}  // namespace mx

}  // namespace rb
