// Matrix-core path for three and four tokens of two-path layers: the structures shared by the host planner and the device
// kernels, and the layout of the expanded input.  The arithmetic is that of rb_mx.h: signs as fp4 +-1, h (.) x as four bf8 terms.
//
// The kernel for one token walks step lists, one sign tile at a time, and fetches the operand of every tile: with four tokens 8 KB for 1 KB
// of signs.  Here a wavefront takes the same columns of all its workgroup's row tiles, so that an operand tile is fetched once, and each
// path has a 16-column operand of its own (four tokens, four terms), so that no column of a matrix instruction is idle at four tokens.
#pragma once
#include <cstddef>
#include <cstdint>

#include "rabit.h"
#include "rb_mx.h"

namespace rb {
namespace flow {

using mx::align_up;
using mx::RESID_CALLER;
using mx::RESID_COPY;
using mx::RESID_NONE;
using mx::ROLE_GATE;
using mx::MAX_CONS;
using mx::MAX_EXPAND;
using mx::MAX_OPS;
using mx::MAX_T;

constexpr int K = 2;               // paths
// Eight wavefronts compute and finish rows, a ninth brings in the signs
constexpr int CWAVES = 8;
constexpr int THREADS = (CWAVES + 1) * 64;
constexpr int MAXSLOT = 8;         // row tiles one workgroup takes per stage; a wavefront finishes one of them
constexpr int GATED_SLOTS = MAXSLOT / 2;   // of a gate-times-up stage: gate in slots 0.., up in slots 4..
constexpr int MAX_STAGE_OPS = 8;   // ops of a stage
constexpr int T = 4;               // tokens of the operand layout (three tokens: the last one's columns are zero)

// The column tiles of an op are cut into one contiguous run per wavefront; a row's sum is over the tiles of a run, then over the
// runs in order, whatever workgroup it falls on and whatever else that workgroup does.
__host__ __device__ constexpr int run_begin(int wave, int CT) { return wave * CT / CWAVES; }
// column tiles whose operands a wavefront holds in registers, 32 registers each; of a longer run they are fetched for every row tile
constexpr int RESIDENT = 3;

// The loading wavefront counts the sign tiles it has asked for, the others the first tile that each of them still needs; the counts may wrap.
// Whether `more` tiles beyond the first `issued` fit a ring of `tiles`, with `used` the least of what is still needed.  Wavefronts that gave up a wait no
// longer wait for tiles to arrive: what they still need may lie ahead of what has been asked for, and there is room then.
__host__ __device__ constexpr bool ring_has_room(uint32_t issued, uint32_t more, uint32_t used, int tiles) { return (int32_t)(issued + more - used) <= tiles; }

// Expanded input ("right operand") of one op, stored as the register image the MFMA wants.
// The 8-bit right operand of v_mfma_scale_f32_16x16x128_f8f6f4 keeps, in lane col + 16 * q
// (col = operand column, q = 0..3), contraction indices 16q..16q+15 in its first four registers and
// 64+16q..64+16q+15 in the next four.  Contraction index == input column inside a 128-column block
// (see rb_layout.h).  Each path has an operand of its own, with column 4 * token + term.
//   [128-column block][half j of the contraction][q][path][4 * token + term][16 bytes]
// A 16-byte group is the 16 input columns one row tile of the producing op writes; all groups that a row tile
// writes, 512 bytes, lie side by side.
constexpr int UP_BLOCK_BYTES = 512 * K * T;

// byte offset of the 16-byte group of (input column block of 16 starting at j0, path, operand column c)
__host__ __device__ inline size_t up_group_offset(int j0, int path, int c)
{
    const int b = j0 >> 7, jj = j0 & 127, q = (jj & 63) >> 4, j = jj >> 6;
    return ((((size_t)b * 2 + j) * 4 + q) * K + path) * (size_t)(64 * T) + (size_t)c * 16;
}

struct alignas(64) Op {
    const uint32_t *bits;     // native sign tiles
    const uint16_t *g;        // fp16 [K][out]
    const uint16_t *h;        // fp16 [K][in]
    const uint16_t *x;        // fp16 [T][in]  input buffer (read by the expansion kernel only)
    uint16_t *y;              // fp16 [T][out] output buffer (null: a later op of the launch overwrites it)
    uint8_t *up;              // expanded input of this op (see up_group_offset)
    int out, in;
    int RT, CT;               // row tiles (16 rows), column tiles (256 columns)
    int dep;                  // op of this launch that writes x (-1: none)
    float sc[K];              // power-of-two input scale per path (max |h| * sc <= 1/2)
    float inv_sc[K];
    int n_cons;               // ops that read y inside this call
    int cons[MAX_CONS];
    // ---- the decoder block around the layer (all unused, zero, in a plain stack)
    const uint16_t *norm_w;   // fp16 [in]: the input is normalised (root mean square) and multiplied by this
    const float *ssq_in;      // [4][n_part]: per token, sums of squares of 16 input rows each
    float *ssq_out;           // [4][RT]: the same of this op's output, for readers that normalise it
    uint32_t *rcopy;          // [T][out]: the fp16 output once more, one word each, for an op that adds it later
    const void *resid;        // what is added to the result: fp16 [T][out] of the caller, the same put aside, or another op's rcopy
    const uint16_t *resid_src;   // the caller's buffer that is put aside (null: none)
    int resid_kind;           // RESID_*
    int n_part;
};
// The gate and the up projection of a feed-forward part run as two ops of a stage whose row tiles are dealt alike; the
// wavefront that finishes a row tile of the gate takes the same rows of the up projection from LDS:
// y = silu(gate) * up leaves through the gate op.

// Ops [op0, op0 + nops) are independent of each other.  Their row tiles, one op after the other, are dealt to the workgroups in
// contiguous, nearly equal shares (of a gate-times-up stage: the row tiles of either op, alike).
struct alignas(64) Stage {
    int op0, nops, tiles, gated;
    int rt[MAX_STAGE_OPS];    // row tiles of each op
    int norm;                 // the ops normalise their input, which is the same for all of them
    int n_slots;              // finishing slots a workgroup may use
    uint32_t rec0;            // index of the stage's first finishing record
};
static_assert(sizeof(Stage) == 64, "one scalar load");

// What a workgroup does in a stage, laid out flat (record stage * n_groups + workgroup) and read one stage ahead, so that nothing on the path from
// one stage to the next waits for a chain of dependent loads
struct alignas(64) Work {
    uint64_t bits[2];         // sign tiles of the first row tile of the share's first op and of its second
    uint32_t up[2];           // their expanded inputs, in units of 256 bytes from the first one of the plan
    uint16_t P[2], CT[2];     // row tiles (0: there is no such op), column tiles
    uint8_t slot1;            // finishing slot of the second op's first row tile
    uint8_t n_fin;            // row tiles to finish
    uint8_t flags;            // WORK_*
    uint8_t pad_;
    uint32_t rec;             // the share's first finishing record
    uint32_t ssq_in;          // sums of squares of the normalised input [4][n_part], in units of 256 bytes from the first expanded input
    float inv_n;              // 1 / in
    uint32_t n_part;
    uint32_t pad2_;
};
static_assert(sizeof(Work) == 64, "one scalar load");
constexpr int WORK_DEP0 = 1, WORK_DEP1 = 2, WORK_GATED = 4, WORK_NORM = 8;

// What the wavefront that finishes a row tile needs: record Work::rec + slot
struct alignas(32) SlotRec {
    uint64_t y;               // fp16 output: row 0 of token 0 (0: not stored)
    uint32_t up[MAX_CONS];    // per reading op: the 16-byte group of path 0, operand column 0 that these rows fill, in units of 16 bytes
    int out;                  // rows of the op
    uint8_t rows, n_cons, resid_kind, pad_;   // rows of the tile; ops that read its output
    uint32_t pad2_;
};
static_assert(sizeof(SlotRec) == 32, "one scalar load");
// More, read only by the form of the kernel that runs decoder blocks (offsets in bytes from the first expanded input; 0: none)
struct alignas(32) SlotExt {
    uint64_t resid;           // element (token 0, row 0 of the tile) of what is added to the result
    uint32_t ssq_out;         // this row tile's entry of the op's own sums of squares, in units of 4 bytes
    int ssq_stride;           // entries per token
    uint32_t rcopy;           // element (token 0, row 0) of the op's copy of its output, in units of 4 bytes
    uint32_t pad_[3];
};
static_assert(sizeof(SlotExt) == 32, "one scalar load");
// per row of a slot: g_k / sc_k of the op (its output scales over the input scaling it was fed with), then
// h_k * sc_k of each reading op (its input scales times its input scaling), [reader][path]
constexpr int VALS_ROW = K * (1 + MAX_CONS);
constexpr size_t VALS_RECORD_BYTES = (size_t)16 * VALS_ROW * sizeof(float);

// workspace: [Op x n_ops][Stage x n_stages][error u32, tiles waited for u32]
//            [indices of the ops whose input is expanded by a kernel of its own]
//            [Work x n_stages x n_groups][SlotRec x records][value records x the same][SlotExt x the same, decoder blocks][up arrays]
//            decoder blocks: [sums of squares and output copies of ops][sums of squares of inputs from outside]
struct Layout {
    size_t ops, stages, error, which, work, slots, vals, ext, up, aux, total;
    size_t aux_poison;        // bytes at the start of aux that every launch marks as not yet written
};

inline __host__ __device__ size_t up_bytes(int in)
{
    const int CB = (in + 255) / 256 * 2;           // whole column tiles: two blocks each
    return (size_t)CB * UP_BLOCK_BYTES;
}

// workgroup g's share [t0, t1) of N row tiles, of G workgroups: contiguous, and shares differ by one tile at most
__host__ __device__ inline void share_of(uint32_t N, uint32_t g, uint32_t G, uint32_t &t0, uint32_t &t1)
{
    if ((G & (G - 1)) == 0) {                 // the usual number of workgroups is a power of two
        const int shift = __builtin_ctz(G);
        t0 = (g * N) >> shift;
        t1 = ((g + 1) * N) >> shift;
        return;
    }
    t0 = g * N / G;
    t1 = (g + 1) * N / G;
}

}  // namespace flow
}  // namespace rb
