// How the ops of a plan hang together, for both persistent decode kernels (host only): who writes what an op reads and adds, and where a
// launch, which has no barriers between ops, needs more than that to give what the ops give one after the other; and which of the two takes a plan.
#pragma once
#include <algorithm>
#include <vector>

#include "rabit.h"
#include "rb_layout.h"
#include "rb_mx.h"

namespace rb {
namespace mx {

// one op of a plan: a layer between two buffers and, in a decoder block, what surrounds it
struct PlanOp {
    int layer, src, dst;      // dst < 0: the result leaves through another op (ROLE_UP)
    int norm;                 // >= 0: which weight vector normalises the input
    int add;                  // >= 0: the buffer added to the result
    int role;
};

// Three and four tokens of two-path layers: which plans take the kernel of rb_flow.hip, which keep the step lists.  The former fetches the operand of a
// column once for all row tiles of a workgroup, so it pays where an op has much to do.  Lines by the mean weights of the plan's ops (by the widest, a head of
// 32000 rows made the eight narrow blocks before it 9 % slower).  us on the step lists and there, three tokens (d x f, number):
//   chains: 512 x 1376 4 63.7 and 65.6, 1024 x 2048 8 127.6 and 129.0, 1024 x 4096 8 141.0 and 137.2; from the line on 1088 x 4352 1 26.0 and 23.2, 1216 x 3328
//   20 425 and 333, 1344 x 2688 1 26.0 and 22.6, 1600 x 4800 8 196 and 159, 2048 x 8192 1 32.2 and 28.4, 4096 x 11008 32 1235 and 921; one op of 1600 x 1600
//   11.6 and 10.7;
//   decoder blocks: 1024 x 2048 8 151 and 165, 1600 x 4800 8 216 and 213, 2048 x 5504 8 214 and 201, 2048 x 6144 8 201 and 210, 2048 x 7168 3 87.2 and 90.6; from
//   the line on 2496 x 4992 4 125 and 116, 2112 x 7360 2 69.9 and 66.3, 3072 x 6144 8 252 and 218, 4096 x 11008 32 1305 and 1032.
// Decoder blocks whose layers mostly leave half of the workgroups without a row tile save little in a stage, in the first five blocks nothing:
// 2048 x 8192 2, 3, 4, 6, 16 61.0 and 61.9, 88.0 and 90.6, 115 and 119, 168 and 168, 433 and 414.
// Of rows of more than RESIDENT_COLS columns a wavefront there does not hold the operands: they are fetched for every row tile, and where a workgroup has more
// than three of those, nothing is saved: 14336 x 8192 25.7 and 26.6, 32768 x 8192 38.5 and 43.6, 32768 x 12288 53.1 and 56.7 (12288 x 12288 28.7 and 28.7;
// 32768 x 6144 32.3 and 22.1).  In two blocks of 8192 x 28672, where they are half of the weights, 279 and 278.
constexpr size_t FLOW_CHAIN_WEIGHTS = 2500000, FLOW_BLOCK_WEIGHTS = 8800000;
constexpr int RESIDENT_COLS = 24 * 256, FLOW_NARROW_BLOCK_OPS = 40;
inline size_t weights_of(const rb_layer &L) { return (size_t)L.out * L.in; }
inline size_t flow_weights(bool block) { return block ? FLOW_BLOCK_WEIGHTS : FLOW_CHAIN_WEIGHTS; }
inline bool takes_flow(const rb_layer *layers, const PlanOp *ops, int n_ops, int tokens, bool block, int groups)
{
    size_t all = 0, beyond = 0;
    int narrow = 0;
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer &L = layers[ops[n].layer];
        all += weights_of(L);
        if (L.in > RESIDENT_COLS && row_tiles(L.out) > 3 * groups) beyond += weights_of(L);
        narrow += 2 * row_tiles(L.out) <= groups;
    }
    if (block && 2 * narrow > n_ops && n_ops < FLOW_NARROW_BLOCK_OPS) return false;
    return tokens > 2 && all >= flow_weights(block) * (size_t)n_ops && 2 * beyond <= all;
}

// Per op of a decoder block, at most: sums of squares of its output and of an input from outside, and the copy of its output that a later op adds.  (What is put
// aside of the caller's is 2 bytes where the copy is 4: a plan is sized for two ops for each of the caller's, and only one of the two adds)
inline size_t block_aux_bound(const rb_layer *layers, int n_layers, int tokens)
{
    size_t most = 0;
    for (int l = 0; l < n_layers; ++l)
        most = std::max(most, align_up((size_t)row_tiles(layers[l].out) * 16, 256) + align_up((size_t)tokens * layers[l].out * 4, 256) +
                                  align_up((size_t)((layers[l].in + 15) / 16) * 16, 256));
    return most;
}

struct OpLinks {
    int producer = -1;        // op that writes the input: the last earlier one that writes that buffer (-1: the caller)
    int addend = -1;          // op whose result is added (-1: nothing is, or what the caller's buffer held before the launch)
    int n_cons = 0, cons[MAX_CONS] = {};   // ops that read the result
    bool squares = false;     // an op that normalises its input reads the result
    bool copied = false;      // a later op adds the result
    bool stores = true;       // no later op writes the same buffer: what the caller finds there is this one's
    bool aside = false;       // what the caller's buffer held is added, and an op that need not come after this one writes that buffer
};

// Workgroups go from op to op as the inputs of each arrive, so a later op that neither reads nor adds, on whatever way, what op n gives
// may store its rows before op n has looked at the caller's buffer
inline bool adds_before_anyone_stores(const PlanOp *ops, const std::vector<OpLinks> &links, int n_ops, int n)
{
    std::vector<bool> after((size_t)n_ops, false);
    after[(size_t)n] = true;
    for (int m = n + 1; m < n_ops; ++m) {
        const OpLinks &l = links[(size_t)m];
        after[(size_t)m] = (l.producer >= 0 && after[(size_t)l.producer]) || (l.addend >= 0 && after[(size_t)l.addend]);
        if (ops[m].dst == ops[n].add && !after[(size_t)m]) return false;
    }
    return true;
}

inline int link_ops(const rb_layer *layers, const PlanOp *ops, int n_ops, std::vector<OpLinks> &links)
{
    links.assign((size_t)n_ops, OpLinks{});
    size_t from_outside = 0;
    for (int n = 0; n < n_ops; ++n) {
        const rb_layer &L = layers[ops[n].layer];
        OpLinks &l = links[(size_t)n];
        auto last_writer = [&](int buf) {
            int m = n - 1;
            while (m >= 0 && ops[m].dst != buf) --m;
            return m;
        };
        l.producer = last_writer(ops[n].src);
        if (ops[n].norm >= 0 && l.producer >= 0) links[(size_t)l.producer].squares = true;
        if (ops[n].add >= 0) {
            l.addend = last_writer(ops[n].add);
            if (l.addend >= 0) {
                if (layers[ops[l.addend].layer].out != L.out) return RB_ERR_SHAPE;
                links[(size_t)l.addend].copied = true;
            }
        }
        if (l.producer < 0) {
            ++from_outside;
        } else {
            OpLinks &p = links[(size_t)l.producer];
            if (p.n_cons >= MAX_CONS) return RB_ERR_UNSUPPORTED;
            if (layers[ops[l.producer].layer].out != L.in) return RB_ERR_SHAPE;
            p.cons[p.n_cons++] = n;
        }
    }
    if (from_outside > MAX_EXPAND || n_ops > MAX_OPS) return RB_ERR_UNSUPPORTED;
    // Readers inside the launch take what they read and add from the expanded inputs and copies of its writer, so only the last writer of a
    // buffer needs to store it; the stores of two, from compute units whose caches are not coherent, could land in either order
    for (int n = 0; n < n_ops; ++n)
        for (int m = n + 1; m < n_ops && links[(size_t)n].stores; ++m) links[(size_t)n].stores = ops[n].dst < 0 || ops[m].dst != ops[n].dst;
    for (int n = 0; n < n_ops; ++n)
        if (ops[n].add >= 0 && links[(size_t)n].addend < 0) links[(size_t)n].aside = !adds_before_anyone_stores(ops, links, n_ops, n);
    return RB_OK;
}

}  // namespace mx
}  // namespace rb
