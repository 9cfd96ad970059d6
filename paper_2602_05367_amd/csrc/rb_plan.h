// How the ops of a plan hang together, for both persistent decode kernels (host only): who writes what an op reads and adds, and where a
// launch, which has no barriers between ops, needs more than that to give what the ops give one after the other.
#pragma once
#include <vector>

#include "rabit.h"
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
