// How the ops of a plan hang together (csrc/rb_plan.h), on lists drawn at random: what the planner says against the definition,
// worked out another way.  Built and run by tests/test_sanitizers.py.
#include <cstdio>
#include <random>
#include <vector>

#include "rb_plan.h"

using namespace rb::mx;

static int fail(const char *what, int trial, int n)
{
    std::printf("trial %d, op %d: %s\n", trial, n, what);
    return 1;
}

// Which plans of three and four tokens take the kernel of rb_flow.hip, on 256 compute units
static int which_kernel()
{
    struct Shape { int out, in; };
    auto takes = [](const std::vector<Shape> &shapes, int tokens, bool block) {
        std::vector<rb_layer> layers;
        std::vector<PlanOp> ops;
        for (const Shape &s : shapes) {
            layers.push_back(rb_layer{s.out, s.in, 2, nullptr, nullptr, nullptr});
            ops.push_back(PlanOp{(int)ops.size(), 0, 1, -1, -1, ROLE_PLAIN});
        }
        return takes_flow(layers.data(), ops.data(), (int)ops.size(), tokens, block, 256);
    };
    auto blocks = [](int d, int f, int n, int head) {
        std::vector<Shape> s;
        for (int i = 0; i < n; ++i)
            for (Shape o : {Shape{d, d}, {d, d}, {d, d}, {d, d}, {f, d}, {f, d}, {d, f}}) s.push_back(o);
        if (head) s.push_back(Shape{head, d});
        return s;
    };
    struct { std::vector<Shape> shapes; bool block, flow; } const cases[] = {
        {blocks(4096, 11008, 32, 0), true, true},  {blocks(4096, 11008, 1, 0), false, true}, {blocks(1024, 2048, 8, 0), false, false},
        {blocks(1216, 3328, 20, 0), false, true},  {blocks(2048, 7168, 3, 0), true, false},  {blocks(2496, 4992, 4, 0), true, true},
        {blocks(2048, 8192, 3, 0), true, false},   {blocks(2048, 8192, 16, 0), true, true},
        // narrow layers before a head, which alone is wide
        {blocks(1024, 2048, 8, 32000), true, false}, {blocks(512, 2048, 16, 32000), false, false}, {blocks(2560, 6592, 4, 32000), true, true},
        // long rows, many of them
        {{{28672, 8192}}, false, false}, {{{32768, 6144}}, false, true}, {{{8192, 28672}}, false, true}, {blocks(8192, 28672, 1, 0), false, true},
        // either side of a line, by one row of the smaller layer
        {{{2500, 1024}, {2383, 1024}}, false, true}, {{{2500, 1024}, {2382, 1024}}, false, false},
    };
    int i = 0;
    for (const auto &c : cases) {
        for (int tokens = 1; tokens <= 4; ++tokens)
            if (takes(c.shapes, tokens, c.block) != (c.flow && tokens > 2)) return fail("the wrong kernel", i, tokens);
        ++i;
    }
    return 0;
}

int main()
{
    if (which_kernel()) return 1;
    std::mt19937 rng(3);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    int asides = 0, in_order = 0;
    for (int trial = 0; trial < 4000; ++trial) {
        rb_layer layer{};
        layer.out = layer.in = 64;
        layer.K = 2;
        const int n_ops = pick(1, 12), n_bufs = pick(2, 9);
        std::vector<PlanOp> ops;
        for (int n = 0; n < n_ops; ++n) {
            const int src = pick(0, n_bufs - 1);
            int dst = pick(0, n_bufs - 1), add = pick(0, 2) ? -1 : pick(0, n_bufs - 1);
            while (dst == src) dst = pick(0, n_bufs - 1);
            if (add == src) add = -1;
            ops.push_back(PlanOp{0, src, dst, pick(0, 1) - 1, add, ROLE_PLAIN});
        }
        // run one after the other, noting who wrote what each op reads
        std::vector<int> writer(n_bufs, -1), producer(n_ops), addend(n_ops), readers(n_ops, 0);
        bool too_many = false;
        for (int n = 0; n < n_ops; ++n) {
            producer[n] = writer[ops[n].src];
            addend[n] = ops[n].add < 0 ? -1 : writer[ops[n].add];
            if (producer[n] >= 0 && ++readers[producer[n]] > MAX_CONS) too_many = true;
            writer[ops[n].dst] = n;
        }
        std::vector<OpLinks> links;
        const int rc = link_ops(&layer, ops.data(), n_ops, links);
        if ((rc == RB_ERR_UNSUPPORTED) != too_many || (rc != RB_OK && rc != RB_ERR_UNSUPPORTED)) return fail("status", trial, rc);
        if (rc != RB_OK) continue;
        // which ops must come after which: paths over what is read and added
        std::vector<std::vector<bool>> before(n_ops, std::vector<bool>(n_ops, false));
        for (int n = 0; n < n_ops; ++n)
            for (int from : {producer[n], addend[n]})
                if (from >= 0) before[from][n] = true;
        for (int k = 0; k < n_ops; ++k)
            for (int i = 0; i < n_ops; ++i)
                for (int j = 0; j < n_ops; ++j)
                    if (before[i][k] && before[k][j]) before[i][j] = true;
        for (int n = 0; n < n_ops; ++n) {
            const OpLinks &l = links[n];
            if (l.producer != producer[n] || l.addend != addend[n] || l.n_cons != readers[n]) return fail("producer, addend or readers", trial, n);
            for (int c = 0; c < l.n_cons; ++c)
                if (producer[l.cons[c]] != n) return fail("a reader", trial, n);
            bool squares = false, copied = false, aside = false, stored_over = false, last = true;
            for (int m = 0; m < n_ops; ++m) {
                squares = squares || (producer[m] == n && ops[m].norm >= 0);
                copied = copied || addend[m] == n;
                last = last && !(m > n && ops[m].dst == ops[n].dst);
                if (m == n || ops[n].add < 0 || addend[n] >= 0 || ops[m].dst != ops[n].add) continue;
                stored_over = true;
                aside = aside || !before[n][m];
            }
            if (l.squares != squares || l.copied != copied) return fail("squares or copy", trial, n);
            if (l.stores != last) return fail("stores", trial, n);
            if (l.aside != aside) return fail("aside", trial, n);
            asides += aside;
            in_order += stored_over && !aside;
        }
    }
    if (asides < 100 || in_order < 100) return fail("too few lists of a kind", asides, in_order);
    std::printf("links of ops: as defined\n");
    return 0;
}
