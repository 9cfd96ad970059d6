"""The few-token kernel (one pass over the weights, two or three paths: stacks of up to 16 tokens, calls of up to 64) and
the three-path form of the fused decode kernel (one token) against the oracle: every op of a stack
recomputed from the input the GPU run actually used."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2602_05367_amd as rb
from helpers import TOL, to_device_layer, random_layer, bf16_bits, max_rel_l2

pytestmark = pytest.mark.gpu


def _branching_stack(rng, K, widths):
    """x -> a; a -> b, c, d (three readers of one output); b -> e; c -> f (e, f, d: stack outputs).
    widths: (x, a, b, c, d, e, f).  Gains keep activations near RMS 1 through the chain."""
    x, a, b, c, d, e, f = widths
    shapes = [(a, x), (b, a), (c, a), (d, a), (e, b), (f, c)]
    layers = []
    for (o, i) in shapes:
        signs, g, h = random_layer(rng, K, o, i)
        # half-normal scales: E[g h] ~ (0.02 * 0.8)^2 per path; bring the output to RMS ~1
        gain = 1.0 / (np.sqrt(i * K) * (0.02 * 0.02))
        layers.append((signs, (g.astype(np.float64) * gain).astype(np.float16), h))
    op_list = [(0, 0, 1), (1, 1, 2), (2, 1, 3), (3, 1, 4), (4, 2, 5), (5, 3, 6)]
    return layers, op_list


def _check_stack(layers, op_list, widths, x, T, label, prepared):
    # one token and three paths in every layer: the fused decode kernel; everything else here: the few-token kernel
    want_path = rb.RB_PATH_MX if (T == 1 and all(l[0].shape[0] == 3 for l in layers)) else rb.RB_PATH_BATCH
    dev_layers = [to_device_layer(*l) for l in layers]
    bufs = [torch.zeros((T, w), dtype=torch.float16, device="cuda") for w in widths]
    bufs[0].copy_(torch.from_numpy(x))
    print(f"{label}: T={T}, prepared={prepared}", flush=True)
    runs = []
    if prepared:
        stack = rb.Stack(dev_layers, op_list, bufs, T)
        stack.prepare()
        for _ in range(2):                      # the second run must repeat the first bit for bit
            stack.run_prepared()
            torch.cuda.synchronize()
            runs.append([b.clone() for b in bufs])
        assert rb.rb_last_path() == want_path
        assert stack.status() == rb.RB_OK, f"gave up: reason {stack.gave_up()}"
        stack.forget()
        for a, b in zip(*runs):
            assert torch.equal(a, b)
    else:
        rb.rb_layer_stack(dev_layers, op_list, bufs, T)
        torch.cuda.synchronize()
        assert rb.rb_last_path() == want_path
    got = [b.cpu().numpy() for b in bufs]
    worst = 0.0
    for n, (l, s, d) in enumerate(op_list):
        assert np.all(np.isfinite(got[d])), n
        ref = oracle.forward(*layers[l], got[s])
        assert np.abs(ref).max() > 0.05, n            # not a comparison of zeros
        err = float(oracle.relative_l2(got[d].astype(np.float64), ref).max())
        worst = max(worst, err)
        assert err <= TOL, (label, n, err)
    print(f"  worst rel_l2={worst:.3e}", flush=True)


# widths: part-filled row blocks (544 = 34 row tiles, 288 = 18), row counts that are not multiples of
# 16 (300, 90), column counts that are not multiples of 256 (1056, 544, 800), several column tiles
WIDTHS = (1056, 544, 288, 800, 300, 90, 1056)


@pytest.mark.parametrize("T", [5, 6, 8, 9, 13, 16])
def test_two_path_stack_small_batches(T):
    rng = synth.child_rng(3, 500, T)
    layers, op_list = _branching_stack(rng, 2, WIDTHS)
    x = synth.outlier_activations(rng, T, WIDTHS[0])
    # from 5 tokens on, rb_layer_stack and prepared stacks alike
    _check_stack(layers, op_list, WIDTHS, x, T, "two paths, branching stack", prepared=(T >= 8 and T % 2 == 0))


@pytest.mark.parametrize("T", [1, 2, 4, 7, 16])
def test_three_path_stack_one_to_sixteen_tokens(T):
    rng = synth.child_rng(3, 501, T)
    layers, op_list = _branching_stack(rng, 3, WIDTHS)
    x = synth.outlier_activations(rng, T, WIDTHS[0])
    _check_stack(layers, op_list, WIDTHS, x, T, "three paths, branching stack", prepared=(T % 2 == 1))


def test_three_path_stack_derived_weights():
    """Paths derived from a Gaussian weight by the oracle (Section 4.2 steps 1-3), three paths."""
    rng = synth.child_rng(3, 502)
    shapes = [(544, 576), (288, 544), (576, 288)]
    layers = []
    x = synth.gaussian_activations(rng, 5, 576)
    cur = x
    for (o, i) in shapes:
        signs, g, h, _ = oracle.derive(synth.gaussian_weight(rng, o, i), 3)
        y = oracle.forward(signs, g, h, cur)
        g = (g.astype(np.float64) / np.sqrt((y ** 2).mean())).astype(np.float16)
        layers.append((signs, g, h))
        cur = oracle.forward(signs, g, h, cur).astype(np.float16)
    _check_stack(layers, [(0, 0, 1), (1, 1, 2), (2, 2, 3)], (576, 544, 288, 576), x, 5, "three paths, derived", True)


def test_mixed_two_and_three_path_layers_in_one_stack():
    rng = synth.child_rng(3, 503)
    shapes = [(544, 288, 2), (288, 544, 3), (320, 544, 2), (90, 288, 3)]
    layers = []
    for (o, i, K) in shapes:
        signs, g, h = random_layer(rng, K, o, i)
        gain = 1.0 / (np.sqrt(i * K) * (0.02 * 0.02))
        layers.append((signs, (g.astype(np.float64) * gain).astype(np.float16), h))
    x = synth.gaussian_activations(rng, 6, 288)          # a three-path layer: the batch kernel at any T
    # op 0: x -> a; ops 1 (K=3) and 2 (K=2) both read a; op 3 reads op 1's output
    _check_stack(layers, [(0, 0, 1), (1, 1, 2), (2, 1, 3), (3, 2, 4)], (288, 544, 288, 320, 90), x, 6, "mixed K", True)


def test_batch_kernel_with_degenerate_scales_and_extreme_inputs():
    """Negative and zero entries in g and h, an all-zero h_k, inputs at the ends of the fp16 range."""
    rng = synth.child_rng(3, 504)
    T, d0, d1, d2 = 9, 1056, 544, 270
    def edge(out, inn, zero_path):
        signs, g, h = random_layer(rng, 2, out, inn)
        g = g.astype(np.float64); h = h.astype(np.float64)
        g[:, rng.integers(0, out, 9)] *= -1.0
        h[:, rng.integers(0, inn, 17)] *= -1.0
        g[0, rng.integers(0, out, 5)] = 0.0
        h[1, rng.integers(0, inn, 11)] = 0.0
        if zero_path is not None:
            h[zero_path] = 0.0
        return signs, g.astype(np.float16), h.astype(np.float16)
    l1 = edge(d1, d0, None)
    x = synth.outlier_activations(rng, T, d0).astype(np.float64)
    idx = rng.choice(d0, size=8, replace=False)
    x[:, idx[0:2]] = 2000.0
    x[:, idx[2:4]] = 3.0e-7                                   # subnormal in fp16
    x[:, idx[4:8]] = 0.0
    x = x.astype(np.float16)
    y1 = oracle.forward(*l1, x)
    l1 = (l1[0], (l1[1].astype(np.float64) / np.sqrt((y1 ** 2).mean())).astype(np.float16), l1[2])
    l2 = edge(d2, d1, 1)
    y2 = oracle.forward(*l2, oracle.forward(*l1, x).astype(np.float16))
    l2 = (l2[0], (l2[1].astype(np.float64) / np.sqrt((y2 ** 2).mean())).astype(np.float16), l2[2])
    _check_stack([l1, l2], [(0, 0, 1), (1, 1, 2)], (d0, d1, d2), x, T, "edge cases", True)


@pytest.mark.parametrize("T,K", [(8, 2), (16, 2), (1, 3), (8, 3)])
def test_full_width_7b_block_on_the_batch_kernel(T, K):
    """One block of the 7B shape exactly as bench.py builds it (signs drawn on the device), at the
    widths and launch shapes that are timed, two and three paths: sampled rows of every op
    against the oracle."""
    import bench
    ops, layers, bufs, op_list, _ = bench.build_stack(rb, synth, torch, "7b", T, K=K)
    ops, layers, op_list = ops[:7], layers[:7], op_list[:7]
    bufs[0].copy_(torch.from_numpy(synth.outlier_activations(synth.child_rng(3, 505, T), T, ops[0].inn)))
    stack = rb.Stack(layers, op_list, bufs, T)
    stack.prepare()
    print(f"full-width 7B block on the batch kernel, T={T}, K={K}", flush=True)
    stack.run_prepared()
    torch.cuda.synchronize()
    assert rb.rb_last_path() == (rb.RB_PATH_MX if (K == 3 and T == 1) else rb.RB_PATH_BATCH) and stack.status() == rb.RB_OK
    stack.forget()
    pick = np.random.default_rng(11)
    worst = 0.0
    for n, op in enumerate(ops):
        L = layers[n]
        y = bufs[op.dst].cpu().numpy().astype(np.float64)
        assert np.all(np.isfinite(y)) and np.any(y != 0), op.name
        native = L.bits.cpu().numpy().view(np.uint32)
        packed = rb.rb_unpack_native(native, K, L.out, L.inn)
        rows = np.unique(np.concatenate([pick.integers(0, L.out, size=40), [0, L.out - 1]]))
        S = rb.rb_unpack(packed[:, rows, :])
        ref = oracle.forward(S, L.g.cpu().numpy()[:, rows], L.h.cpu().numpy(), bufs[op.src].cpu().numpy())
        err = float(oracle.relative_l2(y[:, rows], ref).max())
        worst = max(worst, err)
        assert err <= TOL, (op.name, err)
    print(f"  worst sampled rel_l2={worst:.3e}", flush=True)


@pytest.mark.parametrize("n_ops,T,inn", [(8, 16, 288), (4, 9, 288), (8, 5, 288), (8, 16, 1056), (4, 9, 1056), (2, 5, 1056)])
def test_many_independent_rows_take_larger_row_blocks(n_ops, T, inn):
    """A launch with rows enough lets a workgroup of a layer of more than 1024 columns own up to six row tiles, so that the staged inputs are
    shared by more rows; narrow layers keep to one or two.  The same
    results, other instantiations of the kernel.  Every op reads the one stack input."""
    rng = synth.child_rng(3, 506, n_ops, T)
    out = 8192 - 16 * 5 - 3                           # part-filled last row tile and last row block
    layers = []
    for _ in range(n_ops):
        signs, g, h = random_layer(rng, 2, out, inn)
        gain = 1.0 / (np.sqrt(inn * 2) * (0.02 * 0.02))
        layers.append((signs, (g.astype(np.float64) * gain).astype(np.float16), h))
    x = synth.outlier_activations(rng, T, inn)
    op_list = [(n, 0, 1 + n) for n in range(n_ops)]
    _check_stack(layers, op_list, (inn,) + (out,) * n_ops, x, T, f"{n_ops} independent ops of {out} rows", prepared=(T >= 8))


@pytest.mark.parametrize("narrow,wide,T,K", [(1024, 4096, 16, 2), (32, 4128, 5, 2), (896, 2080, 9, 2), (32, 1056, 16, 3), (1920, 4096, 6, 3), (96, 11008, 8, 2)])
def test_ops_of_different_widths_share_a_launch(narrow, wide, T, K):
    """Two independent ops in one launch, whose workgroups have as many wavefronts as the wider one has use for: some have no columns
    of the narrower op.  Its scales fill an allocation of their own."""
    rng = synth.child_rng(3, 511, narrow, wide, T)
    layers, dev, widths = [], [], (narrow, wide, 300, 130)
    for o, i in ((300, narrow), (130, wide)):
        signs, g, h = random_layer(rng, K, o, i, gain=1.0 / (np.sqrt(i * K) * (0.02 * 0.02)))
        layers.append((signs, g, h))
        dev.append(to_device_layer(signs, g, h))
    xs = [synth.outlier_activations(rng, T, w) for w in (narrow, wide)]
    bufs = [torch.from_numpy(x).cuda() for x in xs] + [torch.zeros((T, w), dtype=torch.float16, device="cuda") for w in widths[2:]]
    print(f"ops of {narrow} and {wide} columns in one launch, T={T} K={K}", flush=True)
    rb.rb_layer_stack(dev, [(0, 0, 2), (1, 1, 3)], bufs, T)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_BATCH
    for n in range(2):
        assert max_rel_l2(bufs[2 + n], oracle.forward(*layers[n], xs[n])) <= TOL, n


@pytest.mark.parametrize("T", [1, 3, 8])
def test_scales_that_are_only_two_byte_aligned(T):
    """g and h need no more than the alignment of their elements: a two-op chain whose scale
    vectors start two bytes past a 16-byte boundary, on the fused kernel (1 and 3 tokens) and on
    the few-token kernel (8 tokens; it reads h sixteen bytes at a time when it can)."""
    rng = synth.child_rng(3, 507, T)
    shapes = [(320, 544), (288, 320)]
    layers = [random_layer(rng, 2, o, i, gain=30.0) for o, i in shapes]

    def off_by_one(a):
        flat = torch.zeros(a.size + 1, dtype=torch.float16, device="cuda")
        flat[1:].copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float16)).flatten())
        t = flat[1:].view(a.shape)
        assert t.data_ptr() % 16 == 2
        return t
    dev_layers = []
    for signs, g, h in layers:
        aligned = to_device_layer(signs, g, h)
        dev_layers.append(rb.Layer(aligned.bits, off_by_one(g), off_by_one(h), 2, signs.shape[1], signs.shape[2]))
    x = synth.outlier_activations(rng, T, 544)
    bufs = [torch.zeros((T, w), dtype=torch.float16, device="cuda") for w in (544, 320, 288)]
    bufs[0].copy_(torch.from_numpy(x))
    print(f"scales two bytes past a 16-byte boundary, T={T}", flush=True)
    rb.rb_layer_stack(dev_layers, [(0, 0, 1), (1, 1, 2)], bufs, T)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == (rb.RB_PATH_BATCH if T == 8 else rb.RB_PATH_MX)
    got = [b.cpu().numpy() for b in bufs]
    for n, (signs, g, h) in enumerate(layers):
        ref = oracle.forward(signs, g, h, got[n])
        assert np.abs(ref).max() > 0.05
        assert oracle.relative_l2(got[n + 1].astype(np.float64), ref).max() <= TOL, n
    y = rb.rb_linear_gemm(dev_layers[0], bufs[0])             # the single-call kernels take the same layers
    torch.cuda.synchronize()
    assert oracle.relative_l2(y.cpu().numpy().astype(np.float64), oracle.forward(*layers[0], got[0])).max() <= TOL


@pytest.mark.parametrize("prepared", [True, False])
def test_three_path_decode_kernel_one_token(prepared):
    """Three paths, one token: the fused decode kernel (its three paths take the place of two
    tokens' two paths in the right operand), a branching stack with ragged widths."""
    rng = synth.child_rng(3, 507, int(prepared))
    layers, op_list = _branching_stack(rng, 3, WIDTHS)
    x = synth.outlier_activations(rng, 1, WIDTHS[0])
    _check_stack(layers, op_list, WIDTHS, x, 1, "three paths, one token", prepared)


def test_three_path_decode_kernel_early_reads_and_degenerate_scales():
    """The same kernel with no hand-over pause at all (nearly every input tile is asked for before
    it is written and has to be read again), negative and zero scales, an all-zero third path."""
    rng = synth.child_rng(3, 508)
    widths = (1056, 544, 288, 800)
    layers = []
    for n, (o, i) in enumerate([(544, 1056), (288, 544), (800, 288)]):
        signs, g, h = random_layer(rng, 3, o, i)
        g = g.astype(np.float64) / (np.sqrt(i * 3) * (0.02 * 0.02)); h = h.astype(np.float64)
        g[:, rng.integers(0, o, 7)] *= -1.0
        h[:, rng.integers(0, i, 9)] *= -1.0
        g[2, rng.integers(0, o, 3)] = 0.0
        if n == 1:
            h[2] = 0.0
        layers.append((signs, g.astype(np.float16), h.astype(np.float16)))
    x = synth.outlier_activations(rng, 1, widths[0])
    for pause in (0, -1):
        rb.rb_stack_set_option(rb.RB_OPT_HANDOVER_PAUSE, pause)
        try:
            _check_stack(layers, [(0, 0, 1), (1, 1, 2), (2, 2, 3)], widths, x, 1, f"three paths, pause {pause}", True)
        finally:
            rb.rb_stack_set_option(rb.RB_OPT_HANDOVER_PAUSE, -1)


@pytest.mark.parametrize("K,out,inn,T,bf16", [
    (2, 20, 32, 3, False), (2, 4112, 288, 16, False), (2, 8200, 288, 5, True), (2, 12304, 160, 16, False), (2, 16390, 288, 7, False),
    (3, 4112, 288, 6, False), (3, 8208, 160, 16, True), (3, 12300, 288, 9, False),       # (several row tiles per workgroup: see below)
    (2, 300, 4384, 17, False), (2, 4112, 288, 32, True), (2, 8200, 96, 31, False), (3, 4100, 288, 18, False),
    (2, 300, 8256, 33, True), (2, 4112, 288, 64, False), (2, 8200, 96, 49, False), (3, 4100, 160, 64, False)])
def test_few_token_calls_element_by_element(K, out, inn, T, bf16):
    """The few-token kernel (token groups of 16, both element
    types; every form of a workgroup in the tests below, which call this one) against fp64, fp32 results.  Products of a scale and an activation are exact, so only the
    additions of the K in terms, the output scale and the path sum round: |error| <= (K in + 8)
    2^-23 sum |g h x| (twice the half-ulp bound; a scale that meets bf16 activations as two terms adds twice as many, which
    half of that bound covers).  One h in eight is an fp16 subnormal, scales have either sign."""
    rng = synth.child_rng(3, 510, K, out, inn, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = g.copy(); h = h.copy()
    g[0, ::5] *= -1; h[1, 1::3] *= -1
    h[:, ::8] = (h[:, ::8].astype(np.float64) * 1e-3).astype(np.float16)
    X = synth.outlier_activations(rng, T, inn)
    Xd = torch.from_numpy(X).cuda()
    if bf16:
        Xd = Xd.to(torch.bfloat16)
        X = Xd.float().cpu().numpy()
    print(f"few-token call K={K} {out}x{inn} T={T} bf16={bf16}", flush=True)
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), Xd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.forward(signs, g, h, X.astype(np.float64))
    size = np.zeros((T, out))
    for k in range(K):
        size += (np.abs(X.astype(np.float64)) @ np.abs(h[k].astype(np.float64)))[:, None] * np.abs(g[k].astype(np.float64))[None, :]
    err = np.abs(Y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= (K * inn + 8) * 2.0 ** -23 * size), float((err / size).max())


@pytest.mark.parametrize("K,out,inn,T,bf16", [
    # sign tiles shared by two wavefronts (9, 17 and 33 units of 128 columns for 8 or 16 of them); several workgroups on a
    # compute unit, many rows of narrow layers
    (2, 300, 1056, 16, False), (2, 300, 4128, 3, True), (3, 60, 2112, 7, False), (2, 28672, 288, 9, False), (2, 22016, 544, 16, True),
    (3, 13824, 544, 6, False), (2, 11008, 544, 64, False), (3, 8208, 288, 40, False), (2, 16400, 544, 24, False), (3, 300, 2080, 17, True),
    # three paths, one to five tokens
    (3, 300, 1056, 1, False), (3, 12300, 288, 2, True), (3, 28672, 160, 5, False), (3, 4100, 2080, 3, True)])
def test_few_token_forms_and_shared_tiles(K, out, inn, T, bf16):
    test_few_token_calls_element_by_element(K, out, inn, T, bf16)


@pytest.mark.parametrize("K,out,inn,T,bf16", [
    # wide enough (more than 1024 columns) that the number of row tiles decides: 1, 2, 3, 4 and 6 per workgroup (three paths: 5 and 7 too), each with one, two and four token
    # groups where that form exists, both element types, eight and sixteen wavefronts
    (2, 300, 1056, 9, False), (2, 4112, 1056, 9, True), (2, 4112, 2080, 15, False), (2, 8200, 1056, 9, False), (2, 12304, 1056, 16, True),
    (2, 16390, 1056, 9, False), (2, 16390, 1056, 3, True), (2, 4112, 1056, 24, False), (2, 8200, 1056, 32, True), (2, 12304, 1056, 24, False),
    (2, 4112, 1056, 48, True), (2, 8200, 1056, 48, False), (3, 4112, 1056, 9, False), (3, 8200, 1056, 9, True), (3, 12304, 1056, 9, False),
    (3, 12304, 1056, 2, True), (3, 16400, 1056, 9, False), (3, 16400, 1056, 16, True), (3, 20500, 1056, 3, False), (3, 20500, 1056, 9, True),
    (3, 24600, 1056, 16, False), (3, 24600, 1056, 7, True), (3, 4112, 1056, 24, True), (3, 8200, 1056, 24, False), (3, 4112, 1056, 48, False), (3, 300, 1056, 48, True),
    # sixteen wavefronts for two, three and four row tiles
    (2, 4112, 5120, 6, False), (2, 8200, 5152, 16, True), (2, 8200, 5152, 11, False), (2, 12304, 5152, 3, False), (2, 12304, 5152, 9, True), (3, 4112, 5152, 13, False),
    # narrow layers: one to eight wavefronts and several workgroups on a compute unit
    (2, 28672, 32, 48, False), (2, 28672, 512, 33, True), (2, 22016, 1024, 24, False), (3, 28672, 1024, 48, True), (3, 5000, 640, 64, False),
    (3, 22016, 512, 9, True), (2, 8200, 896, 17, False)])
def test_few_token_row_tiles_and_narrow_layers(K, out, inn, T, bf16):
    test_few_token_calls_element_by_element(K, out, inn, T, bf16)


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("out,inn,T,act,shift", [
    (16, 32, 6, "f16", 0), (130, 160, 13, "bf16", 1), (1000, 2080, 17, "f16", 1), (4099, 288, 33, "bf16", 0), (70, 4128, 64, "f16", 0),
    (9000, 544, 9, "f16", 0), (9000, 1184, 9, "f16", 1)])
def test_few_token_staging_edges(K, out, inn, T, act, shift):
    """Staged activations of the few-token kernel: token counts that are no multiple of the four a load takes, half
    column tiles, one wavefront per workgroup, two and four token groups, several row tiles per workgroup, scales at an odd
    multiple of two bytes.  Products are exact, so fp32 results are held to 1e-5."""
    rng = synth.child_rng(5, 130, K, out, inn, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = g.copy(); h = h.copy()
    g[1, ::6] *= -1; h[0, ::3] *= -1; h[1, 5] = 0
    X = synth.outlier_activations(rng, T, inn)
    print(f"few tokens K={K} out={out} in={inn} T={T} {act} shift={shift}", flush=True)
    L = to_device_layer(signs, g, h)
    if shift:
        store = torch.zeros(K * inn + shift, dtype=torch.float16, device="cuda")
        store[shift:] = L.h.flatten()
        L.h = store[shift:].view(K, inn)
    Xd = torch.from_numpy(X).cuda()
    if act == "bf16":
        Xd = Xd.to(torch.bfloat16)
        X = oracle.bf16_bits_to_f64(bf16_bits(Xd.cpu())).reshape(T, inn)
    Y = torch.full((T + 1, out), 7.0, dtype=torch.float32, device="cuda")
    rb.rb_linear_gemm(L, Xd, Y=Y[:T])
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    assert torch.all(Y[T] == 7.0)
    assert max_rel_l2(Y[:T], oracle.forward(signs, g, h, X)) <= 1e-5


def _device_layer(gen, K, out, inn):
    """Random signs drawn on the device in native order, scales near those of a derived layer."""
    bits = torch.randint(-2 ** 31, 2 ** 31 - 1, (rb.rb_native_bytes(K, out, inn) // 4,), dtype=torch.int32, device="cuda", generator=gen)
    g = (torch.randn((K, out), device="cuda", generator=gen).abs() * 0.1 + 0.01).half()
    h = (torch.randn((K, inn), device="cuda", generator=gen).abs() * 0.1 + 0.01).half()
    return rb.Layer(bits, g, h, K, out, inn)


def _forward_on_device(L, X):
    """fp64 on the device, a path at a time (plain torch; the signs unpacked by the host's unpacker)."""
    signs = rb.rb_unpack(rb.rb_unpack_native(L.bits.cpu().numpy().view(np.uint32), L.K, L.out, L.inn))
    Y = torch.zeros((X.shape[0], L.out), dtype=torch.float64, device="cuda")
    for k in range(L.K):
        Y += ((X.double() * L.h[k].double()) @ torch.from_numpy(signs[k]).cuda().double().t()) * L.g[k].double()
    return Y


@pytest.mark.parametrize("K,out,inn,T,bf16", [(2, 5, 2 ** 24, 3, False), (3, 17, 2 ** 24 + 96, 1, True), (2, 3, 2 ** 23 + 160, 64, False), (2, 2, 2 ** 25, 20, True)])
def test_few_token_calls_with_offsets_beyond_a_gigabyte(K, out, inn, T, bf16):
    """2^24 columns, or inputs of a gigabyte and more: the few-token kernel's form with 64-bit addresses.  A sum of 2^24 terms of either sign in
    fp32, an eighth of them per wavefront and 32 at a time: 2^16 roundings, each up to 2^-24 of the sum so far, add up in
    quadrature to 2^8 2^-24 = 1.5e-5 of the outputs' norm (of all outputs: a single sum may cancel and its own relative error be any
    size); the bar is six times that, and the root of the number of roundings more for wider layers and for bf16, which takes two
    instructions.  A unit of 128 columns read from the wrong place is 2e-3 of it and more."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(out + T)
    L = _device_layer(gen, K, out, inn)
    X = torch.randn((T, inn), device="cuda", generator=gen).to(torch.bfloat16 if bf16 else torch.float16)
    print(f"wide few-token call K={K} {out}x{inn} T={T} bf16={bf16}", flush=True)
    Y = rb.rb_linear_gemm(L, X, out_dtype=torch.float32)
    ref = _forward_on_device(L, X)
    err = float((Y.double() - ref).norm() / ref.norm())
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= 1e-4 * (inn / 2 ** 24 * (2 if bf16 else 1)) ** 0.5


def test_stack_with_a_wide_op():
    """2^24 columns beside 288 in one launch of a stack, then an op that reads the wide one's output."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    T, shapes = 5, ((64, 2 ** 24), (300, 288), (40, 64))
    layers = [_device_layer(gen, 2, o, i) for o, i in shapes]
    for L in layers:                                           # outputs near RMS 1
        L.g.copy_((L.g.float() * (1.0 / (0.0064 * (2 * L.inn) ** 0.5))).half())
    bufs = [torch.randn((T, w), device="cuda", generator=gen).half() for w in (2 ** 24, 288)] + \
           [torch.zeros((T, w), dtype=torch.float16, device="cuda") for w in (64, 300, 40)]
    print("stack with a wide op", flush=True)
    rb.rb_layer_stack(layers, [(0, 0, 2), (1, 1, 3), (2, 2, 4)], bufs, T)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_BATCH
    for L, src, dst in zip(layers, (0, 1, 2), (2, 3, 4)):
        assert max_rel_l2(bufs[dst], _forward_on_device(L, bufs[src]).cpu().numpy()) <= TOL


@pytest.mark.parametrize("K,n,T", [(2, 8224, 3), (2, 8224, 16), (2, 12320, 7), (2, 4128, 33), (2, 8224, 64), (3, 8224, 6), (3, 4128, 16), (3, 4128, 64)])
def test_few_token_output_over_its_input(K, n, T):
    """From three tokens on (six with three paths) the output may overlap the input, with more row tiles than one
    round of workgroups takes: the input is moved aside first, to the workspace or to the library's scratch
    memory.  The results are those of separate buffers, bit for bit."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(100 * n + T)
    L = _device_layer(gen, K, n, n)
    X = torch.randn((T, n), device="cuda", generator=gen).half()
    want = rb.rb_linear_gemm(L, X)
    print(f"output over its input K={K} {n}x{n} T={T}", flush=True)
    for call in (lambda x, y: rb.rb_linear_gemm(L, x, Y=y), lambda x, y: rb.rb_linear_gemm_noalloc(L, x, y)):
        whole = torch.zeros((3, T, n), dtype=torch.float16, device="cuda")
        # the same buffer, and an output that starts in the middle of the input
        for at in (0, T // 2 * n):
            x, y = whole.flatten()[:T * n].view(T, n), whole.flatten()[at:at + T * n].view(T, n)
            x.copy_(X)
            call(x, y)
            torch.cuda.synchronize()
            assert torch.equal(y, want)
        # bfloat16 in, fp32 out, the input inside the output
        store = torch.zeros(T * n * 4, dtype=torch.uint8, device="cuda")
        y, x = store.view(torch.float32).view(T, n), store[T * n * 2:].view(torch.bfloat16).view(T, n)
        x.copy_(X)
        sep = rb.rb_linear_gemm(L, x.clone(), out_dtype=torch.float32)
        call(x, y)
        torch.cuda.synchronize()
        assert torch.equal(y, sep)


@pytest.mark.parametrize("K,T,prepared", [(2, 5, True), (2, 16, False), (3, 2, False), (3, 8, True)])
def test_stack_buffers_that_overlap_in_memory(K, T, prepared):
    """Buffers of different indices in one piece of memory: an op over its own input (buffer 1 starts in the
    middle of buffer 0), an op that reads what an earlier op of the list has written under another index (4 is
    3's memory), one that overwrites what an earlier op has read (6 is 2's).  Each op's result is that of the
    ops run one after the other on buffers of their own."""
    n = 8224
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7 * K + T)
    layers = [_device_layer(gen, K, n, n) for _ in range(4)]
    for L in layers:                                           # outputs near RMS 1
        L.g.mul_(1.0 / (0.0064 * (K * n) ** 0.5))
    ops = [(0, 0, 1), (1, 2, 3), (2, 4, 5), (3, 5, 6)]
    pool = torch.zeros((6, T, n), dtype=torch.float16, device="cuda").flatten()
    at = lambda i: pool[i * T * n // 2:i * T * n // 2 + T * n].view(T, n)
    bufs = [at(0), at(1), at(4), at(6), at(6), at(8), at(4)]
    x0, x2 = (torch.randn((T, n), device="cuda", generator=gen).half() for _ in range(2))
    print(f"overlapping buffers K={K} T={T} prepared={prepared}", flush=True)
    stack = rb.Stack(layers, ops, bufs, T)
    if prepared:
        stack.prepare()
    for _ in range(2):                                         # (a run leaves other contents behind)
        bufs[0].copy_(x0)
        bufs[2].copy_(x2)
        stack.run_prepared() if prepared else stack.run()
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_BATCH
    stack.forget()
    y1, y3 = rb.rb_linear_gemm(layers[0], x0), rb.rb_linear_gemm(layers[1], x2)
    y5 = rb.rb_linear_gemm(layers[2], bufs[3].clone())
    y6 = rb.rb_linear_gemm(layers[3], bufs[5].clone())
    for got, want in ((bufs[1], y1), (bufs[3], y3), (bufs[5], y5), (bufs[6], y6)):
        assert max_rel_l2(got, want.double().cpu().numpy()) <= TOL


@pytest.mark.parametrize("K,out,inn,T", [(2, 4112, 288, 1), (2, 300, 1056, 2), (2, 4112, 288, 7), (2, 8200, 160, 16), (2, 12304, 160, 5),
                                         (2, 16390, 96, 9), (2, 4112, 1056, 7), (2, 8200, 1056, 16), (2, 12304, 1056, 5), (2, 16390, 1056, 9), (3, 12304, 1056, 6),
                                         (2, 8200, 5152, 3), (2, 300, 544, 18), (2, 4112, 96, 64), (2, 4112, 1056, 64), (3, 300, 288, 6), (3, 4112, 160, 16),
                                         (3, 300, 96, 33), (2, 20, 135200, 2), (3, 16, 135200, 6)])
@pytest.mark.parametrize("size", [3.0e5, 1.0e30, 2.0 ** -15, 2.0 ** -20, 2.0 ** -30, 2.0 ** -80, "mixed"])
def test_few_token_bf16_over_its_whole_range(K, out, inn, T, size):
    """bfloat16 activations far beyond fp16's range, every row tile count per workgroup and token group, more than 64 pieces of
    128 columns per wavefront.  An input scale
    is the exact sum of two bf16 values, so their products with a bf16 activation are exact and only the additions of the
    2 K in terms, the output scale and the path sum round: |error| <= (2 K in + 8) 2^-23 sum |g h x| (twice the
    half-ulp bound).  The scales are the ends of fp16's range too: subnormals, zeros, either sign."""
    rng = synth.child_rng(3, 511, K, out, inn, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = g.copy(); h = h.copy()
    g[0, ::5] *= -1; h[1, 1::3] *= -1; h[0, 4] = 0; h[1, 9] = -0.0; h[0, 6] = 1.0; h[1, 7] = 65504.0; h[0, 8] = 6.0e-8
    h[:, ::8] = (h[:, ::8].astype(np.float64) * 1e-3).astype(np.float16)
    # "mixed": every 128 columns in three of a size of their own, zeros and whole runs that fp16 holds among them
    sizes = torch.from_numpy(2.0 ** rng.uniform(-24, 24, -(-inn // 128))).repeat_interleave(128)[:inn]
    sizes[torch.arange(inn) // 128 % 3 != 0] = 1.0
    Xd = torch.from_numpy(synth.gaussian_activations(rng, T, inn)).double() * (sizes if size == "mixed" else size)
    Xd[:, ::11] = 0.0
    Xd = Xd.cuda().to(torch.bfloat16)
    X = Xd.double().cpu().numpy()
    print(f"bf16 range K={K} {out}x{inn} T={T} size={size}", flush=True)
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), Xd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.forward(signs, g, h, X)
    bound = np.zeros((T, out))
    for k in range(K):
        bound += (np.abs(X) @ np.abs(h[k].astype(np.float64)))[:, None] * np.abs(g[k].astype(np.float64))[None, :]
    err = np.abs(Y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= (2 * K * inn + 8) * 2.0 ** -23 * bound), float((err / bound).max())


@pytest.mark.parametrize("K,T,act", [(2, 2, "bf16"), (2, 7, "bf16"), (3, 6, "bf16"), (2, 7, "f16")])
def test_few_token_infinite_activations(K, T, act):
    """An infinity in one token's input: that token's outputs are what plain arithmetic gives (infinities by the sign of
    the weight, NaN where a scale is zero or the paths disagree), the other tokens' are finite."""
    out, inn = 300, 544
    rng = synth.child_rng(3, 512, K, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = np.abs(g) + np.float16(0.01); h = np.abs(h) + np.float16(0.01)
    h[:, 40] = np.float16(0.5)                                 # a bf16 value
    X = synth.gaussian_activations(rng, T, inn)
    X[1, 40] = np.inf
    print(f"infinite activation K={K} T={T} {act}", flush=True)
    Xd = torch.from_numpy(X).cuda().to(torch.bfloat16 if act == "bf16" else torch.float16)
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), Xd, out_dtype=torch.float32).cpu().numpy()
    paths = signs[:, :, 40].astype(np.float64) * np.inf
    with np.errstate(invalid="ignore"):
        np.testing.assert_array_equal(Y[1], paths.sum(axis=0))
    assert np.all(np.isfinite(np.delete(Y, 1, axis=0)))
