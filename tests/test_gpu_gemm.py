"""Matrix-core GEMM of single calls (the few-token kernel up to 64 tokens and, on layers of few rows, beyond, the
many-token kernel else; both report RB_PATH_GEMM here) vs the fp64 oracle (Section 4.1, Eq. stacked binary
weight), through the C ABI.  Sizes span several workgroup tiles and ragged
tails in every dimension; the 70B-shaped prefill matrices are checked on sampled
outputs the oracle computes one by one."""
import sys

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2602_05367_amd as rb
from helpers import TOL, random_layer, to_device_layer, bf16_bits, max_rel_l2, only_for_many_tokens

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("out,inn,T", [
    (256, 256, 256),        # two blocks of 128 rows, one column tile
    (512, 1024, 300),       # whole row blocks, ragged tokens
    (272, 320, 33),         # few tokens: ragged rows (17 row tiles), ragged columns (in % 256 != 0)
    (1000, 2080, 517),      # everything ragged
    (48, 32, 3),            # few tokens, tiny: three row tiles, the smallest input width
    (4096, 1024, 256),      # whole tiles in every direction
    (8400, 1024, 2048),     # more than one round of the device's workgroups, ragged last row block
    (2816, 512, 2048),      # as many column steps as column groups
])
def test_gemm_matches_oracle(out, inn, T):
    rng = synth.child_rng(5, 100, out, inn, T)
    signs, g, h = random_layer(rng, 2, out, inn)
    X = synth.outlier_activations(rng, T, inn)
    _say(f"gemm out={out} in={inn} T={T}")
    L = to_device_layer(signs, g, h)
    Y = rb.rb_linear_gemm(L, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    err = max_rel_l2(Y, oracle.forward(signs, g, h, X))
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("out,inn,T", [(272, 320, 33), (1000, 2080, 517), (4096, 1024, 256), (8400, 1024, 300)])
def test_three_path_gemm_matches_oracle(out, inn, T):
    """The 3-bit variant: a third path in the effective weight (ragged shapes, scales of either sign); at 33 tokens the
    few-token kernel."""
    rng = synth.child_rng(5, 110, out, inn, T)
    signs, g, h = random_layer(rng, 3, out, inn)
    g = g.copy(); h = h.copy()
    g[2, ::7] *= -1; h[1, ::5] *= -1; h[2, 3::4] *= -1; g[0, 11] = 0
    X = synth.outlier_activations(rng, T, inn)
    _say(f"three-path gemm out={out} in={inn} T={T}")
    L = to_device_layer(signs, g, h)
    Y = rb.rb_linear_gemm(L, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    err = max_rel_l2(Y, oracle.forward(signs, g, h, X))
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("out,inn,T,bf16_in,path", [
    (272, 544, 5, False, "generic"), (272, 544, 6, False, "batch"), (1000, 2080, 8, False, "batch"), (272, 544, 12, False, "batch"),
    (272, 544, 13, False, "gemm"), (1000, 2080, 32, False, "gemm"), (272, 544, 3, True, "generic"), (48, 32, 7, True, "gemm")])
def test_three_path_single_calls_at_few_tokens(out, inn, T, bf16_in, path):
    """One call on a three-path layer from 6 tokens on takes the few-token kernel, which reports itself as RB_PATH_BATCH up
    to 12 fp16 tokens and as RB_PATH_GEMM beyond that and for bf16; fewer tokens take it too and are reported as the generic
    kernel, which served them once."""
    rng = synth.child_rng(5, 111, out, inn, T)
    signs, g, h = random_layer(rng, 3, out, inn)
    g = g.copy(); h = h.copy()
    g[1, ::6] *= -1; h[2, ::3] *= -1
    X = synth.outlier_activations(rng, T, inn)
    _say(f"three-path single call out={out} in={inn} T={T} bf16={bf16_in}")
    L = to_device_layer(signs, g, h)
    Xd = torch.from_numpy(X).cuda()
    if bf16_in:
        Xd = Xd.to(torch.bfloat16)
        X = oracle.bf16_bits_to_f64(bf16_bits(Xd.cpu())).reshape(T, inn)
    Y = rb.rb_linear_gemm(L, Xd)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == {"batch": rb.RB_PATH_BATCH, "gemm": rb.RB_PATH_GEMM, "generic": rb.RB_PATH_SIGNADD}[path]
    err = max_rel_l2(Y, oracle.forward(signs, g, h, X))
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("K", [2, 3])
def test_generic_kernel_beyond_the_matrix_core_kernels(K):
    """2^22 columns are too many for the many-token kernel, 65 tokens for the few-token kernel.  Sums of 2^22 terms in fp32 over the lanes
    and wavefronts of a workgroup: 1e-3."""
    out, inn, T = 3, 2 ** 22 + 32, 65
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    bits = torch.randint(-2 ** 31, 2 ** 31 - 1, (rb.rb_native_bytes(K, out, inn) // 4,), dtype=torch.int32, device="cuda", generator=gen)
    g, h = ((torch.randn((K, n), device="cuda", generator=gen).abs() * 0.1 + 0.01).half() for n in (out, inn))
    L = rb.Layer(bits, g, h, K, out, inn)
    X = torch.randn((T, inn), device="cuda", generator=gen).half()
    _say(f"generic kernel K={K} {out}x{inn} T={T}")
    Y = rb.rb_linear_gemm(L, X, out_dtype=torch.float32)
    assert rb.rb_last_path() == rb.RB_PATH_SIGNADD
    signs = rb.rb_unpack(rb.rb_unpack_native(bits.cpu().numpy().view(np.uint32), K, out, inn))
    ref = torch.zeros((T, out), dtype=torch.float64, device="cuda")
    for k in range(K):
        ref += ((X.double() * h[k].double()) @ torch.from_numpy(signs[k]).cuda().double().t()) * g[k].double()
    err = float((Y.double() - ref).norm() / ref.norm())
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL


def test_gemm_negative_and_zero_scales():
    """Stored output scales of either sign and zero, 40 tokens."""
    out, inn, T = 96, 512, 40
    rng = synth.child_rng(5, 101)
    signs, g, h = random_layer(rng, 2, out, inn)
    g = g.copy(); h = h.copy()
    g[0, ::3] *= -1; g[1, 1::4] *= -1; g[1, 5] = 0
    h[0, ::5] *= -1; h[1, 7] = 0
    X = synth.gaussian_activations(rng, T, inn)
    L = to_device_layer(signs, g, h)
    Y = rb.rb_linear_gemm(L, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    assert max_rel_l2(Y, oracle.forward(signs, g, h, X)) <= TOL


@pytest.mark.parametrize("T", [16, 70, 2800])                   # (the last one on the many-token kernel)
def test_gemm_when_the_magnitude_sits_in_g(T):
    """Section 4.1 leaves the split of a path's magnitude between g and h open.  With h around 3e-5
    and g around 10 the products h x are fp16 subnormals unless the kernel scales each path's h by
    a power of two first (and takes it back out of g); path 2 gets another factor 1/8 on h."""
    out, inn = 272, 1056
    rng = synth.child_rng(5, 109, T)
    signs, g, h = random_layer(rng, 2, out, inn)
    g = (g.astype(np.float64) * 500.0 * np.array([1.0, 8.0])[:, None]).astype(np.float16)
    h = (h.astype(np.float64) * 2.0e-3 * np.array([1.0, 1.0 / 8.0])[:, None]).astype(np.float16)
    assert np.all(np.isfinite(g.astype(np.float64))) and np.count_nonzero(h) > 0.9 * h.size
    X = synth.outlier_activations(rng, T, inn)
    L = to_device_layer(signs, g, h)
    Y = rb.rb_linear_gemm(L, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    assert max_rel_l2(Y, oracle.forward(signs, g, h, X)) <= TOL


def test_gemm_rows_equal_single_token_calls():
    out, inn, T = 320, 1536, 70
    rng = synth.child_rng(5, 102)
    signs, g, h = random_layer(rng, 2, out, inn)
    X = synth.gaussian_activations(rng, T, inn)
    L = to_device_layer(signs, g, h)
    Xd = torch.from_numpy(X).cuda()
    Y = rb.rb_linear_gemm(L, Xd).cpu().numpy().astype(np.float64)
    for t in (0, 31, T - 1):
        yt = rb.rb_linear_gemv(L, Xd[t].contiguous())
        assert max_rel_l2(yt, Y[t][None]) <= 2e-3


@pytest.mark.parametrize("out,inn", [(28672, 8192), (8192, 28672)])
def test_prefill_70b_shapes_sampled(out, inn):
    """Config 5 at full size (T = 2048, bf16 activations, uniform signs drawn on the device in
    native order): 64 sampled outputs per call, each computed by the oracle from the unpacked
    row, plus two whole token rows of a 512-row slice."""
    T = 2048
    gen = torch.Generator(device="cuda"); gen.manual_seed(20260205 + out)
    nbytes = rb.rb_native_bytes(2, out, inn)
    bits = torch.randint(-2 ** 31, 2 ** 31 - 1, (nbytes // 4,), dtype=torch.int32, device="cuda", generator=gen)
    rng = synth.child_rng(5, 103, out)
    g = synth.halfnormal_scales(rng, 2, out); h = synth.halfnormal_scales(rng, 2, inn)
    g[1] *= np.float16(0.3); h[1] *= np.float16(0.3)
    L = rb.Layer(bits, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 2, out, inn)
    Xt = torch.randn((T, inn), device="cuda", generator=gen).to(torch.bfloat16)
    _say(f"prefill {out}x{inn} T={T}")
    Y = rb.rb_linear_gemm(L, Xt, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    # unpack the sampled rows on the host with the library's own (bit-exact, CPU-tested) unpacker
    native = bits.cpu().numpy().view(np.uint32)
    packed = rb.rb_unpack_native(native, 2, out, inn)
    signs_rows = lambda rows: rb.rb_unpack(packed[:, rows, :])
    pick = np.random.default_rng(7)
    rows = np.unique(pick.integers(0, out, size=64)); toks = pick.integers(0, T, size=len(rows))
    S = signs_rows(rows)                                            # [2][n][in]
    X64 = oracle.bf16_bits_to_f64(bf16_bits(Xt[torch.from_numpy(toks).cuda()].cpu())).reshape(len(rows), inn)
    ref = np.array([oracle.forward(S[:, i:i + 1, :], g[:, rows[i]:rows[i] + 1], h, X64[i:i + 1])[0, 0]
                    for i in range(len(rows))])
    got = Y[torch.from_numpy(toks).cuda(), torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    scale = np.sqrt(np.mean(ref ** 2))
    assert np.max(np.abs(got - ref)) <= 4 * TOL * scale, (np.max(np.abs(got - ref)), scale)
    # two whole token rows over a 512-row slice: per-vector relative L2 as everywhere else
    # (for 28672 rows also the last 512)
    for r0 in ([3 * 512, out - 512] if out >= 2048 * 2 else [0]):
        rows2 = np.arange(r0, r0 + 512)
        S2 = signs_rows(rows2)
        for t in (0, T - 1):
            x64 = oracle.bf16_bits_to_f64(bf16_bits(Xt[t:t + 1].cpu())).reshape(1, inn)
            ref2 = oracle.forward(S2, g[:, rows2], h, x64)
            err = max_rel_l2(Y[t:t + 1, r0:r0 + 512], ref2)
            _say(f"  rows {r0}.. t={t} rel_l2={err:.3e}")
            assert err <= TOL


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("out,inn,T,act,res,shift", [
    (40, 32, 65, "f16", "f16", 0),          # fewer rows than a wavefront's, one 32-column step, one token over a block
    (130, 160, 97, "bf16", "f32", 0),       # one row tile in the second workgroup, ragged rows stored one by one
    (1000, 2080, 333, "f16", "bf16", 1),    # column groups of unequal length; scales at an odd multiple of two bytes
    (4096, 288, 500, "bf16", "f16", 0),     # 128 x 64 tiles, last column tile nearly empty
    (8184, 384, 500, "f16", "f32", 0),      # 256 x 64
    (11008, 256, 333, "f16", "f16", 0),     # 256 x 96
    (8200, 256, 1025, "bf16", "bf16", 0),   # 256 x 128, one row and one token over
    # (the first three are few rows for the few-token kernel; the same edges on the many-token kernel)
    (2600, 32, 450, "f16", "f16", 0), (1291, 544, 900, "f16", "f16", 1), (4099, 288, 500, "bf16", "bf16", 0), (2003, 800, 700, "f16", "f32", 5),
    (4099, 2080, 333, "bf16", "f16", 7), (1303, 1056, 700, "f16", "bf16", 3),
])
def test_many_token_shapes(K, out, inn, T, act, res, shift):
    """Every shape of a workgroup of the many-token kernel at its edges, scales of either sign and zero.
    The bar: 1e-3 for results in fp16 and fp32; bf16 results round by up to 2^-9 of each value, 2^-9 / sqrt(3) in
    the mean, on top."""
    rng = synth.child_rng(5, 120, K, out, inn, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = g.copy(); h = h.copy()
    g[1, ::6] *= -1; h[0, ::3] *= -1; g[0, 3] = 0; h[1, 5] = 0
    X = synth.outlier_activations(rng, T, inn)
    _say(f"many-token K={K} out={out} in={inn} T={T} {act} -> {res} shift={shift}")
    L = to_device_layer(signs, g, h)
    if shift:
        store = torch.zeros(K * inn + shift, dtype=torch.float16, device="cuda")
        store[shift:] = L.h.flatten()
        L.h = store[shift:].view(K, inn)
        assert L.h.data_ptr() % 4 == 2
    if out in (2600, 1291, 4099, 2003, 1303):
        assert only_for_many_tokens(K, out, T, act == "bf16")
    Xd = torch.from_numpy(X).cuda()
    if act == "bf16":
        Xd = Xd.to(torch.bfloat16)
        X = oracle.bf16_bits_to_f64(bf16_bits(Xd.cpu())).reshape(T, inn)
    dtype = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[res]
    Y = torch.full((T + 1, out), 7.0, dtype=dtype, device="cuda")
    rb.rb_linear_gemm(L, Xd, Y=Y[:T])
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    assert torch.all(Y[T] == 7.0)
    err = max_rel_l2(Y[:T], oracle.forward(signs, g, h, X))
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL + (2.0 ** -9 / 3 ** 0.5 if res == "bf16" else 0.0)


@pytest.mark.parametrize("K,n,T", [(2, 544, 130), (2, 1312, 640), (3, 1312, 450)])
def test_many_token_output_over_its_input(K, n, T):
    """The output buffer may be the input buffer beyond 64 tokens (the input is moved to the workspace first); few rows, and two sizes of the
    many-token kernel."""
    assert n < 1000 or only_for_many_tokens(K, n, T)
    rng = synth.child_rng(5, 121)
    L = to_device_layer(*random_layer(rng, K, n, n))
    X = torch.from_numpy(synth.outlier_activations(rng, T, n)).cuda()
    want = rb.rb_linear_gemm(L, X)
    got = rb.rb_linear_gemm(L, X, Y=X)
    torch.cuda.synchronize()
    assert torch.equal(got, want)


@pytest.mark.parametrize("K,T", [(2, 70), (2, 500), (3, 70), (2, 800), (3, 600)])       # (the last two on the many-token kernel)
def test_gemm_small_scales_next_to_rows_without_a_path(K, T):
    """Output scales around 2e-5 (fp16 subnormals) and, in the first 512 rows, none for the last path: the power
    of two that lifts the other paths' scales into fp16's normal range must not come from the path that is zero there."""
    out, inn = 1100, 544
    rng = synth.child_rng(5, 122, K, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = (g.astype(np.float64) * 1e-3).astype(np.float16)
    g[K - 1, :512] = 0
    X = synth.outlier_activations(rng, T, inn)
    Xd = torch.from_numpy(X).cuda()
    _say(f"small scales, rows without a path, K={K} T={T}")
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), Xd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM
    ref = oracle.forward(signs, g, h, X)
    for rows in (slice(0, 512), slice(512, out)):
        err = max_rel_l2(Y[:, rows], ref[:, rows])
        _say(f"  rel_l2={err:.3e}")
        assert err <= TOL


@pytest.mark.parametrize("K,n,T,shift", [(2, 544, 70, 1), (3, 544, 70, 3), (2, 1056, 333, 5), (3, 4128, 200, 7), (2, 1312, 640, 1), (3, 1312, 450, 3)])
def test_many_token_scales_off_alignment(K, n, T, shift):
    """Scales that start at an odd multiple of two bytes are moved to the workspace: the same results as aligned ones, bit for
    bit, also when the output lies over the input and on the library's own scratch memory."""
    rng = synth.child_rng(5, 123, K, n, T)
    L = to_device_layer(*random_layer(rng, K, n, n))
    X = torch.from_numpy(synth.outlier_activations(rng, T, n)).cuda()
    want = rb.rb_linear_gemm(L, X)
    store = torch.zeros(K * n + shift, dtype=torch.float16, device="cuda")
    store[shift:] = L.h.flatten()
    L.h = store[shift:].view(K, n)
    _say(f"scales off alignment K={K} {n}x{n} T={T} shift={shift}")
    assert torch.equal(rb.rb_linear_gemm(L, X), want)
    Y = X.clone()
    assert torch.equal(rb.rb_linear_gemm(L, Y, Y=Y), want)
    Y = X.clone()
    assert torch.equal(rb.rb_linear_gemm_noalloc(L, Y, Y), want)


@pytest.mark.parametrize("K,T,case", [(2, 700, "none"), (2, 1100, "small"), (3, 700, "none"), (3, 900, "small"), (2, 700, "inputs"), (3, 700, "outlier")])
def test_gemm_rows_whose_first_path_is_small_or_missing(K, T, case):
    """A row may be built as path 0 plus multiples of it: rows where path 0 has no output scale or one 1e-3 to 1e-6 of the others', layers where it
    has no input scales or one a thousand times the rest, either sign.  Each group of rows by itself against the oracle, fp32 results: two
    roundings to fp16 per weight (2^-12 of it each) stay below 1e-3."""
    out, inn = 1300, 544                                       # (too many tiles of 64 tokens for the few-token kernel)
    rng = synth.child_rng(5, 124, K, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = (g.astype(np.float64) * 20).astype(np.float16)
    g[:, ::3] *= -1; h[1, ::5] *= -1
    groups = [slice(0, 200), slice(200, 600), slice(600, out)]
    if case == "none":
        g[0, groups[0]] = 0
        g[:, 1290:] = 0
    elif case == "small":
        g[0, groups[0]] = (g[0, groups[0]].astype(np.float64) * 1e-6).astype(np.float16)
        g[0, groups[1]] = (g[0, groups[1]].astype(np.float64) * 1e-3).astype(np.float16)
    elif case == "inputs":
        h[0] = 0
    else:
        h[0, 17] *= np.float16(1000)
    X = synth.outlier_activations(rng, T, inn)
    _say(f"first path {case}, K={K} T={T}")
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), torch.from_numpy(X).cuda(), out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.forward(signs, g, h, X)
    for rows in groups:
        err = max_rel_l2(Y[:, rows], ref[:, rows])
        _say(f"  rel_l2={err:.3e}")
        assert err <= TOL
    if case == "none":
        assert torch.all(Y[:, 1290:] == 0)


@pytest.mark.parametrize("K,inn,T,case", [(2, 2080, 700, "outlier"), (3, 2080, 700, "outlier"), (2, 11008, 700, "one column"), (2, 1056, 900, "infinite"),
                                          (2, 544, 1100, "spread"), (3, 544, 900, "spread")])
def test_gemm_rows_that_the_first_path_does_not_carry(K, inn, T, case):
    """The second path's input scales are uneven where the first path has no output scale, one 1e-3 or 0.05 of the others', or a usual
    one, in groups of rows that share workgroups: one scale a thousand times the rest where the activations are a thousandth, or one scale
    only, which leaves the row a single product; scales spread over e^-3 .. e^3; an infinite scale, whose column alone is not finite.
    fp32 results, each group of rows by itself: as many roundings to fp16 per weight as paths (2^-12 of it each, and the largest error of a row of
    several hundred no more than twice the mean) stay below 1e-3."""
    out = 1300                                                 # (too many tiles of 64 tokens for the few-token kernel)
    rng = synth.child_rng(5, 127, K, inn, T)
    signs, g, h = random_layer(rng, K, out, inn)
    g = (np.sign(g.astype(np.float64)) * (0.2 + np.abs(g.astype(np.float64)) * 20)).astype(np.float16)
    h = (0.02 + np.abs(h.astype(np.float64))).astype(np.float16)
    g[:, ::3] *= -1; h[1, ::5] *= -1
    groups = [slice(0, 100), slice(100, 200), slice(200, 230), slice(230, out)]
    for rows, f in zip(groups, (0.0, 1e-3, 0.05, 1.0)):
        g[0, rows] = (g[0, rows].astype(np.float64) * f).astype(np.float16)
    X = synth.outlier_activations(rng, T, inn)
    if case == "outlier":
        h[1, 17] *= np.float16(1000)
        X[:, 17] *= np.float16(1e-3)
    elif case == "one column":
        g[2:] = 0
        g[0, 230:] = 0
        h[1, :17] = 0; h[1, 18:] = 0
    elif case == "spread":
        g = (g.astype(np.float64) * np.exp(rng.standard_normal(g.shape))).astype(np.float16)
        h = (h.astype(np.float64) * np.exp(rng.standard_normal(h.shape))).astype(np.float16)
    else:
        h[1, 17] = np.inf
    _say(f"first path carries not every row, {case}, K={K} in={inn} T={T}")
    Y = rb.rb_linear_gemm(to_device_layer(signs, g, h), torch.from_numpy(X).cuda(), out_dtype=torch.float32)
    torch.cuda.synchronize()
    if case == "infinite":
        assert not torch.any(torch.isfinite(Y[torch.from_numpy(X[:, 17] != 0).cuda()]))
        return
    ref = oracle.forward(signs, g, h, X)
    for rows in groups:
        if case == "one column" and not np.any(ref[:, rows]):
            assert torch.all(Y[:, rows] == 0)
            continue
        got, want = Y[:, rows].cpu().numpy().astype(np.float64), ref[:, rows]
        err = np.sqrt(((got - want) ** 2).sum(0) / (want ** 2).sum(0))         # row by row, over the tokens
        _say(f"  rel_l2={np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum()):.3e} worst row {err.max():.3e}")
        assert err.max() <= TOL


@pytest.mark.parametrize("K,out,inn,T,bf16", [(2, 1290, 800, 700, False), (2, 2600, 96, 1025, True), (3, 1400, 1056, 800, True), (3, 1300, 544, 641, False),
                                              (2, 4100, 2080, 333, False), (2, 5000, 288, 1000, False)])
def test_many_token_kernel_at_ragged_sizes(K, out, inn, T, bf16):
    """Sizes at which calls of more than 64 tokens take the many-token kernel, whose weights are rounded to fp16 (as many roundings as paths, 2^-12 of
    a weight each): within 1e-3 of the oracle."""
    assert only_for_many_tokens(K, out, T, bf16)
    rng = synth.child_rng(5, 125, K, out, inn, T)
    host = random_layer(rng, K, out, inn)
    X = synth.gaussian_activations(rng, T, inn)
    Xd = torch.from_numpy(X).cuda()
    if bf16:
        Xd = Xd.to(torch.bfloat16)
        X = oracle.bf16_bits_to_f64(bf16_bits(Xd.cpu())).reshape(T, inn)
    _say(f"many-token kernel K={K} {out}x{inn} T={T} bf16={bf16}")
    Y = rb.rb_linear_gemm(to_device_layer(*host), Xd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    err = max_rel_l2(Y, oracle.forward(*host, X))
    _say(f"  rel_l2={err:.3e}")
    assert err <= TOL


@pytest.mark.parametrize("K,out,inn,T,bf16", [(2, 300, 800, 65, False), (2, 1000, 2080, 333, True), (3, 700, 1056, 200, False), (2, 33, 4128, 1000, False),
                                              (3, 16, 96, 4097, True), (2, 4100, 544, 100, False)])
def test_many_tokens_of_few_rows(K, out, inn, T, bf16):
    """Few tiles: 64 tokens per workgroup on the few-token kernel.  Its products are exact (fp32 results within 1e-5 of the
    oracle), and every 64 tokens are what a call of their own gives, bit for bit."""
    rng = synth.child_rng(5, 126, K, out, inn, T)
    host = random_layer(rng, K, out, inn)
    L = to_device_layer(*host)
    X = synth.outlier_activations(rng, T, inn)
    Xd = torch.from_numpy(X).cuda()
    if bf16:
        Xd = Xd.to(torch.bfloat16)
        X = oracle.bf16_bits_to_f64(bf16_bits(Xd.cpu())).reshape(T, inn)
    _say(f"few rows K={K} {out}x{inn} T={T} bf16={bf16}")
    Y = torch.full((T + 1, out), 7.0, dtype=torch.float32, device="cuda")
    rb.rb_linear_gemm(L, Xd, Y=Y[:T])
    torch.cuda.synchronize()
    assert rb.rb_last_path() == rb.RB_PATH_GEMM and torch.all(Y[T] == 7.0)
    assert max_rel_l2(Y[:T], oracle.forward(*host, X)) <= 1e-5
    for t in range(0, T - 63, 64 * 7):
        assert torch.equal(rb.rb_linear_gemm(L, Xd[t:t + 64].contiguous(), out_dtype=torch.float32), Y[t:t + 64])
