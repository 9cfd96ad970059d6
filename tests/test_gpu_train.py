"""Training-side kernels against the oracle: the coupled derivation of the binary cores (bit-exact:
the residual's precision is part of the definition) and the gradients of the scales."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2602_05367_amd as rb

pytestmark = pytest.mark.gpu


def _scales(rng, K, n, scale):
    return (np.abs(rng.standard_normal((K, n))) * scale * (0.6 ** np.arange(K))[:, None]).astype(np.float16)


@pytest.mark.parametrize("K,out,inn", [(1, 7, 32), (2, 37, 96), (3, 130, 544), (2, 272, 1056), (2, 1024, 4096)])
def test_couple_bits_and_residual_are_the_oracles(K, out, inn):
    rng = synth.child_rng(5, 600, K, out)
    W = synth.gaussian_weight(rng, out, inn, std=1.0).astype(np.float32)
    W[0, :5] = 0.0                                            # sign(0) = +1
    g, h = _scales(rng, K, out, 0.9), _scales(rng, K, inn, 0.9)
    signs, R = oracle.couple(W, g, h)
    print(f"couple K={K} {out}x{inn}", flush=True)
    packed, native, residual = rb.rb_couple(torch.from_numpy(W).cuda(), torch.from_numpy(g).cuda(),
                                            torch.from_numpy(h).cuda(), want_native=True, want_residual=True)
    torch.cuda.synchronize()
    ref_packed = oracle.pack(signs)
    got_packed = packed.cpu().numpy().view(np.uint32)
    assert np.array_equal(got_packed, ref_packed)
    # the native tiles are what the host repacker makes of the canonical words, padding included
    assert np.array_equal(native.cpu().numpy().view(np.uint32), rb.rb_repack_native(ref_packed))
    assert np.array_equal(residual.cpu().numpy(), R)          # same roundings, bit for bit
    # packed only, native only
    p2, n2, r2 = rb.rb_couple(torch.from_numpy(W).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(),
                              want_native=False)
    assert n2 is None and r2 is None and torch.equal(p2, packed)


def test_coupled_cores_run_through_the_inference_kernels():
    """A training step's forward pass: derive the cores on the device, feed the native tiles to the
    decode kernel, compare with the oracle's forward on the oracle's cores."""
    rng = synth.child_rng(5, 601)
    out, inn, K = 528, 1056, 2
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    _, g, h, _ = oracle.derive(W, K)
    signs, _ = oracle.couple(W, g, h)
    x = synth.gaussian_activations(rng, 1, inn)
    gd, hd = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    _, native, _ = rb.rb_couple(torch.from_numpy(W).cuda(), gd, hd)
    L = rb.Layer(native, gd, hd, K, out, inn)
    y = rb.rb_linear_gemv(L, torch.from_numpy(x[0]).cuda())
    torch.cuda.synchronize()
    ref = oracle.forward(signs, g, h, x)
    assert oracle.relative_l2(y.cpu().numpy().astype(np.float64)[None], ref).max() <= 1e-3


@pytest.mark.parametrize("K,out,inn,N", [(1, 5, 32, 1), (2, 37, 96, 3), (3, 130, 544, 4), (2, 300, 1056, 7)])
def test_scale_gradients_against_the_oracle(K, out, inn, N):
    """fp32 sums of out or in terms against fp64: 1e-5 relative to the gradient's norm (the bound
    for recursive fp32 summation of a few thousand terms of mixed sign is ~n * 2^-24 of the sum of
    magnitudes; the measured error is an order below)."""
    rng = synth.child_rng(5, 602, K, out)
    signs = synth.uniform_signs(rng, K, out, inn)
    g, h = _scales(rng, K, out, 0.5), _scales(rng, K, inn, 0.5)
    X = synth.gaussian_activations(rng, N, inn)
    D = (rng.standard_normal((N, out)) * 0.1).astype(np.float16)
    ref_g, ref_h = oracle.scale_grads(signs, g, h, X, D)
    print(f"scale gradients K={K} {out}x{inn} N={N}", flush=True)
    G = rb.rb_weight_grad(torch.from_numpy(D).cuda(), torch.from_numpy(X).cuda())
    packed = torch.from_numpy(oracle.pack(signs).view(np.int32)).cuda()
    gg, gh = rb.rb_scale_grads(G, packed, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda())
    gg2, gh2 = rb.rb_scale_grads(G, packed, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda())
    torch.cuda.synchronize()
    assert torch.equal(gg, gg2) and torch.equal(gh, gh2)      # fixed summation order
    refG = oracle.weight_grad(D, X)
    assert np.abs(G.cpu().numpy() - refG).max() <= 1e-5 * np.abs(refG).max()
    for got, ref in ((gg, ref_g), (gh, ref_h)):
        err = np.linalg.norm(got.cpu().numpy().astype(np.float64) - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= 1e-5, err


@pytest.mark.parametrize("N,out,inn,shift", [
    (1, 128, 256, 0), (31, 124, 252, 0), (33, 132, 260, 0), (64, 129, 255, 0),      # around one tile of G and one step of samples
    (65, 300, 1056, 1), (40, 4, 32, 0), (7, 1, 1, 0), (100, 64, 2052, 3)])           # pointers at odd elements, tiny and wide
def test_weight_gradient_tiles_and_tails(N, out, inn, shift):
    """Every element of G against fp64.  Bound: products of two fp16 values are exact in fp32, so only
    the N additions round: |error| <= N 2^-23 sum_n |Delta| |X| (twice the half-ulp bound, for an
    accumulator that truncates).  One sample in four has Delta in the fp16 subnormals.  Nothing
    outside G is written."""
    rng = synth.child_rng(5, 603, N, out, inn)
    X = synth.outlier_activations(rng, N, inn)
    D = rng.standard_normal((N, out)) * 0.1
    D[::4] *= 1e-4
    D = D.astype(np.float16)

    def at(a, shift):                                          # `a` in device memory, `shift` elements past an aligned address
        flat = torch.zeros(a.size + shift, dtype=torch.float16, device="cuda")
        flat[shift:].copy_(torch.from_numpy(a).flatten())
        return flat
    Dd, Xd = at(D, shift), at(X, shift)
    G = torch.full((out * inn + 64,), float("nan"), dtype=torch.float32, device="cuda")
    print(f"weight gradient {out}x{inn} N={N} shift={shift}", flush=True)
    assert rb.lib.rb_weight_grad(Dd.data_ptr() + 2 * shift, Xd.data_ptr() + 2 * shift, N, out, inn, G.data_ptr(), None) == rb.RB_OK
    torch.cuda.synchronize()
    assert torch.isnan(G[out * inn:]).all()
    D64, X64 = D.astype(np.float64), X.astype(np.float64)
    err = np.abs(G[:out * inn].cpu().numpy().reshape(out, inn) - D64.T @ X64)
    assert np.all(err <= N * 2.0 ** -23 * (np.abs(D64).T @ np.abs(X64)))


@pytest.mark.parametrize("N,out,inn,shift", [
    # one to seven steps of 32 samples, whole and part-filled; rows of Delta that start at multiples of 2 and 4 bytes, last rows of one to
    # three columns, fewer rows than a tile
    (1, 4, 32, 0), (32, 131, 288, 0), (65, 5, 64, 0), (96, 258, 64, 0), (97, 777, 96, 0), (128, 132, 96, 0), (129, 133, 96, 0),
    (160, 256, 96, 0), (161, 257, 32, 4), (193, 6, 256, 0), (224, 384, 32, 0)])
def test_weight_gradient_steps_and_unaligned_rows(N, out, inn, shift):
    test_weight_gradient_tiles_and_tails(N, out, inn, shift)


@pytest.mark.parametrize("N,out,inn", [(33, 4, 2 ** 23), (1, 5, 2 ** 23 + 4), (65, 12, 2 ** 23 + 260)])
def test_weight_gradient_of_very_wide_layers(N, out, inn):
    """From 2^23 columns on 32 rows of X are beyond the offsets of a buffer: loads of eight bytes where rows are aligned, of two
    where those of Delta are not.  Bound as in test_weight_gradient_tiles_and_tails; the reference is fp64 on the device."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    X = torch.randn((N, inn), device="cuda", generator=gen).half()
    D = (torch.randn((N, out), device="cuda", generator=gen) * 0.1).half()
    print(f"weight gradient {out}x{inn} N={N}", flush=True)
    G = rb.rb_weight_grad(D, X)
    for c in range(0, inn, 2 ** 20):
        x = X[:, c:c + 2 ** 20].double()
        err = (G[:, c:c + 2 ** 20].double() - D.double().t() @ x).abs()
        assert torch.all(err <= N * 2.0 ** -23 * (D.double().abs().t() @ x.abs())), c


@pytest.mark.parametrize("K,out,inn", [(1, 200, 288), (2, 129, 544), (3, 65, 1056)])
def test_scale_gradients_of_part_filled_slices(K, out, inn):
    test_scale_gradients_against_the_oracle(K, out, inn, 3)


@pytest.mark.parametrize("K,out,inn", [(1, 9, 32), (2, 70, 288), (3, 129, 1056)])
def test_scale_gradients_with_an_infinite_scale(K, out, inn):
    """An infinite scale among the first four columns of the first path: its rows' sums are infinite, with the sign of their term, and every
    other gradient is what it is without it.  Columns past the last one must not bring it in a second time."""
    rng = synth.child_rng(5, 605, K, out, inn)
    signs = synth.uniform_signs(rng, K, out, inn)
    G = rng.standard_normal((out, inn)).astype(np.float32)
    G[3] = -np.abs(G[3])
    g, h = synth.halfnormal_scales(rng, K, out), synth.halfnormal_scales(rng, K, inn)
    dev = [torch.from_numpy(a).cuda() for a in (G, rb.rb_pack(signs).view(np.int32), g, h)]
    print(f"scale gradients with an infinite scale K={K} {out}x{inn}", flush=True)
    want_g, want_h = rb.rb_scale_grads(*dev)
    dev[3][0, 2] = float("inf")
    got_g, got_h = rb.rb_scale_grads(*dev)
    torch.cuda.synchronize()
    assert torch.equal(got_h, want_h) and torch.equal(got_g[1:], want_g[1:])
    assert np.array_equal(got_g[0].cpu().numpy(), np.inf * signs[0, :, 2] * np.sign(G[:, 2]))


def test_training_entry_points_reject_bad_arguments():
    W = torch.zeros((4, 32), dtype=torch.float32, device="cuda")
    g = torch.zeros((2, 4), dtype=torch.float16, device="cuda")
    h = torch.zeros((2, 32), dtype=torch.float16, device="cuda")
    out = torch.zeros((2, 4, 1), dtype=torch.int32, device="cuda")
    lib = rb.lib
    assert lib.rb_couple(W.data_ptr(), g.data_ptr(), h.data_ptr(), 2, 4, 32, None, None, None, None) == rb.RB_ERR_NULL
    assert lib.rb_couple(None, g.data_ptr(), h.data_ptr(), 2, 4, 32, out.data_ptr(), None, None, None) == rb.RB_ERR_NULL
    assert lib.rb_couple(W.data_ptr(), g.data_ptr(), h.data_ptr(), 4, 4, 32, out.data_ptr(), None, None, None) == rb.RB_ERR_SHAPE
    assert lib.rb_couple(W.data_ptr(), g.data_ptr(), h.data_ptr(), 2, 4, 33, out.data_ptr(), None, None, None) == rb.RB_ERR_SHAPE
    # the kernels read W sixteen and h eight bytes at a time
    assert lib.rb_couple(W.data_ptr() + 4, g.data_ptr(), h.data_ptr(), 2, 3, 32, out.data_ptr(), None, None, None) == rb.RB_ERR_ALIGN
    assert lib.rb_couple(W.data_ptr(), g.data_ptr(), h.data_ptr() + 2, 1, 4, 32, out.data_ptr(), None, None, None) == rb.RB_ERR_ALIGN
    assert lib.rb_scale_grads(W.data_ptr(), out.data_ptr(), g.data_ptr(), h.data_ptr(), 2, 4, 32, W.data_ptr(), W.data_ptr(),
                              None, 0, None) == rb.RB_ERR_WORKSPACE
    assert lib.rb_scale_grads_workspace_bytes(2, 4, 31) == 0


def test_coupling_of_very_long_rows():
    """More chunks of 512 columns than a grid's second dimension may have (65536)."""
    K, out, inn = 1, 3, 65536 * 512 + 4128
    gen = torch.Generator(device="cuda")
    gen.manual_seed(604)
    W = torch.randn((out, inn), device="cuda", generator=gen) * 0.02
    g, h = torch.full((K, out), 0.1, device="cuda").half(), torch.full((K, inn), 0.1, device="cuda").half()
    print(f"couple {out}x{inn}", flush=True)
    packed, native, _ = rb.rb_couple(W, g, h)
    torch.cuda.synchronize()
    packed = packed.cpu().numpy().view(np.uint32)
    assert np.array_equal(packed[0], np.packbits((W < 0).cpu().numpy(), axis=1, bitorder="little").view(np.uint32))
    assert np.array_equal(rb.rb_unpack_native(native.cpu().numpy().view(np.uint32), K, out, inn), packed)
