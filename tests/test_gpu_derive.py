"""Alg. 1 on the device (rb_derive_iterative) against the oracle's derive_iterative: both sides
decide the signs in fp64, so the stored bits must agree; scales and errors agree to what the
different summation orders leave."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2602_05367_amd as rb

pytestmark = pytest.mark.gpu


def _factors(rng, out, inn, alpha_in, alpha_out):
    s_in = np.abs(rng.standard_normal(inn)) + 0.1
    s_out = np.abs(rng.standard_normal(out)) + 0.1
    rows = (s_out / s_out.max()) ** alpha_out
    cols = (s_in / s_in.max()) ** alpha_in
    return s_in, s_out, rows, cols


def _run(W, K, T_max, rows=None, cols=None):
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()
    packed, g, h, err = rb.rb_derive_iterative(torch.from_numpy(W).cuda(), K, T_max, dev(rows), dev(cols))
    torch.cuda.synchronize()
    return packed.cpu().numpy().view(np.uint32), g.cpu().numpy(), h.cpu().numpy(), err.cpu().numpy()


@pytest.mark.parametrize("K,out,inn,T_max,calibrated", [
    (1, 7, 32, 2, False), (2, 37, 96, 4, True), (3, 130, 544, 3, True), (2, 300, 1056, 3, False), (2, 1024, 2048, 2, True)])
def test_iterative_svid_matches_the_oracle(K, out, inn, T_max, calibrated):
    rng = synth.child_rng(7, 700, K, out)
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    W[0, :3] = 0.0
    print(f"derive K={K} {out}x{inn} T_max={T_max} calibrated={calibrated}", flush=True)
    if calibrated:
        s_in, s_out, rows, cols = _factors(rng, out, inn, 0.5, 0.25)
        signs, g, h, err = oracle.derive_iterative(W, K, T_max, s_in=s_in, s_out=s_out, alpha_in=0.5, alpha_out=0.25)
        got = _run(W, K, T_max, rows, cols)
    else:
        signs, g, h, err = oracle.derive_iterative(W, K, T_max)
        got = _run(W, K, T_max)
    packed, g_d, h_d, err_d = got
    ref_packed = oracle.pack(signs)
    differing = int(np.unpackbits((packed ^ ref_packed).view(np.uint8)).sum())
    assert differing == 0, f"{differing} of {signs.size} signs differ"
    np.testing.assert_allclose(g_d, g, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(h_d, h, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(err_d, err, rtol=1e-9)
    # and what the method promises: every update lowers the error
    flat = err_d.reshape(-1)
    assert np.all(np.diff(flat) <= 1e-12 * flat[0])


def test_one_sweep_is_the_greedy_pass():
    """T_max = 1 against the oracle's greedy derivation, a function of its own."""
    rng = synth.child_rng(7, 701)
    W = synth.gaussian_weight(rng, 272, 544, std=0.02).astype(np.float32)
    signs, g, h, norms = oracle.derive(W, 3, round_scales=False)
    packed, g_d, h_d, err_d = _run(W, 3, 1)
    assert np.array_equal(packed, oracle.pack(signs))
    np.testing.assert_allclose(g_d, g, rtol=1e-8)
    np.testing.assert_allclose(h_d, h, rtol=1e-8)
    np.testing.assert_allclose(err_d[0], norms[1:], rtol=1e-9)
    # residual fractions of a Gaussian weight: 1 - 2/pi, 0.130, 0.058
    frac = (norms[1:] / norms[0]) ** 2
    assert abs(frac[0] - (1 - 2 / np.pi)) < 0.01 and abs(frac[1] - 0.130) < 0.01 and abs(frac[2] - 0.058) < 0.01


# (two passes per iteration; one reading of W; three paths of more columns than the pass after the iteration takes)
@pytest.mark.parametrize("K,zero,out,inn", [(2, (20, 64), 48, 96), (2, (1024, 2080), 1030, 4128), (3, (1024, 8224), 1024, 8224)])
def test_degenerate_weights(K, zero, out, inn):
    # all zero: no scale, every sign +1
    print(f"derive K={K} of zeros {zero}, of one path {out}x{inn}", flush=True)
    packed, g, h, err = _run(np.zeros(zero, dtype=np.float32), K, 2)
    assert not packed.any() and not g.any() and not h.any() and not err.any()
    # a weight that is one path exactly: found in the first update, nothing left for the second
    rng = synth.child_rng(7, 702)
    B = synth.uniform_signs(rng, 1, out, inn)[0].astype(np.float64)
    g0, h0 = np.abs(rng.standard_normal(out)) + 0.5, np.abs(rng.standard_normal(inn)) + 0.5
    W = (g0[:, None] * B * h0[None, :]).astype(np.float32)
    packed, g, h, err = _run(W, K, 1)
    assert np.array_equal(packed[0], oracle.pack(B[None].astype(np.int8))[0])
    np.testing.assert_allclose(g[0][:, None] * h[0][None, :], np.abs(W.astype(np.float64)), rtol=1e-6)
    assert err[0, 0] <= 1e-6 * np.linalg.norm(W) and err[0, 1] <= err[0, 0]


def test_derived_paths_run_through_the_inference_kernel():
    """Initialise on the device, round the scales to fp16, tile the signs, run a token: the
    oracle's forward on the oracle's own initialisation must agree."""
    rng = synth.child_rng(7, 703)
    out, inn, K = 528, 1056, 2
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    signs, g, h, _ = oracle.derive_iterative(W, K, 3)
    packed, g_d, h_d, _ = _run(W, K, 3)
    g16, h16 = g_d.astype(np.float16), h_d.astype(np.float16)
    assert np.array_equal(g16, g.astype(np.float16)) and np.array_equal(h16, h.astype(np.float16))
    native = torch.from_numpy(rb.rb_repack_native(packed).view(np.int32)).cuda()
    L = rb.Layer(native, torch.from_numpy(g16).cuda(), torch.from_numpy(h16).cuda(), K, out, inn)
    x = synth.gaussian_activations(rng, 1, inn)
    y = rb.rb_linear_gemv(L, torch.from_numpy(x[0]).cuda())
    torch.cuda.synchronize()
    ref = oracle.forward(signs, g.astype(np.float16), h.astype(np.float16), x)
    assert oracle.relative_l2(y.cpu().numpy().astype(np.float64)[None], ref).max() <= 1e-3


def test_full_size_layer_as_benchmarked_last_update_against_the_oracle():
    """4096 x 11008, K = 2, the size bench.py times.  The oracle cannot run the whole iteration at
    this size in test time, but the last update of the last sweep is an SVID of one residual that
    numpy can form from what the device returned for the other path: its signs must be the stored
    bits of path 2, the oracle's leading singular pair of its magnitudes the stored scales, and the
    remaining error the last entry of the error table.  The errors must fall from update to update
    and start at the greedy values of a Gaussian weight (residual fractions 1 - 2/pi and 0.130)."""
    out, inn, K, T_max = 4096, 11008, 2, 2
    W = (torch.randn((out, inn), device="cuda", generator=torch.Generator(device="cuda").manual_seed(7)) * 0.02)
    print("derive 4096x11008 on the device", flush=True)
    packed, g, h, err = rb.rb_derive_iterative(W, K, T_max)
    torch.cuda.synchronize()
    Wh = W.cpu().numpy().astype(np.float64)
    packed, g, h, err = packed.cpu().numpy().view(np.uint32), g.cpu().numpy(), h.cpu().numpy(), err.cpu().numpy()
    norm = np.linalg.norm(Wh)
    flat = err.reshape(-1)
    assert np.all(np.diff(flat) < 0)
    assert abs((flat[0] / norm) ** 2 - (1 - 2 / np.pi)) < 0.003 and abs((flat[1] / norm) ** 2 - 0.130) < 0.003
    print("  residual of path 2 in numpy", flush=True)
    B0 = oracle.unpack(packed[0:1])[0]
    R = Wh - g[0][:, None] * B0 * h[0][None, :]
    del B0
    B1 = oracle.sign(R)
    differing = int(np.unpackbits((oracle.pack(B1[None]) ^ packed[1:2]).view(np.uint8)).sum())
    assert differing == 0, differing
    sigma, a, b = oracle.leading_singular_pair(np.abs(R))
    np.testing.assert_allclose(g[1], np.sqrt(sigma) * a, rtol=1e-8)
    np.testing.assert_allclose(h[1], np.sqrt(sigma) * b, rtol=1e-8)
    left = np.linalg.norm(R - g[1][:, None] * B1 * h[1][None, :])
    np.testing.assert_allclose(flat[-1], left, rtol=1e-9)


@pytest.mark.parametrize("K,out,inn,slices_of", [(2, 70, 1056, 32), (2, 70, 1056, 64), (1, 5, 32, 32), (3, 33, 2080, 64)])
def test_slices_of_the_column_pass_and_their_workspace(K, out, inn, slices_of):
    """Ragged rows and columns of both passes (four rows, 1024 columns, 64 columns of the sums); a workspace that holds
    slices of 64 rows only is enough.  Same bars as above."""
    rng = synth.child_rng(7, 705, K, out, slices_of)
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    signs, g, h, err = oracle.derive_iterative(W, K, 2)
    need = rb.lib.rb_derive_workspace_bytes(out, inn)
    if slices_of == 64:
        need -= (-(-out // 32) - -(-out // 64)) * inn * 8 - 256          # (sizes are rounded to 256 bytes)
    Wd = torch.from_numpy(W).cuda()
    packed = torch.empty((K, out, inn // 32), dtype=torch.int32, device="cuda")
    gd, hd = (torch.empty((K, n), dtype=torch.float64, device="cuda") for n in (out, inn))
    ed = torch.empty((2, K), dtype=torch.float64, device="cuda")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    print(f"derive K={K} {out}x{inn}, slices of {slices_of} rows", flush=True)
    rc = rb.lib.rb_derive_iterative(Wd.data_ptr(), None, None, K, 2, out, inn, packed.data_ptr(), gd.data_ptr(), hd.data_ptr(),
                                    ed.data_ptr(), ws.data_ptr(), need, None)
    torch.cuda.synchronize()
    assert rc == rb.RB_OK
    assert np.array_equal(packed.cpu().numpy().view(np.uint32), oracle.pack(signs))
    np.testing.assert_allclose(gd.cpu().numpy(), g, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(hd.cpu().numpy(), h, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(ed.cpu().numpy(), err, rtol=1e-9)


@pytest.mark.parametrize("K,out,inn,calibrated,slow", [
    # one reading of W per iteration: from 1024 rows and 2048 columns to 12288 columns, 2, 4 and 6 groups of 2048; rows that 256 workgroups do
    # not share evenly, groups that end inside a workgroup
    (1, 1024, 2048, True, False), (2, 1030, 4096, False, False), (2, 1025, 4128, True, False), (3, 1024, 6176, True, False),
    (2, 1100, 8224, True, False), (1, 1027, 12288, False, False), (3, 1024, 8288, False, False),
    (1, 1024, 4160, True, False), (3, 1027, 2080, True, False),
    # many more iterations than the host enqueues before it looks: it looks, and goes on, after each
    (1, 1026, 2080, False, True), (2, 1024, 4128, True, True)])
def test_both_passes_in_one_reading(K, out, inn, calibrated, slow):
    """Same bars as above; and the workspace that two passes per iteration need is still enough, with the same signs and, but for
    the order of the sums, the same scales."""
    rng = synth.child_rng(7, 709, K, out)
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    W[0, :3] = 0.0
    if slow:                                                   # two blocks whose leading singular values are a factor of 1.5 apart
        W[:out // 2, inn // 2:] *= 1e-3
        W[out // 2:, :inn // 2] *= 1e-3
        W[out // 2:, inn // 2:] *= 1.5
    print(f"derive K={K} {out}x{inn} calibrated={calibrated}", flush=True)
    s_in, s_out, rows, cols = _factors(rng, out, inn, 0.5, 0.25)
    if not calibrated:
        rows = cols = None
    signs, g, h, err = oracle.derive_iterative(W, K, 2, **(dict(s_in=s_in, s_out=s_out, alpha_in=0.5, alpha_out=0.25) if calibrated else {}))
    packed, g_d, h_d, err_d = _run(W, K, 2, rows, cols)
    assert np.array_equal(packed, oracle.pack(signs))
    np.testing.assert_allclose(g_d, g, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(h_d, h, rtol=1e-8, atol=1e-14)
    np.testing.assert_allclose(err_d, err, rtol=1e-9)
    need = rb.lib.rb_derive_workspace_bytes(out, inn) - (257 - -(-out // 32)) * inn * 8
    Wd = torch.from_numpy(W).cuda()
    rd, cd = (None if a is None else torch.from_numpy(a).cuda() for a in (rows, cols))
    pd = torch.empty((K, out, inn // 32), dtype=torch.int32, device="cuda")
    gd, hd = (torch.empty((K, n), dtype=torch.float64, device="cuda") for n in (out, inn))
    ed = torch.empty((2, K), dtype=torch.float64, device="cuda")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    at = lambda t: None if t is None else t.data_ptr()
    rc = rb.lib.rb_derive_iterative(Wd.data_ptr(), at(rd), at(cd), K, 2, out, inn, pd.data_ptr(), gd.data_ptr(), hd.data_ptr(), ed.data_ptr(),
                                    ws.data_ptr(), need, None)
    torch.cuda.synchronize()
    assert rc == rb.RB_OK and np.array_equal(pd.cpu().numpy().view(np.uint32), packed)
    np.testing.assert_allclose(gd.cpu().numpy(), g_d, rtol=1e-9, atol=1e-14)
    np.testing.assert_allclose(hd.cpu().numpy(), h_d, rtol=1e-9, atol=1e-14)
    np.testing.assert_allclose(ed.cpu().numpy(), err_d, rtol=1e-12)


@pytest.mark.parametrize("K,out,inn,kind", [(1, 1024, 2048, "gaussian"), (2, 1030, 8224, "gaussian"), (3, 1024, 4160, "gaussian"), (2, 1024, 4128, "slow"),
                                            (2, 1024, 2080, "zero"), (3, 1024, 2048, "signs")])
def test_updates_one_after_the_other_without_the_host(K, out, inn, kind):
    """However many passes the host has asked for when it looks (one sweep of four iterations each; a sweep of many more; updates that end at
    once: |R| zero or of equal entries, after which all further residuals are zero), the updates are the same: T sweeps begin with what
    one sweep gives, bit for bit, and the last scales are those of T sweeps with no errors asked for."""
    W = synth.gaussian_weight(synth.child_rng(7, 713, K, out), out, inn, std=0.02).astype(np.float32)
    if kind == "slow":
        W[:out // 2, inn // 2:] *= 1e-3
        W[out // 2:, :inn // 2] *= 1e-3
        W[out // 2:, inn // 2:] *= 1.5
    elif kind == "zero":
        W[:] = 0.0
    elif kind == "signs":
        W = np.where(W >= 0, np.float32(0.25), np.float32(-0.25))
    print(f"derive K={K} {out}x{inn} {kind}", flush=True)
    one = _run(W, K, 1)
    packed, g, h, err = _run(W, K, 7)
    assert np.array_equal(err[:1], one[3]) and np.isfinite(err).all()
    assert np.all(np.diff(err.reshape(-1)) <= 1e-12 * np.linalg.norm(W.astype(np.float64)))
    Wd = torch.from_numpy(W).cuda()
    for T, want in ((1, one), (7, (packed, g, h))):
        pd = torch.empty((K, out, inn // 32), dtype=torch.int32, device="cuda")
        gd, hd = (torch.empty((K, n), dtype=torch.float64, device="cuda") for n in (out, inn))
        need = rb.lib.rb_derive_workspace_bytes(out, inn)
        ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        assert rb.lib.rb_derive_iterative(Wd.data_ptr(), None, None, K, T, out, inn, pd.data_ptr(), gd.data_ptr(), hd.data_ptr(), None, ws.data_ptr(), need, None) == rb.RB_OK
        torch.cuda.synchronize()
        assert np.array_equal(pd.cpu().numpy().view(np.uint32), want[0])
        assert np.array_equal(gd.cpu().numpy(), want[1]) and np.array_equal(hd.cpu().numpy(), want[2])
    if kind == "signs":                                        # the first path is the weight, the others are nothing
        assert np.array_equal(np.unpackbits(packed[0].view(np.uint8), bitorder="little").reshape(out, inn) == 1, W < 0)
        np.testing.assert_allclose(np.outer(g[0], h[0]), 0.25, rtol=1e-12)
        assert err.max() < 1e-11 * 0.25 * np.sqrt(out * inn)
    if kind == "zero":
        assert not err.any() and not g.any() and not h.any()


@pytest.mark.parametrize("K,inn", [(1, 4128), (2, 2080), (2, 8224), (2, 10272), (3, 4128), (3, 8288)])
def test_nothing_beside_the_weight_is_read(K, inn):
    """Groups of 2048 columns that a row fills in part, or not at all (4128, 8224 and 8288 columns: three and five groups' worth in forms
    of four and six): after the weight, the factors and the results lie NaN, as far as the widest form goes, and change nothing."""
    out, beside = 1024, 12288
    W = torch.from_numpy(synth.gaussian_weight(synth.child_rng(7, 710, K, inn), out, inn, std=0.02).astype(np.float32))
    rows, cols = torch.linspace(0.5, 1.0, out, dtype=torch.float64), torch.linspace(0.5, 1.0, inn, dtype=torch.float64)

    def call(fill):
        sizes = {torch.float32: [W.numel()], torch.float64: [out, inn, K * out, K * inn, 2 * K], torch.int32: [K * out * (inn // 32)]}
        held = [torch.full((n + beside,), fill, dtype=t, device="cuda") if t.is_floating_point else torch.full((n + beside,), -1, dtype=t, device="cuda")
                for t, ns in sizes.items() for n in ns]
        Wd, rd, cd, g, h, err, packed = held
        for to, v in ((Wd, W.reshape(-1)), (rd, rows), (cd, cols)):
            to[:v.numel()] = v.cuda()
        need = rb.lib.rb_derive_workspace_bytes(out, inn)
        ws = torch.full((need,), 255, dtype=torch.uint8, device="cuda")
        print(f"derive K={K} {out}x{inn} beside {fill}", flush=True)
        rc = rb.lib.rb_derive_iterative(Wd.data_ptr(), rd.data_ptr(), cd.data_ptr(), K, 2, out, inn, packed.data_ptr(), g.data_ptr(), h.data_ptr(),
                                        err.data_ptr(), ws.data_ptr(), need, None)
        torch.cuda.synchronize()
        assert rc == rb.RB_OK
        for t, n in ((g, K * out), (h, K * inn), (err, 2 * K)):
            assert torch.isfinite(t[:n]).all() and (torch.isnan(t[n:]).all() if fill != fill else not t[n:].any())
        assert (packed[K * out * (inn // 32):] == -1).all()
        return [t[:n].cpu() for t, n in ((packed, K * out * (inn // 32)), (g, K * out), (h, K * inn), (err, 2 * K))]

    for a, b in zip(call(0.0), call(float("nan"))):
        assert torch.equal(a, b)


@pytest.mark.parametrize("K,out,inn,noise", [(1, 300, 1056, 0.14), (1, 1024, 2048, 0.14), (2, 300, 544, 0.3), (3, 70, 4128, 1.0)])
def test_error_of_the_last_update_term_by_term(K, out, inn, noise):
    """The last entry of err against the residual of the returned paths, term by term in extended precision, where
    the residual is a small part of the weight.  Each term W - sum_j What_j rounds K times (2^-53 of a few W each),
    at random over out x in terms, which leaves nothing of it; a sum of squares goes through some 30 additions (in / 64
    of a thread, then trees), 30 x 2^-53 if all round the same way, sqrt(30) x 2^-53 = 6e-16 at random, half of it after
    the root."""
    rng = synth.child_rng(7, 706, K, out)
    W = (1.0 + noise * rng.standard_normal((out, inn))) * synth.uniform_signs(rng, 1, out, inn)[0]
    W = W.astype(np.float32)
    packed, g, h, err = _run(W, K, 1)
    signs = oracle.unpack(packed)
    left = W.astype(np.longdouble)
    for k in range(K):
        left = left - g[k].astype(np.longdouble)[:, None] * signs[k] * h[k].astype(np.longdouble)[None, :]
    want = np.sqrt((left * left).sum())
    print(f"error K={K} {out}x{inn}: off by {float(abs(err[-1, -1] / want - 1)):.2e}, {float((want / np.linalg.norm(W)) ** 2):.4f} of the weight", flush=True)
    assert abs(err[-1, -1] / want - 1) <= 1e-15


@pytest.mark.parametrize("K,out,inn,power", [(2, 70, 1056, -200), (2, 70, 1056, 200), (3, 300, 544, -230), (1, 1024, 2080, 230),
                                             (2, 1024, 4128, -200), (3, 1024, 2080, 200)])
def test_preconditioned_weights_of_any_size(K, out, inn, power):
    """Factors that are powers of two change nothing but the exponents, whatever their size: the same signs and, back in the
    original domain, the same scales, bit for bit, and errors that are the factors times as large."""
    rng = synth.child_rng(7, 707, K, out)
    W = synth.gaussian_weight(rng, out, inn, std=0.02).astype(np.float32)
    one = _run(W, K, 2)
    print(f"derive K={K} {out}x{inn}, factors of 2^{power}", flush=True)
    packed, g, h, err = _run(W, K, 2, np.full(out, 2.0 ** power), np.full(inn, 2.0 ** power))
    assert np.array_equal(packed, one[0])
    assert np.array_equal(g, one[1]) and np.array_equal(h, one[2])
    assert np.array_equal(err, one[3] * 4.0 ** power)


def test_more_rows_than_slices_of_a_grid():
    """More than 65535 slices of 32 rows (a grid's second dimension ends at 65536): one path of a tall matrix against the
    leading eigenvector of |W|^T |W|."""
    out, inn = 65536 * 32 + 37, 32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(708)
    W = torch.randn((out, inn), device="cuda", generator=gen) * 0.02
    print(f"derive {out}x{inn}", flush=True)
    packed, g, h, err = rb.rb_derive_iterative(W, 1, 1)
    A = W.double().abs()
    values, vectors = torch.linalg.eigh((A.T @ A).cpu())
    b = vectors[:, -1].abs()
    sigma = values[-1].sqrt()
    assert torch.allclose(h[0].cpu(), sigma.sqrt() * b, rtol=1e-8, atol=0)
    assert torch.allclose(g[0], (A @ b.cuda()) / sigma.sqrt(), rtol=1e-8, atol=1e-12)
    weights = (1 << torch.arange(32, device="cuda")).long()
    words = ((W < 0).long() * weights).sum(dim=1)
    assert torch.equal(packed[0, :, 0].long() & 0xffffffff, words)
    left = (A - g[0][:, None] * h[0][None, :]).norm()
    assert abs(float(err[0, 0] / left) - 1) <= 1e-9
