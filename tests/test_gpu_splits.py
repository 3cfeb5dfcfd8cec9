"""The splits of the work that a rule on sizes chooses - tiles, runs of steps, chunks - at the sizes where
they begin, end and leave a remainder, against the float64 oracle.

Tolerances: bf16 storage carries eight significant bits (half an ulp: 2^-9 of a value). A result that
passes through k such roundings in sequence (stored input of a pass, operand of a product, result) is off by
k 2^-9 of its scale at most where the factors in between are bounded by one, as decay, gates and their
derivatives are; k = 8 covers the longest chain (gradients: y, dy, x, both gradients of the
pre-activations, dx, du): 2^-6. In fp32 storage the same chain over sums of n terms of equal size gives
8 sqrt(n) 2^-24 with n = 512: 1.1e-5.
"""
import numpy as np
import pytest

import oracle
import rglru_inputs as gen

pytestmark = pytest.mark.gpu

BF16 = 8 * 2.0 ** -9
F32 = 8 * np.sqrt(512) * 2.0 ** -24


def runner():
    import paper_2402_19427_amd.runner as rn
    return rn


def f64(inp):
    return {k: (None if v is None else np.asarray(v, np.float64)) for k, v in inp.items()}


@pytest.mark.parametrize("B,bs,nb", [
    (1, 128, 1), (16, 144, 16), (17, 144, 16),     # one workgroup per (block, sequence): 256 of them at most
    (3, 256, 2), (1, 272, 2), (10, 352, 16), (11, 352, 16), (2, 512, 1), (8, 512, 16), (9, 512, 16),
    (33, 16, 2), (32, 64, 3), (31, 112, 1),        # tiles of 32 sequences, narrow blocks
    (32, 384, 1), (65, 400, 2), (9, 528, 1), (34, 768, 2)])
@pytest.mark.parametrize("how", ["plain", "at", "merge"])
def test_decode_splits(B, bs, nb, how):
    import torch
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, 1, D, nb, act=act, seed=B + bs, h0=True, state=True, decode_tokens=1, bias=True)
    dp = rn.DeviceProblem(inp, B, 1, D, nb, act)
    pos = np.arange(B) % 3 if how == "at" else np.full(B, 4)
    rings = np.stack([gen.ring_from_chrono(inp["state"][b:b + 1], int(pos[b]))[0] for b in range(B)])
    u, h, ring = rn.to_device(inp["u_dec"][0], act), rn.to_device(inp["h0"], "f32"), rn.to_device(rings, act)
    br = gen.make_branch(B, 1, D, act=act, seed=bs)[:, 0]
    if how == "plain":
        y = dp.decode_step(u, h, ring, 4)
    elif how == "at":
        y = dp.decode_step_at(u, h, ring, torch.as_tensor(pos, dtype=torch.int64, device="cuda:0"))
    else:
        y = dp.decode_step_merge(u, rn.to_device(br, act), h, ring, 4)
    q = f64(inp)
    x = np.einsum("kd,kbd->bd", q["conv_w"], np.stack([q["u_dec"][0]] + [q["state"][:, 2 - k] for k in range(3)])) + q["conv_b"]
    h_ref, st_ref = q["h0"].copy(), q["state"].copy()
    y_ref = oracle.decode_step(q["u_dec"][0], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"],
                               h_ref, st_ref, conv_b=q["conv_b"])
    # bound: x enters the products with 8 bits (2^-9 of each term), |sigma'| <= 1/4, log a = c log sigma(Lambda) r
    xb = np.abs(x).reshape(B, nb, bs)
    dp_, dq_ = (2.0 ** -9 * np.einsum("bgi,goi->bgo", xb, np.abs(q[k])).reshape(B, D) for k in ("W_a", "W_x"))
    _, la, i = (lambda p, w: (p, 8.0 * np.log(1 / (1 + np.exp(-q["Lambda"]))) / (1 + np.exp(-p)), 1 / (1 + np.exp(-w))))(
        *((np.einsum("bgi,goi->bgo", x.reshape(B, nb, bs), q[k]).reshape(B, D) + q[b])
          for k, b in (("W_a", "b_a"), ("W_x", "b_x"))))
    a = np.exp(la)
    da = a * 8.0 * np.abs(np.log(1 / (1 + np.exp(-q["Lambda"])))) * dp_ / 4
    m = np.sqrt(1 - a * a)
    bound = np.abs(q["h0"]) * da + np.abs(x) * (i * a * da / np.maximum(m, 1e-3) + m * dq_ / 4) + 1e-4 * (np.abs(h_ref) + np.abs(x))
    assert np.all(np.abs(rn.to_host(h) - h_ref) <= bound)
    if how == "merge":   # the merge rounds y and the product: 2^-8 of the result, and |GeLU(z)| <= |z|
        y_ref, bound = oracle.merge(y_ref, br), bound * np.abs(br)
    assert np.all(np.abs(rn.to_host(y) - y_ref) <= bound + 2.0 ** -7 * np.abs(y_ref) + 1e-30)
    for b in range(B):   # the ring is a copy: bits
        np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(ring)[b:b + 1], int(pos[b]) + 1)[0], st_ref[b])


@pytest.mark.parametrize("B,T,bs,nb", [
    (1, 1, 16, 1), (1, 15, 48, 1), (2, 63, 160, 2), (1, 64, 352, 1), (3, 65, 512, 1), (1, 255, 160, 1), (2, 256, 48, 3),
    (1, 257, 352, 2), (5, 129, 16, 16), (1, 1100, 64, 4)])
@pytest.mark.parametrize("merge", [False, True])
def test_layer_passes(B, T, bs, nb, merge):
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=B + T + bs, h0=True, state=True, dy=True, bias=True)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    pos0 = 5
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h0, dhT = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dhT"], "f32")
    ring, dy, brd = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act), rn.to_device(inp["dy"], act), rn.to_device(br, act)
    q = f64(inp)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    y_ref, hT_ref, st_ref = oracle.forward(q["u"], *w, **kw)
    if merge:
        out, y, hT, st = dp.forward_merge(u, brd, h0=h0, state_in=ring, pos0=pos0)
        got = dp.backward_merge(u, brd, y, dy, h0=h0, state_in=ring, pos0=pos0, dhT=dhT)
        ref = oracle.backward_merge(q["u"], br, *w, q["dy"], dhT=q["dhT"], **kw)
        assert gen.rel_err(rn.to_host(out), oracle.merge(y_ref, br)) < BF16
    else:
        y, hT, st = dp.forward(u, h0=h0, state_in=ring, pos0=pos0)
        got = dp.backward(u, y, dy, h0=h0, state_in=ring, pos0=pos0, dhT=dhT)
        ref = oracle.backward(q["u"], *w, q["dy"], dhT=q["dhT"], **kw)
    assert gen.rel_err(rn.to_host(y), y_ref) < BF16
    assert gen.rel_err(rn.to_host(hT), hT_ref) < BF16
    np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(st), pos0 + T), st_ref)
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k


@pytest.mark.parametrize("B,T,hs,nb", [
    (1, 64, 64, 2), (2, 65, 16, 3), (1, 128, 160, 1), (3, 129, 48, 2), (1, 256, 128, 2), (2, 257, 80, 1), (1, 1025, 32, 2),
    (16, 66, 128, 8), (17, 66, 128, 8), (60, 65, 96, 3)])   # the forward below and above the fused kernel's share
def test_complex_gated_passes(B, T, hs, nb):
    rn = runner()
    D, act = 2 * hs * nb, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=B + T + hs, h0=True, state=True, bias=True, dy=True)
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], 4), act)
    q = f64(inp)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["theta"])
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    y, hT, st = dp.forward(u, h0=h0, state_in=ring, pos0=4)
    y_ref, hT_ref, st_ref = oracle.cg_forward(q["u"], *w, **kw)
    assert gen.rel_err(rn.to_host(y), y_ref) < BF16
    assert gen.rel_err(rn.to_host(hT), hT_ref) < BF16
    np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(st), 4 + T), st_ref)
    got = dp.backward(u, rn.to_device(inp["dy"], act), h0=h0, state_in=ring, pos0=4, dhT=rn.to_device(inp["dhT"], "f32"))
    ref = oracle.cg_backward(q["u"], *w, q["dy"], dhT=q["dhT"], **kw)
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k


@pytest.mark.parametrize("B,T,bs,nb", [(1, 9, 16, 1), (2, 16, 64, 4), (1, 17, 128, 2), (3, 33, 256, 1), (1, 70, 512, 1),
                                       (1, 1025, 64, 2), (2, 300, 48, 2)])
@pytest.mark.parametrize("merge", [False, True])
def test_fp32_forward_in_runs(B, T, bs, nb, merge):
    rn = runner()
    D, act = bs * nb, "f32"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=B + T + bs, h0=True, state=True, bias=True)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], 5), act)
    q = f64(inp)
    y_ref, hT_ref, st_ref = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"],
                                           conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    if merge:
        out, y, hT, st = dp.forward_merge(u, rn.to_device(br, act), h0=h0, state_in=ring, pos0=5)
        assert gen.rel_err(rn.to_host(out), oracle.merge(y_ref, br)) < F32
    else:
        y, hT, st = dp.forward(u, h0=h0, state_in=ring, pos0=5)
    assert gen.rel_err(rn.to_host(y), y_ref) < F32
    assert gen.rel_err(rn.to_host(hT), hT_ref) < F32
    np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(st), 5 + T), st_ref)


@pytest.mark.parametrize("B,T,bs,nb,steps", [(2, 1000, 64, 4, None), (1, 1024, 128, 8, None),   # one piece of 63, 64 runs
                                             (3, 250, 64, 4, 48), (2, 1000, 64, 2, 240), (1, 4100, 32, 2, 1040)])
@pytest.mark.parametrize("merge", [False, True])
def test_fp32_forward_state_in_place_and_in_pieces(B, T, bs, nb, steps, merge):
    """hT in the memory of h0, over many workgroups; `steps`: scratch for that many steps at a time (pieces
    of 3, 15 and 65 runs, at least two of them neither first nor last)."""
    import paper_2402_19427_amd as R
    rn = runner()
    D, act, pos0 = bs * nb, "f32", 5
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, bias=True)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act)
    sh, y, out = dp.shape(), dp.empty_act(B, T, D), dp.empty_act(B, T, D)
    n = R.rglru_workspace_bytes(sh, R.OP_FORWARD_MERGE if merge else R.OP_FORWARD)
    if steps:   # two states, two coefficients per step, the runs' aggregates and (beyond 64 runs) states
        al, nrun = (lambda v: (v + 255) // 256 * 256), -(-steps // 16)
        n = 256 + 2 * al(4 * B * D) + 2 * al(4 * B * steps * D) + al(8 * B * nrun * D) + (al(4 * B * nrun * D) if nrun > 64 else 0)
    ws = dp.empty_f32(n // 4)
    if merge:
        R.rglru_forward_merge(sh, dp.params, u, rn.to_device(br, act), h, ring, pos0, 0, out, y, h, ring, ws, n)
    else:
        R.rglru_forward(sh, dp.params, u, h, ring, pos0, y, h, ring, ws, n)
    q = f64(inp)
    y_ref, hT_ref, st_ref = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"],
                                           conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    assert gen.rel_err(rn.to_host(y), y_ref) < F32
    assert gen.rel_err(rn.to_host(h), hT_ref) < F32
    if merge:   # the error of y times |GeLU(z)| <= |z|
        assert np.all(np.abs(rn.to_host(out) - oracle.merge(y_ref, br)) <= F32 * np.abs(br) * (np.abs(y_ref) + np.sqrt(np.mean(y_ref ** 2))))
    np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(ring), pos0 + T), st_ref)


@pytest.mark.parametrize("B,T,D", [(60, 300, 256), (30, 515, 256), (20, 1030, 256), (1, 4100, 256)])   # 4, 8 and 16 slices, rings that wrap
@pytest.mark.parametrize("adjoint", [False, True])
def test_scan_slices(B, T, D, adjoint):
    import paper_2402_19427_amd as R
    rn = runner()
    inp = gen.make_scan_inputs(B, T, D, act="bf16", seed=B + T)
    a, g, h0 = rn.to_device(inp["a"], "bf16"), rn.to_device(inp["g"], "bf16"), rn.to_device(inp["h0"], "f32")
    if adjoint:
        got, end = rn.scan(a, g, h0, flags=R.SCAN_ADJOINT | R.SCAN_NO_INPUT_SCALE, act="bf16")
        ref, end_ref = oracle.scan_adjoint(inp["a"], inp["g"], inp["h0"])
    else:
        got, end = rn.scan(a, g, h0, act="bf16")
        ref, end_ref = oracle.scan(inp["a"], inp["g"], inp["h0"])
    assert gen.rel_err(rn.to_host(got), ref) < 2.0 ** -8      # stored once, from an fp32 state
    assert gen.rel_err(rn.to_host(end), end_ref) < 1e-4       # (sqrt(1 - a^2) of bf16 a near 1: eight bits cancel)


@pytest.mark.parametrize("B,T", [(20, 1030), (1, 4100)])
def test_scan_slices_with_decays_outside_their_range(B, T):
    """Negative decays and decays above one (unscaled input): products outside [0, 1] pass from slice to slice
    in fp32 too. The state remembers some 30 steps, each with two roundings of 2^-24; twice that for sums that
    cancel, next to the 2^-8 of the stored result."""
    import paper_2402_19427_amd as R
    rn = runner()
    inp = gen.make_scan_inputs(B, T, 256, act="bf16", seed=B + T)
    rng = np.random.default_rng(T)
    a = np.where(rng.random(inp["a"].shape) < 0.02, -1.0, 1.0) * rng.choice([0.9375, 0.96875, 1.015625], inp["a"].shape)
    h, hT = rn.scan(rn.to_device(a, "bf16"), rn.to_device(inp["g"], "bf16"), rn.to_device(inp["h0"], "f32"),
                    flags=R.SCAN_NO_INPUT_SCALE, act="bf16")
    ref, end_ref = oracle.scan(a, inp["g"], inp["h0"], normalize=False)
    assert gen.rel_err(rn.to_host(h), ref) < 2.0 ** -7
    assert gen.rel_err(rn.to_host(hT), end_ref) < 120 * 2.0 ** -24


@pytest.mark.parametrize("B,T,adjoint", [(1, 8192, False), (1, 8192, True), (5, 6000, False), (12, 5000, True)])   # 16, 16, 16 and 10 slices
def test_scan_slices_with_slowly_growing_products(B, T, adjoint):
    """Decays barely above one: the product of a tile of 32 steps, 1 + 5.8e-5, must not lose the bits that
    make the state grow by 1.5 % over the sequence. Each step's decay is an fp32 number beside one, off by
    2^-23 at most, as is its product: 2^-22 per step."""
    import paper_2402_19427_amd as R
    rn = runner()
    D = 256 if B < 12 else 512
    inp = gen.make_scan_inputs(B, T, D, act="bf16", seed=B + T)
    log_a = np.full(inp["a"].shape, gen.round_to_act(np.float32([1.8e-6]), "bf16")[0], np.float32)
    log_a[:, ::7] = gen.round_to_act(np.float32([-4e-7]), "bf16")[0]
    g = gen.round_to_act(0.01 * inp["g"], "bf16")
    flags = R.SCAN_LOG_A | R.SCAN_NO_INPUT_SCALE | (R.SCAN_ADJOINT if adjoint else 0)
    h, hT = rn.scan(rn.to_device(log_a, "bf16"), rn.to_device(g, "bf16"), rn.to_device(inp["h0"], "f32"), flags=flags, act="bf16")
    a = np.exp(log_a.astype(np.float64))
    ref, end_ref = oracle.scan_adjoint(a, g, inp["h0"]) if adjoint else oracle.scan(a, g, inp["h0"], normalize=False)
    assert gen.rel_err(rn.to_host(h), ref) < 2.0 ** -8 + T * 2.0 ** -22
    assert gen.rel_err(rn.to_host(hT), end_ref) < T * 2.0 ** -22


@pytest.mark.parametrize("G", [3, 5, 7])
def test_time_slices_that_do_not_divide_the_ring(G):
    """Rings of 32 and 64 slots over 210 tiles: a slot changes hands between workgroups with every use."""
    import paper_2402_19427_amd as R
    rn = runner()
    B, T, D, act = 1, 6700, 256, "bf16"
    inp = gen.make_inputs(B, T, D, 1, act=act, seed=G, h0=True, dy=True, bias=True)
    q = f64(inp)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    si = gen.make_scan_inputs(B, T, D, act=act, seed=G)
    R.rglru_set_max_time_slices(G)
    try:
        dp = rn.DeviceProblem(inp, B, T, D, 1, act)
        u, h0, dhT = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dhT"], "f32")
        y, hT, _ = dp.forward(u, h0=h0)
        got = dp.backward(u, y, rn.to_device(inp["dy"], act), h0=h0, dhT=dhT)
        h, end = rn.scan(*(rn.to_device(si[k], act) for k in ("a", "g")), rn.to_device(si["h0"], "f32"), act=act)
    finally:
        R.rglru_set_max_time_slices(0)
    y_ref, hT_ref, _ = oracle.forward(q["u"], *w, conv_b=q["conv_b"], h0=q["h0"])
    ref = oracle.backward(q["u"], *w, q["dy"], conv_b=q["conv_b"], h0=q["h0"], dhT=q["dhT"])
    h_ref, _ = oracle.scan(si["a"], si["g"], si["h0"])
    assert gen.rel_err(rn.to_host(y), y_ref) < BF16 and gen.rel_err(rn.to_host(hT), hT_ref) < BF16
    assert gen.rel_err(rn.to_host(h), h_ref) < 2.0 ** -8
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k


@pytest.mark.parametrize("bs", [96, 160, 352])
def test_layer_passes_keep_a_nan_of_a_gate(bs):
    """(Passes at 96 channels, tiles at the others.) A NaN in one channel's gate reaches every gradient it reaches in the oracle, and no other."""
    rn = runner()
    B, T, nb, act = 2, 130, 2, "bf16"
    inp = gen.make_inputs(B, T, bs * nb, nb, act=act, seed=bs, dy=True, bias=True)
    inp["b_x"][bs + 3] = np.nan
    dp = rn.DeviceProblem(inp, B, T, bs * nb, nb, act)
    u, dy, q = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), f64(inp)
    y, hT, _ = dp.forward(u)
    got = dp.backward(u, y, dy)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    y_ref, _, _ = oracle.forward(q["u"], *w, conv_b=q["conv_b"])
    ref = oracle.backward(q["u"], *w, q["dy"], conv_b=q["conv_b"])
    np.testing.assert_array_equal(np.isnan(rn.to_host(y)), np.isnan(y_ref))
    for k in ("db_a", "db_x", "dLambda", "dW_a", "dW_x", "du"):
        np.testing.assert_array_equal(np.isnan(rn.to_host(got[k])), np.isnan(ref[k]), err_msg=k)


def _large(inp, t0):
    """A few inputs past half precision's 65504, through the Conv1D unchanged."""
    inp["conv_w"][:] = 0.0
    inp["conv_w"][0] = 1.0
    inp["conv_b"][:] = 0.0
    for t, d, v in ((t0, 3, 9e4), (t0, 40, -7e4), (t0 + 9, 17, -1.25e5)):
        inp["u"][0, t, d] = gen.round_to_act(np.float32([v]), "bf16")[0]


@pytest.mark.parametrize("T,hs", [(40, 128), (300, 128), (300, 48)])   # fused forward, passes
def test_complex_gated_inputs_past_half_precision(T, hs):
    rn = runner()
    B, nb, act = 1, 2, "bf16"
    inp = gen.make_cg_inputs(B, T, 2 * hs * nb, nb, act=act, seed=T + hs, bias=True, dy=True)
    _large(inp, 20)
    dp, q = rn.CgDeviceProblem(inp, B, T, 2 * hs * nb, nb, act), f64(inp)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["theta"])
    u = rn.to_device(inp["u"], act)
    y, hT, _ = dp.forward(u)
    y_ref, hT_ref, _ = oracle.cg_forward(q["u"], *w, conv_w=q["conv_w"])
    got = dp.backward(u, rn.to_device(inp["dy"], act))
    ref = oracle.cg_backward(q["u"], *w, q["dy"], conv_w=q["conv_w"])
    assert gen.rel_err(rn.to_host(y), y_ref) < BF16 and gen.rel_err(rn.to_host(hT), hT_ref) < BF16
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k


@pytest.mark.parametrize("bs", [96, 160])
def test_layer_passes_stay_finite_past_half_precision(bs):
    """In the backward (passes at 96 channels, tiles at 160) x in half precision feeds products only: an x past its range
    closes or opens gates, it puts no infinity into them. (No reference: with m_t = 0 the oracle has 0 / 0.)"""
    rn = runner()
    B, T, nb, act = 1, 300, 2, "bf16"
    inp = gen.make_inputs(B, T, bs * nb, nb, act=act, seed=7, dy=True, bias=True)
    _large(inp, 20)
    dp = rn.DeviceProblem(inp, B, T, bs * nb, nb, act)
    u = rn.to_device(inp["u"], act)
    y, _, _ = dp.forward(u)
    got = dp.backward(u, y, rn.to_device(inp["dy"], act))
    for k, v in got.items():
        assert np.all(np.isfinite(rn.to_host(v))), k


@pytest.mark.parametrize("bs", [96, 160, 352])
def test_layer_passes_round_what_they_store(bs):
    """(Passes at 96 channels, tiles at the others.) Sums over time: stored adjoints rounded to nearest leave errors of at most 2^-12 each that average
    out, truncated ones shift dx (stored twice) by 2^-11 of its size (2^-12 on average each time)."""
    rn = runner()
    B, T, nb, act = 2, 600, 2, "bf16"
    inp = gen.make_inputs(B, T, bs * nb, nb, act=act, seed=bs + 1, dy=True, bias=True)
    dp = rn.DeviceProblem(inp, B, T, bs * nb, nb, act)
    u, q = rn.to_device(inp["u"], act), f64(inp)
    y, _, _ = dp.forward(u)
    got = dp.backward(u, y, rn.to_device(inp["dy"], act))
    ref = oracle.backward(q["u"], *(q[k] for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "conv_w")), q["dy"], conv_b=q["conv_b"])
    assert np.linalg.norm(rn.to_host(got["dconv_b"]) - ref["dconv_b"]) < 2.0 ** -11 * np.linalg.norm(ref["dconv_b"])


def _smooth(B, T, bs, nb, seed):
    """Gates and decay that do not depend on the input, an upstream gradient and inputs that do not change
    over time: the adjoints vary slowly from step to step."""
    D = bs * nb
    inp = gen.make_inputs(B, T, D, nb, act="bf16", seed=seed, dy=True)
    inp["W_a"][:] = 0.0
    inp["W_x"][:] = 0.0
    inp["b_a"][:] = 0.25
    inp["b_x"][:] = 0.25
    inp["Lambda"][:] = -np.log(np.expm1(0.001 / (8.0 / (1.0 + np.exp(-0.25)))))   # a = exp(-0.001)
    for k in ("u", "dy"):
        inp[k][:] = inp[k][:, :1]
    return inp


@pytest.mark.parametrize("T,bs,nb", [(600, 160, 2), (300, 240, 1), (600, 352, 8), (513, 64, 4), (300, 48, 16)])
def test_input_gradient_is_a_difference_of_adjoints(T, bs, nb):
    """Conv1D taps 1, -1: du is the difference of two neighbours that agree to one part in 200 and more.
    dx is a chain of eight fp32 operations on adjoints that are summed over runs of 64 steps (64 roundings of
    2^-24, then 8 more): 72 2^-24 of dx; half precision anywhere in between would leave 2^-12."""
    rn = runner()
    B, act, D = 2, "bf16", bs * nb
    inp = _smooth(B, T, bs, nb, T + bs)
    inp["conv_w"][:] = 0.0
    inp["conv_w"][0], inp["conv_w"][1] = 1.0, -1.0
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    w = [q[k] for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "conv_w")]
    u = rn.to_device(inp["u"], act)
    y, _, _ = dp.forward(u)
    got = rn.to_host(dp.backward(u, y, rn.to_device(inp["dy"], act))["du"])
    ref = oracle.backward(q["u"], *w, q["dy"])["du"]
    dx = np.abs(np.cumsum(ref[:, ::-1], axis=1)[:, ::-1])   # dx_t = du_t + dx_{t+1}
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 72 * 2.0 ** -24 * dx)


@pytest.mark.parametrize("bs,nb", [(128, 2), (160, 2), (240, 1)])
def test_gates_logits_keep_their_bits(bs, nb):
    """A gate that is open to the same degree in every step and channel: an error of its logit is the same in
    all terms of db_x. r (1 - r) follows it one to one; fp32 leaves 2^-21 at a logit of 8, a few roundings
    of the adjoint (bounded as above by 72 2^-24) and the hardware's exponentials (2^-20)."""
    rn = runner()
    B, T, act, D = 1, 300, "bf16", bs * nb   # (one sequence: terms of one sign)
    inp = _smooth(B, T, bs, nb, bs)
    inp["b_x"][:] = 8.0039
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u = rn.to_device(inp["u"], act)
    y, _, _ = dp.forward(u)
    got = rn.to_host(dp.backward(u, y, rn.to_device(inp["dy"], act))["db_x"])
    ref = oracle.backward(q["u"], *(q[k] for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "conv_w")), q["dy"])["db_x"]
    assert np.all(np.abs(got - ref) <= 2.0 ** -16 * np.abs(ref))


@pytest.mark.parametrize("B,T,bs,nb,size", [(1, 1, 16, 16, 55552), (1, 1, 2048, 1, 33734912), (2, 40, 160, 2, None)])
def test_backward_in_a_workspace_laid_out_before_the_passes(B, T, bs, nb, size):
    """size: what the call asked for then; the general kernels take over where the passes do not fit it."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=bs, h0=True, dy=True, bias=True)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    y, _, _ = dp.forward(u, h0=h0)
    sh = dp.shape()
    n = R.rglru_workspace_bytes(sh, R.OP_BACKWARD)
    size = size or n
    g = dp.alloc_grads()
    pg = R.make_param_grads(*[g[k] for k in ("dW_a", "dW_x", "db_a", "db_x", "dLambda", "dconv_w", "dconv_b")])
    ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    du, dh0 = dp.empty_act(B, T, D), dp.empty_f32(B, D)
    R.rglru_backward(sh, dp.params, u, h0, None, 0, y, dy, None, du, dh0, pg, ws, size, None)
    q = f64(inp)
    ref = oracle.backward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], q["dy"], conv_b=q["conv_b"],
                          h0=q["h0"])
    for k, v in dict(g, du=du, dh0=dh0).items():
        assert gen.rel_err(rn.to_host(v), ref[k]) < BF16, k


@pytest.mark.parametrize("B,T,hs,nb,size", [(1, 17, 256, 1, 753664), (2, 17, 256, 2, 1966080)])
def test_complex_gated_backward_in_a_workspace_laid_out_before_the_passes(B, T, hs, nb, size):
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act = 2 * hs * nb, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=hs, h0=True, dy=True)
    cg = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    need = R.rglru_workspace_bytes(cg.shape(), R.OP_CG_BACKWARD)
    assert size < need
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda:0")
    g = dict(dW_a=f32(nb, hs, 2 * hs), dW_x=f32(nb, hs, 2 * hs), db_a=f32(D // 2), db_x=f32(D // 2), dLambda=f32(D // 2),
             dtheta=f32(D // 2), dconv_w=f32(4, D), dconv_b=f32(D))
    pg = R.make_cg_param_grads(*g.values())
    ws, du, dh0 = torch.empty(size, dtype=torch.uint8, device="cuda:0"), torch.empty_like(u), f32(B, D)
    R.rglru_cg_backward(cg.shape(), cg.params, u, h0, None, 0, dy, None, du, dh0, pg, ws, size, None)
    c = f64(inp)
    ref = oracle.cg_backward(c["u"], c["W_a"], c["W_x"], c["b_a"], c["b_x"], c["Lambda"], c["theta"], c["dy"], conv_w=c["conv_w"],
                             h0=c["h0"])
    for k, v in dict(g, du=du, dh0=dh0).items():
        if k in ref and ref[k] is not None and k != "dconv_b":
            assert gen.rel_err(rn.to_host(v), ref[k]) < BF16, k


def _at(t, off):
    """The tensor's values `off` elements behind a 256-byte boundary."""
    import torch
    room = torch.empty(t.numel() + 128, dtype=t.dtype, device=t.device)
    out = room[off:off + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("off", [1, 2, 4])
def test_complex_gated_passes_at_any_alignment(off):
    """u, dy, the carried ring and the Conv1D's parameters off the 16-byte grid: the matrix-core passes, the same results."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    B, T, hs, nb, act = 2, 300, 64, 2, "bf16"
    D = 2 * hs * nb
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=off, h0=True, state=True, bias=True, dy=True)
    cg = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u, dy, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], 4), act)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda:0")
    sh = cg.shape()

    def call(off):
        at = lambda t: _at(t, off)
        held = [at(cg.t[k]) for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "theta", "conv_w", "conv_b")]   # (params hold addresses)
        params = R.make_cg_params(*held)
        g = dict(dW_a=f32(nb, hs, 2 * hs), dW_x=f32(nb, hs, 2 * hs), db_a=f32(D // 2), db_x=f32(D // 2), dLambda=f32(D // 2),
                 dtheta=f32(D // 2), dconv_w=f32(4, D), dconv_b=f32(D))
        out = dict(y=at(torch.zeros_like(u)), hT=f32(B, D), ring=at(torch.zeros_like(ring)), du=at(torch.zeros_like(u)), dh0=f32(B, D))
        uu, dd, rr = at(u), at(dy), at(ring)
        n = R.rglru_workspace_bytes(sh, R.OP_CG_FORWARD)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        R.rglru_timing_enable(True)
        R.rglru_cg_forward(sh, params, uu, h0, rr, 4, out["y"], out["hT"], out["ring"], ws, n, None)
        n = R.rglru_workspace_bytes(sh, R.OP_CG_BACKWARD)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        R.rglru_cg_backward(sh, params, uu, h0, rr, 4, dd, None, out["du"], out["dh0"], R.make_cg_param_grads(*g.values()), ws, n, None)
        torch.cuda.synchronize()
        names = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        R.rglru_timing_enable(False)
        return dict(g, **out), names

    want, _ = call(0)
    got, names = call(off)
    assert "cg_apply_kernel" in names and "cg_wgrad_kernel" in names and "cg_dgrad_kernel" in names, names
    for k in want:
        np.testing.assert_array_equal(rn.to_host(got[k]), rn.to_host(want[k]), err_msg=k)


def _long_case(rn, cg, T, D, nb, seed):
    """A sequence of T steps with decays that forget within a few hundred steps, made on the GPU."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    act = lambda t: t.to(torch.bfloat16)
    normal = lambda *s, k=1.0: torch.randn(*s, generator=g, device="cuda") * k
    W, bs = (D // 2, D // 2 // nb) if cg else (D, D // nb)
    nin = 2 * bs if cg else bs
    t = dict(W_a=act(normal(nb, bs, nin, k=nin ** -0.5)), W_x=act(normal(nb, bs, nin, k=nin ** -0.5)), b_a=normal(W, k=0.1),
             b_x=normal(W, k=0.1), Lambda=torch.full((W,), 2.0, device="cuda"), conv_w=normal(4, D, k=0.5), conv_b=normal(D, k=0.1))
    if cg:
        t["theta"] = normal(W, k=0.1)
    return t, act(normal(1, T, D)), act(normal(1, T, D))


@pytest.mark.parametrize("cg,T,D,nb", [(False, 210240, 2560, 16), (False, 210240, 2560, 40), (True, 131200, 4096, 16)])
def test_passes_on_sequences_past_32_bit_offsets(cg, T, D, nb):
    """fp32 intermediates of more than 2^31 bytes a sequence: the passes (blocks of 160 channels: the tiles) run, and what they give at the start, around the
    2^31 bytes and at the end is what a short call gives on the steps around it (a decay of 0.6 on average, so that
    512 steps more on either side leave nothing of what is missing)."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    t, u, dy = _long_case(rn, cg, T, D, nb, 7)
    keys = ("W_a", "W_x", "b_a", "b_x", "Lambda") + (("theta",) if cg else ()) + ("conv_w", "conv_b")
    params = (R.make_cg_params if cg else R.make_params)(*[t[k] for k in keys])

    def call(u, dy):
        n = u.shape[1]
        sh = R.make_shape(1, n, D, nb, R.BF16)
        f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda:0")
        g = {k: torch.empty_like(t[k], dtype=torch.float32) for k in keys}
        y, hT, ring, du, dh0 = torch.empty_like(u), f32(1, D), torch.empty(1, 3, D, dtype=u.dtype, device="cuda:0"), torch.empty_like(u), f32(1, D)
        ops = (R.OP_CG_FORWARD, R.OP_CG_BACKWARD) if cg else (R.OP_FORWARD, R.OP_BACKWARD)
        nf, nw = (R.rglru_workspace_bytes(sh, o) for o in ops)
        ws = torch.empty(max(nf, nw, 256), dtype=torch.uint8, device="cuda:0")
        R.rglru_timing_enable(True)
        if cg:
            R.rglru_cg_forward(sh, params, u, None, None, 0, y, hT, ring, ws, nf, None)
            R.rglru_cg_backward(sh, params, u, None, None, 0, dy, None, du, dh0, R.make_cg_param_grads(*g.values()), ws, nw, None)
        else:
            R.rglru_forward(sh, params, u, None, None, 0, y, hT, ring, ws, nf, None)
            R.rglru_backward(sh, params, u, None, None, 0, y, dy, None, du, dh0, R.make_param_grads(*g.values()), ws, nw, None)
        torch.cuda.synchronize()
        names = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        R.rglru_timing_enable(False)
        return y, du, names

    y, du, names = call(u, dy)
    ran = {"cg_wgrad_kernel", "cg_apply_kernel"} if cg else {"fwd_tile_kernel", "bwd_tile_kernel", "tile_wgrad_kernel"} if D // nb >= 112 \
        else {"apply_kernel", "adjoint_kernel", "wgrad_pass_kernel"}
    assert ran <= set(names), names
    at = (1 << 31) // (4 * D)
    for lo, hi in ((0, 300), (at - 150, at + 150), (T - 300, T)):
        a, b = max(lo - 512, 0), min(hi + 512, T)
        ys, dus, _ = call(u[:, a:b].contiguous(), dy[:, a:b].contiguous())
        for got, want in ((y, ys), (du, dus)):
            got, want = got[:, lo:hi].float(), want[:, lo - a:hi - a].float()
            assert torch.isfinite(got).all() and ((got - want).norm() / want.norm()).item() < BF16, (lo, hi)


@pytest.mark.parametrize("T,bs,nb", [(300, 352, 8), (300, 64, 4), (50, 512, 1)])
def test_layer_forward_past_half_precision(T, bs, nb):
    """x past half precision's range leaves the gates of its block finite and enters i_t x_t as it is. (The rows of W of the
    channels it arrives in are zero, so that b_t stays inside half precision there. In the products x stops at 65504: one such
    x per step, at most 1.6 % past it, moves a logit p by 0.016 p and a gate by 0.016 max |p| sigma'(p) = 2^-8 at most.)"""
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=bs, bias=True)
    inp["conv_w"][:], inp["conv_b"][:] = 0.0, 0.0
    inp["conv_w"][0] = 1.0
    for t, d, v in ((20, 3, 66048.0), (24, 40, -66560.0), (29, 17, -66048.0)):   # (bf16 values)
        inp["u"][0, t, d] = v
    for d in (3, 17, 40):
        inp["W_a"][0, d], inp["W_x"][0, d], inp["b_x"][d] = 0.0, 0.0, -3.0
    dp = rn.DeviceProblem(inp, 1, T, D, nb, act)
    y, hT, _ = dp.forward(rn.to_device(inp["u"], act))
    q = f64(inp)
    ref, hT_ref, _ = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], conv_b=q["conv_b"])
    y = rn.to_host(y)
    few = np.isin(np.arange(D), (3, 17, 40))
    for got, want in ((y[..., few], ref[..., few]), (y[..., ~few], ref[..., ~few]), (rn.to_host(hT), hT_ref)):
        assert gen.rel_err(got, want) < BF16


@pytest.mark.parametrize("T,bs,nb,off", [(300, 160, 8, 1), (300, 160, 8, 4), (300, 352, 8, 1), (50, 352, 8, 2),   # the tiles
                                         (300, 64, 8, 1), (50, 96, 8, 2), (130, 64, 4, 4),                       # the passes
                                         (300, 384, 4, 1), (50, 512, 4, 2)])   # the passes with the merge; 512 channels: in the forward, too
@pytest.mark.parametrize("merge", [False, True])
def test_layer_passes_at_any_alignment(T, bs, nb, off, merge):
    """Tensors of the backward off the 16-byte grid, and states of the forward off the 8-byte grid: the tiles or the passes, the same
    results. (The backward's u and dy without the merge stay on the grid: nothing but the passes' own size is asked for.)"""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    B, D, act = 2, bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=bs, h0=True, state=True, bias=True, dy=True)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, dy, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), rn.to_device(inp["h0"], "f32")
    br = rn.to_device(gen.make_branch(B, T, D, act=act, seed=3), act)
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], 4), act)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda:0")
    sh = dp.shape()

    def call(off):
        at = lambda t: _at(t, off)
        par = [at(getattr(dp, k)) for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "conv_w", "conv_b")]
        fpar, bpar = dp.params, R.make_params(*par)
        g = dp.alloc_grads()
        pg = R.make_param_grads(*[g[k] for k in ("dW_a", "dW_x", "db_a", "db_x", "dLambda", "dconv_w", "dconv_b")])
        hh = _at(h0, 1 if off else 0)
        out = dict(y=torch.empty_like(u), hT=_at(torch.zeros_like(h0), 1 if off else 0), ring=torch.empty_like(ring),
                   du=at(torch.zeros_like(u)), dh0=f32(B, D))
        names = []
        R.rglru_timing_enable(True)
        n = R.rglru_workspace_bytes(sh, R.OP_FORWARD)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        R.rglru_forward(sh, fpar, u, hh, ring, 4, out["y"], out["hT"], out["ring"], ws, n, None)
        torch.cuda.synchronize()
        names += [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        R.rglru_timing_enable(True)
        yy, rr, dd, bb = at(out["y"]), at(ring), at(dy) if merge else dy, at(br)
        n = R.rglru_workspace_bytes(sh, R.OP_BACKWARD_MERGE if merge else R.OP_BACKWARD)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        if merge:
            out["dbranch"] = at(torch.zeros_like(u))
            R.rglru_backward_merge(sh, bpar, u, bb, hh, rr, 4, 0, yy, dd, None, out["du"], out["dbranch"], out["dh0"], pg, ws, n, None)
        else:
            R.rglru_backward(sh, bpar, u, hh, rr, 4, yy, dd, None, out["du"], out["dh0"], pg, ws, n, None)
        torch.cuda.synchronize()
        names += [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        R.rglru_timing_enable(False)
        return dict(g, **out), names

    want, _ = call(0)
    got, names = call(off)
    tiles = bs >= 112 and not (merge and bs > 352)
    assert ({"bwd_tile_kernel", "tile_wgrad_kernel"} if tiles else {"adjoint_kernel", "wgrad_pass_kernel"}) <= set(names), names
    assert ("fwd_tile_kernel" if 112 <= bs <= 480 else "apply_kernel") in names, names
    for k in want:
        np.testing.assert_array_equal(rn.to_host(got[k]), rn.to_host(want[k]), err_msg=k)


@pytest.mark.parametrize("B,T", [(1, 33), (8, 64), (8, 512), (8, 513), (16, 256), (16, 257)])   # at most 4 tiles per workgroup, and one more
@pytest.mark.parametrize("tanh", [False, True])
def test_merge_of_narrow_blocks_in_few_tiles(B, T, tanh):
    """The merge as an epilogue against the same call with a merge kernel behind the plain forward: the same bits."""
    import paper_2402_19427_amd as R
    rn = runner()
    bs, nb, act = 160, 8, "bf16"
    D = bs * nb
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=B + T, h0=True, bias=True)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h0, br = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(gen.make_branch(B, T, D, act=act, seed=1), act)
    flags = R.MERGE_GELU_TANH if tanh else 0
    got = dp.forward_merge(u, br, h0=h0, flags=flags, keep_y=True)
    want = dp.forward_merge(u, br, h0=h0, flags=flags | R.MERGE_SEPARATE, keep_y=True)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(rn.to_host(a), rn.to_host(b))
