"""GPU parity of the complex-gated LRU (Appendix B) against its complex128 oracle, through the
C ABI, on the same seeded inputs. Tolerances as for the real layer: 1e-5 in fp32 storage, 2e-2
in bf16 storage (relative error with an rms floor)."""
import numpy as np
import pytest

import oracle
import rglru_inputs as gen

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}

SHAPES = [
    # B, T, D, nb, act
    (2, 37, 96, 3, "f32"),       # hs = 16, ragged T
    (3, 5, 40, 5, "f32"),        # hs = 4, fewer steps than a tile
    (1, 1, 16, 1, "f32"),        # one step, one dense block
    (2, 130, 512, 2, "bf16"),    # hs = 128
    (2, 100, 640, 2, "bf16"),    # hs = 160: ten column blocks of the matrix-core passes
    (3, 70, 192, 2, "bf16"),     # hs = 48: a partial column block
    (2, 70, 384, 2, "bf16"),     # hs = 96: the fused forward with one of its four waves idle
    (1, 200, 256, 2, "bf16"),    # hs = 64: ... with two
    (40, 45, 512, 4, "bf16"),    # 160 (gate block, sequence) pairs: the backward recomputes with the fused kernel
    (1, 300, 1024, 1, "bf16"),   # hs = 512: more outputs than threads
    (4, 20, 24, 12, "bf16"),     # hs = 1: per-channel gates
]


def runner():
    import paper_2402_19427_amd.runner as rn
    return rn


def f64(inp):
    return {k: (None if v is None else np.asarray(v, np.float64)) for k, v in inp.items()}


def params(q):
    return q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["theta"]


@pytest.mark.parametrize("B,T,D,nb,act", SHAPES)
@pytest.mark.parametrize("conv", [True, False])
def test_cg_forward_and_backward_match_oracle(B, T, D, nb, act, conv):
    rn = runner()
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=B * 10 + T + D, h0=True, state=True, bias=True, dy=True)
    pos0 = 7
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act, conv=conv)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act) if conv else None
    y, hT, st = dp.forward(u, h0=h0, state_in=ring, pos0=pos0)
    # the same call without the optional scratch (one pass instead of two)
    y1, hT1, _ = dp.forward(u, h0=h0, state_in=ring, pos0=pos0, scratch=False)
    assert gen.rel_err(rn.to_host(y1), rn.to_host(y)) < (2e-6 if act == "f32" else 1e-2)
    # (bf16 storage: the two-pass form takes x_t in half precision into its gate products)
    assert gen.rel_err(rn.to_host(hT1), rn.to_host(hT)) < (2e-6 if act == "f32" else 1e-2)
    q = f64(inp)
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"], state_in=q["state"]) if conv else {}
    y_ref, hT_ref, st_ref = oracle.cg_forward(q["u"], *params(q), h0=q["h0"], **kw)
    assert gen.rel_err(rn.to_host(y), y_ref) < TOL[act]
    assert gen.rel_err(rn.to_host(hT), hT_ref) < TOL[act]
    if conv:
        np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(st), pos0 + T), st_ref)
    g = dp.backward(u, rn.to_device(inp["dy"], act), h0=h0, state_in=ring, pos0=pos0,
                    dhT=rn.to_device(inp["dhT"], "f32"))
    ref = oracle.cg_backward(q["u"], *params(q), q["dy"], h0=q["h0"], dhT=q["dhT"], **kw)
    assert set(g) == set(ref)
    errs = {k: gen.rel_err(rn.to_host(g[k]), ref[k]) for k in ref}
    print("errors:", {k: float("%.3g" % v) for k, v in errs.items()})
    for k in ref:
        assert errs[k] < TOL[act], (k, errs)


@pytest.mark.parametrize("B,D,nb,act", [(5, 64, 2, "f32"), (19, 512, 2, "bf16"), (3, 1024, 1, "bf16")])
@pytest.mark.parametrize("conv", [True, False])
def test_cg_decode_steps_match_oracle_and_forward(B, D, nb, act, conv):
    rn = runner()
    nsteps = 7
    inp = gen.make_cg_inputs(B, 1, D, nb, act=act, seed=B + D, h0=True, state=True, decode_tokens=nsteps, bias=True)
    dp = rn.CgDeviceProblem(inp, B, 1, D, nb, act, conv=conv)
    pos = 11
    h = rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos), act) if conv else None
    q = f64(inp)
    h_ref, st_ref = q["h0"].copy(), q["state"].copy()
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"]) if conv else {}
    for s in range(nsteps):
        y = dp.decode_step(rn.to_device(inp["u_dec"][s], act), h, ring, pos + s)
        y_ref = oracle.cg_decode_step(q["u_dec"][s], *params(q), h_ref, st_ref, **kw)
        assert gen.rel_err(rn.to_host(y), y_ref) < TOL[act], s
        assert gen.rel_err(rn.to_host(h), h_ref) < TOL[act], s
        if conv:
            np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(ring), pos + s + 1), st_ref)


def test_cg_forward_in_pieces_equals_one_shot():
    rn = runner()
    B, T, D, nb, act = 2, 45, 128, 2, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=3, h0=True, bias=True)
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u = rn.to_device(inp["u"], act)
    y_all, hT_all, st_all = dp.forward(u, h0=rn.to_device(inp["h0"], "f32"))
    h, state, pos, ys = rn.to_device(inp["h0"], "f32"), None, 0, []
    for T1 in (1, 2, 13, 29):
        y, h, state = dp.forward(u[:, pos:pos + T1].contiguous(), h0=h, state_in=state, pos0=pos)
        ys.append(rn.to_host(y))
        pos += T1
    # (short pieces run in one pass with fp32 gate products, long ones on the matrix cores with
    # x_t in half precision: equal up to that rounding, a bf16 step of y here and there)
    assert gen.rel_err(np.concatenate(ys, axis=1), rn.to_host(y_all)) < 1e-2
    assert gen.rel_err(rn.to_host(h), rn.to_host(hT_all)) < 1e-2
    np.testing.assert_array_equal(rn.to_host(state), rn.to_host(st_all))


def test_cg_at_the_paper_s_block_shape_full_width():
    """The complex-gated layer at width 2560 in 10 blocks (hs = 128, the [128][256] gate matrices the
    matrix-core passes are built for), 2048 steps: forward and every gradient against the oracle."""
    rn = runner()
    B, T, D, nb, act = 2, 2048, 2560, 10, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=11, h0=True, bias=True, dy=True)
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    y, hT, _ = dp.forward(u, h0=h0)
    g = dp.backward(u, rn.to_device(inp["dy"], act), h0=h0, dhT=rn.to_device(inp["dhT"], "f32"))
    q = f64(inp)
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"])
    y_ref, hT_ref, _ = oracle.cg_forward(q["u"], *params(q), h0=q["h0"], **kw)
    assert gen.rel_err(rn.to_host(y), y_ref) < TOL[act]
    assert gen.rel_err(rn.to_host(hT), hT_ref) < TOL[act]
    ref = oracle.cg_backward(q["u"], *params(q), q["dy"], h0=q["h0"], dhT=q["dhT"], **kw)
    errs = {k: gen.rel_err(rn.to_host(g[k]), ref[k]) for k in ref}
    print("errors:", {k: float("%.3g" % v) for k, v in errs.items()})
    for k in ref:
        assert errs[k] < TOL[act], (k, errs)


@pytest.mark.parametrize("B,T,hs,nb", [
    (1, 1, 128, 1), (1, 31, 80, 2), (2, 33, 128, 1),    # (the backward only: a sequence of up to 64 steps has the fused forward)
    (1, 65, 128, 2), (3, 96, 96, 2), (1, 257, 80, 4),   # a window per tile; a last tile of one step
    (5, 300, 128, 20), (9, 165, 112, 20),               # windows of two and three tiles, the last one short
    (130, 70, 96, 4)])                                  # one window: nothing in front of it
@pytest.mark.parametrize("conv,turn", [(True, 0.1), (False, 0.1), (True, 1.0)])
def test_cg_tiles(B, T, hs, nb, conv, turn):
    """The kernels in tiles: tile and window edges, blocks that leave part of a wave without channels, the last state in the place of
    the first one, the gradient of the first state in the place of the last one's; phases up to c theta = 8 pi / 10 a step, and 8 pi.

    y and du: half a step of bf16, 2^-8 of an element at most, beside what the 32-bit values behind them may be off. Those: x enters the products in 22
    bits, dp and dq in 16 (2^-17 of each term, and terms of either sign); a step's phase is off by its own rounding, 2^-24 of it and
    the 2^-21 of the sine, and a state holds some hundred steps. Together three to four times the largest error seen over these shapes and three
    draws: 2^-12, for the state, its gradient and dW_a 2^-11 (single elements); ten times that for phases ten times as large."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act, pos0 = 2 * hs * nb, "bf16", 5
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=T + hs, h0=True, state=True, bias=True, dy=True)
    if turn == 1.0:
        inp["theta"] = np.random.default_rng(T).uniform(-np.pi, np.pi, hs * nb).astype(np.float32)
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act, conv=conv)
    u, dy, state = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act) if conv else None
    q = f64(inp)
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"], state_in=q["state"]) if conv else {}
    want = oracle.cg_forward(q["u"], *params(q), h0=q["h0"], **kw)
    ref = oracle.cg_backward(q["u"], *params(q), q["dy"], h0=q["h0"], dhT=q["dhT"], **kw)
    n = max(R.rglru_workspace_bytes(dp.shape(), op) for op in (R.OP_CG_FORWARD, R.OP_CG_BACKWARD))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    y, du, back, names = torch.empty_like(u), torch.empty_like(u), rn.to_device(inp["dhT"], "f32"), []
    g = {k: torch.empty(*ref[k].shape, dtype=torch.float32, device="cuda:0") for k in ref if k not in ("du", "dh0")}
    R.rglru_timing_enable(True)
    try:
        R.rglru_cg_backward(dp.shape(), dp.params, u, state, ring, pos0, dy, back, du, back, R.make_cg_param_grads(**g), ws, n, None)
        R.rglru_cg_forward(dp.shape(), dp.params, u, state, ring, pos0, y, state, None, ws, n, None)
        torch.cuda.synchronize()
        names = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
    finally:
        R.rglru_timing_enable(False)
    assert "cg_bwd_tile_kernel" in names and names.count("cg_tile_prep_kernel") == (2 if T > 64 else 1), names
    tol = lambda k: 10.0 * turn * 2.0 ** (-11 if k in ("hT", "dh0", "dW_a") else -12) + (2.0 ** -8 if k in ("y", "du") else 0.0)
    got = dict(g, y=y, hT=state, du=du, dh0=back)
    errs = {k: gen.rel_err(rn.to_host(got[k]), v) for k, v in dict(ref, y=want[0], hT=want[1]).items()}
    print("errors:", {k: float("%.3g" % v) for k, v in errs.items()})
    for k in errs:
        assert errs[k] < tol(k), (k, errs)


@pytest.mark.parametrize("hs,nb,T", [(48, 2, 40), (128, 2, 70)])
def test_weights_past_half_precision(hs, nb, T):
    """Finite weights stop at 65504 in the products: where they meet inputs of zero, nothing comes of them (an infinity would be a
    NaN). The oracle's results with weights that end there, at the tolerance of the bf16 kernels in tiles and passes."""
    rn = runner()
    D, act, tol = 2 * hs * nb, "bf16", 2.0 ** -6
    inp = gen.make_cg_inputs(1, T, D, nb, act=act, seed=hs, h0=True, dy=True, bias=True)
    for k, v in (("W_a", 1e5), ("W_x", -3e38)):
        inp[k][0, 9, 4] = gen.round_to_act(np.array([v], np.float32), act)[0]
    inp["u"][:, :, 4], inp["conv_b"][4] = 0.0, 0.0
    dp = rn.CgDeviceProblem(inp, 1, T, D, nb, act)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    y, hT, _ = dp.forward(u, h0=h0)
    got = dp.backward(u, dy, h0=h0)
    q = {k: (None if v is None else np.asarray(v, np.float64)) for k, v in inp.items()}
    w = (np.clip(q["W_a"], -65504, 65504), np.clip(q["W_x"], -65504, 65504), q["b_a"], q["b_x"], q["Lambda"], q["theta"])
    kw = dict(conv_w=q["conv_w"], conv_b=q["conv_b"], h0=q["h0"])
    want, ref = oracle.cg_forward(q["u"], *w, **kw), oracle.cg_backward(q["u"], *w, q["dy"], **kw)
    assert gen.rel_err(rn.to_host(y), want[0]) < tol and gen.rel_err(rn.to_host(hT), want[1]) < tol
    for k in ref:
        a, b = rn.to_host(got[k]), ref[k]
        if k in ("du", "dh0", "dconv_w", "dconv_b"):   # (the channel such a weight leads to on a scale of its own)
            a, b = a[..., np.arange(D) != 4], b[..., np.arange(D) != 4]
        assert gen.rel_err(a, b) < tol, k


@pytest.mark.parametrize("B,T,hs,nb,tiles", [(16, 65, 128, 16, False), (12, 96, 128, 16, False), (16, 97, 128, 16, True), (17, 65, 128, 16, True),
                                             (11, 65, 128, 16, True), (24, 96, 128, 10, False), (23, 65, 128, 10, True), (16, 65, 96, 16, True)])
def test_cg_forward_takes_the_faster_kernel(B, T, hs, nb, tiles):
    """Either side of the rule between the tiles and the fused kernel, rows of equal inputs against the oracle's one."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act = 2 * hs * nb, "bf16"
    inp = gen.make_cg_inputs(1, T, D, nb, act=act, seed=T + hs, h0=True, bias=True)
    dp = rn.CgDeviceProblem(inp, 1, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act).expand(B, T, D).contiguous(), rn.to_device(inp["h0"], "f32").expand(B, D).contiguous()
    R.rglru_timing_enable(True)
    try:
        y, hT, _ = dp.forward(u, h0=h0)
        torch.cuda.synchronize()
        names = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
    finally:
        R.rglru_timing_enable(False)
    assert ("cg_tile_kernel" in names) == tiles, names
    q = f64(inp)
    want = oracle.cg_forward(q["u"], *params(q), h0=q["h0"], conv_w=q["conv_w"], conv_b=q["conv_b"])
    assert torch.equal(y, y[:1].expand(B, T, D)) and torch.equal(hT, hT[:1].expand(B, D))
    assert gen.rel_err(rn.to_host(y[:1]), want[0]) < TOL[act] and gen.rel_err(rn.to_host(hT[:1]), want[1]) < TOL[act]


@pytest.mark.parametrize("B,T,hs,nb", [(1, 65, 80, 2), (2, 300, 96, 2), (9, 165, 112, 20), (3, 129, 128, 3), (130, 70, 96, 4)])
@pytest.mark.parametrize("off", [1, 2, 4])
def test_cg_tiles_at_any_alignment(B, T, hs, nb, off):
    """Tensors and parameters off the 16-byte grid, all of them or the outputs only: the tiles, the same bits."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, H, act = 2 * hs * nb, hs * nb, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=off + hs, h0=True, state=True, bias=True, dy=True)
    cg = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    sh = cg.shape()
    u, dy, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], 4), act)
    f32 = lambda *s: torch.empty(*s, dtype=torch.float32, device="cuda:0")
    n = max(R.rglru_workspace_bytes(sh, R.OP_CG_FORWARD), R.rglru_workspace_bytes(sh, R.OP_CG_BACKWARD))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")

    def at(t, off):
        room = torch.empty(t.numel() + 64, dtype=t.dtype, device=t.device)
        out = room[off:off + t.numel()].view(t.shape)
        out.copy_(t)
        return out

    def call(off_in, off_out):
        held = [at(cg.t[k], off_in) for k in ("W_a", "W_x", "b_a", "b_x", "Lambda", "theta", "conv_w", "conv_b")]
        par = R.make_cg_params(*held)
        g = dict(dW_a=f32(nb, hs, 2 * hs), dW_x=f32(nb, hs, 2 * hs), db_a=f32(H), db_x=f32(H), dLambda=f32(H), dtheta=f32(H),
                 dconv_w=f32(4, D), dconv_b=f32(D))
        out = dict(y=at(torch.zeros_like(u), off_out), hT=f32(B, D), ring=at(torch.zeros_like(ring), off_out), du=at(torch.zeros_like(u), off_out),
                   dh0=f32(B, D))
        uu, dd, rr = at(u, off_in), at(dy, off_in), at(ring, off_in)
        R.rglru_timing_enable(True)
        try:
            R.rglru_cg_forward(sh, par, uu, h0, rr, 4, out["y"], out["hT"], out["ring"], ws, n, None)
            R.rglru_cg_backward(sh, par, uu, h0, rr, 4, dd, None, out["du"], out["dh0"], R.make_cg_param_grads(*g.values()), ws, n, None)
            torch.cuda.synchronize()
            names = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        finally:
            R.rglru_timing_enable(False)
        assert names.count("cg_tile_prep_kernel") == 2 and "cg_bwd_tile_kernel" in names, names
        return dict(g, **out)

    want = call(0, 0)
    for got in (call(off, off), call(0, off)):
        for k in want:
            assert torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("B,T,hs,nb", [(1, 130, 128, 8), (1, 90, 80, 16), (1, 100, 112, 12)])
def test_cg_weight_gradients_in_slices(B, T, hs, nb):
    """Fewer slices of the stages than pay, where the workspace has no room for their sums: the same sums in another order, of up to 160
    terms, sqrt(160) 2^-24 < 2^-20 of their scale, 2^-16 for single elements; everything else bit for bit."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act = 2 * hs * nb, "bf16"
    inp = gen.make_cg_inputs(B, T, D, nb, act=act, seed=T + hs, dy=True, bias=True)
    dp = rn.CgDeviceProblem(inp, B, T, D, nb, act)
    u, dy, du, dh0 = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), None, None
    asked = R.rglru_workspace_bytes(dp.shape(), R.OP_CG_BACKWARD)
    ws, one, got, names = torch.empty(asked, dtype=torch.uint8, device="cuda:0"), nb * 4 * hs * hs * 4, {}, {}
    size = asked
    while size > 0:
        g = {k: torch.empty(*dp.t[v].shape, dtype=torch.float32, device="cuda:0") for k, v in
             (("dW_a", "W_a"), ("dW_x", "W_x"), ("db_a", "b_a"), ("db_x", "b_x"), ("dLambda", "Lambda"), ("dtheta", "theta"),
              ("dconv_w", "conv_w"), ("dconv_b", "conv_b"))}
        du, dh0 = torch.empty_like(u), torch.empty(B, D, dtype=torch.float32, device="cuda:0")
        R.rglru_timing_enable(True)
        try:
            R.rglru_cg_backward(dp.shape(), dp.params, u, None, None, 0, dy, None, du, dh0, R.make_cg_param_grads(**g), ws, size, None)
            torch.cuda.synchronize()
            names[size] = [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]
        except R.RglruError as e:
            assert e.code == R.ERR_WORKSPACE
            break
        finally:
            R.rglru_timing_enable(False)
        if "tile_wgrad_kernel" not in names[size]:
            break
        got[size] = dict(g, du=du, dh0=dh0)
        size -= one
    assert len(got) > 1, (asked, one, {n: set(v) for n, v in names.items()})
    for size in got:
        for k, v in got[asked].items():
            if k in ("dW_a", "dW_x"):
                assert gen.rel_err(rn.to_host(got[size][k]), rn.to_host(v)) < 2.0 ** -16, (size, k)
            else:
                assert torch.equal(got[size][k], v), (size, k)
