"""The kernels behind the tiles: what serves the calls whose tensors or workspace the tiles do not accept, against the float64
oracle. Tolerance 2^-6 as for the other bf16 kernels (results of eight bits, products of eleven)."""
import numpy as np
import pytest

import oracle
import rglru_inputs as gen

pytestmark = pytest.mark.gpu
BF16 = 2.0 ** -6


def runner():
    from paper_2402_19427_amd import runner as rn
    return rn


def f64(inp):
    return {k: (None if v is None else np.asarray(v, np.float64)) for k, v in inp.items()}


def at(t, off):
    """The tensor's values `off` elements behind a 256-byte boundary."""
    import torch
    room = torch.empty(t.numel() + 128, dtype=t.dtype, device=t.device)
    out = room[off:off + t.numel()].view(t.shape)
    out.copy_(t)
    return out


class Names:
    """The kernels that ran inside the `with`."""

    def __enter__(self):
        import paper_2402_19427_amd as R
        R.rglru_timing_enable(True)
        return self

    def __exit__(self, *exc):
        import paper_2402_19427_amd as R
        import torch
        torch.cuda.synchronize()
        self.ran = {R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())}
        R.rglru_timing_enable(False)


@pytest.mark.parametrize("B,T,bs,nb,windows", [
    (1, 12400, 256, 2, True), (2, 12320, 160, 2, True), (1, 12300, 128, 1, True),   # one long prompt, ragged ends
    (1, 1500, 256, 1, False), (1, 1100, 192, 2, False), (1, 700, 128, 1, False),    # 16 slices
    (1, 65, 256, 1, False), (3, 97, 144, 2, False), (33, 70, 256, 4, False)])       # few, and none
@pytest.mark.parametrize("how", ["plain", "merge", "tanh", "packed"])
def test_fused_forward_with_inputs_off_the_16_byte_grid(B, T, bs, nb, windows, how):
    """u on the 4-byte grid only; the states in place."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act, pos0 = bs * nb, "bf16", 5
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h = at(rn.to_device(inp["u"], act), 2), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    reset = gen.make_resets(B, T, seed=bs, mean_len=400) if how == "packed" else None
    brd, y, out, sh = rn.to_device(br, act), dp.empty_act(B, T, D), dp.empty_act(B, T, D), dp.shape()
    with Names() as k:
        if how == "packed":
            ws, n = dp.workspace(sh, R.OP_FORWARD_PACKED)
            R.rglru_forward_packed(sh, dp.params, u, torch.from_numpy(reset).cuda(), h, ring, pos0, y, h, ring, ws, n)
        elif how == "plain":
            ws, n = dp.workspace(sh, R.OP_FORWARD)
            R.rglru_forward(sh, dp.params, u, h, ring, pos0, y, h, ring, ws, n)
        else:
            ws, n = dp.workspace(sh, R.OP_FORWARD_MERGE)
            R.rglru_forward_merge(sh, dp.params, u, brd, h, ring, pos0, R.MERGE_GELU_TANH if how == "tanh" else 0, out, y, h, ring, ws, n)
    assert "fwd_tile_kernel" not in k.ran and ("fwd_agg_mfma_kernel" in k.ran) == (windows and how != "packed"), k.ran
    assert k.ran & {"fwd_mfma_kernel", "fwd_merge_mfma_kernel", "fwd_packed_mfma_kernel"}, k.ran
    want = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], conv_b=q["conv_b"], h0=q["h0"],
                          state_in=q["state"], reset=reset)
    assert gen.rel_err(rn.to_host(y), want[0]) < BF16 and gen.rel_err(rn.to_host(h), want[1]) < BF16
    np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(ring), pos0 + T), want[2])
    if how in ("merge", "tanh"):
        assert gen.rel_err(rn.to_host(out), oracle.merge(want[0], br, approx=how == "tanh")) < BF16


def test_windows_replay_as_a_hip_graph():
    """Ring pass, aggregate pass, chain and forward of a long prompt off the 16-byte grid: every replay gives the bits of the
    eager run, whatever the workspace held."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    B, T, D, act = 1, 12500, 256, "bf16"
    inp = gen.make_inputs(B, T, D, 1, act=act, seed=23, h0=True)
    dp = rn.DeviceProblem(inp, B, T, D, 1, act)
    u, h0, sh = at(rn.to_device(inp["u"], act), 2), rn.to_device(inp["h0"], "f32"), dp.shape()
    ws, n = dp.workspace(sh, R.OP_FORWARD)
    outs = dict(y=dp.empty_act(B, T, D), hT=dp.empty_f32(B, D), st=dp.empty_act(B, 3, D))

    def step(stream):
        R.rglru_forward(sh, dp.params, u, h0, None, 0, outs["y"], outs["hT"], outs["st"], ws, n, stream)

    with Names() as k:
        step(torch.cuda.current_stream().cuda_stream)
    assert "fwd_agg_mfma_kernel" in k.ran, k.ran
    eager = {k: v.clone() for k, v in outs.items()}
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(torch.cuda.current_stream().cuda_stream)
    for rep in range(3):
        for v in outs.values():
            v.fill_(7.0)
        ws.fill_(rep + 1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, v in outs.items():
            assert torch.equal(v, eager[k]), (rep, k)


@pytest.mark.parametrize("B,T,nb", [(1, 1, 1), (2, 31, 1), (2, 130, 2), (1, 1500, 1), (33, 70, 4)])
@pytest.mark.parametrize("how", ["plain", "merge", "packed"])
def test_backward_of_256_channels_off_the_16_byte_grid(B, T, nb, how):
    """dy (dout) on the 4-byte grid only: gates, products and weight gradients as kernels of their own."""
    import torch
    rn = runner()
    D, act, pos0 = 256 * nb, "bf16", 7
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + B, h0=True, state=True, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0, dhT = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dhT"], "f32")
    ring, dy = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act), at(rn.to_device(inp["dy"], act), 2)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"], dhT=q["dhT"])
    dev = dict(h0=h0, state_in=ring, pos0=pos0)
    if how == "packed":
        reset = gen.make_resets(B, T, seed=T, mean_len=20)
        rs = torch.from_numpy(reset).cuda()
        y, _, _ = dp.forward_packed(u, rs, **dev)
        with Names() as k:
            got = dp.backward_packed(u, rs, y, dy, dhT=dhT, **dev)
        ref = oracle.backward(q["u"], *w, q["dy"], reset=reset, **kw)
    elif how == "plain":
        y, _, _ = dp.forward(u, **dev)
        with Names() as k:
            got = dp.backward(u, y, dy, dhT=dhT, **dev)
        ref = oracle.backward(q["u"], *w, q["dy"], **kw)
    else:
        br = gen.make_branch(B, T, D, act=act, seed=T)
        brd = rn.to_device(br, act)
        _, y, _, _ = dp.forward_merge(u, brd, **dev)
        with Names() as k:
            got = dp.backward_merge(u, brd, y, dy, dhT=dhT, **dev)
        ref = oracle.backward_merge(q["u"], br, *w, q["dy"], **kw)
    assert ("bwd_gates_packed_kernel" if how == "packed" else "bwd_gates_kernel") in k.ran and "bwd_tile_kernel" not in k.ran, k.ran
    for name in ref:
        assert gen.rel_err(rn.to_host(got[name]), ref[name]) < BF16, name


@pytest.mark.parametrize("B,T,bs,nb", [(1, 16, 112, 1), (2, 100, 128, 2), (1, 300, 160, 2), (2, 65, 240, 1), (2, 300, 352, 2), (1, 257, 448, 1),
                                       (2, 100, 512, 1)])
@pytest.mark.parametrize("merge", [False, True])
def test_backward_in_a_workspace_the_tiles_do_not_fit(B, T, bs, nb, merge):
    """The largest workspace, in steps of a fiftieth of what is asked for, in which the passes take over."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=bs + T, h0=True, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    brd = rn.to_device(br, act)
    y, _, _ = dp.forward(u, h0=h0)
    asked = R.rglru_workspace_bytes(dp.shape(), R.OP_BACKWARD_MERGE if merge else R.OP_BACKWARD)
    ws = torch.empty(asked, dtype=torch.uint8, device="cuda:0")
    for k in range(50, 0, -1):
        size = asked * k // 50 // 256 * 256
        dp.workspace = lambda shape, op: (ws, size)
        with Names() as names:
            got = dp.backward_merge(u, brd, y, dy, h0=h0) if merge else dp.backward(u, y, dy, h0=h0)
        if "bwd_tile_kernel" not in names.ran:
            break
    assert {"adjoint_kernel", "wgrad_pass_kernel"} <= names.ran, (k, names.ran)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"])
    ref = oracle.backward_merge(q["u"], br, *w, q["dy"], **kw) if merge else oracle.backward(q["u"], *w, q["dy"], **kw)
    for name in ref:
        assert gen.rel_err(rn.to_host(got[name]), ref[name]) < BF16, name


@pytest.mark.parametrize("B,T,bs,nb", [(2, 2000, 128, 2), (2, 1500, 352, 1), (1, 600, 384, 2), (1, 333, 448, 4), (1, 40, 272, 16)])
def test_packed_rows_in_fp32_arithmetic(B, T, bs, nb):
    """Packed rows of the blocks that no fused kernel takes run in plain fp32 arithmetic: what leaves in fp32 - the state of the forward, and
    in the backward (given the exact y, rounded once) the gradients that h_{t-1} does not enter - is that of fp32 sums over
    the longest row: 8 sqrt(T) 2^-24 of its scale."""
    import torch
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    reset = gen.make_resets(B, T, seed=bs, mean_len=200)
    rs = torch.from_numpy(reset).cuda()
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], reset=reset)
    y_ref, hT_ref, _ = oracle.forward(q["u"], *w, **kw)
    ref = oracle.backward(q["u"], *w, q["dy"], **kw)
    tol = 8 * np.sqrt(T) * 2.0 ** -24
    n2 = lambda a, b: np.linalg.norm(np.asarray(a, np.float64) - b) / np.linalg.norm(b)
    if bs > 256:
        _, hT, _ = dp.forward_packed(u, rs, h0=h0)
        assert n2(rn.to_host(hT), hT_ref) < tol
    y = rn.to_device(gen.round_to_act(y_ref.astype(np.float32), act), act)
    got = dp.backward_packed(u, rs, y, dy, h0=h0)
    for k in ("dh0", "dW_x", "db_x"):
        assert n2(rn.to_host(got[k]), ref[k]) < tol, k
