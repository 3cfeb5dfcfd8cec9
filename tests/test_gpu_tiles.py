"""The kernels in tiles (rglru_bwd_fused.h, rglru_fwd_tile.h): tile edges, block sizes either side of a wave's 32 channels, the merge,
packed rows, time slices, against the float64 oracle; 2^-6 as for the other bf16 kernels (8-bit results, 11-bit products)."""
import struct

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


def names_of(R):
    return [R.rglru_timing_get(i)[0] for i in range(R.rglru_timing_count())]


@pytest.mark.parametrize("B,T,bs,nb,slices", [
    (1, 1, 128, 1, 0), (2, 31, 144, 2, 0), (1, 33, 160, 1, 0), (3, 32, 176, 1, 1), (1, 63, 192, 2, 0), (2, 64, 208, 1, 0),
    (1, 65, 240, 1, 0), (2, 128, 256, 1, 1), (1, 129, 256, 2, 3), (1, 97, 272, 1, 0), (1, 640, 352, 1, 5), (2, 95, 384, 1, 0),
    (1, 160, 432, 1, 2), (1, 2100, 160, 1, 0), (1, 33, 512, 1, 0), (2, 129, 496, 1, 2),
    (1, 40, 112, 2, 0), (2, 33, 288, 1, 0), (1, 95, 320, 1, 0), (1, 65, 416, 1, 0), (2, 64, 464, 1, 1), (1, 97, 480, 1, 3)])
@pytest.mark.parametrize("how", ["plain", "merge", "tanh", "packed"])
def test_tiles(B, T, bs, nb, slices, how):
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act, pos0 = bs * nb, "bf16", 7
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0, dhT = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dhT"], "f32")
    ring, dy = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act), rn.to_device(inp["dy"], act)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    dev = dict(h0=h0, state_in=ring, pos0=pos0)
    # (room for the tiles at every size)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    dp.workspace = lambda shape, op: (ws, ws.numel())
    R.rglru_set_max_time_slices(slices)
    try:
        if how == "packed":
            reset = gen.make_resets(B, T, seed=bs, mean_len=20)
            rs = torch.from_numpy(reset).cuda()
            y, _, _ = dp.forward_packed(u, rs, **dev)
            R.rglru_timing_enable(True)
            got = dp.backward_packed(u, rs, y, dy, dhT=dhT, **dev)
            ref = oracle.backward(q["u"], *w, q["dy"], dhT=q["dhT"], reset=reset, **kw)
        elif how == "plain":
            y, _, _ = dp.forward(u, **dev)
            R.rglru_timing_enable(True)
            got = dp.backward(u, y, dy, dhT=dhT, **dev)
            ref = oracle.backward(q["u"], *w, q["dy"], dhT=q["dhT"], **kw)
        else:
            br, flags = gen.make_branch(B, T, D, act=act, seed=T), R.MERGE_GELU_TANH if how == "tanh" else 0
            brd = rn.to_device(br, act)
            _, y, _, _ = dp.forward_merge(u, brd, flags=flags, **dev)
            R.rglru_timing_enable(True)
            got = dp.backward_merge(u, brd, y, dy, dhT=dhT, flags=flags, **dev)
            ref = oracle.backward_merge(q["u"], br, *w, q["dy"], dhT=q["dhT"], approx=how == "tanh", **kw)
        names = names_of(R)
    finally:
        R.rglru_timing_enable(False)
        R.rglru_set_max_time_slices(0)
    merged = how in ("merge", "tanh")
    # (LDS does not hold wider tiles with the merge; packed rows of other blocks run on the general kernels)
    assert ("bwd_tile_kernel" in names and "tile_wgrad_kernel" in names) == (bs <= 352 if merged else bs == 256 if how == "packed" else True), names
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k


def least_room(runs, least, most):
    """The smallest workspace, in steps of 256 bytes, in which `runs` says yes (it does at `most`, and not below `least`)."""
    lo, hi = least // 256, most // 256
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if runs(mid * 256) else (mid + 1, hi)
    return hi * 256


@pytest.mark.parametrize("B,T,bs,nb,packed", [
    (1, 16384, 256, 1, False), (1, 16448, 256, 1, False), (8, 2100, 240, 1, False), (3, 1000, 352, 1, False), (12, 300, 512, 1, False),
    (1, 900, 160, 3, False), (1, 700, 112, 1, False), (4, 300, 128, 8, False), (2, 500, 192, 4, False), (3, 200, 320, 2, False),
    (3, 800, 288, 1, False), (2, 300, 256, 2, False), (1, 16384, 256, 1, True), (2, 300, 256, 2, True)])
def test_weight_gradients_in_slices(B, T, bs, nb, packed):
    """Tiles of half and of all columns of a block, in as many slices of the stages as pay (the reported workspace) and in fewer, down to
    those of the smallest workspace in which the tiles run. Half-precision adjoints and inputs (11 bits): 2^-6 as above; sums in another
    order, of up to 16448 terms: sqrt(16448) 2^-24 = 2^-17 of their scale, 2^-14 for single elements."""
    import paper_2402_19427_amd as R
    import torch
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, dy = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act)
    reset = gen.make_resets(B, T, seed=bs, mean_len=90) if packed else None
    rs = torch.from_numpy(reset).cuda() if packed else None
    y, _, _ = dp.forward_packed(u, rs) if packed else dp.forward(u)
    ref = oracle.backward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], q["dy"], conv_b=q["conv_b"], reset=reset)
    asked = R.rglru_workspace_bytes(dp.shape(), R.OP_BACKWARD_PACKED if packed else R.OP_BACKWARD)
    ws, one, got = torch.empty(asked, dtype=torch.uint8, device="cuda:0"), nb * 2 * bs * bs * 4, {}

    def runs(n):
        dp.workspace = lambda shape, op: (ws, n)
        R.rglru_timing_enable(True)
        try:
            got[n] = dp.backward_packed(u, rs, y, dy) if packed else dp.backward(u, y, dy)
            torch.cuda.synchronize()
            return "tile_wgrad_kernel" in names_of(R)
        except R.RglruError as e:
            assert e.code == R.ERR_WORKSPACE
            return False
        finally:
            R.rglru_timing_enable(False)

    least = least_room(runs, 256, asked)
    sizes = sorted({asked, least, min(least + one, asked), min(least + 3 * one, asked)})
    print("workspace:", sizes, "a slice:", one)
    assert len(sizes) > 1 or packed or T > 16000   # (there the general kernels' room is the least that is accepted)
    for n in sizes:
        assert runs(n), n
        for k in ref:
            assert gen.rel_err(rn.to_host(got[n][k]), ref[k]) < BF16, (n, k)
    for n in sizes:
        for k in ("dW_a", "dW_x"):
            assert gen.rel_err(rn.to_host(got[n][k]), rn.to_host(got[asked][k])) < 2.0 ** -14, (n, k)


@pytest.mark.parametrize("B,T,bs,nb,slices", [
    (1, 1, 128, 1, 0), (2, 33, 128, 2, 0), (1, 129, 144, 2, 0), (1, 700, 160, 2, 3), (2, 160, 176, 1, 0), (1, 191, 192, 1, 1),
    (1, 257, 208, 1, 0), (1, 3000, 256, 2, 0), (3, 319, 256, 1, 4), (1, 320, 240, 1, 0), (1, 2, 320, 4, 0), (2, 31, 384, 2, 0),
    (1, 97, 448, 4, 2), (1, 64, 480, 8, 0), (1, 33, 512, 1, 0),
    (1, 70, 112, 16, 0), (2, 65, 288, 8, 0), (1, 40, 416, 8, 0), (1, 66, 464, 16, 1), (1, 600, 352, 8, 5)])
@pytest.mark.parametrize("how", ["plain", "merge", "tanh", "packed"])
def test_forward_tiles(B, T, bs, nb, slices, how):
    """The forward: y, the merge's product, the last state and the ring handed on."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act, pos0 = bs * nb, "bf16", 5
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act)
    w = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    dp.workspace = lambda shape, op: (ws, ws.numel())
    R.rglru_set_max_time_slices(slices)
    R.rglru_timing_enable(True)
    try:
        out = None
        if how == "packed":
            reset = gen.make_resets(B, T, seed=bs, mean_len=20)
            y, hT, st = dp.forward_packed(u, torch.from_numpy(reset).cuda(), h0=h0, state_in=ring, pos0=pos0)
            want = oracle.forward(q["u"], *w, reset=reset, **kw)
        elif how == "plain":
            y, hT, st = dp.forward(u, h0=h0, state_in=ring, pos0=pos0)
            want = oracle.forward(q["u"], *w, **kw)
        else:
            br, flags = gen.make_branch(B, T, D, act=act, seed=T), R.MERGE_GELU_TANH if how == "tanh" else 0
            out, y, hT, st = dp.forward_merge(u, rn.to_device(br, act), flags=flags, h0=h0, state_in=ring, pos0=pos0)
            want = oracle.forward(q["u"], *w, **kw)
        names = names_of(R)
    finally:
        R.rglru_timing_enable(False)
        R.rglru_set_max_time_slices(0)
    if D % 256 == 0 or bs <= 256:
        assert ("fwd_tile_kernel" in names) == (bs <= 480 and (how != "packed" or 128 <= bs <= 256)), names   # (the others: general kernels)
    assert gen.rel_err(rn.to_host(y), want[0]) < BF16
    assert gen.rel_err(rn.to_host(hT), want[1]) < BF16
    np.testing.assert_array_equal(rn.to_host(st), gen.ring_from_chrono(np.asarray(want[2], np.float32), pos0 + T))
    if out is not None:
        assert gen.rel_err(rn.to_host(out), oracle.merge(want[0], br, approx=how == "tanh")) < BF16


@pytest.mark.parametrize("B,T,bs,nb", [(1, 700, 160, 2), (2, 330, 256, 2), (1, 600, 352, 8), (1, 97, 448, 4), (1, 33, 128, 2)])
@pytest.mark.parametrize("how", ["plain", "merge", "packed"])
def test_states_in_place_in_slices(B, T, bs, nb, how):
    """h0 and hT, and the rings, are the same memory while other slices still read it: the bits of the call with separate ones."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    if how == "packed" and bs > 256:
        pytest.skip("packed rows of such blocks run on the general kernels")
    D, act, pos0 = bs * nb, "bf16", 4
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, bias=True)
    dp = rn.DeviceProblem(inp, B, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring0 = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act)
    br, rs = rn.to_device(gen.make_branch(B, T, D, act=act, seed=2), act), torch.from_numpy(gen.make_resets(B, T, seed=bs, mean_len=90)).cuda()
    sh = dp.shape()
    op = {"plain": R.OP_FORWARD, "merge": R.OP_FORWARD_MERGE, "packed": R.OP_FORWARD_PACKED}[how]
    n = R.rglru_workspace_bytes(sh, op)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")

    def call(h_in, h_out, ring_in, ring_out):
        y = dp.empty_act(B, T, D)
        if how == "plain":
            R.rglru_forward(sh, dp.params, u, h_in, ring_in, pos0, y, h_out, ring_out, ws, n)
        elif how == "packed":
            R.rglru_forward_packed(sh, dp.params, u, rs, h_in, ring_in, pos0, y, h_out, ring_out, ws, n)
        else:
            R.rglru_forward_merge(sh, dp.params, u, br, h_in, ring_in, pos0, 0, y, None, h_out, ring_out, ws, n)
        return y, h_out, ring_out

    R.rglru_timing_enable(True)
    try:
        want = call(h0, torch.empty_like(h0), ring0, torch.empty_like(ring0))
        torch.cuda.synchronize()
        assert "fwd_tile_kernel" in names_of(R)
    finally:
        R.rglru_timing_enable(False)
    for _ in range(3):
        h, ring = h0.clone(), ring0.clone()
        for a, b in zip(call(h, h, ring, ring), want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("bs", [160, 256])
def test_a_mark_in_front_of_the_tiles_is_reported_once(bs):
    """The mark an expired wait leaves (planted from the host): sliced calls return NaN until it has been reported."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    B, T, act = 1, 700, "bf16"
    inp = gen.make_inputs(B, T, bs, 1, act=act, seed=3, dy=True)
    dp = rn.DeviceProblem(inp, B, T, bs, 1, act)
    u, dy = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act)
    y, _, _ = dp.forward(u)
    ok = dp.backward(u, y, dy)
    ws, _ = dp.workspace(dp.shape(), R.OP_BACKWARD)
    ws[:16] = torch.tensor(list(struct.pack("<4I", 0x4c474c52, 0x58452d55, 0x45524950, 0xb3d3b3ad)), dtype=torch.uint8, device="cuda:0")
    bad = dp.backward(u, y, dy)
    assert torch.isnan(bad["du"].float()).all()
    with pytest.raises(R.RglruError) as e:
        R.rglru_workspace_status(dp.shape(), R.OP_BACKWARD, ws)
    assert e.value.code == R.ERR_TIMEOUT
    R.rglru_workspace_status(dp.shape(), R.OP_BACKWARD, ws)
    again = dp.backward(u, y, dy)
    for k in ok:
        assert torch.equal(again[k], ok[k]), k


@pytest.mark.parametrize("bs,nb,T", [(128, 2, 33), (160, 2, 161), (192, 2, 130), (240, 2, 321), (256, 2, 321), (384, 2, 289), (448, 4, 333)])
@pytest.mark.parametrize("how", ["plain", "merge", "packed"])
def test_state_behind_infinite_last_inputs(bs, nb, T, how):
    """T is no multiple of the tile: the Conv1D of the steps past the end still sees the last inputs. The state handed on is that of
    the last step whatever they hold (one infinity per block, in its first and in its last step of reach; a decay of zero):
    y in more digits, so that the two differ by half an ulp of bf16."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    if how == "packed" and bs > 256:
        pytest.skip("packed rows of such blocks run on the general kernels")
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=T + bs, h0=True, bias=True)
    inp["u"][0, T - 1, 3] = np.inf
    inp["u"][0, T - 3, bs + 5] = -np.inf
    inp["Lambda"][7] = -1e38
    dp = rn.DeviceProblem(inp, 1, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    dp.workspace = lambda shape, op: (ws, ws.numel())
    R.rglru_timing_enable(True)
    try:
        if how == "packed":
            y, hT, _ = dp.forward_packed(u, torch.from_numpy(gen.make_resets(1, T, seed=bs, mean_len=20)).cuda(), h0=h0)
        elif how == "plain":
            y, hT, _ = dp.forward(u, h0=h0)
        else:
            _, y, hT, _ = dp.forward_merge(u, rn.to_device(gen.make_branch(1, T, D, act=act, seed=1), act), h0=h0)
        torch.cuda.synchronize()
        names = names_of(R)
    finally:
        R.rglru_timing_enable(False)
    assert "tile_prep_kernel" in names, names
    last, hT = rn.to_host(y)[0, -1].astype(np.float64), rn.to_host(hT)[0].astype(np.float64)
    ok = np.isfinite(last)
    assert ok.sum() >= D - 2
    np.testing.assert_array_equal(np.isfinite(hT), ok)
    assert (np.abs(hT[ok] - last[ok]) <= np.abs(hT[ok]) * 2.0 ** -8 + 1e-37).all()


@pytest.mark.parametrize("bs,nb,T", [(112, 2, 33), (160, 2, 70), (256, 2, 97), (352, 2, 50), (416, 1, 33), (512, 1, 45)])
@pytest.mark.parametrize("how", ["plain", "merge", "packed"])
def test_backward_of_a_ragged_tile_ignores_what_lies_past_the_end(bs, nb, T, how):
    """The last y would be h_{t-1} of the first step past the end only (with the merge of dbranch's last step, too): not a bit may depend
    on it. And the Conv1D past the end, infinite here where no step inside the sequence is, adds nothing to any gradient: the channel's gates
    are closed (i_t x_t stays below 2), and the one gradient that takes its inputs as they are is left out."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=T + bs, dy=True, bias=True)
    c = 5
    inp["u"][0, T - 1, c] = gen.round_to_act(np.array([3e38], np.float32), act)[0]
    inp["conv_w"][:, c] = (0.25, 4.0, 0.0, 0.0)
    inp["W_a"][0, c], inp["W_x"][0, c], inp["b_x"][c] = 0.0, 0.0, -100.0
    dp = rn.DeviceProblem(inp, 1, T, D, nb, act)
    u, dy, dhT = rn.to_device(inp["u"], act), rn.to_device(inp["dy"], act), rn.to_device(inp["dhT"], "f32")
    y = rn.to_device(np.random.default_rng(bs).standard_normal((1, T, D), dtype=np.float32), act)
    br = rn.to_device(gen.make_branch(1, T, D, act=act, seed=T), act)
    reset = torch.from_numpy(gen.make_resets(1, T, seed=bs, mean_len=20)).cuda()
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    dp.workspace = lambda shape, op: (ws, ws.numel())

    def call(y):
        R.rglru_timing_enable(True)
        try:
            if how == "plain":
                g = dp.backward(u, y, dy, dhT=dhT)
            elif how == "packed":
                g = dp.backward_packed(u, reset, y, dy, dhT=dhT)
            else:
                g = dp.backward_merge(u, br, y, dy, dhT=dhT)
                g["dbranch"] = g["dbranch"][:, :-1]
            torch.cuda.synchronize()
            assert "tile_prep_kernel" in names_of(R)
        finally:
            R.rglru_timing_enable(False)
        return {k: v.cpu() for k, v in g.items() if v is not None}

    if how == "merge" and bs > 352 or how == "packed" and bs != 256:
        pytest.skip("LDS does not hold the merge of such blocks; packed rows of others than 256 channels run on the general kernels")
    want = call(y)
    for k, v in want.items():
        v = v.float()
        if k == "dconv_w":
            v = torch.cat((v[:, :c], v[:, c + 1:]), 1)
        assert torch.isfinite(v).all(), k
    y[0, -1] = float("inf")
    got = call(y)
    for k in want:
        assert torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("bs,nb,T", [(64, 4, 40), (128, 2, 40), (160, 2, 140), (256, 1, 300), (352, 8, 40), (512, 1, 40)])
def test_weights_past_half_precision(bs, nb, T):
    """Finite weights stop at 65504 in the products (here they meet inputs of zero, where an infinity would be a NaN): the
    oracle's results with weights that end there."""
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=bs, h0=True, dy=True, bias=True)
    for k, v in (("W_a", 1e5), ("W_x", -3e38)):
        inp[k][0, 9, 4] = gen.round_to_act(np.array([v], np.float32), act)[0]
    inp["u"][:, :, 4], inp["conv_b"][4] = 0.0, 0.0
    dp = rn.DeviceProblem(inp, 1, T, D, nb, act)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    y, hT, _ = dp.forward(u, h0=h0)
    got = dp.backward(u, y, dy, h0=h0)
    q = f64(inp)
    w = (np.clip(q["W_a"], -65504, 65504), np.clip(q["W_x"], -65504, 65504), q["b_a"], q["b_x"], q["Lambda"], q["conv_w"])
    want = oracle.forward(q["u"], *w, conv_b=q["conv_b"], h0=q["h0"])
    ref = oracle.backward(q["u"], *w, q["dy"], conv_b=q["conv_b"], h0=q["h0"])
    assert gen.rel_err(rn.to_host(y), want[0]) < BF16 and gen.rel_err(rn.to_host(hT), want[1]) < BF16
    for k in ref:   # (the channel such a weight leads to and the others on scales of their own)
        a, b = rn.to_host(got[k]), ref[k]
        if k in ("dW_a", "dW_x"):
            assert gen.rel_err(a, b) < BF16, k
            continue
        for at in (np.arange(D) == 4, np.arange(D) != 4):
            assert gen.rel_err(a[..., at], b[..., at]) < BF16, k


@pytest.mark.parametrize("B,T,bs,nb,how", [
    (1, 9, 256, 2, "plain"), (2, 20, 256, 1, "plain"), (3, 32, 160, 2, "merge"), (1, 33, 256, 1, "packed"), (2, 64, 224, 1, "tanh"),
    (1, 100, 192, 2, "packed"), (3, 128, 144, 1, "plain"), (1, 255, 208, 2, "merge"), (2, 256, 256, 2, "packed"), (1, 257, 256, 2, "plain"),
    (130, 40, 256, 1, "merge"), (1, 800, 240, 2, "merge")])
def test_short_forward(B, T, bs, nb, how):
    """Short sequences run in tiles of 32 steps in the workspace that is asked for, and on the fused kernel in the least it takes (no
    records where a sequence is one tile: the status word and one gate's weights)."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act, pos0 = bs * nb, "bf16", 9
    inp = gen.make_inputs(B, T, D, nb, act=act, seed=T + bs, h0=True, state=True, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    ring = rn.to_device(gen.ring_from_chrono(inp["state"], pos0), act)
    br = gen.make_branch(B, T, D, act=act, seed=T)
    reset = gen.make_resets(B, T, seed=bs, mean_len=20) if how == "packed" else None
    kw = dict(conv_b=q["conv_b"], h0=q["h0"], state_in=q["state"])
    want = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], reset=reset, **kw)
    dev = dict(h0=h0, state_in=ring, pos0=pos0)
    for least in (False, True) if how == "plain" and T <= 32 else (False,):
        if least:
            ws = torch.empty(256 + nb * 256 * 256 * 2, dtype=torch.uint8, device="cuda:0")
            dp.workspace = lambda shape, op: (ws, ws.numel())
        R.rglru_timing_enable(True)
        try:
            if how == "packed":
                y, hT, st = dp.forward_packed(u, torch.from_numpy(reset).cuda(), **dev)
            elif how == "plain":
                y, hT, st = dp.forward(u, **dev)
            else:
                out, y, hT, st = dp.forward_merge(u, rn.to_device(br, act), flags=R.MERGE_GELU_TANH if how == "tanh" else 0, **dev)
                ref = oracle.merge(want[0], br, approx=how == "tanh")
                assert gen.rel_err(rn.to_host(out), ref) < BF16
            torch.cuda.synchronize()
            names = names_of(R)
        finally:
            R.rglru_timing_enable(False)
        assert ("fwd_tile_kernel" in names) == (not least), names
        assert gen.rel_err(rn.to_host(y), want[0]) < BF16 and gen.rel_err(rn.to_host(hT), want[1]) < BF16
        np.testing.assert_array_equal(gen.chrono_from_ring(rn.to_host(st), pos0 + T), want[2])


@pytest.mark.parametrize("B,T,nb,merge,tiles", [
    (5, 300, 10, False, True), (6, 2000, 10, False, False), (10, 700, 10, False, True), (8, 640, 16, False, True), (8, 700, 16, False, False),
    (4, 640, 10, True, True), (4, 700, 10, True, False), (13, 300, 10, True, True), (14, 300, 16, True, False)])
def test_forward_of_many_units_takes_the_faster_kernel(B, T, nb, merge, tiles):
    """Either side of the rule for 33 units of 256 channels and more."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = 256 * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=T + nb, bias=True)
    dp, q = rn.DeviceProblem(inp, B, T, D, nb, act), f64(inp)
    u = rn.to_device(inp["u"], act).expand(B, T, D).contiguous()
    R.rglru_timing_enable(True)
    try:
        if merge:
            br = gen.make_branch(1, T, D, act=act, seed=T)
            out, y, _, _ = dp.forward_merge(u, rn.to_device(br, act).expand(B, T, D).contiguous())
        else:
            y, _, _ = dp.forward(u)
        torch.cuda.synchronize()
        names = names_of(R)
    finally:
        R.rglru_timing_enable(False)
    assert ("fwd_tile_kernel" in names) == tiles, names
    want = oracle.forward(q["u"], q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"], conv_b=q["conv_b"])[0]
    assert torch.equal(y, y[:1].expand(B, T, D))
    assert gen.rel_err(rn.to_host(y[:1]), want) < BF16
    if merge:
        assert gen.rel_err(rn.to_host(out[-1:]), oracle.merge(want, br)) < BF16


@pytest.mark.parametrize("B,T,bs,nb,merge,tiles", [
    (2, 1400, 256, 16, False, True), (2, 2048, 256, 16, False, False), (3, 2048, 256, 10, False, True),   # 29 - 32 units: not in between
    (1, 512, 256, 16, False, True), (1, 512, 256, 16, True, False), (1, 640, 256, 16, True, True),        # as many rounds, half as many
    (1, 300, 240, 16, False, False), (1, 300, 240, 10, False, True), (2, 4096, 256, 10, True, False), (2, 3000, 256, 10, True, True),
    (1, 1024, 240, 32, False, False), (4, 1024, 176, 16, False, False), (3, 1024, 176, 16, False, True), (4, 200, 176, 16, False, True),
    (8, 300, 176, 16, True, False), (8, 2048, 176, 16, True, True), (1, 1024, 192, 32, False, False), (1, 300, 192, 32, False, True),
    (2, 300, 160, 32, True, False), (2, 400, 160, 32, True, True), (2, 300, 160, 32, False, True)])
def test_forward_takes_the_faster_kernel(B, T, bs, nb, merge, tiles):
    """Either side of the rule between the tiles and the fused kernel; y is the same but for the rounding of its last bits."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    g = torch.Generator(device="cuda").manual_seed(T + bs)
    rand = lambda *s, k=1.0: torch.randn(*s, generator=g, device="cuda") * k
    bf = lambda t: t.to(torch.bfloat16)
    weights = (bf(rand(nb, bs, bs, k=bs ** -0.5)), bf(rand(nb, bs, bs, k=bs ** -0.5)), rand(D, k=0.1), rand(D, k=0.1),
               torch.full((D,), 4.0, device="cuda"), rand(4, D, k=0.5), rand(D, k=0.1))
    par = R.make_params(*weights)
    u, br, y, out, hT = bf(rand(B, T, D)), bf(rand(B, T, D)), bf(rand(B, T, D)), bf(rand(B, T, D)), rand(B, D)
    sh = R.make_shape(B, T, D, nb, R.BF16)

    def call(cap):
        R.rglru_set_max_time_slices(cap)
        n = R.rglru_workspace_bytes(sh, R.OP_FORWARD_MERGE if merge else R.OP_FORWARD)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        R.rglru_timing_enable(True)
        try:
            if merge:
                R.rglru_forward_merge(sh, par, u, br, None, None, 0, 0, out, y, hT, None, ws, n, None)
            else:
                R.rglru_forward(sh, par, u, None, None, 0, y, hT, None, ws, n, None)
            torch.cuda.synchronize()
            return names_of(R), y.float().clone(), hT.clone()
        finally:
            R.rglru_timing_enable(False)
            R.rglru_set_max_time_slices(0)

    names, a, h = call(0)
    # (a merge that neither kernel has as its epilogue there runs behind the plain forward)
    assert ("fwd_tile_kernel" in names and "merge_fwd_kernel" not in names) == tiles, names
    _, b, k = call(1)
    assert ((a - b).norm() / b.norm()).item() < 2.0 ** -9 and ((h - k).norm() / k.norm()).item() < 2.0 ** -9


@pytest.mark.parametrize("B,T,bs,nb,how,tiles", [
    (1, 9, 176, 44, "plain", True), (1, 9, 176, 45, "plain", False), (1, 9, 176, 45, "packed", True), (1, 32, 208, 33, "plain", False),
    (1, 20, 208, 51, "merge", True), (1, 20, 208, 52, "merge", False), (1, 64, 240, 25, "plain", True), (1, 64, 240, 26, "plain", False),
    (1, 64, 240, 19, "merge", True), (1, 64, 240, 20, "merge", False), (1, 200, 208, 51, "plain", True), (1, 200, 208, 52, "plain", False),
    (1, 64, 240, 39, "packed", True), (1, 64, 240, 40, "packed", False), (2, 64, 240, 50, "plain", True), (2, 64, 240, 39, "merge", True),
    (2, 64, 240, 40, "merge", False), (2, 33, 160, 100, "merge", True), (1, 32, 192, 128, "merge", True), (1, 32, 192, 139, "packed", False),
    (8, 64, 208, 24, "plain", False), (8, 32, 208, 24, "plain", True), (8, 64, 208, 24, "merge", True), (8, 160, 240, 16, "plain", False),
    (8, 128, 240, 16, "plain", True), (16, 64, 240, 16, "packed", False), (4, 128, 176, 48, "plain", False), (4, 128, 176, 40, "plain", True),
    (8, 64, 256, 32, "plain", False), (8, 64, 256, 24, "packed", True)])
def test_short_forward_takes_the_faster_kernel(B, T, bs, nb, how, tiles):
    """Either side of the rule by the size of the weights that the tiles prepare; the two kernels' results differ by the rounding of their
    last bits (2^-9 in the 2-norm), seen against the least workspace's fused kernel."""
    import torch
    import paper_2402_19427_amd as R
    D = bs * nb
    g = torch.Generator(device="cuda").manual_seed(T + bs)
    rand = lambda *s, k=1.0: torch.randn(*s, generator=g, device="cuda") * k
    bf = lambda t: t.to(torch.bfloat16)
    weights = (bf(rand(nb, bs, bs, k=bs ** -0.5)), bf(rand(nb, bs, bs, k=bs ** -0.5)), rand(D, k=0.1), rand(D, k=0.1),
               torch.full((D,), 4.0, device="cuda"), rand(4, D, k=0.5), rand(D, k=0.1))
    par, sh = R.make_params(*weights), R.make_shape(B, T, D, nb, R.BF16)
    u, br, y, out, hT = bf(rand(B, T, D)), bf(rand(B, T, D)), bf(rand(B, T, D)), bf(rand(B, T, D)), rand(B, D)
    reset = (torch.rand(B, T, generator=g, device="cuda") < 0.05).to(torch.uint8)
    need = R.rglru_workspace_bytes(sh, {"plain": R.OP_FORWARD, "merge": R.OP_FORWARD_MERGE, "packed": R.OP_FORWARD_PACKED}[how])
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")

    def call(n):
        R.rglru_timing_enable(True)
        try:
            if how == "merge":
                R.rglru_forward_merge(sh, par, u, br, None, None, 0, 0, out, y, hT, None, ws, n, None)
            elif how == "packed":
                R.rglru_forward_packed(sh, par, u, reset, None, None, 0, y, hT, None, ws, n, None)
            else:
                R.rglru_forward(sh, par, u, None, None, 0, y, hT, None, ws, n, None)
            torch.cuda.synchronize()
            return names_of(R), y.float().clone(), hT.clone()
        finally:
            R.rglru_timing_enable(False)

    names, a, h = call(need)
    assert ("fwd_tile_kernel" in names and "merge_fwd_kernel" not in names) == tiles, names
    if tiles:
        names, b, k = call(need - 256)   # (one cell less than the tiles ask for)
        assert "fwd_tile_kernel" not in names, names
        assert ((a - b).norm() / b.norm()).item() < 2.0 ** -9 and ((h - k).norm() / k.norm()).item() < 2.0 ** -9


@pytest.mark.parametrize("T,bs,nb", [(832, 256, 8), (1024, 208, 1), (900, 240, 4)])
@pytest.mark.parametrize("merge", [False, True])
def test_tiles_of_32_steps_in_one_round(T, bs, nb, merge):
    """Where the room makes the plan give up slices, and one round of tiles of 32 steps becomes two, a sequence goes in tiles of 64: the bits
    of a call whose slices are capped at the number of those, which the smaller tiles could only walk in two rounds, too (the state is
    rounded where it enters a tile)."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=T + bs, h0=True, bias=True)
    dp = rn.DeviceProblem(inp, 1, T, D, nb, act)
    u, h0 = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32")
    br = rn.to_device(gen.make_branch(1, T, D, act=act, seed=T), act)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    dp.workspace = lambda shape, op: (ws, ws.numel())

    def call(cap):
        R.rglru_set_max_time_slices(cap)
        R.rglru_timing_enable(True)
        try:
            out = dp.forward_merge(u, br, h0=h0)[1:3] if merge else dp.forward(u, h0=h0)[:2]
            torch.cuda.synchronize()
            assert "fwd_tile_kernel" in names_of(R)
            return out
        finally:
            R.rglru_timing_enable(False)
            R.rglru_set_max_time_slices(0)

    for a, b in zip(call(0), call((T + 63) // 64)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T,bs,nb,merge,tiles,cap", [
    (4096, 112, 1, False, True, 0), (4097, 112, 1, False, False, 0), (6000, 112, 10, False, True, 0), (4096, 192, 1, True, True, 0),
    (4609, 192, 1, True, False, 0), (4096, 224, 1, False, True, 0), (4200, 224, 1, False, False, 0), (3584, 240, 1, True, True, 0),
    (3600, 240, 1, True, False, 0), (15872, 256, 1, True, True, 0), (16000, 256, 1, True, False, 0), (16000, 256, 1, False, True, 0),
    (2560, 320, 1, False, True, 0), (2592, 320, 1, True, False, 0), (2048, 352, 1, True, True, 0), (2100, 352, 1, False, False, 0),
    (4096, 352, 7, False, False, 0), (4096, 352, 8, False, True, 0), (1536, 448, 1, False, True, 0), (1540, 448, 1, False, False, 0),
    (1024, 512, 1, False, True, 0), (1030, 512, 1, False, False, 0), (3584, 512, 11, False, True, 0), (3600, 512, 11, False, False, 0),
    (3600, 512, 12, False, True, 0), (600, 128, 4, False, False, 1)])
def test_backward_takes_the_faster_kernel(T, bs, nb, merge, tiles, cap):
    """Either side of the rule between the tiles and what is parallel over all of time; against the oracle where one block is quick."""
    import torch
    import paper_2402_19427_amd as R
    rn = runner()
    D, act = bs * nb, "bf16"
    inp = gen.make_inputs(1, T, D, nb, act=act, seed=T + bs, h0=True, dy=True, bias=True)
    dp, q = rn.DeviceProblem(inp, 1, T, D, nb, act), f64(inp)
    u, h0, dy = rn.to_device(inp["u"], act), rn.to_device(inp["h0"], "f32"), rn.to_device(inp["dy"], act)
    br = gen.make_branch(1, T, D, act=act, seed=T)
    R.rglru_set_max_time_slices(cap)
    try:
        y, _, _ = dp.forward(u, h0=h0)
        R.rglru_timing_enable(True)
        got = dp.backward_merge(u, rn.to_device(br, act), y, dy, h0=h0) if merge else dp.backward(u, y, dy, h0=h0)
        torch.cuda.synchronize()
        names = names_of(R)
    finally:
        R.rglru_timing_enable(False)
        R.rglru_set_max_time_slices(0)
    assert ("bwd_tile_kernel" in names) == tiles, names
    if nb * T * bs * bs > 600e6:
        return
    w, kw = (q["W_a"], q["W_x"], q["b_a"], q["b_x"], q["Lambda"], q["conv_w"]), dict(conv_b=q["conv_b"], h0=q["h0"])
    ref = oracle.backward_merge(q["u"], br, *w, q["dy"], **kw) if merge else oracle.backward(q["u"], *w, q["dy"], **kw)
    for k in ref:
        assert gen.rel_err(rn.to_host(got[k]), ref[k]) < BF16, k
