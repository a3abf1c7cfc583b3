"""GPU parity of the surrogate-MLP kernels (BF16 matrix cores, FP32
accumulation) with the FP64 oracle that rounds at the same points.

Tolerance (derived from the arithmetic): a BF16 rounding decision taken from
an FP32 sum can differ from the one taken from the FP64 sum by one BF16 step
(2^-8 relative), and FP32 accumulation adds ~K 2^-24.  Each result is
therefore compared with 2^-7 times its magnitude bound (the same products
taken over absolute values), and the median deviation must stay below
1e-4 of the bound, which a dropped term or transposed operand would exceed.
"""
import ctypes as C

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    from paper_2304_01772_amd import _lib
    assert torch.cuda.is_available()
    return _lib.lib()


def _p(t):
    return C.c_void_p(t.data_ptr())


def _close(got, want, bound):
    got, want, bound = (np.asarray(a, np.float64).reshape(-1) for a in (got, want, bound))
    dev = np.abs(got - want)
    assert np.all(dev <= 2.0 ** -7 * bound + 1e-7), np.max(dev / (bound + 1e-30))
    assert np.median(dev / (bound + 1e-30)) < 1e-4


def _run(L, P, x, t, w):
    dev = torch.device("cuda")
    B = x.shape[0]
    Pt = torch.tensor(P, dtype=torch.float32, device=dev)
    xt = torch.tensor(x, dtype=torch.float32, device=dev)
    tt = torch.tensor(t, dtype=torch.float32, device=dev)
    wt = torch.tensor(w, dtype=torch.float32, device=dev)
    y = torch.empty((B, 3), dtype=torch.float32, device=dev)
    act = torch.empty(L.spinmc_mlp_act_floats(B), dtype=torch.float32, device=dev)
    g = torch.empty(mlp.NP, dtype=torch.float32, device=dev)
    dx = torch.empty((B, 4), dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float32, device=dev)
    ws = torch.empty(L.spinmc_mlp_workspace_floats(B), dtype=torch.float32, device=dev)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.spinmc_mlp_forward(_p(Pt), _p(xt), B, _p(y), _p(act), s) == 0
    assert L.spinmc_mlp_backward(_p(Pt), _p(xt), _p(act), _p(tt), _p(wt), B, _p(g), _p(dx),
                                 _p(loss), _p(ws), s) == 0
    torch.cuda.synchronize()
    return y.cpu().numpy(), g.cpu().numpy(), dx.cpu().numpy(), float(loss.item())


@pytest.mark.parametrize("B", [1, 37, 64, 100, 1025])
def test_forward_backward_match_oracle(L, B):
    rng = np.random.default_rng(B)
    P = mlp.init_params(rng)
    P[-3:] = rng.normal(size=3).astype(np.float32) * 0.1
    # nonzero hidden biases
    P[512:640] = rng.normal(size=128).astype(np.float32) * 0.1
    x = rng.normal(size=(B, 4)).astype(np.float32)
    t = rng.normal(size=(B, 3)).astype(np.float32)
    w = np.array([1.0, 0.5, 2.0], np.float32)
    y, g, dx, loss = _run(L, P, x, t, w)
    yo, _ = mlp.forward(P, x)
    go, dxo, losso = mlp.backward(P, x, t, w)
    by, bg, bdx = mlp.magnitude_bounds(P, x, t, w)
    _close(y, yo, by)
    _close(g, go, bg)
    _close(dx, dxo, bdx)
    assert abs(loss - losso) <= 2.0 ** -6 * losso + 1e-6


def test_backward_is_deterministic(L):
    rng = np.random.default_rng(9)
    P = mlp.init_params(rng)
    x = rng.normal(size=(300, 4)).astype(np.float32)
    t = rng.normal(size=(300, 3)).astype(np.float32)
    w = np.ones(3, np.float32)
    a = _run(L, P, x, t, w)
    b = _run(L, P, x, t, w)
    for u, v in zip(a[:3], b[:3]):
        assert np.array_equal(u, v)


def test_adam_matches_oracle(L):
    rng = np.random.default_rng(4)
    dev = torch.device("cuda")
    p = rng.normal(size=mlp.NP).astype(np.float32)
    pt = torch.tensor(p, device=dev)
    mt = torch.zeros(mlp.NP, device=dev)
    vt = torch.zeros(mlp.NP, device=dev)
    po, mo, vo = p.astype(np.float64), np.zeros(mlp.NP), np.zeros(mlp.NP)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for step in range(1, 6):
        g = rng.normal(size=mlp.NP).astype(np.float32)
        gt = torch.tensor(g, device=dev)
        assert L.spinmc_mlp_adam(_p(pt), _p(gt), _p(mt), _p(vt), step, 1e-3, 0.9, 0.999, 1e-8, s) == 0
        po, mo, vo = mlp.adam(po, g, mo, vo, step)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pt.cpu().numpy(), po, rtol=1e-5, atol=1e-6)


def test_train_step_equals_the_separate_calls(L):
    """spinmc_mlp_train_step (forward, backward, reduction fused with Adam)
    leaves parameters, moments, gradient and loss bit-identical to the
    separate forward / backward / adam calls, over three steps, and each
    gradient matches the oracle's."""
    rng = np.random.default_rng(21)
    dev = torch.device("cuda")
    B = 200
    P = mlp.init_params(rng)
    x = torch.tensor(rng.normal(size=(B, 4)).astype(np.float32), device=dev)
    t = torch.tensor(rng.normal(size=(B, 3)).astype(np.float32), device=dev)
    w = torch.tensor([1.0, 0.5, 2.0], dtype=torch.float32, device=dev)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    state = {}
    for name in ("sep", "fused"):
        state[name] = dict(p=torch.tensor(P, device=dev), m=torch.zeros(mlp.NP, device=dev),
                           v=torch.zeros(mlp.NP, device=dev),
                           g=torch.empty(mlp.NP, device=dev), loss=torch.empty(1, device=dev),
                           act=torch.empty(L.spinmc_mlp_act_floats(B), device=dev),
                           ws=torch.empty(L.spinmc_mlp_workspace_floats(B), device=dev))
    y = torch.empty((B, 3), device=dev)
    for step in range(1, 4):
        a = state["sep"]
        p_before = a["p"].cpu().numpy().copy()
        assert L.spinmc_mlp_forward(_p(a["p"]), _p(x), B, _p(y), _p(a["act"]), s) == 0
        assert L.spinmc_mlp_backward(_p(a["p"]), _p(x), _p(a["act"]), _p(t), _p(w), B, _p(a["g"]),
                                     None, _p(a["loss"]), _p(a["ws"]), s) == 0
        assert L.spinmc_mlp_adam(_p(a["p"]), _p(a["g"]), _p(a["m"]), _p(a["v"]), step, 1e-3, 0.9,
                                 0.999, 1e-8, s) == 0
        b = state["fused"]
        assert L.spinmc_mlp_train_step(_p(b["p"]), _p(x), _p(t), _p(w), B, _p(b["g"]), _p(b["m"]),
                                       _p(b["v"]), step, 1e-3, 0.9, 0.999, 1e-8, _p(b["loss"]),
                                       _p(b["act"]), _p(b["ws"]), s) == 0
        torch.cuda.synchronize()
        for k in ("p", "m", "v", "g", "loss"):
            assert torch.equal(a[k], b[k]), (step, k)
        go, _, _ = mlp.backward(p_before, x.cpu().numpy(), t.cpu().numpy(), w.cpu().numpy())
        _, bg, _ = mlp.magnitude_bounds(p_before, x.cpu().numpy(), t.cpu().numpy(),
                                        w.cpu().numpy())
        _close(b["g"].cpu().numpy(), go, bg)


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 65, 32767, 32768, 131073])
def test_forward_sizes_and_alignment(L, B):
    """The forward at the edges of its sample tiles and of its two launch
    forms (from 32768 samples on two tiles a wave), on an input at a 4-byte
    offset from any vector boundary too: outputs and pre-activations against
    the oracle, and the same bits from both alignments."""
    rng = np.random.default_rng(B)
    dev = torch.device("cuda")
    P = mlp.init_params(rng)
    P[512:640] = rng.normal(size=128).astype(np.float32) * 0.1
    x = rng.uniform(-1, 1, size=(B, 4)).astype(np.float32)
    Pt = torch.tensor(P, device=dev)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    outs = []
    for off in (0, 1):
        flat = torch.zeros(4 * B + 4, device=dev)
        flat[off:off + 4 * B] = torch.tensor(x.reshape(-1), device=dev)
        n_act = L.spinmc_mlp_act_floats(B)
        act = torch.full((n_act + 4,), float("nan"), device=dev)
        y = torch.full((B + 1, 3), float("nan"), device=dev)
        assert L.spinmc_mlp_forward(_p(Pt), _p(flat[off:]), B, _p(y), _p(act[off:]), s) == 0
        torch.cuda.synchronize()
        assert torch.isnan(y[B]).all() and torch.isnan(act[off + n_act:]).all()
        outs.append((y[:B].cpu().numpy(), act[off:off + n_act].cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    pick = np.unique(np.linspace(0, B - 1, min(B, 2000)).astype(int))
    yo, cache = mlp.forward(P, x[pick])
    by, _, _ = mlp.magnitude_bounds(P, x[pick], np.zeros((len(pick), 3), np.float32),
                                    np.ones(3, np.float32))
    _close(outs[0][0][pick], yo, by)


@pytest.mark.parametrize("B", [1, 100, 40000])
def test_predict_is_the_scaled_forward(L, B):
    """predict() in one kernel equals scaling, forward and scaling as
    separate tensor operations, bit for bit, and an input that is not a
    contiguous float32 tensor takes those operations."""
    from paper_2304_01772_amd.surrogate import BOX_HI, BOX_LO, SurrogateMLP
    net = SurrogateMLP(seed=3)
    net.y_mu = torch.tensor([0.3, -1.0, 2.0], device="cuda")
    net.y_sd = torch.tensor([0.7, 1.3, 5.0], device="cuda")
    g = np.random.default_rng(B)
    x = torch.tensor(BOX_LO + (BOX_HI - BOX_LO) * g.random((B, 4)), dtype=torch.float32).cuda()
    want = net.forward_normalised(net.normalise_x(x)) * net.y_sd + net.y_mu
    assert torch.equal(net.predict(x), want)
    strided = torch.zeros((B, 8), device="cuda")[:, ::2]
    strided.copy_(x)
    assert torch.equal(net.predict(strided), want)


@pytest.mark.parametrize("B", [1, 16, 63, 64, 65, 1040])
def test_train_step_gradient_at_workgroup_edges(L, B):
    """One training step from zero moments at the edges of the 64-sample
    workgroups and 16-sample tiles, x and act 4 bytes off any vector boundary:
    the gradient, the pre-activations and the loss against the oracle, nothing
    written past the workspace, and a second run with the same bits."""
    rng = np.random.default_rng(300 + B)
    dev = torch.device("cuda")
    P = mlp.init_params(rng)
    P[512:640] = rng.normal(size=128).astype(np.float32) * 0.1
    x = rng.normal(size=(B, 4)).astype(np.float32)
    t = rng.normal(size=(B, 3)).astype(np.float32)
    w = np.array([1.0, 0.5, 2.0], np.float32)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    n_ws = L.spinmc_mlp_workspace_floats(B)
    runs = []
    for _ in range(2):
        p = torch.tensor(P, device=dev)
        xf = torch.zeros(4 * B + 1, device=dev)
        xf[1:] = torch.tensor(x.reshape(-1), device=dev)
        m, v, g = (torch.zeros(mlp.NP, device=dev) for _ in range(3))
        act = torch.empty(L.spinmc_mlp_act_floats(B) + 1, device=dev)
        ws = torch.full((n_ws + 8,), 7.0, device=dev)
        loss = torch.empty(1, device=dev)
        tt, wt = torch.tensor(t, device=dev), torch.tensor(w, device=dev)
        assert L.spinmc_mlp_train_step(_p(p), _p(xf[1:]), _p(tt), _p(wt), B, _p(g), _p(m), _p(v), 1,
                                       1e-3, 0.9, 0.999, 1e-8, _p(loss), _p(act[1:]), _p(ws), s) == 0
        torch.cuda.synchronize()
        assert (ws[n_ws:] == 7.0).all()
        runs.append([a.cpu().numpy() for a in (g, p, loss, act[1:])])
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
    g, _, loss, act = runs[0]
    go, _, losso = mlp.backward(P, x, t, w)
    _, bg, _ = mlp.magnitude_bounds(P, x, t, w)
    _close(g, go, bg)
    assert abs(float(loss[0]) - losso) <= 2.0 ** -6 * losso + 1e-6
    y = torch.empty((B, 3), device=dev)
    act2 = torch.empty(L.spinmc_mlp_act_floats(B), device=dev)
    Pt, xt = torch.tensor(P, device=dev), torch.tensor(x, device=dev)
    assert L.spinmc_mlp_forward(_p(Pt), _p(xt), B, _p(y), _p(act2), s) == 0
    assert np.array_equal(act2.cpu().numpy(), act)


@pytest.mark.parametrize("shapes", [((1,), (4,), (3,), (3,)), ((), (1, 4), (3,), (3,)),
                                    ((4,), (4,), (1,), ()), ((4,), (4,), (1, 3), (5, 3))])
def test_predict_with_broadcast_scaling(L, shapes):
    """Ranges and scales of other shapes than the kernel reads broadcast as
    the separate tensor operations do, and those that need gradients get
    them."""
    from paper_2304_01772_amd.surrogate import SurrogateMLP
    net = SurrogateMLP(seed=4)
    g = np.random.default_rng(5)
    fill = lambda shape, lo: torch.tensor(lo + g.random(shape), dtype=torch.float32).cuda()
    net.x_lo, net.x_hi, net.y_mu, net.y_sd = (
        fill(s, lo) for s, lo in zip(shapes, (-2.0, 1.0, 0.0, 0.5)))
    x = fill((5, 4), 0.0)
    want = net.forward_normalised(net.normalise_x(x)) * net.y_sd + net.y_mu
    assert torch.equal(net.predict(x), want)
    net.y_sd = torch.full((3,), 0.5, device="cuda", requires_grad=True)
    net.predict(x).sum().backward()
    assert net.y_sd.grad is not None


@pytest.mark.parametrize("B", [3, 40000])
def test_silu_of_large_negative_pre_activations(L, B):
    """Pre-activations around -88, where the sigmoid is subnormal but its
    products are not: outputs and gradients through large output weights
    against 64 bits (bf16 of the activation: 2^-8; exponential and subnormal
    sigmoid: below 2^-9), and zero where the exponential overflows."""
    dev = torch.device("cuda")
    P = np.zeros(mlp.NP, np.float32)
    q = mlp.unpack(P)
    q["b2"] = np.linspace(-88.6, -80.0, 128).astype(np.float32).astype(np.float64)
    q["b2"][-1] = -200.0
    q["W3"] = np.zeros((3, 128))
    for j in range(3):  # one neuron an output: the subnormal range, below it, overflow
        q["W3"][j, (5, 90, 127)[j]] = 2.0 ** 100
    P = mlp.pack(q).astype(np.float32)
    x = np.zeros((B, 4), np.float32)
    Pt, xt = torch.tensor(P, device=dev), torch.tensor(x, device=dev)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    y = torch.empty((B, 3), device=dev)
    act = torch.empty(L.spinmc_mlp_act_floats(B), device=dev)
    assert L.spinmc_mlp_forward(_p(Pt), _p(xt), B, _p(y), _p(act), s) == 0
    z = q["b2"][[5, 90, 127]]
    sg = 1.0 / (1.0 + np.exp(-z))
    want = z * sg * 2.0 ** 100
    assert -88.5 < z[0] < -87.5 and 0 < sg[0] < 2.0 ** -126 and z[1] > -87
    yc = y.cpu().numpy()
    assert np.all(np.abs(yc[:, :2] - want[:2]) <= 2.0 ** -7 * np.abs(want[:2]))
    assert np.all(yc[:, 2] == 0)
    # db2 = sum_b 2 w (y - t) / B W3 silu'(z2), with t chosen so that 2 (y - t) / B is 1 / B
    t = torch.tensor(yc - 0.5, device=dev)
    w = torch.ones(3, device=dev)
    g = torch.empty(mlp.NP, device=dev)
    loss = torch.empty(1, device=dev)
    ws = torch.empty(L.spinmc_mlp_workspace_floats(B), device=dev)
    assert L.spinmc_mlp_backward(_p(Pt), _p(xt), _p(act), _p(t), _p(w), B, _p(g), None, _p(loss),
                                 _p(ws), s) == 0
    db2 = mlp.unpack(g.cpu().numpy())["b2"][[5, 90]]
    ref = (sg * (1.0 + z * (1.0 - sg)))[:2] * 2.0 ** 100
    assert np.all(np.abs(db2 - ref) <= 2.0 ** -8 * np.abs(ref))


def test_forward_of_the_largest_batch(L):
    """The last samples of a batch of 2^31 - 1 (34 GB of inputs) are those of
    a small batch."""
    B, n = 2 ** 31 - 1, 100
    if torch.cuda.mem_get_info()[0] < 80 * 2 ** 30:
        pytest.skip("needs 60 GB of free device memory")
    rng = np.random.default_rng(6)
    dev = torch.device("cuda")
    Pt = torch.tensor(mlp.init_params(rng), device=dev)
    tail = torch.tensor(rng.uniform(-1, 1, size=(n, 4)).astype(np.float32), device=dev)
    x = torch.zeros((B, 4), device=dev)
    x[-n:] = tail
    y = torch.full((B, 3), float("nan"), device=dev)
    want = torch.empty((n, 3), device=dev)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.spinmc_mlp_forward(_p(Pt), _p(x), B, _p(y), None, s) == 0
    assert L.spinmc_mlp_forward(_p(Pt), _p(tail), n, _p(want), None, s) == 0
    assert torch.equal(y[-n:], want)
    assert not torch.isnan(y[:: 2 ** 20]).any()
    del x, y
    torch.cuda.empty_cache()
