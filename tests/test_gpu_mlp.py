"""GPU network kernels against the FP64 numpy oracle (BF16 operands, FP32
accumulation).

Element by element: every output and every gradient entry equals the
oracle's network evaluated at BF16 operands (both factors of every product
rounded to BF16, the precision the network is specified in; sums in FP64)
within 2^-8 of the absolute product sums of the GEMM that produced it. As
norms against the plain FP64 oracle: forward and gradients within 2e-2
relative L2, cosine >= 0.999; Adam within FP32 round-off of the oracle's
update applied to the GPU's own gradients."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

DIMS = [5, 256, 256, 256, 192]


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module")
def setup():
    import torch
    from paper_1310_7450_amd import mlp
    rng = np.random.default_rng(1)
    B = 100  # not a multiple of 16: ragged tiles
    x = rng.standard_normal((B, DIMS[0])).astype(np.float32)
    t = (0.3 * rng.standard_normal((B, DIMS[-1]))).astype(np.float32)
    p = mlp.init_params(DIMS, seed=3)
    net = mlp.Net(DIMS, max_batch=256)
    net.set_params(p)
    xd = torch.from_numpy(x).cuda()
    td = torch.from_numpy(t).cuda()
    return net, p, x, t, xd, td


def bf16(a):
    """FP32 -> BF16 -> FP64 with round to nearest, ties to even: keep the top
    16 bits of the FP32 pattern after adding half an ulp of the kept part
    (0x7fff plus the kept part's lowest bit)."""
    b = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    b = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16
    return b.astype(np.uint32).view(np.float32).astype(np.float64)


def test_bf16_rounding_helper():
    """The test's BF16 rounding: exact values stay, halfway cases go to the
    even neighbour, others to the nearest (BF16 keeps 8 significant bits)."""
    assert bf16(np.float32(1.0)) == 1.0
    assert bf16(np.float32(1.0 + 2.0 ** -8)) == 1.0                 # tie, to even
    assert bf16(np.float32(1.0 + 3 * 2.0 ** -8)) == 1.0 + 2.0 ** -6  # tie, to even (up)
    assert bf16(np.float32(1.0 + 2.0 ** -8 + 2.0 ** -20)) == 1.0 + 2.0 ** -7
    assert bf16(np.float32(-3.0)) == -3.0


@pytest.fixture(scope="module")
def setup_bias():
    """The network with random biases (zero biases would hide a bias added to
    the wrong column) and a ragged batch of 77 rows."""
    import torch
    from paper_1310_7450_amd import mlp
    rng = np.random.default_rng(11)
    B = 77
    x = rng.standard_normal((B, DIMS[0])).astype(np.float32)
    p = mlp.init_params(DIMS, seed=4).astype(np.float64)
    o = 0
    for l in range(len(DIMS) - 1):
        o += DIMS[l] * DIMS[l + 1]
        p[o:o + DIMS[l + 1]] = rng.uniform(-0.5, 0.5, DIMS[l + 1])
        o += DIMS[l + 1]
    p = p.astype(np.float32)
    net = mlp.Net(DIMS, max_batch=256)
    net.set_params(p)
    return net, p, x, torch.from_numpy(x).cuda()


# Element-wise tolerance against the oracle at BF16 operands: one BF16 unit
# roundoff (2^-8) of the absolute product sum sum_k |a_ik b_kj| of the GEMM
# that produced the entry. What separates the two is FP32 accumulation (at
# most K 2^-24 of that sum, 1.5e-5 at K = 256) and operands that round to the
# other BF16 neighbour on one side: an activation or a back-propagated dZ
# whose FP32 value differs from the oracle's by the accumulation error can
# cross a rounding midpoint, which changes that term by one BF16 ulp (2^-7 of
# itself). Back-propagated dZ come from sums with much cancellation, so such
# crossings are common there, and a weight gradient sums only the 77 rows of
# the batch. A wrong tile, row or bias gives errors of the size of the
# entries themselves.
TOL_ABS_SUM = 2.0 ** -8


def test_forward_elementwise(setup_bias):
    """Every output of the 5-256-256-256-192 network on a ragged batch of 77
    rows equals the oracle evaluated at BF16 operands within 2^-8 of the
    last layer's absolute product sums; against the FP64 oracle the outputs
    agree within 2e-2 relative L2."""
    import torch
    net, p, x, xd = setup_bias
    y = net.forward(xd)
    torch.cuda.synchronize()
    yg = y.cpu().numpy().astype(np.float64)
    p64, x64 = p.astype(np.float64), x.astype(np.float64)
    yb, cache = omlp.forward(p64, DIMS, x64, operand=bf16)
    W_last = omlp.unpack(p64, DIMS)[-1][0]
    absum = np.abs(bf16(cache[-1][0])) @ np.abs(bf16(W_last)).T
    ratio = np.abs(yg - yb) / (TOL_ABS_SUM * absum)
    y64 = omlp.forward(p64, DIMS, x64)[0]
    print(f"forward: max |err| / tol {ratio.max():.3e}; tol / |y| median "
          f"{np.median(TOL_ABS_SUM * absum / np.abs(yb)):.2e}; vs FP64 rel L2 {rel(yg, y64):.2e}", flush=True)
    assert ratio.max() <= 1.0
    assert rel(yg, y64) < 2e-2


def test_gradients_elementwise(setup_bias):
    """From the oracle's dL/dy (mean squared error against a seeded target),
    every weight gradient dW_l = dZ_l^T H_(l-1) and bias gradient sum_rows dZ_l
    of every layer, through the hidden layers' dZ = (dZ W) * SiLU'(z) path,
    equals the oracle's backward at BF16 operands within 2^-8 of the
    absolute product (or row) sums; against the FP64 oracle the gradients
    agree within 2e-2 relative L2 with cosine > 0.999."""
    import torch
    net, p, x, xd = setup_bias
    rng = np.random.default_rng(12)
    t = 0.3 * rng.standard_normal((x.shape[0], DIMS[-1]))
    p64, x64 = p.astype(np.float64), x.astype(np.float64)
    yb, cache = omlp.forward(p64, DIMS, x64, operand=bf16)
    _, dy = omlp.mse(yb, t)
    dy = dy.astype(np.float32).astype(np.float64)
    gb = omlp.backward(p64, DIMS, cache, dy, operand=bf16)
    net.forward(xd)
    net.backward(torch.from_numpy(dy.astype(np.float32)).cuda())
    g = net.get_grads().astype(np.float64)
    # absolute sums of every gradient entry, from the oracle's own dZ
    layers = omlp.unpack(p64, DIMS)
    dz = dy
    sums = [None] * len(layers)
    for l in range(len(layers) - 1, -1, -1):
        h, _ = cache[l]
        sums[l] = (np.abs(bf16(dz)).T @ np.abs(bf16(h)), np.abs(dz).sum(axis=0))
        if l > 0:
            z = cache[l - 1][1]
            s = 1.0 / (1.0 + np.exp(-z))
            dz = (bf16(dz) @ bf16(layers[l][0])) * (s * (1.0 + z * (1.0 - s)))
    absum = np.concatenate([np.concatenate([a.ravel(), c]) for a, c in sums])
    ratio = np.abs(g - gb) / (TOL_ABS_SUM * absum)
    o = 0
    for l in range(len(DIMS) - 1):
        nW, nb = DIMS[l] * DIMS[l + 1], DIMS[l + 1]
        print(f"layer {l}: dW max |err| / tol {ratio[o:o + nW].max():.3e}, "
              f"db {ratio[o + nW:o + nW + nb].max():.3e}", flush=True)
        o += nW + nb
    go = omlp.backward(p64, DIMS, omlp.forward(p64, DIMS, x64)[1], dy)
    cos = float(g @ go / np.linalg.norm(g) / np.linalg.norm(go))
    print(f"gradients vs FP64: rel L2 {rel(g, go):.2e}, cos {cos:.6f}", flush=True)
    assert ratio.max() <= 1.0
    assert cos > 0.999 and rel(g, go) < 2e-2


def test_forward_matches_oracle(setup):
    import torch
    net, p, x, t, xd, td = setup
    y = net.forward(xd)
    torch.cuda.synchronize()
    yo, _ = omlp.forward(p.astype(np.float64), DIMS, x)
    e = rel(y.cpu().numpy(), yo)
    print(f"forward rel L2 {e:.3e}", flush=True)
    assert e < 2e-2


def test_gradients_match_oracle(setup):
    import torch
    net, p, x, t, xd, td = setup
    y = net.forward(xd)
    dy = torch.empty_like(y)
    loss = net.mse(y, td, dy)
    net.backward(dy)
    g = net.get_grads()
    lo, go = omlp.loss_and_grad(p.astype(np.float64), DIMS, x, t)
    cos = float(g @ go / np.linalg.norm(g) / np.linalg.norm(go))
    e = rel(g, go)
    print(f"loss {loss:.6e} vs {lo:.6e}; grad rel L2 {e:.3e} cos {cos:.6f}", flush=True)
    assert abs(loss - lo) / lo < 2e-2
    assert cos > 0.999 and e < 2e-2


def test_adam_matches_oracle(setup):
    import torch
    from paper_1310_7450_amd import mlp
    net, p, x, t, xd, td = setup
    net2 = mlp.Net(DIMS, max_batch=256)
    net2.set_params(p)
    y = net2.forward(xd)
    dy = torch.empty_like(y)
    net2.mse(y, td, dy)
    net2.backward(dy)
    g = net2.get_grads().astype(np.float64)
    net2.adam_step(lr=1e-3)
    p1 = net2.get_params()
    po, m, v = omlp.adam(p.astype(np.float64), g, np.zeros_like(g), np.zeros_like(g), 1, lr=1e-3)
    assert np.abs(p1 - po).max() < 1e-6


def test_training_reduces_loss():
    """A smooth synthetic regression (outputs are fixed sinusoids of the
    inputs): 300 Adam steps on the GPU cut the loss by more than 10x."""
    import torch
    from paper_1310_7450_amd import mlp
    rng = np.random.default_rng(5)
    x = rng.uniform(-1, 1, (256, 5)).astype(np.float32)
    A = rng.standard_normal((5, 192))
    t = np.sin(x @ A).astype(np.float32)
    net = mlp.Net(DIMS, max_batch=256)
    net.set_params(mlp.init_params(DIMS, seed=0))
    xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
    dy = torch.empty_like(td)
    first = None
    for it in range(300):
        y = net.forward(xd)
        loss = net.mse(y, td, dy, want_loss=(it % 50 == 0 or it == 299))
        if first is None:
            first = loss
        net.backward(dy)
        net.adam_step(lr=2e-3)
    print(f"loss {first:.4e} -> {loss:.4e}", flush=True)
    assert loss < first / 10


def test_train_step_equals_separate_calls():
    """lbml_train_step (rows gathered on the device, one call) gives the same
    loss, gradients and updated parameters, bit for bit, as forward, mse,
    backward and adam_step on the same rows gathered by torch; two steps in a
    row, the second with a smaller batch."""
    import torch
    from paper_1310_7450_amd import mlp
    rng = np.random.default_rng(21)
    X = torch.from_numpy(rng.standard_normal((300, DIMS[0])).astype(np.float32)).cuda()
    Y = torch.from_numpy((0.3 * rng.standard_normal((300, DIMS[-1]))).astype(np.float32)).cuda()
    p0 = mlp.init_params(DIMS, seed=6)
    a, b = mlp.Net(DIMS, max_batch=128), mlp.Net(DIMS, max_batch=128)
    a.set_params(p0)
    b.set_params(p0)
    for batch in (100, 37):
        idx = torch.from_numpy(rng.choice(300, batch, replace=False).astype(np.int32)).cuda()
        la = a.train_step(X, Y, idx, lr=1e-3, want_loss=True)
        xb = X.index_select(0, idx.long()).contiguous()
        yb = Y.index_select(0, idx.long()).contiguous()
        y = b.forward(xb)
        dy = torch.empty_like(y)
        lb = b.mse(y, yb, dy, want_loss=True)
        b.backward(dy)
        b.adam_step(lr=1e-3)
        torch.cuda.synchronize()
        print(f"batch {batch}: loss {la:.6e} vs {lb:.6e}", flush=True)
        assert la == lb
        assert np.array_equal(a.get_grads(), b.get_grads())
        assert np.array_equal(a.get_params(), b.get_params())


# The fused passes (up to four layers of at most 256) and the GEMM per launch
# (deeper or wider networks): every depth, widths of one, of no multiple of a
# tile and of the limit, batches around the 16 rows of a workgroup.
@pytest.mark.parametrize("dims", [[3, 7], [5, 64, 48], [1, 100, 192, 96], [256, 256, 17, 256, 256], [5, 33, 1, 65],
                                  [4, 32, 32, 32, 32, 8], [5, 300, 20]])
@pytest.mark.parametrize("batch", [1, 16, 17, 95])
def test_network_shapes(dims, batch):
    """Forward within 2^-8 of the last layer's absolute product sums of the
    oracle at BF16 operands; gradients of the mean squared error within 2e-2
    (relative L2) of the oracle's at BF16 operands; one training step equal,
    bit for bit, to the separate calls, after a larger batch left its data in
    the workspace."""
    import torch
    from paper_1310_7450_amd import mlp
    rng = np.random.default_rng(sum(dims) + batch)
    p = mlp.init_params(dims, seed=3)
    p = (p + rng.uniform(-0.1, 0.1, p.size)).astype(np.float32)
    X = rng.standard_normal((120, dims[0])).astype(np.float32)
    T = (0.3 * rng.standard_normal((120, dims[-1]))).astype(np.float32)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    a, b = mlp.Net(dims, max_batch=120), mlp.Net(dims, max_batch=120)
    for net in (a, b):
        net.set_params(p)
        net.forward(Xd)  # the whole batch first
    x, t = Xd[:batch].contiguous(), Td[:batch].contiguous()
    y = a.forward(x)
    dy = torch.empty_like(y)
    a.mse(y, t, dy)
    a.backward(dy)
    p64 = p.astype(np.float64)
    yb, cache = omlp.forward(p64, dims, X[:batch].astype(np.float64), operand=bf16)
    absum = np.abs(bf16(cache[-1][0])) @ np.abs(bf16(omlp.unpack(p64, dims)[-1][0])).T
    assert np.all(np.abs(y.cpu().numpy() - yb) <= TOL_ABS_SUM * absum + 2.0 ** -20)
    _, dyo = omlp.mse(yb, T[:batch].astype(np.float64))
    g = omlp.backward(p64, dims, cache, dyo, operand=bf16)
    assert rel(a.get_grads().astype(np.float64), g) < 2e-2
    a.adam_step(lr=1e-3)
    idx = torch.arange(batch, dtype=torch.int32, device="cuda")
    b.train_step(Xd, Td, idx, lr=1e-3, want_loss=False)
    torch.cuda.synchronize()
    assert np.array_equal(a.get_grads(), b.get_grads())
    assert np.array_equal(a.get_params(), b.get_params())
    # a training step keeps its forward pass for another backward
    a.backward(dy)
    b.backward(dy)
    assert np.array_equal(a.get_grads(), b.get_grads())
    assert np.array_equal(a.forward(x).cpu().numpy(), b.forward(x).cpu().numpy())


# The rows a workgroup takes grow with the batch (4 up to 1024 rows, 8 up to
# 2048, then 16): both sides of each limit.
@pytest.mark.parametrize("batch", [1000, 1024, 1025, 2048, 2049])
def test_rows_per_workgroup(batch):
    """A row's prediction does not depend on the batch it is in (bit for bit);
    gradients within 2e-2 (relative L2) of the oracle's at BF16 operands; a
    training step equals the separate calls."""
    import torch
    from paper_1310_7450_amd import mlp
    dims = [5, 64, 256, 40]
    rng = np.random.default_rng(batch)
    p = mlp.init_params(dims, seed=3)
    X = rng.standard_normal((batch, dims[0])).astype(np.float32)
    T = (0.3 * rng.standard_normal((batch, dims[-1]))).astype(np.float32)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    a, b, c = mlp.Net(dims, max_batch=batch), mlp.Net(dims, max_batch=batch), mlp.Net(dims, max_batch=500)
    for net in (a, b, c):
        net.set_params(p)
    y = a.forward(Xd)
    parts = [c.forward(Xd[k:k + 500].contiguous()).cpu().numpy() for k in range(0, batch, 500)]
    assert np.array_equal(y.cpu().numpy(), np.concatenate(parts))
    dy = torch.empty_like(y)
    a.mse(y, Td, dy)
    a.backward(dy)
    p64 = p.astype(np.float64)
    yb, cache = omlp.forward(p64, dims, X.astype(np.float64), operand=bf16)
    _, dyo = omlp.mse(yb, T.astype(np.float64))
    assert rel(a.get_grads().astype(np.float64), omlp.backward(p64, dims, cache, dyo, operand=bf16)) < 2e-2
    a.adam_step(lr=1e-3)
    b.train_step(Xd, Td, torch.arange(batch, dtype=torch.int32, device="cuda"), lr=1e-3, want_loss=False)
    torch.cuda.synchronize()
    assert np.array_equal(a.get_grads(), b.get_grads()) and np.array_equal(a.get_params(), b.get_params())


@pytest.mark.parametrize("dims", [[4, 48, 48, 3], [4, 17, 33, 20, 3], [4, 100, 250, 2], [4, 20, 3]])
def test_infinities_stay_in_their_rows(dims):
    """An infinite activation or gradient, with positive weights everywhere,
    stays an infinity of its sign: no padded column (widths below the kernels'
    padding) turns it into NaN, and rows of finite ones keep their values."""
    import torch
    from paper_1310_7450_amd import mlp
    nl, B = len(dims) - 1, 37
    rng = np.random.default_rng(5)
    p = np.concatenate([np.concatenate([rng.uniform(0.05, 0.1, dims[l] * dims[l + 1]), np.zeros(dims[l + 1])])
                        for l in range(nl)]).astype(np.float32)
    x = rng.uniform(0.5, 1.0, (B, dims[0])).astype(np.float32)
    net = mlp.Net(dims, max_batch=64)
    net.set_params(p)
    finite = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.isfinite(finite).all() and (finite > 0).all()
    # forward: z of row 3 overflows in the first layer
    xi = x.copy()
    xi[3] = 3e38
    p2 = p.copy()
    p2[:dims[0] * dims[1]] = 1.0
    net.set_params(p2)
    want = net.forward(torch.from_numpy(x).cuda()).cpu().numpy()
    got = net.forward(torch.from_numpy(xi).cuda()).cpu().numpy()
    assert np.isposinf(got[3]).all()
    assert np.array_equal(np.delete(got, 3, 0), np.delete(want, 3, 0))
    # backward: an infinite dy in every column of a row, z > 0 throughout
    net.set_params(p)
    net.forward(torch.from_numpy(x).cuda())
    dy = np.full((B, dims[-1]), 1e-3, dtype=np.float32)
    dy[5] = np.inf
    net.backward(torch.from_numpy(dy).cuda())
    assert np.isposinf(net.get_grads()).all()
    dy[5] = 1e-3
    net.backward(torch.from_numpy(dy).cuda())
    assert np.isfinite(net.get_grads()).all()
    net.close()


@pytest.mark.parametrize("dims", [[5, 64, 96], [96, 64, 5], [7, 32, 7]])
@pytest.mark.parametrize("shift", [0, 3])
def test_forward_over_its_input(dims, shift):
    """The output may lie over the input (shift: rows between their starts),
    with more rows than the GPU takes at once."""
    import torch
    from paper_1310_7450_amd import mlp
    B = 20000
    net = mlp.Net(dims, max_batch=B)
    net.set_params(mlp.init_params(dims, seed=2))
    x = torch.randn(B, dims[0], device="cuda")
    want = net.forward(x).clone()
    buf = torch.zeros((B + shift) * max(dims[0], dims[-1]), device="cuda")
    buf[:B * dims[0]] = x.flatten()
    at = shift * dims[-1]
    got = net.forward(buf[:B * dims[0]].view(B, dims[0]), buf[at:at + B * dims[-1]].view(B, dims[-1]))
    assert torch.equal(got, want)
    net.close()


# The least of 32, 64, 128 and 256 columns that holds every layer pads them:
# both sides of each limit, every depth, every number of rows per workgroup.
@pytest.mark.parametrize("batch", [30, 1025, 2049])
@pytest.mark.parametrize("dims", [[5, 32, 7], [32, 8, 30, 1], [5, 33, 7], [5, 17, 9, 64, 31], [5, 65, 7],
                                  [60, 128, 2, 90], [5, 129, 7]])
def test_padded_widths(dims, batch):
    """The same network with its hidden layers widened to 250 by units of
    zero weights (padded to 256) gives the same outputs and gradients, bit for
    bit."""
    import torch
    from paper_1310_7450_amd import mlp
    wide = [dims[0]] + [250] * (len(dims) - 2) + [dims[-1]]
    rng = np.random.default_rng(sum(dims))
    at = 0
    own = []  # positions of the narrow network's parameters in the wide one's
    for l in range(len(dims) - 1):
        ids = at + np.arange(wide[l + 1] * wide[l]).reshape(wide[l + 1], wide[l])
        own.append(ids[:dims[l + 1], :dims[l]].ravel())
        at += ids.size
        own.append(at + np.arange(dims[l + 1]))
        at += wide[l + 1]
    own = np.concatenate(own)
    p = rng.uniform(-0.5, 0.5, own.size).astype(np.float32)
    pw = np.zeros(at, dtype=np.float32)
    pw[own] = p
    x = torch.from_numpy(rng.standard_normal((batch, dims[0])).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.standard_normal((batch, dims[-1])).astype(np.float32)).cuda()
    idx = torch.arange(batch, dtype=torch.int32, device="cuda")
    res = []
    for d, q, pick in ((dims, p, slice(None)), (wide, pw, own)):
        net = mlp.Net(d, max_batch=batch)
        net.set_params(q)
        y = net.forward(x).cpu().numpy()
        loss = net.train_step(x, t, idx, lr=1e-3, want_loss=True)
        res.append((y, net.get_grads()[pick], loss))
        net.close()
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1]) and res[0][2] == res[1][2]
    assert np.abs(res[0][1]).max() > 0
