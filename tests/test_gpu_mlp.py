"""Surrogate network kernels against the FP64 oracle network: forward (bf16
matrix cores, precise split mode), gradients, and a training smoke test."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2109_14403_amd import hom

pytestmark = pytest.mark.gpu

N_IN, N_OUT = 32, 10


def bf16_round(a):
    """Round FP32 values to the nearest bf16 (ties to even)."""
    u = np.ascontiguousarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


@pytest.fixture(scope="module")
def net_and_data():
    rng = np.random.default_rng(3)
    net = hom.MLP(N_IN, N_OUT, seed=11)
    layers = net.layers()
    # perturb the biases so the test sees nonzero bias paths
    flat = net.get_params().copy()
    o = 0
    for (W, b) in layers:
        o += W.size
        flat[o:o + b.size] = rng.normal(scale=0.1, size=b.size)
        o += b.size
    net.set_params(flat)
    xm, xs = rng.normal(size=N_IN), rng.uniform(0.5, 2.0, size=N_IN)
    ym, ys = rng.normal(size=N_OUT), rng.uniform(0.5, 2.0, size=N_OUT)
    lw = rng.uniform(0.5, 2.0, size=N_OUT)
    net.set_scaling(xm, xs, ym, ys, lw)
    x = (xm + xs * rng.normal(size=(333, N_IN))).astype(np.float32)   # 333 rows: a ragged last tile
    y = (ym + ys * rng.normal(size=(333, N_OUT))).astype(np.float32)
    return net, x, y, (xm, xs, ym, ys, lw)


def oracle_forward(params, x, scal):
    xm, xs, ym, ys, _ = scal
    xh = (x.astype(np.float64) - xm) / xs
    yh, _ = omlp.forward(params, xh)
    return yh * ys + ym


def f64(layers, rounding=None):
    return [((rounding(W) if rounding else W).astype(np.float64), b.astype(np.float64)) for W, b in layers]


def test_forward_precise_matches_oracle(net_and_data):
    net, x, _, scal = net_and_data
    ref = oracle_forward(f64(net.layers()), x, scal)
    out = net.forward(x, precise=True)
    err = np.abs(out - ref).max() / np.abs(ref).max()
    print(f"precise forward max rel err {err:.2e}", flush=True)
    assert err < 2e-5


def test_forward_bf16_matches_rounded_weight_oracle(net_and_data):
    net, x, _, scal = net_and_data
    ref = oracle_forward(f64(net.layers(), bf16_round), x, scal)
    out = net.forward(x, precise=False)
    err = np.abs(out - ref).max() / np.abs(ref).max()
    print(f"bf16 forward max rel err {err:.2e}", flush=True)
    assert err < 1e-4


@pytest.mark.parametrize("precise", [False, True])
def test_forward_rows_are_independent(net_and_data, precise):
    """Each row's output depends on that row alone: the same rows give the
    same bits whatever the batch length and wherever the 64-row tiles fall
    (a full tile, a ragged tail, a single row, an offset start)."""
    net, x, _, _ = net_and_data
    full = net.forward(x, precise=precise)
    for lo, hi in [(0, 64), (0, 70), (5, 6), (17, 333), (300, 333)]:
        part = net.forward(np.ascontiguousarray(x[lo:hi]), precise=precise)
        np.testing.assert_array_equal(part, full[lo:hi], err_msg=f"rows {lo}:{hi}")


def test_gated_skip_matches_numpy(net_and_data):
    net, x, _, scal = net_and_data
    xm, xs, ym, ys, _ = scal
    rng = np.random.default_rng(8)
    gates = (7, 6, 26)
    G = rng.normal(scale=0.1, size=(N_OUT, 10, N_IN))
    c = rng.normal(size=N_OUT)
    net.set_skip(gates, G, c)
    try:
        xh = (x.astype(np.float64) - xm) / xs
        s = [np.ones(len(xh))]
        for i in gates:
            s += [xh[:, i], xh[:, i] ** 2, xh[:, i] ** 3]
        s = np.stack(s, axis=1)
        skip = c + np.einsum("rg,jgk,rk->rj", s, G, xh)
        ref = oracle_forward(f64(net.layers()), x, scal) + skip
        out = net.forward(x, precise=True)
        err = np.abs(out - ref).max() / np.abs(ref).max()
        print(f"forward with skip max rel err {err:.2e}", flush=True)
        assert err < 2e-5
    finally:
        net.set_skip(gates, np.zeros_like(G), np.zeros_like(c))


def test_gradients_match_oracle(net_and_data):
    net, x, y, scal = net_and_data
    xm, xs, ym, ys, lw = scal
    L, g = net.loss_grad(x, y, precise=True)
    xh = (x.astype(np.float64) - xm) / xs
    th = (y.astype(np.float64) - ym) / ys
    grads, Lref = omlp.gradients(f64(net.layers()), xh, th, lw)
    assert L == pytest.approx(Lref, rel=1e-5)
    gl = net.layers(g)
    for i, ((gW, gb), (rW, rb)) in enumerate(zip(gl, grads)):
        eW = np.linalg.norm(gW - rW) / np.linalg.norm(rW)
        eb = np.linalg.norm(gb - rb) / np.linalg.norm(rb)
        print(f"layer {i}: dW rel err {eW:.2e}, db rel err {eb:.2e}", flush=True)
        # precise mode carries activations and weights as two bf16 parts
        # (about 16 significant bits), FP32 accumulation
        assert eW < 5e-5 and eb < 5e-5


def test_training_reduces_loss():
    rng = np.random.default_rng(0)
    x = rng.uniform(-1, 1, size=(8192, 8)).astype(np.float32)
    y = np.stack([np.sin(2 * x[:, 0]) + x[:, 1] ** 2, x[:, 2] * x[:, 3], np.cos(x[:, 4] + x[:, 5])], axis=1)
    y = y.astype(np.float32)
    net = hom.MLP(8, 3, seed=1)
    net.set_scaling(x.mean(0), x.std(0), y.mean(0), y.std(0))
    losses = net.train(x, y, epochs=40, batch=256, lr=2e-3, seed=2)
    print(f"loss {losses[0]:.3e} -> {losses[-1]:.3e}", flush=True)
    assert losses[-1] < 1e-2 * losses[0]
    pred = net.forward(x[:512])
    rel = np.abs(pred - y[:512]).max() / np.abs(y).max()
    assert rel < 0.1


def test_row_weights():
    """Row weights enter the loss as w_r (y - t)^2 after scaling to mean 1:
    equal weights reproduce unweighted training bit for bit; weights that
    switch half of the rows off leave those rows' targets unfitted; and the
    weighted skip fit is weighted least squares (equal weights change nothing)."""
    rng = np.random.default_rng(3)
    x = rng.uniform(-1, 1, size=(4096, 6)).astype(np.float32)
    y = np.stack([np.sin(2 * x[:, 0]) + x[:, 1], x[:, 2] * x[:, 3]], axis=1).astype(np.float32)

    def trained(rw, flip=False):
        net = hom.MLP(6, 2, seed=4)
        t = y.copy()
        if flip:
            t[1::2] = -t[1::2]          # contradictory targets on the odd rows
        net.set_scaling(x.mean(0), x.std(0), y.mean(0), y.std(0))
        net.train(x, t, epochs=8, batch=256, lr=2e-3, seed=5, row_weight=rw)
        return net

    a = trained(None).get_params()
    b = trained(np.full(len(x), 2.0, dtype=np.float32)).get_params()
    assert np.array_equal(a, b)
    rw = np.zeros(len(x), dtype=np.float32)
    rw[0::2] = 1.0
    net = trained(rw, flip=True)       # only the even rows (true targets) count
    pred = net.forward(x)
    even = np.abs(pred[0::2] - y[0::2]).mean()
    odd_flipped = np.abs(pred[1::2] + y[1::2]).mean()
    assert even < 0.5 * odd_flipped
    gates = (0, 1, 2)
    s1, s2 = hom.MLP(6, 2, seed=0), hom.MLP(6, 2, seed=0)
    s1.fit_skip(x, y, gates)
    s2.fit_skip(x, y, gates, row_weight=np.full(len(x), 3.0, dtype=np.float32))
    for m in (s1, s2):
        m.set_params(np.zeros(m.param_count, dtype=np.float32))
    assert np.allclose(s1.forward(x[:256]), s2.forward(x[:256]), rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("rows", [1, 4, 17, 63, 65, 1023, 1025, 2500])
def test_gradients_at_batch_edges(rows):
    """Batches around the backward pass's 64-row tiles and its splits of the
    batch. Bound of the fixed batch above: precise mode carries about 16
    significant bits."""
    rng = np.random.default_rng(rows)
    net = hom.MLP(N_IN, N_OUT, seed=5)
    x = rng.normal(size=(rows, N_IN)).astype(np.float32)
    y = rng.normal(size=(rows, N_OUT)).astype(np.float32)
    lw = rng.uniform(0.5, 2.0, size=N_OUT)
    net.set_scaling(np.zeros(N_IN), np.ones(N_IN), np.zeros(N_OUT), np.ones(N_OUT), lw)
    L, g = net.loss_grad(x, y, precise=True)
    grads, Lref = omlp.gradients(f64(net.layers()), x.astype(np.float64), y.astype(np.float64), lw)
    assert L == pytest.approx(Lref, rel=1e-5)
    for i, ((gW, gb), (rW, rb)) in enumerate(zip(net.layers(g), grads)):
        assert np.linalg.norm(gW - rW) < 5e-5 * np.linalg.norm(rW), i
        assert np.linalg.norm(gb - rb) < 5e-5 * np.linalg.norm(rb), i


@pytest.mark.parametrize("precise", [False, True])
def test_forward_rows_alike_on_both_sides_of_the_tile_rule(net_and_data, precise):
    """Launches below 64 * 256 rows take 16 rows a work-group, larger ones 64:
    the same bits for a row in either."""
    net, _, _, (xm, xs, *_rest) = net_and_data
    n = 64 * 256
    x = (xm + xs * np.random.default_rng(9).normal(size=(n + 5, N_IN))).astype(np.float32)
    full = net.forward(x, precise=precise)
    np.testing.assert_array_equal(net.forward(x[:n], precise=precise), full[:n])
    np.testing.assert_array_equal(net.forward(x[:n - 1], precise=precise), full[:n - 1])
    np.testing.assert_array_equal(net.forward(x[n - 30:], precise=precise), full[n - 30:])


@pytest.mark.parametrize("rows,n_out", [(256, 10), (777, 3), (1000, 16)])
def test_targets_normalized_on_the_device_and_on_the_host_are_the_same(rows, n_out):
    """A network with a skip normalizes its targets on the host, one without on
    the device: with a skip of zeros the same training, bit for bit."""
    rng = np.random.default_rng(rows)
    x = rng.normal(size=(rows, 6)).astype(np.float32)
    y = (rng.normal(size=(rows, n_out)) * 10.0 ** rng.integers(-3, 4, n_out)).astype(np.float32)
    nets = [hom.MLP(6, n_out, seed=4) for _ in range(2)]
    for net in nets:
        net.set_scaling(x.mean(0), x.std(0), y.mean(0), y.std(0))
    nets[1].set_skip((0, 1, 2), np.zeros((n_out, 10, 6)), np.zeros(n_out))
    losses = [net.train(x, y, epochs=2, batch=128, lr=2e-3, seed=5) for net in nets]
    np.testing.assert_array_equal(losses[0], losses[1])
    np.testing.assert_array_equal(nets[0].get_params(), nets[1].get_params())


def test_initial_network_of_a_seed():
    """The initial weights are the draws of std::normal_distribution on
    std::mt19937_64(seed), layer by layer (first two and last weight of each
    layer, from a host program that calls the two)."""
    draws = [(0.259052932, -0.316714764, 0.303462267), (-0.100153431, -0.183836535, 0.0187645033),
             (0.0159088224, 0.00444698241, -0.196138665), (0.0302440617, 0.0436188132, 0.0804008171),
             (0.0257088933, -0.0477711968, -0.0274669509)]
    for (w, b), d in zip(hom.MLP(7, 3, seed=11).layers(), draws):
        np.testing.assert_array_equal(np.concatenate([w.ravel()[:2], w.ravel()[-1:]]), np.float32(d))
        assert not b.any()


@pytest.mark.parametrize("rows", [16383, 16384, 20001])
def test_gradients_of_large_batches(rows):
    """Both sides of the row rule of the forward pass that keeps activations (16
    and 64 rows a work-group), and the batch in 64 splits of more than 256
    rows, the last one shorter. Bounds of the smaller batches above."""
    test_gradients_at_batch_edges(rows)


def test_targets_of_more_values_than_a_launch_has_threads():
    """2^28 rows and a few have more than 2^32 padded targets: training takes them.
    Every row is the same and the steps are too small to change a weight: an epoch
    has the loss of one batch."""
    rows, batch = 2**28 + 5, 2**20
    x = np.full((rows, 1), 0.5, np.float32)
    net, few = hom.MLP(1, 1, seed=1), hom.MLP(1, 1, seed=1)
    (loss,) = net.train(x, x, epochs=1, batch=batch, lr=1e-30, seed=0)
    (first,) = few.train(x[:batch], x[:batch], epochs=1, batch=batch, lr=1e-30, seed=0)
    assert loss == pytest.approx(first, rel=1e-6)


@pytest.mark.parametrize("precise,groups", [(False, 768), (True, 640)])
def test_rows_alike_where_the_tiles_change(precise, groups):
    """Up to `groups` work-groups of 16 rows (over all networks) a forward pass
    takes those, beyond 64 rows each: the same bits for a row in either."""
    import torch
    n = 16 * groups
    nets = [hom.MLP(N_IN, N_OUT, seed=s) for s in (1, 2)]
    x = np.random.default_rng(n).normal(size=(n + 1, N_IN)).astype(np.float32)
    full = nets[0].forward(x, precise=precise)
    np.testing.assert_array_equal(nets[0].forward(x[:n], precise=precise), full[:n])
    np.testing.assert_array_equal(nets[0].forward(x[:n - 1], precise=precise), full[:n - 1])
    if precise:
        return  # an ensemble is not
    xd = torch.as_tensor(x[:n // 2 + 1], device="cuda")
    many = hom.mlp_ensemble_infer(nets, xd, 0.1, 1.0)
    few = hom.mlp_ensemble_infer(nets, xd[:-1].contiguous(), 0.1, 1.0)
    for a, b in zip(many, few):
        np.testing.assert_array_equal(a[:-1].cpu().numpy(), b.cpu().numpy())


def test_gradients_where_the_tiles_change():
    """A batch on 64-row tiles of the forward pass that keeps activations against
    its two halves on 16-row ones. The weighted mean of the halves' gradients is
    the batch's; FP32 sums over splits of 256 rows round by 256 eps = 3e-5."""
    rng = np.random.default_rng(12)
    n, h = 16 * 768 + 3, 5000
    net = hom.MLP(N_IN, N_OUT, seed=5)
    net.set_scaling(np.zeros(N_IN), np.ones(N_IN), np.zeros(N_OUT), np.ones(N_OUT), np.ones(N_OUT))
    x = rng.normal(size=(n, N_IN)).astype(np.float32)
    y = rng.normal(size=(n, N_OUT)).astype(np.float32)
    L, g = net.loss_grad(x, y, precise=False)
    (L1, g1), (L2, g2) = net.loss_grad(x[:h], y[:h], precise=False), net.loss_grad(x[h:], y[h:], precise=False)
    assert L == pytest.approx((h * L1 + (n - h) * L2) / n, rel=1e-6)
    for (gW, gb), (aW, ab), (bW, bb) in zip(net.layers(g), net.layers(g1), net.layers(g2)):
        for t, a, b in ((gW, aW, bW), (gb, ab, bb)):
            want = (h * a.astype(np.float64) + (n - h) * b) / n
            assert np.linalg.norm(t - want) < 5e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("rows", [10240, 10241])
def test_precise_gradients_where_the_tiles_change(rows):
    """Bounds of the smaller batches above."""
    test_gradients_at_batch_edges(rows)
