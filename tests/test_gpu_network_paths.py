"""The guess network's three-launch training step and its inference kernel at the edges of their row
tiles, row ranges and padded input and output widths, against the FP64 reference network."""
import numpy as np
import pytest

from oracle import guess

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def thc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_11473_amd import thc as mod
    mod.load()
    return mod


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda")


def _h(t):
    return t.detach().cpu().numpy().astype(np.float64)


def _net(thc, n_in, n_out, rows, seed):
    rng = np.random.default_rng(seed)
    net = thc.MLP(n_in, 256, n_out, seed=seed)
    norm = (rng.standard_normal(n_in), rng.uniform(0.5, 2.0, n_in), rng.standard_normal(n_out),
            rng.uniform(0.5, 2.0, n_out))
    norm = tuple(np.asarray(x, dtype=np.float32).astype(np.float64) for x in norm)
    net.set_norm(*norm)
    net.set_params(net.get_params() + 0.05 * _t(rng.standard_normal(net.n_params)))  # non-zero biases
    X = rng.standard_normal((rows, n_in)).astype(np.float32)
    T = rng.standard_normal((rows, n_out)).astype(np.float32)
    return net, norm, X, T


# one row, around one tile of 16 and one range of 256, more tiles than workgroups (16 x 512) and more
# ranges than 32 (256 x 32) by one row; input and output widths at both ends of the padded class and
# around the two-output instantiation
@pytest.mark.parametrize("n_in,n_out", [(10, 2), (1, 1), (16, 16), (7, 3)])
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 256, 257, 8193])
def test_loss_gradient_and_step(thc, n_in, n_out, rows):
    print(f"[gpu-network] train {n_in} -> {n_out}, {rows} rows", flush=True)
    net, norm, X, T = _net(thc, n_in, n_out, rows, 100 * n_in + rows)
    dims = (n_in, 256, n_out)
    p = _h(net.get_params())
    loss_ref, g_ref = guess.loss_and_grad(p, dims, X.astype(np.float64), T.astype(np.float64), norm)
    loss, g = net.loss_grad(_t(X), _t(T))
    # FP32 sums of 256 terms twice over in the forward pass and twice in the backward pass, each with a
    # relative error of at most 256 2^-24 = 1.5e-5 of the sum of magnitudes: 6e-5 of the largest entry
    # per layer, and a block's entries are compared with the block's largest
    assert abs(loss - loss_ref) < 6e-5 * max(loss_ref, 1e-30)
    for a, b in zip(guess.unpack(_h(g), *dims), guess.unpack(g_ref, *dims)):
        assert np.abs(a - b).max() <= 6e-5 * np.abs(b).max(), (a.shape, np.abs(a - b).max(), np.abs(b).max())
    # one step from zero moments with the gradient just checked: the Adam rule in FP64
    loss2 = net.train_step(_t(X), _t(T), 1e-3)
    assert loss2 == loss
    p1, _, _ = guess.adam(p, _h(g), np.zeros_like(p), np.zeros_like(p), 1, 1e-3)
    # the step is at most lr; FP32 moments and quotients to 2^-20 of it, the parameter to its rounding
    assert np.abs(_h(net.get_params()) - p1).max() <= 1e-3 * 2.0 ** -18 + np.abs(p).max() * 2.0 ** -23


@pytest.mark.parametrize("n_in,n_out", [(10, 2), (1, 16), (16, 1)])
@pytest.mark.parametrize("rows", [1, 16, 17, 63, 8192, 8193, 8260])
def test_inference_rows_do_not_depend_on_the_launch(thc, n_in, n_out, rows):
    """Every row's result is the same bits whichever rows share its launch (the 16- and the 64-row
    workgroups), and the network's to BF16 accuracy."""
    import torch
    print(f"[gpu-network] infer {n_in} -> {n_out}, {rows} rows", flush=True)
    net, norm, X, _ = _net(thc, n_in, n_out, rows, 31 + rows)
    Xd = _t(X)
    y = net.infer(Xd)
    cut = 5 if rows > 5 else rows
    parts = [net.infer(Xd[:cut].contiguous())]
    if rows > cut:
        parts.append(net.infer(Xd[cut:cut + 4096].contiguous()))
    ref = torch.cat(parts)
    assert torch.equal(y[:ref.shape[0]], ref)
    full, yn, _ = guess.forward(_h(net.get_params()), (n_in, 256, n_out), X.astype(np.float64), norm)
    # BF16 operands (2^-9 each) in three layers of up to 256 terms of either sign: a few 2^-9 of the
    # normalized outputs' scale
    err = np.abs((_h(y) - full) / norm[3]).max()
    assert err < 16 * 2.0 ** -9 * max(1.0, np.abs(yn).max()), err
