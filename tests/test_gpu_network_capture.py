"""A training pass of the guess network under stream capture: a pass of the same rows before it has reserved
everything, whichever pass it was."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def thc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_11473_amd import thc as mod
    mod.load()
    return mod


@pytest.mark.parametrize("rows", [1, 300, 1025, 9000])
def test_gradient_is_capturable_after_a_forward_pass(thc, rows):
    import torch
    print(f"[gpu-network-capture] {rows} rows", flush=True)
    rng = np.random.default_rng(rows)
    t = lambda a: torch.from_numpy(a.astype(np.float32)).cuda()
    X, T = t(rng.standard_normal((rows, 10))), t(rng.standard_normal((rows, 2)))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        net = thc.MLP(seed=7)
        net.forward(X)  # reserves for these rows
        grad = torch.empty(net.n_params, dtype=torch.float32, device="cuda")
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin()
        rc = net.lib.thc_mlp_loss_grad(net.net, X.data_ptr(), T.data_ptr(), rows, None, grad.data_ptr())
        graph.capture_end()
        assert rc == thc.THC_OK
        _, want = net.loss_grad(X, T)
        p = net.get_params()
        for k in range(3):
            grad.fill_(float("nan"))
            graph.replay()
            s.synchronize()
            assert torch.equal(grad, want)
            net.set_params(p * (1.0 + 0.01 * (k + 1)))  # eager work between the replays
            _, want = net.loss_grad(X, T)
        graph.replay()
        s.synchronize()
        assert torch.equal(grad, want)
        net.close()
