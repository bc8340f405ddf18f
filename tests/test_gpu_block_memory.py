"""Long blocks of the fused pass lie over the end of the Alg. 6 region (its H block and behind, or all of
it): whatever a pass, or the MP2 density that borrows its buffers, leaves there reaches no later result."""
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


def _inputs(o, v, nL, P, Q, seed):
    import torch
    rng = np.random.default_rng(seed)
    n = o + v
    L = rng.standard_normal((nL, n, n)) * (0.1 / n)
    L = L + L.transpose(0, 2, 1)
    eps = np.concatenate([-np.sort(rng.uniform(0.5, 3.0, o))[::-1], np.sort(rng.uniform(0.3, 4.0, v))])
    x = [rng.standard_normal((k, r)) for r in (P, Q) for k in (o, v)]
    t = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda").contiguous()
    return [t(a) for a in (L, eps, *x)], t(0.01 * rng.standard_normal((o, v)))


# a rank padded to the H-kernel's blocks and tiles (70, 129) and not (64); blocks that cover the end of the
# region (130 of 150 vectors) and, with many vectors of a small rank, all of it; Alg. 4-5 (flags 8)
@pytest.mark.parametrize("o,v,nL,P,Q,flags", [(6, 30, 150, 70, 100, 0), (6, 30, 300, 64, 130, 0), (8, 40, 200, 129, 140, 0),
                                              (4, 8, 2500, 16, 20, 0), (4, 8, 2500, 17, 20, 4), (6, 30, 150, 70, 100, 8)])
def test_nothing_left_by_a_long_block_is_used(thc, o, v, nL, P, Q, flags):
    import torch
    print(f"[gpu-block-memory] o {o} v {v} nL {nL} P {P} Q {Q} flags {flags}", flush=True)
    args, t1 = _inputs(o, v, nL, P, Q, P)
    ctx = thc.THC(o, v, nL, P, Q, flags=flags)
    Z = ctx.build_factors(*args)
    assert ctx.plan()["a_block"] > 64
    first = [x.clone() for x in ctx.residual(Z, t1)]
    assert all(torch.isfinite(x).all() for x in first)
    ctx.mp2_density(torch.full_like(Z, float("nan")))  # the borrowed buffers are NaN throughout
    again = ctx.residual(Z, t1)
    assert all(torch.equal(a, b) for a, b in zip(first, again))
    ctx.close()
    need = thc.plan_query(o, v, nL, P, Q, 270e9, flags=flags)["device_bytes"]
    ws = torch.full(((need + 7) // 8,), float("nan"), dtype=torch.float64, device="cuda")
    ctx = thc.THC(o, v, nL, P, Q, flags=flags, workspace=ws)
    assert torch.equal(ctx.build_factors(*args), Z)
    assert ctx.plan()["a_block"] > 64
    assert all(torch.equal(a, b) for a, b in zip(first, ctx.residual(Z, t1)))
    ctx.close()
