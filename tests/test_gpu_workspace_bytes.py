"""The bytes a context reports are those of its plan: a workspace of that length gives the same plan and bits."""
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


# fewer H-kernel tiles than a generation (short runs in the table), more (P = 260: 1530), and Alg. 4-5
@pytest.mark.parametrize("o,v,nL,P,Q,kw", [(6, 30, 150, 70, 100, {}), (6, 30, 150, 70, 100, {"precision": 1}),
                                           (6, 30, 300, 64, 130, {}), (10, 30, 100, 260, 280, {"flags": 16}),
                                           (6, 30, 150, 70, 100, {"flags": 8})])
def test_reported_bytes_give_the_same_plan(thc, o, v, nL, P, Q, kw):
    import torch
    print(f"[gpu-workspace-bytes] o {o} v {v} nL {nL} P {P} Q {Q} {kw}", flush=True)
    rng = np.random.default_rng(P)
    n = o + v
    L = rng.standard_normal((nL, n, n)) * (0.1 / n)
    L = L + L.transpose(0, 2, 1)
    eps = np.concatenate([-np.sort(rng.uniform(0.5, 3.0, o))[::-1], np.sort(rng.uniform(0.3, 4.0, v))])
    x = [rng.standard_normal((k, r)) for r in (P, Q) for k in (o, v)]
    t = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda").contiguous()
    args = [t(a) for a in (L, eps, *x)]

    def one(bytes_):
        ws = torch.empty(bytes_, dtype=torch.uint8, device="cuda")
        ctx = thc.THC(o, v, nL, P, Q, workspace=ws, **kw)
        Z = ctx.build_factors(*args)
        out = [Z, *[r.clone() for r in ctx.residual(Z)]], ctx.plan(), ctx.memory_bytes()
        ctx.close()
        return out

    big = 2 << 30
    first, plan, need = one(big)
    assert need == plan["device_bytes"] == thc.plan_query(o, v, nL, P, Q, big, **kw)["device_bytes"]
    again, plan2, _ = one(need)
    assert plan2 == plan
    assert all(torch.equal(a, b) for a, b in zip(first, again))
