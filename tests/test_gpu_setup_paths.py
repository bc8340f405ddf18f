"""The set-up's device linear algebra (Cholesky blocks of 64, Householder reduction column by column,
compact WY blocks of 64 reflectors, streamed plane rotations) at the edges of its blocks, against the
generalized eigenproblem E w = e S w on the host."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def thc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_11473_amd import thc as mod
    mod.load()
    return mod


def _inputs(o, v, nL, P, Q, seed):
    rng = np.random.default_rng(seed)
    n = o + v
    L = rng.standard_normal((nL, n, n)) * (0.1 / n)
    L = L + L.transpose(0, 2, 1)
    eps = np.concatenate([-np.sort(rng.uniform(0.5, 3.0, o))[::-1], np.sort(rng.uniform(0.3, 4.0, v))])
    Xo, Xv = rng.standard_normal((o, P)), rng.standard_normal((v, P))
    xo, xv = rng.standard_normal((o, Q)), rng.standard_normal((v, Q))
    return L, eps, Xo, Xv, xo, xv


# P below and at the device eigensolver's smallest size; one more and one less than whole blocks of
# rows, reflectors (P - 2 of them) and rotation tiles; Q around whole Cholesky blocks
@pytest.mark.parametrize("P,Q", [(2, 3), (63, 65), (64, 64), (65, 63), (66, 128), (67, 129), (127, 70), (130, 191),
                                 (131, 192), (194, 193), (300, 320)])
def test_working_basis(thc, P, Q):
    import torch
    from scipy.linalg import eigh
    print(f"[gpu-setup] P {P} Q {Q}", flush=True)
    o, v, nL = 12, 60, 40
    L, eps, Xo, Xv, xo, xv = _inputs(o, v, nL, P, Q, P)
    S = (Xo.T @ Xo) * (Xv.T @ Xv)
    E = (Xo.T @ Xo) * (Xv.T @ (eps[o:, None] * Xv)) - (Xo.T @ (eps[:o, None] * Xo)) * (Xv.T @ Xv)
    w, V = eigh(E, S)
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda").contiguous()
    ctx = thc.THC(o, v, nL, P, Q)
    Z = ctx.build_factors(t(L), t(eps), t(Xo), t(Xv), t(xo), t(xv)).cpu().numpy().reshape(P, P)
    Th = ctx.working()
    Th = (Th[0] if isinstance(Th, tuple) else Th).reshape(P, P)
    # the fit of 0 = e_P + e_Q + delta_P + delta_Q reads the context's eigenvalues: it solves
    # (A + r) delta = -A e with A = P I + 1 1^T and the ridge r = 1e-10 (P + 1)
    _, delta = ctx.guess_targets(Th, Th + 1.0, torch.zeros_like(Th))
    delta = delta.cpu().numpy().ravel()
    e = -(delta + 1e-10 * (P + 1) * np.linalg.solve(P * np.eye(P) + 1.0, delta))
    ctx.close()
    cond = np.linalg.cond(S)
    # eigenvalues: backward error of the factorization and the reduction, n eps each, magnified by cond(S)
    assert np.abs(e - w).max() <= 64 * P * EPS * cond * np.abs(w).max()
    # W W^T = S^-1: the guess in the pair basis is S^-1 M S^-1 whatever the eigenvectors' signs
    B = np.einsum("iX,aX->iaX", Xo, Xv).reshape(o * v, P)
    Lov = L[:, :o, o:].reshape(nL, o * v)
    de = eps[o:][None, :] - eps[:o][:, None]
    t2 = -(Lov.T @ Lov) / (de.reshape(-1, 1) + de.reshape(1, -1))
    M = B.T @ t2 @ B
    Zr = np.linalg.solve(S, np.linalg.solve(S, M).T)
    assert np.abs(Z - Zr).max() <= 64 * P * EPS * cond * np.abs(Zr).max()
    # each eigenvector up to its sign: |W^T M W|, errors of the backward error over the nearest gap
    Tr = np.abs(V.T @ M @ V)
    gap = np.diff(w).min() / np.abs(w).max() if P > 1 else 1.0
    assert np.abs(np.abs(Th.cpu().numpy()) - Tr).max() <= 64 * P * EPS * cond / gap * Tr.max()


def test_metric_not_positive_definite_names_its_block(thc):
    """A zero column of the pair basis in the second block of 64: refused there, at the pivot."""
    import torch
    o, v, nL, P, Q = 8, 40, 20, 100, 60
    L, eps, Xo, Xv, xo, xv = _inputs(o, v, nL, P, Q, 1)
    Xo[:, 70] = 0.0
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda").contiguous()
    ctx = thc.THC(o, v, nL, P, Q)
    with pytest.raises(thc.ThcError, match="amplitude metric S is not positive definite .*block 1 of 2"):
        ctx.build_factors(t(L), t(eps), t(Xo), t(Xv), t(xo), t(xv))
    ctx.close()


@pytest.mark.parametrize("kw", [{}, {"precision": 1}, {"precision": 2}, {"flags": 3}, {"flags": 8}],
                         ids=["fp64", "mixed", "split", "unfused-streamed", "quintic"])
def test_reused_memory_gives_the_same_bits(thc, kw):
    """Nothing depends on what working memory held before: a workspace of NaNs, fresh memory and the
    memory of a context destroyed before give the same bits in set-up, residual, density and solve."""
    import torch
    o, v, nL, P, Q = 6, 30, 40, 70, 100
    L, eps, Xo, Xv, xo, xv = _inputs(o, v, nL, P, Q, 3)
    t = lambda x: torch.tensor(x, dtype=torch.float64, device="cuda").contiguous()
    args = [t(x) for x in (L, eps, Xo, Xv, xo, xv)]

    def one(workspace=None):
        ctx = thc.THC(o, v, nL, P, Q, workspace=workspace, **kw)
        Z = ctx.build_factors(*args)
        t1 = torch.linspace(-0.01, 0.01, o * v, dtype=torch.float64, device="cuda").reshape(o, v)
        res = ctx.residual(Z, t1)
        D = ctx.mp2_density(Z)
        need = ctx.memory_bytes()
        ctx.close()
        flat = [Z, *[x for x in (res if isinstance(res, (tuple, list)) else [res]) if isinstance(x, torch.Tensor)], *D]
        return [x.clone() for x in flat], need

    first, need = one()
    for _ in range(2):
        again, _ = one()
        assert all(torch.equal(a, b) for a, b in zip(first, again))
    ws = torch.full((need // 8,), float("nan"), dtype=torch.float64, device="cuda")
    nans, _ = one(ws)
    assert all(torch.equal(a, b) for a, b in zip(first, nans))
