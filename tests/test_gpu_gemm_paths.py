"""The FP64 product on LDS-staged operands at the edges of its tiles (64, 128), stages (8 k) and row
padding, for every transpose, scale and output form a caller can reach, against host FP64 products."""
import ctypes as C

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


def _padded(rng, batch, rows, cols, ld):
    """batch x rows x ld with NaN in the columns past cols (never part of a product)."""
    X = np.full((batch, rows, ld), np.nan)
    X[:, :, :cols] = rng.standard_normal((batch, rows, cols))
    return X


# M, N around one and several 64- and 128-row tiles; K of less than a stage, of ragged stages and of
# split length; enough rows or batches that the 128 x 64 tiles are taken (512 of them) and not
CASES = [(1, 1, 1, 1), (64, 64, 8, 1), (63, 65, 7, 2), (65, 63, 9, 2), (128, 129, 16, 1), (127, 64, 17, 3),
         (129, 130, 63, 2), (200, 37, 65, 2), (31, 279, 62, 5), (257, 191, 279, 1), (1000, 20, 1000, 1),
         (4099, 1030, 50, 1), (2050, 1100, 71, 1), (620, 620, 279, 8), (130, 70, 33, 300)]


@pytest.mark.parametrize("tA,tB", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("M,N,K,batch", CASES)
def test_products_at_edges(thc, M, N, K, batch, tA, tB):
    import torch
    print(f"[gpu-gemm] {M} x {N} x {K}, batch {batch}, trans {tA} {tB}", flush=True)
    lib = thc.load()
    rng = np.random.default_rng(M * 7 + N * 5 + K * 3 + batch)
    ra, ca = (K, M) if tA else (M, K)
    rb, cb = (N, K) if tB else (K, N)
    lda, ldb, ldc = ca + rng.integers(0, 4), cb + rng.integers(0, 4), N + rng.integers(0, 4)
    shared = batch > 1 and K % 2 == 1  # one B for the whole batch
    A, B = _padded(rng, batch, ra, ca, lda), _padded(rng, 1 if shared else batch, rb, cb, ldb)
    C0 = _padded(rng, batch, M, N, ldc)
    alpha, beta = (1.0, 0.0) if N % 2 else (-0.75, 1.5)
    dA, dB, dC = (torch.from_numpy(x).to("cuda") for x in (A, B, C0))
    ptr = lambda t: C.c_void_p(t.data_ptr())
    rc = lib.thc_dgemm(int(tA), int(tB), M, N, K, alpha, ptr(dA), int(lda), ra * int(lda), ptr(dB), int(ldb),
                       0 if shared else rb * int(ldb), beta, ptr(dC), int(ldc), M * int(ldc), batch,
                       C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    got = dC.cpu().numpy()
    a, b = A[:, :, :ca], B[:, :, :cb]
    a, b = (x.transpose(0, 2, 1) if t else x for x, t in ((a, tA), (b, tB)))
    prev = np.where(beta != 0.0, beta * C0[:, :, :N], 0.0)
    want = alpha * (a @ b) + prev
    # both sides' sums of K products, the scaling and the addition, each rounded: K + 4 ulps of the terms
    bound = 2.0 * (K + 4) * 2.0 ** -53 * (abs(alpha) * (np.abs(a) @ np.abs(b)) + np.abs(prev))
    assert np.all(np.abs(got[:, :, :N] - want) <= bound)
    assert np.all(np.isnan(got[:, :, N:]))  # the padding of C is not written
