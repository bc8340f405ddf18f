"""The length of the fused pass's blocks of Cholesky vectors (host only): whole-nL or long equal blocks where the
panels are small, blocks of 64 at the benchmark workload, and never at the cost of the rest of the plan."""
import random

import pytest

from paper_2111_11473_amd import thc


@pytest.mark.parametrize("o,v,nL,nP,nQ,want", [(6, 22, 70, 50, 110, 70), (10, 40, 150, 120, 300, 150),
                                               (31, 279, 930, 620, 1550, 155), (50, 450, 1500, 1000, 2500, 64),
                                               (4, 8, 2500, 16, 20, 834)])
def test_block_lengths(o, v, nL, nP, nQ, want):
    assert thc.plan_query(o, v, nL, nP, nQ, 270e9)["a_block"] == want


def test_longer_blocks_change_nothing_else():
    """Whatever is planned with explicit blocks of 64 is planned without, with the same H blocks, chunks and
    residency, at every budget (tight ones fall back to 64), and a longer block fits the budget wherever 64 do."""
    rng = random.Random(11)
    longer = 0
    for _ in range(400):
        o = rng.choice([1, 3, 8, 16, 31, 50])
        v = max(1, int(o * rng.uniform(1, 10)))
        nL = max(1, int((o + v) * rng.uniform(0.5, 4)))
        nP = max(1, min(o * v, int(rng.uniform(0.5, 25) * o)))
        nQ = max(1, min(o * v, int(nP * rng.uniform(1, 3))))
        budget = 10 ** rng.uniform(7, 11.43)
        kw = dict(synthetic=rng.random() < 0.3, precision=rng.choice([0, 1]))
        nb = max(1, min(64, int(4.0e9 / (32.0 * nP * nP)), nL))
        try:
            p = thc.plan_query(o, v, nL, nP, nQ, budget, a_block=nb, **kw)
        except thc.ThcError as e:
            assert e.rc == thc.THC_ENOMEM
            with pytest.raises(thc.ThcError):
                thc.plan_query(o, v, nL, nP, nQ, budget, **kw)
            continue
        q = thc.plan_query(o, v, nL, nP, nQ, budget, **kw)
        for key in ("x_block", "i_chunk", "x7_chunk", "lvv_resident", "quintic", "q_pairs", "q_jchunk"):
            assert p[key] == q[key], (key, o, v, nL, nP, nQ, budget, kw)
        assert q["a_block"] >= p["a_block"] and q["device_bytes"] <= max(budget, p["device_bytes"])
        longer += q["a_block"] > p["a_block"]
    assert longer > 50
