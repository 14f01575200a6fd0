"""WRS at the group sizes where its workgroup changes (256 threads where the
largest group has up to 1024 simulations, 1024 threads beyond): weights to the
float32 rounding of their float64 values, every draw inside its interval of
the oracle's running weight sums, copies of the drawn parents."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import resamplers as RS
from paper_2002_12160_amd import scene as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


@pytest.mark.parametrize("sizes", [(1, 255, 1024), (1, 1023, 1025), (2048, 3, 2049), (16384,)], ids=str)
@pytest.mark.parametrize("lam", [0.25, 4.0])
def test_wrs_at_the_workgroup_edges(pt, sizes, lam):
    print(f"WRS groups of {sizes}, lambda {lam}", flush=True)
    K = sum(sizes)
    gs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rng = np.random.default_rng(K)
    cost = rng.lognormal(3.0, 0.8, K).astype(np.float32)
    cost[rng.random(K) < 0.02] = np.inf
    cost[gs[:-1]] = 20.0
    base = S.make_scene(S.CONFIGS["small"], K=4, steps=1)
    st = rng.normal(size=(K, 13)).astype(np.float32)
    sc = S.round_to_f32(dataclasses.replace(base, env_type=np.zeros(K, np.int32), group_start=gs,
                                            state=st.astype(np.float64), params=np.tile([0.1, 0.5, 0, 0, 0], (K, 1))))
    b = pt.Batch.from_scene(sc)
    parent = torch.zeros(K, dtype=torch.int32, device="cuda")
    weights = torch.zeros(K, device="cuda")
    b.resample_wrs(torch.as_tensor(cost).cuda(), 10, 3, lam, parent, weights)
    pmf, _ = RS.group_pmf("wrs", lam, cost.astype(np.float64), 10, gs)
    par = parent.cpu().numpy()
    g_st, _ = b.get_state()
    got = weights.cpu().numpy()
    b.close()
    # exp and the sum in float64 (errors below 1e-12), one rounding to float32
    np.testing.assert_allclose(got, pmf, rtol=2.0 ** -23, atol=1e-38)
    _, cdf, target = RS.draw_parents(pmf, gs, 3, S.CONFIGS["small"].seed)
    for lo, hi in zip(gs[:-1], gs[1:]):
        assert np.all((par[lo:hi] >= lo) & (par[lo:hi] < hi))
        c = np.asarray(cdf)[lo:hi]
        band = 1e-9 * c[-1]
        at = par[lo:hi] - lo
        t = np.asarray(target)[lo:hi]
        assert np.all(c[at] >= t - band) and np.all(np.where(at > 0, c[at - 1], 0.0) <= t + band)
    assert np.array_equal(g_st.astype(np.float32), st[par])
