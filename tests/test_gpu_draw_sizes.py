"""The weighted resamplers at the group sizes where their workgroup changes
(256 threads up to 2048 simulations, 1024 beyond; one entry per thread, ragged
chunks, the largest group) and REPS's temperature from far and near starts:
weights and temperature against the oracle's to 2e-5 (its dual is minimised
directly, good to about 1e-7 in the temperature), every draw inside its
interval of the oracle's running weight sums, copies of the drawn parents."""
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


@pytest.mark.parametrize("sizes", [(1, 2, 255, 257), (1025, 2048), (2049,), (16384,)], ids=str)
@pytest.mark.parametrize("eps", [0.05, 0.3, 2.0])
@pytest.mark.parametrize("lost", [0.0, 0.02])
def test_reps_weights_at_the_workgroup_edges(pt, sizes, eps, lost):
    print(f"REPS groups of {sizes}, epsilon {eps}", flush=True)
    K = sum(sizes)
    gs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rng = np.random.default_rng(K)
    cost = rng.lognormal(3.0, 0.8, K)
    cost = np.where(rng.random(K) < lost, 100 * cost, cost).astype(np.float32)
    base = S.make_scene(S.CONFIGS["small"], K=4, steps=1)
    st = rng.normal(size=(K, 13)).astype(np.float32)
    sc = S.round_to_f32(dataclasses.replace(base, env_type=np.zeros(K, np.int32), group_start=gs,
                                            state=st.astype(np.float64), params=np.tile([0.1, 0.5, 0, 0, 0], (K, 1))))
    b = pt.Batch.from_scene(sc)
    parent = torch.zeros(K, dtype=torch.int32, device="cuda")
    weights, eta = torch.zeros(K, device="cuda"), torch.zeros(b.G, device="cuda")
    b.resample_reps(torch.as_tensor(cost).cuda(), 10, 3, eps, parent, weights, eta)
    pmf, o_eta = RS.group_pmf("reps", float(np.float32(eps)), cost.astype(np.float64), 10, gs)
    # no interior minimum: the eta -> 0+ limit, reported as 0 (the oracle's
    # minimiser then stops at the lower end of its bracket)
    for g, (lo, hi) in enumerate(zip(gs[:-1], gs[1:])):
        if 1 < hi - lo and np.float32(eps) >= np.log((hi - lo) / np.sum(cost[lo:hi] == cost[lo:hi].min())):
            assert o_eta[g] < 1e-12
            o_eta[g] = 0.0
    par, w = parent.cpu().numpy(), weights.cpu().numpy()
    g_st, _ = b.get_state()
    b.close()
    finite = np.isfinite(o_eta)
    assert np.array_equal(finite, np.isfinite(eta.cpu().numpy()))
    np.testing.assert_allclose(eta.cpu().numpy()[finite], np.asarray(o_eta)[finite], rtol=2e-5)
    np.testing.assert_allclose(w, pmf, atol=2e-5 * pmf.max())
    _, cdf, target = RS.draw_parents(pmf, gs, 3, S.CONFIGS["small"].seed)
    for lo, hi in zip(gs[:-1], gs[1:]):
        assert np.all((par[lo:hi] >= lo) & (par[lo:hi] < hi))
        c = np.asarray(cdf)[lo:hi]
        band = 1e-5 * c[-1]
        at = par[lo:hi] - lo
        t = np.asarray(target)[lo:hi]
        assert np.all(c[at] >= t - band) and np.all(np.where(at > 0, c[at - 1], 0.0) <= t + band)
    assert np.array_equal(g_st.astype(np.float32), st[par])
