"""Population-based resampling at the group sizes where the GPU ranks and
copies differently (one workgroup ranks and copies a group of up to 256;
larger ones are ranked 64 simulations per workgroup and copied 16 per
workgroup) against the oracle on the same costs: ties, NaN and infinities
among them.  Parents, copied states and warm caches are exact; the explored
parameters follow the oracle's to 1e-6 (the float32 normals).  The elites of
the refinement come from the same ranking: with no gradient steps it only
lists them."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2002_12160_amd import scene as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


@pytest.mark.parametrize("sizes", [(1,), (2, 3), (63, 64, 65), (256, 15, 1), (257,), (260, 17, 64, 1), (1000, 333),
                                   (4099,)], ids=str)
def test_ranks_and_copies_follow_the_oracle(pt, sizes):
    print(f"resampling groups of {sizes}", flush=True)
    K = sum(sizes)
    gs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    cfg = S.CONFIGS["small"]
    base = S.make_scene(cfg, K=4, steps=1)
    rng = np.random.default_rng(K)
    st = rng.normal(size=(K, 13)).astype(np.float32).astype(np.float64)
    pr = np.concatenate([rng.uniform(0.06, 0.19, (K, 1)), rng.uniform(0.4, 0.9, (K, 1)), np.zeros((K, 3))], axis=1)
    pr = pr.astype(np.float32).astype(np.float64)
    sc = S.round_to_f32(dataclasses.replace(base, env_type=np.zeros(K, np.int32), group_start=gs, state=st, params=pr))
    b = pt.Batch.from_scene(sc)
    keys = rng.integers(0, 1000, size=(K, cfg.C_max)).astype(np.int32)
    imp = rng.normal(size=(K, cfg.C_max, 3)).astype(np.float32).astype(np.float64)
    b.set_warm(keys, imp)
    # every fourth cost from a small set (ties), some NaN and infinite
    cost = rng.lognormal(2.0, 1.0, K).astype(np.float32)
    cost[::4] = rng.integers(1, 4, size=cost[::4].shape)
    cost[rng.random(K) < 0.05] = np.nan
    cost[rng.random(K) < 0.05] = np.inf
    dev = torch.as_tensor(cost).cuda()
    ranked = np.concatenate([lo + np.argsort(np.where(np.isnan(cost[lo:hi]), np.inf, cost[lo:hi]), kind="stable")
                             [:max(1, int(np.float32(hi - lo) * np.float32(cfg.elite_frac)))]
                             for lo, hi in zip(gs[:-1], gs[1:])])
    u = torch.zeros((b.T + 1, b.D), device="cuda")
    gt = torch.zeros((b.T, *b.obs_shape(b.G)), device="cuda")
    elites = b.refine_elites(u, gt, dev.clone(), b.snapshot(), steps=0)
    assert elites.tolist() == ranked.tolist()
    parent = torch.zeros(K, dtype=torch.int32, device="cuda")
    b.resample(dev, 5, parent)
    g_st, g_pr = b.get_state()
    g_k, g_r = b.get_warm()
    o = oracle.Oracle.from_scene(sc) if hasattr(oracle.Oracle, "from_scene") else \
        oracle.Oracle(sc.hand, sc.spheres, sc.n_spheres, sc.inv_inertia, cfg.consts, C_max=cfg.C_max,
                      newton_iters=cfg.newton_iters, D=sc.D)
    o_st, o_pr, o_k, o_r, o_c = sc.state.copy(), sc.params.copy(), keys.copy(), imp.copy(), cost.astype(np.float64)
    o_par = o.resample(oracle.resample_cfg(cfg), gs, 5, o_c, o_st, o_pr, o_k, o_r)
    b.close()
    assert parent.tolist() == o_par.tolist()
    assert np.array_equal(g_st, o_st) and np.array_equal(g_k, o_k) and np.array_equal(g_r, o_r)
    assert np.abs(g_pr - o_pr).max() <= 1e-6
    assert float(dev.abs().sum()) == 0.0
