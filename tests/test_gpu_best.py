"""The running best of every group (pt_cost's and pt_run_window's `best`) at
the group counts where the ranking workgroup's wavefronts divide differently
among the groups: the whole workgroup on one group, teams of wavefronts,
a wavefront per group, several groups per wavefront; from LDS (one workgroup),
from the last workgroup and from a launch of its own.  The lowest index of the
lowest cost, NaN as +inf, exact."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2002_12160_amd import scene as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


def batch(pt, name, K, G, seed):
    """K simulations in G groups of uneven sizes (one simulation at least)."""
    rng = np.random.default_rng(seed)
    gs = np.concatenate([[0], np.sort(rng.choice(np.arange(1, K), G - 1, replace=False)), [K]]).astype(np.int32)
    cfg = S.CONFIGS[name].with_(T=1, newton_iters=1)
    base = S.make_scene(cfg, K=S.CONFIGS[name].G, steps=2)
    types = np.resize(np.arange(base.spheres.shape[0]), K).astype(np.int32)
    st = np.zeros((K, 13))
    st[:, :7] = base.rest_pose[types]
    st[:, 7:] = rng.normal(0.0, 0.05, (K, 6))
    sc = S.round_to_f32(dataclasses.replace(base, env_type=types, group_start=gs, state=st,
                                            params=np.tile([0.1, 0.5, 0.0, 0.0, 0.0], (K, 1))))
    return pt.Batch.from_scene(sc), rng


def lowest(cost, starts):
    c = np.where(np.isnan(cost), np.inf, cost)
    return [int(lo + np.argmin(c[lo:hi])) for lo, hi in zip(starts[:-1], starts[1:])]


# links: 9 (16 wavefronts rank) and 20; simulations: one workgroup, several,
# and more than the ranking in the cost launch takes
@pytest.mark.parametrize("name", ["small", "realtime16384"])
@pytest.mark.parametrize("K", [60, 256, 700, 4096, 5000])
def test_cost_ranks_every_group(pt, name, K):
    for G in (1, 2, 3, 5, 8, 9, 15, 16, 17, 33, 60):
        print(f"cost ranking, {name}: {K} simulations in {G} groups", flush=True)
        b, rng = batch(pt, name, K, G, 100 * K + G)
        cost = rng.lognormal(2.0, 1.0, K).astype(np.float32)
        cost[::3] = rng.integers(1, 4, size=cost[::3].shape)
        cost[rng.random(K) < 0.1] = np.nan
        cost[rng.random(K) < 0.1] = np.inf
        dev = torch.as_tensor(cost).cuda()
        best = torch.full((G,), -1, dtype=torch.int32, device="cuda")
        zero = b.new_obs()          # equal observations add no cost
        gt = torch.zeros(b.obs_shape(G), device="cuda")
        b.cost(zero, gt, dev, best)
        b.cost(zero, gt, dev, best)   # the counter is back at its start
        starts = b.group_start
        b.close()
        assert np.array_equal(dev.cpu().numpy(), cost, equal_nan=True)
        assert best.tolist() == lowest(cost, starts)


@pytest.mark.parametrize("waves", [1, 2, 4])
def test_window_ranks_every_group(pt, waves):
    K = 150
    for G in (1, 2, 3, 4, 5, 9, 60):
        print(f"window ranking: {G} groups, {waves} simulations per workgroup", flush=True)
        b, rng = batch(pt, "small", K, G, G)
        b.set_tuning(waves)
        u = torch.zeros((2, b.D), device="cuda")
        gt = torch.as_tensor(rng.normal(size=(1, *b.obs_shape(G))).astype(np.float32)).cuda()
        c0 = rng.integers(0, 3, K).astype(np.float32)
        cost = torch.as_tensor(c0).cuda()
        best = torch.full((G,), -1, dtype=torch.int32, device="cuda")
        b.run_window(u, gt, cost, best, graph=False)
        starts = b.group_start
        b.close()
        got = cost.cpu().numpy()
        assert not np.array_equal(got, c0)
        assert best.tolist() == lowest(got, starts)
