"""pt_observe and pt_cost at the edges of their workgroups (16 simulations;
256 where the cost also ranks; 32 sensors a pass; ranking in the cost launch
up to 4096 simulations): the observation bit for bit the one that the window
kernel makes of the same step, the cost against float64, and the same bits
with and without the ranking."""
import numpy as np
import pytest
import torch

from tests import tiny

pytestmark = pytest.mark.gpu

R_SPH = 0.004
R_LINK = 0.006


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


def batch(pt, K, L, C_max, cost_mode):
    """Two rows of spheres on the table under L parallel links that press on
    them, each simulation's object at its own height, speed and friction."""
    rng = np.random.default_rng(100 * K + L)
    S = 8
    sph = np.zeros((1, S, 4))
    sph[0, :, 0] = (np.arange(S) // 2) * 0.01
    sph[0, :, 1] = (np.arange(S) % 2) * 0.01
    sph[0, :, 3] = R_SPH
    hand = np.array([tiny.link_row((-0.03, y, R_SPH + R_SPH + R_LINK - 2e-4), (0.06, y, R_SPH + R_SPH + R_LINK - 2e-4),
                                   R_LINK) for y in np.linspace(-0.002, 0.012, L)])
    st = np.repeat(tiny.state(x=(0.0, 0.0, R_SPH))[None], K, 0)
    st[:, 2] += rng.uniform(-2e-4, 2e-4, K)
    st[:, 7:] = rng.normal(0.0, 0.05, (K, 6))
    pr = np.stack([tiny.params(m, mu) for m, mu in zip(rng.uniform(0.05, 0.3, K), rng.uniform(0.2, 0.9, K))])
    g = [0, K] if K < 3 else [0, K // 3, K]
    return pt.Batch(hand=hand, spheres=sph, n_spheres=np.array([S], np.int32),
                    inv_inertia=np.array([[500.0, 500.0, 500.0]]), env_type=np.zeros(K, np.int32),
                    group_start=np.array(g, np.int32), consts=tiny.consts(cost_mode=cost_mode), C_max=C_max,
                    newton_iters=10, T=1, state=st, params=pr), rng


CASES = [(1, 1, 64), (15, 3, 7), (16, 20, 64), (17, 32, 33), (255, 33, 16), (256, 62, 64), (257, 20, 32),
         (4096, 5, 20), (4097, 5, 20)]


@pytest.mark.parametrize("cost_mode", [0, 1])
@pytest.mark.parametrize("K,L,C_max", CASES)
def test_observation_is_the_windows(pt, K, L, C_max, cost_mode):
    print(f"observe: K {K}, L {L}, C_max {C_max}, cost mode {cost_mode}", flush=True)
    b, _ = batch(pt, K, L, C_max, cost_mode)
    start = [t.clone() for t in (b.state, b.params, b.warm)]
    u = torch.zeros(max(b.D, 1), device="cuda")
    b.step(u, u)
    obs = b.observe()
    for t, v in zip((b.state, b.params, b.warm), start):
        t.copy_(v)
    out = b.new_obs(1)
    gt = torch.zeros((1, *b.obs_shape(b.G)), device="cuda")
    b.run_window(torch.zeros((2, max(b.D, 1)), device="cuda"), gt, torch.zeros(K, device="cuda"), None, out, graph=False)
    torch.cuda.synchronize()
    b.close()
    assert (obs[0] > 0).any()
    assert torch.equal(obs.view(torch.int32), out[0].view(torch.int32))


@pytest.mark.parametrize("K,L,C_max", CASES)
def test_cost_against_float64(pt, K, L, C_max):
    print(f"cost: K {K}, L {L}", flush=True)
    b, rng = batch(pt, K, L, C_max, 0)
    c = tiny.consts()
    obs = rng.normal(size=(4, L, K)).astype(np.float32)
    gt = rng.normal(size=(4, L, b.G)).astype(np.float32)
    c0 = rng.uniform(0.0, 5.0, K).astype(np.float32)
    group = np.searchsorted(b.group_start[1:], np.arange(K), side="right")
    d = obs.astype(np.float64) - gt.astype(np.float64)[:, :, group]
    want = c0 + (c.w_mag * d[0] ** 2 + c.w_dir * (d[1:] ** 2).sum(0)).sum(0)
    dev = [torch.as_tensor(x, device="cuda") for x in (obs, gt)]
    ranked, plain = (torch.as_tensor(c0, device="cuda") for _ in range(2))
    ranked = ranked.clone()
    plain = plain.clone()
    best = torch.full((b.G,), -1, dtype=torch.int32, device="cuda")
    b.cost(*dev, ranked, best)
    b.cost(*dev, plain)
    torch.cuda.synchronize()
    starts = b.group_start
    b.close()
    got = ranked.cpu().numpy()
    assert torch.equal(ranked, plain)
    # every term is positive: the sum of L terms and the start loses at most
    # one rounding each, a term at most eight (differences, squares, weights)
    np.testing.assert_allclose(got, want, rtol=(L + 9) * 2.0 ** -24, atol=0)
    assert best.cpu().tolist() == [int(lo + np.argmin(got[lo:hi])) for lo, hi in zip(starts[:-1], starts[1:])]
