"""The cost of Eq. 3 at the edges of its workgroups (16 simulations, or 256
where it also ranks; 32 sensors a pass): against float64, and the same bits
with and without the ranking and in the window kernel."""
import math

import numpy as np
import pytest
import torch

from tests import test_gpu_observe_cost as base
from tests import tiny

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


def rows(rng, L, n):
    """Observations with every state of contact, slip and spin, clear of the
    thresholds."""
    on, slip = rng.random((L, n)) < 0.6, rng.random((L, n)) < 0.5
    way = rng.normal(size=(3, L, n))
    ang = rng.uniform(-math.pi, math.pi, (L, n))
    o = np.zeros((7, L, n))
    o[0] = np.where(on, rng.uniform(0.02, 3.0, (L, n)), rng.uniform(0.0, 0.009, (L, n)))
    o[1:4] = way / np.linalg.norm(way, axis=0) * on
    o[4], o[5] = np.cos(ang) * slip, np.sin(ang) * slip
    o[6] = rng.integers(-1, 2, (L, n))
    return o.astype(np.float32)


def angle(a, b):
    return 2 * np.arctan2(np.sqrt(((a - b) ** 2).sum(0)), np.sqrt(((a + b) ** 2).sum(0)))


@pytest.mark.parametrize("K,L,C_max", base.CASES + [(700, 62, 8), (5, 33, 4)])
def test_cost_against_float64(pt, K, L, C_max):
    print(f"Eq. 3 cost: K {K}, L {L}", flush=True)
    b, rng = base.batch(pt, K, L, C_max, 1)
    c = tiny.consts(cost_mode=1)
    w = np.asarray(c.w_eq3, dtype=np.float32).astype(np.float64)
    obs, gt = rows(rng, L, K), rows(rng, L, b.G)
    c0 = rng.uniform(0.0, 5.0, K).astype(np.float32)
    group = np.searchsorted(b.group_start[1:], np.arange(K), side="right")
    x, y = obs.astype(np.float64), gt.astype(np.float64)[:, :, group]
    touch, slip, spin = [(s(x), s(y)) for s in (lambda o: o[0] > c.tau_contact,
                                                lambda o: (o[4] != 0) | (o[5] != 0), lambda o: o[6] != 0)]
    term = np.where(touch[0] == touch[1], w[1] * np.abs(x[0] - y[0]) + w[2] * angle(x[1:4], y[1:4]) * touch[0], w[0])
    term += np.where(slip[0] == slip[1], w[4] * angle(x[4:6], y[4:6]) * slip[0], w[3])
    term += np.where(spin[0] == spin[1], w[6] * np.abs((x[6] > 0) * 1.0 - (y[6] > 0)) * spin[0], w[5])
    want = c0 + term.sum(0)
    dev = [torch.as_tensor(v, device="cuda") for v in (obs, gt)]
    ranked, plain = (torch.as_tensor(c0).cuda() for _ in range(2))
    best = torch.full((b.G,), -1, dtype=torch.int32, device="cuda")
    b.cost(*dev, ranked, best)
    b.cost(*dev, plain)
    torch.cuda.synchronize()
    starts = b.group_start
    b.close()
    got = ranked.cpu().numpy()
    assert torch.equal(ranked, plain)
    # every term is positive: at most one rounding for each of the L + 1 terms
    # of the sum, 24 in a term (differences, squares and their sums, two
    # roots, atan2f to 4 ulp, the weights, five sums)
    np.testing.assert_allclose(got, want, rtol=(L + 25) * 2.0 ** -24, atol=0)
    assert best.cpu().tolist() == [int(lo + np.argmin(got[lo:hi])) for lo, hi in zip(starts[:-1], starts[1:])]


@pytest.mark.parametrize("K,L,C_max", [(300, 20, 64), (4200, 5, 20)])
def test_cost_is_the_windows(pt, K, L, C_max):
    print(f"Eq. 3 cost, steps and window: K {K}, L {L}", flush=True)
    b, rng = base.batch(pt, K, L, C_max, 1)
    start = [t.clone() for t in (b.state, b.params, b.warm)]
    u = torch.zeros(max(b.D, 1), device="cuda")
    gt = torch.as_tensor(rows(rng, L, b.G)).cuda()
    b.step(u, u)
    obs = b.observe()
    plain, ranked, window = (torch.zeros(K, device="cuda") for _ in range(3))
    b.cost(obs, gt, plain)
    b.cost(obs, gt, ranked, torch.zeros(b.G, dtype=torch.int32, device="cuda"))
    for t, v in zip((b.state, b.params, b.warm), start):
        t.copy_(v)
    b.run_window(torch.zeros((2, max(b.D, 1)), device="cuda"), gt[None].contiguous(), window, graph=False)
    torch.cuda.synchronize()
    b.close()
    assert (plain != plain[0]).any()
    assert torch.equal(plain, ranked) and torch.equal(plain, window)
