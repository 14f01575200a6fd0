"""The float32 solve's narrow phase at the sphere counts where its blocks of
64 end (one block, two, one left over), with lists that hold every candidate
and lists that are cut while they fill: the kept contacts are those of the
float64 solve, whose narrow phase computes the same gaps (and which
test_gpu_cap_cut checks against the oracle).  The scene is that test's: spheres
in a row between the table and parallel links, every pair a candidate."""
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


@pytest.mark.parametrize("S,L,C_max", [(1, 1, 4), (63, 3, 64), (64, 1, 64), (64, 62, 37), (65, 2, 64), (128, 1, 64),
                                       (129, 2, 16), (192, 3, 64), (193, 62, 64), (256, 6, 64)])
def test_float32_keeps_the_same_contacts(pt, S, L, C_max):
    print(f"narrow phase: {S} spheres, {L} links, C_max {C_max}", flush=True)
    rng = np.random.default_rng(S + L)
    sph = np.zeros((1, S, 4))
    sph[0, :, 0] = (np.arange(S) - (S - 1) / 2) * 0.005
    sph[0, :, 2] = (rng.permutation(S) - S / 2) * 2e-5
    sph[0, :, 3] = R_SPH
    half = 0.005 * S / 2 + 0.01
    hand = np.array([tiny.link_row((-half, 0.0, z), (half, 0.0, z), R_LINK)
                     for z in 2 * R_SPH + R_LINK + 1.05e-4 + 3.7e-6 * np.arange(L)])
    kept = []
    for prec in (32, 64):
        b = pt.Batch(hand=hand, spheres=sph, n_spheres=np.array([S], np.int32), inv_inertia=np.array([[50.0, 50.0, 50.0]]),
                     env_type=np.zeros(1, np.int32), group_start=np.array([0, 1], np.int32), consts=tiny.consts(),
                     C_max=C_max, newton_iters=10, T=1, state=tiny.state(x=(0.0, 0.0, R_SPH))[None],
                     params=tiny.params(0.1, 0.5)[None], solve_precision=prec)
        start = b.snapshot()
        u = torch.zeros((2, 1), device="cuda")
        b.step(u[0], u[1])
        kept.append(b.get_warm()[0].tolist())
        for x, v in zip((b.state, b.params, b.warm), start):
            x.copy_(v)
        b.run_window(u, torch.zeros((1, *b.obs_shape(1)), device="cuda"), torch.zeros(1, device="cuda"), graph=False)
        kept.append(b.get_warm()[0].tolist())
        stats = b.read_stats()
        b.close()
        n = S * (L + 1)
        assert stats["candidates"] == 2 * n and stats["dropped"] == 2 * max(0, n - C_max)
    assert kept[0] == kept[1] == kept[2] == kept[3]
    assert sum(k >= 0 for k in kept[0][0]) == min(S * (L + 1), C_max)
