"""The observation at the edges of its small workgroups (4 simulations up to
4096, 16 beyond), bit for bit the window's; and that the observations of Eq. 3
compared so hold slipping and spinning sensors."""
import pytest
import torch

from tests import test_gpu_observe_cost as base

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


@pytest.mark.parametrize("cost_mode", [0, 1])
@pytest.mark.parametrize("K,L,C_max", [(3, 1, 64), (4, 62, 64), (5, 9, 1), (259, 20, 64), (4095, 4, 16), (4096, 7, 40),
                                       (4099, 1, 64)])
def test_observation_at_the_small_workgroups(pt, K, L, C_max, cost_mode):
    base.test_observation_is_the_windows(pt, K, L, C_max, cost_mode)


def test_slip_and_spin_rows_are_there(pt):
    for K, L, C_max in [(256, 20, 64), (4097, 5, 20)]:
        print(f"Eq. 3 observation: K {K}, L {L}", flush=True)
        b, _ = base.batch(pt, K, L, C_max, 1)
        u = torch.zeros(max(b.D, 1), device="cuda")
        b.step(u, u)
        obs = b.observe()
        b.close()
        assert (obs[4:6] != 0).any() and (obs[6] > 0).any() and (obs[6] < 0).any()
