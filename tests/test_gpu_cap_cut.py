"""The contact cap at the candidate counts where its radix select changes
form: 64 (ranked as they are), up to 128, 256 and 512 (cut in one go, two,
four or eight words per lane), past 512 (cut in pieces of 512) and past the
list's capacity of 1536 (cut while the list fills), each with a count at the
edge and one beyond it, against the oracle: spheres in a row between the table
and parallel capsule links stacked 3.7 um apart, every pair a candidate, every
two gaps at least 0.1 um apart (100 times the float32 rounding of a gap), so
the kept keys are exact integers."""
import numpy as np
import pytest
import torch

import oracle
from tests import tiny

pytestmark = pytest.mark.gpu

R_SPH = 0.004
R_LINK = 0.006


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


@pytest.mark.parametrize("S,L,C_max", [(32, 1, 64), (33, 1, 64), (64, 1, 37), (43, 2, 64), (128, 1, 64), (129, 1, 1),
                                       (171, 1, 64), (256, 1, 64), (171, 2, 64), (192, 2, 5), (256, 3, 64),
                                       (256, 5, 64), (255, 6, 63)])
def test_cap_cut_keeps_the_oracles_keys(pt, S, L, C_max):
    ncand = S * (L + 1)
    print(f"cap cut: {ncand} candidates, C_max {C_max}", flush=True)
    rng = np.random.default_rng(1000 + ncand)
    sph = np.zeros((1, S, 4))
    sph[0, :, 0] = (np.arange(S) - (S - 1) / 2) * 0.005
    sph[0, :, 2] = (rng.permutation(S) - S / 2) * 2e-5
    sph[0, :, 3] = R_SPH
    sph = sph.astype(np.float32).astype(np.float64)
    half = 0.005 * S / 2 + 0.01
    hand = np.array([tiny.link_row((-half, 0.0, z), (half, 0.0, z), R_LINK)
                     for z in 2 * R_SPH + R_LINK + 1.05e-4 + 3.7e-6 * np.arange(L)]).astype(np.float32).astype(np.float64)
    inv = np.array([[50.0, 50.0, 50.0]])
    st = tiny.state(x=(0.0, 0.0, R_SPH))[None].astype(np.float32).astype(np.float64)
    pr = tiny.params(0.1, 0.5)[None]
    c = tiny.consts()
    o = oracle.Oracle(hand, sph, np.array([S], np.int32), inv, c, C_max=C_max, newton_iters=10, D=0)
    ost, opr = st.copy(), pr.copy()
    wk, wr = o.new_warm(1)
    o.batch_step(np.zeros(1, np.int32), np.zeros(0), np.zeros(0), ost, opr, wk, wr)
    b = pt.Batch(hand=hand, spheres=sph, n_spheres=np.array([S], np.int32), inv_inertia=inv,
                 env_type=np.zeros(1, np.int32), group_start=np.array([0, 1], np.int32), consts=c,
                 C_max=C_max, newton_iters=10, T=10, state=st, params=pr)
    u = torch.zeros(1, device="cuda")
    b.step(u, u)
    gk, _ = b.get_warm()
    stats = b.read_stats()
    b.close()
    kept = min(ncand, C_max)
    assert stats["candidates"] == ncand and stats["contacts"] == kept and stats["dropped"] == ncand - kept
    # the slots are in (gap, key) order on both sides
    assert gk[0][:kept].tolist() == wk[0][:kept].tolist()
    assert (gk[0][kept:] < 0).all()
