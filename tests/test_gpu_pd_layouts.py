"""The PD hand at the sizes where its solve keeps its blocks elsewhere or
takes its tasks in more turns, against the oracle step by step and the window
against the steps bit for bit: A_oh outside the segment records (two joints on
every link) with the group solutions in the spare words (18 joints) and
outside (24), more joints than one pass of the step cost and more group-solve
tasks than lanes (12 and 16 groups), with A_oh in the segment records (36
joints on 36 links) and outside (64 on 32, the most)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2002_12160_amd import scene as S
from tests import test_gpu_pd as pd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


# fingers, links per finger, two joints on every link, link length
HANDS = [(3, 3, True, 0.04), (4, 3, True, 0.04), (12, 3, False, 0.04), (16, 2, True, 0.055)]


def config(fingers, links, double, length, monkeypatch):
    """A ring of fingers round the small scene's cuboid; with `double` every
    link turns about its z axis too, by joints numbered after the others."""
    cfg = pd._pd_cfg("small")
    cfg = cfg.with_(C_max=64, hand=dataclasses.replace(cfg.hand, n_fingers=fingers, links_per_finger=links,
                                                       link_len=length))
    if double:
        single = S.build_hand

        def build(spec):
            rows, mean = single(spec)
            rows[:, 2] = rows[:, 1] + len(mean)
            rows[:, 6:9] = (0.0, 0.0, 1.0)
            return rows, np.concatenate([mean, np.zeros(len(mean))])

        monkeypatch.setattr(S, "build_hand", build)
    return cfg


@pytest.mark.parametrize("fingers,links,double,length", HANDS)
def test_per_step_parity(pt, fingers, links, double, length, monkeypatch):
    cfg = config(fingers, links, double, length, monkeypatch)
    pd._say(f"PD hand per-step parity: {fingers} fingers of {links} links, {'two joints' if double else 'a joint'} each")
    n_chk, n_ok, n_contact, fails = pd.pd_parity(pt, cfg, 16, 12)
    assert n_contact >= 0.25 * n_chk
    assert n_ok >= 0.15 * n_chk
    assert not fails


@pytest.mark.parametrize("fingers,links,double,length", HANDS)
@pytest.mark.parametrize("K", [21, 1100])
def test_window_equals_steps(pt, fingers, links, double, length, K, monkeypatch):
    cfg = config(fingers, links, double, length, monkeypatch).with_(T=4)
    pd._say(f"PD window vs steps: {fingers} fingers of {links} links, K={K}")
    ref = pd._pd_windows(pt, cfg, K, 2, batched=False)
    got = pd._pd_windows(pt, cfg, K, 2, batched=True)
    for w in range(2):
        for n, x, y in zip(("state", "params", "warm", "hand_state", "cost", "best", "obs", "parent"), ref[w], got[w]):
            assert torch.equal(x, y), f"window {w}: {n} differs"
        force = ref[w][6].view(torch.float32)[:, :fingers * links]
        assert torch.isfinite(force).all()
        # the last fingers' joints are the last groups'
        assert (force[:, -links:] > 0).any() and (force[:, :links] > 0).any()
