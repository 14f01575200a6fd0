"""Empty contact slots beside a contact with the smoothing so small that its
fourth power is no float32 number: the float32 solve's sums must not see the
empty slots' Jacobians, which are not finite there.  Objects of 26 and of
mixed sphere counts dropped on the table, so that some steps leave slots of
the last 16 empty; every simulation stays finite, step by step and in the
window, whose gradient's forward sweep shares the solve."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2002_12160_amd import scene as S

pytestmark = pytest.mark.gpu

STEPS = 8


@pytest.fixture(scope="module")
def pt():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2002_12160_amd import pt as _pt
    return _pt


@pytest.mark.parametrize("name", ["small", "batched4096"])
@pytest.mark.parametrize("delta", [3e-12, 1e-15])
def test_float32_solve_ignores_empty_slots(pt, name, delta):
    print(f"float32 solve, {name}, fb_delta {delta}", flush=True)
    cfg = S.CONFIGS[name]
    cfg = cfg.with_(consts=dataclasses.replace(cfg.consts, fb_delta=delta))
    K = 64
    sc = S.round_to_f32(S.make_scene(cfg, K=K, steps=STEPS))
    b = pt.Batch.from_scene(sc, solve_precision=32, T=STEPS)
    start = b.snapshot()
    u = torch.as_tensor(np.concatenate([sc.u[:1], sc.u]), dtype=torch.float32).cuda().contiguous()
    partly = np.zeros(K, bool)
    for t in range(STEPS):
        b.step(u[t], u[t + 1])
        st, _ = b.get_state()
        keys, _ = b.get_warm()
        n = (keys >= 0).sum(1)
        partly |= (n > 0) & (n % 16 != 0)
        assert np.isfinite(st).all(), f"step {t}: {np.count_nonzero(~np.isfinite(st).all(1))} simulations not finite"
    assert partly.any()
    plain = b.state.clone()
    for x, v in zip((b.state, b.params, b.warm), start):
        x.copy_(v)
    gt = torch.zeros((STEPS, *b.obs_shape(b.G)), device="cuda")
    cost = torch.zeros(K, device="cuda")
    b.run_window(u, gt, cost, graph=False)
    env = torch.arange(K, dtype=torch.int32, device="cuda")
    xi, warm0 = b.start_of(env, *start)
    g_cost, _, g_end, _ = b.window_grad(u, gt, env, xi, warm0, want_grad=False, want_end=True)
    torch.cuda.synchronize()
    assert torch.equal(b.state, plain) and torch.equal(g_end, plain)
    assert torch.isfinite(cost).all() and torch.equal(g_cost, cost)
    b.close()
