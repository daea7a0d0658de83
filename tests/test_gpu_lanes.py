"""Work split over the lanes of a wave, at the body counts where the split
turns: one box, full quads, the last and the first past a wave."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2207_06649_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_06649_amd import pmbs
    return pmbs


def f32(a):
    return np.asarray(a, np.float64).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31])
def test_reward_shared_vertices(pm, n):
    """Four lanes share a box's vertices (16 boxes fill the wave, more take a
    second turn); tilted boxes, the first and the last as target.  FP32
    positions of at most 0.5 m carry 3e-8 m of rounding each, a distance a few
    of them: 1e-6 m, and a relative 1e-5 for its divide and products."""
    rng = np.random.default_rng(n)
    st, bd, _ = scenes.clutter_env(rng, n)
    q = st[:, 3:7] + rng.normal(scale=0.05, size=(n, 4))
    st[:, 3:7] = q / np.linalg.norm(q, axis=1, keepdims=True)
    st, bd = f32(st), f32(bd)
    sim = pm.Sim(max_envs=1, max_bodies=n)
    sim.set_state([0, n], st, bd)
    for target in sorted({0, n - 1}):
        rew, clr = sim.eval_reward([target], 0.08)
        want = O.clearance(st, bd, target)
        if n == 1:
            assert np.isinf(clr[0]) and rew[0] == 1.0
        else:
            assert abs(clr[0] - want) <= 1e-6 + 1e-5 * want
            assert abs(rew[0] - O.reward(st, bd, target, 0.08)) <= 2e-5
