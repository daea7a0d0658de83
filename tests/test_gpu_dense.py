"""Scenes in which boxes mostly touch each other: more row contacts than the
quads take, bodies with long contact lists, many candidate pairs."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

FAR = [5.0, 5.0, 5.1, 5.0]


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_06649_amd import pmbs
    return pmbs


def f32(a):
    return np.asarray(a, np.float64).astype(np.float32).astype(np.float64)


def stepped(pm, st, bd, push, n_sub, waves, contacts):
    sim = pm.Sim(max_envs=1, max_bodies=len(st), max_contacts=contacts)
    sim.set_launch_plan(small_waves=waves, large_waves=waves)
    sim.set_state([0, len(st)], st, bd)
    sim.step(np.asarray(push, np.float32).reshape(1, 4), n_sub)
    return sim.get_state(), sim.env_status(), sim.stats()


def tray(n, seed=0):
    """n - 1 cubes on a plate, apart from each other, four contacts each with it."""
    rng = np.random.default_rng(seed + n)
    st, bd = np.zeros((n, 13)), np.zeros((n, 5))
    st[:, 3] = 1.0
    for i in range(n - 1):
        yaw = rng.uniform(-0.05, 0.05)
        st[i] = [0.03 * (i % 6) - 0.075, 0.03 * (i // 6) - 0.06, 0.0319, np.cos(yaw / 2), 0, 0, np.sin(yaw / 2),
                 *rng.normal(scale=0.02, size=3), *rng.normal(scale=0.1, size=3)]
        bd[i] = [0.012, 0.012, 0.012, rng.uniform(0.01, 0.03), 0.5]
    st[n - 1, 2] = 0.01
    bd[n - 1] = [0.1, 0.1, 0.01, 1.0, 0.4]
    return f32(st), f32(bd)


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("n", [5, 6, 7, 8, 9, 10, 16, 17, 18, 31])
def test_tray_of_cubes_matches_oracle(pm, n, waves):
    """A plate has 4 (n - 1) row contacts and as many pairs as cubes: 16 rows
    with five boxes are the last in quads of lanes, 64 with 17 a wave's first
    slot full; a list of 24 (seven boxes) is the last in a lane's registers; 4,
    8 and 16 pairs fill a pass.  One substep against the oracle under the bars
    of the other one-substep tests (1e-5 m and quaternion, 1e-4 velocity); the
    contact classes bit for bit alike."""
    st, bd = tray(n)
    g, status, stats = stepped(pm, st, bd, FAR, 1, waves, 128)
    o, _, _ = O.step(O.make_config(), np.array([0, n], np.int32), st, bd, f32([FAR]), 1)
    assert status[0] == 0 and stats[0, 0] == 4 * n
    assert np.abs(g[:, :7] - o[:, :7]).max() <= 1e-5
    assert np.abs(g[:, 7:] - o[:, 7:]).max() <= 1e-4
    for contacts in (256, 512):
        other = stepped(pm, st, bd, FAR, 1, waves, contacts)
        assert all(np.array_equal(a, b) for a, b in zip((g, status, stats), other)), contacts


def heap(n, seed):
    """n tilted boxes thrown into each other: face and edge contacts, and pairs
    that an axis keeps apart."""
    rng = np.random.default_rng(seed)
    st, bd = np.zeros((n, 13)), np.zeros((n, 5))
    side = int(np.ceil(n ** (1 / 3)))
    for i in range(n):
        q = rng.normal(size=4) * [1.0, 0.2, 0.2, 1.0]
        bd[i] = [*rng.uniform(0.012, 0.022, size=3), rng.uniform(0.05, 0.2), 0.5]
        cell = np.array([i % side, i // side % side, i // side ** 2])
        st[i, :3] = [0.034, 0.034, 0.034] * cell - [0.017 * (side - 1), 0.017 * (side - 1), -0.02]
        st[i, 3:7] = q / np.linalg.norm(q)
        st[i, 7:10] = rng.normal(scale=0.1, size=3)
        st[i, 10:13] = rng.normal(scale=2.0, size=3)
    return f32(st), f32(bd)


@pytest.mark.parametrize("n", [4, 5, 8, 16, 17, 31])
def test_heap_is_the_same_in_every_kernel(pm, n):
    """One and two waves take different passes over the candidate pairs (five
    to eight pairs: eight lanes a pair and sixteen) and different slots of the
    row contacts; both and every contact class that holds the heap give the
    same bits over 40 substeps of a push through it."""
    push = [-0.02 * n ** 0.5 - 0.06, 0.0, 0.0, 0.0]
    for seed in range(3):
        st, bd = heap(n, 100 * n + seed)
        want = stepped(pm, st, bd, push, 40, 1, 512)
        assert np.isfinite(want[0]).all()
        for contacts in (128, 256):
            one = stepped(pm, st, bd, push, 40, 1, contacts)
            two = stepped(pm, st, bd, push, 40, 2, contacts)
            assert all(np.array_equal(a, b) for a, b in zip(one, two)), (seed, contacts)
            if not one[1][0] & 1:
                assert all(np.array_equal(a, b) for a, b in zip(one, want)), (seed, contacts)


@pytest.mark.parametrize("n_sub", [0, 1, 15, 16, 17])
def test_step_is_ordered_from_16_substeps(pm, n_sub):
    """More environments than resident workgroups: a step of few substeps runs
    one workgroup per environment, one of 16 or more the work-ordered queues;
    states, status and statistics are those of the plain order."""
    from paper_2207_06649_amd import scenes
    b = scenes.concat([scenes.clutter_batch(3, 64, (1, 4))] * 56)   # 3584: past 12 a compute unit
    sim = pm.Sim(max_envs=b.n_envs, max_bodies=b.n_bodies)
    out = []
    for order in (0, 1):
        sim.set_launch_plan(order=order)
        sim.set_state(b.env_offset, f32(b.state), f32(b.body))
        sim.step(b.push.astype(np.float32), n_sub)
        out.append((sim.get_state(), sim.env_status(), sim.stats()))
    assert all(np.array_equal(x, y) for x, y in zip(*out))
