"""Pairs that a face axis keeps apart are left out of the narrowphase until a
bound on their boxes' motion has used up the gap: against runs in which that
bound is past every gap at once."""
import numpy as np
import pytest

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


def stepped(pm, off, st, bd, push, n_sub, waves, contacts):
    sim = pm.Sim(max_envs=len(off) - 1, max_bodies=int(off[-1]), max_contacts=contacts)
    sim.set_launch_plan(small_waves=waves, large_waves=waves)
    sim.set_state(off, st, bd)
    sim.step(np.asarray(push, np.float32).reshape(-1, 4), n_sub)
    return sim.get_state(), sim.env_status(), sim.stats()


@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("n,waves", [(2, 1), (9, 1), (15, 2), (16, 1), (22, 1), (30, 2)])
def test_left_out_pairs_against_none_left_out(pm, n, waves, spin):
    """The bound grows each substep by 4.8e-7 of the farthest box's distance for
    the roundings of positions: a box 1e6 m away makes that 0.48 m, more than
    any gap between boxes whose AABBs overlap, so every such pair is tested in
    every substep.  Upright boxes that slide at each other at up to 1.5 m/s
    without turning (the bound's linear term alone, until they meet), or
    spinning ones; the others' states are bit for bit alike with and without
    the far box."""
    rng = np.random.default_rng(100 * n + 10 * waves + spin)
    E, side = 6, int(np.ceil(np.sqrt(n)))
    st, bd, push = np.zeros((E, n, 13)), np.zeros((E, n, 5)), np.zeros((E, 4))
    for e in range(E):
        for i in range(n):
            yaw = rng.uniform(0, 2 * np.pi)
            h = rng.uniform(0.01, 0.022, size=3)
            at = 0.058 * np.array([i % side - (side - 1) / 2, i // side - (side - 1) / 2])
            st[e, i, :3] = [*at, h[2] + (0.01 if spin else 0.0)]
            st[e, i, 3:7] = [np.cos(yaw / 2), 0, 0, np.sin(yaw / 2)]
            st[e, i, 7:9] = -at * rng.uniform(2.0, 8.0) + rng.normal(scale=0.3, size=2)
            st[e, i, 7:9] *= min(1.0, 1.5 / np.linalg.norm(st[e, i, 7:9]))
            if spin:
                st[e, i, 10:13] = rng.normal(scale=8.0, size=3)
            bd[e, i] = [*h, rng.uniform(0.05, 0.2), rng.uniform(0.05, 0.3)]
        x = 0.058 * side / 2 + 0.06
        push[e] = [-x, rng.uniform(-0.03, 0.03), x, 0.0]
    st, bd = f32(st), f32(bd)
    far_st, far_bd = np.zeros((E, n + 1, 13)), np.zeros((E, n + 1, 5))
    far_st[:, :n], far_bd[:, :n] = st, bd
    far_st[:, n, :4] = [0.0, 0.0, 1.0e6, 1.0]   # above: no contact of its own
    far_bd[:, n] = [0.5, 0.5, 0.5, 1.0, 0.5]
    contacts = 128 if n < 16 else 256
    got, status, _ = stepped(pm, np.arange(E + 1) * n, st.reshape(-1, 13), bd.reshape(-1, 5), push, 120, waves, contacts)
    want, far_status, _ = stepped(pm, np.arange(E + 1) * (n + 1), far_st.reshape(-1, 13), far_bd.reshape(-1, 5), push, 120,
                                  waves, contacts)
    assert np.isfinite(got).all() and np.array_equal(status, far_status) and not np.any(status & 1)
    assert np.array_equal(got, want.reshape(E, n + 1, 13)[:, :n].reshape(-1, 13))
    # boxes did meet: nothing else turns one that slides upright
    if not spin:
        assert np.abs(got.reshape(E, n, 13)[:, :, 3:7] - st[:, :, 3:7]).max() > 0.01
