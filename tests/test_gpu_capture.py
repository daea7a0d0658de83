"""Launches in captured graphs, replayed after environments of other body
counts were loaded: the step kernel's LDS layout for at most 16 boxes must
not meet an environment with more."""
import numpy as np
import pytest

from paper_2207_06649_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_06649_amd import pmbs
    return pmbs


def batch(seed, counts):
    return scenes.concat([scenes.clutter_batch(seed + i, 1, n) for i, n in enumerate(counts)])


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("spare", [0, 2297])
def test_callers_graph_of_a_step_serves_other_body_counts(pm, waves, spare):
    """A step that the caller captured with at most 16 boxes per environment
    is bit for bit the eager step of what is loaded at each replay, also with
    17, 20 and 31 boxes, as one workgroup per environment and (2297 further
    environments of one box) as the work-ordered step."""
    import torch
    loads = [(15, 16, 3), (17, 3, 1), (15, 16, 3), (20, 31, 5), (2, 16, 9)]
    one = scenes.clutter_batch(1, 1, 1)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        E = 3 + spare
        sim = pm.Sim(max_envs=E, max_bodies=64 + spare, stream=stream)
        sim.set_launch_plan(small_waves=waves)
        push = torch.zeros((E, 4), dtype=torch.float32, device="cuda:0")

        def load(k):
            b = batch(10 * k, loads[k])
            off = np.append(b.env_offset, b.env_offset[-1] + 1 + np.arange(spare))
            state = np.concatenate([b.state, np.repeat(one.state, spare, 0)])
            body = np.concatenate([b.body, np.repeat(one.body, spare, 0)])
            pushes = np.concatenate([b.push, np.repeat(one.push, spare, 0)]).astype(np.float32)
            push.copy_(torch.tensor(pushes))
            sim.set_state(off, state, body)

        def result():
            stream.synchronize()
            return sim.get_state(), sim.env_status(), sim.stats()

        want = []
        for k in range(len(loads)):
            load(k)
            sim.step(push, 30)
            want.append(result())
        load(0)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(push, 30)
        for k in range(len(loads)):
            load(k)
            graph.replay()
            assert same(result(), want[k]), loads[k]


@pytest.mark.parametrize("contacts,waves", [(128, 1), (128, 2), (256, 1), (512, 2)])
def test_captured_rollouts_serve_other_body_counts(pm, contacts, waves):
    """Rollouts of the same launch arguments on one simulator, the largest
    environment at most 16 boxes, then more, then fewer again: the kernels
    captured for one load are not replayed on the other, and both sets of
    kernels are kept.  Every replay is bit for bit the eager rollout of a fresh
    simulator."""
    import torch
    loads = [(12, 16, 3), (17, 20, 3), (15, 16, 8), (18, 5, 30), (31, 2, 16), (16, 16, 16)]
    E, H = 3, 2
    off = np.array([0, 2, 4, 6], np.int32)
    sim = pm.Sim(max_envs=E, max_bodies=64, max_contacts=contacts, max_horizon=H)
    rew = torch.zeros((E, H), dtype=torch.float32, device="cuda:0")
    cnt = torch.zeros(E, dtype=torch.int32, device="cuda:0")

    def roll(s, k, flags, rewards=None, counts=None):
        b = batch(10 * k, loads[k])
        s.set_launch_plan(small_max_bodies=31, small_waves=waves, large_waves=waves)
        s.load(b)
        acts = np.array([8 * (i % n) + 3 * i % 8 for n in loads[k] for i in range(2)], np.int32)
        got = s.rollout(acts, off, np.zeros(E, np.int32), n_substeps=20, max_h=H,
                        flags=flags | pm.ROLLOUT_WRITE_STATE, rewards=rewards, counts=counts)
        return got[0].copy(), got[1].copy(), s.get_state(), s.env_status()

    want = [roll(pm.Sim(max_envs=E, max_bodies=64, max_contacts=contacts, max_horizon=H), k, pm.ROLLOUT_QUEUE)
            for k in range(len(loads))]
    for turn in range(3):
        for k in range(len(loads)):
            rew.fill_(-1.0)
            cnt.zero_()
            got = roll(sim, k, pm.ROLLOUT_QUEUE | pm.ROLLOUT_GRAPH, rew, cnt)
            assert same(got, want[k]), (turn, loads[k])
