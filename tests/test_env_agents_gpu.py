"""Environment-only kernels with one lane per agent, and the ragged variant of the lane-per-env rollout: an environment's
trajectory depends on its index alone, so a small batch repeats the first environments of a large one bit for bit, and so
do single steps fed with the recorded actions.  The large batch runs another kernel for 3 to 10 agents of simple spread and
for predator-prey with 2, 3, 5, 6 and 8 agents.  Predator-prey with 4 and 10 agents has no other rollout kernel: those two
are compared with the oracle below.  1 and 2 agents of simple spread run the writer kernel at every size (its ragged
variant throughout, as the large batch is odd); its aligned variant with 3 agents is one more size."""
import numpy as np
import pytest

from tests import helpers as Hp

pytestmark = pytest.mark.gpu

TAG = ((4, 2, 3), (2, 1, 1), (3, 0, 2), (6, 2, 4), (5, 2, 4), (8, 2, 6), (10, 3, 8))
CASES = [("spread", n, n, 0, mode) for n in range(1, 11) for mode in (0, 1)] + [("tag",) + t + (0,) for t in TAG]


@pytest.mark.parametrize("scenario,agents,landmarks,adversaries,reward_mode", CASES)
def test_small_ragged_and_stepped_batches_repeat_the_large_one(scenario, agents, landmarks, adversaries, reward_mode):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    T, big = 11, 42001

    def make(E):
        if scenario == "tag":
            cfg = synth.tag_config(E, agents, landmarks, adversaries, max_episode_steps=4)
        else:
            cfg = synth.spread_config(E, agents, max_episode_steps=4, reward_mode=reward_mode)
        env = MpeEnv(MpeConfig(**cfg))
        env.reset(17)
        return env

    env = make(big)
    ref = [x[:, :128].clone() for x in env.rollout(T, *env.empty_traj(T))[:4]]
    last = env.rollout(1, None, None, None, None, env.empty_obs())[4][:128].clone()
    env.close()
    if scenario == "spread" and agents == 3:            # past the lane-per-agent range, whole waves, aligned slices
        E = 65 * torch.cuda.get_device_properties(0).multi_processor_count // 64 * 64 + 64
        env = make(E)
        out = env.rollout(T, *env.empty_traj(T))
        for k in range(4):
            assert torch.equal(out[k][:, :128], ref[k]), (E, k)
        env.close()
    for E in (1, 21, 64, 127):
        env = make(E)
        out = env.rollout(T, *env.empty_traj(T))
        for k in range(4):
            assert torch.equal(out[k], ref[k][:, :E]), (E, k)
        assert torch.equal(env.rollout(1, None, None, None, None, env.empty_obs())[4], last[:E]), (E, "last_obs")
        env.reset(17)
        obs, rew, done = env.empty_obs(), torch.empty(env.rew_shape, device="cuda"), torch.empty(E, dtype=torch.uint8, device="cuda")
        for t in range(T):
            env.step(ref[1][t, :E].contiguous(), obs, rew, done)
            assert torch.equal(rew, ref[2][t, :E]) and torch.equal(done, ref[3][t, :E]), (E, t)
            if t + 1 < T:
                assert torch.equal(obs, ref[0][t + 1, :E]), (E, t)
        env.close()


@pytest.mark.parametrize("shape", [(4, 2, 3), (10, 3, 8)])
def test_predator_prey_without_another_kernel_against_the_oracle(shape):
    """Many blocks, the last one ragged: the first envs and the last ones.  Actions, flags and episode starts as the oracle
    has them, positions of the first steps within the episode tolerance of the parity tests."""
    import torch
    from oracle import Oracle
    from paper_2311_10090_amd.binding import MpeEnv
    T, E, n = 30, 1003, 40
    env = MpeEnv(Hp.tag_gpu_config(E, *shape, 1, 0))
    env.reset(9)
    out = [o.cpu().numpy() for o in env.rollout(T, *env.empty_traj(T))]
    torch.cuda.synchronize()
    env.close()
    for off in (0, E - n):
        orc = Oracle(Hp.tag_oracle_config(n, *shape, 1, 0, env_offset=off), threads=4)
        orc.reset(9)
        ref = orc.rollout(T)
        obs, act, rew, done = [o[:, off:off + n] for o in out[:4]]
        assert np.array_equal(act, ref[1]) and np.array_equal(done, ref[3]), off
        assert np.abs(obs[0] - ref[0][0]).max() <= 1e-6 and np.abs(obs[25] - ref[0][25]).max() <= 1e-6, off
        assert np.abs(obs[:5] - ref[0][:5]).max() <= Hp.EPISODE_ATOL, off
