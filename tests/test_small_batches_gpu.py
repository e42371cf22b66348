"""The small-batch kernel (one 16-row tile per wavefront, service and critic wavefronts) against the kernels for full
batches: an environment's trajectory depends on its index alone, so the first environments of a batch of any size are
the same bit for bit.  Sizes: one env, a ragged block, two blocks; just past one 8-env and one 16-env block per CU, both
ragged, where other instantiations take over (16-env blocks with 6, 8 and 10 agents; operands read from LDS), as far as a
shape's range goes; episodes of 5 steps so that resets are frequent."""
import pytest

pytestmark = pytest.mark.gpu

SPREAD = [(1, 0), (1, 1), (2, 0), (2, 1), (3, 0), (3, 1), (4, 0), (5, 0), (6, 0), (7, 0), (8, 0), (9, 0), (10, 0)]     # agents, bf16
TAG = [(n, l, a, wd) for n, l, a in ((4, 2, 3), (2, 1, 1), (3, 0, 2), (6, 2, 4), (5, 2, 4), (8, 2, 6), (10, 3, 8)) for wd in (0, 1)]
CASES = [("spread", n, n, 0, wd) for n, wd in SPREAD] + [("tag",) + t for t in TAG]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries,wd", CASES)
def test_first_envs_do_not_depend_on_the_batch(scenario, agents, landmarks, adversaries, wd, ac):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T, big, small = 12, 40961 if agents > 3 else 57345, (1, 21, 32, 8 * cus + 5, 16 * cus + 5)
    D = synth.tag_obs_dim(agents, landmarks, adversaries) if scenario == "tag" else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    policy, critic = dev(synth.policy_weights_with_bias(3, 1, D, 64)), dev(synth.critic_weights(3, 1, D, 64))

    def outputs(E):
        if scenario == "tag":
            cfg = synth.tag_config(E, agents, landmarks, adversaries, 1, 64, wd, max_episode_steps=5)
        else:
            cfg = synth.spread_config(E, agents, 1, 64, wd, max_episode_steps=5, reward_mode=agents % 2)
        env = MpeEnv(MpeConfig(**cfg))
        env.set_policy(*policy)
        env.reset(11)
        if ac:
            env.set_critic(*critic)
            out = env.rollout_ac(T, *env.empty_traj_ac(T))
        else:
            out = env.rollout(T, *env.empty_traj(T))
        keep = min(E, max(small))
        out = [(o[:, :keep] if o.shape[0] == T and o.dim() > 1 and o.shape[1] == E else o[:keep]).clone() for o in out]
        state = [s[..., :keep].clone() for s in env.get_state()[:4]]
        env.close()
        return out, state

    ref, ref_state = outputs(big)
    for E in small:
        out, state = outputs(E)
        for k, (a, b) in enumerate(zip(out, ref)):
            b = b[:, :E] if b.shape[0] == T and a.shape[0] == T and a.shape != b.shape[:1] else b[:E]
            assert torch.equal(a, b), (E, "output", k)
        for k, (a, b) in enumerate(zip(state, ref_state)):
            assert torch.equal(a, b[..., :E]), (E, "state", k)
