"""The service lanes of the recurrent kernel (sampling noise one step ahead, outputs of the sampling): a block of 16 envs
with a ragged last one against the large blocks of a full batch, bit for bit, with rows that fill 1 to 3 wavefronts, and
the one shape whose LDS has no room for the noise in its large block (3 agents of predator-prey, actor-critic).  Episodes
of 5 steps, two rollouts in turn."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries", [
    ("spread", 1, 1, 0), ("spread", 3, 3, 0), ("spread", 5, 5, 0), ("tag", 3, 0, 2), ("tag", 4, 2, 3), ("tag", 6, 2, 4)])
def test_small_blocks_agree_with_large_ones(scenario, agents, landmarks, adversaries, ac):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    T, few, many, H = 7, 101, 8261, synth.GRU_HIDDEN
    tag = scenario == "tag"
    D = synth.tag_obs_dim(agents, landmarks, adversaries) if tag else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    policy, critic = dev(synth.gru_weights(5, 1, D)), dev(synth.gru_critic_weights(5, 1))

    def outputs(E):
        if tag:
            cfg = synth.tag_config(E, agents, landmarks, adversaries, 1, H, 1, max_episode_steps=5)
        else:
            cfg = synth.spread_config(E, agents, 1, H, 1, max_episode_steps=5, reward_mode=agents % 2)
        env = MpeEnv(MpeConfig(**cfg))
        env.set_gru_policy(*policy)
        if ac:
            env.set_gru_critic(*critic)
        env.reset(11)
        kept = []
        for _ in range(2):
            out = env.rollout_ac(T, *env.empty_traj_ac(T)) if ac else env.rollout(T, *env.empty_traj(T))
            kept += [(o[:, :few] if o.dim() > 1 and o.shape[1] == E else o[:few]).clone() for o in out]
        kept += [s[..., :few].clone() for s in env.get_state()[:4]]
        kept.append(env.get_hidden().reshape(E, -1)[:few].clone())
        env.close()
        return kept

    for k, (a, b) in enumerate(zip(outputs(few), outputs(many))):
        assert torch.equal(a, b), ("output", k)
