"""The independent-wavefront kernel of full batches, at the edges of its block shapes: an environment's trajectory depends
on its run and index alone, so a batch that ends inside a block, inside a wavefront, or just past a whole round of blocks
agrees bit for bit with the start of another one, and a few runs (the small-batch kernel) with the start of many, also
where a run is no whole number of blocks.  Episodes of 5 steps."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [("spread", 3, 3, 0), ("spread", 4, 4, 0), ("spread", 6, 6, 0), ("spread", 7, 7, 0), ("spread", 10, 10, 0),
          ("tag", 3, 0, 2), ("tag", 4, 2, 3), ("tag", 5, 2, 4), ("tag", 10, 3, 8)]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries", SHAPES)
def test_batches_and_runs_agree_on_what_they_share(scenario, agents, landmarks, adversaries, ac):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    T, tag = 7, scenario == "tag"
    D = synth.tag_obs_dim(agents, landmarks, adversaries) if tag else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]

    def outputs(E, runs, keep, wd):
        if tag:
            cfg = synth.tag_config(E, agents, landmarks, adversaries, runs, 64, wd, max_episode_steps=5)
        else:
            cfg = synth.spread_config(E, agents, runs, 64, wd, max_episode_steps=5, reward_mode=agents % 2)
        env = MpeEnv(MpeConfig(**cfg))
        env.set_policy(*[w[:runs].contiguous() for w in policy])
        env.reset(11)
        if ac:
            env.set_critic(*[w[:runs].contiguous() for w in critic])
            out = env.rollout_ac(T, *env.empty_traj_ac(T))
        else:
            out = env.rollout(T, *env.empty_traj(T))
        TE = E * runs
        out = [(o[:, :keep] if o.dim() > 1 and o.shape[1] == TE else o[:keep]).clone() for o in out]
        out += [s[..., :keep].clone() for s in env.get_state()[:4]]
        env.close()
        return out

    per_wave = 64 // agents
    round4 = 256 * 4 * per_wave                      # one block of 4 wavefronts per CU of a 256-CU card
    for wd in (0, 1) if tag else (0,):
        policy, critic = dev(synth.policy_weights_with_bias(3, 1, D, 64)), dev(synth.critic_weights(3, 1, D, 64))
        full = 2 * round4 + per_wave + 1
        want = outputs(full, 1, full, wd)
        for E in (round4 * 3 // 2 + 5, round4 + per_wave - 1, round4 * 3 // 2 * 5 // 4):
            for k, (a, b) in enumerate(zip(outputs(E, 1, E, wd), want)):
                b = b[:, :E] if b.dim() > 1 and b.shape[1] == full else b[..., :E] if b.shape[-1] == full and a.shape[0] == b.shape[0] else b[:E]
                assert torch.equal(a, b), (wd, E, "output", k)
        many = 1200
        E = 48 if tag else 64
        policy, critic = dev(synth.policy_weights_with_bias(3, many, D, 64)), dev(synth.critic_weights(3, many, D, 64))
        for k, (a, b) in enumerate(zip(outputs(E, 3, 3 * E, wd), outputs(E, many, 3 * E, wd))):
            assert torch.equal(a, b), (wd, "runs", k)
