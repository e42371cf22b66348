"""The recurrent rollout in independent wavefronts (mpe_gru_waves.hip) against the block kernel (mpe_policy_gru.hip), bit for bit.
Per shape three batches of one run: a few envs (blocks); a batch just above what one round of blocks takes, all of it in
independent wavefronts, whose last one is partly filled; and a larger one that is split between the two kernels or, where that
is faster, all in blocks.  What an env does depends on (seed, run, env) only, so batches agree on the envs they share: state
carried over two rollouts, episodes of 5 steps, outputs left out in the second rollout of half the shapes."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [("spread", 1, 1, 0, 50001, 66000), ("spread", 2, 2, 0, 17001, 40000), ("spread", 3, 3, 0, 16500, 30000),
          ("spread", 4, 4, 0, 9001, 20000), ("spread", 5, 5, 0, 9001, 16400), ("spread", 6, 6, 0, 8301, 12000),
          ("spread", 7, 7, 0, 4201, 9000), ("spread", 8, 8, 0, 4201, 9000), ("spread", 9, 9, 0, 4201, 8000),
          ("spread", 10, 10, 0, 4201, 8000), ("tag", 4, 2, 3, 8301, 20000), ("tag", 2, 1, 1, 17001, 40000), ("tag", 3, 0, 2, 16500, 30000),
          ("tag", 6, 2, 4, 8301, 12000), ("tag", 5, 2, 4, 9001, 16400), ("tag", 8, 2, 6, 4201, 9000), ("tag", 10, 3, 8, 4201, 8000)]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries,mid,large", SHAPES)
def test_wavefronts_agree_with_blocks(scenario, agents, landmarks, adversaries, mid, large, ac):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    T, few, H = 7, 101, synth.GRU_HIDDEN
    tag = scenario == "tag"
    D = synth.tag_obs_dim(agents, landmarks, adversaries) if tag else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    policy, critic = dev(synth.gru_weights(5, 1, D)), dev(synth.gru_critic_weights(5, 1))

    def outputs(E, keep):
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
        for k in range(2):
            bufs = list(env.empty_traj_ac(T) if ac else env.empty_traj(T))
            if k and agents % 2:
                bufs[0] = bufs[2] = bufs[-1] = None
            out = env.rollout_ac(T, *bufs) if ac else env.rollout(T, *bufs)
            kept += [(o[:, :keep] if o.dim() > 1 and o.shape[1] == E else o[:keep]).clone() for o in out if o is not None]
        kept += [s[..., :keep].clone() for s in env.get_state()[:4]]
        kept.append(env.get_hidden().reshape(E, -1)[:keep].clone())
        env.close()
        return kept

    print("recurrent %s, %d agents, %s" % (scenario, agents, "actor-critic" if ac else "plain"), flush=True)
    for small, big in ((few, mid), (mid, large)):
        for k, (a, b) in enumerate(zip(outputs(small, small), outputs(big, small))):
            assert torch.equal(a, b), ("output", k, small, big)
