"""Several runs that are no whole number of the large kernels' blocks, and the bf16 block shapes between the small-batch
kernel and the large ones.  Jobs on both sides of a dispatch line run different kernels and agree bit for bit on the runs
(or environments) that they share: a trajectory depends on its run, its index in it and the seed alone.  The lines are
stated in 16-env blocks per CU, as in the dispatch, so the sizes follow the card.  Episodes of 5 steps."""
import pytest

pytestmark = pytest.mark.gpu

T = 11
TAG = {2: (2, 1, 1), 4: (4, 2, 3), 5: (5, 2, 4), 6: (6, 2, 4), 8: (8, 2, 6), 10: (10, 3, 8)}

# agents, bf16, actor-critic, envs per run, 16-env blocks per CU on either side of a line
TAG_RUNS = [(4, 0, 0, 16, 3.4, 3.7), (4, 0, 0, 160, 3.0, 9.0), (4, 1, 0, 16, 2.7, 3.0), (4, 1, 0, 48, 2.5, 8.2), (4, 1, 1, 16, 2.4, 2.7),
            (4, 1, 1, 32, 5.0, 7.2), (5, 1, 0, 16, 2.4, 2.7), (6, 1, 0, 16, 1.4, 1.7), (6, 1, 1, 48, 1.4, 1.7), (8, 0, 0, 16, 1.4, 1.7),
            (8, 1, 0, 48, 1.1, 1.5), (8, 1, 1, 16, 1.4, 1.7), (2, 1, 0, 16, 4.4, 4.8), (2, 1, 1, 48, 3.4, 3.7),
            # runs that stay with the small-batch kernel or end inside a block of independent wavefronts
            (5, 0, 1, 32, 1.2, 2.9), (6, 0, 0, 48, 1.2, 3.2), (10, 0, 0, 32, 1.0, 3.0)]
SPREAD_RUNS = [(2, 1, 0, 16, 5.8, 6.3), (2, 1, 0, 48, 5.8, 6.3), (2, 1, 1, 32, 4.8, 5.3), (2, 1, 1, 96, 7.7, 8.3), (3, 1, 1, 32, 5.8, 6.3),
               (3, 1, 1, 32, 8.2, 12.3), (3, 1, 0, 64, 5.8, 6.3), (6, 0, 0, 64, 1.8, 7.0), (9, 0, 0, 32, 1.0, 5.0), (10, 0, 1, 32, 1.0, 5.0)]
# one run, ragged: scenario, agents, bf16, actor-critic, 16-env blocks per CU on either side
ONE_RUN = [("tag", 4, 1, 1, 1.9, 2.3), ("tag", 4, 1, 1, 5.9, 6.1), ("tag", 8, 1, 0, 1.9, 3.9), ("tag", 8, 1, 0, 3.9, 4.2),
           ("spread", 3, 1, 0, 5.9, 7.9), ("spread", 3, 1, 0, 7.9, 8.2), ("spread", 10, 0, 0, 1.0, 2.0)]
CASES = [("tag",) + c for c in TAG_RUNS] + [("spread",) + c for c in SPREAD_RUNS] + [c[:4] + (0,) + c[4:] for c in ONE_RUN]


@pytest.mark.parametrize("scenario,agents,wd,ac,run_envs,low,high", CASES)
def test_both_sides_of_a_line_agree(scenario, agents, wd, ac, run_envs, low, high):
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tag = scenario == "tag"
    print(scenario, agents, wd, ac, run_envs, low, high, flush=True)
    D = synth.tag_obs_dim(*TAG[agents]) if tag else 6 * agents
    sizes = [(max(2, int(b * 16 * cus) // run_envs), run_envs) if run_envs else (1, int(b * 16 * cus) - 3) for b in (low, high)]
    most = max(runs for runs, _ in sizes)
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    policy, critic = dev(synth.policy_weights_with_bias(3, most, D, 64)), dev(synth.critic_weights(3, most, D, 64))

    def outputs(runs, E):
        if tag:
            cfg = synth.tag_config(E, *TAG[agents], runs, 64, wd, max_episode_steps=5)
        else:
            cfg = synth.spread_config(E, agents, runs, 64, wd, max_episode_steps=5, reward_mode=run_envs // 16 % 2)
        env = MpeEnv(MpeConfig(**cfg))
        env.set_policy(*[w[:runs].contiguous() for w in policy])
        env.reset(11)
        if ac:
            env.set_critic(*[w[:runs].contiguous() for w in critic])
            out = env.rollout_ac(T, *env.empty_traj_ac(T))
        else:
            out = env.rollout(T, *env.empty_traj(T))
        state = env.get_state()[:4]
        env.close()
        return out, state

    (few_runs, few_envs), (many_runs, many_envs) = sizes
    assert few_runs * few_envs < many_runs * many_envs
    shared = few_runs * few_envs
    (a_out, a_state), (b_out, b_state) = outputs(few_runs, few_envs), outputs(many_runs, many_envs)
    per_step = 6 if ac else 4                       # outputs [T][envs]...; the rest are [envs]...
    for k, (a, b) in enumerate(zip(a_out, b_out)):
        assert torch.equal(a, b[:, :shared] if k < per_step else b[:shared]), ("output", k)
    for k, (a, b) in enumerate(zip(a_state, b_state)):
        assert torch.equal(a, b[..., :shared]), ("state", k)
    del a_out, b_out
    torch.cuda.empty_cache()
