"""The recurrent rollout in blocks of one, two and four row tiles, whose last rows may belong to no env, against blocks of 16
envs, bit for bit.  What an env does depends on (seed, run, env) only, so batches agree on the envs they share; each batch is the
largest of its block size less one env: the last block is partly filled.  State carried over two rollouts, episodes of 5
steps, outputs left out in the second rollout of half the shapes."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [("spread", n, n, 0) for n in range(2, 11)] + [("tag", *s) for s in ((4, 2, 3), (2, 1, 1), (3, 0, 2), (6, 2, 4), (5, 2, 4), (8, 2, 6), (10, 3, 8))]


def _outputs(scenario, agents, landmarks, adversaries, ac):
    """outputs(E): everything two rollouts of a batch of E envs write, the env axis first."""
    import torch
    from paper_2311_10090_amd import synth
    from paper_2311_10090_amd.binding import MpeConfig, MpeEnv
    T, H = 7, synth.GRU_HIDDEN
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
        for k in range(2):
            bufs = list(env.empty_traj_ac(T) if ac else env.empty_traj(T))
            if k and agents % 2:
                bufs[0] = bufs[2] = bufs[-1] = None
            out = env.rollout_ac(T, *bufs) if ac else env.rollout(T, *bufs)
            kept += [(o.transpose(0, 1) if o.shape[0] == T else o).clone() for o in out if o is not None]
        kept += [s.movedim(-1, 0).clone() for s in env.get_state()[:4]]
        kept.append(env.get_hidden().reshape(E, -1).clone())
        env.close()
        return kept

    print("recurrent %s, %d agents, %s" % (scenario, agents, "actor-critic" if ac else "plain"), flush=True)
    return outputs


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries", SHAPES)
def test_small_blocks_agree_with_blocks_of_16_envs(scenario, agents, landmarks, adversaries, ac):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    outputs = _outputs(scenario, agents, landmarks, adversaries, ac)
    full = outputs(16 * cus)
    for block in sorted({16 * tiles // agents for tiles in (1, 2, 4)}):
        E = max(block * cus - 1, 1)
        if block == 16 or block > 21:
            continue
        keep = min(E, 16 * cus)
        for k, (a, b) in enumerate(zip(outputs(E), full)):
            assert torch.equal(a[:keep], b[:keep]), ("output", k, E)


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("agents", [2, 3, 6, 10])
def test_small_blocks_behind_a_round_of_independent_wavefronts(agents, ac):
    """A whole round of independent wavefronts and a remainder in blocks of one tile, against two whole rounds."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    outputs = _outputs("spread", agents, agents, 0, ac)
    turn = cus * 8 * (32 // agents)
    E = turn + cus * (16 // agents) - 1
    for k, (a, b) in enumerate(zip(outputs(E), outputs(2 * turn))):
        assert torch.equal(a, b[:E]), ("output", k)
