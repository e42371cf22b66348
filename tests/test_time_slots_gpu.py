"""Rollouts in slots of time: see tests/time_slots.py.  Steps: two slots, some (with a remainder), many; sizes: one env, partly
filled last groups, several blocks."""
import pytest

pytestmark = pytest.mark.gpu

EPISODES = [(25, 50), (25, 128), (5, 101), (1, 64), (40, 81)]        # steps of an episode, of a rollout


@pytest.mark.parametrize("kind", ["alike", "stretches", "own"])
@pytest.mark.parametrize("max_ep,T", EPISODES)
@pytest.mark.parametrize("scenario,agents,envs", [("spread", 1, 1), ("spread", 1, 1027), ("spread", 2, 512), ("spread", 3, 65),
                                                  ("spread", 3, 1024), ("spread", 3, 6000), ("spread", 4, 1001), ("spread", 10, 130),
                                                  ("tag", 2, 77), ("tag", 3, 1003), ("tag", 4, 1500), ("tag", 10, 100)])
def test_environment_only(scenario, agents, envs, max_ep, T, kind):
    from tests.time_slots import assert_slots_change_nothing, config
    assert_slots_change_nothing(config(scenario, agents, envs, max_ep), T, kind, max_ep)


@pytest.mark.parametrize("scenario,agents", [("spread", 2), ("spread", 3), ("spread", 6), ("tag", 4)])
@pytest.mark.parametrize("left_out", [(0, 4), (1, 2), (3,), (0, 1, 2, 3)])
def test_environment_only_without_some_outputs(scenario, agents, left_out):
    from tests.time_slots import assert_slots_change_nothing, config
    assert_slots_change_nothing(config(scenario, agents, 200, 25), 77, "alike", 25, left_out=left_out)


# (scenario, agents, bf16) x (envs, runs, steps of an episode, of a rollout): blocks of the small-batch kernel with operands in
# registers and in LDS, partly filled; wavefronts in blocks of 4, 8 and 12 with lanes of several slots, ends of runs inside one
SHAPES = [("spread", 1, 0), ("spread", 1, 1), ("spread", 2, 0), ("spread", 2, 1), ("spread", 3, 0), ("spread", 3, 1), ("spread", 4, 0),
          ("spread", 6, 0), ("spread", 8, 0), ("spread", 10, 0), ("tag", 2, 0), ("tag", 3, 1), ("tag", 4, 0), ("tag", 6, 0), ("tag", 8, 1), ("tag", 10, 0)]
SIZES = [(1, 1, 25, 77), (67, 1, 5, 101), (1003, 1, 25, 128), (16, 24, 25, 128), (48, 7, 25, 110)]
LARGE = [("spread", 1, 0, 9001), ("spread", 2, 1, 7001), ("spread", 3, 0, 5001), ("spread", 3, 0, 8200), ("spread", 3, 0, 11000), ("spread", 3, 1, 9003),
         ("spread", 5, 0, 4099), ("spread", 7, 0, 2500), ("spread", 8, 0, 4100), ("spread", 9, 0, 2300), ("spread", 10, 0, 3400), ("tag", 2, 1, 9005),
         ("tag", 3, 0, 8001), ("tag", 4, 0, 7003), ("tag", 5, 1, 2501), ("tag", 6, 0, 3999), ("tag", 8, 0, 3001), ("tag", 10, 1, 3333)]


def networks(scenario, agents, runs, ac):
    import torch
    from paper_2311_10090_amd import synth
    from tests.time_slots import config
    c = config(scenario, agents, 16, 25)
    D = synth.tag_obs_dim(agents, c["num_landmarks"], c["num_adversaries"]) if scenario == "tag" else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    return dict(policy=dev(synth.policy_weights_with_bias(3, runs, D, 64)), critic=dev(synth.critic_weights(3, runs, D, 64)) if ac else ())


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("envs,runs,max_ep,T", SIZES)
@pytest.mark.parametrize("scenario,agents,wd", SHAPES)
def test_policies(scenario, agents, wd, envs, runs, max_ep, T, ac):
    from tests.time_slots import assert_slots_change_nothing, config
    if runs > 1 and scenario == "spread" and agents > 3:
        envs = 64
    cfg = config(scenario, agents, envs, max_ep, runs, 64, wd)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, T, kind, max_ep, **networks(scenario, agents, runs, ac))


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,wd,envs", LARGE)
def test_policies_in_wavefronts(scenario, agents, wd, envs, ac):
    from tests.time_slots import assert_slots_change_nothing, config
    cfg = config(scenario, agents, envs, 25, 1, 64, wd)
    for kind in ("stretches", "own"):
        assert_slots_change_nothing(cfg, 128, kind, 25, **networks(scenario, agents, 1, ac))


@pytest.mark.parametrize("runs,envs", [(1024, 16), (300, 32), (77, 48), (100, 64)])
@pytest.mark.parametrize("agents,ac", [(3, False), (3, True), (2, True)])
def test_runs_in_wavefronts(agents, runs, envs, ac):
    from tests.time_slots import assert_slots_change_nothing, config
    cfg = config("spread", agents, envs, 25, runs, 64, 0)
    assert_slots_change_nothing(cfg, 128, "own", 25, **networks("spread", agents, runs, ac))


@pytest.mark.parametrize("left_out", [(0, 6), (1, 2, 7), (3, 4), (5, 6, 7)])
@pytest.mark.parametrize("envs", [500, 6000])
def test_actor_critic_without_some_outputs(envs, left_out):
    from tests.time_slots import assert_slots_change_nothing, config
    assert_slots_change_nothing(config("spread", 3, envs, 25, 1, 64, 0), 128, "alike", 25, left_out=left_out, **networks("spread", 3, 1, True))


# recurrent policy: blocks of every number of row tiles (spare rows too), partly filled; runs; wavefronts whose first rows are the end
# of a slot and whose last ones the start of the next.  Counters of its own also leave envs that run all steps in slot 0.
RECURRENT = [("spread", 1, 1, 1), ("spread", 1, 5000, 1), ("spread", 2, 903, 1), ("spread", 3, 3, 1), ("spread", 3, 251, 1), ("spread", 3, 509, 1),
             ("spread", 3, 1030, 1), ("spread", 3, 1500, 1), ("spread", 3, 3100, 1), ("spread", 3, 6007, 1), ("spread", 3, 16, 12), ("spread", 3, 32, 90),
             ("spread", 3, 64, 60), ("spread", 4, 2501, 1), ("spread", 6, 333, 1), ("spread", 6, 2222, 1), ("spread", 10, 130, 1),
             ("spread", 10, 1601, 1), ("tag", 2, 1003, 1), ("tag", 3, 4001, 1), ("tag", 4, 200, 1), ("tag", 4, 16, 33), ("tag", 6, 1999, 1),
             ("tag", 8, 777, 1), ("tag", 10, 601, 1)]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("max_ep,T", [(25, 128), (5, 75), (40, 81)])
@pytest.mark.parametrize("scenario,agents,envs,runs", RECURRENT)
def test_recurrent_policies(scenario, agents, envs, runs, max_ep, T, ac):
    import torch
    from paper_2311_10090_amd import synth
    from tests.time_slots import assert_slots_change_nothing, config
    cfg = config(scenario, agents, envs, max_ep, runs, synth.GRU_HIDDEN, 1)
    D = synth.tag_obs_dim(agents, cfg["num_landmarks"], cfg["num_adversaries"]) if scenario == "tag" else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    nets = dict(policy=dev(synth.gru_weights(5, runs, D)), critic=dev(synth.gru_critic_weights(5, runs)) if ac else (), gru=True)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, T, kind, max_ep, **nets)
    if envs == 6007 or envs == 509:
        assert_slots_change_nothing(cfg, T, "stretches", max_ep, left_out=(0, 4) if not ac else (0, 1, 5, 7), **nets)
