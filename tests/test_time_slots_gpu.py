"""Rollouts in slots of time: see tests/time_slots.py.  Steps: two slots, some (with a remainder), many; sizes: one env, partly
filled last groups, several blocks."""
import pytest

from tests.time_slots import RUNS, assert_slots_change_nothing, batches, config, networks

pytestmark = pytest.mark.gpu

EPISODES = [(25, 50), (25, 128), (5, 101), (1, 64), (40, 81)]        # steps of an episode, of a rollout


@pytest.mark.parametrize("kind", ["alike", "stretches", "own"])
@pytest.mark.parametrize("max_ep,T", EPISODES)
@pytest.mark.parametrize("scenario,agents,envs", [("spread", 1, 1), ("spread", 1, 1027), ("spread", 2, 512), ("spread", 3, 65),
                                                  ("spread", 3, 1024), ("spread", 3, 6000), ("spread", 4, 1001), ("spread", 10, 130),
                                                  ("tag", 2, 77), ("tag", 3, 1003), ("tag", 4, 1500), ("tag", 10, 100)])
def test_environment_only(scenario, agents, envs, max_ep, T, kind):
    assert_slots_change_nothing(config(scenario, agents, envs, max_ep), T, kind, max_ep)


@pytest.mark.parametrize("scenario,agents", [("spread", 2), ("spread", 3), ("spread", 6), ("tag", 4)])
@pytest.mark.parametrize("left_out", [(0, 4), (1, 2), (3,), (0, 1, 2, 3)])
def test_environment_only_without_some_outputs(scenario, agents, left_out):
    assert_slots_change_nothing(config(scenario, agents, 200, 25), 77, "alike", 25, left_out=left_out)


# (scenario, agents, bf16) x (envs, runs, steps of an episode, of a rollout): blocks of the small-batch kernel with operands in
# registers and in LDS, partly filled; wavefronts in blocks of 4, 8 and 12 with lanes of several slots, ends of runs inside one
SHAPES = [("spread", 1, 0), ("spread", 1, 1), ("spread", 2, 0), ("spread", 2, 1), ("spread", 3, 0), ("spread", 3, 1), ("spread", 4, 0),
          ("spread", 6, 0), ("spread", 8, 0), ("spread", 10, 0), ("tag", 2, 0), ("tag", 3, 1), ("tag", 4, 0), ("tag", 6, 0), ("tag", 8, 1), ("tag", 10, 0)]
SIZES = [(1, 1, 25, 77), (67, 1, 5, 101), (1003, 1, 25, 128), (16, 24, 25, 128), (48, 7, 25, 110)]
LARGE = [("spread", 1, 0, 9001), ("spread", 2, 1, 7001), ("spread", 3, 0, 5001), ("spread", 3, 0, 8200), ("spread", 3, 0, 11000), ("spread", 3, 1, 9003),
         ("spread", 5, 0, 4099), ("spread", 7, 0, 2500), ("spread", 8, 0, 4100), ("spread", 9, 0, 2300), ("spread", 10, 0, 3400), ("tag", 2, 1, 9005),
         ("tag", 3, 0, 8001), ("tag", 4, 0, 7003), ("tag", 5, 1, 2501), ("tag", 6, 0, 3999), ("tag", 8, 0, 3001), ("tag", 10, 1, 3333)]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("envs,runs,max_ep,T", SIZES)
@pytest.mark.parametrize("scenario,agents,wd", SHAPES)
def test_policies(scenario, agents, wd, envs, runs, max_ep, T, ac):
    if runs > 1 and scenario == "spread" and agents > 3:
        envs = 64
    cfg = config(scenario, agents, envs, max_ep, runs, 64, wd)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, T, kind, max_ep, **networks(scenario, agents, runs, ac))


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,wd,envs", LARGE)
def test_larger_batches(scenario, agents, wd, envs, ac):
    cfg = config(scenario, agents, envs, 25, 1, 64, wd)
    for kind in ("stretches", "own"):
        assert_slots_change_nothing(cfg, 128, kind, 25, **networks(scenario, agents, 1, ac))


@pytest.mark.parametrize("runs,envs,agents,ac", RUNS)
def test_runs_in_wavefronts(agents, runs, envs, ac):
    cfg = config("spread", agents, envs, 25, runs, 64, 0)
    assert_slots_change_nothing(cfg, 128, "own", 25, **networks("spread", agents, runs, ac))


@pytest.mark.parametrize("left_out", [(0, 6), (1, 2, 7), (3, 4), (5, 6, 7)])
@pytest.mark.parametrize("envs", [500, 6000])
def test_actor_critic_without_some_outputs(envs, left_out):
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
    cfg = config(scenario, agents, envs, max_ep, runs, 128, 1)
    nets = networks(scenario, agents, runs, ac, gru=True)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, T, kind, max_ep, **nets)
    if envs == 6007 or envs == 509:
        assert_slots_change_nothing(cfg, T, "stretches", max_ep, left_out=(0, 4) if not ac else (0, 1, 5, 7), **nets)


@pytest.mark.parametrize("batch", batches(), ids=lambda b: b.kernel.replace(" ", ""))
def test_every_instance(batch):
    """tests/test_time_slots_cpu.py: that the batch runs in this instance, and that none is missing."""
    b = batch
    nets = networks(b.scenario, b.agents, b.runs, b.critic, b.policy == "gru") if b.policy != "none" else {}
    cfg = config(b.scenario, b.agents, b.envs, b.max_ep, b.runs, {"none": 0, "mlp": 64, "gru": 128}[b.policy], b.wd, b.reward)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, b.T, kind, b.max_ep, **nets)


@pytest.mark.parametrize("reward", [0, 1], ids=["shared", "mixed"])
@pytest.mark.parametrize("agents", [1, 2, 3, 6])
@pytest.mark.parametrize("policy,envs", [("none", 200), ("none", 8192), ("mlp", 500), ("mlp", 20011), ("gru", 300), ("gru", 6007)])
def test_both_rewards(policy, envs, agents, reward):
    nets = networks("spread", agents, 1, False, policy == "gru") if policy != "none" else {}
    cfg = config("spread", agents, envs, 25, 1, {"none": 0, "mlp": 64, "gru": 128}[policy], int(policy == "gru"), reward)
    for kind in ("alike", "own"):
        assert_slots_change_nothing(cfg, 110, kind, 25, **nets)
