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
