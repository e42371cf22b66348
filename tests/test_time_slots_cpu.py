"""Which rollouts run in slots of time (mpe_slots.h), from recorded launches: the blocks of all slots, eight XCDs at a time; and what the
blocks and the slots cover (mpe_slot_map.h), by counting."""
import os
import subprocess

import pytest

from tests.launch_record import ROOT, build_recorder, launches, record
from tests.time_slots import RUNS, Batch, batches, record_commands


def test_blocks_and_slots_cover_everything_once(tmp_path):
    exe = str(tmp_path / "slot_map")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-o", exe, os.path.join(ROOT, "tests", "slot_map.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "slots ok\n", r.stdout


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return build_recorder(tmp_path_factory.mktemp("recorder"))


@pytest.mark.parametrize("T", [6400, 6425, 1 << 17, 1 << 20, 1 << 24])
def test_slots_are_few(recorder, T):
    """A block walks over the slots before its own: no more than 256 of them, of longer spans where a rollout holds more episodes."""
    _, grid = blocks(recorder, "0 3 3 0 64 1", T)
    span = 25 * -(-(T // 257 + 1) // 25)
    assert grid == padded(4 * (T // span)) and T // span <= 256


def blocks(recorder, shape, T, call="rollout", policy=()):
    out = record(recorder, ["create " + shape, *policy, "reset", "%s %d" % (call, T)])
    (name, grid), = launches(out[-1][1])
    return name.split("<")[0], grid


def padded(n):
    return (n + 7) // 8 * 8


@pytest.mark.parametrize("shape,T,kernel,groups,slots", [
    ("0 3 3 0 1000 1", 128, "rollout_agents_kernel", 50, 5),              # 20 envs to a block; 28 + 4 x 25 steps
    ("0 3 3 0 1000 1", 74, "rollout_agents_kernel", 50, 2),
    ("0 3 3 0 1000 1", 49, "rollout_agents_kernel", 50, 1),               # no two episodes
    ("0 3 3 0 1000 8", 128, "rollout_uniform_ws_kernel", 125, 5),         # runs side by side are one batch
    ("0 3 3 0 16384 1", 128, "rollout_uniform_ws_kernel", 256, 2),        # near the rate of the writes: two
    ("0 3 3 0 65536 1", 128, "rollout_uniform_ws_kernel", 1024, 1),
    ("0 1 1 0 32768 1", 100, "rollout_uniform_ws_kernel", 512, 4),
    ("0 10 10 0 1000 1", 128, "rollout_agents_kernel", 167, 5),
    ("1 4 2 3 1000 1", 2048, "rollout_agents_kernel", 63, 81),
])
def test_environment_only(recorder, shape, T, kernel, groups, slots):
    assert blocks(recorder, shape, T) == (kernel, padded(groups * slots))


def spread(n):
    return (n + 31) // 32 * 32


@pytest.mark.parametrize("shape,T,call,kernel,grid", [
    ("0 3 3 0 64 1", 128, "rollout", "rollout_gru_kernel", padded(13 * 5)),               # 5-env blocks, one slot each
    ("0 3 3 0 64 1", 49, "rollout", "rollout_gru_kernel", padded(13)),                    # no two episodes
    ("0 3 3 0 1000 1", 128, "rollout_ac", "rollout_gru_kernel", padded(48 * 5)),          # 21 envs
    ("0 3 3 0 16 12", 128, "rollout", "rollout_gru_kernel", padded(12 * 5)),              # runs: blocks inside one
    ("0 3 3 0 4096 1", 128, "rollout", "rollout_gru_waves_kernel", spread(256)),          # wavefronts with lanes of several slots
    ("0 3 3 0 12000 1", 128, "rollout_ac", "rollout_gru_waves_kernel", spread(750)),
    ("0 10 10 0 3000 1", 64, "rollout", "rollout_gru_waves_kernel", spread(250)),
    ("0 3 3 0 20480 1", 128, "rollout_ac", "rollout_gru_waves_kernel", 256),              # a whole round in one slot
])
def test_recurrent_policies(recorder, shape, T, call, kernel, grid):
    assert blocks(recorder, shape, T, call, ("gru", "critic")) == (kernel, grid)


def test_set_state_clears_the_tickets(recorder):
    """With and without a reset before: one that a capture has recorded has not run."""
    for first in ([], ["reset"]):
        out = record(recorder, ["create 0 3 3 0 1000 1", *first, "set_state"])
        assert [name for name, _ in launches(out[-1][1])] == ["read_counters_kernel"]


@pytest.mark.parametrize("shape,T,call,policy,alike,unlike", [
    # in a block kernel, whose blocks have slots only where their envs' counters are alike
    ("0 3 3 0 1000 1 0 0 25", 128, "rollout", (), "rollout_agents_kernel", "rollout_agents_kernel"),
    ("0 3 3 0 4800 1 0 0 25", 128, "rollout", (), "rollout_uniform_ws_kernel", "rollout_agents_kernel"),
    ("0 1 1 0 4800 1 0 0 25", 128, "rollout", (), "rollout_uniform_ws_kernel", "rollout_uniform_ws_kernel"),
    ("1 4 2 3 1000 1 0 0 25", 128, "rollout", (), "rollout_agents_kernel", "rollout_agents_kernel"),
    ("0 6 6 0 256 1 64 0 25", 50, "rollout", ("mlp",), "rollout_small_kernel", "rollout_small_kernel"),
    ("1 8 2 6 200 1 64 0 25", 50, "rollout_ac", ("mlp", "mlp_critic"), "rollout_small_kernel", "rollout_small_kernel"),
    ("0 3 3 0 1000 1 128 1 25", 128, "rollout", ("gru",), "rollout_gru_kernel", "rollout_gru_kernel"),
    ("0 3 3 0 16 12 128 1 25", 128, "rollout_ac", ("gru", "critic"), "rollout_gru_kernel", "rollout_gru_kernel"),
])
def test_unlike_counters_in_blocks(recorder, shape, T, call, policy, alike, unlike):
    """They run in one slot, as after no other call than mpe_set_state."""
    def route(*before):
        (name, _), = launches(record(recorder, ["create " + shape, *policy, *before, "%s %d" % (call, T)])[-1][1])
        return name
    several, fresh = route("reset"), route("counters 0", "set_state")
    assert several == fresh and several.startswith(alike) and ("SlotGrid" in several or several.endswith("true>"))
    one = route("counters 7", "set_state")
    assert one.startswith(unlike) and "SlotGrid" not in one and (not one.startswith("rollout_uniform_ws") or one.endswith("false>"))
    assert route("counters 7", "set_state", "reset") == several and route("counters 7", "set_state", "counters 0", "set_state") == several
    # what was found last holds until the next state's kernel has run
    assert route("counters 7", "set_state", "rollout 1") == one


def test_unlike_counters_in_wavefronts(recorder):
    """Lanes have a slot of their own: slots as ever, also of smaller batches, whose blocks can have none."""
    for envs, alike in ((20011, "rollout_waves_kernel"), (1000, "rollout_small_kernel")):
        for unit, kernel in ((0, alike), (7, "rollout_waves_kernel"), (48, alike)):
            out = record(recorder, ["create 0 3 3 0 %d 1 64 0 25" % envs, "mlp", "counters %d" % unit, "set_state", "rollout 128"])
            (name, _), = launches(out[-1][1])
            assert name.startswith(kernel) and "SlotGrid" in name, (envs, unit, name)


@pytest.mark.parametrize("shape,T", [("0 3 3 0 48 450 64 0 25", 86), ("0 3 3 0 48 200 64 1 25", 86)])
def test_runs_that_one_slot_suits_better(recorder, shape, T):
    """Actor-critic, 8 to 9 % slower in slots, whose long blocks share their compute units."""
    (name, _), = launches(record(recorder, ["create " + shape, "mlp", "mlp_critic", "reset", "rollout_ac %d" % T])[-1][1])
    assert name.startswith("rollout_small_kernel") and "SlotGrid" not in name


def single_launches(recorder, cases):
    """The kernel that each batch's rollout launches."""
    commands = [record_commands(b) for b in cases]
    out, names = record(recorder, [c for cs in commands for c in cs]), []
    for cs in commands:
        (name, _), = launches(out[len(cs) - 2][1])
        names.append(name)
        out = out[len(cs):]
    return names


def test_every_instance_with_slots_has_its_batch(recorder):
    """The GPU test of all instances runs these: each in the instance that it is listed for, and no instance without one."""
    cases = list(batches())
    assert single_launches(recorder, cases) == [b.kernel for b in cases]
    (_, lines), = record(recorder, ["kernels"])
    instances = {k[len("kernel "):] for k in lines if "SlotGrid" in k or (k.startswith("kernel rollout_uniform_ws_kernel<") and k.endswith("true>"))}
    assert {b.kernel for b in cases} == instances and len(instances) > 400


def test_runs_of_the_gpu_test_share_wavefronts(recorder):
    cases = [Batch("spread", agents, 0, "mlp", ac, envs, runs, 25, 128, 0, "") for runs, envs, agents, ac in RUNS]
    for b, name in zip(cases, single_launches(recorder, cases)):
        assert name.startswith("rollout_waves_kernel<WaveSpread<%d>" % b.agents) and "SlotGrid" in name, b
