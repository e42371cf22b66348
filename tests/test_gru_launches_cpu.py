"""Launches of the recurrent rollout, recorded without a device: a call that the runtime refuses leaves the handle as it was or
makes it ask for a new state, and between them the kernels of a batch cover each of its envs once."""
import re

import pytest

from paper_2311_10090_amd.binding import MPE_EHIP, MPE_ESTATE, MPE_OK
from tests.gru_batches import SHAPES, batches, whole_rounds
from tests.launch_record import build_recorder, launches, record

SPLIT = ["0 3 3 0 65536 1", "0 6 6 0 10500 1", "0 10 10 0 6300 1", "1 4 2 3 20500 1"]    # independent wavefronts, then blocks


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return build_recorder(tmp_path_factory.mktemp("recorder"))


def _setup(shape):
    return ["create " + shape, "gru", "critic", "reset"]


@pytest.mark.parametrize("call", ["rollout 4", "rollout_ac 4"])
@pytest.mark.parametrize("shape", SPLIT)
def test_refused_preparation_launches_nothing(recorder, shape, call):
    for k in (1, 2):                                       # either kernel's LDS
        *_, (rc, lines), (_, step), (again, then) = record(recorder, _setup(shape) + ["fail attribute %d" % k, call, "abs_step", call])
        assert rc == MPE_EHIP and not launches(lines) and "FAILS" in lines[-1]
        assert step == ["abs_step 0"] and again == MPE_OK and len(launches(then)) == 2


@pytest.mark.parametrize("call", ["rollout 4", "rollout_ac 4"])
@pytest.mark.parametrize("shape", SPLIT)
def test_refused_launch(recorder, shape, call):
    # the first of the two: nothing has run
    *_, (rc, _), (again, then) = record(recorder, _setup(shape) + ["fail launch 1", call, call])
    assert rc == MPE_EHIP and again == MPE_OK and len(launches(then)) == 2
    # the second: part of the batch has been stepped
    rcs = [rc for rc, _ in record(recorder, _setup(shape) + ["fail launch 2", call, call, "reset", call])]
    assert rcs[-4:] == [MPE_EHIP, MPE_ESTATE, MPE_OK, MPE_OK]
    rcs = [rc for rc, _ in record(recorder, _setup(shape) + ["fail launch 2", call, "set_state", call])]
    assert rcs[-3:] == [MPE_EHIP, MPE_OK, MPE_OK]


# envs per block of the second template argument, the scenario's agents before it
BLOCK = re.compile(r"launch rollout_gru_kernel<Gru(?:Spread|Tag)<(\d+)[^>]*>, (\d+), .* first (\d+) groups (\d+)$")
WAVES = re.compile(r"launch rollout_gru_waves_kernel<.* envs (\d+)$")


@pytest.mark.parametrize("call", ["rollout 4", "rollout_ac 4"])
@pytest.mark.parametrize("units", [256, 80, 27])
def test_kernels_cover_the_batch(recorder, units, call):
    shapes = [(0, n, n, 0) for n in range(1, 11)] + [(1, 4, 2, 3), (1, 10, 3, 8)]
    sizes = sorted({max(1, int(units * x) + d) for x in (0.01, 1, 2, 5, 10, 15.5, 21, 32, 40, 64, 80, 100, 130, 256, 300, 400) for d in (-1, 0, 1)})
    cases = [(s, e) for s in shapes for e in sizes]
    commands = [c for s, e in cases for c in ["create %d %d %d %d" % s + " %d 1" % e, "gru", "critic", "reset", call, "destroy"]]
    out = record(recorder, commands, units)
    for (shape, envs), (rc, lines) in zip(cases, out[4::6]):
        assert rc == MPE_OK
        done = 0
        for line in (x for x in lines if x.startswith("launch ")):
            waves, block = WAVES.match(line), BLOCK.match(line)
            if waves:
                assert done == 0
                done = int(waves[1])
            else:
                agents, eb, first, groups = (int(v) for v in block.groups())
                assert done == (first if agents * eb % 16 else first * eb), (shape, envs, line)      # spare rows: counted in envs
                assert done + (groups - 1) * eb < envs <= done + groups * eb
                done = envs
        assert done == envs, (shape, envs, lines)


def test_batches_between_blocks_and_wavefronts_with_a_critic(recorder):
    """Where a round of blocks costs about a round of independent wavefronts: 9 agents, blocks while at most two thirds of the
    compute units have one; 10 agents, wavefronts from the first batch on that small blocks leave."""
    def kernel(agents, envs):
        out = record(recorder, ["create 0 %d %d 0 %d 1" % (agents, agents, envs), "gru", "critic", "reset", "rollout_ac 4"])
        return [name.split("<")[0] for name, _ in launches(out[-1][1])]
    for agents, envs, waves in ((8, 2000, False), (8, 4000, False), (9, 1800, False), (9, 2400, False), (9, 3000, True), (9, 4096, True),
                                (10, 1600, True), (10, 4096, True)):
        assert kernel(agents, envs) == ["rollout_gru_waves_kernel" if waves else "rollout_gru_kernel"], (agents, envs)


@pytest.mark.parametrize("shape", ["0 3 3 0 256 1", "0 6 6 0 6000 1", "0 10 10 0 2000 1", "0 3 3 0 65536 1", "1 4 2 3 20500 1", "0 3 3 0 64 8"])
def test_weights_are_packed_in_one_launch(recorder, shape):
    """Also where a batch may run in both kernels, which read images of their own."""
    out = record(recorder, _setup(shape) + ["gru", "critic"])
    assert [name for name, _ in launches(out[4][1])] == ["pack_gru_kernel"]
    assert [name for name, _ in launches(out[5][1])] == ["pack_gru_critic_kernel"]


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
def test_batches_of_the_gpu_tests_reach_their_kernels(recorder, ac):
    cases = [(s, kernels, envs) for s in SHAPES for kernels, envs in batches(*s, ac) + [("waves", whole_rounds(s[1]))]]
    out = record(recorder, [c for s, _, envs in cases for c in ["create %d %d %d %d" % (s[0] == "tag", *s[1:]) + " %d 1" % envs, "gru", "critic",
                                                               "reset", "rollout_ac 1" if ac else "rollout 1", "destroy"]])
    for (shape, kernels, envs), (rc, lines) in zip(cases, out[4::6]):
        found = []
        for line in (x for x in lines if x.startswith("launch ")):
            block = BLOCK.match(line)
            found.append("blocks" + block[2] if block else "waves")
        assert rc == MPE_OK and "+".join(found) == kernels, (shape, envs)
