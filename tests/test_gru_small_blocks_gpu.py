"""The recurrent rollout in blocks of one, two and four row tiles, whose last rows may belong to no env, alone and behind a round of
independent wavefronts, against two whole rounds of those, bit for bit over all envs.  The last block is partly filled, but in
blocks of one env (tests/test_gru_launches_cpu.py checks which kernels a batch reaches)."""
import pytest

from tests.gru_batches import SHAPES, assert_same, batches, outputs_of, small_blocks, whole_rounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries", [s for s in SHAPES if s[1] > 1])
def test_small_blocks_agree_with_wavefronts(scenario, agents, landmarks, adversaries, ac):
    outputs = outputs_of(scenario, agents, landmarks, adversaries, ac)
    whole = outputs(whole_rounds(agents))
    for kernels, envs in batches(scenario, agents, landmarks, adversaries, ac):
        if small_blocks(kernels):
            assert_same(outputs, envs, whole)
