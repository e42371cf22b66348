"""The recurrent rollout's kernels against each other, bit for bit over all envs of each batch: blocks of 16, 32 and 64 envs
(mpe_policy_gru.hip) alone and behind independent wavefronts, and a batch of wavefronts whose last one is partly filled, against two
whole rounds of independent wavefronts (mpe_gru_waves.hip).  tests/test_gru_launches_cpu.py checks which kernels a batch reaches."""
import pytest

from tests.gru_batches import SHAPES, assert_same, batches, outputs_of, small_blocks, whole_rounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ac", [False, True], ids=["plain", "actor_critic"])
@pytest.mark.parametrize("scenario,agents,landmarks,adversaries", SHAPES)
def test_blocks_agree_with_wavefronts(scenario, agents, landmarks, adversaries, ac):
    outputs = outputs_of(scenario, agents, landmarks, adversaries, ac)
    whole = outputs(whole_rounds(agents))
    for kernels, envs in batches(scenario, agents, landmarks, adversaries, ac):
        if not small_blocks(kernels):
            assert_same(outputs, envs, whole)
