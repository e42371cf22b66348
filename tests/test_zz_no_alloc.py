"""mpe_rollout_noalloc -- the entry point for callers that cannot allocate device memory -- against the
handle-based calls it stands for (mpe_create + mpe_reset + mpe_set_policy + mpe_rollout): every output bit
for bit, on two calls in a row of which the second is the smaller one (the static scratch array keeps the
first call's contents), plus the refusals.  Through the C ABI."""
import numpy as np
import pytest

from tests import helpers as Hp
from paper_2311_10090_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _reference(cfg, seed, weights, T):
    from paper_2311_10090_amd.binding import MpeEnv
    env = MpeEnv(cfg)
    if weights is not None:
        env.set_policy(*weights)
    env.reset(seed)
    out = env.rollout(T, *env.empty_traj(T))
    torch.cuda.synchronize()
    bufs = env.empty_traj(T)
    env.close()
    return out, bufs


def _call(cfg, seed, weights, T, bufs):
    from paper_2311_10090_amd.binding import rollout_noalloc
    for b in bufs:
        b.view(torch.uint8).fill_(0xA5)      # whatever the call does not write stays visible
    out = rollout_noalloc(cfg, seed, weights, T, *bufs)
    torch.cuda.synchronize()
    return out


# (first call, second smaller call): (envs, agents, runs, hidden, weight dtype, T)
PAIRS = [
    ((65536, 3, 1, 64, 0, 30), (4096, 3, 1, 64, 0, 30)),      # headline launch (256-env blocks), then 32-env blocks
    ((4096, 3, 1, 64, 0, 40), (100, 2, 1, 64, 0, 26)),        # fewer agents, ragged size
    ((64, 3, 64, 64, 0, 27), (16, 3, 8, 64, 0, 27)),          # one set of weights per run
    ((2048, 10, 1, 128, 1, 26), (70, 4, 1, 64, 1, 26)),       # lane-per-agent bf16 kernel, two shapes
    ((8192, 3, 1, 0, 0, 50), (130, 3, 1, 0, 0, 50)),          # no policy: seeded uniform actions
    ((300, 5, 1, 0, 0, 30), (64, 1, 1, 64, 1, 30)),           # uniform actions, then a bf16 policy
    ((1024, 6, 1, 64, 0, 26), (100, 4, 1, 64, 0, 26)),        # fp32 weights with 4 and more agents
    ((512, 10, 1, 64, 0, 26), (70, 8, 1, 64, 0, 26)),         # ... with layer 1 over two K slices
    ((107000, 3, 1, 64, 0, 60), (1000, 3, 1, 64, 0, 128)),    # no room for the tickets of slots of time, then room
    ((107000, 3, 1, 0, 0, 60), (1000, 3, 1, 0, 0, 128)),
]


@pytest.mark.parametrize("first,second", PAIRS)
def test_two_calls_in_a_row_match_the_handle_based_calls(first, second):
    for k, (E, N, R, H, wd, T) in enumerate((first, second)):
        cfg = Hp.gpu_config(E, N, R, H, wd)
        weights = Hp.to_dev(synth.policy_weights_with_bias(11 + k, R, 6 * N, H)) if H else None
        seed = 5 + k
        print("no-alloc call %d: E=%d N=%d R=%d H=%d dtype=%d T=%d" % (k, E, N, R, H, wd, T), flush=True)
        ref, bufs = _reference(cfg, seed, weights, T)
        got = _call(cfg, seed, weights, T, bufs)
        for name, a, b in zip(("obs", "act", "rew", "done", "last_obs"), got, ref):
            assert torch.equal(a, b), "%s differs (call %d)" % (name, k)


def test_mixed_reward_and_absent_outputs():
    from paper_2311_10090_amd.binding import rollout_noalloc
    E, N, T = 1000, 3, 30
    cfg = Hp.gpu_config(E, N, 1, 64, 0, reward_mode=1, local_ratio=0.3)
    weights = Hp.to_dev(synth.policy_weights_with_bias(3, 1, 6 * N, 64))
    ref, bufs = _reference(cfg, 9, weights, T)
    got = _call(cfg, 9, weights, T, bufs)
    assert got[2].shape == (T, E, N)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
    # only the rewards asked for
    rew = torch.empty_like(ref[2])
    rollout_noalloc(cfg, 9, weights, T, None, None, rew, None, None)
    torch.cuda.synchronize()
    assert torch.equal(rew, ref[2])


def test_refusals():
    from paper_2311_10090_amd.binding import rollout_noalloc, MpeError, MPE_EINVAL, MpeConfig
    from paper_2311_10090_amd.binding import load_library
    import ctypes as C
    lib = load_library()
    scratch_bytes = 8 << 20
    w = Hp.to_dev(synth.policy_weights(1, 1, 18, 64))
    # the state of 120,000 envs of 3 agents (76 bytes each) does not fit the 8 MiB array; 100,000 do
    with pytest.raises(MpeError) as ei:
        rollout_noalloc(Hp.gpu_config(120000, 3, 1, 64, 0), 1, w, 2)
    assert ei.value.code == MPE_EINVAL and b"scratch" in lib.mpe_last_error()
    assert 120000 * 76 > scratch_bytes > 100000 * 76
    rollout_noalloc(Hp.gpu_config(100000, 3, 1, 64, 0), 1, w, 2)
    for bad in (dict(T=0), dict(T=(1 << 24) + 1)):
        with pytest.raises(MpeError) as ei:
            rollout_noalloc(Hp.gpu_config(64, 3, 1, 64, 0), 1, w, bad["T"])
        assert ei.value.code == MPE_EINVAL
    with pytest.raises(MpeError) as ei:                      # only some of the six arrays
        rollout_noalloc(Hp.gpu_config(64, 3, 1, 64, 0), 1, w[:5] + [None], 2)
    assert ei.value.code == MPE_EINVAL
    with pytest.raises(MpeError) as ei:                      # a policy shape that mpe_set_policy refuses
        rollout_noalloc(Hp.gpu_config(64, 8, 1, 128, 0), 1, Hp.to_dev(synth.policy_weights(1, 1, 48, 128)), 2)
    assert ei.value.code == MPE_EINVAL
    with pytest.raises(MpeError) as ei:                      # the second scenario is not built here
        rollout_noalloc(Hp.tag_gpu_config(64), 1, None, 2)
    assert ei.value.code == MPE_EINVAL
    with pytest.raises(MpeError) as ei:                      # bad config
        rollout_noalloc(MpeConfig(num_envs=0), 1, None, 2)
    assert ei.value.code == MPE_EINVAL
    obs = torch.empty(64 * 3 * 18 + 1, dtype=torch.float32, device="cuda")[1:]   # misaligned output
    with pytest.raises(MpeError) as ei:
        rollout_noalloc(Hp.gpu_config(64, 3), 1, None, 1, obs.view(1, 64, 3, 18))
    assert ei.value.code == MPE_EINVAL
    torch.cuda.synchronize()
