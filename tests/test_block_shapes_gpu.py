"""The fused feed-forward rollout picks its kernel and block shape by batch size (the small-batch kernel's 16-env blocks,
independent wavefronts of whole envs, 32- or 64-env blocks, 256-env blocks of four sync groups).
All shapes run the same arithmetic in the same order and an env's trajectory depends only on (seed, run,
env index), so jobs of different sizes must agree bit for bit on the envs they share; sampled ranges of
every job, including its ragged tail, are also compared with the oracle."""
import numpy as np
import pytest

from tests import helpers as Hp
from paper_2311_10090_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

T = 30


def say(msg):
    print(msg, flush=True)


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.fail("gpu tests need a device; the library has no CPU fallback")
    from paper_2311_10090_amd.binding import MpeEnv
    from oracle import Oracle
    return MpeEnv, Oracle


def _job(mods, E, N, wd, mixed, ac, w, cw, seed):
    env = mods[0](Hp.gpu_config(E, N, 1, 64, wd, reward_mode=1 if mixed else 0, local_ratio=0.5))
    env.set_policy(*Hp.to_dev(w))
    if ac:
        env.set_critic(*Hp.to_dev(cw))
    env.reset(seed)
    out = env.rollout_ac(T, *env.empty_traj_ac(T)) if ac else env.rollout(T, *env.empty_traj(T))
    state = env.get_state()
    torch.cuda.synchronize()
    env.close()
    return out, state


# sizes (256 CUs): the small-batch kernel up to 32,768 envs (24,576 with bf16 weights or a critic, for 2 agents 16,384 and
# with a critic 12,288); then 3 agents fp32: independent wavefronts up to 43,008, bf16: 32-env blocks up to 32,768; 64-env
# blocks (1 and 2 agents: 32-row wavefronts) up to 65,535 (with a critic 32,767), 256-env blocks beyond
@pytest.mark.parametrize("N,wd,mixed,ac,sizes", [
    (3, 0, False, False, (8192, 8200, 16384, 20001, 65600)),
    (3, 0, True, False, (5000, 12000, 30000)),
    (3, 1, False, False, (8190, 16000, 16390)),
    (3, 0, False, True, (8192, 16384, 16400)),
    (2, 0, False, False, (1000, 30000, 65700)),
    (2, 0, False, True, (1000, 40000)),
    (1, 0, False, False, (333, 65536 + 64)),
    (1, 1, True, False, (100, 50000)),
])
def test_block_shapes_agree_bit_for_bit_and_with_the_oracle(mods, N, wd, mixed, ac, sizes):
    say("block shapes N=%d wd=%d mixed=%d ac=%d sizes=%s" % (N, wd, mixed, ac, sizes))
    w = synth.policy_weights_with_bias(21, 1, 6 * N, 64)
    cw = synth.critic_weights(21, 1, 6 * N, 64)
    jobs = [(E,) + _job(mods, E, N, wd, mixed, ac, w, cw, 8) for E in sizes]
    E0, out0, st0 = jobs[0]
    nper = 6 if ac else 4          # outputs shaped [T][TE]...; the rest are [TE]...
    for E, out, st in jobs[1:]:
        n = min(E, E0)
        for k, (a, b) in enumerate(zip(out0, out)):
            same = torch.equal(a[:, :n], b[:, :n]) if k < nper else torch.equal(a[:n], b[:n])
            assert same, "output %d of the %d-env job differs from the %d-env job's" % (k, E, E0)
        for a, b in zip(st0[:2], st[:2]):      # agent positions and velocities [2][N][TE]
            assert torch.equal(a[..., :n], b[..., :n])
    # oracle: the first envs of the first job and the ragged tail of every job
    for E, out, st in jobs:
        for off, n in [(max(0, E - 40), min(40, E))] + ([(0, 48)] if E == E0 else []):
            orc = mods[1](Hp.oracle_config(n, N, 1, 64, wd, env_offset=off, reward_mode=1 if mixed else 0,
                                           local_ratio=0.5), threads=8)
            orc.set_policy(*w)
            if ac:
                orc.set_critic(*cw)
            orc.reset(8)
            ref = orc.rollout_ac(T) if ac else orc.rollout(T)
            obs, act = out[0][:, off:off + n].cpu().numpy(), out[1][:, off:off + n].cpu().numpy()
            done = out[5 if ac else 3][:, off:off + n].cpu().numpy()
            assert np.array_equal(done, ref[5 if ac else 3])
            assert np.array_equal(obs[0].astype(np.float64), ref[0][0]) and np.array_equal(obs[25].astype(np.float64), ref[0][25])
            same = (act == ref[1]).all(axis=2)
            alive = np.logical_and.accumulate(same[:25], axis=0)
            assert alive[-1].mean() >= (0.9 if wd else 0.97), "envs %d.. of the %d-env job" % (off, E)
            prior = np.vstack([np.ones((1, n), bool), alive[:4]])
            err = np.abs(obs[:5].astype(np.float64) - ref[0][:5]).reshape(5, n, -1).max(axis=2)
            assert (err * prior).max() <= Hp.EPISODE_ATOL, "envs %d.. of the %d-env job" % (off, E)


def _tag_job(mods, E, shape, wd, ac, w, cw, seed):
    env = mods[0](Hp.tag_gpu_config(E, *shape, 1, 64, wd=wd))
    env.set_policy(*Hp.to_dev(w))
    if ac:
        env.set_critic(*Hp.to_dev(cw))
    env.reset(seed)
    out = env.rollout_ac(T, *env.empty_traj_ac(T)) if ac else env.rollout(T, *env.empty_traj(T))
    state = env.get_state()
    torch.cuda.synchronize()
    env.close()
    return out, state


# predator-prey (256 CUs): the small-batch kernel up to 12,697 envs with 4 agents (8,192 bf16 with a critic), 24,576 with 3,
# 16,384 with 2 (12,288 with a critic); then 2 agents 64-env blocks of 32-row wavefronts up to 32,768, 4 agents independent
# wavefronts up to 32,768 (any size with a critic), the regular blocks beyond
@pytest.mark.parametrize("shape,wd,ac,sizes", [
    ((4, 2, 3), 0, False, (8192, 8200, 20001)),
    ((4, 2, 3), 1, False, (8000, 9000)),
    ((4, 2, 3), 0, True, (8192, 16384, 16500)),
    ((2, 1, 1), 0, False, (1000, 32768, 33000)),
    ((2, 1, 1), 0, True, (1000, 40000)),
    ((3, 0, 2), 0, False, (5000, 8193)),
    ((3, 0, 2), 0, True, (8192, 8200)),
])
def test_predator_prey_block_shapes_agree_bit_for_bit_and_with_the_oracle(mods, shape, wd, ac, sizes):
    say("tag block shapes %s wd=%d ac=%d sizes=%s" % (shape, wd, ac, sizes))
    N, D = shape[0], Hp.tag_obs_dim(*shape)
    w = synth.policy_weights_with_bias(22, 1, D, 64)
    cw = synth.critic_weights(22, 1, D, 64)
    jobs = [(E,) + _tag_job(mods, E, shape, wd, ac, w, cw, 9) for E in sizes]
    E0, out0, st0 = jobs[0]
    nper = 6 if ac else 4
    for E, out, st in jobs[1:]:
        n = min(E, E0)
        for k, (a, b) in enumerate(zip(out0, out)):
            same = torch.equal(a[:, :n], b[:, :n]) if k < nper else torch.equal(a[:n], b[:n])
            assert same, "output %d of the %d-env job differs from the %d-env job's" % (k, E, E0)
        for a, b in zip(st0[:2], st[:2]):
            assert torch.equal(a[..., :n], b[..., :n])
    for E, out, st in jobs:
        off, n = E - 40, 40
        orc = mods[1](Hp.tag_oracle_config(n, *shape, 1, 64, wd=wd, env_offset=off), threads=8)
        orc.set_policy(*w)
        if ac:
            orc.set_critic(*cw)
        orc.reset(9)
        ref = orc.rollout_ac(T) if ac else orc.rollout(T)
        obs, act = out[0][:, off:off + n].cpu().numpy(), out[1][:, off:off + n].cpu().numpy()
        done = out[5 if ac else 3][:, off:off + n].cpu().numpy()
        assert np.array_equal(done, ref[5 if ac else 3])
        # episode starts: exact up to the fp32 rounding of differences of off-grid landmark coordinates
        assert np.abs(obs[0] - ref[0][0]).max() <= 1e-6 and np.abs(obs[25] - ref[0][25]).max() <= 1e-6
        same = (act == ref[1]).all(axis=2)
        alive = np.logical_and.accumulate(same[:25], axis=0)
        assert alive[-1].mean() >= (0.9 if wd else 0.97), "envs %d.. of the %d-env job" % (off, E)
        prior = np.vstack([np.ones((1, n), bool), alive[:4]])
        err = np.abs(obs[:5].astype(np.float64) - ref[0][:5]).reshape(5, n, -1).max(axis=2)
        assert (err * prior).max() <= Hp.EPISODE_ATOL, "envs %d.. of the %d-env job" % (off, E)


# recurrent policy: 16-env blocks up to 4,096 envs, 32-env blocks up to 8,192, 64-env blocks beyond
@pytest.mark.parametrize("N,sizes", [(3, (4096, 4100, 8192, 8200)), (1, (100, 5000, 9000)), (2, (4090, 8300)),
                                     (4, (3000, 4200, 9000)), (5, (4096, 8200))])
def test_recurrent_block_shapes_agree_bit_for_bit_and_with_the_oracle(mods, N, sizes):
    say("recurrent block shapes N=%d sizes=%s" % (N, sizes))
    w = synth.gru_weights(23, 1, 6 * N)
    jobs = []
    for E in sizes:
        env = mods[0](Hp.gpu_config(E, N, 1, 128, 1))
        env.set_gru_policy(*Hp.to_dev(w))
        env.reset(10)
        out = env.rollout(T, *env.empty_traj(T))
        hid = env.get_hidden()
        torch.cuda.synchronize()
        env.close()
        jobs.append((E, out, hid))
    E0, out0, hid0 = jobs[0]
    for E, out, hid in jobs[1:]:
        n = min(E, E0)
        for k, (a, b) in enumerate(zip(out0, out)):
            same = torch.equal(a[:, :n], b[:, :n]) if k < 4 else torch.equal(a[:n], b[:n])
            assert same, "output %d of the %d-env job differs from the %d-env job's" % (k, E, E0)
        assert torch.equal(hid0[:n], hid[:n]), "carried state"
    for E, out, hid in jobs:
        off, n = E - 40, 40
        orc = mods[1](Hp.oracle_config(n, N, 1, 128, 1, env_offset=off), threads=8)
        orc.set_gru(*w)
        orc.reset(10)
        ref = orc.rollout(T)
        obs, act = out[0][:, off:off + n].cpu().numpy(), out[1][:, off:off + n].cpu().numpy()
        assert np.array_equal(out[3][:, off:off + n].cpu().numpy(), ref[3])
        assert np.array_equal(obs[0].astype(np.float64), ref[0][0]) and np.array_equal(obs[25].astype(np.float64), ref[0][25])
        same = (act == ref[1]).all(axis=2)
        alive = np.logical_and.accumulate(same[:25], axis=0)
        assert alive[-1].mean() >= 0.9, "envs %d.. of the %d-env job" % (off, E)
        prior = np.vstack([np.ones((1, n), bool), alive[:4]])
        err = np.abs(obs[:5].astype(np.float64) - ref[0][:5]).reshape(5, n, -1).max(axis=2)
        assert (err * prior).max() <= Hp.EPISODE_ATOL, "envs %d.. of the %d-env job" % (off, E)


# several runs of 16 k envs each (the paper's IPPO setting on MPE is 16 envs per run, App. G): the small-batch kernel's
# blocks of 16 envs inside one run, with its weights (many runs: test_run_blocks_gpu.py)
@pytest.mark.parametrize("N,E,R,wd,mixed,ac", [
    (3, 16, 40, 0, False, False), (3, 48, 5, 0, False, False), (3, 80, 3, 0, True, False), (3, 16, 9, 0, False, True),
    (3, 16, 12, 1, False, False), (1, 16, 7, 0, False, False), (2, 32, 9, 0, False, False), (2, 16, 5, 0, True, True),
    (1, 48, 3, 0, False, True), (3, 96, 3, 0, False, False), (3, 32, 6, 0, True, True),
])
def test_small_runs_with_their_own_weights_against_the_oracle(mods, N, E, R, wd, mixed, ac):
    from scipy.special import log_softmax
    say("small runs N=%d E=%d R=%d wd=%d mixed=%d ac=%d" % (N, E, R, wd, mixed, ac))
    D, TE = 6 * N, E * R
    w = synth.policy_weights_with_bias(31, R, D, 64)
    cw = synth.critic_weights(31, R, D, 64)
    rm = dict(reward_mode=1 if mixed else 0, local_ratio=0.5)
    env = mods[0](Hp.gpu_config(E, N, R, 64, wd, **rm))
    orc = mods[1](Hp.oracle_config(E, N, R, 64, wd, **rm), threads=8)
    env.set_policy(*Hp.to_dev(w))
    orc.set_policy(*w)
    if ac:
        env.set_critic(*Hp.to_dev(cw))
        orc.set_critic(*cw)
    env.reset(11)
    orc.reset(11)
    out = env.rollout_ac(T, *env.empty_traj_ac(T)) if ac else env.rollout(T, *env.empty_traj(T))
    ref = orc.rollout_ac(T) if ac else orc.rollout(T)
    obs, act = out[0].cpu().numpy(), out[1].cpu().numpy()
    rew, done = out[4 if ac else 2].cpu().numpy(), out[5 if ac else 3].cpu().numpy()
    assert np.array_equal(done, ref[5 if ac else 3])
    assert np.array_equal(obs[0].astype(np.float64), ref[0][0]) and np.array_equal(obs[25].astype(np.float64), ref[0][25])
    same = (act == ref[1]).all(axis=2)
    alive = np.logical_and.accumulate(same[:25], axis=0)
    assert alive[-1].mean() >= (0.9 if wd else 0.97)
    prior = np.vstack([np.ones((1, TE), bool), alive[:4]])
    err = np.abs(obs[:5].astype(np.float64) - ref[0][:5]).reshape(5, TE, -1).max(axis=2)
    assert (err * prior).max() <= Hp.EPISODE_ATOL
    if not mixed:
        assert (np.abs(rew[:5] - ref[4 if ac else 2][:5]) * alive[:5]).max() <= Hp.EPISODE_ATOL
    # the runs use their own weights and streams: first actions differ from run to run
    a0 = act[0].reshape(R, E, N)
    assert any(not np.array_equal(a0[0], a0[r]) for r in range(1, R))
    if ac and not wd:
        logp, val = out[2].cpu().numpy(), out[3].cpu().numpy()
        for run in range(R):
            sl = slice(run * E, (run + 1) * E)
            rows = obs[:, sl].reshape(-1, D).astype(np.float64)
            z = orc.policy_logits(rows, run=run)
            ref_lp = log_softmax(z, axis=1)[np.arange(z.shape[0]), act[:, sl].reshape(-1)]
            Hp.assert_close_step(logp[:, sl].reshape(-1), ref_lp, "log-prob from recorded obs and actions")
            Hp.assert_close_step(val[:, sl].reshape(-1), orc.value(rows, run=run), "value from recorded obs")
    env.close()


@pytest.mark.parametrize("shape,E,R,wd,ac", [
    ((4, 2, 3), 16, 20, 0, False), ((4, 2, 3), 48, 4, 1, False), ((4, 2, 3), 16, 6, 0, True), ((4, 2, 3), 64, 3, 0, True),
    ((2, 1, 1), 16, 9, 0, False), ((2, 1, 1), 80, 2, 0, True), ((3, 0, 2), 16, 10, 0, False), ((3, 0, 2), 48, 3, 0, True),
])
def test_predator_prey_small_runs_with_their_own_weights_against_the_oracle(mods, shape, E, R, wd, ac):
    from scipy.special import log_softmax
    say("tag small runs %s E=%d R=%d wd=%d ac=%d" % (shape, E, R, wd, ac))
    N, D, TE = shape[0], Hp.tag_obs_dim(*shape), E * R
    w = synth.policy_weights_with_bias(32, R, D, 64)
    cw = synth.critic_weights(32, R, D, 64)
    env = mods[0](Hp.tag_gpu_config(E, *shape, R, 64, wd=wd))
    orc = mods[1](Hp.tag_oracle_config(E, *shape, R, 64, wd=wd), threads=8)
    env.set_policy(*Hp.to_dev(w))
    orc.set_policy(*w)
    if ac:
        env.set_critic(*Hp.to_dev(cw))
        orc.set_critic(*cw)
    env.reset(12)
    orc.reset(12)
    out = env.rollout_ac(T, *env.empty_traj_ac(T)) if ac else env.rollout(T, *env.empty_traj(T))
    ref = orc.rollout_ac(T) if ac else orc.rollout(T)
    obs, act = out[0].cpu().numpy(), out[1].cpu().numpy()
    rew, done = out[4 if ac else 2].cpu().numpy(), out[5 if ac else 3].cpu().numpy()
    assert np.array_equal(done, ref[5 if ac else 3])
    assert np.abs(obs[0] - ref[0][0]).max() <= 1e-6 and np.abs(obs[25] - ref[0][25]).max() <= 1e-6
    same = (act == ref[1]).all(axis=2)
    alive = np.logical_and.accumulate(same[:25], axis=0)
    assert alive[-1].mean() >= (0.9 if wd else 0.97)
    prior = np.vstack([np.ones((1, TE), bool), alive[:4]])
    err = np.abs(obs[:5].astype(np.float64) - ref[0][:5]).reshape(5, TE, -1).max(axis=2)
    assert (err * prior).max() <= Hp.EPISODE_ATOL
    a0 = act[0].reshape(R, E, N)
    assert any(not np.array_equal(a0[0], a0[r]) for r in range(1, R))
    if ac:
        logp, val = out[2].cpu().numpy(), out[3].cpu().numpy()
        for run in range(R):
            sl = slice(run * E, (run + 1) * E)
            rows = obs[:, sl].reshape(-1, D).astype(np.float64)
            z = orc.policy_logits(rows, run=run)
            ref_lp = log_softmax(z, axis=1)[np.arange(z.shape[0]), act[:, sl].reshape(-1)]
            Hp.assert_close_step(logp[:, sl].reshape(-1), ref_lp, "log-prob from recorded obs and actions")
            Hp.assert_close_step(val[:, sl].reshape(-1), orc.value(rows, run=run), "value from recorded obs")
    env.close()
