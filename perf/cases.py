"""What a user of the library has it do, as measurable cases over the range of sizes, shapes and options.

A case names one entry point and its configuration (plain values):
  call       "step" (mpe_step), "rollout" (mpe_rollout) or "rollout_ac" (mpe_rollout_ac)
  scenario   "spread" or "tag" (predator-prey; then also landmarks, adversaries)
  envs, runs, agents, steps      environments per run, independent runs, agents per env, steps of one rollout
  policy     "none" (actions from the caller or seeded uniform ones), "mlp" or "gru"; hidden, dtype
  reward     "shared" or "mixed" (one value per agent)
  learner    the weights are installed again before every rollout, as a training loop does after each update

prepare() makes what such a program holds before the call (handle, weights, trajectory buffers, actions), run() is
one call of the loop, and its outputs are the trajectory buffers the call fills.
"""
import math

import torch

from paper_2311_10090_amd import synth
from paper_2311_10090_amd.binding import MpeConfig, MpeEnv

DEVICE = "cuda:0"
GRU = synth.GRU_HIDDEN
TAG_SHAPES = ((4, 2, 3), (2, 1, 1), (3, 0, 2), (6, 2, 4), (5, 2, 4), (8, 2, 6), (10, 3, 8))   # agents, landmarks, adversaries


def _case(name, call, envs, agents=3, runs=1, steps=128, scenario="spread", landmarks=None, adversaries=0, policy="none",
          hidden=0, dtype="fp32", reward="shared", learner=False):
    case = dict(call=call, scenario=scenario, envs=envs, runs=runs, agents=agents,
                landmarks=agents if landmarks is None else landmarks, adversaries=adversaries, steps=steps,
                policy=policy, hidden=hidden, dtype=dtype, reward=reward, learner=learner)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # one transition of a few environments under given actions: an evaluation or debugging loop, all latency
        _case("step_64", "step", 64, steps=1),
        # the same call at the size of a large batch: a program with an agent of its own steps the environments
        _case("step_65536", "step", 65536, steps=1),
        # random-action throughput at the 10,000 environments that environment speed is usually quoted on
        _case("env_10000", "rollout", 10000, steps=100),
        # random-action throughput of a batch that fills the chip: bound by the trajectory writes
        _case("env_65536", "rollout", 65536),
        # rollout of the small training batch, policy evaluated in the loop
        _case("mlp_4096", "rollout", 4096, policy="mlp", hidden=64),
        # the headline shape: rollout of a batch that fills the chip
        _case("mlp_65536", "rollout", 65536, policy="mlp", hidden=64),
        # more agents with their own rewards, an environment count that is no multiple of anything
        _case("mlp_6_agents", "rollout", 20011, agents=6, policy="mlp", hidden=64, reward="mixed"),
        # the scaled scenario: ten agents, wide network, bf16 weights
        _case("mlp_10_agents_bf16", "rollout", 16384, agents=10, policy="mlp", hidden=128, dtype="bf16"),
        # independent runs side by side, every run with its own weights
        _case("runs_1024x64", "rollout", 64, runs=1024, policy="mlp", hidden=64),
        # the collection phase of 1,024 training runs of 16 environments each: new weights, then an actor-critic rollout
        _case("train_1024x16", "rollout_ac", 16, runs=1024, policy="mlp", hidden=64, learner=True),
        # the collection phase of one large training run in the predator-prey scenario
        _case("train_tag", "rollout_ac", 65536, agents=4, scenario="tag", landmarks=2, adversaries=3, policy="mlp", hidden=64,
              learner=True),
        # the collection phase of one large training run with a recurrent agent
        _case("train_gru", "rollout_ac", 65536, policy="gru", hidden=GRU, dtype="bf16", learner=True),
    ]


def _log_int(rng, lo, hi):
    """A whole number in [lo, hi], even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("step", "env", "mlp", "mlp", "runs", "train", "train_runs", "tag", "gru"))
    steps = _log_int(rng, 32, 128)
    reward = rng.choice(("shared", "shared", "mixed"))
    agents = rng.choice((1, 2, 3, 3, 3, 4, 5, 6, 7, 8, 9, 10))
    rows = 196608                                    # agent rows of the largest batch
    if kind == "step":
        return _case(None, "step", _log_int(rng, 16, 65536 // max(1, agents // 3)), agents, steps=1, reward=reward)
    if kind == "env":
        # a row of ten agents is 240 bytes: the batch shrinks with the square of the agents
        return _case(None, "rollout", _log_int(rng, 64, min(65536, 65536 * 9 // agents ** 2)), agents, steps=steps, reward=reward)
    if kind in ("mlp", "train"):
        dtype = rng.choice(("fp32", "fp32", "bf16"))
        hidden = rng.choice((64, 128)) if dtype == "bf16" and agents >= 4 else 64
        ac = kind == "train"
        return _case(None, "rollout_ac" if ac else "rollout", _log_int(rng, 64, rows // max(3, agents)), agents, steps=steps,
                     policy="mlp", hidden=hidden, dtype=dtype, reward=reward, learner=ac)
    if kind in ("runs", "train_runs"):
        ac = kind == "train_runs"
        runs = _log_int(rng, 16, 1024)
        return _case(None, "rollout_ac" if ac else "rollout", rng.choice((16, 32, 48, 64)), rng.choice((1, 2, 3, 3)), runs=runs,
                     steps=steps, policy="mlp", hidden=64, dtype=rng.choice(("fp32", "fp32", "bf16")), reward=reward, learner=ac)
    if kind == "tag":
        agents, landmarks, adversaries = rng.choice(TAG_SHAPES)
        call = rng.choice(("rollout", "rollout_ac"))
        return _case(None, call, _log_int(rng, 64, rows // max(3, agents)), agents, steps=steps, scenario="tag", landmarks=landmarks,
                     adversaries=adversaries, policy="mlp", hidden=64, dtype=rng.choice(("fp32", "fp32", "bf16")),
                     learner=call == "rollout_ac")
    call = rng.choice(("rollout", "rollout_ac"))
    agents = rng.choice((1, 2, 3, 3, 3, 4, 5, 6))
    return _case(None, call, _log_int(rng, 64, rows // 2 // max(3, agents)), agents, steps=steps, policy="gru", hidden=GRU, dtype="bf16",
                 reward=reward, learner=call == "rollout_ac")


def _obs_dim(case):
    if case["scenario"] == "tag":
        return synth.tag_obs_dim(case["agents"], case["landmarks"], case["adversaries"])
    return 6 * case["agents"]


def _config(case):
    wd = 1 if case["dtype"] == "bf16" else 0
    if case["scenario"] == "tag":
        return synth.tag_config(case["envs"], case["agents"], case["landmarks"], case["adversaries"], case["runs"],
                                case["hidden"], wd)
    return synth.spread_config(case["envs"], case["agents"], case["runs"], case["hidden"], wd,
                               reward_mode=1 if case["reward"] == "mixed" else 0)


def _mlp_weights(gen, runs, obs_dim, hidden, outputs):
    """N(0, 1/fan_in) matrices and small biases, [runs][fan_in][fan_out]; outputs None: a critic's single output."""
    def mat(*shape):
        return torch.randn((runs,) + shape, generator=gen, device=DEVICE) / math.sqrt(shape[0])

    def vec(*shape):
        return torch.rand((runs,) + shape, generator=gen, device=DEVICE) * 0.2 - 0.1
    last = (hidden,) if outputs is None else (hidden, outputs)
    return [mat(obs_dim, hidden), vec(hidden), mat(hidden, hidden), vec(hidden), mat(*last),
            vec() if outputs is None else vec(outputs)]


def _gru_weights(gen, runs, obs_dim):
    def mat(*shape):
        return torch.randn((runs,) + shape, generator=gen, device=DEVICE) / math.sqrt(shape[0])

    def vec(*shape):
        return torch.rand((runs,) + shape, generator=gen, device=DEVICE) * 0.2 - 0.1
    policy = [mat(obs_dim, GRU), vec(GRU), mat(GRU, 3 * GRU), vec(3 * GRU), mat(GRU, 3 * GRU), vec(3 * GRU),
              mat(GRU, GRU), vec(GRU), mat(GRU, synth.NUM_ACTIONS), vec(synth.NUM_ACTIONS)]
    critic = [mat(GRU, GRU), vec(GRU), mat(GRU), vec()]
    return policy, critic


def _install(state):
    env, case = state["env"], state["case"]
    if case["policy"] == "mlp":
        env.set_policy(*state["policy"])
        if case["call"] == "rollout_ac":
            env.set_critic(*state["critic"])
    elif case["policy"] == "gru":
        env.set_gru_policy(*state["policy"])
        if case["call"] == "rollout_ac":
            env.set_gru_critic(*state["critic"])


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    env = MpeEnv(MpeConfig(**_config(case)), DEVICE)
    state = {"case": case, "env": env}
    if case["policy"] == "mlp":
        state["policy"] = _mlp_weights(gen, case["runs"], env.D, case["hidden"], synth.NUM_ACTIONS)
        state["critic"] = _mlp_weights(gen, case["runs"], env.D, case["hidden"], None)
    elif case["policy"] == "gru":
        state["policy"], state["critic"] = _gru_weights(gen, case["runs"], env.D)
    _install(state)
    env.reset(seed & 0xFFFFFFFF)
    if case["call"] == "step":
        state["actions"] = torch.randint(0, synth.NUM_ACTIONS, (env.TE, env.N), generator=gen, device=DEVICE, dtype=torch.uint8)
        state["out"] = (env.empty_obs(), torch.empty(env.rew_shape, dtype=torch.float32, device=DEVICE),
                        torch.empty((env.TE,), dtype=torch.uint8, device=DEVICE))
    elif case["call"] == "rollout":
        state["out"] = env.empty_traj(case["steps"])
    else:
        state["out"] = env.empty_traj_ac(case["steps"])
    return state


def run(state):
    env, case = state["env"], state["case"]
    if case["call"] == "step":
        return env.step(state["actions"], *state["out"])
    if case["learner"]:
        _install(state)
    out = (env.rollout if case["call"] == "rollout" else env.rollout_ac)(case["steps"], *state["out"])
    if case["policy"] == "gru":
        # a learner keeps the carried state that the next segment starts from
        return tuple(out) + (env.get_hidden(),)
    return out


def _flops_per_agent_step(case):
    """Multiply-adds of the networks, two operations each (the environment's own arithmetic is left out)."""
    d, h, a = _obs_dim(case), case["hidden"], synth.NUM_ACTIONS
    ac = case["call"] == "rollout_ac"
    if case["policy"] == "mlp":
        return 2 * (d * h + h * h + h * a) + (2 * (d * h + h * h + h) if ac else 0)
    if case["policy"] == "gru":
        return 2 * (d * h + 2 * h * 3 * h + h * h + h * a) + (2 * (h * h + h) if ac else 0)
    return 0


def work(case):
    n, d, lm = case["agents"], _obs_dim(case), case["landmarks"]
    te, t = case["envs"] * case["runs"], case["steps"]
    per_agent_reward = case["reward"] == "mixed" or case["scenario"] == "tag"
    rewards = 4 * (n if per_agent_reward else 1)
    state = 2 * (16 * n + 4) + 8 * lm                 # positions, velocities, counter in and out; landmarks in
    if case["call"] == "step":
        return {"bytes": te * (state + n + 4 * n * d + rewards + 1), "flops": 0}
    step = 4 * n * d + n + rewards + 1 + (8 * n if case["call"] == "rollout_ac" else 0)
    hidden = case["hidden"]
    weights = 0
    if case["policy"] == "mlp":
        weights = 4 * (d * hidden + hidden * hidden + 7 * hidden) * (2 if case["call"] == "rollout_ac" else 1)
    elif case["policy"] == "gru":
        weights = 4 * (d * hidden + 7 * hidden * hidden)
        state += 2 * 4 * n * hidden                   # carried state in and out
    return {"bytes": te * (t * step + state + 4 * n * d) + case["runs"] * weights,
            "flops": te * t * n * _flops_per_agent_step(case)}


def tolerance(case):
    if case["call"] == "step":
        # one fp32 transition; the force between nearly coincident agents amplifies a rounding of their distance
        return {"rel": 1e-5, "max": 1e-3}
    if case["policy"] == "none":
        # Contacts are stiff (a position difference grows about 2.3 times per step while two agents overlap), so a
        # few episodes in ten thousand, with ten agents one in ten, leave a rounding difference above 1e-4 until
        # their reset; an overlap that a rounding decides is worth half a unit of reward.
        return {"rel": 1e-3, "max": 0.9}
    # Sampling turns a rounding difference of two logits into another action now and then, and the environment is
    # on another path from there to the end of its episode: about one action in 1e7 with fp32 weights, a few in 1e5
    # with bf16 ones (a value at a rounding boundary of bf16 moves a logit by 1e-3).
    if case["dtype"] == "fp32":
        return {"rel": 5e-3, "max": 0.99, "differ": 1e-4}
    return {"rel": 0.03, "max": 0.99, "differ": 3e-3}
