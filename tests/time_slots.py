"""Rollouts whose time runs in slots side by side, against the same steps in calls that are too short for slots: an
environment's trajectory does not depend on how its steps are divided among calls, bit for bit."""
import collections
import os

import torch

from paper_2311_10090_amd import synth
from paper_2311_10090_amd.binding import MpeConfig, MpeEnv

SHORT = 30           # two slots are at least 32 steps


def counters(kind, envs, max_ep):
    """Episode counters at the start: all alike; alike in stretches of 500 envs; each its own, also beyond the episode's end
    and below zero."""
    if kind == "alike":
        return torch.full((envs,), 7 % max_ep, dtype=torch.int32)
    if kind == "stretches":
        return (torch.arange(envs) // 500 % max_ep).to(torch.int32)
    return torch.randint(-3, max_ep + 4, (envs,), generator=torch.Generator().manual_seed(5), dtype=torch.int32)


def outputs(cfg, T, start, pieces, policy=(), critic=(), gru=False, left_out=(), captured=False):
    """Everything that two rollouts of T steps write, each in calls of the given lengths.  captured: the state and the first rollout's
    calls come from a graph, whose calls were chosen when the new counters were not known."""
    assert sum(pieces) == T
    env = MpeEnv(MpeConfig(**cfg))
    if policy:
        (env.set_gru_policy if gru else env.set_policy)(*policy)
    if critic:
        (env.set_gru_critic if gru else env.set_critic)(*critic)
    env.reset(11)
    pa, va, pl, _, step = env.get_state()
    start = start.cuda()
    kept = []
    for first in (True, False):
        sets = []
        for n in pieces:
            sets.append(list(env.empty_traj_ac(n) if critic else env.empty_traj(n)))
            for k in left_out:
                sets[-1][k] = None

        def calls():
            if first:
                env.set_state(pa, va, pl, start, 11, int(step))
            return [(env.rollout_ac if critic else env.rollout)(n, *bufs) for n, bufs in zip(pieces, sets)]
        if first and captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                parts = calls()
            graph.replay()
        else:
            parts = calls()
        parts = [[None if o is None else o.clone() for o in out] for out in parts]
        last = 2 if critic else 1
        for k in range(len(parts[0])):
            if parts[0][k] is not None:
                kept.append(parts[-1][k] if k >= len(parts[0]) - last else torch.cat([p[k] for p in parts]))
        kept += [s.clone() for s in env.get_state()[:4]]
        if gru:
            kept.append(env.get_hidden().clone())
    env.close()
    return kept


def assert_slots_change_nothing(cfg, T, kind, max_ep, **more):
    envs = cfg["num_envs"] * cfg["num_runs"]
    print("slots: %d envs, %d agents, %d steps, episodes of %d, counters %s" % (envs, cfg["num_agents"], T, max_ep, kind), flush=True)
    start = counters(kind, envs, max_ep)
    short = [SHORT] * (T // SHORT) + ([T % SHORT] if T % SHORT else [])
    expected = outputs(cfg, T, start, short, **more)
    for captured in (False, True) if kind != "alike" else (False,):
        for k, (a, b) in enumerate(zip(outputs(cfg, T, start, [T], captured=captured, **more), expected)):
            assert torch.equal(a, b), ("output", k, captured)


TAG = {2: (1, 1), 3: (0, 2), 4: (2, 3), 5: (2, 4), 6: (2, 4), 8: (2, 6), 10: (3, 8)}      # landmarks, adversaries


def config(scenario, agents, envs, max_ep, runs=1, hidden=0, wd=0, reward=None):
    if scenario == "tag":
        landmarks, adversaries = TAG[agents]
        return synth.tag_config(envs, agents, landmarks, adversaries, runs, hidden, wd, max_episode_steps=max_ep)
    return synth.spread_config(envs, agents, runs, hidden, wd, max_episode_steps=max_ep, reward_mode=agents % 2 if reward is None else reward)


# Runs whose slots share wavefronts: (runs, envs of one, agents, critic)
RUNS = [(1024, 16, 3, False), (300, 32, 3, False), (150, 48, 3, False), (100, 64, 3, False), (1024, 16, 3, True), (300, 32, 3, True),
        (256, 48, 3, True), (100, 64, 3, True), (128, 48, 2, True), (512, 48, 2, True), (300, 64, 2, True), (77, 64, 2, True)]

Batch = collections.namedtuple("Batch", "scenario agents wd policy critic envs runs max_ep T reward kernel")


def batches():
    """A batch for every kernel instance with slots."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "slot_batches.txt")
    for line in open(path):
        if not line.startswith("#"):
            s, n, wd, policy, ac, *numbers = line.split(maxsplit=10)[:10]
            yield Batch(s, int(n), int(wd), policy, ac == "1", *map(int, numbers), line.split(maxsplit=10)[10].strip())


def networks(scenario, agents, runs, ac, gru=False):
    D = synth.tag_obs_dim(agents, *TAG[agents]) if scenario == "tag" else 6 * agents
    dev = lambda arrs: [torch.from_numpy(a).cuda() for a in arrs]
    if gru:
        return dict(policy=dev(synth.gru_weights(5, runs, D)), critic=dev(synth.gru_critic_weights(5, runs)) if ac else (), gru=True)
    return dict(policy=dev(synth.policy_weights_with_bias(3, runs, D, 64)), critic=dev(synth.critic_weights(3, runs, D, 64)) if ac else ())


def record_commands(b):
    """For tests/launch_record.py: the batch's rollout is the command before the last."""
    landmarks, adversaries = TAG[b.agents] if b.scenario == "tag" else (b.agents, 0)
    hidden = {"none": 0, "mlp": 64, "gru": synth.GRU_HIDDEN}[b.policy]
    return ["create %d %d %d %d %d %d %d %d %d %d" % (b.scenario == "tag", b.agents, landmarks, adversaries, b.envs, b.runs, hidden, b.wd, b.max_ep, b.reward),
            *{"none": (), "mlp": ("mlp", "mlp_critic"), "gru": ("gru", "critic")}[b.policy], "reset", "%s %d" % ("rollout_ac" if b.critic else "rollout", b.T), "destroy"]
