"""Performance cases of the rollout library: what its users have it do, through its Python entry points.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare(case, seed)`` makes what a
program holds before the call (env state, policy weights with their packed copy, trajectory buffers, workspace),
``run(state)`` is one call (or, for the actor-critic rollout, the rollout and the advantage estimate that follows
it), ``work(case)`` its unavoidable bytes and operations, ``tolerance(case)`` how far outputs may be off and
``exact(case, seed)`` the outputs in float64 where they do not hang on a sampled trajectory.

Rollouts go on where the previous call of the same state stopped (t0 advances), as a training loop's do.  Env
sizes and networks are the library's workloads (paper_2609_13716_amd/workloads.py):

    op "step"    rollout_step, injected actions: an external policy drives the envs
    op "run"     rollout_run, the fused rollout of one shared policy
    op "ac"      rollout_run_ac, then gae over the stored trajectory: what a PPO-style learner consumes
    op "pop"     rollout_run_pop, an ego policy paired with the teammates of a population
    op "teams"   rollout_run_teams, an ego policy paired with heuristic teammates
    op "s5"      rollout_run_s5, the recurrent S5 actor-critic
    op "policy"  policy_forward on stored observations: evaluation of a batch, a learner's forward pass
"""

import numpy as np
import torch

from paper_2609_13716_amd import rollout as R
from paper_2609_13716_amd import workloads

# Env configurations and the policies that act in them: (config, observation size, actions, hidden widths).
_LBF8 = dict(grid_h=8, grid_w=8, n_agents=2, n_food=3, max_agent_level=2, max_food_level=3, max_steps=50)
_LBF7 = dict(grid_h=7, grid_w=7, n_agents=2, n_food=3, max_agent_level=1, max_food_level=2, max_steps=50,
             const_levels=True)
_LBF12 = dict(grid_h=12, grid_w=12, n_agents=3, n_food=6, max_agent_level=3, max_food_level=6, max_steps=50)
ENVS = {
    "lbf8": dict(D=192, nA=6, A=2, hidden=(128, 128), cfg=lambda E, s: R.EnvConfig(E, seed=s, **_LBF8)),
    "lbf8_small": dict(D=192, nA=6, A=2, hidden=(64, 64), cfg=lambda E, s: R.EnvConfig(E, seed=s, **_LBF8)),
    "lbf7": dict(D=147, nA=6, A=2, hidden=(128, 128), cfg=lambda E, s: R.EnvConfig(E, seed=s, **_LBF7)),
    "lbf12": dict(D=432, nA=6, A=3, hidden=(256, 256), cfg=lambda E, s: R.EnvConfig(E, seed=s, **_LBF12)),
    "oc": dict(D=1170, nA=6, A=2, hidden=(256, 256), cfg=lambda E, s: R.overcooked_config(E, seed=s)),
    "hn": dict(D=658, nA=20, A=2, hidden=(512, 512), cfg=lambda E, s: R.hanabi_config(E, seed=s)),
    "hn_mini": dict(D=278, nA=16, A=2, hidden=(256, 256),
                    cfg=lambda E, s: R.hanabi_config(E, seed=s, colours=3, ranks=3)),
}
# Mean number of non-zero features of an observation (for the stored observations of op "policy").
NONZERO = {"lbf8": 6, "lbf8_small": 6, "lbf7": 6, "lbf12": 10, "oc": 36, "hn": 150, "hn_mini": 70}
S5 = dict(d_model=128, d_state=128, head_width=1024)
POPULATION = 9
GAMMA, LAM = 0.99, 0.95


def listed():
    return [
        # one step of a small batch driven from outside: the shortest call a program makes, all latency
        dict(name="step_lbf8_256x1_f32", op="step", env="lbf8", envs=256, steps=1, dtype="f32"),
        # a debugging / unit-size rollout in float32: one workgroup's chain, the chip idle
        dict(name="run_lbf8_16x128_f32", op="run", env="lbf8_small", envs=16, steps=128, dtype="f32"),
        # the headline rollout: 4096 envs of 8x8 Level-Based Foraging
        dict(name="run_lbf8_4096x128_bf16", op="run", env="lbf8", envs=4096, steps=128, dtype="bf16"),
        # the largest grid and batch: three agents, 256-wide layers
        dict(name="run_lbf12_16384x128_bf16", op="run", env="lbf12", envs=16384, steps=128, dtype="bf16"),
        # kitchens over a full episode
        dict(name="run_oc_4096x400_bf16", op="run", env="oc", envs=4096, steps=400, dtype="bf16"),
        # Hanabi self-play with legality masks
        dict(name="run_hn_4096x80_bf16", op="run", env="hn", envs=4096, steps=80, dtype="bf16"),
        # a learner's data collection: values, log-probabilities, then advantages; a ragged batch
        dict(name="ac_lbf8_3000x128_bf16", op="ac", env="lbf8", envs=3000, steps=128, dtype="bf16"),
        # ad hoc teamwork evaluation: one ego, eight teammates in blocks of envs
        dict(name="pop_lbf8_4096x128_bf16", op="pop", env="lbf8", envs=4096, steps=128, dtype="bf16", blocks=True),
        # the recurrent ego agent
        dict(name="s5_lbf8_4096x128_bf16", op="s5", env="lbf8", envs=4096, steps=128, dtype="bf16"),
        # a learner's forward pass over a stored kitchen batch
        dict(name="policy_oc_262144_bf16", op="policy", env="oc", rows=262144, dtype="bf16", masked=False),
        # the same for Hanabi, with legality masks and an odd number of rows
        dict(name="policy_hn_100003_bf16", op="policy", env="hn", rows=100003, dtype="bf16", masked=True),
        # Hanabi games driven from outside, observations and legality masks out
        dict(name="step_hn_4096x80_bf16", op="step", env="hn", envs=4096, steps=80, dtype="bf16"),
    ]


# (op, env, dtypes, most envs, most steps) of the drawn rollouts; the products stay within the listed cases' work.
_DRAWN = [
    ("step", "lbf8", ("f32", "bf16"), 4096, 128), ("step", "lbf7", ("f32", "bf16"), 4096, 128),
    ("step", "lbf12", ("bf16",), 8192, 64), ("step", "oc", ("f32", "bf16"), 4096, 100),
    ("step", "hn", ("f32", "bf16"), 4096, 80), ("step", "hn_mini", ("bf16",), 4096, 80),
    ("run", "lbf8_small", ("f32", "bf16"), 1024, 128), ("run", "lbf8", ("f32", "bf16"), 16384, 128),
    ("run", "lbf7", ("bf16",), 4096, 128), ("run", "lbf12", ("bf16",), 16384, 64),
    ("run", "oc", ("bf16",), 4096, 200), ("run", "hn", ("bf16",), 4096, 80), ("run", "hn_mini", ("bf16",), 4096, 80),
    ("ac", "lbf8", ("bf16",), 8192, 128), ("pop", "lbf8", ("bf16",), 4096, 128), ("teams", "lbf7", ("bf16",), 4096, 128),
    ("s5", "lbf8", ("bf16",), 4096, 64),
]
_DRAWN_POLICY = [("lbf8", ("f32", "bf16"), 1 << 20), ("lbf8_small", ("f32", "bf16"), 1 << 20), ("lbf7", ("bf16",), 1 << 19),
                 ("lbf12", ("bf16",), 1 << 18), ("oc", ("bf16",), 1 << 18), ("hn", ("bf16",), 1 << 17),
                 ("hn_mini", ("bf16",), 1 << 18)]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    if rng.random() < 0.3:
        env, dtypes, most = rng.choice(_DRAWN_POLICY)
        return dict(op="policy", env=env, rows=_log_uniform(rng, 1, most), dtype=rng.choice(dtypes),
                    masked=env.startswith("hn"))
    op, env, dtypes, most_envs, most_steps = rng.choice(_DRAWN)
    case = dict(op=op, env=env, envs=_log_uniform(rng, 8, most_envs), steps=_log_uniform(rng, 1, most_steps),
                dtype=rng.choice(dtypes))
    if op == "pop":  # teammates in contiguous blocks of envs, or dealt round-robin
        case["blocks"] = rng.random() < 0.7
    return case


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _dims(case):
    e = ENVS[case["env"]]
    return (e["D"], *e["hidden"], e["nA"] + (1 if case["op"] == "ac" else 0))


def _policy_inputs(case, seed):
    """Weights, biases, observations and masks of op "policy" (torch only: exact() starts from them too)."""
    D, H1, H2, nA = _dims(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ws, bs = [], []
    for n, k in ((H1, D), (H2, H1), (nA, H2)):
        ws.append((torch.randn(n, k, generator=g, device="cuda") / k ** 0.5).to(_torch_dtype(case)))
        bs.append((0.1 * torch.randn(n, generator=g, device="cuda")).to(_torch_dtype(case)))
    rows = case["rows"]
    # sparse observations of small whole numbers: mostly ones, an occasional level
    u = torch.rand(rows, D, generator=g, device="cuda")
    p = NONZERO[case["env"]] / D
    one, two = (1.0, 1.0) if case["env"].startswith("hn") else (1.0, 2.0)
    obs = torch.where(u < 0.75 * p, one, torch.where(u < p, two, 0.0)).to(_torch_dtype(case))
    legal = None
    if case["masked"]:
        legal = (torch.rand(rows, nA, generator=g, device="cuda") < 0.6).to(torch.uint8)
    return ws, bs, obs, legal


def prepare(case, seed):
    op, dt = case["op"], case["dtype"]
    e = ENVS[case["env"]]
    st = dict(case=case)
    if op == "policy":
        ws, bs, st["obs"], st["legal"] = _policy_inputs(case, seed)
        st["policy"] = R.Policy(ws, bs, dt)
        st["logits"] = torch.empty(case["rows"], e["nA"], device="cuda")
        return st
    E, T, A, D, nA = case["envs"], case["steps"], e["A"], e["D"], e["nA"]
    cfg = st["cfg"] = e["cfg"](E, seed)
    st["state"] = R.new_state(cfg)
    R.rollout_init(cfg, st["state"])
    st["t"] = 0
    tdt = _torch_dtype(case)
    new = lambda *shape, dtype=torch.float32: torch.empty(*shape, dtype=dtype, device="cuda")  # noqa: E731
    if op == "step":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        # (Hanabi: most uniform actions are illegal and act as the lowest legal one)
        st["actions"] = torch.randint(0, nA, (T, E, A), generator=g, device="cuda", dtype=torch.int32)
        st["out"] = dict(obs_out=new(T, E, A, D, dtype=tdt), reward=new(T, E), done=new(T, E, dtype=torch.uint8))
        if case["env"].startswith("hn"):
            st["out"]["legal_out"] = new(T, E, A, nA, dtype=torch.uint8)
        return st
    out = st["out"] = dict(obs=new(T, E, A, D, dtype=tdt), actions=new(T, E, A, dtype=torch.int32),
                           logits=new(T, E, A, nA), reward=new(T, E), done=new(T, E, dtype=torch.uint8),
                           obs_last=new(E, A, D, dtype=tdt))
    if op in ("ac", "s5"):
        out.update(value=new(T, E, A), logp=new(T, E, A), value_last=new(E, A))
    if op == "ac":
        st["adv"], st["ret"] = new(T, E, A), new(T, E, A)
    if op == "s5":
        st["policy"] = R.S5Policy(workloads.s5_params(D, S5["d_model"], S5["d_state"], S5["head_width"], nA, seed))
        st["carry"] = torch.zeros(E * A, 2, S5["d_state"], device="cuda")
        st["workspace"] = new(R.s5_workspace_bytes(cfg, st["policy"]), dtype=torch.uint8)
    elif op == "pop":
        nets = [workloads.policy_weights(_dims(case), seed + q, bias_scale=0.1) for q in range(POPULATION)]
        st["policy"] = R.Population([w for w, _ in nets], [b for _, b in nets], dt)
        mates = np.arange(E) * (POPULATION - 1) // E if case["blocks"] else np.arange(E) % (POPULATION - 1)
        idx = np.zeros((E, A), np.int32)
        idx[:, 1:] = 1 + mates[:, None]
        st["index"] = torch.from_numpy(idx).cuda()
    else:
        ws, bs = workloads.policy_weights(_dims(case), seed, bias_scale=0.1)
        st["policy"] = R.Policy(ws, bs, dt)
        if op == "teams":  # agent 0 the policy, agent 1 heuristic kind e mod 11
            kinds = np.full((E, A), -1, np.int32)
            kinds[:, 1] = np.arange(E) % len(R.HEURISTICS)
            st["kinds"] = torch.from_numpy(kinds).cuda()
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "policy":
        return R.policy_forward(st["policy"], st["obs"], st["legal"], st["logits"])
    cfg, state, t, out = st["cfg"], st["state"], st["t"], st["out"]
    st["t"] = t + case["steps"]
    if op == "step":
        R.rollout_step(cfg, state, t, st["actions"], **out)
        return dict(out, state=state)
    if op == "run":
        R.rollout_run(cfg, st["policy"], state, t, case["steps"], **out)
        return dict(out, state=state)
    if op == "pop":
        R.rollout_run_pop(cfg, st["policy"], st["index"], state, t, case["steps"], **out)
        return dict(out, state=state)
    if op == "teams":
        R.rollout_run_teams(cfg, st["policy"], st["kinds"], state, t, case["steps"], **out)
        return dict(out, state=state)
    if op == "s5":
        R.rollout_run_s5(cfg, st["policy"], state, st["carry"], t, case["steps"], workspace=st["workspace"], **out)
        return dict(out, state=state, carry=st["carry"])
    R.rollout_run_ac(cfg, st["policy"], state, t, case["steps"], **out)
    R.gae(out["reward"], out["done"], out["value"], out["value_last"], GAMMA, LAM, adv=st["adv"], ret=st["ret"])
    return dict(out, state=state, adv=st["adv"], ret=st["ret"])


def work(case):
    e = ENVS[case["env"]]
    es = 2 if case["dtype"] == "bf16" else 4
    D, nA = e["D"], e["nA"]
    dims = _dims(case)
    row_flops = 2 * sum(a * b for a, b in zip(dims, dims[1:]))
    weights = es * sum(a * b + b for a, b in zip(dims, dims[1:]))
    if case["op"] == "policy":
        rows = case["rows"]
        return dict(bytes=rows * (D * es + 4 * nA + (nA if case["masked"] else 0)) + weights, flops=rows * row_flops)
    E, T, A = case["envs"], case["steps"], e["A"]
    # observation, actions, reward and done of every step; the env state in and out once
    nbytes = T * E * (A * D * es + 4 * A + 5) + 2 * R.rl_state_bytes(e["cfg"](E, 0))
    if case["op"] == "step":
        return dict(bytes=nbytes + (T * E * A * nA if case["env"].startswith("hn") else 0), flops=0)
    nbytes += T * E * A * nA * 4 + E * A * D * es  # logits, the last observation
    if case["op"] == "s5":
        H, P, F = S5["d_model"], S5["d_state"], S5["head_width"]
        row_flops = 2 * (D * H + 2 * P * H + 2 * P * H + 2 * (H * F + 2 * F * F) + F * (nA + 1))
        # values and log-probabilities; the carried state in and out once
        nbytes += T * E * A * 8 + 2 * E * A * 2 * P * 4 + 2 * (D * H + 2 * (H * F + 2 * F * F)) + 16 * P * H
        return dict(bytes=nbytes, flops=(T + 1) * E * A * row_flops)
    rows = T * E * (1 if case["env"].startswith("hn") else A)  # Hanabi: only the mover's policy runs
    if case["op"] == "ac":
        nbytes += T * E * A * (8 + 4 + 8) + T * E * 5  # values, log pi; the estimate reads and writes
    return dict(bytes=nbytes + weights * (POPULATION if case["op"] == "pop" else 1), flops=rows * row_flops)


def tolerance(case):
    if case["op"] == "step":
        return "exact"  # whole-number env dynamics; the reward is one IEEE division
    if case["op"] == "policy":
        # bf16: the hidden activations are rounded to bf16 (measured 2.0e-3 .. 2.6e-3 against float64);
        # float32: sums of up to 192 products
        return {"rel": 1e-2, "max": 5e-2} if case["dtype"] == "bf16" else {"rel": 5e-6, "max": 5e-5}
    # A rollout feeds its sampled actions back, so one differing action changes all that follows in its env:
    # the same sums in the same order give the same bits, and only the float32 outputs that nothing is
    # sampled from (values, log-probabilities, advantages) have room for another order of a sum.
    return {"rel": 1e-5, "max": 1e-4, "differ": 1e-4}


def exact(case, seed):
    """Float64 logits of op "policy"; the other outputs hang on a sampled trajectory or are whole numbers."""
    if case["op"] != "policy":
        return None
    ws, bs, obs, legal = _policy_inputs(case, seed)
    out = []
    for part in torch.split(obs, 1 << 15):
        x = part.double()
        for l in range(3):
            x = x @ ws[l].double().T + bs[l].double()
            if l < 2:
                x = torch.tanh(x)
        out.append(x)
    logits = torch.cat(out)
    return logits if legal is None else logits.masked_fill(legal == 0, float("-inf"))
