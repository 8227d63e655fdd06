"""What a user of this library has it do, as cases to be timed and compared.

A case is one call of a training (or evaluation) loop -- `step`, `rollout`, `step_decoupled` -- on an agent of
a given environment, network, batch and unroll length:

    call        "step" (unroll + update), "rollout" (acting alone), "decoupled" (actor beside a V-trace learner)
    env         "catch", "pendulum" or "maze"; rows, cols: the board; max_steps: the episode's length
    hidden      widths of the hidden layers, "256-256"
    dtype       "fp32" or "bf16"
    B, T        environments and interactions per unroll
    lam         lambda of the returns
    updates     Adam updates per unroll; sequential: each chunk's gradient at the parameters as they are by then
    pathwise    policy gradient through the pendulum's dynamics

The five `*_step` cases named like a workload are the repository's own configurations; the others take the same
environments to the options, board sizes, widths and batch sizes beside them.
"""
import math

import numpy as np
import torch

from paper_2104_06272_amd import binding, workloads

DEVICE = "cuda:0"


def _case(name, workload=None, **over):
    c = dict(call="step", updates=1, sequential=False, pathwise=False)
    if workload:
        w = workloads.get(workload)
        c.update(env=w["env"]["kind"], rows=w["env"]["rows"], cols=w["env"]["cols"], max_steps=w["env"]["max_steps"],
                 hidden="-".join(str(x) for x in w["net"]["hidden"]), dtype=w["net"]["dtype"], B=w["B"], T=w["T"],
                 lam=w["net"]["lambda"])
    c.update(over)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a debugging-size run: one small agent whose step is all latency
        _case("catch_small_step", "catch_small"),
        # the headline configuration: grid-world agent, a few thousand environments on one device
        _case("catch_4096_step", "catch_4096"),
        # continuous control with lambda-returns
        _case("pendulum_8192_step", "pendulum_8192"),
        # the largest agent: bf16 layers, a maze per environment
        _case("maze_16384_step", "maze_16384"),
        # throughput with a tiny network: hundreds of thousands of environments
        _case("catch_262144_step", "catch_262144"),
        # a maze of another size in full precision, a batch and an unroll that are no powers of two
        _case("maze_fp32_odd_step", env="maze", rows=9, cols=13, max_steps=128, hidden="128-64", dtype="fp32", B=1040, T=23, lam=0.95),
        # a narrow bf16 policy for control, an ordinary batch
        _case("pendulum_bf16_step", "pendulum_8192", hidden="128-128", dtype="bf16", B=1024),
        # layers of different widths, a batch that is a multiple of 16 only
        _case("catch_wide_ragged_step", "catch_4096", hidden="512-256", B=2000, T=15),
        # actor and learner side by side, off-policy by one update
        _case("catch_4096_decoupled", "catch_4096", call="decoupled"),
        # the gradient taken through the environment
        _case("pendulum_8192_pathwise", "pendulum_8192", pathwise=True),
        # four minibatch updates per unroll, each at the parameters the one before left
        _case("pendulum_minibatch_step", "pendulum_8192", hidden="128-128", B=2048, updates=4, sequential=True),
        # evaluating a policy on a larger board: acting alone, three layers
        _case("catch_eval_rollout", "catch_4096", call="rollout", rows=13, cols=7, max_steps=12, hidden="256-128-64", B=1008, T=24),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        env = rng.choice(["catch", "catch", "pendulum", "pendulum", "maze"])
        dtype = "bf16" if rng.random() < 0.35 else "fp32"
        layers = rng.choice([1, 2, 2, 2, 3])
        widths = [64, 128, 256, 512] if layers > 1 else [32, 64, 128, 256]
        if rng.random() < 0.5:                               # most users give every layer one width
            hidden = [rng.choice(widths)] * layers
        else:
            hidden = [rng.choice(widths) for _ in range(layers)]
        if dtype == "bf16":                                  # what bf16 is for: layers wide enough for the matrix cores
            hidden = [max(128, h) for h in hidden]
        c = _case(None, env=env, dtype=dtype, lam=rng.choice([1.0, 0.95, 0.9]))
        # powers of two and multiples of 64 are the usual batches; any multiple of 16 is allowed
        B = _log_int(rng, 16, 65536)
        quantum = rng.choice([16, 64, 64])
        c["B"] = max(quantum, B // quantum * quantum)
        c["T"] = _log_int(rng, 4, 64)
        if env == "catch":
            c["rows"], c["cols"] = rng.choice([(10, 5), (10, 5), (rng.randint(5, 16), rng.randint(3, 12))])
            c["max_steps"] = c["rows"] - 1
        elif env == "maze":
            c["rows"], c["cols"] = rng.choice([(16, 16), (8, 8), (rng.randint(5, 16), rng.randint(5, 16))])
            c["max_steps"] = rng.choice([64, 128, 256])
        else:
            c["rows"], c["cols"], c["max_steps"] = 0, 0, 200
        kind = rng.random()
        if kind < 0.15:
            c["call"] = "rollout"
        elif kind < 0.30:
            c["call"] = "decoupled"
        elif kind < 0.42:
            c["updates"] = rng.choice([2, 4])
            c["sequential"] = rng.random() < 0.5
            c["T"] = max(1, c["T"] // c["updates"]) * c["updates"]
        elif kind < 0.54 and env == "pendulum" and dtype == "fp32":
            hidden = [rng.choice([64, 128, 256])] * 2
            c["pathwise"] = True
        c["hidden"] = "-".join(str(h) for h in hidden)
        if _cost(c) <= _cost(_case(None, "maze_16384")) and c["B"] * c["T"] <= 1 << 22 and _accepted(c):
            return c


def _config(c):
    net = dict(workloads.CONFIGS["catch_small"]["net"])      # the hyper-parameters all workloads share
    net.update(hidden=[int(x) for x in c["hidden"].split("-")], dtype=c["dtype"],
               policy="tanh_gaussian" if c["env"] == "pendulum" else "categorical")
    net["lambda"] = c["lam"]
    env = dict(kind=c["env"], rows=c["rows"], cols=c["cols"], max_steps=c["max_steps"], p_wall=0.2 if c["env"] == "maze" else 0.0)
    return dict(env=env, net=net, B=c["B"], T=c["T"])


def _accepted(c):
    """Whether the library takes the shape; several updates go with batches that cut into whole row groups."""
    if c["updates"] > 1 and (c["B"] % (256 if c["dtype"] == "bf16" else 64) or c["B"] * c["T"] // c["updates"] < 1024):
        return False
    return binding.workspace_bytes(_config(c)) > 0


class _State:
    pass


def _f32(ws, off, n):
    return ws[off:off + 4 * n].view(torch.float32)


def prepare(c, seed):
    """An agent in the middle of training: parameters of the seed, moments of earlier gradients, environments inside
    their episodes."""
    cfg = _config(c)
    g = binding.Anakin(cfg, seed=seed, device=DEVICE)
    rng = np.random.default_rng([seed, 2104])
    B, T, P = g.B, g.T, g.P
    if c["updates"] > 1:
        g.set_updates_per_unroll(c["updates"], sequential=c["sequential"])
    if c["pathwise"]:
        g.set_policy_gradient(binding.PG_PATHWISE)
    theta = g.get_params()
    m = (1e-4 * rng.standard_normal(P)).astype(np.float32)
    v = (1e-6 * rng.uniform(0.1, 1.0, P)).astype(np.float32)

    si = np.zeros((B, 4), np.int32)
    sf = np.zeros((B, 2), np.float32)
    if c["env"] == "catch":
        si[:, 0] = rng.integers(0, c["cols"], B)
        si[:, 1] = rng.integers(0, c["rows"] - 1, B)
        si[:, 2] = rng.integers(0, c["cols"], B)
    elif c["env"] == "pendulum":
        si[:, 0] = rng.integers(0, c["max_steps"], B)
        sf[:, 0] = rng.uniform(-3.1, 3.1, B)
        sf[:, 1] = rng.uniform(-2.0, 2.0, B)
    else:
        cells = c["rows"] * c["cols"]
        walls = g.get_walls()
        cell = rng.integers(0, cells - 1, B)
        blocked = (walls[np.arange(B), cell >> 5] >> (cell & 31).astype(np.uint32)) & 1
        si[:, 0] = np.where(blocked, 0, cell)
        si[:, 1] = rng.integers(0, c["max_steps"] // 2, B)

    def place(step):
        g.set_params(theta)
        g.set_opt_state(m, v, 100)
        g.set_env_state(si, sf)
        g.global_step = step

    start = 1000 * T
    place(start)
    s = _State()
    s.g = g
    # The workspace is the caller's memory: the outputs of a call stay in it.  theta, gradient and the two moments
    # stand at its beginning, on multiples of 256 bytes; the trajectory where the library says.
    pitch = (4 * P + 255) // 256 * 256
    own = {name: _f32(g.ws, k * pitch, P) for k, name in enumerate(("theta", "grad", "m", "v"))}
    for name, want in (("theta", theta), ("m", m), ("v", v)):
        if not np.array_equal(own[name].cpu().numpy(), want):
            raise RuntimeError("the workspace does not begin with theta, gradient, m and v")

    def views():
        t = binding.TrajView()
        g._chk(g.L.anakin_get_trajectory(g.h, t))

        def at(off, rows, dtype, width=None):
            n = rows * B * (width or 1) * dtype.itemsize
            x = g.ws[off:off + n].view(dtype)
            return x.view(rows, B) if width is None else x.view(rows, B, width)

        o = {"state": at(t.off_state_s0, T + 1, torch.int32), "reward": at(t.off_reward, T, torch.float32),
             "done": at(t.off_done, T, torch.uint8), "value": at(t.off_value, T + 1, torch.float32),
             "head": at(t.off_head, T + 1, torch.float32, t.head_stride)[:, :, :t.num_heads]}
        if c["env"] == "pendulum":
            o.update(theta_t=at(t.off_state_f0, T + 1, torch.float32), theta_dot=at(t.off_state_f1, T + 1, torch.float32),
                     noise=at(t.off_eps, T, torch.float32), action=at(t.off_action_f, T, torch.float32))
        else:
            o["action"] = at(t.off_action, T, torch.uint8)
        if c["call"] != "rollout":
            o.update(adv=at(t.off_adv, T, torch.float32), ret=at(t.off_ret, T, torch.float32), **own)
        return o

    if c["call"] == "decoupled":
        # two record sets take turns: one unroll is stored before the first call, and the learner starts from the
        # parameters that collected it
        g.rollout()
        first = views()
        g.step_decoupled()
        second = views()
        place(start + 2 * T)
        s.outputs, s.turn = (first, second), 0
    else:
        s.outputs, s.turn = (views(),), 0
    s.call = {"step": g.step, "rollout": g.rollout, "decoupled": g.step_decoupled}[c["call"]]
    return s


def run(s):
    s.call()
    out = s.outputs[s.turn]
    s.turn = (s.turn + 1) % len(s.outputs)
    return out


def _shape(c):
    """(multiply-adds per sample between hidden layers and in the heads, width of the first layer, parameters, head
    outputs, first-layer rows read per sample)"""
    h = [int(x) for x in c["hidden"].split("-")]
    A = {"catch": 3, "pendulum": 2, "maze": 4}[c["env"]]
    D = {"catch": c["rows"] * c["cols"], "pendulum": 3, "maze": 3 * c["rows"] * c["cols"]}[c["env"]]
    NH = A + 1
    mid = sum(a * b for a, b in zip(h, h[1:]))
    P = D * h[0] + h[0] + sum(a * b + b for a, b in zip(h, h[1:])) + h[-1] * NH + NH
    return mid, h[-1] * NH, h[0], P, NH, {"catch": 2, "pendulum": 3, "maze": 1}[c["env"]]


def work(c):
    mid, heads, H1, P, NH, rows = _shape(c)
    B, T = c["B"], c["T"]
    M = B * T
    forward = 2.0 * (mid + heads + rows * H1)
    flops = forward * B * (T + 1)
    if c["env"] == "maze":                                   # the walls of a maze are the same all through the unroll
        flops += 2.0 * B * 0.2 * c["rows"] * c["cols"] * H1
    state = 4 if c["env"] != "pendulum" else 12
    action = 1 if c["env"] != "pendulum" else 8
    bits = c["rows"] * c["cols"] / 8 if c["env"] == "maze" else 0
    n_bytes = 4.0 * P + B * (2 * state + bits) + B * (T + 1) * (state + 4 + 4 * NH) + M * (action + 5)
    if c["call"] != "rollout":
        # both products of every layer but the first, which has no gradient of its input to form
        flops += M * (4.0 * mid + 4.0 * heads + 2.0 * rows * H1)
        if c["env"] == "maze":
            flops += 2.0 * B * 0.2 * c["rows"] * c["cols"] * H1
        n_bytes += 4.0 * P * 6 + M * 8.0
        if c["pathwise"]:                                    # the adjoint's own way back through the network
            flops += M * 2.0 * (mid + rows * H1)
        if c["call"] == "decoupled":                         # the learner's forward pass over the stored unroll
            flops += forward * B * (T + 1)
            n_bytes += B * (T + 1) * (state + 4 + 4 * NH) + M * (action + 5)
        if c["updates"] > 1:
            n_bytes += 4.0 * P * 6 * (c["updates"] - 1)
            if c["sequential"]:                              # every chunk but the first is evaluated anew
                flops += forward * M * (c["updates"] - 1) / c["updates"]
    return {"bytes": n_bytes, "flops": flops}


def _cost(c):
    """Rough relative cost of a case, for draw(): arithmetic at the type's rate plus memory traffic of the activations."""
    w = work(c)
    h = sum(int(x) for x in c["hidden"].split("-"))
    wide = 2 if c["dtype"] == "bf16" else 4
    return w["flops"] / (2.0e15 if c["dtype"] == "bf16" else 1.3e14) + (w["bytes"] + 4.0 * wide * h * c["B"] * c["T"]) / 5e12


def tolerance(c):
    # Acting in fp32 is bit for bit; the update's sums over samples may be taken in another order.  bf16 layers round
    # every activation to eight bits of significand, and an action drawn on the edge may fall to the other side.
    if c["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.5, "differ": 2e-3}
    return {"rel": 2e-5, "max": 1e-3}
