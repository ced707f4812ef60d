"""What a program built on this framework spends its GPU time on, as cases that can be timed.

The work comes in five kinds, one per way the library is called:

  predict   one batch of states through ``Ga3c.predict`` (the predictor of Sec. 4.1): policy, value and sampled action
  train     one update on N agents x t_max steps through ``Ga3c.train_step`` (the trainer of Sec. 4.1)
  ragged    one update on segments of unequal length (episodes that ended) through ``Ga3c.train_step_ragged``
  step      the balanced pipeline of Sec. 4.2: t_max predictions of all agents on one stream, an update on another
  sched     a closed loop of agents through ``Scheduler``: requests, results, segments and the updates made of them

Networks: the small net of Sec. 3.2, the larger net of the workload list (three conv layers, fc 512) and the paper's
larger-network family of Sec. 5 (conv1 stride 4, 3, 2 or 1).  ``math`` 0 is fp32 accuracy, 1 rounds the operands of
every contraction to bfloat16.  Frames are game-like: rectangles on black that move a little from plane to plane, and
salt noise.
"""
from __future__ import annotations

import math as _math

import numpy as np
import torch

import paper_1611_06256_amd as g

T_MAX = 5
PLANES, SIDE = 4, 84
FRAME = PLANES * SIDE * SIDE


def _case(name, kind, net, n, actions=18, math=0):
    """``n``: frames of a prediction, agents (or segments) of everything else."""
    return {"name": name, "kind": kind, "net": net, "n": n, "actions": actions, "math": math}


def listed():
    return [
        # one state: an agent that plays alone, and the latency floor of a call
        _case("predict small 1", "predict", "small", 1),
        # whatever happens to be queued when a predictor looks: an odd handful
        _case("predict small 37", "predict", "small", 37),
        # the largest batch of the prediction sweep
        _case("predict small 1024", "predict", "small", 1024),
        # the larger net's prediction batch
        _case("predict large 256", "predict", "large", 256),
        # the paper's fastest setting, 128 agents, on a member of its larger-network family (odd map widths)
        _case("predict paper3 128", "predict", "paper3", 128),
        # the smallest update: 8 agents with Pong's six actions
        _case("train small 8x5", "train", "small", 8, actions=6),
        # an update in which a good part of the episodes ended early
        _case("ragged small 128", "ragged", "small", 128),
        # the headline workload: 512 agents, five predictions each and one update of 2560 frames, on two streams
        _case("step small 512", "step", "small", 512),
        # the larger net's update in both arithmetics
        _case("train large 256x5", "train", "large", 256),
        _case("train large 256x5 bf16", "train", "large", 256, math=1),
        # the largest network of the paper (conv1 stride 1, fc 1024), 128 agents
        _case("train paper1 128x5", "train", "paper1", 128),
        # 256 agents in lockstep through the two queues
        _case("sched small 256", "sched", "small", 256),
    ]


# Largest n that a network of each kind is run with.
_MOST = {
    "predict": {"small": 1024, "large": 512, "paper4": 256, "paper3": 256, "paper2": 256, "paper1": 256},
    "train": {"small": 512, "large": 256, "paper4": 128, "paper3": 128, "paper2": 128, "paper1": 128},
    "ragged": {"small": 512, "large": 256, "paper4": 128, "paper3": 128, "paper2": 128, "paper1": 128},
    "step": {"small": 512, "large": 256},
    "sched": {"small": 256, "large": 256},
}


def draw(rng):
    kind = rng.choice(["predict", "predict", "predict", "train", "train", "ragged", "step", "sched"])
    net = rng.choice([k for k in ("small", "small", "small", "large", "large", "paper4", "paper3", "paper2", "paper1")
                      if k in _MOST[kind]])
    least, most = (16 if kind in ("step", "sched") else 1), _MOST[kind][net]
    n = round(_math.exp(rng.uniform(_math.log(least), _math.log(most))))
    c = _case("", kind, net, max(least, min(most, n)), actions=rng.randint(3, 18),
              math=0 if kind == "sched" else int(rng.random() < 0.25))
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs --

def _desc(case):
    net, a = case["net"], case["actions"]
    if net == "small":
        d = g.SMALL_NET(a)
    elif net == "large":
        d = g.LARGE_NET(a)
    else:
        stride = int(net[len("paper"):])
        d = g.NetDesc(conv=((32, 8, stride), (32, 4, 2), (64, 4, 2)), fc_units=1024 if stride == 1 else 256, n_actions=a)
    d.math = case["math"]
    return d


def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _frames(n, gen):
    """n stacks of four planes: 3 to 12 rectangles, each shifted a little in every plane, and 2 % salt."""
    def ints(lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=gen, device="cuda")

    out = torch.zeros(n, PLANES, SIDE, SIDE, dtype=torch.uint8, device="cuda")
    count = ints(3, 13, n)
    at = torch.arange(SIDE, device="cuda")
    for k in range(12):
        inside = []
        for _ in range(2):                        # rows, then columns
            lo = ints(0, SIDE - 2, n, 1) + ints(-2, 3, n, PLANES)
            hi = lo + ints(2, 32, n, 1)
            inside.append((at >= lo[..., None]) & (at < hi[..., None]))
        drawn = inside[0][..., :, None] & inside[1][..., None, :] & (count > k)[:, None, None, None]
        out = torch.where(drawn, ints(1, 256, n).to(torch.uint8)[:, None, None, None], out)
    salt = torch.rand(out.shape, generator=gen, device="cuda") < 0.02
    return out.masked_fill_(salt, 255)


def _rewards(gen, *shape):
    u = torch.rand(*shape, generator=gen, device="cuda")
    return (u >= 0.95).float() - (u < 0.05).float()


def _answers(n, actions, gen):
    """Uniforms for the draw and the tensors that a prediction fills."""
    return {"uniforms": torch.rand(n, generator=gen, device="cuda"),
            "logits": torch.empty(n, actions, device="cuda"), "values": torch.empty(n, device="cuda"),
            "probs": torch.empty(n, actions, device="cuda"),
            "actions": torch.empty(n, dtype=torch.int32, device="cuda")}


def _results(net):
    """Where an update's results are read out to."""
    return {k: torch.empty(net.n_params, device="cuda") for k in ("theta", "g", "grad")}


def _lengths(n, seed):
    """Steps per segment: t_max, or fewer where the episode ended (three in ten)."""
    r = np.random.default_rng(seed)
    return np.where(r.random(n) < 0.3, r.integers(1, T_MAX, size=n), T_MAX).astype(np.int32)


def prepare(case, seed):
    kind, n, a = case["kind"], case["n"], case["actions"]
    gen = _rng(seed)
    s = {"kind": kind, "hp": g.HParams(clip_norm=40.0)}
    if kind == "predict":
        s["net"] = g.Ga3c(_desc(case), n, 0)
        s["frames"] = _frames(n, gen)
        s["answers"] = _answers(n, a, gen)
    elif kind == "train":
        s["net"] = net = g.Ga3c(_desc(case), n, n * T_MAX)
        s["batch"] = (_frames(n * T_MAX, gen).view(n, T_MAX, PLANES, SIDE, SIDE),
                      torch.randint(0, a, (n, T_MAX), dtype=torch.int32, generator=gen, device="cuda"),
                      _rewards(gen, n, T_MAX),
                      (torch.rand(n, T_MAX, generator=gen, device="cuda") < 0.02).to(torch.uint8),
                      torch.randn(n, generator=gen, device="cuda"))
        s["results"] = _results(net)
        s["stats"] = torch.zeros(8, device="cuda")
    elif kind == "ragged":
        lens = _lengths(n, seed)
        start = np.zeros(n + 1, np.int32)
        np.cumsum(lens, out=start[1:])
        total = int(start[-1])
        dones = np.zeros(total, np.uint8)
        dones[start[1:][lens < T_MAX] - 1] = 1
        s["net"] = net = g.Ga3c(_desc(case), n, n * T_MAX)
        s["batch"] = (_frames(total, gen),
                      torch.randint(0, a, (total,), dtype=torch.int32, generator=gen, device="cuda"),
                      _rewards(gen, total), torch.from_numpy(dones).cuda(), torch.from_numpy(start).cuda(),
                      torch.randn(n, generator=gen, device="cuda"))
        s["results"] = _results(net)
        s["stats"] = torch.zeros(8, device="cuda")
    elif kind == "step":
        s["net"] = net = g.Ga3c(_desc(case), n, n * T_MAX)
        s["shown"] = [_frames(n, gen) for _ in range(T_MAX)]         # what the agents see in this pass
        s["answers"] = [_answers(n, a, gen) for _ in range(T_MAX)]
        s["batch"] = (_frames(n * T_MAX, gen).view(n, T_MAX, PLANES, SIDE, SIDE),    # their segment before that
                      torch.randint(0, a, (n, T_MAX), dtype=torch.int32, generator=gen, device="cuda"),
                      _rewards(gen, n, T_MAX),
                      (torch.rand(n, T_MAX, generator=gen, device="cuda") < 0.02).to(torch.uint8))
        s["results"] = _results(net)
        s["stats"] = torch.zeros(8, device="cuda")
        s["streams"] = torch.cuda.Stream(), torch.cuda.Stream()
        s["told"] = torch.cuda.Event()
    else:
        s["net"] = net = g.Ga3c(_desc(case), n, n * T_MAX)
        s["sched"] = g.Scheduler(net, s["hp"], t_max=T_MAX, predict_cap=n, train_min=min(40, n * T_MAX), train_cap=n * T_MAX)
        s["frames"] = _frames(n * T_MAX, gen)                         # [agent][step]
        r = np.random.default_rng(seed)
        s["agents"] = np.arange(n, dtype=np.int32)
        s["first"] = np.uint64(s["frames"].data_ptr()) + np.arange(n, dtype=np.uint64) * np.uint64(T_MAX * FRAME)
        s["uniforms"] = r.random((T_MAX, n), dtype=np.float32)
        u = r.random((n, T_MAX))
        s["rewards"] = (u >= 0.95).astype(np.float32) - (u < 0.05).astype(np.float32)
        s["dones"] = (r.random((n, T_MAX)) < 0.02).astype(np.uint8)
        s["results"] = _results(net)
    s["net"].params_init(seed)
    torch.cuda.synchronize()
    return s


# --------------------------------------------------------------- the passes --

def _read_out(s, stream=None):
    net, out = s["net"], s["results"]
    net.params_get(0, out["theta"], stream=stream)
    net.params_get(1, out["g"], stream=stream)
    net.params_get(2, out["grad"], stream=stream)
    return out


def _shown(answers):
    return {k: answers[k] for k in ("logits", "values", "probs", "actions")}


def _run_step(s):
    net, (sp, st) = s["net"], s["streams"]
    for k in range(T_MAX):
        net.predict(s["shown"][k], stream=sp, **s["answers"][k])
        if k == 0:
            s["told"].record(sp)
    st.wait_event(s["told"])       # the value after a segment is the one told by the first prediction after it
    net.train_step(*s["batch"], s["answers"][0]["values"], s["hp"], stats=s["stats"], stream=st)
    done = _read_out(s, st)
    sp.wait_stream(st)             # the next pass's first prediction writes what this update reads
    return {"told": [_shown(x) for x in s["answers"]], "update": done, "stats": s["stats"][:5]}


def _run_sched(s):
    sched, agents, n = s["sched"], s["agents"], len(s["agents"])
    acts = np.empty((n, T_MAX), np.int32)
    values = np.empty((n, T_MAX), np.float32)
    version = None
    for k in range(T_MAX):
        sched.submit_predict_many(agents, s["first"] + np.uint64(k * FRAME), s["uniforms"][k])
        sched.tick()
        got = 0
        while got < n:
            who, act, val, ver = sched.poll_arrays(with_version=True)
            acts[who, k], values[who, k] = act, val
            if k == 0 and who.size:
                version = np.full(n, ver[0], np.int64)
            got += who.size
    sched.submit_segment_many(agents, s["first"], np.full(n, T_MAX, np.int32), acts, s["rewards"], s["dones"],
                              values[:, 0].copy(), version)
    sched.tick()
    return {"actions": acts, "values": values, "update": _read_out(s)}


def run(s):
    kind = s["kind"]
    if kind == "predict":
        s["net"].predict(s["frames"], **s["answers"])
        return _shown(s["answers"])
    if kind == "train":
        s["net"].train_step(*s["batch"], s["hp"], stats=s["stats"])
        return {"update": _read_out(s), "stats": s["stats"][:5]}
    if kind == "ragged":
        s["net"].train_step_ragged(*s["batch"], s["hp"], stats=s["stats"])
        return {"update": _read_out(s), "stats": s["stats"][:5]}
    return _run_step(s) if kind == "step" else _run_sched(s)


# ------------------------------------------------------- what a pass takes --

def _network(case):
    """Multiply-adds of a frame forward and of its first layer, and the number of parameters."""
    d = _desc(case)
    c, h, macs, params, first = d.in_c, d.in_h, 0, 0, 0
    for oc, k, st in d.conv:
        h = (h - k) // st + 1
        macs += oc * c * k * k * h * h
        params += oc * (c * k * k + 1)
        first = first or macs
        c = oc
    flat = c * h * h
    macs += flat * d.fc_units + d.fc_units * (d.n_actions + 1)
    params += (flat + 1) * d.fc_units + (d.fc_units + 1) * (d.n_actions + 1)
    return macs, first, params


def work(case):
    kind, n, a = case["kind"], case["n"], case["actions"]
    macs, first, params = _network(case)
    predict = {"bytes": n * (FRAME + 4 * (2 * a + 3)), "flops": 2 * n * macs}
    if kind == "predict":
        return {"bytes": predict["bytes"] + 4 * params, "flops": predict["flops"]}
    frames = n * T_MAX if kind != "ragged" else n * T_MAX * 3 // 4 + n // 10      # three in ten are half as long
    # forward, and both gradients of every layer but the first, whose input needs none; theta and g are read and
    # written, and they and the gradient are handed out
    update = {"bytes": frames * (FRAME + 9) + 4 * n + 4 * params * 7, "flops": 2 * frames * (3 * macs - first)}
    if kind in ("train", "ragged"):
        return update
    return {k: T_MAX * predict[k] + update[k] for k in ("bytes", "flops")}


def tolerance(case):
    if case["math"]:
        # operands are bfloat16: a value on the edge between two of them may fall either way
        return {"rel": 1e-2, "max": 0.3, "differ": 0.01}
    if case["kind"] == "predict":
        return {"rel": 1e-5, "max": 2e-4, "differ": 0.002}
    # sums of 32-bit products through several layers; a pre-activation within rounding of zero may be cut off or not
    return {"rel": 5e-5, "max": 5e-3, "differ": 0.002}
