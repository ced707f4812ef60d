"""Kernels whose operands are two float16 terms each (split_f16.hpp): sizes at which their work is split differently, and
values that float16 does not hold unscaled."""
import numpy as np
import pytest

import ga3c_synth as synth
import oracle as orc
import test_gpu_parity as P

pytestmark = pytest.mark.gpu

# A sum of n products carries about sqrt(n / 32) roundings of 2^-24 of itself, two terms leave 2^-23 of an operand at most: below 1e-6
# for the 256 to 3136 products of a layer here, five layers one after the other.
TOL = 5e-6


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_1611_06256_amd as g
    assert torch.cuda.is_available()
    return g


def scaled(net, theta, layer, power):
    """Layer `layer` (from 1) times 2^power, the next one divided by it: the same network, other sizes in between."""
    theta, off = theta.copy(), net.offsets()

    def times(name, p):
        at, shape = off[name]
        theta[at:at + int(np.prod(shape))] *= np.float32(2.0 ** p)

    times(f"conv{layer}.W", power)
    times(f"conv{layer}.b", power)
    times(f"conv{layer + 1}.W" if f"conv{layer + 1}.W" in off else "fc.W", -power)
    return theta


def network(G, which, A):
    if which == "small":
        return G.SMALL_NET(A)
    return G.LARGE_NET(A) if which == "large" else G.NetDesc(conv=((32, 8, int(which[-1])), (32, 4, 2), (64, 4, 2)), fc_units=256, n_actions=A)


# one, two and three frames a block; activations beyond float16's largest number and below its smallest; a filter of zeros
@pytest.mark.parametrize("which,B,layer,power",
                         [(which, *c) for which in ("large", "paper4", "paper3") for c in
                          [(1, 1, 0), (256, 1, 0), (257, 1, 0), (513, 1, 0), (3, 1, 30), (3, 1, -30), (3, 2, 30), (3, 2, -30), (3, 3, 30), (3, 3, -40)]] +
                         [("small", *c) for c in [(65, 1, 0), (256, 1, 0), (257, 1, 0), (515, 1, 0), (1025, 1, 0), (67, 1, 30), (67, 1, -30), (67, 2, 30), (67, 2, -40)]])
def test_predictions_with_the_convolutions_in_one_kernel(G, which, B, layer, power):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9100 + B)
    theta = scaled(net, theta, layer, power)
    at, shape = net.offsets()[f"conv{layer}.W"]
    theta[at:at + int(np.prod(shape[1:]))] = 0
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9101 + B, B)
    if power:
        frames[0] = 0
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    assert P.rel_err(lg, ref["logits"]) <= TOL and P.rel_err(vl, ref["values"]) <= TOL
    net.close()


# Weights that two terms of one scale do not hold: a single huge one per layer, whose output the rectifier cuts off where the input is not
# zero; a channel of other sizes, which the next layer's weights undo
@pytest.mark.parametrize("which,B,what", [(n, b, w) for n, b in (("large", 2), ("paper4", 2), ("paper3", 258), ("small", 67))
                                          for w in ("huge", "channel 1", "channel 2") if n != "small" or w != "channel 2"])
def test_predictions_with_weights_far_apart(G, which, B, what):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9150 + B)
    if what == "huge":
        for name, (at, shape) in net.offsets().items():
            if name.startswith("conv") and name.endswith(".W"):
                theta[at + int(np.prod(shape)) // 3] = -3.4e38
    else:
        l = int(what[-1])
        v = orc.views(onet, theta)
        for name, part, p in ((f"conv{l}.W", np.s_[3], 24), (f"conv{l}.b", np.s_[3], 24), (f"conv{l + 1}.W", np.s_[:, 3], -24)):
            w = v[name].copy()
            w[part] *= np.float32(2.0 ** p)
            at = net.offsets()[name][0]
            theta[at:at + w.size] = w.ravel()
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9151 + B, B)
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    assert np.isfinite(ref["logits"]).all() and P.rel_err(lg, ref["logits"]) <= TOL and P.rel_err(vl, ref["values"]) <= TOL
    net.close()


# The small net's filters for predictions follow every update, a filter per wavefront of the kernel that updates the parameters: the
# same bits as in a context that was given those parameters.  The second network ends soon behind the filters (3113 vectors of four).
@pytest.mark.parametrize("conv,F", [(((16, 8, 4), (32, 4, 2)), 256), (((16, 8, 4), (32, 4, 2), (1, 1, 1)), 1)])
def test_predictions_read_the_filters_that_an_update_leaves(G, conv, F):
    import torch
    A, B, N = 3, 70, 6
    desc = G.NetDesc(conv=conv, fc_units=F, n_actions=A)
    net, other = G.Ga3c(desc, B, 5 * N), G.Ga3c(desc, B, 0)
    net.params_init(9201)
    frames = torch.from_numpy(synth.uniform_frames(9202, (B, 4, 84, 84))).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9203, N, 5, A).items()}
    u = torch.from_numpy(synth.uniforms(9204, B)).cuda()

    def told(n):
        o = dict(logits=torch.full((B, A), float("nan"), device="cuda"), values=torch.full((B,), float("nan"), device="cuda"))
        n.predict(frames, uniforms=u, **o)
        return o

    before = told(net)
    for step in range(2):
        net.train_step(frames[:5 * N].view(N, 5, 4, 84, 84), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.05))
        theta = net.params_get(0).clone()
        other.params_set(theta, 0)
        got, want = told(net), told(other)
        torch.cuda.synchronize()
        for k in want:
            assert torch.isfinite(want[k]).all() and not torch.equal(want[k], before[k]) and torch.equal(got[k], want[k]), (step, k)
    net.close(); other.close()


# Gradients, whose operands are scaled by what a block has met so far: one frame a block and several, rewards (and with them gradients) of
# very different sizes in one block, a layer whose map is zero.  Each layer on its own, from the tensors that the update has left, in 64
# bits: sums of n products carry sqrt(n / 32) roundings of 2^-24 of the running sum, observed 3e-7 of the result at most.
@pytest.mark.parametrize("which,N,spread,dead", [(w, *c) for w in ("small", "large", "paper4") for c in [(1, 0, 0), (157, 0, 0), (160, 6, 0), (40, 0, 1)]])
def test_gradients_of_the_convolutions(G, which, N, spread, dead):
    import torch
    A, T = 6, 5
    B = N * T
    net, onet, theta = P.make(G, network(G, which, A), 1, B, 9300 + N)
    off = net.offsets()
    if dead:
        at, shape = off["conv1.b"]
        theta[at:at + int(np.prod(shape))] = -50
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9301 + N, B).reshape(B, 4, 84, 84)
    tr = synth.trajectories(9302 + N, N, T, A)
    sizes = np.float32(10.0) ** np.random.default_rng(9303).uniform(-spread, spread, N).astype(np.float32)
    rewards = (tr["rewards"] + np.float32(0.5)) * sizes[:, None]
    net.train_step(torch.from_numpy(frames).cuda().view(N, T, 4, 84, 84), torch.from_numpy(tr["actions"]).cuda(), torch.from_numpy(rewards).cuda(),
                   torch.from_numpy(tr["dones"]).cuda(), None, G.HParams())

    def get(which, *shape):
        return net.train_debug_get(which, torch.empty(int(np.prod(shape)), device="cuda")).cpu().double().view(shape)

    def close(got, want, what):
        assert torch.isfinite(got).all() and float((got - want).norm()) <= 1e-6 * float(want.norm()), what

    x, grad = torch.from_numpy(frames).double() / 255, net.params_get(2).cpu().double()
    conv = onet.conv
    for l, (oc, k, s) in enumerate(conv):
        oh = (x.shape[-1] - k) // s + 1
        y, dy = get(4 + l, B, oc, oh, oh), get(10 + l, B, oc, oh, oh)
        at, shape = off[f"conv{l + 1}.W"]
        n = int(np.prod(shape))
        close(grad[at:at + n].view(*shape), torch.nn.grad.conv2d_weight(x, tuple(shape), dy, stride=s), f"conv{l + 1}.W")
        at_b = off[f"conv{l + 1}.b"][0]
        close(grad[at_b:at_b + oc], dy.sum((0, 2, 3)), f"conv{l + 1}.b")
        if l:
            w = torch.from_numpy(theta[at:at + n]).double().view(*shape)
            close(get(10 + l - 1, *x.shape), torch.nn.grad.conv2d_input(x.shape, w, dy, stride=s) * (x > 0), f"input of conv{l + 1}")
        x = y
    net.close()


# The first layer's weight gradient where a block takes all 32 filters of a frame (more than 128 frames) and where it takes 16, in both
# arithmetics; with rounded operands its sums are of bytes times dY rounded to bfloat16, products that are exact in fp32.  Bound as above.
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("which,N", [("large", 128), ("large", 129), ("large", 515), ("small", 257)])
def test_first_layers_weight_gradient(G, which, N, math):
    import torch
    A = 4
    desc = network(G, which, A)
    desc.math = math
    net = G.Ga3c(desc, 1, N)
    net.params_init(9400)
    frames = torch.from_numpy(synth.rectangle_frames(9401, N))
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9402, N, 1, A).items()}
    net.train_step(frames.cuda().view(N, 1, 4, 84, 84), tr["actions"], tr["rewards"] + 0.5, tr["dones"], None, G.HParams())
    oc = desc.conv[0][0]
    dy = net.train_debug_get(10, torch.empty((N, oc, 20, 20), device="cuda")).cpu()
    dy = (dy.bfloat16() if math else dy).double()
    grad, off = net.params_get(2).cpu().double(), net.offsets()
    for name, want in (("conv1.W", torch.nn.grad.conv2d_weight(frames.double(), (oc, 4, 8, 8), dy, stride=4) / 255), ("conv1.b", dy.sum((0, 2, 3)))):
        got = grad[off[name][0]:off[name][0] + want.numel()].view(want.shape)
        assert float((got - want).norm()) <= 1e-6 * float(want.norm()), name
    net.close()


def err2(x, y):
    return float(np.linalg.norm(np.asarray(x, np.float64) - y) / np.linalg.norm(y))


# Frames of which little is lit, and no bias that would cover it: a byte of 1 counts as much as one of 255.  Bound: five layers of 1e-6 each (TOL above), as norms add up.
@pytest.mark.parametrize("which,B", [("small", 67), ("large", 3), ("paper4", 3), ("paper3", 3)])
@pytest.mark.parametrize("what", [1, 3, 15, "dots"])
def test_predictions_of_dark_frames(G, which, B, what):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9120)
    for name, (at, shape) in net.offsets().items():
        if name.endswith(".b"):
            theta[at:at + int(np.prod(shape))] = 0
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    r = synth.rng(9121)
    if what == "dots":                 # six pixels of 1 or 2
        frames = np.zeros((B, 4 * 84 * 84), np.uint8)
        for b in range(B):
            frames[b, r.integers(0, 4 * 84 * 84, 6)] = r.integers(1, 3, 6)
        frames = frames.reshape(B, 4, 84, 84)
    else:
        frames = r.integers(0, what + 1, (B, 4, 84, 84)).astype(np.uint8)
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    e = err2(lg, ref["logits"]), err2(vl, ref["values"])
    print(f"dark {which} {what}: {e[0]:.2e} {e[1]:.2e}", flush=True)
    assert max(e) <= 2.5e-6
    net.close()


# A channel that the next layer does not look at, whose values lie far above all others: their scale is not its.  The first layer's bias, the
# second one's (the small net's second map stays fp32).  2^9: still one scale, in frames of zeros and ones too.
@pytest.mark.parametrize("which,B,layer", [("large", 2, 1), ("large", 2, 2), ("paper4", 2, 1), ("paper4", 2, 2), ("paper3", 258, 1), ("paper3", 2, 2),
                                           ("small", 67, 1)])
@pytest.mark.parametrize("power", [9, 14, 27])
def test_predictions_with_a_bias_that_nothing_reads(G, which, B, layer, power):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9130)
    at, _ = net.offsets()[f"conv{layer}.b"]
    theta[at + 5] = 2.0 ** power
    at, shape = net.offsets()[f"conv{layer + 1}.W"]
    w = theta[at:at + int(np.prod(shape))].reshape(shape)
    w[:, 5] = 0
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9131, B) >> (7 if power == 9 else 0)
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    e = err2(lg, ref["logits"]), err2(vl, ref["values"])
    print(f"bias {which} {layer} {power}: {e[0]:.2e} {e[1]:.2e}", flush=True)
    assert max(e) <= 2.5e-6
    net.close()


# Filters of few weights, of which the large ones meet nothing but zeros: what is left is as exact as any.
@pytest.mark.parametrize("which,B", [("large", 2), ("paper4", 2), ("paper3", 2), ("small", 67)])
@pytest.mark.parametrize("layer", [1, 2])
def test_predictions_with_few_weights_in_a_filter(G, which, B, layer):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9140)
    off = net.offsets()

    def tensor(name):
        at, shape = off[name]
        return theta[at:at + int(np.prod(shape))].reshape(shape)

    w = tensor(f"conv{layer}.W")
    if layer == 2:                     # channel 0 of the first map stays zero
        tensor("conv1.W")[0] = 0
        tensor("conv1.b")[0] = 0
    keep = w[:, 1, :2, :4].copy()
    w[:] = 0
    w[:, 1, :2, :4] = keep
    w[:, 0, 0, 0] = 2.0 ** 24
    tensor(f"conv{layer}.b")[:] = 0
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9141, B)
    frames[:, 0] = 0
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    e = err2(lg, ref["logits"]), err2(vl, ref["values"])
    print(f"few {which} {layer}: {e[0]:.2e} {e[1]:.2e}", flush=True)
    assert max(e) <= 2.5e-6
    net.close()


# Gradients of a network one of whose channels is 2^`power` times the others, which the next layer undoes: every filter's and every input
# channel's part has the error of a sum of fp32 products, not that of the largest.  Each layer from what the update left, in 64 bits; bound
# as in test_gradients_of_the_convolutions, for parts.
@pytest.mark.parametrize("which,N,layer", [(w, n, l) for w in ("small", "large", "paper4") for n in (1, 157) for l in (1, 2, 3) if w != "small" or l < 3])
@pytest.mark.parametrize("power", [24, -24])
def test_gradients_with_a_channel_of_another_size(G, which, N, layer, power):
    import torch
    A, T = 6, 5
    B = N * T
    net, onet, theta = P.make(G, network(G, which, A), 1, B, 9350 + N)
    off = net.offsets()

    def tensor(name, *shape):
        at, sh = off[name]
        return theta[at:at + int(np.prod(sh))].reshape(shape or sh)

    def times(part, p):
        part *= np.float32(2.0 ** p)

    times(tensor(f"conv{layer}.W")[3], power)
    times(tensor(f"conv{layer}.b")[3:4], power)
    if f"conv{layer + 1}.W" in off:
        times(tensor(f"conv{layer + 1}.W")[:, 3], -power)
    else:
        oc = onet.conv[layer - 1][0]
        times(tensor("fc.W", off["fc.W"][1][0], oc, -1)[:, 3], -power)
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9351 + N, B).reshape(B, 4, 84, 84)
    tr = synth.trajectories(9352 + N, N, T, A)
    print(f"gradients {which} N={N} layer={layer} power={power}", flush=True)
    net.train_step(torch.from_numpy(frames).cuda().view(N, T, 4, 84, 84), torch.from_numpy(tr["actions"]).cuda(),
                   torch.from_numpy(tr["rewards"] + np.float32(0.5)).cuda(), torch.from_numpy(tr["dones"]).cuda(), None, G.HParams())

    def get(which, *shape):
        return net.train_debug_get(which, torch.empty(int(np.prod(shape)), device="cuda")).cpu().double().view(shape)

    def worst(got, want, dim):
        other = [d for d in range(want.dim()) if d != dim]
        d, n = (got - want).pow(2).sum(other).sqrt(), want.pow(2).sum(other).sqrt()
        assert torch.isfinite(got).all()
        return float((d[n > 0] / n[n > 0]).max())

    x, grad, errors = torch.from_numpy(frames).double() / 255, net.params_get(2).cpu().double(), {}
    for l, (oc, k, s) in enumerate(onet.conv):
        oh = (x.shape[-1] - k) // s + 1
        y, dy = get(4 + l, B, oc, oh, oh), get(10 + l, B, oc, oh, oh)
        at, shape = off[f"conv{l + 1}.W"]
        n = int(np.prod(shape))
        got, want = grad[at:at + n].view(*shape), torch.nn.grad.conv2d_weight(x, tuple(shape), dy, stride=s)
        errors[f"conv{l + 1}.W filter"], errors[f"conv{l + 1}.W channel"] = worst(got, want, 0), worst(got, want, 1)
        at_b = off[f"conv{l + 1}.b"][0]
        errors[f"conv{l + 1}.b"] = worst(grad[at_b:at_b + oc][:, None], dy.sum((0, 2, 3))[:, None], 1)
        if l:
            w = torch.from_numpy(theta[at:at + n]).double().view(*shape)
            errors[f"input of conv{l + 1}"] = worst(get(10 + l - 1, *x.shape), torch.nn.grad.conv2d_input(x.shape, w, dy, stride=s) * (x > 0), 1)
        x = y
    print("  " + ", ".join(f"{k} {v:.1e}" for k, v in errors.items()), flush=True)
    off_by = {k: v for k, v in errors.items() if v > 2e-6}
    assert not off_by, off_by
    net.close()
