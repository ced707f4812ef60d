"""The batch sizes at which a launch rule of the prediction and update paths changes its kernel or its split of the work,
and the order of calls that come on more than one stream."""
import numpy as np
import pytest

import ga3c_synth as synth
import test_gpu_parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_1611_06256_amd as g
    assert torch.cuda.is_available()
    return g


@pytest.mark.parametrize("A,batches", [(18, (1, 2, 5, 6, 10, 11, 21, 22, 42, 43, 64, 65)), (63, (4, 9, 20, 41, 64))])
def test_small_net_predictions_across_the_splits_of_a_frame(G, A, batches):
    # up to 42 frames one launch, 21 with 63 actions; the slices of the fc layer per frame and the frames per block change with the batch,
    # and many actions leave no room in LDS for two frames
    for B in batches:
        P.check_predict(G, G.SMALL_NET(A), B, 7000 + B)


# The last batch of one launch and the first of three: 42 and 43 frames, 21 and 22 where two frames do not fit a block; from the caller's own
# parameters too.
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("A,B", [(18, 42), (18, 43), (63, 21), (63, 22)])
def test_where_the_one_launch_of_a_prediction_ends(G, A, B, math):
    import dataclasses
    import torch
    desc = dataclasses.replace(G.SMALL_NET(A), math=math)
    # (a seed at which no uniform is within 1e-5 of an edge of the distribution: 63 actions of 21 frames, one draw in forty sets has one there)
    P.check_predict(G, desc, B, 7080 + B)
    net, onet, theta = P.make(G, desc, B, 0, 7060 + B)
    frames = synth.rectangle_frames(7061, B)
    lg, vl, _, _ = P.run_predict(G, net, frames)
    got = {k: torch.full(s, float("nan"), device="cuda") for k, s in (("logits", (B, A)), ("values", (B,)))}
    G.predict_static(A, math, torch.from_numpy(theta).cuda(), torch.from_numpy(frames).cuda(), **got)
    torch.cuda.synchronize()
    # the same kernels on the same filters; three launches take the fc weights from another buffer, with the same sums
    np.testing.assert_array_equal(got["logits"].cpu().numpy(), lg)
    np.testing.assert_array_equal(got["values"].cpu().numpy(), vl)
    net.close()


@pytest.mark.parametrize("F,B", [(256, 3), (256, 66), (512, 1), (512, 5), (512, 130), (1024, 2), (1024, 65)])
def test_heads_after_few_and_many_partial_sums(G, F, B):
    desc = G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=18)
    P.check_predict(G, desc, B, 7100 + B)


# 256 units: the kernel that takes split operands.  96 units are no multiple of 64: the kernel that splits both itself, whose input
# gradient's tile changes at 256 tiles of 64x64 (41 columns of them: 6 rows up to 384 frames).
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("F,N", [(F, N) for F in (256, 96) for N in (76, 77, 128, 129)])
def test_fc_gradients_where_the_tile_changes(G, F, N, math):
    desc = G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=6, math=math)
    P.run_train(G, desc, N, 5, 7200 + N, dict(clip_norm=40.0), frames=synth.rectangle_frames(7201, N * 5).reshape(N, 5, 4, 84, 84))


# (the family's members at fp32 accuracy only: the medians for rounded operands are bounds of the two-layer nets)
@pytest.mark.parametrize("stride,F,A,N,math", [(0, F, A, N, m) for m in (0, 1) for F, A, N in
                                               [(256, 6, 1), (256, 6, 31), (256, 6, 32), (256, 6, 65), (256, 18, 1024), (256, 18, 1030), (64, 6, 530), (512, 40, 77)]] +
                         [(3, 256, 6, 70, 0), (2, 320, 6, 34, 0)])
def test_fc_gradients_at_the_edges_of_tiles_and_chunks(G, stride, F, A, N, math):
    # k-steps of 32 frames, tiles of 64 frames, units and columns (2592, 1600 and 4096 columns); chunks in a block or a block each;
    # heads that split their own gradients and heads that do not (40 actions).  Uniform bytes: frames made of a few drawn ones
    # repeat one operand's rounding a thousandfold, and the median of the forward outputs, bounded for roundings that are
    # independent, says nothing about them.
    conv = ((32, 8, stride), (32, 4, 2), (64, 4, 2)) if stride else ((16, 8, 4), (32, 4, 2))
    P.run_train(G, G.NetDesc(conv=conv, fc_units=F, n_actions=A, math=math), N, 1, 7250 + N, dict(clip_norm=40.0))


@pytest.mark.parametrize("math,line", [(0, 1024), (1, 640)])
def test_fc_gradients_of_updates_of_changing_size_in_one_context(G, math, line):
    # with and without partial sums in turn, at a capacity above the update's size: the bits of contexts of the update's own size
    import torch
    A = 6
    desc = G.SMALL_NET(A)
    desc.math = math
    cap = line + 70
    frames = torch.from_numpy(synth.uniform_frames(7261, (cap, 1, 4, 84, 84))).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7262, cap, 1, A).items()}

    def gradient(net, n):
        print(f"train {n} frames, math {math}", flush=True)
        net.train_step(frames[:n], tr["actions"][:n], tr["rewards"][:n], tr["dones"][:n], None, G.HParams(lr=0.0))
        return net.params_get(2).clone()

    net = G.Ga3c(desc, 1, cap)
    net.params_init(7263)
    for n in (cap, line, 40, line + 1, line, cap):
        own = G.Ga3c(desc, 1, n)
        own.params_init(7263)
        got, want = gradient(net, n), gradient(own, n)
        torch.cuda.synchronize()
        own.close()
        assert float(want.abs().max()) > 0 and torch.equal(got, want), n
    net.close()


# the most actions whose fused heads fit the 160 KB of LDS, and fewer: two passes over the units, a last block of five frames
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("A", [6, 12])
def test_fused_heads_of_1024_units(G, A, math):
    P.run_train(G, G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=1024, n_actions=A, math=math), 77, 1, 7280 + A, dict(clip_norm=40.0))


# heads too large for the fused kernel: blocks of 256 columns of the fc layer (one, one and a rest, four), a last block of five
# frames; outputs around the eight that are read ahead
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("F,A", [(256, 32), (300, 39), (1024, 15), (1024, 18)])
def test_separate_heads_backward(G, F, A, math):
    P.run_train(G, G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=A, math=math), 13, 1, 7290 + A, dict(clip_norm=40.0))


# Layer by layer only: both sides then round the same numbers and P.STAGE_TOL_BF16 holds at every size.  End to end a single operand
# that rounds differently on the two sides reaches every gradient behind it, so a median over 32 biases (observed 1.3e-3 at 641 frames)
# is a matter of how many such operands there are, and not of the kernels.
# Small net: a block of the fc weight gradient takes all chunks up to 640 frames.  Larger net: rounded operands leave room for two
# blocks of its convolutions per compute unit, a frame each up to 384 frames, then two frames in one block, and from 513 second
# frames of two blocks.
@pytest.mark.parametrize("which,N", [("small", 640), ("small", 641), ("large", 384), ("large", 385), ("large", 513), ("large", 1280)])
def test_rounded_updates_layer_by_layer(G, which, N):
    import torch
    desc = G.SMALL_NET(6) if which == "small" else G.LARGE_NET(6)
    desc.math = 1
    net, onet, theta = P.make(G, desc, 1, N, 7290 + N)
    frames = synth.uniform_frames(7291 + N, (N, 1, 4, 84, 84))
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7292 + N, N, 1, 6).items()}
    print(f"train {N} frames, {which} net, math 1", flush=True)
    net.train_step(torch.from_numpy(frames).cuda(), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
    torch.cuda.synchronize()
    P.check_layers(net, onet, theta, frames.reshape(N, 4, 84, 84), N)
    net.close()


def test_rounded_predictions_of_the_larger_net(G):
    desc = G.LARGE_NET(6)
    desc.math = 1
    P.check_predict(G, desc, 300, 7295)


@pytest.mark.parametrize("F,A,N", [(256, 3, 1), (256, 3, 17), (64, 7, 33), (256, 4, 129), (64, 3, 136), (256, 11, 264)])
def test_partial_gradients_added_up_at_the_ends_of_rows_and_rounds(G, F, A, N):
    # 1 to 264 matrices of partial sums (sixteen to a thread and round); rows of F + 1 = 257 and 65 columns of which groups of four
    # outputs take the bias with them, segments of 771, 455 and 195 outputs whose last group is not whole, and some without groups
    P.run_train(G, G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=A), N, 1, 7270 + N, dict(clip_norm=40.0))


# (frames of a batch, frames of the parts that it is predicted in once more): both are cut into the same chunks of k.  Small net, fp32
# accuracy: 512 and 256 blocks of the fc product, with two and three k-steps in LDS; 700 frames besides stage early in the fused
# convolutions, their parts between barriers; rounded: 960 and 512 blocks, two and three steps.  Stride-1
# member: 512 blocks with three steps (its weights and the activations of 128 frames exceed the Infinity Cache), 512 with two, 256
# with three; rounded: three.
@pytest.mark.parametrize("net,math,B,parts", [("small", 0, 512, (256, 256)), ("small", 0, 700, (450, 250)), ("small", 1, 900, (450, 450)),
                                              ("paper1", 0, 128, (64, 64)), ("paper1", 0, 128, (100, 28)), ("paper1", 1, 128, (64, 64))])
def test_fc_product_has_the_same_bits_with_two_and_three_steps_in_lds(G, net, math, B, parts):
    import torch
    A = 18
    desc = G.SMALL_NET(A) if net == "small" else P.paper_family_net(G, 1, A)
    desc.math = math
    net = G.Ga3c(desc, B, 0)
    net.params_init(7801)
    frames = torch.from_numpy(synth.uniform_frames(7802, (B, 4, 84, 84))).cuda()
    whole, split = torch.empty(B, A, device="cuda"), torch.empty(B, A, device="cuda")
    print(f"predict B={B} math={math}", flush=True)
    net.predict(frames, logits=whole)
    at = 0
    for n in parts:
        net.predict(frames[at:at + n], logits=split[at:at + n])
        at += n
    torch.cuda.synchronize()
    assert float(whole.abs().max()) > 0 and torch.equal(whole, split)
    net.close()


# two and three frames a block at fp32 accuracy, five and six with rounded operands: staged between barriers and early
@pytest.mark.parametrize("math,B", [(0, 512), (0, 520), (1, 1280), (1, 1290)])
def test_training_convolutions_have_the_same_bits_in_batches_of_any_size(G, math, B):
    import torch
    A = 6
    desc = G.SMALL_NET(A)
    desc.math = math
    net = G.Ga3c(desc, B, B)
    net.params_init(7811)
    frames = torch.from_numpy(synth.uniform_frames(7812, (B, 1, 4, 84, 84))).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7813, B, 1, A).items()}

    def convolutions(at, n):
        print(f"train {n} frames of {B}, math {math}", flush=True)
        net.train_step(frames[at:at + n], tr["actions"][at:at + n], tr["rewards"][at:at + n], tr["dones"][at:at + n], None, G.HParams(lr=0.0))
        return [net.train_debug_get(4 + l, torch.empty(n * k, device="cuda")).clone() for l, k in enumerate((16 * 400, 32 * 81))]

    whole = convolutions(0, B)
    parts = [convolutions(at, min(256, B - at)) for at in range(0, B, 256)]
    torch.cuda.synchronize()
    for l in range(2):
        assert float(whole[l].abs().max()) > 0 and torch.equal(whole[l], torch.cat([p[l] for p in parts])), f"layer {l + 1}"
    net.close()


def test_parameters_read_out_to_any_place(G):
    import torch
    net, _, theta = P.make(G, G.NetDesc(**P.ODD), 1, 0, 7300)
    for off in range(5):
        buf = torch.full((net.n_params + 9,), 7.0, device="cuda")
        net.params_get(0, out=buf[off:off + net.n_params])
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        np.testing.assert_array_equal(got[off:off + net.n_params], theta)
        assert (got[:off] == 7).all() and (got[off + net.n_params:] == 7).all()
    net.close()


def test_calls_that_move_to_a_second_stream_wait_for_the_first(G):
    # one stream alone records no event; the first call elsewhere has to wait for everything before it all the same
    import torch
    N, T, A = 128, 5, 18
    desc = G.SMALL_NET(A)
    frames = torch.from_numpy(synth.rectangle_frames(7401, N * T).reshape(N, T, 4, 84, 84)).cuda()
    first = frames[:, 0].contiguous()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7402, N, T, A).items()}
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for several in (False, True):
        net = G.Ga3c(desc, N, N * T)
        a, b = streams if several else streams[:1] * 2
        out = torch.empty(N, A, device="cuda")
        torch.cuda.synchronize()
        print("several streams" if several else "one stream", flush=True)
        net.params_init(7403, stream=a)
        for _ in range(3):
            net.predict(first, logits=out, stream=a)
            net.train_step(frames, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.01), stream=a)
        net.predict(first, logits=out, stream=b)
        net.train_step(frames, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.01), stream=b)
        net.predict(first, logits=out, stream=a)
        torch.cuda.synchronize()
        got.append((out.cpu().numpy(), net.params_get(0).cpu().numpy()))
        net.close()
    for x, y in zip(*got):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("B", [5, 64, 70])
def test_captured_predictions_replay_as_called(G, B):
    # a stream under capture gets its fences as nodes of their own (a launch that completes an event cannot be captured)
    import torch
    A = 18
    net = G.Ga3c(G.SMALL_NET(A), B, 0)
    s = torch.cuda.Stream()
    frames = torch.from_numpy(synth.rectangle_frames(7501, B)).cuda()
    got, want = torch.zeros(B, A, device="cuda"), torch.zeros(B, A, device="cuda")
    net.params_init(7502)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        net.predict(frames, logits=got, stream=s)
    for _ in range(3):
        got.zero_()
        net.predict(frames, logits=want, stream=s)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), want.cpu().numpy())
    assert want.abs().max().item() > 0
    net.close()


@pytest.mark.parametrize("which", ["small", "large", "paper3"])
def test_updates_in_place_give_the_same_parameters(G, which):
    # updates without a prediction between them overwrite the published parameters, and what is derived from them; with one
    # between them they write the other copy
    import torch
    N, T, A = 9, 5, 6
    desc = {"small": G.SMALL_NET(A), "large": G.LARGE_NET(A)}.get(which) or P.paper_family_net(G, 3, A)
    frames = torch.from_numpy(synth.rectangle_frames(7601, N * T).reshape(N, T, 4, 84, 84)).cuda()
    first = frames[:, 0].contiguous()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7602, N, T, A).items()}
    got = []
    for predictions in (1, 2, 0):                 # before every update, before every second one, only at the end
        net = G.Ga3c(desc, N, N * T)
        net.params_init(7603)
        out = torch.empty(N, A, device="cuda")
        for k in range(6):
            if predictions and k % predictions == 0:
                net.predict(first, logits=out)
            net.train_step(frames, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.01))
        net.predict(first, logits=out)
        torch.cuda.synchronize()
        got.append((out.cpu().numpy(), net.params_get(0).cpu().numpy(), net.params_get(1).cpu().numpy()))
        net.close()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            np.testing.assert_array_equal(x, y)


# four, two blocks per frame and one in the larger net's convolutions (up to 64 and 128 frames), four and one in its first layer (up to 64)
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129])
def test_larger_net_convolutions_have_the_same_bits_with_several_blocks_per_frame(G, n):
    import torch
    A, B = 6, 260
    desc = G.LARGE_NET(A)
    net = G.Ga3c(desc, B, B)
    net.params_init(7821)
    frames = torch.from_numpy(synth.uniform_frames(7822, (B, 1, 4, 84, 84))).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(7823, B, 1, A).items()}

    def convolutions(k):
        print(f"train {k} frames", flush=True)
        net.train_step(frames[:k], tr["actions"][:k], tr["rewards"][:k], tr["dones"][:k], None, G.HParams(lr=0.0))
        acts = [net.train_debug_get(4 + l, torch.empty(k * m, device="cuda")).clone() for l, m in enumerate((32 * 400, 64 * 81, 64 * 49))]
        return acts, [net.train_debug_get(10 + l, torch.empty(k * m, device="cuda")).clone() for l, m in enumerate((32 * 400, 64 * 81, 64 * 49))]

    (whole, dwhole), (part, dpart) = convolutions(B), convolutions(n)
    torch.cuda.synchronize()
    for l in range(3):
        assert float(part[l].abs().max()) > 0 and torch.equal(whole[l][:part[l].numel()], part[l]), f"layer {l + 1}"
    # what the fc layer sends back, and the last layer's input gradient: the fc layer adds its 3136 products up in other chunks where
    # there are fewer frames, which moves its outputs and all that follows from them by about sqrt(3136) fp32 roundings, 3e-6
    for l in (2, 1):
        scale = float(dpart[l].abs().max())
        assert scale > 0 and float((dwhole[l][:dpart[l].numel()] - dpart[l]).abs().max()) <= 1e-5 * scale, f"input gradient of layer {l + 2}"
    net.close()


def predictions(G, desc, frames, sizes):
    import torch
    net, B, A = G.Ga3c(desc, len(frames), 0), len(frames), desc.n_actions
    net.params_init(7831)
    u = torch.from_numpy(synth.uniforms(7833, B)).cuda()
    o = dict(logits=torch.full((B, A), float("nan"), device="cuda"), values=torch.full((B,), float("nan"), device="cuda"),
             probs=torch.full((B, A), float("nan"), device="cuda"), actions=torch.full((B,), -1, dtype=torch.int32, device="cuda"))
    lo = 0
    for n in sizes:
        print(f"predict {n} F={desc.fc_units} A={A} math={desc.math}", flush=True)
        net.predict(frames[lo:lo + n], uniforms=u[lo:lo + n], **{k: v[lo:lo + n] for k, v in o.items()})
        lo += n
    torch.cuda.synchronize()
    net.close()
    return o, lo


# Heads with a block per frame (up to 256 frames) and four frames per block form the same sums.  256 and 257 frames of 512 units are
# cut into the same chunks of the fc product, so everything is the same bits.
@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("A", [15, 16, 63])
def test_predictions_have_the_same_heads_with_one_and_four_frames_per_block(G, A, math):
    import torch
    frames = torch.from_numpy(synth.uniform_frames(7832, (257, 4, 84, 84))).cuda()
    desc = G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=512, n_actions=A, math=math)
    (four, _), (one, n) = predictions(G, desc, frames, [257]), predictions(G, desc, frames, [256])
    for k in four:
        assert torch.isfinite(four[k]).all() and torch.equal(four[k][:n], one[k][:n]), k


# 256 and 1024 units: wherever the one kernel takes over from the other the fc product is cut into other chunks of k, so results differ by
# the rounding of fp32 sums (and a draw now and then)
@pytest.mark.parametrize("F,A,sizes", [(256, 18, [132, 132]), (256, 3, [132, 132]), (1024, 6, [132, 132])])
def test_predictions_have_level_heads_with_one_and_four_frames_per_block(G, F, A, sizes):
    import torch
    frames = torch.from_numpy(synth.uniform_frames(7832, (264, 4, 84, 84))).cuda()
    desc = G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=A)
    (four, _), (one, _) = predictions(G, desc, frames, [264]), predictions(G, desc, frames, sizes)
    for k in ("logits", "values"):
        assert torch.isfinite(four[k]).all() and float((four[k] - one[k]).abs().max() / four[k].abs().max()) <= 2e-6, k
    assert float((four["actions"] != one["actions"]).float().mean()) <= 0.01


# segments longer than a wavefront's lanes hold the rewards of (64), as long, and shorter; units in fours and not, several
# frames of a block beyond the last, one output and the most that the fused kernel has
@pytest.mark.parametrize("T", [1, 63, 64, 65, 150])
@pytest.mark.parametrize("F,A", [(12, 6), (13, 1), (260, 31)])
def test_ragged_update_of_equal_segments_is_the_rectangular_one(G, T, F, A):
    import torch
    N = 3
    desc = G.NetDesc(conv=((16, 8, 4), (32, 4, 2)), fc_units=F, n_actions=A)
    frames = torch.from_numpy(synth.uniform_frames(7841, (N, T, 4, 84, 84))).cuda()
    tr = synth.trajectories(7842, N, T, A)
    ac, rw, dn = (torch.from_numpy(tr[k]).cuda() for k in ("actions", "rewards", "dones"))
    boot = torch.from_numpy(synth.rng(7843).standard_normal(N).astype(np.float32)).cuda()
    print(f"train T={T} F={F} A={A}", flush=True)
    out = []
    for ragged in (False, True):
        net = G.Ga3c(desc, 4, N * T)
        net.params_init(7844)
        if ragged:
            start = torch.from_numpy(np.arange(N + 1, dtype=np.int32) * T).cuda()
            net.train_step_ragged(frames.reshape(N * T, 4, 84, 84), ac.reshape(-1), rw.reshape(-1), dn.reshape(-1), start, boot, G.HParams())
        else:
            net.train_step(frames, ac, rw, dn, boot, G.HParams())
        torch.cuda.synchronize()
        out.append((net.params_get(0).cpu().numpy(), net.params_get(2).cpu().numpy(), net.train_debug_get(0, torch.empty(N * T, device="cuda")).cpu().numpy()))
        net.close()
    for x, y in zip(*out):
        assert np.isfinite(x).all()
        np.testing.assert_array_equal(x, y)
