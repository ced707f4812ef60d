"""The any-size kernels of the paper's larger-network family (csrc/conv_band.hpp, conv_bytes.hpp, conv_band_f32.hpp)
at the sizes where their bands can go wrong, layer by layer against the fp64 oracle, and bit for bit against the
any-shape kernels where the two form the same sums."""
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


def frames_of(seed, n, h):
    return synth.rectangle_frames(seed, n, h=h)


# conv1 -> conv2 -> conv3 maps: odd and even, one row or column, one band and several, a last band that is short
SHAPES = [
    dict(in_h=60, conv=((32, 8, 2), (32, 4, 2), (64, 4, 2))),      # 27x39 -> 12x18 -> 5x8
    dict(in_h=32, conv=((32, 8, 3), (64, 4, 2))),                  # 9x26 -> 3x12
    dict(in_h=50, conv=((16, 8, 1), (32, 3, 2), (32, 4, 2))),      # 43x77, 16 filters; 21x38 (general) -> 9x18
    dict(in_h=84, conv=((32, 8, 5), (32, 4, 2))),                  # 16x16 -> 7x7
    dict(in_h=36, conv=((32, 8, 9), (64, 4, 2))),                  # 4x9 -> 1x3
]


@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_band_shapes(G, shape, math):
    desc = G.NetDesc(in_c=4, in_w=84, fc_units=32, n_actions=5, math=math, **shape)
    P.check_predict(G, desc, 3, 9100, frames=frames_of(9101, 3, desc.in_h))
    P.run_train(G, desc, 2, 3, 9110, dict(clip_norm=40.0), frames=frames_of(9111, 6, desc.in_h).reshape(2, 3, 4, desc.in_h, 84))


@pytest.mark.parametrize("math", [0, 1])
def test_several_frames_per_item(G, math):
    # maps so small and a batch so large that an item holds several frames, the last item fewer
    desc = G.NetDesc(in_c=4, in_h=40, in_w=84, conv=((32, 8, 8), (32, 4, 2)), fc_units=16, n_actions=4, math=math)
    N, T = 421, 5
    fr = np.tile(frames_of(9201, 131, 40), (17, 1, 1, 1))[:N * T]
    P.run_train(G, desc, N, T, 9200, dict(clip_norm=40.0), frames=fr.reshape(N, T, 4, 40, 84))
    P.check_predict(G, desc, 1100, 9210, frames=fr[:1100])


@pytest.mark.parametrize("shape,n", [(SHAPES[0], 7), (SHAPES[2], 3), (SHAPES[3], 300),
                                     (dict(in_h=84, conv=((32, 8, 1), (32, 4, 2), (64, 4, 2))), 5)])
def test_training_activations_are_the_any_shape_kernels_bits(G, shape, n):
    import torch
    desc = G.NetDesc(in_c=4, in_w=84, fc_units=16, n_actions=4, **shape)
    fr = torch.from_numpy(np.tile(frames_of(9301, min(n, 20), desc.in_h), (n // min(n, 20), 1, 1, 1))).cuda()
    n = int(fr.shape[0])
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9302, n, 1, 4).items()}
    acts = []
    for generic in (True, False):
        net = G.Ga3c(desc, n, n)
        net.params_init(9303)
        net.use_generic_kernels(generic)
        print(f"train n={n} generic={generic}", flush=True)
        net.train_step(fr.view(n, 1, *fr.shape[1:]), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
        c, h, w, got = 4, desc.in_h, 84, []
        for l, (oc, k, s) in enumerate(desc.conv):
            c, h, w = oc, (h - k) // s + 1, (w - k) // s + 1
            got.append(net.train_debug_get(4 + l, torch.empty(n * c * h * w, device="cuda")))
        torch.cuda.synchronize()
        acts.append(got)
        net.close()
    for l, (a, b) in enumerate(zip(*acts)):
        assert float(a.abs().max()) > 0 and torch.equal(a, b), f"layer {l}"


@pytest.mark.parametrize("math", [0, 1])
@pytest.mark.parametrize("stride,h,N", [(1, 35, 30), (2, 37, 60), (3, 38, 80)])
def test_gradients_with_several_items_per_block(G, stride, h, N, math):
    # more bands than blocks: 28x77 / 15x39 / 11x26 pixels of conv1, then 13x37 / 6x18 / 4x12 of the second layer, whose rows are
    # filled up to octets and whose bands do not divide the map; the last band of a frame is short
    desc = G.NetDesc(in_c=4, in_h=h, in_w=84, conv=((32, 8, stride), (32 if stride > 1 else 64, 4, 2)), fc_units=16, n_actions=4, math=math)
    fr = np.tile(frames_of(9401, 25, h), (N // 5, 1, 1, 1))[:5 * N]
    P.run_train(G, desc, N, 5, 9400, dict(clip_norm=40.0), frames=fr.reshape(N, 5, 4, h, 84))


def test_gradients_do_not_meet_what_an_earlier_larger_batch_left(G):
    # rows end inside a vector, and what lies behind the last frame of a batch is an earlier batch's, here not numbers
    import torch
    desc = G.NetDesc(in_c=4, in_h=36, in_w=84, conv=((32, 8, 2), (32, 4, 2)), fc_units=16, n_actions=4)
    fr = torch.from_numpy(frames_of(9501, 10, 36)).cuda().view(5, 2, 4, 36, 84)
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9502, 5, 2, 4).items()}
    grads = []
    for dirty in (False, True):
        net = G.Ga3c(desc, 5, 10)
        if dirty:
            net.params_set(torch.full((net.n_params,), float("nan"), device="cuda"), 0)
            net.train_step(fr, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams())
        net.params_init(9503)
        cut = {k: v[:3].contiguous() for k, v in tr.items()}
        net.train_step(fr[:3].contiguous(), cut["actions"], cut["rewards"], cut["dones"], None, G.HParams())
        grads.append(net.params_get(2))
        torch.cuda.synchronize()
        net.close()
    assert float(grads[0].abs().max()) > 0 and torch.equal(grads[0], grads[1])


@pytest.mark.parametrize("n", [20, 40, 60, 140])
def test_training_activations_are_the_any_shape_kernels_bits_across_the_launch_rules(G, n):
    # the second layer's 9 n tiles of 64 filters: a block per tile, one filter tile per wavefront, two, and one again with more rounds
    test_training_activations_are_the_any_shape_kernels_bits(G, dict(in_h=84, conv=((32, 8, 3), (64, 4, 2))), n)


@pytest.mark.parametrize("shape,n", [(SHAPES[0], 7), (SHAPES[0], 1), (dict(in_h=84, conv=((32, 8, 3), (32, 4, 2), (64, 4, 2))), 5),
                                     (dict(in_h=36, conv=((32, 8, 9), (64, 4, 2))), 300)])
def test_masks_as_bits_are_the_masks_as_values(G, shape, n):
    # frames that are not 16-byte aligned go through the any-shape kernel of the first layer, which has the same sums and leaves no
    # bits: the input gradient of the second layer then takes its mask from the activations
    import torch
    desc = G.NetDesc(in_c=4, in_w=84, fc_units=32, n_actions=4, **shape)
    fr = np.tile(frames_of(9401, min(n, 20), desc.in_h), (-(-n // min(n, 20)), 1, 1, 1))[:n]
    room = torch.empty(fr.size + 4, dtype=torch.uint8, device="cuda")
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9402, n, 1, 4).items()}
    h, w = (desc.in_h - desc.conv[0][1]) // desc.conv[0][2] + 1, (84 - desc.conv[0][1]) // desc.conv[0][2] + 1
    got = []
    for shift in (0, 4):
        x = room[shift:shift + fr.size].view(n, 1, 4, desc.in_h, 84)
        x.copy_(torch.from_numpy(fr).view(n, 1, 4, desc.in_h, 84))
        net = G.Ga3c(desc, n, n)
        net.params_init(9403)
        print(f"n={n} shift={shift}", flush=True)
        net.train_step(x, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
        got.append([net.train_debug_get(which, torch.empty(n * 32 * h * w, device="cuda")) for which in (4, 10)])
        torch.cuda.synchronize()
        net.close()
    for a, b in zip(*got):
        assert float(a.abs().max()) > 0 and torch.equal(a, b)
    assert bool(((got[0][0] > 0) | (got[0][1] == 0)).all()) and bool((got[0][0] == 0).any())


@pytest.mark.parametrize("in_h", [49, 50])
def test_byte_layer_with_two_blocks_per_compute_unit_has_the_any_shape_kernels_bits(G, in_h):
    # 40 frames: 42x77 maps are 8085 tiles, whole rounds for two blocks per compute unit; 43x77 are a tile a block more, and take one
    test_training_activations_are_the_any_shape_kernels_bits(G, dict(in_h=in_h, conv=((32, 8, 1), (32, 4, 2))), 40)


@pytest.mark.parametrize("oc,n", [(64, 256), (32, 512)])
def test_input_gradient_of_a_tall_narrow_map(G, oc, n):
    # 514x4 with one term: LDS and registers would hold all 257 rows of the phase grid in one item, more than a staging unit can name
    import torch
    import torch.nn.functional as F
    desc = G.NetDesc(in_c=4, in_h=521, in_w=11, conv=((32, 8, 1), (oc, 4, 2)), fc_units=16, n_actions=4, math=1)
    net = G.Ga3c(desc, 1, n)
    net.params_init(9601)
    fr = torch.from_numpy(synth.uniform_frames(9602, (n, 1, 4, 521, 11))).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9603, n, 1, 4).items()}
    print(f"train {n} frames, {oc} filters", flush=True)
    net.train_step(fr, tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
    at = net.offsets()["conv2.W"][0]
    w = net.params_get(0)[at:at + oc * 32 * 16].cpu().view(oc, 32, 4, 4)
    act, dact, dy = (net.train_debug_get(which, torch.empty((n, *shape), device="cuda"))[::51].cpu()
                     for which, shape in ((4, (32, 514, 4)), (10, (32, 514, 4)), (11, (oc, 256, 1))))
    torch.cuda.synchronize()
    net.close()
    assert bool((dy[:, :, -2:] != 0).any())
    ref = F.conv_transpose2d(dy.bfloat16().double(), w.bfloat16().double(), stride=2) * (act > 0)
    # products of bfloat16 are exact; at most 2 x 2 x oc of them are added in fp32
    bound = 4 * oc * 2.0 ** -24 * F.conv_transpose2d(dy.bfloat16().double().abs(), w.bfloat16().double().abs(), stride=2)
    assert bool(((dact - ref).abs() <= bound).all())


@pytest.mark.parametrize("shape", [SHAPES[0], dict(in_h=50, conv=((32, 8, 1), (32, 4, 2), (64, 4, 2))), dict(in_h=84, conv=((32, 8, 3), (32, 4, 2), (64, 4, 2)))])
def test_gradients_are_as_near_to_the_exact_sums_as_those_of_the_fp32_instruction(G, shape):
    # every layer's gradients from the library's own activations and dY, against products and sums in 64 bits: three bf16 terms an
    # operand (csrc/conv_band_grads.hpp), and the any-shape kernels' chains of the fp32 instruction
    import torch
    import torch.nn.functional as F
    n = 6
    desc = G.NetDesc(in_c=4, in_w=84, fc_units=32, n_actions=4, **shape)
    fr = torch.from_numpy(frames_of(9701, n, desc.in_h))
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9702, n, 1, 4).items()}
    off = {}
    for generic in (False, True):
        net = G.Ga3c(desc, n, n)
        net.params_init(9703)
        net.use_generic_kernels(generic)
        print(f"train generic={generic}", flush=True)
        net.train_step(fr.cuda().view(n, 1, 4, desc.in_h, 84), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
        theta, grad, at = net.params_get(0).cpu(), net.params_get(2).cpu(), net.offsets()
        x, h, w = fr.double() / 255, desc.in_h, 84
        for l, (oc, k, s) in enumerate(desc.conv):
            oh, ow = (h - k) // s + 1, (w - k) // s + 1
            act, dy = (net.train_debug_get(which + l, torch.empty((n, oc, oh, ow), device="cuda")).cpu().double() for which in (4, 10))
            o, sh = at[f"conv{l + 1}.W"]
            W, dW = (v[o:o + oc * sh[1] * k * k].view(*sh).double() for v in (theta, grad))
            off[f"dW{l + 1}", generic] = float((dW - torch.nn.grad.conv2d_weight(x, W.shape, dy, stride=s)).norm() / dW.norm())
            o = at[f"conv{l + 1}.b"][0]
            db = grad[o:o + oc].double()
            off[f"db{l + 1}", generic] = float((db - dy.sum((0, 2, 3))).norm() / db.norm())
            if l:
                dx = F.conv_transpose2d(dy, W, stride=s, output_padding=((h - k) % s, (w - k) % s)) * (x > 0)
                off[f"dX{l + 1}", generic] = float((below - dx).norm() / dx.norm())
            x, below, h, w = act, dy, oh, ow
        net.close()
    print({k[0]: (f"{v:.1e}", f"{off[k[0], True]:.1e}") for k, v in off.items() if not k[1]}, flush=True)
    for (what, generic), v in off.items():
        if not generic:
            assert 0 < v <= off[what, True] and (what[:2] != "dX" or v <= 8e-8), (what, v, off[what, True])


def test_an_infinite_activation_stays_in_its_channel(G):
    # a vector of eight columns ends in the next row, in the next channel or behind the last frame: what lies there meets zeros of dY,
    # and infinity times zero is no number.  11x38 -> 4x18 with dY all zero (the fc layer's sums are no numbers, its rectifier makes them 0)
    import torch
    desc = G.NetDesc(in_c=4, in_h=30, in_w=84, conv=((32, 8, 2), (32, 4, 2)), fc_units=32, n_actions=4)
    n, c = 5, 3
    net = G.Ga3c(desc, n, n)
    net.params_init(9801)
    theta, at = net.params_get(0), net.offsets()
    theta[at["conv1.b"][0] + c] = float("inf")
    net.params_set(theta, 0)
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9802, n, 1, 4).items()}
    net.train_step(torch.from_numpy(frames_of(9803, n, 30)).cuda().view(n, 1, 4, 30, 84), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
    o = at["conv2.W"][0]
    dw = net.params_get(2)[o:o + 32 * 32 * 16].view(32, 32, 16)
    torch.cuda.synchronize()
    net.close()
    assert bool(dw[:, c].isnan().all())
    dw[:, c] = 0
    assert bool((dw == 0).all())


@pytest.mark.parametrize("shape", [SHAPES[0], dict(in_h=84, conv=((32, 8, 3), (32, 4, 2), (64, 4, 2)))])
def test_weights_beyond_the_largest_bfloat16(G, shape):
    # -3.4e38 is a number, though its first term would round to minus infinity: outputs with it are cut off, gradients of the rest stay
    import torch
    n = 4
    desc = G.NetDesc(in_c=4, in_w=84, fc_units=32, n_actions=4, **shape)
    fr = torch.from_numpy(frames_of(9901, n, desc.in_h)).cuda()
    tr = {k: torch.from_numpy(v).cuda() for k, v in synth.trajectories(9902, n, 1, 4).items()}
    got = []
    for generic in (False, True):
        net = G.Ga3c(desc, n, n)
        net.params_init(9903)
        theta, at = net.params_get(0), net.offsets()
        for layer, k in (("conv1.W", 500), ("conv2.W", 5000), ("conv3.W", 9000)):
            theta[at[layer][0] + k] = -3.4e38
        net.params_set(theta, 0)
        net.use_generic_kernels(generic)
        print(f"generic={generic}", flush=True)
        logits, values = torch.empty((n, 4), device="cuda"), torch.empty(n, device="cuda")
        net.predict(fr, logits=logits, values=values)
        net.train_step(fr.view(n, 1, 4, desc.in_h, 84), tr["actions"], tr["rewards"], tr["dones"], None, G.HParams(lr=0.0))
        got.append([logits, values, net.params_get(2)])
        torch.cuda.synchronize()
        net.close()
    for a, b in zip(*got):
        assert bool(torch.isfinite(a).all()) and float((a - b).norm() / b.norm()) <= 5e-5      # sums of fp32 products through the layers
