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
    return G.LARGE_NET(A) if which == "large" else G.NetDesc(conv=((32, 8, int(which[-1])), (32, 4, 2), (64, 4, 2)), fc_units=256, n_actions=A)


# one, two and three frames a block; activations beyond float16's largest number and below its smallest; a filter of zeros
@pytest.mark.parametrize("which", ["large", "paper4", "paper3"])
@pytest.mark.parametrize("B,layer,power", [(1, 1, 0), (256, 1, 0), (257, 1, 0), (513, 1, 0), (3, 1, 30), (3, 1, -30), (3, 2, 30), (3, 2, -30), (3, 3, 30), (3, 3, -40)])
def test_predictions_with_three_convolutions_in_one_kernel(G, which, B, layer, power):
    import torch
    net, onet, theta = P.make(G, network(G, which, 6), B, 0, 9100 + B)
    theta = scaled(net, theta, layer, power)
    at, shape = net.offsets()[f"conv{layer}.W"]
    theta[at:at + int(np.prod(shape[1:]))] = 0
    net.params_set(torch.from_numpy(theta).cuda(), 0)
    frames = synth.rectangle_frames(9101 + B, B)
    if B == 3:
        frames[0] = 0
    lg, vl, _, _ = P.run_predict(G, net, frames)
    ref = orc.forward(onet, theta, frames)
    assert P.rel_err(lg, ref["logits"]) <= TOL and P.rel_err(vl, ref["values"]) <= TOL
    net.close()
