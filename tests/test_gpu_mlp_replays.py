"""Inference of the learned demapper around stream capture: parameters that a replayed update has
changed, and captured inference whose parameters change between replays.  The reference is a fresh
handle with the same parameters, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def md():
    import paper_2104_06311_amd as m
    return m


def fresh(net, y):
    other = md().MLP(net.D, net.hidden, net.m, seed=99)
    other.set(net.get(0))
    return md().llr_learned(other, y)


SHAPES = [(4, 64, 5), (17, 288, 4)]                     # weights resident in LDS, and streamed


def setup(D, H, m):
    rng = np.random.default_rng(D)
    y = torch.from_numpy(rng.standard_normal((256, D)).astype(np.float32)).cuda()
    t = torch.from_numpy((4 * rng.standard_normal((256, m))).astype(np.float32)).cuda()
    net = md().MLP(D, H, m, seed=1)
    net.train_step(y, t, 1e-2)                          # allocates what a capture must not
    md().llr_learned(net, y)
    torch.cuda.synchronize()
    return net, y, t


@pytest.mark.parametrize("D,H,m", SHAPES)
def test_inference_follows_replayed_updates(D, H, m):
    net, y, t = setup(D, H, m)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.train_step(y, t, 1e-2)
    for k in range(3):
        before = md().llr_learned(net, y)
        g.replay()
        torch.cuda.synchronize()
        after = md().llr_learned(net, y)
        assert not torch.equal(after, before) and torch.equal(after, fresh(net, y)), k


@pytest.mark.parametrize("D,H,m", SHAPES)
def test_captured_inference_follows_the_parameters(D, H, m):
    net, y, t = setup(D, H, m)
    out = torch.empty(256, m, device="cuda")
    net.train_step(y, t, 1e-2)                          # the copies are out of date at the capture
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        md().llr_learned(net, y, out=out)
    assert torch.equal(md().llr_learned(net, y), fresh(net, y))     # nothing has been replayed yet
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, fresh(net, y)), k
        net.train_step(y, t, 1e-2)
        torch.cuda.synchronize()
