"""Training of the learned demapper after an allocation that failed: the handle's working memory is gone
then, and what it held must not be taken for current.  Compared with a handle that met no failure, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def md():
    import paper_2104_06311_amd as m
    return m


def batch(n, D, m, seed):
    rng = np.random.default_rng(seed)
    return (torch.from_numpy(rng.standard_normal((n, D)).astype(np.float32)).cuda(),
            torch.from_numpy((4 * rng.standard_normal((n, m))).astype(np.float32)).cuda())


@pytest.mark.parametrize("D,H,m", [(4, 64, 5), (4, 40, 5)])    # fused kernels, and the layer-by-layer form
def test_update_after_a_failed_larger_batch(D, H, m):
    small, large = batch(64, D, m, 1), batch(20000, D, m, 2)
    net, ref = md().MLP(D, H, m, seed=3), md().MLP(D, H, m, seed=3)
    for n in (net, ref):
        n.train_step(*small, 1e-2)
    torch.cuda.synchronize()
    md().alloc_fault_inject(0)
    try:
        with pytest.raises(md().MdemapError) as e:
            net.grad(*large)
        assert e.value.status == -5
    finally:
        md().alloc_fault_inject(-1)
    for n in (net, ref):
        n.adam_step(1e-2)                                   # with the gradient both still hold
        n.train_step(*small, 1e-2)
        n.train_step(*large, 1e-2)
    for which in range(4):
        assert np.array_equal(net.get(which), ref.get(which)), which
