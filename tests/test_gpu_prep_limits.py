"""The one-launch preparation at the upper edges of its range: the most labels with the most
coordinates that go with them (M * (D | 1) = 24576 floats and 8192 labels, 128 KiB of LDS), M = 1024
with the longest rows (130 KiB, with the search for factors), and the first shapes beyond, which take
three launches; labels broken in place at each."""
import math

import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_product import product

pytestmark = pytest.mark.gpu


def md():
    import paper_2104_06311_amd as m
    return m


def check(X, labels, snr_db, maxlog, atol, rtol):
    M, D = X.shape
    s2 = synth.sigma2_from_snr_db(X, snr_db)
    rng = np.random.default_rng(M)
    y = (X[rng.integers(0, M, 130)] + math.sqrt(s2) * rng.standard_normal((130, D))).astype(np.float32)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    ld = torch.from_numpy(labels.astype(np.int32)).cuda()
    f, ref = (md().llr_maxlog, oracle.llr_maxlog) if maxlog else (md().llr_exact, oracle.llr_exact)
    L = f(Xd, ld, yd, s2).cpu().numpy()
    want = ref(X, labels, y, s2)
    assert np.all(np.abs(L - want) <= atol + rtol * np.abs(want)), np.abs(L - want).max()
    keep = ld[M // 2].item()
    for bad in (ld[M // 2 - 1].item(), M):     # used twice, out of range
        ld[M // 2] = bad
        assert torch.isnan(f(Xd, ld, yd, s2)).all()
    ld[M // 2] = keep
    assert np.array_equal(f(Xd, ld, yd, s2).cpu().numpy(), L)
    md().release_cache()                       # the host's label check is cached by address


@pytest.mark.parametrize("M,D", [(8192, 2), (8192, 3), (8192, 4), (4096, 5), (4096, 6), (1024, 30)])
@pytest.mark.parametrize("maxlog", [False, True])
def test_without_factors(M, D, maxlog):
    X, _ = synth.gaussian_constellation(M, D, 300 + M + D)
    check(X, synth.random_labels(M, M + 5 * D), 9.0, maxlog, 2e-3, 2e-4)   # the split-FP16 score bound


@pytest.mark.parametrize("maxlog", [False, True])
def test_factors_of_the_longest_rows(maxlog):
    """Five groups of four points in six coordinates each."""
    rng = np.random.default_rng(1)
    X, labels = product(*[(rng.standard_normal((4, 6)), rng.permutation(4)) for _ in range(5)])
    perm = rng.permutation(1024)
    # FP64 distances, FP32 sums of two terms and their logarithms: the product tests' bound
    check(X[perm], labels[perm], 3.0, maxlog, 1e-9 if maxlog else 4e-6, 2.0 ** -23)
    assert md().llr_path_counts() == (0, 0)
