"""Exact and max-log LLRs where FP32 squared distances, the noise's reciprocal or their product
leave the FP32 range: constellations and noise scaled by 1e20 and 1e-20, noise far below the
points' distances, and symbols at equal distance from several points.

Tolerances.  Factors of up to four points, and constellations of up to 16: those of test_gpu_product.py
for M <= 16; other products: those of its FP32 distances; 32 and 64 points without structure, whose
symbols all go to their FP64 pass here, the rounding of the result and 1e-9; and 8 roundings of the
farthest point's FP64 score, where scores cancel."""
import math

import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_product import pam, product, shape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def forget_labels():
    """Label buffers are checked on the host once per address: leave none behind."""
    yield
    import paper_2104_06311_amd as m
    m.release_cache()

DOUBLE = ["bpsk", "8psk", "gauss4", "gauss16", "qam4", "qam16", "2xqam16"]     # FP64 distances
SINGLE = ["qam64", "qam256", "psk8x2", "rect32", "three", "planes256", "flat64", "quarter64"]   # some FP32
GENERAL = ["gauss32", "gauss64"]


def md():
    import paper_2104_06311_amd as m
    return m


def points(name):
    if name in ("gauss4", "gauss32", "gauss64"):           # gauss4: one factor of four points
        return synth.gaussian_constellation(int(name[5:]), 2, 4)
    if name == "quarter64":                                # factors of four and of sixteen points
        return product(pam(4), pam(16))
    return shape(name)


def bound(name):
    if name in GENERAL:
        return 1e-9, 2.0 ** -23
    if name in DOUBLE:
        return 4e-6, 2.0 ** -23
    return 3 * 2.0 ** -24 * 256 * math.log(2.0) + 4e-6, 4 * 2.0 ** -24


def received(X, s2, n, seed):
    rng = np.random.default_rng(seed)
    X64 = X.astype(np.float64)
    y = X64[rng.integers(0, len(X), n)] + math.sqrt(s2) * rng.standard_normal((n, X.shape[1]))
    y[0] = 0.0                                             # between the points of every axis
    y[1] = X64[0]
    y[2] = 0.5 * (X64[0] + X64[1])
    y[3:6] *= 7.0                                          # outside the constellation
    return y.astype(np.float32)


def check_exact(X, labels, y, s2, atol, rtol):
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    ld = torch.from_numpy(labels.astype(np.int32)).cuda()
    want = oracle.llr_exact(X, labels, y, s2)
    assert np.isfinite(want).all()
    L = md().llr_exact(Xd, ld, yd, s2)
    got = L.cpu().numpy().astype(np.float64)
    far = ((y.astype(np.float64)[:, None] - X.astype(np.float64)) ** 2).sum(2).max(1, keepdims=True) / (2.0 * s2)
    good = np.abs(got - want) <= atol + rtol * np.abs(want) + 8 * 2.0 ** -53 * far      # not where NaN
    assert good.all(), (np.argwhere(~good)[:3], got[~good][:3], want[~good][:3])
    tx = torch.zeros(len(y), dtype=torch.int32, device="cuda")
    Lg, g, _ = md().llr_exact_gmi(Xd, ld, yd, tx, s2)
    assert torch.equal(Lg, L) and torch.isfinite(g).all()
    return Xd, ld, yd


@pytest.mark.parametrize("name", DOUBLE + SINGLE)
@pytest.mark.parametrize("scale", [1e20, 1e19, 1e6, 1e-6, 1e-20])
def test_scales(name, scale):
    X, labels = points(name)
    X = (X.astype(np.float64) * scale).astype(np.float32)
    s2 = synth.sigma2_from_snr_db(X, 10.0)
    y = received(X, s2, 517, 3)
    Xd, ld, yd = check_exact(X, labels, y, s2, *bound(name))
    got = md().llr_maxlog(Xd, ld, yd, s2).cpu().numpy().astype(np.float64)
    want = oracle.llr_maxlog(X, labels, y, s2)
    assert np.all(np.abs(got - want) <= 1e-9 + 2.0 ** -23 * np.abs(want))


@pytest.mark.parametrize("name", GENERAL)
@pytest.mark.parametrize("scale", [1e20, 1e19, 1e-20])
def test_scales_without_structure(name, scale):
    X, labels = points(name)
    X = (X.astype(np.float64) * scale).astype(np.float32)
    s2 = synth.sigma2_from_snr_db(X, 10.0)
    check_exact(X, labels, received(X, s2, 517, 3), s2, *bound(name))


@pytest.mark.parametrize("name", DOUBLE + SINGLE + GENERAL)
@pytest.mark.parametrize("snr_db", [60.0, 100.0, 115.0, 200.0, 290.0])
def test_little_noise(name, snr_db):
    X, labels = points(name)
    s2 = synth.sigma2_from_snr_db(X, snr_db)
    check_exact(X, labels, received(X, s2, 517, 4), s2, *bound(name))


@pytest.mark.parametrize("seed", range(6))
def test_logarithms_of_small_constellations(seed):
    """16 points of which some lie on the received value and the others out of reach: every subset's
    sum is a whole number k of terms 1 and the LLR ln (k0 / k1), FP64 but for its last rounding
    (and the 1e-10 that the logarithm's series leaves)."""
    rng = np.random.default_rng(seed)
    labels = np.arange(16, dtype=np.uint32)
    near = rng.random(16) < 0.6
    near[[0, 15]] = True                                   # no subset without one
    X = np.where(near, 0.25, 1e4 + np.arange(16)).astype(np.float32)[:, None]
    bits = (labels[:, None] >> np.arange(3, -1, -1)) & 1
    k1 = (bits & near[:, None]).sum(0)
    want = np.log((near.sum() - k1) / k1)
    L = md().llr_exact(torch.from_numpy(X).cuda(), torch.from_numpy(labels.astype(np.int32)).cuda(),
                       torch.full((3, 1), 0.25, device="cuda"), 0.5).cpu().numpy()
    assert np.all(np.abs(L - want) <= 2.0 ** -24 * np.abs(want) + 2e-10), (L[0], want)


def coinciding(n, seed):
    """n points of which some lie at 0.25, in both halves of every bit, and the others out of reach."""
    near = np.random.default_rng(seed).random(n) < 0.6
    near[[0, n - 1]] = True
    return np.where(near, 0.25, 1e4 + np.arange(n)), near


@pytest.mark.parametrize("n,other", [(8, 4), (8, 8), (8, 16), (16, 2), (16, 4), (16, 8), (16, 16)])
@pytest.mark.parametrize("seed", range(3))
def test_far_symbols_are_demapped_in_fp64(n, other, seed):
    """As above, in a product whose other factor's points are out of the FP32 sums' reach: ln (k0 / k1)
    but for the last rounding (2e-12: FP64 exponentials and logarithms)."""
    x, near = coinciding(n, seed)
    X, labels = product((x, np.arange(n)), (1e3 * np.arange(other), np.arange(other)))
    mf = n.bit_length() - 1
    bits = (np.arange(n)[:, None] >> np.arange(mf - 1, -1, -1)) & 1
    k1 = (bits & near[:, None]).sum(0)
    want = np.log((near.sum() - k1) / k1)
    L = md().llr_exact(torch.from_numpy(X).cuda(), torch.from_numpy(labels.astype(np.int32)).cuda(),
                       torch.tensor([[0.25, 0.0], [0.25, 1e3]], device="cuda"), 0.5)
    assert md().llr_path_counts() == (0, 0)
    assert np.all(np.abs(L.cpu().numpy()[:, :mf] - want) <= 2.0 ** -24 * np.abs(want) + 2e-12), (L[:, :mf], want)


@pytest.mark.parametrize("M,D", [(32, 1), (64, 1), (64, 3), (32, 8)])
@pytest.mark.parametrize("seed", range(3))
def test_left_symbols_are_demapped_in_fp64(M, D, seed):
    """The same without structure: the points with the highest label bit set are all out of reach."""
    x, near = coinciding(M // 2, seed)
    x, near = np.concatenate([x, 2e4 + np.arange(M // 2) ** 2]), np.concatenate([near, np.zeros(M // 2, bool)])
    X = np.zeros((M, D), np.float32)
    X[:, D - 1] = x
    m = M.bit_length() - 1
    k1 = (((np.arange(M)[:, None] >> np.arange(m - 2, -1, -1)) & 1) & near[:, None]).sum(0)
    want = np.log((near.sum() - k1) / k1)
    y = torch.zeros(70, D, device="cuda")
    y[:, D - 1] = 0.25
    L = md().llr_exact(torch.from_numpy(X).cuda(), torch.arange(M, dtype=torch.int32, device="cuda"), y, 0.5)
    assert md().llr_path_counts() == (70, 0)
    L = L.cpu().numpy()
    assert np.all(np.abs(L[:, 1:] - want) <= 2.0 ** -24 * np.abs(want) + 2e-12), (L[0], want)
    assert np.allclose(L[:, 0], (2e4 - 0.25) ** 2, rtol=1e-6)


@pytest.mark.parametrize("name", ["qam64", "qam256", "2xqam16", "planes256", "gauss64"])
@pytest.mark.parametrize("snr_db", [16.0, 24.0, 27.0, 40.0])
def test_fused_gmi_takes_left_symbols_from_their_llrs(name, snr_db):
    """None, some and all symbols left: the fused loss terms against gmi_reduce of the same LLRs.  A term is
    2^-22 of itself and of its LLRs' rounding (2^-24 of up to 1e4 here, where it is not near zero) off."""
    X, labels = points(name)
    s2 = synth.sigma2_from_snr_db(X, snr_db)
    Xd, ld = torch.from_numpy(X).cuda(), torch.from_numpy(labels.astype(np.int32)).cuda()
    tx, y = md().awgn_sample(Xd, 11, 0, 70001, math.sqrt(s2))
    tx[:50] = (tx[:50] + 1) % len(X)                        # some wrong ones, so that terms are large
    L, g, se = md().llr_exact_gmi(Xd, ld, y, tx, s2)
    assert torch.equal(L, md().llr_exact(Xd, ld, y, s2))
    G, _, SE = md().gmi_reduce(L, tx, ld)
    loss = (len(labels).bit_length() - 1) - G.item()
    assert abs(g.item() - G.item()) <= 2e-6 * (loss + 1.0) and abs(se.item() - SE.item()) <= 1e-4 * SE.item()


@pytest.mark.parametrize("name", ["qam64", "qam256"])
def test_captured_calls_with_and_without_left_symbols(name):
    """One graph replayed with received values of which some, then none, then all are left."""
    X, labels = points(name)
    s2 = synth.sigma2_from_snr_db(X, 25.0)
    Xd, ld = torch.from_numpy(X).cuda(), torch.from_numpy(labels.astype(np.int32)).cuda()
    m = len(labels).bit_length() - 1
    rng = np.random.default_rng(8)
    near = X[np.argsort((X ** 2).sum(1))[:4]]               # next to the axes: no far subset
    some = X[rng.integers(0, len(X), 3000)]
    ys = [some, near[rng.integers(0, 4, 3000)] * 0.2, 40.0 * some, some]
    ys = [torch.from_numpy((v + math.sqrt(s2) * rng.standard_normal(v.shape)).astype(np.float32)).cuda() for v in ys]
    y, out = torch.empty_like(ys[0]), torch.empty(3000, m, device="cuda")
    y.copy_(ys[0])
    md().llr_exact_noalloc(Xd, ld, y, s2, out=out)          # looks the array's address up
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        md().llr_exact_noalloc(Xd, ld, y, s2, out=out)
    for v in ys:
        want = md().llr_exact(Xd, ld, v, s2)
        y.copy_(v)
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
