"""gmi_reduce and ber_count where a thread's symbols in flight end and the grid is at its largest
(2048 blocks of 256 threads, four symbols each): one symbol less, exactly as many, and a second trip
with few symbols.  Tolerances as in test_gpu_reductions.py; error counts are whole numbers."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FULL = 2048 * 256 * 4


@pytest.mark.parametrize("m", [1, 3, 4, 5])
@pytest.mark.parametrize("n", [FULL - 1, FULL, FULL + 1, FULL + 3, FULL + 2048 * 256 + 1])
def test_second_trip(m, n):
    import paper_2104_06311_amd as md
    g = torch.Generator(device="cuda")
    g.manual_seed(n + m)
    labels = torch.randperm(1 << m, device="cuda", generator=g).to(torch.int32)
    tx = torch.randint(0, 1 << m, (n,), device="cuda", generator=g).to(torch.int32)
    shifts = torch.arange(m - 1, -1, -1, device="cuda", dtype=torch.int32)
    sent = ((labels[tx.long()][:, None] >> shifts) & 1).to(torch.float32)
    llr = (1.0 - 2.0 * sent) * 3.0 + 2.5 * torch.randn((n, m), device="cuda", generator=g)
    llr[-1] = -40.0 * (1.0 - 2.0 * sent[-1])                 # the last symbol: wrong in every bit, and heavy
    G, pb, se = md.gmi_reduce(llr, tx, labels)
    x = llr.double() * (2.0 * sent.double() - 1.0)
    terms = torch.logaddexp(torch.zeros_like(x), x) / np.log(2.0)
    T = terms.sum(1)
    mean = T.mean().item()
    assert abs(G.item() - (m - mean)) <= 2e-6 * (mean + 1.0)
    assert torch.all((pb - (1.0 - terms.mean(0))).abs() <= 5e-7 * (terms.mean(0) + 1.0))
    assert abs(se.item() - T.std().item() / np.sqrt(n)) <= 1e-5 * se.item()
    err, per = md.ber_count(llr, tx, labels)
    wrong = ((llr < 0) != (sent == 1)).sum(0)
    assert per.cpu().tolist() == wrong.cpu().tolist() and err.item() == wrong.sum().item()
