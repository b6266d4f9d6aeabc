"""The sparse call's row list on the matrix cores (bf16 caches): lists are padded to whole groups of 16 rows with
a listed row that no head takes, and a window in blocks of its own is listed too. Rows that nobody selected hold
NaN, so a read of one that reaches a product shows. Against attention over the same rows in 64 bits."""
import math

import pytest
import torch

from paper_2606_31519_amd import rbq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("n,w,tail,every", [
    (2048, 0, True, 7),      # ragged lists, no window
    (2048, 19, True, 97),    # a few rows and the folded window behind them
    (1024, 19, False, 1),    # full lists; the window in a block of its own, one full group and three rows
    (3000, 300, False, 2900),   # one row in a whole call (splits without any), two window blocks
    (1111, 0, True, 1),
])
def test_unlisted_rows_stay_out(G, D, n, w, tail, every):
    Hkv = 2
    Hq, tau = Hkv * G, 1.0 / math.sqrt(D)
    g = torch.Generator(device="cuda").manual_seed(n + w + G)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    q = r(1, Hq, D)
    cap = n + w
    K, V = r(1, Hkv, cap, D).to(torch.bfloat16), r(1, Hkv, cap, D).to(torch.bfloat16)
    sel = torch.zeros(Hq, n, dtype=torch.bool, device="cuda")
    for h in range(Hq):
        sel[h, (h % 3)::every] = True     # (position 0, 1 or 2 and every `every`-th from there)
    unlisted = ~sel.view(Hkv, G, n).any(1)
    K[0, :, :n][unlisted] = float("nan")
    V[0, :, :n][unlisted] = float("nan")
    Kl, Vl, ld = (K[:, :, n:], V[:, :, n:], cap) if tail else \
        (K[:, :, n:].clone().contiguous(), V[:, :, n:].clone().contiguous(), max(w, 1))
    idx = torch.zeros(Hq, n, dtype=torch.int32, device="cuda")
    cnt = sel.sum(1).to(torch.int32)
    for h in range(Hq):
        idx[h, :cnt[h]] = sel[h].nonzero()[:, 0].to(torch.int32)
    out = torch.empty(1, Hq, D, device="cuda")
    lse = torch.empty(1, Hq, device="cuda")
    ws = rbq.workspace(rbq.RBQ_OP_SPARSE_DECODE, 1, Hq, Hkv, D, n, w)
    rbq.rbq_sparse_decode(1, Hq, Hkv, D, q, K, V, cap, n, idx, cnt, Kl if w else None, Vl if w else None, ld, w, tau,
                          out, lse, ws)
    torch.cuda.synchronize()
    for h in range(Hq):
        rows = torch.cat([sel[h].nonzero()[:, 0], torch.arange(n, n + w, device="cuda")])
        k, v = K[0, h // G, rows].double(), V[0, h // G, rows].double()
        lg = k @ q[0, h].double() * tau
        ref = torch.softmax(lg, 0) @ v
        # probabilities as two bf16 parts (2^-17 of each), logits and sums in fp32 (some 1e-6)
        assert (out[0, h].double() - ref).abs().max() <= 3e-5 * v.abs().max()
        assert abs(float(lse[0, h]) - float(torch.logsumexp(lg, 0))) <= 1e-5 * max(1.0, float(lg.abs().max()))
