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


@pytest.mark.parametrize("B,Hkv,D,w", [(40, 8, 64, 0), (64, 4, 128, 9), (65, 4, 128, 9), (2, 3, 64, 30), (64, 9, 128, 9),
                                       (64, 13, 64, 0), (65, 9, 128, 9)])
def test_ragged_batches_in_any_order(B, Hkv, D, w):
    """Launches of more blocks than are resident at once, in chunks of 512 keys or more, take the densest sequences first
    (64 sequences x 9 or 13 KV heads here; the others keep their order): every sequence still gets its own rows, also
    empty ones and equal densities."""
    G, n, tau = 2, 1100, 1.0 / math.sqrt(D)
    Hq, cap = Hkv * G, n + w
    g = torch.Generator(device="cuda").manual_seed(B)
    r = lambda *s: torch.randn(*s, device="cuda", generator=g)
    q, K, V = r(B, Hq, D), r(B, Hkv, cap, D).to(torch.bfloat16), r(B, Hkv, cap, D).to(torch.bfloat16)
    seq_n = torch.tensor([(0, n, 1, 257, 1024, 700, 700)[b % 7] for b in range(B)], dtype=torch.int32, device="cuda")
    seq_w = torch.tensor([b % (w + 1) for b in range(B)], dtype=torch.int32, device="cuda")
    idx = torch.zeros(B, Hq, n, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(B, Hq, dtype=torch.int32, device="cuda")
    lists = {}
    for b in range(B):
        for h in range(Hq):
            rows = torch.arange(0, int(seq_n[b]), 1 + (b * 5 + h) % 9, device="cuda")
            lists[b, h] = rows
            idx[b, h, :len(rows)] = rows.to(torch.int32)
            cnt[b, h] = len(rows)
    out, lse = torch.empty(B, Hq, D, device="cuda"), torch.empty(B, Hq, device="cuda")
    ws = rbq.workspace(rbq.RBQ_OP_SPARSE_DECODE, B, Hq, Hkv, D, n, w)
    rbq.rbq_sparse_decode_varlen(B, Hq, Hkv, D, q, K, V, cap, n, w, seq_n, seq_w, idx, cnt, tau, out, lse, ws)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(Hq):
            nb, wb = int(seq_n[b]), int(seq_w[b])
            rows = torch.cat([lists[b, h], torch.arange(nb, nb + wb, device="cuda")])
            if len(rows) == 0:
                assert float(lse[b, h]) == -math.inf and (out[b, h] == 0).all()
                continue
            k, v = K[b, h // G, rows].double(), V[b, h // G, rows].double()
            lg = k @ q[b, h].double() * tau
            # (as above)
            assert (out[b, h].double() - torch.softmax(lg, 0) @ v).abs().max() <= 3e-5 * v.abs().max()
            assert abs(float(lse[b, h]) - float(torch.logsumexp(lg, 0))) <= 1e-5 * max(1.0, float(lg.abs().max()))
