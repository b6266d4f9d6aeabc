"""The Top-p selection's forms (one block per row up to 32768 keys, three passes
beyond, each with its irregular rows) against the oracle, at the sizes where one
takes over from the other and on rows that leave the logarithmic grid."""
import math

import numpy as np
import pytest
import torch

import parity_util as pu
from paper_2606_31519_amd import pipeline, rbq
from workloads import gen

pytestmark = pytest.mark.gpu
TAU = 1 / math.sqrt(128)


def _select(S, p, tau):
    rows, n = S.shape
    dS = torch.from_numpy(np.ascontiguousarray(S, dtype=np.float32)).cuda()
    sel = torch.full((rows, n), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(rows, dtype=torch.int32, device="cuda")
    rbq.rbq_topp_select(1, rows, n, dS, p, tau, sel, cnt, rbq.workspace(rbq.RBQ_OP_TOPP, 1, rows, rows, 128, n))
    torch.cuda.synchronize()
    return sel.cpu().numpy(), cnt.cpu().numpy()


def _rows(n, seed):
    r = np.random.default_rng(seed)
    x = r.standard_normal(n)
    tail = np.concatenate([[40.0 / TAU], np.full(n - 1, 0.0)]) if n > 1 else np.zeros(1)
    return np.stack([
        x * 3.0 / TAU,                                     # a few octaves: some keys per bin
        x * 1e-3 / TAU,                                    # everything inside one bin or two
        x * 0.08 / TAU,                                    # hundreds to thousands of candidates
        np.round(x * 4.0) / TAU,                           # ties
        x * 1e6,                                           # bins past 2^24, where a bin is one fp32 value
        np.where(r.random(n) < 0.3, -np.inf, x / TAU),     # masked keys
        np.where(np.arange(n) % 7 == 0, x / TAU, np.finfo(np.float32).min),   # the same with the lowest value
        -np.abs(x) * 1e-30,                                # around zero
        tail,                                              # one key 58 octaves above all others
    ])


@pytest.mark.parametrize("n", [1, 63, 1024, 4096, 4097, 8193, 16384, 16385, 28673, 32768, 32769, 49152, 131071])
@pytest.mark.parametrize("p", [0.05, 0.9, 0.999])
def test_forms_against_the_oracle(n, p):
    S = _rows(n, n)
    sel, cnt = _select(S, p, TAU)
    for r in range(S.shape[0]):
        pu.check_topp(S[r].astype(np.float32), p, TAU, sel[r, :cnt[r]])


@pytest.mark.parametrize("n", [20000, 40000])
def test_boundary_far_below_the_maximum(n):
    """The top key alone holds less than p of the mass (0.99999953 at n = 20000, 0.99999907 at 40000), and the keys tied
    34.5 octaves below it (45 units of 2^-40 each) hold more than the rest of p: exactly these n / 2 keys."""
    S = np.zeros((1, n))
    S[0, 5] = 34.5 * math.log(2) / TAU
    S[0, n // 2:] -= 2.0 / TAU
    m = np.exp((S[0] - S[0, 5]) * TAU)
    p = float(np.float32(1.0 - 2e-7))
    assert m[5] < p * m.sum() < 0.99 * m[:n // 2].sum() + 0.01 * m[5]
    sel, cnt = _select(S, p, TAU)
    assert cnt[0] == n // 2 and np.array_equal(sel[0, :cnt[0]], np.arange(n // 2))


@pytest.mark.parametrize("n", [5000, 40000])
def test_rows_without_a_finite_maximum(n):
    """An infinite maximum leaves no key a mass: every key is selected (NaN scores add no mass)."""
    x = np.random.default_rng(n).standard_normal(n)
    S = np.stack([np.where(np.arange(n) == 77, np.inf, x), np.full(n, -np.inf), x])
    sel, cnt = _select(S, 0.9, 1.0)
    for r in (0, 1):
        assert cnt[r] == n and np.array_equal(sel[r], np.arange(n))
    S[2, 11] = np.nan
    got, c2 = _select(S[2:], 0.9, 1.0)
    want = np.setdiff1d(sel[2, :cnt[2]], [11])
    assert np.setxor1d(got[0, :c2[0]], want).size <= 2


def test_long_row_without_a_bitmap():
    """More than four sub-chunks per part: the separate call keeps no bitmap and compares the scores again."""
    n = 4_300_001
    S = (np.random.default_rng(3).standard_normal((1, n)) * 3.0 / TAU).astype(np.float32)
    sel, cnt = _select(S, 0.9, TAU)
    pu.check_topp(S[0], 0.9, TAU, sel[0, :cnt[0]])


@pytest.mark.parametrize("n,w", [(4095, 9), (32768, 0), (32771, 33), (70000, 256)])
def test_step_equals_calls(n, w):
    """The fused step selects into its bitmaps, the separate call into its workspace: the same keys and outputs."""
    wl = gen.random_case(2, 8, 2, n, seed=n, w=w, p=0.9)
    a, b = pipeline.DecodeState.from_workload(wl), pipeline.DecodeState.from_workload(wl)
    for st in (a, b):
        st.build_index()
    a.step(0.9, flush=False)
    b.step_calls(0.9, flush=False)
    torch.cuda.synchronize()
    cnt = a.sel_count.cpu().numpy()
    assert np.array_equal(cnt, b.sel_count.cpu().numpy())
    ia, ib = a.sel_idx.cpu().numpy(), b.sel_idx.cpu().numpy()
    for s in range(2):
        for h in range(8):
            assert np.array_equal(ia[s, h, :cnt[s, h]], ib[s, h, :cnt[s, h]])
    assert torch.equal(a.out, b.out) and torch.equal(a.lse, b.lse)


@pytest.mark.parametrize("n", [200, 32768, 32769])
def test_bins_at_the_end_of_the_fractions(n):
    """Products S * c of -2^23 + 1/2 and -2^23 share a bin (below -2^23 every fp32 value is an integer): p = 0.3 of 100
    keys of each is reached within the first."""
    S = np.full((1, n), -1.1e6, np.float32)
    S[0, 0:100], S[0, 100:200] = -1027875.0625, -1027875.125
    c = np.float32(np.float32(float(np.float32(TAU)) * 1.4426950408889634) * np.float32(64.0))
    assert S[0, 0] * c == np.float32(-8388607.5) and S[0, 100] * c == np.float32(-8388608.0)
    sel, cnt = _select(S, 0.3, TAU)
    assert cnt[0] == 100 and np.array_equal(sel[0, :100], np.arange(100))


@pytest.mark.parametrize("n,sigma,p", [(1 << 20, 1.5, 0.9), (1 << 20, 2.0, 0.95), (1 << 21, 1.5, 0.9)])
def test_long_gaussian_rows_are_regular(n, sigma, p):
    """Thousands of candidates in a row, some tens in each of its parts: no row of these is settled by the exact select
    of irregular ones (the fifth word of its state, the workspace's last piece), which reads a row 3 times per part."""
    S = (np.random.default_rng(n).standard_normal((1, n)) * sigma / TAU).astype(np.float32)
    dS = torch.from_numpy(S).cuda()
    sel = torch.full((1, n), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = rbq.workspace(rbq.RBQ_OP_TOPP, 1, 1, 1, 128, n)
    size = rbq.rbq_workspace_bytes(rbq.RBQ_OP_TOPP, 1, 1, 1, 128, n, 0)
    rbq.rbq_topp_select(1, 1, n, dS, p, TAU, sel, cnt, ws)
    state = ws[size - 256:size - 256 + 32].cpu().numpy().view(np.uint32)
    assert state[0] == np.float32(S.max()).view(np.uint32) and state[4] == 0
    pu.check_topp(S[0], p, TAU, sel[0, :int(cnt[0])].cpu().numpy())


@pytest.mark.parametrize("n", [4096, 8192, 8193, 12289, 16385, 32768, 32769])
def test_rows_of_few_scores(n):
    """All keys in one bin, in as many keys as one block ranks from LDS and in more: one score (every key is selected),
    and two next to each other (half of the keys hold half of the mass and a little more)."""
    one = np.full(n, 3.25, np.float32)
    two = one.copy()
    two[::2] = np.nextafter(np.float32(3.25), np.float32(4))
    sel, cnt = _select(np.stack([one, two]), 0.49, TAU)
    assert cnt[0] == n and np.array_equal(sel[0], np.arange(n))
    assert cnt[1] == (n + 1) // 2 and np.array_equal(sel[1, :cnt[1]], np.arange(0, n, 2))


def _deep_row(n, first, seed):
    """One key 37 octaves above keys `first` .. n - 1, which spread over half a nat; no other key counts. p = 1 - 2^-24
    leaves 2^-24 of the total to be found among them."""
    S = np.full(n, -1e6, np.float32)
    S[first:] = -0.5 * np.random.default_rng(seed).random(n - first)
    S[5] = 37.0 * math.log(2)
    return S, 1.0 - 2.0 ** -24


@pytest.mark.parametrize("n", [16385, 20000, 32768])
def test_masses_far_below_the_maximum(n):
    """The keys' masses are 5 to 8 units of 2^-40. Of units of 2^-48 a mass loses less than one: all of them together no
    more than 16384, which moves the boundary by at most that over the smallest mass, 2^11 e^-1/2 units."""
    S, p = _deep_row(n, n - 16384 if n > 16385 else 16, 7)
    sel, cnt = _select(S[None], p, 1.0)
    m = np.exp(S.astype(np.float64) - float(S[5]))
    order = np.argsort(-S, kind="stable")
    want = int(np.searchsorted(np.cumsum(m[order]), p * m.sum())) + 1
    assert 1000 < want < 16000
    slack = 16384 / (2.0 ** 11 * math.exp(-0.5)) + 1
    assert abs(int(cnt[0]) - want) <= slack, (cnt[0], want)
    assert np.array_equal(sel[0, :cnt[0]], np.sort(order[:cnt[0]]))


def test_a_row_alone_and_in_a_longer_batch():
    """A sequence of a ragged batch selects the keys that it selects alone, also where the batch's longest row takes the
    other form and the boundary lies where the units of the masses tell."""
    n, lens = 40000, [16384, 16385, 20000, 32768, 32769, 40000, 9000]
    S = np.full((len(lens), n), -math.inf, np.float32)
    ps = []
    for i, nr in enumerate(lens):
        if nr < 16384:
            S[i, :nr], p = np.random.default_rng(i).standard_normal(nr) * 3, 0.9
        else:
            S[i, :nr], p = _deep_row(nr, nr - 15000, i)
        ps.append(float(np.float32(p)))
    dS, B = torch.from_numpy(S).cuda(), len(lens)
    sel = torch.full((B, n), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(B, dtype=torch.int32, device="cuda")
    rbq.rbq_topp_select_varlen(B, 1, n, torch.tensor(lens, dtype=torch.int32, device="cuda"), dS,
                               torch.tensor(ps, device="cuda"), 1.0, sel, cnt,
                               rbq.workspace(rbq.RBQ_OP_TOPP, B, 1, 1, 128, n))
    sel, cnt = sel.cpu().numpy(), cnt.cpu().numpy()
    for i, nr in enumerate(lens):
        s1, c1 = _select(S[i:i + 1, :nr], ps[i], 1.0)
        assert cnt[i] == c1[0] and np.array_equal(sel[i, :cnt[i]], s1[0, :c1[0]]), nr


@pytest.mark.parametrize("n,spread", [(1 << 19, 0.8), (1 << 20, 1.5)])
def test_step_equals_calls_on_long_rows(n, spread):
    """The same where a row has thousands of candidates (normal scores of `spread` nats): step and calls settle it alike,
    by sums of the same form."""
    H, D = 2, 64
    g = torch.Generator(device="cuda").manual_seed(n)
    K, V = (torch.randn(1, H, n, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(1, H, D, device="cuda", generator=g)
    q *= spread * math.sqrt(D) / q.norm(dim=2, keepdim=True)
    st = pipeline.DecodeState(1, H, H, D, n, n, 0, K, V, q, torch.from_numpy(gen.haar_rotation(D)).cuda())
    st.build_index()
    got = []
    for step in (st.step_calls, st.step):
        st.sel_idx.fill_(-1)
        step(0.9, flush=False)
        got.append([t.clone() for t in (st.scores, st.sel_count, st.sel_idx, st.out, st.lse)])
    for x, y in zip(*got):
        assert torch.equal(x, y)
    assert 0.2 * n < int(got[0][1][0, 0]) < 0.95 * n
