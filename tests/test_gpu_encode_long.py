"""The encoder on long runs of keys (a prefill) against the oracle: more keys than
any window, ragged last tiles, few and many (sequence, head) groups, both head
dimensions and key types, scales far from one, degenerate keys, and the same rows
whether a run is encoded whole or in pieces."""
import math

import numpy as np
import pytest
import torch

import parity_util as pu
from paper_2606_31519_amd import rbq
from workloads import gen

pytestmark = pytest.mark.gpu


def _encode(K, P, c_q, c_k=None, offset=0, pad=0, rot=True):
    B, H, n, D = K.shape
    cap = n + offset + pad
    f = dict(dtype=torch.float32, device="cuda")
    ck = torch.zeros(B, H, D, **f) if c_k is None else c_k
    codes = torch.full((B, H, cap, D // 32), -1, dtype=torch.int32, device="cuda")
    kfac = torch.full((B, H, cap, 2), -7.0, **f)
    alpha = torch.zeros(B, H, n, **f)
    rot_out = torch.zeros(B, H, n, D, **f) if rot else None
    flags = rbq.RBQ_ENCODE_SET_CENTROID if c_k is None else 0
    ws = rbq.workspace(rbq.RBQ_OP_ENCODE, B, H, H, D, n)
    rbq.rbq_encode_keys(B, H, D, K, n, n, offset, cap, P, c_q, ck, codes, kfac, flags, alpha, ws, rot_out=rot_out)
    torch.cuda.synchronize()
    return ck, codes, kfac, alpha, rot_out


@pytest.mark.parametrize("B,H,n,D,kv,scale,offset", [
    (1, 1, 4097, 128, "bf16", 1.0, 0), (2, 3, 4127, 128, "bf16", 1.0, 5), (1, 2, 9000, 128, "f32", 1.0, 0),
    (1, 2, 4100, 64, "bf16", 1.0, 3), (2, 1, 5001, 64, "f32", 1.0, 0), (1, 1, 4200, 128, "bf16", 1e-18, 0),
    (1, 1, 4200, 128, "f32", 1e15, 0), (1, 1, 33000, 128, "bf16", 1.0, 0)])
def test_against_the_oracle(B, H, n, D, kv, scale, offset):
    wl = gen.random_case(B, H, H, n, D=D, seed=n, kv_dtype="f32", c_q_scale=0.5, key_offset=1.0)
    dt = torch.bfloat16 if kv == "bf16" else torch.float32
    K = (torch.from_numpy(wl.K[:, :, :n]) * scale).to(dt).cuda().contiguous()
    c_q = torch.from_numpy(wl.c_q).cuda()
    P = torch.from_numpy(wl.P).cuda()
    ck, codes, kfac, alpha, rot = _encode(K, P, c_q, offset=offset, pad=2)
    assert (codes[:, :, :offset] == -1).all() and (codes[:, :, offset + n:] == -1).all()
    assert (kfac[:, :, :offset] == -7).all() and (kfac[:, :, offset + n:] == -7).all()
    flips = 0
    for b in range(B):
        for h in range(H):
            k64 = K[b, h].float().cpu().numpy().astype(np.float64)
            c = pu.u32(codes)[b, h, offset:offset + n]
            # (factors and centroid in units of the scale: the checks' absolute terms are meant for keys near 1)
            fac = kfac[b, h, offset:offset + n].cpu().numpy().astype(np.float64)
            flips += pu.check_encode_group(c, fac / scale, ck[b, h].cpu().numpy().astype(np.float64) / scale, k64 / scale,
                                           wl.P, wl.c_q[b, h], rot=rot[b, h].cpu().numpy().astype(np.float64) / scale,
                                           alpha=alpha[b, h].cpu().numpy())
    assert flips <= 1e-5 * B * H * n * D   # |r| within rounding of zero: about 1e-7 of the components


def test_more_groups_than_blocks():
    B, H, n, D = 75, 4, 4097, 64
    g = torch.Generator(device="cuda").manual_seed(1)
    K = torch.randn(B, H, n, D, device="cuda", generator=g).to(torch.bfloat16)
    P = torch.from_numpy(gen.haar_rotation(D)).cuda()
    ck, codes, kfac, alpha, _ = _encode(K, P, None, rot=False)
    for b, h in ((0, 0), (37, 2), (74, 3)):
        pu.check_encode_group(pu.u32(codes[b, h]), kfac[b, h].cpu().numpy(), ck[b, h].cpu().numpy(),
                              K[b, h].double().cpu().numpy(), P.cpu().numpy(), None)


def test_zero_components_and_keys_at_the_centroid():
    """With P = I the rotated components are the centred keys' own: an exact zero gives bit 0, and a key equal to the
    centroid gives no bits and f = 0. One component far above the others leaves the small ones their signs."""
    n, D = 4100, 128
    x = torch.randn(1, 1, n, D, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    x[0, 0, ::3, ::5] = 0.0
    x[0, 0, 7] = 0.0
    x[0, 0, 11] = -0.0
    x[0, 0, 13, 4] = 3e4
    K = x.to(torch.bfloat16)
    zero = torch.zeros(1, 1, D, device="cuda")
    _, codes, kfac, _, rot = _encode(K, torch.eye(D, device="cuda"), None, c_k=zero)
    bits = np.unpackbits(pu.u32(codes[0, 0]).view(np.uint8), axis=1, bitorder="little").astype(bool)
    assert np.array_equal(bits, (K[0, 0] > 0).cpu().numpy())
    assert kfac[0, 0, 7, 0] == 0 and kfac[0, 0, 11, 0] == 0
    assert torch.equal(rot[0, 0], K[0, 0].float())


@pytest.mark.parametrize("D,kv", [(128, "bf16"), (64, "bf16"), (128, "f32")])
def test_rebuilt_index_is_the_appended_one(D, kv):
    """A run of keys has the rows of the same keys appended piece by piece (rebuilding an index that windows were flushed
    into changes none of it), for every rotation, and a key that is no number gives no number in both."""
    H, n = 2, 9001
    g = torch.Generator(device="cuda").manual_seed(D)
    K = torch.randn(1, H, n, D, device="cuda", generator=g)
    K[0, 0, 5, 3], K[0, 1, 4500, 0], K[0, 1, 8999, 1] = math.inf, math.nan, -math.inf
    K = K.to(torch.bfloat16 if kv == "bf16" else torch.float32)
    ck = torch.randn(1, H, D, device="cuda", generator=g)
    had = torch.ones(1, 1, device="cuda")
    while had.shape[0] < D:
        had = torch.cat([torch.cat([had, had], 1), torch.cat([had, -had], 1)])
    signs = torch.randint(0, 2, (D, 1), device="cuda", generator=g).float() * 2 - 1
    for P in (torch.from_numpy(gen.haar_rotation(D)).cuda(), torch.eye(D, device="cuda"), signs * had / math.sqrt(D)):
        P = P.contiguous()
        for c_q in (torch.randn(1, H, D, device="cuda", generator=g), torch.zeros(1, H, D, device="cuda")):
            _, codes, kfac, alpha, rot = _encode(K, P, c_q, c_k=ck)
            for lo, hi in ((0, 4096), (4096, 4097), (4097, 8193), (8193, n)):
                _, c1, f1, a1, r1 = _encode(K[:, :, lo:hi].contiguous(), P, c_q, c_k=ck)
                assert torch.equal(c1, codes[:, :, lo:hi])
                for whole, piece in ((kfac, f1), (alpha, a1), (rot, r1)):
                    assert torch.equal(whole[:, :, lo:hi].nan_to_num(nan=7e30), piece.nan_to_num(nan=7e30))
            assert bool(kfac[0, 1, 4500, 1].isnan())


def test_whole_values_through_a_permutation():
    """Every bit of a key takes part in its rotated components: a P that only permutes and negates gives them exactly,
    however far apart a key's components are."""
    n, D = 4099, 128
    g = torch.Generator(device="cuda").manual_seed(4)
    K = torch.randn(1, 1, n, D, device="cuda", generator=g)
    K *= torch.exp2(torch.randint(-60, 60, (1, 1, n, D), device="cuda", generator=g).float())
    perm = torch.randperm(D, device="cuda", generator=g)
    sign = torch.randint(0, 2, (D,), device="cuda", generator=g).float() * 2 - 1
    P = torch.zeros(D, D, device="cuda")
    P[perm, torch.arange(D, device="cuda")] = sign
    _, codes, _, _, rot = _encode(K, P, None, c_k=torch.zeros(1, 1, D, device="cuda"))
    want = K[0, 0][:, perm] * sign
    assert torch.equal(rot[0, 0], want)
    bits = np.unpackbits(pu.u32(codes[0, 0]).view(np.uint8), axis=1, bitorder="little").astype(bool)
    assert np.array_equal(bits, (want > 0).cpu().numpy())
