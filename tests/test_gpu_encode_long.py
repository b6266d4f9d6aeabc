"""The encoder of long runs (more than 4096 new keys per head: two fp16 parts per
value on the matrix cores) against the oracle, at its edges: the first size it
takes, ragged last tiles, fewer and more (sequence, head) groups than its blocks,
both head dimensions and key types, scales far from one, and degenerate keys."""
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
    # the parts hold 22 bits: each component within 2^-21 of itself
    assert ((rot[0, 0] - K[0, 0].float()).abs() <= 2.0 ** -21 * K[0, 0].float().abs()).all()


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("kv", ["bf16", "f32"])
@pytest.mark.parametrize("n", [40000, 4100])
def test_every_sign_is_that_of_64_bits(D, kv, n):
    """Components within rounding of zero are formed again in 64 bits: no bit differs from the sign there, with some
    components of each key made small on purpose (n = 4100: every key, through P's columns)."""
    H = 6
    g = torch.Generator(device="cuda").manual_seed(n + D)
    P = torch.from_numpy(gen.haar_rotation(D)).cuda()
    K = torch.randn(1, H, n, D, device="cuda", generator=g)
    if n == 4100:   # r ~ 1e-7 in two components of every key, on either side of zero
        r = torch.randn(1, H, n, D, device="cuda", generator=g).double()
        r[..., 5] *= 1e-7
        r[..., D - 2] *= 1e-7
        K = (r @ P.double().T).float()
    K = K.to(torch.bfloat16 if kv == "bf16" else torch.float32).contiguous()
    ck, codes, _, _, _ = _encode(K, P, None, rot=False)
    r = (K[0].double() - ck[0].double()[:, None]) @ P.double()
    bits = torch.stack([(codes[0, :, :, d // 32] >> (d % 32)) & 1 for d in range(D)], 2).bool()
    assert int((bits != (r > 0)).sum()) == 0
