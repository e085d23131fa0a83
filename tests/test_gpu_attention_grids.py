"""The attention kernels' workgroup shapes (256 queries; 128 queries with the
keys split over two wave groups, for small grids; dQ and dK/dV in one grid
up to 256 blocks of each) at sequence lengths
whose last block is half full and whose first block leaves the second group
without a visible key: against float64 of the same fp16/bf16 q, k, v."""
import math

import pytest
import torch

from paper_2606_11169_amd import libchunk as lc
from tests.gpu_util import DEV, banner

pytestmark = pytest.mark.gpu


def rel(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("dt", ["fp16", "bf16"])
@pytest.mark.parametrize("B,S,H,kv", [(1, 128, 1, 1), (2, 384, 2, 1), (1, 1152, 3, 3), (2, 1152, 16, 4),
                                      (8, 384, 32, 32),
                                      (16, 256, 32, 8), (2, 128, 70, 35)])
def test_both_shapes(B, S, H, kv, dt):
    banner(f"attention grids B={B} S={S} H={H}/{kv} {dt}")
    tdt, ldt = (torch.float16, lc.LC_FP16) if dt == "fp16" else (torch.bfloat16, lc.LC_BF16)
    g = torch.Generator(device=DEV)
    g.manual_seed(S + H)
    T, ld = B * S, (H + 2 * kv) * 128
    qkv = torch.randn((T, ld), generator=g, device=DEV).to(tdt)
    dout = torch.randn((T, H * 128), generator=g, device=DEV).to(torch.bfloat16)
    o, dqkv = torch.empty_like(dout), torch.empty((T, ld), dtype=torch.bfloat16, device=DEV)
    lse = torch.empty((B, H, S), device=DEV)
    q, dq = qkv.data_ptr(), dqkv.data_ptr()
    off = (H * 256, (H + kv) * 256)
    lc.lc_attention_forward(ldt, lc.LC_BF16, B, S, H, 128, q, q + off[0], q + off[1], ld, o, H * 128,
                            lse, Hkv=kv)
    nb = lc.lc_attention_scratch_bytes(B, S, H, kv)
    scratch = torch.empty(nb, dtype=torch.uint8, device=DEV)
    lc.lc_attention_backward(ldt, lc.LC_BF16, B, S, H, 128, q, q + off[0], q + off[1], ld, o, dout,
                             H * 128, lse, dq, dq + off[0], dq + off[1], ld, None, None, scratch, nb,
                             Hkv=kv)
    mask = torch.ones((S, S), dtype=torch.bool, device=DEV).triu(1)
    x = qkv.view(B, S, H + 2 * kv, 128)
    ro, rl = torch.empty((B, S, H, 128), dtype=torch.float64, device=DEV), torch.empty_like(lse, dtype=torch.float64)
    rg = torch.zeros((B, S, H + 2 * kv, 128), dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(H):
            j = H + h * kv // H
            t = [x[b, :, i].double().requires_grad_() for i in (h, j, j + kv)]
            sc = (t[0] @ t[1].t() / math.sqrt(128)).masked_fill(mask, -math.inf)
            oh = torch.softmax(sc, -1) @ t[2]
            oh.backward(dout.view(B, S, H, 128)[b, :, h].double())
            ro[b, :, h], rl[b, h] = oh.detach(), torch.logsumexp(sc, -1).detach()
            rg[b, :, h] += t[0].grad
            rg[b, :, j] += t[1].grad
            rg[b, :, j + kv] += t[2].grad
    # P to 16 bits (2^-9 for bf16), outputs to bf16: 2^-8 in the 2-norm covers both;
    # the gradients' products round P, dS and their operands once more each
    assert rel(o.view_as(ro), ro) < 2 ** -8
    assert rel(lse, rl) < 1e-5
    assert rel(dqkv.view_as(rg), rg) < 2 ** -6.5


@pytest.mark.parametrize("dt", ["fp16", "bf16"])
@pytest.mark.parametrize("B,S,H,kv", [(1, 1024, 4, 4), (1, 2048, 16, 16), (1, 1024, 4, 2)])
def test_key_gradients_in_place(B, S, H, kv, dt):
    """dk, dv over k, v give what separate buffers give (sizes at which dQ and dK/dV
    otherwise share a grid). The sums that form D and dQ may then be added in another
    order: a few fp32 roundings before the one to bf16, so at most a small share of the
    values one bf16 step (2^-8) apart."""
    banner(f"attention key gradients in place B={B} S={S} H={H}/{kv} {dt}")
    tdt, ldt = (torch.float16, lc.LC_FP16) if dt == "fp16" else (torch.bfloat16, lc.LC_BF16)
    g = torch.Generator(device=DEV)
    g.manual_seed(S + H)
    T, d, dkv = B * S, H * 128, kv * 128
    q = torch.randn((T, d), generator=g, device=DEV).to(tdt)
    k, v = (torch.randn((T, d), generator=g, device=DEV).to(tdt) for _ in range(2))  # rows of d: one stride
    dout = torch.randn((T, d), generator=g, device=DEV).to(torch.bfloat16)
    o, lse = torch.empty_like(dout), torch.empty((B, H, S), device=DEV)
    lc.lc_attention_forward(ldt, lc.LC_BF16, B, S, H, 128, q, k, v, d, o, d, lse, Hkv=kv)
    nb = lc.lc_attention_scratch_bytes(B, S, H, kv)
    scratch = torch.empty(nb, dtype=torch.uint8, device=DEV)

    def backward(dk, dv):
        dq = torch.empty_like(dout)
        lc.lc_attention_backward(ldt, lc.LC_BF16, B, S, H, 128, q, k, v, d, o, dout, d, lse, dq, dk, dv, d,
                                 None, None, scratch, nb, Hkv=kv)
        return [t.view(torch.bfloat16)[:, :w].clone() for t, w in ((dq, d), (dk, dkv), (dv, dkv))]

    want = backward(torch.empty_like(dout), torch.empty_like(dout))
    got = backward(k, v)
    for a, b in zip(got, want):
        assert bool(torch.isfinite(b).all())
        assert rel(a, b.double()) < 2 ** -10
