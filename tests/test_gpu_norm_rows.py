"""RMSNorm backward at the edges of its row shapes (one to eight waves per row,
one or two chunks per lane, rows too long for registers) and of the 16-row blocks,
against float64, for the stages' type mixes and a mixed one."""
import pytest
import torch

from paper_2606_11169_amd import libchunk as lc
from tests.gpu_util import DEV, banner

pytestmark = pytest.mark.gpu
F32, BF16 = lc.LC_FP32, lc.LC_BF16
DT = {F32: torch.float32, BF16: torch.bfloat16}


@pytest.mark.parametrize("x,w,dres,out", [(F32, BF16, F32, F32), (F32, BF16, BF16, F32), (BF16, BF16, F32, BF16),
                                          (F32, F32, F32, F32), (BF16, F32, None, F32)])
@pytest.mark.parametrize("T,d", [(1, 8), (17, 512), (33, 520), (16, 1024), (40, 1032), (15, 2048), (50, 2056),
                                 (31, 4104), (18, 8192), (18, 8200)])
def test_backward(T, d, x, w, dres, out):
    banner(f"rmsnorm rows T={T} d={d} {x}{w}{dres}{out}")
    g = torch.Generator(device=DEV)
    g.manual_seed(T + d)
    xs = torch.randn((T, d), generator=g, device=DEV).to(DT[x])
    gain = (1 + 0.1 * torch.randn(d, generator=g, device=DEV)).to(DT[w])
    dn = torch.randn((T, d), generator=g, device=DEV)
    dr = None if dres is None else torch.randn((T, d), generator=g, device=DEV).to(DT[dres])
    rstd = torch.empty(T, device=DEV)
    n = torch.empty((T, d), dtype=DT[w], device=DEV)
    lc.lc_rmsnorm_forward(T, d, xs, gain, 1e-5, n, rstd, x, w, w)
    dx = torch.empty((T, d), dtype=DT[out], device=DEV)
    cp = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
    dg0 = torch.randn(d, generator=g, device=DEV)
    dg = dg0.clone()
    nb = lc.lc_rmsnorm_scratch_bytes(T, d)
    scratch = torch.full((nb // 4 + 64,), -3.0, device=DEV)
    lc.lc_rmsnorm_backward(T, d, dn, xs, rstd, gain, dr, dx, dg, scratch, nb, F32, x, w,
                           F32 if dres is None else dres, out, dx_copy=cp)
    xd, gd, dd = xs.double(), gain.double(), dn.double()
    r = torch.rsqrt(xd.square().mean(-1, keepdim=True) + 1e-5)
    dxh = dd * gd
    ref = r * (dxh - xd * r * (dxh * xd * r).mean(-1, keepdim=True))
    if dr is not None:
        ref = ref + dr.double()

    def rel(a, b):
        return float((a.double() - b).norm() / b.norm())

    assert rel(n, xd * r * gd) < (2 ** -8 if w == BF16 else 1e-6)  # bf16: one rounding
    assert rel(dx, ref) < (2 ** -8 if out == BF16 else 1e-6)
    assert rel(cp, ref) < 2 ** -8
    assert rel(dg, dg0.double() + (dd * xd * r).sum(0)) < 1e-6
    assert bool((scratch[nb // 4:] == -3.0).all())
