"""Chunk B's input- and weight-gradient products in one launch where both are small:
outputs and gradient equal, bit for bit, the same backward with a launch for each (the
split backward, and a stage whose weight products are timed), at sizes that combine the
32 and 64 tiles in every way (input gradient with weight gradient, both epilogues), the
fp32 pair, sizes too large to pair, grouped-query attention and a mixture of experts."""
import pytest
import torch

from paper_2606_11169_amd import libchunk as lc
from paper_2606_11169_amd.runner import random_stage
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu


def run(desc, split, timed):
    r = random_stage(desc, 2, seed=3, max_w_pending=2)
    r.alloc_random_microbatches(2, seed=4)
    if timed:
        lc.lc_stage_timer_enable(r.stage, 1000)
    r.zero_grad()
    r.run_order(lc.lc_order_1f1b_split(2, 2, 0, 0) if split else lc.lc_order_1f1b(2, 2, 0))
    torch.cuda.synchronize()
    out = [t.clone() for t in (*r.Y, *r.dX, r.grad)]
    r.close()
    return out


@pytest.mark.parametrize("bf16,d,heads,f,seq,batch,more", [
    (True, 256, 2, 128, 128, 1, {}), (True, 512, 4, 1408, 256, 1, {}), (True, 640, 5, 704, 384, 1, {}),
    (True, 384, 3, 1024, 128, 3, {}), (True, 1024, 8, 2816, 512, 1, {}),
    # SwiGLU backward of 64 tiles with a weight gradient of 32 and the other way round;
    # a stored input gradient of 64 with 32
    (True, 256, 2, 704, 512, 1, {}), (True, 512, 4, 1408, 128, 1, {}), (True, 256, 2, 704, 256, 5, {}),
    (True, 512, 4, 704, 256, 1, {"n_kv_heads": 2, "qk_norm": True}),
    (True, 256, 2, 320, 128, 2, {"n_experts": 4, "top_k": 2, "d_ff_expert": 320}),
    (False, 128, 4, 344, 64, 2, {}), (False, 96, 3, 250, 40, 1, {}), (False, 512, 8, 1024, 130, 2, {})])
def test_one_launch_or_two(bf16, d, heads, f, seq, batch, more):
    banner(f"grad pairs bf16={bf16} d={d} f={f} T={seq}x{batch} {more}")
    desc = lc.make_desc(2, d, heads, d // heads, f, seq, batch, bf16, **more)
    ref = run(desc, True, False)
    for timed in (False, True):
        for a, b in zip(ref, run(desc, False, timed)):
            assert torch.equal(a, b)
    assert all(bool(torch.isfinite(t).all()) for t in ref)
