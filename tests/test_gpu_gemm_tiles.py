"""The bf16 GEMM's output tiles (256, 128, 64 and 32, chosen by the product's size)
at the edges of tiles, rings and k-steps, against float64 products of the same
operands: the plain and accumulating products in every layout on every tile, the
residual add on every tile, the SwiGLU and RoPE epilogues on every tile and (the
rounding test) with other element types than the stages'. Integer-valued operands
make the plain products exact in fp32 (|sum| < 2^24), so those are compared bit for
bit."""
import numpy as np
import pytest
import torch

from paper_2606_11169_amd import libchunk as lc
from tests.gpu_util import DEV, banner

pytestmark = pytest.mark.gpu

BF16, FP32, FP16 = lc.LC_BF16, lc.LC_FP32, lc.LC_FP16
# (M, N): 32 tiles, 64 tiles, 128 tiles (over 256 of 64, ragged both ways; m/n-major
# rows need a multiple of 8), 256 tiles
SIZES = [(1, 8), (72, 136), (520, 712), (1096, 1928), (1480, 6152)]
# stages of 256 (32 tile), 128 (64 tile) or 64 (128, 256): none full, one, the ring's wrap, a
# ragged last stage
DEPTHS = [8, 128, 200, 520, 1032, 2056]


def ints(g, *shape):
    return torch.randint(-4, 5, shape, generator=g, device=DEV).to(torch.bfloat16)


def gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


@pytest.mark.parametrize("layout", [(1, 1), (1, 0), (0, 0)], ids=["NT", "NN", "TN"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_tiles_bit_exact(size, layout):
    M, N = size
    ak, bk = layout
    if not ak:
        M = (M + 7) // 8 * 8
    for K in DEPTHS:
        banner(f"gemm tiles {M}x{N}x{K} layout {layout}")
        g = gen(M + N + K)
        A, B = ints(g, *((M, K) if ak else (K, M))), ints(g, *((N, K) if bk else (K, N)))
        ref = (A if ak else A.t()).double() @ (B if bk else B.t()).double().t()
        C = torch.full((M + 1, N), -3.0, dtype=torch.float32, device=DEV)
        lc.lc_gemm(BF16, lc.LC_EPI_STORE_F32, M, N, K, A, A.shape[1], ak, B, B.shape[1], bk, C, N)
        assert torch.equal(C[:M].double(), ref)
        assert bool((C[M] == -3.0).all())
        if ak == bk:  # the accumulating epilogue adds the same sum once
            lc.lc_gemm(BF16, lc.LC_EPI_ACCUM_F32, M, N, K, A, A.shape[1], ak, B, B.shape[1], bk, C, N)
            assert torch.equal(C[:M].double(), 2 * ref)
            assert bool((C[M] == -3.0).all())


def rel(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("T,f,d", [(40, 64, 264), (520, 320, 520), (1003, 960, 136), (2056, 3136, 72)])
def test_tiles_swiglu_and_residual(T, f, d):
    """Gate/up with SwiGLU, down with the residual and the SwiGLU backward. The
    sums are exact, so gate and up are too; bf16 outputs are one rounding off
    (2^-9 relative each, a 2-norm of 2^-9), fp32 ones a few fp32 roundings and
    the hardware reciprocal's ulp."""
    banner(f"gemm tiles swiglu T={T} f={f} d={d}")
    g = gen(T + f + d)
    x, w13 = ints(g, T, d), ints(g, 2 * f, d)
    gate, up = (torch.empty((T, f), dtype=torch.float32, device=DEV) for _ in range(2))
    act = torch.empty((T, f), dtype=torch.bfloat16, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_SWIGLU, T, f, d, x, d, 1, w13, d, 1, act, f, aux0=gate, aux1=up,
               ld_aux=f, aux_dtype=FP32)
    gr, ur = x.double() @ w13[:f].double().t(), x.double() @ w13[f:].double().t()
    assert torch.equal(gate.double(), gr) and torch.equal(up.double(), ur)
    sg = torch.sigmoid(gr)
    assert rel(act, gr * sg * ur) < 2 ** -9
    w2, h = ints(g, d, f), torch.randn((T, d), generator=g, device=DEV)
    a2 = ints(g, T, f)
    y = torch.empty((T, d), dtype=torch.float32, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_RESIDUAL, T, d, f, a2, f, 1, w2, f, 1, y, d, R=h, ldr=d,
               c_dtype=FP32, r_dtype=FP32)
    assert rel(y, h.double() + a2.double() @ w2.double().t()) < 1e-6
    dy = ints(g, T, d)
    da = torch.empty((T, 2 * f), dtype=torch.bfloat16, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_SWIGLU_BWD, T, f, d, dy, d, 1, w2, f, 0, da, 2 * f, aux0=gate,
               aux1=up, ld_aux=f, aux_dtype=FP32)
    dact = dy.double() @ w2.double()
    assert rel(da[:, :f], dact * ur * sg * (1 + gr * (1 - sg))) < 2 ** -9
    assert rel(da[:, f:], dact * gr * sg) < 2 ** -9


@pytest.mark.parametrize("types", ["fp32", "bf16 residual", "bf16 result"])
@pytest.mark.parametrize("T,N,K", [(20, 264, 64), (520, 520, 320), (1003, 1928, 960), (1480, 6152, 328)])
def test_tiles_residual(T, N, K, types):
    """The residual add, ragged both ways: the sums are exact; one fp32 rounding, and one
    to bf16 (2^-9 relative) where the result is bf16."""
    banner(f"gemm tiles residual {T}x{N}x{K} {types}")
    g = gen(T + N)
    a, w = ints(g, T, K), ints(g, N, K)
    h = torch.randn((T, N), generator=g, device=DEV)
    h = h.to(torch.bfloat16) if types == "bf16 residual" else h
    y = torch.full((T + 1, N), -3.0, dtype=torch.bfloat16 if types == "bf16 result" else torch.float32, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_RESIDUAL, T, N, K, a, K, 1, w, K, 1, y, N, R=h, ldr=N,
               c_dtype=BF16 if types == "bf16 result" else FP32,
               r_dtype=BF16 if types == "bf16 residual" else FP32)
    ref = h.double() + a.double() @ w.double().t()
    assert rel(y[:T], ref) < (2 ** -9 if types == "bf16 result" else 1e-6)
    assert bool((y[T] == -3.0).all())


@pytest.mark.parametrize("T,H,seq", [(40, 1, 8), (520, 2, 130), (1003, 5, 59), (1480, 16, 1480)])
def test_tiles_rope(T, H, seq):
    """q|k|v of H heads each, q and k rotated, with the bf16 copy."""
    banner(f"gemm tiles rope T={T} H={H}")
    g = gen(T + H)
    N, K = 3 * H * 128, 72
    x, w = ints(g, T, K), ints(g, N, K)
    ang = torch.rand((seq, 64), generator=g, device=DEV)
    cos, sin = torch.cos(ang), torch.sin(ang)
    q = torch.empty((T, N), dtype=torch.float16, device=DEV)
    qb = torch.empty((T, N), dtype=torch.bfloat16, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_ROPE, T, N, K, x, K, 1, w, K, 1, q, N, aux0=qb, ld_aux=N,
               rope_cos=cos, rope_sin=sin, rope_seq=seq, rope_cols=2 * H * 128, head_dim=128,
               c_dtype=FP16, aux_dtype=BF16)
    ref = (x.double() @ w.double().t()).view(T, 3 * H, 128)
    pos = torch.arange(T, device=DEV) % seq
    c, s = cos.double()[pos, None], sin.double()[pos, None]
    a, b = ref[:, :2 * H, :64].clone(), ref[:, :2 * H, 64:].clone()
    ref[:, :2 * H, :64], ref[:, :2 * H, 64:] = a * c - b * s, a * s + b * c
    assert rel(q.view(T, 3 * H, 128), ref) < 2 ** -11
    assert rel(qb.view(T, 3 * H, 128), ref) < 2 ** -8


def test_epilogues_round_alike_on_every_tile():
    """RoPE, SwiGLU and the SwiGLU backward of 1480, 520, 40 and 20 rows (256, 128, 64 and 32
    tiles): exact sums, so the same rows get the same bits."""
    banner("gemm tiles, epilogue bits")
    g = gen(7)
    T, N, K = 1480, 6144, 72
    x, w = ints(g, T, K), ints(g, 2 * N, K)
    ang = torch.rand((T, 64), generator=g, device=DEV) * 6
    cos, sin = torch.cos(ang), torch.sin(ang)
    gate, up = (torch.randn((T, N), generator=g, device=DEV) for _ in range(2))

    def rope(rows, types):
        q, qb = (torch.empty((rows, N), dtype=t[0], device=DEV) for t in types)
        lc.lc_gemm(BF16, lc.LC_EPI_ROPE, rows, N, K, x, K, 1, w, K, 1, q, N, aux0=qb, ld_aux=N, rope_cos=cos,
                   rope_sin=sin, rope_seq=T, rope_cols=N // 2, head_dim=128, c_dtype=types[0][1],
                   aux_dtype=types[1][1])
        return q, qb

    def swiglu(rows, c, aux):
        h = N // 2
        act = torch.empty((rows, h), dtype=c[0], device=DEV)
        a0, a1 = (torch.empty((rows, h), dtype=aux[0], device=DEV) for _ in range(2))
        lc.lc_gemm(BF16, lc.LC_EPI_SWIGLU, rows, h, K, x, K, 1, w, K, 1, act, h, aux0=a0, aux1=a1, ld_aux=h,
                   c_dtype=c[1], aux_dtype=aux[1])
        return act, a0, a1

    def swiglu_bwd(rows, c, nt):
        b = w[:N] if nt else w[:N].t().contiguous()
        da = torch.empty((rows, 2 * N), dtype=c[0], device=DEV)
        lc.lc_gemm(BF16, lc.LC_EPI_SWIGLU_BWD, rows, N, K, x, K, 1, b, b.shape[1], int(nt), da, 2 * N, aux0=gate,
                   aux1=up, ld_aux=N, c_dtype=c[1], aux_dtype=FP32)
        return (da,)

    f32, f16, b16 = (torch.float32, FP32), (torch.float16, FP16), (torch.bfloat16, BF16)
    for call in (lambda r: rope(r, (f16, b16)), lambda r: rope(r, (f32, f32)), lambda r: swiglu(r, b16, f32),
                 lambda r: swiglu(r, f32, f16), lambda r: swiglu_bwd(r, b16, False),
                 lambda r: swiglu_bwd(r, f32, False), lambda r: swiglu_bwd(r, b16, True)):
        full = call(T)
        for rows in (520, 40, 20):
            for a, b in zip(call(rows), full):
                assert torch.equal(a, b[:rows])
    # and the values: the stage's types against float64
    (da,) = swiglu_bwd(T, f32, True)
    v, sg = x.double() @ w[:N].double().t(), torch.sigmoid(gate.double())
    assert rel(da[:, :N], v * up.double() * sg * (1 + gate.double() * (1 - sg))) < 1e-6
    assert rel(da[:, N:], v * gate.double() * sg) < 1e-6


@pytest.mark.parametrize("sizes,N", [([30, 0, 50, 1], 72), ([300, 0, 17, 512, 256, 1], 264),
                                     ([900, 40, 0, 700], 1416)], ids=["32", "64", "128"])
def test_tiles_grouped(sizes, N):
    banner(f"gemm tiles grouped {sizes} N={N}")
    g = gen(N)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    G, R, K = len(sizes), int(off[-1]) + 40, 328
    offd = torch.from_numpy(off).to(DEV)
    A, B = ints(g, R, K), ints(g, G, N, K)
    C = torch.full((R, N), -3.0, dtype=torch.float32, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_STORE_F32, R, N, K, A, K, 1, B, K, 1, C, N, group_mode=1,
               n_groups=G, group_offsets=offd, group_stride_b=N * K)
    for e in range(G):
        r = slice(off[e], off[e + 1])
        assert torch.equal(C[r].double(), A[r].double() @ B[e].double().t()), e
    assert bool((C[off[-1]:] == -3.0).all())
    # weight gradients: k runs over each group's rows
    M = 200
    X, Y = ints(g, R, M), ints(g, R, N)
    D = torch.ones((G, M, N), dtype=torch.float32, device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_ACCUM_F32, M, N, R, X, M, 0, Y, N, 0, D, N, group_mode=2,
               n_groups=G, group_offsets=offd, group_stride_c=M * N)
    for e in range(G):
        r = slice(off[e], off[e + 1])
        assert torch.equal(D[e].double(), 1 + X[r].double().t() @ Y[r].double()), e


@pytest.mark.parametrize("sizes,N,K", [
    ([900, 0, 2000, 129, 1, 1671, 128, 700], 1160, 520), ([33 * i % 257 for i in range(64)], 520, 512),
    ([0, 0, 0, 12000], 264, 520), ([700, 0, 1300, 128, 1, 900], 1416, 504)],
    ids=["uneven", "64groups", "one", "few_k"])
def test_tiles_grouped_mapped_to_xcds(sizes, N, K):
    """Over 264 tiles of 128, which the map spreads over the XCDs by the tiles that the groups
    have (few_k: in launch order): every row of a group, none past the last. Integers: exact."""
    banner(f"gemm tiles grouped, mapped {len(sizes)} groups N={N} K={K}")
    assert sum(-(-n // 128) for n in sizes) * -(-N // 128) > 264
    g = gen(N + K)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    G, R = len(sizes), int(off[-1]) + 40
    offd = torch.from_numpy(off).to(DEV)
    A, B = ints(g, R, K), ints(g, G, N, K)
    Bt = B.transpose(1, 2).contiguous()
    for b, kmajor in ((B, 1), (Bt, 0)):
        C = torch.full((R, N), -3.0, dtype=torch.float32, device=DEV)
        lc.lc_gemm(BF16, lc.LC_EPI_STORE_F32, R, N, K, A, K, 1, b, K if kmajor else N, kmajor, C, N,
                   group_mode=1, n_groups=G, group_offsets=offd, group_stride_b=N * K)
        for e in range(G):
            r = slice(off[e], off[e + 1])
            assert torch.equal(C[r].double(), A[r].double() @ B[e].double().t()), e
        assert bool((C[off[-1]:] == -3.0).all())


def test_widest_grouped_output():
    """64 groups, eight of one row each, of 30 million columns: the smaller tiles' upper
    bound of workgroups passes what a launch takes. Integer operands: exact."""
    G, N, K = 64, 30_000_000, 8
    banner(f"gemm tiles grouped 8x{N}x{K}")
    g = gen(G)
    A, B = ints(g, 8, K), ints(g, N, K)
    off = torch.tensor([min(i, 8) for i in range(G + 1)], dtype=torch.int32, device=DEV)
    C = torch.zeros((8, N), device=DEV)
    lc.lc_gemm(BF16, lc.LC_EPI_STORE_F32, 8, N, K, A, K, 1, B, K, 1, C, N, group_mode=1, n_groups=G,
               group_offsets=off, group_stride_b=0)
    assert torch.equal(C, A.float() @ B.float().t())
