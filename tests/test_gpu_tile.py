"""The tiled GEMM (more than 16 activation rows) against plain products in 64 bits: every
block shape that is built, in every format, with fp16 and with int8 activations
(test_tile_plan.py checks on the CPU that the sizes here select each of them), chunk counts
1, 2, 3 and odd ones, partial tiles in both directions, rows of Y at odd offsets
(n % 4 != 0) and at a misaligned pointer.

Tolerance: fp16 outputs of fp32 sums. An output carries its own rounding, 2^-11 of it, and
at most k + 2 fp32 roundings of partial sums, bounded by 2^-24 (k + 2) sum |w x|; with fp16
activations W' is taken as the dequantized matrix, so no other rounding enters."""
import numpy as np
import pytest

from helpers import random_quant

pytestmark = pytest.mark.gpu

U3, U4, C3, C4 = (3, 0), (4, 0), (3, 1), (4, 1)
FORMATS = [(*f, g) for f in (U3, U4, C3, C4) for g in (32, 64, 128)] + [(4, 2, 64)]
# Few blocks, one and more rounds of blocks, last blocks of 1 or few rows; the shapes that
# split k over a block's waves with fewer chunks than waves, as many, and numbers that leave
# some waves one chunk short.
SIZES = [(500, 128, 70), (1376, 1024, 77), (4001, 1408, 40), (1001, 1152, 17), (333, 11008, 65), (4096, 11008, 100),
         (11008, 256, 64), (4099, 128, 500), (11009, 384, 258), (11008, 256, 521), (5506, 640, 1025), (22013, 256, 1030),
         (4096, 128, 2048),
         # 17 to 64 rows in the 32 x 32 tiles of gemm.hip (fp16): an odd number of chunks, one and two tiles
         (12305, 640, 21), (12309, 1024, 50),
         # with odd chunk counts, the shapes (and the remaining forms of gemm.hip) that the ones above leave out
         (228, 1408, 2063), (234, 384, 2087), (2208, 384, 2189), (201, 384, 1261), (456, 384, 2125), (225, 2432, 2162),
         (4868, 384, 1590), (344, 9088, 2081), (7577, 384, 2061), (521, 8576, 1997)]
# int8 rows of uniform weights: the sizes at which a shape is taken instead of gemm_a8.hip
UNIFORM_A8 = [(4283, 896, 1868), (1884, 1408, 2118), (2723, 2176, 2166), (2023, 2944, 2026), (4311, 1152, 1911),
              (6086, 1920, 2002), (2888, 6784, 2089)]


def sizes(fmt, a8):
    return SIZES + (UNIFORM_A8 if a8 and fmt[1] == 0 else [])


def quant(fmt, n, k):
    bits, kind, group = fmt
    if kind < 2:
        return random_quant(n, k, bits, group, kind, seed=n + k + bits)
    rng = np.random.default_rng(n + k)
    G = k // 64
    q = random_quant(n, k, 4, 64, 1, seed=n)  # codes
    q.kind, q.codebook = 2, np.sort(rng.standard_normal((4, 16)), -1).astype(np.float16).view(np.uint16)
    q.scales = rng.uniform(2e-3, 2e-2, (n, G)).astype(np.float16).view(np.uint16)
    q.selectors = rng.integers(0, 4, (n, G), dtype=np.uint8)
    return q


def half(t, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(t).view(np.float16)).to(dev)


def levels(q, dev):
    """The exact levels in 64 bits (s (q - z), table entries, s CB[t][q])."""
    import torch
    G = q.k // q.group
    code = torch.from_numpy(q.codes).to(dev).view(q.n, G, q.group).long()
    if q.kind == 0:
        w = (code.double() - half(q.zeros, dev).double()[..., None]) * half(q.scales, dev).double()[..., None]
    elif q.kind == 1:
        w = half(q.codebook, dev).double().gather(-1, code)
    else:
        cb = half(q.codebook, dev).double()[torch.from_numpy(q.selectors).to(dev).long()]
        w = cb.gather(-1, code) * half(q.scales, dev).double()[..., None]
    return w.view(q.n, q.k)


def check(y, x, w):
    import torch
    ref, size = x @ w.t(), x.abs() @ w.abs().t()
    bound = ref.abs() * 2.0**-11 + 2.0**-24 * (1 + (x.shape[1] + 2) * size)
    assert torch.isfinite(y).all()
    bad = (y.double() - ref).abs() > bound
    assert not bad.any(), (int(bad.sum()), bad.nonzero()[:4].tolist())


@pytest.mark.parametrize("a8", [False, True], ids=["f16", "a8"])
@pytest.mark.parametrize("fmt", FORMATS, ids=lambda f: f"b{f[0]}kind{f[1]}g{f[2]}")
def test_tile_shapes(gpu, fmt, a8):
    import torch
    qx, dev = gpu, "cuda"
    for n, k, m in sizes(fmt, a8):
        print(f"tile {fmt} a8={a8} {n}x{k} m={m}", flush=True)
        q = quant(fmt, n, k)
        pw = qx.PackedWeight.from_quant(q)
        g = torch.Generator(device=dev).manual_seed(n + m)
        X = torch.randn(m, k, generator=g, device=dev).half()
        if a8:
            Xq, sx = qx.quantize_a8(X)
            check(pw.gemm_a8(Xq, sx), Xq.double() * sx.double()[:, None], levels(q, dev))
        else:
            check(pw.gemm(X), X.double(), pw.dequant().double())
        del pw


@pytest.mark.parametrize("m", [50, 500])  # k split over waves, and one round of blocks
@pytest.mark.parametrize("n", [4097, 4098, 4099, 4100])
def test_tile_output_offset(gpu, n, m):
    """Y may start at any multiple of 2 bytes, and with it every row and its stores of 8 bytes;
    what lies around it stays untouched."""
    import torch
    qx, dev, k = gpu, "cuda", 256
    pw = qx.PackedWeight.from_quant(quant((4, 0, 64), n, k))
    X = torch.randn(m, k, generator=torch.Generator(device=dev).manual_seed(1), device=dev).half()
    check(pw.gemm(X), X.double(), pw.dequant().double())
    want = pw.gemm(X)
    for at in (1, 2, 3):
        buf = torch.full((m * n + 16,), 7.0, dtype=torch.float16, device=dev)
        pw.gemm(X, buf[at:at + m * n].view(m, n))
        assert torch.equal(buf[at:at + m * n].view(m, n), want)
        assert (buf[:at] == 7).all() and (buf[at + m * n:] == 7).all()


def test_tile_one_hot_rows(gpu):
    """One-hot activations give columns of W' exactly (every k of two chunks, every format)."""
    import torch
    qx, dev, k = gpu, "cuda", 384
    for fmt in FORMATS:
        for n in (500, 11009):
            print(f"tile one-hot {fmt} n={n}", flush=True)
            pw = qx.PackedWeight.from_quant(quant(fmt, n, k))
            Y = pw.gemm(torch.eye(k, device=dev).half())
            assert torch.equal(Y, pw.dequant().t()), fmt
