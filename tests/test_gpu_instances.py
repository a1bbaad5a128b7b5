"""Every instance of the cloud projection's matrix-core kernels, with K long
enough that its counted waits run and its stages go round, against 64-bit sums
on the GPU; and a row's logits, which are the same in every one of them."""

import pytest
import torch

import paper_2607_13093_amd as sph

import kernel_rules as rules
import parity as P

pytestmark = pytest.mark.gpu

CLIP = 6.0


def _operands(M, n, K, wtype, pad, bias, seed):
    """h [M, K], weight rows of a vocabulary larger than the subset whose rows
    start `pad` bytes past the whole lines that K takes, and the subset."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    item, vocab = (2 if wtype == "bf16" else 1), n + 300
    ld = -(-K * item // 128) * 128 + pad
    h = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((vocab, ld // item), device="cuda", generator=g) * K ** -0.5
    w = w.to(torch.bfloat16 if wtype == "bf16" else torch.float8_e4m3fn)[:, :K]
    ws = torch.rand((vocab,), device="cuda", generator=g) + 0.5 if wtype == "fp8" else None
    b = torch.randn((vocab,), device="cuda", generator=g) if bias else None
    ids = torch.randperm(vocab, device="cuda", generator=g)[:n].sort().values
    return h, w, ws, b, ids


def _check(M, n, K, wtype, pad, bias, seed):
    h, w, ws, b, ids = _operands(M, n, K, wtype, pad, bias, seed)
    sub = sph.Subset(ids.to(torch.int32).cpu().numpy(), vocab=w.shape[0])
    q, s, z = sph.cloud_partial(h, w, sub, CLIP, w_row_scale=ws, bias=b, want_z=True)
    sub.close()
    hd = h.double()
    for j in range(0, n, 16384):
        sel = ids[j:j + 16384]
        wd = (w.view(torch.uint8)[sel].view(w.dtype) if wtype == "fp8" else w[sel]).float().double()
        if ws is not None:
            wd *= ws[sel].double()[:, None]
        ref, tol = hd @ wd.t(), hd.abs() @ wd.abs().t()
        if b is not None:
            ref += b[sel].double()
            tol += b[sel].double().abs()
        d = (z[:, j:j + 16384].double() - ref).abs()
        bad = d > P.tol_of(tol)
        assert not bad.any(), (int(bad.sum()), float(d.max()), bad.nonzero()[:3].tolist())
    # codes and scales of the logits written
    y = z.clamp(-CLIP, CLIP)
    sc = (y.abs().amax(1).double() / 127.0).float()
    assert torch.equal(sc, s)
    t = (y.double() / sc[:, None].double()).float().round()
    assert torch.equal(t.to(torch.int8), q)


# (rows, positions): with both weight types, every instance of the streaming kernel
# (tests/test_kernel_rules.py checks that)
STREAM = [
    (20, 15001), (18, 30001), (18, 45001), (50, 9001), (60, 30001), (64, 60001), (90, 9001), (90, 45001), (90, 60001),
    (120, 9001), (100, 30001), (128, 60001), (110, 40001), (155, 45001), (150, 64001), (129, 36001), (190, 9001),
    (175, 30001), (165, 45001), (190, 65001), (170, 40001),
    # row groups
    (300, 30001), (450, 15001), (700, 9001),
]


def stream_columns(M, n, wtype, pad):
    """Six stages more than are in flight, the last one partial (E4M3 and rows off
    the lines: one 16-byte chunk; bf16 on lines: five)."""
    bm, bn, ra, rw, lines = rules.stream_tile(M, n, wtype)
    columns = (64 if wtype == "bf16" else 128) * lines
    return columns * (max(ra, rw) + 5) + (16 if wtype == "fp8" else 8 if pad else 40)


@pytest.mark.parametrize("pad", [0, 16], ids=["lines", "off_lines"])
@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
@pytest.mark.parametrize("M,n", STREAM)
def test_streaming_instances(M, n, wtype, pad):
    assert rules.cloud_kernel(M, n, 64, wtype) == "stream"
    _check(M, n, stream_columns(M, n, wtype, pad), wtype, pad, bool(n & 8), M + n)


# (rows, positions, columns, weights, kernel): past the streaming rule.  Three
# stages of weights from six steps on (three rounds of six: the steady state), two
# from two steps on, odd and partial steps on the two-wave kernels.
TILES = [
    (1100, 6001, 6 * 64, "bf16", "w1<3>"),
    (1030, 5000, 18 * 64, "bf16", "w1<3>"),
    (512, 33025, 12 * 64, "bf16", "w1<3>"),
    (1025, 257, 24 * 64, "bf16", "w1<3>"),
    (1280, 2049, 2 * 64, "bf16", "w1<2>"),
    (1100, 6001, 4 * 64, "bf16", "w1<2>"),
    (500, 33025, 10 * 64, "bf16", "w1<2>"),
    (1025, 300, 16 * 64, "bf16", "w1<2>"),
    (1100, 6001, 64, "bf16", "dma256"),
    (1030, 5000, 7 * 64, "bf16", "dma256"),
    (512, 33025, 15 * 64, "bf16", "dma256"),
    (1100, 6001, 9 * 64 + 8, "bf16", "dma256"),
    (1590, 3001, 12 * 64, "bf16", "dma320"),
    (300, 33025, 7 * 64, "bf16", "dma320"),
    (640, 33025, 3 * 64 + 56, "bf16", "dma320"),
    (1100, 6001, 64, "fp8", "dma8_256"),
    (1030, 5000, 7 * 64, "fp8", "dma8_256"),
    (512, 33025, 8 * 64 + 16, "fp8", "dma8_256"),
    (300, 33025, 6 * 64, "fp8", "dma8_320"),
    (1590, 3001, 9 * 64 + 48, "fp8", "dma8_320"),
]


@pytest.mark.parametrize("bias", [False, True], ids=["", "bias"])
@pytest.mark.parametrize("M,n,K,wtype,kernel", TILES, ids=[f"M{m}n{n}K{k}-{x}" for m, n, k, w, x in TILES])
def test_tiled_instances(M, n, K, wtype, kernel, bias):
    assert rules.cloud_kernel(M, n, K, wtype) == kernel
    _check(M, n, K, wtype, 0, bias, M + n + K)


# (columns, weights, [(rows, positions, kernel)])
SAME = [
    (12 * 64, "bf16", [(20, 33025, "stream"), (160, 33025, "stream"), (1100, 4001, "w1<3>"), (512, 33025, "w1<3>"),
                       (300, 33025, "dma320"), (256, 20000, "stream")]),
    (4 * 64, "bf16", [(20, 4001, "stream"), (1100, 4001, "w1<2>"), (1590, 4001, "dma320")]),
    (5 * 64, "bf16", [(20, 4001, "stream"), (1100, 4001, "dma256"), (1590, 4001, "dma320")]),
    (5 * 64 + 24, "bf16", [(60, 4001, "stream"), (1100, 4001, "dma256"), (1590, 4001, "dma320")]),
    (5 * 64 + 16, "fp8", [(20, 4001, "stream"), (100, 33025, "stream"), (1100, 4001, "dma8_256"),
                          (300, 33025, "dma8_320")]),
]


@pytest.mark.parametrize("K,wtype,shapes", SAME, ids=[f"K{k}-{w}" for k, w, x in SAME])
def test_rows_have_the_same_logits_in_every_kernel(K, wtype, shapes):
    """The first 20 rows of every batch, over the positions that all have, bit for
    bit (blocks of positions and row tiles start elsewhere in each)."""
    n0 = min(n for _, n, _ in shapes)
    h, w, ws, b, ids = _operands(max(m for m, _, _ in shapes), max(n for _, n, _ in shapes), K, wtype, 0, True, K)
    first = None
    for M, n, kernel in shapes:
        assert rules.cloud_kernel(M, n, K, wtype) == kernel
        sub = sph.Subset(ids[:n].to(torch.int32).cpu().numpy(), vocab=w.shape[0])
        _, _, z = sph.cloud_partial(h[:M], w, sub, CLIP, w_row_scale=ws, bias=b, want_z=True)
        sub.close()
        z = z[:20, :n0].contiguous()
        first = z if first is None else first
        assert torch.equal(z.view(torch.int32), first.view(torch.int32)), (M, n, kernel)
