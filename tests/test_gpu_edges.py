"""GPU parity at the edges of the MFMA kernels' tiles and K steps: partial K
steps (any multiple of 8 columns), row tiles with one or all rows in use,
subsets that end one position into a tile, and payload rows at every
alignment, through the staged checks of tests/parity.py against the oracle.
"""

import numpy as np
import pytest
import torch

import paper_2607_13093_amd as sph
from oracle import gcm as ogcm
from synth import Config, make_workload

import kernel_rules as rules
from test_gpu_payload import run_format_case

pytestmark = pytest.mark.gpu

ENDPOINT = [
    # (sessions, R, d_end, n): the small tiles of the endpoint projection
    (3, 3, 8, 257),      # 9 rows, one 8-column step, a tile of one position
    (4, 8, 48, 1535),    # 32 rows, one partial step
    (11, 3, 72, 519),    # 33 rows, a whole and an 8-column step
    (32, 4, 120, 1009),  # 128 rows
    (43, 3, 96, 770),    # 129 rows
    (64, 4, 56, 513),    # 256 rows
    (53, 6, 184, 1031),  # 318 rows
    # the large ones (many positions; long K up to 192 rows)
    (31, 5, 264, 33057),  # 155 rows of the 256-row tile
    (64, 4, 56, 33025),   # 256 rows, a tile of one position
    (80, 4, 72, 33000),   # 320 rows
    (2, 5, 8, 262145),    # few rows, more positions than the small tiles have slots for
]


@pytest.mark.parametrize("fmt", [(8, 0), (4, 0), (8, 256)], ids=["b8", "b4", "b8blk256"])
@pytest.mark.parametrize("shape", ENDPOINT, ids=[f"S{s}R{r}de{e}n{n}" for s, r, e, n in ENDPOINT])
def test_endpoint_partial_steps_and_unaligned_rows(shape, fmt):
    S, R, de, n = shape
    cfg = Config("edge", 400 + sum(shape) + fmt[0], d=de + 128, d_end=de, vocab=n + 300, n_sub=n,
                 subset_kind="choice", sessions=S, rows_per_session=R)
    sessions = None if S * R * n < 2_000_000 else [0, S - 1]
    run_format_case(make_workload(cfg), fmt[0], fmt[1], f"endpoint edge {shape} {fmt}", sessions=sessions)


# (sessions, R, d_cloud, n): the row tiles of the streaming cloud projection at
# the edges of their rows, widths (32 ... 256 positions per block) and K steps
# (one chunk, partial steps; tests/test_gpu_instances.py has every instance with
# long K), weight rows that start at every 16-byte place of a line
STREAM = [
    (3, 3, 8, 33),        # 9 rows, one chunk
    (4, 8, 136, 8193),    # 32 rows, 33 positions per block, the last one
    (11, 3, 200, 16500),  # 33 rows, 65 per block
    (16, 4, 264, 33000),  # 64 rows, 129 per block
    (13, 5, 328, 40001),  # 65 rows, 157 per block
    (12, 8, 72, 65536),   # 96 rows, 256 per block
    (97, 1, 520, 1),      # 97 rows, one position
    (16, 8, 448, 61441),  # 128 rows, 241 per block
    (43, 3, 312, 61440),  # 129 rows, 240 per block
    (32, 5, 960, 65537),  # 160 rows, two rounds
    (23, 7, 152, 45001),  # 161 rows
    (24, 8, 64, 300),     # 192 rows, one whole step
    (19, 5, 264, 24000),  # 95 rows, 94 positions per block
    (23, 4, 200, 9001),   # 92 rows, 36
    (31, 5, 136, 31000),  # 155 rows, 122
    (35, 5, 328, 14000),  # 175 rows, 55
    (5, 3, 136, 4001),    # 15 rows, two lines a stage: the last one's second half empty
    (31, 4, 1160, 9000),  # 124 rows, several rounds of its three stages
    (12, 5, 904, 30001),  # 60 rows, 118 positions per block
]


@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", STREAM, ids=[f"S{s}R{r}dc{c}n{n}" for s, r, c, n in STREAM])
def test_streaming_cloud_projection(shape, wtype):
    S, R, dc, n = shape
    if wtype == "fp8":
        dc = -(-dc // 16) * 16
    cfg = Config("stream", 500 + sum(shape) % 1000, d=dc + 8, d_end=8, vocab=n + 77, n_sub=n,
                 subset_kind="choice", sessions=S, rows_per_session=R, wtype=wtype,
                 with_bias=S % 2 == 0)
    # one session of a large case stands for its row tile's first and last rows
    sessions = None if S * R * n < 1_000_000 else [0, S - 1]
    run_format_case(make_workload(cfg), 8, 0, f"stream {shape} {wtype}", sessions=sessions)


# (sessions, R, n, tau, top_p): rows whose passes are spread over several
# blocks, at the edges of the rule, with every mass below the cut, with one
# part listing too much (tau large) and with a nucleus of a few ids
LONG_ROWS = [
    (1, 5, 32768, 0.7, 0.9),
    (1, 1, 40001, 0.7, 1.0),
    (2, 3, 70003, 3.0, 0.95),
    (1, 2, 33027, 0.25, 0.5),
    (64, 1, 32769, 0.9, 0.8),
    (32, 4, 65537, 0.6, 0.9),
]


@pytest.mark.parametrize("shape", LONG_ROWS, ids=[f"S{s}R{r}n{n}t{t}p{p}" for s, r, n, t, p in LONG_ROWS])
def test_sampling_few_long_rows(shape):
    import numpy as np
    import torch

    from paper_2607_13093_amd import api as sph
    from test_gpu_sampling import run_sample_case

    S, R, n, tau, top_p = shape
    cfg = Config("long_rows", 700 + S + R, d=192, d_end=64, vocab=n + 50, n_sub=n, subset_kind="choice",
                 sessions=S, rows_per_session=R, mode="sample", temperature=tau, top_p=top_p,
                 philox_seed=0xABCDEF12345 + n)
    if S * R <= 8:
        run_sample_case(make_workload(cfg), tag=f"long rows {shape}")
    # the same tokens from a workspace without the optional scratch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    M = S * R
    q = (torch.randn((M, n), generator=g, device="cuda") * 30).round().clamp(-127, 127).to(torch.int8)
    sc = torch.rand((M,), generator=g, device="cuda") * 0.05 + 0.01
    ids = np.sort(np.random.default_rng(n).choice(n + 50, n, replace=False)).astype(np.int32)
    sub = sph.Subset(ids, vocab=n + 50)
    drafts = torch.zeros((S, R - 1), dtype=torch.int32, device="cuda") if R > 1 else None
    full = sph.fuse_verify_workspace(M, sub, sph.SAMPLE)
    base = (M * 16384 + 255) // 256 * 256 + (M * n * 4 + 255) // 256 * 256
    assert full > base
    got = []
    for size in (full, base):
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        tok, acc, _ = sph.fuse_verify(q, sc, None, None, sub, S, R, drafts, mode=sph.SAMPLE,
                                      temperature=tau, top_p=top_p, seed=n, workspace=ws)
        torch.cuda.synchronize()
        got.append((tok.cpu().numpy(), acc.cpu().numpy()))
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    with pytest.raises(sph.SphError):
        sph.fuse_verify(q, sc, None, None, sub, S, R, drafts, mode=sph.SAMPLE, temperature=tau,
                        top_p=top_p, seed=n,
                        workspace=torch.empty((base - 256,), dtype=torch.uint8, device="cuda"))
    sub.close()


def _rows(M, n, kind, seed):
    """Fused logits of M rows at tau 1: normal ones of deviation s, for "top" with
    one id besides that has share p of the mass, for "zipf" 200 ids that have it
    (through the payload: 8-bit codes of their logits), for "crowd" with all ids
    but the first 4096 far below."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape, s, p = kind
    h = torch.randn((M, 64), device="cuda", generator=g)
    h = (h * (8.0 / h.norm(dim=1, keepdim=True))).to(torch.bfloat16)
    w = (torch.randn((n, 64), device="cuda", generator=g) * (s / 8.0)).to(torch.bfloat16)
    q = torch.zeros((M, n), dtype=torch.int8, device="cuda")
    scale = torch.ones((M,), device="cuda")
    if shape == "crowd":
        q[:, 4096:] = -127
        scale[:] = 0.4
    elif shape != "normal":
        ids = torch.stack([torch.randperm(n, device="cuda", generator=g)[:1 if shape == "top" else 200] for _ in range(M)])
        lw = -1.1 * torch.log(torch.arange(1, ids.shape[1] + 1, device="cuda").double())
        lw += np.log(n) + s * s / 2 + np.log(p / (1 - p)) - torch.logsumexp(lw, 0)
        scale[:] = float(lw.max()) / 127.0
        q.scatter_(1, ids, (lw * (127.0 / lw.max())).round().clamp(0, 127).to(torch.int8).expand(M, -1).contiguous())
    return q, scale, h, w


# (kind, top_p): a few ids hold much of the mass and the cut lies just past them
# (in a thin tail or a crowded one), between them, or where ids are far apart;
# and a window whose ids all lie in one block's part, which cannot list them
PEAKED = [(("top", 1.0, 0.8), 0.8), (("top", 0.3, 0.5), 0.5), (("top", 1.0, 0.8), 0.9), (("top", 2.0, 0.8), 0.8),
          (("zipf", 1.5, 0.7), 0.8), (("normal", 4.0, 0), 0.9), (("normal", 6.0, 0), 0.95),
          (("crowd", 0.05, 0), 0.7)]


@pytest.mark.parametrize("split", [True, False], ids=["split", "one_block"])
@pytest.mark.parametrize("kind,top_p", PEAKED, ids=[f"{k[0]}s{k[1]}m{k[2]}-p{p}" for k, p in PEAKED])
def test_sampling_peaked_rows(kind, top_p, split):
    """Rows with a few large weights sample what the oracle does, in one exact pass
    like flat ones: a second one over 65536 positions takes longer than half of the
    whole launch."""
    import oracle
    from test_gpu_sampling import _exempt

    M, n, seed = 48, 65536, 11
    sub = sph.Subset(vocab=n, full=True)
    full = sph.fuse_verify_workspace(M, sub, sph.SAMPLE)
    base = M * 16384 + M * n * 4
    assert full > base and base % 256 == 0
    ws = torch.empty((full if split else base,), dtype=torch.uint8, device="cuda")
    best, out = [], None
    for k, p in ((("normal", 1.5, 0), 0.9), (kind, top_p)):
        q, s, h, w = _rows(M, n, k, seed)
        sph.trace_start(400)
        for _ in range(20):
            out = sph.fuse_verify(q, s, h, w, sub, M, 1, None, mode=sph.SAMPLE, temperature=1.0, top_p=p, seed=seed,
                                  want_fused=True, workspace=ws)
        torch.cuda.synchronize()
        best.append(min(ms for name, ms in sph.trace_collect(400) if name == "fuse_sample"))
    tok, _, f = out
    rows = [0, 1, M // 2, M - 1]
    ref, info = oracle.sample_select(f[rows].cpu().numpy(), np.arange(n, dtype=np.int32), 1.0, np.float32(top_p), seed, 1,
                                     row_index=np.asarray(rows))
    bad = (tok[rows].cpu().numpy() != ref) & ~_exempt(info)
    assert not bad.any(), (tok[rows], ref)
    print(f"sampler: flat {best[0] * 1e3:.1f} us, {kind} {best[1] * 1e3:.1f} us", flush=True)
    if kind[0] != "crowd":
        assert best[1] < 1.3 * best[0], best
    sub.close()


BUCKET = np.float32(24.0 / 4096)


def _off_middle(d, p, per, mass, before, n=65536):
    """Logits (largest 0, tau 1) whose bucket counts mislead: a head of large weights,
    `per` logits in each of 60 buckets around the cut of top_p = p, each of `mass` of
    the total, and a tail; those in front of the cut lie at the start (d < 0) or the
    end of their buckets, those behind it at the other."""
    s, rng = float(BUCKET), np.random.default_rng(per)
    front, back = (0.02, 0.97) if d < 0 else (0.97, 0.02)
    head = np.r_[0.0, 3 + np.arange(20) * 2 + front]
    q0 = int(-np.log(mass * np.exp(-head * s).sum() / p) / s)
    i = np.arange(60)
    cut = np.repeat(q0 + i + np.where(i < 60 * before, front, back), per)
    w, k = np.exp(-cut * s), int(60 * before) * per
    nt = n - len(head) - len(cut)
    tail = (np.exp(-head * s).sum() + w[:k].sum()) * (1 - p) / p - w[k:].sum()
    q1 = np.floor(-np.log(tail / nt) / s) + np.arange(nt) % 7 - 3 + back
    return -(rng.permutation(np.r_[head, cut, q1]) * s).astype(np.float32)


def _windows(f, p):
    """The sampler's window of one row and what becomes of it: a replay of its rules
    in 64 bits."""
    n, last = f.size, 4095
    b = np.minimum((f.max() - f) * np.float32(4096.0 / 24.0), np.float32(last)).astype(int)
    count = np.bincount(b, minlength=4096)
    k = count.astype(float)
    k[last] = 0
    w = np.exp(-float(BUCKET) * (np.arange(4096) + 0.5))
    m = k * w
    m[0] += 1 - w[0]
    A, C = np.cumsum(m), np.r_[0, np.cumsum(k)]
    err = 2.96e-3 * ((1 - p) * np.maximum(A - 1, 0) + p * (A[-1] - A)) + p * n * 3.9e-11

    def first(x):
        h = np.nonzero(A + x * err >= p * A[-1])[0]
        return int(h[0]) if len(h) else 4096

    for share, most in ((1.0, 64), (0.25, 1024), (0.0625, 1024), (0.0, n)):
        lo, hi = min(first(share), last), first(-share)
        if share == 0.0:
            hi = lo
        if (C[hi + 1] if hi <= last else n) - C[lo] <= most:
            hi = min(hi, last)
            break
    e = np.cumsum(np.bincount(b, weights=np.exp(f.astype(float) - f.max()), minlength=4096))
    cut = int(np.nonzero(e >= p * e[-1])[0][0])
    path = []
    while True:
        below, over = lo > 0 and e[lo - 1] >= p * e[-1], count[lo:hi + 1].sum() > 1024
        if lo <= cut <= hi and not over:
            return path
        if len(path) < 3 and below:
            lo, hi = max(0, lo - 2), lo - 1
            path.append("down")
        elif len(path) < 3 and over and hi > lo:
            hi -= 1
            path.append("shrink")
        elif len(path) < 3 and not over and hi < last:
            lo, hi = hi + 1, min(hi + 2, last)
            path.append("up")
        else:
            return path + ["group"]


# (direction, top_p, logits a bucket, weight of one, share of the 60 buckets in front
# of the cut) and the moves of the window
MISSED = [
    ((-1, 0.9, 100, 5e-6, 0.3), ["down"]),
    ((1, 0.9, 100, 5e-6, 0.3), ["up"]),
    ((1, 0.9, 520, 2e-6, 0.2), ["up", "shrink"]),
    ((-1, 0.9, 520, 2e-6, 0.2), ["down", "shrink", "up", "group"]),
    ((-1, 0.5, 1, 2e-5, 0.3), ["down", "down", "down", "group"]),
    ((1, 0.5, 1, 2e-5, 0.3), ["up", "up", "up", "group"]),
    ((-1, 0.5, 350, 4e-7, 0.2), ["group"]),
]


@pytest.mark.parametrize("split", [True, False], ids=["split", "one_block"])
@pytest.mark.parametrize("row,path", MISSED, ids=["-".join(p) for _, p in MISSED])
def test_sampling_rows_whose_window_misses(row, path, split):
    """A window that misses the cut, or whose neighbours overflow the list, moves until
    it is found; rows of the same logits sample with other random numbers."""
    import oracle
    from test_gpu_sampling import _exempt

    M, n, p = 128, 65536, row[1]
    f0 = _off_middle(*row)
    assert _windows(f0, p) == path
    # the logits as three bf16 numbers each: every sum of them is exact
    rest, parts = torch.from_numpy(f0).cuda(), []
    for _ in range(3):
        parts.append(rest.to(torch.bfloat16))
        rest = rest - parts[-1].float()
    w = torch.zeros((n, 8), device="cuda", dtype=torch.bfloat16)
    w[:, :3] = torch.stack(parts, 1)
    h = torch.ones((M, 8), device="cuda", dtype=torch.bfloat16)
    sub = sph.Subset(vocab=n, full=True)
    full, base = sph.fuse_verify_workspace(M, sub, sph.SAMPLE), M * 16384 + M * n * 4
    assert full > base and base % 256 == 0
    ws = torch.empty((full if split else base,), dtype=torch.uint8, device="cuda")
    q, s = torch.zeros((M, n), dtype=torch.int8, device="cuda"), torch.ones((M,), device="cuda")
    tok, _, f = sph.fuse_verify(q, s, h, w, sub, M, 1, None, mode=sph.SAMPLE, temperature=1.0, top_p=p, seed=5,
                                want_fused=True, workspace=ws)
    assert torch.equal(f, torch.from_numpy(f0).cuda().expand(M, -1))
    ref, info = oracle.sample_select(np.broadcast_to(f0, (M, n)), np.arange(n, dtype=np.int32), 1.0, np.float32(p), 5, 1,
                                     row_index=np.arange(M))
    bad = (tok.cpu().numpy() != ref) & ~_exempt(info)
    assert not bad.any(), (tok, ref)
    assert (~_exempt(info)).sum() > M // 2  # (a tenth of them logits near the cut)
    sub.close()


# (sessions, R, d_cloud, n): partial K steps and ragged edges, first of the row
# groups of the streaming kernel (193 to 1024 rows over few positions), then of
# the 256- and 320-row tiles
TILES = [
    (193, 1, 8, 300),      # groups of 97 and 96 rows, 32 positions per block
    (64, 4, 72, 513),      # two groups of 128
    (52, 5, 200, 255),     # 260 rows, fewer shares than one XCD group
    (64, 5, 312, 1025),
    (57, 9, 456, 770),     # 513 rows: four groups
    (37, 7, 1000, 256),    # 259 rows
    (97, 4, 136, 16384),   # 388 rows: four groups, 256 positions per block
    (205, 1, 88, 32768),   # 205 rows: two groups, the last positions of the rule
    (1021, 1, 264, 333),   # eight groups, the last one short
    (257, 4, 8, 300),      # 1028 rows: 256-row tiles, one chunk
    (320, 4, 72, 513),     # 1280 rows, every row of the tiles
    (260, 6, 200, 255),    # 1560 rows: 320-row tiles
    (400, 4, 312, 1025),   # 1600 rows, one position past the tiles
    (391, 4, 456, 770),    # 1564 rows: 320-row tiles
    (257, 5, 1000, 256),   # 1285 rows, one whole tile of positions
    (257, 4, 256, 300),    # two whole steps at a time
    (258, 4, 384, 513),    # six
]


@pytest.mark.parametrize("fmt", [(8, 0), (4, 256)], ids=["b8", "b4blk256"])
@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", TILES, ids=[f"S{s}R{r}dc{c}n{n}" for s, r, c, n in TILES])
def test_tiled_cloud_projection_partial_steps(shape, wtype, fmt):
    S, R, dc, n = shape
    if wtype == "fp8":
        dc = -(-dc // 16) * 16
    cfg = Config("tiles", 800 + sum(shape) % 1000, d=dc + 8, d_end=8, vocab=n + 33, n_sub=n,
                 subset_kind="choice", sessions=S, rows_per_session=R, wtype=wtype,
                 with_bias=S % 2 == 1)
    sessions = None if S * R * n < 2_000_000 else [0, S // 2, S - 1]
    run_format_case(make_workload(cfg), fmt[0], fmt[1], f"tiles {shape} {wtype} {fmt}", sessions=sessions)


@pytest.mark.parametrize("wtype,d_cloud", [("bf16", 72), ("fp8", 2064)])
def test_block_quantising_epilogue_with_a_partial_step(wtype, d_cloud):
    """1028 rows x 52736 positions: enough tiles (five row tiles by 206) for the
    quantising epilogue in spite of the partial K step."""
    cfg = Config("tiles_q", 870, d=d_cloud + 8, d_end=8, vocab=53000, n_sub=52736, subset_kind="choice",
                 sessions=257, rows_per_session=4, wtype=wtype, with_bias=True)
    run_format_case(make_workload(cfg), 4, 256, f"quantising tiles {wtype}", sessions=[0, 128, 256])


@pytest.mark.parametrize("bits", [8, 4])
def test_codes_of_the_quantising_epilogue_are_those_of_its_logits(bits):
    """E4M3 weights with a bias: every code is the one that the written logit rounds
    to, among enough logits (66 million) that computing them twice in two roundings
    shows."""
    M, n, K = 1100, 60000, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    h = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((n, K), device="cuda", generator=g).to(torch.float8_e4m3fn)
    ws = torch.rand((n,), device="cuda", generator=g) * 0.3 + 0.1
    bias = torch.randn((n,), device="cuda", generator=g)
    sub = sph.Subset(vocab=n, full=True)
    sph.trace_start(10)
    q, s, z = sph.cloud_partial(h, w, sub, 6.0, w_row_scale=ws, bias=bias, want_z=True, bits=bits, block=256)
    torch.cuda.synchronize()
    assert [k for k, _ in sph.trace_collect(10)] == ["cloud_mfma"]  # no quantiser of its own
    if bits == 4:
        q = torch.stack((q & 15, q >> 4), 2).view(M, n).to(torch.int8)
        q = torch.where(q >= 8, q - 16, q)
    qmax = 127.0 if bits == 8 else 7.0
    for r in range(0, M, 100):
        y = z[r:r + 100].clamp(-6.0, 6.0)
        a = torch.nn.functional.pad(y.abs(), (0, -n % 256)).view(len(y), -1, 256).amax(2)
        # fp32 quotients, correctly rounded (exact enough in 64 bits before the rounding)
        sc = (a.double() / qmax).float()
        assert torch.equal(sc, s[r:r + 100])
        t = (y.double() / sc.repeat_interleave(256, 1)[:, :n].double()).float().round()
        assert torch.equal(t.to(torch.int8), q[r:r + 100]), int((t != q[r:r + 100]).sum())
    sub.close()


@pytest.mark.parametrize("bits,block", [(8, 0), (4, 0), (8, 256), (4, 1024)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8, 255, 1022, 4093, 4094, 4095, 4096, 4097, 4098, 4099, 8193, 12287])
def test_quantiser_at_the_ends_of_rows(n, bits, block):
    """Rows whose last four columns straddle a chunk of the quantiser or are fewer,
    from partial logits n apart (any alignment) and whole lines apart: the codes
    and scales are those of the logits."""
    M, K = 5, 64
    g = torch.Generator(device="cuda").manual_seed(n)
    h = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((n, K), device="cuda", generator=g).to(torch.bfloat16)
    sub = sph.Subset(vocab=n, full=True)
    q, s, z = sph.cloud_partial(h, w, sub, 12.0, want_z=True, bits=bits, block=block)
    q2, s2, _ = sph.cloud_partial(h, w, sub, 12.0, bits=bits, block=block)
    sub.close()
    qmax = 127.0 if bits == 8 else 7.0
    y, wide = z.clamp(-12.0, 12.0), block or n
    a = torch.nn.functional.pad(y.abs(), (0, -n % wide)).view(M, -1, wide).amax(2)
    sc = (a.double() / qmax).float()
    code = (y.double() / sc.repeat_interleave(wide, 1)[:, :n].double()).float().round().to(torch.int8)
    if bits == 4:
        code = torch.nn.functional.pad(code, (0, n & 1)).to(torch.uint8) & 15
        code = code[:, 0::2] | (code[:, 1::2] << 4)
    assert torch.equal(sc.view(s.shape), s) and torch.equal(code, q)
    assert torch.equal(s, s2) and torch.equal(q, q2)


def test_a_partial_chunk_costs_what_its_columns_do():
    """Rows of 1500 columns take the quantiser 0.52 to 0.55 of the time of 4096 (with
    loads in branches for the ends of rows 0.62 to 0.64)."""
    ratio = []
    for _ in range(3):
        us = []
        for n in (1500, 4096):
            us.append(_cloud_us(2048, n, 64, 0, "cloud_quantize")[0])
        ratio.append(us[0] / us[1])
    print(f"1500 columns against 4096: {ratio}", flush=True)
    assert min(ratio) < 0.6


def _cloud_us(M, n, K, block, only=None):
    g = torch.Generator(device="cuda").manual_seed(K)
    h = torch.randn((M, K), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((n, K), device="cuda", generator=g).to(torch.bfloat16)
    sub = sph.Subset(vocab=n, full=True)
    sph.trace_start(400)
    for _ in range(60):
        sph.cloud_partial(h, w, sub, 30.0, block=block)
    torch.cuda.synchronize()
    t = sph.trace_collect(400)
    sub.close()
    names = sorted({k for k, _ in t if k == (only or k)})
    return sum(min(ms for k, ms in t if k == name) for name in names) * 1e3, names


def test_few_tiles_with_a_partial_step_quantise_apart():
    """32 tiles of a 208-column projection: blocks of 256 positions cost what blocks
    of 1024 do (both by the separate quantiser), as the epilogue would keep a CU per
    tile for longer than all the rest takes."""
    t1024, n1 = _cloud_us(1964, 863, 208, 1024)
    t256, n2 = _cloud_us(1964, 863, 208, 256)
    print(f"blocks of 1024 {t1024:.1f} us, of 256 {t256:.1f} us", flush=True)
    assert n1 == n2 == ["cloud_mfma", "cloud_quantize"]
    assert t256 < 1.5 * t1024


# (key bytes, rows, segment bytes, aad bytes): batches whose lanes take one block
# each (the last piece of a row one block, three, a few), short rows in large
# numbers, blocks over two and three segments, and sums whose workgroup has no
# thread left for the other terms
SEALED = [
    (32, 520, (5, 2, 3), 7),       # 520 rows of one block over three segments
    (16, 520, (0,), 33),           # no data
    (32, 667, (37,), 1024),        # rows of 65 other terms, over one wave and the next
    (16, 700, (4, 30), 1000),      # 64, the last one short
    (32, 130, (16381, 4), 20),     # 1025 blocks a row
    (16, 33, (65535, 9), 0),       # 4097
    (16, 41, (30007, 20008), 16),  # a boundary inside a block, a ragged end
    (32, 24, (49153, 4), 1024),    # 768 threads, the largest AAD beside one block
    (16, 9, (8128, 16), 23),       # 509 blocks, 3 other terms: one workgroup of 512 threads
    (32, 9, (8144, 16), 23),       # one term more: two workgroups and a sum of sums
    (16, 40, (49136,), 1024),      # 1024 threads, 1023 blocks in the last sum: a second pass
]


# the same and the blocks that a lane chains: a last piece with a shorter chain and
# a first round that is partly empty, pieces that are all whole, and segments that
# meet inside a chained piece
CHAINED = [
    (32, 60, (200000,), 0, 2),          # last piece 84 blocks, two rounds
    (16, 64, (123457,), 13, 2),
    (16, 64, (131072, 118928), 7, 3),   # boundary on a block, last piece 73 of 192
    (32, 320, (60000, 4), 32, 4),       # 167 of 256: three rounds, the first 39 blocks
    (16, 1024, (16384,), 0, 4),         # whole pieces only
    (32, 128, (150001, 49999), 64, 6),  # a boundary inside a block of a chained piece
    (16, 256, (131, 260869), 1000, 10),
]


@pytest.mark.parametrize("case", CHAINED, ids=[f"k{k}r{r}L{'_'.join(map(str, b))}a{a}c{c}" for k, r, b, a, c in CHAINED])
def test_sealed_batches_with_chains(case):
    assert rules.gcm_chain(case[1], sum(case[2]), case[3]) == case[4]
    _sealed(*case[:4])


@pytest.mark.parametrize("case", SEALED, ids=[f"k{k}r{r}L{'_'.join(map(str, b))}a{a}" for k, r, b, a in SEALED])
def test_sealed_batches(case):
    assert rules.gcm_chain(case[1], sum(case[2]), case[3]) <= 1
    _sealed(*case)


def _sealed(klen, rows, seg, la):
    """A batch's rows equal the same rows sealed one at a time (and the oracle),
    and open; a changed byte fails its row alone."""
    rng = np.random.default_rng(rows + sum(seg) + la)
    key = sph.GcmKey(k := rng.bytes(klen))
    x = [rng.integers(0, 256, (rows, b), dtype=np.uint8) for b in seg]
    iv = rng.integers(0, 256, (rows, 12), dtype=np.uint8)
    aad = rng.integers(0, 256, (rows, la), dtype=np.uint8)
    dx, div = [torch.from_numpy(a).cuda() for a in x], torch.from_numpy(iv).cuda()
    daad = torch.from_numpy(aad).cuda() if la else None
    ct, tag = sph.gcm_seal_segments(key, dx, div, daad)
    for r in sorted({0, 1, rows // 2, rows - 1}):
        one, t1 = sph.gcm_seal_segments(key, [a[r:r + 1] for a in dx], div[r:r + 1], daad[r:r + 1] if la else None)
        assert torch.equal(t1, tag[r:r + 1]), r
        for a, b in zip(one, ct):
            assert torch.equal(a, b[r:r + 1]), r
    ref, tref = ogcm.seal_rows(k, np.concatenate([a[-1:] for a in x], 1), iv[-1:], aad[-1:])
    np.testing.assert_array_equal(torch.cat(list(ct), 1)[-1:].cpu().numpy(), ref)
    np.testing.assert_array_equal(tag[-1:].cpu().numpy(), tref)
    bad = rows // 3
    tag[bad, 5] ^= 1
    pt, ok = sph.gcm_open_segments(key, ct, div, tag, daad)
    for a, b in zip(pt, dx):
        assert torch.equal(a, b)
    want = torch.ones_like(ok)
    want[bad] = 0
    assert torch.equal(ok, want)


def test_sealing_with_associated_data_costs_what_it_hashes():
    """1 KB of AAD to every row of a batch is as many blocks more as 1 KB of data
    without its encryption: not more time than that (the terms of a row are summed
    before they meet in memory)."""
    rows = 1500
    key = sph.GcmKey(bytes(range(32)))
    g = torch.Generator(device="cuda").manual_seed(5)
    iv = torch.randint(0, 256, (rows, 12), dtype=torch.uint8, device="cuda", generator=g)
    best = []
    for data, la in ((37 + 1024, 0), (37, 1024)):
        x = torch.randint(0, 256, (rows, data), dtype=torch.uint8, device="cuda", generator=g)
        aad = torch.randint(0, 256, (rows, la), dtype=torch.uint8, device="cuda", generator=g) if la else None
        sph.trace_start(400)
        for _ in range(20):
            sph.gcm_seal_segments(key, (x,), iv, aad)
        torch.cuda.synchronize()
        best.append(min(ms for name, ms in sph.trace_collect(400)))
    print(f"sealed: data {best[0] * 1e3:.1f} us, AAD {best[1] * 1e3:.1f} us", flush=True)
    assert best[1] < 1.3 * best[0], best


@pytest.mark.parametrize("M,n", [(37, 1001), (300, 33025), (1030, 259)], ids=["stream", "tiles320", "tiles256"])
def test_payload_with_and_without_padded_rows(M, n):
    """The partial logits' row stride (whole lines in a workspace of the queried
    size, n in the smallest one accepted or in z_out) changes no payload bit."""
    g = torch.Generator(device="cuda").manual_seed(M)
    h = torch.randn((M, 72), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((n, 72), device="cuda", generator=g).to(torch.bfloat16)
    sub = sph.Subset(vocab=n, full=True)
    full = sph.cloud_partial_workspace(M, sub)
    least = (M * n * 4 + 255) // 256 * 256 + (M * 8192 + 255) // 256 * 256
    assert least < full
    got = [sph.cloud_partial(h, w, sub, 8.0, workspace=torch.full((size,), 0x7F, dtype=torch.uint8, device="cuda"),
                             want_z=want)
           for size, want in ((full, False), (least, False), (full, True))]
    for q, s, _ in got[1:]:
        assert torch.equal(q, got[0][0]) and torch.equal(s, got[0][1])
    assert torch.equal(got[2][2].abs().clamp(max=8.0).amax(1) / 127.0, got[2][1])
    with pytest.raises(sph.SphError):
        sph.cloud_partial(h, w, sub, 8.0, workspace=torch.empty((least - 256,), dtype=torch.uint8, device="cuda"),
                          want_z=False)
    sub.close()


# (rows, d_cloud, d_end, n): rows of h that fill the skinny kernels' LDS in one
# launch (8 x 8704 columns), just exceed it (two launches) and need four
SKINNY = [(8, 8704, 64, 301), (8, 8720, 64, 301), (7, 9952, 8712, 77), (8, 30720, 24, 70)]


@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", SKINNY, ids=[f"M{m}dc{c}de{e}n{n}" for m, c, e, n in SKINNY])
def test_skinny_rows_at_the_lds_limit(shape, wtype):
    M, dc, de, n = shape
    cfg = Config("skinny", 900 + dc % 100, d=dc + de, d_end=de, vocab=n + 9, n_sub=n, subset_kind="choice",
                 sessions=1, rows_per_session=M, wtype=wtype, with_bias=True)
    run_format_case(make_workload(cfg), 8, 0, f"skinny {shape} {wtype}")


def test_skinny_row_longer_than_its_lds_is_refused():
    h = torch.zeros((1, 30728), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((4, 30728), dtype=torch.bfloat16, device="cuda")
    sub = sph.Subset(vocab=4, full=True)
    with pytest.raises(sph.SphError, match="too large"):
        sph.cloud_partial(h, w, sub, 8.0)
    sub.close()


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M", [1, 3, 8])
def test_few_rows_without_endpoint_columns(M, bits):
    """d_end = 0 on the skinny kernel: the fused logits are the dequantised payload,
    the token its largest."""
    n = 1571
    g = torch.Generator(device="cuda").manual_seed(M)
    sub = sph.Subset(vocab=n, full=True)
    scale = torch.rand((M,), device="cuda", generator=g) * 0.05 + 0.01
    top = 127 if bits == 8 else 7
    codes = torch.randint(-top, top, (M, n), device="cuda", generator=g)
    best = torch.arange(M, device="cuda") * 97 + 5
    codes[torch.arange(M, device="cuda"), best] = top
    if bits == 8:
        q = codes.to(torch.int8)
    else:
        c = torch.nn.functional.pad(codes, (0, 1)).to(torch.uint8) & 15
        q = c[:, 0::2] | (c[:, 1::2] << 4)
    tok, acc, f = sph.fuse_verify(q, scale, None, None, sub, 1, M, best[:M - 1].to(torch.int32)[None] if M > 1 else None,
                                  want_fused=True, bits=bits)
    assert torch.equal(f, codes.float() * scale[:, None])
    assert torch.equal(tok, best.to(torch.int32)) and int(acc) == M - 1
    sub.close()


@pytest.mark.parametrize("n", [300, 4096, 70001])
@pytest.mark.parametrize("R", [1, 2, 4, 5, 8, 9, 16, 17, 40])
def test_final_selection_at_its_rows_per_session(R, n):
    """One, two and four waves a row, few keys and many: the largest of every row,
    the lowest of its ties, and the drafts up to the first that differs."""
    S = 3
    M = S * R
    g = torch.Generator(device="cuda").manual_seed(R + n)
    q = torch.randint(-100, 100, (M, n), device="cuda", generator=g).to(torch.int8)
    best = torch.randint(0, n, (M,), device="cuda", generator=g)
    tie = torch.randint(0, n, (M,), device="cuda", generator=g)
    q[torch.arange(M), best] = 127
    q[torch.arange(M), tie] = 127
    want = torch.minimum(best, tie).to(torch.int32)
    drafts = want.view(S, R)[:, :R - 1].clone()
    match = [R - 1, 0, max(0, R - 2)]
    for i, k in enumerate(match):
        if k < R - 1:
            drafts[i, k] = (drafts[i, k] + 1) % n
    sub = sph.Subset(vocab=n, full=True)
    tok, acc, _ = sph.fuse_verify(q, torch.full((M,), 0.01, device="cuda"), None, None, sub, S, R,
                                  drafts if R > 1 else None)
    sub.close()
    assert torch.equal(tok, want)
    assert acc.tolist() == [min(k, R - 1) for k in match]


@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
@pytest.mark.parametrize("M", [2, 20])
def test_no_cloud_columns(M, wtype):
    """d_cloud = 0 (through the C interface): the partial logits are the bias, on the
    skinny kernel as on the streaming one."""
    from paper_2607_13093_amd import _lib

    n = 777
    g = torch.Generator(device="cuda").manual_seed(n)
    bias = torch.randn((n,), device="cuda", generator=g)
    w = torch.zeros((n, 16), device="cuda", dtype=torch.bfloat16)
    ones = torch.ones((n,), device="cuda")
    sub = sph.Subset(vocab=n, full=True)
    q = torch.empty((M, n), dtype=torch.int8, device="cuda")
    s, z = torch.empty((M,), device="cuda"), torch.full((M, n), float("nan"), device="cuda")
    ws = torch.empty((sph.cloud_partial_workspace(M, sub),), dtype=torch.uint8, device="cuda")
    fp8 = wtype == "fp8"
    _lib.check(_lib.load().sph_cloud_partial_fmt(
        None, 0, M, 0, w.data_ptr(), 16, _lib.SPH_W_FP8_E4M3 if fp8 else _lib.SPH_W_BF16, ones.data_ptr() if fp8 else None,
        bias.data_ptr(), sub.handle, 30.0, 8, 0, q.data_ptr(), s.data_ptr(), z.data_ptr(), ws.data_ptr(), ws.numel(),
        torch.cuda.current_stream().cuda_stream))
    assert torch.equal(z, bias.expand(M, -1))
    amax = bias.abs().max()
    assert torch.equal(s, (amax / 127.0).expand(M))
    assert torch.equal(q, torch.round(bias / (amax / 127.0)).to(torch.int8).expand(M, -1))
    sub.close()
