"""Performance cases of the split-head vocabulary projection.

Each case is work that a program using the library does through its Python
binding: a decoding step (cloud call, then endpoint call), one side's call on
its own (cloud and endpoint are different machines in the paper's setting, so
each is a program by itself), or the sealing and opening of a payload batch.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare`` makes a case's inputs, plan and buffers, ``run`` is one pass and
``work``, ``tolerance`` and ``exact`` say what a pass has to do, how far two
correct implementations may differ and what 64-bit arithmetic gives.

Ranges: hidden sizes 512 to 8192 with endpoint slices of 48 to 512 columns
(the paper: D = 4096, D_end = 48 ... 512), vocabularies of 8192 to 152064 ids,
subsets of 5% to 100% of them (the paper's languages: 30%, 40%, 100%), windows
of 1 to 9 rows (drafts N = 0 ... 8) of 1 to 256 sessions, bf16 and E4M3 cloud
weights, 8- and 4-bit payloads with one scale per row or per block, greedy and
sampled selection, bf16 and int8 hidden states.
"""

import math

import numpy as np
import torch

from paper_2607_13093_amd import api as sph

CLIP = 30.0
KEY = bytes(range(32))
AAD_BYTES = 32


def _case(name, path, **kw):
    c = {"name": name, "path": path, "d": 4096, "d_end": 256, "vocab": 128256, "n": 49152,
         "sessions": 1, "rows": 5, "wtype": "bf16", "bits": 8, "block": 0, "mode": "greedy",
         "temperature": 1.0, "top_p": 1.0, "hidden_codes": False, "bias": False}
    c.update(kw)
    return c


def listed():
    return [
        # a toy-sized head: every kernel is a few microseconds, launches and host code count
        _case("tiny_step", "step", d=512, d_end=64, vocab=8192, n=4096, rows=3),
        # one user's step: five rows against 49152 weight rows, a stream from memory
        _case("decode_step", "step"),
        # the same on a server that keeps E4M3 weights, with the larger hidden size
        _case("decode_fp8_cloud", "cloud", d=5120, d_end=320, vocab=152064, n=65536, wtype="fp8"),
        # one user's endpoint with temperature and top-p: few rows, each sampled over 65536 ids
        _case("decode_sample_endpoint", "endpoint", d=5120, d_end=320, vocab=152064, n=65536,
              mode="sample", temperature=0.7, top_p=0.9),
        # the paper's model (D 4096, D_end 96, 150000 ids, 30% of them) with two users' windows
        # of eight drafts: more rows than the streaming kernel takes, few for the matrix cores
        _case("paper_two_users_step", "step", d_end=96, vocab=150000, n=45001, sessions=2, rows=9),
        # the same model with 40% of the ids and a moderate batch of users
        _case("paper_batch_step", "step", d_end=96, vocab=150000, n=60000, sessions=31, rows=5),
        # a batch of 64 users' windows: as many bytes as operations
        _case("batched_step", "step", d_end=512, vocab=152064, n=60000, sessions=64),
        # a large server batch over the whole vocabulary
        _case("dense_full_step", "step", d=8192, d_end=512, n=128256, sessions=256, rows=8),
        # the same batch on a subset with the compact options: 4-bit codes with block scales and
        # the hidden state as int8 codes
        _case("dense_sub_compact_step", "step", d=8192, d_end=512, n=32768, sessions=256, rows=8,
              bits=4, block=256, hidden_codes=True),
        # E4M3 weights with a batch of users
        _case("batch_fp8_cloud", "cloud", d=5120, d_end=320, vocab=152064, n=65536, sessions=128,
              wtype="fp8"),
        # that batch's endpoint: sampling 640 rows of 65536 ids
        _case("batch_sample_endpoint", "endpoint", d=5120, d_end=320, vocab=152064, n=65536,
              sessions=128, mode="sample", temperature=0.7, top_p=0.9),
        # a batch's payload, codes and scales as one message per row, sealed and opened
        _case("batch_seal_open", "seal", vocab=152064, n=60000, sessions=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "cloud", "endpoint", "endpoint", "seal"])
    while True:
        vocab = rng.choice([32000, 100352, 128256, 150000, 152064])
        rows = rng.choice([1, 2, 3, 5, 6, 7, 8, 9])
        sessions = _log(rng, 1, 256)
        d = rng.choice([2048, 4096, 4096, 5120, 8192])
        n = min(vocab, _log(rng, vocab // 20, vocab))
        if rng.random() < 0.4:
            n = min(vocab, n // 64 * 64)
        if sessions * rows <= 2048 and sessions * rows * n * d <= 2048 * 128256 * 8192 * 0.9:
            break
    # endpoints sample; whole steps do not, as one payload code on the other side of a rounding
    # boundary can change a sampled token
    sampled = path == "endpoint" and rng.random() < 0.75
    bits, block = rng.choice([(8, 0), (8, 0), (8, 0), (4, 256), (8, 256), (4, 0), (8, 1024)])
    return _case(
        "", path, d=d, d_end=rng.choice([48, 64, 96, 128, 256, 320, 512]), vocab=vocab, n=n,
        sessions=sessions, rows=rows,
        wtype=rng.choice(["bf16", "bf16", "fp8"]), bits=bits, block=block,
        mode="sample" if sampled else "greedy",
        temperature=round(rng.uniform(0.4, 1.2), 2) if sampled else 1.0,
        top_p=rng.choice([0.8, 0.9, 0.95, 1.0]) if sampled else 1.0,
        hidden_codes=path in ("step", "endpoint") and rng.random() < 0.25,
        bias=path in ("step", "cloud") and rng.random() < 0.25)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + stream)
    return g


def _normal_bf16(rows, cols, seed, stream, scale=1.0):
    """Normal values (times scale) rounded to bf16, a block of rows at a time."""
    g = _gen(seed, stream)
    out = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    for r in range(0, rows, 32768):
        e = min(rows, r + 32768)
        out[r:e] = torch.randn((e - r, cols), generator=g, device="cuda") * scale
    return out


def _ids(case, seed):
    if case["n"] == case["vocab"]:
        return np.arange(case["vocab"], dtype=np.int32)
    rng = np.random.default_rng([int(seed), 7])
    return np.sort(rng.choice(case["vocab"], size=case["n"], replace=False)).astype(np.int32)


def _scale_shape(case):
    M = case["sessions"] * case["rows"]
    return (M,) if case["block"] == 0 else (M, -(-case["n"] // case["block"]))


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    M, d, de = case["sessions"] * case["rows"], case["d"], case["d_end"]
    x = {"ids": _ids(case, seed)}
    inv = 1.0 / math.sqrt(d)
    if case["path"] == "seal":
        x["codes"], x["scale"] = _payload(case, seed)
        g = _gen(seed, 5)
        x["iv"] = torch.randint(0, 256, (M, 12), generator=g, device="cuda", dtype=torch.uint8)
        x["aad"] = torch.randint(0, 256, (M, AAD_BYTES), generator=g, device="cuda", dtype=torch.uint8)
        return x
    x["h"] = _normal_bf16(M, d, seed, 0)
    if case["path"] != "cloud":
        x["w_end"] = _normal_bf16(case["vocab"], de, seed, 1, inv)
    if case["path"] != "endpoint":
        w = _normal_bf16(case["vocab"], d - de, seed, 2, inv)
        if case["wtype"] == "fp8":
            codes = torch.empty(w.shape, dtype=torch.float8_e4m3fn, device="cuda")
            rs = torch.empty((case["vocab"],), dtype=torch.float32, device="cuda")
            for r in range(0, case["vocab"], 32768):
                f = w[r:r + 32768].float()
                s = f.abs().amax(dim=1) / 448.0
                codes[r:r + 32768] = (f / s[:, None]).to(torch.float8_e4m3fn)
                rs[r:r + 32768] = s
            x["w_cloud"], x["w_scale"] = codes, rs
        else:
            x["w_cloud"], x["w_scale"] = w, None
        x["bias"] = (torch.randn((case["vocab"],), generator=_gen(seed, 3), device="cuda") * 0.5
                     if case["bias"] else None)
    else:
        x["codes"], x["scale"] = _payload(case, seed)
        if case["hidden_codes"]:
            f = x["h"].float()
            s = f.abs().amax(dim=1) / 127.0
            x["hq"], x["hs"] = torch.round(f / s[:, None]).clamp(-127, 127).to(torch.int8), s
    if case["path"] != "cloud" and case["rows"] > 1:
        x["drafts"] = _drafts(case, x, seed)
    else:
        x["drafts"] = None
    return x


def _payload(case, seed):
    """A received payload: codes of normal partial logits in the case's format."""
    M, n, bits, block = case["sessions"] * case["rows"], case["n"], case["bits"], case["block"]
    g = _gen(seed, 4)
    qmax = 127.0 if bits == 8 else 7.0
    codes = torch.empty((M, n if bits == 8 else (n + 1) // 2), device="cuda",
                        dtype=torch.int8 if bits == 8 else torch.uint8)
    scale = torch.empty(_scale_shape(case), dtype=torch.float32, device="cuda")
    for m in range(M):
        z = torch.randn((n,), generator=g, device="cuda")
        if block:
            nb = -(-n // block)
            zp = torch.nn.functional.pad(z, (0, nb * block - n)).view(nb, block)
            s = zp.abs().amax(dim=1) / qmax
            q = torch.round(zp / s[:, None]).view(-1)[:n]
        else:
            s = z.abs().max() / qmax
            q = torch.round(z / s)
        scale[m] = s
        q = q.clamp(-qmax, qmax).to(torch.int8)
        if bits == 4:
            q = torch.nn.functional.pad(q, (0, n & 1)).to(torch.uint8) & 15
            q = q[0::2] | (q[1::2] << 4)
        codes[m] = q
    return codes, scale


def _drafts(case, x, seed):
    """Half of the drafts are what the head would say, half other ids of the subset."""
    S, R = case["sessions"], case["rows"]
    rng = np.random.default_rng([int(seed), 8])
    ids = x["ids"]
    rand = ids[rng.integers(0, len(ids), size=(S, R - 1))]
    if case["path"] == "step" and case["wtype"] == "bf16":
        sel = torch.from_numpy(ids.astype(np.int64)).cuda()
        z = x["h"][:, case["d_end"]:] @ x["w_cloud"][sel].t()
        z += x["h"][:, :case["d_end"]] @ x["w_end"][sel].t()
        guess = ids[z.argmax(dim=1).cpu().numpy()].reshape(S, R)[:, :R - 1]
        rand = np.where(rng.random((S, R - 1)) < 0.5, guess, rand)
    return torch.from_numpy(np.ascontiguousarray(rand.astype(np.int32))).cuda()


# ---------------------------------------------------------------------------
# a pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    x = _inputs(case, seed)
    M, n = case["sessions"] * case["rows"], case["n"]
    dev = torch.device("cuda")

    def bytes_(count):
        return torch.empty(max(1, count), dtype=torch.uint8, device=dev)

    st = {"case": dict(case), "x": x}
    if case["path"] == "seal":
        st["key"] = sph.GcmKey(KEY)
        codes, scales = x["codes"].view(torch.uint8), x["scale"].view(M, -1).view(torch.uint8)
        st["segs"] = (codes, scales)
        st["sealed"] = (torch.empty_like(codes), torch.empty_like(scales))
        st["opened"] = (torch.empty_like(codes), torch.empty_like(scales))
        st["tag"] = torch.empty((M, 16), dtype=torch.uint8, device=dev)
        st["ok"] = torch.empty((M,), dtype=torch.int32, device=dev)
        st["ws"] = bytes_(sph.gcm_workspace(M, codes.shape[1] + scales.shape[1]))
        return st
    full = n == case["vocab"]
    st["sub"] = sub = (sph.Subset(vocab=n, full=True) if full
                       else sph.Subset(x["ids"], vocab=case["vocab"]))
    mode = sph.SAMPLE if case["mode"] == "sample" else sph.GREEDY
    if case["path"] != "endpoint":
        codes = torch.empty((M, sph.payload_code_bytes(n, case["bits"])), device=dev,
                            dtype=torch.int8 if case["bits"] == 8 else torch.uint8)
        st["payload"] = (codes, torch.empty(_scale_shape(case), dtype=torch.float32, device=dev))
        st["ws_cloud"] = bytes_(sph.cloud_partial_workspace(M, sub))
    else:
        st["payload"] = (x["codes"], x["scale"])
    if case["path"] != "cloud":
        want = case["path"] == "endpoint"
        st["out"] = (torch.empty((M,), dtype=torch.int32, device=dev),
                     torch.empty((case["sessions"],), dtype=torch.int32, device=dev),
                     torch.empty((M, n), dtype=torch.float32, device=dev) if want else None)
        if case["hidden_codes"]:
            st["ws_end"] = bytes_(sph.fuse_verify_hq_workspace(M, case["d_end"], sub, mode))
            st["hidden"] = ((x["hq"], x["hs"]) if want else
                            (torch.empty((M, case["d"]), dtype=torch.int8, device=dev),
                             torch.empty((M,), dtype=torch.float32, device=dev)))
        else:
            st["ws_end"] = bytes_(sph.fuse_verify_workspace(M, sub, mode))
        st["select"] = {"mode": mode, "temperature": case["temperature"], "top_p": case["top_p"],
                        "seed": int(seed) + 0x5EED}
    return st


def run(st):
    case, x = st["case"], st["x"]
    if case["path"] == "seal":
        sph.gcm_seal_segments(st["key"], st["segs"], x["iv"], x["aad"], out=st["sealed"],
                              tag=st["tag"], workspace=st["ws"])
        sph.gcm_open_segments(st["key"], st["sealed"], x["iv"], st["tag"], x["aad"],
                              out=st["opened"], ok=st["ok"], workspace=st["ws"])
        return {"sealed": st["sealed"], "tag": st["tag"], "opened": st["opened"], "ok": st["ok"]}
    h, de = x["h"], case["d_end"]
    q, s = st["payload"]
    fmt = {"bits": case["bits"], "block": case["block"]}
    res = {}
    if case["path"] != "endpoint":
        sph.cloud_partial(h[:, de:], x["w_cloud"], st["sub"], CLIP, w_row_scale=x["w_scale"],
                          bias=x["bias"], workspace=st["ws_cloud"], out=(q, s, None), **fmt)
        res["codes"], res["scale"] = q, s
        if case["path"] == "cloud":
            return res
    S, R = case["sessions"], case["rows"]
    if case["hidden_codes"]:
        hq, hs = st["hidden"]
        if case["path"] == "step":
            sph.hidden_quantize(h, out=(hq, hs))
            res["hidden_codes"], res["hidden_scale"] = hq, hs
        tok, acc, fused = sph.fuse_verify_hq(q, s, hq, hs, de, x["w_end"], st["sub"], S, R,
                                             x["drafts"], workspace=st["ws_end"], out=st["out"],
                                             **st["select"], **fmt)
    else:
        tok, acc, fused = sph.fuse_verify(q, s, h[:, :de], x["w_end"], st["sub"], S, R,
                                          x["drafts"], workspace=st["ws_end"], out=st["out"],
                                          **st["select"], **fmt)
    res["tokens"], res["accept"] = tok, acc
    if fused is not None:
        res["fused"] = fused
    return res


# ---------------------------------------------------------------------------
# what a pass has to do
# ---------------------------------------------------------------------------

def work(case):
    M, n, d, de = case["sessions"] * case["rows"], case["n"], case["d"], case["d_end"]
    payload = M * (-(-n * case["bits"] // 8)) + 4 * int(np.prod(_scale_shape(case)))
    if case["path"] == "seal":
        # sealed and opened: each reads and writes every byte once
        return {"bytes": 4 * payload + M * (12 + AAD_BYTES + 16) * 2, "flops": 0}
    b = f = 0
    if case["path"] != "endpoint":
        wb = 2 if case["wtype"] == "bf16" else 1
        b += n * (d - de) * wb + 4 * n + M * (d - de) * 2 + payload
        b += 4 * n * ((case["wtype"] == "fp8") + bool(case["bias"]))
        f += 2 * M * n * (d - de)
    if case["path"] != "cloud":
        hb = 1 if case["hidden_codes"] else 2
        b += n * de * 2 + 4 * n + M * de * hb + payload + 4 * M
        f += 2 * M * n * de
        if case["path"] == "endpoint":
            b += 4 * M * n
        elif case["hidden_codes"]:
            b += M * d * 3
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Measured against 64 bits over these ranges: scales and fused logits are up to 4.8e-7 off
    (2-norm) and 2.3e-6 at the largest, so another order of the fp32 sums may show four times
    that.  Up to 1.1e-5 of the 8-bit codes lie on the other side of a rounding boundary (a few
    codes of a small call), and one row in some 100000 has another best id, so that a batch
    may have one such row."""
    if case["path"] == "seal":
        return "exact"
    M = case["sessions"] * case["rows"]
    differ = max(5e-5, 3.0 / (M * case["n"]))
    return {"rel": 2e-6, "max": 1e-5, "differ": differ if M < 200 else min(0.01, 1.5 / M)}


def exact(case, seed):
    """Scales and fused logits in 64 bits; codes, tokens and bytes have no such value."""
    if case["path"] == "seal":
        return None
    x = _inputs(case, seed)
    M, n, de = case["sessions"] * case["rows"], case["n"], case["d_end"]
    ids = torch.from_numpy(x["ids"].astype(np.int64)).cuda()
    h = x["h"].double()
    res = {}
    step = 16384
    if case["path"] != "endpoint":
        res["codes"] = None
        qmax = 127.0 if case["bits"] == 8 else 7.0
        block = case["block"]
        best = torch.zeros(_scale_shape(case), dtype=torch.float64, device="cuda")
        for j in range(0, n, step):
            sel = ids[j:j + step]
            w = x["w_cloud"][sel] if case["wtype"] == "bf16" else x["w_cloud"].view(torch.uint8)[sel].view(torch.float8_e4m3fn).float()
            w = w.double()
            if x["w_scale"] is not None:
                w *= x["w_scale"][sel].double()[:, None]
            z = h[:, de:] @ w.t()
            if x["bias"] is not None:
                z += x["bias"][sel].double()[None, :]
            z = z.clamp(-CLIP, CLIP).abs()
            if block == 0:
                best = torch.maximum(best, z.amax(dim=1))
            else:
                nb = -(-z.shape[1] // block)
                zp = torch.nn.functional.pad(z, (0, nb * block - z.shape[1]))
                best[:, j // block:j // block + nb] = zp.view(M, nb, block).amax(dim=2)
        res["scale"] = best / qmax
        if case["path"] == "cloud":
            return res
        if case["hidden_codes"]:
            res["hidden_codes"], res["hidden_scale"] = None, h.abs().amax(dim=1) / 127.0
    res["tokens"] = res["accept"] = None
    if case["path"] == "endpoint":
        q = x["codes"]
        if case["bits"] == 4:
            nib = torch.stack((q & 15, q >> 4), dim=2).view(M, -1)[:, :n].to(torch.int8)
            q = torch.where(nib >= 8, nib - 16, nib)
        he = h[:, :de]
        if case["hidden_codes"]:
            he = x["hq"][:, :de].double() * x["hs"].double()[:, None]
        fused = torch.empty((M, n), dtype=torch.float64, device="cuda")
        for j in range(0, n, step):
            e = min(n, j + step)
            fused[:, j:e] = he @ x["w_end"][ids[j:e]].double().t()
        for m in range(M):
            s = x["scale"][m].double()
            if case["block"]:
                s = s.repeat_interleave(case["block"])[:n]
            fused[m] += q[m].double() * s
        res["fused"] = fused
    return res
