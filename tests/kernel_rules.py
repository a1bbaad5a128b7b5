"""Which kernel a shape takes, asked of the built library's own dispatch rules
(host functions, no GPU), so that a test whose shapes are meant for a kernel can
say so and fails when a rule moves them elsewhere."""

import ctypes

from paper_2607_13093_amd import _lib

_I64 = ctypes.c_int64


def _rule(symbol, args, res=ctypes.c_int):
    f = _lib.load()[symbol]
    f.argtypes, f.restype = args, res
    return f


def stream_groups(M, n):
    return _rule("_ZN3sph13stream_groupsEii", [ctypes.c_int] * 2)(M, n)


def stream_width(M, n):
    return _rule("_ZN3sph12stream_widthEii", [ctypes.c_int] * 2)(M, n)


def mfma_bm(M):
    return _rule("_ZN3sph7mfma_bmEi", [ctypes.c_int])(M)


def stream_tile(M, n, wtype):
    """(row tile, positions per block at most, stages of h, stages of weights,
    lines a stage) of k_mfma_stream."""
    out = (ctypes.c_int * 5)()
    _rule("_ZN3sph11stream_tileEiiiPi", [ctypes.c_int] * 3 + [ctypes.c_void_p], None)(M, n, int(wtype == "fp8"), out)
    return tuple(out)


def cloud_kernel(M, n, K, wtype="bf16", bits=8, block=0):
    """"gemv", "stream", "w1<2>", "w1<3>", "dma256", "dma320" (bf16 weights),
    "dma8_256", "dma8_320" (E4M3), with "q" where the epilogue quantises."""
    if M <= 8:
        return "gemv"
    if stream_groups(M, n) > 0:
        return "stream"
    bm = mfma_bm(M)
    fp8 = wtype == "fp8"
    quant = _rule("_ZN3sph26mfma_quantises_in_epilogueEiiiii", [ctypes.c_int] * 5, ctypes.c_bool)
    if block == 256 and quant(M, n, K, int(fp8), bits):
        return f"dma8_{bm}q" if fp8 else f"dma{bm}q"
    if bm == 256 and not fp8:
        stages = _rule("_ZN3sph14mfma_w1_stagesEi", [ctypes.c_int])(K)
        if stages:
            return f"w1<{stages}>"
    return f"dma8_{bm}" if fp8 else f"dma{bm}"


def gcm_chain(rows, row_bytes, aad_bytes):
    """Blocks that a lane of k_gcm_bulk chains at most; 0: k_gcm_blocks."""
    n, na = -(-row_bytes // 16), -(-aad_bytes // 16)
    chain = max(1, min(16, -(-(rows * n) // 32768)))  # a partial sum's blocks / 256
    data = -(-n // (256 * chain))
    last = n - (data - 1) * 256 * chain if data else 256
    parts = data + (0 if data and (chain > 1 or 256 - last >= na + 2) else 1)
    if chain <= 4 and rows * parts <= 512:
        return 0
    return _rule("_ZN3sph14gcm_bulk_chainElll", [_I64] * 3)(rows, n, na)
