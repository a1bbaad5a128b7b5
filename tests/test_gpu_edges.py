"""GPU parity at the edges of the MFMA kernels' tiles and K steps: partial K
steps (any multiple of 8 columns), row tiles with one or all rows in use,
subsets that end one position into a tile, and payload rows at every
alignment, through the staged checks of tests/parity.py against the oracle.
"""

import pytest

from synth import Config, make_workload

from test_gpu_payload import run_format_case

pytestmark = pytest.mark.gpu

ENDPOINT = [
    # (sessions, R, d_end, n): every row tile of the endpoint projection
    (3, 3, 8, 257),      # 9 rows, one 8-column step, a tile of one position
    (4, 8, 48, 1535),    # 32 rows, one partial step
    (11, 3, 72, 519),    # 33 rows, a whole and an 8-column step
    (32, 4, 120, 1009),  # 128 rows
    (43, 3, 96, 770),    # 129 rows: 256-row tile
    (64, 4, 56, 513),    # 256 rows
    (53, 6, 184, 1031),  # 318 rows: 320-row tile
]


@pytest.mark.parametrize("fmt", [(8, 0), (4, 0), (8, 256)], ids=["b8", "b4", "b8blk256"])
@pytest.mark.parametrize("shape", ENDPOINT, ids=[f"S{s}R{r}de{e}n{n}" for s, r, e, n in ENDPOINT])
def test_endpoint_partial_steps_and_unaligned_rows(shape, fmt):
    S, R, de, n = shape
    cfg = Config("edge", 400 + sum(shape) + fmt[0], d=de + 128, d_end=de, vocab=n + 300, n_sub=n,
                 subset_kind="choice", sessions=S, rows_per_session=R)
    run_format_case(make_workload(cfg), fmt[0], fmt[1], f"endpoint edge {shape} {fmt}")


# (sessions, R, d_cloud, n): every row tile of the streaming cloud projection
# and each of its widths (32 ... 256 positions per block), one-chunk and
# partial K steps, weight rows that start at every 16-byte place of a line
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
