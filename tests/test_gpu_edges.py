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
