"""The shapes of the GPU tests reach the kernels that they are meant for: the
dispatch rules are host functions, so this needs no GPU."""

import pytest

import kernel_rules as rules
import test_gpu_instances as inst


def _instances():
    """Every instance of the streaming kernel that the rule can pick."""
    found = set()
    for M in list(range(9, 193)) + list(range(193, 1025, 7)):
        for n in [1, 300] + list(range(4096, 65537, 1024)) + list(range(65537, 200000, 9973)):
            if rules.stream_groups(M, n) > 0:
                found |= {(w,) + rules.stream_tile(M, n, w) for w in ("bf16", "fp8")}
    return found


def test_every_streaming_instance_has_a_case():
    want = _instances()
    have = {(w,) + rules.stream_tile(M, n, w) for M, n in inst.STREAM for w in ("bf16", "fp8")}
    assert want - have == set()
    assert len(want) == 37


@pytest.mark.parametrize("pad", [0, 16])
@pytest.mark.parametrize("wtype", ["bf16", "fp8"])
def test_streaming_cases_reach_the_counted_waits(wtype, pad):
    # the wait of step t is a counted one for t <= steps - (stages in flight)
    for M, n in inst.STREAM:
        assert rules.cloud_kernel(M, n, 64, wtype) == "stream"
        _, _, ra, rw, lines = rules.stream_tile(M, n, wtype)
        steps = -(-inst.stream_columns(M, n, wtype, pad) // ((64 if wtype == "bf16" else 128) * lines))
        assert steps - max(ra, rw) >= 5


def test_tiled_cases_reach_their_kernels():
    for M, n, K, wtype, kernel in inst.TILES:
        assert rules.cloud_kernel(M, n, K, wtype) == kernel
    for K, wtype, shapes in inst.SAME:
        for M, n, kernel in shapes:
            assert rules.cloud_kernel(M, n, K, wtype) == kernel, (M, n, K)
