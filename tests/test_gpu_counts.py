"""GPU parity of the counting screen: candidates proved free of waiting from counts per replica and window, and those
that fail the proof and go on to the slot rings and the replay, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2604_07144_amd import traces                    # noqa: E402
from tests.gpu_harness import GpuWorkload, assert_same, oracle_for, to_records   # noqa: E402

# R, M, B, mean gap (us): requests take 2 .. 22 ms, so a gap of g has about 20000 / g of them in a window
CASES = [
    (2048, 3, 24, 40000),       # buckets of 16 (eight per step), whole steps
    (2051, 5, 16, 30000),       # 16 or 32, odd row length
    (1000, 11, 16, 20000),      # 32 or 64, ragged last step
    (129, 40, 12, 20000),       # one position into the second step
    (127, 63, 12, 20000),       # the last table with a lane per replica
    (130, 64, 12, 20000),       # the first without
    (5000, 45, 24, 4000),       # buckets of 128
    (20000, 65, 48, 1000),      # a bucket of several steps, two passes over the replicas
    (33001, 128, 64, 400),      # 16-byte loads, every alignment of a row
    (40960, 130, 64, 400),      # rows of whole 512-request steps
    (9000, 1000, 8, 400),       # the largest tables
    (1, 4, 8, 1000), (2, 4, 8, 1000), (511, 200, 8, 3000), (513, 200, 64, 3000),
]


def _trace(R, M, B, gap, seed):
    rng = np.random.default_rng(seed)
    arrival = np.cumsum(rng.integers(0, 2 * gap, R)).astype(np.uint64) + np.uint64(5_000_000_019)
    return traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [traces.COEF_STANDARD] * M, B=B)


def _rows(tr, C, seed):
    """Even rows, then rows that crowd ever fewer replicas, one with an unknown id at each end, one with a single replica."""
    rng = np.random.default_rng(seed)
    rows = rng.integers(0, tr.M, size=(C, tr.R)).astype(np.uint16)
    for i, c in enumerate(range(C // 2, C - 3)):
        rows[c] %= max(1, tr.M >> (i % 4))
    rows[C - 3, 0], rows[C - 2, -1] = tr.M, 0xFFFF
    rows[C - 1] = tr.M - 1
    return rows


@pytest.mark.parametrize("R,M,B,gap", CASES)
@pytest.mark.parametrize("C", [13, 40])
def test_counted_rows_match_the_oracle(R, M, B, gap, C):
    tr = _trace(R, M, B, gap, R + M)
    rows = _rows(tr, C, R + C)
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"R={R} M={M} B={B} gap={gap} C={C}")


@pytest.mark.parametrize("offset", range(1, 8))
def test_rows_that_start_anywhere(offset):
    """The batch itself on any 2-byte boundary: 16-byte and 4-byte loads begin inside the first unit."""
    for R, M, B, gap in ((33001, 128, 64, 400), (5001, 45, 24, 4000), (2051, 5, 16, 30000)):
        tr = _trace(R, M, B, gap, 77)
        rows = _rows(tr, 9, offset)
        flat = torch.zeros(rows.size + 8, dtype=torch.int16, device="cuda")
        flat[offset:offset + rows.size] = torch.from_numpy(rows.reshape(-1).view(np.int16)).cuda()
        with GpuWorkload(tr) as g:
            got = to_records(g.eval_device(flat[offset:offset + rows.size].view(rows.shape)))
        assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"offset {offset} R={R}")


@pytest.mark.parametrize("extra", [0, 1])
def test_exactly_full_and_one_too_many(extra):
    """B requests at one instant on one replica fill it (nobody waits); one more waits."""
    B, M, R = 16, 33, 4096
    tr = _trace(R, M, B, 40000, 3)
    arrival = tr.arrival_us.copy()
    at = 2000
    arrival[at:at + B + extra] = arrival[at]
    tr = traces.custom_trace(np.maximum.accumulate(arrival), tr.prompt_len, tr.out_len, [traces.COEF_STANDARD] * M, B=B)
    rows = np.tile((np.arange(R) % (M - 1)).astype(np.uint16), (4, 1))
    rows[1:, at:at + B + extra] = M - 1
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
        replayed = g.counts()[1]
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=4), f"extra {extra}")
    assert (replayed == 0) == (extra == 0)
