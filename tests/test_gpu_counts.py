"""GPU parity of the counting screen: candidates proved free of waiting from counts per replica and window, and those
that fail the proof and go on to the slot rings and the replay, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2604_07144_amd import traces                    # noqa: E402
from tests.gpu_harness import GpuWorkload, assert_same, oracle_for, to_records   # noqa: E402

# R, M, B, mean gap (us), and the form of the counting screen: bucket size and columns (16, 8 or 4 for tables up to 159, 319 and more
# replicas; buckets of 512 requests or more are read 16 bytes at a time).  Requests take 2 .. 22 ms, so a gap of g has about
# 20000 / g of them in a window.
FORMS = [
    (33001, 45, 32, 400, 128, 16), (33001, 45, 48, 150, 256, 16), (33001, 45, 64, 150, 512, 16), (33001, 128, 64, 150, 1024, 16),
    (33001, 200, 16, 400, 128, 8), (33001, 200, 24, 150, 256, 8), (33001, 200, 32, 150, 512, 8), (33001, 200, 64, 150, 2048, 8),
    (33001, 900, 10, 400, 128, 4), (33001, 400, 16, 150, 256, 4), (33001, 400, 24, 150, 512, 4), (33001, 400, 48, 150, 2048, 4),
    (40960, 128, 64, 150, 1024, 16),       # rows of whole steps
]
# the same on shorter rows, which it screens in calls of many
SHORT_FORMS = [
    (8191, 45, 32, 400, 128, 16), (8191, 45, 64, 150, 512, 16), (8191, 200, 16, 400, 128, 8), (8191, 200, 48, 150, 1024, 8),
    (8191, 400, 12, 400, 128, 4), (8191, 400, 32, 150, 1024, 4), (8192, 128, 64, 150, 1024, 16),
]
# Identical, always available replicas in calls that are too small for it: rings, streamed evaluation or lists.
CASES = [
    (2048, 3, 24, 40000), (2051, 5, 16, 30000), (1000, 11, 16, 20000), (129, 40, 12, 20000), (127, 63, 12, 20000),
    (130, 64, 12, 20000), (5000, 45, 24, 4000), (20000, 65, 48, 1000), (9000, 1000, 8, 400), (1, 4, 8, 1000), (2, 4, 8, 1000),
    (511, 200, 8, 3000), (513, 200, 64, 3000),
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


@pytest.mark.parametrize("R,M,B,gap,bucket,columns", FORMS)
@pytest.mark.parametrize("C", [13, 40])
def test_counted_rows_match_the_oracle(R, M, B, gap, bucket, columns, C):
    """Few long rows, so several wavefronts share one, each on another 2-byte boundary where R is odd."""
    tr = _trace(R, M, B, gap, R + M)
    rows = _rows(tr, C, R + C)
    with GpuWorkload(tr) as g:
        assert g.route(C)["counts"][:2] == (bucket, columns) and g.route(C)["counts"][2] > 1
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"R={R} M={M} B={B} gap={gap} C={C}")


@pytest.mark.parametrize("R,M,B,gap,bucket,columns", SHORT_FORMS)
def test_counted_rows_of_a_large_call_match_the_oracle(R, M, B, gap, bucket, columns):
    """So many rows that each has one wavefront; 23 different ones over and over."""
    tr = _trace(R, M, B, gap, R + M)
    rows = _rows(tr, 23, R)
    C = 23 * 183
    with GpuWorkload(tr) as g:
        assert g.route(C)["counts"] == (bucket, columns, 1)
        got = to_records(g.eval_device(torch.from_numpy(rows.view(np.int16)).cuda().repeat(183, 1)))
    assert_same(got, np.tile(oracle_for(tr).eval_batch(rows, nthreads=8), 183), f"R={R} M={M} B={B}")


@pytest.mark.parametrize("R,M,B,gap", CASES)
@pytest.mark.parametrize("C", [13, 40])
def test_smaller_calls_match_the_oracle(R, M, B, gap, C):
    tr = _trace(R, M, B, gap, R + M)
    rows = _rows(tr, C, R + C)
    with GpuWorkload(tr) as g:
        assert g.route(C)["counts"] == (0, 0, 0)
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"R={R} M={M} B={B} gap={gap} C={C}")


@pytest.mark.parametrize("offset", range(1, 8))
@pytest.mark.parametrize("R,M,B,gap", [(33001, 128, 64, 150), (33001, 45, 32, 400), (33002, 400, 24, 150), (5001, 45, 24, 4000)])
def test_rows_that_start_anywhere(offset, R, M, B, gap):
    """The batch itself on any 2-byte boundary: 16-byte and 4-byte loads begin inside the first unit."""
    tr = _trace(R, M, B, gap, 77)
    rows = _rows(tr, 9, offset)
    flat = torch.zeros(rows.size + 8, dtype=torch.int16, device="cuda")
    flat[offset:offset + rows.size] = torch.from_numpy(rows.reshape(-1).view(np.int16)).cuda()
    with GpuWorkload(tr) as g:
        assert (g.route(9)["counts"][0] > 0) == (R > 32768)
        got = to_records(g.eval_device(flat[offset:offset + rows.size].view(rows.shape)))
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"offset {offset} R={R}")


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("R,M,B,gap,at", [(33001, 45, 32, 400, 2000), (33001, 128, 64, 150, 1000), (33001, 200, 16, 400, 32900),
                                          (33001, 400, 24, 150, 511), (4096, 33, 16, 40000, 2000)])
def test_exactly_full_and_one_too_many(R, M, B, gap, at, extra):
    """B requests at one instant on a replica that gets no others fill it (nobody waits); one more waits."""
    tr = _trace(R, M, B, gap, 3)
    arrival = tr.arrival_us.copy()
    arrival[at:at + B + extra] = arrival[at]
    tr = traces.custom_trace(np.maximum.accumulate(arrival), tr.prompt_len, tr.out_len, [traces.COEF_STANDARD] * M, B=B)
    rows = np.tile((np.arange(R) % (M - 1)).astype(np.uint16), (4, 1))
    rows[1:, at:at + B + extra] = M - 1
    with GpuWorkload(tr) as g:
        assert (g.route(4)["counts"][0] > 0) == (R > 32768)
        got = g.eval(rows)
        replayed = g.counts()[1]
    want = oracle_for(tr).eval_batch(rows, nthreads=4)
    assert_same(got, want, f"extra {extra}")
    assert (int(want[1]["sum_ttft_us"]) > int(want[0]["sum_ttft_us"])) == bool(extra)
    assert (replayed == 0) == (extra == 0)
