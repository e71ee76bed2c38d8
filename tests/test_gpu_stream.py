"""GPU parity of the streamed evaluation (replicas that are always there, nobody expected to wait), of what it hands to the
listed evaluation, and of both with edit lists, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2604_07144_amd import traces                    # noqa: E402
from tests.gpu_harness import GpuWorkload, assert_same, oracle_for, to_records   # noqa: E402

KINDS = (traces.COEF_STANDARD, traces.COEF_FAST, traces.COEF_SLOW)


def _trace(R, M, B, gap, kinds, seed, **kw):
    rng = np.random.default_rng(seed)
    arrival = np.cumsum(rng.integers(0, 2 * gap, R)).astype(np.uint64) + np.uint64(5_000_000_019)
    return traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % kinds] for m in range(M)], B=B, **kw)


def _rows(tr, C, seed):
    """Even rows; rows on ever fewer replicas (some wait), rows on one kind only (fewer large values than an even spread),
    unknown ids here and there, and at both ends."""
    rng = np.random.default_rng(seed)
    rows = rng.integers(0, tr.M, size=(C, tr.R)).astype(np.uint16)
    for i, c in enumerate(range(C // 2, C - 4)):
        rows[c] = rows[c] % max(1, tr.M >> (i % 4)) if i % 2 else np.minimum(rows[c] // 3 * 3 + i // 2 % 3, tr.M - 1)
    rows[C - 4][rng.random(tr.R) < 0.1] = tr.M + 3
    rows[C - 3, 0], rows[C - 2, -1] = tr.M, 0xFFFF
    rows[C - 1] = tr.M - 1
    return rows


# R, M, B, mean gap (us), kinds: the slowest kind takes up to 35 ms, so a window holds about 35000 / gap requests
CASES = [
    (256, 4, 8, 50000, 1),         # identical replicas, a table too small for the slot rings: buckets of a few requests
    (300, 2, 4, 90000, 2), (257, 3, 8, 60000, 3), (1000, 7, 12, 20000, 3),
    (2048, 32, 16, 4000, 3), (2049, 33, 24, 4000, 3), (127, 20, 12, 9000, 3), (128, 20, 12, 9000, 3), (129, 20, 12, 9000, 3),
    (9001, 48, 32, 1250, 3),       # buckets of whole steps, long rows: many wavefronts per row
    (3000, 255, 8, 1500, 3), (3000, 256, 8, 1500, 3), (700, 1024, 8, 1500, 3),
    (70001, 64, 48, 700, 3),       # 65536 requests and more
    (1, 5, 4, 1000, 3), (2, 5, 4, 1000, 3), (3, 5, 4, 1000, 3),
]


@pytest.mark.parametrize("R,M,B,gap,kinds", CASES)
@pytest.mark.parametrize("tabled", [False, True])
def test_streamed_rows_match_the_oracle(R, M, B, gap, kinds, tabled):
    tr = _trace(R, M, B, gap, kinds, R + M)
    rows = _rows(tr, 14 if R < 50000 else 8, R)
    tables, want = None, oracle_for(tr)
    if tabled:
        rng = np.random.default_rng(R)
        tables = (np.arange(M, dtype=np.uint32) % kinds, rng.integers(0, 9000, (kinds, R)).astype(np.uint32),
                  rng.integers(0, 60, (kinds, R)).astype(np.uint32))
        want.set_cost_tables(*tables)
    with GpuWorkload(tr, tables=tables) as g:
        got = g.eval(rows)
    assert_same(got, want.eval_batch(rows, nthreads=8), f"R={R} M={M} B={B} gap={gap} kinds={kinds} tabled={tabled}")


@pytest.mark.parametrize("penalty", [0, 1, 5000, 40_000, 10_000_000])
@pytest.mark.parametrize("slo", [(500_000, 50_000), (5000, 40)])
def test_penalties_below_among_and_above_the_latencies(penalty, slo):
    tr = _trace(3000, 30, 24, 3000, 3, 5, penalty_us=penalty, slo_ttft_us=slo[0], slo_tpot_us=slo[1])
    rows = np.random.default_rng(6).integers(0, 30, size=(12, 3000)).astype(np.uint16)
    for c in range(12):                                    # 0, 3, 6 ... rejected requests; 31 are needed for the 99th percentile
        rows[c, 100:100 + 3 * c * c // 4] = 30
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"penalty {penalty} slo {slo}")


def test_odd_batches_and_a_second_call():
    """The batch itself on a 2-byte boundary, rows of odd length, and a call after one that left pending marks."""
    tr = _trace(2051, 33, 24, 4000, 3, 9)
    want = oracle_for(tr)
    with GpuWorkload(tr) as g:
        for seed, C in ((1, 9), (2, 30), (3, 5)):
            rows = _rows(tr, C, seed)
            flat = torch.zeros(rows.size + 8, dtype=torch.int16, device="cuda")
            flat[seed:seed + rows.size] = torch.from_numpy(rows.reshape(-1).view(np.int16)).cuda()
            got = to_records(g.eval_device(flat[seed:seed + rows.size].view(rows.shape)))
            assert_same(got, want.eval_batch(rows, nthreads=8), f"call {seed}")


def test_children_of_a_mixed_cluster():
    tr = _trace(4099, 33, 24, 4000, 3, 11)
    parent = np.random.default_rng(1).integers(0, 33, 4099).astype(np.uint16)
    first, request, replica = traces.draw_edit_lists(3, 25, 4099, 33, 120.0, replica_range=34)
    with GpuWorkload(tr) as g:
        g.set_parent(parent, 25)
        got = g.eval_children(first, request, replica)
    assert_same(got, oracle_for(tr).eval_children(parent, first, request, replica), "children")
