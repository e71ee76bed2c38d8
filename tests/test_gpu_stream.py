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


# R, M, B, mean gap (us), kinds: the slowest kind takes up to 35 ms, so a window holds about 35000 / gap requests.
# With linear costs no more than B are in service at once, and the costs that `tabled` draws need counts here and there.
CASES = [
    (256, 4, 8, 50000, 1),         # identical replicas, a table too small for the slot rings
    (300, 2, 4, 90000, 2), (257, 3, 8, 60000, 3), (1000, 7, 12, 20000, 3),
    (2048, 32, 16, 4000, 3), (2049, 33, 24, 4000, 3), (127, 20, 12, 9000, 3), (128, 20, 12, 9000, 3), (129, 20, 12, 9000, 3),
    (9001, 48, 32, 1250, 3),       # long rows: many wavefronts per row
    (70001, 64, 48, 700, 3),       # 65536 requests and more
    (1, 5, 4, 1000, 3), (2, 5, 4, 1000, 3), (3, 5, 4, 1000, 3),
    (3000, 255, 8, 1500, 3), (3000, 256, 8, 1500, 3),   # more than B at once, and counts that leave no room: listed
]
# More than B at once, and the bucket size that the proof by counting takes.
COUNTED = [
    (300, 5, 64, 200, 2, 4), (9001, 5, 64, 400, 3, 8), (2048, 48, 16, 700, 3, 8), (300, 255, 8, 4000, 3, 16), (257, 64, 12, 1250, 2, 16),
    (9001, 48, 12, 4000, 3, 16), (2049, 255, 12, 200, 2, 32), (2048, 64, 16, 1250, 3, 32), (9001, 7, 64, 200, 2, 32),
    (257, 1024, 8, 1250, 2, 64), (1000, 130, 16, 200, 2, 64), (9001, 256, 16, 200, 2, 128), (2049, 130, 48, 100, 3, 128),
    (70001, 20, 64, 300, 3, 128), (70001, 20, 48, 450, 3, 128),
]


def _linear_tables(tr, kinds):
    """The trace's linear costs as tables."""
    p = tr.prompt_len.astype(np.int64)
    return (np.arange(len(tr.coef), dtype=np.uint32) % kinds, np.stack([a + b * p for a, b, _, _ in KINDS[:kinds]]).astype(np.uint32),
            np.stack([c + d * ((p + 1023) // 1024) for _, _, c, d in KINDS[:kinds]]).astype(np.uint32))


@pytest.mark.parametrize("R,M,B,gap,kinds,bucket", COUNTED)
@pytest.mark.parametrize("tabled", [False, True])
def test_counted_rows_match_the_oracle(R, M, B, gap, kinds, bucket, tabled):
    tr = _trace(R, M, B, gap, kinds, R + M)
    rows = _rows(tr, 14 if R < 50000 else 8, R)
    tables, want = _linear_tables(tr, kinds) if tabled else None, oracle_for(tr)
    with GpuWorkload(tr, tables=tables) as g:
        route = g.route(len(rows))
        assert (route["rings"], route["stream"], route["stream_bucket"]) == (0, 1, bucket)
        got = g.eval(rows)
    assert_same(got, want.eval_batch(rows, nthreads=8), f"R={R} M={M} B={B} gap={gap} kinds={kinds} tabled={tabled}")


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("R,M,B,gap,kinds", [(9001, 48, 12, 4000, 3), (9001, 256, 16, 200, 2), (70001, 20, 48, 450, 3)])
@pytest.mark.parametrize("at", [0, 1001, -100])
def test_exactly_full_and_one_too_many(R, M, B, gap, kinds, at, extra):
    """B requests at one instant on a replica that gets no others: nobody waits.  One more does."""
    tr = _trace(R, M, B, gap, kinds, 3)
    at %= R
    arrival = tr.arrival_us.copy()
    arrival[at:at + B + extra] = arrival[at]
    tr = traces.custom_trace(np.maximum.accumulate(arrival), tr.prompt_len, tr.out_len, [KINDS[m % kinds] for m in range(M)], B=B)
    rows = np.tile((np.arange(R) % (M - 1)).astype(np.uint16), (4, 1))
    rows[1:, at:at + B + extra] = M - 1
    with GpuWorkload(tr) as g:
        assert g.route(4)["stream"] == 1
        got = g.eval(rows)
    want = oracle_for(tr).eval_batch(rows, nthreads=4)
    waits = int(oracle_for(tr, B=64).eval_batch(rows[1:2])[0]["sum_ttft_us"]) < int(want[1]["sum_ttft_us"])
    assert_same(got, want, f"extra {extra} at {at}")
    assert waits == bool(extra)


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
    tr = _trace(3000, 30, 24, 1000, 3, 5, penalty_us=penalty, slo_ttft_us=slo[0], slo_tpot_us=slo[1])
    rows = np.random.default_rng(6).integers(0, 30, size=(12, 3000)).astype(np.uint16)
    for c in range(12):                                    # 0, 3, 6 ... rejected requests; 31 are needed for the 99th percentile
        rows[c, 100:100 + 3 * c * c // 4] = 30
    with GpuWorkload(tr) as g:
        assert g.route(12)["stream"] == 1
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"penalty {penalty} slo {slo}")


def test_odd_batches_and_a_second_call():
    """The batch itself on a 2-byte boundary, rows of odd length, and a call after one that left pending marks."""
    tr = _trace(2051, 33, 24, 1000, 3, 9)
    want = oracle_for(tr)
    with GpuWorkload(tr) as g:
        assert g.route(9)["stream"] == 1
        for seed, C in ((1, 9), (2, 30), (3, 5)):
            rows = _rows(tr, C, seed)
            flat = torch.zeros(rows.size + 8, dtype=torch.int16, device="cuda")
            flat[seed:seed + rows.size] = torch.from_numpy(rows.reshape(-1).view(np.int16)).cuda()
            got = to_records(g.eval_device(flat[seed:seed + rows.size].view(rows.shape)))
            assert_same(got, want.eval_batch(rows, nthreads=8), f"call {seed}")


def test_children_of_a_mixed_cluster():
    tr = _trace(4099, 33, 24, 1000, 3, 11)
    parent = np.random.default_rng(1).integers(0, 33, 4099).astype(np.uint16)
    first, request, replica = traces.draw_edit_lists(3, 25, 4099, 33, 120.0, replica_range=34)
    with GpuWorkload(tr) as g:
        assert g.route(25)["stream"] == 1
        g.set_parent(parent, 25)
        got = g.eval_children(first, request, replica)
    assert_same(got, oracle_for(tr).eval_children(parent, first, request, replica), "children")


# ------------------------------------------------------------------ light clusters: no more than B requests in service at once
@pytest.mark.parametrize("R,M,B,gap,kinds", [
    (1, 5, 4, 1000, 3), (2, 5, 4, 1000, 2), (127, 5, 4, 90000, 3), (128, 20, 12, 9000, 3), (129, 7, 12, 9000, 2),
    (2051, 33, 24, 4000, 3), (9001, 48, 32, 2500, 3), (4096, 4, 8, 20000, 1), (3000, 256, 16, 6000, 3), (700, 1024, 8, 15000, 3),
    (70001, 64, 48, 1500, 3)])
@pytest.mark.parametrize("tabled", [False, True])
def test_light_clusters_settle_every_row(R, M, B, gap, kinds, tabled):
    """Crowded on one replica or not, on one kind or not: nobody can wait, so every row is settled where it is read."""
    tr = _trace(R, M, B, gap, kinds, R + M)
    rows = _rows(tr, 15 if R < 50000 else 9, R)
    tables, want = None, oracle_for(tr)
    if tabled:
        rng = np.random.default_rng(R)
        tables = (np.arange(M, dtype=np.uint32) % kinds, rng.integers(0, 9000, (kinds, R)).astype(np.uint32),
                  rng.integers(0, 30, (kinds, R)).astype(np.uint32))
        want.set_cost_tables(*tables)
    with GpuWorkload(tr, tables=tables) as g:
        assert g.route(len(rows))["stream"] == 2
        for part in (rows, rows[:3], rows[3:]):
            assert_same(g.eval(part), want.eval_batch(part, nthreads=8), f"R={R} M={M} B={B} kinds={kinds} tabled={tabled}")
        assert g.counts()[1] == 0


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("kinds", [1, 3])
def test_as_many_at_once_as_slots_and_one_more(extra, kinds):
    """B requests at one instant: even on one replica nobody waits, and nothing has to be counted.  One more may wait."""
    B, M, R, at = 8, 3, 300, 100
    tr = _trace(R, M, B, 90000, kinds, 4)
    arrival = tr.arrival_us.copy()
    arrival[at:at + B + extra] = arrival[at]
    arrival[at + B + extra:] += np.uint64(10_000_000)
    tr = traces.custom_trace(np.maximum.accumulate(arrival), tr.prompt_len, tr.out_len, [KINDS[m % kinds] for m in range(M)], B=B)
    rows = np.stack([np.full(R, m, dtype=np.uint16) for m in range(M)] + [(np.arange(R) % M).astype(np.uint16)])
    want = oracle_for(tr).eval_batch(rows, nthreads=4)
    assert (int(want[0]["sum_ttft_us"]) > int(oracle_for(tr, B=64).eval_batch(rows[:1])[0]["sum_ttft_us"])) == bool(extra)
    with GpuWorkload(tr) as g:
        assert (g.route(4)["stream"] == 2) == (extra == 0)
        assert_same(g.eval(rows), want, f"extra {extra} kinds {kinds}")


@pytest.mark.parametrize("penalty", [0, 1, 5000, 40_000, 10_000_000])
def test_penalties_where_nobody_can_wait(penalty):
    """Rejected requests are counted without the proof; rows on the fastest kind are read a second time."""
    tr = _trace(3000, 30, 24, 9000, 3, 5, penalty_us=penalty, slo_ttft_us=5000, slo_tpot_us=40)
    rows = np.random.default_rng(6).integers(0, 30, size=(14, 3000)).astype(np.uint16)
    for c in range(14):
        if c % 2:
            rows[c] = rows[c] // 3 * 3 + 1
        rows[c, 100:100 + 3 * c * c // 4] = 30
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=8), f"penalty {penalty}")


@pytest.mark.parametrize("prefill,tpot", [(0, 0), (0, 5), (5, 0), (1, 1)])
def test_costs_that_are_all_alike(prefill, tpot):
    """All values in one bin, the lowest one among them."""
    tr = _trace(500, 4, 16, 9000, 1, 6)
    rows = _rows(tr, 9, 3)
    tables = (np.zeros(4, dtype=np.uint32), np.full((1, 500), prefill, dtype=np.uint32), np.full((1, 500), tpot, dtype=np.uint32))
    want = oracle_for(tr)
    want.set_cost_tables(*tables)
    with GpuWorkload(tr, tables=tables) as g:
        assert_same(g.eval(rows), want.eval_batch(rows, nthreads=4), f"prefill {prefill} tpot {tpot}")


def test_light_clusters_need_no_lists_and_do_not_mind_crowded_rows():
    """16384 requests at 400 a second on 48 replicas of three kinds: the cost model takes no scratch for lists, and rows on one
    replica or on the fast kind are not replayed queue by queue (which took 30 and 6 times as long as even rows)."""
    R, M, C = 16384, 48, 2048
    tr = _trace(R, M, 32, 2500, 3, 12)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    even = torch.randint(0, M, (C, R), generator=g, device="cuda", dtype=torch.int16)
    batches = [even, torch.ones_like(even), even // 3 * 3 + 1]
    out = torch.zeros((C, 8), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with GpuWorkload(tr) as w:
        assert (w.route(C)["stream"], w.route(C)["lists"]) == (2, 0)
        assert free - torch.cuda.mem_get_info()[0] < 64 << 20
        took = []
        for rows in batches:
            best = float("inf")
            for _ in range(5):
                start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                start.record()
                w.eval_device(rows, out)
                end.record()
                torch.cuda.synchronize()
                best = min(best, start.elapsed_time(end))
            took.append(best)
            assert_same(to_records(out[:2]), oracle_for(tr).eval_batch(rows[:2].cpu().numpy().view(np.uint16), nthreads=2))
    assert max(took) < 4.0 * took[0], took


@pytest.mark.parametrize("R,C", [(16001, 14), (16000, 600), (70000, 9)])
@pytest.mark.parametrize("tabled", [False, True])
def test_a_busy_beginning_is_all_that_is_listed(R, C, tabled):
    """More than B requests at once only in the first 1500: a row that fails the proof has those listed and the rest scored on
    arrival, or is handed to the general replay, and the scratch area holds no more than their lists (2.2 GB for all of R = 16001)."""
    M, B = 20, 48
    tr = _trace(R, M, B, 12000, 3, 13)
    rng = np.random.default_rng(2)
    gap = np.where(np.arange(R) < 1500, 450, 12000)
    tr = traces.custom_trace(np.cumsum(rng.integers(0, 2 * gap)), tr.prompt_len, tr.out_len, [KINDS[m % 3] for m in range(M)], B=B)
    rows = _rows(tr, C, R)
    rows[1], rows[2] = 2, np.where(np.arange(R) < 1490, np.arange(R) % M, 2)
    tables, want = _linear_tables(tr, 3) if tabled else None, oracle_for(tr)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with GpuWorkload(tr, tables=tables) as g:
        assert free - torch.cuda.mem_get_info()[0] < 1_400_000_000
        assert (g.route(C)["stream"], g.route(C)["lists"]) == (1, 2)
        assert_same(g.eval(rows), want.eval_batch(rows, nthreads=8), f"R={R} C={C} tabled={tabled}")


@pytest.mark.parametrize("gap,settles", [(1000, False), (4000, True)])
def test_captured_in_a_graph_and_replayed(gap, settles):
    """Launches only, with counts and without: replays with new rows, eager calls and synchronisations in between."""
    tr = _trace(3001, 33, 24, gap, 3, 21)
    want = oracle_for(tr)
    d_rows = torch.zeros((20, 3001), dtype=torch.int16, device="cuda")
    d_out = torch.full((20, 8), -1, dtype=torch.int64, device="cuda")
    with GpuWorkload(tr) as g:
        assert g.route(20)["stream"] == (2 if settles else 1)
        g.eval_device(d_rows, d_out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            g.eval_device(d_rows, d_out)
        for it in range(4):
            rows = _rows(tr, 20, it) if it != 2 else np.random.default_rng(it).integers(0, 33, size=(20, 3001)).astype(np.uint16)
            d_rows.copy_(torch.from_numpy(rows.view(np.int16)).cuda())
            d_out.fill_(-1)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert_same(to_records(d_out), want.eval_batch(rows, nthreads=8), f"replay {it}")
            assert_same(g.eval(rows), to_records(d_out), f"eager call after replay {it}")


def test_one_workload_between_slot_counts():
    """The slot count decides whether nothing has to be counted, counts are kept, or everything is listed: back and forth, tables
    too, on one workload, whose buffers are reused."""
    from paper_2604_07144_amd import binding
    tr = _trace(3001, 33, 24, 1000, 3, 22)
    rows = _rows(tr, 30, 5)
    with GpuWorkload(tr) as g:
        for B, stream, tabled in ((24, 1, False), (64, 2, False), (2, 0, False), (64, 2, True), (24, 1, True), (64, 2, False), (24, 1, False)):
            if tabled:
                binding.ap_costtable_set(g.handle, _linear_tables(tr, 3)[0], tr.t_on_us, tr.t_off_us, B, tr.slo_ttft_us, tr.slo_tpot_us,
                                         tr.penalty_us, *_linear_tables(tr, 3)[1:])
            else:
                binding.ap_costmodel_set(g.handle, binding.make_replicas(tr.coef, tr.t_on_us, tr.t_off_us), B, tr.slo_ttft_us, tr.slo_tpot_us,
                                         tr.penalty_us)
            assert g.route(30)["stream"] == stream
            assert_same(g.eval(rows), oracle_for(tr, B=B).eval_batch(rows, nthreads=8), f"B={B} tabled={tabled}")


@pytest.mark.parametrize("R,M,B", [(64, 3, 8), (128, 3, 8), (1000, 7, 12), (9001, 7, 12)])
@pytest.mark.parametrize("few", [False, True])
def test_steps_full_of_large_values_and_ids_at_the_edge(R, M, B, few):
    """Equal requests: all values are large, or all but a handful are, so that the buffer of large values is filled by every step;
    ids M - 1, M and M + 1 in whole steps."""
    rng = np.random.default_rng(R)
    prompt, out = np.full(R, 700), np.full(R, 90)
    if few:
        prompt[rng.random(R) < 0.02] = 3000
    arrival = np.cumsum(rng.integers(10_000, 60_000, R)).astype(np.uint64)
    tr = traces.custom_trace(arrival, prompt, out, [KINDS[m % 2] for m in range(M)], B=B)
    rows = np.tile((np.arange(R) % M).astype(np.uint16), (5, 1))
    rows[1], rows[2, R // 2], rows[3, R // 2] = M - 1, M, M + 1
    rows[4, ::3] = M
    with GpuWorkload(tr) as g:
        assert g.route(5)["stream"] != 0
        got = g.eval(rows)
    assert_same(got, oracle_for(tr).eval_batch(rows, nthreads=4), f"R={R} few={few}")
