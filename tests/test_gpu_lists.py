"""GPU parity of the lists' edges (tile and run remainders, rows that list everything or nothing, replicas gone early), of small
calls that are left to the fused replay, and of the list replay's register groups, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2604_07144_amd import traces                    # noqa: E402
from tests.gpu_harness import GpuWorkload, assert_same, oracle_for   # noqa: E402

KINDS = (traces.COEF_STANDARD, traces.COEF_FAST, traces.COEF_SLOW)
U64MAX = 0xFFFFFFFFFFFFFFFF


def _elastic(R, M, B, gap, seed, steady, **kw):
    rng = np.random.default_rng(seed)
    arrival = np.cumsum(rng.integers(0, 2 * gap, R)).astype(np.uint64) + np.uint64(1_000_003)
    at = rng.integers(int(arrival[0]), int(arrival[-1]) + 1, size=(M, 2))
    stays = rng.random(M) < steady
    t_on = np.where(stays, 0, at.min(axis=1)).astype(np.uint64)
    t_off = np.where(stays, np.uint64(U64MAX), at.max(axis=1).astype(np.uint64))
    return traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(M)], t_on, t_off,
                               B=B, **kw)


def _rows(tr, C, seed):
    """Even rows; rows on few replicas (lists are long); rows that only use replicas as long as they are there
    (nothing rejected, so the histograms are needed); unknown ids."""
    rng = np.random.default_rng(seed)
    rows = rng.integers(0, tr.M, size=(C, tr.R)).astype(np.uint16)
    third = C // 3
    for i, c in enumerate(range(third, 2 * third)):
        rows[c] %= max(1, tr.M >> (i % 5))
    there = (tr.arrival_us[:, None] >= tr.t_on_us[None]) & (tr.arrival_us[:, None] + np.uint64(10_000_000) < tr.t_off_us[None])
    for c in range(2 * third, C - 1):
        pick = rng.random((tr.R, tr.M)) * there
        rows[c] = pick.argmax(axis=1).astype(np.uint16)
    rows[C - 1][rng.random(tr.R) < 0.02] = tr.M
    return rows


@pytest.mark.parametrize("R,M,B,gap,steady", [
    (6000, 50, 24, 1200, 0.5), (6001, 33, 24, 1500, 0.9), (5000, 70, 16, 1500, 0.5), (2047, 20, 12, 4000, 0.7), (2048, 12, 8, 9000, 0.7),
    (1025, 64, 32, 900, 0.9), (1024, 65, 32, 900, 0.9), (66000, 40, 48, 600, 0.8), (300, 5, 16, 30000, 0.6),
    # nothing streamed: crowded, so that every request is listed; few and many bits in an id, a row a tile and one more
    (1023, 3, 8, 20, 0.5), (2049, 64, 16, 3, 0.0), (3000, 65, 16, 3, 0.5), (4097, 129, 8, 2, 0.3), (70001, 300, 64, 1, 0.3)])
@pytest.mark.parametrize("tabled", [False, True])
def test_elastic_rows_match_the_oracle(R, M, B, gap, steady, tabled):
    tr = _elastic(R, M, B, gap, R + M, steady)
    rows = _rows(tr, 13 if R < 20000 else 7, R)
    tables, want = None, oracle_for(tr)
    if tabled:
        rng = np.random.default_rng(R)
        tables = (np.arange(M, dtype=np.uint32) % 3, rng.integers(0, 9000, (3, R)).astype(np.uint32), rng.integers(0, 60, (3, R)).astype(np.uint32))
        want.set_cost_tables(*tables)
    with GpuWorkload(tr, tables=tables) as g:
        for part in (rows, rows[:5], rows[5:]):
            assert_same(g.eval(part), want.eval_batch(part, nthreads=8), f"R={R} M={M} B={B} gap={gap} steady={steady} tabled={tabled}")


@pytest.mark.parametrize("B", [1, 7, 8, 9, 12, 13, 16, 17, 24, 25, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("slow", [False, True])
def test_queues_that_fill_drain_and_fill_again(B, slow):
    """Quiet stretches and bursts in turn, so that a queue has few, half or all of its slots in use: every group of slot registers
    holds still at some time.  `slow`: tokens so slow that the tpot bins span more than a byte."""
    rng = np.random.default_rng(B)
    R, M = 4000, 4
    gap = np.repeat(rng.choice([60, 400, 1500, 6000], 40), R // 40)
    coef = [(2000, 3, 25, 5), (1200, 2, 15, 3), (3500, 5, 40, 2000 if slow else 8), (2000, 3, 25, 5)]
    tr = traces.custom_trace(np.cumsum(rng.integers(0, 2 * gap)), rng.integers(1, 8000, R), rng.integers(1, 60 if slow else 300, R), coef, B=B)
    rows = rng.integers(0, M, size=(70, R)).astype(np.uint16)
    rows[1], rows[2] = 2, np.arange(R) // 1000
    with GpuWorkload(tr) as g:
        assert_same(g.eval(rows), oracle_for(tr).eval_batch(rows, nthreads=8), f"B={B} slow={slow}")


@pytest.mark.parametrize("R,C", [(800, 9), (801, 9), (800, 512), (800, 513), (5, 1)])
def test_small_calls_on_either_side_of_the_line(R, C):
    tr = _elastic(R, 6, 8, 3000, R, 0.5)
    rows = np.random.default_rng(C).integers(0, 6, size=(C, R)).astype(np.uint16)
    with GpuWorkload(tr) as g:
        want = oracle_for(tr).eval_batch(rows, nthreads=8)
        for _ in range(2):
            assert_same(g.eval(rows), want, f"R={R} C={C}")


@pytest.mark.parametrize("stride", [2048, 2049])
def test_a_workgroup_whose_first_candidate_needs_no_merge(stride):
    """More candidates than the merge has workgroups: one goes through several, and the first of them, settled by penalty, must
    not keep the others from their histograms (all rows up to `stride` rejected, then one in 64 with nothing rejected)."""
    R, M, C = 130, 4, 3 * 2048
    tr = _elastic(R, M, 8, 3000, 7, 1.0, penalty_us=3_600_000_000)
    tr = traces.custom_trace(tr.arrival_us, tr.prompt_len, tr.out_len, [KINDS[m % 3] for m in range(M)],
                             np.where(np.arange(M) == 0, int(tr.arrival_us[R // 2]), 0), np.full(M, U64MAX, dtype=np.uint64), B=8)
    rows = np.full((C, R), M, dtype=np.uint16)
    some = np.random.default_rng(3).integers(0, M, size=(48, R)).astype(np.uint16)
    at = np.arange(stride, C, 64)[:48]
    rows[at] = some[:at.shape[0]]
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
    want = np.repeat(oracle_for(tr).eval_batch(rows[:1]), C)
    want[at] = oracle_for(tr).eval_batch(some[:at.shape[0]])
    assert_same(got, want, f"stride {stride}")


@pytest.mark.parametrize("R,M,C,fused", [(256, 4, 1, True), (256, 4, 512, True), (256, 4, 513, False), (200, 65, 256, True),
                                         (200, 65, 257, False), (200, 128, 3, True), (200, 129, 3, False), (200, 129, 4, True),
                                         (800, 2, 40, True), (801, 2, 40, False)])
def test_small_calls_report_what_larger_ones_do(R, M, C, fused):
    """A trace so crowded that every request is listed: no row counts as replayed, whether few rows are scored or many."""
    rng = np.random.default_rng(R + M)
    tr = traces.custom_trace(np.cumsum(rng.integers(0, 3, R)), rng.integers(1, 4000, R), rng.integers(1, 200, R),
                             [KINDS[m % 3] for m in range(M)], B=2)
    rows = rng.integers(0, M, size=(C, R)).astype(np.uint16)
    rows[C // 2] = 1
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] == (3 if fused else 1)
        assert_same(g.eval(rows), oracle_for(tr).eval_batch(rows, nthreads=8), f"R={R} M={M} C={C}")
        assert g.counts() == (C, 0)


@pytest.mark.parametrize("R,fused", [(200, True), (584, True), (720, False)])
def test_small_calls_of_replicas_that_come_and_go(R, fused):
    """Lists next to empty and the rest streamed, on either side of the line up to which the fused replay takes such calls."""
    rng = np.random.default_rng(R)
    arrival = np.cumsum(rng.integers(1, 2_000_000, R))
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(8)], B=8,
                             t_off_us=[int(arrival[R // 5])] + [traces.UINT64_MAX] * 7)
    rows = rng.integers(0, 8, size=(97, R)).astype(np.uint16)
    rows[40], rows[41] = 0, 1
    with GpuWorkload(tr) as g:
        assert g.route(97)["lists"] == (3 if fused else 2)
        assert_same(g.eval(rows), oracle_for(tr).eval_batch(rows, nthreads=8), f"R={R}")


@pytest.mark.parametrize("R", [1023, 2048, 2049, 3073, 5121])
@pytest.mark.parametrize("M,B,C", [(3, 24, 700), (5, 64, 1025), (70, 48, 600)])
def test_equally_long_lists_over_many_blocks_of_candidates(R, M, B, C):
    """Every request listed on permanent replicas: odd numbers of tiles, runs that end with a block, lanes without requests, and a number
    of workgroups that does not divide evenly among the XCDs."""
    rng = np.random.default_rng(R + M)
    tr = traces.custom_trace(np.cumsum(rng.integers(0, 40 if M < 70 else 4, R)), rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[0]] * M, B=B)
    rows = rng.integers(0, M, size=(C, R)).astype(np.uint16)
    rows[1], rows[2], rows[C - 1] = 0, np.arange(R) // 8 % M, M
    rows[300:320] = np.sort(rows[300:320], axis=1)
    some = np.unique(np.concatenate([np.arange(4), np.arange(4, C, 37), np.arange(255, 258), np.arange(300, 304), np.arange(C - 3, C)]))
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] == 1
        got = g.eval(rows)
    assert_same(got[some], oracle_for(tr).eval_batch(rows[some], nthreads=8), f"R={R} M={M} B={B}")


@pytest.mark.parametrize("M", [772, 773, 784, 794, 795])
def test_tables_that_fill_the_lds(M):
    """Large tables, up to the line from which they are left to the general replay (794 replicas of three kinds with 16-bit counts).  Nothing
    rejected, a part listed and a part streamed, bins from both."""
    rng = np.random.default_rng(M)
    R, B = 3000, 4
    arrival = np.cumsum(np.concatenate([rng.integers(0, 3, R // 2), rng.integers(20_000, 60_000, R - R // 2)])).astype(np.uint64)
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(M)],
                             np.where(np.arange(M) % 5 == 0, int(arrival[R // 4]), 0), B=B)
    rows = rng.integers(0, M, size=(700, R)).astype(np.uint16)
    rows[3] = rows[3] % 7
    some = np.concatenate([np.arange(6), np.arange(6, 700, 60)])
    with GpuWorkload(tr) as g:
        assert g.route(700)["lists"] == (2 if M < 795 else 0)
        got = g.eval(rows)
    assert_same(got[some], oracle_for(tr).eval_batch(rows[some], nthreads=8), f"M={M}")


@pytest.mark.parametrize("load", [1, 8, 200])
@pytest.mark.parametrize("slow", [False, True])
@pytest.mark.parametrize("kinds", [1, 3])
def test_bins_few_and_many(load, slow, kinds):
    """From a trace on which next to no listed request leaves a bins word to one on which all do, in one word and in two; one queue takes
    most requests of a row, others none."""
    rng = np.random.default_rng(load)
    R, M, B = 5000, 9, 12
    arrival = np.cumsum(rng.integers(0, max(2, 3200 // load), R)).astype(np.uint64)
    coef = [KINDS[m % kinds] for m in range(M)]
    if slow:
        coef[0] = (3500, 5, 40, 2000)
    tr = traces.custom_trace(arrival, rng.integers(1, 8000, R), rng.integers(1, 60 if slow else 300, R), coef, B=B)
    rows = rng.integers(0, M, size=(300, R)).astype(np.uint16)
    rows[1], rows[2] = np.where(rng.random(R) < 0.9, 4, rows[1]), 8
    rows[3, ::7] = M
    with GpuWorkload(tr) as g:
        assert_same(g.eval(rows)[:24], oracle_for(tr).eval_batch(rows[:24], nthreads=8), f"load {load}")


@pytest.mark.parametrize("R", [7000, 9217])
def test_a_wavefront_with_nothing_left_to_start_beside_others(R):
    """64 rows that crowd a replica until no slot comes free before it leaves, next to rows that do not: their wavefront only counts
    its requests from then on, stage after stage, while the workgroup's others replay theirs."""
    rng = np.random.default_rng(R)
    M, B = 3, 8
    arrival = np.cumsum(rng.integers(0, 60, R)).astype(np.uint64)
    t_off = [int(arrival[-1]) - 1, int(arrival[R // 2]), traces.UINT64_MAX]
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(M)], t_off_us=t_off, B=B)
    rows = rng.integers(1, M, size=(700, R)).astype(np.uint16)
    rows[64:][:, ::40] = 0
    rows[:64] = np.where(rng.random((64, R)) < 0.9, 0, rows[:64])
    some = np.concatenate([np.arange(0, 64, 5), np.arange(64, 700, 41)])
    with GpuWorkload(tr) as g:
        got = g.eval(rows)
    assert_same(got[some], oracle_for(tr).eval_batch(rows[some], nthreads=8), f"R={R}")


@pytest.mark.parametrize("R", [1024, 5000, 8193])
@pytest.mark.parametrize("B", [12, 64])
def test_queues_that_few_rows_use(R, B):
    """More blocks of candidates than compute units, and most wavefronts of the list replay find tiles, or whole queues, without a
    request among blocks that have some: rows on a few of the replicas, on one for a stretch of the trace, on all."""
    rng = np.random.default_rng(R + B)
    M, C = 130, 700
    arrival = np.cumsum(rng.integers(0, 8, R)).astype(np.uint64)
    t_off = np.where(np.arange(M) % 3 == 1, int(arrival[2 * R // 3]), U64MAX).astype(np.uint64)
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(M)], t_off_us=t_off, B=B)
    rows = rng.integers(0, 9, size=(C, R)).astype(np.uint16)
    rows[70] = np.arange(R) * M // R
    rows[71], rows[C - 1] = M - 1, rng.integers(0, M, R)
    rows[640:650, 3000:] = M
    some = np.unique(np.concatenate([np.arange(0, C, 60), np.arange(69, 73), np.arange(638, 652, 3), [C - 1]]))
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] != 3
        got = g.eval(rows)
    assert_same(got[some], oracle_for(tr).eval_batch(rows[some], nthreads=8), f"R={R} B={B}")


@pytest.mark.parametrize("C", [40, 700])
def test_a_queue_that_closes_early_in_rows_that_need_histograms(C):
    """A crowded replica leaves in the first third of the trace, and so few requests name it that the p99 values come from the
    histograms: its wavefronts have bins to leave at first and nothing to start after that, tile after tile."""
    rng = np.random.default_rng(C)
    R, M, B = 9000, 5, 8
    arrival = np.cumsum(rng.integers(0, 400, R)).astype(np.uint64)
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[m % 3] for m in range(M)],
                             t_off_us=[int(arrival[R // 3])] + [U64MAX] * (M - 1), B=B)
    rows = rng.integers(1, M, size=(C, R)).astype(np.uint16)
    rows[:, R // 4:R // 4 + 60] = 0
    rows[1::2, R // 3 + 100:R // 3 + 120] = 0
    want = oracle_for(tr).eval_batch(rows[:40], nthreads=8)
    assert (want["n_rejected"] > 0).any() and (want["n_rejected"] < R // 100).all()
    with GpuWorkload(tr) as g:
        assert_same(g.eval(rows)[:40], want, f"C={C}")


@pytest.mark.parametrize("M,R", [(1, 3000), (2, 2500), (63, 4000), (64, 4000), (129, 5000), (300, 5000), (513, 3000), (790, 3000), (520, 66000)])
@pytest.mark.parametrize("slow", [False, True])
def test_bins_of_one_long_queue_among_short_ones(M, R, slow):
    """What the merge adds up lies in one queue, in a few, in all of them or in the last, with empty queues before, between and behind;
    one word per request and two, histograms of both widths, more queues than the workgroup has threads."""
    rng = np.random.default_rng(M + R)
    arrival = np.cumsum(rng.integers(0, 3, R)).astype(np.uint64)
    coef = [(3500, 5, 40, 2000) if slow and m == M // 2 else KINDS[m % 3] for m in range(M)]
    longest = 200 if not slow else 60 if R < 60000 else 9                       # all requests one after the other stay below 2^32 us
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, longest, R), coef, B=8)
    rows = rng.integers(0, M, size=(9, R)).astype(np.uint16)
    rows[0], rows[1], rows[2] = M // 2, M - 1, 0
    rows[3] = np.where(rng.random(R) < 0.95, M // 3, rows[3])
    rows[4] = rows[4] // 7 * 7
    rows[5] = np.minimum(M - 1, M // 2 + rows[5] % 3)
    C = 530
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] in (1, 2)
        got = g.eval(np.resize(rows, (C, R)) if R < 60000 else rows)
    assert_same(got[:9], oracle_for(tr).eval_batch(rows, nthreads=8), f"M={M} R={R} slow={slow}")
    assert (got == got[np.arange(len(got)) % 9]).all()


@pytest.mark.parametrize("B", [8, 16, 24, 48, 64])
@pytest.mark.parametrize("count", [1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 1023, 1024])
def test_runs_that_end_anywhere_in_a_block(B, count):
    """A replica's run of a tile has exactly `count` requests, another's the rest: sixteen entries are read ahead, four replayed at a time,
    in every row alike, so that no other lane makes a wavefront go on; odd numbers of tiles."""
    rng = np.random.default_rng(B + count)
    R = 3 * 1024 + min(count, 500)
    tr = traces.custom_trace(np.cumsum(rng.integers(0, 40, R)), rng.integers(1, 4000, R), rng.integers(1, 200, R), [KINDS[0]] * 3, B=B)
    row = np.ones(R, dtype=np.uint16)
    for t in range(0, R, 1024):
        n = min(1024, R - t)
        row[t + rng.permutation(n)[:count]] = 0
    rows = np.repeat(row[None], 70, axis=0)
    with GpuWorkload(tr) as g:
        assert g.route(70)["lists"] == 1
        got = g.eval(rows)
    assert_same(got, np.repeat(oracle_for(tr).eval_batch(rows[:1]), 70), f"B={B} count={count}")


@pytest.mark.parametrize("M,B,C", [(129, 16, 700), (64, 64, 1100), (66, 24, 1537), (31, 48, 2305), (257, 8, 520)])
@pytest.mark.parametrize("slow", [False, True])
def test_equally_long_lists_with_more_workgroups_than_compute_units(M, B, C, slow):
    """As many blocks of candidates times replicas as put the list replay beyond a workgroup per compute unit, with bins in one word and in
    two: every queue of every block is replayed once, in whatever order the workgroups take them, also where replicas, blocks or
    both do not divide evenly; and rows that crowd neighbouring replicas."""
    rng = np.random.default_rng(M + C)
    R = 2049
    assert M * ((C + 255) // 256) > torch.cuda.get_device_properties(0).multi_processor_count
    arrival = np.cumsum(rng.integers(0, 3, R)).astype(np.uint64)
    coef = [(3500, 5, 40, 2000) if slow else KINDS[0]] * M
    tr = traces.custom_trace(arrival, rng.integers(1, 4000, R), rng.integers(1, 60 if slow else 200, R), coef, B=B)
    rows = rng.integers(0, M, size=(C, R)).astype(np.uint16)
    rows[::7] %= max(1, M // 6)
    rows[1], rows[2], rows[C - 1] = 0, np.arange(R) // 8 % M, M - 1
    some = np.unique(np.concatenate([np.arange(4), np.arange(4, C, 97), np.arange(255, 258), np.arange(0, C, 133), np.arange(C - 3, C)]))
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] == 1
        got = g.eval(rows)
    assert_same(got[some], oracle_for(tr).eval_batch(rows[some], nthreads=8), f"M={M} B={B} C={C} slow={slow}")


@pytest.mark.parametrize("B", [13, 16, 17, 23, 24, 25, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("kind", ["equal", "wide", "mostly short", "closing"])
def test_slots_taken_from_the_front(B, kind):
    """The slot times a lane keeps in order are merged with the others when one of the next four starts may not be among them.  A backlog
    that all becomes ready at once, then a trickle, then a burst, with service times that are all alike, that span five orders, or of
    which most end before the slots taken first come free again, so that they are taken from the front over and over; and replicas that
    leave while some lanes still start requests."""
    rng = np.random.default_rng(B)
    R, M, C = 2600, 3, 130
    gap = np.repeat([0, 900, 0, 20_000, 25, 0], [500, 600, 300, 200, 700, 300])
    arrival = np.cumsum(gap + rng.integers(0, 2, R))
    out = {"equal": np.full(R, 40), "wide": np.exp(rng.uniform(0, 11, R)).astype(int) + 1,
           "mostly short": np.where(rng.random(R) < 0.1, 20_000, 1 + rng.integers(0, 3, R)), "closing": rng.integers(1, 400, R)}[kind]
    t_on = [int(arrival[450]), 0, int(arrival[900])]
    t_off = [U64MAX] * 3 if kind != "closing" else [int(arrival[450]) + 60_000, int(arrival[1300]), int(arrival[-1]) + 1]
    tr = traces.custom_trace(arrival, rng.integers(1, 60, R), out, [(5, 1, 3, 2), (0, 0, 1, 1), (2000, 3, 25, 5)], t_on, t_off, B=B)
    rows = rng.integers(0, M, size=(C, R)).astype(np.uint16)
    rows[1], rows[2], rows[3] = 0, 1, 2
    rows[64:80] %= 2
    with GpuWorkload(tr) as g:
        assert g.route(C)["lists"] in (1, 2)
        assert_same(g.eval(rows), oracle_for(tr).eval_batch(rows, nthreads=8), f"B={B} {kind}")


@pytest.mark.parametrize("B", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", ["crowded", "last before", "long first", "stay"])
def test_starts_that_come_too_late_with_few_slots(B, kind):
    """With fewer than four slots a start may be later than every slot time of four requests before: each of the four may wait for the one
    before it.  Replicas that leave while a crowd waits, right after a request becomes ready, after three of the longest services in a row
    that fit exactly or by a microsecond not, and replicas that stay."""
    rng = np.random.default_rng(B)
    R, M, C = 2500, 5, 70
    long = 2000 + 3 * 40 + 25 * 400 + 5 * 400                            # the longest service: 40 tokens in, 400 out
    prompt, out = rng.integers(1, 40, R), rng.integers(1, 40, R)
    arrival = np.cumsum(rng.integers(0, {"crowded": 300, "stay": 300, "last before": 60_000, "long first": 400}[kind], R)).astype(np.uint64)
    prompt[::97], out[::97] = 40, 400
    if kind == "long first":
        prompt[1200:1300], out[1200:1300] = 40, 400
    at = int(arrival[1250])
    t_on = np.array([0, 0, int(arrival[1100]), 0, 0], np.uint64)
    t_off = {"crowded": [int(arrival[2000]), int(arrival[2400]) + 9_000_000, at + 400_000, 30_000_000, U64MAX],
             "last before": [at + 1, at + long, at + 3 * long, at + 3 * long + 1, at + 3 * long - 1],
             "long first": [at + 1, at + long, int(arrival[1100]) + 3 * long, int(arrival[1100]) + 3 * long + 1, at + 40 * long],
             "stay": [U64MAX] * 5}[kind]
    tr = traces.custom_trace(arrival, prompt, out, [(2000, 3, 25, 5)] * 3 + [(1200, 2, 15, 3)] * 2, t_on, np.array(t_off, np.uint64), B=B, penalty_us=10**9)
    rows = rng.integers(0, M, size=(C, R)).astype(np.uint16)
    for m in range(M):
        rows[m] = m
        rows[8 + m, 1150:] = m
    with GpuWorkload(tr) as g:
        assert g.route(600)["lists"] in (1, 2)
        got = g.eval(np.resize(rows, (600, R)))
    assert_same(got[:C], oracle_for(tr).eval_batch(rows, nthreads=8), f"B={B} {kind}")
    assert (got == got[np.arange(600) % C]).all()


@pytest.mark.parametrize("M,R", [(1, 1030), (2, 2048), (40, 1000), (64, 4 * 1024 + 65), (130, 9 * 1024 + 1)])
def test_tiles_that_crowd_a_replica(M, R):
    """A tile whose first requests name one replica often enough has its places, and those of one more replica, counted another way: rows on
    one to five replicas, on one replica and now and then another, with unknown ids in front and in between, tiles that crowd in turn with
    tiles that do not, and replicas that are gone by a tile or in its middle."""
    rng = np.random.default_rng(M + R)
    B = 6
    arrival = np.cumsum(rng.integers(0, 200, R)).astype(np.uint64)
    t_off = np.where(np.arange(M) % 3 == 2, arrival[rng.integers(R // 3, R, M)], traces.UINT64_MAX).astype(np.uint64)
    tr = traces.custom_trace(arrival, rng.integers(1, 800, R), rng.integers(1, 100, R), [(2000, 3, 25, 5)] * M, None, t_off, B=B)
    rows = rng.integers(0, M, size=(40, R)).astype(np.uint16)
    for c in range(20):
        some = rng.choice(M, size=min(M, 1 + c % 5), replace=False)
        rows[c] = rng.choice(some, size=R)
        if c >= 5:                                                       # a share of others, unknown ones among them
            rows[c] = np.where(rng.random(R) < (0.02, 0.3, 0.7)[c % 3], rng.integers(0, M + 2, R), rows[c])
    rows[20:28] = np.where(np.arange(R) // 1024 % 2 == 0, rows[0:8], rows[20:28])
    rows[22, ::1024] = rows[23, :64] = M
    rows[24:28, 32:64] = rows[28:32, 32:64]
    with GpuWorkload(tr) as g:
        assert g.route(600)["lists"] == 1
        got = g.eval(np.resize(rows, (600, R)))
        odd = g.eval(rows[:7])                                           # few rows: eight wavefronts each
    want = oracle_for(tr).eval_batch(rows, nthreads=8)
    assert_same(got[:40], want, f"M={M} R={R}")
    assert (got == got[np.arange(600) % 40]).all()
    assert_same(odd, want[:7], f"M={M} R={R}, few rows")


@pytest.mark.parametrize("bins", [False, True])
@pytest.mark.parametrize("kind", ["comes up late", "one slot", "two slots", "late, two slots"])
@pytest.mark.parametrize("beyond", [-1, 0, 1, 100_000_000, 700_000_000])
def test_latencies_on_either_side_of_a_quarter_of_the_range(kind, beyond, bins):
    """Four latencies are added up in 32 bits where the host's bound on a latency - the latest window's beginning, all service over the
    slots and one service more - is below 2^30 us, and one by one where it is not: bounds one below it, at it, one above and far above, by a
    replica that comes up behind a backlog, by an overload of one or two slots, and by both, with latencies next to the bound.  bins: with and
    without rejected requests that settle the p99 values."""
    rng = np.random.default_rng(abs(beyond))
    R, M = 2304, 3
    bound = (1 << 30) + beyond                                           # what the host compares with 2^30
    B = {"comes up late": 8, "one slot": 1, "two slots": 2, "late, two slots": 2}[kind]
    arrival = np.arange(R, dtype=np.uint64)
    on_replica = {"comes up late": bound - 2_000_000, "one slot": 0, "two slots": 0, "late, two slots": bound // 2}[kind]
    tpot, out = 10, 20
    service = (bound - on_replica) * B // (R + B)                        # of each request, and a microsecond more for some of them
    extra = np.zeros(R, int)
    while on_replica + (service * R + int(extra.sum())) // B + service + int(extra.max()) < bound:
        extra[int(extra.argmin())] += 1
    assert on_replica + (service * R + int(extra.sum())) // B + service + int(extra.max()) == bound
    t_on = np.array([0, 0, on_replica], np.uint64)
    t_off = np.array([U64MAX, 5_000_000 if not bins else U64MAX, U64MAX], np.uint64)
    tr = traces.custom_trace(arrival, 1 + extra, np.full(R, out), [(service - tpot * out - 1, 1, tpot, 0)] * M, t_on, t_off, B=B,
                             penalty_us=(1 << 32) - 1 if bins else 1 << 40)
    rows = rng.integers(0, M, size=(70, R)).astype(np.uint16)
    rows[0] = rows[1] = 2
    rows[1, ::3] = M
    rows[2, :40] = 1
    rows[3] = 0
    want = oracle_for(tr).eval_batch(rows, nthreads=8)
    if beyond > 1:
        assert int(want["p99_e2e_us"][0]) > (1 << 30)                    # one request in a hundred: four in a row do not fit 32 bits
    with GpuWorkload(tr) as g:
        assert g.route(600)["lists"] in (1, 2)
        got = g.eval(np.resize(rows, (600, R)))
    assert_same(got[:70], want, f"{kind} {beyond}")
    assert (got == got[np.arange(600) % 70]).all()
