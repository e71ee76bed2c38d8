// Candidate-assignment evaluator for MI355X (gfx950): kernels and C ABI.
//
// One workgroup scores one candidate at a time.  The trace is walked in time chunks;
// for every chunk the workgroup
//   (1) counts the chunk's requests per replica        (replica histogram, LDS atomics),
//   (2) turns the counts into offsets                  (wavefront exclusive scans),
//   (3) scatters request indices by replica, stably    (rank inside a wavefront by ballots),
//   (4) replays every replica's queue segment, one wavefront per replica: the B
//       slot-free times live one per lane and persist in LDS between chunks,
//   (5) feeds TTFT / TPOT / E2E of every served request into LDS histograms and
//       per-lane sums.
// After the last chunk the histograms give the p99 values and one 64-byte record is
// written.  Grouping by replica in arrival order is the per-instance queue order of
// Section 8.3 (Setup); the B-slot queue is continuous batching with maximum batch size
// b^max (Section 5.3 "Serving simulator"); the reductions are the per-request
// objectives of Appendix "Discussion and Limitation" (adaptability to diverse serving
// objectives).
//
// Time on the device is 32-bit microseconds relative to the first arrival;
// ap_costmodel_set proves that no finish time can overflow before it enables the path.
//
// This file holds the host side: planning, the workload object and the C ABI.  The kernels are in
// ap_counts.hpp and ap_screen.hpp (screening), ap_stream.hpp (replicas that are always there), ap_replay.hpp (fused replay), ap_pipeline.hpp (three-kernel replay) and
// ap_children.hpp (sparse candidates), ap_split.hpp (replicas that differ or come and go: listed and streamed
// part), ap_roofline.hpp (roofline cost tables, trace time) and ap_agentic.hpp (agentic workflows); ap_common.hpp
// has what they share.
#include <cmath>
#include <mutex>

#include "ap_common.hpp"
#include "ap_screen.hpp"
#include "ap_counts.hpp"
#include "ap_replay.hpp"
#include "ap_pipeline.hpp"
#include "ap_children.hpp"
#include "ap_split.hpp"
#include "ap_stream.hpp"
#include "ap_roofline.hpp"
#include "ap_agentic.hpp"

namespace {

// ----------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------
inline uint32_t align_up(uint32_t v, uint32_t a) { return (v + a - 1u) / a * a; }

// LDS layout for a given chunk size; returns total bytes.
uint32_t plan_lds(EvalParams& p, uint32_t chunk, bool hist16, bool len16) {
    uint32_t off = 3u * kBins * (hist16 ? 2u : 4u);
    p.off_slots = off;  off += align_up(p.M * p.B * 4u, 16u);
    p.off_sorted = off; off += align_up(p.M * 4u, 16u);
    p.off_close = off;  off += align_up((p.M + 1u) * 4u, 16u);
    p.off_cnt = off;    off += align_up(kWaves * (p.M + 1u) * 4u, 16u);
    p.off_qstart = off; off += align_up((p.M + 2u) * 4u, 16u);
    p.off_list = off;   off += align_up(chunk * 2u, 16u);
    p.off_arr = off;    off += chunk * 4u;
    p.off_prompt = off; off += align_up(chunk * (len16 ? 2u : 4u), 16u);
    p.off_out = off;    off += align_up(chunk * (len16 ? 2u : 4u), 16u);
    p.off_misc = off;   off += 64u + 3u * kWaves * 4u;
    p.chunk = chunk;
    return off;
}

using EvalKernel = void (*)(EvalParams, const uint16_t*, ap_metrics*, uint32_t, uint32_t, PendingWord);

EvalKernel eval_kernel(bool hist16, bool len16, bool tabled) {
    static const EvalKernel variants[8] = {
        k_eval_candidates<false, false, false>, k_eval_candidates<true, false, false>,
        k_eval_candidates<false, true, false>,  k_eval_candidates<true, true, false>,
        k_eval_candidates<false, false, true>,  k_eval_candidates<true, false, true>,
        k_eval_candidates<false, true, true>,   k_eval_candidates<true, true, true>};
    return variants[(hist16 ? 1 : 0) + (len16 ? 2 : 0) + (tabled ? 4 : 0)];
}

}  // namespace

constexpr size_t kNominalSumsBytes = 3u * kBins * sizeof(uint32_t) + 3u * sizeof(unsigned long long) + 4u * sizeof(uint32_t);

namespace {
// Every failed device call ends here: HIP keeps the error of a failed call until somebody reads it, and the next,
// unrelated call must not find it.
ap_status device_error() {
    (void)hipGetLastError();
    return AP_ERR_DEVICE;
}

// Device buffers of one roofline computation; freed when the object goes out of scope.
struct RoofBuffers {
    RoofGroup* groups = nullptr;
    unsigned long long* prefill_ns = nullptr;
    unsigned long long* step_ns = nullptr;
    unsigned long long* prefix_ns = nullptr;
    double* weight_bytes = nullptr;
    uint32_t* feasible = nullptr;
    uint32_t* prefill_us = nullptr;
    uint32_t* tpot_us = nullptr;
    uint32_t cap_groups = 0, cap_seq = 0;       // what the table buffers hold; a later computation that fits reuses them
    void release() {
        for (void* q : {(void*)groups, (void*)prefill_ns, (void*)step_ns, (void*)prefix_ns, (void*)weight_bytes,
                        (void*)feasible, (void*)prefill_us, (void*)tpot_us})
            if (q) (void)hipFree(q);
        groups = nullptr; prefill_ns = step_ns = prefix_ns = nullptr; weight_bytes = nullptr; feasible = nullptr;
        prefill_us = tpot_us = nullptr;
        cap_groups = cap_seq = 0;
    }
    ~RoofBuffers() { release(); }
};
}  // namespace

// One plan of the listed / streamed evaluation.
struct SplitPlan {
    bool short_chain = false;         // calls of few rows are left to the fused replay
    bool all_within = false;          // no request's prefill or time per token can exceed the objectives
    uint32_t list_waves_most = 0, split_waves_most[2] = {};   // wavefronts of a workgroup that LDS has room for: k_list_candidates, k_split_candidates
                                      //   without and with histograms
    uint32_t off_wave[2] = {};        // where the latter's areas begin
    bool expect_lazy = false;         // stream without histograms first
    uint32_t batch = 0;               // candidates per batch (what the scratch area holds)
    unsigned char* tables = nullptr;  // ranges, kinds, coefficients, queues, order
    size_t tables_bytes = 0;
    size_t o_lists = 0, o_bins = 0, o_desc = 0, o_part = 0, o_hist = 0, o_bin_base = 0, o_bin_count = 0;   // where its parts lie in the scratch area
    SplitParams params{};
};

struct ap_workload {
    int device = 0;
    uint32_t R = 0;
    uint64_t base_us = 0;             // first arrival
    uint64_t span_us = 0;             // last arrival - first arrival
    std::vector<int32_t> h_prompt, h_out;
    std::vector<uint32_t> h_arrival;  // relative to base_us (clamped; a span beyond 32 bits is refused anyway)
    uint32_t* d_arrival = nullptr;
    uint32_t* d_prompt = nullptr;
    uint32_t* d_out = nullptr;
    DevReplica* d_rep = nullptr;      // capacity AP_MAX_REPLICAS
    uint32_t* d_tab_prefill = nullptr;  // [T][R] cost tables (ap_costtable_set), kept for the largest T seen
    uint32_t* d_tab_tpot = nullptr;
    size_t tab_entries = 0;
    bool tabled = false;              // the current cost model reads the tables
    RoofBuffers* roof = nullptr;             // device buffers of ap_costtable_set_roofline, kept for the next call
    unsigned char* d_bounds = nullptr;       // TableBounds, then the replica types in use [AP_MAX_REPLICAS]
    uint32_t* d_span = nullptr;       // [R] contention-free service intervals in ticks, valid when screen is set
    uint32_t* d_span_t = nullptr;     // the same, lane-major for the one-wavefront screening kernel
    uint32_t* d_pair = nullptr;       // one word per two requests (eight-wavefront screening kernel, when it fits)
    bool screen_packed = false;       // that kernel reads d_pair instead of d_span
    ap_metrics* d_nominal = nullptr;  // record shared by all contention-free candidates
    unsigned char* d_nominal_sums = nullptr;   // k_nominal_metrics: three histograms of 32-bit counts, then its sums and counters
    uint32_t* d_pending = nullptr;    // [2] "this call has left pending marks", taken in turn by the calls; [2] = candidates replayed;
                                      //   [3]: those the fused replay scored in place of the lists
    mutable uint32_t turn = 0;        // which of the two the next call uses
    mutable uint64_t n_scored = 0;    // candidates scored since the cost model was set
    bool has_model = false;
    bool screen = false;              // homogeneous, always-on replicas: screening applies
    bool hist16 = false;              // R < 65536: 16-bit histogram counters
    bool len16 = false;               // every prompt and output length < 65536: 16-bit staging
    EvalParams params{};
    ScreenParams screen_params{};
    uint32_t lds_bytes = 0;
    uint32_t screen_lds_bytes = 0;
    uint32_t* d_count_lo = nullptr;   // counting screen: first bucket of every bucket's window
    bool counts = false;              // the counting screen runs in front of the slot rings
    CountParams count_params{};
    bool screen_wide = false;         // eight wavefronts per candidate (large replica tables)
    uint32_t screen_wide_lds_bytes = 0;
    uint32_t max_grid = 0;
    uint32_t resident_grid = 0;       // workgroups of the replay kernel behind a screen: a multiple of what the device holds at once
    uint32_t n_cu = 0;
    // three-kernel replay: request records, scratch for one batch of candidates, launch parameters
    uint4* d_req = nullptr;           // [R] {arrival, prompt_len, out_len, 0}
    unsigned char* d_scratch = nullptr;
    size_t scratch_bytes = 0;
    uint32_t batch = 0;               // candidates per batch
    GroupParams group_params{};
    ReplayParams replay_params{};
    ReduceParams reduce_params{};
    EvalParams reduce_eval{};
    uint32_t group_lds_bytes = 0, replay_lds_bytes = 0, reduce_lds_bytes = 0;
    bool small_table = false;         // identical replicas, but too few and too small for the slot rings
    bool pipeline = false;
    // sparse candidates (ap_parent_set / ap_eval_children)
    uint16_t* d_parent = nullptr;     // [R]
    uint32_t* d_peak = nullptr;       // [AP_MAX_REPLICAS + 1] depth of the parent per replica, then its unknown ids
    uint32_t* d_room = nullptr;       // [AP_MAX_REPLICAS]
    unsigned char* h_stage = nullptr; // pinned: the parent row on its way in, then the depths on their way out
    uint16_t* d_rows = nullptr;       // [max_children][R]
    size_t rows_bytes = 0;
    uint32_t max_children = 0;
    bool has_parent = false;
    ChildParams child_params{};
    // streamed evaluation (replicas always there, nobody expected to wait): its own tables, one allocation
    bool stream = false;
    bool stream_settles = false;      // nobody can wait: it leaves nothing behind
    uint32_t* d_stream_tab = nullptr;
    size_t stream_tab_bytes = 0;
    StreamParams stream_params{};
    uint32_t stream_lds_bytes = 0;
    // split evaluation (replicas that differ or have windows): listed part replayed, streamed part scored on arrival
    uint2* d_req8 = nullptr;          // [R] {arrival, prompt | out << 16}; only when every length is below 65536
    uint2* d_tab_pair = nullptr;      // [T][R] the cost tables side by side, for the split evaluation of a tabulated model
    size_t tab_pair_entries = 0;
    unsigned char* d_split_scratch = nullptr;
    size_t split_scratch_bytes = 0;
    bool split = false;               // the split evaluation runs in front of the general replay
    SplitPlan split_plan{};
};

// Wavefronts of a kernel that the registers of a SIMD hold at once.
static uint32_t waves_by_registers(const hipFuncAttributes& attr) {
    return std::min(8u, 512u / align_up((uint32_t)std::max(attr.numRegs, 1), 8u));
}

// Do a kernel's dynamic tables begin at LDS address 0?  k_stream_candidates and k_split_candidates read their first table by address, and
// whatever a kernel declares itself (__shared__) would come before it.
static bool tables_at_lds_zero(const void* kernel) {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, kernel) == hipSuccess && attr.sharedSizeBytes == 0u;
}

typedef void (*stream_fn)(StreamParams, const uint16_t*, ap_metrics*, uint32_t, PendingWord);
static stream_fn stream_kernel(bool settles, bool tabled) {
    return settles ? (tabled ? k_stream_candidates<true, false> : k_stream_candidates<false, false>)
                   : (tabled ? k_stream_candidates<true, true> : k_stream_candidates<false, true>);
}

typedef void (*split_fn)(SplitParams, const uint16_t*, uint32_t, uint32_t, uint32_t, PendingWord);
static split_fn split_kernel(uint32_t hist_mode, bool tabled, bool within) {
    static const split_fn variants[12] = {
        k_split_candidates<0u, false, false>, k_split_candidates<1u, false, false>, k_split_candidates<2u, false, false>,
        k_split_candidates<0u, true, false>,  k_split_candidates<1u, true, false>,  k_split_candidates<2u, true, false>,
        k_split_candidates<0u, false, true>,  k_split_candidates<1u, false, true>,  k_split_candidates<2u, false, true>,
        k_split_candidates<0u, true, true>,   k_split_candidates<1u, true, true>,   k_split_candidates<2u, true, true>};
    return variants[hist_mode + (tabled ? 3u : 0u) + (within ? 6u : 0u)];
}

typedef void (*replay_lists_fn)(SplitParams, uint32_t, uint32_t);
template <uint32_t kBins_, bool kFew>
static replay_lists_fn replay_lists_kernel_of(uint32_t B) {
    return B < 4u ? k_replay_lists<4u, kBins_, kFew> : B <= 8u ? k_replay_lists<8u, kBins_, kFew> : B <= 12u ? k_replay_lists<12u, kBins_, kFew> : B <= 16u ? k_replay_lists<16u, kBins_, kFew>
           : B <= 24u ? k_replay_lists<24u, kBins_, kFew> : B <= 32u ? k_replay_lists<32u, kBins_, kFew>
           : B <= 48u ? k_replay_lists<48u, kBins_, kFew> : k_replay_lists<64u, kBins_, kFew>;
}

// The dense path on C rows: screening where it applies, then the exact replay of what is left.
// marked: only rows whose record carries the pending mark are looked at (screening applies).
static PendingWord take_pending_word(const ap_workload* w) {
    const uint32_t t = w->turn;
    w->turn = t ^ 1u;
    return PendingWord{w->d_pending + t, w->d_pending + (t ^ 1u)};
}

// The counting screen is one launch more in front of the rings, 2 us, which calls of 12 to 30 us do not get back.  It pays from
// about 2^25 requests, and on long rows, which are a chain of blocks of 512 or 1024 requests for the rings.  Even rows, without
// and with it: of 4096 requests on 45 replicas 19 and 21 us at 2^24 requests, 29 and 28 at 2^25, 49 and 44 at 2^26; of 16384 on
// 128 replicas 15.1 and 16.5, 24 and 20, 40 and 30; of 32768 on 128, 16.6 and 16.4 at 2^24, 14 and 11 at 2^16.
static bool counts_first(const ap_workload* w, uint32_t C) { return w->counts && (w->R >= 32768u || (uint64_t)C * w->R >= (1u << 25)); }

// Wavefronts per row of the counting screen: several while there are fewer rows than the chip holds wavefronts (8192 at eight per
// SIMD), as long as a wavefront's share stays at least four steps and at least as long as what it has to count again before it.
static uint32_t count_waves_per_row(const ap_workload* w, uint32_t C) {
    const CountParams& p = w->count_params;
    const uint32_t step = p.w_log2 >= 9u ? 512u : 128u, again = (p.ring_mask + 1u) << p.w_log2;
    uint32_t per_row = 1u;
    while (per_row < kCountMaxWaves && (uint64_t)C * per_row * 2u <= (uint64_t)w->n_cu * 32u &&
           w->R / (per_row * 2u) >= std::max(4u * step, again / 2u) &&
           std::max(4u, per_row * 2u) * p.wave_words * 4u <= kCountLdsBytes)
        per_row *= 2u;
    return per_row;
}

// Calls of few rows that go to the fused replay in place of the lists: up to two rows per compute unit with up to 64 replicas, one
// with more, whose slots leave room for one workgroup or slow two down (even rows of 800 requests on replicas that come and go, lists and
// fused replay: 512 rows on 64 replicas 36 and 29 us, on 128 34 and 37, 256 rows there 32 and 30).  A wavefront works through the queues of
// many replicas one after the other, while the launches of the lists cost the same for any number: beyond 128 replicas one row is better
// off with lists (200 requests on 500 replicas: one row 27 and 30, 4 rows 32 and 31; 800 on 500: 39 and 46, 52 and 46).
static bool fused_replay(const ap_workload* w, uint32_t C) {
    const uint32_t M = w->params.M;
    return w->split && w->split_plan.short_chain && C <= (M <= 64u ? 2u : 1u) * w->n_cu && (M <= 128u || C >= 4u);
}

// The counting screen on C rows.
static ap_status launch_counts(const ap_workload* w, const uint16_t* d_assign, uint32_t C, ap_metrics* d_out, hipStream_t stream,
                               PendingWord flags) {
    typedef void (*count_fn)(CountParams, const uint16_t*, ap_metrics*, uint32_t, PendingWord);
    CountParams p = w->count_params;
    const bool quad = p.w_log2 >= 9u;                        // buckets of 512 requests or more: 16-byte loads
    static const count_fn variants[6] = {k_screen_counts<1u, 2u>, k_screen_counts<1u, 3u>, k_screen_counts<1u, 4u>,
                                         k_screen_counts<4u, 2u>, k_screen_counts<4u, 3u>, k_screen_counts<4u, 4u>};
    const count_fn kernel = variants[p.columns_log2 - 2u + (quad ? 3u : 0u)];
    const uint32_t per_row = count_waves_per_row(w, C);
    p.waves_per_row = per_row;
    const uint32_t waves = std::max(4u, per_row);
    const uint32_t grid = (C + waves / per_row - 1u) / (waves / per_row);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * kWave), waves * p.wave_words * 4u, stream, p, d_assign, d_out, C, flags);
    return hipGetLastError() == hipSuccess ? AP_OK : device_error();
}

// Histograms and accumulators, and behind them two words per queue.
static uint32_t merge_lds_bytes(const ap_workload* w, const SplitParams& sp) { return w->reduce_lds_bytes + 8u * sp.n_queues; }

// The listed / streamed evaluation, a batch of candidates at a time; what it hands back carries the pending mark.
// pending: only candidates that carry the pending mark already (behind the streamed evaluation).
static ap_status launch_split(const ap_workload* w, const SplitPlan& plan, const uint16_t* d_assign, uint32_t C, ap_metrics* d_out,
                              hipStream_t stream, PendingWord flags, bool pending) {
    SplitParams sp = plan.params;
    sp.lists = reinterpret_cast<uint16_t*>(w->d_split_scratch + plan.o_lists);
    sp.bins = w->d_split_scratch + plan.o_bins;
    sp.desc = reinterpret_cast<uint32_t*>(w->d_split_scratch + plan.o_desc);
    sp.part = reinterpret_cast<SplitPartial*>(w->d_split_scratch + plan.o_part);
    sp.hist = reinterpret_cast<uint32_t*>(w->d_split_scratch + plan.o_hist);
    sp.bin_base = reinterpret_cast<uint32_t*>(w->d_split_scratch + plan.o_bin_base);
    sp.bin_count = reinterpret_cast<uint32_t*>(w->d_split_scratch + plan.o_bin_count);
    const replay_lists_fn replay_lean = replay_lists_kernel_of<0u, false>(sp.B);
    // batches of equal size (whole wavefronts of the list replay), none above what the scratch area holds
    const uint32_t n_batches = (C + plan.batch - 1u) / plan.batch;
    const uint32_t per_batch = std::min(plan.batch, ((C + n_batches - 1u) / n_batches + 63u) / 64u * 64u);
    for (uint32_t c0 = 0; c0 < C; c0 += per_batch) {
        const uint32_t n = std::min(per_batch, C - c0);
        if (pending) {
            sp.pending = d_out + c0;
            sp.pending_word = flags.mine;
        }
        const uint32_t grid = std::min(n, w->n_cu * 16u);
        // Where something is streamed: first without histograms if the candidates are expected to be settled by penalty; then
        // with histograms, for every candidate or for those the first pass marked.
        const bool plain_first = plan.expect_lazy;
        // A workgroup per row: four wavefronts, or eight where rows leave the chip less than two per SIMD (300 rows of 20001 requests on 61
        // replicas 1.2 to 1.3 times less time).  Not more beyond: LDS is what they wait for, and a row's tiles take as many turns
        // with five wavefronts as with four (1024 rows of 131072 on 128, 172 us with four, 179 with six; 700 rows of 16384 on 64, 52 and 63 with five).
        auto waves_of = [&](uint32_t most) { return n <= 2u * w->n_cu ? std::max(kBuildMinWaves, std::min(most, sp.n_tiles)) : kBuildMinWaves; };
        auto launch_split_kernel = [&](uint32_t hist_mode, uint32_t blocks, uint32_t only_flagged) {
            const uint32_t h = hist_mode != 0u ? 1u : 0u, waves = waves_of(plan.split_waves_most[h]);
            sp.off_wave = plan.off_wave[h];
            hipLaunchKernelGGL(split_kernel(hist_mode, w->tabled, plan.all_within), dim3(blocks), dim3(waves * kWave),
                               sp.off_wave + waves * sp.wave_bytes, stream, sp, d_assign, c0, n, only_flagged, flags);
        };
        if (sp.any_streamed == 0u) {
            const uint32_t waves = waves_of(plan.list_waves_most);
            hipLaunchKernelGGL(k_list_candidates, dim3(grid), dim3(waves * kWave), sp.l_wave + waves * sp.l_wave_bytes, stream, sp, d_assign, c0, n, flags);
        } else {
            if (plain_first) launch_split_kernel(0u, grid, 0u);
            // (behind a plain pass: usually nothing to do, so few workgroups)
            launch_split_kernel(sp.wide ? 2u : 1u, plain_first ? std::min(n, w->n_cu * 3u) : grid, plain_first ? 1u : 0u);
        }
        // the list replay: where most candidates are settled by penalty, those go through the variant that leaves no bins, and
        // the wavefronts of the other variant find the few that remain
        if (sp.n_queues != 0u) {
            const uint32_t blocks = (n + kReplayListThreads - 1u) / kReplayListThreads;
            const uint32_t groups = sp.even_lists != 0u ? align_up((sp.n_queues + kNeighbours - 1u) / kNeighbours * blocks, kXcds) * kNeighbours
                                                        : sp.n_queues * blocks;
            const bool lean = plan.expect_lazy;
            const bool few = sp.n_queues * blocks <= w->n_cu;
            const replay_lists_fn replay_bins = sp.wide_bins ? (few ? replay_lists_kernel_of<2u, true>(sp.B) : replay_lists_kernel_of<2u, false>(sp.B))
                                                             : (few ? replay_lists_kernel_of<1u, true>(sp.B) : replay_lists_kernel_of<1u, false>(sp.B));
            if (lean) hipLaunchKernelGGL(replay_lean, dim3(groups), dim3(kReplayListThreads), 0, stream, sp, n, 1u);
            hipLaunchKernelGGL(replay_bins, dim3(groups), dim3(kReplayListThreads), 0, stream, sp, n, lean ? 2u : 0u);
        }
        hipLaunchKernelGGL(sp.wide ? k_merge_candidates<false> : k_merge_candidates<true>, dim3(std::min(n, w->n_cu * 8u)),
                           dim3(kThreads), merge_lds_bytes(w, sp), stream, w->reduce_eval, sp, d_out, c0, n, flags);
    }
    return hipGetLastError() == hipSuccess ? AP_OK : device_error();
}

static ap_status launch_stream(const ap_workload* w, const uint16_t* d_assign, uint32_t C, ap_metrics* d_out, hipStream_t stream,
                               PendingWord flags) {
    // A workgroup per row: four wavefronts, or more where rows are fewer than the chip holds wavefronts and long enough that
    // each still has four steps.
    uint32_t waves = 4u;
    while (waves < kStreamMaxThreads / kWave && (uint64_t)C * waves * 2u <= (uint64_t)w->n_cu * 32u && w->R / 128u >= 8u * waves) waves *= 2u;
    const uint32_t grid = std::min(C, w->n_cu * 64u);
    hipLaunchKernelGGL(stream_kernel(w->stream_settles, w->tabled), dim3(grid), dim3(waves * kWave),
                       w->stream_lds_bytes + waves * kStreamLargeBytes, stream, w->stream_params, d_assign, d_out, C, flags);
    return hipGetLastError() == hipSuccess ? AP_OK : device_error();
}

static ap_status launch_dense(const ap_workload* w, const uint16_t* d_assign, uint32_t C, ap_metrics* d_out,
                              hipStream_t stream, bool marked, PendingWord flags) {
    if (!marked && counts_first(w, C)) {
        const ap_status st = launch_counts(w, d_assign, C, d_out, stream, flags);
        if (st != AP_OK) return st;
        marked = true;                                       // the rings look at what it has left
    }
    if (w->screen) {
        const uint32_t blocks = std::min((C + kScreenWaves - 1u) / kScreenWaves, w->n_cu * 64u);
        // rows start on 4-byte boundaries when R is even and the batch itself does
        const bool aligned = (w->R % 2u == 0u) && (reinterpret_cast<uintptr_t>(d_assign) % 4u == 0u);
        typedef void (*screen_fn)(ScreenParams, const uint16_t*, ap_metrics*, uint32_t, PendingWord);
        if (w->screen_wide) {
            static const screen_fn wide[8] = {
                k_screen_candidates_wide<false, false, false>, k_screen_candidates_wide<true, false, false>,
                k_screen_candidates_wide<false, true, false>,  k_screen_candidates_wide<true, true, false>,
                k_screen_candidates_wide<false, false, true>,  k_screen_candidates_wide<true, false, true>,
                k_screen_candidates_wide<false, true, true>,   k_screen_candidates_wide<true, true, true>};
            // one candidate per workgroup while the grid stays moderate: workgroups finish at different
            // times, and the hardware's queue of waiting workgroups balances that better than fixed shares
            // marked: runs of candidates per workgroup (at most one per thread), few workgroups
            const uint32_t grid = marked ? std::max((C + kWideThreads - 1u) / kWideThreads, std::min(C, w->n_cu * 4u))
                                         : std::min(C, w->n_cu * 64u);
            hipLaunchKernelGGL(wide[(aligned ? 1 : 0) + (w->screen_packed ? 2 : 0) + (marked ? 4 : 0)], dim3(grid),
                               dim3(kWideThreads), w->screen_wide_lds_bytes, stream, w->screen_params, d_assign, d_out, C, flags);
        } else {
            static const screen_fn narrow[4] = {k_screen_candidates<false, false>, k_screen_candidates<true, false>,
                                                k_screen_candidates<false, true>, k_screen_candidates<true, true>};
            const uint32_t grid = marked ? std::max((C + kScreenThreads - 1u) / kScreenThreads, std::min(blocks, w->n_cu * 8u))
                                         : blocks;
            hipLaunchKernelGGL(narrow[(aligned ? 1 : 0) + (marked ? 2 : 0)], dim3(grid), dim3(kScreenThreads),
                               w->screen_lds_bytes, stream, w->screen_params, d_assign, d_out, C, flags);
        }
        if (hipGetLastError() != hipSuccess) return device_error();
    }
    const bool fused = !marked && fused_replay(w, C);
    bool split_behind = false;
    if (w->stream && !marked) {
        const ap_status st = launch_stream(w, d_assign, C, d_out, stream, flags);
        if (st != AP_OK || w->stream_settles) return st;
        split_behind = true;
    }
    if (w->split && !marked && !fused) {
        const ap_status st = launch_split(w, w->split_plan, d_assign, C, d_out, stream, flags, split_behind);
        if (st != AP_OK) return st;
        if (w->split_plan.params.any_streamed == 0u) return AP_OK;                   // with every request listed nothing is handed back
    }
    const uint32_t pending_only = (w->screen || split_behind || (w->split && !marked && !fused)) ? 1u : 0u;
    if (w->pipeline) {
        for (uint32_t c0 = 0; c0 < C; c0 += w->batch) {
            const uint32_t n = std::min(w->batch, C - c0);
            hipLaunchKernelGGL(k_group_requests, dim3(n), dim3(kGroupThreads), w->group_lds_bytes, stream, w->group_params,
                               d_assign, d_out, c0, n, pending_only);
            const uint32_t n_wg = (n * w->params.M + kReplayThreads - 1u) / kReplayThreads;
            hipLaunchKernelGGL(k_replay_queues, dim3(n_wg), dim3(kReplayThreads), w->replay_lds_bytes, stream,
                               w->replay_params, d_out, c0, n, pending_only);
            hipLaunchKernelGGL(w->hist16 ? k_reduce_candidates<true> : k_reduce_candidates<false>, dim3(n), dim3(kThreads),
                               w->reduce_lds_bytes, stream, w->reduce_eval, w->reduce_params, d_out, c0, n, pending_only);
        }
        if (hipGetLastError() != hipSuccess) return device_error();
        return AP_OK;
    }
    // After screening, most workgroups only find out that nothing is left for them: as many as can be
    // resident at once look at all the records together.
    const uint32_t grid = std::min(C, pending_only ? w->resident_grid : w->max_grid);
    EvalParams p = w->params;
    if (fused) p.replayed = w->d_pending + 3;                // in place of the lists: not what ap_eval_counts_get reports
    hipLaunchKernelGGL(eval_kernel(w->hist16, w->len16, w->tabled), dim3(grid), dim3(kThreads), w->lds_bytes, stream, p, d_assign, d_out, C,
                       pending_only, flags);
    if (hipGetLastError() != hipSuccess) return device_error();
    return AP_OK;
}

extern "C" {

const char* ap_status_str(ap_status s) {
    switch (s) {
        case AP_OK: return "ok";
        case AP_ERR_INVALID: return "invalid argument";
        case AP_ERR_RANGE: return "capacity of the device path exceeded";
        case AP_ERR_ALLOC: return "allocation failed";
        case AP_ERR_DEVICE: return "HIP call failed";
        case AP_ERR_STATE: return "no cost model (or, for children, no parent) set";
    }
    return "unknown status";
}

uint32_t ap_hist_bin(uint64_t v) {
    if (v < 128u) return (uint32_t)v;
    uint32_t e = 0;
    for (uint64_t t = v; t > 1u; t >>= 1) ++e;         // floor(log2 v)
    if (e > 37u) return kBins - 1u;
    return ((e - 6u) << 7) | (uint32_t)((v >> (e - 7u)) & 127u);
}

uint64_t ap_hist_lower(uint32_t bin) {
    if (bin < 128u) return bin;
    return (uint64_t)(128u | (bin & 127u)) << ((bin >> 7) - 1u);
}

ap_status ap_workload_create(const uint64_t* arrival_us, const int32_t* prompt_len, const int32_t* out_len,
                             uint32_t R, ap_workload** out) {
    if (!arrival_us || !prompt_len || !out_len || !out || R == 0) return AP_ERR_INVALID;
    for (uint32_t r = 0; r < R; ++r) {
        if (prompt_len[r] < 1 || out_len[r] < 1) return AP_ERR_INVALID;
        if (r && arrival_us[r] < arrival_us[r - 1]) return AP_ERR_INVALID;
    }
    ap_workload* w = new (std::nothrow) ap_workload;
    if (!w) return AP_ERR_ALLOC;
    std::vector<uint32_t> rel;
    try {
        w->h_prompt.assign(prompt_len, prompt_len + R);
        w->h_out.assign(out_len, out_len + R);
        rel.resize(R);
    } catch (const std::bad_alloc&) {
        delete w;
        return AP_ERR_ALLOC;
    }
    w->R = R;
    w->len16 = true;
    for (uint32_t r = 0; r < R; ++r) w->len16 = w->len16 && prompt_len[r] < 65536 && out_len[r] < 65536;
    w->base_us = arrival_us[0];
    w->span_us = arrival_us[R - 1] - arrival_us[0];
    // relative 32-bit arrivals; a span that does not fit is refused later by ap_costmodel_set
    for (uint32_t r = 0; r < R; ++r) rel[r] = (uint32_t)std::min<uint64_t>(arrival_us[r] - w->base_us, kNever);
    w->h_arrival = rel;

    ap_status st = AP_OK;
    if (hipGetDevice(&w->device) != hipSuccess) st = AP_ERR_DEVICE;
    const size_t bytes = (size_t)R * 4u;
    const size_t padded = ((size_t)R + kScreenBlock - 1u) / kScreenBlock * kScreenBlock * 4u;
    if (st == AP_OK && (hipMalloc(&w->d_arrival, bytes) != hipSuccess || hipMalloc(&w->d_prompt, bytes) != hipSuccess ||
                        hipMalloc(&w->d_out, bytes) != hipSuccess ||
                        hipMalloc(&w->d_rep, sizeof(DevReplica) * AP_MAX_REPLICAS) != hipSuccess ||
                        hipMalloc(&w->d_span, bytes) != hipSuccess ||
                        hipMalloc(&w->d_span_t, padded) != hipSuccess ||
                        hipMalloc(&w->d_pair, ((size_t)R + 1u) / 2u * 4u) != hipSuccess ||
                        hipMalloc(&w->d_count_lo, ((size_t)R + kCountShift + kCountMinBucket) / kCountMinBucket * 4u) != hipSuccess ||
                        hipMalloc(&w->d_nominal, sizeof(ap_metrics)) != hipSuccess ||
                        hipMalloc(&w->d_nominal_sums, kNominalSumsBytes) != hipSuccess ||
                        hipMalloc(&w->d_pending, 4u * sizeof(uint32_t)) != hipSuccess))
        st = AP_ERR_ALLOC;
    if (st == AP_OK && hipMemset(w->d_pending, 0, 4u * sizeof(uint32_t)) != hipSuccess) st = AP_ERR_DEVICE;
    std::vector<uint4> recs;
    if (st == AP_OK) {
        try {
            recs.resize(R);
        } catch (const std::bad_alloc&) {
            st = AP_ERR_ALLOC;
        }
    }
    if (st == AP_OK) {
        for (uint32_t r = 0; r < R; ++r) recs[r] = make_uint4(rel[r], (uint32_t)prompt_len[r], (uint32_t)out_len[r], 0u);
        if (hipMalloc(&w->d_req, sizeof(uint4) * (size_t)R) != hipSuccess) st = AP_ERR_ALLOC;
        else if (hipMemcpy(w->d_req, recs.data(), sizeof(uint4) * (size_t)R, hipMemcpyHostToDevice) != hipSuccess)
            st = AP_ERR_DEVICE;
    }
    if (st == AP_OK && w->len16) {
        // arrival and both lengths of a request in 8 bytes, for the kernels that read whole records
        std::vector<uint2> packed;
        try {
            packed.assign((size_t)R + 1u, make_uint2(0u, 0u));       // one spare record: pairs of records are read at once
        } catch (const std::bad_alloc&) {
            st = AP_ERR_ALLOC;
        }
        if (st == AP_OK) {
            for (uint32_t r = 0; r < R; ++r) packed[r] = make_uint2(rel[r], (uint32_t)prompt_len[r] | ((uint32_t)out_len[r] << 16));
            if (hipMalloc(&w->d_req8, sizeof(uint2) * ((size_t)R + 1u)) != hipSuccess) st = AP_ERR_ALLOC;
            else if (hipMemcpy(w->d_req8, packed.data(), sizeof(uint2) * ((size_t)R + 1u), hipMemcpyHostToDevice) != hipSuccess)
                st = AP_ERR_DEVICE;
        }
    }
    if (st == AP_OK && (hipMemcpy(w->d_arrival, rel.data(), bytes, hipMemcpyHostToDevice) != hipSuccess ||
                        hipMemcpy(w->d_prompt, prompt_len, bytes, hipMemcpyHostToDevice) != hipSuccess ||
                        hipMemcpy(w->d_out, out_len, bytes, hipMemcpyHostToDevice) != hipSuccess))
        st = AP_ERR_DEVICE;
    if (st != AP_OK) {
        (void)hipGetLastError();
        ap_workload_destroy(w);
        return st;
    }
    *out = w;
    return AP_OK;
}

// The cost tables side by side for the evaluations that read them in pairs, rows up to the highest type in use.
// ready: false where there is no room for them (the general replay scores the calls then).
static ap_status pair_tables(ap_workload* w, const uint32_t* rep_type, uint32_t M, bool& ready) {
    ready = false;
    size_t entries = 0;
    for (uint32_t m = 0; m < M; ++m) entries = std::max(entries, ((size_t)rep_type[m] + 1u) * w->R);
    if (entries > w->tab_pair_entries) {
        if (w->d_tab_pair && hipFree(w->d_tab_pair) != hipSuccess) return device_error();
        w->d_tab_pair = nullptr;
        w->tab_pair_entries = 0;
        if (hipMalloc(&w->d_tab_pair, entries * sizeof(uint2)) != hipSuccess) {
            (void)hipGetLastError();
            return AP_OK;
        }
        w->tab_pair_entries = entries;
    }
    hipLaunchKernelGGL(k_pair_tables, dim3((uint32_t)std::min<size_t>(4096u, (entries + kThreads - 1u) / kThreads)), dim3(kThreads), 0,
                       nullptr, w->d_tab_prefill, w->d_tab_tpot, w->d_tab_pair, entries);
    if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) return device_error();
    ready = true;
    return AP_OK;
}

// For every multiple k of `grain`: the first request still in service, nobody waiting, when request k * grain - shift (0 if
// that is negative) arrives.  It only moves forward.
static std::vector<uint32_t> first_in_service(const ap_workload* w, const std::vector<uint32_t>& worst_service, uint32_t grain,
                                              uint32_t shift) {
    std::vector<uint32_t> first((w->R + shift) / grain + 1u);
    const uint32_t* arr = w->h_arrival.data();
    for (uint32_t k = 0, q = 0; k < first.size(); ++k) {
        const uint32_t i = std::min(w->R - 1u, k * grain < shift ? 0u : k * grain - shift);
        while (q < i && (uint64_t)arr[q] + worst_service[q] <= arr[i]) ++q;
        first[k] = q;
    }
    return first;
}

// Is a row that is spread evenly over the replicas all but sure to have at most B requests per replica in every one of
// n_windows windows of `window` requests?  Chernoff's bound on a Poisson count: one chance in 10^7 per row.  Behind the streamed
// evaluation a single row that fails makes its call wait for the serial replay of the row's queues; behind the counting screen
// it is a pass of the rings over one row, and the line was not tried elsewhere there.
static bool windows_fit(double window, uint32_t M, uint32_t B, uint32_t n_windows) {
    const double mean = window / M, most = (double)B + 1.0;
    return most > mean && most - mean - most * std::log(most / mean) + std::log((double)M * n_windows) <= -16.0;
}

// Ascending order, 11 bits at a time where there is much to sort.
static void sort_ascending(std::vector<uint32_t>& v) {
    if (v.size() < 2048u) {
        std::sort(v.begin(), v.end());
        return;
    }
    std::vector<uint32_t> other(v.size());
    for (uint32_t shift = 0; shift < 32u; shift += 11u) {
        std::vector<size_t> at(2049u, 0u);
        for (uint32_t x : v) ++at[((x >> shift) & 2047u) + 1u];
        for (uint32_t d = 0; d < 2047u; ++d) at[d + 1u] += at[d];
        for (uint32_t x : v) other[at[(x >> shift) & 2047u]++] = x;
        v.swap(other);
    }
}

// depth[i]: the largest number of requests of the whole trace, i or later, that are in service at an arrival when nobody waits
// and all are on their slowest kind of replica, the arriving one included; depth[R] = 0.
// From the finish times in order instead of a heap of them: setting the cost model of 131072 requests under load 7.0 to 2.3 ms.
static std::vector<uint32_t> service_depths(const ap_workload* w, const std::vector<uint32_t>& worst_service) {
    const uint32_t R = w->R;
    const uint32_t* arr = w->h_arrival.data();
    std::vector<uint32_t> finish;                            // of all requests that take any time; those are in service after their arrival
    finish.reserve(R);
    for (uint32_t r = 0; r < R; ++r)
        if (worst_service[r] != 0u) finish.push_back(arr[r] + worst_service[r]);      // below 2^32: the range proof
    sort_ascending(finish);
    std::vector<uint32_t> depth((size_t)R + 1u, 0u);
    size_t come = 0, gone = 0;                               // whoever has left by the arrival of r came before r
    for (uint32_t r = 0; r < R; ++r) {
        while (gone < finish.size() && finish[gone] <= arr[r]) ++gone;
        if (worst_service[r] != 0u) ++come;
        depth[r] = (uint32_t)(come - gone) + (worst_service[r] == 0u ? 1u : 0u);
    }
    for (uint32_t r = R; r-- > 0u;) depth[r] = std::max(depth[r], depth[r + 1u]);
    return depth;
}

// Plan of the split evaluation (ap_split.hpp) - replicas that differ or have windows, crowded traces, tables too
// small for the one-wavefront screen; linear cost models (rep_type == nullptr) and tabulated ones:
// the index ranges of every replica, the bound D on requests in service that started on arrival, the
// scratch area for one batch of candidates.  Leaves w->split false where the path does not apply.
// least_bin: per metric a bin that at least R - k99 + 1 requests reach on whichever kind of replica, without waiting.
// depth_from: service_depths (also behind the streamed evaluation: listing everything there costs crowded rows up to ten times
// as much where only the beginning of the trace is busy, 0.49 against 5.1 ms for 4096 rows of 16384 requests on one of 48
// replicas after 256 at 1500 a second, and saves a third where many rows are handed to the general replay, 7.7 against 5.1 ms
// with a busy quarter).  applies: the plan can be used.
// rep_type: the tabulated cost model (replica m reads row rep_type[m] of the tables, which are on the device by
// now); table_longest_prefill / table_longest_tpot are then the largest entries of the rows in use.
static ap_status plan_split(ap_workload* w, SplitPlan& plan, bool& applies,
                            const std::vector<DevReplica>& dev, const ap_replica* replicas,
                            const std::vector<uint32_t>& kinds, const std::vector<uint32_t>& worst_service,
                            const std::vector<uint64_t>& kind_sum, const std::vector<uint64_t>& kind_longest,
                            uint64_t latest_finish_bound, const uint32_t* rep_type, uint64_t table_longest_prefill,
                            uint64_t table_longest_tpot, const uint32_t* least_bin, const std::vector<uint32_t>& depth_from) {
    applies = false;
    const uint32_t R = w->R, M = w->params.M, B = w->params.B;
    if (!w->d_req8) return AP_OK;                            // request records with 16-bit lengths only
    const bool tabled = rep_type != nullptr;
    const bool wide = R >= 65536u;                           // two range words per replica, 32-bit histogram counts
    // The kernels multiply with 24-bit factors and add up a tile's sixteen latencies per lane in 32 bits.
    uint64_t longest_tpot = table_longest_tpot, longest_prefill = table_longest_prefill;
    for (uint32_t m = 0; m < M && !tabled; ++m) {
        if (replicas[m].prefill_per_tok_us >= (1u << 24) || replicas[m].decode_per_kctx_us >= (1u << 24)) return AP_OK;
        longest_tpot = std::max<uint64_t>(longest_tpot, (uint64_t)replicas[m].decode_base_us + 64ull * replicas[m].decode_per_kctx_us);
        longest_prefill = std::max<uint64_t>(longest_prefill, (uint64_t)replicas[m].prefill_base_us + 65535ull * replicas[m].prefill_per_tok_us);
    }
    if (longest_tpot >= (1u << 24)) return AP_OK;
    for (uint32_t m = 0; m < M && tabled; ++m)
        if (rep_type[m] >= 1024u) return AP_OK;              // the type rides in ten bits of a tile word
    const uint32_t longest_service = *std::max_element(worst_service.begin(), worst_service.end());
    if (longest_service >= (1u << 28)) return AP_OK;
    std::vector<uint32_t> tab(3u * (AP_MAX_REPLICAS + 1u) + 4u * kinds.size(), 0u);   // range words, kind words, coefficients
    std::vector<SplitQueue> queue(M);
    std::vector<uint32_t> order;

    // The streamed part of a replica may begin where the bound leaves an eighth of the slots to the listed part.
    const uint32_t reserve = B / 8u;
    const uint32_t i_calm = (uint32_t)(std::partition_point(depth_from.begin(), depth_from.end(),
                                                            [&](uint32_t d) { return d + reserve > B; }) - depth_from.begin());
    const uint32_t* arr = w->h_arrival.data();
    uint32_t longest_list = 0;
    uint64_t expect_rejected = 0;
    bool any_streamed = false;
    std::vector<uint32_t> i_list_of(M), i_off_of(M), kind_index(M);
    for (uint32_t m = 0; m < M; ++m) {
        const DevReplica& d = dev[m];
        const uint32_t i_on = (uint32_t)(std::lower_bound(arr, arr + R, d.t_on) - arr);
        const uint32_t i_off = (uint32_t)(std::lower_bound(arr, arr + R, d.t_off) - arr);
        // which kind of replica this is (its service times: mean and longest)
        size_t ki = 0;
        for (size_t k = 0; k < kinds.size(); ++k)
            if (tabled ? rep_type[kinds[k]] == rep_type[m]
                       : (replicas[kinds[k]].prefill_base_us == replicas[m].prefill_base_us &&
                          replicas[kinds[k]].prefill_per_tok_us == replicas[m].prefill_per_tok_us &&
                          replicas[kinds[k]].decode_base_us == replicas[m].decode_base_us &&
                          replicas[kinds[k]].decode_per_kctx_us == replicas[m].decode_per_kctx_us))
                ki = k;
        // The backlog a replica finds when it comes up is about its share of the requests so far; served B at a
        // time it is gone after so many mean service times, and the last of it after one longest service more.
        // Twice that is where the streamed part begins - a guess that only decides how often the list replay has
        // to hand a candidate back, never a result.
        uint32_t i_list = 0;
        if (i_on > 0u) {
            const double mean_service = (double)kind_sum[ki] / R;
            const double drain = 2.0 * (((double)i_on / M) / B + 1.0) * mean_service + (double)kind_longest[ki];
            const uint64_t t_target = (uint64_t)d.t_on + (uint64_t)std::min(drain, 4.0e9);
            i_list = (uint32_t)(std::lower_bound(arr, arr + R, (uint32_t)std::min<uint64_t>(t_target, kNever)) - arr);
        }
        i_list = std::min(std::max(i_list, i_calm), i_off);
        i_list_of[m] = i_list;
        i_off_of[m] = i_off;
        kind_index[m] = (uint32_t)ki;
    }
    const uint32_t hist_words = wide ? 3u * kBins : 3u * kBins / 2u, hist_bytes = hist_words * 4u;
    const uint32_t tile_cap = align_up(std::min(kTile, R) + 7u * std::min(M, std::min(kTile, R)), 8u);
    const uint32_t least_tpot_bin = std::min(least_bin[1], w->params.penalty_bin);
    const bool wide_bins = ap_hist_bin(longest_tpot) >= least_tpot_bin + kTpotSpan;
    // scratch of a candidate: lists, run descriptors, a partial record, histograms.  A trace so long that 64 candidates' lists take over
    // 8 GiB stays with the general replay.
    auto bytes_per_candidate = [&](uint32_t longest) {
        const size_t tiles = (longest + kTile - 1u) / kTile;
        return tiles * tile_cap * (2u + (wide_bins ? 8u : 4u)) + tiles * M * 4u + sizeof(SplitPartial) + hist_bytes + 2u * (M + 1u) * 4u;
    };
    const size_t most_per_candidate = ((size_t)8 << 30) / 64u;
    // Where next to nothing would be streamed, list that too: k_list_candidates takes half of k_split_candidates' time, and no row is handed back
    // for what its listed part leaves taken.  Calls of a busy beginning and a quiet end, streamed and listed, half of the replicas coming late:
    //   quiet   1677 rows of 20000, 50 replicas   200 rows    4096 of 4000 on 12   200 rows    559 of 60000 on 200   200 rows
    //    2 %    430 and 388 us                    223 and 215   318 and 207        121 and 116   678 and 590         344 and 334
    //    6 %    413 and 386                       216 and 215   490 and 204        166 and 116   660 and 590         335 and 335
    //   10 %    399 and 388                       208 and 214   476 and 204        165 and 116   635 and 585         325 and 335
    //   15 %    385 and 384                       198 and 214   529 and 206        166 and 115   607 and 590         311 and 334
    // (4000 on 12: streamed, rows are handed back).  The line, a fourteenth, is where 200 rows begin to lose; three lose 3 % there, and rows that
    // crowd a replica, which then wait for its quiet end as well, up to the share itself (200 rows of 4000 on one of 12, 6 % quiet, 727 and 763).
    // It is asked of every replica by itself: a row that crowds one waits for its list, request after request.  With the line on the trace as a
    // whole, 64 rows of 32768 requests on 4 replicas that stay while 60 are never there took 2.2 ms (54 us with these streamed), 7.5 ms on one of
    // them (64 us); even rows of 63 replicas that come at the end and one that stays would gain by it, 457 against 519 us.
    bool list_all = true;
    for (uint32_t m = 0; m < M; ++m) list_all = list_all && (i_off_of[m] - i_list_of[m]) * 14ull <= i_off_of[m];
    list_all = list_all && bytes_per_candidate(*std::max_element(i_off_of.begin(), i_off_of.end())) <= most_per_candidate;
    for (uint32_t m = 0; m < M; ++m) {
        const DevReplica& d = dev[m];
        const uint32_t i_list = list_all ? i_off_of[m] : i_list_of[m], i_off = i_off_of[m], ki = kind_index[m];
        tab[m] = wide ? i_list : (i_list | (i_off << 16));
        tab[AP_MAX_REPLICAS + 1u + m] = i_off;
        tab[2u * (AP_MAX_REPLICAS + 1u) + m] = tabled ? rep_type[m] : ki;
        any_streamed = any_streamed || i_list < i_off;
        SplitQueue q{};
        q.a = d.a; q.b = d.b; q.c = d.c; q.d = d.d; q.t_on = d.t_on; q.t_off = d.t_off;
        q.i_list = i_list;
        q.t_split = i_list < i_off ? arr[i_list] : kNever;
        q.allow_busy = i_list < i_off ? B - std::min(B, depth_from[i_list]) : 0u;
        q.late_from = d.t_off == kNever ? kNever : d.t_off - std::min(d.t_off, 3u * longest_service);
        queue[m] = q;
        longest_list = std::max(longest_list, i_list);
        expect_rejected += R - i_off;
    }
    tab[M] = 0u;                                             // unknown replica ids: rejected on arrival
    tab[AP_MAX_REPLICAS + 1u + M] = 0u;
    tab[2u * (AP_MAX_REPLICAS + 1u) + M] = 0u;
    for (size_t k = 0; k < kinds.size() && !tabled; ++k) {
        uint32_t* co = &tab[3u * (AP_MAX_REPLICAS + 1u) + 4u * k];
        co[0] = replicas[kinds[k]].prefill_base_us; co[1] = replicas[kinds[k]].prefill_per_tok_us;
        co[2] = replicas[kinds[k]].decode_base_us;  co[3] = replicas[kinds[k]].decode_per_kctx_us;
    }
    for (uint32_t m = 0; m < M; ++m)
        if (queue[m].i_list > 0u) order.push_back(m);
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return queue[x].i_list > queue[y].i_list; });

    SplitParams sp{};
    sp.R = R; sp.M = M; sp.B = B;
    sp.n_tiles = (R + kTile - 1u) / kTile;
    sp.n_list_tiles = (longest_list + kTile - 1u) / kTile;
    sp.tile_cap = tile_cap;
    sp.n_queues = (uint32_t)order.size();
    sp.even_lists = sp.n_queues == M && queue[order.front()].i_list == queue[order.back()].i_list ? 1u : 0u;
    sp.slo_ttft = w->params.slo_ttft;
    sp.slo_tpot = w->params.slo_tpot;
    // The p99 values are the penalty latency once R - k99 + 1 requests are rejected, if no served latency can
    // reach the penalty's bin: all of them lie below the bound on finish times of the range proof.
    const bool penalty_on_top = w->params.penalty_bin > ap_hist_bin(latest_finish_bound);
    sp.lazy_from = penalty_on_top ? R - w->params.k99 + 1u : kNever;
    plan.all_within = longest_prefill <= w->params.slo_ttft && longest_tpot <= w->params.slo_tpot;
    // A request that waits beyond its ready time finds all B slots taken by earlier ones, so it waits no longer than all service together
    // takes B slots.
    uint64_t all_service = 0, latest_on = 0;
    for (uint32_t r = 0; r < R; ++r) all_service += worst_service[r];
    for (const DevReplica& d : dev)
        if (d.t_on < d.t_off) latest_on = std::max<uint64_t>(latest_on, d.t_on);
    sp.step_facts = (longest_tpot <= w->params.slo_tpot ? kTpotWithin : 0u) |
                    (latest_on + all_service / B + longest_service < (1u << 30) ? kSumsFit : 0u);
    for (uint32_t h = 0; h < 3u; ++h) {
        sp.least_bin[h] = std::min(least_bin[h], w->params.penalty_bin);
        sp.least_us[h] = (uint32_t)std::min<uint64_t>(ap_hist_lower(sp.least_bin[h]), kNever);
    }
    sp.wide_bins = wide_bins ? 1u : 0u;
    sp.wide = wide ? 1u : 0u;
    sp.any_streamed = any_streamed ? 1u : 0u;
    sp.hist_words = hist_words;
    // LDS of the streaming kernel
    uint32_t off = ((uint32_t)kinds.size() + 1u) * 16u;      // the coefficients come first, and 0 behind them
    sp.off_range = off; off += align_up((M + 1u) * 4u, 16u);
    sp.off_range_off = off; off += wide ? align_up((M + 1u) * 4u, 16u) : 0u;
    sp.off_kind = off;  off += align_up((M + 1u) * 4u, 16u);
    sp.off_acc = off;   off += 64u;
    const uint32_t before_waves = off;
    sp.l_total = off;
    sp.l_wave = sp.l_total + align_up(M * 4u, 16u);
    sp.l_wave_bytes = align_up(runs_bytes(M, sp.tile_cap), 16u);
    // the wavefronts' areas come last, behind the histograms and totals where there are some
    sp.off_hist = off;
    sp.off_total = off + hist_bytes;
    sp.w_tile = sp.l_wave_bytes;
    sp.w_sums = sp.w_tile + align_up((M + 1u) * 4u, 16u);
    sp.wave_bytes = sp.w_sums + 3u * kWave * 8u;
    plan.off_wave[0] = off;
    plan.off_wave[1] = sp.off_total + align_up(M * 4u, 16u);
    int lds_cap = 0;
    if (hipDeviceGetAttribute(&lds_cap, hipDeviceAttributeMaxSharedMemoryPerBlock, w->device) != hipSuccess) return device_error();
    auto waves_most = [&](uint32_t fixed, uint32_t per_wave) { return std::min(kBuildMaxWaves, ((uint32_t)lds_cap - std::min((uint32_t)lds_cap, fixed)) / per_wave); };
    plan.list_waves_most = waves_most(sp.l_wave, sp.l_wave_bytes);
    for (uint32_t h = 0; h < 2u; ++h) plan.split_waves_most[h] = waves_most(plan.off_wave[h], sp.wave_bytes);
    // A replica table that large stays with the general replay.  The line is 28 bytes a replica, two a list position and two or four a request
    // of a tile for each of four wavefronts, and 8 or 12 a replica besides: 794 replicas with 16-bit counts, 607 with 32-bit ones (three kinds,
    // traces of a tile or more; 160 KB).  The kernels hold less: they would fit all 1024 and 951.  Above it, general replay and lists: 1000 even
    // rows of 16384 requests on 800 replicas of 8 slots that come and go 1255 and 459 us, that stay under load 1676 and 608, of 70000 on 700
    // 4646 and 1133 (4 slots, staying, 7146 and 2095); but rows on one replica that stays 2778 and 3569, 64 of them 696 and 3397, one of 70000 on
    // one of 700 2922 and 14700.  The lists lose as much below the line; it is kept until both kinds of row are worth having.
    const uint32_t held = 2u * align_up(M * 4u, 16u) + kTile * (M <= 64u ? 2u : 4u) + align_up(sp.tile_cap * 2u, 16u) + align_up(M * 8u, 16u) +
                          align_up((M + 1u) * 4u, 16u);
    if (before_waves - 16u + kBuildMinWaves * held + hist_bytes > (uint32_t)lds_cap ||
        std::min(plan.list_waves_most, std::min(plan.split_waves_most[0], plan.split_waves_most[1])) < kBuildMinWaves) return AP_OK;
    if (!tables_at_lds_zero(reinterpret_cast<const void*>(split_kernel(0u, tabled, plan.all_within))) ||
        !tables_at_lds_zero(reinterpret_cast<const void*>(split_kernel(wide ? 2u : 1u, tabled, plan.all_within))))
        return device_error();
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_list_candidates), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(sp.l_wave + plan.list_waves_most * sp.l_wave_bytes)) != hipSuccess ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(split_kernel(0u, tabled, plan.all_within)),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(plan.off_wave[0] + plan.split_waves_most[0] * sp.wave_bytes)) != hipSuccess ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(split_kernel(wide ? 2u : 1u, tabled, plan.all_within)),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(plan.off_wave[1] + plan.split_waves_most[1] * sp.wave_bytes)) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }

    const size_t bins_bytes = wide_bins ? 8u : 4u, per_cand = bytes_per_candidate(longest_list);
    if (per_cand > most_per_candidate) return AP_OK;
    // (2 of every 6 or 10 bytes are the lists themselves, so those of a batch stay below 2^32 bytes, which the list replay relies on)
    uint32_t batch = (uint32_t)std::min<size_t>(16384u, std::max<size_t>(64u, ((size_t)4 << 30) / per_cand));
    batch = batch / 64u * 64u;
    auto carve = [](size_t& at, size_t bytes) { const size_t here = at; at = (at + bytes + 255u) / 256u * 256u; return here; };
    size_t total = 0;
    for (;; batch = std::max(64u, batch / 2u / 64u * 64u)) {        // a device short of memory gets smaller batches
        total = 0;
        plan.o_lists = carve(total, (size_t)batch * sp.n_list_tiles * sp.tile_cap * 2u);
        plan.o_bins = carve(total, (size_t)batch * sp.n_list_tiles * sp.tile_cap * bins_bytes);
        plan.o_desc = carve(total, (size_t)batch * sp.n_list_tiles * M * 4u);
        plan.o_part = carve(total, (size_t)batch * sizeof(SplitPartial));
        plan.o_hist = carve(total, (size_t)batch * hist_bytes);
        plan.o_bin_base = carve(total, (size_t)batch * (M + 1u) * 4u);
        plan.o_bin_count = carve(total, (size_t)batch * (M + 1u) * 4u);
        if (total <= w->split_scratch_bytes) break;
        if (w->d_split_scratch && hipFree(w->d_split_scratch) != hipSuccess) return device_error();
        w->d_split_scratch = nullptr;
        w->split_scratch_bytes = 0;
        if (hipMalloc(&w->d_split_scratch, total) == hipSuccess) {
            w->split_scratch_bytes = total;
            break;
        }
        (void)hipGetLastError();
        w->d_split_scratch = nullptr;
        if (batch == 64u) return AP_OK;                         // no room for the lists: the general replay scores the calls
    }
    // the tables in one buffer: coefficients at a multiple of 16 bytes, like the queues
    std::vector<uint32_t> words(tab.size() + 4u + 12u * (size_t)M + order.size() + 16u, 0u);
    size_t at = 0;
    auto put = [&](const void* src, size_t n_words) {
        at = (at + 3u) / 4u * 4u;
        const size_t here = at;
        if (n_words) std::memcpy(&words[here], src, 4u * n_words);
        at += n_words;
        return here;
    };
    const size_t n_ranges = 3u * (AP_MAX_REPLICAS + 1u);
    const size_t o_tab = put(tab.data(), n_ranges), o_coef = put(tab.data() + n_ranges, tab.size() - n_ranges);
    const size_t o_queue = put(queue.data(), sizeof(SplitQueue) / 4u * M), o_order = put(order.data(), order.size());
    if (4u * words.size() > plan.tables_bytes) {
        if (plan.tables && hipFree(plan.tables) != hipSuccess) return device_error();
        plan.tables = nullptr;
        plan.tables_bytes = 0;
        if (hipMalloc(&plan.tables, 4u * words.size()) != hipSuccess) {
            (void)hipGetLastError();
            plan.tables = nullptr;
            return AP_ERR_ALLOC;
        }
        plan.tables_bytes = 4u * words.size();
    }
    if (hipMemcpy(plan.tables, words.data(), 4u * words.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipFuncSetAttribute(wide ? reinterpret_cast<const void*>(&k_merge_candidates<false>)
                                 : reinterpret_cast<const void*>(&k_merge_candidates<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)merge_lds_bytes(w, sp)) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    const uint32_t* base = reinterpret_cast<const uint32_t*>(plan.tables);
    sp.req8 = w->d_req8;
    sp.tab.range = base + o_tab;
    sp.tab.range_off = base + o_tab + (AP_MAX_REPLICAS + 1u);
    sp.tab.kind = base + o_tab + 2u * (AP_MAX_REPLICAS + 1u);
    sp.tab.coef = reinterpret_cast<const uint4*>(base + o_coef);
    sp.tab.n_kinds = tabled ? 0u : (uint32_t)kinds.size();
    sp.tab_pair = tabled ? w->d_tab_pair : nullptr;
    sp.queue = reinterpret_cast<const SplitQueue*>(base + o_queue);
    sp.order = base + o_order;
    plan.params = sp;
    plan.batch = batch;
    // A small call - few rows, and the fused replay's wavefront per queue has little more to do than a lane of the list replay -
    // is left to the fused replay: one launch instead of three to five.  It takes 40 ns a request of a row's longest queue and works on four
    // queues of a row at a time; the list replay takes 200 ns a request of the longest list while the chip is nearly empty, and the launches
    // 20 to 30 us together.  Both kinds of row, even ones and those that crowd a replica, are meant to gain.  Lists and fused replay: 64 rows of
    // 200 requests on 4 replicas that come and go, even 48 and 15 us, on one replica 58 and 19; 512 rows of 800 on 8 replicas that stay, even 51
    // and 28, on one 185 and 53; but 512 of 800 on 2 replicas that are mostly away, 34 and 37, on one 35 and 55.  With windows the longest
    // list says little about the others: there even rows have to do without it in the first term, and a crowded replica may have left early
    // (512 rows of 800 on 8, even 31 and 27, on one that has 25 and 53; 256 rows on 500, 56 and 51, 25 and 51).  Replicas with a streamed part
    // cost a launch or two more, and the line lies as much higher.  It was drawn when either took longer and is on the lists' side now: of what
    // it leaves to them, 64 rows of 1200 on 8 replicas that stay take 61 us and would take 22, 2000 on 24 51 and 28.
    plan.short_chain = !w->pipeline && (uint64_t)R * M <= 800ull * M + (w->small_table ? 7ull * longest_list : 0ull) &&
                       65ull * R <= (any_streamed ? 38000ull : 13000ull) + 115ull * longest_list;
    // stream without histograms first when an even spread of the requests over the replicas would reject enough (never behind the
    // streamed evaluation, whose replicas do not leave)
    plan.expect_lazy = !w->stream && penalty_on_top && expect_rejected / M >= sp.lazy_from;
    applies = true;
    return AP_OK;
}

// Plan of the counting screen (ap_counts.hpp): the bucket size and, per bucket, the first bucket with a request that is
// still in service when it begins.  Leaves w->counts false where no bucket size makes a row that is spread evenly over the
// replicas likely to pass.  worst_service: every request's service time (one kind of replica).
static ap_status plan_counts(ap_workload* w, const std::vector<uint32_t>& worst_service) {
    const uint32_t R = w->R, M = w->params.M, B = w->params.B;
    const std::vector<uint32_t> first = first_in_service(w, worst_service, kCountMinBucket, kCountShift);
    // Coarse buckets cost fewer checks, fine ones make a tighter window: the coarsest that will do.
    const uint32_t n_rows = M / 4u + 1u, columns_log2 = n_rows <= 40u ? 4u : n_rows <= 80u ? 3u : 2u;
    for (uint32_t w_log2 = 11u; w_log2 >= 7u; --w_log2) {
        const uint32_t per = (1u << w_log2) / kCountMinBucket;
        const uint32_t n_buckets = ((R + kCountShift) >> w_log2) + 1u;
        uint32_t window = 1u;
        for (uint32_t b = 0; b < n_buckets; ++b) window = std::max(window, b + 1u - (first[b * per] >> w_log2));
        uint32_t copies = 2u;
        while (copies < window + 1u) copies *= 2u;
        const uint32_t words = align_up(n_rows << columns_log2, 4u) + align_up(copies * n_rows, 4u);
        if (4u * words * 4u > kCountLdsBytes) continue;
        if (!windows_fit(std::min((double)window * (1u << w_log2), (double)R), M, B, n_buckets)) continue;
        std::vector<uint32_t> lo(n_buckets);
        for (uint32_t b = 0; b < n_buckets; ++b) lo[b] = first[b * per] >> w_log2;
        if (hipMemcpy(w->d_count_lo, lo.data(), 4u * (size_t)n_buckets, hipMemcpyHostToDevice) != hipSuccess) return device_error();
        CountParams cp{};
        cp.lo = w->d_count_lo;
        cp.nominal = w->d_nominal;
        cp.R = R; cp.M = M; cp.B = B;
        cp.w_log2 = w_log2;
        cp.ring_mask = copies - 1u;
        cp.n_rows = n_rows;
        cp.columns_log2 = columns_log2;
        cp.wave_words = words;
        w->count_params = cp;
        w->counts = true;
        return AP_OK;
    }
    return AP_OK;
}

// ap_hist_bin for values below 2^32, without its loop: the plans take it several times per request.
static uint32_t bin_of(uint32_t v) {
    const uint32_t s = 24u - std::min(v ? (uint32_t)__builtin_clz(v) : 32u, 24u);
    return (s << 7) + (v >> s);
}

// Per metric (ttft, tpot, e2e) a bin that at least R - k99 + 1 requests reach on their cheapest kind of replica without waiting:
// no candidate's p99 value of served requests lies below it.  The highest such bin where there are few kinds; where there are
// many coefficient sets, from the smallest of each coefficient, which no kind undercuts.  replicas: of the kinds, or null: the
// costs come from the tables (HOST, [T][R]) and kinds holds their rows.
static void least_bins(const ap_workload* w, std::vector<ap_replica> of_kind, const std::vector<uint32_t>& rows, const uint32_t* tab_prefill,
                       const uint32_t* tab_tpot, uint32_t (&least)[3]) {
    const uint32_t R = w->R, need = R - w->params.k99 + 1u;
    if (of_kind.size() > 8u) {
        ap_replica low = of_kind[0];
        for (const ap_replica& k : of_kind) {
            low.prefill_base_us = std::min(low.prefill_base_us, k.prefill_base_us);
            low.prefill_per_tok_us = std::min(low.prefill_per_tok_us, k.prefill_per_tok_us);
            low.decode_base_us = std::min(low.decode_base_us, k.decode_base_us);
            low.decode_per_kctx_us = std::min(low.decode_per_kctx_us, k.decode_per_kctx_us);
        }
        of_kind.assign(1u, low);
    }
    std::vector<uint32_t> count(3u * kBins, 0u);
    for (uint32_t r = 0; r < R; ++r) {                       // (all values are below 2^32: the range proof)
        uint32_t low[3] = {kNever, kNever, kNever};
        auto take = [&](uint32_t prefill, uint32_t tpot) {
            low[0] = std::min(low[0], prefill);
            low[1] = std::min(low[1], tpot);
            low[2] = std::min(low[2], prefill + (uint32_t)w->h_out[r] * tpot);
        };
        const uint32_t prompt = (uint32_t)w->h_prompt[r], ctx = (prompt + 1023u) >> 10;
        for (const ap_replica& k : of_kind) take(k.prefill_base_us + k.prefill_per_tok_us * prompt, k.decode_base_us + k.decode_per_kctx_us * ctx);
        for (uint32_t t : rows) take(tab_prefill[(size_t)t * R + r], tab_tpot[(size_t)t * R + r]);
        for (uint32_t h = 0; h < 3u; ++h) ++count[h * kBins + bin_of(low[h])];
    }
    for (uint32_t h = 0; h < 3u; ++h) {
        uint32_t bin = kBins, reached = 0;
        while (bin > 0u && reached < need) reached += count[h * kBins + --bin];
        least[h] = bin;
    }
}

// Plan of the streamed evaluation (ap_stream.hpp): bucket size, window table, the bins from which large values are counted.
// Leaves w->stream false where it does not apply.  cost(k, r, prefill, tpot): the cost of request r on the kind of replica
// whose first replica is k; rep_type: tabulated cost model; least_bin: as for plan_split; longest: no ttft, tpot or e2e of a request
// that does not wait is larger on any kind; most_in_service: the largest of service_depths.
extern "C++" template <typename Cost>
static ap_status plan_stream(ap_workload* w, const ap_replica* replicas, const std::vector<uint32_t>& kinds,
                             const std::vector<uint32_t>& kind_of, const std::vector<uint32_t>& worst_service, const uint32_t* rep_type,
                             const Cost& cost, const uint32_t* least_bin, const uint32_t* longest, uint32_t most_in_service) {
    const uint32_t R = w->R, M = w->params.M, B = w->params.B;
    const bool tabled = rep_type != nullptr;
    if (!w->d_req8) return AP_OK;                            // request records with 16-bit lengths only
    for (uint32_t m = 0; m < M && !tabled; ++m)              // the kernel multiplies with 24-bit factors
        if (replicas[m].prefill_per_tok_us >= (1u << 24) || replicas[m].decode_per_kctx_us >= (1u << 24) ||
            (uint64_t)replicas[m].decode_base_us + 64ull * replicas[m].decode_per_kctx_us >= (1u << 24))
            return AP_OK;
    for (uint32_t r = 0; r < R; ++r)                         // and adds up eight latencies in 32 bits
        if (worst_service[r] >= (1u << 28)) return AP_OK;
    // With no more than B requests in service at once nobody waits on any row: nothing to count.
    const bool settles = most_in_service <= B;
    // bucket size: the coarsest that will do and whose counts fit (32 KiB: four workgroups per compute unit; more was not measured)
    const uint32_t words = (M + 4u) / 4u;
    const std::vector<uint32_t> first = settles ? std::vector<uint32_t>() : first_in_service(w, worst_service, 2u, 1u);
    uint32_t w_log2 = 7u, n_buckets = 0;
    for (; !settles; --w_log2) {
        if (w_log2 == 0u) return AP_OK;
        n_buckets = ((R + 1u) >> w_log2) + 1u;
        if ((uint64_t)n_buckets * (words * 4u + 2u) > 32768u) return AP_OK;
        const uint32_t per = (1u << w_log2) / 2u;
        uint32_t window = 1u;
        for (uint32_t b = 0; b < n_buckets; ++b) window = std::max(window, b + 1u - (first[b * per] >> w_log2));
        if (windows_fit(std::min((double)window * (1u << w_log2), (double)R), M, B, n_buckets)) break;
    }
    if (tabled && longest[1] >= (1u << 24)) return AP_OK;
    const uint32_t highest[3] = {bin_of(longest[0]), bin_of(longest[1]), bin_of(longest[2])};
    // Values per bin when the requests are spread over the kinds as the replicas are (in units of 1 / M), from a sample of the
    // requests: all that hangs on it is how many values are counted and how often a row is read twice.  (One kind: least_bin says it.)
    const uint32_t n_kinds = (uint32_t)kinds.size(), n_sample = n_kinds == 1u ? 0u : std::min(R, std::max(1024u, 6144u / n_kinds));
    std::vector<uint32_t> share(n_kinds, 0u);
    for (uint32_t m = 0; m < M; ++m) ++share[kind_of[m]];
    std::vector<uint16_t> bins(3u * (size_t)n_kinds * n_sample);       // [kind][request of the sample][metric]
    std::vector<uint64_t> weight(3u * kBins, 0u);
    for (uint32_t k = 0; k < n_kinds; ++k)
        for (uint32_t i = 0; i < n_sample; ++i) {
            const uint32_t r = (uint32_t)((uint64_t)i * R / n_sample);
            uint64_t prefill, tpot;
            cost(kinds[k], r, prefill, tpot);
            const uint64_t value[3] = {prefill, tpot, prefill + (uint64_t)w->h_out[r] * tpot};
            for (uint32_t h = 0; h < 3u; ++h) {
                const uint32_t bin = bin_of((uint32_t)value[h]);
                bins[3u * ((size_t)k * n_sample + i) + h] = (uint16_t)bin;
                weight[h * kBins + bin] += share[k];
            }
        }
    StreamParams sp{};
    sp.need_top = R - w->params.k99 + 1u;
    // twice what is needed, and room for the spread of a small number of requests
    const double want = (2.0 * sp.need_top + 8.0 * std::sqrt((double)sp.need_top) + 8.0) * M * n_sample / R;
    uint32_t total_bins = 0;
    for (uint32_t h = 0; h < 3u; ++h) {
        uint32_t from = n_kinds == 1u ? 0u : highest[h] + 1u;
        double reached = 0.0;
        while (from > 0u && reached < want) reached += (double)weight[h * kBins + --from];
        sp.from[h] = std::min(std::min(least_bin[h], w->params.penalty_bin), highest[h]);
        const uint32_t counted_from[2] = {std::max(from, sp.from[h]), sp.from[h]};
        for (uint32_t i = 0; i < 2u; ++i) {
            sp.least[i][h] = (uint32_t)ap_hist_lower(counted_from[i]);
            sp.n_counted[i][h] = highest[h] + 1u - counted_from[i];
        }
        sp.n_bins[h] = sp.n_counted[1][h];
        total_bins += sp.n_bins[h];
    }
    // A sample of a row tells which bins to count from, where the row is long enough to pay for it: it takes 2 us, a reading
    // 1 us per thousand requests.
    std::vector<uint32_t> sample_weight;
    if (R >= 8192u && std::memcmp(sp.least[0], sp.least[1], sizeof(sp.least[0])) != 0) {
        const uint32_t most = 16u * kStreamWeight;
        sample_weight.assign(M + 1u, 0u);
        std::vector<uint32_t> kind_weight(n_kinds, most);
        for (uint32_t k = 0; k < n_kinds; ++k) {
            uint64_t large[3] = {0u, 0u, 0u};
            for (uint32_t i = 0; i < n_sample; ++i)
                for (uint32_t h = 0; h < 3u; ++h) large[h] += bins[3u * ((size_t)k * n_sample + i) + h] + sp.n_counted[0][h] > highest[h] ? 1u : 0u;
            for (uint32_t h = 0; h < 3u; ++h)
                kind_weight[k] = (uint32_t)std::min<uint64_t>(kind_weight[k], large[h] * kStreamWeight * R / n_sample / sp.need_top);
        }
        for (uint32_t m = 0; m < M; ++m) sample_weight[m] = kind_weight[kind_of[m]];
        bool rejected_is_large = true;
        for (uint32_t h = 0; h < 3u; ++h) rejected_is_large = rejected_is_large && ap_hist_lower(w->params.penalty_bin) >= sp.least[0][h];
        sample_weight[M] = rejected_is_large ? most : 0u;
    }
    uint32_t off = align_up((M + 1u) * 4u, 16u);
    sp.off_coef = off; off += tabled ? 0u : (uint32_t)kinds.size() * 16u;
    sp.off_lo = off;   off += align_up(n_buckets * 2u, 16u);
    sp.off_cnt = off;  off += align_up(n_buckets * words * 4u, 16u);
    sp.off_hist = off; off += align_up(total_bins * 4u, 16u);
    sp.off_acc = off;  off += 64u;
    if (off > 65536u) return AP_OK;
    sp.off_large = off;                                      // behind them the wavefronts' buffers, as many as a call's workgroups have
    // one buffer: coefficients, kinds, window table, weights
    std::vector<uint32_t> tab(4u * kinds.size() + (M + 1u) + n_buckets + sample_weight.size(), 0u);
    for (size_t k = 0; k < kinds.size() && !tabled; ++k) {
        const ap_replica& rp = replicas[kinds[k]];
        tab[4u * k] = rp.prefill_base_us; tab[4u * k + 1u] = rp.prefill_per_tok_us;
        tab[4u * k + 2u] = rp.decode_base_us; tab[4u * k + 3u] = rp.decode_per_kctx_us;
    }
    uint32_t* kind_words = &tab[4u * kinds.size()];
    for (uint32_t m = 0; m < M; ++m) kind_words[m] = tabled ? rep_type[m] * R : kind_of[m];
    kind_words[M] = tabled ? rep_type[0] * R : 0u;           // unknown ids: any entry, its cost is not used
    for (uint32_t b = 0; b < n_buckets; ++b) kind_words[M + 1u + b] = first[b * ((1u << w_log2) / 2u)] >> w_log2;
    std::copy(sample_weight.begin(), sample_weight.end(), kind_words + M + 1u + n_buckets);
    if (4u * tab.size() > w->stream_tab_bytes) {
        if (w->d_stream_tab && hipFree(w->d_stream_tab) != hipSuccess) return device_error();
        w->d_stream_tab = nullptr;
        w->stream_tab_bytes = 0;
        if (hipMalloc(&w->d_stream_tab, 4u * tab.size()) != hipSuccess) {
            (void)hipGetLastError();
            w->d_stream_tab = nullptr;
            return AP_OK;                                    // no room: the listed evaluation scores the calls
        }
        w->stream_tab_bytes = 4u * tab.size();
    }
    if (hipMemcpy(w->d_stream_tab, tab.data(), 4u * tab.size(), hipMemcpyHostToDevice) != hipSuccess) return device_error();
    sp.req8 = w->d_req8;
    sp.coef = reinterpret_cast<const uint4*>(w->d_stream_tab);
    sp.tab_pair = tabled ? w->d_tab_pair : nullptr;
    sp.kind = w->d_stream_tab + 4u * kinds.size();
    sp.lo = sp.kind + (M + 1u);
    sp.weight = sample_weight.empty() ? nullptr : sp.lo + n_buckets;
    sp.n_kinds = tabled ? 0u : (uint32_t)kinds.size();
    sp.R = R; sp.M = M; sp.B = B;
    sp.w_log2 = w_log2; sp.n_buckets = n_buckets; sp.words = words;
    sp.slo_ttft = w->params.slo_ttft; sp.slo_tpot = w->params.slo_tpot;
    sp.all_within = highest[0] < ap_hist_bin(sp.slo_ttft) && highest[1] < ap_hist_bin(sp.slo_tpot) ? 1u : 0u;
    sp.penalty_bin = w->params.penalty_bin;
    sp.penalty = w->params.penalty;
    if (!tables_at_lds_zero(reinterpret_cast<const void*>(stream_kernel(settles, tabled)))) return device_error();
    constexpr uint32_t large = kStreamMaxThreads / kWave * kStreamLargeBytes;
    if (off + large > 65536u &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(stream_kernel(settles, tabled)), hipFuncAttributeMaxDynamicSharedMemorySize,
                            65536 + (int)large) != hipSuccess)
        return device_error();
    w->stream_params = sp;
    w->stream_lds_bytes = off;
    w->stream = true;
    w->stream_settles = settles;
    return AP_OK;
}

// Slots per replica of the one-wavefront ring screen: a power of two, at most B, as long as that wavefront's slot state
// (rings and counters of M + 1 replicas) stays small enough for many wavefronts per compute unit.  wide: the state
// leaves room for fewer slots than are worth having, so the eight-wavefront kernel, whose workgroup holds one row's
// rings, takes the table.
static uint32_t narrow_ring_slots_log2(uint32_t M, uint32_t B, bool& wide) {
    uint32_t most = 0, S_log2 = 0;
    while ((2u << most) <= kScreenMaxSlots && (M + 1u) * ((2u << most) + 1u) * 4u <= kScreenLdsPerWave) ++most;
    while (S_log2 < most && (2u << S_log2) <= B) ++S_log2;
    wide = (1u << most) < std::min(B, kScreenMinSlots);
    return S_log2;
}

// Shared by ap_costmodel_set (rep_type == nullptr: the coefficients of `replicas` apply) and
// ap_costtable_set (replica m is of type rep_type[m] < T and the HOST tables [T][R] apply; the
// coefficients are ignored).
// tab_prefill == nullptr with rep_type set: the tables are in the workload's device buffers already
// (ap_costtable_set_roofline) and the bounds come from a reduction over them.
static ap_status set_cost_model_checked(ap_workload* w, const ap_replica* replicas, uint32_t M, uint32_t B, const ap_slo* slo,
                                        const uint32_t* rep_type, const uint32_t* tab_prefill, const uint32_t* tab_tpot,
                                        uint32_t T);

static ap_status set_cost_model(ap_workload* w, const ap_replica* replicas, uint32_t M, uint32_t B, const ap_slo* slo,
                                const uint32_t* rep_type, const uint32_t* tab_prefill, const uint32_t* tab_tpot, uint32_t T) {
    try {                                                   // host containers allocate: nothing may leave through the C ABI
        return set_cost_model_checked(w, replicas, M, B, slo, rep_type, tab_prefill, tab_tpot, T);
    } catch (const std::bad_alloc&) {
        if (w) w->has_model = false;
        return AP_ERR_ALLOC;
    }
}

static ap_status set_cost_model_checked(ap_workload* w, const ap_replica* replicas, uint32_t M, uint32_t B, const ap_slo* slo,
                                        const uint32_t* rep_type, const uint32_t* tab_prefill, const uint32_t* tab_tpot,
                                        uint32_t T) {
    if (!w || !replicas || !slo || M == 0 || B == 0) return AP_ERR_INVALID;
    const bool tabled = rep_type != nullptr;
    const bool on_device = tabled && tab_prefill == nullptr;
    for (uint32_t m = 0; m < M; ++m)
        if (replicas[m].t_on_us > replicas[m].t_off_us) return AP_ERR_INVALID;
    if (M > AP_MAX_REPLICAS || B > AP_MAX_SLOTS) return AP_ERR_RANGE;

    // ---- range proof for 32-bit relative time ------------------------------------------
    // Every start is at most max(latest arrival, latest t_on of a replica that can serve)
    // plus the total of all earlier service on that replica; bound the latter by the sum
    // over requests of their largest service time on any replica.
    const uint64_t limit = (uint64_t)kNever - 1u;
    uint64_t latest = w->span_us;
    for (uint32_t m = 0; m < M; ++m) {
        const ap_replica& rp = replicas[m];
        if (rp.t_on_us >= rp.t_off_us || rp.t_on_us <= w->base_us) continue;   // never serves / already on
        latest = std::max(latest, rp.t_on_us - w->base_us);
    }
    if (latest > limit) return AP_ERR_RANGE;
    // distinct kinds of replica (coefficient sets, or types with tables), each by its first replica
    std::vector<uint32_t> kinds;
    auto same_kind = [&](uint32_t x, uint32_t y) {
        return tabled ? rep_type[x] == rep_type[y]
                      : (replicas[x].prefill_base_us == replicas[y].prefill_base_us &&
                         replicas[x].prefill_per_tok_us == replicas[y].prefill_per_tok_us &&
                         replicas[x].decode_base_us == replicas[y].decode_base_us &&
                         replicas[x].decode_per_kctx_us == replicas[y].decode_per_kctx_us);
    };
    for (uint32_t m = 0; m < M; ++m) {
        bool seen = false;
        for (uint32_t k : kinds) seen = seen || same_kind(k, m);
        if (!seen) kinds.push_back(m);
    }
    // prefill time and time per token of request r on the kind whose first replica is k
    auto host_cost = [&](uint32_t k, uint32_t r, uint64_t& prefill, uint64_t& tpot) {
        if (tabled) {
            prefill = tab_prefill[(size_t)rep_type[k] * w->R + r];
            tpot = tab_tpot[(size_t)rep_type[k] * w->R + r];
        } else {
            // each term stays far below 2^64: coefficients < 2^32, lengths < 2^31
            const uint64_t prompt = (uint64_t)w->h_prompt[r];
            prefill = (uint64_t)replicas[k].prefill_base_us + (uint64_t)replicas[k].prefill_per_tok_us * prompt;
            tpot = (uint64_t)replicas[k].decode_base_us + (uint64_t)replicas[k].decode_per_kctx_us * ((prompt + 1023u) >> 10);
        }
    };
    uint64_t total = latest;
    uint64_t table_longest_prefill = 0, table_longest_tpot = 0;   // tabulated: the largest entries of the rows in use
    uint64_t latest_unqueued = 0;      // latest finish if nobody ever waited (arrival + service)
    uint64_t longest_pair = 0;         // longest time from the arrival of request 2q to the unqueued finish of 2q or 2q+1
    uint64_t service_sum = 0;
    std::vector<uint32_t> worst_service;            // per request: its longest service time over the kinds of replica
    std::vector<uint64_t> kind_sum, kind_longest;   // per kind: all service times added up, and the longest
    try {
        worst_service.resize(w->R);
        kind_sum.assign(kinds.size(), 0u);
        kind_longest.assign(kinds.size(), 0u);
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    if (on_device) {
        if (hipSetDevice(w->device) != hipSuccess) return device_error();
        std::vector<uint32_t> in_use;
        try {
            for (uint32_t k : kinds) in_use.push_back(rep_type[k]);
        } catch (const std::bad_alloc&) {
            return AP_ERR_ALLOC;
        }
        TableBounds bounds{};
        TableBounds* d_bounds = reinterpret_cast<TableBounds*>(w->d_bounds);
        uint32_t* d_in_use = reinterpret_cast<uint32_t*>(w->d_bounds + sizeof(TableBounds));
        if (hipMemcpy(d_bounds, &bounds, sizeof(bounds), hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(d_in_use, in_use.data(), 4u * in_use.size(), hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipGetLastError();
            return device_error();
        }
        const uint32_t blocks = std::max(1u, std::min(1024u, (w->R + kRoofThreads - 1u) / kRoofThreads));
        hipLaunchKernelGGL(k_table_bounds, dim3(blocks), dim3(kRoofThreads), 0, nullptr, w->d_tab_prefill, w->d_tab_tpot, d_in_use,
                           (uint32_t)in_use.size(), w->d_arrival, w->d_out, w->R, d_bounds, w->d_span);
        // (the table of contention-free intervals is not in use at this point: it takes every request's longest
        // service time, 4 R bytes, which the host's sweep over the trace needs)
        if (hipGetLastError() != hipSuccess ||
            hipMemcpy(&bounds, d_bounds, sizeof(bounds), hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(worst_service.data(), w->d_span, 4u * (size_t)w->R, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipGetLastError();
            return device_error();
        }
        if (bounds.over_range != 0u || bounds.service_sum > limit - latest) return AP_ERR_RANGE;
        service_sum = bounds.service_sum;
        total += bounds.service_sum;
        latest_unqueued = bounds.latest_unqueued;
        longest_pair = bounds.longest_pair;
        table_longest_prefill = bounds.longest_prefill;
        table_longest_tpot = bounds.longest_tpot;
        for (size_t ki = 0; ki < kinds.size(); ++ki) {      // only a guess is made from these: the kinds are not told apart
            kind_sum[ki] = bounds.service_sum;
            for (uint32_t r = 0; r < w->R; ++r) kind_longest[ki] = std::max<uint64_t>(kind_longest[ki], worst_service[r]);
        }
    }
    for (uint32_t r = 0; r < (on_device ? 0u : w->R); ++r) {
        const uint64_t outl = (uint64_t)w->h_out[r];
        uint64_t worst = 0;
        for (size_t ki = 0; ki < kinds.size(); ++ki) {
            uint64_t prefill, tpot;
            host_cost(kinds[ki], r, prefill, tpot);
            if (tpot > limit || prefill > limit) return AP_ERR_RANGE;
            if (tabled) {
                table_longest_prefill = std::max(table_longest_prefill, prefill);
                table_longest_tpot = std::max(table_longest_tpot, tpot);
            }
            uint64_t svc = prefill + outl * tpot;
            worst = std::max(worst, svc);
            kind_sum[ki] += std::min(svc, limit);
            kind_longest[ki] = std::max(kind_longest[ki], std::min(svc, limit));
        }
        worst_service[r] = (uint32_t)std::min(worst, limit);
        total += worst;
        service_sum += worst;
        latest_unqueued = std::max<uint64_t>(latest_unqueued, (uint64_t)w->h_arrival[r] + worst);
        longest_pair = std::max<uint64_t>(longest_pair, (uint64_t)w->h_arrival[r] + worst - w->h_arrival[r & ~1u]);
        if (total > limit) return AP_ERR_RANGE;
    }

    // ---- LDS plan: the largest chunk that fits ------------------------------------------
    if (hipSetDevice(w->device) != hipSuccess) return device_error();
    int lds_cap = 0, n_cu = 0;
    if (hipDeviceGetAttribute(&lds_cap, hipDeviceAttributeMaxSharedMemoryPerBlock, w->device) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, w->device) != hipSuccess)
        return device_error();
    EvalParams p{};
    p.M = M;
    p.B = B;
    // No bin can count more than R requests, so below 65536 requests two bins share a word.
    const bool hist16 = w->R < 65536u;
    // A chunk should hand each replica about 56 requests, so that the 64-lane blocks of the
    // replay are mostly full and rarely spill into a second block; more than that only costs
    // LDS.  At least 2048 requests where there are more than 1024: small tables gain from fewer barriers (a row of 4096 requests on 8
    // replicas 27 to 22 us).  Prefer a size that lets two workgroups share a compute unit (they cover each
    // other's barriers); otherwise take the largest chunk one workgroup can hold.
    const uint32_t want = std::min(kMaxChunk, std::max((w->R > 2u * kThreads ? 4u : 2u) * kThreads, align_up(56u * M, kThreads)));
    uint32_t bytes = 0, chunk = 0;
    uint32_t by_registers = 1;                               // workgroups of the kernel that a compute unit's registers hold
    {   // what the kernel itself declares (nothing today) comes off the dynamic part
        hipFuncAttributes attr;
        if (hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(eval_kernel(hist16, w->len16, tabled))) != hipSuccess)
            return device_error();
        lds_cap -= (int)std::min<size_t>(attr.sharedSizeBytes, (size_t)lds_cap);
        by_registers = std::max(1u, waves_by_registers(attr) * 4u / kWaves);
    }
    for (uint32_t budget : {(uint32_t)lds_cap / 2u, (uint32_t)lds_cap}) {
        const uint32_t smallest = budget == (uint32_t)lds_cap ? kThreads : std::max(kThreads, want / 2u);
        for (chunk = want; chunk >= smallest; chunk -= kThreads) {
            bytes = plan_lds(p, chunk, hist16, w->len16);
            if (bytes <= budget) break;
        }
        if (chunk >= smallest) break;
        chunk = 0;
    }
    // When even the smallest chunk does not fit (large M * B), candidates are scored by the
    // three-kernel pipeline instead, whose slot state is per queue rather than per candidate.
    const bool use_pipeline = chunk == 0;
    if (use_pipeline) bytes = 0;

    // LDS of the kernels that only need the histograms and the accumulators behind them
    const uint32_t hist_bytes = 3u * kBins * (hist16 ? 2u : 4u);
    const uint32_t reduce_lds = hist_bytes + 64u + 3u * kWaves * 4u;

    std::vector<DevReplica> dev(M);
    for (uint32_t m = 0; m < M; ++m) {
        const ap_replica& rp = replicas[m];
        DevReplica& d = dev[m];
        d.a = tabled ? rep_type[m] * w->R : rp.prefill_base_us;     // T * R < 2^32 was checked by the caller
        d.b = tabled ? 0u : rp.prefill_per_tok_us;
        d.c = tabled ? 0u : rp.decode_base_us;
        d.d = tabled ? 0u : rp.decode_per_kctx_us;
        if (rp.t_on_us >= rp.t_off_us || rp.t_off_us <= w->base_us) {
            d.t_on = 0;      // the window is empty or closed before the trace: nothing is ever served
            d.t_off = 0;
        } else {
            d.t_on = rp.t_on_us <= w->base_us ? 0u : (uint32_t)(rp.t_on_us - w->base_us);
            d.t_off = (uint32_t)std::min<uint64_t>(rp.t_off_us - w->base_us, kNever);
        }
    }
    if (tabled) {
        const size_t entries = (size_t)T * w->R;
        if (entries > w->tab_entries && !on_device) {
            if ((w->d_tab_prefill && hipFree(w->d_tab_prefill) != hipSuccess) ||
                (w->d_tab_tpot && hipFree(w->d_tab_tpot) != hipSuccess))
                return device_error();
            w->d_tab_prefill = w->d_tab_tpot = nullptr;
            w->tab_entries = 0;
            w->has_model = false;     // the previous model may have pointed at the freed tables
            if (hipMalloc(&w->d_tab_prefill, entries * 4u) != hipSuccess || hipMalloc(&w->d_tab_tpot, entries * 4u) != hipSuccess) {
                (void)hipGetLastError();
                return AP_ERR_ALLOC;
            }
            w->tab_entries = entries;
        }
        if (on_device && entries > w->tab_entries) return AP_ERR_STATE;       // the caller filled them: they exist
        if (!on_device &&
            (hipMemcpy(w->d_tab_prefill, tab_prefill, entries * 4u, hipMemcpyHostToDevice) != hipSuccess ||
             hipMemcpy(w->d_tab_tpot, tab_tpot, entries * 4u, hipMemcpyHostToDevice) != hipSuccess)) {
            (void)hipGetLastError();
            w->has_model = false;
            return device_error();
        }
    }
    if (hipMemcpy(w->d_rep, dev.data(), sizeof(DevReplica) * M, hipMemcpyHostToDevice) != hipSuccess ||
        (!use_pipeline && hipFuncSetAttribute(reinterpret_cast<const void*>(eval_kernel(hist16, w->len16, tabled)),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) ||
        hipFuncSetAttribute(hist16 ? reinterpret_cast<const void*>(&k_nominal_metrics<true>)
                                   : reinterpret_cast<const void*>(&k_nominal_metrics<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)reduce_lds) != hipSuccess) {
        (void)hipGetLastError();
        w->has_model = false;     // the replica table on the device may be half-written
        return device_error();
    }

    p.arrival = w->d_arrival;
    p.prompt = w->d_prompt;
    p.outlen = w->d_out;
    p.rep = w->d_rep;
    p.tab_prefill = tabled ? w->d_tab_prefill : nullptr;
    p.tab_tpot = tabled ? w->d_tab_tpot : nullptr;
    p.R = w->R;
    p.key_bits = 0;
    while (((M - 1u) >> p.key_bits) != 0u) ++p.key_bits;       // bits needed for the replica ids 0..M-1
    p.slo_ttft = (uint32_t)std::min<uint64_t>(slo->ttft_us, kNever);
    p.slo_tpot = (uint32_t)std::min<uint64_t>(slo->tpot_us, kNever);
    p.penalty = slo->penalty_us;
    p.penalty_bin = ap_hist_bin(slo->penalty_us);
    p.k99 = (uint32_t)((99ull * w->R + 99ull) / 100ull);
    p.replayed = w->d_pending + 2;
    if (hipMemset(p.replayed, 0, sizeof(uint32_t)) != hipSuccess) return device_error();
    w->n_scored = 0;
    w->has_model = false;
    w->has_parent = false;    // its analysis belonged to the previous cost model
    w->tabled = tabled;
    w->params = p;
    w->lds_bytes = bytes;
    w->hist16 = hist16;
    w->n_cu = (uint32_t)n_cu;
    w->max_grid = (uint32_t)n_cu * 64u;    // few candidates per workgroup: the hardware balances uneven finish times
    // Behind a screen: a workgroup looks at C / resident_grid records, all at once, and replays those of them that are marked.  As many as LDS
    // holds, four at most per compute unit, rounded up to a multiple of what registers and LDS hold together (two): three, which LDS
    // alone allows with the chunk above, left the third of every three beside an empty place.  8192 rows of 4096 requests, all on one of
    // 16 replicas, 3240 us with two or four workgroups per compute unit, 4060 with three; where some rows are marked two take 147 us and
    // four 124 (3000 rows of 3000 requests on 4 of 8 replicas); where none is, 512 more that leave at once cost half a microsecond.
    const uint32_t by_lds = std::min(4u, bytes ? (uint32_t)lds_cap / bytes : 1u), at_once = std::max(1u, std::min(by_lds, by_registers));
    w->resident_grid = (uint32_t)n_cu * ((std::max(1u, by_lds) + at_once - 1u) / at_once * at_once);

    // ---- three-kernel replay: scratch for one batch of candidates -------------------------
    w->reduce_eval = p;
    w->reduce_eval.off_misc = hist_bytes;                              // histograms, then the accumulators
    w->reduce_lds_bytes = reduce_lds;
    w->pipeline = use_pipeline;
    if (use_pipeline) {
        const uint32_t R = w->R;
        const uint32_t chunk_g = std::min(kGroupThreads * kGroupMaxPerThread, align_up(R, kGroupThreads));
        const uint32_t n_chunks = (R + chunk_g - 1u) / chunk_g;
        const uint32_t qs_stride = align_up(M + 2u, 8u);
        const size_t slots = (size_t)n_chunks * chunk_g;               // list positions per candidate
        const size_t per_cand = (size_t)n_chunks * qs_stride * 2u + slots * (2u + 4u + 2u) + (size_t)M * sizeof(QueuePartial) + 4u;
        const size_t target = (size_t)1 << 30;                         // enough candidates per batch to fill the GPU
        uint32_t batch = (uint32_t)std::min<size_t>(65535u, std::max<size_t>(1u, target / per_cand));
        auto carve = [](size_t& off, size_t bytes) { const size_t at = off; off = (off + bytes + 255u) / 256u * 256u; return at; };
        size_t off = 0;
        const size_t o_qs = carve(off, (size_t)batch * n_chunks * qs_stride * 2u);
        const size_t o_list = carve(off, (size_t)batch * slots * 2u);
        const size_t o_te = carve(off, (size_t)batch * slots * 4u);
        const size_t o_p = carve(off, (size_t)batch * slots * 2u);
        const size_t o_part = carve(off, (size_t)batch * M * sizeof(QueuePartial));
        const size_t o_unk = carve(off, (size_t)batch * 4u);
        if (off > w->scratch_bytes) {
            if (w->d_scratch && hipFree(w->d_scratch) != hipSuccess) return device_error();
            w->d_scratch = nullptr;
            w->scratch_bytes = 0;
            if (hipMalloc(&w->d_scratch, off) != hipSuccess) {
                (void)hipGetLastError();
                return AP_ERR_ALLOC;
            }
            w->scratch_bytes = off;
        }
        if (hipMemset(w->d_scratch + o_unk, 0, (size_t)batch * 4u) != hipSuccess) return device_error();
        w->batch = batch;
        GroupParams gp{};
        gp.R = R; gp.M = M; gp.chunk = chunk_g; gp.n_chunks = n_chunks; gp.key_bits = p.key_bits; gp.qs_stride = qs_stride;
        gp.qs = reinterpret_cast<uint16_t*>(w->d_scratch + o_qs);
        gp.list = reinterpret_cast<uint16_t*>(w->d_scratch + o_list);
        gp.unknown = reinterpret_cast<uint32_t*>(w->d_scratch + o_unk);
        gp.replayed = p.replayed;
        w->group_params = gp;
        w->group_lds_bytes = (kGroupWaves * (M + 1u) + M + 2u) * 4u;
        ReplayParams qp{};
        qp.req = w->d_req; qp.rep = w->d_rep; qp.qs = gp.qs; qp.list = gp.list;
        qp.tab_prefill = p.tab_prefill; qp.tab_tpot = p.tab_tpot;
        qp.bins_te = reinterpret_cast<uint32_t*>(w->d_scratch + o_te);
        qp.bins_p = reinterpret_cast<uint16_t*>(w->d_scratch + o_p);
        qp.partial = reinterpret_cast<QueuePartial*>(w->d_scratch + o_part);
        qp.R = R; qp.M = M; qp.B = B; qp.chunk = chunk_g; qp.n_chunks = n_chunks; qp.qs_stride = qs_stride;
        qp.slo_ttft = p.slo_ttft; qp.slo_tpot = p.slo_tpot;
        w->replay_params = qp;
        w->replay_lds_bytes = kReplayWaves * B * kWave * 4u;
        ReduceParams rd{};
        rd.qs = gp.qs; rd.bins_te = qp.bins_te; rd.bins_p = qp.bins_p; rd.partial = qp.partial; rd.unknown = gp.unknown;
        rd.M = M; rd.chunk = chunk_g; rd.n_chunks = n_chunks; rd.qs_stride = qs_stride;
        w->reduce_params = rd;
        if (hipFuncSetAttribute(hist16 ? reinterpret_cast<const void*>(&k_reduce_candidates<true>)
                                       : reinterpret_cast<const void*>(&k_reduce_candidates<false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)w->reduce_lds_bytes) != hipSuccess)
            return device_error();
    }

    // ---- screening plan: only for identical replicas that are available throughout ------
    bool always_on = true;
    for (const DevReplica& d : dev) always_on = always_on && d.t_on == 0u && d.t_off == kNever;
    w->screen = always_on && kinds.size() == 1 && w->R <= (1u << 30);      // the kernels' byte offsets are 32-bit
    // Screening proves that nobody waits; where the mean number of requests in service per replica (total service time
    // over the trace's span, by Little's law) is a quarter of the slots or more, hardly any candidate will pass, and
    // the trace goes straight to the listed evaluation, which replays every queue.
    const bool crowded = w->span_us == 0 || (double)service_sum / (double)w->span_us / M >= 0.25 * B;
    if (w->screen && crowded && w->d_req8) w->screen = false;
    w->counts = false;
    if (w->screen) {
        const ap_status st = plan_counts(w, worst_service);
        if (st != AP_OK) return st;
    }
    // The one-wavefront screening kernel hands a step's 64 requests to rings of S slots in no particular order: with
    // few replicas and few slots (64 / M requests per ring and step against S slots) a ring wraps within one step
    // and hardly any candidate passes.  Such tables go to the listed evaluation as well.
    {
        bool wide = false;
        const uint32_t S_log2 = narrow_ring_slots_log2(M, B, wide);
        w->small_table = w->screen && !w->counts && !wide && 128u >= M * (1u << S_log2) && w->d_req8;
        if (w->small_table) w->screen = false;
    }
    if (w->screen) {
        ScreenParams sp{};
        sp.span = w->d_span;
        sp.span_t = w->d_span_t;
        sp.pair = w->d_pair;
        // the smallest tick that brings every contention-free finish time below 2^16 ticks
        uint64_t tick_us = std::max<uint64_t>(1u, latest_unqueued / 0xFFFDu);
        while (latest_unqueued / tick_us + 2u > 0xFFFFu) ++tick_us;
        sp.nominal = w->d_nominal;
        sp.R = w->R;
        sp.M = M;
        // Screening slots per replica: a power of two, at most B.  One wavefront per candidate as
        // long as that wavefront's slot state (rings and counters of M + 1 replicas) stays small
        // enough for many wavefronts per compute unit with a useful number of slots; otherwise
        // the eight-wavefront kernel, whose workgroup holds one candidate's rings.
        uint32_t S_log2 = narrow_ring_slots_log2(M, B, w->screen_wide);
        if (w->screen_wide) {
            S_log2 = 0;
            while ((2u << S_log2) <= std::min(B, kWideMaxSlots) && M * (2u << S_log2) * 4u <= kWideLdsBytes) ++S_log2;
        }
        // The eight-wavefront kernel can read one word per pair of requests if the tick is coarse
        // enough for the pair's two tick counts to fit 8 bits (count <= longest_pair / tick + 2).
        // Take that tick when it is not out of proportion: at most twice the other one, or at
        // most an eighth of the mean service time.
        const uint64_t tick_packed = std::max<uint64_t>(tick_us, (longest_pair + 252u) / 253u);
        w->screen_packed = w->screen_wide &&
                           (tick_packed <= 2u * tick_us || tick_packed * 8u <= service_sum / w->R);
        if (w->screen_packed) tick_us = tick_packed;
        sp.slots_log2 = S_log2;
        const uint32_t ring_bytes = 4u << S_log2;
        sp.wave_bytes = ((M + 1u) * (ring_bytes + 4u) + ring_bytes - 1u) / ring_bytes * ring_bytes;
        w->screen_params = sp;
        w->screen_wide_lds_bytes = (((M + 1u) << S_log2) + 4u) * 4u;
        w->screen_lds_bytes = kScreenWaves * sp.wave_bytes;
        // a thread takes two requests per turn; enough workgroups for four turns each, at most one per compute unit
        const uint32_t n_groups = std::max(1u, std::min((uint32_t)n_cu, (w->R + 8u * kThreads - 1u) / (8u * kThreads)));
        if (hipMemsetAsync(w->d_nominal_sums, 0, kNominalSumsBytes, nullptr) != hipSuccess) return device_error();
        hipLaunchKernelGGL(hist16 ? k_nominal_metrics<true> : k_nominal_metrics<false>, dim3(n_groups), dim3(kThreads),
                           reduce_lds, nullptr, w->reduce_eval, w->d_span, w->d_span_t,
                           w->screen_packed ? w->d_pair : nullptr, (uint32_t)tick_us,
                           reinterpret_cast<uint32_t*>(w->d_nominal_sums),
                           reinterpret_cast<unsigned long long*>(w->d_nominal_sums + 3u * kBins * sizeof(uint32_t)), w->d_nominal);
        if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
            (void)hipGetLastError();
            return device_error();
        }
    }
    // ---- streamed and split evaluation: replicas that differ or have windows, crowded traces, small tables ----
    w->split = w->stream = w->stream_settles = false;
    bool tables_ready = true;
    if (!w->screen && tabled && w->d_req8) {
        const ap_status st = pair_tables(w, rep_type, M, tables_ready);
        if (st != AP_OK) return st;
    }
    if (!w->screen && w->d_req8 && tables_ready) {
        const std::vector<uint32_t> depths = service_depths(w, worst_service);
        uint32_t least_bin[3] = {0u, 0u, 0u};
        if (!on_device) {
            std::vector<ap_replica> of_kind;
            std::vector<uint32_t> rows;
            for (uint32_t k : kinds) {
                if (tabled) rows.push_back(rep_type[k]);
                else of_kind.push_back(replicas[k]);
            }
            least_bins(w, std::move(of_kind), rows, tab_prefill, tab_tpot, least_bin);
        }
        if (always_on && !on_device) {
            const uint32_t longest_prompt = (uint32_t)*std::max_element(w->h_prompt.begin(), w->h_prompt.end());
            uint32_t longest[3] = {(uint32_t)table_longest_prefill, (uint32_t)table_longest_tpot, *std::max_element(worst_service.begin(), worst_service.end())};
            for (uint32_t k : kinds)
                if (!tabled) {                               // both grow with the prompt
                    longest[0] = std::max(longest[0], replicas[k].prefill_base_us + replicas[k].prefill_per_tok_us * longest_prompt);
                    longest[1] = std::max(longest[1], replicas[k].decode_base_us + replicas[k].decode_per_kctx_us * ((longest_prompt + 1023u) >> 10));
                }
            std::vector<uint32_t> kind_of(M);
            for (uint32_t m = 0; m < M; ++m)
                for (size_t k = 0; k < kinds.size(); ++k)
                    if (same_kind(kinds[k], m)) kind_of[m] = (uint32_t)k;
            const ap_status st = plan_stream(w, replicas, kinds, kind_of, worst_service, tabled ? rep_type : nullptr, host_cost,
                                             least_bin, longest, depths[0]);
            if (st != AP_OK) return st;
        }
        if (!w->stream_settles) {
            const ap_status st = plan_split(w, w->split_plan, w->split, dev, replicas, kinds, worst_service, kind_sum,
                                            kind_longest, total, tabled ? rep_type : nullptr, table_longest_prefill, table_longest_tpot,
                                            least_bin, depths);
            if (st != AP_OK) return st;
        }
    }
    w->has_model = true;
    return AP_OK;
}

ap_status ap_costmodel_set(ap_workload* w, const ap_replica* replicas, uint32_t M, uint32_t B, const ap_slo* slo) {
    return set_cost_model(w, replicas, M, B, slo, nullptr, nullptr, nullptr, 0u);
}

ap_status ap_costtable_set(ap_workload* w, const ap_typed_replica* replicas, uint32_t M, uint32_t B, const ap_slo* slo,
                           const uint32_t* prefill_us, const uint32_t* tpot_us, uint32_t n_types) {
    if (!w || !replicas || !slo || !prefill_us || !tpot_us || M == 0 || B == 0 || n_types == 0) return AP_ERR_INVALID;
    if (M > AP_MAX_REPLICAS) return AP_ERR_RANGE;
    if ((uint64_t)n_types * w->R > 0xFFFFFFFFull) return AP_ERR_RANGE;      // table offsets are 32-bit on the device
    std::vector<ap_replica> plain;
    std::vector<uint32_t> types;
    try {
        plain.resize(M);
        types.resize(M);
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    for (uint32_t m = 0; m < M; ++m) {
        if (replicas[m].type >= n_types) return AP_ERR_INVALID;
        types[m] = replicas[m].type;
        plain[m] = ap_replica{0u, 0u, 0u, 0u, replicas[m].t_on_us, replicas[m].t_off_us};
    }
    return set_cost_model(w, plain.data(), M, B, slo, types.data(), prefill_us, tpot_us, n_types);
}

ap_status ap_eval_candidates(const ap_workload* w, const uint16_t* d_assign, uint32_t C, ap_metrics* d_out,
                             void* hip_stream) {
    if (!w) return AP_ERR_INVALID;
    if (!w->has_model) return AP_ERR_STATE;
    if (C == 0) return AP_OK;
    if (!d_assign || !d_out) return AP_ERR_INVALID;
    w->n_scored += C;
    return launch_dense(w, d_assign, C, d_out, static_cast<hipStream_t>(hip_stream), false, take_pending_word(w));
}

// What a call of C rows goes through, for tests that have to know which kernels they reach (not part of the header):
//   [0] bucket size of the counting screen in requests (0: not launched), [1] its columns, [2] its wavefronts per row;
//   [3] wavefronts per row of the slot rings (0: none);
//   [4] streamed evaluation: 0 none, 1 counts, 2 has nothing to count; [5] bucket size of its counts;
//   [6] behind that (or first): 0 no lists, 1 every request listed, 2 a listed and a streamed part, 3 the fused replay instead.
ap_status ap_route_get(const ap_workload* w, uint32_t C, uint32_t out[7]) {
    if (!w || !out) return AP_ERR_INVALID;
    if (!w->has_model) return AP_ERR_STATE;
    const bool counts = counts_first(w, C);
    out[0] = counts ? 1u << w->count_params.w_log2 : 0u;
    out[1] = counts ? 1u << w->count_params.columns_log2 : 0u;
    out[2] = counts ? count_waves_per_row(w, C) : 0u;
    out[3] = !w->screen ? 0u : w->screen_wide ? kWideWaves : 1u;
    out[4] = !w->stream ? 0u : w->stream_settles ? 2u : 1u;
    out[5] = w->stream && !w->stream_settles ? 1u << w->stream_params.w_log2 : 0u;
    out[6] = fused_replay(w, C) ? 3u : !w->split ? 0u : w->split_plan.params.any_streamed != 0u ? 2u : 1u;
    return AP_OK;
}

ap_status ap_eval_counts_get(const ap_workload* w, ap_eval_counts* out) {
    if (!w || !out) return AP_ERR_INVALID;
    if (!w->has_model) return AP_ERR_STATE;
    uint32_t replayed = 0;
    if (hipSetDevice(w->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(&replayed, w->d_pending + 2, sizeof(uint32_t), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    out->candidates = w->n_scored;
    out->replayed = replayed;
    return AP_OK;
}

ap_status ap_parent_set(ap_workload* w, const uint16_t* parent, uint32_t max_children) {
    if (!w || !parent || max_children == 0) return AP_ERR_INVALID;
    if (!w->has_model) return AP_ERR_STATE;
    if (hipSetDevice(w->device) != hipSuccess) return device_error();
    w->has_parent = false;
    if ((uint64_t)max_children > (UINT64_MAX / sizeof(uint16_t)) / w->R) return AP_ERR_ALLOC;     // the rows cannot exist
    const size_t need = (size_t)max_children * w->R * sizeof(uint16_t);
    const size_t row_bytes = (size_t)w->R * sizeof(uint16_t), peak_bytes = sizeof(uint32_t) * (AP_MAX_REPLICAS + 1u);
    if ((!w->d_parent && hipMalloc(&w->d_parent, row_bytes + 16u) != hipSuccess) ||
        (!w->d_peak && hipMalloc(&w->d_peak, peak_bytes) != hipSuccess) ||
        (!w->d_room && hipMalloc(&w->d_room, sizeof(uint32_t) * AP_MAX_REPLICAS) != hipSuccess) ||
        (!w->h_stage && hipHostMalloc(reinterpret_cast<void**>(&w->h_stage), std::max(row_bytes, peak_bytes), hipHostMallocDefault) != hipSuccess)) {
        (void)hipGetLastError();
        return AP_ERR_ALLOC;
    }
    if (need > w->rows_bytes) {
        if (w->d_rows && hipFree(w->d_rows) != hipSuccess) return device_error();
        w->d_rows = nullptr;
        w->rows_bytes = 0;
        if (hipMalloc(&w->d_rows, need) != hipSuccess) {
            (void)hipGetLastError();
            return AP_ERR_ALLOC;
        }
        w->rows_bytes = need;
    }
    // through the pinned buffer: upload, analysis and read-back are queued together and waited for once
    std::memcpy(w->h_stage, parent, row_bytes);
    if (hipMemcpyAsync(w->d_parent, w->h_stage, row_bytes, hipMemcpyHostToDevice, nullptr) != hipSuccess) return device_error();
    const uint32_t M = w->params.M;
    bool certify = false;
    if (w->screen) {
        // the shortcut needs the nominal record, i.e. identical replicas that are always available
        hipLaunchKernelGGL(k_parent_occupancy, dim3(M), dim3(kOccupancyThreads), 0, nullptr, w->params, w->d_parent, w->d_peak,
                           w->d_room);
        // (the kernel is queued behind the upload, which has therefore read the pinned buffer before the depths land in it)
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(w->h_stage, w->d_peak, sizeof(uint32_t) * (M + 1u), hipMemcpyDeviceToHost, nullptr) != hipSuccess ||
            hipStreamSynchronize(nullptr) != hipSuccess) {
            (void)hipGetLastError();
            return device_error();
        }
        const uint32_t* peak = reinterpret_cast<const uint32_t*>(w->h_stage);
        // ... and a parent that is contention-free itself and names only replicas of the table
        certify = peak[M] == 0u;
        for (uint32_t m = 0; m < M; ++m) certify = certify && peak[m] <= w->params.B;
    } else if (hipStreamSynchronize(nullptr) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    ChildParams cp{};
    cp.parent = w->d_parent;
    cp.room = w->d_room;
    cp.nominal = w->d_nominal;
    cp.rows = w->d_rows;
    cp.R = w->R;
    cp.M = M;
    cp.key_bits = 0;
    while (((w->R - 1u) >> cp.key_bits) != 0u) ++cp.key_bits;
    cp.certify = certify ? 1u : 0u;
    w->child_params = cp;
    w->max_children = max_children;
    w->has_parent = true;
    return AP_OK;
}

ap_status ap_eval_children(const ap_workload* w, const uint32_t* d_edit_first, const uint32_t* d_edit_request,
                           const uint16_t* d_edit_replica, uint32_t C, ap_metrics* d_out, void* hip_stream) {
    if (!w) return AP_ERR_INVALID;
    if (!w->has_model || !w->has_parent) return AP_ERR_STATE;
    if (C == 0) return AP_OK;
    if (!d_edit_first || !d_edit_request || !d_edit_replica || !d_out) return AP_ERR_INVALID;
    if (C > w->max_children) return AP_ERR_RANGE;
    w->n_scored += C;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const PendingWord flags = take_pending_word(w);
    if (w->child_params.certify != 0u) {
        const uint32_t blocks = std::min((C + kChildWaves - 1u) / kChildWaves, w->n_cu * 64u);
        hipLaunchKernelGGL(k_certify_children, dim3(blocks), dim3(kChildThreads), (kChildWaves + 1u) * w->child_params.M * 4u, stream,
                           w->child_params, d_edit_first, d_edit_request, d_edit_replica, d_out, C, flags);
    } else {
        hipLaunchKernelGGL(k_write_children, dim3(std::min(C, w->n_cu * 64u)), dim3(kRowThreads), 0, stream, w->child_params,
                           d_edit_first, d_edit_request, d_edit_replica, C, flags);
    }
    if (hipGetLastError() != hipSuccess) return device_error();
    return launch_dense(w, w->d_rows, C, d_out, stream, w->child_params.certify != 0u, flags);
}

// ---- roofline cost tables -------------------------------------------------------------
namespace {

// Validate the descriptions and run the table kernels; leaves prefill_ns / prefix_ns / weight_bytes /
// feasible filled on the device.
ap_status roofline_tables_on_device(const ap_model* models, uint32_t n_models, const ap_gpu* gpus, uint32_t n_gpus,
                                    const ap_group* groups, uint32_t n_groups, uint32_t max_seq, RoofBuffers& buf) {
    if (!models || !gpus || !groups || n_models == 0 || n_gpus == 0 || n_groups == 0 || max_seq == 0) return AP_ERR_INVALID;
    if (n_groups > 65535u || max_seq > (1u << 24)) return AP_ERR_RANGE;
    std::vector<RoofGroup> host;
    try {
        host.resize(n_groups);
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    for (uint32_t i = 0; i < n_groups; ++i) {
        const ap_group& gr = groups[i];
        if (gr.model >= n_models || gr.gpu >= n_gpus || gr.tp == 0 || gr.batch == 0) return AP_ERR_INVALID;
        const ap_model& m = models[gr.model];
        const ap_gpu& g = gpus[gr.gpu];
        if (m.layers == 0 || m.hidden == 0 || m.intermediate == 0 || m.vocab == 0 || m.heads == 0 || m.kv_heads == 0 ||
            m.kv_heads > m.heads || m.weight_bits == 0)
            return AP_ERR_INVALID;
        if (!(g.flops > 0.0) || !(g.hbm_bytes_per_s > 0.0) || !(g.mem_bytes > 0.0) || g.gpus_per_node == 0 ||
            !(g.link_intra_bytes_per_s > 0.0) || !(g.link_inter_bytes_per_s > 0.0))
            return AP_ERR_INVALID;
        RoofGroup& o = host[i];
        o.L = m.layers; o.H = m.hidden; o.I = m.intermediate; o.V = m.vocab; o.A = m.heads; o.K = m.kv_heads;
        o.e = (double)m.weight_bits / 8.0;
        o.b = gr.batch; o.t = gr.tp;
        o.flops = g.flops; o.hbm = g.hbm_bytes_per_s;
        o.link = gr.tp <= g.gpus_per_node ? g.link_intra_bytes_per_s : g.link_inter_bytes_per_s;
        o.mem = g.mem_bytes;
    }
    const size_t per_group = (size_t)max_seq + 1u;
    if (n_groups > buf.cap_groups || max_seq > buf.cap_seq) {
        buf.release();
        if (hipMalloc(&buf.groups, sizeof(RoofGroup) * n_groups) != hipSuccess ||
            hipMalloc(&buf.prefill_ns, 8u * per_group * n_groups) != hipSuccess ||
            hipMalloc(&buf.step_ns, 8u * per_group * n_groups) != hipSuccess ||
            hipMalloc(&buf.prefix_ns, 8u * (per_group + 1u) * n_groups) != hipSuccess ||
            hipMalloc(&buf.weight_bytes, 8u * n_groups) != hipSuccess || hipMalloc(&buf.feasible, 4u * n_groups) != hipSuccess) {
            (void)hipGetLastError();
            buf.release();
            return AP_ERR_ALLOC;
        }
        buf.cap_groups = n_groups;
        buf.cap_seq = max_seq;
    }
    if (hipMemcpy(buf.groups, host.data(), sizeof(RoofGroup) * n_groups, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    hipLaunchKernelGGL(k_roofline_steps, dim3((max_seq + kRoofThreads) / kRoofThreads, n_groups), dim3(kRoofThreads), 0, nullptr,
                       buf.groups, n_groups, max_seq, buf.prefill_ns, buf.step_ns, buf.weight_bytes, buf.feasible);
    hipLaunchKernelGGL(k_roofline_prefix, dim3(n_groups), dim3(kRoofThreads), 0, nullptr, buf.step_ns, max_seq, buf.prefix_ns);
    if (hipGetLastError() != hipSuccess) return device_error();
    return AP_OK;
}

}  // namespace

ap_status ap_costtable_set_roofline(ap_workload* w, const ap_typed_replica* replicas, uint32_t M, uint32_t B,
                                    const ap_slo* slo, const ap_model* models, uint32_t n_models, const ap_gpu* gpus,
                                    uint32_t n_gpus, const ap_group* groups, uint32_t n_groups) {
    if (!w || !replicas || !slo || M == 0 || B == 0 || n_groups == 0) return AP_ERR_INVALID;
    if (M > AP_MAX_REPLICAS) return AP_ERR_RANGE;
    if ((uint64_t)n_groups * w->R > 0xFFFFFFFFull) return AP_ERR_RANGE;     // table offsets are 32-bit on the device
    if (hipSetDevice(w->device) != hipSuccess) return device_error();
    std::vector<ap_replica> plain;
    std::vector<uint32_t> types;
    try {
        plain.resize(M);
        types.resize(M);
        if (!w->roof) w->roof = new RoofBuffers;
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    for (uint32_t m = 0; m < M; ++m) {
        if (replicas[m].type >= n_groups) return AP_ERR_INVALID;
        types[m] = replicas[m].type;
        plain[m] = ap_replica{0u, 0u, 0u, 0u, replicas[m].t_on_us, replicas[m].t_off_us};
    }
    uint64_t longest = 0;                                  // prompt + output of the longest request
    for (uint32_t r = 0; r < w->R; ++r) longest = std::max<uint64_t>(longest, (uint64_t)w->h_prompt[r] + (uint64_t)w->h_out[r]);
    if (longest > (1u << 24)) return AP_ERR_RANGE;
    const ap_status st = roofline_tables_on_device(models, n_models, gpus, n_gpus, groups, n_groups, (uint32_t)longest, *w->roof);
    if (st != AP_OK) return st;
    // from here on the previous cost model is gone: the tables it may have read are overwritten
    w->has_model = false;
    const size_t entries = (size_t)n_groups * w->R;
    if (entries > w->tab_entries) {
        if ((w->d_tab_prefill && hipFree(w->d_tab_prefill) != hipSuccess) || (w->d_tab_tpot && hipFree(w->d_tab_tpot) != hipSuccess)) {
            (void)hipGetLastError();
            return device_error();
        }
        w->d_tab_prefill = w->d_tab_tpot = nullptr;
        w->tab_entries = 0;
        if (hipMalloc(&w->d_tab_prefill, entries * 4u) != hipSuccess || hipMalloc(&w->d_tab_tpot, entries * 4u) != hipSuccess) {
            (void)hipGetLastError();
            return AP_ERR_ALLOC;
        }
        w->tab_entries = entries;
    }
    if (!w->d_bounds && hipMalloc(&w->d_bounds, sizeof(TableBounds) + 4u * AP_MAX_REPLICAS) != hipSuccess) {
        (void)hipGetLastError();
        return AP_ERR_ALLOC;
    }
    hipLaunchKernelGGL(k_roofline_request_costs, dim3((w->R + kRoofThreads - 1u) / kRoofThreads, n_groups), dim3(kRoofThreads),
                       0, nullptr, w->roof->prefill_ns, w->roof->prefix_ns, (uint32_t)longest, w->d_prompt, w->d_out, w->R,
                       w->d_tab_prefill, w->d_tab_tpot);
    if (hipGetLastError() != hipSuccess) return device_error();
    return set_cost_model(w, plain.data(), M, B, slo, types.data(), nullptr, nullptr, n_groups);
}

ap_status ap_roofline_tables(const ap_model* models, uint32_t n_models, const ap_gpu* gpus, uint32_t n_gpus,
                             const ap_group* groups, uint32_t n_groups, uint32_t max_seq, uint64_t* prefill_ns,
                             uint64_t* decode_prefix_ns, double* weight_bytes, uint8_t* feasible) {
    if (!prefill_ns || !decode_prefix_ns || !weight_bytes || !feasible) return AP_ERR_INVALID;
    RoofBuffers buf;
    const ap_status st = roofline_tables_on_device(models, n_models, gpus, n_gpus, groups, n_groups, max_seq, buf);
    if (st != AP_OK) return st;
    std::vector<uint32_t> ok;
    try {
        ok.resize(n_groups);
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    const size_t per_group = (size_t)max_seq + 1u;
    if (hipMemcpy(prefill_ns, buf.prefill_ns, 8u * per_group * n_groups, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(decode_prefix_ns, buf.prefix_ns, 8u * (per_group + 1u) * n_groups, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(weight_bytes, buf.weight_bytes, 8u * n_groups, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(ok.data(), buf.feasible, 4u * n_groups, hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    for (uint32_t i = 0; i < n_groups; ++i) feasible[i] = ok[i] ? 1u : 0u;
    return AP_OK;
}

ap_status ap_roofline_costs(const ap_workload* w, const ap_model* models, uint32_t n_models, const ap_gpu* gpus,
                            uint32_t n_gpus, const ap_group* groups, uint32_t n_groups, uint32_t* prefill_us,
                            uint32_t* tpot_us) {
    if (!w || !prefill_us || !tpot_us) return AP_ERR_INVALID;
    if (hipSetDevice(w->device) != hipSuccess) return device_error();
    uint64_t longest = 0;                                  // prompt + output of the longest request
    for (uint32_t r = 0; r < w->R; ++r) longest = std::max<uint64_t>(longest, (uint64_t)w->h_prompt[r] + (uint64_t)w->h_out[r]);
    if (longest > (1u << 24)) return AP_ERR_RANGE;
    RoofBuffers buf;
    const ap_status st = roofline_tables_on_device(models, n_models, gpus, n_gpus, groups, n_groups, (uint32_t)longest, buf);
    if (st != AP_OK) return st;
    const size_t entries = (size_t)n_groups * w->R;
    if (hipMalloc(&buf.prefill_us, 4u * entries) != hipSuccess || hipMalloc(&buf.tpot_us, 4u * entries) != hipSuccess) {
        (void)hipGetLastError();
        return AP_ERR_ALLOC;
    }
    hipLaunchKernelGGL(k_roofline_request_costs, dim3((w->R + kRoofThreads - 1u) / kRoofThreads, n_groups), dim3(kRoofThreads),
                       0, nullptr, buf.prefill_ns, buf.prefix_ns, (uint32_t)longest, w->d_prompt, w->d_out, w->R, buf.prefill_us,
                       buf.tpot_us);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpy(prefill_us, buf.prefill_us, 4u * entries, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(tpot_us, buf.tpot_us, 4u * entries, hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    return AP_OK;
}

ap_status ap_trace_time(const ap_model* models, const double* pcie_coef, uint32_t n_models, const ap_gpu* gpus, uint32_t n_gpus,
                        const ap_placement* d_plans, const uint32_t* d_n_intervals, const uint64_t* d_sched_ns,
                        const uint64_t* d_stale_ns, const uint64_t* d_serve_ns, uint32_t C, uint32_t N_max,
                        uint32_t load_scope, ap_breakdown* d_out, void* hip_stream) {
    if (!models || !pcie_coef || !gpus || n_models == 0 || n_gpus == 0 || N_max == 0) return AP_ERR_INVALID;
    if (load_scope != AP_LOAD_DEPLOYED && load_scope != AP_LOAD_CHANGED) return AP_ERR_INVALID;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (C == 0) return AP_OK;
    if (!d_plans || !d_n_intervals || !d_sched_ns || !d_stale_ns || !d_serve_ns || !d_out) return AP_ERR_INVALID;
    if ((uint64_t)n_models * n_gpus > (1u << 20)) return AP_ERR_RANGE;
    std::vector<RoofGroup> host;
    std::vector<double> pcie;
    try {
        host.resize(n_models);
        pcie.resize(n_gpus);
    } catch (const std::bad_alloc&) {
        return AP_ERR_ALLOC;
    }
    for (uint32_t z = 0; z < n_models; ++z) {
        const ap_model& m = models[z];
        if (m.layers == 0 || m.hidden == 0 || m.intermediate == 0 || m.vocab == 0 || m.heads == 0 || m.kv_heads == 0 ||
            m.kv_heads > m.heads || m.weight_bits == 0 || !(pcie_coef[z] > 0.0))
            return AP_ERR_INVALID;
        RoofGroup o{};
        o.L = m.layers; o.H = m.hidden; o.I = m.intermediate; o.V = m.vocab; o.A = m.heads; o.K = m.kv_heads;
        o.e = (double)m.weight_bits / 8.0;
        host[z] = o;
    }
    for (uint32_t g = 0; g < n_gpus; ++g) {
        if (!(gpus[g].pcie_bytes_per_s > 0.0)) return AP_ERR_INVALID;
        pcie[g] = gpus[g].pcie_bytes_per_s;
    }
    struct Temp {
        RoofGroup* models = nullptr;
        double* coef = nullptr;
        double* pcie = nullptr;
        unsigned long long* tau = nullptr;
        ~Temp() {
            for (void* q : {(void*)models, (void*)coef, (void*)pcie, (void*)tau})
                if (q) (void)hipFree(q);
        }
    } tmp;
    if (hipMalloc(&tmp.models, sizeof(RoofGroup) * n_models) != hipSuccess || hipMalloc(&tmp.coef, 8u * n_models) != hipSuccess ||
        hipMalloc(&tmp.pcie, 8u * n_gpus) != hipSuccess || hipMalloc(&tmp.tau, 8u * (size_t)n_models * n_gpus) != hipSuccess) {
        (void)hipGetLastError();
        return AP_ERR_ALLOC;
    }
    // the descriptions are on the device when these copies return; the kernels then run on the caller's stream,
    // behind whatever produced the device inputs there
    if (hipMemcpy(tmp.models, host.data(), sizeof(RoofGroup) * n_models, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(tmp.coef, pcie_coef, 8u * n_models, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(tmp.pcie, pcie.data(), 8u * n_gpus, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    hipLaunchKernelGGL(k_transfer_times, dim3((n_models * n_gpus + kRoofThreads - 1u) / kRoofThreads), dim3(kRoofThreads), 0, stream,
                       tmp.models, tmp.coef, n_models, tmp.pcie, n_gpus, tmp.tau);
    TraceTimeParams tp{};
    tp.tau_ns = tmp.tau;
    tp.plans = d_plans;
    tp.n_intervals = d_n_intervals;
    tp.sched_ns = reinterpret_cast<const unsigned long long*>(d_sched_ns);
    tp.stale_ns = reinterpret_cast<const unsigned long long*>(d_stale_ns);
    tp.serve_ns = reinterpret_cast<const unsigned long long*>(d_serve_ns);
    tp.C = C; tp.N_max = N_max; tp.Z = n_models; tp.G = n_gpus;
    tp.load_changed_only = load_scope == AP_LOAD_CHANGED ? 1u : 0u;
    hipLaunchKernelGGL(k_trace_time, dim3((C + kRoofThreads - 1u) / kRoofThreads), dim3(kRoofThreads), 0, stream, tp, d_out);
    // the temporary tables are freed on return: wait for the stream
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(stream) != hipSuccess) {
        (void)hipGetLastError();
        return device_error();
    }
    return AP_OK;
}

// ---- trace time for callers that cannot allocate ------------------------------------------
// The transfer-time table of ap_trace_time_static lives in this array (one copy per device, held until the
// process ends).  In host code the array's name is only a stand-in for the symbol: its device address is asked
// for once per device and kept in trace_scratch_at.
static __device__ __align__(256) unsigned long long scratch[kTransferArgModels * kTransferArgGpus];
constexpr int kScratchDevices = 64;
static unsigned long long* trace_scratch_at[kScratchDevices] = {};
static std::mutex trace_scratch_lock;

ap_status ap_trace_time_static(const ap_model* models, const double* pcie_coef, uint32_t n_models, const ap_gpu* gpus,
                               uint32_t n_gpus, const ap_placement* d_plans, const uint32_t* d_n_intervals,
                               const uint64_t* d_sched_ns, const uint64_t* d_stale_ns, const uint64_t* d_serve_ns, uint32_t C,
                               uint32_t N_max, uint32_t load_scope, ap_breakdown* d_out, void* hip_stream) {
    if (!models || !pcie_coef || !gpus || n_models == 0 || n_gpus == 0 || N_max == 0) return AP_ERR_INVALID;
    if (load_scope != AP_LOAD_DEPLOYED && load_scope != AP_LOAD_CHANGED) return AP_ERR_INVALID;
    if (n_models > AP_STATIC_MAX_MODELS || n_gpus > AP_STATIC_MAX_GPU_TYPES) return AP_ERR_RANGE;
    if (C == 0) return AP_OK;
    if (!d_plans || !d_n_intervals || !d_sched_ns || !d_stale_ns || !d_serve_ns || !d_out) return AP_ERR_INVALID;
    TransferArgs args{};
    for (uint32_t z = 0; z < n_models; ++z) {
        const ap_model& m = models[z];
        if (m.layers == 0 || m.hidden == 0 || m.intermediate == 0 || m.vocab == 0 || m.heads == 0 || m.kv_heads == 0 ||
            m.kv_heads > m.heads || m.weight_bits == 0 || !(pcie_coef[z] > 0.0))
            return AP_ERR_INVALID;
        args.model[z] = m;
        args.coef[z] = pcie_coef[z];
    }
    for (uint32_t g = 0; g < n_gpus; ++g) {
        if (!(gpus[g].pcie_bytes_per_s > 0.0)) return AP_ERR_INVALID;
        args.pcie[g] = gpus[g].pcie_bytes_per_s;
    }
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return device_error();
    if (device < 0 || device >= kScratchDevices) return AP_ERR_RANGE;
    unsigned long long* tau = nullptr;
    {
        std::lock_guard<std::mutex> hold(trace_scratch_lock);
        if (!trace_scratch_at[device]) {                      // the first call on this device, which is current
            void* at = nullptr;
            if (hipGetSymbolAddress(&at, HIP_SYMBOL(scratch)) != hipSuccess || !at) {
                (void)hipGetLastError();
                return device_error();
            }
            trace_scratch_at[device] = static_cast<unsigned long long*>(at);
        }
        tau = trace_scratch_at[device];
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // every entry the second kernel reads is written by the first: nothing of an earlier call is looked at
    hipLaunchKernelGGL(k_transfer_times_from_args, dim3((n_models * n_gpus + kRoofThreads - 1u) / kRoofThreads), dim3(kRoofThreads), 0,
                       stream, args, n_models, n_gpus, tau);
    TraceTimeParams tp{};
    tp.tau_ns = tau;
    tp.plans = d_plans;
    tp.n_intervals = d_n_intervals;
    tp.sched_ns = reinterpret_cast<const unsigned long long*>(d_sched_ns);
    tp.stale_ns = reinterpret_cast<const unsigned long long*>(d_stale_ns);
    tp.serve_ns = reinterpret_cast<const unsigned long long*>(d_serve_ns);
    tp.C = C; tp.N_max = N_max; tp.Z = n_models; tp.G = n_gpus;
    tp.load_changed_only = load_scope == AP_LOAD_CHANGED ? 1u : 0u;
    hipLaunchKernelGGL(k_trace_time, dim3((C + kRoofThreads - 1u) / kRoofThreads), dim3(kRoofThreads), 0, stream, tp, d_out);
    if (hipGetLastError() != hipSuccess) return device_error();
    return AP_OK;
}

// ---- agentic workflows ------------------------------------------------------------------
struct ap_agentic {
    int device = 0;
    AgenticParams params{};
    uint32_t lds_bytes = 0;
    uint32_t n_cu = 0;
    uint32_t chunks = 0;              // which kernel
    uint32_t waves = 0;               // wavefronts (candidates) per workgroup
    uint32_t row_waves = 0, row_lds_bytes = 0;   // k_agentic_rows; 0: it does not apply
    uint32_t wave_plans = 0, row_plans = 0;      // how many plans a compute unit's LDS holds, by either kernel (the latter: its registers too)
    void* d_block = nullptr;          // one allocation behind all the tables
};

typedef void (*agentic_fn)(AgenticParams, const uint16_t*, const uint16_t*, const uint32_t*, ap_agentic_metrics*, uint32_t);
static uint32_t agentic_chunks(uint32_t K) {
    const uint32_t n = (K + kWave - 1u) / kWave;
    return n <= 4u ? n : n <= 6u ? 6u : n <= 8u ? 8u : n <= 12u ? 12u : 16u;
}
static agentic_fn agentic_kernel(uint32_t chunks) {
    return chunks == 1u ? k_agentic_eval<1u> : chunks == 2u ? k_agentic_eval<2u> : chunks == 3u ? k_agentic_eval<3u>
           : chunks == 4u ? k_agentic_eval<4u> : chunks == 6u ? k_agentic_eval<6u> : chunks == 8u ? k_agentic_eval<8u>
           : chunks == 12u ? k_agentic_eval<12u> : k_agentic_eval<16u>;
}

ap_status ap_agentic_create(const uint64_t* arrival_us, const uint64_t* slo_us, uint32_t W, const uint32_t* wf,
                            const uint32_t* in_len, const uint32_t* out_len, const uint32_t* pred_first, const uint32_t* pred,
                            uint32_t K, const ap_prefill_instance* prefill, uint32_t P, const ap_decode_instance* decode,
                            uint32_t Q, uint64_t penalty_permille, ap_agentic** out) {
    if (!arrival_us || !slo_us || !wf || !in_len || !out_len || !pred_first || !prefill || !decode || !out || W == 0 || K == 0 ||
        P == 0 || Q == 0)
        return AP_ERR_INVALID;
    if (W > AP_AGENTIC_MAX_WORKFLOWS || K > AP_AGENTIC_MAX_CALLS || P > AP_AGENTIC_MAX_INSTANCES || Q > AP_AGENTIC_MAX_INSTANCES)
        return AP_ERR_RANGE;
    if (pred_first[0] != 0u) return AP_ERR_INVALID;
    for (uint32_t k = 0; k < K; ++k) {
        if (wf[k] >= W || in_len[k] == 0 || out_len[k] == 0 || pred_first[k + 1u] < pred_first[k]) return AP_ERR_INVALID;
        if (pred_first[k + 1u] > pred_first[k] && !pred) return AP_ERR_INVALID;
        for (uint32_t i = pred_first[k]; i < pred_first[k + 1u]; ++i)
            if (pred[i] >= k || wf[pred[i]] != wf[k]) return AP_ERR_INVALID;
    }
    uint64_t first = arrival_us[0], last = arrival_us[0];
    for (uint32_t w = 0; w < W; ++w) {
        if (slo_us[w] == 0) return AP_ERR_INVALID;
        first = std::min(first, arrival_us[w]);
        last = std::max(last, arrival_us[w]);
    }
    for (uint32_t i = 0; i < P; ++i)
        if ((uint64_t)prefill[i].base_us + prefill[i].per_tok_us == 0) return AP_ERR_INVALID;
    for (uint32_t i = 0; i < Q; ++i)
        if ((uint64_t)decode[i].base_us + decode[i].per_kctx_us == 0) return AP_ERR_INVALID;
    // 32-bit time: no completion can lie beyond the last arrival plus every call's slowest stages in a row
    const uint64_t limit = (uint64_t)kNever - 1u;
    uint64_t total = last - first;
    if (total > limit) return AP_ERR_RANGE;
    for (uint32_t k = 0; k < K; ++k) {
        uint64_t slow_pre = 0, slow_dec = 0;
        for (uint32_t i = 0; i < P; ++i)
            slow_pre = std::max<uint64_t>(slow_pre, (uint64_t)prefill[i].base_us + (uint64_t)prefill[i].per_tok_us * in_len[k]);
        for (uint32_t i = 0; i < Q; ++i)
            slow_dec = std::max<uint64_t>(slow_dec, (uint64_t)out_len[k] * ((uint64_t)decode[i].base_us +
                                                    (uint64_t)decode[i].per_kctx_us * (((uint64_t)in_len[k] + 1023u) >> 10)));
        if (slow_pre > limit || slow_dec > limit) return AP_ERR_RANGE;
        total += slow_pre + slow_dec;
        if (total > limit) return AP_ERR_RANGE;
        if ((uint64_t)in_len[k] + out_len[k] > limit) return AP_ERR_RANGE;
    }

    ap_agentic* a = new (std::nothrow) ap_agentic;
    if (!a) return AP_ERR_ALLOC;
    ap_status st = AP_OK;
    const uint32_t n_pred = pred_first[K];
    std::vector<uint32_t> rel, pa, pb, qc, qd, cap;
    try {
        rel.resize(W); pa.resize(P); pb.resize(P); qc.resize(Q); qd.resize(Q); cap.resize(Q);
    } catch (const std::bad_alloc&) {
        delete a;
        return AP_ERR_ALLOC;
    }
    for (uint32_t w = 0; w < W; ++w) rel[w] = (uint32_t)(arrival_us[w] - first);
    // the kernel counts down a call's outstanding predecessors, so it wants the lists the other way round
    std::vector<uint32_t> n_pred_of, succ_first, succ;
    try {
        n_pred_of.assign(K, 0u);
        succ_first.assign(K + 1u, 0u);
        succ.assign(std::max(1u, n_pred), 0u);
    } catch (const std::bad_alloc&) {
        delete a;
        return AP_ERR_ALLOC;
    }
    try {                                                   // the temporaries below allocate
        for (uint32_t k = 0; k < K; ++k) {
            // a predecessor listed twice counts once: keep distinct ones
            std::vector<uint32_t> mine(pred + pred_first[k], pred + pred_first[k + 1u]);
            std::sort(mine.begin(), mine.end());
            mine.erase(std::unique(mine.begin(), mine.end()), mine.end());
            if (mine.size() > 255u) { delete a; return AP_ERR_RANGE; }
            n_pred_of[k] = (uint32_t)mine.size();
            for (uint32_t j : mine) ++succ_first[j + 1u];
        }
        for (uint32_t k = 0; k < K; ++k) succ_first[k + 1u] += succ_first[k];
        {
            std::vector<uint32_t> fill(succ_first.begin(), succ_first.end() - 1);
            for (uint32_t k = 0; k < K; ++k) {
                std::vector<uint32_t> mine(pred + pred_first[k], pred + pred_first[k + 1u]);
                std::sort(mine.begin(), mine.end());
                mine.erase(std::unique(mine.begin(), mine.end()), mine.end());
                for (uint32_t j : mine) succ[fill[j]++] = k;
            }
        }
    } catch (const std::bad_alloc&) {
        delete a;
        return AP_ERR_ALLOC;
    }
    for (uint32_t i = 0; i < P; ++i) { pa[i] = prefill[i].base_us; pb[i] = prefill[i].per_tok_us; }
    for (uint32_t i = 0; i < Q; ++i) { qc[i] = decode[i].base_us; qd[i] = decode[i].per_kctx_us; cap[i] = decode[i].capacity_tokens; }
    // what every workgroup keeps in LDS, laid out as it is copied there
    std::vector<unsigned char> blob;
    AgenticParams& p = a->params;
    try {
        std::vector<uint32_t> by_arrival(W);
        for (uint32_t w = 0; w < W; ++w) by_arrival[w] = w;
        std::stable_sort(by_arrival.begin(), by_arrival.end(), [&](uint32_t x, uint32_t y) { return rel[x] < rel[y]; });
        std::vector<uint16_t> root;                              // calls without predecessors, workflow by workflow in order of arrival
        std::vector<uint32_t> start(4u * ((size_t)W + 1u), 0u), n_roots(W, 0u), fill(W, 0u);
        for (uint32_t k = 0; k < K; ++k) n_roots[wf[k]] += n_pred_of[k] == 0u ? 1u : 0u;
        uint32_t n_root = 0;
        for (uint32_t i = 0; i < W; ++i) {
            const uint32_t w = by_arrival[i];
            start[4u * i] = rel[w];
            start[4u * i + 1u] = fill[w] = n_root;
            start[4u * i + 2u] = n_roots[w];
            start[4u * i + 3u] = w;
            n_root += n_roots[w];
        }
        start[4u * W] = kNever;
        root.assign(std::max(1u, n_root), 0u);
        for (uint32_t k = 0; k < K; ++k)
            if (n_pred_of[k] == 0u) root[fill[wf[k]]++] = (uint16_t)k;
        std::vector<uint16_t> succ16(succ.begin(), succ.begin() + std::max(1u, succ_first[K]));
        std::vector<unsigned char> left(n_pred_of.begin(), n_pred_of.end());
        std::vector<uint32_t> info(4u * (size_t)K);
        for (uint32_t k = 0; k < K; ++k) {
            info[4u * k] = in_len[k];
            info[4u * k + 1u] = out_len[k];
            const uint32_t n = succ_first[k + 1u] - succ_first[k];
            info[4u * k + 2u] = n == 1u ? succ[succ_first[k]] : succ_first[k];
            info[4u * k + 3u] = wf[k] | (n << 16);               // both at most 1023
        }
        auto put = [&](const void* src, size_t n) {
            const uint32_t at = (uint32_t)blob.size();
            blob.resize((blob.size() + n + 15u) / 16u * 16u, 0u);
            std::memcpy(blob.data() + at, src, n);
            return at;
        };
        p.o_info = put(info.data(), 4u * info.size());
        p.o_start = put(start.data(), 4u * start.size());
        p.o_arrival = put(rel.data(), 4u * (size_t)W);
        p.o_root = put(root.data(), 2u * root.size());
        p.o_n_pred = put(left.data(), left.size());
        p.blob_bytes = (uint32_t)blob.size();
        const uint32_t o_succ = put(succ16.data(), 2u * succ16.size());
        p.o_succ = succ16.size() <= kAgenticLdsSuccessors ? o_succ : 0u;      // not 0: it is never the first piece
        if (p.o_succ != 0u) p.blob_bytes = (uint32_t)blob.size();
        p.succ = reinterpret_cast<const uint16_t*>((size_t)o_succ);           // the device address once there is one
    } catch (const std::bad_alloc&) {
        delete a;
        return AP_ERR_ALLOC;
    }
    // one block on the device: the blob, the objectives (8-byte entries), the instances
    const size_t o_slo = blob.size(), o_inst = o_slo + 8u * (size_t)W, bytes = o_inst + 4u * (2u * (size_t)P + 3u * (size_t)Q);
    if (hipGetDevice(&a->device) != hipSuccess) st = AP_ERR_DEVICE;
    if (st == AP_OK && hipMalloc(&a->d_block, bytes) != hipSuccess) st = AP_ERR_ALLOC;
    int n_cu = 0, lds_cap = 0;
    if (st == AP_OK && (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, a->device) != hipSuccess ||
                        hipDeviceGetAttribute(&lds_cap, hipDeviceAttributeMaxSharedMemoryPerBlock, a->device) != hipSuccess))
        st = AP_ERR_DEVICE;
    if (st == AP_OK) {
        unsigned char* base = static_cast<unsigned char*>(a->d_block);
        uint32_t* at = reinterpret_cast<uint32_t*>(base + o_inst);
        auto put = [&](const uint32_t* src, size_t n) {
            uint32_t* here = at;
            if (n && hipMemcpy(here, src, 4u * n, hipMemcpyHostToDevice) != hipSuccess) st = AP_ERR_DEVICE;
            at += n;
            return here;
        };
        if (hipMemcpy(base, blob.data(), blob.size(), hipMemcpyHostToDevice) != hipSuccess ||
            hipMemcpy(base + o_slo, slo_us, 8u * (size_t)W, hipMemcpyHostToDevice) != hipSuccess)
            st = AP_ERR_DEVICE;
        p.blob = reinterpret_cast<const uint4*>(base);
        p.succ = reinterpret_cast<const uint16_t*>(base + reinterpret_cast<size_t>(p.succ));
        p.slo = reinterpret_cast<const unsigned long long*>(base + o_slo);
        p.pa = put(pa.data(), P);
        p.pb = put(pb.data(), P);
        p.qc = put(qc.data(), Q);
        p.qd = put(qd.data(), Q);
        p.cap = put(cap.data(), Q);
        p.penalty = penalty_permille;
        p.W = W; p.K = K; p.P = P; p.Q = Q;
        a->chunks = agentic_chunks(K);
        uint32_t off = align_up(std::max(8u * W, 4u * K), 16u);
        p.o_over = 0u;
        p.o_call = off;   off += align_up(2u * K, 16u);
        p.o_rank = off;   off += align_up(2u * K, 16u);
        p.o_ids = off;    off += align_up(2u * K, 16u);
        p.o_left = off;   off += align_up(K, 16u);
        p.o_comp = off;   off += align_up(4u * W, 16u);
        p.o_failed = off; off += align_up(W, 16u);
        p.o_over_phase = off; off += align_up(K, 16u);
        p.o_queue = off;  off += (P + Q) * 2u * a->chunks * 4u;
        p.wave_bytes = align_up(off, 16u);
        a->waves = kAgenticWaves;
        while (a->waves > 1u && p.blob_bytes + a->waves * p.wave_bytes > (uint32_t)lds_cap) a->waves /= 2u;
        a->lds_bytes = p.blob_bytes + a->waves * p.wave_bytes;
        a->wave_plans = (uint32_t)lds_cap / a->lds_bytes * a->waves;
        a->n_cu = (uint32_t)n_cu;
        // a row of lanes per plan: as many plans per compute unit as its LDS takes, in workgroups of up to kAgenticWaves wavefronts
        off = align_up(std::max(8u * W, 4u * align_up(K, kRowLanes)), 16u);
        p.g_call = off;    off += align_up(4u * K, 16u);
        p.g_call_of = off; off += align_up(2u * K, 16u);
        p.g_left = off;    off += align_up(K, 16u);
        p.g_comp = off;    off += align_up(4u * W, 16u);
        p.g_failed = off;  off += align_up((W + 31u) / 32u * 4u, 16u);
        p.g_queue = off;   off += (P + Q) * ((K + 31u) / 32u) * 4u;
        p.g_bytes = align_up(off, 16u);
        bool by_rows = P <= kRowLanes && Q <= kRowLanes && p.o_succ != 0u;   // it multiplies with 24-bit factors
        for (uint32_t k = 0; k < K; ++k) by_rows = by_rows && in_len[k] < (1u << 24) && out_len[k] < (1u << 24);
        for (uint32_t i = 0; i < P; ++i) by_rows = by_rows && pb[i] < (1u << 24);
        for (uint32_t i = 0; i < Q; ++i) by_rows = by_rows && qd[i] < (1u << 24) && (uint64_t)qc[i] + ((uint64_t)qd[i] << 14) < (1u << 24);
        if (by_rows) {
            uint32_t most = 0;
            for (uint32_t waves = kAgenticWaves; waves >= 1u; waves /= 2u) {
                const uint32_t bytes = p.blob_bytes + waves * (kWave / kRowLanes) * p.g_bytes;
                const uint32_t plans = bytes <= (uint32_t)lds_cap ? (uint32_t)lds_cap / bytes * waves : 0u;
                if (plans <= most) continue;
                most = plans;
                a->row_waves = waves;
                a->row_plans = plans * (kWave / kRowLanes);
                a->row_lds_bytes = bytes;
            }
        }
        if (a->row_waves != 0u) {
            hipFuncAttributes attr;
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_agentic_rows), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)a->row_lds_bytes) != hipSuccess ||
                hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&k_agentic_rows)) != hipSuccess)
                st = AP_ERR_DEVICE;
            else a->row_plans = std::min(a->row_plans, waves_by_registers(attr) * 4u * (kWave / kRowLanes));
        }
        if (a->lds_bytes > (uint32_t)lds_cap) st = AP_ERR_RANGE;
        else if (hipFuncSetAttribute(reinterpret_cast<const void*>(agentic_kernel(a->chunks)), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)a->lds_bytes) != hipSuccess)
            st = AP_ERR_DEVICE;
    }
    if (st != AP_OK) {
        (void)hipGetLastError();
        ap_agentic_destroy(a);
        return st;
    }
    *out = a;
    return AP_OK;
}

// Four plans per wavefront (k_agentic_rows) where the wavefronts of single plans would crowd the chip or not all be in service at
// once: those take as long for one plan as for all that are resident, and 0.036 of what a round of k_agentic_rows takes for each further
// plan of a compute unit.  In us, single plans against four, for plans of 317 calls on 4 + 4 instances, of which a compute unit holds 32:
// 1024 plans 659 and 1004, 6144 1030 and 1107, 6656 1382 and 1106, 8192 1458 and 1105.  More plans than that are several
// rounds.  A round that is not half full takes nearly as long as a full one: 8704 plans 1540 and 1971, 10240 1653 and 1985, 12288 1909 and
// 1982 (1917 and 1680 on 1 + 1 instances, 2155 and 1986 on 8 + 8), 14336 2256 and 2206, 16384 2476 and 2206, 20480 3050 and 2980, 32768
// 4691 and 4329.  Where a compute unit holds 48 (161 calls) no fill matters: 14336 plans 1134 and 792, 32768 2363 and 1468; 44 calls, 64 by
// registers: 8704 plans 207 and 172, 98304 1684 and 1049.  Where it holds 24 or fewer a second round never pays (362 calls: 5632 plans
// 1543 and 1310, 6656 1623 and 2281, 32768 5913 and 7185; 627 calls, 16: 4096 plans 2681 and 2140, 8192 4232 and 4278), and none does where
// it holds no more than single plans (486 calls: 4096 plans 1286 and 1604).
static bool agentic_by_rows(const ap_agentic* a, uint32_t C) {
    const uint32_t at_once = a->n_cu * a->row_plans;
    if (C <= a->n_cu * std::min(24u, a->wave_plans) || at_once == 0u) return false;
    if (C <= at_once || a->row_plans >= 48u) return true;
    return a->row_plans >= 32u && (C % at_once == 0u || C % at_once >= at_once / 2u);
}

// Which kernel C plans go through, for tests (not part of the header): 1 k_agentic_rows, 0 k_agentic_eval.
ap_status ap_agentic_route_get(const ap_agentic* a, uint32_t C, uint32_t* out) {
    if (!a || !out) return AP_ERR_INVALID;
    *out = agentic_by_rows(a, C) ? 1u : 0u;
    return AP_OK;
}

ap_status ap_agentic_eval(const ap_agentic* a, const uint16_t* d_prefill, const uint16_t* d_decode, const uint32_t* d_key,
                          uint32_t C, ap_agentic_metrics* d_out, void* hip_stream) {
    if (!a) return AP_ERR_INVALID;
    if (C == 0) return AP_OK;
    if (!d_prefill || !d_decode || !d_key || !d_out) return AP_ERR_INVALID;
    if (agentic_by_rows(a, C)) {
        const uint32_t plans = a->row_waves * (kWave / kRowLanes);
        hipLaunchKernelGGL(k_agentic_rows, dim3(std::min((C + plans - 1u) / plans, a->n_cu * 64u)), dim3(a->row_waves * kWave), a->row_lds_bytes,
                           static_cast<hipStream_t>(hip_stream), a->params, d_prefill, d_decode, d_key, d_out, C);
        if (hipGetLastError() != hipSuccess) return device_error();
        return AP_OK;
    }
    const uint32_t blocks = std::min((C + a->waves - 1u) / a->waves, a->n_cu * 64u);
    hipLaunchKernelGGL(agentic_kernel(a->chunks), dim3(blocks), dim3(a->waves * kWave), a->lds_bytes,
                       static_cast<hipStream_t>(hip_stream), a->params, d_prefill, d_decode, d_key, d_out, C);
    if (hipGetLastError() != hipSuccess) return device_error();
    return AP_OK;
}

ap_status ap_agentic_destroy(ap_agentic* a) {
    if (!a) return AP_OK;
    const bool ok = !a->d_block || hipFree(a->d_block) == hipSuccess;
    delete a;
    return ok ? AP_OK : AP_ERR_DEVICE;
}

ap_status ap_workload_destroy(ap_workload* w) {
    if (!w) return AP_OK;
    bool ok = true;
    if (w->d_arrival) ok = (hipFree(w->d_arrival) == hipSuccess) && ok;
    if (w->d_prompt) ok = (hipFree(w->d_prompt) == hipSuccess) && ok;
    if (w->d_out) ok = (hipFree(w->d_out) == hipSuccess) && ok;
    if (w->d_rep) ok = (hipFree(w->d_rep) == hipSuccess) && ok;
    if (w->d_tab_prefill) ok = (hipFree(w->d_tab_prefill) == hipSuccess) && ok;
    if (w->d_tab_tpot) ok = (hipFree(w->d_tab_tpot) == hipSuccess) && ok;
    if (w->d_req) ok = (hipFree(w->d_req) == hipSuccess) && ok;
    if (w->d_scratch) ok = (hipFree(w->d_scratch) == hipSuccess) && ok;
    if (w->d_span) ok = (hipFree(w->d_span) == hipSuccess) && ok;
    if (w->d_span_t) ok = (hipFree(w->d_span_t) == hipSuccess) && ok;
    if (w->d_pair) ok = (hipFree(w->d_pair) == hipSuccess) && ok;
    if (w->d_stream_tab) ok = (hipFree(w->d_stream_tab) == hipSuccess) && ok;
    if (w->d_count_lo) ok = (hipFree(w->d_count_lo) == hipSuccess) && ok;
    if (w->d_nominal) ok = (hipFree(w->d_nominal) == hipSuccess) && ok;
    if (w->d_nominal_sums) ok = (hipFree(w->d_nominal_sums) == hipSuccess) && ok;
    if (w->d_pending) ok = (hipFree(w->d_pending) == hipSuccess) && ok;
    if (w->h_stage) ok = (hipHostFree(w->h_stage) == hipSuccess) && ok;
    if (w->d_parent) ok = (hipFree(w->d_parent) == hipSuccess) && ok;
    if (w->d_peak) ok = (hipFree(w->d_peak) == hipSuccess) && ok;
    if (w->d_room) ok = (hipFree(w->d_room) == hipSuccess) && ok;
    if (w->d_rows) ok = (hipFree(w->d_rows) == hipSuccess) && ok;
    if (w->d_req8) ok = (hipFree(w->d_req8) == hipSuccess) && ok;
    if (w->split_plan.tables) ok = (hipFree(w->split_plan.tables) == hipSuccess) && ok;
    if (w->d_split_scratch) ok = (hipFree(w->d_split_scratch) == hipSuccess) && ok;
    if (w->d_bounds) ok = (hipFree(w->d_bounds) == hipSuccess) && ok;
    if (w->d_tab_pair) ok = (hipFree(w->d_tab_pair) == hipSuccess) && ok;
    delete w->roof;
    delete w;
    return ok ? AP_OK : AP_ERR_DEVICE;
}

}  // extern "C"
