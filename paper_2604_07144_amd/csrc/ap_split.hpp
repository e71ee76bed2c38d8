// Exact evaluation for replicas that differ or come and go: the trace of every replica is cut in two.
#ifndef AP_SPLIT_HPP
#define AP_SPLIT_HPP

#include <type_traits>

#include "ap_common.hpp"
#include "ap_runs.hpp"
#include "ap_screen.hpp"

namespace {

// ----------------------------------------------------------------------------------
// split evaluation: a listed part that is replayed, a streamed part that provably never waits
// ----------------------------------------------------------------------------------
// Replica m serves during [t_on, t_off) (the snapshot holds cluster availability, Section 4; Section 8.2
// "Elastic Cluster Dynamics").  Requests are in arrival order, so for every replica three index ranges are
// fixed by the trace alone, whatever the candidate:
//   r >= i_off[m]             arrives when the replica is gone: rejected on arrival;
//   r <  i_list[m]            the LISTED part: everything that arrives before the replica is up (its backlog)
//                             and while that backlog drains.  These requests are grouped by replica and
//                             replayed exactly through the B-slot queue (k_replay_lists);
//   i_list[m] <= r < i_off[m] the STREAMED part: scored where the assignment row is read, as requests that
//                             start on arrival (ttft = prefill), without a queue.
// Why the streamed part may skip the queue.  Let D(r) be the number of requests r' <= r of the whole trace,
// on any replica, whose service interval [arrival, arrival + longest service over the replica kinds) holds
// arrival(r): no candidate can have more requests that started on arrival in service on one replica at that
// moment.  Let busy(c, m) be the number of slots of replica m that the listed part of candidate c leaves taken
// beyond t_split[m] = arrival(i_list[m]).  If busy(c, m) + max over r >= i_list[m] of D(r) <= B, then by
// induction in arrival order every streamed request of (c, m) finds a free slot when it arrives: the requests
// of m in service at that moment are listed ones still running (at most busy) and earlier streamed ones, which
// started on arrival by the induction hypothesis and are therefore counted by D(r) - 1.  The host picks
// i_list[m] so that the bound leaves room (ap_costmodel_set); k_replay_lists counts busy(c, m) at the end of
// every list and hands the candidate to the general replay if the room is not there.  A trace too dense for
// any room (D above B) simply has every request listed.
//
// Per candidate the record is put together from three parts that add up (sums, counts) or combine by max
// (latest finish): the streamed part (k_split_candidates), the listed part (k_replay_lists, one atomic update per
// queue) and the rejected requests at the penalty latency (k_merge_candidates).
//
// The p99 fields need the histograms only when fewer than R - k99 + 1 requests are rejected.  Otherwise the
// k99-th smallest value of each metric is the penalty latency itself (rejected requests are charged it,
// Appendix "Serving Simulator", Memory Feasibility), provided every served latency falls in a lower bin, which
// the host checks against its bound on all finish times.  Such a candidate is called settled-by-penalty below
// and carries kFlagLazy; the others keep histograms: the streamed requests are counted in LDS while the row is
// read (and parked in device memory), the list replay leaves, queue by queue, the bins of the listed requests that any p99 value can
// depend on, and k_merge_candidates adds the two up.
constexpr uint32_t kBuildMinWaves = 4, kBuildMaxWaves = 8;   // of a workgroup of the kernels that build the lists
constexpr uint32_t kTile = 1024;                  // requests per tile: a list position fits 10 bits
constexpr uint32_t kTileSteps = kTile / kWave;
constexpr uint32_t kCrowd = 16;                   // of a tile's first 64 requests on one replica (k_list_candidates)
constexpr uint32_t kFlagNeedHist = 1u;            // streamed without histograms, but they are needed: stream again
constexpr uint32_t kFlagFallback = 2u;            // the listed part left too many slots taken: general replay
constexpr uint32_t kFlagLazy = 4u;                // the p99 values are the penalty latency
constexpr uint32_t kFlagNoStreamHist = 8u;        // histograms needed, and no request of the candidate was streamed
constexpr uint32_t kTpotWithin = 1u;              // no request's time per token can exceed the objective
constexpr uint32_t kSumsFit = 2u;                 // four latencies (e2e) add up to less than 2^32
// A list entry is 16 times the request's index in its tile: the list replay reads 16-byte records.
constexpr uint32_t kEntryShift = 4;
constexpr uint32_t kPadding = kTile << kEntryShift;   // the entry of a run's padding: names a record that never starts
// Bins word of a listed request: for each metric 0 (not served, or below least_bin), or bin - least_bin + 1.  Finish times are
// below 2^32, so bins are below 3328: 12 bits for ttft and for e2e, and 8 for tpot where its bins span no more than 255 from
// least_bin on.  Two words otherwise: ttft and e2e in the first, tpot in the second.
constexpr uint32_t kTpotSpan = 255u;

// Per replica, for the streaming kernel, as three arrays (copied to LDS; an entry per replica and one more, index
// M, for unknown replica ids: everything rejected).  Lanes look entries up by replica id, so consecutive ids must
// fall into different LDS banks: one 32-bit word per replica holds both ranges when R is below 65536 (else one
// word each), and the cost coefficients are stored once per kind of replica, which another word names.
struct SplitTables {
    const uint32_t* range;                        // [M + 1] i_list | i_off << 16; wide: i_list
    const uint32_t* range_off;                    // wide only: [M + 1] i_off
    const uint32_t* kind;                         // [M + 1] index into coef; tabulated cost model: the replica's type
                                                  //   (either way below 1024: it rides in the upper bits of a tile word)
    const uint4* coef;                            // [n_kinds] a, b, c, d
    uint32_t n_kinds;
};

struct SplitQueue {                               // per replica, for the list replay, 48 bytes
    uint32_t a, b, c, d, t_on, t_off;
    uint32_t i_list;
    uint32_t t_split;                             // arrival of request i_list; kNever: nothing is streamed
    uint32_t allow_busy;                          // slots that may still be taken beyond t_split
    uint32_t late_from;                           // t_off less three of the longest services; kNever: the replica stays
    uint32_t pad0, pad1;
};

struct SplitPartial {                             // per candidate of a batch, 64 bytes
    unsigned long long s_e2e, s_ttft, s_tpot;     // served requests only
    uint32_t last_fin, n_ok, n_rej, flags;
    uint32_t pad[6];
};

struct SplitParams {
    const uint2* req8;                            // [R] {arrival, prompt | out << 16}
    SplitTables tab;
    const SplitQueue* queue;                      // [M]
    const uint32_t* order;                        // [n_queues] replicas with a listed part, longest first
    uint32_t* desc;                               // [batch][n_list_tiles][M] count << 16 | first list position of
                                                  //   the replica's run
    uint16_t* lists;                              // [batch][n_list_tiles][tile_cap] entries of tile-local request indices by replica
    SplitPartial* part;                           // [batch]
    uint32_t* hist;                               // [batch][hist_words] the streamed requests' histograms
    void* bins;                                   // [batch][n_list_tiles * tile_cap] what listed requests add to the histograms, where it is
                                                  //   anything: a bins word as above, or two where the tpot bins span too much
    uint32_t* bin_base;                           // [batch][M + 1] where a queue's words begin (see place_bins)
    uint32_t* bin_count;                          // [batch][M + 1] how many the list replay has left
    uint32_t wide_bins;                           // the latter
    uint32_t least_bin[3], least_us[3];           // no p99 value (ttft, tpot, e2e) can lie below this bin: the list replay leaves smaller ones out
    uint32_t step_facts;                          // of the list replay: kTpotWithin, kSumsFit
    const uint2* tab_pair;                        // tabulated cost model: [T][R] {prefill time, time per token}; the kind
                                                  //   word of a replica then holds its type, SplitQueue::a type * R
    // Set when the listed evaluation runs behind the streamed one (ap_stream.hpp): only candidates whose record in `pending`
    // (the batch's) carries the pending mark are looked at, and none if the call has not raised its word.
    const ap_metrics* pending;
    const uint32_t* pending_word;
    uint32_t hist_words;                          // 3 * kBins / 2 (16-bit counts, R < 65536) or 3 * kBins
    uint32_t wide;                                // R >= 65536: two range words per replica
    uint32_t any_streamed;                        // some replica has a streamed part
    uint32_t R, M, B;
    uint32_t n_tiles, n_list_tiles, tile_cap, n_queues;
    uint32_t even_lists;                          // every replica has a list, and all are equally long
    uint32_t slo_ttft, slo_tpot;
    uint32_t lazy_from;                           // rejected requests from which the p99 values are the penalty; kNever: never
    // byte offsets into the streaming kernel's dynamic LDS
    uint32_t off_range, off_range_off, off_kind, off_acc, off_wave, wave_bytes, w_tile, w_sums, off_hist;
    uint32_t off_total;                                  // listed requests per replica
    uint32_t l_wave, l_wave_bytes, l_total;      // k_list_candidates: its wavefronts' areas (last), and the same
};

// Is candidate cb of the batch one to look at?
__device__ __forceinline__ bool split_wanted(const SplitParams& p, uint32_t cb) { return p.pending == nullptr || is_pending(p.pending[cb]); }
__device__ __forceinline__ bool split_nothing_pending(const SplitParams& p) {
    return p.pending != nullptr && __hip_atomic_load(p.pending_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
}

// The two cost tables of a tabulated model side by side, so that a request's prefill time and time per token come
// with one 8-byte load.
__global__ __launch_bounds__(kThreads) void k_pair_tables(const uint32_t* __restrict__ prefill, const uint32_t* __restrict__ tpot,
                                                          uint2* __restrict__ pair, size_t n) {
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (size_t)gridDim.x * kThreads)
        pair[i] = make_uint2(prefill[i], tpot[i]);
}

// Ranks by LDS additions.  A wavefront's LDS instructions execute in order; of the lanes of one addition that name the same word, lower
// ones have been seen to come first, always, but nothing promises it.  So every lane looks, once a tile's entries are in their runs, at
// the entry before its own, and a tile in which one is larger has its runs sorted (tests/device hands places out in any order).  A random
// read of 64 entries is 5 LDS cycles; ranks that need no such look, from ballots, are 30 vector instructions.
__device__ __forceinline__ void sort_runs(uint16_t* list, const uint32_t* first_of, const uint32_t* desc, uint32_t M) {
    for (uint32_t m = threadIdx.x & 63u; m < M; m += kWave) sort_run(list + first_of[m], desc[m] >> 16);
}

// A wavefront's LDS area for a tile's runs: [M] the runs' lengths, then where they begin; [64] words for what is not listed, one a lane; a list
// of tile_cap entries with eight more on either side.  What is not listed gets half of the list's length for a place, and one more than that
// for a run's beginning, which makes it write to the second spot behind the list, and finds 0 in the first.
__host__ __device__ inline uint32_t runs_list_offset(uint32_t M) { return (M + kWave) * 4u; }
__host__ __device__ inline uint32_t runs_bytes(uint32_t M, uint32_t tile_cap) { return ((runs_list_offset(M) + 15u) & ~15u) + tile_cap * 2u + 32u; }
__device__ __forceinline__ void init_runs(const SplitParams& p, unsigned char* area, uint32_t lane) {
    uint32_t* run = reinterpret_cast<uint32_t*>(area);
    for (uint32_t m = lane; m < p.M; m += kWave) run[m] = 0u;
    run[p.M + lane] = p.tile_cap / 2u + 1u;
    uint16_t* list = reinterpret_cast<uint16_t*>(area + ((runs_list_offset(p.M) + 15u) & ~15u)) + 8u;
    if (lane < 8u) list[p.tile_cap + lane] = 0u;
}

// A tile's runs and their descriptors, from the lengths of the runs (cleared again).  at: the LDS address of a request's run length or, if it is
// not listed, of its lane's word; place: the request's place in the run.  on_run(m, c): replica m has c requests here.
template <typename OnRun>
__device__ __forceinline__ void write_runs(const SplitParams& p, size_t tile_at, uint32_t lane, unsigned char* area,
                                           uint32_t (&at)[kTileSteps], const uint32_t (&place)[kTileSteps], const OnRun& on_run) {
    const uint32_t M = p.M;
    uint32_t* run = reinterpret_cast<uint32_t*>(area);
    uint16_t* list = reinterpret_cast<uint16_t*>(area + ((runs_list_offset(M) + 15u) & ~15u)) + 8u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t total = 0;
    for (uint32_t base = 0; base < M; base += kWave) {
        const uint32_t m = base + lane;
        const uint32_t c = m < M ? run[m] : 0u;
        const uint32_t room = (c + 7u) & ~7u;                                        // runs start on multiples of 8 positions
        const uint32_t upto = wave_inclusive_scan(room, lane);
        if ((c & 7u) != 0u) {                                                        // the run's last block: what no request takes is padding
            uint32_t pad = kPadding * 0x10001u;                                      // (made here: kept from tile to tile it costs a spill)
            asm volatile("" : "+v"(pad));
            reinterpret_cast<uint4*>(list)[(total + upto - room + c) / 8u] = make_uint4(pad, pad, pad, pad);
        }
        if (m < M) {
            run[m] = total + upto - room;
            p.desc[tile_at * M + m] = (c << 16) | (total + upto - room);
            on_run(m, c);
        }
        total += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    }
    if (total != 0u) {
        typedef __attribute__((address_space(3))) uint16_t lds_half;
        const uint32_t before_list = lds_address(list) - 2u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s) at[s] = *(lds_word*)(uintptr_t)at[s];
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s) {
            at[s] = before_list + 2u * (at[s] + place[s]);
            ((lds_half*)(uintptr_t)at[s])[1] = (uint16_t)((s * kWave + lane) << kEntryShift);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s) at[s] = *(lds_half*)(uintptr_t)at[s];   // the entry before (that of the first in a run is not looked at)
        unsigned long long disorder = 0ull;
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s)
            disorder |= __ballot(at[s] > (s * kWave + lane) << kEntryShift) & __ballot(place[s] != 0u);
        if (disorder != 0ull) sort_runs(list, run, p.desc + tile_at * M, M);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint4* dst = reinterpret_cast<uint4*>(p.lists + tile_at * p.tile_cap);       // 16 bytes (8 positions) at a time
        typedef uint32_t four_words __attribute__((ext_vector_type(4)));
        const four_words* from = reinterpret_cast<const four_words*>(list);
        four_words* to = reinterpret_cast<four_words*>(dst);
        for (uint32_t v = lane; v < total / 8u; v += 2u * kWave) {
            const uint32_t u = v + kWave;
            const four_words first = from[v], second = from[min(u, total / 8u - 1u)];
            to[v] = first;
            if (u < total / 8u) to[u] = second;
        }
    }
    for (uint32_t m = lane; m < M; m += kWave) run[m] = 0u;                          // for the wavefront's next tile
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// The ids of tile j, a lane's request of every 64; M beyond the row.
__device__ __forceinline__ void fetch_ids(uint32_t (&into)[kTileSteps], const uint16_t* row, uint32_t j, uint32_t lane, uint32_t R, uint32_t M) {
    if (j * kTile + kTile <= R) {
        const uint16_t* ids = row + j * kTile + lane;
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s) into[s] = __builtin_nontemporal_load(ids + s * kWave);
    } else {
#pragma unroll
        for (uint32_t s = 0; s < kTileSteps; ++s) {
            const uint32_t r = j * kTile + s * kWave + lane;
            into[s] = r < R ? (uint32_t)__builtin_nontemporal_load(row + r) : M;
        }
    }
}

// Where the bins of each replica's queue begin: the sums of the requests listed for the replicas before it, a tile's counted up to
// the next multiple of four, which is how the list replay writes (one wavefront).
__device__ __forceinline__ void place_bins(const SplitParams& p, uint32_t cb, const uint32_t* total_of) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t before = 0;
    for (uint32_t base = 0; base < p.M; base += kWave) {
        const uint32_t m = base + lane, v = m < p.M ? total_of[m] : 0u;
        const uint32_t upto = wave_inclusive_scan(v, lane);
        if (m < p.M) p.bin_base[(size_t)cb * (p.M + 1u) + m] = before + upto - v;
        before += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    }
}

// Streaming kernel, where something is streamed.  One workgroup per candidate at a time;
// its wavefronts take the tiles of the row in turn and share nothing but the accumulators (and the histograms), so there is no barrier inside a
// candidate.
// Per tile a wavefront classifies its 1024 requests, accumulates the streamed ones, finds the places of the listed ones in their replicas'
// runs by LDS additions (see sort_runs) and writes the runs, which start on multiples of 8 list positions, and their descriptors out.
// Bound by instruction issue and, with five wavefronts per SIMD, by what they wait for.  43 instructions for 64 requests and 404 us for 8192
// rows of 32768 requests on 64 replicas that come and go (3001 of 20011 on 50 with tables: 199) when listed requests were queued in LDS, counted and
// ranked from a second pass over the queue; 36 and 356 (144) now.  Of the 356 the runs are 110 and the costs 60; without a coefficient of 0 for
// requests that cost nothing, a branch for each instead, 405; with the sums in registers, 101 of them and four wavefronts, 400.
// kHistMode: 0 keeps no histograms of the streamed requests (enough when the candidate is settled by penalty), 1 keeps them
// with 16-bit counts (R < 65536), 2 with 32-bit counts.
// only_flagged: look only at candidates that an earlier launch marked kFlagNeedHist.
// kWithin: no request's prefill or time per token can exceed the objectives.
// kTabled: prefill time and time per token are read from the tables (one 8-byte load per request, issued with the
// table look-ups of the quarter tile) instead of being evaluated from a kind's coefficients.
template <uint32_t kHistMode, bool kTabled, bool kWithin>
__global__ __launch_bounds__(kBuildMaxWaves * kWave, kHistMode == 0u ? 5 : 4) void k_split_candidates(SplitParams p, const uint16_t* __restrict__ assign,
                                                                    uint32_t c0, uint32_t n_cand, uint32_t only_flagged,
                                                                    PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    pending_clear_next(flags);
    constexpr bool kHist = kHistMode != 0u, kHist16 = kHistMode == 1u;
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds + p.off_hist);          // kHist only
    uint32_t* range_of = reinterpret_cast<uint32_t*>(lds + p.off_range);
    uint32_t* range_off_of = reinterpret_cast<uint32_t*>(lds + p.off_range_off);   // wide only
    uint32_t* kind_of = reinterpret_cast<uint32_t*>(lds + p.off_kind);
    uint4* coef_of = reinterpret_cast<uint4*>(lds);
    unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(lds + p.off_acc);
    uint32_t* acc32 = reinterpret_cast<uint32_t*>(lds + p.off_acc + 24);    // latest finish, within objectives, rejected
    const uint32_t tid = threadIdx.x, w = wave_index(), n_waves = blockDim.x >> 6;
    uint32_t lane = tid & 63u;
    unsigned char* mine = lds + p.off_wave + w * p.wave_bytes;
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(mine + p.w_sums);   // [3][64] per lane: e2e, ttft, tpot
    uint32_t* tile_of = reinterpret_cast<uint32_t*>(mine + p.w_tile);        // [M + 1] the replica's ranges within the tile in hand
    uint32_t* total = reinterpret_cast<uint32_t*>(lds + p.off_total);        // kHist only: [M]
    // The coefficients lie at LDS address 0 (read by address: through the array's name every access costs an addition of its base).  The
    // kernel must declare no __shared__ variable of its own: the host asks (tables_at_lds_zero).
    typedef uint32_t four_words __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const four_words lds_four;
    const uint32_t R = p.R, M = p.M;

    // Mode 0 never runs behind the streamed evaluation, and need not ask.
    if (kHist && split_nothing_pending(p)) return;
    if (only_flagged) {                                                             // usually nothing is: leave at once
        bool any = false;
        for (uint32_t cb = blockIdx.x; cb < n_cand; cb += gridDim.x) any = any || (p.part[cb].flags & kFlagNeedHist) != 0u;
        if (!any) return;                                                           // the same words for every thread
    }
    for (uint32_t i = tid; i <= M; i += blockDim.x) {
        range_of[i] = p.tab.range[i];
        if (p.wide != 0u) range_off_of[i] = p.tab.range_off[i];
        kind_of[i] = p.tab.kind[i];
    }
    for (uint32_t i = tid; i <= p.tab.n_kinds; i += blockDim.x) coef_of[i] = i < p.tab.n_kinds ? p.tab.coef[i] : make_uint4(0u, 0u, 0u, 0u);
    init_runs(p, mine, lane);
    const uint32_t runs_at = lds_address(mine), nowhere_at = runs_at + 4u * (M + (tid & 63u));

    for (uint32_t cb = blockIdx.x; cb < n_cand; cb += gridDim.x) {
        if ((only_flagged && (p.part[cb].flags & kFlagNeedHist) == 0u) || (kHist && !split_wanted(p, cb))) continue;   // the same for every thread
        __syncthreads();                                                            // the last candidate's totals were read
        if (kHist) {
            for (uint32_t i = tid; i < p.hist_words; i += blockDim.x) hist[i] = 0u;
            for (uint32_t m = tid; m < M; m += blockDim.x) total[m] = 0u;
        }
        if (tid < 10u) reinterpret_cast<uint32_t*>(acc64)[tid] = 0u;
        __syncthreads();
        const uint16_t* row = assign + (size_t)(c0 + cb) * R;
        uint32_t last_fin = 0, n_ok = 0, n_rej = 0, n_streamed = 0;
        for (uint32_t k = 0; k < 3u; ++k) sums[k * kWave + lane] = 0ull;

        // A wavefront's tiles.  A lane holds a request of every 64.  The ids of the next tile are requested before the runs of
        // this one are written, the records and table look-ups of a quarter tile together before it is worked on.
        constexpr uint32_t kParts = 4u, kPart = kTileSteps / kParts;
        uint32_t at[kTileSteps], at_next[kTileSteps];                               // the replica
        // one tile; kWhole: all of its 1024 requests exist
        auto work_tile = [&](auto whole_tag, uint32_t j) {
            constexpr bool kWhole = decltype(whole_tag)::value;
            const uint32_t r0 = j * kTile, n = min(kTile, R - r0);
            asm volatile("" : "+v"(lane));                                          // positions are made here, not kept in registers
            // The replica ranges cut down to this tile, one word per replica: in the halves, listed below position `lo` of the tile and
            // gone from position `hi` on (both 0 .. 1024), and below them, in five bits each, the replica's kind
            // (or its type, when the costs come from tables), so that a request needs one look-up, and a half of it is
            // compared as it stands with the request's position, shifted alike and filled with ones.
            // (The wavefront's own LDS accesses execute in order.)
            for (uint32_t m = lane; m <= M; m += kWave) {
                const uint32_t word = range_of[m];
                const uint32_t i_list = p.wide != 0u ? word : (word & 0xFFFFu);
                const uint32_t i_off = p.wide != 0u ? range_off_of[m] : (word >> 16);
                const uint32_t lo = min(max(i_list, r0) - r0, kTile), hi = min(max(i_off, r0) - r0, kTile), kind = kind_of[m];
                tile_of[m] = (lo << 5) | (kind & 31u) | (((hi << 5) | (kind >> 5)) << 16);
            }
            const char* records = reinterpret_cast<const char*>(p.req8 + r0);
            uint32_t n_listed = 0;                                                  // (the same in every lane)
            uint32_t t_e2e = 0, t_ttft = 0, t_tpot = 0;                             // the tile's sums: 16 values below 2^28 each
            uint32_t place[kTileSteps];                                             // in the replica's run
#pragma unroll
            for (uint32_t h = 0; h < kParts; ++h) {
                unsigned long long record[kPart];                                   // (relaxed loads: others are moved to where they are used)
                uint32_t word[kPart], kind[kPart];
                uint32_t cost_prefill[kTabled ? kPart : 1u], cost_tpot[kTabled ? kPart : 1u];
#pragma unroll
                for (uint32_t i = 0; i < kPart; ++i) {
                    const uint32_t rl = (h * kPart + i) * kWave + lane;
                    record[i] = 0ull;
                    if (kWhole || rl < n)
                        record[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(records + (h * kPart + i) * kWave * 8u + lane * 8u),
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    word[i] = tile_of[at[h * kPart + i]];
                }
#pragma unroll
                for (uint32_t i = 0; i < kPart; ++i) {
                    if (kTabled) {
                        const uint32_t type = (word[i] & 31u) | ((word[i] >> 11) & 0x3E0u);
                        kind[i] = R < (1u << 24) ? __umul24(type, R) : type * R;    // the type's first table entry
                    } else {
                        kind[i] = (word[i] & 31u) << 4;                             // where the coefficients are
                    }
                }
                if (!kTabled && p.tab.n_kinds > 32u) {
#pragma unroll
                    for (uint32_t i = 0; i < kPart; ++i) {
                        kind[i] |= (word[i] >> 7) & 0x3E00u;
                        asm volatile("" : "+v"(kind[i]));                           // (a branch, not a choice for each)
                    }
                }
                if (kTabled) {
#pragma unroll
                    for (uint32_t i = 0; i < kPart; ++i) {                          // whether streamed or not: the entry exists
                        const uint32_t r = kWhole ? r0 + (h * kPart + i) * kWave + lane : min(r0 + (h * kPart + i) * kWave + lane, R - 1u);
                        const unsigned long long cost = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p.tab_pair) + (kind[i] + r),
                                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                        cost_prefill[i] = (uint32_t)cost;
                        cost_tpot[i] = (uint32_t)(cost >> 32);
                    }
                }
                // which of the lanes' requests start on arrival
                unsigned long long streamed[kPart], any_streamed = 0ull;
#pragma unroll
                for (uint32_t i = 0; i < kPart; ++i) {
                    const uint32_t s = h * kPart + i, rl = s * kWave + lane, position = (rl << 5) | 31u;
                    const unsigned long long in = kWhole ? ~0ull : __ballot(rl < n);
                    const unsigned long long listed = __ballot(position < (word[i] & 0xFFFFu)) & in;    // lo <= hi
                    const unsigned long long rejected = __ballot(position >= word[i] >> 16) & in;
                    streamed[i] = ~(listed | rejected) & in;
                    any_streamed |= streamed[i];
                    n_rej += (uint32_t)__popcll(rejected);
                    n_listed += (uint32_t)__popcll(listed);
                    asm volatile("" : "+s"(n_rej), "+s"(n_listed));                 // counted here, not kept as masks
                    const bool is_listed = __builtin_amdgcn_inverse_ballot_w64(listed);
                    at[s] = is_listed ? runs_at + 4u * at[s] : nowhere_at;
                    place[s] = p.tile_cap / 2u;
                    if (is_listed) place[s] = lds_add_rtn(at[s], 1u);
                }
                if (any_streamed == 0ull) continue;
                // ttft = prefill for these; the others cost nothing, from coefficients of 0 or instead of what the tables say
                uint32_t prefill[kPart], tpot[kPart], e2e[kPart], fin[kPart];
#pragma unroll
                for (uint32_t i = 0; i < kPart; ++i) {
                    const bool is_streamed = __builtin_amdgcn_inverse_ballot_w64(streamed[i]);
                    const uint32_t arrival = (uint32_t)record[i], lens = (uint32_t)(record[i] >> 32);
                    const uint32_t prompt = lens & 0xFFFFu, out = lens >> 16;
                    if (kTabled) {
                        prefill[i] = is_streamed ? cost_prefill[i] : 0u;
                        tpot[i] = is_streamed ? cost_tpot[i] : 0u;
                    } else {
                        const four_words co = *reinterpret_cast<lds_four*>(is_streamed ? kind[i] : p.tab.n_kinds * 16u);
                        prefill[i] = co.x + __umul24(co.y, prompt);                 // the host keeps all factors below 2^24
                        tpot[i] = co.z + __umul24(co.w, (prompt + 1023u) >> 10);
                    }
                    e2e[i] = prefill[i] + __umul24(out, tpot[i]);
                    fin[i] = is_streamed ? arrival + e2e[i] : 0u;
                    if (!kWithin) n_ok += (is_streamed && prefill[i] <= p.slo_ttft && tpot[i] <= p.slo_tpot) ? 1u : 0u;
                    if (kHist && is_streamed) {                                     // (a test per value against least_us costs more than it
                        hist_add<kHist16>(hist, 0u, hist_bin_u32(prefill[i]), 1u);  // saves: 3 rows of 30000 requests 46 against 37 us,
                        hist_add<kHist16>(hist, 1u, hist_bin_u32(tpot[i]), 1u);     // 2236 rows 261 against 252 in all)
                        hist_add<kHist16>(hist, 2u, hist_bin_u32(e2e[i]), 1u);
                    }
                }
                static_assert(kPart == 4u, "four added up");
                t_ttft += prefill[0] + prefill[1] + prefill[2] + prefill[3];
                t_e2e += e2e[0] + e2e[1] + e2e[2] + e2e[3];
                t_tpot += tpot[0] + tpot[1] + tpot[2] + tpot[3];
                last_fin = max(max(max(last_fin, fin[0]), max(fin[1], fin[2])), fin[3]);
            }
            atomicAdd(&sums[lane], (unsigned long long)t_e2e);                      // (in LDS they take no six registers)
            atomicAdd(&sums[kWave + lane], (unsigned long long)t_ttft);
            atomicAdd(&sums[2u * kWave + lane], (unsigned long long)t_tpot);
            fetch_ids(at_next, row, j + n_waves, lane, R, M);
            n_streamed += n - n_listed;                                             // (the rejected ones are taken off at the end)
            if (j >= p.n_list_tiles) return;                                        // nothing can be listed there
            write_runs(p, (size_t)cb * p.n_list_tiles + j, lane, mine, at, place, [&](uint32_t m, uint32_t c) {
                if (kHist && c != 0u) atomicAdd(&total[m], (c + 3u) & ~3u);
            });
        };
        fetch_ids(at_next, row, w, lane, R, M);
        for (uint32_t j = w; j < p.n_tiles; j += n_waves) {
#pragma unroll
            for (uint32_t s = 0; s < kTileSteps; ++s) at[s] = min(at_next[s], M);
            if ((j + 1u) * kTile <= R) work_tile(std::true_type{}, j);
            else work_tile(std::false_type{}, j);
        }

        // the workgroup's totals
        const unsigned long long s_e2e = wave_sum_u64(sums[lane]), s_ttft = wave_sum_u64(sums[kWave + lane]), s_tpot = wave_sum_u64(sums[2u * kWave + lane]);
        last_fin = wave_all_max(last_fin);
        n_ok = kWithin ? n_streamed - n_rej : wave_sum_u32(n_ok);
        if (lane == 0u) {
            atomicAdd(&acc64[0], s_e2e);
            atomicAdd(&acc64[1], s_ttft);
            atomicAdd(&acc64[2], s_tpot);
            atomicMax(&acc32[0], last_fin);
            atomicAdd(&acc32[1], n_ok);
            atomicAdd(&acc32[2], n_rej);                                            // already a wavefront total
        }
        __syncthreads();
        const uint32_t rejected = acc32[2];
        const bool lazy = rejected >= p.lazy_from;
        if (tid == 0u) {
            SplitPartial sp{};
            sp.s_e2e = acc64[0];
            sp.s_ttft = acc64[1];
            sp.s_tpot = acc64[2];
            sp.last_fin = acc32[0];
            sp.n_ok = acc32[1];
            sp.n_rej = rejected;
            sp.flags = lazy ? kFlagLazy : (kHist ? 0u : kFlagNeedHist);
            p.part[cb] = sp;
        }
        if (kHist && !lazy && w == 0u) place_bins(p, cb, total);
        if (kHist && !lazy) {
            uint32_t* dst = p.hist + (size_t)cb * p.hist_words;
            for (uint32_t i = tid; i < p.hist_words; i += blockDim.x) dst[i] = hist[i];
        }
    }
}

// `before`, and the lanes of `lanes` below this one.
__device__ __forceinline__ uint32_t lanes_before(unsigned long long lanes, uint32_t before) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, before));
}

// Lists where nothing is streamed: every request is listed, or its replica is gone.  No record, cost or queue is needed then, so a
// tile's ids stay in registers, a lane's request of every 64, together with what an LDS addition to the length of its replica's run returned:
// the request's place in the run (see sort_runs).
// Lanes that add to one word are served one after the other, so a tile that crowds a replica has the places on it, and on one more, counted
// by ballots instead: 2048 rows of 32768 requests on one of 64 replicas 254 to 78 us (122 with ballots alone), on two 157 to 79 (122), on three
// 126 to 111, four 110 to 107; from six on few tiles reach kCrowd, and even rows take 74 either way.  (Both forms behind a test in one loop cost
// even rows 109: registers.)
// Bound by LDS accesses, about 30 cycles for 64 requests: the addition, the run's beginning, the entry's store and the look at the entry
// before it, all at random banks.  1024 rows of 131072 requests on 128 replicas 166 us (61 vector instructions for 64 requests and 287 us
// with places from one ballot per bit of the replica id), 4096 rows of 32768 on 64 that come and go 137 (222).
__global__ __launch_bounds__(kBuildMaxWaves * kWave, 6) void k_list_candidates(SplitParams p, const uint16_t* __restrict__ assign, uint32_t c0,
                                                                      uint32_t n_cand, PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    pending_clear_next(flags);
    if (split_nothing_pending(p)) return;
    const uint32_t tid = threadIdx.x, w = wave_index(), n_waves = blockDim.x >> 6;
    uint32_t lane = tid & 63u;
    const uint32_t R = p.R, M = p.M;
    uint32_t* end_of = reinterpret_cast<uint32_t*>(lds + p.off_range);               // [M + 1] the replica's list ends here
    uint32_t* rejected_of_row = reinterpret_cast<uint32_t*>(lds + p.off_acc);
    uint32_t* total_of = reinterpret_cast<uint32_t*>(lds + p.l_total);               // [M] listed requests of the row
    unsigned char* mine = lds + p.l_wave + w * p.l_wave_bytes;
    init_runs(p, mine, tid & 63u);
    const uint32_t runs_at = lds_address(mine), nowhere_at = runs_at + 4u * (M + (tid & 63u));
    for (uint32_t i = tid; i <= M; i += blockDim.x) end_of[i] = p.wide != 0u ? p.tab.range[i] : p.tab.range[i] & 0xFFFFu;
    uint32_t least_end = kNever;
    for (uint32_t m = lane; m < M; m += kWave) least_end = min(least_end, p.wide != 0u ? p.tab.range[m] : p.tab.range[m] & 0xFFFFu);
    least_end = kNever - wave_all_max(kNever - least_end);
    for (uint32_t cb = blockIdx.x; cb < n_cand; cb += gridDim.x) {
        if (!split_wanted(p, cb)) continue;                                          // the same record for every thread
        __syncthreads();                                                             // the last candidate's totals were read
        if (tid == 0u) rejected_of_row[0] = 0u;
        for (uint32_t m = tid; m < M; m += blockDim.x) total_of[m] = 0u;
        __syncthreads();
        const uint16_t* row = assign + (size_t)(c0 + cb) * R;
        uint32_t n_seen = 0, n_listed = 0, listed_here = 0;                          // the last: of replica `lane`
        uint32_t at_next[kTileSteps];                                                // the replica
        // Tiles from j on while they are crowded, or while they are not: kCrowd or more of the first 64 requests name one replica.
        auto work_tiles = [&](auto crowded_tag, uint32_t j) {
            constexpr bool kCrowded = decltype(crowded_tag)::value;
            for (; j < p.n_tiles; j += n_waves) {
                // the replica that the tile's first lane with one names
                const unsigned long long known = __ballot(at_next[0] < M);
                const uint32_t some = known != 0ull ? (uint32_t)__builtin_amdgcn_readlane((int)at_next[0], __builtin_ctzll(known)) : kNever;
                const unsigned long long of_some = __ballot(at_next[0] == some);
                if (((uint32_t)__popcll(of_some) >= kCrowd) != kCrowded) break;
                const uint32_t r0 = j * kTile;
                n_seen += min(kTile, R - r0);
                asm volatile("" : "+v"(lane));                                       // positions are made here, not kept in registers
                uint32_t at[kTileSteps];
#pragma unroll
                for (uint32_t s = 0; s < kTileSteps; ++s) at[s] = min(at_next[s], M);
                fetch_ids(at_next, row, j + n_waves, lane, R, M);
                uint32_t place[kTileSteps];                                          // in the run
                if (r0 + kTile <= least_end) {                                       // all but unknown replicas': the next look-ups say nothing
#pragma unroll
                    for (uint32_t s = 0; s < kTileSteps; ++s) place[s] = at[s] < M ? kNever : 0u;
                } else {
#pragma unroll
                    for (uint32_t s = 0; s < kTileSteps; ++s) place[s] = end_of[at[s]];  // entry M is 0
                }
                if constexpr (!kCrowded) {
#pragma unroll
                    for (uint32_t s = 0; s < kTileSteps; ++s) {
                        const bool listed = r0 + s * kWave + lane < place[s];        // and below R
                        n_listed += (uint32_t)__popcll(__ballot(listed));
                        at[s] = listed ? runs_at + 4u * at[s] : nowhere_at;
                        place[s] = p.tile_cap / 2u;
                        if (listed) place[s] = lds_add_rtn(at[s], 1u);
                    }
                } else {
                    // that replica's places, and those of the first one beside it, are counted by ballots
                    const unsigned long long others = known & ~of_some;
                    const uint32_t other = others != 0ull ? (uint32_t)__builtin_amdgcn_readlane((int)at[0], __builtin_ctzll(others)) : kNever;
                    uint32_t n_some = 0, n_other = 0;
#pragma unroll
                    for (uint32_t s = 0; s < kTileSteps; ++s) {
                        const unsigned long long listed = __ballot(r0 + s * kWave + lane < place[s]);
                        const unsigned long long lanes_some = __ballot(at[s] == some) & listed, lanes_other = __ballot(at[s] == other) & listed;
                        at[s] = __builtin_amdgcn_inverse_ballot_w64(listed) ? runs_at + 4u * at[s] : nowhere_at;
                        place[s] = __builtin_amdgcn_inverse_ballot_w64(lanes_some) ? lanes_before(lanes_some, n_some) : p.tile_cap / 2u;
                        place[s] = __builtin_amdgcn_inverse_ballot_w64(lanes_other) ? lanes_before(lanes_other, n_other) : place[s];
                        if (__builtin_amdgcn_inverse_ballot_w64(listed & ~(lanes_some | lanes_other))) place[s] = lds_add_rtn(at[s], 1u);
                        n_listed += (uint32_t)__popcll(listed);
                        n_some += (uint32_t)__popcll(lanes_some);
                        n_other += (uint32_t)__popcll(lanes_other);
                        __builtin_amdgcn_sched_barrier(0);                           // counted here, not kept as masks
                    }
                    if (lane == 0u) {
                        uint32_t* run = reinterpret_cast<uint32_t*>(mine);
                        run[some] = n_some;
                        if (other != kNever) run[other] = n_other;
                    }
                }
                if (j >= p.n_list_tiles) continue;                                   // nothing is listed: no tile of the lists either
                write_runs(p, (size_t)cb * p.n_list_tiles + j, lane, mine, at, place, [&](uint32_t m, uint32_t c) {
                    if (m < kWave) listed_here += (c + 3u) & ~3u;
                    else if (c != 0u) atomicAdd(&total_of[m], (c + 3u) & ~3u);
                });
            }
            return j;
        };
        fetch_ids(at_next, row, w, lane, R, M);
        for (uint32_t j = w; j < p.n_tiles;) {
            j = work_tiles(std::false_type{}, j);
            if (j < p.n_tiles) j = work_tiles(std::true_type{}, j);
        }
        if (lane == 0u) atomicAdd(&rejected_of_row[0], n_seen - n_listed);           // wavefront totals
        if (listed_here != 0u) atomicAdd(&total_of[lane], listed_here);
        __syncthreads();
        if (tid == 0u) {
            SplitPartial sp{};
            sp.n_rej = rejected_of_row[0];
            sp.flags = sp.n_rej >= p.lazy_from ? kFlagLazy : kFlagNoStreamHist;
            p.part[cb] = sp;
        }
        if (w == 0u && rejected_of_row[0] < p.lazy_from) place_bins(p, cb, total_of);
    }
}

// a becomes the median of three: with a <= c it is min(c, max(a, b)), in one instruction.  In place, so that a's register
// stays the same along every path through the code around it.
__device__ __forceinline__ void median3(uint32_t& a, uint32_t b, uint32_t c) { asm("v_med3_u32 %0, %0, %1, %2" : "+v"(a) : "v"(b), "v"(c)); }

__device__ __forceinline__ void raise(uint32_t& a, uint32_t b) { asm("v_max_u32 %0, %0, %1" : "+v"(a) : "v"(b)); }

// List replay.  One lane per (candidate, replica) queue: the 64 lanes of a wavefront replay the listed part of
// replica m under 64 candidates of the batch, and the kListWaves wavefronts of a workgroup take neighbouring
// candidates of the same replica.  All lanes share the replica, hence its cost coefficients and window (scalar
// registers) and - roughly - the pace at which they move through the trace, so the request records of
// kReplayTiles tiles are staged in LDS once per workgroup and read by every lane; inside such a stage the
// wavefronts run free (no barrier), and within a wavefront the lanes meet again at every tile, where the lane
// with the most requests of the tile sets the pace.  Staging several tiles at a time for several wavefronts is
// what keeps the share of idle lane-steps down: the counts of a stage differ less, relative to their mean, than
// those of a single tile.
// A lane keeps its B slot-free times in registers, as two ascending sequences: the front, kFront of them, and the rest.  A request
// starts at max(ready, s[0]), and its finish time f replaces s[0] in the front by one median per register:
// s'[i] = med3(s[i], f, s[i+1]), i.e. min(s[i+1], max(s[i], f)).  A lane without a request in a step has a record that inserts 0,
// which leaves the registers as they are, and adds one microsecond to the sum of latencies, taken off in the end: nothing in a step asks
// whether a request was served.  Requests that would start too late are given that record before their step; lanes look for them
// only when one of four starts may be that late: where a queue closes, and then until the tile ends, for the other lanes too.
// Is s[0] the earliest slot?  Slots that are free when a request is ready are as good as each other, then and later, whatever time
// they hold.  So four requests may take theirs from the front if s[3] <= max(earliest of the rest, ready time of the first): of
// s[0..3] one is still there at each of the four.  Where that does not hold in some lane, all lanes merge the two sequences
// (Batcher's network) and the front is the kFront earliest again, which is good for kFront requests at least, and for any
// number while slots are free: as a queue fills up, after its backlog has drained, on a light trace.
// Starts do not decrease along a queue, so once a start reaches t_off every later request is rejected too: a tile in which no
// lane's earliest slot comes free in time is only counted, and a workgroup without such a lane stages nothing more.
// kSlots: B rounded up to 8, 12, 16, 24, 32, 48 or 64, and 4 below four; registers beyond B hold kNever and stay there.  Below four slots a
// start may be later than all of them were four requests before, and the bound is another (see below): with s[3], which is none there, the
// look was taken at every step, 300 rows of 16384 requests that crowd 8 of 48 replicas 676 us, 562 now (stay, any load), 368 and 255 (leave).
//
// Bound by instruction issue, and where the longest of 64 lanes' runs sets the pace by the idle steps of the others.  What every lane would
// evaluate for itself is done once while staging (the request's prefill and decode time on this replica, from coefficients or tables),
// records are read from LDS four at a time before they are needed, a tile's steps are counted once.
// Of 64 slots a front of 16 takes 16 operations a request and a merge about 300 and its register moves, at most once in 16: half of the 64
// medians over one sorted sequence, and a quarter while slots are free (fronts of 8 and 32 are 38 and 42).  With 16, 24 and 32 slots it is a
// front of 8, below that the front is all.  One sorted sequence, whose lower registers held still where slots were free, and this: kernels of
// 8192 rows of 32768 requests on 64 replicas of 64 slots that come and go 380 and 300 us, of 1024 of 131072 on 128 crowded 665 and 550; calls of
// 4096 rows of 16384 on 48 that come and go, half their slots in use: 16 slots 233 and 229 us, 32 280 and 260, 64 345 and 280.
// Loads run ahead: a lane's descriptors a stage, its next block of entries a block, also into the next tile, and the
// records of a stage four per thread at a time.  A register whose
// load is in flight is neither moved nor chosen from in between (either waits for it), hence one block ahead, e_next as vectors
// and the empty asm where they are waited for.  Blocks of eight entries come too late for queues of few slots: a wavefront by itself takes
// 200 ns a request there, a line from HBM and the stores before it more than eight of those (400 rows of 16384 requests on one of 2 replicas
// of 8 slots 3842 us, 3356 with sixteen).  With more than 48 slots a pair of steps that
// no lane needs is left out; up to there the branch costs more (crowds of one queue 6 % at 8 and 16 slots, 4 % at 24 to 48).
// Where all lists are as long as the trace, a few neighbouring replicas share an XCD, whose L2 then holds their runs once.
// A queue's words for the histograms follow one another (place_bins), four requests at a time where one of the four has a value
// that a p99 value can reach: on a trace that is not hopelessly overloaded one in fifty to one in ten has, and a word per list
// position would be a gigabyte of 16-byte stores to as many cache lines for 1024 rows of 131072 requests.
// kBins: 0 leaves no bins, 1 one word per request, 2 two words.  which: 0 every candidate, 1 only those settled by penalty,
// 2 only the others; a workgroup without a lane to work on ends at once.
// kFew: no more than a workgroup per compute unit; bins are then taken of every four requests, without a test whether any of them counts.  A
// crowded queue's wavefront, which has its SIMD to itself, gains 3 % by that at any number of workgroups, one of even rows gains or loses
// little where replicas are of several kinds and loses up to a fifth where they are of one and few of its values count.  With the test and
// without: 8192 requests on 64 replicas of 8 slots, 256 rows that crowd 10 of them 259 and 251 us, even rows 86 and 85; 16384 on 24 of 16 slots,
// 256 rows, crowds 1130 and 1089, even 276 and 263; 131072 on 128 of 64 slots, 256 rows (128 workgroups), crowds 2680 and 2618, even 742 and 785, of
// three kinds 904 and 892; 3 rows, even, 466 and 559; 1024 rows (512 workgroups), crowds 2965 and 2913, even 1078 and 1129.  The line is at the
// compute units: beyond it even rows, which are the larger calls, lose as much as crowds gain.
constexpr uint32_t kListWaves = 4;
constexpr uint32_t kReplayListThreads = kListWaves * kWave;
constexpr uint32_t kXcds = 8;                     // workgroups go to them in turn
constexpr uint32_t kNeighbours = 4;               // replicas whose workgroups for the same candidates share an XCD
constexpr uint32_t kReplayTiles = 2;              // tiles staged at a time: 32 KiB of records per workgroup
constexpr uint32_t kStageAtOnce = 4;
constexpr uint32_t kStagedTile = kTile + 1u;      // a tile's records, then the one that padding names

__device__ __forceinline__ uint32_t bin_above(uint32_t v, uint32_t least_us, uint32_t least_bin) {
    return v >= least_us ? hist_bin_u32(v) - least_bin + 1u : 0u;
}

// hi:lo += v in two instructions (the compiler's 64-bit add takes a register for the upper half of v as well), the two wait states that
// the compiler keeps between a vector instruction that writes vcc and one that reads it among them
__device__ __forceinline__ void add_wide(uint32_t& lo, uint32_t& hi, uint32_t v) {
    asm("v_add_co_u32 %0, vcc, %0, %2\n\ts_nop 1\n\tv_addc_co_u32 %1, vcc, 0, %1, vcc" : "+v"(lo), "+v"(hi) : "v"(v) : "vcc");
}

// Merge of two ascending sequences by Batcher's odd-even network (K. E. Batcher, Sorting networks and their applications, 1968), in place:
// the kM elements s[kAt], s[kAt + kStride], .. and the kN behind them (kM a power of two, kN >= kM).  A single element goes in by a
// median per place.  The asm keeps the order of the exchanges, and with it the registers to the elements and one more: left to the
// compiler's schedule, 64 elements take 35 registers more, written so 14.
template <uint32_t kSlots, uint32_t kAt, uint32_t kStride, uint32_t kM, uint32_t kN>
__device__ __forceinline__ void merge_sorted(uint32_t (&s)[kSlots]) {
    if constexpr (kM == 1u) {
        const uint32_t v = s[kAt];
        asm volatile("v_min_u32 %0, %1, %2" : "=&v"(s[kAt]) : "v"(v), "v"(s[kAt + kStride]));
#pragma unroll
        for (uint32_t i = 1; i < kN; ++i)
            median3(s[kAt + i * kStride], v, s[kAt + (i + 1u) * kStride]);
        raise(s[kAt + kN * kStride], v);
    } else {
        merge_sorted<kSlots, kAt, 2u * kStride, kM / 2u, (kN + 1u) / 2u>(s);
        merge_sorted<kSlots, kAt + kStride, 2u * kStride, kM / 2u, kN / 2u>(s);
#pragma unroll
        for (uint32_t i = 1; i + 1u < kM + kN; i += 2u) {
            uint32_t& a = s[kAt + i * kStride];
            uint32_t& b = s[kAt + (i + 1u) * kStride];
            uint32_t low;
            asm volatile("v_min_u32 %0, %1, %2\n\tv_max_u32 %2, %1, %2" : "=&v"(low), "+v"(a), "+v"(b));
            a = low;
        }
    }
}

template <uint32_t kSlots, uint32_t kBins_, bool kFew>
__global__ __launch_bounds__(kReplayListThreads, kSlots > 32u ? 3 : 5) void k_replay_lists(SplitParams p, uint32_t n_cand, uint32_t which) {
    __shared__ uint4 recs[kReplayTiles * kStagedTile];                              // {arrival, prefill + decode, decode, tpot}
    __shared__ uint32_t goes_on[kListWaves];                                        // the wavefront has a lane with something to replay
    if (split_nothing_pending(p)) return;
    const uint32_t tid = threadIdx.x;
    const uint32_t n_blocks = (n_cand + kReplayListThreads - 1u) / kReplayListThreads;
    // Longest lists first; where all are as long as the trace, kNeighbours replicas next to each other and the same candidates on one XCD:
    // their runs share cache lines.  Such units go round the XCDs, the blocks of candidates of the same replicas one after the other, so
    // that the long queues of rows that crowd neighbouring replicas are spread over the XCDs and over the compute units of each (a
    // contiguous eighth of all workgroups per XCD put them side by side: 1500 rows of 30000 requests that crowd 50 of 300 replicas 624
    // against 454 us, calls of 11184 of 3000 on one of 8, 1134 against 923; even rows, and units of 4, 8 and 16, alike to 1 %).
    uint32_t at_queue = blockIdx.x / n_blocks, at_block = blockIdx.x % n_blocks;
    if (p.even_lists != 0u) {
        const uint32_t in_xcd = blockIdx.x / kXcds, unit = in_xcd / kNeighbours * kXcds + blockIdx.x % kXcds;
        at_queue = unit / n_blocks * kNeighbours + in_xcd % kNeighbours;
        at_block = unit % n_blocks;
        if (at_queue >= p.n_queues) return;
    }
    // (which is settled here: left to the compiler, a row of 3000 requests on one of 8 replicas takes 663 us, with this 614)
    asm volatile("" : "+s"(at_queue), "+s"(at_block));
    const uint32_t m = p.order[at_queue];
    const uint32_t cb = at_block * kReplayListThreads + tid;
    bool live = cb < n_cand && split_wanted(p, cb);
    const uint32_t flags = live ? p.part[cb].flags : 0u;
    const bool lazy = (flags & kFlagLazy) != 0u;
    live = live && (which == 0u || lazy == (which == 1u));
    if (__syncthreads_or(live ? 1 : 0) == 0) return;
    const bool with_hist = kBins_ != 0u && live && !lazy;                           // leave bins
    SplitQueue q = p.queue[m];
    q.a = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.a);
    q.b = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.b);
    q.c = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.c);
    q.d = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.d);
    q.t_on = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.t_on);
    q.t_off = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.t_off);
    q.i_list = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.i_list);
    q.late_from = (uint32_t)__builtin_amdgcn_readfirstlane((int)q.late_from);

    constexpr bool kBelowFour = kSlots == 4u;                                       // slots
    constexpr uint32_t kFront = kSlots >= 48u ? 16u : kSlots >= 16u ? 8u : kSlots;  // a power of two where there is a rest
    constexpr bool kPairs = kSlots > 48u;                                           // two steps are worth a branch
    constexpr uint32_t kHalves = 2u, kBlock = 8u * kHalves;                         // entries ahead
    uint32_t s[kSlots];
#pragma unroll
    for (uint32_t i = 0; i < kSlots; ++i) s[i] = i < p.B ? 0u : kNever;
    static_assert(kFront == kSlots || (kFront >= 4u && (kFront & (kFront - 1u)) == 0u && 2u * kFront <= kSlots), "four at a time; merge_sorted");
    auto earliest = [&]() { return kFront < kSlots ? min(s[0], s[kFront < kSlots ? kFront : 0u]) : s[0]; };
    uint32_t e2e_lo = 0, e2e_hi = 0, dec_lo = 0, dec_hi = 0, tpot_lo = 0, tpot_hi = 0;
    uint32_t n_ok = 0, n_rej = 0, n_over = 0, n_run = 0, n_here = 0;       // steps, and requests among them

    const uint32_t n_t = (q.i_list + kTile - 1u) / kTile;
    uint32_t j0 = 0;
    const size_t desc_at = (size_t)(live ? cb : 0u) * p.n_list_tiles;
    auto desc_of = [&](uint32_t j) { return live && j < n_t ? p.desc[(desc_at + j) * p.M + m] : 0u; };
    auto run_of = [&](uint32_t d, uint32_t& count) {                                // a descriptor that was never written that way lists nothing
        const uint32_t first = d & 0xFFFFu;
        count = (((first & 7u) != 0u) | (first + (((d >> 16) + 7u) & ~7u) > p.tile_cap)) ? 0u : d >> 16;
        return first;
    };
    typedef uint32_t four_words __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const four_words lds_four;
    // The kBlock entries from kBlock * b on of a run.  A lane without them reads where all such lanes do, the area's first bytes, so that there
    // is no branch around the loads and next to no traffic: where each read its own tile's first block, one that no lane needed, 8388 rows
    // of 8000 requests that crowd 50 of 300 replicas took 605 us in here, 351 before anything was read ahead, 359 with this.
    const uint32_t lists_at = 2u * p.tile_cap * (uint32_t)desc_at;                  // bytes: plan_split keeps a batch's lists below 2^32
    four_words e_next[kHalves] = {};                                                      // the block after the one in hand
    auto request_block = [&](uint32_t d, uint32_t j, uint32_t b) {
        uint32_t count;
        const uint32_t first = run_of(d, count), run_at = lists_at + 2u * (j * p.tile_cap + first + kBlock * b);
#pragma unroll
        for (uint32_t h = 0; h < kHalves; ++h) {
            const uint32_t at = kBlock * b + 8u * h < count ? run_at + 16u * h : 0u;
            e_next[h] = *reinterpret_cast<const four_words*>(reinterpret_cast<const char*>(p.lists) + at);
        }
    };
    static_assert(kReplayTiles == 2u, "descriptors of a stage and of the next one");
    uint32_t d_here[2], d_next[2] = {desc_of(0u), desc_of(1u)};
    // the words of the queue's large values, in fours with at least one of them
    const size_t bins_at = with_hist ? (size_t)cb * p.n_list_tiles * p.tile_cap + p.bin_base[(size_t)cb * (p.M + 1u) + m] : 0u;
    uint32_t n_left = 0;
    for (; j0 < n_t; j0 += kReplayTiles) {
        const uint32_t r0 = j0 * kTile, n = min(kReplayTiles * kTile, p.R - r0);
        if ((tid & 63u) == 0u) goes_on[wave_index()] = 0u;
        if (__ballot(live && earliest() < q.t_off) != 0ull && (tid & 63u) == 0u) goes_on[wave_index()] = 1u;
        __syncthreads();                                                            // also: the last stage's records were read
        uint32_t any = 0u;
#pragma unroll
        for (uint32_t ww = 0; ww < kListWaves; ++ww) any |= goes_on[ww];
        if (__builtin_amdgcn_readfirstlane((int)any) == 0) break;
        d_here[0] = d_next[0];
        d_here[1] = d_next[1];
        // several records per thread at a time, requested together
        for (uint32_t i0 = tid; i0 < n; i0 += kStageAtOnce * kReplayListThreads) {
            uint2 rq[kStageAtOnce], cost[kStageAtOnce];
#pragma unroll
            for (uint32_t k = 0; k < kStageAtOnce; ++k) rq[k] = p.req8[r0 + min(i0 + k * kReplayListThreads, n - 1u)];
            if (p.tab_pair != nullptr) {
#pragma unroll
                for (uint32_t k = 0; k < kStageAtOnce; ++k) cost[k] = p.tab_pair[q.a + r0 + min(i0 + k * kReplayListThreads, n - 1u)];
            } else {
#pragma unroll
                for (uint32_t k = 0; k < kStageAtOnce; ++k) {
                    const uint32_t prompt = rq[k].y & 0xFFFFu;
                    cost[k] = make_uint2(q.a + __umul24(q.b, prompt),               // the host keeps all factors below 2^24
                                         q.c + __umul24(q.d, (prompt + 1023u) >> 10));
                }
            }
#pragma unroll
            for (uint32_t k = 0; k < kStageAtOnce; ++k) {
                const uint32_t i = i0 + k * kReplayListThreads;
                if (i < n) {
                    const uint32_t decode = __umul24(rq[k].y >> 16, cost[k].y);
                    recs[i + i / kTile] = make_uint4(rq[k].x, cost[k].x + decode, decode, cost[k].y);
                }
            }
        }
        if (tid < kReplayTiles) recs[tid * kStagedTile + kTile] = make_uint4(kNever, 1u, 0u, 0u);
        __syncthreads();
        if (j0 == 0u) request_block(d_here[0], 0u, 0u);
        for (uint32_t j = j0; j < min(j0 + kReplayTiles, n_t); ++j) {
            const uint32_t records_at = lds_address(recs) + (j - j0) * kStagedTile * 16u;
            uint32_t d = j == j0 ? d_here[0] : d_here[1];
            uint32_t count;
            (void)run_of(d, count);
            const bool open = live && earliest() < q.t_off;                         // else nothing starts any more: its run is left alone
            n_over += open ? 0u : count;
            d = open ? d : 0u;
            count = open ? count : 0u;
            n_here += count;
            uint32_t closes = open ? q.t_off : kNever;
            if constexpr (kBelowFour) {
                const uint32_t latest = max(recs[(j - j0) * kStagedTile + min(kTile, p.R - j * kTile) - 1u].x, q.t_on);   // of the tile's ready times
                closes = !open ? kNever : latest < q.late_from ? q.late_from : 0u;
            }
            // Steps of the tile; where nothing can start there is one all the same, in which only the next tile's block and the next
            // stage's descriptors are requested.
            const uint32_t most = __ballot(open) != 0ull ? wave_all_max(count) : 0u;
            uint32_t n_steps = max(most, 1u);
            uint32_t e[4u * kHalves];                                               // two entries each, the next ones first
#pragma unroll
            for (uint32_t i = 0; i < 4u * kHalves; ++i) e[i] = kPadding * 0x10001u;
            for (uint32_t k0 = 0; k0 < n_steps; k0 += 4u) {                         // four requests at a time
                if (k0 % kBlock == 0u) {
                    const bool last = k0 + kBlock >= n_steps;                       // the last block of every lane: on to the next tile's
                    // waited for here, before the next requests
#pragma unroll
                    for (uint32_t h = 0; h < kHalves; ++h) asm volatile("" : "+v"(e_next[h]));
                    asm volatile("" : "+v"(d_next[0]), "+v"(d_next[1]));
#pragma unroll
                    for (uint32_t i = 0; i < 4u * kHalves; ++i) e[i] = k0 + (i < 4u ? 0u : 8u) < count ? e_next[i / 4u][i % 4u] : kPadding * 0x10001u;
                    // (short traces have no next tile: 106 to 92 us for 512 rows of 800 requests on 755 replicas)
                    if (!last || j + 1u < n_t)
                        request_block(!last ? d : j == j0 ? d_here[1] : d_next[0], last ? j + 1u : j, last ? 0u : k0 / kBlock + 1u);
                    if (k0 == 0u && j == j0) {
                        d_next[0] = desc_of(j0 + 2u);
                        d_next[1] = desc_of(j0 + 3u);
                    }
                } else {
#pragma unroll
                    for (uint32_t i = 0; i + 2u < 4u * kHalves; ++i) e[i] = e[i + 2u];
                }
                if (most == 0u) continue;
                const uint32_t word[2] = {e[0], e[1]};
                four_words rec[4];
#pragma unroll
                for (uint32_t k = 0; k < 4u; ++k)
                    rec[k] = *reinterpret_cast<lds_four*>(records_at + ((k & 1u) ? word[k >> 1] >> 16 : word[k >> 1] & 0xFFFFu));
                // do the next four starts come from the front in every lane? (a lane without a request is ready at kNever)
                if (kFront < kSlots && __ballot(s[kFront < kSlots ? 3u : 0u] > max(s[kFront < kSlots ? kFront : 0u], max(rec[0].x, q.t_on))) != 0ull)
                    merge_sorted<kSlots, 0u, 1u, kFront, kSlots - kFront>(s);
                const bool short_four = kPairs && k0 + 2u >= n_steps;               // no lane has a third
                // No start is later than s[3], or ready time; with fewer than four slots, where s[3] is none, than the later of s[0] and the
                // ready times and three services on top.  Where some lane's four may start too late, those of them that do are made
                // padding first: which they are comes from the four earliest slots.
                if (__ballot(s[kBelowFour ? 0u : 3u] >= closes) != 0ull) {
                    // (A way out of the loop here costs every step three branches: 1024 rows of 131072 requests, all on one replica, 37.3 ms
                    // instead of 36.4, even rows 1106 us instead of 1080.)
                    if (__ballot(open && earliest() < q.t_off) == 0ull) {           // nothing starts any more: these four are the last
                        n_rej += count - min(count, k0 + 4u);
                        n_steps = k0;
                    }
                    uint32_t early[4];
#pragma unroll
                    for (uint32_t i = 0; i < 4u; ++i) early[i] = s[i];
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k) {
                        const uint32_t start = max(max(rec[k].x, q.t_on), early[0]);
                        const bool served = start < q.t_off;
                        const uint32_t f = served ? start + rec[k].y : 0u;
#pragma unroll
                        for (uint32_t i = 0; i < 3u; ++i) median3(early[i], f, early[i + 1u]);
                        raise(early[3], f);
                        n_rej += !served && rec[k].x != kNever ? 1u : 0u;
                        rec[k].x = served ? rec[k].x : kNever;
                        rec[k].y = served ? rec[k].y : 1u;
                        rec[k].z = served ? rec[k].z : 0u;
                        rec[k].w = served ? rec[k].w : 0u;
                    }
                }
                uint32_t e2e[4] = {1u, 1u, 1u, 1u}, ttft[4];
#pragma unroll
                for (uint32_t k = 0; k < 4u; ++k) {
                    if (k >= 2u && short_four) continue;
                    const uint32_t f = max(max(rec[k].x, q.t_on), s[0]) + rec[k].y; // padding: kNever + 1
#pragma unroll
                    for (uint32_t i = 0; i < kFront; ++i) {
                        if (i + 1u < kFront) median3(s[i], f, s[i + 1u < kFront ? i + 1u : i]);
                        else raise(s[i], f);
                    }
                    e2e[k] = f - rec[k].x;                                          // padding: 1
                }
                n_run += 4u;
                add_wide(dec_lo, dec_hi, rec[0].z + rec[1].z + rec[2].z + rec[3].z);   // each below 2^28
                add_wide(tpot_lo, tpot_hi, rec[0].w + rec[1].w + rec[2].w + rec[3].w);
#pragma unroll
                for (uint32_t k = 0; k < 4u; ++k) ttft[k] = e2e[k] - rec[k].z;
                if (p.step_facts == (kTpotWithin | kSumsFit)) {
                    add_wide(e2e_lo, e2e_hi, e2e[0] + e2e[1] + e2e[2] + e2e[3]);
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k) n_ok += ttft[k] <= p.slo_ttft ? 1u : 0u;
                } else {
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k) {
                        add_wide(e2e_lo, e2e_hi, e2e[k]);
                        n_ok += (ttft[k] <= p.slo_ttft && rec[k].w <= p.slo_tpot) ? 1u : 0u;
                    }
                }
                if constexpr (kBins_ != 0u) {
                    const bool any_large = (max(max(ttft[0], ttft[1]), max(ttft[2], ttft[3])) >= p.least_us[0]) |
                                           (max(max(rec[0].w, rec[1].w), max(rec[2].w, rec[3].w)) >= p.least_us[1]) |
                                           (max(max(e2e[0], e2e[1]), max(e2e[2], e2e[3])) >= p.least_us[2]);
                    if ((kFew || any_large) && with_hist) {
                        uint32_t bins[4], tpot_bins[4];
#pragma unroll
                        for (uint32_t k = 0; k < 4u; ++k) {
                            tpot_bins[k] = rec[k].x == kNever ? 0u : bin_above(rec[k].w, p.least_us[1], p.least_bin[1]);
                            bins[k] = rec[k].x == kNever ? 0u : bin_above(ttft[k], p.least_us[0], p.least_bin[0]) | (bin_above(e2e[k], p.least_us[2], p.least_bin[2]) << 12) |
                                                                (kBins_ == 2u ? 0u : tpot_bins[k] << 24);
                        }
                        if ((bins[0] | bins[1] | bins[2] | bins[3] | (kBins_ == 2u ? tpot_bins[0] | tpot_bins[1] | tpot_bins[2] | tpot_bins[3] : 0u)) != 0u) {
                            if (kBins_ == 2u) {
                                uint4* dst = reinterpret_cast<uint4*>(reinterpret_cast<uint2*>(p.bins) + bins_at + n_left);
                                dst[0] = make_uint4(bins[0], tpot_bins[0], bins[1], tpot_bins[1]);
                                dst[1] = make_uint4(bins[2], tpot_bins[2], bins[3], tpot_bins[3]);
                            } else {
                                *reinterpret_cast<uint4*>(reinterpret_cast<uint32_t*>(p.bins) + bins_at + n_left) = make_uint4(bins[0], bins[1], bins[2], bins[3]);
                            }
                            n_left += 4u;
                        }
                    }
                }
            }
        }
    }
    if (kBins_ != 0u && with_hist) p.bin_count[(size_t)cb * (p.M + 1u) + m] = n_left;
    for (; j0 < n_t; ++j0)                                                          // nothing starts any more: only counted
        n_over += live ? p.desc[((size_t)cb * p.n_list_tiles + j0) * p.M + m] >> 16 : 0u;
    // steps without a request that was served: each has left a latency of one microsecond, and was within the objectives if that is
    const uint32_t n_padding = n_run - (n_here - n_rej);
    if (p.slo_ttft >= 1u) n_ok -= n_padding;
    const unsigned long long s_e2e = (((unsigned long long)e2e_hi << 32) | e2e_lo) - n_padding;
    const unsigned long long s_tpot = ((unsigned long long)tpot_hi << 32) | tpot_lo;
    const unsigned long long s_ttft = s_e2e - (((unsigned long long)dec_hi << 32) | dec_lo);
    uint32_t last_fin = 0;                                                          // a slot's time is replaced by a later one only: the latest stays
#pragma unroll
    for (uint32_t i = 0; i < kSlots; ++i) last_fin = max(last_fin, s[i] == kNever ? 0u : s[i]);
    if (!live) return;
    // does the listed part leave the streamed part the room the host counted on?
    uint32_t flag = 0u;
    if (q.t_split != kNever) {
        uint32_t busy = 0u;
#pragma unroll
        for (uint32_t i = 0; i < kSlots; ++i) busy += (i < p.B && s[i] > q.t_split) ? 1u : 0u;
        if (busy > q.allow_busy) flag = kFlagFallback;
    }
    SplitPartial* sp = p.part + cb;
    if (s_e2e) atomicAdd(&sp->s_e2e, s_e2e);
    if (s_ttft) atomicAdd(&sp->s_ttft, s_ttft);
    if (s_tpot) atomicAdd(&sp->s_tpot, s_tpot);
    if (last_fin) atomicMax(&sp->last_fin, last_fin);
    if (n_ok) atomicAdd(&sp->n_ok, n_ok);
    if (n_rej + n_over) atomicAdd(&sp->n_rej, n_rej + n_over);
    if (flag) atomicOr(&sp->flags, flag);
}

// Merge: one record per candidate from its partial sums.  A candidate settled by penalty is written by one
// thread; one that the list replay handed back gets the pending mark (the general replay scores it next); for
// the others a workgroup takes the streamed requests' histograms from device memory, adds the bins the list replay
// left and goes through the usual block-wide reduction.
template <bool kHist16>
__global__ __launch_bounds__(kThreads) void k_merge_candidates(EvalParams p, SplitParams sp, ap_metrics* __restrict__ out,
                                                               uint32_t c0, uint32_t n_cand, PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds);
    unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(lds + p.off_misc);
    uint32_t* acc32 = reinterpret_cast<uint32_t*>(lds + p.off_misc + 24);
    uint32_t* wtot = reinterpret_cast<uint32_t*>(lds + p.off_misc + 64);
    uint32_t* n_before = wtot + 3u * kWaves;                                         // [n_queues], and then
    uint32_t* at_of = n_before + sp.n_queues;                                        // [n_queues]
    const uint32_t tid = threadIdx.x;
    if (split_nothing_pending(sp)) return;
    // One workgroup per candidate that needs its histograms; the others are one thread's work each, so a
    // workgroup first settles a run of kThreads of them.
    for (uint32_t base = blockIdx.x * kThreads; base < n_cand; base += gridDim.x * kThreads) {
        const uint32_t cb = base + tid;
        if (cb < n_cand && split_wanted(sp, cb)) {
            const SplitPartial part = sp.part[cb];
            if (part.flags & kFlagFallback) {
                unsigned long long* dst = reinterpret_cast<unsigned long long*>(&out[c0 + cb]);
#pragma unroll
                for (uint32_t i = 0; i < 8u; ++i) dst[i] = ~0ull;
                pending_raise(flags);
            } else if (part.flags & kFlagLazy) {
                const unsigned long long penalty = (unsigned long long)part.n_rej * p.penalty;
                const unsigned long long edge = hist_lower_edge(p.penalty_bin);
                ap_metrics mt;
                mt.sum_e2e_us = part.s_e2e + penalty;
                mt.sum_ttft_us = part.s_ttft + penalty;
                mt.sum_tpot_us = part.s_tpot + penalty;
                mt.makespan_us = part.last_fin;
                mt.p99_ttft_us = edge;
                mt.p99_tpot_us = edge;
                mt.p99_e2e_us = edge;
                mt.slo_ok = part.n_ok;
                mt.n_rejected = part.n_rej;
                out[c0 + cb] = mt;
            }
        }
    }
    // Where all are settled, the workgroup learns it from one load per thread instead of one after the other (8192 candidates:
    // 9 against 6 us).
    bool any = false;
    for (uint32_t c = blockIdx.x + tid * gridDim.x; c < n_cand; c += kThreads * gridDim.x)
        any = any || (sp.part[c].flags & (kFlagFallback | kFlagLazy)) == 0u;
    const bool any_here = __ballot(any) != 0ull;                                     // one store per wavefront
    if ((tid & 63u) == 0u) wtot[wave_index()] = any_here ? 1u : 0u;
    __syncthreads();
    uint32_t n_any = 0u;
    for (uint32_t ww = 0; ww < kWaves; ++ww) n_any += wtot[ww];
    if (n_any == 0u) return;
    for (uint32_t c = blockIdx.x; c < n_cand; c += gridDim.x) {
        const SplitPartial part = sp.part[c];                                       // the same for every thread
        if (!split_wanted(sp, c) || (part.flags & (kFlagFallback | kFlagLazy))) continue;
        const uint32_t* src = sp.hist + (size_t)c * sp.hist_words;
        const bool parked = (part.flags & kFlagNoStreamHist) == 0u;
        // (a word at a time this is 20 waits in a row: 54 against 42 us for 3895 rows of 1920 requests)
        static_assert(3u * kBins / 2u % 4u == 0u, "histograms are copied 16 bytes at a time");
        for (uint32_t i = tid; i < sp.hist_words / 4u; i += kThreads)
            reinterpret_cast<uint4*>(hist)[i] = parked ? reinterpret_cast<const uint4*>(src)[i] : make_uint4(0u, 0u, 0u, 0u);
        if (tid < 16u) reinterpret_cast<uint32_t*>(acc64)[tid] = 0u;
        __syncthreads();
        // The words of all queues as one sequence, four at a time and a four per thread, however they are spread over the queues:
        // n_before[i] fours lie before queue i's, and the sequence's f-th four is the candidate's (f + at_of[i])-th.  (With a queue per
        // wavefront, or per lane where there are many, one long queue kept the workgroup waiting: 559 rows of 60000 requests that crowd 42
        // of 256 replicas 383 us, 131 before bins were compact, 80 now; 11184 of 3000 on one of 8, 472, 261 and 135; one row of 16384 on
        // 2 replicas, 57, 26 and 19.)
        const size_t bins_at = (size_t)c * sp.n_list_tiles * sp.tile_cap, queues_at = (size_t)c * (sp.M + 1u);
        uint32_t n_fours = 0;
        for (uint32_t base = 0; base < sp.n_queues; base += kThreads) {
            const uint32_t i = base + tid, m = i < sp.n_queues ? sp.order[i] : 0u;
            const uint32_t n = i < sp.n_queues ? sp.bin_count[queues_at + m] / 4u : 0u, first = sp.bin_base[queues_at + m] / 4u;
            const uint32_t upto = wave_inclusive_scan(n, tid & 63u);
            if ((tid & 63u) == 63u) wtot[wave_index()] = upto;
            __syncthreads();
            uint32_t before = n_fours + upto - n;
#pragma unroll
            for (uint32_t ww = 0; ww < kWaves; ++ww) {
                before += ww < wave_index() ? wtot[ww] : 0u;
                n_fours += wtot[ww];
            }
            if (i < sp.n_queues) {
                n_before[i] = before;
                at_of[i] = first - before;
            }
            __syncthreads();
        }
        auto add = [&](uint32_t both, uint32_t tpot) {
            const uint32_t ttft = both & 0xFFFu, e2e = (both >> 12) & 0xFFFu;
            if (ttft != 0u) hist_add<kHist16>(hist, 0u, min(sp.least_bin[0] + ttft - 1u, kBins - 1u), 1u);
            if (tpot != 0u) hist_add<kHist16>(hist, 1u, min(sp.least_bin[1] + tpot - 1u, kBins - 1u), 1u);
            if (e2e != 0u) hist_add<kHist16>(hist, 2u, min(sp.least_bin[2] + e2e - 1u, kBins - 1u), 1u);
        };
        for (uint32_t f = tid; f < n_fours; f += kThreads) {
            uint32_t i = 0;                                                         // the last queue that begins at or before it
            for (uint32_t step = 1u << (31u - (uint32_t)__clz((int)sp.n_queues)); step != 0u; step /= 2u)
                if (i + step < sp.n_queues && n_before[i + step] <= f) i += step;
            const size_t at = bins_at / 4u + (uint32_t)(f + at_of[i]);
            if (sp.wide_bins != 0u) {
                const uint4 v = reinterpret_cast<const uint4*>(sp.bins)[2u * at], u = reinterpret_cast<const uint4*>(sp.bins)[2u * at + 1u];
                add(v.x, v.y);
                add(v.z, v.w);
                add(u.x, u.y);
                add(u.z, u.w);
            } else {
                const uint4 v = reinterpret_cast<const uint4*>(sp.bins)[at];
                add(v.x, v.x >> 24);
                add(v.y, v.y >> 24);
                add(v.z, v.z >> 24);
                add(v.w, v.w >> 24);
            }
        }
        __syncthreads();
        const bool first_thread = tid == 0u;
        finish_candidate<kHist16, true>(p, hist, acc64, acc32, wtot, first_thread ? part.s_e2e : 0ull,
                                        first_thread ? part.s_ttft : 0ull, first_thread ? part.s_tpot : 0ull,
                                        first_thread ? part.last_fin : 0u, first_thread ? part.n_ok : 0u,
                                        first_thread ? part.n_rej : 0u, &out[c0 + c]);
        __syncthreads();
    }
}

}  // namespace

#endif  // AP_SPLIT_HPP
