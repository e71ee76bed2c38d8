// Screening by counting: prove a candidate contention-free from how many requests each replica gets in a window.
#ifndef AP_COUNTS_HPP
#define AP_COUNTS_HPP

#include "ap_common.hpp"
#include "ap_screen.hpp"

namespace {

// ----------------------------------------------------------------------------------
// counting screen
// ----------------------------------------------------------------------------------
// Applies where the slot-ring screens do: identical replicas, always available, so a request that does not wait is in
// service during [arrival, arrival + service) on whichever replica it is.  The row is cut into buckets of w consecutive
// requests.  For every bucket b the host knows from the trace alone the first bucket lo(b) that holds a request still in
// service when bucket b begins (nobody waiting).  If replica m gets at most B requests in buckets lo(b) .. b, for every b,
// then by induction in arrival order none of them waits: whoever is in service on m when a request of bucket b arrives came
// in these buckets and is not the request itself, so at most B - 1 slots are taken.  Hence a candidate that passes for all
// replicas and buckets has the nominal record.  The test is sufficient, not necessary; a candidate that fails (or names an
// unknown replica) gets the pending mark and goes to the slot rings, which look at every interval by itself.
//
// What it takes is one LDS add per request - no per-request table, no answer from the LDS, nothing shared between
// wavefronts - so the kernel reads the rows and little else.  Where the add goes decides the pace: one counter per replica
// sends the 64 lanes of an instruction to random banks (14 LDS cycles each, 0.82 ms on 16384 rows of 131072 requests and
// 128 replicas).  So a lane picks its column: four replicas share a word (a byte each), and every word exists once per column,
// column lane mod n_columns.  Of 64 lanes only those that share a column (4, 8 or 16 of them with 16, 8 or 4 columns) can meet in
// a bank or a word.  When a bucket ends, lane r adds up row r (the four replicas 4 r .. 4 r + 3) over the columns, as whole words.
// Nothing is ever cleared: the words are running sums modulo 2^32, and the difference of two of them is
// n0 + n1 * 2^8 + n2 * 2^16 + n3 * 2^24 modulo 2^32, the four counts of the requests in between, as long as all are below
// 256.  Should one not be, it reads too small and its neighbour too large, and the bytes add up to less than the requests
// in the window - which is therefore compared, summed over all windows of the row, before a candidate passes.
// Counting does not depend on what came before, so several wavefronts can share a row, each starting at lo(its first
// bucket): a call with few candidates is not one serial chain per candidate.
//
// Rows start on any 2-byte boundary.  A lane loads 4 * kVec bytes (2 * kVec requests) from an aligned address, so the
// row is seen as beginning `a` positions into its first aligned unit.  lo(b) allows for every `a`.
struct CountParams {
    const uint32_t* lo;           // [n_buckets] as above, for rows that begin up to kCountShift positions into their first unit
    const ap_metrics* nominal;
    uint32_t R, M, B;
    uint32_t w_log2;              // requests per bucket, log2
    uint32_t ring_mask;           // sums kept per row - 1 (a power of two of them, at least b - lo(b) + 2)
    uint32_t n_rows;              // words per column: a byte for each of the M replicas and one more, for unknown ids
    uint32_t columns_log2;
    uint32_t wave_words;          // LDS words of one wavefront: counters and kept sums
    uint32_t waves_per_row;       // power of two
};
constexpr uint32_t kCountShift = 7u;
constexpr uint32_t kCountMinBucket = 128u;
constexpr uint32_t kCountMaxWaves = 16u;          // wavefronts of a workgroup (and of a row) at most
constexpr uint32_t kCountLdsBytes = 65536u - 256u; // and of counters per workgroup

// lo(b) is the same for every lane: read through the constant address space it stays on the scalar unit.
__device__ __forceinline__ uint32_t count_lo(const uint32_t* lo, uint32_t b) {
    return ((const __attribute__((address_space(4))) uint32_t*)(uintptr_t)lo)[b];
}

// kVec: 4-byte words a lane loads per step (1: 128 requests a step, 4: 512); a bucket is one or more whole steps.
// kColumnsLog2: as CountParams::columns_log2, which it depends on n_rows for; n_rows is at most 64 where it is 4.
template <uint32_t kVec, uint32_t kColumnsLog2>
__global__ __launch_bounds__(kCountMaxWaves * kWave) void k_screen_counts(CountParams p, const uint16_t* __restrict__ assign,
                                                                          ap_metrics* __restrict__ out, uint32_t C,
                                                                          PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t failed[kCountMaxWaves];
    pending_clear_next(flags);
    constexpr uint32_t kStep = 128u * kVec, kPer = 2u * kVec, kDepth = kVec == 1u ? 8u : 2u;
    constexpr uint32_t kColumns = 1u << kColumnsLog2, kQuads = kColumns / 4u;
    constexpr bool kOnePass = kColumnsLog2 == 4u;                            // a lane per row
    const uint32_t lane = threadIdx.x & 63u, wv = wave_index(), n_waves = blockDim.x >> 6;
    const uint32_t R = p.R, M = p.M, n_rows = p.n_rows, ring_mask = p.ring_mask;
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds) + wv * p.wave_words;    // [n_rows][kColumns]
    uint32_t* ring = cnt + n_rows * kColumns;                                // [ring_mask + 1][n_rows]
    const uint32_t rows_here = n_waves / p.waves_per_row;
    const uint32_t part = wv % p.waves_per_row;
    const uint32_t c = blockIdx.x * rows_here + wv / p.waves_per_row;        // the host launches enough workgroups for all of C
    if (threadIdx.x < kCountMaxWaves) failed[threadIdx.x] = 0u;
    if (p.waves_per_row > 1u) __syncthreads();
    bool bad = false;
    if (c < C) {
        const uint16_t* row = assign + (size_t)c * R;
        const uint32_t a = (uint32_t)(reinterpret_cast<uintptr_t>(row) >> 1) & (kPer - 1u);
        const uint32_t n = R + a;                                            // positions
        const uint32_t n_steps = (n + kStep - 1u) / kStep;
        const uint32_t n_buckets = (n + (1u << p.w_log2) - 1u) >> p.w_log2;
        const uint32_t steps_log2 = p.w_log2 - (kVec == 1u ? 7u : 9u);       // steps per bucket
        // this wavefront's buckets, and where it has to begin counting for the first of them
        const uint32_t share = (n_buckets + p.waves_per_row - 1u) / p.waves_per_row;
        const uint32_t b_first = min(part * share, n_buckets), b_end = min(b_first + share, n_buckets);
        const uint32_t b_count = b_first < b_end && b_first != 0u ? count_lo(p.lo, b_first) : 0u;
        const uint32_t s_first = b_count << steps_log2;
        const uint32_t s_end = b_first < b_end ? min(b_end << steps_log2, n_steps) : s_first;
        for (uint32_t i = lane; i < n_rows * kColumns; i += kWave) cnt[i] = 0u;
        for (uint32_t i = lane; i < n_rows; i += kWave) ring[((b_count - 1u) & ring_mask) * n_rows + i] = 0u;
        uint32_t seen = 0, meant = 0;                                        // requests found and requests there, over the checked windows

        // 127 less the limit of each of the row's replicas: a byte above its limit has its top bit set once that is added,
        // or has it already.  The last row: byte M has limit 0, those behind it stay 0.
        auto room_of = [&](uint32_t r) {
            const uint32_t room = (127u - p.B) * 0x01010101u;
            if (4u * r + 4u <= M) return room;
            const uint32_t shift = 8u * (M - 4u * r);
            return (room & ((1u << shift) - 1u)) | (127u << shift);
        };
        const uint32_t my_room = lane < n_rows ? room_of(lane) : 0u;
        auto check_row = [&](uint32_t r, uint32_t room, const uint32_t* old, uint32_t* now, bool full) {
            const uint4* line = reinterpret_cast<const uint4*>(cnt + r * kColumns);
            uint32_t sum = 0;
#pragma unroll
            for (uint32_t i = 0; i < kQuads; ++i) {                          // lanes begin at different columns: different banks
                const uint4 v = line[(i + (r >> 1)) & (kQuads - 1u)];
                sum += v.x + v.y + v.z + v.w;
            }
            now[r] = sum;
            const uint32_t got = sum - old[r];
            if (full) {
                bad = bad || ((got | ((got & 0x7F7F7F7Fu) + room)) & 0x80808080u) != 0u;
                seen = __builtin_amdgcn_sad_u8(got, 0u, seen);               // the four bytes added up
            }
        };
        auto check = [&](uint32_t b) {                                       // bucket b has been counted
            const uint32_t lo = count_lo(p.lo, b);
            const uint32_t* old = ring + ((lo - 1u) & ring_mask) * n_rows;
            uint32_t* now = ring + (b & ring_mask) * n_rows;
            const bool full = b >= b_first;
            if (kOnePass) {
                if (lane < n_rows) check_row(lane, my_room, old, now, full);
            } else {
                for (uint32_t r = lane; r < n_rows; r += kWave) check_row(r, room_of(r), old, now, full);
            }
            if (full) meant += min((b + 1u) << p.w_log2, n) - max(lo << p.w_log2, a);
        };
        auto step_done = [&](uint32_t s) {
            if (((s + 1u) & ((1u << steps_log2) - 1u)) == 0u || s + 1u == n_steps) check(s >> steps_log2);
        };

        // Two ids (the halves of a word) at a time.  `at`: LDS byte addresses of their words in this lane's column, 16 bits
        // each (all of a workgroup's LDS is below 64 KiB); shifts take the lower five bits of their count, 8 (id mod 4).
        typedef unsigned short pair_t __attribute__((ext_vector_type(2)));
        const unsigned short column = (unsigned short)(lds_address(cnt) + (lane & (kColumns - 1u)) * 4u);
        const unsigned short top = (unsigned short)M;
        auto add_pair = [&](uint32_t word, bool first_there, bool second_there) {
            pair_t id;
            __builtin_memcpy(&id, &word, 4);
            id = __builtin_elementwise_min(id, pair_t{top, top});            // unknown replicas: entry M
            const pair_t at = (id & (unsigned short)0xFFFC) * (unsigned short)kColumns + column;
            uint32_t ids, addresses;
            __builtin_memcpy(&ids, &id, 4);
            __builtin_memcpy(&addresses, &at, 4);
            if (first_there) lds_add(addresses & 0xFFFFu, 1u << ((ids << 3) & 31u));
            if (second_there) lds_add(addresses >> 16, 1u << ((ids >> 13) & 31u));
        };
        auto edge_step = [&](uint32_t s) {                                   // a unit that is not all the row's
            for (uint32_t e = 0; e < kVec; ++e) {
                const uint32_t pos = s * kStep + lane * kPer + 2u * e;
                const bool in0 = pos >= a && pos < n, in1 = pos + 1u >= a && pos + 1u < n;
                const uint32_t id0 = in0 ? (uint32_t)row[pos - a] : 0u, id1 = in1 ? (uint32_t)row[pos + 1u - a] : 0u;
                add_pair(id0 | (id1 << 16), in0, in1);
            }
            step_done(s);
        };
        const uint32_t f_first = s_first == 0u && a != 0u ? min(1u, s_end) : s_first;      // whole steps: [f_first, f_end)
        const uint32_t f_end = max(f_first, min(s_end, n / kStep));
        if (f_first > s_first) edge_step(s_first);
        if (f_first < f_end) {
            typedef uint32_t load_t __attribute__((ext_vector_type(kVec)));
            struct Loaded {
                load_t word[kDepth];
            };
            const char* lane_base = reinterpret_cast<const char*>(row - a) + lane * (4u * kVec);
            auto fetch = [&](Loaded& into, uint32_t s0) {                    // a step beyond the end loads the last one again
#pragma unroll
                for (uint32_t d = 0; d < kDepth; ++d)
                    into.word[d] = __builtin_nontemporal_load(reinterpret_cast<const load_t*>(lane_base + (size_t)min(s0 + d, f_end - 1u) * (2u * kStep)));
            };
            auto work = [&](const Loaded& now, uint32_t s0) {
#pragma unroll
                for (uint32_t d = 0; d < kDepth; ++d) {
                    const uint32_t s = s0 + d;
                    if (s >= f_end) break;
#pragma unroll
                    for (uint32_t e = 0; e < kVec; ++e) add_pair(now.word[d][e], true, true);
                    step_done(s);
                }
            };
            Loaded set_a, set_b;
            fetch(set_a, f_first);
            for (uint32_t s = f_first; s < f_end; s += 2u * kDepth) {
                fetch(set_b, s + kDepth);
                work(set_a, s);
                fetch(set_a, s + 2u * kDepth);
                work(set_b, s + kDepth);
                if (__ballot(bad) != 0ull) break;
            }
        }
        bad = __ballot(bad) != 0ull;
        if (!bad && f_end < s_end) edge_step(f_end);
        bad = __ballot(bad) != 0ull || wave_sum_u32(seen) != meant;          // both modulo 2^32
    }
    if (p.waves_per_row > 1u) {
        if (bad && lane == 0u) failed[wv / p.waves_per_row] = 1u;
        __syncthreads();
        bad = failed[wv / p.waves_per_row] != 0u;
    }
    if (c < C && part == 0u) {
        if (lane < 8u) reinterpret_cast<unsigned long long*>(&out[c])[lane] =
            bad ? ~0ull : reinterpret_cast<const unsigned long long*>(p.nominal)[lane];
        if (bad && lane == 0u) pending_raise(flags);
    }
}

}  // namespace

#endif  // AP_COUNTS_HPP
