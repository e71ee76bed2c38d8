// Sparse candidates: parent occupancy and the per-child shortcut / row writer.
#ifndef AP_CHILDREN_HPP
#define AP_CHILDREN_HPP

#include "ap_common.hpp"

namespace {

// ----------------------------------------------------------------------------------
// sparse candidates: children of one parent row, given as lists of (request, replica) edits
// ----------------------------------------------------------------------------------
// Children are small modifications of a parent (Section 5.4 "Synthesis Configuration",
// trade-off-aware mutation; Section 6.1 "Warm-start re-evolution": top candidates along with
// their mutations).  A child's row is the parent's with its edits applied front to back; a later
// edit of a request replaces an earlier one and an edit naming a request >= R changes nothing.
//
// With identical, always-available replicas the parent is analysed once (k_parent_occupancy):
// peak[m] is the largest number of the parent's requests replica m has in service at the same
// moment when nobody waits, i.e. the depth of the intervals [arrival, arrival + service).  A
// child's requests on replica m are a subset of the parent's there plus the requests its edits
// send to m, so their depth is at most peak[m] + (edits naming m).  Where that stays within B for
// every replica no request of the child ever finds the B slots taken, nobody waits, and the
// child's record is the nominal one - decided from the edit list alone, without its row.  Every
// other child gets its row written out and goes through the dense path (screening, then replay).
struct ChildParams {
    const uint16_t* parent;       // [R]
    const uint32_t* room;         // [M] B - peak[m], or 0 where the parent already exceeds B
    const ap_metrics* nominal;
    uint16_t* rows;               // [max_children][R] rows of the children the dense path has to look at
    uint32_t R, M, key_bits;      // key_bits: bits of R - 1
    uint32_t certify;             // 0: no shortcut (replicas differ, windows, parent not contention-free): rows for all
};

constexpr uint32_t kChildWaves = 4;
constexpr uint32_t kChildThreads = kChildWaves * kWave;
constexpr uint32_t kOccupancyThreads = 1024;
constexpr uint32_t kOccupancyWaves = kOccupancyThreads / kWave;
constexpr uint32_t kOccupancyPerThread = 8;       // parent ids per thread and step
constexpr uint32_t kOccupancyStep = kOccupancyThreads * kOccupancyPerThread;
constexpr uint32_t kOccupancyTile = 2u * kOccupancyThreads;                 // requests whose depths are counted together
constexpr uint32_t kOccupancyListCap = kOccupancyStep + kOccupancyTile;

// One workgroup per replica walks the parent row in steps of 8192 ids.  All its threads pick out
// the replica's requests of the step (each thread 8 consecutive ids; counts scanned across the
// workgroup; request indices appended to an LDS list in arrival order).  Whenever the list holds a
// tile of 2048 requests, and once more at the end, the depths of the tile's requests are counted,
// two requests per thread: the depth at a request's arrival is one plus the number of earlier
// requests whose unqueued finish time is later than that arrival.  Earlier requests of the same
// tile are looked at backwards from the request, as far as an arrival plus the tile's longest
// service time still reaches past this arrival (arrivals are in order, so nothing before that can
// still be in service).  Requests of earlier tiles are represented by the 64 latest finish times
// seen so far (`latest`, ascending across the lanes of the first wavefront, kept by dropping the
// earliest and inserting the new one where it belongs): if fewer than 64 earlier requests are
// still in service they are all among those, and 64 or more make the depth exceed every B anyway.
// A depth above 64 is reported as 65.  peak[M] counts the parent's requests that name no replica
// of the table.
__global__ __launch_bounds__(kOccupancyThreads) void k_parent_occupancy(EvalParams p, const uint16_t* __restrict__ parent,
                                                                        uint32_t* __restrict__ peak,
                                                                        uint32_t* __restrict__ room) {
    __shared__ uint32_t list[kOccupancyListCap];  // this replica's requests not yet counted, in arrival order
    __shared__ uint32_t tile_arrival[kOccupancyTile], tile_finish[kOccupancyTile];
    __shared__ uint32_t carry[kWave];             // `latest` as the tile being counted sees it
    __shared__ uint32_t wave_total[kOccupancyWaves];
    __shared__ uint32_t longest;                  // longest service time of the tile
    __shared__ uint32_t wg_deepest;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = wave_index(), m = blockIdx.x;
    const DevReplica rp = p.rep[0];
    uint32_t latest = 0u, deepest = 0u, unknown = 0u, n_list = 0u;
    bool have_carry = false;
    if (tid == 0u) {
        longest = 0u;
        wg_deepest = 0u;
    }

    // Counts the depths of list[0 .. n_tile) and takes them off the list.  Called by all threads with the same
    // arguments; more_follow: requests after this tile may exist, so `latest` has to be brought up to date.
    auto count_tile = [&](uint32_t n_tile, bool more_follow) {
        uint32_t my_arrival[2] = {0u, 0u}, my_longest = 0u;
#pragma unroll
        for (uint32_t q = 0; q < 2u; ++q) {
            const uint32_t i = tid + q * kOccupancyThreads;
            if (i < n_tile) {
                const uint32_t r = list[i];
                uint32_t prefill, tpot;
                request_cost(p.tab_prefill, p.tab_tpot, rp, r, p.prompt[r], prefill, tpot);
                const uint32_t service = prefill + p.outlen[r] * tpot;
                my_arrival[q] = p.arrival[r];
                tile_arrival[i] = my_arrival[q];
                tile_finish[i] = my_arrival[q] + service;
                my_longest = max(my_longest, service);
            }
        }
        my_longest = wave_all_max(my_longest);
        if (lane == 0u && my_longest != 0u) atomicMax(&longest, my_longest);
        if (wv == 0u) carry[lane] = latest;
        __syncthreads();
        const uint32_t reach = longest;
#pragma unroll
        for (uint32_t q = 0; q < 2u; ++q) {
            const uint32_t i = tid + q * kOccupancyThreads;
            if (i < n_tile) {
                const uint32_t a = my_arrival[q];
                uint32_t depth = 1u;
                if (have_carry)
                    for (uint32_t l = 0; l < kWave; ++l) depth += carry[l] > a ? 1u : 0u;
                for (uint32_t j = i; j > 0u && tile_arrival[j - 1u] + reach > a; --j) depth += tile_finish[j - 1u] > a ? 1u : 0u;
                deepest = max(deepest, min(depth, 65u));
            }
        }
        if (more_follow && wv == 0u) {
            for (uint32_t i0 = 0; i0 < n_tile; i0 += kWave) {
                const uint32_t finish = i0 + lane < n_tile ? tile_finish[i0 + lane] : 0u;
                const uint32_t n_here = min(kWave, n_tile - i0);
                for (uint32_t k = 0; k < n_here; ++k) {
                    const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)finish, (int)k);
                    latest = min(wave_shift_down(latest, kNever), max(latest, f));
                }
            }
        }
        __syncthreads();                          // everyone is done with the tile and with list[0 .. n_tile)
        // close the gap: a thread only touches the positions congruent to its own index, front to back
        for (uint32_t d = tid; d + n_tile < n_list; d += kOccupancyThreads) list[d] = list[d + n_tile];
        if (tid == 0u) longest = 0u;
        n_list -= n_tile;
        have_carry = true;
        __syncthreads();
    };

    // my 8 ids of a step: one 16-byte load where the row has them all (the parent buffer is 16-byte aligned
    // and a thread's run starts at a multiple of 8 ids), one by one at the ragged end
    auto fetch = [&](uint4& into, uint32_t r0) {
        const uint32_t at = r0 + tid * kOccupancyPerThread;
        if (at + kOccupancyPerThread <= p.R) {
            into = *reinterpret_cast<const uint4*>(parent + at);
        } else {
            uint32_t w[4];
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                const uint32_t lo = at + 2u * k < p.R ? (uint32_t)parent[at + 2u * k] : 0xFFFFu;
                const uint32_t hi = at + 2u * k + 1u < p.R ? (uint32_t)parent[at + 2u * k + 1u] : 0xFFFFu;
                w[k] = lo | (hi << 16);
            }
            into = make_uint4(w[0], w[1], w[2], w[3]);
        }
    };
    uint4 ids_next;
    fetch(ids_next, 0u);
    __syncthreads();                              // longest and wg_deepest are set
    for (uint32_t r0 = 0; r0 < p.R; r0 += kOccupancyStep) {
        // as a bit mask: which of my 8 ids name this replica (absent ones read as 0xFFFF and are skipped below)
        const uint32_t mine = r0 + tid * kOccupancyPerThread;
        const uint32_t w[4] = {ids_next.x, ids_next.y, ids_next.z, ids_next.w};
        if (r0 + kOccupancyStep < p.R) fetch(ids_next, r0 + kOccupancyStep);   // in flight during the rest of this step
        uint32_t hits = 0u;
#pragma unroll
        for (uint32_t k = 0; k < kOccupancyPerThread; ++k) {
            const uint32_t id = (w[k >> 1] >> ((k & 1u) << 4)) & 0xFFFFu;
            const bool present = mine + k < p.R;
            hits |= (present && id == m ? 1u : 0u) << k;
            unknown += (present && id >= p.M) ? 1u : 0u;
        }
        const uint32_t n_mine = (uint32_t)__popc(hits);
        const uint32_t upto = wave_inclusive_scan(n_mine, lane);
        if (lane == 63u) wave_total[wv] = upto;
        __syncthreads();
        uint32_t at = n_list + upto - n_mine, n_step = 0u;
#pragma unroll
        for (uint32_t j = 0; j < kOccupancyWaves; ++j) {
            at += j < wv ? wave_total[j] : 0u;
            n_step += wave_total[j];
        }
        for (uint32_t h = hits; h != 0u; h &= h - 1u) list[at++] = mine + (uint32_t)__ffs((int)h) - 1u;
        n_list += n_step;                         // below kOccupancyListCap: less than a tile was left over
        __syncthreads();                          // the list is written; wave_total may be rewritten
        const bool last_step = r0 + kOccupancyStep >= p.R;
        while (n_list >= kOccupancyTile) count_tile(kOccupancyTile, !(last_step && n_list == kOccupancyTile));
        if (last_step && n_list > 0u) count_tile(n_list, false);
    }
    deepest = wave_all_max(deepest);
    if (lane == 0u) atomicMax(&wg_deepest, deepest);
    __syncthreads();
    if (tid == 0u) {
        const uint32_t d = wg_deepest;
        peak[m] = d;
        room[m] = d <= p.B ? p.B - d : 0u;
    }
    if (m == 0u) {
        unknown = wave_sum_u32(unknown);
        if (lane == 0u) wave_total[wv] = unknown;
        __syncthreads();
        if (tid == 0u) {
            uint32_t total = 0u;
            for (uint32_t j = 0; j < kOccupancyWaves; ++j) total += wave_total[j];
            peak[p.M] = total;
        }
    }
}

// Eight ids of the parent from any position on, as four words.  The parent is 4-byte aligned and has 16 bytes behind it.
__device__ __forceinline__ uint4 parent_ids(const uint16_t* __restrict__ parent, uint32_t at) {
    const uint32_t* s = reinterpret_cast<const uint32_t*>(parent) + at / 2u;
    if (at % 2u == 0u) return make_uint4(s[0], s[1], s[2], s[3]);
    return make_uint4((s[0] >> 16) | (s[1] << 16), (s[1] >> 16) | (s[2] << 16), (s[2] >> 16) | (s[3] << 16), (s[3] >> 16) | (s[4] << 16));
}

// A wavefront copies the parent to a row that begins on any 2-byte boundary: 16-byte stores to aligned addresses.
__device__ __forceinline__ void copy_row(uint16_t* __restrict__ row, const uint16_t* __restrict__ parent, uint32_t R, uint32_t lane) {
    const uint32_t head = min(R, (uint32_t)((16u - (reinterpret_cast<uintptr_t>(row) & 15u)) & 15u) / 2u);   // ids before the first unit
    const uint32_t n_units = (R - head) / 8u;
    if (lane < head) row[lane] = parent[lane];
    for (uint32_t i = head + 8u * n_units + lane; i < R; i += kWave) row[i] = parent[i];
    uint4* dst = reinterpret_cast<uint4*>(row + head);
#pragma unroll 4
    for (uint32_t i = lane; i < n_units; i += kWave) dst[i] = parent_ids(parent, head + 8u * i);
}

// The rows of all children, where none can be settled from its edits alone (replicas that differ, a parent that queues
// itself).  A workgroup per child; the row goes by in chunks.  For every request of the chunk in hand the LDS holds the
// number of the last edit that names it (atomic maximum, so the order of the list decides and nothing has to be done in
// order), then every thread puts eight ids together and stores them at once.  1097 rows of 30284 requests with 1202 edits
// each take 0.06 ms; one wavefront per child that copied the parent and then stored edit after edit took 0.4 ms (a fence, a
// ballot per bit of the request number and 64 scattered 2-byte stores per batch of 64 edits).
constexpr uint32_t kRowThreads = 256;
constexpr uint32_t kRowChunk = 8192;              // requests per chunk: 32 KiB of LDS, five workgroups per compute unit
__global__ __launch_bounds__(kRowThreads) void k_write_children(ChildParams p, const uint32_t* __restrict__ first,
                                                                const uint32_t* __restrict__ request,
                                                                const uint16_t* __restrict__ replica, uint32_t C, PendingWord flags) {
    __shared__ __align__(16) uint32_t last[kRowChunk];                       // 1 + number of the edit within the list; 0: none
    pending_clear_next(flags);
    const uint32_t tid = threadIdx.x;
    for (uint32_t c = blockIdx.x; c < C; c += gridDim.x) {
        const uint32_t e0 = first[c], e1 = first[c + 1u], n_edits = e0 < e1 ? e1 - e0 : 0u;   // empty or reversed: no edits
        uint16_t* row = p.rows + (size_t)c * p.R;
        // the row as beginning `a` positions into its first 16-byte unit
        const uint32_t a = (uint32_t)(reinterpret_cast<uintptr_t>(row) >> 1) & 7u, n = p.R + a;
        for (uint32_t p0 = 0; p0 < n; p0 += kRowChunk) {
            const uint32_t here = min(kRowChunk, (n - p0 + 7u) & ~7u);
            for (uint32_t i = 4u * tid; i < here; i += 4u * kRowThreads) *reinterpret_cast<uint4*>(&last[i]) = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            for (uint32_t e = tid; e < n_edits; e += kRowThreads) {
                const uint32_t r = request[e0 + e];
                if (r < p.R && r + a >= p0 && r + a - p0 < kRowChunk) atomicMax(&last[r + a - p0], e + 1u);
            }
            __syncthreads();
            for (uint32_t i = 8u * tid; i < here; i += 8u * kRowThreads) {
                const uint4 l0 = *reinterpret_cast<const uint4*>(&last[i]), l1 = *reinterpret_cast<const uint4*>(&last[i + 4u]);
                const uint32_t from[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
                const uint32_t at = p0 + i;                                  // position of the first of the eight
                if (at >= a && at + 8u <= n) {
                    const uint4 v = parent_ids(p.parent, at - a);
                    uint32_t word[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (uint32_t k = 0; k < 8u; ++k)
                        if (from[k] != 0u) {
                            const uint32_t shift = (k & 1u) * 16u;
                            word[k >> 1] = (word[k >> 1] & ~(0xFFFFu << shift)) | ((uint32_t)replica[e0 + from[k] - 1u] << shift);
                        }
                    *reinterpret_cast<uint4*>(row - a + at) = make_uint4(word[0], word[1], word[2], word[3]);
                } else {
                    for (uint32_t k = 0; k < 8u; ++k)
                        if (at + k >= a && at + k < n) row[at + k - a] = from[k] != 0u ? replica[e0 + from[k] - 1u] : p.parent[at + k - a];
                }
            }
            __syncthreads();
        }
    }
}

// One wavefront per child, where the parent leaves room: count the child's edits per replica in LDS and compare with
// the room the parent leaves; a child that passes gets the nominal record.  A child that does not
// pass (too many edits for some replica, or an edit naming a replica outside the table) gets the
// pending mark and its row: the parent's, then its edits in batches of 64, the lanes of a batch
// that name the same request settled in favour of the highest lane, batches in list order.
__global__ __launch_bounds__(kChildThreads, 7) void k_certify_children(ChildParams p, const uint32_t* __restrict__ first,
                                                                    const uint32_t* __restrict__ request,
                                                                    const uint16_t* __restrict__ replica,
                                                                    ap_metrics* __restrict__ out, uint32_t C,
                                                                    PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    pending_clear_next(flags);
    const uint32_t lane = threadIdx.x & 63u, w = wave_index();
    uint32_t* count = reinterpret_cast<uint32_t*>(lds) + w * p.M;            // this wavefront's: edits per replica
    uint32_t* room = reinterpret_cast<uint32_t*>(lds) + kChildWaves * p.M;   // the workgroup's copy of p.room
    for (uint32_t m = lane; m < p.M; m += kWave) count[m] = 0u;
    unsigned long long nominal_word = 0ull;                                  // lanes 0..7: the record of a child that passes
    for (uint32_t m = threadIdx.x; m < p.M; m += kChildThreads) room[m] = p.room[m];
    if (lane < 8u) nominal_word = reinterpret_cast<const unsigned long long*>(p.nominal)[lane];
    __syncthreads();
    for (uint32_t c = blockIdx.x * kChildWaves + w; c < C; c += gridDim.x * kChildWaves) {
        const unsigned long long e0 = first[c], e1 = first[c + 1u];          // empty or reversed: no edits
        bool fail = false;
        // rounds of kInFlight loads of both arrays per lane; the next round is requested before the
        // current one is counted, so the lists stream in without a pause between rounds
        constexpr uint32_t kInFlight = 8;
        uint32_t r[kInFlight], m[kInFlight], r_next[kInFlight], m_next[kInFlight];
        auto fetch = [&](uint32_t (&rq)[kInFlight], uint32_t (&rp)[kInFlight], unsigned long long b) {
#pragma unroll
            for (uint32_t k = 0; k < kInFlight; ++k) {
                const unsigned long long e = b + k * kWave + lane;
                rq[k] = e < e1 ? request[e] : kNoKey;                    // past the end: names no request
                rp[k] = e < e1 ? (uint32_t)replica[e] : 0u;
            }
        };
        if (e0 < e1) fetch(r_next, m_next, e0);
        for (unsigned long long b = e0; b < e1; b += kInFlight * kWave) {
#pragma unroll
            for (uint32_t k = 0; k < kInFlight; ++k) {
                r[k] = r_next[k];
                m[k] = m_next[k];
            }
            if (b + kInFlight * kWave < e1) fetch(r_next, m_next, b + kInFlight * kWave);
#pragma unroll
            for (uint32_t k = 0; k < kInFlight; ++k) {
                if (r[k] < p.R) {
                    if (m[k] < p.M) atomicAdd(&count[m[k]], 1u);
                    else fail = true;
                }
            }
        }
        for (uint32_t m = lane; m < p.M; m += kWave) {
            fail = fail || count[m] > room[m];
            count[m] = 0u;
        }
        const bool dense = __ballot(fail) != 0ull;
        if (lane < 8u) reinterpret_cast<unsigned long long*>(&out[c])[lane] = dense ? ~0ull : nominal_word;
        if (dense && lane == 0u) pending_raise(flags);
        if (!dense) continue;
        uint16_t* row = p.rows + (size_t)c * p.R;
        copy_row(row, p.parent, p.R, lane);
        // A wavefront's stores to one address take effect in the order of its instructions, whichever lanes make them, so between
        // the copy and a batch, and between batches, only the compiler has to be held (a device-wide fence writes the L2 back
        // each time: 2.4 ms for 9262 rows of 12421 requests with 547 edits each, 0.35 ms so).
        for (unsigned long long b = e0; b < e1; b += kWave) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const unsigned long long e = b + lane;
            const uint32_t r = e < e1 ? request[e] : kNoKey;
            const uint16_t m = e < e1 ? replica[e] : (uint16_t)0;
            bool mine = e < e1 && r < p.R;
            // a batch in increasing order names no request twice
            const uint32_t before = wave_shift_up(r, 0u);                    // all lanes take part
            if (__ballot(lane != 0u && e < e1 && before >= r) != 0ull) {
                uint32_t lo, hi;
                wave_peers(r, p.R, p.key_bits, lo, hi);                      // lanes of this batch naming my request
                const unsigned long long peers = ((unsigned long long)hi << 32) | lo;
                mine = mine && ((peers >> lane) >> 1) == 0ull;
            }
            if (mine) row[r] = m;
        }
    }
}

}  // namespace

#endif  // AP_CHILDREN_HPP
