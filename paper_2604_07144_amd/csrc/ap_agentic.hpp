// Agentic workflows on a disaggregated prefill/decode cluster: one wavefront replays one candidate plan.
#ifndef AP_AGENTIC_HPP
#define AP_AGENTIC_HPP

#include "ap_common.hpp"

namespace {

// ----------------------------------------------------------------------------------
// candidate plans for multi-call workflows (Section 8.3; Appendix, Formulation for Agentic Request)
// ----------------------------------------------------------------------------------
// A call is released when its workflow has arrived and all its predecessors have completed; it is
// prefilled on its prefill instance (one call at a time, the waiting call with the smallest
// (key, index) first), then decoded on its decode instance, which admits its first waiting call as
// soon as the call's in + out tokens fit the free part of the instance's token budget (no
// overtaking).  Events of one instant are applied as decode completions, prefill completions,
// releases, decode admissions, prefill starts.  A call that names no prefill instance fails at its
// release, one that names no decode instance or can never fit fails at the end of its prefill; a
// failed call completes at that instant and its workflow is charged the penalty ratio.  Per
// workflow: ratio = completion time * 1000 / SLO; per candidate: their sum, nearest-rank 95th and
// 99th percentiles, the number of late and of failed workflows, the makespan.
//
// The event loop is serial in time, so the parallelism is across candidates: one wavefront each, and next to nothing of
// it is done lane by lane.  What is running, who waits and what happens next is held so that a step touches only what it
// changes:
//  * the calls in service sit in 64 slots, one per lane (end of the stage, and which call);
//    the next instant is the minimum over them and the next arrival of a workflow.  Calls beyond 64 in service wait
//    for their end in an LDS table by call, which is gone through only when one of them ends;
//  * the calls of a plan are ranked by (key, index) once, before the loop; an instance's queue is a bit mask over ranks in
//    LDS, so its first waiting call is the first bit set, and joining or leaving a queue is one bit;
//  * a completion, release or arrival notes which instances it concerns, and only those try to admit or start a call;
//  * workflows are taken in order of arrival, each with the list of its calls without predecessors.
// Tables that are the same for all plans (lengths, successors, arrivals) are copied to LDS once per workgroup; the
// wavefronts of a workgroup share nothing else and never meet at a barrier after that.
// It is bound by the issue of scalar instructions (225 per call, 178 vector and 25 LDS ones).  Scanning the
// calls' phases at every instant (a lane per 64 calls, masks per lane) took 2.58 ms for 8192 plans of a 330-call slice,
// 1.64 ms now.
struct AgenticParams {
    const uint4* blob;            // the tables that go to LDS, laid out as below
    uint32_t blob_bytes;          // a multiple of 16
    // byte offsets into it
    uint32_t o_lens;              // uint2 [K] {in_len, out_len}
    uint32_t o_arrival;           // uint32 [W] microseconds after the earliest arrival
    uint32_t o_succ_first;        // uint32 [K + 1] successors of call k: succ[succ_first[k] .. succ_first[k + 1])
    uint32_t o_wf;                // uint16 [K]
    uint32_t o_order;             // uint16 [W] workflows by arrival
    uint32_t o_root_first;        // uint16 [W + 1] calls without predecessors of workflow w: root[root_first[w] .. root_first[w + 1])
    uint32_t o_root;              // uint16 [..]
    uint32_t o_n_pred;            // uint8 [K], padded to 4 bytes
    uint32_t o_succ;              // uint16 [..], or 0: too long for LDS, read from `succ`
    const uint16_t* succ;
    const unsigned long long* slo;  // [W]
    const uint32_t* pa;           // [P] prefill: pa + pb * in_len
    const uint32_t* pb;
    const uint32_t* qc;           // [Q] decode: out_len * (qc + qd * ceil(in_len / 1024))
    const uint32_t* qd;
    const uint32_t* cap;          // [Q]
    unsigned long long penalty;
    uint32_t W, K, P, Q;
    // byte offsets into a wavefront's own LDS, which begins behind the blob
    uint32_t o_call;              // uint16 [K] call of a rank
    uint32_t o_rank;              // uint16 [K] rank of a call
    uint32_t o_ids;               // uint16 [K] prefill instance | decode instance << 8 (P resp. Q: none)
    uint32_t o_left;              // uint8 [K] predecessors still to complete
    uint32_t o_comp;              // uint32 [W] completion time per workflow
    uint32_t o_failed;            // uint8 [W]
    uint32_t o_queue;             // uint32 [P + Q][2 chunks] waiting calls by rank
    uint32_t o_over;              // uint32 [K] end of the stage of a call in service without a slot, else kNever
    uint32_t o_over_phase;        // uint8 [K] its phase
    uint32_t wave_bytes;          // LDS per wavefront (offset 0: uint64 ratios [W], once the event loop is over, before that o_over)
};

constexpr uint32_t kAgenticWaves = 4;             // at most; fewer where the tables are large
constexpr uint32_t kAgenticThreads = kAgenticWaves * kWave;
constexpr uint32_t kAgenticLdsSuccessors = 4096;  // successor lists up to this length are kept in LDS

__device__ __forceinline__ void wave_sync_lds() {
    // LDS writes of any lane of this wavefront are visible to the lanes' later reads; keeps the compiler
    // from carrying LDS values across the point
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Wavefront-wide reductions on the cross-lane data path of the vector ALU (no trip through LDS, which
// the per-lane shuffles would take): an inclusive scan inside each row of 16 lanes by shifting the row
// right by 1, 2, 4 and 8 lanes (a lane with no source keeps the identity), then the last lane of row 0
// and of row 2 sent to rows 1 and 3, then lane 31 to rows 2 and 3; lane 63 holds the result, which is
// handed to every lane as a uniform value.
#define AP_DPP(identity, v, ctrl, rows) \
    (uint32_t)__builtin_amdgcn_update_dpp((int)(identity), (int)(v), ctrl, rows, 0xF, false)
__device__ __forceinline__ uint32_t wave_all_or(uint32_t v) {
    v |= AP_DPP(0u, v, 0x111, 0xF);                                          // row_shr:1
    v |= AP_DPP(0u, v, 0x112, 0xF);                                          // row_shr:2
    v |= AP_DPP(0u, v, 0x114, 0xF);                                          // row_shr:4
    v |= AP_DPP(0u, v, 0x118, 0xF);                                          // row_shr:8
    v |= AP_DPP(0u, v, 0x142, 0xA);                                          // row_bcast:15 into rows 1 and 3
    v |= AP_DPP(0u, v, 0x143, 0xC);                                          // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_all_min(uint32_t v) {
    v = min(v, AP_DPP(kNever, v, 0x111, 0xF));
    v = min(v, AP_DPP(kNever, v, 0x112, 0xF));
    v = min(v, AP_DPP(kNever, v, 0x114, 0xF));
    v = min(v, AP_DPP(kNever, v, 0x118, 0xF));
    v = min(v, AP_DPP(kNever, v, 0x142, 0xA));
    v = min(v, AP_DPP(kNever, v, 0x143, 0xC));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
#undef AP_DPP
__device__ __forceinline__ unsigned long long wave_all_or64(unsigned long long v) {
    return ((unsigned long long)wave_all_or((uint32_t)(v >> 32)) << 32) | wave_all_or((uint32_t)v);
}

__device__ __forceinline__ uint32_t wave_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint32_t wave_lane(uint32_t v, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane); }

// kChunks: 64-call chunks of a plan, at least ceil(K / 64).
template <uint32_t kChunks>
__global__ __launch_bounds__(kAgenticThreads) void k_agentic_eval(AgenticParams p, const uint16_t* __restrict__ pre_inst,
                                                                  const uint16_t* __restrict__ dec_inst,
                                                                  const uint32_t* __restrict__ key,
                                                                  ap_agentic_metrics* __restrict__ out, uint32_t C) {
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t lane = threadIdx.x & 63u, wv = wave_index(), n_waves = blockDim.x >> 6;
    const uint32_t K = p.K, W = p.W, P = p.P, Q = p.Q;
    constexpr uint32_t kWords = 2u * kChunks;                    // 32-bit words of a queue's mask
    constexpr uint32_t kInPrefill = 0u, kInDecode = 1u, kUnplaced = 2u;   // phases; unplaced: over at this instant, naming no prefill instance
    for (uint32_t i = threadIdx.x; i < p.blob_bytes / 16u; i += blockDim.x) reinterpret_cast<uint4*>(lds)[i] = p.blob[i];
    __syncthreads();
    const uint2* lens = reinterpret_cast<const uint2*>(lds + p.o_lens);
    const uint32_t* arrival = reinterpret_cast<const uint32_t*>(lds + p.o_arrival);
    const uint32_t* succ_first = reinterpret_cast<const uint32_t*>(lds + p.o_succ_first);
    const uint16_t* wf = reinterpret_cast<const uint16_t*>(lds + p.o_wf);
    const uint16_t* order = reinterpret_cast<const uint16_t*>(lds + p.o_order);
    const uint16_t* root_first = reinterpret_cast<const uint16_t*>(lds + p.o_root_first);
    const uint16_t* root = reinterpret_cast<const uint16_t*>(lds + p.o_root);
    const uint16_t* succ_lds = reinterpret_cast<const uint16_t*>(lds + p.o_succ);
    unsigned char* mine = lds + p.blob_bytes + wv * p.wave_bytes;
    unsigned long long* ratio = reinterpret_cast<unsigned long long*>(mine);
    uint16_t* call_of = reinterpret_cast<uint16_t*>(mine + p.o_call);
    uint16_t* rank_of = reinterpret_cast<uint16_t*>(mine + p.o_rank);
    uint16_t* ids = reinterpret_cast<uint16_t*>(mine + p.o_ids);
    unsigned char* left = mine + p.o_left;
    uint32_t* comp = reinterpret_cast<uint32_t*>(mine + p.o_comp);
    unsigned char* wf_failed = mine + p.o_failed;
    uint32_t* queue = reinterpret_cast<uint32_t*>(mine + p.o_queue);           // prefill instances, then decode instances
    uint32_t* over = reinterpret_cast<uint32_t*>(mine + p.o_over);
    unsigned char* over_phase = mine + p.o_over_phase;
    // lane i holds the constants of prefill instance i and of decode instance i
    const uint32_t pa = lane < P ? p.pa[lane] : 0u, pb = lane < P ? p.pb[lane] : 0u;
    const uint32_t qc = lane < Q ? p.qc[lane] : 0u, qd = lane < Q ? p.qd[lane] : 0u, cap = lane < Q ? p.cap[lane] : 0u;

    for (uint32_t c = blockIdx.x * n_waves + wv; c < C; c += gridDim.x * n_waves) {
        uint32_t my_key[kChunks], rank[kChunks];
#pragma unroll
        for (uint32_t j = 0; j < kChunks; ++j) {
            const uint32_t k = j * kWave + lane;
            my_key[j] = k < K ? key[(size_t)c * K + k] : 0u;
            rank[j] = 0u;
            if (k < K) {
                over[k] = kNever;
                ids[k] = (uint16_t)(min((uint32_t)pre_inst[(size_t)c * K + k], P) | (min((uint32_t)dec_inst[(size_t)c * K + k], Q) << 8));
            }
        }
        for (uint32_t i = lane; i < (K + 3u) / 4u; i += kWave)
            reinterpret_cast<uint32_t*>(left)[i] = reinterpret_cast<const uint32_t*>(lds + p.o_n_pred)[i];
        for (uint32_t w = lane; w < W; w += kWave) {
            comp[w] = arrival[w];                                // a workflow without calls completes on arrival
            wf_failed[w] = 0;
        }
        for (uint32_t i = lane; i < (P + Q) * kWords; i += kWave) queue[i] = 0u;
        wave_sync_lds();
        // rank by (key, index): earlier calls count at equal keys, later ones do not
#pragma unroll
        for (uint32_t jv = 0; jv < kChunks; ++jv) {
            const uint32_t n = K > jv * kWave ? min(K - jv * kWave, kWave) : 0u;
#pragma unroll 4
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t o = wave_lane(my_key[jv], i);
#pragma unroll
                for (uint32_t j = 0; j < kChunks; ++j) {
                    if (j > jv) rank[j] += o <= my_key[j] ? 1u : 0u;
                    else if (j < jv) rank[j] += o < my_key[j] ? 1u : 0u;
                    else rank[j] += (o < my_key[j] || (o == my_key[j] && i < lane)) ? 1u : 0u;
                }
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kChunks; ++j) {
            const uint32_t k = j * kWave + lane;
            if (k < K) {
                rank_of[k] = (uint16_t)rank[j];
                call_of[rank[j]] = (uint16_t)k;
            }
        }
        wave_sync_lds();

        uint32_t ends = kNever, who = 0u;                        // this lane's slot: end of the stage (kNever: free), call | phase << 10
        uint32_t t_over = kNever;                                // the first end among the calls in service without one
        uint32_t room = cap;                                     // lane q: free tokens of decode instance q
        unsigned long long busy = 0ull;                          // prefill instances at work
        unsigned long long try_pre = 0ull, try_dec = 0ull;       // instances something has changed for
        uint32_t t = 0u, last_done = 0u, n_arrived = 0u;         // times are relative to the earliest arrival: the first instant is 0
        uint32_t next_arrival = 0u;
        bool again = false;

        auto occupy = [&](uint32_t end, uint32_t k, uint32_t phase) {
            const unsigned long long free = __ballot(ends == kNever);
            if (free != 0ull) {
                const bool me = lane == (uint32_t)__ffsll((long long)free) - 1u;
                ends = me ? end : ends;
                who = me ? k | (phase << 10) : who;
            } else {
                if (lane == 0u) {
                    over[k] = end;
                    over_phase[k] = (unsigned char)phase;
                }
                t_over = min(t_over, end);
                wave_sync_lds();
            }
        };
        // the lanes with `ready` set release their call s: it waits at its prefill instance, or fails if it names none
        auto release = [&](bool ready, uint32_t s) {
            const uint32_t inst = ready ? (uint32_t)ids[s] & 0xFFu : 0u, r = ready ? (uint32_t)rank_of[s] : 0u;
            if (ready && inst < P) atomicOr(&queue[inst * kWords + (r >> 5)], 1u << (r & 31u));
            for (unsigned long long m = __ballot(ready); m != 0ull; m &= m - 1ull) {
                const uint32_t b = (uint32_t)__ffsll((long long)m) - 1u, i = wave_lane(inst, b);
                if (i < P) {
                    try_pre |= 1ull << i;
                } else {                                         // completes at this instant: looked at once more below
                    occupy(t, wave_lane(s, b), kUnplaced);
                    again = true;
                }
            }
        };
        auto complete = [&](uint32_t k, bool failed) {           // call k is over; those waiting for it have one predecessor less
            const uint32_t w = wf[k];
            if (lane == 0u) {
                comp[w] = t;
                if (failed) wf_failed[w] = 1;
            }
            last_done = t;
            const uint32_t first = wave_uniform(succ_first[k]), end = wave_uniform(succ_first[k + 1u]);
            for (uint32_t i0 = first; i0 < end; i0 += kWave) {       // usually none or one
                const uint32_t i = i0 + lane;
                uint32_t s = 0u;
                bool ready = false;
                if (i < end) {
                    s = p.o_succ != 0u ? succ_lds[i] : p.succ[i];
                    // (byte counters, through the word that holds the byte: each is decremented exactly as often as it was set)
                    const uint32_t shift = (s & 3u) * 8u;
                    const uint32_t old = atomicSub(reinterpret_cast<uint32_t*>(left + (s & ~3u)), 1u << shift);
                    ready = ((old >> shift) & 0xFFu) == 1u;      // its workflow has arrived: a call of it has completed
                }
                release(ready, s);
            }
        };
        // the first waiting call of a queue, by rank; K if there is none
        auto first_waiting = [&](uint32_t inst) {
            const uint32_t word = lane < kWords ? queue[inst * kWords + lane] : 0u;
            const unsigned long long any = __ballot(word != 0u);
            if (any == 0ull) return K;
            const uint32_t i = (uint32_t)__ffsll((long long)any) - 1u;
            return i * 32u + (uint32_t)__ffs((int)wave_lane(word, i)) - 1u;
        };
        auto leave = [&](uint32_t inst, uint32_t r) {
            if (lane == 0u) atomicAnd(&queue[inst * kWords + (r >> 5)], ~(1u << (r & 31u)));
            wave_sync_lds();
        };

        for (;;) {
            // ---- 1. completions, arrivals and the releases that follow (again when a call failed at its release) ----
            do {
                again = false;
                auto over_now = [&](uint32_t k, uint32_t phase) {    // the stage of call k has ended
                    const uint32_t id = wave_uniform(ids[k]), i = id & 0xFFu, q = id >> 8;
                    const uint2 len = lens[k];
                    const uint32_t need = wave_uniform(len.x + len.y);
                    bool done = true, failed = false;
                    if (phase == kInDecode) {
                        room += lane == q ? need : 0u;
                        try_dec |= 1ull << q;
                    } else if (phase == kInPrefill) {
                        busy &= ~(1ull << i);
                        try_pre |= 1ull << i;
                        failed = done = q >= Q || need > wave_lane(cap, q & 63u);
                        if (!failed) {
                            const uint32_t r = wave_uniform(rank_of[k]);
                            if (lane == 0u) atomicOr(&queue[(P + q) * kWords + (r >> 5)], 1u << (r & 31u));
                            try_dec |= 1ull << q;
                        }
                    } else {
                        failed = true;
                    }
                    if (done) complete(k, failed);
                };
                unsigned long long due = __ballot(ends == t);
                const uint32_t was = who;                        // a slot may be taken again meanwhile
                ends = ends == t ? kNever : ends;
                while (due != 0ull) {
                    const uint32_t x = wave_lane(was, (uint32_t)__ffsll((long long)due) - 1u);
                    due &= due - 1ull;
                    over_now(x & 1023u, x >> 10);
                }
                if (t_over == t) {                               // one pass: what is due, and the first end among the others
                    uint32_t rest = kNever;
                    t_over = kNever;                             // (a call that fails at its release lowers it again, and sets `again`)
                    for (uint32_t k0 = 0; k0 < K; k0 += kWave) {
                        const uint32_t end = k0 + lane < K ? over[k0 + lane] : kNever;
                        rest = min(rest, end == t ? kNever : end);
                        for (unsigned long long here = __ballot(end == t); here != 0ull; here &= here - 1ull) {
                            const uint32_t k = k0 + (uint32_t)__ffsll((long long)here) - 1u, phase = wave_uniform(over_phase[k]);
                            if (lane == 0u) over[k] = kNever;
                            wave_sync_lds();
                            over_now(k, phase);
                        }
                    }
                    t_over = min(t_over, wave_all_min(rest));
                }
                while (next_arrival <= t) {                      // kNever once all have arrived
                    const uint32_t w = wave_uniform(order[n_arrived]);
                    const uint32_t first = wave_uniform(root_first[w]), end = wave_uniform(root_first[w + 1u]);
                    for (uint32_t i0 = first; i0 < end; i0 += kWave) {
                        const bool ready = i0 + lane < end;
                        release(ready, ready ? (uint32_t)root[i0 + lane] : 0u);
                    }
                    ++n_arrived;
                    next_arrival = n_arrived < W ? wave_uniform(arrival[wave_uniform(order[n_arrived])]) : kNever;
                }
                wave_sync_lds();
            } while (again);
            // ---- 2. decode admissions: the first waiting call of an instance, while it fits ----
            for (; try_dec != 0ull; try_dec &= try_dec - 1ull) {
                const uint32_t q = (uint32_t)__ffsll((long long)try_dec) - 1u;
                for (;;) {
                    const uint32_t r = first_waiting(P + q);
                    if (r >= K) break;
                    const uint32_t k = wave_uniform(call_of[r]);
                    const uint2 len = lens[k];
                    const uint32_t n_in = wave_uniform(len.x), n_out = wave_uniform(len.y), need = n_in + n_out;
                    if (need > wave_lane(room, q)) break;
                    room -= lane == q ? need : 0u;
                    occupy(t + n_out * (wave_lane(qc, q) + wave_lane(qd, q) * ((n_in + 1023u) >> 10)), k, kInDecode);
                    leave(P + q, r);
                }
            }
            // ---- 3. prefill starts on idle instances ----
            for (try_pre &= ~busy; try_pre != 0ull; try_pre &= try_pre - 1ull) {
                const uint32_t i = (uint32_t)__ffsll((long long)try_pre) - 1u;
                const uint32_t r = first_waiting(i);
                if (r >= K) continue;
                const uint32_t k = wave_uniform(call_of[r]);
                const uint32_t n_in = wave_uniform(lens[k].x);
                busy |= 1ull << i;
                occupy(t + wave_lane(pa, i) + wave_lane(pb, i) * n_in, k, kInPrefill);
                leave(i, r);
            }
            // ---- 4. the next instant ----
            t = min(min(wave_all_min(ends), t_over), next_arrival);
            if (t == kNever) break;
        }
        wave_sync_lds();

        // ---- workflows -> completion ratios -> metrics --------------------------------------------
        unsigned long long sum = 0ull;
        uint32_t n_late = 0u, n_failed = 0u;
        for (uint32_t w = lane; w < W; w += kWave) {
            const unsigned long long took = comp[w] - arrival[w];
            const bool failed = wf_failed[w] != 0;
            const unsigned long long r = failed ? p.penalty : took * 1000ull / p.slo[w];
            ratio[w] = r;
            sum += r;
            n_late += (failed || took > p.slo[w]) ? 1u : 0u;
            n_failed += failed ? 1u : 0u;
        }
        sum = wave_sum_u64(sum);
        n_late = wave_sum_u32(n_late);
        n_failed = wave_sum_u32(n_failed);
        wave_sync_lds();
        // nearest rank: the value whose rank among all ratios (ties by workflow index) is the wanted one
        const uint32_t rank95 = (uint32_t)((95ull * W + 99ull) / 100ull) - 1u, rank99 = (uint32_t)((99ull * W + 99ull) / 100ull) - 1u;
        unsigned long long p95 = 0ull, p99 = 0ull;
        for (uint32_t w = lane; w < W; w += kWave) {
            const unsigned long long r = ratio[w];
            uint32_t rank = 0u;
            for (uint32_t v = 0; v < W; ++v) {
                const unsigned long long o = ratio[v];
                rank += (o < r || (o == r && v < w)) ? 1u : 0u;
            }
            if (rank == rank95) p95 = r;
            if (rank == rank99) p99 = r;
        }
        p95 = wave_all_or64(p95);                                // exactly one lane holds each
        p99 = wave_all_or64(p99);
        if (lane == 0u) {
            ap_agentic_metrics m;
            m.sum_ratio_permille = sum;
            m.p95_permille = p95;
            m.p99_permille = p99;
            m.makespan_us = last_done;
            m.n_late = n_late;
            m.n_failed = n_failed;
            out[c] = m;
        }
        wave_sync_lds();
    }
}

}  // namespace

#endif  // AP_AGENTIC_HPP
