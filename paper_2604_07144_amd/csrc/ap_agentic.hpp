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
//  * a completion, release or arrival notes which instances it concerns, and only those try to admit or start a call; lane i keeps the
//    first waiting call of instance i with what it takes, so that whether it goes needs no look into the tables (8 % less for
//    plans of 320 calls by themselves, three LDS round trips for each attempt before);
//  * workflows are taken in order of arrival, each with the list of its calls without predecessors.
// Tables that are the same for all plans (lengths, successors, arrivals) are copied to LDS once per workgroup; the
// wavefronts of a workgroup share nothing else and never meet at a barrier after that.
// It is bound by instruction issue (per call 214 vector instructions, 196 scalar and 19 LDS ones): 8192 plans of a 330-call slice take
// 1.51 ms, 2.58 when the calls' phases were scanned at every instant (a lane per 64 calls, masks per lane).
struct AgenticParams {
    const uint4* blob;            // the tables that go to LDS, laid out as below
    uint32_t blob_bytes;          // a multiple of 16
    // byte offsets into it
    uint32_t o_info;              // uint4 [K] {in_len, out_len, where its successors begin (the successor itself if it is the
                                  //   only one), workflow | number of successors << 16}
    uint32_t o_start;             // uint4 [W + 1] workflows by arrival: {arrival, first root, number of roots, workflow}; roots are the
                                  //   calls without predecessors; entry W arrives at kNever
    uint32_t o_arrival;           // uint32 [W] microseconds after the earliest arrival
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
    // k_agentic_rows: byte offsets into a plan's own LDS, likewise behind the blob (offset 0: uint32 [K, up to a multiple of 16] keys,
    // then ends of the calls in service without a slot, then uint64 ratios [W])
    uint32_t g_call;              // uint32 [K] rank << 22 | call << 12 | prefill instance << 6 | decode instance
    uint32_t g_call_of;           // uint16 [K] call of a rank
    uint32_t g_left;              // uint8 [K] predecessors still to complete
    uint32_t g_comp;              // uint32 [W] completion time per workflow
    uint32_t g_failed;            // uint32 [ceil(W / 32)] a bit per workflow
    uint32_t g_queue;             // uint32 [P + Q][ceil(K / 32)] waiting calls by rank
    uint32_t g_bytes;             // LDS per plan
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
    const uint4* info = reinterpret_cast<const uint4*>(lds + p.o_info);
    const uint4* start = reinterpret_cast<const uint4*>(lds + p.o_start);
    const uint32_t* arrival = reinterpret_cast<const uint32_t*>(lds + p.o_arrival);
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

        // lane i: the first waiting call of prefill instance i and of decode instance i (its rank; K: none), and what it takes
        uint32_t pre_head = K, pre_head_call = 0u, pre_head_takes = 0u;
        uint32_t dec_head = K, dec_head_call = 0u, dec_head_takes = 0u, dec_head_need = 0u;

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
            const uint32_t inst = ready ? (uint32_t)ids[s] & 0xFFu : 0u, r = ready ? (uint32_t)rank_of[s] : 0u, in_len = ready ? info[s].x : 0u;
            if (ready && inst < P) atomicOr(&queue[inst * kWords + (r >> 5)], 1u << (r & 31u));
            for (unsigned long long m = __ballot(ready); m != 0ull; m &= m - 1ull) {
                const uint32_t b = (uint32_t)__ffsll((long long)m) - 1u, i = wave_lane(inst, b);
                if (i < P) {
                    try_pre |= 1ull << i;
                    const uint32_t rank_b = wave_lane(r, b), call_b = wave_lane(s, b), in_b = wave_lane(in_len, b);
                    const bool earlier = lane == i && rank_b < pre_head;
                    pre_head = earlier ? rank_b : pre_head;
                    pre_head_call = earlier ? call_b : pre_head_call;
                    pre_head_takes = earlier ? pa + pb * in_b : pre_head_takes;
                } else {                                         // completes at this instant: looked at once more below
                    occupy(t, wave_lane(s, b), kUnplaced);
                    again = true;
                }
            }
        };
        auto complete = [&](uint32_t k, bool failed) {           // call k is over; those waiting for it have one predecessor less
            const uint4 call = info[k];
            if (lane == 0u) {
                comp[call.w & 0xFFFFu] = t;
                if (failed) wf_failed[call.w & 0xFFFFu] = 1;
            }
            last_done = t;
            const uint32_t first = wave_uniform(call.z), end = first + wave_uniform(call.w >> 16);
            for (uint32_t i0 = first; i0 < end; i0 += kWave) {       // usually none or one
                const uint32_t i = i0 + lane;
                uint32_t s = 0u;
                bool ready = false;
                if (i < end) {
                    s = end - first == 1u ? first : p.o_succ != 0u ? succ_lds[i] : p.succ[i];
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
        // the first waiting call of a decode or prefill instance has left: the next one
        auto next_decode = [&](uint32_t q) {
            leave(P + q, wave_lane(dec_head, q));
            const uint32_t r = first_waiting(P + q), k = r < K ? wave_uniform(call_of[r]) : 0u;
            const uint32_t n_in = wave_uniform(info[k].x), n_out = wave_uniform(info[k].y);
            const bool ours = lane == q;
            dec_head = ours ? r : dec_head;
            dec_head_call = ours ? k : dec_head_call;
            dec_head_need = ours ? n_in + n_out : dec_head_need;
            dec_head_takes = ours ? n_out * (qc + qd * ((n_in + 1023u) >> 10)) : dec_head_takes;
        };
        auto next_prefill = [&](uint32_t i) {
            leave(i, wave_lane(pre_head, i));
            const uint32_t r = first_waiting(i), k = r < K ? wave_uniform(call_of[r]) : 0u, n_in = wave_uniform(info[k].x);
            const bool ours = lane == i;
            pre_head = ours ? r : pre_head;
            pre_head_call = ours ? k : pre_head_call;
            pre_head_takes = ours ? pa + pb * n_in : pre_head_takes;
        };

        for (;;) {
            // ---- 1. completions, arrivals and the releases that follow (again when a call failed at its release) ----
            do {
                again = false;
                auto over_now = [&](uint32_t k, uint32_t phase) {    // the stage of call k has ended
                    const uint32_t id = wave_uniform(ids[k]), i = id & 0xFFu, q = id >> 8;
                    const uint32_t n_in = wave_uniform(info[k].x), n_out = wave_uniform(info[k].y), need = n_in + n_out;
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
                            const bool earlier = lane == q && r < dec_head;
                            dec_head = earlier ? r : dec_head;
                            dec_head_call = earlier ? k : dec_head_call;
                            dec_head_need = earlier ? need : dec_head_need;
                            dec_head_takes = earlier ? n_out * (qc + qd * ((n_in + 1023u) >> 10)) : dec_head_takes;
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
                    const uint4 now = start[n_arrived];
                    const uint32_t first = wave_uniform(now.y), end = first + wave_uniform(now.z);
                    for (uint32_t i0 = first; i0 < end; i0 += kWave) {
                        const bool ready = i0 + lane < end;
                        release(ready, ready ? (uint32_t)root[i0 + lane] : 0u);
                    }
                    ++n_arrived;
                    next_arrival = wave_uniform(start[n_arrived].x);
                }
                wave_sync_lds();
            } while (again);
            // ---- 2. decode admissions: the first waiting call of an instance, while it fits ----
            for (;;) {
                const unsigned long long fits = __ballot(dec_head < K && dec_head_need <= room) & try_dec;
                if (fits == 0ull) break;
                const uint32_t q = (uint32_t)__ffsll((long long)fits) - 1u;
                room -= lane == q ? dec_head_need : 0u;
                occupy(t + wave_lane(dec_head_takes, q), wave_lane(dec_head_call, q), kInDecode);
                next_decode(q);
            }
            try_dec = 0ull;
            // ---- 3. prefill starts on idle instances ----
            for (try_pre &= __ballot(pre_head < K) & ~busy; try_pre != 0ull; try_pre &= try_pre - 1ull) {
                const uint32_t i = (uint32_t)__ffsll((long long)try_pre) - 1u;
                busy |= 1ull << i;
                occupy(t + wave_lane(pre_head_takes, i), wave_lane(pre_head_call, i), kInPrefill);
                next_prefill(i);
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

// ---- four plans per wavefront -----------------------------------------------------------------
// The same event loop for up to 16 instances of either kind, a row of 16 lanes per plan.  With a wavefront per plan every step of
// the loop is scalar work (196 scalar and 214 vector instructions per call of a plan, both issued at most once per SIMD and
// four cycles); here a step is vector work that four plans share, each at its own instant:
//  * lane i of a row owns prefill instance i and decode instance i: what runs on the former, the free tokens of the latter, the
//    first waiting call of both queues with what it takes (so a decision needs registers only), and which words of the queue's mask
//    hold a bit.  The masks themselves are in LDS and are read when a queue's first call leaves;
//  * decoding calls sit in 64 slots, four per lane; one that finds none free has its end in a table by call;
//  * one ended call or one arrival per plan and pass: a minimum over the row (rotations on the vector ALU's cross-lane path) says
//    which, and tells every lane of the row.
// Rows are at different instants, and all go through what one of them needs; values that concern a plan are the same in
// its 16 lanes.  A pass is some 220 vector instructions, 60 scalar ones and six LDS round trips one after the other (per call of a plan 166
// vector instructions, 43 scalar and 11 LDS ones), so a wavefront by itself takes 1.00 ms for plans of 317 calls, two per SIMD 1.11, and
// there they are bound by instruction issue.  8192 plans of 330 calls 1.16 ms, 1.51 by k_agentic_eval, measured in turn.  Which kernel
// takes a call: agentic_by_rows.
constexpr uint32_t kRowLanes = 16;
constexpr uint32_t kRowSlots = 4;                 // decoding calls per lane

template <uint32_t kBy>
__device__ __forceinline__ uint32_t row_rotated(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + kBy, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t row_all_min(uint32_t v) {
    v = min(v, row_rotated<8>(v));
    v = min(v, row_rotated<4>(v));
    v = min(v, row_rotated<2>(v));
    return min(v, row_rotated<1>(v));
}
__device__ __forceinline__ uint32_t row_all_or(uint32_t v) {
    v |= row_rotated<8>(v);
    v |= row_rotated<4>(v);
    v |= row_rotated<2>(v);
    return v | row_rotated<1>(v);
}
__device__ __forceinline__ uint32_t row_all_sum(uint32_t v) {
    v += row_rotated<8>(v);
    v += row_rotated<4>(v);
    v += row_rotated<2>(v);
    return v + row_rotated<1>(v);
}
__device__ __forceinline__ unsigned long long row_all_sum64(unsigned long long v) {
    auto add = [&](uint32_t lo, uint32_t hi) { v += ((unsigned long long)hi << 32) | lo; };
    add(row_rotated<8>((uint32_t)v), row_rotated<8>((uint32_t)(v >> 32)));
    add(row_rotated<4>((uint32_t)v), row_rotated<4>((uint32_t)(v >> 32)));
    add(row_rotated<2>((uint32_t)v), row_rotated<2>((uint32_t)(v >> 32)));
    add(row_rotated<1>((uint32_t)v), row_rotated<1>((uint32_t)(v >> 32)));
    return v;
}
__device__ __forceinline__ bool any_lane(bool b) { return __ballot(b) != 0ull; }
// which lanes of this lane's row
__device__ __forceinline__ uint32_t row_lanes(bool b) {
    const unsigned long long all = __ballot(b);
    const uint32_t half = (threadIdx.x & 32u) != 0u ? (uint32_t)(all >> 32) : (uint32_t)all;
    return (half >> (threadIdx.x & 16u)) & 0xFFFFu;
}
// LDS accesses of a wavefront execute in order; this keeps the compiler from moving them across
__device__ __forceinline__ void row_order_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__global__ __launch_bounds__(kAgenticThreads) void k_agentic_rows(AgenticParams p, const uint16_t* __restrict__ pre_inst,
                                                                 const uint16_t* __restrict__ dec_inst, const uint32_t* __restrict__ key,
                                                                 ap_agentic_metrics* __restrict__ out, uint32_t C) {
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t K = p.K, W = p.W, P = p.P, Q = p.Q;
    for (uint32_t i = threadIdx.x; i < p.blob_bytes / 16u; i += blockDim.x) reinterpret_cast<uint4*>(lds)[i] = p.blob[i];
    __syncthreads();
    const uint32_t i0 = threadIdx.x & (kRowLanes - 1u);          // the lane's place in its row: the instances it owns
    const uint32_t n_plans = blockDim.x / kRowLanes, plan = threadIdx.x / kRowLanes;
    const uint4* info = reinterpret_cast<const uint4*>(lds + p.o_info);
    const uint4* start_of = reinterpret_cast<const uint4*>(lds + p.o_start);
    const uint32_t* arrival = reinterpret_cast<const uint32_t*>(lds + p.o_arrival);
    unsigned char* mine = lds + p.blob_bytes + plan * p.g_bytes;
    uint32_t* over = reinterpret_cast<uint32_t*>(mine);
    unsigned long long* ratio = reinterpret_cast<unsigned long long*>(mine);
    uint32_t* call_word = reinterpret_cast<uint32_t*>(mine + p.g_call);
    uint16_t* call_of = reinterpret_cast<uint16_t*>(mine + p.g_call_of);
    unsigned char* left = mine + p.g_left;
    uint32_t* comp = reinterpret_cast<uint32_t*>(mine + p.g_comp);
    uint32_t* failed_wf = reinterpret_cast<uint32_t*>(mine + p.g_failed);
    const uint32_t n_words = (K + 31u) / 32u;
    uint32_t* queues = reinterpret_cast<uint32_t*>(mine + p.g_queue);
    uint32_t* pre_queue = queues + min(i0, P - 1u) * n_words;    // the lane's own queues, where it has the instance
    uint32_t* dec_queue = queues + (P + min(i0, Q - 1u)) * n_words;
    const uint32_t pa = i0 < P ? p.pa[i0] : 0u, pb = i0 < P ? p.pb[i0] : 0u;
    const uint32_t qc = i0 < Q ? p.qc[i0] : 0u, qd = i0 < Q ? p.qd[i0] : 0u, cap = i0 < Q ? p.cap[i0] : 0u;
    constexpr uint32_t kNone = kNever, kIsPrefill = 1u << 10, kOver = kNever - 1u;   // kOver: the instant of a plan that is over

    for (uint32_t c0 = blockIdx.x * n_plans; c0 < C; c0 += gridDim.x * n_plans) {
        if (c0 + wave_index() * (kWave / kRowLanes) >= C) break;
        const uint32_t c = min(c0 + plan, C - 1u);               // rows beyond the last plan repeat it and write nothing
        const uint32_t n_seg = (K + kRowLanes - 1u) / kRowLanes;
        for (uint32_t k = i0; k < n_seg * kRowLanes; k += kRowLanes) {
            over[k] = k < K ? key[(size_t)c * K + k] : kNever;
            if (k < K) {
                const uint32_t pre = min((uint32_t)pre_inst[(size_t)c * K + k], P), dec = min((uint32_t)dec_inst[(size_t)c * K + k], Q);
                const bool fits = dec < Q && info[k].x + info[k].y <= p.cap[min(dec, Q - 1u)];
                call_word[k] = (k << 12) | (pre << 6) | (fits ? dec : Q);   // one that can never fit fails where one without an instance does
            }
        }
        for (uint32_t i = i0; i < (K + 3u) / 4u; i += kRowLanes)
            reinterpret_cast<uint32_t*>(left)[i] = reinterpret_cast<const uint32_t*>(lds + p.o_n_pred)[i];
        for (uint32_t w = i0; w < W; w += kRowLanes) comp[w] = arrival[w];   // a workflow without calls completes on arrival
        for (uint32_t w = i0; w < (W + 31u) / 32u; w += kRowLanes) failed_wf[w] = 0u;
        for (uint32_t i = i0; i < (P + Q) * n_words; i += kRowLanes) queues[i] = 0u;
        row_order_lds();
        // rank by (key, index): earlier calls count at equal keys, later ones do not; 16 calls against eight per lane at a time
        for (uint32_t b = 0; b < n_seg; b += 8u) {
            uint32_t my_key[8], rank[8];
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) {
                my_key[j] = over[min(b + j, n_seg - 1u) * kRowLanes + i0];
                rank[j] = 0u;
            }
            for (uint32_t seg = 0; seg < n_seg; ++seg) {
                uint32_t o[kRowLanes];
#pragma unroll
                for (uint32_t e = 0; e < kRowLanes / 4u; ++e) {
                    const uint4 v = reinterpret_cast<const uint4*>(over)[seg * (kRowLanes / 4u) + e];
                    o[4u * e] = v.x; o[4u * e + 1u] = v.y; o[4u * e + 2u] = v.z; o[4u * e + 3u] = v.w;
                }
#pragma unroll
                for (uint32_t j = 0; j < 8u; ++j) {
                    if (seg < b + j) {
#pragma unroll
                        for (uint32_t e = 0; e < kRowLanes; ++e) rank[j] += o[e] <= my_key[j] ? 1u : 0u;
                    } else if (seg > b + j) {
#pragma unroll
                        for (uint32_t e = 0; e < kRowLanes; ++e) rank[j] += o[e] < my_key[j] ? 1u : 0u;
                    } else {
#pragma unroll
                        for (uint32_t e = 0; e < kRowLanes; ++e) rank[j] += (o[e] < my_key[j] || (o[e] == my_key[j] && e < i0)) ? 1u : 0u;
                    }
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) {
                const uint32_t k = (b + j) * kRowLanes + i0;
                if (k < K) {
                    call_word[k] |= rank[j] << 22;
                    call_of[rank[j]] = (uint16_t)k;
                }
            }
        }
        row_order_lds();
        for (uint32_t k = i0; k < K; k += kRowLanes) over[k] = kNever;
        row_order_lds();

        // the lane's instances
        uint32_t pre_end = kNever, pre_call = kNone;             // what runs on the prefill instance (kNever: idle)
        uint32_t pre_head = kNone, pre_head_call = 0u, pre_head_takes = 0u, pre_any = 0u;   // first waiting call (rank); words of the mask with a bit
        uint32_t room = cap;                                     // free tokens of the decode instance
        uint32_t dec_head = kNone, dec_head_call = 0u, dec_head_takes = 0u, dec_head_need = 0u, dec_any = 0u;
        uint32_t end[kRowSlots], who[kRowSlots];                 // decoding calls, of any instance (kNever: free; who then names none to come)
#pragma unroll
        for (uint32_t j = 0; j < kRowSlots; ++j) end[j] = kNever, who[j] = kNone;
        // the plan's
        uint32_t t = 0u, t_over = kNever, last_done = 0u, n_arrived = 0u;
        uint4 next = start_of[0];                                // the workflow that arrives next

        auto decode_takes = [&](const uint4& call) { return __umul24(call.y, qc + __umul24(qd, (call.x + 1023u) >> 10)); };

        // A pass: at the plan's next instant (its present one while something is left to do there) one call ends or one workflow
        // arrives, and, once no more do at that instant, idle prefill instances start and one call is admitted.
        for (;;) {
            const bool can = (dec_any != 0u && dec_head_need <= room) || (pre_any != 0u && pre_end == kNever);
            uint32_t first = can ? t : pre_end;
#pragma unroll
            for (uint32_t j = 0; j < kRowSlots; ++j) first = min(first, end[j]);
            t = min(row_all_min(first), min(next.x, t_over));
            if (!any_lane(t != kNever)) break;
            t = min(t, kOver);
            // ---- which call, which workflow ----
            uint32_t x = pre_end == t ? pre_call | kIsPrefill : kNone;
#pragma unroll
            for (uint32_t j = 0; j < kRowSlots; ++j) x = min(x, end[j] == t ? who[j] : kNone);
            x = row_all_min(x);
            if (any_lane(x == kNone && t_over == t)) {           // in the table, once the slots hold none
                uint32_t found = kNone;
                for (uint32_t k = i0; k < K; k += kRowLanes)
                    if (over[k] == t) found = min(found, k);
                found = row_all_min(found);
                if (x == kNone && t_over == t) {
                    x = found;
                    if ((found & (kRowLanes - 1u)) == i0) over[found] = kNever;
                }
                row_order_lds();
                uint32_t rest = kNever;                          // (once for every call that ends there: rare)
                for (uint32_t k = i0; k < K; k += kRowLanes) rest = min(rest, over[k]);
                t_over = row_all_min(rest);
            }
            const bool ended = x != kNone, arrives = !ended && next.x == t;
            const uint32_t k = ended ? x & 1023u : 0u;
            const uint32_t word = call_word[k];
            const uint4 call = info[k];
            const uint4 arrival_now = next;
            if (arrives) next = start_of[++n_arrived];
            if ((pre_call | kIsPrefill) == x) pre_end = kNever;
#pragma unroll
            for (uint32_t j = 0; j < kRowSlots; ++j) end[j] = who[j] == x ? kNever : end[j];   // a call is in one slot, once
            // ---- what ends ----
            const uint32_t rank = word >> 22, pre = (word >> 6) & 63u, dec = word & 63u, need = call.x + call.y;
            const bool prefilled = ended && (x & kIsPrefill) != 0u, unplaced = pre >= P;
            const bool decodes = prefilled && dec < Q, done = ended && !decodes;
            if (done && !prefilled && !unplaced && i0 == dec) room += need;
            {                                                    // it waits for the tokens
                const bool ours = decodes && i0 == dec, earlier = ours && rank < dec_head;
                if (ours) atomicOr(&dec_queue[rank >> 5], 1u << (rank & 31u));
                const uint32_t takes = decode_takes(call);
                dec_any |= ours ? 1u << (rank >> 5) : 0u;
                dec_head = earlier ? rank : dec_head;
                dec_head_call = earlier ? k : dec_head_call;
                dec_head_need = earlier ? need : dec_head_need;
                dec_head_takes = earlier ? takes : dec_head_takes;
            }
            last_done = done ? t : last_done;
            if (done && i0 == 0u) {
                comp[call.w & 0xFFFFu] = t;
                if (prefilled || unplaced) atomicOr(&failed_wf[(call.w & 0xFFFFu) >> 5], 1u << (call.w & 31u));
            }
            // ---- what is released: successors whose last predecessor this was, or the roots of a workflow ----
            const uint32_t n = done ? call.w >> 16 : arrives ? arrival_now.z : 0u;
            if (any_lane(n != 0u)) {
                const bool one = done && n == 1u;                // the successor itself is in the call's entry
                const uint32_t list = done ? p.o_succ + 2u * call.z : p.o_root + 2u * arrival_now.y;
                uint32_t l0 = i0;
                do {
                    const bool here = l0 < n;
                    uint32_t s = one ? call.z : 0u;
                    if (here && !one) s = *reinterpret_cast<const uint16_t*>(lds + list + 2u * l0);
                    const uint32_t of = call_word[s], in_len = info[s].x, inst = (of >> 6) & 63u;
                    bool ready = here;
                    if (here && done) {
                        const uint32_t shift = (s & 3u) * 8u;
                        const uint32_t old = atomicSub(reinterpret_cast<uint32_t*>(left + (s & ~3u)), 1u << shift);
                        ready = ((old >> shift) & 0xFFu) == 1u;  // its workflow has arrived: a call of it has completed
                    }
                    if (ready && inst < P) atomicOr(queues + __umul24(inst, n_words) + (of >> 27), 1u << ((of >> 22) & 31u));
                    if (any_lane(ready && inst >= P)) {          // completes at this instant: by way of the table
                        if (ready && inst >= P) over[s] = t;
                        if (row_lanes(ready && inst >= P) != 0u) t_over = t;
                        row_order_lds();
                    }
                    uint32_t of_s = ready && inst < P ? of : kNone;
                    while (any_lane(of_s != kNone)) {            // tell the owners, one per plan at a time
                        const uint32_t m = row_all_min(of_s), m_in = row_all_min(of_s == m ? in_len : kNone);
                        const uint32_t m_rank = m >> 22;
                        const bool ours = m != kNone && i0 == ((m >> 6) & 63u), earlier = ours && m_rank < pre_head;
                        pre_any |= ours ? 1u << (m >> 27) : 0u;
                        pre_head = earlier ? m_rank : pre_head;
                        pre_head_call = earlier ? (m >> 12) & 1023u : pre_head_call;
                        pre_head_takes = earlier ? pa + __umul24(pb, m_in) : pre_head_takes;
                        of_s = of_s == m ? kNone : of_s;
                    }
                    l0 += kRowLanes;
                } while (any_lane(l0 < n));
            }
            row_order_lds();
            // ---- when no more ends or arrives at this instant: prefill starts, one decode admission per plan ----
            uint32_t soonest = pre_end;
#pragma unroll
            for (uint32_t j = 0; j < kRowSlots; ++j) soonest = min(soonest, end[j]);
            const bool more = row_lanes(soonest == t) != 0u || t_over == t || next.x == t;
            const bool fits = !more && dec_any != 0u && dec_head_need <= room, starts = !more && pre_any != 0u && pre_end == kNever;
            if (!any_lane(fits || starts)) continue;
            pre_end = starts ? t + pre_head_takes : pre_end;
            pre_call = starts ? pre_head_call : pre_call;
            const uint32_t admitted = row_all_min(fits ? dec_head_call : kNone);
            const bool leaves = fits && dec_head_call == admitted;
            {                                                    // the admitted call takes a slot of the first lane with a free one
                const uint32_t until = row_all_min(leaves ? t + dec_head_takes : kNever);
                uint32_t latest = end[0];
#pragma unroll
                for (uint32_t j = 1; j < kRowSlots; ++j) latest = max(latest, end[j]);
                const uint32_t with_room = row_lanes(latest == kNever);
                bool take = admitted != kNone && (uint32_t)__ffs((int)with_room) == i0 + 1u;
#pragma unroll
                for (uint32_t j = 0; j < kRowSlots; ++j) {
                    const bool here = take && end[j] == kNever;
                    end[j] = here ? until : end[j];
                    who[j] = here ? admitted : who[j];
                    take = take && !here;
                }
                if (any_lane(admitted != kNone && with_room == 0u)) {   // or goes to the table
                    if (admitted != kNone && with_room == 0u) {
                        if (i0 == 0u) over[admitted] = until;
                        t_over = min(t_over, until);
                    }
                    row_order_lds();
                }
            }
            room -= leaves ? dec_head_need : 0u;
            // The queues whose first call has left, both at once: the word that held it, and the next one with a bit.
            {
                const uint32_t pre_at = starts ? pre_head >> 5 : 0u, dec_at = leaves ? dec_head >> 5 : 0u;
                const uint32_t pre_rest = pre_any & ~(1u << pre_at), dec_rest = dec_any & ~(1u << dec_at);
                const uint32_t pre_then = pre_rest != 0u ? (uint32_t)__ffs((int)pre_rest) - 1u : 0u;
                const uint32_t dec_then = dec_rest != 0u ? (uint32_t)__ffs((int)dec_rest) - 1u : 0u;
                const uint32_t pre_word = pre_queue[pre_at] & ~(1u << (pre_head & 31u)), dec_word = dec_queue[dec_at] & ~(1u << (dec_head & 31u));
                const uint32_t pre_next = pre_queue[pre_then], dec_next = dec_queue[dec_then];
                if (starts) pre_queue[pre_at] = pre_word;
                if (leaves) dec_queue[dec_at] = dec_word;
                // (a row's first word with a bit is the head's: ranks ascend)
                const uint32_t pre_bits = pre_word != 0u ? pre_word : pre_next, dec_bits = dec_word != 0u ? dec_word : dec_next;
                const uint32_t pre_left = pre_word != 0u ? pre_any : pre_rest, dec_left = dec_word != 0u ? dec_any : dec_rest;
                uint32_t pre_to = (pre_word != 0u ? pre_at : pre_then) * 32u + (uint32_t)__ffs((int)pre_bits) - 1u;
                uint32_t dec_to = (dec_word != 0u ? dec_at : dec_then) * 32u + (uint32_t)__ffs((int)dec_bits) - 1u;
                const bool pre_more = starts && pre_left != 0u, dec_more = leaves && dec_left != 0u;
                const uint32_t pre_k = call_of[pre_more ? pre_to : 0u], dec_k = call_of[dec_more ? dec_to : 0u];
                const uint32_t pre_in = info[pre_k].x;
                const uint4 dec_info = info[dec_k];
                pre_any = starts ? pre_left : pre_any;
                pre_head = starts ? (pre_more ? pre_to : kNone) : pre_head;
                pre_head_call = pre_more ? pre_k : pre_head_call;
                pre_head_takes = pre_more ? pa + __umul24(pb, pre_in) : pre_head_takes;
                dec_any = leaves ? dec_left : dec_any;
                dec_head = leaves ? (dec_more ? dec_to : kNone) : dec_head;
                dec_head_call = dec_more ? dec_k : dec_head_call;
                dec_head_need = dec_more ? dec_info.x + dec_info.y : dec_head_need;
                dec_head_takes = dec_more ? decode_takes(dec_info) : dec_head_takes;
            }
            row_order_lds();
        }
        row_order_lds();

        // ---- workflows -> completion ratios -> metrics --------------------------------------------
        unsigned long long sum = 0ull;
        uint32_t n_late = 0u, n_failed = 0u;
        for (uint32_t w = i0; w < W; w += kRowLanes) {
            const unsigned long long took = comp[w] - arrival[w];
            const bool failed = ((failed_wf[w >> 5] >> (w & 31u)) & 1u) != 0u;
            const unsigned long long r = failed ? p.penalty : took * 1000ull / p.slo[w];
            ratio[w] = r;
            sum += r;
            n_late += (failed || took > p.slo[w]) ? 1u : 0u;
            n_failed += failed ? 1u : 0u;
        }
        sum = row_all_sum64(sum);
        n_late = row_all_sum(n_late);
        n_failed = row_all_sum(n_failed);
        row_order_lds();
        const uint32_t rank95 = (uint32_t)((95ull * W + 99ull) / 100ull) - 1u, rank99 = (uint32_t)((99ull * W + 99ull) / 100ull) - 1u;
        unsigned long long p95 = 0ull, p99 = 0ull;
        for (uint32_t w = i0; w < W; w += kRowLanes) {
            const unsigned long long r = ratio[w];
            uint32_t rank = 0u;
            for (uint32_t v = 0; v < W; ++v) {
                const unsigned long long o = ratio[v];
                rank += (o < r || (o == r && v < w)) ? 1u : 0u;
            }
            if (rank == rank95) p95 = r;
            if (rank == rank99) p99 = r;
        }
        ap_agentic_metrics m;                                    // exactly one lane of the row holds each percentile
        m.p95_permille = ((unsigned long long)row_all_or((uint32_t)(p95 >> 32)) << 32) | row_all_or((uint32_t)p95);
        m.p99_permille = ((unsigned long long)row_all_or((uint32_t)(p99 >> 32)) << 32) | row_all_or((uint32_t)p99);
        m.sum_ratio_permille = sum;
        m.makespan_us = last_done;
        m.n_late = n_late;
        m.n_failed = n_failed;
        if (i0 == 0u && c0 + plan < C) out[c] = m;
        row_order_lds();
    }
}

}  // namespace

#endif  // AP_AGENTIC_HPP
