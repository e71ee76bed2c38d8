// Scoring in one pass over the row, for replicas that are always there: nobody waits, proved by counting.
#ifndef AP_STREAM_HPP
#define AP_STREAM_HPP

#include "ap_common.hpp"
#include "ap_counts.hpp"
#include "ap_screen.hpp"

namespace {

// ----------------------------------------------------------------------------------
// streamed evaluation
// ----------------------------------------------------------------------------------
// For replicas that are available throughout but differ (or a table too small for the slot rings).  Every request is scored
// where its id is read, as one that starts on arrival: ttft = prefill, e2e = prefill + decode on its replica's kind.  That
// is its record in the B-slot queue too if nobody waits.  Where no more than B requests of the whole trace are ever in service
// at once, on the slowest kind, nobody can, whatever the row, and nothing is left to prove (kCounted false).  Elsewhere it is
// proved for each row as in the counting screen (ap_counts.hpp): no replica gets more than B requests in the buckets lo(b) .. b,
// for any bucket b, where lo(b) is the first bucket with a request that could still be in service when b begins, on the slowest
// kind.  Here a candidate belongs to one workgroup and the counts of all buckets stay in LDS (a byte each, a bucket has at most
// 128 requests), so the windows are looked at once, at the end, and buckets can be as small as two requests.  A candidate that
// fails the proof gets the pending mark; the listed evaluation scores it next.
//
// A p99 value is the need_top-th largest of R values, so only large ones have to be told apart.  The host picks a bin per metric
// (and its lower edge, least[0]) that twice the needed number of requests reaches when the row is spread over the kinds as the
// replicas are; values from that bin on are counted, one in fifty, instead of every request in three histograms (three LDS
// atomics per request, time per token on a handful of addresses).  A row that prefers the fast kinds has fewer than need_top
// values there.  Its values are counted from the bin that enough requests reach on whichever kind (least[1]), where the p99
// value always is.  On long rows a sample of the row, a request per thread, tells; where there is no sample, or it was wrong, the
// row is read a second time.  (4096 rows of 16384 requests on the fast third of 48 replicas took 132 us with the sample, 231 without,
// 1009 when such rows went to the listed evaluation; before the change of the next paragraph.)
//
// Bound by instruction issue, 38 vector and 32 scalar instructions per 64 requests without counts, so the common case is kept
// short: in 128 requests that all exist and name a replica, which one packed compare per lane tells, nothing is tested
// request by request, the two requests of a lane are added up together, and large values are set aside and counted 64 at a time.
// Every request by the general form, its large values counted on the spot: 67 and 55 instructions, 136 us for 4096 rows of 16384
// requests on 48 replicas of three kinds; 91 now.  (Two wavefronts per row instead of four, fewer instructions still, take 10 % longer.)
struct StreamParams {
    const uint2* req8;            // [R + 1] {arrival, prompt | out << 16}
    const uint32_t* lo;           // [n_buckets] for rows that begin up to one position into their first 4-byte unit
    const uint32_t* kind;         // [M + 1] index into coef; tabulated cost model: first table entry of the replica's type
    const uint4* coef;            // [n_kinds] a, b, c, d
    const uint2* tab_pair;        // tabulated cost model: [T][R] {prefill time, time per token}
    uint32_t n_kinds;
    uint32_t R, M, B;
    uint32_t w_log2, n_buckets;
    uint32_t words;               // 4-byte words of counts per bucket: a byte per replica and one for unknown ids
    uint32_t slo_ttft, slo_tpot, all_within;
    // Per metric (ttft, tpot, e2e): the lowest bin that is ever counted and the bins that can occur from there on; for the first
    // and the second reading of a row, the lower edge of the first counted bin and the bins from that one on.
    uint32_t from[3], n_bins[3], least[2][3], n_counted[2][3];
    uint32_t need_top;            // R - k99 + 1
    const uint32_t* weight;       // [M + 1] or null: what a request on the replica adds to a sample of the row, kStreamWeight if a row
                                  //   of such requests has just need_top large values
    uint32_t penalty_bin;
    uint64_t penalty;
    uint32_t off_coef, off_lo, off_cnt, off_hist, off_acc, off_large;   // byte offsets into dynamic LDS
};
constexpr uint32_t kStreamMaxThreads = 1024;
constexpr uint32_t kStreamWeight = 64;
constexpr uint32_t kStreamLarge = 256;            // room for 63 requests with a large value that wait to be counted and the 128 of a step
constexpr uint32_t kStreamLargeBytes = 3u * 4u * kStreamLarge;   // per wavefront

// Two 16-bit ids, each cut down to `most`.
__device__ __forceinline__ uint32_t both_below(uint32_t ids, uint32_t most) {
    typedef uint16_t two_ids __attribute__((ext_vector_type(2)));
    two_ids v, m = {(uint16_t)most, (uint16_t)most};
    __builtin_memcpy(&v, &ids, 4);
    v = __builtin_elementwise_min(v, m);
    __builtin_memcpy(&ids, &v, 4);
    return ids;
}

template <bool kTabled, bool kCounted>
__global__ __launch_bounds__(kStreamMaxThreads, 6) void k_stream_candidates(StreamParams p, const uint16_t* __restrict__ assign,
                                                                            ap_metrics* __restrict__ out, uint32_t C,
                                                                            PendingWord flags) {
    extern __shared__ __align__(16) unsigned char lds[];
    pending_clear_next(flags);
    uint32_t* kind_of = reinterpret_cast<uint32_t*>(lds);
    uint4* coef_of = reinterpret_cast<uint4*>(lds + p.off_coef);
    uint16_t* lo_of = reinterpret_cast<uint16_t*>(lds + p.off_lo);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + p.off_cnt);            // [n_buckets][words], kCounted only
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds + p.off_hist);          // the three counted parts, one after the other
    unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(lds + p.off_acc);   // e2e, ttft, tpot
    uint32_t* acc32 = reinterpret_cast<uint32_t*>(lds + p.off_acc + 24);     // latest finish, within objectives, rejected, windows failed, p99 bins[3], too few counted, the sample's weight
    const uint32_t tid = threadIdx.x, n_threads = blockDim.x, lane = tid & 63u, wv = wave_index(), n_waves = n_threads >> 6;
    uint32_t* large = reinterpret_cast<uint32_t*>(lds + p.off_large + wv * kStreamLargeBytes);   // [3][kStreamLarge]
    const uint32_t R = p.R, M = p.M;
    const uint32_t hist_at[3] = {0u, p.n_bins[0], p.n_bins[0] + p.n_bins[1]};
    const uint32_t n_hist = hist_at[2] + p.n_bins[2], n_cnt = kCounted ? p.n_buckets * p.words : 0u;
    bool staged = false;
    uint32_t reading = 0;                                                    // 1: the row is read a second time
    for (uint32_t c = blockIdx.x; c < C;) {
        const uint16_t* row = assign + (size_t)c * R;
        const uint32_t a = (uint32_t)(reinterpret_cast<uintptr_t>(row) >> 1) & 1u, n = R + a;   // positions, as in the counting screen
        const uint32_t n_steps = (n + 127u) / 128u;
        // A lane takes two requests of every 128; the wavefronts take the steps in turn.  The next step's ids and records
        // are requested before the current one is worked on.
        typedef uint32_t two_records __attribute__((ext_vector_type(4), aligned(8)));
        struct Step {
            uint32_t ids;
            two_records rec;
        };
        auto whole = [&](uint32_t s) { return (s != 0u || a == 0u) && (s + 1u) * 128u <= n; };
        auto fetch = [&](uint32_t s) {
            Step st;
            const uint32_t pos = s * 128u + 2u * lane;
            if (whole(s)) {                                                  // uniform bases and offsets that stay: no address arithmetic per lane
                st.ids = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(
                    reinterpret_cast<const char*>(row + ((size_t)s * 128u - a)) + 4u * lane));
                st.rec = *reinterpret_cast<const two_records*>(reinterpret_cast<const char*>(p.req8 + ((size_t)s * 128u - a)) + 16u * lane);
            } else {                                                         // positions outside the row: an id no replica has, told apart below
                const bool in0 = pos >= a && pos < n, in1 = pos + 1u < n;
                const uint2 r0 = in0 ? p.req8[pos - a] : make_uint2(0u, 0u), r1 = in1 ? p.req8[pos + 1u - a] : make_uint2(0u, 0u);
                st.ids = (in0 ? (uint32_t)row[pos - a] : 0u) | ((in1 ? (uint32_t)row[pos + 1u - a] : 0u) << 16);
                st.rec = two_records{r0.x, r0.y, r1.x, r1.y};
            }
            return st;
        };
        Step next{};
        if (wv < n_steps) next = fetch(wv);
        uint32_t weight = 0;
        if (p.weight != nullptr && reading == 0u) weight = p.weight[min((uint32_t)row[(uint32_t)((uint64_t)tid * R / n_threads)], M)];
        if (!staged) {                                                       // behind the row's first loads: a short call waits once
            for (uint32_t i = tid; i <= M; i += n_threads) kind_of[i] = kTabled ? p.kind[i] : p.off_coef + p.kind[i] * 16u;
            for (uint32_t i = tid; i < p.n_kinds; i += n_threads) coef_of[i] = p.coef[i];
            if (kCounted)
                for (uint32_t i = tid; i < p.n_buckets; i += n_threads) lo_of[i] = (uint16_t)p.lo[i];
            staged = true;
        }
        for (uint32_t i = tid; i < n_cnt; i += n_threads) cnt[i] = 0u;
        for (uint32_t i = tid; i < n_hist; i += n_threads) hist[i] = 0u;
        if (tid < 16u) reinterpret_cast<uint32_t*>(acc64)[tid] = 0u;
        __syncthreads();
        if (p.weight != nullptr && reading == 0u) {
            weight = wave_sum_u32(weight);
            if (lane == 0u) atomicAdd(&acc32[8], weight);
            __syncthreads();
            reading = acc32[8] < n_threads * (kStreamWeight + kStreamWeight / 4u) ? 1u : 0u;   // the same word for every thread
        }
        const uint32_t least[3] = {p.least[reading][0], p.least[reading][1], p.least[reading][2]};
        unsigned long long s_e2e = 0, s_ttft = 0, s_tpot = 0;
        uint32_t t_e2e = 0, t_ttft = 0, t_tpot = 0, last_fin = 0, n_ok = 0, n_rej = 0;  // a wavefront's sums of up to four steps: 8 values below 2^28

        // Large values go through a buffer of the wavefront's own and are counted 64 at a time: with one request in twenty large some
        // lane of nearly every step has one, and counted on the spot each metric's bin costs every lane its instructions.
        uint32_t n_large = 0, n_counted_large = 0;
        auto count_large = [&](uint32_t n) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < n) {
                const uint32_t at = (n_counted_large + lane) & (kStreamLarge - 1u);
                const uint32_t value[3] = {large[at], large[kStreamLarge + at], large[2u * kStreamLarge + at]};
#pragma unroll
                for (uint32_t h = 0; h < 3u; ++h)
                    if (value[h] >= least[h]) atomicAdd(&hist[hist_at[h] + min(hist_bin_u32(value[h]) - p.from[h], p.n_bins[h] - 1u)], 1u);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            n_counted_large += n;
        };
        auto keep_large = [&](unsigned long long all, uint32_t prefill, uint32_t tpot, uint32_t e2e) {
            if (all == 0ull) return;
            if (__builtin_amdgcn_inverse_ballot_w64(all)) {
                const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(all >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all, n_large)) &
                                    (kStreamLarge - 1u);
                large[at] = prefill;
                large[kStreamLarge + at] = tpot;
                large[2u * kStreamLarge + at] = e2e;
            }
            n_large += (uint32_t)__popcll(all);
        };
        // kPlain: all 128 requests exist and name a replica.
        uint32_t prefill[2], tpot[2], e2e[2];
        unsigned long long is_large[2];                                      // which lanes' requests
        // (by LDS address, which begins at 0 with the kinds: through the array's name every access costs an addition of its base.  The
        // kernel must declare no __shared__ variable of its own: the host asks, tables_at_lds_zero)
        typedef __attribute__((address_space(3))) const uint32_t lds_word;
        typedef uint32_t four_words __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) const four_words lds_four;
        lds_word* const kind_at = reinterpret_cast<lds_word*>(0u);
        auto coef_from = [&](uint32_t at) {
            const four_words v = *reinterpret_cast<lds_four*>(at);
            return make_uint4(v.x, v.y, v.z, v.w);
        };
        auto score = [&](auto plain_tag, const Step& st, uint32_t s, uint32_t ids) {
            constexpr bool kPlain = decltype(plain_tag)::value;
            const uint32_t pos = s * 128u + 2u * lane;
            uint32_t* mine = kCounted ? cnt + (pos >> p.w_log2) * p.words : nullptr;   // w is even: both requests are in one bucket
            const uint32_t id[2] = {ids & 0xFFFFu, ids >> 16};
            const uint32_t kind[2] = {*(kind_at + id[0]), *(kind_at + id[1])};
            const bool in[2] = {kPlain || (pos >= a && pos < n), kPlain || pos + 1u < n};
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e) {
                const uint32_t lens = e ? st.rec.w : st.rec.y, len = lens >> 16;
                if (kTabled) {
                    const uint32_t r = kPlain ? pos + e - a : (in[e] ? pos + e - a : 0u);
                    const uint2 cost = p.tab_pair[kind[e] + r];
                    prefill[e] = cost.x;
                    tpot[e] = cost.y;
                } else {
                    const uint32_t prompt = lens & 0xFFFFu;
                    const uint4 co = coef_from(kind[e]);
                    prefill[e] = co.x + __umul24(co.y, prompt);              // the host keeps all factors below 2^24
                    tpot[e] = co.z + __umul24(co.w, (prompt + 1023u) >> 10);
                }
                e2e[e] = prefill[e] + __umul24(len, tpot[e]);
            }
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e) {
                const bool known = kPlain || (in[e] && id[e] < M);
                if (kCounted && (kPlain || in[e])) atomicAdd(&mine[id[e] >> 2], 1u << ((id[e] & 3u) * 8u));
                if (!kCounted && !kPlain) n_rej += in[e] && id[e] >= M ? 1u : 0u;
                if (!known) prefill[e] = tpot[e] = e2e[e] = 0u;              // rejected: adds nothing here
                t_ttft += prefill[e];
                t_e2e += e2e[e];
                t_tpot += tpot[e];
                if (p.all_within == 0u) n_ok += (known && prefill[e] <= p.slo_ttft && tpot[e] <= p.slo_tpot) ? 1u : 0u;
                is_large[e] = __ballot(prefill[e] >= least[0]) | __ballot(tpot[e] >= least[1]) | __ballot(e2e[e] >= least[2]);
                if (!kPlain) is_large[e] &= __ballot(known);
                if (!kPlain && known) last_fin = max(last_fin, (e ? st.rec.z : st.rec.x) + e2e[e]);
            }
            if (kPlain) last_fin = max(last_fin, max(st.rec.x + e2e[0], st.rec.z + e2e[1]));
        };
        if (wv < n_steps) {
            uint32_t turn = 0;
            for (uint32_t s = wv; s < n_steps; s += n_waves) {
                const Step now = next;
                if (s + n_waves < n_steps) next = fetch(s + n_waves);
                if (whole(s) && __ballot(both_below(now.ids, M - 1u) != now.ids) == 0ull) score(std::true_type{}, now, s, now.ids);
                else score(std::false_type{}, now, s, both_below(now.ids, M));
#pragma unroll
                for (uint32_t e = 0; e < 2u; ++e) keep_large(is_large[e], prefill[e], tpot[e], e2e[e]);
                while (n_large - n_counted_large >= kWave) count_large(kWave);   // leaves 63 at most
                if ((++turn & 3u) == 0u) {
                    s_e2e += t_e2e;
                    s_ttft += t_ttft;
                    s_tpot += t_tpot;
                    t_e2e = t_ttft = t_tpot = 0u;
                }
            }
            if (n_large != n_counted_large) count_large(n_large - n_counted_large);
            s_e2e = wave_sum_u64(s_e2e + t_e2e);
            s_ttft = wave_sum_u64(s_ttft + t_ttft);
            s_tpot = wave_sum_u64(s_tpot + t_tpot);
            last_fin = wave_all_max(last_fin);
            if (p.all_within == 0u) n_ok = wave_sum_u32(n_ok);
            if (!kCounted) n_rej = wave_sum_u32(n_rej);
            if (lane == 0u) {
                atomicAdd(&acc64[0], s_e2e);
                atomicAdd(&acc64[1], s_ttft);
                atomicAdd(&acc64[2], s_tpot);
                atomicMax(&acc32[0], last_fin);
                atomicAdd(&acc32[1], n_ok);
                if (!kCounted) atomicAdd(&acc32[2], n_rej);
            }
        }
        __syncthreads();

        // The windows: a thread takes one word of the buckets (four replicas) and a share of the buckets, and keeps the
        // window's sum as it moves.  No byte can run over: it is looked at whenever something was added, and a bucket adds
        // at most 128 to a sum of at most 127 that has passed.
        if (kCounted) {
            bool bad = false;
            const uint32_t shares = max(1u, n_threads / p.words), per = (p.n_buckets + shares - 1u) / shares;
            for (uint32_t job = tid; job < shares * p.words; job += n_threads) {
                const uint32_t q = job % p.words, b0 = job / p.words * per, b1 = min(b0 + per, p.n_buckets);
                if (b0 >= b1) continue;
                uint32_t room = (127u - p.B) * 0x01010101u, top = 0x80808080u, unknown_shift = 32u;
                if (4u * q + 4u > M) {                                       // the last word: byte M counts unknown ids, without a limit
                    unknown_shift = 8u * (M - 4u * q);
                    const uint32_t known = (1u << unknown_shift) - 1u;
                    room &= known;
                    top &= known;
                }
                uint32_t l = lo_of[b0], sum = 0, n_unknown = 0;
                for (uint32_t b = l; b < b0; ++b) {
                    sum += cnt[b * p.words + q];
                    bad = bad || ((sum | (sum + room)) & top) != 0u;
                }
                for (uint32_t b = b0; b < b1; ++b) {
                    for (const uint32_t lo = lo_of[b]; l < lo; ++l) sum -= cnt[l * p.words + q];
                    const uint32_t here = cnt[b * p.words + q];
                    sum += here;
                    bad = bad || ((sum | (sum + room)) & top) != 0u;
                    if (unknown_shift < 32u) n_unknown += (here >> unknown_shift) & 0xFFu;
                }
                if (n_unknown != 0u) atomicAdd(&acc32[2], n_unknown);
            }
            if (bad) acc32[3] = 1u;
            __syncthreads();
        }

        // p99: from the top down, the rejected requests at the penalty's bin
        const uint32_t rejected = acc32[2];
        for (uint32_t h = wv; h < 3u; h += n_waves) {
            const uint32_t* counts = hist + hist_at[h];
            uint32_t above = p.penalty_bin >= p.from[h] + p.n_bins[h] ? rejected : 0u, found = kNoKey;
            if (above >= p.need_top) found = p.penalty_bin;
            const uint32_t n_counted = p.n_counted[reading][h];
            for (uint32_t k = 0; k < n_counted && found == kNoKey; k += kWave) {
                const uint32_t down = k + lane, i = p.n_bins[h] - 1u - down;
                uint32_t v = down < n_counted ? counts[i] : 0u;
                if (down < n_counted && p.from[h] + i == p.penalty_bin) v += rejected;
                const uint32_t upto = above + wave_inclusive_scan(v, lane);
                const unsigned long long reached = __ballot(down < n_counted && upto >= p.need_top);
                if (reached != 0ull) found = p.from[h] + p.n_bins[h] - 1u - (k + (uint32_t)__ffsll((long long)reached) - 1u);
                above = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
            }
            if (lane == 0u) {
                if (found == kNoKey) acc32[7] = 1u;                          // the row has fewer large values than the host expected
                else acc32[4u + h] = found;
            }
        }
        __syncthreads();
        const bool again = reading == 0u && acc32[3] == 0u && acc32[7] != 0u;
        if (tid == 0u && !again) {
            ap_metrics mt;
            if (acc32[3] != 0u || acc32[7] != 0u) {
                __builtin_memset(&mt, 0xFF, sizeof(mt));
                pending_raise(flags);
            } else {
                mt.sum_e2e_us = acc64[0] + (unsigned long long)rejected * p.penalty;
                mt.sum_ttft_us = acc64[1] + (unsigned long long)rejected * p.penalty;
                mt.sum_tpot_us = acc64[2] + (unsigned long long)rejected * p.penalty;
                mt.makespan_us = acc32[0];
                mt.p99_ttft_us = hist_lower_edge(acc32[4]);
                mt.p99_tpot_us = hist_lower_edge(acc32[5]);
                mt.p99_e2e_us = hist_lower_edge(acc32[6]);
                mt.slo_ok = p.all_within != 0u ? R - rejected : acc32[1];
                mt.n_rejected = rejected;
            }
            out[c] = mt;
        }
        __syncthreads();                                                     // the totals were read
        reading = again ? 1u : 0u;
        if (!again) c += gridDim.x;
    }
}

}  // namespace

#endif  // AP_STREAM_HPP
