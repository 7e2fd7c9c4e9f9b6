// Algorithm 1 on block counts (Sec. 3.3: the runtime state of each decoder,
// Eq. (6), Algorithm 1, and the atomic reservation of B_need after each
// dispatch) on gfx950.
//
//   rsc_state           one workgroup per decoder: held and reserved blocks of
//                       its residents (and of requests whose prompt KV is
//                       still in transfer) summed in 64-bit integers;
//   static_independent  every arrival against the reported state: a workgroup
//                       sorts the decoders by (queue, index) in LDS, keeps
//                       the records of B_eff in that order, and each arrival
//                       takes the first record that holds its B_need by a
//                       binary search;
//   static_reserve      arrivals one after another, each reserving its B_need
//                       and joining its decoder's queue before the next: one
//                       wavefront holds the state of up to 1,024 decoders in
//                       registers (ceil(D/64) per lane, a template parameter)
//                       and computes the needs itself, 64 arrivals at a time.
//                       The chain is serial by definition, so this kernel runs
//                       at the latency of one wavefront: arrivals with a
//                       feasible decoder are matched up to 64 at once, the
//                       others take a wavefront maximum each.
#include <type_traits>

#include "maps_internal.hpp"

namespace maps {
namespace {

constexpr int kRscNT = 512;
constexpr int kRscPer = 4;           // residents per thread whose loads are in flight together
constexpr int kIndNT = 1024;         // one decoder of a tile per thread
constexpr int kResSlots = MAPS_MAX_RESERVE_DECODERS / kWave;
constexpr int64_t kBlockLimit = int64_t(1) << 52;

// ceil(tokens / S) for 0 <= tokens < 2^32 with inv = min(floor(2^32 / S), 2^32 - 1):
// the product's high word is the quotient or one less (tokens (2^32 / S - inv) < 2^32),
// so the remainder against it stays below 2 S.  Five instructions against about
// forty of a 64-bit division, which bounded the sums over the residents.
__device__ inline uint32_t ceil_blocks(uint32_t tokens, uint32_t S, uint32_t inv) {
    const uint32_t q = __umulhi(tokens, inv);
    const uint32_t r = tokens - q * S;
    return q + (r > 0) + (r > S);
}
inline uint32_t block_inverse(int32_t S) {
    const uint64_t q = (uint64_t(1) << 32) / uint32_t(S);
    return q < UINT32_MAX ? uint32_t(q) : UINT32_MAX;
}

// ---------------------------------------------------------------------------
// Runtime state
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kRscNT) void rsc_state(int32_t D, const int64_t* __restrict__ seg_off,
                                                    int64_t n_total, const int32_t* __restrict__ p,
                                                    const int32_t* __restrict__ g, const int32_t* __restrict__ U,
                                                    const uint8_t* __restrict__ in_flight,
                                                    const int32_t* __restrict__ cap, int32_t S, uint32_t inv,
                                                    int64_t* __restrict__ b_free, int64_t* __restrict__ b_res,
                                                    int64_t* __restrict__ b_eff, uint32_t* dev_err) {
    __shared__ int64_t tmp[2][kRscNT / kWave];
    const int d = blockIdx.x;
    int64_t lo = seg_off[d], hi = seg_off[d + 1];
    if (!(0 <= lo && lo <= hi && hi <= n_total)) {
        if (threadIdx.x == 0) {
            raise_error(dev_err, MAPS_ERR_SEG_OFFSETS);
            b_free[d] = b_res[d] = b_eff[d] = 0;
        }
        return;
    }
    int64_t held = 0, res = 0;
    bool bad = false;
    for (int64_t r0 = lo + threadIdx.x; r0 < hi; r0 += kRscNT * kRscPer) {
        int32_t pr[kRscPer], gr[kRscPer], ur[kRscPer];
        uint8_t fl[kRscPer];
#pragma unroll
        for (int k = 0; k < kRscPer; ++k) {
            const int64_t r = r0 + k * kRscNT;
            const bool in = r < hi;   // past the segment: nothing held, nothing reserved
            pr[k] = in ? p[r] : 0;
            gr[k] = in ? g[r] : 0;
            ur[k] = in ? U[r] : 0;
            fl[k] = in && in_flight ? in_flight[r] : 0;
        }
#pragma unroll
        for (int k = 0; k < kRscPer; ++k) {
            const uint32_t pk = uint32_t(pr[k]), uk = ur[k] < 0 ? 0u : uint32_t(ur[k]);
            const uint32_t budget = ceil_blocks(pk + uk, uint32_t(S), inv);
            // staged reservation: prompt KV still in transfer, nothing held,
            // the whole budget (the prompt's blocks without a bound) reserved
            const bool staged = fl[k] != 0;
            bad |= (pr[k] < 0) | (!staged & (gr[k] < 0));
            const uint32_t now = staged ? 0u : ceil_blocks(pk + uint32_t(gr[k]), uint32_t(S), inv);
            held += now;
            if ((staged || ur[k] >= 0) && budget > now) res += budget - now;
        }
    }
    if (bad) raise_error(dev_err, MAPS_ERR_NEG_LEN);
    held = block_reduce_add<kRscNT>(held, tmp[0]);
    res = block_reduce_add<kRscNT>(res, tmp[1]);
    if (threadIdx.x == 0) {
        const int32_t c = cap[d];
        if (c < 0) raise_error(dev_err, MAPS_ERR_NEG_LEN);
        const int64_t fr = int64_t(c) / S - held;
        b_free[d] = fr;
        b_res[d] = res;
        b_eff[d] = fr - res;
    }
}

struct StaticArgs {
    int32_t D;
    const int64_t* beff;
    const int32_t* qlen;
    int32_t S;
    uint32_t inv;      // block_inverse(S)
    const int32_t* ap;
    const int32_t* aU;
    int64_t A;
    int32_t policy;
    int64_t rr_offset;
    int32_t* choice;
    int64_t* need;
    uint8_t* flags;
    int64_t* beff_out;
    int32_t* q_out;
    uint32_t* dev_err;
};

// ---------------------------------------------------------------------------
// Every arrival against the reported state
// ---------------------------------------------------------------------------
// The choice depends on the arrival only through its B_need: with the decoders
// in (queue, index) order, the shortest feasible queue is the first whose
// B_eff holds B_need, and only a B_eff above all those before it (a record)
// can be that first one.  Each workgroup sorts the decoders, 1,024 at a time,
// and keeps the records, so an arrival costs a binary search over a handful
// of them instead of a comparison with every decoder: with rsc_state before it,
// 262,144 arrivals on 256 decoders take 19 us a pass instead of 82.
template <int kPer>
__global__ __launch_bounds__(kIndNT) void static_independent(StaticArgs a) {
    __shared__ uint64_t skey[kIndNT];   // sort exchange, then the records' (queue, decoder)
    __shared__ int64_t rec[kIndNT];     // the records' B_eff, increasing
    __shared__ int64_t tmp64[kIndNT / kWave];
    __shared__ int32_t tmp32[kIndNT / kWave];
    const int t = threadIdx.x;
    const int64_t first = int64_t(blockIdx.x) * (kIndNT * kPer) + t;
    int32_t pr[kPer], ur[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {   // in flight during the first sort
        const int64_t i = first + k * kIndNT;
        pr[k] = i < a.A ? a.ap[i] : 0;
        ur[k] = i < a.A ? a.aU[i] : -1;
    }
    uint64_t best[kPer];                // (queue, decoder) of the shortest feasible queue so far
#pragma unroll
    for (int k = 0; k < kPer; ++k) best[k] = ~0ull;
    int64_t most_b = INT64_MIN;         // the largest B_eff and its first decoder
    int32_t most = 0;
    for (int64_t t0 = 0; t0 < a.D; t0 += kIndNT) {
        const int n = a.D - t0 < kIndNT ? int(a.D - t0) : kIndNT;
        int64_t B = INT64_MIN;
        uint64_t key = ~0ull;
        if (t < n) {
            B = a.beff[t0 + t];
            key = (uint64_t(uint32_t(a.qlen[t0 + t]) ^ 0x80000000u) << 32) | uint32_t(t0 + t);
            if (blockIdx.x == 0) {      // the reported state stays: independent arrivals reserve nothing
                if (a.beff_out) a.beff_out[t0 + t] = B;
                if (a.q_out) a.q_out[t0 + t] = int32_t(uint32_t(key >> 32) ^ 0x80000000u);
            }
        }
        const int64_t tile_b = block_reduce_max<kIndNT>(B, tmp64);
        const int32_t tile_d = -block_reduce_max<kIndNT>(t < n && B == tile_b ? -t : -kIndNT, tmp32);
        if (tile_b > most_b) { most_b = tile_b; most = int32_t(t0) + tile_d; }
        if (a.policy != MAPS_POLICY_MQ) continue;
        int n2 = kWave;
        while (n2 < n) n2 <<= 1;
        key = block_sort(key, n2, skey);
        __syncthreads();
        rec[t] = B;
        __syncthreads();
        const int64_t b = t < n ? rec[uint32_t(key) - uint32_t(t0)] : INT64_MIN;
        int64_t all;
        const int64_t before = block_excl_scan<kIndNT, true>(b, INT64_MIN, tmp64, &all);
        const bool is_rec = t < n && (t == 0 || b > before);
        int32_t records;
        const int32_t at = block_excl_scan<kIndNT, false>(int32_t(is_rec), 0, tmp32, &records);
        if (is_rec) { rec[at] = b; skey[at] = key; }   // every thread read rec before the scans' barriers
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (ur[k] < 0) continue;
            const int64_t need = ceil_blocks(uint32_t(pr[k]) + uint32_t(ur[k]), uint32_t(a.S), a.inv);
            int lo = 0, hi = records;   // the first record that holds the need
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (rec[mid] < need) lo = mid + 1; else hi = mid;
            }
            const uint64_t c = lo < records ? skey[lo] : ~0ull;
            best[k] = c < best[k] ? c : best[k];
        }
        __syncthreads();   // rec and skey are reused by the next tile
    }
    bool bad = false;
    uint32_t rr = uint32_t((a.rr_offset + first) % a.D);
    const uint32_t rr_step = uint32_t(kIndNT % a.D);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int64_t i = first + k * kIndNT;
        if (i < a.A) {
            int64_t need = -1;
            int32_t d = int32_t(rr);
            uint8_t f = 2;
            if (ur[k] >= 0) {
                bad |= pr[k] < 0;
                need = ceil_blocks(uint32_t(pr[k]) + uint32_t(ur[k]), uint32_t(a.S), a.inv);
                const bool feasible = best[k] != ~0ull;   // (queue, decoder) is never all ones: decoder < 2^31
                d = feasible ? int32_t(uint32_t(best[k])) : most;
                f = feasible || need <= most_b ? 1 : 0;
            }
            a.choice[i] = d;
            a.need[i] = need;
            a.flags[i] = f;
        }
        rr += rr_step;
        rr = rr >= uint32_t(a.D) ? rr - uint32_t(a.D) : rr;
    }
    if (bad) raise_error(a.dev_err, MAPS_ERR_NEG_LEN);
}

// ---------------------------------------------------------------------------
// One arrival after another, with reservation
// ---------------------------------------------------------------------------
// 64-bit wavefront minimum and maximum as two 32-bit reductions, high word
// first (a 32-bit DPP step is one instruction, a 64-bit one is five)
__device__ inline uint32_t wave_max_u32(uint32_t v) {
    return wave_last(wave_incl_scan(v, 0u, [](uint32_t x, uint32_t y) { return x > y ? x : y; }));
}

__device__ inline uint64_t wave_max_u64(uint64_t v) {
    const uint32_t hi = wave_max_u32(uint32_t(v >> 32));
    const uint32_t lo = wave_max_u32(uint32_t(v >> 32) == hi ? uint32_t(v) : 0u);
    return (uint64_t(hi) << 32) | lo;
}

__device__ inline uint64_t wave_min_u64(uint64_t v) {
    return ~wave_max_u64(~v);
}

// A value that is the same in every lane, as a scalar.
__device__ inline int64_t uniform64(int64_t v) {
    return int64_t((uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int32_t(uint64_t(v) >> 32)))) << 32) |
                   uint32_t(__builtin_amdgcn_readfirstlane(int32_t(v))));
}

// Largest-B_eff key of one decoder: (B_eff + 2^52) above (1023 - decoder);
// 0 (below every key) for a slot past the last decoder.
__device__ inline uint64_t best_b_key(int64_t B, int32_t d, int32_t D) {
    return d < D ? (uint64_t(B + kBlockLimit) << 10) | uint64_t(1023 - d) : 0;
}

// kSlots decoders per lane: decoder lane + 64 s in slot s, its B_eff and queue
// length in registers.  The arrivals go 64 at a time (one per lane, read out
// with readlane).

// A run of up to 64 arrivals with 64-bit keys.  The largest B_eff key over
// all decoders is kept between arrivals (only the chosen decoder's changes):
// an arrival whose B_need exceeds it takes that decoder at once; only a
// feasible shortest-queue choice scans every decoder.
template <int kSlots>
__device__ __forceinline__ void reserve_run_wide(const StaticArgs& a, int cnt, int64_t my_need, int32_t my_rr,
                                                 int64_t (&B)[kSlots], int64_t (&Q)[kSlots], int64_t& top,
                                                 bool& range_bad, int32_t& out) {
    const int lane = threadIdx.x;
    const bool mq = a.policy == MAPS_POLICY_MQ;
    uint64_t K[kSlots];
    auto lane_best = [&]() {
        uint64_t m = K[0];
#pragma unroll
        for (int s = 1; s < kSlots; ++s) m = K[s] > m ? K[s] : m;
        return m;
    };
#pragma unroll
    for (int s = 0; s < kSlots; ++s) K[s] = best_b_key(B[s], lane + s * kWave, a.D);
    uint64_t kb = wave_max_u64(lane_best());
    for (int j = 0; j < cnt; ++j) {
        const int64_t need = (int64_t(uint32_t(__builtin_amdgcn_readlane(int32_t(uint64_t(my_need) >> 32), j)))
                              << 32) |
                             uint32_t(__builtin_amdgcn_readlane(int32_t(my_need), j));
        int32_t best, f;
        if (need < 0) {
            best = __builtin_amdgcn_readlane(my_rr, j);
            f = 2;
        } else {
            const int64_t bmax = int64_t(kb >> 10) - kBlockLimit;
            if (mq && need <= bmax) {
                // feasible decoders exist: (Q, decoder) among them, smallest first
                uint64_t kf = ~0ull;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const int32_t d = lane + s * kWave;
                    const uint64_t k1 = (uint64_t(Q[s]) << 20) | uint64_t(d);
                    if (d < a.D && need <= B[s] && k1 < kf) kf = k1;
                }
                best = int32_t(wave_min_u64(kf) & 0xFFFFF);
                f = 1;
            } else {
                best = 1023 - int32_t(kb & 1023);
                f = need <= bmax ? 1 : 0;
            }
        }
        // the owning lane reserves and enqueues; a reservation changes the largest B_eff
        const int owner = best % kWave, slot = best / kWave;
        if (lane == owner) {
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                if (s == slot) {   // uniform: a scalar branch
                    if (need >= 0) {
                        B[s] -= need;
                        K[s] = best_b_key(B[s], best, a.D);
                    }
                    Q[s] += 1;
                    range_bad |= B[s] <= -kBlockLimit || B[s] >= kBlockLimit;
                }
            }
        }
        if (need >= 0) kb = wave_max_u64(lane_best());
        out = lane == j ? best | (f << 30) : out;
    }
    top = int64_t(kb >> 10) - kBlockLimit;
}

// The same run in 32 bits: R = kSlots (B_eff - top) + kSlots - 1 - slot (top: the
// largest B_eff at the run's start; the difference saturated at kRelLow), and the
// queue keys (Q << 10) | decoder.  Taken when the needs sum to less than 2^25
// blocks and every queue is in [0, 2^21 - 64).  Under policy MQ every B_eff counts
// as at most kMostB here: one that starts the run at 2^25 or more holds every
// need of it, so what it has beyond never decides.  A saturated decoder then has
// B_eff < 0 under MQ and is never feasible; nor is it ever the largest, which
// stays above top - 2^25; so neither its R nor its B_eff is used.  A feasible
// difference stays above -2^26 after its reservation, as does the largest.
// The slot makes a lane's maximum its lowest decoder with the largest B_eff.
// An arrival without a feasible decoder takes about 160 ns with one slot a
// lane, 220 with 4 (256 decoders) and 325 with 16 (1,000); looking for the slot
// in every register and updating each under a mask took 195, 303 and 650.
//
// Runs of arrivals that all find a feasible decoder are matched level by level
// of the queue lengths instead of one after another.  Every arrival prefers
// the decoders in the same (Q, index) order and a dispatch only makes its
// decoder worse (less B_eff, a longer queue), so taking the arrivals in turn
// gives the same pairs as taking the decoders of the shortest queue length in
// index order, each with the first arrival still waiting that it holds, then
// those of the next length (the matched ones among them, with what they have
// left), and so on.  A decoder's turn then depends on the others only through
// the set of waiting arrivals, a 64-bit mask: one compare of its R against the
// 64 thresholds and a bit search, instead of a wavefront minimum and a masked
// update of every slot an arrival.  An arrival left without a decoder takes
// the largest B_eff at its turn: the matching is undone, repeated for the
// arrivals before it (which the later ones never influence) and goes on after
// it, over at most as many arrivals at first as that attempt matched.
// One wavefront issues an instruction about every 4 ns, and that bounds the
// chain: an arrival takes 110 ns this way, against 220 ns with a wavefront
// minimum each and 375 ns with branches on the chosen lane and slot as well
// (65,536 arrivals on 256 decoders, 99.8% with a feasible one).
static_assert(kResSlots <= 16, "a slot in the four bits that kRelLow leaves free");
constexpr int32_t kRelLow = -(1 << 26);
constexpr int64_t kMostB = (int64_t(1) << 26) - 1;
constexpr int64_t kRunSpan = int64_t(1) << 25;
constexpr int64_t kRunQueue = int64_t(1) << 21;

__device__ inline uint32_t wave_min_u32(uint32_t v) {
    return wave_last(wave_incl_scan(v, ~0u, [](uint32_t x, uint32_t y) { return x < y ? x : y; }));
}
__device__ inline int32_t wave_max_i32(int32_t v) {
    return wave_last(wave_incl_scan(v, INT32_MIN, [](int32_t x, int32_t y) { return x > y ? x : y; }));
}

// fn(slot as a constant) for a slot in [kLo, kHi) that is the same in every
// lane: a tree of scalar branches.
template <int kLo, int kHi, typename Fn>
__device__ __forceinline__ void at_slot(int slot, Fn fn) {
    if constexpr (kHi - kLo == 1) {
        fn(std::integral_constant<int, kLo>{});
        // keeps the branches apart: merged, they index the registers by a variable, through memory
        asm volatile("" ::"i"(kLo));
    } else {
        constexpr int kMid = (kLo + kHi) / 2;
        if (slot < kMid) at_slot<kLo, kMid>(slot, fn);
        else at_slot<kMid, kHi>(slot, fn);
    }
}

template <int kSlots>
__device__ __forceinline__ void reserve_run(const StaticArgs& a, int cnt, int32_t my_need, int32_t my_rr,
                                            int64_t (&B)[kSlots], int64_t (&Q)[kSlots], int64_t& top,
                                            int32_t& out) {
    constexpr int kBits = kSlots > 8 ? 4 : kSlots > 4 ? 3 : kSlots > 2 ? 2 : kSlots - 1;
    constexpr int32_t kLow = (1 << kBits) - 1;
    const int lane = threadIdx.x;
    const bool mq = a.policy == MAPS_POLICY_MQ;
    const int64_t most = mq ? kMostB : INT64_MAX;
    top = uniform64(top);
    const bool capped = top > most;
    const int64_t ref = capped ? most : top;
    int32_t R[kSlots], R0[kSlots];
    uint32_t K[kSlots];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const int32_t d = lane + s * kWave;
        int64_t r = B[s] - ref;
        if (capped) r = r < 0 ? r : 0;
        // past the last decoder: below every threshold and every maximum
        R0[s] = R[s] = d >= a.D ? INT32_MIN : (r > kRelLow ? int32_t(r) : kRelLow) * (1 << kBits) + (kLow - s);
        K[s] = (uint32_t(Q[s]) << 10) | uint32_t(d);
    }
    // a decoder holds the need when R >= 2^kBits (need - ref); under MC ref may lie far above, then the largest does
    const int64_t thr64 = int64_t(my_need) - ref;
    const int32_t my_thr = thr64 >= (INT32_MAX >> kBits) ? INT32_MAX
                                                         : (thr64 > kRelLow ? int32_t(thr64) : kRelLow) * (1 << kBits);
    const int32_t my_cost = my_need * (1 << kBits);
    // the first arrival at or after `cur` with any bit of `set`, else 64
    auto first_from = [&](uint64_t set, int cur) {
        set = set >> cur << cur;
        return set != 0 ? __ffsll((unsigned long long)set) - 1 : kWave;
    };
    // arrivals [lo, hi)
    auto range = [](int lo, int hi) { return (hi >= kWave ? ~0ull : (1ull << hi) - 1ull) & (~0ull << lo); };
    const uint64_t no_bound = __builtin_amdgcn_ballot_w64(my_need < 0);   // past the batch as well
    int span = kWave;   // arrivals a matching tries
    for (int cur = 0; cur < cnt;) {
        if ((no_bound >> cur) & 1) {   // round robin: the request only joins the queue
            const int32_t d = __builtin_amdgcn_readlane(my_rr, cur);
#pragma unroll
            for (int s = 0; s < kSlots; ++s) K[s] += lane + s * kWave == d ? 1024u : 0u;
            out = lane == cur ? int32_t(uint32_t(d) | 0x80000000u) : out;
            ++cur;
            continue;
        }
        int32_t m;
        for (;;) {
            int32_t mine = R[0];
#pragma unroll
            for (int s = 1; s < kSlots; ++s) mine = R[s] > mine ? R[s] : mine;
            m = wave_max_i32(mine);
            const int32_t thr = __builtin_amdgcn_readlane(my_thr, cur);
            if (mq && m >= thr) break;
            // the lowest decoder with the largest B_eff
            const int l = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(mine == m)) - 1;
            const int slot = kLow - (m & kLow);
            const int32_t cost = lane == l ? __builtin_amdgcn_readlane(my_cost, cur) : 0;
            const uint32_t joins = lane == l ? 1024u : 0u;
            at_slot<0, kSlots>(slot, [&](auto s) {
                R[s] -= cost;
                K[s] += joins;
            });
            out = lane == cur ? (slot * kWave + l) | (m >= thr ? 1 << 30 : 0) : out;
            ++cur;
            if (cur >= cnt || ((no_bound >> cur) & 1) != 0) break;
        }
        if (cur >= cnt || ((no_bound >> cur) & 1) != 0) continue;
        // up to the first arrival that no decoder holds now or that has no bound
        int end = first_from(no_bound | __builtin_amdgcn_ballot_w64(my_thr > m), cur);
        end = end < cur + span ? end : cur + span;
        span = span < kWave ? 2 * span : kWave;
        int32_t R1[kSlots];
        uint32_t K1[kSlots];
#pragma unroll
        for (int s = 0; s < kSlots; ++s) { R1[s] = R[s]; K1[s] = K[s]; }
        for (;;) {
            uint64_t wait = range(cur, end);
            uint32_t level = 0;   // every shorter queue is done
            while (wait != 0) {
                const bool mine = ((wait >> lane) & 1) != 0;
                const int32_t low = -wave_max_i32(mine ? -my_thr : -INT32_MAX);
                uint32_t k = ~0u;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const uint32_t k1 = R[s] >= low && K[s] >= level ? K[s] : ~0u;
                    k = k1 < k ? k1 : k;
                }
                k = wave_min_u32(k);
                if (k == ~0u) break;   // no decoder holds any waiting arrival
                const uint32_t top_k = k | 1023u;   // the last key of this queue length
                level = top_k + 1;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    uint64_t at = __builtin_amdgcn_ballot_w64(R[s] >= low && K[s] <= top_k && K[s] >= k);
                    if (at == 0 || wait == 0) continue;
                    // the loop's first instruction at the start of a 32-byte fetch: where
                    // it fell by chance an arrival took between 1 and 1.12 times as long
                    asm volatile(".p2align 5");
                    do {
                        const int l = __ffsll((unsigned long long)at) - 1;
                        at &= at - 1;
                        const int32_t r = __builtin_amdgcn_readlane(R[s], l);
                        const uint64_t c = __builtin_amdgcn_ballot_w64(my_thr <= r) & wait;
                        if (c == 0) continue;
                        const int j = __ffsll((unsigned long long)c) - 1;
                        wait &= ~(1ull << j);
                        const int32_t cost = __builtin_amdgcn_readlane(my_cost, j);
                        const bool own = lane == l;
                        R[s] -= own ? cost : 0;
                        K[s] += own ? 1024u : 0u;
                        out = lane == j ? (l + s * kWave) | (1 << 30) : out;
                    } while (at != 0 && wait != 0);
                }
            }
            if (wait == 0) break;
            // the first arrival of the run finds its decoder whatever follows, so this stays above cur
            end = __ffsll((unsigned long long)wait) - 1;
#pragma unroll
            for (int s = 0; s < kSlots; ++s) { R[s] = R1[s]; K[s] = K1[s]; }
            span = end - cur > 4 ? end - cur : 4;
            if (end <= cur) { end = cur + 1; break; }   // unreachable: an end of the loop in any case
        }
        cur = end;
    }
    int32_t m = INT32_MIN;
    uint64_t key = 0;
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        if (lane + s * kWave < a.D) {
            B[s] += (R[s] - R0[s]) >> kBits;
            Q[s] = int64_t(K[s] >> 10);
        }
        m = R[s] > m ? R[s] : m;
    }
    if (!capped) {
        top += wave_max_i32(m) >> kBits;
    } else {
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            const uint64_t k = best_b_key(B[s], lane + s * kWave, a.D);
            key = k > key ? k : key;
        }
        top = int64_t(wave_max_u64(key) >> 10) - kBlockLimit;
    }
}

template <int kSlots>
__global__ __launch_bounds__(kWave) void static_reserve(StaticArgs a) {
    const int lane = threadIdx.x;
    int64_t B[kSlots];
    int64_t Q[kSlots];
    uint64_t k0 = 0;
    bool range_bad = false, neg = false;
    // the first run's arrivals
    int32_t p = lane < a.A ? a.ap[lane] : 0, U = lane < a.A ? a.aU[lane] : -1;
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const int32_t d = lane + s * kWave;
        B[s] = d < a.D ? a.beff[d] : 0;
        Q[s] = d < a.D ? a.qlen[d] : 0;
        range_bad |= B[s] <= -kBlockLimit || B[s] >= kBlockLimit;   // outside the packed keys
        const uint64_t k = best_b_key(B[s], d, a.D);
        k0 = k > k0 ? k : k0;
    }
    int64_t top = int64_t(wave_max_u64(k0) >> 10) - kBlockLimit;   // the largest B_eff
    // the run's first round-robin decoder; runs advance by 64 arrivals
    int32_t rr = int32_t(a.rr_offset % a.D);
    const int32_t rr_step = kWave % a.D;
    for (int64_t c0 = 0; c0 < a.A; c0 += kWave) {
        const int64_t mine = c0 + lane;
        neg |= U >= 0 && p < 0;
        const int64_t my_need = U < 0 ? int64_t(-1)
                                      : int64_t(ceil_blocks(uint32_t(p) + uint32_t(U), uint32_t(a.S), a.inv));
        // the next run's arrivals are on their way during this one
        p = mine + kWave < a.A ? a.ap[mine + kWave] : 0;
        U = mine + kWave < a.A ? a.aU[mine + kWave] : -1;
        const int32_t my_rr = int32_t(uint32_t(rr + lane) % uint32_t(a.D));
        rr += rr_step;
        rr = rr >= a.D ? rr - a.D : rr;
        int32_t out = 0;
        const int cnt = a.A - c0 < kWave ? int(a.A - c0) : kWave;
        // the run's needs and the queues decide the width (the same in every lane)
        bool long_queue = false;   // or a negative one
#pragma unroll
        for (int s = 0; s < kSlots; ++s) long_queue |= uint64_t(Q[s]) >= uint64_t(kRunQueue - kWave);
        const bool queues = __builtin_amdgcn_ballot_w64(long_queue) == 0;
        const int64_t need_sum = wave_reduce_add(my_need > 0 ? my_need : int64_t(0));
        if (queues && need_sum < kRunSpan)
            reserve_run<kSlots>(a, cnt, int32_t(my_need), my_rr, B, Q, top, out);
        else
            reserve_run_wide<kSlots>(a, cnt, my_need, my_rr, B, Q, top, range_bad, out);
        if (mine < a.A) {
            a.choice[mine] = out & 0x3FFFFFFF;
            a.need[mine] = my_need;
            a.flags[mine] = uint8_t(uint32_t(out) >> 30);
        }
    }
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const int32_t d = lane + s * kWave;
        range_bad |= B[s] <= -kBlockLimit;   // B_eff only falls: the end shows whether any left the keys' range
        if (d < a.D) {
            if (a.beff_out) a.beff_out[d] = B[s];
            if (a.q_out) a.q_out[d] = int32_t(Q[s]);
        }
    }
    if (neg) raise_error(a.dev_err, MAPS_ERR_NEG_LEN);
    if (range_bad) raise_error(a.dev_err, MAPS_ERR_BLOCK_RANGE);
}

}  // namespace
}  // namespace maps

using namespace maps;

extern "C" maps_status maps_rsc_state(int32_t D, const int64_t* seg_off, int64_t n_total, const int32_t* prompt,
                                      const int32_t* generated, const int32_t* upper, const uint8_t* in_flight,
                                      const int32_t* capacity,
                                      int32_t block_size, int64_t* b_free, int64_t* b_res, int64_t* b_eff,
                                      uint32_t* dev_err, hipStream_t stream) {
    if (D < 1 || n_total < 0 || block_size < 1) return MAPS_E_SIZE;
    if (!seg_off || !capacity || !b_free || !b_res || !b_eff || !dev_err ||
        (n_total > 0 && (!prompt || !generated || !upper)))
        return MAPS_E_NULL;
    hipLaunchKernelGGL(rsc_state, dim3(unsigned(D)), dim3(kRscNT), 0, stream, D, seg_off, n_total, prompt,
                       generated, upper, in_flight, capacity, block_size, block_inverse(block_size), b_free, b_res,
                       b_eff, dev_err);
    MAPS_CHECK_LAUNCH();
    return MAPS_OK;
}

extern "C" maps_status maps_place_static(int32_t D, const int64_t* b_eff, const int32_t* queue_len,
                                         int32_t block_size, const int32_t* a_prompt, const int32_t* a_upper,
                                         int64_t A, int32_t policy, int64_t rr_offset, int32_t reserve,
                                         int32_t* choice, int64_t* b_need, uint8_t* flags, int64_t* b_eff_out,
                                         int32_t* queue_out, uint32_t* dev_err, hipStream_t stream) {
    if (D < 1 || A < 0 || block_size < 1 || rr_offset < 0 || (reserve && D > MAPS_MAX_RESERVE_DECODERS))
        return MAPS_E_SIZE;
    if (policy != MAPS_POLICY_MQ && policy != MAPS_POLICY_MC) return MAPS_E_POLICY;
    if (!b_eff || !queue_len || !dev_err || (A > 0 && (!a_prompt || !a_upper || !choice || !b_need || !flags)))
        return MAPS_E_NULL;
    StaticArgs a{D, b_eff, queue_len, block_size, block_inverse(block_size), a_prompt, a_upper, A, policy,
                 rr_offset, choice, b_need, flags, b_eff_out, queue_out, dev_err};
    if (reserve) {
        const int slots = (D + kWave - 1) / kWave;
        if (slots <= 1) hipLaunchKernelGGL(static_reserve<1>, dim3(1), dim3(kWave), 0, stream, a);
        else if (slots <= 2) hipLaunchKernelGGL(static_reserve<2>, dim3(1), dim3(kWave), 0, stream, a);
        else if (slots <= 4) hipLaunchKernelGGL(static_reserve<4>, dim3(1), dim3(kWave), 0, stream, a);
        else if (slots <= 8) hipLaunchKernelGGL(static_reserve<8>, dim3(1), dim3(kWave), 0, stream, a);
        else hipLaunchKernelGGL(static_reserve<kResSlots>, dim3(1), dim3(kWave), 0, stream, a);
        MAPS_CHECK_LAUNCH();
        return MAPS_OK;
    }
    if (A == 0 && !b_eff_out && !queue_out) return MAPS_OK;
    // One arrival per thread up to two workgroups per compute unit (each sorts
    // the decoders for itself), four beyond.
    const int64_t blocks = (A + kIndNT - 1) / kIndNT;
    if (blocks <= 2 * int64_t(device_compute_units()))
        hipLaunchKernelGGL(static_independent<1>, dim3(unsigned(blocks > 0 ? blocks : 1)), dim3(kIndNT), 0, stream, a);
    else
        hipLaunchKernelGGL(static_independent<4>, dim3(unsigned((blocks + 3) / 4)), dim3(kIndNT), 0, stream, a);
    MAPS_CHECK_LAUNCH();
    return MAPS_OK;
}
