// KV pressure of decoders under round-robin or MAPS routing (App. A) on
// gfx950: a batch of independent simulations, one wavefront each.
//
// Each simulation follows the requests of one arrival sequence through N
// decoders of C KV tokens (App. A: demand M = L_p + L_out held from admission
// to completion, FIFO admission while K + M <= C, one token per millisecond
// per decoder shared by its admitted requests in one-token time slices) and
// records the high-pressure intervals (K / C >= theta) of every decoder.
//
// The state only changes at arrivals and completions, so the wavefront jumps
// from one such event to the next instead of stepping through milliseconds,
// and a decoder's ready queue is brought up to date lazily: after m one-token
// slices over n requests, the request at position k has received
// m / n + [k < m mod n] tokens and has moved to position (k - m) mod n, and the
// request at position k with l tokens left completes after (l - 1) n + k + 1
// slices, so the decoder's next completion is a wavefront minimum that stays
// valid until its queue changes.  The request that completes is the last of
// the queue then, and an admission appends at the end.
//
// A single wavefront issues an instruction about every 4 ns, so the time is
// the number of instructions an event takes.  simulate_fast keeps a decoder's
// requests one per lane in no particular order, with their position and tokens
// left: bringing a queue up to date, removing and appending are then a few
// lane-local instructions with nothing moved, the decoder in hand stays in two
// registers from event to event (the others wait in LDS), and times, tokens
// and divisions are 32-bit.  It needs valid inputs, times and C below 2^31,
// outputs below 2^24 (checked by one pass over the inputs) and at most 64
// admitted requests per decoder at a time; a simulation that does not fit
// starts in, or at the event where a queue outgrows the lanes goes over to,
// simulate_general: up to 1,024 requests per decoder in LDS in service order,
// in 64-bit, rotated by every update.  128 simulations of 10,000 requests on 4
// decoders: 45 ms all in simulate_general, 19 ms in simulate_fast.
//
// The next 64 arrivals (time, prompt, output, bound) sit in the lanes'
// registers, so an arrival waits on no global load.  The FIFO queues live in
// the workspace (one ring per decoder, 16 bytes an entry: id, prompt, output,
// bound).  simulate_general holds the head's entry in the decoder's lane;
// simulate_fast holds each queue's first entries, up to 64, in LDS, since a
// wait for one loaded entry is a wait for every store before it (one counter
// counts both).  Every loop is bounded: an arrival or a completion is consumed
// per event, and a simulation that could not progress reports an error instead
// of spinning.
#include "maps_internal.hpp"

namespace maps {
namespace {

constexpr int kSimNT = kWave;      // one wavefront per simulation
constexpr int kMaxDec = MAPS_MAX_SIM_DECODERS;
static_assert(kMaxDec <= kWave, "each decoder's state lives in one lane");
constexpr int kReady = MAPS_MAX_SIM_READY;
constexpr int kPerLane = kReady / kWave;
constexpr int64_t kNever = INT64_MAX;

struct SimArgs {
    int32_t N;
    int64_t C;
    int32_t theta_ppm;
    int64_t n;
    int32_t S;
    const int64_t* arrival;   // [S][n]
    const int32_t* prompt;    // [n]
    const int32_t* output;    // [n]
    const int32_t* bound;     // [n]
    const int32_t* policy;    // [S]
    int64_t* finish;          // [S][n]
    int32_t* routed;          // [S][n] (nullable)
    int64_t* stats;           // [S][5][N]: hp_time, hp_max, hp_count, max_queue, queue_area
    int64_t* span;            // [S][2]
    int4* fifo;               // workspace [S][N][n]: {id, prompt, output, bound}
    uint32_t* dev_err;
};

// Decoder d's state lives in lane d's registers (N <= 8 < 64): every lane
// reads it with readlane at the uniform index d, lane d alone writes it.
struct DecRegs {
    int64_t K, R;             // tokens held; needs reserved by queued requests (policy 1)
    int64_t next_done;        // time of the next completion (kNever when the ready queue is empty)
    int64_t t_sync;           // the ready queue's tokens-left are as of this time
    int64_t run, hp_time, hp_max, hp_count, max_queue, queue_area;
    int32_t nready, q_head, q_count;
    int4 head;                // the FIFO head's {id, prompt, output, bound} while q_count > 0
};

__device__ inline int32_t rl32(int32_t v, int j) { return __builtin_amdgcn_readlane(v, j); }
__device__ inline int64_t rl64(int64_t v, int j) {
    return int64_t((uint64_t(uint32_t(__builtin_amdgcn_readlane(int32_t(uint64_t(v) >> 32), j))) << 32) |
                   uint32_t(__builtin_amdgcn_readlane(int32_t(v), j)));
}

// A simulation between two steps of an event, or before its first (t = the
// first arrival).  The next 64 arrivals are in lane registers (lane k: request
// wbase + k), refilled by one coalesced load when the arrivals pass them; read
// with readlane at a uniform index.
struct SimState {
    DecRegs me;               // this lane's decoder (lanes < N)
    int64_t wbase, w_arr;
    int32_t w_p, w_o, w_b;
    int64_t t, next, done, last;
    bool resumed;             // the completions at t are done; every decoder is synced to t
};

__device__ inline void refill(const SimArgs& a, const int64_t* arr, SimState& st, int64_t base) {
    st.wbase = base;
    const int64_t i = base + threadIdx.x;
    st.w_arr = i < a.n ? arr[i] : kNever;
    st.w_p = i < a.n ? a.prompt[i] : 0;
    st.w_o = i < a.n ? a.output[i] : 0;
    st.w_b = i < a.n ? a.bound[i] : -1;
}

// LDS: general queues [N][kReady] x {id, tokens left, demand}.  The fast path's
// [N][64] x FIFO entries, {tokens left, position} and {id, demand} lie in the
// ids of each decoder past the first 64, which is all that the handover writes:
// beside the queues they left room for two instead of three workgroups a CU
// with 4 decoders and three instead of four with 3 (2,048 simulations of 1,500
// requests on 3 decoders in the general form: 17.4 instead of 14.3 ms).
__device__ inline void simulate_general(const SimArgs& a, SimState& st, int32_t* lds) {
    const int s = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t N = a.N;
    const int64_t n = a.n, C = a.C;
    int32_t* rid = lds;                         // [N][kReady] request ids in service order
    int32_t* rleft = lds + N * kReady;          // [N][kReady] tokens left as of t_sync
    uint32_t* rdem = reinterpret_cast<uint32_t*>(lds + 2 * N * kReady);   // [N][kReady] demands L_p + L_out
    const int64_t* arr = a.arrival + int64_t(s) * n;
    int64_t* fin = a.finish + int64_t(s) * n;
    int32_t* rout = a.routed ? a.routed + int64_t(s) * n : nullptr;
    int4* fifo = a.fifo + int64_t(s) * N * n;
    const int32_t policy = a.policy[s];
    bool bad_input = false, ready_full = false;
    DecRegs& me = st.me;

    // arrival time of request `next` (kNever past the last), the window moved up to it when passed
    auto arrival_of_next = [&](int64_t nx) -> int64_t {
        if (nx >= n) return kNever;
        if (nx >= st.wbase + kWave) refill(a, arr, st, nx);
        return rl64(st.w_arr, int(nx - st.wbase));
    };

    // bring decoder d's ready queue to time t: m slices since t_sync
    auto sync = [&](int d, int64_t t) {
        const int32_t nr = rl32(me.nready, d);
        const int64_t m = t - rl64(me.t_sync, d);
        if (nr > 0 && m > 0) {
            const int64_t q = m / nr;
            const int32_t r = int32_t(m % nr);
            int32_t id[kPerLane], lf[kPerLane];
            uint32_t dm[kPerLane];
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {   // new position k takes old position (k + r) mod nr
                if (j * kWave >= nr) break;         // uniform: only the rows of 64 that hold entries
                const int32_t k = lane + j * kWave;
                if (k < nr) {
                    int32_t src = k + r;
                    src = src >= nr ? src - nr : src;
                    id[j] = rid[d * kReady + src];
                    lf[j] = int32_t(rleft[d * kReady + src] - q - (src < r ? 1 : 0));
                    dm[j] = rdem[d * kReady + src];
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                if (j * kWave >= nr) break;
                const int32_t k = lane + j * kWave;
                if (k < nr) {
                    rid[d * kReady + k] = id[j];
                    rleft[d * kReady + k] = lf[j];
                    rdem[d * kReady + k] = dm[j];
                }
            }
            __syncthreads();
        }
        if (lane == d) me.t_sync = t;
    };
    // decoder d's next completion after a change of its ready queue (synced to t)
    auto schedule = [&](int d, int64_t t) {
        const int32_t nr = rl32(me.nready, d);
        int64_t best = kNever;
        for (int j = 0; j < kPerLane; ++j) {
            if (j * kWave >= nr) break;
            const int32_t k = lane + j * kWave;
            if (k < nr) {
                const int64_t sk = int64_t(rleft[d * kReady + k] - 1) * nr + k + 1;
                best = sk < best ? sk : best;
            }
        }
        best = -wave_reduce_max(-best);   // the wavefront minimum (kNever = INT64_MAX negates safely)
        if (lane == d) me.next_done = nr > 0 ? t + best : kNever;
    };
    // append request i (output o, demand dem) to the ready queue (synced to t)
    auto admit = [&](int d, int64_t i, int32_t o, int64_t dem, int64_t t) {
        if (rl32(me.nready, d) >= kReady) { ready_full = true; return false; }
        sync(d, t);
        const int32_t k = rl32(me.nready, d);
        if (lane == 0) {
            rid[d * kReady + k] = int32_t(i);
            rleft[d * kReady + k] = o;
            rdem[d * kReady + k] = uint32_t(dem);
        }
        if (lane == d) {
            me.nready = k + 1;
            me.K += dem;
        }
        __syncthreads();
        return true;
    };

    int64_t t = st.t, next = st.next, done = st.done, last = st.last;
    uint32_t dirty = st.resumed ? (1u << N) - 1u : 0;   // decoders whose ready queue changed at t (bit d)
    bool completions = !st.resumed;
    const int64_t max_events = 2 * n + 8;
    // Where the loop falls in the 32-byte instruction fetches decides 3%: 2,048
    // simulations of 1,500 requests on 8 decoders take 51.0 ms with it at 16,
    // 52.8, 51.7 and 52.0 at 0, 8 and 24.  Executed once.
    asm volatile(".p2align 5\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0");
    for (int64_t ev = 0;; ++ev) {
        if (ev > max_events) { bad_input = true; break; }
        // 1. completions at t: the completing request is the last of the synced queue
        for (int d = 0; d < N; ++d) {
            if (!completions || rl64(me.next_done, d) != t) continue;
            sync(d, t);
            const int32_t k = rl32(me.nready, d) - 1;
            const int64_t i = rid[d * kReady + k];
            const int64_t dem = int64_t(rdem[d * kReady + k]);
            if (lane == d) {
                me.nready = k;
                me.K -= dem;
            }
            if (lane == 0) fin[i] = t;
            done += 1;
            last = t;
            dirty |= 1u << d;
        }
        completions = true;
        if (done >= n) break;
        // 2. FIFO admission
        for (int d = 0; d < N; ++d) {
            while (rl32(me.q_count, d) > 0) {
                const int4 h = make_int4(rl32(me.head.x, d), rl32(me.head.y, d), rl32(me.head.z, d),
                                         rl32(me.head.w, d));
                const int64_t dem = int64_t(h.y) + h.z;
                if (rl64(me.K, d) + dem > C) break;
                if (!admit(d, h.x, h.z, dem, t)) break;
                const int32_t qh = rl32(me.q_head, d), qc = rl32(me.q_count, d) - 1;
                const int32_t nh = qh + 1 == n ? 0 : qh + 1;
                if (lane == d) {
                    me.q_head = nh;
                    me.q_count = qc;
                    if (policy == 1 && h.w >= 0) me.R -= int64_t(h.y) + h.w;
                    // the next head's entry: one 16-byte load, only after an admission (lane d wrote it)
                    if (qc > 0) me.head = fifo[int64_t(d) * n + nh];
                }
                dirty |= 1u << d;
            }
        }
        // 3. arrivals at t, in index order
        while (next < n) {
            const int64_t ai = arrival_of_next(next);
            if (ai > t) break;
            const int j = int(next - st.wbase);
            const int32_t pi = rl32(st.w_p, j), oi = rl32(st.w_o, j), bi = rl32(st.w_b, j);
            const int64_t i = next++;
            const int64_t dem = int64_t(pi) + oi, nd = int64_t(pi) + bi;
            if (ai < t || pi < 0 || oi < 1 || dem > C) {
                bad_input = true;   // out of order or never admissible: dropped
                if (lane == 0) fin[i] = t;
                done += 1;
                continue;
            }
            int d;
            if (policy == 1 && bi >= 0) {   // Algorithm 1 at block size 1
                int feas = -1, most = 0;
                int32_t fq = 0;
                int64_t most_beff = 0;
                for (int k = 0; k < N; ++k) {
                    const int64_t beff = C - rl64(me.K, k) - rl64(me.R, k);
                    const int32_t qk = rl32(me.q_count, k);
                    if (nd <= beff && (feas < 0 || qk < fq)) {
                        feas = k;
                        fq = qk;
                    }
                    if (k == 0 || beff > most_beff) {
                        most = k;
                        most_beff = beff;
                    }
                }
                d = feas >= 0 ? feas : most;
            } else {
                d = int(i % N);
            }
            if (lane == 0 && rout) rout[i] = d;
            bool queued = true;
            if (rl32(me.q_count, d) == 0 && rl64(me.K, d) + dem <= C) {
                queued = !admit(d, i, oi, dem, t);
                if (!queued) dirty |= 1u << d;
            }
            if (queued) {
                const int32_t qh = rl32(me.q_head, d), qc = rl32(me.q_count, d);
                int64_t tail = int64_t(qh) + qc;
                tail = tail >= n ? tail - n : tail;
                const int4 e = make_int4(int32_t(i), pi, oi, bi);
                if (lane == d) {   // the lane that reads the ring writes it
                    fifo[int64_t(d) * n + tail] = e;
                    if (qc == 0) me.head = e;
                    me.q_count = qc + 1;
                    if (policy == 1 && bi >= 0) me.R += nd;
                }
            }
        }
        if (done >= n) break;   // only dropped requests were left
        for (int d = 0; d < N; ++d)
            if (dirty & (1u << d)) schedule(d, t);
        dirty = 0;
        // the next event, and the state recorded over [t, t_next)
        int64_t t_next = arrival_of_next(next);
        for (int d = 0; d < N; ++d) {
            const int64_t nd = rl64(me.next_done, d);
            t_next = nd < t_next ? nd : t_next;
        }
        if (t_next == kNever || t_next <= t) { bad_input = true; break; }
        const int64_t len = t_next - t;
        if (lane < N) {
            if (me.K * 1000000 >= int64_t(a.theta_ppm) * C) {
                if (me.run == 0) me.hp_count += 1;
                me.run += len;
                me.hp_time += len;
                me.hp_max = me.run > me.hp_max ? me.run : me.hp_max;
            } else {
                me.run = 0;
            }
            me.queue_area += int64_t(me.q_count) * len;
            me.max_queue = me.q_count > me.max_queue ? me.q_count : me.max_queue;
        }
        t = t_next;
    }
    st.last = last;
    if (lane == 0) {
        if (bad_input) raise_error(a.dev_err, MAPS_ERR_SIM_INPUT);
        if (ready_full) raise_error(a.dev_err, MAPS_ERR_SIM_READY);
    }
}

// Whether simulate_fast's 32-bit times and unchecked inputs hold: arrival times
// that do not decrease, requests that can be admitted, and a last completion
// (at most all the outputs after the last arrival) below 2^31 ms after the
// first arrival.
__device__ inline bool fits_fast(const SimArgs& a, const int64_t* arr) {
    constexpr int kPer = 8;
    if (a.C >= (int64_t(1) << 31) || a.n >= (int64_t(1) << 28)) return false;
    bool bad = false;
    int64_t work = 0;
    for (int64_t i0 = 0; i0 < a.n; i0 += kPer * kWave) {
        int64_t t0[kPer], t1[kPer];
        int32_t p[kPer], o[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int64_t i = i0 + k * kWave + threadIdx.x;
            const bool in = i < a.n;
            t0[k] = in ? arr[i > 0 ? i - 1 : 0] : 0;
            t1[k] = in ? arr[i] : 0;
            p[k] = in ? a.prompt[i] : 0;
            o[k] = in ? a.output[i] : 1;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            bad |= t1[k] < t0[k] || p[k] < 0 || o[k] < 1 || o[k] >= (1 << 24) || int64_t(p[k]) + o[k] > a.C;
            work += o[k];
        }
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0) return false;
    const int64_t first = arr[0], last = arr[a.n - 1];   // in order: last - first cannot wrap below 0
    const uint64_t span = uint64_t(last) - uint64_t(first);
    return span < (uint64_t(1) << 31) && int64_t(span) + wave_reduce_add(work) < (int64_t(1) << 31) - 1;
}

// A value that is the same in every lane, as a scalar.  The compiler takes the
// loop-carried ones for divergent and would run every branch on them by
// execution masks, about a fifth slower.
__device__ inline int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Minimum of a 32-bit value and maximum of a 64-bit value over lanes 0..7.
__device__ inline uint32_t min8(uint32_t v) {
    auto op = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
    v = op(v, dpp_move<kDppRowShr1, 0xf>(~0u, v));
    v = op(v, dpp_move<kDppRowShr2, 0xf>(~0u, v));
    v = op(v, dpp_move<kDppRowShr4, 0xf>(~0u, v));
    return __builtin_amdgcn_readlane(v, kMaxDec - 1);
}
__device__ inline int64_t max8(int64_t v) {
    auto op = [](int64_t x, int64_t y) { return x > y ? x : y; };
    v = op(v, dpp_move<kDppRowShr1, 0xf>(INT64_MIN, v));
    v = op(v, dpp_move<kDppRowShr2, 0xf>(INT64_MIN, v));
    v = op(v, dpp_move<kDppRowShr4, 0xf>(INT64_MIN, v));
    return rl64(v, kMaxDec - 1);
}

// Runs the simulation from its start with 32-bit times relative to the first
// arrival; returns true when it is done, false when a ready queue would
// outgrow the lanes: st then holds the state for simulate_general, between the
// completions at st.t and the admissions.
__device__ inline bool simulate_fast(const SimArgs& a, SimState& st, int32_t* lds) {
    const int s = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t N = a.N, n = int32_t(a.n), C = int32_t(a.C);
    int4* q_fifo = reinterpret_cast<int4*>(lds + kWave);                // entry i of a FIFO in slot i mod 64
    int2* q_state = reinterpret_cast<int2*>(lds + kWave + 4 * kWave);   // {tokens left, position}
    int2* q_req = q_state + kWave;                                      // {id, demand}
    static_assert(kReady >= kWave + (4 + 2 + 2) * kWave && kReady % 4 == 0, "the fast arrays past the first 64 ids");
    constexpr int kStep2 = kReady / 2, kStep4 = kReady / 4;             // from one decoder's to the next
    const int64_t* arr = a.arrival + int64_t(s) * n;
    int64_t* fin = a.finish + int64_t(s) * n;
    int32_t* rout = a.routed ? a.routed + int64_t(s) * n : nullptr;
    int4* rings = a.fifo + int64_t(s) * N * n;
    const int32_t policy = a.policy[s];
    const int64_t origin = st.t;
    constexpr int32_t kFree = INT32_MAX;   // position of a lane without a request
    // high pressure: K 10^6 >= theta C
    const int32_t k_high = int32_t((int64_t(a.theta_ppm) * C + 999999) / 1000000);

    // lane d < N: decoder d
    int32_t K = 0, nready = 0;
    // the FIFO: entries [q_head, q_head + q_count) in the order they came (at
    // most n in all: the ring does not wrap), those below q_end in LDS
    int32_t q_head = 0, q_count = 0, q_end = kWave;
    int64_t R = 0, area = 0;
    uint32_t due = ~0u, synced = 0;       // the next completion (~0: none); the ready queue's time
    int32_t run = 0, hp_time = 0, hp_max = 0, hp_count = 0, max_queue = 0;

    // the ready queue in hand
    int cur = -1;
    int32_t left = 0, pos = kFree, count = 0;
    for (int d = 0; d < N; ++d) q_state[d * kStep2 + lane] = make_int2(0, kFree);

    uint32_t t = 0;
    int32_t next = 0, done = 0, rr = 0;   // rr = next mod N
    int32_t wbase = 0;
    uint32_t w_arr = 0;
    auto fill = [&](int32_t base) {   // the arrivals' window
        refill(a, arr, st, base);
        wbase = base;
        w_arr = base + lane < n ? uint32_t(st.w_arr - origin) : ~0u;
        // waited for here: a wait at each use would be one for the stores in flight there
        asm volatile("" : "+v"(w_arr), "+v"(st.w_p), "+v"(st.w_o), "+v"(st.w_b));
    };
    fill(0);
    auto next_arrival = [&]() -> uint32_t {   // ~0 past the last
        next = uniform(next);
        wbase = uniform(wbase);
        if (next >= n) return ~0u;
        if (next >= wbase + kWave) fill(next);
        return __builtin_amdgcn_readlane(w_arr, next - wbase);
    };
    // take decoder d's ready queue in hand, brought up to time t
    auto enter = [&](int d) {
        cur = uniform(cur);
        count = uniform(count);
        if (cur != d) {
            if (cur >= 0) q_state[cur * kStep2 + lane] = make_int2(left, pos);
            const int2 x = q_state[d * kStep2 + lane];
            left = x.x;
            pos = x.y;
            cur = d;
            count = rl32(nready, d);
        }
        const uint32_t m = t - uint32_t(rl32(int32_t(synced), d));
        if (m != 0 && count > 0) {
            uint32_t q, r;
            if (m < (1u << 22)) {   // the float quotient is off by at most one
                q = uint32_t(float(m) * __builtin_amdgcn_rcpf(float(count)));
                r = m - q * uint32_t(count);
                if (int32_t(r) < 0) { r += uint32_t(count); q -= 1; }
                if (r >= uint32_t(count)) { r -= uint32_t(count); q += 1; }
            } else {
                q = m / uint32_t(count);
                r = m % uint32_t(count);
            }
            const bool again = pos < int32_t(r);
            left -= int32_t(q) + int32_t(again);
            const int32_t moved = pos - int32_t(r) + (again ? count : 0);
            pos = pos < count ? moved : kFree;
        }
        if (lane == d) synced = t;
    };
    // append a request to the queue in hand (decoder d's); false: no lane is free
    auto admit = [&](int d, int32_t i, int32_t o, int32_t dem) -> bool {
        enter(d);
        if (count >= kWave) return false;
        const uint64_t used = __builtin_amdgcn_ballot_w64(pos != kFree);
        const int slot = __ffsll((unsigned long long)~used) - 1;
        if (lane == slot) {
            left = o;
            pos = count;
            q_req[d * kStep2 + lane] = make_int2(i, dem);
        }
        count += 1;
        if (lane == d) {
            nready = count;
            K += dem;
        }
        return true;
    };

    int over = 0;   // a queue outgrew the lanes
    const int64_t max_events = 2 * int64_t(n) + 8;
    for (int64_t ev = 0; ev <= max_events; ++ev) {
        t = uint32_t(uniform(int32_t(t)));
        rr = uniform(rr);
        done = uniform(done);
        // 1. completions at t: the completing request is the last of its queue
        const uint64_t completed = __builtin_amdgcn_ballot_w64(due == t && lane < N);
        for (uint64_t c = completed; c != 0; c &= c - 1) {
            const int d = __ffsll((unsigned long long)c) - 1;
            enter(d);
            const uint64_t at = __builtin_amdgcn_ballot_w64(pos == count - 1);
            const int slot = at != 0 ? __ffsll((unsigned long long)at) - 1 : 0;
            const int2 req = q_req[d * kStep2 + slot];
            pos = lane == slot ? kFree : pos;
            count -= 1;
            if (lane == d) {
                nready = count;
                K -= req.y;
            }
            if (lane == 0) fin[req.x] = origin + t;
            done += 1;
        }
        uint64_t dirty = completed;
        if (completed != 0) st.last = origin + t;
        if (done >= n) break;
        // 2. FIFO admission (only a completion can make room for a head)
        for (uint64_t c = completed & __builtin_amdgcn_ballot_w64(q_count > 0); c != 0 && uniform(over) == 0; c &= c - 1) {
            const int d = __ffsll((unsigned long long)c) - 1;
            while (rl32(q_count, d) > 0) {
                const int32_t at = rl32(q_head, d);
                if (at == rl32(q_end, d)) {   // the next 64 entries into LDS
                    const int32_t i = at + lane;
                    __builtin_amdgcn_s_waitcnt(0);   // the ring's stores have reached L2, where it is read
                    if (lane < rl32(q_count, d)) {
                        const uint64_t* e = reinterpret_cast<const uint64_t*>(rings + int64_t(d) * n + i);
                        const uint64_t lo = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const uint64_t hi = __hip_atomic_load(e + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        q_fifo[d * kStep4 + i % kWave] = make_int4(int32_t(lo), int32_t(lo >> 32), int32_t(hi),
                                                                  int32_t(hi >> 32));
                    }
                    if (lane == d) q_end += kWave;
                }
                const int4 h = q_fifo[d * kStep4 + at % kWave];
                const int32_t hi = uniform(h.x), hp = uniform(h.y), ho = uniform(h.z), hb = uniform(h.w);
                if (uint32_t(rl32(K, d)) + uint32_t(hp + ho) > uint32_t(C)) break;   // both at most C < 2^31
                if (!admit(d, hi, ho, hp + ho)) { over = 1; break; }
                if (lane == d) {
                    if (policy == 1 && hb >= 0) R -= int64_t(hp) + hb;
                    q_head += 1;
                    q_count -= 1;
                }
            }
        }
        // 3. arrivals at t, in index order
        while (uniform(over) == 0 && next_arrival() == t) {
            const int j = next - wbase;
            const int32_t pi = rl32(st.w_p, j), oi = rl32(st.w_o, j), bi = rl32(st.w_b, j);
            int d;
            if (policy == 1 && bi >= 0) {   // Algorithm 1 at block size 1
                const int64_t need = int64_t(pi) + bi;
                const int64_t eff = lane < N ? int64_t(C) - K - R : INT64_MIN;
                const bool feasible = need <= eff;
                if (__builtin_amdgcn_ballot_w64(feasible) != 0) {
                    d = int(min8(feasible ? (uint32_t(q_count) << 3) | uint32_t(lane) : ~0u) & 7u);
                } else {
                    const int64_t most = max8(eff);
                    d = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(eff == most)) - 1;
                }
            } else {
                d = rr;
            }
            d = uniform(d);
            if (rl32(q_count, d) == 0 && uint32_t(rl32(K, d)) + uint32_t(pi + oi) <= uint32_t(C)) {
                if (!admit(d, next, oi, pi + oi)) { over = 1; break; }
                dirty |= 1ull << d;
            } else if (lane == d) {
                const int4 e = make_int4(next, pi, oi, bi);
                const int32_t tail = q_head + q_count;
                if (tail < q_end) q_fifo[d * kStep4 + tail % kWave] = e;
                else rings[int64_t(d) * n + tail] = e;
                q_count += 1;
                if (policy == 1 && bi >= 0) R += int64_t(pi) + bi;
            }
            if (lane == 0 && rout) rout[next] = d;
            next += 1;
            rr = rr + 1 == N ? 0 : rr + 1;
        }
        if (uniform(over) != 0) break;
        // the changed queues' next completions
        for (uint64_t c = dirty; c != 0; c &= c - 1) {
            const int d = __ffsll((unsigned long long)c) - 1;
            if (uniform(cur) != d) enter(d);   // the one in hand is at t: it has just changed
            const uint32_t slices = pos < count ? __umul24(uint32_t(left - 1), uint32_t(count)) + uint32_t(pos) + 1u
                                                : ~0u;
            const uint32_t least = wave_last(
                wave_incl_scan(slices, ~0u, [](uint32_t x, uint32_t y) { return x < y ? x : y; }));
            if (lane == d) due = count > 0 ? t + least : ~0u;
        }
        // the next event, and the state recorded over [t, t_next)
        const uint32_t first_due = min8(lane < N ? due : ~0u), arrives = next_arrival();
        const uint32_t t_next = uint32_t(uniform(int32_t(first_due < arrives ? first_due : arrives)));
        if (t_next == ~0u) break;   // unreachable: requests are left, so one arrives or completes
        const int32_t len = int32_t(t_next - t);
        const bool high = K >= k_high;
        hp_count += high && run == 0;
        run = high ? run + len : 0;
        hp_time += high ? len : 0;
        hp_max = run > hp_max ? run : hp_max;
        area += int64_t(uint64_t(uint32_t(q_count)) * uint32_t(len));
        max_queue = q_count > max_queue ? q_count : max_queue;
        t = t_next;
    }
    DecRegs& me = st.me;
    me.K = K;
    me.R = R;
    me.run = run;
    me.hp_time = hp_time;
    me.hp_max = hp_max;
    me.hp_count = hp_count;
    me.max_queue = max_queue;
    me.queue_area = area;
    me.nready = nready;
    if (!over) {
        if (done < n && lane == 0) raise_error(a.dev_err, MAPS_ERR_SIM_INPUT);
        return true;
    }
    // every queue in service order at t
    int32_t* rid = lds;
    int32_t* rleft = lds + N * kReady;
    uint32_t* rdem = reinterpret_cast<uint32_t*>(lds + 2 * N * kReady);
    for (int d = 0; d < N; ++d) {
        enter(d);
        if (pos < count) {
            const int2 req = q_req[d * kStep2 + lane];
            rid[d * kReady + pos] = req.x;
            rleft[d * kReady + pos] = left;
            rdem[d * kReady + pos] = uint32_t(req.y);
        }
        // the FIFO entries in LDS into the ring
        const int32_t i = rl32(q_head, d) + lane;
        if (lane < rl32(q_count, d) && i < rl32(q_end, d))
            rings[int64_t(d) * n + i] = q_fifo[d * kStep4 + i % kWave];
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the ring is read through the vector L1 from here on
    me.q_head = q_head == n ? 0 : q_head;
    me.q_count = q_count;
    if (lane < N && q_count > 0) me.head = rings[int64_t(lane) * n + q_head];
    st.t = origin + t;
    me.t_sync = st.t;
    me.next_done = kNever;   // scheduled again by simulate_general
    st.next = next;
    st.done = done;
    st.resumed = true;
    return false;
}

__global__ __launch_bounds__(kSimNT) void simulate_kernel(SimArgs a) {
    extern __shared__ __align__(16) int32_t lds[];
    const int s = blockIdx.x;
    const int lane = threadIdx.x;
    const int32_t N = a.N;
    const int64_t* arr = a.arrival + int64_t(s) * a.n;
    SimState st{};
    st.t = arr[0];
    st.last = st.t;
    st.me.next_done = kNever;
    st.me.t_sync = st.t;   // the first arrival
    if (!fits_fast(a, arr)) {
        refill(a, arr, st, 0);
        simulate_general(a, st, lds);
    } else if (!simulate_fast(a, st, lds)) {
        simulate_general(a, st, lds);
    }
    const DecRegs& me = st.me;
    if (lane < N) {
        int64_t* o = a.stats + int64_t(s) * 5 * N;
        o[0 * N + lane] = me.hp_time;
        o[1 * N + lane] = me.hp_max;
        o[2 * N + lane] = me.hp_count;
        o[3 * N + lane] = me.max_queue;
        o[4 * N + lane] = me.queue_area;
    }
    if (lane == 0) {
        a.span[2 * int64_t(s)] = arr[0];
        a.span[2 * int64_t(s) + 1] = st.last;
    }
}

}  // namespace
}  // namespace maps

using namespace maps;

extern "C" size_t maps_simulate_workspace_size(int32_t N, int64_t n, int32_t S) {
    if (N < 1 || N > MAPS_MAX_SIM_DECODERS || n < 1 || S < 0) return 0;
    return align256(size_t(S) * size_t(N) * size_t(n) * sizeof(int4));
}

extern "C" maps_status maps_simulate(int32_t N, int64_t C, int32_t theta_ppm, int64_t n, int32_t S,
                                     const int64_t* arrival_ms, const int32_t* prompt, const int32_t* output,
                                     const int32_t* bound, const int32_t* policy, int64_t* finish_ms,
                                     int32_t* routed, int64_t* stats, int64_t* span, uint32_t* dev_err,
                                     void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (N < 1 || N > MAPS_MAX_SIM_DECODERS || C < 1 || n < 1 || n > INT32_MAX || S < 0 || theta_ppm < 1 ||
        theta_ppm > 1000000)
        return MAPS_E_SIZE;
    if (S == 0) return MAPS_OK;
    if (!arrival_ms || !prompt || !output || !bound || !policy || !finish_ms || !stats || !span || !dev_err ||
        !workspace)
        return MAPS_E_NULL;
    if (workspace_bytes < maps_simulate_workspace_size(N, n, S)) return MAPS_E_WORKSPACE;
    SimArgs a{N, C, theta_ppm, n, S, arrival_ms, prompt, output, bound, policy, finish_ms, routed, stats, span,
              static_cast<int4*>(workspace), dev_err};
    const size_t lds = size_t(N) * kReady * 3 * sizeof(int32_t);
    allow_dynamic_lds(simulate_kernel, lds);
    hipLaunchKernelGGL(simulate_kernel, dim3(unsigned(S)), dim3(kSimNT), lds, stream, a);
    MAPS_CHECK_LAUNCH();
    return MAPS_OK;
}
