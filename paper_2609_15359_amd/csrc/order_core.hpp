#pragma once
// Local SJF order and admission (Sec. 3.3, Eq. (7); App. A, Eq. (10)) on gfx950:
// the device code, shared by the local-order launch and the launch that ends
// placement and orders every local queue.
//
// One workgroup per decoder:
//   1. bitonic sort of the packed keys (promoted?0:1, promoted? index :
//      bound, index) -- unique keys, so the order is the stable one;
//   2. a second bitonic sort of (bound, index) gives the queue by bound, with
//      the start of each run of equal bounds;
//   (a queue of at most 64 requests is ordered by counting instead, each
//   wavefront counting against 4 of its requests);
//   3. admitted = the largest k whose prefix keeps the projected peak within
//      the capacity.  For a prefix, residents plus admitted requests form
//      a curve that increases between breakpoints -- the residents' event
//      times and the requests' bounds -- so the peak is its maximum over those
//      points, and k is the least, over the points, of the largest prefix that
//      fits there.  The order is the promoted requests, then the others by
//      bound, so at a point t a prefix past the promoted ones holds the
//      promoted requests with bound >= t (masked suffix sums over the
//      bound-sorted queue) and a contiguous run of the others (a difference of
//      prefix sums): one pass over the points, each with one search of its
//      place among the bounds and, only where the wavefront's best prefix so
//      far does not fit, a search of the prefix.  Where the promoted requests
//      alone do not fit, a few of them are added up in order; of more, the
//      prefix that fits at the worst point is an upper end, and is the answer
//      when it fits at every point, else the next one comes from the point
//      that it exceeds most (see admit_promoted).
//      Residents' occupancy comes from the projection's LDS where the
//      workgroup has just built it (an event a thread), else from the snapshot
//      (record S + t N at the rank of t).
//      A binary search over k with one pass a probe, the points handed out by
//      whole rank words (32 steps each, and the events crowd at the low
//      steps), took 45 us of a projection of 4 decoders x 64 residents and 120
//      us of 61 x 1,021 with room in the queues; this pass takes 1 and 2.5 us
//      of them, 5 us with 2,100 events and 6 with 3,600 a decoder.
#include "maps_internal.hpp"

namespace maps {
namespace order {

constexpr int kOrderNT = 1024;
constexpr int kMaxQ = MAPS_MAX_LOCAL_QUEUE;
// Up to so many promoted requests are added up in order at each point where
// they do not all fit; more of them go through admit_promoted, which takes some
// 10 us whatever their number, against 0.3 us a request (a queue of 200 beside
// 64 residents: 30, 35, 40 and 45 us with 4, 24, 48 and 64 of them added up, 40 to
// 44 us the other way).
constexpr int kAddUp = 48;

struct LocalArgs {
    SnapLayout L;
    const void* snap;
    const int32_t* cap;
    const int64_t* q_off;
    int64_t total;
    const int32_t* qp;
    const int32_t* qU;
    const int32_t* qwait;
    int32_t max_wait;
    int32_t* order;
    int32_t* admitted;
    uint32_t* dev_err;
};

struct LocalLds {
    // the sort keys (steps 1-2) and the prompt suffix sums (step 3) are never
    // live together, nor the bounds by index (steps 1-2) and the prefix sums
    // (step 3): sharing their space leaves room for two workgroups per CU
    union {
        uint64_t keys[kMaxQ];
        int64_t psuf[kMaxQ + 1];  // prompts summed over the requests csuf counts
    };
    union {
        int32_t ue[kMaxQ];        // bound of entry i (missing bound -> u_max)
        int64_t ppre[kMaxQ + 1];  // prompts of the unpromoted requests before a position of the new order
        int2 pro[kMaxQ];          // the promoted requests in order, {prompt, bound}, once ppre is not needed
    };
    int32_t pos[kMaxQ];       // position of queue entry i in the new order
    int32_t pp[kMaxQ];        // prompt of entry i
    int32_t uidx[kMaxQ];      // entries sorted by (bound, index)
    int32_t us[kMaxQ];        // their bounds
    int32_t csuf[kMaxQ + 1];  // step 3: promoted requests with bound >= that position's bound;
                              // until then the entry at each position of the new order
    int2 pro64[kWave];        // the promoted requests in order, up to 64
    int64_t red64[kOrderNT / kWave];
    int32_t red32[kOrderNT / kWave];
    int32_t promoted;         // promoted requests
    int64_t worst_t, worst_room;   // the point that a prefix exceeds most
};

// keys[0..n2), n2 a power of two from 64 to kMaxQ, ascending; begins and ends with
// a barrier.  Up to one key per thread they are sorted in registers.
__device__ inline void sort_keys(uint64_t* keys, int n2) {
    __syncthreads();
    if (n2 <= kOrderNT) {
        const uint64_t mine = int(threadIdx.x) < n2 ? keys[threadIdx.x] : ~0ull;
        const uint64_t key = block_sort(mine, n2, keys);
        __syncthreads();
        if (int(threadIdx.x) < n2) keys[threadIdx.x] = key;
        __syncthreads();
        return;
    }
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += kOrderNT) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const uint64_t a = keys[i], b = keys[ixj];
                    const bool up = (i & k) == 0;
                    if ((a > b) == up) { keys[i] = b; keys[ixj] = a; }
                }
            }
            __syncthreads();
        }
    }
}

// First bound-sorted position with bound >= t.
__device__ inline int first_bound(const LocalLds& s, int n, int64_t t) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s.us[mid] < t) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// a * b of values below 2^32: one instruction.
__device__ inline int64_t mul_wide(int64_t a, int64_t b) { return int64_t(uint64_t(uint32_t(a)) * uint32_t(b)); }

// fn(valid, t, O(t), first bound-sorted position with bound >= t) at every
// resident event of the snapshot's slice, over the workgroup's threads;
// called by whole wavefronts (valid: the lane has a point).  A thread takes 4
// steps of a rank word at a time, or the whole word where the step axis is
// long and the events are sparse on it, and loads the rank words and first
// records of 4 such units together.
template <typename Fn>
__device__ inline void for_each_event(const LocalLds& s, int n, const uint2* rank, const int2* cold, int32_t E,
                                      int32_t W, Fn fn) {
    constexpr int kU = 4;
    const int lg = W <= 4096 ? 3 : 0, nb = 32 >> lg;   // 2^lg units of nb steps a word
    const int64_t units = int64_t(W) << lg;
    for (int64_t u0 = 0; u0 < units; u0 += kU * kOrderNT) {
        uint2 rw[kU];
        uint32_t bits[kU], e[kU];
        int32_t t0[kU];
        int2 r[kU];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int64_t u = u0 + j * kOrderNT + threadIdx.x;
            rw[j] = u < units ? rank[u >> lg] : make_uint2(0u, 0u);
            t0[j] = int32_t(u << (5 - lg));
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int sh = t0[j] & 31;
            bits[j] = lg == 0 ? rw[j].x : (rw[j].x >> sh) & ((1u << nb) - 1u);
            e[j] = rw[j].y + uint32_t(__popc(rw[j].x & ((1u << sh) - 1u)));
            if (e[j] >= uint32_t(E)) { e[j] = uint32_t(E); bits[j] = 0u; }
            r[j] = bits[j] != 0u ? cold[e[j]] : make_int2(0, 1);
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            int lo = -1;
            while (__builtin_amdgcn_ballot_w64(bits[j] != 0u) != 0) {
                const bool valid = bits[j] != 0u;
                int64_t tau = 0, occ = 0;
                int2 next = r[j];
                if (valid) {
                    tau = int64_t(t0[j]) + (__ffs(bits[j]) - 1);
                    occ = int64_t(r[j].x) + mul_wide(tau, r[j].y - 1);
                    bits[j] &= bits[j] - 1u;
                    ++e[j];
                    if (e[j] >= uint32_t(E)) bits[j] = 0u;
                    else if (bits[j] != 0u) next = cold[e[j]];   // in flight during fn
                    if (lo < 0) lo = first_bound(s, n, tau);
                    else
                        while (lo < n && s.us[lo] < tau) ++lo;
                }
                fn(valid, tau, occ, lo < 0 ? 0 : lo);
                r[j] = next;
            }
        }
    }
}

// The events of the decoder that this workgroup has just projected, still in
// its LDS: times, and the occupancy at each (cap: where the occupancies start;
// 0: not there).
struct LdsEvents {
    const uint32_t* base;
    int64_t cap;
};

// fn(valid, t, O(t), first bound-sorted position with bound >= t) at every
// point, the decoder's events and the queue's bounds, by whole wavefronts.
template <typename Fn>
__device__ inline void for_each_point(const LocalLds& s, int n, const uint2* rank, const int2* cold, int32_t E,
                                      int32_t W, const LdsEvents& ev, Fn point) {
    // the bounds' records are on their way during the events
    const int32_t ucl_max = 32 * W - 1;
    const int i0 = int(threadIdx.x);
    auto record = [&](int i, int64_t& t) -> int2 {
        t = s.us[i];
        const int32_t tc = t < ucl_max ? int32_t(t) : ucl_max;
        const uint2 w = rank[tc >> 5];
        const uint32_t at = w.y + __popc(w.x & ((1u << (tc & 31)) - 1u));
        return at < uint32_t(E) ? cold[at] : make_int2(0, 1);
    };
    int64_t t0 = 0;
    int2 r0 = make_int2(0, 1);
    if (i0 < n) r0 = record(i0, t0);
    if (ev.cap > 0) {
        for (int e0 = 0; e0 < E; e0 += kOrderNT) {
            const int e = e0 + int(threadIdx.x);
            const bool valid = e < E;
            if (__builtin_amdgcn_ballot_w64(valid) == 0) break;
            const int64_t tau = valid ? int64_t(ev.base[e]) : 0;
            const int64_t occ = valid ? int64_t(int32_t(ev.base[ev.cap + e])) : 0;
            point(valid, tau, occ, valid ? first_bound(s, n, tau) : 0);
        }
    } else {
        for_each_event(s, n, rank, cold, E, W, point);
    }
    for (int b0 = 0; b0 < n; b0 += kOrderNT) {
        const int i = b0 + i0;
        const bool valid = i < n;
        if (__builtin_amdgcn_ballot_w64(valid) == 0) break;
        if (b0 > 0 && valid) r0 = record(i, t0);
        point(valid, t0, valid ? int64_t(r0.x) + mul_wide(t0, r0.y - 1) : 0, valid ? first_bound(s, n, t0) : 0);
    }
}

// The point that a prefix exceeds most, over the workgroup's threads, each
// with its own in (over, t, room); over <= 0: none.  Returns whether there is
// one, then in worst_t and worst_room.  Ends with a barrier.
__device__ inline bool worst_point(LocalLds& s, int64_t over, int64_t t, int64_t room) {
    const int64_t most = block_reduce_max<kOrderNT>(over, s.red64);
    if (most <= 0) return false;   // the same in every thread
    const int32_t who = block_reduce_max<kOrderNT>(over == most ? int32_t(threadIdx.x) : -1, s.red32);
    if (int32_t(threadIdx.x) == who) {
        s.worst_t = t;
        s.worst_room = room;
    }
    __syncthreads();
    return true;
}

// The largest prefix of the promoted requests that fits, where not all do (the
// point in worst_t and worst_room does not hold them).  What the promoted requests hold at one point only grows with the
// prefix, so the largest one that fits there, a masked prefix sum in order, is
// an upper end; a pass over the points (with the masked suffix sums over the
// bounds for this prefix) shows whether it fits everywhere or which point it
// exceeds most.  Mostly one to three such passes; from the fifth on every second
// one takes the middle of what is left, so that there are at most some twenty.
// 256 decoders with 64 residents and 2,048 promoted requests, of which a third
// fits, take 117 us, and 61 with 512; adding the requests up at every point took
// 1,207 and 283, the binary search over k 191 and 110.
__device__ inline int admit_promoted(LocalLds& s, int n, int32_t C, const uint2* rank, const int2* cold, int32_t E,
                                     int32_t W, const LdsEvents& ev) {
    const int np = s.promoted;
    __syncthreads();   // ppre is done with
    for (int i = int(threadIdx.x); i < n; i += kOrderNT) {
        const int j = s.uidx[i], at = s.pos[j];
        if (at < np) s.pro[at] = make_int2(s.pp[j], s.us[i]);
    }
    __syncthreads();
    auto fit_at_worst = [&]() {
        const int64_t t = s.worst_t, room = s.worst_room;
        int32_t fit = 0;
        block_scan<kOrderNT, false, false, false, int64_t>(
            np, int64_t(0), [&](int64_t i) { const int2 r = s.pro[i]; return r.y >= t ? int64_t(r.x) + t : int64_t(0); },
            [&](int64_t, int64_t v) { fit += v <= room; }, s.red64);
        return block_reduce_add<kOrderNT>(fit, s.red32);
    };
    int lo = 0, up = fit_at_worst();   // lo fits, nothing past up does
    for (int turn = 0; lo < up; ++turn) {
        const int k = turn >= 4 && turn % 2 == 0 ? (lo + up + 1) / 2 : up;
        block_scan<kOrderNT, false, true, false, int32_t>(
            n, 0, [&](int64_t i) { return int32_t(s.pos[s.uidx[i]] < k); },
            [&](int64_t i, int32_t v) { s.csuf[i] = v; }, s.red32);
        block_scan<kOrderNT, false, true, false, int64_t>(
            n, int64_t(0),
            [&](int64_t i) { const int j = s.uidx[i]; return s.pos[j] < k ? int64_t(s.pp[j]) : int64_t(0); },
            [&](int64_t i, int64_t v) { s.psuf[i] = v; }, s.red64);   // csuf[n] and psuf[n] stay 0
        int64_t over = 0, at = 0, room_at = 0;
        for_each_point(s, n, rank, cold, E, W, ev, [&](bool valid, int64_t t, int64_t occ, int first) {
            const int64_t room = int64_t(C) - occ;
            const int64_t x = s.psuf[first] + mul_wide(t, s.csuf[first]) - room;
            if (valid && x > over) {
                over = x;
                at = t;
                room_at = room;
            }
        });
        if (!worst_point(s, over, at, room_at)) {
            lo = k;
        } else {
            const int fit = fit_at_worst();   // below k
            up = fit < up ? fit : up;
        }
    }
    return lo;
}

// The largest k whose prefix fits (the residents alone do): see step 3 above.
// The prefix sums and the promoted requests' suffix sums are ready.
__device__ inline int admit(LocalLds& s, int n, int32_t C, const uint2* rank, const int2* cold, int32_t E, int32_t W,
                            const LdsEvents& ev) {
    const int np = s.promoted;
    int best = n;   // the largest prefix that fits at every point of this wavefront so far
    int64_t most = 0, most_t = 0, most_room = 0;   // this thread's point that the promoted requests exceed most
    for_each_point(s, n, rank, cold, E, W, ev, [&](bool valid, int64_t t, int64_t occ, int lo) {
        const int c = s.csuf[lo];
        const int64_t room = int64_t(C) - occ;
        const int64_t rest = room - (s.psuf[lo] + mul_wide(t, c));   // with every promoted request there
        const int first = lo + c;   // the new order's first unpromoted request with bound >= t
        const int64_t base = s.ppre[first];
        auto fits = [&](int k) { return k <= first || s.ppre[k] - base + mul_wide(t, k - first) <= rest; };
        const bool over = valid && rest < 0;
        const bool search = valid && rest >= 0 && !fits(best);
        if (__builtin_amdgcn_ballot_w64(search || over) == 0) return;   // the usual case after the first few points
        int mine = best;
        if (search) {
            int a = first, b = best - 1;   // fits(first), not fits(best)
            while (a < b) {
                const int mid = (a + b + 1) >> 1;
                if (fits(mid)) a = mid; else b = mid - 1;
            }
            mine = a;
        }
        if (over && -rest > most) {
            most = -rest;
            most_t = t;
            most_room = room;
        }
        if (np <= kAddUp && __builtin_amdgcn_ballot_w64(over) != 0) {   // add the promoted requests up
            int64_t sum = 0;
            bool held = over;
            for (int j = 0; j < (best < np ? best : np); ++j) {
                const int2 r = s.pro64[j];
                sum += r.y >= t ? int64_t(r.x) + t : int64_t(0);
                if (held && sum > room) {
                    mine = j;
                    held = false;
                }
                if (__builtin_amdgcn_ballot_w64(held) == 0) break;
            }
        }
        best = -wave_reduce_max(-mine);
    });
    // above every -best: somewhere the promoted requests alone do not fit
    const int most_k = block_reduce_max<kOrderNT>(np > kAddUp && most > 0 ? 1 : -best, s.red32);
    if (most_k <= 0) return -most_k;
    worst_point(s, most, most_t, most_room);
    return admit_promoted(s, n, C, rank, cold, E, W, ev);
}

// Decoder d's queue bounds and capacity, and, when the queue holds at most
// one wavefront of requests, request i's prompt, bound and wait in lane i of
// every wavefront (0 elsewhere).  Called early by a launch that has other work first, so
// that these loads are in flight during it.
struct QueueFetch {
    int64_t qlo, qhi;
    int32_t C, pr, u, wait;
};

__device__ inline QueueFetch fetch_queue(const LocalArgs& g, int32_t d) {
    QueueFetch f;
    f.qlo = g.q_off[d];
    f.qhi = g.q_off[d + 1];
    f.C = g.cap[d];
    f.pr = 0;
    f.u = 0;
    f.wait = 0;
    const int64_t i = f.qlo + int64_t(threadIdx.x % kWave);   // every wavefront holds the short queue
    if (0 <= f.qlo && f.qlo <= f.qhi && f.qhi <= g.total && f.qhi - f.qlo <= kWave && i < f.qhi) {
        f.pr = g.qp[i];
        f.u = g.qU[i];
        f.wait = g.qwait != nullptr ? g.qwait[i] : 0;
    }
    return f;
}

// The whole local order of decoder d by one workgroup of kOrderNT threads, in
// the LDS `s` (free for it when every thread arrives here).
// built != nullptr: the snapshot's decoder d was written by this workgroup
// (the projection's launch), which passes the header it wrote (the
// snapshot's own header, written by another workgroup, cannot be read back
// reliably) and the resident count.  pre (nullable): fetch_queue's values.
// ev: the decoder's events in LDS outside `s`, if there.
__device__ inline void order_queue(const LocalArgs& g, int32_t d, LocalLds& s, int64_t built_n_total = -1,
                                   const DecHeader* built = nullptr, const QueueFetch* pre = nullptr,
                                   const LdsEvents& ev = LdsEvents{nullptr, 0}) {
    const SnapLayout& L = g.L;
    const SnapView V = snap_view(const_cast<void*>(g.snap), L);
    int64_t n_total = built_n_total;
    if (built == nullptr) {
        const SnapHeader hdr = *V.hdr;
        if (!(hdr.magic == kSnapMagic && hdr.D == L.D && hdr.u_max == L.u_max && hdr.W == L.W)) {
            if (d == 0 && threadIdx.x == 0) raise_error(g.dev_err, MAPS_ERR_SNAPSHOT);
            return;
        }
        n_total = hdr.n_total;
    }
    const DecHeader h = built != nullptr ? *built : V.dec[d];
    if (!slice_ok(h, n_total, L)) {
        if (threadIdx.x == 0) raise_error(g.dev_err, MAPS_ERR_SNAPSHOT);
        return;
    }
    const QueueFetch f = pre != nullptr ? *pre : fetch_queue(g, d);
    const int64_t qlo = f.qlo, qhi = f.qhi;
    if (!(0 <= qlo && qlo <= qhi && qhi <= g.total)) {
        if (threadIdx.x == 0) { raise_error(g.dev_err, MAPS_ERR_SEG_OFFSETS); g.admitted[d] = 0; }
        return;
    }
    const int64_t n64 = qhi - qlo;
    if (n64 > kMaxQ) {
        if (threadIdx.x == 0) { raise_error(g.dev_err, MAPS_ERR_QUEUE_TOO_LONG); g.admitted[d] = 0; }
        return;
    }
    const int n = int(n64);
    const int32_t C = f.C;
    if (threadIdx.x == 0 && C < 0) raise_error(g.dev_err, MAPS_ERR_NEG_LEN);
    int n2 = 1;
    while (n2 < n) n2 <<= 1;

    if (n2 <= kWave) {
        // A queue of at most one wavefront: request i in lane i of every
        // wavefront.  Both orders by counting: the new position of i is the
        // number of requests before it by (class and key, index), its place
        // by bound the number before it by (bound, index).  Wavefront
        // w counts against requests [4w, 4w + 4); wave 0 adds the counts.
        constexpr int kWaves = kOrderNT / kWave;
        constexpr int kPer = kWave / kWaves;   // requests each wavefront counts against
        const int i = int(threadIdx.x % kWave), w = int(threadIdx.x / kWave);
        bool neg = false, promoted = false;
        uint32_t key = ~0u, ue = ~0u;   // past the queue: after every request
        if (i < n) {
            neg = f.pr < 0;
            ue = uint32_t(f.u < 0 ? L.u_max : f.u);
            promoted = g.qwait != nullptr && f.wait >= g.max_wait;
            key = promoted ? uint32_t(i) : (0x80000000u | ue);   // class bit, then index or bound
        }
        if (neg && w == 0) raise_error(g.dev_err, MAPS_ERR_NEG_LEN);
        uint32_t r1 = 0, r2 = 0;
#pragma unroll
        for (int jj = 0; jj < kPer; ++jj) {
            const int j = w * kPer + jj;
            if (j >= n) break;   // uniform
            const uint32_t hj = __builtin_amdgcn_readlane(key, j), uj = __builtin_amdgcn_readlane(ue, j);
            r1 += (hj < key) | ((hj == key) & (j < i));
            r2 += (uj < ue) | ((uj == ue) & (j < i));
        }
        uint32_t* part = reinterpret_cast<uint32_t*>(s.keys);   // [2][kWaves][kWave], free until step 3
        part[(0 * kWaves + w) * kWave + i] = r1;
        part[(1 * kWaves + w) * kWave + i] = r2;
        __syncthreads();
        if (w == 0 && i < n) {
            uint32_t a1 = 0, a2 = 0;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) {
                a1 += part[(0 * kWaves + v) * kWave + i];
                a2 += part[(1 * kWaves + v) * kWave + i];
            }
            g.order[qlo + a1] = i;
            s.pos[i] = int32_t(a1);
            s.pp[i] = f.pr < 0 ? 0 : f.pr;
            s.uidx[a2] = i;
            s.us[a2] = int32_t(ue);
            s.csuf[a1] = i;
        }
        __syncthreads();
        // step 3's sums in one wavefront
        if (w == 0 && h.base_peak <= C) {
            const int np = __popcll(__builtin_amdgcn_ballot_w64(promoted));
            const bool in = i < n;
            const int64_t p1 = in && i >= np ? s.pp[s.csuf[i]] : 0;
            const int j = in ? s.uidx[i] : 0;
            const bool m = in && s.pos[j] < np;
            const int64_t p2 = m ? s.pp[j] : 0;
            const int64_t q1 = wave_incl_scan_add(p1), q2 = wave_incl_scan_add(p2);
            const int32_t c2 = wave_incl_scan_add(int32_t(m));
            const int64_t all2 = wave_last(q2);
            const int32_t allc = wave_last(c2);
            const int32_t own = in ? s.csuf[i] : 0;
            const int32_t own_p = s.pp[own], own_u = __shfl(int(ue), own, kWave);
            if (in) {   // part (the keys) and the entries by position were last read above, by this wavefront
                s.pro64[i] = make_int2(own_p, own_u);   // for i < np the promoted requests in order
                s.ppre[i + 1] = q1;
                s.psuf[i] = all2 - q2 + p2;
                s.csuf[i] = allc - c2 + int32_t(m);
            }
            if (i == 0) {
                s.ppre[0] = 0;
                s.psuf[n] = 0;
                s.csuf[n] = 0;
                s.promoted = np;
            }
        }
        __syncthreads();
    } else {
        // 1. the new order (Eq. (7) with promotion)
        bool neg = false;
        for (int i = threadIdx.x; i < n2; i += kOrderNT) {
            if (i < n) {
                int32_t pr = g.qp[qlo + i], u = g.qU[qlo + i];
                neg |= pr < 0;
                s.pp[i] = pr < 0 ? 0 : pr;
                const int32_t ue = u < 0 ? L.u_max : u;
                s.ue[i] = ue;
                const bool promoted = g.qwait != nullptr && g.qwait[qlo + i] >= g.max_wait;
                const uint64_t cls = promoted ? 0ull : (1ull << 63);
                const uint64_t val = promoted ? uint64_t(i) : uint64_t(ue);
                s.keys[i] = cls | (val << 32) | uint64_t(uint32_t(i));
            } else {
                s.keys[i] = ~0ull;
            }
        }
        if (neg) raise_error(g.dev_err, MAPS_ERR_NEG_LEN);
        if (threadIdx.x == 0) s.promoted = 0;
        sort_keys(s.keys, n2);
        for (int i = threadIdx.x; i < n; i += kOrderNT) {
            const int idx = int(uint32_t(s.keys[i]));
            g.order[qlo + i] = idx;
            s.pos[idx] = i;
            s.csuf[i] = idx;
            if (!(s.keys[i] >> 63) && (i + 1 == n || (s.keys[i + 1] >> 63))) s.promoted = i + 1;
        }
        __syncthreads();

        if (h.base_peak <= C) {   // else nothing is admitted, and only the order is wanted
            // 2. the queue sorted by bound
            for (int i = threadIdx.x; i < n2; i += kOrderNT)
                s.keys[i] = i < n ? ((uint64_t(uint32_t(s.ue[i])) << 32) | uint64_t(uint32_t(i))) : ~0ull;
            sort_keys(s.keys, n2);
            for (int i = threadIdx.x; i < n; i += kOrderNT) {
                s.uidx[i] = int(uint32_t(s.keys[i]));
                s.us[i] = int32_t(s.keys[i] >> 32);
            }
            __syncthreads();
            // step 3's sums: the prompts of the unpromoted requests before each
            // position, and the promoted requests' suffix sums by bound
            const int np = s.promoted;
            if (np <= kWave && int(threadIdx.x) < np) {   // the scan's barriers precede its writes over the bounds
                const int idx = s.csuf[threadIdx.x];
                s.pro64[threadIdx.x] = make_int2(s.pp[idx], s.ue[idx]);
            }
            block_scan<kOrderNT, false, false, false, int64_t>(
                n, int64_t(0), [&](int64_t i) { return i >= np ? int64_t(s.pp[s.csuf[i]]) : int64_t(0); },
                [&](int64_t i, int64_t v) { s.ppre[i + 1] = v; }, s.red64);
            block_scan<kOrderNT, false, true, false, int32_t>(
                n, 0, [&](int64_t i) { return int32_t(s.pos[s.uidx[i]] < np); },
                [&](int64_t i, int32_t v) { s.csuf[i] = v; }, s.red32);
            block_scan<kOrderNT, false, true, false, int64_t>(
                n, int64_t(0),
                [&](int64_t i) { const int j = s.uidx[i]; return s.pos[j] < np ? int64_t(s.pp[j]) : int64_t(0); },
                [&](int64_t i, int64_t v) { s.psuf[i] = v; }, s.red64);
            if (threadIdx.x == 0) { s.ppre[0] = 0; s.csuf[n] = 0; s.psuf[n] = 0; }
            __syncthreads();
        }
    }

    // 3. admission: largest k with peak(k) <= C
    const uint2* rank = slice_rank(V, h);
    const int2* cold = slice_cold(V, h, L);
    const int k = h.base_peak <= C ? admit(s, n, C, rank, cold, h.E, L.W, ev) : 0;
    if (threadIdx.x == 0) g.admitted[d] = k;
}

}  // namespace order
}  // namespace maps
