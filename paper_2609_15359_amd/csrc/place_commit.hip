// Placement with sequential commit (Sec. 3.3: each dispatch atomically
// reserves its demand before the next request is placed; Algorithm 1) on
// gfx950.
//
// Arrivals are placed in order.  Each is evaluated against every decoder's
// projected occupancy, which includes the arrivals already committed to that
// decoder (a committed arrival (p, U) holds p + t at step t while t <= U), and
// is then committed to the decoder it chose.  Per decoder the dense step axis
// t = 0..T (T = u_max) is kept in the workspace:
//   O(t)   occupancy,
//   PF(u)  max_{t <= u} (O(t) + t)         (stored, see the floors below),
//   SA(u)  max_{t > u} O(t)                (0 at u = T),
// so that peak(p, U) = max(p + PF(U), SA(U)) is two reads.  Committing (p, U)
// changes O only on [0, U]; there PF and SA are derived again by workgroup
// scans.  Above U, PF(u) becomes max(PF(u), v) with v = PF(U) after the
// commit.  That tail is rewritten only up to the end of U's block of kFloorBlock
// steps; for the blocks after it v is recorded as a floor of the block
// (FB[k] = max(FB[k], v)), and a lookup takes max(PF(u), FB[block of u]).  A
// floor never exceeds the true prefix maximum (O only grows), and every change
// above the stored values is restored by the largest floor of an earlier
// block or the rewritten tail within the block, so the lookup is exact.
//
//   commit_init    one 1,024-thread workgroup per decoder: O(t) from the
//                  snapshot (the rank of t among the events, then S_e + t N_e),
//                  PF and SA by prefix and suffix scans, floors cleared.
//   commit_serial  one 512-thread workgroup for the whole chain: per arrival
//                  every decoder's peak (PF, SA and the block floor at U), the
//                  choice by a workgroup argmin, then the commit on [0, U] of
//                  the chosen decoder with its tail and block floors.
//                  Queue lengths and capacities live in LDS; with at most 512
//                  decoders the next arrival's lookups are issued with the
//                  commit's loads.
//   commit_rounds  the same chain with the commits of a round of arrivals in
//                  parallel, for policy MQ while decoders are feasible: see
//                  there.  commit_serial goes on where it ends.
#include "maps_internal.hpp"

namespace maps {
namespace {

constexpr int kCommitNT = 1024;            // threads of a workgroup building one decoder's curves
constexpr int kWaves = kCommitNT / kWave;
constexpr int kSerialNT = 512;             // threads of the chain's workgroup (256 VGPRs each: no spills)
constexpr int kSerialWaves = kSerialNT / kWave;
constexpr int64_t kFeasibleBias = int64_t(1) << 62;

constexpr int kFloorBlock = 1024;  // steps per floor block
constexpr int kFloorPer = 2;       // block floors a thread updates per commit: blocks up to 2 * kSerialNT
constexpr int kTailPer = kFloorBlock / kSerialNT;   // steps of a commit's own block above it per thread

struct CommitLayout {
    int32_t D, L, NB;      // decoders, steps per decoder (u_max + 1), floor blocks per decoder
    size_t off_O, off_PF, off_SA, off_F, off_ctl, bytes;
};

// The exchange of commit_rounds between the master and the owners, in device
// memory: every access is a device-coherent load or store (no cache holds it).
constexpr int kWindow = 128;        // arrivals evaluated ahead in a round
constexpr int kMaskWords = kWindow / 64;
constexpr int kRoundDecoders = 1024;
constexpr int kMaxOwners = 1024;
constexpr uint32_t kRun = 1u << 30, kDeclined = 1u << 31, kOwnerCount = kRun - 1u;   // of `entry`
// `round`, one word: the last round published above the arrivals it placed and
// whether another follows; kEnded: none does, whatever that says.
constexpr uint64_t kEnded = 1ull << 63;
constexpr uint32_t kMore = 1u << 31;
__host__ __device__ inline uint64_t round_word(uint32_t r, uint32_t placed, bool more) {
    return (uint64_t(r) << 32) | placed | (more ? kMore : 0u);
}
struct RoundControl {
    uint64_t round;
    uint32_t entry;        // owners that have checked in, and whether the rounds run
    uint32_t owners;       // those that had when the rounds began
    int64_t resume;        // the serial chain's first arrival
    uint32_t ready[kMaxOwners];                      // the round each owner has evaluated
    int32_t assign[kRoundDecoders];                  // the window's arrival committed to each decoder, or -1
    uint64_t feasible[kRoundDecoders][kMaskWords];   // the window's arrivals that each decoder holds
    int64_t over[kRoundDecoders];                    // overflow of the window's first arrival with a bound
    int32_t queue[kRoundDecoders];                   // queue lengths after the rounds (for the next launch)
};

CommitLayout commit_layout(int32_t D, int32_t u_max) {
    CommitLayout c;
    c.D = D;
    c.L = u_max + 1;
    c.NB = (c.L + kFloorBlock - 1) / kFloorBlock;
    const size_t dense = align256(size_t(D) * size_t(c.L) * sizeof(int64_t));
    c.off_O = 0;
    c.off_PF = dense;
    c.off_SA = 2 * dense;
    c.off_F = 3 * dense;
    c.off_ctl = c.off_F + align256(size_t(D) * size_t(c.NB) * sizeof(int64_t));
    c.bytes = c.off_ctl + align256(sizeof(RoundControl));
    return c;
}
// the blocks after a commit's own: at most NB - 1
static_assert((MAPS_MAX_COMMIT_U_MAX + kFloorBlock) / kFloorBlock - 1 <= kFloorPer * kSerialNT,
              "block floors per thread");
static_assert(kTailPer * kSerialNT >= kFloorBlock - 1, "steps of a block above a commit per thread");

struct CommitArgs {
    SnapLayout S;
    const void* snap;
    int64_t* O;
    int64_t* PF;
    int64_t* SA;
    int64_t* F;        // [D][NB] block floors: the largest v of a commit in an earlier block
    int32_t L, NB;
    int32_t stage_cap;   // range entries the chain stages in LDS
    const int32_t* cap;
    const int32_t* qlen;
    const int32_t* ap;
    const int32_t* aU;
    int64_t A;
    int32_t policy;
    int64_t rr_offset;
    int32_t* choice;
    int64_t* chosen_peak;
    int64_t* chosen_over;
    uint8_t* flags;
    int32_t* queue_out;
    uint32_t* dev_err;
    RoundControl* ctl;
    int32_t owners;      // workgroups of commit_rounds that may own decoders
    CommitWaits waits;
};

__device__ inline int64_t max64(int64_t a, int64_t b) { return a > b ? a : b; }

// ---------------------------------------------------------------------------
// Dense curves of every decoder from the snapshot
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kCommitNT) void commit_init(CommitArgs a) {
    __shared__ int64_t tmp[2][kWaves];
    const int d = blockIdx.x;
    const int32_t L = a.L;
    int64_t* O = a.O + int64_t(d) * L;
    int64_t* PF = a.PF + int64_t(d) * L;
    int64_t* SA = a.SA + int64_t(d) * L;
    int64_t* F = a.F + int64_t(d) * a.NB;
    for (int32_t i = threadIdx.x; i < a.NB; i += kCommitNT) F[i] = 0;
    if (d == 0 && a.owners > 0) {   // the exchange of the rounds starts open
        if (threadIdx.x == 0) {
            a.ctl->round = 0;
            a.ctl->entry = a.ctl->owners = 0;
            a.ctl->resume = 0;
        }
        for (int32_t i = threadIdx.x; i < kMaxOwners; i += kCommitNT) a.ctl->ready[i] = 0;
    }

    const SnapView V = snap_view(const_cast<void*>(a.snap), a.S);
    const SnapHeader* hs = V.hdr;
    bool ok = hs->magic == kSnapMagic && hs->D == a.S.D && hs->u_max == a.S.u_max && hs->W == a.S.W &&
              hs->P == a.S.P;
    DecHeader h{};
    if (ok) {
        h = V.dec[d];
        ok = slice_ok(h, hs->n_total, a.S);
    }
    if (!ok) {
        if (threadIdx.x == 0) raise_error(a.dev_err, MAPS_ERR_SNAPSHOT);
        for (int32_t t = threadIdx.x; t < L; t += kCommitNT) O[t] = PF[t] = SA[t] = 0;
        return;
    }
    const uint2* rank = slice_rank(V, h);
    const int2* cold = slice_cold(V, h, a.S);
    const uint32_t E = uint32_t(h.E);
    // occupancy at step t: the rank e of t among the events, then S_e + t N_e
    auto occ = [&](int32_t t) -> int64_t {
        const uint2 w = rank[t >> 5];
        uint32_t e = w.y + __popc(w.x & ((1u << (t & 31)) - 1u));
        e = e < E ? e : E;
        const int2 c = cold[e];
        return int64_t(c.x) + int64_t(t) * (c.y - 1);
    };
    // Each wavefront takes one segment of whole rows of 64 steps, a step per
    // lane, so that every array is written in whole cache lines (with a chunk
    // of consecutive steps per thread the 201 MB of 256 decoders x 32,769 steps
    // took 539 us): the segments' maxima first, then the rows upwards for PF and
    // downwards for SA, each with a wavefront scan and a carry.
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    const int32_t rows = (L + kWave - 1) / kWave, per = (rows + kWaves - 1) / kWaves;
    const int32_t r0 = wid * per < rows ? wid * per : rows, r1 = r0 + per < rows ? r0 + per : rows;
    int64_t mpre = 0, msuf = 0;
    for (int32_t r = r0; r < r1; ++r) {
        const int32_t t = r * kWave + lane;
        if (t < L) {
            const int64_t o = occ(t);
            mpre = max64(mpre, o + t);
            msuf = max64(msuf, o);
        }
    }
    mpre = wave_reduce_max(mpre);
    msuf = wave_reduce_max(msuf);
    if (lane == 0) { tmp[0][wid] = mpre; tmp[1][wid] = msuf; }
    __syncthreads();
    int64_t run = 0, after = 0;   // over the segments below and above this one
    for (int i = 0; i < kWaves; ++i) {
        if (i < wid) run = max64(run, tmp[0][i]);
        if (i > wid) after = max64(after, tmp[1][i]);
    }
    for (int32_t r = r0; r < r1; ++r) {
        const int32_t t = r * kWave + lane;
        const int64_t o = t < L ? occ(t) : 0;
        const int64_t pf = max64(run, wave_incl_scan_max(t < L ? o + t : int64_t(0)));
        if (t < L) {
            O[t] = o;
            PF[t] = pf;
        }
        run = wave_last(pf);
    }
    for (int32_t r = r1 - 1; r >= r0; --r) {
        // lane i takes the row's step 63 - i: the scan runs down the steps
        const int32_t t = r * kWave + (kWave - 1 - lane);
        const int64_t o = t < L ? occ(t) : 0;
        const int64_t incl = max64(after, wave_incl_scan_max(o));
        if (t < L) SA[t] = wave_shift_up1(incl, after);
        after = wave_last(incl);
    }
}

// ---------------------------------------------------------------------------
// The serial chain
// ---------------------------------------------------------------------------

constexpr int kRowBatch = 8;   // rows of 64 steps a wavefront loads at once

// Barrier that orders LDS traffic only: each wave waits for its own LDS
// operations, not for its global stores in flight (a full __syncthreads waits
// for those too, about a microsecond after the commit's stores).  The memory
// clobber keeps the compiler from moving memory accesses across it.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One decoder's peak inputs at step u: the stored prefix maximum, the floor
// of u's block, and the suffix maximum.
struct PeakIn {
    int64_t pf, fl, sa;
};

// Issued as three independent loads; the caller reads them once it needs them.
__device__ inline PeakIn peak_load(const CommitArgs& a, int32_t d, int32_t u) {
    const int64_t off = int64_t(d) * a.L + u;
    return PeakIn{a.PF[off], a.F[int64_t(d) * a.NB + u / kFloorBlock], a.SA[off]};
}

// Selection key of decoder d for the arrival (p, U): its peak and key.
__device__ inline int64_t commit_key(const PeakIn& in, int64_t p, int32_t C, int32_t Q, int32_t policy,
                                     int64_t* peak_out) {
    const int64_t peak = max64(p + max64(in.pf, in.fl), in.sa);
    const int64_t over = peak - C;
    *peak_out = peak;
    return (policy == MAPS_POLICY_MQ && over <= 0) ? int64_t(Q) - kFeasibleBias : over;
}

// Workgroup argmin of (key, d), lowest d on ties; every thread gets the
// result.  Wavefront minima by DPP, then one LDS round over the wavefronts.
__device__ inline void block_argmin(int64_t& key, int32_t& d, int64_t* skey, int32_t* sd) {
    const int64_t wk = wave_last(wave_incl_scan(key, INT64_MAX, [](int64_t x, int64_t y) { return x < y ? x : y; }));
    const int32_t wd =
        wave_last(wave_incl_scan(key == wk ? d : INT32_MAX, INT32_MAX,
                                 [](int32_t x, int32_t y) { return x < y ? x : y; }));
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    if (lane == 0) { skey[wid] = wk; sd[wid] = wd; }
    lds_barrier();
    key = skey[0];
    d = sd[0];
    for (int i = 1; i < kSerialWaves; ++i)
        if (skey[i] < key || (skey[i] == key && sd[i] < d)) { key = skey[i]; d = sd[i]; }
}

// Values of the committed decoder at the next arrival's step, taken while
// its arrays are rewritten: the new PF there (next step <= U) and the new SA
// (next step < U).
struct Capture {
    int64_t pf, sa;
};

// Holds a loaded value in a register from this point on: the wait for its
// load is placed here, before the stores that follow (on gfx9 one counter
// covers loads and stores, so a later first use would also wait for those).
__device__ inline void pin(int64_t& x) { asm volatile("" : "+v"(x)); }

// Commit (p, Uc) to decoder bd: O += p + t on [0, Uc], PF and SA derived
// again there, and the new PF(Uc) recorded as a floor above Uc.  Each
// wavefront takes one segment of whole rows of 64 steps, a step per lane, so
// that every access covers whole cache lines; the segments' maxima are
// exchanged once, then each row's PF and SA are a wavefront scan and a carry.
// (With a chunk of consecutive steps per thread each access touched 64 lines,
// and a range of 10,000 steps took 22 us, one past 18,000 about 60.)
// V = int32_t: every value fits (see commit_any) and the new O values stay in
// LDS (`stage`, Uc + 1 entries) between the passes; int64_t: they are read back
// from HBM.  `un` is the next arrival's step (-1: none): the lanes that rewrite
// PF(un) and SA(un) below Uc leave them in `cap`, and a thread with pre_d >= 0
// loads decoder pre_d's peak inputs at un into *pre_out, issued with the
// range's loads.  Returns the new PF(Uc), the same in every thread.  Ends with
// a barrier after which every store of the commit is visible to the workgroup.
template <typename V>
__device__ inline int64_t commit_range(const CommitArgs& a, V* stage, int32_t bd, int64_t p, int32_t Uc, int32_t un,
                                       int32_t pre_d, PeakIn* pre_out, Capture* cap, int64_t* scan_tmp,
                                       int64_t* scan_tmp2) {
    constexpr bool kStaged = sizeof(V) == 4;
    const int32_t L = a.L;
    const int lane = threadIdx.x % kWave, wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int64_t* O = a.O + int64_t(bd) * L;
    int64_t* PF = a.PF + int64_t(bd) * L;
    int64_t* SA = a.SA + int64_t(bd) * L;
    int64_t* Fd = a.F + int64_t(bd) * a.NB;
    const int32_t n = Uc + 1;
    const int32_t rows = (n + kWave - 1) / kWave, per = (rows + kSerialWaves - 1) / kSerialWaves;
    const int32_t r0 = wid * per < rows ? wid * per : rows, r1 = r0 + per < rows ? r0 + per : rows;
    // above Uc: the rest of its block (up to kTailPer steps per thread) and
    // the block floors after it (up to kFloorPer per thread), read with the
    // range and raised to v last
    const int32_t kc = Uc / kFloorBlock;
    const int32_t tail_end = (kc + 1) * kFloorBlock < L ? (kc + 1) * kFloorBlock : L;
    int64_t tail_old[kTailPer];
#pragma unroll
    for (int k = 0; k < kTailPer; ++k) {
        const int32_t tt = Uc + 1 + int32_t(threadIdx.x) + k * kSerialNT;
        tail_old[k] = tt < tail_end ? PF[tt] : 0;
    }
    int64_t fb_old[kFloorPer];
#pragma unroll
    for (int k = 0; k < kFloorPer; ++k) {
        const int32_t blk = kc + 1 + int32_t(threadIdx.x) + k * kSerialNT;
        fb_old[k] = blk < a.NB ? Fd[blk] : 0;
    }
    int64_t sa_top = SA[Uc];   // max of O beyond Uc: unchanged by the commit
    const bool pre = un >= 0 && pre_d >= 0;
    PeakIn pl{0, 0, 0};
    if (pre) pl = peak_load(a, pre_d, un);
    int64_t o[kRowBatch];
    auto load_rows = [&](int32_t rb) {
#pragma unroll
        for (int j = 0; j < kRowBatch; ++j) {
            const int32_t t = (rb + j) * kWave + lane;
            o[j] = rb + j < r1 && t < n ? O[t] : 0;
        }
    };
    load_rows(r0);
    // the loads issued before the range's are waited for now, ahead of its stores
    pin(sa_top);
    pin(pl.pf);
    pin(pl.fl);
    pin(pl.sa);
#pragma unroll
    for (int k = 0; k < kTailPer; ++k) pin(tail_old[k]);
#pragma unroll
    for (int k = 0; k < kFloorPer; ++k) pin(fb_old[k]);
    V mpre = 0, msuf = 0;
    for (int32_t rb = r0; rb < r1; rb += kRowBatch) {
        if (rb != r0) load_rows(rb);
#pragma unroll
        for (int j = 0; j < kRowBatch; ++j) {
            const int32_t t = (rb + j) * kWave + lane;
            if (rb + j < r1 && t < n) {
                const int64_t x = o[j] + p + t;
                O[t] = x;
                if constexpr (kStaged) stage[t] = V(x);
                mpre = V(x) + t > mpre ? V(x) + t : mpre;
                msuf = V(x) > msuf ? V(x) : msuf;
            }
        }
    }
    mpre = wave_reduce_max(mpre);
    msuf = wave_reduce_max(msuf);
    lds_barrier();   // every wave has read the scan arrays' earlier contents
    if (lane == 0) {
        scan_tmp[wid] = mpre;
        scan_tmp2[wid] = msuf;
    }
    lds_barrier();
    V run = 0, all = 0, after = V(sa_top);   // over the segments below and above this one
#pragma unroll
    for (int i = 0; i < kSerialWaves; ++i) {
        const V x = V(scan_tmp[i]), y = V(scan_tmp2[i]);
        if (i < wid) run = x > run ? x : run;
        if (i > wid) after = y > after ? y : after;
        all = x > all ? x : all;
    }
    const int64_t v = all;
    if (pre) *pre_out = pl;
    // the wavefront's own new O values, a step per lane (kDown: from the row's top down)
    V x[kRowBatch];
    auto fetch_rows = [&](int32_t rb, bool down) {
#pragma unroll
        for (int j = 0; j < kRowBatch; ++j) {
            const int32_t t = (rb + j) * kWave + (down ? kWave - 1 - lane : lane);
            const bool in = rb + j >= r0 && rb + j < r1 && t < n;
            if constexpr (kStaged) x[j] = in ? stage[t] : V(0);
            else x[j] = in ? V(O[t]) : V(0);
        }
    };
    if constexpr (!kStaged) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's O stores
    for (int32_t rb = r0; rb < r1; rb += kRowBatch) {
        fetch_rows(rb, false);
#pragma unroll
        for (int j = 0; j < kRowBatch; ++j) {
            const int32_t t = (rb + j) * kWave + lane;
            const bool in = rb + j < r1 && t < n;
            const V incl = wave_incl_scan_max(in ? V(x[j] + t) : V(0));
            const V pf = incl > run ? incl : run;
            if (in) {
                PF[t] = pf;
                if (t == un) cap->pf = pf;
            }
            run = wave_last(pf);
        }
    }
    // SA from the top down; lane i takes a row's step 63 - i
    const int32_t batches = (r1 - r0 + kRowBatch - 1) / kRowBatch;
    for (int32_t rb = r0 + (batches - 1) * kRowBatch; rb >= r0; rb -= kRowBatch) {
        fetch_rows(rb, true);
#pragma unroll
        for (int j = kRowBatch - 1; j >= 0; --j) {
            if (rb + j >= r1) continue;   // uniform
            const int32_t t = (rb + j) * kWave + (kWave - 1 - lane);
            const V scan = wave_incl_scan_max(x[j]);
            const V incl = scan > after ? scan : after;
            const V sa = wave_shift_up1(incl, after);
            if (t < Uc) {
                SA[t] = sa;
                if (t == un) cap->sa = sa;
            }
            after = wave_last(incl);
        }
    }
    // the new PF(Uc) = v is a floor for every step above Uc
#pragma unroll
    for (int k = 0; k < kTailPer; ++k) {
        const int32_t tt = Uc + 1 + int32_t(threadIdx.x) + k * kSerialNT;
        if (tt < tail_end) PF[tt] = max64(tail_old[k], v);
    }
#pragma unroll
    for (int k = 0; k < kFloorPer; ++k) {
        const int32_t blk = kc + 1 + int32_t(threadIdx.x) + k * kSerialNT;
        if (blk < a.NB) Fd[blk] = max64(fb_old[k], v);
    }
    __syncthreads();
    return v;
}

// LDS of the chain's workgroup beside the dynamic part.
struct ChainLds {
    int32_t tile_p[2][kSerialNT], tile_U[2][kSerialNT];   // arrivals of the current and next tile
    int64_t skey[kSerialWaves], scan_tmp[kSerialWaves], scan_tmp2[kSerialWaves];
    int32_t sd[kSerialWaves];
    int64_t speak;
    Capture cap;
};

// The new O values of a commit, and PF and SA on its range, fit 32 bits when
// its peak plus U does: O(t) + t <= PF(Uc) <= peak - p before it, plus p + t
// after it, and SA there is at most the larger of those and SA(Uc) <= peak.
__device__ inline int64_t commit_any(const CommitArgs& a, int32_t* stage, int64_t peak, int32_t bd, int64_t p,
                                     int32_t Uc, int32_t un, int32_t pre_d, PeakIn* cur, ChainLds& w) {
    if (peak + Uc < int64_t(INT32_MAX) && Uc < a.stage_cap)
        return commit_range<int32_t>(a, stage, bd, p, Uc, un, pre_d, cur, &w.cap, w.scan_tmp, w.scan_tmp2);
    return commit_range<int64_t>(a, nullptr, bd, p, Uc, un, pre_d, cur, &w.cap, w.scan_tmp, w.scan_tmp2);
}

// One workgroup for the chain from arrival `first` on (the queue lengths in Q
// and the capacities in C are ready).  kPre (D <= kSerialNT): thread d owns
// decoder d, and the next arrival's peak inputs are loaded while the current
// arrival is committed; only the committed decoder's inputs change, and its
// thread patches them from the values the commit captured.  Otherwise every
// thread evaluates its decoders d, d + kSerialNT, ... after each commit.
template <bool kPre>
__device__ inline void serial_chain(const CommitArgs& a, int64_t first, int32_t* Q, int32_t* C, int32_t* ostage,
                                    ChainLds& w) {
    auto& tile_p = w.tile_p;
    auto& tile_U = w.tile_U;
    auto& skey = w.skey;
    auto& sd = w.sd;
    auto& speak = w.speak;
    auto& cap = w.cap;
    const int32_t D = a.S.D, L = a.L, T = L - 1;
    const int tid = threadIdx.x;
    auto stage = [&](int64_t tile) {   // arrivals of `tile` into its buffer
        const int64_t j = tile * kSerialNT + tid;
        tile_p[tile & 1][tid] = j < a.A ? a.ap[j] : 0;
        tile_U[tile & 1][tid] = j < a.A ? a.aU[j] : -1;
    };
    stage(first / kSerialNT);
    if (first % kSerialNT != 0) stage(first / kSerialNT + 1);
    __syncthreads();
    PeakIn cur{0, 0, 0};
    int64_t have = -1;   // the arrival whose inputs `cur` holds
    for (int64_t i = first; i < a.A; ++i) {
        // the next tile is staged at the first arrival of a tile; the
        // barriers of that arrival precede every read of it
        if (i % kSerialNT == 0) stage(i / kSerialNT + 1);
        // uniform values read from LDS, made scalar so that every address derived from them is
        const int32_t p0 = __builtin_amdgcn_readfirstlane(tile_p[(i / kSerialNT) & 1][i % kSerialNT]);
        const int32_t U = __builtin_amdgcn_readfirstlane(tile_U[(i / kSerialNT) & 1][i % kSerialNT]);
        if (U < 0) {   // no bound: round robin, the request only joins the queue
            if (tid == 0) {
                const int32_t d = int32_t((a.rr_offset + i) % D);
                a.choice[i] = d;
                a.chosen_peak[i] = -1;
                a.chosen_over[i] = 0;
                a.flags[i] = 2;
                Q[d] += 1;
            }
            lds_barrier();
            continue;
        }
        if (tid == 0) {
            if (p0 < 0) raise_error(a.dev_err, MAPS_ERR_NEG_LEN);
            if (U > T) raise_error(a.dev_err, MAPS_ERR_BOUND_RANGE);
        }
        const int64_t p = p0 < 0 ? 0 : p0;
        const int32_t Uc = U < T ? U : T;
        // every decoder's peak with this arrival, and the thread's best key
        int64_t key = INT64_MAX, peak_best = 0;
        int32_t best = INT32_MAX;
        if constexpr (kPre) {
            if (tid < D) {
                if (have != i) cur = peak_load(a, tid, Uc);
                key = commit_key(cur, p, C[tid], Q[tid], a.policy, &peak_best);
                best = tid;
            }
        } else {
            for (int32_t d = tid; d < D; d += kSerialNT) {
                int64_t pk;
                const int64_t k = commit_key(peak_load(a, d, Uc), p, C[d], Q[d], a.policy, &pk);
                if (k < key) { key = k; best = d; peak_best = pk; }
            }
        }
        int64_t bkey = key;
        int32_t bd = best;
        block_argmin(bkey, bd, skey, sd);
        bd = __builtin_amdgcn_readfirstlane(bd);
        if (bd < 0 || bd >= D) bd = 0;   // unreachable with D >= 1; keeps every index in range
        if (best == bd && bd != INT32_MAX) speak = peak_best;   // the owner of the chosen decoder
        lds_barrier();
        const int64_t peak = speak;
        if (tid == 0) {
            const int64_t over = peak - C[bd];
            a.choice[i] = bd;
            a.chosen_peak[i] = peak;
            a.chosen_over[i] = over > 0 ? over : 0;
            a.flags[i] = over <= 0 ? 1 : 0;
            Q[bd] += 1;
        }
        // the next arrival's step, when it has a bound: its inputs go out with the commit's loads
        int32_t un = -1;
        if constexpr (kPre) {
            const int64_t j = i + 1;
            const int32_t Un =
                j < a.A ? __builtin_amdgcn_readfirstlane(tile_U[(j / kSerialNT) & 1][j % kSerialNT]) : -1;
            if (Un >= 0) un = Un < T ? Un : T;
        }
        const int32_t pre_d = kPre && tid < D ? tid : -1;
        const int64_t v = commit_any(a, ostage, peak, bd, p, Uc, un, pre_d, &cur, w);
        if constexpr (kPre) {
            if (un >= 0) {
                if (tid < D) {
                    if (tid == bd) {   // rewritten on [0, Uc] (SA below Uc); above Uc, v is a floor
                        if (un <= Uc) cur.pf = cap.pf;
                        else cur.fl = max64(cur.fl, v);
                        if (un < Uc) cur.sa = cap.sa;
                    }
                }
                have = i + 1;
            }
        }
    }
    if (a.queue_out)
        for (int32_t d = tid; d < D; d += kSerialNT) a.queue_out[d] = Q[d];
}

// The chain over the whole batch, or from where the rounds ended.
template <bool kPre>
__global__ __launch_bounds__(kSerialNT) void commit_serial(CommitArgs a) {
    extern __shared__ __align__(16) int32_t lds[];   // [D] queue lengths, [D] capacities, the stage
    __shared__ ChainLds w;
    const int32_t D = a.S.D;
    int32_t* Q = lds;
    int32_t* C = lds + D;
    bool neg = false;
    for (int32_t d = threadIdx.x; d < D; d += kSerialNT) {
        Q[d] = a.qlen[d];
        C[d] = a.cap[d];
        neg |= Q[d] < 0 || C[d] < 0;
        if (a.owners > 0 && a.ctl->resume > 0) Q[d] = a.ctl->queue[d];
    }
    if (neg) raise_error(a.dev_err, MAPS_ERR_NEG_LEN);
    serial_chain<kPre>(a, a.owners > 0 ? a.ctl->resume : 0, Q, C, lds + 2 * D, w);
}

// ---------------------------------------------------------------------------
// Rounds of arrivals with their commits in parallel (policy MQ)
// ---------------------------------------------------------------------------
//
// With feasible decoders an arrival takes the first of them in (queue length,
// index) order, and a commit only makes its decoder worse: a longer queue and
// higher peaks.  So against the curves as they stand at the start of a round,
// arrivals in order can each take their first feasible decoder until one meets
// a decoder taken earlier in the round (which needs that decoder's new curve,
// unless the old one did not hold the arrival either: then the new one does
// not): up to there every choice is the serial one, the decoders are distinct,
// and their commits run in parallel.  An arrival that no decoder holds takes
// the smallest overflow, which is known exactly for the first of a round.
// A round is about one level of the queue lengths: 4,096 arrivals on 256
// decoders with queues of 0..63 take about 60 rounds.
//
// Each decoder belongs to one owner workgroup (they are dealt in turn to those
// that have checked in), which keeps its curves in the L2 of its XCD: it evaluates the window of the next 128 arrivals against them
// (a bit each), and commits what the round gives its decoders.  Workgroup 0,
// the master, matches the window in one wavefront (decoder lane + 64 s in slot
// s).  Only the bits and the matches pass between them, by device-coherent
// stores followed by a round number; the curves never leave their XCD.
//
// The master starts the rounds when every owner has checked in, or after
// kCheckIn with those that have (workgroups of other kernels hold the other
// compute units; who comes later leaves at once), if they are two or more and
// one for 64 decoders.  1,024 arrivals: 7.7 ms in the serial chain on 256
// decoders, 7.1 / 4.4 / 2.3 / 1.8 ms with 2 / 4 / 16 / 255 owners; 11.7 ms
// on 1,000 decoders, 16.8 / 11.4 / 6.6 ms with 8 / 16 / 255.  The rounds also
// end when they hold too few arrivals to pay (no decoder is feasible any more,
// and commits do not make any feasible again).  The serial chain's launch takes
// up what is left.
//
// Every wait is bounded, and one that expires costs time but no arrival: two
// words change by compare-and-swap only, so that everyone agrees on what they
// hold.  `entry` goes to kRun or to kDeclined once: an owner that stops waiting
// for the master declines the rounds for all, or finds that they run and joins
// them.  `round` is that of the next round, or gets kEnded once: an owner that stops waiting
// for a round, and a master that stops waiting for an owner, end the rounds
// after the last one published, whose commits every owner still makes (the
// exchange of a round is written only when all have read the one before).  The
// serial chain goes on after that round.
// 4,096 arrivals on 256 decoders (queues of 0..63, bounds of 3,600 steps on
// average, 32,768 at most), nearly all feasible: 49 ms in the serial chain
// before, 3.7 ms with the rounds and the commits by rows.
constexpr int kReviewRounds = 8;             // rounds after which the master looks at what they held
constexpr uint32_t kCheckIn = 20000;         // 200 us at the 100 MHz of the constant clock
constexpr uint32_t kOwnerDecoders = 64;      // the most an owner takes
constexpr uint32_t kMostPolls = 1u << 22;    // an owner or the master that is not heard of for seconds

template <typename T>
__device__ inline T co_load(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void co_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// *p goes from `from` to `to`; returns what it held before.
template <typename T>
__device__ inline T co_swap(T* p, T from, T to) {
    __hip_atomic_compare_exchange_strong(p, &from, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return from;
}
// Every store of this wavefront has reached memory, and none of its later
// accesses is issued before.
__device__ inline void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// What an owner's first thread learned, for the others.
struct Published {
    int32_t own, owners;
    uint64_t round;   // the round's word, or the last one before it
};

// The check-in of an owner (one thread): its place among the owners, or -1
// where the rounds do not run or began without it.
__device__ inline int32_t owner_enters(const CommitArgs& a) {
    uint32_t e = __hip_atomic_fetch_add(&a.ctl->entry, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((e & (kRun | kDeclined)) != 0) return -1;
    const int32_t own = int32_t(e);
    for (uint32_t i = 0; i < a.waits.entry_polls && (e & (kRun | kDeclined)) == 0; ++i) {
        __builtin_amdgcn_s_sleep(4);
        e = co_load(&a.ctl->entry);
    }
    // not decided for seconds: decline (a swap fails only when another owner
    // checks in or the word is decided)
    while ((e & (kRun | kDeclined)) == 0) {
        const uint32_t held = co_swap(&a.ctl->entry, e, e | kDeclined);
        e = held == e ? e | kDeclined : held;
    }
    asm volatile("" ::: "memory");
    return (e & kRun) != 0 ? own : -1;
}

// Waits for the round after the word `last` (one thread of an owner): its word,
// or `last` where the rounds have ended before it.
__device__ inline uint64_t owner_waits(const CommitArgs& a, uint64_t last) {
    uint64_t seen = co_load(&a.ctl->round);
    for (uint32_t i = 0; i < a.waits.owner_polls && seen == last; ++i) {
        __builtin_amdgcn_s_sleep(2);
        seen = co_load(&a.ctl->round);
    }
    if (seen == last) seen = co_swap(&a.ctl->round, last, last | kEnded);   // not heard of for seconds: end there
    return seen & ~kEnded;
}

__device__ inline void owner_rounds(const CommitArgs& a, int32_t* ostage, ChainLds& w, Published& pub) {
    const int tid = threadIdx.x, lane = tid % kWave;
    const int32_t D = a.S.D, T = a.L - 1;
    if (tid == 0) {
        pub.own = owner_enters(a);
        pub.owners = int32_t(co_load(&a.ctl->owners));
    }
    __syncthreads();
    const int32_t own = __builtin_amdgcn_readfirstlane(pub.own);   // decoders own, own + P, ...
    const int32_t P = __builtin_amdgcn_readfirstlane(pub.owners);
    if (own < 0 || own >= P) return;
    int64_t pos = 0;
    uint64_t last = 0;
    for (uint32_t round = 1;; ++round) {
        // the window against this owner's decoders: kSerialNT / kWindow of them at a time
        constexpr int kTogether = kSerialNT / kWindow;
        const int j = tid % kWindow;
        const int64_t i = pos + j;
        const int32_t U = i < a.A ? a.aU[i] : -1, p0 = i < a.A ? a.ap[i] : 0;
        const int32_t Uc = U < T ? U : T;
        const int64_t p = p0 < 0 ? 0 : p0;
        // the window's first arrival with a bound: in the first half, else in the second
        if (tid < kWindow) w.skey[tid / kWave] = int64_t(__builtin_amdgcn_ballot_w64(U >= 0));
        __syncthreads();
        const uint64_t b0 = uint64_t(w.skey[0]), b1 = uint64_t(w.skey[1]);
        const int j0 = b0 != 0 ? __ffsll((unsigned long long)b0) - 1
                               : b1 != 0 ? kWave + __ffsll((unsigned long long)b1) - 1 : -1;
        for (int32_t k = tid / kWindow; own + int64_t(k) * P < D; k += kTogether) {
            const int32_t d = own + k * P;
            bool holds = false;
            if (U >= 0) {
                const PeakIn in = peak_load(a, d, Uc);
                const int64_t over = max64(p + max64(in.pf, in.fl), in.sa) - a.cap[d];
                holds = over <= 0;
                if (j == j0) co_store(&a.ctl->over[d], over);
            }
            const uint64_t bits = __builtin_amdgcn_ballot_w64(holds);
            if (lane == 0) co_store(&a.ctl->feasible[d][j / kWave], bits);
        }
        stores_done();
        __syncthreads();
        if (tid == 0) {
            co_store(&a.ctl->ready[own], round);
            pub.round = owner_waits(a, last);
            asm volatile("" ::: "memory");
        }
        __syncthreads();
        if (pub.round == last) return;   // the rounds have ended before this one
        last = pub.round;
        for (int32_t d = own; d < D; d += P) {
            const int32_t at = __builtin_amdgcn_readfirstlane(co_load(&a.ctl->assign[d]));
            if (at < 0 || at >= kWindow || pos + at >= a.A) continue;
            const int64_t i = pos + at;
            const int32_t p0 = a.ap[i], U = a.aU[i], C = a.cap[d];
            if (tid == 0) {
                if (p0 < 0) raise_error(a.dev_err, MAPS_ERR_NEG_LEN);
                if (U > T) raise_error(a.dev_err, MAPS_ERR_BOUND_RANGE);
            }
            const int64_t p = p0 < 0 ? 0 : p0;
            const int32_t Uc = __builtin_amdgcn_readfirstlane(U < 0 ? 0 : U < T ? U : T);
            const PeakIn in = peak_load(a, d, Uc);
            const int64_t peak = max64(p + max64(in.pf, in.fl), in.sa);
            if (tid == 0) {
                const int64_t over = peak - C;
                a.choice[i] = d;
                a.chosen_peak[i] = peak;
                a.chosen_over[i] = over > 0 ? over : 0;
                a.flags[i] = over <= 0 ? 1 : 0;
            }
            __syncthreads();   // every thread has read the curves that the commit rewrites
            PeakIn unused{0, 0, 0};
            commit_any(a, ostage, peak, d, p, Uc, -1, -1, &unused, w);   // ends with a barrier
        }
        if ((uint32_t(last) & kMore) == 0u) return;
        pos += uint32_t(last) & ~kMore;
    }
}

// The master's rounds by one wavefront.
template <int kSlots>
__device__ inline void master_rounds(const CommitArgs& a) {
    const int lane = threadIdx.x;
    const int32_t D = a.S.D;
    // packed keys (Q << 10) | decoder: every queue stays in [0, 2^21)
    bool wide = false;
    uint32_t K[kSlots];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        const int32_t d = lane + s * kWave;
        const int32_t q = d < D ? a.qlen[d] : 0;
        wide |= q < 0 || q + a.A >= (1 << 21);
        K[s] = d < D ? (uint32_t(q) << 10) | uint32_t(d) : ~0u;
    }
    bool run = __builtin_amdgcn_ballot_w64(wide) == 0;
    uint32_t e = 0;
    if (lane == 0) {
        e = co_load(&a.ctl->entry);
        if (run) {
            const uint64_t t0 = wall_clock64();
            while (e < uint32_t(a.owners) && wall_clock64() - t0 < a.waits.check_in) {   // kDeclined is above every count
                __builtin_amdgcn_s_sleep(4);
                e = co_load(&a.ctl->entry);
            }
        }
        while ((e & (kRun | kDeclined)) == 0) {
            co_store(&a.ctl->owners, e);
            stores_done();
            const uint32_t to = e | (run && e >= 2u && e * kOwnerDecoders >= uint32_t(D) ? kRun : kDeclined);
            const uint32_t held = co_swap(&a.ctl->entry, e, to);
            e = held == e ? to : held;
        }
    }
    e = __builtin_amdgcn_readfirstlane(e);
    if ((e & kRun) == 0) return;   // ctl->resume stays 0
    const int32_t P = int32_t(e & kOwnerCount);

    int64_t pos = 0, pos0 = 0;   // the first arrival after the rounds so far, and before the last of them
    uint32_t K0[kSlots];         // the queues before the last round
    uint64_t word = 0, word0 = 0, swapped = 0;   // the last round's, the one before, and what its publication found
#pragma unroll
    for (int s = 0; s < kSlots; ++s) K0[s] = K[s];
    // an owner has ended the rounds before the last one, which is void then
    auto void_last = [&]() {
        if (__builtin_amdgcn_ballot_w64(lane == 0 && swapped != word0) == 0) return false;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) K[s] = K0[s];
        pos = pos0;
        return true;
    };
    int held = 0;   // arrivals placed since the last review
    bool few = false;
    for (uint32_t round = 1;; ++round) {
        // every owner has evaluated the window
        bool late = false;
        uint32_t heard = co_load(&a.ctl->ready[lane < P ? lane : 0]);
        // looked at with a load in flight behind it: waiting for the swap at
        // once took 0.7 us a round
        if (round > 1 && void_last()) break;
        for (int32_t o = lane; o - lane < P && !late; o += kWave) {
            if (o != lane) heard = co_load(&a.ctl->ready[o < P ? o : 0]);
            uint32_t n = 0;
            while (__builtin_amdgcn_ballot_w64(o < P && heard < round) != 0) {
                if (++n > a.waits.master_polls) { late = true; break; }
                heard = co_load(&a.ctl->ready[o < P ? o : 0]);
            }
        }
        if (late) {   // end after the round before; an owner may have done so already
            if (lane == 0) (void)co_swap(&a.ctl->round, word, word | kEnded);
            break;
        }
        asm volatile("" ::: "memory");
        uint32_t bits[kSlots][2 * kMaskWords];
        uint64_t taken[kSlots];
        int32_t mine[kSlots];   // the arrival assigned to this lane's decoder
        pos0 = pos;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            K0[s] = K[s];
            const int32_t d = lane + s * kWave;
#pragma unroll
            for (int h = 0; h < kMaskWords; ++h) {
                const uint64_t m = d < D ? co_load(&a.ctl->feasible[d][h]) : 0;
                bits[s][2 * h] = uint32_t(m);
                bits[s][2 * h + 1] = uint32_t(m >> 32);
            }
            taken[s] = 0;
            mine[s] = -1;
        }
        const int32_t U0 = pos + lane < a.A ? a.aU[pos + lane] : 0;
        const int32_t U1 = pos + kWave + lane < a.A ? a.aU[pos + kWave + lane] : 0;
        const uint64_t none[2] = {__builtin_amdgcn_ballot_w64(U0 < 0), __builtin_amdgcn_ballot_w64(U1 < 0)};
        const int cnt = a.A - pos < kWindow ? int(a.A - pos) : kWindow;
        int done = 0;
        bool first = true, stop = false;
        if (round == 1) {
            // fewer than half of the window's arrivals find a decoder: the chain is better off from the start
            int held_by_any = 0;
#pragma unroll
            for (int word = 0; word < 2 * kMaskWords; ++word) {
                uint32_t m = 0;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) m |= bits[s][word];
                held_by_any += __popc(wave_last(wave_incl_scan(m, 0u, [](uint32_t x, uint32_t y) { return x | y; })));
            }
            const int bounded = cnt - __popcll(none[0]) - __popcll(none[1]);
            few = 2 * held_by_any < bounded;
            stop |= few;
        }
        auto take = [&](int32_t d, int j) {   // decoder d (uniform) takes the window's arrival j
#pragma unroll
            for (int s = 0; s < kSlots; ++s) {
                const bool own = lane + s * kWave == d;
                K[s] += own ? 1024u : 0u;
                mine[s] = own ? j : mine[s];
                taken[s] |= d / kWave == s ? 1ull << (d % kWave) : 0ull;
            }
        };
#pragma unroll
        for (int word = 0; word < 2 * kMaskWords; ++word) {
            for (int jj = 0; jj < 32 && !stop; ++jj) {
                const int j = word * 32 + jj;
                if (j >= cnt) break;
                if ((none[word / 2] >> (j % kWave)) & 1) {   // round robin: the request only joins the queue
                    const int32_t d = int32_t((a.rr_offset + pos + j) % D);
#pragma unroll
                    for (int s = 0; s < kSlots; ++s) K[s] += lane + s * kWave == d ? 1024u : 0u;
                    if (lane == 0) {
                        a.choice[pos + j] = d;
                        a.chosen_peak[pos + j] = -1;
                        a.chosen_over[pos + j] = 0;
                        a.flags[pos + j] = 2;
                    }
                    done = j + 1;
                    continue;
                }
                uint32_t k = ~0u;
#pragma unroll
                for (int s = 0; s < kSlots; ++s) {
                    const uint32_t k1 = (bits[s][word] >> jj) & 1u ? K[s] : ~0u;
                    k = k1 < k ? k1 : k;
                }
                k = wave_last(wave_incl_scan(k, ~0u, [](uint32_t x, uint32_t y) { return x < y ? x : y; }));
                int32_t d;
                if (k != ~0u) {
                    d = int32_t(k & 1023u);
                    uint64_t t = 0;
#pragma unroll
                    for (int s = 0; s < kSlots; ++s) t = d / kWave == s ? taken[s] : t;
                    if ((t >> (d % kWave)) & 1) { stop = true; break; }   // its new curve decides
                } else {
                    if (!first) { stop = true; break; }   // the overflows are those of the first
                    int64_t least = INT64_MAX, over[kSlots];
#pragma unroll
                    for (int s = 0; s < kSlots; ++s) {
                        over[s] = lane + s * kWave < D ? co_load(&a.ctl->over[lane + s * kWave]) : INT64_MAX;
                        least = over[s] < least ? over[s] : least;
                    }
                    least = wave_last(wave_incl_scan(least, INT64_MAX, [](int64_t x, int64_t y) { return x < y ? x : y; }));
                    d = 0;
#pragma unroll
                    for (int s = kSlots - 1; s >= 0; --s) {
                        const uint64_t at = __builtin_amdgcn_ballot_w64(over[s] == least);
                        d = at != 0 ? s * kWave + __ffsll((unsigned long long)at) - 1 : d;
                    }
                }
                first = false;
                take(d, j);
                done = j + 1;
            }
        }
        held += done;
        bool more = pos + done < a.A && !few;
        if (more && round % kReviewRounds == 0) {
            more = held >= kReviewRounds + kReviewRounds / 2;
            held = 0;
        }
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
            if (lane + s * kWave < D) co_store(&a.ctl->assign[lane + s * kWave], mine[s]);
        stores_done();
        word0 = word;
        word = round_word(round, uint32_t(done), more);
        if (lane == 0) swapped = co_swap(&a.ctl->round, word0, word);
        pos += done;
        if (!more) {
            (void)void_last();
            break;
        }
    }
    if (lane == 0) a.ctl->resume = pos;
#pragma unroll
    for (int s = 0; s < kSlots; ++s)
        if (lane + s * kWave < D) a.ctl->queue[lane + s * kWave] = int32_t(K[s] >> 10);
}

template <int kSlots>
__global__ __launch_bounds__(kSerialNT) void commit_rounds(CommitArgs a) {
    extern __shared__ __align__(16) int32_t lds[];   // an owner's stage, placed as in commit_serial
    __shared__ ChainLds w;
    __shared__ Published pub;
    if (blockIdx.x != 0) owner_rounds(a, lds + 2 * a.S.D, w, pub);
    else if (threadIdx.x < kWave) master_rounds<kSlots>(a);
}

}  // namespace
}  // namespace maps

using namespace maps;

extern "C" size_t maps_place_commit_workspace_size(int32_t D, int32_t u_max) {
    if (D < 1 || D > MAPS_MAX_COMMIT_DECODERS || u_max < 0 || u_max > MAPS_MAX_COMMIT_U_MAX) return 0;
    return commit_layout(D, u_max).bytes;
}

extern "C" maps_status maps_internal_place_commit(const void* snapshot, int32_t D, int32_t u_max,
                                                  const int32_t* capacity, const int32_t* queue_len,
                                                  const int32_t* a_prompt, const int32_t* a_upper, int64_t A,
                                                  int32_t policy, int64_t rr_offset, int32_t* choice,
                                                  int64_t* chosen_peak, int64_t* chosen_overflow, uint8_t* flags,
                                                  int32_t* queue_out, uint32_t* dev_err, void* workspace,
                                                  size_t workspace_bytes, hipStream_t stream, CommitWaits waits) {
    if (D < 1 || D > MAPS_MAX_COMMIT_DECODERS || A < 0 || rr_offset < 0 || u_max < 0 ||
        u_max > MAPS_MAX_COMMIT_U_MAX)
        return MAPS_E_SIZE;
    if (policy != MAPS_POLICY_MQ && policy != MAPS_POLICY_MC) return MAPS_E_POLICY;
    if (!snapshot || !capacity || !queue_len || !dev_err || !workspace ||
        (A > 0 && (!a_prompt || !a_upper || !choice || !chosen_peak || !chosen_overflow || !flags)))
        return MAPS_E_NULL;
    const CommitLayout c = commit_layout(D, u_max);
    if (workspace_bytes < c.bytes) return MAPS_E_WORKSPACE;
    char* w = static_cast<char*>(workspace);
    CommitArgs a{};
    a.S = snap_layout(D, 0, u_max);   // region offsets do not depend on the resident count
    a.snap = snapshot;
    a.O = reinterpret_cast<int64_t*>(w + c.off_O);
    a.PF = reinterpret_cast<int64_t*>(w + c.off_PF);
    a.SA = reinterpret_cast<int64_t*>(w + c.off_SA);
    a.F = reinterpret_cast<int64_t*>(w + c.off_F);
    a.L = c.L;
    a.NB = c.NB;
    a.cap = capacity;
    a.qlen = queue_len;
    a.ap = a_prompt;
    a.aU = a_upper;
    a.A = A;
    a.policy = policy;
    a.rr_offset = rr_offset;
    a.choice = choice;
    a.chosen_peak = chosen_peak;
    a.chosen_over = chosen_overflow;
    a.flags = flags;
    a.queue_out = queue_out;
    a.dev_err = dev_err;
    a.ctl = reinterpret_cast<RoundControl*>(w + c.off_ctl);
    a.waits = waits;
    // Rounds where arrivals can find different feasible decoders, from 8
    // arrivals on (starting the owners costs about one serial arrival); the
    // master and the owners fill a compute unit each.
    const int cus = device_compute_units();
    const bool rounds = policy == MAPS_POLICY_MQ && D >= 3 && D <= kRoundDecoders && A >= 8 && cus >= 4;
    a.owners = rounds ? (D < cus - 1 ? D : cus - 1) : 0;
    if (a.owners > kMaxOwners) a.owners = kMaxOwners;
    auto serial = D <= kSerialNT ? commit_serial<true> : commit_serial<false>;
    // The master walks its slots at every arrival: as few as hold the decoders
    // (1,024 arrivals on 257 decoders 1.85 ms with 8 slots, 2.40 with 16; on 16
    // decoders 2.26 ms with 1 slot, 2.40 with 4).
    auto round = D <= 1 * kWave   ? commit_rounds<1>
                 : D <= 2 * kWave ? commit_rounds<2>
                 : D <= 4 * kWave ? commit_rounds<4>
                 : D <= 8 * kWave ? commit_rounds<8>
                                  : commit_rounds<kRoundDecoders / kWave>;
    // dynamic LDS of the chain: queue lengths and capacities, then as many
    // staged range entries as the workgroup's LDS holds beside the kernel's
    // static LDS (less 256 bytes for the alignment of the dynamic part)
    const size_t qc = size_t(2) * D * sizeof(int32_t);   // a multiple of 8 bytes
    size_t fixed = kernel_static_lds(serial);
    if (rounds && kernel_static_lds(round) > fixed) fixed = kernel_static_lds(round);
    fixed += qc + 256;
    if (fixed > kLdsPerWorkgroup) return MAPS_E_SIZE;   // unreachable with D <= MAPS_MAX_COMMIT_DECODERS
    a.stage_cap = int32_t((kLdsPerWorkgroup - fixed) / sizeof(int32_t));
    const size_t lds = qc + size_t(a.stage_cap) * sizeof(int32_t);
    hipLaunchKernelGGL(commit_init, dim3(unsigned(D)), dim3(kCommitNT), 0, stream, a);
    MAPS_CHECK_LAUNCH();
    if (rounds) {
        allow_dynamic_lds(round, lds);
        hipLaunchKernelGGL(round, dim3(unsigned(1 + a.owners)), dim3(kSerialNT), lds, stream, a);
        MAPS_CHECK_LAUNCH();
    }
    allow_dynamic_lds(serial, lds);
    hipLaunchKernelGGL(serial, dim3(1), dim3(kSerialNT), lds, stream, a);
    MAPS_CHECK_LAUNCH();
    return MAPS_OK;
}

extern "C" maps_status maps_place_commit(const void* snapshot, int32_t D, int32_t u_max, const int32_t* capacity,
                                         const int32_t* queue_len, const int32_t* a_prompt, const int32_t* a_upper,
                                         int64_t A, int32_t policy, int64_t rr_offset, int32_t* choice,
                                         int64_t* chosen_peak, int64_t* chosen_overflow, uint8_t* flags,
                                         int32_t* queue_out, uint32_t* dev_err, void* workspace,
                                         size_t workspace_bytes, hipStream_t stream) {
    return maps_internal_place_commit(snapshot, D, u_max, capacity, queue_len, a_prompt, a_upper, A, policy, rr_offset,
                                      choice, chosen_peak, chosen_overflow, flags, queue_out, dev_err, workspace,
                                      workspace_bytes, stream, CommitWaits{kCheckIn, kMostPolls, kMostPolls, kMostPolls});
}
