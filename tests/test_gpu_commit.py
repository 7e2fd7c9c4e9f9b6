"""Placement with sequential commit on the GPU (maps_place_commit) against
the CPU oracle, bit for bit: arrivals in order, each committed to its
decoder's projected occupancy and queue before the next (Sec. 3.3, Algorithm
1).  Random ragged decoders and arrival mixes, both policies, round-robin
arrivals, capacity ties, the seeded workloads (literal and with room), the
single-arrival case against maps_place, and the device error bits."""
import ctypes

import numpy as np
import pytest

import oracle
import workload
from tests.gpu_common import assert_same, fit_capacity, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    return oracle.Oracle()


def _cuda(x, dtype=np.int32):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, dtype=dtype)).cuda()


class Waits(ctypes.Structure):
    """Of the rounds: ticks of the 100 MHz clock for all owners to check in, and polls of an owner for
    that decision, of an owner for a round and of the master for the owners."""
    _fields_ = [(n, ctypes.c_uint32) for n in ("check_in", "entry_polls", "owner_polls", "master_polls")]


MOST = 1 << 22
PATIENT = (10**8, MOST, MOST, MOST)   # a second for the check-in, whatever else the card is busy with
RUN, DECLINED = 1 << 30, 1 << 31      # of the entry word


def _exchange(ws, D, u_max):
    """The entry word, the owners of the rounds and the first arrival left to the serial chain, from the
    exchange behind the curves (three of u_max + 1 int64 a decoder) and the floors (one int64 per 1,024 steps)."""
    a = lambda x: (x + 255) // 256 * 256  # noqa: E731
    at = 3 * a(8 * D * (u_max + 1)) + a(8 * D * (u_max // 1024 + 1))
    words = ws[at:at + 24].cpu().numpy()
    entry, owners = words[8:16].view(np.uint32)
    return int(entry), int(owners), int(words[16:].view(np.int64)[0])


def _gpu(seg, p, g, U, u_max, cap, Q, a_p, a_U, policy=0, rr=0, waits=None):
    """maps_place_commit's outputs, and the exchange of its rounds; waits: through the internal entry."""
    import torch

    import paper_2609_15359_amd as maps
    D, A = len(cap), len(a_p)
    snap, _, err = maps.project(_cuda(seg, np.int64), _cuda(p), _cuda(g), _cuda(U), u_max)
    ws = torch.zeros(maps.place_commit_workspace_bytes(D, u_max), dtype=torch.uint8, device="cuda")
    args = _cuda(cap), _cuda(Q), _cuda(a_p), _cuda(a_U)
    if waits is None:
        out = maps.place_commit(snap, *args, policy, rr, dev_err=err, workspace=ws)
    else:
        new = lambda n, t: torch.empty(n, dtype=t, device="cuda")  # noqa: E731
        out = maps.CommitPlacement(choice=new(A, torch.int32), chosen_peak=new(A, torch.int64),
                                   chosen_overflow=new(A, torch.int64), flags=new(A, torch.uint8),
                                   queue_out=new(D, torch.int32), dev_err=err)
        fn = maps.library().maps_internal_place_commit
        fn.restype, fn.argtypes = ctypes.c_int32, maps.library().maps_place_commit.argtypes + [Waits]
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
        st = fn(ptr(snap.data), D, u_max, *(ptr(t) for t in args), A, policy, rr, ptr(out.choice),
                ptr(out.chosen_peak), ptr(out.chosen_overflow), ptr(out.flags), ptr(out.queue_out), ptr(err),
                ptr(ws), ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), Waits(*waits))
        assert st == 0
    torch.cuda.synchronize()
    entry, owners, resume = _exchange(ws, D, u_max)
    return dict(choice=out.choice.cpu().numpy(), chosen_peak=out.chosen_peak.cpu().numpy(),
                chosen_overflow=out.chosen_overflow.cpu().numpy(), flags=out.flags.cpu().numpy(),
                queue_out=out.queue_out.cpu().numpy(), err=int(err.item()) & 0xFFFFFFFF, entry=entry, owners=owners,
                resume=resume)


def _compare(g, r, q_after, tag):
    assert g["err"] == 0, tag
    for f in ("choice", "chosen_peak", "chosen_overflow", "flags"):
        assert_same(f"{tag} {f}", g[f], getattr(r, f))
    assert_same(f"{tag} queue_out", g["queue_out"], q_after)


def _random_case(rng, D, nmax, A, u_max):
    counts = rng.integers(0, nmax + 1, size=D)
    seg = np.zeros(D + 1, np.int64)
    seg[1:] = np.cumsum(counts)
    n = int(seg[-1])
    U = rng.integers(0, u_max + 1, size=n)
    g = rng.integers(0, u_max + 1, size=n)           # g may exceed U: remaining length 0
    p = rng.integers(0, 3000, size=n)
    a_p = rng.integers(0, 3000, size=A)
    a_U = np.where(rng.random(A) < 0.1, -1, rng.integers(0, u_max + 1, size=A))
    return seg, p, g, U, a_p, a_U


@pytest.mark.parametrize("D,nmax,A,u_max", [(1, 5, 40, 50), (3, 30, 300, 2000), (17, 200, 700, 9000),
                                            (64, 40, 2100, 1023), (300, 8, 900, 70),
                                            # ranges longer than the chain's LDS stage, many floor blocks
                                            (4, 60, 500, 40000),
                                            # more decoders than threads: no lookups ahead
                                            (1100, 3, 250, 2500),
                                            # the most decoders the chain takes: the smallest LDS stage
                                            (8192, 2, 60, 100)])
def test_random(orc, D, nmax, A, u_max):
    rng = np.random.default_rng(D * 1000 + A)
    seg, p, g, U, a_p, a_U = _random_case(rng, D, nmax, A, u_max)
    base = orc.project(seg, p, g, U)
    # capacities around the base peaks plus a few arrivals: both branches, and queue growth matters
    cap = (base + rng.integers(0, 4 * (3000 + u_max), size=D)).astype(np.int32)
    Q = rng.integers(0, 5, size=D)
    for policy in (0, 1):
        rr = int(rng.integers(0, 1000))
        r, q_after = orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, policy=policy, rr_offset=rr)
        got = _gpu(seg, p, g, U, u_max, cap, Q, a_p, a_U, policy, rr)
        _compare(got, r, q_after, f"D={D} A={A} policy={policy}")
        say(f"[commit] D={D} A={A} policy={policy}: feasible {np.mean(r.flags & 1):.3f}")


# (D, A, u_max): batches at the edges of the rounds' window of 128 arrivals, decoders at the edges of a
# wavefront's slots, one and several decoders an owner workgroup, and the most decoders the rounds take
@pytest.mark.parametrize("D,A,u_max", [(3, 8, 300), (3, 129, 300), (64, 127, 500), (65, 128, 500), (255, 640, 400),
                                       (256, 257, 400), (257, 900, 200), (600, 1500, 150), (1024, 2100, 100)])
@pytest.mark.parametrize("room", ["most", "half", "none", "long queues"])
def test_rounds(orc, D, A, u_max, room):
    """Rounds of parallel commits: decoders that hold nearly every arrival, about
    half of them and none (where the rounds give way to the serial chain), in
    batches with arrivals without a bound, past u_max's profile and with equal
    and unequal queues; and queues too long for the rounds."""
    rng = np.random.default_rng(D + A)
    seg, p, g, U, a_p, a_U = _random_case(rng, D, 12, A, u_max)
    base = orc.project(seg, p, g, U)
    demand = int((a_p + np.maximum(a_U, 0)).mean()) * max(1, A // D)
    share = {"most": 4 * demand, "half": demand, "none": 0, "long queues": demand}[room]
    cap = (base + rng.integers(0, share + 1, size=D)).astype(np.int32)
    Q = rng.integers(0, 7, size=D) + (2**21 - 5 if room == "long queues" else 0)
    rr = int(rng.integers(0, 2**40))
    r, q_after = orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, policy=0, rr_offset=rr)
    say(f"[commit] rounds D={D} A={A} {room}: feasible {np.mean(r.flags & 1):.3f}")
    got = _gpu(seg, p, g, U, u_max, cap, Q, a_p, a_U, 0, rr, waits=PATIENT)
    _compare(got, r, q_after, f"rounds D={D} A={A} {room}")
    say(f"[commit] rounds D={D} A={A} {room}: entry {got['entry']:#x}, {got['owners']} owners, serial from {got['resume']}")
    # who placed the arrivals: the rounds, the rounds until too few of a window fit, or the serial chain alone
    assert got["entry"] & (DECLINED if room == "long queues" else RUN)
    first, last = {"most": (A, A), "half": (1, A), "none": (0, 0), "long queues": (0, 0)}[room]
    assert first <= got["resume"] <= last


@pytest.mark.parametrize("waits", [(0, MOST, MOST, MOST), (10**8, 0, MOST, MOST), (10**8, MOST, 0, MOST),
                                   (10**8, MOST, 2, MOST), (10**8, MOST, 20, MOST), (10**8, MOST, 100, MOST),
                                   (10**8, MOST, MOST, 0), (10**8, MOST, MOST, 3), (10**8, MOST, MOST, 20),
                                   (10**8, MOST, MOST, 100), (10**8, MOST, 15, 15), (0, 0, 0, 0)])
def test_waits_that_expire(orc, waits):
    """Owners and a master that stop waiting, before the rounds and anywhere in them: every arrival is placed
    and no error raised, whoever gave up first."""
    for D, A, u_max in ((3, 300, 300), (65, 700, 9000), (300, 900, 2000)):
        rng = np.random.default_rng(D + A)
        seg, p, g, U, a_p, a_U = _random_case(rng, D, 12, A, u_max)
        base = orc.project(seg, p, g, U)
        demand = int((a_p + np.maximum(a_U, 0)).mean()) * max(1, A // D)
        cap = (base + rng.integers(0, 4 * demand + 1, size=D)).astype(np.int32)
        Q = rng.integers(0, 7, size=D)
        r, q_after = orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, policy=0, rr_offset=5)
        say(f"[commit] waits {waits} D={D} A={A}")
        got = _gpu(seg, p, g, U, u_max, cap, Q, a_p, a_U, 0, 5, waits=waits)
        _compare(got, r, q_after, f"waits {waits} D={D} A={A}")
        say(f"[commit] waits {waits} D={D} A={A}: the serial chain took up at {got['resume']}")
        assert 0 <= got["resume"] <= A and bool(got["entry"] & RUN) != bool(got["entry"] & DECLINED)


def test_rounds_without_a_compute_unit(orc):
    """A kernel of another stream holds a compute unit for longer than the owners have to check in: the rounds
    run with the others.  One simulation of 8 decoders takes 96 KB of its compute unit's LDS for some
    20 ms, so that an owner, which takes all of it, finds no place there."""
    import torch

    import paper_2609_15359_amd as maps
    D, A, u_max = 300, 900, 2000
    rng = np.random.default_rng(1)
    seg, p, g, U, a_p, a_U = _random_case(rng, D, 12, A, u_max)
    cap = (orc.project(seg, p, g, U) + 40000).astype(np.int32)
    Q = rng.integers(0, 7, size=D)
    r, q_after = orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, policy=0, rr_offset=5)
    n = 8000
    requests = [_cuda(rng.integers(lo, hi, size=n)) for lo, hi in ((1, 2000), (1, 800), (1, 800))]
    arrival = _cuda(np.sort(rng.integers(0, 60 * n, size=n))[None, :], np.int64)
    policy = _cuda([1])
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        sim = maps.simulate(8, 50000, 850000, arrival, *requests, policy)
    done = torch.cuda.Event()
    done.record(other)
    got = _gpu(seg, p, g, U, u_max, cap, Q, a_p, a_U, 0, 5)   # ends with a synchronize
    _compare(got, r, q_after, "a compute unit less")
    launched = min(D, torch.cuda.get_device_properties(0).multi_processor_count - 1)
    say(f"[commit] a compute unit less: {got['owners']} of {launched} owners, serial from {got['resume']}")
    assert got["entry"] & RUN and got["resume"] == A and 0 < got["owners"] < launched
    assert int(sim.dev_err.item()) == 0


def _two_batches(orc, seed):
    """Two batches for the rounds: inputs, and what the oracle makes of them."""
    out = []
    for D, A, u_max in ((300, 700, 2000), (65, 500, 3000)):
        rng = np.random.default_rng(seed + D)
        seg, p, g, U, a_p, a_U = _random_case(rng, D, 12, A, u_max)
        cap = (orc.project(seg, p, g, U) + rng.integers(0, 60000, size=D)).astype(np.int32)
        Q = rng.integers(0, 7, size=D)
        out.append(((seg, p, g, U, u_max, cap, Q, a_p, a_U), orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, rr_offset=3)))
    return out


class _Call:
    """maps.place_commit with its buffers, for calls on several streams and under capture."""

    def __init__(self, seg, p, g, U, u_max, cap, Q, a_p, a_U):
        import torch

        import paper_2609_15359_amd as maps
        self.snap, _, self.err = maps.project(_cuda(seg, np.int64), _cuda(p), _cuda(g), _cuda(U), u_max)
        self.args = [_cuda(cap), _cuda(Q), _cuda(a_p), _cuda(a_U)]
        self.ws = torch.empty(maps.place_commit_workspace_bytes(len(cap), u_max), dtype=torch.uint8, device="cuda")
        self.out = None
        self.place()

    def place(self):
        import paper_2609_15359_amd as maps
        self.out = maps.place_commit(self.snap, *self.args, 0, 3, dev_err=self.err, workspace=self.ws, out=self.out)

    def forget(self):
        for t in (self.out.choice, self.out.chosen_peak, self.out.chosen_overflow, self.out.queue_out):
            t.fill_(-7)
        self.out.flags.fill_(77)

    def check(self, want, tag):
        o = self.out
        _compare(dict(choice=o.choice.cpu().numpy(), chosen_peak=o.chosen_peak.cpu().numpy(),
                      chosen_overflow=o.chosen_overflow.cpu().numpy(), flags=o.flags.cpu().numpy(),
                      queue_out=o.queue_out.cpu().numpy(), err=int(self.err.item()) & 0xFFFFFFFF), *want, tag)


def test_two_streams(orc):
    """Two calls in flight on two streams, whose owners compete for the compute units."""
    import torch
    batches = _two_batches(orc, 40)
    calls, streams = [_Call(*b) for b, _ in batches], [torch.cuda.Stream() for _ in batches]
    for turn in range(4):
        for c in calls:
            c.forget()
        torch.cuda.synchronize()
        for c, s in list(zip(calls, streams))[:: 1 if turn % 2 else -1]:
            with torch.cuda.stream(s):
                c.place()
        torch.cuda.synchronize()
        for i, (c, (_, want)) in enumerate(zip(calls, batches)):
            c.check(want, f"two streams, turn {turn}, call {i}")


def test_capture_and_replay(orc):
    """A captured call, replayed on other arrivals, capacities and queues with eager work between the replays."""
    import torch
    (seg, p, g, U, u_max, cap, Q, a_p, a_U), _ = _two_batches(orc, 50)[0]
    call, stream = _Call(seg, p, g, U, u_max, cap, Q, a_p, a_U), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call.place()
    rng = np.random.default_rng(6)
    for turn in range(4):
        if turn:
            cap, Q = rng.permutation(cap), rng.permutation(Q)
            a_p, a_U = rng.permutation(a_p), rng.permutation(a_U)
        want = orc.place_commit(seg, p, g, U, cap, Q, a_p, a_U, rr_offset=3)
        for old, x in zip(call.args, (cap, Q, a_p, a_U)):
            old.copy_(_cuda(x))
        call.forget()
        graph.replay()
        torch.cuda.synchronize()
        call.check(want, f"replay, turn {turn}")
        call.forget()
        call.place()   # eager, on the same workspace
        torch.cuda.synchronize()
        call.check(want, f"eager, turn {turn}")


def test_ties_and_empty_decoders(orc):
    # identical decoders (every key ties: lowest index first, then queue growth spreads them), empty decoders
    D = 6
    seg = np.array([0, 2, 4, 4, 6, 8, 8], np.int64)
    p = np.array([10, 20] * 4)
    g = np.array([1, 2] * 4)
    U = np.array([5, 7] * 4)
    a_p = np.full(40, 3)
    a_U = np.full(40, 4)
    cap = np.full(D, 10**6)
    for policy in (0, 1):
        r, q_after = orc.place_commit(seg, p, g, U, cap, np.zeros(D), a_p, a_U, policy=policy)
        got = _gpu(seg, p, g, U, 16, cap, np.zeros(D), a_p, a_U, policy)
        _compare(got, r, q_after, f"ties policy={policy}")


def test_single_arrival_is_maps_place(orc):
    import torch

    import paper_2609_15359_amd as maps
    rng = np.random.default_rng(5)
    seg, p, g, U, a_p, a_U = _random_case(rng, 9, 50, 1, 3000)
    a_U[:] = 1234
    cap = rng.integers(0, 300000, size=9)
    Q = rng.integers(0, 4, size=9)
    got = _gpu(seg, p, g, U, 3000, cap, Q, a_p, a_U)
    snap, _, err = maps.project(_cuda(seg, np.int64), _cuda(p), _cuda(g), _cuda(U), 3000)
    pl = maps.place(snap, _cuda(cap), _cuda(Q), _cuda(a_p), _cuda(a_U), dev_err=err)
    torch.cuda.synchronize()
    assert int(got["choice"][0]) == int(pl.choice[0]) and int(got["chosen_peak"][0]) == int(pl.chosen_peak[0])
    assert int(got["flags"][0]) == int(pl.flags[0])


@pytest.mark.parametrize("name,arrivals", [("tiny", None), ("small", None), ("medium", 6000), ("large", 3000)])
def test_workload(orc, name, arrivals):
    """The seeded workloads (bounds from the oracle's calibration of the
    batch): literal capacities, where every decoder is overloaded and each
    arrival takes the largest slack, and capacities with room; medium and
    large on their first arrivals (the oracle derives a decoder's maxima over
    the whole step axis at every commit)."""
    b = workload.make(name)
    o = oracle.step(b, orc, want_pairs=False)
    U_res, U_arr, _ = b.split_bounds(o.U)
    k = b.arrivals if arrivals is None else arrivals
    ap, aU = b.arr_prompt[:k], U_arr[:k]
    fit = fit_capacity(b, {"U": o.U, "base_peak": o.base_peak})
    for tag, cap in (("literal", b.capacity), ("room", fit)):
        r, q_after = orc.place_commit(b.seg_off, b.res_prompt, b.res_gen, U_res, cap, b.queue_len, ap, aU,
                                      rr_offset=11)
        got = _gpu(b.seg_off, b.res_prompt, b.res_gen, U_res, b.u_max, cap, b.queue_len, ap, aU, 0, 11)
        _compare(got, r, q_after, f"{name} {tag}")
        say(f"[commit] {name} {tag}: {k} arrivals, feasible fraction {np.mean(r.flags & 1):.3f}")


def test_error_bits():
    seg = np.array([0, 2], np.int64)
    ok = _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [100], [0], [1, 2], [3, 4])
    assert ok["err"] == 0
    assert _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [100], [0], [-1, 2], [3, 4])["err"] & 1
    assert _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [100], [0], [-1, 2], [-1, 4])["err"] == 0   # no bound: RR
    assert _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [-100], [0], [1, 2], [3, 4])["err"] & 1
    assert _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [100], [-3], [1, 2], [3, 4])["err"] & 1
    assert _gpu(seg, [5, 1], [0, 0], [3, 3], 10, [100], [0], [1, 2], [3, 11])["err"] & 16


def test_snapshot_mismatch_is_reported():
    import torch

    import paper_2609_15359_amd as maps
    seg = np.array([0, 2], np.int64)
    snap, _, err = maps.project(_cuda(seg, np.int64), _cuda([5, 1]), _cuda([0, 0]), _cuda([3, 3]), 10)
    torch.cuda.synchronize()
    wrong = maps.Snapshot(data=snap.data, D=1, n_total=2, u_max=12)   # built for u_max 10
    e = maps.new_error_word()
    maps.place_commit(wrong, _cuda([100]), _cuda([0]), _cuda([1]), _cuda([3]), dev_err=e)
    torch.cuda.synchronize()
    assert int(e.item()) & 32
