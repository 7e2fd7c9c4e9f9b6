"""Admission in the local order (maps_local_order, maps_project_order) against
the CPU oracle, bit for bit, where the prefix search can go wrong: queue
lengths at the edges of the one-wavefront and one-key-per-thread forms, no,
some and only promoted requests and numbers of them at the edges of adding them
up, capacities from the base peak to past the
whole queue, and decoders whose events the projection keeps in LDS (with and
without a dense profile) or not."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    return oracle.Oracle()


def _cuda(x, dtype=np.int32):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, dtype=dtype)).cuda()


@pytest.mark.parametrize("u_max,residents", [(700, 300), (20000, 900), (20000, 9000)],
                         ids=["profile", "events-in-lds", "events-in-hbm"])
@pytest.mark.parametrize("promoted", [0.0, 0.1, 1.0, 47, 48, 49, 64, 65])
def test_admission(orc, u_max, residents, promoted):
    import torch

    import paper_2609_15359_amd as maps
    rng = np.random.default_rng(residents + int(10 * promoted))
    qlens = [0, 1, 2, 33, 63, 64, 65, 200, 1023, 1024, 1025, 2048]
    D = len(qlens)
    counts = rng.integers(residents // 2, residents + 1, size=D)
    counts[3] = 0
    counts[-1] = residents
    seg = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(seg[-1])
    p, g = rng.integers(0, 3000, size=n), rng.integers(0, u_max // 2, size=n)
    U = np.minimum(g + rng.integers(0, u_max, size=n), u_max)
    q_off = np.concatenate([[0], np.cumsum(qlens)]).astype(np.int64)
    nq = int(q_off[-1])
    q_p = rng.integers(0, 2000, size=nq)
    q_U = rng.integers(-1, u_max + 1, size=nq)
    q_U[rng.random(nq) < 0.3] = u_max // 3                  # runs of equal bounds
    wait = np.where(rng.random(nq) < promoted, 1000, 999)
    if promoted > 1:                                        # so many of each queue
        wait = np.concatenate([np.where(rng.permutation(k) < promoted, 1000, 999) for k in qlens])
    base = orc.project(seg, p, g, U)
    dev = [_cuda(x) for x in (p, g, U)]
    demand = np.array([(q_p[a:b] + np.maximum(q_U[a:b], 0)).sum() for a, b in zip(q_off, q_off[1:])])
    for share in (0.0, 0.02, 0.3, 0.7, 2.0):
        cap = np.minimum(base + (share * demand).astype(np.int64), 2**31 - 1).astype(np.int32)
        want_order, want_adm = orc.local_order(seg, p, g, U, cap, q_off, q_p, q_U, wait, 1000, u_max)
        say(f"[order] residents {residents} promoted {promoted} share {share}: {want_adm.tolist()}")
        args = (_cuda(cap), _cuda(q_off, np.int64), _cuda(q_p), _cuda(q_U), _cuda(wait), 1000)
        snap, b, order, adm, err = maps.project_order(_cuda(seg, np.int64), *dev, u_max, *args)
        order2, adm2, err2 = maps.local_order(snap, *args)
        torch.cuda.synchronize()
        assert int(err.item()) == 0 and int(err2.item()) == 0
        assert_same("base peak", b.cpu().numpy(), base)
        for tag, o, a in (("project_order", order, adm), ("local_order", order2, adm2)):
            assert_same(f"{tag} order", o.cpu().numpy(), want_order)
            assert_same(f"{tag} admitted", a.cpu().numpy(), want_adm)


@pytest.mark.parametrize("n,N,growth", [(65, 200, 1.1), (300, 200, 1.03), (2048, 1000, 1.003)])
def test_promoted_prefix_one_point_at_a_time(orc, n, N, growth):
    """Promoted requests of which each exceeds the room at its own bound, a little more than the one before
    it, beside N residents: a pass over the points lowers the prefix that may fit by one, unless it halves
    what is left.  The three take 10, 16 and 21 passes."""
    import torch

    import paper_2609_15359_amd as maps
    free = 20                                               # requests at the front that always fit
    q_p = np.minimum(100 * growth ** np.arange(n), 10**5).astype(np.int64)
    q_p[:free] = 1
    room0 = int(q_p.sum()) + 300 * (N + n)                  # at step 0; falls by N a step
    before = np.concatenate([[0], np.cumsum(q_p)[:-1]])
    q_U = (room0 - before) // (N + np.arange(n))
    q_U[:free] = 0
    u_max = int(q_U.max())
    seg = np.array([0, N], np.int64)
    p, g, U = np.full(N, 5), np.zeros(N, np.int64), np.full(N, u_max)
    cap = np.array([5 * N + room0])
    q_off, wait = np.array([0, n], np.int64), np.full(n, 1000)
    assert 0 <= orc.project(seg, p, g, U)[0] <= cap[0] < 2**31
    want_order, want_adm = orc.local_order(seg, p, g, U, cap, q_off, q_p, q_U, wait, 1000, u_max)
    args = (_cuda(cap), _cuda(q_off, np.int64), _cuda(q_p), _cuda(q_U), _cuda(wait), 1000)
    snap, b, order, adm, err = maps.project_order(_cuda(seg, np.int64), _cuda(p), _cuda(g), _cuda(U), u_max, *args)
    order2, adm2, err2 = maps.local_order(snap, *args)
    torch.cuda.synchronize()
    say(f"[order] one point at a time, {n}: {want_adm.tolist()}")
    assert int(err.item()) == 0 and int(err2.item()) == 0 and 0 < want_adm[0] < n
    for o, a in ((order, adm), (order2, adm2)):
        assert_same("order", o.cpu().numpy(), want_order)
        assert_same("admitted", a.cpu().numpy(), want_adm)
