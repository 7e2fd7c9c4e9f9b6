"""The App. A pressure simulation on the GPU (maps_simulate, one wavefront
per simulation, event to event) against the CPU oracle (one millisecond at a
time), bit for bit: completion times, routing, high-pressure time, longest
interval, interval count, queue maxima and areas, span.  Hand-worked
timelines, random small cases (both policies, thresholds hit exactly,
queueing), the App. A setup at full size over a utilisation sweep, limits and
the device error bits."""
import numpy as np
import pytest

import oracle
import workload.appa as appa
from tests.gpu_common import assert_same, say
from tests.oracle_pins import SIM_FIELDS, _sim_case, golden

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def orc():
    return oracle.Oracle()


def _cuda(x, dtype=np.int32):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, dtype=dtype)).cuda()


def _gpu(N, C, theta, arrivals, prompt, output, bound, policies):
    """One call: row s of `arrivals` with policy policies[s]."""
    import torch

    import paper_2609_15359_amd as maps
    arr = np.atleast_2d(np.asarray(arrivals, np.int64))
    r = maps.simulate(N, C, theta, _cuda(arr, np.int64), _cuda(prompt), _cuda(output), _cuda(bound),
                      _cuda(policies))
    torch.cuda.synchronize()
    st = r.stats.cpu().numpy()
    out = []
    for s in range(arr.shape[0]):
        out.append(dict(finish_ms=r.finish_ms[s].cpu().numpy(), routed=r.routed[s].cpu().numpy(),
                        hp_time=st[s, 0], hp_max=st[s, 1], hp_count=st[s, 2], max_queue=st[s, 3],
                        queue_area=st[s, 4], span=r.span[s].cpu().numpy()))
    return out, int(r.dev_err.item()) & 0xFFFFFFFF


def _compare(g, r, tag):
    for f in SIM_FIELDS:
        assert_same(f"{tag} {f}", g[f], getattr(r, f))


def test_hand_worked(orc):
    for c in golden("simulate_hand.json")["cases"]:
        got, err = _gpu(c["N"], c["C"], c["theta_ppm"], [c["arrival_ms"]], c["prompt"], c["output"], c["bound"],
                        [c["policy"]])
        assert err == 0
        for f in SIM_FIELDS:
            assert np.asarray(got[0][f]).tolist() == c[f], (c["name"], f)


def test_random_small(orc):
    rng = np.random.default_rng(77)
    for trial in range(150):
        N, C, theta, arr, prompt, output, bound = _sim_case(rng, n_max=40)
        got, err = _gpu(N, C, theta, [arr, arr], prompt, output, bound, [0, 1])
        assert err == 0, trial
        for pol in (0, 1):
            _compare(got[pol], orc.simulate(N, C, theta, arr, prompt, output, bound, pol), f"trial {trial} p{pol}")


@pytest.mark.parametrize("N", [1, 3, 8])
def test_heavy_queueing(orc, N):
    """Many requests at once on tight decoders: long FIFO queues, many
    admissions per completion, ready queues of tens of requests."""
    rng = np.random.default_rng(N)
    n = 3000
    prompt = rng.integers(0, 200, size=n).astype(np.int32)
    output = rng.integers(1, 400, size=n).astype(np.int32)
    bound = (output + rng.integers(-50, 200, size=n)).clip(-1).astype(np.int32)
    C = 6000
    arr = np.sort(rng.integers(0, 20000, size=n)).astype(np.int64)
    burst = np.zeros(n, np.int64)   # everything at t = 0
    got, err = _gpu(N, C, 700000, [arr, arr, burst, burst], prompt, output, bound, [0, 1, 0, 1])
    assert err == 0
    for s, (a, pol) in enumerate(((arr, 0), (arr, 1), (burst, 0), (burst, 1))):
        _compare(got[s], orc.simulate(N, C, 700000, a, prompt, output, bound, pol), f"N={N} case {s}")


def test_appendix_a_setup(orc):
    """App. A: 10,000 requests, N = 4, C = 50,000 tokens, theta = 0.85,
    t_tok = 1 ms, bounds from the oracle's calibration of the synthetic
    predictor, over a sweep of utilisation."""
    w = appa.make()
    q, _ = orc.calibrate(w.cal_pred, w.cal_truth, w.edges, appa.ALPHA_PPM)
    U = orc.apply_bounds(w.pred, w.edges, q, appa.U_MAX)
    rhos = [0.8, 0.9, 0.96, 1.0, 1.05, 1.1]
    arr = [w.arrivals(r) for r in rhos for _ in (0, 1)]
    pols = [p for _ in rhos for p in (0, 1)]
    got, err = _gpu(appa.N_DECODERS, appa.CAPACITY, appa.THETA_PPM, arr, w.prompt, w.output, U, pols)
    assert err == 0
    for s, (a, pol) in enumerate(zip(arr, pols)):
        r = orc.simulate(appa.N_DECODERS, appa.CAPACITY, appa.THETA_PPM, a, w.prompt, w.output, U, pol)
        _compare(got[s], r, f"rho={rhos[s // 2]} policy={pol}")
        T = r.span[1] - r.span[0]
        say(f"[appa] rho={rhos[s // 2]} policy={pol}: f_hp {np.round(r.hp_time / T, 3).tolist()} "
            f"max queue {r.max_queue.tolist()}")


def test_error_bits():
    ok, err = _gpu(1, 10, 500000, [[0, 1]], [2, 3], [4, 5], [4, 5], [0])
    assert err == 0
    _, err = _gpu(1, 10, 500000, [[0, 1]], [2, 8], [4, 5], [4, 5], [0])    # 8 + 5 > C
    assert err & 2048
    _, err = _gpu(1, 10, 500000, [[3, 1]], [2, 3], [4, 5], [4, 5], [0])    # arrival times decrease
    assert err & 2048
    _, err = _gpu(1, 10, 500000, [[0, 1]], [2, 3], [4, 0], [4, 5], [0])    # an empty output
    assert err & 2048
    n = 1100   # more admitted requests at once than a ready queue holds
    _, err = _gpu(1, 10**6, 500000, [np.zeros(n)], np.zeros(n), np.full(n, 3), np.full(n, 3), [0])
    assert err & 4096


@pytest.mark.parametrize("N,C,tokens", [(1, 3000, 20), (3, 1500, 12), (8, 4000, 30)])
def test_queues_outgrow_the_lanes(orc, N, C, tokens):
    """Small requests in bursts: the ready queues pass 64 requests in the middle
    of an event (arrivals, or a completion that makes room for many), where the
    simulation goes over from one request per lane to the queues in LDS; in the
    same launch one whose queues stay short and one with a last arrival past 32
    bits of milliseconds."""
    rng = np.random.default_rng(N)
    n = 700
    prompt = rng.integers(0, tokens, size=n)
    output = rng.integers(1, tokens, size=n)
    bound = np.where(rng.random(n) < 0.1, -1, output + rng.integers(0, 4, size=n))
    prompt[rng.random(n) < 0.02] = C // 2
    prompt[-1], output[-1], bound[-1] = 5, 7, 7
    burst = np.sort(rng.integers(0, 12, size=n)) * 97
    spread = np.arange(n) * (tokens * 2)
    late = np.concatenate([burst[:-1], [2**33]])
    rows = [burst, burst, spread, spread, late, late]
    got, err = _gpu(N, C, 850000, rows, prompt, output, bound, [0, 1] * 3)
    assert err == 0
    for s in range(4):
        _compare(got[s], orc.simulate(N, C, 850000, rows[s], prompt, output, bound, s % 2), f"N={N} case {s}")
    for s in (4, 5):   # the oracle steps through every millisecond: without the last request
        want = orc.simulate(N, C, 850000, burst[:-1], prompt[:-1], output[:-1], bound[:-1], s % 2)
        assert_same(f"N={N} late finish", got[s]["finish_ms"][:-1], want.finish_ms)
        assert_same(f"N={N} late routed", got[s]["routed"][:-1], want.routed)
        assert_same(f"N={N} late queue area", got[s]["queue_area"], want.queue_area)
        assert got[s]["finish_ms"][-1] == 2**33 + 7


@pytest.mark.parametrize("name,arrival,output", [
    ("gap of 2^22 - 1", [0, 0], [2**21, 2**21 + 9]),               # the last of the float quotients
    ("gap of 2^22 + 1", [0, 0], [2**21 + 1, 2**21 + 9]),           # the first of the integer divisions
    ("three in turn", [0, 0, 0], [2**22 + 5] * 3),
    ("arrival at 2^22 - 1", [0, 0, 2**22 - 1], [2**22, 2**22 + 2, 7]),
    ("arrival at 2^22", [0, 0, 2**22], [2**22, 2**22 + 2, 7]),
    ("arrival at 2^22 + 1", [0, 0, 2**22 + 1], [2**22, 2**22 + 2, 7]),
    ("longest output in 24 bits", [3, 5, 9], [2**24 - 1, 4, 2**22]),
    ("output of 2^24", [3, 5, 9], [2**24, 4, 2**22]),               # past the fast form
])
def test_long_outputs(orc, name, arrival, output):
    """Queues that stay as they are over millions of milliseconds, on both sides of where the slices since the
    last event are divided as floats, and outputs on both sides of the fast form's limit."""
    n = len(output)
    prompt, bound = np.arange(n), np.array(output) + 3
    got, err = _gpu(1, 2**30, 10000, [arrival, arrival], prompt, output, bound, [0, 1])
    assert err == 0
    for s in (0, 1):
        want = orc.simulate(1, 2**30, 10000, np.array(arrival, np.int64), prompt, output, bound, s)
        _compare(got[s], want, f"{name} policy {s}")
        say(f"[appa] {name}: done at {want.finish_ms.tolist()}")
