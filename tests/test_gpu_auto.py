"""PASUR_SCHED_AUTO on large rounds: enqueued without a wait, captured and
replayed, side by side on several streams.  The schedules run the same operations
in the same order: states are compared bit for bit."""
import threading

import pytest

import synth
from gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def game(pa):
    """The whole game of deal 1: rounds 4 and 6 have 1.4e7 and 9.7e6 nodes."""
    deck, roots = synth.full_game_root(1)
    return pa.SubgameSolver(deck, 0, roots)


def fresh(pa, torch, rr, dtype):
    st = pa.CfrState(rr.fgt, dtype)
    V = None
    if rr.round < 5:
        g = torch.Generator(device="cuda").manual_seed(3)
        V = torch.empty(rr.fgt.n_next, dtype=torch.float64, device="cuda").uniform_(-9, 9, generator=g)
    pa.leaf_utilities(rr.fgt, V, dtype, st.u[8])
    pa.cfr_init(st)
    return st


def tensors(st):
    return st.sigma[1:] + st.R[1:] + st.u + [st.vacc]


# the call before the capture, and the captured one: segments or streaming sweeps
# (three iterations), of either state type
@pytest.mark.parametrize("before,captured", [((12, "F32"), (12, "F32")), ((12, "F32"), (9, "F64")),
                                             ((2, "F32"), (12, "F64")), ((12, "F64"), (2, "F32"))])
@pytest.mark.parametrize("k", [5, 3])
def test_auto_captured_after_a_warm_up(k, before, captured):
    pa = require_gpu()
    import torch
    s = game(pa)
    rr = s.rounds[k]
    n0, t0 = before[0], getattr(pa, "PASUR_" + before[1])
    n1, t1 = captured[0], getattr(pa, "PASUR_" + captured[1])
    print(f"[auto] round {k + 1}, {before} then {captured}", flush=True)
    pa.cfr_iterate(fresh(pa, torch, rr, t0), n0)
    ref = fresh(pa, torch, rr, t1)
    pa.cfr_iterate(ref, n1, pa.paper_params(pa.SCHED_LEVEL_SYNC))
    want = [t.clone() for t in tensors(ref)]
    st = fresh(pa, torch, rr, t1)
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            pa.cfr_init(st, side)
            pa.cfr_iterate(st, n1, stream=side)
    torch.cuda.current_stream().wait_stream(side)
    other = fresh(pa, torch, rr, t0)
    for i in range(4):
        for t in tensors(st)[:-1]:
            if t is not st.u[8]:
                t.fill_(0.25)
        if i % 2:  # eager work between the replays
            pa.cfr_iterate(other, n0)
            torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for j, (a, b) in enumerate(zip(tensors(st), want)):
            assert torch.equal(a, b), (i, j)
    s.free()


def test_auto_returns_before_its_work_is_done():
    """20 iterations of 1.4e7 nodes behind 50 ms of other work, on a tree whose first
    call is over."""
    pa = require_gpu()
    import torch
    s = game(pa)
    rr = s.rounds[3]
    pa.cfr_iterate(fresh(pa, torch, rr, pa.PASUR_F32), 20)
    ref = fresh(pa, torch, rr, pa.PASUR_F32)
    pa.cfr_iterate(ref, 20, pa.paper_params(pa.SCHED_ROOT))
    pa.cfr_iterate(ref, 20, pa.paper_params(pa.SCHED_ROOT))
    st = fresh(pa, torch, rr, pa.PASUR_F32)
    torch.cuda.synchronize()
    torch.cuda._sleep(100_000_000)
    pa.cfr_iterate(st, 20)
    pa.cfr_iterate(st, 20)
    assert not torch.cuda.current_stream().query()
    torch.cuda.synchronize()
    for a, b in zip(tensors(st) + st.Sbar[1:], tensors(ref) + ref.Sbar[1:]):
        assert torch.equal(a, b)
    s.free()


def test_auto_on_two_streams_and_from_two_threads():
    """Roots of up to 26,000 nodes, whose far arrays are scratch of the call: calls
    on states of their own that run at the same time."""
    pa = require_gpu()
    import torch
    s = game(pa)
    rr = s.rounds[3]
    ref = fresh(pa, torch, rr, pa.PASUR_F32)
    for _ in range(3):
        pa.cfr_iterate(ref, 10)
    states = [fresh(pa, torch, rr, pa.PASUR_F32) for _ in range(4)]
    streams = [torch.cuda.Stream() for _ in states]
    torch.cuda.synchronize()
    for _ in range(3):  # two streams, one thread
        for st, q in list(zip(states, streams))[:2]:
            pa.cfr_iterate(st, 10, stream=q)
    failed = []

    def work(st, q):
        try:
            for _ in range(3):
                pa.cfr_iterate(st, 10, stream=q)
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    threads = [threading.Thread(target=work, args=x) for x in list(zip(states, streams))[2:]]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for st in states:
        for a, b in zip(tensors(st) + st.Sbar[1:], tensors(ref) + ref.Sbar[1:]):
            assert torch.equal(a, b)
    s.free()


def scheduled(pa, torch, rr, dtype, iters):
    """The schedule that AUTO takes, by the kernels that it launches (on a state that
    is not solved: what the launches compute does not matter here)."""
    st = fresh(pa, torch, rr, dtype)
    pa.profile_enable(True)
    pa.cfr_iterate(st, iters)
    kernels = set(int(k) for k in pa.profile_read()[0])
    pa.profile_enable(False)
    assert kernels <= {2, 3} or not kernels & {2, 3}, kernels
    return "segments" if kernels & {2, 3} else "stream"


# 3.4e8 nodes, 18% of them below roots of 15,000 to 27,000 nodes; 1.5e8; 1.9e8, 9%
# below roots of more than 60,000; 1.2e8, small roots
@pytest.mark.parametrize("seed,k,dtype_name,line", [
    (48, 5, "PASUR_F32", 38), (40, 4, "PASUR_F64", 20), (4, 4, "PASUR_F32", 72),
    (7, 4, "PASUR_F64", 17), (7, 4, "PASUR_F32", 17)])
def test_auto_switches_by_size_iterations_and_roots(seed, k, dtype_name, line):
    pa = require_gpu()
    import torch
    deck, roots = synth.full_game_root(seed)
    s = pa.SubgameSolver(deck, 0, roots)
    rr = s.rounds[k]
    least = 5 + sum(rr.fgt.n) // 10_000_000
    assert line in (least, 3 * least)
    dtype = getattr(pa, dtype_name)
    print(f"[auto] deal {seed} round {k + 1}, {sum(rr.fgt.n)} nodes, {dtype_name}", flush=True)
    assert scheduled(pa, torch, rr, dtype, line - 1) == "stream"
    assert scheduled(pa, torch, rr, dtype, line) == "segments"
    s.free()


def test_auto_streams_a_root_that_one_workgroup_would_take_too_long_for():
    """One root of 1.6e7 nodes, iterated in place by one workgroup otherwise."""
    from test_gpu_values import wide_start
    pa = require_gpu()
    import torch
    deck, roots = wide_start()
    s = pa.SubgameSolver(deck, 5, roots)
    rr = s.rounds[0]
    assert sum(rr.fgt.n) > 9_000_000
    print(f"[auto] one root of {sum(rr.fgt.n)} nodes", flush=True)
    assert scheduled(pa, torch, rr, pa.PASUR_F32, 100) == "stream"
    s.free()
