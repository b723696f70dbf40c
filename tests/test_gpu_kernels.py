"""Each kernel variant where it can go wrong, against the oracle or against the
kernels that the other tests hold to it: the forms of the segment schedule, the
schedule that AUTO picks, the ends of a batch, external sampling beyond its
on-chip lists, tree values of many roots, feature rows that are not aligned,
trees wider than the scans' tiles, built in several threads.

The schedules run the same operations in the same order, so states are compared
bit for bit; the tree values' tolerance is stated where it is used."""
import threading

import numpy as np
import pytest

import oracle
import synth
from oracle import mlp as omlp
from gpu_common import oracle_rounds, require_gpu, roots_from_array, to_np
from test_gpu_trees import compare_round

pytestmark = pytest.mark.gpu


def playout(pa, seed, start):
    deck = synth.deal(seed)
    return deck, roots_from_array([pa.playout_root(deck, start, synth.playout_draws(seed, start))])


def arrays(st):
    return [to_np(t).copy() for t in st.sigma[1:] + st.R[1:] + st.Sbar[1:] + st.reachA[:8]
            + st.reachB[:8] + st.u] + [to_np(st.vacc).copy()]


def disturb(torch, rr, st, how):
    """A state that the solver's own calls do not make (single-child edges
    included), but which the level-synchronous kernels iterate."""
    g = torch.Generator(device="cuda").manual_seed(5)
    if how == "regrets":  # as a warm start leaves them
        for l in range(1, 9):
            st.R[l].uniform_(-2.0, 2.0, generator=g)
            st.Sbar[l].uniform_(0.0, 2.0, generator=g)
    elif how == "sigma":  # no chain is forced
        for l in range(1, 9):
            st.sigma[l].mul_(0.75)
    elif how == "leaf":  # an infinite utility spreads, and turns into NaN
        st.u[8][::101] = float("inf")


# seed 102, round 5: one root of 15,424 nodes; from round 3: 36 roots of 15,424 to
# 36,722 nodes (on chip up to 14,000 nodes in FP32 and 7,000 in FP64, the far
# arrays apart up to 32,000 and 16,000, all of them beyond); seed 101: 179 roots,
# groups of up to 12 children
@pytest.mark.parametrize("seed,start,dtype_name,rule,block,seg_nodes,how", [
    (102, 5, "PASUR_F32", "dcfr", 0, 0, ""), (102, 5, "PASUR_F64", "dcfr", 0, 0, ""),
    (102, 3, "PASUR_F32", "dcfr", 0, 0, "regrets"), (102, 3, "PASUR_F64", "plus", 0, 0, ""),
    (102, 3, "PASUR_F32", "vanilla", 0, 0, ""), (102, 3, "PASUR_F64", "dcfr+", 256, 0, "regrets"),
    (101, 3, "PASUR_F32", "plus", 0, 0, "regrets"), (101, 3, "PASUR_F64", "dcfr", 512, 0, ""),
    (101, 3, "PASUR_F32", "dcfr0", 0, 9000, ""), (101, 4, "PASUR_F32", "dcfr", 256, 0, "leaf"),
    (102, 3, "PASUR_F32", "dcfr", 0, 0, "sigma"), (101, 4, "PASUR_F64", "dcfr+", 0, 20000, "sigma")])
def test_segment_forms_equal_level_sync(seed, start, dtype_name, rule, block, seg_nodes, how):
    pa = require_gpu()
    import torch
    dtype = getattr(pa, dtype_name)
    deck, roots = playout(pa, seed, start)
    s = pa.SubgameSolver(deck, start, roots, dtype=dtype)
    rr = s.rounds[-1]
    print(f"[segments] {sum(rr.fgt.n)} nodes, {rr.fgt.n[0]} roots, {dtype_name} {rule} "
          f"block={block} seg_nodes={seg_nodes} {how}", flush=True)
    out = []
    for sched in (pa.SCHED_LEVEL_SYNC, pa.SCHED_ROOT):
        p = pa.paper_params(sched, block, seg_nodes)
        if rule == "plus":
            p.variant, p.rm_mode = pa.CFR_PLUS, pa.RM_POSITIVE
        elif rule == "vanilla":
            p.variant, p.rm_mode = pa.CFR_VANILLA, pa.RM_POSITIVE
        elif rule == "dcfr+":
            p.rm_mode = pa.RM_POSITIVE
        elif rule == "dcfr0":
            p.eps = 0.0
        st = pa.CfrState(rr.fgt, dtype)
        for t in st.reachA[1:8] + st.reachB[1:8] + st.u[:8]:
            t.zero_()
        pa.leaf_utilities(rr.fgt, None, dtype, st.u[8])
        pa.cfr_init(st)
        disturb(torch, rr, st, how)
        pa.cfr_iterate(st, 4, p)
        pa.cfr_iterate(st, 5, p)
        torch.cuda.synchronize()
        out.append(arrays(st))
    for k, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b, equal_nan=how == "leaf"), k
    s.free()


def test_auto_picks_by_iterations_on_large_rounds():
    """A round of 9.7e6 nodes: streamed for three iterations (no sums below
    forced chains), in segments for eight."""
    pa = require_gpu()
    import torch
    deck, roots = synth.full_game_root(1)
    s = pa.SubgameSolver(deck, 0, roots)
    rr = s.rounds[5]
    assert 9_000_000 <= sum(rr.fgt.n) < 12_000_000
    for iters, sched in ((3, pa.SCHED_STREAM), (8, pa.SCHED_ROOT)):
        out = []
        for x in (sched, pa.SCHED_AUTO):
            print(f"[auto] {iters} iterations, schedule {x}", flush=True)
            st = pa.CfrState(rr.fgt, pa.PASUR_F32)
            pa.leaf_utilities(rr.fgt, None, pa.PASUR_F32, st.u[8])
            pa.cfr_init(st)
            pa.cfr_iterate(st, iters, pa.paper_params(x))
            torch.cuda.synchronize()
            out.append([to_np(t) for t in st.sigma[1:] + st.R[1:] + st.Sbar[1:]])
        for a, b in zip(*out):
            assert np.array_equal(a, b)
    s.free()


@pytest.mark.parametrize("dtype_name", ["PASUR_F32", "PASUR_F64"])
@pytest.mark.parametrize("n", [1, 8, 11])
def test_batch_ends_equal_single_calls(dtype_name, n):
    """Eight trees fill a launch."""
    pa = require_gpu()
    import torch
    dtype = getattr(pa, dtype_name)
    b = pa.BatchSolver([synth.two_round_root(i + 1) for i in range(n)], 4, 5, dtype=dtype)
    print(f"[batch ends] {dtype_name} {n} deals", flush=True)
    b.solve()
    torch.cuda.synchronize()
    for sv in b.deals:
        V = None
        for k in (1, 0):
            rr = sv.rounds[k]
            st = pa.CfrState(rr.fgt, dtype)
            pa.leaf_utilities(rr.fgt, V, dtype, st.u[8])
            pa.cfr_init(st)
            pa.cfr_iterate(st, 5, pa.paper_params(pa.SCHED_LEVEL_SYNC))
            pa.average_strategy(st)
            V = torch.empty(rr.fgt.n[0], dtype=torch.float64, device="cuda")
            pa.round_values(st, pa.V_ITERATE_MEAN, V)
            torch.cuda.synchronize()
            assert np.array_equal(to_np(V), to_np(rr.V))
            for x, y in zip(st.sigma_bar[1:] + st.R[1:] + st.u, rr.state.sigma_bar[1:]
                            + rr.state.R[1:] + rr.state.u):
                assert np.array_equal(to_np(x), to_np(y))
    with pytest.raises(pa.PasurError, match="next round's root values"):
        b.ends[0].begin([None] * n)
    b.free()


@pytest.mark.parametrize("dtype_name", ["PASUR_F32", "PASUR_F64"])
def test_init_writes_its_arrays_only(dtype_name):
    """Arrays that begin and end between 16-byte boundaries."""
    pa = require_gpu()
    import torch
    dtype = getattr(pa, dtype_name)
    deck, roots = synth.last_round_roots(3)
    s = pa.SubgameSolver(deck, 5, roots, dtype=dtype)
    rr = s.rounds[0]
    for shift in (1, 2, 3):
        st = pa.CfrState(rr.fgt, dtype)
        big = {}
        for name in ("R", "Sbar", "sigma"):
            for l in range(1, 9):
                t = torch.full((rr.fgt.n[l] + 8,), 7.0, dtype=st.R[1].dtype, device="cuda")
                big[name, l] = t
                getattr(st.c, name)[l] = t[shift:].data_ptr()
        pa.cfr_init(st)
        torch.cuda.synchronize()
        for (name, l), t in big.items():
            x, n = to_np(t), rr.fgt.n[l]
            assert np.all(x[:shift] == 7.0) and np.all(x[shift + n:] == 7.0), (name, l)
            if name == "sigma":
                k = np.diff(rr.fgt.read(pa.FGT_CHILD_BEGIN, l - 1))
                assert np.array_equal(x[shift:shift + n], np.repeat((1.0 / k).astype(x.dtype), k))
            else:
                assert np.all(x[shift:shift + n] == 0.0), (name, l)
    s.free()


@pytest.mark.parametrize("dtype_name,rm", [("PASUR_F32", "RM_FLOOR"), ("PASUR_F64", "RM_POSITIVE")])
@pytest.mark.parametrize("per_wg", [1, 5, 62])
def test_external_sampling_beyond_on_chip_lists(dtype_name, rm, per_wg):
    """A wave with 62 roots reaches some thousand nodes in a pass, more than it
    holds on chip; the level schedule visits every node."""
    pa = require_gpu()
    import torch
    dtype = getattr(pa, dtype_name)
    deck, roots = playout(pa, 8, 4)
    s = pa.SubgameSolver(deck, 4, roots, dtype=dtype)
    rr = s.rounds[1]
    assert rr.fgt.n[0] == 62
    out = []
    for sched in (pa.ES_LEVEL, pa.ES_FRONTIER):
        print(f"[es] {dtype_name} {rm} schedule {sched}, {per_wg} roots a wave", flush=True)
        st = pa.CfrState(rr.fgt, dtype)
        for t in st.u[:8]:
            t.zero_()
        pa.leaf_utilities(rr.fgt, None, dtype, st.u[8])
        pa.cfr_init(st)
        pa.es_iterate(st, 6, 11, getattr(pa, rm), schedule=sched, roots_per_wg=per_wg)
        pa.es_iterate(st, 5, 11, getattr(pa, rm), schedule=sched, roots_per_wg=per_wg)
        torch.cuda.synchronize()
        out.append([to_np(t).copy() for t in st.sigma[1:] + st.R[1:] + st.Sbar[1:] + st.u])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    s.free()


def values_np(n, cb, sigma, leaf, mode, tv):
    v = leaf
    for l in range(7, -1, -1):
        at = cb[l][:-1].astype(np.int64)
        if l % 2 == 0 and mode in (tv["BR_A"], tv["MINIMAX"]):
            v = np.maximum.reduceat(v, at)
        elif l % 2 == 1 and mode in (tv["BR_B"], tv["MINIMAX"]):
            v = np.minimum.reduceat(v, at)
        else:
            v = np.add.reduceat(sigma[l + 1].astype(np.float64) * v, at)
    return v


@pytest.mark.parametrize("seed,start", [(101, 3), (1, 0)])
def test_tree_values_of_many_and_wide_roots(seed, start):
    """179 roots, some with more than 1,024 nodes on level 5, and 3,211 roots.
    Tolerance: a level adds at most 13 products, each with one rounding and
    summed in another order: 8 levels of 14 roundings of values below 100
    differ by at most 8 * 14 * 2^-53 * 100 < 1.3e-12."""
    pa = require_gpu()
    import torch
    if start == 0:
        deck, roots = synth.full_game_root(seed)
    else:
        deck, roots = playout(pa, seed, start)
    s = pa.SubgameSolver(deck, start, roots)
    rr = s.rounds[-1]
    st = pa.CfrState(rr.fgt, pa.PASUR_F32)
    pa.leaf_utilities(rr.fgt, None, pa.PASUR_F32, st.u[8])
    pa.cfr_init(st)
    pa.cfr_iterate(st, 5)
    pa.average_strategy(st)
    leaf = st.u[8].double()
    sb = [None] + [to_np(t) for t in st.sigma_bar[1:]]
    cb = [rr.fgt.read(pa.FGT_CHILD_BEGIN, l) for l in range(8)]
    tv = {k: getattr(pa, "TV_" + k) for k in ("EXPECT", "BR_A", "BR_B", "MINIMAX")}
    V = torch.empty(rr.fgt.n[0], dtype=torch.float64, device="cuda")
    for mode in tv.values():
        print(f"[values] {rr.fgt.n[0]} roots, mode {mode}", flush=True)
        pa.tree_values(rr.fgt, leaf, pa.PASUR_F32, st.sigma_bar, mode, V)
        torch.cuda.synchronize()
        want = values_np(rr.fgt.n, cb, sb, to_np(leaf), mode, tv)
        assert np.max(np.abs(to_np(V) - want)) <= 1.3e-12
    s.free()


@pytest.mark.parametrize("which", ["a", "b", "v", "ab", "bv", "abv"])
def test_exploitability_outputs_one_at_a_time(which):
    """Outputs asked for together or alone are the same numbers."""
    pa = require_gpu()
    import torch
    deck, roots = playout(pa, 101, 3)
    s = pa.SubgameSolver(deck, 3, roots)
    s.solve(5)
    want = [to_np(t) for t in s.exploitability()]
    out = [torch.full((len(roots),), 9.0, dtype=torch.float64, device="cuda") if c in which else None
           for c in "abv"]
    pa.exploitability([rr.fgt for rr in s.rounds], [rr.state.sigma_bar for rr in s.rounds],
                      pa.PASUR_F32, *out)
    torch.cuda.synchronize()
    for got, ref in zip(out, want):
        assert got is None or np.array_equal(to_np(got), ref)
    s.free()


def test_results_of_a_solver_with_its_own_stream():
    """Solves and best responses on a stream of the solver's own: what they return
    is read on the caller's stream without waiting."""
    pa = require_gpu()
    import torch
    deck, roots = playout(pa, 101, 3)
    ref = pa.SubgameSolver(deck, 3, roots)
    s = pa.SubgameSolver(deck, 3, roots, stream=torch.cuda.Stream())
    for iters in (3, 40, 10):
        want = [float(ref.solve(iters)[0])] + [float(x[0]) for x in ref.exploitability()]
        for _ in range(3):
            V = s.solve(iters)
            got = [float(V[0])]
            a, b, v = s.exploitability()
            assert float(((a - b) / 2).max()) >= 0.0
            assert got + [float(x[0]) for x in (a, b, v)] == want
            m = s.selfplay(1000, 7)
            assert int(m.sum()) == int(ref.selfplay(1000, 7).sum())
    s.free()
    ref.free()


@pytest.mark.parametrize("n", [1, 7, 31, 32, 33, 257])
def test_feature_rows_at_any_offset(n):
    """Rows of 384 bytes to aligned and unaligned places, all edges in order or
    a list of them."""
    pa = require_gpu()
    import torch
    deck, roots = synth.two_round_root(2)
    s = pa.SubgameSolver(deck, 4, roots, keep_gt=True)
    rr = s.rounds[1]
    l = 4
    width = omlp.N_IN
    full = torch.empty((rr.fgt.n[l], width), dtype=torch.int16, device="cuda")
    pa.edge_features(rr.gt, rr.fgt, l, None, rr.fgt.n[l], full)
    pick = torch.randperm(rr.fgt.n[l], generator=torch.Generator().manual_seed(n))[:n].int().cuda()
    for edges, rows in ((None, rr.fgt.n[l]), (pick, n)):
        want = to_np(full if edges is None else full[pick.long()]).reshape(-1)
        for shift in (0, 1, 3):
            buf = torch.full((rows * width + 16,), 21, dtype=torch.int16, device="cuda")
            pa.edge_features(rr.gt, rr.fgt, l, edges, rows, buf[shift:])
            torch.cuda.synchronize()
            got = to_np(buf)
            assert np.array_equal(got[shift:shift + rows * width], want)
            assert np.all(got[:shift] == 21) and np.all(got[shift + rows * width:] == 21)
    s.free()


def test_wide_trees_match_oracle():
    """Rounds whose levels span several tiles of the scans and sorts."""
    pa = require_gpu()
    deck, roots = playout(pa, 102, 4)
    for k, (gt, f) in enumerate(oracle_rounds(deck, 4, roots)):
        compare_round(pa, deck, 4 + k, roots)
        if k == 0:
            roots = roots_from_array(f.get(oracle.FGT_NEXT_ROOTS))


def test_trees_built_in_several_threads():
    """Trees that take and give back device memory at once in four threads, each
    on a stream of its own, are those that one thread builds."""
    pa = require_gpu()
    import torch

    def build(seed, stream):
        with torch.cuda.stream(stream):
            deck, roots = playout(pa, seed, 3)
            s = pa.SubgameSolver(deck, 3, roots, stream=stream)
            out = [rr.fgt.read(f, l) for rr in s.rounds for l in range(8)
                   for f in (pa.FGT_GT, pa.FGT_SID, pa.FGT_CHILD_BEGIN)]
            s.free()
        return out

    seeds = [5, 6, 7, 8]
    want = {x: build(x, torch.cuda.Stream()) for x in seeds}
    failed = []

    def work(seed):
        try:
            stream = torch.cuda.Stream()
            for _ in range(3):
                for a, b in zip(build(seed, stream), want[seed]):
                    assert np.array_equal(a, b)
        except Exception as e:  # noqa: BLE001
            failed.append((seed, repr(e)))

    threads = [threading.Thread(target=work, args=(x,)) for x in seeds]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_cached_blocks_follow_the_games_built():
    """Trees of 8.5e8 and of 6.4e8 nodes, more than the cache holds together: the
    last game's blocks stay, so that building it again asks the device for none."""
    pa = require_gpu()
    import torch
    slack = 256 << 20  # the tensors of the driver and of other libraries

    def build_and_free(seed):
        deck, roots = synth.full_game_root(seed)
        s = pa.SubgameSolver(deck, 0, roots)
        built = torch.cuda.mem_get_info()[0]
        s.free()
        return built, torch.cuda.mem_get_info()[0]

    pa.lib().pasur_release_cache()
    start = torch.cuda.mem_get_info()[0]
    _, free = build_and_free(40)
    assert start - free <= (16 << 30) + slack
    _, free = build_and_free(22)
    assert start - free <= (16 << 30) + slack
    built, again = build_and_free(22)
    assert abs(built - free) <= slack and abs(again - free) <= slack
    pa.lib().pasur_release_cache()
    assert start - torch.cuda.mem_get_info()[0] <= slack


# one game per thread up to 2^18 games of two uniform players and 2^19 others,
# several beyond: the same game under its number in both
@pytest.mark.parametrize("dtype_name", ["PASUR_F32", "PASUR_F64"])
@pytest.mark.parametrize("start", [4, 5])
def test_games_do_not_depend_on_their_number(start, dtype_name):
    pa = require_gpu()
    import torch
    deck, roots = playout(pa, 102, start)
    s = pa.SubgameSolver(deck, start, roots, dtype=getattr(pa, dtype_name))
    s.solve(30)
    S, U = pa.PLAY_SIGMA_BAR, pa.PLAY_UNIFORM
    for pol, line in (((S, S), 1 << 19), ((S, U), 1 << 19), ((U, S), 1 << 19), ((U, U), 1 << 18)):
        want = s.selfplay(line, 3, *pol)
        for n in (1, 257, line - 1, line + 1, 2 * line + 255):
            got = s.selfplay(n, 3, *pol)
            assert got.shape == (n,)
            m = min(n, line)
            assert torch.equal(got[:m], want[:m]), (pol, n)
        assert len(torch.unique(want)) > (pol != (S, S)), pol
    s.free()
