"""Which form of the segment schedule runs: the plan says it, the device counts the
segments that ran otherwise, and every form's state is that of the
level-synchronous kernels.  Also the games of self-play beyond one per thread,
against the oracle's."""
import numpy as np
import pytest

import synth
from gpu_common import oracle_rounds, require_gpu, to_np
from oracle import selfplay as sp
from test_gpu_kernels import arrays, disturb, playout
from test_gpu_values import wide_root

pytestmark = pytest.mark.gpu


def level_sizes(pa, f):
    """Nodes of every root on every level (levels are root-major): [9][roots]."""
    at = np.arange(f.n[0] + 1, dtype=np.int64)
    n = [np.diff(at)]
    for l in range(8):
        at = f.read(pa.FGT_CHILD_BEGIN, l).astype(np.int64)[at]
        n.append(np.diff(at))
    return np.array(n)


# 179 roots of up to 33,000 nodes (seed 101), 36 of 15,424 to 36,722 (102), one of
# 1.3e5, which has no compact form
@pytest.mark.parametrize("case,dtype_name,how", [
    ((101, 3), "PASUR_F32", ""), ((101, 3), "PASUR_F64", "regrets"), ((102, 3), "PASUR_F32", ""),
    ((102, 3), "PASUR_F64", ""), ((102, 3), "PASUR_F32", "sigma"), ("wide", "PASUR_F32", "")])
def test_form_that_runs_is_the_planned_one(case, dtype_name, how):
    """An edge takes 4 values in LDS (2 and its node's words apart with far arrays), an
    edge below level 5 two more, a node one and 14 bytes of words, the tables up to
    8.2 KB and 2 bytes a node; 159 KB are there.  Nodes above level 6 always count,
    those of levels 6 and 7 unless they are forced chains."""
    pa = require_gpu()
    import torch
    dtype = getattr(pa, dtype_name)
    if case == "wide":
        (deck, roots), start = wide_root(7, 8), 5
    else:
        (deck, roots), start = playout(pa, *case), case[1]
    s = pa.SubgameSolver(deck, start, roots, dtype=dtype)
    rr = s.rounds[-1]
    out = []
    for planned in (False, True):
        st = pa.CfrState(rr.fgt, dtype)
        for t in st.reachA[1:8] + st.reachB[1:8] + st.u[:8]:
            t.zero_()
        pa.leaf_utilities(rr.fgt, None, dtype, st.u[8])
        pa.cfr_init(st)
        disturb(torch, rr, st, how)
        if planned:
            plan = pa.Plan([st], pa.paper_params(pa.SCHED_ROOT), 1, 8)
            plan.iterate(1, 3)
            plan.iterate(4, 5)
            torch.cuda.synchronize()
            forms = plan.forms()
            print(f"[forms] {sum(rr.fgt.n)} nodes {dtype_name} {how}: {forms}", flush=True)
            n, v, room = level_sizes(pa, rr.fgt), 4 if dtype == pa.PASUR_F32 else 8, 159 * 1024
            few, all_ = n[1:7].sum(0), n[1:].sum(0)          # edges
            inner, nodes = n[:6].sum(0), n[:8].sum(0)
            tables = 8400 + 2 * nodes
            lds = (4 * v * few + (v + 14) * inner,
                   4 * v * all_ + 2 * v * n[7:].sum(0) + (v + 14) * nodes + tables)
            far = (2 * v * few + v * inner, 2 * v * all_ + v * nodes + tables)
            for (least, most), count in ((lds, forms["lds"]), (far, forms["lds"] + forms["far"])):
                assert np.sum(most <= room) <= count <= np.sum(least <= room)
            assert forms["in_place"] == np.sum(all_ > 100000)
            n = n[0]
            assert forms["lds"] + forms["far"] + forms["all_far"] + forms["in_place"] == len(n)
            assert plan.n_segs == len(n)
            assert plan.block == forms["most_threads"] >= forms["least_threads"] >= 256
            # a chain that is not forced makes the form larger than planned
            assert (forms["unplanned"] > 0) == (how == "sigma")
            plan.free()
        else:
            pa.cfr_iterate(st, 8, pa.paper_params(pa.SCHED_LEVEL_SYNC))
        torch.cuda.synchronize()
        out.append(arrays(st))
    for k, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b), k
    s.free()


def test_threads_that_a_plan_reports_are_those_it_launches():
    """Small roots, of which four fit a compute unit: workgroups of 256."""
    pa = require_gpu()
    deck, roots = synth.full_game_root(1)
    s = pa.SubgameSolver(deck, 0, roots)
    rr = s.rounds[2]  # 586 roots of some 2,600 nodes
    plan = pa.Plan([pa.CfrState(rr.fgt, pa.PASUR_F32)], pa.paper_params(pa.SCHED_ROOT), 1, 2)
    f = plan.forms()
    print(f"[forms] {f}", flush=True)
    assert f["least_threads"] == 256 and plan.block == f["most_threads"]
    other = pa.Plan(plan.states, pa.paper_params(pa.SCHED_ROOT, 512), 1, 2)
    f = other.forms()
    assert f["least_threads"] == f["most_threads"] == other.block == 512
    for x in (plan, other):
        x.free()
    s.free()


def test_games_beyond_one_per_thread_match_the_oracle():
    """Two uniform players, two average strategies and both mixtures: games from all
    over a call in which a thread plays several."""
    pa = require_gpu()
    deck, roots = playout(pa, 102, 4)
    s = pa.SubgameSolver(deck, 4, roots, dtype=pa.PASUR_F64)
    s.solve(30)
    rounds = []
    for (gt, f), rr in zip(oracle_rounds(deck, 4, roots), s.rounds):
        rounds.append({"cb": f.child_begin(), "sbar": [None] + [to_np(t) for t in rr.state.sigma_bar[1:]],
                       "link": rr.fgt.read(pa.FGT_LINK) if rr.round < 5 else None,
                       "base": rr.fgt.read(pa.FGT_LEAF_BASE)})
    S, U = pa.PLAY_SIGMA_BAR, pa.PLAY_UNIFORM
    for pol in ((S, S), (S, U), (U, S), (U, U)):
        n = (1 << 19) + 1000
        got = to_np(s.selfplay(n, 9, *pol))
        games = np.unique(np.concatenate([np.arange(50), np.linspace(0, n - 1, 400).astype(int)]))
        for g in games:
            q, m = 0, 0
            for r, R in enumerate(rounds):
                for l in range(8):
                    b, e = int(R["cb"][l][q]), int(R["cb"][l][q + 1])
                    u = sp.splitmix_uniform(9, int(g) * 64 + r * 8 + l)
                    q = b + sp.choose(u, R["sbar"][l + 1][b:e], pol[l & 1])
                m += int(R["base"][q])
                if r + 1 < len(rounds):
                    q = int(R["link"][q])
            assert got[g] == m, (pol, g)
    s.free()


@pytest.mark.parametrize("beta,dtype_name", [(-1.0, "PASUR_F32"), (-1.0, "PASUR_F64"),
                                             (400.0, "PASUR_F64")])
def test_discounts_that_are_not_numbers(beta, dtype_name):
    """0^beta for beta < 0 and 9^400 are infinite, their discounts NaN: regrets of
    forced chains follow them as in the level-synchronous kernels, from the first
    iteration on or from where the power overflows.  Such segments run in place."""
    pa = require_gpu()
    import torch
    deck, roots = playout(pa, 8, 4)
    s = pa.SubgameSolver(deck, 4, roots, dtype=getattr(pa, dtype_name))
    rr = s.rounds[1]
    out = []
    for sched in (pa.SCHED_LEVEL_SYNC, pa.SCHED_ROOT):
        p = pa.paper_params(sched)
        p.beta = beta
        st = pa.CfrState(rr.fgt, s.dtype)
        for t in st.reachA[1:8] + st.reachB[1:8] + st.u[:8]:
            t.zero_()
        pa.leaf_utilities(rr.fgt, None, s.dtype, st.u[8])
        pa.cfr_init(st)
        pa.cfr_iterate(st, 4, p)
        pa.cfr_iterate(st, 8, p)
        torch.cuda.synchronize()
        out.append(arrays(st))
    assert any(np.isnan(a).any() for a in out[0])
    plan = pa.Plan([st], p, 1, 12)
    assert plan.forms()["in_place"] == plan.n_segs == rr.fgt.n[0]
    plan.free()
    for k, (a, b) in enumerate(zip(*out)):
        assert np.array_equal(a, b, equal_nan=True), k
    s.free()
