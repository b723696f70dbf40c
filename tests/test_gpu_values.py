"""Exact values of rounds with few large roots, which are split over workgroups,
against the oracle's, one node at a time in FP64."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import oracle_exploitability, oracle_rounds, require_gpu, to_np

pytestmark = pytest.mark.gpu


def wide_root(seed, n_pool, rnd=5):
    """A start state of round `rnd` whose pool holds n_pool numerics."""
    deck = synth.deal(seed)
    cards = [c for c in sorted(deck[:4 + 8 * rnd]) if c < 40][::2][:n_pool]
    return deck, [synth.Root(sum(1 << c for c in cards), 0, 0, 0, 1)]


def wide_start():
    """Aces, twos and threes in hand and fourteen numerics in the pool: 139 moves at
    the root, 4,586 nodes on level 2."""
    alex, bob = [0, 4, 8, 40], [1, 5, 44, 48]
    pool = [c for s in (2, 3, 1, 0) for c in range(s, 40, 4) if c not in alex + bob][:14]
    deck = [c for c in range(52) if c not in alex + bob] + alex + bob
    return deck, [synth.Root(sum(1 << c for c in pool), 0, 0, 0, 1)]


# one root of 6.1e3 nodes, which is not split, and of 1.3e5, 7.0e5, 2.5e6 and 1.6e7,
# which fit one workgroup from level 3, 2, 2 and 1 on
ROUNDS = [("pool 4", lambda pa: wide_root(7, 4)), ("pool 8", lambda pa: wide_root(7, 8)),
          ("pool 10", lambda pa: wide_root(7, 10)), ("pool 12", lambda pa: wide_root(7, 12)),
          ("fourteen", lambda pa: wide_start())]


@pytest.mark.parametrize("dtype_name", ["PASUR_F32", "PASUR_F64"])
@pytest.mark.parametrize("case", range(len(ROUNDS)))
def test_values_of_large_roots(case, dtype_name):
    """Tolerance: a node's sum of at most K products of one rounding each, over 8
    levels, of values of at most |leaf|: 8 (K + 1) 2^-53 max |leaf|, if the oracle
    sums in another order; best responses round no more than that."""
    pa = require_gpu()
    import torch
    name, make = ROUNDS[case]
    deck, roots = make(pa)
    dtype = getattr(pa, dtype_name)
    s = pa.SubgameSolver(deck, 5, roots, dtype=dtype)
    f = s.rounds[0].fgt
    cb = [f.read(pa.FGT_CHILD_BEGIN, l) for l in range(8)]
    rng = np.random.default_rng(case)
    sig = [None]
    for l in range(8):
        k = np.diff(cb[l])
        w = rng.random(f.n[l + 1]) + 0.01
        sig.append(w / np.repeat(np.add.reduceat(w, cb[l][:-1]), k))
    tdt = torch.float32 if dtype == pa.PASUR_F32 else torch.float64
    dev = [None] + [torch.from_numpy(x).to("cuda", tdt) for x in sig[1:]]
    sig = [None] + [to_np(t).astype(np.float64) for t in dev[1:]]
    leaf = torch.empty(f.n[8], dtype=torch.float64, device="cuda")
    pa.leaf_utilities(f, None, pa.PASUR_F64, leaf)
    K = max(int(np.diff(c).max()) for c in cb)
    tol = 8 * (K + 1) * 2.0 ** -53 * float(leaf.abs().max())
    out, again = (torch.empty(f.n[0], dtype=torch.float64, device="cuda") for _ in range(2))
    for mode in (pa.TV_EXPECT, pa.TV_BR_A, pa.TV_BR_B, pa.TV_MINIMAX):
        print(f"[values] {name} {dtype_name} {sum(f.n)} nodes, mode {mode}", flush=True)
        sg = None if mode == pa.TV_MINIMAX else dev
        pa.tree_values(f, leaf, dtype, sg, mode, out)
        if max(f.n[:8]) <= 1 << 21:  # what it takes
            pa.tree_values_noalloc(f, leaf, dtype, sg, mode, again)
        else:
            pa.tree_values(f, leaf, dtype, sg, mode, again)
        torch.cuda.synchronize()
        want = oracle.tree_values(f.n, cb, to_np(leaf), sig, mode)
        assert np.max(np.abs(to_np(out) - want)) <= tol
        assert torch.equal(out, again)
    # and as a round's value, from leaves of the state's type
    st = pa.CfrState(f, dtype)
    pa.leaf_utilities(f, None, dtype, st.u[8])
    pa.cfr_init(st)
    for l in range(1, 9):
        st.sigma_bar[l].copy_(dev[l])
    pa.round_values(st, pa.V_SIGMA_BAR, again)
    pa.tree_values(f, st.u[8].double(), dtype, dev, pa.TV_EXPECT, out)
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    s.free()


def test_exploitability_of_rounds_with_large_roots():
    """From round 4 with a pool of eight numerics: its root and many of the next
    round's are split.  Tolerance as above, over two rounds."""
    pa = require_gpu()
    import torch
    deck, roots = wide_root(5, 8, rnd=4)
    s = pa.SubgameSolver(deck, 4, roots, dtype=pa.PASUR_F64)
    print(f"[values] {[sum(rr.fgt.n) for rr in s.rounds]} nodes, "
          f"{[rr.fgt.n[0] for rr in s.rounds]} roots", flush=True)
    s.solve(2)
    got = [to_np(x) for x in s.exploitability()]
    rounds = oracle_rounds(deck, 4, roots)
    sbars = [[None] + [to_np(t) for t in rr.state.sigma_bar[1:]] for rr in s.rounds]
    want = oracle_exploitability(rounds, sbars)
    K = max(int(np.diff(c).max()) for _, f in rounds for c in f.child_begin())
    for g, w in zip(got, want):
        assert np.max(np.abs(g - w)) <= 2 * 8 * (K + 1) * 2.0 ** -53 * 200
    one = torch.empty(1, dtype=torch.float64, device="cuda")
    pa.exploitability([rr.fgt for rr in s.rounds], [rr.state.sigma_bar for rr in s.rounds],
                      pa.PASUR_F64, None, one, None)
    torch.cuda.synchronize()
    assert float(one[0]) == got[1][0]
    s.free()


def test_values_of_a_large_root_take_more_than_one_compute_unit():
    """2.5e6 nodes below one root: 0.1 ms over the chip, 32 ms in one workgroup."""
    pa = require_gpu()
    import torch
    deck, roots = wide_root(7, 12)
    s = pa.SubgameSolver(deck, 5, roots)
    f = s.rounds[0].fgt
    leaf = torch.empty(f.n[8], dtype=torch.float64, device="cuda")
    pa.leaf_utilities(f, None, pa.PASUR_F64, leaf)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    times = []
    for call in (pa.tree_values, pa.tree_values_noalloc) * 3:
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        call(f, leaf, pa.PASUR_F32, None, pa.TV_MINIMAX, out)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    print(f"[values] {sum(f.n)} nodes: {times} ms", flush=True)
    assert min(times[0::2]) < 4 and min(times[1::2]) < 4
    s.free()
