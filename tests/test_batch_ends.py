"""The ends of a batch hold no handle of a tree or a state beyond a call.  The
library's host code runs over a HIP runtime without a device (fake_hip.c)."""
import fake_hip


def test_batch_with_a_freed_tree_is_refused(tmp_path):
    fake_hip.run("""
        import paper_2508_06559_amd as pa
        pa._stream = lambda s=None: None
        one = (C.c_double * 64)()

        class Ptr:
            def data_ptr(self):
                return C.addressof(one)

        class State:
            def __init__(self):
                st, g = fake_hip.build_round(fake, L, 7)
                st, h = fake_hip.unfold(fake, L, g, 7)
                assert st == 0
                self.fgt = pa.UnfoldedTree(h, 5)
                self.c = pa._State()
                for name in ("sigma", "R", "Sbar", "reachA", "reachB", "u"):
                    for l in range(9):
                        getattr(self.c, name)[l] = C.addressof(one)
                self.c.vacc = C.addressof(one)
                self.sb_ptrs = (C.c_void_p * 9)(*[C.addressof(one)] * 9)
                self.t = 1

        states = [State(), State(), State()]
        ends = pa.BatchEnds(states)
        def both():
            ends.begin([None] * 3)
            for st in states:
                st.t = 6
            ends.end([Ptr()] * 3)
        both()
        states[1].t = 5   # sums over five iterations divided by four
        try:
            ends.end([Ptr()] * 3)
            raise SystemExit("different iteration counts accepted")
        except ValueError:
            pass
        states[1].fgt.free()
        launches = fake.launches
        for call in (lambda: ends.begin([None] * 3), both):
            try:
                call()
                raise SystemExit("a freed tree was accepted")
            except pa.PasurError as e:
                assert "item 1 is NULL" in str(e)
        for st in states:
            st.t = 6
        try:
            ends.end([Ptr()] * 3)
            raise SystemExit("a freed tree was accepted")
        except pa.PasurError as e:
            assert "item 1 is NULL" in str(e)
        assert fake.launches == launches
    """, tmp_path)


def test_empty_batch_is_solved(monkeypatch):
    import torch

    import paper_2508_06559_amd as pa
    monkeypatch.setattr(pa.solver, "_torch", lambda: torch)
    b = pa.BatchSolver([], 4, 5)
    b.solve()
    assert b.deals == [] and b.edges() == 0 and b.exploitability() == []
    b.free()
