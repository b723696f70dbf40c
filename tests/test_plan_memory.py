"""Plans and AUTO's calls that get no memory for the segments' far arrays.  The
library's host code runs over a HIP runtime without a device (fake_hip.c)."""
import fake_hip
from test_auto import SETUP


def test_plan_without_memory_for_far_arrays_runs_in_place(tmp_path):
    fake_hip.run("""
        import numpy as np
        import paper_2508_06559_amd as pa
        # one root with 3,000 nodes on each level, 600 active ones on levels 6 and 7
        # with 700 children each: too large for LDS in any form but the one that
        # keeps everything in device memory
        n = 3000
        off = np.tile(np.array([0, n], np.int32), 9)
        counts = np.array([600, 600, 700, 700], np.int32)
        st, g = fake_hip.build_round(fake, L, 1)
        for k in range(31):
            fake.words[k] = 0 if k in (0, 3) else 1 if k < 4 else n
        fake.copy_from, fake.copy_bytes = off.ctypes.data, off.nbytes
        f, r = C.c_void_p(), fake_hip.roots(1)
        assert L.pasur_unfold_scores(g, r, 1, C.byref(f), None) == 0, L.pasur_last_error()
        fake.copy_from, fake.copy_bytes = counts.ctypes.data, counts.nbytes
        one = (C.c_double * 64)()
        s = pa._State()
        for name in ("sigma", "R", "Sbar", "reachA", "reachB", "u"):
            for l in range(9):
                getattr(s, name)[l] = C.addressof(one)
        s.vacc = C.addressof(one)
        p = pa.paper_params(pa.SCHED_ROOT)
        def create():
            h = C.c_void_p()
            fg, sp = (C.c_void_p * 1)(f.value), (C.c_void_p * 1)(C.addressof(s))
            st = L.pasur_plan_create(fg, sp, 1, C.byref(p), 1, 10, C.byref(h), None)
            info = (C.c_int64 * 8)()
            assert st == 0 and L.pasur_plan_forms(h, info) == 0, L.pasur_last_error()
            return h, list(info)
        h, info = create()
        assert info[:5] == [0, 0, 1, 0, 1], info
        assert L.pasur_plan_iterate(C.c_void_p(h.value), 1, 3, None) == 0
        L.pasur_plan_free(h)
        L.pasur_release_cache()
        # the anchor, then the far arrays: none, not even of what is released
        fake.failing_after, fake.failing_mallocs = 1, 2
        h, info = create()
        assert fake.failing_mallocs == 0
        assert info[:5] == [0, 0, 0, 1, 1], info
        launches = fake.launches
        assert L.pasur_plan_iterate(C.c_void_p(h.value), 1, 3, None) == 0
        assert fake.launches == launches + 1
        L.pasur_plan_free(h)
    """, tmp_path)


def test_auto_without_memory_for_segments_streams(tmp_path):
    fake_hip.run(SETUP + """
        assert run(f32, 20, 8) == 0   # segments: their index is there
        segments = fake.launches
        assert run(f32, 20, 8) == 0
        segments = fake.launches - segments
        L.pasur_release_cache()       # (what the calls had has ended)
        fake.failing_mallocs = 2      # scratch of the next call: none
        launches = fake.launches
        assert run(f32, 20, 8) == 0, L.pasur_last_error()
        assert fake.failing_mallocs == 0
        assert fake.launches - launches > 10 * segments   # sweeps, level by level
        assert run(f32, 20, 8) == 0
    """, tmp_path)
