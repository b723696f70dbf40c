"""PASUR_SCHED_AUTO on large rounds: its calls enqueue work and wait for nothing,
and can be captured once a tree's index is there.  The library's host code runs
over a HIP runtime without a device (fake_hip.c)."""
import fake_hip

SETUP = """
        import paper_2508_06559_amd as pa
        n = 1000001   # nodes per level, 9e6 in all, as many roots
        st, g = fake_hip.build_round(fake, L, n)
        st, f = fake_hip.unfold(fake, L, g, n)
        assert st == 0, L.pasur_last_error()
        L.pasur_gt_free(g)
        one = (C.c_double * 64)()
        def state(dtype):
            s = pa._State()
            s.dtype = dtype
            for name in ("sigma", "R", "Sbar", "reachA", "reachB", "u"):
                for l in range(9):
                    getattr(s, name)[l] = C.addressof(one)
            s.vacc = C.addressof(one)
            return s
        f32, f64 = state(pa.PASUR_F32), state(pa.PASUR_F64)
        def run(s, iters, stream=0, sched=pa.SCHED_AUTO):
            p = pa.paper_params(sched)
            return L.pasur_cfr_iterate(f, C.byref(s), C.byref(p), 1, iters, C.c_void_p(stream))
"""


def test_auto_only_enqueues_on_large_rounds(tmp_path):
    fake_hip.run(SETUP + """
        assert run(f32, 20) == 0, L.pasur_last_error()
        syncs, mallocs = fake.syncs, fake.mallocs
        assert run(f32, 20) == 0 and run(f64, 300) == 0 and run(f32, 20) == 0
        assert fake.syncs == syncs
        fake.pending = 0
    """, tmp_path)


def test_auto_is_captured_after_any_call_on_the_tree(tmp_path):
    """Whatever that call's state type and iterations: a capture may neither wait
    nor allocate."""
    for first in ("f32, 20", "f64, 20", "f32, 2", "f64, 2"):
        fake_hip.run(SETUP + f"""
        assert run({first}) == 0, L.pasur_last_error()
        fake.capturing = 1
        syncs, mallocs, launches = fake.syncs, fake.mallocs, fake.launches
        for s in (f32, f64):
            for iters in (2, 20, 300):
                assert run(s, iters, 8) == 0, L.pasur_last_error()
                assert (fake.syncs, fake.mallocs) == (syncs, mallocs), (s.dtype, iters)
        assert fake.launches > launches
        assert fake.mallocs_async == fake.frees_async
        fake.capturing = 0
        """, tmp_path)


def test_scratch_of_enqueued_calls_is_not_shared(tmp_path):
    """A later call on the same stream follows the first one; a call on another
    stream has scratch of its own until the first one's work has ended."""
    fake_hip.run(SETUP + """
        assert run(f32, 20, 8) == 0
        fake.unfinished = 1
        assert run(f32, 20, 8) == 0    # the first call's scratch has come from the cache
        mallocs, waits = fake.mallocs, fake.event_waits
        for _ in range(5):
            assert run(f32, 20, 8) == 0
        assert fake.mallocs == mallocs and fake.event_waits == waits + 5
        assert run(f32, 20, 16) == 0
        assert fake.mallocs == mallocs + 1
        assert run(f32, 20, 16) == 0 and run(f32, 20, 8) == 0
        assert fake.mallocs == mallocs + 1
        fake.unfinished = 0            # all have ended: any stream may have either
        waits = fake.event_waits
        assert run(f32, 20, 24) == 0
        assert fake.mallocs == mallocs + 1 and fake.event_waits == waits
        L.pasur_fgt_free(f)
    """, tmp_path)
