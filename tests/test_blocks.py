"""Device memory that freed trees and plans leave to later ones: it is idle when
it is handed out again, and it is not kept where it is needed.  The library's
host code runs over a HIP runtime without a device (fake_hip.c)."""
import pytest

import fake_hip


def test_blocks_of_a_handle_wait_for_a_failed_free(tmp_path):
    """The wait for the device that comes before a tree's blocks go back is refused,
    as while another thread captures: nobody gets these blocks until it has
    succeeded."""
    fake_hip.run("""
        st, g = fake_hip.build_round(fake, L, 7)
        assert st == 0, L.pasur_last_error()
        fake.pending = 1   # a caller's work on the tree
        fake.free_status = 900
        L.pasur_gt_free(g)
        fake.free_status = 0
        before = fake.mallocs
        fake.pending = 1   # it still runs, and the wait is refused again
        fake.free_status = 900
        st, h = fake_hip.build_round(fake, L, 7)
        assert st == 0
        assert fake.mallocs - before >= 9, fake.mallocs - before
        # once a wait succeeds they are handed out again
        fake.free_status = 0
        L.pasur_gt_free(h)
        before = fake.mallocs
        st, a = fake_hip.build_round(fake, L, 7)
        st, b = fake_hip.build_round(fake, L, 7)
        assert fake.mallocs - before == 2, fake.mallocs - before   # their anchors
    """, tmp_path)


def test_blocks_of_a_plan_wait_for_a_failed_wait(tmp_path):
    """A call whose own wait for the stream fails does not leave its memory to
    others."""
    fake_hip.run("""
        import paper_2508_06559_amd as pa
        st, g = fake_hip.build_round(fake, L, 7)
        st, f = fake_hip.unfold(fake, L, g, 7)
        assert st == 0, L.pasur_last_error()
        one = (C.c_double * 64)()
        s = pa._State()
        for name in ("sigma", "R", "Sbar", "reachA", "reachB", "u"):
            for l in range(9):
                getattr(s, name)[l] = C.addressof(one)
        s.vacc = C.addressof(one)
        p = pa.paper_params(pa.SCHED_ROOT)
        run = lambda: L.pasur_cfr_iterate(f, C.byref(s), C.byref(p), 1, 2, None)
        assert run() == 0
        before = fake.mallocs
        assert run() == 0
        assert fake.mallocs == before   # the first call's memory again
        syncs = [0]
        def fail(): # the second wait, behind the launch, fails
            syncs[0] += 1
            fake.sync_status = 0 if syncs[0] < 2 else 719
        hook = fake_hip.HOOK(fail)
        fake.in_sync = C.cast(hook, C.c_void_p)
        assert run() != 0
        fake.in_sync, fake.sync_status = None, 0
        assert run() == 0
        assert fake.mallocs > before, "memory of the failed call handed out again"
    """, tmp_path)


def test_scan_scratch_is_kept_until_its_scan_has_ended(tmp_path):
    """An error that an earlier, unrelated call left behind comes up in the middle of
    a scan: its scratch does not go back while its kernels may run."""
    fake_hip.run("""
        n = 5000   # more than a tile, so that a scan has scratch
        st, g = fake_hip.build_round(fake, L, n)
        st, f = fake_hip.unfold(fake, L, g, n)
        assert st == 0, L.pasur_last_error()
        L.pasur_release_cache()
        seg, edges = (C.c_int32 * (n + 1))(), (C.c_int32 * n)()
        a, b = C.c_int64(), C.c_int64()
        sample = lambda: L.pasur_sample_parents(f, 8, 1, 0.5, seg, edges, C.byref(a), C.byref(b), None)
        # another thread releases the cache while the call waits
        def release():
            assert not fake.freed_pending
            L.pasur_release_cache()
        hook = fake_hip.HOOK(release)
        fake.pending = fake.freed_pending = 0
        fake.in_sync = C.cast(hook, C.c_void_p)
        fake.last_error = 1
        assert sample() != 0
        assert fake.freed_pending == 0, "scratch given back while its scan is pending"
        fake.in_sync = None
        for k in range(31): fake.words[k] = 1
        assert sample() == 0, L.pasur_last_error()
        assert fake.freed_pending == 0
    """, tmp_path)


def test_build_that_runs_out_of_memory_waits_for_its_kernels(tmp_path):
    """No memory for the first level's scan: the roots' scratch, which the kernel
    before it reads, goes back only after that kernel has ended."""
    fake_hip.run("""
        n = 5000
        fake.failing_after, fake.failing_mallocs = 3, 2   # anchor, scratch, level 0; then none
        st, g = fake_hip.build_round(fake, L, n)
        assert st == -5 and not g.value, L.pasur_last_error()
        assert fake.launches > 0 and fake.failing_mallocs == 0
        assert fake.freed_pending == 0, "memory given back while a kernel is pending"
    """, tmp_path)


def test_anchors_are_allocated_from_released_memory(tmp_path):
    """The device is full but for what the library keeps: it gives that back for a
    handle's anchor too, and a failed allocation leaves no error behind."""
    fake_hip.run("""
        st, g = fake_hip.build_round(fake, L, 7)
        L.pasur_gt_free(g)
        frees = fake.frees
        fake.failing_mallocs = 1
        st, g = fake_hip.build_round(fake, L, 7)
        assert st == 0, L.pasur_last_error()
        assert fake.frees - frees >= 9   # the cached blocks
        fake.failing_mallocs = 2
        st, h = fake_hip.build_round(fake, L, 7)
        assert st == -5 and fake.last_error == 0
    """, tmp_path)


def test_a_block_is_kept_by_what_its_own_device_has_free(tmp_path):
    """A tree of device 0, freed while device 1 is current, and the other way
    round."""
    fake_hip.run("""
        for full, current, kept in ((1, 1, True), (0, 1, False), (1, 0, True)):
            fake.device = 0
            L.pasur_release_cache()
            st, g = fake_hip.build_round(fake, L, 2 << 20)   # blocks of 88 MB
            assert st == 0
            fake.free_bytes[0] = fake.free_bytes[1] = 1 << 40
            fake.free_bytes[full] = 1 << 30
            fake.device = current
            frees = fake.frees
            L.pasur_gt_free(g)
            assert fake.device == current
            assert (fake.frees - frees == 1) == kept, (full, current, fake.frees - frees)
    """, tmp_path)


def test_frees_do_not_hold_up_other_threads(tmp_path):
    """A free waits for the device: meanwhile other threads allocate, free and
    release."""
    fake_hip.run("""
        import threading
        done = []
        def other():
            st, g = fake_hip.build_round(fake, L, 7)
            L.pasur_gt_free(g)
            L.pasur_release_cache()
            done.append(st)
        def hook():
            fake.in_free = None
            t = threading.Thread(target=other, daemon=True)
            t.start()
            t.join(10)
        h = fake_hip.HOOK(hook)
        def in_next_free(f):
            del done[:]
            fake.in_free = C.cast(h, C.c_void_p)
            f()
            assert done == [0], "a free held the lock"
        st, g = fake_hip.build_round(fake, L, 7)
        L.pasur_gt_free(g)
        in_next_free(L.pasur_release_cache)
        # no room: the block itself is freed
        st, g = fake_hip.build_round(fake, L, 2 << 20)
        def full():   # the anchor's wait is over: the next free is a block's
            fake.free_bytes[0] = 0
            fake.in_free = C.cast(h, C.c_void_p)
        first = fake_hip.HOOK(full)
        del done[:]
        fake.in_free = C.cast(first, C.c_void_p)
        L.pasur_gt_free(g)
        assert done == [0], "a block's free held the lock"
    """, tmp_path)


def test_tensors_are_allocated_from_released_memory(monkeypatch):
    """The package's tensors find no room while the library keeps freed trees'
    memory: it is given back, and the allocation tried again, once."""
    import torch

    import paper_2508_06559_amd as pa
    log = []

    room = [False]

    def empty(shape, dtype, device):
        log.append("empty")
        if not room[0]:
            raise torch.OutOfMemoryError("full")
        return (shape, dtype, device)

    def release():
        log.append("release")
        room[0] = True

    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(pa, "release_cache", release)
    for allocate in (lambda: pa.device_empty(3, torch.int8),
                     lambda: pa.on_device(lambda: torch.empty(3, dtype=torch.int8, device="cuda"))):
        room[0] = False
        assert allocate() == (3, torch.int8, "cuda")
        assert log == ["empty", "release", "empty"]
        del log[:]
    room[0] = False
    monkeypatch.setattr(pa, "release_cache", lambda: log.append("release"))
    with pytest.raises(torch.OutOfMemoryError):
        pa.device_empty(3, torch.int8)
    assert log == ["empty", "release", "empty"]
