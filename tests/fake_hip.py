"""The library's host code without a GPU: libpasur.so over the HIP runtime of
fake_hip.c, in a process of its own."""
import ctypes as C
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Fake(C.Structure):
    """`fake` of fake_hip.c."""
    _fields_ = ([(n, C.c_int) for n in
                 ("free_status", "sync_status", "last_error", "failing_mallocs", "failing_after",
                  "device", "capturing", "pending", "freed_pending", "mallocs", "frees",
                  "host_mallocs", "syncs", "launches", "mallocs_async", "frees_async",
                  "unfinished", "event_waits")] +
                [("free_bytes", C.c_int64 * 2), ("total_bytes", C.c_int64 * 2),
                 ("copy_from", C.c_void_p), ("copy_bytes", C.c_int64),
                 ("words", C.c_int64 * 31), ("in_sync", C.c_void_p), ("in_free", C.c_void_p)])


HOOK = C.CFUNCTYPE(None)


def load(so):
    """(fake, library) in this process; `so` is fake_hip.c built."""
    f = C.CDLL(so, mode=C.RTLD_GLOBAL)
    fake = Fake.in_dll(f, "fake")
    for d in (0, 1):
        fake.free_bytes[d] = fake.total_bytes[d] = 1 << 40
    sys.path.insert(0, ROOT)
    import paper_2508_06559_amd as pa
    return fake, pa.lib()


def roots(n):
    """n entries of the size of pasur_root."""
    return (C.c_byte * (16 * n))()


def build_round(fake, L, n, rnd=5):
    """A handle of a round tree whose levels have n nodes each (and n roots), as
    the kernels would report; (status, handle)."""
    deck = (C.c_uint8 * 52)(*range(52))
    for k in range(31):
        fake.words[k] = n if k else 0
    h = C.c_void_p()
    r = roots(max(n, 1))
    st = L.pasur_build_round_tree(deck, rnd, r, max(n, 1), C.byref(h), None)
    return st, h


def unfold(fake, L, gt, n):
    """A handle of its unfolding, n nodes on each level; (status, handle)."""
    for k in range(31):
        fake.words[k] = 0 if k in (0, 3) else n
    h = C.c_void_p()
    r = roots(max(n, 1))
    st = L.pasur_unfold_scores(gt, r, max(n, 1), C.byref(h), None)
    return st, h


def run(body, tmp_path):
    """Runs `body` with `fake` and the library `L` in a process of its own."""
    so = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")],
                   check=True)
    code = ("import ctypes as C, sys\n"
            f"sys.path.insert(0, {HERE!r})\n"
            "import fake_hip\n"
            f"fake, L = fake_hip.load({so!r})\n" + textwrap.dedent(body))
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
