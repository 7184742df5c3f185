"""No exception leaves the C interface: a failed host allocation is LC_ENOMEM.
In a process of its own whose address space has no room for the tables of a
batch of many grids."""
import subprocess
import sys
import textwrap

CODE = textwrap.dedent("""
    import ctypes, resource, sys
    sys.path.insert(0, {root!r})
    from paper_1907_13415_amd import lc
    n = 2_000_000
    grids = (lc.lc_grid * n)()
    g = lc.make_grid(lc.LC_D2Q9, lc.LC_FP32_DEV, 3, 2, 1)
    ctypes.memmove(grids, ctypes.byref(g), ctypes.sizeof(g))
    for k in (1 << b for b in range(21)):
        ctypes.memmove(ctypes.byref(grids, k * ctypes.sizeof(g)), grids, min(k, n - k) * ctypes.sizeof(g))
    size = ctypes.c_size_t()
    args = (n, grids, ctypes.byref(size), None, None, None, None)
    pages = int(open("/proc/self/statm").read().split()[0])
    limit = resource.getrlimit(resource.RLIMIT_AS)
    resource.setrlimit(resource.RLIMIT_AS, (pages * resource.getpagesize() + (100 << 20), limit[1]))
    rc = lc._lib.lc_batch_layout(*args)
    msg = lc._lib.lc_last_error()
    resource.setrlimit(resource.RLIMIT_AS, limit)
    print(rc, msg)
    assert rc == lc.LC_ENOMEM and msg, (rc, msg)
    assert lc._lib.lc_batch_layout(*args) == lc.LC_OK and size.value >= n * 9 * 6 * 4
""")


def test_failed_host_allocation_is_a_status():
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE.format(root=root)], text=True, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, timeout=300)
    print(r.stdout[-2000:])
    assert r.returncode == 0
