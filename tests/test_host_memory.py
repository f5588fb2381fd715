"""Host memory that runs out at a C entry is PHUB_ENOMEM, not a C++ exception
through it (CPU; in a process of its own with a limited address space)."""

import subprocess
import sys
import textwrap

CODE = textwrap.dedent("""
    import ctypes, resource, numpy as np
    from paper_1805_07891_amd import phub
    lib = phub.Library().lib
    keys = np.zeros(1 << 26, np.int64)  # empty keys: no memory of their own
    grads = (ctypes.c_void_p * 1)()
    used = int(open('/proc/self/statm').read().split()[0]) * resource.getpagesize()
    resource.setrlimit(resource.RLIMIT_AS, (used + (256 << 20),) * 2)
    rc = lib.phub_step_noalloc(1, len(keys), keys.ctypes.data, 32768, 0.1, 0.9, 0.0, 1,
                               ctypes.addressof(grads), None, None, None)
    print(rc, phub.PHUB_ENOMEM)
""")


def test_noalloc_reports_host_memory():
    out = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    got, want = out.stdout.split()
    assert got == want
