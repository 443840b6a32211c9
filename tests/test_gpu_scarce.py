"""Calls that find less memory than they would like: without pinned blocks they
take pageable memory, and the results are the same.

A small library in front of the HIP runtime refuses the allocation; the call
runs in a process of its own, which loads it before the simulator."""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FRONT = r"""
#include <dlfcn.h>
#include <stddef.h>
typedef int (*host_fn)(void**, size_t, unsigned);
typedef int (*dev_fn)(void**, size_t, void*);
static host_fn real_host;
static dev_fn real_dev;
int refuse_host = 0, refused = 0;
size_t most = ~(size_t)0;
void setup(const char* path) {
  void* h = dlopen(path, RTLD_NOW);
  real_host = (host_fn)dlsym(h, "hipHostMalloc");
  real_dev = (dev_fn)dlsym(h, "hipMallocAsync");
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  if (!refuse_host) return real_host(p, n, flags);
  ++refused;
  return real_host(NULL, n, flags); /* an error of the runtime's own, which it remembers */
}
int hipMallocAsync(void** p, size_t n, void* s) {
  if (n <= most) return real_dev(p, n, s);
  ++refused;
  real_host(NULL, n, 0); /* as above */
  return 2; /* out of memory */
}
"""

HEAD = """
import ctypes, sys
import numpy as np
import torch
torch.zeros(1, device="cuda")
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
front = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
front.setup(path.encode())
sys.path.insert(0, sys.argv[2])
import paper_2204_11404_amd as qs
refuse_host = ctypes.c_int.in_dll(front, "refuse_host")
refused = ctypes.c_int.in_dll(front, "refused")
most = ctypes.c_size_t.in_dll(front, "most")
same = lambda a, b: all((a[k] is None and b[k] is None) or np.array_equal(a[k], b[k]) for k in a
                        if k in ("records", "final_bits", "p1", "states"))
"""


def _run(tmp_path, body):
    src, so = tmp_path / "front.c", tmp_path / "front.so"
    src.write_text(FRONT)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(so), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(body), str(so), ROOT], capture_output=True,
                       text=True, timeout=110)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_no_pinned_block(tmp_path):
    print("case no pinned block", flush=True)
    _run(tmp_path, """
        kw = dict(d=3, gateset="cr", rounds=2, n_traj=5, seed=3, p=0.02, eps=0.02, dtype="c128", want_p1=True)
        refuse_host.value = 1
        a = qs.run_rounds(**kw)
        assert refused.value > 0
        refuse_host.value = 0
        assert same(a, qs.run_rounds(**kw))
    """)
