"""Calls that find less memory than they would like: without pinned blocks they
take pageable memory, without device memory for the trajectories side by side
they run fewer at a time, and the results are the same.

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
typedef int (*free_fn)(void*, void*);
static host_fn real_host;
static dev_fn real_dev;
static free_fn real_free;
int refuse_host = 0, refused = 0;
size_t most = ~(size_t)0; /* bytes allocated in stream order at a time */
static size_t live, size_of[1024];
static void* ptr_of[1024];
void setup(const char* path) {
  void* h = dlopen(path, RTLD_NOW);
  real_host = (host_fn)dlsym(h, "hipHostMalloc");
  real_dev = (dev_fn)dlsym(h, "hipMallocAsync");
  real_free = (free_fn)dlsym(h, "hipFreeAsync");
}
int hipHostMalloc(void** p, size_t n, unsigned flags) {
  if (!refuse_host) return real_host(p, n, flags);
  ++refused;
  return real_host(NULL, n, flags); /* an error of the runtime's own, which it remembers */
}
int hipMallocAsync(void** p, size_t n, void* s) {
  if (n > most || live > most - n) {
    ++refused;
    real_host(NULL, n, 0); /* as above */
    return 2;              /* out of memory */
  }
  const int r = real_dev(p, n, s);
  for (int i = 0; r == 0 && i < 1024; ++i)
    if (!ptr_of[i]) {
      ptr_of[i] = *p;
      size_of[i] = n;
      live += n;
      break;
    }
  return r;
}
int hipFreeAsync(void* p, void* s) {
  for (int i = 0; p && i < 1024; ++i)
    if (ptr_of[i] == p) {
      ptr_of[i] = NULL;
      live -= size_of[i];
      break;
    }
  return real_free(p, s);
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


# d = 5: four registers fit and the tables beside them do not; d = 4 (also with
# two registers each: the predicted passes): room for some of the registers;
# d <= 3: for some of the results
@pytest.mark.parametrize("mib,kw", [
    (1024, dict(d=5, rounds=2, n_traj=4, dtype="c64")),
    (40, dict(d=4, rounds=2, n_traj=150, dtype="c64", zeta=0.01)),
    (40, dict(d=4, rounds=2, n_traj=60, dtype="c64", zeta=0.0)),
    (6, dict(d=3, rounds=2, n_traj=2000, dtype="c128", zeta=0.01, want_states=True)),
])
def test_short_device_memory(tmp_path, mib, kw):
    print(f"case short device memory {mib} {kw}", flush=True)
    _run(tmp_path, f"""
        kw = dict(gateset="cr", seed=3, p=0.02, eps=0.02, **{kw!r})
        most.value = {mib} << 20
        a = qs.run_rounds(**kw)
        assert refused.value > 0
        n = refused.value
        most.value = 1 << 40
        assert same(a, qs.run_rounds(**kw)) and refused.value == n
    """)


def test_small_runs_stay_within_their_limit(tmp_path):
    """Ten million d = 2 trajectories of one round: seven bytes of results each
    and 32 of parameters, 256 MiB at a time and 1 MiB for the tables."""
    print("case limit of small runs", flush=True)
    _run(tmp_path, """
        most.value = 257 << 20
        a = qs.run_rounds(d=2, gateset="cr", rounds=1, n_traj=10_000_000, seed=3, p=0.02, eps=0.02, dtype="c64")
        assert refused.value == 0
        n = 8_000_000
        b = qs.run_rounds(d=2, gateset="cr", rounds=1, n_traj=1000, seed=3, p=0.02, eps=0.02, dtype="c64", traj0=n)
        assert np.array_equal(a["records"][n:n + 1000], b["records"])
        assert np.array_equal(a["final_bits"][n:n + 1000], b["final_bits"])
    """)
