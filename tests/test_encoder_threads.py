"""The host encoder of the local-column row blocks shares its segments (4,096 rows or more) among threads from two
segments on.  A preloaded pthread_create counts the threads that one r3mg_analyze starts: with the blocks of a
local-column shape encoded it starts more of them than without, on a matrix of three segments."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COUNTER = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <pthread.h>
static int made;
int threads_made(void) { return __atomic_load_n(&made, __ATOMIC_SEQ_CST); }
int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* p) {
  __atomic_add_fetch(&made, 1, __ATOMIC_SEQ_CST);
  int (*real)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*) =
      (int (*)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*))dlsym(RTLD_NEXT, "pthread_create");
  return real(t, a, f, p);
}
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
import fixtures as F, paper_2607_28235_amd as P
made = ctypes.CDLL(sys.argv[2]).threads_made
prob = F.structured_qp(3, 12, 2)
assert prob.n == 15625
out = []
for fine in (0, 6):
    o = P.Options(dim=3, coarse_degree=1, leaf_size=256, skip_leaf_level=1, fine_kernel=fine, multi_rhs_kernel=0)
    before = made()
    P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, o, factor=False).close()
    out.append(made() - before)
print("threads", *out)
"""


def test_local_blocks_are_encoded_by_several_threads(tmp_path):
    if (os.cpu_count() or 1) < 2 or len(os.sched_getaffinity(0)) < 2:
        pytest.skip("one processor")
    src, lib = tmp_path / "counter.c", tmp_path / "counter.so"
    src.write_text(COUNTER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib), "-ldl", "-lpthread"], check=True)
    env = dict(os.environ, LD_PRELOAD=(str(lib) + " " + os.environ.get("LD_PRELOAD", "")).strip())
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(lib)], env=env, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    without, encoded = map(int, r.stdout.split("threads", 1)[1].split())
    assert encoded >= without + 2
