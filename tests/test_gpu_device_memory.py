"""Device memory and streams: what a handle or a group solve holds, and what a handle does where the memory for an
optional copy is not to be had.

Each check runs in a child process whose hipMalloc, hipFree and hipStreamCreateWithFlags pass through a preloaded
recorder: it counts the live allocations of a given size and the streams made, and refuses chosen sizes
(hipErrorOutOfMemory, as the runtime answers), so that nothing depends on how much memory the card has left.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORDER = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <link.h>
#include <pthread.h>
#include <stddef.h>
#include <stdlib.h>
#include <string.h>
#define SLOTS 65536
static void* at[SLOTS];
static size_t size[SLOTS], refuse[16];
static int used, nrefuse, refused;
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static int runtime(struct dl_phdr_info* i, size_t n, void* path) {
  (void)n;
  if (!i->dlpi_name || !strstr(i->dlpi_name, "libamdhip64.so")) return 0;
  *(const char**)path = i->dlpi_name;
  return 1;
}
static void* real_of(const char* name) {  /* the loaded HIP runtime's own function */
  const char* path = 0;
  dl_iterate_phdr(runtime, &path);
  void* lib = path ? dlopen(path, RTLD_NOLOAD | RTLD_LAZY) : 0;
  void* f = lib ? dlsym(lib, name) : 0;
  if (!f) exit(3);
  return f;
}
void rec_refuse(size_t n) { refuse[nrefuse++] = n; }
void rec_allow(void) { nrefuse = 0; }
int rec_refused(void) { return refused; }
int rec_live(size_t n) {
  int c = 0;
  for (int i = 0; i < used; ++i) c += at[i] && size[i] == n;
  return c;
}
int hipMalloc(void** p, size_t n) {
  int (*real)(void**, size_t) = (int (*)(void**, size_t))real_of("hipMalloc");
  for (int i = 0; i < nrefuse; ++i)
    if (refuse[i] == n) {
      ++refused;
      return 2;
    }
  int rc = real(p, n);
  pthread_mutex_lock(&mu);
  int i = 0;
  while (i < used && at[i]) ++i;
  if (rc == 0 && i < SLOTS) {
    at[i] = *p;
    size[i] = n;
    if (i == used) ++used;
  }
  pthread_mutex_unlock(&mu);
  return rc;
}
static size_t left;
void rec_left(size_t n) { left = n; }  /* what hipMemGetInfo says is left; 0: the truth */
int hipMemGetInfo(size_t* f, size_t* t) {
  int (*real)(size_t*, size_t*) = (int (*)(size_t*, size_t*))real_of("hipMemGetInfo");
  int rc = real(f, t);
  if (left) *f = left;
  return rc;
}
static int streams;
int rec_streams(void) { return streams; }
int hipStreamCreateWithFlags(void** s, unsigned flags) {
  int (*real)(void**, unsigned) = (int (*)(void**, unsigned))real_of("hipStreamCreateWithFlags");
  ++streams;
  return real(s, flags);
}
int hipFree(void* p) {
  int (*real)(void*) = (int (*)(void*))real_of("hipFree");
  pthread_mutex_lock(&mu);
  for (int i = 0; p && i < used; ++i)
    if (at[i] == p) at[i] = 0;
  pthread_mutex_unlock(&mu);
  return real(p);
}
"""

PRELUDE = r"""
import ctypes, dataclasses, sys
sys.path.insert(0, sys.argv[1])
import numpy as np, torch
import fixtures as F
import paper_2607_28235_amd as P
rec = ctypes.CDLL(sys.argv[2])
rec.rec_refuse.argtypes = rec.rec_live.argtypes = rec.rec_left.argtypes = [ctypes.c_size_t]
torch.zeros(1, device="cuda")

def problem(d, N, p):
    prob = F.structured_qp(d, N, p, jitter=0.2 if d == 2 else 0.0, cfg=2)
    prob.chunks = int(np.sum((np.diff(prob.row_ptr) + 3) // 4))
    return prob

def handle(prob, **kw):
    o = P.Options(dim=prob.d, coarse_degree=1, leaf_size=64 if prob.d == 2 else 150, max_coarse_dofs=600,
                  skip_leaf_level=int(prob.d == 3))
    return P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, dataclasses.replace(o, **kw))

def solve(h, prob, nr=1, seed=1):
    b = np.random.default_rng(seed).standard_normal((nr, prob.n))
    b[:, prob.boundary] = 0.0
    b = torch.from_numpy(b if nr > 1 else b[0]).cuda()
    x = torch.zeros_like(b)
    it, _, ok = h.pcg(b, x, rtol=1e-10, maxit=300)
    assert ok
    return x.cpu().numpy()

def refuse(*sizes):
    for n in sizes:
        rec.rec_refuse(n)
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = tmp_path_factory.mktemp("recorder")
    (d / "rec.c").write_text(RECORDER)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(d / "rec.c"), "-o", str(d / "rec.so"), "-ldl", "-lpthread"],
                   check=True)
    return str(d / "rec.so")


def _child(recorder, body, tune):
    env = dict(os.environ, LD_PRELOAD=(recorder + " " + os.environ.get("LD_PRELOAD", "")).strip(),
               R3MG_TUNE_CACHE=str(tune))
    r = subprocess.run([sys.executable, "-u", "-c", PRELUDE + body, ROOT, recorder], env=env, capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-3000:]
    return r.stdout


def test_recorder_sees_the_library(recorder, tmp_path):
    print("[gpu-case] recorder", flush=True)
    _child(recorder, r"""
prob = problem(2, 24, 3)
h = handle(prob, fine_kernel=0)
assert rec.rec_live(4 * (prob.n + 1)) >= 1          # row pointers
h.close()
assert rec.rec_live(4 * (prob.n + 1)) == 0
""", tmp_path / "tune")


# the arrays refused at set-up: chunked values in float32, in float64, the positions, everything
@pytest.mark.parametrize("what", ["16", "32", "4", "4, 16, 32"])
@pytest.mark.parametrize("fp32", [0, 1])
def test_setup_without_room_for_the_chunked_matrix(recorder, what, fp32, tmp_path):
    """Without room for a chunked copy the fine level takes CSR shape 0, which gives bitwise the same solution; the
    choice is not written to the tuning cache, and a cached chunk choice falls back likewise."""
    print(f"[gpu-case] no room for {what} bytes a chunk, fp32={fp32}", flush=True)
    tune = tmp_path / "tune"
    _child(recorder, rf"""
fp32, what = {fp32}, [{what}]
prob = problem(3, 10, 2)
ref = handle(prob, fine_kernel=0, vcycle_fp32=fp32, tune_cache=0)
want = solve(ref, prob)
hit = any(w in (4, 16 if fp32 else 32, 32) for w in what)
refuse(*[w * prob.chunks for w in what])
for known in (0, 1):
    if known:                                        # a cached choice of the chunk shape for both operators
        rec.rec_allow()
        h = handle(prob, vcycle_fp32=fp32)
        h.close()
        keys = sorted({{ln.rsplit(" ", 1)[0] for ln in open({str(tune)!r}) if "/fine1/" in ln}})
        open({str(tune)!r}, "a").writelines(f"{{k}} 1414\n" for k in keys)
        refuse(*[w * prob.chunks for w in what])
    before = rec.rec_refused()
    h = handle(prob, vcycle_fp32=fp32)
    assert (rec.rec_refused() > before) == hit
    if hit and not known:
        assert "/fine1/" not in (open({str(tune)!r}).read() if __import__("os").path.exists({str(tune)!r}) else "")
    if 4 in what or (16 if fp32 else 32) in what:
        assert h.info()[0]["kernel"].startswith("k_level_stream<"), h.info()[0]["kernel"]
    assert np.array_equal(solve(h, prob), want)
    h.update_values(torch.from_numpy(2.0 * prob.val).cuda())
    assert np.linalg.norm(2.0 * solve(h, prob) - want) <= 1e-8 * np.linalg.norm(want)
    h.close()
""", tune)


@pytest.mark.parametrize("fp32", [0, 1])
def test_block_solve_without_room_for_the_chunked_matrix(recorder, fp32, tmp_path):
    """The first block solve without room for the block lists, or for either precision's values, takes the kernels over
    the CSR arrays; a later one with room works as well."""
    print(f"[gpu-case] block solve without room, fp32={fp32}", flush=True)
    _child(recorder, rf"""
prob = problem(3, 10, 2)
ref = handle(prob, fine_kernel=0, multi_rhs_kernel=3, vcycle_fp32={fp32}, tune_cache=0)
want = solve(ref, prob, 4)
for what in ([4], [16], [32], [4, 16, 32]):
    h = handle(prob, fine_kernel=0, vcycle_fp32={fp32}, tune_cache=0)
    before = rec.rec_refused()
    refuse(*[w * prob.chunks for w in what])
    x = solve(h, prob, 4)
    assert (rec.rec_refused() > before) == (what != [16] or {fp32})
    rec.rec_allow()
    assert np.linalg.norm(x - want) <= 1e-9 * np.linalg.norm(want)
    assert np.linalg.norm(solve(h, prob, 8)[:4] - solve(ref, prob, 8)[:4]) <= 1e-9 * np.linalg.norm(want)
    assert np.linalg.norm(solve(h, prob, 4) - want) <= 1e-9 * np.linalg.norm(want)
    h.close()
""", tmp_path / "tune")


def test_rejected_chunk_copies_are_given_back(recorder, tmp_path):
    """No chunk array stays with a handle whose choices read none: shape 0 for one column and the column-split kernel
    for several, from the tuning cache or timed (where the timing picks it)."""
    print("[gpu-case] rejected chunk copies", flush=True)
    tune = str(tmp_path / "tune")
    _child(recorder, rf"""
prob = problem(2, 40, 2)
def held():
    return sum(rec.rec_live(w * prob.chunks) for w in (1, 4, 16, 32))
assert held() == 0
h = handle(prob, vcycle_fp32=1)
solve(h, prob, 8)
h.close()
assert held() == 0
lines = [ln.split() for ln in open({tune!r})]
keys = sorted({{k for k, v in lines if "/fine1/" in k}})
open({tune!r}, "a").writelines(f"{{k}} 0\n" for k in keys)
h = handle(prob, vcycle_fp32=1)
assert h.info()[0]["kernel"].startswith("k_level_stream<")
assert held() == 0
split = {{k: 208 for k, v in lines if "/mr/0/" in k or "/mr/-1/" in k}}
open({tune!r}, "a").writelines(f"{{k}} {{v}}\n" for k, v in split.items())
solve(h, prob, 8)
assert held() == 0
h.close()
# timed: copies only where the choice is a chunk kernel
h = handle(prob, vcycle_fp32=1, tune_cache=1)
for nr in (2, 4, 16):
    solve(h, prob, nr)
lines = [ln.split() for ln in open({tune!r})]
if not any(int(v) >= 400 for k, v in lines if "/mr/0/" in k or "/mr/-1/" in k):
    assert held() == 0
h.close()
""", tmp_path / "tune")


@pytest.mark.parametrize("fp32", [0, 1])
def test_setup_scratch_stays_only_with_handles_that_are_set_up_again(recorder, fp32, tmp_path):
    """r3mg_factor gives back the dense factorisation's two n x n arrays, the Lanczos vectors and the partial Galerkin
    blocks; they come with the first r3mg_update_values and stay for the next one."""
    print(f"[gpu-case] set-up scratch, fp32={fp32}", flush=True)
    _child(recorder, rf"""
prob = problem(2, 40, 3)
h = handle(prob, vcycle_fp32={fp32}, max_coarse_dofs=1200)
nc = h.info()[-1]["n"]
dense, lanczos = 8 * nc * nc, 5 * 8 * prob.n
def counts():
    return rec.rec_live(dense), rec.rec_live(lanczos)
assert nc > 300 and counts() == (1, 0), counts()     # the inverse alone
want = solve(h, prob)
for rep in range(3):
    h.update_values(torch.from_numpy(prob.val).cuda())
    assert counts() == (3, 1), counts()
assert np.array_equal(solve(h, prob), want)
h.close()
assert counts() == (0, 0)
""", tmp_path / "tune")


# (cells, p', levels, fp32, whether the packed inverse is read): two-level float64 up to 1,024 unknowns reads the rows of the
# full inverse, and forms no packed one
@pytest.mark.parametrize("N,pc,levels,fp32,packed", [(48, 1, 2, 0, 0), (48, 1, 2, 1, 1), (32, 2, 2, 0, 1), (48, 1, 3, 0, 1)])
def test_packed_coarsest_inverse_only_where_it_is_read(recorder, N, pc, levels, fp32, packed, tmp_path):
    print(f"[gpu-case] packed inverse N={N} p'={pc} levels={levels} fp32={fp32}", flush=True)
    _child(recorder, rf"""
prob = problem(2, {N}, 2)
h = handle(prob, coarse_degree={pc}, leaf_size={40 if N == 48 else 64}, max_coarse_dofs=3000 if {levels} == 2 else 300,
           max_levels={levels}, vcycle_fp32={fp32})
assert h.nlevels == {levels}
nt = -(-h.info()[-1]["n"] // 64)
size = nt * (nt + 1) // 2 * 64 * 64 * (4 if {fp32} else 8)
assert rec.rec_live(size) == {packed}
solve(h, prob)
solve(h, prob, 4)
""", tmp_path / "tune")


def test_group_solves_keep_a_bounded_number_of_streams(recorder, tmp_path):
    """Twelve problems share eight streams, which every later group solve reuses, with the solutions of single solves."""
    print("[gpu-case] streams of a group solve", flush=True)
    _child(recorder, r"""
probs = [problem(3, n, 2) for n in (5, 6, 7, 8, 5, 6, 7, 8, 5, 6, 7, 8)]
hs = [handle(p, use_graph=0, tune_cache=0, vcycle_fp32=k % 2) for k, p in enumerate(probs)]
bs = [torch.from_numpy(np.where(p.boundary, 0.0, np.random.default_rng(1).standard_normal((1, p.n))[0])).cuda()
      for p in probs]
before = rec.rec_streams()
for rtol in (1e-6, 1e-10, 1e-10):
    xs = [torch.zeros_like(b) for b in bs]
    it, rr, ok = P.solve_group(hs, bs, xs, rtol=rtol, maxit=100)
    assert ok and rec.rec_streams() - before == 8, rec.rec_streams() - before
for p, h, x in zip(probs, hs, xs):
    assert np.array_equal(solve(h, p), x.cpu().numpy())
""", tmp_path / "tune")


@pytest.mark.parametrize("fp32", [0, 1])
def test_chunked_values_leave_room_for_a_solve(recorder, fp32, tmp_path):
    """A chunked copy that leaves less than a one-column solve's vectors is not taken, from the tuning cache or not."""
    print(f"[gpu-case] room for a solve, fp32={fp32}", flush=True)
    _child(recorder, rf"""
prob = problem(3, 10, 2)
want = solve(handle(prob, fine_kernel=0, vcycle_fp32={fp32}, tune_cache=0), prob)
held = lambda: sum(rec.rec_live(w * prob.chunks) for w in (4, 16, 32))
assert held() == 0
for known in (0, 1):
    for left, kept in ((64 * prob.n - 1, False), (64 * prob.n, True)):
        rec.rec_left(left)
        h = handle(prob, vcycle_fp32={fp32}, tune_cache=known)
        rec.rec_left(0)
        chunk = h.info()[0]["kernel"].startswith("k_level_chunk<")
        assert chunk == (held() > 0) and (kept or not chunk)
        assert np.array_equal(solve(h, prob), want)
        h.close()
    h = handle(prob, vcycle_fp32={fp32})                 # fills the cache
    assert h.info()[0]["kernel"].startswith("k_level_chunk<")
    h.close()
""", tmp_path / "tune")


# what is refused at 16 columns: PCG's vectors, the V-cycle's of the fine level, PCG's partial sums
@pytest.mark.parametrize("what", ["pcg", "level", "partials"])
@pytest.mark.parametrize("fp32", [0, 1])
def test_smaller_solve_after_a_block_solve_without_memory(recorder, what, fp32, tmp_path):
    """A block solve whose vectors find no device memory says so; afterwards solves that fit give bitwise what they gave
    before it, and the block solve works once there is room."""
    print(f"[gpu-case] block solve without memory: {what}, fp32={fp32}", flush=True)
    _child(recorder, rf"""
prob = problem(2, 24, 3)
opt = dict(fine_kernel=0, vcycle_fp32={fp32})     # the first handle's timed choices, by way of the tuning cache
ref = handle(prob, **opt)
want = {{nr: solve(ref, prob, nr) for nr in (1, 4, 16)}}
h = handle(prob, **opt)
for nr in (1, 4):
    assert np.array_equal(solve(h, prob, nr), want[nr])
refuse(dict(pcg=8 * 16 * prob.n, level={4 if fp32 else 8} * 16 * prob.n, partials=8 * 1024 * 2 * 16)["{what}"])
for rep in range(2):
    before = rec.rec_refused()
    try:
        solve(h, prob, 16)
        assert False, "solved without memory"
    except P.R3mgError as e:
        assert "hipMalloc" in str(e), e
    assert rec.rec_refused() > before
    for nr in (1, 4, 1):
        assert np.array_equal(solve(h, prob, nr), want[nr]), nr
rec.rec_allow()
for nr in (16, 4, 1):
    assert np.array_equal(solve(h, prob, nr), want[nr]), nr
h.close()
""", tmp_path / "tune")
