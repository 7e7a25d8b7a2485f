"""Host code that allocates, sizes and launches, on the CPU: the library runs
in a child process on a stand-in for the HIP runtime (host_runtime.cpp), which
records the launches and can refuse one chosen call."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_over.restype = ctypes.c_char_p
for f in (stub.stub_launches, stub.stub_attributes, stub.stub_seen):
    f.restype = ctypes.c_int64
import numpy as np
from paper_2409_13958_amd import binding as B, meshgen as mg

def context(prob, **kw):
    return B.Context.from_problem(prob, device=0, stream=1, **kw)

def film(nx, ny, nz=1, grid=(16, 16, 4), periodic=0b011):
    return mg.kuhn_box((nx, ny, nz), 1e-9, periodic=periodic, jitter=0.1, grid=grid)

def seen(watch):
    buf = np.zeros(4096, np.uint64)
    return buf[:stub.stub_seen(watch, buf.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(4096))]

def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)

def heff(ctx):
    m, h = np.zeros((ctx.n, 3), np.float32), np.zeros((ctx.n, 3), np.float32)
    return ctx.lib.pmfem_heff(ctx.h, ptr(m), ptr(h), 3, None)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    lib = tmp_path_factory.mktemp("runtime") / "host_runtime.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(HERE, "host_runtime.cpp"), "-o", str(lib)], check=True)
    return str(lib)


def child(runtime, code, *args):
    r = subprocess.run([sys.executable, "-c", PRELUDE + code, runtime, *map(str, args)],
                       cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


# the refused call: every allocation and copy of the workspace in turn
@pytest.mark.parametrize("scheme", ["midpoint", "adaptive"])
@pytest.mark.parametrize("call, nth", [("hipHostGetDevicePointer", 1), ("hipHostMalloc", 1),
                                       ("hipMemcpy", 1)]
                         + [("hipMalloc", k) for k in range(1, 16)])
def test_implicit_workspace_after_a_refused_call(runtime, scheme, call, nth):
    """A step whose workspace could not be set up reports it, and the next one
    sets up what is missing: no kernel is launched with a null buffer."""
    child(runtime, """
scheme, call, nth = sys.argv[2:]
ctx = context(film(4, 4))
m = np.zeros((ctx.n, 3)); m[:, 2] = 1.0

def step(kdim):
    if scheme == "midpoint":
        return ctx.lib.pmfem_llg_implicit(ctx.h, ptr(m), 1e-15, 0.5, 1, 3, None, 1e-8, kdim, None)
    dt = np.array([1e-15])
    return ctx.lib.pmfem_llg_implicit_adaptive(ctx.h, ptr(m), 2e-15, ptr(dt), 0.5, 3, None, 1e-6,
                                               1e-8, kdim, 0, None, None, 0)
watches = [(k, a, stub.stub_watch(k.encode(), a)) for k, a in (
    ("k_mid_point", 1), ("k_mid_point", 2), ("k_mid_point", 4), ("k_mid_point", 5),
    ("k_mid_residual", 1), ("k_mid_residual", 2), ("k_mid_residual", 3), ("k_mid_residual", 4),
    ("k_mid_residual", 5), ("k_mid_residual", 10), ("k_mid_residual", 11), ("k_mid_residual", 12),
    ("k_gs_next", 1), ("k_gs_next", 2), ("k_gs_next", 3), ("k_gs_next", 6), ("k_gs_next", 7),
    ("k_gs_next", 8), ("k_gs_next", 9), ("k_lincomb", 7))]
for kdim in (4, 8):               # a first workspace, then a larger one
    stub.stub_fail(call.encode(), ctypes.c_int64(int(nth)))
    rc = step(kdim)
    refused = stub.stub_failed()
    stub.stub_fail(b"", ctypes.c_int64(0))
    assert rc != 0 if refused else rc == 0
    assert step(4) == 0
    assert step(kdim) == 0
for k, a, w in watches:
    assert len(seen(w)) > 0 or (k, scheme) == ("k_lincomb", "midpoint")
    assert (seen(w) != 0).all(), (k, a)
""", scheme, call, nth)


@pytest.mark.parametrize("p, rb, grid", [
    (1, 0, (5, 7, 5)), (2, 1, (10, 10, 49)), (3, 2, (50, 50, 81)), (4, 1, (18, 18, 16)),
    (5, 1, (14, 14, 14)), (5, 1, (75, 75, 75)), (5, 1, (125, 125, 20)),
])
def test_scatter_tiles_launch_without_an_attribute(runtime, p, rb, grid):
    """The largest footprints of every order, one context's and a batch's, fit
    in the LDS that a launch may have without a function attribute (an
    attribute belongs to the function: one context would set another's)."""
    child(runtime, """
p, rb, *grid = map(int, sys.argv[2:])
ctx = context(film(5, 5, 5, tuple(grid), 0b111), order_p=p, near_boxes=rb)
assert heff(ctx) == 0
b = B.Batch([ctx], stream=1)
m, h = np.zeros((ctx.n, 3), np.float32), np.zeros((ctx.n, 3), np.float32)
assert b.lib.pmfem_batch_heff(b.h, ptr(m), ptr(h), 3) == 0
assert stub.stub_launches(b"k_anterp_scatter") == 2
assert stub.stub_over() == b"", stub.stub_over()
assert stub.stub_attributes(b"k_anterp_scatter") == 0
""", p, rb, *grid)


def test_plane_transforms_of_every_extent_that_fits(runtime):
    """The plane form of the transforms can be asked for wherever the twiddle
    tables and two buffers of a plane's row pairs or columns fit in LDS, and
    nowhere else; it is the automatic choice, alone and in a batch, where they
    also fit at padded strides."""
    child(runtime, """
edge = [(48, 400), (49, 400), (60, 324), (125, 160), (392, 50), (400, 49), (486, 40), (490, 40)]
for nx, ny in edge + [(16, 16), (128, 128), (140, 140), (144, 140), (490, 42), (512, 512)]:
    ctx = context(film(4, 4, 2, (nx, ny, 4)))
    Hx, pairs = nx // 2 + 1, (ny + 1) // 2
    fits = 8 * (nx + ny + 2 * max(pairs * nx, Hx * ny)) <= 160 * 1024
    assert (ctx.lib.pmfem_set_variant(ctx.h, b"fft", 2) == 0) == fits, (nx, ny)
    assert fits or (nx, ny) not in edge
    planes = lambda: stub.stub_launches(b"k_fft_xy_fwd")
    before = planes()
    assert heff(ctx) == 0
    assert planes() - before == int(fits)
    ctx.lib.pmfem_set_variant(ctx.h, b"fft", 0)
    b = B.Batch([ctx], stream=1)
    before = planes()
    assert heff(ctx) == 0
    m = np.zeros((ctx.n, 3), np.float32)
    assert b.lib.pmfem_batch_heff(b.h, ptr(m), ptr(m.copy()), 3) == 0
    assert planes() - before == 2 * int(fits and (nx, ny) not in edge)
    assert stub.stub_over() == b"", stub.stub_over()
""")


def test_an_exception_in_a_parallel_loop_reaches_its_caller(tmp_path):
    """The set-up's loops run on threads that allocate: what one of them throws
    is thrown to the loop's caller (which reports it as a status), once all
    threads have ended, and does not end the process."""
    src = tmp_path / "loop.cpp"
    src.write_text("""
#include "internal.h"
#include <cstdio>
#include <new>
int main() {
  for (int64_t bad : {0, 1, 777, 4095}) {
    std::atomic<int> in(0);
    bool caught = false;
    try {
      pmfem::parallel_for(4096, [&](int64_t i) {
        ++in;
        if (i == bad) { --in; throw std::bad_alloc(); }
        --in;
      }, 1);
    } catch (const std::bad_alloc&) { caught = true; }
    if (!caught || in != 0) return 1;
  }
  std::atomic<int64_t> sum(0);
  pmfem::parallel_for(1001, [&](int64_t i) { sum += i; }, 7);
  return sum == 1001 * 500 ? 0 : 2;
}
""")
    exe = tmp_path / "loop"
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{ROOT}/paper_2409_13958_amd/csrc",
                    f"-I{ROOT}/include", str(src), "-o", str(exe), "-lpthread"], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0


@pytest.mark.parametrize("nth, more", [(k, 1) for k in range(1, 9)] + [(1, 2), (8, 2)])
def test_surrogate_after_refused_training_buffers(runtime, nth, more):
    """A gradient whose buffers are refused leaves the network usable for
    inference and for a later gradient; where even the buffers of inference
    are refused afterwards (more = 2), inference is refused too. No kernel is
    launched with a null buffer."""
    child(runtime, """
nth, more = map(int, sys.argv[2:])
ctx = context(film(4, 4))
ctx.surrogate_init(depth=4)
p, _ = ctx.surrogate_get_params()
ctx.surrogate_set_params(p, scales=(1.0, 1.0))
q = np.zeros(ctx._grid_shape(), np.float32); u = q.copy()
watches = [(k, a, stub.stub_watch(k.encode(), a)) for k, a in (
    ("k_sg_in", 1), ("k_sg_in", 5), ("k_sg_mid", 1), ("k_sg_mid", 4), ("k_sg_out", 1),
    ("k_sg_out", 5), ("k_sg_loss", 4), ("k_sg_wgradE", 4))]
apply = lambda: ctx.lib.pmfem_surrogate_apply(ctx.h, ptr(q), ptr(u))
grad = lambda: ctx.lib.pmfem_surrogate_loss_grad(ctx.h, ptr(q), ptr(u), None, None, 0)
profile = lambda: ctx.lib.pmfem_surrogate_profile(ctx.h, ptr(q), ptr(u), 1, ptr(np.zeros(12)))
stub.stub_fail_run(b"hipMalloc", ctypes.c_int64(nth), ctypes.c_int64(more))
assert grad() != 0
stub.stub_fail(b"", ctypes.c_int64(0))
# the second refused call is the one that would bring inference back
assert (apply() == 0) == (more == 1)
assert (profile() == 0) == (more == 1)
ctx.surrogate_enable(True)
assert (heff(ctx) == 0) == (more == 1)
assert grad() == 0 and apply() == 0 and profile() == 0 and heff(ctx) == 0
for k, a, w in watches:
    assert len(seen(w)) > 0 and (seen(w) != 0).all(), (k, a)
""", nth, more)


@pytest.mark.parametrize("call", ["hipMalloc", "hipMemcpy"])
def test_a_batch_that_could_not_be_set_up_is_refused(runtime, call):
    """Whichever allocation or copy of a batch's set-up is refused, its
    evaluation and steps say so and launch nothing."""
    child(runtime, """
call = sys.argv[2]
cells = [context(film(4, 4)), context(film(5, 4))]
lib = cells[0].lib
arr = (ctypes.c_void_p * 2)(*[c.h for c in cells])
n = sum(c.n for c in cells)
m, m64 = np.zeros((n, 3), np.float32), np.zeros((n, 3))
nth = 0
while True:
    nth += 1
    stub.stub_fail(call.encode(), ctypes.c_int64(nth))
    b = ctypes.c_void_p()
    rc = lib.pmfem_batch_create(ctypes.byref(b), 2, ctypes.cast(arr, ctypes.c_void_p),
                                ctypes.c_void_p(1), 0)
    refused = stub.stub_failed()
    stub.stub_fail(b"", ctypes.c_int64(0))
    if not refused:
        assert rc == 0
        break
    assert rc != 0
    before = stub.stub_launches(b"")
    if b.value:
        assert lib.pmfem_batch_heff(b, ptr(m), ptr(m.copy()), 3) == B.Status.ESTATE, nth
        assert lib.pmfem_batch_llg_step(b, ptr(m64), 1e-15, 0.5, 1) == B.Status.ESTATE, nth
        assert lib.pmfem_batch_llg_step_graph(b, ptr(m64), 1e-15, 0.5, 1) == B.Status.ESTATE, nth
        lib.pmfem_batch_destroy(b)
    assert stub.stub_launches(b"") == before
assert nth > 10     # calls of the set-up were refused
""", call)
