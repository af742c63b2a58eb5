"""Which compiled form of the one-launch CG chunks (csrc/cg_grid.hip) runs, asked of
the library, and that it ran: every form against the launch-per-phase iterations,
and the states a solve can find its chunks in."""
import numpy as np
import pytest

import basin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NU = (1e3, 1e-2)
DT = 3600.0


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1207_0486_amd import hns  # noqa: F401
    return torch.device("cuda", 0)


def _operator(m, bit, keep_fp32=False):
    from paper_1207_0486_amd.hns import Operator
    op = Operator(m, NU[0], NU[1], DT, kind="poisson" if bit < 0 else "helmholtz",
                  keep_fp32=keep_fp32, gpu_assembly=True)
    op.set_param("small_n", 0)
    return op


def _rhs(m, bit, seed, dev):
    d = None if bit < 0 else ((m.bc >> bit) & 1) == 1
    b = basin.normal_rhs(m.n, seed, zero_mean=bit < 0, dirichlet=d)
    return torch.as_tensor(b, device=dev)


def _rel(x, y):
    return float((x - y).norm() / y.norm())


# values of a row that a form moves through memory per iteration, by rows per
# thread (FP64): lower diagonals beyond those kept on chip, and x twice
STREAMED = {1: 0, 2: 0, 4: 0, 6: 2, 8: 5, 12: 11}

# rows per thread of the form that 256 CUs take, in FP64 and FP32
FORMS = [((30, 28, 7), 1, 1), ((61, 47, 13), 2, 2), ((90, 80, 11), 4, 4), ((180, 190, 21), 6, 8),
         ((240, 189, 17), 8, 8), ((237, 192, 18), 8, 8), ((250, 200, 22), 12, 12)]


@pytest.mark.parametrize("grid, rows64, rows32", FORMS,
                         ids=["x".join(map(str, g)) for g, _, _ in FORMS])
def test_the_expected_form_runs_and_equals_the_launches(dev, grid, rows64, rows32):
    """40 FP64 iterations equal those of a launch per phase to rounding (the dot
    products' order differs); a mixed velocity solve meets its tolerance in the
    same number of iterations."""
    if torch.cuda.get_device_properties(dev).multi_processor_count != 256:
        pytest.skip("tilings of 256 CUs")
    m = basin.basin_mesh(*grid, seed=5)
    b = _rhs(m, -1, 21, dev)
    op = _operator(m, -1)
    assert op.one_launch_info()["workgroups"] == 0          # nothing planned yet
    xs = {}
    for one in (0, -1):
        op.set_param("one_launch", one)
        xs[one], info = op.solve(b, tol=1e-12, max_iter=40, check=False)
        assert info.iterations == 40
        assert (op.one_launch_info()["chunks"] > 0) == (one == -1)
    got = op.one_launch_info()
    assert got["rows_per_thread"] == rows64 and got["missed"] == 0
    assert got["streamed"] == STREAMED[rows64]
    op.close()
    assert _rel(xs[-1], xs[0]) <= 1e-11
    b = _rhs(m, 1, 22, dev)
    op = _operator(m, 1, keep_fp32=True)
    it = {}
    for one in (0, -1):
        op.set_param("one_launch", one)
        x, info = op.solve(b, tol=1e-11, mask_bit=1, mode="mixed")
        assert info.status == 0 and info.relres_true <= 1e-11
        it[one] = info.iterations
        assert (op.one_launch_info("mixed")["chunks"] > 0) == (one == -1)
    got = op.one_launch_info("mixed")
    assert got["rows_per_thread"] == rows32 and got["missed"] == 0
    assert op.one_launch_info()["chunks"] == 0              # FP64 chunks: none in a mixed solve
    op.close()
    assert abs(it[-1] - it[0]) <= 1


def test_a_missed_meeting_is_counted(dev):
    m = basin.basin_mesh(40, 36, 6, seed=5)
    for mode in ("fp64", "mixed"):
        b = _rhs(m, 1, 41, dev)
        op = _operator(m, 1, keep_fp32=True)
        op.set_param("meet_polls", 0)
        x, info = op.solve(b, tol=1e-10, mask_bit=1, mode=mode)
        got = op.one_launch_info(mode)
        op.close()
        assert info.status == 0 and got["missed"] == 1 and got["chunks"] == 0


def test_bad_queries_refused(dev):
    import ctypes as C
    from paper_1207_0486_amd import _lib as L
    op = _operator(basin.box_mesh(4, 4, 2), -1)
    info = L.hns_one_launch_info()
    for args in ((None, 0, C.byref(info)), (op._h, 2, C.byref(info)), (op._h, 0, None)):
        assert L.lib().hns_one_launch_read(*args) == L.HNS_ERR_INVALID
    op.close()


def test_operators_on_one_form(dev):
    """Operators that share a compiled form (4 rows per thread) with unlike tiles:
    the larger solves as before after a smaller one was planned."""
    m, small = basin.basin_mesh(160, 140, 20, seed=5), basin.basin_mesh(90, 80, 11, seed=5)
    b, bs = _rhs(m, 1, 51, dev), _rhs(small, 1, 52, dev)
    op, other = _operator(m, 1), _operator(small, 1)
    x, info = op.solve(b, tol=1e-10, mask_bit=1)
    y, _ = other.solve(bs, tol=1e-10, mask_bit=1)
    z, again = op.solve(b, tol=1e-10, mask_bit=1)
    one, two = op.one_launch_info(), other.one_launch_info()
    op.close()
    other.close()
    assert one["rows_per_thread"] == two["rows_per_thread"] == 4
    assert one["lds_bytes"] > two["lds_bytes"] and one["chunks"] >= 2 and two["chunks"] >= 1
    assert again.status == 0 and again.iterations == info.iterations and torch.equal(x, z)


@pytest.mark.parametrize("mode", ["fp64", "mixed"])
def test_solves_that_run_together(dev, mode):
    """Threads with an operator and a stream each, whose chunks fit the GPU side by
    side or take turns (51 to 255 workgroups), as solves and as sessions: every
    answer is the one of the solve alone, bit for bit, and no meeting is missed."""
    import threading
    from paper_1207_0486_amd.hns import BatchSession
    grids = [((24, 24, 8), -1), ((24, 24, 8), 1), ((61, 47, 13), -1), ((61, 47, 13), 0),
             ((128, 64, 20), 1), ((128, 128, 16), 2), ((180, 190, 21), 0)]
    cases = []
    for k, (grid, bit) in enumerate(grids):
        m = basin.basin_mesh(*grid, seed=5)
        op = _operator(m, bit, keep_fp32=True)
        b = _rhs(m, bit, 60 + k, dev)
        x, info = op.solve(b, tol=1e-9, mask_bit=bit, mode=mode)
        cases.append((op, bit, b, x, info))
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        op, bit, b, want, winfo = cases[k]
        torch.cuda.set_device(dev)
        s = torch.cuda.Stream(dev)
        with torch.cuda.stream(s):
            sess = BatchSession(op, 2, mode)
            for _ in range(4 if bit < 0 else 12):
                x, info = op.solve(b, tol=1e-9, mask_bit=bit, mode=mode, stream=s)
                sess.add([1], [bit], [b], [1e-9], [100000], stream=s)
                while sess.advance(64, stream=s):
                    pass
                y, got = sess.take(1, stream=s)
                s.synchronize()
                if not (torch.equal(x, want) and torch.equal(y, want)
                        and info.iterations == got.iterations == winfo.iterations):
                    wrong.append(k)
            sess.close()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    missed = [c[0].one_launch_info(mode)["missed"] for c in cases]
    for c in cases:
        c[0].close()
    assert not wrong and not any(missed)


# A hipLaunchKernel in front of the runtime's that refuses the chunks (the only
# launches of 512 threads in more than one workgroup) while a flag is set.
REFUSE_C = """
#include <stdint.h>
#include <stddef.h>
typedef struct { uint32_t x, y, z; } dim3;
typedef int (*launch_t)(const void *, dim3, dim3, void **, size_t, void *);
static launch_t real;
static int refuse, refused;
void set_real(void *f) { real = (launch_t)f; }
void set_refuse(int on) { refuse = on; }
int get_refused(void) { return refused; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s)
{
    if (!real) return 1;
    if (refuse && b.x == 512 && g.x > 1) { ++refused; return 701; }
    return real(f, g, b, args, lds, s);
}
"""

REFUSE_PY = """
import ctypes, os, sys
front = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library that it stands in front of
sys.path.insert(0, sys.argv[2])
import torch   # loads the runtime; every launch below, torch's too, goes through the front
hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
front.set_real.argtypes = [ctypes.c_void_p]
front.set_real(ctypes.cast(ctypes.CDLL(hip).hipLaunchKernel, ctypes.c_void_p))
import basin
from paper_1207_0486_amd.hns import BatchSession, Operator
dev = torch.device("cuda", 0)
m = basin.basin_mesh(40, 36, 6, seed=5)
d = ((m.bc >> 1) & 1) == 1
b = torch.as_tensor(basin.normal_rhs(m.n, 41, dirichlet=d), device=dev)
for mode in ("fp64", "mixed"):
    op = Operator(m, 1e3, 1e-2, 3600.0, kind="helmholtz", keep_fp32=True, gpu_assembly=True)
    op.set_param("small_n", 0)
    op.set_param("check_every", 4)
    op.set_param("one_launch", 0)
    want, i = op.solve(b, tol=1e-10, mask_bit=1, mode=mode)
    op.set_param("one_launch", -1)
    front.set_refuse(1)
    got, j = op.solve(b, tol=1e-10, mask_bit=1, mode=mode)
    assert j.status == 0 and i.iterations == j.iterations and torch.equal(got, want), mode
    info = op.one_launch_info(mode)
    assert info["chunks"] == 0 and info["refused"] == 1, info
    # refused in the middle: the rest of the iterations, from where it is
    front.set_refuse(0)
    s = BatchSession(op, 1, mode)
    s.add([0], [1], [b], [1e-10], [1000])
    s.advance(4)
    front.set_refuse(1)
    while s.advance(4):
        pass
    y, k = s.take(0)
    info = op.one_launch_info(mode)
    assert k.status == 0 and abs(k.iterations - i.iterations) <= 1 and info["chunks"] == 1, (k, info)
    assert info["refused"] == 2, info
    assert float((y - want).norm() / want.norm()) <= 1e-9
    s.close()
    front.set_refuse(0)
    op.close()
assert front.get_refused() == 4
print("refused launches fell back")
"""


def test_a_refused_launch_falls_back(dev, tmp_path):
    """The device refuses the chunk's launch: the solve takes the launches per
    phase, to their bits, and so does the rest of one that has begun."""
    import os
    import subprocess
    import sys
    c, so = tmp_path / "refuse.c", tmp_path / "librefuse.so"
    c.write_text(REFUSE_C)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), str(c)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", REFUSE_PY, str(so), root], capture_output=True,
                         text=True, timeout=100, cwd=root)
    assert out.returncode == 0 and "refused launches fell back" in out.stdout, out.stderr[-2000:]


@pytest.mark.parametrize("bit, mode", [(-1, "fp64"), (1, "fp64"), (-1, "mixed"), (1, "mixed")])
def test_a_meeting_missed_later(dev, bit, mode):
    """Chunks that run, then one whose workgroups give up: the iterations that x
    does not hold are dropped and not counted.  FP64 starts again from the guess, to
    the launches' bits; mixed precision from its last replacement."""
    from paper_1207_0486_amd.hns import BatchSession
    m = basin.basin_mesh(40, 36, 6, seed=5)
    b = _rhs(m, bit, 71, dev)
    op = _operator(m, bit, keep_fp32=True)
    op.set_param("one_launch", 0)
    want, winfo = op.solve(b, tol=1e-10, mask_bit=bit, mode=mode)
    op.set_param("one_launch", -1)
    s = BatchSession(op, 1, mode)
    # (the cap: mixed solves restart their directions at the miss)
    cap = winfo.iterations if mode == "fp64" else 2 * winfo.iterations
    s.add([0], [bit], [b], [1e-10], [cap])
    for n in (3, 5, 7):
        assert s.advance(n) == 1
    before = op.one_launch_info(mode)["chunks"]
    op.set_param("meet_polls", 0)
    while s.advance(1000):
        pass
    x, info = s.take(0)
    s.close()
    got = op.one_launch_info(mode)
    assert before >= 3 and got["chunks"] == before and got["missed"] == 1
    assert info.status == 0 and info.relres_true <= 1e-10 and info.iterations <= cap
    if mode == "fp64":
        assert info.iterations == winfo.iterations and torch.equal(x, want)
    op.close()


def test_a_missed_meeting_is_remembered(dev):
    """The next 16 solves of the operator take launches per phase without trying
    (32 after the next miss), until a setting asks for one launch again."""
    m = basin.basin_mesh(40, 36, 6, seed=5)
    b = _rhs(m, 1, 81, dev)
    op = _operator(m, 1)
    op.set_param("meet_polls", 0)
    missed = []
    for _ in range(60):
        assert op.solve(b, tol=1e-6, mask_bit=1)[1].status == 0
        missed.append(op.one_launch_info()["missed"])
    assert missed == [1] * 17 + [2] * 33 + [3] * 10
    assert op.one_launch_info()["chunks"] == 0
    op.set_param("meet_polls", 1 << 21)
    op.solve(b, tol=1e-6, mask_bit=1)
    got = op.one_launch_info()
    op.close()
    assert got["chunks"] == 1 and got["missed"] == 3
