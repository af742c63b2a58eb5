"""Edges of the step's forms in diagonal storage: non-finite values reach exactly
the nodes they are coupled to, vectors that overlap, calls that run together."""
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


def _operator(m):
    from paper_1207_0486_amd.hns import Operator
    return Operator(m, *NU, DT, kind="helmholtz", step_aux=True)


# a uniform box, where a tenth of the couplings of B are exactly 0 (half of its
# diagonal among them), and a mesh with a bumpy floor
MESHES = {"box": lambda: basin.box_mesh(6, 5, 4), "basin": lambda: basin.basin_mesh(7, 5, 4, seed=2)}


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("mesh", MESHES)
def test_non_finite_values_reach_the_coupled_nodes(dev, mesh, value):
    """0 times a non-finite value is NaN, so every node that shares a
    tetrahedron with the value's node is non-finite, and no other node is."""
    m = MESHES[mesh]()
    op = _operator(m)
    at = m.n // 2 + 1
    near = np.zeros(m.n, dtype=bool)
    near[m.tets[(m.tets == at).any(axis=1)].ravel()] = True
    x = torch.ones(m.n, dtype=torch.float64, device=dev)
    x[at] = value

    def spread(y):
        return ~torch.isfinite(y).cpu().numpy()

    for name in ("B1", "B2", "B3", "B1T", "B2T", "B3T"):
        assert np.array_equal(spread(op.apply_aux(name, x)), near), name
    one = torch.ones(3, m.n, dtype=torch.float64, device=dev)
    for c in range(3):
        ut = one.clone()
        ut[c] = x
        assert np.array_equal(spread(op.step_pressure_rhs(ut)), near)
    free = [((m.bc >> c) & 1) == 0 for c in range(3)]
    for y in (op.step_correct(one, x), op.step_correct_rhs(7.0, one, x),
              op.step_velocity_rhs(one, x)):
        for c in range(3):
            assert np.array_equal(spread(y[c]), near & free[c]), c
    op.close()


@pytest.mark.parametrize("shift", [0, 1, 5])
def test_pressure_inside_the_velocity(dev, shift):
    """p += q comes first, also where p lies in u~ (then the forms read the
    updated u~) or in the result (then the result replaces it)."""
    m = basin.basin_mesh(19, 23, 6, seed=2)
    op = _operator(m)
    n = m.n
    rng = np.random.default_rng(3)
    ut = torch.as_tensor(rng.standard_normal((3, n)), device=dev)
    q = torch.as_tensor(rng.standard_normal(n), device=dev)
    for name, args in (("step_correct", ()), ("step_correct_rhs", (7.0,))):
        call = getattr(op, name)
        a, b = ut.clone(), ut.clone()
        b.view(-1)[n + shift:2 * n + shift] += q
        got = call(*args, a, q, a.view(-1)[n + shift:2 * n + shift])
        assert torch.equal(a, b)
        want = call(*args, b, q)
        # the launches sum a row's entries in another order than the one pass
        assert float((got - want).abs().max()) <= 1e-13 * float(want.abs().max())
        out = torch.zeros_like(ut)
        call(*args, ut, q, out.view(-1)[n + shift:2 * n + shift], out=out)
        want = call(*args, ut, q)
        assert float((out - want).abs().max()) <= 1e-13 * float(want.abs().max())
    op.close()


def test_calls_that_run_together(dev):
    """Threads with a stream each call the forms of one operator at the same
    time: every result is the one of the call alone, bit for bit."""
    import threading
    m = basin.basin_mesh(64, 60, 10, seed=2)
    op = _operator(m)
    rng = np.random.default_rng(3)
    us = [torch.as_tensor(rng.standard_normal((3, m.n)), device=dev) for _ in range(4)]

    def forms(k, stream=None):
        adv = op.step_advection(us[k], stream=stream)
        return adv, op.step_velocity_rhs_bdf(7.0, 1.0, us[k], adv=adv, stream=stream)

    want = [forms(k) for k in range(4)]
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        torch.cuda.set_device(dev)
        s = torch.cuda.Stream(dev)
        with torch.cuda.stream(s):
            for _ in range(30):
                got = forms(k, s)
                s.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, want[k])):
                    wrong.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    op.close()
