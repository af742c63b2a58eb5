"""Served requests above the single-workgroup size: the sessions of several operators
run their one-launch chunks at the same time, and every answer is the one of the same
request alone, bit for bit."""
import numpy as np
import pytest

import basin

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# 5,625 to 282,897 rows: chunks that fit the GPU side by side and one that does not
MESHES = [(24, 24, 8), (32, 32, 8), (64, 64, 10), (128, 128, 16)]


def _make(key):
    idx, kind = key
    return basin.basin_mesh(*MESHES[idx], seed=10 + idx), 1e3, 1e-2, 3600.0, kind


@pytest.mark.parametrize("mode", ["fp64", "mixed"])
def test_served_together_equals_alone(mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1207_0486_amd.hns import Operator
    from paper_1207_0486_amd.serve import GpuBackend, Request, Server
    be = GpuBackend(_make, mode=mode, check_every=16)
    srv = Server(be, budget_bytes=16 << 30, capacity=2, chunk=32)
    rng = np.random.default_rng(7)
    reqs = []
    for i in range(32):
        idx, kind = i % 4, "poisson" if i % 8 < 4 else "helmholtz"
        m = be.make_operator((idx, kind))[0]
        bit = -1 if kind == "poisson" else int(rng.integers(0, 3))
        d = None if bit < 0 else ((m.bc >> bit) & 1) == 1
        reqs.append(Request(key=(idx, kind), b=basin.normal_rhs(m.n, 2000 + i, dirichlet=d),
                            mask_bit=bit, tol=1e-8))
    results = [f.result(timeout=100) for f in [srv.submit(r) for r in reqs]]
    missed = [r.entry.op.one_launch_info(mode)["missed"] for r in srv.resident.values()]
    chunks = [r.entry.op.one_launch_info(mode)["chunks"] for r in srv.resident.values()]
    srv.close()
    assert not srv.errors and len(missed) == 8 and not any(missed) and all(chunks)
    ops = {}
    for r, out in zip(reqs, results):
        if r.key not in ops:
            m, nu_h, nu_v, dt, kind = be.make_operator(r.key)
            ops[r.key] = Operator(m, nu_h, nu_v, dt, kind=kind, keep_fp32=mode == "mixed",
                                  gpu_assembly=True)
        x, info = ops[r.key].solve(torch.as_tensor(r.b, device="cuda"), tol=1e-8,
                                   mask_bit=r.mask_bit, mode=mode)
        assert out.info.status == info.status == 0 and out.info.iterations == info.iterations
        assert np.array_equal(out.x, x.cpu().numpy()), r.key
    for op in ops.values():
        op.close()
