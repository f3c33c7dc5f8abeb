"""Block-Jacobi PCG on a matrix that turns out indefinite after some
iterations, at the sizes where the iteration changes its launches: x is the
last good iterate.

The right-hand side of a chain sits in its first row, so the search direction
of iteration k reaches row k; the block of row 5 is -I / 1000 there, and p.Ap
is first negative in the sixth iteration, after five good ones.  The
iterations before do the same operations in the same order however many are
asked for, so x equals the five iterations' x bit for bit, in every entry
point: the counted ones, which report the breakdown, and the enqueue-only
call, which cannot.  (The paper's termination stops after the five: r.z is
negative by then.)
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from test_gpu_pcg_sizes import _chain, _matrix, gp  # noqa: E402,F401

K = 5


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("V", [1536, 1537, 4096, 4097, 65536, 65537, 98304, 98305])
def test_x_at_a_late_breakdown(gp, V, dtype):  # noqa: F811
    dt = gp.F64 if dtype == "f64" else gp.F32
    rows, cols, vals = _chain(V)
    if dt == gp.F32:
        vals = vals.astype(np.float32).astype(np.float64)
    vals[(rows == K) & (cols == K)] = -1e-3 * np.eye(3)
    b = np.zeros((V, 3))
    b[0] = [1.0, -2.0, 0.5]
    bt = torch.tensor(b, device="cuda")
    A = _matrix(gp, V, rows, cols, vals, dt)
    ctx = gp.Context()
    good, it, _, st = gp.pcg(ctx, A, bt, rtol=0.0, maxit=K)
    assert it == K and st == gp.OK
    ref, _, _ = oracle.pcg(V, rows, cols, vals, b, rtol=0.0, maxit=K)
    err = np.linalg.norm(good.cpu().numpy().reshape(-1) - ref) / np.linalg.norm(ref)
    assert err <= (1e-10 if dt == gp.F64 else 1e-5), err  # as for the positive definite chains
    for maxit in (K + 1, 40):
        x = torch.zeros_like(bt)
        with pytest.raises(gp.GipcError) as e:
            gp.pcg(ctx, A, bt, x=x, rtol=0.0, maxit=maxit)
        assert e.value.status == gp.ERR_BREAKDOWN
        assert torch.equal(x, good), maxit
    x = torch.zeros_like(bt)
    with pytest.raises(gp.GipcError) as e:
        gp.pcg_static(A, bt, x=x, rtol=0.0, maxit=40)
    assert e.value.status == gp.ERR_BREAKDOWN and torch.equal(x, good)
    x = torch.zeros_like(bt)
    gp.pcg_static(A, bt, x=x, rtol=0.0, maxit=40, counts=False)
    torch.cuda.synchronize()
    assert torch.equal(x, good)
    ctx.close()
