"""Block-Jacobi PCG at the sizes where the iteration changes its launches (one
workgroup for everything between two products up to 4096 rows, scalars formed
by every workgroup up to 65536, kernels of their own beyond): caller-made
block-tridiagonal systems against the oracle's PCG, FP64 and FP32 blocks.

* a fixed number of iterations (odd and even, beyond the host's poll): the
  oracle's iterate; FP64 to 1e-10 of its norm (a well-conditioned system:
  rounding, about 1e-16 a step, is not amplified), FP32 to 1e-5 (products in
  FP32, unit roundoff 6e-8, a few dozen operations a step);
* stopped by the residual: the oracle's iteration count within one;
* a negative definite matrix breaks down at the first iteration.
"""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09400_amd as gp
    torch.cuda.set_device(0)
    return gp


def _chain(V):
    """Rows, columns, blocks of a symmetric positive definite chain."""
    rng = np.random.default_rng(V)
    B = 0.3 * rng.standard_normal((V, 3, 3))
    D = np.einsum("vab,vcb->vac", B, B) + np.diag([2.5, 3.0, 3.5])
    off = 0.2 * rng.standard_normal((max(V - 1, 0), 3, 3))
    rows = np.concatenate([np.arange(V), np.arange(V - 1), np.arange(1, V)])
    cols = np.concatenate([np.arange(V), np.arange(1, V), np.arange(V - 1)])
    vals = np.concatenate([D, off, off.transpose(0, 2, 1)])
    order = np.lexsort((cols, rows))
    return rows[order].astype(np.int32), cols[order].astype(np.int32), np.ascontiguousarray(vals[order])


def _matrix(gp, V, rows, cols, vals, dtype):
    dev = torch.device("cuda", 0)
    rp = torch.tensor(np.searchsorted(rows, np.arange(V + 1)).astype(np.int32), device=dev)
    ci = torch.tensor(cols, device=dev)
    tdt = torch.float64 if dtype == gp.F64 else torch.float32
    val = torch.tensor(np.ascontiguousarray(vals.reshape(-1, 9).T), device=dev).to(tdt).contiguous()
    desc = gp.Bsr(V, len(rows), rp.data_ptr(), ci.data_ptr(), val.data_ptr(), dtype, None, None)
    return SimpleNamespace(desc=desc, keep=(rp, ci, val))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("V", [1, 2, 1024, 1025, 4096, 4097, 65536, 65537])
def test_pcg_sizes(gp, V, dtype):
    dt = gp.F64 if dtype == "f64" else gp.F32
    rows, cols, vals = _chain(V)
    if dt == gp.F32:
        vals = vals.astype(np.float32).astype(np.float64)
    b = np.random.default_rng(7).standard_normal((V, 3))
    A = _matrix(gp, V, rows, cols, vals, dt)
    bt = torch.tensor(b, device="cuda")
    ctx = gp.Context()
    # in exact arithmetic a system of 3 V unknowns is solved in 3 V iterations
    for maxit in [m for m in (1, 2, 5, 18) if m < 3 * V]:
        ref, _, _ = oracle.pcg(V, rows, cols, vals, b, rtol=0.0, maxit=maxit)
        x, it, rr, st = gp.pcg(ctx, A, bt, rtol=0.0, maxit=maxit)
        err = np.linalg.norm(x.cpu().numpy().reshape(-1) - ref) / np.linalg.norm(ref)
        assert it == maxit and st == gp.OK
        assert err <= (1e-10 if dt == gp.F64 else 1e-5), (V, maxit, err)
    tol = 1e-8 if dt == gp.F64 else 1e-4
    _, ito, _ = oracle.pcg(V, rows, cols, vals, b, rtol=tol, maxit=200)
    x, it, rr, st = gp.pcg(ctx, A, bt, rtol=tol, maxit=200)
    assert st == gp.OK and rr <= tol and abs(it - ito) <= 1
    N = _matrix(gp, V, rows, cols, -vals, dt)
    with pytest.raises(gp.GipcError) as e:
        gp.pcg(ctx, N, bt, rtol=tol, maxit=10)
    assert e.value.status == gp.ERR_BREAKDOWN
    ctx.close()
