"""Block-Jacobi PCG with each of its products at the sizes where the iteration
changes its launches: one workgroup for everything between two products up to
1536 rows (1024 without a matrix), scalars formed by every workgroup up to
98304, kernels of their own beyond.

* chains with the row-start map, whose product walks the matrix backwards in
  every other iteration, against the oracle's PCG: 1e-10 of the iterate's norm
  (well-conditioned systems: rounding, about 1e-16 a step, is not amplified);
* the matrix-free operator and both dense products of a small scene with
  vertices of their own added, the diagonal as large as the largest entry of
  the contact blocks, against gipc_pcg on the assembled matrix: 1e-10 again;
* both: the same number of iterations to a tolerance, within one.
"""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import scenes  # noqa: E402
from test_gpu_pcg_sizes import _chain, _matrix, gp  # noqa: E402,F401


def _with_map(gp, V, rows, cols, vals):
    A = _matrix(gp, V, rows, cols, vals, gp.F64)
    rp = np.searchsorted(rows, np.arange(V + 1))
    bits = np.zeros(-(-len(rows) // 64) * 64, np.uint8)
    bits[rp[:-1]] = 1
    head = torch.tensor(np.packbits(bits, bitorder="little").view(np.int64), device="cuda")
    wrow = torch.tensor(rows[::64].copy(), device="cuda")
    A.desc.wave_head, A.desc.wave_row = head.data_ptr(), wrow.data_ptr()
    return SimpleNamespace(desc=A.desc, keep=(A, head, wrow))


def _rel(x, ref):
    return np.linalg.norm(x.cpu().numpy().reshape(-1) - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("V", [1, 2, 1024, 1025, 1536, 1537, 98304, 98305])
def test_entry_product(gp, V):  # noqa: F811
    rows, cols, vals = _chain(V)
    b = np.random.default_rng(11).standard_normal((V, 3))
    A = _with_map(gp, V, rows, cols, vals)
    bt = torch.tensor(b, device="cuda")
    ctx = gp.Context()
    for maxit in [m for m in (1, 2, 5, 18) if m < 3 * V]:
        ref, _, _ = oracle.pcg(V, rows, cols, vals, b, rtol=0.0, maxit=maxit)
        x, it, _, st = gp.pcg(ctx, A, bt, rtol=0.0, maxit=maxit)
        assert it == maxit and st == gp.OK and _rel(x, ref) <= 1e-10, (maxit, _rel(x, ref))
    _, ito, _ = oracle.pcg(V, rows, cols, vals, b, rtol=1e-8, maxit=200)
    x, it, rr, st = gp.pcg(ctx, A, bt, rtol=1e-8, maxit=200)
    assert st == gp.OK and rr <= 1e-8 and abs(it - ito) <= 1
    ctx.close()


@pytest.mark.parametrize("V", [512, 1024, 1025, 98304, 98305])
def test_products_without_a_matrix(gp, V):  # noqa: F811
    s = scenes.two_sheets(n=16, seed=1)
    x = np.concatenate([s.x, np.random.default_rng(V).uniform(10.0, 20.0, (V - s.V, 3))])
    rest = np.concatenate([s.x_rest, x[s.V:]])
    X, XR = torch.tensor(x, device="cuda"), torch.tensor(rest, device="cuda")
    T = torch.tensor(np.asarray(s.tuples, np.int32).reshape(-1, 4), device="cuda")
    prm = gp.params(dhat=s.dhat, kappa=s.kappa)
    ctx = gp.Context()
    gp.pairs_build(ctx, X, T, prm, x_rest=XR)
    A = gp.BsrMatrix(ctx)
    gp.eval_assemble(ctx, X, prm, A, x_rest=XR)
    D = torch.full((V,), A.val.abs().max().item(), dtype=torch.float64, device="cuda")
    gp.eval_assemble(ctx, X, prm, A, diag=D, x_rest=XR)
    hess = gp.proxy_dense(ctx, X, prm, x_rest=XR)
    b = torch.tensor(np.random.default_rng(13).standard_normal((V, 3)), device="cuda")
    other = gp.Context()
    solves = [lambda **k: gp.pcg_mf(ctx, b, diag=D, **k)]
    solves += [lambda scheme=c, **k: gp.pcg_dense(ctx, hess, b, diag=D, scheme=scheme, **k)
               for c in (gp.DENSE_ENTRY, gp.DENSE_THREAD)]
    for maxit in (1, 2, 5, 18):
        ref = gp.pcg(other, A, b, rtol=0.0, maxit=maxit, by_rows=True)[0].cpu().numpy().reshape(-1)
        for solve in solves:
            got, it, _, st = solve(rtol=0.0, maxit=maxit)
            assert it == maxit and st == gp.OK and _rel(got, ref) <= 1e-10, (maxit, _rel(got, ref))
    _, ita, _, _ = gp.pcg(other, A, b, rtol=1e-8, maxit=200, by_rows=True)
    for solve in solves:
        _, it, rr, st = solve(rtol=1e-8, maxit=200)
        assert st == gp.OK and rr <= 1e-8 and abs(it - ita) <= 1
    ctx.close()
    other.close()
