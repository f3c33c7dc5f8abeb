"""Contact candidates on grids of many cells, against brute force.

A few hundred small pairs of triangles far apart: 2^25, 2^26 and nearly 2^28
cells (the limit), nearly all empty, in slices of the passes that take one
wavefront per cell.  The set and the order (point-triangle by point, then
edge-edge by first edge) are those of brute force, also when the pairs stand
at the first and the last cell and across the borders of the slices.
"""
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


@pytest.mark.parametrize("n", [321, 323, 407, 645])  # 2^25 cells lie between 322^3 and 323^3, 2^26 below 407^3
def test_many_cells(gp, n):
    # cells of 2 (extent 1 plus dhat 1) from 4 dhat below the smallest coordinate
    dhat, span = 1.0, 2.0 * (n - 1) - 4.5
    rng = np.random.default_rng(n)
    at = rng.uniform(0.0, span - 1.5, (300, 3))
    at[0], at[1] = 0.0, span - 1.5
    for k, border in enumerate(c for c in range(1 << 25, n ** 3, 1 << 25)):  # the cells beside a slice's border
        cell = np.array([border // n ** 2, border // n % n, border % n])
        at[2 + k] = np.clip(2.0 * cell - 4.0, 0.0, span - 1.5)
    tri = np.array([[0.0, 0.0, 0.0], [1.0, 0.2, 0.1], [0.3, 1.0, 1.0]])
    x = np.concatenate([np.concatenate([p + tri, p + 0.5 + tri]) for p in at])
    i = np.arange(len(x)).reshape(-1, 3)
    tris = np.ascontiguousarray(i, dtype=np.int32)
    edges = np.ascontiguousarray(np.concatenate([i[:, [0, 1]], i[:, [1, 2]], i[:, [0, 2]]]), dtype=np.int32)
    vobj = (np.arange(len(x)) // 3).astype(np.int32)
    dev = torch.device("cuda", 0)
    ctx = gp.Context()
    c = gp.candidates(ctx, torch.tensor(x, device=dev), *(torch.tensor(a, device=dev) for a in (vobj, tris, edges)),
                      dhat).cpu().numpy()
    ctx.close()
    ref = oracle.candidates(x, vobj, tris, edges, dhat)
    assert len(ref) >= 15 * len(at)  # 6 point-triangle and 9 edge-edge pairs each
    assert len(c) == len(ref) and set(map(tuple, c.tolist())) == set(map(tuple, ref.tolist()))
    npt = int((c[:, 0] < 0).sum())
    assert (c[:npt, 0] < 0).all() and (np.diff(~c[:npt, 0]) >= 0).all()
    first = {tuple(e): k for k, e in enumerate(edges.tolist())}
    assert (np.diff([first[tuple(e)] for e in c[npt:, :2].tolist()]) >= 0).all()
