"""Contact candidates where boxes touch and objects mix, against brute force.

The pair tests decide by integer steps within a cell and compare coordinates
only where those tie; a vertex shared across objects is looked for only where
a primitive's vertices belong to different ones.  Strips of vertices on a
lattice (boxes that touch exactly, faces of cells hit exactly), in tenths
(touching up to rounding), flat in one axis, far from the origin, in cells
with more than 64 primitives, with objects per strip or per vertex: the set
equals the brute-force set exactly.
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


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("strips,length,unit,origin,dhat", [
    (2, 3, 1.0, 0.0, 1.0),        # a few cells, boxes exactly dhat apart
    (6, 40, 1.0, 0.0, 1.0),
    (6, 40, 0.1, 0.0, 0.1),       # tenths: equal up to rounding
    (5, 30, 1.0, 1048576.0, 1.0),  # far away, still exact
    (4, 25, 0.1, 1048576.3, 0.2),
    (6, 40, 1.0, 0.0, 0.0),       # closed boxes that touch
    (40, 6, 1.0, 0.0, 3.0),       # more than 64 primitives in a cell
])
def test_touching_boxes_and_mixed_objects(gp, strips, length, unit, origin, dhat, mixed):
    rng = np.random.default_rng(strips * 100 + length)
    g = np.zeros((strips, length, 3))
    g[..., 0] = np.arange(length)
    g[..., 1] = np.arange(length) % 2 + rng.integers(0, 3, (strips, 1))
    g[..., 2] = rng.integers(0, 2, (strips, 1))
    x = (g * unit + origin).reshape(-1, 3)
    i = np.arange(strips * length).reshape(strips, length)
    tris = np.stack([i[:, :-2], i[:, 1:-1], i[:, 2:]], 2).reshape(-1, 3)
    edges = np.concatenate([np.stack([i[:, :-1], i[:, 1:]], 2).reshape(-1, 2),
                            np.stack([i[:, :-2], i[:, 2:]], 2).reshape(-1, 2)])
    vobj = rng.integers(0, 3, x.shape[0]) if mixed else np.repeat(np.arange(strips) % 3, length)
    order = rng.permutation(len(edges))
    edges = edges[order]
    dev = torch.device("cuda", 0)
    ctx = gp.Context()
    c = gp.candidates(ctx, torch.tensor(x, device=dev), *(torch.tensor(a, dtype=torch.int32, device=dev)
                                                         for a in (vobj, tris, edges)), dhat).cpu().numpy()
    ref = oracle.candidates(x, vobj, tris, edges, dhat)
    assert len(ref) > 0 and len(c) == len(ref)
    assert set(map(tuple, c.tolist())) == set(map(tuple, ref.tolist()))
    ctx.close()


@pytest.mark.parametrize("first", [True, False])
def test_a_box_of_nan_is_apart_from_nothing(gp, first):
    # a comparison with NaN never says that boxes are apart, and NaN falls into
    # the grid's first cell, where this triangle lies too
    nan = np.full((2, 3), np.nan)
    x = np.concatenate([[[0.0, 0.0, 0.0], [1.0, 0.0, 0.1], [0.0, 1.0, 0.2]], nan])
    vobj = np.array([0, 0, 0, 1, 1])
    tris = np.array([[0, 1, 2]])
    edges = np.array([[0, 1], [1, 2], [0, 2]])
    edges = np.concatenate([[[3, 4]], edges] if first else [edges, [[3, 4]]])
    dev = torch.device("cuda", 0)
    ctx = gp.Context()
    c = gp.candidates(ctx, torch.tensor(x, device=dev), *(torch.tensor(a, dtype=torch.int32, device=dev)
                                                         for a in (vobj, tris, edges)), 1e-3).cpu().numpy()
    want = [(-4, 0, 1, 2), (-5, 0, 1, 2)]
    want += [(3, 4, a, b) if first else (a, b, 3, 4) for a, b in [(0, 1), (1, 2), (0, 2)]]
    assert len(c) == len(want) and set(map(tuple, c.tolist())) == set(want)
    ctx.close()
