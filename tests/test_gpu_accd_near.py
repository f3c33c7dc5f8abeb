"""Additive CCD on the GPU for pairs that touch or nearly do.

* Pairs at distance 0 (a point on an end of a segment or triangle, edges
  that share a point) give time 0 and are counted, at either end of every
  edge, and so do pairs of which an edge is far below the others' size.
* A point (or a parallel edge) at distance d beside an axis-aligned edge of
  length L, 1e-6 L down to 1e-13 L, falling onto it at speed v: the closed
  form (1 - s) d / v.  The coordinates across the edge are exact, so the
  distance errs by the foot's place along the edge only: its parameter comes
  from a rounded product over a rounded square (three roundings) and its
  product with the edge is one more, 2^-51 L in all; d^2 + (2^-51 L)^2 is
  d (1 + (2^-51 L / d)^2 / 2), and 2^-48 covers the few roundings besides.
* The first sub-step is the quotient (1 - s) d / l_p, and the mean motion a
  quotient by the number of vertices, to the last bit: a point at a distance
  that is exact falls onto a point, an edge or a triangle, so all of l_p's
  roundings are those of the same sums in numpy (the root of a rounded square
  is the number itself).
* A displacement with a NaN has no rate of approach: tc, not counted, as for
  no relative motion.  An infinite one has no sub-step: the search ends at
  max_iter and is counted as capped, not as touching.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

S = 0.1


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09400_amd as gp
    torch.cuda.set_device(0)
    return gp


@pytest.fixture(scope="module")
def ctx(gp):
    c = gp.Context()
    yield c
    c.close()


def _run(gp, ctx, X, D, tup, tc):
    toi, info = gp.accd(ctx, torch.tensor(X.reshape(-1, 3), device="cuda"),
                        torch.tensor(D.reshape(-1, 3), device="cuda"), torch.tensor(tup, device="cuda"), s=S, tc=tc,
                        max_iter=1000)
    return toi.cpu().numpy(), info


def _neg(i):
    return -(i + 1)


def _tuples(kind, P):
    """P tuples of their own four vertices each."""
    i = np.arange(4 * P, dtype=np.int32).reshape(P, 4)
    a, b, c, d = i.T
    m = np.full(P, -1, np.int32)
    cols = dict(ee=(a, b, c, d), pt=(_neg(a), b, c, d), pe=(_neg(a), b, c, m), pp=(_neg(a), b, m, m),
                pe_par=(_neg(a), _neg(b), c, _neg(d)), pp_par=(_neg(a), _neg(b), _neg(c), _neg(d)))[kind]
    return np.ascontiguousarray(np.stack(cols, 1), dtype=np.int32)


# vertices of the two primitives, by slot of the tuple
ENDS = dict(ee=([0, 1], [2, 3]), pt=([0], [1, 2, 3]), pe=([0], [1, 2]), pp=([0], [1]), pe_par=([0], [2, 3]),
            pp_par=([0], [2]))


@pytest.mark.parametrize("kind", sorted(ENDS))
def test_touching_at_any_end(gp, ctx, kind):
    rng = np.random.default_rng(3)
    at = [(i, j) for i in ENDS[kind][0] for j in ENDS[kind][1]]
    P = 64 * len(at)
    X, D = rng.normal(size=(P, 4, 3)), rng.normal(size=(P, 4, 3))
    for k in range(P):
        i, j = at[k % len(at)]
        X[k, j] = X[k, i]
        if k % 3 == 0:  # another edge of length 0, 1e-170 or 1e-20 at the touching end
            for o in set(ENDS[kind][1]) - {j}:
                X[k, o] = X[k, j]
                X[k, o, k // 3 % 3] += (0.0, 1e-170, 1e-20)[k // 9 % 3]
                break
    toi, info = _run(gp, ctx, X, D, _tuples(kind, P), tc=1.0)
    assert (toi == 0.0).all() and info["n_touching"] == P and info["step"] == 0.0 and info["n_capped"] == 0


@pytest.mark.parametrize("ratio", [1e-6, 1e-9, 1e-10, 1e-11, 1e-12, 1e-13])
@pytest.mark.parametrize("kind", ["pt", "pe", "pe_par", "ee"])
def test_near_an_axis_aligned_edge(gp, ctx, kind, ratio):
    rng = np.random.default_rng(int(-np.log10(ratio)))
    P = 500
    L, f, v = rng.uniform(0.5, 2.0, P), rng.uniform(0.05, 0.95, P), rng.uniform(0.5, 2.0, P)
    d = ratio * L
    X, D = np.zeros((P, 4, 3)), np.zeros((P, 4, 3))
    e0, e1 = dict(pt=(1, 2), pe=(1, 2), pe_par=(2, 3), ee=(2, 3))[kind]
    X[:, e1, 0] = L                                    # the edge along x, from the origin
    X[:, 0, 0], X[:, 0, 1], D[:, 0, 1] = f * L, d, -v  # the point beside it, falling onto it
    if kind == "pt":
        X[:, 3, 0], X[:, 3, 1] = 0.5 * L, -L           # the triangle on the edge's other side
    elif kind in ("ee", "pe_par"):                     # an edge parallel to it from the point on, past the end
        X[:, 1, 0], X[:, 1, 1], D[:, 1, 1] = 3.0 * L, d, -v
    toi, info = _run(gp, ctx, X, D, _tuples(kind, P), tc=1e9)
    ref = (1.0 - S) * d / v
    bound = 0.5 * (2.0 ** -51 * L / d) ** 2 + 2.0 ** -48
    err = np.abs(toi - ref) / ref
    print(f"accd near {kind} d/L={ratio:g}: largest error {err.max():.2e}, of its bound {(err / bound).max():.2e}",
          flush=True)
    assert info["n_touching"] == 0 and info["n_capped"] == 0
    assert (err <= bound).all()


@pytest.mark.parametrize("kind", ["pp", "pe", "pt"])
def test_first_sub_step_to_the_last_bit(gp, ctx, kind):
    rng = np.random.default_rng(17)
    P, nv = 2000, dict(pp=2, pe=3, pt=4)[kind]
    d, v = rng.uniform(0.5, 2.0, P), rng.uniform(0.5, 2.0, P)
    X, D = np.zeros((P, 4, 3)), np.zeros((P, 4, 3))
    X[:, 0, 1], D[:, 0, 1] = d, -v
    if kind != "pp":  # the point above (0, 0, 0), a quarter along the edge, or both edges of a triangle of area 8
        X[:, 1, 0], X[:, 2, 0] = -1.0, 3.0
        if kind == "pt":
            X[:, 1:3, 2], X[:, 3, 0], X[:, 3, 2] = -1.0, -1.0, 3.0
    toi, info = _run(gp, ctx, X, D, _tuples(kind, P), tc=1e9)
    m = -v / nv
    lp = np.abs(-v - m) + np.abs(0.0 - m)
    assert info["max_steps"] == 2
    assert np.array_equal(toi, (1.0 - S) * d / lp)


@pytest.mark.parametrize("kind", sorted(ENDS))
def test_displacement_not_finite(gp, ctx, kind):
    rng = np.random.default_rng(23)
    used = sorted(ENDS[kind][0] + ENDS[kind][1])
    P = 12 * len(used)
    for value, capped in ((np.nan, 0), (np.inf, P), (-np.inf, P)):
        X, D = rng.normal(size=(P, 4, 3)), rng.normal(size=(P, 4, 3))
        D[np.arange(P), np.resize(used, P), np.arange(P) // len(used) % 3] = value
        toi, info = _run(gp, ctx, X, D, _tuples(kind, P), tc=0.75)
        assert info["n_touching"] == 0 and info["n_capped"] == capped
        if np.isnan(value):
            assert (toi == 0.75).all() and info["step"] == 0.75
