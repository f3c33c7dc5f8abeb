"""gipc_pairs_check of pairs whose distance sits at dhat up to rounding.

A point just past the end of an edge 10^8 times as long as dhat: the
classification's difference (p - a) - (b - a) and the evaluation's p - b round
differently, and the points here are those that the first puts beyond dhat by
1e-8 and more, the second within dhat by 1e-9 and more of dhat^2 (both are
exact differences of doubles, the same in numpy).  The staged pair still
contributes there, so it counts as changed, not as left; clearly beyond dhat
it has left.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DH = 1e-8


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09400_amd as gp
    torch.cuda.set_device(0)
    return gp


def test_left_only_where_the_evaluation_agrees(gp):
    rng = np.random.default_rng(1)
    a, b = -rng.uniform(0.3, 0.9, 4096), rng.uniform(0.3, 0.9, 4096)
    p = b + DH * (1.0 - rng.uniform(0.0, 2e-8, 4096))
    pick = (((p - a) - (b - a)) ** 2 > (1.0 + 1e-8) * DH * DH) & ((p - b) ** 2 < (1.0 - 1e-9) * DH * DH)
    a, b, p = a[pick], b[pick], p[pick]
    n = len(p)
    assert n > 50

    def at(point):
        x = np.zeros((n, 3, 3))
        x[:, 0, 0], x[:, 1, 0], x[:, 2, 0] = point, a, b
        return torch.tensor(x.reshape(-1, 3), device="cuda")

    i = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    tup = torch.tensor(np.stack([-(i[:, 0] + 1), i[:, 1], i[:, 2], np.full(n, -1, np.int32)], 1), device="cuda")
    prm = gp.params(dhat=DH, kappa=1e4)
    ctx = gp.Context()
    built = at(b + 0.9 * DH)
    info = gp.pairs_build(ctx, built, tup, prm)
    assert info["n_active"] == n
    stale, c = gp.pairs_check(ctx, at(p), tup, prm, x_rest=built)
    assert stale and (c["n_entered"], c["n_left"], c["n_changed"]) == (0, 0, n)
    stale, c = gp.pairs_check(ctx, at(b + 1.1 * DH), tup, prm, x_rest=built)
    assert not stale and (c["n_entered"], c["n_left"], c["n_changed"]) == (0, n, 0)
    ctx.close()
