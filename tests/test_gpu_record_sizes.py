"""Records and sums that end raggedly, against the oracle.

Barrier and friction records are written by quads of lanes and energies are
summed over pieces of 1024 vertices: a random part of the tuples of two
jittered sheets (every type, mollified pairs too), from one tuple to ends
inside a quad, a wavefront and a workgroup, with the vertices renumbered at
random among V.  Energies, gradients and blocks of barrier and friction
within 1e-9 (energies relative, the others of the largest entry), the
tolerance of the larger scenes: sums of at most a few hundred terms in FP64.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import scenes  # noqa: E402

TOL = 1e-9
MU, EPS_V, DT = 0.3, 1e-2, 1e-2


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_09400_amd as gp
    torch.cuda.set_device(0)
    return gp


@pytest.mark.parametrize("P,V", [(1, 1023), (2, 1024), (3, 1025), (4, 2047), (5, 2048), (63, 2049), (65, 1024),
                                 (255, 1025), (257, 9000), (1027, 4097)])
def test_records_and_sums(gp, P, V):
    s = scenes.two_sheets(n=12, dhat=0.08, kappa=10.0, seed=3, offset=0.5, jitter=0.3)
    rng = np.random.default_rng(P)
    perm = rng.permutation(V)[:s.V]
    t = np.asarray(s.tuples, np.int64)
    po = oracle.params(dhat=s.dhat, kappa=s.kappa)
    # tuples in contact (of positive energy), a third of them mollified
    ev = oracle.eval_scene(s.x, t, po, x_rest=s.x_rest, per_pair=True)
    moll = np.asarray(ev["mollified"]) != 0
    near, para = (np.flatnonzero((ev["pairE"] > 0) & m) for m in (~moll, moll))
    m = min((P + 2) // 3, len(para))
    pick = np.concatenate([rng.choice(para, m, replace=False), rng.choice(near, P - m, replace=False)])
    t = t[np.sort(pick)]
    vert = np.where(t < 0, -t - 1, t)
    t = np.where(t < 0, -perm[vert] - 1, perm[vert])
    x, xr = rng.uniform(50.0, 60.0, (V, 3)), rng.uniform(50.0, 60.0, (V, 3))
    x[perm], xr[perm] = s.x, s.x_rest
    xm = x + rng.normal(scale=0.3 * EPS_V * DT, size=x.shape)
    ev = oracle.eval_scene(x, t, po, x_rest=xr, per_pair=True)
    fr = oracle.friction_scene(x, xm, t, po, oracle.fparams(MU, EPS_V, DT), x_rest=xr, per_pair=True)
    diag = np.full(V, 10.0)
    rows, cols, vals = oracle.assemble(V, t, ev["pairH"] + fr["pairH"], diag)

    dev = torch.device("cuda", 0)
    X, XR, XM, D = (torch.tensor(a, device=dev) for a in (x, xr, xm, diag))
    pg = gp.params(dhat=s.dhat, kappa=s.kappa)
    ctx = gp.Context()
    info = gp.pairs_build(ctx, X, torch.tensor(t, dtype=torch.int32, device=dev), pg, x_rest=XR)
    assert info["n_active"] == P
    gp.friction_lag(ctx, X, pg, MU, EPS_V, DT, x_rest=XR)
    A = gp.BsrMatrix(ctx)
    Eb, gb = gp.eval_assemble(ctx, X, pg, A, diag=D, x_rest=XR)
    Ef, gf = gp.friction_eval(ctx, XM, pg, A)
    assert Eb.item() == pytest.approx(ev["E"], rel=TOL) and Ef.item() == pytest.approx(fr["E"], rel=TOL)
    assert np.abs(gb.cpu().numpy() - ev["grad"]).max() <= TOL * np.abs(ev["grad"]).max()
    assert np.abs(gf.cpu().numpy() - fr["grad"]).max() <= TOL * np.abs(fr["grad"]).max()
    rp, ci = A.row_ptr().cpu().numpy(), A.col_idx().cpu().numpy()
    got = dict(zip(zip(np.repeat(np.arange(V), np.diff(rp)).tolist(), ci.tolist()),
                   A.val[:, :A.nnzb].cpu().numpy().T.reshape(-1, 3, 3)))
    want = dict(zip(zip(rows.tolist(), cols.tolist()), vals))
    worst = max(np.abs(got.get(k, 0.0) - want.get(k, 0.0)).max() for k in set(got) | set(want))
    assert worst <= TOL * max(np.abs(B).max() for B in vals)
    ctx.close()
