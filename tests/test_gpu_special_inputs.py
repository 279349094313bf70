"""Inputs outside the ordinary: infinite charges, and points closer together
than the square of their distance can be told from 0."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_15269_amd as F
    return F


# charge counts around a wave's 64 lanes, target counts of every number of
# targets a wave
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nt", [(1, 1), (63, 5), (64, 5), (65, 5), (130, 300), (200, 600),
                                  (1025, 1030)])
def test_direct_sum_keeps_an_infinite_charge_apart(fmm, prec, n, nt):
    """An infinite charge gives infinite sums at every other point (and NaN,
    0 times infinity, at its own), whatever the number of charges."""
    _say(f"[direct, infinite charge] {prec} n={n} nt={nt}")
    rng = np.random.default_rng(50 + n)
    pos, q = rng.random((n, 3)), rng.uniform(-1, 1, n)
    q[0] = np.inf
    tg = rng.integers(0, n, nt)
    tg[0] = 0
    dt = torch.float64 if prec == "fp64" else torch.float32
    u, f = fmm.direct(torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda().to(dt),
                      torch.from_numpy(tg).cuda())
    u, f = u.cpu().numpy(), f.cpu().numpy()
    away = tg != 0
    assert np.all(np.isnan(u[~away]))
    assert np.all(u[away] == -np.inf)  # u = -1/(4 pi) sum q / r
    assert np.array_equal(f[away], -np.inf * np.sign(pos[tg[away]] - pos[0]))


def _near_reference(pos, q, skip):
    """Direct sums in FP64 without the pairs of the points in skip."""
    d = pos[:, None] - pos[None]
    r2 = (d * d).sum(-1)
    np.fill_diagonal(r2, np.inf)
    for a in skip:
        for b in skip:
            r2[a, b] = np.inf
    w = q[None] / np.sqrt(r2)
    with np.errstate(over="ignore", invalid="ignore"):
        return -w.sum(1) / (4 * np.pi), -((w / r2)[..., None] * d).sum(1) / (4 * np.pi)


# pairs whose squared distance is 0 in the plan's precision though the points
# differ, on both sides of a median split (so in different leaves): about the
# origin, and about odd multiples of half the cell by which near points are
# looked for
@pytest.mark.parametrize("prec,rhs,gap", [("fp32", 1, 1e-25), ("fp32", 8, 1e-25),
                                          ("fp64", 1, 1e-170)])
@pytest.mark.parametrize("where", ["origin", "edge", "corner"])
@pytest.mark.parametrize("axis,n", [(0, 200), (2, 1200)])
def test_pairs_too_close_to_tell_apart_contribute_nothing(fmm, prec, rhs, gap, where, axis, n):
    _say(f"[close points] {prec} {rhs} vectors gap {gap} {where} axis {axis} n={n}")
    rng = np.random.default_rng(60)
    pos = rng.uniform(0.1, 1.0, (n, 3))
    pos[: n // 2, axis] *= -1.0
    pos[:, axis] *= 4.0  # the axis of the first split
    half = (2.0 ** -51 if prec == "fp32" else 2.0 ** -501)
    along = [axis] if where != "corner" else [0, 1, 2]
    a, b = 3, n - 4
    pos[a] = pos[b] = 0.0
    for k in along:
        c = 0.0 if where == "origin" else 3 * half
        # (a gap below the spacing of numbers about c rounds away: then a is
        # the next number below)
        pos[a, k] = min(c - gap, np.nextafter(c, -1.0))
        pos[b, k] = c + gap
        d = pos[b, k] - pos[a, k]
        assert d > 0 and (np.float32(d) ** 2 if prec == "fp32" else d * d) == 0
    dt = torch.float64 if prec == "fp64" else torch.float32
    Q = torch.from_numpy(rng.uniform(-1, 1, (rhs, n))).to(dt)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=2, leaf_max=n // 4, splits=2, theta=0.01,
                    precision=prec, max_rhs=rhs)
    assert plan.info()["n_m2l"] == 0  # near field only
    perm, starts = plan.tree()[:2]
    leaf = np.searchsorted(starts, np.argsort(perm)[[a, b]], "right")
    assert leaf[0] != leaf[1]
    U, F = plan.evaluate(Q.cuda() if rhs > 1 else Q[0].cuda())
    U, F = U.reshape(rhs, n).double().cpu().numpy(), F.reshape(rhs, n, 3).double().cpu().numpy()
    tol = 1e-12 if prec == "fp64" else 1e-5
    for r in range(rhs):
        u0, f0 = _near_reference(pos, Q[r].double().numpy(), (a, b))
        assert np.abs(U[r] - u0).max() <= tol * np.abs(u0).max()
        assert np.abs(F[r] - f0).max() <= tol * np.abs(f0).max()


@pytest.mark.parametrize("prec,far", [("fp32", 1e-15), ("fp64", 1e-150)])
def test_near_points_that_can_be_told_apart_still_count(fmm, prec, far):
    """A pair of one search cell whose distance can be told from 0."""
    _say(f"[close points] {prec} told apart at {far}")
    rng = np.random.default_rng(61)
    pos = rng.uniform(0.1, 1.0, (60, 3))
    pos[:30, 0] *= -4.0
    pos[30:, 0] *= 4.0
    pos[3], pos[40] = 0.0, 0.0
    pos[3, 0], pos[40, 0] = -far / 8, far / 8
    q = rng.uniform(0.5, 1, 60)
    dt = torch.float64 if prec == "fp64" else torch.float32
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=2, leaf_max=16, splits=2, theta=0.01,
                    precision=prec)
    u, _ = plan.evaluate(torch.from_numpy(q).cuda().to(dt), field=False)
    u0, _ = _near_reference(pos, q, ())
    u = u.double().cpu().numpy()
    tol = 1e-12 if prec == "fp64" else 1e-5
    assert np.all(np.abs(u - u0) <= tol * np.abs(u0))
