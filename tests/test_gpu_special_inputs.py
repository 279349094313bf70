"""Inputs outside the ordinary: infinite charges."""
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
