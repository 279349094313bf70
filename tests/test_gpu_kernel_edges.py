"""Edges of the tiles, forms and pools that the kernels and plans choose among.

Bounds are those of the other parity tests, for the same reasons: FP64 sums
of the same terms in another order stay within 1e-10 of the oracle FMM (1e-13
for a plain sum), FP32 within 1e-5.
"""
import sys
import threading

import numpy as np
import pytest

import workloads
from _norms import parity as _rel

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


# targets around the steps of the targets per wave (512, 1024) and of the
# slices; sources around a wave's 64 lanes
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("fp32", 1e-5)])
@pytest.mark.parametrize("n,nt", [(2, 1), (63, 17), (64, 255), (65, 257), (1000, 511),
                                  (1025, 512), (700, 1023), (129, 1025), (300, 4099)])
def test_direct_sum_target_and_source_edges(fmm, prec, tol, n, nt):
    from oracle.direct import direct
    _say(f"[direct edges] {prec} n={n} nt={nt}")
    pos, q = workloads.uniform_cube(n, 30)
    q = np.abs(q) + 0.5  # no cancellation: the bounds are relative to the sums
    tg = np.random.default_rng(31).integers(0, n, nt)
    dt = torch.float64 if prec == "fp64" else torch.float32
    args = (torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda().to(dt),
            torch.from_numpy(tg).cuda())
    u, f = fmm.direct(*args)
    u1, _ = fmm.direct(*args, field=False)
    ud, gd = direct(pos, q, pos[tg], field=True)
    assert _rel(u.double().cpu().numpy(), ud) <= tol
    assert _rel(f.double().cpu().numpy(), -gd) <= tol
    assert torch.equal(u, u1)


# leaf sizes on both sides of the near field's forms: two targets a thread in
# blocks of 64 or 128, whole waves, more targets than a block holds; most and
# least points of a leaf differ by one
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("per_leaf", [4, 5, 15, 16, 17, 31, 32, 33, 42, 43, 49, 63, 64, 65, 86,
                                      100, 127, 128, 129, 200, 256, 257, 300])
def test_near_field_leaf_size_edges(fmm, prec, tol, per_leaf):
    from oracle.fmm import fmm as oracle_fmm
    n = 16 * per_leaf - 3
    _say(f"[near-field forms] {prec} {per_leaf} points a leaf")
    pos, q = workloads.uniform_cube(n, 32)
    if per_leaf % 3 == 0:
        pos[n // 2] = pos[1]  # coincident points in different leaves
    u0, f0 = oracle_fmm(pos, q, 4, per_leaf, 2, 0.6)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=4, leaf_max=per_leaf, splits=2, theta=0.6,
                    precision=prec)
    qt = torch.from_numpy(q).cuda().to(torch.float64 if prec == "fp64" else torch.float32)
    u, f = plan.evaluate(qt)
    assert _rel(u.double().cpu().numpy(), u0) <= tol
    assert _rel(f.double().cpu().numpy(), f0) <= tol
    u1, _ = plan.evaluate(qt, field=False)
    assert torch.equal(u, u1)


# targets and sources of unlike leaf sizes (source leaves of more points than
# a block stages at a time, target leaves of a few)
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("ns,nt,leaf", [(300, 7, 300), (517, 40, 520), (70, 900, 128),
                                        (2000, 90, 128)])
def test_near_field_between_unlike_leaves(fmm, prec, tol, ns, nt, leaf):
    from oracle.fmm import fmm_st
    _say(f"[unlike leaves] {prec} {ns} charges {nt} targets leaf={leaf}")
    src, q = workloads.uniform_cube(ns, 33)
    tgt, _ = workloads.uniform_cube(nt, 34)
    u0, f0 = fmm_st(src, q, tgt, 5, leaf, 2, 0.6)
    plan = fmm.Plan(torch.from_numpy(src).cuda(), p=5, leaf_max=leaf, splits=2, theta=0.6,
                    precision=prec, targets=torch.from_numpy(tgt).cuda())
    u, f = plan.evaluate(torch.from_numpy(q).cuda().to(
        torch.float64 if prec == "fp64" else torch.float32))
    assert _rel(u.double().cpu().numpy(), u0) <= tol
    assert _rel(f.double().cpu().numpy(), f0) <= tol


# every order's M2L (its waves per block, its lanes per item)
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("p", range(1, 11))
def test_m2l_of_every_order(fmm, prec, tol, p):
    from oracle.fmm import fmm as oracle_fmm
    _say(f"[M2L] {prec} p={p}")
    pos, q = workloads.uniform_cube(2900, 35)
    u0, f0 = oracle_fmm(pos, q, p, 24, 2, 0.7)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=p, leaf_max=24, splits=2, theta=0.7,
                    precision=prec)
    u, f = plan.evaluate(torch.from_numpy(q).cuda().to(
        torch.float64 if prec == "fp64" else torch.float32))
    assert _rel(u.double().cpu().numpy(), u0) <= tol
    assert _rel(f.double().cpu().numpy(), f0) <= tol


# vectors taken one by one, in one or two column halves, and in a second pass
# (coincident points: distance 0 is looked for everywhere)
@pytest.mark.parametrize("n,leaf", [(2600, 47), (17000, 64)])
@pytest.mark.parametrize("R", [4, 5, 6, 7, 16, 17, 37])
def test_vector_counts(fmm, n, leaf, R):
    from oracle.fmm import fmm as oracle_fmm
    _say(f"[vectors] n={n} R={R}")
    pos, _ = workloads.uniform_cube(n, 36)
    if n == 2600:
        pos[n // 2] = pos[1]
    Q = np.random.default_rng(37).uniform(-1, 1, (R, n))
    pt, Qt = torch.from_numpy(pos).cuda(), torch.from_numpy(Q).cuda().float()
    kw = dict(p=5, leaf_max=leaf, splits=2, theta=0.6, precision="fp32")
    U, Fd = fmm.Plan(pt, max_rhs=R, **kw).evaluate(Qt)
    single = fmm.Plan(pt, **kw)
    for r in range(R):
        u1, f1 = single.evaluate(Qt[r])
        assert _rel(U[r].double().cpu().numpy(), u1.double().cpu().numpy()) <= 1e-6
        assert _rel(Fd[r].double().cpu().numpy(), f1.double().cpu().numpy()) <= 1e-6
    u0, f0 = oracle_fmm(pos, Q[R - 1], 5, leaf, 2, 0.6)
    assert _rel(U[R - 1].double().cpu().numpy(), u0) <= 1e-5
    assert _rel(Fd[R - 1].double().cpu().numpy(), f0) <= 1e-5


def test_plans_made_and_dropped_share_no_state(fmm):
    """Plans of several sizes made, evaluated and dropped in turn, from two
    threads on their own streams and around a captured graph, give each time
    what the first plan of their size gave."""
    sizes = [1, 700, 5000, 12000]
    data = {}
    for n in sizes:
        pos, q = workloads.uniform_cube(n, 40 + n)
        pt, qt = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda()
        data[n] = (pt, qt, *fmm.Plan(pt, p=5, leaf_max=40).evaluate(qt))
    torch.cuda.synchronize()
    pt, qt, u0, f0 = data[5000]
    kept = fmm.Plan(pt, p=5, leaf_max=40)
    kept.evaluate(qt)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ug, fg = kept.evaluate(qt)
    bad = []

    def work():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for n in sizes * 3:
                p_, q_, u_, f_ = data[n]
                u, f = fmm.Plan(p_, p=5, leaf_max=40).evaluate(q_)
                stream.synchronize()
                if not (torch.equal(u, u_) and torch.equal(f, f_)):
                    bad.append(n)

    threads = [threading.Thread(target=work) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    torch.cuda.synchronize()
    assert not bad and not any(t.is_alive() for t in threads)
    for _ in range(3):
        ug.zero_()
        fg.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ug, u0) and torch.equal(fg, f0)


# a pass for each vector, or one for all: small plans and low orders take them
# together, where a pass alone is short against the pass of many
@pytest.mark.parametrize("n,leaf,s,p,R,passes", [
    (60, 32, 2, 6, 2, 1), (300, 32, 2, 5, 2, 1), (300, 32, 2, 5, 3, 1), (3000, 64, 2, 8, 3, 3),
    (3000, 64, 2, 8, 4, 1), (20000, 128, 3, 4, 5, 1), (20000, 128, 3, 4, 2, 2),
    (130000, 64, 2, 10, 5, 5), (130000, 64, 2, 10, 6, 1), (130000, 64, 2, 10, 37, 6)])
def test_few_vectors_take_the_quicker_way(fmm, n, leaf, s, p, R, passes):
    _say(f"[few vectors] n={n} p={p} R={R}")
    pos, _ = workloads.uniform_cube(n, 38)
    Q = torch.from_numpy(np.random.default_rng(39).uniform(-1, 1, (R, n))).cuda().float()
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=p, leaf_max=leaf, splits=s, theta=0.7,
                    precision="fp32", max_rhs=R)
    U, Fd = plan.evaluate(Q)
    plan.set_profiling(True)
    u, f = plan.evaluate(Q)
    assert plan.read_profile()[1] == passes
    assert torch.equal(u, U) and torch.equal(f, Fd)
    plan.set_profiling(False)
    u1, f1 = plan.evaluate(Q[R - 1])
    assert _rel(U[R - 1].double().cpu().numpy(), u1.double().cpu().numpy()) <= 1e-6
    assert _rel(Fd[R - 1].double().cpu().numpy(), f1.double().cpu().numpy()) <= 1e-6


# both directions' partial rows of split direct lists lie in one buffer
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_split_lists_of_both_directions_share_their_rows(fmm, prec):
    _say(f"[split lists] {prec} forward and transposed in turn")
    pos, q = workloads.clustered(24000, 41)
    dt = torch.float64 if prec == "fp64" else torch.float32
    pt, qt = torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda().to(dt)
    kw = dict(p=4, leaf_max=64, splits=2, theta=0.6, precision=prec)
    plan = fmm.Plan(pt, **kw)
    assert plan.info()["p2p_items"] > plan.info()["nleaf"]
    forward = fmm.Plan(pt, **kw).evaluate(qt)
    back = fmm.Plan(pt, **kw).evaluate_transposed(qt)
    for _ in range(2):
        for got, want in ((plan.evaluate(qt), forward), (plan.evaluate_transposed(qt), back)):
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
