"""The near field's forms against each other.

A leaf's form depends on its size, its direct list and the number of work
items of the whole plan, so the leaves of one problem take other forms when
the problem is evaluated by itself and inside a set of many.  In FP32 every
form adds the same terms in the same order: the results agree bit for bit.
"""
import ctypes
import sys

import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ONE_WAVE = 0  # fmm_near_runs: threads of an item's block, 0 for one wave


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def fmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_15269_amd as F
    return F


def _forms(plan, field):
    """{threads of a block (0: one wave, one target a lane): items}"""
    from paper_2511_15269_amd import _lib
    threads, items = (ctypes.c_int * 4)(), (ctypes.c_int64 * 4)()
    n = _lib.lib().fmm_near_runs(plan._h, 0, int(field), threads, items)
    assert 0 < n <= 4
    out = {}
    for k in range(n):
        if items[k]:
            out[threads[k]] = out.get(threads[k], 0) + items[k]
    return out


def _plan(fmm, pos, leaf, sizes=None):
    return fmm.Plan(pos, p=2, leaf_max=leaf, splits=2, theta=0.8, precision="fp32", sizes=sizes)


def _problem(per_leaf, seed):
    n = 256 * per_leaf - 85  # 256 leaves of per_leaf points and of one less
    pos, q = workloads.uniform_cube(n, seed)
    return torch.from_numpy(pos).cuda(), torch.from_numpy(q).cuda().float()


# copies of a problem of 256 leaves: thousands and tens of thousands of items
# choose other forms (in a potential-only pass too); leaf sizes about the steps of two
# targets a thread in 64, 128 and 256 threads and about whole waves.  wide, pot:
# forms that have to be among those seen
@pytest.mark.parametrize("per_leaf,wide,pot", [
    (33, {256, 128, 64}, {256, 128, 64}), (42, {256, 128, 64}, {256, 128, 64}),
    (43, {256, 128, 64}, {256, 128, 64}), (49, {256, 128}, {256, 128}),
    (56, {256, ONE_WAVE}, {256, 64}), (64, {256, ONE_WAVE}, {256, 128, 64}),
    (65, {256, 128, ONE_WAVE}, {256, 128, 64}), (86, {256, 128, ONE_WAVE}, {256, 128}),
    (128, {256, ONE_WAVE}, {256, 128}), (130, {256, ONE_WAVE}, {256, ONE_WAVE}),
    (160, {256, ONE_WAVE}, {256, ONE_WAVE})])
def test_fp32_forms_agree_bit_for_bit(fmm, per_leaf, wide, pot):
    pos, q = _problem(per_leaf, 70)
    n = pos.shape[0]
    seen, seen_pot, ref = set(), set(), None
    for copies in (1, 8, 24, 80):
        plan = _plan(fmm, pos.repeat(copies, 1), per_leaf, [n] * copies if copies > 1 else None)
        assert plan.info()["nleaf"] == 256 * copies
        _say(f"[near forms] {per_leaf} a leaf, {copies} problems: {_forms(plan, True)}, "
             f"potential {_forms(plan, False)}")
        seen |= set(_forms(plan, True))
        seen_pot |= set(_forms(plan, False))
        u, f = plan.evaluate(q.repeat(copies))
        v, _ = plan.evaluate(q.repeat(copies), field=False)
        assert torch.equal(u, v)
        if ref is None:
            ref = u, f
        assert torch.equal(u, ref[0].repeat(copies))
        assert torch.equal(f, ref[1].repeat(copies, 1))
    assert wide <= seen and pot <= seen_pot


@pytest.mark.parametrize("per_leaf,leaves", [(160, 512), (200, 256), (256, 256)])
def test_potential_only_items_of_short_lists_keep_one_wave(fmm, per_leaf, leaves):
    """Leaves of more points than 128 threads take in one round of targets,
    whose items keep one wave with a field, keep it without one."""
    pos, _ = workloads.uniform_cube(per_leaf * leaves, 75)
    plan = fmm.Plan(torch.from_numpy(pos).cuda(), p=2, leaf_max=per_leaf, splits=1, theta=0.8,
                    precision="fp32")
    items = plan.info()["p2p_items"]
    _say(f"[near forms] {leaves} leaves of {per_leaf}: {_forms(plan, True)}, "
         f"potential {_forms(plan, False)}")
    assert 5000 < items < 14500
    assert _forms(plan, True) == _forms(plan, False) == {ONE_WAVE: items}


def test_potential_only_items_of_leaves_larger_than_the_block(fmm):
    """The remaining items of a potential-only pass take one form by their
    mean size: larger leaves among them run in several rounds of targets."""
    small, qs = _problem(56, 71)
    large, ql = _problem(128, 72)
    k = 72
    plan = _plan(fmm, torch.cat([small] * k + [large]), 128,
                 [small.shape[0]] * k + [large.shape[0]])
    _say(f"[near forms] mixed: {_forms(plan, True)}, potential {_forms(plan, False)}")
    assert _forms(plan, True)[ONE_WAVE] > 18000 and _forms(plan, False)[64] > 18000
    q = torch.cat([qs] * k + [ql])
    u, f = plan.evaluate(q)
    v, _ = plan.evaluate(q, field=False)
    assert torch.equal(u, v)
    for pos, qq, at in ((small, qs, 0), (large, ql, small.shape[0] * k)):
        u0, f0 = _plan(fmm, pos, 128).evaluate(qq)
        assert torch.equal(u[at:at + qq.shape[0]], u0)
        assert torch.equal(f[at:at + qq.shape[0]], f0)


# sources in leaves of a few points: runs of direct lists of more leaves than a
# block has threads
@pytest.mark.parametrize("prec,tol,leaf,splits,ns,nt", [
    ("fp32", 1e-5, 33, 3, 6500, 264), ("fp32", 1e-5, 64, 3, 6500, 512),
    ("fp64", 1e-12, 2, 1, 900, 16), ("fp64", 1e-12, 4, 1, 3000, 30)])
def test_lists_longer_than_the_block(fmm, prec, tol, leaf, splits, ns, nt):
    from oracle.direct import direct
    src, q = workloads.uniform_cube(ns, 73)
    tgt, _ = workloads.uniform_cube(nt, 74)
    dt = torch.float64 if prec == "fp64" else torch.float32
    plan = fmm.Plan(torch.from_numpy(src).cuda(), p=2, leaf_max=leaf, splits=splits, theta=0.01,
                    precision=prec, targets=torch.from_numpy(tgt).cuda())
    inf = plan.info()
    _say(f"[near forms] {prec} {inf['n_p2p']} leaf pairs in {inf['p2p_items']} items: "
         f"{_forms(plan, True)}")
    assert inf["n_m2l"] == 0 and inf["n_p2p"] > 64 * inf["p2p_items"]
    Q = torch.from_numpy(abs(q) + 0.5).cuda().to(dt)
    u, f = plan.evaluate(Q)
    u0, g0 = direct(src, Q.double().cpu().numpy(), tgt, field=True)
    assert abs(u.double().cpu().numpy() - u0).max() <= tol * abs(u0).max()
    assert abs(f.double().cpu().numpy() + g0).max() <= tol * abs(g0).max()
