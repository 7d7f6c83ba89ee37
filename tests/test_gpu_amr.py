"""Adaptive refinement on the GPU (Sec. IV.A): refinement flags by the N_ref
criterion, box placement by the library's Berger-Rigoutsos clustering, and the
solve on the resulting tree of boxes (several per level, two levels deep),
against the oracle's tree solve."""
from __future__ import annotations

import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1511_08200_amd import ndgp, synth  # noqa: E402

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu-amr] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ndgp.lib()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / np.linalg.norm(np.ravel(b)))


def nref_flags(delta, n_particles, n_ref):
    return ((delta + 1.0) * n_particles / delta.size > n_ref).astype(np.uint8)


def build_tree(n=64, seed=31, n_particles=None, n_ref=20.0, n_ref1=2.0, max_level1=4):
    """Flags on the domain -> level-1 boxes; flags on the largest level-1 box
    (threshold n_ref1) -> level-2 boxes inside it.  Every flag array is the
    library's (ndgp_refine_flags) and equals the criterion's definition
    exactly."""
    f = synth.make_field(n, 1.0, seed, n_tophats=6)
    N = n**3 if n_particles is None else n_particles
    grid0 = ndgp.Grid(n=n, h=ndgp.cell_size(float(n), n))
    flags, counts = ndgp.refine_flags(grid0, [dev(f.delta)], N, n_ref)
    want = nref_flags(f.delta, N, n_ref)
    assert np.array_equal(flags[0].cpu().numpy(), want) and counts[0] == int(want.sum())
    boxes = ndgp.refine_boxes(flags[0], n, periodic=True)
    assert boxes == ndgp.refine_boxes(want, n, periodic=True)  # device and host flags agree
    boxes = sorted(boxes, key=lambda b: -b.n)[:max_level1]
    chains = [[b.origin] for b in boxes]
    deltas = [f.delta] + [synth.patch_delta(f, n, ch, b.n) for ch, b in zip(chains, boxes)]
    # level 2 inside the largest level-1 box: the box's own density and flags
    b0 = boxes[0]
    g1 = ndgp.Grid(n=n, h=grid0.h, patches=[ndgp.Patch(b0.n, b0.origin)])
    fl1, _ = ndgp.refine_flags(g1, [dev(deltas[0]), dev(deltas[1])], N, n_ref1)
    # a level-1 cell holds (delta + 1) N / (2n)^3 particles
    want1 = ((deltas[1] + 1.0) * N / (2 * n) ** 3 > n_ref1).astype(np.uint8)
    assert np.array_equal(fl1[1].cpu().numpy(), want1) and want1.sum() > 0
    kids = ndgp.refine_boxes(fl1[1], b0.n, periodic=False, parent_index=0)
    kids = sorted(kids, key=lambda b: -b.n)[:3]
    for k in kids:
        boxes.append(k)
        chains.append(chains[0] + [k.origin])
        deltas.append(synth.patch_delta(f, n, chains[-1], k.n))
    return f, grid0, boxes, deltas


def test_amr_tree_solve_matches_oracle():
    f, grid, boxes, deltas = build_tree()
    say(f"tree: {[(b.parent, b.n, b.origin) for b in boxes]}")
    assert len(boxes) >= 3 and any(b.parent >= 0 for b in boxes)
    rc = 1.0
    beta = O.beta_lcdm(1.0, 0.3, rc)
    tree = [(b.parent, b.n, b.origin) for b in boxes]
    phio, infos = O.solve_tree(deltas, grid.h, rc, beta, tree)
    assert all(i.status == 0 for i in infos)
    phig, rep, per_box = ndgp.solve_amr(grid, ndgp.Params(rc=rc, tol=0.0, max_cycles=200), boxes,
                                        [dev(d) for d in deltas])
    torch.cuda.synchronize()
    say(f"domain cycles={rep.cycles[0]}; boxes {per_box}")
    assert rep.status == 0
    for lvl in range(len(phig)):
        e = rel(phig[lvl].cpu().numpy(), phio[lvl])
        say(f"  level {lvl}: rel err {e:.2e}")
        assert e <= 1e-11
    # interpolated mode: every box is the oracle's interpolation of its GPU parent
    phii, rep_i, per_i = ndgp.solve_amr(grid, ndgp.Params(rc=rc, tol=1e-10,
                                                          mode=ndgp.MODE_INTERPOLATED),
                                        boxes, [dev(deltas[0])] + [None] * len(boxes))
    torch.cuda.synchronize()
    assert all(p["rel_res"] == -1.0 and p["cycles"] == 0 for p in per_i)
    host = [x.cpu().numpy() for x in phii]
    for b, x in enumerate(boxes):
        par = host[0] if x.parent < 0 else host[1 + x.parent]
        want = O.interpolate(par, x.parent < 0, x.origin, 0, x.n)
        assert np.abs(host[1 + b] - want).max() <= 1e-14 * np.abs(want).max()
    # truncated at depth 2: level-1 boxes relaxed (as in the full run), level 2 interpolated
    phit, rep_t, per_t = ndgp.solve_amr(grid, ndgp.Params(rc=rc, tol=0.0, max_cycles=200,
                                                          mode=ndgp.MODE_TRUNCATED,
                                                          trunc_level=2),
                                        boxes, [dev(d) for d in deltas])
    torch.cuda.synchronize()
    for b, x in enumerate(boxes):
        if x.parent < 0:
            assert torch.equal(phit[1 + b], phig[1 + b])
        else:
            assert per_t[b]["cycles"] == 0


def test_amr_rejects_bad_trees_and_inputs():
    f, grid, boxes, deltas = build_tree(max_level1=2)
    bad = list(boxes) + [ndgp.Box(len(boxes) + 3, 8, (0, 0, 0))]
    with pytest.raises(ndgp.NdgpError):
        ndgp.solve_amr(grid, ndgp.Params(rc=1.0), bad, [dev(d) for d in deltas] + [None])
    nan = [d.copy() for d in deltas]
    nan[1][2, 3, 4] = np.nan
    with pytest.raises(ndgp.NdgpError) as e:
        ndgp.solve_amr(grid, ndgp.Params(rc=1.0), boxes, [dev(d) for d in nan])
    assert e.value.status == ndgp.NDGP_EINVAL


def many_box_tree(n=128, seed=41, n_ref=12.0, n_ref1=2.0, deep=3):
    """A tree the way N_ref flags make it on a mildly clustered field (sigma_ln
    0.8, 12 top-hats; clustering efficiency 0.3): 74 boxes of 8^3 to 32^3
    (solved one workgroup each) and one of 64^3 (solved level by level), and
    inside the largest boxes the boxes their own flags ask for (a level-1 cell
    holds (delta + 1) N / (2n)^3 particles)."""
    f = synth.make_field(n, 0.8, seed, n_tophats=12)
    grid = ndgp.Grid(n=n, h=ndgp.cell_size(float(n), n))
    flags = nref_flags(f.delta, n**3, n_ref)
    boxes = ndgp.refine_boxes(flags, n, periodic=True, efficiency=0.3)
    chains = [[b.origin] for b in boxes]
    deltas = [f.delta] + [synth.patch_delta(f, n, ch, b.n) for ch, b in zip(chains, boxes)]
    parents = sorted(range(len(boxes)), key=lambda b: -boxes[b].n)[:deep]
    for p in parents:
        bp = boxes[p]
        fl = ((deltas[1 + p] + 1.0) * n**3 / (2 * n) ** 3 > n_ref1).astype(np.uint8)
        kids = ndgp.refine_boxes(fl, bp.n, periodic=False, parent_index=p, efficiency=0.7)
        for k in sorted(kids, key=lambda b: -b.n)[:4]:
            boxes.append(k)
            chains.append(chains[p] + [k.origin])
            deltas.append(synth.patch_delta(f, n, chains[-1], k.n))
    return f, grid, boxes, deltas


@pytest.mark.parametrize("case", ["tol", "stagnation", "damped"])
def test_small_boxes_in_one_launch_equal_box_by_box(case):
    """Boxes of at most 32^3 cells solved one workgroup each (all of a tree
    level in one launch) give the same bits, cycles, restart cycles, residuals
    and event counts as relaxing them one after the other (NDGP_TWO_PASS), on
    a tree with boxes of 8^3 to 64^3 at two depths."""
    f, grid, boxes, deltas = many_box_tree()
    sizes = sorted({b.n for b in boxes})
    say(f"{case}: {len(boxes)} boxes of sizes {sizes}, depths "
        f"{sorted({0 if b.parent < 0 else 1 for b in boxes})}")
    assert {8, 16, 32, 64} <= set(sizes) and any(b.parent >= 0 for b in boxes)
    kw = dict(rc=1.0, tol=1e-10)
    if case == "stagnation":
        kw = dict(rc=1.0, tol=0.0, max_cycles=200)
    if case == "damped":
        kw = dict(rc=5.0, tol=1e-10, damped=True)
    dd = [dev(d) for d in deltas]
    a, ra, pa = ndgp.solve_amr(grid, ndgp.Params(**kw), boxes, dd)
    b, rb, pb = ndgp.solve_amr(grid, ndgp.Params(two_pass=True, **kw), boxes, dd)
    torch.cuda.synchronize()
    say(f"  cycles {sorted({p['cycles'] for p in pa})}, domain {ra.cycles[0]}")
    assert ra.status == rb.status == 0
    assert pa == pb
    assert ra.fallbacks == rb.fallbacks and ra.holds == rb.holds
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    if case == "damped":
        assert all(p["damped_from"] == 1 for p in pa)


def test_small_boxes_reject_bad_density():
    f, grid, boxes, deltas = many_box_tree(deep=0)
    small = next(q for q, b in enumerate(boxes) if b.n <= 32)
    bad = [d.copy() for d in deltas]
    bad[1 + small][1, 2, 3] = np.inf
    with pytest.raises(ndgp.NdgpError) as e:
        ndgp.solve_amr(grid, ndgp.Params(rc=1.0), boxes, [dev(d) for d in bad])
    assert e.value.status == ndgp.NDGP_EINVAL


def test_empty_tree_is_the_plain_solve():
    """A tree with no boxes is ndgp_solve of the domain, bit for bit."""
    f = synth.make_field(32, 1.0, 5, n_tophats=2)
    grid = ndgp.Grid(n=32, h=ndgp.cell_size(64.0, 32))
    params = ndgp.Params(rc=1.0, tol=1e-10)
    d = dev(f.delta)
    a, ra, pa = ndgp.solve_amr(grid, params, [], [d])
    b, rb = ndgp.solve(grid, params, [d])
    torch.cuda.synchronize()
    assert pa == [] and ra.cycles[0] == rb.cycles[0] and ra.rel_res[0] == rb.rel_res[0]
    assert torch.equal(a[0], b[0])


@pytest.mark.parametrize("count", [6, 7])
def test_few_32_boxes_on_a_level_equal_box_by_box(count):
    """Six 32^3 boxes on a tree level are relaxed one after the other, seven in one
    launch: both give the bits and reports of the per-colour box-by-box path."""
    n, rng = 64, np.random.default_rng(60 + count)
    grid = ndgp.Grid(n=n, h=1.0)
    boxes = [ndgp.Box(-1, 32, (16 * (q % 4), 16 * (q // 4), 16 * (q % 3))) for q in range(count)]
    d0 = rng.lognormal(0.0, 0.8, (n,) * 3)
    dd = [dev(d0 - d0.mean())] + [dev(rng.lognormal(0.0, 0.8, (32,) * 3) - 1.3) for _ in boxes]
    a, b = (ndgp.solve_amr(grid, ndgp.Params(rc=1.0, tol=1e-10, two_pass=t), boxes, dd)
            for t in (False, True))
    torch.cuda.synchronize()
    assert a[1].status == b[1].status == 0 and a[2] == b[2]
    assert (a[1].fallbacks, a[1].holds) == (b[1].fallbacks, b[1].holds)
    assert all(torch.equal(x, y) for x, y in zip(a[0], b[0]))
