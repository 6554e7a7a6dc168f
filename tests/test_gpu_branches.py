"""Branches that ordinary inputs do not reach, and kernels that must agree.

* The residual alone and the residual beside the matrix come from two kernels. In the
  mixed forms they are the same bits (each states the order of every rounding), in
  FP64 the same sums in another order: on hanging nodes and on cut elements whose
  items hold point counts that are no multiple of 8, 16 or 64. FP64 tolerance:
  items of up to 128 points of similar size, 10^3 eps = 2e-13 of the norm.
* Steps of BiCGStab that end early (rh . v = 0, |s| small, t = 0, omega = 0) and
  GMRES on an operator that closes the space at once: systems of two coupled nodes
  with dyadic entries, where every product and quotient is exact.
* The second stream of the overlapped schedule unlimited, with limited items, with a
  limited relabel too, and started after the OUT elements: the limits are the ones
  meant, and the outputs equal those in order bit for bit.
* OUT elements two per workgroup, the last of an odd count alone, in every form: the
  matrix against the matrix-free action (FP64 1e-12, mixed 1e-5 of the norm: sums of
  under 10^3 products in FP64, FP32 products of under 10^2 terms).
* Labels of points whose bin holds more triangles than one numbering of a wave's
  pairs takes.
"""
import numpy as np
import pytest

from paper_2009_00706_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2009_00706_amd import vms
    vms.lib()
    return torch, vms


def context(vms, tree, surf, prec, seed=81):
    asm = vms.Assembler(tree, surf, vms.make_params(quad_depth=3, precision=getattr(vms, prec)))
    xyz = asm.export(vms.VMS_EXPORT_NODE_XYZ).T / float(1 << tree.max_level) * tree.root_len + np.asarray(tree.origin)
    asm.set_fields(I.make_fields(xyz, seed))
    return asm


@pytest.mark.parametrize("prec", ["VMS_FP64", "VMS_MIXED_BF16", "VMS_MIXED_FP16"])
@pytest.mark.parametrize("geometry", ["hanging", "cut", "cut and hanging"])
def test_residual_alone_equals_the_one_beside_the_matrix(env, oracle, geometry, prec):
    torch, vms = env
    c = tuple(0.5 + o for o in I.BODY_OFFSET)
    if geometry == "hanging":
        tree, surf = I.sphere_refined_octree(c, 0.3, 3, 6, 1.5), None
    elif geometry == "cut":
        tree, surf = I.uniform_octree(4), I.icosphere(3, 0.3, c)
    else:  # the surface off the refined shell: cut elements with hanging corners
        tree, surf = I.sphere_refined_octree(c, 0.2, 3, 6, 1.5), I.icosphere(3, 0.24, c)
    asm = context(vms, tree, surf, prec)
    print(f"[paths] {geometry} {prec}: {tree.n} octants", flush=True)
    if surf is not None:
        counts = np.unique(asm.export(vms.VMS_EXPORT_SUBGP)["el"], return_counts=True)[1]
        assert counts.max() > 64 and all((counts % k).any() for k in (8, 16, 64))
    if "hanging" in geometry:
        ms = oracle.derive_mesh(tree.ax, tree.ay, tree.az, tree.level, tree.max_level)
        hang = ms.vertex_is_hanging[ms.elem_vertex].any(1)
        assert hang[asm.export(vms.VMS_EXPORT_MARKERS) == (2 if surf else 0)].sum() > 50
    asm.assemble()
    beside = asm.resid.clone()
    asm.resid.fill_(float("nan"))
    asm.apply()
    torch.cuda.synchronize()
    assert torch.isfinite(beside).all()
    err = (torch.linalg.vector_norm(asm.resid - beside) / torch.linalg.vector_norm(beside)).item()
    print(f"[paths] {geometry} {prec}: difference {err:.2e}", flush=True)
    assert err <= 2e-13 if prec == "VMS_FP64" else torch.equal(asm.resid, beside)
    asm.close()


# 2 x 2 operator [[1, c], [d, 1]] (times the 4 x 4 identity) between two neighbouring
# nodes, right-hand side, and what BiCGStab does with it: x, steps, |b - A x| / |b|
ENDS = {
    "s small": (0.0, 0.0, (3.0, 5.0), (3.0, 5.0), 1, 0.0),
    "t = 0": (2.0, 0.5, (1.0, 2.0), (0.5, 1.0), 1, 0.75),
    "rh . v = 0": (-3.0, 1.0, (1.0, 1.0), (0.0, 0.0), 0, 1.0),
    "omega = 0": (0.0, 2.0, (1.0, 1.0), (0.5, 0.5), 1, 0.5),
}


def two_node_system(env, prec, c, d, b):
    """Identity but for nodes 0 and 1, which are coupled by c and d."""
    torch, vms = env
    asm = context(vms, I.uniform_octree(1), None, prec)
    rp, ci = asm.export(vms.VMS_EXPORT_ROW_PTR), asm.export(vms.VMS_EXPORT_COL_IDX)
    row = np.repeat(np.arange(rp.size - 1), np.diff(rp))
    same = (row & 3) == (ci & 3)
    v = (row == ci).astype(np.float64)
    for i, j, w in ((0, 1, c), (1, 0, d)):
        at = (row >> 2 == i) & (ci >> 2 == j) & same
        assert at.sum() == 4
        v[at] = w
    asm.vals.copy_(torch.as_tensor(v))
    rhs = np.zeros(rp.size - 1)
    rhs[:4], rhs[4:8] = b
    return asm, torch.as_tensor(rhs, device="cuda")


@pytest.mark.parametrize("prec", ["VMS_FP64", "VMS_MIXED_BF16"])
@pytest.mark.parametrize("case", list(ENDS))
def test_bicgstab_steps_that_end_early(env, case, prec):
    torch, vms = env
    c, d, b, want, steps, rr_want = ENDS[case]
    asm, rhs = two_node_system(env, prec, c, d, b)
    x, it, rr = asm.solve(rhs, method=vms.VMS_KSP_BCGS, max_iter=9, rtol=1e-12, dirichlet=False)
    torch.cuda.synchronize()
    got = x.cpu().numpy()
    print(f"[ends] {case} {prec}: {it} steps, residual {rr}", flush=True)
    assert it == steps and rr == pytest.approx(rr_want, abs=1e-14)
    assert np.array_equal(got[:8], np.repeat(want, 4)) and not got[8:].any()
    asm.close()


def test_gmres_ends_when_the_space_closes(env):
    torch, vms = env
    asm, rhs = two_node_system(env, "VMS_FP64", 0.0, 0.0, (3.0, 4.0))
    x, it, rr = asm.solve(rhs, method=vms.VMS_KSP_GMRES, restart=5, max_iter=9, rtol=1e-12, dirichlet=False)
    torch.cuda.synchronize()
    assert it == 1 and rr <= 1e-15 and torch.linalg.vector_norm(x - rhs) <= 1e-14
    asm.close()


def test_labels_where_one_bin_holds_very_many_triangles(env):
    """A sphere of 81,920 triangles far smaller than a bin beside a large one: the
    points in its bin have more pairs than the wave's points are numbered for
    together, so each point's pairs are numbered alone."""
    torch, vms = env
    cs, rs, cb, rb = np.array([2.0, 0.51, 0.49]), 1e-5, np.array([0.5, 0.5, 0.5]), 0.5
    surf = I.merge_surfaces([I.icosphere(3, rb, cb), I.icosphere(6, rs, cs)])
    rng = np.random.default_rng(4)
    d = rng.normal(size=(40, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    near = cs + d * (rs * rng.choice([0.3, 0.9, 1.1, 3.0], 40))[:, None]       # in the small sphere's bin
    line = np.column_stack([rng.uniform(-0.2, 2.2, 20), np.full(20, cs[1]), np.full(20, cs[2])])
    wide = rng.uniform([-0.1, 0.0, 0.0], [2.1, 1.0, 1.0], (400, 3))
    p = rng.permutation(np.concatenate([near, line, wide]))
    # inside either, the icospheres' facets within 1% of their radius
    ds, db = np.linalg.norm(p - cs, axis=1) / rs, np.linalg.norm(p - cb, axis=1) / rb
    sure = (np.abs(ds - 1) > 0.02) & (np.abs(db - 1) > 0.02)
    want = ((ds < 1) | (db < 1)).astype(np.uint8)
    assert sure.sum() > 400 and 10 < want[sure].sum() < sure.sum()
    px, py, pz = (torch.as_tensor(np.ascontiguousarray(p[:, k]), device="cuda") for k in range(3))
    lab = torch.full((p.shape[0],), 7, dtype=torch.uint8, device="cuda")
    print(f"[labels] {surf.n_tri} triangles, {p.shape[0]} points", flush=True)
    vms.inout_classify(surf, px, py, pz, lab)
    torch.cuda.synchronize()
    assert np.array_equal(lab.cpu().numpy()[sure], want[sure])


# geometry, precision, relabel, whether (items, relabel) are limited
PLANS = [("sphere", "VMS_FP64", 1, (False, False)), ("boxes", "VMS_FP64", 1, (True, True)),
         ("boxes", "VMS_FP64", 0, (True, False)), ("boxes", "VMS_MIXED_BF16", 1, (True, True)),
         ("boxes", "VMS_MIXED_BF16", 0, (True, False)),  # starts after the OUT elements
         ("finer boxes", "VMS_MIXED_FP16", 1, (True, False)), ("finest boxes", "VMS_FP64", 1, (False, False))]


@pytest.mark.parametrize("geometry,prec,relabel,limited", PLANS)
def test_plans_of_the_second_stream(env, geometry, prec, relabel, limited):
    torch, vms = env
    n_face = {"boxes": 30, "finer boxes": 45, "finest boxes": 91}
    tree, surf = I.sphere_workload(4, 7, 4.0, 3, 0.15) if geometry == "sphere" else \
        I.two_box_workload(5, 9, 8.0, n_face[geometry])
    asm = context(vms, tree, surf, prec)
    outs = []
    for overlap in (False, True, True):
        vms.vms_set_overlap(asm.ctx, overlap)
        asm.vals.fill_(float("nan"))
        asm.resid.fill_(float("nan"))
        asm.assemble(flags=vms.VMS_RELABEL * relabel)
        torch.cuda.synchronize()
        outs.append((asm.vals.clone(), asm.resid.clone()))
        got = vms.vms_overlap_limits(asm.ctx)
        print(f"[plans] {geometry} {prec} relabel {relabel} overlap {overlap}: limits {got}", flush=True)
        assert (got[0] > 0, got[1] > 0) == (limited if overlap else (False, False))
    asm.apply()   # has no second stream: the limits stay those of the assembly
    assert vms.vms_overlap_limits(asm.ctx) == got
    for v, r in outs[1:]:
        assert torch.equal(v, outs[0][0]) and torch.equal(r, outs[0][1])
    assert torch.isfinite(outs[0][0]).all()
    vms.vms_sizes(asm.ctx)
    asm.close()


def test_overlap_limits_reject_null():
    from paper_2009_00706_amd import vms
    assert vms.lib().vms_overlap_limits(None, None) == vms.VMS_EINVAL


@pytest.mark.parametrize("prec,tol", [("VMS_FP64", 1e-12), ("VMS_MIXED_BF16", 1e-5), ("VMS_MIXED_FP16", 1e-5)])
def test_out_elements_two_per_workgroup(env, prec, tol):
    torch, vms = env
    tree = I.refined_octree(5, 5, lambda x, y, z, h, l: np.zeros(x.shape, bool), ext=(27, 27, 25))
    assert tree.n == 18225  # over four rounds of 16 workgroups on each of 256 CUs
    asm = context(vms, tree, None, prec)
    asm.vals.fill_(float("nan"))
    asm.assemble()
    beside = asm.resid.clone()
    asm.apply()
    x = torch.as_tensor(np.random.default_rng(6).normal(size=asm.sizes["n_rows"]), device="cuda")
    a, b = asm.spmv(x), asm.jacobian_action(x)
    torch.cuda.synchronize()
    err = (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()
    res = (torch.linalg.vector_norm(asm.resid - beside) / torch.linalg.vector_norm(beside)).item()
    print(f"[two] {prec}: J x {err:.1e}, residual {res:.1e}", flush=True)
    assert err <= tol and res <= 2e-13
    if prec != "VMS_FP64":
        assert torch.equal(asm.resid, beside)
    asm.close()
