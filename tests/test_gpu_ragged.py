"""The kernels at the edges of their tiles and rules.

* Uniform grids of 1, 2, 27, 3072, 3136 and 3179 elements: fewer elements than a
  wave has lanes, one element per workgroup and (over 3072) two, the last one of
  an odd count alone. Matrix and residual, residual alone and Jacobian action
  against the reference; in the mixed forms residual alone and residual beside
  the matrix are the same bits.
* Two boxes and a sphere: the overlapped schedule, whose second stream is limited
  in one and not in the other, against the in-order one, bit for bit.
* Triquadratic grids of 1, 6 and 576 elements (persistent workgroups: 512).
* Network gradients of 1 sample, around one tile of 64 and over 512 tiles.

Tolerances: FP64 1e-12 of the norm (sums of under 10^3 terms of similar size,
10^3 eps with a margin of 5); mixed forms and the FP32 network 1e-5 (FP32 products
and sums of under 10^2 terms, 10^2 eps = 6e-6).
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


def grid(nx, ny, nz, level):
    return I.refined_octree(level, level, lambda x, y, z, h, l: np.zeros(x.shape, bool), ext=(nx, ny, nz))


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec,tol", [("VMS_FP64", 1e-12), ("VMS_MIXED_BF16", 1e-5), ("VMS_MIXED_FP16", 1e-5)])
@pytest.mark.parametrize("ext", [(1, 1, 1, 1), (1, 2, 1, 2), (3, 3, 3, 2), (16, 16, 12, 4), (16, 14, 14, 4),
                                 (17, 17, 11, 5)], ids=lambda e: str(e[0] * e[1] * e[2]))
def test_ragged_element_counts(env, oracle, ext, prec, tol):
    torch, vms = env
    t = grid(*ext)
    assert t.n == ext[0] * ext[1] * ext[2]
    ms = oracle.derive_mesh(t.ax, t.ay, t.az, t.level, t.max_level)
    asm = vms.Assembler(t, None, vms.make_params(precision=getattr(vms, prec)))
    f = I.make_fields(ms.node_xyz_int / float(1 << t.max_level) * t.root_len, 77)
    asm.set_fields(f)
    V, R = oracle.assemble(t, ms, f)
    x = np.random.default_rng(5).normal(size=R.size)
    y_ref = oracle.jacobian_apply(t, ms, f, x)
    asm.assemble()
    vals, res = asm.vals.cpu().numpy().astype(np.float64), asm.resid.clone()
    asm.apply()
    y = asm.jacobian_action(torch.as_tensor(x, device="cuda")).cpu().numpy()
    errs = [rel(vals, V), rel(res.cpu().numpy(), R), rel(asm.resid.cpu().numpy(), R), rel(y, y_ref)]
    print(f"{t.n} elements {prec}: J {errs[0]:.1e}, R {errs[1]:.1e}, R alone {errs[2]:.1e}, Jx {errs[3]:.1e}", flush=True)
    assert max(errs) <= tol
    if prec != "VMS_FP64":
        assert torch.equal(asm.resid, res)
    asm.close()


@pytest.mark.parametrize("prec", ["VMS_FP64", "VMS_MIXED_BF16"])
@pytest.mark.parametrize("geometry", ["boxes", "sphere"])
def test_schedules_agree(env, geometry, prec):
    torch, vms = env
    tree, surf = I.two_box_workload(5, 9, 8.0, 30) if geometry == "boxes" else I.sphere_workload(4, 7, 4.0, 3, 0.15)
    asm = vms.Assembler(tree, surf, vms.make_params(quad_depth=3, precision=getattr(vms, prec)))
    xyz = asm.export(vms.VMS_EXPORT_NODE_XYZ).T / float(1 << tree.max_level) * tree.root_len + np.asarray(tree.origin)
    asm.set_fields(I.make_fields(xyz, 78))
    outs = []
    for overlap, timing in ((False, False), (True, False), (True, True), (True, False)):
        vms.vms_set_overlap(asm.ctx, overlap)
        vms.vms_set_timing(asm.ctx, timing)
        asm.assemble(flags=vms.VMS_RELABEL)
        torch.cuda.synchronize()
        outs.append((asm.vals.clone(), asm.resid.clone()))
        asm.vals.zero_()
        asm.resid.zero_()
    for v, r in outs[1:]:
        assert torch.equal(v, outs[0][0]) and torch.equal(r, outs[0][1])
    asm.close()


@pytest.mark.parametrize("ext", [(1, 1, 1, 1), (3, 2, 1, 2), (9, 8, 8, 4)], ids=lambda e: str(e[0] * e[1] * e[2]))
def test_q2_ragged_element_counts(env, oracle, ext):
    torch, vms = env
    from oracle import q2 as Q
    t = grid(*ext)
    m = Q.derive_q2_mesh(t)
    q = vms.vms_q2_create(t)
    f = I.make_fields(Q.node_xyz(t, m), 79)
    fd = {k: torch.as_tensor(f[k], device="cuda") for k in f}
    vals = torch.zeros(m.nnz, dtype=torch.float64, device="cuda")
    res = torch.zeros(4 * m.n_nodes, dtype=torch.float64, device="cuda")
    vms.vms_q2_assemble(q, fd, vals, res)
    torch.cuda.synchronize()
    V, R = Q.assemble(t, m, f)
    errs = rel(vals.cpu().numpy(), V), rel(res.cpu().numpy(), R)
    print(f"Q2 {t.n} elements: J {errs[0]:.1e}, R {errs[1]:.1e}", flush=True)
    assert max(errs) <= 1e-12
    vms.vms_q2_destroy(q)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 32768 + 65])
def test_network_gradient_ragged_batches(env, n):
    torch, vms = env
    from oracle import mlp as M
    lo, hi = np.zeros(3), np.ones(3)
    th, B = M.init_params(7).astype(np.float32), M.fourier_matrix(7, 2.0).astype(np.float32)
    rng = np.random.default_rng(n)
    x, sdf = rng.uniform(lo, hi, (n, 3)), rng.normal(0, 0.05, n)
    h = vms.vms_mlp_create(lo, hi, th, B, 0.05)
    p = [torch.as_tensor(np.ascontiguousarray(x[:, k]), device="cuda") for k in range(3)]
    g = torch.zeros(M.N_PARAMS, dtype=torch.float32, device="cuda")
    loss = vms.vms_mlp_grad(h, *p, torch.as_tensor(sdf, device="cuda"), g)
    ref_loss, ref = M.loss_and_grad(th.astype(np.float64), x, sdf, lo, hi, B.astype(np.float64), 0.05)
    err = rel(g.cpu().numpy().astype(np.float64), ref)
    print(f"{n} samples: gradient {err:.1e}, loss {abs(loss - ref_loss) / ref_loss:.1e}", flush=True)
    assert err <= 1e-5 and abs(loss - ref_loss) <= 1e-5 * ref_loss
    vms.vms_mlp_destroy(h)
