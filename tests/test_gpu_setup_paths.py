"""GPU setup paths against a second formulation of the same thing, at the
sizes where their launches have edges."""
import numpy as np
import pytest

import workload

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("name,cons", [
    ("tiny3", ("corners",)),                      # fewer coarse DOFs than one launch's columns
    ("c3s", ("corners", "faces", "edges")),       # an odd count, uneven subregions
    ((24, 4), ("corners", "faces")),              # several launches, the last one partly filled
])
def test_explicit_coarse_operator_is_the_chain(name, cons):
    """The dense level-2 operator, assembled some hundred columns a launch, is
    the subregion chain: M^{-1} r equal to rounding (a sum of at most a few
    thousand products of size ~1: 1e-12 of the largest entry)."""
    torch = _torch()
    from paper_2412_17543_amd.solver import Solver
    if isinstance(name, tuple):
        nx, sub = name
        s = dict(nx=nx, elem_to_sub=workload.cube_partition(nx, sub), coef=np.ones(nx ** 3), elem_keep=None,
                 sub_to_subregion=workload.cube_subregions(nx // sub, 2))
    else:
        s = workload.workload(name)
    kw = dict(sub_to_subregion=s["sub_to_subregion"], elem_keep=s["elem_keep"], constraints=cons, autotune=False)
    a = Solver(s["nx"], s["elem_to_sub"], s["coef"], coarse_form="explicit", **kw)
    b = Solver(s["nx"], s["elem_to_sub"], s["coef"], coarse_form="chain", **kw)
    print("[gpu] %s %s: %d coarse DOFs" % (name, cons, a.info()["n_coarse"]), flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    for _ in range(2):
        r = torch.randn(a.n_gamma, dtype=torch.float64, device="cuda", generator=g)
        za, zb = a.apply_precond(r), b.apply_precond(r)
        assert (za - zb).abs().max().item() <= 1e-12 * zb.abs().max().item()


def _box(nx, cells):
    cell = (np.arange(nx) * cells) // nx
    return (cell[None, None, :] + cells * (cell[None, :, None] + cells * cell[:, None, None])).ravel().astype(np.int32)


@pytest.mark.parametrize("nx,part", [
    (4, _box(4, 2)),         # one interior node a subdomain, at most 19 interface nodes: rows within one wave
    (15, _box(15, 2)),       # 7^3 / 6^3 interiors, interfaces past 64 and 128 columns
    (15, _box(15, 3)),       # an interior of exactly 64 pivots beside 80 to 125
    (24, _box(24, 2)),       # 12^3 subdomains: 1,331 interior nodes and more, two dozen panels
    (6, np.minimum(np.arange(216) % 6, 2).astype(np.int32)),   # the middle slab has no interior node
])
def test_local_operators(nx, part):
    """Interior eliminations, saddle inverses and the couplings K_IB, K_BI at
    sizes around their panels and waves: the condensed right-hand side, A p,
    M^{-1} r and the recovered solution against the oracle's substructuring
    (local condition numbers up to ~1e3 on 1e-16 rounding: 1e-11 of the
    largest entry)."""
    torch = _torch()
    from oracle.sequence import OracleSolver
    from paper_2412_17543_amd.solver import Solver
    coef = workload.lognormal_coef(nx ** 3, 0.5)
    print("[gpu] couplings %d^3, %d subdomains" % (nx, part.max() + 1), flush=True)
    g = Solver(nx, part, coef, constraints=("corners", "faces"), autotune=False)
    o = OracleSolver(nx, part, coef)
    F = workload.rhs_sequence(nx, 1)
    b = g.condense(torch.tensor(F[0], device="cuda")).cpu().numpy()
    bo = o.ss.condense(F[0])
    bo = bo[0] if isinstance(bo, tuple) else bo
    assert np.abs(b - bo).max() <= 1e-11 * np.abs(bo).max()
    x = np.random.default_rng(nx).standard_normal(g.n_gamma)
    for got, want in ((g.apply_schur, o.ss.apply_A), (g.apply_precond, o.M.apply)):
        y, yo = got(torch.tensor(x, device="cuda")).cpu().numpy(), want(x)
        assert np.abs(y - yo).max() <= 1e-11 * np.abs(yo).max()
    U, its, rr = g.solve_sequence(torch.tensor(F, device="cuda"), 1e-12)
    uo, _, _ = o.solve_sequence(F, 1e-12)
    assert np.abs(U[0].cpu().numpy() - uo[0]).max() <= 1e-10 * np.abs(uo[0]).max()


@pytest.mark.parametrize("nx,part,cons,prec", [
    (8, _box(8, 2), ("corners", "faces"), 64),                 # 18 coarse DOFs
    (24, "c3s", ("corners", "edges"), 32),                    # an odd count, uneven subdomains
    (40, _box(40, 5), ("corners", "faces"), 16),               # 444: two passes of r_C, several groups of rows
    (20, _box(20, 5), ("corners", "faces", "edges"), 64),      # above the limit: both calls the separate kernels
])
def test_coarse_solve_inside_the_prolongation(nx, part, cons, prec):
    """Small coarse spaces are solved by the prolongation's own blocks, in the
    summation order of the separate kernels (which run while the kernel classes
    are timed): bitwise equal."""
    torch = _torch()
    from paper_2412_17543_amd.solver import Solver
    s = workload.workload("c3s") if isinstance(part, str) else dict(elem_to_sub=part, sub_to_subregion=None, elem_keep=None)
    g = Solver(nx, s["elem_to_sub"], workload.lognormal_coef(nx ** 3, 0.5), sub_to_subregion=s["sub_to_subregion"],
               elem_keep=s["elem_keep"], constraints=cons, local_prec=prec, autotune=False)
    print("[gpu] coarse solve in the prolongation: %d^3, %d coarse DOFs" % (nx, g.info()["n_coarse"]), flush=True)
    r = torch.randn(g.n_gamma, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    z = g.apply_precond(r)
    g.enable_timing(True)
    assert torch.equal(z, g.apply_precond(r))


@pytest.mark.parametrize("nx,cells,group,cons,form", [
    (24, 6, None, ("corners", "faces"), "auto"),             # two levels, 665 DOFs: 11 panels, 25 rows in the last
    (24, 6, 3, ("corners", "faces"), "explicit"),            # the same number in explicit form
    (27, 9, 3, ("corners",), "explicit"),                    # 512 DOFs: the most held as rows
    (20, 10, 5, ("corners", "faces"), "explicit"),           # 3,429 DOFs: 54 panels
    (24, 12, 2, ("corners", "edges", "faces"), "chain"),     # level 3 in panels (1,115 DOFs)
])
def test_coarse_operators_in_panels(nx, cells, group, cons, form):
    """Coarse operators on both sides of the size from which they are held in
    panels: M^{-1} r against the oracle (both are sums of at most a few thousand
    products of size ~1, through coarse matrices of condition up to ~1e4: 1e-11
    of the largest entry), and a block adjoint against the single ones (both
    solved to 1e-12: 1e-9)."""
    torch = _torch()
    from oracle.sequence import OracleSolver
    from paper_2412_17543_amd.solver import Solver
    part, coef = _box(nx, cells), workload.lognormal_coef(nx ** 3, 0.5)
    sr = None if group is None else workload.cube_subregions(cells, group)
    g = Solver(nx, part, coef, sub_to_subregion=sr, constraints=cons, coarse_form=form, autotune=False)
    print("[gpu] %d^3, %d^3 subdomains, %s: %d coarse DOFs" % (nx, cells, form, g.info()["n_coarse"]), flush=True)
    o = OracleSolver(nx, part, coef, sub_to_subregion=sr, constraints=cons)
    r = np.random.default_rng(nx).standard_normal(g.n_gamma)
    z, zo = g.apply_precond(torch.tensor(r, device="cuda")).cpu().numpy(), o.M.apply(r)
    assert np.abs(z - zo).max() <= 1e-11 * np.abs(zo).max()
    u = torch.tensor(workload.rhs_sequence(nx, 3), device="cuda")
    one, gf1 = g.adjoint_grad(u, u, 1e-12)
    blk, gfb, its = g.adjoint_grad_block(u, u, 1e-12)
    assert (one - blk).abs().max().item() <= 1e-9 * one.abs().max().item()
    assert (gf1 - gfb).abs().max().item() <= 1e-9 * gf1.abs().max().item()


@pytest.mark.parametrize("form,ncols", [("auto", 8), ("auto", 9), ("chain", 1), ("chain", 17), ("chain", 32)])
def test_block_prolongation(form, ncols):
    """Block adjoints of full and partly filled column groups, on a partition
    whose middle subdomain has over 128 coarse DOFs (a cube of 4^3 cells among
    152 single ones), two levels (coarse parts added by the prolongation) and a
    chain of three: each equals the column-by-column gradient, both solved to
    1e-12 (1e-9 of the largest entry)."""
    torch = _torch()
    from paper_2412_17543_amd.solver import Solver
    nx, cells = 12, 6
    cell = _box(nx, cells).astype(np.int64)
    xyz = np.stack([cell % cells, (cell // cells) % cells, cell // cells ** 2])
    cell[((xyz >= 1) & (xyz <= 4)).all(axis=0)] = -1
    ids, part = np.unique(cell, return_inverse=True)
    part = part.reshape(-1).astype(np.int32)
    sr = (ids >= 108).astype(np.int32) if form == "chain" else None
    g = Solver(nx, part, workload.lognormal_coef(nx ** 3, 0.5), sub_to_subregion=sr, coarse_form=form, autotune=False)
    print("[gpu] %s, %d columns: %d coarse DOFs" % (form, ncols, g.info()["n_coarse"]), flush=True)
    u = torch.tensor(workload.rhs_sequence(nx, ncols), device="cuda")
    one, gf1 = g.adjoint_grad(u, u, 1e-12)
    blk, gfb, its = g.adjoint_grad_block(u, u, 1e-12)
    assert (one - blk).abs().max().item() <= 1e-9 * one.abs().max().item()
    assert (gf1 - gfb).abs().max().item() <= 1e-9 * gf1.abs().max().item()


@pytest.mark.parametrize("nx,ncols,cons", [
    (24, 17, ("corners", "faces")),             # 386 interface nodes: 24 tile rows and a strip; 16 + 4 columns a block
    (24, 20, ("corners", "faces", "edges")),    # the same, 26 coarse DOFs (two groups of 16)
    (24, 21, ("corners", "faces")),             # two chunks of columns
    (27, 20, ("corners", "faces")),             # 488 interface nodes: above the LDS of two blocks
])
def test_block_products_with_four_more_columns(nx, ncols, cons):
    """Block adjoints around 16 columns equal the column-by-column ones, both
    solved to 1e-12 (1e-9 of the largest entry)."""
    torch = _torch()
    from paper_2412_17543_amd.solver import Solver
    g = Solver(nx, _box(nx, 3), workload.lognormal_coef(nx ** 3, 0.5), constraints=cons, autotune=False)
    print("[gpu] %d^3, %d columns: %d coarse DOFs" % (nx, ncols, g.info()["n_coarse"]), flush=True)
    u = torch.tensor(workload.rhs_sequence(nx, ncols), device="cuda")
    one, gf1 = g.adjoint_grad(u, u, 1e-12)
    blk, gfb, its = g.adjoint_grad_block(u, u, 1e-12)
    assert (one - blk).abs().max().item() <= 1e-9 * one.abs().max().item()
    assert (gf1 - gfb).abs().max().item() <= 1e-9 * gf1.abs().max().item()
