"""Forms chosen by size, at the sizes where they change: the block product with
the most tile rows, and the coarse solve inside and outside the prolongation."""
import numpy as np
import pytest

import workload

pytestmark = pytest.mark.gpu

FUSED_MAX_NC = 512                  # coarse DOFs solved for by the prolongation's blocks


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _around(nx, edge):
    """3 x 3 x 3 subdomains of an nx^3 cube, the middle one of edge[0] x edge[1] x
    edge[2] elements and away from the boundary: its nodes on its own boundary
    are its interface."""
    cell = []
    for e in edge:
        lo = (nx - e) // 2
        cell.append((np.arange(nx) >= lo).astype(np.int32) + (np.arange(nx) >= lo + e))
    x, y, z = cell
    return (x[None, None, :] + 3 * (y[None, :, None] + 3 * z[:, None, None])).ravel().astype(np.int32)


@pytest.mark.parametrize("edge,nB", [((9, 9, 10), 524), ((8, 9, 11), 520)])    # 33 tile rows, the last of 12 and 8
@pytest.mark.parametrize("ncols", [3, 20])
def test_block_product_with_the_most_tile_rows(edge, nB, ncols):
    """One interface above 512 nodes (a fifth group of tile columns a wave)
    beside small ones: the block adjoint equals the column-by-column one, both
    solved to 1e-12 (1e-9 of the largest entry).  The same subdomain's interior
    is above the block product's rows, so condensation and recovery go one by
    one."""
    torch = _torch()
    from paper_2412_17543_amd.solver import Solver
    nx = 20
    g = Solver(nx, _around(nx, edge), workload.lognormal_coef(nx ** 3, 0.5), autotune=False)
    print("[gpu] %s, %d columns: %d interface nodes" % (edge, ncols, g.info()["max_nB"]), flush=True)
    assert g.info()["max_nB"] == nB
    u = torch.tensor(workload.rhs_sequence(nx, ncols), device="cuda")
    one, gf1 = g.adjoint_grad(u, u, 1e-12)
    blk, gfb, its = g.adjoint_grad_block(u, u, 1e-12)
    assert (one - blk).abs().max().item() <= 1e-9 * one.abs().max().item()
    assert (gf1 - gfb).abs().max().item() <= 1e-9 * gf1.abs().max().item()


def test_block_product_refuses_larger_interfaces():
    torch = _torch()
    from paper_2412_17543_amd._lib import BddcError
    from paper_2412_17543_amd.solver import Solver
    nx = 20
    g = Solver(nx, _around(nx, (9, 10, 10)), np.ones(nx ** 3), autotune=False)
    assert g.info()["max_nB"] == 562
    u = torch.tensor(workload.rhs_sequence(nx, 2), device="cuda")
    with pytest.raises(BddcError) as e:
        g.adjoint_grad_block(u, u, 1e-8)
    assert e.value.code == -1 and "block product" in str(e.value)
    g.adjoint_grad(u, u, 1e-8)


@pytest.mark.parametrize("nx,cells,cons,inside", [
    (8, 2, ("corners", "faces"), True),                 # 18 coarse DOFs
    (24, "c3s", ("corners", "edges"), True),            # an odd count, uneven subdomains
    (20, 5, ("corners", "faces"), True),                # 444
    (20, 5, ("corners", "faces", "edges"), False),      # 684: by blocks of the operator, outside
])
def test_coarse_solve_on_both_sides_of_the_limit(nx, cells, cons, inside):
    """M^{-1} r against the oracle (sums of at most a few thousand products of
    size ~1, local condition numbers up to ~1e3: 1e-11 of the largest entry), as
    solved and with the kernel classes timed, and the coarse space on the side
    of the limit that the case is for."""
    torch = _torch()
    from oracle.sequence import OracleSolver
    from paper_2412_17543_amd.solver import Solver
    if cells == "c3s":
        s = workload.workload("c3s")
        part, sr, keep = s["elem_to_sub"], s["sub_to_subregion"], s["elem_keep"]
    else:
        c = (np.arange(nx) * cells) // nx
        part = (c[None, None, :] + cells * (c[None, :, None] + cells * c[:, None, None])).ravel().astype(np.int32)
        sr = keep = None
    coef = workload.lognormal_coef(nx ** 3, 0.5)
    g = Solver(nx, part, coef, sub_to_subregion=sr, elem_keep=keep, constraints=cons, autotune=False)
    print("[gpu] %d^3 %s: %d coarse DOFs" % (nx, cons, g.info()["n_coarse"]), flush=True)
    assert (g.info()["n_coarse"] <= FUSED_MAX_NC) == inside
    o = OracleSolver(nx, part, coef, elem_keep=keep, sub_to_subregion=sr, constraints=cons)
    r = np.random.default_rng(nx).standard_normal(g.n_gamma)
    zo = o.M.apply(r)
    for timed in (False, True):
        g.enable_timing(timed)
        z = g.apply_precond(torch.tensor(r, device="cuda")).cpu().numpy()
        assert np.abs(z - zo).max() <= 1e-11 * np.abs(zo).max()
