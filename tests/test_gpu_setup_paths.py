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
