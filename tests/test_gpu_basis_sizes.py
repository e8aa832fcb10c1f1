"""Deflation-basis sizes on both sides of the register buckets of the vector
and recycling kernels, against the oracle (as the other float64 parity tests:
rtol 1e-10, iterations within +-1, solutions to 1e-9)."""
import numpy as np
import pytest

import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 8, 9, 24, 25, 40, 41, 64])
def test_basis_size(R):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.sequence import OracleSolver
    from paper_2412_17543_amd.solver import Solver
    s = workload.workload("tiny3")
    print("[gpu] tiny3 R %d" % R, flush=True)
    kw = dict(sub_to_subregion=s["sub_to_subregion"], R=R, reorth=R in (9, 41))
    g = Solver(16, s["elem_to_sub"], s["coef"], autotune=False, **kw)
    o = OracleSolver(16, s["elem_to_sub"], s["coef"], **kw)
    F = workload.rhs_sequence(16, 6)
    U, its, rr = g.solve_sequence(torch.tensor(F, device="cuda"), 1e-10)
    uo, ito, _ = o.solve_sequence(F, 1e-10)
    assert np.all(np.abs(its - ito) <= 1), (its, ito)
    assert np.all(rr < 1e-10)
    assert g.info()["deflation_cols"] == o.rec.basis(o.ss.n_gamma).shape[1]
    for k in range(len(F)):
        assert np.abs(U[k].cpu().numpy() - uo[k]).max() <= 1e-9 * np.abs(uo[k]).max()
