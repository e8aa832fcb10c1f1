"""Work splits of the batched products with fewer blocks than one per compute
unit: the operators against the oracle, and a tuned configuration read back
and pinned."""
import numpy as np
import pytest

import workload

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _solver(name, **kw):
    from paper_2412_17543_amd.solver import Solver
    s = workload.workload(name)
    return Solver(s["nx"], s["elem_to_sub"], s["coef"], sub_to_subregion=s["sub_to_subregion"],
                  elem_keep=s["elem_keep"], **kw)


@pytest.mark.parametrize("name", ["c16", "c3s"])                # 8 equal subdomains; uneven ones
@pytest.mark.parametrize("cfg", [(1, 2, 4, 4), (1, 4, 8, 2), (8, 3, 4, 2), (1, 1000, 8, 4)])
def test_fractions_of_the_blocks(name, cfg):
    """A p and M^{-1} r (local condition numbers up to ~1e3 on 1e-16 rounding:
    1e-11 of the largest entry)."""
    torch = _torch()
    from oracle.sequence import OracleSolver
    s = workload.workload(name)
    g = _solver(name, product_cfg=list(cfg) * 2, autotune=False)
    o = OracleSolver(s["nx"], s["elem_to_sub"], s["coef"], sub_to_subregion=s["sub_to_subregion"], elem_keep=s["elem_keep"])
    t = g.tuning()
    print("[gpu] %s %s: %d blocks" % (name, cfg, t["schur"]["blocks"]), flush=True)
    for w in ("schur", "neumann"):
        assert [t[w][k] for k in ("blocks_per_cu", "per_subdomain", "waves", "unroll")] == list(cfg)
    x = np.random.default_rng(1).standard_normal(g.n_gamma)
    for got, want in ((g.apply_schur, o.ss.apply_A), (g.apply_precond, o.M.apply)):
        y, yo = got(torch.tensor(x, device="cuda")).cpu().numpy(), want(x)
        assert np.abs(y - yo).max() <= 1e-11 * np.abs(yo).max()


@pytest.mark.parametrize("name", ["c16", "tiny3", "c3s"])
def test_tuned_configuration_is_the_pinned_one(name):
    torch = _torch()
    keys = ("blocks_per_cu", "per_subdomain", "waves", "unroll")
    a = _solver(name)
    t = a.tuning()
    b = _solver(name, product_cfg=[int(t[w][k]) for w in ("schur", "neumann") for k in keys])
    u = b.tuning()
    print("[gpu] %s: %s" % (name, t), flush=True)
    for w in ("schur", "neumann"):
        assert [t[w][k] for k in ("blocks",) + keys] == [u[w][k] for k in ("blocks",) + keys]
    x = torch.randn(a.n_gamma, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    assert torch.equal(a.apply_schur(x), b.apply_schur(x))
    assert torch.equal(a.apply_precond(x), b.apply_precond(x))
