"""GPU parity of the stencil fit, the rows S and the preconditioner.

* class stencils (Section 3.1, 3.2): the GPU's Gram eigenvectors span the
  same 3-dimensional space as the oracle's thin-SVD alpha: projector
  difference <= 1e-9 (the subspace is unique up to a 3x3 mix, so projectors
  and gauge-invariant products are compared, not vectors); the three Gram
  eigenvalues equal the oracle's squared singular values to 1e-9 relative;
* beta = B^H alpha and the rows S of Eq. (11): compared after mapping the
  GPU alpha onto the oracle's basis (alpha_gpu = alpha_oracle X);
* the preconditioner S^-1 Q v, which is invariant to the 3x3 mix, element
  by element against the oracle's sparse LU: 1e-9 relative.
"""
import numpy as np
import pytest

from oracle import sparse as osp
from oracle import stencil as ost
from paper_1804_02297_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _plan(n, m, max_rhs=1):
    from paper_1804_02297_amd.binding import Plan
    return Plan(n, I.wavenumber_for(n), _dev(m), max_rhs=max_rhs)


@pytest.mark.parametrize("n", [4, 6, 8, 13])
def test_class_stencils_match_oracle(lib, n):
    k = I.wavenumber_for(n)
    m = I.medium_bumps(n, 2)
    print(f"class fit n={n}", flush=True)
    plan = _plan(n, m)
    plan.stencil_fit()
    al, be, ev = plan.class_stencils()
    oal, obe, osg = ost.fit_all_classes(n, k)
    for kap in range(27):
        R = oal[kap].shape[0]
        ag = al[kap, :R]
        assert np.abs(ag.conj().T @ ag - np.eye(3)).max() <= 1e-10
        assert np.abs(ost.projector(ag) - ost.projector(oal[kap])).max() <= 1e-9, kap
        assert np.allclose(ev[kap], osg[kap][:3] ** 2, rtol=1e-9, atol=1e-14 * osg[kap][-1] ** 2), kap
        # beta in the oracle's basis: alpha_gpu = alpha_or X -> beta_gpu = beta_or X
        X = oal[kap].conj().T @ ag
        assert np.abs(be[kap, :R] - obe[kap] @ X).max() <= 1e-9 * np.abs(obe[kap]).max()


def test_rows_match_oracle_assembly(lib):
    n = 7
    k = I.wavenumber_for(n)
    m = I.medium_bumps(n, 4)
    plan = _plan(n, m)
    plan.stencil_fit()
    al, be, _ = plan.class_stencils()
    rows = plan.rows()
    oal, obe, _ = ost.fit_all_classes(n, k)
    # oracle assembly with the GPU's stencils: identical rows up to rounding
    gal = [al[kap, :oal[kap].shape[0]] for kap in range(27)]
    gbe = [be[kap, :oal[kap].shape[0]] for kap in range(27)]
    S, _ = osp.assemble(n, m, gal, gbe)
    from test_host_solver import csr_to_rows
    ref = csr_to_rows(S, n)
    assert np.abs(rows - ref).max() <= 1e-13 * np.abs(ref).max()


@pytest.mark.parametrize("n", [6, 10])
def test_preconditioner_matches_oracle(lib, n):
    k = I.wavenumber_for(n)
    m = I.medium_bumps(n, 5)
    plan = _plan(n, m, max_rhs=2)
    plan.stencil_fit()
    plan.factor()
    v = I.random_field(2, n, 6)
    z = plan.precond(_dev(v)).cpu().numpy()
    oal, obe, _ = ost.fit_all_classes(n, k)
    S, Q = osp.assemble(n, m, oal, obe)
    P = osp.Preconditioner(S, Q)
    ref = np.stack([P(vv) for vv in v])
    assert np.abs(z - ref).max() <= 1e-9 * np.abs(ref).max()


def test_zero_contrast_preconditioner_is_identity(lib):
    n = 8
    m = np.zeros((n, n, n), complex)
    plan = _plan(n, m)
    plan.stencil_fit()
    plan.factor()
    v = I.random_field(1, n, 2)
    z = plan.precond(_dev(v)).cpu().numpy()
    assert np.abs(z - v).max() <= 1e-10 * np.abs(v).max()


@pytest.mark.parametrize("n,nrhs", [(4, 7), (5, 1), (11, 3), (18, 16)])
def test_class_stencil_product_over_boxes(lib, n, nrhs):
    """Q v with the class stencils by the classes' boxes: extents n - 2 odd and
    even (a thread's second point missing), boxes of less than a workgroup and
    workgroups that cross right-hand sides.  Without contrast S = Q, so
    S^-1 Q v = v up to the factor's rounding."""
    plan = _plan(n, np.zeros((n, n, n), complex), max_rhs=nrhs)
    plan.stencil_fit()
    plan.factor()
    v = I.random_field(nrhs, n, 12)
    z = plan.precond(_dev(v)).cpu().numpy()
    print(f"n={n} x{nrhs} {np.abs(z - v).max() / np.abs(v).max():.2e}", flush=True)
    assert np.abs(z - v).max() <= 1e-10 * np.abs(v).max()
