"""The first kernel group of tetrahedra and pyramids (double-precision matrix
cores) at its tiles' edges: less than one workgroup of eight elements, a
remainder, several workgroups; every order's remainders of 16 rows and four
k-steps; against the oracle in extended precision.  Tolerances: FP64 1e-12, the
FP32 floor of the precision split 2e-5."""

import numpy as np
import pytest

import paper_2401_06132_amd as frmi
from oracle.mesh import Mesh, elements_mesh
from oracle.rhs import Params, rhs as oracle_rhs
from paper_2401_06132_amd import inputs
from test_gpu_lds_nan import _staged_rhs_after_nan_fills
from test_mesh_elements import sheared_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["tet", "pyr"])
@pytest.mark.parametrize("dims,p", [(d, p) for p in (1, 2, 3, 4) for d in ((1, 1, 1), (1, 2, 2))])
def test_tile_edges(dims, p, kind, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("disu case", dims, p, kind, prec, flush=True)
    m = Mesh(*dims, p, kind)
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=17)
    ref = oracle_rhs(m, {t: u.astype(np.longdouble) for t, u in zip(m.types, U)}, Params(pref=inputs.P0),
                     dtype=np.longdouble)
    s = frmi.Solver(dims, p, kind, prec=prec, pref=inputs.P0, rho_ref=inputs.RHO0)
    u = torch.from_numpy(np.concatenate([x.reshape(-1) for x in U])).cuda()
    du = torch.empty_like(u)
    frmi.fill_lds(float("nan"))
    s.rhs(u, du)
    torch.cuda.synchronize()
    err = np.max([(np.abs(g - ref[t]).max(axis=(0, 2)) / np.abs(ref[t]).max(axis=(0, 2))).astype(np.float64)
                  for g, t in zip(s.split(du.cpu().numpy()), m.types)], axis=0)
    print("rel err per variable", err, flush=True)
    assert np.all(err < (1e-12 if prec == "fp64" else 2e-5)), err


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["tet", "pyr"])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_partial_last_group(p, kind, prec):
    """18 elements: two whole workgroups of eight and one with two elements, LDS filled with NaN before each
    kernel group."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("partial group case", p, kind, prec, flush=True)
    # three cubic cells in a row
    verts, lat, _ = sheared_case((1, 1, 3), p, kind, A=np.diag([1.0, 1.0, 3.0]))
    m = elements_mesh(p, verts, lat)
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=18)
    assert len(U[0]) == 18
    ref = oracle_rhs(m, {t: u.astype(np.longdouble) for t, u in zip(m.types, U)}, Params(pref=inputs.P0),
                     dtype=np.longdouble)
    s = frmi.Solver(None, p, "elements", verts=verts, period=lat, prec=prec, pref=inputs.P0, rho_ref=inputs.RHO0)
    du = _staged_rhs_after_nan_fills(s, np.concatenate([x.reshape(-1) for x in U]))
    assert np.all(np.isfinite(du))
    err = np.max([(np.abs(g - ref[t]).max(axis=(0, 2)) / np.abs(ref[t]).max(axis=(0, 2))).astype(np.float64)
                  for g, t in zip(s.split(du), m.types)], axis=0)
    print("rel err per variable", err, flush=True)
    assert np.all(err < (1e-12 if prec == "fp64" else 2e-5)), err


@pytest.mark.parametrize("node", [0, -1])
@pytest.mark.parametrize("kind,p", [("tet", 2), ("tet", 4), ("pyr", 1), ("pyr", 2), ("pyr", 3), ("pyr", 4)])
def test_infinity_reaches_the_face_values(kind, p, node):
    """FP64, point counts that are no multiple of the k-steps' four: an infinite energy makes the element's face
    values infinite, and so the wave speed and every residual of the element not finite, whichever node holds it.
    The zero padding of the operator must not turn it into a NaN (which a maximum drops)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("infinity case", kind, p, node, flush=True)
    s = frmi.Solver(3, p, kind, pref=inputs.P0, rho_ref=inputs.RHO0)
    U = inputs.element_state(s.upts_coords(), seed=21)
    E = len(U[0])
    U[0][E // 2, 4, node] = np.inf
    u = torch.from_numpy(U[0].reshape(-1)).cuda()
    du = torch.empty_like(u)
    s.rhs(u, du)
    torch.cuda.synchronize()
    assert not np.isfinite(s.split(du.cpu().numpy())[0][E // 2]).any()
