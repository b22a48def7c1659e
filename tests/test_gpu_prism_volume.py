"""The prism volume kernels (single precision: matrix cores, one column per
lane; double precision: operator rows in scalar registers) where their tiles
can go wrong: element counts one off a workgroup's, a single workgroup half
filled, every order's row remainders, affine and curved, against the oracle in
extended precision.  Tolerances: the FP32 floor of the precision split, 2e-5
per variable (curved elements, which keep the unsplit energy flux, 1e-4);
FP64 1e-12."""

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

# prisms: two per cell; workgroups of 8, 7, 4 and 5 elements at p = 1..4 (FP64: 8, 5, 3, 2)
CASES = [(d, p, k) for p in (1, 2, 3, 4) for k in ("prism", "prism_warp")
         for d in ((2, 1, 1), (3, 1, 1), (1, 5, 1), (2, 2, 3)) if not (k == "prism_warp" and min(d[0], d[2]) < 2)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("dims,p,kind", CASES)
def test_volume_tile_edges(dims, p, kind, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("volume case", dims, p, kind, prec, flush=True)
    m = Mesh(*dims, p, kind)
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=11)
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
    assert np.all(err < (1e-12 if prec == "fp64" else (1e-4 if "warp" in kind else 2e-5))), err


# prisms per workgroup of the volume kernel, by precision and order
GROUP = {"fp32": {1: 8, 2: 7, 3: 4, 4: 5}, "fp64": {1: 8, 2: 5, 3: 3, 4: 2}}


def _check(m, U, s, tol):
    """The staged right-hand side, LDS filled with NaN before each kernel group, against the oracle."""
    ref = oracle_rhs(m, {t: u.astype(np.longdouble) for t, u in zip(m.types, U)}, Params(pref=inputs.P0),
                     dtype=np.longdouble)
    du = _staged_rhs_after_nan_fills(s, np.concatenate([x.reshape(-1) for x in U]))
    assert np.all(np.isfinite(du))
    err = np.max([(np.abs(g - ref[t]).max(axis=(0, 2)) / np.abs(ref[t]).max(axis=(0, 2))).astype(np.float64)
                  for g, t in zip(s.split(du), m.types)], axis=0)
    print("rel err per variable", err, flush=True)
    assert np.all(err < tol), err


@pytest.mark.parametrize("prec,p,dims", [("fp32", p, (3, 3, 3)) for p in (1, 2, 3, 4)] +
                         [("fp64", 1, (3, 3, 3)), ("fp64", 2, (3, 3, 3)), ("fp64", 3, (2, 2, 2))])
def test_curved_partial_last_group(prec, p, dims):
    """Curved prisms whose last workgroup is partly filled (box meshes hold an even number of prisms, so groups of
    two, FP64 p = 4, are always whole there).  At least two cells per axis: where a curved element pairs with
    itself, the rounding of two equal centroid coordinates decides which side is L."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("curved case", dims, p, prec, flush=True)
    m = Mesh(*dims, p, "prism_warp")
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=12)
    assert len(U[0]) % GROUP[prec][p] != 0
    s = frmi.Solver(dims, p, "prism_warp", prec=prec, pref=inputs.P0, rho_ref=inputs.RHO0)
    _check(m, U, s, 1e-12 if prec == "fp64" else 1e-4)


def odd_prisms(dims):
    """Vertices and lattice of a prism box with the first prism cut from its centre into a pyramid on each
    quadrilateral and a tetrahedron on each triangle: an odd number of prisms."""
    verts, lat, _ = sheared_case(dims, 1, "prism", A=np.eye(3))
    x, rest = verts["prism"][0], verts["prism"][1:]
    c = x.mean(axis=0)
    tet = [[x[a], x[b], x[d], c] for a, b, d in ((0, 2, 1), (3, 4, 5))]
    pyr = [[x[a], x[b], x[a + 3], x[b + 3], c] for a, b in ((0, 1), (1, 2), (2, 0))]

    def positive(e, flip):
        e = np.array(e)
        return e if np.linalg.det(np.stack([e[1] - e[0], e[2] - e[0], e[-1] - e[0]])) > 0 else e[flip]

    return {"prism": rest, "tet": np.array([positive(e, [0, 2, 1, 3]) for e in tet]),
            "pyr": np.array([positive(e, [0, 2, 1, 3, 4]) for e in pyr])}, lat


@pytest.mark.parametrize("dims", [(2, 2, 2), (2, 3, 2)])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_odd_prism_count(p, dims):
    """FP64 with 15 and 23 prisms: a half-filled last group of two at p = 4."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("odd prism case", dims, p, flush=True)
    verts, lat = odd_prisms(dims)
    m = elements_mesh(p, verts, lat)
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=13)
    assert len(verts["prism"]) == 2 * np.prod(dims) - 1
    s = frmi.Solver(None, p, "elements", verts=verts, period=lat, pref=inputs.P0, rho_ref=inputs.RHO0)
    assert s.n_prism % GROUP["fp64"][4] == 1
    _check(m, U, s, 1e-12)
