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
from oracle.mesh import Mesh
from oracle.rhs import Params, rhs as oracle_rhs
from paper_2401_06132_amd import inputs

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
