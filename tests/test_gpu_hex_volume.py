"""The hexahedral volume kernels with a partly filled last workgroup (27
elements; groups of 7, 6, 5, 4 and 2, and of one element) and LDS filled with
NaN before each kernel group, against the oracle in extended precision: affine
with flux anti-aliasing, with surface-flux anti-aliasing as well, and curved.
Tolerances: FP64 1e-12; FP32 2e-5, curved (unsplit energy flux) 1e-4."""

import numpy as np
import pytest

import paper_2401_06132_amd as frmi
from oracle.mesh import Mesh
from oracle.rhs import Params, rhs as oracle_rhs
from paper_2401_06132_amd import inputs
from test_gpu_lds_nan import _staged_rhs_after_nan_fills

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,saa", [("hex", False), ("hex", True), ("hex_warp", False)])
@pytest.mark.parametrize("p", [1, 2, 3, 4])
def test_partial_last_group(p, kind, saa, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("hex volume case", p, kind, "saa" if saa else "", prec, flush=True)
    dims = (3, 3, 3)
    m = Mesh(*dims, p, kind, surf_aa=saa)
    U = inputs.element_state([m.upts_coords(t) for t in m.types], seed=19)
    ref = oracle_rhs(m, {t: u.astype(np.longdouble) for t, u in zip(m.types, U)}, Params(pref=inputs.P0),
                     dtype=np.longdouble)
    s = frmi.Solver(dims, p, kind, prec=prec, pref=inputs.P0, rho_ref=inputs.RHO0, surface_aa=saa)
    du = _staged_rhs_after_nan_fills(s, np.concatenate([x.reshape(-1) for x in U]))
    assert np.all(np.isfinite(du))
    err = np.max([(np.abs(g - ref[t]).max(axis=(0, 2)) / np.abs(ref[t]).max(axis=(0, 2))).astype(np.float64)
                  for g, t in zip(s.split(du), m.types)], axis=0)
    print("rel err per variable", err, flush=True)
    assert np.all(err < (1e-12 if prec == "fp64" else (1e-4 if kind == "hex_warp" else 2e-5))), err
