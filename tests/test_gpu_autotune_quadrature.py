"""Tuned 16-column task sets of a matrix whose close entries come from a quadrature: low-precision cycles
apply the FP32 copy of the stored tiles, so the tuner has to time that form."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_tuned_block_solve(precision):
    from paper_2501_17656_amd import H2Matrix, bem_panels, bem_quadrature7
    V, T = synth.bumpy_torus_mesh(40, 20)
    Vd, Td = torch.from_numpy(V).cuda(), torch.from_numpy(T.astype(np.int64)).cuda()
    y, s, d = bem_panels(Vd, Td)
    g = H2Matrix(y, "laplace", 1.0, 0.0, 64, 0.7, 3, scale=s, diag=d)
    g.set_near_quadrature(*bem_quadrature7(Vd, Td))
    B = torch.from_numpy(synth.normal_vector(len(T), 5, nrhs=16)).cuda()
    kw = {"rtol": 1e-8, "precision": precision, "smoother": "bj"}
    X, info = g.solve_multi(B, **kw)
    g.set_autotune(True)
    Xt, tuned = g.solve_multi(B, **kw)
    assert set(g.block_tuning()) >= {"near", "fine"}
    # another order of the sums; both solve to 1e-8
    assert tuned["converged"] and abs(tuned["cycles"] - info["cycles"]) <= 1
    for k in range(16):
        assert float((g.matvec(Xt[:, k].contiguous()) - B[:, k]).norm()) < 1e-8 * float(B[:, k].norm())
    g.close()
