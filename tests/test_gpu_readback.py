"""State and fluence readback: the doubles handed out are the device's own
values, exactly (FP64 copied straight into the caller's buffer, FP32 widened)."""
import numpy as np
import pytest

import rte_inputs as ri

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,N", [(16, 0), (16, 2), (48, 1)])
def test_readback_is_exact(n, N, prec):
    from paper_1801_06364_amd.rte import Solver
    M = (N + 1) ** 2
    psi0 = np.random.default_rng(n + N).standard_normal((M, n, n, n))
    s = Solver(n, N, 0.5, 0.3, 0.0, *ri.homogeneous_maps(n, 0.1, 2.0, 0.8), psi0=psi0, W=0, precision=prec)
    state, phi = s.get_state(), s.fluence()
    s.close()
    held = psi0.astype(np.float32).astype(np.float64) if prec == "f32" else psi0
    assert np.array_equal(state, held)
    assert np.array_equal(phi, held[0])
