"""The plane passes against the oracle where their work is split unevenly: two
planes per workgroup (16^3, 48^3) with an odd number of moments, so that a
workgroup holds planes of two z (P_2: nine moments) or one moment only (P_0:
both planes carry fluence sums), rows of one wavefront in two planes (48^3),
three column stages (96^3; 32^3 FP64), and every grid's standalone forward pass
(first step) and fused one (later steps). Layer, source on some planes only,
RK4: state, integrated fluence (FP64 sums of the last stage) and the per-step
fluence change (partial sums per z-plane).

Tolerances: the bars of the parity tests, relative L2 1e-12 (FP64) and 1e-5
(FP32); the fluence change is a ratio of two sums of n^3 terms, each with the
relative error of the state's change, 1e-9 and 1e-3.
"""
import numpy as np
import pytest

from oracle import pn

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "f64": 1e-12}
CASES = [(16, 0), (16, 2), (32, 1), (48, 0), (48, 2), (64, 1), (96, 1)]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,N", CASES)
def test_planes_against_oracle(n, N, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1801_06364_amd.rte import Solver
    print(f"\n[planes] n={n} N={N} {prec}", flush=True)
    M, W, steps, dx, c, dt = (N + 1) ** 2, n // 8, 3, 0.25, 0.3, 0.16
    rng = np.random.default_rng(7 * n + N)
    mu_a, mu_s, g = rng.uniform(0.01, 0.1, (n,) * 3), rng.uniform(1, 9, (n,) * 3), rng.uniform(0.5, 0.9, (n,) * 3)
    psi0 = rng.uniform(0.5, 1.5, (M, n, n, n))
    q = np.zeros((M, n, n, n))
    q[:, n // 2, W:n - W, W:n - W] = rng.uniform(0, 1, (M, n - 2 * W, n - 2 * W))
    q[:, n // 2 + 3] = q[:, n // 2]
    ref = pn.solve(n, N, dx, c, dt, mu_a, mu_s, g, psi0, q, W, 0.01, 1.0, steps)
    s = Solver(n, N, dx, c, dt, mu_a, mu_s, g, psi0=psi0, q=q, W=W, precision=prec, record_steps=steps,
               stream=torch.cuda.Stream())
    s.step(steps)

    def rel(a, b):
        return np.linalg.norm(a - b) / np.linalg.norm(b)

    assert rel(s.get_state(), ref["state"]) <= TOL[prec]
    assert rel(s.fluence(1), ref["phi_int"]) <= TOL[prec]
    res = s.residuals()
    s.close()
    assert np.allclose(res, ref["residual"], rtol=1e-9 if prec == "f64" else 1e-3, atol=0.0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,N", [(16, 0), (16, 3), (48, 2), (64, 5)])
def test_growth_threshold_of_a_device_state(n, N, prec):
    """The runaway-growth threshold of a state set from device memory (block
    sums, then one block; fewer vectors than threads at 16^3) equals that of
    the same state set from the host: sums of at most 64 n^3 positive FP64
    terms in two orders, so within (64 n^3) 2^-53 < 2e-9 of each other. The
    snapshot carries it after the 32 bytes magic, hash, step, flags."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import struct

    from paper_1801_06364_amd.rte import Solver
    print(f"\n[growth] n={n} N={N} {prec}", flush=True)
    M = (N + 1) ** 2
    psi = np.random.default_rng(n + N).standard_normal((M, n, n, n)).astype(np.float32).astype(np.float64)
    flat = np.full((n, n, n), 0.5)
    s = Solver(n, N, 0.25, 0.3, 0.0, flat, flat, flat, precision=prec, stream=torch.cuda.Stream())
    limits = []
    s.set_state(psi)
    limits.append(struct.unpack_from("d", s.snapshot(), 32)[0])
    dev = torch.from_numpy(psi.ravel()).cuda()
    torch.cuda.synchronize()   # the solver runs on a stream of its own
    s.set_state_device(dev)
    limits.append(struct.unpack_from("d", s.snapshot(), 32)[0])
    s.close()
    w = np.repeat(2 * np.arange(N + 1) + 1, 2 * np.arange(N + 1) + 1)
    assert abs(limits[0] / (1e16 * (w * (psi ** 2).reshape(M, -1).sum(1)).sum()) - 1) <= 2e-9
    assert abs(limits[1] / limits[0] - 1) <= 2e-9
