"""Reverse sweep after a run that left the finite numbers: the recomputed states
behind the step that raises the stop flag hold that step's state, as the run
itself does, whatever the workspace held before. (One segment: its states are the
workspace section behind the checkpoint.) Both forms of the last stage's pass
(plane grids, row passes of 256^3) and both schemes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["rk4", "euler"])
@pytest.mark.parametrize("n,N", [(16, 1), (48, 0), (256, 0)])
def test_recomputed_states_behind_a_stop_are_held(n, N, scheme):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1801_06364_amd.rte import RTE_EUNSTABLE, RteError, Solver
    print(f"\n[stopped] n={n} N={N} {scheme}", flush=True)
    M, steps = (N + 1) ** 2, 14
    mu_a = np.full((n, n, n), 10.0)   # mu_a c dt = 6000: a factor 6000 (Euler) or 5e13 (RK4) a step
    s = Solver(n, N, 0.25, 0.3, 2000.0, mu_a, mu_a, 0 * mu_a, psi0=np.ones((1, n, n, n)), precision="f32",
               det_index=[0], record_steps=steps, scheme=scheme, stream=torch.cuda.Stream())
    with pytest.raises(RteError) as e:
        s.forward_checkpointed(steps, steps)
    assert e.value.code == RTE_EUNSTABLE
    F = M * n ** 3 * 4
    seg = s.adj_ws[(F + 255) // 256 * 256:][:steps * F].view(torch.float32)
    with torch.cuda.stream(s.stream):
        seg.fill_(7.0)
    s.adjoint(np.ones((steps, 1)))
    u = seg.view(torch.int32).view(steps, -1).cpu()
    bad = [k for k in range(steps) if not np.isfinite(u[k].numpy().view(np.float32)).all()]
    s.close()
    assert bad and 0 < bad[0] < steps - 2
    for k in range(bad[0] + 1, steps):
        assert torch.equal(u[k], u[bad[0]]), k
