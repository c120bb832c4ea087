"""Compulsory-byte model of the passes that the bench's roofline lines divide by
measured times, for the schedules that run (no GPU needed)."""
import bench


def test_bytes_of_the_128_p7_step_with_the_streaming_pass():
    # four stages of one sweep over the spectrum (2F) and one fused plane pass
    n, N, M, s = 128, 7, 64, 4
    F = M * n ** 3 * s
    assert bench.algorithmic_bytes("stream", n, M, N, s) == 2 * F
    step = 4 * (bench.algorithmic_bytes("stream", n, M, N, s) + bench.algorithmic_bytes("inv_plane", n, M, N, s))
    assert abs(step - (27 * F + 32 * n ** 3 * 4 + 16 * n ** 3)) < 1
    assert abs(step / 1e9 - 14.80) < 0.01


def test_bytes_of_an_arnoldi_step_of_the_propagator():
    # 128^3 P_5, 20 steps per application, restart 30. One application: copy,
    # forward pass and difference 7F; a step's four stages 7F + maps each, less
    # one F. Orthogonalisation of cycle position j: two passes of j + 2 and j + 3
    # vectors, norm and scaling 3F.
    n, N, M, s, m, K = 128, 5, 36, 4, 30, 20
    F, maps = M * n ** 3 * s, (N + 1) * n ** 3 * s
    app = 7 * F + K * (27 * F + 4 * maps)
    gs = sum(2 * (2 * j + 5) + 3 for j in range(m)) / m * F
    got = bench.gmres_iteration_bytes(n, M, N, s, m, K)
    assert abs(got - (app + gs)) < 1
    assert abs(got / 1e9 - 190.7) < 0.05


def test_bytes_of_an_arnoldi_step_of_the_operator():
    # S + Sigma: forward pass 2F, streaming pass 2F, inverse pass 3F + maps
    n, N, M, s, m = 64, 3, 16, 8, 10
    F, maps = M * n ** 3 * s, (N + 1) * n ** 3 * s
    gs = sum(2 * (2 * j + 5) + 3 for j in range(m)) / m * F
    assert abs(bench.gmres_iteration_bytes(n, M, N, s, m, 0) - (7 * F + maps + gs)) < 1
