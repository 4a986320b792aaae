"""The shared-code EM step at the edges of its kernels' tiles: 16, 32 and 64 padded centres, sub-spaces around a multiple
of 16 (and odd), points around the 8 of a workgroup's round, around 8 x 256 workgroups, and more than 32 a workgroup.
Oracle: oracle.em_step_shared (fp64)."""
import numpy as np
import pytest

from test_gpu_em import em_shared, shared_calibration  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# The right-hand sides are fp32 sums of up to 36 points per wavefront, 8 wavefronts and 256 partial sums: 300 roundings of
# 2^-24, 1.8e-5, if all went one way (observed: 7e-7).  Operands of 16 bits would show 2^-9.
TOL_PHI = 2e-5


@pytest.mark.parametrize("J,Nc,N", [(1, 1, 40), (2, 16, 1031), (15, 17, 2048), (17, 32, 2049), (33, 33, 777), (64, 48, 2305), (5, 64, 4099),
                                    (3, 12, 8193), (16, 8, 8449), (64, 5, 9)])
def test_tile_edges_match_oracle(em_shared, oracle, J, Nc, N):  # noqa: F811
    data, start = shared_calibration(J, N, Nc, seed=J * 1000 + Nc)
    T = 0.3 * np.sqrt(J)
    print(f"case group={J} Nc={Nc} N={N} T={T:.2f}", flush=True)
    got = em_shared(data, start, T)
    ref, _ = oracle.em_step_shared(data, start, temperature=T)
    worst = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  max relative deviation of phi: {worst:.3e}", flush=True)
    assert worst <= TOL_PHI


def test_a_point_on_a_centre(em_shared, oracle):  # noqa: F811
    """Squared distances that come out negative by rounding count as zero."""
    data, start = shared_calibration(8, 600, 9, seed=5, noise=0.0)
    hidden = (start[..., 0] + 1j * start[..., 1]).astype(np.complex64)
    for i in range(100):
        c = hidden[:, i % 9] + 1j * hidden[:, (i * 5) % 9]
        data[i, :, 0], data[i, :, 1] = c.real, c.imag
    got = em_shared(data, start, 0.5)
    ref, _ = oracle.em_step_shared(data, start, temperature=0.5)
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= TOL_PHI * np.abs(ref).max()


@pytest.mark.parametrize("T", [1e-40, 1e-37, 1e-20, 1e-10, 1e-9, 1e6, 1e30, float("inf")])
@pytest.mark.parametrize("J,Nc,N", [(8, 12, 3000), (5, 16, 1500), (8, 33, 9000)])
def test_temperatures_from_hard_to_uniform_assignment(em_shared, oracle, J, Nc, N, T):  # noqa: F811
    """Every temperature above zero: as T -> 0 a point belongs to its nearest centre, as T -> infinity to all alike.

    Points whose two nearest centres differ by less than 1e-3 are left out (fp32 distances would decide them), so that for
    the small temperatures both sides assign every point to the same centre and N_ab is a sum of whole numbers."""
    data, start = shared_calibration(J, N, Nc, seed=J * 77 + Nc)
    z = start[..., 0].astype(np.complex128) + 1j * start[..., 1]
    cen = (z[:, :, None] + 1j * z[:, None, :]).reshape(J, -1)                      # [J][Nc^2]
    k = data[..., 0].astype(np.complex128) + 1j * data[..., 1]                     # [N][J]
    d2 = (np.abs(k) ** 2).sum(1)[:, None] + (np.abs(cen) ** 2).sum(0) - 2 * (k @ cen.conj()).real
    near = np.sqrt(np.sort(d2, axis=1)[:, :2])
    data = data[near[:, 1] - near[:, 0] > 1e-3]
    print(f"case group={J} Nc={Nc} N={len(data)} T={T:g}", flush=True)
    got = em_shared(data, start, T)
    ref, _ = oracle.em_step_shared(data, start, temperature=None if T < 1e-8 else T)
    assert np.isfinite(got).all()
    worst = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  max relative deviation of phi: {worst:.3e}", flush=True)
    assert worst <= TOL_PHI
