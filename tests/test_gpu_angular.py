"""The angular transform Y = P Phi (Sec. 4.1) on the GPU through the C ABI,
against the FP64 oracle, and composed with the radial DSBT."""
import math

import numpy as np
import pytest
from scipy import special

from oracle import angular, dsbt as odsbt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def dev(x, dtype):
    return torch.from_numpy(np.ascontiguousarray(x).reshape(-1)).to(dtype).cuda()


# tolerances: FP32 arithmetic, or FP64.  The complex64 cases take every matrix-core
# tile count of both axis steps (16 to 64 rows; the DFT up to 128), and N_phi = 63
# in complex128 the vector kernel of the azimuthal step (2 N_phi > 64).
CASES = [(8, 9, 100, "c64", 2e-6), (16, 17, 256, "c64", 2e-6), (64, 63, 70, "c64", 2e-6), (1, 1, 64, "c64", 1e-6),
         (33, 31, 130, "c64", 2e-6), (20, 5, 64, "c64", 2e-6),
         # 64 < 2 N_phi <= 128: the DFT matrix in LDS, 5, 6, 7 and 8 row blocks
         (8, 33, 100, "c64", 2e-6), (4, 45, 70, "c64", 2e-6), (3, 53, 130, "c64", 2e-6),
         # fewer radial points than one block: every load past the last point is clamped
         (5, 3, 3, "c64", 2e-6), (33, 31, 1, "c64", 2e-6), (5, 3, 3, "c128", 1e-12), (40, 31, 1, "c128", 1e-12),
         (8, 9, 100, "c128", 1e-12), (16, 31, 130, "c128", 1e-12), (64, 63, 65, "c128", 1e-12)]


@pytest.mark.parametrize("nt,nphi,nr,precision,tol", CASES)
def test_forward_inverse_match_oracle(nt, nphi, nr, precision, tol):
    from paper_1509_07115_amd import AngularTransform
    rng = np.random.default_rng(nt * 100 + nphi)
    psi = rng.standard_normal((nt, nphi, nr)) + 1j * rng.standard_normal((nt, nphi, nr))
    Y = AngularTransform(nr, nt, nphi, precision)
    c = Y.forward(dev(psi, Y.dtype)).cpu().numpy().reshape(nphi, nt, nr)
    ref = angular.forward(psi, nt, nphi)
    assert np.linalg.norm(c - ref) <= tol * np.linalg.norm(ref)
    back = Y.inverse(dev(c, Y.dtype)).cpu().numpy().reshape(nt, nphi, nr)
    assert np.linalg.norm(back - psi) <= 2 * tol * np.linalg.norm(psi)
    refi = angular.inverse(ref, nt, nphi)
    got_i = Y.inverse(dev(ref, Y.dtype)).cpu().numpy().reshape(nt, nphi, nr)
    assert np.linalg.norm(got_i - refi) <= tol * np.linalg.norm(refi)


@pytest.mark.parametrize("nt,nphi,nr,precision,tol", [(64, 17, 4096, "c64", 2e-6), (64, 63, 1024, "c64", 2e-6),
                                                      (64, 17, 4096, "c128", 1e-12)])
def test_timed_sizes_match_oracle(nt, nphi, nr, precision, tol):
    """The sizes the angular timing runs: there each matrix-core workgroup loops
    over several point blocks with its loads prefetched (3 and 4 blocks at
    64 x 17 x 4096 in complex64, 2 for the FP64 Legendre step; 2 for the
    Legendre step at 64 x 63 x 1024), which the small cases above do not reach.
    Element by element against the oracle."""
    from paper_1509_07115_amd import AngularTransform
    rng = np.random.default_rng(nr + nphi)
    psi = rng.standard_normal((nt, nphi, nr)) + 1j * rng.standard_normal((nt, nphi, nr))
    Y = AngularTransform(nr, nt, nphi, precision)
    ref = angular.forward(psi, nt, nphi)
    c = Y.forward(dev(psi, Y.dtype)).cpu().numpy().reshape(nphi, nt, nr)
    scale = np.abs(ref).max()
    assert np.abs(c - ref).max() <= tol * scale * math.sqrt(nt)
    assert np.linalg.norm(c - ref) <= tol * np.linalg.norm(ref)
    refi = angular.inverse(ref, nt, nphi)
    got_i = Y.inverse(dev(ref, Y.dtype)).cpu().numpy().reshape(nt, nphi, nr)
    assert np.abs(got_i - refi).max() <= tol * np.abs(refi).max() * math.sqrt(nt)
    assert np.linalg.norm(got_i - refi) <= tol * np.linalg.norm(refi)


@pytest.mark.parametrize("l,m", [(0, 0), (2, -1), (5, 3), (8, -7), (8, 8)])
def test_sampled_harmonic_has_one_coefficient(l, m):
    # Y_lm (library routine) sampled with sqrt(w_j dphi), l <= N_theta - 1: the
    # transform puts all of it on channel (l, m), at every radial point
    from paper_1509_07115_amd import AngularTransform
    nt, nphi, nr = 9, 17, 3
    eta, w, phi = angular.grid(nt, nphi)
    h = special.sph_harm_y(l, m, np.arccos(eta)[:, None], phi[None, :]) * np.sqrt(w)[:, None] * math.sqrt(2 * math.pi / nphi)
    psi = h[:, :, None] * np.array([1.0, -2.0, 0.5j])[None, None, :]
    Y = AngularTransform(nr, nt, nphi, "c128")
    c = Y.forward(dev(psi, Y.dtype)).cpu().numpy().reshape(nphi, nt, nr)
    ref = np.zeros_like(c)
    ref[m + 8, l - abs(m), :] = [1.0, -2.0, 0.5j]
    np.testing.assert_allclose(c, ref, atol=1e-12)


def test_composed_with_the_radial_transform():
    # c = B Y psi (eq. BYpsi): the coefficient layout is a DSBT channel layout
    from paper_1509_07115_amd import AngularTransform, Plan
    nt, nphi, nr, rmax = 6, 9, 128, 12.8
    rng = np.random.default_rng(8)
    psi = rng.standard_normal((nt, nphi, nr)) + 1j * rng.standard_normal((nt, nphi, nr))
    Y = AngularTransform(nr, nt, nphi)
    plan = Plan(Y.channels(rmax))
    b = plan.forward(Y.forward(dev(psi, torch.complex64))).cpu().numpy().reshape(nphi, nt, nr)
    a = angular.forward(psi, nt, nphi)
    for q in range(nphi):
        for t in range(nt):
            l = abs(q - 4) + t
            ref = odsbt.forward(a[q, t], l)
            assert np.linalg.norm(b[q, t] - ref) <= 1e-5 * np.linalg.norm(ref), (q, t)
    assert Y.lm()[0] == (4, -4) and Y.lm()[4 * nt] == (0, 0)


def test_rejected_sizes_and_buffers():
    from paper_1509_07115_amd import AngularTransform, DsbtError
    for nt, nphi in ((0, 5), (65, 5), (8, 4), (8, 65)):
        with pytest.raises(DsbtError, match="UNSUPPORTED"):
            AngularTransform(16, nt, nphi)
    Y = AngularTransform(16, 4, 5)
    with pytest.raises(TypeError):
        Y.forward(torch.zeros(16 * 20, dtype=torch.complex128, device="cuda"))
    with pytest.raises(ValueError):
        Y.forward(torch.zeros(10, dtype=torch.complex64, device="cuda"))


# (N_theta, N_phi, Nr): one and two row blocks of node pairs at their edges (1, 32,
# 33, 64; odd counts have a middle node), 1 to 8 steps of element pairs (N_phi 1 to
# 63), points below, at and past the workgroup's 16, and both sides of the size
# where two launches take over (704 values, 512 points; 1280 values at most)
ONE_LAUNCH = [(1, 1, 1), (2, 1, 17), (31, 3, 15), (32, 15, 16), (33, 17, 33), (64, 1, 100), (64, 11, 5), (63, 11, 47),
              (30, 23, 19), (22, 25, 31), (15, 45, 9), (14, 47, 513), (11, 63, 21), (20, 63, 515), (64, 19, 600),
              (64, 11, 512), (64, 13, 512), (64, 13, 513), (64, 21, 520)]


@pytest.mark.parametrize("nt,nphi,nr", ONE_LAUNCH)
def test_both_steps_in_one_launch(nt, nphi, nr):
    """Against the oracle to the complex64 tolerance of the cases above, into a new
    buffer, in place, and into a buffer shifted by one element over the input (which
    goes through the work buffer in two launches)."""
    from paper_1509_07115_amd import AngularTransform
    rng = np.random.default_rng(nt * 100 + nphi)
    psi = rng.standard_normal((nt, nphi, nr)) + 1j * rng.standard_normal((nt, nphi, nr))
    Y = AngularTransform(nr, nt, nphi)
    ref = angular.forward(psi, nt, nphi)
    for call, x, want in ((Y.forward, psi, ref), (Y.inverse, ref, angular.inverse(ref, nt, nphi))):
        want = np.asarray(want).reshape(-1)
        n = want.size
        room = torch.zeros(n + 1, dtype=Y.dtype, device="cuda")
        for off in (None, 0, 1):
            room[:n] = dev(x, Y.dtype)
            out = torch.full_like(room[:n], float("nan")) if off is None else room[off:off + n]
            call(room[:n], out=out)
            got = out.cpu().numpy()
            assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want), (call.__name__, off)


@pytest.mark.parametrize("nt,nphi,nr", [(64, 17, 20), (33, 11, 16), (64, 1, 40), (9, 1, 3), (20, 63, 530)])
def test_one_launch_takes_values_up_to_the_largest(nt, nphi, nr):
    """A power of two times the data is the same power of two times the result (to one
    rounding, and to terms below the normal range of the unscaled result), up to the
    largest finite values: the symmetric and antisymmetric sums of element and node pairs
    must not overflow where the result does not.  Two values of nearly 2^128 per point:
    an azimuth pair (+k, -k), a node pair (j, -j), equal and opposite."""
    from paper_1509_07115_amd import AngularTransform
    Y = AngularTransform(nr, nt, nphi)
    rng = np.random.default_rng(nt + nphi)
    grid, coef = np.zeros((nt, nphi, nr), np.complex64), np.zeros((nphi, nt, nr), np.complex64)
    for i in range(nr):
        j, k, q, t = (int(rng.integers(n)) for n in (nt, nphi, nphi, nt))
        v = np.complex64(complex(*rng.uniform(1.7, 1.99, 2)))
        s = (1, -1)[i // 2 % 2]
        grid[j, k, i] = v
        grid[(j, (nphi - k) % nphi, i) if i % 2 else (nt - 1 - j, k, i)] += s * v * (i % 2 == 0 or k > 0)
        grid[j, k, i] = v
        coef[q, t, i] = v
        coef[nphi - 1 - q, t, i] = s * v
    two = 2.0 ** 127
    for call, x in ((Y.forward, grid), (Y.inverse, coef)):
        small = torch.from_numpy(x.reshape(-1)).cuda()
        large = torch.view_as_complex(torch.view_as_real(small) * two)
        assert torch.isfinite(torch.view_as_real(large)).all()
        want = torch.view_as_real(call(small)) * two
        got = torch.view_as_real(call(large))
        ok = torch.isfinite(want)                    # (a result of 2 or more overflows in earnest)
        assert ok.float().mean() > 0.9
        assert torch.allclose(got[ok], want[ok], rtol=2.0 ** -23, atol=two * 2.0 ** -120), call.__name__


def _us_per_call(f, n=20):
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(n):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / n)
    return best


@pytest.mark.parametrize("nt,nphi,nr", [(1, 1, 1 << 19), (4, 1, 1 << 18)])
def test_many_points_of_a_small_angular_grid_are_not_held_up(nt, nphi, nr):
    """A transform reads and writes its data once or twice: four copies' time and the two
    launches are ample (one workgroup per 16 points takes twice that)."""
    from paper_1509_07115_amd import AngularTransform
    Y = AngularTransform(nr, nt, nphi)
    x = torch.randn(Y.size, 2, device="cuda").view(-1, 2)
    x = torch.view_as_complex(x)
    out = torch.empty_like(x)
    copy = _us_per_call(lambda: out.copy_(x))
    for call in (Y.forward, Y.inverse):
        t = _us_per_call(lambda: call(x, out=out))
        print(f"{nt} x {nphi} x {nr} {call.__name__}: {t:.1f} us, copy {copy:.1f}")
        assert t <= 4 * copy + 12


# both sides of the line between one launch and two for many points
@pytest.mark.parametrize("nt,nphi,nr", [(3, 1, 16384), (3, 1, 16385), (17, 7, 16401), (18, 7, 16401), (24, 5, 16390),
                                        (8, 15, 16400), (40, 1, 20001),
                                        (16, 1, 20480), (16, 1, 20481), (23, 5, 20483), (24, 5, 20483), (40, 3, 20481),
                                        (15, 1, 32768), (15, 1, 32769), (5, 3, 32771),
                                        (33, 5, 65536), (33, 5, 65537)])
def test_many_points(nt, nphi, nr):
    from paper_1509_07115_amd import AngularTransform
    rng = np.random.default_rng(nr + nt)
    psi = rng.standard_normal((nt, nphi, nr)) + 1j * rng.standard_normal((nt, nphi, nr))
    Y = AngularTransform(nr, nt, nphi)
    for call, ref in ((Y.forward, angular.forward(psi, nt, nphi)),
                      (Y.inverse, angular.inverse(psi.reshape(nphi, nt, nr), nt, nphi))):
        want = np.asarray(ref).reshape(-1)
        got = call(dev(psi, Y.dtype)).cpu().numpy()
        assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want), call.__name__
