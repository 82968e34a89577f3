"""The eight-wave moment pipeline (tiles of 64) at the edges of its range, and
the potential tables shared between channels, against the dense oracle."""
import numpy as np
import pytest

from oracle import dsbt as odsbt
from oracle import tdse as otdse

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


# as for the other moment kernels: complex64 transforms to the stated small-N
# bound, complex64 data with FP64 arithmetic to two FP32 roundings, FP64 to 1e-12
TOL = {"c64": 2e-6, "c64x": 2.5e-7, "c128": 1e-12}


def _dtype(precision):
    return torch.complex128 if precision == "c128" else torch.complex64


def _channels(N, counts, gap=0):
    out, off = [], gap
    for ell, n in counts:
        for _ in range(n):
            out.append((N, ell, 0.1 * N, off))
            off += N + gap
    return out, off


def _check(chans, total, precision, tile=0):
    from paper_1509_07115_amd import Plan
    rng = np.random.default_rng(len(chans) + chans[0][0])
    x = rng.standard_normal(total) + 1j * rng.standard_normal(total)
    plan = Plan(chans, precision=precision, tile=tile)
    xd = torch.from_numpy(x).to(_dtype(precision)).cuda()
    b, y = plan.forward(xd).cpu().numpy(), plan.inverse(xd).cpu().numpy()
    x = xd.cpu().numpy().astype(np.complex128)
    for N, ell, _, off in chans:
        s = slice(off, off + N)
        for got, ref in ((b[s], odsbt.forward(x[s], ell)), (y[s], odsbt.inverse(x[s], ell))):
            assert np.linalg.norm(got - ref) <= TOL[precision] * np.linalg.norm(ref), (N, ell, off)


@pytest.mark.parametrize("precision", ["c64", "c64x", "c128"])
@pytest.mark.parametrize("N", [64, 128, 192 + 64, 512])
def test_tiles_of_64_at_the_edges_of_k(N, precision):
    # k = ceil(l/2) at 0, 1 and around each multiple of 16 up to 64; 1, 8 and 9
    # channels per l; odd gaps between the channels (8-byte aligned complex64 rows)
    counts = [(ell, n) for ell, n in ((0, 1), (1, 8), (2, 1), (31, 9), (32, 1), (33, 8), (63, 1), (64, 9), (65, 1),
                                      (95, 1), (96, 8), (97, 1), (126, 1), (127, 9)) if ell <= 2 * N - 2]
    _check(*_channels(N, counts, gap=3), precision, tile=64)


def test_two_column_blocks_per_item():
    # more items than compute units and l above 62: FP32 items of 16 channels
    N = 64
    counts = [(ell, 97) for ell in range(33, 60)] + [(100, 25), (126, 1)]
    chans, total = _channels(N, counts)
    _check(chans, total, "c64")


@pytest.mark.parametrize("precision", ["c64", "c128"])
def test_potential_tables_shared_between_equal_channels(precision):
    from paper_1509_07115_amd import Plan
    N, dt = 128, 0.02
    chans, total = _channels(N, [(2, 3), (5, 4), (70, 2)], gap=1)
    rng = np.random.default_rng(3)
    x = rng.standard_normal(total) + 1j * rng.standard_normal(total)
    plan = Plan(chans, precision=precision)
    shapes = rng.standard_normal((len(chans), N))
    # few distinct potentials, then one per channel (more table space), then all equal
    for pick in ([0, 0, 1, 1, 0, 2, 0, 1, 2], list(range(9)), [4] * 9):
        V = np.zeros(total)
        for (_, _, _, off), j in zip(chans, pick):
            V[off:off + N] = shapes[j]
        plan.set_potential(V, dt)
        xd = torch.from_numpy(x).to(_dtype(precision)).cuda()
        got = plan.kinetic_step(xd.clone(), 2).cpu().numpy()
        x0 = xd.cpu().numpy().astype(np.complex128)
        for (_, ell, rmax, off), j in zip(chans, pick):
            s = slice(off, off + N)
            E = otdse.kinetic_energies(N, rmax, ell)
            ref = otdse.propagate(x0[s], ell, shapes[j], E, dt, np.ones(2))
            # two steps of two transforms each, and their phase products
            tol = 2 * (2 * TOL[precision] + 4e-7 * (precision == "c64"))
            assert np.linalg.norm(got[s] - ref) <= tol * np.linalg.norm(ref), (ell, off, pick)


@pytest.mark.parametrize("precision", ["c64", "c64x", "c128"])
@pytest.mark.parametrize("sizes", [(16,), (32,), (64,), (128,), (256,), (512,), (1024,), (2048,), (4096,),
                                   (4096, 16, 2048, 32, 1024, 64, 512, 128, 256)])
def test_sine_cosine_stage_of_every_size(sizes, precision):
    # l = 0 and 1 (the two reorderings): the passes of every size, last passes of
    # radix 2, 4 and 8, groups of channels with a remainder, and all sizes in one launch
    chans, off = [], 1
    for N in sizes:
        for ell, n in ((0, 2), (1, 1 + max(1, 2048 // N) % 3)):
            for _ in range(n):
                chans.append((N, ell, 0.1 * N, off))
                off += N + 1
    _check(chans, off, precision)


def _check_steps(chans, total, precision, kind, sample):
    """Two steps against the dense oracle on the sampled channels: two transforms and their
    phase products per step, errors relative to the input (no factor is above one)."""
    from paper_1509_07115_amd import Plan
    dt = 0.02
    rng = np.random.default_rng(total)
    x = rng.standard_normal(total) + 1j * rng.standard_normal(total)
    V = np.abs(rng.standard_normal(total))
    plan = Plan(chans, precision=precision)
    plan.set_potential(V, dt, imaginary=kind == "imaginary")
    xd = torch.from_numpy(x).to(_dtype(precision)).cuda()
    got = plan.kinetic_step(xd.clone(), 2, adjoint=kind == "adjoint").cpu().numpy()
    x0 = xd.cpu().numpy().astype(np.complex128)
    tol = 2 * (2 * TOL[precision] + 4e-7 * (precision == "c64"))
    for N, ell, rmax, off in sample:
        s = slice(off, off + N)
        E, ref = otdse.kinetic_energies(N, rmax, ell), x0[s]
        for _ in range(2):
            ref = (otdse.imag_step(ref, ell, V[s], E, dt) if kind == "imaginary" else
                   otdse.step(ref, ell, V[s], E, dt, adjoint=kind == "adjoint"))
        assert np.linalg.norm(got[s] - ref) <= tol * np.linalg.norm(x0[s]), (kind, N, ell, off)


@pytest.mark.parametrize("precision", ["c64", "c64x", "c128"])
@pytest.mark.parametrize("kind", ["step", "adjoint", "imaginary"])
def test_steps_with_two_to_four_moment_blocks(kind, precision):
    # the kinetic factors at the edges of the moment blocks, one to four tiles, beside channels
    # of small l, with remainders of channels
    chans, off = [], 1
    for N in (64, 128, 256):
        for ell, n in ((3, 2), (33, 9), (64, 1), (65, 9), (95, 1), (96, 3), (97, 8), (126, 9), (127, 1)):
            for _ in range(n if ell <= 2 * N - 2 else 0):
                chans.append((N, ell, 0.1 * N, off))
                off += N + 3
    _check_steps(chans, off, precision, kind, chans)


@pytest.mark.parametrize("kind", ["step", "adjoint", "imaginary"])
def test_steps_of_two_column_blocks(kind):
    # FP32 with more items of 8 channels than compute units: items of 16 channels, whose column
    # blocks share the kinetic factors; 41 channels per l leave an item of 8 and one of 1
    chans, total = _channels(64, [(ell, 41) for ell in range(64, 127)], gap=1)
    _check_steps(chans, total, "c64", kind, [c for i, c in enumerate(chans) if i % 41 in (0, 8, 15, 31, 32, 40)])
