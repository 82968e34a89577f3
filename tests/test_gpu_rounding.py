"""Rounding of the moment stage: what the choice of tile and the other channels of
a plan may and may not change in a channel's result."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _packed(N, ells):
    return [(N, ell, 0.05 * N, i * N) for i, ell in enumerate(ells)]


def _random(n, dtype, seed=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.view_as_complex(torch.randn(n, 2, dtype=torch.float64, device="cuda", generator=g)).to(dtype)


LOW = [ell for ell in (0, 1, 2, 5, 9, 15, 16, 20, 31, 32, 40, 47, 50, 62) for _ in range(8)]


@pytest.mark.parametrize("N", [512, 2048])
def test_tiles_of_64_round_no_more_than_tiles_of_32(N):
    # error of complex64 against complex128 over 112 channels of random data; the bound
    # is the four-wave pipeline's own error on the same data
    from paper_1509_07115_amd import Plan
    chans = _packed(N, LOW)
    x = _random(N * len(chans), torch.complex64)
    exact = Plan(chans, precision="c128")
    for call in ("forward", "inverse"):
        ref = getattr(exact, call)(x.to(torch.complex128))
        err = {}
        for tile in (32, 64):
            got = getattr(Plan(chans, tile=tile), call)(x).to(torch.complex128)
            err[tile] = (torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref)).item()
        print(f"N={N} {call}: tiles of 32 {err[32]:.4g}, of 64 {err[64]:.4g}")
        assert err[64] <= err[32], (call, err)



def test_long_chains_of_large_l():
    """Errors over 128 tiles, against complex128: the channels of the uneven batch with N =
    8192 and l >= 96.  Bounds 5% above what an FP32 sum over each block row in column order
    gives (2.53e-7 forward), and a tenth below the inverse's 3.44e-7, whose terms came in
    the worst order."""
    from paper_1509_07115_amd import Plan, workloads
    w = workloads.uneven()
    chans = [c for c in w.channels if c[0] == 8192 and c[1] >= 96]
    assert len(chans) > 10
    x = torch.from_numpy(w.psi).to(torch.complex64).cuda()
    plan, exact = Plan(chans), Plan(chans, precision="c128")
    b = plan.forward(x)
    for name, got, ref, bound in (("forward", b, exact.forward(x.to(torch.complex128)), 2.66e-7),
                                  ("inverse", plan.inverse(b), exact.inverse(b.to(torch.complex128)), 3.1e-7)):
        errs = [(torch.linalg.vector_norm(got[o:o + N] - ref[o:o + N]) / torch.linalg.vector_norm(ref[o:o + N])).item()
                for N, _, _, o in chans]
        rms = float(np.sqrt(np.mean(np.square(errs))))
        print(f"{name}: rms {rms:.3e}, largest {max(errs):.3e}")
        assert rms <= bound, name


def _with_potential(chans, mode="batched"):
    from paper_1509_07115_amd import Plan
    plan = Plan(chans, mode=mode)
    V = np.zeros(plan.elems)
    for N, ell, rmax, off in chans:
        V[off:off + N] = -1.0 / np.sqrt(((np.arange(N) + 0.5) * rmax / N) ** 2 + 0.01)
    plan.set_potential(V, 0.02)
    return plan


# (sizes, l of the channels looked at, channels of each, l of the others, channels of each): more and
# fewer items than compute units (two items of a tile size in a workgroup, or one), items of one and two
# column blocks, one tile per channel, unequal sizes (items that share a workgroup end at different tiles)
COMPANY = [((512,), (0, 1, 2, 15, 31, 32, 33, 62), 3, (71,), 1),
           ((64, 512, 128), (0, 1, 2, 15, 31, 32, 33, 62), 2, (65, 96, 100), 3),
           ((64,), tuple(range(0, 63, 3)), 9, (64, 70, 97, 126), 40),
           ((32, 64, 256, 128), tuple(range(50)), 9, (64, 90, 110), 30),
           ((64,), tuple(range(64)), 72, (100, 120), 100),
           ((64,), (0, 5, 40), 9, tuple(range(64, 127)), 40)]


@pytest.mark.parametrize("sizes,low,n_low,high,n_high", COMPANY)
def test_fp32_results_do_not_depend_on_the_other_channels(sizes, low, n_low, high, n_high):
    """complex64 channels with l <= 63 get the same bits with and without channels of
    larger l in the plan: transforms, steps and adjoint steps; and the batched plan the
    bits of the per-channel one."""
    chans, off = [], 1
    for N in sizes:
        for ell, n in [(ell, n_low) for ell in low] + [(ell, n_high) for ell in high if N >= 64]:
            if ell > 2 * N - 2:
                continue
            for _ in range(n):
                chans.append((N, ell, 0.05 * N, off))
                off += N + 1
    alone = [c for c in chans if c[1] <= 63]
    x = _random(off, torch.complex64, seed=7)
    a, b, plain = _with_potential(alone), _with_potential(chans), _with_potential(chans, mode="plain")

    def at(y, some):   # the values of some channels
        return torch.cat([y[o:o + N] for N, _, _, o in some])

    for call in ("forward", "inverse"):
        got = getattr(b, call)(x)
        assert torch.equal(at(getattr(a, call)(x), alone), at(got, alone)), call
        assert torch.equal(at(getattr(plain, call)(x), chans), at(got, chans)), call
    for adjoint in (False, True):
        y, z, w = x.clone(), x.clone(), x.clone()
        a.kinetic_step(y, 3, adjoint=adjoint)
        b.kinetic_step(z, 3, adjoint=adjoint)
        plain.kinetic_step(w, 3, adjoint=adjoint)
        assert torch.equal(at(y, alone), at(z, alone)), adjoint
        assert torch.equal(at(w, chans), at(z, chans)), adjoint


def test_autotuned_complex64_plans_keep_the_default_tile(tmp_path):
    # few items, where tiles of 64 would be the fastest; then a stored line that holds one
    import json

    from paper_1509_07115_amd import Plan
    chans = _packed(2048, [ell for ell in range(16) for _ in range(8)])
    cache = tmp_path / "tune.jsonl"
    first = Plan.autotuned(chans, nrep=5, cache=str(cache)).tuning
    assert first["tile"] in (0, 32)
    line = json.loads(cache.read_text())
    line["tile"] = 64
    cache.write_text(json.dumps(line) + "\n")
    again = Plan.autotuned(chans, nrep=5, cache=str(cache))
    assert again.tuning["tile"] in (0, 32) and len(cache.read_text().splitlines()) == 2
    x = _random(2048 * len(chans), torch.complex64)
    assert torch.equal(again.forward(x), Plan(chans).forward(x))
    # FP64 arithmetic: a stored tile of 64 is taken
    Plan.autotuned(chans, nrep=1, cache=str(cache), precision="c128")
    lines = cache.read_text().splitlines()
    line = json.loads(lines[-1])
    line["tile"] = 64
    cache.write_text("\n".join(lines[:-1] + [json.dumps(line)]) + "\n")
    assert Plan.autotuned(chans, nrep=1, cache=str(cache), precision="c128").tuning["tile"] == 64


@pytest.mark.parametrize("precision", ["c128", "c64x"])
@pytest.mark.parametrize("N", [128, 512, 1024, 2048])
def test_fp64_tile_follows_the_items_per_compute_unit(N, precision):
    # one item of 8 channels per compute unit is the line, at every size; the bits of the
    # results say which tile a plan took
    from paper_1509_07115_amd import Plan
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    for items, tile in ((ncu // 2 + 16, 64), (ncu, 64), (ncu + 1, 32)):
        ells = [3 + i % 13 for i in range(items)]          # 13 l, a remainder in some of them
        chans = _packed(N, [ell for ell in sorted(ells) for _ in range(8)])
        x = _random(N * len(chans), torch.complex64 if precision == "c64x" else torch.complex128)
        b = Plan(chans, precision=precision).forward(x)
        assert torch.equal(b, Plan(chans, precision=precision, tile=tile).forward(x)), (items, tile)
        assert precision == "c64x" or not torch.equal(b, Plan(chans, precision=precision, tile=96 - tile).forward(x))


def test_forty_fp32_steps_of_small_and_large_l_in_one_plan():
    """complex64 against complex128 after 40 steps of random data, 112 channels with l <= 62
    and 96 with l >= 64.  Per step the error is that of two transforms and three unit
    factors, 40 steps add it up at random: sqrt(40) (1.41e-7^2 + 1.57e-7^2 + 3 (1.1e-7)^2)^.5
    = 1.8e-6 for l <= 62 (the transforms' measured errors), with a fifth more allowed for
    what is not random; sums over up to 128 slots and moments may add another tenth.  The
    norm may grow by 3e-7 (2.0e-7 before there were tiles of 64 in FP32 plans)."""
    from paper_1509_07115_amd import Plan
    N = 2048
    high = [ell for ell in (64, 65, 70, 80, 90, 95, 96, 97, 100, 110, 120, 127) for _ in range(8)]
    chans = _packed(N, LOW + high)
    x = _random(N * len(chans), torch.complex64)
    V = np.tile(-1.0 / np.sqrt(((np.arange(N) + 0.5) * 0.05) ** 2 + 0.01), len(chans))
    y = {}
    for precision in ("c64", "c128"):
        plan = Plan(chans, precision=precision)
        plan.set_potential(V, 0.01)
        y[precision] = plan.kinetic_step(x.to(plan.dtype, copy=True), 40).to(torch.complex128).reshape(-1, N)
    cut = len(LOW)
    for name, s, bound in (("l <= 62", slice(0, cut), 2.2e-6), ("l >= 64", slice(cut, None), 2.4e-6)):
        a, b = y["c64"][s], y["c128"][s]
        err = (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()
        growth = (torch.linalg.vector_norm(a) / torch.linalg.vector_norm(b)).item() - 1.0
        print(f"{name}: error {err:.3e}, norm {growth:+.3e}")
        assert err <= bound and abs(growth) <= 3e-7, name
