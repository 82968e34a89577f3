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

