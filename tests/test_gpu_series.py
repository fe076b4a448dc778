"""GPU parity of the matrix-core kernel for short univariate series (sets of kernels of one dilation) against the CPU
oracle, at the sizes where its steps, sets and choice of path can go wrong.  Needs an MI355X."""
import numpy as np
import pytest

from kernels_of import sampled
from paper_2301_08527_amd import rocket
from parity import check_forward

pytestmark = pytest.mark.gpu


def _run(B, L, K, mask, lam=10.0, u8=False):
    import torch
    h, kr = sampled(L + K, K, 1, L)
    rng = np.random.default_rng(L)
    print("series", B, L, K, mask, lam, flush=True)
    if u8:
        import oracle
        raw = rng.integers(0, 256, size=(B, 1, L)).astype(np.uint8)
        out = rocket.rocket_transform_u8(h, torch.from_numpy(raw).cuda(), mask, lam).cpu().numpy()
        x = oracle.znormalize_u8(raw)
    else:
        x = rng.standard_normal((B, 1, L)).astype(np.float32)
        out = rocket.rocket_transform(h, torch.from_numpy(x).cuda(), mask, lam).cpu().numpy()
    check_forward(x, kr, out, mask, lam=lam)


@pytest.mark.parametrize("mask", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("B,L,K", [(2, 11, 9), (3, 33, 70), (5, 97, 200)])    # shorter than a step of 32; sets of one to sixteen kernels
def test_every_mask_on_small_series(B, L, K, mask):
    _run(B, L, K, mask)


@pytest.mark.parametrize("B,L,K,mask", [
    (3, 2400, 600, 7), (2, 4900, 300, 3),       # four, two and one workgroup to a CU
    (2, 9700, 100, 7), (2, 10400, 100, 7),      # either side of the longest series that LDS holds
    (11, 9700, 9700, 3), (10, 10400, 10400, 2),     # the same, with enough kernels for the sets to be taken
    (40, 3000, 3000, 3), (25, 4900, 4900, 7),
    (40, 1500, 3000, 3),                        # several sets to a wavefront
    (64, 3000, 300, 7), (40, 8000, 200, 2),     # few kernels to a dilation: those go through the job kernels
])
def test_long_and_thin(B, L, K, mask):
    _run(B, L, K, mask)


@pytest.mark.parametrize("lam", [-2.0, 0.0, 0.3, 1000.0])
def test_slope_of_any_sign(lam):
    _run(3, 150, 120, 7, lam=lam)


def test_raw_bytes():
    _run(5, 701, 333, 7, u8=True)
