"""Small batches run streaming contraction kernels instead of the tile kernels,
with the same products in the same order: every signal of a single-B plan
equals, bit for bit, the same signal in a mixed plan (whose work lists always
run the tile kernels; the oracle tests cover those).

The sizes are where the streaming kernels differ: one to four row tiles of 16
degrees, N not a multiple of 4 or 16, pair lists with and without a self-mirror
middle tile and without mirror symmetry, whole and partial groups of 4 signals
(8 in real plans), spectra read directly or through LDS, and batches on both
sides of the switch to the tile kernels.
"""
import numpy as np
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu

CASES = ([(B, "complex") for B in (6, 12, 18, 24, 27, 32, 36, 54, 64, 72, 81, 96)] +
         [(B, kind) for kind in ("real", "so3") for B in (16, 24, 64)])


def _random(shape, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if dtype.is_complex:
        real = torch.float64 if dtype == torch.complex128 else torch.float32
        return torch.view_as_complex(torch.randn(*shape, 2, generator=g, dtype=real, device="cuda"))
    return torch.randn(*shape, generator=g, dtype=dtype, device="cuda")


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("B,kind", CASES + [(128, "complex")])
def test_small_batches_bitwise_equal_tile_kernels(B, kind, dtype, monkeypatch):
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    total = 17 if B <= 64 else 9
    big = su2.MixedPlan([B] * total, dtype, **kw)
    one = su2.Plan(B, 1, dtype, **kw)
    x = _random((total, *one.sample_shape[1:]), one.sample_dtype, B)
    c = _random((total, one.ncoef), one.torch_dtype, B + 1)
    one.close()
    want = [big.forward(x.view(-1)).view(total, -1).cpu().numpy(), big.inverse(c.view(-1)).view(x.shape).cpu().numpy(),
            big.adjoint(c.view(-1)).view(x.shape).cpu().numpy()]
    big.close()
    for batch in (1, 2, 4, 5, 8, 17) if B <= 64 else (1, 2, 5):
        plan = su2.Plan(B, batch, dtype, **kw)
        # signals from both ends
        at = list(range(batch - batch // 2)) + list(range(total - batch // 2, total))
        got = [plan.forward(x[at]).cpu().numpy(), plan.inverse(c[at]).cpu().numpy(), plan.adjoint(c[at]).cpu().numpy()]
        plan.close()
        for name, g, w in zip(("forward", "inverse", "adjoint"), got, want):
            assert np.array_equal(g, w[at]), (batch, name)
