"""Signals share waves, products and LDS tiles in the contractions and the small
grids' kernels: an infinity or a NaN in one signal leaves every bit of the others
as it is without it."""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu

# batches of one and two groups of signals, and past the streaming kernels
CASES = [(4, 5), (6, 5), (8, 5), (9, 4), (12, 9), (24, 4), (24, 60), (36, 7), (64, 4), (64, 8), (64, 9), (72, 6), (96, 4)]


@pytest.mark.parametrize("dtype", ["c64", "c128", "c64_bf16x3"])
@pytest.mark.parametrize("kind", ["complex", "so3"])
@pytest.mark.parametrize("B,batch", CASES)
def test_other_signals_keep_their_bits(B, batch, kind, dtype):
    plan = su2.Plan(B, batch, dtype, **(dict(group="so3") if kind == "so3" else {}))
    g = torch.Generator(device="cuda").manual_seed(B)
    real = torch.float64 if dtype == "c128" else torch.float32
    bad = batch // 2
    keep = [s for s in range(batch) if s != bad]
    for call, shape in (("forward", plan.sample_shape), ("inverse", plan.coeff_shape), ("adjoint", plan.coeff_shape)):
        a = torch.view_as_complex(torch.randn(*shape, 2, generator=g, dtype=real, device="cuda"))
        want = getattr(plan, call)(a).clone()
        for value in (float("inf"), float("nan")):
            b = a.clone()
            b.view(batch, -1)[bad] = complex(value, 0.0)
            got = getattr(plan, call)(b)
            assert not torch.isfinite(torch.view_as_real(got[bad])).all()
            assert torch.equal(got[keep], want[keep]), (call, value)
    plan.close()
