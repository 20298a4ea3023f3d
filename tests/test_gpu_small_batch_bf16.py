"""Small batches of split-BF16 plans run streaming contraction kernels with the
products of the tile kernels: every signal equals, bit for bit, the same signal
in a mixed plan (whose work lists run the tile kernels; the oracle tests cover
those).  Sizes: one to four row tiles, N not a multiple of 8, 16 or 32, lists
with and without mirror symmetry, partial groups of signals, and batches on
both sides of the switch.
"""
import numpy as np
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,kind", [(B, "complex") for B in (9, 18, 27, 32, 36, 54, 64, 81, 128)] +
                         [(B, kind) for kind in ("real", "so3") for B in (16, 32, 64)])
def test_small_bf16_batches_bitwise_equal_tile_kernels(B, kind, monkeypatch):
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    total = 33 if B <= 64 else 9
    big = su2.MixedPlan([B] * total, "c64_bf16x3", **kw)
    one = su2.Plan(B, 1, "c64_bf16x3", **kw)
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(total, *one.sample_shape[1:], generator=g, dtype=torch.float64, device="cuda").to(one.sample_dtype)
    if x.is_complex():
        x = x * (1 + 0.5j)
    c = torch.complex(*(torch.randn(total, one.ncoef, generator=g, dtype=torch.float32, device="cuda") for _ in range(2)))
    one.close()
    want = [big.forward(x.reshape(-1)).view(total, -1).cpu().numpy(),
            big.inverse(c.view(-1)).view(x.shape).cpu().numpy(), big.adjoint(c.view(-1)).view(x.shape).cpu().numpy()]
    big.close()
    for batch in (1, 3, 4, 9, 16, 33) if B <= 64 else (1, 2, 5):
        plan = su2.Plan(B, batch, "c64_bf16x3", **kw)
        at = list(range(batch - batch // 2)) + list(range(total - batch // 2, total))  # signals from both ends
        got = [plan.forward(x[at]).cpu().numpy(), plan.inverse(c[at]).cpu().numpy(), plan.adjoint(c[at]).cpu().numpy()]
        plan.close()
        for name, a, w in zip(("forward", "inverse", "adjoint"), got, want):
            assert np.array_equal(a, w[at]), (batch, name)


@pytest.mark.parametrize("B,batch", [(24, 130), (72, 17), (81, 33), (128, 13)])
def test_bf16_forward_tiles_bitwise_equal_work_lists(B, batch, monkeypatch):
    """The single-plan forward tile kernels at one row tile (two workgroups per
    CU) and four (one pair per wave), whole and partial 16-signal tiles."""
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    big, plan = su2.MixedPlan([B] * batch, "c64_bf16x3"), su2.Plan(B, batch, "c64_bf16x3")
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(*plan.sample_shape, 2, generator=g, device="cuda")
    x = torch.view_as_complex(x)
    want = big.forward(x.view(-1)).view(plan.coeff_shape)
    assert torch.equal(plan.forward(x), want)
    big.close()
    plan.close()
