"""Calls of the grids N = 12 and 16 run as one kernel up to some signals per
compute unit and as two kernels above: on both sides of every limit each signal
has the bits it has alone."""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu

# (B, dtype, kind, call): signals per compute unit of the last batch in one kernel
LIMITS = [
    (6, "c128", "complex", "forward", 5),
    (6, "c128", "so3", "forward", 5),
    (6, "c128", "real", "inverse", 24),
    (8, "c128", "complex", "inverse", 5),
    (8, "c128", "complex", "adjoint", 5),
    (6, "c64", "complex", "inverse", 12),
    (8, "c64", "complex", "adjoint", 12),
    (6, "c64", "so3", "inverse", 16),
    # none, or one kernel again where the spectra outgrow the cache
    (8, "c128", "complex", "forward", 20),
    (8, "c64", "complex", "inverse", 64),
]


@pytest.mark.parametrize("B,dtype,kind,call,per_cu", LIMITS)
def test_both_sides_of_the_limit(B, dtype, kind, call, per_cu):
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    one = su2.Plan(B, 1, dtype, **kw)
    shape = one.sample_shape[1:] if call == "forward" else one.coeff_shape[1:]
    dt = one.sample_dtype if call == "forward" else one.torch_dtype
    g = torch.Generator(device="cuda").manual_seed(B)
    few = torch.randn(5, *shape, generator=g, dtype=torch.float64, device="cuda")
    if dt.is_complex:
        few = torch.complex(few, torch.randn(5, *shape, generator=g, dtype=torch.float64, device="cuda"))
    few = few.to(dt)
    want = torch.cat([getattr(one, call)(few[i:i + 1]) for i in range(5)])
    one.close()
    edge = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    for batch in (edge - 1, edge, edge + 1):
        at = torch.arange(batch, device="cuda") % 5
        plan = su2.Plan(B, batch, dtype, **kw)
        got = getattr(plan, call)(few[at])
        plan.close()
        for i in range(5):
            assert torch.equal(got[i::5], want[i].expand_as(got[i::5])), (batch, i)
