"""Single-B plans switch from the streaming contractions to the tile kernels at
batches that depend on bandlimit, type, direction and kind of plan: the last
batch of the one and the first of the other give every signal the bits it has in
a mixed plan, whose work lists always run the tile kernels.

The limits are the dispatch rules' for the compute units of the device, with the
pair tiles of the plan's layout.
"""
import pytest
import torch

import paper_2605_23923_amd as su2
from test_table_padding import PT, _degrees

pytestmark = pytest.mark.gpu

CASES = [(B, "complex", dtype) for B in (18, 24, 27, 36, 48, 54, 64, 72, 108) for dtype in ("c64", "c128", "c64_bf16x3")]
CASES += [(B, "so3", dtype) for B in (32, 72, 96) for dtype in ("c64", "c128", "c64_bf16x3")]
CASES += [(B, "real", dtype) for B in (16, 32, 64) for dtype in ("c64", "c128", "c64_bf16x3")]


def _limits(B, kind, dtype):
    """Largest streaming batch of the forward and the inverse."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    half = kind == "real" and B in (8, 16, 32, 64)  # half-spectrum: a pair per wave, tiles from 2m = 0 up
    tiles = len(_degrees(B, kind == "so3", True)) // PT
    if half:
        low = sum(1 for m in range(-(B - 1), 0) for n in range(-(B - 1), B) if (m - n) % 2 == 0)
        units = tiles - (low + PT - 1) // PT
    else:
        units = (tiles + 1) // 2
    fills, few = 4 * units >= 3 * cus, B <= 32
    if dtype == "c64_bf16x3":
        fwd = (12 if 64 < B <= 108 else 8) if fills else (2500 if few else 1800) // units
        inv = (12 if 64 < B <= 96 else 8) if fills else ((1000 if B <= 16 else 520) if half else 4000 if B <= 54 else 2200) // units
    elif dtype == "c64":
        fwd = (12 if B > 64 else 8) if fills else 1600 // units
        inv = (12 if B > 64 else 8) if fills else min(40, 3600 // units)
    else:
        fwd = 8 if fills else (1600 if few else 2300 if B <= 54 else 1200) // units
        inv = (4 if half else 8) if fills else (2550 if few else 2900 if B <= 54 else 1200) // units
    return fwd, inv


def _random(n, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if dtype.is_complex:
        real = torch.float64 if dtype == torch.complex128 else torch.float32
        return torch.view_as_complex(torch.randn(n, 2, generator=g, dtype=real, device="cuda"))
    return torch.randn(n, generator=g, dtype=dtype, device="cuda")


@pytest.mark.parametrize("B,kind,dtype", CASES)
def test_last_streaming_and_first_tile_batch(B, kind, dtype, monkeypatch):
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    ref = su2.MixedPlan([B] * 3, dtype, **kw)
    x, c = _random(ref.total_samples, ref.sample_dtype, B), _random(ref.total_coeffs, ref.torch_dtype, B + 1)
    want = {"forward": ref.forward(x).view(3, -1), "inverse": ref.inverse(c).view(3, -1), "adjoint": ref.adjoint(c).view(3, -1)}
    ref.close()
    fwd, inv = _limits(B, kind, dtype)
    for call, limit in (("forward", fwd), ("inverse", inv), ("adjoint", inv)):
        for batch in (limit, limit + 1):
            plan = su2.Plan(B, batch, dtype, **kw)
            at = torch.arange(batch, device="cuda") % 3
            src = (x if call == "forward" else c).view(3, -1)[at].reshape(plan.sample_shape if call == "forward" else plan.coeff_shape)
            got = getattr(plan, call)(src).view(batch, -1)
            plan.close()
            for s in range(3):
                assert torch.equal(got[s::3], want[call][s].expand_as(got[s::3])), (call, batch, s)
            del src, got
