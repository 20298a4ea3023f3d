"""The FP32 rings of mixed-radix lengths are as exact as transforms with one
radix per pass: normwise errors of single-precision plans against
double-precision ones on the same inputs, compared with those that one-radix
kernels had on them (golden/one_radix_errors.json).

The inputs are fixed, so a length's figure moves only with its arithmetic.  Each
is the mean over at least 2e5 rounded values, which pins it to a few parts per
thousand: 1 % is allowed, and 2 % below N = 12, where a handful of roots decide.
"""
import json
import os

import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "one_radix_errors.json")
BANDLIMITS = (3, 4, 6, 9, 12, 18, 24, 27, 36, 48, 54, 72, 81, 96, 108)
KINDS = ("complex", "so3")
CALLS = ("forward", "inverse", "adjoint")


def errors(B, kind):
    """Normwise error of the c64 plan's forward, inverse and adjoint."""
    kw = dict(group="so3") if kind == "so3" else {}
    batch = max(1, min(1024, 4_000_000 // (2 * B) ** 3))
    p64, p32 = su2.Plan(B, batch, "c128", **kw), su2.Plan(B, batch, "c64", **kw)
    g = torch.Generator().manual_seed(B)
    x = torch.view_as_complex(torch.rand(p32.total_samples, 2, generator=g) * 2 - 1).to("cuda")
    c = torch.view_as_complex(torch.randn(p32.total_coeffs, 2, generator=g)).to("cuda")
    out = []
    for call in CALLS:
        a = x if call == "forward" else c
        want = getattr(p64, call)(a.to(torch.complex128))
        out.append(float((getattr(p32, call)(a) - want).norm() / want.norm()))
    p64.close()
    p32.close()
    return out


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("B", BANDLIMITS)
def test_errors_no_larger_than_one_radix_per_pass(B, kind):
    with open(GOLDEN) as fh:
        before = json.load(fh)[f"{kind} {B}"]
    allowed = 1.02 if B < 6 else 1.01
    for call, now, was in zip(CALLS, errors(B, kind), before):
        assert now <= allowed * was, (call, now, was)
