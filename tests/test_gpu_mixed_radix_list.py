"""Mixed plans run the rings of several small groups of mixed-radix lengths in
one launch: every signal has the bits of its own single-B plan, in each
direction, precision and kind of plan.

The mixes hold every length of that launch, partly filled last workgroups (the
rings of a group are not a multiple of the rings per workgroup), a longer
mixed-radix group beside them, register-resident groups beside them or none, and
one such group alone (which keeps its own launch).
"""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu

MIXES = {
    "every_length": [1, 2, 3, 4, 6, 9, 12, 18, 24, 27],
    "ragged": [27, 3, 18, 3, 9, 27, 3, 24, 1, 18, 18],
    "beside_others": [36, 8, 24, 16, 12, 6, 12],
    "one_group": [12, 32, 12],
}


def _random(n, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if dtype.is_complex:
        real = torch.float64 if dtype == torch.complex128 else torch.float32
        return torch.view_as_complex(torch.randn(n, 2, generator=g, dtype=real, device="cuda"))
    return torch.randn(n, generator=g, dtype=dtype, device="cuda")


@pytest.mark.parametrize("dtype", ["c128", "c64", "c64_bf16x3"])
@pytest.mark.parametrize("kind", ["complex", "real", "so3"])
@pytest.mark.parametrize("mix", sorted(MIXES))
def test_ring_list_bitwise_equals_single_plans(mix, kind, dtype, monkeypatch):
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    Bs = MIXES[mix]
    mp = su2.MixedPlan(Bs, dtype, **kw)
    x = _random(mp.total_samples, mp.sample_dtype, 7)
    c = _random(mp.total_coeffs, mp.torch_dtype, 8)
    got = mp.forward(x), mp.inverse(c), mp.adjoint(c)
    mp.close()
    xo = co = 0
    for s, B in enumerate(Bs):
        p = su2.Plan(B, 1, dtype, **kw)
        xs, cs = x[xo:xo + p.total_samples], c[co:co + p.total_coeffs]
        want = p.forward(xs), p.inverse(cs), p.adjoint(cs)
        for name, g, w in zip(("forward", "inverse", "adjoint"), got, want):
            part = g[co:co + p.total_coeffs] if name == "forward" else g[xo:xo + p.total_samples]
            assert torch.equal(part, w.view(-1)), (s, B, name)
        xo, co = xo + p.total_samples, co + p.total_coeffs
        p.close()
