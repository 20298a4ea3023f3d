"""The mixed-radix ring kernels at every N = 2B they take, in both types: their
splits differ per N and type (slices per ring, DFT lengths up to 18, several
rings per workgroup below N = 24), so each is checked on its own.

Per B: an exact round trip (every coefficient, hence every bin of every ring),
and sampled coefficients of a non-bandlimited signal and sampled synthesis
points against the oracle.  Three signals, so that workgroups of several rings
and slice groups end in the middle.  Tolerances as in test_gpu_parity.py
(1e-10 / 1e-6 against the oracle), twice that for the round trip's two
transforms in FP32, and 1e-11 in FP64.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_23923_amd as su2
import synth

pytestmark = pytest.mark.gpu

NPDT = {"c128": np.complex128, "c64": np.complex64}
TOL = {"c128": 1e-10, "c64": 1e-6}
TOL_RT = {"c128": 1e-11, "c64": 2e-6}


def _rel(got, ref):
    got, ref = np.asarray(got, np.complex128).reshape(-1), np.asarray(ref, np.complex128).reshape(-1)
    assert np.all(np.isfinite(got))
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 6, 9, 12, 18, 24, 27, 36, 48, 54, 72, 81, 96, 108])
def test_mixed_radix_rings(B, dtype):
    batch = 3
    plan = su2.Plan(B, batch, dtype)
    c = synth.coeffs(B, batch, seed=300 + B, dtype=NPDT[dtype])
    x = plan.inverse(torch.from_numpy(c).cuda())
    assert _rel(plan.forward(x).cpu().numpy(), c) <= TOL_RT[dtype]
    rng = np.random.default_rng(B)
    pts = rng.choice((2 * B) ** 3, min((2 * B) ** 3, 24), replace=False)
    assert _rel(x[2].cpu().numpy().reshape(-1)[pts], oracle.inverse(B, c[2].astype(np.complex128), pts)) <= TOL[dtype]
    u = synth.samples_uniform(B, batch, seed=400 + B, dtype=NPDT[dtype])
    f = plan.forward(torch.from_numpy(u).cuda()).cpu().numpy()
    sel = rng.choice(oracle.num_coeffs(B), min(oracle.num_coeffs(B), 12), replace=False)
    assert _rel(f[1][sel], oracle.forward(B, u[1].astype(np.complex128), sel)) <= TOL[dtype]
    plan.close()


def test_noalloc_limit_is_the_documented_one():
    """The scratch limit counts P rounded up to 16 at the mixed-radix sizes
    too, whatever padding their pair lists carry: B = 24 in c64 fits up to
    8 x 48 x 1120 x batch <= 64 MiB."""
    N, P16 = 48, 1120
    fits = (64 << 20) // (8 * N * P16)
    for batch, ok in ((fits, True), (fits + 1, False)):
        plan = su2.Plan(24, batch, "c64")
        x = torch.view_as_complex(torch.randn(batch, N, N, N, 2, device="cuda"))
        out = torch.empty(plan.coeff_shape, dtype=torch.complex64, device="cuda")
        if ok:
            assert torch.equal(plan.forward_noalloc(x, out), plan.forward(x))
        else:
            with pytest.raises(su2.SU2Error) as ei:
                plan.forward_noalloc(x, out)
            assert ei.value.status == 2
        plan.close()
