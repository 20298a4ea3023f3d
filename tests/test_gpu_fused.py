"""Calls of small grids (B <= 8) run as one kernel per call, spectra in LDS.
They and their neighbours equal the stage by stage launches bit for bit, for one signal and
for more signals than the chip has compute units, and leave the ring spectra in
the plan's workspace as the stages do."""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["complex", "real", "so3"])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 6, 8, 9, 12])
def test_one_kernel_calls_equal_stages(B, kind, dtype):
    kw = {"complex": {}, "real": dict(real=True), "so3": dict(group="so3")}[kind]
    for batch in (1, 3, 300):
        plan = su2.Plan(B, batch, dtype, **kw)
        g = torch.Generator(device="cuda").manual_seed(B)
        x = torch.randn(*plan.sample_shape, generator=g, dtype=torch.float64, device="cuda")
        if kind != "real":
            x = torch.complex(x, torch.randn(*plan.sample_shape, generator=g, dtype=torch.float64, device="cuda"))
        x = x.to(plan.sample_dtype)
        c = torch.complex(*(torch.randn(*plan.coeff_shape, generator=g, dtype=torch.float64, device="cuda")
                            for _ in range(2))).to(plan.torch_dtype)
        want_f, want_i, want_a = torch.empty_like(c), torch.empty_like(x), torch.empty_like(x)
        plan.run_stage("ring_forward", x, None)
        plan.run_stage("beta_forward", None, want_f)
        plan.run_stage("beta_inverse", c, None)
        plan.run_stage("ring_inverse", None, want_i)
        plan.run_stage("beta_adjoint", c, None)
        plan.run_stage("ring_adjoint", None, want_a)
        again = torch.empty_like(x)
        for call, stage, want in ((plan.inverse, "ring_inverse", want_i), (plan.adjoint, "ring_adjoint", want_a)):
            assert torch.equal(call(c), want), batch
            plan.run_stage(stage, None, again)
            assert torch.equal(again, want), batch
        assert torch.equal(plan.forward(x), want_f), batch
        again = torch.empty_like(c)
        plan.run_stage("beta_forward", None, again)
        assert torch.equal(again, want_f), batch
        plan.close()
