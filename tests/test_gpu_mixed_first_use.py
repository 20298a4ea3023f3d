"""A mixed plan's call is launched directly the first time its direction,
buffers and stream are used, captured into a graph the second time and
replayed from then on: all three give the same bits, also when more
combinations are in use than the plan remembers, on a second stream, and with
eager work between."""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu


def test_direct_captured_and_replayed_calls_agree(monkeypatch):
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    plan = su2.MixedPlan([16, 24, 9, 32, 24], "c64")
    x = torch.view_as_complex(torch.randn(plan.total_samples, 2, device="cuda"))
    ref_c = plan.forward(x)
    ref_x = plan.inverse(ref_c)
    ref_a = plan.adjoint(ref_c)
    # 40 output buffers: more than the 32 remembered first uses and 16 graphs
    outs = [torch.empty_like(ref_c) for _ in range(40)]
    for _ in range(3):
        for o in outs:
            o.zero_()
            assert plan.forward(x, out=o) is o
        assert all(torch.equal(o, ref_c) for o in outs)
        back = torch.zeros_like(ref_x)
        for ref, call in ((ref_x, plan.inverse), (ref_a, plan.adjoint)):
            for _ in range(3):
                back.zero_()
                assert torch.equal(call(ref_c, out=back), ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = [plan.forward(x, out=outs[0]).clone() for _ in range(3)]
    torch.cuda.current_stream().wait_stream(side)
    assert all(torch.equal(g, ref_c) for g in got)
