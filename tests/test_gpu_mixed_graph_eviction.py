"""A mixed plan keeps the graphs of 16 combinations of direction, buffers and
stream: with more in use the oldest is destroyed, and its combination is launched
directly, captured and replayed again when it returns, always with the same bits."""
import pytest
import torch

import paper_2605_23923_amd as su2

pytestmark = pytest.mark.gpu


def test_evicted_graphs_return(monkeypatch):
    monkeypatch.setenv("SU2_AUTOTUNE", "0")
    plan = su2.MixedPlan([16, 24, 9, 32, 24], "c64")
    x = torch.view_as_complex(torch.randn(plan.total_samples, 2, device="cuda"))
    c = plan.forward(x)
    want = {"forward": c.clone(), "inverse": plan.inverse(c), "adjoint": plan.adjoint(c)}
    # 20 buffers, each used three times in a row: launched, captured, replayed; from the
    # 17th on the oldest graph goes.  Then the first five again, and a few others' replays.
    for call, src in (("forward", x), ("inverse", c), ("adjoint", c)):
        outs = [torch.empty_like(want[call]) for _ in range(20)]
        for o in outs + outs[:5] + outs[12:17]:
            for _ in range(3):
                o.zero_()
                assert getattr(plan, call)(src, out=o) is o
                assert torch.equal(o, want[call])
    plan.close()
