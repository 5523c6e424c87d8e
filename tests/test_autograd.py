"""CPU tests of the autograd scores' host side (the kernels' calls replaced)."""
import contextlib

import pytest
import torch

import paper_2506_20043_amd as pv


@pytest.mark.parametrize("requires,mode,want", [(True, contextlib.nullcontext, True), (False, contextlib.nullcontext, False),
                                                (True, torch.no_grad, False), (True, torch.inference_mode, False)])
def test_the_gradient_is_computed_where_it_is_recorded(monkeypatch, requires, mode, want):
    """Only a forward pass that a backward may follow asks the kernel for the gradient and keeps it."""
    asked = []

    def score(ctx, grids, ligs, lp, bp, dof, grad=True):
        asked.append(grad)
        return {"energy": dof.sum(1), **({"grad_dof": torch.ones_like(dof)} if grad else {})}

    monkeypatch.setattr(pv, "score_grad", score)
    monkeypatch.setattr(pv, "_scale_grad", lambda ctx, ligs, lp, grad, of_xyz, g: grad * g[:, None])
    dof = torch.arange(12.0).reshape(3, 4).requires_grad_(requires)
    with mode():
        e = pv.ScoreGrad.apply(dof, (None,) * 5)
    assert asked == [want] and e.requires_grad == want
    if want:
        (g,) = torch.autograd.grad(e, dof, torch.tensor([1.0, 2.0, 3.0]))
        assert torch.equal(g, torch.tensor([1.0, 2.0, 3.0])[:, None].expand(3, 4))
