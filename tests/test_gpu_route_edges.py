"""discretize() where memory is short (GPU): the outputs come first, and the workspace of
the two-launch form is taken only if it can be had beside them.
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from test_gpu_route import _inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_outputs_before_the_workspace(monkeypatch):
    from paper_2604_09993_amd import api
    print("[gpu] route, memory for the outputs alone", flush=True)
    args = _inputs(api, "quad13", 64, torch.float64)
    one = api.discretize(*args, 3, layout="throughput")
    two = api.discretize(*args, 3)
    assert not all(torch.equal(one[k], two[k]) for k in one)
    left = [sum(v.numel() * v.element_size() for v in one.values())]
    empty = torch.empty

    def limited(shape, **kw):
        need = int(np.prod(shape)) * torch.tensor([], dtype=kw["dtype"]).element_size()
        if need > left[0]:
            raise torch.cuda.OutOfMemoryError("limit of the test")
        left[0] -= need
        return empty(shape, **kw)

    monkeypatch.setattr(api.torch, "empty", limited)
    got = api.discretize(*args, 3)
    monkeypatch.undo()
    torch.cuda.synchronize()
    assert left[0] == 0
    assert all(torch.equal(got[k], one[k]) for k in one)
