"""discretize(): where memory is short and where substeps are few (GPU).  The outputs come
first, and the workspace of the two-launch form is taken only if it can be had beside them;
one or two substeps take one launch longer than more do.
"""
import numpy as np
import pytest

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


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name,waves64,waves32", [("hopper", 1, 1), ("cheetah7", 2, 1),
                                                  ("quad13", 6, 2)])
def test_few_substeps(name, waves64, waves32, dtype):
    """One and two substeps: one launch past the line of more, two from some rounds of
    the CUs on; the routed call is bitwise the form that the rule names."""
    from paper_2604_09993_amd import api
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    fp32 = dtype == torch.float32
    groups = waves32 if fp32 else waves64
    rounds = 16 if fp32 and name == "hopper" else (2 if fp32 else 3.2)
    for K in (1, 2):
        line = int(rounds * cus / K) // groups
        for N in (line, line + 1):
            print(f"[gpu] route {name} {dtype} N={N} K={K}", flush=True)
            args = _inputs(api, name, N, dtype)
            got = api.discretize(*args, K)
            form = {k: torch.empty_like(v) for k, v in got.items()}
            if N > line:
                form = api.discretize_split(*args, K)
            else:
                api.discretize_into(*args, K, form)   # (one launch always)
            torch.cuda.synchronize()
            assert all(torch.equal(got[k], form[k]) for k in form), (N, K)
