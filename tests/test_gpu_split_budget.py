"""Register budget of the FP32 tangent launch with 13 pairs (GPU): it changes at two and a
half intervals per CU; both sides of the line against the oracle, and each other.
"""
import pytest

from test_gpu_reduced import _case, _check, _dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_line():
    from paper_2604_09993_amd import api
    line = 5 * torch.cuda.get_device_properties(0).multi_processor_count // 2
    out = []
    model, d = _case(4, 3, "flat", line + 1)
    for N in (line, line + 1):
        print(f"[gpu] split FP32 4x3 flat N={N}", flush=True)
        e = dict(d, X=d["X"][:N + 1], U=d["U"][:N + 1], s=d["s"][:N])
        cm, X, U, s, p = _dev(model, e, torch.float32)
        out.append(api.discretize_split(cm, X, U, s, p, 2))
        torch.cuda.synchronize()
        _check(model, e, 2, out[-1], torch.float32)
    # (the same arithmetic at either budget)
    assert all(torch.equal(out[0][k], out[1][k][..., :line]) for k in out[0])
