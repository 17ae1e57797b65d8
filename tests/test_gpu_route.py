"""Route of discretize(): one launch or two by the interval count (GPU).

Around the counts where the rule changes, for both types, padded node strides, an
output left out and a stream of the caller's, the routed call is bitwise the form
the rule names and within the bars of tests/parity.py of the other; beyond the
workspace limit it stays with one launch.
"""
import numpy as np
import pytest

from paper_2604_09993_amd import synth
from parity import PHI32, PHI64, TOL32, TOL64, compare_outputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _inputs(api, name, N, dtype, pad=0):
    rng = np.random.default_rng([900, N])
    model = synth.MODEL_MAKERS[name](rng)
    d = synth.gen_nodes(model, N, rng, T=0.02 * N)
    ld = N + 1 + pad
    return (api.CisModel(model), api.to_device_soa(d["X"], dtype=dtype, ld=ld),
            api.to_device_soa(d["U"], dtype=dtype, ld=ld),
            torch.tensor(d["s"], device="cuda", dtype=dtype),
            torch.tensor(d["p"], device="cuda", dtype=dtype))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name,waves64,waves32", [("hopper", 1, None), ("biped5", 2, 1),
                                                  ("cheetah7", 2, 1), ("quad13", 6, 2)])
def test_route_at_the_line(name, waves64, waves32, dtype):
    from paper_2604_09993_amd import api
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    groups = waves64 if dtype == torch.float64 else waves32
    line = 2 * cus if groups is None else cus // groups
    fp32 = dtype == torch.float32
    for N, pad, xprop in ((line, 0, True), (line + 1, 0, True), (line + 1, 3, False)):
        print(f"[gpu] route {name} {dtype} N={N} pad={pad}", flush=True)
        args = _inputs(api, name, N, dtype, pad)
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        got = api.discretize(*args, 3, with_xprop=xprop, stream=stream)
        stream.synchronize()
        two = api.discretize_split(*args, 3)
        one = api.discretize(*args, 3, layout="throughput")
        torch.cuda.synchronize()
        keys = [k for k in two if got[k] is not None]
        assert ("xprop" in keys) == xprop
        routed = all(torch.equal(got[k], two[k]) for k in keys)
        assert routed == (N > line)
        errs = compare_outputs({k: v.double().cpu().numpy() for k, v in
                                api.as_interval_major({k: got[k] for k in keys}).items()},
                               {k: v.double().cpu().numpy() for k, v in
                                api.as_interval_major({k: one[k] for k in keys}).items()},
                               keys, PHI32 if fp32 else PHI64)
        bad = {k: e for k, e in errs.items() if not e <= (TOL32 if fp32 else TOL64)}
        assert not bad, bad


def test_route_workspace_limit(monkeypatch):
    from paper_2604_09993_amd import api
    args = _inputs(api, "quad13", 64, torch.float64)
    two = api.discretize(*args, 3)
    monkeypatch.setattr(api, "SPLIT_WS_MAX", 0)
    got = api.discretize(*args, 3)
    one = api.discretize(*args, 3, layout="throughput")
    torch.cuda.synchronize()
    assert all(torch.equal(got[k], one[k]) for k in one)
    assert not all(torch.equal(got[k], two[k]) for k in two)
