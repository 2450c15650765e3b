"""The device calls' argument checks in C++ (_marshal.so) against the ctypes path of the same
functions: same results, keywords accepted, everything refused that was refused, with the same text."""
import pytest
import torch

import harness as Hn
import paper_2504_19925_amd as symi
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def layer():
    c = wl.scaled(wl.get_config("c1"), T=96)
    st = Hn.State(c)
    X, logits, dY = Hn.draw_inputs(c, 0)
    return st, logits


def test_every_device_call_is_marshalled_and_equals_the_ctypes_path(layer):
    st, logits = layer
    assert {n for n in symi.EXPORTS if hasattr(getattr(symi, n, None), "__wrapped__")} == set(symi.binding._marshal)
    got = []
    for f in (symi.symi_route, symi.symi_route.__wrapped__):
        st.idx.fill_(-1)
        f(st.ctx, logits, st.idx, st.gate, st.hist)
        got.append((st.idx.clone(), st.gate.clone(), st.hist.clone()))
    symi.symi_route(st.ctx, logits=logits, idx=st.idx, gate=st.gate, hist=st.hist)
    got.append((st.idx, st.gate, st.hist))
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    p = torch.nn.Parameter(logits)   # a tensor like any other
    symi.symi_route(st.ctx, p, st.idx, st.gate, st.hist)
    assert torch.equal(got[0][0], st.idx)


@pytest.mark.parametrize("break_it", ["dtype", "short", "strided", "cpu", "not a tensor", "count", "ctx"])
def test_refusals_are_those_of_the_ctypes_path(layer, break_it):
    st, logits = layer
    args = [st.ctx, logits, st.idx, st.gate, st.hist]
    if break_it == "dtype":
        args[2] = st.idx.long()
    elif break_it == "short":
        args[1] = logits[:-1]
    elif break_it == "strided":
        args[3] = torch.empty(st.gate.shape[0], st.gate.shape[1] * 2, device="cuda")[:, ::2]
    elif break_it == "cpu":
        args[4] = st.hist.cpu()
    elif break_it == "not a tensor":
        args[4] = [0] * 8
    elif break_it == "count":
        args.pop()
    else:
        args[0] = symi.SymiCtx(None, st.cfg, 0)
    said = []
    for f in (symi.symi_route, symi.symi_route.__wrapped__):
        with pytest.raises((symi.SymiError, TypeError)) as e:
            f(*args)
        said.append((type(e.value), str(e.value)))
    assert said[0] == said[1]


def test_the_current_stream_is_used(layer):
    st, logits = layer
    symi.symi_route(st.ctx, logits, st.idx, st.gate, st.hist)
    want = st.idx.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        z = logits.flip(0).contiguous()
        for _ in range(50):
            z = z * 1.0
        symi.symi_route(st.ctx, z, st.idx, st.gate, st.hist)
        got = st.idx.clone()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    assert torch.equal(got, want.flip(0))
