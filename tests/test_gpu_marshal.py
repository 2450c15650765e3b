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


def _arguments(st, X, logits, dY):
    """A valid argument list of every device call; every tensor is exactly as large as the call needs."""
    E, S, d, f = st.c.E, st.c.S_tot, st.c.d, st.c.f
    new = lambda *n, dtype=st.cfg.torch_dtype: torch.zeros(*n, dtype=dtype, device="cuda")
    f32 = torch.float32
    fwd = [X, st.idx, st.hist, st.counts, st.first_slot, st.row_of_assign, st.assign_of_row, st.slot_offsets, st.Xp]
    bwd = [st.dYp, st.Xp, st.UV, st.H, st.slot_offsets, st.first_slot, st.W1s, st.W2s, st.dXp]
    dW = [st.dW1, st.dW2]
    dWs = [new(S, 2 * f, d, dtype=f32), new(S, d, f, dtype=f32)]
    opt = [Hn.make_adam()[0], *dW, st.master, st.m, st.v]
    Wr, b = new(E, d), new(E, dtype=f32)
    calls = {
        "symi_route": [logits, st.idx, st.gate, st.hist],
        "symi_place": [st.hist, st.counts, st.placement, st.first_slot],
        "symi_dispatch": [*fwd, st.ws],
        "symi_dispatch_noalloc": fwd,
        "symi_dispatch_capacity": [st.c.A, *fwd, st.ws],
        "symi_expert_fwd": [st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws],
        "symi_combine": [st.Yp, st.row_of_assign, st.gate, st.Y],
        "symi_combine_bwd": [dY, st.Yp, st.row_of_assign, st.gate, st.dYp, st.dgate],
        "symi_expert_bwd": [*bwd, *dW, st.ws],
        "symi_expert_bwd_active": [*bwd, *dW, st.ws],
        "symi_expert_bwd_slots": [*bwd, *dWs, st.ws],
        "symi_replica_allreduce": [st.first_slot, 1.0, *dWs],
        "symi_dispatch_bwd": [st.dXp, st.row_of_assign, st.dX],
        "symi_route_bwd": [logits, st.idx, st.gate, st.dgate, st.dlogits],
        "symi_router_fwd": [X, Wr, b, new(st.c.T, E, dtype=f32)],
        "symi_router_bwd": [X, Wr, st.dlogits, new(E, d, dtype=f32), new(E, dtype=f32), st.dX, st.ws],
        "symi_adam_to_replicas": [*opt, st.first_slot, st.W1s, st.W2s],
        "symi_adam_to_replicas_active": [*opt, st.slot_offsets, st.first_slot, st.first_slot, st.W1s, st.W2s],
    }
    return {n: [st.ctx, *a] for n, a in calls.items()}


OTHER = {torch.float32: torch.int32, torch.int32: torch.float32, torch.bfloat16: torch.float16,
         torch.uint8: torch.int8}   # of the same size


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_every_call_takes_exact_sizes_and_refuses_less(dtype):
    """Every tensor of every call: accepted in C++ at exactly the size the call needs; one element
    less, or another type of the same size, is refused with the ctypes path's words.  Sizes differ between
    any two quantities, so that a mistaken one shows."""
    c = wl.scaled(wl.get_config("c1"), dtype=dtype, E=6, k=3, d=40, f=56, T=97, S_tot=11, N=2, router_matmul=False)
    st = Hn.State(c)
    X, logits, dY = Hn.draw_inputs(c, 0)
    st.place_current()
    calls = _arguments(st, X, logits, dY)
    assert set(calls) == set(symi.binding._marshal)
    for name, args in calls.items():      # in the order of an iteration
        assert symi.binding._marshal[name](*args) == 0, name
        for i, t in enumerate(args):
            if not isinstance(t, torch.Tensor):
                continue
            for bad in (t.view(-1)[:-1], t.view(OTHER[t.dtype])):   # (the memory is whole either way)
                wrong = args[:i] + [bad] + args[i + 1:]
                assert symi.binding._marshal[name](*wrong) is None, (name, i)
                said = []
                for call in (getattr(symi, name), getattr(symi, name).__wrapped__):
                    with pytest.raises(symi.SymiError, match="needs at least|expected dtype") as e:
                        call(*wrong)
                    said.append(str(e.value))
                assert said[0] == said[1], name
    torch.cuda.synchronize()
    for name, i in (("symi_router_fwd", 3), ("symi_router_bwd", 5)):      # the bias may be left out
        args = list(calls[name])
        args[i] = None
        assert symi.binding._marshal[name](*args) == 0, name
