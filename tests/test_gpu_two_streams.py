"""The expert backward on two streams, at a size that takes them (T*k*d*f = 5.4e8, a few rounds of tiles), at one just
below the size where the helper stream begins, and (bf16) at a smaller one with 101 MB of class gradients, which takes it too:
the same bits as on one stream, eager and replayed from a HIP graph."""
import pytest
import torch

import paper_2504_19925_amd as symi
import workloads as wl
import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("E,d,f,T", [(16, 512, 512, 1024), (16, 328, 512, 1024), (64, 256, 512, 256)])
def test_two_streams(dtype, E, d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype=dtype, E=E, k=2, d=d, f=f, T=T, S_tot=E + E // 2, N=1, iters=1, router_matmul=False)
    print(f"[two streams] {dtype} E={E} d={d} f={f} T={T}", flush=True)
    weights = wl.make_class_weights(c, "cuda")
    X, logits, dY = Hn.draw_inputs(c, 0)
    outs = []
    for flags, how in ((symi.CTX_NO_OVERLAP, "eager"), (0, "eager"), (0, "graph")):
        st = Hn.State(c, weights=weights, flags=flags)
        st.place_current()
        st.forward(X, logits)
        results = (st.dX, st.dW1, st.dW2, st.dgate, st.dlogits)

        def clear():
            for t in results:
                t.fill_(float("nan"))

        if how == "eager":
            clear()
            st.backward(dY, logits)
            Hn.sync()
            outs.append([t.clone() for t in results])
            continue
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        Hn.sync()
        with torch.cuda.stream(s):
            st.backward(dY, logits)
            s.synchronize()
            g.capture_begin()
            st.backward(dY, logits)
            g.capture_end()
        for _ in range(3):
            clear()
            Hn.sync()
            g.replay()
            Hn.sync()
            outs.append([t.clone() for t in results])
            clear()
            st.backward(dY, logits)   # the program's own work between the replays
            Hn.sync()
            outs.append([t.clone() for t in results])
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert torch.equal(a, b)
