"""The 128 x 128 tile of the bf16 variable-row products (few or short tiles) against the oracle's layer: slots of one
row up to three tiles, both sides of the 64 rows below which half the wavefronts rest, reductions of one to six 64-deep
steps with and without a ragged end, ragged columns, numbers of column tiles that are and are not multiples of eight,
and sizes on both sides of the rule that chooses it."""
import pytest
import torch

import paper_2504_19925_amd as symi
import workloads as wl
import harness as Hn
from tests.checks import check_iteration

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,S,d,f,T", [(2, 1, 2, 8, 8, 70), (3, 2, 4, 64, 72, 129), (4, 1, 5, 136, 520, 641),
                                         (6, 2, 9, 200, 328, 333), (4, 2, 6, 392, 264, 500), (2, 1, 3, 320, 1032, 385),
                                         # 128 rows per slot on average and one more, K = 1024 and 1032
                                         (4, 1, 4, 1024, 72, 512), (4, 1, 4, 1024, 72, 513), (4, 1, 4, 1032, 72, 512),
                                         (16, 4, 16, 256, 1024, 4100)])
def test_layer(E, k, S, d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=E, k=k, d=d, f=f, T=T, S_tot=S, N=1, iters=1,
                  router_matmul=False, seed=d + T)
    print(f"[mid tile] E={E} S={S} d={d} f={f} T={T}", flush=True)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)


# given slot offsets: row counts at the tile's edges, empty slots in front, between and behind, more slots than a
# workgroup has threads; binary64 on the stored inputs of every product.  A stored value is a 32-bit sum rounded to
# bf16: half of 2^-8 of itself, and the sum's own error, far below 2^-9 of the row's scale
@pytest.mark.parametrize("d,f,extra", [(72, 136, 0), (264, 192, 0), (128, 520, 300)])
def test_tile_edges(d, f, extra):
    rows = [0, 1, 63, 64, 65, 0, 127, 128, 129, 191, 193, 257, 10, 300, 300] + [0] * extra + [5, 0]
    S, T = len(rows), sum(rows)
    c = wl.scaled(wl.get_config("c2"), E=4, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    st = Hn.State(c, shard=0)
    g = torch.Generator(device="cuda").manual_seed(d)
    for t, std in ((st.Xp, 1.0), (st.dYp, 1.0), (st.W1s, d ** -0.5), (st.W2s, f ** -0.5)):
        t.normal_(0.0, std, generator=g)
    st.slot_offsets.copy_(torch.tensor([0] + rows).cumsum(0))
    st.first_slot.copy_(torch.tensor([0, 3, 7, 9, S]))
    print(f"[mid edges] d={d} f={f} S={S}", flush=True)
    symi.symi_expert_fwd(st.ctx, st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws)
    symi.symi_expert_bwd(st.ctx, st.dYp, st.Xp, st.UV, st.H, st.slot_offsets, st.first_slot, st.W1s, st.W2s, st.dXp,
                         st.dW1, st.dW2, st.ws)
    off = [0]
    for n in rows:
        off.append(off[-1] + n)

    def near(a, b):
        assert bool(((a - b).abs() <= b.abs() * 2 ** -8 + b.abs().max() * 2 ** -9).all())

    for q, n in enumerate(rows):
        if not n:
            continue
        s = slice(off[q], off[q + 1])
        W1, W2 = st.W1s[q].double(), st.W2s[q].double()
        uv, h = st.UV[s].double(), st.H[s].double()
        u, v = uv[:, :f], uv[:, f:]
        want = st.Xp[s].double() @ W1.T
        near(uv, want)
        near(h, torch.nn.functional.silu(want[:, :f]) * want[:, f:])
        near(st.Yp[s].double(), h @ W2.T)
        dh = st.dYp[s].double() @ W2
        sg = torch.sigmoid(u)
        duv = torch.cat([dh * v * sg * (1 + u * (1 - sg)), dh * u * sg], 1)
        # du, dv live in the workspace: the input gradient from them rounded to bf16, whose roundings add up like noise
        want = duv.bfloat16().double() @ W1
        got = st.dXp[s].double()
        assert float((got - want).norm() / want.norm()) < 2 ** -8
