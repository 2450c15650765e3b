"""The hidden gradient du = dh v s (1 + u (1 - s)), dv = dh u s, s = sigmoid(u), where s is near the smallest normal number:
dh s on its own would be subnormal and lose its bits, dh v does not.  The permuted tokens are the unit vectors, so
the W1 gradient holds du and dv themselves; dh is a product of two bf16 numbers, exact in 32 bits."""
import pytest
import torch

import paper_2504_19925_amd as symi
import workloads as wl
import harness as Hn

pytestmark = pytest.mark.gpu


# the 128 x 128 tile (few short tiles) and the 256 x 256 one (A > 128 S and 9 x 65 tiles of K = 1024)
@pytest.mark.parametrize("d,f", [(64, 72), (1024, 8256)])
def test_small_sigmoid(d, f):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=1, k=1, d=d, f=f, T=d, S_tot=1, N=1, iters=1, router_matmul=False)
    print(f"[hidden gradient] d={d} f={f}", flush=True)
    st = Hn.State(c, shard=0)
    g = torch.Generator(device="cuda").manual_seed(d)
    eye = torch.eye(d, dtype=torch.bfloat16, device="cuda")
    st.Xp.copy_(eye)
    st.dYp.copy_(eye * 2.0 ** -20)                                   # dh[r, j] = 2^-20 W2[r, j]
    st.W2s.uniform_(1.0, 2.0, generator=g)
    st.W1s.normal_(generator=g)
    st.H.zero_()
    st.UV[:, :f].uniform_(-87.0, -84.0, generator=g)                 # s from 1.6e-38 to 3e-37
    st.UV[:, f:].uniform_(2.0 ** 49, 2.0 ** 50, generator=g)
    st.slot_offsets.copy_(torch.tensor([0, d]))
    st.first_slot.copy_(torch.tensor([0, 1]))
    symi.symi_expert_bwd(st.ctx, st.dYp, st.Xp, st.UV, st.H, st.slot_offsets, st.first_slot, st.W1s, st.W2s, st.dXp,
                         st.dW1, st.dW2, st.ws)
    dh = st.dYp.double().diagonal()[:, None] * st.W2s[0].double()
    u, v = st.UV[:, :f].double(), st.UV[:, f:].double()
    s = torch.sigmoid(u)
    got = st.dW1[0, :f].T.double()
    want = dh * v * s * (1 + u * (1 - s))
    # rounding to bf16, 2^-8, and the exponential of an argument of 126 in 32 bits, below 2^-14
    assert float(((got - want).abs() / want.abs()).max()) <= 2.0 ** -8 + 2.0 ** -14
