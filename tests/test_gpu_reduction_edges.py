"""GPU parity of the bf16 expert products where their pipelines can go wrong: reductions of one to ten
64-deep steps with and without a partial last step (the large tile: two stages of one operand, three of the
other; the smaller tiles: two or three of both), classes of few rows, and slots on both sides of the half-height tile's
128 rows."""
import pytest
import torch

import paper_2504_19925_amd as symi
import workloads as wl
import harness as Hn
from tests.checks import bf16_tiles, check_iteration, launches, products_against_binary64

pytestmark = pytest.mark.gpu


# on the 128 x 128 tile; the weight gradients, here and below, on the large one
@pytest.mark.parametrize("d,f,T", [(8, 8, 40), (64, 56, 90), (72, 64, 128), (120, 136, 129), (128, 192, 250),
                                   (192, 200, 258), (256, 248, 380), (264, 320, 390), (328, 384, 515), (448, 440, 700)])
def test_steps_of_the_reduction(d, f, T):
    assert bf16_tiles(T, 3, 2, 4, d, f) == ("mmmm" if T > 64 else "ffmm")
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=3, k=2, d=d, f=f, T=T, S_tot=4, N=1, iters=1,
                  router_matmul=False, seed=d + T)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)


# at most 32 rows per slot on average: the forward products take their small tile.  One row, slots of
# one, several and (a uniform placement under skewed popularity) more than four 64-row parts, reductions of
# one to four steps with and without a partial one, column remainders, and the first size beyond the rule
@pytest.mark.parametrize("E,k,S,d,f,T", [(1, 1, 1, 8, 8, 1), (4, 2, 6, 72, 136, 33), (16, 2, 24, 128, 256, 64),
                                         (24, 1, 24, 200, 64, 768), (24, 1, 24, 200, 64, 769), (64, 4, 80, 136, 328, 640),
                                         (8, 1, 64, 264, 72, 2048)])
def test_few_rows_per_slot(E, k, S, d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=E, k=k, d=d, f=f, T=T, S_tot=S, N=1, iters=1,
                  router_matmul=False, seed=3 * T + d)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)


# A rank whose experts got nothing brings slot offsets that are all zero with a positive token count: no
# row exists, so nothing is computed and nothing written, whatever an earlier call (here one with every
# row in the first slot) left in the workspace
@pytest.mark.parametrize("dtype,T,S", [("bf16", 192, 24), ("bf16", 200, 220), ("bf16", 400, 6), ("f32", 192, 24), ("f32", 9000, 6)])
def test_no_slot_has_rows(dtype, T, S):
    c = wl.scaled(wl.get_config("c2"), dtype=dtype, E=4, k=2, d=136, f=520, T=T, S_tot=S, N=1, iters=1,
                  router_matmul=False)
    st = Hn.State(c, shard=0)
    st.Xp.normal_()
    st.W1s.normal_()
    st.W2s.normal_()

    def forward(kept):
        st.slot_offsets.fill_(kept)
        st.slot_offsets[0] = 0
        for t in (st.UV, st.H, st.Yp):
            t.fill_(3.0)
        symi.symi_expert_fwd(st.ctx, st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws)
        return [bool((t == 3.0).all()) for t in (st.UV, st.H, st.Yp)]

    print(f"[no rows] {dtype} T={T} S={S}", flush=True)
    assert forward(c.A) == [False] * 3
    assert forward(0) == [True] * 3


# Rows are few per slot on average but sit in some of the slots: the 64-row tiles of the small-batch forward
# products at their edges, 25 of them (three rounds of 8 and one more) in 1, 2, 3, 6, 8, 16, 27 and 28 column tiles,
# counted by the workgroups and, beyond 8 workgroups per compute unit, from a table, against binary64.  A stored value is a 32-bit sum rounded to bf16 (half of
# 2^-8), h of the unrounded u and v; the second product is compared on the stored h
@pytest.mark.parametrize("d,f", [(8, 72), (264, 328), (1024, 1000), (264, 1728), (264, 1792)])
def test_a_small_batch_in_a_few_slots(d, f):
    rows = [0, 1, 63, 64, 65, 0, 127, 128, 129, 191, 193, 257, 10] + [0] * 35
    S, T = len(rows), sum(rows)
    assert T <= 32 * S
    c = wl.scaled(wl.get_config("c2"), E=4, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    st = Hn.State(c, shard=0, flags=symi.CTX_TIMING)
    g = torch.Generator(device="cuda").manual_seed(d)
    for t, std in ((st.Xp, 1.0), (st.W1s, d ** -0.5), (st.W2s, f ** -0.5)):
        t.normal_(0.0, std, generator=g)
    st.slot_offsets.copy_(torch.tensor([0] + rows).cumsum(0))
    print(f"[few slots] d={d} f={f}", flush=True)
    symi.symi_expert_fwd(st.ctx, st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert launches(st.ctx, "tile_map") == int((T // 64 + S) * (-(-f // 64) - (-d // 128)) > 8 * cus)
    slot = torch.repeat_interleave(torch.arange(S), torch.tensor(rows))
    X, W1, W2, UV, H, Yp = (t.cpu().double() for t in (st.Xp, st.W1s, st.W2s, st.UV, st.H, st.Yp))
    for s in slot.unique().tolist():
        at = slot == s
        uv = X[at] @ W1[s].T
        h = torch.nn.functional.silu(uv[:, :f]) * uv[:, f:]
        for got, want in ((UV[at], uv), (H[at], h), (Yp[at], H[at] @ W2[s].T)):
            assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all(), (s, rows[s])


# Indices beyond the end of a reduction are zeros in both operands, whatever lies behind them in memory: the rows of the
# next class (weight gradients), the next row of the activations or of the weights (the other products).  NaN in
# every second class must stay there.  1 to 5 steps, full and ragged, an odd and an even number of them
@pytest.mark.parametrize("d,f,rows", [(8, 72, 1), (64, 128, 64), (72, 64, 65), (136, 200, 191), (192, 264, 193), (320, 136, 300)])
def test_nothing_beyond_the_reduction(d, f, rows):
    E = 4
    c = wl.scaled(wl.get_config("c2"), E=E, k=1, d=d, f=f, T=E * rows, S_tot=E, N=1, iters=1, router_matmul=False)
    st = Hn.State(c, shard=0)
    g = torch.Generator(device="cuda").manual_seed(d + rows)
    for t, std in ((st.Xp, 1.0), (st.dYp, 1.0), (st.W1s, d ** -0.5), (st.W2s, f ** -0.5)):
        t.normal_(0.0, std, generator=g)
    st.slot_offsets.copy_(torch.arange(E + 1) * rows)
    st.first_slot.copy_(torch.arange(E + 1))

    def run():
        symi.symi_expert_fwd(st.ctx, st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws)
        symi.symi_expert_bwd(st.ctx, st.dYp, st.Xp, st.UV, st.H, st.slot_offsets, st.first_slot, st.W1s, st.W2s, st.dXp,
                             st.dW1, st.dW2, st.ws)
        return [t.view(E, -1).clone() for t in (st.UV, st.H, st.Yp, st.dXp, st.dW1, st.dW2)]

    print(f"[beyond K] d={d} f={f} rows={rows}", flush=True)
    clean = run()
    for e in (1, 3):
        st.Xp[e * rows:(e + 1) * rows] = float("nan")
        st.dYp[e * rows:(e + 1) * rows] = float("nan")
        st.W1s[e], st.W2s[e] = float("nan"), float("nan")
    for a, b in zip(clean, run()):
        assert torch.isfinite(a).all()
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
        assert torch.isnan(b[1]).all() and torch.isnan(b[3]).all()


# The same on the large tile, which takes short reductions only with many rows and wide outputs: one to ten steps of the first
# forward product and the hidden gradient (d), then of the second forward product (f) and the input gradient (2 f).
# Slots of every height around 64, 128 and 256 rows, and empty ones; the rest of the rows in the last five.  All four products
# on the large tile, every output against binary64; then NaN in every second slot's operands, which must stay there
@pytest.mark.parametrize("d,f,T", [(40, 8200, 27000), (64, 4104, 33000), (72, 4104, 29000), (128, 2056, 32000), (136, 2056, 30000),
                                   (200, 1544, 27000), (256, 1544, 22000), (264, 1544, 22000), (328, 1032, 24000),
                                   (400, 1032, 20000), (456, 1032, 18000), (512, 1032, 17000), (520, 1032, 17000), (584, 1032, 15000),
                                   (8200, 40, 21000), (4104, 64, 26000), (4104, 72, 24000), (2056, 136, 24000), (1544, 200, 29000),
                                   (1544, 256, 23000), (1032, 328, 27000), (1032, 520, 17000)])
def test_steps_of_the_large_tile(d, f, T):
    rows = [0, 1, 63, 64, 65, 127, 128, 129, 0, 191, 255, 256, 257, 0, 511, 513]
    left = T - sum(rows)
    rows += [left // 5 + i - 2 for i in range(5)]
    rows[-1] += T - sum(rows)
    S = len(rows)
    assert bf16_tiles(T, S, 1, S, d, f) == "LLLL"
    c = wl.scaled(wl.get_config("c2"), E=S, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    st = Hn.State(c, shard=0)
    print(f"[large tile] d={d} f={f} T={T}", flush=True)
    products_against_binary64(st, rows, list(range(S + 1)), d + f)
    if min(d, f) % 64 == 0 and min(d, f) > 64:
        return
    outs = (st.UV, st.H, st.Yp, st.dXp)
    clean, grads = [t.clone() for t in outs], [st.dW1.clone(), st.dW2.clone()]
    off = torch.tensor([0] + rows).cumsum(0).tolist()
    for q in range(1, S, 2):
        for t in (st.Xp[off[q]:off[q + 1]], st.dYp[off[q]:off[q + 1]], st.W1s[q], st.W2s[q]):
            t.fill_(float("nan"))
    symi.symi_expert_fwd(st.ctx, st.Xp, st.slot_offsets, st.W1s, st.W2s, st.UV, st.H, st.Yp, st.ws)
    symi.symi_expert_bwd(st.ctx, st.dYp, st.Xp, st.UV, st.H, st.slot_offsets, st.first_slot, st.W1s, st.W2s, st.dXp,
                         st.dW1, st.dW2, st.ws)
    for q in range(S):
        for a, b in zip(clean, outs):
            a, b = a[off[q]:off[q + 1]], b[off[q]:off[q + 1]]
            assert torch.isnan(b).all() if q & 1 else torch.equal(a, b), q
        for a, b in zip(grads, (st.dW1[q], st.dW2[q])):
            assert torch.isnan(b).all() if q & 1 and rows[q] else torch.equal(a[q], b), q
