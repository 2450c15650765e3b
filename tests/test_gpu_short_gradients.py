"""The 128 x 256 tile of weight gradients with short reductions: tile edges in rows and columns, reductions of a row to several
steps with a remainder, empty and skipped classes, per class and per slot, against binary64; and on both sides of the line in mean rows the
same bits as the large tile gives the same class."""
import pytest
import torch

import paper_2504_19925_amd as symi

pytestmark = pytest.mark.gpu


def layer(rows, first, d, f, seed, T=None):
    """dUV comes from the layer's own backward: u = v = 0 makes it 0, so the saved u, v are drawn too."""
    E, S, A = len(first) - 1, len(rows), sum(rows)
    cfg = symi.SymiCfg.make(T or A, E, 1, d, f, S, 1, 0, "bf16", 1)
    n = T or A
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *m, std=1.0: (torch.randn(*m, generator=g, device="cuda") * std).bfloat16()
    off = torch.tensor([0] + rows, dtype=torch.int32).cumsum(0).to(torch.int32)
    s = dict(ctx=symi.symi_create(cfg), Xp=r(n, d), dYp=r(n, d), W1=r(S, 2 * f, d, std=d ** -0.5), W2=r(S, d, f, std=f ** -0.5),
             UV=r(n, 2 * f), H=r(n, f), dXp=r(n, d), off=off.cuda(), first=torch.tensor(first, dtype=torch.int32, device="cuda"),
             ws=torch.empty(symi.symi_workspace_bytes(cfg), dtype=torch.uint8, device="cuda"), offs=off.tolist())
    return s


def backward(s, E, d, f, fn):
    dW1, dW2 = torch.full((E, 2 * f, d), 7.0, device="cuda"), torch.full((E, d, f), 7.0, device="cuda")
    fn(s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"], dW1, dW2, s["ws"])
    return dW1, dW2


SHAPES = {
    "one row": ([1], [0, 1], 8, 8),
    "a step, two, three and a remainder": ([31, 32, 33, 64, 65, 96, 97, 95], list(range(9)), 136, 264),
    "tile edges": ([20, 0, 61, 7], [0, 2, 3, 4], 256, 128),
    "one column piece over": ([50, 3, 0, 77], [0, 1, 2, 3, 4], 264, 520),
    "64 rows in the last tile": ([40] * 8, [0, 2, 4, 6, 8], 192, 328),
    "whole rounds per XCD": ([17, 80, 5, 33], [0, 1, 2, 3, 4], 1024, 2048),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_against_binary64(name):
    rows, first, d, f = SHAPES[name]
    E, S = len(first) - 1, len(rows)
    print(f"[short gradients {name}] rows {rows} d={d} f={f}", flush=True)
    s = layer(rows, first, d, f, 1)
    want1, want2 = torch.zeros(S, 2 * f, d, device="cuda", dtype=torch.float64), torch.zeros(S, d, f, device="cuda", dtype=torch.float64)
    for q, n in enumerate(rows):
        r = slice(s["offs"][q], s["offs"][q] + n)
        u, v, dY = s["UV"][r, :f].double(), s["UV"][r, f:].double(), s["dYp"][r].double()
        dh, sg = dY @ s["W2"][q].double(), torch.sigmoid(u)
        duv = torch.cat([dh * v * sg * (1 + u * (1 - sg)), dh * u * sg], 1).bfloat16().double()
        want1[q], want2[q] = duv.T @ s["Xp"][r].double(), dY.T @ s["H"][r].double()
    got = {"slots": backward(s, S, d, f, symi.symi_expert_bwd_slots), "classes": backward(s, E, d, f, symi.symi_expert_bwd),
           "active": backward(s, E, d, f, symi.symi_expert_bwd_active)}
    for kind, (g1, g2) in got.items():
        w1, w2 = want1, want2
        if kind != "slots":
            w1, w2 = (torch.stack([w[first[e]:first[e + 1]].sum(0) for e in range(E)]) for w in (w1, w2))
        for e in range(w1.shape[0]):
            if kind == "active" and not sum(rows[first[e]:first[e + 1]]):
                assert bool((g1[e] == 7).all()) and bool((g2[e] == 7).all())    # not written
                continue
            # dW2: 32-bit sums of exact products.  dW1: du, dv rounded to bf16 by the kernel and by the oracle, from
            # fp32 and from binary64: apart by one rounding, 2^-8, where the two sit on different sides of a tie
            assert float((g2[e].double() - w2[e]).abs().max()) <= 2.0 ** -18 * float(w2[e].abs().max()) if w2[e].any() else not g2[e].any(), (kind, e)
            assert float((g1[e].double() - w1[e]).norm()) <= 2.0 ** -9 * float(w1[e].norm()), (kind, e)


def test_same_bits_as_the_large_tile():
    """A class of 96 rows alone (short), and in front of a class of 1500 (mean beyond the line, the large tile)."""
    d, f = 264, 392
    s = layer([96], [0, 1], d, f, 2)
    short = backward(s, 1, d, f, symi.symi_expert_bwd)
    big = layer([96, 1500], [0, 1, 2], d, f, 3)
    for n in ("Xp", "dYp", "UV", "H"):
        big[n][:96] = s[n]
    big["W1"][0], big["W2"][0] = s["W1"][0], s["W2"][0]
    large = backward(big, 2, d, f, symi.symi_expert_bwd)
    assert torch.equal(short[0][0], large[0][0]) and torch.equal(short[1][0], large[1][0])


@pytest.mark.parametrize("fn", ["symi_expert_bwd", "symi_expert_bwd_slots"])
def test_same_bits_on_both_sides_of_the_gradients_line(fn):
    """65 classes just below 1 GiB of gradients, 66 just above it, the large tile where the helper stream runs."""
    d, f = 336, 4096
    rows = [1 + 7 * q % 40 for q in range(65)]
    n = sum(rows)
    s = layer(rows, list(range(66)), d, f, 4)
    below = backward(s, 65, d, f, getattr(symi, fn))
    big = layer(rows + [5], list(range(67)), d, f, 5)
    for name in ("Xp", "dYp", "UV", "H"):
        big[name][:n] = s[name]
    big["W1"][:65], big["W2"][:65] = s["W1"], s["W2"]
    above = backward(big, 66, d, f, getattr(symi, fn))
    assert torch.equal(below[0], above[0][:65]) and torch.equal(below[1], above[1][:65])
