"""fp32 expert products at the ends of the fp32 range, where the sums of bf16 parts give way to the fp32 instruction."""
import pytest
import torch

import paper_2504_19925_amd as symi
from tests.test_gpu_f32_split import expected, layer, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [1.0, 2.0 ** 41, float("inf")])
def test_active_leaves_classes_without_rows(value):
    """Some seven tiles to a workgroup, those of the classes without rows behind the others: none of them is written, whatever
    the values of the others are."""
    rows = [64] * 24 + [0] * 40
    s = layer(rows, list(range(65)), 264, 520, seed=5)
    run(s)
    s["Xp"][7::64, 5] = value
    s["dYp"][9::64, 3] = value
    s["dW1"].fill_(7.0)
    s["dW2"].fill_(7.0)
    symi.symi_expert_bwd_active(s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"],
                                s["dW1"], s["dW2"], s["ws"])
    for e in range(64):
        kept = bool((s["dW1"][e] == 7.0).all()) and bool((s["dW2"][e] == 7.0).all())
        assert kept == (e >= 24), e


def close(got, want, K, what):
    """Finite results within the bound of 32-bit sums of K products: 4e-7 of the 2-norm (test_gpu_f32_split), and 2^-149, the spacing of
    subnormal numbers, for each of up to K partial sums."""
    got, err = got.double(), float((got.double() - want).norm())
    assert err <= 4e-7 * float(want.norm()) + 2.0 ** -149 * (got.numel() * K) ** 0.5, (what, err / max(float(want.norm()), 1e-300))


def test_values_without_bf16_parts():
    """Values that round to 0 in bf16 (2^-136) against large ones: the sums are normal fp32 numbers in every product, though all
    bf16 parts of one operand vanish.  Each slot is a class of its own, so nothing else is in its tiles."""
    d, f, n, tiny, large = 264, 328, 100, 2.0 ** -136, 2.0 ** 30
    s = layer([n] * 24, list(range(25)), d, f, seed=7)
    r = [slice(n * q, n * q + n) for q in range(24)]
    s["Xp"][r[0]] *= tiny           # u, v near 2^-106
    s["W1"][0] *= large
    s["Xp"][r[1]] *= 2.0 ** -68     # h near 2^-137
    s["W2"][1] *= large
    symi.symi_expert_fwd(s["ctx"], s["Xp"], s["off"], s["W1"], s["W2"], s["UV"], s["H"], s["Yp"], s["ws"])
    want = expected(s)
    for q in range(24):
        close(s["UV"][r[q]], want["UV"][r[q]], d, ("UV", q))
        close(s["Yp"][r[q]], want["Yp"][r[q]], f, ("Yp", q))
    assert float(s["UV"][r[0]].abs().max()) > 2.0 ** -110 and float(s["Yp"][r[1]].abs().max()) > 2.0 ** -112
    s["dYp"][r[2]] *= tiny          # dh near 2^-106
    s["W2"][2] *= large
    s["dYp"][r[3]] *= tiny          # du, dv near 2^-136
    s["W1"][3] *= large
    s["dYp"][r[4]] *= tiny
    s["Xp"][r[4]] *= large
    s["dYp"][r[5]] *= tiny
    s["H"][r[5]] *= large
    b = (s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"])
    want = expected(s)
    for call, names in ((symi.symi_expert_bwd, ("dW1", "dW2")), (symi.symi_expert_bwd_active, ("dW1", "dW2")),
                        (symi.symi_expert_bwd_slots, ("sW1", "sW2"))):
        for t in ("dXp", *names):
            s[t].fill_(7.0)
        call(*b, s[names[0]], s[names[1]], s["ws"])
        for q in range(24):
            # du, dv are stored in fp32 and may be subnormal there, as may be the sums: 2^-149 of each, times the other operand
            slack = 2.0 ** -149 * max(1.0, float(s["W1"][q].abs().max())) * (2 * f * n * d) ** 0.5
            assert float((s["dXp"][r[q]].double() - want["dXp"][r[q]]).norm()) <= 4e-7 * float(want["dXp"][r[q]].norm()) + slack, q
            slack = 2.0 ** -149 * max(1.0, float(s["Xp"][r[q]].abs().max())) * (2 * f * n * d) ** 0.5
            assert float((s[names[0]][q].double() - want[names[0]][q]).norm()) <= 4e-7 * float(want[names[0]][q].norm()) + slack, q
            close(s[names[1]][q], want[names[1]][q], n, (names[1], q))
        assert min(float(t.abs().max()) for t in (s["dXp"][r[2]], s["dXp"][r[3]], s[names[0]][4], s[names[1]][5])) > 2.0 ** -112


def test_classes_with_few_rows():
    """Weight gradients of one and two rows among classes of hundreds: as exact as products rounded once each, class by class (in
    the norm of a whole output they would not be seen)."""
    d, f = 264, 328
    rows = [1, 2, 200, 1, 3, 2, 0, 500] * 8
    s = layer(rows, list(range(65)), d, f, seed=11)
    s["Xp"][:, 0] = 1.0     # the first column of dW1 is the sum of du, dv
    run(s)
    b = (s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"])
    aW1, aW2 = torch.zeros_like(s["dW1"]), torch.zeros_like(s["dW2"])
    symi.symi_expert_bwd_active(*b, aW1, aW2, s["ws"])
    for gW1, gW2 in ((s["dW1"], s["dW2"]), (s["sW1"], s["sW2"]), (aW1, aW2)):
        for e, n in enumerate(rows):
            r = slice(s["offs"][e], s["offs"][e] + n)
            dY, H, X = (s[t][r].double() for t in ("dYp", "H", "Xp"))
            # n products and n - 1 additions of them, each rounded to 2^-24 of at most the sum of their magnitudes
            err = (gW2[e].double() - dY.T @ H).abs()
            assert bool((err <= n * 2.0 ** -24 * (dY.abs().T @ H.abs())).all()), (e, n)
            if n == 1:
                want = gW1[e].double()[:, :1] @ X
                assert bool(((gW1[e].double() - want).abs() <= 2.0 ** -24 * want.abs()).all()), e


def out_of_range(s, r):
    """Infinities, NaN and values beyond what three bf16 parts hold, one kind to a slot: those of the forward in place, those of
    the backward by the returned function."""
    s["Xp"][r[1]][5, 7] = float("inf")
    s["Xp"][r[2]][6, 3] = float("nan")
    s["W1"][3][9, 11] = float("-inf")
    s["W2"][4][5, 7] = float("inf")
    s["W2"][5][2] = 1e33
    s["Xp"][r[6]][70, 100] = 2e33
    s["W1"][6] *= 1e-20

    def later():
        s["dYp"][r[8]][3, 3] = float("inf")
        s["dYp"][r[9]] *= 1e33
        s["H"][r[10]][12, 9] = float("nan")
        s["H"][r[11]] *= 1e33
        s["UV"][r[13]][1, 4] = float("inf")
        s["UV"][r[14]][60, -3] = float("-inf")
        s["Xp"][r[15]] *= 1e33
        s["W2"][16][3, 4] = float("nan")
        s["W1"][17][:, 5] = 1e33
    return later


def same(got, want, size, what):
    """The same infinities and NaN, and finite results to 2e-5 of `size`, the sum of the magnitudes (32-bit sums of up to 1040 products,
    rounded in turn, of values that are such sums themselves: 1040 2^-24 and less)."""
    got, want = got.double(), want.float().double()     # beyond fp32: infinite
    assert torch.equal(torch.isnan(got), torch.isnan(want)), what
    assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.equal(got[torch.isinf(got)], want[torch.isinf(want)]), what
    ok = torch.isfinite(want)
    assert bool(((got - want).abs()[ok] <= 2e-5 * size[ok] + 1e-37).all()), what


@pytest.mark.parametrize("d,f", [(264, 520), (328, 392)])
def test_every_product_out_of_range(d, f):
    """Six products, gradients per class, per slot and of the active classes, several tiles to a workgroup, remainders of rows and
    columns and classes without rows: what 32-bit products give, in the tiles that are computed once more and in the others."""
    rows = [100, 130, 64, 0, 77, 200] * 8
    rows[3], rows[9], rows[15] = 70, 90, 80
    first = [0, 1, 2, 3, 5, 8] + list(range(9, 49))
    s = layer(rows, first, d, f, seed=13)
    r = [slice(s["offs"][q], s["offs"][q + 1]) for q in range(48)]
    later = out_of_range(s, r)
    D, big = torch.float64, lambda t: t.double().abs().nan_to_num(0, 0, 0)
    symi.symi_expert_fwd(s["ctx"], s["Xp"], s["off"], s["W1"], s["W2"], s["UV"], s["H"], s["Yp"], s["ws"])
    for q in range(48):
        X, W1, W2, H = s["Xp"][r[q]], s["W1"][q], s["W2"][q], s["H"][r[q]]
        same(s["UV"][r[q]], X.to(D) @ W1.to(D).T, big(X) @ big(W1).T, ("UV", q))
        same(s["Yp"][r[q]], H.to(D) @ W2.to(D).T, big(H) @ big(W2).T, ("Yp", q))
    later()
    dX, mX = torch.zeros_like(s["dXp"], dtype=D), torch.zeros_like(s["dXp"], dtype=D)
    duv, mduv = torch.zeros_like(s["UV"], dtype=D), torch.zeros_like(s["UV"], dtype=D)
    for q in range(48):
        dY, W1, W2 = s["dYp"][r[q]], s["W1"][q], s["W2"][q]
        u, v = s["UV"][r[q]][:, :f], s["UV"][r[q]][:, f:]
        dh, mh, sg = (dY.to(D) @ W2.to(D)).float(), big(dY) @ big(W2), torch.sigmoid(u)
        duv[r[q]] = torch.cat([dh * v * sg * (1 + u * (1 - sg)), dh * u * sg], 1).to(D)
        mduv[r[q]] = torch.cat([mh * big(v * sg * (1 + u * (1 - sg))), mh * big(u * sg)], 1)
        dX[r[q]], mX[r[q]] = duv[r[q]] @ W1.to(D), mduv[r[q]] @ big(W1)
    b = (s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"])
    slots = [(q, q + 1) for q in range(48)]
    for call, n1, n2, groups in ((symi.symi_expert_bwd, "dW1", "dW2", list(zip(first, first[1:]))),
                                 (symi.symi_expert_bwd_active, "dW1", "dW2", list(zip(first, first[1:]))),
                                 (symi.symi_expert_bwd_slots, "sW1", "sW2", slots)):
        for t in ("dXp", n1, n2):
            s[t].fill_(7.0)
        call(*b, s[n1], s[n2], s["ws"])
        for q in range(48):
            same(s["dXp"][r[q]], dX[r[q]], mX[r[q]], ("dXp", call.__name__, q))
        for g, (q0, q1) in enumerate(groups):
            at = slice(s["offs"][q0], s["offs"][q1])
            if at.start == at.stop:
                kept = 7.0 if call is symi.symi_expert_bwd_active else 0.0
                assert bool((s[n1][g] == kept).all()) and bool((s[n2][g] == kept).all()), (call.__name__, g)
                continue
            X, H, dY = s["Xp"][at], s["H"][at], s["dYp"][at]
            same(s[n1][g], duv[at].T @ X.to(D), mduv[at].T @ big(X), (n1, call.__name__, g))
            same(s[n2][g], dY.to(D).T @ H.to(D), big(dY).T @ big(H), (n2, call.__name__, g))
