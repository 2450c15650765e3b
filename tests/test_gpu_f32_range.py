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
