"""The fp32 expert products that split every value into three bf16 ones: tile, step and class edges against binary64 with
the bound of 32-bit sums, and the values that three bf16 ones do not hold (infinities, NaN, the ends of the range), which
have to give what 32-bit products give."""
import pytest
import torch

import paper_2504_19925_amd as symi

pytestmark = pytest.mark.gpu
DEV = "cuda"


def layer(rows, first, d, f, seed=0):
    """A layer whose slots hold the given rows; class c has the slots first[c] .. first[c + 1]."""
    E, S, A = len(first) - 1, len(rows), sum(rows)
    cfg = symi.SymiCfg.make(A, E, 1, d, f, S, 1, 0, "f32", 1)
    g = torch.Generator(device=DEV).manual_seed(seed)
    r = lambda *n, std=1.0: torch.randn(*n, generator=g, device=DEV) * std
    z = lambda *n: torch.full(n, 7.0, device=DEV)
    off = torch.tensor([0] + rows, dtype=torch.int32).cumsum(0).to(torch.int32)
    s = dict(ctx=symi.symi_create(cfg), Xp=r(A, d), dYp=r(A, d), W1=r(S, 2 * f, d, std=d ** -0.5), W2=r(S, d, f, std=f ** -0.5),
             UV=z(A, 2 * f), H=z(A, f), Yp=z(A, d), dXp=z(A, d), dW1=z(E, 2 * f, d), dW2=z(E, d, f),
             sW1=z(S, 2 * f, d), sW2=z(S, d, f), off=off.to(DEV), first=torch.tensor(first, dtype=torch.int32, device=DEV),
             ws=torch.empty(symi.symi_workspace_bytes(cfg), dtype=torch.uint8, device=DEV))
    s["rows"], s["offs"] = rows, off.tolist()
    return s


def run(s):
    symi.symi_expert_fwd(s["ctx"], s["Xp"], s["off"], s["W1"], s["W2"], s["UV"], s["H"], s["Yp"], s["ws"])
    b = (s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"])
    symi.symi_expert_bwd(*b, s["dW1"], s["dW2"], s["ws"])
    symi.symi_expert_bwd_slots(*b, s["sW1"], s["sW2"], s["ws"])


def expected(s):
    """The six products in binary64, slot by slot, from the fp32 values that the forward stored."""
    f = s["W2"].shape[2]
    first = s["first"].tolist()
    out = {n: torch.zeros_like(s[n], dtype=torch.float64) for n in ("UV", "H", "Yp", "dXp", "dW1", "dW2", "sW1", "sW2")}
    for q, n in enumerate(s["rows"]):
        r = slice(s["offs"][q], s["offs"][q] + n)
        W1, W2, X, dY = (t.double() for t in (s["W1"][q], s["W2"][q], s["Xp"][r], s["dYp"][r]))
        out["UV"][r] = X @ W1.T
        uv = s["UV"][r].double()
        u, v = uv[:, :f], uv[:, f:]
        sg = torch.sigmoid(u)
        out["H"][r] = u * sg * v
        out["Yp"][r] = s["H"][r].double() @ W2.T
        dh = dY @ W2
        duv = torch.cat([dh * v * sg * (1 + u * (1 - sg)), dh * u * sg], 1)
        out["dXp"][r] = duv @ W1
        out["sW1"][q], out["sW2"][q] = duv.T @ X, dY.T @ s["H"][r].double()
    for e in range(len(first) - 1):
        out["dW1"][e], out["dW2"][e] = out["sW1"][first[e]:first[e + 1]].sum(0), out["sW2"][first[e]:first[e + 1]].sum(0)
    return out


CASES = {
    # rows of the slots, first slot of each class, d, f
    "tile edges": ([1, 63, 64, 65, 127, 128, 129, 0, 200, 31, 33, 500] * 2, list(range(25)), 328, 264),
    "one step": ([64, 70] * 40, list(range(0, 81, 2)), 24, 1032),
    "step and a piece": ([200] * 30, list(range(0, 31, 3)), 40, 520),
    "column of 8": ([90] * 24, list(range(25)), 136, 584),
    "most rows in one class": ([3000, 1, 0, 40, 8, 0, 17, 300], [0, 1, 2, 3, 5, 8], 520, 328),
    "many small slots": ([17, 30, 5, 64] * 32, list(range(0, 129, 4)), 264, 328),
}


@pytest.mark.parametrize("name", list(CASES))
def test_against_binary64(name):
    rows, first, d, f = CASES[name]
    print(f"[f32 split {name}] rows {sum(rows)} in {len(rows)} slots d={d} f={f}", flush=True)
    s = layer(rows, first, d, f)
    run(s)
    want = expected(s)
    for n, w in want.items():
        g = s[n].double()
        # A sum of K rounded products of which each partial sum is rounded once: relative 2-norm within 2^-24 sqrt(K / 16),
        # K up to 2f and the rows of a class; the gradients go through one stored fp32 value more.  Measured 0.6e-7 - 2.3e-7.
        assert float((g - w).norm()) <= 4e-7 * float(w.norm()), (n, float((g - w).norm() / w.norm()))
        assert float((g - w).abs().max()) <= 2e-5 * float(w.pow(2).mean().sqrt()) + 2.0 ** -20 * float(w.abs().max()), n


def test_ends_of_the_range():
    """Infinities, NaN, values that bf16 rounds to infinity and values whose third part is subnormal: the same non-finite
    results as 32-bit products, and the finite ones as exact."""
    d, f = 264, 328
    rows, first = [100] * 24, list(range(25))
    s = layer(rows, first, d, f, seed=3)
    X, W1 = s["Xp"], s["W1"]
    X[5, 7] = float("inf")
    X[105, 3], X[106, 3] = float("nan"), float("-inf")
    X[205, 9] = 3.4e38                              # rounds to infinity in bf16
    W1[2, :, 9] *= 1e-3
    X[300:400] *= 2.0 ** -115                       # a slot of small values: u, v near 2^-115
    X[400:500] *= 2.0 ** -128                       # subnormal ones
    W1[5] *= 2.0 ** 100                             # small values against large ones
    X[500:600] *= 2.0 ** -118
    run(s)
    for q in range(7):
        r = slice(100 * q, 100 * q + 100)
        want = X[r].double() @ W1[q].double().T
        got = s["UV"][r].double()
        odd = ~torch.isfinite(want) | (want.abs() > 3.4e38)
        assert torch.equal(torch.isfinite(got), ~odd), q
        # an infinity keeps its sign; NaN where infinities meet or one was there
        assert torch.equal(torch.isnan(got), torch.isnan(want)), q
        assert torch.equal(got[torch.isinf(got)] > 0, want[torch.isinf(got)] > 0), q
        ok = torch.isfinite(want).all(1) & (want.abs() < 1e38).all(1)
        a, b = got[ok], want[ok]
        # 2^-149 is the spacing of subnormal numbers, to which each of up to d partial sums is rounded
        assert float((a - b).norm()) <= 4e-7 * float(b.norm()) + 2.0 ** -149 * (a.numel() * d) ** 0.5, (q, float((a - b).norm() / b.norm()))
    # the other slots are as without them
    for q in (7, 12, 23):
        r = slice(100 * q, 100 * q + 100)
        want = X[r].double() @ W1[q].double().T
        assert float((s["UV"][r].double() - want).norm()) <= 4e-7 * float(want.norm())
