"""The small fp32 products: dh and dW2, dX and dW1 in one launch each, with four and with eight wavefronts to a reduction and an odd
number of tiles in the last workgroup, rows found from the slot offsets.  The same bits as one launch for each product (a
context that times every launch), per class and per slot, and every value against binary64."""
import pytest
import torch

import paper_2504_19925_amd as symi
from tests.checks import launches
from tests.test_gpu_f32_split import expected

pytestmark = pytest.mark.gpu
NAMES = ("UV", "H", "Yp", "dXp", "dW1", "dW2", "sW1", "sW2")

CASES = {
    # rows of the slots, first slot of each class, d, f
    "one row": ([1], [0, 1], 8, 8),
    "eight share, no class empty": ([33, 1, 64, 31], [0, 1, 3, 4], 72, 136),
    "empty slots and classes": ([0, 0, 40, 0, 95, 0, 0, 7, 0], [0, 1, 4, 6, 9], 40, 264),
    "four share dh, eight dX": ([128] * 16, list(range(0, 17, 2)), 128, 256),
    "four share both, odd tile counts": ([97, 3, 130, 160, 61, 99, 128, 127, 33, 1, 5, 250, 290, 64, 90, 110], list(range(0, 17, 2)), 296, 104),
    "more slots than threads": ([0, 1, 0, 0, 2] * 52, list(range(0, 261, 52)), 24, 40),
}


def layer(rows, first, d, f, flags):
    E, S, A = len(first) - 1, len(rows), sum(rows)
    cfg = symi.SymiCfg.make(A, E, 1, d, f, S, 1, 0, "f32", 1)
    g = torch.Generator(device="cuda").manual_seed(A)
    r = lambda *n, std=1.0: torch.randn(*n, generator=g, device="cuda") * std
    z = lambda *n: torch.full(n, 7.0, device="cuda")
    off = torch.tensor([0] + rows, dtype=torch.int32).cumsum(0).to(torch.int32)
    s = dict(ctx=symi.symi_create(cfg, flags), Xp=r(A, d), dYp=r(A, d), W1=r(S, 2 * f, d, std=d ** -0.5), W2=r(S, d, f, std=f ** -0.5),
             UV=z(A, 2 * f), H=z(A, f), Yp=z(A, d), dXp=z(A, d), dW1=z(E, 2 * f, d), dW2=z(E, d, f), sW1=z(S, 2 * f, d),
             sW2=z(S, d, f), off=off.cuda(), first=torch.tensor(first, dtype=torch.int32, device="cuda"),
             ws=torch.full((symi.symi_workspace_bytes(cfg),), 0xFF, dtype=torch.uint8, device="cuda"), rows=rows, offs=off.tolist())
    symi.symi_expert_fwd(s["ctx"], s["Xp"], s["off"], s["W1"], s["W2"], s["UV"], s["H"], s["Yp"], s["ws"])
    b = (s["ctx"], s["dYp"], s["Xp"], s["UV"], s["H"], s["off"], s["first"], s["W1"], s["W2"], s["dXp"])
    symi.symi_expert_bwd(*b, s["dW1"], s["dW2"], s["ws"])
    symi.symi_expert_bwd_slots(*b, s["sW1"], s["sW2"], s["ws"])
    return s


@pytest.mark.parametrize("name", list(CASES))
def test_pairs(name):
    rows, first, d, f = CASES[name]
    print(f"[f32 pairs {name}] rows {sum(rows)} in {len(rows)} slots d={d} f={f}", flush=True)
    s = layer(rows, first, d, f, 0)
    one = layer(rows, first, d, f, symi.CTX_TIMING)
    # no table where all products of a call are small; the weight gradients of 260 single slots are not
    assert launches(one["ctx"], "tile_map") == (1 if len(rows) == 260 else 0)
    want = expected(s)
    for n in NAMES:
        assert torch.equal(s[n], one[n]), n
        # 32-bit sums of up to 2f terms or a class's rows, each partial sum rounded once: 2^-24 sqrt(K / 16) at most
        g, w = s[n].double(), want[n]
        assert float((g - w).norm()) <= 4e-7 * float(w.norm()), (n, float((g - w).norm() / w.norm()))
