"""The gate network's backward where its launches change: one chunk of tokens, whose sums are the gradients, and two; the weight
gradient's workgroups beside those of dX and of the bias gradient; classes that are no multiple of 8 or of the four of a lane
group.  Against binary64, with a workspace that ends in a pattern nobody may write."""
import pytest
import torch

import paper_2504_19925_amd as symi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("T", [1, 127, 128, 129, 256, 257, 513, 1100])
@pytest.mark.parametrize("dtype,E,d", [("bf16", 8, 136), ("bf16", 128, 1032), ("bf16", 12, 264), ("bf16", 136, 72),
                                       ("f32", 8, 72), ("f32", 5, 64), ("f32", 30, 264)])
def test_against_binary64(dtype, E, d, T, bias):
    cfg = symi.SymiCfg.make(T, E, 1, d, 8, E, 1, 0, dtype, 1)
    ctx, dt, dev = symi.symi_create(cfg), cfg.torch_dtype, "cuda"
    g = torch.Generator(device=dev).manual_seed(T + E)
    r = lambda *n, std=1.0, t=torch.float32: (torch.randn(*n, generator=g, device=dev) * std).to(t)
    X, Wr, b, dX0, dl = r(T, d, t=dt), r(E, d, std=0.05, t=dt), r(E), r(T, d, t=dt), r(T, E, std=0.1)
    n = symi.symi_workspace_bytes(cfg)
    ws = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=dev)
    logits, dWr, db, dX = torch.full((T, E), 7.0, device=dev), torch.full((E, d), 7.0, device=dev), torch.full((E,), 7.0, device=dev), dX0.clone()
    symi.symi_router_fwd(ctx, X, Wr, b if bias else None, logits)
    symi.symi_router_bwd(ctx, X, Wr, dl, dWr, db if bias else None, dX, ws)
    assert bool((ws[n:] == 0xA5).all())
    Xd, Wd, dld = X.double(), Wr.double(), dl.double()
    # dlogits enter the bf16 products rounded to bf16 and dX is rounded to it: 2^-9 each, independent; fp32: sums of 32-bit products
    tol = 2.0 ** -8 if dtype == "bf16" else 4e-7
    for name, got, want, t in (("logits", logits, Xd @ Wd.T + (b.double() if bias else 0), 4e-7), ("dWr", dWr, dld.T @ Xd, tol),
                               ("dX", dX, dX0.double() + dld @ Wd, tol), ("db", db, dld.sum(0) if bias else torch.full_like(db, 7.0).double(), 4e-7)):
        err = float((got.double() - want).norm() / want.norm())
        assert err <= t, (name, err)
