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


def test_scores_beyond_the_threads_of_one_dimension():
    """2^21 tokens of 1024 classes in fp32: 2^32 threads, more than one dimension of a launch takes."""
    T, E, d = 1 << 21, 1024, 8
    ctx, dev = symi.symi_create(symi.SymiCfg.make(T, E, 1, d, 8, E, 1, 0, "f32", 1)), "cuda"
    X, Wr = torch.randn(T, d, device=dev), torch.randn(E, d, device=dev)
    logits = torch.full((T, E), 7.0, device=dev)
    symi.symi_router_fwd(ctx, X, Wr, None, logits)
    for t in (0, 1 << 19, T - 512):
        want = X[t:t + 512].double() @ Wr.double().T
        assert float((logits[t:t + 512].double() - want).norm() / want.norm()) <= 4e-7, t


def test_gradients_beyond_the_threads_of_one_dimension():
    """2^20 tokens of d = 2048, E = 256 in fp32: 2^32 threads and some; 2^31 elements of X."""
    T, E, d = 1 << 20, 256, 2048
    cfg = symi.SymiCfg.make(T, E, 1, d, 8, E, 1, 0, "f32", 1)
    ctx, dev = symi.symi_create(cfg), "cuda"
    X, Wr, dl = torch.randn(T, d, device=dev), torch.randn(E, d, device=dev), torch.randn(T, E, device=dev)
    dX, dWr, db = torch.ones(T, d, device=dev), torch.full((E, d), 7.0, device=dev), torch.full((E,), 7.0, device=dev)
    ws = torch.empty(symi.symi_workspace_bytes(cfg), dtype=torch.uint8, device=dev)
    symi.symi_router_bwd(ctx, X, Wr, dl, dWr, db, dX, ws)
    wW, wb = torch.zeros(E, d, dtype=torch.float64, device=dev), torch.zeros(E, dtype=torch.float64, device=dev)
    for t in range(0, T, 1 << 17):
        r = slice(t, t + (1 << 17))
        wW += dl[r].double().T @ X[r].double()
        wb += dl[r].double().sum(0)
        q = slice(t + (1 << 17) - 256, t + (1 << 17))
        want = 1 + dl[q].double() @ Wr.double()
        assert float((dX[q].double() - want).norm() / want.norm()) <= 4e-7, t
    # sums of 2^20 terms: chunks of 512 and then 2048 chunks in ascending order, 2^-24 sqrt(2048) at most
    assert float((dWr.double() - wW).norm() / wW.norm()) <= 3e-6
    assert float((db.double() - wb).norm() / wb.norm()) <= 3e-6


@pytest.mark.parametrize("T", [100, 700])
def test_fp32_buffers_at_any_element(T):
    """fp32 buffers that begin 4 bytes behind a 16-byte boundary, as slices of a flat parameter buffer do: wide loads and stores."""
    E, d, dev = 12, 136, "cuda"
    cfg = symi.SymiCfg.make(T, E, 1, d, 8, E, 1, 0, "f32", 1)
    ctx = symi.symi_create(cfg)
    at = lambda *n: torch.randn(1 + torch.Size(n).numel() + 7, device=dev)[1:1 + torch.Size(n).numel()].view(*n)
    X, Wr, dl, dX, dWr, logits = at(T, d), at(E, d), at(T, E), at(T, d), at(E, d), at(T, E)
    dX0, ws = dX.double(), torch.empty(symi.symi_workspace_bytes(cfg), dtype=torch.uint8, device=dev)
    symi.symi_router_fwd(ctx, X, Wr, None, logits)
    symi.symi_router_bwd(ctx, X, Wr, dl, dWr, None, dX, ws)
    for name, got, want in (("logits", logits, X.double() @ Wr.double().T), ("dWr", dWr, dl.double().T @ X.double()),
                            ("dX", dX, dX0 + dl.double() @ Wr.double())):
        assert float((got.double() - want).norm() / want.norm()) <= 4e-7, name
