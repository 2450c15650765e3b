"""Kernels that choose between two kinds of loads by size (combine, dispatch backward, replica all-reduce) on both sides of
their rules, in both types: rows of 528 and of 496 MiB, gradients and activations of 518 and 500, slot gradients of 281
and 226; against plain torch in binary64.  A combined value is a 32-bit sum of k products in order, rounded to its type."""
import pytest
import torch

import paper_2504_19925_amd as symi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mb,f", [(528, 8), (496, 8), (160, 352), (160, 320)])
def test_combine_and_dispatch_backward(dtype, mb, f):
    w, d, k, E = (2 if dtype == "bf16" else 4), 1024, 3, 8
    T = (mb << 20) // (w * d * k)
    cfg = symi.SymiCfg.make(T, E, k, d, f, E, 1, 0, dtype, 1)
    ctx = symi.symi_create(cfg)
    dt, dev, A = cfg.torch_dtype, "cuda", T * k
    g = torch.Generator(device=dev).manual_seed(mb)
    rows = torch.randn(A, d, generator=g, device=dev, dtype=dt)
    roa = torch.randperm(A, generator=g, device=dev).to(torch.int32)
    roa[::17] = -1                                          # dropped by a capacity rule
    gate = torch.rand(T, k, generator=g, device=dev)
    Y, dX = torch.full((T, d), 7.0, dtype=dt, device=dev), torch.full((T, d), 7.0, dtype=dt, device=dev)
    print(f"[hints] {dtype} {mb} MB f={f}", flush=True)
    symi.symi_combine(ctx, rows, roa, gate, Y)
    symi.symi_dispatch_bwd(ctx, rows, roa, dX)
    for out, weights in ((Y, gate), (dX, torch.ones_like(gate))):
        for t0 in range(0, T, 16384):
            at = roa.view(T, k)[t0:t0 + 16384].long()
            wt = torch.where(at >= 0, weights[t0:t0 + 16384], 0.0).double()
            x = rows[at.clamp(min=0)].double() * wt[..., None]
            want, scale = x.sum(1), x.abs().sum(1)
            eps = (2.0 ** -8 * want.abs() if dtype == "bf16" else 0.0) + 4 * 2.0 ** -24 * scale
            assert bool(((out[t0:t0 + 16384].double() - want).abs() <= eps).all())


@pytest.mark.parametrize("f", [2000, 1608])
def test_replica_all_reduce(f):
    E, S, d = 4, 12, 1024
    ctx = symi.symi_create(symi.SymiCfg.make(16, E, 1, d, f, S, 1, 0, "bf16", 1))
    first = torch.tensor([0, 1, 3, 7, 12], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(f)
    g1, g2 = torch.randn(S, 2 * f, d, generator=g, device="cuda"), torch.randn(S, d, f, generator=g, device="cuda")
    want = [t.clone() for t in (g1, g2)]
    print(f"[hints] all-reduce {12 * S * d * f / 1e6:.0f} MB", flush=True)
    symi.symi_replica_allreduce(ctx, first, 0.5, g1, g2)
    for got, x in zip((g1, g2), want):
        for e in range(E):
            a, b = int(first[e]), int(first[e + 1])
            s = x[a].clone()
            for q in range(a + 1, b):                       # slot order, in 32 bits
                s += x[q]
            s *= 0.5
            assert all(torch.equal(got[q], s) for q in range(a, b))
