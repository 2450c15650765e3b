"""The fp32 expert products at the edges of their three tilings (32 x 32 with the reduction shared by
wavefronts, 64 x 64, 64 x 128): every stage of an iteration against the oracle.  The tolerance is the
one every fp32 stage has (harness.metrics): 32-bit products summed 16 at a time."""
import pytest

import harness as Hn
import workloads as wl
from tests.checks import check_iteration

pytestmark = pytest.mark.gpu

SHAPES = {
    # one row, reductions of a single 8-deep piece
    "one row": dict(T=1, E=1, k=1, S_tot=1, N=1, d=8, f=8),
    # 32-row tiles with a remainder of one row and one column piece, reductions no multiple of 16
    "shared reduction": dict(T=33, E=3, k=2, S_tot=6, N=3, d=40, f=72),
    # reductions longer than the wavefronts' 16-deep rounds, classes without rows
    "long reduction": dict(T=700, E=16, k=1, S_tot=20, N=4, d=264, f=128),
    # 64-wide tiles: 8 columns in the last column tile, 32-deep steps with a remainder of 8
    "64 x 64": dict(T=2050, E=8, k=2, S_tot=12, N=2, d=136, f=520),
    # 128-wide tiles for every product, the last one with less than one 32-column block
    "64 x 128": dict(T=4100, E=8, k=2, S_tot=12, N=2, d=264, f=1096),
}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("active", [False, True])
def test_fp32_products(name, active):
    c = wl.scaled(wl.get_config("c1"), router_matmul=False, **SHAPES[name])
    st = Hn.State(c)
    st.active_grads = active
    X, logits, dY = Hn.draw_inputs(c, 0)
    print(f"[f32 {name}] active={active} {c}", flush=True)
    check_iteration(st, X, logits, dY)
