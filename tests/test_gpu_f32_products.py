"""The fp32 expert products at the edges of their tilings (32 x 32 with the reduction shared by
wavefronts, 64 x 64 in 32-deep and 16-deep steps, 64 x 128): every stage of an iteration against the oracle.  The tolerance is the
one every fp32 stage has (harness.metrics): 32-bit products summed 16 at a time."""
import pytest
import torch

import harness as Hn
import workloads as wl
from tests.checks import check_iteration

pytestmark = pytest.mark.gpu

# shape, and the tiling of the six products (the two forward ones, dh, dX, dW2, dW1): "s" shared reduction,
# 64 and 128 columns wide, 16: 64 wide in 16-deep steps
SHAPES = {
    # one row, reductions of a single 8-deep piece
    "one row": (dict(T=1, E=1, k=1, S_tot=1, N=1, d=8, f=8), ("s", "s", "s", "s", "s", "s")),
    # 32-row tiles with a remainder of one row and one column piece, reductions no multiple of 16
    "shared reduction": (dict(T=33, E=3, k=2, S_tot=6, N=3, d=40, f=72), ("s", "s", "s", "s", "s", "s")),
    # reductions longer than the wavefronts' 16-deep rounds, classes without rows
    "long reduction": (dict(T=700, E=16, k=1, S_tot=20, N=4, d=264, f=128), ("s", "s", "s", "s", "s", "s")),
    # all three tilings in one iteration: 8 columns in the last column tile, 32-deep steps with a remainder of 8
    "all three": (dict(T=2050, E=8, k=2, S_tot=12, N=2, d=136, f=520), (128, "s", 64, "s", "s", 64)),
    # 64-wide tiles wherever there are any, 8 rows and columns in the last one
    "64 x 64": (dict(T=4100, E=16, k=2, S_tot=24, N=2, d=200, f=520), (128, 64, 16, 64, 64, 64)),
    # the last 128-wide tile with two whole 32-column blocks and 8 columns of a third
    "64 and 128 wide": (dict(T=4100, E=8, k=2, S_tot=12, N=2, d=264, f=1096), (128, 64, 128, 64, 64, 64)),
    # 16-deep steps in three stages: both operands reduction-contiguous and the right one strided, remainders of 8
    "16 deep": (dict(T=4100, E=8, k=2, S_tot=12, N=2, d=520, f=264), (128, 16, 64, 16, "s", 64)),
    # a reduction of one step in three stages, and of two
    "16 deep, short": (dict(T=8200, E=4, k=2, S_tot=8, N=2, d=264, f=16), (128, 16, 64, 16, "s", "s")),
    # 128-wide tiles for every product, the last one with less than one 32-column block
    "64 x 128": (dict(T=6600, E=16, k=2, S_tot=24, N=2, d=520, f=1096), (128, 128, 128, 128, 128, 128)),
}


def tilings(T, E, k, S_tot, d, f, cus, **_):
    """The dispatch rule of the fp32 products: 64 x 128 tiles of each against the compute units."""
    up = lambda a, b: -(-a // b)
    rows = T * k // 64 + S_tot // 2
    heights = (rows,) * 4 + (up(d, 64) * E, up(2 * f, 64) * E)
    widths = (f, d, f, d, f, d)

    def one(i):
        n = heights[i] * up(widths[i], 128 if i else 64)
        if n < cus:
            return "s"
        if i == 0 or n >= 4 * cus:
            return 128
        return 64 if i >= 4 or heights[i] * up(widths[i], 64) <= 4 * cus else 16

    return tuple(one(i) for i in range(6))


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("active", [False, True])
def test_fp32_products(name, active):
    shape, want = SHAPES[name]
    assert tilings(cus=torch.cuda.get_device_properties(0).multi_processor_count, **shape) == want
    c = wl.scaled(wl.get_config("c1"), router_matmul=False, **shape)
    st = Hn.State(c)
    st.active_grads = active
    X, logits, dY = Hn.draw_inputs(c, 0)
    print(f"[f32 {name}] active={active} {c}", flush=True)
    check_iteration(st, X, logits, dY)
