"""The tables of row tiles: the 128 x 128 tile's, written where a product has many tiles, and no table at all where no product of a
backward reads one and the gradients are short.  Launches counted, every product against binary64."""
import pytest

import harness as Hn
import paper_2504_19925_amd as symi
import workloads as wl
from tests.checks import launches, products_against_binary64

pytestmark = pytest.mark.gpu


def spread(S, T, empty=()):
    """T rows over S slots, from few to twice the mean, none in some."""
    rows = [0] * S
    for i in range(T):
        rows[int(S * (i / T) ** 0.5)] += 1
    for q in empty:
        rows[-1], rows[q] = rows[-1] + rows[q], 0
    return rows


# (T / 128 + S) x column tiles, 16 workgroups per compute unit (256): forward on both sides, hidden gradient on both sides
@pytest.mark.parametrize("S,T,d,f,E,tables", [
    (40, 2400, 72, 4480, 8, (1, 1)),        # 58 x 70 = 4060 first forward; the large tile in the second and in dX: its table
    (40, 2400, 72, 4544, 8, (1, 1)),        # 58 x 71 = 4118
    (300, 9000, 72, 1400, 60, (1, 1)),      # 370 x 22: small batch's own table; 370 x 11 = 4070, and more than 4096 rows: the order of the classes
    (300, 9000, 72, 1416, 60, (1, 1)),      # 370 x 12 = 4440
    (24, 900, 136, 264, 12, (0, 0)),        # small: no table, no order
    (24, 900, 136, 264, 2, (0, 1)),         # gradients of 450 rows per class
    (65, 4097, 136, 264, 65, (0, 1)),       # one row more than goes without an order
])
def test_launches_and_values(S, T, d, f, E, tables):
    c = wl.scaled(wl.get_config("c2"), E=E, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    rows = spread(S, T, empty=(0, S // 2))
    first = [S * e // E for e in range(E + 1)]
    print(f"[row tables] S={S} T={T} d={d} f={f} E={E}", flush=True)
    st = Hn.State(c, shard=0, flags=symi.CTX_TIMING | symi.CTX_NO_OVERLAP)
    products_against_binary64(st, rows, first, T + d)
    assert launches(st.ctx, "tile_map") == sum(tables)
