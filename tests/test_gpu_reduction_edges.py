"""GPU parity of the bf16 expert products where their pipelines can go wrong: reductions of one to
seven 64-deep steps with and without a partial last step (two stages of one operand, three of the
other), classes of few rows, and slots on both sides of the half-height tile's 128 rows."""
import pytest

import workloads as wl
import harness as Hn
from tests.checks import check_iteration

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f,T", [(8, 8, 40), (64, 56, 90), (72, 64, 128), (120, 136, 129), (128, 192, 250),
                                   (192, 200, 258), (256, 248, 380), (264, 320, 390), (328, 384, 515), (448, 440, 700)])
def test_steps_of_the_reduction(d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=3, k=2, d=d, f=f, T=T, S_tot=4, N=1, iters=1,
                  router_matmul=False, seed=d + T)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)


# at most 32 rows per slot on average: the forward products take their small tile.  One row, slots of
# one, several and (a uniform placement under skewed popularity) more than four 64-row parts, reductions of
# one to four steps with and without a partial one, column remainders, and the first size beyond the rule
@pytest.mark.parametrize("E,k,S,d,f,T", [(1, 1, 1, 8, 8, 1), (4, 2, 6, 72, 136, 33), (16, 2, 24, 128, 256, 64),
                                         (24, 1, 24, 200, 64, 768), (24, 1, 24, 200, 64, 769), (64, 4, 80, 136, 328, 640),
                                         (8, 1, 64, 264, 72, 2048)])
def test_few_rows_per_slot(E, k, S, d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=E, k=k, d=d, f=f, T=T, S_tot=S, N=1, iters=1,
                  router_matmul=False, seed=3 * T + d)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)
