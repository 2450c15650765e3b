"""The 128 x 128 tile of the bf16 variable-row products (few or short tiles) against the oracle's layer: slots of one
row up to three tiles, both sides of the 64 rows below which half the wavefronts rest, reductions of one to six 64-deep
steps with and without a ragged end, ragged columns, numbers of column tiles that are and are not multiples of eight; and
both sides of the rule that chooses it, against binary64."""
import pytest
import torch

import paper_2504_19925_amd as symi
import workloads as wl
import harness as Hn
from tests.checks import bf16_tiles, check_iteration, launches, products_against_binary64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,S,d,f,T", [(2, 1, 2, 8, 8, 70), (3, 2, 4, 64, 72, 129), (4, 1, 5, 136, 520, 641),
                                         (6, 2, 9, 200, 328, 333), (4, 2, 6, 392, 264, 500), (2, 1, 3, 320, 1032, 385),
                                         # long reductions; many rows, where the forward and the input gradient take the large tile
                                         (4, 1, 4, 1024, 72, 512), (4, 1, 4, 1024, 72, 513), (4, 1, 4, 1032, 72, 512),
                                         (16, 4, 16, 256, 1024, 4100)])
def test_layer(E, k, S, d, f, T):
    c = wl.scaled(wl.get_config("c2"), dtype="bf16", E=E, k=k, d=d, f=f, T=T, S_tot=S, N=1, iters=1,
                  router_matmul=False, seed=d + T)
    print(f"[mid tile] E={E} S={S} d={d} f={f} T={T}", flush=True)
    st = Hn.State(c, shard=0)
    X, logits, dY = Hn.draw_inputs(c, 0)
    check_iteration(st, X, logits, dY)


# given slot offsets: row counts at the tile's edges, empty slots in front, between and behind, more slots than a
# workgroup has threads
@pytest.mark.parametrize("d,f,extra", [(72, 136, 0), (264, 192, 0), (128, 520, 300)])
def test_tile_edges(d, f, extra):
    rows = [0, 1, 63, 64, 65, 0, 127, 128, 129, 191, 193, 257, 10, 300, 300] + [0] * extra + [5, 0]
    S, T = len(rows), sum(rows)
    c = wl.scaled(wl.get_config("c2"), E=4, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    print(f"[mid edges] d={d} f={f} S={S}", flush=True)
    products_against_binary64(Hn.State(c, shard=0), rows, [0, 3, 7, 9, S], d)


# both sides of every line of the rule, in mean rows per slot and in reduction length, and of the limit of tiles x K (at and above
# 128 rows on average), with one stream, and of the backward's limit with two; which tile the four products take.  Rows spread
# from none to twice the mean
@pytest.mark.parametrize("S,T,d,f,want", [
    (16, 1024, 1536, 1360, "mmmL"), (16, 1025, 1536, 1360, "LmmL"), (16, 1024, 1544, 1360, "LmmL"),    # first forward: 64, 1536
    (32, 3584, 640, 1200, "mmmL"), (32, 3585, 640, 1200, "LmmL"), (32, 3584, 648, 1200, "LmmL"),       # 112, 640
    (64, 4096, 640, 1984, "mmmL"), (64, 4097, 640, 1984, "mLmL"), (64, 4096, 640, 1992, "mLmL"),       # second forward: 64, 1984
    (64, 7168, 640, 1024, "mmmL"), (64, 7169, 640, 1024, "LLmL"), (64, 7168, 640, 1032, "mLmL"),       # 112, 1024
    (16, 640, 1792, 2320, "LLmL"), (16, 641, 1792, 2320, "LLLL"), (16, 640, 1800, 2320, "LLLL"),       # hidden gradient: 40, 1792
    (16, 1280, 1536, 2320, "LLmL"), (16, 1281, 1536, 2320, "LLLL"), (16, 1280, 1544, 2320, "LLLL"),    # 80, 1536
    (32, 4096, 512, 2696, "LLmL"), (32, 4097, 512, 2696, "LLLL"), (32, 4096, 520, 2696, "LLLL"),       # 128, 512
    (32, 1536, 1032, 768, "mmmm"), (32, 1537, 1032, 768, "mmmL"), (32, 1536, 1032, 776, "mmmL"),       # input gradient: 48, 1536
    (32, 3072, 1928, 320, "mmmm"), (32, 3073, 1928, 320, "mmmL"), (32, 3072, 1928, 328, "mmmL"),       # 96, 640
    (8, 1024, 1024, 2688, "mLmL"), (8, 1024, 1024, 2752, "LLmL"),                                      # tiles x K
    (4, 2048, 512, 1792, "mmmL"), (4, 2048, 512, 1856, "LmmL"),                                        # half of it, 512 rows
    (4, 2048, 128, 992, "mmmm"), (4, 2048, 128, 1000, "mmmL"),                                         # 31 and 32 steps
    (4, 8192, 512, 712, "Lmmm2"), (4, 8192, 512, 720, "LmLL2"),                                        # two streams: 3e9
    (128, 5120, 1024, 408, "mmmm2"), (129, 5120, 1024, 408, "mmmL2")])                                 # 4 tiles per unit
def test_both_sides_of_the_rule(S, T, d, f, want):
    streams, want = 2 if want[4:] else 1, want[:4]
    c = wl.scaled(wl.get_config("c2"), E=2, k=1, d=d, f=f, T=T, S_tot=S, N=1, iters=1, router_matmul=False)
    assert bf16_tiles(T, 2, 1, S, d, f, streams) == want
    st = Hn.State(c, shard=0, flags=symi.CTX_TIMING | (0 if streams == 2 else symi.CTX_NO_OVERLAP))
    rows = [0] * S
    for i in range(T):
        rows[int(S * (i / T) ** 0.5)] += 1
    rows[0], rows[-1] = 0, rows[-1] + rows[0]
    print(f"[mid rule] S={S} T={T} d={d} f={f} {want}", flush=True)
    products_against_binary64(st, rows, [0, S // 2, S], T + d)
    # the table of the large tile's rows is written unless neither forward product takes it, and always by the backward
    assert launches(st.ctx, "tile_map") == 1 + ("L" in want[:2])
