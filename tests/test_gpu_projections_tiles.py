"""Selection projections at the edges of the tiles: sequences shorter than a
vector, groups of positions that end inside one (L % 4), channel counts off a
step (16 fp32, 32 bf16), every split of a tile over waves, ranks off a vector,
and a last row block that is partly timescale rows. Against the fp64 oracle at
the tolerances of the other projections."""
import pytest

import oracle
import workloads
from gpu_util import BF16_TOL, FP32_TOL, assert_close, log, to_f64
from test_gpu_projections import draw_u, run

pytestmark = pytest.mark.gpu

CASES = [  # batch, K, Dc, L, N, R
    (1, 1, 1, 1, 1, 1),
    (3, 2, 15, 2, 2, 1),
    (2, 4, 31, 3, 16, 2),
    (2, 4, 33, 5, 16, 3),       # two positions a lane, L odd
    (1, 3, 16, 63, 8, 16),
    (2, 4, 48, 1027, 16, 17),   # four positions a lane, four waves: a partial group
    (4, 4, 17, 1025, 4, 33),
    (1, 1, 70, 16390, 16, 4),
    (4097, 4, 17, 1, 8, 5),     # positions over the batch: a partial tile
    (1403, 4, 33, 3, 16, 3),
    (11001, 4, 20, 3, 4, 2),    # the same, two waves a tile in bf16
    (8, 4, 20, 8195, 16, 5),    # two waves a tile, more waves than steps
    (8, 4, 100, 8197, 1, 18),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,K,Dc,L,N,R", CASES)
def test_tile_edges(batch, K, Dc, L, N, R, dtype):
    log(f"projections b={batch} K={K} Dc={Dc} L={L} N={N} R={R} {dtype}")
    u, ut = draw_u(batch, K, Dc, L, seed=Dc + L, dtype=dtype)
    pw = workloads.make_projection_weights(K, Dc, N, R, seed=R)
    d, B, C = run(ut, pw, N)
    rd, rB, rC = oracle.projections(u, pw.W, pw.W_dt, N=N)
    tol = FP32_TOL if dtype == "f32" else BF16_TOL
    for got, ref, nm in ((B, rB, "B"), (C, rC, "C"), (d, rd, "delta")):
        assert_close(to_f64(got), ref, **tol, what=f"{nm} {dtype}")
