"""GPU: batches between decode and prefill at the lines of the rules that choose their tiles (rows per expert, rows
of the shared experts, token limits of the split down projection) and at the edges of those tiles, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,E,k,S,hosted", [
    (65, 256, 1024, 4, 2, 0, 3),       # split down projection: fewest tokens, shortest contractions
    (256, 320, 1088, 4, 2, 1, 4),      # ragged columns, last size of the streaming tiles
    (257, 320, 1088, 4, 4, 0, 4),      # every expert 257 rows: a third row tile of one row
    (512, 256, 1024, 8, 2, 1, 5),      # last split size
    (513, 256, 1024, 8, 2, 1, 5),
    (448, 1088, 1088, 4, 2, 0, 3),     # last size in 128 x 128 tiles: ragged columns
    (449, 1088, 1088, 4, 2, 1, 3),     # and one token more, in 128 x 256 ones
    (256, 2624, 1024, 4, 2, 0, 3),     # more columns, last size of the streaming tiles
    (257, 2624, 1088, 4, 4, 0, 4),     # and a third row tile of one row
    (130, 256, 2048, 4, 2, 0, 3),      # F = 8 H
    (360, 256, 4096, 8, 2, 0, 5),      # a contraction long enough for the cut, not cut any more
    (384, 192, 192, 48, 2, 0, 40),     # 16 rows per expert, shortest ring
    (385, 192, 192, 48, 2, 0, 40),     # one pick over it
    (128, 192, 704, 32, 4, 4, 20),     # 512 shared rows
    (129, 192, 704, 32, 4, 4, 20),     # 516
    (1152, 320, 448, 24, 3, 0, 24),    # 144 rows per expert: last size of the 128-row tiles of a small layer
    (1153, 320, 448, 24, 3, 1, 24),
    (3584, 320, 192, 256, 8, 0, 200),  # 112 rows per expert of a layer with many: last size of the 128-row tiles
    (3585, 320, 192, 256, 8, 0, 200),
    # One pick per token, the popular experts with several row tiles.  (All experts hosted: with a share p of
    # the tokens local, the rms of the batch is sqrt(p) of a local row's, and a rounding error of 3e-3 of the
    # row's rms counts as 3e-3 / sqrt(p) against the bar of 2e-2; one token of 1025 would count 9e-2.)
    (1024, 192, 192, 64, 1, 0, 64),    # last size of the 64-row tiles
    (1025, 192, 192, 65, 1, 0, 65),
    (2560, 192, 192, 64, 1, 0, 64),    # last size of the 128-row tiles
    (2561, 192, 192, 64, 1, 0, 64),
    (128, 192, 320, 2, 2, 1, 2),       # full 128-row tiles
    (129, 192, 320, 2, 2, 1, 1),       # and one row more
    (70, 128, 192, 64, 2, 0, 64),      # contraction below the rings': prefill tiles
])
def test_mid_batch_tiles(T, H, F, E, k, S, hosted):
    from gpu_util import check_layer, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=k, S=S, bias_group_tokens=0)
    mask = np.zeros(E, np.uint8)
    mask[np.random.default_rng([T, E]).permutation(E)[:hosted]] = 1
    inp = make_inputs(cfg)
    ref = oracle_layer(inp, mask)
    for layout in ("row_major", "tiled"):
        check_layer(cfg, run_layer(cfg, inp, mask, weight_table(inp, mask, tiled=layout == "tiled"),
                                   weight_layout=layout), ref)
