"""GPU: the expert intermediate in 16 x 32 tiles, and row-major in a workspace that has no room for the up to 15 rows
the tiles add: both against the oracle and bit for bit the same."""
import numpy as np
import pytest
import torch

import paper_2508_12851_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,E,k,S", [
    (1, 64, 64, 4, 1, 0),          # one row, one tile column pair
    (7, 256, 1024, 4, 2, 1),       # decode, 21 rows
    (67, 192, 192, 24, 1, 0),      # small tiles
    (131, 320, 448, 8, 3, 1),      # 128-row tiles, experts that start inside a tile
    (203, 256, 1088, 4, 2, 0),     # split down projection, ragged columns
    (777, 128, 320, 3, 1, 0),      # 256-row tiles
])
def test_tiled_and_plain_intermediate(T, H, F, E, k, S):
    from gpu_util import check_layer, desc_of, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=k, S=S, bias_group_tokens=0)
    mask = (np.arange(E) != 1).astype(np.uint8)
    inp = make_inputs(cfg)
    wt = weight_table(inp, mask)
    rows = T * (k + S)

    def section(r):
        return -(-r * F * 2 // 256) * 256

    full = P.workspace_bytes(desc_of(cfg), T)
    plain = full - (section(-(-rows // 16) * 16) - section(rows))
    assert plain < full
    a = run_layer(cfg, inp, mask, wt, ws=torch.empty(full, dtype=torch.uint8, device="cuda").fill_(255))
    check_layer(cfg, a, oracle_layer(inp, mask))
    b = run_layer(cfg, inp, mask, wt, ws=torch.empty(plain, dtype=torch.uint8, device="cuda").fill_(255))
    assert torch.equal(a.out.view(torch.int16), b.out.view(torch.int16))
    with pytest.raises(Exception):
        run_layer(cfg, inp, mask, wt, ws=torch.empty(plain - 256, dtype=torch.uint8, device="cuda"))
