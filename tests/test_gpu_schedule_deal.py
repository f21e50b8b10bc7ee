"""GPU: the deal of routed and shared work items over the XCDs at its edges (fewer than 8 shared items, none, only
shared ones, fewer items than XCDs), against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,E,S,hosted", [
    (70, 64, 64, 2, 1, 2),       # one column tile: 1 shared item, counted as a routed one
    (257, 64, 64, 4, 3, 4),      # 6 shared items
    (257, 64, 64, 4, 4, 4),      # 8 shared items, 4 to 8 routed ones
    (300, 256, 128, 8, 2, 0),    # shared items only
    (1100, 320, 704, 64, 1, 64),
    (600, 192, 1408, 128, 16, 3),
    (900, 256, 256, 8, 0, 5),    # no shared items
])
def test_deal_of_routed_and_shared_items(T, H, F, E, S, hosted):
    from gpu_util import check_layer, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=min(2, E), S=S, bias_group_tokens=0)
    mask = np.zeros(E, np.uint8)
    mask[np.random.default_rng([T, E]).permutation(E)[:hosted]] = 1
    inp = make_inputs(cfg)
    check_layer(cfg, run_layer(cfg, inp, mask, weight_table(inp, mask)), oracle_layer(inp, mask))
