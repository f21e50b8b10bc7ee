"""GPU: the router inside the layer (experts and hidden elements spread over workgroups, picks counted per placement
block; decode batches of at most 16 experts: the decode front end) at its edges, against the oracle, whole numbers
bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,E,k", [
    (65, 64, 2, 1),          # fewest tokens, 2 slices of the hidden dimension for 8 wavefronts
    (65, 64, 256, 1),        # partial logits larger than the FFN buffers they would borrow: one-launch router
    (97, 2112, 17, 3),       # ragged tiles, odd number of slices; 48 assignments per workgroup straddle blocks
    (513, 320, 65, 8),       # 5 of 8 expert tiles, 4104 assignments
    (1366, 128, 60, 6),      # 8196 assignments: first size with blocks of 2048
    (700, 1024, 129, 7),     # 9 of 16 expert tiles
    (300, 256, 256, 5),
    (5000, 64, 16, 2),
    (1, 256, 17, 1),         # decode batches: fewest experts, one token
    (24, 2048, 64, 6),
    (64, 192, 256, 8),
    (3, 64, 256, 1),         # partial logits larger than the FFN buffers: a decode batch has a region for them
    (16, 64, 33, 1),
    (64, 4160, 65, 8),       # long hidden dimension, most assignments
    (64, 320, 16, 2),        # last expert count of the decode front end
])
@pytest.mark.parametrize("gates", ["renormalized", "softmax_all"])
def test_split_router_in_layer(T, H, E, k, gates):
    from gpu_util import check_layer, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=64, E=E, k=k, S=1, bias_group_tokens=100)
    mask = (np.random.default_rng([T, E]).random(E) < 0.3).astype(np.uint8)
    mask[E - 1] = 1
    inp = make_inputs(cfg)
    o = run_layer(cfg, inp, mask, weight_table(inp, mask), gate_mode=gates)
    check_layer(cfg, o, oracle_layer(inp, mask, renormalize=gates == "renormalized"))


@pytest.mark.parametrize("T,E,k", [(6112, 60, 4), (6113, 60, 4), (8192, 60, 4), (8193, 60, 4), (10001, 8, 2)])
def test_router_of_large_batches(T, E, k):
    """Both sides of the lines between the router in one launch (6113 to 8192 tokens) and the spread one, the whole layer."""
    from gpu_util import check_layer, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    H, F = 64, 256
    # the spread router borrows the FFN's h and y for the histograms of blocks of at least 512 picks and one part of the
    # logits (experts in tiles of 16, up to a power of two of them); a layer that lacks the room takes the other one
    experts = 16 * next(n for n in (1, 2, 4, 8, 16) if 16 * n >= E)
    assert T * k * (H + F) * 2 >= -(-T * k // 512) * E * 4 + 256 + T * experts * 8
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=k, S=0, bias_group_tokens=100)
    mask = (np.random.default_rng([T, E]).random(E) < 0.5).astype(np.uint8)
    inp = make_inputs(cfg)
    o = run_layer(cfg, inp, mask, weight_table(inp, mask))
    check_layer(cfg, o, oracle_layer(inp, mask))
