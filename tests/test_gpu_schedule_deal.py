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


@pytest.mark.parametrize("T,H,F", [
    (600, 1280, 4096),       # 30 items: lists of 3 and 4
    (1100, 768, 4160),       # 30 items, 130 k-tiles
    (2100, 1088, 4096),      # 90 items: lists of 11 and 12, last round not full
])
def test_lists_of_a_cut_last_round_take_equal_slices(T, H, F):
    """The longest list decides how thin the slices of all lists are (read from the schedule in the workspace)."""
    import paper_2508_12851_amd as P
    from gpu_util import check_layer, desc_of, oracle_layer, run_layer, weight_table
    from prism_inputs import make_config, make_inputs
    E = 2                                   # two picks of two experts: T rows each
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=2, S=0, bias_group_tokens=0, n_local=E)
    inp = make_inputs(cfg)
    mask = np.ones(E, np.uint8)
    ws = P.alloc_workspace(desc_of(cfg), T)
    o = run_layer(cfg, inp, mask, weight_table(inp, mask), ws=ws)
    check_layer(cfg, o, oracle_layer(inp, mask))

    # the workspace: local_src, local_offsets, inv, histograms, then the two schedules
    def up(n, a):
        return -(-n // a) * a

    A = 2 * T
    start = 2 * up(4 * A, 256) + up(4 * (E + 1), 256) + up(4 * (-(-A // 2048)) * E, 256)
    row_tiles64 = A // 64 + E + 1
    ints = up(32 + 64 * (row_tiles64 * -(-(-(-max(H, F) // 64)) // 8) + 32) + 8 * 16 * 8, 64)
    head = ws[start + 4 * ints:start + 4 * ints + 128].view(torch.int32).cpu().numpy()
    items = E * -(-T // 256) * -(-H // 256)
    assert head[0] == E * -(-T // 256)
    slices = set()
    for x in range(8):
        n = items * (x + 1) // 8 - items * x // 8
        cut = n - head[4 + x]
        assert cut == n % 32
        slices.add(int(head[20 + x]) // cut)
        assert head[20 + x] % cut == 0
    assert slices == {min(16, 32 // (-(-items // 8) % 32), F // 32 // 8)}
