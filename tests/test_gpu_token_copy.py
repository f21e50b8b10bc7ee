"""GPU: the copy of the token rows that prefill batches of wide layers multiply (rows past the last whole tile of 16, which
the copy keeps behind y; shared experts; hidden sizes that are no multiple of the 1024 columns of a workgroup; experts
hosted elsewhere), in the whole layer and in prism_expert_ffn with a y of the caller's, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2508_12851_amd as P
from ffn_paths import packs_rows
from oracle import prism_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,E,k,S,hosted,tiled", [
    (777, 1088, 4096, 16, 8, 1, 3, True),       # 6993 rows: the last tile has one
    (513, 2112, 4160, 8, 4, 1, 2, True),        # fewest tokens; 2565 rows, 5 past a tile
    (601, 1024, 4608, 8, 8, 0, 2, True),        # whole chunks of columns, no shared experts; 4808 rows, 8 past a tile
    (1501, 2112, 4096, 16, 8, 2, 2, False),     # row-major weights; 15010 rows, 2 past a tile
    (1024, 1984, 4096, 8, 8, 6, 0, False),      # shared experts only; whole tiles
])
def test_token_copy(T, H, F, E, k, S, hosted, tiled):
    from gpu_util import TOL, check_layer, desc_of, oracle_layer, rel_err, run_layer, to_dev, to_f32, weight_table
    from prism_inputs import make_config, make_inputs
    assert packs_rows(H, F, E, k, S, T, tiled)
    layout = "tiled" if tiled else "row_major"
    cfg = make_config("cfg4_finegrained", T=T, H=H, F=F, E=E, k=k, S=S, bias_group_tokens=0, zipf_s=1.0)
    mask = np.zeros(E, np.uint8)
    mask[np.random.default_rng([T, E]).permutation(E)[:hosted]] = 1
    inp = make_inputs(cfg)
    wt = weight_table(inp, mask, tiled=tiled)
    ref = oracle_layer(inp, mask)
    check_layer(cfg, run_layer(cfg, inp, mask, wt, weight_layout=layout), ref)

    # prism_expert_ffn: the copy lies in the workspace, not in the caller's y
    desc = desc_of(cfg, weight_layout=layout)
    ws = P.alloc_workspace(desc, T)
    d = P.prism_dispatch(desc, to_dev(ref.route.topk_idx), to_dev(mask), ws)
    y = torch.full((T * (k + S), H), -7.0, dtype=torch.bfloat16, device="cuda")
    P.prism_expert_ffn(desc, to_dev(inp.x), wt, d.local_src, d.local_offsets, ws, y=y)
    f, nl, A = inp.f32, ref.dispatch.n_local, T * k
    got = to_f32(y)
    assert (got[nl:A] == -7.0).all()
    want = O.expert_ffn(f(inp.x), lambda e: tuple(f(w) for w in inp.expert(e)),
                        [tuple(f(w) for w in inp.shared(s)) for s in range(S)], ref.dispatch.local_src,
                        ref.dispatch.local_offsets, k)
    assert rel_err(np.concatenate([got[:nl], got[A:]]), want) <= TOL["bf16"]
