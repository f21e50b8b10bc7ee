"""The remote call end to end on one GPU: the requesting server's layer, the rows it ships
(prism_pack_remote), the hosting side's grouped FFN on the shipped rows (prism_expert_ffn with
one slot per row and no shared experts), and the aggregation of the returned rows
(prism_combine_remote).  Local partial + returned rows must give the layer with every expert
hosted."""
import numpy as np
import pytest
import torch

import paper_2508_12851_amd as P
from oracle import prism_oracle as O
from prism_inputs import make_config, make_inputs

from gpu_util import TOL, check_layer, desc_of, oracle_layer, rel_err, run_layer, to_dev, to_f32, weight_table

pytestmark = pytest.mark.gpu

CASES = {
    "tiny_f32": dict(name="cfg1_tiny_f32"),
    "mixtral_small": dict(name="cfg2_mixtral_prefill", T=333, H=256, F=448),
    "mixtral_decode": dict(name="cfg3_mixtral_decode", T=32, H=256, F=448),
    "finegrained_small": dict(name="cfg4_finegrained", T=700, H=128, F=192, bias_group_tokens=128),
    "dsv2_small": dict(name="cfg5_dsv2lite_migration", T=515, H=128, F=192),
}


@pytest.mark.parametrize("case", list(CASES))
def test_remote_call_completes_the_layer(case):
    kw = dict(CASES[case])
    cfg = make_config(kw.pop("name"), **kw)
    inp = make_inputs(cfg)
    f = inp.f32
    desc = desc_of(cfg)
    ws = P.alloc_workspace(desc, cfg.T)
    wt_all = weight_table(inp, all_experts=True)
    x = to_dev(inp.x)

    # requesting server: local partial sum and the remote list
    part_ref = oracle_layer(inp)
    o = run_layer(cfg, inp, wt=wt_all, ws=ws)
    check_layer(cfg, o, part_ref)
    R = int(o.n_local_remote[1])
    assert R == part_ref.dispatch.n_remote and R > 0

    # rows it ships: bit-exact copies of the remote assignments' tokens
    packed = P.prism_pack_remote(desc, x, o.remote_src, o.remote_offsets)
    torch.cuda.synchronize()
    shipped_ref = O.pack_remote(inp.x, part_ref.dispatch.remote_src, cfg.k)
    got = packed.view(torch.int16).cpu().numpy().view(np.uint16) if cfg.dtype == "bf16" \
        else packed.cpu().numpy()
    assert np.array_equal(got[:R], shipped_ref)
    assert not got[R:].any()

    # hosting side: grouped FFN over the shipped rows, one slot per row, no shared experts
    peer = P.make_desc(cfg.H, cfg.F, cfg.E, 1, 0, cfg.dtype)
    ws_peer = P.alloc_workspace(peer, R)
    rows = torch.arange(R, dtype=torch.int32, device="cuda")
    y_remote = P.prism_expert_ffn(peer, packed[:R].contiguous(), wt_all, rows, o.remote_offsets, ws_peer)
    torch.cuda.synchronize()
    experts = lambda e: tuple(f(w) for w in inp.expert(e))
    y_ref = O.expert_ffn(f(inp.x), experts, [], part_ref.dispatch.remote_src,
                         part_ref.dispatch.remote_offsets, cfg.k)
    assert rel_err(to_f32(y_remote), y_ref) <= TOL[cfg.dtype]

    # requesting server again: add the returned rows to the local partial sum
    out = o.out.clone()
    P.prism_combine_remote(desc, y_remote, o.remote_src, o.remote_offsets, o.topk_gate, out, ws)
    torch.cuda.synchronize()
    done_ref = O.combine_remote(part_ref.out, y_ref, part_ref.dispatch.remote_src,
                                part_ref.route.topk_gate, cfg.dtype)
    err = rel_err(to_f32(out), done_ref)
    assert err <= TOL[cfg.dtype], err
    # = the layer with every expert hosted, computed in one go (one rounding fewer)
    ones = np.ones(cfg.E, np.uint8)
    full_ref = oracle_layer(inp, ones)
    full = run_layer(cfg, inp, mask=ones, wt=wt_all, ws=ws)
    assert rel_err(to_f32(out), full_ref.out) <= 1.5 * TOL[cfg.dtype]
    assert rel_err(to_f32(out), to_f32(full.out)) <= 1.5 * TOL[cfg.dtype]
    print(f"{case}: R={R}, completed-layer err {err:.3g}")


def test_nothing_remote_leaves_out_untouched():
    cfg = make_config("cfg2_mixtral_prefill", T=100, H=128, F=128)
    inp = make_inputs(cfg)
    desc = desc_of(cfg)
    ws = P.alloc_workspace(desc, cfg.T)
    ones = np.ones(cfg.E, np.uint8)
    o = run_layer(cfg, inp, mask=ones, wt=weight_table(inp, all_experts=True), ws=ws)
    assert o.n_local_remote.cpu().tolist() == [cfg.A, 0]
    before = o.out.clone()
    y_none = torch.zeros((1, cfg.H), dtype=torch.bfloat16, device="cuda")
    P.prism_combine_remote(desc, y_none, o.remote_src, o.remote_offsets, o.topk_gate, o.out, ws)
    packed = P.prism_pack_remote(desc, to_dev(inp.x), o.remote_src, o.remote_offsets)
    torch.cuda.synchronize()
    assert torch.equal(o.out, before) and not packed.any()


@pytest.mark.parametrize("dtype,H", [("f32", 8), ("bf16", 64)])
@pytest.mark.parametrize("fill", [0, 1, 255])
def test_combine_on_a_workspace_that_holds_other_places(dtype, H, fill):
    """The inverse of a list is scattered over whatever the workspace held: entries of assignments that are not in
    the list must not count, whether they hold a possible row, one past the end or nothing sensible."""
    T, E, k = 37, 5, 3
    rng = np.random.default_rng([H, fill])
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    desc = P.make_desc(H, 64, E, k, 0, dtype)
    y = torch.from_numpy(rng.standard_normal((T * k, H)).astype(np.float32)).to(td).cuda()
    gate = torch.from_numpy(rng.random((T, k)).astype(np.float32)).cuda()
    ws = P.alloc_workspace(desc, T)
    ws.fill_(fill)
    for local in (0, 1, 40, T * k):             # the later calls find the places of the earlier ones
        src = rng.permutation(T * k)[:local].astype(np.int32)
        lst = torch.full((T * k,), -1, dtype=torch.int32, device="cuda")
        lst[:local] = torch.from_numpy(src).cuda()
        off = torch.from_numpy(np.linspace(0, local, E + 1).astype(np.int32)).cuda()
        got = P.prism_combine(desc, y, lst, off, gate, ws).double().cpu().numpy()
        start = torch.full((T, H), 0.5, dtype=td, device="cuda")
        added = P.prism_combine_remote(desc, y, lst, off, gate, start, ws).double().cpu().numpy()
        ref = np.zeros((T, H))
        for r, a in enumerate(src):
            ref[a // k] += gate[a // k, a % k].item() * y[r].double().cpu().numpy()
        # one rounding of the result to p significant bits, which is off by at most half a unit in the last place,
        # 2^-p of it (p = 24, and 8 for bf16), and up to 4 of the fp32 sum, whose terms are below 8
        for v, w in ((got, ref), (added, ref + 0.5)):
            assert np.all(np.abs(v - w) <= 2.0 ** (-24 if dtype == "f32" else -8) * np.abs(w) + 32 * 2.0 ** -24)


@pytest.mark.parametrize("dtype,H,n_rows,first", [("bf16", 8, 1, 0), ("bf16", 2056, 700, 3), ("f32", 24, 700, 699), ("f32", 8, 5, 5)])
def test_clear_rows(dtype, H, n_rows, first):
    desc = P.make_desc(H, 64, 2, 1, 0, dtype)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    rows = torch.ones((n_rows + 1, H), dtype=td, device="cuda")
    off = torch.tensor([0, 0, first], dtype=torch.int32, device="cuda")
    P.binding._clear_rows(desc, off, n_rows, rows, None)
    ref = torch.ones_like(rows)
    ref[first:n_rows] = 0
    assert torch.equal(rows, ref)


@pytest.mark.parametrize("dtype,T", [("f32", 70), ("bf16", 700)])
def test_expert_ffn_of_a_list_that_starts_later(dtype, T):
    """A caller's own list whose first segment starts at row 9: the rows before it are zeros, as those after the last."""
    H, F, E = 128, 192, 3
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(T)
    draw = lambda *s: (torch.randn(s, generator=gen, device="cuda") * s[1] ** -0.5).to(td)
    x, w = draw(T, H) * H ** 0.5, [(draw(F, H), draw(F, H), draw(H, F)) for _ in range(E)]
    off = [9, 9 + T // 3, 9 + T // 3, T - 7]
    src = torch.randperm(T, generator=gen, device="cuda").to(torch.int32)
    desc = P.make_desc(H, F, E, 1, 0, dtype)
    ws = P.alloc_workspace(desc, T)
    torch.full((T, H), 7.0, dtype=td, device="cuda")      # freed at once: what the allocator hands out next
    y = P.prism_expert_ffn(desc, x, P.WeightTable(w), src, torch.tensor(off, dtype=torch.int32, device="cuda"), ws)
    assert not y[:9].any() and not y[T - 7:].any()
    for e in range(E):
        xr = x[src[off[e]:off[e + 1]].long()].float()
        g, u, d = (m.float() for m in w[e])
        h = (torch.nn.functional.silu(xr @ g.t()) * (xr @ u.t())).to(td).float()
        if len(xr):
            assert rel_err(to_f32(y[off[e]:off[e + 1]]), (h @ d.t()).cpu().numpy()) <= TOL[dtype]


@pytest.mark.parametrize("first,last", [(0, 0), (3, 3), (2, 5), (0, 11), (11, 11)])
def test_clear_rows_before_and_after_the_list(first, last):
    desc = P.make_desc(24, 64, 2, 1, 0, "f32")
    rows = torch.ones((12, 24), device="cuda")
    P.binding._clear_rows(desc, torch.tensor([first, first, last], dtype=torch.int32, device="cuda"), 11, rows, None)
    ref = torch.ones_like(rows)
    ref[:first] = 0
    ref[last:11] = 0
    assert torch.equal(rows, ref)
