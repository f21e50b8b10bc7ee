"""Performance cases of the placement-aware MoE layer: the work one edge server has it do.

A server keeps its layers resident (router, bias, the hosted experts, a placement mask), its
workspace and its output buffers, and calls the layer once per layer and batch.  The cases take
that call through its range: a single token to 8192, few wide and many narrow experts, both
element types, both weight layouts, both gate conventions.  A last kind of pass uses the separate
entry points the way a server that cooperates with others does: it runs its local part step by
step, packs the rows it ships, serves a peer's request and adds the rows that came back.

Inputs follow prism_inputs: tokens N(0, 1), router and expert weights N(0, 1/H), a Zipf-skewed
popularity bias, masks that host the most popular experts.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2508_12851_amd as P
from prism_inputs.generate import top_popular_mask, zipf_bias

# The layer shapes of this repository's workloads: few wide experts, and many narrow ones beside
# always-on shared experts in two variants; `many` has the most experts and picks the layer takes.
WIDE = dict(H=4096, F=14336, E=8, k=2, S=0, n_local=5, zipf_s=1.0, bias_group_tokens=0)
FINE = dict(H=2048, F=1408, E=60, k=4, S=4, n_local=36, zipf_s=1.2, bias_group_tokens=512)
FINE2 = dict(H=2048, F=1408, E=64, k=6, S=2, n_local=32, zipf_s=1.0, bias_group_tokens=0)
MANY = dict(H=1024, F=1024, E=256, k=8, S=0, n_local=128, zipf_s=1.0, bias_group_tokens=0)
SMALL_F32 = dict(H=256, F=512, E=8, k=2, S=0, n_local=4, zipf_s=1.0, bias_group_tokens=0)
LAYER_F32 = dict(H=1024, F=2048, E=8, k=2, S=0, n_local=5, zipf_s=1.0, bias_group_tokens=0)


def _case(name, shape, T, path="layer", dtype="bf16", layout="row_major", gates="renormalized"):
    c = dict(shape, T=T, path=path, dtype=dtype, layout=layout, gates=gates)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer in use (fp32, 64 tokens): launches and host work
        _case("f32_tiny", SMALL_F32, 64, dtype="f32"),
        # an fp32 layer of ordinary size: the arithmetic of the fp32 path
        _case("f32_layer", LAYER_F32, 500, dtype="f32"),
        # one sequence generating: a single token, two experts' weights streamed
        _case("wide_decode_1", WIDE, 1),
        # decode batch of 32 sequences: every hosted expert's weights streamed once
        _case("wide_decode_32", WIDE, 32, layout="tiled"),
        # decode batch of the narrow-expert layer, ragged size: many small experts, a few rows each
        _case("fine_decode_24", FINE2, 24, layout="tiled"),
        # larger decode batch or short prompt on the wide layer, weights as they come from a checkpoint
        _case("wide_mid_200", WIDE, 200),
        # short prompt on the narrow-expert layer: a dozen rows per expert
        _case("fine_mid_333", FINE, 333, layout="tiled"),
        # prefill of the wide layer: the headline batch, bound by the matrix cores
        _case("wide_prefill_4096", WIDE, 4096, layout="tiled"),
        # prefill of the narrow-expert layer, packed weights
        _case("fine_prefill_8192", FINE, 8192, layout="tiled"),
        # ragged prefill of its variant, row-major weights, the other gate convention
        _case("fine_prefill_5001", FINE2, 5001, gates="softmax_all"),
        # the largest number of experts and picks: routing and bucketing weigh most
        _case("many_experts_3000", MANY, 3000, layout="tiled"),
        # cooperating server: separate steps, remote rows packed and aggregated, a peer served
        _case("remote_call_1500", FINE2, 1500, path="remote", layout="tiled"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "wide", "wide", "fine", "fine", "fine2", "many", "remote"])
    layout = rng.choice(["row_major", "tiled"])
    gates = rng.choice(["renormalized", "renormalized", "softmax_all"])
    if kind == "f32":
        shape = dict(LAYER_F32, H=8 * _log_int(rng, 8, 128), F=8 * _log_int(rng, 8, 256),
                     n_local=rng.randint(2, 8))
        return _case(None, shape, _log_int(rng, 1, 500), dtype="f32", gates=gates)
    if kind == "wide":
        shape = dict(WIDE, H=64 * rng.randint(16, 64), F=64 * rng.randint(64, 224), n_local=rng.randint(2, 6))
        return _case(None, shape, _log_int(rng, 1, 4096), layout=layout, gates=gates)
    if kind == "fine":
        shape = dict(FINE, n_local=rng.randint(12, 60), zipf_s=rng.choice([0.0, 1.0, 1.2]))
        return _case(None, shape, _log_int(rng, 1, 8192), layout=layout, gates=gates)
    if kind == "fine2":
        shape = dict(FINE2, n_local=rng.randint(12, 64), F=64 * rng.randint(12, 32))
        return _case(None, shape, _log_int(rng, 1, 8192), layout=layout, gates=gates)
    if kind == "many":
        shape = dict(MANY, E=rng.randint(65, 256), k=rng.randint(4, 8), F=64 * rng.randint(8, 24))
        shape["n_local"] = rng.randint(16, min(shape["E"], 160))
        return _case(None, shape, _log_int(rng, 1, 4096), layout=layout, gates=gates)
    shape = dict(rng.choice([FINE, FINE2]), n_local=rng.randint(12, 48))
    return _case(None, shape, _log_int(rng, 8, 3000), path="remote", layout=layout, gates=gates)


# ---------------------------------------------------------------------------------------------
def _routing(case, seed):
    """(bias [G, E] fp32, mask [E] uint8) of a server: seeded popularity ranks, most popular hosted."""
    rng = np.random.default_rng([seed, 17])
    groups = -(-case["T"] // case["bias_group_tokens"]) if case["bias_group_tokens"] else 1
    ranks = np.stack([rng.permutation(case["E"]) + 1 for _ in range(groups)])
    bias = np.stack([zipf_bias(r, case["zipf_s"]) for r in ranks])
    return bias, top_popular_mask(ranks, case["zipf_s"], case["n_local"])


def prepare(case, seed):
    T, H, F, E, k, S = (case[n] for n in ("T", "H", "F", "E", "k", "S"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std=1.0):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dt).mul_(std)

    desc = P.make_desc(H, F, E, k, S, case["dtype"], case["bias_group_tokens"], case["gates"], case["layout"])
    bias_host, mask_host = _routing(case, seed)
    bias, mask = torch.from_numpy(bias_host).cuda(), torch.from_numpy(mask_host).cuda()
    x, w_router = normal((T, H)), normal((E, H), H ** -0.5)

    def triples(n):
        w = [normal(s, H ** -0.5) for s in ((n, F, H), (n, F, H), (n, H, F))]
        pack = P.prism_pack_weights if case["layout"] == "tiled" else (lambda m: m)
        return [tuple(pack(w[j][i]) for j in range(3)) for i in range(n)]

    hosted = iter(triples(int(mask_host.sum())))
    weights = P.WeightTable([next(hosted) if mask_host[e] else None for e in range(E)],
                            triples(S) if S else ())
    st = dict(case=case, desc=desc, x=x, w_router=w_router, bias=bias, mask=mask, weights=weights,
              ws=P.alloc_workspace(desc, T))
    if case["path"] == "layer":
        st["out"] = P.alloc_layer_out(desc, T)
        st["accum"] = torch.zeros(E, dtype=torch.int64, device="cuda")
    else:
        # a peer's request: rows for the experts hosted here, in expert order, as many as this
        # server's own batch has tokens (their number comes with the message)
        R = T
        split = np.random.default_rng([seed, 18]).multinomial(R, mask_host / mask_host.sum())
        peer = P.make_desc(H, F, E, 1, 0, case["dtype"], weight_layout=case["layout"])
        st.update(peer=peer, peer_x=normal((R, H)), peer_ws=P.alloc_workspace(peer, R),
                  peer_rows=torch.arange(R, dtype=torch.int32, device="cuda"),
                  peer_offsets=torch.from_numpy(np.concatenate([[0], np.cumsum(split)]).astype(np.int32)).cuda(),
                  y_returned=normal((T * k, H), 0.5))
    return st


def run(st):
    d, x = st["desc"], st["x"]
    if st["case"]["path"] == "layer":
        o = P.prism_moe_layer(d, x, st["w_router"], st["bias"], st["weights"], st["mask"], st["ws"],
                              outputs=st["out"], counts_accum=st["accum"])
        return dict(vars(o), accum=st["accum"])
    # requesting server: its own part, and the rows it ships
    r = P.prism_route(d, x, st["w_router"], st["bias"], want_logits=False)
    s = P.prism_dispatch(d, r.topk_idx, st["mask"], st["ws"])
    shipped = P.prism_pack_remote(d, x, s.remote_src, s.remote_offsets)
    y = P.prism_expert_ffn(d, x, st["weights"], s.local_src, s.local_offsets, st["ws"])
    out = P.prism_combine(d, y, s.local_src, s.local_offsets, r.topk_gate, st["ws"])
    # serving a peer meanwhile
    served = P.prism_expert_ffn(st["peer"], st["peer_x"], st["weights"], st["peer_rows"],
                                st["peer_offsets"], st["peer_ws"])
    # what the peers sent back
    P.prism_combine_remote(d, st["y_returned"], s.remote_src, s.remote_offsets, r.topk_gate, out, st["ws"])
    return dict(out=out, shipped=shipped, served=served, counts=r.counts, idx=r.topk_idx, gate=r.topk_gate,
                **{n: getattr(s, n) for n in ("local_src", "local_offsets", "remote_src", "remote_offsets",
                                              "n_local_remote", "remote_bytes")})


# ---------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _expected_routing(T, E, k, n_local, zipf_s, bias_group_tokens):
    """Expected (local assignments, hosted experts that receive a token) of a batch, from sampled
    N(0, 1) router logits plus the popularity bias."""
    case = dict(T=T, E=E, n_local=n_local, zipf_s=zipf_s, bias_group_tokens=bias_group_tokens)
    gen = torch.Generator().manual_seed(0)
    local, touched, passes = 0.0, 0.0, max(1, min(32, 4096 // T))
    for p in range(passes):
        bias, mask = _routing(case, p)
        n = min(T, 4096)
        rows = torch.arange(n) * T // n // bias_group_tokens if bias_group_tokens else torch.zeros(n, dtype=torch.long)
        picks = (torch.randn((n, E), generator=gen) + torch.from_numpy(bias)[rows]).topk(k, dim=1).indices
        hits = torch.bincount(picks.reshape(-1), minlength=E) * torch.from_numpy(mask)
        local += float(hits.sum()) * T / n / passes
        touched += float((hits > 0).sum()) / passes
    return local, touched


def work(case):
    T, H, F, E, k, S = (case[n] for n in ("T", "H", "F", "E", "k", "S"))
    es = 4 if case["dtype"] == "f32" else 2
    local, touched = _expected_routing(T, E, k, case["n_local"], case["zipf_s"], case["bias_group_tokens"])
    rows = local + S * T
    expert = 3.0 * H * F * es
    # tokens, router, the experts that have rows, output rows; picks, gates and the remote list
    nbytes = (2.0 * T + E) * H * es + (touched + S) * expert + 12.0 * T * k
    flops = 2.0 * T * H * E + 6.0 * H * F * rows
    if case["path"] == "remote":
        # shipped rows, returned rows, the peer's rows in and out (its experts are the same ones)
        nbytes += (2.0 * (T * k - local) + 2.0 * T) * H * es + 4.0 * T * k
        flops += 6.0 * H * F * T
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # About four times what is seen against the same layer in 64 bits.  fp32: sums of up to 2048
    # terms, 2e-7 of the norm and 1.2e-6 of the rms as the path adds them, 1.2e-6 and 5.5e-6 when the
    # products are added one after the other.  bf16: the intermediate, the expert rows and the output
    # are each rounded once, 3e-3 of the norm and 1.2e-2 to 1.8e-2 of the rms.  Indices, counts, lists
    # and offsets are whole numbers and agree exactly.
    return {"rel": 5e-6, "max": 2.5e-5} if case["dtype"] == "f32" else {"rel": 1.2e-2, "max": 6e-2}
