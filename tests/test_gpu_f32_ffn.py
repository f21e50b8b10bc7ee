"""GPU: the fp32 expert FFN at the edges of its tiles (64 rows x 32 / 64 columns, k-tiles of 16, eighths of the
contraction), against 64-bit arithmetic."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,rows,S", [
    (1, 8, 1, [0, 1, 0], 0),                    # one element per row of the down projection
    (5, 16, 3, [2, 0, 3], 1),                   # rows shorter than a 16-byte load
    (70, 24, 5, [64, 1, 5], 2),                 # full tile, single row; misaligned rows of W_down
    (130, 136, 18, [65, 32, 33], 0),            # both halves of a tile and one row more
    (160, 200, 33, [63, 0, 97], 1),
    (40, 1024, 2047, [7, 33, 0], 1),            # the longest chains; every weight row at another alignment
    (300, 264, 130, [129, 128, 43], 0),
    (1000, 64, 2048, [500, 300, 97, 65, 33], 0),   # gate/up in tiles of 64 rows, down in tiles of 32
    (200, 40, 4096, [100, 64, 33], 3),          # the same with shared rows
    (1100, 2056, 320, [600, 65, 33, 400], 0),   # fp32 products: gate/up in tiles of 64 rows (200 items), ...
    (1100, 2056, 512, [600, 65, 33, 400], 0),   # ... and of 32 (320 items of 64 rows are two rounds, 592 of 32 three)
])
def test_f32_ffn_edges(T, H, F, rows, S):
    import paper_2508_12851_amd as P
    rng = np.random.default_rng([T, H, F])
    E, A = len(rows), T                          # top_k = 1: at most one row per token
    assert sum(rows) <= A
    x = rng.standard_normal((T, H)).astype(np.float32)
    w = [[(rng.standard_normal(s) / np.sqrt(s[1])).astype(np.float32) for s in ((F, H), (F, H), (H, F))]
         for _ in range(E + S)]
    src = rng.permutation(A)[:sum(rows)].astype(np.int32)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)

    def dev(a):
        return torch.from_numpy(a).cuda()

    desc = P.make_desc(H, F, E, 1, S, "f32")
    table = P.WeightTable([tuple(map(dev, t)) for t in w[:E]], [tuple(map(dev, t)) for t in w[E:]])
    y = torch.full((A + S * T, H), -7.0, device="cuda")
    local_src = torch.full((A,), -1, dtype=torch.int32, device="cuda")
    local_src[:len(src)] = dev(src)
    P.prism_expert_ffn(desc, dev(x), table, local_src, dev(off), P.alloc_workspace(desc, T), y=y)
    y = y.cpu().numpy()

    def ffn(xr, t):
        g, u, d = (m.astype(np.float64) for m in t)
        a = xr.astype(np.float64)
        z = a @ g.T
        return (z / (1.0 + np.exp(-z)) * (a @ u.T)) @ d.T

    # Each sum passes at most 4 + 2 + K/128 + 3 < 32 roundings of 2^-24; they are independent, so the
    # relative 2-norm of a sum's error stays below sqrt(32) * 2^-24 = 3.4e-7; gate, up and down add up.
    def check(got, ref):
        if ref.size:
            assert np.linalg.norm(got - ref) <= 1e-6 * np.linalg.norm(ref)

    for e in range(E):
        check(y[off[e]:off[e + 1]], ffn(x[src[off[e]:off[e + 1]]], w[e]))
    assert (y[off[E]:A] == -7.0).all()           # rows without an assignment are not written
    for s in range(S):
        check(y[A + s * T:A + (s + 1) * T], ffn(x, w[E + s]))


@pytest.mark.parametrize("T,H,F", [(70, 40, 24), (33, 264, 130), (65, 2056, 40), (40, 64, 2056)])
def test_f32_ffn_values_without_bf16_parts(T, H, F):
    """Values that round up to infinity in bf16, infinities and NaN, on both sides of the longest contraction
    that is multiplied in parts (2048): finite rows as in 64 bits, the others infinite or NaN in the same places."""
    import paper_2508_12851_amd as P
    rng = np.random.default_rng([T, H, F])
    x = rng.standard_normal((T, H)).astype(np.float32)
    w = [(rng.standard_normal(s) / np.sqrt(s[1])).astype(np.float32) for s in ((F, H), (F, H), (H, F))]
    for m in w[:2]:
        m[:, 7] *= np.float32(1e-38)
    x[5, 7] = 3.4e38                             # below the largest fp32 value, above the largest bf16 one
    x[9, 1], x[T - 1, H - 1] = np.inf, -np.inf
    x[11, 2] = np.nan
    dev = lambda a: torch.from_numpy(a).cuda()
    desc = P.make_desc(H, F, 1, 1, 0, "f32")
    y = P.prism_expert_ffn(desc, dev(x), P.WeightTable([tuple(map(dev, w))]), torch.arange(T, dtype=torch.int32, device="cuda"),
                           torch.tensor([0, T], dtype=torch.int32, device="cuda"), P.alloc_workspace(desc, T)).cpu().numpy()
    with np.errstate(all="ignore"):
        g, u, d = (m.astype(np.float64) for m in w)
        z = x.astype(np.float64) @ g.T
        ref = (z / (1.0 + np.exp(-z)) * (x.astype(np.float64) @ u.T)) @ d.T
    odd = [9, 11, T - 1]
    assert (np.isnan(ref[odd]) | np.isinf(ref[odd])).all()
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(y), np.isinf(ref))
    rest = np.setdiff1d(np.arange(T), odd)       # bound: test_f32_ffn_edges
    assert np.linalg.norm(y[rest] - ref[rest]) <= 1e-6 * np.linalg.norm(ref[rest])


def test_f32_ffn_of_more_tiles_than_one_grid_dimension_holds():
    """16392 row tiles x 512 column tiles = 8.4 million workgroups of 512 threads, more than 2^32 threads in a row
    (h takes 69 GB).  Every row written, rows at the edges of every expert against 64-bit arithmetic."""
    import paper_2508_12851_amd as P
    T, H, F, E = 131072, 64, 16384, 8
    A = T * E                                    # every token picks every expert
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda") / (shape[-1] ** 0.5 if len(shape) == 2 and shape != (T, H) else 1)

    x = normal(T, H)
    w = [(normal(F, H), normal(F, H), normal(H, F)) for _ in range(E)]
    desc = P.make_desc(H, F, E, E, 0, "f32")
    off = torch.arange(0, A + 1, T, dtype=torch.int32, device="cuda")
    tok = torch.arange(T, dtype=torch.int32, device="cuda")
    src = torch.cat([tok * E + e for e in range(E)])
    y = torch.full((A, H), float("nan"), device="cuda")
    P.prism_expert_ffn(desc, x, P.WeightTable(w, []), src, off, P.alloc_workspace(desc, T), y=y)
    assert bool(torch.isfinite(y).all())
    picks = torch.cat([torch.arange(0, 130), torch.arange(T - 130, T), torch.arange(0, T, 997)]).cuda()
    for e in range(E):
        g, u, d = (m.double() for m in w[e])
        a = x[picks].double()
        z = a @ g.T
        ref = (z / (1 + torch.exp(-z)) * (a @ u.T)) @ d.T
        got = y[e * T:(e + 1) * T][picks].double()
        # 4 + 2 + F / 128 + 3 roundings of 2^-24, independent: sqrt(137) * 6e-8 = 7e-7 of a sum's norm; three sums
        assert float((got - ref).norm() / ref.norm()) <= 2e-6


def run_one_expert(x, wg, wu, wd):
    """prism_expert_ffn of one expert that takes every row of x once; numpy in, numpy out."""
    import paper_2508_12851_amd as P
    T, (F, H) = len(x), wg.shape
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    desc = P.make_desc(H, F, 1, 1, 0, "f32")
    y = P.prism_expert_ffn(desc, dev(x), P.WeightTable([(dev(wg), dev(wu), dev(wd))]),
                           torch.arange(T, dtype=torch.int32, device="cuda"),
                           torch.tensor([0, T], dtype=torch.int32, device="cuda"), P.alloc_workspace(desc, T))
    return y.cpu().numpy()


def normal_operands(T, H, F, seed=0):
    rng = np.random.default_rng([T, H, F, seed])
    x = rng.standard_normal((T, H)).astype(np.float32)
    return [x] + [(rng.standard_normal(s) / np.sqrt(s[1])).astype(np.float32) for s in ((F, H), (F, H), (H, F))]


@pytest.mark.parametrize("T,H,F", [(33, 8, 8), (70, 264, 130), (40, 2048, 40), (300, 40, 2048)])
@pytest.mark.parametrize("ex,eg,eu,ed", [
    (118, -118, -118, 0),                        # weights of which bf16 parts keep about 13 bits, ordinary sums
    (-118, 118, 118, 0),                         # the same of the tokens
    (122, -125, -125, 0),                        # weights next to the smallest normal fp32 value, and below
    (0, 0, 0, -118),                             # small weights of the down projection: all results are small
    (-40, 40, -50, 100),                         # small sums of one matrix, large weights after them
])
def test_f32_ffn_small_operands(T, H, F, ex, eg, eu, ed):
    """Operands whose bf16 parts fall below the smallest bf16 value: as good as any others (bound: test_f32_ffn_edges;
    scaled by powers of two, so that the operands are the same ones but for what falls below the smallest fp32 value,
    which the reference sees too)."""
    ops = [np.ldexp(m, e).astype(np.float32) for m, e in zip(normal_operands(T, H, F), (ex, eg, eu, ed))]
    y = run_one_expert(*ops)
    x, g, u, d = (m.astype(np.float64) for m in ops)
    z = x @ g.T
    ref = (z / (1.0 + np.exp(-z)) * (x @ u.T)) @ d.T
    assert np.linalg.norm(y - ref) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("T,H,F", [(33, 64, 40), (70, 264, 130), (300, 1024, 72)])
@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38, 1e-36, 0.0])
def test_f32_ffn_rows_do_not_depend_on_their_neighbours(T, H, F, value):
    """A token or an output column of which the products of parts are not enough must not change a bit of the others."""
    x, wg, wu, wd = normal_operands(T, H, F)
    plain = run_one_expert(x, wg, wu, wd)
    odd = x.copy()
    odd[5, :] = value                            # one whole row ...
    odd[T - 1, H // 2] = value                   # ... one element of another
    rest = np.setdiff1d(np.arange(T), [5, T - 1])
    with np.errstate(all="ignore"):
        np.testing.assert_array_equal(run_one_expert(odd, wg, wu, wd)[rest], plain[rest])
        odd = wd.copy()
        odd[3, :] = value
        odd[H - 1, F // 2] = value
        rest = np.setdiff1d(np.arange(H), [3, H - 1])
        np.testing.assert_array_equal(run_one_expert(x, wg, wu, odd)[:, rest], plain[:, rest])


def test_f32_ffn_marks_more_items_than_a_workgroup_has_marks():
    """Small rows in the first and last tiles of 271392 items, 1060 per workgroup: only their rows are redone."""
    T, H, F = 66 * 1024, 8, 8200                 # 1056 row tiles of 64 rows x 257 column tiles of h
    x, wg, wu, wd = normal_operands(T, H, F)
    plain = run_one_expert(x, wg, wu, wd)
    odd = x.copy()
    odd[[0, T - 1]] = np.float32(1e-36)
    odd[7] = np.inf
    rest = np.setdiff1d(np.arange(T), [0, 7, T - 1])
    np.testing.assert_array_equal(run_one_expert(odd, wg, wu, wd)[rest], plain[rest])


def test_f32_ffn_single_products():
    """Contractions of one term: a million products of full fp32 values, each rounded once.  Tokens and the gate are
    powers of two (silu(32) = 32 in fp32), so h = 32 W_up exactly, and a row of W_down has one element."""
    T = H = F = 1024
    rng = np.random.default_rng(11)
    x = np.eye(T, H, dtype=np.float32)
    wu = rng.standard_normal((F, H)).astype(np.float32)
    pick, wd = rng.integers(0, F, H), np.zeros((H, F), np.float32)
    wd[np.arange(H), pick] = rng.standard_normal(H)
    y = run_one_expert(x, np.full((F, H), 32, np.float32), wu, wd).astype(np.float64)
    ref = 32.0 * wu[pick, :].T.astype(np.float64) * wd[np.arange(H), pick].astype(np.float64)[None, :]
    # one rounding to fp32, 2^-24; the seven smaller products of parts (at most 2^-8 of the product each, two
    # roundings of 2^-24 apiece) add less than 14 * 2^-32, the ninth, left out, 2^-34
    assert np.all(np.abs(y - ref) <= 2.0 ** -24 * (1 + 2.0 ** -4) * np.abs(ref))


def test_f32_ffn_down_projection_of_subnormal_weights():
    """Weights so small that their bf16 parts are all zero: the sums come out as zeros and are looked at again."""
    T, H, F = 40, 72, 136
    x, wg, wu, wd = normal_operands(T, H, F)
    wd = np.ldexp(wd * np.float32(np.sqrt(F)), -139).astype(np.float32)
    y = run_one_expert(x, wg, wu, wd).astype(np.float64)
    g, u, d = (m.astype(np.float64) for m in (wg, wu, wd))
    z = x.astype(np.float64) @ g.T
    ref = (z / (1.0 + np.exp(-z)) * (x.astype(np.float64) @ u.T)) @ d.T
    # results are multiples of 2^-149, each of the F products is rounded to one, half of it at most
    assert np.abs(ref).max() > 2.0 ** -138 and np.all(np.abs(y - ref) <= F * 2.0 ** -150)


@pytest.mark.parametrize("T,H,F", [(33, 64, 40), (300, 1024, 72), (200, 72, 1024)])
def test_f32_ffn_sparse_rows(T, H, F):
    """Rows with few elements or none: most sums of a wavefront are zeros.  Bound: test_f32_ffn_edges."""
    x, wg, wu, wd = normal_operands(T, H, F)
    rng = np.random.default_rng(T)
    x[rng.random((T, H)) < 0.97] = 0
    x[::7] = 0
    wd[rng.random((H, F)) < 0.97] = 0
    y = run_one_expert(x, wg * 4, wu * 4, wd * 4)
    g, u, d = (4 * m.astype(np.float64) for m in (wg, wu, wd))
    z = x.astype(np.float64) @ g.T
    ref = (z / (1.0 + np.exp(-z)) * (x.astype(np.float64) @ u.T)) @ d.T
    assert np.linalg.norm(y - ref) <= 1e-6 * np.linalg.norm(ref) and not y[::7].any()
