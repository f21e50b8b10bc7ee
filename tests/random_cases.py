"""Seeded random layer shapes, batch sizes, masks, gate conventions and weight layouts (all
within the library's documented limits), shared by the GPU parity test that runs them and
the CPU test that settles which error measure each of them is held to.  No arithmetic of the
method lives here."""
import os

import numpy as np

N_CASES = int(os.environ.get("PRISM_RANDOM_CASES", "32"))   # more for a longer hunt
N_WIDE_CASES, N_STREAMING_CASES = 12, 24

# Cases whose layer output is held to the per-row form of the error measure, max |a - ref| /
# (|ref| + rms of the token's own row), instead of the whole-batch rms: their tokens differ by
# orders of magnitude in size (256 experts, a random mask, gates that are not renormalised),
# and the bf16 roundings the layer is defined with, carried out in otherwise exact arithmetic,
# already exceed the 2e-2 bar against the whole-batch rms.  tests/test_error_measure.py proves
# this membership on the CPU, case by case, and that no other case needs it.
PER_ROW_CASES = frozenset({12})
PER_ROW_STREAMING_CASES = frozenset({12})   # the same for draw_streaming_case: 234 of 1672 picks hosted


def draw_case(i):
    """-> (make_config overrides, gate mode, tiled weights?) of random case i."""
    rng = np.random.default_rng(7000 + i)
    pick = lambda seq: seq[int(rng.integers(0, len(seq)))]
    f32 = i % 8 == 7
    E = pick([2, 3, 5, 8, 12, 16, 40, 60, 64, 100, 256])
    k = int(rng.integers(1, min(8, E) + 1))
    S = pick([0, 0, 0, 1, 2, 4])
    if f32:
        H, F = pick([8, 72, 136]), pick([24, 200])
    else:
        H, F = pick([64, 128, 192, 256, 320, 512, 1024]), pick([64, 128, 192, 448, 1024, 1088, 1536])
    T = int(pick([rng.integers(1, 65), rng.integers(65, 513), rng.integers(513, 1500)]))
    if f32:
        T = min(T, 200)
    # keep the fp64 oracle to a few seconds
    while T * (k + S) * H * F > 3e9 and T > 1:
        T = max(1, T // 2)
    n_local = int(pick([0, E, rng.integers(0, E + 1), rng.integers(0, E + 1)]))
    return dict(dtype="f32" if f32 else "bf16", T=T, H=H, F=F, E=E, k=k, S=S, n_local=n_local,
                n_swapped=0, bias_group_tokens=pick([0, 0, 16, 64, 128]), mask_kind=pick(["top", "random"]),
                zipf_s=pick([0.0, 1.0, 1.2]), seed=100 + i), \
        pick(["renormalized", "softmax_all"]), (not f32) and H % 32 == 0 and F % 32 == 0 and bool(rng.integers(0, 2))


def draw_wide_case(i):
    """Random prefill batches of layers with a long down-projection contraction (F >= 4096), where
    the schedule cuts a partly filled last round of work items into slices: few experts, so that
    the number of row tiles -- and with it the number of items left over -- varies from case to case."""
    rng = np.random.default_rng(9000 + i)
    pick = lambda seq: seq[int(rng.integers(0, len(seq)))]
    E = pick([2, 3, 4, 6, 8])
    k = int(rng.integers(1, min(3, E) + 1))
    S = pick([0, 0, 1])
    H, F = pick([128, 256, 512]), pick([4096, 4160, 4608, 5120])
    T = int(rng.integers(513, 2600))         # smaller batches split the whole down projection instead
    while T * (k + S) * H * F > 3e9 and T > 513:
        T = max(513, T * 3 // 4)
    n_local = int(pick([E, E, max(1, E - 1), int(rng.integers(1, E + 1))]))
    return dict(dtype="bf16", T=T, H=H, F=F, E=E, k=k, S=S, n_local=n_local, n_swapped=0,
                bias_group_tokens=pick([0, 0, 256]), mask_kind=pick(["top", "random"]),
                zipf_s=pick([0.0, 1.0]), seed=300 + i), bool(rng.integers(0, 2))


def draw_streaming_case(i):
    """Random batches of up to 512 tokens of layers wide enough for the paths that stream the
    weights (H >= 256, F >= 1024): decode tiles up to 64 tokens, 128 x 128 tiles dealt item by item up to
    256, 128 x 128 or 128 x 256 ones beyond, by the hidden size, each with the down projection split into a
    number of slices that the schedule builder picks from the number of experts that received tokens --
    which the expert count, the mask and the popularity skew vary from case to case."""
    rng = np.random.default_rng(12000 + i)
    pick = lambda seq: seq[int(rng.integers(0, len(seq)))]
    E = pick([2, 4, 8, 8, 16, 32])
    k = int(rng.integers(1, min(4, E) + 1))
    S = pick([0, 0, 1])
    H, F = pick([256, 512, 1024, 2048, 2624, 3072]), pick([1024, 1536, 2048, 4096])
    T = int(pick([rng.integers(1, 65), rng.integers(65, 257), rng.integers(257, 513), rng.integers(257, 513)]))
    n_local = int(pick([E, max(1, E - 1), int(rng.integers(1, E + 1))]))
    return dict(dtype="bf16", T=T, H=H, F=F, E=E, k=k, S=S, n_local=n_local, n_swapped=0,
                bias_group_tokens=pick([0, 0, 32]), mask_kind=pick(["top", "random"]),
                zipf_s=pick([0.0, 1.0, 2.0]), seed=500 + i), bool(rng.integers(0, 2))
