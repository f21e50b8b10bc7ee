"""CPU: the rules that choose the tiles of the expert FFN (csrc/ffn_paths.h)."""
import pytest

from ffn_paths import cuts_last_round, ffn_path, packs_rows


@pytest.mark.parametrize("H,F,E,k,S,T,tiled,path", [
    (4096, 14336, 8, 2, 0, 32, True, "kDecodeTiled"),
    (4096, 14336, 8, 2, 0, 64, False, "kDecode"),
    (64, 64, 8, 2, 0, 64, False, "kDecodeShort"),
    (4096, 14336, 8, 2, 0, 300, True, "kSplitWide"),
    (1024, 4096, 8, 2, 0, 300, False, "kSplitSquare"),
    (2048, 1408, 60, 4, 4, 333, True, "kFewRows128"),
    (1024, 1024, 256, 8, 0, 100, True, "kFewRows64"),
    (4096, 14336, 8, 2, 0, 4096, True, "kPrefill"),
    (64, 64, 8, 2, 0, 65, False, "kPrefillShort"),
])
def test_path_of_the_usual_sizes(H, F, E, k, S, T, tiled, path):
    assert ffn_path(H, F, E, k, S, T, tiled) == path


def test_cut_and_copy_of_the_usual_sizes():
    assert cuts_last_round(4096, 14336, 8, 2, 0, 4096) and packs_rows(4096, 14336, 8, 2, 0, 4096, True)
    assert not cuts_last_round(2048, 1408, 60, 4, 4, 8192) and not packs_rows(2048, 1408, 60, 4, 4, 8192)
    assert cuts_last_round(4096, 4096, 16, 2, 0, 400)       # too many row tiles for the split path


@pytest.mark.parametrize("T", [65, 128, 129, 200, 256])
@pytest.mark.parametrize("H,F,E,k,S", [
    (4096, 14336, 8, 2, 0), (4096, 14336, 8, 1, 0), (4096, 4096, 8, 2, 0), (3072, 8192, 8, 2, 0), (2304, 9216, 8, 2, 0),
    (2560, 10240, 8, 2, 0), (2048, 8192, 4, 2, 0), (2048, 4096, 16, 2, 1), (1536, 6144, 8, 2, 0), (1024, 2048, 8, 2, 0),
])
def test_weight_streaming_batches_take_the_small_tiles(H, F, E, k, S, T):
    """Few hosted experts (the host cannot know) leave most of the machine idle in wider tiles."""
    assert ffn_path(H, F, E, k, S, T) == "kStream"


@pytest.mark.parametrize("H,F,E,k,S,T,path", [
    (2048, 1408, 256, 1, 0, 1024, "kFewRows64"),      # a peer's rows: few hosted experts may get them all
    (2048, 1408, 256, 1, 0, 1025, "kFewRows128"),
    (2048, 1408, 256, 1, 0, 2560, "kFewRows128"),
    (2048, 1408, 256, 1, 0, 2561, "kPrefill"),
    (2048, 1408, 64, 1, 0, 4096, "kPrefill"),
    (1024, 1024, 256, 8, 0, 512, "kFewRows64"),       # 16 rows per expert
    (1024, 1024, 256, 8, 0, 513, "kFewRows128"),
    (1024, 1024, 256, 8, 0, 3584, "kFewRows128"),     # 112 rows per expert
    (1024, 1024, 256, 8, 0, 3585, "kPrefill"),
    (2048, 1408, 60, 4, 4, 2150, "kPrefill"),
    (2048, 1408, 64, 6, 2, 1500, "kPrefill"),
    (896, 448, 32, 6, 0, 768, "kFewRows128"),         # small layers, 144 rows per expert: (18 + 16) x 4 full-tile items
    (896, 448, 32, 6, 0, 769, "kPrefill"),
    (2048, 448, 32, 6, 0, 682, "kFewRows128"),        # 128 rows, 32 x 8 items
    (2048, 448, 32, 6, 0, 683, "kPrefill"),           # 33 x 8
])
def test_lines_of_the_few_rows_tiles(H, F, E, k, S, T, path):
    assert ffn_path(H, F, E, k, S, T) == path


@pytest.mark.parametrize("H,T,path", [
    (1024, 257, "kSplitSquare"), (1024, 512, "kSplitSquare"), (1088, 448, "kSplitSquare"), (1088, 449, "kSplitWide"),
    (2560, 257, "kSplitSquare"), (2560, 448, "kSplitSquare"), (2560, 449, "kSplitWide"), (2560, 512, "kSplitWide"),
    (2624, 257, "kSplitWide"), (4096, 512, "kSplitWide"),
])
def test_lines_of_the_split_tiles(H, T, path):
    assert ffn_path(H, 8192, 8, 2, 0, T) == path


@pytest.mark.parametrize("H,F,T,tiled,packs", [
    (4096, 14336, 512, True, False), (4096, 14336, 513, True, True),
    (4096, 14336, 513, False, False), (4096, 14336, 936, False, False), (4096, 14336, 937, False, True),
    (4096, 4096, 800, False, False), (2048, 8192, 655, True, False), (2048, 8192, 656, True, True),
])
def test_lines_of_the_token_row_copy(H, F, T, tiled, packs):
    assert packs_rows(H, F, 8, 2, 0, T, tiled) == packs


def test_random_cases_span_the_paths():
    """The random parity cases reach every path, those of wide and of streaming layers the ones they are drawn for."""
    from collections import Counter

    from random_cases import N_STREAMING_CASES, N_WIDE_CASES, draw_case, draw_streaming_case, draw_wide_case

    def args(kw, tiled):
        return kw["H"], kw["F"], kw["E"], kw["k"], kw["S"], kw["T"], tiled

    layers = [(kw, tiled) for kw, _, tiled in map(draw_case, range(32)) if kw["dtype"] == "bf16"]
    wide = list(map(draw_wide_case, range(N_WIDE_CASES)))
    streaming = list(map(draw_streaming_case, range(N_STREAMING_CASES)))
    assert all(cuts_last_round(*args(*c)) for c in wide)
    count = Counter(ffn_path(*args(*c)) for c in streaming)
    for path in ("kDecode", "kDecodeTiled", "kStream", "kSplitSquare", "kSplitWide"):
        assert count[path] >= 2, count
    assert {ffn_path(*args(*c)) for c in layers + wide + streaming} == {
        "kDecodeTiled", "kDecode", "kDecodeShort", "kStream", "kSplitSquare", "kSplitWide", "kFewRows64",
        "kFewRows128", "kPrefill", "kPrefillShort"}
