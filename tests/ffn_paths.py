"""The tile rules of csrc/ffn_paths.h, compiled for the host: which path a batch takes, without a GPU."""
import ctypes
import functools
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2508_12851_amd", "csrc", "ffn_paths.h")

_SOURCE = """
#include "ffn_paths.h"
static prism_layer_desc desc(const int* a) {
  prism_layer_desc d{};
  d.hidden = a[0]; d.ffn = a[1]; d.n_experts = a[2]; d.top_k = a[3]; d.n_shared = a[4];
  d.dtype = PRISM_BF16; d.weight_layout = a[5];
  return d;
}
extern "C" int ffn_path_of(const int* a, int T) { return (int)prism::ffn_path(desc(a), T); }
extern "C" int packs_rows(const int* a, int T) {
  return prism::ffn_path(desc(a), T) == prism::FfnPath::kPrefill && prism::pack_rows_pays(desc(a), T);
}
extern "C" int cuts_last_round(const int* a, int T) {
  return prism::ffn_path(desc(a), T) == prism::FfnPath::kPrefill && prism::down_slicing_applies(desc(a), T);
}
"""


@functools.lru_cache(maxsize=1)
def _lib():
    d = tempfile.mkdtemp(prefix="ffn_paths_")
    src, so = os.path.join(d, "p.cpp"), os.path.join(d, "p.so")
    with open(src, "w") as f:
        f.write(_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.dirname(HEADER),
                    "-I", os.path.join(ROOT, "include"), src, "-o", so], check=True, timeout=120)
    lib = ctypes.CDLL(so)
    text = open(HEADER).read()
    body = text[text.index("enum class FfnPath {"):]
    lib.names = re.findall(r"^\s*(k\w+)", body[:body.index("};")], re.M)
    return lib


def _args(H, F, E, k, S=0, tiled=False):
    return (ctypes.c_int * 6)(H, F, E, k, S, int(tiled))


def ffn_path(H, F, E, k, S, T, tiled=False):
    """Name of the path of a bf16 batch of T tokens."""
    return _lib().names[_lib().ffn_path_of(_args(H, F, E, k, S, tiled), T)]


def packs_rows(H, F, E, k, S, T, tiled=False):
    return bool(_lib().packs_rows(_args(H, F, E, k, S, tiled), T))


def cuts_last_round(H, F, E, k, S, T, tiled=False):
    return bool(_lib().cuts_last_round(_args(H, F, E, k, S, tiled), T))
