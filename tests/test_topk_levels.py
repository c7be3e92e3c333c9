"""The level rule of top-k scoring (csrc/topk_levels.h, host arithmetic only, compiled here with the host compiler):
the levels cover the labels, and a row's candidate list holds what a level appends also where the scores after the first
level are more spread than those in it."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "topk_levels.h"
extern "C" int topk_level_ends(int64_t L, int Bp, int k, int slabs, int64_t* ends, int* list) {
  const elmo::TopkLevels t = elmo::topk_levels(L, Bp, k, slabs);
  for (int i = 0; i <= t.n; ++i) ends[i] = t.end(i);
  *list = elmo::topk_list(Bp);
  return t.n + 1;
}
"""


@pytest.fixture(scope="module")
def level_ends(tmp_path_factory):
    d = tmp_path_factory.mktemp("topk_levels")
    (d / "shim.cpp").write_text(SHIM)
    lib = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2510_11168_amd", "csrc"), "-o", lib, str(d / "shim.cpp")], check=True)
    f = ctypes.CDLL(lib).topk_level_ends
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int)]

    def ends(L, Bp, k, slabs=6):
        e, n = (ctypes.c_int64 * 256)(), ctypes.c_int()
        m = f(L, Bp, k, slabs, e, ctypes.byref(n))
        return list(e[:m]), n.value
    return ends


def test_levels_cover_the_labels(level_ends):
    for L in (1, 127, 4095, 4096, 4097, 8192, 131072, 133080, 1 << 20, 3_000_001, 1 << 31):
        for Bp in (64, 128, 192, 256, 1024, 4096, 65536):
            for k in (1, 2, 7, 10, 100, 128):
                if k > L:
                    continue
                ends, n = level_ends(L, Bp, k, 1 + (L + k) % 64)
                assert n == (8192 if Bp <= 128 else 4096)
                assert ends[0] == min(L, 4096) and ends[-1] == L and len(ends) <= 24
                assert all(a < b for a, b in zip(ends, ends[1:])) or ends == [L]      # no level is empty
                assert all(e % 256 == 0 for e in ends[:-1])                           # and all but the last are whole label tiles


@pytest.mark.parametrize("Bp", [64, 128, 256, 1024])
@pytest.mark.parametrize("spread", [1.0, 1.5, 2.0])
def test_lists_hold_what_a_level_appends(level_ends, Bp, spread):
    """Scores N(0, 1) for the first 4096 labels and N(0, spread) for the others, sixteen rows: at every level the k best of
    the levels before and the scores above the k-th of them fit the row's list."""
    rng = np.random.default_rng(int(10 * spread))
    worst = {}
    for _ in range(16):
        z = rng.standard_normal(3_000_000, dtype=np.float32)
        z[4096:] *= np.float32(spread)
        for L in (131072, 524288, 670091, 1_000_000, 3_000_000):
            for k in (1, 5, 10, 34, 100, 128):
                ends, n = level_ends(L, Bp, k)
                top = np.partition(z[:ends[0]], -k)[-k:]
                for a, e in zip(ends, ends[1:]):
                    passed = z[a:e][z[a:e] > top.min()]
                    worst[L, k] = max(worst.get((L, k), 0), (k + len(passed)) / n)
                    top = np.partition(np.concatenate([top, passed]), -k)[-k:]
    assert max(worst.values()) <= 1.0, {c: round(w, 2) for c, w in worst.items() if w > 1.0}


@pytest.mark.parametrize("slabs,L,rows,k,levels", [
    # d = 768 (12 slabs: BF16, 6: E4M3); levels after the first, the fastest measured
    (12, 50000, 256, 1, 1), (6, 50000, 512, 1, 1), (12, 131072, 256, 100, 2), (12, 140000, 256, 10, 2), (6, 140000, 256, 5, 2), (12, 140000, 1024, 34, 3),
    (12, 131072, 1024, 100, 3), (6, 131072, 2048, 100, 4), (6, 3000000, 1024, 100, 5), (12, 670091, 64, 10, 2),
])
def test_number_of_levels_follows_the_measured_times(level_ends, slabs, L, rows, k, levels):
    assert len(level_ends(L, rows, k, slabs)[0]) == levels + 1
