"""How a step splits a head into passes (csrc/plan.h, host arithmetic only, compiled here with the host compiler): the passes
cover the labels, their gradients fit where they are put, and the launches that are priced are those that are made."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "plan.h"
// out: off_g, end of its region, slots, off_topk, total, number of passes, then the passes' labels (at most 4096)
extern "C" int step_passes(int64_t L, int d, int fmt, int64_t chunk, int max_B, int B, int kahan_bf16_drop, int want_dx, int64_t* out) {
  elmo::Plan p{};
  p.L = L; p.d = d; p.fmt = fmt; p.chunk = (chunk + 127) / 128 * 128; p.maxB = max_B; p.max_nnz = 64 * max_B;
  elmo::lay_out(p);
  const int Bp = elmo::round_up(B, 64);
  const bool small = Bp <= 128 && d % 256 == 0 && !kahan_bf16_drop;
  const elmo::Pass ps = elmo::choose_pass(p, Bp, small, want_dx != 0);
  out[0] = ps.off_g; out[1] = ps.off_g == p.off_g ? p.off_dx : ps.slots; out[2] = ps.slots; out[3] = p.off_topk; out[4] = p.total;
  int64_t n = 0, c0 = 0;
  for (; c0 < L && n < 4096; c0 += ps.take(L - c0)) out[6 + n++] = ps.take(L - c0);
  out[5] = n;
  int64_t largest = 0;
  for (int i = 0; i < n; ++i) largest = out[6 + i] > largest ? out[6 + i] : largest;
  return c0 == L && largest == ps.largest(L) ? 0 : -1;
}
"""


def load(tmp):
    (tmp / "shim.cpp").write_text(SHIM)
    lib = str(tmp / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2510_11168_amd", "csrc"), "-o", lib, str(tmp / "shim.cpp")], check=True)
    f = ctypes.CDLL(lib).step_passes
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int64)]

    def passes(L, d, fmt, chunk, B, max_B=None, separate=False, want_dx=True):
        out = (ctypes.c_int64 * 4200)()
        assert f(L, d, fmt, chunk, max_B or B, B, int(separate), int(want_dx), out) == 0
        return dict(off=out[0], end=out[1], slots=out[2], off_topk=out[3], total=out[4], labels=list(out[6:6 + out[5]]))
    return passes


@pytest.fixture(scope="module")
def passes(tmp_path_factory):
    return load(tmp_path_factory.mktemp("step_passes"))


def test_passes_cover_the_labels_and_their_gradients_fit(passes):
    rng = random.Random(1)

    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))
    for _ in range(3000):
        L, d, fmt = log_int(1, 3_000_000), 128 * rng.randint(1, 16), rng.randint(0, 1)
        max_B = log_int(1, 8192)
        B = rng.choice([max_B, log_int(1, max_B)])
        chunk = rng.choice([1, 128, log_int(1, L), L, 2 * L])
        if L > 2000 * max(chunk, 1):
            chunk = L // 2000 + 1
        r = passes(L, d, fmt, chunk, B, max_B, rng.random() < 0.2, rng.random() < 0.8)
        n, chunk128, Bp = r["labels"], (chunk + 127) // 128 * 128, (B + 63) // 64 * 64
        assert sum(n) == L and all(x % 128 == 0 for x in n[:-1]) and all(x >= min(chunk128, L) for x in n[:-1])
        # whole tiles of 128 labels, and the last rows are read 512 bytes wide
        assert r["off"] + (max(n) + 127) // 128 * 128 * Bp * 2 + 4096 <= r["end"]
        # tile losses of 128 x 128 tiles, behind everything else
        assert r["slots"] == 0 or (r["off_topk"] <= r["slots"] and r["slots"] + (L + 127) // 128 * ((Bp + 127) // 128) * 4 <= r["total"])


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("B", [2048, 3000])
def test_an_input_gradient_that_is_not_asked_for_is_not_priced(passes, B, fmt):
    """60000 labels at d = 768 go in three passes: the input gradient's slabs favour a shorter last one, the two launches
    that are left without dX equal ones (2 to 5 % faster)."""
    assert passes(60000, 768, fmt, 16384, B)["labels"] == [21760, 21760, 16480]
    assert passes(60000, 768, fmt, 16384, B, want_dx=False)["labels"] == [20096, 20096, 19808]


def planes(labels, B, d, kahan_rows=0):
    """Planes of input-gradient partials that a pass over `labels` labels fills: label groups of 32-label tiles for a small
    batch, slices of 64-label slabs otherwise."""
    Bp = (B + 63) // 64 * 64
    if Bp <= 128 and d % 256 == 0:
        def groups(n):
            t = -(-n // 32)
            return -(-t // -(-t // max(1, 256 // (d // 256))))
        parts = [n for n in (min(kahan_rows, labels), labels - min(kahan_rows, labels)) if n]
        return max(groups(n) for n in parts)
    slabs = -(-labels // 64)
    S = min(max(1, 256 // (-(-Bp // 256) * -(-d // 256))), 64, slabs)
    return -(-slabs // -(-slabs // S))


def test_heads_of_the_gpu_tests_split_as_they_say(passes):
    """The GPU tests of later passes are worth something only while their heads really go in several."""
    gpu = pytest.importorskip("test_gpu_shapes")
    for B, d, L, chunk, kahan_rows, n, first, last in gpu.PLANES:
        labels = passes(L, d, gpu.o.E4M3, chunk, B)["labels"]
        assert len(labels) == n and planes(labels[0], B, d, kahan_rows) == first and planes(labels[-1], B, d, kahan_rows) == last, (labels, B, d, L)
    for fmt, flags, B, d, L, chunk, kahan_rows, T, wd, n in gpu.SEVERAL:
        separate = T and fmt == gpu.o.BF16 and flags & gpu.KA
        assert len(passes(L, d, fmt, chunk, B, separate=bool(separate))["labels"]) == n, (fmt, flags, B, d, L)
        assert len(passes(L, d, fmt, L, B, separate=bool(separate))["labels"]) == 1
