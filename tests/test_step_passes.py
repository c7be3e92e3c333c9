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
// out: off_g, end of its region, slots, off_topk, total, kernels of the backward half, planes, rows of a plane, rows of all planes that there is
// room for, number of passes, then for each (at most 2000) its labels and the planes that it has labels for
extern "C" int step_plan(int64_t L, int d, int fmt, int64_t chunk, int max_B, int B, int64_t kahan_rows, int flags, int drop_thresh, int want_dx, int64_t* out) {
  elmo::Plan p{};
  p.L = L; p.d = d; p.fmt = fmt; p.chunk = (chunk + 127) / 128 * 128; p.maxB = max_B; p.max_nnz = 64 * max_B;
  p.flags = flags; p.kahan_rows = flags & ELMO_KAHAN ? (kahan_rows ? kahan_rows : L) : 0; p.drop_thresh = drop_thresh;
  elmo::lay_out(p);
  const elmo::StepPlan s = elmo::plan_step(p, elmo::round_up(B, 64), want_dx != 0);
  const elmo::Pass& ps = s.ps;
  out[0] = ps.off_g; out[1] = ps.off_g == p.off_g ? p.off_dx : ps.slots; out[2] = ps.slots; out[3] = p.off_topk; out[4] = p.total;
  out[5] = s.kernels; out[6] = s.planes; out[7] = s.plane_rows; out[8] = p.dx_rows;
  int64_t n = 0, c0 = 0, largest = 0;
  for (; c0 < L && n < 2000; c0 += ps.take(L - c0), ++n) {
    const int64_t labels = ps.take(L - c0), head = std::max<int64_t>(0, std::min(labels, p.kahan_rows - c0));
    const int64_t slabs = (labels + 31) / 32, per = (slabs + s.slices - 1) / s.slices;    // as k_dx cuts them
    out[10 + 2 * n] = labels;
    out[11 + 2 * n] = s.one_pass() ? std::max(s.groups(head), s.groups(labels - head)) : (slabs + per - 1) / per;
    largest = std::max(largest, labels);
  }
  out[9] = n;
  return c0 == L && largest == ps.largest(L) ? 0 : -1;
}
"""
SEPARATE, ONE_PASS_256, ONE_PASS_128 = 0, 1, 2
SR, KAHAN = 1, 2


def load(tmp):
    (tmp / "shim.cpp").write_text(SHIM)
    lib = str(tmp / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2510_11168_amd", "csrc"), "-o", lib, str(tmp / "shim.cpp")], check=True)
    f = ctypes.CDLL(lib).step_plan
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                  ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]

    def passes(L, d, fmt, chunk, B, max_B=None, kahan_rows=0, flags=SR, drop=0, want_dx=True):
        out = (ctypes.c_int64 * 4200)()
        assert f(L, d, fmt, chunk, max_B or B, B, kahan_rows, flags, drop, int(want_dx), out) == 0
        n = out[9]
        return dict(off=out[0], end=out[1], slots=out[2], off_topk=out[3], total=out[4], kernels=out[5], planes=out[6], plane_rows=out[7],
                    dx_rows=out[8], labels=list(out[10:10 + 2 * n:2]), filled=list(out[11:11 + 2 * n:2]))
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
        if L > 1900 * max(chunk, 1):
            chunk = L // 1900 + 1
        kahan = rng.random() < 0.5
        r = passes(L, d, fmt, chunk, B, max_B, L // 3 // 128 * 128 if kahan and rng.random() < 0.5 else 0, SR | KAHAN if kahan else SR,
                   64 if rng.random() < 0.2 else 0, rng.random() < 0.8)
        n, chunk128, Bp = r["labels"], (chunk + 127) // 128 * 128, (B + 63) // 64 * 64
        assert sum(n) == L and all(x % 128 == 0 for x in n[:-1]) and all(x >= min(chunk128, L) for x in n[:-1])
        # whole tiles of 128 labels
        assert r["off"] + (max(n) + 127) // 128 * 128 * Bp * 2 <= r["end"]
        # every plane of partial sums has its room, and is written by some pass
        assert r["planes"] * r["plane_rows"] <= r["dx_rows"] and max(r["filled"]) <= r["planes"]
        # tile losses of 128 x 128 tiles, behind everything else
        assert r["slots"] == 0 or (r["off_topk"] <= r["slots"] and r["slots"] + (L + 127) // 128 * ((Bp + 127) // 128) * 4 <= r["total"])


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("B", [2048, 3000])
def test_an_input_gradient_that_is_not_asked_for_is_not_priced(passes, B, fmt):
    """60000 labels at d = 768 go in three passes: the input gradient's slabs favour a shorter last one, the two launches
    that are left without dX equal ones (2 to 5 % faster)."""
    assert passes(60000, 768, fmt, 16384, B)["labels"] == [21760, 21760, 16480]
    assert passes(60000, 768, fmt, 16384, B, want_dx=False)["labels"] == [20096, 20096, 19808]


@pytest.mark.parametrize("L,d,fmt,chunk,B,n", [(1500000, 640, 0, 16384, 32, 16), (562459, 640, 1, 16384, 25, 6), (1000000, 768, 1, 30000, 160, 19),
                                             (1202307, 768, 1, 16384, 129, 23)])
def test_one_pass_heads_are_not_cut_for_update_tiles(passes, L, d, fmt, chunk, B, n):
    """A pass of a one-pass kernel has no waves of update tiles to fill; what it costs besides its labels is its launches and planes."""
    r = passes(L, d, fmt, chunk, B)
    assert (r["kernels"], len(r["labels"])) == (ONE_PASS_128, n)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("L,B", [(4097, 16), (5000, 128), (8192, 64)])
def test_one_label_tile_per_workgroup_where_there_are_cus(passes, L, B, fmt):
    """An update without an input gradient has no planes to write: up to 256 tiles of 32 labels each has a workgroup of its own at d = 256."""
    r = passes(L, 256, fmt, L, B, want_dx=False)
    assert (r["kernels"], r["labels"], r["filled"]) == (ONE_PASS_256, [L], [-(-L // 32)])


def test_heads_of_the_gpu_tests_split_as_they_say(passes):
    """The GPU tests of later passes and of single kernels are worth something only while their heads really go that way."""
    gpu = pytest.importorskip("test_gpu_shapes")
    kernels = {"separate": SEPARATE, "256": ONE_PASS_256, "128": ONE_PASS_128}
    for kernel, B, d, L, chunk, kahan_rows, n, first, last in gpu.PLANES:
        r = passes(L, d, gpu.o.E4M3, chunk, B, kahan_rows=kahan_rows, flags=gpu.SR | (gpu.KA if kahan_rows else 0))
        assert (r["kernels"], len(r["labels"]), r["filled"][0], r["filled"][-1]) == (kernels[kernel], n, first, last), (r, B, d, L)
    for kernel, fmt, flags, B, d, L, chunk, kahan_rows, T, wd, n in gpu.SEVERAL:
        for ch, several in ((chunk, n), (L, 1)):
            r = passes(L, d, fmt, ch, B, kahan_rows=kahan_rows, flags=flags, drop=T)
            assert (r["kernels"], len(r["labels"])) == (kernels[kernel], several), (r["kernels"], len(r["labels"]), fmt, flags, B, d, L)
    for kernel, B, d, L, kahan_rows in gpu.ONE_PASS:
        for fmt, flags, T, wd in gpu.ONE_PASS_MODES:
            r = passes(L, d, fmt, L, B, kahan_rows=kahan_rows if flags & gpu.KA else 0, flags=flags, drop=T)
            no_room = T and fmt == gpu.o.BF16 and flags & gpu.KA
            assert r["kernels"] == (ONE_PASS_128 if no_room else kernels[kernel]), (r, fmt, flags, B, d, L)
