"""GPU parity at the sizes where a kernel's split of the work can go wrong: edges of tiles, remainders, the
smallest and largest of a range.  Oracle, inputs and bounds as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

from oracle import elmo_oracle as o
from paper_2510_11168_amd import synth
from test_gpu_parity import Case, assert_dx_close, assert_far_misses_are_tiny, b, check_step, ordered, say  # noqa: F401  (b is the module's fixture)

pytestmark = pytest.mark.gpu


def batch(L, d, B, seed=5, rule="lognormal5"):
    rng = np.random.default_rng(seed)
    X = synth.make_x(rng, B, d)
    indptr, indices = synth.ZipfLabels(L, 1.0).draw_csr(rng, B, rule)
    return X, indptr, indices


# (kernels of the backward half, B, d, L, chunk, kahan_rows, passes of the step, planes that its first pass has labels for, its last):
# test_step_passes.py holds the library to the first and the last three.  "256" / "128": one pass over 256- or 128-column tiles.
PLANES = [
    ("256", 40, 256, 246016, 9600, 0, 3, 234, 256),         # a later pass has more label groups than the first
    ("256", 40, 512, 8193, 8193, 0, 1, 86, 86),             # the fewest labels; groups of three tiles, the last of two, one label in its last
    ("256", 100, 256, 20000, 20000, 128, 1, 207, 207),      # one pass in two parts, the first with four groups for 207 planes
    ("128", 40, 512, 128 * 3 + 5, 128, 0, 1, 13, 13),       # fewer label tiles than groups; a ragged last tile
    ("128", 100, 256, 1024, 1024, 128, 1, 28, 28),          # one pass in two parts, the first with fewer groups than the second
    ("128", 130, 384, 70, 1000, 0, 1, 3, 3),
    ("separate", 300, 128, 65624, 6400, 0, 2, 61, 64),      # 64 label slices, three of them without labels in the first pass
    ("separate", 300, 384, 70, 1000, 0, 1, 2, 2),           # three label slabs on two slices, half a column tile
    ("separate", 130, 128, 70, 1000, 0, 1, 2, 2),
]


@pytest.mark.parametrize("B,d,L,chunk,kahan_rows,passes", [row[1:7] for row in PLANES])
def test_input_gradient_planes(b, B, d, L, chunk, kahan_rows, passes):  # noqa: F811
    """The first launch of a step writes every plane of partial sums that the end adds up, whether it has labels
    for it or not; later launches add to them."""
    fmt, flags = o.E4M3, o.FLAG_SR | (o.FLAG_KAHAN if kahan_rows else 0)
    case = Case(b, L, d, fmt, chunk, flags, B, w_std=0.05, seed=8, kahan_rows=kahan_rows)
    case.head.workspace.fill_(0x7F)         # whatever the planes held before must not matter
    X, indptr, indices = batch(L, d, B)
    dX, _ = case.step(X, indptr, indices, 0.05, 1, 2)
    assert case.passes == passes
    ref, _ = o.input_gradient_rows(case.W0, X, indptr, indices, fmt, np.arange(B))
    assert_dx_close(dX, ref, 6e-2)


@pytest.mark.parametrize("B,per_row,L", [
    (1, 1, 128),            # one positive, one bin
    (129, 9, 128 * 3 + 1),  # one more row than a pass of the index covers, one more positive than the lanes of a row
    (1030, 5, 300000),      # rows beyond one batch of passes, more bins than threads
    (128, 256, 20000),      # 32768 positives by one workgroup
    (256, 256, 20000),      # 65536: the separate index kernels
])
def test_label_index_sizes(b, B, per_row, L):  # noqa: F811
    """The positives of a batch reach their labels whatever the number of rows, positives and bins: the weights are the
    oracle's on labels drawn from the whole head, most of them with positives, and the loss where that is all labels
    (every positive of larger heads: test_every_positive_reaches_its_label)."""
    d, fmt, flags = 128, o.E4M3, 0
    case = Case(b, L, d, fmt, L, flags, B, max_nnz=B * per_row, w_std=0.05, seed=4)
    rng = np.random.default_rng(6)
    X = synth.make_x(rng, B, d)
    indices = np.concatenate([np.sort(rng.choice(L, size=per_row, replace=False)) for _ in range(B)]).astype(np.int32)
    indptr = (np.arange(B + 1) * per_row).astype(np.int32)
    case.head.workspace.fill_(0x7F)
    _, loss = case.step(X, indptr, indices, 0.05, 0, 0, want_dx=False)
    hot = np.unique(indices)
    rows = np.unique(np.concatenate([rng.choice(hot, min(len(hot), 3500), replace=False), rng.integers(0, L, 300), np.arange(min(L, 128)), np.arange(max(0, L - 128), L)]))
    rows = np.arange(L) if L <= 4096 else rows
    ref = o.head_step(case.W0[rows], None, X, indptr, indices, 0.05, 0, 0, fmt, flags, label_ids=rows)
    Wn = case.W()[rows]
    assert np.mean(Wn == ref["W_new"]) >= 0.999
    if len(rows) == L:
        assert abs(loss - ref["loss"]) <= 2e-3 * abs(ref["loss"])


def uneven(B, lens, L, seed=3):
    """CSR of rows of the given lengths, ids spread over the whole head, the first and the last label in every long row."""
    rng = np.random.default_rng(seed)
    rows = []
    for n in lens:
        r = np.sort(rng.choice(L, size=n, replace=False))
        if n > 1:
            r[0], r[-1] = 0, L - 1
        rows.append(r)
    assert len(rows) == B
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.concatenate(rows + [np.zeros(0, np.int64)]).astype(np.int32)


def index_case(B, what, L):
    rng = np.random.default_rng(9)
    lens = {"none": np.zeros(B, int), "one": np.ones(B, int), "five": np.full(B, 5), "eight": np.full(B, 8),
            "eight and one more": np.full(B, 8) + (np.arange(B) == B // 2), "every third": np.arange(B) % 3 // 2 * 7,
            "most": np.full(B, 65536 // B), "long": np.where(np.arange(B) % 128 == 5, 1000, 1), "longer": np.where(np.arange(B) % 128 == 5, 3000, 1), "mixed": rng.integers(0, 40, B)}[what]
    return uneven(B, lens, L)


@pytest.mark.parametrize("B,what,L", [
    (1, "one", 128), (1, "most", 70000), (2, "none", 300), (7, "mixed", 5000), (128, "most", 20000), (129, "five", 385),
    (300, "every third", 70000),                                    # empty rows
    (1024, "long", 100000), (1024, "longer", 100000),               # rows of 1000 positives among rows of one; 3000: the separate kernels
    (400, "mixed", 300000), (1030, "five", 300000),                 # more rows than one round of the workgroup
    (1500, "one", 9000), (1700, "one", 9000), (2000, "eight", 9000),    # on both sides of the line to the separate kernels
    (16, "mixed", 4194304), (3000, "one", 4194304), (16, "mixed", 4194305),   # the most bins, and one more
])
def test_every_positive_reaches_its_label(b, B, what, L):  # noqa: F811
    """Zero weights make every logit zero and G = 1/2 - Y exactly; with inputs of +-1/8 that cancel in pairs the new weights
    lr (Y^T X - sum(X) / 2) are exact, so each of the L x d shows exactly the positives of its label."""
    d, lr = 128, 0.5
    indptr, indices = index_case(B, what, L)
    rng = np.random.default_rng(2)
    X = rng.choice([-0.125, 0.125], (B, d)).astype(np.float32)
    X[1::2] = -X[:B // 2 * 2:2]
    head = b.Head(L, d, o.BF16, 131072, 0, B, max(len(indices), 1))
    head.workspace.fill_(0x7F)
    Xd, ip, ix = (torch.from_numpy(v).to("cuda:0") for v in (o.round_bf16(X).view(np.int16), indptr, indices))
    head.step(Xd, ip, ix, lr, 0, 0)
    Xf = torch.from_numpy(X).to("cuda:0")
    want = (-lr / 2 * Xf.double().sum(0)).float().expand(L, d).clone()
    want.index_add_(0, ix.long(), lr * Xf[torch.repeat_interleave(torch.arange(B, device="cuda:0"), ip.diff().long())])
    assert torch.equal(head.weights().view(torch.bfloat16).float(), want.bfloat16().float())


def test_malformed_rows_are_skipped_and_reported(b):  # noqa: F811
    """Rows whose pointers fall, leave the list or name ids out of order: skipped or taken as they stand, and the next call says so."""
    L, d, B = 1000, 128, 6
    X = torch.from_numpy(o.round_bf16(np.full((B, d), 0.125, np.float32)).view(np.int16)).to("cuda:0")
    for indptr, indices in (([0, 2, 1, 2, 3, 4, 5], [1, 2, 3, 4, 5, 6]), ([0, 1, 2, 3, 4, 5, 9], [1, 2, 3, 4, 5, 6]), ([0, 2, 3, 4, 5, 6, 6], [7, 7, 1, 2, 3, 4]),
                            ([0, 1, 2, 3, 4, 5, 6], [1, 2, -1, 4, 5, 6])):
        head = b.Head(L, d, o.BF16, L, b.ELMO_VALIDATE, B, 6)
        head.step(X, torch.tensor(indptr, dtype=torch.int32, device="cuda:0"), torch.tensor(indices, dtype=torch.int32, device="cuda:0"), 0.5, 0, 0)
        rows = [(r, indices[p]) for r in range(B) if indptr[r] <= indptr[r + 1] <= len(indices) for p in range(indptr[r], indptr[r + 1])]
        G = np.full((B, L), 0.5)
        for r, l in rows:
            if l >= 0:
                G[r, l] = -0.5
        assert np.array_equal(head.weights().view(torch.bfloat16).float().cpu().numpy()[:, 0], -0.5 * 0.125 * G.sum(0).astype(np.float32))
        with pytest.raises(b.ElmoError) as e:
            head.step(X, torch.zeros(B + 1, dtype=torch.int32, device="cuda:0"), torch.zeros(0, dtype=torch.int32, device="cuda:0"), 0.5, 0, 1)
        assert e.value.code == -4


def test_set_up_does_not_wait_for_uneven_rows(b):  # noqa: F811
    """Eight rows of 1000 positives 128 rows apart among rows of one: the set-up takes about what the same number of positives
    in even rows takes (thirty times that where a few threads walk them one after another)."""
    B, L, d = 1024, 100000, 128
    us = []
    for lens in (np.where(np.arange(B) % 128 == 5, 1000, 1), np.full(B, 9)):
        indptr, indices = uneven(B, lens, L)
        head = b.Head(L, d, o.E4M3, L, 0, B, len(indices))
        args = [torch.from_numpy(v).to("cuda:0") for v in (synth.make_x(np.random.default_rng(1), B, d).view(np.int16), indptr, indices)]
        b.elmo_head_profile(head.h, True)
        for _ in range(3):
            head.step(*args, 0.0, 0, 0)
        b.elmo_head_profile_read(head.h)
        for _ in range(10):
            head.step(*args, 0.0, 0, 0)
        us.append(100 * b.elmo_head_profile_read(head.h)["setup"][0])
    say(f"   set-up: uneven rows {us[0]:.1f} us, even rows {us[1]:.1f} us")
    assert us[0] <= 4 * us[1]


@pytest.mark.parametrize("fmt", [o.BF16, o.E4M3])
@pytest.mark.parametrize("n,first,shift", [
    (1, 0, 0), (7, 3, 0), (8, 8, 0), (2049, 16, 0),     # fewer than a group, one group, a remainder
    (4096 + 5, 13, 0),                                  # groups that span two blocks of fields
    (4096 + 5, 13, 1), (2048, 0, 3),                    # buffers that are not aligned to the wide accesses
    (256 * 32 * 256 * 8 + 24, 40, 0),                   # more groups than threads
    ((2 << 20) - 1, 13, 0), ((2 << 20) + 5, 13, 0),     # on both sides of the line between the two forms of stochastic rounding
])
def test_quantize_sizes_and_alignment(b, fmt, n, first, shift):  # noqa: F811
    """Whatever the size, the first element and the alignment, the bits are the oracle's and nothing else is written."""
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n) * 0.05).astype(np.float32)
    src = torch.zeros(n + 8, dtype=torch.float32, device="cuda:0")
    src[shift:shift + n] = torch.from_numpy(x)
    tdt, ndt = (torch.int16, np.uint16) if fmt == o.BF16 else (torch.uint8, np.uint8)
    for mode in (0, 1):
        dst = torch.full((n + 16,), 85, dtype=tdt, device="cuda:0")
        b.elmo_quantize(src[shift:], n, fmt, mode, 77, 5, first, dst[shift:])
        got = dst.cpu().numpy().view(ndt)
        pick = np.arange(n) if n <= 1 << 16 else np.unique(np.concatenate([np.arange(4096), n - 1 - np.arange(4096), rng.integers(0, n, 4096)]))
        r = o.sr_fields(77, 5, (first + pick).astype(np.uint64)) if mode else None
        assert np.array_equal(got[shift + pick], o.quantize(x[pick], fmt, r))
        assert (got[:shift] == 85).all() and (got[shift + n:] == 85).all()


SR, KA = o.FLAG_SR, o.FLAG_KAHAN
# (kernels, fmt, flags, B, d, L, chunk, kahan_rows, dropout threshold, weight decay, passes)
SEVERAL = [
    ("256", o.E4M3, SR, 40, 256, 250000, 9600, 0, 0, 0.0, 3),
    ("256", o.E4M3, SR | KA, 40, 256, 250000, 9600, 128 * 800, 0, 0.0, 3),      # compensation ends inside a pass
    ("256", o.E4M3, SR | KA, 70, 256, 100000, 512, 0, 77, 0.01, 2),             # masked tile copy
    ("256", o.BF16, SR, 100, 256, 100000, 512, 0, 128, 0.0, 2),
    ("256", o.BF16, KA, 70, 256, 100000, 512, 128 * 500, 0, 0.01, 2),
    ("128", o.BF16, KA, 70, 256, 100000, 512, 0, 26, 0.0, 2),                   # no room for the masked copy of 256 columns
    ("128", o.E4M3, SR | KA, 130, 640, 100003, 30000, 128 * 300, 0, 0.0, 2),    # the last pass ragged
    ("separate", o.E4M3, SR, 300, 384, 150000, 20000, 0, 0, 0.0, 4),            # passes in the top-k scratch
    ("separate", o.E4M3, SR | KA, 300, 128, 100000, 512, 128 * 500, 64, 0.01, 2),
    ("separate", o.E4M3, SR | KA, 70, 128, 100000, 512, 128 * 500, 64, 0.01, 2),    # a small batch
    ("separate", o.BF16, SR, 300, 128, 60000, 512, 0, 128, 0.0, 2),
    ("separate", o.BF16, KA, 600, 256, 60000, 512, 0, 26, 0.01, 2),             # the last pass larger than the first
    ("128", o.E4M3, SR, 5, 256, 5000, 128, 0, 0, 0.0, 1),                       # everything in one pass
]


@pytest.mark.parametrize("fmt,flags,B,d,L,chunk,kahan_rows,T,wd,passes", [row[1:] for row in SEVERAL])
def test_passes_larger_than_the_chunk(b, fmt, flags, B, d, L, chunk, kahan_rows, T, wd, passes):  # noqa: F811
    """A head whose passes are made of several chunks computes what one with a single chunk does: the same weights and
    compensation bit by bit, dX and loss to the order of FP32 sums (BF16 rounding of dX: one spacing, 2^-8 in norm), and
    a top-k between two steps, whose scratch holds a pass's gradients, disturbs neither.  Labels of every pass against
    the oracle too, so that an offset lost in both -- the masks, the rounding fields -- shows."""
    X, indptr, indices = batch(L, d, B)
    got, like = [], None
    for ch in (chunk, L):
        case = Case(b, L, d, fmt, ch, flags, B, w_std=0.05, seed=8, kahan_rows=kahan_rows, dropout_p=T / 256, weight_decay=wd, like=like)
        like = case
        case.head.workspace.fill_(0x7F)
        idx = torch.zeros((B, 7), dtype=torch.int32, device="cuda:0")
        Xd = torch.from_numpy(X.view(np.int16)).to("cuda:0")
        out = [case.step(X, indptr, indices, 0.05, 1, 2)]
        assert case.passes == (passes if ch == chunk else 1)
        first = case.W()
        case.head.topk(Xd, 7, idx, None)
        out += [case.step(X, indptr, indices, 0.05, 1, 3), (idx.cpu().numpy(), 0.0), (case.W(), case.C())]
        got.append(out)
        case.head.close()
    (d0, d1, i, w), (e0, e1, j, v) = got
    assert np.array_equal(w[0], v[0]) and np.array_equal(i[0], j[0])
    assert w[1] is None or np.array_equal(w[1], v[1])
    for (x, lx), (y, ly) in ((d0, e0), (d1, e1)):
        assert_dx_close(x, y, 2.0 ** -8)
        assert abs(lx - ly) <= 1e-5 * abs(ly)
    rows = np.unique(np.concatenate([np.arange(l, min(l + 64, L)) for l in range(0, L, max(L // 24, 1))] + [np.arange(L - 64, L)]))
    C = None
    if flags & KA:
        C = np.zeros((len(rows), d), np.uint16)
        held = rows < (kahan_rows or L)
        C[held] = case.C0[rows[held]]
    ref = o.head_step(case.W0[rows], C, X, indptr, indices, 0.05, 1, 2, fmt, flags, label_ids=rows, weight_decay=wd, dropout=T,
                      **({"kahan_rows": kahan_rows} if kahan_rows else {}))
    dist = np.abs(ordered(first[rows], fmt) - ordered(ref["W_new"], fmt))
    assert np.mean(dist <= 1) >= 0.999
    assert_far_misses_are_tiny(first[rows], ref["W_new"], dist, fmt, 0.05)
    ref, _ = o.input_gradient_rows(case.W0, X, indptr, indices, fmt, np.arange(min(B, 8)), dropout=T, seed=1, step=2)
    assert_dx_close(d0[0][:8], ref, 6e-2)


@pytest.mark.parametrize("fmt", [o.BF16, o.E4M3])
@pytest.mark.parametrize("B,L,d,levels", [
    (1, 40, 128, 3),            # fewer labels than k allows, all in the first level
    (1, 4096, 256, 5),          # exactly the first level
    (64, 4097, 128, 9),         # one label more
    (65, 30011, 384, 9),        # two more 64-row groups than one tile holds: the 128-row tile
    (128, 21000, 128, 17),      # one slab per E4M3 tile
    (129, 25000, 128, 9),       # the first batch on the 256-row tiles
    (3, 70000, 128, 2),         # a handful of distinct scores: thousands of labels tie with the k-th
])
def test_topk_is_exact_with_ties(b, fmt, B, L, d, levels):  # noqa: F811
    """Weights and inputs on a coarse grid make every score a small multiple of 2^-4, exact in FP32, so ids and scores
    have one right answer, ties by smaller id included: across level and tile edges, through buckets that hold
    more candidates than a workgroup can rank, and for signed zeros and negative scores."""
    rng = np.random.default_rng(L + B)
    W = (rng.integers(0, levels, (L, d)) - levels // 2).astype(np.float32) / 8
    X = rng.integers(-1, 2, (B, d)).astype(np.float32) * (rng.random((B, d)) < 0.2) / 2
    if B > 2:
        X[0] = 0.0                                   # every score is zero
        X[1] = -np.abs(X[1])
    Wq = o.quantize(W, fmt)
    assert np.array_equal(o.decode(Wq, fmt), W)
    Wd = torch.from_numpy(Wq.view(np.int16) if fmt == o.BF16 else Wq).to("cuda:0")
    Xd = torch.from_numpy(o.round_bf16(X).view(np.int16)).to("cuda:0")
    head = b.Head(L, d, fmt, 4096, 0, B, B)
    head.weights().copy_(Wd)
    Z = torch.from_numpy(X) @ torch.from_numpy(W).T
    for k in (1, 100, 128, 130):
        k = min(k, L)
        ref_sc, ref_idx = torch.sort(Z, dim=1, descending=True, stable=True)
        ref_sc, ref_idx = ref_sc[:, :k].numpy(), ref_idx[:, :k].numpy()
        outs = [lambda i, s: head.topk(Xd, k, i, s)]
        if B <= 128:
            outs.append(lambda i, s: b.elmo_topk_static(Wd, L, d, fmt, Xd, B, k, i, s))
        for call in outs:
            idx, sc = torch.full((B, k), -7, dtype=torch.int32, device="cuda:0"), torch.full((B, k), 7.0, device="cuda:0")
            head.workspace.fill_(0x7F)
            call(idx, sc)
            assert np.array_equal(idx.cpu().numpy(), ref_idx)
            assert np.array_equal(sc.cpu().numpy(), ref_sc)


@pytest.mark.parametrize("fmt", [o.BF16, o.E4M3])
@pytest.mark.parametrize("B", [3, 100, 200])        # lists of 8192 on 64-row and on 128-row tiles, lists of 4096
@pytest.mark.parametrize("above", [4096 - 5, 4097, 8192 - 5, 8192 - 4, 9000])
def test_topk_list_lengths(b, fmt, B, above):  # noqa: F811
    """`above` labels after the first 4096 beat every label of the first level: with the five that are kept as many as a list of
    4096 (where one level takes them all) or 8192 holds, one more (the overflow path), or well beyond.  Scores are small
    multiples of 1/16, so thousands tie, and ids and scores have one right answer."""
    L, d, k = 60000, 128, 5
    rng = np.random.default_rng(above)
    W = np.zeros((L, d), np.float32)
    W[:, 0] = rng.integers(-8, 9, L) / 8
    W[rng.choice(np.arange(4096, 20000), above, replace=False), 0] = rng.integers(9, 17, above) / 8
    X = np.zeros((B, d), np.float32)
    X[:, 0] = 0.5
    Wq = o.quantize(W, fmt)
    assert np.array_equal(o.decode(Wq, fmt), W)
    Xd = torch.from_numpy(o.round_bf16(X).view(np.int16)).to("cuda:0")
    head = b.Head(L, d, fmt, 4096, 0, B, B)
    head.weights().copy_(torch.from_numpy(Wq.view(np.int16) if fmt == o.BF16 else Wq).to("cuda:0"))
    head.workspace.fill_(0x7F)
    idx, sc = torch.full((B, k), -7, dtype=torch.int32, device="cuda:0"), torch.full((B, k), 7.0, device="cuda:0")
    head.topk(Xd, k, idx, sc)
    ref_sc, ref_idx = torch.sort(torch.from_numpy(W[:, 0] / 2), descending=True, stable=True)
    assert np.array_equal(idx.cpu().numpy(), np.tile(ref_idx[:k].numpy(), (B, 1)))
    assert np.array_equal(sc.cpu().numpy(), np.tile(ref_sc[:k].numpy(), (B, 1)))


@pytest.mark.parametrize("B,k", [(1, 1), (1024, 3), (1025, 3), (3000, 300), (7, 1000)])
def test_precision_hits_sizes(b, B, k):  # noqa: F811
    """Row groups of 1024 and scans of 256 positions: the counts are the definition's."""
    rng = np.random.default_rng(B)
    n = 2000
    idx = np.stack([rng.choice(n, k, replace=False) for _ in range(B)]).astype(np.int32)
    rows = [np.sort(rng.choice(n, rng.integers(0, 12), replace=False)) for _ in range(B)]
    indptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    indices = np.concatenate(rows + [np.zeros(1, np.int64)]).astype(np.int32)
    want = np.cumsum(np.sum([np.isin(idx[i], rows[i]) for i in range(B)], axis=0))
    hits = torch.full((k,), -1, dtype=torch.int64, device="cuda:0")
    b.elmo_precision_hits(torch.from_numpy(idx).to("cuda:0"), B, k, torch.from_numpy(indptr).to("cuda:0"),
                          torch.from_numpy(indices).to("cuda:0"), hits)
    assert np.array_equal(hits.cpu().numpy(), want)


@pytest.mark.parametrize("fmt,flags", [(o.BF16, o.FLAG_SR), (o.E4M3, o.FLAG_SR | o.FLAG_KAHAN)])
@pytest.mark.parametrize("B,L", [
    (129, 2000), (300, 257), (520, 130),    # 128-row tiles of a larger batch: the last one ragged, or with no rows of the padded batch
    (200, 33000 + 7), (300, 16384 + 5),     # just too many tiles for them: the 256-row tiles, ragged both ways
])
def test_logits_tile_choice(b, fmt, flags, B, L):  # noqa: F811
    case = Case(b, L, 128, fmt, L, flags, B, w_std=0.05, seed=9)
    case.head.workspace.fill_(0x7F)
    check_step(case, *batch(L, 128, B), 0.05, 1, 2, 6e-2)


@pytest.mark.parametrize("B,d", [(40, 256), (300, 384)])
@pytest.mark.parametrize("shift", [1, 3, 4])
def test_inputs_of_an_fp8_head_may_begin_at_any_element(b, B, d, shift):  # noqa: F811
    """X is staged before use: the same step and the same top-k, bit for bit, whatever its first element's address."""
    L, fmt, flags = 3000, o.E4M3, o.FLAG_SR | o.FLAG_KAHAN
    X, indptr, indices = batch(L, d, B)
    Xh = torch.from_numpy(X.view(np.int16))
    out = []
    for s in (0, shift):
        case = Case(b, L, d, fmt, L, flags, B, w_std=0.05, seed=8)
        buf = torch.zeros(B * d + 8, dtype=torch.int16, device="cuda:0")
        Xd = buf[s:s + B * d].view(B, d)
        Xd.copy_(Xh)
        dX = torch.zeros((B, d), dtype=torch.int16, device="cuda:0")
        idx, sc = torch.zeros((B, 9), dtype=torch.int32, device="cuda:0"), torch.zeros((B, 9), device="cuda:0")
        case.head.topk(Xd, 9, idx, sc)
        case.head.step(Xd, torch.from_numpy(indptr).to("cuda:0"), torch.from_numpy(indices).to("cuda:0"), 0.05, 1, 2, dX, None)
        out.append((case.W(), case.C(), dX.cpu().numpy(), idx.cpu().numpy(), sc.cpu().numpy()))
    for p, q in zip(*out):
        assert np.array_equal(p, q)


@pytest.mark.parametrize("B,d,L", [
    (1, 384, 33),       # two slabs of samples, fewer than the ring's stages; one label slab and one row per slice
    (128, 128, 31),     # four, as many as stages; less than one label block
    (300, 640, 257),    # ten; half a column tile, one row beyond a label tile
    (321, 256, 1025),   # the last samples in a slab of their own
])
@pytest.mark.parametrize("fmt,flags,T", [(o.BF16, o.FLAG_SR, 0), (o.E4M3, o.FLAG_SR | o.FLAG_KAHAN, 0), (o.E4M3, o.FLAG_SR, 64), (o.BF16, o.FLAG_SR, 64)])
def test_short_rings_and_cut_blocks(b, fmt, flags, T, B, d, L):  # noqa: F811
    """Products over fewer slabs than the rings have stages, and gradients whose label blocks and octets of samples are cut."""
    case = Case(b, L, d, fmt, L, flags, B, w_std=0.05, seed=11, **({"dropout_p": T / 256} if T else {}))
    case.head.workspace.fill_(0x7F)
    X, indptr, indices = batch(L, d, B, rule="fixed5")
    tol = 6e-2 if fmt == o.E4M3 else 2e-2
    if not T:
        check_step(case, X, indptr, indices, 0.05, 3, 1, tol)
        return
    ref = o.head_step(case.W0, None, X, indptr, indices, 0.05, 3, 1, fmt, flags, dropout=T)
    dX, _ = case.step(X, indptr, indices, 0.05, 3, 1)
    dist = np.abs(ordered(case.W(), fmt) - ordered(ref["W_new"], fmt))
    assert np.mean(dist <= 1) >= 0.999
    assert_dx_close(dX, ref["dX_partial"], tol)


# (kernel, B, d, L, kahan_rows)
ONE_PASS = [
    ("128", 129, 256, 31, 0),       # the fewest rows, less than a label tile
    ("128", 192, 640, 97, 0),       # the second half of the samples half empty
    ("128", 193, 384, 4133, 128),   # one row beyond 192; compensation for the first tiles, a launch each
    ("128", 256, 768, 3000, 0),     # the most rows; groups of three label tiles, the last with fewer
    ("128", 1, 384, 33, 0),         # one row, where 256 does not divide the width
    ("128", 128, 640, 4100, 128),   # three groups of samples for the lower waves' steps, none for half of the upper waves
    ("128", 64, 256, 16384, 0),     # the most tiles of a small batch that still takes 128 columns,
    ("256", 64, 256, 16385, 0),     # one label more: the last of three to a group holds one label,
    ("256", 65, 256, 16385, 8192),  # and one more row; compensation for half of the labels
]
ONE_PASS_MODES = [(o.E4M3, SR | KA, 0, 0.0), (o.E4M3, SR, 64, 0.01), (o.BF16, KA, 64, 0.0), (o.BF16, SR, 0, 0.0)]


@pytest.mark.parametrize("B,d,L,kahan_rows", [row[1:] for row in ONE_PASS])
@pytest.mark.parametrize("fmt,flags,T,wd", ONE_PASS_MODES)
def test_one_pass_kernels(b, fmt, flags, T, wd, B, d, L, kahan_rows):  # noqa: F811
    """Input gradient and update in one pass over the weights, over 128-column tiles (the update a tile late) and 256-column ones; the
    update alone, which other kernels do beyond 128 rows and at other widths, gives the same bits."""
    kr = kahan_rows if flags & o.FLAG_KAHAN else 0
    case = Case(b, L, d, fmt, L, flags, B, w_std=0.05, comp_std=2e-4 if flags & o.FLAG_KAHAN else 0.0, seed=12, kahan_rows=kr, weight_decay=wd, dropout_p=T / 256)
    case.head.workspace.fill_(0x7F)
    X, indptr, indices = batch(L, d, B, rule="fixed5")
    C0 = case.C0
    if kr:
        C0 = np.zeros((L, d), np.uint16)
        C0[:kr] = case.C0
    ref = o.head_step(case.W0, C0, X, indptr, indices, 0.05, 3, 1, fmt, flags, kahan_rows=kr or None, weight_decay=wd, dropout=T)
    dX, loss = case.step(X, indptr, indices, 0.05, 3, 1)
    dist = np.abs(ordered(case.W(), fmt) - ordered(ref["W_new"], fmt))
    assert np.mean(dist <= 1) >= 0.999
    assert_far_misses_are_tiny(case.W(), ref["W_new"], dist, fmt, 0.05)
    assert_dx_close(dX, ref["dX_partial"], 6e-2 if fmt == o.E4M3 else 2e-2)
    assert abs(loss - ref["loss"]) <= 2e-3 * abs(ref["loss"])
    if flags & o.FLAG_KAHAN:
        n = kr or L
        same = dist[:n] == 0
        err = np.abs(o.decode_bf16(case.C()[:n]) - o.decode_bf16(ref["comp_new"][:n]))[same] / np.maximum(np.abs(o.decode(ref["W_new"][:n], fmt)), 2.0**-9)[same]
        assert np.quantile(err, 0.999) <= 2.0**-8
    alone = Case(b, L, d, fmt, L, flags, B, w_std=0.05, comp_std=2e-4 if flags & o.FLAG_KAHAN else 0.0, seed=12, kahan_rows=kr, weight_decay=wd, dropout_p=T / 256, like=case)
    alone.head.workspace.fill_(0x7F)
    alone.step(X, indptr, indices, 0.05, 3, 1, want_dx=False)
    assert np.array_equal(alone.W(), case.W()) and (not flags & o.FLAG_KAHAN or np.array_equal(alone.C(), case.C()))


@pytest.mark.parametrize("B,L,d,per_row", [(1, 100, 128, 1), (3, 129, 256, 40), (64, 8192, 256, 5), (128, 1000, 384, 16), (127, 70000, 256, 2), (128, 300, 256, 17)])
def test_small_bf16_steps_find_their_positives(b, B, L, d, per_row):  # noqa: F811
    """A BF16 step of at most 128 rows and 2048 positives has no label index and transposes X beside its logits; one positive list
    beyond (128 x 17) and the validating head go the other way, and all give the same bits."""
    rng = np.random.default_rng(3)
    X = synth.make_x(rng, B, d)
    indices = np.concatenate([np.sort(rng.choice(L, size=per_row, replace=False)) for _ in range(B)]).astype(np.int32)
    indptr = (np.arange(B + 1) * per_row).astype(np.int32)
    case = Case(b, L, d, o.BF16, L, SR, B, max_nnz=B * per_row, w_std=0.05, seed=4)
    case.head.workspace.fill_(0x7F)
    check_step(case, X, indptr, indices, 0.05, 0, 0, 2e-2)
    other = Case(b, L, d, o.BF16, L, SR | b.ELMO_VALIDATE, B, max_nnz=B * per_row, w_std=0.05, seed=4, like=case)
    other.head.workspace.fill_(0x7F)
    dX, loss = other.step(X, indptr, indices, 0.05, 0, 0)
    again = Case(b, L, d, o.BF16, L, SR, B, max_nnz=B * per_row, w_std=0.05, seed=4, like=case)
    dX2, loss2 = again.step(X, indptr, indices, 0.05, 0, 0)
    assert np.array_equal(other.W(), again.W()) and np.array_equal(dX, dX2) and loss == loss2


def test_small_bf16_steps_skip_malformed_rows(b):  # noqa: F811
    """Row pointers that fall, leave the list or stand at the ends of their type: those rows are skipped, the others count, and a list that
    begins before the first row or goes on behind the last."""
    L, d, top = 1000, 128, 2**31 - 1
    for indptr in ([0, 2, 1, 2, 3, 4, 5], [0, 1, 2, 3, 4, 5, 9], [-1, 1, 2, 3, -2**31, 4, 6], [0, top, top, 1, 2, top - 1, 3], [top, 0, 6, 6, top - 2, 5, 6], [1, 2, 2, 4], [0, 0, 0, 6, 5]):
        indices = [1, 2, 300, 4, 999, 6]
        B = len(indptr) - 1
        X = torch.from_numpy(o.round_bf16(np.full((B, d), 0.125, np.float32)).view(np.int16)).to("cuda:0")
        head = b.Head(L, d, o.BF16, L, 0, B, 6)
        head.workspace.fill_(0x7F)
        head.step(X, torch.tensor(indptr, dtype=torch.int32, device="cuda:0"), torch.tensor(indices, dtype=torch.int32, device="cuda:0"), 0.5, 0, 0)
        G = np.full((B, L), 0.5)
        for r in range(B):
            if 0 <= indptr[r] <= indptr[r + 1] <= len(indices):
                G[r, indices[indptr[r]:indptr[r + 1]]] = -0.5
        assert np.array_equal(head.weights().view(torch.bfloat16).float().cpu().numpy(), np.repeat(-0.5 * 0.125 * G.sum(0).astype(np.float32)[:, None], d, 1))


@pytest.mark.parametrize("B,what,L", [(1, "all", 300), (1, "all", 70000), (2, "all", 70000), (64, "one long", 8192), (127, "mixed", 5000), (128, "every third", 3000), (128, "last", 9000), (128, "none", 300)])
def test_small_bf16_steps_with_uneven_rows(b, B, what, L):  # noqa: F811
    """Up to 2048 positives however they are spread over the rows: exact weights, as in test_every_positive_reaches_its_label."""
    d, lr = 128, 0.5
    rng = np.random.default_rng(4)
    lens = {"all": np.full(B, min(2048 // B, L)), "one long": np.where(np.arange(B) == B // 2, 1900, 2), "mixed": rng.integers(0, 30, B),
            "every third": np.arange(B) % 3 // 2 * 40, "last": np.where(np.arange(B) == B - 1, 2048, 0), "none": np.zeros(B, int)}[what]
    indptr, indices = uneven(B, lens, L)
    assert len(indices) <= 2048
    X = rng.choice([-0.125, 0.125], (B, d)).astype(np.float32)
    X[1::2] = -X[:B // 2 * 2:2]
    head = b.Head(L, d, o.BF16, 131072, 0, B, max(len(indices), 1))
    head.workspace.fill_(0x7F)
    Xd, ip, ix = (torch.from_numpy(v).to("cuda:0") for v in (o.round_bf16(X).view(np.int16), indptr, indices))
    head.step(Xd, ip, ix, lr, 0, 0)
    Xf = torch.from_numpy(X).to("cuda:0")
    want = (-lr / 2 * Xf.double().sum(0)).float().expand(L, d).clone()
    want.index_add_(0, ix.long(), lr * Xf[torch.repeat_interleave(torch.arange(B, device="cuda:0"), ip.diff().long())])
    assert torch.equal(head.weights().view(torch.bfloat16).float(), want.bfloat16().float())


def test_small_bf16_steps_do_not_wait_for_uneven_rows(b):  # noqa: F811
    """One row with most of 2000 positives: the logits of many label tiles take about what they take with even rows (four times that
    where a row's positives are walked by a few threads in every tile)."""
    B, L, d = 64, 500000, 256
    us = []
    for lens in (np.where(np.arange(B) == 5, 1800, 2), np.full(B, 30)):
        indptr, indices = uneven(B, lens, L)
        head = b.Head(L, d, o.BF16, L, 0, B, len(indices))
        args = [torch.from_numpy(v).to("cuda:0") for v in (synth.make_x(np.random.default_rng(1), B, d).view(np.int16), indptr, indices)]
        b.elmo_head_profile(head.h, True)
        for _ in range(3):
            head.step(*args, 0.0, 0, 0)
        b.elmo_head_profile_read(head.h)
        for _ in range(10):
            head.step(*args, 0.0, 0, 0)
        us.append(100 * b.elmo_head_profile_read(head.h)["logits"][0])
    say(f"   logits: uneven rows {us[0]:.1f} us, even rows {us[1]:.1f} us")
    assert us[0] <= 1.5 * us[1]
