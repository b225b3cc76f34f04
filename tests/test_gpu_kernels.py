"""GPU parity of the share kernels at the sizes where their tilings can go wrong: every output element
against the oracle's Eq. 1, at tile edges, remainders of the contraction units and the longest runs
between two recombinations."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as co                                   # noqa: E402
from workloads import rng                             # noqa: E402
from workloads.launches import kernels, places        # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_07239_amd as comet
    c = comet.Context(0)
    yield c
    c.close()


def up(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def down(t):
    return t.cpu().numpy().view(np.uint64)


def u64(seed, stream, *shape):
    return rng.uniform_u64(seed, stream, int(np.prod(shape))).reshape(shape)


def check(ctx, kind, m, other, bs, kept, fmt, full, party=1, seed=900, kernel=None):
    """One share call: ``other`` is the axis that is not indexed (k of SOMM, n of SIMM).  ``kernel``: how the name of the
    kernel that has to take the call begins."""
    print("[gpu-kernels] %s m=%d other=%d bs=%d blocks=%d %s full=%s" % (kind, m, other, bs, len(kept), fmt, full),
          flush=True)
    sys.stdout.flush()
    idx = np.array(kept, dtype=np.int32)
    t, nb = len(idx), int(idx.max()) + 2
    na, nf = t * bs, nb * bs
    if kind == "somm":
        e, a, f, b, c = u64(seed, 1, m, other), u64(seed, 2, m, other), u64(seed, 3, other, na), u64(seed, 4, other, nf), \
            u64(seed, 5, m, na)
        a_sel, b_sel = a, co.index_cols(b, idx, bs)
    else:
        e, a, f, b, c = u64(seed, 1, m, na), u64(seed, 2, m, nf), u64(seed, 3, na, other), u64(seed, 4, nf, other), \
            u64(seed, 5, m, other)
        a_sel, b_sel = co.index_cols(a, idx, bs), co.index_rows(b, idx, bs)
    want = co.beaver_share(party, e, f, a_sel, b_sel, c)
    gi = torch.from_numpy(idx).cuda()
    b = b if full else b_sel
    tr = fmt == "neuron_major"
    e_d, a_d, f_d, b_d, c_d = up(e), up(a if full else a_sel), up(f.T if tr else f), up(b.T if tr else b), up(c)
    if fmt == "planes":
        f_d, b_d = ctx.open_weight_planes(f_d), ctx.open_weight_planes(b_d)

    def call():
        if kind == "somm":
            return ctx.somm_share(party, bs, gi, None, t, e_d, f_d, a_d, b_d, c_d, b_full=full, neuron_major=tr)
        return ctx.simm_share(party, bs, gi, None, t, e_d, f_d, a_d, b_d, c_d, a_full=full, b_full=full)

    z = call()
    torch.cuda.synchronize()
    assert np.array_equal(down(z), want)
    if kernel:
        ran = kernels(call)
        assert len([name for name in ran if name.startswith(kernel)]) == 1, ran


# Contraction of one half in words (steps of 32, stacked and taken in pairs): one step (the only pair
# takes one step of each half), odd and even step counts.  The 64 x 64 tile (forced: products this small take the few-row
# and the one-launch kernel), and whatever the size takes.
@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("m", [33, 64, 65, 128, 129])
@pytest.mark.parametrize("k", [1, 31, 33, 64, 95, 160])
def test_planes_tiles_and_step_pairs(ctx, m, k, tile):
    import paper_2505_07239_amd as comet
    kernel = "ring_planes_kernel<2, 2, 2, 2," if tile else "ring_direct_kernel<" if k <= 100 else "ring_fewrow_kernel<"
    ctx.set_tuning(comet.TUNE_GEMM_TILE, tile)
    try:
        check(ctx, "somm", m, k, 16, (0, 2, 3, 5, 6), "planes", True, kernel=kernel)
        if k >= 16:
            check(ctx, "simm", m, 65, 16, tuple(range(0, 2 * ((k + 15) // 16), 2)), "planes", True, kernel=kernel)
    finally:
        ctx.set_tuning(comet.TUNE_GEMM_TILE, 0)


@pytest.mark.parametrize("m,n", [(33, 64), (128, 64)])
def test_planes_long_contraction(ctx, m, n):
    """One workgroup, 4 x 128 + 1 pairs: the planes are flushed between the runs."""
    import paper_2505_07239_amd as comet
    ctx.set_tuning(comet.TUNE_GEMM_GRID, 1)
    try:
        check(ctx, "somm", m, 513 * 32, n, (0,), "planes", True, kernel="ring_planes_kernel<2, 2, 2, 2,")
    finally:
        ctx.set_tuning(comet.TUNE_GEMM_GRID, 0)


def check_columns(ctx, kind, m, k, n, fmt, grid=0, seed=920, kernel=None, bs=16):
    """One share call too large for the oracle as a whole: the first and last column of every 64, compared
    in full.  Every second block of the indexed axis (n of SOMM, k of SIMM) is kept."""
    import paper_2505_07239_amd as comet
    print("[gpu-kernels] columns %s m=%d k=%d n=%d bs=%d %s grid=%d" % (kind, m, k, n, bs, fmt, grid), flush=True)
    t = (n if kind == "somm" else k) // bs
    idx = np.arange(0, 2 * t, 2, dtype=np.int32)
    e, c = u64(seed, 1, m, k), u64(seed, 5, m, n)
    f = torch.randint(-2 ** 63, 2 ** 63 - 1, (k, n), dtype=torch.int64, device="cuda")
    full = (k, 2 * n) if kind == "somm" else (2 * k, n)
    b = torch.randint(-2 ** 63, 2 ** 63 - 1, full, dtype=torch.int64, device="cuda")
    a = u64(seed, 2, m, k if kind == "somm" else 2 * k)
    sel = np.repeat(idx.astype(np.int64), bs) * bs + np.tile(np.arange(bs), t)     # gathered position of a compact one
    cols = np.unique(np.concatenate([np.arange(0, n, 64), np.minimum(np.arange(63, n + 64, 64), n - 1)]))
    cols_d = torch.from_numpy(cols).cuda()
    if kind == "somm":
        b_sel, a_sel = down(b[:, torch.from_numpy(sel[cols]).cuda()]), a
    else:
        b_sel, a_sel = down(b[:, cols_d][torch.from_numpy(sel).cuda()]), np.ascontiguousarray(a[:, sel])
    want = co.beaver_share(1, e, down(f[:, cols_d]), a_sel, b_sel, np.ascontiguousarray(c[:, cols]))
    if fmt == "planes":
        f, b = ctx.open_weight_planes(f), ctx.open_weight_planes(b)
    gi, e, a, c = torch.from_numpy(idx).cuda(), up(e), up(a), up(c)
    call = lambda: (ctx.somm_share if kind == "somm" else ctx.simm_share)(1, bs, gi, None, t, e, f, a, b, c)
    ctx.set_tuning(comet.TUNE_GEMM_GRID, grid)
    try:
        z = call()
        ran = kernels(call) if kernel else []
    finally:
        ctx.set_tuning(comet.TUNE_GEMM_GRID, 0)
    assert np.array_equal(down(z[:, cols_d]), want)
    assert not kernel or len([name for name in ran if name.startswith(kernel)]) == 1, ran


# The 128 x 64 tile of a single call (more than 32 tiles, rows not ragged): shared tiles; and owned ones
# (the forced grid divides the tiles), with a contraction of more than 128 pairs that one run may not cover.
@pytest.mark.parametrize("kind,m,k,n,grid", [("somm", 128, 33, 2112, 0), ("somm", 250, 95, 2112, 0), ("somm", 250, 1, 2112, 0),
                                             ("simm", 128, 48, 2100, 0), ("simm", 250, 112, 2100, 0),
                                             ("somm", 128, 33, 2112, 11), ("simm", 128, 48, 2112, 11),
                                             ("somm", 250, 129 * 32 + 5, 2112, 33), ("simm", 250, 129 * 32 + 16, 2112, 33)])
def test_planes_128x64_single_calls(ctx, kind, m, k, n, grid):
    check_columns(ctx, kind, m, k, n, "planes", grid, kernel="ring_planes_kernel<2, 2, 4, 2,")


# The choice between 64 x 64 and 64 x 128: below and from 32 pairs per compute unit on (5 x 15 tiles), a multiple of 64
# tiles below and from 256 pairs on, a single row tile.
@pytest.mark.parametrize("kind,m,k,n,wide", [("somm", 320, 3488, 960, False), ("somm", 320, 3520, 960, True), ("simm", 300, 3520, 912, True),
                                             ("somm", 192, 1664, 4096, False), ("somm", 192, 10928, 4096, True),
                                             ("simm", 64, 4096, 2560, False)])
def test_planes_narrow_tile_choice(ctx, kind, m, k, n, wide):
    check_columns(ctx, kind, m, k, n, "planes", kernel="ring_planes_kernel<1, 4, 4, 2," if wide else "ring_planes_kernel<2, 2, 2, 2,")


# The 32 x 256 tile on words where it is taken without being asked for (more than sixteen units of the few-row kernel per
# compute unit), below 320 MB: rows of B_i gathered by blocks of a power of two, of another length, and column gathers.
@pytest.mark.parametrize("kind,m,k,n,bs", [("simm", 16, 4096, 2560, 32), ("simm", 32, 4095, 2500, 21), ("simm", 9, 4096, 2600, 16),
                                           ("somm", 32, 4001, 2496, 32), ("somm", 16, 4100, 2499, 21)])
def test_words_32x256_tile(ctx, kind, m, k, n, bs):
    check_columns(ctx, kind, m, k, n, "words", kernel="ring_gemm_kernel<1, 4, 1, 2,", bs=bs)


# Weight words beyond 320 MB, read past the caches up to 64 rows.
@pytest.mark.parametrize("kind", ["somm", "simm"])
@pytest.mark.parametrize("m", [9, 33, 64, 128, 129, 192, 193, 300, 768, 769])
def test_words_beyond_the_cache(ctx, kind, m):
    k, n = (2048, 10512) if kind == "somm" else (10512, 2048)
    check_columns(ctx, kind, m, k, n, "words")


# The 32 x 128 tile on planes and the 32 x 256 tile on words, whatever the size, with the few-row kernels switched off:
# remainders of the contraction and of the columns, rows of B_i as they come, gathered by blocks of a power of two and of
# any other length, neuron-major weights.
@pytest.mark.parametrize("kind,fmt,bs", [(kind, fmt, bs) for kind in ("somm", "simm") for fmt, bs in (
    ("planes", 16), ("planes", 48), ("words", 32), ("words", 21), ("words", 8), ("words", 5))] + [("somm", "neuron_major", 16)])
@pytest.mark.parametrize("m,other", [(1, 31), (9, 33), (31, 64), (32, 95), (32, 300)])
def test_32_row_tiles(ctx, kind, m, other, fmt, bs):
    import paper_2505_07239_amd as comet
    other += fmt == "neuron_major" and other % 2
    kernel = "ring_planes_kernel<1, 4, 2, 2," if fmt == "planes" else "ring_gemm_kernel<1, 4, 1, 2,"
    ctx.set_tuning(comet.TUNE_SKINNY, 1)
    try:
        check(ctx, kind, m, other, bs, (0, 2, 3, 5, 6, 7, 9, 10, 13), fmt, True, kernel=kernel)
        check(ctx, kind, m, other, bs, (1, 4), fmt, False, kernel=kernel)
    finally:
        ctx.set_tuning(comet.TUNE_SKINNY, 0)


def masked_mask(m, nb, per_block, seed=950):
    """Every block belongs to one token, and to per_block - 1 more at random: most steps of a row tile are
    there for a single token, and the row tiles list different ones."""
    mask = np.zeros((m, nb), np.uint8)
    r = rng.uniform_u64(seed + m, 60, nb * per_block).reshape(nb, per_block)
    for j in range(nb):
        mask[(7 * j) % m, j] = 1
        mask[(r[j, 1:] % np.uint64(m)).astype(np.int64), j] = 1
    return mask


def check_masked(ctx, m, nb, bs, n, fmt, per_block, full=True, replays=0, kernel=None):
    print("[gpu-kernels] masked m=%d nb=%d bs=%d n=%d %s full=%s" % (m, nb, bs, n, fmt, full), flush=True)
    k, seed = nb * bs, 940
    e, a, f, b, c = u64(seed, 1, m, k), u64(seed, 2, m, k), u64(seed, 3, k, n), u64(seed, 4, k, n), u64(seed, 5, m, n)
    idx = torch.arange(nb, dtype=torch.int32, device="cuda")
    f_d, b_d = up(f), up(b)
    if fmt == "planes":
        f_d, b_d = ctx.open_weight_planes(f_d), ctx.open_weight_planes(b_d)
    e_d, a_d, c_d = up(e), up(a), up(c)
    tm, z = torch.zeros((m, nb), dtype=torch.uint8, device="cuda"), torch.zeros((m, n), dtype=torch.int64, device="cuda")

    def call():
        ctx.simm_share_masked(1, bs, idx, None, nb, tm, e_d, f_d, a_d, b_d, c_d, a_full=full, b_full=full, out=z)

    def inputs(rep):
        mask = masked_mask(m, nb, per_block, 950 + rep)
        tm.copy_(torch.from_numpy(mask))
        return co.beaver_share_sparse_input(1, e, f, a, b, c, np.repeat(mask, bs, axis=1))

    want = inputs(0)
    call()
    assert np.array_equal(down(z), want)
    if kernel:
        ran = kernels(call)
        assert len([name for name in ran if name.startswith(kernel)]) == 1, ran
    if not replays:
        return
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep in range(1, replays + 1):
        want = inputs(rep)
        z.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(down(z), want), "replay %d" % rep
        z.zero_()
        call()
        assert np.array_equal(down(z), want), "eager after replay %d" % rep


# Per-token row sets on weight planes: the 32 x 128, 64 x 64 and (from 32 pairs per compute unit on, 24 with one
# row tile) 64 x 128 tiles.
@pytest.mark.parametrize("m,nb,bs,n", [(9, 12, 16, 40), (32, 30, 32, 130), (33, 12, 16, 64), (64, 20, 48, 65),
                                       (129, 16, 16, 200), (260, 40, 32, 96), (64, 512, 32, 768), (200, 512, 32, 257)])
@pytest.mark.parametrize("full", [True, False])
def test_masked_planes(ctx, m, nb, bs, n, full):
    check_masked(ctx, m, nb, bs, n, "planes", 3, full)


# Step lists of more than one chunk (1024 steps of 32 neurons): blocks that end with a chunk, are cut by its
# end, and single neurons; rows that are no multiple of four.
@pytest.mark.parametrize("m,nb,bs", [(70, 1056, 32), (70, 702, 48), (67, 1605, 21), (35, 33001, 1), (130, 2064, 16)])
@pytest.mark.parametrize("fmt", ["words", "planes"])
def test_masked_step_list_chunks(ctx, m, nb, bs, fmt):
    check_masked(ctx, m, nb, bs, 40, fmt, 1, fmt == "words" or bs % 16 == 0)


# One workgroup: runs of more than 128 listed pairs (256 steps) in both kernels of 64 rows on words, rows of B_i found by
# sixteen, one by one and as they come; one row tile and two with different lists.
@pytest.mark.parametrize("m,nb,bs,full", [(40, 560, 16, True), (70, 560, 16, True), (40, 930, 9, True), (70, 930, 9, False)])
@pytest.mark.parametrize("tile", [2, 3])
def test_masked_words_long_runs(ctx, m, nb, bs, full, tile):
    import paper_2505_07239_amd as comet
    ctx.set_tuning(comet.TUNE_GEMM_GRID, 1)
    ctx.set_tuning(comet.TUNE_GEMM_TILE, tile)
    try:
        check_masked(ctx, m, nb, bs, 70, "words", 2, full, kernel="ring_words_kernel<" if tile == 2 else "ring_gemm_kernel<2, 2, 1, 1,")
    finally:
        ctx.set_tuning(comet.TUNE_GEMM_GRID, 0)
        ctx.set_tuning(comet.TUNE_GEMM_TILE, 0)


# The counter of finished workgroups starts from zero in every call, replayed or not.
@pytest.mark.parametrize("fmt", ["words", "planes"])
def test_masked_replays(ctx, fmt):
    check_masked(ctx, 200, 60, 16, 96, fmt, 2, replays=3)


# Masked shares and opened words are stored through the caches up to 192 MB and past them beyond: just below, at
# and just above the line.
@pytest.mark.parametrize("words", [(192 << 17) - 512, 192 << 17, (192 << 17) + 512])
def test_store_rule_of_the_streaming_kernels(ctx, words):
    import paper_2505_07239_amd as comet
    print("[gpu-kernels] stores, %d words" % words, flush=True)
    a = torch.randint(-2 ** 63, 2 ** 63 - 1, (words // 512, 512), dtype=torch.int64, device="cuda")
    b = a.roll(1, 0)
    assert torch.equal(ctx.mask_share(a, b), a - b) and torch.equal(ctx.open(a, b), a + b)
    for axis, bs in ((comet.AXIS_ROWS, 1), (comet.AXIS_COLS, 2)):
        idx = torch.arange(a.shape[axis == comet.AXIS_COLS] // bs, dtype=torch.int32, device="cuda")
        assert torch.equal(ctx.mask_share_gather(a, b, axis, bs, idx, None, idx.numel()), a - b)


@pytest.mark.parametrize("neuron_major", [False, True])
@pytest.mark.parametrize("k", [(112 << 17) // 512 - 32, (112 << 17) // 512 + 32])
def test_large_planes(ctx, k, neuron_major):
    """Digit t of word (row, col) sits at byte row % 16 of unit (row / 32, col / 64, t, row / 16 % 2, col % 64)."""
    print("[gpu-kernels] plane stores, k=%d neuron_major=%s" % (k, neuron_major), flush=True)
    w = torch.randint(-2 ** 63, 2 ** 63 - 1, (k, 512), dtype=torch.int64, device="cuda")
    buf = ctx.open_weight_planes(w.t().contiguous() if neuron_major else w, neuron_major=neuron_major).buf
    bias = 0x0080808080808080
    want = ((w + bias) ^ bias).view(torch.uint8).view(k // 32, 2, 16, 8, 64, 8).permute(0, 3, 5, 1, 4, 2)
    assert torch.equal(buf.view(-1)[:w.numel() * 8].view(want.shape), want)


# Where a chunk's run of indices starts: from the words of at most three chunks before it (16384 blocks a
# chunk), from at most 255 counts, or from the scanned counts; and the one-workgroup masks of several tokens.
@pytest.mark.parametrize("n_tok,nb", [(2, 16384), (2, 16385), (3, 49153), (2, 65536), (2, 65537), (1, 65537),
                                      (1, 256 * 16384), (1, 256 * 16384 + 1), (4, 4096), (5, 4096), (31, 4096), (33, 3971), (70, 17)])
@pytest.mark.parametrize("density", [0.0, 0.3, 1.0])
def test_compact_chunk_starts(ctx, n_tok, nb, density):
    print("[gpu-kernels] compact %d x %d, %g" % (n_tok, nb, density), flush=True)
    mask = (rng.uniform_u64(7 + nb, 1, n_tok * nb) < np.uint64(min(int(density * 2 ** 64), 2 ** 64 - 1))).astype(np.uint8).reshape(n_tok, nb)
    idx, n = ctx.compact_mask(torch.from_numpy(mask).cuda())
    want = np.nonzero(mask.any(axis=0))[0]
    assert int(n.item()) == len(want) and np.array_equal(idx[:len(want)].cpu().numpy(), want)


# One workgroup of four or of sixteen wavefronts, either side of each line between them.
@pytest.mark.parametrize("n_tok,nb", [(1024, 48), (1025, 48), (12, 4096), (13, 4096), (3328, 32), (3329, 32),
                                      (95, 344), (96, 344), (20, 1001), (5, 4095), (6, 4095), (5, 1025), (20, 1025),
                                      (292, 56), (293, 56), (963, 17), (964, 17), (3, 4095), (16385, 1), (131072, 1)])
@pytest.mark.parametrize("lead", [0, 5])
def test_compact_one_workgroup(ctx, n_tok, nb, lead):
    print("[gpu-kernels] compact, one workgroup %d x %d from byte %d" % (n_tok, nb, lead), flush=True)
    flags = (rng.uniform_u64(9 + nb, 1, n_tok * nb) < np.uint64(2 ** 64 // 100)).astype(np.uint8)
    flags[-1] = 255
    buf = torch.full((n_tok * nb + 32,), 7, dtype=torch.uint8, device="cuda")      # flags around the mask count for nothing
    mask = buf[lead:lead + n_tok * nb].view(n_tok, nb)
    mask.copy_(torch.from_numpy(flags.reshape(n_tok, nb)))
    idx, n = ctx.compact_mask(mask)
    want = np.nonzero(flags.reshape(n_tok, nb).any(axis=0))[0]
    assert int(n.item()) == len(want) and np.array_equal(idx[:len(want)].cpu().numpy(), want)


# Members of a grouped call that name the same opened activations (whole tiles and ragged ones of the packing kernel).
@pytest.mark.parametrize("kind", ["somm", "simm"])
@pytest.mark.parametrize("m,k", [(65, 64), (130, 95), (256, 192)])
@pytest.mark.parametrize("names", [(0, 0), (0, 0, 1, 1), (0, 1, 0, 1, 2), (1, 1, 1, 1, 1, 1, 1, 1)])
def test_group_members_share_activations(ctx, kind, m, k, names):
    import paper_2505_07239_amd as comet
    print("[gpu-kernels] shared activations %s m=%d k=%d %s" % (kind, m, k, names), flush=True)
    bs, idx = 16, np.array([0, 2, 3, 5, 6, 7], dtype=np.int32)
    t, nb = len(idx), 9
    na, nf = t * bs, nb * bs
    es = {q: u64(300 + q, 1, m, k if kind == "somm" else na) for q in set(names)}
    es_d = {q: up(e) for q, e in es.items()}
    members, wants = [], []
    for j, q in enumerate(names):
        seed, party = 310 + j, j & 1
        if kind == "somm":
            f, a, b, c = u64(seed, 2, k, na), u64(seed, 3, m, k), u64(seed, 4, k, nf), u64(seed, 5, m, na)
            wants.append(co.beaver_share(party, es[q], f, a, co.index_cols(b, idx, bs), c))
        else:
            f, a, b, c = u64(seed, 2, na, k), u64(seed, 3, m, nf), u64(seed, 4, nf, k), u64(seed, 5, m, k)
            wants.append(co.beaver_share(party, es[q], f, co.index_cols(a, idx, bs), co.index_rows(b, idx, bs), c))
        members.append((party, es_d[q], ctx.open_weight_planes(up(f)), up(a), ctx.open_weight_planes(up(b)), up(c)))
    ctx.set_tuning(comet.TUNE_GROUP, 1)
    try:
        got = ctx.share_group(kind, bs, torch.from_numpy(idx).cuda(), None, t, members)
    finally:
        ctx.set_tuning(comet.TUNE_GROUP, 0)
    for j, want in enumerate(wants):
        assert np.array_equal(down(got[j]), want), "member %d" % j


# Up to 8 rows: one round of workgroups fills the chip as far as the kernel's registers allow (two columns per lane; two rows
# take two or three rounds, long runs of opened ones about sixteen workgroups a unit), six or seven a unit word by word.
@pytest.mark.parametrize("unopened", [False, True])
@pytest.mark.parametrize("kind", ["somm", "simm"])
@pytest.mark.parametrize("m", [2, 3, 6, 7])
def test_slices_fill_the_chip(ctx, kind, m, unopened):
    units = torch.cuda.get_device_properties(0).multi_processor_count
    draw = lambda *shape: torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda")

    def plan(k, n, bs):
        print("[gpu-kernels] slices %s m=%d k=%d n=%d unopened=%s" % (kind, m, k, n, unopened), flush=True)
        t = (n if kind == "somm" else k) // bs
        idx = torch.arange(t, dtype=torch.int32, device="cuda")
        e, a, c, b, w = draw(m, k), draw(m, k), draw(m, n), draw(k, n), [draw(k, n) for _ in range(1 + unopened)]
        z = torch.empty_like(c)
        call = getattr(ctx, "%s_share%s" % (kind, "_unopened" if unopened else ""))
        return places(lambda: call(1, bs, idx, None, t, e, *w, a, b, c, out=z), "ring_skinny_kernel<")

    grid, most = plan(1 << 15, 256, 32)                       # two tiles of columns
    rounds = (3 if unopened else 2) if m == 2 else 1
    assert grid == rounds * most * units, (grid, most)
    grid, most = plan(1 << 14, 128 if kind == "simm" else 127, 1)
    assert grid == (7 if m == 2 else 6) * units and most >= grid // units, (grid, most)
    if not unopened and m > 2 and (m != 6 or kind == "simm"):
        grid, most = plan(512 * 40, 128 * units // 8, 32)     # thirty-two tiles on 256 units
        tiles = units // 8
        assert 14 * units <= grid <= 16 * units and grid % tiles == 0, (grid, most)
