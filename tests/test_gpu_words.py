"""GPU parity of the share kernels that small products and products on weight words take: every output
element against the oracle's Eq. 1, at tile edges, remainders of the contraction and the longest runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as co                                   # noqa: E402
from workloads import rng                             # noqa: E402
from workloads.launches import kernels                # noqa: E402


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


def operands(kind, m, other, bs, t, full, seed):
    """Host operands of one share with every second block kept, and the indexed triple parts."""
    idx = np.arange(0, 2 * t, 2, dtype=np.int32)
    na, nf = t * bs, 2 * t * bs
    if kind == "somm":
        e, a, f, b, c = u64(seed, 1, m, other), u64(seed, 2, m, other), u64(seed, 3, other, na), \
            u64(seed, 4, other, nf), u64(seed, 5, m, na)
        a_sel, b_sel = a, co.index_cols(b, idx, bs)
    else:
        e, a, f, b, c = u64(seed, 1, m, na), u64(seed, 2, m, nf), u64(seed, 3, na, other), u64(seed, 4, nf, other), \
            u64(seed, 5, m, other)
        a_sel, b_sel = co.index_cols(a, idx, bs), co.index_rows(b, idx, bs)
    return idx, e, a if full else a_sel, f, b if full else b_sel, c, a_sel, b_sel


def check(ctx, kind, fmt, m, other, bs, t, full=True, party=1, kernel=None, **tuning):
    """``kernel``: how the name of the kernel that has to take the call begins (for a forced tile: the tile's)."""
    import paper_2505_07239_amd as comet
    if tuning.get("TUNE_GEMM_TILE"):
        kernel = "ring_planes_kernel<" if fmt == "planes" else \
            "ring_words_kernel<" if tuning["TUNE_GEMM_TILE"] == 2 else "ring_gemm_kernel<2, 2, 1, 1,"
    print("[gpu-words] %s %s m=%d other=%d bs=%d blocks=%d full=%s %s" % (kind, fmt, m, other, bs, t, full, tuning), flush=True)
    idx, e, a, f, b, c, a_sel, b_sel = operands(kind, m, other, bs, t, full, 940)
    want = co.beaver_share(party, e, f, a_sel, b_sel, c)
    tr = fmt == "neuron_major"
    f_d, b_d = (up(f.T if tr else f), up(b.T if tr else b))
    if fmt == "planes":
        f_d, b_d = ctx.open_weight_planes(f_d), ctx.open_weight_planes(b_d)
    gi, e_d, a_d, c_d = torch.from_numpy(idx).cuda(), up(e), up(a), up(c)

    def call():
        if kind == "somm":
            return ctx.somm_share(party, bs, gi, None, t, e_d, f_d, a_d, b_d, c_d, b_full=full, neuron_major=tr)
        return ctx.simm_share(party, bs, gi, None, t, e_d, f_d, a_d, b_d, c_d, a_full=full, b_full=full)

    for key, value in tuning.items():
        ctx.set_tuning(getattr(comet, key), value)
    try:
        z = call()
        torch.cuda.synchronize()
        ran = kernels(call) if kernel else []
    finally:
        for key in tuning:
            ctx.set_tuning(getattr(comet, key), 0)
    assert np.array_equal(down(z), want)
    assert not kernel or len([name for name in ran if name.startswith(kernel)]) == 1, ran


# Contraction lengths at the edges of a step (32), a pair (64) and the one-launch path (100 words).  tile 0: the one-launch
# path and the few-row kernel; 2 and 3: the tiles of 64 rows whatever the size, on words of both kernels.
@pytest.mark.parametrize("fmt,tile", [(fmt, tile) for fmt in ("words", "planes", "neuron_major") for tile in (0, 2, 3)
                                      if (fmt, tile) != ("planes", 3)])
@pytest.mark.parametrize("m", [9, 32, 33, 64, 130])
def test_small_somm(ctx, fmt, tile, m):
    for k in (1, 2, 31, 32, 33, 64, 65, 95, 97, 100, 101, 160, 193, 224):
        if fmt != "neuron_major" or k % 2 == 0:
            check(ctx, "somm", fmt, m, k, 5 if k % 3 == 0 and fmt == "words" else 16, 5, party=k & 1, TUNE_GEMM_TILE=tile)


# Blocks of 7 neurons (rows looked up one by one), of 16 (sixteen at a time) and of 32; compact operands.
@pytest.mark.parametrize("m", [9, 32, 33, 64, 130])
@pytest.mark.parametrize("fmt,bs,tile", [("words", bs, tile) for bs in (7, 16, 32) for tile in (0, 2, 3)] +
                         [("planes", bs, tile) for bs in (16, 48) for tile in (0, 2)])
def test_small_simm(ctx, fmt, bs, m, tile):
    for t in (1, 2, 3, 5, 6, 7, 14):
        check(ctx, "simm", fmt, m, 65 if t & 1 else 33, bs, t, party=t & 1, TUNE_GEMM_TILE=tile)
    check(ctx, "simm", fmt, m, 64, bs, 5, full=False, TUNE_GEMM_TILE=tile)


# One workgroup: several tiles, more than 128 pairs (256 steps) of each, so that the planes are flushed between runs.
@pytest.mark.parametrize("kind,fmt,m,other,bs,t", [("somm", "words", 33, 257 * 32 + 5, 16, 5), ("somm", "neuron_major", 33, 8228, 16, 5),
                                                   ("simm", "words", 40, 70, 16, 515), ("simm", "words", 40, 70, 9, 915),
                                                   ("somm", "words", 12, 257 * 32 + 5, 16, 5), ("simm", "words", 12, 70, 9, 915)])
def test_words_long_contraction(ctx, kind, fmt, m, other, bs, t):
    check(ctx, kind, fmt, m, other, bs, t, TUNE_GEMM_GRID=1)
    for tile in (2, 3):
        check(ctx, kind, fmt, m, other, bs, t, TUNE_GEMM_GRID=1, TUNE_GEMM_TILE=tile)


# How the contraction is shared out: a slice of one tile, even shares (72 tiles on 256 workgroups and on 7, which cut every
# tile at other places), two and four row tiles side by side, whole tiles.
@pytest.mark.parametrize("fmt", ["words", "planes"])
@pytest.mark.parametrize("m,k,n,grid", [(64, 200, 320, 0), (64, 300, 72 * 64, 0), (128, 300, 72 * 32, 0), (250, 260, 72 * 16, 0),
                                        (128, 300, 192, 7), (200, 330, 192, 4), (128, 100, 256, 8)])
def test_work_split(ctx, fmt, m, k, n, grid):
    for tile in ((2,) if fmt == "planes" else (2, 3)):
        check(ctx, "somm", fmt, m, k, 16, n // 16, TUNE_GEMM_TILE=tile, TUNE_GEMM_GRID=grid)
        if grid == 0:
            check(ctx, "simm", fmt, m, n // 4, 16, k // 16, TUNE_GEMM_TILE=tile)


# The same with fewer blocks on the device than the capacity the launch was planned for: even shares with and without teams
# of row tiles, slices, owned tiles (128 x 256 on 8 workgroups), down to one block and none.
@pytest.mark.parametrize("fmt", ["words", "planes", "neuron_major"])
@pytest.mark.parametrize("m,other,cap,grid", [(64, 300, 288, 0), (128, 300, 144, 0), (250, 260, 72, 0), (150, 300, 60, 7), (250, 260, 72, 12),
                                              (128, 100, 16, 8), (64, 200, 20, 0)])
def test_work_split_device_counts(ctx, fmt, m, other, cap, grid):
    import paper_2505_07239_amd as comet
    for kind in ("somm", "simm") if fmt != "neuron_major" else ("somm",):
        bs, seed = 16, 945
        for t in sorted({cap - 1, cap * 2 // 3, cap // 3, 1, 0}, reverse=True):
            print("[gpu-words] %s %s m=%d other=%d blocks=%d of %d grid=%d" % (kind, fmt, m, other, t, cap, grid), flush=True)
            ld, nf = cap * bs, 2 * cap * bs
            idx = np.arange(0, 2 * cap, 2, dtype=np.int32)
            on, sel = t * bs, idx[:t]
            if kind == "somm":
                e, a, f, b, c = u64(seed, 1, m, other), u64(seed, 2, m, other), u64(seed, 3, other, ld), u64(seed, 4, other, nf), \
                    u64(seed, 5, m, ld)
                want = co.beaver_share(1, e, f[:, :on], a, co.index_cols(b, sel, bs), c[:, :on]) if t else None
            else:
                e, a, f, b, c = u64(seed, 1, m, ld), u64(seed, 2, m, nf), u64(seed, 3, ld, other), u64(seed, 4, nf, other), \
                    u64(seed, 5, m, other)
                want = co.beaver_share(1, e[:, :on], f[:on], co.index_cols(a, sel, bs), co.index_rows(b, sel, bs), c) if t else c
            turn = (lambda w: up(w.T)) if fmt == "neuron_major" else up
            f_d, b_d = turn(f), turn(b)
            if fmt == "planes":
                f_d, b_d = ctx.open_weight_planes(f_d), ctx.open_weight_planes(b_d)
            gi, n_dev, e_d, a_d, c_d = torch.from_numpy(idx).cuda(), torch.tensor([t], dtype=torch.int32, device="cuda"), up(e), up(a), up(c)
            for tile in (2, 3) if fmt != "planes" else (2,):
                z = torch.full(c.shape, 77, dtype=torch.int64, device="cuda")
                ctx.set_tuning(comet.TUNE_GEMM_TILE, tile)
                ctx.set_tuning(comet.TUNE_GEMM_GRID, grid)
                try:
                    if kind == "somm":
                        ctx.somm_share(1, bs, gi, n_dev, cap, e_d, f_d, a_d, b_d, c_d, neuron_major=fmt == "neuron_major", out=z)
                    else:
                        ctx.simm_share(1, bs, gi, n_dev, cap, e_d, f_d, a_d, b_d, c_d, out=z)
                    torch.cuda.synchronize()
                finally:
                    ctx.set_tuning(comet.TUNE_GEMM_TILE, 0)
                    ctx.set_tuning(comet.TUNE_GEMM_GRID, 0)
                got = down(z)
                if kind == "simm":
                    assert np.array_equal(got, want), tile
                else:
                    assert (not t or np.array_equal(got[:, :on], want)) and np.all(got[:, on:] == 77), tile


STAGED, WORDS = "ring_gemm_kernel<2, 2, 1, 1,", "ring_words_kernel<"


def either_kernel(ctx, call, kernel):
    """The kernel that takes the call, and the same words from the two kernels on words of 64-row tiles."""
    import paper_2505_07239_amd as comet
    ran, z = kernels(call), call().clone()
    assert len([name for name in ran if name.startswith(kernel)]) == 1, ran
    for tile, other in ((2, WORDS), (3, STAGED)):
        ctx.set_tuning(comet.TUNE_GEMM_TILE, tile)
        try:
            assert any(name.startswith(other) for name in kernels(call)) and torch.equal(call(), z)
        finally:
            ctx.set_tuning(comet.TUNE_GEMM_TILE, 0)


# Either side of the lines between the two kernels on words: one pair of steps per compute unit; even shares without teams that
# slices of twice as many workgroups would replace, slices a tenth longer, few slices; neuron-major weights; rows looked up one
# by one.
@pytest.mark.parametrize("kind,fmt,m,k,n,bs,kernel", [
    ("somm", "words", 64, 512, 1024, 32, STAGED), ("somm", "words", 64, 513, 1024, 32, WORDS), ("somm", "words", 40, 1001, 256, 32, STAGED),
    ("simm", "words", 64, 512, 1024, 32, STAGED), ("simm", "words", 64, 512, 1024, 16, STAGED), ("simm", "words", 64, 513, 1024, 27, WORDS),
    ("simm", "words", 64, 510, 1024, 30, WORDS), ("somm", "words", 400, 2560, 640, 32, STAGED), ("somm", "words", 400, 2560, 1024, 32, WORDS),
    ("somm", "words", 320, 1664, 2048, 32, WORDS), ("somm", "words", 150, 256, 3008, 32, STAGED), ("somm", "words", 128, 2560, 640, 32, WORDS),
    ("somm", "neuron_major", 150, 4096, 960, 32, STAGED), ("somm", "neuron_major", 256, 1024, 2560, 32, STAGED),
    ("somm", "neuron_major", 128, 2560, 640, 32, WORDS)])
def test_which_kernel_on_words(ctx, kind, fmt, m, k, n, bs, kernel):
    print("[gpu-words] %s %s m=%d k=%d n=%d bs=%d: %s" % (kind, fmt, m, k, n, bs, kernel), flush=True)
    draw = lambda *shape: torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda")
    t = (n if kind == "somm" else k) // bs
    idx = torch.arange(0, 2 * t, 2, dtype=torch.int32, device="cuda")
    c, z = draw(m, n), torch.empty((m, n), dtype=torch.int64, device="cuda")
    if kind == "somm":
        e, a, f, b = draw(m, k), draw(m, k), draw(k, n), draw(k, 2 * n)
        if fmt == "neuron_major":
            f, b = f.t().contiguous(), b.t().contiguous()
        call = lambda: ctx.somm_share(1, bs, idx, None, t, e, f, a, b, c, neuron_major=fmt == "neuron_major", out=z)
    else:
        e, a, f, b = draw(m, k), draw(m, 2 * k), draw(k, n), draw(2 * k, n)
        call = lambda: ctx.simm_share(1, bs, idx, None, t, e, f, a, b, c, out=z)
    either_kernel(ctx, call, kernel)


# The same with row sets (which lists a row tile has does not matter) and with result blocks.
@pytest.mark.parametrize("m,nb,bs,n,kernel", [(33, 60, 16, 96, STAGED), (64, 256, 32, 64, STAGED), (64, 257, 32, 64, WORDS),
                                              (65, 60, 16, 96, WORDS), (77, 512, 16, 512, STAGED), (77, 511, 16, 512, WORDS),
                                              (77, 512, 16, 513, WORDS), (128, 512, 16, 512, WORDS), (77, 171, 48, 96, WORDS)])
def test_which_kernel_with_row_sets(ctx, m, nb, bs, n, kernel):
    print("[gpu-words] row sets m=%d nb=%d bs=%d n=%d: %s" % (m, nb, bs, n, kernel), flush=True)
    draw = lambda *shape: torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda")
    mask = torch.from_numpy(((np.arange(m)[:, None] * 7 + np.arange(nb)[None, :] * 5) % 31 < 3).astype(np.uint8)).cuda()
    idx = torch.arange(nb, dtype=torch.int32, device="cuda")
    e, a, f, b, c = draw(m, nb * bs), draw(m, nb * bs), draw(nb * bs, n), draw(nb * bs, n), draw(m, n)
    z = torch.empty_like(c)
    either_kernel(ctx, lambda: ctx.simm_share_masked(1, bs, idx, None, nb, mask, e, f, a, b, c, out=z), kernel)


@pytest.mark.parametrize("m,nb,k,kernel", [(33, 60, 200, STAGED), (64, 128, 2048, STAGED), (64, 128, 2049, WORDS), (65, 60, 200, WORDS)])
def test_which_kernel_with_result_blocks(ctx, m, nb, k, kernel):
    print("[gpu-words] result blocks m=%d nb=%d k=%d: %s" % (m, nb, k, kernel), flush=True)
    draw = lambda *shape: torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda")
    mask = torch.from_numpy((np.arange(m)[:, None] % 3 == np.arange(nb)[None, :] % 3).astype(np.uint8)).cuda()
    cc = ctx.components(mask)
    e, a, f, b, c = draw(m, k), draw(m, k), draw(k, nb * 32), draw(k, nb * 32), draw(m, nb * 32)
    z = torch.zeros_like(c)
    either_kernel(ctx, lambda: ctx.somm_share_blocks(1, 32, cc["blk_idx"], cc["blk_comp"], cc["n_blk"], nb, cc["row_comp"], cc["n_row"],
                                                     e, f, a, b, c, out=z), kernel)


# Groups up to 32 rows share their launches whatever the size; more rows while the products are small (twenty units).
@pytest.mark.parametrize("kind", ["somm", "simm"])
@pytest.mark.parametrize("m,other,t,n_mem", [(5, 64, 3, 2), (32, 200, 9, 3), (33, 100, 5, 4), (65, 330, 20, 2), (128, 768, 40, 4)])
def test_small_groups(ctx, kind, m, other, t, n_mem):
    print("[gpu-words] group %s m=%d other=%d blocks=%d members=%d" % (kind, m, other, t, n_mem), flush=True)
    members, want, e0 = [], [], None
    for j in range(n_mem):
        idx, e, a, f, b, c, a_sel, b_sel = operands(kind, m, other, 16, t, True, 960 + j)
        e0 = (e, up(e)) if j % 2 == 0 else e0                                 # every second member shares its E
        want.append(co.beaver_share(j & 1, e0[0], f, a_sel, b_sel, c))
        members.append((j & 1, e0[1], ctx.open_weight_planes(up(f)), up(a), ctx.open_weight_planes(up(b)), up(c)))
    outs = ctx.share_group(kind, 16, torch.from_numpy(idx).cuda(), None, t, members)
    torch.cuda.synchronize()
    for z, w in zip(outs, want):
        assert np.array_equal(down(z), w)
