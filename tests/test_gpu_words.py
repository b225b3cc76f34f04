"""GPU parity of the share kernels that small products and products on weight words take: every output
element against the oracle's Eq. 1, at tile edges, remainders of the contraction and the longest runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle as co                                   # noqa: E402
from workloads import rng                             # noqa: E402


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


def check(ctx, kind, fmt, m, other, bs, t, full=True, party=1, **tuning):
    import paper_2505_07239_amd as comet
    print("[gpu-words] %s %s m=%d other=%d bs=%d blocks=%d full=%s %s" % (kind, fmt, m, other, bs, t, full, tuning), flush=True)
    idx, e, a, f, b, c, a_sel, b_sel = operands(kind, m, other, bs, t, full, 940)
    want = co.beaver_share(party, e, f, a_sel, b_sel, c)
    tr = fmt == "neuron_major"
    f_d, b_d = (up(f.T if tr else f), up(b.T if tr else b))
    if fmt == "planes":
        f_d, b_d = ctx.open_weight_planes(f_d), ctx.open_weight_planes(b_d)
    for key, value in tuning.items():
        ctx.set_tuning(getattr(comet, key), value)
    try:
        gi = torch.from_numpy(idx).cuda()
        if kind == "somm":
            z = ctx.somm_share(party, bs, gi, None, t, up(e), f_d, up(a), b_d, up(c), b_full=full,
                               **({"neuron_major": True} if tr else {}))
        else:
            z = ctx.simm_share(party, bs, gi, None, t, up(e), f_d, up(a), b_d, up(c), a_full=full, b_full=full)
        torch.cuda.synchronize()
    finally:
        for key in tuning:
            ctx.set_tuning(getattr(comet, key), 0)
    assert np.array_equal(down(z), want)


# Contraction lengths at the edges of a step (32), a pair (64) and the one-launch path (100 words).  tile 0: the one-launch
# path and the few-row kernel; 2: the 64 x 64 tile whatever the size.
@pytest.mark.parametrize("fmt", ["words", "planes", "neuron_major"])
@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("m", [9, 32, 33, 64, 130])
def test_small_somm(ctx, fmt, tile, m):
    for k in (1, 2, 31, 32, 33, 64, 65, 95, 97, 100, 101, 160, 193, 224):
        if fmt != "neuron_major" or k % 2 == 0:
            check(ctx, "somm", fmt, m, k, 5 if k % 3 == 0 and fmt == "words" else 16, 5, party=k & 1, TUNE_GEMM_TILE=tile)


# Blocks of 7 neurons (rows looked up one by one), of 16 (sixteen at a time) and of 32; compact operands.
@pytest.mark.parametrize("tile", [0, 2])
@pytest.mark.parametrize("m", [9, 32, 33, 64, 130])
@pytest.mark.parametrize("fmt,bs", [("words", 7), ("words", 16), ("words", 32), ("planes", 16), ("planes", 48)])
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


# How the contraction is shared out: a slice of one tile, even shares (72 tiles on 256 workgroups and on 7, which cut every
# tile at other places), two and four row tiles side by side, whole tiles.
@pytest.mark.parametrize("fmt", ["words", "planes"])
@pytest.mark.parametrize("m,k,n,grid", [(64, 200, 320, 0), (64, 300, 72 * 64, 0), (128, 300, 72 * 32, 0), (250, 260, 72 * 16, 0),
                                        (128, 300, 192, 7), (200, 330, 192, 4), (128, 100, 256, 8)])
def test_work_split(ctx, fmt, m, k, n, grid):
    check(ctx, "somm", fmt, m, k, 16, n // 16, TUNE_GEMM_TILE=2, TUNE_GEMM_GRID=grid)
    if grid == 0:
        check(ctx, "simm", fmt, m, n // 4, 16, k // 16, TUNE_GEMM_TILE=2)


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
