"""GPU parity of the packing of the activations where their words are fetched one by one: odd row lengths, indexed A_i with
blocks of any length, the remainder of a 64-word piece, per-token row sets.  Every output element against the oracle's Eq. 1."""
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


def u64(seed, stream, *shape):
    return rng.uniform_u64(seed, stream, int(np.prod(shape))).reshape(shape)


# Rows around a tile of 64 and the 32 rows of the few-row kernel; pieces of 64 words that are whole, end early and start past
# the end of the contraction; blocks that divide 64 and blocks that straddle it.
@pytest.mark.parametrize("row_sets", [False, True])
@pytest.mark.parametrize("m", [9, 32, 33, 64, 65, 130])
@pytest.mark.parametrize("bs,t", [(1, 127), (3, 64), (16, 9), (21, 7), (24, 8), (32, 7), (48, 5), (65, 3)])
def test_word_by_word(ctx, bs, t, m, row_sets):
    print("[gpu-pack] m=%d bs=%d blocks=%d row_sets=%s" % (m, bs, t, row_sets), flush=True)
    n, party = 40, t & 1
    idx = np.arange(1, 2 * t, 2, dtype=np.int32)
    e, a, f, b, c = u64(970, 1, m, t * bs), u64(970, 2, m, 2 * t * bs), u64(970, 3, t * bs, n), u64(970, 4, 2 * t * bs, n), \
        u64(970, 5, m, n)
    a_sel, b_sel, e_sel = co.index_cols(a, idx, bs), co.index_rows(b, idx, bs), e
    if row_sets:
        mask = (np.arange(m)[:, None] * 7 + np.arange(2 * t)[None, :] * 5) % 3 != 0
        on = np.repeat(mask[:, idx], bs, axis=1)
        a_sel, e_sel = np.where(on, a_sel, np.uint64(0)), np.where(on, e, np.uint64(0))
    want = co.beaver_share(party, e_sel, f, a_sel, b_sel, c)
    gi = torch.from_numpy(idx).cuda()
    if row_sets:
        z = ctx.simm_share_masked(party, bs, gi, None, t, torch.from_numpy(mask.astype(np.uint8)).cuda(), up(e), up(f), up(a),
                                  up(b), up(c))
    else:
        z = ctx.simm_share(party, bs, gi, None, t, up(e), up(f), up(a), up(b), up(c), a_full=True, b_full=True)
    torch.cuda.synchronize()
    assert np.array_equal(z.cpu().numpy().view(np.uint64), want)


@pytest.mark.parametrize("m", [9, 33, 64, 130])
@pytest.mark.parametrize("k", [101, 127, 128, 129, 191, 255])
def test_odd_row_length(ctx, k, m):
    print("[gpu-pack] m=%d k=%d" % (m, k), flush=True)
    idx = np.arange(0, 6, 2, dtype=np.int32)
    e, a, f, b, c = u64(971, 1, m, k), u64(971, 2, m, k), u64(971, 3, k, 48), u64(971, 4, k, 96), u64(971, 5, m, 48)
    want = co.beaver_share(k & 1, e, f, a, co.index_cols(b, idx, 16), c)
    z = ctx.somm_share(k & 1, 16, torch.from_numpy(idx).cuda(), None, 3, up(e), up(f), up(a), up(b), up(c), b_full=True)
    torch.cuda.synchronize()
    assert np.array_equal(z.cpu().numpy().view(np.uint64), want)
