"""The native marshalling of the binding against the binding's own way through every form a call accepts, and what
it has to decline."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def both():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_07239_amd as comet
    native, plain = comet.Context(0), comet.Context(0)
    plain._host.close()
    plain._host = comet.binding._NoHost(plain.h.value, 0)      # what stands in its place where it is missing
    assert type(native._host).__name__ == "Host"
    yield native, plain
    native.close(), plain.close()


def words(*shape):
    return torch.randint(-2 ** 63, 2 ** 63 - 1, shape, dtype=torch.int64, device="cuda")


def i32(*values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def same(both, call):
    """The call through both contexts: equal tensors, or the same exception with the same message."""
    got = []
    for ctx in both:
        try:
            r = call(ctx)
            got.append([t.clone() for t in (r if isinstance(r, (list, tuple)) else [getattr(r, "buf", r)])])
        except Exception as err:                              # noqa: BLE001
            got.append((type(err), str(err)))
    a, b = got
    if isinstance(a, tuple) or isinstance(b, tuple):
        assert a == b
        return False
    assert len(a) == len(b) and all(x.shape == y.shape and torch.equal(x, y) for x, y in zip(a, b))
    return True


def test_streaming_calls(both):
    x, a, idx, n = words(6, 40), words(6, 40), i32(0, 2), i32(2)
    for call in ("mask_share", "open"):
        assert same(both, lambda c: getattr(c, call)(x, a))
        assert same(both, lambda c: getattr(c, call)(x.view(-1), a, out=torch.empty_like(x)))    # numbers of words, not shapes
        for bad in (a[:, ::2], a[:3], a.to(torch.int32), a.cpu(), None):
            assert not same(both, lambda c: getattr(c, call)(x, bad))
        assert not same(both, lambda c: getattr(c, call)(x, a, out=torch.empty(3, dtype=torch.int64, device="cuda")))
    for axis, bs in ((0, 8), (1, 2)):
        assert same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx, n, 2))
        assert same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx, None, 2))
        same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx, n, 0))
        assert not same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx, None, 3))       # more than the list holds
        assert not same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx.long(), n, 2))
        assert not same(both, lambda c: c.mask_share_gather(x, a, axis, bs, idx, n, 200))
    assert not same(both, lambda c: c.mask_share_gather(x, a, 7, 2, idx, n, 2))
    for nm in (False, True):
        # (columns beyond the matrix are padding that no call writes or reads)
        buf = torch.zeros(64 * 64 * 8, dtype=torch.uint8, device="cuda")
        assert same(both, lambda c: c.open_weight_planes(x, a, out=buf.zero_(), neuron_major=nm))
        assert same(both, lambda c: c.open_weight_planes(x, out=buf.zero_(), neuron_major=nm))
        assert not same(both, lambda c: c.open_weight_planes(x, a[:3], neuron_major=nm))
        assert not same(both, lambda c: c.open_weight_planes(x, a, out=buf[:16], neuron_major=nm))
    for mask in (torch.ones(70, dtype=torch.uint8, device="cuda"), (torch.rand(5, 70, device="cuda") < 0.3).to(torch.uint8)):
        assert same(both, lambda c: c.compact_mask(mask, torch.zeros(70, dtype=torch.int32, device="cuda"), i32(0)))
        assert not same(both, lambda c: c.compact_mask(mask.bool()))


@pytest.mark.parametrize("fmt", ["words", "planes", "neuron_major"])
@pytest.mark.parametrize("kind", ["somm", "simm"])
def test_share_calls(both, kind, fmt):
    m, k, bs, t, nb = 9, 48, 16, 2, 5
    idx, n = i32(0, 3), i32(t)
    somm, tr = kind == "somm", fmt == "neuron_major"
    if tr and not somm:
        pytest.skip("neuron-major weights belong to SOMM")
    turn = (lambda w: w.t().contiguous()) if tr else (lambda w: w)
    pack = (lambda c, w: c.open_weight_planes(w)) if fmt == "planes" else (lambda c, w: w)
    kw = dict(neuron_major=True) if tr else {}
    e, a, c_i = (words(m, k), words(m, k), words(m, t * bs)) if somm else (words(m, t * bs), words(m, nb * bs), words(m, k))
    f, b = (turn(words(k, t * bs)), turn(words(k, nb * bs))) if somm else (words(t * bs, k), words(nb * bs, k))

    def share(c, e=e, f=f, a=a, b=b, z=None, party=1, idx=idx, n=n, cap=t, block=bs, **more):
        call = c.somm_share if somm else c.simm_share
        return call(party, block, idx, n, cap, e, pack(c, f), a, pack(c, b), c_i, out=z, **kw, **more)

    assert same(both, share)
    assert same(both, lambda c: share(c, z=torch.empty_like(c_i), party=0))
    assert same(both, lambda c: share(c, n=None))
    compact = turn(words(k, t * bs)) if somm else words(t * bs, k)
    assert same(both, lambda c: share(c, b=compact, b_full=False, **({} if somm else dict(a_full=True))))
    for bad in (dict(party=2), dict(e=e[:, 1:]), dict(e=e.cpu()), dict(a=a[:3]), dict(cap=3), dict(cap=-1), dict(idx=None), dict(idx=idx.long()),
                dict(n=n.long()), dict(z=torch.empty(2, 2, dtype=torch.int64, device="cuda")), dict(b=compact), dict(block=np.int64(bs))):
        same(both, lambda c: share(c, **bad))                 # the same answer, whichever it is
    if fmt != "neuron_major":
        members = [(j, e, f, a, b, c_i) for j in (0, 1)]
        group = lambda c, ms, **more: c.share_group(kind, bs, idx, n, t, [(p, x, pack(c, y), u, pack(c, v), w) for p, x, y, u, v, w in ms],
                                                    **more)
        assert same(both, lambda c: group(c, members))
        assert same(both, lambda c: group(c, members[:1], out=[torch.empty_like(c_i)]))
        assert same(both, lambda c: group(c, members, out=(torch.empty_like(c_i), torch.empty_like(c_i))))
        for bad in ([None, None], [torch.empty_like(c_i), None], [torch.empty_like(c_i)], [torch.empty_like(c_i), 3]):
            assert not same(both, lambda c: group(c, members, out=list(bad)))
        assert not same(both, lambda c: group(c, []))
        assert not same(both, lambda c: group(c, members * 5))
        assert not same(both, lambda c: group(c, [members[0], (1, e[:4].contiguous(), f, a[:4].contiguous(), b, c_i[:4].contiguous())]))
        assert not same(both, lambda c: group(c, [(0, e, f, a, b[:, :8].contiguous(), c_i)]))
    if fmt == "words":
        e8, a8, c8 = e[:8].contiguous(), a[:8].contiguous(), c_i[:8].contiguous()
        g = words(*f.shape)
        un = lambda c, g1, **more: (c.somm_share_unopened if somm else c.simm_share_unopened)(1, bs, idx, n, t, e8, f, g1, a8, b, c8, **more)
        assert same(both, lambda c: un(c, g))
        assert not same(both, lambda c: un(c, None))
        assert not same(both, lambda c: un(c, g[:8].contiguous()))


def test_what_is_not_plain_is_declined(both):
    native = both[0]
    x = words(4, 4)

    class Sub(torch.Tensor):
        pass

    for t in (x.as_subclass(Sub), x.cpu(), x.double(), x.t(), None, 3):
        if t is not None and isinstance(t, torch.Tensor) and t.is_cuda and t.dtype == torch.int64 and t.is_contiguous():
            assert native._host.elementwise(False, t, t, None) is None and native.mask_share(t, x).shape == x.shape
        assert native._host.elementwise(False, t, x, None) is None
        assert native._host.open_planes(t, None, None, False) is None
    assert native._host.elementwise(0, x, x, None) is None and native._host.elementwise(False, x, x) is None
    assert native._host.gather(x, x, 0, 1.0, i32(0), None, 1, None) is None
    assert native._host.compact(None, torch.ones(5000, dtype=torch.uint8, device="cuda"), i32(0), i32(0)) is None   # no workspace
    torch.cuda.synchronize()


def test_current_stream_and_capture(both):
    """The native part follows torch's current stream, also while it is captured."""
    x, a = words(64, 512), words(64, 512)
    want = x - a
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    out = torch.empty_like(x)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        both[0].mask_share(x, a, out=out)
    s.synchronize()
    assert torch.equal(out, want)
    with torch.cuda.graph(g, stream=s):
        both[0].mask_share(x, a, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def test_an_allocation_that_fails_leaves_nothing_behind(both):
    """The second result of a group does not fit: the exception is torch's, and the first one is given back."""
    import gc
    m, k, bs, t = 8192, 2, 16, 64                             # results of 64 MB
    idx, e, a, c_i = i32(*range(t)), words(m, k), words(m, k), words(m, t * bs)
    f, b = words(k, t * bs), words(k, t * bs)
    both[0].workspace(1 << 26)
    gc.collect()
    torch.cuda.empty_cache()
    before, total = torch.cuda.memory_allocated(), torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (100 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            both[0].share_group("somm", bs, idx, None, t, [(j, e, f, a, b, c_i) for j in (0, 1)])
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    gc.collect()
    assert torch.cuda.memory_allocated() == before
