"""The chunk kernels of regular layouts at the edges of what their compact 32-bit program takes: every number of levels that a
kernel is compiled for and one more, elements just below and just past 2^30 bytes, extents past 32 bits, and typed copies
between two such layouts with counts on both sides."""
import numpy as np
import pytest

from gpu_util import first_diff, to_dev, to_host, zeros_dev
from oracle import build_type as obuild
from paper_2402_12274_amd import inputs

pytestmark = pytest.mark.gpu

COUNTS = [9, 3, 2, 3, 2, 3, 2]


@pytest.fixture(scope="module")
def env():
    from gpu_util import torch_cuda

    torch = torch_cuda()
    from paper_2402_12274_amd import mdt

    return torch, mdt


def _nest(levels, run, negative=False, gap=0):
    """(spec, bytes before the origin) of `levels` loops, none of which merge, over one run."""
    spec, step, before = ("contiguous", run, inputs.BYTE), run + 80 + gap, 0
    for i, n in enumerate(COUNTS[:levels]):
        back = negative and i % 2
        spec = ("hvector", n, 1, -step if back else step, spec)
        before += (n - 1) * step if back else 0
        step = n * step + 13
    return ("resized", 0, step + 100, spec), before


@pytest.mark.parametrize("negative", [False, True])
@pytest.mark.parametrize("levels", range(8))
def test_every_number_of_levels(env, levels, negative):
    torch, mdt = env
    spec, before = _nest(levels, 24 if levels else 72, negative)
    t, o = mdt.build_type(spec), obuild(spec)
    count = 70000 // t.size() + 2
    host = inputs.random_bytes(before + count * spec[2] + 64, seed=levels)
    src = to_dev(host)
    ms = mdt.Stream(torch.cuda.current_stream().cuda_stream)
    total = count * t.size()
    for i, (off, nbytes) in enumerate([(0, -1), (t.size() - 5, 4096 * 16 + 11), (16 * 256 - 7, 16 * 256 + 14), (total - 33, -1)]):
        ref = o.pack(host, before, count, off, nbytes)
        want = np.full(host.size, 0xCD, np.uint8)
        o.unpack(ref, want, before, count, off)
        shift = 3 * i
        for batched in (False, True):
            out, back = zeros_dev(ref.size + 32, 0xEE), zeros_dev(host.size, 0xCD)
            if batched:
                b = mdt.Batch()
                b.add_pack(src.data_ptr() + before, count, t, off, out.data_ptr() + shift, nbytes)
                b.add_unpack(out.data_ptr() + shift, ref.size, back.data_ptr() + before, count, t, off)
                b.launch(ms)
            else:
                mdt.mdt_pack(src.data_ptr() + before, count, t, off, out.data_ptr() + shift, nbytes)
                mdt.mdt_unpack(out.data_ptr() + shift, ref.size, back.data_ptr() + before, count, t, off)
            got = to_host(out)
            assert first_diff(got[shift:shift + ref.size], ref) is None, (off, nbytes, batched)
            assert (got[:shift] == 0xEE).all() and (got[shift + ref.size:] == 0xEE).all(), (off, nbytes, batched)
            assert first_diff(to_host(back), want) is None, (off, nbytes, batched)


@pytest.mark.parametrize("runs", [4329604, 4329605])
def test_elements_around_the_size_limit(env, runs):
    # runs of 248 bytes in 264: 2^30 - 32 bytes of data, and 216 past 2^30
    torch, mdt = env
    t = mdt.build_type(("contiguous", runs, ("resized", 0, 264, ("contiguous", 248, inputs.BYTE))))
    size, count = t.size(), 2
    assert (size < 1 << 30) == (runs == 4329604)
    g = torch.Generator(device="cuda")
    g.manual_seed(runs)
    src = torch.randint(0, 256, (count * runs * 264,), dtype=torch.uint8, device="cuda", generator=g)
    ref = src.view(-1, 264)[:, :248].reshape(-1)
    windows = [(0, 1 << 20), (size - 100003, 300007), (size - 5, 11), (2 * size - 70001, 70001)]
    for off, nbytes in windows:
        out = zeros_dev(nbytes + 16, 0xEE)
        assert mdt.mdt_pack(src.data_ptr(), count, t, off, out.data_ptr() + 5, nbytes) == nbytes
        assert torch.equal(out[5:5 + nbytes], ref[off:off + nbytes]), (off, nbytes)
        assert bool((out[:5] == 0xEE).all()) and bool((out[5 + nbytes:] == 0xEE).all())
    out = torch.empty_like(ref)
    assert mdt.mdt_pack(src.data_ptr(), count, t, 0, out.data_ptr(), -1) == 2 * size
    assert torch.equal(out, ref)
    back = torch.full_like(src, 0xCD)
    mdt.mdt_unpack(out.data_ptr(), 2 * size, back.data_ptr(), count, t, 0)
    assert torch.equal(back.view(-1, 264)[:, :248].reshape(-1), ref)
    assert bool((back.view(-1, 264)[:, 248:] == 0xCD).all())


def test_extent_past_32_bits(env):
    # one element has the compact program, a count of them the general one
    torch, mdt = env
    extent = (3 << 30) + 40
    one = ("vector", 3000, 3, 17, inputs.DOUBLE)
    t, o = mdt.build_type(("resized", 0, extent, one)), obuild(one)
    span = o.attrs()["true_ub"]
    hosts = [inputs.random_bytes(span, seed=s) for s in (1, 2)]
    src = torch.zeros(extent + span, dtype=torch.uint8, device="cuda")
    src[:span], src[extent:] = to_dev(hosts[0]), to_dev(hosts[1])
    ref = np.concatenate([o.pack(h, 0, 1) for h in hosts])
    for count, off, nbytes in [(1, 0, -1), (2, 0, -1), (2, 71999, 4), (2, 5, 20000), (2, 72000, 72000)]:
        want = ref[off:off + nbytes] if nbytes >= 0 else ref[off:72000 * count]
        out = zeros_dev(want.size, 0)
        assert mdt.mdt_pack(src.data_ptr(), count, t, off, out.data_ptr(), nbytes) == want.size
        assert first_diff(to_host(out), want) is None, (count, off, nbytes)
        back = torch.full_like(src, 0xCD)
        mdt.mdt_unpack(out.data_ptr(), want.size, back.data_ptr(), count, t, off)
        full = np.full(2 * span, 0xCD, np.uint8)
        for e in range(2):
            lo, hi = max(off - 72000 * e, 0), min(off + want.size - 72000 * e, 72000)
            if lo < hi:
                o.unpack(want[72000 * e + lo - off:72000 * e + hi - off], full[e * span:(e + 1) * span], 0, 1, lo)
        got = np.concatenate([to_host(back[:span]), to_host(back[extent:])])
        assert first_diff(got, full) is None, (count, off, nbytes)
        assert bool((back[span:extent] == 0xCD).all())


@pytest.mark.parametrize("levels", [(0, 6), (6, 1), (3, 3), (5, 2)])
@pytest.mark.parametrize("nbytes", [60000, 9 << 20])
def test_copies_with_counts_on_both_sides(env, levels, nbytes):
    # tiles of 256 chunks below 8 MiB and of 1024 from there on; runs of 24 against runs of 20, 72 or 100 bytes
    torch, mdt = env
    (a, _), (b, _) = _nest(levels[0], 24 if levels[0] else 72), _nest(levels[1], 20 if levels[1] % 2 else 100, gap=8)
    ta, tb, oa, ob = mdt.build_type(a), mdt.build_type(b), obuild(a), obuild(b)
    ca = nbytes // ta.size() + 2
    cb = ca * ta.size() // tb.size() + 2
    host = inputs.random_bytes(ca * a[2], seed=sum(levels))
    src = to_dev(host)
    total = ca * ta.size()
    for off, mx in [(0, -1), (ta.size() - 3, 16 * 256 + 1), (tb.size() - 3, nbytes // 2), (total - 17, -1)]:
        stream = oa.pack(host, 0, ca, off, mx)
        want = np.full(cb * b[2], 0xA5, np.uint8)
        ob.unpack(stream, want, 0, cb, off)
        dst = zeros_dev(want.size, 0xA5)
        assert mdt.mdt_typed_copy(src.data_ptr(), ca, ta, dst.data_ptr(), cb, tb, off, mx) == stream.size
        assert first_diff(to_host(dst), want) is None, (off, mx)
