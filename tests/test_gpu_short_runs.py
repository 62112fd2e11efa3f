"""Run tables of short blocks (one run per lane, packed bytes in LDS) against the oracle: tile edges, remainders, runs up
to the longest the kernel takes and one past it, partial ranges, elements that share tiles, odd addresses."""
import numpy as np
import pytest

import oracle
from gpu_util import first_diff, to_dev, to_host, zeros_dev
from paper_2402_12274_amd import inputs

pytestmark = pytest.mark.gpu

# (blocks, mean, longest) and the packed ranges (offset, bytes; -1: all)
LAYOUTS = [(3, 400, 512), (300, 3, 40), (900, 24, 256), (5000, 24, 512), (5000, 24, 513), (2500, 120, 512), (20000, 1, 2)]


@pytest.mark.parametrize("n,mean,longest", LAYOUTS)
@pytest.mark.parametrize("count,off,nbytes,shift", [(1, 0, -1, 0), (2, 0, -1, 3), (1, 5, 4096, 0), (1, 1000, 1023, 7),
                                                    (3, 77, -1, 15), (2, 17, 65537, 1)])
def test_pack_unpack(n, mean, longest, count, off, nbytes, shift):
    from paper_2402_12274_amd import mdt

    lens, disps = inputs.hindexed_blocks(nblocks=n, span=n * (mean + 200) + 4096, mean=float(mean), maxlen=longest, seed=n)
    lens[n // 2] = longest  # the longest run is there, in a gap of its own past the others
    disps[n // 2] = n * (mean + 200) + 8192 + 3
    spec = ("resized", 0, n * (mean + 200) + 16384, inputs.hindexed_type(lens, disps))
    t, o = mdt.build_type(spec), oracle.build_type(spec)
    host = inputs.random_bytes(count * spec[2], seed=mean)
    ref = o.pack(host, 0, count, off, nbytes)
    if ref.size == 0:
        pytest.skip("range past the stream")
    src, out = to_dev(host), zeros_dev(ref.size + 32, 0xEE)
    assert mdt.mdt_pack(src.data_ptr(), count, t, off, out.data_ptr() + shift, nbytes) == ref.size
    got = to_host(out)
    assert first_diff(got[shift:shift + ref.size], ref) is None
    assert (got[:shift] == 0xEE).all() and (got[shift + ref.size:] == 0xEE).all()
    want = np.full(host.size, 0xCD, np.uint8)
    o.unpack(ref, want, 0, count, off)
    for batched in (False, True):
        back = zeros_dev(host.size, 0xCD)
        if batched:
            b, s = mdt.Batch(), mdt.Stream()
            b.add_unpack(out.data_ptr() + shift, ref.size, back.data_ptr(), count, t, off)
            b.launch(s)
        else:
            mdt.mdt_unpack(out.data_ptr() + shift, ref.size, back.data_ptr(), count, t, off)
        assert first_diff(to_host(back), want) is None
