"""Run tables in batches against the oracle: tables of short runs (one run per lane) and of longer ones (a cached slice of
the table, each chunk's runs searched), packed, unpacked and relayed over whole and partial ranges, at every kind of
launch and tile size, and the longer ones in single launches too."""
import numpy as np
import pytest

from gpu_util import first_diff, note, to_dev, to_host, zeros_dev
from oracle import build_type as obuild
from paper_2402_12274_amd import inputs

pytestmark = pytest.mark.gpu

CONFIGS = [(1024, 4, 0, 1, 0), (256, 4, 1, 0, 0), (1024, 0, 2, 0, 0), (4096, 0, 2, 1, 1), (2048, 2, 0, 0, 1)]
# (offset, bytes; -1: all): tile edges, a range inside one tile, one that ends in the middle of a chunk
RANGES = [(0, -1), (5, 4099), (16 * 1024 - 3, 16 * 1024 + 6), (1000, 50001)]


@pytest.fixture(scope="module")
def env():
    from gpu_util import torch_cuda

    torch = torch_cuda()
    from paper_2402_12274_amd import mdt

    return torch, mdt


def _spec(n, mean, longest):
    """n runs of at most `longest` bytes, one of them that long, and an extent that leaves a gap behind them."""
    lens, disps = inputs.hindexed_blocks(nblocks=n, span=n * (mean + 60) + 4096, mean=float(mean), maxlen=longest, seed=n + mean)
    lens[n // 3] = longest
    disps[n // 3] = n * (mean + 60) + 8192 + 5
    return ("resized", 0, n * (mean + 60) + 16384 + longest, inputs.hindexed_type(lens, disps))


def _check(env, spec, count, relay_to=None):
    torch, mdt = env
    ms = mdt.Stream(torch.cuda.current_stream().cuda_stream)
    t, o = mdt.build_type(spec), obuild(spec)
    host = inputs.random_bytes(count * spec[2], seed=count)
    src = to_dev(host)
    for cfg in CONFIGS:
        bp, bu, br = mdt.Batch(), mdt.Batch(), mdt.Batch()
        keep = []
        for i, (off, nbytes) in enumerate(RANGES):
            ref = o.pack(host, 0, count, off, nbytes)
            if ref.size == 0:
                continue
            shift = 7 * i % 16
            out, pk = zeros_dev(ref.size + 32, 0xEE), zeros_dev(ref.size + 32, 0)
            pk[shift:shift + ref.size] = to_dev(ref)
            want = np.full(host.size, 0xCD, np.uint8)
            o.unpack(ref, want, 0, count, off)
            back = zeros_dev(host.size, 0xCD)
            assert bp.add_pack(src.data_ptr(), count, t, off, out.data_ptr() + shift, nbytes) == ref.size
            bu.add_unpack(pk.data_ptr() + shift, ref.size, back.data_ptr(), count, t, off)
            item = [pk, shift, ref, out, want, back]
            if relay_to is not None:
                t2, o2 = mdt.build_type(relay_to), obuild(relay_to)
                far = np.full(relay_to[2], 0x5A, np.uint8)
                o2.unpack(ref, far, 0, 1, off)
                mid, dst = zeros_dev(ref.size + 32, 0xEE), zeros_dev(relay_to[2], 0x5A)
                br.add_relay(src.data_ptr(), count, t, mid.data_ptr() + shift, dst.data_ptr(), 1, t2, off, nbytes)
                item += [mid, far, dst]
            keep.append(item)
        for b in (bp, bu, br) if relay_to is not None else (bp, bu):
            note(f"run table batch cfg={cfg} requests={len(keep)}")
            b.set_config(mdt.BatchConfig(*cfg))
            b.launch(ms)
            torch.cuda.synchronize()
        for _, shift, ref, out, want, back, *relay in keep:
            for buf in [out] + relay[:1]:
                got = to_host(buf)
                assert first_diff(got[shift:shift + ref.size], ref) is None, cfg
                assert (got[:shift] == 0xEE).all() and (got[shift + ref.size:] == 0xEE).all(), cfg
            assert first_diff(to_host(back), want) is None, cfg
            if relay:
                assert first_diff(to_host(relay[2]), relay[1]) is None, cfg


def _table(total, run, gap):
    """A table of runs of `run` bytes that holds at least `total`, and the extent that it lies in."""
    n = total // run + 1
    return ("resized", 0, n * (run + gap) + 64, inputs.hindexed_type(np.full(n, run, np.int64), np.arange(n) * (run + gap) + 3))


# runs of a few bytes: a step of 1024 chunks is many runs for each lane; 200 runs an element: steps of several elements
@pytest.mark.parametrize("n,mean,longest,count", [(30000, 1, 2, 1), (12000, 12, 512, 1), (9000, 24, 256, 1), (900, 100, 512, 3),
                                                  (200, 24, 256, 40)])
def test_short_runs(env, n, mean, longest, count):
    spec = _spec(n, mean, longest)
    total = obuild(spec).attrs()["size"] * count
    _check(env, spec, count, _table(total, 40, 10))


# one run past the longest that a lane takes alone, a mean past theirs, runs longer than a tile's step of chunks; counts
# of such elements
LONG = [(5000, 24, 513, 1), (5000, 24, 513, 2), (900, 200, 4096, 1), (700, 220, 500, 3), (300, 400, 40000, 1)]


@pytest.mark.parametrize("n,mean,longest,count", LONG)
def test_longer_runs(env, n, mean, longest, count):
    spec = _spec(n, mean, longest)
    total = obuild(spec).attrs()["size"] * count
    _check(env, spec, count, _table(total, 700, 30))


@pytest.mark.parametrize("short_src", [False, True])
def test_relay_between_short_and_longer_runs(env, short_src):
    spec = _spec(4000, 24, 256 if short_src else 513)
    total = obuild(spec).attrs()["size"]
    _check(env, spec, 1, _table(total, 700 if short_src else 40, 20))


@pytest.mark.parametrize("n,mean,longest,count", LONG)
def test_longer_runs_single_launches(env, n, mean, longest, count):
    torch, mdt = env
    spec = _spec(n, mean, longest)
    t, o = mdt.build_type(spec), obuild(spec)
    host = inputs.random_bytes(count * spec[2], seed=n)
    src = to_dev(host)
    for i, (off, nbytes) in enumerate(RANGES):
        ref = o.pack(host, 0, count, off, nbytes)
        shift = 5 * i % 16
        out, back = zeros_dev(ref.size + 32, 0xEE), zeros_dev(host.size, 0xCD)
        assert mdt.mdt_pack(src.data_ptr(), count, t, off, out.data_ptr() + shift, nbytes) == ref.size
        got = to_host(out)
        assert first_diff(got[shift:shift + ref.size], ref) is None, (off, nbytes)
        assert (got[:shift] == 0xEE).all() and (got[shift + ref.size:] == 0xEE).all(), (off, nbytes)
        want = np.full(host.size, 0xCD, np.uint8)
        o.unpack(ref, want, 0, count, off)
        mdt.mdt_unpack(out.data_ptr() + shift, ref.size, back.data_ptr(), count, t, off)
        assert first_diff(to_host(back), want) is None, (off, nbytes)
