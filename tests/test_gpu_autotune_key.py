"""The file of saved tunings: entries of batches that run other kernels, or that an older library timed, are not taken."""
import pytest

from gpu_util import zeros_dev
from paper_2402_12274_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    from gpu_util import torch_cuda

    torch = torch_cuda()
    from paper_2402_12274_amd import mdt

    return torch, mdt


def _runs(a, b, n=4000):
    """n records of 512 bytes that hold a run of a bytes and, 192 bytes on, one of b."""
    return ("contiguous", n, ("resized", 0, 512, ("struct", [a, b], [0, 192], [inputs.BYTE] * 2)))


def _batch(mdt, t, src, out):
    b = mdt.Batch()
    b.add_pack(src.data_ptr(), 1, t, 0, out.data_ptr(), -1)
    return b


def test_layouts_that_run_other_kernels_are_timed_apart(env, tmp_path, monkeypatch):
    # equal kind of layout, size, runs and bytes: the first has runs of one length and spacing, which the chunk kernels
    # locate through the compact program, the second has not
    torch, mdt = env
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("MDT_AUTOTUNE_CACHE", str(cache))
    ms = mdt.Stream(torch.cuda.current_stream().cuda_stream)
    types = [mdt.build_type(_runs(96, 96)), mdt.build_type(_runs(64, 128))]
    assert types[0].layout_info() == types[1].layout_info() and types[0].size() == types[1].size()
    src, out = zeros_dev(4000 * 512), zeros_dev(4000 * 192)
    for i, t in enumerate(types):
        _batch(mdt, t, src, out).autotune(ms)
        assert cache.read_text().count('": [') == i + 1


def _fnv1a(h, v):
    for byte in int(v).to_bytes(8, "little"):
        h = ((h ^ byte) * 1099511628211) & (2 ** 64 - 1)
    return h


def test_choices_of_older_kernels_are_timed_again(env, tmp_path, monkeypatch):
    # the key as it was while the chunk kernels had the general program only: library version 100, compute units, and of
    # the one request direction, body (4: chunk) and kind (2: one group), type size, runs, bits of the packed bytes
    torch, mdt = env
    ms = mdt.Stream(torch.cuda.current_stream().cuda_stream)
    t = mdt.build_type(_runs(96, 96))
    h = 1469598103934665603
    for v in (100, torch.cuda.get_device_properties(0).multi_processor_count, 4 << 32 | 2, t.size(), 8000,
              t.size().bit_length()):
        h = _fnv1a(h, v)
    cache = tmp_path / "tune.json"
    cache.write_text('{\n  "%016x-1": [2048, 0, 2, 0, 0]\n}\n' % h)  # a tile that no tuning tries
    monkeypatch.setenv("MDT_AUTOTUNE_CACHE", str(cache))
    src, out = zeros_dev(4000 * 512), zeros_dev(4000 * 192)
    cfg = _batch(mdt, t, src, out).autotune(ms)
    assert mdt.config_dict(cfg)["tile_chunks"] != 2048
    assert cache.read_text().count('": [') == 2
