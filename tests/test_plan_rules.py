"""The split rules of the plans on the CPU, through the C ABI: a finer split
never takes a shape away from the entry point with the fixed scratch, nor from a
workspace that is kept while max_seqlen changes."""
import ctypes

import pytest

from paper_2606_07317_amd import gbla

ALIGNED = 1 << 20


@pytest.fixture(scope="module")
def lib():
    return gbla.load_library()


def _coarse_bytes(batch, heads, n, d, ragged):
    """Scratch of the fp32 forward with state units of at least 256 tokens."""
    tokens = n if ragged else batch * n
    chunk = 256
    while chunk < 2048 and chunk * 256 < tokens * heads:
        chunk *= 2
    rec = (d * d + d + 2 + 63) // 64 * 64 * 4
    frag = (d // 16 + 1) * (d // 32) * 64 * 32
    units = tokens // chunk + batch
    up = lambda x: (x + 255) // 256 * 256
    return up(up(units * heads * rec) + batch * heads * up(frag))


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_fp32_noalloc_still_takes_what_the_coarse_split_fits(lib, d, ragged):
    """Status 4 is the refusal; an accepted call ends in the HIP runtime, which
    has no device here (status 5).  The kernels are not reached on a CPU."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch on the fake pointers")
    taken = 0
    for heads in (1, 2, 3, 8, 16):
        for batch in (1, 2, 7, 16, 40, 55, 60, 110, 200):
            for n in (0, 1, 63, 64, 65, 300, 999, 2048, 4000, 8191, 16384, 32768):
                if _coarse_bytes(batch, heads, n, d, ragged) > gbla.NOALLOC_SCRATCH_BYTES:
                    continue
                s = gbla.Shape(batch, heads, n, d, 4, n if ragged else 0, gbla.GBLA_F32, 1e-6, 0)
                args = [ALIGNED] * 7 + [ALIGNED if ragged else None, ALIGNED, None]
                assert lib.gbla_forward_noalloc(ctypes.byref(s), *args) != 4, (batch, heads, n)
                taken += 1
    assert taken > 50


def _backward_need(lib, shape):
    """Smallest workspace that the ragged gbla_backward call does not refuse."""
    lo, hi = 0, 1 << 33
    while lo < hi:
        mid = (lo + hi) // 2
        args = [ALIGNED] * 7 + [ALIGNED] * 3 + [mid] + [ALIGNED] * 7 + [None]
        if lib.gbla_backward(ctypes.byref(shape), *args) == 4:
            lo = mid + 1
        else:
            hi = mid
    return lo


@pytest.mark.parametrize("d", [32, 64, 128])
def test_backward_workspace_serves_every_max_seqlen(lib, d):
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch on the fake pointers")
    for heads, batch, T in ((1, 1, 60000), (4, 3, 2000), (8, 40, 30000), (3, 7, 255)):
        need = set()
        for longest in (0, 1, 100, 700, 5000, 20000, T, 1 << 30):
            s = gbla.Shape(batch, heads, T, d, 4, longest, gbla.GBLA_BF16, 1e-6, 0)
            need.add(_backward_need(lib, s))
            assert gbla.backward_workspace_bytes(s) >= max(need)
        assert len(need) == 1, (heads, batch, T, need)
