"""The placement probe's own pass on the real memory."""

import gc

import numpy as np
import pytest
import torch

from paper_2410_11998_amd import binding as B

DEV = "cuda:0"
GIB = 1 << 30


@pytest.fixture(autouse=True)
def memory_goes_back():
    gc.collect()
    torch.cuda.empty_cache()
    yield
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.gpu
def test_the_probe_copies_inside_the_chunks_it_names_and_nowhere_else():
    """Three chunks: the sources of a chunk keep their contents, its outputs hold copies of sources, all else is untouched."""
    chunk, step, buf = B.PROBE_CHUNK_BYTES, B.PROBE_STEP_BYTES, 64 << 20
    span = 2 * step + chunk
    arena = torch.empty((span + (64 << 20)) // 4, dtype=torch.float32, device=DEV)
    part = arena[:arena.numel()].view(-1, buf // 4)
    for k in range(part.shape[0]):
        part[k].fill_(float(k))
    print("case", arena.data_ptr() % (2 << 20), flush=True)
    assert arena.data_ptr() % (2 << 20) == 0
    _, rep = B.dadam_place_by_timing(arena.data_ptr(), span, 0, [8 << 20] * 4, 288 * GIB)
    torch.cuda.synchronize()
    assert rep.note != B.DADAM_NOTE_NO_PROBE and rep.n_stretches >= 1
    in_chunk = [k for c in range(3) for k in range(c * step // buf, (c * step + chunk) // buf)]
    low, high = part.amin(1).cpu().numpy(), part.amax(1).cpu().numpy()
    assert np.array_equal(low, high)                                        # every buffer holds one value throughout
    sources = {k for c in range(3) for k in range(c * step // buf, c * step // buf + 8)}
    for k in range(part.shape[0]):
        if k not in in_chunk or k in sources:
            assert low[k] == k, k
        else:
            assert low[k] in sources, (k, low[k])


@pytest.mark.gpu
def test_the_probe_sees_a_picture_of_a_free_devices_memory():
    """On a device whose memory is free the pass tells chunks of one third from chunks of two: the first look gives
    stretches, whether or not the buffers then find room, and nothing is timed twice."""
    free, total = torch.cuda.mem_get_info(DEV)
    if free < (250 << 30):
        pytest.skip("needs a device with 250 GiB free")
    unit = 2 << 20
    arena = torch.empty((free - (12 << 30)) // unit * unit + unit, dtype=torch.uint8, device=DEV)
    shift = -arena.data_ptr() % unit
    span = (arena.numel() - unit) // unit * unit
    _, rep = B.dadam_place_by_timing(arena.data_ptr() + shift, span, 0, [48 << 20] * 64, total)
    found = [(s.third, s.lo >> 30, s.hi >> 30) for s in rep.stretches[:rep.n_stretches]]
    print("case", found, rep.note, rep.probe_launches, rep.rate_across, list(rep.rate_inside), flush=True)
    chunks = (span - B.PROBE_CHUNK_BYTES) // B.PROBE_STEP_BYTES + 1
    assert rep.note != B.DADAM_NOTE_NO_PICTURE and len({t for t, _, _ in found}) >= 2
    assert rep.probe_launches <= 8 * (2 * (chunks - 1) + 3)
