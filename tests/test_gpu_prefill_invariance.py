"""A row's prefill output does not depend on how the call is cut: the same bytes
alone, beside other sequences, as a chunk and under a page table wider than the
sequence.  The calls below run the same rows in every kind of work item (32 rows
with the KV tiles over the waves, 128 and 256 rows), so equal bytes between them
hold for the items as well.  No tolerance: FP32 sums in the same order."""
import numpy as np
import pytest
import torch

from tests import helpers as H
from tests.test_gpu_prefill_few import _chunks, _dev, mp  # noqa: F401

pytestmark = pytest.mark.gpu


def _bits(run, new, flags, pages=0):
    """Output bits per sequence of the last new[b] rows, page table at least `pages` wide."""
    args, out = _chunks(run, new)
    if pages:
        wide = torch.zeros((run.B, pages), dtype=torch.int32, device="cuda")
        wide[:, :run.pt.shape[1]] = args["page_table"]
        args["page_table"] = wide
    run.mp.prefill(**args, flags=flags)
    torch.cuda.synchronize()
    got, cu = H.bits(out), np.concatenate([[0], np.cumsum(new)])
    return [got[cu[b]:cu[b + 1]] for b in range(run.B)]


# the compared sequence (keys, rows) and what runs beside it: rows that take the split
# items alone and whole items next to a prompt that fills the chip
@pytest.mark.parametrize("mxfp4,smooth", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("total,new", [(4000, 256), (2049, 33), (3001, 1), (1500, 700)])
def test_alone_and_beside_others(orc, mp, total, new, mxfp4, smooth):  # noqa: F811
    flags = (mp.SMOOTH if smooth else 0) | (mp.MXFP4 if mxfp4 else 0)
    run = H.Run(orc, mp, 95, [total, 6000], 8, 2, mxfp4=mxfp4, smooth=smooth, stale_fill=True)
    small = _bits(run, [new, 1], flags)[0]                   # few rows in the call
    beside = _bits(run, [new, 6000], flags)[0]               # a whole prompt beside it
    assert np.array_equal(small, beside)


@pytest.mark.parametrize("mxfp4", [False, True])
@pytest.mark.parametrize("h_q,h_kv,total", [(8, 2, 1000), (4, 2, 2305), (32, 8, 777), (16, 8, 1300)])
def test_chunks_and_wide_tables(orc, mp, h_q, h_kv, total, mxfp4):  # noqa: F811
    flags = mp.SMOOTH | (mp.MXFP4 if mxfp4 else 0)
    run = H.Run(orc, mp, 96, [total], h_q, h_kv, mxfp4=mxfp4, stale_fill=True)
    whole = _bits(run, [total], flags)[0]
    for pages in (64, 2048):
        for seed in (0, mp.SEED_MFMA):   # a wide table's whole items form the seed as the flag says
            assert np.array_equal(_bits(run, [total], flags | seed, pages)[0], whole), (pages, seed)
    for rows in (1, 40, 300):
        assert np.array_equal(_bits(run, [rows], flags)[0], whole[-rows:]), rows
        assert np.array_equal(_bits(run, [rows], flags, 2048)[0], whole[-rows:]), rows
