"""GPU parity of prefill calls whose items have 128 rows, or may have: row counts around
the 128- and 256-row tiles, ragged batches, chunks behind short and long contexts, both
formats, with and without the compensation; calls on both sides of the workgroup limit;
wide page tables.  Outputs against the oracle at the bar of the other parity tests; the
mixed step, which keeps 256-row items, gives the same bytes.  Two tests hold the times
of calls against each other."""
import numpy as np
import pytest
import torch

from tests import helpers as H
from tests.test_gpu_prefill_few import _check_chunks, _chunks, _dev, mp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mxfp4,smooth", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("total,new", [(129, 129), (255, 255), (256, 256), (257, 257), (640, 640), (1700, 900)])
def test_half_items(orc, mp, total, new, mxfp4, smooth):  # noqa: F811
    run = H.Run(orc, mp, 91, [total], 32, 8, mxfp4=mxfp4, smooth=smooth, stale_fill=True)
    flags = (mp.SMOOTH if smooth else 0) | (mp.MXFP4 if mxfp4 else 0)
    args, out = _check_chunks(run, [new], flags)
    ref = H.bits(out)
    out.fill_(float("nan"))
    qq = mp.QuantQ(1, 1, 32)
    qq.codes.copy_(run.qq.codes[-1:])
    qq.scales.copy_(run.qq.scales[-1:])
    qq.tscale.copy_(run.qq.tscale)
    dec = torch.full((1, 32, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    most = (total + 255) // 256
    ws = torch.zeros(mp.mixed_workspace_size(1, 32, 8, most) // 4, dtype=torch.float32, device="cuda")
    mp.mixed_step(args, dict(qq=qq, cache=run.cache, stats=run.stats, kv_len=_dev([total]), page_table=_dev(run.pt),
                             out=dec, partition_tokens=256, max_partitions=most), ws, flags)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits(out), ref)


@pytest.mark.parametrize("totals,new", [([130, 1, 257, 600], [130, 1, 257, 600]), ([900, 2000, 300], [300, 129, 5]),
                                        ([1664], [1664]), ([1665], [1665])])
def test_half_items_ragged_and_limit(orc, mp, totals, new):  # noqa: F811
    """Ragged batches, and the last call of the rule (13 x 32 workgroups) beside the next."""
    run = H.Run(orc, mp, 93, totals, 32 if len(totals) == 1 else 16, 8)
    _check_chunks(run, new, mp.SMOOTH)


# Workgroups of 128 rows whose items the device cuts by the contexts: 128 rows of a prompt,
# 256 behind a long prefix (32:8; 8:2 heads the same under a wide table, in 32-row blocks)
@pytest.mark.parametrize("mxfp4", [False, True])
@pytest.mark.parametrize("total,new,h_q,h_kv", [(1600, 1600, 32, 8), (5000, 1500, 32, 8), (10000, 6000, 8, 2),
                                                (4500, 1281, 32, 8)])
def test_items_by_context(orc, mp, total, new, h_q, h_kv, mxfp4):  # noqa: F811
    run = H.Run(orc, mp, 94, [total], h_q, h_kv, mxfp4=mxfp4, stale_fill=True)
    flags = mp.SMOOTH | (mp.MXFP4 if mxfp4 else 0)
    args, out = _check_chunks(run, [new], flags)
    ref = H.bits(out)
    table = args["page_table"]
    for pages, seed in ((table.shape[1], mp.SEED_MFMA), (2048, 0), (2048, mp.SEED_MFMA)):
        wide = torch.zeros((1, pages), dtype=torch.int32, device="cuda")
        wide[:, :table.shape[1]] = table
        out.fill_(float("nan"))
        mp.prefill(**dict(args, page_table=wide), flags=flags | seed)
        torch.cuda.synchronize()
        assert np.array_equal(H.bits(out), ref), (pages, seed)


def _time(mp, args, flags):  # noqa: F811
    """Median time of a call in microseconds, of nine batches of 20."""
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    times = []
    for _ in range(10):   # the first is a warm-up
        start.record()
        for _ in range(20):
            mp.prefill(**args, flags=flags)
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end) * 50)
    return float(np.median(times[1:]))


@pytest.mark.parametrize("h_q,h_kv,total,few,many", [(32, 8, 10100, 1600, 2048), (8, 2, 12400, 6000, 8192)])
def test_fewer_rows_take_no_longer(orc, mp, h_q, h_kv, total, few, many):  # noqa: F811
    """The items of fewer rows behind the same context: 128-row ones, two rounds of them
    where 256-row ones are one, took 1.6 and 1.9 times as long as the larger call."""
    run = H.Run(orc, mp, 97, [total], h_q, h_kv)
    took = [_time(mp, _chunks(run, [n])[0], mp.SMOOTH) for n in (few, many)]
    assert took[0] <= 1.15 * took[1], took


@pytest.mark.parametrize("rows", [250, 777])
def test_wide_page_table_costs_nothing(orc, mp, rows):  # noqa: F811
    """A short prompt under a page table of the model's maximum length: the same items
    (256-row ones took 1.2 times as long), twelve percent for the larger grid."""
    run = H.Run(orc, mp, 98, [rows], 32, 8)
    args = _chunks(run, [rows])[0]
    wide = torch.zeros((1, 2048), dtype=torch.int32, device="cuda")
    wide[:, :args["page_table"].shape[1]] = args["page_table"]
    tight = _time(mp, args, mp.SMOOTH)
    assert _time(mp, dict(args, page_table=wide), mp.SMOOTH) <= 1.12 * tight, tight
