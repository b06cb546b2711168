"""GPU parity of prefill calls that run in 128-row workgroups: row counts around the
128- and 256-row tiles, ragged batches, a chunk behind a context, both formats, with
and without the compensation; calls on both sides of the workgroup limit.  Outputs against the oracle at the bar of the other parity tests; the
mixed step, which keeps 256-row workgroups, gives the same bytes."""
import numpy as np
import pytest
import torch

from tests import helpers as H
from tests.test_gpu_prefill_few import _check_chunks, _dev, mp  # noqa: F401

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
