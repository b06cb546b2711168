"""GPU parity of prefill calls with few query rows (32-row workgroups whose KV tiles
are spread over the waves) and of the dispatch order of batches whose sequences
start at different positions: row counts around 32, contexts around the eight-tile
rounds, ragged batches in which some sequences split and others do not, shards
with few heads, both formats and with and without the compensation.  Outputs against the
oracle at the bar of the other parity tests; the mixed step gives the same bytes."""
import numpy as np
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp():
    import paper_2609_33135_amd as mp
    assert torch.cuda.is_available()
    mp.lib()
    return mp


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _chunks(run, new):
    """The last new[b] rows of every sequence as one chunked call's arguments and output."""
    mp = run.mp
    idx = np.concatenate([np.arange(run.cu[b + 1] - n, run.cu[b + 1]) for b, n in enumerate(new)])
    qq = mp.QuantQ(len(idx), run.B, run.h_q)
    qq.codes.copy_(run.qq.codes[torch.from_numpy(idx).cuda()])
    qq.scales.copy_(run.qq.scales[torch.from_numpy(idx).cuda()])
    qq.tscale.copy_(run.qq.tscale)
    out = torch.full((len(idx), run.h_q, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    args = dict(qq=qq, cache=run.cache, stats=run.stats, cu_seqlens_q=_dev(np.concatenate([[0], np.cumsum(new)])),
                q_start=_dev([s - n for s, n in zip(run.seqlens, new)]), kv_len=_dev(run.seqlens), page_table=_dev(run.pt),
                out=out, max_seqlen_q=max(new))
    return args, out


def _check_chunks(run, new, flags):
    args, out = _chunks(run, new)
    run.mp.prefill(**args, flags=flags)
    torch.cuda.synchronize()
    got = H.bits(out)
    items, at, pos = [], [], 0
    for b, n in enumerate(new):
        for i in sorted({0, 1, n // 2, n - 1} & set(range(n))):
            for h in range(run.h_q):
                items.append((b, run.seqlens[b] - n + i, h))
                at.append((pos + i, h))
        pos += n
    ref, _ = run.prefill_oracle(np.array(items, np.int32))
    got = np.stack([got[r, h] for r, h in at])
    assert not np.isnan(H.bf16_f64(got)).any()
    max_abs, mean_rel, n_bad = H.compare_bf16(got, ref)
    assert n_bad == 0 and mean_rel <= H.TOL_MEAN_REL, (max_abs, mean_rel, n_bad)
    return args, out


@pytest.mark.parametrize("mxfp4,smooth", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("total,new", [(1024, 1), (1025, 31), (2048, 32), (2050, 33), (1151, 64), (3000, 100), (700, 700)])
def test_few_rows(orc, mp, total, new, mxfp4, smooth):
    run = H.Run(orc, mp, 81, [total], 4, 2, mxfp4=mxfp4, smooth=smooth, stale_fill=True)
    _check_chunks(run, [new], (mp.SMOOTH if smooth else 0) | (mp.MXFP4 if mxfp4 else 0))


@pytest.mark.parametrize("totals,new", [([2500, 90, 1300], [300, 90, 40]), ([40, 4000], [40, 33]),
                                        ([129, 1, 2000, 600, 257], [1, 1, 17, 600, 256])])
def test_few_rows_ragged(orc, mp, totals, new):
    """Sequences that split beside sequences that do not."""
    run = H.Run(orc, mp, 82, totals, 8, 8)
    _check_chunks(run, new, mp.SMOOTH)


@pytest.mark.parametrize("totals,new", [([3000, 1100, 2300, 400], [900, 1100, 300, 257]),
                                        ([600, 5000, 512], [600, 513, 1]), ([300] * 70, [300 - 4 * i for i in range(70)])])
def test_order_of_unequal_starts(orc, mp, totals, new):
    """Enough heads and rows for the 256-row items; sequences that start apart (and a batch past 64)."""
    run = H.Run(orc, mp, 83, totals, 48 if len(totals) < 10 else 8, 16 if len(totals) < 10 else 8)
    _check_chunks(run, new, mp.SMOOTH)


@pytest.mark.parametrize("total,new", [(2100, 40), (3000, 700)])
def test_mixed_step_same_bytes(orc, mp, total, new):
    run = H.Run(orc, mp, 84, [total], 4, 2)
    args, out = _check_chunks(run, [new], mp.SMOOTH)
    ref, dec_ref = H.bits(out), run.decode_last_gpu(256)
    out.fill_(float("nan"))
    qq = mp.QuantQ(1, 1, 4)
    qq.codes.copy_(run.qq.codes[-1:])
    qq.scales.copy_(run.qq.scales[-1:])
    qq.tscale.copy_(run.qq.tscale)
    dec = torch.full((1, 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    most = (total + 255) // 256
    ws = torch.zeros(mp.mixed_workspace_size(1, 4, 2, most) // 4, dtype=torch.float32, device="cuda")
    mp.mixed_step(args, dict(qq=qq, cache=run.cache, stats=run.stats, kv_len=_dev([total]), page_table=_dev(run.pt),
                             out=dec, partition_tokens=256, max_partitions=most), ws, mp.SMOOTH)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits(out), ref) and np.array_equal(H.bits(dec), dec_ref)


# maximum row counts above the call's: blocks of the grid past the rows, in one sequence
# and in a batch
@pytest.mark.parametrize("totals,new,most", [([900], [300], 1000), ([300], [1], 257), ([2000, 70], [33, 70], 640)])
def test_fewer_rows_than_the_maximum(orc, mp, totals, new, most):
    run = H.Run(orc, mp, 85, totals, 8, 2)
    args, out = _check_chunks(run, new, mp.SMOOTH)
    ref = H.bits(out)
    out.fill_(float("nan"))
    mp.prefill(**dict(args, max_seqlen_q=most), flags=mp.SMOOTH)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits(out), ref)
