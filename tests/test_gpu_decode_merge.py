"""GPU parity of the decode at the edges of its partition counts: one to eight
partitions (merged in the partitions' own workgroup of 1, 2, 4 or 8 waves), up to
the 8, 16 and 32 states a one-wave merge holds, and chunk edges of the many-wave
merge, with a second sequence of fewer partitions beside the first.  Outputs
against the oracle; the one-launch mixed step's merge gives the same bytes."""
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


def _check(got, ref):
    max_abs, mean_rel, n_bad = H.compare_bf16(got, ref)
    assert not np.isnan(H.bf16_f64(got)).any()
    assert n_bad == 0 and mean_rel <= H.TOL_MEAN_REL, (max_abs, mean_rel, n_bad)


@pytest.mark.parametrize("nparts", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 257])
def test_partition_counts(orc, mp, nparts):
    lens = [nparts * 128 - 5, max(1, nparts * 128 // 3)]
    run = H.Run(orc, mp, 71, lens, 4, 2, mxfp4=nparts % 2 == 0)
    _check(run.decode_last_gpu(128), run.decode_last_oracle(128))


@pytest.mark.parametrize("mxfp4,smooth", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("h_q,h_kv", [(1, 1), (8, 1), (10, 2)])
def test_eight_wave_groups(orc, mp, h_q, h_kv, mxfp4, smooth):
    """More workgroups than compute units: 5 to 8 partitions in one workgroup; ragged, down to one."""
    lens = [1024 - 41 * i for i in range(20)]
    run = H.Run(orc, mp, 72, lens, h_q, h_kv, mxfp4=mxfp4, smooth=smooth)
    _check(run.decode_last_gpu(128), run.decode_last_oracle(128))


@pytest.mark.parametrize("nparts", [3, 33, 70])
def test_mixed_merge_same_bytes(orc, mp, nparts):
    n = nparts * 128 - 9
    run = H.Run(orc, mp, 73, [n], 4, 2)
    ref = run.decode_last_gpu(128)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qq = mp.QuantQ(1, 1, 4)
    qq.codes.copy_(run.qq.codes[-1:])
    qq.scales.copy_(run.qq.scales[-1:])
    qq.tscale.copy_(run.qq.tscale)
    out = torch.full((n, 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    dec = torch.full((1, 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.zeros(mp.mixed_workspace_size(1, 4, 2, nparts) // 4, dtype=torch.float32, device="cuda")
    pre = dict(qq=run.qq, cache=run.cache, stats=run.stats, cu_seqlens_q=run.cu_d, q_start=dev([0]), kv_len=dev([n]),
               page_table=dev(run.pt), out=out, max_seqlen_q=n)
    mp.mixed_step(pre, dict(qq=qq, cache=run.cache, stats=run.stats, kv_len=dev([n]), page_table=dev(run.pt), out=dec,
                            partition_tokens=128, max_partitions=nparts), ws, mp.SMOOTH)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits(dec), ref)


@pytest.mark.parametrize("h_q,h_kv,batch,nparts", [(32, 8, 2, 33), (33, 11, 2, 33), (40, 8, 2, 40), (2, 1, 1, 515)])
def test_split_merge_limit(orc, mp, h_q, h_kv, batch, nparts):
    """Both sides of the 64 heads that two workgroups per head merge, and a second round of sixteen waves."""
    lens = [nparts * 128 - 5, 128 * 32 + 1][:batch]
    run = H.Run(orc, mp, 74, lens, h_q, h_kv)
    _check(run.decode_last_gpu(128), run.decode_last_oracle(128))
