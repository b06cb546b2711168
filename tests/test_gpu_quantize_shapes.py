"""Bit-exact parity of the quantization pass at the edges of its launch shapes: the
one-launch calls (sequences up to 64 tokens, in one workgroup or one per part),
the per-KV-head-group kernels (small calls, group sizes up to the limit) and the
whole-chunk kernels past it, statistics in one block, two, and at the limit of the
short finish, empty sequences among the others, fresh and frozen statistics, slots
that start inside a page or run backwards, and the V copies of the other PV
precisions.  Every byte equals the oracle's."""
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


def _compare(got, ref, what):
    for key, g in got.items():
        r = np.asarray(ref[key])
        g = np.asarray(g)
        if g.dtype == np.float32:
            g, r = g.view(np.uint32), r.astype(np.float32).view(np.uint32)
        bad = np.argwhere(g.reshape(r.shape) != r)
        assert not len(bad), (what, key, len(bad), bad[:3].tolist())


def _both(orc, mp, lens, h_q, h_kv, flags, slots, n_pages, stats=None, seed=5):
    """The call through the library and the oracle on the same bits, over 0xFF-filled planes."""
    B, T = len(lens), sum(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    g = torch.Generator().manual_seed(seed)
    rnd = lambda h: (torch.randn(T, h, 128, generator=g) * 2 + torch.randn(1, h, 128, generator=g)).bfloat16().cuda()
    q, k, v = rnd(h_q), rnd(h_kv), rnd(h_kv)
    pv = flags & (mp.PV_BF16 | mp.PV_NVFP4)
    cache = mp.PagedCache(n_pages, h_q, h_kv, pv=pv)
    for t in (cache.k_codes, cache.k_scales, cache.v_codes):
        t.fill_(0xFF)
    cache.ds.view(torch.int16).fill_(-1)
    st = mp.SeqStats(B, h_q, h_kv)
    okw = {}
    if stats is not None:
        st.q_mean.copy_(stats[0])
        st.k_mean.copy_(stats[1])
        st.k_tscale.copy_(stats[2])
        okw = dict(q_mean=H.bits(stats[0]), k_mean=H.bits(stats[1]), k_tscale=stats[2].cpu().numpy())
    qq = mp.QuantQ(T, B, h_q)
    ocache = dict(k_codes=np.full((n_pages, h_kv, 64, 64), 0xFF, np.uint8),
                  k_scales=np.full((n_pages, h_kv, 64, 8), 0xFF, np.uint8),
                  v_codes=np.full((n_pages, h_kv, 128, 64), 0xFF, np.uint8),
                  ds=np.full((n_pages, h_q, 64), 0xFFFF, np.uint16))
    oflags = 0
    for a, b in ((mp.SMOOTH, orc.SMOOTH), (mp.COMPUTE_STATS, orc.COMPUTE_STATS), (mp.TSCALE_UNIT, orc.TSCALE_UNIT),
                 (mp.MXFP4, orc.MXFP4), (mp.PV_BF16, orc.PV_BF16), (mp.PV_NVFP4, orc.PV_NVFP4)):
        oflags |= b if flags & a else 0
    mp.quantize_qk(q, k, v, torch.from_numpy(cu).cuda(), torch.from_numpy(slots).cuda(), cache, st, qq, flags, max(lens))
    torch.cuda.synchronize()
    ref = orc.quantize_qk(H.bits(q), H.bits(k), H.bits(v), cu, slots, n_pages, oflags, cache=ocache, **okw)
    ref = dict(ref, **ref["cache"])
    got = dict(q_codes=qq.codes.cpu(), q_scales=qq.scales.cpu(), q_tscale=qq.tscale.cpu().numpy(),
               q_mean=H.bits(st.q_mean), k_mean=H.bits(st.k_mean), k_tscale=st.k_tscale.cpu().numpy(),
               k_codes=cache.k_codes.cpu(), k_scales=cache.k_scales.cpu(), v_codes=cache.v_codes.cpu())
    if flags & mp.SMOOTH:
        got["ds"] = H.bits(cache.ds)
    if pv:
        got["v_aux"] = H.bits(cache.v_aux) if pv == mp.PV_BF16 else cache.v_aux.cpu()
    _compare(got, ref, (lens, h_q, h_kv, flags))
    return st


def _pages(lens, start=0, backwards=False):
    """Slots of packed sequences, each in pages of its own from slot `start` of its first page."""
    out, page = [], 0
    for n in lens:
        s = page * 64 + start + np.arange(n, dtype=np.int64)
        out.append(s[::-1].copy() if backwards else s)
        page += (start + n + 63) // 64
    return np.concatenate(out), page + 1


# heads: groups of 1, 4, 5, the largest the group kernels take (16) and one past it (17)
@pytest.mark.parametrize("h_q,h_kv", [(1, 1), (8, 2), (10, 2), (16, 1), (17, 1)])
@pytest.mark.parametrize("lens", [[1], [0, 8, 1], [9, 64, 0, 63], [65, 1], [127, 128, 129, 64], [300]])
def test_shapes_fresh_and_frozen(orc, mp, lens, h_q, h_kv):
    slots, n_pages = _pages(lens)
    for mode in (mp.SMOOTH, 0, mp.SMOOTH | mp.MXFP4, mp.SMOOTH | mp.TSCALE_UNIT):
        st = _both(orc, mp, lens, h_q, h_kv, mode | mp.COMPUTE_STATS, slots, n_pages)
        s2, p2 = _pages(lens, start=37)
        _both(orc, mp, lens, h_q, h_kv, mode, s2, p2, stats=(st.q_mean, st.k_mean, st.k_tscale), seed=6)


@pytest.mark.parametrize("lens", [[64, 5], [200, 64]])
def test_slots_backwards(orc, mp, lens):
    slots, n_pages = _pages(lens, backwards=True)
    _both(orc, mp, lens, 8, 2, mp.SMOOTH | mp.COMPUTE_STATS, slots, n_pages)


@pytest.mark.parametrize("lens", [[40, 64], [64, 130, 7]])
@pytest.mark.parametrize("pv", ["PV_BF16", "PV_NVFP4"])
def test_v_copies(orc, mp, lens, pv):
    slots, n_pages = _pages(lens)
    _both(orc, mp, lens, 8, 2, mp.SMOOTH | mp.COMPUTE_STATS | getattr(mp, pv), slots, n_pages)


# statistics blocks at the short finish's limit (64 blocks) and past it; many sequences (one
# workgroup per group instead of one per part); a call past the group kernels' chunk limit
@pytest.mark.parametrize("lens,h_q,h_kv", [([8192], 2, 1), ([8193, 130], 2, 1), ([16] * 300, 4, 2), ([70] * 80, 8, 8),
                                           ([33300], 1, 1)])
def test_limits(orc, mp, lens, h_q, h_kv):
    slots, n_pages = _pages(lens)
    _both(orc, mp, lens, h_q, h_kv, mp.SMOOTH | mp.COMPUTE_STATS, slots, n_pages)


# one long sequence among many short ones: grids of the blocks that the call has, with
# empty sequences and more than one round of 64 sequences in the search for a block
@pytest.mark.parametrize("lens", [[1] * 70 + [0] * 3 + [700, 130] + [1] * 20, [1, 0, 900, 1, 1, 1], [1500] + [0] * 40])
def test_skewed_batches(orc, mp, lens):
    slots, n_pages = _pages(lens)
    for mode in (mp.SMOOTH, 0, mp.SMOOTH | mp.MXFP4):
        st = _both(orc, mp, lens, 8, 2, mode | mp.COMPUTE_STATS, slots, n_pages)
        _both(orc, mp, lens, 8, 2, mode, slots, n_pages, stats=(st.q_mean, st.k_mean, st.k_tscale), seed=6)


def test_short_sequences_beside_a_long_one_cost_little(mp):
    """One token each in 31 more sequences: grids of (blocks of the longest) x (sequences)
    took 1.26 times as long as the long sequence alone."""
    took = []
    for lens in ([30000], [30000] + [1] * 31):
        T, B = sum(lens), len(lens)
        q, k, v = (torch.randn((T, h, 128), device="cuda", dtype=torch.bfloat16) for h in (32, 8, 8))
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
        slots, n_pages = _pages(lens)
        args = (q, k, v, cu, torch.from_numpy(slots).cuda(), mp.PagedCache(n_pages, 32, 8), mp.SeqStats(B, 32, 8), mp.QuantQ(T, B, 32),
                mp.SMOOTH | mp.COMPUTE_STATS, max(lens))
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(8):   # the first is a warm-up
            start.record()
            for _ in range(10):
                mp.quantize_qk(*args)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        took.append(float(np.median(times[1:])))
    assert took[1] <= 1.15 * took[0], took
