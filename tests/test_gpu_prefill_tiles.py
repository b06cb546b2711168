"""GPU parity of the prefill at the edges of its tiles: query counts around the
32-row wave and 256-row workgroup boundaries, first tiles that end inside a page,
inside a 128-key tile and on its edge, and chunks behind prefixes of odd length,
for both Q/K formats and with and without the compensation.  Outputs against the
oracle at the bar of the other parity tests (BF16 rounding plus flips of single
E4M3 probabilities)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from tests import helpers as H

pytestmark = pytest.mark.gpu

LENS = [[1, 31, 32, 33], [127, 128, 129], [255, 256, 257], [64, 65, 191, 193, 511, 513]]


@pytest.fixture(scope="module")
def mp():
    import paper_2609_33135_amd as mp
    assert torch.cuda.is_available()
    mp.lib()
    return mp


def check(run, out, items, ref):
    got = np.stack([out[run.cu[b] + i, h] for b, i, h in items])
    max_abs, mean_rel, n_bad = H.compare_bf16(got, ref)
    assert n_bad == 0 and mean_rel <= H.TOL_MEAN_REL, (max_abs, mean_rel, n_bad)


@pytest.mark.parametrize("mxfp4", [False, True])
@pytest.mark.parametrize("smooth", [True, False])
@pytest.mark.parametrize("lens", LENS)
def test_tile_edges(orc, mp, lens, smooth, mxfp4):
    run = H.Run(orc, mp, 61, lens, 4, 2, smooth=smooth, mxfp4=mxfp4, stale_fill=True)
    items = np.array([(b, i, h) for b, n in enumerate(lens) for i in sorted({0, n // 2, max(n - 2, 0), n - 1})
                      for h in range(4)], np.int32)
    ref, _ = run.prefill_oracle(items)
    check(run, run.prefill_gpu(), items, ref)


@pytest.mark.parametrize("start", [1, 63, 127, 128, 129, 255, 700])
def test_chunk_edges(orc, mp, start):
    """The last rows of a sequence as a chunk at `start`: bit-identical to the same rows of
    the whole prefill (each row sees the same tiles in the same order)."""
    n = 900
    run = H.Run(orc, mp, 62, [n], 4, 2)
    whole = run.prefill_gpu()
    rows = n - start
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    qq = mp.QuantQ(rows, 1, 4)
    qq.codes.copy_(run.qq.codes[start:])
    qq.scales.copy_(run.qq.scales[start:])
    qq.tscale.copy_(run.qq.tscale)
    out = torch.full((rows, 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    mp.prefill(qq, run.cache, run.stats, dev([0, rows]), dev([start]), dev([n]), dev(run.pt), out, rows, mp.SMOOTH)
    torch.cuda.synchronize()
    assert np.array_equal(H.bits(out), whole[start:])
