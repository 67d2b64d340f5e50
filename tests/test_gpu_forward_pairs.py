"""The forward without the mask where it takes two query tiles at a time (256 rows): parity with the fp64 oracle on bags that reach it.

The bag: sequences of 17 and 14 query tiles, odd and even, so that some pairs fall apart at the end of a head (their tiles are then
taken singly), with 33 and 36 rows in the last tile, and short ones that are never paired."""
import numpy as np
import pytest

from knap_inputs import BagSpec, make_qkv_dout
from oracle import attention as A

import queue_model as Q
from gpu_util import GpuRun, say

pytestmark = pytest.mark.gpu

LENS = [2081, 130, 1700, 64, 1]
# more than two and three rounds of 128-row items
HEADS = {128: 48, 64: 104}


def _compare(run, d, strict, lse_tol):
    """First, middle and last heads.  strict: 1e-2, on N(0, 1) inputs.  Else the bound of rows that few keys dominate: every
    probability carries a relative error of up to 2^-9, sum_i w_i e_i (v_i - out), and the stored result another 2^-9 of itself:
    2^-9 (2 max|v| + |ref|).  lse relative to its own size where scores are large (fp32 scores of hundreds)."""
    worst = worst_lse = 0.0
    cu = [int(c) for c in run.cu]
    H = run.bag.H
    for s in range(len(LENS)):
        rows = slice(cu[s], cu[s + 1])
        for h in (0, 1, 2, H // 8, H // 2, H - 1):
            q, k, v = (run.host(n, rows, h) for n in ("q", "k", "v"))
            O, LSE = A.attn_fwd_dense(q, k, v, run.bag.scale)
            bar = 1e-2 if strict else 2.0 ** -9 * (2 * np.abs(v).max() + np.abs(O))
            worst = max(worst, float((np.abs(run.host("out", rows, h) - O) / bar).max()))
            worst_lse = max(worst_lse, float((np.abs(run.lse[h, rows] - LSE) / np.maximum(1.0, np.abs(LSE) / 64)).max()))
    say(f"[pairs] d={d}: fwd error / bar={worst:.3f} lse={worst_lse:.3e}")
    assert worst <= 1.0 and worst_lse <= lse_tol


def _bag(d, seed):
    w = Q.walk_pairs(LENS, HEADS[d], d)
    assert w.items > 100 and w.draws and w.most < Q.walk("fwd", LENS, HEADS[d], d, False).most
    return BagSpec("pairs", LENS, H=HEADS[d], d=d, seed=seed + d)


@pytest.mark.parametrize("d", [64, 128])
def test_pairs_of_query_tiles(d):
    _compare(GpuRun(_bag(d, 9100), backward=False), d, d == 128, 1e-3 if d == 128 else 3e-3)


@pytest.mark.parametrize("power", [3, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_pairs_with_keys_far_above_the_first_64(d, power):
    """Behind the first 64 keys of the long sequences some are 2^power times as large, in every second head: probabilities far above
    one, which take the second term (3), and ones beyond the range, which send the item through the narrow form (8)."""
    bag = _bag(d, 9200)
    tensors = make_qkv_dout(bag)
    for first in (900, 2081 + 130 + 1650):
        big = tensors["k"][first:first + 3, ::2]
        big[(big & 0x7f80) != 0] += np.uint16(power << 7)
    _compare(GpuRun(bag, tensors=tensors, backward=False), d, False, 3e-3)


@pytest.mark.parametrize("d,H", [(128, 65536), (64, 131072)])
def test_pairs_at_rows_of_16_mb(d, H):
    """256 rows of q or out are 2^32 bytes, the first size that a 32-bit byte count does not hold.  One tensor for q, k and v (24 GB);
    a scale of 1 / d, so that a row's weights are spread over its keys and not on itself.  Bar: as in _compare, and 1e-3 for lse."""
    import torch
    import paper_2508_06001_amd as K
    L, scale = 1450, 1.0 / d
    assert Q.walk_pairs([L], H, d).items > 0
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of GPU memory")
    say(f"[pairs] 16 MB rows: d={d} H={H}")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9300 + d)
    x = torch.empty((L, H, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    attn = K.VarlenAttention([0, L], H, d, scale)
    attn.out.fill_(float("nan"))
    attn.forward(x, x, x)
    torch.cuda.synchronize()
    for h in (0, 1, H // 2 + 1, H - 1):
        v = x[:, h].double().cpu().numpy()
        O, LSE = A.attn_fwd_dense(v, v, v, scale)
        err = np.abs(attn.out[:, h].double().cpu().numpy() - O) / (2.0 ** -9 * (2 * np.abs(v).max() + np.abs(O)))
        assert err.max() <= 1.0 and np.abs(attn.lse[h].cpu().numpy() - LSE).max() <= 1e-3, (h, err.max())
    assert all(bool(torch.isfinite(rows).all()) for rows in attn.out.split(64))
    del attn, x
    torch.cuda.empty_cache()
