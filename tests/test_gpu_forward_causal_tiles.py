"""The causal forward on whole query tiles of 128 rows, at the edges of its loop: one key tile, two (of which half of the waves see one), odd
and even numbers of them, ragged ends, pairs of tiles and middle ones; parity with the fp64 oracle."""
import numpy as np
import pytest

from knap_inputs import BagSpec
from oracle import attention as A

import queue_model as Q
from gpu_util import GpuRun, say

pytestmark = pytest.mark.gpu

LENS = [1, 32, 63, 64, 65, 127, 128, 129, 191, 193, 256, 257, 320, 385, 641]


@pytest.mark.parametrize("d,H", [(128, 30), (64, 45)])
def test_causal_forward_on_whole_tiles(d, H):
    """Bars: rows that see few keys return single entries of v, rounded once to bf16, 2^-8 of the reference or 1e-2; a sum of
    probabilities of relative error 2^-9 each is off by at most as much, so lse by at most 2^-9, and the fp32 rest."""
    w = Q.walk("fwd", LENS, H, d, True)
    assert w.parts == 0 and w.draws
    run = GpuRun(BagSpec("causal_tiles", LENS, H=H, d=d, seed=9800 + d), backward=False, causal=True)
    cu = [int(c) for c in run.cu]
    worst = worst_lse = 0.0
    for s in range(len(LENS)):
        rows = slice(cu[s], cu[s + 1])
        for h in (0, H // 2, H - 1):
            O, LSE = A.attn_fwd_dense(*(run.host(n, rows, h) for n in ("q", "k", "v")), run.bag.scale, True)
            worst = max(worst, float((np.abs(run.host("out", rows, h) - O) / np.maximum(1e-2, 2.0 ** -8 * np.abs(O))).max()))
            worst_lse = max(worst_lse, float(np.abs(run.lse[h, rows] - LSE).max()))
    say(f"[causal tiles] d={d}: error / bar={worst:.3f} lse={worst_lse:.3e}")
    assert worst <= 1.0 and worst_lse <= 2.0 ** -9 + 1e-4
