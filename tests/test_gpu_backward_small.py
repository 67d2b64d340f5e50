"""The backward of small bags, in items of 64 keys and of 64 queries (knap_attn_bwd_small.hip): parity with the fp64 oracle on bags that
launch it, and the launch of 128-row items with every query tile in parts on bags that still take it.

Bars: dq, dk, dv are sums of products of bf16-rounded factors (P and dS, relative 2^-9 each) stored in bf16: 2^-9 from either, so 2 times
2^-9 in the 2-norm of a head where errors are independent; 4 times as the bound."""
import numpy as np
import pytest

from knap_inputs import BagSpec
from oracle import attention as A

import queue_model as Q
from gpu_util import GpuRun, rel_fro, say

pytestmark = pytest.mark.gpu

BAR = 4 * 2.0 ** -9


def _compare(bag, causal, heads):
    run = GpuRun(bag, causal=causal)
    cu = [int(c) for c in run.cu]
    worst = 0.0
    for h in heads:
        got = {n: np.zeros((bag.total_tokens, bag.d)) for n in ("dq", "dk", "dv")}
        want = {n: np.zeros((bag.total_tokens, bag.d)) for n in got}
        for s in range(len(bag.seq_lens)):
            rows = slice(cu[s], cu[s + 1])
            if rows.start == rows.stop:
                continue
            q, k, v, dout = (run.host(n, rows, h) for n in ("q", "k", "v", "dout"))
            for n, ref in zip(("dq", "dk", "dv"), A.attn_bwd_dense(q, k, v, dout, bag.scale, causal)):
                want[n][rows], got[n][rows] = ref, run.host(n, rows, h)
                # no sequence is hidden behind the others' size; single rows have dq = dk = 0 up to rounding
                if rows.stop - rows.start > 8:
                    assert rel_fro(run.host(n, rows, h), ref) <= 2 * BAR, (n, h, s)
        for n in got:
            worst = max(worst, rel_fro(got[n], want[n]))
    say(f"[small] {bag.name} d={bag.d} causal={causal}: worst rel={worst:.3e}")
    assert worst <= BAR
    return run


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,H", [
    ([1, 31, 32, 33, 63, 64, 65, 0, 95, 97, 127, 128, 129, 191, 193, 255], 2),     # edges of the 32- and 64-row blocks and steps
    ([1537], 3), ([700, 333, 5], 4)])
def test_small_backward(lens, H, d, causal):
    import torch
    from paper_2508_06001_amd.runtime import bf16_device_to_bits
    assert Q.bwd_small(lens, H, d, causal)
    run = _compare(BagSpec("small", lens, H=H, d=d, seed=9500 + H + d), causal, range(H))
    # the same bits with a workspace that holds anything
    a, x = run.attn, run.dev
    a.workspace.fill_(0xff)
    for t in (a.dq, a.dk, a.dv):
        t.fill_(float("nan"))
    a.backward(x["q"], x["k"], x["v"], x["dout"])
    torch.cuda.synchronize()
    for got, want in zip((a.dq, a.dk, a.dv), (run.dq_bits, run.dk_bits, run.dv_bits)):
        assert np.array_equal(bf16_device_to_bits(got), want)


@pytest.mark.parametrize("d,lens,H,causal", [
    (128, [129] * 30, 4, True), (64, [129] * 30, 6, True),               # more items than workgroups: several draws; the last three take 128 rows
    (128, [1, 200] * 5, 12, False), (64, [1, 129, 129, 65], 44, False)])    # sequences that the average makes look shorter
def test_small_backward_draws(d, lens, H, causal):
    w = Q.walk_small(lens, H, d)
    assert Q.bwd_small(lens, H, d, causal) and w.draws and w.most > w.per
    _compare(BagSpec("small_draws", lens, H=H, d=d, seed=9600 + H + d), causal, [0, H // 2, H - 1])


@pytest.mark.parametrize("d,lens,H,causal", [(128, [160] * 22, 6, True), (64, [320] * 20, 6, True), (64, [700, 333, 5, 64], 24, True)])
def test_small_backward_draws_where_items_of_64_rows_pay(d, lens, H, causal):
    w = Q.walk_small(lens, H, d)
    s = Q.small_items(lens, H, d, causal)
    assert s.host > 0 and s.pays and w.draws and w.most > w.per
    _compare(BagSpec("small_draws", lens, H=H, d=d, seed=9650 + H + d), causal, [0, H // 2, H - 1])


@pytest.mark.parametrize("d,lens,H,causal,pays", [
    (128, [1, 200] * 20, 3, False, False), (64, [1, 200] * 40, 2, False, False), (128, [128] * 40, 3, False, True),
    (64, [128] * 96, 2, False, True),
    (128, [64] * 30 + [1, 0], 6, True, True), (128, [9176, 1], 3, True, False), (128, [96] * 70, 3, True, False), (128, [128] * 93, 3, True, True),
    (64, [20644, 0, 0], 2, True, False), (64, [160] * 105, 2, True, False), (64, [64] * 34 + [1], 12, True, True),
    (64, [0, 8] * 200 + [320] * 4, 1, True, True)])
def test_small_backward_of_bags_whose_lengths_decide(d, lens, H, causal, pays):
    """The kernel in front of the launch writes the decision behind the launch's counters, 256 bytes from the workspace's end: up to 64
    sequences, more, and more than a workgroup has threads; empty ones."""
    import torch
    from paper_2508_06001_amd.runtime import bf16_device_to_bits
    s = Q.small_items(lens, H, d, causal)
    assert s.host == 1 and s.pays == pays
    run = _compare(BagSpec("small_decided", lens, H=H, d=d, seed=9900 + H + d), causal, sorted({0, H // 2, H - 1}))
    a, x = run.attn, run.dev
    for fill in (0xff, 0):
        a.workspace.fill_(fill)
        for t in (a.dq, a.dk, a.dv):
            t.fill_(float("nan"))
        a.backward(x["q"], x["k"], x["v"], x["dout"])
        torch.cuda.synchronize()
        assert int(a.workspace[-256:].view(torch.int32)[8]) == pays
        for got, want in zip((a.dq, a.dk, a.dv), (run.dq_bits, run.dk_bits, run.dv_bits)):
            assert np.array_equal(bf16_device_to_bits(got), want)


@pytest.mark.parametrize("d,lens,H,causal", [(128, [700, 450], 14, False), (64, [700, 450], 21, False),
                                             # empty sequences, which the host's rule counts as tiles
                                             (128, [1537] + [0] * 40, 7, True), (64, [1537] + [0] * 40, 11, True)])
def test_128_row_items_with_every_query_tile_in_parts(d, lens, H, causal):
    w = Q.walk_joint(lens, H, d, causal)
    assert Q.bwd_joint(lens, H, d, causal) and not Q.bwd_small(lens, H, d, causal)
    assert w.parts == w.items * (4 if causal else 2) and not w.draws
    _compare(BagSpec("joint_parts", lens, H=H, d=d, seed=9700 + H + d), causal, [0, H // 2, H - 1])


def test_captured_small_backward_decides_at_every_replay():
    """Two bags of the same tokens and number of sequences, one of which takes items of 128 rows: a captured call follows the lengths that
    stand in cu_seqlens when it is replayed."""
    import torch
    from paper_2508_06001_amd.runtime import bf16_device_to_bits
    H, d, bags = 3, 128, ([96] * 70, [64] * 69 + [96 * 70 - 64 * 69])
    for lens, pays in zip(bags, (False, True)):
        s = Q.small_items(lens, H, d, True)
        assert s.host == 1 and s.pays == pays
    runs = [GpuRun(BagSpec("small_captured", lens, H=H, d=d, seed=9990), causal=True) for lens in bags]
    a, x = runs[0].attn, runs[0].dev
    # the first one's buffers are those of the captured call
    given = [{"cu": r.attn.cu.clone(), "out": r.attn.out.clone(), "lse": r.attn.lse.clone(), **{n: r.dev[n].clone() for n in x}} for r in runs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        a.backward(x["q"], x["k"], x["v"], x["dout"])
    for i in (0, 1, 1, 0, 1):
        run = runs[i]
        for n, t in (("cu", a.cu), ("out", a.out), ("lse", a.lse), *x.items()):
            t.copy_(given[i][n])
        for t in (a.dq, a.dk, a.dv):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(a.workspace[-256:].view(torch.int32)[8]) == i
        for got, want in zip((a.dq, a.dk, a.dv), (run.dq_bits, run.dk_bits, run.dv_bits)):
            assert np.array_equal(bf16_device_to_bits(got), want), i
