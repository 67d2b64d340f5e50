"""The forward without the mask where it takes two query tiles at a time (256 rows): parity with the fp64 oracle on bags that reach it.

The bag: sequences of 17 and 14 query tiles, odd and even, so that some pairs fall apart at the end of a head (their tiles are then
taken singly), with 33 and 36 rows in the last tile, and short ones that are never paired."""
import math

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
# lse on N(0, 1) inputs: a sum of probabilities of relative error 2^-9 each is off by at most as much, and the fp32 rest
LSE_MOST = 2.0 ** -9 + 1e-4


def _compare(run, d, strict, lse_tol, sequences=None, heads=None):
    """First, middle and last heads.  strict: 1e-2, on N(0, 1) inputs.  Else the bound of rows that few keys dominate: every
    probability carries a relative error of up to 2^-9, sum_i w_i e_i (v_i - out), and the stored result another 2^-9 of itself:
    2^-9 (2 max|v| + |ref|).  lse relative to its own size where scores are large (fp32 scores of hundreds)."""
    worst = worst_lse = 0.0
    cu = [int(c) for c in run.cu]
    H = run.bag.H
    for s in range(len(cu) - 1) if sequences is None else sequences:
        rows = slice(cu[s], cu[s + 1])
        for h in (0, 1, 2, H // 8, H // 2, H - 1) if heads is None else heads:
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
    _compare(GpuRun(_bag(d, 9100), backward=False), d, True, 1e-3 if d == 128 else LSE_MOST)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("length", [2048, 1984, 2012, 1660])
def test_pairs_at_the_ends_of_the_loop_over_the_keys(d, length):
    """The last tile whole, in either buffer (32 and 31 tiles; the ticket is then drawn in the loop), or ragged behind an odd number of whole
    ones (31 and 25)."""
    lens = [length, 130, length, 64]
    w = Q.walk_pairs(lens, HEADS[d], d)
    assert w.items > 100 and w.draws
    _compare(GpuRun(BagSpec("pair_ends", lens, H=HEADS[d], d=d, seed=9400 + d + length), backward=False), d, True, LSE_MOST)


@pytest.mark.parametrize("d,H", [(128, 4), (64, 8)])
def test_pairs_of_more_sequences_than_a_wave_has_lanes(d, H):
    """How many items are paired is counted by one wave, 64 sequences at a time."""
    lens = [1409 + (37 * i) % 192 for i in range(90)]
    assert min(lens) == 1409 and Q.walk_pairs(lens, H, d).items > 8 * 50
    _compare(GpuRun(BagSpec("many_pairs", lens, H=H, d=d, seed=9500 + d), backward=False), d, True, LSE_MOST, range(0, 90, 11), [0, H - 1])


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


# Inputs of known probabilities: keys of zeros but for a few with one entry, so that against the reference (the maximum of the first 64 keys,
# 0) a key's probability is 1 or 2^x.  One sequence of so many heads that most of its query tiles are paired.
L_ONE, HEADS_ONE = 1700, {128: 256, 64: 512}
# A probability of 2^x with x from here is 2^16 (1 + 0.56 .. 0.96 2^-8), which bf16 takes down to 2^16: alone, that is an error of 2.2e-3 to
# 3.7e-3 of lse, where such keys dominate the row.  With the second term 2^-17 of P is left, 7.6e-6 of lse; fp32 exponents of up to
# 64 and the logarithm of their sum take the rest of the bar.
X_DOWN = (16.0032, 16.0054)
LSE_BAR = 5e-5


def _entries(d, low, high):
    """Entries of a query and a key, exact in bf16, and the exponent x in [low, high] of their probability."""
    for i in range(128, 256):
        for j in range(128, 256):
            for e in range(-4, 5):
                a, b = i / 16.0, j / 128.0 * 2.0 ** e
                if low <= a * b * d ** -0.5 / math.log(2.0) <= high:
                    return a, b, a * b * d ** -0.5 / math.log(2.0)
    raise AssertionError((d, low, high))


def _lse_of_one_sequence(d, fill):
    """lse (H, L) of the sequence behind fill(q, k), in float64."""
    import torch
    import paper_2508_06001_amd as K
    H = HEADS_ONE[d]
    w = Q.walk_pairs([L_ONE], H, d)
    assert 2 * w.items > 7 * H          # of 14 H query tiles
    q, k, v = (torch.zeros((L_ONE, H, d), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    fill(q, k)
    out, lse = K.VarlenAttention([0, L_ONE], H, d, d ** -0.5).forward(q, k, v)
    assert bool((out == 0).all())
    return lse.double().cpu().numpy()


@pytest.mark.parametrize("huge_first", [True, False])
@pytest.mark.parametrize("d", [64, 128])
def test_second_term_of_a_row_beside_one_of_a_huge_sum(d, huge_first):
    """A lane holds two rows, 32 apart.  Those of one block have a key of 2^60, beside which the other block's three keys of 2^16 are nothing;
    they take their second term all the same."""
    a, b, x = _entries(d, *X_DOWN)
    a0, b0, x0 = _entries(d, 59.5, 60.5)
    rows = np.arange(L_ONE) % 64 < 32
    huge = rows if huge_first else ~rows

    def fill(q, k):
        import torch
        at = torch.from_numpy(huge).to("cuda")
        q[at, :, 0] = a0
        q[~at, :, 1] = a
        k[100, :, 0] = b0
        k[900:903, :, 1] = b

    lse = _lse_of_one_sequence(d, fill)
    want = np.where(huge, math.log(L_ONE - 1 + 2.0 ** x0), math.log(L_ONE - 3 + 3 * 2.0 ** x))
    assert math.log(L_ONE - 3 + 3 * 2.0 ** x) - math.log(L_ONE - 3 + 3 * 2.0 ** 16) > 20 * LSE_BAR      # without the second term
    err = float(np.abs(lse - want).max())
    say(f"[pairs] d={d} beside a huge sum: lse error={err:.2e}")
    assert err <= LSE_BAR


@pytest.mark.parametrize("keys", [(900, 901, 902), (930, 951, 959), (1665, 1670, 1695), (1696, 1698, 1699), (910, 940, 1690)])
@pytest.mark.parametrize("d", [64, 128])
def test_second_term_where_three_keys_dominate(d, keys):
    """In the first half of a tile, in the second, in either half of the ragged last tile (1664 to 1699), in several.  Rounded once their
    probabilities put lse off by more than 20 times the bar."""
    a, b, x = _entries(d, *X_DOWN)

    def fill(q, k):
        q[:, :, 1] = a
        k[list(keys), :, 1] = b

    want = math.log(L_ONE - 3 + 3 * 2.0 ** x)
    assert want - math.log(L_ONE - 3 + 3 * 2.0 ** 16) > 20 * LSE_BAR
    err = float(np.abs(_lse_of_one_sequence(d, fill) - want).max())
    say(f"[pairs] d={d} keys {keys}: lse error={err:.2e}")
    assert err <= LSE_BAR


def _one_sequence(d, change):
    """The sequence of known pairs with N(0, 1) inputs behind change(q, k, v): inputs and results of three heads in float64."""
    import torch
    import paper_2508_06001_amd as K
    H = HEADS_ONE[d]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9700 + d)
    q, k, v = (torch.empty((L_ONE, H, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(3))
    change(q, k, v)
    out, lse = K.VarlenAttention([0, L_ONE], H, d, d ** -0.5).forward(q, k, v)
    for h in (0, H // 2, H - 1):
        yield tuple(x[:, h].double().cpu().numpy() for x in (q, k, v, out)) + (lse[h].double().cpu().numpy(),)


@pytest.mark.parametrize("n", [32, 63, 64, 96, 200])
@pytest.mark.parametrize("d", [64, 128])
def test_pairs_behind_keys_of_minus_infinity(d, n):
    """The first n keys have scores of -inf: from 64 on the pair has no reference, and its rows are done again in parts.  Bars as in
    _compare, strict."""
    def change(q, k, v):
        q[:, :, 0] = 1.0
        k[:n, :, 0] = -math.inf

    for q, k, v, out, lse in _one_sequence(d, change):
        O, LSE = A.attn_fwd_dense(q, k[n:], v[n:], d ** -0.5)
        assert np.abs(out - O).max() <= 1e-2 and np.abs(lse - LSE).max() <= LSE_MOST


@pytest.mark.parametrize("what,value", [("q", math.nan), ("k", math.nan), ("v", math.nan), ("v", math.inf), ("k", math.inf)])
@pytest.mark.parametrize("d", [64, 128])
def test_pairs_with_infinities_and_nan(d, what, value):
    """One entry, behind the first 64 keys.  Rows whose fp64 result is finite are as without it (k = +inf: where q's entry is negative the
    score is -inf), the others not finite; a NaN or an infinity in q or v stays in its row or column."""
    def change(q, k, v):
        {"q": q, "k": k, "v": v}[what][700, :, 3] = value

    for q, k, v, out, lse in _one_sequence(d, change):
        with np.errstate(all="ignore"):
            O, LSE = A.attn_fwd_dense(q, k, v, d ** -0.5)
        finite = np.isfinite(O)
        assert 0 < int((~finite).sum()) and (what == "k" and value != math.inf or finite.any())
        assert not np.isfinite(out[~finite]).any()
        assert not finite.any() or np.abs(out[finite] - O[finite]).max() <= 1e-2
        rows = np.isfinite(LSE)
        assert not rows.any() or np.abs(lse[rows] - LSE[rows]).max() <= LSE_MOST
        assert not np.isfinite(lse[~rows]).any()
