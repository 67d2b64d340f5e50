"""The kernels' work queues and the host's rules about them, walked through on the CPU (tests/queue_model.cpp compiles the same
headers): every item, or every part of it, is dealt out exactly once."""
import random

import pytest

import queue_model as Q


def _random_bag(rng):
    n = rng.choice((1, 1, 2, 3, 4, 7, 16, 33, 200))
    top = rng.choice((64, 300, 1500, 6000, 40000))
    lens = [max(0, int(top ** rng.random())) for _ in range(n)]
    if rng.random() < 0.3:
        lens[rng.randrange(n)] = 0
    if rng.random() < 0.3:
        lens = [lens[0]] * n
    return lens


@pytest.mark.parametrize("causal", [False, True])
def test_every_item_of_one_kind_once(causal):
    rng = random.Random(1 + causal)
    draws = {True: 0, False: 0}
    for _ in range(600):
        lens, H, d = _random_bag(rng), rng.choice((1, 2, 3, 6, 12, 24, 48)), rng.choice((64, 128))
        cus = rng.choice((256, 256, 256, 304, 80, 37))          # 37: no multiple of eight workgroups, one queue
        for pairs in (2, 4) if d == 128 else (2,):              # d = 64: no form with four
            for kernel in ("fwd", "dq", "dkdv"):
                w = Q.walk(kernel, lens, H, d, causal, pairs, cus)
                assert w.wrong == 0, (kernel, lens, H, d, causal, pairs, cus, w)
                draws[w.draws] += 1
    assert min(draws.values()) > 300, draws


def test_bags_that_the_kernels_deal_out_in_each_way():
    """The model tells apart what the GPU tests rely on: all parts, whole items and parts, whole items with draws."""
    assert Q.walk("fwd", [37, 128, 200, 311], 2, 64, False) == Q.Walk(14, 28, 96, 4, False, 0)
    w = Q.walk("dq", [2081], 31, 128, False)
    assert w.items == 17 * 31 and w.parts == 2 * (17 * 31 - 512) and w.draws
    w = Q.walk("dkdv", [450] * 32, 24, 128, False)
    assert Q.dkdv_pairs([450] * 32, 24, 128, False) == 2 and w.items == 32 * 24 * 4 and w.draws and not w.parts
    # few items behind a single round: in parts where the round's shortest item and one of them take longer than the longest
    w = Q.walk("fwd", [1536, 1000], 27, 128, False)
    assert w.items == 20 * 27 and 0 < w.parts < w.items and w.draws
    assert Q.walk("fwd", [8192, 6000, 4500, 4400], 3, 128, False).parts > 0
    for lens, H in (([8192, 8192, 4300, 4300], 3), ([8192, 8192, 4096, 4096], 3), ([3000, 1500, 1000], 12)):
        w = Q.walk("fwd", lens, H, 128, False)
        assert w.items > 512 and w.draws and not w.parts


@pytest.mark.parametrize("causal", [False, True])
def test_every_item_of_both_kinds_once(causal):
    """The launch of both kinds of items: random bags and grids, all parts, thin last rounds and none."""
    rng = random.Random(30 + causal)
    seen = {"all": 0, "thin": 0, "none": 0}
    for _ in range(1500):
        lens, H, d = _random_bag(rng), rng.choice((1, 2, 3, 6, 12, 24, 48)), rng.choice((64, 128))
        cus = rng.choice((256, 256, 256, 304, 80, 37))
        w = Q.walk_joint(lens, H, d, causal, cus)
        assert w.wrong == 0, (lens, H, d, causal, cus, w)
        split = 4 if causal else 2
        seen["none" if w.parts == 0 else "all" if w.parts == w.items * split else "thin"] += 1
    assert min(seen.values()) > 20, seen


def test_every_item_of_the_unmasked_forward_once():
    """Its tickets: pairs of items, single ones, parts; random bags and grids, with and without pairs, all in parts."""
    rng = random.Random(77)
    seen = {"pairs": 0, "no pairs": 0, "all parts": 0}
    for _ in range(1500):
        lens, H, d = _random_bag(rng), rng.choice((1, 2, 3, 6, 12, 24, 48)), rng.choice((64, 128))
        cus = rng.choice((256, 256, 256, 304, 80, 37))
        w = Q.walk_pairs(lens, H, d, cus)
        assert w.wrong == 0, (lens, H, d, cus, w)
        items = H * sum((x + 127) // 128 for x in lens)
        seen["pairs" if w.items else "all parts" if items and w.parts == 2 * items else "no pairs"] += 1
    assert min(seen.values()) > 100, seen


@pytest.mark.parametrize("lens,H,d,pairs", [([6000] + [250] * 10, 48, 64, False), ([6000] + [250] * 20, 24, 128, True), ([10000], 48, 64, True)])
def test_a_few_pairs_are_none_at_d_64(lens, H, d, pairs):
    assert (Q.walk_pairs(lens, H, d).items > 0) == pairs


def test_every_item_of_the_small_backward_once():
    """Tiles of 64 rows of both kinds; random bags and grids, drawn and not.  Where the rule takes it, one launch is the rule as well."""
    rng = random.Random(99)
    seen = {False: 0, True: 0}
    for _ in range(1500):
        lens, H, d = _random_bag(rng), rng.choice((1, 2, 3, 6, 12, 24, 48)), rng.choice((64, 128))
        cus = rng.choice((256, 256, 256, 304, 80, 37))
        w = Q.walk_small(lens, H, d, cus)
        assert w.wrong == 0 and w.parts == 0, (lens, H, d, cus, w)
        seen[w.draws] += 1
        for causal in (False, True):
            assert not Q.bwd_small(lens, H, d, causal, cus) or Q.bwd_joint(lens, H, d, causal, cus), (lens, H, d, causal)
    assert min(seen.values()) > 100, seen


def test_small_items_are_left_to_the_device_where_the_lengths_decide():
    """Where the host takes tiles of 64 rows by itself the device would for any lengths of that sum and number; random bags near the
    limits of every rule."""
    rng = random.Random(123)
    seen = {0: 0, 1: 0, 2: 0, "not": 0}
    for _ in range(6000):
        H, d, causal = rng.choice((1, 2, 3, 6, 12, 24, 48)), rng.choice((64, 128)), rng.random() < 0.6
        cus = rng.choice((256, 256, 304, 80, 37))
        room = max(1, int(rng.uniform(0.1, 0.6) * cus * (3 if d == 64 else 2) / H))        # tiles of 128 rows
        top = rng.choice((64, 128, 192, 256, 320, 600, 128 * room))
        lens = []
        while sum((x + 127) // 128 for x in lens) < room and len(lens) < 2048:
            lens.append(rng.choice((0, 1, top, rng.randint(1, top))))
        if sum(lens) == 0:
            continue
        s = Q.small_items(lens, H, d, causal, cus)
        assert s.host < 2 or s.pays, (lens, H, d, causal, cus)
        assert bool(s.host) == Q.bwd_small(lens, H, d, causal, cus)
        seen[s.host] += 1
        seen["not"] += s.host == 1 and not s.pays
    assert min(seen.values()) > 100, seen


@pytest.mark.parametrize("lens,H,d,causal,pays", [
    ([10019], 3, 128, True, None), ([10019, 1], 3, 128, True, False), ([20644, 0, 0], 2, 64, True, False),    # one long sequence, alone or not
    ([5262] + [300] * 17, 3, 128, True, True),
    ([1, 200] * 20, 3, 128, False, False), ([1, 200] * 7, 12, 64, False, False), ([1, 200] * 17, 3, 128, False, True),
    ([128] * 40, 6, 128, True, False), ([128] * 46, 6, 128, True, True), ([64] * 46, 6, 128, True, True), ([96] * 24, 12, 64, True, False),
    ([160] * 35, 6, 64, True, False), ([256] * 24, 6, 64, True, True), ([256] * 35, 6, 64, True, False), ([320] * 23, 6, 64, True, True)])
def test_small_items_of_bags_measured_both_ways(lens, H, d, causal, pays):
    """pays: None where the host does not ask."""
    s = Q.small_items(lens, H, d, causal)
    assert s.host == (0 if pays is None else s.host) and (pays is None or (s.host in ((1, 2) if pays else (1,)) and s.pays == pays)), s


@pytest.mark.parametrize("start", [0, (1 << 32) - 20000])
def test_counter_sets_are_cleared_between_two_uses_far_from_either(start):
    """Eager forward calls: between two calls that draw from one set some call clears it, and calls that touch a set (draw from
    it or clear it) are at least 4096 apart, so that none of them meet as long as no call runs beside one that much younger.
    Captured calls have sets of their own."""
    start -= start % 12288
    touched, cleared = {}, {}
    for call in range(start, start + 5 * 12288):
        got, clear = Q.eager_set(call)
        for s in ([] if clear is None else range(clear, clear + 4096)):
            assert call - touched.get(s, call - 4096) >= 4096
            touched[s] = call
            cleared[s] = True
        assert 0 <= got < 12288 and call - touched.get(got, call - 4096) >= 4096
        if call >= start + 12288:
            assert cleared[got]
        touched[got], cleared[got] = call, False
    assert {Q.captured_set(c) for c in range(9000)} == set(range(12288, 16384))
