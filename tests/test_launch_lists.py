"""CPU tests of the lists that the launches run: every (block of rows, key tile) and every (key block, row tile) exactly
once, partial results in slots of their own inside the workspace, every sum over exactly its block's slots."""
import numpy as np
import pytest

import paper_2507_07966_amd as pa
from tests.random_shapes import random_shapes
from tests.test_plan_abi import host_plan

TILE, BLOCK, KEYS = 64, 256, 128


def check_slots(slots_of_block, sums, num_slots):
    """slots_of_block: block -> the slots its items leave, for cut blocks; sums: block -> (first slot, slots)."""
    assert set(slots_of_block) == set(sums)
    seen = []
    for block, slots in slots_of_block.items():
        first, n = sums[block]
        assert n > 1 and slots == list(range(first, first + n)), block
        seen += slots
    assert sorted(seen) == list(range(num_slots))


def check_row_lists(plan, which, P, lens, group):
    """Lists 0 and 1: the key sequence [prefix | own keys] of every block, in parts that its items sweep."""
    off = np.concatenate([[0], np.cumsum(lens)])
    blocks, cut = {}, {}
    for g, row0, c, nkeys, key0, pkeys, okey0, slot in plan.launch_items(which).tolist():
        if g < 0:
            continue
        assert key0 % TILE == 0 and okey0 % TILE == 0 and nkeys >= 0 and pkeys >= 0 and nkeys + pkeys > 0
        parts = ([(key0, key0 + pkeys)] if pkeys else []) + ([(P + okey0, P + okey0 + nkeys)] if nkeys else [])
        if which == 0 and not pkeys:
            assert okey0 <= row0 // group             # every row of the block sees the range's first key
        blocks.setdefault((g, row0, c), []).append((slot, parts))
        if slot >= 0:
            cut.setdefault((g, row0, c), []).append(slot)
    want = {(g, row0, c): P + (min(row0 + BLOCK, n * group) - 1) // group + 1
            for g, n in enumerate(lens) for row0 in range(0, n * group, BLOCK) for c in range(plan_heads(plan))}
    assert set(blocks) == set(want)
    for block, items in blocks.items():
        items.sort()
        assert items[0][0] >= 0 or len(items) == 1    # a block is whole or cut
        parts = sorted(p for _, ps in items for p in ps)
        assert parts[0][0] == 0 and parts[-1][1] == want[block]
        assert all(a[1] == b[0] for a, b in zip(parts, parts[1:])), (block, parts)
    sums = {}
    for off_g, row0, c, rows, first, n in plan.launch_sums(which).tolist():
        g = int(np.searchsorted(off, off_g, side="right") - 1)
        assert off[g] == off_g and rows == min(BLOCK, lens[g] * group - row0)
        assert (g, row0, c) not in sums
        sums[(g, row0, c)] = (first, n)
    check_slots({b: sorted(s) for b, s in cut.items()}, sums, plan.launch_slots(which))
    return len(cut), len(blocks) - len(cut)


def plan_heads(plan):
    return int(max(it[2] for it in plan.items(1))) + 1


def check_key_list(plan, P, lens, group):
    """List 2: the row tiles of every key block: all of them for prefix keys, from the block's first row on for own keys."""
    off = np.concatenate([[0], np.cumsum(lens)])
    row_tiles = -(-int(off[-1]) * group // TILE)
    tiles, cut, n_keys = {}, {}, {}
    for g, key0, c, nkeys, t0, t1, extra, slot in plan.launch_items(2).tolist():
        if c < 0:
            continue
        assert t0 <= t1 and 0 < nkeys <= KEYS
        own = int(g != -1)
        at = key0 if g < 0 else int(off[g]) + key0
        r = int(np.searchsorted(off, at, side="right") - 1) if own else -1
        if g == -2:                                   # the mask-free kernel: every row of the tiles sees every key
            assert t0 * TILE >= (at + nkeys - 1) * group and t1 * TILE <= off[r + 1] * group
        else:
            assert g == r
        streamed = list(range(t0, t1)) + ([extra] if g >= 0 and extra >= 0 else [])
        tiles.setdefault((own, at, c), []).extend(streamed)
        assert n_keys.setdefault((own, at, c), nkeys) == nkeys
        if slot >= 0:
            cut.setdefault((own, at, c), []).append(slot)
        else:
            assert len(tiles[(own, at, c)]) == len(streamed)   # it writes the result: the block's only item
    first = plan.mask_free_items()                    # a launch of the mask-free kernel, then one of the masked kernel
    if first >= 0:
        items = plan.launch_items(2)
        assert (items[:first, 0][items[:first, 2] >= 0] < 0).all() and (items[first:, 0][items[first:, 2] >= 0] >= 0).all()
    heads = plan_heads(plan)
    want = {(0, k, c): range(row_tiles) for k in range(0, P, KEYS) for c in range(heads)}
    for g, n in enumerate(lens):
        for k in range(0, n, KEYS):
            for c in range(heads):
                want[(1, int(off[g]) + k, c)] = range((int(off[g]) + k) * group // TILE, -(-int(off[g + 1]) * group // TILE))
    assert set(tiles) == set(want)
    for block, t in tiles.items():
        assert sorted(t) == list(want[block]), block
    sums = {(own, k, c): (first, n) for own, k, c, nkeys, first, n in plan.launch_sums(2).tolist() if nkeys == n_keys[(own, k, c)]}
    assert len(sums) == len(plan.launch_sums(2))
    check_slots({b: sorted(s) for b, s in cut.items()}, sums, plan.launch_slots(2))


def check_plan(Hq, Hkv, D, P, lens):
    plan = host_plan(num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, prefix_len=P, suffix_lens=list(lens))
    group, T = Hq // Hkv, sum(lens)
    fwd = (0, 0)
    if len(plan.launch_items(0)):
        fwd = check_row_lists(plan, 0, P, lens, group)
        assert fwd[0] > 0
    images = Hkv * (-(-P // TILE) + sum(-(-n // TILE) for n in lens)) * D * TILE * 2
    assert plan.workspace_bytes >= plan.launch_slots(0) * BLOCK * (D + 1) * 4 + T * Hq * 4 + images
    dq = check_row_lists(plan, 1, P, lens, group)
    check_key_list(plan, P, lens, group)
    mpad = -(-T * group // TILE) * TILE
    fixed = 2 * T * Hq * 4 + 2 * Hkv * mpad * D * 2 + 3 * Hkv * mpad * 4 + images
    slots = plan.launch_slots(1) * BLOCK * D * 4 + plan.launch_slots(2) * 2 * KEYS * D * 4
    assert fixed + slots <= plan.backward_workspace_bytes <= fixed + slots + 12 * 256
    return plan, fwd, dq


def shapes(n=70, seed=11):
    """Beside the shared random shapes: prefixes up to 2^17 with short rollouts, ordinary and long own key sets."""
    rng = np.random.default_rng(seed)
    out = list(random_shapes())
    for i in range(n):
        Hkv, group, D = int(rng.choice([1, 2, 3, 4, 8])), int(rng.choice([1, 2, 4, 7])), int(rng.choice([64, 128]))
        kind = i % 3
        P = int(2 ** rng.uniform(0, (17, 13, 16)[kind])) if rng.random() < 0.8 else 0
        lens = tuple(int(2 ** rng.uniform(0, (6, 11, 13)[kind])) for _ in range(int(rng.integers(1, 18 if kind == 0 else 6))))
        out.append((Hkv * group, Hkv, D, P, lens))
    return out


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", shapes())
def test_launch_lists_cover_every_pair_once(Hq, Hkv, D, P, lens):
    check_plan(Hq, Hkv, D, P, lens)


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [
    (28, 4, 128, 50000, (8,) * 16), (28, 4, 128, 60000, (1,) * 8), (4, 4, 128, 29000, (300,) * 16),
    (16, 8, 128, 26000, (32,) * 8), (16, 8, 64, 49000, (64,) * 16), (16, 8, 128, 20000, (32,) * 16),
    (28, 4, 128, 40000, (1,) * 32), (28, 4, 128, 0, (32768,)), (4, 4, 128, 0, (9115,)), (28, 4, 128, 4096, (1152,) * 8),
    (28, 4, 128, 3000, (2400, 100)), (14, 2, 128, 1377, (1500, 37, 1200, 60)), (14, 2, 128, 700, (2600,)),
    (6, 3, 64, 70, (6100,)), (8, 2, 64, 0, (4200, 1)), (14, 2, 64, 5377, (1500, 37, 1200, 1901, 60)), (4, 4, 128, 0, (3000,)),
])
def test_launch_lists_of_named_shapes(Hq, Hkv, D, P, lens):
    """Prefixes near the size of the static workspace (the prefix stays in key ranges if blocks of rows cannot be cut: room
    for a partial of every range and of the own keys), one long sequence, the ordinary short-video batch."""
    plan, fwd, _ = check_plan(Hq, Hkv, D, P, lens)
    splits = len({int(k) for k in plan.items(0)[:, 4]}) if P else 1
    if splits > 1 and fwd == (0, 0):
        assert plan.workspace_bytes >= (splits + 1) * sum(lens) * Hq * (D + 1) * 4


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [
    (1, 1, 64, 256, (96, 96)), (8, 2, 128, 1000, (70, 300, 111, 299)), (4, 4, 64, 0, (1,) * 2000), (28, 4, 128, 40, (300, 1)),
    (8, 2, 64, 33, (1, 5) * 150),
])
def test_f32_blocks_cover_every_row_once(Hq, Hkv, D, P, lens):
    plan = host_plan(num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, prefix_len=P, suffix_lens=list(lens), dtype="f32")
    group = Hq // Hkv
    for which in (3, 4):
        seen = [[np.zeros(n * group, dtype=np.int32) for n in lens] for _ in range(Hkv)]
        items = plan.launch_items(which)
        assert (items[:, 3] == items[0, 3]).all() and items[0, 3] in (16, 32) and (which == 3 or items[0, 3] == 16)
        for g, row0, c, rows in items[:, :4].tolist():
            assert row0 % rows == 0 and row0 < lens[g] * group
            seen[c][g][row0:row0 + rows] += 1
        assert all((s == 1).all() for per_head in seen for s in per_head)
    many_short = len(lens) > 100
    assert plan.launch_items(3)[0, 4] == (1 if many_short else 8)


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,cut", [
    (8, 2, 128, 1000, (70, 300, 111, 299), (False, True)), (1, 1, 64, 3000, (200, 50), (True, False)),
    (7, 1, 128, 0, (900,), (False, True)), (2, 1, 64, 65, (700,), (True, True)), (3, 3, 64, 17, (16, 1, 15), (False, False)),
    (4, 2, 128, 1, (513, 1, 700), (False, True)), (2, 1, 128, 3000, (257, 9), (True, False)),
])
def test_f32_backward_cuts_cover_every_pair_once(Hq, Hkv, D, P, lens, cut):
    """Lists 6 and 7 (empty: whole blocks): every 16-key block of a block of rows, every stacked row of a block of keys,
    in exactly one item; the slots of a block side by side and summed once."""
    plan = host_plan(num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, prefix_len=P, suffix_lens=list(lens), dtype="f32")
    group, off, np_ = Hq // Hkv, np.concatenate([[0], np.cumsum(lens)]).tolist(), -(-P // 16)
    rows, keys = plan.launch_items(6).tolist(), plan.launch_items(7).tolist()
    assert (len(plan.launch_sums(6)) > 0, len(plan.launch_sums(7)) > 0) == cut
    parts, slots = {}, {}
    for g, row0, c, nkeys, key0, _, _, slot in rows:
        parts.setdefault((g, row0, c), []).append((key0, key0 + nkeys))
        if slot >= 0:
            slots.setdefault((g, row0, c), []).append(slot)
    if rows:
        want = {(g, r, c): np_ + ((min(r + 16, n * group) - 1) // group + 16) // 16
                for g, n in enumerate(lens) for r in range(0, n * group, 16) for c in range(Hkv)}
        check_parts(parts, {b: (0, n) for b, n in want.items()})
    sums = {(off.index(o), r, c): (first, n) for o, r, c, nrows, first, n in plan.launch_sums(6).tolist()
            if nrows == min(16, lens[off.index(o)] * group - r)}
    check_slots({b: sorted(s) for b, s in slots.items()}, sums, plan.launch_slots(6))
    parts, slots = {}, {}
    for g, key0, c, nkeys, r0, r1, _, slot in keys:
        assert nkeys == min(16, (P if g < 0 else lens[g]) - key0)
        parts.setdefault((g, key0, c), []).append((r0, r1))
        if slot >= 0:
            slots.setdefault((int(g >= 0), key0 + (off[g] if g >= 0 else 0), c), []).append(slot)
    if keys:
        want = {(-1, k, c): (0, off[-1] * group) for k in range(0, P, 16) for c in range(Hkv)}
        want.update({(g, k, c): ((off[g] + k) * group, off[g + 1] * group)
                     for g, n in enumerate(lens) for k in range(0, n, 16) for c in range(Hkv)})
        check_parts(parts, want)
    sums = {(own, k, c): (first, n) for own, k, c, _, first, n in plan.launch_sums(7).tolist()}
    check_slots({b: sorted(s) for b, s in slots.items()}, sums, plan.launch_slots(7))
    need = plan.launch_slots(6) * 16 * D * 4 + plan.launch_slots(7) * 2 * 16 * D * 4 + 2 * sum(lens) * Hq * 4
    assert need <= plan.backward_workspace_bytes <= need + 2 * 256


def check_parts(parts, want):
    assert set(parts) == set(want)
    for block, p in parts.items():
        p.sort()
        assert (p[0][0], p[-1][1]) == want[block] and all(a < b for a, b in p)
        assert all(a[1] == b[0] for a, b in zip(p, p[1:])), block


def tiles_in_a_row(plan):
    """Key tiles of the longest item of a whole bf16 call, times the rounds that its items take on 256 CUs."""
    items = plan.launch_items(0) if len(plan.launch_items(0)) else plan.items(3) if plan.prefix_len else plan.items(1)
    items = items[items[:, 0] >= 0]
    return -(-len(items) // 256) * int((-(-items[:, 3] // TILE) + -(-items[:, 5] // TILE)).max())


CUT = (333, 400, 67, 90)


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,tiles,cut", [
    (4, 4, 128, 64 * 124, (256,) * 64, 128, False), (4, 4, 128, 64 * 124 + 1, (256,) * 64, 129, False),   # whole blocks, one round
    (4, 4, 64, 64 * 252, (256,) * 64, 256, False), (4, 4, 64, 64 * 252 + 1, (256,) * 64, 257, False),
    (28, 4, 128, 64 * 249, CUT, 128, True), (28, 4, 128, 64 * 249 + 1, CUT, 129, True),     # two ranges of the longest block
    (28, 4, 64, 64 * 505, CUT, 256, True), (28, 4, 64, 64 * 505 + 1, CUT, 257, True),
    (8, 8, 128, 0, (2688,) * 8, 126, False), (8, 8, 128, 0, (2689,) * 8, 129, False),       # no prefix, three rounds of 42 and 43
    (8, 8, 64, 0, (5440,) * 4, 255, False), (8, 8, 64, 0, (5441,) * 4, 258, False),
])
def test_short_calls_end_at_their_limit(Hq, Hkv, D, P, lens, tiles, cut):
    """Up to 128 (D = 64: 256) key tiles in a row are a short call."""
    plan = host_plan(num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, prefix_len=P, suffix_lens=list(lens))
    assert (len(plan.launch_items(0)) > 0) == cut and tiles_in_a_row(plan) == tiles
    assert plan.short_call == (tiles <= (128 if D == 128 else 256))


def test_short_calls_are_whole_bf16_calls():
    from paper_2507_07966_amd import binding
    assert host_plan(prefix_len=256, suffix_lens=[100]).short_call
    assert not host_plan(prefix_len=256, suffix_lens=[100], dtype="f32").short_call
    assert not host_plan(prefix_len=32768, suffix_lens=[2304] * 8).short_call          # the 32K-prefix workload: one sweep
    assert not host_plan(prefix_len=230400, suffix_lens=[2304] * 8).short_call         # separate passes
    assert binding.load_library().prefix_attn_plan_short_call(None) == -1


def test_launch_list_arguments():
    from paper_2507_07966_amd import binding
    lib = binding.load_library()
    plan = host_plan()
    assert lib.prefix_attn_plan_num_launch_items(plan.handle, 5) == -1 and lib.prefix_attn_plan_num_launch_items(None, 0) == -1
    assert lib.prefix_attn_plan_launch_items(plan.handle, 0, None) == 1
    assert lib.prefix_attn_plan_num_launch_sums(plan.handle, 3) == -1 and lib.prefix_attn_plan_launch_slots(plan.handle, -1) == -1
    f32 = host_plan(dtype="f32")
    assert all(len(f32.launch_items(w)) == 0 for w in (0, 1, 2)) and all(len(plan.launch_items(w)) == 0 for w in (3, 4))


def best_plan_time(repeats=12, **kw):
    import time
    best = float("inf")
    for _ in range(repeats):
        t = time.perf_counter()
        host_plan(**kw)
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("heads,D,lens", [((4, 4), 64, 15976), ((4, 4), 128, 15000), ((14, 2), 64, 4400)])
def test_search_for_cuts_is_a_small_part_of_making_a_plan(heads, D, lens):
    """A plan whose own key blocks are candidates for cuts against one of twice the length, which has too many blocks for
    the search: 1.4 to 2.2 times its time.  (A search that scheduled every candidate took 7 to 13 times.)  And the cuts are
    bounded: four partial-gradient slots per CU."""
    kw = dict(num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=D, prefix_len=0)
    plan = host_plan(suffix_lens=[lens], **kw)
    assert plan.launch_slots(2) <= 4 * 256
    assert best_plan_time(suffix_lens=[lens], **kw) < 5 * best_plan_time(suffix_lens=[2 * lens], **kw)


@pytest.mark.parametrize("heads,D,lens,longer", [((4, 4), 128, 3900, 4300), ((2, 2), 64, 7900, 8400)])
def test_search_for_fp32_cuts_is_a_small_part_of_making_a_plan(heads, D, lens, longer):
    """An fp32 plan whose blocks are candidates for cuts (and stay whole) against a slightly longer one, which has four blocks a CU
    and no search: 1.5 to 1.8 times its time.  (A search item by item, with every number of ranges tried, took 2.6 times.)"""
    kw = dict(num_q_heads=heads[0], num_kv_heads=heads[1], head_dim=D, prefix_len=0, dtype="f32")
    best = {lens: float("inf"), longer: float("inf")}
    for _ in range(20):                               # in turn: both see the same machine
        for n in best:
            best[n] = min(best[n], best_plan_time(repeats=4, suffix_lens=[n], **kw))
    assert best[lens] < 2.2 * best[longer]


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,cut", [
    (4, 4, 128, 54411, (1, 3, 19, 2, 7, 1), False), (16, 8, 128, 30115, (9, 2), False), (4, 4, 128, 46606, (5, 132, 127, 24, 42, 1), False),
    (4, 4, 128, 7922, (9, 2, 5, 1), True), (28, 4, 128, 1024, (128,), True), (28, 4, 128, 100000, (2, 3), True),
])
def test_cuts_that_the_workspace_limits_yield_to_key_ranges_of_the_prefix(Hq, Hkv, D, P, lens, cut):
    """Few short blocks over a long prefix: the 256-row slots that fit beside the layout copy allow a few ranges a block
    only (392 us for the first shape), fewer than the prefix pass has (166 us).  Calls whose cuts have room keep them."""
    plan, fwd, _ = check_plan(Hq, Hkv, D, P, lens)
    assert (fwd[0] > 0) == cut
    assert len({int(k) for k in plan.items(0)[:, 4]}) > 1
