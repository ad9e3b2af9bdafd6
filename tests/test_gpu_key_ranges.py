"""The keys [prefix | own keys] of some or all blocks of rows are cut into ranges, one work item each, and a merge adds
their partials.  Shapes where the cuts can go wrong: a ragged last prefix tile next to a cut, cuts inside
the own keys (at or before the block's first position), blocks whose lengths differ, as many ranges as the prefix has
tiles, whole calls with and without the caller's LSE and partials over a shard.  Against the fp64 oracle."""
import numpy as np
import pytest

from oracle import cref
from paper_2507_07966_amd import workloads as wl
from tests.gpu_util import check, forward_variant, run_hip, to_device

pytestmark = pytest.mark.gpu

SHAPES = [  # all have cut blocks (asserted); `whole`: whole blocks beside them in the same launch
    (28, 4, 128, 1024, (128,)),            # 16 blocks
    (28, 4, 128, 1000, (5, 3)),            # tiny rollouts, ragged last prefix tile
    (4, 4, 128, 193, (900,)),              # own keys outweigh the prefix: cuts inside them
    (1, 1, 64, 130, (2000,)),              # three prefix tiles
    (16, 2, 128, 3000, (1500,)),           # 94 blocks: two ranges
    (8, 2, 64, 5377, (40, 3, 300)),        # ragged everything
]
SHAPES = [s + (False,) for s in SHAPES] + [s + (True,) for s in [
    (28, 4, 128, 3000, (2400, 100)),       # 69 blocks of a kv head for 64 CUs: five cut, the others whole in the same launch
    (6, 3, 64, 700, (9000, 77)),           # kv heads that share no layout over the XCDs, 216 blocks
    (14, 2, 64, 5377, (1500, 37, 1200, 1901, 60)),   # 131 blocks of a kv head for 128 CUs
    (4, 4, 128, 0, (3000,)),               # own keys only: cut up to the diagonal, the first blocks whole
    (8, 8, 64, 0, (1, 63, 64, 65, 1281)),
]]


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,whole", SHAPES)
def test_key_ranges_whole_call_and_partial(Hq, Hkv, D, P, lens, whole):
    import torch
    import paper_2507_07966_amd as pa
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=P + Hq)
    print(f"key ranges {Hq}/{Hkv}/{D} P={P} lens={lens}", flush=True)
    ro, rl, _ = cref.prefix_shared_attention(x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix, x.suffix_lens, x.workload.scale)
    out, lse = run_hip(x)
    check(out, lse, ro, rl, f"key ranges {Hq}/{Hkv}/{D} P={P} {lens}")
    dev = [to_device(x, n) for n in ("q", "k_prefix", "v_prefix", "k_suffix", "v_suffix")]
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, list(lens), x.workload.scale, dtype="bf16", device=0)
    items = plan.launch_items(0)
    slots = items[items[:, 0] >= 0][:, 7]
    assert (slots >= 0).any() and (slots < 0).any() == whole
    T = sum(lens)
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda").random_(0, 255)
    o = torch.full((T, Hq, D), float("nan"), device="cuda")
    l = torch.full((T, Hq), float("nan"), device="cuda")
    pa.prefix_attn_forward_partial(plan, *dev, True, o, l, ws)
    # static entry point: the merge writes the caller's [Hq, T] LSE itself, or none at all
    so = torch.full((T, Hq, D), float("nan"), device="cuda", dtype=torch.bfloat16)
    sl = torch.full((Hq, T), float("nan"), device="cuda")
    if plan.workspace_bytes <= pa.STATIC_SCRATCH_BYTES:
        pa.prefix_attn_forward_static(plan, *dev, so, sl)
        torch.cuda.synchronize()
        assert np.array_equal(so.double().cpu().numpy(), out) and np.array_equal(sl.double().cpu().numpy(), lse)
        so.fill_(float("nan"))
        pa.prefix_attn_forward_static(plan, *dev, so, None)
        torch.cuda.synchronize()
        assert np.array_equal(so.double().cpu().numpy(), out)
    torch.cuda.synchronize()
    plan.destroy()
    check(o.double().cpu().numpy(), l.t().double().cpu().numpy(), ro, rl, f"key ranges, partial {Hq}/{Hkv}/{D} P={P} {lens}")


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [
    (28, 4, 128, 50000, (8,) * 16), (28, 4, 128, 60000, (1,) * 8), (28, 4, 128, 40000, (1,) * 32),
    (4, 4, 128, 29000, (300,) * 16), (16, 8, 128, 26000, (32,) * 8), (16, 8, 64, 49000, (64,) * 16),
    (16, 8, 128, 15360, (32,) * 16), (16, 8, 128, 20000, (32,) * 16), (16, 8, 128, 25344, (32,) * 16),
])
def test_split_prefix_near_the_size_of_the_static_workspace(Hq, Hkv, D, P, lens):
    """Few short blocks of rows over a long prefix: the values' layout copy leaves little of the library's own workspace,
    so the blocks may not be cut into ranges; the prefix pass's partials of every key range then have to be merged."""
    import torch
    import paper_2507_07966_amd as pa
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=P + Hq)
    label = f"split prefix {Hq}/{Hkv}/{D} P={P} {len(lens)} x {lens[0]}"
    print(label, flush=True)
    rows = np.arange(0, sum(lens), max(1, Hq * P * sum(lens) // 100_000_000))   # what the oracle does in about a second
    ro, rl, _ = cref.prefix_shared_attention(x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix, x.suffix_lens,
                                             x.workload.scale, rows=rows)
    out, lse, plan, dev, ws, _, _ = run_hip(x, return_plan=True)
    check(out[rows], lse[:, rows], ro, rl, label)
    assert len({int(k) for k in plan.items(0)[:, 4]}) > 1 and len(plan.launch_items(0)) == 0
    assert plan.workspace_bytes <= pa.STATIC_SCRATCH_BYTES
    T = sum(lens)
    names = ("q", "k_prefix", "v_prefix", "k_suffix", "v_suffix")
    so = torch.full((T, Hq, D), float("nan"), device="cuda", dtype=torch.bfloat16)
    sl = torch.full((Hq, T), float("nan"), device="cuda")
    pa.prefix_attn_forward_static(plan, *[dev[n] for n in names], so, sl)
    o = torch.full((T, Hq, D), float("nan"), device="cuda")
    l = torch.full((T, Hq), float("nan"), device="cuda")
    pa.prefix_attn_forward_partial(plan, *[dev[n] for n in names], True, o, l, ws)
    torch.cuda.synchronize()
    plan.destroy()
    assert np.array_equal(so.double().cpu().numpy(), out) and np.array_equal(sl.double().cpu().numpy(), lse)
    check(o[rows].double().cpu().numpy(), l[rows].t().double().cpu().numpy(), ro, rl, f"{label}, partial")


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,variant,hidden", [
    (28, 4, 128, 960, (128,), "short, cut", (256, 704)),           # whole ranges of prefix keys, and first tiles of ranges
    (4, 4, 128, 0, (3000,), "short, cut", (700, 1900)),            # own keys
    (14, 2, 64, 5377, (1500, 37, 1200, 1901, 60), "short, cut", (1000, 4500)),   # beside whole blocks
    # long calls, with a second launch for the items given up; a whole range is hidden (asserted)
    (28, 4, 128, 20000, (333, 400, 67, 90), "ranges", (0, 12000)),
    (14, 2, 64, 60000, (300, 400, 500, 77), "ranges", (15000, 45000)),
])
def test_key_ranges_whose_scores_are_all_minus_infinity(Hq, Hkv, D, P, lens, variant, hidden):
    """Keys that a bias channel of minus infinity hides: a range may then hold no key that counts, and adds nothing."""
    import torch
    import paper_2507_07966_amd as pa
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=41)
    print(f"hidden keys {Hq}/{Hkv}/{D} P={P} lens={lens}", flush=True)
    x.q[:, :, 0] = 1.0
    for k in (x.k_prefix, x.k_suffix):
        k[:, :, 0] = 0.0
    (x.k_prefix if P else x.k_suffix)[hidden[0]:hidden[1], :, 0] = -np.inf
    for n in ("q", "k_prefix", "k_suffix"):
        x.bits[n], _ = wl.round_to_bf16(getattr(x, n))
    step = max(1, sum(lens) // (300 if P < 10000 else 60))   # what the oracle does in a few seconds
    rows = np.arange(0, sum(lens), step)
    ro, rl, _ = cref.prefix_shared_attention(x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix, x.suffix_lens,
                                             x.workload.scale, rows=rows)
    out, lse, plan, dev, ws, _, _ = run_hip(x, return_plan=True)
    assert forward_variant(plan) == variant and plan.launch_slots(0) > 0
    if P:
        assert any(slot >= 0 and nkeys == 0 and hidden[0] <= key0 and key0 + pkeys <= hidden[1]
                   for g, _, _, nkeys, key0, pkeys, _, slot in plan.launch_items(0).tolist() if g >= 0)
    check(out[rows], lse[:, rows], ro, rl, "hidden keys")
    o = torch.full((sum(lens), Hq, D), float("nan"), device="cuda")
    l = torch.full((sum(lens), Hq), float("nan"), device="cuda")
    pa.prefix_attn_forward_partial(plan, *[dev[n] for n in ("q", "k_prefix", "v_prefix", "k_suffix", "v_suffix")], True, o, l, ws)
    torch.cuda.synchronize()
    plan.destroy()
    check(o[rows].double().cpu().numpy(), l[rows].t().double().cpu().numpy(), ro, rl, "hidden keys, partial")


@pytest.mark.parametrize("P,lens,variant", [(960, (128,), "short, cut"), (20000, (333, 400, 67, 90), "ranges")])
def test_key_ranges_keep_an_infinite_value_infinite(P, lens, variant):
    """An infinity in the value of a rollout's first token, which all of its rows see: the channel is infinite in every one of
    them, for its kv head, and nothing else changes (the merge reads the last range, which holds it, several times)."""
    x = wl.make_custom("bf16", 28, 4, 128, P, lens, seed=43)
    print(f"infinite value P={P}", flush=True)
    clean, clean_lse = run_hip(x)
    x.v_suffix[0, 0, 5] = np.inf
    x.bits["v_suffix"], _ = wl.round_to_bf16(x.v_suffix)
    out, lse, plan, *_ = run_hip(x, return_plan=True)
    assert forward_variant(plan) == variant and plan.launch_slots(0) > 0
    n = lens[0]
    assert np.isposinf(out[:n, :7, 5]).all()
    out[:n, :7, 5] = clean[:n, :7, 5]
    assert np.array_equal(out, clean) and np.array_equal(lse, clean_lse)
