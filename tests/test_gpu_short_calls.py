"""Short calls (whole bf16 calls of few key tiles: one launch that reads V as it is) next to the general path with its V^T
images: the same bits as the fp32 partial of the same call, which always takes the general path; and nothing behind the last
key of a key set reaches a result, whichever path reads it."""
import numpy as np
import pytest

from paper_2507_07966_amd import workloads as wl
from tests.gpu_util import forward_variant, to_device

pytestmark = pytest.mark.gpu
NAMES = ("q", "k_prefix", "v_prefix", "k_suffix", "v_suffix")


def run(plan, dev, lse_too=True):
    import torch
    import paper_2507_07966_amd as pa
    T, Hq, D = dev["q"].shape
    ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda").random_(0, 255)
    out = torch.full((T, Hq, D), float("nan"), device="cuda", dtype=torch.bfloat16)
    lse = torch.full((Hq, T), float("nan"), device="cuda")
    args = [dev[n] if dev[n].numel() else None for n in NAMES]
    pa.prefix_attn_forward(plan, *args, out, ws)
    pa.prefix_attn_lse(plan, ws, lse)
    o = torch.full((T, Hq, D), float("nan"), device="cuda")
    l = torch.full((T, Hq), float("nan"), device="cuda")
    pa.prefix_attn_forward_partial(plan, *args, True, o, l, ws)
    torch.cuda.synchronize()
    return out, lse, o, l


SHAPES = [
    # ragged prefixes and rollouts; blocks whole, cut, without a prefix
    (28, 4, 128, 130, (70, 41), "short"), (28, 4, 128, 1021, (67, 200), "short, cut"), (7, 1, 128, 0, (321, 65), "short"),
    (4, 4, 128, 0, (3001, 5), "short, cut"), (14, 2, 64, 515, (129, 300), "short"), (8, 2, 64, 5377, (40, 3, 300), "short, cut"),
    (4, 4, 64, 0, (700, 1, 64), "short"), (16, 16, 64, 77, (1, 1, 2, 33), "short"),
    # and of long calls
    (28, 4, 128, 20001, (333, 400, 67, 90), "ranges"), (4, 4, 64, 16253, (250, 33) * 32, "sweep"), (4, 2, 64, 0, (16500, 9), "own keys"),
]


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,variant", SHAPES)
def test_nothing_behind_the_last_key_reaches_a_result(Hq, Hkv, D, P, lens, variant):
    """K and V are slices at the start of larger tensors that hold NaN after their last row, and the second rollout's K and V, which
    share the first one's last tile, are NaN: everything but the second rollout's own rows keeps its bits."""
    import torch
    import paper_2507_07966_amd as pa
    print(f"behind the last key {Hq}/{Hkv}/{D} P={P} {lens[:4]} {variant}", flush=True)
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=71)
    dev = {n: to_device(x, n) for n in NAMES}
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, list(lens), x.workload.scale, dtype="bf16", device=0)
    assert forward_variant(plan) == variant
    clean = run(plan, dev)
    assert all(torch.isfinite(t).all() for t in clean)
    if plan.short_call:   # the general path's fp32 partial of the same call, rounded
        assert torch.equal(clean[2].bfloat16(), clean[0]) and torch.equal(clean[3].t(), clean[1])
    hostile = dict(dev)
    for n in NAMES[1:]:
        big = torch.full((len(dev[n]) + 256, Hkv, D), float("nan"), device="cuda", dtype=torch.bfloat16)
        hostile[n] = big[:len(dev[n])]
        hostile[n].copy_(dev[n])
    got = run(plan, hostile)
    assert all(torch.equal(a, b) for a, b in zip(got, clean))
    for n in ("k_suffix", "v_suffix"):
        hostile[n][lens[0]:lens[0] + lens[1]] = float("nan")
    got = run(plan, hostile)
    others = torch.ones(sum(lens), dtype=torch.bool)
    others[lens[0]:lens[0] + lens[1]] = False
    others = others.cuda()
    for a, b, token_axis in zip(got, clean, (0, 1, 0, 0)):
        assert torch.isnan(a[~others] if token_axis == 0 else a[:, ~others]).all()
        assert torch.equal(a[others], b[others]) if token_axis == 0 else torch.equal(a[:, others], b[:, others])
    plan.destroy()
