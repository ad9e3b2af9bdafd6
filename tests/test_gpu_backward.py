"""GPU parity of the backward: the HIP path (through the C ABI) against the fp64 oracle, element by
element on the same seeded inputs.  Tolerances are relative to each gradient tensor's
root-mean-square (see tests/gpu_util.py)."""
import numpy as np
import pytest

from oracle import cref
from oracle import ref_attention as ref
from paper_2507_07966_amd import workloads as wl
from tests.gpu_util import GRAD_NAMES, check_grads, delta_error_sigma, few_keys_floor, run_hip_backward

pytestmark = pytest.mark.gpu


def oracle_backward(x, d_out, scale=None):
    scale = x.workload.scale if scale is None else scale
    return cref.prefix_shared_attention_backward(x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix,
                                                 x.suffix_lens, scale, d_out)[:5]


def test_c1_tiny_fp32_backward_full_tensor():
    x = wl.make_inputs(wl.WORKLOADS["C1"])
    do, _ = wl.make_d_out(x)
    got = run_hip_backward(x, do)
    check_grads(got, oracle_backward(x, do), "f32", "C1")


EDGE = [
    # dtype, Hq, Hkv, D, P, suffix_lens
    ("bf16", 28, 4, 128, 300, (70, 1, 129, 64)),     # ragged, P and S not multiples of any tile
    ("bf16", 28, 4, 128, 0, (200, 37)),              # no prefix
    ("bf16", 4, 4, 128, 64, (1,)),                   # G = 1, S = 1, Hq = Hkv
    ("bf16", 8, 1, 128, 1, (65, 64, 63)),            # single prefix key, one kv head
    ("bf16", 14, 2, 64, 257, (100, 300)),            # head_dim 64
    ("bf16", 7, 1, 128, 1000, (37,) * 5),            # one GQA group, many short rollouts
    ("bf16", 2, 2, 128, 129, (513,)),                # group = 1, key blocks with a ragged tail
    ("bf16", 6, 2, 128, 200, (130, 127, 1, 129)),    # rollout boundaries inside row tiles and key blocks
    ("bf16", 8, 2, 64, 300, (1500, 700, 1)),         # short prefix, many rows: prefix key blocks split over row ranges
    ("bf16", 28, 4, 128, 5000, (40, 3)),             # few rows, long prefix: dQ over 9 prefix key ranges
    ("bf16", 8, 2, 64, 3000, (17,)),                 # the same with head_dim 64
    ("bf16", 7, 1, 128, 8192, (1200,)),              # one kv head: prefix key ranges (forward, dQ) and row ranges (dK/dV) at once
    ("bf16", 6, 3, 128, 300, (100, 57)),             # 3 kv heads do not divide the 8 XCDs: lists are not interleaved
    ("f32", 4, 2, 64, 100, (33, 70)),
    ("f32", 6, 2, 128, 0, (50, 1)),
    ("f32", 3, 3, 128, 65, (1, 2, 3)),
]


@pytest.mark.parametrize("dtype,Hq,Hkv,D,P,lens", EDGE)
def test_backward_edge_shapes_full_tensor(dtype, Hq, Hkv, D, P, lens):
    x = wl.make_custom(dtype, Hq, Hkv, D, P, lens, seed=3)
    do, bits = wl.make_d_out(x)
    print(f"backward edge case {dtype} Hq={Hq} Hkv={Hkv} D={D} P={P} lens={lens}", flush=True)
    got = run_hip_backward(x, do, bits)
    sig = delta_error_sigma(x, do)   # what the bf16-rounded forward output leaves in dQ and dK, from the definition
    check_grads(got, oracle_backward(x, do), dtype, f"edge {dtype} {Hq}/{Hkv}/{D} P={P} {lens}", sigmas=sig)
    # also against the plain definition (numpy: chain rule on the forward formula, softmax Jacobian written out),
    # which has none of the two-phase structure that the C version shares with the kernels
    if Hq * sum(lens) * (P + max(lens)) <= 3e7:
        plain = ref.prefix_shared_attention_backward(x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix,
                                                     x.suffix_lens, x.workload.scale, do)
        check_grads(got, plain, dtype, f"edge vs the plain definition {dtype} {Hq}/{Hkv}/{D} P={P} {lens}", sigmas=sig)


@pytest.mark.parametrize("std", [1.7, 2.5, 3.2])
@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [(14, 2, 128, 700, (150, 90)), (8, 2, 64, 300, (400, 37)), (7, 1, 128, 1, (171, 205))])
def test_backward_peaked_softmax_full_tensor(std, Hq, Hkv, D, P, lens):
    """Inputs of standard deviation 1.7 ... 3.2 give logits of standard deviation 3 ... 10: most rows put nearly
    all their weight on one or two keys.  Their exact dQ cancels to almost zero while the error that the
    bf16-rounded forward output leaves in delta does not, so the per-vector rounding model alone is not a
    bound here; delta_error_sigma() works that error out from the definition, element by element, and the
    tolerance is the sum of both (no term fitted to this test)."""
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=5, std=std)
    do, bits = wl.make_d_out(x)
    print(f"backward, peaked softmax: std={std} Hq={Hq} Hkv={Hkv} D={D} P={P} lens={lens}", flush=True)
    got = run_hip_backward(x, do, bits)
    check_grads(got, oracle_backward(x, do), "bf16", f"peaked std={std} {Hq}/{Hkv}/{D} P={P}", sigmas=delta_error_sigma(x, do))


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [(28, 4, 128, 500, (300, 129)), (8, 2, 64, 300, (1500, 700, 1))])
def test_backward_bitwise_reproducible(Hq, Hkv, D, P, lens):
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=7)
    do, bits = wl.make_d_out(x)
    a = run_hip_backward(x, do, bits)
    b = run_hip_backward(x, do, bits)
    for n in GRAD_NAMES:
        assert np.array_equal(a[n], b[n]), n


def test_c2_backward_full_tensor():
    x = wl.make_inputs(wl.WORKLOADS["C2"])
    do, bits = wl.make_d_out(x)
    got = run_hip_backward(x, do, bits)
    check_grads(got, oracle_backward(x, do), "bf16", "C2")


def test_backward_direct_key_block_path_full_tensor():
    """Element by element on the dK/dV path the long-prefix configurations take: head_dim 128, 7 query heads per
    kv head, 512 prefix key blocks (two rounds of workgroups, the last block of a head ragged), every block one
    work item that streams ALL stacked rows (no row ranges, no partial gradients), ragged rollouts."""
    import paper_2507_07966_amd as pa
    shape = (28, 4, 128, 16350, (500, 333, 129, 467, 71))
    plan = pa.prefix_attn_plan(*shape[:4], list(shape[4]), 128 ** -0.5, dtype="bf16", device=-1)
    ki = plan.key_items(0)
    ki = ki[ki[:, 2] >= 0]
    row_tiles = (sum(shape[4]) * 7 + 63) // 64
    assert len(ki) == 4 * 128 and (ki[:, 4] == 0).all() and (ki[:, 5] == row_tiles).all()    # direct path
    plan.destroy()
    x = wl.make_custom("bf16", *shape, seed=19)
    do, bits = wl.make_d_out(x)
    got = run_hip_backward(x, do, bits)
    check_grads(got, oracle_backward(x, do), "bf16", "direct dK/dV path, 16K prefix")


@pytest.mark.parametrize("D,P,lens", [(128, 64, (5000, 33, 5300)), (64, 64, (5000, 33, 5300)), (128, 1, (171, 605, 5377))])
def test_backward_long_rollouts_masked_and_mask_free_items_full_tensor(D, P, lens):
    """Rollouts long enough (512 row tiles and more) that the dK/dV pass over their own keys is split: per key
    block a masked item on the diagonal tiles (plus the rollout's last tile, which here also holds rows of the
    next rollout) and a mask-free item that walks the tiles between backwards, two fp32 partial gradients and
    their sum.  Element by element against the oracle; one kv head keeps the oracle at a few 1e11 FLOP.  The
    third shape has a one-key prefix: its first rows see two or three keys while the long rollout makes the
    gradient tensors small on average, the case that needs the few-keys term of the tolerance to be absolute."""
    import paper_2507_07966_amd as pa
    shape = (7, 1, D, P, lens)
    plan = pa.prefix_attn_plan(*shape[:4], list(shape[4]), D ** -0.5, dtype="bf16", device=-1)
    free = plan.key_items(2)
    long_ones = sum(1 for n in lens if n >= 4700)
    assert (free[:, 0] == -2).sum() >= 30 * long_ones and (plan.key_item_extra_tiles(1) >= 0).sum() >= 30 * (long_ones - 1)
    plan.destroy()
    x = wl.make_custom("bf16", *shape, seed=29)
    do, bits = wl.make_d_out(x)
    got = run_hip_backward(x, do, bits)
    check_grads(got, oracle_backward(x, do), "bf16", f"long rollouts, split dK/dV pass, D={D} P={P} {lens}",
                few_keys_floor(x, do))


def test_backward_and_logprob_on_side_stream_and_graph_replay():
    """Neither call allocates or synchronises, so both can run on any stream and be captured into a HIP graph;
    every replay must reproduce the eager result bit for bit (stale workspace contents must not matter)."""
    import torch
    import paper_2507_07966_amd as pa
    from tests.gpu_util import run_hip_backward
    x = wl.make_custom("bf16", 28, 4, 128, 700, (300, 129), seed=9)
    do, bits = wl.make_d_out(x)
    eager, (plan, args, grads) = run_hip_backward(x, do, bits, keep=True)
    bws = args[-1]
    lpw = wl.make_logprob_inputs(wl.LogprobWorkload("g", 300, 128, 1000, head_std=0.05, seed=2))
    h = torch.from_numpy(lpw.bits["hidden"].view(np.int16)).cuda().view(torch.bfloat16)
    W = torch.from_numpy(lpw.bits["lm_head"].view(np.int16)).cuda().view(torch.bfloat16)
    y = torch.from_numpy(lpw.targets).cuda()
    lws = torch.empty(pa.token_logprob_workspace(300, 128, 1000), dtype=torch.uint8, device="cuda")
    lp = torch.zeros(300, dtype=torch.float32, device="cuda")
    pa.token_logprob_forward(h, W, y, 1.0, lp, None, lws)
    torch.cuda.synchronize()
    lp_eager = lp.cpu().numpy().copy()

    def enqueue():
        pa.prefix_attn_backward(*args)
        pa.token_logprob_forward(h, W, y, 1.0, lp, None, lws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        enqueue()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        enqueue()
    for rep in range(3):
        for t in grads.values():
            t.zero_()
        lp.zero_()
        bws.random_(0, 255)
        lws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in GRAD_NAMES:
            assert np.array_equal(grads[n].float().cpu().numpy().astype(np.float64), eager[n]), f"replay {rep} {n}"
        assert np.array_equal(lp.cpu().numpy(), lp_eager), f"replay {rep} logprob"
    plan.destroy()


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [
    (14, 2, 64, 700, (1900, 37, 640)), (7, 1, 128, 0, (1111, 5)), (12, 2, 128, 129, (1025, 400)), (16, 2, 64, 0, (513,)),
])
def test_backward_own_key_blocks_cut_into_row_ranges_full_tensor(Hq, Hkv, D, P, lens):
    """Few key blocks: the rows of a rollout's first key blocks are cut into ranges, each a work item with a partial
    gradient (the workspace then holds slots of 2 x 128 x D fp32), in the same launch as the prefix blocks.  Ragged
    last blocks, row tiles that two rollouts share."""
    import paper_2507_07966_amd as pa
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, list(lens), D ** -0.5, dtype="bf16", device=-1)
    T, group = sum(lens), Hq // Hkv
    mpad = -(-T * group // 64) * 64
    tiles = -(-P // 64) + sum(-(-n // 64) for n in lens)
    fixed = 2 * T * Hq * 4 + 2 * Hkv * mpad * D * 2 + 3 * Hkv * mpad * 4 + Hkv * tiles * D * 64 * 2 + 12 * 256
    longest = max(plan.key_items(1)[:, 5] - plan.key_items(1)[:, 4])
    pre = plan.key_items(0)
    prefix_slots = len(pre[pre[:, 2] >= 0]) if len(pre) and pre[0, 5] - pre[0, 4] < mpad // 64 else 0
    dq_splits = len({int(k) for k in plan.items(2)[:, 4]})
    fixed += prefix_slots * 2 * 128 * D * 4 + (dq_splits if dq_splits > 1 else 0) * T * Hq * D * 4
    assert longest >= 32 and plan.backward_workspace_bytes >= fixed + 2 * 2 * 128 * D * 4
    plan.destroy()
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=31)
    do, bits = wl.make_d_out(x)
    # without a prefix the first rows see one or two keys, so their dQ is a difference of rounded terms: the absolute
    # few-keys term of few_keys_floor bounds it, as for the one-key prefix above
    check_grads(run_hip_backward(x, do, bits), oracle_backward(x, do), "bf16", f"own blocks cut {Hq}/{Hkv}/{D} P={P} {lens}",
                few_keys_floor(x, do))


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,whole", [
    (28, 4, 128, 3000, (2400, 100), True),         # 69 blocks of a kv head for 64 CUs: five cut, the others whole
    (14, 2, 128, 1377, (1500, 37, 1200, 60), False),   # fewer blocks than CUs: all cut, at and inside the own keys
    (14, 2, 128, 700, (2600,), True),              # the longest blocks cut, the others whole
    (6, 3, 64, 70, (6100,), True),                 # kv heads that share no layout over the XCDs
    (8, 2, 64, 0, (4200, 1), True),                # own keys only: ranges that some or all rows of a wavefront do not see
])
def test_backward_dq_blocks_cut_into_key_ranges_full_tensor(Hq, Hkv, D, P, lens, whole):
    """dQ of blocks of rows that do not fill the chip in whole rounds: ranges of [prefix | own keys] with fp32 partials,
    beside whole blocks, against the fp64 oracle."""
    import paper_2507_07966_amd as pa
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, list(lens), D ** -0.5, dtype="bf16", device=0)
    items = plan.launch_items(1)
    plan.destroy()
    real = items[items[:, 0] >= 0]
    cut = real[real[:, 7] >= 0]
    assert len(cut) and (cut[:, 6] > 0).any() and (len(cut) < len(real)) == whole
    x = wl.make_custom("bf16", Hq, Hkv, D, P, lens, seed=37)
    do, bits = wl.make_d_out(x)
    check_grads(run_hip_backward(x, do, bits), oracle_backward(x, do), "bf16", f"dq ranges {Hq}/{Hkv}/{D} P={P} {lens}",
                few_keys_floor(x, do))
