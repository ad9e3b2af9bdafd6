"""The fp32 kernels at the sizes where their tiling can go wrong: 16-row and 32-row blocks, 16-key blocks, eight
wavefronts that share the keys (or rows) between them, and the switch to 32-row blocks.  Against the fp64 oracle.

Tolerance of the forward: 1e-5 absolute on out and LSE, as for the fp32 configuration of tests/test_gpu_parity.py: a
score is a sum of D <= 128 fp32 products of size <= 5 (error <= 128 * 2^-24 * 5 * sqrt(D) * scale < 4e-6 at the worst,
1e-6 typically), which moves a probability by as much relative to itself, and values are <= 5."""
import numpy as np
import pytest

from oracle import cref
from paper_2507_07966_amd import workloads as wl
from tests.gpu_util import check, check_grads, run_hip, run_hip_backward

pytestmark = pytest.mark.gpu

# Hq, Hkv, D, P, suffix_lens, the forward's blocks (rows of a block, wavefronts that share its keys)
SHAPES = [
    (1, 1, 64, 0, (1,), (16, 1)),             # one row, one key
    (2, 1, 128, 1, (1, 2), (16, 8)),          # seven of the eight wavefronts see nothing
    (1, 1, 128, 15, (16, 17, 15), (16, 8)),   # edges of the row and key blocks
    (3, 1, 64, 16, (5, 6), (16, 8)),          # 15 and 18 stacked rows
    (7, 1, 128, 129, (33, 64), (16, 8)),      # one key into a second round of the wavefronts
    (4, 2, 64, 257, (128, 1, 130), (16, 8)),
    (28, 4, 128, 500, (90, 70), (32, 8)),     # 7 heads per kv head; 284 blocks of 16 rows: 32-row blocks (one round of workgroups, not two)
    (28, 4, 128, 200, (150, 55), (32, 8)),
    (28, 4, 128, 40, (300, 1), (32, 8)),      # 532 blocks of 16 rows, three rounds; 268 of 32 rows, two
    (16, 2, 64, 33, (1000, 31), (32, 8)),     # 1,032 and 516 blocks, head_dim 64
    (16, 2, 64, 300, (900, 90), (32, 8)),     # 990 blocks: 32-row blocks, ragged against both sizes
    (28, 4, 128, 500, (90,) + (1,) * 60, (16, 8)),   # 400 blocks of 16 rows or 320 of 32, two rounds either way: 16-row blocks
    (16, 2, 64, 300, (700,) + (1,) * 90, (16, 8)),   # the same with head_dim 64: four rounds of 880 blocks, three of 530
    (4, 4, 128, 0, (1, 2, 17) * 100, (16, 1)),       # many short rollouts: one wavefront a block, one or two 16-key blocks each
    (8, 2, 64, 33, (1, 5) * 150, (16, 1)),           # the same with a ragged prefix
    (6, 1, 128, 1000, (1,) * 600, (16, 8)),          # many blocks that are nearly empty, over many keys
]


@pytest.mark.parametrize("Hq,Hkv,D,P,lens,blocks", SHAPES)
def test_f32_forward_and_backward_tiles(Hq, Hkv, D, P, lens, blocks):
    import paper_2507_07966_amd as pa
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, lens, D ** -0.5, dtype="f32", device=-1)
    assert blocks is None or tuple(plan.launch_items(3)[0, 3:5]) == blocks
    plan.destroy()
    x = wl.make_custom("f32", Hq, Hkv, D, P, lens, seed=31)
    do, _ = wl.make_d_out(x)
    print(f"fp32 tiles Hq={Hq} Hkv={Hkv} D={D} P={P} lens={lens}", flush=True)
    args = (x.q, x.k_prefix, x.v_prefix, x.k_suffix, x.v_suffix, x.suffix_lens, x.workload.scale)
    ro, rl, _ = cref.prefix_shared_attention(*args)
    out, lse = run_hip(x)
    mx, _, ml = check(out, lse, ro, rl, "fp32 tiles")
    assert mx < 1e-5 and ml < 1e-5
    got = run_hip_backward(x, do)
    check_grads(got, cref.prefix_shared_attention_backward(*args, do)[:5], "f32", f"fp32 tiles {Hq}/{Hkv}/{D} P={P} {lens}")


def test_f32_bitwise_reproducible():
    x = wl.make_custom("f32", 8, 2, 128, 300, (100, 57), seed=32)
    do, _ = wl.make_d_out(x)
    a, b = run_hip_backward(x, do), run_hip_backward(x, do)
    for n in a:
        if isinstance(a[n], np.ndarray):
            assert np.array_equal(a[n], b[n]), n


def test_f32_a_million_one_token_rollouts():
    """More blocks of rows than one launch dimension holds work-items for (2^32): forward and backward against a
    float64 evaluation of the four keys that each row sees.  Tolerance on the largest error, relative to each tensor's
    root mean square: 1e-4.  A dot product of 64 N(0, 1) channels has partial sums of at most 40 (five sigma), so it is
    off by up to sqrt(64) 2^-24 40 = 2e-5, dS (a difference of two) by 4e-5 p; times a key element of up to 5.7 and
    the scale 1/8 that is 2.7e-5 on dQ, whose elements are 0.4 in size: 7e-5 of it.  The output, dV and dK are products
    of fewer rounded terms; a prefix gradient is a sum of 10^6 terms of mixed sign, added in fp32 by eight
    wavefronts: 3 * 10^4 additions each of a sum of up to 400 terms' size, off by sqrt(3e4) 2^-24 = 1e-5 of it."""
    import torch
    import paper_2507_07966_amd as pa
    G, P, D = 1_100_000, 3, 64
    print(f"fp32 {G} one-token rollouts", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    q, ks, vs, do = (rand(G, 1, D) for _ in range(4))
    kp, vp = rand(P, 1, D), rand(P, 1, D)
    plan = pa.prefix_attn_plan(1, 1, D, P, np.ones(G, dtype=np.int32), D ** -0.5, dtype="f32", device=0)
    ws = torch.empty(max(plan.workspace_bytes, plan.backward_workspace_bytes), dtype=torch.uint8, device="cuda")
    out, lse = torch.full_like(q, float("nan")), torch.full((1, G), float("nan"), device="cuda")
    pa.prefix_attn_forward(plan, q, kp, vp, ks, vs, out, ws)
    pa.prefix_attn_lse(plan, ws, lse)
    torch.cuda.synchronize()
    grads = [torch.full_like(t, float("nan")) for t in (q, kp, vp, ks, vs)]
    pa.prefix_attn_backward(plan, q, kp, vp, ks, vs, out, do, lse, *grads, ws)
    torch.cuda.synchronize()
    plan.destroy()
    q6, ks6, vs6, do6, kp6, vp6 = (t[:, 0].double() for t in (q, ks, vs, do, kp, vp))
    s = torch.cat([(q6[:, None, :] * kp6[None]).sum(-1), (q6 * ks6).sum(-1, keepdim=True)], 1) * D ** -0.5
    l6 = torch.logsumexp(s, 1)
    p = torch.exp(s - l6[:, None])
    o6 = sum(p[:, j:j + 1] * vp6[j] for j in range(P)) + p[:, P:] * vs6
    dw = torch.cat([(do6[:, None, :] * vp6[None]).sum(-1), (do6 * vs6).sum(-1, keepdim=True)], 1)
    ds = p * (dw - (do6 * o6).sum(-1, keepdim=True)) * D ** -0.5
    want = [sum(ds[:, j:j + 1] * kp6[j] for j in range(P)) + ds[:, P:] * ks6,
            torch.stack([(ds[:, j:j + 1] * q6).sum(0) for j in range(P)]),
            torch.stack([(p[:, j:j + 1] * do6).sum(0) for j in range(P)]), ds[:, P:] * q6, p[:, P:] * do6]
    assert (lse[0].double() - l6).abs().max() < 1e-5
    for name, got, ref in zip(("out", "dq", "dk_prefix", "dv_prefix", "dk_suffix", "dv_suffix"), [out] + grads, [o6] + want):
        err = (got[:, 0].double() - ref).abs().max() / ref.square().mean().sqrt()
        print(f"{name}: {float(err):.2e}", flush=True)
        assert err < 1e-4, name


BAD = 37   # token whose value (key, query, upstream gradient) is not finite: inside a 16-row block, a 16-key block
CH = 5


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [(1, 1, 64, 0, (90,)), (4, 2, 128, 19, (130, 33)), (28, 4, 128, 40, (300, 1)),
                                             (4, 4, 128, 0, (47,) + (1, 2, 17) * 100)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_f32_non_finite_values_reach_only_the_rows_that_see_them(Hq, Hkv, D, P, lens, bad):
    """One bad value of the first rollout, or of the last prefix key (which masked steps past the prefix's end repeat),
    must leave every result that does not depend on it as it is without it; forward, dQ and dK / dV."""
    print(f"fp32 non-finite {bad} {Hq}/{Hkv}/{D} P={P} lens={lens}", flush=True)

    def run(name, row, value):
        x = wl.make_custom("f32", Hq, Hkv, D, P, lens, seed=33)
        do, _ = wl.make_d_out(x)
        (do if name == "d_out" else getattr(x, name))[row, 0, CH] = value
        out, lse = run_hip(x)
        return dict(run_hip_backward(x, do), out=out, lse=lse.T)   # all [tokens, heads ...]

    T, group = sum(lens), Hq // Hkv
    seen = np.arange(BAD, lens[0])
    rest = np.setdiff1d(np.arange(T), seen)
    before = np.setdiff1d(np.arange(T), np.arange(BAD + 1))   # keys that the bad row does not see
    same = lambda a, b: np.allclose(a, b, rtol=1e-5, atol=1e-6)
    # a value: one channel of the rows that see it, nothing else of the forward
    clean, got = run("v_suffix", BAD, 0.5), run("v_suffix", BAD, bad)
    want = got["out"][seen, :group, CH]
    assert np.isnan(want).all() if np.isnan(bad) else (want == bad).all()
    got["out"][seen, :group, CH] = clean["out"][seen, :group, CH]
    assert same(got["out"], clean["out"]) and same(got["lse"], clean["lse"])
    # a key: the rows that see it
    clean, got = run("k_suffix", BAD, 0.5), run("k_suffix", BAD, bad)
    for n in ("out", "lse", "dq"):
        assert same(got[n][rest], clean[n][rest]) and same(got[n][:, group:], clean[n][:, group:]), n
    # a query row or its upstream gradient: its own dQ, and the keys it sees
    for name in ("q", "d_out"):
        clean, got = run(name, BAD, 0.5), run(name, BAD, bad)
        other = np.setdiff1d(np.arange(T), [BAD])
        for n in ("out", "lse", "dq"):
            assert same(got[n][other], clean[n][other]), (name, n)
        for n in ("dk_suffix", "dv_suffix"):
            assert same(got[n][before], clean[n][before]) and same(got[n][:, 1:], clean[n][:, 1:]), (name, n)
    if P:
        clean, got = run("v_prefix", P - 1, 0.5), run("v_prefix", P - 1, bad)
        want = got["out"][:, :group, CH]
        assert np.isnan(want).all() if np.isnan(bad) else (want == bad).all()
        got["out"][:, :group, CH] = clean["out"][:, :group, CH]
        assert same(got["out"], clean["out"]) and same(got["lse"], clean["lse"])


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", [
    (1, 1, 64, 3000, (200, 50)), (7, 1, 128, 0, (900,)), (2, 1, 64, 65, (700,)), (4, 2, 128, 1, (513, 1, 700)), (2, 1, 128, 3000, (257, 9)),
    (4, 2, 128, 512, (300, 40)),   # rows and keys cut at D = 128
])
def test_f32_backward_cut_into_ranges(Hq, Hkv, D, P, lens):
    """Launches of few blocks, whose blocks of rows or keys are cut into ranges with partial sums: ranges that end inside a
    rollout, on its diagonal and in its ragged last block; a value that is not finite in the first of them."""
    import paper_2507_07966_amd as pa
    plan = pa.prefix_attn_plan(Hq, Hkv, D, P, lens, D ** -0.5, dtype="f32", device=-1)
    assert len(plan.launch_sums(6)) + len(plan.launch_sums(7)) > 0
    test_f32_forward_and_backward_tiles(Hq, Hkv, D, P, lens, None)
    test_f32_non_finite_values_reach_only_the_rows_that_see_them(Hq, Hkv, D, P, lens, float("inf"))
