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

SHAPES = [
    # Hq, Hkv, D, P, suffix_lens
    (1, 1, 64, 0, (1,)),                      # one row, one key: seven of the eight wavefronts see nothing
    (2, 1, 128, 1, (1, 2)),
    (1, 1, 128, 15, (16, 17, 15)),            # edges of the row and key blocks
    (3, 1, 64, 16, (5, 6)),                   # 15 and 18 stacked rows
    (7, 1, 128, 129, (33, 64)),               # one key into a second round of the wavefronts
    (4, 2, 64, 257, (128, 1, 130)),
    (28, 4, 128, 500, (90, 70)),              # 7 heads per kv head, 16-row blocks
    (28, 4, 128, 200, (150, 55)),             # 359 blocks of 16 rows: 32-row blocks (one round of workgroups, not two)
    (28, 4, 128, 40, (300, 1)),               # 527 blocks: three rounds of 16-row blocks
    (16, 2, 64, 33, (1000, 31)),              # 1,031 blocks, head_dim 64: 16-row blocks, 5 rounds
    (16, 2, 64, 300, (900, 90)),              # 990 blocks: 32-row blocks, ragged against both sizes
]


@pytest.mark.parametrize("Hq,Hkv,D,P,lens", SHAPES)
def test_f32_forward_and_backward_tiles(Hq, Hkv, D, P, lens):
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
