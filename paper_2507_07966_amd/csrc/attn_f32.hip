// fp32 attention for fp32 inputs (exact checks, gradient checks, small debugging runs): the whole call in one kernel,
// a sweep over [prefix keys | the rollout's own keys] per block of rows with fp32 MFMAs (v_mfma_f32_16x16x4_f32: fp32
// products and sums, nothing is rounded below fp32).
//
// What bounds it: at its sizes (tens to a few thousand rows) the latency of one block's sweep, then the fp32 matrix
// rate (157 TFLOP/s nominal, 153 reached by a large product).  Hence the split: a workgroup owns only 16 * NQ stacked
// rows m = i * group + (h % group), and its 8 wavefronts take the keys between them, 32 (NQ = 1) or 16 (NQ = 2) at a
// time, each with an online softmax of its own; at the end the 8 partial results are combined through LDS in a fixed
// order.  A wavefront reads its K and V rows straight into MFMA operand registers: no two wavefronts of a workgroup
// need the same ones, so staging them in LDS would only add barriers.
//   - S^T = K Q^T: the A operand's lane (key l16, channel quarter g4) loads 16 consecutive bytes, four contraction
//     steps of K; Q sits in registers in the same channel order.
//   - The accumulator then holds, per lane, keys 4 g4 + i (i = 0..3) of query column l16, which is exactly the B
//     operand of O^T += V^T P^T when step j contracts over keys 4 g4 + j: P needs no data movement at all.
//   - V^T operands: a lane loads 4 consecutive channels of key 4 g4 + j, one for each of four MFMAs; row r of
//     accumulator (B, e) is channel 64 B + 4 r + e.
// NQ = 2 reads every key once for 32 rows (half the L2 traffic), NQ = 1 has twice the workgroups; with few keys a block
// has one wavefront (WAVES = 1) and takes 16 keys at a time: build_f32_blocks in plan.cpp chooses.
// Measured against one wavefront per row with scalar products (what this replaced): one head of 64 channels, 192 rows,
// 256 + 96 keys 2,223 -> 22 us for the call; 8 / 2 heads of 128 channels, 740 tokens over 1,000 + 70..300 keys 13.3 ms ->
// 62 us (67 TFLOP/s); 28 / 4 heads, 9,600 tokens over 4,000 + 600 keys 102 TFLOP/s, two thirds of the fp32 matrix rate.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "f32_rows.h"

namespace pa {
namespace {

using namespace f32rows;

__device__ inline float quad_max(float x) {  // over the lanes l16, l16 + 16, l16 + 32, l16 + 48 of a query column
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ inline float quad_sum(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

template <int D, int NQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 2) void pass_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_pre, const float* __restrict__ v_pre,
    const float* __restrict__ k_own, const float* __restrict__ v_own, float* __restrict__ out, float* __restrict__ lse,
    const WorkItem* __restrict__ items, int64_t num_items, const int32_t* __restrict__ cu, int P, bool with_own, int Hq,
    int Hkv, int group, float scale) {
  constexpr int ROWS = 16 * NQ;                              // rows of a workgroup
  constexpr int KB = NQ == 1 && WAVES > 1 ? 2 : 1;              // 16-key blocks per step of a wavefront
  constexpr int KS = D / 16, VB = D / 64;                    // 16-byte loads per key: along its row / per key of a step
  constexpr int LD = D + 4;                                  // padded row of the combine buffer (bank spread)
  __shared__ __attribute__((aligned(16))) float o_s[WAVES][ROWS][LD];
  __shared__ float m_s[WAVES][ROWS], l_s[WAVES][ROWS];

  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (block >= num_items) return;
  const WorkItem it = items[block];
  const int row0 = it.row0, off_g = cu[it.g];
  const int nrows = (cu[it.g + 1] - off_g) * group;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  auto packed_row = [&](int m) { return (int64_t)(off_g + m / group) * Hq + it.c * group + m % group; };

  // ---- this lane's query columns; rows past the rollout's end repeat its last row and are not written
  f32x4 Q[NQ][KS];
  int pos[NQ];
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    const int m = min(row0 + nq * 16 + l16, nrows - 1);
    pos[nq] = m / group;
    const float* qp = q + packed_row(m) * D + 4 * g4;
#pragma unroll
    for (int s = 0; s < KS; ++s) Q[nq][s] = *reinterpret_cast<const f32x4*>(qp + 16 * s);
  }
  const int nown = with_own ? (min(row0 + ROWS, nrows) - 1) / group + 1 : 0;  // own keys the last row sees
  const int np = (P + 15) / 16, nb = np + (nown + 15) / 16;                   // 16-key blocks: prefix, then own

  const int diagonal = np + (row0 / group + 1) / 16;  // own blocks from here on hold keys that some rows do not see

  f32x4 O[NQ][4 * VB];
  float m_run[NQ], l_run[NQ];
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    m_run[nq] = -INFINITY;
    l_run[nq] = 0.f;
#pragma unroll
    for (int b = 0; b < 4 * VB; ++b) O[nq][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // keys [key0, ..) of block b (a block past the last one: the last one again, masked away)
  struct Block { const float *k, *v; int key0, last; };
  auto block_of = [&](int b) {
    b = min(b, nb - 1);
    const bool pre = b < np;
    const int64_t first = ((int64_t)(pre ? 0 : off_g) * Hkv + it.c) * D;
    return Block{(pre ? k_pre : k_own) + first, (pre ? v_pre : v_own) + first, (pre ? b : b - np) * 16, (pre ? P : nown) - 1};
  };
  const int64_t stride = (int64_t)Hkv * D;
  f32x4 K[KB][KS], V[KB][4][VB];
  auto load_k = [&](int b0) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const Block b = block_of(b0 + kb);
      const float* p = b.k + min(b.key0 + l16, b.last) * stride + 4 * g4;
#pragma unroll
      for (int s = 0; s < KS; ++s) K[kb][s] = *reinterpret_cast<const f32x4*>(p + 16 * s);
    }
  };
  auto load_v = [&](int b0) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const Block b = block_of(b0 + kb);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* p = b.v + min(b.key0 + 4 * g4 + j, b.last) * stride + 4 * l16;
#pragma unroll
        for (int B = 0; B < VB; ++B) V[kb][j][B] = *reinterpret_cast<const f32x4*>(p + 64 * B);
      }
    }
  };

  bool bad = false;  // some value of the diagonal blocks is not finite
  if (wave * KB < nb) load_k(wave * KB);
  for (int b0 = wave * KB; b0 < nb; b0 += WAVES * KB) {
    load_v(b0);
    f32x4 S[KB][NQ];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int nq = 0; nq < NQ; ++nq) S[kb][nq] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int nq = 0; nq < NQ; ++nq)
            S[kb][nq] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[kb][s][j], Q[nq][s][j], S[kb][nq], 0, 0, 0);
    if (b0 + WAVES * KB < nb) load_k(b0 + WAVES * KB);
    // register i of S[kb][nq]: key 4 g4 + i of block b0 + kb, query column l16
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const bool pre = b0 + kb < np;
        const int key0 = (pre ? b0 + kb : b0 + kb - np) * 16 + 4 * g4;
        const int limit = b0 + kb >= nb ? -1 : pre ? P - 1 : pos[nq];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S[kb][nq][i] = key0 + i <= limit ? S[kb][nq][i] * scale : -INFINITY;
          mx = fmaxf(mx, S[kb][nq][i]);
        }
      }
      const float m_new = fmaxf(m_run[nq], quad_max(mx));
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // no visible key yet: every weight below is exp(-inf) = 0
      if (__any(m_new > m_run[nq])) {
        const float alpha = expf(m_run[nq] - m_ref);
        l_run[nq] *= alpha;
#pragma unroll
        for (int b = 0; b < 4 * VB; ++b) O[nq][b] *= alpha;
        m_run[nq] = m_new;
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          S[kb][nq][i] = expf(S[kb][nq][i] - m_ref);
          l_run[nq] += S[kb][nq][i];
        }
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int b = b0 + kb, keys = b >= nb ? 0 : b < np ? P - b * 16 : nown - (b - np) * 16;  // that exist in the block
      if (keys < 16) clear_rows_from(V[kb], keys, g4);
      if (b >= diagonal && clear_bad(V[kb])) bad = true;
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int B = 0; B < VB; ++B)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int nq = 0; nq < NQ; ++nq)
              O[nq][4 * B + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[kb][j][B][e], S[kb][nq][j], O[nq][4 * B + e], 0, 0, 0);
  }
  if (bad)  // the values that were cleared, for the rows that see them
    for (int b = diagonal; b < nb; ++b) {
      if (b / KB % WAVES != wave) continue;
      load_k(b);
#pragma unroll
      for (int nq = 0; nq < NQ; ++nq) {
        f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int j = 0; j < 4; ++j) p = __builtin_amdgcn_mfma_f32_16x16x4f32(K[0][s][j], Q[nq][s][j], p, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = expf(p[i] * scale - m_run[nq]);
        const int key0 = (b - np) * 16;
        add_bad<D>(O[nq], p, min(16, nown - key0), lane, [&](int r) { return key0 + r <= pos[nq]; },
                   [&](int r) { return v_own + ((int64_t)(off_g + key0 + r) * Hkv + it.c) * D; });
      }
    }

  // ---- combine the wavefronts: register i of O[nq][4 B + e] is channel 64 B + 4 (4 g4 + i) + e of query column l16
#pragma unroll
  for (int nq = 0; nq < NQ; ++nq) {
    const int r = nq * 16 + l16;
#pragma unroll
    for (int B = 0; B < VB; ++B)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(&o_s[wave][r][64 * B + 16 * g4 + 4 * i]) =
            f32x4{O[nq][4 * B][i], O[nq][4 * B + 1][i], O[nq][4 * B + 2][i], O[nq][4 * B + 3][i]};
    const float l = quad_sum(l_run[nq]);
    if (g4 == 0) {
      m_s[wave][r] = m_run[nq];
      l_s[wave][r] = l;
    }
  }
  __syncthreads();
  for (int n = threadIdx.x; n < ROWS * (D / 4); n += WAVES * 64) {
    const int r = n / (D / 4), ch = n % (D / 4) * 4;
    if (row0 + r >= nrows) continue;
    float m = m_s[0][r];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) m = fmaxf(m, m_s[w][r]);  // finite: every row sees a key
    float l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float a = expf(m_s[w][r] - m);  // a wavefront without a visible key: exp(-inf) = 0
      l += a * l_s[w][r];
      acc += a * *reinterpret_cast<const f32x4*>(&o_s[w][r][ch]);
    }
    const int64_t row = packed_row(row0 + r);
    *reinterpret_cast<f32x4*>(out + row * D + ch) = acc * (1.0f / l);
    if (ch == 0) lse[row] = m + logf(l);
  }
}

}  // namespace

int launch_pass_f32(const PassArgs& a, void* stream) {
  if (a.num_items == 0) return 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto f = [](const void* p) { return static_cast<const float*>(p); };
  const int P = a.k_pre ? (int)a.P : 0;
  const dim3 grid((unsigned)std::min(a.num_items, MAX_GRID_X), (unsigned)((a.num_items + MAX_GRID_X - 1) / MAX_GRID_X));
#define PA_LAUNCH(DD, NQ, WAVES)                                                                                   \
  pass_f32_kernel<DD, NQ, WAVES><<<grid, WAVES * 64, 0, s>>>(f(a.q), f(a.k_pre), f(a.v_pre), f(a.k), f(a.v), a.o_part, \
      a.lse_part, a.items, a.num_items, a.cu, P, a.causal, a.Hq, a.Hkv, a.group, a.scale)
#define PA_LAUNCH_D(DD)                                                                                            \
  if (a.block_rows == 32) PA_LAUNCH(DD, 2, 8);                                                                     \
  else if (a.block_waves == 8) PA_LAUNCH(DD, 1, 8);                                                                \
  else PA_LAUNCH(DD, 1, 1)
  if (a.D == 128) {
    PA_LAUNCH_D(128);
  } else {
    PA_LAUNCH_D(64);
  }
#undef PA_LAUNCH_D
#undef PA_LAUNCH
  return (int)hipGetLastError();
}

}  // namespace pa
