// Backward in fp32 (exact checks, gradient checks, small debugging runs) with fp32 MFMAs (v_mfma_f32_16x16x4_f32):
// a query-stationary kernel for dQ and a key-stationary one for dK and dV, no atomics, fixed summation order.
//   W_j = exp(scale <q, k_j> - LSE),  dS_j = W_j (<dO, v_j> - delta),
//   dQ = scale sum_j dS_j k_j,  dK_j = scale sum_rows dS_j q,  dV_j = sum_rows W_j dO,
// a prefix key summing over the rows of all rollouts (paper Sec. 5.1: shared video prefix).
//
// What bounds it: at these sizes latency, then the fp32 matrix rate.  Both kernels keep 16 columns (query rows, keys)
// per workgroup and deal the streamed side out to 8 wavefronts 16 at a time, so even a few hundred rows or keys give
// every CU work; the 8 partial sums are added through LDS at the end.  As in the forward (attn_f32.hip) a streamed row
// is read twice, straight into MFMA operand registers: once with lane (row l16, channel quarter g4) for the products
// over channels, once with lane (row 4 g4 + j, channels 4 l16 ..) for the products over rows, where the accumulator of
// the first product (rows 4 g4 + i of column l16) is the B operand of step j = i without any data movement.
// Measured (8 / 2 heads of 128 channels, 740 tokens over 1,000 + 70..300 keys), against one wavefront per row / per key
// with wavefront reductions for every dot product: dQ 1,350 -> 105 us, dK/dV 1,890 -> 182 us (59 and 45 TFLOP/s).
// At most two of the four loads of a block are in registers at a time: each is issued one product ahead of its use.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bwd.h"
#include "f32_rows.h"

namespace pa {
namespace {

using namespace f32rows;

constexpr int BF_WAVES = 8;

template <int D>
struct Col {  // 16 columns (rows of q / dO / k / v) as MFMA B operands over channels: lane (l16, g4) holds 16 s + 4 g4 ..
  f32x4 x[D / 16];
  __device__ inline void load(const float* row, int g4) {
#pragma unroll
    for (int s = 0; s < D / 16; ++s) x[s] = *reinterpret_cast<const f32x4*>(row + 16 * s + 4 * g4);
  }
};
template <int D>
struct Rows {  // 16 streamed rows as MFMA A operands over rows: lane holds channels 64 B + 4 l16 .. of rows 4 g4 + j
  f32x4 x[4][D / 64];
  __device__ inline void load(const float* base, const int (&row)[4], int64_t stride, int l16) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int B = 0; B < D / 64; ++B) x[j][B] = *reinterpret_cast<const f32x4*>(base + row[j] * stride + 64 * B + 4 * l16);
  }
};
// [16 streamed rows] x [16 columns] over all channels; two accumulation chains
template <int D>
__device__ inline f32x4 dot16(const Col<D>& a, const Col<D>& b) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s][0], b.x[s][0], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s][1], b.x[s][1], s1, 0, 0, 0);
    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s][2], b.x[s][2], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[s][3], b.x[s][3], s1, 0, 0, 0);
  }
  return s0 + s1;
}
// acc[4 B + e] (16 channels x 16 columns; row r is channel 64 B + 4 r + e) += rows^T w
template <int D>
__device__ inline void outer16(f32x4 (&acc)[D / 16], const Rows<D>& r, f32x4 w) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int B = 0; B < D / 64; ++B)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[4 * B + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.x[j][B][e], w[j], acc[4 * B + e], 0, 0, 0);
}

// Sum of the wavefronts' accumulators: LDS [wavefront][column][D], padded rows; column c, channels ch .. ch + 3.
template <int D>
struct Partials {
  float x[BF_WAVES][16][D + 4];
  __device__ inline void put(const f32x4 (&acc)[D / 16], int wave, int l16, int g4) {
#pragma unroll
    for (int B = 0; B < D / 64; ++B)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *reinterpret_cast<f32x4*>(&x[wave][l16][64 * B + 16 * g4 + 4 * i]) =
            f32x4{acc[4 * B][i], acc[4 * B + 1][i], acc[4 * B + 2][i], acc[4 * B + 3][i]};
  }
  __device__ inline f32x4 sum(int c, int ch) const {
    f32x4 r = *reinterpret_cast<const f32x4*>(&x[0][c][ch]);
#pragma unroll
    for (int w = 1; w < BF_WAVES; ++w) r += *reinterpret_cast<const f32x4*>(&x[w][c][ch]);
    return r;
  }
};

// dQ of 16 stacked rows m = i * group + (h % group) of one (rollout, kv head): sweep over the prefix and own keys.
template <int D>
__global__ __launch_bounds__(BF_WAVES * 64, 2) void bwd_dq_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ d_out, const float* __restrict__ k_prefix,
    const float* __restrict__ v_prefix, const float* __restrict__ k_suffix, const float* __restrict__ v_suffix,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dq,
    const WorkItem* __restrict__ items, int64_t num_items, const int32_t* __restrict__ cu, int P, int Hq, int Hkv, int group,
    float scale) {
  __shared__ __attribute__((aligned(16))) Partials<D> part;
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (block >= num_items) return;
  const WorkItem it = items[block];
  const int row0 = it.row0, off_g = cu[it.g];
  const int nrows = (cu[it.g + 1] - off_g) * group;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  auto packed_row = [&](int m) { return (int64_t)(off_g + m / group) * Hq + it.c * group + m % group; };
  const int m = min(row0 + l16, nrows - 1);  // rows past the end repeat the last one and are not written
  const int pos = m / group;
  const int64_t row = packed_row(m);
  Col<D> Q, dO;
  Q.load(q + row * D, g4);
  dO.load(d_out + row * D, g4);
  const float l = lse[row], dl = delta[row];
  const int nown = (min(row0 + 16, nrows) - 1) / group + 1;
  const int np = (P + 15) / 16, nb = np + (nown + 15) / 16;
  const int diagonal = np + (row0 / group + 1) / 16;  // own blocks from here on hold keys that some rows do not see
  const int64_t stride = (int64_t)Hkv * D;
  bool bad = false;  // some value of the diagonal blocks is not finite

  f32x4 acc[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  Col<D> K;
  auto base = [&](const float* pre, const float* own, int b) {
    return (b < np ? pre : own + off_g * stride) + (int64_t)it.c * D;
  };
  auto key_of = [&](int b, int r) {  // clamped: what a key past the end gives is masked
    return b < np ? min(b * 16 + r, P - 1) : min((b - np) * 16 + r, nown - 1);
  };
  if (wave < nb) K.load(base(k_prefix, k_suffix, wave) + key_of(wave, l16) * stride, g4);
  for (int b = wave; b < nb; b += BF_WAVES) {
    Col<D> V;
    V.load(base(v_prefix, v_suffix, b) + key_of(b, l16) * stride, g4);
    const f32x4 S = dot16<D>(K, Q);
    Rows<D> KR;
    const int keys[4] = {key_of(b, 4 * g4), key_of(b, 4 * g4 + 1), key_of(b, 4 * g4 + 2), key_of(b, 4 * g4 + 3)};
    KR.load(base(k_prefix, k_suffix, b), keys, stride, l16);
    const f32x4 W = dot16<D>(V, dO);
    const int next = b + BF_WAVES;
    if (next < nb) K.load(base(k_prefix, k_suffix, next) + key_of(next, l16) * stride, g4);
    const int key0 = (b < np ? b : b - np) * 16 + 4 * g4, limit = b < np ? P - 1 : pos;
    f32x4 ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) ds[i] = key0 + i <= limit ? expf(scale * S[i] - l) * (W[i] - dl) : 0.f;
    const int there = b < np ? P - b * 16 : nown - (b - np) * 16;  // keys that exist in the block
    if (there < 16) clear_rows_from(KR.x, there, g4);
    if (b >= diagonal && clear_bad(KR.x)) bad = true;
    outer16<D>(acc, KR, ds);
  }
  if (bad)  // the values that were cleared, for the rows that see them
    for (int b = wave; b < nb; b += BF_WAVES) {
      if (b < diagonal) continue;
      const int key0 = (b - np) * 16;
      Col<D> V;
      K.load(base(k_prefix, k_suffix, b) + key_of(b, l16) * stride, g4);
      V.load(base(v_prefix, v_suffix, b) + key_of(b, l16) * stride, g4);
      const f32x4 S = dot16<D>(K, Q), W = dot16<D>(V, dO);
      f32x4 ds;
#pragma unroll
      for (int i = 0; i < 4; ++i) ds[i] = expf(scale * S[i] - l) * (W[i] - dl);
      add_bad<D>(acc, ds, min(16, nown - key0), lane, [&](int r) { return key0 + r <= pos; },
                 [&](int r) { return base(k_prefix, k_suffix, b) + (key0 + r) * stride; });
    }
  part.put(acc, wave, l16, g4);
  __syncthreads();
  for (int n = threadIdx.x; n < 16 * (D / 4); n += BF_WAVES * 64) {
    const int r = n / (D / 4), ch = n % (D / 4) * 4;
    if (row0 + r < nrows) *reinterpret_cast<f32x4*>(dq + packed_row(row0 + r) * D + ch) = scale * part.sum(r, ch);
  }
}

// dK, dV of 16 keys of one kv head: workgroups first over the blocks of prefix keys, then over every rollout's own keys.
// The streamed rows of a prefix key are all stacked rows M = t * group + j of the kv head, of an own key those of its
// rollout from its position on.
template <int D>
__global__ __launch_bounds__(BF_WAVES * 64, 2) void bwd_dkv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ d_out, const float* __restrict__ k_prefix,
    const float* __restrict__ v_prefix, const float* __restrict__ k_suffix, const float* __restrict__ v_suffix,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dk_prefix,
    float* __restrict__ dv_prefix, float* __restrict__ dk_suffix, float* __restrict__ dv_suffix,
    const int32_t* __restrict__ cu, int G, int T, int P, int Hq, int Hkv, int group, float scale) {
  __shared__ __attribute__((aligned(16))) Partials<D> part;
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int np = (P + 15) / 16;
  if (block >= ((int64_t)np + T / 16 + G) * Hkv) return;
  const int c = (int)(block % Hkv);
  int kb = (int)(block / Hkv), g = -1, off_g = 0, nkeys = P, t_end = T;
  if (kb >= np) {
    // which rollout the block of own keys belongs to: rollout g owns the blocks from cu[g] / 16 + g on, enough for its
    // keys with at most one block too many (found by bisection; a walk over the rollouts, 10,000 of one token and 100 prefix
    // keys, took 40 of the 51 ms of a backward pass)
    kb -= np;
    g = 0;
    for (int end = G; end - g > 1;) {
      const int mid = (g + end) / 2;
      if (cu[mid] / 16 + mid <= kb) g = mid; else end = mid;
    }
    off_g = cu[g];
    t_end = cu[g + 1];
    nkeys = t_end - off_g;
    kb -= off_g / 16 + g;
    if (kb * 16 >= nkeys) return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int64_t stride = (int64_t)Hkv * D;
  const int64_t first = ((int64_t)(g < 0 ? 0 : off_g) * Hkv + c) * D;
  const int key0 = kb * 16, key = min(key0 + l16, nkeys - 1);
  Col<D> K, V;
  K.load((g < 0 ? k_prefix : k_suffix) + first + key * stride, g4);
  V.load((g < 0 ? v_prefix : v_suffix) + first + key * stride, g4);
  const int m_key = g < 0 ? 0 : (off_g + key) * group;              // first stacked row that sees this lane's key
  const int m0 = g < 0 ? 0 : (off_g + key0) * group, m1 = t_end * group;
  const int m_all = g < 0 ? 0 : (off_g + min(key0 + 15, nkeys - 1)) * group;  // rows from here on see every key
  bool bad = false;  // some value of the rows before is not finite

  f32x4 dK[D / 16], dV[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) dK[b] = dV[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto packed_row = [&](int m) { m = min(m, m1 - 1); return (m / group) * Hq + c * group + m % group; };  // T * Hq <= 2^31
  Col<D> Q;
  int mrow = m0 + wave * 16;
  unsigned row = mrow < m1 ? (unsigned)packed_row(mrow + l16) : 0u;
  if (mrow < m1) Q.load(q + (int64_t)row * D, g4);
  for (; mrow < m1; mrow += BF_WAVES * 16) {
    Col<D> dO;
    dO.load(d_out + (int64_t)row * D, g4);
    int rows[4];
    f32x4 l, dl;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rows[j] = __shfl((int)row, 4 * g4 + j);
      l[j] = lse[(unsigned)rows[j]];
      dl[j] = delta[(unsigned)rows[j]];
    }
    const f32x4 S = dot16<D>(Q, K);
    Rows<D> R;
    R.load(d_out, rows, D, l16);
    const f32x4 W = dot16<D>(dO, V);
    f32x4 p, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = mrow + 4 * g4 + i;
      const bool seen = m >= m_key && m < m1;
      p[i] = seen ? expf(scale * S[i] - l[i]) : 0.f;
      ds[i] = seen ? p[i] * (W[i] - dl[i]) : 0.f;
    }
    const int there = m1 - mrow;  // rows that exist
    if (there < 16) clear_rows_from(R.x, there, g4);
    if (mrow < m_all && clear_bad(R.x)) bad = true;
    Rows<D> R2;
    R2.load(q, rows, D, l16);
    outer16<D>(dV, R, p);
    const int next = mrow + BF_WAVES * 16;
    if (next < m1) {
      row = (unsigned)packed_row(next + l16);
      Q.load(q + (int64_t)row * D, g4);
    }
    if (there < 16) clear_rows_from(R2.x, there, g4);
    if (mrow < m_all && clear_bad(R2.x)) bad = true;
    outer16<D>(dK, R2, ds);
  }
  if (bad)  // the values that were cleared, for the keys that see their rows
    for (mrow = m0 + wave * 16; mrow < m_all; mrow += BF_WAVES * 16) {
      row = (unsigned)packed_row(mrow + l16);
      Col<D> dO;
      Q.load(q + (int64_t)row * D, g4);
      dO.load(d_out + (int64_t)row * D, g4);
      const f32x4 S = dot16<D>(Q, K), W = dot16<D>(dO, V);
      f32x4 p, ds;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned at = (unsigned)__shfl((int)row, 4 * g4 + i);
        p[i] = expf(scale * S[i] - lse[at]);
        ds[i] = p[i] * (W[i] - delta[at]);
      }
      auto seen = [&](int r) { return mrow + r >= m_key; };
      auto row_of = [&](const float* x) {
        return [x, row](int r) { return x + (int64_t)(unsigned)__shfl((int)row, r) * D; };
      };
      add_bad<D>(dV, p, min(16, m1 - mrow), lane, seen, row_of(d_out));
      add_bad<D>(dK, ds, min(16, m1 - mrow), lane, seen, row_of(q));
    }
  float* dk = (g < 0 ? dk_prefix : dk_suffix) + first;
  float* dv = (g < 0 ? dv_prefix : dv_suffix) + first;
  auto finish = [&](float* dst, float factor) {
    __syncthreads();
    for (int n = threadIdx.x; n < 16 * (D / 4); n += BF_WAVES * 64) {
      const int r = n / (D / 4), ch = n % (D / 4) * 4;
      if (key0 + r < nkeys) *reinterpret_cast<f32x4*>(dst + (key0 + r) * stride + ch) = factor * part.sum(r, ch);
    }
  };
  part.put(dV, wave, l16, g4);
  finish(dv, 1.0f);
  __syncthreads();
  part.put(dK, wave, l16, g4);
  finish(dk, scale);
}

const float* f(const void* p) { return static_cast<const float*>(p); }
float* fw(void* p) { return static_cast<float*>(p); }
dim3 grid_of(int64_t blocks) {
  return dim3((unsigned)std::min(blocks, MAX_GRID_X), (unsigned)((blocks + MAX_GRID_X - 1) / MAX_GRID_X));
}

}  // namespace

int launch_bwd_dq_f32(const BwdF32Args& a, void* stream) {
  if (a.num_items == 0) return 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid = grid_of(a.num_items);
#define PA_LAUNCH(DD)                                                                                           \
  bwd_dq_f32_kernel<DD><<<grid, BF_WAVES * 64, 0, s>>>(f(a.q), f(a.d_out), f(a.k_prefix), f(a.v_prefix),        \
                                                       f(a.k_suffix), f(a.v_suffix), a.lse, a.delta, fw(a.dq),  \
                                                       a.items, a.num_items, a.cu, (int)a.P, a.Hq, a.Hkv, a.group, \
                                                       a.scale)
  if (a.D == 128) PA_LAUNCH(128); else PA_LAUNCH(64);
#undef PA_LAUNCH
  return (int)hipGetLastError();
}

int launch_bwd_dkv_f32(const BwdF32Args& a, void* stream) {
  // 16-key blocks: the prefix's, and every rollout's (at most one partly filled each, see the kernel)
  const int64_t blocks = (a.P + 15) / 16 + a.T / 16 + a.G;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid = grid_of(blocks * a.Hkv);
#define PA_LAUNCH(DD)                                                                                              \
  bwd_dkv_f32_kernel<DD><<<grid, BF_WAVES * 64, 0, s>>>(f(a.q), f(a.d_out), f(a.k_prefix), f(a.v_prefix),          \
                                                        f(a.k_suffix), f(a.v_suffix), a.lse, a.delta,              \
                                                        fw(a.dk_prefix), fw(a.dv_prefix), fw(a.dk_suffix),         \
                                                        fw(a.dv_suffix), a.cu, a.G, (int)a.T, (int)a.P, a.Hq,      \
                                                        a.Hkv, a.group, a.scale)
  if (a.D == 128) PA_LAUNCH(128); else PA_LAUNCH(64);
#undef PA_LAUNCH
  return (int)hipGetLastError();
}

}  // namespace pa
