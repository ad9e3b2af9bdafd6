// Backward in fp32 (exact checks, gradient checks, small debugging runs) with fp32 MFMAs (v_mfma_f32_16x16x4_f32):
// a query-stationary kernel for dQ and a key-stationary one for dK and dV, no atomics, fixed summation order.
//   W_j = exp(scale <q, k_j> - LSE),  dS_j = W_j (<dO, v_j> - delta),
//   dQ = scale sum_j dS_j k_j,  dK_j = scale sum_rows dS_j q,  dV_j = sum_rows W_j dO,
// a prefix key summing over the rows of all rollouts (paper Sec. 5.1: shared video prefix).
//
// What bounds it: at these sizes latency, then the fp32 matrix rate.  Both kernels keep 16 columns (query rows, keys)
// per workgroup and deal the streamed side out to 8 wavefronts 16 rows at a time, so even a few hundred rows or keys give
// every CU work; the 8 partial sums are added through LDS at the end.  A streamed row is used twice: with lane (row l16,
// channel quarter g4) as operand of the products over channels, and with lane (row 4 g4 + j, channels 4 l16 ..) as operand
// of the products over rows, where the accumulator of the first product (rows 4 g4 + i of column l16) is the B operand of
// step j = i without any data movement.
// The rows travel global -> LDS with direct 16-byte loads, whole rows at a time, into a region of the wavefront's own (no
// barrier), and both operands are read from there.  (Loaded straight into registers, the first operand has 16 consecutive
// lanes on 16 rows, 16 bytes each: the address unit took about 64 cycles per load, as long as all the MFMAs, and every row was fetched
// twice.)
// Measured, 8 / 2 heads of 128 channels, 900 tokens over 1,000 + 179..289 keys: dQ 105 us with the loads into registers, 90 now
// (73 TFLOP/s); dK/dV 178 -> 147 us, and 110 + 5 us with its few long blocks cut into ranges of rows (61 TFLOP/s).  The matrix
// pipe is then busy 55 % of the cycles (dQ: 51 %): about 80 % inside the loops (a step, by blocks of different length, takes 4.6 ... 5.0 us
// for 8,192 MFMA cycles a SIMD at 2.1 GHz, dQ 3.7 us for 6,144), the rest is the start and end of two items a CU and the uneven third.
// (4 wavefronts a workgroup, two workgroups a CU: 87 and 101 us here, but half the wavefronts where blocks are few.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bwd.h"
#include "f32_rows.h"
#include "mfma_tiles.h"

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
};
// 16 streamed rows in LDS, owned by one wavefront: chunk ch (4 channels) of row r at chunk position ch ^ r of its row, so that both
// operand reads spread over all banks.
template <int D>
struct Staged {
  static constexpr int CHUNKS = D / 4, ROWS_PER_LOAD = 64 / CHUNKS, LOADS = 16 / ROWS_PER_LOAD;
  float x[16][D];
  // Load n brings rows row(n, lane) = n * ROWS_PER_LOAD + ...; this lane's part of it is channels channel(n, lane) .. + 3.
  static __device__ inline int row(int n, int lane) { return n * ROWS_PER_LOAD + lane / CHUNKS; }
  static __device__ inline int channel(int n, int lane) { return (lane % CHUNKS ^ row(n, lane)) * 4; }
  // from(n): this lane's source of load n.  What was read from here before has to be in registers (drained()).
  template <class From>
  __device__ inline void issue(From from) {
#pragma unroll
    for (int n = 0; n < LOADS; ++n) mt::load16_to_lds(from(n), reinterpret_cast<unsigned char*>(x) + n * 1024);
  }
  __device__ inline f32x4 col(int s, int l16, int g4) const {
    return *reinterpret_cast<const f32x4*>(&x[l16][((4 * s + g4) ^ l16) * 4]);
  }
  __device__ inline void rows(Rows<D>& out, int l16, int g4) const {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int B = 0; B < D / 64; ++B)
        out.x[j][B] = *reinterpret_cast<const f32x4*>(&x[4 * g4 + j][((16 * B + l16) ^ (4 * g4 + j)) * 4]);
  }
};
// The wavefront's loads have landed / its LDS reads are in registers; nothing is moved across.
__device__ inline void landed() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}
__device__ inline void drained() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  asm volatile("" ::: "memory");
}
// [16 streamed rows] x [16 columns] over all channels; two accumulation chains
template <int D, class Operand>
__device__ inline f32x4 dot16(Operand a, const Col<D>& b) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const f32x4 x = a(s);
    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], b.x[s][0], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1], b.x[s][1], s1, 0, 0, 0);
    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2], b.x[s][2], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[3], b.x[s][3], s1, 0, 0, 0);
  }
  return s0 + s1;
}
template <int D>
__device__ inline f32x4 dot16(const Col<D>& a, const Col<D>& b) {
  return dot16<D>([&](int s) { return a.x[s]; }, b);
}
template <int D>
__device__ inline f32x4 dot16(const Staged<D>& a, const Col<D>& b, int l16, int g4) {
  return dot16<D>([&](int s) { return a.col(s, l16, g4); }, b);
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

// Sum of the wavefronts' accumulators: LDS [wavefront][column][D], padded rows; column c, channels ch .. ch + 3.  Takes the
// place of the staged rows once every wavefront is done with them.
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

template <int D>
union Shared {
  Staged<D> staged[BF_WAVES][2];
  Partials<D> part;
};

// dQ of 16 stacked rows m = i * group + (h % group) of one (rollout, kv head): sweep over the prefix and own keys.  CUT (a
// launch of few blocks): an item with a slot (it.split >= 0) sweeps the 16-key blocks [key0, key0 + nkeys) of that sequence
// only and leaves its unscaled sum in the slot (16 rows each); bwd_f32_sum_kernel adds a block's slots.
template <int D, bool CUT>
__global__ __launch_bounds__(BF_WAVES * 64, 2) void bwd_dq_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ d_out, const float* __restrict__ k_prefix,
    const float* __restrict__ v_prefix, const float* __restrict__ k_suffix, const float* __restrict__ v_suffix,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dq, float* __restrict__ partial,
    const WorkItem* __restrict__ items, int64_t num_items, const int32_t* __restrict__ cu, int P, int Hq, int Hkv, int group,
    float scale) {
  __shared__ __attribute__((aligned(1024))) Shared<D> lds;
  Partials<D>& part = lds.part;
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
  const int np = (P + 15) / 16;
  const bool part_of = CUT && it.split >= 0;
  const int b_first = part_of ? it.key0 : 0, nb = part_of ? it.key0 + it.nkeys : np + (nown + 15) / 16;
  const int diagonal = np + (row0 / group + 1) / 16;  // own blocks from here on hold keys that some rows do not see
  const int64_t stride = (int64_t)Hkv * D;
  bool bad = false;  // some value of the diagonal blocks is not finite

  f32x4 acc[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  Staged<D>&K = lds.staged[wave][0], &V = lds.staged[wave][1];
  auto base = [&](const float* pre, const float* own, int b) {
    return (b < np ? pre : own + off_g * stride) + (int64_t)it.c * D;
  };
  auto key_of = [&](int b, int r) {  // clamped: what a key past the end gives is masked
    return b < np ? min(b * 16 + r, P - 1) : min((b - np) * 16 + r, nown - 1);
  };
  int64_t lane_off[Staged<D>::LOADS];  // of this lane's parts inside a block of 16 keys that all exist
#pragma unroll
  for (int n = 0; n < Staged<D>::LOADS; ++n) lane_off[n] = Staged<D>::row(n, lane) * stride + Staged<D>::channel(n, lane);
  auto issue = [&](Staged<D>& dst, const float* pre, const float* own, int b) {
    const float* p = base(pre, own, b);
    if (b < np ? b * 16 + 16 <= P : (b - np) * 16 + 16 <= nown) {
      p += (b < np ? b : b - np) * 16 * stride;
      dst.issue([&](int n) { return p + lane_off[n]; });
    } else {
      dst.issue([&](int n) { return p + key_of(b, Staged<D>::row(n, lane)) * stride + Staged<D>::channel(n, lane); });
    }
  };
  const int b_wave = b_first + wave;
  if (b_wave < nb) {
    issue(K, k_prefix, k_suffix, b_wave);
    issue(V, v_prefix, v_suffix, b_wave);
  }
  for (int b = b_wave; b < nb; b += BF_WAVES) {
    const int next = b + BF_WAVES;
    landed();
    const f32x4 W = dot16<D>(V, dO, l16, g4);
    drained();
    if (next < nb) issue(V, v_prefix, v_suffix, next);
    const f32x4 S = dot16<D>(K, Q, l16, g4);
    Rows<D> KR;
    K.rows(KR, l16, g4);
    drained();
    if (next < nb) issue(K, k_prefix, k_suffix, next);
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
    for (int b = b_wave; b < nb; b += BF_WAVES) {
      if (b < diagonal) continue;
      const int key0 = (b - np) * 16;
      Col<D> KC, VC;
      KC.load(base(k_prefix, k_suffix, b) + key_of(b, l16) * stride, g4);
      VC.load(base(v_prefix, v_suffix, b) + key_of(b, l16) * stride, g4);
      const f32x4 S = dot16<D>(KC, Q), W = dot16<D>(VC, dO);
      f32x4 ds;
#pragma unroll
      for (int i = 0; i < 4; ++i) ds[i] = expf(scale * S[i] - l) * (W[i] - dl);
      add_bad<D>(acc, ds, min(16, nown - key0), lane, [&](int r) { return key0 + r <= pos; },
                 [&](int r) { return base(k_prefix, k_suffix, b) + (key0 + r) * stride; });
    }
  __syncthreads();  // no wavefront reads staged rows any more
  part.put(acc, wave, l16, g4);
  __syncthreads();
  for (int n = threadIdx.x; n < 16 * (D / 4); n += BF_WAVES * 64) {
    const int r = n / (D / 4), ch = n % (D / 4) * 4;
    if (part_of) *reinterpret_cast<f32x4*>(partial + ((int64_t)it.split * 16 + r) * D + ch) = part.sum(r, ch);
    else if (row0 + r < nrows) *reinterpret_cast<f32x4*>(dq + packed_row(row0 + r) * D + ch) = scale * part.sum(r, ch);
  }
}

// dK, dV of 16 keys of one kv head: workgroups first over the blocks of prefix keys, then over every rollout's own keys.
// The streamed rows of a prefix key are all stacked rows M = t * group + j of the kv head, of an own key those of its
// rollout from its position on.  CUT (a launch of few blocks): the workgroups run a list instead, whose items stream the
// stacked rows [tile0, tile1); one with a slot leaves its unscaled sums there ([2][16 keys][D]: dK, dV).
template <int D, bool CUT>
__global__ __launch_bounds__(BF_WAVES * 64, 2) void bwd_dkv_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ d_out, const float* __restrict__ k_prefix,
    const float* __restrict__ v_prefix, const float* __restrict__ k_suffix, const float* __restrict__ v_suffix,
    const float* __restrict__ lse, const float* __restrict__ delta, float* __restrict__ dk_prefix,
    float* __restrict__ dv_prefix, float* __restrict__ dk_suffix, float* __restrict__ dv_suffix,
    float* __restrict__ partial, const KeyItem* __restrict__ items, int64_t num_items,
    const int32_t* __restrict__ cu, int G, int T, int P, int Hq, int Hkv, int group, float scale) {
  __shared__ __attribute__((aligned(1024))) Shared<D> lds;
  Partials<D>& part = lds.part;
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int np = (P + 15) / 16;
  if (block >= (CUT ? num_items : ((int64_t)np + T / 16 + G) * Hkv)) return;
  KeyItem it{};
  if (CUT) it = items[block];
  const int c = CUT ? it.c : (int)(block % Hkv);
  int kb = CUT ? it.key0 / 16 : (int)(block / Hkv), g = CUT ? it.g : -1, off_g = 0, nkeys = P, t_end = T;
  if (CUT) {
    if (g >= 0) {
      off_g = cu[g];
      t_end = cu[g + 1];
      nkeys = t_end - off_g;
    }
  } else if (kb >= np) {
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
  const int r0 = CUT ? it.tile0 : m0, r1 = CUT ? it.tile1 : m1;  // the rows streamed here
  const int m_all = g < 0 ? 0 : (off_g + min(key0 + 15, nkeys - 1)) * group;  // rows from here on see every key
  bool bad = false;  // some value of the rows before is not finite

  f32x4 dK[D / 16], dV[D / 16];
#pragma unroll
  for (int b = 0; b < D / 16; ++b) dK[b] = dV[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto packed_row = [&](int m) { m = min(m, m1 - 1); return (m / group) * Hq + c * group + m % group; };  // T * Hq <= 2^31
  Staged<D>&Q = lds.staged[wave][0], &dO = lds.staged[wave][1];
  int mrow = r0 + wave * 16;
  // of the block in flight: packed row of its stacked row l16, that row's LSE and delta, this lane's parts of the rows
  unsigned row = 0u;
  float l_row = 0.f, dl_row = 0.f;
  int64_t lane_off[Staged<D>::LOADS];
  auto locate = [&](int m) {
    row = (unsigned)packed_row(m + l16);
    unsigned of[Staged<D>::LOADS];
#pragma unroll
    for (int n = 0; n < Staged<D>::LOADS; ++n) of[n] = (unsigned)__shfl((int)row, Staged<D>::row(n, lane));
    l_row = lse[row];
    dl_row = delta[row];
#pragma unroll
    for (int n = 0; n < Staged<D>::LOADS; ++n) lane_off[n] = (int64_t)of[n] * D + Staged<D>::channel(n, lane);
  };
  auto issue = [&](Staged<D>& dst, const float* x) {
    dst.issue([&](int n) { return x + lane_off[n]; });
  };
  if (mrow < r1) {
    locate(mrow);
    issue(Q, q);
    issue(dO, d_out);
  }
  for (; mrow < r1; mrow += BF_WAVES * 16) {
    landed();
    f32x4 l, dl;  // of rows 4 g4 ..
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      l[i] = __shfl(l_row, 4 * g4 + i);
      dl[i] = __shfl(dl_row, 4 * g4 + i);
    }
    const f32x4 S = dot16<D>(Q, K, l16, g4);
    const f32x4 W = dot16<D>(dO, V, l16, g4);
    Rows<D> R;
    dO.rows(R, l16, g4);
    f32x4 p, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = mrow + 4 * g4 + i;
      const bool seen = m >= m_key && m < m1;
      p[i] = seen ? expf(scale * S[i] - l[i]) : 0.f;
      ds[i] = seen ? p[i] * (W[i] - dl[i]) : 0.f;
    }
    const int there = m1 - mrow;  // rows that exist
    drained();
    const int next = mrow + BF_WAVES * 16;
    if (next < r1) {
      locate(next);
      issue(dO, d_out);
    }
    if (there < 16) clear_rows_from(R.x, there, g4);
    if (mrow < m_all && clear_bad(R.x)) bad = true;
    outer16<D>(dV, R, p);
    Q.rows(R, l16, g4);
    drained();
    if (next < r1) issue(Q, q);
    if (there < 16) clear_rows_from(R.x, there, g4);
    if (mrow < m_all && clear_bad(R.x)) bad = true;
    outer16<D>(dK, R, ds);
  }
  if (bad)  // the values that were cleared, for the keys that see their rows
    for (mrow = r0 + wave * 16; mrow < min(m_all, r1); mrow += BF_WAVES * 16) {
      row = (unsigned)packed_row(mrow + l16);
      Col<D> QC, dOC;
      QC.load(q + (int64_t)row * D, g4);
      dOC.load(d_out + (int64_t)row * D, g4);
      const f32x4 S = dot16<D>(QC, K), W = dot16<D>(dOC, V);
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
  auto finish = [&](float* dst, float* slot, float factor) {
    __syncthreads();
    for (int n = threadIdx.x; n < 16 * (D / 4); n += BF_WAVES * 64) {
      const int r = n / (D / 4), ch = n % (D / 4) * 4;
      if (CUT && it.slot >= 0) *reinterpret_cast<f32x4*>(slot + r * D + ch) = part.sum(r, ch);
      else if (key0 + r < nkeys) *reinterpret_cast<f32x4*>(dst + (key0 + r) * stride + ch) = factor * part.sum(r, ch);
    }
  };
  float* slot = CUT ? partial + (int64_t)it.slot * (2 * 16 * D) : nullptr;
  __syncthreads();  // no wavefront reads staged rows any more
  part.put(dV, wave, l16, g4);
  finish(dv, slot + 16 * D, 1.0f);
  __syncthreads();
  part.put(dK, wave, l16, g4);
  finish(dk, slot, scale);
}

// Adds the slots of cut blocks, in their order: workgroups first over the blocks of rows (dQ), then over the blocks of keys.
template <int D>
__global__ __launch_bounds__(256) void bwd_f32_sum_kernel(
    const float* __restrict__ dq_partial, const float* __restrict__ key_partial, const RangeSum* __restrict__ dq_sums,
    const KeySum* __restrict__ key_sums, int num_dq_sums, float* __restrict__ dq, float* __restrict__ dk_prefix,
    float* __restrict__ dv_prefix, float* __restrict__ dk_suffix, float* __restrict__ dv_suffix, int Hq, int Hkv, int group,
    float scale) {
  constexpr int PER_ROW = D / 4, SLOT = 16 * D;
  auto sum = [](const float* p, int n, int64_t step) {
    f32x4 acc = *reinterpret_cast<const f32x4*>(p);
#pragma unroll 4
    for (int i = 1; i < n; ++i) acc += *reinterpret_cast<const f32x4*>(p + i * step);
    return acc;
  };
  if ((int)blockIdx.x < num_dq_sums) {
    const RangeSum s = dq_sums[blockIdx.x];
    for (int n = threadIdx.x; n < s.nrows * PER_ROW; n += 256) {
      const int m = s.row0 + n / PER_ROW, ch = n % PER_ROW * 4;
      const int64_t row = (int64_t)(s.off_g + m / group) * Hq + s.c * group + m % group;
      *reinterpret_cast<f32x4*>(dq + row * D + ch) = scale * sum(dq_partial + (int64_t)s.slot0 * SLOT + n * 4, s.nslots, SLOT);
    }
    return;
  }
  const KeySum s = key_sums[blockIdx.x - num_dq_sums];
  float* dk = s.own ? dk_suffix : dk_prefix;
  float* dv = s.own ? dv_suffix : dv_prefix;
  const float* p = key_partial + (int64_t)s.slot0 * (2 * SLOT);
  for (int n = threadIdx.x; n < s.nkeys * PER_ROW; n += 256) {
    const int64_t at = ((int64_t)(s.key0 + n / PER_ROW) * Hkv + s.c) * D + n % PER_ROW * 4;
    *reinterpret_cast<f32x4*>(dk + at) = scale * sum(p + n * 4, s.nslots, 2 * SLOT);
    *reinterpret_cast<f32x4*>(dv + at) = sum(p + SLOT + n * 4, s.nslots, 2 * SLOT);
  }
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
#define PA_LAUNCH(DD, CC)                                                                                       \
  bwd_dq_f32_kernel<DD, CC><<<grid, BF_WAVES * 64, 0, s>>>(f(a.q), f(a.d_out), f(a.k_prefix), f(a.v_prefix),    \
                                                           f(a.k_suffix), f(a.v_suffix), a.lse, a.delta, fw(a.dq), \
                                                           a.dq_partial, a.items, a.num_items, a.cu, (int)a.P, a.Hq, \
                                                           a.Hkv, a.group, a.scale)
  if (a.D == 128) {
    if (a.num_dq_sums) PA_LAUNCH(128, true); else PA_LAUNCH(128, false);
  } else {
    if (a.num_dq_sums) PA_LAUNCH(64, true); else PA_LAUNCH(64, false);
  }
#undef PA_LAUNCH
  return (int)hipGetLastError();
}

int launch_bwd_dkv_f32(const BwdF32Args& a, void* stream) {
  // 16-key blocks: the prefix's, and every rollout's (at most one partly filled each, see the kernel)
  const int64_t blocks = (a.P + 15) / 16 + a.T / 16 + a.G;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool cut = a.num_key_items > 0;
  const dim3 grid = grid_of(cut ? a.num_key_items : blocks * a.Hkv);
#define PA_LAUNCH(DD, CC)                                                                                          \
  bwd_dkv_f32_kernel<DD, CC><<<grid, BF_WAVES * 64, 0, s>>>(f(a.q), f(a.d_out), f(a.k_prefix), f(a.v_prefix),      \
                                                            f(a.k_suffix), f(a.v_suffix), a.lse, a.delta,          \
                                                            fw(a.dk_prefix), fw(a.dv_prefix), fw(a.dk_suffix),     \
                                                            fw(a.dv_suffix), a.key_partial, a.key_items,           \
                                                            a.num_key_items, a.cu, a.G, (int)a.T, (int)a.P, a.Hq,  \
                                                            a.Hkv, a.group, a.scale)
  if (a.D == 128) {
    if (cut) PA_LAUNCH(128, true); else PA_LAUNCH(128, false);
  } else {
    if (cut) PA_LAUNCH(64, true); else PA_LAUNCH(64, false);
  }
#undef PA_LAUNCH
  if (hipGetLastError() != hipSuccess) return 1;
  const int64_t sums = a.num_dq_sums + a.num_key_sums;  // those of dQ, launched before, too
  if (sums == 0) return 0;
#define PA_LAUNCH(DD)                                                                                            \
  bwd_f32_sum_kernel<DD><<<(unsigned)sums, 256, 0, s>>>(a.dq_partial, a.key_partial, a.dq_sums, a.key_sums,      \
                                                        (int)a.num_dq_sums, fw(a.dq), fw(a.dk_prefix),           \
                                                        fw(a.dv_prefix), fw(a.dk_suffix), fw(a.dv_suffix), a.Hq, \
                                                        a.Hkv, a.group, a.scale)
  if (a.D == 128) PA_LAUNCH(128); else PA_LAUNCH(64);
#undef PA_LAUNCH
  return (int)hipGetLastError();
}

}  // namespace pa
