// Log-sum-exp merge of the prefix partial and the suffix partial, and the LSE export.
//
// Two attention results over disjoint key sets A and B of the same query combine as
//   LSE = ln(e^{LSE_A} + e^{LSE_B}),  O = e^{LSE_A - LSE} O_A + e^{LSE_B - LSE} O_B,
// which is exactly the softmax over A u B.  Here A = the shared video prefix (Sec. 5.1 of
// the paper: computed once, reused by all rollouts) and B = the rollout's own tokens.
// Pure streaming work: 2 fp32 partial rows in, one output row out; HBM-bound.
#include <hip/hip_runtime.h>

#include "common.h"

namespace pa {
namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One thread handles 4 consecutive channels of one row; rows are walked grid-stride.  The result is an fp32 partial (a
// whole call combines the two in the suffix pass's epilogue instead, see attn_bf16.hip).
__global__ __launch_bounds__(256) void merge_kernel(const float* __restrict__ o1, const float* __restrict__ lse1,
                                                    const float* __restrict__ o2, const float* __restrict__ lse2,
                                                    float* __restrict__ out, float* __restrict__ lse, int64_t rows,
                                                    int D, bool has_prefix) {
  const int per_row = D / 4;
  const int64_t total = rows * per_row;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
    const int64_t row = idx / per_row;
    const int ch = (int)(idx - row * per_row);
    const float l2 = lse2[row];
    float a1 = 0.f, a2 = 1.f, l = l2;
    if (has_prefix) {
      const float l1 = lse1[row];
      const float m = fmaxf(l1, l2);  // finite: every row sees at least its own key
      const float w1 = expf(l1 - m), w2 = expf(l2 - m);
      const float tot = w1 + w2;
      const float inv = 1.0f / tot;
      a1 = w1 * inv;
      a2 = w2 * inv;
      l = m + logf(tot);
    }
    f32x4 r = a2 * *reinterpret_cast<const f32x4*>(o2 + idx * 4);
    if (has_prefix) r += a1 * *reinterpret_cast<const f32x4*>(o1 + idx * 4);
    *reinterpret_cast<f32x4*>(out + idx * 4) = r;
    if (ch == 0) lse[row] = l;
  }
}

// n-way merge: one thread handles 4 consecutive channels of one (token, head) row.  Bound by reading the partials; STEP of
// them (a divisor of n) are in flight together, as non-temporal loads since nothing reads them again.  8 partials of 18,432
// tokens x 28 heads x 128 channels: 457 us one after the other, 423 us now (2.24 GB at 5.3 TB/s).  Whole calls back to back, one after
// the other -> now: 1 partial 85 -> 80 us, 2 130 -> 119, 3 179 -> 174, 4 232 -> 227, 5 288 -> 282, 6 343 -> 316, 7 398 -> 391, 8 453 -> 436,
// 10 566 -> 516, 16 897 -> 842; an odd n keeps one load in flight and gains by the non-temporal loads only.
template <bool OUT_BF16, int STEP>
__global__ __launch_bounds__(256) void merge_n_kernel(MergeNArgs a) {
  const int per_row = a.D / 4;
  const int64_t rows = a.T * a.Hq;
  const int64_t total = rows * per_row;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
    const int64_t row = idx / per_row;
    const int ch = (int)(idx - row * per_row);
    float m = -INFINITY;
    for (int i = 0; i < a.n; i += STEP)
#pragma unroll
      for (int e = 0; e < STEP; ++e) m = fmaxf(m, a.lse[i + e][row]);
    float tot = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < a.n; i += STEP) {
      f32x4 o[STEP];
#pragma unroll
      for (int e = 0; e < STEP; ++e) o[e] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(a.o[i + e] + idx * 4));
#pragma unroll
      for (int e = 0; e < STEP; ++e) {
        const float w = expf(a.lse[i + e][row] - m);  // a partial over no keys has LSE = -inf and weight 0
        tot += w;
        acc += w * o[e];
      }
    }
    const f32x4 r = acc * (1.0f / tot);
    if (OUT_BF16) {
      *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(a.out) + idx * 4) = __builtin_convertvector(r, bf16x4);
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + idx * 4) = r;
    }
    if (ch == 0) {
      const float l = m + logf(tot);
      if (a.lse_out) {
        const int64_t t = row / a.Hq, h = row - t * a.Hq;
        a.lse_out[h * a.T + t] = l;
      }
      if (a.lse_th_out) a.lse_th_out[row] = l;
    }
  }
}

// Merge of the range slots of the cut blocks: one thread handles 4 channels of one row, a workgroup 256 / (D / 4) rows of
// one block.  A call of a few blocks is bound by the latency of the loads, so the slots are taken four at a time, with all
// loads of a step in flight together and the weights rescaled when a later step holds a larger LSE (two loops over the
// slots, the LSEs first, took 8.7 us for 128 tokens of 28 heads in 6 ranges; now 4.1).
struct SlotArgs {  // what the kernel reads of MergeNArgs
  const RangeSum* sums;
  const float* o_slots;
  const float* lse_slots;
  void* out;
  float* lse_out;
  float* lse_th_out;
  int64_t T;
  int32_t Hq, group;
};
template <int D, bool OUT_BF16>
__global__ __launch_bounds__(256) void merge_slots_kernel(SlotArgs a) {
  constexpr int PER_ROW = D / 4, ROWS = 256 / PER_ROW, PARTS = ROWS_PER_ITEM / ROWS, STEP = 4;
  const RangeSum b = a.sums[blockIdx.x / PARTS];
  const int r = (blockIdx.x % PARTS) * ROWS + threadIdx.x / PER_ROW, ch = threadIdx.x % PER_ROW;
  if (r >= b.nrows) return;
  const float* lp = a.lse_slots + (int64_t)b.slot0 * ROWS_PER_ITEM + r;
  const float* op = a.o_slots + ((int64_t)b.slot0 * ROWS_PER_ITEM + r) * D + ch * 4;
  float mx = -INFINITY, tot = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < b.nslots; i0 += STEP) {
    float l[STEP];
    f32x4 o[STEP];
#pragma unroll
    for (int e = 0; e < STEP; ++e) {
      const int i = min(i0 + e, b.nslots - 1);
      l[e] = lp[i * ROWS_PER_ITEM];
      o[e] = *reinterpret_cast<const f32x4*>(op + (int64_t)i * (ROWS_PER_ITEM * D));
    }
    float top = mx;
#pragma unroll
    for (int e = 0; e < STEP; ++e) top = fmaxf(top, l[e]);
    const float ref = top == -INFINITY ? 0.f : top;  // no key that counts so far (see the range kernel): weights of 0
    const float old = expf(mx - ref);
    tot *= old;
    acc *= old;
#pragma unroll
    for (int e = 0; e < STEP; ++e) {
      if (i0 + e < b.nslots) {  // a repeated slot is left out, not weighted by 0: it may hold an infinity
        const float w = expf(l[e] - ref);
        tot += w;
        acc += w * o[e];
      }
    }
    mx = top;
  }
  const f32x4 v = acc * (1.0f / tot);
  const int m = b.row0 + r, t = b.off_g + m / a.group, h = b.c * a.group + m % a.group;
  const int64_t row = (int64_t)t * a.Hq + h;
  if (OUT_BF16) {
    *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(a.out) + row * D + ch * 4) = __builtin_convertvector(v, bf16x4);
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + row * D + ch * 4) = v;
  }
  if (ch == 0) {
    const float l = mx + logf(tot);
    if (a.lse_out) a.lse_out[h * a.T + t] = l;
    if (a.lse_th_out) a.lse_th_out[row] = l;
  }
}

// [T, Hq] -> [Hq, T]
__global__ __launch_bounds__(256) void lse_export_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                         int64_t T, int Hq) {
  const int64_t total = T * Hq;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
    const int64_t h = idx / T, t = idx - h * T;
    out[idx] = in[t * Hq + h];
  }
}

}  // namespace

int launch_merge(const MergeArgs& a, void* stream) {
  if (a.rows == 0) return 0;
  const int64_t total = a.rows * (a.D / 4);
  const int64_t want = (total + 255) / 256;
  const int blocks = (int)(want < 256 * 32 ? want : 256 * 32);
  hipStream_t s = static_cast<hipStream_t>(stream);
  merge_kernel<<<blocks, 256, 0, s>>>(a.o1, a.lse1, a.o2, a.lse2, a.out, a.lse, a.rows, a.D, a.has_prefix);
  return (int)hipGetLastError();
}

static int launch_merge_slots(const MergeNArgs& m, hipStream_t s) {
  if (m.num_sums == 0) return 0;
  const unsigned grid = (unsigned)(m.num_sums * (ROWS_PER_ITEM * m.D / 4 / 256));
  const SlotArgs a{m.sums, m.o_slots, m.lse_slots, m.out, m.lse_out, m.lse_th_out, m.T, m.Hq, m.group};
  if (m.D == 128) {
    if (m.dtype == PA_BF16) merge_slots_kernel<128, true><<<grid, 256, 0, s>>>(a);
    else merge_slots_kernel<128, false><<<grid, 256, 0, s>>>(a);
  } else {
    if (m.dtype == PA_BF16) merge_slots_kernel<64, true><<<grid, 256, 0, s>>>(a);
    else merge_slots_kernel<64, false><<<grid, 256, 0, s>>>(a);
  }
  return (int)hipGetLastError();
}

int launch_merge_n(const MergeNArgs& a, void* stream) {
  if (a.sums) return launch_merge_slots(a, static_cast<hipStream_t>(stream));
  const int64_t total = a.T * a.Hq * (a.D / 4);
  if (total == 0) return 0;
  const int64_t want = (total + 255) / 256;
  const int blocks = (int)(want < 256 * 32 ? want : 256 * 32);
  hipStream_t s = static_cast<hipStream_t>(stream);
#define PA_MERGE(STEP)                                                          \
  if (a.dtype == PA_BF16) merge_n_kernel<true, STEP><<<blocks, 256, 0, s>>>(a); \
  else merge_n_kernel<false, STEP><<<blocks, 256, 0, s>>>(a)
  if (a.n % 8 == 0) {
    PA_MERGE(8);
  } else if (a.n % 4 == 0) {
    PA_MERGE(4);
  } else if (a.n % 2 == 0) {
    PA_MERGE(2);
  } else {
    PA_MERGE(1);
  }
#undef PA_MERGE
  return (int)hipGetLastError();
}

int launch_lse_export(const float* lse_th, float* lse_ht, int64_t T, int32_t Hq, void* stream) {
  const int64_t total = T * Hq;
  if (total == 0) return 0;
  const int64_t want = (total + 255) / 256;
  const int blocks = (int)(want < 256 * 16 ? want : 256 * 16);
  lse_export_kernel<<<blocks, 256, 0, static_cast<hipStream_t>(stream)>>>(lse_th, lse_ht, T, Hq);
  return (int)hipGetLastError();
}

}  // namespace pa
