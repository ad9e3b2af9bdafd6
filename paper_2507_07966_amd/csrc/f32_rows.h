// Device helpers of the fp32 kernels for values that are not finite.  A streamed row (a key's V or K, a query's dO or q) is
// an MFMA operand for 16 columns at once, and a column that must not see the row gives it weight 0; 0 times an infinity or
// a NaN would still reach that column.  So rows past the end of their set are cleared, and in blocks that only some columns
// see (those on the causal diagonal) values that are not finite are cleared too and, if there were any, added at the end to
// the columns that see them.
#pragma once

#include <hip/hip_runtime.h>

namespace pa {
namespace f32rows {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline bool finite(float x) { return x * 0.f == 0.f; }

// x[j][B]: channels 64 B + 4 l16 .. of row 4 g4 + j.  Clears the rows from `first` on.
template <int VB>
__device__ inline void clear_rows_from(f32x4 (&x)[4][VB], int first, int g4) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (4 * g4 + j >= first) {
#pragma unroll
      for (int B = 0; B < VB; ++B) x[j][B] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// Clears the values that are not finite; true (in every lane) if the wavefront's 16 rows held one.
template <int VB>
__device__ inline bool clear_bad(f32x4 (&x)[4][VB]) {
  bool bad = false;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int B = 0; B < VB; ++B)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (!finite(x[j][B][e])) {
          bad = true;
          x[j][B][e] = 0.f;
        }
  return __any(bad);
}

// acc[4 B + e], register i: channel 64 B + 4 (4 g4 + i) + e of column l16.  Adds w_r x for every value x of row r < n that is
// not finite, where visible(r) says that this lane's column sees the row; the weights are laid out as an MFMA result (w[i]:
// row 4 g4 + i of column l16), row_of(r) points at a row in memory.
template <int D, class Visible, class RowOf>
__device__ inline void add_bad(f32x4 (&acc)[D / 16], f32x4 w, int n, int lane, Visible visible, RowOf row_of) {
  const int l16 = lane & 15, g4 = lane >> 4;
#pragma unroll 1
  for (int r = 0; r < n; ++r) {
    const float mine = (r & 2) ? ((r & 1) ? w[3] : w[2]) : ((r & 1) ? w[1] : w[0]);
    const float wr = __shfl(mine, l16 + 16 * (r >> 2));
    const bool seen = visible(r);
    const float* x = row_of(r) + 16 * g4;
#pragma unroll
    for (int B = 0; B < D / 64; ++B)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(x + 64 * B + 4 * i);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * B + e][i] += seen && !finite(v[e]) ? wr * v[e] : 0.f;
      }
  }
}

}  // namespace f32rows
}  // namespace pa
