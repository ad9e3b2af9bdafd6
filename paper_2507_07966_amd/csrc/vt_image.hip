// Layout pre-pass of the bf16 forward: the V^T tile images of vt_image.h.
#include <hip/hip_runtime.h>

#include "vt_image.h"

namespace pa {
namespace {

template <int D>
__global__ __launch_bounds__(256) void vt_image_kernel(const unsigned short* __restrict__ v_prefix,
                                                       const unsigned short* __restrict__ v_suffix,
                                                       unsigned short* __restrict__ vt_prefix,
                                                       unsigned short* __restrict__ vt_suffix,
                                                       const int32_t* __restrict__ cu,
                                                       const int32_t* __restrict__ vt_off, int64_t P, int tiles_prefix,
                                                       int tiles_suffix, int G, int Hkv) {
  __shared__ vt::ImageTile<D> tile;
  vt::make_image<D, false>(tile.t, blockIdx.x, v_prefix, v_suffix, vt_prefix, vt_suffix, cu, vt_off, P, tiles_prefix,
                           tiles_suffix, G, Hkv);
}

}  // namespace

int launch_vt_images(const VtArgs& a, void* stream) {
  const int64_t blocks = (int64_t)a.Hkv * (a.tiles_prefix + a.tiles_suffix);
  if (blocks == 0) return 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto vp = static_cast<const unsigned short*>(a.v_prefix);
  auto vs = static_cast<const unsigned short*>(a.v_suffix);
  auto tp = static_cast<unsigned short*>(a.vt_prefix);
  auto ts = static_cast<unsigned short*>(a.vt_suffix);
#define PA_VT(DD)                                                                                            \
  vt_image_kernel<DD><<<(unsigned)blocks, 256, 0, s>>>(vp, vs, tp, ts, a.cu, a.vt_off, a.P, a.tiles_prefix, \
                                                       a.tiles_suffix, a.G, a.Hkv)
  if (a.D == 128) PA_VT(128); else PA_VT(64);
#undef PA_VT
  return (int)hipGetLastError();
}

}  // namespace pa
