// The decode step in one launch (decode_body.h), compiled once per entmax exponent mode
// (-DDASH_DEC_MODE=0..4, see stage1_common.h), each object providing launch_decode_route_m<MODE>.
#include "decode_body.h"

namespace dash {

#ifndef DASH_DEC_MODE
#error "compile with -DDASH_DEC_MODE=<exponent mode: 0..4>"
#endif

template <int D, bool WIDE>
static hipError_t launch_t(const DecArgs& a, unsigned grid, size_t lds, hipStream_t st) {
  auto kern = s2_decode_kernel<D, DEC_ROUTE, DASH_DEC_MODE, WIDE>;
  static LdsOptIn opt_in;
  if (hipError_t e = allow_dyn_lds((const void*)kern, lds, opt_in); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, a);
  return hipGetLastError();
}

#define DASH_CAT2(a_, b_) a_##b_
#define DASH_CAT(a_, b_) DASH_CAT2(a_, b_)

hipError_t DASH_CAT(launch_decode_route_m, DASH_DEC_MODE)(const DecArgs& a, int head_dim, unsigned grid, size_t lds, hipStream_t st) {
  if (head_dim == 128) return a.s.g_q > 4 ? launch_t<128, true>(a, grid, lds, st) : launch_t<128, false>(a, grid, lds, st);
  return a.s.g_q > 4 ? launch_t<64, true>(a, grid, lds, st) : launch_t<64, false>(a, grid, lds, st);
}

}  // namespace dash
