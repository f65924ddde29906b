// Per-call NTT kernels: plain transforms and ternary polynomials.
#include "ntt_core.h"

namespace pencil {

template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_ntt_plain(uint64_t* data, int inverse, Consts C, Tables T) {
  extern __shared__ uint64_t lds[];
  do_ntt_plain<LOGN, LOGE, F60>(lds, data, inverse, C, T, blockIdx.x);
}

template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_ntt_ternary(uint64_t* dst, uint64_t nonce, uint64_t obj_base,
                                                      uint32_t purpose, int form, int64_t count, Consts C, Tables T) {
  extern __shared__ uint64_t lds[];
  do_ntt_ternary<LOGN, LOGE, F60>(lds, dst, nonce, obj_base, purpose, form, count, C, T, blockIdx.x);
}

hipError_t launch_ntt_plain(uint64_t* data, int64_t polys, bool inverse, const Consts& C, const Tables& T,
                            hipStream_t s) {
  if (polys <= 0) return hipSuccess;
  NTT_DISPATCH(k_ntt_plain, dim3((unsigned)(polys * C.L)), C, s, data, inverse ? 1 : 0, C, T);
  return hipGetLastError();
}

hipError_t launch_ntt_ternary(uint64_t* dst, int64_t count, uint64_t nonce, uint64_t obj_base, uint32_t purpose, int form,
                              const Consts& C, const Tables& T, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  NTT_DISPATCH(k_ntt_ternary, dim3((unsigned)(count * C.L)), C, s, dst, nonce, obj_base, purpose, form, count, C, T);
  return hipGetLastError();
}

hipError_t configure_lds_ntt() {
  const int max_lds = 160 * 1024;
  hipError_t e = hipSuccess;
#define PENCIL_RAISE(LN, LE, F)                                                                            \
  for (const void* f : {(const void*)k_ntt_plain<LN, LE, F>, (const void*)k_ntt_ternary<LN, LE, F>}) {            \
    hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);         \
    if (r != hipSuccess) e = r;                                                                          \
  }
  PENCIL_RAISE(13, 4, false)
  PENCIL_RAISE(13, 4, true)
  PENCIL_RAISE(13, 5, false)
  PENCIL_RAISE(13, 5, true)
  PENCIL_RAISE(14, 4, false)
  PENCIL_RAISE(14, 4, true)
  PENCIL_RAISE(14, 5, false)
  PENCIL_RAISE(14, 5, true)
#undef PENCIL_RAISE
  return e;
}

}  // namespace pencil
