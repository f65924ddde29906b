// Batched step: every forward and inverse NTT of a step's products, one
// launch per ring degree, over a device-side segment table.
#include "ntt_core.h"

namespace pencil {

// Every NTT of one phase, for one ring degree: the forward transforms of the
// inputs (k_step_ntt: ciphertexts, plaintexts, re-randomisation masks) or the
// inverse transforms of the outputs (k_step_intt).
template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE)
    k_step_ntt(const StepSeg* __restrict__ segs, int nseg, const Consts* __restrict__ consts,
               const Tables* __restrict__ tabs, const uint64_t* __restrict__ nonce) {
  extern __shared__ uint64_t lds[];
  const StepSeg& S = segs[find_seg(segs, nseg, blockIdx.x)];
  const Consts& C = consts[S.ctx];
  const Tables& T = tabs[S.ctx];
  const int64_t p = (int64_t)blockIdx.x - S.block_begin;
  switch (S.kind) {
    case SEG_CT: do_ntt_ct<LOGN, LOGE, F60>(lds, S.src, S.dst, S.count, S.tensor, S.G, S.V, C, T, p); break;
    case SEG_PT: do_ntt_pt<LOGN, LOGE, F60>(lds, S.tensor, S.dst, S.count, S.side, S.G, S.V, C, T, p); break;
    case SEG_TERN: do_ntt_ternary<LOGN, LOGE, F60>(lds, S.dst, *nonce + S.nonce_off, S.obj_base, S.purpose, S.V.form, S.count, C, T, p); break;
    default: break;
  }
}

// The forward transforms of one product (per-call path).  One launch: at the
// smallest layers each of the two to four launches it replaces took 11-15 us, one
// after the other, for a few polynomials.
template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_call_ntt(const NttCall A) {
  extern __shared__ uint64_t lds[];
  const int64_t b = blockIdx.x;
  int i = 0;
#pragma unroll
  for (int k = 0; k < kNttSegs - 1; ++k) i += b >= A.seg[k].block_end ? 1 : 0;
  const NttSeg& S = A.seg[i];
  const int64_t p = b - (i ? A.seg[i - 1].block_end : 0);
  switch (S.kind) {
    case SEG_CT:
      do_ntt_ct<LOGN, LOGE, F60>(lds, S.src, S.dst, S.count, S.tensor, A.G, S.V, A.C, A.T, p);
      break;
    case SEG_PT:
      do_ntt_pt<LOGN, LOGE, F60>(lds, S.tensor, S.dst, S.count, S.side, A.G, S.V, A.C, A.T, p);
      break;
    default:
      do_ntt_ternary<LOGN, LOGE, F60>(lds, S.dst, A.nonce, S.obj_base, S.purpose, S.V.form, S.count, A.C, A.T, p);
      break;
  }
}

template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE)
    k_step_intt(const StepSeg* __restrict__ segs, int nseg, const Consts* __restrict__ consts,
                const Tables* __restrict__ tabs) {
  extern __shared__ uint64_t lds[];
  const StepSeg& S = segs[find_seg(segs, nseg, blockIdx.x)];
  const int64_t p = (int64_t)blockIdx.x - S.block_begin;
  do_ntt_plain<LOGN, LOGE, F60>(lds, S.dst, 1, consts[S.ctx], tabs[S.ctx], p);
}

hipError_t launch_step_ntt(int log2n, int width, bool inverse, const StepPhase& P, int64_t blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  Consts C{};  // only log2n, n, ntt_loge and fold60 are read by the dispatch
  C.log2n = log2n;
  C.n = 1 << log2n;
  C.ntt_loge = width % 8;
  C.fold60 = width >= 8;
  const dim3 grid((unsigned)blocks);
  if (P.call)
    NTT_DISPATCH(k_call_ntt, grid, C, s, *P.call);
  else if (inverse)
    NTT_DISPATCH(k_step_intt, grid, C, s, P.segs, P.nseg, P.consts, P.tabs);
  else
    NTT_DISPATCH(k_step_ntt, grid, C, s, P.segs, P.nseg, P.consts, P.tabs, P.nonce);
  return hipGetLastError();
}

hipError_t configure_lds_step() {
  const int max_lds = 160 * 1024;
  hipError_t e = hipSuccess;
#define PENCIL_RAISE(LN, LE, F)                                                                            \
  for (const void* f : {(const void*)k_step_ntt<LN, LE, F>, (const void*)k_step_intt<LN, LE, F>,                \
                        (const void*)k_call_ntt<LN, LE, F>}) {           \
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
