// The data owner's ends: public-key encryption in the NTT domain, the
// decryption phase and exact-CRT decode, and key generation.
#include "ntt_core.h"

namespace pencil {

// Encryption in the NTT domain: ct_c = pk_c * u + NTT(e_c (+ round(q m / t) on
// c = 0)), with m the encoded share at each slot, each residue stored in the
// multiply-accumulate's split form; the product path consumes ciphertexts in
// this form.  Grid: n_ct * 2 * L, u_ntt is [n][L][N].
template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_encrypt(const uint64_t* u_ntt, const int64_t* share, uint64_t* ct, int side,
                                                  Geo G, View V, const uint64_t* pk_ntt, const uint64_t* pk_sh,
                                                  uint64_t nonce, uint64_t obj_base, Consts C, Tables T) {
  extern __shared__ uint64_t lds[];
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int64_t p = blockIdx.x;
  const int l = (int)(p % L);
  const int c = (int)((p / L) % 2);
  const int64_t j = p / (2 * L);
  const LimbConst& lc = C.limb[l];
  const uint64_t* u = u_ntt + (j * L + l) * n;
  const uint64_t* pk = pk_ntt + ((int64_t)c * L + l) * n;
  const uint64_t* pks = pk_sh + ((int64_t)c * L + l) * n;
  const uint64_t obj = obj_base + (uint64_t)j;
  const TileOrigin to = tile_origin(side, G, j);
  for (int blk = threadIdx.x; blk < n / 4; blk += blockDim.x) {
    U64x4 e = philox((uint64_t)blk, obj, c ? P_ENC_E1 : P_ENC_E0, 0, C.seed, nonce);
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const int i = blk * 4 + z;
      uint64_t v = small_to_mod(cbd21(e.v[z]), lc.q);
      if (c == 0) {
        const int64_t off = slot_at(side, G, V, to, i);
        if (off >= 0) {
          uint64_t m = (uint64_t)share[off];
          v = add_mod(v, delta_scale(m, round_rho(m, C), lc), lc.q);
        }
      }
      lds[lpad(i)] = v;
    }
  }
  __syncthreads();
  ntt_fwd<LOGN, LOGE, F60, F60>(lds, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  uint64_t* o = ct + p * n;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    o[i] = split30(add_mod(mul_shoup(u[i], pk[i], pks[i], lc.q), lds[lpad(i)], lc.q));
}

// Decryption phase per limb: x = c0 + INTT(NTT(c1) * s).  Grid: n * L, x is [n][L][N].
template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_phase(const uint64_t* ct, uint64_t* x, const uint64_t* s_ntt,
                                                const uint64_t* s_sh, Consts C, Tables T) {
  extern __shared__ uint64_t lds[];
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int64_t p = blockIdx.x;
  const int l = (int)(p % L);
  const int64_t j = p / L;
  const LimbConst& lc = C.limb[l];
  const uint64_t* c0 = ct + ((j * 2 + 0) * L + l) * n;
  // residues as the caller has them, sums of ciphertexts unreduced: any
  // representative for the F60 butterflies, below 16 q for the others; read by the
  // first pass itself
  const PENCIL_GLOBAL uint64_t* c1 = gview(ct + ((j * 2 + 1) * L + l) * n);
  if constexpr (F60) {
    const BflyK<true> bk = bfly_consts<true>(lc.q);
    ntt_fwd_in<LOGN, LOGE, F60>(lds, [&](int i) { return fold60(c1[i], bk); }, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  } else {
    ntt_fwd_in<LOGN, LOGE, F60>(lds, [c1](int i) { return c1[i]; }, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  }
  const uint64_t* sv = s_ntt + (int64_t)l * n;
  const uint64_t* ss = s_sh + (int64_t)l * n;
  for (int i = threadIdx.x; i < n; i += blockDim.x) lds[lpad(i)] = mul_shoup(lds[lpad(i)], sv[i], ss[i], lc.q);
  __syncthreads();
  uint64_t* o = x + p * n;
  uint64_t* poly = lds;
  ntt_inv_in<LOGN, LOGE, F60>(
      lds, [poly](int i) { return poly[lpad(i)]; },
      [o, c0, &lc](int i, uint64_t v) { o[i] = add_mod(c0[i], v, lc.q); }, iw_table<LOGN, LOGE>(T, C, l), lc.q);
}

// Exact decryption of the output slots: with y_l = x_l * (q/q_l)^-1 mod q_l and
// y_l t = alpha_l q_l + beta_l,  t x / q = sum alpha_l + sum beta_l / q_l - v t,
// so m = (sum alpha_l + round(F / q)) mod t with F = sum beta_l (q / q_l); the
// rounding compares 2F with (2j + 1) q.  One thread per output element.
// With `noise` set, the distance |F / q - round(F / q)| = |t x / q - m'| (m' the
// unreduced message), which is the noise as a fraction of q / t, is also
// computed in double precision (sum of beta_l / q_l, error ~L 2^-53) and its
// maximum kept in *noise (float bits; non-negative floats order like integers).
//
// What bounds it: vector instruction issue.  Indices are 32-bit (the launcher
// splits a call of 2^31 outputs or more) and the limb count is a template
// parameter: 2F < 2 L q < 2^(60 L + 3) fits L words, and a threshold is compared
// by the borrow of one multiword subtraction.  64-bit indices, division by t
// and loops over all words took 124 us for the outputs of a 64 -> 64 channel layer
// on 32 x 32, batch 64 (N = 16384, L = 4), this 91 us.
template <int L>
__global__ void __launch_bounds__(256) k_decode(const uint64_t* x, int64_t* share, uint32_t o_base, uint32_t count,
                                                uint32_t per, Geo G, View OV, Consts C, uint32_t* noise) {
  const uint32_t g = blockIdx.x * 256 + threadIdx.x;
  if (g >= count) return;
  const uint32_t oo = g / per;
  uint32_t e = g - oo * per;
  const uint32_t o = o_base + oo;
  const uint32_t ye = e / (uint32_t)G.ow, x_ = e - ye * (uint32_t)G.ow;
  const uint32_t re = ye / (uint32_t)G.oh, y = ye - re * (uint32_t)G.oh;
  const uint32_t mm = re / (uint32_t)G.rt, rr = re - mm * (uint32_t)G.rt;
  const uint32_t ty = o / (uint32_t)G.nOX, oxi = o - ty * (uint32_t)G.nOX;
  const uint32_t tr = ty / (uint32_t)G.nOY, oyi = ty - tr * (uint32_t)G.nOY;
  const uint32_t mi = tr / (uint32_t)G.nR, ri = tr - mi * (uint32_t)G.nR;
  const int m = (int)(mi * G.mt + mm), r = (int)(ri * G.rt + rr), yy = (int)(oyi * G.oh + y), xx = (int)(oxi * G.ow + x_);
  if (m >= G.M || r >= G.R || yy >= G.OH || xx >= G.OW) return;
  const int slot = (int)mm * G.RS + G.O + (int)rr * G.S + (int)y * G.wa + (int)x_;
  const PENCIL_GLOBAL uint64_t* xp = gview(x + (int64_t)o * L * C.n + slot);
  uint64_t F[L];
#pragma unroll
  for (int w = 0; w < L; ++w) F[w] = 0;
  uint64_t alpha = 0;
  double fsum = 0.0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const LimbConst& lc = C.limb[l];
    const uint64_t yl = mul_shoup(xp[(int64_t)l * C.n], lc.qhat_inv, lc.qhat_inv_sh, lc.q);
    uint64_t est = __umul64hi(yl, lc.t_sh);
    uint64_t beta = yl * C.t - est * lc.q;
    if (beta >= lc.q) {
      beta -= lc.q;
      est += 1;
    }
    if (noise) fsum += (double)beta / (double)lc.q;
    alpha += est;  // each alpha_l < t
    // F += beta * qhat_l, which has L - 1 words (one for L = 1)
    uint64_t carry = 0;
#pragma unroll
    for (int w = 0; w < (L > 1 ? L - 1 : 1); ++w) {
      uint64_t ph, pl;
      mul_wide(beta, C.qhat[l][w], ph, pl);
      uint64_t s1 = F[w] + pl;
      uint64_t c1 = s1 < pl;
      uint64_t s2 = s1 + carry;
      c1 += s2 < carry;
      F[w] = s2;
      carry = ph + c1;
    }
    if (L > 1) F[L - 1] += carry;
  }
  // rnd = number of thresholds below 2F
  uint64_t rnd = 0;
#pragma unroll
  for (int j = 0; j < L; ++j) {
    uint64_t borrow = 0;
#pragma unroll
    for (int w = 0; w < L; ++w) {
      const uint64_t d = (F[w] << 1) | (w ? F[w - 1] >> 63 : 0), h = C.thr[j][w];
      borrow = h < d || (h == d && borrow) ? 1 : 0;
    }
    rnd += borrow;
  }
  const uint64_t mres = reduce64(alpha + rnd, C.one_sh_t, C.t);
  gview(share)[m * OV.s0 + r * OV.s1 + yy * OV.sy + xx * OV.sx] = (int64_t)mres;
  if (noise) {
    const float frac = (float)fabs(fsum - (double)rnd);
    atomicMax(noise, __float_as_uint(frac));
  }
}

// Key generation, one block per limb: s ternary (stream P_SK), a uniform mod q_l
// (stream P_PK_A, limb l, two words per coefficient), e CBD21 (stream P_PK_E);
// pk = (-(a s + e), a), kept in both coefficient and NTT form.  One LDS buffer;
// every thread re-reads only the global entries it wrote itself.
template <int LOGN, int LOGE, bool F60>
__global__ void PENCIL_NTT_BOUNDS(LOGN, LOGE) k_keygen(uint64_t* s_ntt, int64_t* s_coeff, uint64_t* pk_coeff,
                                                 uint64_t* pk_ntt, Consts C, Tables T) {
  extern __shared__ uint64_t lds[];
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int l = blockIdx.x;
  const LimbConst& lc = C.limb[l];
  const uint64_t nonce = kKeygenNonce;
  const TW* tw = fw_table<LOGN, LOGE>(T, C, l);
  for (int blk = threadIdx.x; blk < n / 8; blk += blockDim.x) {
    U64x4 w = philox((uint64_t)blk, 0, P_SK, 0, C.seed, nonce);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      int64_t sv = ternary32((uint32_t)(w.v[h >> 1] >> (32 * (h & 1))));
      lds[lpad(blk * 8 + h)] = small_to_mod(sv, lc.q);
      if (l == 0) s_coeff[blk * 8 + h] = sv;
    }
  }
  __syncthreads();
  ntt_fwd<LOGN, LOGE, F60>(lds, tw, lc.q);
  for (int i = threadIdx.x; i < n; i += blockDim.x) s_ntt[(int64_t)l * n + i] = lds[lpad(i)];
  __syncthreads();
  for (int blk = threadIdx.x; blk < n / 2; blk += blockDim.x) {
    U64x4 w = philox((uint64_t)blk, 0, P_PK_A, (uint64_t)l, C.seed, nonce);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // (w_lo + 2^64 w_hi) mod q
      uint64_t hi = reduce64(w.v[2 * h + 1], lc.one_sh, lc.q);
      uint64_t v = add_mod(mul_shoup(hi, lc.r64, lc.r64_sh, lc.q), reduce64(w.v[2 * h], lc.one_sh, lc.q), lc.q);
      lds[lpad(blk * 2 + h)] = v;
      pk_coeff[((int64_t)1 * L + l) * n + blk * 2 + h] = v;
    }
  }
  __syncthreads();
  ntt_fwd<LOGN, LOGE, F60>(lds, tw, lc.q);
  // a * s pointwise (128-bit product, Barrett), then inverse transform
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const uint64_t av = lds[lpad(i)];
    pk_ntt[((int64_t)1 * L + l) * n + i] = av;
    uint64_t ph, pl;
    mul_wide(av, s_ntt[(int64_t)l * n + i], ph, pl);
    lds[lpad(i)] = reduce128(ph, pl, lc.q, lc.mu_lo, lc.mu_hi);
  }
  __syncthreads();
  ntt_inv<LOGN, LOGE, F60>(lds, iw_table<LOGN, LOGE>(T, C, l), lc.q);
  __syncthreads();
  for (int blk = threadIdx.x; blk < n / 4; blk += blockDim.x) {
    U64x4 w = philox((uint64_t)blk, 0, P_PK_E, 0, C.seed, nonce);
#pragma unroll
    for (int z = 0; z < 4; ++z) {
      const int i = blk * 4 + z;
      uint64_t as = lds[lpad(i)];
      uint64_t v = add_mod(as, small_to_mod(cbd21(w.v[z]), lc.q), lc.q);
      v = v == 0 ? 0 : lc.q - v;
      lds[lpad(i)] = v;
      pk_coeff[(int64_t)l * n + i] = v;
    }
  }
  __syncthreads();
  ntt_fwd<LOGN, LOGE, F60>(lds, tw, lc.q);
  for (int i = threadIdx.x; i < n; i += blockDim.x) pk_ntt[(int64_t)l * n + i] = lds[lpad(i)];
}

hipError_t launch_encrypt(const uint64_t* u_ntt, const int64_t* share, uint64_t* ct, int64_t n_ct, int side,
                          const Geo& G, const View& V, const uint64_t* pk_ntt, const uint64_t* pk_sh, uint64_t nonce,
                          uint64_t obj_base, const Consts& C, const Tables& T, hipStream_t s) {
  if (n_ct <= 0) return hipSuccess;
  NTT_DISPATCH(k_encrypt, dim3((unsigned)(n_ct * 2 * C.L)), C, s, u_ntt, share, ct, side, G, V, pk_ntt, pk_sh, nonce,
               obj_base, C, T);
  return hipGetLastError();
}

hipError_t launch_phase(const uint64_t* ct, uint64_t* x, int64_t n_ct, const uint64_t* s_ntt, const uint64_t* s_sh,
                        const Consts& C, const Tables& T, hipStream_t s) {
  if (n_ct <= 0) return hipSuccess;
  NTT_DISPATCH(k_phase, dim3((unsigned)(n_ct * C.L)), C, s, ct, x, s_ntt, s_sh, C, T);
  return hipGetLastError();
}

hipError_t launch_decode(const uint64_t* x, int64_t* share, int64_t n_out, const Geo& G, const View& outV,
                         const Consts& C, uint32_t* noise, hipStream_t s) {
  const int64_t per = (int64_t)G.mt * G.rt * G.oh * G.ow;
  if (n_out <= 0 || per <= 0) return hipSuccess;
  if (n_out >= ((int64_t)1 << 32) || per >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const int64_t polys = (((int64_t)1 << 31) - 1) / per;  // of one launch
  for (int64_t o = 0; o < n_out; o += polys) {
    const uint32_t count = (uint32_t)((n_out - o < polys ? n_out - o : polys) * per);
    const dim3 grid((count + 255) / 256);
    switch (C.L) {
      case 1: hipLaunchKernelGGL(k_decode<1>, grid, dim3(256), 0, s, x, share, (uint32_t)o, count, (uint32_t)per, G, outV, C, noise); break;
      case 2: hipLaunchKernelGGL(k_decode<2>, grid, dim3(256), 0, s, x, share, (uint32_t)o, count, (uint32_t)per, G, outV, C, noise); break;
      case 3: hipLaunchKernelGGL(k_decode<3>, grid, dim3(256), 0, s, x, share, (uint32_t)o, count, (uint32_t)per, G, outV, C, noise); break;
      case 4: hipLaunchKernelGGL(k_decode<4>, grid, dim3(256), 0, s, x, share, (uint32_t)o, count, (uint32_t)per, G, outV, C, noise); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

hipError_t launch_keygen(uint64_t* s_ntt, int64_t* s_coeff, uint64_t* pk_coeff, uint64_t* pk_ntt, const Consts& C,
                         const Tables& T, hipStream_t s) {
  NTT_DISPATCH(k_keygen, dim3((unsigned)C.L), C, s, s_ntt, s_coeff, pk_coeff, pk_ntt, C, T);
  return hipGetLastError();
}


hipError_t configure_lds_do() {
  const int max_lds = 160 * 1024;
  hipError_t e = hipSuccess;
#define PENCIL_RAISE(LN, LE, F)                                                                            \
  for (const void* f : {(const void*)k_encrypt<LN, LE, F>, (const void*)k_phase<LN, LE, F>,                    \
                        (const void*)k_keygen<LN, LE, F>}) {                                                \
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
