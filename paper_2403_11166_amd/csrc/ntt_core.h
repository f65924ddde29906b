// Negacyclic NTT of one limb-polynomial per workgroup, staged in LDS, and
// the forward-transform front ends of the product path (input ciphertexts
// with the model owner's share, encoded plaintexts, ternary masks).
#pragma once
#include "device_common.h"

namespace pencil {

// ----------------------------------------------------------------- NTT core
// One workgroup transforms one limb-polynomial held in LDS.  N/E threads each
// keep E residues in registers (E = 16, or 32 if tuned so) and run several
// butterfly stages per LDS round trip; the log2 N stages are split into
// ceil(log2 N / log2 E) passes of near-equal size.  LDS rows are padded by one
// word every 32 so that strided passes spread over the banks.
__device__ __forceinline__ int lpad(int i) { return i + (i >> 5); }

template <int LOGN, int LOGE_>
struct NttShape {
  static constexpr int LOGE = LOGE_;
  static constexpr int E = 1 << LOGE;
  static constexpr int T = (1 << LOGN) / E;  // threads per block
  static constexpr int NP = ntt_pass_count(LOGN, LOGE);
  static constexpr int size(int i) { return ntt_pass_size(LOGN, LOGE, i); }
  static constexpr int start(int i) { return ntt_pass_start(LOGN, LOGE, i); }
};

// Limb l's twiddles in the order of this width's passes.
template <int LOGN, int LOGE>
__device__ __forceinline__ const TW* fw_table(const Tables& T, const Consts& C, int l) {
  return T.fw + (((int64_t)(LOGE - 4) * 2 * C.L + l) << LOGN);
}
template <int LOGN, int LOGE>
__device__ __forceinline__ const TW* iw_table(const Tables& T, const Consts& C, int l) {
  return T.iw + (((int64_t)(LOGE - 4) * 2 * C.L + l) << LOGN);
}

// Launch bounds of a kernel that transforms one polynomial per workgroup:
// N / E threads (1024 only for E = 16 at N = 16384, one workgroup per CU by
// LDS) and the waves per SIMD the registers must allow (4 with 16 residues per
// thread, 2 with 32).
constexpr int ntt_threads(int logn, int loge) { return (1 << logn) >> loge; }
constexpr int ntt_min_waves(int logn, int loge) { return ntt_threads(logn, loge) > 512 || loge < 5 ? 4 : 2; }
#define PENCIL_NTT_BOUNDS(LOGN, LOGE) __launch_bounds__(ntt_threads(LOGN, LOGE), ntt_min_waves(LOGN, LOGE))

// What bounds the transforms: vector instruction issue (68 % of the SIMD cycles of
// the forward launch at N = 16384 with four cycles an instruction, more by the costs
// below; 52 % of the inverse's), then, for the inverse, the loads and stores
// that nothing overlaps at one workgroup per CU.  Issue costs measured here, in
// cycles per wave: v_and, v_add 2.5; v_alignbit, v_mul_hi, v_lshl_or 4.4-4.6;
// 64-bit shifts and adds 5; v_mad_u64_u32 5.3.  Forward launch of three conv layers
// (107 k polynomials, N = 16384, L = 4) 12.9 -> 10.2 ms, inverse 3.86 -> 2.74 ms:
// the F60 product 85 -> 62 cycles per butterfly, twiddles in the passes' order,
// N^-1 in the last stage's twiddles, results stored from registers, 1024 threads
// of 16 residues instead of 512 of 32.
//
// Two kinds of butterfly.  F60 is for moduli q = 2^60 - delta with delta <= 2^26
// (the library's own 60-bit primes; a context qualifies if all its limbs do),
// the other for every modulus a context accepts.
//
// Butterfly constants of one modulus q < 2^60, hidden from the optimiser so
// that x - 4q stays the single 64-bit addition x + (2^64 - 4q) instead of a
// borrow chain.  F60: 4q, 5q, 8q, 2^64 - q, and delta, 2 delta,
// 4 delta.  Else: 8q, 4q and
// 2^64 minus each, 2^64 - q, and for the final reduction the bit length B of q
// (q < 2^B), 2^B - 1 and delta = 2^B - q.
template <bool F60>
struct BflyK;
template <>
struct BflyK<false> {
  uint64_t q8, nq8, q4, nq4, nq, top_mask;
  uint32_t top_bits, top_delta;
};
template <>
struct BflyK<true> {
  uint64_t q4, q5, q8, nq;
  uint32_t delta, delta2, delta4;
};

template <bool F60>
__device__ __forceinline__ BflyK<F60> bfly_consts(uint64_t q) {
  if constexpr (F60) {
    const uint32_t delta = (uint32_t)((1ull << 60) - q);
    BflyK<true> k{4 * q, 5 * q, 8 * q, 0 - q, delta, 2 * delta, 4 * delta};
    asm volatile("" : "+s"(k.q4), "+s"(k.q5), "+s"(k.q8), "+s"(k.nq), "+s"(k.delta), "+s"(k.delta2), "+s"(k.delta4));
    return k;
  } else {
    const uint32_t b = 64 - (uint32_t)__builtin_clzll(q);
    BflyK<false> k{8 * q, 0 - 8 * q, 4 * q, 0 - 4 * q, 0 - q, (1ull << b) - 1, b, (uint32_t)((1ull << b) - q)};
    asm volatile("" : "+s"(k.q8), "+s"(k.nq8), "+s"(k.q4), "+s"(k.nq4), "+s"(k.nq), "+s"(k.top_mask),
                 "+s"(k.top_bits), "+s"(k.top_delta));
    return k;
  }
}

// x - c if x >= c, else x, for x < 2c and c <= 2^63 (nc = 2^64 - c): x - c
// taken as a signed 64-bit value is negative exactly when x < c.
__device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t c, uint64_t nc) {
  const uint64_t d = x + nc;
  return (int64_t)d < 0 ? x : d;
}

// Lazy Shoup product y w mod q in [0, 4q) for any y < 2^64, w < q, with
// companion ws = floor(w 2^64 / q).  Of y ws / 2^64 = y1 ws1 + (y1 ws0 + y0 ws1)
// / 2^32 + y0 ws0 / 2^64 (32-bit halves) the estimate keeps y1 ws1 +
// hi(y0 ws1) + hi(y1 ws0): three multiplies instead of four.  The dropped parts
// sum to less than 3, so the estimate is at most 2 below floor(y ws / 2^64),
// which is itself at most 1 below floor(y w / q); y w - est q is then below 4q.
__device__ __forceinline__ uint64_t mul_lazy(uint64_t y, const TW w, const BflyK<false>& k) {
  const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
  const uint32_t s0 = (uint32_t)w.ws, s1 = (uint32_t)(w.ws >> 32);
  uint64_t est = (uint64_t)y1 * s1 + __umulhi(y0, s1);
  est += __umulhi(y1, s0);
  return y * w.w + est * k.nq;
}

// F60: y w mod q for any y < 2^64, from the split forms of w and of w' = w 2^32
// mod q.  With y = y0 + y1 2^32, V = y0 w + y1 w' <= 2 (2^32 - 1)(q - 1) < 2^93;
// its 30-bit parts are c0 + Q 2^30 (four multiply-adds, Q < 2^63).  Cutting Q at
// bit 31 or 32, Q = l + h 2^31 or l + h 2^32, and using 2^61 = 2 delta and 2^62 =
// 4 delta (mod q), V = c0 + l 2^30 + 2 delta h (below 2^61 + 2^59 < 3q) or c0 +
// l 2^30 + 4 delta h (below 2^62 + 2^59 < 5q, two instructions fewer: the forward
// transform, whose values have room to grow, takes this one).  Five 32-bit
// multiplies and no quotient, where Shoup's form takes nine; the transforms are
// bound by instruction issue.
template <bool CUT32 = false>
__device__ __forceinline__ uint64_t mul_lazy(uint64_t y, const TW w, const BflyK<true>& k) {
  const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
  uint64_t p = (uint64_t)y0 * (uint32_t)w.w;
  p += (uint64_t)y1 * (uint32_t)w.ws;
  uint64_t c = (uint64_t)y0 * (uint32_t)(w.w >> 32) + (p >> 30);
  asm("" : "+v"(c));  // p >> 30 enters a multiply-add instead of an addition of its own
  c += (uint64_t)y1 * (uint32_t)(w.ws >> 32);
  const uint32_t cl = (uint32_t)c;
  // c0 | l << 30 in one instruction (written out, it becomes a 64-bit shift and masks)
  uint32_t lo;
  asm("v_lshl_or_b32 %0, %1, 30, %2" : "=v"(lo) : "v"(cl), "v"((uint32_t)p & 0x3FFFFFFFu));
  if constexpr (CUT32) return ((uint64_t)(cl >> 2) << 32 | lo) + (uint64_t)(uint32_t)(c >> 32) * k.delta4;
  uint32_t hi;
  asm("v_bfe_u32 %0, %1, 2, 29" : "=v"(hi) : "v"(cl));
  return ((uint64_t)hi << 32 | lo) + (uint64_t)(uint32_t)(c >> 31) * k.delta2;
}

// F60: x < 2^64 -> below 2^60 + 15 delta, the same residue.
__device__ __forceinline__ uint64_t fold60(uint64_t x, const BflyK<true>& k) {
  const uint32_t h = (uint32_t)(x >> 60);
  return (x & ((1ull << 60) - 1)) + (uint64_t)h * k.delta;
}

// Lazy Cooley-Tukey butterfly of stage s (a compile-time constant after
// unrolling).  Plain moduli reduce x by 8q on even stages: x and y in [0, 16q)
// give a = x mod 8q in [0, 8q) and outputs in [0, 12q); on odd stages inputs in
// [0, 12q) give outputs in [0, 16q).  The Shoup product t is below 4q for any y,
// and 16q < 2^64 for q < 2^60.  F60: t < 5q, so a stage adds at most 5q, and x
// folds every third stage: from at most 2^60 - 1 + 15 delta three stages stay
// below 2^60 + 15 delta + 15 q = 2^64.
__device__ __forceinline__ void ct_bfly(uint64_t& x, uint64_t& y, const TW w, const BflyK<false>& k, const int s) {
  const uint64_t a = s % 2 == 0 ? csub(x, k.q8, k.nq8) : x;
  const uint64_t t = mul_lazy(y, w, k);
  x = a + t;
  y = (a + k.q4) - t;
}
__device__ __forceinline__ void ct_bfly(uint64_t& x, uint64_t& y, const TW w, const BflyK<true>& k, const int s) {
  const uint64_t a = s % 3 == 0 && s > 0 ? fold60(x, k) : x;
  const uint64_t t = mul_lazy<true>(y, w, k);
  x = a + t;
  y = (a + k.q5) - t;
}

// Lazy Gentleman-Sande butterfly of stage s.  Plain moduli: u, v in [0, 4q) ->
// [0, 4q).  F60: even stages take [0, 4q) and leave sums unreduced below 8q;
// odd stages take [0, 8q), fold the sums (below 16q < 2^64) to 2^60 + 15 delta,
// and products are below 2^61 + 2^59 < 4q throughout.
__device__ __forceinline__ void gs_bfly(uint64_t& u, uint64_t& v, const TW w, const BflyK<false>& k, const int) {
  const uint64_t s = csub(u + v, k.q4, k.nq4);
  const uint64_t d = (u + k.q4) - v;
  v = mul_lazy(d, w, k);
  u = s;
}
__device__ __forceinline__ void gs_bfly(uint64_t& u, uint64_t& v, const TW w, const BflyK<true>& k, const int s) {
  const uint64_t sum = u + v;
  const uint64_t d = (u + (s % 2 ? k.q8 : k.q4)) - v;
  v = mul_lazy<false>(d, w, k);
  u = s % 2 ? fold60(sum, k) : sum;
}

// The last stage, with N^-1 in both its twiddles: u + v and u - v times w0, w1.
template <bool F60>
__device__ __forceinline__ void gs_last(uint64_t& u, uint64_t& v, const TW w0, const TW w1, const BflyK<F60>& k,
                                        const int s) {
  uint64_t c;
  if constexpr (F60) c = s % 2 ? k.q8 : k.q4;
  else c = k.q4;
  const uint64_t sum = u + v, d = (u + c) - v;
  u = mul_lazy(sum, w0, k);
  v = mul_lazy(d, w1, k);
}

// x < 2^64 (F60) or x in [0, 16q) -> x mod q.  With x = h 2^B + r (r < 2^B,
// h < 16), x = r + h delta (mod q), and r + h delta < 2^B + 15 delta < 2q because
// the moduli lie within 2^B / 17 of 2^B (checked when the context is made).
__device__ __forceinline__ uint64_t reduce_16q(uint64_t x, uint64_t q, const BflyK<false>& k) {
  const uint32_t h = (uint32_t)(x >> k.top_bits);
  const uint64_t y = (uint64_t)h * k.top_delta + (x & k.top_mask);
  return csub(y, q, k.nq);
}
__device__ __forceinline__ uint64_t reduce_16q(uint64_t x, uint64_t q, const BflyK<true>& k) {
  return csub(fold60(x, k), q, k.nq);
}

// Twiddle of a pass: entry e (1 <= e < 2^S) of block blk (B0 bits), stored at
// (e << B0) + blk, so that the lanes of a wave, which take consecutive blocks,
// read consecutive entries.  (In the tables' natural order a thread's entries
// are adjacent instead: each 16-byte load then touched 64 cache lines and the
// L1, which 16 waves overran, fetched every line several times: an inverse
// transform of 128 KB, N = 16384, read 1.15 MB from the L2, and 0.79 MB now.)  With blocks of 64 or more groups a whole wave uses the
// same entries, which SCALAR passes read through the scalar cache.  All do but the
// encryption's with plain moduli (k_encrypt), N = 4096, L = 2, 50-bit moduli, scalar
// against vector loads: 30 ciphertexts 22.7 and 21.8 us, 1024 189 and 186 us, but the
// forward transforms of a step 103.7 and 104.3 us, its inverse 35.4 and 35.7 us.
template <int B0, bool UNIFORM>
__device__ __forceinline__ TW twiddle_at(const PENCIL_GLOBAL TW* tw, int e, int blk) {
  if constexpr (UNIFORM) {
    const auto* p = (const __attribute__((address_space(4))) TW*)(tw + ((e << B0) + __builtin_amdgcn_readfirstlane(blk)));
    return TW{p->w, p->ws};
  } else {
    const PENCIL_GLOBAL TW* p = tw + ((e << B0) + blk);
    return TW{p->w, p->ws};
  }
}

// Forward (merged negacyclic Cooley-Tukey, psi^rev twiddles; natural order in,
// bit-reversed out) stages S0 .. S0+S-1.  At stage l (t = N >> (l+1)) the pair
// (i0, i0 + t) of group i = i0 >> (log2 N - l) uses psi^rev(2^l + i).  A thread
// takes E / 2^S groups of 2^S residues {base + k * 2^LT}, LT = log2 N - S0 - S.
// `in(i)` supplies input residue i: the LDS polynomial, or for the first pass
// values the caller computes (an encoding), which then skip the LDS.
template <int LOGN, int LOGE, bool F60, int S0, int S, bool LAST, bool SCALAR, typename In>
__device__ __forceinline__ void fwd_pass(uint64_t* a, In in, const PENCIL_GLOBAL TW* tw, uint64_t q,
                                         const BflyK<F60>& bk) {
  using Sh = NttShape<LOGN, LOGE>;
  constexpr int T = Sh::T, G = Sh::E >> S, K = 1 << S, LT = LOGN - S0 - S;
  const int tid = threadIdx.x;
  uint64_t v[Sh::E];
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const int g = r * T + tid;
    const int base = ((g >> LT) << (LOGN - S0)) + (g & ((1 << LT) - 1));
#pragma unroll
    for (int k = 0; k < K; ++k) v[r * K + k] = in(base + (k << LT));
  }
  // A wave whose first-pass inputs are all zero (most waves of a sparse K
  // tile) skips the butterflies: its outputs are zero, a representative of
  // the same residues the lazy butterflies would give.
  bool work = true;
  if constexpr (S0 == 0) {
    uint64_t any = 0;
#pragma unroll
    for (int i = 0; i < Sh::E; ++i) any |= v[i];
    work = __builtin_amdgcn_ballot_w64(any != 0) != 0;
  }
  if (work) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int h = 1 << (S - 1 - s);
#pragma unroll
      for (int r = 0; r < G; ++r) {
        const int blk = (r * T + tid) >> LT;
#pragma unroll
        for (int j = 0; j < (1 << s); ++j) {
          const TW w = twiddle_at<S0, (SCALAR && LT >= 6)>(tw, (1 << s) + j, blk);
#pragma unroll
          for (int k = j << (S - s); k < ((j + 1) << (S - s)); ++k) {
            if (k & h) continue;
            ct_bfly(v[r * K + k], v[r * K + k + h], w, bk, S0 + s);
          }
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const int g = r * T + tid;
    const int base = ((g >> LT) << (LOGN - S0)) + (g & ((1 << LT) - 1));
#pragma unroll
    for (int k = 0; k < K; ++k) {
      uint64_t x = v[r * K + k];
      if (LAST) x = reduce_16q(x, q, bk);
      a[lpad(base + (k << LT))] = x;
    }
  }
}

// Inverse (Gentleman-Sande, psi^-rev twiddles; bit-reversed in, natural out)
// stages with t = 2^L0 .. 2^(L0+S-1): pair (i0, i0 + t), i = i0 >> (l + 1),
// twiddle psi^-rev((N >> (l + 1)) + i).  Groups are {base + k * 2^L0}.  Table
// entries 0 and 1 hold N^-1 and N^-1 psi^-rev(1), the twiddles of the last stage.
// `out(i, x)` takes result i (reduced to [0, q) in the last pass).
template <int LOGN, int LOGE, bool F60, int L0, int S, typename In, typename Out>
__device__ __forceinline__ void inv_pass(In in, Out out, const PENCIL_GLOBAL TW* tw, uint64_t q,
                                         const BflyK<F60>& bk) {
  constexpr bool LAST = L0 + S == LOGN;
  using Sh = NttShape<LOGN, LOGE>;
  constexpr int T = Sh::T, G = Sh::E >> S, K = 1 << S;
  const int tid = threadIdx.x;
  uint64_t v[Sh::E];
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const int g = r * T + tid;
    const int base = ((g >> L0) << (L0 + S)) + (g & ((1 << L0) - 1));
#pragma unroll
    for (int k = 0; k < K; ++k) v[r * K + k] = in(base + (k << L0));
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int h = 1 << s;
#pragma unroll
    for (int r = 0; r < G; ++r) {
      const int blk = (r * T + tid) >> L0;
#pragma unroll
      for (int j = 0; j < (K >> (s + 1)); ++j) {
        const TW w = twiddle_at<LOGN - L0 - S, (L0 >= 6)>(tw, (K >> (s + 1)) + j, blk);
#pragma unroll
        for (int k = j << (s + 1); k < ((j + 1) << (s + 1)); ++k) {
          if (k & h) continue;
          if (LAST && s == S - 1)
            gs_last(v[r * K + k], v[r * K + k + h], twiddle_at<0, true>(tw, 0, 0), w, bk, L0 + s);
          else
            gs_bfly(v[r * K + k], v[r * K + k + h], w, bk, L0 + s);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < G; ++r) {
    const int g = r * T + tid;
    const int base = ((g >> L0) << (L0 + S)) + (g & ((1 << L0) - 1));
#pragma unroll
    for (int k = 0; k < K; ++k) out(base + (k << L0), LAST ? reduce_16q(v[r * K + k], q, bk) : v[r * K + k]);
  }
}

// Forward transform into the LDS polynomial `a` (outputs in [0, q)) of the
// inputs in [0, q) that `in(i)` supplies to the first pass; the transform's
// first LDS access is the first pass' store, so `a` must not be in use.
// Callers synchronise after (outputs read).
template <int LOGN, int LOGE, bool F60, bool SCALAR = true, typename In>
__device__ __forceinline__ void ntt_fwd_in(uint64_t* a, In in, const TW* tw_generic, uint64_t q) {
  using Sh = NttShape<LOGN, LOGE>;
  const BflyK<F60> bk = bfly_consts<F60>(q);
  const PENCIL_GLOBAL TW* tw = gview(tw_generic);
  auto lds = [a](int i) { return a[lpad(i)]; };
  fwd_pass<LOGN, LOGE, F60, Sh::start(0), Sh::size(0), Sh::NP == 1, SCALAR>(a, in, tw, q, bk);
  __syncthreads();
  if constexpr (Sh::NP > 1) {
    fwd_pass<LOGN, LOGE, F60, Sh::start(1), Sh::size(1), Sh::NP == 2, SCALAR>(a, lds, tw, q, bk);
    __syncthreads();
  }
  if constexpr (Sh::NP > 2) {
    fwd_pass<LOGN, LOGE, F60, Sh::start(2), Sh::size(2), Sh::NP == 3, SCALAR>(a, lds, tw, q, bk);
    __syncthreads();
  }
  if constexpr (Sh::NP > 3) {
    fwd_pass<LOGN, LOGE, F60, Sh::start(3), Sh::size(3), true, SCALAR>(a, lds, tw, q, bk);
    __syncthreads();
  }
}

// Forward transform of the LDS polynomial (inputs in [0, q), outputs in [0, q)).
// Callers synchronise before (inputs written) and after (outputs read).
template <int LOGN, int LOGE, bool F60, bool SCALAR = true>
__device__ __forceinline__ void ntt_fwd(uint64_t* a, const TW* tw_generic, uint64_t q) {
  ntt_fwd_in<LOGN, LOGE, F60, SCALAR>(a, [a](int i) { return a[lpad(i)]; }, tw_generic, q);
}

// Inverse transform (inputs in [0, 4q), results in [0, q)) by way of the LDS
// polynomial `a`, of the inputs `in(i)` supplies to the first pass (as for
// ntt_fwd_in, `a` must not be in use); `out(i, x)` takes result i from the thread
// that computed it.  A wave's 64 results of a store are consecutive.
template <int LOGN, int LOGE, bool F60, typename In, typename Out>
__device__ __forceinline__ void ntt_inv_in(uint64_t* a, In in, Out out, const TW* tw_generic, uint64_t q) {
  using Sh = NttShape<LOGN, LOGE>;
  static_assert(Sh::NP == 3 || Sh::NP == 4, "pass counts of log2 N = 10 .. 14");
  const BflyK<F60> bk = bfly_consts<F60>(q);
  const PENCIL_GLOBAL TW* tw = gview(tw_generic);
  auto lds = [a](int i) { return a[lpad(i)]; };
  auto put = [a](int i, uint64_t x) { a[lpad(i)] = x; };
  inv_pass<LOGN, LOGE, F60, Sh::start(0), Sh::size(0)>(in, put, tw, q, bk);
  __syncthreads();
  inv_pass<LOGN, LOGE, F60, Sh::start(1), Sh::size(1)>(lds, put, tw, q, bk);
  __syncthreads();
  if constexpr (Sh::NP == 3) {
    inv_pass<LOGN, LOGE, F60, Sh::start(2), Sh::size(2)>(lds, out, tw, q, bk);
  } else {
    inv_pass<LOGN, LOGE, F60, Sh::start(2), Sh::size(2)>(lds, put, tw, q, bk);
    __syncthreads();
    inv_pass<LOGN, LOGE, F60, Sh::start(3), Sh::size(3)>(lds, out, tw, q, bk);
  }
}

// Inverse transform in place of the LDS polynomial (its last pass writes where
// it read); callers synchronise before and after.
template <int LOGN, int LOGE, bool F60>
__device__ __forceinline__ void ntt_inv(uint64_t* a, const TW* tw_generic, uint64_t q) {
  ntt_inv_in<LOGN, LOGE, F60>(
      a, [a](int i) { return a[lpad(i)]; }, [a](int i, uint64_t x) { a[lpad(i)] = x; }, tw_generic, q);
}

// ------------------------------------------------------------------ kernels

// In-place forward or inverse NTT of [polys][L][N].
template <int LOGN, int LOGE, bool F60>
__device__ __forceinline__ void do_ntt_plain(uint64_t* lds, uint64_t* data, int inverse, const Consts& C,
                                             const Tables& T, int64_t p) {
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int l = (int)(p % L);
  const LimbConst& lc = C.limb[l];
  // the first butterfly pass reads its residues straight from memory; results
  // leave the LDS in 16-byte pairs (a pair never straddles an LDS pad word)
  PENCIL_GLOBAL u64x2* g = (PENCIL_GLOBAL u64x2*)gview(data + p * n);
  const PENCIL_GLOBAL uint64_t* g1 = gview(data + p * n);
  auto src = [g1](int i) { return g1[i]; };
  if (!inverse) {
    // F60: any 64-bit representative, folded here; plain butterflies take one below 16 q as it is
    auto red = [&](int i) {
      if constexpr (F60) return fold60(g1[i], bfly_consts<true>(lc.q));
      else return g1[i];
    };
    ntt_fwd_in<LOGN, LOGE, F60>(lds, red, fw_table<LOGN, LOGE>(T, C, l), lc.q);
    for (int i = threadIdx.x; i < n / 2; i += blockDim.x) g[i] = u64x2{lds[lpad(2 * i)], lds[lpad(2 * i) + 1]};
  } else {
    // results go from registers to memory
    PENCIL_GLOBAL uint64_t* o1 = gview(data + p * n);
    ntt_inv_in<LOGN, LOGE, F60>(lds, src, [o1](int i, uint64_t x) { o1[i] = x; }, iw_table<LOGN, LOGE>(T, C, l), lc.q);
  }
}

// Input ciphertexts (NTT domain, split form) of the products that add the
// model owner's share: component 0 gains the transform of round(q m / t) of
// the share (Alg. 1, product step) and is written, split, to the staging
// copy; component 1 is read in place by the multiply-accumulate.
// Grid: count * L blocks, polynomial p = (j, l) in [count][L] order; src is
// [count][2][L][N], and so is dst (component 0 only) in split form; for the
// matrix-core multiply-accumulate dst holds component 0 alone, in V.form.
template <int LOGN, int LOGE, bool F60>
__device__ __forceinline__ void do_ntt_ct(uint64_t* lds, const uint64_t* src, uint64_t* dst, int64_t count, const int64_t* share, const Geo& G, const View& V, const Consts& C,
                                          const Tables& T, int64_t p) {
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int l = (int)(p % L);
  const int64_t j = p / L;
  const int form = V.form;
  const int64_t at = (j * 2 * L + l) * n;  // component 0, limb l of ciphertext j
  const LimbConst& lc = C.limb[l];
  const PENCIL_GLOBAL int64_t* gshare = gview(share);
  const TileOrigin to = a_tile_origin(G, j);
  auto enc = [&](int i) {
    uint64_t v = 0;
    const int64_t off = a_slot_at(G, V, to, i);
    if (off >= 0) {
      const uint64_t m = (uint64_t)gshare[off];
      v = delta_scale(m, round_rho(m, C), lc);
    }
    return v;
  };
  ntt_fwd_in<LOGN, LOGE, F60>(lds, enc, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  // 16-byte accesses: a polynomial is 16-byte aligned
  const PENCIL_GLOBAL u64x2* g2 = (const PENCIL_GLOBAL u64x2*)gview(src + at);
  if (form_blocked(form)) {
    PENCIL_GLOBAL uint64_t* o = gview(dst + ((int64_t)l * (n / kMxGroup) * count + j) * kMxGroup);
    const int64_t group = count * kMxGroup;
    for (int i = threadIdx.x; i < n / 2; i += blockDim.x) {
      const u64x2 v = g2[i];
      const int s = 2 * i;
      *(PENCIL_GLOBAL u64x2*)(o + (s / kMxGroup) * group + s % kMxGroup) =
          u64x2{form_value(add_mod(unsplit30(v[0]), lds[lpad(s)], lc.q), form),
                form_value(add_mod(unsplit30(v[1]), lds[lpad(s) + 1], lc.q), form)};
    }
    return;
  }
  PENCIL_GLOBAL u64x2* o2 = (PENCIL_GLOBAL u64x2*)gview(dst + at);
  for (int i = threadIdx.x; i < n / 2; i += blockDim.x) {
    const u64x2 v = g2[i];
    o2[i] = u64x2{split30(add_mod(unsplit30(v[0]), lds[lpad(2 * i)], lc.q)),
                  split30(add_mod(unsplit30(v[1]), lds[lpad(2 * i) + 1], lc.q))};
  }
}

// Plaintext tiles: encode (side 0: forward A tile, 1: reverse K tile), centred
// lift of Z_t into Z_{q_l}, forward NTT.  Grid: count * L, output [count][L][N]
// or slot-blocked, in V.form.
template <int LOGN, int LOGE, bool F60>
__device__ __forceinline__ void do_ntt_pt(uint64_t* lds, const int64_t* tensor, uint64_t* dst, int64_t count,
                                          int side, const Geo& G, const View& V, const Consts& C, const Tables& T, int64_t p) {
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int l = (int)(p % L);
  const int64_t j = p / L;
  const LimbConst& lc = C.limb[l];
  const PENCIL_GLOBAL int64_t* gt = gview(tensor);
  const TileOrigin to = tile_origin(side, G, j);
  auto lift = [&](int64_t off) {
    const uint64_t w = (uint64_t)gt[off];
    return w <= C.t_half ? w : lc.q - (C.t - w);
  };
  if (side == 0) {
    // A tiles are dense: each slot gathers its value in the first pass
    auto enc = [&](int i) {
      const int64_t off = a_slot_at(G, V, to, i);
      return off >= 0 ? lift(off) : (uint64_t)0;
    };
    ntt_fwd_in<LOGN, LOGE, F60>(lds, enc, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  } else {
    // K tiles hold rt kt kh kw entries, often far fewer than N (a kernel
    // window per channel pair): zero the polynomial, then scatter the entries
    for (int i = threadIdx.x; i < n; i += blockDim.x) lds[lpad(i)] = 0;
    __syncthreads();
    const int nnz = G.rt * G.kt * G.kh * G.kw;
    for (int e = threadIdx.x; e < nnz; e += blockDim.x) {
      int slot;
      const int64_t off = k_entry_at(G, V, to, e, slot);
      if (off >= 0 && slot >= 0 && slot < n) lds[lpad(slot)] = lift(off);
    }
    __syncthreads();
    ntt_fwd<LOGN, LOGE, F60>(lds, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  }
  store_form<LOGN>(dst, V.form, count, L, l, j, [&](int i) { return form_value(lds[lpad(i)], V.form); });
}

// Fresh ternary polynomials (object obj_base + j, stream `purpose`), lifted and
// transformed.  Coefficient i uses the 32-bit half i mod 2 of stream word i/2,
// so one Philox block covers 8 coefficients.  Grid: count * L, output
// [count][L][N] or slot-blocked, in `form`.
template <int LOGN, int LOGE, bool F60>
__device__ __forceinline__ void do_ntt_ternary(uint64_t* lds, uint64_t* dst, uint64_t nonce, uint64_t obj_base,
                                               uint32_t purpose, int form, int64_t count, const Consts& C,
                                               const Tables& T, int64_t p) {
  constexpr int n = 1 << LOGN;
  const int L = C.L;
  const int l = (int)(p % L);
  const int64_t j = p / L;
  const LimbConst& lc = C.limb[l];
  for (int blk = threadIdx.x; blk < n / 8; blk += blockDim.x) {
    U64x4 w = philox((uint64_t)blk, obj_base + j, purpose, 0, C.seed, nonce);
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      uint32_t half = (uint32_t)(w.v[h >> 1] >> (32 * (h & 1)));
      lds[lpad(blk * 8 + h)] = small_to_mod(ternary32(half), lc.q);
    }
  }
  __syncthreads();
  ntt_fwd<LOGN, LOGE, F60>(lds, fw_table<LOGN, LOGE>(T, C, l), lc.q);
  store_form<LOGN>(dst, form, count, L, l, j, [&](int i) { return form_value(lds[lpad(i)], form); });
}

}  // namespace pencil
