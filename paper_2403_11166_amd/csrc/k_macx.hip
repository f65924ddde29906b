// Pointwise multiply-accumulate of the product path on the int8 matrix cores.
#include "mx_common.h"

namespace pencil {

// Per NTT slot the multiply-accumulate is a small matrix product over Z_q,
// out[i, j] = sum_k X[i, k] Y[k, j], X the A rows and Y the K rows.
// Each residue v < 2^60 becomes eight signed digits d_0 .. d_7 in [-128, 128),
// v = sum d_i 2^(8 i): adding 0x80 to every byte position with carries and then
// flipping the bytes' top bits gives their two's complement bytes.  A product
// is sum_s 2^(8 s) D_s with D_s = sum_{i + j = s} x_i y_j, and each diagonal
// D_s (15 of them) is one int32 matrix accumulator over the whole contraction:
// |D_s| <= 2^17 per index, so kMxMaxK indices stay below 2^31.
//
// v_mfma_i32_16x16x64_i8 takes 64 contraction bytes: four digits of 16
// contraction indices.  With Y's bytes reversed into R (R byte p = y_(7-p)) and
// W(o) the four bytes o .. o + 3 of R (zero outside it), the low digits of X
// against W(o) land on diagonal 7 - o and its high digits on 11 - o, so 11
// windows o = -3 .. 7 and 22 instructions cover a block's 64 digit products of
// 16 x 16 x 16 residues with 27 % of the multiplies on zero padding.
//
// A workgroup owns 16 slots of one limb (a 128-byte run of every operand row)
// and a 16 x 16 tile of outputs, one slot per wave: 15 x 4 accumulators leave
// four waves per SIMD.  Contraction blocks of 16 indices are loaded by all
// threads, brought into digits and transposed through LDS; two buffers, so the
// loads of a block are in flight while the one before it is multiplied.  Rows
// are (A row, component) pairs for a product with one term, and A rows of one
// component for the weight gradient, whose terms carry the ciphertext on
// different sides.
//
// Buffers the library writes itself (plaintexts, staged ciphertext components,
// u') are slot-blocked, [limb][slot group][tile][kMxGroup slots], plaintexts and
// staged components already in digits: a workgroup reads them from one
// contiguous range.  Ciphertexts in the caller's buffers are a 128-byte run per
// tile.  With both sides so (32 rows at strides of tens of MiB) the CU's
// first-level address translations missed several times as often; they miss on 0.5
// % of the requests here.
//
// What bounds it: the operand loads.  The products of a training step of three
// conv layers (64, 128 and 256 channels, batch 64, N = 16384, L = 4) take 9.3 ms
// against 18.8 ms in the vector kernel; 25 GB come from memory, 46 GB through the vector L1 (each row is
// read once per 16 x 16 tile).  With the loads left out it takes 6.0 ms, with the
// matrix instructions left out 8.3 ms.  8-slot workgroups (two per CU, 64-byte
// runs) measured the same on these and 3 % slower on memory traffic; letting half
// the waves multiply while the others convert was 3 % slower.
constexpr int kMxTile = 16, kMxKB = 16;
constexpr int kMxSlots = 16;  // slots of a workgroup, one per wave
constexpr int kMxPairs = kMxSlots / 2;
static_assert(kMxThreads == kMxSlots * 64, "one wave per slot");
// LDS layout of one slot's operand: [4 index groups][low, high digits][16 rows]
// [4 indices]; a wave's 16-byte reads are contiguous.  The staging threads' writes
// (8 slot pairs x 4 indices of one row) fall on distinct banks: planes and slots
// are padded by 16 bytes, and the upper eight slots swap neighbouring rows (in
// the output tile: pairs of entries).
constexpr int kMxPlaneBytes = kMxTile * 16 + 16;
constexpr int kMxGroupBytes = 2 * kMxPlaneBytes;
constexpr int kMxSlotBytes = 4 * kMxGroupBytes + 16;
constexpr int kMxOpBytes = kMxSlots * kMxSlotBytes;
constexpr int kMxBufBytes = 2 * kMxOpBytes;
constexpr int kMxLds = 2 * kMxBufBytes;
constexpr int kMxDiag = 15;

// Split-form residue -> digit bytes (low and high words).
__device__ __forceinline__ mx_u2 mx_digits(mx_u2 s) {
  const uint64_t v = ((uint64_t)(s[1] >> 2) << 32 | (s[0] | s[1] << 30)) + 0x8080808080808080ull;
  return mx_u2{(uint32_t)v ^ 0x80808080u, (uint32_t)(v >> 32) ^ 0x80808080u};
}

// The same bytes in reverse order.
__device__ __forceinline__ mx_u2 mx_reversed(mx_u2 d) {
  return mx_u2{__builtin_bswap32(d[1]), __builtin_bswap32(d[0])};
}

// The two instructions of window O.  Windows are formed one at a time: eleven at
// once would not fit the registers.
template <int O>
__device__ __forceinline__ void mx_step(mx_v4i (&acc)[kMxDiag], const mx_v4i xl, const mx_v4i xh, const mx_u4 r0,
                                        const mx_u4 r1) {
  mx_v4i w;
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (int)mx_window<O>(r0[i], r1[i]);
  acc[7 - O] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xl, w, acc[7 - O], 0, 0, 0);
  acc[11 - O] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xh, w, acc[11 - O], 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void mx_block(mx_v4i (&acc)[kMxDiag], const uint8_t* buf, int wave, int lane) {
  const uint8_t* p = buf + wave * kMxSlotBytes + ((lane & 15) ^ wave >> 3) * 16 + (lane >> 4) * kMxGroupBytes;
  const mx_v4i xl = *(const mx_v4i*)p, xh = *(const mx_v4i*)(p + kMxPlaneBytes);
  const mx_u4 r0 = *(const mx_u4*)(p + kMxOpBytes), r1 = *(const mx_u4*)(p + kMxOpBytes + kMxPlaneBytes);
  mx_step<0>(acc, xl, xh, r0, r1);
  mx_step<4>(acc, xl, xh, r0, r1);
  mx_step<1>(acc, xl, xh, r0, r1);
  mx_step<2>(acc, xl, xh, r0, r1);
  mx_step<3>(acc, xl, xh, r0, r1);
  mx_step<-1>(acc, xl, xh, r0, r1);
  mx_step<5>(acc, xl, xh, r0, r1);
  mx_step<-2>(acc, xl, xh, r0, r1);
  mx_step<6>(acc, xl, xh, r0, r1);
  mx_step<-3>(acc, xl, xh, r0, r1);
  mx_step<7>(acc, xl, xh, r0, r1);
}

// One output from its 15 diagonals: sum_s D_s 2^(8 s) + pk u' mod q.  The
// diagonals combine in four positive 64-bit groups g_h = 2^56 + sum_{s < 4}
// D_(4 h + s) 2^(8 s); then, with everything in 30-bit halves (c0, c1),
//   s0 + s1 2^30 + s2 2^60 = g_0 + g_1 2^32 + g_2 r64 + g_3 r96 + pk u' + mx_off
// where mx_off cancels the four offsets mod q.  Moduli just below 2^60
// (q = 2^60 - delta, delta <= 2^26) fold 2^60 = delta twice and leave a value
// below 2^61 + 2^57 < 4 q, which the inverse transform takes; others are
// Barrett-reduced.
template <bool FOLD60>
__device__ __forceinline__ uint64_t mx_combine(const mx_v4i (&acc)[kMxDiag], int r, uint64_t pk, uint64_t u,
                                               int32_t m8, int32_t m16, int32_t m24, const LimbConst& lc) {
  uint64_t g[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    int64_t v = mx_mad(acc[4 * h][r], 1, 1ll << 56);
    v = mx_mad(acc[4 * h + 1][r], m8, v);
    v = mx_mad(acc[4 * h + 2][r], m16, v);
    if (4 * h + 3 < kMxDiag) v = mx_mad(acc[4 * h + 3][r], m24, v);
    g[h] = (uint64_t)v;
  }
  constexpr uint32_t k30 = 0x3FFFFFFFu;
  uint64_t s0 = g[0] + lc.mx_off, s1 = g[1] << 2, s2 = 0;
  auto mac = [&](uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1) {
    s0 += (uint64_t)a0 * b0;
    s1 += (uint64_t)a0 * b1;
    asm volatile("" : "+v"(s1));
    s1 += (uint64_t)a1 * b0;
    s2 += (uint64_t)a1 * b1;
  };
  mac((uint32_t)u, (uint32_t)(u >> 32), (uint32_t)pk, (uint32_t)(pk >> 32));
  mac((uint32_t)g[2] & k30, (uint32_t)(g[2] >> 30), (uint32_t)lc.r64_split, (uint32_t)(lc.r64_split >> 32));
  mac((uint32_t)g[3] & k30, (uint32_t)(g[3] >> 30), (uint32_t)lc.r96_split, (uint32_t)(lc.r96_split >> 32));
  s1 += s0 >> 30;
  s2 += s1 >> 30;
  const uint32_t c0 = (uint32_t)s0 & k30, c1 = (uint32_t)s1 & k30;
  const uint64_t lo60 = (uint64_t)(c1 >> 2) << 32 | (c0 | c1 << 30);
  if constexpr (FOLD60) {
    const uint64_t p0 = (uint64_t)(uint32_t)s2 * lc.delta60;
    const uint64_t p1 = (uint64_t)(uint32_t)(s2 >> 32) * lc.delta60 + (p0 >> 32);  // < 2^58
    const uint64_t rem = (uint64_t)((uint32_t)p1 & 0x0FFFFFFFu) << 32 | (uint32_t)p0;
    return lo60 + rem + (uint64_t)(uint32_t)(p1 >> 28) * lc.delta60;
  }
  const uint64_t hi = s2 >> 4, t = s2 << 60;  // lo60 has no bits there
  return reduce128(hi, lo60 | t, lc.q, lc.mu_lo, lc.mu_hi);
}

// FOLD60: see mx_combine.
template <bool FOLD60>
__device__ __forceinline__ void mx_tile(uint8_t* lds, const MacArgs& A, const Geo& G, const Consts& C, int slot_group,
                                        int tile) {
  const int n = C.n, L = C.L;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // The thread's index, taken from the hardware at each use and opaque to the
  // compiler: what follows from it is not held in registers over the loop,
  // where the accumulators leave few.
  auto thread_id = [&] {
    uint32_t id = (uint32_t)wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(id));
    return id;
  };
  const int per_limb = n / kMxSlots;
  const int l = slot_group / per_limb;
  const int64_t ln = (int64_t)l * n + (int64_t)(slot_group - l * per_limb) * kMxSlots;
  // slot-blocked buffers: group and first slot in it
  const int64_t lg = slot_group / (kMxGroup / kMxSlots), ls = slot_group % (kMxGroup / kMxSlots) * kMxSlots;
  const LimbConst& lc = C.limb[l];
  const int64_t pt_stride = (int64_t)L * n, ct_stride = 2 * pt_stride;
  const int sp = G.nOY * G.nOX, kspan = G.nKY * G.nKX, ksteps = G.nK * kspan;
  // tile -> row tile, column tile (and component for two terms)
  const bool packed = A.n_terms == 1;
  const int ct_tiles = (G.nR + kMxTile - 1) / kMxTile;
  int rt = tile / ct_tiles;
  const int ctile = tile - rt * ct_tiles;
  const int comp = packed ? 0 : rt & 1;
  if (!packed) rt >>= 1;
  const int nb = (ksteps + kMxKB - 1) / kMxKB, total = nb * A.n_terms;
  // Staging: wave w loads row w of the A side (X) and of the K side (Y), each
  // lane two contraction indices of two slots.  The row addresses are
  // wave-uniform; sx, sy are the byte strides of a contraction index (A tiles of
  // a row are one apart, or sp apart where kspan = 1).
  const char *px, *py;
  uint32_t sx, sy;
  bool x_split = false;  // term 0's X row holds split residues, to be turned into digits
  auto set_term = [&](int t) {
    const int f = rt * kMxTile + wave;
    int am = packed ? f >> 1 : f;
    const int c = packed ? f & 1 : comp;
    if (am >= A.m_rows) am = A.m_rows - 1;  // padding rows read the last row (never stored)
    int col = ctile * kMxTile + wave;
    if (col >= G.nR) col = G.nR - 1;
    const int mi = am / sp;
    const int64_t arow = ((int64_t)mi * (G.nK - 1) * sp + am) * kspan, krow = (int64_t)col * ksteps;
    const int64_t na = (int64_t)A.m_rows * ksteps, nk = (int64_t)G.nR * ksteps;
    const uint32_t ctb = (uint32_t)(ct_stride * 8), blk = kMxGroup * 8;
    const MacTerm& T = A.term[t];
    // rows in the caller's buffers: ciphertext strides, split residues
    const bool cx = t == 0 && (c || !A.stage), cy = t == 1;
    if (t == 0) x_split = cx;
    sx = cx ? ctb : blk;
    sy = cy ? ctb : blk;
    px = cx ? (const char*)(T.a + c * pt_stride + ln + arow * ct_stride)
            : (const char*)((t == 0 ? A.stage : T.a) + (lg * na + arow) * kMxGroup + ls);
    py = cy ? (const char*)(T.k + comp * pt_stride + ln + krow * ct_stride)
            : (const char*)(T.k + (lg * nk + krow) * kMxGroup + ls);
    if (kspan == 1) sx *= (uint32_t)sp;
    px = uni(px);
    py = uni(py);
  };
  struct Regs {
    u64x2 x[2], y[2];
  };
  // A lane holds indices kp and kp + 8 (kp = id / 8 % 8) of two slots.
  auto load = [&](int k0) {
    const uint32_t id = thread_id(), pair = id % kMxPairs * 16, kp = id / kMxPairs % 8;
    Regs v;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      uint32_t k = kp + 8 * i;
      if (k0 + kMxKB > ksteps) k = min(k, (uint32_t)(ksteps - 1 - k0));  // a valid index; masked in store
      v.x[i] = *(const PENCIL_GLOBAL u64x2*)((const PENCIL_GLOBAL char*)px + (k * sx + pair));
      v.y[i] = *(const PENCIL_GLOBAL u64x2*)((const PENCIL_GLOBAL char*)py + (k * sy + pair));
    }
    px = uni(px + (uint64_t)kMxKB * sx);
    py = uni(py + (uint64_t)kMxKB * sy);
    return v;
  };
  auto store = [&](const Regs v, uint8_t* buf, int k0, bool xs, bool ys) {
    const uint32_t id = thread_id(), spair = id % kMxPairs, kp = id / kMxPairs % 8;
    mx_u2 x[2][2], y[2][2];  // [index][slot]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        x[i][s] = mx_u2{(uint32_t)v.x[i][s], (uint32_t)(v.x[i][s] >> 32)};
        y[i][s] = mx_u2{(uint32_t)v.y[i][s], (uint32_t)(v.y[i][s] >> 32)};
      }
    if (xs)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i >> 1][i & 1] = mx_digits(x[i >> 1][i & 1]);
    if (ys)
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i >> 1][i & 1] = mx_reversed(mx_digits(y[i >> 1][i & 1]));
    if (k0 + kMxKB > ksteps)  // digit strings of zeros past the contraction's end
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k0 + (int)kp + 8 * (i >> 1) >= ksteps) y[i >> 1][i & 1] = mx_u2{0, 0};
    uint8_t* p = buf + 2 * spair * kMxSlotBytes + (kp >> 2) * kMxGroupBytes + ((uint32_t)wave ^ spair >> 2) * 16 +
                 (kp & 3) * 4;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint8_t* q = p + s * kMxSlotBytes + i * 2 * kMxGroupBytes;
        *(uint32_t*)q = x[i][s][0];
        *(uint32_t*)(q + kMxPlaneBytes) = x[i][s][1];
        *(uint32_t*)(q + kMxOpBytes) = y[i][s][0];
        *(uint32_t*)(q + kMxOpBytes + kMxPlaneBytes) = y[i][s][1];
      }
  };
  // The outputs a thread moves, entries e = id / kMxPairs + 128 t of the tile,
  // slots 2 (id % kMxPairs) and the next: the output's number and component, or -1.
  auto out_tile = [&](uint32_t id, int t, int& c) {
    const int e = (int)(id / kMxPairs) + 128 * t;
    const int fr = rt * kMxTile + (e >> 4), oc = ctile * kMxTile + (e & 15);
    const int m = packed ? fr >> 1 : fr;
    c = packed ? fr & 1 : comp;
    const int mi = sp == 1 ? m : fdiv(m, G.dv_sp);
    return m < A.m_rows && oc < G.nR ? (mi * (G.nR - 1) + oc) * sp + m : -1;
  };
  // The loads of block b; for b = total, u' of this tile's outputs.
  const int64_t n_out = (int64_t)A.m_rows * G.nR;
  auto index_of = [&](int b) { return (b >= nb ? b - nb : b) * kMxKB; };
  auto fetch = [&](int b) {
    if (b >= total) {
      const uint32_t id = thread_id();
      const uint64_t* u = A.u + lg * n_out * kMxGroup + ls;
      Regs v{};
      if (b == total)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          int c;
          const int o = out_tile(id, t, c);
          v.x[t] = *(const PENCIL_GLOBAL u64x2*)(gview(u) + (int64_t)(o < 0 ? 0 : o) * kMxGroup + 2 * (id % kMxPairs));
        }
      return v;
    }
    if (b == nb) set_term(1);
    return load(index_of(b));
  };
  auto tail_at = [&](uint32_t id, int t) { return ((id / kMxPairs ^ (id % kMxPairs >> 2) * 2) + 128 * t) * 8; };
  // Block b to its buffer, and the loads of the next.
  auto put = [&](const Regs v, int b) {
    uint8_t* buf = lds + (b & 1) * kMxBufBytes;
    if (b == total) {
      const uint32_t id = thread_id();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s)
          *(uint64_t*)(buf + (2 * (id % kMxPairs) + s) * kMxSlotBytes + tail_at(id, t)) = v.x[t][s];
      return v;
    }
    store(v, buf, index_of(b), b < nb && x_split, b >= nb);
    return fetch(b + 1);
  };
  set_term(0);
  const Regs v0 = fetch(0);
  Regs v = fetch(1);
  store(v0, lds, 0, x_split, false);
  mx_v4i acc[kMxDiag];
#pragma unroll
  for (int s = 0; s < kMxDiag; ++s) acc[s] = mx_v4i{0, 0, 0, 0};
  __syncthreads();
  // Turn b converts and stores block b, whose loads went out a turn earlier,
  // starts the loads of the block after it, and multiplies block b - 1.
  for (int b = 1; b <= total; ++b) {
    v = put(v, b);
    mx_block(acc, lds + ((b - 1) & 1) * kMxBufBytes, wave, (int)(thread_id() & 63));
    __syncthreads();
  }
  // + pk_c u', recombination and reduction: a lane holds the outputs of rows
  // 4 (lane / 16) + r, column lane % 16
  uint8_t* const fin = lds + (total & 1) * kMxBufBytes;
  uint8_t* tail = fin + wave * kMxSlotBytes;
  const PENCIL_GLOBAL uint64_t* gpk = gview(A.pk);
  const uint64_t pk0 = gpk[ln + wave], pk1 = gpk[pt_stride + ln + wave];
  int32_t m8 = 1 << 8, m16 = 1 << 16, m24 = 1 << 24;
  asm volatile("" : "+v"(m8), "+v"(m16), "+v"(m24));
  const int lane = (int)(thread_id() & 63);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * (lane >> 4) + r;
    uint64_t* slot = (uint64_t*)(tail + ((row * kMxTile + (lane & 15)) ^ (wave >> 3) * 2) * 8);
    const int c = packed ? r & 1 : comp;
    *slot = mx_combine<FOLD60>(acc, r, c ? pk1 : pk0, *slot, m8, m16, m24, lc);
    __builtin_amdgcn_sched_barrier(0);  // one output at a time: the accumulators leave few registers
  }
  __syncthreads();
  const uint32_t id = thread_id();
  PENCIL_GLOBAL uint64_t* gout = gview(A.out);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int c;
    const int o = out_tile(id, t, c);
    if (o < 0) continue;
    const uint8_t* p = fin + 2 * (id % kMxPairs) * kMxSlotBytes + tail_at(id, t);
    *(PENCIL_GLOBAL u64x2*)(gout + o * ct_stride + c * pt_stride + ln + 2 * (id % kMxPairs)) =
        u64x2{*(const uint64_t*)p, *(const uint64_t*)(p + kMxSlotBytes)};
  }
}

__device__ __forceinline__ void mx_work(uint8_t* lds, const MacArgs& A, const Geo& G, const Consts& C, int slot_group,
                                        int tile) {
  if (C.fold60)
    mx_tile<true>(lds, A, G, C, slot_group, tile);
  else
    mx_tile<false>(lds, A, G, C, slot_group, tile);
}

// Work items: slot groups x tiles, the tiles of one slot group adjacent (they
// share operand rows) and neighbouring slot groups, which share 128-byte
// lines, next to each other on one XCD.
__global__ void __launch_bounds__(kMxThreads, 4) k_mac_matrix(MacArgs A, Geo G, Consts C, int tiles, int64_t total) {
  extern __shared__ __align__(16) uint8_t mx_lds[];
  const int w = (int)xcd_work(blockIdx.x, total);
  mx_work(mx_lds, A, G, C, w / tiles, w % tiles);
}

__global__ void __launch_bounds__(kMxThreads, 4) k_step_mac_matrix(const StepSeg* __restrict__ segs, int nseg,
                                                            const Consts* __restrict__ consts) {
  extern __shared__ __align__(16) uint8_t mx_lds[];
  const StepSeg& S = segs[find_seg(segs, nseg, blockIdx.x)];
  const int64_t local = (int64_t)blockIdx.x - S.block_begin;
  const int tiles = mac_matrix_tiles(S.mac.n_terms, S.mac.m_rows, S.G.nR);
  const int64_t work = S.slot_blocks * tiles, padded = (work + 7) & ~(int64_t)7;
  const int w = (int)xcd_work(local, padded);
  if (w >= work) return;
  mx_work(mx_lds, S.mac, S.G, consts[S.ctx], w / tiles, w % tiles);
}

hipError_t launch_mac_matrix(const MacArgs& A, const Geo& G, const Consts& C, hipStream_t s) {
  if (A.n_terms < 1 || A.n_terms > 2 || !A.term[0].a_is_ct || (A.n_terms == 2 && A.term[1].a_is_ct))
    return hipErrorInvalidValue;
  const int tiles = mac_matrix_tiles(A.n_terms, A.m_rows, G.nR);
  const int64_t total = mac_matrix_groups(C.n, C.L) * tiles;
  if (total <= 0) return hipSuccess;
  if (total > kMxMaxBlocks) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_mac_matrix, dim3((unsigned)total), dim3(kMxThreads), kMxLds, s, A, G, C, tiles, total);
  return hipGetLastError();
}

hipError_t launch_step_mac_matrix(const StepPhase& P, int64_t blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  if (blocks > kMxMaxBlocks) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(k_step_mac_matrix, dim3((unsigned)blocks), dim3(kMxThreads), kMxLds, s, P.segs, P.nseg, P.consts);
  return hipGetLastError();
}

hipError_t configure_lds_macx() {
  hipError_t a = hipFuncSetAttribute((const void*)k_mac_matrix, hipFuncAttributeMaxDynamicSharedMemorySize, kMxLds);
  hipError_t b = hipFuncSetAttribute((const void*)k_step_mac_matrix, hipFuncAttributeMaxDynamicSharedMemorySize, kMxLds);
  return a != hipSuccess ? a : b;
}

}  // namespace pencil
