// Exact Z_t packed correlation on the int8 matrix cores.
#include <climits>

#include "mx_common.h"

namespace pencil {

// out[m, r, y, x] = sum_{k, dy, dx} A[m, k, y+dy, x+dx] K[r, k, dy, dx] mod t for
// t < 2^46, as a tiled contraction of 64 x 64 outputs ((m, y, x) rows, r columns)
// per workgroup.  A value v < t is six signed digits d_i in [-128, 128), v = sum
// d_i 2^(8 i); a product has eleven diagonals D_s = sum_{i + j = s} a_i b_j, each
// an int32 matrix accumulator over the contraction (|D_s| <= 6 2^14 per index, so
// kZxMaxK indices stay below 2^31), and the sum is recombined exactly in 128
// bits and reduced mod t once per output.
//
// One v_mfma_i32_16x16x64_i8 takes four digits of 16 contraction indices: with K's
// digits reversed (R byte p = k_(5-p)) and W(o) bytes o .. o + 3 of R, A's digits
// 0-3 against W(o) give diagonal 5 - o (o = -3 .. 5), its digits 4-5 diagonal 9 -
// o (o = -1 .. 5): 16 instructions per 16 x 16 x 16 block.  512 threads stage 16
// indices of 64 A rows and 64 K rows per turn: 16 lanes take consecutive indices
// (coalesced along a contiguous contraction), each lane two rows of either side;
// digits go to LDS in the order the waves read them, in two buffers.  A wave
// multiplies 32 x 16 outputs.
//
// Grids too small to fill the GPU split the contraction over gridDim.y; the
// parts' residues are then added atomically to a zeroed output, which a last
// kernel reduces mod t.
//
// What bounds it: the staging's address and digit arithmetic (about as many
// cycles as the matrix instructions), and short contractions per workgroup.  64 ->
// 64 channels, 3 x 3, on 16 x 16, batch 64 (604 M multiply-adds): forward 334 us
// with the f64 matrix kernel, 48 us here; weight gradient 290 and 67 us.  The same
// on 32 x 32: 1289 and 174 us, 1744 and 169 us (28 T multiply-adds per second).
constexpr int kZxTile = 64, kZxKB = 16, kZxThreads = 512, kZxDiag = 11;
constexpr int kZxGroupBytes = kZxTile * 16 + 32;  // [64 rows][4 indices] of one digit half, padded by 8 banks
constexpr int kZxPlaneBytes = 4 * kZxGroupBytes;
constexpr int kZxOpBytes = 2 * kZxPlaneBytes;
constexpr int kZxBufBytes = 2 * kZxOpBytes;

template <int O, bool LO, bool HI>
__device__ __forceinline__ void zx_step(mx_v4i (&acc)[2][kZxDiag], const mx_v4i (&xl)[2], const mx_v4i (&xh)[2],
                                        const mx_u4 r0, const mx_u4 r1) {
  mx_v4i w;
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (int)mx_window<O>(r0[i], r1[i]);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (LO) acc[i][5 - O] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xl[i], w, acc[i][5 - O], 0, 0, 0);
    if constexpr (HI) acc[i][9 - O] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xh[i], w, acc[i][9 - O], 0, 0, 0);
  }
}

template <bool WIN>
__global__ void __launch_bounds__(kZxThreads, 2) k_zt_matrix(const int64_t* a, const int64_t* kt, int64_t* out, Geo G,
                                                             View AV, View KV, View OV, Consts C, DotStep D,
                                                             int col_blocks, int64_t per) {
  __shared__ __align__(16) uint8_t lds[2 * kZxBufBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ohw = G.OH * G.OW, P = G.M * ohw, R = G.R, kk = G.KH * G.KW;
  const int rb = (int)blockIdx.x / col_blocks, cb = (int)blockIdx.x - rb * col_blocks;
  const PENCIL_GLOBAL int64_t* ga = gview(a);
  const PENCIL_GLOBAL int64_t* gk = gview(kt);
  // staging: this thread's contraction index (mod 16) and rows rg, rg + 32
  const int rg = tid >> 4;
  int abase[2], kbase[2];  // element offsets (below 2^31, see the launcher)
  int ay[2], ax[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = rb * kZxTile + rg + 32 * i, col = cb * kZxTile + rg + 32 * i;
    const int rr = row < P ? row : 0;
    const int m = WIN ? rr / ohw : rr, rem = rr - m * ohw, y = WIN ? rem / G.OW : 0, x = WIN ? rem - y * G.OW : 0;
    ay[i] = row < P ? y - AV.pady : INT_MIN / 2;  // a padding row is outside for every window position
    ax[i] = x - AV.pad;
    abase[i] = m * (int)AV.s0 + (WIN ? (y - AV.pady) * (int)AV.sy + ax[i] * (int)AV.sx : 0);
    kbase[i] = col < R ? col * (int)KV.s0 : -1;
  }
  const int64_t ctot = (int64_t)G.K * kk;
  const int64_t c_begin = blockIdx.y * per, c_end = c_begin + per < ctot ? c_begin + per : ctot;
  int c = (int)c_begin + (tid & 15);
  int k = c, dy = 0, dx = 0;
  if constexpr (WIN) {
    k = c / kk;
    const int rem = c - k * kk;
    dy = rem / G.KW;
    dx = rem - dy * G.KW;
  }
  uint64_t va[2], vk[2];
  // the loads of 16 indices; entries outside the tensors or the range read as zero
  auto load = [&] {
    const bool live = c < c_end;
    if constexpr (WIN) {
      const int ky = KV.flip ? KV.KH - 1 - dy : dy, kx = KV.flip ? KV.KW - 1 - dx : dx;
      const int koff = k * (int)KV.s1 + ky * (int)KV.sy + kx * (int)KV.sx;
      const int aoff = k * (int)AV.s1 + dy * (int)AV.sy + dx * (int)AV.sx;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bool in = live && (uint32_t)(ay[i] + dy) < (uint32_t)AV.H && (uint32_t)(ax[i] + dx) < (uint32_t)AV.W;
        va[i] = in ? (uint64_t)ga[abase[i] + aoff] : 0;
        vk[i] = live && kbase[i] >= 0 ? (uint64_t)gk[kbase[i] + koff] : 0;
      }
      dx += D.ddx;
      if (dx >= G.KW) {
        dx -= G.KW;
        ++dy;
      }
      dy += D.ddy;
      if (dy >= G.KH) {
        dy -= G.KH;
        ++k;
      }
      k += D.dk;
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        va[i] = live && ay[i] >= 0 ? (uint64_t)ga[abase[i] + k * (int)AV.s1] : 0;
        vk[i] = live && kbase[i] >= 0 ? (uint64_t)gk[kbase[i] + k * (int)KV.s1] : 0;
      }
      k += kZxKB;
    }
    c += kZxKB;
  };
  auto store = [&](uint8_t* buf) {
    constexpr uint64_t k80 = 0x808080808080ull;
    uint8_t* p = buf + ((tid & 15) >> 2) * kZxGroupBytes + rg * 16 + (tid & 3) * 4;
#pragma unroll
    for (int i = 0; i < 2; ++i, p += 32 * 16) {
      const uint64_t da = (va[i] + k80) ^ k80, dk = (vk[i] + k80) ^ k80;
      const uint32_t kl = (uint32_t)dk, kh = (uint32_t)(dk >> 32);
      *(uint32_t*)p = (uint32_t)da;
      *(uint32_t*)(p + kZxPlaneBytes) = (uint32_t)(da >> 32);
      // digits 5 4 3 2, then 1 0 and two zeros
      *(uint32_t*)(p + kZxOpBytes) = __builtin_amdgcn_perm(kh, kl, 0x02030405u);
      *(uint32_t*)(p + kZxOpBytes + kZxPlaneBytes) = __builtin_amdgcn_perm(kh, kl, 0x0c0c0001u);
    }
  };
  mx_v4i acc[2][kZxDiag];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int s = 0; s < kZxDiag; ++s) acc[i][s] = mx_v4i{0, 0, 0, 0};
  const int wrow = (wave & 1) * 32, wcol = (wave >> 1) * 16;
  const int turns = (int)((c_end - c_begin + kZxKB - 1) / kZxKB);
  load();
  store(lds);
  __syncthreads();
  for (int t = 0; t < turns; ++t) {
    if (t + 1 < turns) load();
    const uint8_t* buf = lds + (t & 1) * kZxBufBytes + (lane >> 4) * kZxGroupBytes + (lane & 15) * 16;
    mx_v4i xl[2], xh[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      xl[i] = *(const mx_v4i*)(buf + (wrow + 16 * i) * 16);
      xh[i] = *(const mx_v4i*)(buf + (wrow + 16 * i) * 16 + kZxPlaneBytes);
    }
    const mx_u4 r0 = *(const mx_u4*)(buf + kZxOpBytes + wcol * 16);
    const mx_u4 r1 = *(const mx_u4*)(buf + kZxOpBytes + wcol * 16 + kZxPlaneBytes);
    zx_step<0, true, true>(acc, xl, xh, r0, r1);
    zx_step<4, true, true>(acc, xl, xh, r0, r1);
    zx_step<1, true, true>(acc, xl, xh, r0, r1);
    zx_step<2, true, true>(acc, xl, xh, r0, r1);
    zx_step<3, true, true>(acc, xl, xh, r0, r1);
    zx_step<5, true, true>(acc, xl, xh, r0, r1);
    zx_step<-1, true, true>(acc, xl, xh, r0, r1);
    zx_step<-2, true, false>(acc, xl, xh, r0, r1);
    zx_step<-3, true, false>(acc, xl, xh, r0, r1);
    if (t + 1 < turns) store(lds + ((t + 1) & 1) * kZxBufBytes);
    __syncthreads();
  }
  // a lane holds outputs (row 4 (lane / 16) + r, column lane % 16) of its tiles:
  // S = g0 + g1 2^32 + g2 2^64 >= 0 with signed groups g_h = sum_{s < 4} D_(4 h + s) 2^(8 s)
  int32_t m8 = 1 << 8, m16 = 1 << 16, m24 = 1 << 24;
  asm volatile("" : "+v"(m8), "+v"(m16), "+v"(m24));
  const int col = cb * kZxTile + wcol + (lane & 15);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int64_t g[3];
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        int64_t v = mx_mad(acc[i][4 * h + 2][r], m16, mx_mad(acc[i][4 * h + 1][r], m8, acc[i][4 * h][r]));
        if (4 * h + 3 < kZxDiag) v = mx_mad(acc[i][4 * h + 3][r], m24, v);
        g[h] = v;
      }
      uint64_t lo = (uint64_t)g[0], hi = (uint64_t)(g[0] >> 63);
      const uint64_t t1 = (uint64_t)g[1] << 32;
      lo += t1;
      hi += (uint64_t)(g[1] >> 32) + (lo < t1 ? 1 : 0) + (uint64_t)g[2];
      const uint64_t v = add_mod(mul_shoup(reduce64(hi, C.one_sh_t, C.t), C.r64t, C.r64t_sh, C.t),
                                 reduce64(lo, C.one_sh_t, C.t), C.t);
      const int row = rb * kZxTile + wrow + 16 * i + 4 * (lane >> 4) + r;
      if (row < P && col < R) {
        const int m = WIN ? row / ohw : row, rem = row - m * ohw, y = WIN ? rem / G.OW : 0, x = rem - y * G.OW;
        int64_t* o = out + ((int64_t)m * OV.s0 + (int64_t)col * OV.s1 + (WIN ? (int64_t)y * OV.sy + (int64_t)x * OV.sx : 0));
        if (gridDim.y == 1)
          *gview(o) = (int64_t)v;
        else
          atomicAdd((unsigned long long*)o, (unsigned long long)v);
      }
    }
}

__global__ void __launch_bounds__(256) k_zt_zero(int64_t* out, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) gview(out)[i] = 0;
}

__global__ void __launch_bounds__(256) k_zt_mod(int64_t* out, int64_t count, Consts C) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) gview(out)[i] = (int64_t)reduce64((uint64_t)gview(out)[i], C.one_sh_t, C.t);
}

hipError_t launch_zt_matrix(const int64_t* a, const int64_t* k, int64_t* out, const Geo& G, const View& AV,
                            const View& KV, const View& OV, const Consts& C, bool win, hipStream_t s) {
  const int64_t rows = (int64_t)G.M * G.OH * G.OW, ctot = (int64_t)G.K * G.KH * G.KW, count = rows * G.R;
  const int64_t rbs = (rows + kZxTile - 1) / kZxTile, cbs = ((int64_t)G.R + kZxTile - 1) / kZxTile;
  const int64_t splits = zt_matrix_splits(rbs * cbs, ctot, OV.s1 == 1);
  const int64_t turns = (ctot + kZxKB - 1) / kZxKB, per = (turns + splits - 1) / splits * kZxKB;
  const int kk = G.KH * G.KW;
  const DotStep D{kZxKB / kk, (kZxKB % kk) / G.KW, (kZxKB % kk) % G.KW, 0};
  const dim3 grid((unsigned)(rbs * cbs), (unsigned)((ctot + per - 1) / per));
  const dim3 flat((unsigned)((count + 255) / 256));
  if (grid.y > 1) hipLaunchKernelGGL(k_zt_zero, flat, dim3(256), 0, s, out, count);
  if (win)
    hipLaunchKernelGGL(k_zt_matrix<true>, grid, dim3(kZxThreads), 0, s, a, k, out, G, AV, KV, OV, C, D, (int)cbs, per);
  else
    hipLaunchKernelGGL(k_zt_matrix<false>, grid, dim3(kZxThreads), 0, s, a, k, out, G, AV, KV, OV, C, D, (int)cbs, per);
  if (grid.y > 1) hipLaunchKernelGGL(k_zt_mod, flat, dim3(256), 0, s, out, count, C);
  return hipGetLastError();
}

}  // namespace pencil
