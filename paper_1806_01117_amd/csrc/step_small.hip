// One-launch step kernels for small batches (fp32, gfx950).
//
// A kernel launch costs ~3 us on its own here, so each recurrent step is one
// launch.  For a batch of 64 the gate GEMM (B x G*H x (D+H)) must still be
// spread over all 256 CUs, and what bounds a workgroup is the bytes it streams
// from L2 (~30 GB/s per workgroup), so the tile is the smallest that still
// covers the whole reduction: 16 batch rows x U hidden units, all G gates
// (U = 8 for the LSTM, i.e. 32 weight rows; U = 16 for the tanh RNN).  The 8
// waves of a workgroup split the reduction; their partial products meet in
// LDS and are summed in wave order (bit-reproducible), then one thread per
// (row, unit) runs the cell math.
//
// Within the workgroup's G*U columns the weight rows are gate-major:
// column n = g*U + u is row g*H + j0 + u of W, so the epilogue thread of unit
// u finds its gates at columns u, U+u, 2U+u, 3U+u.
//
// The adjoint launch of step t also computes hbar_{t+1} = zbar_{t+1} W_h for
// its (rows, units) tile, the one product that needs the previous launch's
// output; W_h is read through its transpose WhT[j][k] = W[k][D+j] so both
// products are row-contiguous in the reduction index.
//
// Loads.  A vector load costs by the 128-byte lines it touches, so one
// instruction reads 8 rows x 128 bytes (lane l: row l >> 3, bytes 16 (l & 7))
// of W, [x | h], zbar or W_h^T where the reduction is long, not the MFMA
// operand's 16 rows x 64 bytes (kept for short ones); each
// wave turns its rows into fragments through swizzled LDS tiles of its own (no
// workgroup barrier in the loop).  A row of x or h (and the weights' part that
// meets it) that ends in the middle of a 128-byte block reads zeros after it.
//
// Operands are fp32 (v_mfma_f32_16x16x4_f32, 4 per 16 bytes of a lane) or bf16
// (v_mfma_f32_16x16x32_bf16, one per 16 bytes): either way a block is 128
// bytes of an operand row, two fragments.  With bf16 the
// stored h, the copy of h_t for the weight gradient and zbar (the adjoint
// GEMMs' operand) are rounded to bf16 (nearest even); accumulation, the cell
// state and its adjoint stay fp32.
#include <hip/hip_runtime.h>

#include "ambptt.h"
#include "kernels.hpp"
#include "mfma.hpp"

namespace ambptt {
namespace {

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return mfma_f32_16x16x4(a, b, c); }

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

template <class T>
struct Op;
template <>
struct Op<float> {
  using V = f4;
  static constexpr int CW = 16;  // reduction indices per chunk
  static __device__ __forceinline__ f4 mma(const V& a, const V& b, f4 c) {
    c = mfma4(a.x, b.x, c);
    c = mfma4(a.y, b.y, c);
    c = mfma4(a.z, b.z, c);
    return mfma4(a.w, b.w, c);
  }
  static __device__ __forceinline__ float store(float v) { return v; }
  static __device__ __forceinline__ float load(float v) { return v; }
};
template <>
struct Op<__bf16> {
  using V = bf16x8;
  static constexpr int CW = 32;
  static __device__ __forceinline__ f4 mma(const V& a, const V& b, f4 c) {
    return mfma_bf16_16x16x32(a, b, c);
  }
  static __device__ __forceinline__ __bf16 store(float v) { return (__bf16)v; }  // nearest even
  static __device__ __forceinline__ float load(__bf16 v) { return (float)v; }
};

constexpr int kWaves = 8;
constexpr int kU = 2;  // chunks per prefetch group

// acc[nb] += sum over chunks [c0, c1) of a(ch) . b(ch, nb); loads run one group
// of kU chunks ahead of the MFMAs.
template <class T, int NB, class LA, class LB>
__device__ __forceinline__ void chunks(int c0, int c1, f4 (&acc)[NB], LA la, LB lb) {
  using V = typename Op<T>::V;
  if (c0 >= c1) return;
  V a[kU], b[kU][NB];
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int ch = min(c0 + u, c1 - 1);
    a[u] = la(ch);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) b[u][nb] = lb(ch, nb);
  }
  for (int g = c0; g < c1; g += kU) {
    V an[kU], bn[kU][NB];
    const bool more = g + kU < c1;
    if (more) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int ch = min(g + kU + u, c1 - 1);
        an[u] = la(ch);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) bn[u][nb] = lb(ch, nb);
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (g + u < c1) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = Op<T>::mma(a[u], b[u][nb], acc[nb]);
      }
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        a[u] = an[u];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) b[u][nb] = bn[u][nb];
      }
    }
  }
}

constexpr int kS = 2;          // blocks of loads in flight per wave
constexpr int kTile = 2048;    // one 16-row x 128-byte scratch tile
constexpr unsigned kPast = 0x7f000000u;  // an offset past any Rows8

typedef unsigned int u4v __attribute__((ext_vector_type(4)));

// Eight consecutive rows of an operand from `base` on (bytes past the last
// row read zero); `stride` bytes from row to row.  The range check takes the
// sum of a load's two offsets, without wrapping: rows that are all past the
// batch (no bytes) read zero at any offset.
struct Rows8 {
  unsigned long long base;
  unsigned bytes;
  __device__ __forceinline__ u4v load(unsigned voff, unsigned soff) const {
    return __builtin_amdgcn_raw_buffer_load_b128(
        __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000), voff, soff, 0);
  }
};
__device__ __forceinline__ Rows8 rows8(const void* p, size_t row0, int rows, size_t stride) {
  const unsigned long long q = (unsigned long long)p + row0 * stride;
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(q)), hi = __builtin_amdgcn_readfirstlane(unsigned(q >> 32));
  return {((unsigned long long)hi << 32) | lo,
          unsigned(__builtin_amdgcn_readfirstlane(unsigned(size_t(max(0, min(rows, 8))) * stride)))};
}

// acc[nb] += the wave's blocks [c0, c1) of A (16 rows) and B (16 rows per
// column block nb).  ld(blk, v) loads a block's 2 + 2 NB pieces of 8 rows: A's
// rows 0-7 and 8-15, then B's.
template <class T, int NB, class LD>
__device__ __forceinline__ void blocks(int c0, int c1, char* scr, f4 (&acc)[NB], LD ld) {
  using V = typename Op<T>::V;
  if (c0 >= c1) return;
  const int lane = threadIdx.x & 63, t = lane >> 3, k = lane & 7, r = lane & 15, q = lane >> 4;
  // row t's 16-byte piece k lies in slot k ^ (t & 7) of the row
  const int w0 = t * 128 + 16 * (k ^ t), r0 = r * 128 + 16 * (q ^ (r & 7)), r1 = r * 128 + 16 * ((q + 4) ^ (r & 7));
  u4v v[kS][2 + 2 * NB];
#pragma unroll
  for (int s = 0; s < kS; ++s) ld(min(c0 + s, c1 - 1), v[s]);
  for (int c = c0; c < c1; c += kS) {
#pragma unroll
    for (int s = 0; s < kS; ++s) {
      if (c + s >= c1) break;
#pragma unroll
      for (int i = 0; i < 2 + 2 * NB; ++i) *(u4v*)(scr + (i >> 1) * kTile + (i & 1) * 1024 + w0) = v[s][i];
      if (c + s + kS < c1) ld(c + s + kS, v[s]);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const V a = *(const V*)(scr + (h ? r1 : r0));
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = Op<T>::mma(a, *(const V*)(scr + (1 + nb) * kTile + (h ? r1 : r0)), acc[nb]);
      }
      __builtin_amdgcn_wave_barrier();  // the tiles are read before the next block is stored
    }
  }
}

// CACHED (adjoint): the step's pre-activations are kept (a.zc_in) and its
// gate product is not formed again.
// RG, RH: the gate product's and the h-adjoint product's loads go by rows
// through LDS (blocks), else by fragments (chunks).
template <class T, int G, int MODE, bool RG, bool RH, bool CACHED>
__global__ __launch_bounds__(64 * kWaves) void step_small(StepArgs a) {
  constexpr size_t E = sizeof(T);
  using V = typename Op<T>::V;
  constexpr int CW = Op<T>::CW, LE = CW / 4;  // a chunk's elements, a lane's (16 bytes)
  constexpr int U = (G == 4) ? 8 : 16;  // units per workgroup
  constexpr int NC = G * U;             // gate columns (32 or 16)
  constexpr int NB = NC / 16;           // MFMA column blocks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int B = a.B, D = a.D, H = a.H, GH = G * H, K1 = D + H;
  const unsigned lrow = lane >> 3, lpiece = 16 * (lane & 7);  // this lane's row and bytes of a load
  // XCD-aware tile order.  Workgroups are dealt to the 8 XCDs round-robin by
  // id, so ids with equal id % 8 share an L2.  Tiles are numbered unit-group
  // major (w = ug * mtiles + mt) and each XCD takes a contiguous run of them:
  // the row tiles of one unit group then read its weight rows through one L2.
  const int mtiles = (B + 15) / 16, ntile = mtiles * (H / U);
  const int per = (ntile + 7) / 8;
  const int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (w >= ntile) return;  // grid padding (the whole workgroup leaves together)
  const int m0 = (w % mtiles) * 16;
  const int j0 = (w / mtiles) * U;
  const int wg_slot = w;   // loss accumulator of this tile
  const int row = min(m0 + r, B - 1);  // chunks: rows >= B are loaded clamped, their results dropped

  __shared__ float zs[CACHED ? 1 : kWaves][16][NC + 1];
  __shared__ float hs[kWaves][16][17];
  __shared__ __attribute__((aligned(16))) char scratch[RG || RH ? kWaves : 1][(1 + NB) * kTile];
  char* scr = scratch[RG || RH ? wave : 0];

  if (MODE != kFinal && !CACHED) {
    f4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (RG) {
      // blocks of x, then of h
      const unsigned xrow = unsigned(D * E), hrow = unsigned(H * E), wrow = xrow + hrow;  // row bytes
      const int nx = int(xrow + 127) / 128, nblk = nx + int(hrow + 127) / 128;
      const int c0 = (nblk * wave) / kWaves, c1 = (nblk * (wave + 1)) / kWaves;
      const int xh = xrow % 128 ? nx - 1 : -1, hh = hrow % 128 ? nblk - 1 : -1;  // blocks that end in the middle
      const Rows8 xr[2] = {rows8(a.x, m0, B - m0, xrow), rows8(a.x, m0 + 8, B - m0 - 8, xrow)};
      const Rows8 hr[2] = {rows8(a.h, m0, B - m0, hrow), rows8(a.h, m0 + 8, B - m0 - 8, hrow)};
      Rows8 wr[2 * NB];  // 8 columns: the LSTM's units of one gate, or half the RNN's units
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) wr[i] = rows8(a.W, G == 4 ? size_t(i) * H + j0 : size_t(j0 + 8 * i), 8, wrow);
      const unsigned xv = lrow * xrow + lpiece, hv = lrow * hrow + lpiece, wv = lrow * wrow + lpiece;
      blocks<T, NB>(c0, c1, scr, acc, [&](int blk, u4v* v) {
        const bool inx = blk < nx;  // selects, not branches: the same for the whole wave
        const bool cut = (blk == xh || blk == hh) && lpiece >= 64;
        const unsigned so = unsigned(inx ? blk : blk - nx) * 128u;
        const unsigned av = cut ? kPast : inx ? xv : hv, bv = cut ? kPast : wv;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const Rows8 s{inx ? xr[i].base : hr[i].base, inx ? xr[i].bytes : hr[i].bytes};
          v[i] = s.load(av, so);
        }
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) v[2 + i] = wr[i].load(bv, so + (inx ? 0u : xrow));
      });
    } else {
      const int nch = K1 / CW;
      const int c0 = (nch * wave) / kWaves, c1 = (nch * (wave + 1)) / kWaves;
      const T* xr = (const T*)a.x + (size_t)row * D;
      const T* hr = (const T*)a.h + (size_t)row * H;
      const T* wr[NB];
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = nb * 16 + r;  // column of this lane in block nb
        wr[nb] = (const T*)a.W + (size_t)((n / U) * H + j0 + (n % U)) * K1;
      }
      chunks<T, NB>(c0, c1, acc,
                    [&](int ch) -> V {
                      const int k = ch * CW + LE * q;
                      return *(const V*)(ch * CW < D ? xr + k : hr + (k - D));
                    },
                    [&](int ch, int nb) -> V { return *(const V*)(wr[nb] + ch * CW + LE * q); });
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 4; ++v) zs[wave][4 * q + v][nb * 16 + r] = acc[nb][v];
  }
  const bool do_hbar = (MODE == kFinal) || (MODE == kAdjoint && !a.first);
  if (do_hbar) {
    f4 acc[1] = {f4{0.f, 0.f, 0.f, 0.f}};
    if constexpr (RH) {
      const unsigned zrow = unsigned(GH * E);
      const int nblk = int(zrow + 127) / 128, zh = zrow % 128 ? nblk - 1 : -1;
      const int c0 = (nblk * wave) / kWaves, c1 = (nblk * (wave + 1)) / kWaves;
      const Rows8 zr[2] = {rows8(a.zbar_in, m0, B - m0, zrow), rows8(a.zbar_in, m0 + 8, B - m0 - 8, zrow)};
      // U units: 8 (columns 8 .. 15 of the product are unused) or 16
      const Rows8 tr[2] = {rows8(a.WhT, j0, 8, zrow), rows8(a.WhT, j0 + 8, U == 16 ? 8 : 0, zrow)};
      const unsigned zv = lrow * zrow + lpiece;
      blocks<T, 1>(c0, c1, scr, acc, [&](int blk, u4v* v) {
        const unsigned vo = blk == zh && lpiece >= 64 ? kPast : zv, so = unsigned(blk) * 128u;
        v[0] = zr[0].load(vo, so);
        v[1] = zr[1].load(vo, so);
        v[2] = tr[0].load(vo, so);
        v[3] = U == 16 ? tr[1].load(vo, so) : u4v{0u, 0u, 0u, 0u};
      });
    } else {
      const int nch = GH / CW;
      const int c0 = (nch * wave) / kWaves, c1 = (nch * (wave + 1)) / kWaves;
      const T* zr = (const T*)a.zbar_in + (size_t)row * GH;
      // U units; lanes r >= U (LSTM) repeat units so no extra rows are fetched
      const T* wt = (const T*)a.WhT + (size_t)(j0 + (r % U)) * GH;
      chunks<T, 1>(c0, c1, acc, [&](int ch) -> V { return *(const V*)(zr + ch * CW + LE * q); },
                   [&](int ch, int) -> V { return *(const V*)(wt + ch * CW + LE * q); });
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) hs[wave][4 * q + v][r] = acc[0][v];
  }
  __syncthreads();

  // epilogue: thread (m, u) for m < 16, u < U
  float lterm = 0.f;
  if (tid < 16 * U) {
#pragma clang fp contract(on)  // the same bits with and without the gate product
    const int ml = tid / U, u = tid % U;
    const int m = m0 + ml, j = j0 + u;
    if (m < B) {
      const size_t o = (size_t)m * H + j;
      float hbar = 0.f;
      if (do_hbar) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) hbar += hs[w][ml][u];
      }
      if (MODE == kFinal) {
        a.dh0[o] = hbar;
        if (G == 4) a.dc0[o] = a.cbar_in[o];
      } else {
        float z[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (CACHED) {
            z[g] = a.zc_in[(size_t)m * GH + g * H + j];
          } else {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) s += zs[w][ml][g * U + u];
            z[g] = s + a.bias[g * H + j];
            if (MODE == kForward && a.zc_out) a.zc_out[(size_t)m * GH + g * H + j] = z[g];
          }
        }
        float h1, c1 = 0.f, tc = 0.f, ig = 0.f, fg = 0.f, gg = 0.f, og = 0.f, cold = 0.f;
        if (G == 4) {
          ig = sigm(z[0]);
          fg = sigm(z[1 % G]);
          gg = tanhf(z[2 % G]);
          og = sigm(z[3 % G]);
          cold = a.c[o];
          c1 = fg * cold + ig * gg;
          tc = tanhf(c1);
          h1 = og * tc;
        } else {
          h1 = tanhf(z[0]);
        }
        const T h1s = Op<T>::store(h1);  // the stored state
        if (MODE == kForward) {
          ((T*)a.h_out)[o] = h1s;
          if (G == 4) a.c_out[o] = c1;
        } else {
          const float hl = Op<T>::load(h1s);  // loss and seed read the stored h_{t+1}
          float sd = 0.f;
          if (a.loss == AMBPTT_LOSS_MEAN_SQ_ALL) {
            sd = 2.f * hl * a.inv_bh;
            lterm = hl * hl;
          } else if (a.last) {
            if (a.loss == AMBPTT_LOSS_HALF_SQ_LAST) {
              sd = hl;
              lterm = hl * hl;
            } else {
              sd = a.inv_bh;
              lterm = hl;
            }
          }
          const float hb = hbar + sd;
          T* zo = (T*)a.zbar_out + (size_t)m * GH + j;
          if (G == 4) {
            const float cb = a.first ? 0.f : a.cbar_in[o];
            const float ob = hb * tc;
            const float ch = cb + hb * og * (1.f - tc * tc);
            zo[0] = Op<T>::store(ch * gg * ig * (1.f - ig));
            zo[H] = Op<T>::store(ch * cold * fg * (1.f - fg));
            zo[2 * H] = Op<T>::store(ch * ig * (1.f - gg * gg));
            zo[3 * H] = Op<T>::store(ob * og * (1.f - og));
            a.cbar_out[o] = ch * fg;
          } else {
            zo[0] = Op<T>::store(hb * (1.f - h1 * h1));
          }
          ((T*)a.hwin_out)[o] = ((const T*)a.h)[o];
        }
      }
    }
  }
  if (MODE == kAdjoint) {
    // threads >= 16 U hold 0; waves beyond the epilogue contribute nothing
    const float s = wave_sum(lterm);
    __shared__ float wsum[kWaves];
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += wsum[w];
      a.loss_acc[wg_slot] += (double)t;
    }
  }
}

}  // namespace

void step_small_grid(int G, int B, int H, dim3* grid, dim3* block) {
  const int U = (G == 4) ? 8 : 16;
  const int ntile = ((B + 15) / 16) * (H / U);
  *grid = dim3(8 * ((ntile + 7) / 8), 1, 1);
  *block = dim3(64 * kWaves, 1, 1);
}

hipError_t launch_step_small(int G, int bf16, int mode, const StepArgs& a, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1) {
  dim3 grid, block;
  step_small_grid(G, a.B, a.H, &grid, &block);
  // By rows where the reduction is long enough (128-byte blocks of it): with
  // one or two blocks per wave the trip through LDS costs more than the lines
  // it saves.  Forward by rows / by fragments: 40 blocks (32 x 1024, D 256, fp32)
  // 9.5 / 11.5 us, 30 (tanh RNN, 64 x 896) 6.9 / 7.0, 17.5 (16 x 544) 7.1 / 6.6,
  // 9 (5 x 80) 6.2 / 5.7.  Adjoint, h-adjoint product: 128 blocks 14.6 / 21.0,
  // 32 (20 x 512, bf16) 6.0 / 8.4, 16 (40 x 256, bf16) 5.4 / 6.0, 10 (5 x 80)
  // 6.6 / 6.2.
  const size_t e = bf16 ? 2 : 4;
  const bool rg = size_t(a.D + a.H) * e >= 20 * 128, rh = size_t(G) * a.H * e >= 16 * 128;
#define AMB_K(T_, G_, M_, RG_, RH_, C_) \
  hipExtLaunchKernelGGL((step_small<T_, G_, M_, RG_, RH_, C_>), grid, block, 0, s, e0, e1, 0, a)
#define AMB_T(T_, G_)                                                          \
  do {                                                                         \
    if (mode == kForward) {                                                    \
      if (rg) AMB_K(T_, G_, kForward, true, false, false);                     \
      else AMB_K(T_, G_, kForward, false, false, false);                       \
    } else if (mode == kFinal) {                                               \
      if (rh) AMB_K(T_, G_, kFinal, false, true, false);                       \
      else AMB_K(T_, G_, kFinal, false, false, false);                         \
    } else if (a.zc_in) {                                                      \
      if (rh) AMB_K(T_, G_, kAdjoint, false, true, true);                      \
      else AMB_K(T_, G_, kAdjoint, false, false, true);                        \
    } else if (rg) {                                                           \
      if (rh) AMB_K(T_, G_, kAdjoint, true, true, false);                      \
      else AMB_K(T_, G_, kAdjoint, true, false, false);                        \
    } else {                                                                   \
      if (rh) AMB_K(T_, G_, kAdjoint, false, true, false);                     \
      else AMB_K(T_, G_, kAdjoint, false, false, false);                       \
    }                                                                          \
  } while (0)
  if (bf16) {
    if (G == 4) AMB_T(__bf16, 4);
    else AMB_T(__bf16, 1);
  } else {
    if (G == 4) AMB_T(float, 4);
    else AMB_T(float, 1);
  }
#undef AMB_T
#undef AMB_K
  return hipGetLastError();
}

}  // namespace ambptt
