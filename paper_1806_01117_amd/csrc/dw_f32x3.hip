// fp32 weight-gradient window on the bf16 matrix cores (gfx950).
//
// dW[k][c] (+)= sum_r Z[r][k] X[r][c], db[k] (+)= sum_r Z[r][k] over the R
// rows of one window; Z = zbar [R][GH], X = [x | h] [R][D + H], both stored
// with the reduction index r as the row.  Operands are split in three bf16
// parts and multiplied as in gemm_f32x3.hip (f32x3.hpp has the stage
// pipeline).  A workgroup owns a TM x TN tile of dW; a stage is 32 rows.
//
// Both operands are split on their way to LDS.  An MFMA operand wants 8
// consecutive r of one column per lane, so a thread reads 4 rows of 4 (Z) or
// 2 (X) neighbouring columns, and after the split the 4 rows of one column are
// the 8 bytes that it writes per plane: the transpose costs no instruction.
// The 32 lanes of a half wave read 512 (Z) or 256 (X) consecutive bytes of a
// row.  In LDS the 16-column blocks are 16 bytes further apart than their
// size, so that a write's lanes spread over all banks.
//
// db comes from the Z values that the tiles of the first 128 columns load
// anyway: a thread sums its own rows, and the 8 threads of a column are added
// in order.
//
// Bound: the matrix cores, 63 % busy in the 4096-LSTM's window at the 1.8 GHz
// that this load leaves of 2.4 (MFMAs alone on such operands run at 2.0 GHz);
// its waves wait a quarter of the time.  That window (16384 x 5120, 8192 rows,
// 8.2 TFLOP of bf16 products) takes 7.0 ms against 10.8-11.6 ms on fp32 MFMAs,
// 1.17 PFLOP/s; 4096 x 1120 over 7200 rows 0.51 ms against 0.99; 4096 x 1280
// over 1024 rows 77 us against 124; one fp32 residual MLP layer, 1040 x 1040
// over 70 rows, 9.5 us against 14.0; 320 x 288 over 320 rows 21 us against 34.
#include <hip/hip_runtime.h>

#include "f32x3.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace ambptt {
namespace {

constexpr int kBlkP = kBlk + 16;  // padded block stride in LDS

template <int TM, int TN, int WM, int WN>
struct DwTile {
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int MI = TM / WM / 16, NI = TN / WN / 16;
  static constexpr int ABYTES = TM / 16 * kBlkP, STAGE = ABYTES + TN / 16 * kBlkP;
  static constexpr int LZ = TN + 4;
  static constexpr int LDS = 2 * STAGE > TM * LZ * 4 ? 2 * STAGE : TM * LZ * 4;
  // wave w: r 8 g .. +7 with g = w / (NW / 4); its lanes 32 column groups x 2 halves of 4 rows
  static_assert(TM == 32 * NW && TN == 16 * NW, "one column group of each operand per thread");

  template <bool BIAS>
  static __device__ __forceinline__ void body(const DwArgs& a, int k0, int c0, char* lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, q = lane >> 4;
    const int D = a.D, H = a.H, GH = a.GH, R = a.R, N = D + H;
    const int g = wave / (NW / 4), half = lane >> 5, cg = (wave % (NW / 4)) * 32 + (lane & 31);
    const int r0 = 8 * g + 4 * half;  // the thread's first row of a stage

    // Z: rows at or past R read as zero (the buffer ends there); columns past
    // GH read something, their results are unused
    const unsigned zbytes = unsigned(R) * unsigned(GH) * 4u;
    const unsigned zoff = (unsigned(r0) * unsigned(GH) + unsigned(k0 + 4 * cg)) * 4u;
    const int aoff = (cg >> 2) * kBlkP + (16 * g + 4 * (cg & 3)) * 16 + 8 * half;
    // X: rows past the last read it again, against zeros of Z
    const int c = c0 + 2 * cg;
    const float* xb = c < D ? (const float*)a.x + c : (const float*)a.hwin + (c < N ? c - D : 0);
    const int ldx = c < D ? D : H;
    const int boff = ABYTES + (cg >> 3) * kBlkP + (16 * g + 2 * (cg & 7)) * 16 + 8 * half;

    f4 zr[4];
    f2 xr[4];
    float bs[4] = {0.f, 0.f, 0.f, 0.f};
    auto gload = [&](int st, int p) {  // piece 1: Z, piece 2: X
      if (p == 1) {
        const __amdgpu_buffer_rsrc_t rz = rsrc(a.zbar, zbytes);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          zr[e] = __builtin_bit_cast(f4, bload(rz, zoff, unsigned(st * kSt + e) * unsigned(GH) * 4u));
      } else if (p == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e) xr[e] = *(const f2*)(xb + (size_t)min(st * kSt + r0 + e, R - 1) * ldx);
      }
    };
    auto column = [&](char* d, float v0, float v1, float v2, float v3) {
      u2v p0, p1, p2;
      unsigned t0, t1, t2;
      split2(v0, v1, t0, t1, t2);
      p0.x = t0, p1.x = t1, p2.x = t2;
      split2(v2, v3, t0, t1, t2);
      p0.y = t0, p1.y = t1, p2.y = t2;
      *(u2v*)d = p0;
      *(u2v*)(d + kFrag) = p1;
      *(u2v*)(d + 2 * kFrag) = p2;
    };
    auto put = [&](int buf, int p) {  // pieces 0, 1: columns 0-1 and 2-3 of Z; 2: X
      char* s = lds + buf * STAGE;
      if (p < 2) {
        const float sc = buf ? -kScale : kScale;
#pragma unroll
        for (int j = 2 * p; j < 2 * p + 2; ++j) {
          if (BIAS) bs[j] += (zr[0][j] + zr[1][j]) + (zr[2][j] + zr[3][j]);
          column(s + aoff + 16 * j, zr[0][j] * sc, zr[1][j] * sc, zr[2][j] * sc, zr[3][j] * sc);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          column(s + boff + 16 * j, xr[0][j] * kScale, xr[1][j] * kScale, xr[2][j] * kScale, xr[3][j] * kScale);
      }
    };

    f4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    x3_pipeline<MI, NI, 3, STAGE, kBlkP>(lds, wm * MI * kBlkP + lane * 16, ABYTES + wn * NI * kBlkP + lane * 16, 0,
                                         (R + kSt - 1) / kSt, gload, put, acc);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] *= kUnscale;
    if (any_bad(acc)) {  // fp32 MFMAs over 4 rows each, straight from global memory
      const float* zc[MI];
      const float* xc[NI];
      int lx[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) zc[i] = (const float*)a.zbar + min(k0 + (wm * MI + i) * 16 + r, GH - 1);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int cc = min(c0 + (wn * NI + j) * 16 + r, N - 1);
        xc[j] = cc < D ? (const float*)a.x + cc : (const float*)a.hwin + (cc - D);
        lx[j] = cc < D ? D : H;
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
      for (int rr = 0; rr < R; rr += 4) {
        const int row = rr + q;
        const bool in = row < R;  // rows past R: zero on both sides
        float zv[MI], xv[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) zv[i] = in ? zc[i][(size_t)row * GH] : 0.f;
#pragma unroll
        for (int j = 0; j < NI; ++j) xv[j] = in ? xc[j][(size_t)row * lx[j]] : 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mfma_f32_16x16x4(zv[i], xv[j], acc[i][j]);
      }
    }

    // the tile through LDS: 16 bytes of dW per lane
    float* t = (float*)lds;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          t[((wm * MI + i) * 16 + 4 * q + v) * LZ + (wn * NI + j) * 16 + r] = acc[i][j][v];
    __syncthreads();
    constexpr int TPR = TN / 4;  // threads per row
    const int cl = 4 * (tid % TPR);
    if (c0 + cl < N) {
#pragma unroll 4
      for (int row = tid / TPR; row < TM; row += NT / TPR) {
        if (k0 + row >= GH) break;
        f4* d = (f4*)(a.dW + (size_t)(k0 + row) * N + c0 + cl);
        f4 o = *(const f4*)(t + row * LZ + cl);
        if (a.accumulate) o += *d;
        *d = o;
      }
    }
    if (BIAS) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 4; ++j) t[(2 * g + half) * TM + 4 * cg + j] = bs[j];
      __syncthreads();
      if (tid < TM && k0 + tid < GH) {
        float s = t[tid];
#pragma unroll
        for (int e = 1; e < 8; ++e) s += t[e * TM + tid];
        a.db[k0 + tid] = a.accumulate ? a.db[k0 + tid] + s : s;
      }
    }
  }
};

template <int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void dw_f32x3(DwArgs a) {
  using T = DwTile<TM, TN, WM, WN>;
  __shared__ __attribute__((aligned(16))) char lds[T::LDS];
  // consecutive workgroups take consecutive k tiles: an XCD's share of a
  // round is then an (8-apart) set of k tiles against a few column tiles
  if (blockIdx.y == 0) T::template body<true>(a, blockIdx.x * TM, 0, lds);
  else T::template body<false>(a, blockIdx.x * TM, blockIdx.y * TN, lds);
}

}  // namespace

bool dw_f32x3_pays(const DwArgs& a) {
  // a short window of a small gradient is two stages and their prologue here:
  // 208 x 208 over 18 rows 8.5 us, dw_lds_f32 7.0
  return a.R > 64 || (a.GH >= 256 && a.D + a.H >= 256);
}

bool dw_f32x3_fits(const DwArgs& a) {
  // Z's offsets are 32-bit, those past its end included: stages go in pairs
  // and are loaded two ahead (db takes in the first of these two, whose rows
  // must read zero), and a tile's columns may end 255 past GH
  const long long stages = (a.R + kSt - 1ll) / kSt;
  const unsigned long long rows = (stages + stages % 2 + 2ull) * kSt;
  return a.R >= 1 && a.GH >= 16 && a.GH % 16 == 0 && a.D % 16 == 0 && a.H % 16 == 0 &&
         4ull * (rows * a.GH + 256) < (1ull << 32);
}

hipError_t launch_dw_f32x3(const DwArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (!dw_f32x3_fits(a)) return hipErrorInvalidValue;
  const int N = a.D + a.H;
  // A 32-row stage of a 256 x 128 tile takes 2.05 us, of two 128 x 64 tiles
  // sharing a CU 1.3 us: the fewer rounds times those (4096 x 1120: 144 tiles
  // in one round 496 us, 576 in two 588 us over 7200 rows)
  const auto rounds = [](int t, int slots) { return double((t + slots - 1) / slots); };
  const int big = ((a.GH + 255) / 256) * ((N + 127) / 128), small = ((a.GH + 127) / 128) * ((N + 63) / 64);
  if (2.05 * rounds(big, 256) <= 1.3 * rounds(small, 512)) {
    hipExtLaunchKernelGGL((dw_f32x3<256, 128, 4, 2>), dim3((a.GH + 255) / 256, (N + 127) / 128), dim3(512), 0, s, e0, e1,
                          0, a);
  } else {
    hipExtLaunchKernelGGL((dw_f32x3<128, 64, 4, 1>), dim3((a.GH + 127) / 128, (N + 63) / 64), dim3(256), 0, s, e0, e1, 0,
                          a);
  }
  return hipGetLastError();
}

}  // namespace ambptt
