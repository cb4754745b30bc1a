// fp32 products on the bf16 matrix cores (gfx950), for the large-batch
// recurrent cells: the gate product with the cell epilogue, the adjoint's
// h-adjoint product, and the copies of the weights that they read.
//
// An fp32 value is the exact sum of three bf16 values, a = a0 + a1 + a2 (each
// the nearest bf16 to what the ones before it leave: 3 x 8 significant bits
// and two signs cover fp32's 24).  Of the nine products of two such sums six
// are formed, a0 b0 + a0 b1 + a1 b0 + a1 b1 + a0 b2 + a2 b0.  With |a1| <=
// 2^-8 and |a2| <= 2^-17 of a's power of two, a1 b2 + a2 b1, the larger of
// what is left out, comes to at most 2^-24 of |a b| (2^-26.5 rms over random
// operands): no more than one rounding to fp32.  Every product of two bf16
// values is exact in the fp32 accumulators, so a 32-wide reduction step costs
// 6 v_mfma_f32_16x16x32_bf16 (96 cycles) where v_mfma_f32_16x16x4_f32 takes 8
// (256 cycles): six MFMAs summed from zero, then one VALU add to the
// accumulators (f32x3.hpp).
//
// Infinities, NaNs and sums past fp32's range do not split (inf - inf): every
// wave looks at its finished accumulators and, if one is not finite, forms
// its block again with fp32 MFMAs straight from global memory, so such inputs
// give what the fp32 kernels give.  Operands are scaled before they are split
// (f32x3.hpp), so that the split is exact down to fp32's subnormals.
//
// Data flow.  B (the weights, fixed for a pass) is split once per pass into
// fragment order: the 1 KiB that a wave's MFMA operand needs (16 rows x 32
// reduction indices, lane l: row l & 15, indices 8 (l >> 4) .. +7) lie
// together, three planes one after the other.  A (activations, or zbar) is
// read as fp32 rows and split on its way to LDS: the split's VALU work hides
// under the MFMAs, and the operand moves 4 bytes per element from L2 instead
// of 6.  LDS holds two stages of 32 reduction indices.
#include <hip/hip_runtime.h>

#include "ambptt.h"
#include "f32x3.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace ambptt {
namespace {

__host__ __device__ __forceinline__ int stages(int k) { return (k + kSt - 1) / kSt; }

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ void tile_of(int i, int mt, int nt, int* tm, int* tn) {
  if (nt % 8 == 0) {  // the row tiles of one column tile share an XCD
    const int xcd = i & 7, k = i >> 3;
    *tn = xcd * (nt >> 3) + k / mt;
    *tm = k % mt;
  } else {
    *tm = i % mt;
    *tn = i / mt;
  }
}

// One workgroup's product on a TM x TN tile: KG groups of WM x WN waves, each
// wave (TM / WM) x (TN / WN).  A: rows of [x | h], fp32; B: planes in fragment
// order.  A group takes its own part of the stages, in LDS buffers of its own
// (two groups give a SIMD two waves where the grid has fewer tiles than the
// chip has CUs); the groups' sums meet in the epilogue.
template <int TM, int TN, int WM, int WN, int KG>
struct Tile {
  static constexpr int NW = WM * WN, NT = 64 * NW;  // of one group
  static constexpr int MI = TM / WM / 16, NI = TN / WN / 16;
  static constexpr int PA = TM * 8 / NT;            // float4 of A per thread and stage
  static constexpr int PB = TN / 16 * 3 / NW;       // 16-byte pieces of B per thread and stage
  static constexpr int ABYTES = TM / 16 * kBlk, BBYTES = TN / 16 * kBlk;
  static constexpr int STAGE = ABYTES + BBYTES;
  static constexpr int LDS = KG * 2 * STAGE;
  static_assert(TM * 8 % NT == 0 && TN / 16 * 3 % NW == 0 && MI % 2 == 0, "whole loads per thread, row blocks in pairs");

  // A's rows are [x | h], x: [M][D], h: [M][H], each padded to whole stages
  // (TWO false: h alone).  bblk(b) is the packed block row of the tile's
  // 16-column block b; kb its 32-wide steps.  What a padded stage reads of A
  // past the end of a row meets zeros of B.  Stages st0 .. st1 - 1; len: the
  // most stages that any group of the workgroup has (their barriers are
  // common).  lds: the group's buffers.
  template <bool TWO, class BBlk>
  static __device__ __forceinline__ void run(const float* x, const float* h, int M, int D, int H, int m0,
                                             const char* Bp, unsigned bbytes, int kb, int st0, int st1, int len,
                                             BBlk bblk, char* lds, f4 (&acc)[MI][NI]) {
    const int tid = threadIdx.x % NT, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, q = lane >> 4;
    const int kx = TWO ? (D + kSt - 1) / kSt : 0;  // x's stages
    // A loader: thread t takes float4 t % 8 of rows t / 8 + (NT / 8) p of a
    // stage, so 8 lanes read one 128-byte line.  In LDS the 16 bytes of (row
    // r, indices 8 g .. +7) of a fragment lie in slot 16 g + (r ^ swz(g)),
    // swz = 0, 12, 4, 8: the four g of a write then fall on distinct banks,
    // and the lanes that one pass of a 16-byte read serves (0-3, 12-15 and
    // 20-27 of a half wave) still do
    const int lr = tid >> 3, c4 = tid & 7;
    const auto swz = [](int g) { return 4 * ((g >> 1) ^ (3 * (g & 1))); };
    const unsigned xbytes = unsigned(M) * unsigned(D) * 4u, hbytes = unsigned(M) * unsigned(H) * 4u;
    static_assert(NT % 128 == 0, "a thread's rows share their place in a fragment");
    const int aoff = (lr >> 4) * kBlk + (16 * (c4 >> 1) + ((lr & 15) ^ swz(c4 >> 1))) * 16 + 8 * (c4 & 1);
    // B loader: wave w moves PB of the tile's 3 TN / 16 plane fragments
    unsigned bsrc[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int f = wave * PB + p;  // block f / 3, plane f % 3
      bsrc[p] = unsigned(bblk(f / 3)) * unsigned(kb) * unsigned(kBlk) + unsigned(f % 3) * unsigned(kFrag);
    }
    const int boff = ABYTES + wave * PB * kFrag + lane * 16;

    // piece p of stage st to registers: float4 p of A, or (p = PA) the B
    // planes; of a stage past the last, its A again and zeros for B (the
    // stages go in pairs; of two groups and one stage the first has none, and
    // takes stage 0's A)
    f4 ra[PA];
    u4v rb[PB];
    auto gload = [&](int st_, int p) {
      const int st = max(0, min(st_, st1 - 1));
      if (p < PA) {
        // selects, not a branch: the stage stays one block for the scheduler
        const bool inx = TWO && st < kx;
        const unsigned long long base = inx ? (unsigned long long)x : (unsigned long long)h;
        const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, inx ? xbytes : hbytes, 0x00020000);
        const unsigned m = unsigned(min(m0 + lr + (NT / 8) * p, M - 1));  // rows past M: clamped, their results unused
        ra[p] = __builtin_bit_cast(f4, bload(ru, m * unsigned(inx ? 4 * D : 4 * H) + 16u * unsigned(c4),
                                             unsigned(inx ? st : st - kx) * 128u));
      } else {
#pragma unroll
        for (int f = 0; f < PB; ++f)
          rb[f] = bload(rsrc(Bp, st_ < st1 ? bbytes : 0u), 16u * unsigned(lane), bsrc[f] + unsigned(st) * unsigned(kBlk));
      }
    };
    // piece p, split, to LDS; the stages of buffer 1 hold -A
    auto put = [&](int buf, int p) {
      char* s = lds + buf * STAGE;
      if (p < PA) {
        const f4 v = ra[p] * (buf ? -kScale : kScale);
        u2v p0, p1, p2;
        unsigned t0, t1, t2;
        split2(v.x, v.y, t0, t1, t2);
        p0.x = t0, p1.x = t1, p2.x = t2;
        split2(v.z, v.w, t0, t1, t2);
        p0.y = t0, p1.y = t1, p2.y = t2;
        char* d = s + aoff + p * (NT / 128) * kBlk;
        *(u2v*)d = p0;
        *(u2v*)(d + kFrag) = p1;
        *(u2v*)(d + 2 * kFrag) = p2;
      } else {
#pragma unroll
        for (int f = 0; f < PB; ++f) *(u4v*)(s + boff + f * kFrag) = rb[f];
      }
    };
    const int ard = (wm * MI) * kBlk + (16 * q + (r ^ swz(q))) * 16;
    const int brd = ABYTES + (wn * NI) * kBlk + lane * 16;
    x3_pipeline<MI, NI, PA + 1, STAGE, kBlk>(lds, ard, brd, st0, st0 + len, gload, put, acc);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] *= kUnscale;
  }

  // The same sums by fp32 MFMAs from global memory; bval(j, k) is B of the
  // lane's column (l & 15) of the wave's column block j at reduction indices
  // k .. k + 3 of [x | h].  D and H are multiples of 16.
  template <class BVal>
  static __device__ __forceinline__ void exact(const float* x, const float* h, int M, int D, int H, int m0, int st0,
                                               int st1, BVal bval, f4 (&acc)[MI][NI]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % NW;
    const int wm = wave / WN, kx = stages(D);
    const int r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    for (int c = 2 * st0; c < 2 * st1; ++c) {  // 16 reduction indices each
      const bool inx = c < 2 * kx;
      const float* base = inx ? x : h;
      const int ld = inx ? D : H, kk = 16 * (inx ? c : c - 2 * kx);
      if (kk >= ld) continue;  // the padding of a segment
      f4 av[MI], bv[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i)
        av[i] = *(const f4*)(base + (size_t)min(m0 + (wm * MI + i) * 16 + r, M - 1) * ld + kk + 4 * q);
#pragma unroll
      for (int j = 0; j < NI; ++j) bv[j] = bval(j, (inx ? kk : D + kk) + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mfma_f32_16x16x4(av[i][e], bv[j][e], acc[i][j]);
    }
  }
};

// ---- epilogue of the gate product ----------------------------------------------
// Every thread takes four consecutive units of a row, so that the global
// accesses are 16 bytes per lane; zget(g, row, j) gives the pre-activations
// (bias included) of gate g, tile row `row`, units j .. j + 3.  Forward: the
// cell update; adjoint: loss term (returned), seed, cell adjoint, zbar_t,
// cbar_t and the copy of h_t.  Contractions are fixed by the source, so that
// the kernels that share this give the same bits.
template <int G, int MODE, int TM, int U, int NT, class Z>
__device__ __forceinline__ float cell_epilogue(const StepArgs& a, int m0, int j0, Z zget) {
#pragma clang fp contract(on)
  float lterm = 0.f;
  constexpr int TPR = U / 4;  // threads per row
  const int B = a.B, H = a.H, GH = G * H, tid = threadIdx.x;
  const int j = j0 + 4 * (tid % TPR);
  if (j < H) {
#pragma unroll 2
    for (int row = tid / TPR; row < TM; row += NT / TPR) {
      const int m = m0 + row;
      if (m >= B) break;
      const size_t o = (size_t)m * H + j;
      f4 z[G];
#pragma unroll
      for (int g = 0; g < G; ++g) z[g] = zget(g, row, j);
      f4 h1, c1, tc, ig, fg, gg, og, cold;
      if (G == 4) {
        cold = *(const f4*)(a.c + o);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ig[e] = sigm(z[0][e]);
          fg[e] = sigm(z[1 % G][e]);
          gg[e] = tanhf(z[2 % G][e]);
          og[e] = sigm(z[3 % G][e]);
          c1[e] = fg[e] * cold[e] + ig[e] * gg[e];
          tc[e] = tanhf(c1[e]);
          h1[e] = og[e] * tc[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) h1[e] = tanhf(z[0][e]);
      }
      if (MODE == kForward) {
        *(f4*)((float*)a.h_out + o) = h1;
        if (G == 4) *(f4*)(a.c_out + o) = c1;
        if (a.zc_out) {
#pragma unroll
          for (int g = 0; g < G; ++g) *(f4*)(a.zc_out + (size_t)m * GH + g * H + j) = z[g];
        }
        continue;
      }
      // adjoint: loss term of h_{t+1} and its seed dL/dh_{t+1}
      f4 hbar = {0.f, 0.f, 0.f, 0.f};
      if (!a.first) {  // the product's partial sums, in order
        hbar = *(const f4*)(a.hbar_in + o);
        for (int ps = 1; ps < a.hbar_parts; ++ps) hbar += *(const f4*)(a.hbar_in + o + (size_t)ps * B * H);
      }
      if (a.loss == AMBPTT_LOSS_MEAN_SQ_ALL) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          hbar[e] += 2.f * h1[e] * a.inv_bh;
          lterm += h1[e] * h1[e];
        }
      } else if (a.last) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool sq = a.loss == AMBPTT_LOSS_HALF_SQ_LAST;
          hbar[e] += sq ? h1[e] : a.inv_bh;
          lterm += sq ? h1[e] * h1[e] : h1[e];
        }
      }
      float* zo = (float*)a.zbar_out + (size_t)m * GH + j;
      if (G == 4) {
        f4 cb = {0.f, 0.f, 0.f, 0.f};
        if (!a.first) cb = *(const f4*)(a.cbar_in + o);
        f4 d0, d1, d2, d3, cn;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ob = hbar[e] * tc[e];
          const float ch = cb[e] + hbar[e] * og[e] * (1.f - tc[e] * tc[e]);
          d0[e] = ch * gg[e] * ig[e] * (1.f - ig[e]);
          d1[e] = ch * cold[e] * fg[e] * (1.f - fg[e]);
          d2[e] = ch * ig[e] * (1.f - gg[e] * gg[e]);
          d3[e] = ob * og[e] * (1.f - og[e]);
          cn[e] = ch * fg[e];
        }
        *(f4*)zo = d0;
        *(f4*)(zo + H) = d1;
        *(f4*)(zo + 2 * H) = d2;
        *(f4*)(zo + 3 * H) = d3;
        *(f4*)(a.cbar_out + o) = cn;
      } else {
        f4 d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = hbar[e] * (1.f - h1[e] * h1[e]);
        *(f4*)zo = d;
      }
      *(f4*)((float*)a.hwin_out + o) = *(const f4*)((const float*)a.h + o);
    }
  }
  return lterm;
}

// the waves' loss terms, summed in wave order
template <int NW>
__device__ __forceinline__ void add_loss(const StepArgs& a, float lterm, float* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float s = wave_sum(lterm);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < NW; ++w) t += (double)red[w];
    a.loss_acc[blockIdx.x] += t;
  }
}

// ---- gate product with the cell epilogue --------------------------------------
// Tile: TM batch rows x TN gate columns = U = TN / G units of all G gates
// (16-column block b of the tile: gate b / (U / 16)).  The finished tile goes
// to the epilogue through LDS.
template <int G, int MODE, int TM, int TN, int WM, int WN, int KG>
__global__ __launch_bounds__(64 * WM * WN * KG) void cell_f32x3(StepArgs a) {
  using T = Tile<TM, TN, WM, WN, KG>;
  constexpr int U = TN / G, UB = U / 16, LZ = TN + 4;
  constexpr int LDS = T::LDS > KG * TM * LZ * 4 ? T::LDS : KG * TM * LZ * 4;
  __shared__ __attribute__((aligned(16))) char lds[LDS];
  __shared__ float red[T::NW * KG];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wv / T::NW, wave = wv % T::NW;
  const int wm = wave / WN, wn = wave % WN;
  const int r = lane & 15, q = lane >> 4;
  const int B = a.B, D = a.D, H = a.H, K1 = D + H, GH = G * H;
  const int mt = (B + TM - 1) / TM, nt = (H + U - 1) / U;
  int tm, tn;
  tile_of(blockIdx.x, mt, nt, &tm, &tn);
  const int m0 = tm * TM, j0 = tn * U;
  const int hb = H / 16;
  // units past H (the last tile): the last 16 units again, unused
  auto bblk = [&](int b) { return (b / UB) * hb + min(j0 / 16 + b % UB, hb - 1); };

  f4 acc[T::MI][T::NI];
#pragma unroll
  for (int i = 0; i < T::MI; ++i)
#pragma unroll
    for (int j = 0; j < T::NI; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  const int kb = stages(D) + stages(H);
  const int st0 = kg * kb / KG, st1 = (kg + 1) * kb / KG, len = (kb + KG - 1) / KG;
  T::template run<true>((const float*)a.x, (const float*)a.h, B, D, H, m0, (const char*)a.Wx3,
                               unsigned(GH / 16) * unsigned(kb) * unsigned(kBlk), kb, st0, st1, len, bblk,
                               lds + kg * 2 * T::STAGE, acc);
  if (KG > 1) __syncthreads();  // every group has left its buffers
  if (any_bad(acc)) {
    const float* W = (const float*)a.W;
    T::exact((const float*)a.x, (const float*)a.h, B, D, H, m0, st0, st1,
             [&](int j, int k) {
               return *(const f4*)(W + (size_t)(16 * bblk(wn * T::NI + j) + r) * K1 + k);
             },
             acc);
  }
  float* z = (float*)lds;  // one tile per group
#pragma unroll
  for (int i = 0; i < T::MI; ++i)
#pragma unroll
    for (int j = 0; j < T::NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        z[kg * TM * LZ + ((wm * T::MI + i) * 16 + 4 * q + v) * LZ + (wn * T::NI + j) * 16 + r] = acc[i][j][v];
  __syncthreads();

  const float lterm = cell_epilogue<G, MODE, TM, U, T::NT * KG>(a, m0, j0, [&](int g, int row, int j) {
    const float* zr = z + row * LZ + g * U + (j - j0);
    f4 v = *(const f4*)zr;
#pragma unroll
    for (int k = 1; k < KG; ++k) v += *(const f4*)(zr + k * TM * LZ);
    return v + *(const f4*)(a.bias + g * H + j);
  });
  if (MODE == kAdjoint) add_loss<T::NW * KG>(a, lterm, red);
}

// The adjoint of a step whose pre-activations are kept: the same tiles and
// the same threads for the same elements (so the same loss sums), without the
// product.  Bound by HBM: 5 [B][4 H] or so arrays of the LSTM in and out.
template <int G, int TM, int TN, int NW>
__global__ __launch_bounds__(64 * NW) void cell_back_f32x3(StepArgs a) {
  constexpr int U = TN / G;
  __shared__ float red[NW];
  int tm, tn;
  tile_of(blockIdx.x, (a.B + TM - 1) / TM, (a.H + U - 1) / U, &tm, &tn);
  const float lterm = cell_epilogue<G, kAdjoint, TM, U, 64 * NW>(a, tm * TM, tn * U, [&](int g, int row, int j) {
    return *(const f4*)(a.zc_in + (size_t)(tm * TM + row) * (G * a.H) + g * a.H + j);
  });
  add_loss<NW>(a, lterm, red);
}

// ---- h-adjoint product: out = zbar W_h, the reduction split --------------------
// Part s of `parts` contiguous runs of stages goes to out + s M N; the
// adjoint (or sum_parts) adds the parts in order.
template <int TM, int TN, int WM, int WN, int KG>
__global__ __launch_bounds__(64 * WM * WN * KG) void prod_f32x3(ProdArgs a, int parts) {
  using T = Tile<TM, TN, WM, WN, KG>;
  __shared__ __attribute__((aligned(16))) char lds[T::LDS];
  static_assert(T::LDS >= (KG - 1) * T::NT * T::MI * T::NI * 16, "the groups' sums fit the stages' LDS");
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wv / T::NW, wave = wv % T::NW;
  const int wm = wave / WN, wn = wave % WN;
  const int r = lane & 15, q = lane >> 4;
  const int M = a.M, N = a.N, K = a.K;
  const int mt = (M + TM - 1) / TM, nt = (N + TN - 1) / TN;
  int tm, tc;
  tile_of(blockIdx.x, mt, nt * parts, &tm, &tc);
  const int tn = tc / parts, part = tc % parts;
  const int m0 = tm * TM, n0 = tn * TN;
  const int kb = stages(K);
  const int np = parts * KG, pt = part * KG + kg;
  const int st0 = int((long)pt * kb / np), st1 = int((long)(pt + 1) * kb / np), len = (kb + np - 1) / np;
  auto bblk = [&](int b) { return min(n0 / 16 + b, N / 16 - 1); };  // columns past N: the last 16 again, unused
  f4 acc[T::MI][T::NI];
#pragma unroll
  for (int i = 0; i < T::MI; ++i)
#pragma unroll
    for (int j = 0; j < T::NI; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  T::template run<false>((const float*)a.A, (const float*)a.A, M, 0, K, m0, (const char*)a.B,
                               unsigned(N / 16) * unsigned(kb) * unsigned(kBlk), kb, st0, st1, len, bblk,
                               lds + kg * 2 * T::STAGE, acc);
  if (any_bad(acc)) {
    const float* W = a.Bf;  // B(k, n) = W[k ldb + n]
    T::exact((const float*)a.A, (const float*)a.A, M, 0, K, m0, st0, st1,
             [&](int j, int k) {
               const float* s = W + (size_t)k * a.ldb + 16 * bblk(wn * T::NI + j) + r;
               return f4{s[0], s[a.ldb], s[2 * (size_t)a.ldb], s[3 * (size_t)a.ldb]};
             },
             acc);
  }
  if (KG > 1) {  // the other groups' sums, in order, through LDS
    f4* g = (f4*)lds;
    const int t = threadIdx.x % T::NT;
    __syncthreads();
    if (kg > 0)
#pragma unroll
      for (int i = 0; i < T::MI; ++i)
#pragma unroll
        for (int j = 0; j < T::NI; ++j) g[(((kg - 1) * T::MI + i) * T::NI + j) * T::NT + t] = acc[i][j];
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int k = 0; k < KG - 1; ++k)
#pragma unroll
      for (int i = 0; i < T::MI; ++i)
#pragma unroll
        for (int j = 0; j < T::NI; ++j) acc[i][j] += g[((k * T::MI + i) * T::NI + j) * T::NT + t];
  }
  float* out = a.out + (size_t)part * M * N;
#pragma unroll
  for (int i = 0; i < T::MI; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = m0 + (wm * T::MI + i) * 16 + 4 * q + v;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < T::NI; ++j) {
        const int n = n0 + (wn * T::NI + j) * 16 + r;
        if (n < N) out[(size_t)m * N + n] = acc[i][j][v];
      }
    }
}

__global__ void sum_parts_f32(const float* __restrict__ p, int parts, size_t n4, float* __restrict__ out) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n4) return;
  f4 s = ((const f4*)p)[i];
  for (int k = 1; k < parts; ++k) s += ((const f4*)p)[i + (size_t)k * n4];
  ((f4*)out)[i] = s;
}

// dst <- the planes of src's N rows of K values (scaled) in fragment order, K padded
// with zeros to whole stages: steps kb0 .. of the kb steps of a block row.  A
// thread makes one lane's 16 bytes of the three planes.  TR: src(n, k) =
// src[k ld + n] (the columns of W_h).
template <bool TR>
__global__ __launch_bounds__(256) void pack_f32x3(const float* __restrict__ src, int N, int K, int ld, int kb, int kb0,
                                                  char* __restrict__ dst) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the four waves of a block take neighbouring fragments along the rows of src
  const int nb = TR ? blockIdx.y * 4 + wave : blockIdx.y, ks = TR ? blockIdx.x : blockIdx.x * 4 + wave;
  if (nb >= N / 16 || ks >= stages(K)) return;
  const int n = nb * 16 + (lane & 15), k = ks * kSt + 8 * (lane >> 4);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e)
    v[e] = k < K ? src[TR ? (size_t)(k + e) * ld + n : (size_t)n * ld + k + e] * kScale : 0.f;  // K is a multiple of 8
  u4v p0, p1, p2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    unsigned t0, t1, t2;
    split2(v[2 * e], v[2 * e + 1], t0, t1, t2);
    p0[e] = t0, p1[e] = t1, p2[e] = t2;
  }
  char* d = dst + ((size_t)nb * kb + kb0 + ks) * kBlk + lane * 16;
  *(u4v*)d = p0;
  *(u4v*)(d + kFrag) = p1;
  *(u4v*)(d + 2 * kFrag) = p2;
}

}  // namespace

size_t f32x3_bytes(int N, int K0, int K1) { return size_t(N / 16) * size_t(stages(K0) + stages(K1)) * kBlk; }

hipError_t launch_pack_f32x3(const float* src, int N, int K0, int K1, int ld, bool transposed, void* dst, hipStream_t s) {
  if (N < 16 || N % 16 || K0 % 8 || K1 % 8 || K0 < 0 || K1 < 8) return hipErrorInvalidValue;
  const int kb = stages(K0) + stages(K1);
  for (int seg = 0; seg < 2; ++seg) {
    const int K = seg ? K1 : K0, kb0 = seg ? stages(K0) : 0;
    if (K == 0) continue;
    const float* p = src + (seg ? (transposed ? size_t(K0) * ld : size_t(K0)) : 0);
    if (transposed)
      hipLaunchKernelGGL((pack_f32x3<true>), dim3(stages(K), (N / 16 + 3) / 4), dim3(256), 0, s, p, N, K, ld, kb, kb0,
                         (char*)dst);
    else
      hipLaunchKernelGGL((pack_f32x3<false>), dim3((stages(K) + 3) / 4, N / 16), dim3(256), 0, s, p, N, K, ld, kb, kb0,
                         (char*)dst);
  }
  return hipGetLastError();
}

bool f32x3_fits(int G, int B, int D, int H) {
  const unsigned long long lim = 1ull << 32;  // buffer offsets are 32-bit
  return (G == 1 || G == 4) && B >= 1 && D >= 0 && D % 16 == 0 && H >= 16 && H % 16 == 0 &&
         4ull * B * H * G + 4096 < lim && 4ull * B * D + 4096 < lim && f32x3_bytes(G * H, D, H) < lim &&
         f32x3_bytes(H, 0, G * H) < lim;
}

namespace {

// The two tiles: 256 x 128 on 8 waves moves the fewest operand bytes per MFMA;
// 128 x 64 on two groups of 4 waves makes more workgroups of a small grid.
// One workgroup of either fills a CU.  A 32-wide stage of the first takes
// 2.05 us (300 x 9856 x 2672, 84 stages, 154 tiles: 167 us; 2.55 us with all
// CUs at it, whose clock then falls), of the second 0.75 us (the same in two
// rounds of 462 tiles: 126 us; 300 x 4096 x 1120: 31.5 us, with one group of 4
// waves 39.5 us), so the second is taken where its rounds over the 256 CUs are
// fewer than 2.7 times the first's (300 x 12288 x 3136, 3 rounds against 1:
// 214 us against 202).
constexpr double kBigStage = 2.05, kSmallStage = 0.75;
double rounds(int tiles) { return double((tiles + 255) / 256); }
bool big_tiles(int big, int small) { return rounds(big) * kBigStage <= rounds(small) * kSmallStage; }

template <int G, int MODE>
hipError_t cell_launch(const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const auto tiles = [&](int tm, int tn) { return ((a.B + tm - 1) / tm) * ((a.H + tn / G - 1) / (tn / G)); };
  const int big = tiles(256, 128), small = tiles(128, 64);
  const bool back = MODE == kAdjoint && a.zc_in;
  if (big_tiles(big, small)) {
    if (back) hipExtLaunchKernelGGL((cell_back_f32x3<G, 256, 128, 8>), dim3(big), dim3(512), 0, s, e0, e1, 0, a);
    else hipExtLaunchKernelGGL((cell_f32x3<G, MODE, 256, 128, 4, 2, 1>), dim3(big), dim3(512), 0, s, e0, e1, 0, a);
  } else {
    if (back) hipExtLaunchKernelGGL((cell_back_f32x3<G, 128, 64, 8>), dim3(small), dim3(512), 0, s, e0, e1, 0, a);
    else hipExtLaunchKernelGGL((cell_f32x3<G, MODE, 128, 64, 4, 1, 2>), dim3(small), dim3(512), 0, s, e0, e1, 0, a);
  }
  return hipGetLastError();
}

// the h-adjoint product's tile and split: the least of rounds x stages
struct ProdPlan {
  bool big;
  int parts, tiles;
};
ProdPlan prod_plan(int M, int N, int K) {
  const int kb = stages(K);
  const int t[2] = {((M + 127) / 128) * ((N + 63) / 64), ((M + 255) / 256) * ((N + 127) / 128)};
  ProdPlan best{false, 1, t[0]};
  double least = 1e30;
  for (int big = 0; big < 2; ++big)
    for (int parts = 1; parts <= kProdSplitMax && parts * 16 <= kb; parts *= 2) {
      const double c = rounds(t[big] * parts) * ((kb + parts - 1) / parts) * (big ? kBigStage : kSmallStage);
      if (c < 0.97 * least) least = c, best = ProdPlan{big == 1, parts, t[big]};  // more parts must pay for their sum
    }
  return best;
}
}  // namespace

int cell_f32x3_tiles(int G, int B, int H) {  // the most workgroups that its launches have
  return ((B + 127) / 128) * ((H + 64 / G - 1) / (64 / G));
}

hipError_t launch_cell_f32x3(int G, int mode, const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (!f32x3_fits(G, a.B, a.D, a.H) || !a.Wx3 || (mode == kAdjoint && !a.first && !a.hbar_in)) return hipErrorInvalidValue;
  if (mode != kForward && mode != kAdjoint) return hipErrorInvalidValue;
  if (G == 4) return mode == kForward ? cell_launch<4, kForward>(a, s, e0, e1) : cell_launch<4, kAdjoint>(a, s, e0, e1);
  return mode == kForward ? cell_launch<1, kForward>(a, s, e0, e1) : cell_launch<1, kAdjoint>(a, s, e0, e1);
}

int prod_f32x3_parts(int M, int N, int K) { return prod_plan(M, N, K).parts; }

hipError_t launch_prod_f32x3(const ProdArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.M < 1 || a.N < 16 || a.N % 16 || a.K < 16 || a.K % 16 || a.add || !a.Bf) return hipErrorInvalidValue;
  const ProdPlan p = prod_plan(a.M, a.N, a.K);
  const dim3 grid(p.tiles * p.parts), block(512);
  if (p.big) hipExtLaunchKernelGGL((prod_f32x3<256, 128, 4, 2, 1>), grid, block, 0, s, e0, e1, 0, a, p.parts);
  else hipExtLaunchKernelGGL((prod_f32x3<128, 64, 4, 1, 2>), grid, block, 0, s, e0, e1, 0, a, p.parts);
  return hipGetLastError();
}

hipError_t launch_sum_parts_f32(const float* p, int parts, size_t n, float* out, hipStream_t s, hipEvent_t e0,
                                hipEvent_t e1) {
  if (n % 4 || parts < 1) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(sum_parts_f32, dim3(unsigned((n / 4 + 255) / 256)), dim3(256), 0, s, e0, e1, 0, p, parts, n / 4,
                        out);
  return hipGetLastError();
}

}  // namespace ambptt
