// fp32 products on the bf16 matrix cores (gfx950): the exact split of an fp32
// value in three bf16 parts, and the stage pipeline of the kernels that
// multiply split operands (gemm_f32x3.hip, dw_f32x3.hip).
//
// Range.  Both operands are scaled by 2^32 before they are split (and their
// products' sums by 2^-64): an fp32 value down to the smallest subnormal then
// has its parts in bf16's normal range (unscaled, values below about 2^-110
// would lose bits).  Values of 2^96 and more and sums of 2^64 and more
// overflow; such tiles are formed again (any_bad).
//
// Rounding.  The matrix cores round a bf16 MFMA's sum of products down (not
// to nearest), a bias that grows with the length of the chain of
// accumulations: with one chain through the whole reduction db of the
// 4096-LSTM, a sum over thousands of rows, was 3.4e-6 off (8e-7 with fp32
// MFMAs).  So each stage's six products are summed from zero and added to the
// accumulators by VALU adds, which round to nearest, and every other stage
// multiplies -A and is subtracted, which turns its bias around.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "mfma.hpp"

namespace ambptt {

typedef unsigned int u2v __attribute__((ext_vector_type(2)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kSt = 32;                         // reduction indices per stage
constexpr int kFrag = 1024;                     // bytes of one plane of a 16-row fragment
constexpr int kBlk = 3 * kFrag;                 // ... of its three planes
constexpr float kScale = 4294967296.0f;         // 2^32, of either operand
constexpr float kUnscale = 1.0f / 18446744073709551616.0f;  // 2^-64, of their products

__device__ __forceinline__ unsigned pk_bf16(float a, float b) {
  const f2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float lo_f(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float hi_f(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, unsigned bytes) {
  const unsigned long long p = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(p)), hi = __builtin_amdgcn_readfirstlane(unsigned(p >> 32));
  void* ub = (void*)(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
// reads past the buffer's end return zero
__device__ __forceinline__ u4v bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
}

// the three planes of a pair of values
__device__ __forceinline__ void split2(float a, float b, unsigned& p0, unsigned& p1, unsigned& p2) {
  p0 = pk_bf16(a, b);
  const float a1 = a - lo_f(p0), b1 = b - hi_f(p0);
  p1 = pk_bf16(a1, b1);
  p2 = pk_bf16(a1 - lo_f(p1), b1 - hi_f(p1));
}

// whether any of a wave's accumulators is an infinity or a NaN
template <int MI, int NI>
__device__ __forceinline__ bool any_bad(const f4 (&acc)[MI][NI]) {
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) bad |= !(fabsf(acc[i][j][v]) <= 3.402823466e38f);
  return __any(bad);
}

// The stages st0 .. st1 - 1 of one wave's MI x NI blocks of 16 x 16.
// gload(st, p) brings piece p (of NP) of stage st to registers, put(buf, p)
// splits it and writes it to LDS buffer `buf` (buffer 1: -A).  The stages go
// in pairs (st1 - st0 is rounded up): of a stage past the last that counts,
// gload must give zeros for one operand.
// ard, brd: the lane's first fragments in a buffer of STAGE bytes; BLK: bytes
// from one 16-row block to the next, its planes kFrag apart.
//
// A stage is MI row blocks of 6 NI MFMAs.  In the blocks but the last the
// next stage goes to the other buffer, a piece at a time, and the piece's
// loads for the stage after that are issued (so a load has a whole stage to
// arrive).  The one barrier of a stage comes before its last block, whose
// operands are in registers by then: during that block the next stage's first
// operands are read, each plane of B once its last use is issued, and the
// matrix cores find them there after it.
template <int MI, int NI, int NP, int STAGE, int BLK, class GLoad, class Put>
__device__ __forceinline__ void x3_pipeline(const char* lds, int ard, int brd, int st0, int st1, GLoad gload, Put put,
                                            f4 (&acc)[MI][NI]) {
  static_assert(MI % 2 == 0, "row blocks in pairs");
  bf16x8 b[3][NI], a[2][3];
  auto lda = [&](int buf, int i) {
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) a[i & 1][pl] = *(const bf16x8*)(lds + buf * STAGE + ard + i * BLK + pl * kFrag);
  };
  auto ldb = [&](int buf, int pl) {
#pragma unroll
    for (int j = 0; j < NI; ++j) b[pl][j] = *(const bf16x8*)(lds + buf * STAGE + brd + j * BLK + pl * kFrag);
  };

#pragma unroll
  for (int p = 0; p < NP; ++p) gload(st0, p);
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    put(0, p);
    gload(st0 + 1, p);
  }
  __syncthreads();
  lda(0, 0);
  ldb(0, 2);
  ldb(0, 1);
  ldb(0, 0);
  f4 tl[NI];  // the last row block's sums, added one block later
#pragma unroll
  for (int j = 0; j < NI; ++j) tl[j] = f4{0.f, 0.f, 0.f, 0.f};
  auto stage = [&](int st, auto cur_) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_)::value;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const bool tail = i == MI - 1;
      if (tail) __syncthreads();
      f4 t[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) t[j] = f4{0.f, 0.f, 0.f, 0.f};
      auto mul = [&](int pa, int pb) {
#pragma unroll
        for (int j = 0; j < NI; ++j)
          t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i & 1][pa], b[pb][j], t[j], 0, 0, 0);
      };
      if (!tail) {
        lda(cur, i + 1);
        mul(0, 2);
        mul(1, 1);
        mul(0, 1);
        mul(2, 0);
        mul(1, 0);
        mul(0, 0);
#pragma unroll
        for (int p = 0; p < NP; ++p)
          if (p * (MI - 1) / NP == i) {
            put(cur ^ 1, p);
            gload(st + 2, p);
          }
      } else {
        lda(cur ^ 1, 0);
        mul(0, 2);
        __builtin_amdgcn_sched_barrier(0);
        ldb(cur ^ 1, 2);
        mul(1, 1);
        mul(0, 1);
        __builtin_amdgcn_sched_barrier(0);
        ldb(cur ^ 1, 1);
        mul(2, 0);
        mul(1, 0);
        mul(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        ldb(cur ^ 1, 0);
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {  // (the row block before the first is the stage before's last)
        if ((i == 0) != (cur == 1)) acc[(i + MI - 1) % MI][j] -= tl[j];
        else acc[i == 0 ? MI - 1 : i - 1][j] += tl[j];
        tl[j] = t[j];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int st = st0; st < st1; st += 2) {
    stage(st, std::integral_constant<int, 0>{});
    stage(st + 1, std::integral_constant<int, 1>{});
  }
#pragma unroll
  for (int j = 0; j < NI; ++j) acc[MI - 1][j] -= tl[j];
  __syncthreads();  // the last stage's reads of the buffers are done
}

}  // namespace ambptt
