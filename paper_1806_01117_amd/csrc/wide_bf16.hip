// Wide-batch bf16 step kernels (gfx950): the LSTM / tanh-RNN cell and the
// residual MLP for batches of 48 rows and more and for smaller ones whose
// weights are many.
//
// At these shapes a step is a short, fat GEMM (the 2048-wide LSTM: 128 x 8192
// x 3072 with a 50 MB weight matrix; the 4096-wide MLP layer: 256 x 4096 x
// 4096).  What bounds it is how fast every CU pulls its operands through L2,
// not the MFMA rate.  Two choices follow from that:
//   * Tiles move the fewest bytes per CU: a 64 x 64 output tile per
//     workgroup for the cell's gate GEMM (64 batch rows x 16 LSTM units, all
//     four gates) and for the MLP layer, 32 x 32 for the h-adjoint product.
//     Problems that would leave most of the 256 CUs without a tile take 32 or
//     16 rows per tile instead (tile_rows).
//     The adjoint's products hbar = zbar W_h (cell) and zbar W_{l+1} (MLP)
//     are launches of their own: each reads the whole zbar of its rows, and
//     fused into the cell kernel's tile they would move twice the bytes.
//   * Loads cover whole 128-byte lines.  The activation operand is read as
//     rows, one load instruction covering 8 rows x 128 bytes (lane l: row
//     l >> 3, bytes 16 (l & 7) ..), which pulls about twice the bandwidth of
//     the MFMA operand layout (16 rows x 64 bytes per instruction); each wave
//     turns its rows into MFMA fragments through LDS scratch tiles of its own
//     (swizzled 16 x 128-byte tiles), so no workgroup barrier sits in the
//     main loop.  The recurrent cell's weights, fixed for a pass, are read
//     from a copy in fragment order (pack_nt below): one load instruction
//     reads a fragment's 1 KiB contiguously into the lanes that multiply it,
//     with no trip through LDS.
// Inside a workgroup the 8 waves split the reduction in 64-wide blocks, so no
// byte is loaded twice; the loads of the next block(s) are in flight while
// the current one is multiplied.  The partial products meet in LDS and are
// summed in wave order (bit-reproducible).
//
// Operands are bf16 on v_mfma_f32_16x16x32_bf16 (lane l: row or column
// l & 15, reduction indices 8 (l >> 4) .. +7 of a 32-wide chunk; result:
// column l & 15, rows 4 (l >> 4) .. +3).  Stored h / y, zbar and the copies
// kept for the weight gradient are bf16 (nearest even); accumulation, the
// LSTM cell state, its adjoint and the carried MLP adjoint stay fp32.
#include <hip/hip_runtime.h>

#include "ambptt.h"
#include "kernels.hpp"
#include "mfma.hpp"

namespace ambptt {
namespace {

constexpr int kWaves = 8;  // waves per workgroup of the launched kernels
constexpr int kSlot = 2048;  // one 16-row x 128-byte scratch tile

typedef unsigned int u4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Workgroup id -> tile, XCD-aware: ids are dealt to the 8 XCDs round-robin,
// and each XCD takes a contiguous run of tiles numbered column-group major,
// so the row groups that share weight rows share one L2.
__device__ __forceinline__ int tile_of(int ntile) {
  const int per = (ntile + 7) / 8;
  return int(blockIdx.x % 8) * per + int(blockIdx.x / 8);
}

// Buffer descriptor of a whole operand.  Every buffer here is the same for
// all lanes of a wave; readfirstlane states that, so the descriptor sits in
// scalar registers.  Reads at or past `bytes` return zero (rows beyond the
// batch).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, unsigned bytes) {
  const unsigned long long p = (unsigned long long)base;
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(p)), hi = __builtin_amdgcn_readfirstlane(unsigned(p >> 32));
  void* ub = (void*)(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
__device__ __forceinline__ u4v bload(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
}

// Rows of a row-major operand, read in 16-row groups and 64-wide reduction
// blocks (128 bytes of a bf16 row).  Instruction h of group g covers rows
// row0 + 16 g + 8 h + (lane >> 3), bytes 16 (lane & 7) .. +15 of the block.
// A row of cols values that ends in the middle of a block (cols an odd
// multiple of 32) reads zeros for the block's second half.
struct Rows {
  __amdgpu_buffer_rsrc_t r;
  unsigned voff;    // lane part: (lane >> 3) stride + 16 (lane & 7)
  unsigned vtail;   // ... in the block that the row ends in: past the buffer for its second half
  unsigned base;    // row0 stride (the same for the wave)
  unsigned stride;  // row stride in bytes
  int half;         // the block that the row ends in the middle of (-1: none)
  __device__ __forceinline__ u4v load(int g, int h, int blk) const {
    return bload(r, blk == half ? vtail : voff, base + unsigned(16 * g + 8 * h) * stride + unsigned(blk) * 128u);
  }
};
__device__ __forceinline__ Rows rows_of(const void* p, unsigned bytes, int row0, int cols) {
  const int lane = threadIdx.x & 63;
  Rows s;
  s.r = rsrc(p, bytes);
  s.voff = unsigned((lane >> 3) * (2 * cols) + 16 * (lane & 7));
  s.vtail = (lane & 7) < 4 ? s.voff : bytes;
  s.base = unsigned(row0) * unsigned(2 * cols);
  s.stride = unsigned(2 * cols);
  s.half = cols % 64 ? cols / 64 : -1;
  return s;
}
__host__ __device__ __forceinline__ int blocks(int cols) { return (cols + 63) / 64; }

// An NT operand Bm(k, n) = B[n][k] in fragment order: the fragment of n tile
// jt (columns 16 jt ..) and 32-wide reduction step ks is 1 KiB, lane l's 16
// bytes being B[16 jt + (l & 15)][32 ks + 8 (l >> 4) .. +7], the operand
// layout of v_mfma_f32_16x16x32_bf16; the fragments of an n tile are
// consecutive (n tile major), two per 64-wide block, padded with zeros.
struct Frags {
  __amdgpu_buffer_rsrc_t r;
  unsigned voff;  // 16 lane
  unsigned tile;  // bytes of one n tile: its blocks' fragments
  __device__ __forceinline__ u4v load(int jt, int ks) const {
    return bload(r, voff, unsigned(jt) * tile + unsigned(ks) * 1024u);
  }
};
__device__ __forceinline__ Frags frags_of(const void* p, int N, int nblk) {
  Frags f;
  f.tile = unsigned(nblk) * 2048u;
  f.r = rsrc(p, unsigned(N / 16) * f.tile);
  f.voff = unsigned(threadIdx.x & 63) * 16u;
  return f;
}

// Per-lane LDS offsets within one 16 x 128-byte scratch tile.  Row t's
// 16-byte group k sits at slot k ^ (t & 7): the 8 lanes that write one row hit
// 8 different slots, and the reads of one fragment column spread over the
// banks (measured free of bank conflicts on gfx950, where an extra flip for
// rows 8..15 was not).
struct Xpose {
  unsigned w0, w1;  // writes of the rows-0..7 and rows-8..15 instructions
  unsigned r0, r1;  // fragment reads: reduction indices 0..31 and 32..63 of the block
  __device__ __forceinline__ void init() {
    const int lane = threadIdx.x & 63;
    auto sw = [](int t) { return t & 7; };
    const int t0 = lane >> 3, t1 = 8 + (lane >> 3), k = lane & 7;
    w0 = unsigned(t0 * 128 + 16 * (k ^ sw(t0)));
    w1 = unsigned(t1 * 128 + 16 * (k ^ sw(t1)));
    const int r = lane & 15, q = lane >> 4;
    r0 = unsigned(r * 128 + 16 * (q ^ sw(r)));
    r1 = unsigned(r * 128 + 16 * ((q + 4) ^ sw(r)));
  }
  __device__ __forceinline__ void put(char* tile, const u4v& v0, const u4v& v1) const {
    *(u4v*)(tile + w0) = v0;
    *(u4v*)(tile + w1) = v1;
  }
  // the MFMA fragment of the block's 32-wide chunk c
  __device__ __forceinline__ bf16x8 get(const char* tile, int c) const {
    return __builtin_bit_cast(bf16x8, *(const u4v*)(tile + (c ? r1 : r0)));
  }
};

// Software pipeline over reduction blocks [c0, c1): ld(blk, s) issues the
// loads of block blk into register buffer s, use(s) consumes buffer s.  The
// loads of S - 1 blocks are in flight while one is used.  c0 and c1 are the
// same for the whole wave, so every branch is scalar; the steady-state body
// has no branch and the stages keep their order, so the wait before each use
// leaves the younger blocks' loads outstanding.
template <int S, class LD, class USE>
__device__ __forceinline__ void pipeline(int c0, int c1, LD ld, USE use) {
  if (c1 <= c0) return;
  // unconditional prologue (a short range loads its last block again) in
  // stage order: the wait at the loop head is the worst case over the loop's
  // entry and its back edge
#pragma unroll
  for (int s = 0; s < S; ++s) {
    ld(min(c0 + s, c1 - 1), s);
    __builtin_amdgcn_sched_barrier(0);
  }
  int ch = c0;
  for (; ch + 2 * S <= c1; ch += S) {  // blocks ch .. ch + S - 1 are in buffers 0 .. S - 1
#pragma unroll
    for (int s = 0; s < S; ++s) {
      use(s);
      ld(ch + S + s, s);
      // keep the stages in order: the compiler would otherwise gather every
      // MFMA of the body ahead of every load and wait for all loads at once
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the last S .. 2S - 1 blocks
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if (ch + s < c1) {
      use(s);
      if (ch + S + s < c1) ld(ch + S + s, s);
    }
  }
  ch += S;
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (ch + s < c1) use(s);
}

// acc[i][nb] += A_i . B_nb over the wave's blocks [c0, c1); la(g, h, blk) and
// lb(g, h, blk) load instruction h of 16-row group g of block blk.  The wave's
// scratch `scr` holds NB + RT tiles.  With PB, lb(g, c, blk) loads the
// fragment of B's group g for the block's 32-wide chunk c (Frags), which the
// MFMAs take as loaded.
template <int RT, int NB, int S, bool PB = false, class LA, class LB>
__device__ __forceinline__ void nt_rows(int c0, int c1, char* scr, const Xpose& X, f4 (&acc)[RT][NB], LA la, LB lb) {
  u4v va[S][RT][2], vb[S][NB][2];
  pipeline<S>(
      c0, c1,
      [&](int blk, int s) {
#pragma unroll
        for (int g = 0; g < RT; ++g)
#pragma unroll
          for (int h = 0; h < 2; ++h) va[s][g][h] = la(g, h, blk);
#pragma unroll
        for (int g = 0; g < NB; ++g)
#pragma unroll
          for (int h = 0; h < 2; ++h) vb[s][g][h] = lb(g, h, blk);
      },
      [&](int s) {
        if constexpr (!PB) {
#pragma unroll
          for (int g = 0; g < NB; ++g) X.put(scr + g * kSlot, vb[s][g][0], vb[s][g][1]);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) X.put(scr + (NB + i) * kSlot, va[s][i][0], va[s][i][1]);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          bf16x8 fb[NB];
#pragma unroll
          for (int g = 0; g < NB; ++g) fb[g] = PB ? __builtin_bit_cast(bf16x8, vb[s][g][c]) : X.get(scr + g * kSlot, c);
#pragma unroll
          for (int i = 0; i < RT; ++i) {
            const bf16x8 fa = X.get(scr + (NB + i) * kSlot, c);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[i][nb] = mfma_bf16_16x16x32(fa, fb[nb], acc[i][nb]);
          }
        }
        __builtin_amdgcn_wave_barrier();  // the tiles are read before the next block is stored
      });
}

// The wave's partial products -> ps[wave][row][col] (LDS, after every wave
// has left its main loop); the workgroup-wide sum runs in wave order.
template <int RT, int NB>
__device__ __forceinline__ void put_partials(float* ps, int wave, const f4 (&acc)[RT][NB]) {
  constexpr int LD = 16 * NB + 1;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  float* p = ps + wave * (16 * RT) * LD;
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 4; ++v) p[(16 * i + 4 * q + v) * LD + nb * 16 + r] = acc[i][nb][v];
}
template <int RT, int NB, int NW>
__device__ __forceinline__ float sum_partials(const float* ps, int row, int col) {
  constexpr int LD = 16 * NB + 1, W = 16 * RT * LD;
  float s = 0.f;
#pragma unroll
  for (int wv = 0; wv < NW; ++wv) s += ps[wv * W + row * LD + col];
  return s;
}

// LDS of a kernel: the partial sums, or the waves' scratch, whichever is larger
template <int RT, int NB, int SCR, int NW>
constexpr int lds_bytes() {
  constexpr int ps = NW * 16 * RT * (16 * NB + 1) * 4;
  constexpr int sc = NW * SCR;
  return ps > sc ? ps : sc;
}

// ---- the recurrent cell: gate GEMM + cell update ----------------------------
//
// Workgroup tile: 16 RT batch rows x UN hidden units, all G gates (64 gate
// columns: UN = 16 for the LSTM, 64 for the tanh RNN).  Gate column n =
// g UN + u is weight row g H + j0 + u; a 16-column group is 16 consecutive
// weight rows, one n tile of the fragment-order copy of W (a.W: pack_nt of
// the [G H][D + H] weights).  Forward: h_{t+1}, c_{t+1}.  Adjoint (gate recomputation of
// step t): with hbar_{t+1} from the product launch before it (absent for the
// first turn) it forms zbar_t, cbar_t, the loss term and the copy of h_t for
// the weight-gradient window.
// CACHED (adjoint): the pre-activations are kept (a.zc_in) and the gate
// product is not formed again; the same tiles and threads take the same
// elements.
template <int G, int MODE, int RT, bool CACHED = false, int NW = kWaves, int S = RT == 4 ? 2 : 3>
__global__ __launch_bounds__(64 * NW) void cell_wide(StepArgs a) {
  constexpr int NB = 4, TM = 16 * RT;
  constexpr int UN = 64 / G;  // hidden units of the tile
  constexpr int SCR = (RT + NB) * kSlot;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int B = a.B, D = a.D, H = a.H, GH = G * H;
  const int mg = (B + TM - 1) / TM, ntile = mg * ((H + UN - 1) / UN);
  const int w = tile_of(ntile);
  if (w >= ntile) return;  // grid padding (the whole workgroup leaves together)
  const int m0 = (w % mg) * TM, j0 = (w / mg) * UN;

  __shared__ __attribute__((aligned(16))) char lds[CACHED ? 16 : lds_bytes<RT, NB, SCR, NW>()];
  float* ps = (float*)lds;
  if (!CACHED) {
    f4 acc[RT][NB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f4{0.f, 0.f, 0.f, 0.f};
    Xpose X;
    X.init();
    const int nbx = blocks(D), nbk = nbx + blocks(H);
    const int c0 = (nbk * wave) / NW, c1 = (nbk * (wave + 1)) / NW;
    const unsigned xbytes = unsigned(size_t(B) * D * 2), hbytes = unsigned(size_t(B) * H * 2);  // < 4 GiB: cell_wide_fits
    const Rows xs = rows_of(a.x, xbytes, m0, D), hs = rows_of(a.h, hbytes, m0, H);
    const Frags wf = frags_of(a.W, GH, nbk);
    nt_rows<RT, NB, S, true>(
        c0, c1, lds + wave * SCR, X, acc,
        [&](int g, int h, int blk) -> u4v {
          // an x or an h block: the same choice for the whole wave, made by
          // selects (with branches around the loads a step of the 2048-LSTM
          // took 19.6 us instead of 16.2)
          const bool inx = blk < nbx;
          const int bk = inx ? blk : blk - nbx;
          const unsigned v = inx ? xs.voff : hs.voff, vt = inx ? xs.vtail : hs.vtail;
          const unsigned long long p = inx ? (unsigned long long)a.x : (unsigned long long)a.h;
          return bload(__builtin_amdgcn_make_buffer_rsrc((void*)p, 0, inx ? xbytes : hbytes, 0x00020000),
                       bk == (inx ? xs.half : hs.half) ? vt : v,
                       (inx ? xs.base : hs.base) + unsigned(16 * g + 8 * h) * (inx ? xs.stride : hs.stride) +
                           unsigned(bk) * 128u);
        },
        [&](int g, int c, int blk) -> u4v {  // units past H (the tanh RNN's last tile): the last 16 again, unused
          return wf.load((16 * g / UN) * (H / 16) + min((j0 + (16 * g) % UN) / 16, H / 16 - 1), 2 * blk + c);
        });
    __syncthreads();  // every wave has left its scratch
    put_partials<RT, NB>(ps, wave, acc);
  }
  __syncthreads();

  // epilogue: pair (row ml, unit u), consecutive threads on consecutive units
  float lterm = 0.f;
  for (int pi = tid; pi < TM * UN; pi += 64 * NW) {
#pragma clang fp contract(on)  // the same bits with and without the gate product
    const int ml = pi / UN, u = pi % UN;
    const int m = m0 + ml, j = j0 + u;
    if (m >= B || j >= H) continue;
    const int o = m * H + j;
    float z[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const size_t zo = (size_t)m * GH + g * H + j;
      if (CACHED) {
        z[g] = a.zc_in[zo];
      } else {
        z[g] = sum_partials<RT, NB, NW>(ps, ml, g * UN + u) + a.bias[g * H + j];
        if (MODE == kForward && a.zc_out) a.zc_out[zo] = z[g];
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
    const __bf16 h1s = (__bf16)h1;  // the stored state (nearest even)
    if (MODE == kForward) {
      ((__bf16*)a.h_out)[o] = h1s;
      if (G == 4) a.c_out[o] = c1;
    } else {
      const float hl = (float)h1s;  // loss and seed read the stored h_{t+1}
      float sd = 0.f, lt = 0.f;
      if (a.loss == AMBPTT_LOSS_MEAN_SQ_ALL) {
        sd = 2.f * hl * a.inv_bh;
        lt = hl * hl;
      } else if (a.last) {
        if (a.loss == AMBPTT_LOSS_HALF_SQ_LAST) {
          sd = hl;
          lt = hl * hl;
        } else {
          sd = a.inv_bh;
          lt = hl;
        }
      }
      lterm += lt;
      const float hb = (a.first ? 0.f : a.hbar_in[o]) + sd;
      __bf16* zo = (__bf16*)a.zbar_out + (size_t)m * GH + j;
      if (G == 4) {
        const float cb = a.first ? 0.f : a.cbar_in[o];
        const float ob = hb * tc;
        const float ch = cb + hb * og * (1.f - tc * tc);
        zo[0] = (__bf16)(ch * gg * ig * (1.f - ig));
        zo[H] = (__bf16)(ch * cold * fg * (1.f - fg));
        zo[2 * H] = (__bf16)(ch * ig * (1.f - gg * gg));
        zo[3 * H] = (__bf16)(ob * og * (1.f - og));
        a.cbar_out[o] = ch * fg;
      } else {
        zo[0] = (__bf16)(hb * (1.f - h1 * h1));
      }
      ((__bf16*)a.hwin_out)[o] = ((const __bf16*)a.h)[o];
    }
  }
  if (MODE == kAdjoint) {
    const float s = wave_sum(lterm);
    __shared__ float wsum[NW];
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) t += wsum[wv];
      a.loss_acc[w] += (double)t;
    }
  }
}

// The NN product's B block in LDS: row t (one k, 64 columns n) is 128 bytes,
// its 32-byte segments (16 columns each) permuted by nn_swz(t) so that the
// 16 rows one transposing read touches (rows kb + 8 g + 0..3, g = 0..3) fall
// on distinct banks within each half wave.
__device__ __forceinline__ int nn_swz(int t) { return ((t >> 1) & 1) | (((t >> 3) & 1) << 1); }

// Fragment of the block's 16 x 32 piece (columns 16 nb .., rows kb .. kb + 31):
// lane l receives rows kb + 8 (l >> 4) .. +7 of column l & 15.  Each
// ds_read_b64_tr_b16 gives lane j of a 16-lane group rows r .. r + 3 of
// column j, the group's lane i naming 4 consecutive values (row r + (i >> 2),
// columns 4 (i & 3) ..) of that 16-column segment.
__device__ __forceinline__ bf16x8 nn_frag(const char* bt, int kb, int nb) {
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  const int r0 = kb + 8 * g + (i >> 2), r1 = r0 + 4;
  typedef short s4 __attribute__((ext_vector_type(4)));
  typedef short s8 __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s4 lds_s4;
  const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(bt + r0 * 128 + 32 * (nb ^ nn_swz(r0)) + 8 * (i & 3)));
  const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(bt + r1 * 128 + 32 * (nb ^ nn_swz(r1)) + 8 * (i & 3)));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// ---- products of the adjoint ------------------------------------------------
//
// out[m][n] = add[m][n] (if given) + sum_k A[m][k] Bm(k, n), A [M][K] bf16,
// over a TM x TN tile (TM = 16 RT, TN = 16 NB) per workgroup.
//   NN = false: Bm(k, n) = B[n][k] (the cell's W_h^T), B in fragment order
//     (pack_nt of the [N][K] rows);
//   NN = true:  Bm(k, n) = B[k][n] (the MLP's W_{l+1}, contiguous in n; TN =
//     64): each block's 64 x 64 elements of B go to the wave's scratch as
//     loaded (rows k of 128 bytes) and come back as fragments through
//     gfx950's transposing LDS read, so no transposed copy of the weights
//     is kept.
template <int RT, bool NN, int NB>
constexpr int prod_scr() { return NN ? RT * kSlot + 64 * 128 : (RT + NB) * kSlot; }

// the tile's partial sums in LDS (ready after the barrier that ends it)
template <int RT, int NB, bool NN, int NW, int S>
__device__ __forceinline__ void prod_tile(const ProdArgs& a, int m0, int n0, char* lds) {
  constexpr int SCR = prod_scr<RT, NN, NB>();
  static_assert(!NN || 16 * NB == 64, "the NN product takes 64-column tiles");
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.M, N = a.N, K = a.K;
  f4 acc[RT][NB];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f4{0.f, 0.f, 0.f, 0.f};
  const int nbk = blocks(K);
  const int c0 = (nbk * wave) / NW, c1 = (nbk * (wave + 1)) / NW;
  Xpose X;
  X.init();
  char* scr = lds + wave * SCR;
  const Rows as = rows_of(a.A, unsigned(size_t(M) * K * 2), m0, K);  // < 4 GiB: the fits checks
  if constexpr (!NN) {
    const Frags bf = frags_of(a.B, N, nbk);
    nt_rows<RT, NB, S, true>(
        c0, c1, scr, X, acc, [&](int g, int h, int blk) -> u4v { return as.load(g, h, blk); },
        [&](int g, int c, int blk) -> u4v { return bf.load(n0 / 16 + g, 2 * blk + c); });
  } else {
    // B block: instruction p covers k rows 8 p + (lane >> 3) of the block, columns n0 + 8 (lane & 7) .. +7.
    // Row t of the block is stored as 128 bytes, its four 32-byte segments (16 columns each) permuted by
    // nn_swz(t), and a fragment (column l & 15 of a 16-column segment, 8 consecutive k) comes back with two
    // transposing reads (nn_frag).
    const int lane = tid & 63;
    // (rows k past K read zero, columns past N something whose results are unused)
    const Rows bs = rows_of(a.B, unsigned(size_t(K) * N * 2), 0, N);
    const unsigned bcol = unsigned(n0) * 2u;
    char* bt = scr + RT * kSlot;
    const int lr = lane >> 3, lp = lane & 7;  // row within the instruction, 16-byte piece of the row
    u4v va[S][RT][2], vb[S][8];
    pipeline<S>(
        c0, c1,
        [&](int blk, int s) {
#pragma unroll
          for (int g = 0; g < RT; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) va[s][g][h] = as.load(g, h, blk);
#pragma unroll
          for (int p = 0; p < 8; ++p) vb[s][p] = bload(bs.r, bs.voff, bcol + unsigned(blk * 64 + 8 * p) * bs.stride);
        },
        [&](int s) {
#pragma unroll
          for (int i = 0; i < RT; ++i) X.put(scr + i * kSlot, va[s][i][0], va[s][i][1]);
#pragma unroll
          for (int p = 0; p < 8; ++p) {
            const int t = 8 * p + lr;
            *(u4v*)(bt + t * 128 + 32 * ((lp >> 1) ^ nn_swz(t)) + 16 * (lp & 1)) = vb[s][p];
          }
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            bf16x8 fb[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) fb[nb] = nn_frag(bt, 32 * c, nb);
#pragma unroll
            for (int i = 0; i < RT; ++i) {
              const bf16x8 fa = X.get(scr + i * kSlot, c);
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) acc[i][nb] = mfma_bf16_16x16x32(fa, fb[nb], acc[i][nb]);
            }
          }
          __builtin_amdgcn_wave_barrier();  // the tiles are read before the next block is stored
        });
  }
  __syncthreads();  // every wave has left its scratch
  put_partials<RT, NB>((float*)lds, wave, acc);
  __syncthreads();
}

template <int RT, int NB, bool NN, int NW = kWaves, int S = NN ? 2 : (RT * NB >= 4 ? 3 : 4)>
__global__ __launch_bounds__(64 * NW) void prod_wide(ProdArgs a) {
  constexpr int TM = 16 * RT, TN = 16 * NB;
  const int tid = threadIdx.x, M = a.M, N = a.N;
  const int mg = (M + TM - 1) / TM, ntile = mg * ((N + TN - 1) / TN);
  const int w = tile_of(ntile);
  if (w >= ntile) return;
  const int m0 = (w % mg) * TM, n0 = (w / mg) * TN;
  __shared__ __attribute__((aligned(16))) char lds[lds_bytes<RT, NB, prod_scr<RT, NN, NB>(), NW>()];
  const float* ps = (const float*)lds;
  prod_tile<RT, NB, NN, NW, S>(a, m0, n0, lds);
  for (int pi = tid; pi < TM * TN; pi += 64 * NW) {
    const int ml = pi / TN, nl = pi % TN;
    const int m = m0 + ml;
    if (m >= M || n0 + nl >= N) continue;
    const float s = sum_partials<RT, NB, NW>(ps, ml, nl);
    const size_t o = (size_t)m * N + n0 + nl;
    a.out[o] = a.add ? a.add[o] + s : s;
  }
}

// ---- the residual MLP layer -------------------------------------------------
//
// z_l = y_l W_l^T + b_l over a 64 x 64 tile (rows x output columns).
// Forward: y_{l+1} = y_l + relu(z_l).  Adjoint (recomputation of layer l):
// ybar_{l+1} = nn_in (= ybar_{l+2} + zbar_{l+1} W_{l+1}, from the product
// launch before it) plus the loss seed; zbar_l = ybar_{l+1} 1[z_l > 0].
// The epilogue over a 16 RT x 64 tile: zsum(ml, nl) is z_l without its bias
// (or, CACHED, unused: z_l is a.zc_in), nn(ml, nl, o) is nn_in's element.
template <int MODE, int RT, bool CACHED, int NW, class ZS, class NNI>
__device__ __forceinline__ void mlp_epilogue(const MlpArgs& a, int tile, int m0, int n0, ZS zsum, NNI nn) {
  constexpr int TM = 16 * RT, TN = 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, B = a.B, w = a.w;
  float lterm = 0.f;
  for (int pi = tid; pi < TM * TN; pi += 64 * NW) {
#pragma clang fp contract(on)  // the same bits with and without the product
    const int ml = pi / TN, nl = pi % TN;
    const int m = m0 + ml, c = n0 + nl;
    if (m >= B || c >= w) continue;
    const size_t o = (size_t)m * w + c;
    const float z = CACHED ? a.zc_in[o] : zsum(ml, nl) + a.bias[c];
    if (MODE == kForward && a.zc_out) a.zc_out[o] = z;
    const float yv = (float)((const __bf16*)a.y)[o];
    const __bf16 y1s = (__bf16)(yv + fmaxf(z, 0.f));
    if (MODE == kForward) {
      ((__bf16*)a.y_out)[o] = y1s;
    } else {
      const float hl = (float)y1s;  // the loss reads the stored y_{l+1}
      float yb;
      if (a.first) {
        if (a.loss == AMBPTT_LOSS_HALF_SQ_LAST) {
          yb = hl;
          lterm += hl * hl;
        } else if (a.loss == AMBPTT_LOSS_MEAN_LAST) {
          yb = a.inv_bw;
          lterm += hl;
        } else {
          yb = 2.f * hl * a.inv_bw;
          lterm += hl * hl;
        }
      } else {
        yb = nn(ml, nl, o);
        if (a.loss == AMBPTT_LOSS_MEAN_SQ_ALL) {
          yb += 2.f * hl * a.inv_bw;
          lterm += hl * hl;
        }
      }
      a.ybar_out[o] = yb;
      ((__bf16*)a.zbar_out)[o] = (__bf16)(z > 0.f ? yb : 0.f);
      ((__bf16*)a.ywin_out)[o] = ((const __bf16*)a.y)[o];
    }
  }
  if (MODE == kAdjoint) {
    const float s = wave_sum(lterm);
    __shared__ float wsum[NW];
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) t += wsum[wv];
      a.loss_acc[tile] += (double)t;
    }
  }
}

template <int MODE, int RT, int NW = kWaves, int S = RT == 4 ? 2 : 3>
__global__ __launch_bounds__(64 * NW) void mlp_wide(MlpArgs a) {
  constexpr int NB = 4, TM = 16 * RT, TN = 64;
  constexpr int SCR = (RT + NB) * kSlot;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int B = a.B, w = a.w;
  const int mg = (B + TM - 1) / TM, ntile = mg * ((w + TN - 1) / TN);
  const int tile = tile_of(ntile);
  if (tile >= ntile) return;
  const int m0 = (tile % mg) * TM, n0 = (tile / mg) * TN;

  __shared__ __attribute__((aligned(16))) char lds[lds_bytes<RT, NB, SCR, NW>()];
  float* ps = (float*)lds;
  {
    f4 acc[RT][NB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[i][nb] = f4{0.f, 0.f, 0.f, 0.f};
    Xpose X;
    X.init();
    const int nbk = blocks(w);
    const int c0 = (nbk * wave) / NW, c1 = (nbk * (wave + 1)) / NW;
    const Rows ys = rows_of(a.y, unsigned(size_t(B) * w * 2), m0, w);  // < 4 GiB: mlp_wide_fits
    const Rows ws = rows_of(a.W, unsigned(size_t(w) * w * 2), n0, w);
    nt_rows<RT, NB, S>(
        c0, c1, lds + wave * SCR, X, acc, [&](int g, int h, int blk) -> u4v { return ys.load(g, h, blk); },
        [&](int g, int h, int blk) -> u4v { return ws.load(g, h, blk); });
    __syncthreads();  // every wave has left its scratch
    put_partials<RT, NB>(ps, wave, acc);
  }
  __syncthreads();

  mlp_epilogue<MODE, RT, false, NW>(
      a, tile, m0, n0, [&](int ml, int nl) { return sum_partials<RT, NB, NW>(ps, ml, nl); },
      [&](int, int, size_t o) { return a.nn_in[o]; });
}

// The adjoint of a layer whose z_l is kept: the product zbar_{l+1} W_{l+1}
// (on the same tiles) and the layer's own adjoint in one launch.
template <int RT, int NW = kWaves>
__global__ __launch_bounds__(64 * NW) void mlp_back_wide(MlpArgs a) {
  constexpr int TM = 16 * RT;
  const int mg = (a.B + TM - 1) / TM, ntile = mg * ((a.w + 63) / 64);
  const int tile = tile_of(ntile);
  if (tile >= ntile) return;
  const int m0 = (tile % mg) * TM, n0 = (tile / mg) * 64;
  __shared__ __attribute__((aligned(16))) char lds[lds_bytes<RT, 4, prod_scr<RT, true, 4>(), NW>()];
  const float* ps = (const float*)lds;
  const ProdArgs pa{a.zbar_in, a.Wn, nullptr, nullptr, a.B, a.w, a.w};
  prod_tile<RT, 4, true, NW, 2>(pa, m0, n0, lds);
  mlp_epilogue<kAdjoint, RT, true, NW>(
      a, tile, m0, n0, [](int, int) { return 0.f; },
      [&](int ml, int nl, size_t o) { return a.ybar_in[o] + sum_partials<RT, 4, NW>(ps, ml, nl); });
}

// 16-row groups per tile for M rows and `cols` column tiles: 64 rows where
// that makes 160 tiles or more, else 32, else 16.  Fewer rows read the weights
// more often from L2 but put more CUs to work (forward step, 64 / 32 / 16
// rows): 100 x 1536 x 1600 (tanh RNN) 12.7 / 9.6 / 7.2 us on 48 / 96 / 168
// tiles; the LSTM at B = 128, D = 256, H = 1024 11.3 / 8.5 / 10.6 on 128 / 256
// / 512; residual MLP layers 70 x 512 8.3 / 6.3 / 5.4, 128 x 2048 12.6 / 9.6 /
// 8.2, 256 x 2048 12.9 / 10.6 / 13.7; the 2048-LSTM (256 tiles of 64 rows)
// 16.0 / 20.3 / 25.9.
int tile_rows(int M, int cols) {
  for (int rt = 4; rt > 1; rt /= 2)
    if (((M + 16 * rt - 1) / (16 * rt)) * cols >= 160) return rt;
  return 1;
}
int row_tiles(int M, int cols) { return (M + 16 * tile_rows(M, cols) - 1) / (16 * tile_rows(M, cols)); }

unsigned grid_for(int ntile) { return unsigned(8 * ((ntile + 7) / 8)); }

// dst (fragment order, Frags) <- the [N][K0 + K1] rows of src (row stride ld),
// the two segments each padded to whole blocks: one thread per 16-byte lane
// chunk, written in order.
__global__ __launch_bounds__(256) void pack_nt(const char* __restrict__ src, int K0, int K1, int ld, size_t chunks,
                                               char* __restrict__ dst) {
  const size_t t = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= chunks) return;
  const int l = int(t & 63), b0 = blocks(K0);
  const size_t f = t >> 6, kf = 2 * size_t(b0 + blocks(K1));
  const size_t jt = f / kf;
  const int ks = int(f % kf);
  const bool first = ks < 2 * b0;
  const int k = 32 * (first ? ks : ks - 2 * b0) + 8 * (l >> 4);  // within the segment
  u4v v = {0u, 0u, 0u, 0u};
  if (k < (first ? K0 : K1)) {
    const size_t row = 16 * jt + size_t(l & 15);
    v = *(const u4v*)(src + 2 * (row * size_t(ld) + size_t(first ? k : K0 + k)));
  }
  *(u4v*)(dst + 16 * t) = v;
}

}  // namespace

size_t pack_nt_bytes(int N, int K0, int K1) { return size_t(N / 16) * size_t(blocks(K0) + blocks(K1)) * 2048; }

hipError_t launch_pack_nt_bf16(const void* src, int N, int K0, int K1, int ld, void* dst, hipStream_t s) {
  const size_t bytes = pack_nt_bytes(N, K0, K1);
  if (N < 16 || N % 16 != 0 || K0 < 0 || K1 < 32 || K0 % 32 != 0 || K1 % 32 != 0 || ld < K0 + K1 || ld % 8 != 0 ||
      bytes > 0xFFFFFFFFull)  // Frags addresses the copy with 32-bit offsets
    return hipErrorInvalidValue;
  const size_t chunks = bytes / 16;
  hipLaunchKernelGGL(pack_nt, dim3(unsigned((chunks + 255) / 256)), dim3(256), 0, s, (const char*)src, K0, K1, ld, chunks,
                     (char*)dst);
  return hipGetLastError();
}

// Every operand is addressed with 32-bit buffer offsets: each must stay under 4 GiB.
static bool under_4g(size_t rows, size_t cols) { return rows * (cols + 128) * 2 <= 0xFFFFFFFFull; }

bool cell_wide_fits(int G, int B, int D, int H) {
  return D % 32 == 0 && H % 32 == 0 && H > 0 && B > 0 && under_4g(size_t(B), size_t(D) + size_t(H)) &&
         under_4g(size_t(G) * H, size_t(D) + size_t(H)) && under_4g(size_t(B), size_t(G) * H) &&
         under_4g(size_t(H), size_t(G) * H);
}

bool mlp_wide_fits(int B, int w) { return w % 32 == 0 && w > 0 && B > 0 && under_4g(size_t(w) + 64, size_t(w)) && under_4g(size_t(B), size_t(w)); }

static int cell_cols(int G, int H) { return (H + 64 / G - 1) / (64 / G); }
int cell_wide_tiles(int G, int B, int H) { return row_tiles(B, cell_cols(G, H)) * cell_cols(G, H); }

template <int G, int RT>
static hipError_t launch_cell_wide_rt(int mode, const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(grid_for(cell_wide_tiles(G, a.B, a.H))), block(64 * kWaves);
  if (mode == kForward) hipExtLaunchKernelGGL((cell_wide<G, kForward, RT>), grid, block, 0, s, e0, e1, 0, a);
  else if (a.zc_in) hipExtLaunchKernelGGL((cell_wide<G, kAdjoint, RT, true>), grid, block, 0, s, e0, e1, 0, a);
  else hipExtLaunchKernelGGL((cell_wide<G, kAdjoint, RT>), grid, block, 0, s, e0, e1, 0, a);
  return hipGetLastError();
}

template <int G>
static hipError_t launch_cell_wide_g(int mode, const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (tile_rows(a.B, cell_cols(G, a.H))) {
    case 4: return launch_cell_wide_rt<G, 4>(mode, a, s, e0, e1);
    case 2: return launch_cell_wide_rt<G, 2>(mode, a, s, e0, e1);
    default: return launch_cell_wide_rt<G, 1>(mode, a, s, e0, e1);
  }
}

hipError_t launch_cell_wide(int G, int mode, const StepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if ((mode != kForward && mode != kAdjoint) || !cell_wide_fits(G, a.B, a.D, a.H)) return hipErrorInvalidValue;
  return G == 4 ? launch_cell_wide_g<4>(mode, a, s, e0, e1) : launch_cell_wide_g<1>(mode, a, s, e0, e1);
}

bool prod_wide_big(int M, int N) { return N % 32 == 0 && ((M + 31) / 32) * (N / 32) >= 192; }

hipError_t launch_prod_nt(const ProdArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.K % 32 != 0 || a.N % 16 != 0 || a.M < 1) return hipErrorInvalidValue;
  const dim3 block(64 * kWaves);
  if (prod_wide_big(a.M, a.N)) {
    const dim3 grid(grid_for(((a.M + 31) / 32) * (a.N / 32)));
    hipExtLaunchKernelGGL((prod_wide<2, 2, false>), grid, block, 0, s, e0, e1, 0, a);
  } else {
    const dim3 grid(grid_for(((a.M + 15) / 16) * (a.N / 16)));
    hipExtLaunchKernelGGL((prod_wide<1, 1, false>), grid, block, 0, s, e0, e1, 0, a);
  }
  return hipGetLastError();
}

int mlp_wide_tiles(int B, int w) { return row_tiles(B, blocks(w)) * blocks(w); }

hipError_t launch_prod_nn(const ProdArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.K % 32 != 0 || a.N % 32 != 0 || a.M < 1) return hipErrorInvalidValue;
  const dim3 grid(grid_for(mlp_wide_tiles(a.M, a.N))), block(64 * kWaves);
  switch (tile_rows(a.M, blocks(a.N))) {
    case 4: hipExtLaunchKernelGGL((prod_wide<4, 4, true>), grid, block, 0, s, e0, e1, 0, a); break;
    case 2: hipExtLaunchKernelGGL((prod_wide<2, 4, true>), grid, block, 0, s, e0, e1, 0, a); break;
    default: hipExtLaunchKernelGGL((prod_wide<1, 4, true>), grid, block, 0, s, e0, e1, 0, a); break;
  }
  return hipGetLastError();
}

template <int RT>
static hipError_t launch_mlp_wide_rt(int mode, const MlpArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(grid_for(mlp_wide_tiles(a.B, a.w))), block(64 * kWaves);
  if (mode == kForward) hipExtLaunchKernelGGL((mlp_wide<kForward, RT>), grid, block, 0, s, e0, e1, 0, a);
  else if (a.zc_in) hipExtLaunchKernelGGL((mlp_back_wide<RT>), grid, block, 0, s, e0, e1, 0, a);
  else hipExtLaunchKernelGGL((mlp_wide<kAdjoint, RT>), grid, block, 0, s, e0, e1, 0, a);
  return hipGetLastError();
}

static hipError_t launch_mlp_wide_any(int mode, const MlpArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  switch (tile_rows(a.B, blocks(a.w))) {
    case 4: return launch_mlp_wide_rt<4>(mode, a, s, e0, e1);
    case 2: return launch_mlp_wide_rt<2>(mode, a, s, e0, e1);
    default: return launch_mlp_wide_rt<1>(mode, a, s, e0, e1);
  }
}

hipError_t launch_mlp_back_wide(const MlpArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (!mlp_wide_fits(a.B, a.w) || a.first || !a.zc_in) return hipErrorInvalidValue;
  return launch_mlp_wide_any(kAdjoint, a, s, e0, e1);
}

hipError_t launch_mlp_wide(int mode, const MlpArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if ((mode != kForward && mode != kAdjoint) || !mlp_wide_fits(a.B, a.w) || (mode == kAdjoint && a.zc_in))
    return hipErrorInvalidValue;
  return launch_mlp_wide_any(mode, a, s, e0, e1);
}

}  // namespace ambptt
