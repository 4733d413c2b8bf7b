// bf16 MFMA GEMM for gfx950 with fused epilogues: C[M x N] = A[M x K] B[K x N],
// float32 accumulation (v_mfma_f32_32x32x16_bf16).
//
// Operand layouts: kOpKMajor (row r of the operand has K contiguous:
// X[r * ld + k]) and kOpRowMajorMN (X[k * ld + r]).
//
// Three kernels (launch_gemm_bf16 chooses): whole-K tiles
// (gemm_bf16_whole_kernel; over a very long K its parts side by side, with
// partial sums), few rows (gemm_bf16_few_kernel), and for the rest (few tiles
// over a long K, few columns over a short one, operands without 16-byte rows, the
// log-mel epilogues) the split-K kernel with its partial sums:
//
// Tiles of 128 x 128 x 32 per 256-thread workgroup (four wavefronts in 2 x 2,
// each 64 x 64 as 2 x 2 MFMA 32 x 32 blocks).  Tiles are staged in LDS as
// [row][k] with K contiguous (rows padded by 16 bytes, 16-byte k-chunks
// permuted per row, swz_k), so every lane's 8-element MFMA fragment is one
// 16-byte LDS read; the LDS tiles are double
// buffered and the next k-step is prefetched into registers.
//
// MFMA 32x32x16 lane layout (verified on gfx950): A fragment = row (lane % 32),
// k = 8 (lane / 32) .. +7; B fragment = column (lane % 32), same k; the 16
// accumulators of a lane are column (lane % 32), rows 8 (v / 4) + 4 (lane / 32)
// + (v % 4), v = 0..15.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "synth_internal.h"

namespace synth {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int BM = 128, BN = 128, BK = 32, PADK = BK + 8;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// float -> bf16, round to nearest even (NaN stays NaN)
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u));
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float gelu_erf(float x) {
  return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f));
}
// d/dx x Phi(x) = Phi(x) + x phi(x)
__device__ __forceinline__ float gelu_erf_grad(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752440f)) +
         x * 0.39894228040143267794f * expf(-0.5f * x * x);
}

__device__ __forceinline__ bool aligned16(const void* p) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

// 16 elements as eight 4-byte loads (rows of an even leading dimension that
// is not a multiple of 8, e.g. the MLP's 78-wide output rows)
__device__ __forceinline__ void load16_by4(const uint16_t* p, uint4& r0, uint4& r1) {
  const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
  r0 = make_uint4(q[0], q[1], q[2], q[3]);
  r1 = make_uint4(q[4], q[5], q[6], q[7]);
}

// Staging of a 128 x 32 tile (rows row0.., k k0..) of an operand into
// dst[row][k], in two phases so that the loads of the next k-step can be in
// flight during the MFMAs: load() fills two 16-byte registers per thread,
// store() writes them to LDS.
//   K-major: thread t takes row t / 2, k (t & 1) * 16 .. +15 (32 bytes).
//   row-major (X[k * ld + r]): thread t takes k t / 8, rows (t % 8) * 16 ..
//   +15, written to LDS transposed (16 two-byte writes).
// Rows of an even leading dimension that is not a multiple of 8 are read as
// 4-byte words.  Tiles at the matrix edge or at the end K of the k-range (or
// unaligned operands) are read element by element with bounds checks and zero
// fill.
template <int OP>
__device__ __forceinline__ void load_tile(uint4& r0, uint4& r1, int64_t K, const void* srcv,
                                          int64_t ld, int64_t row0, int64_t nrows, int64_t k0) {
  constexpr int G = 8;                // row-major: groups of 16 rows per k
  const int t = threadIdx.x;
  const uint16_t* src = reinterpret_cast<const uint16_t*>(srcv);
  uint16_t v[16];
  if constexpr (OP == kOpKMajor) {
    const int64_t gr = row0 + (t >> 1);
    const int64_t kb = k0 + (t & 1) * 16;
    if (gr < nrows && kb + 16 <= K && ((ld & 7) == 0) && aligned16(src)) {
      const uint4* p = reinterpret_cast<const uint4*>(src + gr * ld + kb);
      r0 = p[0];
      r1 = p[1];
      return;
    }
    if (gr < nrows && kb + 16 <= K && ((ld & 1) == 0) &&
        (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
      load16_by4(src + gr * ld + kb, r0, r1);
      return;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
      v[e] = (gr < nrows && kb + e < K) ? src[gr * ld + kb + e] : (uint16_t)0;
  } else {
    const int64_t gk = k0 + t / G;
    const int64_t gr = row0 + (t % G) * 16;
    if (gk < K && gr + 16 <= nrows && ((ld & 7) == 0) && aligned16(src)) {
      const uint4* p = reinterpret_cast<const uint4*>(src + gk * ld + gr);
      r0 = p[0];
      r1 = p[1];
      return;
    }
    if (gk < K && gr + 16 <= nrows && ((ld & 1) == 0) &&
        (reinterpret_cast<uintptr_t>(src) & 3u) == 0) {
      load16_by4(src + gk * ld + gr, r0, r1);
      return;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
      v[e] = (gk < K && gr + e < nrows) ? src[gk * ld + gr + e] : (uint16_t)0;
  }
  r0 = make_uint4(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16),
                  v[4] | ((uint32_t)v[5] << 16), v[6] | ((uint32_t)v[7] << 16));
  r1 = make_uint4(v[8] | ((uint32_t)v[9] << 16), v[10] | ((uint32_t)v[11] << 16),
                  v[12] | ((uint32_t)v[13] << 16), v[14] | ((uint32_t)v[15] << 16));
}

// LDS column of element k of tile row `row`: the four 8-element (16-byte)
// k-chunks of a row are permuted by (row / 16) mod 4.  The transposed stores
// of row-major operands (the lanes of a wavefront at 8 k values, 16 rows
// apart, rows 20 dwords apart) then spread over 16 banks instead of 4 (a
// 2-way instead of an 8-way conflict), and an MFMA fragment (8 consecutive
// k from a multiple of 8) is still one 16-byte read.
__device__ __forceinline__ int swz_k(int row, int k) { return k ^ (((row >> 4) & 3) << 3); }

template <int OP>
__device__ __forceinline__ void store_tile(const uint4& r0, const uint4& r1,
                                           uint16_t (*dst)[PADK]) {
  constexpr int G = 8;
  const int t = threadIdx.x;
  if constexpr (OP == kOpKMajor) {
    const int r = t >> 1, kk = (t & 1) * 16;
    *reinterpret_cast<uint4*>(&dst[r][swz_k(r, kk)]) = r0;
    *reinterpret_cast<uint4*>(&dst[r][swz_k(r, kk + 8)]) = r1;
  } else {
    const int kk = t / G, rr = (t % G) * 16;
    const uint32_t w[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
    const int kc = swz_k(rr, kk);       // rows rr .. rr + 15 share the permutation
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      dst[rr + 2 * e][kc] = (uint16_t)(w[e] & 0xFFFFu);
      dst[rr + 2 * e + 1][kc] = (uint16_t)(w[e] >> 16);
    }
  }
}

// Element (row, col) of the standard epilogues: x is alpha A B (+ bias added here).
__device__ __forceinline__ void epi_store(const GemmArgs& g, int64_t row, int64_t col, float x) {
  const int64_t o = row * g.ldc + col;
  if (g.bias) x += g.bias[col];
  if (g.pre) g.pre[o] = x;
  if (g.epilogue == kEpiGelu) x = gelu_erf(x);
  else if (g.epilogue == kEpiSigmoid) x = 1.0f / (1.0f + expf(-x));
  else if (g.epilogue == kEpiGeluGrad) x = x * gelu_erf_grad(g.aux[o]);
  if (g.beta != 0.0f)
    x += g.beta * (g.c_bf16 ? bf2f(reinterpret_cast<const uint16_t*>(g.C)[o])
                            : reinterpret_cast<const float*>(g.C)[o]);
  if (g.c_bf16) reinterpret_cast<uint16_t*>(g.C)[o] = f2bf(x);
  else reinterpret_cast<float*>(g.C)[o] = x;
}

// The standard epilogue for the 16 accumulators of one lane (column col,
// rows row0 + 8 (v / 4) + (v % 4)): the GELU' pre-activations it reads are
// loaded for all 16 first, so the loads are in flight together instead of
// one round trip per element.
__device__ __forceinline__ void epi_store16(const GemmArgs& g, int64_t row0, int64_t col,
                                            f32x16 acc) {
  if (col >= g.N) return;
  float aux[16];
  if (g.epilogue == kEpiGeluGrad) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t row = row0 + 8 * (v >> 2) + (v & 3);
      aux[v] = row < g.M ? g.aux[row * g.ldc + col] : 0.0f;
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int64_t row = row0 + 8 * (v >> 2) + (v & 3);
    if (row >= g.M) continue;
    float x = acc[v] * g.alpha;
    if (g.epilogue == kEpiGeluGrad) {
      const int64_t o = row * g.ldc + col;
      if (g.bias) x += g.bias[col];
      if (g.pre) g.pre[o] = x;
      x *= gelu_erf_grad(aux[v]);
      if (g.beta != 0.0f)
        x += g.beta * (g.c_bf16 ? bf2f(reinterpret_cast<const uint16_t*>(g.C)[o])
                                : reinterpret_cast<const float*>(g.C)[o]);
      if (g.c_bf16) reinterpret_cast<uint16_t*>(g.C)[o] = f2bf(x);
      else reinterpret_cast<float*>(g.C)[o] = x;
    } else {
      epi_store(g, row, col, x);
    }
  }
}

template <int AOP, int BOP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
    gemm_bf16_kernel(GemmArgs g) {
  __shared__ __align__(16) uint16_t As[2][BM][PADK];
  __shared__ __align__(16) uint16_t Bs[2][BN][PADK];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t tiles_n = (g.N + BN - 1) / BN;
  const int64_t tiles = ((g.M + BM - 1) / BM) * tiles_n;
  const int64_t tile = blockIdx.x % tiles;
  const int64_t tm = tile / tiles_n, tn = tile % tiles_n;
  const int64_t m0 = tm * BM, n0 = tn * BN;
  // split K: workgroup part p takes [kbeg, kend), a whole number of k-steps
  const int split = g.split > 1 ? g.split : 1;
  const int64_t part = blockIdx.x / tiles;
  const int64_t kper = ((g.K + split - 1) / split + BK - 1) / BK * BK;
  const int64_t kbeg = part * kper;
  const int64_t kend = kbeg + kper < g.K ? kbeg + kper : g.K;

  // four named accumulators (an array of them is not kept in registers)
  f32x16 s00 = {}, s01 = {}, s10 = {}, s11 = {};
#define SYNTH_SACC(i, j) ((i) == 0 ? ((j) == 0 ? s00 : s01) : ((j) == 0 ? s10 : s11))

  // LDS double buffer; the next k-step's tiles are loaded into registers
  // before this step's MFMAs and written to the other buffer after them.
  uint4 a0, a1, b0, b1;
  load_tile<AOP>(a0, a1, kend, g.A, g.lda, m0, g.M, kbeg);
  load_tile<BOP>(b0, b1, kend, g.B, g.ldb, n0, g.N, kbeg);
  store_tile<AOP>(a0, a1, As[0]);
  store_tile<BOP>(b0, b1, Bs[0]);
  __syncthreads();
  const int64_t nk = kend > kbeg ? (kend - kbeg + BK - 1) / BK : 0;
  for (int64_t ks = 0; ks < nk; ++ks) {
    const int buf = (int)(ks & 1);
    const bool more = ks + 1 < nk;
    if (more) {
      load_tile<AOP>(a0, a1, kend, g.A, g.lda, m0, g.M, kbeg + (ks + 1) * BK);
      load_tile<BOP>(b0, b1, kend, g.B, g.ldb, n0, g.N, kbeg + (ks + 1) * BK);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      const int kq = kk + 8 * (lane >> 5);
      bf16x8 af[2], bfr[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = wm * 64 + i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8*>(&As[buf][r][swz_k(r, kq)]);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int r = wn * 64 + j * 32 + (lane & 31);
        bfr[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf][r][swz_k(r, kq)]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          SYNTH_SACC(i, j) = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], SYNTH_SACC(i, j), 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (more) {
      store_tile<AOP>(a0, a1, As[buf ^ 1]);
      store_tile<BOP>(b0, b1, Bs[buf ^ 1]);
    }
    __syncthreads();
  }

  // ---- epilogue ----
  if (split > 1) {
    // raw partial sums; the reduction applies the epilogue
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int64_t col = n0 + wn * 64 + j * 32 + (lane & 31);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t row = m0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          if (col < g.N && row < g.M) g.partial[(part * g.M + row) * g.N + col] = SYNTH_SACC(i, j)[v];
        }
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t col = n0 + wn * 64 + j * 32 + (lane & 31);
      const bool col_ok = col < g.N;
      if (g.epilogue <= kEpiGeluGrad) {
        epi_store16(g, m0 + wm * 64 + i * 32 + 4 * (lane >> 5), col, SYNTH_SACC(i, j));
        continue;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = m0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        float x = SYNTH_SACC(i, j)[v] * g.alpha;
        if (g.epilogue == kEpiPowerPairs) {
          x += (g.bias && col_ok) ? g.bias[col] : 0.0f;
          // (Re, Im) sit in adjacent columns = adjacent lanes; every lane shuffles
          const float other = __shfl_xor(x, 1);
          if ((col & 1) == 0 && col_ok && row < g.M) {
            const float p = x * x + other * other;
            const int64_t o = row * g.ldc + (col >> 1);
            if (g.c_bf16) reinterpret_cast<uint16_t*>(g.C)[o] = f2bf(p);
            else reinterpret_cast<float*>(g.C)[o] = p;
          }
        } else if (col_ok && row < g.M) {    // kEpiLogMelT
          if (g.bias) x += g.bias[col];
          const int64_t o = (row / 64) * 8192 + col * 64 + (row % 64);
          reinterpret_cast<float*>(g.C)[o] = logf(x + 1e-6f);
        }
      }
    }
}

#undef SYNTH_SACC

// ---------------------------------------------------------------------------
// GEMM without partials: one workgroup computes its tile over the whole of K,
// the parts of a split reduction one after another.  A part's product starts
// from zero and is added to the running sum in part order, as the split-K
// kernels and their sum do, so the result is theirs bit for bit; what goes is
// the partials' way through memory (4 x 16.8 MB written and read for the
// MLP's first layer at batch 4096) and the second launch.
//
// Tile (32 MB WM) x (32 NB WN) x 64, WM x WN wavefronts, each MB x NB MFMA
// blocks of 32 x 32.  Operand tiles go from global memory straight to LDS
// (global_load_lds, 16 bytes per lane, 1 KB per wave instruction), two stages:
// the next stage's loads are issued behind the barrier that ends the previous
// stage's reads and have a whole stage of MFMAs to arrive.  The instruction
// writes the lanes' 16-byte pieces one after another, so the swizzles below,
// which spread a fragment's reads over all banks, are applied to the address
// each lane reads from:
//   K-major   [row][8 pieces of 8 k], piece c of row r in slot c ^ (r / 2 & 7):
//             a fragment (row = lane % 32, 8 consecutive k) is one 16-byte
//             read, and 16 neighbouring rows cover all 64 banks.
//   row-major [k][row], 64-byte runs of a k-row permuted by its index: a
//             fragment is two transposing reads (ds_read_b64_tr_b16: 16 lanes
//             read 4 k-rows of 16 elements and get 4 k of one row each;
//             lane layout checked on gfx950), the 4 k-rows in 4 different
//             64-byte runs, so no operand is transposed by stores.
//
// Bound by LDS bandwidth (a 128 x 128 stage moves 32 KB in and 96 KB out for
// 512 clocks of MFMA per SIMD): with the MFMAs taken out the 4096 x 1024 x 8192
// product takes 74 us, with the LDS reads out 71, whole 93 (737 TFLOP/s);
// eight wavefronts rather than four 64 x 64 ones 107 -> 93.  MLP training step
// at batch 4096: 562 -> 390 us (first layer with its GELU 100 + 22 -> 95 us,
// its weight gradient 124 + 18 -> 89, the 1024-wide products 33 + 20 -> 25 to
// 30, the weight gradient of the second layer 34 + 13 -> 34, the K = 78 input
// gradient 44 -> 24).
// ---------------------------------------------------------------------------
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;

constexpr int SK = 64;                       // k per stage
__device__ __align__(16) uint4 g_zero16;     // source of the k past a part's end

template <int TM>
__device__ __forceinline__ int run_swz(int k) {       // permutation of a k-row's 64-byte runs
  return TM >= 128 ? (k & 3) : ((k >> 1) & 1);
}

// 16-byte slot `at` of a staged tile: the row (row-major: the first of its 8
// rows) and the k it holds.
template <int OP, int TM>
__device__ __forceinline__ void slot_at(int at, int& row, int& kk) {
  if constexpr (OP == kOpKMajor) {
    row = at >> 3;
    kk = ((at & 7) ^ ((row >> 1) & 7)) * 8;
  } else {
    constexpr int PR = TM / 8;                                   // pieces per k-row
    kk = at / PR;
    const int p = at % PR;
    row = (((p >> 2) ^ run_swz<TM>(kk)) << 5) | ((p & 3) << 3);
  }
}

// One 16-byte-per-lane load from global memory straight to LDS (lds: the
// wavefront's 1 KB).  As asm, because behind the builtin the compiler waits
// for every such load in flight before the next LDS read, which it cannot tell
// from the bytes being loaded; the kernel waits for the stage it reads
// (wait_loads) and for nothing later.  The instruction writes no register.
__device__ __forceinline__ uint32_t lds_addr(const uint16_t* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint16_t*)p;
}
__device__ __forceinline__ void load_to_lds(uint32_t lds, const char* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds(uint32_t lds, const char* p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds), "v"(p)
               : "memory", "m0");
}

// One operand's loads, NW wavefronts, PW wave instructions each per stage.
// Rows past the operand's end are clamped (their products are not stored); k
// past a part's end read zeros.  ANY: an operand without 16-byte rows (an odd
// leading dimension or pointer, or a k or row count that is not a multiple of
// 8) goes element by element through registers, zero outside.
template <int OP, int TM, int NW, bool ANY>
struct Stager {
  static constexpr int PW = TM / (8 * NW);
  const char* ptr;               // element (tile row 0, next stage's k 0)
  int64_t ld;
  int row_lim;
  uint32_t lds0;                 // this wavefront's first slot in the first buffer
  uint32_t off[PW];

  __device__ __forceinline__ void init(const void* base, int64_t ld_, int64_t row0, int64_t rows,
                                       const uint16_t* lds) {
    ld = ld_;
    ptr = reinterpret_cast<const char*>(base) + 2 * (OP == kOpKMajor ? row0 * ld : row0);
    row_lim = (int)min((int64_t)TM, rows - row0);
    lds0 = __builtin_amdgcn_readfirstlane(lds_addr(lds) + (threadIdx.x >> 6) * PW * 1024);
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      int row, kk;
      slot_at<OP, TM>(slot(i), row, kk);
      if (OP == kOpKMajor) row = row < row_lim ? row : row_lim - 1;
      else row = row + 8 <= row_lim ? row : row_lim - 8;
      off[i] = OP == kOpKMajor ? 2u * ((uint32_t)row * (uint32_t)ld + (uint32_t)kk)
                               : 2u * ((uint32_t)kk * (uint32_t)ld + (uint32_t)row);
    }
  }
  __device__ __forceinline__ int slot(int i) const {
    return (int)((((threadIdx.x >> 6) * PW + i) << 6) + (threadIdx.x & 63));
  }
  // lds: the buffer's offset in bytes, kleft: the k that remain in the part
  __device__ __forceinline__ void load(uint32_t buf, uint16_t* lds, int kleft) {
    if constexpr (ANY) {
      load_any(lds, kleft);
    } else if (kleft >= SK) {
#pragma unroll
      for (int i = 0; i < PW; ++i) load_to_lds(lds0 + buf + i * 1024, ptr, off[i]);
    } else {
#pragma unroll
      for (int i = 0; i < PW; ++i) {
        int row, kk;
        slot_at<OP, TM>(slot(i), row, kk);
        load_to_lds(lds0 + buf + i * 1024,
                    kk < kleft ? ptr + off[i] : reinterpret_cast<const char*>(&g_zero16));
      }
    }
    ptr += 2 * (OP == kOpKMajor ? (int64_t)1 : ld) * (kleft < SK ? kleft : SK);
  }
  __device__ __forceinline__ void load_any(uint16_t* lds, int kleft) const {
    const uint16_t* src = reinterpret_cast<const uint16_t*>(ptr);
    const bool words = (ld & 1) == 0 && (reinterpret_cast<uintptr_t>(src) & 3u) == 0;
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      int row, kk;
      slot_at<OP, TM>(slot(i), row, kk);
      // 8 elements along k (K-major) or along the rows
      const uint16_t* p = src + (OP == kOpKMajor ? (int64_t)row * ld + kk : (int64_t)kk * ld + row);
      const int n = OP == kOpKMajor ? (row < row_lim ? kleft - kk : 0)
                                    : (kk < kleft ? row_lim - row : 0);
      uint32_t w[4] = {0, 0, 0, 0};
      if (words && n >= 8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = reinterpret_cast<const uint32_t*>(p)[e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e < n) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
      }
      *reinterpret_cast<uint4*>(lds + slot(i) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
};

// The MFMA fragment of the 32 rows from r0 at k (16 per MFMA, from k0) of a
// staged tile.
template <int OP, int TM>
__device__ __forceinline__ bf16x8 fragment(const uint16_t* lds, int r0, int k0) {
  const int lane = threadIdx.x & 63;
  if constexpr (OP == kOpKMajor) {
    const int row = r0 + (lane & 31), c = (k0 >> 3) + (lane >> 5);
    return *reinterpret_cast<const bf16x8*>(lds + ((row << 3) | (c ^ ((row >> 1) & 7))) * 8);
  } else {
    typedef __attribute__((address_space(3))) s16x4* tptr;
    // 16 lanes: 4 k-rows x 4 pieces of 4 elements
    const int k = k0 + 8 * (lane >> 5) + ((lane & 15) >> 2);
    const int c = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;       // within the 32 rows
    const uint16_t* p0 = lds + k * TM + (((r0 >> 5) ^ run_swz<TM>(k)) << 5) + c;
    const uint16_t* p1 = lds + (k + 4) * TM + (((r0 >> 5) ^ run_swz<TM>(k + 4)) << 5) + c;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr)p0);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tptr)p1);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

// The standard epilogue (as epi_store) of W neighbouring elements of one row.
template <int W>
struct alignas(4 * W) Vals {
  float v[W];
};
template <int W>
__device__ __forceinline__ Vals<W> epi_aux(const GemmArgs& g, int64_t o) {
  Vals<W> y = {};
  if (g.epilogue == kEpiGeluGrad) {
    if constexpr (W == 4) {
      const float4 a = *reinterpret_cast<const float4*>(g.aux + o);
      y = {a.x, a.y, a.z, a.w};
    } else {
      y.v[0] = g.aux[o];
    }
  }
  return y;
}
template <int W>
__device__ __forceinline__ void epi_row(const GemmArgs& g, int64_t o, Vals<W> x, const Vals<W>& bias,
                                        const Vals<W>& aux) {
#pragma unroll
  for (int e = 0; e < W; ++e) {
    x.v[e] = x.v[e] * g.alpha;
    if (g.bias) x.v[e] += bias.v[e];
  }
  if (g.pre) {
    if constexpr (W == 4)
      *reinterpret_cast<float4*>(g.pre + o) = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
    else
      g.pre[o] = x.v[0];
  }
  if (g.epilogue == kEpiGelu) {
#pragma unroll
    for (int e = 0; e < W; ++e) x.v[e] = gelu_erf(x.v[e]);
  } else if (g.epilogue == kEpiSigmoid) {
#pragma unroll
    for (int e = 0; e < W; ++e) x.v[e] = 1.0f / (1.0f + expf(-x.v[e]));
  } else if (g.epilogue == kEpiGeluGrad) {
#pragma unroll
    for (int e = 0; e < W; ++e) x.v[e] *= gelu_erf_grad(aux.v[e]);
  }
  float* cf = reinterpret_cast<float*>(g.C) + o;
  uint16_t* ch = reinterpret_cast<uint16_t*>(g.C) + o;
  if (g.beta != 0.0f) {
#pragma unroll
    for (int e = 0; e < W; ++e) x.v[e] += g.beta * (g.c_bf16 ? bf2f(ch[e]) : cf[e]);
  }
  if (g.c_bf16) {
    if constexpr (W == 4)
      *reinterpret_cast<uint2*>(ch) =
          make_uint2(f2bf(x.v[0]) | ((uint32_t)f2bf(x.v[1]) << 16),
                     f2bf(x.v[2]) | ((uint32_t)f2bf(x.v[3]) << 16));
    else
      ch[0] = f2bf(x.v[0]);
  } else {
    if constexpr (W == 4) *reinterpret_cast<float4*>(cf) = make_float4(x.v[0], x.v[1], x.v[2], x.v[3]);
    else cf[0] = x.v[0];
  }
}

// The epilogue of a TM x TN tile of sums in LDS ([TM][TN] float32): each
// thread takes W columns of every (NT W / TN)-th row, four rows at a time so
// that their reads of the pre-activations are in flight together.  From LDS
// and in a loop because 64 copies of erff as straight-line code (one per
// accumulator) cost more than the product: the instructions did not fit the
// cache (45 us of a 50 us kernel).
template <int TM, int TN, int NT, int W>
__device__ __forceinline__ void epi_tile(const GemmArgs& g, const float* c, int64_t m0, int64_t n0) {
  constexpr int TPR = TN / W, RS = NT / TPR;
  const int col = (threadIdx.x % TPR) * W, r0 = threadIdx.x / TPR;
  if (n0 + col >= g.N) return;
  Vals<W> bias = {};
  if (g.bias)
#pragma unroll
    for (int e = 0; e < W; ++e) bias.v[e] = g.bias[n0 + col + e];
  const int rows = (int)min((int64_t)TM, g.M - m0);
  const int64_t o = m0 * g.ldc + n0 + col;
  int r = r0;
#pragma unroll 1
  for (; r + 3 * RS < rows; r += 4 * RS) {
    Vals<W> y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = epi_aux<W>(g, o + (r + u * RS) * g.ldc);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      epi_row<W>(g, o + (r + u * RS) * g.ldc,
                 *reinterpret_cast<const Vals<W>*>(c + (r + u * RS) * TN + col), bias, y[u]);
  }
#pragma unroll 1
  for (; r < rows; r += RS)
    epi_row<W>(g, o + r * g.ldc, *reinterpret_cast<const Vals<W>*>(c + r * TN + col), bias,
               epi_aux<W>(g, o + r * g.ldc));
}

// s_waitcnt vmcnt(N), the other counters left free
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// PARTS: the parts of the sum are spread over grid.y, a run of them to each
// workgroup, and every part's product goes to g.partial for the split reduction.
template <int AOP, int BOP, int MB, int NB, int WM, int WN, int NS, bool AANY, bool PARTS>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2, 2)))
    gemm_bf16_whole_kernel(GemmArgs g) {
  constexpr int TM = 32 * MB * WM, TN = 32 * NB * WN, NW = WM * WN;
  constexpr int STAGE = (TM + TN) * SK;
  __shared__ __align__(16) uint16_t tile[NS][STAGE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int64_t tiles_n = (g.N + TN - 1) / TN;
  // each XCD takes a contiguous run of tiles (row-major): they share A's rows
  // and all of B through that XCD's L2
  const int64_t nblk = gridDim.x;
  const int64_t id = (nblk % 8 == 0) ? (int64_t)(blockIdx.x % 8) * (nblk / 8) + blockIdx.x / 8
                                     : (int64_t)blockIdx.x;
  const int64_t m0 = id / tiles_n * TM, n0 = id % tiles_n * TN;
  const int split = g.split > 1 ? g.split : 1;
  const int kper = (int)(((g.K + split - 1) / split + BK - 1) / BK * BK);
  // this workgroup's parts, their first k and (K) their end
  const int run = PARTS ? (split + (int)gridDim.y - 1) / (int)gridDim.y : split;
  const int p0 = PARTS ? (int)blockIdx.y * run : 0, p1 = min(split, p0 + run);
  const int k0 = (int)min(g.K, (int64_t)p0 * kper), K = (int)min(g.K, (int64_t)p1 * kper);

  Stager<AOP, TM, NW, AANY> sa;
  Stager<BOP, TN, NW, false> sb;
  sa.init(g.A, g.lda, m0, g.M, tile[0]);
  sb.init(g.B, g.ldb, n0, g.N, tile[0] + TM * SK);
  if constexpr (PARTS) {
    sa.ptr += 2 * (AOP == kOpKMajor ? (int64_t)1 : g.lda) * k0;
    sb.ptr += 2 * (BOP == kOpKMajor ? (int64_t)1 : g.ldb) * k0;
  }
  f32x16 sum[MB][NB] = {};
  // the stage to load next, NS - 1 ahead of the one computed: its k, its
  // part's end and its buffer
  int lk = k0, lend = min(k0 + kper, K), lbuf = 0;
  auto load_next = [&]() {
    if (lk >= K) return;
    const int left = lend - lk;
    sa.load(lbuf * STAGE * 2, tile[lbuf], left);
    sb.load(lbuf * STAGE * 2, tile[lbuf] + TM * SK, left);
    lbuf = lbuf + 1 < NS ? lbuf + 1 : 0;
    lk += SK;
    if (left <= SK) {
      lk = lend;
      lend = min(lend + kper, K);
    }
  };
  constexpr int LOADS = (AANY ? 0 : sa.PW) + sb.PW;          // per wave and stage
#pragma unroll
  for (int i = 0; i < NS - 1; ++i) load_next();
  // Fragments are read one k-step (16) ahead of the MFMAs that take them, the
  // next stage's first ones too: read at the head of their own step, the LDS
  // reads and the MFMAs of a wavefront follow one another instead of
  // overlapping (2000 clocks a stage against the 512 of its MFMAs).
  bf16x8 af[2][MB], bf[2][NB];
  auto read = [&](int slot, int b, int kk) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
      af[slot][i] = fragment<AOP, TM>(tile[b], (wm * MB + i) * 32, kk);
#pragma unroll
    for (int j = 0; j < NB; ++j)
      bf[slot][j] = fragment<BOP, TN>(tile[b] + TM * SK, (wn * NB + j) * 32, kk);
  };
  auto next_stage = [&](bool more) {
    // the next stage's tile is whole once the loads but those of the NS - 3
    // stages behind it have arrived in every wave; the barrier also ends the
    // reads of the previous stage's buffer, which load_next fills
    if (more) wait_loads<LOADS*(NS - 3)>();
    else wait_loads<0>();
    if constexpr (AANY) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  next_stage(lk < K);
  read(0, 0, 0);
  int buf = 0;
  for (int p = p0; p < p1; ++p) {
    f32x16 acc[MB][NB] = {};
    for (int left = min((int64_t)kper, K - (int64_t)p * kper); left > 0; left -= SK) {
      const int nbuf = buf + 1 < NS ? buf + 1 : 0;
#pragma unroll
      for (int q = 0; q < SK / 16; ++q) {
        if (q + 1 < SK / 16) read((q + 1) & 1, buf, (q + 1) * 16);
        else read((q + 1) & 1, nbuf, 0);             // past the last stage: not used
        if (q == SK / 16 - 2) {
          next_stage(lk < K);
          load_next();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[q & 1][i], bf[q & 1][j],
                                                                acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      buf = nbuf;
    }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if constexpr (PARTS) {
          const int64_t col = n0 + (wn * NB + j) * 32 + (lane & 31);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int64_t row = m0 + (wm * MB + i) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (col < g.N && row < g.M) g.partial[(p * g.M + row) * g.N + col] = acc[i][j][v];
          }
        } else {
          sum[i][j] += acc[i][j];
        }
      }
  }
  if constexpr (PARTS) return;
  // the sums to LDS (the last stage's reads are over behind the barrier)
  static_assert(sizeof(tile) >= TM * TN * sizeof(float), "the staging buffers hold the sums");
  __syncthreads();
  float* c = reinterpret_cast<float*>(tile);
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        c[((wm * MB + i) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * TN +
          (wn * NB + j) * 32 + (lane & 31)] = sum[i][j][v];
  __syncthreads();
  const bool vec = ((g.ldc | g.N) & 3) == 0 &&
                   ((reinterpret_cast<uintptr_t>(g.C) | reinterpret_cast<uintptr_t>(g.pre) |
                     reinterpret_cast<uintptr_t>(g.aux)) & 15u) == 0;
  if (vec) epi_tile<TM, TN, 64 * NW, 4>(g, c, m0, n0);
  else epi_tile<TM, TN, 64 * NW, 1>(g, c, m0, n0);
}

// ---------------------------------------------------------------------------
// Few rows (the proposal asked about some sounds): one workgroup per 32 x 32
// tile of C, its eight wavefronts each multiplying one part of the split
// reduction, K-major fragments read from memory straight into registers (128 k
// at a time, 16 loads in flight).  Up to 8 parts (grid.y 1) are added in part
// order from LDS: the split-K kernel's numbers without its partials' way
// through memory, its second launch and the padding of its 128-row tiles.
// More parts are spread over grid.y workgroups of 8, which write partials for
// gemm_split_reduce_kernel (all of the first layer's 64 parts in one
// workgroup kept only 32 CUs busy: 29 us at 16 rows against 20 in two
// launches before).  Bound by the latency of its few loads.
// ---------------------------------------------------------------------------
constexpr int kFewWaves = 8;

__global__ void __launch_bounds__(64 * kFewWaves) gemm_bf16_few_kernel(GemmArgs g) {
  __shared__ float part[kFewWaves][32 * 32];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int r = lane & 31, h = 8 * (lane >> 5);
  const int64_t tiles_n = (g.N + 31) / 32;
  const int64_t m0 = blockIdx.x / tiles_n * 32, n0 = blockIdx.x % tiles_n * 32;
  const int K = (int)g.K, split = g.split > 1 ? g.split : 1;
  const int kper = (int)(((g.K + split - 1) / split + BK - 1) / BK * BK);
  const int p = blockIdx.y * kFewWaves + wave;
  const bool a_ok = m0 + r < g.M, b_ok = n0 + r < g.N;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(g.A) + (a_ok ? m0 + r : 0) * g.lda + h;
  const uint16_t* B = reinterpret_cast<const uint16_t*>(g.B) + (b_ok ? n0 + r : 0) * g.ldb + h;
  const int kbeg = (int)min((int64_t)p * kper, g.K), kend = p < split ? min(kbeg + kper, K) : kbeg;
  f32x16 acc = {};
  for (int k = kbeg; k < kend; k += 128) {
    bf16x8 af[8], bf[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bool in = k + 16 * s + h < kend;
      af[s] = in && a_ok ? *reinterpret_cast<const bf16x8*>(A + k + 16 * s) : bf16x8{};
      bf[s] = in && b_ok ? *reinterpret_cast<const bf16x8*>(B + k + 16 * s) : bf16x8{};
    }
#pragma unroll
    for (int s = 0; s < 8; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s], bf[s], acc, 0, 0, 0);
  }
  if (gridDim.y > 1) {
    if (p < split && b_ok) {
      float* dst = g.partial + (p * g.M + m0) * g.N + n0 + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (m0 + row < g.M) dst[row * g.N] = acc[v];
      }
    }
    return;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v)
    part[wave][(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 32 + r] = acc[v];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 1024; e += 64 * kFewWaves) {
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < kFewWaves; ++q)
      if (q < split) sum += part[q][t + e];
    const int64_t row = m0 + ((t + e) >> 5), col = n0 + (t & 31);
    if (row < g.M && col < g.N) epi_store(g, row, col, sum * g.alpha);
  }
}

// Sum of the split-K partials in part order, then the epilogue.
__global__ void __launch_bounds__(256) gemm_split_reduce_kernel(GemmArgs g) {
  // One workgroup per output row (rows strided over the grid): the row's
  // columns are read from each part as 16-byte vectors when N is a multiple
  // of 4 and the workspace 16-byte aligned, else one by one; no index
  // division.
  const int64_t n = g.M * g.N;
  const int t = threadIdx.x;
  const bool vec = (g.N & 3) == 0 && (reinterpret_cast<uintptr_t>(g.partial) & 15u) == 0;
  for (int64_t row = blockIdx.x; row < g.M; row += gridDim.x) {
    const float* src = g.partial + row * g.N;
    if (vec) {
      for (int64_t c4 = t; 4 * c4 < g.N; c4 += 256) {
        float4 x = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int p = 0;
        for (; p + 4 <= g.split; p += 4) {     // four parts' loads in flight, added in order
          float4 v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(src + (p + u) * n + 4 * c4);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            x.x += v[u].x;
            x.y += v[u].y;
            x.z += v[u].z;
            x.w += v[u].w;
          }
        }
        for (; p < g.split; ++p) {
          const float4 v = *reinterpret_cast<const float4*>(src + p * n + 4 * c4);
          x.x += v.x;
          x.y += v.y;
          x.z += v.z;
          x.w += v.w;
        }
        epi_store(g, row, 4 * c4, x.x * g.alpha);
        epi_store(g, row, 4 * c4 + 1, x.y * g.alpha);
        epi_store(g, row, 4 * c4 + 2, x.z * g.alpha);
        epi_store(g, row, 4 * c4 + 3, x.w * g.alpha);
      }
    } else {
      for (int64_t col = t; col < g.N; col += 256) {
        float x = 0.0f;
        int p = 0;
        for (; p + 4 <= g.split; p += 4) {
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = src[(p + u) * n + col];
#pragma unroll
          for (int u = 0; u < 4; ++u) x += v[u];
        }
        for (; p < g.split; ++p) x += src[p * n + col];
        epi_store(g, row, col, x * g.alpha);
      }
    }
  }
}

// The same sum of a small output (up to 2^17 elements), where one workgroup a
// row leaves most CUs idle and one thread adds 4 columns' parts 4 at a time:
// one element per thread, 16 parts' loads in flight (16 x 1024 of 64 parts:
// 9 -> 4 us).
__global__ void __launch_bounds__(64) gemm_split_reduce_small_kernel(GemmArgs g) {
  const int64_t n = g.M * g.N, i = blockIdx.x * (int64_t)64 + threadIdx.x;
  if (i >= n) return;
  const float* src = g.partial + i;
  float x = 0.0f;
  int p = 0;
  for (; p + 16 <= g.split; p += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = src[(p + u) * n];
#pragma unroll
    for (int u = 0; u < 16; ++u) x += v[u];
  }
  for (; p < g.split; ++p) x += src[p * n];
  epi_store(g, i / g.N, i % g.N, x * g.alpha);
}

hipError_t launch_reduce(const GemmArgs& g, hipStream_t s) {
  if (g.M * g.N <= ((int64_t)1 << 17)) {
    hipLaunchKernelGGL(gemm_split_reduce_small_kernel, dim3((unsigned)((g.M * g.N + 63) / 64)),
                       dim3(64), 0, s, g);
  } else {
    const int64_t blocks = g.M < 65535 ? g.M : 65535;
    hipLaunchKernelGGL(gemm_split_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, g);
  }
  return hipGetLastError();
}

template <int AOP>
hipError_t launch_b(const GemmArgs& g, int b_op, dim3 grid, hipStream_t s) {
  if (b_op == kOpKMajor)
    hipLaunchKernelGGL((gemm_bf16_kernel<AOP, kOpKMajor>), grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((gemm_bf16_kernel<AOP, kOpRowMajorMN>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

// Whether an operand's tiles can be loaded in 16-byte pieces (rows is the
// operand's row count, the offsets in a tile 32-bit).
bool pieces16(const void* p, int op, int64_t ld, int64_t rows, int64_t K) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && ld % 8 == 0 && ld <= ((int64_t)1 << 22) &&
         (op == kOpKMajor ? K : rows) % 8 == 0;
}

// Tiles of 32 MB WM x 32 NB WN.
template <int AOP, int BOP, int MB, int NB, int WM, int WN, int NS>
hipError_t launch_whole(const GemmArgs& g, bool a16, hipStream_t s) {
  constexpr int TM = 32 * MB * WM, TN = 32 * NB * WN;
  const int64_t tiles = ((g.M + TM - 1) / TM) * ((g.N + TN - 1) / TN);
  if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (a16)
    hipLaunchKernelGGL((gemm_bf16_whole_kernel<AOP, BOP, MB, NB, WM, WN, NS, false, false>),
                       dim3((unsigned)tiles), dim3(64 * WM * WN), 0, s, g);
  else
    hipLaunchKernelGGL((gemm_bf16_whole_kernel<AOP, BOP, MB, NB, WM, WN, NS, true, false>),
                       dim3((unsigned)tiles), dim3(64 * WM * WN), 0, s, g);
  return hipGetLastError();
}

// 128 x 128 tiles of K-major operands, the parts spread over `groups` workgroups
// a tile, then their sum.
hipError_t launch_parts(const GemmArgs& g, int groups, hipStream_t s) {
  const int64_t tiles = ((g.M + 127) / 128) * ((g.N + 127) / 128);
  hipLaunchKernelGGL((gemm_bf16_whole_kernel<kOpKMajor, kOpKMajor, 2, 1, 2, 4, 4, false, true>),
                     dim3((unsigned)tiles, (unsigned)groups), dim3(512), 0, s, g);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_reduce(g, s);
}

template <int... T>
hipError_t launch_whole_ops(const GemmArgs& g, int a_op, int b_op, bool a16, hipStream_t s) {
  if (a_op == kOpKMajor)
    return b_op == kOpKMajor ? launch_whole<kOpKMajor, kOpKMajor, T...>(g, a16, s)
                             : launch_whole<kOpKMajor, kOpRowMajorMN, T...>(g, a16, s);
  return b_op == kOpKMajor ? launch_whole<kOpRowMajorMN, kOpKMajor, T...>(g, a16, s)
                           : launch_whole<kOpRowMajorMN, kOpRowMajorMN, T...>(g, a16, s);
}

}  // namespace

constexpr int64_t kLongK = 12288, kFewWork = (int64_t)1 << 20;   // see launch_gemm_bf16

// The number of parts a product's sum over K is taken in.  Each part starts
// from zero and the parts are added in order, so the number is part of the
// result; every kernel here keeps to it, whether it spreads the parts over
// workgroups or takes them one after another.
int gemm_split_for(int64_t M, int64_t N, int64_t K) {
  int64_t split = 1;
  if (M % 256 == 0 && N % 256 == 0 && K % BK == 0 && K > 0) {
    const int64_t tiles = (M / 256) * (N / 256);
    while (tiles * split < 256 && K >= split * 2 * 8 * BK) split *= 2;
    return (int)split;
  }
  const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  while (tiles * split < 512 && K >= split * 2 * 4 * BK) split *= 2;
  return (int)split;
}

size_t gemm_split_bytes(int64_t M, int64_t N, int split) {
  return split > 1 ? (size_t)split * (size_t)M * (size_t)N * sizeof(float) : 0;
}

hipError_t launch_gemm_bf16(const GemmArgs& g, int a_op, int b_op, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  const int split = g.split > 1 ? g.split : 1;
  if (split > 1 && (!g.partial || g.epilogue > kEpiGeluGrad)) return hipErrorInvalidValue;
  if ((a_op != kOpKMajor && a_op != kOpRowMajorMN) || (b_op != kOpKMajor && b_op != kOpRowMajorMN))
    return hipErrorInvalidValue;
  hipError_t e;
  if (g.epilogue <= kEpiGeluGrad && g.K > 0 && g.K < ((int64_t)1 << 30) &&
      pieces16(g.B, b_op, g.ldb, g.N, g.K)) {
    const bool a16 = pieces16(g.A, a_op, g.lda, g.M, g.K);
    const int64_t t32 = ((g.M + 31) / 32) * ((g.N + 31) / 32);
    const int64_t t64 = ((g.M + 63) / 64) * ((g.N + 63) / 64);
    const int64_t t256 = ((g.M + 255) / 256) * ((g.N + 127) / 128);
    const int64_t t128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    const bool k_major = a_op == kOpKMajor && b_op == kOpKMajor && a16;
    // Few rows.  With more than 8 parts every 32 x 32 tile re-reads its
    // operands over all of K: up to tiles x K of 2^20 (MLP forward, us: 16 rows 45
    // -> 23, 128 rows 46 -> 44; 200 rows by this kernel 57, by the split one 40;
    // of 16384 inputs 64 rows 51 -> 41, 128 rows by this kernel 59, split 50).
    if (k_major && split > 1 && (split > kFewWaves ? t32 * g.K <= kFewWork : t32 <= 512)) {
      const int groups = (split + kFewWaves - 1) / kFewWaves;
      hipLaunchKernelGGL(gemm_bf16_few_kernel, dim3((unsigned)t32, (unsigned)groups),
                         dim3(64 * kFewWaves), 0, s, g);
      e = hipGetLastError();
      return e != hipSuccess || groups == 1 ? e : launch_reduce(g, s);
    }
    // A long K over up to half as many tiles as CUs: its parts side by side
    // (MLP forward of 65536 inputs, us, split kernel, whole tiles, parts: 512 rows
    // 179, 339, 141; 1100 rows 551, 582, 284; of 16384 inputs 512 rows 86, 109,
    // 73).  Below this line whole tiles are no slower than the split kernel was.
    if (k_major && split > 1 && g.K >= kLongK && t128 <= 128)
      return launch_parts(g, (int)(256 / t128 < split ? 256 / t128 : split), s);
    // Up to 32 columns and a short K over more than a tile a CU: whole tiles, one
    // workgroup a CU, have nothing to hide their loads and stores behind; the split
    // kernel has four (1000000 x 16, us, whole and split: K = 32 140 and 94, 64 141
    // and 124, 128 172 and 188; K-major 262144 x 32 x 96 45 and 42, row-major 46
    // and 46; 20000 rows 8.3 and 9).
    const bool narrow = g.N <= 32 && g.K <= (a_op == kOpKMajor ? 96 : 64) && t128 > 256;
    // 256 x 128 tiles where they fill the chip and K is more than their
    // longer prologue (1024 x 8192 x 4096: 106 -> 81 us against 128 x 128);
    // 128 x 128 from where 64 x 64 ones would need a second round (0.7 us a
    // stage against 0.4 twice).  Few 64 x 64 tiles over a long K leave CUs
    // idle for all of it: those keep to the split kernel (MLP forward of 333
    // rows: 65 us split, 77 whole; 512 rows: 88 and 70).
    if (t256 >= 192 && g.K > 512) return launch_whole_ops<2, 2, 4, 2, 3>(g, a_op, b_op, a16, s);
    if (t64 > 256 && !narrow) return launch_whole_ops<2, 1, 2, 4, 4>(g, a_op, b_op, a16, s);
    if (!narrow && (split == 1 || t64 >= (g.K > 2048 ? 128 : 64)))
      return launch_whole_ops<1, 1, 2, 2, 8>(g, a_op, b_op, a16, s);
  }
  const int64_t tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  if (tiles * split > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(tiles * split));
  e = a_op == kOpKMajor ? launch_b<kOpKMajor>(g, b_op, grid, s)
                        : launch_b<kOpRowMajorMN>(g, b_op, grid, s);
  if (e != hipSuccess || split == 1) return e;
  return launch_reduce(g, s);
}

}  // namespace synth
