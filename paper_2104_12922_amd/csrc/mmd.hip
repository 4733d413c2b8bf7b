// Sums of pairwise L1 distances between two sets of embeddings, and the
// maximum mean discrepancy built from them (Section 5, equation "mmd": sets
// of sounds compared through an auditory distance d; here d is the L1
// distance between embedding vectors):
//   S(A, B) = sum_{i < n, j < m} sum_k |A[i][k] - B[j][k]|
//   MMD(X, Y) = 2 S(X, Y) / (n m) - S(X, X) / n^2 - S(Y, Y) / m^2.
//
// Two kernels: one sorts each dimension's values (sets of up to 2048 sounds,
// sorted_pair_sum_kernel below), one takes all pairs (l1_pair_sum_kernel, beyond
// that and where the dimensions are too few for a sort, there in float64):
//
// Workgroups of 256 threads take tiles of 64 x 64 pairs and one share of
// the embedding dimension (whole runs of 256 dimensions, so tiles x shares
// fills the chip even for sets of a few hundred sounds).  The dimension is
// walked in chunks of 32 staged in LDS (rows padded to 36 floats).  Thread
// (ty, tx) holds the 4 x 4 pairs rows ty + 16 a, columns tx + 16 b: per four
// staged dimensions, 8 16-byte LDS reads (conflict-free: the A reads are
// broadcasts, B rows 36 floats apart cover distinct banks) feed 64 |x - y|
// accumulations.  A pair's distance is accumulated in float32 (or float64) over
// each run of 256 dimensions, then added to a float64 accumulator; a workgroup sums
// its pairs in a fixed order, and a second kernel sums the workgroups in
// order, so S is bitwise reproducible and S(X, X) equals S(A = X, B = X).
// Bound by VALU issue: two instructions (subtract, add of the absolute
// value) per pair and dimension (float64 at half the rate); padding past the last
// dimension is skipped by fours (2000 x 2000 of 8 dimensions 15 -> 14 us for one
// sum, which its launches bound, 5000 x 5000 58 -> 36).
#include <algorithm>

#include "synth_internal.h"

namespace synth {
namespace {

constexpr int kPT = 64;          // pairs per tile side
constexpr int kPK = 32;          // dimensions per LDS chunk
constexpr int kPLd = 36;         // padded LDS row (floats)
constexpr int kF32Run = 256;     // dimensions accumulated in float32 before promotion
constexpr int64_t kFillBlocks = 1024;

struct PairPlan {
  int64_t tiles_n, tiles_m, shares, runs_per_share;
};

PairPlan pair_plan(int64_t n, int64_t m, int64_t dim) {
  PairPlan p;
  p.tiles_n = (n + kPT - 1) / kPT;
  p.tiles_m = (m + kPT - 1) / kPT;
  const int64_t tiles = p.tiles_n * p.tiles_m;
  const int64_t runs = dim > 0 ? (dim + kF32Run - 1) / kF32Run : 1;
  int64_t want = tiles >= kFillBlocks ? 1 : (kFillBlocks + tiles - 1) / (tiles > 0 ? tiles : 1);
  if (want > runs) want = runs;
  p.runs_per_share = (runs + want - 1) / want;
  p.shares = (runs + p.runs_per_share - 1) / p.runs_per_share;
  return p;
}

// Stage rows r0 .. r0 + 63, dimensions k0 .. k0 + 31 of X (rows < rows, dims
// < dim; anything outside reads as 0, and |0 - 0| adds nothing).
template <class T>
struct alignas(16) Vec4 {
  T x, y, z, w;
};
template <class T>
__device__ __forceinline__ void stage_rows(T (*S)[kPLd], const float* __restrict__ X,
                                           int64_t ld, int64_t rows, int64_t r0, int64_t k0,
                                           int64_t dim, bool vec) {
  const int t = threadIdx.x;
  const int lr = t >> 2, lk = (t & 3) * 8;
  const int64_t r = r0 + lr, k = k0 + lk;
  float4 v0 = make_float4(0.f, 0.f, 0.f, 0.f), v1 = v0;
  if (r < rows) {
    const float* p = X + r * ld + k;
    if (vec && k + 8 <= dim) {
      v0 = *reinterpret_cast<const float4*>(p);
      v1 = *reinterpret_cast<const float4*>(p + 4);
    } else {
      float e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = (k + i < dim) ? p[i] : 0.0f;
      v0 = make_float4(e[0], e[1], e[2], e[3]);
      v1 = make_float4(e[4], e[5], e[6], e[7]);
    }
  }
  typedef Vec4<T> V;
  *reinterpret_cast<V*>(&S[lr][lk]) = V{(T)v0.x, (T)v0.y, (T)v0.z, (T)v0.w};
  *reinterpret_cast<V*>(&S[lr][lk + 4]) = V{(T)v1.x, (T)v1.y, (T)v1.z, (T)v1.w};
}

__device__ __forceinline__ float magnitude(float x) { return fabsf(x); }
__device__ __forceinline__ double magnitude(double x) { return fabs(x); }

// T: of the differences and their sums over a run.
template <class T>
__global__ void __launch_bounds__(256) l1_pair_sum_kernel(const float* __restrict__ A, int64_t lda,
                                                          int64_t n, const float* __restrict__ B,
                                                          int64_t ldb, int64_t m, int64_t dim,
                                                          PairPlan plan, int vec,
                                                          double* __restrict__ partial) {
  __shared__ __align__(16) T As[kPT][kPLd];
  __shared__ __align__(16) T Bs[kPT][kPLd];
  __shared__ double red[256];
  const int t = threadIdx.x;
  const int tx = t & 15, ty = t >> 4;
  const int64_t share = blockIdx.x % plan.shares;
  const int64_t tile = blockIdx.x / plan.shares;
  const int64_t i0 = (tile / plan.tiles_m) * kPT, j0 = (tile % plan.tiles_m) * kPT;
  const int64_t kbeg = share * plan.runs_per_share * kF32Run;
  int64_t kend = kbeg + plan.runs_per_share * kF32Run;
  if (kend > dim) kend = dim;
  T acc[4][4] = {};
  double dacc[4][4] = {};
  for (int64_t k0 = kbeg; k0 < kend; k0 += kPK) {
    stage_rows(As, A, lda, n, i0, k0, kend, vec != 0);
    stage_rows(Bs, B, ldb, m, j0, k0, kend, vec != 0);
    __syncthreads();
    const int left = (int)min(kend - k0, (int64_t)kPK);
#pragma unroll
    for (int kk = 0; kk < kPK; kk += 4) {
      if (kk >= left) break;               // nothing but padding
      Vec4<T> xa[4], yb[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) xa[a] = *reinterpret_cast<const Vec4<T>*>(&As[ty + 16 * a][kk]);
#pragma unroll
      for (int b = 0; b < 4; ++b) yb[b] = *reinterpret_cast<const Vec4<T>*>(&Bs[tx + 16 * b][kk]);
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          acc[a][b] += magnitude(xa[a].x - yb[b].x);
          acc[a][b] += magnitude(xa[a].y - yb[b].y);
          acc[a][b] += magnitude(xa[a].z - yb[b].z);
          acc[a][b] += magnitude(xa[a].w - yb[b].w);
        }
    }
    __syncthreads();
    if ((k0 + kPK - kbeg) % kF32Run == 0 || k0 + kPK >= kend) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          dacc[a][b] += (double)acc[a][b];
          acc[a][b] = 0;
        }
    }
  }
  // this thread's pairs inside the sets, in a fixed order
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (i0 + ty + 16 * a < n && j0 + tx + 16 * b < m) s += dacc[a][b];
  red[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) partial[blockIdx.x] = red[0];
}

// out[0] = sum of partial[0 .. count) in order (one workgroup: per-thread
// strided sums, then a fixed tree).
__global__ void __launch_bounds__(256) ordered_sum_kernel(const double* __restrict__ partial,
                                                          int64_t count, double* __restrict__ out) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  double s = 0.0;
  for (int64_t i = t; i < count; i += 256) s += partial[i];
  red[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) out[0] = red[0];
}

// out[0] = 2 s_xy / (n m) - s_xx / n^2 - s_yy / m^2 from out[1..3].
__global__ void mmd_combine_kernel(double* out, int64_t n, int64_t m) {
  if (threadIdx.x == 0) {
    const double dn = (double)n, dm = (double)m;
    out[0] = 2.0 * out[1] / (dn * dm) - out[2] / (dn * dn) - out[3] / (dm * dm);
  }
}

// ---------------------------------------------------------------------------
// Pair sums by sorting.  S(A, B) needs no single pair's distance, only the sum
// over all pairs, and that follows from each dimension's values in ascending
// order: the gap between neighbours k and k + 1 of the merged values of A and
// B counts once for every pair it separates, so with a and b values of A and
// B up to k
//   S(A, B) = sum_k gap_k (a (m - b) + b (n - a)),
//   S(A, A) = sum_k gap_k 2 a (n - a),   S(B, B) = sum_k gap_k 2 b (m - b):
// (n + m) log^2(n + m) operations per dimension instead of n m + n n + m m,
// all terms non-negative and all sums float64 (the all-pairs kernel adds a
// distance in float32 over runs of 256 dimensions; against float64 the three
// sums of 1000 x 1000 x 8192 log-mel-like features were 4.1e-8 off and are
// 1e-15 off).  For B = A every term of the three sums is the same number, so
// MMD(X, X) is exactly 0 here too.
//
// One wavefront sorts one dimension in registers: lanes 0-31 hold A, lanes
// 32-63 hold B, R values each (32 R >= max(n, m), the rest padded with the
// largest float).  Bitonic sort in the form whose merges begin with a mirrored
// exchange, so every comparison is ascending: distances below R are register
// pairs (one min and one max), lane distances are DPP moves and one median
// with +-infinity per value.  The last merge, of A with B, has to remember
// where a value came from: it runs on the values as float64, whose 29 spare
// mantissa bits hold the mark.  A workgroup of C wavefronts stages C
// neighbouring dimensions of all rows through LDS (C floats = 64 bytes of a
// row, padded to C + 1: the lanes of a wavefront read 32 rows of one dimension
// from distinct banks).
//
// Bound by VALU issue at R = 32 (5200 instructions per wavefront, which sorts a
// dimension; by counter the VALU is busy for 79% of the launch, at 2.9 of the
// four wavefronts per SIMD that fit).  MMD of 1000 x 1000 sounds of 8192
// features: 1.31 ms (three all-pairs launches) -> 0.08 ms.
// ---------------------------------------------------------------------------
constexpr int kSortFlagNan = 1, kSortFlagPos = 2, kSortFlagNeg = 4;

__device__ __forceinline__ int sort_key(float x) {      // monotone int of a float
  const int i = __float_as_int(x);
  return i ^ ((i >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float sort_value(int k) {    // and back
  return __int_as_float(k ^ ((k >> 31) & 0x7FFFFFFF));
}

__device__ __forceinline__ int med3_i32(int x, int y, int z) {
  // z = INT_MAX gives max(x, y), INT_MIN gives min(x, y): the compiler folds
  // this shape to one v_med3_i32
  const int lo = x < y ? x : y, hi = x < y ? y : x;
  const int c = hi < z ? hi : z;
  return lo > c ? lo : c;
}

// Value of lane (lane ^ D) for D = 1, 2, 4, 8, 16 and of the mirrored lane of
// a group of 2, 4, 8, 16, 32, 64 lanes.
template <int CTRL>
__device__ __forceinline__ int dpp(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}
template <int D>
__device__ __forceinline__ int lane_xor(int x) {
  if constexpr (D == 1) return dpp<0xB1>(x);                       // quad_perm 1,0,3,2
  else if constexpr (D == 2) return dpp<0x4E>(x);                  // quad_perm 2,3,0,1
  else if constexpr (D == 4) return dpp<0x1B>(dpp<0x141>(x));      // half mirror (^7), then ^3
  else if constexpr (D == 8) return dpp<0x128>(x);                 // rotate a row of 16 by 8
  else return __shfl_xor(x, D);
}
template <int G>
__device__ __forceinline__ int lane_mirror(int x) {
  if constexpr (G == 2) return dpp<0xB1>(x);
  else if constexpr (G == 4) return dpp<0x1B>(x);
  else if constexpr (G == 8) return dpp<0x141>(x);
  else if constexpr (G == 16) return dpp<0x140>(x);
  else return __shfl_xor(x, G - 1);
}

__device__ __forceinline__ double pack(int lo, int hi) {
  return __hiloint2double(hi, lo);
}
template <int D>
__device__ __forceinline__ double lane_xor(double x) {
  return pack(lane_xor<D>(__double2loint(x)), lane_xor<D>(__double2hiint(x)));
}
template <int G>
__device__ __forceinline__ double lane_mirror(double x) {
  return pack(lane_mirror<G>(__double2loint(x)), lane_mirror<G>(__double2hiint(x)));
}

// The lane keeps the smaller (up false) or the larger of its value and p.
__device__ __forceinline__ int keep(int x, int p, bool, int sel) { return med3_i32(x, p, sel); }
__device__ __forceinline__ double keep(double x, double p, bool up, int) {
  return (p < x) != up ? p : x;
}
__device__ __forceinline__ void order2(int& a, int& b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  a = lo;
  b = hi;
}
__device__ __forceinline__ void order2(double& a, double& b) {
  const double lo = fmin(a, b), hi = fmax(a, b);
  a = lo;
  b = hi;
}

// One exchange at lane distance D (after a merge's mirrored first exchange).
template <int D, int R, class T>
__device__ __forceinline__ void exchange_lanes(T (&x)[R], int lane) {
  const bool up = (lane & D) != 0;
  const int sel = up ? 0x7FFFFFFF : (int)0x80000000;
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = keep(x[r], lane_xor<D>(x[r]), up, sel);
}
// Exchanges at register distances R / 2 .. 1.
template <int R, int FROM, class T>
__device__ __forceinline__ void exchange_regs(T (&x)[R]) {
#pragma unroll
  for (int d = FROM; d >= 1; d >>= 1)
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & d) == 0) order2(x[r], x[r | d]);
}
// Merge the two sorted halves of every group of G lanes (G R values).
template <int G, int R, class T>
__device__ __forceinline__ void merge_lanes(T (&x)[R], int lane) {
  {
    const bool up = (lane & (G >> 1)) != 0;
    const int sel = up ? 0x7FFFFFFF : (int)0x80000000;
#pragma unroll
    for (int r = 0; r < R / 2; ++r) {
      const T p = lane_mirror<G>(x[R - 1 - r]), q = lane_mirror<G>(x[r]);
      x[r] = keep(x[r], p, up, sel);
      x[R - 1 - r] = keep(x[R - 1 - r], q, up, sel);
    }
  }
  if constexpr (G >= 64) exchange_lanes<16>(x, lane);
  if constexpr (G >= 32) exchange_lanes<8>(x, lane);
  if constexpr (G >= 16) exchange_lanes<4>(x, lane);
  if constexpr (G >= 8) exchange_lanes<2>(x, lane);
  if constexpr (G >= 4) exchange_lanes<1>(x, lane);
  exchange_regs<R, R / 2>(x);
}

// Inclusive sum over the lanes of the wavefront.
__device__ __forceinline__ int lane_scan(int v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(v, d);
    if (lane >= d) v += o;
  }
  return v;
}

// partial[3 block + 0..2] = S(A, B), S(A, A), S(B, B) of the block's C
// dimensions.  Grid: ceil(dim / C) workgroups of C wavefronts.
template <int R, int C>
__global__ void __launch_bounds__(64 * C) sorted_pair_sum_kernel(
    const float* __restrict__ A, int64_t lda, int n, const float* __restrict__ B, int64_t ldb,
    int m, int64_t dim, int vec, double* __restrict__ partial) {
  __shared__ float tile[64 * R * (C + 1)];           // [n + m][C + 1]
  __shared__ double sums[3][C];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // neighbouring dimensions on one XCD (workgroups go to the 8 XCDs in turn),
  // whose L2 then serves the 64-byte halves of a row's 128-byte lines
  const int64_t nblk = gridDim.x;
  const int64_t blk = (nblk % 8 == 0) ? (int64_t)(blockIdx.x % 8) * (nblk / 8) + blockIdx.x / 8
                                      : (int64_t)blockIdx.x;
  const int64_t k0 = blk * C;
  constexpr int Q = C / 4;                           // 16-byte pieces of a row
  const int q = (t % Q) * 4;
  for (int row = t / Q; row < n + m; row += 64 * C / Q) {
    const float* p = row < n ? A + (int64_t)row * lda + k0 + q : B + (int64_t)(row - n) * ldb + k0 + q;
    float* d = tile + row * (C + 1) + q;
    if (vec && k0 + q + 4 <= dim) {
      const float4 v = *reinterpret_cast<const float4*>(p);
      d[0] = v.x;
      d[1] = v.y;
      d[2] = v.z;
      d[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = k0 + q + e < dim ? p[e] : 0.0f;
    }
  }
  __syncthreads();

  const bool is_b = lane >= 32;
  const int rows = is_b ? m : n, base = is_b ? n : 0;
  int flags = 0;
  int x[R];
  bool finite = true;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * 32 + (lane & 31);
    const float v = i < rows ? tile[(base + i) * (C + 1) + wave] : 3.402823466e38f;
    finite = finite && fabsf(v) <= 3.402823466e38f;
    x[r] = sort_key(v);
  }
  if (__any(!finite)) {                  // noted, and out of the other set's own sum
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float v = sort_value(x[r]);
      if (!(fabsf(v) <= 3.402823466e38f)) {
        flags |= v != v ? kSortFlagNan : v > 0.0f ? kSortFlagPos : kSortFlagNeg;
        x[r] = 0;
      }
    }
  }
  // sort the R values of every lane, then lanes 0-31 (A) and 32-63 (B)
#pragma unroll
  for (int s = 2; s <= R; s <<= 1) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & (s >> 1)) == 0) order2(x[r], x[r ^ (s - 1)]);
#pragma unroll
    for (int d = s >> 2; d >= 1; d >>= 1)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if ((r & d) == 0) order2(x[r], x[r | d]);
  }
  merge_lanes<2>(x, lane);
  merge_lanes<4>(x, lane);
  merge_lanes<8>(x, lane);
  merge_lanes<16>(x, lane);
  merge_lanes<32>(x, lane);
  // merge A with B, each value marked in its lowest bit
  double z[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const double v = (double)sort_value(x[r]);
    z[r] = pack(__double2loint(v) | (is_b ? 1 : 0), __double2hiint(v));
  }
  merge_lanes<64>(z, lane);

  int nb = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) nb += __double2loint(z[r]) & 1;
  int b = lane_scan(nb, lane) - nb;                  // values of B before this lane's
  const double first = pack(__double2loint(z[0]) & ~1, __double2hiint(z[0]));
  const double after = pack(__shfl_down(__double2loint(first), 1), __shfl_down(__double2hiint(first), 1));
  double sxy = 0.0, sxx = 0.0, syy = 0.0;
  double v = first;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = lane * R + r;                      // position in the merged order
    b += __double2loint(z[r]) & 1;
    const int a = k + 1 - b;
    const double w = r + 1 < R ? pack(__double2loint(z[r + 1 < R ? r + 1 : r]) & ~1,
                                      __double2hiint(z[r + 1 < R ? r + 1 : r]))
                               : after;
    const double gap = k + 1 < n + m ? w - v : 0.0;  // the padding has no gaps
    const int an = __mul24(a, n - a), bm = __mul24(b, m - b);
    const int ab = __mul24(a, m - b) + __mul24(b, n - a);
    sxy = fma(gap, (double)ab, sxy);
    sxx = fma(gap, (double)(2 * an), sxx);
    syy = fma(gap, (double)(2 * bm), syy);
    v = w;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    sxy += __shfl_xor(sxy, d);
    sxx += __shfl_xor(sxx, d);
    syy += __shfl_xor(syy, d);
  }
  // what |x - y| gives where values are not finite: a set's own sum has the
  // pair of a value with itself (inf - inf), two sets' sum has infinities of
  // equal sign
  const unsigned long long lo = 0xFFFFFFFFull;
  const unsigned long long fn = __ballot(flags & kSortFlagNan), fp = __ballot(flags & kSortFlagPos),
                           fm = __ballot(flags & kSortFlagNeg);
  if (fn | fp | fm) {
    const double nan = __longlong_as_double(0x7FF8000000000000ll);
    if ((fn | fp | fm) & lo) sxx = nan;
    if ((fn | fp | fm) >> 32) syy = nan;
    const bool same = ((fp & lo) && (fp >> 32)) || ((fm & lo) && (fm >> 32));
    sxy = fn || same ? nan : __longlong_as_double(0x7FF0000000000000ll);
  }
  if (lane == 0) {
    sums[0][wave] = sxy;
    sums[1][wave] = sxx;
    sums[2][wave] = syy;
  }
  __syncthreads();
  if (t < 3) {
    double s = 0.0;
    for (int c = 0; c < C; ++c)
      if (k0 + c < dim) s += sums[t][c];
    partial[3 * blk + t] = s;
  }
}

// The blocks' sums in order: with mmd, out[0..3] = {MMD, S(A, B), S(A, A),
// S(B, B)}; without, out[0] = S(A, B).
__global__ void __launch_bounds__(256) sorted_final_kernel(const double* __restrict__ partial,
                                                           int64_t count, int64_t n, int64_t m,
                                                           int mmd, double* __restrict__ out) {
  __shared__ double red[3][256];
  const int t = threadIdx.x;
  double s[3] = {0.0, 0.0, 0.0};
  int64_t i = t;
  for (; i + 7 * 256 < count; i += 8 * 256) {   // eight blocks' loads in flight, added in order
    double v[8][3];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k) v[u][k] = partial[3 * (i + 256 * u) + k];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k) s[k] += v[u][k];
  }
  for (; i < count; i += 256)
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] += partial[3 * i + k];
#pragma unroll
  for (int k = 0; k < 3; ++k) red[k][t] = s[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w)
#pragma unroll
      for (int k = 0; k < 3; ++k) red[k][t] += red[k][t + w];
    __syncthreads();
  }
  if (t == 0) {
    if (mmd) {
      const double dn = (double)n, dm = (double)m;
      out[0] = 2.0 * red[0][0] / (dn * dm) - red[1][0] / (dn * dn) - red[2][0] / (dm * dm);
      out[1] = red[0][0];
      out[2] = red[1][0];
      out[3] = red[2][0];
    } else {
      out[0] = red[0][0];
    }
  }
}

// Registers per lane for sets of at most 32 R values; 0 beyond 2048.
int sort_regs(int64_t n, int64_t m) {
  const int64_t top = n > m ? n : m;
  int r = 4;
  while (r < 64 && 32 * r < top) r *= 2;
  return 32 * r >= top ? r : 0;
}
// Dimensions per workgroup: 16 (64 bytes of a row); 8 at R = 64, whose 4096
// rows fill the LDS, and at R = 32, where two workgroups of 70 KB share a CU
// and one stages while the other sorts (1000 x 1000: 85 -> 79 us).
int sort_cols(int r) { return r >= 32 ? 8 : 16; }

int64_t tiled(int64_t n) { return (n + kPT - 1) / kPT * kPT; }

// The ways of a sum.  kSorted and kPairs64 keep every difference and sum in
// float64; a pair's distance over runs of 256 dimensions is float32 in kPairs32.
enum class Way { kSorted, kPairs64, kPairs32 };

// Sorting takes at least the latency of one wavefront's sort of 32 R values a
// set, however few the dimensions (8 or 16 a workgroup leave most of the chip
// idle), and all pairs in float64 at least its launches; so the way is chosen by
// what both take, us as measured (sets of features; sorted and all pairs):
//   one sum:    2000 x 2000 of 8      49 and 14    1000 x 1000 of 64   27 and 14
//               300 x 300 of 128      22 and 20    1000 x 1000 of 256  27 and 35
//               64 x 64 of 65536      69 and 35    256 x 256 of 8192   22 and 49
//   an MMD:     1100 x 1100 of 16     48 and 32    1000 x 1000 of 8    26 and 29
//               1 x 2048 of 33        51 and 44    2000 x 2000 of 64   50 and 82
// The sort: a floor by its registers, then a rate per dimension.
double sort_us(int r, int64_t dim) {
  const double floor_us = r <= 8 ? 14.5 : r == 16 ? 22.0 : r == 32 ? 26.5 : 48.5;
  const double rate = r == 4 ? 0.98e-3 : r == 8 ? 1.8e-3 : r == 16 ? 4.6e-3 : r == 32 ? 7.7e-3 : 24e-3;
  return std::max(floor_us, 5.0 + rate * (double)dim);
}
// All pairs: what is left of the launches beside the kernel, and per 32 staged
// dimensions of a share (fewer at the end cost about half and the rest by their
// number) 3.1 us alone on a CU, 2.7 for every 256 workgroups.
double pairs64_us(int64_t n, int64_t m, int64_t dim) {
  const PairPlan p = pair_plan(n, m, dim);
  const int64_t blocks = p.tiles_n * p.tiles_m * p.shares;
  const int64_t d = std::min(dim, p.runs_per_share * kF32Run), rest = d % kPK;
  const double chunks = (double)(d / kPK) + (rest ? 0.45 + 0.55 * (double)rest / kPK : 0.0);
  return 6.0 + chunks * std::max(3.1, 2.7 * (double)((blocks + 255) / 256));
}

// The three sums of an MMD: one pass against three sums' launches.
Way mmd_way(int64_t n, int64_t m, int64_t dim) {
  const int r = n > 0 && m > 0 && dim > 0 ? sort_regs(n, m) : 0;
  if (r == 0) return Way::kPairs32;
  const double pairs = pairs64_us(n, m, dim) + pairs64_us(n, n, dim) + pairs64_us(m, m, dim);
  return sort_us(r, dim) <= std::max(28.5, pairs) ? Way::kSorted : Way::kPairs64;
}

// One sum alone is left to float32 runs where one set of more than 256 sounds is
// much the larger, and sorting it would outweigh the pairs (in whole tiles) at
// any number of dimensions: at 1000 x 64 of 8192 all pairs take 31 us and the
// sort 74, at 1000 x 256 116 and 75, at 2000 x 64 64 and 191, at 2000 x 256 226
// and 192.
Way one_way(int64_t n, int64_t m, int64_t dim) {
  const int r = n > 0 && m > 0 && dim > 0 ? sort_regs(n, m) : 0;
  if (r == 0 || (r > 8 && tiled(n) * tiled(m) < 6400 * (int64_t)r)) return Way::kPairs32;
  return sort_us(r, dim) <= std::max(14.3, pairs64_us(n, m, dim)) ? Way::kSorted : Way::kPairs64;
}

template <int R, int C>
hipError_t launch_sorted(const float* A, int64_t lda, int64_t n, const float* B, int64_t ldb,
                         int64_t m, int64_t dim, int vec, double* partial, int64_t blocks,
                         hipStream_t s) {
  hipLaunchKernelGGL((sorted_pair_sum_kernel<R, C>), dim3((unsigned)blocks), dim3(64 * C), 0, s, A,
                     lda, (int)n, B, ldb, (int)m, dim, vec, partial);
  return hipGetLastError();
}

hipError_t launch_sort_sums(const float* A, int64_t lda, int64_t n, const float* B, int64_t ldb,
                            int64_t m, int64_t dim, double* partial, int mmd, double* out,
                            hipStream_t s) {
  const int r = sort_regs(n, m);
  const int64_t blocks = (dim + sort_cols(r) - 1) / sort_cols(r);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const int vec = ((lda | ldb) % 4 == 0) && (reinterpret_cast<uintptr_t>(A) % 16 == 0) &&
                  (reinterpret_cast<uintptr_t>(B) % 16 == 0);
  hipError_t e;
  switch (r) {
    case 4: e = launch_sorted<4, 16>(A, lda, n, B, ldb, m, dim, vec, partial, blocks, s); break;
    case 8: e = launch_sorted<8, 16>(A, lda, n, B, ldb, m, dim, vec, partial, blocks, s); break;
    case 16: e = launch_sorted<16, 16>(A, lda, n, B, ldb, m, dim, vec, partial, blocks, s); break;
    case 32: e = launch_sorted<32, 8>(A, lda, n, B, ldb, m, dim, vec, partial, blocks, s); break;
    default: e = launch_sorted<64, 8>(A, lda, n, B, ldb, m, dim, vec, partial, blocks, s); break;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sorted_final_kernel, dim3(1), dim3(256), 0, s, partial, blocks, n, m, mmd, out);
  return hipGetLastError();
}

size_t sort_bytes(int64_t n, int64_t m, int64_t dim) {
  const int c = sort_cols(sort_regs(n, m));
  return (size_t)((dim + c - 1) / c) * 3 * sizeof(double);
}

size_t pairs_bytes(int64_t n, int64_t m, int64_t dim) {
  const PairPlan p = pair_plan(n, m, dim);
  return (size_t)(p.tiles_n * p.tiles_m * p.shares) * sizeof(double);
}

// Bytes that hold the partial sums of every call of at most these sizes, so that
// a workspace for the largest sets serves all: it grows with each size, where
// the need of a call does not (which way it goes depends on the sizes, and a
// few tiles take more shares each).  All pairs of t tiles take t max(1, about
// 1024 / t) partials: fewer than 2048 or one a tile, and at most one a run of
// 256 dimensions and tile.
size_t any_smaller_bytes(int64_t n, int64_t m, int64_t dim) {
  const int64_t tiles = ((n + kPT - 1) / kPT) * ((m + kPT - 1) / kPT);
  const int64_t runs = dim > 0 ? (dim + kF32Run - 1) / kF32Run : 1;
  const int64_t pairs = std::min(tiles * runs, std::max(tiles, 2 * kFillBlocks));
  return std::max((size_t)pairs * sizeof(double),
                  sort_bytes(std::min<int64_t>(n, 2048), std::min<int64_t>(m, 2048), dim));
}

template <class T>
hipError_t launch_all_pairs(const float* A, int64_t lda, int64_t n, const float* B, int64_t ldb,
                            int64_t m, int64_t dim, double* partial, double* out, hipStream_t s) {
  const PairPlan p = pair_plan(n, m, dim);
  const int64_t blocks = p.tiles_n * p.tiles_m * p.shares;
  if (blocks > 0 && dim > 0) {
    const int vec = ((lda | ldb) % 4 == 0) && (reinterpret_cast<uintptr_t>(A) % 16 == 0) &&
                    (reinterpret_cast<uintptr_t>(B) % 16 == 0);
    hipLaunchKernelGGL(l1_pair_sum_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, A, lda, n, B,
                       ldb, m, dim, p, vec, partial);
  }
  hipLaunchKernelGGL(ordered_sum_kernel, dim3(1), dim3(256), 0, s, partial,
                     dim > 0 ? blocks : (int64_t)0, out);
  return hipGetLastError();
}

}  // namespace

size_t l1_pair_sum_need(int64_t n, int64_t m, int64_t dim) {
  return one_way(n, m, dim) == Way::kSorted ? sort_bytes(n, m, dim) : pairs_bytes(n, m, dim);
}

size_t l1_pair_sum_workspace(int64_t n, int64_t m, int64_t dim) { return any_smaller_bytes(n, m, dim); }

hipError_t launch_l1_pair_sum(const float* A, int64_t lda, int64_t n, const float* B, int64_t ldb,
                              int64_t m, int64_t dim, double* partial, double* out, hipStream_t s) {
  switch (one_way(n, m, dim)) {
    case Way::kSorted: return launch_sort_sums(A, lda, n, B, ldb, m, dim, partial, 0, out, s);
    case Way::kPairs64: return launch_all_pairs<double>(A, lda, n, B, ldb, m, dim, partial, out, s);
    default: return launch_all_pairs<float>(A, lda, n, B, ldb, m, dim, partial, out, s);
  }
}

size_t mmd_l1_need(int64_t n, int64_t m, int64_t dim) {
  if (mmd_way(n, m, dim) == Way::kSorted) return sort_bytes(n, m, dim);
  return std::max({pairs_bytes(n, m, dim), pairs_bytes(n, n, dim), pairs_bytes(m, m, dim)});
}

size_t mmd_l1_workspace(int64_t n, int64_t m, int64_t dim) {
  const int64_t top = std::max(n, m);
  return any_smaller_bytes(top, top, dim);
}

hipError_t launch_mmd_l1(const float* X, int64_t n, const float* Y, int64_t m, int64_t dim,
                         double* ws, double* out, hipStream_t s) {
  const Way way = mmd_way(n, m, dim);
  if (way == Way::kSorted) return launch_sort_sums(X, dim, n, Y, dim, m, dim, ws, 1, out, s);
  // the three sums reuse the workspace in stream order
  const auto sum = way == Way::kPairs64 ? launch_all_pairs<double> : launch_all_pairs<float>;
  hipError_t e = sum(X, dim, n, Y, dim, m, dim, ws, out + 1, s);
  if (e == hipSuccess) e = sum(X, dim, n, X, dim, n, dim, ws, out + 2, s);
  if (e == hipSuccess) e = sum(Y, dim, m, Y, dim, m, dim, ws, out + 3, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mmd_combine_kernel, dim3(1), dim3(64), 0, s, out, n, m);
  return hipGetLastError();
}

}  // namespace synth
