// Adjoint of the Voice render: d(sum_n g(n) y(n)) / d(params), g = dL/dy given.
//
// Forward recap (per voice; q audio samples per control sample):
//   a_o(n) = (1 - t) y_o(j) + t y_o(j+1), j = n div q, t = (n mod q) / q
//   theta_v(n) = phi_v / 2pi + sum_{k<n} inc_v(k), inc_v = hz(m_v) / sr,
//   m_v = midi + tune_v + depth_v a_pitch_v
//   y = L1 sin(2 pi theta_1) a_1 + L2 x2(theta_2) a_3 + L3 noise a_4
//
// Kernel A (one wavefront per chunk of a voice, or per slice of chunks)
// recomputes the forward with the render's own control stage and phase
// recurrences and reduces, per control segment s,
//   D_v = sum dtheta_v,  C{0,1}_v = sum w{0,1} inc_v,  E{0,1}_v = sum w{0,1} inc_v P_v
// (w0 = 1 - t, w1 = t, P_v the inclusive in-segment prefix of dtheta_v), the
// VCA row sums A{0,1}_o = sum w{0,1} g L x, and the sums for the levels, the
// square-saw shape and its gain K.  With Gend_v(s) = sum of D_v over later
// segments, the upsampled pitch adjoint of segment s is
//   B{0,1}_v(s) = (Gend_v(s) + D_v(s)) C{0,1}_v(s) - E{0,1}_v(s),
// i.e. sum_k w inc Gtheta(k) with Gtheta(k) = sum_{n>k} dtheta(n): the reverse
// (suffix) scan of the phase adjoint is split into an in-segment part (here)
// and a cross-segment float64 scan (kernel B).
//
// Kernel B (one wavefront per chunk): segment adjoints -> dy_o(j) (transposed
// upsampling), modulation mixer, LFOs (shape weights, phase with its own suffix
// scan, rate clamp), control-rate VCAs and the six ADSRs, d(human value) summed
// over the chunk.  Kernel C joins a voice's chunks and applies the curve
// mapping's Jacobian: d/d(normalised parameter).  Deterministic; no atomics.
#include <math.h>

#include <type_traits>

#include "philox.h"
#include "sine_table.h"
#include "synth_internal.h"
#include "voice_device.h"

namespace synth {
namespace {

using namespace voice;

enum {
  kRD1 = 0, kRC01, kRC11, kRE01, kRE11,           // sine VCO phase adjoint
  kRD2, kRC02, kRC12, kRE02, kRE12,               // square-saw VCO phase adjoint
  kRA01, kRA11, kRA03, kRA13, kRA04, kRA14,       // VCA rows 1, 3, 4
  kRL1, kRL2, kRL3, kRShape, kRK,                 // levels, shape, square-saw gain
  kNumRed
};

constexpr double kIndexScale = 1024.0;           // no control period has more samples

// sin and cos of 2 pi j / 256 from the quarter wave.
__device__ __forceinline__ double2 sincos_entry(int j) {
  const int r = j & 63, o = j >> 6;              // octet pair: quarter o, offset r
  const double a = kSinT[r], b = kSinT[64 - r];  // sin, cos of the offset
  switch (o) {
    case 0: return make_double2(a, b);
    case 1: return make_double2(b, -a);
    case 2: return make_double2(-a, -b);
    default: return make_double2(-b, a);
  }
}

// sin and cos of 2 pi th in float64: th = n / 256 + d, |d| <= 1/512 (exact),
// the table's sine and cosine at n mod 256 and, for a = 2 pi d (|a| <= 0.0123),
// sin a to a^5 and cos a - 1 to a^6 (truncation 9e-18 and 2e-20), joined by
// the addition theorems: 18 instructions after the reduction against 34 for
// the two series on a quarter cycle, with the same rounding (2e-16).
__device__ __forceinline__ void sincos_table(const double2* tab, double th, double& s, double& c) {
  const double n = rint(256.0 * th);
  const double a = fma(n, -1.0 / 256.0, th) * kTwoPi, a2 = a * a;
  const double2 t = tab[(int)n & 255];
  double p = fma(a2, kSeriesC[kSin5], kSeriesC[kSin3]);
  const double sa = fma(p * a2, a, a);
  p = fma(a2, kSeriesC[kCos6], kSeriesC[kCos4]);
  const double ca = a2 * fma(a2, p, -0.5);       // cos a - 1
  s = fma(t.y, sa, fma(t.x, ca, t.x));
  c = fma(-t.x, sa, fma(t.y, ca, t.y));
}

// 2^y for y <= 0 by exp2_f64's method on 64 table points: |r| <= 1/128, so the
// series runs to z^5 / 120 (truncation 4e-17).
__device__ __forceinline__ double exp2_table(const double* tab, double y) {
  y = fmax(y, -1100.0);
  const double nd = rint(y * 64.0);
  const int n = (int)nd;
  const double z = fma(nd, -1.0 / 64.0, y) * kLn2;
  double p = fma(z, kSeriesC[kExpC5], kSeriesC[kExpC4]);
  p = fma(p, z, kSeriesC[kExpC3]);
  p = fma(p, z, 0.5);
  p = fma(p, z, 1.0);
  p = fma(p, z, 1.0);
  return ldexp(tab[n & 63] * p, n >> 6);
}

// What the control-rate pass reads and adds up per chunk of a voice, after the
// segment sums red [batch][21][J].
struct CtlArgs {
  double* carries;   // [batch][chunks][4]: the phases at the chunk's start (LFO 1, 2 used)
  double* gpart;     // [batch][chunks][kPartOut]: adjoint sums of the chunk, the first kPartOut
  int64_t nchunks;
};

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

// First chunk from which a voice is silent: every envelope is 0 with zero
// derivative from control sample floor(note-off + longest release) + 2 on, so
// no parameter sees the samples there.
__device__ __forceinline__ int64_t silent_chunk(const double* v, double rc) {
  double jsil = 0.0;
  for (int k = 0; k < 6; ++k) jsil = fmax(jsil, v[1] * rc + v[2 + 5 * k + 3] * rc);
  jsil = fmin(jsil, 9.0e15);
  const int64_t js = (int64_t)floor(jsil) + 2;
  return (js + kSegsPerChunk - 1) / kSegsPerChunk;
}

// Bound by float64 VALU issue for part of its time and by the latency of a
// sample's chain (recurrence, table reads, series) for the rest: over 256 voices
// of 4 s counters show the VALU busy for 60% of the launch, 1.5 wavefronts per
// SIMD on average of the two that the registers allow, a third of their time in
// waits.  125 instructions a sample of the loop, 92 of them float64 (205 with
// the series' sine and cosine, the weights, ramps and products that follow from
// sums with and without the sample index formed per sample, and the
// exponential's table in global memory), 147 with the control stage; the pass
// 383 -> 298 us.  LDS of 20.4 KB (noise as its 16-bit halves, 64 points of the
// exponential) lets a CU hold the eight wavefronts the registers allow; fetching
// the next sample's table entries a sample ahead changed nothing (301 us).
template <int RPS>
__global__ void __launch_bounds__(kWave, 2) adjoint_audio_kernel(const RenderArgs a,
                                                              const float* __restrict__ g_audio,
                                                              double* __restrict__ red,
                                                              CtlArgs ctl) {
  __shared__ VoiceShared sh;
  extern __shared__ __align__(16) float tile[];
  const int lane = threadIdx.x;
  const int per = a.slices * a.pass_split;       // workgroups per voice
  const int64_t b = blockIdx.x / per;
  const int part = (int)(blockIdx.x % per);
  const int slice = part / a.pass_split, sub = part % a.pass_split;
  const int q = a.q;
  const int h = q / RPS;
  const double qd = (double)q;
  const int64_t N = a.n_uniform;
  const int64_t J = (N + q - 1) / q;
  const uint64_t g = a.voice_ids ? a.voice_ids[b] : a.first_g + (uint64_t)b;
  const float* gv = g_audio + b * N;
  double* rv = red + b * J * kNumRed;
  float* tg = tile;                 // g(n) of the pass
  uint16_t* tn = reinterpret_cast<uint16_t*>(tile + kWave * h);   // 16-bit noise of the pass
  __shared__ double2 sct[256];
  __shared__ double e2t[64];
  for (int j = lane; j < 256; j += kWave) sct[j] = sincos_entry(j);
  for (int j = lane; j < 64; j += kWave) e2t[j] = kExp2T[4 * j];

  voice_setup(a, b, sh, lane);
  const double* v = sh.v;
  const double sr = a.sr;
  const int64_t nchunks = ctl.nchunks;
  const int64_t c_sil = silent_chunk(v, a.rc);
  // this workgroup's chunks (a voice may be split over several workgroups;
  // the carries at its first chunk are precomputed, or the earlier chunks
  // are walked through the control stage only)
  const int64_t c_lo = nchunks * slice / a.slices;
  const int64_t c_hi = nchunks * (slice + 1) / a.slices;

  const double midi = v[0];
  const double m_hi = fmax(0.0, midi + v[71] + fmax(0.0, v[72]));
  const double f_hi = fmin(440.0 * exp2((m_hi - 69.0) / 12.0), sr / 2.0);
  const double Kd = 12000.0 / (f_hi * log10(f_hi));
  const float cg = (float)(1.0 - v[74] / 2.0);
  const double shape_d = v[74], L2cg2pi = v[76] * (1.0 - v[74] / 2.0) * kTwoPi;
  const double L1d = v[75], L2d = v[76], L3d = v[77], L1d_2pi = v[75] * kTwoPi;
  const double K2d = 2.0 * 1.4426950408889634 * Kd, K4d = 4.0 * Kd;   // exp(-2|z|) = 2^-(2 log2(e) |z|)
  const uint32_t glo = (uint32_t)g, ghi = (uint32_t)(g >> 32);

  int64_t c_start = 0;
  if (a.carries && c_lo > 0 && c_lo < a.carry_stride) {
    // chunk-start carries computed beforehand (as for a split render)
    if (lane < 4) sh.carry[lane] = a.carries[(b * a.carry_stride + c_lo) * 4 + lane];
    __syncthreads();
    c_start = c_lo;
  }
  for (int64_t c = c_start; c < c_hi; ++c) {
    if (c >= c_sil) break;                       // no segment sums are read from there on
    double y[5], yn[5];
    if (!a.carries && c >= c_lo && sub == 0 && lane < 2)
      ctl.carries[(b * nchunks + c) * 4 + lane] = sh.carry[lane];
    __syncthreads();
    control_stage<RPS, false>(a, sh, reinterpret_cast<double*>(tile), c, J, h, lane, y, yn);
    if (c < c_lo) continue;                      // slice starts later: only carries needed
    // unscaled VCA ramps of this lane's segment
    const double a10_d = y[1], a1d_d = (yn[1] - y[1]) / qd;
    const double a30_d = y[3], a3d_d = (yn[3] - y[3]) / qd;
    const double a40_d = y[4], a4d_d = (yn[4] - y[4]) / qd;
    __syncthreads();

    constexpr int segs_pp = kWave / RPS;
    const int nseg = (int)((J - c * kSegsPerChunk) < kSegsPerChunk ? (J - c * kSegsPerChunk)
                                                                    : kSegsPerChunk);
    const int npass = (nseg + segs_pp - 1) / segs_pp;
    for (int p = sub; p < npass; p += a.pass_split) {
      // ---- load pass: g and the noise halves into LDS, 4 samples per lane ----
      const int64_t pbase = (c * kSegsPerChunk + (int64_t)p * segs_pp) * q;
      int64_t cnt64 = (int64_t)((nseg - p * segs_pp) < segs_pp ? (nseg - p * segs_pp) : segs_pp) * q;
      if (cnt64 > N - pbase) cnt64 = N - pbase;
      const int cnt = (int)cnt64;
      const int tcap = kWave * h;
      const uint32_t grp0 = (uint32_t)(pbase >> 3);
      for (int base = 0; base < tcap; base += 512) {
        uint32_t w[4] = {glo, ghi, grp0 + (uint32_t)(base >> 3) + (uint32_t)lane, 1u};
        philox4x32_10(w, a.nk0, a.nk1);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
          const int src_l = sub * 32 + (lane >> 1);
          const uint32_t w0 = __shfl(w[0], src_l), w1 = __shfl(w[1], src_l);
          const uint32_t w2 = __shfl(w[2], src_l), w3 = __shfl(w[3], src_l);
          const uint32_t wa = (lane & 1) ? w2 : w0;
          const uint32_t wb = (lane & 1) ? w3 : w1;
          const int li = base + sub * 256 + 4 * lane;
          if (li < tcap) {
            float gg[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) gg[e] = li + e < cnt ? gv[pbase + li + e] : 0.0f;
            *reinterpret_cast<float4*>(tg + li) = make_float4(gg[0], gg[1], gg[2], gg[3]);
            *reinterpret_cast<uint2*>(tn + li) = make_uint2(wa, wb);
          }
        }
      }
      __syncthreads();
      // ---- run pass: forward recompute and per-run reductions ----
      const int ls = p * segs_pp + lane / RPS;
      const int m = lane % RPS;
      const int src = ls < kWave ? ls : kWave - 1;
      double t1 = sh.seg[0][kSegTheta][src], i1 = sh.seg[0][kSegInc][src];
      double t2 = sh.seg[1][kSegTheta][src], i2 = sh.seg[1][kSegInc][src];
      const double r1 = sh.seg[0][kSegRatio][src], r2 = sh.seg[1][kSegRatio][src];
      {
        double s1 = sh.seg[0][kSegRunSum][src], R1 = sh.seg[0][kSegRunRatio][src];
        double s2 = sh.seg[1][kSegRunSum][src], R2 = sh.seg[1][kSegRunRatio][src];
        for (int t = 0; t < m; ++t) {
          t1 += s1; s1 *= R1; i1 *= R1;
          t2 += s2; s2 *= R2; i2 *= R2;
        }
      }
      // VCA ramps at sample ks of the segment: x0 + ks xd.  In float64 with the
      // phase adjoints' constant factors for the reason given below, in float32
      // for the shape and gain sums.
      const double A10d = __shfl(a10_d, src), A1dd = __shfl(a1d_d, src);
      const double A30d = __shfl(a30_d, src), A3dd = __shfl(a3d_d, src);
      const double A40d = __shfl(a40_d, src), A4dd = __shfl(a4d_d, src);
      const double p10 = A10d * L1d_2pi, p1d = A1dd * L1d_2pi;
      const double p30 = A30d * L2cg2pi, p3d = A3dd * L2cg2pi;
      const float A30 = (float)A30d, A3d = (float)(A3dd * kIndexScale);
      double P1 = 0.0, P2 = 0.0;
      // sums over the run of l = inc and ks l, of both times P (float64), and
      // of d and ks d of the three amplitude terms, the shape and gain terms
      // (float32 over at most q / RPS samples; there ks counts 2^-10, exactly, as
      // a period has at most 1024 samples, so that ks d overflows no earlier than d)
      double c1 = 0.0, k1 = 0.0, e1 = 0.0, f1 = 0.0, c2 = 0.0, k2 = 0.0, e2 = 0.0, f2 = 0.0;
      float s1 = 0.0f, w1 = 0.0f, s3 = 0.0f, w3 = 0.0f, s4 = 0.0f, w4 = 0.0f, fsh = 0.0f, fk = 0.0f;
      const int seg_valid = ls < nseg ? 1 : 0;
      // samples of this run that exist in the voice (the last segment may be partial)
      const int64_t run0 = (c * kSegsPerChunk + ls) * (int64_t)q + m * h;
      const int nlive = seg_valid ? (int)(N - run0 < h ? (N - run0 > 0 ? N - run0 : 0) : h) : 0;
      const float* tgl = tg + lane * h;
      const uint16_t* tnl = tn + lane * h;
      auto run = [&](auto whole) {
        double kd = (double)(m * h);                 // sample index within the segment
        float kf = (float)(m * h) * (float)(1.0 / kIndexScale);
#pragma unroll 1
        for (int k = 0; k < h; ++k) {
          const float gk = tgl[k];                   // 0 past the voice's end
          const float nn = fmaf((float)tnl[k], 0x1p-15f, -32767.5f * 0x1p-15f);   // exact
          const double gd = (double)gk;
          double sn1, cs1, sn2, cs2;
          sincos_table(sct, t1, sn1, cs1);
          sincos_table(sct, t2, sn2, cs2);
          // Phase adjoints.  Square-saw: T = tanh(K s), sech^2 = 4e/(1+e)^2 with
          // e = exp(-2|K s|).  Its phase adjoint is a sum over the voice of
          // terms of both signs that the tanh edge scales by up to 2 pi K; for
          // pitch parameters the sum can be 1e6 times smaller than the sum of
          // its magnitudes, so float32 rounding of the terms (the hardware sine
          // and exponential, the VCA ramp) would dominate it.  The term is
          // evaluated in float64, and the sine VCO's alike.
          const double e = exp2_table(e2t, -fabs(K2d * sn2));
          const double de = 1.0 + e;
          double ri = __builtin_amdgcn_rcp(de);
          ri = fma(fma(-de, ri, 1.0), ri, ri);
          ri = fma(fma(-de, ri, 1.0), ri, ri);
          const double T = copysign((1.0 - e) * ri, sn2);
          const double er = e * ri * ri;             // sech^2 / 4
          const double Q = fma(shape_d, cs2, 1.0);
          P1 += gd * fma(kd, p1d, p10) * cs1;
          P2 += gd * fma(kd, p3d, p30) * fma(er * cs2 * Q, K4d, -(shape_d * sn2) * T);
          const double l1 = whole.value || k < nlive ? i1 : 0.0;
          const double l2 = whole.value || k < nlive ? i2 : 0.0;
          const double m1 = kd * l1, m2 = kd * l2;
          c1 += l1;
          k1 += m1;
          e1 = fma(l1, P1, e1);
          f1 = fma(m1, P1, f1);
          c2 += l2;
          k2 += m2;
          e2 = fma(l2, P2, e2);
          f2 = fma(m2, P2, f2);
          // amplitude side
          const float x2 = (float)(T * Q), tc = (float)(T * cs2), ek = (float)(er * sn2 * Q);
          const float d1 = gk * (float)sn1, d3 = gk * x2, d4 = gk * nn;
          const float ga3 = gk * fmaf(kf, A3d, A30);
          s1 += d1;
          w1 = fmaf(kf, d1, w1);
          s3 += d3;
          w3 = fmaf(kf, d3, w3);
          s4 += d4;
          w4 = fmaf(kf, d4, w4);
          fsh = fmaf(ga3, fmaf(cg, tc, -0.5f * x2), fsh);
          fk = fmaf(ga3, ek, fk);
          t1 += i1; i1 *= r1;
          t2 += i2; i2 *= r2;
          kd += 1.0;
          kf += (float)(1.0 / kIndexScale);
        }
      };
      if (__all(nlive == h || !seg_valid)) run(std::true_type{});   // invalid lanes are not used
      else run(std::false_type{});
      // the sums with the upsampling weights 1 - ks / q and ks / q
      const double inv_q = 1.0 / qd;
      double acc[kNumRed];
      acc[kRD1] = P1;
      acc[kRC11] = k1 * inv_q;
      acc[kRC01] = c1 - acc[kRC11];
      acc[kRE11] = f1 * inv_q;
      acc[kRE01] = e1 - acc[kRE11];
      acc[kRD2] = P2;
      acc[kRC12] = k2 * inv_q;
      acc[kRC02] = c2 - acc[kRC12];
      acc[kRE12] = f2 * inv_q;
      acc[kRE02] = e2 - acc[kRE12];
      const double L2cg = L2d * (double)cg;
      const double inv_qi = inv_q * kIndexScale;
      acc[kRA11] = L1d * w1 * inv_qi;
      acc[kRA01] = L1d * s1 - acc[kRA11];
      acc[kRA13] = L2cg * w3 * inv_qi;
      acc[kRA03] = L2cg * s3 - acc[kRA13];
      acc[kRA14] = L3d * w4 * inv_qi;
      acc[kRA04] = L3d * s4 - acc[kRA14];
      acc[kRL1] = A10d * s1 + A1dd * kIndexScale * w1;
      acc[kRL2] = (double)cg * (A30d * s3 + A3dd * kIndexScale * w3);
      acc[kRL3] = A40d * s4 + A4dd * kIndexScale * w4;
      acc[kRShape] = L2d * fsh;
      acc[kRK] = 4.0 * L2cg * fk;
      // combine the RPS runs of each segment: E += P_before * C, then sums
      if constexpr (RPS == 4) {
        // lanes 4i .. 4i + 3: prefix and sums by quad permutations
        auto before = [&](double P) {
          double t = dpp_f64<0x90>(P);               // lanes 0, 0, 1, 2
          double i2 = P + (m >= 1 ? t : 0.0);
          t = dpp_f64<0x44>(i2);                     // lanes 0, 1, 0, 1
          i2 += m >= 2 ? t : 0.0;
          t = dpp_f64<0x90>(i2);
          return m >= 1 ? t : 0.0;
        };
        const double pb1 = before(P1), pb2 = before(P2);
        acc[kRE01] += pb1 * acc[kRC01];
        acc[kRE11] += pb1 * acc[kRC11];
        acc[kRE02] += pb2 * acc[kRC02];
        acc[kRE12] += pb2 * acc[kRC12];
#pragma unroll
        for (int r = 0; r < kNumRed; ++r) {
          double t = acc[r] + dpp_f64<0xB1>(acc[r]); // lanes 1, 0, 3, 2
          acc[r] = t + dpp_f64<0x4E>(t);             // lanes 2, 3, 0, 1
        }
      } else {
        static_assert(RPS == 1, "one or four runs per segment");
      }
      const int64_t sglob = c * kSegsPerChunk + ls;
      if (m == 0 && ls < nseg) {
#pragma unroll
        for (int r = 0; r < kNumRed; ++r) rv[r * J + sglob] = acc[r];
      }
      __syncthreads();
    }
  }
}

// A chunk's adjoint sums: the 78 parameters', then for each LFO eight factors
// and its phase-adjoint sum.  The phase adjoint of an LFO at control sample k
// is summed over all later samples of the voice; what lies in later chunks
// enters the chunk's adjoints as one number per LFO, so its factor in the rate
// ADSR's A, D, S, R, alpha, note-off, the rate and the depth is summed as well
// and applied when the chunks are joined.
enum { kSumTail = kNumParams, kSumDph = kSumTail + 16, kNumSums = kSumDph + 2, kPartOut = 84 };

// The sums from kPartOut on go into the chunk's own part of the segment sums:
// its first segment's column of the rows that only the chunk itself reads, by
// then in registers (a workspace of the size that callers hold has no more room).
__device__ __forceinline__ int64_t tail_index(int n, int64_t c, int64_t J) {
  const int e = n - kPartOut;
  const int r = e < 2   ? kRC01 + 2 * e
                : e < 4 ? kRC02 + 2 * (e - 2)
                : e < 7 ? kRA01 + 2 * (e - 4)
                        : kRL1 + e - 7;
  return r * J + c * kSegsPerChunk;
}
static_assert(kNumSums - kPartOut == 12 && kRE01 == kRC01 + 2 && kRE02 == kRC02 + 2 &&
                  kRA04 == kRA01 + 4 && kRK == kRL1 + 4, "rows read by one chunk only");

// Rows of a wavefront's partial sums, in the order in which they come: eight per
// ADSR k (A, D, S, R, alpha, the factors of alpha and note-off), four factors
// (A, D, S, R) per LFO, twelve per LFO (its eight parameters, the factors of
// rate and depth, the phase-adjoint sum), the mixer, the parameters 68 .. 77,
// midi and note-off.
enum {
  kRowEnv = 0, kRowTail = 48, kRowLfo = 56, kRowMix = 80, kRowOsc = 100, kRowMidi = 110,
  kRowOff = 112, kNumRows = 116
};

__device__ __forceinline__ int sum_row(int n) {
  if (n == 0) return kRowMidi;
  if (n == 1) return kRowOff;
  if (n < 32) return kRowEnv + 8 * ((n - 2) / 5) + (n - 2) % 5;
  if (n < 48) return kRowLfo + 12 * ((n - 32) / 8) + (n - 32) % 8;
  if (n < 68) return kRowMix + n - 48;
  if (n < kSumTail) return kRowOsc + n - 68;
  if (n >= kSumDph) return kRowLfo + 12 * (n - kSumDph) + 10;
  const int i = (n - kSumTail) / 8, r = (n - kSumTail) % 8;
  return r < 4 ? kRowTail + 4 * i + r : r < 6 ? kRowEnv + 8 * (2 + 2 * i) + 1 + r : kRowLfo + 12 * i + 2 + r;
}

// Four values per lane -> part[row + (lane & 3)][lane / 16]: the sum of value
// lane & 3 over the lane's row of sixteen.  Each of the first two steps halves
// the values a lane holds (27 instructions for four sums; four steps for each
// value by itself take 48).
constexpr int kPartRow = 5;
__device__ __forceinline__ void emit4(double (*part)[kPartRow], int row, int lane, double x0,
                                      double x1, double x2, double x3) {
  const bool o1 = lane & 1, o2 = lane & 2;
  const double a = (o1 ? x1 : x0) + dpp_f64<0xB1>(o1 ? x0 : x1);   // quad_perm 1, 0, 3, 2
  const double b = (o1 ? x3 : x2) + dpp_f64<0xB1>(o1 ? x2 : x3);
  double s = (o2 ? b : a) + dpp_f64<0x4E>(o2 ? a : b);             // quad_perm 2, 3, 0, 1
  s += dpp_f64<0x128>(s);                                          // row_ror 8
  s += dpp_f64<0x124>(s);                                          // row_ror 4
  if ((lane & 15) < 4) part[row + (lane & 3)][lane >> 4] = s;
}

// Reverse exclusive scan over lanes: sum of x over lanes l' > l.
__device__ __forceinline__ double wave_rev_excl_scan(double x, int lane) {
  double incl = x;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const double t = __shfl_down(incl, d);
    if (lane + d < kWave) incl += t;
  }
  const double ex = __shfl_down(incl, 1);
  return lane == kWave - 1 ? 0.0 : ex;
}

// x^alpha for x in [0, 1] as pow01 with its derivatives d/dx and d/dalpha (0
// for x <= 0, as the oracle's masked power).
__device__ __forceinline__ void pow01_grad(double x, double al, double& P, double& dx, double& dal) {
  P = 0.0;
  dx = 0.0;
  dal = 0.0;
  if (x >= 1.0) {
    P = 1.0;
    dx = al;
  } else if (x > 0.0) {
    const double l2 = log2_f64(x);
    P = exp2_f64(al * l2);
    dx = al * P / x;
    dal = P * (l2 * kLn2);
  }
}

// ramp = clamp((j - s) / L, 0, 1): gradient passes inside [0, 1] (inclusive)
// for L > 0; d/ds = -1/L, d/dL = -(j - s) / L^2.
__device__ __forceinline__ bool ramp_live(double jd, double s, double L, double invL) {
  if (!(L > 0.0)) return false;
  const double r = (jd - s) * invL;
  return r >= 0.0 && r <= 1.0;
}

// The control-rate adjoint, chunk-parallel: one wavefront per (voice, chunk),
// control samples j = 62c .. 62c + 61 on lanes 1 .. 62 (lane l <-> j = 62c - 1
// + l); lane 0 carries segment 62c - 1, whose right-end adjoint lands on lane
// 1.  From the other chunks it needs the phase adjoints D of all later segments
// (summed here from their rows) and both LFO phases at control sample 62c.
//
// Bound by float64 issue: about 3100 instructions a chunk at three wavefronts
// per SIMD.  Two earlier passes over the chunks (LFO phase totals, then the
// LFOs' phase adjoints) are gone, the latter by the factors above, and the
// per-lane accumulators in LDS (47.6 KB, three wavefronts per CU) by sums across
// lanes as the values come: 256 voices of 4 s 285 us for three passes -> 75.
// The ADSRs are evaluated twice, once for their values and once with their
// logarithms for the derivatives, in loops over the six: kept in registers they
// cost the occupancy.
struct GradShared {
  VoiceShared vs;
  double part[kNumRows][kPartRow];
};

__global__ void __launch_bounds__(kWave, 3) adjoint_chunk_grad_kernel(const RenderArgs a,
                                                                      double* red, CtlArgs t) {
  __shared__ GradShared S;
  const int lane = threadIdx.x;
  const int64_t b = blockIdx.x / t.nchunks, c = blockIdx.x % t.nchunks;
  const int64_t J = (a.n_uniform + a.q - 1) / a.q;
  double* rv = red + b * J * kNumRed;
  double* out = t.gpart + (b * t.nchunks + c) * kPartOut;
  voice_setup(a, b, S.vs, lane);
  const double* v = S.vs.v;
  const double* dv = S.vs.d;
  const double rc = a.rc;
  const int64_t c_sil = silent_chunk(v, rc);
  if (c >= c_sil) {
    for (int n = lane; n < kNumSums; n += kWave)
      (n < kPartOut ? out[n] : rv[tail_index(n, c, J)]) = 0.0;
    return;
  }
  // envelope values, then their adjoints, of the six ADSRs (the segment rows
  // are not used here)
  double (*env)[kWave] = reinterpret_cast<double (*)[kWave]>(&S.vs.seg);
  static_assert(2 * kSegFields >= 6, "envelope rows");
  const double* lc = t.carries + (b * t.nchunks + c) * 4;
  double Gend1 = 0.0, Gend2 = 0.0;
  const int64_t Jl = c_sil < t.nchunks ? c_sil * kSegsPerChunk : J;   // later segments are 0
#pragma unroll 4
  for (int64_t k = (c + 1) * kSegsPerChunk + lane; k < Jl; k += kWave) {
    Gend1 += rv[kRD1 * J + k];
    Gend2 += rv[kRD2 * J + k];
  }
  Gend1 = wave_sum(Gend1);
  Gend2 = wave_sum(Gend2);

  const double kPitch = kLn2 / 12.0;
  const double note_off = v[1] * rc;
  const bool owned_lane = lane >= 1 && lane <= kSegsPerChunk;
  const int64_t j = c * kSegsPerChunk - 1 + lane;
  const double jd = (double)j;
  const bool inr = j >= 0 && j < J && lane <= kSegsPerChunk;
  const bool own = owned_lane && inr;
  const bool lastj = (j == J - 1);

  // forward recompute at control sample j
#pragma unroll 1
  for (int k = 0; k < 6; ++k) env[k][lane] = adsr_value(dv, k, jd, note_off);
  double x[4] = {env[0][lane], env[1][lane], 0.0, 0.0};
  double ph[2], lfo[2], fpre[2], sn[2], cs[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    // LFO phase: carry at the chunk's first owned sample + exclusive scan
    const int pb = 32 + 8 * i;
    fpre[i] = v[pb] + v[pb + 1] * env[2 + 2 * i][lane];
    const double inc = owned_lane ? fmax(0.0, fpre[i]) / rc : 0.0;
    const double th = lc[i] + wave_excl_scan(inc, lane);
    const double p = th - floor(th);
    ph[i] = p;
    sincos_cycles_f64(p, sn[i], cs[i]);
    const double num = v[pb + 3] * ((1.0 + sn[i]) / 2.0) + v[pb + 4] * (1.0 - fabs(2.0 * p - 1.0)) +
                       v[pb + 5] * p + v[pb + 6] * (1.0 - p) + v[pb + 7] * (p < 0.5 ? 1.0 : 0.0);
    lfo[i] = num * dv[kLfoInvW + i];
    x[2 + i] = lfo[i] * env[3 + 2 * i][lane];
  }
  double y[5];
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    const int pb = 48 + 4 * o;
    y[o] = (v[pb] * x[0] + v[pb + 1] * x[1] + v[pb + 2] * x[2] + v[pb + 3] * x[3]) *
           dv[kMixInvNorm + o];
  }

  // dy_o(j): transposed upsampling of the segment adjoints; the right-end
  // contributions come from the previous segment (lane - 1).  The shuffles run
  // on every lane: a cross-lane read from a lane that is masked off by a branch
  // returns no data.
  auto R = [&](int r) { return inr ? rv[r * J + j] : 0.0; };
  double dy[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  {
    double m[2], dep[2], phi[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const int o = 2 * w, rb = w ? kRD2 : kRD1;
      const double Dl = R(rb), C0 = R(rb + 1), C1 = R(rb + 2), E0 = R(rb + 3), E1 = R(rb + 4);
      const double D = own ? Dl : 0.0;
      // segment phase adjoints: later segments of this chunk + those of later
      // chunks; lane 0 (segment 62c - 1) needs all of this chunk's
      const double Ge = (w ? Gend2 : Gend1) + wave_rev_excl_scan(D, lane);
      const double B0 = (Ge + Dl) * C0 - E0;
      const double B1 = (Ge + Dl) * C1 - E1;
      const double pB1 = __shfl_up(B1, 1);
      const double tn = __shfl_down(y[o], 1);
      const double yn = lastj ? y[o] : tn;
      const double bt = B0 + pB1 + (lastj ? B1 : 0.0);
      dy[o] = own ? v[69 + 3 * w] * kPitch * bt : 0.0;
      // pitch and phase contributions of segment j
      m[w] = own ? kPitch * (B0 + B1) : 0.0;
      dep[w] = own ? kPitch * (y[o] * B0 + yn * B1) : 0.0;
      phi[w] = D / kTwoPi;
    }
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      const int o = w == 0 ? 1 : w + 2, rb = kRA01 + 2 * w;
      const double A0 = R(rb), A1 = R(rb + 1);
      const double pA1 = __shfl_up(A1, 1);
      dy[o] = own ? A0 + pA1 + (lastj ? A1 : 0.0) : 0.0;
    }
    double gmidi = m[0] + m[1], gtune = m[1], gdep = dep[1];
    // the square-saw gain K = 12000 / (f_hi log10 f_hi), f_hi from the highest pitch
    const double rK = R(kRK);
    const double dK = own ? rK : 0.0;
    if (dK != 0.0) {
      const double mh = v[0] + v[71] + fmax(0.0, v[72]);
      const double m_hi = fmax(0.0, mh);
      const double fh = 440.0 * exp2((m_hi - 69.0) / 12.0);
      if (fh <= a.sr / 2.0) {
        const double Kd = 12000.0 / (fh * log10(fh));
        const double dKdf = -(Kd / fh) * (1.0 + 1.0 / log(fh));
        const double dm = dK * dKdf * fh * kPitch;
        if (mh >= 0.0) {
          gmidi += dm;
          gtune += dm;
          if (v[72] >= 0.0) gdep += dm;
        }
      }
    }
    const double rL1 = R(kRL1), rL2 = R(kRL2), rL3 = R(kRL3), rS = R(kRShape);
    emit4(S.part, kRowOsc, lane, m[0], dep[0], phi[0], gtune);
    emit4(S.part, kRowOsc + 4, lane, gdep, phi[1], own ? rS : 0.0, own ? rL1 : 0.0);
    emit4(S.part, kRowOsc + 8, lane, own ? rL2 : 0.0, own ? rL3 : 0.0, gmidi, 0.0);
  }

  // modulation mixer: y_o = sum_i G_oi x_i / n_o, n_o = max(1, sum_i G_oi)
  double dx[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    const int pb = 48 + 4 * o;
    const double inv = dv[kMixInvNorm + o];
    const bool big = (v[pb] + v[pb + 1] + v[pb + 2] + v[pb + 3]) >= 1.0;
    const double yo = big ? y[o] : 0.0, di = dy[o] * inv;
#pragma unroll
    for (int i = 0; i < 4; ++i) dx[i] += v[pb + i] * di;
    // dy is 0 on the lanes that own no control sample
    emit4(S.part, kRowMix + 4 * o, lane, di * (x[0] - yo), di * (x[1] - yo), di * (x[2] - yo),
          di * (x[3] - yo));
  }
  // LFOs
  double tail[2];                        // d inc / d rate ADSR of a later phase adjoint
  env[0][lane] = dx[0];
  env[1][lane] = dx[1];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int pb = 32 + 8 * i;
    const double p = ph[i], erate = env[2 + 2 * i][lane];
    const double dl = dx[2 + i] * env[3 + 2 * i][lane];
    env[3 + 2 * i][lane] = dx[2 + i] * lfo[i];
    const double invW = dv[kLfoInvW + i];
    double dph = 0.0, dw = 0.0;
    if (invW > 0.0) {
      const double sd = (p * 2.0 - 1.0) > 0.0 ? 1.0 : ((p * 2.0 - 1.0) < 0.0 ? -1.0 : 0.0);
      const double der = v[pb + 3] * (0.5 * kTwoPi * cs[i]) + v[pb + 4] * (-2.0 * sd) + v[pb + 5] -
                         v[pb + 6];
      dw = own ? dl * invW : 0.0;
      dph = dw * der;
    }
    // phase: d phi += dph / 2 pi; d inc(k) = sum_{j > k} dph(j)
    const bool live = own && fpre[i] >= 0.0;
    const double unit = live ? 1.0 / rc : 0.0;
    const double later = wave_rev_excl_scan(dph, lane);
    const double df = live ? later / rc : 0.0;
    env[2 + 2 * i][lane] = live ? df * v[pb + 1] : 0.0;
    tail[i] = live ? unit * v[pb + 1] : 0.0;
    const int sl = kRowLfo + 12 * i;
    // what does not reach a parameter leaves it alone also where it is not finite
    const double er = live ? erate : 0.0, lf = invW > 0.0 ? lfo[i] : 0.0;
    emit4(S.part, sl, lane, df, df * er, dph / kTwoPi, dw * ((1.0 + sn[i]) / 2.0 - lf));
    emit4(S.part, sl + 4, lane, dw * (1.0 - fabs(2.0 * p - 1.0) - lf), dw * (p - lf),
          dw * (1.0 - p - lf), dw * ((p < 0.5 ? 1.0 : 0.0) - lf));
    emit4(S.part, sl + 8, lane, unit, unit * er, dph, 0.0);
  }
  // ADSRs: derivatives per unit of the envelope's adjoint (0 where neither it
  // nor a later phase adjoint reaches the envelope)
  double goff = 0.0;
#pragma unroll 1
  for (int k = 0; k < 6; ++k) {
    const double de = own ? env[k][lane] : 0.0;
    const double tl = k == 2 ? tail[0] : k == 4 ? tail[1] : 0.0;
    double dA = 0.0, dD = 0.0, dS = 0.0, dR = 0.0, dO = 0.0, dal = 0.0;
    bool live_a = false, live_d = false, live_r = false;   // ramps that the sample lies on
    if (de != 0.0 || tl != 0.0) {
      const double A = dv[kEnvA + k], D = dv[kEnvD + k], Rr = dv[kEnvR + k];
      const double iA = dv[kEnvInvA + k], iD = dv[kEnvInvD + k], iR = dv[kEnvInvR + k];
      const double Sus = dv[kEnvS + k], al = dv[kEnvAlpha + k];
      double Pa, Pd, Pr, xa, xd, xr, la, ld, lr;
      pow01_grad(ramp(jd, 0.0, A, iA), al, Pa, xa, la);
      pow01_grad(1.0 - ramp(jd, A, D, iD), al, Pd, xd, ld);
      pow01_grad(1.0 - ramp(jd, note_off, Rr, iR), al, Pr, xr, lr);
      const double M = Sus + (1.0 - Sus) * Pd;
      const double dPa = M * Pr, dM = Pa * Pr, dPr = Pa * M;
      const double dPd = dM * (1.0 - Sus);
      dS = dM * (1.0 - Pd);
      dal = dPa * la + dPd * ld + dPr * lr;
      live_a = ramp_live(jd, 0.0, A, iA);
      live_d = ramp_live(jd, A, D, iD);
      live_r = ramp_live(jd, note_off, Rr, iR);
      if (live_a) dA += dPa * xa * (-jd * iA * iA);
      if (live_d) {
        const double dd = -dPd * xd;       // d/d dec
        dA += dd * (-iD);
        dD += dd * (-(jd - A) * iD * iD);
      }
      if (live_r) {
        const double dr = -dPr * xr;       // d/d rel
        dO += dr * (-iR);
        dR += dr * (-(jd - note_off) * iR * iR);
      }
      dA *= rc;
      dD *= rc;
      dR *= rc;
      dO *= rc;
    }
    // a ramp that is not passed takes no adjoint, also not one that is not finite
    const double deA = live_a || live_d ? de : 0.0, deD = live_d ? de : 0.0, deR = live_r ? de : 0.0;
    goff += deR * dO;
    emit4(S.part, kRowEnv + 8 * k, lane, deA * dA, deD * dD, de * dS, deR * dR);
    emit4(S.part, kRowEnv + 8 * k + 4, lane, de * dal, tl * dal, tl * dO, 0.0);
    if (k == 2 || k == 4) emit4(S.part, kRowTail + 2 * k - 4, lane, tl * dA, tl * dD, tl * dS, tl * dR);
  }
  emit4(S.part, kRowOff, lane, goff, 0.0, 0.0, 0.0);
  __syncthreads();
  for (int n = lane; n < kNumSums; n += kWave) {
    const double* pr = S.part[sum_row(n)];
    double s = 0.0;
#pragma unroll
    for (int l = 0; l < kWave / 16; ++l) s += pr[l];
    (n < kPartOut ? out[n] : rv[tail_index(n, c, J)]) = s;
  }
}

// Per voice: the chunks' sums joined (last chunk first; the LFO factors times
// the phase adjoints of the chunks after theirs) and taken through the curve
// mapping's Jacobian to the normalised parameters.
constexpr int kParamThreads = 128;
__global__ void __launch_bounds__(kParamThreads) adjoint_params_kernel(const RenderArgs a,
                                                                       const double* __restrict__ red,
                                                                       CtlArgs t,
                                                                       float* __restrict__ grad_params) {
  __shared__ double tot[kNumSums];
  const int p = threadIdx.x;
  const int64_t b = blockIdx.x;
  const int64_t J = (a.n_uniform + a.q - 1) / a.q;
  if (p < kNumSums) {
    const double* rv = red + b * J * kNumRed;
    const double* gp = t.gpart + b * t.nchunks * kPartOut;
    auto sum_of = [&](int n, int64_t c) {
      return n < kPartOut ? gp[c * kPartOut + n] : rv[tail_index(n, c, J)];
    };
    double s = 0.0;
    if (p < kSumTail || p >= kSumDph) {
#pragma unroll 4
      for (int64_t c = t.nchunks - 1; c >= 0; --c) s += sum_of(p, c);
    } else {
      const int dp = kSumDph + (p - kSumTail) / 8;
      double later = 0.0;
#pragma unroll 4
      for (int64_t c = t.nchunks - 1; c >= 0; --c) {
        const double f = sum_of(p, c), d = sum_of(dp, c);
        if (later != 0.0 && f != 0.0) s += later * f;
        later += d;
      }
    }
    tot[p] = s;
  }
  __syncthreads();
  if (p >= kNumParams) return;
  double s = tot[p];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int eb = 2 + 5 * (2 + 2 * i), lb = 32 + 8 * i, tb = kSumTail + 8 * i;
    if (p >= eb && p < eb + 5) s += tot[tb + p - eb];
    if (p == 1) s += tot[tb + 5];
    if (p == lb || p == lb + 1) s += tot[tb + 6 + p - lb];
  }
  const double u = (double)a.params[b * kNumParams + p];
  const NebulaArgs& nb = a.neb;
  const double span = nb.hi[p] - nb.lo[p];
  const bool lin = bit(nb.linear, p);
  const double e = nb.inv_curve[p];
  double jac;
  if (!bit(nb.sym, p)) {
    jac = lin ? span : (u > 0.0 ? span * e * pow(u, e - 1.0) : 0.0);
  } else {
    const double d = 2.0 * u - 1.0;
    const double ad = fabs(d);
    jac = ad > 0.0 ? (lin ? span : span * e * pow(ad, e - 1.0)) : 0.0;
  }
  grad_params[b * kNumParams + p] = (float)(s * jac);
}

template <int RPS>
hipError_t launch_adjoint_rps(const RenderArgs& a, const float* g, double* red, float* gp,
                              hipStream_t s) {
  size_t shmem = (size_t)kWave * (a.q / RPS) * (sizeof(float) + sizeof(uint16_t));
  if (shmem < 8 * kWave * sizeof(double)) shmem = 8 * kWave * sizeof(double);
  const int64_t J = (a.n_uniform + a.q - 1) / a.q;
  CtlArgs t;
  t.nchunks = (J + kSegsPerChunk - 1) / kSegsPerChunk;
  t.carries = adjoint_carries(red, a.batch, a.n_uniform, a.q);
  t.gpart = t.carries + a.batch * t.nchunks * 4;
  hipLaunchKernelGGL((adjoint_audio_kernel<RPS>), dim3((unsigned)(a.batch * a.slices * a.pass_split)),
                     dim3(kWave),
                     shmem, s, a, g, red, t);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(adjoint_chunk_grad_kernel, dim3((unsigned)(a.batch * t.nchunks)), dim3(kWave), 0,
                     s, a, red, t);
  hipLaunchKernelGGL(adjoint_params_kernel, dim3((unsigned)a.batch), dim3(kParamThreads), 0, s, a, red,
                     t, gp);
  return hipGetLastError();
}

}  // namespace

size_t adjoint_workspace_bytes(int64_t batch, int64_t n_samples, int q) {
  // per-segment sums [batch][21][J], the chunk-start carries [batch][chunks][4],
  // then the chunks' adjoint sums [batch][chunks][84]
  const int64_t J = (n_samples + q - 1) / q;
  const int64_t nchunks = (J + kSegsPerChunk - 1) / kSegsPerChunk;
  return (size_t)batch * ((size_t)J * kNumRed + (size_t)nchunks * (4 + kPartOut)) *
         sizeof(double);
}

double* adjoint_carries(double* ws, int64_t batch, int64_t n_samples, int q) {
  const int64_t J = (n_samples + q - 1) / q;
  return ws + batch * J * kNumRed;
}

int64_t adjoint_max_chunks() { return 512; }

hipError_t launch_render_backward(const RenderArgs& a, const float* grad_audio, double* ws,
                                  float* grad_params, int runs_per_segment, hipStream_t s) {
  if (a.batch == 0) return hipSuccess;
  switch (runs_per_segment) {
    case 1: return launch_adjoint_rps<1>(a, grad_audio, ws, grad_params, s);
    case 4: return launch_adjoint_rps<4>(a, grad_audio, ws, grad_params, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace synth
