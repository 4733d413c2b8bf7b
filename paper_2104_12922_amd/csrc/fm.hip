// Four-operator FM voice (the FM architecture Sections 3.2 and 7 announce).
// Four sine operators on the keyboard pitch, operator i at f_i = 440
// 2^((midi_f0 - 69) / 12) ratio_i 2^(detune_i / 1200) (at most sr / 2), each
// scaled by its level and its own ADSR (the Voice's envelope at the control
// rate, upsampled linearly, holding the last control value); operator j
// modulates operator i < j's phase with index M[i][j] cycles:
//   o_i(n) = level_i env_i(n) sin(2 pi (n f_i / sr + sum_{j > i} M[i][j] o_j(n)))
// for i = 3, 2, 1, 0, and y(n) = sum_i w_i o_i(n) / max(1, sum_i w_i).
//
// No operator feeds back on itself, so every sample is a closed-form
// function of n: one wavefront per voice takes 64 control periods (a chunk)
// at a time; lane l evaluates the four envelopes at control sample
// 64c + l + 1 (float64, the Voice's ADSR code; 64c is the previous chunk's
// last) into LDS, then every lane renders four
// consecutive samples per step (lanes on consecutive 16-byte groups, so each
// store instruction writes 1 KB of contiguous audio).  The four samples share
// a control period; the phase n f_i / sr of the first is a whole number of
// 2^-64 cycles that wraps by itself and advances by one 64-bit addition per
// step (off by at most n 2^-64 cycles from the truncation of f_i / sr to that
// unit, against n f_i / sr 2^-53 from a float64 product).  Its upper 32 bits are
// the float32 phase in [0, 1], cut to whole 2^-32 cycles: a phase below 2^-8 has
// fewer significant bits than a float32 of its own scale would (2.3e-10 cycles
// at most).  The next three samples add f_i / sr in float32 (within 2e-7
// cycles), and the float32 hardware sine takes revolutions.  Periods after every
// envelope has reached 0 are zero-filled without computation.  Bound by VALU
// issue (busy for the whole launch by counter): four sines, at half rate, and
// about 25 other instructions per sample, 32.9 in all with the control stage, at
// five wavefronts per SIMD (91 registers; with the operators' constants in
// vector registers 123 and four).  16384 voices of 1, 2 and 4 s: 1970 us with a
// float64 product, floor and conversion per operator and step, 1790 with
// fixed-point phases and envelope pairs read as vectors, 1774 with the constants
// formed by a lane each and kept in scalar registers; 65536 voices of 500
// samples 144, 164 and 128.
#include "voice_device.h"

namespace synth {
namespace {

using voice::adsr_value;
using voice::kEnvA;
using voice::kEnvAlpha;
using voice::kEnvD;
using voice::kEnvInvA;
using voice::kEnvInvD;
using voice::kEnvInvR;
using voice::kEnvR;
using voice::kEnvS;
using voice::kDerived;
using voice::map_param;

constexpr int kFmParams = 44;
constexpr int kOpBase[4] = {2, 10, 18, 26};
constexpr int kModBase = 34, kMixBase = 40;

struct FmArgs {
  const float* params;       // [B][44] normalised
  const int64_t* offsets;    // [B + 1] or null
  int64_t n_uniform;
  int64_t batch;
  float* audio;
  double sr, rc;
  int q;
  uint32_t q_magic;          // x / q == umulhi(x, q_magic) for x < 2^16
  NebulaArgs neb;            // first 44 entries used
  const int32_t* order;      // null, or the voices in the order workgroups take them
};

// Lane `from`'s value in a scalar register.
__device__ __forceinline__ float of_lane(float x, int from) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), from));
}
__device__ __forceinline__ uint64_t of_lane(uint64_t x, int from) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(x >> 32), from) << 32 |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)x, from);
}

__global__ void __launch_bounds__(64) fm_render_kernel(FmArgs a) {
  __shared__ double v[kFmParams];
  __shared__ double dv[kDerived];
  __shared__ __align__(16) float env0[64][4], envd[64][4];   // per period: value at its start, slope
  __shared__ __align__(16) float last[4];                    // value at the last chunk's end
  const int lane = threadIdx.x;
  const int64_t b = a.order ? (int64_t)a.order[blockIdx.x] : (int64_t)blockIdx.x;
  if (b < 0 || b >= a.batch) return;         // an order entry out of range renders nothing
  int64_t start, L;
  if (a.offsets) {
    packed_range(a.offsets, a.batch, b, start, L);
  } else {
    start = b * a.n_uniform;
    L = a.n_uniform;
  }
  if (L <= 0) return;
  float* out = a.audio + start;
  if (lane < kFmParams) v[lane] = map_param((double)a.params[b * kFmParams + lane], lane, a.neb);
  __syncthreads();
  const double rc = a.rc;
  if (lane < 4) {                          // envelope of operator `lane`, in control samples
    const int pb = kOpBase[lane] + 3;
    const double A = v[pb] * rc, D = v[pb + 1] * rc, R = v[pb + 3] * rc;
    dv[kEnvA + lane] = A;
    dv[kEnvInvA + lane] = 1.0 / A;
    dv[kEnvD + lane] = D;
    dv[kEnvInvD + lane] = 1.0 / D;
    dv[kEnvR + lane] = R;
    dv[kEnvInvR + lane] = 1.0 / R;
    dv[kEnvS + lane] = v[pb + 2];
    dv[kEnvAlpha + lane] = v[pb + 4];
  }
  __syncthreads();
  const double note_off = v[1] * rc;
  // operator constants and the envelope's first value: lane i forms operator i's,
  // the constants then go to scalar registers (formed by every lane for all four,
  // 65536 voices of 100 samples took 127 us)
  uint64_t incx[4];                        // cycles per sample in units of 2^-64
  float lvl[4], incf[4];
  {
    const int pb = kOpBase[0] + (kOpBase[1] - kOpBase[0]) * (lane & 3);
    const double f = 440.0 * voice::exp2_f64((v[0] - 69.0) / 12.0) * v[pb] *
                     voice::exp2_f64(v[pb + 1] / 1200.0);
    // limited from above only: whole cycles below -1/2 are taken out (exactly),
    // and a negative increment is the wrapped negative of its magnitude (a
    // conversion of a negative number to unsigned is undefined)
    double inc = fmin(f, a.sr / 2.0) / a.sr;
    inc -= rint(inc);
    const uint64_t mag = (uint64_t)(fabs(inc) * 0x1p64);
    if (lane < 4) last[lane] = (float)v[pb + 2] * (float)adsr_value(dv, lane, 0.0, note_off);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      incx[i] = of_lane(inc < 0.0 ? 0 - mag : mag, i);
      incf[i] = of_lane((float)inc, i);
      lvl[i] = of_lane((float)v[pb + 2], i);
    }
  }
  __syncthreads();
  float nan0[4];                           // 0, or NaN for a frequency of minus infinity
#pragma unroll
  for (int i = 0; i < 4; ++i) nan0[i] = 0.0f * incf[i];
  const float m01 = of_lane((float)v[kModBase], 0), m02 = of_lane((float)v[kModBase + 1], 0);
  const float m03 = of_lane((float)v[kModBase + 2], 0), m12 = of_lane((float)v[kModBase + 3], 0);
  const float m13 = of_lane((float)v[kModBase + 4], 0), m23 = of_lane((float)v[kModBase + 5], 0);
  const double wsum = v[kMixBase] + v[kMixBase + 1] + v[kMixBase + 2] + v[kMixBase + 3];
  const double wn = 1.0 / fmax(1.0, wsum);
  const float w0 = of_lane((float)(v[kMixBase] * wn), 0), w1 = of_lane((float)(v[kMixBase + 1] * wn), 0);
  const float w2 = of_lane((float)(v[kMixBase + 2] * wn), 0), w3 = of_lane((float)(v[kMixBase + 3] * wn), 0);
  // every envelope is exactly 0 from control sample note_off + R_i on; a
  // period whose two control values are 0 is silent
  double rel_end = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) rel_end = fmax(rel_end, note_off + dv[kEnvR + i]);
  const int64_t J = (L + a.q - 1) / a.q;
  const int64_t j_silent = (int64_t)fmin((double)J, floor(rel_end) + 2.0);
  const float inv_q = 1.0f / (float)a.q;
  const bool vec = ((start & 3) == 0);
  for (int64_t j0 = 0; j0 < J; j0 += 64) {
    const int64_t c0 = j0 * a.q;
    const int cnt = (int)min((int64_t)64 * a.q, L - c0);
    if (j0 >= j_silent) {                  // silent from here on: zero-fill the rest
      for (int64_t p = c0 + 4 * lane; p < L; p += 256) {
        if (vec && p + 4 <= L) {
          *reinterpret_cast<float4*>(out + p) = make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
          for (int e = 0; e < 4 && p + e < L; ++e) out[p + e] = 0.0f;
        }
      }
      break;
    }
    // control values at j0 + 0 .. 64 (the last period holds its value): lane
    // l evaluates j0 + l + 1, the end of period l, and takes its start from
    // lane l - 1; the value at j0 is the previous chunk's last one (the same
    // control sample; before the first chunk, the one at 0).  Operator 0
    // modulates nothing: its mix weight is in its envelope.
    {
      const double jd = (double)min(j0 + lane + 1, J - 1);
      float r[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = lvl[i] * (float)adsr_value(dv, i, jd, note_off);
      float l[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        l[i] = __shfl_up(r[i], 1);
        if (lane == 0) l[i] = last[i];
      }
      *reinterpret_cast<float4*>(env0[lane]) = make_float4(w0 * l[0], l[1], l[2], l[3]);
      *reinterpret_cast<float4*>(envd[lane]) =
          make_float4(w0 * (r[0] - l[0]), r[1] - l[1], r[2] - l[2], r[3] - l[3]);
      __syncthreads();                     // last is read before it is written
      if (lane == 63) *reinterpret_cast<float4*>(last) = make_float4(r[0], r[1], r[2], r[3]);
    }
    __syncthreads();
    uint64_t ph64[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      ph64[i] = (uint64_t)c0 * incx[i] + (uint64_t)(uint32_t)(4 * lane) * incx[i];
    for (int p = 4 * lane; p < cnt; p += 256) {
      // samples p .. p + 3 lie in one control period (q and p are multiples
      // of 4): one period index, one phase per operator, the other three
      // phases and envelope values by float32 steps from it
      const int seg = (int)__umulhi((uint32_t)p, a.q_magic);
      const float t0 = (float)(p - seg * a.q) * inv_q;
      const float4 ev = *reinterpret_cast<const float4*>(env0[seg]);
      const float4 dvv = *reinterpret_cast<const float4*>(envd[seg]);
      const float e0[4] = {ev.x, ev.y, ev.z, ev.w}, de[4] = {dvv.x, dvv.y, dvv.z, dvv.w};
      float ph0[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ph0[i] = fmaf((float)(uint32_t)(ph64[i] >> 32), 0x1p-32f, nan0[i]);
        ph64[i] += incx[i] << 8;
      }
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = fmaf((float)e, inv_q, t0);
        float ph[4], en[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          ph[i] = fmaf((float)e, incf[i], ph0[i]);
          en[i] = fmaf(t, de[i], e0[i]);
        }
        const float o3 = en[3] * __builtin_amdgcn_sinf(ph[3]);
        const float o2 = en[2] * __builtin_amdgcn_sinf(fmaf(m23, o3, ph[2]));
        const float o1 = en[1] * __builtin_amdgcn_sinf(fmaf(m12, o2, fmaf(m13, o3, ph[1])));
        const float s0 = __builtin_amdgcn_sinf(fmaf(m01, o1, fmaf(m02, o2, fmaf(m03, o3, ph[0]))));
        y[e] = fmaf(en[0], s0, fmaf(w1, o1, fmaf(w2, o2, w3 * o3)));
      }
      const int64_t n0 = c0 + p;
      if (vec && p + 4 <= cnt) {
        *reinterpret_cast<float4*>(out + n0) = make_float4(y[0], y[1], y[2], y[3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (p + e < cnt) out[n0 + e] = y[e];
      }
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_fm_render(const float* params, const int64_t* offsets, int64_t batch,
                            int64_t n_samples, float* audio, double sr, double rc, int q,
                            const NebulaArgs& neb, const int32_t* order, hipStream_t s) {
  if (batch == 0) return hipSuccess;
  FmArgs a;
  a.params = params;
  a.offsets = offsets;
  a.n_uniform = offsets ? 0 : n_samples;
  a.batch = batch;
  a.audio = audio;
  a.sr = sr;
  a.rc = rc;
  a.q = q;
  a.q_magic = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)q - 1) / (uint64_t)q);
  a.neb = neb;
  a.order = order;
  hipLaunchKernelGGL(fm_render_kernel, dim3((unsigned)batch), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace synth
