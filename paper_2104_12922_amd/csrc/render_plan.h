// The library's default launch plan of a render (host arithmetic only).
#pragma once

#include <math.h>
#include <stdint.h>

namespace synth {

constexpr int kChunkSegments = 62;   // control periods per chunk

inline int64_t chunks_of(int64_t n_samples, int q) {
  const int64_t J = (n_samples + q - 1) / q;
  return (J + kChunkSegments - 1) / kChunkSegments;
}

struct RenderPlan {
  int rps;          // runs per segment
  int slices;       // parts of a voice's chunks, workgroups of their own
  int pass_split;   // workgroups that share a slice's passes
};

// Runs per segment 4 (1 if q is not a multiple of 4); uniform batches
// (n_samples > 0) of fewer than 2048 voices split each voice over workgroups so
// that the grid covers the chip - at most a quarter of its chunks when the
// slices walk the earlier chunks for their carries.
//
// When the carries are computed first (carried), every chunk is a workgroup:
// the finest parts even out the notes' silent ends best (us: 256 voices of 43
// chunks, 8 parts 187, 16 177, 31 167, 43 148; 512 of 64, 16 parts 366, 64 335;
// 1500 of 72, 6 parts 1135, 72 1034; 8192 workgroups as the aim took 239, 483
// and 1118).
//
// Then the passes (of 16 control periods) of a chunk, up to 4, are split while
// the chip has fewer than two workgroups per CU: each part forms the chunk's
// control stage for itself, so only where no carries are walked, and a part
// without a pass would be idle.  The passes halve the render of 8 voices of 1 s
// (25 -> 16 us).
inline RenderPlan default_render_plan(double sample_rate, double control_rate, int64_t batch,
                                      int64_t n_samples, bool carried) {
  RenderPlan p = {4, 1, 1};
  if (!(control_rate > 0.0)) return p;
  const double q = nearbyint(sample_rate / control_rate);
  if (fmod(q, 4.0) != 0.0) p.rps = 1;
  if (!(n_samples > 0 && batch > 0 && q >= 4.0)) return p;
  const int64_t nchunks = chunks_of(n_samples, (int)q);
  int64_t want = (2048 + batch - 1) / batch;
  if (carried && want > 1 && nchunks <= 0x7FFFFFFF / batch) want = nchunks;
  else if (want > nchunks / 4) want = nchunks / 4;
  if (want > 1) p.slices = (int)want;
  if (p.rps == 4 && (carried ? p.slices > 1 : nchunks == 1)) {
    const int64_t passes = ((n_samples + (int)q - 1) / (int)q + 15) / 16;
    while (p.pass_split < 4 && p.pass_split < passes && batch * p.slices * p.pass_split < 512)
      p.pass_split *= 2;
  }
  return p;
}

}  // namespace synth
