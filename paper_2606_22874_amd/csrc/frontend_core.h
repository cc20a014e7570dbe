// Shared by the selector front end's kernels: the rotary frequencies and the
// angle of one (position, pair).
#pragma once

#include "spot_internal.h"

namespace spot {

constexpr int kMaxRopePairs = 64;

// base^(-2i / rope_dim) for the rotary pairs i < rope_dim / 2 (FP64).
struct RopeFreq {
  double f[kMaxRopePairs];
};

// Sine and cosine of pos * freq: the angle in FP64, reduced in FP64 by a
// multiple of pi/2 (in two parts) to [-pi/4, pi/4], then the minimax
// polynomials of Moshier's Cephes library for that range in FP32 (a general
// sincosf brings its own reduction for large arguments along, three times the
// instructions).  Errors against the sine and cosine of the FP64 angle are below
// 1e-7 for angles up to 2^40; past 2^53, which only a rope_base below 1 gives,
// the quarter turns are no longer exact, and the clamp keeps the values bounded
// (the angle itself, rounded to FP64, has no fraction of a turn left there).
// (On the host for its test.)
__host__ __device__ __forceinline__ void rope_sincos(int pos, double freq, float& s, float& c) {
  const double theta = (double)pos * freq;
  const double k = rint(theta * 0.6366197723675814);    // 2 / pi
  double red = fma(-k, 1.5707963267948966, theta);      // pi / 2, high part
  red = fma(-k, 6.123233995736766e-17, red);            // pi / 2, low part
  const int q = (int)(k - 4.0 * floor(k * 0.25));       // quarter turns, 0 .. 3
  const float x = fminf(fmaxf((float)red, -0.79f), 0.79f), z = x * x;
  const float sn =
      fmaf(fmaf(fmaf(-1.9515295891e-4f, z, 8.3321608736e-3f), z, -1.6666654611e-1f) * z, x, x);
  const float cs = fmaf(
      fmaf(fmaf(2.443315711809948e-5f, z, -1.388731625493765e-3f), z, 4.166664568298827e-2f) * z,
      z, fmaf(-0.5f, z, 1.f));
  const float a = q & 1 ? cs : sn, b = q & 1 ? sn : cs;
  s = q & 2 ? -a : a;
  c = (q + 1) & 2 ? -b : b;
}

// Arguments of a projection, as spot_selector_project documents them.
struct ProjectArgs {
  const uint16_t *h, *w_q, *w_k, *w_w;
  const int32_t* pos;
  int rows, d_model, h_s, d_s, rope_dim;
  RopeFreq freq;
  uint16_t* q_out;
  float* w_out;
  uint16_t* k_cache;
  int rows_per_seq, l_cap;
};

// Projection of many rows on the matrix cores (frontend_mfma.hip), and which
// calls it takes.
bool project_mfma_takes(int rows, int d_model);
hipError_t launch_project_mfma(const ProjectArgs& a, hipStream_t s);

}  // namespace spot
