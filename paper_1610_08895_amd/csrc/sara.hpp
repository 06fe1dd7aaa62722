// Internal state of the SARA sparsity dictionary (Sec. III): Dirac plus Daubechies bases.
#pragma once

#include "common.hpp"

namespace ri {

constexpr int MAX_WAVELETS = 8;
constexpr int MAX_TAPS = 16;  // db8

// Filters of the wavelet bases, by wavelet slot.  On the device they live in one buffer,
// FILT_STRIDE floats per slot (lowpass h in [0, 16), highpass g in [16, 32)), read through
// a pointer with uniform indices (scalar loads).
constexpr int FILT_STRIDE = 2 * MAX_TAPS;
struct SaraFilters {
  float h[MAX_WAVELETS][MAX_TAPS];
  float g[MAX_WAVELETS][MAX_TAPS];
  int len[MAX_WAVELETS];
};

struct Sara {
  int n = 0, levels = 0;
  int dirac = 0;  // 1 if basis 0 is the Dirac basis
  int nw = 0;     // number of wavelet bases
  int b = 0;      // dirac + nw
  SaraFilters filt{};
  float* dfilt = nullptr;  // nw * FILT_STRIDE
  int* dlen = nullptr;     // nw
  size_t tmp_stride = 0;        // floats of LL scratch per wavelet
  size_t tmp_off[8] = {0};      // offset of LL_l (l = 1..levels-1) inside a wavelet's scratch
  float* tmp = nullptr;         // nw * tmp_stride
  float* coef_tmp = nullptr;    // b * n * n, power iterations
  float* vec_tmp = nullptr;     // n * n, power iterations
  double* dsum = nullptr;
};

// s = Psi^dagger x, or with clip: s = clip(s + Psi^dagger x, -alpha, alpha) (step 13 Moreau form);
// with weights wts (b*n*n, the layout of s) the bound of coefficient k is alpha * wts[k].
int psi_adj_apply(const Sara& S, const float* x, float* s, bool clip, float alpha, hipStream_t st,
                  const float* wts = nullptr);
// x = Psi s.
int psi_apply(const Sara& S, const float* s, float* x, hipStream_t st);
// Steps 13 and 14: the clipped analysis of x into s, then out = Psi s (bit for bit the two calls
// above, in fewer launches where levels are small).
int sparsity_apply(const Sara& S, const float* x, float* s, float alpha, const float* wts, float* out, hipStream_t st);

// ---- kernel arguments ----
struct DwtArgs {
  const float* x;  // level-1 input (n x n)
  float* tmp;
  size_t tmp_stride, in_off, out_off;
  float* s;
  int n, m, level, levels, dirac, nw;
  int clip;
  float alpha;
  const float* wts;  // per-coefficient weights of the clip bound (layout of s), or null
  // reverse sweep: s <- |gate| < bound ? s + scale v : 0 instead of the clip (gate: layout of s)
  const float* gate;
  float scale;
};

struct IdwtArgs {
  const float* s;
  float* tmp;
  size_t tmp_stride, ll_off, out_off;
  int n, m, level, levels, dirac, nw;
  float* x;  // top level only: the image Psi s
};

constexpr int DEEP = 64;  // largest input of the deep levels
struct DeepArgs {
  DwtArgs a;
  int first;      // first level
  size_t ll_off;  // offset of its input (analysis) and output (synthesis) in a wavelet's scratch
  int analyse, synth;
};

// The sparsity branch cut into jobs that ride on the launches of the data branch, as workgroups
// added to theirs (wgs = 0: nothing to add).
enum { SIDE_NONE = 0, SIDE_DWT = 1, SIDE_IDWT = 2, SIDE_DEEP = 3, SIDE_TOP = 4, SIDE_DWT_GATE = 5, SIDE_DEEP_GATE = 6 };
struct SideJob {
  int wgs = 0, nx = 0, ny = 0;
  const float* filt = nullptr;
  const int* flen = nullptr;
  DwtArgs a{};
  IdwtArgs i{};
  DeepArgs e{};
};
struct SideJobs {
  SideJob first, second;  // analysis levels 1 and 2 (SIDE_DWT; second only if the deep levels start at 3)
  SideJob deep;           // SIDE_DEEP
  SideJob lower;          // synthesis level 2 (SIDE_IDWT; only with second)
  SideJob top;            // finest synthesis level (SIDE_TOP)
};
// The jobs of sparsity_apply, each to run after the one before it; false if the dictionary has
// other levels than they cover.
bool side_jobs(const Sara& S, const float* x, float* s, float alpha, const float* wts, float* out, SideJobs& j);
// Of the reverse sweep: out = Psi s (deep, then top), and s <- |gate| < bound ? s + scale Psi^dagger x
// : 0, then out = Psi s (first, deep, top; of the kinds that heed the gate).  False unless the deep
// levels start at the second.
bool side_synthesis(const Sara& S, const float* s, float* out, SideJobs& j);
bool side_gated(const Sara& S, const float* x, float* s, const float* gate, float scale, float alpha, const float* wts,
                float* out, SideJobs& j);
// The job `top` in a launch of its own.
int side_top(const Sara& S, const SideJob& j, hipStream_t st);

}  // namespace ri
