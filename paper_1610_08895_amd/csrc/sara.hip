// SARA dictionary: Psi^dagger (analysis, Algorithm 1 step 13) and Psi (synthesis,
// step 14) for the Dirac basis plus Daubechies wavelets, as periodic separable 2D filter
// banks.  One analysis level of an m x m input, per axis:
//   a[k] = sum_j h[j] x[(2k + j) mod m],   d[k] = sum_j g[j] x[(2k + j) mod m],
// x (columns) first, then y (rows), written in Mallat layout; synthesis is the transpose.
//
// Each workgroup owns an output tile and stages the input it needs in LDS together with
// its periodic halo (filter length - 2 samples), then runs the row and the column filters
// from LDS; the filter length is a compile-time constant per basis.  Levels small enough for
// one workgroup's LDS run together in one launch.  Synthesis computes
// output pairs (2q, 2q + 1) from the same coefficients a[q - u], d[q - u].  Analysis of
// level 1 reads x~ once per wavelet from L2; the dual update of step 13,
// s = clip(s + Psi^dagger x~, -alpha, alpha), is applied as each coefficient is produced,
// with the old coefficients loaded before the input is staged; for the weighted l1 prior of
// reweighted SARA the bound is alpha w_k, with the weights w laid out like s.  The last
// synthesis level sums all bases.
#include <cmath>
#include <new>
#include <vector>

#include "host_math.hpp"
#include "handles.hpp"
#include "sara.hpp"
#include "sara_dev.hpp"

namespace ri {
namespace {

__global__ __launch_bounds__(ST) void k_dwt_level(DwtArgs A, const float* __restrict__ filt,
                                                  const int* __restrict__ flen, int nx, int ny) {
  __shared__ __align__(16) char smem[DWT_SMEM];
  dwt_body<false>(A, filt, flen, blockIdx.x, nx, ny, smem);
}

__global__ __launch_bounds__(ST) void k_idwt_level(IdwtArgs A, const float* __restrict__ filt,
                                                   const int* __restrict__ flen, int nx, int ny) {
  __shared__ __align__(16) char smem[IDWT_SMEM];
  idwt_body(A, filt, flen, blockIdx.x, nx, ny, smem);
}

template <int TG>
__global__ __launch_bounds__(ST * TG) void k_idwt_top(IdwtArgs A, const float* __restrict__ filt,
                                                      const int* __restrict__ flen, int nx, int ny) {
  __shared__ __align__(16) char smem[TOP_SMEM<TG>];
  top_body<TG>(A, filt, flen, blockIdx.x, nx, ny, smem);
}

__global__ __launch_bounds__(DEEP_THREADS) void k_sara_deep(DeepArgs E, const float* __restrict__ filt,
                                                            const int* __restrict__ flen) {
  __shared__ __align__(16) char smem[DEEP_SMEM];
  deep_body<false>(E, filt, flen, blockIdx.x, smem);
}

int tiles(int outputs, int t) { return (outputs + t - 1) / t; }

DwtArgs dwt_args(const Sara& S, int lev, const float* x, float* s, bool clip, float alpha, const float* wts) {
  return DwtArgs{x, S.tmp, S.tmp_stride, lev >= 2 ? S.tmp_off[lev - 1] : 0, lev < S.levels ? S.tmp_off[lev] : 0,
                 s, S.n, S.n >> (lev - 1), lev, S.levels, S.dirac, S.nw, clip ? 1 : 0, alpha, wts, nullptr, 0.f};
}

IdwtArgs idwt_args(const Sara& S, int lev, const float* s, float* x) {
  return IdwtArgs{s, S.tmp, S.tmp_stride, lev < S.levels ? S.tmp_off[lev] : 0, lev >= 2 ? S.tmp_off[lev - 1] : 0,
                  S.n, S.n >> (lev - 1), lev, S.levels, S.dirac, S.nw, x};
}

// The first level of the deep kernel (levels + 1: none).
int deep_first(const Sara& S) {
  if (S.nw == 0) return S.levels + 1;
  int lev = 2;
  while (lev <= S.levels && (S.n >> (lev - 1)) > DEEP) ++lev;
  return lev;
}

DeepArgs deep_args(const Sara& S, float* s, bool analyse, bool synth, bool clip, float alpha, const float* wts) {
  const int first = deep_first(S);
  return DeepArgs{dwt_args(S, first, nullptr, s, clip, alpha, wts), first, S.tmp_off[first - 1], analyse ? 1 : 0,
                  synth ? 1 : 0};
}

int launch_deep(const Sara& S, const DeepArgs& e, hipStream_t st) {
  hipLaunchKernelGGL(k_sara_deep, dim3(S.nw), dim3(DEEP_THREADS), 0, st, e, S.dfilt, S.dlen);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

// Analysis of levels 1 .. last, one launch each.
int analysis_levels(const Sara& S, const float* x, float* s, bool clip, float alpha, const float* wts, int last,
                    hipStream_t st) {
  for (int lev = 1; lev <= last; ++lev) {
    const int t = tiles(S.n >> lev, TO), z = S.nw + ((lev == 1 && S.dirac) ? 1 : 0);
    if (z == 0) continue;
    hipLaunchKernelGGL(k_dwt_level, dim3(t * t * z), dim3(ST), 0, st, dwt_args(S, lev, x, s, clip, alpha, wts),
                       S.dfilt, S.dlen, t, t);
    RI_LAUNCH_CHECK();
  }
  return RI_OK;
}

// Synthesis of levels first .. 2, one launch each, then the finest.
int synthesis_levels(const Sara& S, const float* s, float* x, int first, hipStream_t st) {
  for (int lev = first; lev >= 2 && S.nw > 0; --lev) {
    const int t = tiles(S.n >> (lev - 1), TS);
    hipLaunchKernelGGL(k_idwt_level, dim3(t * t * S.nw), dim3(ST), 0, st, idwt_args(S, lev, s, nullptr), S.dfilt,
                       S.dlen, t, t);
    RI_LAUNCH_CHECK();
  }
  const int t = tiles(S.n, TS);
  const IdwtArgs A = idwt_args(S, 1, s, x);
  if (t * t <= 2 * 256)  // at most two tiles per CU
    hipLaunchKernelGGL(k_idwt_top<TOP_GROUPS>, dim3(t * t), dim3(ST * TOP_GROUPS), 0, st, A, S.dfilt, S.dlen, t, t);
  else
    hipLaunchKernelGGL(k_idwt_top<1>, dim3(t * t), dim3(ST), 0, st, A, S.dfilt, S.dlen, t, t);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

void destroy_sara(Sara& S) {
  dev_free(S.tmp);
  dev_free(S.coef_tmp);
  dev_free(S.vec_tmp);
  dev_free(S.dsum);
  dev_free(S.dfilt);
  dev_free(S.dlen);
}

int create_sara(Sara& S, int n, int levels, uint32_t bases) {
  if (bases == 0) bases = 0x1FF;
  if (bases & ~0x1FFu) return fail(RI_EINVAL, "bases bitmask 0x%x has bits above db8", bases);
  if (levels < 1 || levels > 6) return fail(RI_EINVAL, "levels=%d must be in [1, 6]", levels);
  if (!is_pow2(n) || n > 4096 || n < (1 << levels) || n < 4)
    return fail(RI_EINVAL, "n=%d must be a power of two in [max(4, 2^levels), 4096] (levels=%d)", n, levels);
  S.n = n;
  S.levels = levels;
  S.dirac = (bases & 1u) ? 1 : 0;
  S.nw = 0;
  for (int N = 1; N <= 8; ++N) {
    if (!(bases & (1u << N))) continue;
    std::vector<double> h;
    double err = 1.0;
    daubechies_lowpass(N, h, &err);
    if (!(err < 1e-12)) return fail(RI_EINVAL, "db%d filter orthonormality error %.3g", N, err);
    const int w = S.nw++;
    S.filt.len[w] = 2 * N;
    for (int j = 0; j < 2 * N; ++j) {
      S.filt.h[w][j] = float(h[j]);
      S.filt.g[w][j] = float(((j & 1) ? -1.0 : 1.0) * h[2 * N - 1 - j]);
    }
  }
  S.b = S.dirac + S.nw;
  S.tmp_stride = 0;
  for (int l = 1; l < levels; ++l) {
    S.tmp_off[l] = S.tmp_stride;
    S.tmp_stride += size_t(n >> l) * (n >> l);
  }
  RI_TRY(dev_alloc(&S.tmp, size_t(S.nw) * S.tmp_stride));
  RI_TRY(dev_alloc(&S.coef_tmp, size_t(S.b) * n * n));
  RI_TRY(dev_alloc(&S.vec_tmp, size_t(n) * n));
  RI_TRY(dev_alloc(&S.dsum, SUMSQ_SCRATCH));
  if (S.nw > 0) {
    std::vector<float> f(size_t(S.nw) * FILT_STRIDE, 0.f);
    for (int w = 0; w < S.nw; ++w)
      for (int j = 0; j < MAX_TAPS; ++j) {
        f[size_t(w) * FILT_STRIDE + j] = S.filt.h[w][j];
        f[size_t(w) * FILT_STRIDE + MAX_TAPS + j] = S.filt.g[w][j];
      }
    RI_TRY(dev_alloc(&S.dfilt, f.size()));
    RI_TRY(dev_alloc(&S.dlen, size_t(S.nw)));
    RI_HIP(hipMemcpy(S.dfilt, f.data(), f.size() * sizeof(float), hipMemcpyHostToDevice));
    RI_HIP(hipMemcpy(S.dlen, S.filt.len, S.nw * sizeof(int), hipMemcpyHostToDevice));
  }
  return RI_OK;
}

}  // namespace

int psi_adj_apply(const Sara& S, const float* x, float* s, bool clip, float alpha, hipStream_t st,
                  const float* wts) {
  const int first = deep_first(S);
  RI_TRY(analysis_levels(S, x, s, clip, alpha, wts, first - 1, st));
  return first <= S.levels ? launch_deep(S, deep_args(S, s, true, false, clip, alpha, wts), st) : RI_OK;
}

int psi_apply(const Sara& S, const float* s, float* x, hipStream_t st) {
  const int first = deep_first(S);
  if (first <= S.levels)  // the coefficients are only read
    RI_TRY(launch_deep(S, deep_args(S, const_cast<float*>(s), false, true, false, 0.f, nullptr), st));
  return synthesis_levels(S, s, x, first - 1, st);
}

int sparsity_apply(const Sara& S, const float* x, float* s, float alpha, const float* wts, float* out, hipStream_t st) {
  const int first = deep_first(S);
  RI_TRY(analysis_levels(S, x, s, true, alpha, wts, first - 1, st));
  if (first <= S.levels) RI_TRY(launch_deep(S, deep_args(S, s, true, true, true, alpha, wts), st));
  return synthesis_levels(S, s, out, first - 1, st);
}

bool side_jobs(const Sara& S, const float* x, float* s, float alpha, const float* wts, float* out, SideJobs& j) {
  const int first = deep_first(S);
  if (first > S.levels || first > 3) return false;
  auto dwt = [&](int lev) {
    const int t = tiles(S.n >> lev, TO), z = S.nw + ((lev == 1 && S.dirac) ? 1 : 0);
    SideJob q{t * t * z, t, t, S.dfilt, S.dlen};
    q.a = dwt_args(S, lev, x, s, true, alpha, wts);
    return q;
  };
  j.first = dwt(1);
  j.second = first == 3 ? dwt(2) : SideJob{};
  j.deep = SideJob{S.nw, 0, 0, S.dfilt, S.dlen};
  j.deep.e = deep_args(S, s, true, true, true, alpha, wts);
  const int t2 = tiles(S.n >> 1, TS), t = tiles(S.n, TS);
  j.lower = first == 3 ? SideJob{t2 * t2 * S.nw, t2, t2, S.dfilt, S.dlen} : SideJob{};
  j.lower.i = idwt_args(S, 2, s, nullptr);
  j.top = SideJob{t * t, t, t, S.dfilt, S.dlen};
  j.top.i = idwt_args(S, 1, s, out);
  return true;
}

bool side_synthesis(const Sara& S, const float* s, float* out, SideJobs& j) {
  if (deep_first(S) != 2 || S.levels < 2) return false;
  const int t = tiles(S.n, TS);
  j.deep = SideJob{S.nw, 0, 0, S.dfilt, S.dlen};
  j.deep.e = deep_args(S, const_cast<float*>(s), false, true, false, 0.f, nullptr);  // s is only read
  j.top = SideJob{t * t, t, t, S.dfilt, S.dlen};
  j.top.i = idwt_args(S, 1, s, out);
  return true;
}

bool side_gated(const Sara& S, const float* x, float* s, const float* gate, float scale, float alpha, const float* wts,
                float* out, SideJobs& j) {
  if (deep_first(S) != 2 || !side_jobs(S, x, s, alpha, wts, out, j)) return false;
  for (DwtArgs* a : {&j.first.a, &j.deep.e.a}) {
    a->gate = gate;
    a->scale = scale;
  }
  return true;
}

int side_top(const Sara& S, const SideJob& j, hipStream_t st) {
  return synthesis_levels(S, j.i.s, j.i.x, 1, st);
}

}  // namespace ri

using ri::fail;

extern "C" {

int ri_sara_create(ri_sara* out, int n, int levels, uint32_t bases, hipStream_t stream) {
  (void)stream;
  if (!out) return fail(RI_EINVAL, "out is NULL");
  *out = nullptr;
  ri_sara h = new (std::nothrow) ri_sara_s;
  if (!h) return fail(RI_ENOMEM, "host allocation failed");
  const int rc = ri::create_sara(h->s, n, levels, bases);
  if (rc != RI_OK) {
    ri::destroy_sara(h->s);
    delete h;
    return rc;
  }
  *out = h;
  return RI_OK;
}

void ri_sara_destroy(ri_sara sara) {
  if (!sara) return;
  ri::destroy_sara(sara->s);
  delete sara;
}

int ri_sara_bases(ri_sara sara, int* b) {
  if (!sara || !b) return fail(RI_EINVAL, "NULL argument");
  *b = sara->s.b;
  return RI_OK;
}

int ri_psi(ri_sara sara, const float* s, float* x, hipStream_t stream) {
  if (!sara || !s || !x) return fail(RI_EINVAL, "NULL argument");
  return ri::psi_apply(sara->s, s, x, stream);
}

int ri_psi_adj(ri_sara sara, const float* x, float* s, hipStream_t stream) {
  if (!sara || !s || !x) return fail(RI_EINVAL, "NULL argument");
  return ri::psi_adj_apply(sara->s, x, s, false, 0.f, stream);
}

int ri_psi_norm(ri_sara sara, float* x0, int max_it, double rtol, double* norm_host, int* iters_host,
                hipStream_t stream) {
  if (!sara || !x0 || !norm_host || max_it < 1) return fail(RI_EINVAL, "bad argument");
  ri::Sara& S = sara->s;
  const size_t N = size_t(S.n) * S.n;
  float* cur = x0;
  float* nxt = S.vec_tmp;
  double lam = 0.0, lam_prev = 0.0, sq = 0.0;
  int it;
  RI_TRY(ri::sumsq_f32(cur, N, S.dsum, stream));
  RI_TRY(ri::scale_by_rsqrt(cur, N, S.dsum, stream));
  for (it = 1; it <= max_it; ++it) {
    RI_TRY(ri::psi_adj_apply(S, cur, S.coef_tmp, false, 0.f, stream));
    RI_TRY(ri::psi_apply(S, S.coef_tmp, nxt, stream));
    RI_TRY(ri::sumsq_f32(nxt, N, S.dsum, stream));
    RI_HIP(hipMemcpyAsync(&sq, S.dsum, sizeof(double), hipMemcpyDeviceToHost, stream));
    RI_HIP(hipStreamSynchronize(stream));
    lam = std::sqrt(sq);
    RI_TRY(ri::scale_by_rsqrt(nxt, N, S.dsum, stream));
    std::swap(cur, nxt);
    if (lam == 0.0 || std::fabs(lam - lam_prev) <= rtol * lam) break;
    lam_prev = lam;
  }
  if (cur != x0) RI_HIP(hipMemcpyAsync(x0, cur, N * sizeof(float), hipMemcpyDeviceToDevice, stream));
  RI_HIP(hipStreamSynchronize(stream));
  *norm_host = std::sqrt(lam);
  if (iters_host) *iters_host = it > max_it ? max_it : it;
  return RI_OK;
}

}  // extern "C"
