// Pruned 2D FFTs of the measurement operator: b~ = F Z S x (Algorithm 1 step 4) and its
// adjoint Re S Z^dagger F^dagger (step 17), on the K x K grid, K = 2n.
//
// Pixel (r, c) has centred coordinates l = (r - n/2, c - n/2) and lands on grid index
// q = l mod K, so only n of the K inputs per axis are nonzero: q in [0, n/2) maps back to
// pixel q + n/2 and q in [K - n/2, K) to pixel q - K + n/2.  The forward transform runs a
// row pass over the n nonzero image rows (K-point FFTs of zero-padded, S-scaled rows) into
// an n x K buffer, then a column pass over all K columns that reads only the n nonzero
// rows and writes the full grid.  The adjoint runs the column pass first, keeping only
// the n output rows that map back to pixels, then a row pass keeping n of K outputs and
// the real part, scaled by S.
#include "fft.hpp"
#include "plan.hpp"
#include "sara_dev.hpp"

namespace ri {

namespace {

__device__ __forceinline__ int pix_of(int q, int n, int K) {
  // grid index -> pixel index, or -1 outside the image support
  return q < n / 2 ? q + n / 2 : (q >= K - n / 2 ? q - K + n / 2 : -1);
}

// Grids of up to 1024 cells take the smallest panels that fill a wavefront with radix-8 jobs (rows)
// or four columns (a 32-byte segment of a row): their passes are as long as one workgroup's
// chain of passes, and more workgroups shorten it: forward columns 9.7 -> 7.6 us at K = 1024 (64
// -> 256 workgroups), 7.0 -> 5.6 at 512 (32 -> 128); the rows keep their 3 to 6 us.
template <int K>
struct RowCfg {
  static constexpr int W = K > WINDOWED_K ? 1 : (K >= 512 ? 1 : (512 / K < K / 2 ? 512 / K : K / 2));
  static constexpr int NT = K == 4096 ? 512 : (K > WINDOWED_K ? 256 : (W * K / 8 < 64 ? 64 : W * K / 8));
};
template <int K>
struct ColCfg {
  static constexpr int W = K <= WINDOWED_K ? 4 : 16384 / K;
  static constexpr int NT = K > WINDOWED_K ? 512 : (W * K / 16 < 64 ? 64 : W * K / 16);
};

// Adjoint column panels of windowed plans.  Up to SIDE_K a sparsity job may ride on the launch
// (KIND), whose workgroup size decides the panel; launches without a job use the same kernel, so
// that both give the same bits (another instance may contract its products differently).
template <int K>
struct WinColCfg {
  static constexpr int KIND = K < SIDE_K ? SIDE_TOP : (K == SIDE_K ? SIDE_IDWT : SIDE_NONE);
  static constexpr int W = K <= SIDE_K ? 8 : 4;
  static constexpr int NT = KIND == SIDE_TOP ? ST * TOP_GROUPS : 256;
  static constexpr int RADIX = K >= 256 ? 16 : 8;
};

// Column panel of workgroup b of nb: consecutive blocks go round-robin to the eight XCDs,
// so neighbouring panels, which share 128-byte rows of the grid, are given to blocks on
// the same XCD (and its L2) when nb is a multiple of 8.
__device__ __forceinline__ int panel_of(int b, int nb) {
  return nb % 8 == 0 ? (b % 8) * (nb / 8) + b / 8 : b;
}

// Twiddles are staged in LDS when the panel and the table fit in 144 KiB together.
template <int K, int W>
struct TwLds {
  static constexpr bool fits = (K * W + K) * 8 <= 144 * 1024;
  static constexpr int size = fits ? K : 1;
};

template <int K, int W, int NT>
__global__ __launch_bounds__(NT) void k_fwd_rows(const float* __restrict__ x, const float* __restrict__ S,
                                                 float2* __restrict__ rows, const float2* __restrict__ tw) {
  constexpr int n = K / 2;
  __shared__ float2 lds[K * W];
  __shared__ float2 twl[TwLds<K, W>::size];
  const int r0 = blockIdx.x * W;
  auto load = [&](int w, int q) -> float2 {
    const int c = pix_of(q, n, K);
    if (c < 0) return make_float2(0.f, 0.f);
    const int r = r0 + w;
    return make_float2(x[size_t(r) * n + c] * (S[r] * S[c]), 0.f);
  };
  auto store = [&](int w, int k, float2 v) { rows[size_t(r0 + w) * K + k] = v; };
  FftPanel<K, W, NT, -1, false>::template run<TwLds<K, W>::fits>(lds, tw, twl, load, store);
}

template <int K, int W, int NT>
__global__ __launch_bounds__(NT) void k_fwd_cols(const float2* __restrict__ rows, float2* __restrict__ grid,
                                                 const float2* __restrict__ tw) {
  constexpr int n = K / 2;
  __shared__ float2 lds[K * W];
  __shared__ float2 twl[TwLds<K, W>::size];
  const int c0 = panel_of(blockIdx.x, gridDim.x) * W;
  auto load = [&](int w, int q) -> float2 {
    const int r = pix_of(q, n, K);
    if (r < 0) return make_float2(0.f, 0.f);
    return rows[size_t(r) * K + c0 + w];
  };
  auto store = [&](int w, int k, float2 v) { grid[size_t(k) * K + c0 + w] = v; };
  FftPanel<K, W, NT, -1, true>::template run<TwLds<K, W>::fits>(lds, tw, twl, load, store);
}

template <int K, int W, int NT>
__global__ __launch_bounds__(NT) void k_adj_cols(const float2* __restrict__ grid, float2* __restrict__ rows,
                                                 const float2* __restrict__ tw) {
  constexpr int n = K / 2;
  __shared__ float2 lds[K * W];
  __shared__ float2 twl[TwLds<K, W>::size];
  const int c0 = panel_of(blockIdx.x, gridDim.x) * W;
  auto load = [&](int w, int k) -> float2 { return grid[size_t(k) * K + c0 + w]; };
  // the data branch's kernels issue ahead of the sparsity branch's waves sharing their SIMDs
  __builtin_amdgcn_s_setprio(3);
  auto store = [&](int w, int q, float2 v) {
    const int r = pix_of(q, n, K);
    if (r >= 0) rows[size_t(r) * K + c0 + w] = v;
  };
  FftPanel<K, W, NT, +1, true>::template run<TwLds<K, W>::fits>(lds, tw, twl, load, store);
}

// The adjoint column pass of a windowed plan, whose grid comes as the gridding tiles' patches:
// stored column s holds grid column s - 3 (mod K), so that tile tx's region starts at stored
// column GSIDE tx, and stored row likewise; a cell in the first 7 rows or columns of its tile
// also lies in the reach of the tile above, to the left, or both.  All four are loaded for every
// cell, the absent ones from a cell of the own patch that is always zero: loads under a branch
// would be waited for one after the other (36 us at K = 1024, against 9.8 so; the pass over a
// merged grid took 9.2, and the halo pass before it 7.0).
constexpr int REACH = KB_J - 1;
constexpr int SHIFT = KB_J / 2 - 1;

// KIND: the workgroups after the K / W panels' are those of a sparsity job.
template <int K, int W, int NT, int KIND>
__global__ __launch_bounds__(NT) void k_adj_cols_win(const float2* __restrict__ patch, float2* __restrict__ rows,
                                                     const float2* __restrict__ tw, SideJob side) {
  constexpr int n = K / 2, TA = K / GSIDE;
  constexpr int OWN = (K * W + TwLds<K, W>::size) * int(sizeof(float2)), JOB = KIND != SIDE_NONE ? side_smem<NT>() : 0;
  __shared__ __align__(16) char smem[OWN > JOB ? OWN : JOB];
  if constexpr (KIND != SIDE_NONE) {
    if (blockIdx.x >= K / W) {
      side_body<NT, KIND>(side, int(blockIdx.x) - K / W, smem);
      return;
    }
  }
  float2* lds = reinterpret_cast<float2*>(smem);
  float2* twl = lds + K * W;
  const int c0 = panel_of(blockIdx.x, K / W) * W;
  // the data branch's kernels issue ahead of the sparsity branch's waves sharing their SIMDs
  __builtin_amdgcn_s_setprio(3);
  auto load = [&](int w, int k) -> float2 {
    const int s = c0 + w, sy = (k + SHIFT) & (K - 1);
    const int tx = s / GSIDE, lx = s % GSIDE, ty = sy / GSIDE, ly = sy % GSIDE;
    const int tl = (tx - 1) & (TA - 1), tu = (ty - 1) & (TA - 1);
    const int o = ly * PATCH_W + lx, own = (ty * TA + tx) * PATCH_CELLS, zero = own + PATCH_CELLS - 1;
    const bool left = lx < REACH, up = ly < REACH;
    const float2 a = patch[own + o];
    const float2 b = patch[left ? (ty * TA + tl) * PATCH_CELLS + o + GSIDE : zero];
    const float2 c = patch[up ? (tu * TA + tx) * PATCH_CELLS + o + GSIDE * PATCH_W : zero];
    const float2 d = patch[left && up ? (tu * TA + tl) * PATCH_CELLS + o + GSIDE * PATCH_W + GSIDE : zero];
    return cadd(cadd(a, b), cadd(c, d));
  };
  auto store = [&](int w, int q, float2 v) {
    const int r = pix_of(q, n, K);
    if (r >= 0) rows[size_t(r) * K + ((c0 + w - SHIFT) & (K - 1))] = v;
  };
  FftPanel<K, W, NT, +1, true, WinColCfg<K>::RADIX>::template run<TwLds<K, W>::fits>(lds, tw, twl, load, store);
}

// UPD: the output g = Re S (...) feeds steps 17-18 (PrimalUpdate) instead of being stored.
template <int K, int W, int NT, bool UPD>
__global__ __launch_bounds__(NT) void k_adj_rows(const float2* __restrict__ rows, const float* __restrict__ S,
                                                 float* __restrict__ x, const float2* __restrict__ tw,
                                                 PrimalUpdate u, int add) {
  constexpr int n = K / 2;
  __shared__ float2 lds[K * W];
  __shared__ float2 twl[TwLds<K, W>::size];
  const int r0 = blockIdx.x * W;
  // With one row per workgroup, K / 8 threads and a radix-8 last pass, thread t stores the
  // outputs t + i K / 8, i < 8, of which i = 0, 1, 6, 7 are pixels: their x and s~ are
  // loaded before the transform, so the update does not wait for them at the end.
  constexpr bool PREF = UPD && W == 1 && NT == K / 8 && FftPanel<K, W, NT, +1, false>::RB == 8;
  float xp[4] = {0.f, 0.f, 0.f, 0.f}, sp[4] = {0.f, 0.f, 0.f, 0.f};
  if constexpr (PREF) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = threadIdx.x + (i < 2 ? i : i + 4) * (K / 8);
      const size_t o = size_t(r0) * n + pix_of(q, n, K);
      xp[i] = u.x[o];
      sp[i] = u.st[o];
    }
  }
  auto load = [&](int w, int k) -> float2 { return rows[size_t(r0 + w) * K + k]; };
  auto store = [&](int w, int q, float2 v) {
    const int c = pix_of(q, n, K);
    if (c >= 0) {
      const int r = r0 + w;
      const size_t o = size_t(r) * n + c;
      const float g = v.x * (S[r] * S[c]);
      if (UPD) {
        float xo, so;
        if constexpr (PREF) {
          const int i = q < K / 8 ? 0 : (q < K / 4 ? 1 : (q < 7 * K / 8 ? 2 : 3));
          xo = i == 0 ? xp[0] : (i == 1 ? xp[1] : (i == 2 ? xp[2] : xp[3]));
          so = i == 0 ? sp[0] : (i == 1 ? sp[1] : (i == 2 ? sp[2] : sp[3]));
        } else {
          xo = u.x[o];
          so = u.st[o];
        }
        float gr;
        if constexpr (K <= WINDOWED_K) gr = fmaf(u.varsigma, g, fmaf(u.varsigma_lo, g, u.sigma * so));
        else gr = u.sigma * so + u.varsigma * g;
        const float xn = fmaxf(0.f, xo - u.tau * gr);
        u.x[o] = xn;
        u.xt[o] = 2.f * xn - xo;
      } else {
        x[o] = add != 0 ? x[o] + g : g;
      }
    }
  };
  FftPanel<K, W, NT, +1, false>::template run<TwLds<K, W>::fits>(lds, tw, twl, load, store);
}

template <int K>
int fwd_rows_impl(const Plan& p, const float* x, float2*, hipStream_t s) {
  using RC = RowCfg<K>;
  hipLaunchKernelGGL((k_fwd_rows<K, RC::W, RC::NT>), dim3(K / 2 / RC::W), dim3(RC::NT), 0, s, x, p.scale,
                     p.rowbuf, p.twiddle);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

template <int K>
int fwd_cols_impl(const Plan& p, const float*, float2* grid, hipStream_t s) {
  using CC = ColCfg<K>;
  hipLaunchKernelGGL((k_fwd_cols<K, CC::W, CC::NT>), dim3(K / CC::W), dim3(CC::NT), 0, s, p.rowbuf, grid,
                     p.twiddle);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

template <int K>
int adj_cols_impl(const Plan& p, const float2* grid, const SideJob* side, hipStream_t s) {
  const int jobs = side != nullptr ? side->wgs : 0;
  if (jobs > 0 && K > SIDE_K) return fail(RI_EINVAL, "adjoint column pass: no side job at K=%d", K);
  if constexpr (K <= WINDOWED_K) {
    using WC = WinColCfg<K>;
    hipLaunchKernelGGL((k_adj_cols_win<K, WC::W, WC::NT, WC::KIND>), dim3(K / WC::W + jobs), dim3(WC::NT), 0, s, grid,
                       p.rowbuf, p.twiddle, jobs > 0 ? *side : SideJob{});
  } else {
    using CC = ColCfg<K>;
    hipLaunchKernelGGL((k_adj_cols<K, CC::W, CC::NT>), dim3(K / CC::W), dim3(CC::NT), 0, s, grid, p.rowbuf,
                       p.twiddle);
  }
  RI_LAUNCH_CHECK();
  return RI_OK;
}

template <int K>
int adj_rows_impl(const Plan& p, bool add, float* x, hipStream_t s) {
  using RC = RowCfg<K>;
  hipLaunchKernelGGL((k_adj_rows<K, RC::W, RC::NT, false>), dim3(K / 2 / RC::W), dim3(RC::NT), 0, s, p.rowbuf,
                     p.scale, x, p.twiddle, PrimalUpdate{}, add ? 1 : 0);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

template <int K>
int adj_rows_update_impl(const Plan& p, const PrimalUpdate& u, hipStream_t s) {
  using RC = RowCfg<K>;
  hipLaunchKernelGGL((k_adj_rows<K, RC::W, RC::NT, true>), dim3(K / 2 / RC::W), dim3(RC::NT), 0, s, p.rowbuf,
                     p.scale, nullptr, p.twiddle, u, 0);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

}  // namespace

#define RI_FFT_DISPATCH(FN, ...)                                          \
  switch (p.K) {                                                          \
    case 32: return FN<32>(__VA_ARGS__);                                  \
    case 64: return FN<64>(__VA_ARGS__);                                  \
    case 128: return FN<128>(__VA_ARGS__);                                \
    case 256: return FN<256>(__VA_ARGS__);                                \
    case 512: return FN<512>(__VA_ARGS__);                                \
    case 1024: return FN<1024>(__VA_ARGS__);                              \
    case 2048: return FN<2048>(__VA_ARGS__);                              \
    case 4096: return FN<4096>(__VA_ARGS__);                              \
    default: return fail(RI_EINVAL, "unsupported FFT size K=%d", p.K);    \
  }

int fft_forward_rows(const Plan& p, const float* x, hipStream_t s) {
  RI_FFT_DISPATCH(fwd_rows_impl, p, x, nullptr, s)
}

int fft_forward_cols(const Plan& p, float2* grid, hipStream_t s) {
  RI_FFT_DISPATCH(fwd_cols_impl, p, nullptr, grid, s)
}

int fft_adjoint_cols(const Plan& p, const float2* grid, hipStream_t s, const SideJob* side) {
  RI_FFT_DISPATCH(adj_cols_impl, p, grid, side, s)
}

int fft_adjoint_rows(const Plan& p, float* x, hipStream_t s, bool add) {
  RI_FFT_DISPATCH(adj_rows_impl, p, add, x, s)
}

int fft_adjoint_rows_update(const Plan& p, const PrimalUpdate& u, hipStream_t s) {
  RI_FFT_DISPATCH(adj_rows_update_impl, p, u, s)
}

int fft_forward(const Plan& p, const float* x, float2* grid, hipStream_t s) {
  RI_TRY(fft_forward_rows(p, x, s));
  return fft_forward_cols(p, grid, s);
}

int fft_adjoint(const Plan& p, const float2* grid, float* x, hipStream_t s) {
  RI_TRY(fft_adjoint_cols(p, grid, s));
  return fft_adjoint_rows(p, x, s);
}

}  // namespace ri
