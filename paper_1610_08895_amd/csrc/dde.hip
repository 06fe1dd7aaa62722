// Direction-dependent effects in the interpolation G (Eq. 1's D(l, u), folded into G's
// kernels as Sec. II describes): the DDE of visibility m is band limited on the
// oversampled grid, D_m(l) = sum_{p,q} d_m[q, p] exp(-2 pi i (p l_x + q l_y) / K), so its
// row of G is the jd x jd kernel d_m convolved with the Kaiser-Bessel kernel (the plain
// kernel at a frequency shifted by (p, q) whole cells is the same 8 weights on shifted
// cells):
//
//   W_m[ty][tx] = sum_{p,q} d_m[q, p] w_y[ty - h - q] w_x[tx - h - p],   0 <= tx, ty < S,
//
// on the S = J + 2h cells per axis starting at floor(kappa) - J/2 + 1 - h.  The S^2 weights are
// never stored: streaming them bound both directions to HBM (1152 bytes per visibility at
// S = 12), while the 25 taps they come from are 200 bytes, and the sum over p, q and the kernel's
// taps separates into about 1500 multiply-adds, 91 cycles of a SIMD.  The taps are stored
// tap-major, d[t * M + m], so the 64 lanes of a wavefront, which take 64 consecutive visibilities,
// read 512 contiguous bytes per tap, and by visibility for the adjoint, whose lanes are spread.  300007 visibilities, 512^2 image, jd = 5, 16 blocks: G 131 us
// with stored weights, 30 without (13 of multiply-adds); its adjoint 148 and 37 us (15 of
// multiply-adds, about as much of LDS atomics), merging the patches 19 and 16 us.
//
// Degridding stages a tile plus the kernel's reach in LDS, as the plain kernel does, and forms
// y_m = sum_{q,p} d_m[q, p] (sum of the kernel's taps shifted by (q, p)).  Gridding (the
// adjoint, conjugate weights) is owner-computes per unit of a tile's items: one workgroup
// accumulates a group of about GROUP_VIS visibilities at a time exactly in fixed point with
// 64-bit LDS integer atomics (a power-of-two scale from the largest sum of max_t |W_m| |v_m|
// over the visibilities m in reach of one cell), and writes the tile's whole region (tile plus
// reach) to the unit's patch; a merge pass then adds, for every grid cell, the patches of the up
// to four tiles whose regions cover it, in a fixed order.  Results are deterministic.
#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "handles.hpp"

namespace ri {
namespace {

constexpr int DT = 256;                 // threads per workgroup
constexpr int DNV = MAX_BIN / DT;       // visibilities per thread per item (degridding)
constexpr int MAX_H = 3;                // jd <= 7
constexpr int GROUP_VIS = 512;           // visibilities that share one scale (one item may be larger)
constexpr int GRID_UNIT_VIS = 512;      // visibilities of a gridding unit, if M is not larger than 2^19

template <int T, int H>
struct DdeGeom {
  static constexpr int S = KB_J + 2 * H;      // taps per axis
  static constexpr int R0 = KB_J / 2 - 1 + H;  // reach before the tile
  static constexpr int TW = T + S - 1;         // region: tile plus reach
  static constexpr int TP = TW + 1;            // LDS pitch
  // bins of BC x BC of the tile's cells: a region cell is in reach of visibilities of at most
  // BW x BW adjacent bins
  static constexpr int BC = 4, NB = T / BC;
  static constexpr int BW = (S + BC - 2) / BC + 1 < NB ? (S + BC - 2) / BC + 1 : NB;
};

// The tap polynomials' row ty of W for taps d (any factor included): e[p] = sum_q w_y[ty - q] d[q][p],
// then row[tx] = init + sum_p w_x[tx - p] e[p].  ty is a constant where this is unrolled.
template <int H>
__device__ __forceinline__ void weight_row(int ty, const float* wx, const float* wy, const float2* d, float init,
                                           float2* row) {
  constexpr int JD = 2 * H + 1, S = KB_J + 2 * H;
#pragma unroll
  for (int tx = 0; tx < S; ++tx) row[tx] = make_float2(init, init);
#pragma unroll
  for (int p = 0; p < JD; ++p) {
    float2 e = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < JD; ++q) {
      if (ty - q < 0 || ty - q >= KB_J) continue;
      e.x = fmaf(wy[ty - q], d[q * JD + p].x, e.x);
      e.y = fmaf(wy[ty - q], d[q * JD + p].y, e.y);
    }
#pragma unroll
    for (int j = 0; j < KB_J; ++j) {
      row[j + p].x = fmaf(wx[j], e.x, row[j + p].x);
      row[j + p].y = fmaf(wx[j], e.y, row[j + p].y);
    }
  }
}

// An upper bound of |z|, at most 8.3 % above it.
__device__ __forceinline__ float modulus_bound(float2 z) {
  const float a = fabsf(z.x), b = fabsf(z.y);
  return fmaf(0.41421357f, fminf(a, b), fmaxf(a, b));
}

// One thread per visibility: its taps into tap-major order, and the bound of its weights,
// max over the taps of |W|.
template <int H>
__global__ __launch_bounds__(DT) void k_dde_taps(int64_t M, const uint2* __restrict__ coord,
                                                 const float2* __restrict__ in, KBPoly P, float2* __restrict__ taps,
                                                 float* __restrict__ wmax) {
  constexpr int JD = 2 * H + 1, S = KB_J + 2 * H;
  for (int64_t m = blockIdx.x * int64_t(DT) + threadIdx.x; m < M; m += int64_t(gridDim.x) * DT) {
    float wx[KB_J], wy[KB_J];
    int cx, cy;
    kb_weights(coord[m].x, P, wx, cx);
    kb_weights(coord[m].y, P, wy, cy);
    float2 d[JD * JD];
#pragma unroll
    for (int t = 0; t < JD * JD; ++t) {
      d[t] = in[m * (JD * JD) + t];
      taps[size_t(t) * M + m] = d[t];
    }
    float mx = 0.f;
#pragma unroll
    for (int ty = 0; ty < S; ++ty) {
      float2 row[S];
      weight_row<H>(ty, wx, wy, d, 0.f, row);
#pragma unroll
      for (int tx = 0; tx < S; ++tx) mx = fmaxf(mx, modulus_bound(row[tx]));
    }
    wmax[m] = mx;
  }
}

enum { DD_APPLY = 0, DD_RESIDUAL = 1 };

// Degridding over units {tile, first, end} of items; MODE as k_degrid in gridding.hip
// (residual: r = v + G b - y into out and FP64 partial norms of r and of G b - y per wavefront).
template <int T, int H, int MODE>
__global__ __launch_bounds__(DT) void k_degrid_dde(const int4* __restrict__ units, int nunits,
                                                   const Item* __restrict__ items, const uint8_t* __restrict__ mask,
                                                   const uint2* __restrict__ coord, const float2* __restrict__ taps,
                                                   int64_t M, KBPoly P, const float2* __restrict__ grid, int K, int tpa,
                                                   float2* __restrict__ out, const float2* __restrict__ y,
                                                   const float2* __restrict__ v, double* __restrict__ part) {
  using G = DdeGeom<T, H>;
  constexpr int S = G::S, TW = G::TW, TP = G::TP, R0 = G::R0, JD = 2 * H + 1;
  constexpr int NWV = DT / 64;
  __shared__ float2 tile[TW * TP];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int u = blockIdx.x; u < nunits; u += gridDim.x) {
    const int4 un = units[u];
    bool any = mask == nullptr && un.y < un.z;  // empty units fill gaps of the XCD order
    for (int q = un.y; q < un.z && !any; ++q) any = mask[items[q].x] != 0;
    if (!any) continue;
    const int ty = un.x / tpa, tx = un.x - (un.x / tpa) * tpa;
    const int gy0 = ty * T - R0, gx0 = tx * T - R0;
    for (int idx = threadIdx.x; idx < TW * TW; idx += DT) {
      const int ly = idx / TW, lx = idx - ly * TW;
      tile[ly * TP + lx] = grid[size_t((gy0 + ly) & (K - 1)) * K + ((gx0 + lx) & (K - 1))];
    }
    __syncthreads();
    for (int q = un.y; q < un.z; ++q) {
      const Item it = items[q];
      if (mask != nullptr && mask[it.x] == 0) continue;
      double sr = 0.0, se = 0.0;
      const int rw = (wv + q) & (NWV - 1);  // items are often short: their first wavefronts rotate
      for (int k = 0; k < DNV; ++k) {
        const int s = rw * 64 + lane + k * DT;
        if (s >= it.w) break;
        const int64_t m = it.z + s;
        const uint2 c = coord[m];
        float wx[KB_J], wy[KB_J];
        int cx, cy;
        kb_weights(c.x, P, wx, cx);
        kb_weights(c.y, P, wy, cy);
        // region row / column of the first tap: cell - 3 - h - (tile origin - R0)
        const float2* base = &tile[(cy - ty * T) * TP + (cx - tx * T)];
        // vs[q][p]: the kernel's sum at shift (q, p)
        float2 vs[JD][JD];
#pragma unroll
        for (int q = 0; q < JD; ++q)
#pragma unroll
          for (int p = 0; p < JD; ++p) vs[q][p] = make_float2(0.f, 0.f);
#pragma unroll
        for (int a = 0; a < S; ++a) {
          float2 row[S];
#pragma unroll
          for (int b = 0; b < S; ++b) row[b] = base[a * TP + b];
#pragma unroll
          for (int p = 0; p < JD; ++p) {
            float2 t = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < KB_J; ++j) {
              t.x = fmaf(wx[j], row[j + p].x, t.x);
              t.y = fmaf(wx[j], row[j + p].y, t.y);
            }
#pragma unroll
            for (int q = 0; q < JD; ++q) {
              if (a - q < 0 || a - q >= KB_J) continue;
              vs[q][p].x = fmaf(wy[a - q], t.x, vs[q][p].x);
              vs[q][p].y = fmaf(wy[a - q], t.y, vs[q][p].y);
            }
          }
        }
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int q = 0; q < JD; ++q)
#pragma unroll
          for (int p = 0; p < JD; ++p) {
            const float2 d = taps[size_t(q * JD + p) * M + m];
            acc.x = fmaf(d.x, vs[q][p].x, fmaf(-d.y, vs[q][p].y, acc.x));
            acc.y = fmaf(d.x, vs[q][p].y, fmaf(d.y, vs[q][p].x, acc.y));
          }
        if (MODE == DD_APPLY) {
          out[m] = acc;
        } else {
          const float2 yy = y[m], vv = v[m];
          const float2 e = make_float2(acc.x - yy.x, acc.y - yy.y);
          const float2 r = make_float2(vv.x + e.x, vv.y + e.y);
          if (out != nullptr) out[m] = r;
          sr += double(r.x) * r.x + double(r.y) * r.y;
          se += double(e.x) * e.x + double(e.y) * e.y;
        }
      }
      if (MODE == DD_RESIDUAL) {
        sr = wave_sum(sr);
        se = wave_sum(se);
        if (lane == 0) {
          part[(size_t(it.y) * NWV + rw) * 2] = sr;
          part[(size_t(it.y) * NWV + rw) * 2 + 1] = se;
        }
      }
    }
    __syncthreads();
  }
}

// N taps of one visibility, two to a load (8-byte alignment).
template <int N>
__device__ __forceinline__ void load_taps(const float2* __restrict__ p, float2* d) {
  typedef float tap2 __attribute__((ext_vector_type(4), aligned(8)));
#pragma unroll
  for (int t = 0; t + 1 < N; t += 2) {
    const tap2 q = *reinterpret_cast<const tap2*>(p + t);
    d[t] = make_float2(q.x, q.y);
    d[t + 1] = make_float2(q.z, q.w);
  }
  d[N - 1] = p[N - 1];
}

// Gridding with conjugate DDE weights over units of one tile's items {tile, first, end, patch}.
// PROJECT: the values are the step-8 dual changes (v_new = r shrink_i stored, v_new - v_old
// gridded), else y.  The tile's region goes to the unit's patch (stored), or is added to the tile's
// (ADDP; each tile then has one unit).  A unit is taken in groups of items of together at most
// GROUP_VIS visibilities (or one item of up to MAX_BIN): the wavefronts take the active items in
// turn, list their visibilities without gaps, and sum the fixed-point bound; the group's threads
// then take the list.  An item at a time, as a block's part of a tile comes, left most of a
// workgroup idle (blocks cut a tile into pieces of a few dozen visibilities): 160 us, at 300007
// visibilities and jd = 5, against 73 in list order and 49 with a wavefront's lanes spread over the
// list; 41 with room for all taps of a visibility in registers at once, 37 with the taps read by
// visibility: tap-major, the spread lanes fetched each line of taps up to 16 times (at 2^22
// visibilities, 1024^2 and jd = 5, 810 us, by visibility 512). 128 registers hold the taps up to jd
// = 5, and four wavefronts per SIMD: with three, the per-block form, whose workgroups are short and
// many, waits for slots (64 blocks over the whole plane, 200000 visibilities at 512^2: 560 us, now
// 398), and 2^21 visibilities take 268 us instead of 246.
// The scale: a group's items come from many blocks, and the sum of all its bounds, which no cell
// reaches, left few bits to each (2^21 visibilities in 64 blocks at 1024^2, error of Phi^dagger
// 2.3e-6; 4.6e-7 with the bounds summed by bins of 4 x 4 cells and groups of 512, 5.2e-7 with 1024;
// each item by itself, which has a scale of its own, 4.8e-7).  The bins cost 39 -> 41 us at 300007
// visibilities, and with the smaller groups 217 -> 246 at 2^21.
template <int T, int H, bool PROJECT, bool ADDP>
__global__ __launch_bounds__(DT, H <= 2 ? 4 : 2) void k_grid_dde(const int4* __restrict__ units, int nunits,
                                                 const Item* __restrict__ items, const uint8_t* __restrict__ mask,
                                                 const uint2* __restrict__ coord, const float2* __restrict__ vtaps,
                                                 const float* __restrict__ wmax, KBPoly P,
                                                 const float2* __restrict__ y, const float2* __restrict__ e,
                                                 float2* __restrict__ v, const float* __restrict__ shrink,
                                                 float2* __restrict__ patch, int tpa) {
  using G = DdeGeom<T, H>;
  constexpr int S = G::S, TW = G::TW, TP = G::TP, JD = 2 * H + 1, NB = G::NB, BW = G::BW, PB = NB - BW + 1;
  constexpr int NWV = DT / 64;
  static_assert(NB * NB <= DT, "one thread per bin, and a bin in a byte");
  __shared__ unsigned long long acci[TW * TP];
  __shared__ float2 val[MAX_BIN];
  __shared__ int vis[MAX_BIN];
  __shared__ float amp[MAX_BIN];          // the bound of each visibility's contributions
  __shared__ unsigned char bin[MAX_BIN];  // its bin
  __shared__ unsigned bsum[NB * NB];      // the bins' sums of the bounds, in units of 2^-24 of their total
  __shared__ float red[NWV];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int k = threadIdx.x; k < TW * TP; k += DT) acci[k] = 0ull;
  if (threadIdx.x < NB * NB) bsum[threadIdx.x] = 0u;
  for (int u = blockIdx.x; u < nunits; u += gridDim.x) {
    const int4 un = units[u];
    const int ty = un.x / tpa, tx = un.x - (un.x / tpa) * tpa;
    float2* pt = patch + size_t(ADDP ? un.x : un.w) * TW * TW;
    bool first = !ADDP;
    for (int q = un.y; q < un.z || first;) {
      // list the group's visibilities; every wavefront scans the items' widths
      int cnt = 0;
      float babs = 0.f;
      for (bool full = false; q < un.z && !full;) {
        const int have = min(64, un.z - q);
        Item it{};
        int w = 0;
        if (lane < have) {
          it = items[q + lane];
          w = mask == nullptr || mask[it.x] != 0 ? it.w : 0;
        }
        int end = w;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int t = __shfl_up(end, o);
          if (lane >= o) end += t;
        }
        const int fit = __popcll(__ballot(lane < have && (cnt + end <= GROUP_VIS || cnt + end == w)));
        full = fit < have;
        for (int i = wv; i < fit; i += NWV) {
          const int iw = __shfl(w, i), im = __shfl(it.z, i), s0 = cnt + __shfl(end, i) - iw;
          const float sh = PROJECT && iw > 0 ? shrink[__shfl(it.x, i)] : 0.f;
#pragma unroll 1
          for (int s = lane; s < iw; s += 64) {
            const int64_t m = im + s;
            float2 x;
            if (PROJECT) {
              const float2 vo = v[m], rr = e[m];  // r = v_old + G b - y from the degridding
              const float2 vn = make_float2(rr.x * sh, rr.y * sh);
              v[m] = vn;
              x = make_float2(vn.x - vo.x, vn.y - vo.y);
            } else {
              x = y[m];
            }
            const uint2 c = coord[m];
            const float a = wmax[m] * modulus_bound(x);
            val[s0 + s] = x;
            vis[s0 + s] = int(m);
            amp[s0 + s] = a;
            const int by = (int(c.y >> FRAC_BITS) - ty * T) / G::BC, bx = (int(c.x >> FRAC_BITS) - tx * T) / G::BC;
            bin[s0 + s] = static_cast<unsigned char>(by * NB + bx);
            babs += a;
          }
        }
        if (fit > 0) cnt += __shfl(end, fit - 1);
        q += fit;
      }
      babs = wave_sum(babs);
      if (lane == 0) red[wv] = babs;
      __syncthreads();
      float bound = 0.f;
#pragma unroll
      for (int k = 0; k < NWV; ++k) bound += red[k];
      float inv = 0.f;
      if (bound > 0.f) {
        // the largest sum of the bounds in reach of one cell (whole numbers: the same in any order)
        const float unit = bound * (1.f / 16777216.f), per = 1.f / unit;
        for (int s = threadIdx.x; s < cnt; s += DT) atomicAdd(&bsum[bin[s]], unsigned(amp[s] * per) + 1u);
        __syncthreads();
        unsigned most = 0;
        for (int p = lane; p < PB * PB; p += 64) {
          unsigned t = 0;
#pragma unroll
          for (int i = 0; i < BW; ++i)
#pragma unroll
            for (int j = 0; j < BW; ++j) t += bsum[(p / PB + i) * NB + p % PB + j];
          most = max(most, t);
        }
        // 2^E with reach * 2^E < 2^31: no cell's sum of either part can leave 32 bits (the factor guards
        // the bounds' own rounding and that of up to MAX_BIN contributions)
        const float reach = wave_max(float(most)) * unit;
        int ex = 0;
        frexpf(reach * 1.0001f, &ex);
        const int e2 = min(31 - ex, 126);  // (both powers are normal numbers)
        const float scale = ldexpf(1.f, e2);
        inv = ldexpf(1.f, -e2);
        // neighbours in the list share cells, which one instruction's atomics would take in turn: a
        // wavefront's lanes take visibilities `nw` apart
        const int nw = (cnt + 63) / 64;
#pragma unroll 1
        for (int w = wv; w < nw; w += NWV) {
          const int s = lane * nw + w;
          if (s >= cnt) continue;
          const int64_t m = vis[s];
          const float vr = val[s].x * scale, vi = val[s].y * scale;
          const uint2 c = coord[m];
          float2 d[JD * JD];  // conj(d) v
          load_taps<JD * JD>(vtaps + m * (JD * JD), d);
#pragma unroll
          for (int t = 0; t < JD * JD; ++t) {
            const float2 g = d[t];
            d[t] = make_float2(fmaf(g.x, vr, g.y * vi), fmaf(g.x, vi, -g.y * vr));
          }
          float wx[KB_J], wy[KB_J];
          int cx, cy;
          kb_weights(c.x, P, wx, cx);
          kb_weights(c.y, P, wy, cy);
          unsigned long long* base = &acci[(cy - ty * T) * TP + (cx - tx * T)];
#pragma unroll
          for (int a = 0; a < S; ++a) {
            float2 row[S];
            weight_row<H>(a, wx, wy, d, 0.5f, row);
#pragma unroll
            for (int b = 0; b < S; ++b) {  // rounded to nearest
              const int ir = static_cast<int>(floorf(row[b].x)), ii = static_cast<int>(floorf(row[b].y));
              const unsigned hi = unsigned(ii) + unsigned(ir >> 31);
              atomicAdd(base + a * TP + b, (static_cast<unsigned long long>(hi) << 32) | unsigned(ir));
            }
          }
        }
      }
      __syncthreads();
      if (threadIdx.x < NB * NB) bsum[threadIdx.x] = 0u;
      if (first || bound > 0.f) {
#pragma unroll 2
        for (int c = threadIdx.x; c < TW * TW; c += DT) {
          unsigned long long* cell = &acci[c + c / TW];
          const unsigned long long w64 = *cell;
          float2 x = make_float2(0.f, 0.f);
          if (w64) {
            *cell = 0ull;
            const int ir = static_cast<int>(static_cast<unsigned>(w64));
            const int ii = static_cast<int>(static_cast<unsigned>(
                (w64 - static_cast<unsigned long long>(static_cast<long long>(ir))) >> 32));
            x = make_float2(float(ir) * inv, float(ii) * inv);
          }
          if (first) {
            pt[c] = x;
          } else if (w64) {
            const float2 o = pt[c];
            pt[c] = make_float2(o.x + x.x, o.y + x.y);
          }
        }
      }
      first = false;
    }
  }
}

// The sum of the patches that cover cell (iy, ix) of tile (ty, tx): its own, and in each axis at
// most one neighbour's (above or to the left of the near edge, below or to the right of the far
// one).  All four are loaded, the absent ones from the own patch and dropped, so that no load
// waits for another.  more: the further patches of tile t are [more[t], more[t + 1]) (NULL: none).
template <int T, int H>
__device__ __forceinline__ float2 covering(const float2* __restrict__ patch, const int* __restrict__ more, int tpa,
                                           int ty, int tx, int iy, int ix) {
  using G = DdeGeom<T, H>;
  constexpr int TW = G::TW, R0 = G::R0, NEAR = TW - T - R0, FAR = T - R0;
  static_assert(NEAR <= FAR, "one neighbour per axis");
  const int dy = iy < NEAR ? -1 : (iy >= FAR ? 1 : 0), dx = ix < NEAR ? -1 : (ix >= FAR ? 1 : 0);
  const int ny = (ty + dy + tpa) & (tpa - 1), nx = (tx + dx + tpa) & (tpa - 1);
  const int oy = iy + R0, ox = ix + R0;
  const int t[4] = {ty * tpa + tx, ty * tpa + nx, ny * tpa + tx, ny * tpa + nx};
  const int o[4] = {oy * TW + ox, oy * TW + ox - dx * T, (oy - dy * T) * TW + ox, (oy - dy * T) * TW + ox - dx * T};
  const bool on[4] = {true, dx != 0, dy != 0, dx != 0 && dy != 0};
  float2 a[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) a[k] = patch[size_t(on[k] ? t[k] : t[0]) * TW * TW + (on[k] ? o[k] : o[0])];
  if (more != nullptr) {
    int f[4], n[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[k] = more[t[k]];
      n[k] = on[k] ? more[t[k] + 1] - f[k] : 0;
    }
    const int most = max(max(n[0], n[1]), max(n[2], n[3]));
    for (int j = 0; j < most; ++j) {
      float2 x[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = patch[size_t(j < n[k] ? f[k] + j : t[k]) * TW * TW + (on[k] ? o[k] : o[0])];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (j < n[k]) a[k] = cadd(a[k], x[k]);
    }
  }
  float2 s = a[0];
#pragma unroll
  for (int k = 1; k < 4; ++k)
    if (on[k]) s = cadd(s, a[k]);
  return s;
}

// grid cell (=, or += with ADD) the sum of the patches of the tiles whose regions cover
// it, neighbours in a fixed order; one workgroup per tile.
template <int T, int H, bool ADD>
__global__ __launch_bounds__(DT) void k_dde_merge(float2* __restrict__ grid, const float2* __restrict__ patch,
                                                  const int* __restrict__ more, int K, int tpa) {
  const int t = blockIdx.x;
  const int ty = t / tpa, tx = t - (t / tpa) * tpa;
  for (int k = threadIdx.x; k < T * T; k += DT) {
    const int iy = k / T, ix = k - (k / T) * T;
    const float2 acc = covering<T, H>(patch, more, tpa, ty, tx, iy, ix);
    float2* g = &grid[size_t(ty * T + iy) * K + tx * T + ix];
    if (!ADD) {
      *g = acc;
    } else if (acc.x != 0.f || acc.y != 0.f) {
      const float2 o = *g;
      *g = make_float2(o.x + acc.x, o.y + acc.y);
    }
  }
}

// The sum of the DDE tiles' patches covering each cell of a gridding tile (neighbours in a fixed
// order) into that tile's own cells of the patch array (=, or += with ADD); without ADD the
// rest of its slot, where the plain kernel stores its reach, becomes zero.  One workgroup per
// gridding tile.
template <int T, int H, bool ADD>
__global__ __launch_bounds__(DT) void k_dde_merge_win(float2* __restrict__ sum, const float2* __restrict__ patch,
                                                      const int* __restrict__ more, int K, int tpa, int gta) {
  const int gty = blockIdx.x / gta, gtx = blockIdx.x - (blockIdx.x / gta) * gta;
  float2* out = sum + size_t(blockIdx.x) * PATCH_CELLS;
  if (!ADD)
    for (int k = threadIdx.x; k < PATCH_CELLS; k += DT)
      if (k / PATCH_W >= GSIDE || k % PATCH_W >= GSIDE) out[k] = make_float2(0.f, 0.f);
  for (int i = threadIdx.x; i < GSIDE * GSIDE; i += DT) {
    const int R = i / GSIDE, C = i % GSIDE, k = R * PATCH_W + C;
    const int gy = (gty * GSIDE - (KB_J / 2 - 1) + R) & (K - 1), gx = (gtx * GSIDE - (KB_J / 2 - 1) + C) & (K - 1);
    const int ty = gy / T, iy = gy % T, tx = gx / T, ix = gx % T;
    const float2 acc = covering<T, H>(patch, more, tpa, ty, tx, iy, ix);
    if (!ADD) {
      out[k] = acc;
    } else if (acc.x != 0.f || acc.y != 0.f) {
      const float2 o = out[k];
      out[k] = make_float2(o.x + acc.x, o.y + acc.y);
    }
  }
}

int wgs(const Plan& p, int units) {
  const int g = p.persistent_wgs > 0 ? p.persistent_wgs : units;
  return units < g ? (units > 0 ? units : 1) : g;
}

// Calls F.template operator()<T, H>() for the plan's tile and DDE half-width.
template <class F>
int dispatch(const Plan& p, F&& f) {
#define RI_DDE_H(TT)                                                 \
  switch (p.dde.h) {                                                 \
    case 0: return f.template operator()<TT, 0>();                   \
    case 1: return f.template operator()<TT, 1>();                   \
    case 2: return f.template operator()<TT, 2>();                   \
    case 3: return f.template operator()<TT, 3>();                   \
    default: return fail(RI_EINVAL, "unsupported DDE half-width %d", p.dde.h); \
  }
  switch (p.tile) {
    case 16: RI_DDE_H(16)
    case 32: RI_DDE_H(32)
    case 64: RI_DDE_H(64)
    default: return fail(RI_EINVAL, "unsupported tile %d", p.tile);
  }
#undef RI_DDE_H
}

size_t region_cells(const Plan& p) {
  const size_t tw = size_t(p.tile) + p.dde.S - 1;
  return tw * tw;
}

}  // namespace

void dde_destroy(Dde& dd) {
  dev_free(dd.taps);
  dev_free(dd.vtaps);
  dev_free(dd.wmax);
  dev_free(dd.tunits);
  dev_free(dd.more);
  dev_free(dd.patch);
  dd = Dde{};
}

int dde_degrid(const Plan& p, const int4* units, int nunits, const Item* items, const uint8_t* mask,
               const float2* grid, float2* out, const float2* y, const float2* v, double* part, hipStream_t s) {
  if (nunits <= 0) return RI_OK;
  const bool resid = y != nullptr;
  return dispatch(p, [&]<int T, int H>() -> int {
    if (resid)
      hipLaunchKernelGGL((k_degrid_dde<T, H, DD_RESIDUAL>), dim3(wgs(p, nunits)), dim3(DT), 0, s, units, nunits,
                         items, mask, p.coord, p.dde.taps, p.M, p.poly, grid, p.K, p.tpa, out, y, v, part);
    else
      hipLaunchKernelGGL((k_degrid_dde<T, H, DD_APPLY>), dim3(wgs(p, nunits)), dim3(DT), 0, s, units, nunits, items,
                         mask, p.coord, p.dde.taps, p.M, p.poly, grid, p.K, p.tpa, out, y, v, part);
    RI_LAUNCH_CHECK();
    return RI_OK;
  });
}

int dde_grid(const Plan& p, const int4* units, int nunits, const Item* items, const uint8_t* mask, const float2* y,
             const float2* e, float2* v, const float* shrink, bool project, bool add_patch, hipStream_t s) {
  if (nunits <= 0) return RI_OK;
  return dispatch(p, [&]<int T, int H>() -> int {
    const dim3 g(wgs(p, nunits)), b(DT);
#define RI_GDDE(PR, AD)                                                                                        \
  hipLaunchKernelGGL((k_grid_dde<T, H, PR, AD>), g, b, 0, s, units, nunits, items, mask, p.coord, p.dde.vtaps,    \
                     p.dde.wmax, p.poly, y, e, v, shrink, p.dde.patch, p.tpa)
    if (project && add_patch) RI_GDDE(true, true);
    else if (project) RI_GDDE(true, false);
    else if (add_patch) RI_GDDE(false, true);
    else RI_GDDE(false, false);
#undef RI_GDDE
    RI_LAUNCH_CHECK();
    return RI_OK;
  });
}

int dde_merge(const Plan& p, float2* grid, bool add, bool units, hipStream_t s) {
  const int* more = units ? p.dde.more : nullptr;
  return dispatch(p, [&]<int T, int H>() -> int {
    const dim3 g(p.windowed ? p.n_gtiles : p.n_tiles), b(DT);
    if (p.windowed && add)
      hipLaunchKernelGGL((k_dde_merge_win<T, H, true>), g, b, 0, s, grid, p.dde.patch, more, p.K, p.tpa, p.gta);
    else if (p.windowed)
      hipLaunchKernelGGL((k_dde_merge_win<T, H, false>), g, b, 0, s, grid, p.dde.patch, more, p.K, p.tpa, p.gta);
    else if (add)
      hipLaunchKernelGGL((k_dde_merge<T, H, true>), g, b, 0, s, grid, p.dde.patch, more, p.K, p.tpa);
    else
      hipLaunchKernelGGL((k_dde_merge<T, H, false>), g, b, 0, s, grid, p.dde.patch, more, p.K, p.tpa);
    RI_LAUNCH_CHECK();
    return RI_OK;
  });
}

int dde_zero_patches(const Plan& p, hipStream_t s) {
  return zero_c64(p.dde.patch, size_t(p.n_tiles) * region_cells(p), s);
}

}  // namespace ri

using ri::fail;

extern "C" int ri_plan_dde(ri_plan plan, int jd, const float* d_host, hipStream_t stream) {
  if (!plan) return fail(RI_EINVAL, "plan is NULL");
  ri::Plan& p = plan->p;
  if (jd == 0 || d_host == nullptr) {
    if (jd != 0 || d_host != nullptr) return fail(RI_EINVAL, "removing DDEs takes jd = 0 and d = NULL");
    RI_HIP(hipStreamSynchronize(stream));
    ri::dde_destroy(p.dde);
    return RI_OK;
  }
  if (jd < 1 || jd % 2 == 0 || jd > 2 * ri::MAX_H + 1)
    return fail(RI_EINVAL, "jd = %d must be odd, 1 <= jd <= %d", jd, 2 * ri::MAX_H + 1);
  const int jd2 = jd * jd;
  for (int64_t k = 0; k < 2 * p.M * jd2; ++k)
    if (!std::isfinite(d_host[k])) return fail(RI_EINVAL, "non-finite DDE tap at visibility %lld", (long long)(k / (2 * jd2)));
  RI_HIP(hipStreamSynchronize(stream));
  ri::dde_destroy(p.dde);
  ri::Dde& dd = p.dde;
  const int h = jd / 2;
  dd.h = h;
  dd.S = ri::KB_J + 2 * h;
  int rc = RI_OK;
  try {
    // taps into plan order on the host
    std::vector<float2> dp(size_t(p.M) * jd2);
    const float2* du = reinterpret_cast<const float2*>(d_host);
    for (int64_t k = 0; k < p.M; ++k)
      std::copy(du + size_t(p.order_host[k]) * jd2, du + size_t(p.order_host[k] + 1) * jd2, dp.begin() + k * jd2);
    // the tiles' units: runs of items of at most `cap` visibilities, so that the densest tiles are
    // not one workgroup's work (300007 visibilities: 44 us at 256, 42 at 384, 41 at 512; more than
    // 512 leaves the chip fewer units than it holds at once) and the further patches stay fewer
    // than about 1024
    const int64_t cap = std::max<int64_t>(ri::GRID_UNIT_VIS, p.M / 1024);
    std::vector<int4> tunits;
    std::vector<int> count(p.n_tiles, 0), more(size_t(p.n_tiles) + 1, p.n_tiles);
    for (const int4& un : p.tile_units_host) {
      int64_t acc = 0;
      int a = un.y;
      for (int q = un.y; q <= un.z; ++q) {
        const int w = q < un.z ? p.titem_vis_host[q] : 0;
        if (q < un.z && (q == a || acc + w <= cap)) {
          acc += w;
          continue;
        }
        tunits.push_back(make_int4(un.x, a, q, count[un.x]++));
        a = q;
        acc = w;
      }
    }
    for (int t = 0; t < p.n_tiles; ++t) more[t + 1] = more[t] + std::max(0, count[t] - 1);
    for (int4& un : tunits) un.w = un.w == 0 ? un.x : more[un.x] + un.w - 1;
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.vtaps, dp.size());
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.taps, size_t(jd2) * p.M);
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.wmax, size_t(p.M));
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.tunits, tunits.size());
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.more, more.size());
    if (rc == RI_OK) rc = ri::dev_alloc(&dd.patch, size_t(more[p.n_tiles]) * ri::region_cells(p));
    if (rc == RI_OK) {
      dd.n_tunits = int(tunits.size());
      if (hipMemcpyAsync(dd.vtaps, dp.data(), dp.size() * sizeof(float2), hipMemcpyHostToDevice, stream) != hipSuccess ||
          hipMemcpyAsync(dd.tunits, tunits.data(), tunits.size() * sizeof(int4), hipMemcpyHostToDevice, stream) !=
              hipSuccess ||
          hipMemcpyAsync(dd.more, more.data(), more.size() * sizeof(int), hipMemcpyHostToDevice, stream) !=
              hipSuccess)
        rc = fail(RI_EHIP, "copy of the DDE tables failed");
    }
    if (rc == RI_OK) rc = ri::dde_zero_patches(p, stream);
    if (rc == RI_OK) {
      const unsigned g = unsigned(std::min<int64_t>((p.M + ri::DT - 1) / ri::DT, 65536));
      switch (h) {
        case 0: hipLaunchKernelGGL(ri::k_dde_taps<0>, dim3(g), dim3(ri::DT), 0, stream, p.M, p.coord, dd.vtaps, p.poly, dd.taps, dd.wmax); break;
        case 1: hipLaunchKernelGGL(ri::k_dde_taps<1>, dim3(g), dim3(ri::DT), 0, stream, p.M, p.coord, dd.vtaps, p.poly, dd.taps, dd.wmax); break;
        case 2: hipLaunchKernelGGL(ri::k_dde_taps<2>, dim3(g), dim3(ri::DT), 0, stream, p.M, p.coord, dd.vtaps, p.poly, dd.taps, dd.wmax); break;
        default: hipLaunchKernelGGL(ri::k_dde_taps<3>, dim3(g), dim3(ri::DT), 0, stream, p.M, p.coord, dd.vtaps, p.poly, dd.taps, dd.wmax); break;
      }
      if (hipGetLastError() != hipSuccess) rc = fail(RI_EHIP, "DDE tap kernel launch failed");
    }
    if (rc == RI_OK && hipStreamSynchronize(stream) != hipSuccess) rc = fail(RI_EHIP, "stream sync failed");
  } catch (const std::bad_alloc&) {
    rc = fail(RI_ENOMEM, "host allocation failed");
  }
  if (rc != RI_OK) ri::dde_destroy(dd);
  return rc;
}
