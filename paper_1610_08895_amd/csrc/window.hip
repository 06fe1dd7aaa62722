// Gridding by windows, for plans with grids of up to WINDOWED_K cells per axis (gridding.hip
// holds the kernel for larger grids, and the degridding of both): G_i^dagger with the dual
// update of step 8 fused in, as in gridding.hip.
//
// A window is an aligned 8 x 8 group of grid cells; the footprints of all visibilities whose
// cell lies in it fall in one 16 x 16 patch of the grid (15 x 15 of it), so with wx_m and wy_m
// the 8 weights of visibility m placed at its cell's offset in a zero row of 16,
//
//   patch[i][j] += sum_m wy_m[i] (v_m wx_m[j])      (rows x visibilities x columns),
//
// an FP32 matrix product on the matrix cores (v_mfma_f32_16x16x4_f32, exact FP32
// multiply-adds).  The placed weight rows pass through a per-wavefront LDS buffer: 64 lanes
// evaluate the x and the y weights of 32 visibilities (a chunk) at once, store them as columns
// of a [row][visibility] array over zeros, and read them back in the operands' layouts.  The
// plan sorts a block's visibilities by tile and window, so that the visibilities of a window
// are one contiguous run (a segment) per block.
//
// The matrix accumulators hold one chunk's sum at a time, which is added to the window's by
// Kahan's compensated summation: a chain of FP32 additions over all of a window's visibilities
// loses bits with their number.  65536 visibilities in one window of a 512^2 image, error of
// Phi^dagger against FP64, one chain -> chunks: equal samples 2.7e-4 -> 4.8e-7, ones at random places
// 3.1e-5 -> 1.6e-7, random values 2.5e-6 -> 4.3e-7 (gridding.hip's integer sums: 2.1e-6, 3.0e-7,
// 1.7e-6).  It costs 32 vector instructions a chunk: the adjoint of 1.5 10^6 visibilities at 512^2, the
// whole call 63.1 -> 64.5 us.
//
// Why only small grids: the matrix product takes 16 cycles of a SIMD's matrix unit per
// visibility, the placing and the loads as much again on the VALU and the LDS, and together
// they are no faster than gridding.hip's 64 atomics per visibility on a chip that those keep
// full (2^22 visibilities at 1024^2: 98 us here, before the sums were compensated, 92 us there).  But a 32 x 32 tile per
// workgroup leaves most of the chip idle on a small grid and its densest tile decides the time;
// a window per wavefront or less spreads the same work over 16 times as many.  Per launch in the
// solver and the adjoint, tiles with their halo pass -> windows: 2^13 visibilities at 64^2 25.3 ->
// 10.8 us and 82000 of 327680 (masked) at 256^2 47 -> 24 (both with the deep wavelet levels in the
// launch), 500000 of 10^6 (masked) at 512^2 67 -> 26.6, 1.5 10^6 (a tenth of them spread evenly) at
// 512^2 92.6 -> 37; the error of Phi^dagger at the last 1.9e-6 -> 4.0e-7.
#include <algorithm>

#include "plan.hpp"
#include "sara_dev.hpp"

namespace ri {

namespace {

constexpr int CH = 32;  // visibilities per chunk: two lanes each (one per axis, or per component)
// Row pitch of a chunk's weight array in LDS: the 16-byte reads of 16 rows touch every bank
// equally often.
constexpr int WP = CH + 4;
constexpr int WROWS = 16;
constexpr int WBUF = 2 * WROWS * WP;  // x rows, then y rows

using f32x4 = float __attribute__((ext_vector_type(4)));

// Orders LDS traffic of one wavefront (whose LDS operations execute in program order): the
// compiler may not move accesses across it, and no instruction is emitted.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Takes over a value loaded ahead, as a move that the compiler cannot merge or delay: the
// register the value was loaded into is then free for the next load, which would otherwise go
// to a fresh one and be waited for at once to be copied.
template <class T>
__device__ __forceinline__ T take(T x) {
  T r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// Lanes of a chunk: lane l = 16 g + m holds component (or axis) g & 1 of visibility
// 16 (g >> 1) + m.
__device__ __forceinline__ int lane_vis(int lane) { return ((lane >> 5) << 4) | (lane & 15); }

// Places the weights of this lane's packed coordinate in the chunk's array `w` (x rows, then y
// rows) as a column over zeros.
__device__ __forceinline__ void place_weights(float* w, int lane, unsigned packed, const KBPoly& P) {
  float k[KB_J];
  int cell;
  kb_weights(packed, P, k, cell);
  f32x4* z = reinterpret_cast<f32x4*>(w);
#pragma unroll
  for (int i = 0; i < WBUF / 4; i += 64)
    if (i + 64 <= WBUF / 4 || lane < WBUF / 4 - i) z[i + lane] = f32x4{0.f, 0.f, 0.f, 0.f};
  wave_lds_fence();
  float* col = w + ((lane >> 4) & 1) * (WROWS * WP) + (cell & (WIN - 1)) * WP + lane_vis(lane);
#pragma unroll
  for (int j = 0; j < KB_J; ++j) col[j * WP] = k[j];
}

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// s += p by Kahan's summation, whose error does not grow with the number of terms (c: by how much
// rounding has left s too large).
__device__ __forceinline__ void add_compensated(f32x4& s, f32x4& c, const f32x4 p) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float y = p[k] - c[k], t = s[k] + y;
    c[k] = (t - s[k]) - y;
    s[k] = t;
  }
}

// APPLY: grid y.  PROJECT: step 8 from r and v_old, grid v_new - v_old.  FRESH: every block
// active, step 8 from r alone, grid v_new.
enum { GR_APPLY = 0, GR_PROJECT = 1, GR_FRESH = 2 };

// Inclusive prefix sum over the 64 lanes (all active).
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// One workgroup per unit, a tile of 16 x 16 cells or a part of a dense one's visibilities, with SPLIT
// wavefronts per window of it, which take the window's chunks in turn.  A wavefront goes through its
// window's segments (all blocks; those of inactive blocks count as empty) in batches of 64, one lane
// per segment: the prefix sums of their counts go to a table in LDS, in which each lane of a chunk
// then finds its visibility by bisection.  The patch stays in registers until the window is done;
// the wavefronts' patches are then summed into the tile's 23 x 23 region and stored in the tile's
// own slot of the patch array (added to it with `add`; a dense tile's further parts are always
// stored, each in its own slot of xpatch, for k_win_merge), which nobody else writes: no atomics and
// no order dependence, so results are deterministic.  The adjoint column pass adds the overlapping
// regions.
// SIDE: the workgroups after the tiles' are those of a sparsity job.
template <int MODE, int SPLIT, bool SIDE>
__global__ __launch_bounds__(256 * SPLIT, 4) void k_win_grid(const int* __restrict__ slots, int nunits,
                                                                 const int* __restrict__ woff, const int4* __restrict__ wsegs,
                                                                 const uint8_t* __restrict__ mask,
                                                                 const unsigned* __restrict__ coord, float2* __restrict__ patch,
                                                                 float2* __restrict__ xpatch, int ntiles, KBPoly P,
                                                                 const float* __restrict__ y, const float* __restrict__ e,
                                                                 float* __restrict__ v, const float* __restrict__ shrink, int add, int stride,
                                                                 SideJob side) {
  constexpr int NW = 4 * SPLIT, GT = 64 * NW;
  constexpr int DP = WROWS + 1;  // pitch of a window's patch in LDS
  static_assert(WROWS * DP * 2 <= WBUF, "a window's patch takes the place of its weights");
  struct Shared {
    float wbuf[NW][WBUF];
    float vbuf[NW][2 * CH];
    int4 tab[NW][64];
    int touched[NW];
  };
  constexpr int SIDE_BYTES = SIDE ? side_smem<GT>() : 0;
  __shared__ __align__(16) char smem[SIDE_BYTES > int(sizeof(Shared)) ? SIDE_BYTES : int(sizeof(Shared))];
  if constexpr (SIDE) {
    if (int(blockIdx.x) >= stride) {
      // (the operator form is the reverse sweep's)
      side_body<GT, MODE == GR_APPLY ? SIDE_DEEP_GATE : SIDE_DEEP>(side, int(blockIdx.x) - stride, smem);
      return;
    }
  }
  // the data branch's kernels issue ahead of the sparsity branch's waves sharing their SIMDs
  __builtin_amdgcn_s_setprio(3);
  Shared& sh = *reinterpret_cast<Shared*>(smem);
  auto& wbuf = sh.wbuf;
  auto& vbuf = sh.vbuf;
  auto& tab = sh.tab;
  auto& touched = sh.touched;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, m = lane & 15, comp = g & 1, sl = lane_vis(lane);
  float* w = wbuf[wv];
  for (int u = blockIdx.x; u < nunits; u += stride) {
    const int win = wv / SPLIT, first = (wv % SPLIT) * CH;
    const int s0 = woff[4 * u + win], s1 = woff[4 * u + win + 1];
    f32x4 dr = {0.f, 0.f, 0.f, 0.f}, di = {0.f, 0.f, 0.f, 0.f}, cr = dr, ci = di;
    bool any = false;
    for (int b0 = s0; b0 < s1; b0 += 64) {
      const int nb = min(64, s1 - b0);
      int4 sg = make_int4(0, 0, 0, 0);
      if (lane < nb) sg = wsegs[b0 + lane];
      bool act = lane < nb;
      if (act && mask != nullptr) act = mask[sg.z] != 0;
      const int cnt = act ? sg.y : 0;
      float fac = 0.f;
      if (MODE != GR_APPLY && act) fac = shrink[sg.z];
      const int incl = wave_scan(cnt);
      const int total = __builtin_amdgcn_readlane(incl, 63);
      if (total == 0) continue;
      any = true;
      wave_lds_fence();
      tab[wv][lane] = make_int4(incl - cnt, sg.x, __float_as_int(fac), sg.w);
      wave_lds_fence();
      int step0 = 0;  // the largest power of two below nb
      if (nb > 1) step0 = 1 << (31 - __builtin_clz(nb - 1));
      // this lane's operands of the chunk at q (of the batch's last visibility past its end)
      unsigned cn;
      float rn, on = 0.f, shn = 0.f;
      int pn;
      auto load_vis = [&](int q) {
        const int s = min(q + sl, total - 1);
        int k = 0;
        for (int st = step0; st > 0; st >>= 1)
          if (tab[wv][k + st].x <= s) k += st;
        const int4 en = tab[wv][k];
        pn = en.y + s - en.x;
        shn = __int_as_float(en.z);
        const size_t i = 2 * size_t(pn) + comp;
        cn = coord[i];
        if (MODE == GR_APPLY) {
          rn = y[i];
        } else {
          rn = e[i];
          if (MODE == GR_PROJECT) on = v[i];
        }
      };
      load_vis(first);
      for (int q = first; q < total; q += SPLIT * CH) {
        const unsigned cw = take(cn);
        const int pos = pn;
        const float old = MODE == GR_PROJECT ? take(on) : 0.f;
        float val = take(rn);
        if (MODE != GR_APPLY) val *= shn;
        __builtin_amdgcn_sched_barrier(0);
        load_vis(q + SPLIT * CH);
        const bool in = q + sl < total;
        if (MODE != GR_APPLY && in) v[2 * size_t(pos) + comp] = val;
        if (MODE == GR_PROJECT) val -= old;
        if (!in) val = 0.f;
        if (__ballot(val != 0.f) == 0ull) continue;  // duals that did not change
        wave_lds_fence();
        place_weights(w, lane, cw, P);
        vbuf[wv][comp * CH + sl] = val;
        wave_lds_fence();
        f32x4 pr = {0.f, 0.f, 0.f, 0.f}, pi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if (t > 0 && q + 16 * t >= total) continue;
          const int o = 16 * t + 4 * g;
          const f32x4 a = *reinterpret_cast<const f32x4*>(w + (WROWS + m) * WP + o);
          const f32x4 x = *reinterpret_cast<const f32x4*>(w + m * WP + o);
          const f32x4 vr = *reinterpret_cast<const f32x4*>(&vbuf[wv][o]);
          const f32x4 vi = *reinterpret_cast<const f32x4*>(&vbuf[wv][CH + o]);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            pr = mfma(a[k], x[k] * vr[k], pr);
            pi = mfma(a[k], x[k] * vi[k], pi);
          }
        }
        add_compensated(dr, cr, pr);
        add_compensated(di, ci, pi);
      }
    }
    // the window's patch, rows 4 g + k and column m in this lane, to LDS
    wave_lds_fence();
    float2* d = reinterpret_cast<float2*>(w);
#pragma unroll
    for (int k = 0; k < 4; ++k) d[(4 * g + k) * DP + m] = make_float2(dr[k], di[k]);
    if (lane == 0) touched[wv] = any;
    __syncthreads();
    const int slot = slots[u];
    const bool store = !add || slot >= ntiles;
    bool changed = store;
#pragma unroll
    for (int k = 0; k < NW; ++k) changed = changed || touched[k] != 0;
    if (changed) {
      float2* pt = slot < ntiles ? patch + size_t(slot) * PATCH_CELLS : xpatch + size_t(slot - ntiles) * PATCH_CELLS;
      for (int c = threadIdx.x; c < PATCH_CELLS; c += GT) {
        const int R = c / PATCH_W, C = c - (c / PATCH_W) * PATCH_W;
        float2 s = make_float2(0.f, 0.f);
#pragma unroll
        for (int wy = 0; wy < 2; ++wy)
#pragma unroll
          for (int wx = 0; wx < 2; ++wx) {
            const int r = R - WIN * wy, cc = C - WIN * wx;
            if (r >= 0 && r < WROWS && cc >= 0 && cc < WROWS) {
#pragma unroll
              for (int k = 0; k < SPLIT; ++k) {
                const float2 t = reinterpret_cast<const float2*>(wbuf[(2 * wy + wx) * SPLIT + k])[r * DP + cc];
                s.x += t.x;
                s.y += t.y;
              }
            }
          }
        if (store) {
          pt[c] = s;
        } else if (s.x != 0.f || s.y != 0.f) {
          const float2 old = pt[c];
          pt[c] = make_float2(old.x + s.x, old.y + s.y);
        }
      }
    }
    __syncthreads();
  }
}

// Adds a dense tile's further parts to its own slot: one workgroup per 64 cells of a tile, its
// wavefronts taking every 16th part (compensated sums, so that many parts cost no bits) and then
// summed in order.
constexpr int MW = 16, MERGE_BLOCKS = PATCH_CELLS / 64;
static_assert(PATCH_CELLS % 64 == 0, "whole wavefronts of cells");
__global__ __launch_bounds__(64 * MW) void k_win_merge(const int4* __restrict__ split, float2* __restrict__ patch,
                                                       const float2* __restrict__ xpatch) {
  __shared__ float2 part[MW][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int4 sp = split[blockIdx.x / MERGE_BLOCKS];
  const int c = (blockIdx.x % MERGE_BLOCKS) * 64 + lane;
  const float2* x = xpatch + size_t(sp.y) * PATCH_CELLS + c;
  float2 s = make_float2(0.f, 0.f), e = s;
#pragma unroll 4
  for (int j = wv; j < sp.z; j += MW) {
    const float2 v = x[size_t(j) * PATCH_CELLS];
    const float2 y = csub(v, e), t = cadd(s, y);
    e = csub(csub(t, s), y);
    s = t;
  }
  part[wv][lane] = s;
  __syncthreads();
  if (wv > 0) return;
  float2* p = patch + size_t(sp.x) * PATCH_CELLS + c;
  float2 a = *p;
  for (int k = 0; k < MW && k < sp.z; ++k) a = cadd(a, part[k][lane]);
  *p = a;
}

const float* words(const float2* p) { return reinterpret_cast<const float*>(p); }
float* words(float2* p) { return reinterpret_cast<float*>(p); }

struct Units {
  const int *slots, *woff;
  const int4* segs;
  int n;
};

template <int MODE, int SPLIT>
int launch(const Plan& p, const Units& q, const uint8_t* mask, float2* patch, const float2* y, const float2* e,
           float2* v, const float* shrink, bool add, hipStream_t s, const SideJob* side) {
  const int g = p.persistent_wgs > 0 ? std::min(p.persistent_wgs, q.n) : q.n;
  const unsigned* coord = reinterpret_cast<const unsigned*>(p.coord);
  if (side != nullptr && side->wgs > 0) {
    if constexpr (SPLIT == 4) {
      static_assert(256 * SPLIT == DEEP_THREADS, "the job's workgroup size");
      hipLaunchKernelGGL((k_win_grid<MODE, SPLIT, true>), dim3(g + side->wgs), dim3(256 * SPLIT), 0, s, q.slots, q.n,
                         q.woff, q.segs, mask, coord, patch, p.xpatch, p.n_gtiles, p.poly, words(y), words(e),
                         words(v), shrink, add ? 1 : 0, g, *side);
    } else {
      return fail(RI_EINVAL, "windowed gridding: no side job here");
    }
  } else {
    hipLaunchKernelGGL((k_win_grid<MODE, SPLIT, false>), dim3(g), dim3(256 * SPLIT), 0, s, q.slots, q.n, q.woff,
                       q.segs, mask, coord, patch, p.xpatch, p.n_gtiles, p.poly, words(y), words(e), words(v),
                       shrink, add ? 1 : 0, g, SideJob{});
  }
  RI_LAUNCH_CHECK();
  return RI_OK;
}

template <int MODE>
int grid_units(const Plan& p, const Units& q, const uint8_t* mask, float2* patch, const float2* y, const float2* e,
               float2* v, const float* shrink, bool add, hipStream_t s, const SideJob* side = nullptr) {
  if (q.n <= 0) return RI_OK;
  return p.win_split == 1 ? launch<MODE, 1>(p, q, mask, patch, y, e, v, shrink, add, s, side)
                          : launch<MODE, 4>(p, q, mask, patch, y, e, v, shrink, add, s, side);
}

// Over every unit (tiles without visibilities among them, so that a fresh pass also clears what the
// DDE kernels may have left there), and the parts of the dense tiles together.
template <int MODE>
int grid_tiles(const Plan& p, const uint8_t* mask, float2* patch, const float2* y, const float2* e, float2* v,
               const float* shrink, bool add, hipStream_t s, const SideJob* side) {
  const Units all{p.wslots, p.woff, p.wsegs, p.n_wunits};
  RI_TRY(grid_units<MODE>(p, all, mask, patch, y, e, v, shrink, add, s, side));
  if (p.n_wsplit > 0) {
    hipLaunchKernelGGL(k_win_merge, dim3(p.n_wsplit * MERGE_BLOCKS), dim3(64 * MW), 0, s, p.wsplit, patch, p.xpatch);
    RI_LAUNCH_CHECK();
  }
  return RI_OK;
}

}  // namespace

int win_apply(const Plan& p, const float2* y, const uint8_t* mask, float2* patch, hipStream_t s, const SideJob* side) {
  return grid_tiles<GR_APPLY>(p, mask, patch, y, nullptr, nullptr, nullptr, false, s, side);
}

int win_project(const Plan& p, const float2* e, float2* v, const float* shrink, const uint8_t* mask, float2* patch,
                hipStream_t s, const SideJob* side) {
  return grid_tiles<GR_PROJECT>(p, mask, patch, nullptr, e, v, shrink, true, s, side);
}

int win_project_all(const Plan& p, const float2* r, float2* v, const float* shrink, float2* patch, hipStream_t s,
                    const SideJob* side) {
  return grid_tiles<GR_FRESH>(p, nullptr, patch, nullptr, r, v, shrink, false, s, side);
}

int win_project_block(const Plan& p, int block, const float2* e, float2* v, const float* shrink, float2* patch,
                      hipStream_t s) {
  const int a = p.bwoff_host[block], b = p.bwoff_host[block + 1];
  const Units mine{p.bslots + a, p.bwoff + 4 * a, p.bsegs, b - a};
  return grid_units<GR_PROJECT>(p, mine, nullptr, patch, nullptr, e, v, shrink, true, s);
}

}  // namespace ri
