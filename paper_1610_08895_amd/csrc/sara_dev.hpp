// Device code of the SARA filter banks (sara.hip), shared with the kernels that carry parts of
// the sparsity branch as further workgroups of their launches.
#pragma once

#include "sara.hpp"

namespace ri {

constexpr int ST = 256;  // threads per workgroup
constexpr int TO = 16;   // analysis: outputs per subband per axis per workgroup
constexpr int TS = 32;   // synthesis: outputs per axis per workgroup
constexpr int STAGE_ROWS = ST / 32;  // rows per step of a staging with 32 threads to a row

__device__ __forceinline__ float clampf(float v, float a) { return fminf(fmaxf(v, -a), a); }

// Tile (tx, ty) of workgroup b of an nx x ny tile grid.  Consecutive workgroups go round-robin
// to the eight XCDs, so with a row-major order neighbouring tiles, whose staged regions overlap,
// would sit on different XCDs; when the row count is a multiple of 8, each XCD takes a band of
// whole tile rows instead, and the overlaps are fetched once into its L2.
__device__ __forceinline__ void band_tile(int b, int nx, int ny, int& tx, int& ty) {
  if (ny % 8 != 0) {
    ty = b / nx;
    tx = b - (b / nx) * nx;
    return;
  }
  const int i = b / 8;
  ty = (b % 8) * (ny / 8) + i / nx;
  tx = i - (i / nx) * nx;
}

// Two neighbouring floats of a caller's buffer, which is aligned to one float only; and the value
// at a byte offset, which an address register and a 32-bit offset reach (no array here is larger
// than 2^32 bytes per basis).
typedef float floatpair __attribute__((ext_vector_type(2), aligned(4)));
template <class V>
__device__ __forceinline__ V& at_byte(const float* base, unsigned off) {
  return *reinterpret_cast<V*>(const_cast<char*>(reinterpret_cast<const char*>(base)) + off);
}

// bound of the clip at coefficient k of s: alpha, or alpha w_k (the same FP32 product
// wherever it is formed, so a clipped value equals the bound exactly)
__device__ __forceinline__ float clip_bound(const DwtArgs& A, size_t k) {
  return A.wts != nullptr ? A.alpha * A.wts[k] : A.alpha;
}

// the new coefficient from the old one and v, its analysis (g: the gate's value)
template <bool GATE>
__device__ __forceinline__ float new_coef(const DwtArgs& A, float old, float bound, float g, float v) {
  if (GATE) return fabsf(g) < bound ? fmaf(A.scale, v, old) : 0.f;
  return A.clip ? clampf(old + v, bound) : v;
}

// One analysis level for wavelet w with filters of (compile-time) length L on an output
// tile (i0, j0) of each subband.  Sizes are powers of two, so indices wrap with masks.
// Bound by instructions more than by memory: of level 1 at 1024^2, 21.9 us, 13 were vector
// instructions, a third of them filters and most others addresses.  With pairs, constant steps and
// 32-bit offsets they take 9 of 17 us (36 MB written); the finest synthesis level, staged the same
// way, 22.3 -> 18 us.
template <int L, bool GATE>
__device__ __forceinline__ void analysis_tile(const DwtArgs& A, const float* __restrict__ hw, int w, int i0,
                                              int j0, float* in, float2* lh) {
  const float* __restrict__ gw = hw + MAX_TAPS;
  constexpr int RE = 2 * TO + L - 2;       // input rows / columns the tile reads
  constexpr int RW = 2 * TO + MAX_TAPS - 2; // LDS row stride
  const int n = A.n, m = A.m, mo = A.m / 2, mm = A.m - 1;
  const float* src = A.level == 1 ? A.x : A.tmp + w * A.tmp_stride + A.in_off;
  float* sb = A.s + size_t(w + A.dirac) * n * n;
  // the coefficients this thread updates (one output position per thread: TO * TO == ST),
  // loaded now so that their latency overlaps the staging and the filters
  static_assert(TO * TO == ST, "one output position per thread");
  const int pi = threadIdx.x / TO, pj = threadIdx.x - (threadIdx.x / TO) * TO;
  const int qi = i0 + pi, qj = j0 + pj;
  const bool mine = qi < mo && qj < mo;
  float old[4] = {0.f, 0.f, 0.f, 0.f}, bnd[4] = {A.alpha, A.alpha, A.alpha, A.alpha};
  const size_t sbo = size_t(w + A.dirac) * n * n;
  const unsigned k0 = 4u * (__umul24(qi, n) + qj), kx = 4u * mo, ky = 4u * __umul24(mo, n);
  const unsigned ko[4] = {k0, k0 + kx, k0 + ky, k0 + ky + kx};  // byte offsets in the basis
  if (A.clip && mine) {
    if (A.level == A.levels) old[0] = at_byte<const float>(sb, ko[0]);
#pragma unroll
    for (int c = 1; c < 4; ++c) old[c] = at_byte<const float>(sb, ko[c]);
    if (A.wts != nullptr)
#pragma unroll
      for (int c = 0; c < 4; ++c) bnd[c] = A.alpha * at_byte<const float>(A.wts + sbo, ko[c]);
  }
  float gate[4] = {0.f, 0.f, 0.f, 0.f};
  if (GATE && mine)
#pragma unroll
    for (int c = 0; c < 4; ++c) gate[c] = at_byte<const float>(A.gate + sbo, ko[c]);
  // staged by pairs, 32 threads to a row, so that a thread's column stays and its rows step by 8;
  // the rows wrap, so those after the tile's last are loaded like the others (a load of each row
  // under its own condition would wait for the one before)
  {
    const int lx = threadIdx.x % 32, ly0 = threadIdx.x / 32;
    if (lx < RE / 2) {
      constexpr int PER = (RE + STAGE_ROWS - 1) / STAGE_ROWS;
      const unsigned col = 4u * ((2 * j0 + 2 * lx) & mm);
      floatpair r[PER];
#pragma unroll
      for (int e = 0; e < PER; ++e)
        r[e] = at_byte<const floatpair>(src, 4u * __umul24((2 * i0 + ly0 + e * STAGE_ROWS) & mm, m) + col);
#pragma unroll
      for (int e = 0; e < PER; ++e)
        *reinterpret_cast<float2*>(&in[(ly0 + e * STAGE_ROWS) * RW + 2 * lx]) = make_float2(r[e].x, r[e].y);
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < (RE * TO + ST - 1) / ST; ++e) {
    if (int(threadIdx.x) + e * ST >= RE * TO) break;
    const float2* row = reinterpret_cast<const float2*>(&in[(pi + e * (ST / TO)) * RW + 2 * pj]);
    float a = 0.f, d = 0.f;
#pragma unroll
    for (int t = 0; t < L / 2; ++t) {
      const float2 v = row[t];
      a = fmaf(hw[2 * t], v.x, a);
      d = fmaf(gw[2 * t], v.x, d);
      a = fmaf(hw[2 * t + 1], v.y, a);
      d = fmaf(gw[2 * t + 1], v.y, d);
    }
    lh[threadIdx.x + e * ST] = make_float2(a, d);
  }
  __syncthreads();
  if (!mine) return;
  float ll = 0.f, hi = 0.f, hl = 0.f, hh = 0.f;  // hi: low along y, high along x
#pragma unroll
  for (int t = 0; t < L; ++t) {
    const float2 v = lh[(2 * pi + t) * TO + pj];
    ll = fmaf(hw[t], v.x, ll);
    hi = fmaf(hw[t], v.y, hi);
    hl = fmaf(gw[t], v.x, hl);
    hh = fmaf(gw[t], v.y, hh);
  }
  auto put = [&](int c, float v) { at_byte<float>(sb, ko[c]) = new_coef<GATE>(A, old[c], bnd[c], gate[c], v); };
  if (A.level < A.levels) at_byte<float>(A.tmp + w * A.tmp_stride + A.out_off, 4u * (__umul24(qi, mo) + qj)) = ll;
  else put(0, ll);
  put(1, hi);
  put(2, hl);
  put(3, hh);
}

#define RI_SWITCH_L(LEN, CALL)          \
  switch (LEN) {                        \
    case 2: CALL(2); break;             \
    case 4: CALL(4); break;             \
    case 6: CALL(6); break;             \
    case 8: CALL(8); break;             \
    case 10: CALL(10); break;           \
    case 12: CALL(12); break;           \
    case 14: CALL(14); break;           \
    default: CALL(16); break;           \
  }

// Analysis level: workgroup b of nx * ny * (wavelets, and the Dirac basis at level 1).
constexpr int DWT_RW = 2 * TO + MAX_TAPS - 2;
constexpr int DWT_IN = (DWT_RW + STAGE_ROWS - 1) / STAGE_ROWS * STAGE_ROWS * DWT_RW * 4;  // whole steps of rows
constexpr int DWT_SMEM = DWT_IN + DWT_RW * TO * 8;
template <bool GATE>
__device__ __forceinline__ void dwt_body(const DwtArgs& A, const float* __restrict__ filt,
                                         const int* __restrict__ flen, int b, int nx, int ny, char* smem) {
  float* in = reinterpret_cast<float*>(smem);
  float2* lh = reinterpret_cast<float2*>(smem + DWT_IN);
  const int n = A.n, z = b / (nx * ny);
  int tx, ty;
  band_tile(b - z * (nx * ny), nx, ny, tx, ty);
  const int i0 = ty * TO, j0 = tx * TO;
  if (z == A.nw) {  // Dirac basis at level 1: coefficient = pixel
    for (int idx = threadIdx.x; idx < 4 * TO * TO; idx += ST) {
      const int r = 2 * i0 + idx / (2 * TO), c = 2 * j0 + idx % (2 * TO);
      if (r >= n || c >= n) continue;
      const size_t k = size_t(r) * n + c;
      A.s[k] = new_coef<GATE>(A, A.clip ? A.s[k] : 0.f, A.clip ? clip_bound(A, k) : 0.f, GATE ? A.gate[k] : 0.f, A.x[k]);
    }
    return;
  }
#define RI_ANALYSIS(LL) analysis_tile<LL, GATE>(A, filt + z * FILT_STRIDE, z, i0, j0, in, lh)
  RI_SWITCH_L(flen[z], RI_ANALYSIS)
#undef RI_ANALYSIS
}

constexpr int RS = TS / 2 + MAX_TAPS / 2;  // LDS stride of a staged subband region

// Coefficients of one synthesis tile: output tile (p0, q0) of wavelet w (half filter
// length H) reads rows / columns [p0 / 2 - H, p0 / 2 + TS / 2) and [q0 / 2 - H, ...) of
// each of its four subbands (periodic): RL x RL, RL = TS / 2 + H.  Of 256 threads, 32 take a row,
// so that a thread's column stays and its rows step by 8; rows after the region's last are staged
// too (indices wrap), without a condition that would make each load wait for the one before.
constexpr int STAGE_PER = (RS + STAGE_ROWS - 1) / STAGE_ROWS;
static_assert(RS <= 32 && RS % STAGE_ROWS == 0, "a row of the region is one group of 32 threads; whole steps");
struct Stage {
  float v[4][STAGE_PER];
};

__device__ __forceinline__ void fetch_stage(const IdwtArgs& A, int w, int H, int p0, int q0, int tid, Stage& r) {
  const int RL = TS / 2 + H;
  const int n = A.n, mo = A.m / 2, mk = A.m / 2 - 1;
  const int kx = tid % 32, ky0 = tid / 32;
  if (kx >= RL) return;
  const int gx = (q0 / 2 - H + kx) & mk, gy0 = p0 / 2 - H + ky0;
  const float* sw = A.s + size_t(w + A.dirac) * n * n;
  const bool ll_coef = A.level == A.levels;
  const float* ll = ll_coef ? sw : A.tmp + w * A.tmp_stride + A.ll_off;
  const int ll_stride = ll_coef ? n : mo;
  const unsigned ox = 4u * mo, oy = 4u * __umul24(mo, n);
#pragma unroll
  for (int e = 0; e < STAGE_PER; ++e) {
    const int gy = (gy0 + e * STAGE_ROWS) & mk;
    const unsigned k = 4u * (__umul24(gy, n) + gx);
    r.v[0][e] = at_byte<const float>(ll, 4u * (__umul24(gy, ll_stride) + gx));
    r.v[1][e] = at_byte<const float>(sw, k + ox);       // low-y, high-x
    r.v[2][e] = at_byte<const float>(sw, k + oy);       // high-y, low-x
    r.v[3][e] = at_byte<const float>(sw, k + oy + ox);  // high-y, high-x
  }
}

__device__ __forceinline__ void deposit_stage(int H, const Stage& r, int tid, float4* sb) {
  const int RL = TS / 2 + H, kx = tid % 32, ky0 = tid / 32;
  if (kx >= RL) return;
#pragma unroll
  for (int e = 0; e < STAGE_PER; ++e) {
    sb[(ky0 + e * STAGE_ROWS) * RS + kx] = make_float4(r.v[0][e], r.v[1][e], r.v[2][e], r.v[3][e]);
  }
}

// One synthesis level for one wavelet (filters of length L) on a tile whose coefficients
// are staged in sb: out[2q + r] = sum_u h[2u + r] a[q - u] + g[2u + r] d[q - u] along each
// axis (the transpose of the analysis), columns (y) first into lh (low and high along x), then
// rows (x).  Returns through `emit(k, pl, q, v_even, v_odd)` the output pairs (p0 + pl, q0 + 2q
// + {0, 1}).  tid: the thread within the 256 that share sb and lh.  Requires sb complete (a
// barrier after staging); ends after the barrier between its two passes, so sb may be
// overwritten once it returns.  A coefficient's four subbands and a column sum's two halves lie
// together in LDS, so that one instruction reads them.
template <int L, class Emit>
__device__ __forceinline__ void synthesis_staged(const float* __restrict__ hw, const float4* sb, float2* lh, int tid,
                                                 Emit& emit) {
  const float* __restrict__ gw = hw + MAX_TAPS;
  constexpr int H = L / 2;
  constexpr int RL = TS / 2 + H;
  for (int idx = tid; idx < (TS / 2) * RL; idx += ST) {
    const int qy = idx / RL, jl = idx - qy * RL;
    float le = 0.f, lo = 0.f, he = 0.f, ho = 0.f;
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const float4 c = sb[(qy + H - u) * RS + jl];
      le = fmaf(hw[2 * u], c.x, fmaf(gw[2 * u], c.z, le));
      lo = fmaf(hw[2 * u + 1], c.x, fmaf(gw[2 * u + 1], c.z, lo));
      he = fmaf(hw[2 * u], c.y, fmaf(gw[2 * u], c.w, he));
      ho = fmaf(hw[2 * u + 1], c.y, fmaf(gw[2 * u + 1], c.w, ho));
    }
    lh[(2 * qy) * RS + jl] = make_float2(le, he);
    lh[(2 * qy + 1) * RS + jl] = make_float2(lo, ho);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < TS * TS / 2 / ST; ++k) {
    const int idx = tid + k * ST;
    const int pl = idx / (TS / 2), qx = idx - pl * (TS / 2);
    float ve = 0.f, vo = 0.f;
#pragma unroll
    for (int u = 0; u < H; ++u) {
      const float2 c = lh[pl * RS + qx + H - u];
      ve = fmaf(hw[2 * u], c.x, fmaf(gw[2 * u], c.y, ve));
      vo = fmaf(hw[2 * u + 1], c.x, fmaf(gw[2 * u + 1], c.y, vo));
    }
    emit(k, pl, qx, ve, vo);
  }
}

// Synthesis level: workgroup b of nx * ny * wavelets.
constexpr int IDWT_SMEM = RS * RS * 16 + TS * RS * 8;
__device__ __forceinline__ void idwt_body(const IdwtArgs& A, const float* __restrict__ filt,
                                          const int* __restrict__ flen, int b, int nx, int ny, char* smem) {
  float4* sb = reinterpret_cast<float4*>(smem);
  float2* lh = reinterpret_cast<float2*>(smem + RS * RS * 16);
  const int w = b / (nx * ny);
  int tx, ty;
  band_tile(b - w * (nx * ny), nx, ny, tx, ty);
  const int p0 = ty * TS, q0 = tx * TS, m = A.m;
  float* out = A.tmp + w * A.tmp_stride + A.out_off;
  auto emit = [&](int, int pl, int qx, float ve, float vo) {
    const int p = p0 + pl, q = q0 + 2 * qx;
    if (p < m && q < m) at_byte<floatpair>(out, 4u * (__umul24(p, m) + q)) = floatpair{ve, vo};
  };
  const int L = flen[w], tid = threadIdx.x;
  Stage r;
  fetch_stage(A, w, L / 2, p0, q0, tid, r);
  deposit_stage(L / 2, r, tid, sb);
  __syncthreads();
#define RI_SYNTH(LL) synthesis_staged<LL>(filt + w * FILT_STRIDE, sb, lh, tid, emit)
  RI_SWITCH_L(L, RI_SYNTH)
#undef RI_SYNTH
}

// Last level: each workgroup sums all wavelets' syntheses of its tile, in order.  Its TG groups
// of 256 threads take the wavelets in turn (a long filter after a short one); a group loads its
// next wavelet's coefficients into registers while the current one is computed.  With one group
// the sums stay in registers; with four the wavelets' tiles are added through LDS, which
// shortens the chain of eight loads, two passes and their barriers where there are too few
// tiles to hide it, and costs where there are enough: 14.4 -> 7.8 us at 64^2 (4 tiles), 16.4 -> 8.7 at 512^2 (256),
// but 22.7 -> 29.2 at 1024^2 (1024).
constexpr int TOP_GROUPS = 4;

template <int TG>
constexpr int TOP_SMEM = TG * IDWT_SMEM;

template <int TG>
__device__ __forceinline__ void top_body(const IdwtArgs& A, const float* __restrict__ filt,
                                         const int* __restrict__ flen, int b, int nx, int ny, char* smem) {
  constexpr int PER = TS * TS / 2 / ST;  // output pairs per thread
  constexpr int ROUNDS = MAX_WAVELETS / TG;
  float4* sb0 = reinterpret_cast<float4*>(smem);
  const int grp = TG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / ST), tid = threadIdx.x % ST;
  float4* sb = sb0 + grp * (RS * RS);
  float2* lh = reinterpret_cast<float2*>(sb0 + TG * (RS * RS)) + grp * (TS * RS);
  int tx, ty;
  band_tile(b, nx, ny, tx, ty);
  const int p0 = ty * TS, q0 = tx * TS, n = A.n;
  auto wavelet = [&](int r) { return r * TG + (r % 2 == 0 ? grp : TG - 1 - grp); };
  // the Dirac basis' pixels that this thread stores
  constexpr int DIR = TG == 1 ? 2 * PER : 1;
  static_assert(TG == 1 || TS * TS == ST * TG, "one output per thread");
  auto pixel = [&](int k) {  // row << 16 | column, within the tile
    if (TG > 1) return (int(threadIdx.x) / TS) << 16 | int(threadIdx.x) % TS;
    const int idx = tid + (k / 2) * ST;
    return (idx / (TS / 2)) << 16 | (2 * (idx % (TS / 2)) + k % 2);
  };
  float dir[DIR];
#pragma unroll
  for (int k = 0; k < DIR; ++k) {
    const int p = p0 + (pixel(k) >> 16), q = q0 + (pixel(k) & 0xffff);
    dir[k] = A.dirac && p < n && q < n ? A.s[size_t(p) * n + q] : 0.f;
  }
  float2 val[TG == 1 ? 1 : ROUNDS][PER];  // the sums, or each of the group's wavelets
  if (TG == 1)
#pragma unroll
    for (int k = 0; k < PER; ++k) val[0][k] = make_float2(0.f, 0.f);
  Stage st;
  if (wavelet(0) < A.nw) {
    fetch_stage(A, wavelet(0), flen[wavelet(0)] / 2, p0, q0, tid, st);
    deposit_stage(flen[wavelet(0)] / 2, st, tid, sb);
  }
  __syncthreads();
  auto round = [&](int r, float2* v) {
    const int w = wavelet(r), wn = r + 1 < ROUNDS ? wavelet(r + 1) : A.nw;
    const int Hn = wn < A.nw ? flen[wn] / 2 : 0;
    if (wn < A.nw) fetch_stage(A, wn, Hn, p0, q0, tid, st);
    if (w < A.nw) {
      auto emit = [&](int k, int, int, float ve, float vo) {
        v[k] = TG == 1 ? make_float2(v[k].x + ve, v[k].y + vo) : make_float2(ve, vo);
      };
#define RI_SYNTH(LL) synthesis_staged<LL>(filt + w * FILT_STRIDE, sb, lh, tid, emit)
      RI_SWITCH_L(flen[w], RI_SYNTH)
#undef RI_SYNTH
    } else {
      __syncthreads();
    }
    if (wn < A.nw) deposit_stage(Hn, st, tid, sb);
    __syncthreads();
  };
  if constexpr (TG == 1) {
    for (int r = 0; r < A.nw; ++r) round(r, val[0]);
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) round(r, val[r]);
  }
  float* part = reinterpret_cast<float*>(sb0);  // [wavelet][row][column]
  if (TG > 1) {
    static_assert(TG == 1 || sizeof(float) * MAX_WAVELETS * TS * TS <= sizeof(float4) * TG * RS * RS, "the tiles take the place of sb");
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
      if (wavelet(r) < A.nw)
#pragma unroll
        for (int k = 0; k < PER; ++k)
          reinterpret_cast<float2*>(part + wavelet(r) * TS * TS)[tid + k * ST] = val[TG == 1 ? 0 : r][k];
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < DIR; ++k) {
    const int p = p0 + (pixel(k) >> 16), q = q0 + (pixel(k) & 0xffff);
    float acc = 0.f;
    if (TG == 1) acc = k % 2 == 0 ? val[0][k / 2].x : val[0][k / 2].y;
    else
      for (int w = 0; w < A.nw; ++w) acc += part[w * TS * TS + threadIdx.x];
    if (p < n && q < n) A.x[size_t(p) * n + q] = acc + dir[k];
  }
}

// The deep levels of one wavelet in one workgroup: every level whose input is at most DEEP x
// DEEP, from level e.first (2 or more) to the last, with the input, the filtered rows and the
// coefficients (in Mallat layout) in LDS.  Analysis with the dual clip, synthesis, or both
// without leaving LDS.  On such levels a launch per level costs more than its work: levels 2 to
// 4 of a 64^2 image took six launches of 3.1 to 5.2 us, and take 11 us together, most of them
// hidden behind the gridding whose launch they share (8.3 us by itself).
constexpr int DEEP_THREADS = 1024;
constexpr int DEEP_SMEM = 3 * DEEP * DEEP * 4;

template <int L, bool GATE>
__device__ __forceinline__ void deep_levels(const DeepArgs& E, const float* __restrict__ hw, int w, char* smem) {
  const float* __restrict__ gw = hw + MAX_TAPS;
  constexpr int H = L / 2;
  float* in = reinterpret_cast<float*>(smem);
  float2* lh = reinterpret_cast<float2*>(in + DEEP * DEEP);
  float* sc = reinterpret_cast<float*>(lh + DEEP * DEEP / 2);  // coefficients, rows DEEP apart
  const DwtArgs& A = E.a;
  const int n = A.n, m0 = n >> (E.first - 1), tid = threadIdx.x;
  float* sb = A.s + size_t(w + A.dirac) * n * n;
  float* ll0 = A.tmp + w * A.tmp_stride + E.ll_off;
  if (E.analyse ? A.clip != 0 : E.synth != 0)
    for (int k = tid; k < m0 * m0; k += DEEP_THREADS) sc[(k / m0) * DEEP + k % m0] = sb[size_t(k / m0) * n + k % m0];
  if (E.analyse) {
    for (int k = tid; k < m0 * m0; k += DEEP_THREADS) in[k] = ll0[k];
    for (int lev = E.first; lev <= A.levels; ++lev) {
      const int m = n >> (lev - 1), mo = m / 2, mm = m - 1;
      __syncthreads();
      for (int k = tid; k < m * mo; k += DEEP_THREADS) {
        const int r = k / mo, j = k - (k / mo) * mo;
        float a = 0.f, d = 0.f;
#pragma unroll
        for (int t = 0; t < L; ++t) {
          const float v = in[r * m + ((2 * j + t) & mm)];
          a = fmaf(hw[t], v, a);
          d = fmaf(gw[t], v, d);
        }
        lh[k] = make_float2(a, d);
      }
      __syncthreads();
      for (int k = tid; k < mo * mo; k += DEEP_THREADS) {
        const int qi = k / mo, qj = k - (k / mo) * mo;
        float c[4] = {0.f, 0.f, 0.f, 0.f};  // low-low, low-y/high-x, high-y/low-x, high-high
#pragma unroll
        for (int t = 0; t < L; ++t) {
          const float2 v = lh[((2 * qi + t) & mm) * mo + qj];
          c[0] = fmaf(hw[t], v.x, c[0]);
          c[1] = fmaf(hw[t], v.y, c[1]);
          c[2] = fmaf(gw[t], v.x, c[2]);
          c[3] = fmaf(gw[t], v.y, c[3]);
        }
        if (lev < A.levels) in[k] = c[0];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (b == 0 && lev < A.levels) continue;
          const int r = qi + (b >> 1) * mo, q = qj + (b & 1) * mo;
          const size_t o = size_t(r) * n + q, k = size_t(w + A.dirac) * n * n + o;
          const float v = new_coef<GATE>(A, A.clip ? sc[r * DEEP + q] : 0.f, A.clip ? clip_bound(A, k) : 0.f,
                                         GATE ? A.gate[k] : 0.f, c[b]);
          sb[o] = v;
          sc[r * DEEP + q] = v;
        }
      }
    }
  }
  if (E.synth) {
    for (int lev = A.levels; lev >= E.first; --lev) {
      const int m = n >> (lev - 1), mo = m / 2, mk = mo - 1;
      __syncthreads();
      for (int k = tid; k < mo * mo; k += DEEP_THREADS) {
        const int qy = k / mo, jl = k - (k / mo) * mo;
        float le = 0.f, lo = 0.f, he = 0.f, ho = 0.f;
#pragma unroll
        for (int u = 0; u < H; ++u) {
          const float* c = sc + ((qy - u) & mk) * DEEP + jl;
          const float c0 = c[0], c1 = c[mo], c2 = c[mo * DEEP], c3 = c[mo * DEEP + mo];
          le = fmaf(hw[2 * u], c0, fmaf(gw[2 * u], c2, le));
          lo = fmaf(hw[2 * u + 1], c0, fmaf(gw[2 * u + 1], c2, lo));
          he = fmaf(hw[2 * u], c1, fmaf(gw[2 * u], c3, he));
          ho = fmaf(hw[2 * u + 1], c1, fmaf(gw[2 * u + 1], c3, ho));
        }
        lh[(2 * qy) * mo + jl] = make_float2(le, he);
        lh[(2 * qy + 1) * mo + jl] = make_float2(lo, ho);
      }
      __syncthreads();
      for (int k = tid; k < m * mo; k += DEEP_THREADS) {
        const int p = k / mo, qx = k - (k / mo) * mo;
        float ve = 0.f, vo = 0.f;
#pragma unroll
        for (int u = 0; u < H; ++u) {
          const float2 c = lh[p * mo + ((qx - u) & mk)];
          ve = fmaf(hw[2 * u], c.x, fmaf(gw[2 * u], c.y, ve));
          vo = fmaf(hw[2 * u + 1], c.x, fmaf(gw[2 * u + 1], c.y, vo));
        }
        if (lev == E.first) {
          reinterpret_cast<float2*>(ll0 + p * m0)[qx] = make_float2(ve, vo);
        } else {
          sc[p * DEEP + 2 * qx] = ve;
          sc[p * DEEP + 2 * qx + 1] = vo;
        }
      }
    }
  }
}

template <bool GATE>
__device__ __forceinline__ void deep_body(const DeepArgs& E, const float* __restrict__ filt,
                                          const int* __restrict__ flen, int w, char* smem) {
#define RI_DEEP(LL) deep_levels<LL, GATE>(E, filt + w * FILT_STRIDE, w, smem)
  RI_SWITCH_L(flen[w], RI_DEEP)
#undef RI_DEEP
}

// A part of the sparsity branch as further workgroups of another kernel's launch (SideJob).
// THREADS: that kernel's workgroup size, which decides the kinds it can hold.
template <int THREADS>
constexpr int side_smem() {
  return THREADS == ST ? (DWT_SMEM > IDWT_SMEM ? DWT_SMEM : IDWT_SMEM)
                       : (DEEP_SMEM > TOP_SMEM<TOP_GROUPS> ? DEEP_SMEM : TOP_SMEM<TOP_GROUPS>);
}

template <int THREADS, int KIND>
__device__ __forceinline__ void side_body(const SideJob& j, int b, char* smem) {
  static_assert((KIND == SIDE_DWT || KIND == SIDE_DWT_GATE || KIND == SIDE_IDWT) == (THREADS == ST),
                "the job's workgroup size");
  if constexpr (KIND == SIDE_DWT || KIND == SIDE_DWT_GATE)
    dwt_body<KIND == SIDE_DWT_GATE>(j.a, j.filt, j.flen, b, j.nx, j.ny, smem);
  if constexpr (KIND == SIDE_IDWT) idwt_body(j.i, j.filt, j.flen, b, j.nx, j.ny, smem);
  if constexpr (KIND == SIDE_DEEP || KIND == SIDE_DEEP_GATE)
    deep_body<KIND == SIDE_DEEP_GATE>(j.e, j.filt, j.flen, b, smem);
  if constexpr (KIND == SIDE_TOP) top_body<TOP_GROUPS>(j.i, j.filt, j.flen, b, j.nx, j.ny, smem);
}

}  // namespace ri
