// Measurement-operator plan and the Phi / Phi^dagger entry points (Eq. 3, Eq. 8).
//
// Plan creation:
//   * each u-v coordinate becomes kappa = u K / (2 pi) wrapped to [0, K), stored as a
//     12-bit cell plus a 20-bit fraction (position error <= 2^-21 cell, i.e. < 1e-6 rad of
//     phase at the image edge), in FP64 on the device (plan_sort.hip);
//   * the visibilities are sorted by (block, grid tile, cell) on the device, and inside each
//     block cut on the host into work items of at most `bin` visibilities of one tile;
//   * Kaiser-Bessel weights are fitted per tap by degree-7 polynomials (Chebyshev
//     interpolation of the kernel evaluated with an I0 power series);
//   * twiddles exp(-2 pi i k / K) and the pre-compensation S = 1/phi_hat(l/K) are
//     evaluated in FP64 and rounded to FP32.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>
#include <thread>
#include <vector>

#include "host_math.hpp"
#include "handles.hpp"

namespace ri {
namespace {

// Bound by its random 8-byte accesses: the plan moves a visibility only inside its block, so
// each XCD is given a contiguous run of chunks (the dispatcher deals consecutive workgroups
// round-robin over the eight XCDs), and the lines that a block's scattered accesses share meet
// in one L2; each thread keeps four of them in flight.  M = 2^22
// in 64 blocks, plan to user order: 61 us (one per thread, any XCD, 8-byte indices) -> 31 us.
constexpr int PERM_CHUNK = 1024, PERM_XCDS = 8;

template <bool TO_PLAN>
__global__ __launch_bounds__(256) void k_permute(const float2* __restrict__ src, float2* __restrict__ dst,
                                                 const int* __restrict__ order, int64_t M, int per_xcd) {
  const int64_t chunk = int64_t(blockIdx.x % PERM_XCDS) * per_xcd + blockIdx.x / PERM_XCDS;
  const int64_t k0 = chunk * PERM_CHUNK + threadIdx.x;
  if (k0 >= M) return;
  int o[4];
  float2 v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) o[j] = k0 + j * 256 < M ? order[k0 + j * 256] : 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (k0 + j * 256 >= M) continue;
    v[j] = src[TO_PLAN ? int64_t(o[j]) : k0 + j * 256];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (k0 + j * 256 >= M) continue;
    dst[TO_PLAN ? k0 + j * 256 : int64_t(o[j])] = v[j];
  }
}

__global__ void k_copy_f32(const float* __restrict__ a, float* __restrict__ b, size_t n) {
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    b[i] = a[i];
}

void destroy_plan(Plan& p) {
  dev_free(p.coord);
  dev_free(p.order);
  dev_free(p.items);
  dev_free(p.item_box);
  dev_free(p.item_pairs);
  dev_free(p.item_off);
  dev_free(p.block_off);
  dev_free(p.twiddle);
  dev_free(p.scale);
  dev_free(p.grid);
  dev_free(p.rowbuf);
  dev_free(p.titems);
  dev_free(p.units);
  dev_free(p.bunits);
  dev_free(p.dunits);
  dev_free(p.unit_patch);
  dev_free(p.tile_sp_off);
  dev_free(p.tile_sp);
  dev_free(p.spatch);
  dev_free(p.item_part);
  dev_free(p.block_tmp);
  dev_free(p.halo);
  dev_free(p.empty_tiles);
  dev_free(p.wslots);
  dev_free(p.woff);
  dev_free(p.wsegs);
  dev_free(p.wsplit);
  dev_free(p.xpatch);
  dev_free(p.bslots);
  dev_free(p.bwoff);
  dev_free(p.bsegs);
  dev_free(p.patch);
  dev_free(p.norm_tmp);
  dev_free(p.dsum);
  dde_destroy(p.dde);
}

template <class T>
int upload(T** dst, const std::vector<T>& src, hipStream_t s) {
  RI_TRY(dev_alloc(dst, src.size()));
  if (!src.empty()) RI_HIP(hipMemcpyAsync(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice, s));
  return RI_OK;
}

using KV = std::pair<uint64_t, int64_t>;  // (tile << 32 | tile-local cell ly * T + lx, index)

// Reorders a list of visibilities (or of same-cell pairs, by their first member) so that
// every 64 consecutive ones, which one wavefront processes together, spread their
// staged-tile addresses ly * (T + TILE_PAD) + lx evenly over the LDS banks: they are dealt
// round-robin from one queue per bank (32 banks of 8-byte words).
template <class E, class Key>
void lds_bank_order(std::vector<E>& v, int T, Key key) {
  constexpr int NB = 32;
  std::vector<E> q[NB];
  for (const E& e : v) {
    const uint32_t local = uint32_t(key(e));
    const uint32_t ly = local / T, lx = local % T;
    q[(ly * uint32_t(T + TILE_PAD) + lx) % NB].push_back(e);
  }
  size_t head[NB] = {}, out = 0;
  while (out < v.size())
    for (int b = 0; b < NB; ++b)
      if (head[b] < q[b].size()) v[out++] = q[b][head[b]++];
}

// Orders the w visibilities of one work item (sorted by tile-local cell) for the kernels.
// Thread t of a gridding workgroup takes positions t + k GRID_LANES, k = 0 .. MAX_BIN /
// GRID_LANES - 1, and treats slots 2j and 2j + 1 as a pair when t < P_j: two visibilities
// of the same cell whose 64 taps it adds with one atomic each.  Same-cell visibilities are
// paired greedily, and the pairs are placed at positions (t + 2j L, t + (2j + 1) L), t < P_j,
// where L = GRID_LANES and P_j is as many whole wavefronts (64) of pairs as fit; the rest
// (odd members and pairs that do not fit) fill the other positions as singles.  Pairs and singles are each dealt over the LDS
// banks.  Returns P_0 | P_1 << 16.
uint32_t item_order(KV* kv, int64_t w, int T) {
  constexpr int L = GRID_LANES;
  static_assert(MAX_BIN == 4 * L, "two slot pairs per thread");
  std::vector<std::pair<KV, KV>> pairs;
  std::vector<KV> singles;
  for (int64_t k = 0; k < w;) {
    int64_t e = k;
    while (e < w && uint32_t(kv[e].first) == uint32_t(kv[k].first)) ++e;
    for (; k + 1 < e; k += 2) pairs.push_back({kv[k], kv[k + 1]});
    if (k < e) singles.push_back(kv[k++]);
  }
  const int64_t cap0 = std::clamp<int64_t>(w - L, 0, L), cap1 = std::clamp<int64_t>(w - 3 * L, 0, L);
  // whole wavefronts of pairs, so that no wavefront runs both the pair and the single path
  const int64_t p0 = std::min<int64_t>(int64_t(pairs.size()), cap0) / 64 * 64;
  const int64_t p1 = std::min<int64_t>(int64_t(pairs.size()) - p0, cap1) / 64 * 64;
  for (size_t j = size_t(p0 + p1); j < pairs.size(); ++j) {
    singles.push_back(pairs[j].first);
    singles.push_back(pairs[j].second);
  }
  pairs.resize(size_t(p0 + p1));
  lds_bank_order(pairs, T, [](const std::pair<KV, KV>& e) { return e.first.first; });
  lds_bank_order(singles, T, [](const KV& e) { return e.first; });
  std::vector<KV> out(w);
  std::vector<char> used(w, 0);
  for (int64_t j = 0; j < p0 + p1; ++j) {
    const int64_t a = j < p0 ? j : 2 * L + (j - p0);
    out[a] = pairs[j].first;
    out[a + L] = pairs[j].second;
    used[a] = used[a + L] = 1;
  }
  size_t next = 0;
  for (int64_t a = 0; a < w; ++a)
    if (!used[a]) out[a] = singles[next++];
  std::copy(out.begin(), out.end(), kv);
  return uint32_t(p0) | uint32_t(p1) << 16;
}

// Fourier transform at f of the kernel that the tap polynomials make up: tap j at distance
// t = g + 3 - j, g in [0, 1), weighs E_j(x^2) + x O_j(x^2), x = 2 g - 1, and tap 7 - j the
// mirrored value, so the pair contributes 2 w cos(2 pi f t).  Gauss-Legendre on 12 nodes:
// exact for degree 23, the integrand's degree 7 times a cosine of less than pi / 2 per unit.
double poly_hat(const KBPoly& P, double f) {
  static const double node[6] = {0.1252334085114689, 0.3678314989981802, 0.5873179542866175,
                                 0.7699026741943047, 0.9041172563704749, 0.9815606342467193};
  static const double weight[6] = {0.2491470458134028, 0.2334925365383548, 0.2031674267230659,
                                   0.1600783285433462, 0.1069393259953184, 0.0471753363865118};
  double sum = 0.0;
  for (int j = 0; j < KB_J / 2; ++j)
    for (int k = 0; k < 12; ++k) {
      const double x = k < 6 ? node[k] : -node[k - 6], x2 = x * x;
      double e = P.e[j][KB_HALF_DEG], o = P.o[j][KB_HALF_DEG];
      for (int q = KB_HALF_DEG - 1; q >= 0; --q) {
        e = e * x2 + P.e[j][q];
        o = o * x2 + P.o[j][q];
      }
      const double t = 0.5 * (x + 1.0) + (KB_J / 2 - 1) - j;
      sum += weight[k % 6] * 0.5 * 2.0 * (e + x * o) * std::cos(2.0 * M_PI * f * t);
    }
  return sum;
}

// Four wavefronts per window up to this many tiles.  Per launch with 1, 2 and 4: 12.2, 9.1, 8.5 us at
// 64^2 (64 tiles), 24.4, 17.8, 16.1 at 256^2 (1024), 25.9, 26.8, 57.3 at 512^2 (4096): on the larger
// grids the tiles fill the chip by themselves (one workgroup of 16 wavefronts per CU, by its LDS, is
// 1024 windows at once), and the split only adds wavefronts without work.
constexpr int WIN_SPLIT_TILES = 1024;

// Host copies of a windowed plan's gridding lists (Plan::wslots and the following).
struct WinLists {
  std::vector<int> slots, woff, bslots, bwoff, block_off;
  std::vector<int4> segs, bsegs, split;
};

// The units of the windowed gridding over all blocks, and each block's own.  A tile of 16 x 16 cells is
// one unit, or P of them, each with the P-th part of each window's visibilities (blocks in order,
// segments cut where a part ends): a window is the work of one to four wavefronts, which take 0.78 us
// per 32 visibilities one after the other, so that a dense window alone decides the launch's time.
// P is the least that leaves a window 1024 visibilities for one wavefront or 2048 for four (25 and 13
// us; less costs ordinary coverages the merging, 5 us: a dirty image of 1.5 10^6 visibilities at 512^2
// takes 64.7 us, with 768 65.6, with 512 69.8; with 4096 for four, 1.3 10^6 at 256^2 take 54 us instead
// of 44) or win_split M / 4096, its share if the windows that the chip holds at once (1024 of four
// wavefronts) had the same; and at least what slice_vis asks for, where that does not cut finer than
// the tile's work items.  Gridding 2^20 visibilities of a Gaussian of 16 cells at 512^2: 958 -> 47 us
// (tiles of 32 x 32 cells 4118, sliced by 4096 328), of 3 cells 6316 -> 70; 2^18 of 16 cells at 256^2
// 122 -> 35.
void window_lists(const std::vector<std::vector<int4>>& block_segs, const Plan& p, int64_t M, WinLists& out) {
  const int d = int(block_segs.size());
  // segments by tile and window, blocks in order
  std::vector<int> off(4 * size_t(p.n_gtiles) + 1, 0);
  for (const auto& v : block_segs)
    for (const int4& sg : v) off[sg.w + 1] += 1;
  for (size_t q = 0; q + 1 < off.size(); ++q) off[q + 1] += off[q];
  std::vector<int4> segs(off.back());
  std::vector<int> fill(off.begin(), off.end() - 1);
  out.block_off.assign(1, 0);
  out.bwoff.assign(1, 0);
  out.bsegs.reserve(segs.size());
  for (const auto& v : block_segs) {
    for (size_t k = 0; k < v.size();) {
      const int t = v[k].w / 4;
      out.bslots.push_back(t);
      for (int w = 0; w < 4; ++w) {
        for (; k < v.size() && v[k].w == 4 * t + w; ++k) {
          segs[fill[v[k].w]++] = v[k];
          out.bsegs.push_back(v[k]);
        }
        out.bwoff.push_back(int(out.bsegs.size()));
      }
    }
    out.block_off.push_back(int(out.bslots.size()));
  }
  struct Unit {
    int slot;
    int64_t vis;
    int off[5];  // ranges of `parts`
  };
  std::vector<Unit> units;
  std::vector<int4> parts;
  parts.reserve(segs.size());
  const int64_t most = std::max<int64_t>(p.win_split == 1 ? 1024 : 2048, p.win_split * (M / 4096));
  int extra = 0;
  for (int t = 0; t < p.n_gtiles; ++t) {
    int64_t vis = 0, P = 1, items = 0, in_block = 0, count[4];
    for (int w = 0; w < 4; ++w) {
      count[w] = 0;
      for (int k = off[4 * t + w]; k < off[4 * t + w + 1]; ++k) count[w] += segs[k].y;
      vis += count[w];
      P = std::max(P, (count[w] + most - 1) / most);
    }
    if (p.slice_vis > 0 && vis > p.slice_vis) {
      std::vector<std::pair<int, int64_t>> blocks;  // the tile's visibilities by block
      for (int k = off[4 * t]; k < off[4 * t + 4]; ++k) blocks.push_back({segs[k].z, segs[k].y});
      std::sort(blocks.begin(), blocks.end());
      for (size_t k = 0; k < blocks.size(); ++k) {
        in_block += blocks[k].second;
        if (k + 1 < blocks.size() && blocks[k + 1].first == blocks[k].first) continue;
        items += (in_block + p.bin - 1) / p.bin;
        in_block = 0;
      }
      P = std::max(P, std::min(items, (vis + p.slice_vis - 1) / p.slice_vis));
    }
    if (P > 1) out.split.push_back(make_int4(t, extra, int(P - 1), 0));
    int at[4];
    int64_t used[4] = {0, 0, 0, 0};  // of segment at[w]
    for (int w = 0; w < 4; ++w) at[w] = off[4 * t + w];
    for (int64_t k = 0; k < P; ++k) {
      Unit u{k == 0 ? t : p.n_gtiles + extra++, 0, {int(parts.size()), 0, 0, 0, 0}};
      for (int w = 0; w < 4; ++w) {
        int64_t left = count[w] * (k + 1) / P - count[w] * k / P;
        u.vis += left;
        while (left > 0) {
          const int4 sg = segs[at[w]];
          const int64_t n = std::min<int64_t>(left, sg.y - used[w]);
          parts.push_back(make_int4(int(sg.x + used[w]), int(n), sg.z, 0));
          left -= n;
          used[w] += n;
          if (used[w] == sg.y) {
            ++at[w];
            used[w] = 0;
          }
        }
        u.off[w + 1] = int(parts.size());
      }
      units.push_back(u);
    }
  }
  // most visibilities first: the dispatcher hands freed slots the next one
  std::stable_sort(units.begin(), units.end(), [](const Unit& l, const Unit& r) { return l.vis > r.vis; });
  out.woff.assign(1, 0);
  out.segs.reserve(parts.size());
  for (const Unit& u : units) {
    out.slots.push_back(u.slot);
    for (int w = 0; w < 4; ++w) {
      out.segs.insert(out.segs.end(), parts.begin() + u.off[w], parts.begin() + u.off[w + 1]);
      out.woff.push_back(int(out.segs.size()));
    }
  }
}

int create_plan(Plan& p, int n, int64_t M, const float* uv, int d, const int64_t* off, int J, double beta,
                const ri_tuning* tune, hipStream_t s) {
  if (!is_pow2(n) || n < 16 || n > 2048) return fail(RI_EINVAL, "n=%d must be a power of two in [16, 2048]", n);
  if (M < 1 || M > (int64_t(1) << 31) - 1) return fail(RI_EINVAL, "M=%lld out of range", (long long)M);
  if (d < 1 || d > 4096) return fail(RI_EINVAL, "d=%d must be in [1, 4096]", d);
  if (!uv || !off) return fail(RI_EINVAL, "uv and block_off must not be NULL");
  if (J != KB_J) return fail(RI_EINVAL, "only J=%d is supported (got %d)", KB_J, J);
  if (off[0] != 0 || off[d] != M) return fail(RI_EINVAL, "block_off must start at 0 and end at M");
  for (int i = 0; i < d; ++i)
    if (off[i + 1] <= off[i]) return fail(RI_EINVAL, "block %d is empty or offsets decrease", i);
  for (int64_t m = 0; m < 2 * M; ++m)
    if (!std::isfinite(uv[m])) return fail(RI_EINVAL, "non-finite u-v coordinate at %lld", (long long)(m / 2));

  p.n = n;
  p.K = 2 * n;
  p.M = M;
  p.d = d;
  p.J = J;
  p.beta = beta > 0 ? beta : 2.34 * J;
  p.tile = tune && tune->tile ? tune->tile : 32;
  if (p.tile != 16 && p.tile != 32 && p.tile != 64) return fail(RI_EINVAL, "tile must be 16, 32 or 64");
  // gridding phases need two tiles per axis at least (same-colour tiles must not touch)
  while (p.tile > 16 && p.tile > p.K / 2) p.tile /= 2;
  p.bin = tune && tune->bin > 0 ? tune->bin : MAX_BIN;
  if (p.bin > MAX_BIN) return fail(RI_EINVAL, "bin=%d exceeds %d", p.bin, MAX_BIN);
  if (tune && tune->fft_panel != 0) return fail(RI_EINVAL, "fft_panel is reserved and must be 0");
  p.fft_panel = 0;
  p.persistent_wgs = tune ? tune->persistent_wgs : 0;
  p.slice_vis = tune && tune->slice_vis != 0 ? tune->slice_vis : -1;
  p.tpa = p.K / p.tile;
  p.windowed = p.K <= WINDOWED_K;
  p.block_off_host.assign(off, off + d + 1);

  // Kaiser-Bessel polynomials
  std::vector<double> mono;
  kb_fit_taps(J, p.beta, 2 * KB_HALF_DEG + 1, mono, &p.poly_err);
  if (!(p.poly_err < 2e-7)) return fail(RI_EINVAL, "kernel polynomial fit error %.3g too large (beta %.3f)", p.poly_err, p.beta);
  for (int j = 0; j < KB_J / 2; ++j)
    for (int k = 0; k <= KB_HALF_DEG; ++k) {
      p.poly.e[j][k] = float(mono[size_t(j) * (2 * KB_HALF_DEG + 2) + 2 * k]);
      p.poly.o[j][k] = float(mono[size_t(j) * (2 * KB_HALF_DEG + 2) + 2 * k + 1]);
    }

  // coordinates and the sort on the device (plan_sort), then the work items of each block
  // on the host (blocks are independent: one host thread each)
  const int K = p.K, T = p.tile, tpa = p.tpa;
  uint2* packed = nullptr;  // M packed coordinates, user order (device)
  std::vector<uint64_t> skeys;
  std::vector<int> sidx;
  RI_TRY(plan_sort(uv, M, off, d, K, T, tpa, p.windowed, &packed, skeys, sidx, s));
  struct Freer {
    uint2*& q;
    ~Freer() { dev_free(q); }
  } free_packed{packed};
  p.order_host.resize(M);
  std::vector<std::vector<Item>> block_items(d);
  std::vector<std::vector<uint32_t>> block_pairs(d), block_boxes(d);
  // {first position, count, block, 4 gridding tile + its window}, by the last
  std::vector<std::vector<int4>> block_segs(d);
  // Windowed plans keep the sorted order, which the gridding's windows need; pairs and bank dealing
  // inside their items would save the degridding 6 % where a cell holds a dozen visibilities of one
  // block (27.8 -> 26.6 us at 1.5 10^6, 512^2) and nothing on sparser ones.  Their degridding items are cut smaller where M would
  // not give every CU four workgroups (8192 visibilities at 64^2: 14.8 us with items of up to
  // 1024 and units of 2048, 4.7 with 256 and 256), unless the (block, tile) runs alone may come
  // near the count of items that the norms' scratch allows.
  const int wpt = T / WIN;
  int64_t kbin = p.bin, dunit_vis = DUNIT_VIS;
  if (p.windowed && int64_t(d) * tpa * tpa <= 32768) {
    dunit_vis = std::clamp<int64_t>((M / 1024 + 255) / 256 * 256, DUNIT_VIS_MIN, DUNIT_VIS);
    kbin = std::min(kbin, dunit_vis);
  }
  std::atomic<int> items_info{0};
  std::atomic<int> bad{0};
  const unsigned nthreads = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
  auto work = [&](int i) {
    const int64_t lo = off[i], hi = off[i + 1];
    std::vector<KV> kv(hi - lo);
    for (int64_t k = lo; k < hi; ++k) {
      const uint64_t key = skeys[k];
      if (int64_t(key >> 28) != i) bad = 1;  // the sort keeps the blocks where they are
      kv[k - lo] = {(((key >> 12) & 0xFFFFu) << 32) | (key & 0xFFFu), int64_t(sidx[k])};
    }
    auto& its = block_items[i];
    auto& prs = block_pairs[i];
    auto& bxs = block_boxes[i];
    int64_t k = 0;
    while (k < hi - lo) {
      const uint64_t tile = kv[k].first >> 32;
      int64_t e = k;
      while (e < hi - lo && (kv[e].first >> 32) == tile) ++e;
      items_info += int((e - k + p.bin - 1) / p.bin);
      for (int64_t a = k; a < e; a += kbin) {
        const int64_t w = std::min<int64_t>(kbin, e - a);
        if (!p.windowed) {
          // footprint box: the item's smallest and largest tile-local row and column
          int b[4] = {T, -1, T, -1};
          for (int64_t m = a; m < a + w; ++m) {
            const int local = int(uint32_t(kv[m].first)), ly = local / T, lx = local % T;
            b[0] = std::min(b[0], ly);
            b[1] = std::max(b[1], ly);
            b[2] = std::min(b[2], lx);
            b[3] = std::max(b[3], lx);
          }
          bxs.push_back(uint32_t(b[0]) | uint32_t(b[1]) << 8 | uint32_t(b[2]) << 16 | uint32_t(b[3]) << 24);
          prs.push_back(item_order(kv.data() + a, w, T));
        } else {
          prs.push_back(0);  // no same-cell pairs are placed
        }
        its.push_back(make_int4(i, int(tile), int(lo + a), int(w)));
      }
      for (int64_t a = k; p.windowed && a < e;) {  // one segment per window
        const int sub = int(uint32_t(kv[a].first) >> 6);
        int64_t z = a + 1;
        while (z < e && int(uint32_t(kv[z].first) >> 6) == sub) ++z;
        const int wy = int(tile) / tpa * wpt + sub / wpt, wx = int(tile) % tpa * wpt + sub % wpt;
        block_segs[i].push_back(make_int4(int(lo + a), int(z - a), i,
                                          4 * ((wy / 2) * (K / GSIDE) + wx / 2) + (wy % 2) * 2 + wx % 2));
        a = z;
      }
      k = e;
    }
    std::sort(block_segs[i].begin(), block_segs[i].end(), [](const int4& l, const int4& r) { return l.w < r.w; });
    for (int64_t k = 0; k < hi - lo; ++k) p.order_host[lo + k] = int(kv[k].second);
  };
  {
    std::vector<std::thread> th;
    std::atomic<int> next{0};
    for (unsigned t = 0; t < nthreads; ++t)
      th.emplace_back([&] {
        for (int i = next++; i < d; i = next++) work(i);
      });
    for (auto& t : th) t.join();
  }
  if (bad) return fail(RI_EHIP, "device sort returned visibilities outside their block");
  std::vector<Item> items;
  std::vector<uint32_t> item_pairs, item_box;
  p.item_off_host.assign(d + 1, 0);
  for (int i = 0; i < d; ++i) {
    p.item_off_host[i] = int(items.size());
    items.insert(items.end(), block_items[i].begin(), block_items[i].end());
    item_pairs.insert(item_pairs.end(), block_pairs[i].begin(), block_pairs[i].end());
    item_box.insert(item_box.end(), block_boxes[i].begin(), block_boxes[i].end());
  }
  p.item_off_host[d] = int(items.size());
  p.n_items = int(items.size());
  p.n_items_info = items_info;

  WinLists win;
  if (p.windowed) {
    p.gta = K / GSIDE;
    p.n_gtiles = p.gta * p.gta;
    p.win_split = p.n_gtiles <= WIN_SPLIT_TILES ? 4 : 1;
    window_lists(block_segs, p, M, win);
    p.n_wunits = int(win.slots.size());
    p.n_wsplit = int(win.split.size());
    p.bwoff_host = win.block_off;
  }

  // items grouped by tile, and tiles grouped into the four gridding colours
  p.n_tiles = tpa * tpa;
  std::vector<int> tile_cnt(p.n_tiles + 1, 0), tile_vis(p.n_tiles, 0);
  for (const Item& it : items) {
    tile_cnt[it.y + 1] += 1;
    tile_vis[it.y] += it.w;
  }
  for (int t = 0; t < p.n_tiles; ++t) tile_cnt[t + 1] += tile_cnt[t];
  std::vector<int> tile_items(items.size()), fill(tile_cnt.begin(), tile_cnt.end() - 1);
  for (int k = 0; k < int(items.size()); ++k) tile_items[fill[items[k].y]++] = k;
  std::vector<int> empty_tiles;
  for (int t = 0; t < p.n_tiles; ++t)
    if (tile_vis[t] == 0) empty_tiles.push_back(t);
  p.n_empty = int(empty_tiles.size());
  std::vector<int4> units, bunits;
  {
    std::vector<int> ts;
    for (int t = 0; t < p.n_tiles; ++t)
      if (tile_vis[t] > 0) ts.push_back(t);
    std::stable_sort(ts.begin(), ts.end(), [&](int a, int b) { return tile_vis[a] > tile_vis[b]; });
    for (int t : ts) units.push_back(make_int4(t, tile_cnt[t], tile_cnt[t + 1], tile_vis[t]));
  }
  p.tile_units_host = units;
  p.titem_vis_host.clear();
  for (int k : tile_items) p.titem_vis_host.push_back(items[k].w);
  if (p.windowed) {  // none of what follows but the degridding units
    units.clear();
    empty_tiles.clear();
    p.n_empty = 0;
  }
  // split dense tiles into slices of whole items
  std::vector<int> unit_patch;
  std::vector<std::vector<int>> tile_patches(p.n_tiles);
  {
    std::vector<int4> sliced;
    for (const int4& un : units) {
      if (p.slice_vis <= 0 || un.w <= p.slice_vis) {
        sliced.push_back(un);
        unit_patch.push_back(-1);
        continue;
      }
      int a = un.y, acc = 0;
      bool first = true;
      auto emit = [&](int e) {
        sliced.push_back(make_int4(un.x, a, e, acc));
        if (first) {
          unit_patch.push_back(-1);
        } else {
          tile_patches[un.x].push_back(p.n_spatch);
          unit_patch.push_back(p.n_spatch++);
        }
        first = false;
      };
      for (int q = un.y; q < un.z; ++q) {
        const int w = items[tile_items[q]].w;
        if (q > a && acc + w > p.slice_vis) {
          emit(q);
          a = q;
          acc = 0;
        }
        acc += w;
      }
      emit(un.z);
    }
    // densest first
    std::vector<int> idx(sliced.size());
    for (size_t k = 0; k < idx.size(); ++k) idx[k] = int(k);
    std::stable_sort(idx.begin(), idx.end(), [&](int l, int r) { return sliced[l].w > sliced[r].w; });
    units.clear();
    std::vector<int> up;
    for (int k : idx) {
      units.push_back(sliced[k]);
      up.push_back(unit_patch[k]);
    }
    unit_patch.swap(up);
  }
  std::vector<int> tile_sp_off(p.n_tiles + 1, 0), tile_sp;
  for (int t = 0; t < p.n_tiles; ++t) {
    tile_sp_off[t + 1] = tile_sp_off[t] + int(tile_patches[t].size());
    tile_sp.insert(tile_sp.end(), tile_patches[t].begin(), tile_patches[t].end());
  }
  p.n_units = int(units.size());
  std::vector<int4> dunits;
  for (const int4& un : p.windowed ? p.tile_units_host : units) {
    int a = un.y, acc = 0;
    for (int q = un.y; q < un.z; ++q) {
      const int w = items[tile_items[q]].w;
      if (q > a && acc + w > dunit_vis) {
        dunits.push_back(make_int4(un.x, a, q, acc));
        a = q;
        acc = 0;
      }
      acc += w;
    }
    dunits.push_back(make_int4(un.x, a, un.z, acc));
  }
  // The longest first, so that none starts when the others are done.  An item costs a windowed plan's
  // unit as long as some hundreds of visibilities do (its loads), so that a sparse tile with a few
  // visibilities of each block is among the longest: by visibilities alone such tiles came last, and the
  // launch took 27.7 us (6 visibilities per pixel at 256^2, 16 blocks over the whole plane), 37.4 (20 per
  // pixel), 40.7 (3.8 at 512^2); so 22.1, 30.9, 35.3, with 256 per item as with 1024.  The finer units of
  // windowed plans (dunit_vis) are what leaves such tails: other plans' order is by visibilities.
  const int item_cost = p.windowed ? 1024 : 0;
  auto unit_cost = [&](const int4& u) { return int64_t(u.w) + int64_t(item_cost) * (u.z - u.y); };
  std::stable_sort(dunits.begin(), dunits.end(),
                   [&](const int4& l, const int4& r) { return unit_cost(l) > unit_cost(r); });
  p.n_dunits = int(dunits.size());
  {
    // XCD-aware order of the degridding units.  The dispatcher deals consecutive
    // workgroups round-robin over the eight XCDs, and a dense tile has several units, each
    // staging the same tile and reach: the tiles are dealt to the XCDs in density order and
    // all units of a tile are placed at positions equal modulo 8, so that their stagings hit
    // the one XCD's L2.  Gaps (XCDs with fewer units) hold empty units.
    constexpr int NX = 8;
    std::vector<std::vector<int4>> per_xcd(NX);
    std::vector<int> tile_xcd(p.n_tiles, -1);
    int next = 0;
    if (p.windowed)  // in density order also where the units' order is another
      for (const int4& un : p.tile_units_host) tile_xcd[un.x] = next++ % NX;
    for (int k = 0; k < p.n_dunits; ++k) {
      int& x = tile_xcd[dunits[k].x];
      if (x < 0) x = next++ % NX;
      per_xcd[x].push_back(dunits[k]);
    }
    size_t L = 0;
    for (const auto& v : per_xcd) L = std::max(L, v.size());
    std::vector<int4> ordered(L * NX, make_int4(0, 0, 0, 0));
    for (int x = 0; x < NX; ++x)
      for (size_t j = 0; j < per_xcd[x].size(); ++j) ordered[j * NX + x] = per_xcd[x][j];
    dunits.swap(ordered);
    p.n_dunits = int(dunits.size());
  }
  p.bunit_off_host.assign(size_t(d) + 1, 0);
  for (int i = 0; i < d; ++i) {
    p.bunit_off_host[i] = int(bunits.size());
    for (int k = p.item_off_host[i]; k < p.item_off_host[i + 1];) {
      int e = k, vis = 0;
      while (e < p.item_off_host[i + 1] && items[e].y == items[k].y) vis += items[e++].w;
      bunits.push_back(make_int4(items[k].y, k, e, vis));
      k = e;
    }
  }
  p.bunit_off_host[d] = int(bunits.size());
  // device copies: y = index in block order
  std::vector<Item> items_dev(items), titems(items.size());
  for (size_t k = 0; k < items.size(); ++k) items_dev[k].y = int(k);
  for (size_t q = 0; q < items.size(); ++q) titems[q] = items_dev[tile_items[q]];

  std::vector<float2> tw(K);
  for (int k = 0; k < K; ++k) {
    const double a = -2.0 * M_PI * k / K;
    tw[k] = make_float2(float(std::cos(a)), float(std::sin(a)));
  }
  std::vector<float> sc(n);
  // Windowed plans take the transform of the kernel that is evaluated, its FP32 coefficients
  // included: their rounding alone (3e-8 of the weights, the same for every visibility) would
  // scale Phi, and through many iterations decide the error of gradients.  Larger grids keep the
  // closed form and with it the results they had: no gradient is measured there that would show it.
  for (int r = 0; r < n; ++r) {
    const double f = double(r - n / 2) / K;
    sc[r] = float(1.0 / (p.windowed ? poly_hat(p.poly, f) : kb_hat(f, J, p.beta)));
  }

  RI_TRY(dev_alloc(&p.coord, M));
  RI_TRY(upload(&p.order, p.order_host, s));
  RI_TRY(plan_gather_coord(packed, p.order, M, p.coord, s));
  RI_TRY(upload(&p.items, items_dev, s));
  RI_TRY(upload(&p.titems, titems, s));
  RI_TRY(upload(&p.item_box, item_box, s));
  RI_TRY(upload(&p.item_pairs, item_pairs, s));
  RI_TRY(upload(&p.item_off, p.item_off_host, s));
  RI_TRY(upload(&p.block_off, p.block_off_host, s));
  RI_TRY(upload(&p.twiddle, tw, s));
  RI_TRY(upload(&p.scale, sc, s));
  RI_TRY(upload(&p.units, units, s));
  RI_TRY(upload(&p.bunits, bunits, s));
  RI_TRY(upload(&p.dunits, dunits, s));
  RI_TRY(upload(&p.unit_patch, unit_patch, s));
  RI_TRY(upload(&p.tile_sp_off, tile_sp_off, s));
  RI_TRY(upload(&p.tile_sp, tile_sp, s));
  RI_TRY(upload(&p.empty_tiles, empty_tiles, s));
  RI_TRY(upload(&p.wslots, win.slots, s));
  RI_TRY(upload(&p.woff, win.woff, s));
  RI_TRY(upload(&p.wsegs, win.segs, s));
  RI_TRY(upload(&p.wsplit, win.split, s));
  RI_TRY(upload(&p.bslots, win.bslots, s));
  RI_TRY(upload(&p.bwoff, win.bwoff, s));
  RI_TRY(upload(&p.bsegs, win.bsegs, s));
  RI_TRY(dev_alloc(&p.grid, size_t(K) * K));
  RI_TRY(dev_alloc(&p.rowbuf, size_t(n) * K));
  if (p.n_spatch > 0) RI_TRY(dev_alloc(&p.spatch, size_t(p.n_spatch) * (p.tile + 8) * (p.tile + 8)));
  RI_TRY(dev_alloc(&p.item_part, 2 * size_t(PART_WAVES) * items.size()));
  RI_TRY(dev_alloc(&p.block_tmp, 2 * size_t(d)));
  RI_TRY(dev_alloc(&p.norm_tmp, size_t(n) * n));
  RI_TRY(dev_alloc(&p.dsum, SUMSQ_SCRATCH));
  if (p.windowed) {
    RI_TRY(dev_alloc(&p.patch, p.adj_cells()));
    RI_TRY(dev_alloc(&p.xpatch, size_t(p.n_wunits - p.n_gtiles) * PATCH_CELLS));
  } else {
    // tiles without visibilities keep an all-zero halo patch forever
    RI_TRY(dev_alloc(&p.halo, size_t(p.n_tiles) * ring_cells(p.tile)));
    RI_TRY(zero_c64(p.halo, size_t(p.n_tiles) * ring_cells(p.tile), s));
  }
  RI_HIP(hipStreamSynchronize(s));
  return RI_OK;
}

}  // namespace

int phi_apply(const Plan& p, const float* x, float* y, const uint8_t* mask, hipStream_t s) {
  RI_TRY(fft_forward(p, x, p.grid, s));
  return degrid_apply(p, p.grid, reinterpret_cast<float2*>(y), mask, s);
}

int phi_adj_apply(const Plan& p, const float* y, float* x, const uint8_t* mask, hipStream_t s) {
  RI_TRY(grid_apply(p, reinterpret_cast<const float2*>(y), mask, p.adj_buffer(), s));
  return fft_adjoint(p, p.adj_buffer(), x, s);
}

}  // namespace ri

using ri::fail;

extern "C" {

int ri_plan_create(ri_plan* out, int n, int64_t M, const float* uv_host, int d, const int64_t* block_off_host,
                   int J, double beta, const ri_tuning* tune, hipStream_t stream) {
  if (!out) return fail(RI_EINVAL, "out is NULL");
  *out = nullptr;
  ri_plan h = new (std::nothrow) ri_plan_s;
  if (!h) return fail(RI_ENOMEM, "host allocation failed");
  int rc;
  try {
    rc = ri::create_plan(h->p, n, M, uv_host, d, block_off_host, J, beta, tune, stream);
  } catch (const std::bad_alloc&) {
    rc = fail(RI_ENOMEM, "host allocation failed during plan creation");
  }
  if (rc != RI_OK) {
    ri::destroy_plan(h->p);
    delete h;
    return rc;
  }
  *out = h;
  return RI_OK;
}

void ri_plan_destroy(ri_plan plan) {
  if (!plan) return;
  ri::destroy_plan(plan->p);
  delete plan;
}

int ri_plan_info(ri_plan plan, int* n, int64_t* M, int* d, int* K, int* tile, int* n_items) {
  if (!plan) return fail(RI_EINVAL, "plan is NULL");
  if (n) *n = plan->p.n;
  if (M) *M = plan->p.M;
  if (d) *d = plan->p.d;
  if (K) *K = plan->p.K;
  if (tile) *tile = plan->p.tile;
  if (n_items) *n_items = plan->p.n_items_info;
  return RI_OK;
}

int ri_plan_order(ri_plan plan, int64_t* order_host) {
  if (!plan || !order_host) return fail(RI_EINVAL, "NULL argument");
  std::copy(plan->p.order_host.begin(), plan->p.order_host.end(), order_host);
  return RI_OK;
}

int ri_plan_permute(ri_plan plan, const float* src, float* dst, int to_plan, hipStream_t stream) {
  if (!plan || !src || !dst) return fail(RI_EINVAL, "NULL argument");
  if (src == dst) return fail(RI_EINVAL, "src and dst must differ");
  const int64_t chunks = (plan->p.M + ri::PERM_CHUNK - 1) / ri::PERM_CHUNK;
  const int per_xcd = int((chunks + ri::PERM_XCDS - 1) / ri::PERM_XCDS);
  const float2* in = reinterpret_cast<const float2*>(src);
  float2* out = reinterpret_cast<float2*>(dst);
  if (to_plan)
    hipLaunchKernelGGL(ri::k_permute<true>, dim3(per_xcd * ri::PERM_XCDS), dim3(256), 0, stream, in, out,
                       plan->p.order, plan->p.M, per_xcd);
  else
    hipLaunchKernelGGL(ri::k_permute<false>, dim3(per_xcd * ri::PERM_XCDS), dim3(256), 0, stream, in, out,
                       plan->p.order, plan->p.M, per_xcd);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

int ri_phi(ri_plan plan, const float* x, float* y, const uint8_t* mask, hipStream_t stream) {
  if (!plan || !x || !y) return fail(RI_EINVAL, "NULL argument");
  return ri::phi_apply(plan->p, x, y, mask, stream);
}

int ri_phi_adj(ri_plan plan, const float* y, float* x, const uint8_t* mask, hipStream_t stream) {
  if (!plan || !x || !y) return fail(RI_EINVAL, "NULL argument");
  return ri::phi_adj_apply(plan->p, y, x, mask, stream);
}

int ri_block_sumsq(ri_plan plan, const float* y, double* out, hipStream_t stream) {
  if (!plan || !y || !out) return fail(RI_EINVAL, "NULL argument");
  return ri::block_sumsq(plan->p, reinterpret_cast<const float2*>(y), out, stream);
}

int ri_phi_norm(ri_plan plan, float* x0, int max_it, double rtol, double* norm_host, int* iters_host,
                hipStream_t stream) {
  if (!plan || !x0 || !norm_host || max_it < 1) return fail(RI_EINVAL, "bad argument");
  ri::Plan& p = plan->p;
  const size_t N = size_t(p.n) * p.n;
  float* y = nullptr;
  RI_TRY(ri::dev_alloc(&y, 2 * size_t(p.M)));
  float* cur = x0;
  float* nxt = p.norm_tmp;
  double lam = 0.0, lam_prev = 0.0, sq = 0.0;
  int it = 0, rc = RI_OK;
  rc = ri::sumsq_f32(cur, N, p.dsum, stream);
  if (rc == RI_OK) rc = ri::scale_by_rsqrt(cur, N, p.dsum, stream);
  for (it = 1; rc == RI_OK && it <= max_it; ++it) {
    rc = ri::phi_apply(p, cur, y, nullptr, stream);
    if (rc == RI_OK) rc = ri::phi_adj_apply(p, y, nxt, nullptr, stream);
    if (rc == RI_OK) rc = ri::sumsq_f32(nxt, N, p.dsum, stream);
    if (rc == RI_OK && hipMemcpyAsync(&sq, p.dsum, sizeof(double), hipMemcpyDeviceToHost, stream) != hipSuccess)
      rc = fail(RI_EHIP, "copy of the norm failed");
    if (rc == RI_OK && hipStreamSynchronize(stream) != hipSuccess) rc = fail(RI_EHIP, "stream sync failed");
    if (rc != RI_OK) break;
    lam = std::sqrt(sq);
    rc = ri::scale_by_rsqrt(nxt, N, p.dsum, stream);
    std::swap(cur, nxt);
    if (lam == 0.0 || std::fabs(lam - lam_prev) <= rtol * lam) break;
    lam_prev = lam;
  }
  if (rc == RI_OK && cur != x0) {
    hipLaunchKernelGGL(ri::k_copy_f32, dim3(1024), dim3(256), 0, stream, cur, x0, N);
    if (hipGetLastError() != hipSuccess) rc = fail(RI_EHIP, "copy launch failed");
  }
  if (rc == RI_OK && hipStreamSynchronize(stream) != hipSuccess) rc = fail(RI_EHIP, "stream sync failed");
  ri::dev_free(y);
  if (rc != RI_OK) return rc;
  *norm_host = std::sqrt(lam);
  if (iters_host) *iters_host = std::min(it, max_it);
  return RI_OK;
}

}  // extern "C"
