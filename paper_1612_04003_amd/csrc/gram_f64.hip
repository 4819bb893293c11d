// Dense FP64 Gram of gathered rows: the one-problem launches (split-K Gram
// kernel and its deterministic reduction) and the launch planner.  The device
// code and its design notes are in gram_dev.h.
#include "gram_dev.h"

#include <algorithm>
#include <cmath>

namespace cabcd {
namespace {

using namespace gdev;

// Several row lists per launch: step blockIdx.y reads idx + step * m and
// writes its partials (and its Y u, when u is given) at partials + step * pstride.
template <int NB>
__global__ __launch_bounds__(Cfg<NB>::THREADS) void gram_f64_dma_kernel(
    const double* __restrict__ A, int64_t ld, int64_t cols, const int32_t* __restrict__ idx,
    int m, const double* __restrict__ u, int64_t chunk, double* __restrict__ partials,
    int64_t pstride) {
  using C = Cfg<NB>;
  __shared__ __attribute__((aligned(16))) double t0[DN<NB>::TILE], t1[DN<NB>::TILE];
  idx += (int64_t)blockIdx.y * m;
  partials += (int64_t)blockIdx.y * pstride;
  const int64_t k_begin = (int64_t)blockIdx.x * chunk;
  const int64_t k_end = std::min(cols, k_begin + chunk);
  gram_slab_dma<NB>(A, ld, k_begin, k_end, idx, m, u,
                    partials + (int64_t)blockIdx.x * (C::NBLK * 256 + C::SBP), t0, t1);
}

template <int NB>
__global__ __launch_bounds__(Tri<NB>::THREADS) void gram_f64_tri_kernel(
    const double* __restrict__ A, int64_t ld, int64_t cols, const int32_t* __restrict__ idx,
    int m, const double* __restrict__ u, int64_t chunk, double* __restrict__ partials,
    int64_t pstride) {
  using C = Tri<NB>;
  __shared__ __attribute__((aligned(16))) double t0[C::TILE], t1[C::TILE], t2[C::TILE];
  idx += (int64_t)blockIdx.y * m;
  partials += (int64_t)blockIdx.y * pstride;
  const int64_t k_begin = (int64_t)blockIdx.x * chunk;
  const int64_t k_end = std::min(cols, k_begin + chunk);
  gram_slab_tri<C>(A, ld, k_begin, k_end, idx, m, 0, u,
                   partials + (int64_t)blockIdx.x * (C::NBLK * 256 + C::SBP), TriLds{t0, t1, t2});
}

// Entries of a part of a Gram above 256 rows: its blocks, then a triangle's Y u.
__host__ __device__ constexpr int64_t big_entries(int kind) {
  return kind > 0 ? (int64_t)kind * (kind + 1) / 2 * 256 + 16 * kind : (int64_t)-kind * 16 * 256;
}

// A Gram of 257 to 512 rows: workgroup x of Gram y computes one slab of one part.  The
// parts differ in work a column, so each gets workgroups (and so slabs) in proportion:
// one round of equally long workgroups.  384 x 65536: 183 us and 15 to reduce 63 MB of
// partial sums; as four 256-row Grams of 256 slabs (544 blocks of work for 300) 331 us
// and 76 for 286 MB.
__global__ __launch_bounds__(512) void gram_f64_big_kernel(
    const double* __restrict__ A, int64_t ld, int64_t cols, const int32_t* __restrict__ idx,
    int m, const double* __restrict__ u, double* __restrict__ partials, GramBig p) {
  constexpr int TILE = Rect<8>::TILE;   // the largest
  __shared__ __attribute__((aligned(16))) double t0[TILE], t1[TILE], t2[TILE];
  const TriLds L{t0, t1, t2};
  idx += (int64_t)blockIdx.y * m;
  int q = 0;
  while ((int)blockIdx.x >= p.wg[q + 1]) ++q;
  const int slab = (int)blockIdx.x - p.wg[q];
  double* part = partials + (int64_t)blockIdx.y * p.off[p.parts] + p.off[q] +
                 slab * big_entries(p.kind[q]);
  const int64_t k0 = slab * p.chunk[q], k1 = std::min(cols, k0 + p.chunk[q]);
  const int base = p.base[q];
  switch (p.kind[q]) {
    case 4: gram_slab_tri<Tri<4>>(A, ld, k0, k1, idx, m, base, u, part, L); break;
    case 8: gram_slab_tri<Tri<8>>(A, ld, k0, k1, idx, m, base, u, part, L); break;
    case 12: gram_slab_tri<Tri<12>>(A, ld, k0, k1, idx, m, base, u, part, L); break;
    case 16: gram_slab_tri<Tri<16>>(A, ld, k0, k1, idx, m, base, u, part, L); break;
    case -4: gram_slab_tri<Rect<4>>(A, ld, k0, k1, idx, m, base, nullptr, part, L); break;
    default: gram_slab_tri<Rect<8>>(A, ld, k0, k1, idx, m, base, nullptr, part, L); break;
  }
}

// MODE 1: the Gram with the previous step's update folded in; MODE 2: the
// update alone (one slab per workgroup, the Gram's slabs).
template <int MODE>
__global__ __launch_bounds__(D16::THREADS) void gram_f64_dma16_upd_kernel(
    const double* __restrict__ A, int64_t ld, int64_t cols, const int32_t* __restrict__ idx,
    int m, int64_t chunk, double* __restrict__ partials, D16Upd up) {
  __shared__ __attribute__((aligned(16))) double lds[D16::LDS_UPD];
  const int64_t k_begin = (int64_t)blockIdx.x * chunk;
  const int64_t k_end = std::min(cols, k_begin + chunk);
  double* part =
      MODE == 1 ? partials + (int64_t)blockIdx.x * (D16::NBLK * 256 + D16::SBP) : nullptr;
  gram_slab_dma16<MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up);
}

// A reduction workgroup has 1024 threads: GROUPS split groups (a wave or more
// each) for 1024 / GROUPS entries.  Many splits take 16 groups of 64 entries;
// a few splits take one group, each thread summing all of its entry's splits.
constexpr int kRedThreads = 1024;
// So does a launch of many entries with up to 16 splits: 16 groups of one split
// each add in the same order, but load one value a thread (73 MB of 13 Grams'
// partials: 2.3 TB/s).
int red_groups(int nsplit, int64_t entries) {
  return nsplit <= 4 || (nsplit <= 16 && entries >= (1 << 18)) ? 1 : 16;
}

// Partial set blockIdx.y: partials + set * nsplit * pstride.  MODE 0: the
// Gram of step blockIdx.y (idx + step * m, G and add + step * m * m; Yu is
// NULL for several steps).  MODE 1 / 2: the diagonal / cross sets of a Gram of m in
// (256, 512] rows (store_entry_big).
template <int MODE, int GROUPS>
__global__ __launch_bounds__(kRedThreads) void gram_reduce_kernel(
    const double* __restrict__ partials, int nsplit, int nb, const int32_t* __restrict__ idx,
    int m, double scale, double shift, int overlap, double* __restrict__ G,
    double* __restrict__ Yu, int layout, const float* __restrict__ rs,
    const double* __restrict__ add) {
  constexpr int kRedElems = kRedThreads / GROUPS;
  constexpr int kRedGroups = GROUPS;
  __shared__ double red[kRedGroups][kRedElems];
  const int nblk = nb * (nb + 1) / 2;
  const int64_t pstride = (int64_t)nblk * 256 + 16 * nb;
  partials += (int64_t)blockIdx.y * nsplit * pstride;
  const int gram = MODE == 0 ? (int)blockIdx.y : 0;
  idx += (int64_t)gram * m;
  G += (int64_t)gram * m * m;
  if (add != nullptr) add += (int64_t)gram * m * m;
  const int el = threadIdx.x % kRedElems;
  const int grp = threadIdx.x / kRedElems;
  const int64_t e = (int64_t)blockIdx.x * kRedElems + el;
  // Each wave sums a contiguous range of splits for 64 consecutive entries;
  // the ranges are then added in group order, so the result is deterministic.
  const int spg = (nsplit + kRedGroups - 1) / kRedGroups;   // splits per group
  const int sp0 = grp * spg;
  int sp1 = min(nsplit, sp0 + spg);
  // blocks of padding rows are not read (130 rows of codes as sixteen block rows: 45 of
  // the 136 blocks)
  if (MODE == 0 && m <= 16 * (nb - 1) && e < (int64_t)nblk * 256) {
    int r = 0;
    while (blk_index(r + 1, 0) <= (int)(e >> 8)) ++r;
    if (16 * r >= m) sp1 = sp0;
  }
  double s = 0.0;
  if (layout == 2 && e < (int64_t)nblk * 256) {   // FP32 block entries
    const float* p = reinterpret_cast<const float*>(partials) + e;
    const int64_t fstride = 2 * pstride;
    int sp = sp0;
    for (; sp + 8 <= sp1; sp += 8) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = p[(int64_t)(sp + q) * fstride];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += (double)v[q];
    }
    for (; sp < sp1; ++sp) s += (double)p[(int64_t)sp * fstride];
  } else if (e < pstride) {
    const double* p = partials + e;
    int sp = sp0;
    for (; sp + 8 <= sp1; sp += 8) {
      double v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = p[(int64_t)(sp + q) * pstride];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += v[q];
    }
    for (; sp < sp1; ++sp) s += p[(int64_t)sp * pstride];
  }
  red[grp][el] = s;
  __syncthreads();
  if (grp != 0 || e >= pstride) return;
  double t = red[0][el];
#pragma unroll
  for (int g = 1; g < kRedGroups; ++g) t += red[g][el];
  if constexpr (MODE == 0)
    store_entry(e, t, nblk, idx, m, scale, shift, overlap, G, Yu, layout, rs, add);
  else
    gdev::store_entry_big(e, t, MODE - 1, (int)blockIdx.y, idx, m, scale, shift, overlap, G, Yu,
                          layout, rs);
}

// The parts' partial sums into G and Y u (Gram blockIdx.y), in slab order by GROUPS
// ranges as in gram_reduce_kernel.
template <int GROUPS>
__global__ __launch_bounds__(kRedThreads) void gram_big_reduce_kernel(
    const double* __restrict__ partials, const int32_t* __restrict__ idx, int m, double scale,
    double shift, int overlap, double* __restrict__ G, double* __restrict__ Yu,
    const double* __restrict__ add, GramBig p) {
  constexpr int kElems = kRedThreads / GROUPS;
  __shared__ double red[GROUPS][kElems];
  idx += (int64_t)blockIdx.y * m;
  G += (int64_t)blockIdx.y * m * m;
  if (add != nullptr) add += (int64_t)blockIdx.y * m * m;
  const int el = threadIdx.x % kElems, grp = threadIdx.x / kElems;
  const int64_t ge = (int64_t)blockIdx.x * kElems + el;
  const bool on = ge < p.entry[p.parts];
  int q = 0;
  while (on && ge >= p.entry[q + 1]) ++q;
  const int64_t e = ge - p.entry[q];
  double s = 0.0;
  if (on) {
    const int n = p.wg[q + 1] - p.wg[q];
    const int64_t stride = big_entries(p.kind[q]);
    const double* in = partials + (int64_t)blockIdx.y * p.off[p.parts] + p.off[q] + e;
    const int per = (n + GROUPS - 1) / GROUPS;
    const int s1 = min(n, (grp + 1) * per);
    int sp = grp * per;
    for (; sp + 8 <= s1; sp += 8) {
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = in[(int64_t)(sp + j) * stride];
#pragma unroll
      for (int j = 0; j < 8; ++j) s += v[j];
    }
    for (; sp < s1; ++sp) s += in[(int64_t)sp * stride];
  }
  red[grp][el] = s;
  __syncthreads();
  if (grp != 0 || !on) return;
  double t = red[0][el];
#pragma unroll
  for (int g = 1; g < GROUPS; ++g) t += red[g][el];
  const int kind = p.kind[q], base = p.base[q];
  int row, col;
  if (kind > 0) {
    const int nblk = kind * (kind + 1) / 2;
    if (e >= (int64_t)nblk * 256) {   // Y u follows a triangle's blocks
      const int r = base + (int)(e - (int64_t)nblk * 256);
      if (Yu != nullptr && r < m) Yu[r] = t;
      return;
    }
    bool lower;
    entry_rc(e, 0, row, col, lower);
    if (!lower) return;
    row += base;
    col += base;
  } else {
    const int blk = (int)(e >> 8), item = (int)(e >> 6) & 3, lane = (int)e & 63;
    row = base + 16 * (blk >> 4) + 4 * item + (lane >> 4);
    col = 16 * (blk & 15) + (lane & 15);
  }
  if (row >= m) return;
  const bool same = overlap ? idx[row] == idx[col] : row == col;
  if (add != nullptr) t += add[(int64_t)row * m + col];
  const double v = scale * t + (same ? shift : 0.0);
  G[(int64_t)row * m + col] = v;
  G[(int64_t)col * m + row] = v;
}

// The index lists (gdev::big_lists) of a low-precision Gram above 256 rows.
__global__ __launch_bounds__(512) void big_index_kernel(const int32_t* __restrict__ idx, int m,
                                                        int32_t* __restrict__ ia,
                                                        int32_t* __restrict__ ib) {
  gdev::big_lists(idx, m, ia, ib, threadIdx.x, 512);
}

template <int NB>
hipError_t launch_nb(const GramPlan& p, const double* A, int64_t ld, int64_t cols,
                     const int32_t* idx, int m, int nsteps, const double* u, double* partials,
                     hipStream_t st) {
  const int64_t pstride = (int64_t)gram_partial_doubles(p);
  const dim3 grid((unsigned)p.nsplit, (unsigned)nsteps);
  if constexpr (NB >= kTriMin)
    hipLaunchKernelGGL((gram_f64_tri_kernel<NB>), grid, dim3(Tri<NB>::THREADS), 0, st, A, ld, cols,
                       idx, m, u, p.chunk, partials, pstride);
  else
    hipLaunchKernelGGL((gram_f64_dma_kernel<NB>), grid, dim3(Cfg<NB>::THREADS), 0, st, A, ld, cols,
                       idx, m, u, p.chunk, partials, pstride);
  return hipGetLastError();
}

}  // namespace

// Block rows of a Gram of m <= 256 rows: a power of two up to 8 (the k-split kernels),
// even numbers above (the matrix cores bound those, and 150 rows as sixteen block rows
// were 136 blocks of work for 55; odd numbers would save 8 % more at most).
int gram_f64_blocks(int m) {
  int nb = 1;
  while (16 * nb < m && nb < 8) nb *= 2;
  return 16 * nb >= m ? nb : tri_rows((m + 15) / 16);
}

GramPlan plan_gram_f64(int m, int64_t cols) {
  GramPlan p{};
  const int nb = gram_f64_blocks(m);
  p.nb = nb;
  p.nblk = nb * (nb + 1) / 2;
  const bool tri = nb >= kTriMin;
  p.kt = tri ? 16 : 256 / nb;
  const int bw = nb >= 2 ? nb / 2 : 1;
  const int kg = tri ? 1 : 8 / bw;
  const int nacc = tri ? (p.nblk + 7) / 8 : nb >= 2 ? nb + 1 : 1;
  // Cost model (alpha-beta-gamma style, eq. comm): matrix-core time of the
  // slowest round of workgroups, HBM time of the gathered rows, and the traffic
  // of writing and re-reading the partial Grams.  Pick the cheapest chunk.
  const double clock = 2.4e9, hbm = 6.0e12;
  // The plan depends on m only through nb, so every m of one class gets the
  // same split and the workspace bound over classes is exact.
  const double ybytes = 16.0 * nb * (double)cols * 8.0;
  const double pbytes_per = ((double)p.nblk * 256 + 16.0 * nb) * 8.0;
  double best = 1e300;
  int64_t best_chunk = cols;
  // A CU streams at most its share of the HBM rate, so fewer slabs than CUs
  // leave bandwidth unused.
  auto hbm_time = [&](int64_t nsplit) {
    return ybytes / (hbm * std::min(1.0, (double)nsplit / 256.0));
  };
  for (int64_t chunk = p.kt; ; chunk *= 2) {
    const int64_t nsplit = (cols + chunk - 1) / chunk;
    const double per_wg = 2.0 * ((double)chunk / (4.0 * kg)) * nacc * 64.0 / clock;
    const double rounds = std::ceil((double)nsplit / 256.0);
    const double t = std::max(rounds * per_wg, hbm_time(nsplit)) +
                     2.0 * nsplit * pbytes_per / hbm + (nsplit > 1024 ? 1e-3 : 0.0);
    if (t < best) {
      best = t;
      best_chunk = chunk;
    }
    if (nsplit <= 1) break;
  }
  // Also try the chunk that gives exactly one workgroup per CU.
  {
    int64_t chunk = (cols + 255) / 256;
    chunk = ((chunk + p.kt - 1) / p.kt) * p.kt;
    const int64_t nsplit = (cols + chunk - 1) / chunk;
    const double per_wg = 2.0 * ((double)chunk / (4.0 * kg)) * nacc * 64.0 / clock;
    const double t = std::max(per_wg, hbm_time(nsplit)) + 2.0 * nsplit * pbytes_per / hbm;
    if (t < best) {
      best = t;
      best_chunk = chunk;
    }
  }
  p.chunk = best_chunk;
  p.nsplit = (int)((cols + best_chunk - 1) / best_chunk);
  return p;
}

// Microseconds a workgroup spends on one tile of a part (two waves a SIMD), at least
// the latency of the DMA: one tile is in flight.
static double big_tile_us(int kind) {
  const int blocks = kind > 0 ? kind * (kind + 1) / 2 : -kind * 16;
  return std::max(0.9, (blocks + 7) / 8 * 4 * 64 * 2 / 2400.0);
}

GramBig plan_gram_big_f64(int m, int64_t cols, int wgs) {
  GramBig p{};
  const int rest = (m - 256 + 63) / 64 * 4;   // block rows from 256 on, in fours
  auto part = [&](int kind, int base) {
    p.kind[p.parts] = kind;
    p.base[p.parts++] = base;
  };
  part(16, 0);
  part(rest, 256);
  for (int r = 0; r < rest; r += 8) part(-std::min(8, rest - r), 256 + 16 * r);
  double total = 0.0;
  for (int q = 0; q < p.parts; ++q) total += big_tile_us(p.kind[q]);
  const int64_t tiles = (cols + 15) / 16;
  for (int q = 0; q < p.parts; ++q) {
    // (rounded down, so that the workgroups are one round)
    int64_t n = (int64_t)(wgs * big_tile_us(p.kind[q]) / total);
    n = std::min(std::max<int64_t>(n, 1), tiles);
    p.chunk[q] = 16 * ((tiles + n - 1) / n);
    n = (cols + p.chunk[q] - 1) / p.chunk[q];
    p.wg[q + 1] = p.wg[q] + (int)n;
    p.entry[q + 1] = p.entry[q] + big_entries(p.kind[q]);
    p.off[q + 1] = p.off[q] + n * big_entries(p.kind[q]);
  }
  return p;
}

size_t gram_big_doubles_max(int m_max, int64_t cols, int wgs) {
  size_t best = 0;
  for (int m = 320; m - 64 < m_max; m += 64) {
    const GramBig p = plan_gram_big_f64(m, cols, wgs);
    best = std::max(best, (size_t)p.off[p.parts]);
  }
  return best;
}

size_t gram_partial_doubles(const GramPlan& p) {
  return (size_t)p.nsplit * ((size_t)p.nblk * 256 + 16 * (size_t)p.nb);
}

hipError_t launch_gram_f64(const GramPlan& p, const double* A, int64_t ld, int64_t cols,
                           const int32_t* idx, int m, const double* u, double* partials,
                           hipStream_t st, int nsteps) {
  if (nsteps < 1 || nsteps > 65535) return hipErrorInvalidValue;
  switch (p.nb) {
    case 1: return launch_nb<1>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 2: return launch_nb<2>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 4: return launch_nb<4>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 8: return launch_nb<8>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 10: return launch_nb<10>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 12: return launch_nb<12>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 14: return launch_nb<14>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    case 16: return launch_nb<16>(p, A, ld, cols, idx, m, nsteps, u, partials, st);
    default: return hipErrorInvalidValue;
  }
}

bool gram_f64_takes_update(const GramPlan& p, int m) { return p.nb == 16 && m == D16::SBP; }

hipError_t launch_gram_f64_upd(const GramPlan& p, const double* A, int64_t ld, int64_t cols,
                               const int32_t* idx, int m, double* partials, const D16Upd& up,
                               hipStream_t st) {
  if (!gram_f64_takes_update(p, m) || up.idx == nullptr || up.delta == nullptr ||
      up.r == nullptr)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((gram_f64_dma16_upd_kernel<1>), dim3((unsigned)p.nsplit), dim3(D16::THREADS),
                     0, st, A, ld, cols, idx, m, p.chunk, partials, up);
  return hipGetLastError();
}

hipError_t launch_update_f64(const GramPlan& p, const double* A, int64_t ld, int64_t cols,
                             const D16Upd& up, hipStream_t st) {
  if (p.nb != 16 || up.idx == nullptr || up.delta == nullptr || up.r == nullptr)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((gram_f64_dma16_upd_kernel<2>), dim3((unsigned)p.nsplit), dim3(D16::THREADS),
                     0, st, A, ld, cols, nullptr, 0, p.chunk, nullptr, up);
  return hipGetLastError();
}

template <int MODE>
void launch_reduce(int groups, dim3 grid, hipStream_t st, const double* partials, int nsplit,
                   int nb, const int32_t* idx, int m, double scale, double shift, int overlap,
                   double* G, double* Yu, int layout, const float* rs, const double* add) {
  if (groups == 1)
    hipLaunchKernelGGL((gram_reduce_kernel<MODE, 1>), grid, dim3(kRedThreads), 0, st, partials,
                       nsplit, nb, idx, m, scale, shift, overlap, G, Yu, layout, rs, add);
  else
    hipLaunchKernelGGL((gram_reduce_kernel<MODE, 16>), grid, dim3(kRedThreads), 0, st, partials,
                       nsplit, nb, idx, m, scale, shift, overlap, G, Yu, layout, rs, add);
}

hipError_t launch_gram_reduce(const GramPlan& p, const double* partials, const int32_t* idx,
                              int m, double scale, double shift, bool overlap, double* G,
                              double* Yu, hipStream_t st, int layout, const float* rs,
                              int nsteps, const double* add) {
  if (nsteps < 1 || nsteps > 65535 || (nsteps > 1 && Yu != nullptr)) return hipErrorInvalidValue;
  const int64_t entries = (int64_t)p.nblk * 256 + 16 * p.nb;
  const int groups = red_groups(p.nsplit, entries * nsteps);
  const int64_t blocks = (entries + kRedThreads / groups - 1) / (kRedThreads / groups);
  launch_reduce<0>(groups, dim3((unsigned)blocks, (unsigned)nsteps), st, partials, p.nsplit, p.nb,
                   idx, m, scale, shift, overlap ? 1 : 0, G, Yu, layout, rs, add);
  return hipGetLastError();
}

hipError_t launch_gram_big_f64(const GramBig& p, const double* A, int64_t ld, int64_t cols,
                               const int32_t* idx, int m, const double* u, double* partials,
                               hipStream_t st, int ngram) {
  if (m <= 256 || m > 512 || ngram < 1 || ngram > 65535 || (ngram > 1 && u != nullptr))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(gram_f64_big_kernel, dim3((unsigned)p.wg[p.parts], (unsigned)ngram), dim3(512),
                     0, st, A, ld, cols, idx, m, u, partials, p);
  return hipGetLastError();
}

hipError_t launch_gram_big_reduce_f64(const GramBig& p, const double* partials,
                                      const int32_t* idx, int m, double scale, double shift,
                                      bool overlap, double* G, double* Yu, hipStream_t st,
                                      int ngram, const double* add) {
  if (m <= 256 || m > 512 || ngram < 1 || ngram > 65535 || (ngram > 1 && Yu != nullptr))
    return hipErrorInvalidValue;
  int most = 0;
  for (int q = 0; q < p.parts; ++q) most = std::max(most, p.wg[q + 1] - p.wg[q]);
  const int groups = red_groups(most, p.entry[p.parts] * ngram);
  const int per = kRedThreads / groups;
  const dim3 grid((unsigned)((p.entry[p.parts] + per - 1) / per), (unsigned)ngram);
  if (groups == 1)
    hipLaunchKernelGGL((gram_big_reduce_kernel<1>), grid, dim3(kRedThreads), 0, st, partials, idx,
                       m, scale, shift, overlap ? 1 : 0, G, Yu, add, p);
  else
    hipLaunchKernelGGL((gram_big_reduce_kernel<16>), grid, dim3(kRedThreads), 0, st, partials, idx,
                       m, scale, shift, overlap ? 1 : 0, G, Yu, add, p);
  return hipGetLastError();
}

hipError_t launch_big_index(const int32_t* idx, int m, int32_t* ia, int32_t* ib, hipStream_t st) {
  if (m <= 256 || m > 512) return hipErrorInvalidValue;
  hipLaunchKernelGGL(big_index_kernel, dim3(1), dim3(512), 0, st, idx, m, ia, ib);
  return hipGetLastError();
}

int big_cross_steps(int m) { return m - 256 > 128 ? 4 : 2; }

hipError_t launch_gram_reduce_big(const GramPlan& p, const double* partials, const int32_t* idx,
                                  int m, double scale, double shift, bool overlap, double* G,
                                  double* Yu, hipStream_t st, int layout, const float* rs) {
  if (p.nb != 16 || m <= 256 || m > 512) return hipErrorInvalidValue;
  const int64_t entries = (int64_t)p.nblk * 256 + 16 * p.nb;
  const int groups = red_groups(p.nsplit, entries * 2);
  const int64_t blocks = (entries + kRedThreads / groups - 1) / (kRedThreads / groups);
  launch_reduce<1>(groups, dim3((unsigned)blocks, 2), st, partials, p.nsplit, p.nb, idx, m, scale,
                   shift, overlap ? 1 : 0, G, Yu, layout, rs, nullptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_reduce<2>(groups, dim3((unsigned)blocks, (unsigned)big_cross_steps(m)), st,
                   partials + 2 * gram_partial_doubles(p), p.nsplit, p.nb, idx, m, scale, shift,
                   overlap ? 1 : 0, G, nullptr, layout, rs, nullptr);
  return hipGetLastError();
}

}  // namespace cabcd
