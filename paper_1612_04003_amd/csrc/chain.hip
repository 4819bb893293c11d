// The dependent chain of outer steps whose Grams are computed ahead.
//
// The s inner solves of an outer step are one block forward substitution with
// the lower block triangle T of the overlap-augmented Gram (solve_dev.h).  T
// depends on the sampled indices only, so for Grams computed ahead its inverse
// is formed ahead too, off the chain, and the solves of a step become one
// product delta = T^-1 c with no dependent inner steps.  (As one workgroup's
// forward substitution they took 15.5 us of a 38 us dense dual step at b = 8,
// s = 32 and 42 us of an 81 us sparse one at b = 16, s = 32.)
//
// T^-1 is formed in superblocks of gb = b floor(16 / b) <= 16 rows, padded to
// 16 with the identity:
//   * chain_diag_kernel: the superblocks on the diagonal (block lower triangular
//     inside) by Gauss-Jordan elimination, one row per lane; their pivots are
//     those of the b x b blocks Gamma_j, and a pivot <= 0 or NaN is noted in the
//     step's links, which report it when the step is run;
//   * chain_panel_kernel: a first inverse Z by rows, Z_IJ = -(sum_{J<t<=I} Z_It T_tJ)
//     D_J^-1, one workgroup per superblock row I on the FP64 matrix cores, which
//     work on Z transposed: an FP64 MFMA result holds item i at row 4 i + lane /
//     16, which is the operand layout of k-slice i, so Z feeds the next product
//     from the registers it was written from (kept in LDS);
//   * chain_resid_kernel, chain_refine_kernel: T^-1 = Z + (I - Z T) Z for the rows
//     that need it, the residual summed in twice the working precision.
// (chain_small_kernel does all of it for up to four superblocks.)  The order and the
// refinement are for accuracy.  With c = T delta the product Z c is off by (Z T - I) delta, which the substitution has no counterpart to: where
// the rows are nearly collinear, c is far smaller than |T| |delta|.  An inverse by
// columns keeps T Z - I small and leaves Z T - I large: w of 256 x 4096, b = 8, s =
// 32, row correlation 0.9999, lambda 1e-5, was off by 5.3e-7 where the substitution
// is off by 8.7e-12.  By rows w is right, but the errors of a step's deltas are
// independent of each other, where later blocks of the substitution make up for
// those of earlier ones, and the companion takes them up: on the CPU a dual w of 300
// x 600, b = s = 16, was off by 4.3e-10, against 1.5e-11.  The refined inverse is
// exact to the rounding of its entries, and Z c to the rounding of the product, which
// c scales: w and r of that primal run are off by 1.1e-11 and 1.2e-11, by substitution
// by 8.7e-12 and 1.0e-11.  Refining every row adds 2 us to a step of 256 rows and 11 to
// one of 512; where none is refined there are two short launches a batch more.
// T^-1 is stored as its lower 16 x 16 superblocks in that result layout, items
// 2 i and 2 i + 1 of a lane side by side (256 doubles each, row-major over the
// block triangle), which the product reads with two 16-byte loads a lane.
//
// Dense steps then take one launch each (chain_step_kernel): the companion u is
// cut into column slabs, one workgroup per slab.  Every workgroup adds the
// slabs' partial Y u of the step (written by the launch before), forms c and
// delta = T^-1 c for itself (T^-1 comes from L2), updates its slab of u with
// the step's rows, and forms its slab's partial products of the next step's
// rows with the updated slab, which it still holds.  One more workgroup
// updates x and gathers x at the next step's indices.  What bounds a launch is
// latency: the partial sums come from other XCDs' workgroups, and delta needs
// all of them; the rows are prefetched into registers before that wait.  Sparse
// steps keep their row products and updates and take chain_delta_kernel between
// them.
//
// Measured per outer step in a long run, before -> now (us): dense primal d =
// 64, n = 1024, b = 4, s = 8: 14 -> 8.5 (the launch 7.9); d = 2048, n = 2^18, b =
// 8, s = 1: 28 -> 15.8 (12.0: 33.5 MB of rows at 2.8 TB/s); dense dual d = 2048, b
// = 8, s = 32: 38.6 in four launches -> 17.2 (13.2, of which T^-1 c takes 3.9: 278
// KB of T^-1 into each of 64 CUs); sparse dual b = 16, s = 8: 25 -> 16.5; s = 32: 81
// -> 46, now the Gram's pace.
#include "chain_dev.h"
#include "gram_dev.h"
#include "lowp_dev.h"
#include "solve_dev.h"

#include <algorithm>
#include <type_traits>

namespace cabcd {
namespace {

using cdev::kLinkBad;
using cdev::kLinkFirst;
using cdev::rhs_of;
using cdev::tri_at;
using cdev::tri_block;
using gdev::d16_row_sum;
using gdev::d4;

// v / b for v < 16, 1 <= b <= 16, as a product with bm = block_mul(b).
__host__ __device__ constexpr int block_mul(int b) { return (255 + b) / b; }
__device__ __forceinline__ int block_of(int v, int bm) { return (v * bm) >> 8; }

// ------------------------------------------------------------------ T^-1

// Row u of the inverse of superblock I (a group of sixteen lanes holds one), the
// identity past nsb; true when a pivot is not positive (the same in the group).
__device__ __forceinline__ bool diag_inverse(const double* __restrict__ G, int m, int b, int gb,
                                             int nsb, int I, int u, double (&e)[16]) {
  const int r0 = I * gb;
  const bool live = I < nsb && u < gb && r0 + u < m;
  // unconditional loads at clamped places, so that they go out together
#pragma unroll
  for (int v = 0; v < 16; ++v) e[v] = G[(int64_t)min(r0 + v, m - 1) * m + min(r0 + u, m - 1)];
  const int bm = block_mul(b), bu = block_of(u, bm);
#pragma unroll
  for (int v = 0; v < 16; ++v)
    e[v] = live && block_of(v, bm) <= bu && v < gb && r0 + v < m ? e[v] : (u == v ? 1.0 : 0.0);
  bool bad = false;
  sdev::gj_rows16<0>(e, u, bad);   // every lane takes part in the row broadcasts
  return bad;
}

// Superblock I of step blockIdx.y: four per wave, one row per lane.
__global__ __launch_bounds__(64) void chain_diag_kernel(const double* __restrict__ G, int m, int b,
                                                        int gb, int nsb, double* __restrict__ tri,
                                                        double* __restrict__ dinv,
                                                        int* __restrict__ bad_block) {
  G += (int64_t)blockIdx.y * m * m;
  tri += (int64_t)blockIdx.y * tri_block(nsb, 0) * 256;
  dinv += (int64_t)blockIdx.y * nsb * 256;
  const int I = blockIdx.x * 4 + (threadIdx.x >> 4);
  const int u = threadIdx.x & 15;
  double e[16];
  const bool bad = diag_inverse(G, m, b, gb, nsb, I, u, e);
  if (I >= nsb) return;
  if (u == 0) bad_block[(int)blockIdx.y * nsb + I] = bad ? 1 : 0;
  double* t = tri + (int64_t)tri_block(I, I) * 256;
  double* d = dinv + (int64_t)I * 256 + 16 * u;   // the transposed operand: k-slice, lane
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    t[tri_at(u >> 2, (u & 3) * 16 + v)] = e[v];
    d[v] = e[v];
  }
}

// Rows of superblock t of T in the columns of superblock J < t, transposed, as an operand:
// 16 consecutive doubles a row.  FULL: gb = 16 and m a multiple of 16.
template <bool FULL>
__device__ __forceinline__ void load_t(gptr<const double> Gs, int m, int gb, int t, int J,
                                       int lane, double (&a)[4]) {
  const int l15 = lane & 15, l16 = lane >> 4, col = J * gb + l15;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int kk = 4 * s + l16, row = t * gb + kk;
    if constexpr (FULL) {
      a[s] = Gs[(int64_t)row * m + col];
    } else {
      const bool ok = kk < gb && l15 < gb && row < m && col < m;
      const double v = Gs[ok ? (int64_t)row * m + col : 0];
      a[s] = ok ? v : 0.0;
    }
  }
}

// -D_J^-1 from the right to the sum v, all transposed (da: the operand of D_J^-1).
__device__ __forceinline__ d4 times_dinv(const double (&da)[4], const double (&v)[4]) {
  d4 z0 = {0.0, 0.0, 0.0, 0.0}, z1 = {0.0, 0.0, 0.0, 0.0};
  z0 = gdev::mfma(da[0], -v[0], z0);
  z1 = gdev::mfma(da[1], -v[1], z1);
  z0 = gdev::mfma(da[2], -v[2], z0);
  z1 = gdev::mfma(da[3], -v[3], z1);
  return z0 + z1;
}

// Link word of row p of the m rows ix; sb_bad: whether its superblock is.
__device__ __forceinline__ int link_word(const int* ix, int m, int p, int sb_bad) {
  const int i = ix[p];
  bool first = true;
  for (int q = 0; q < p; ++q) first &= ix[q] != i;
  int next = 0;
  for (int q = m - 1; q > p; --q) next = ix[q] == i ? q + 1 : next;
  return (first ? kLinkFirst : 0) | next | (sb_bad != 0 ? kLinkBad : 0);
}

// A row needs no refinement where |Z_rk| sqrt(T_kk T_rr), which bounds the amplification
// |Z| |T| whatever the scales of the rows, is at most kRefineFrom: in CPU runs of 160 steps
// of all block sizes, correlations 0 to 0.999 and lambda 1e-6 to 0.1, Z as it is then came
// within 10 % of the substitution (mean error of x and of the companion; 25 % above 32, 37 %
// from 128 on).
constexpr double kRefineFrom = 16.0;
__device__ __forceinline__ double amplified(double z, double gk, double gr) {
  const double v = z * z * gk * gr;
  return v >= 0.0 ? v : __builtin_inf();
}

// Workgroup x < gridDim.x - 1: superblock row I = nsb - 1 - x of step blockIdx.y by
// four waves (the longest rows first); the last workgroup builds the step's links.
// Z to `tri`, and to `out` too where the row needs no refinement, which `need` notes.
//
// A row is a chain over its columns: column R (superblock I - R) needs Z of every
// column before it.  Wave w holds the columns r = w mod 4 and adds their products to
// its part of column R; the parts meet in LDS and wave R mod 4, the only one that
// reads Z_R afterwards, finishes it.  So the other waves run ahead into
// the next column meanwhile (the parts are double-buffered), and one barrier a column
// is enough.  PF operand blocks a wave are in flight; Z goes to memory at the
// end (stores in the loop made the loads after them wait: 50 us for 13 steps of
// 256 rows with one wave a row and stores in the loop, 190 us for 16 of 512).
constexpr int kPanelWaves = 4;
template <bool FULL>
__global__ __launch_bounds__(64 * kPanelWaves) void chain_panel_kernel(
    const double* __restrict__ G, int m, int gb, int nsb, double* __restrict__ tri,
    const double* __restrict__ dinv, const int32_t* __restrict__ idx, int* __restrict__ link,
    const int* __restrict__ bad_block, double* __restrict__ out, int* __restrict__ need) {
  extern __shared__ __attribute__((aligned(16))) double zs[];
  const int64_t step = blockIdx.y;
  if (blockIdx.x == gridDim.x - 1) {
    int* ix = reinterpret_cast<int*>(zs);
    idx += step * m;
    link += step * m;
    for (int p = threadIdx.x; p < m; p += blockDim.x) ix[p] = idx[p];
    __syncthreads();
    for (int p = threadIdx.x; p < m; p += blockDim.x)
      link[p] = link_word(ix, m, p, bad_block[step * nsb + p / gb]);
    return;
  }
  constexpr int PF = 4;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l15 = lane & 15, l16 = lane >> 4;
  const int I = nsb - 1 - (int)blockIdx.x, nr = I + 1;
  const gptr<const double> Gs = glb(G) + step * m * m;
  const gptr<double> T = glb(tri) + step * tri_block(nsb, 0) * 256;
  const gptr<const double> D = glb(dinv) + step * nsb * 256 + lane;
  double* part = zs + lane;                       // two sets of four parts
  double* Zs = zs + 2 * kPanelWaves * 256;        // Z of column r, transposed, at r * 256
  double* Z = Zs + lane;

  // operand block (R, r): rows of superblock I - r of T in the columns of I - R
  auto load = [&](int R, int r, double(&a)[4]) { load_t<FULL>(Gs, m, gb, I - r, I - R, lane, a); };
  double ring[PF][4], da[4];
  int Rn = w + 1, rn = w;   // the next block to load (clamped past the last)
  auto next_load = [&](double(&a)[4]) {
    load(min(Rn, nr - 1), min(rn, nr - 1), a);
    rn += kPanelWaves;
    const bool end = rn >= Rn;
    Rn += end ? 1 : 0;
    rn = end ? w : rn;
  };
  int Rd = w == 0 ? kPanelWaves : w;   // the next column this wave finishes
  auto load_d = [&] {
#pragma unroll
    for (int s = 0; s < 4; ++s) da[s] = D[(int64_t)(I - min(Rd, nr - 1)) * 256 + 64 * s];
  };
#pragma unroll
  for (int q = 0; q < PF; ++q) next_load(ring[q]);
  load_d();
  if (w == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      Z[64 * i] =
          T[(int64_t)tri_block(I, I) * 256 + tri_at(l15 >> 2, (l15 & 3) * 16 + 4 * i + l16)];
  }
  int R = 1, r = w;
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
  auto end_column = [&] {
    double* set = part + (R & 1) * kPanelWaves * 256;
    const d4 sum = acc[0] + acc[1];
    acc[0] = acc[1] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) set[w * 256 + 64 * s] = sum[s];
    lds_barrier();
    if (w == (R & (kPanelWaves - 1))) {
      double v[4];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        v[s] = (set[64 * s] + set[256 + 64 * s]) + (set[512 + 64 * s] + set[768 + 64 * s]);
      const d4 z = times_dinv(da, v);
#pragma unroll
      for (int s = 0; s < 4; ++s) Z[R * 256 + 64 * s] = z[s];
      Rd += kPanelWaves;
      load_d();
    }
    ++R;
    r = w;
  };
  while (R < nr) {
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      while (R < nr && r >= R) end_column();   // uniform
      if (R < nr) {
        const double* z = Z + r * 256;
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[s & 1] = gdev::mfma(ring[q][s], z[64 * s], acc[s & 1]);
        next_load(ring[q]);
        r += kPanelWaves;
      }
    }
  }
  // wave w wrote the columns R = w mod 4
  double* gd = zs;                       // the diagonal of G up to this row (kMaxRows at most)
  double* top = zs + kPanelWaves * 256;   // a wave's largest amplification
  lds_barrier();
  for (int p = threadIdx.x; p < nr * gb; p += 64 * kPanelWaves) {
    const double v = Gs[(int64_t)min(p, m - 1) * (m + 1)];
    gd[p] = p < m ? v : 0.0;
  }
  lds_barrier();
  double big = 0.0;
  for (int R1 = w; R1 < nr; R1 += kPanelWaves) {
    const double* z = Zs + R1 * 256 + 16 * l15 + l16;
    const double gk = l15 < gb ? gd[(I - R1) * gb + l15] : 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double gr = 4 * s + l16 < gb ? gd[I * gb + 4 * s + l16] : 0.0;
      big = fmax(big, amplified(z[4 * s], gk, gr));
    }
  }
  for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
  if (lane == 0) top[w] = big;
  lds_barrier();
  const bool refine =
      fmax(fmax(top[0], top[1]), fmax(top[2], top[3])) > kRefineFrom * kRefineFrom;
  if (threadIdx.x == 0) need[step * nsb + I] = refine ? 1 : 0;
  const gptr<double> To = glb(out) + step * tri_block(nsb, 0) * 256;
  for (int R1 = w; R1 < nr; R1 += kPanelWaves) {
    const int64_t at = (int64_t)tri_block(I, I - R1) * 256;
    const double* z = Zs + R1 * 256 + 16 * l15 + l16;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (R1 > 0) T[at + tri_at(s, lane)] = z[4 * s];
      if (!refine) To[at + tri_at(s, lane)] = z[4 * s];
    }
  }
}

// This lane's items of the stored superblock at t.
__device__ __forceinline__ void tri_load(gptr<const double> t, int lane, double (&v)[4]) {
  typedef double dv2 __attribute__((ext_vector_type(2)));
  const dv2 x = *(gptr<const dv2>)(t + 2 * lane), y = *(gptr<const dv2>)(t + 128 + 2 * lane);
  v[0] = x.x;
  v[1] = x.y;
  v[2] = y.x;
  v[3] = y.y;
}

// Superblock (I, J) of the block triangle that is number x in it.
__device__ __forceinline__ void tri_place(int x, int& I, int& J) {
  I = 0;
  while (tri_block(I + 1, 0) <= x) ++I;
  J = x - tri_block(I, 0);
}

// h + l += a b in twice the working precision: the rounding errors of the product and
// of the sum (TwoProduct and TwoSum; Ogita, Rump and Oishi, SIAM J. Sci. Comput. 2005,
// algorithm Dot2).
__device__ __forceinline__ void dot2(double a, double b, double& h, double& l) {
#pragma clang fp contract(off)   // (h + p must round p)
  const double p = a * b, e = fma(a, b, -p);
  const double q = h + p, z = q - h;
  l += ((h - (q - z)) + (p - z)) + e;
  h = q;
}

// Superblock (I, J) of I - Z T by a workgroup of kResWaves waves, to `out` in the matrix
// cores' operand order (Zr: row I of Z).  Wave w adds the products t = J + w mod 4, a lane
// rows 4 (lane / 16) .. + 3 of column lane % 16.  The vector units bound it: ten FP64
// operations an element product, one product's loads ahead.
constexpr int kResWaves = 4;
struct ResLds {
  static constexpr int ZS = 18;   // (16-byte pieces of a row aligned; two-way bank conflicts)
  __attribute__((aligned(16))) double zt[kResWaves][16 * ZS];   // Z_It, transposed
  double tt[kResWaves][256];                                    // T_tJ
  double part[kResWaves][2][256];
};
template <bool FULL>
__device__ __forceinline__ void resid_block(gptr<const double> Gs, int m, int b, int gb,
                                            gptr<const double> Zr, int I, int J, ResLds& L,
                                            gptr<double> out) {
  typedef double dv2 __attribute__((ext_vector_type(2)));
  constexpr int ZS = ResLds::ZS;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l15 = lane & 15, l16 = lane >> 4;
  const int bm = block_mul(b);
  const int col = J * gb + l15;
  double zv[4], tv[4], h[4], l[4];
  auto load = [&](int t) {
    t = min(t, I);
    tri_load(Zr + (int64_t)t * 256, lane, zv);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int kk = 4 * s + l16, row = t * gb + kk;
      const bool in = FULL || (kk < gb && l15 < gb && row < m && col < m);
      const bool ok = in && (t != J || block_of(l15, bm) <= block_of(kk, bm));
      const double v = Gs[ok ? (int64_t)row * m + col : 0];
      tv[s] = ok ? v : (t == J && kk == l15 ? 1.0 : 0.0);
    }
  };
#pragma unroll
  for (int s = 0; s < 4; ++s) h[s] = l[s] = 0.0;
  load(J + w);
  for (int t0 = J; t0 <= I; t0 += kResWaves) {   // uniform
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      L.zt[w][l15 * ZS + 4 * s + l16] = zv[s];
      L.tt[w][64 * s + lane] = tv[s];
    }
    lds_barrier();
    load(t0 + kResWaves + w);
    if (t0 + w <= I) {   // uniform in a wave
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double t = L.tt[w][16 * k + l15];
        const dv2 z0 = *reinterpret_cast<const dv2*>(&L.zt[w][k * ZS + 4 * l16]);
        const dv2 z1 = *reinterpret_cast<const dv2*>(&L.zt[w][k * ZS + 4 * l16 + 2]);
        dot2(z0.x, t, h[0], l[0]);
        dot2(z0.y, t, h[1], l[1]);
        dot2(z1.x, t, h[2], l[2]);
        dot2(z1.y, t, h[3], l[3]);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    L.part[w][0][64 * s + lane] = h[s];
    L.part[w][1][64 * s + lane] = l[s];
  }
  lds_barrier();
  const int at = threadIdx.x, row = 4 * l16 + (at >> 6);   // (column l15)
  double sh = I == J && row == l15 ? -1.0 : 0.0, sl = 0.0;
#pragma unroll
  for (int q = 0; q < kResWaves; ++q) {
    const double p = L.part[q][0][at], s = sh + p, d = s - sh;
    sl += ((sh - (s - d)) + (p - d)) + L.part[q][1][at];
    sh = s;
  }
  out[16 * l15 + row] = -(sh + sl);
}

// Superblock x of step blockIdx.y of the residual of Z (`tri`), for the rows in need.
template <bool FULL>
__global__ __launch_bounds__(64 * kResWaves) void chain_resid_kernel(
    const double* __restrict__ G, int m, int b, int gb, int nsb, const double* __restrict__ tri,
    const int* __restrict__ need, double* __restrict__ res) {
  __shared__ ResLds L;
  const int64_t step = blockIdx.y;
  int I, J;
  tri_place((int)(gridDim.x - 1 - blockIdx.x), I, J);   // (the longest first)
  if (need[step * nsb + I] == 0) return;
  const int64_t at = step * tri_block(nsb, 0);
  resid_block<FULL>(glb(G) + step * m * m, m, b, gb, glb(tri) + (at + tri_block(I, 0)) * 256, I, J,
                    L, glb(res) + (at + tri_block(I, J)) * 256);
}

// Superblock (I, J) of T^-1 = Z + R Z by a wave, all three of one step.
__device__ __forceinline__ void refine_block(gptr<const double> Z, gptr<const double> R, int I,
                                             int J, int lane, gptr<double> out) {
  typedef double dv2 __attribute__((ext_vector_type(2)));
  constexpr int U = 4;   // products in flight
  double a[U][4], z[U][4], z0[4];
  const gptr<const double> Rr = R + (int64_t)tri_block(I, 0) * 256 + lane;
  auto load = [&](int t, int q) {
    t = min(t, I);
#pragma unroll
    for (int s = 0; s < 4; ++s) a[q][s] = Rr[(int64_t)t * 256 + 64 * s];
    tri_load(Z + (int64_t)tri_block(t, J) * 256, lane, z[q]);
  };
  tri_load(Z + (int64_t)tri_block(I, J) * 256, lane, z0);
#pragma unroll
  for (int q = 0; q < U; ++q) load(J + q, q);
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
  for (int t0 = J; t0 <= I; t0 += U) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (t0 + q <= I) {   // uniform
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[s & 1] = gdev::mfma(a[q][s], z[q][s], acc[s & 1]);
      }
      load(t0 + U + q, q);
    }
  }
  const d4 c = acc[0] + acc[1];
  const gptr<double> o = out + (int64_t)tri_block(I, J) * 256;
  *(gptr<dv2>)(o + 2 * lane) = dv2{z0[0] + c[0], z0[1] + c[1]};
  *(gptr<dv2>)(o + 128 + 2 * lane) = dv2{z0[2] + c[2], z0[3] + c[3]};
}

// Superblock 4 x + wave of step blockIdx.y of T^-1 from Z (`tri`) and the residual, for the
// rows in need.
__global__ __launch_bounds__(256) void chain_refine_kernel(int nsb, const double* __restrict__ tri,
                                                           const int* __restrict__ need,
                                                           const double* __restrict__ res,
                                                           double* __restrict__ out) {
  const int n = tri_block(nsb, 0);
  const int x = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
  if (x >= n) return;
  int I, J;
  tri_place(n - 1 - x, I, J);   // (the longest first)
  const int64_t step = blockIdx.y;
  if (need[step * nsb + I] == 0) return;
  refine_block(glb(tri) + step * n * 256, glb(res) + step * n * 256, I, J, threadIdx.x & 63,
               glb(out) + step * n * 256);
}

// Steps of up to kSmallSuper superblocks: all of the above by one workgroup, wave w
// superblock row w, with T and Z in registers (Z comes transposed and is the next product's
// operand as it is).  As launches of their own the parts took 20 us of a call of one step.
constexpr int kSmallSuper = 4;
template <bool FULL>
__global__ __launch_bounds__(64 * kSmallSuper) void chain_small_kernel(
    const double* __restrict__ G, int m, int b, int gb, int nsb, const int32_t* __restrict__ idx,
    double* __restrict__ tri, double* __restrict__ raw, double* __restrict__ res,
    int* __restrict__ link) {
  static_assert(kSmallSuper == kResWaves, "resid_block takes the workgroup");
  constexpr int S = kSmallSuper;
  __shared__ double dt[S][256], zw[tri_block(S, 0)][256], gd[16 * S];
  __shared__ int ix[16 * S], bad[S], need[S];
  __shared__ ResLds L;
  const int64_t step = blockIdx.x;
  const int n = tri_block(nsb, 0);
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, l16 = lane >> 4;
  const int I = __builtin_amdgcn_readfirstlane(tid >> 6);
  G += step * m * m;
  const gptr<const double> Gs = glb(G);
  const gptr<double> T = glb(tri) + step * n * 256;
  double a[S][S][4];   // T_tJ of this row's columns
#pragma unroll
  for (int J = 0; J < S; ++J)
#pragma unroll
    for (int t = J + 1; t < S; ++t)
      if (t <= I && I < nsb) load_t<FULL>(Gs, m, gb, t, J, lane, a[J][t]);   // uniform
  if (I == 0) {
    double e[16];
    const bool bd = diag_inverse(G, m, b, gb, nsb, l16, l15, e);
#pragma unroll
    for (int v = 0; v < 16; ++v) dt[l16][16 * l15 + v] = e[v];
    if (l15 == 0) bad[l16] = bd ? 1 : 0;
  } else if (I == 1) {
    const int p = min(lane, m - 1);
    const double v = Gs[(int64_t)p * (m + 1)];
    gd[lane] = lane < m ? v : 0.0;
    ix[lane] = idx[step * m + p];
  }
  __syncthreads();
  if (tid < m) link[step * m + tid] = link_word(ix, m, tid, bad[tid / gb]);
  if (I < nsb) {
    double W[S][4];   // Z_It, transposed
    gdev::static_for<0, S>([&](auto r) {
      constexpr int J = S - 1 - r;
      if (J == I) {   // uniform
#pragma unroll
        for (int s = 0; s < 4; ++s) W[J][s] = dt[J][16 * l15 + 4 * s + l16];
      } else if (J < I) {
        d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = J + 1; t < S; ++t)
          if (t <= I) {
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = gdev::mfma(a[J][t][s], W[t][s], acc);
          }
        double da[4], v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          da[s] = dt[J][64 * s + lane];
          v[s] = acc[s];
        }
        const d4 z = times_dinv(da, v);
#pragma unroll
        for (int s = 0; s < 4; ++s) W[J][s] = z[s];
      }
    });
    double big = 0.0;
    const double gr = l15 < gb ? gd[I * gb + l15] : 0.0;
#pragma unroll
    for (int t = 0; t < S; ++t)
      if (t <= I) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int k = 4 * s + l16;
          big = fmax(big, amplified(W[t][s], k < gb ? gd[t * gb + k] : 0.0, gr));
          zw[tri_block(I, t)][16 * k + l15] = W[t][s];
        }
      }
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    // (with one block a step its inverse is what the solve uses too)
    if (lane == 0) need[I] = m > b && big > kRefineFrom * kRefineFrom ? 1 : 0;
  } else if (lane == 0) {
    need[I] = 0;
  }
  __syncthreads();
  const int any = __builtin_amdgcn_readfirstlane(need[0] | need[1] | need[2] | need[3]);
  const gptr<double> Z = glb(raw) + step * n * 256, R = glb(res) + step * n * 256;
  for (int x = I; x < n; x += S) {   // a wave a superblock
    int i, j;
    tri_place(x, i, j);
    const bool final = need[i] == 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double z = zw[x][16 * l15 + 4 * s + l16];
      if (final) T[x * 256 + tri_at(s, lane)] = z;
      if (any) Z[x * 256 + tri_at(s, lane)] = z;
    }
  }
  if (!any) return;
  __syncthreads();
  for (int i = 0; i < nsb; ++i) {
    if (__builtin_amdgcn_readfirstlane(need[i]) == 0) continue;
    for (int j = 0; j <= i; ++j) {
      resid_block<FULL>(Gs, m, b, gb, Z + (int64_t)tri_block(i, 0) * 256, i, j, L,
                        R + (int64_t)tri_block(i, j) * 256);
      __syncthreads();
    }
  }
  for (int x = I; x < n; x += S) {
    int i, j;
    tri_place(x, i, j);
    if (need[i] != 0) refine_block(Z, R, i, j, lane, T);
  }
}

// ------------------------------------------------------------------ delta = T^-1 c

// Bit i: item i of this lane in a diagonal superblock is in the lower block
// triangle.
__device__ __forceinline__ int diag_mask(int bm, int lane) {
  int mask = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (block_of(lane & 15, bm) <= block_of(4 * i + (lane >> 4), bm)) mask |= 1 << i;
  return mask;
}

// Adds a superblock's products to the four row sums of this lane (cj: the
// right-hand side at this lane's column).  Entries above the block diagonal are
// skipped (mask), not multiplied by zero, so a non-finite entry of c reaches
// its own block and the later ones only.
__device__ __forceinline__ void tri_fma(const double (&v)[4], double cj, bool diag, int mask,
                                        double (&acc)[4]) {
  if (diag) {   // uniform
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double t = fma(v[i], cj, acc[i]);
      acc[i] = (mask >> i) & 1 ? t : acc[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = fma(v[i], cj, acc[i]);
  }
}

constexpr int kStepThreads = 512;
constexpr int kMaxSuper = 32;   // superblocks of a chain step
constexpr int kMaxRows = 512;

// Sparse steps: Y u comes from the row products, x is updated by the companion
// update's launch.  Workgroup i takes superblock rows i and nsb - 1 - i, four
// waves each (wave w the columns J = w mod 4).
__global__ __launch_bounds__(kStepThreads) void chain_delta_kernel(
    const double* __restrict__ tri, const double* __restrict__ Yu, const int32_t* __restrict__ idx,
    const double* __restrict__ x, const double* __restrict__ y, int m, int b, int gb, int nsb,
    int mode, double lambda, double n, double* __restrict__ delta, int* status) {
  __shared__ double c[kMaxSuper * 16];
  __shared__ double red[2][4][16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int I = wave < 4 ? (int)blockIdx.x : nsb - 1 - (int)blockIdx.x;
  const int w = wave & 3;
  const gptr<const double> T = glb(tri) + (int64_t)tri_block(I, 0) * 256;
  const int diag = diag_mask(block_mul(b), lane);
  constexpr int U = 8;   // columns in flight (at most 8 per wave: J < 32)
  double v[U][4];
#pragma unroll
  for (int q = 0; q < U; ++q) tri_load(T + (int64_t)min(w + 4 * q, I) * 256, lane, v[q]);
  c[tid] = 0.0;
  lds_barrier();
  if (tid < m) {
    const int i = idx[tid];
    c[tid / gb * 16 + tid % gb] =
        rhs_of(mode, lambda, n, Yu[tid], x[i], mode == 0 ? 0.0 : y[i]);
  }
  lds_barrier();
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const int J = w + 4 * q;
    if (J <= I) tri_fma(v[q], c[J * 16 + (lane & 15)], J == I, diag, acc);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double s = d16_row_sum(acc[i]);
    if ((lane & 15) == 0) red[wave >> 2][w][4 * i + (lane >> 4)] = s;
  }
  lds_barrier();
  if (tid < 32) {
    const int h = tid >> 4, r = tid & 15;
    const int Ir = h == 0 ? (int)blockIdx.x : nsb - 1 - (int)blockIdx.x;
    const int p = Ir * gb + r;
    if (r < gb && p < m && (h == 0 || Ir != (int)blockIdx.x)) {
      const double d = (red[h][0][r] + red[h][1][r]) + (red[h][2][r] + red[h][3][r]);
      delta[p] = d;
      if (!isfinite(d)) raise_status(status, DEV_NONFINITE);
    }
  }
}

// ------------------------------------------------------------------ dense steps

template <int FMT>
struct Chunk {
  static constexpr int ES = FMT == CABCD_F64 ? 8 : (FMT == CABCD_BF16 ? 2 : 1);
  static constexpr int EPC = 16 / ES;
  // 16 bytes of a row.  FP64 rows may start on any 8-byte boundary: the load
  // needs dword alignment only (codes: 16-byte boundaries).
  static __device__ __forceinline__ uint4 load(gptr<const uint8_t> p) {
    typedef unsigned int uv4 __attribute__((ext_vector_type(4)));
    typedef unsigned int uv4_8 __attribute__((ext_vector_type(4), aligned(8)));
    if constexpr (FMT == CABCD_F64) {
      const uv4_8 t = *(gptr<const uv4_8>)p;
      return make_uint4(t.x, t.y, t.z, t.w);
    } else {
      const uv4 t = *(gptr<const uv4>)p;
      return make_uint4(t.x, t.y, t.z, t.w);
    }
  }
  static __device__ __forceinline__ void decode(const uint4& x, double (&e)[EPC]) {
    if constexpr (FMT == CABCD_F64)
      __builtin_memcpy(e, &x, 16);
    else
      ldev::lp_decode_all<FMT>(x, e);
  }
  // element e of a row
  static __device__ __forceinline__ double one(gptr<const uint8_t> row, int64_t e) {
    if constexpr (FMT == CABCD_F64)
      return *(gptr<const double>)(row + 8 * e);
    else if constexpr (FMT == CABCD_BF16)
      return decode_bf16(*(gptr<const uint16_t>)(row + 2 * e));
    else
      return (double)__builtin_amdgcn_cvt_pk_f32_fp8((int)row[e], false)[0];
  }
};

__device__ __forceinline__ double wave_total(double v) {
  v = d16_row_sum(v);
  return (gdev::d16_read_lane(v, 0) + gdev::d16_read_lane(v, 16)) +
         (gdev::d16_read_lane(v, 32) + gdev::d16_read_lane(v, 48));
}

// LDS of a step launch (doubles): the row sums of Y u, c, delta, then the slab
// of u, then the region where row groups and waves meet.
__host__ __device__ constexpr int64_t step_lds(int epc, int lc, int m) {
  const int slab = lc * epc;
  const int groups = lc >= 64 ? kStepThreads : 8 * lc;   // (row group, chunk) pairs that meet
  const int part = lc > 64 ? lc / 64 * m : 0;
  return 2 * kStepThreads + kMaxSuper * 16 + kMaxRows + slab +
         (groups * epc > part ? groups * epc : part);
}

// One launch of the chain of dense steps (see the file header).  Workgroups
// x < slabs take LC = 2^lc whole 16-byte chunks of the columns each: thread t
// owns chunk t % LC for the rows t / LC + RG q (RG = 512 / LC row groups; LC is
// 16 or at least 64, so a chunk's lanes meet inside rows of sixteen or whole
// waves).  With `tail` one more takes the columns past the last whole chunk,
// thread p row p.  The last one updates x.
//
// Everything a workgroup reads from memory is asked for up front, with no
// branch between the loads (clamped places instead), because the launch is a
// chain of latencies: row indices, rows, partial sums and T^-1 in one go, then
// LDS-only barriers, which leave the loads in flight.  Sums over slabs, row
// groups and lanes run in fixed orders, and the products with the next step's
// rows are the same code with and without the step before them, so a run gives
// the same bits however it is split into calls.
//
// TALL: more than kFewRows rows a step (few slabs, deep prefetch, one workgroup
// a CU); else two workgroups fit a CU, so that 256 wide slabs and the
// workgroup that updates x run at once.
constexpr int kFewRows = 32;
constexpr int kPrefetchWgs = 8;
template <int FMT, bool TALL>
__global__ __launch_bounds__(kStepThreads, TALL ? 2 : 4) void chain_step_kernel(ChainStep a) {
  using C = Chunk<FMT>;
  constexpr int ES = C::ES, EPC = C::EPC;
  // rows in flight per thread and pass
  constexpr int U = FMT == CABCD_F64 ? 8 : TALL || FMT == CABCD_BF16 ? 4 : 2;
  constexpr int PT = TALL ? 6 : 2;                 // superblocks of T^-1 in flight per wave
  constexpr int UP = TALL ? 12 : 2;                // partial sums in flight per thread
  extern __shared__ __attribute__((aligned(16))) double sm[];
  const int m = a.m, LC = 1 << a.lc, RG = kStepThreads >> a.lc;
  double* red = sm;
  double* c = red + 2 * kStepThreads;
  double* dl = c + kMaxSuper * 16;
  double* us = dl + kMaxRows;
  double* meet = us + (int64_t)LC * EPC;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroups past the one that updates x bring the next step's T^-1 into the
  // L2 caches (workgroups go to the eight XCDs in turn)
  const int nwork = (int)gridDim.x - (a.tri1 != nullptr ? kPrefetchWgs : 0);
  if ((int)blockIdx.x >= nwork) {
    const gptr<const uint4> t1 = (gptr<const uint4>)glb(a.tri1);
    const int n = tri_block(a.nsb, 0) * 128;   // 16-byte pieces
    for (int q = threadIdx.x; q < n; q += 4 * kStepThreads) {
      typedef unsigned int uv4 __attribute__((ext_vector_type(4)));
      uv4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *(gptr<const uv4>)(t1 + min(q + i * kStepThreads, n - 1));
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(v[i]));
    }
    return;
  }
  const bool xwg = (int)blockIdx.x == nwork - 1;            // updates x
  const bool twg = a.tail && (int)blockIdx.x == a.nslab - 1;   // the ragged columns
  const int cp = tid & (LC - 1), rg = tid >> a.lc;
  const int64_t nchunk = a.cols / EPC;
  const int64_t chunk = (int64_t)blockIdx.x * LC + cp;
  const bool live = chunk < nchunk;
  const bool upd = a.step && a.upd;
  const bool dots = a.idx1 != nullptr;
  const int64_t kb = (live ? chunk : 0) * 16;               // byte offset in a row
  const gptr<const uint8_t> A = glb(a.A) + kb;
  const int32_t* ixa = upd ? a.idx : a.ix;                  // a.ix: any step's indices
  const int32_t* ixb = dots ? a.idx1 : a.ix;

  // ---- the loads
  int i0[U], i1[U];
  auto load_index = [&](const int32_t* ix, int p0, int(&i)[U]) {
#pragma unroll
    for (int q = 0; q < U; ++q) i[q] = ix[min(p0 + q * RG, m - 1)];
  };
  load_index(ixa, rg, i0);
  load_index(ixb, rg, i1);
  // partial Y u: a thread adds two neighbouring rows of the slabs gp + NG t
  typedef double dv2 __attribute__((ext_vector_type(2)));
  const int PS = 1 << a.ps, PH = PS >> 1, gp = tid >> (a.ps - 1), NG = kStepThreads >> (a.ps - 1);
  const int pt = min(tid, m - 1);
  const double xi = a.xg[pt];
  const double sc = FMT != CABCD_F64 ? a.xg[m + pt] : 1.0;
  dv2 pv[UP];
  const gptr<const double> P = glb(a.P) + 2 * (tid & (PH - 1));
  const int np = (a.nslab + NG - 1) / NG;   // partial sums a thread adds
  auto pload = [&](int t0) {
#pragma unroll
    for (int t = 0; t < UP; ++t)
      pv[t] = *(gptr<const dv2>)(P + (int64_t)min(gp + (t0 + t) * NG, a.nslab - 1) * PS);
  };
  pload(0);
  // this wave's superblocks: the rows w, 15 - w, 16 + w and 31 - w below nsb
  double ring[PT][4];
  int In = wave, Jn = 0;   // the next superblock to load
  int I = wave, J = 0;     // the next superblock to use
  const gptr<const double> T = glb(a.tri);
  auto tload = [&](double(&v)[4]) {
    const int blk = In < a.nsb ? tri_block(In, Jn) : 0;
    tri_load(T + (int64_t)blk * 256, lane, v);
    const bool end = Jn == In;
    Jn = end ? 0 : Jn + 1;
    In += !end ? 0 : (In & 8) ? 2 * wave + 1 : 15 - 2 * wave;
  };
#pragma unroll
  for (int t = 0; t < PT; ++t) tload(ring[t]);
  uint4 c0[U], c1[U];
  auto load_rows = [&](const int(&ix)[U], uint4(&v)[U]) {
#pragma unroll
    for (int q = 0; q < U; ++q) v[q] = C::load(A + (int64_t)ix[q] * a.ld * ES);
  };
  load_rows(i0, c0);
  load_rows(i1, c1);
  double uo[EPC];   // (the owners of u are the threads below LC)
  {
    const gptr<const double> ug = glb(a.u) + (live ? chunk : 0) * EPC;
#pragma unroll
    for (int e = 0; e < EPC; ++e) uo[e] = ug[e];
  }

  // ---- c and delta = T^-1 c
  if (a.step) {
    double y0 = 0.0, y1 = 0.0;
    for (int t0 = 0;;) {
#pragma unroll
      for (int t = 0; t < UP; ++t) {
        const bool in = gp + (t0 + t) * NG < a.nslab;
        y0 += in ? pv[t].x : 0.0;
        y1 += in ? pv[t].y : 0.0;
      }
      t0 += UP;
      if (t0 >= np) break;
      pload(t0);
    }
    for (int off = PH; off < 64; off <<= 1) {
      y0 += __shfl_xor(y0, off, 64);
      y1 += __shfl_xor(y1, off, 64);
    }
    const int groups = PH < 64 ? 8 : NG;
    if (PH >= 64 || lane < PH)
      *reinterpret_cast<dv2*>(red + (PH >= 64 ? gp : wave) * PS + 2 * (tid & (PH - 1))) =
          dv2{y0, y1};
    c[tid] = 0.0;
    lds_barrier();
    if (tid < m) {
      double v[8], s = 0.0;
#pragma unroll
      for (int g = 0; g < 8; ++g) v[g] = red[min(g, groups - 1) * PS + tid];
#pragma unroll
      for (int g = 0; g < 8; ++g) s += g < groups ? v[g] : 0.0;
      const int sb = (tid * a.gbm) >> 16;   // tid / gb
      c[16 * sb + tid - sb * a.gb] = rhs_of(a.mode, a.lambda, a.n, sc * s, xi, 0.0);
    }
    lds_barrier();
    const int diag = diag_mask(a.bm, lane);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    while (I < a.nsb) {
#pragma unroll
      for (int t = 0; t < PT; ++t) {
        if (I < a.nsb) {   // uniform
          tri_fma(ring[t], c[J * 16 + (lane & 15)], J == I, diag, acc);
          tload(ring[t]);
          if (J++ == I) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const double s = d16_row_sum(acc[i]);
              acc[i] = 0.0;
              const int row = 4 * i + (lane >> 4);
              if ((lane & 15) == 0 && row < a.gb && I * a.gb + row < m) dl[I * a.gb + row] = s;
            }
            J = 0;
            I += (I & 8) ? 2 * wave + 1 : 15 - 2 * wave;
          }
        }
      }
    }
    lds_barrier();
  }

  // ---- x[idx] += delta, and x at the next step's indices
  if (xwg) {
    if (a.step) {
      if (tid < m && !isfinite(dl[tid])) raise_status(a.status, DEV_NONFINITE);
      cdev::scatter_delta<kStepThreads>(a.idx, a.link, dl, m, a.x, a.status);
      __syncthreads();
    }
    if (dots && tid < m) {   // (the dual's right-hand side takes x + y)
      const int i = a.idx1[tid];
      a.xg1[tid] = a.mode != 0 ? a.x[i] + a.y[i] : a.x[i];
      if (FMT != CABCD_F64) a.xg1[m + tid] = a.rs != nullptr ? (double)a.rs[i] : 1.0;
    }
    return;
  }
  if (FMT != CABCD_F64 && upd && a.rs != nullptr) {
    if (tid < m) dl[tid] *= sc;
    lds_barrier();
  }

  // ---- the ragged columns: thread p holds row p's elements
  if (twg) {
    const int rem = (int)(a.cols - nchunk * EPC);
    // (u is read once, into LDS: the barriers below do not order global memory)
    if (tid < rem) us[tid] = glb(a.u)[nchunk * EPC + tid];
    lds_barrier();
    const gptr<const uint8_t> At = glb(a.A);
    const gptr<const uint8_t> row0 = At + (int64_t)ixa[pt] * a.ld * ES;
    const gptr<const uint8_t> row1 = At + (int64_t)ixb[pt] * a.ld * ES;
    double t1 = 0.0;
    for (int e = 0; e < rem; ++e) {
      const int64_t k = nchunk * EPC + e;
      double un = us[e];
      if (upd) {
        const double d = tid < m ? dl[tid] : 0.0;
        const double x = tid < m ? C::one(row0, k) : 0.0;
        const double w = wave_total(x * d);
        if (lane == 0) red[wave] = w;
        lds_barrier();
        double s = 0.0;
#pragma unroll
        for (int g = 0; g < 8; ++g) s += red[g];
        lds_barrier();
        un += a.gamma * s;
        if (tid == 0) glb(a.u)[k] = un;
      }
      if (dots && tid < m) t1 = fma(C::one(row1, k), un, t1);
    }
    if (dots && tid < m) a.P1[(int64_t)blockIdx.x * PS + tid] = t1;
    return;
  }

  // ---- the slab of u
  if (upd) {
    double acc[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) acc[e] = 0.0;
    for (int p0 = rg;;) {
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int p = p0 + q * RG;
        double x[EPC];
        C::decode(c0[q], x);
        const double d = dl[min(p, m - 1)];
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[e] = p < m ? fma(x[e], d, acc[e]) : acc[e];
      }
      p0 += U * RG;
      if (p0 - rg >= m) break;   // uniform
      load_index(ixa, p0, i0);
      load_rows(i0, c0);
    }
    // the row groups of a chunk: inside a wave, then through LDS
    if (LC == 16) {
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] += __shfl_xor(acc[e], 16, 64);
#pragma unroll
      for (int e = 0; e < EPC; ++e) acc[e] += __shfl_xor(acc[e], 32, 64);
    }
    const int groups = LC == 16 ? 8 : RG;
    if (groups > 1) {
      if (LC >= 64 || lane < 16) {
#pragma unroll
        for (int e = 0; e < EPC; ++e)
          meet[((LC == 16 ? wave : rg) * EPC + e) * LC + cp] = acc[e];
      }
      lds_barrier();
      if (tid < LC) {
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
          double s = 0.0, v[8];
#pragma unroll
          for (int g = 0; g < 8; ++g) v[g] = meet[(min(g, groups - 1) * EPC + e) * LC + tid];
#pragma unroll
          for (int g = 0; g < 8; ++g) s += g < groups ? v[g] : 0.0;
          acc[e] = s;
        }
      }
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) uo[e] += a.gamma * acc[e];
    if (tid < LC && live) {
      const gptr<double> ug = glb(a.u) + chunk * EPC;
#pragma unroll
      for (int e = 0; e < EPC; ++e) ug[e] = uo[e];
    }
  }
  if (!dots) return;

  // ---- the slab's products with the next step's rows
  if (tid < LC) {
#pragma unroll
    for (int e = 0; e < EPC; ++e) us[e * LC + tid] = uo[e];
  }
  lds_barrier();
  double ul[EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) ul[e] = us[e * LC + cp];
  const gptr<double> P1 = glb(a.P1) + (int64_t)blockIdx.x * PS;
  for (int p0 = rg;;) {
    double t[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      double x[EPC];
      C::decode(c1[q], x);
      t[q] = 0.0;
#pragma unroll
      for (int e = 0; e < EPC; ++e) t[q] = fma(x[e], ul[e], t[q]);
      t[q] = live ? t[q] : 0.0;
    }
    if (LC == 16) {
#pragma unroll
      for (int q = 0; q < U; ++q) t[q] = d16_row_sum(t[q]);
      if (cp == 0) {
#pragma unroll
        for (int q = 0; q < U; ++q)
          if (p0 + q * RG < m) P1[p0 + q * RG] = t[q];
      }
    } else {
#pragma unroll
      for (int q = 0; q < U; ++q) t[q] = wave_total(t[q]);
      if (lane == 0) {
#pragma unroll
        for (int q = 0; q < U; ++q)
          if (p0 + q * RG < m) {
            if (LC == 64)
              P1[p0 + q * RG] = t[q];
            else
              meet[(wave & (LC / 64 - 1)) * m + p0 + q * RG] = t[q];
          }
      }
    }
    p0 += U * RG;
    if (p0 - rg >= m) break;   // uniform
    load_index(ixb, p0, i1);
    load_rows(i1, c1);
  }
  if (LC > 64) {
    lds_barrier();
    if (tid < m) {
      double s = 0.0;
      for (int w = 0; w < LC / 64; ++w) s += meet[w * m + tid];
      P1[tid] = s;
    }
  }
}

// ------------------------------------------------------------- few and short rows
// Runs of steps in one launch by one workgroup, where a step's rows fit its registers
// (32 elements a thread: 128 KiB) and T^-1 has at most a row of superblocks a wave.  The
// companion stays in LDS and a thread holds its elements of the step's rows from the
// products with u to the update; the next step's come from the L2 after that.  What
// bounds a step is one chain of latencies (rows, sums over the wave and the workgroup,
// T^-1 c, the sums of the update) and, towards 128 KiB, the 50 GB/s or so that a CU
// reads.  A launch a step also waits for its own start and for the other XCDs' partial
// sums.  Marginal time of a step, launches -> here (us): dense dual b s = 32, d = 64:
// 8.1 -> 3.8; 64, 128: 9.2 -> 5.3; 32, 512: 8.4 -> 6.7; 64, 256: 9.2 -> 7.2; primal d =
// 64, n = 256, b s = 32: 8.3 -> 4.9.  With 64 elements a thread (256 KiB) 32, 1024 was 8.4
// -> 8.4 and 64, 512 9.5 -> 10.7, so the line is at half of that; rows asked for a step
// ahead into registers of their own gained nothing.
//
// Column c + LC j (c = thread % LC) and row rg + RG q (rg = thread / LC, RG = 512 / LC)
// is slot q CJ + j; LC is a power of two from 64 on, CJ = columns / LC, so a wave's 64
// lanes lie in one row.
constexpr int kSoloThreads = 512;
constexpr int kSoloSlots = 32;                 // elements a thread holds
constexpr int kSoloSuper = 8;                  // superblocks of T^-1, at most: one a wave
// Columns a thread holds of a row: a power of two.
int solo_cj(int64_t cols) {
  int cj = 1;
  while (cj * kSoloThreads < cols) cj *= 2;
  return cj;
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <bool HALF32>   // swaps halves of 32 lanes, or neighbouring rows of 16
__device__ __forceinline__ double swap_add(double a, double b) {
  const unsigned alo = __double2loint(a), ahi = __double2hiint(a);
  const unsigned blo = __double2loint(b), bhi = __double2hiint(b);
  u32x2 lo, hi;
  if constexpr (HALF32) {
    const auto l = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
    lo = u32x2{l[0], l[1]};
    hi = u32x2{h[0], h[1]};
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
    lo = u32x2{l[0], l[1]};
    hi = u32x2{h[0], h[1]};
  }
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// The sums over a wave of its lanes' sixteen values; lane l gets that of value l / 4.
// Every exchange halves the values a lane holds, so sixteen sums take 15 + 2 additions.
__device__ __forceinline__ double wave_sums16(double (&v)[16], int lane) {
  double a[8], b[4];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = swap_add<true>(v[i], v[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = swap_add<false>(a[i], a[i + 4]);
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
  const double c0 = (b3 ? b[2] : b[0]) + dpp<0x128>(b3 ? b[0] : b[2]);   // row_ror:8
  const double c1 = (b3 ? b[3] : b[1]) + dpp<0x128>(b3 ? b[1] : b[3]);
  double d = (b2 ? c1 : c0) + dpp<0x141>(b2 ? c0 : c1);                  // row_half_mirror
  d += dpp<0xB1>(d);   // the four lanes of a quad
  d += dpp<0x4E>(d);
  return d;
}

template <int CJ>
__global__ __launch_bounds__(kSoloThreads) void chain_solo_kernel(ChainSolo a,
                                                                 const int32_t* __restrict__ idx) {
  constexpr int QN = kSoloSlots / CJ;   // rows a thread holds
  extern __shared__ __attribute__((aligned(16))) double sm[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = a.m, cols = (int)a.cols, LC = 1 << a.lc, RG = kSoloThreads >> a.lc;
  const int cp = tid & (LC - 1), rg = __builtin_amdgcn_readfirstlane(tid >> a.lc);
  const int W = LC / 64, wq = wave & (W - 1);   // waves side by side in a row
  double* c = sm;                               // kMaxSuper * 16
  double* dl = c + kMaxSuper * 16;              // kMaxRows
  double* red = dl + kMaxRows;                  // kSoloThreads CJ, at least W m
  double* us = red + kSoloThreads * CJ;         // LC CJ
  const bool owner = wave * 64 < m;             // holds rows of x

  const gptr<const double> A = glb(a.A);
  double x[kSoloSlots];                         // the step's rows
  // (opaque: keeps the places of a step's rows out of the registers between steps)
  auto first_row = [&] {
    int r = rg;
    asm volatile("" : "+s"(r));
    return r;
  };
  // lane q holds the index of the wave's row q, a step ahead of its rows
  auto load_index = [&](int step) {
    return glb(idx)[(int64_t)min(step, a.steps - 1) * m + min(rg + lane * RG, m - 1)];
  };
  // eight rows at a time (spares registers), as far as there are rows
  constexpr int B = QN < 8 ? QN : 8;
  auto load_rows = [&](int ix) {
    gdev::static_for<0, QN / B>([&](auto g) {
      __builtin_amdgcn_sched_barrier(0);
      if (B * g * RG < m) {
#pragma unroll
        for (int q = B * g; q < B * g + B; ++q) {
          const gptr<const double> row = A + (int64_t)__builtin_amdgcn_readlane(ix, q) * a.ld;
#pragma unroll
          for (int j = 0; j < CJ; ++j) x[q * CJ + j] = row[min(cp + j * LC, cols - 1)];
        }
      }
    });
  };
#pragma unroll
  for (int q = 0; q < kSoloSlots; ++q) x[q] = 0.0;
  load_rows(load_index(0));
  int nidx = load_index(1);
  c[tid] = 0.0;
  for (int k = tid; k < LC * CJ; k += kSoloThreads) us[k] = k < cols ? glb(a.u)[k] : 0.0;
  const int sb = (tid * a.gbm) >> 16;           // tid / gb
  const int cat = 16 * sb + tid - sb * a.gb;
  const int diag = diag_mask(a.bm, lane);
  __syncthreads();

  for (int step = 0; step < a.steps; ++step) {
    const int32_t* ix = idx + (int64_t)step * m;
    const gptr<const double> T = glb(a.tri) + step * a.tri_stride;
    double xi = 0.0;
    if (tid < m) {   // (the dual's right-hand side takes x + y)
      const int i = ix[tid];
      xi = a.mode != 0 ? glb(a.x)[i] + glb(a.y)[i] : glb(a.x)[i];
    }
    // this wave's row of superblocks of T^-1
    double tr[kSoloSuper][4];
    const int I = min(wave, a.nsb - 1);
#pragma unroll
    for (int J = 0; J < kSoloSuper; ++J)
      tri_load(T + (int64_t)tri_block(I, min(J, I)) * 256, lane, tr[J]);
    // ---- Y u
    {
      double ul[CJ];
#pragma unroll
      for (int j = 0; j < CJ; ++j) ul[j] = us[cp + j * LC];
      constexpr int G = QN < 16 ? QN : 16;
      gdev::static_for<0, QN / G>([&](auto g) {
        constexpr int q0 = g * G;
        __builtin_amdgcn_sched_barrier(0);
        if (q0 * RG < m) {   // uniform
          double t[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            t[q] = 0.0;
            if (q < G) {
#pragma unroll
              for (int j = 0; j < CJ; ++j) t[q] = fma(x[(q0 + q) * CJ + j], ul[j], t[q]);
            }
          }
          const double s = wave_sums16(t, lane);
          const int p = rg + (q0 + (lane >> 2)) * RG;
          if ((lane & 3) == 0 && (lane >> 2) < G && p < m) red[wq * m + p] = s;
        }
      });
    }
    lds_barrier();
    if (tid < m) {
      double v[8], s = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) v[w] = red[min(w, W - 1) * m + tid];
#pragma unroll
      for (int w = 0; w < 8; ++w) s += w < W ? v[w] : 0.0;
      c[cat] = rhs_of(a.mode, a.lambda, a.n, s, xi, 0.0);
    }
    lds_barrier();
    // ---- delta = T^-1 c
    if (wave < a.nsb) {
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int J = 0; J < kSoloSuper; ++J)
        if (J <= I) tri_fma(tr[J], c[J * 16 + (lane & 15)], J == I, diag, acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double s = d16_row_sum(acc[i]);
        const int row = 4 * i + (lane >> 4);
        if ((lane & 15) == 0 && row < a.gb && I * a.gb + row < m) dl[I * a.gb + row] = s;
      }
    }
    lds_barrier();
    // ---- u += gamma Y^T delta
    if (step + 1 < a.steps || a.last_upd) {
      double acc[CJ];
#pragma unroll
      for (int j = 0; j < CJ; ++j) acc[j] = 0.0;
      const int r0 = first_row();
      gdev::static_for<0, QN / B>([&](auto g) {
        __builtin_amdgcn_sched_barrier(0);
        if (B * g * RG < m) {
#pragma unroll
          for (int q = B * g; q < B * g + B; ++q) {
            const int p = r0 + q * RG;
            const double d = dl[min(p, m - 1)];
#pragma unroll
            for (int j = 0; j < CJ; ++j) acc[j] = p < m ? fma(x[q * CJ + j], d, acc[j]) : acc[j];
          }
        }
      });
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        if (RG > 1)
          red[rg * LC + cp] = acc[j];   // (CJ = 1)
        else if (cp + j * LC < cols)   // (u stays 0 past the last column)
          us[cp + j * LC] += a.gamma * acc[j];
      }
    }
    // ---- x[idx] += delta: one writer per coordinate
    if (tid < m) {
      if (!isfinite(dl[tid])) raise_status(a.status, DEV_NONFINITE);
      cdev::scatter_delta<kSoloThreads>(ix, a.link + (int64_t)step * m, dl, m, a.x, a.status);
    }
    if (owner) __builtin_amdgcn_s_waitcnt(0);   // x is read again after the barrier
    asm volatile("" ::: "memory");
    lds_barrier();
    asm volatile("" ::: "memory");
    load_rows(nidx);
    nidx = load_index(step + 2);
    if (RG > 1 && (step + 1 < a.steps || a.last_upd)) {
      if (tid < cols) {
        double v[8], s = 0.0;
#pragma unroll
        for (int g = 0; g < 8; ++g) v[g] = red[min(g, RG - 1) * LC + tid];
#pragma unroll
        for (int g = 0; g < 8; ++g) s += g < RG ? v[g] : 0.0;
        us[tid] += a.gamma * s;
      }
      lds_barrier();
    }
  }
  if (a.steps > 1 || a.last_upd) {
    __syncthreads();
    for (int k = tid; k < cols; k += kSoloThreads) glb(a.u)[k] = us[k];
  }
}

}  // namespace

ChainPlan chain_plan(int m, int b) {
  ChainPlan p{};
  if (b < 1 || b > 16 || m < 1 || m > kMaxRows || m % b != 0) return p;
  p.gb = 16 / b * b;
  p.nsb = (m + p.gb - 1) / p.gb;
  p.ok = p.nsb <= kMaxSuper;
  p.tri = (size_t)tri_block(p.nsb, 0) * 256;
  p.work = (size_t)p.nsb * 257 + 2 * p.tri;
  return p;
}

hipError_t launch_chain_prepare(const ChainPlan& p, const double* G, int nsteps, int m, int b,
                                const int32_t* idx, double* tri, double* work, int* link,
                                hipStream_t st) {
  if (!p.ok || nsteps < 1 || nsteps > 65535) return hipErrorInvalidValue;
  double* raw = work;
  double* res = raw + (size_t)nsteps * p.tri;
  double* dinv = res + (size_t)nsteps * p.tri;
  int* bad_block = reinterpret_cast<int*>(dinv + (size_t)nsteps * p.nsb * 256);
  int* need = bad_block + (size_t)nsteps * p.nsb;
  const bool full = p.gb == 16 && m % 16 == 0;
  if (p.nsb <= kSmallSuper) {
    hipLaunchKernelGGL(full ? chain_small_kernel<true> : chain_small_kernel<false>,
                       dim3((unsigned)nsteps), dim3(64 * kSmallSuper), 0, st, G, m, b, p.gb, p.nsb,
                       idx, tri, raw, res, link);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(chain_diag_kernel, dim3((unsigned)((p.nsb + 3) / 4), (unsigned)nsteps),
                     dim3(64), 0, st, G, m, b, p.gb, p.nsb, raw, dinv, bad_block);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = std::max((size_t)(2 * kPanelWaves + p.nsb) * 256 * sizeof(double),
                              (size_t)m * sizeof(int));
  auto kern = full ? chain_panel_kernel<true> : chain_panel_kernel<false>;
  if (lds > 64 * 1024) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)p.nsb + 1, (unsigned)nsteps), dim3(64 * kPanelWaves),
                     lds, st, G, m, p.gb, p.nsb, raw, dinv, idx, link, bad_block, tri, need);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const unsigned n = (unsigned)tri_block(p.nsb, 0);
  hipLaunchKernelGGL(full ? chain_resid_kernel<true> : chain_resid_kernel<false>,
                     dim3(n, (unsigned)nsteps), dim3(64 * kResWaves), 0, st, G, m, b, p.gb, p.nsb,
                     raw, need, res);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(chain_refine_kernel, dim3((n + 3) / 4, (unsigned)nsteps), dim3(256), 0, st,
                     p.nsb, raw, need, res, tri);
  return hipGetLastError();
}

hipError_t launch_chain_delta(const ChainPlan& p, const double* tri, const double* Yu,
                              const int32_t* idx, const double* x, const double* y, int m, int b,
                              int mode, double lambda, double n, double* delta, int* status,
                              hipStream_t st) {
  if (!p.ok) return hipErrorInvalidValue;
  hipLaunchKernelGGL(chain_delta_kernel, dim3((unsigned)((p.nsb + 1) / 2)), dim3(kStepThreads), 0,
                     st, tri, Yu, idx, x, y, m, b, p.gb, p.nsb, mode, lambda, n, delta, status);
  return hipGetLastError();
}

// The slabs of u: 16 or 64 to 512 chunks a workgroup, so that at most 256
// workgroups share the columns.  Narrow slabs spread a step's rows over more
// CUs; every workgroup reads all slabs' partial Y u.
ChainSlabs chain_slabs(int dtype, int m, int64_t cols) {
  const int epc = dtype == CABCD_F64 ? 2 : (dtype == CABCD_BF16 ? 8 : 16);
  const int64_t chunks = cols / epc;
  ChainSlabs s{};
  s.lc = 4;
  while (s.lc < 9 && chunks > (int64_t)256 << s.lc) s.lc = s.lc == 4 ? 6 : s.lc + 1;
  s.tail = cols % epc != 0 ? 1 : 0;
  s.nslab = (int)((chunks + (1 << s.lc) - 1) >> s.lc) + s.tail;
  s.ps = 1;
  while ((1 << s.ps) < m) ++s.ps;
  s.partial = (size_t)s.nslab << s.ps;
  return s;
}

hipError_t launch_chain_step(int dtype, const ChainStep& step, hipStream_t st) {
  ChainStep a = step;
  const int epc = dtype == CABCD_F64 ? 2 : (dtype == CABCD_BF16 ? 8 : 16);
  if (a.m < 1 || a.m > kMaxRows || a.nsb > kMaxSuper || a.lc < 4 || a.lc == 5 || a.lc > 9 ||
      a.ps < 1 || (1 << a.ps) < a.m || (1 << a.ps) > kStepThreads || a.cols < epc)
    return hipErrorInvalidValue;
  const unsigned grid = ((a.step && a.upd) || a.idx1 != nullptr ? a.nslab : 0) + 1 +
                        (a.tri1 != nullptr ? kPrefetchWgs : 0);
  const size_t lds = (size_t)step_lds(epc, 1 << a.lc, a.m) * sizeof(double);
  a.bm = block_mul(a.b);
  a.gbm = (65535 + a.gb) / a.gb;
  const bool tall = a.m > kFewRows;
  using Kern = void (*)(ChainStep);
  const Kern kerns[3][2] = {
      {chain_step_kernel<CABCD_F64, false>, chain_step_kernel<CABCD_F64, true>},
      {chain_step_kernel<CABCD_BF16, false>, chain_step_kernel<CABCD_BF16, true>},
      {chain_step_kernel<CABCD_FP8_E4M3, false>, chain_step_kernel<CABCD_FP8_E4M3, true>}};
  const Kern kern = kerns[dtype == CABCD_F64 ? 0 : (dtype == CABCD_BF16 ? 1 : 2)][tall ? 1 : 0];
  if (lds > 64 * 1024) {   // beyond the default limit (wide slabs of codes)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kStepThreads), lds, st, a);
  return hipGetLastError();
}

// Column lanes (log2) of chain_solo_kernel for m rows of cols FP64 columns with nsb
// superblocks, or -1 where a launch a step is the way (see there).
int chain_solo_lc(int m, int64_t cols, int nsb) {
  if (nsb > kSoloSuper || cols > 8 * kSoloThreads) return -1;
  int lc = 6;
  while ((1 << lc) < cols && lc < 9) ++lc;
  const int64_t cj = solo_cj(cols);
  return cj * ((m + (kSoloThreads >> lc) - 1) / (kSoloThreads >> lc)) <= kSoloSlots ? lc : -1;
}

hipError_t launch_chain_solo(const ChainSolo& args, hipStream_t st) {
  ChainSolo a = args;
  if (a.steps < 1 || chain_solo_lc(a.m, a.cols, a.nsb) != a.lc || a.lc < 0)
    return hipErrorInvalidValue;
  a.bm = block_mul(a.b);
  a.gbm = (65535 + a.gb) / a.gb;
  const int cj = solo_cj(a.cols);
  const size_t lds = sizeof(double) *
                     (kMaxSuper * 16 + kMaxRows + (size_t)kSoloThreads * cj + ((size_t)cj << a.lc));
  auto go = [&](auto kernel) -> hipError_t {
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSoloThreads), lds, st, a, a.idx);
    return hipGetLastError();
  };
  switch (cj) {
    case 1: return go(chain_solo_kernel<1>);
    case 2: return go(chain_solo_kernel<2>);
    case 4: return go(chain_solo_kernel<4>);
    case 8: return go(chain_solo_kernel<8>);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace cabcd
