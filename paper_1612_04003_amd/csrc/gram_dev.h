// Device code of the dense FP64 Gram of gathered rows on the CDNA4 matrix
// cores, shared by the one-problem kernels and the batched persistent kernel.
//
// Computes the s-step Gram Y Y^T of Alg. 2 (Y = [I_1..I_s]^T X, rows of X) and
// Alg. 4 (Y = X[I_1..I_s], rows of X^T), together with Y u for the companion
// vector u (the residual products of eq. recur / the dual recurrence).  The
// paper forms this with MKL on CSR on every MPI rank (Section 5.2); here it is
// one launch per outer step:
//
// * The reduction dimension (cols of A) is split into `chunk`-wide slabs, one
//   workgroup each (split-K), so that hundreds of workgroups cover a thin
//   m x m output with K in the hundreds of thousands.
// * A workgroup streams its slab through LDS in KT-wide tiles: the m gathered
//   rows go from HBM straight into LDS (LDS-DMA of 16 bytes a lane, which needs
//   dword alignment only, so rows may start on any 8-byte boundary: 6.0 TB/s
//   from odd ones as from 16-byte ones), double-buffered, and Y u is accumulated
//   in FP64 from the tile, so Y is read from HBM exactly once.
// * The lower triangle of 16x16 output blocks is computed with
//   v_mfma_f64_16x16x4_f64.  Each wave owns the blocks of two block rows
//   (r, NB-1-r), so every wave has NB+1 accumulators and reads at most NB
//   fragments per k-step.  For small NB the waves also split the k-steps of a
//   tile and are summed through LDS at the end.
// * The MFMA reduction index is permuted: lane group g of a 128-bit fragment
//   read supplies columns 8p+2g and 8p+2g+1 to two consecutive MFMAs.  Any
//   bijection of k works because both operands use the same one.
// * Each workgroup writes its partial blocks; they are summed in split order
//   (deterministic) by a second kernel or, in the batched persistent kernel,
//   by the problem's last workgroup, which applies scale and shift in FP64 and
//   mirrors the result into both triangles.
#pragma once

#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace cabcd {
namespace gdev {

typedef double d4 __attribute__((ext_vector_type(4)));

// Wave layout: eight waves, two per SIMD, a wave owns block rows w and NB-1-w, so
// every wave owns the same number of lower blocks.  Waves that own the same rows
// (KG > 1, small NB) split the k-steps of a tile instead.
template <int NB>
struct Cfg {
  static constexpr int SBP = 16 * NB;                       // padded rows
  static constexpr int NBLK = NB * (NB + 1) / 2;            // lower 16x16 blocks
  static constexpr int KT = 256 / NB;                       // tile width: SBP*KT = 4096
  static constexpr int CH = KT / 2;                         // 16-byte chunks per row
  static constexpr int BW = NB >= 2 ? NB / 2 : 1;           // waves splitting the blocks
  static constexpr int KG = 8 / BW;                         // waves splitting the k-steps
  static constexpr int THREADS = 512;
  static constexpr int NCH = SBP * CH / THREADS;            // chunks per thread per tile
  static constexpr int PAIRS = KT / 8;                      // 128-bit fragment reads per tile
  static constexpr int NACC = NB >= 2 ? NBLK / BW : 1;      // accumulators per wave
  static constexpr int YUS = SBP * CH;
  static_assert(NCH * THREADS == SBP * CH, "tile must split evenly");
  static_assert(PAIRS % KG == 0, "k-steps must split evenly");
  static_assert(NB < 2 || NACC * BW == NBLK, "blocks must split evenly");
};

// Index of lower block (r, c) in row-major lower-triangular order.
__host__ __device__ constexpr int blk_index(int r, int c) { return r * (r + 1) / 2 + c; }

// i-th block row owned by wave w.
__host__ __device__ constexpr int owned_row(int NB, int w, int i) {
  return NB == 1 ? 0 : (i == 0 ? w : NB - 1 - w);
}

// First accumulator of owned row i (accumulators of row r are its r+1 blocks).
__host__ __device__ constexpr int acc_offset(int NB, int w, int i) {
  return i == 0 ? 0 : owned_row(NB, w, 0) + 1;
}

// Block index of accumulator a of wave bw.
template <int NB>
__device__ __forceinline__ int acc_block(int bw, int a) {
  if (NB < 2) return 0;
  return a <= bw ? blk_index(bw, a) : blk_index(NB - 1 - bw, a - bw - 1);
}

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Stores and loads of a slab's partial sums.  AGENT: at agent scope (written
// through to, and read from, where every XCD sees them), for a reader in the same
// launch, which then needs no fence: publishing ordinary stores with one writes
// the XCD's whole L2 back, 37 us an item in the batched rounds.
template <bool AGENT>
__device__ __forceinline__ void put(gptr<double> p, double v) {
  if constexpr (AGENT)
    __hip_atomic_store((double*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}
__device__ __forceinline__ double get_agent(gptr<const double> p) {
  return __hip_atomic_load((const double*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// s_waitcnt immediate: no vector memory load outstanding (LDS and scalar counters free).
constexpr int kWaitVm0 = 0x0F70;

// ---------------------------------------------------------------------------
// NB <= 8: waves own block-row pairs and split a tile's k-steps.  A 32 KiB tile of
// SBP rows x
// KT = 256 / NB columns goes from HBM straight into LDS, rows unpadded with the
// 16-byte chunks of each aligned group of sixteen XOR-swizzled by the row
// (chunk c of row r at c ^ (r & 15)), so the sixteen rows of a fragment read
// fall in distinct banks; a thread forms Y u for its four (row, chunk) pairs
// from LDS after the tile lands.  Rows of 256 bytes (NB = 8) to 2 KiB (NB = 1)
// per tile keep the HBM pages busy.
template <int NB>
struct DN {
  using C = Cfg<NB>;
  static constexpr int DMA_PER_WAVE = C::SBP * C::CH / 64 / 8;   // 4 instructions
  static constexpr int UDMA = (C::KT / 2 + 63) / 64;              // u slots, 64 a time
  static constexpr int TILE = C::SBP * C::KT + C::KT;            // doubles: rows, then u
  // accumulators a wave brings to the other k-groups' at a time: what a tile buffer holds
  static constexpr int HA =
      C::KG > 1 ? std::min(C::NACC, TILE / ((C::KG - 1) * C::BW * 256)) : C::NACC;
  static_assert(HA >= 1 && C::YUS <= TILE, "the sums fit a tile buffer");
};

template <int NB, int W>
__device__ __forceinline__ void mma_tile_dma(const double* __restrict__ tile, int lane, int kg,
                                             d4 (&acc)[Cfg<NB>::NACC]) {
  using C = Cfg<NB>;
  constexpr int NR = NB >= 2 ? 2 : 1;
  const int rl = lane & 15, g = lane >> 4;
#pragma unroll
  for (int p = 0; p < C::PAIRS / C::KG; ++p) {
    const int ch = 4 * (kg + p * C::KG) + g;            // chunk (two columns) of this lane
    const double* base = tile + rl * C::KT + 2 * (ch ^ rl);
    auto frag = [&](int r) { return *reinterpret_cast<const double2*>(base + r * 16 * C::KT); };
    double2 fo[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) fo[i] = frag(owned_row(NB, W, i));
    constexpr int CMAX = NB >= 2 ? NB - 1 - W : 0;        // largest owned row
#pragma unroll
    for (int c = 0; c <= CMAX; ++c) {
      double2 fc = {0.0, 0.0};
      bool own = false;
#pragma unroll
      for (int i = 0; i < NR; ++i)
        if (owned_row(NB, W, i) == c) {
          fc = fo[i];
          own = true;
        }
      if (!own) fc = frag(c);
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int r = owned_row(NB, W, i);
        if (c <= r) {
          const int a = acc_offset(NB, W, i) + c;
          acc[a] = mfma(fo[i].x, fc.x, acc[a]);
          acc[a] = mfma(fo[i].y, fc.y, acc[a]);
        }
      }
    }
  }
}

template <int NB, int W = 0>
__device__ __forceinline__ void mma_dispatch_dma(int bw, const double* __restrict__ tile, int lane,
                                                 int kg, d4 (&acc)[Cfg<NB>::NACC]) {
  if constexpr (W < Cfg<NB>::BW) {
    if (bw == W)
      mma_tile_dma<NB, W>(tile, lane, kg, acc);
    else
      mma_dispatch_dma<NB, W + 1>(bw, tile, lane, kg, acc);
  }
}

// One workgroup's slab of the Gram: columns [k_begin, k_end) of the rows
// idx[0..m) of A (m <= 16 NB; idx may point to LDS), u indexed by absolute
// column (NULL: no Y u).  Writes the partial blocks and the partial Y u to
// part[0 .. NBLK*256 + SBP).  t0 and t1: the tile buffers (DN<NB>::TILE doubles),
// __shared__ arrays of their own, as in TriLds: with both in one array every tile waited
// for the next one's DMA before its first read.  Every thread of the workgroup must
// call it.
template <int NB, bool AGENT = false>
__device__ __forceinline__ void gram_slab_dma(const double* __restrict__ A, int64_t ld,
                                              int64_t k_begin, int64_t k_end, const int32_t* idx,
                                              int m, const double* __restrict__ u,
                                              double* __restrict__ part, double* t0, double* t1) {
  using C = Cfg<NB>;
  using D = DN<NB>;
  typedef __attribute__((address_space(3))) void* lds_vptr;
  typedef __attribute__((address_space(1))) const void* glb_vptr;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int bw = __builtin_amdgcn_readfirstlane(wave % C::BW);
  const int kg = __builtin_amdgcn_readfirstlane(wave / C::BW);
  const int ntiles = (int)((k_end - k_begin + C::KT - 1) / C::KT);

  // DMA instruction i of this wave fills slots (4 wave + i) * 64 + lane:
  // row slot / CH, position slot % CH, chunk position ^ (row % 16).
  // Rows past m (padding of the last block row) are never loaded: they are
  // zeroed once in both buffers.
  gptr<const double> src[D::DMA_PER_WAVE];
  int cofs[D::DMA_PER_WAVE];
  bool live[D::DMA_PER_WAVE];
  const gptr<const double> Ag = glb(A);
#pragma unroll
  for (int i = 0; i < D::DMA_PER_WAVE; ++i) {
    const int q = (D::DMA_PER_WAVE * wave + i) * 64 + lane;
    const int r = q / C::CH;
    cofs[i] = 2 * ((q % C::CH) ^ (r & 15));
    live[i] = r < m;
    src[i] = Ag + (int64_t)idx[r < m ? r : 0] * ld;
    if (!live[i]) {
      const int at = (D::DMA_PER_WAVE * wave + i) * 128 + 2 * lane;
      *reinterpret_cast<double2*>(t0 + at) = double2{0.0, 0.0};
      *reinterpret_cast<double2*>(t1 + at) = double2{0.0, 0.0};
    }
  }
  const bool want_u = u != nullptr;
  const gptr<const double> ug = glb(u);
  // (padding rows stay zero; u: the tile's KT entries, unswizzled after the rows)
  auto issue = [&](int t, double* T) {
    const int64_t k0 = k_begin + (int64_t)t * C::KT;
    double* const ud = T + C::SBP * C::KT;
    const bool u_wave = want_u && wave == 7;
    if (k0 + C::KT <= k_end) {
#pragma unroll
      for (int i = 0; i < D::DMA_PER_WAVE; ++i)   // 64 slots of 2 doubles each
        if (live[i])
          __builtin_amdgcn_global_load_lds((glb_vptr)(src[i] + (k0 + cofs[i])),
                                           (lds_vptr)(T + (D::DMA_PER_WAVE * wave + i) * 128), 16,
                                           0, 0);
      if (u_wave) {
#pragma unroll
        for (int j = 0; j < D::UDMA; ++j)
          if (64 * j + lane < C::KT / 2)
            __builtin_amdgcn_global_load_lds((glb_vptr)(ug + (k0 + 2 * (64 * j + lane))),
                                             (lds_vptr)(ud + 128 * j), 16, 0, 0);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < D::DMA_PER_WAVE; ++i) {
      const int64_t k = k0 + cofs[i];
      double2 v;
      v.x = live[i] && k < k_end ? src[i][k] : 0.0;
      v.y = live[i] && k + 1 < k_end ? src[i][k + 1] : 0.0;
      *reinterpret_cast<double2*>(T + (D::DMA_PER_WAVE * wave + i) * 128 + 2 * lane) = v;
    }
    if (u_wave) {
#pragma unroll
      for (int j = 0; j < D::UDMA; ++j)
        if (64 * j + lane < C::KT / 2) {
          const int64_t k = k0 + 2 * (64 * j + lane);
          double2 v;
          v.x = k < k_end ? ug[k] : 0.0;
          v.y = k + 1 < k_end ? ug[k + 1] : 0.0;
          *reinterpret_cast<double2*>(ud + 128 * j + 2 * lane) = v;
        }
    }
  };

  // Y u: chunk c of rows tid / CH + (THREADS / CH) i
  const int c = tid % C::CH;
  int rho[C::NCH];
#pragma unroll
  for (int i = 0; i < C::NCH; ++i) rho[i] = tid / C::CH + (C::THREADS / C::CH) * i;
  double yu[C::NCH];
#pragma unroll
  for (int i = 0; i < C::NCH; ++i) yu[i] = 0.0;

  d4 acc[C::NACC];
#pragma unroll
  for (int a = 0; a < C::NACC; ++a) acc[a] = d4{0.0, 0.0, 0.0, 0.0};

  auto step = [&](int t, const double* tile, double* next) {
    if (t + 1 < ntiles) issue(t + 1, next);
    mma_dispatch_dma<NB>(bw, tile, lane, kg, acc);
    if (want_u) {
      const double2 ub = *reinterpret_cast<const double2*>(tile + C::SBP * C::KT + 2 * c);
#pragma unroll
      for (int i = 0; i < C::NCH; ++i) {
        const int r = rho[i];
        const double2 v =
            *reinterpret_cast<const double2*>(tile + r * C::KT + 2 * (c ^ (r & 15)));
        yu[i] = fma(v.x, ub.x, yu[i]);
        yu[i] = fma(v.y, ub.y, yu[i]);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);   // tile t + 1 is in LDS
    __syncthreads();
  };
  issue(0, t0);
  __builtin_amdgcn_s_waitcnt(0);   // the LDS-DMA writes count on the vector memory counter
  __syncthreads();
  for (int t = 0; t < ntiles; t += 2) {
    step(t, t0, t1);
    if (t + 1 < ntiles) step(t + 1, t1, t0);
  }

  // Sum the k-groups (waves with the same blocks) through LDS, in group order,
  // HA of a wave's blocks at a time.
  if constexpr (C::KG > 1) {
#pragma unroll
    for (int a0 = 0; a0 < C::NACC; a0 += D::HA) {
      auto at = [&](int g, int a) {
        return t0 + (((g - 1) * C::BW + bw) * D::HA + (a - a0)) * 256 + lane;
      };
      if (kg > 0) {
#pragma unroll
        for (int a = a0; a < std::min(a0 + D::HA, C::NACC); ++a)
#pragma unroll
          for (int i = 0; i < 4; ++i) at(kg, a)[64 * i] = acc[a][i];
      }
      __syncthreads();
      if (kg == 0) {
        for (int g = 1; g < C::KG; ++g) {
#pragma unroll
          for (int a = a0; a < std::min(a0 + D::HA, C::NACC); ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[a][i] += at(g, a)[64 * i];
        }
      }
      if (a0 + D::HA < C::NACC) __syncthreads();
    }
  }
  if (kg == 0) {
#pragma unroll
    for (int a = 0; a < C::NACC; ++a) {
      gptr<double> dst = glb(part) + acc_block<NB>(bw, a) * 256 + lane;
#pragma unroll
      for (int i = 0; i < 4; ++i) put<AGENT>(dst + 64 * i, acc[a][i]);
    }
  }
  if (want_u) {
    __syncthreads();   // LDS is reused for the row sums of Y u
#pragma unroll
    for (int i = 0; i < C::NCH; ++i) t0[rho[i] * C::CH + c] = yu[i];
    __syncthreads();
    if (tid < C::SBP) {
      double sum = 0.0;
      for (int q = 0; q < C::CH; ++q) sum += t0[tid * C::CH + q];
      put<AGENT>(glb(part) + C::NBLK * 256 + tid, sum);
    }
  }
}

// ---------------------------------------------------------------------------
// NB = 10, 12, 14, 16 (129 to 256 rows): the matrix cores bound it.  The lower 16x16
// blocks are dealt to the eight waves in row-major runs of equal length, and a wave
// runs through its blocks column by column, so that it holds few rows of fragments at
// a time.  Tiles are 16 columns, three in LDS: one is computed, the next is in, the
// one after is on its way.  Rows are unpadded 128-byte slots whose eight 16-byte
// chunks are XOR-swizzled, chunk c of row r at c ^ ((r >> 1) & 7), so the sixteen rows
// of a fragment read fall in distinct banks.
//
// The order of a tile is fixed by hand (sched_barrier): before each block the fragments
// kTriLead ahead are read, at the end of a tile from the next one, so that the matrix
// cores start on it straight after the barrier.  256 x 2^18 (17.2 GFLOP): 317 us as two
// buffers whose reads the compiler let wait for the DMA into the other one, 296 with
// that wait gone, 291 with the third buffer and the fixed order (250 us more for each
// 2^18 columns more, the rest is writing 71 MB of partial sums at the end); 150 x 100003
// as sixteen block rows 125 us, as ten 55.
constexpr int kTriMin = 9;       // block rows from which on these kernels run
constexpr int kTriLead = 4;
constexpr int tri_rows(int nb) { return nb < kTriMin ? nb : (nb + 1) / 2 * 2; }

// A wave's blocks (block row r, block column c, index q in the partial) in the order
// they are computed, the block rows in the order their fragments are first used, how
// many of them block i needs, and the block rows whose Y u is this wave's (its diagonal
// blocks').
struct WaveBlocks {
  int n = 0, nf = 0, nd = 0;
  int r[17] = {}, c[17] = {}, q[17] = {}, need[17] = {};
  int fr[24] = {}, diag[16] = {};
  bool have[24] = {};
  constexpr void add(int row, int col, int k) {
    if (!have[row]) {
      have[row] = true;
      fr[nf++] = row;
    }
    if (!have[col]) {
      have[col] = true;
      fr[nf++] = col;
    }
    r[n] = row;
    c[n] = col;
    q[n] = k;
    need[n] = nf;
    ++n;
    if (row == col) diag[nd++] = row;
  }
};

// Block rows NR whose rows a tile holds, and blocks NBLK of the shape's partial.
template <int NROWS, int NBLOCKS>
struct SlabShape {
  static constexpr int NR = NROWS, NBLK = NBLOCKS, SBP = 16 * NR, KT = 16, CH = KT / 2;
  static constexpr int PP = KT / 8;                  // 128-bit fragment reads per tile
  static constexpr int THREADS = 512;
  static constexpr int TILE = SBP * KT + KT;         // doubles per buffer: rows, then u
  static constexpr int DMA = SBP * CH / 64;          // instructions of 64 chunks a tile
};

// The lower triangle of NB block rows, rows base + r; wave W takes an eighth of the
// row-major order.
template <int NB>
struct Tri : SlabShape<NB, NB * (NB + 1) / 2> {
  static __device__ __forceinline__ int row(int base, int r) { return base + r; }
  template <int W>
  static constexpr WaveBlocks blocks() {
    WaveBlocks b{};
    const int n = NB * (NB + 1) / 2, q0 = W * n / 8, q1 = (W + 1) * n / 8;
    for (int col = 0; col < NB; ++col)
      for (int row = col; row < NB; ++row) {
        const int k = blk_index(row, col);
        if (k >= q0 && k < q1) b.add(row, col, k);
      }
    return b;
  }
};

// R block rows (rows base + r) against the first sixteen: block (i, j) at i * 16 + j; a
// wave takes two block rows of R and 4 R / 4 block columns.
template <int R>
struct Rect : SlabShape<16 + R, 16 * R> {
  static __device__ __forceinline__ int row(int base, int r) {
    return r < 256 ? r : base + (r - 256);
  }
  template <int W>
  static constexpr WaveBlocks blocks() {
    WaveBlocks b{};
    const int i0 = 2 * (W % (R / 2)), j0 = R * (W / (R / 2));
    for (int j = j0; j < j0 + R; ++j)
      for (int i = i0; i < i0 + 2; ++i) b.add(16 + i, j, i * 16 + j);
    return b;
  }
};

// The three tile buffers (a shape's TILE doubles each).  In the one-problem kernels
// each is a __shared__ array of its own and the tile loop is unrolled over the three,
// which is what tells the compiler that a read of one need not wait for the DMA into
// another.
struct TriLds {
  double *t0, *t1, *t2;
};

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <class C, int W, bool AGENT>
__device__ __forceinline__ void tri_slab(const double* __restrict__ A, int64_t ld,
                                         int64_t k_begin, int64_t k_end, const int32_t* idx,
                                         int m, int base, const double* __restrict__ u,
                                         double* __restrict__ part, const TriLds L) {
  typedef __attribute__((address_space(3))) void* lds_vptr;
  typedef __attribute__((address_space(1))) const void* glb_vptr;
  constexpr WaveBlocks T = C::template blocks<W>();
  constexpr int LEAD = T.nf < kTriLead ? T.nf : kTriLead;
  constexpr int ND = (C::DMA - W + 7) / 8;   // this wave's DMA instructions: W + 8 i
  const int lane = threadIdx.x & 63;
  // The ragged tile of a slab that ends inside one comes first, by ordinary loads.
  const int nfull = (int)((k_end - k_begin) / C::KT);
  const bool ragged = k_begin + (int64_t)nfull * C::KT < k_end;
  const int ntiles = nfull + (ragged ? 1 : 0);

  // DMA instruction i of a wave fills slots (W + 8 i) * 64 + lane: row slot / 8,
  // position slot % 8; rows past m: any valid row
  auto slot_row = [&](int i) { return 8 * (W + 8 * i) + (lane >> 3); };
  auto chunk_of = [&](int r) { return (lane & 7) ^ ((r >> 1) & 7); };
  const gptr<const double> Ag = glb(A);
  const bool want_u = u != nullptr;
  const gptr<const double> ug = glb(u);
  gptr<const double> src[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int r = slot_row(i), p = C::row(base, r);
    src[i] = Ag + (int64_t)idx[p < m ? p : 0] * ld + k_begin + 2 * chunk_of(r);
  }
  // full tile f (columns k_begin + 16 f ..)
  auto issue = [&](int f, double* B) {
#pragma unroll
    for (int i = 0; i < ND; ++i)
      __builtin_amdgcn_global_load_lds((glb_vptr)(src[i] + (int64_t)f * C::KT),
                                       (lds_vptr)(B + (W + 8 * i) * 128), 16, 0, 0);
    if (W == 7 && want_u && lane < C::CH)   // the tile's u after the rows
      __builtin_amdgcn_global_load_lds((glb_vptr)(ug + k_begin + (int64_t)f * C::KT + 2 * lane),
                                       (lds_vptr)(B + C::SBP * C::KT), 16, 0, 0);
  };
  const int shift = ragged ? 1 : 0;   // tile t is full tile t - shift
  if (ragged) {
    const int64_t k0 = k_begin + (int64_t)nfull * C::KT;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int64_t off = (int64_t)nfull * C::KT, k = k0 + 2 * chunk_of(slot_row(i));
      double2 v;
      v.x = k < k_end ? src[i][off] : 0.0;
      v.y = k + 1 < k_end ? src[i][off + 1] : 0.0;
      *reinterpret_cast<double2*>(L.t0 + (W + 8 * i) * 128 + 2 * lane) = v;
    }
    if (W == 7 && lane < C::KT)
      L.t0[C::SBP * C::KT + lane] = want_u && k0 + lane < k_end ? ug[k0 + lane] : 0.0;
  } else {
    issue(0, L.t0);
  }
  if (ntiles > 1) issue(1 - shift, L.t1);

  // fragment offsets of the two k-pairs: row lane % 16 of a block row, chunk 4 pp +
  // lane / 16, swizzled
  const int g = lane >> 4, rl = lane & 15;
  int lane_off[C::PP];
#pragma unroll
  for (int pp = 0; pp < C::PP; ++pp)
    lane_off[pp] = rl * C::KT + 2 * ((4 * pp + g) ^ ((rl >> 1) & 7));
  auto frag = [&](const double* B, int pp, int r) {
    return *reinterpret_cast<const double2*>(B + lane_off[pp] + r * 16 * C::KT);
  };

  d4 acc[T.n];
#pragma unroll
  for (int a = 0; a < T.n; ++a) acc[a] = d4{0.0, 0.0, 0.0, 0.0};
  double yu[T.nd > 0 ? T.nd : 1];
#pragma unroll
  for (int a = 0; a < T.nd; ++a) yu[a] = 0.0;
  double2 pre[LEAD];   // the next tile's first fragments

  __builtin_amdgcn_s_waitcnt(0);   // the LDS-DMA writes count on the vector memory counter
  __syncthreads();
#pragma unroll
  for (int i = 0; i < LEAD; ++i) pre[i] = frag(L.t0, 0, T.fr[i]);

  // Tile t in cur, tile t + 1 in nxt, tile t + 2 on its way into far.
  auto step = [&](int t, const double* cur, const double* nxt, double* far) {
    double2 F[C::PP][C::NR];
    double2 ut[C::PP];
    static_for<0, LEAD>([&](auto i) { F[0][T.fr[i]] = pre[i]; });
    static_for<0, C::PP * T.n>([&](auto I) {
      constexpr int pp = I / T.n, i = I % T.n;
      // fragments read before this block: all that the one before it had asked for
      constexpr int last = I == 0 ? 0 : I - 1;
      constexpr int before =
          I == 0 ? LEAD : std::max(LEAD, last / T.n * T.nf + T.need[last % T.n] + LEAD);
      constexpr int after = std::max(before, pp * T.nf + T.need[i] + LEAD);
      static_for<before, after>([&](auto l) {
        constexpr int tile = l / (C::PP * T.nf), lp = l / T.nf % C::PP, f = l % T.nf;
        if constexpr (tile == 0)
          F[lp][T.fr[f]] = frag(cur, lp, T.fr[f]);
        else
          pre[f] = frag(nxt, 0, T.fr[f]);
      });
      if constexpr (T.nd > 0 && i == 0)   // u at the same two columns
        ut[pp] = *reinterpret_cast<const double2*>(cur + C::SBP * C::KT + 8 * pp + 2 * g);
      const double2 fr = F[pp][T.r[i]], fc = F[pp][T.c[i]];
      acc[i] = mfma(fr.x, fc.x, acc[i]);
      acc[i] = mfma(fr.y, fc.y, acc[i]);
      if constexpr (i == T.n - 1)
        static_for<0, T.nd>([&](auto d) {
          yu[d] = fma(F[pp][T.diag[d]].x, ut[pp].x, yu[d]);
          yu[d] = fma(F[pp][T.diag[d]].y, ut[pp].y, yu[d]);
        });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (I == 1) {
        if (t + 2 < ntiles) issue(t + 2 - shift, far);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __builtin_amdgcn_s_waitcnt(kWaitVm0);   // tile t + 2 is in LDS
    lds_barrier();
  };
  for (int t = 0; t < ntiles; t += 3) {
    step(t, L.t0, L.t1, L.t2);
    if (t + 1 < ntiles) step(t + 1, L.t1, L.t2, L.t0);
    if (t + 2 < ntiles) step(t + 2, L.t2, L.t0, L.t1);
  }

  gptr<double> pg = glb(part);
  static_for<0, T.n>([&](auto a) {
    gptr<double> dst = pg + T.q[a] * 256 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) put<AGENT>(dst + 64 * i, acc[a][i]);
  });
  if (want_u) {   // Y u of the wave's diagonal rows: sum the four lane groups
    static_for<0, T.nd>([&](auto d) {
      double v = yu[d];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (lane < 16) put<AGENT>(pg + C::NBLK * 256 + 16 * T.diag[d] + lane, v);
    });
  }
}

// The slab of a shape (Tri: arguments and partial layout as gram_slab_dma; Rect: without
// Y u): rows idx[C::row(base, .)], the m-th on replaced by the first.
template <class C, bool AGENT = false>
__device__ __forceinline__ void gram_slab_tri(const double* __restrict__ A, int64_t ld,
                                              int64_t k_begin, int64_t k_end, const int32_t* idx,
                                              int m, int base, const double* __restrict__ u,
                                              double* __restrict__ part, const TriLds L) {
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: tri_slab<C, 0, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 1: tri_slab<C, 1, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 2: tri_slab<C, 2, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 3: tri_slab<C, 3, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 4: tri_slab<C, 4, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 5: tri_slab<C, 5, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    case 6: tri_slab<C, 6, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
    default: tri_slab<C, 7, AGENT>(A, ld, k_begin, k_end, idx, m, base, u, part, L); break;
  }
}

// ---------------------------------------------------------------------------
// The 256-row Gram with the previous step's companion update folded in
// (CABCD_FLAG_FOLD_UPDATE), and that update alone.  Two tiles in LDS, rows as in Tri;
// wave W owns block rows W and 15 - W.  Y u is accumulated from the waves' own-row
// fragments and summed over the four lane groups at the end.
struct D16 {
  static constexpr int NB = 16, SBP = 256, NBLK = 136, KT = 16, CH = KT / 2;
  static constexpr int PP = KT / 8;                  // 128-bit fragment reads per tile
  static constexpr int THREADS = 512;
  static constexpr int TILE = SBP * KT + KT;         // doubles per buffer: rows, then u
  static constexpr int DMA_PER_WAVE = SBP * CH / THREADS;   // 4 instructions
  // two more buffers for the previous step's rows (and the tile's old companion
  // entries), then gamma * delta of the previous step; one array (as arrays of their
  // own with the tile loop unrolled over them a step took 0.388 ms, not 0.371)
  static constexpr int YT = SBP * KT + KT;           // doubles per update buffer
  static constexpr int YOFF = 2 * TILE;
  static constexpr int DOFF = 2 * TILE + 2 * YT;
  static constexpr int LDS_UPD = DOFF + SBP;
};

// x of the lane N places along in the lane's row of sixteen (DPP row_ror),
// as two 32-bit moves
template <int N>
__device__ __forceinline__ double d16_ror(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + N, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + N, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// The sum over a row of sixteen lanes, in every lane of the row.
__device__ __forceinline__ double d16_row_sum(double x) {
  x += d16_ror<8>(x);
  x += d16_ror<4>(x);
  x += d16_ror<2>(x);
  x += d16_ror<1>(x);
  return x;
}
// x of lane l (the same l in every lane) in every lane.
__device__ __forceinline__ double d16_read_lane(double x, int l) {
  const long long b = __double_as_longlong(x);
  return __hiloint2double(__builtin_amdgcn_readlane((int)(b >> 32), l),
                          __builtin_amdgcn_readlane((int)b, l));
}

// Chunk swizzle of row r: the sixteen rows of a fragment read land on
// distinct banks (8 chunks a row: (r >> 1) & 7; 16 chunks a row: r & 15).
__device__ __forceinline__ int d16_swz(int r) { return D16::CH == 8 ? (r >> 1) & 7 : r & 15; }

// The whole slab for wave W (block rows W and 15 - W); gram_slab_dma16 picks
// the instantiation once, so each wave's tile loop is one straight-line path
// for the register allocator.
// MODE 1: the Gram slab with the previous step's companion update applied to the
// slab's columns first; Y u uses the updated companion.  MODE 2: the update alone
// (the last step of a call, or one followed by a check), by the same code, so
// a column's update has the same rounding whichever way it runs.
//
// The update of tile t's 16 columns: wave W sums column pair W over the 256
// rows (lane l: rows l + 64 j, then a butterfly over the wave, lane 0's total
// kept), adds the old entries, writes the companion and, in MODE 1, the
// tile's u slot.  In MODE 1 it runs one tile ahead of the Gram (tile t + 1
// during tile t), so the end-of-tile barrier publishes the u slot; the
// previous step's rows are DMA'd two tiles ahead, their chunks swizzled as
// the Gram's tiles are ((r >> 1) & 7), so the column-pair reads of sixteen
// consecutive rows fall in distinct banks.
template <int W, int MODE>
__device__ __forceinline__ void d16_slab(const double* __restrict__ A, int64_t ld,
                                         int64_t k_begin, int64_t k_end, const int32_t* idx,
                                         int m, double* __restrict__ part, double* lds,
                                         const D16Upd up) {
  using C = D16;
  typedef __attribute__((address_space(3))) void* lds_vptr;
  typedef __attribute__((address_space(1))) const void* glb_vptr;
  constexpr int R0 = W, R1 = 15 - W;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int ntiles = (int)((k_end - k_begin + C::KT - 1) / C::KT);

  // DMA instruction i of this wave fills slots (4 W + i) * 64 + lane.
  gptr<const double> src[C::DMA_PER_WAVE];
  int cofs[C::DMA_PER_WAVE];
  const gptr<const double> Ag = glb(A);
#pragma unroll
  for (int i = 0; i < C::DMA_PER_WAVE; ++i) {
    const int q = (C::DMA_PER_WAVE * W + i) * 64 + lane;
    const int r = q / C::CH;
    cofs[i] = 2 * ((q % C::CH) ^ d16_swz(r));
    // rows past m: any valid row (MODE 2 reads no Gram rows)
    src[i] = MODE == 2 ? Ag : Ag + (int64_t)idx[r < m ? r : 0] * ld;
  }

  // The previous step's rows: DMA instruction i of this wave
  // fills slots q = (4 W + i) * 64 + lane of an update buffer: row q / 8 =
  // 8 (4 W + i) + lane / 8, chunk (q % 8) ^ ((row >> 1) & 7), the swizzle
  // being (4 i + lane / 16) & 7.  The rows are kept as indices and the
  // addresses formed at each issue, to spare registers.
  int yrow[C::DMA_PER_WAVE];
  const gptr<double> rg = glb(up.r);
#pragma unroll
  for (int i = 0; i < C::DMA_PER_WAVE; ++i)
    yrow[i] = up.idx[8 * (C::DMA_PER_WAVE * W + i) + (lane >> 3)];
  if (tid < C::SBP) lds[C::DOFF + tid] = up.gamma * up.delta[tid];
  auto issue_y = [&](int t, int slot) {
    const int64_t k0 = k_begin + (int64_t)t * C::KT;
    double* Y = lds + C::YOFF + slot * C::YT;
#pragma unroll
    for (int i = 0; i < C::DMA_PER_WAVE; ++i) {
      double* dst = Y + (C::DMA_PER_WAVE * W + i) * 128;
      const int64_t k = k0 + 2 * ((lane & 7) ^ ((4 * i + (lane >> 4)) & 7));
      const gptr<const double> row = Ag + (int64_t)yrow[i] * ld;
      if (k + 1 < k_end) {
        __builtin_amdgcn_global_load_lds((glb_vptr)(row + k), (lds_vptr)dst, 16, 0, 0);
      } else {
        double2 v;
        v.x = k < k_end ? row[k] : 0.0;
        v.y = 0.0;
        *reinterpret_cast<double2*>(dst + 2 * lane) = v;
      }
    }
    // the old companion entries of the tile's columns: lanes 0..CH-1 of wave 7
    if (W == 7 && lane < C::CH) {
      double* dst = Y + C::SBP * C::KT;
      const int64_t k = k0 + 2 * lane;
      if (k + 1 < k_end) {
        __builtin_amdgcn_global_load_lds((glb_vptr)(rg + k), (lds_vptr)dst, 16, 0, 0);
      } else {
        double2 v;
        v.x = k < k_end ? rg[k] : 0.0;
        v.y = k + 1 < k_end ? rg[k + 1] : 0.0;
        *reinterpret_cast<double2*>(dst + 2 * lane) = v;
      }
    }
  };
  // tile t's update from update buffer yslot; MODE 1 also fills the u slot
  // of Gram buffer uslot
  auto update = [&](int t, int yslot, int uslot) {
    const double* Y = lds + C::YOFF + yslot * C::YT;
    const double* dl = lds + C::DOFF;
    double p0 = 0.0, p1 = 0.0;
#pragma unroll 2
    for (int j = 0; j < C::SBP / 64; ++j) {
      const int r = lane + 64 * j;
      const double2 y = *reinterpret_cast<const double2*>(Y + r * C::KT + 2 * (W ^ d16_swz(r)));
      const double dj = dl[r];
      p0 = fma(y.x, dj, p0);
      p1 = fma(y.y, dj, p1);
    }
    // the wave's total: each row of 16 lanes by DPP rotations, then the four
    // row sums (lanes 0, 16, 32, 48) in a fixed order
    p0 = d16_row_sum(p0);
    p1 = d16_row_sum(p1);
    p0 = (d16_read_lane(p0, 0) + d16_read_lane(p0, 16)) +
         (d16_read_lane(p0, 32) + d16_read_lane(p0, 48));
    p1 = (d16_read_lane(p1, 0) + d16_read_lane(p1, 16)) +
         (d16_read_lane(p1, 32) + d16_read_lane(p1, 48));
    if (lane == 0) {
      const int64_t k = k_begin + (int64_t)t * C::KT + 2 * W;
      const double* ro = Y + C::SBP * C::KT;
      const double n0 = ro[2 * W] + p0, n1 = ro[2 * W + 1] + p1;
      if (k < k_end) rg[k] = n0;
      if (k + 1 < k_end) rg[k + 1] = n1;
      if constexpr (MODE == 1) {
        double* us = lds + uslot * C::TILE + C::SBP * C::KT;
        us[2 * W] = k < k_end ? n0 : 0.0;
        us[2 * W + 1] = k + 1 < k_end ? n1 : 0.0;
      }
    }
  };
  if constexpr (MODE == 2) {
    issue_y(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int t = 0; t < ntiles; ++t) {
      if (t + 1 < ntiles) issue_y(t + 1, (t + 1) & 1);
      update(t, t & 1, -1);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
    return;
  }

  auto issue = [&](int t, int slot) {
    const int64_t k0 = k_begin + (int64_t)t * C::KT;
    double* T = lds + slot * C::TILE;
#pragma unroll
    for (int i = 0; i < C::DMA_PER_WAVE; ++i) {
      double* dst = T + (C::DMA_PER_WAVE * W + i) * 128;   // 64 slots of 2 doubles
      const int64_t k = k0 + cofs[i];
      if (k + 1 < k_end) {
        __builtin_amdgcn_global_load_lds((glb_vptr)(src[i] + k), (lds_vptr)dst, 16, 0, 0);
      } else {
        double2 v;
        v.x = k < k_end ? src[i][k] : 0.0;
        v.y = 0.0;
        *reinterpret_cast<double2*>(dst + 2 * lane) = v;
      }
    }
  };

  // This lane's fragment offsets (doubles) for the two k-pairs of a tile: row
  // lane & 15 of every block row, chunk 4 pp + lane / 16, swizzled.
  const int g = lane >> 4;
  const int rl = lane & 15;
  int lane_off[C::PP];
#pragma unroll
  for (int pp = 0; pp < C::PP; ++pp) lane_off[pp] = rl * C::KT + 2 * ((4 * pp + g) ^ d16_swz(rl));

  d4 acc[17];
#pragma unroll
  for (int a = 0; a < 17; ++a) acc[a] = d4{0.0, 0.0, 0.0, 0.0};
  double yua[2] = {0.0, 0.0};

  issue(0, 0);
  issue_y(0, 0);
  if (ntiles > 1) issue_y(1, 1);
  __builtin_amdgcn_s_waitcnt(0);   // the LDS-DMA writes count on the vector memory counter
  __syncthreads();
  update(0, 0, 0);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    if (t + 1 < ntiles) issue(t + 1, (t + 1) & 1);
    // update buffer t & 1 held tile t (updated during tile t - 1); tile t + 1
    // arrived during tile t - 1.  Waves 0-3 update before their matrix
    // instructions, waves 4-7 (the other wave of each SIMD) after them, so
    // the update's latency runs beside the other wave's MFMA chain.
    if (t + 2 < ntiles) issue_y(t + 2, t & 1);
    if (W < 4 && t + 1 < ntiles) update(t + 1, (t + 1) & 1, (t + 1) & 1);
    const double* tile = lds + (t & 1) * C::TILE;
#pragma unroll
    for (int pp = 0; pp < C::PP; ++pp) {
      const double* base = tile + lane_off[pp];
      auto frag = [&](int r) {   // rows 16 r .. 16 r + 15, this lane's chunk of pair pp
        return *reinterpret_cast<const double2*>(base + r * 16 * C::KT);
      };
      const double2 f0 = frag(R0);
      const double2 f1 = frag(R1);
      const double2 ut =   // u at the same two columns (unswizzled, after the rows)
          *reinterpret_cast<const double2*>(tile + C::SBP * C::KT + 8 * pp + 2 * g);
      yua[0] = fma(f0.x, ut.x, yua[0]);
      yua[0] = fma(f0.y, ut.y, yua[0]);
      yua[1] = fma(f1.x, ut.x, yua[1]);
      yua[1] = fma(f1.y, ut.y, yua[1]);
#pragma unroll
      for (int c = 0; c <= R1; ++c) {
        const double2 fc = c == R0 ? f0 : (c == R1 ? f1 : frag(c));
        if (c <= R0) {
          acc[c] = mfma(f0.x, fc.x, acc[c]);
          acc[c] = mfma(f0.y, fc.y, acc[c]);
        }
        acc[R0 + 1 + c] = mfma(f1.x, fc.x, acc[R0 + 1 + c]);
        acc[R0 + 1 + c] = mfma(f1.y, fc.y, acc[R0 + 1 + c]);
      }
    }
    if (W >= 4 && t + 1 < ntiles) update(t + 1, (t + 1) & 1, (t + 1) & 1);
    __builtin_amdgcn_s_waitcnt(0);   // tile t + 1 is in LDS
    __syncthreads();
  }

  gptr<double> pg = glb(part);
#pragma unroll
  for (int a = 0; a < 17; ++a) {
    const int blk = a <= R0 ? blk_index(R0, a) : blk_index(R1, a - R0 - 1);
    gptr<double> dst = pg + blk * 256 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[64 * i] = acc[a][i];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {   // Y u of the two owned block rows: sum the four lane groups
    double v = yua[i];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < 16) pg[C::NBLK * 256 + 16 * (i == 0 ? R0 : R1) + lane] = v;
  }
}

// The folded slab (MODE 1) or its update alone (MODE 2); partial layout as gram_slab_dma.
template <int MODE>
__device__ __forceinline__ void gram_slab_dma16(const double* __restrict__ A, int64_t ld,
                                                int64_t k_begin, int64_t k_end,
                                                const int32_t* idx, int m,
                                                double* __restrict__ part, double* lds,
                                                const D16Upd up) {
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: d16_slab<0, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 1: d16_slab<1, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 2: d16_slab<2, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 3: d16_slab<3, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 4: d16_slab<4, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 5: d16_slab<5, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    case 6: d16_slab<6, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
    default: d16_slab<7, MODE>(A, ld, k_begin, k_end, idx, m, part, lds, up); break;
  }
}

// Element e of a partial block (lane-major: e = item*64 + lane) sits at
// column lane%16 of its 16x16 block and row 4*item + lane/16 (layout 0: the
// output order of v_mfma_f64_16x16x4_f64 on gfx950) or 4*(lane/16) + item
// (layout 1: the FP32-output MFMAs).  Both were checked on the hardware with
// probes of known integer matrices.
__device__ __forceinline__ void entry_rc(int64_t e, int layout, int& row, int& col, bool& lower) {
  const int q = (int)(e >> 8);
  int r = 0;
  while (blk_index(r + 1, 0) <= q) ++r;
  const int cb = q - blk_index(r, 0);
  const int item = (int)(e >> 6) & 3;
  const int lane = (int)e & 63;
  row = 16 * r + (layout == 0 ? 4 * item + (lane >> 4) : 4 * (lane >> 4) + item);
  col = 16 * cb + (lane & 15);
  lower = r != cb || row >= col;
}

// Writes the reduced entry e (sum t of its partials) to Gov / Yu.  add (may be
// NULL): an m x m row-major term added to the sum before scaling, read at
// (row, col) with row >= col (the light-column part of a split sparse Gram).
__device__ __forceinline__ void store_entry(int64_t e, double t, int nblk, const int32_t* idx,
                                            int m, double scale, double shift, int overlap,
                                            double* __restrict__ G, double* __restrict__ Yu,
                                            int layout, const float* __restrict__ rs,
                                            const double* __restrict__ add = nullptr) {
  if (e >= (int64_t)nblk * 256) {          // the Y u entries follow the blocks
    const int p = (int)(e - (int64_t)nblk * 256);
    if (Yu != nullptr && p < m) glb(Yu)[p] = rs ? (double)glb(rs)[idx[p]] * t : t;
    return;
  }
  int row, col;
  bool lower;
  entry_rc(e, layout, row, col, lower);
  if (row < m && col < m && lower) {
    const bool on = overlap ? (idx[row] == idx[col]) : (row == col);
    const double sc =
        rs ? scale * (double)glb(rs)[idx[row]] * (double)glb(rs)[idx[col]] : scale;
    if (add != nullptr) t += glb(add)[(int64_t)row * m + col];
    const double v = sc * t + (on ? shift : 0.0);
    glb(G)[(int64_t)row * m + col] = v;
    glb(G)[(int64_t)col * m + row] = v;
  }
}

// Index lists of a Gram of m in (256, 512] rows of codes or of a batched problem: ia = the m indices padded to
// 512 with idx[0] (two 256-row Grams: the diagonal blocks); ib[t] (t < nc,
// nc = 4 when m > 384, else 2) = idx[128 x .. 128 x + 128) followed by
// ia[256 + 128 y .. 256 + 128 y + 128), x = t % 2, y = t / 2, whose 256-row
// Gram holds the cross block of rows 256 + 128 y.. and columns 128 x.. .
// Padding rows are multiplied and never stored.  m may be below 256 (the ragged
// last step of a batched problem): every row past m is idx[0], also in the first
// half, whose entries past m are whatever the caller's list held before.  Thread
// t of nthreads.
__device__ __forceinline__ void big_lists(const int32_t* idx, int m, int32_t* ia, int32_t* ib,
                                          int t, int nthreads) {
  const int nc = m - 256 > 128 ? 4 : 2;
  for (int q = t; q < 512; q += nthreads) ia[q] = idx[q < m ? q : 0];
  for (int slot = t; slot < 256 * nc; slot += nthreads) {
    const int list = slot >> 8, pos = slot & 255;
    const int x = list & 1, y = list >> 1;
    const int r = pos < 128 ? 128 * x + pos : 256 + 128 * y + (pos - 128);
    ib[slot] = idx[r < m ? r : 0];
  }
}

// Where the reduced entry e of step `step` of a Gram of more than 256 rows
// goes (m in (256, 512], assembled from 256-row Grams; see
// launch_big_index): set 0 holds the two diagonal 256 x 256 blocks (step k:
// rows and columns 256 k + local) and Y u; set 1 holds the cross blocks, step
// t giving rows 256 + 128 (t / 2) + (local row - 128) and columns
// 128 (t % 2) + local column from the local block rows 8..15 x columns 0..7.
__device__ __forceinline__ void store_entry_big(int64_t e, double t, int set, int step,
                                                const int32_t* idx, int m, double scale,
                                                double shift, int overlap,
                                                double* __restrict__ G, double* __restrict__ Yu,
                                                int layout, const float* __restrict__ rs) {
  constexpr int kNblk = 136;
  if (e >= (int64_t)kNblk * 256) {          // the Y u entries follow the blocks
    const int p = 256 * step + (int)(e - (int64_t)kNblk * 256);
    if (set == 0 && Yu != nullptr && p < m) glb(Yu)[p] = rs ? (double)glb(rs)[idx[p]] * t : t;
    return;
  }
  int row, col;
  bool lower;
  entry_rc(e, layout, row, col, lower);
  if (!lower) return;
  int gr, gc;
  if (set == 0) {
    gr = 256 * step + row;
    gc = 256 * step + col;
  } else {
    if (row < 128 || col >= 128) return;
    gr = 256 + 128 * (step >> 1) + (row - 128);
    gc = 128 * (step & 1) + col;
  }
  if (gr >= m || gc >= m) return;
  const bool on = overlap ? (idx[gr] == idx[gc]) : (gr == gc);
  const double sc = rs ? scale * (double)glb(rs)[idx[gr]] * (double)glb(rs)[idx[gc]] : scale;
  const double v = sc * t + (on ? shift : 0.0);
  glb(G)[(int64_t)gr * m + gc] = v;
  glb(G)[(int64_t)gc * m + gr] = v;
}

// out[e] = the sum over q < n of in[e + q stride], in q order, by T threads;
// every value at agent scope (gdev::put<true>).
template <int T, class Out>
__device__ __forceinline__ void sum_sets(const double* __restrict__ in, int n, int64_t stride,
                                         int64_t count, Out out) {
  for (int64_t e = threadIdx.x; e < count; e += T) {
    const gptr<const double> p = glb(in) + e;
    double s = 0.0;
    for (int q = 0; q < n; q += 8) {
      double v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = get_agent(p + (int64_t)std::min(q + j, n - 1) * stride);
#pragma unroll
      for (int j = 0; j < 8; ++j) s += q + j < n ? v[j] : 0.0;
    }
    out(e, s);
  }
}

// The whole reduction by one workgroup of T threads: n partial sets (stride
// doubles apart) are added in set order for every entry.
template <int T>
__device__ __forceinline__ void reduce_wg(const double* __restrict__ partials, int n,
                                          int64_t stride, int nb, const int32_t* idx, int m,
                                          double scale, double shift, double* __restrict__ G,
                                          double* __restrict__ Yu, int layout,
                                          const float* __restrict__ rs) {
  const int nblk = nb * (nb + 1) / 2;
  sum_sets<T>(partials, n, stride, (int64_t)nblk * 256 + 16 * nb, [&](int64_t e, double s) {
    store_entry(e, s, nblk, idx, m, scale, shift, 1, G, Yu, layout, rs);
  });
}

// The reduction of a Gram of m <= 512 rows assembled from 256-row Grams, by
// one workgroup of T threads: set q's partial Gram g (g < 2: the diagonal
// blocks, then the cross blocks; nsets = 2 + big_cross_steps(m)) is at
// partials + q stride + g pstride16; every entry sums its sets in order and is
// stored once (store_entry_big).
template <int T>
__device__ __forceinline__ void reduce_wg_big(const double* __restrict__ partials, int n,
                                              int64_t stride, int nsets, const int32_t* idx,
                                              int m, double scale, double shift,
                                              double* __restrict__ G, double* __restrict__ Yu,
                                              int layout, const float* __restrict__ rs) {
  constexpr int64_t pstride = (int64_t)136 * 256 + 16 * 16;
  for (int g = 0; g < nsets; ++g)
    sum_sets<T>(partials + g * pstride, n, stride, pstride, [&](int64_t e, double s) {
      store_entry_big(e, s, g < 2 ? 0 : 1, g < 2 ? g : g - 2, idx, m, scale, shift, 1, G, Yu,
                      layout, rs);
    });
}

}  // namespace gdev
}  // namespace cabcd
