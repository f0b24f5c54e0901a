// Blocked SpMV core for gfx950 (paper §4.2: one index per dense block).
//
// A group of G lanes (G a power of two dividing the 64-lane wavefront) owns one
// block row.  Lane l takes blocks k0+l, k0+l+G, ... of the row: consecutive lanes
// read consecutive blocks, so a wave's value loads cover one contiguous stretch of
// the value array.  Each lane keeps one whole block in registers, gathers the
// BC*NRHS entries of x it multiplies, and accumulates BR*NRHS partial sums; the
// group then reduces them with cross-lane shuffles (no LDS, no atomics), so the
// result is deterministic.  The per-row epilogue is a template parameter, which
// lets the smoother, residual and CG kernels fuse their vector updates into the
// product instead of making extra passes over HBM.
#pragma once

#include <algorithm>

#include "internal.hpp"

namespace blk {

constexpr int kBlock = 256;

template <class T>
__device__ __forceinline__ T fmadd(T a, T b, T c) { return a * b + c; }

template <int N, class T>
__device__ __forceinline__ T pick(const T (&v)[N], int i) {
  T r = T(0);
#pragma unroll
  for (int t = 0; t < N; ++t)
    if (t == i) r = v[t];
  return r;
}

template <int BR, int BC, int NR, class TM, class TX, class TA>
__device__ __forceinline__ void block_fma(const TM* __restrict__ b, const TA (&xv)[BC * NR], TA (&acc)[BR * NR]) {
#pragma unroll
  for (int i = 0; i < BR; ++i) {
#pragma unroll
    for (int j = 0; j < BC; ++j) {
      const TA a = ld<TA>(b + i * BC + j);
#pragma unroll
      for (int q = 0; q < NR; ++q) acc[i * NR + q] = fmadd(a, xv[j * NR + q], acc[i * NR + q]);
    }
  }
}

// Lanes of a group stride over the blocks of the row; each lane takes U blocks per
// step and issues all their loads before the multiply-adds, so a wave keeps
// U * 64 blocks of loads in flight.
//
// SYM (square blocks, a structurally symmetric matrix): the strictly lower blocks
// of the row are not read from their own position but as the transpose of their
// mirror in the upper triangle, mir[k] = position of block (colidx[k], row).  Only
// the upper triangle and the diagonal are then streamed from HBM; each mirrored
// block was read by its own (earlier) row shortly before, so its second read is
// mostly served by the caches.  For a symmetric matrix the products are the same,
// in the same order within a lane.
template <int BR, int BC, int NR, int G, int U, class TM, class TX, class TA, bool SYM = false>
__device__ __forceinline__ void row_product(const int32_t* __restrict__ colidx,
                                            const TM* __restrict__ val, const TX* __restrict__ x,
                                            int k0, int k1, int lane, TA (&acc)[BR * NR], int row = 0,
                                            const int32_t* __restrict__ mir = nullptr) {
  static_assert(!SYM || BR == BC, "symmetric reads need square blocks");
#pragma unroll
  for (int t = 0; t < BR * NR; ++t) acc[t] = TA(0);
  for (int kb = k0 + lane; kb < k1; kb += G * U) {
    TM bv[U][BR * BC];
    TA xv[U][BC * NR];
    bool low[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = kb + u * G;
      low[u] = false;
      if (k < k1) {
        // with symmetric reads the block's source position comes from the mirror index
        // (k itself for the diagonal and upper blocks), loaded alongside the column
        // index, so the value load waits for one index load as in the full reads
        const int c = colidx[k];
        int src = k;
        if constexpr (SYM) src = mir[k];
        const TX* xc = x + static_cast<size_t>(c) * (BC * NR);
#pragma unroll
        for (int t = 0; t < BC * NR; ++t) xv[u][t] = ld<TA>(xc + t);
        if constexpr (SYM) low[u] = c < row;
        const TM* b = val + static_cast<size_t>(src) * (BR * BC);
#pragma unroll
        for (int t = 0; t < BR * BC; ++t) bv[u][t] = b[t];
      } else {
#pragma unroll
        for (int t = 0; t < BC * NR; ++t) xv[u][t] = TA(0);
#pragma unroll
        for (int t = 0; t < BR * BC; ++t) bv[u][t] = TM{};
      }
    }
    if constexpr (SYM) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < BR; ++i) {
#pragma unroll
          for (int j = i + 1; j < BC; ++j) {
            const TM a = bv[u][i * BC + j], b = bv[u][j * BC + i];
            bv[u][i * BC + j] = low[u] ? b : a;
            bv[u][j * BC + i] = low[u] ? a : b;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) block_fma<BR, BC, NR, TM, TX, TA>(bv[u], xv[u], acc);
  }
#pragma unroll
  for (int t = 0; t < BR * NR; ++t) acc[t] = group_sum<G>(acc[t]);
}

// Generic kernel: one tile of kBlock / G block rows per workgroup; logical
// workgroups are XCD-contiguous (the hardware hands workgroup b to XCD b mod 8 and
// each XCD has its own L2), so neighbouring rows, which gather the same x entries,
// run on the same XCD at the same time.  A reducing epilogue (dot products) leaves
// one partial sum per workgroup; every thread reaches that block reduction.
template <int BR, int BC, int NR, int G, int U, class TM, class TX, class TA, class Epi, bool SYM = false>
__global__ __launch_bounds__(kBlock) void spmv_kernel(int nbr, const int32_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colidx,
                                                      const TM* __restrict__ val,
                                                      const TX* __restrict__ x, Epi epi,
                                                      const int32_t* __restrict__ mir = nullptr,
                                                      int chunk = kSpmvChunk) {
  constexpr int kRows = kBlock / G;
  const int lb = xcd_chunked_block(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), chunk);
  const int row = lb * kRows + static_cast<int>(threadIdx.x) / G;
  const int lane = static_cast<int>(threadIdx.x) % G;
  TA acc[BR * NR];
  const bool active = row < nbr;
  // the row's extent is loaded first and the epilogue's own-row operands right after
  // it, before the product: loads complete in issue order, so waiting for the extent
  // does not wait for the operands, whose latency then overlaps the block loads
  int k0 = 0, k1 = 0;
  if (active) {
    k0 = rowptr[row];
    k1 = rowptr[row + 1];
  }
  const auto pre = epi.template prefetch<BR, NR, G>(active, row);
  if (active) {
    row_product<BR, BC, NR, G, U, TM, TX, TA, SYM>(colidx, val, x, k0, k1, lane, acc, row, mir);
  } else {
#pragma unroll
    for (int z = 0; z < BR * NR; ++z) acc[z] = TA(0);
  }
  const double part = epi.template apply<BR, NR, G>(active, row, lane, acc, pre);
  if constexpr (Epi::kReduce) {
    __shared__ double lds[4];
    const double sum = block_sum_256(part, lds);
    if (threadIdx.x == 0) epi.partial[lb] = sum;
  }
}


// Eight right-hand sides: kColLanes lanes share a block, each with 16 bytes of every
// gathered panel row (two FP64 or four FP32 columns).
template <class TX>
constexpr int kColLanes = 8 * static_cast<int>(sizeof(TX)) / 16;

// 16 bytes of a panel row; element alignment only, as the caller's vectors have
template <class TX>
struct alignas(sizeof(TX)) PanelCols {
  static constexpr int N = 8 / kColLanes<TX>;
  TX v[N];
};
template <class TA, class TX>
__device__ __forceinline__ void ld_cols(const TX* p, TA (&v)[PanelCols<TX>::N]) {
  PanelCols<TX> c;
  __builtin_memcpy(&c, p, sizeof(c));
#pragma unroll
  for (int q = 0; q < PanelCols<TX>::N; ++q) v[q] = static_cast<TA>(c.v[q]);
}
template <class TA, class TX>
__device__ __forceinline__ void st_cols(TX* p, const TA (&v)[PanelCols<TX>::N]) {
  PanelCols<TX> c;
#pragma unroll
  for (int q = 0; q < PanelCols<TX>::N; ++q) c.v[q] = static_cast<TX>(v[q]);
  __builtin_memcpy(p, &c, sizeof(c));
}

// v of lane SRC of every group of CL (2 or 4) lanes, by quad permutation
template <int CL, int SRC>
__device__ __forceinline__ int col_bcast(int v) {
  constexpr int perm = CL == 4 ? SRC * 0x55 : (SRC == 0 ? 0xA0 : 0xF5);
  return __builtin_amdgcn_mov_dpp(v, perm, 0xf, 0xf, true);
}
template <int CL, int SRC, class TA>
__device__ __forceinline__ TA col_bcast_t(TA v) {
  int w[sizeof(TA) / 4];
  __builtin_memcpy(w, &v, sizeof(TA));
#pragma unroll
  for (int t = 0; t < static_cast<int>(sizeof(TA) / 4); ++t) w[t] = col_bcast<CL, SRC>(w[t]);
  __builtin_memcpy(&v, w, sizeof(TA));
  return v;
}

// acc += block * panel: the block's value e (row e / BC, column e % BC) comes from the lane
// of the group that loaded it
template <int E, int BE, int BC, int CL, int PER, int CPL, int BR, class TA>
__device__ __forceinline__ void panel_fma(const TA (&raw)[PER], const TA (&xv)[BC][CPL], TA (&acc)[BR][CPL]) {
  if constexpr (E < BE) {
    constexpr int src = E / PER < CL - 1 ? E / PER : CL - 1;
    constexpr int base = src * PER < BE - PER ? src * PER : BE - PER;
    const TA a = col_bcast_t<CL, src>(raw[E - base]);
#pragma unroll
    for (int q = 0; q < CPL; ++q) acc[E / BC][q] = fmadd(a, xv[E % BC][q], acc[E / BC][q]);
    panel_fma<E + 1, BE, BC, CL, PER, CPL, BR, TA>(raw, xv, acc);
  }
}

// The partial sums of a lane: its columns of the row's BR entries.
template <int BR, int CPL, class TA>
struct ColSums {
  TA v[BR][CPL];
  __device__ __forceinline__ void add(const ColSums& o) {
#pragma unroll
    for (int i = 0; i < BR; ++i)
#pragma unroll
      for (int q = 0; q < CPL; ++q) v[i][q] += o.v[i][q];
  }
};

// A row's blocks are added as V lanes with one chain of blocks each would (block k on chain
// k % V), in xor-tree order: whatever G is, FP32 and FP64 take as many roundings as with one
// lane per block.  Adding a slot's blocks one after the other instead was 10 % (FP64, 27 3x3
// blocks: 162 us) and 5 % (FP32, 84 us) faster, and 1.5 and 5 % further from the exact product.
template <class TX, int G, int U>
constexpr int kChains = U == 1 && sizeof(TX) == 4 ? 2 * G : G;

// G lanes per block row: G / CL block slots of CL lanes.  The V chains of a row are dealt to
// the S slots, T = V / S each; a slot's CL lanes load a block's values in CL pieces and 16
// bytes each of the BC panel rows, and pass the values around by quad permutations.  A load
// instruction of a wave so covers the whole 64- or 32-byte panel rows of 16 or 32 blocks, where
// one lane per block touched 64 different lines for 16 bytes each: the kernel was bound by
// those L1 accesses.  The tree's upper levels join a slot's chains, the lower ones the slots;
// every lane then holds its columns of all BR rows, and slot s finishes rows s, s + S, ...
// 262,144 rows of 27 3x3 blocks: FP64 248 -> 179 us (3.5 TB/s on the bytes of A, x and y), FP32
// 116 -> 88; its prolongator 79 -> 45 and restriction 95 -> 50 us in FP64.  The vector units
// bound it as much as the loads do, so the chains are loops and the 3x3 kernel is held to 72
// registers (seven waves a SIMD): unrolled it takes 138, or 72 with spills, and 265 us.
template <int BR, int BC, int G, int U, class TM, class TX, class TA, class Epi>
__global__ __launch_bounds__(kBlock, BR * BC == 9 && U == 1 ? 7 : 1) void spmm8_kernel(
    int nbr, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx, const TM* __restrict__ val,
    const TX* __restrict__ x, Epi epi) {
  constexpr int CL = kColLanes<TX>, CPL = 8 / CL, S = G / CL;
  constexpr int BE = BR * BC, PER = (BE + CL - 1) / CL;
  constexpr int V = kChains<TX, G, U>, T = V / S;
  static_assert(G % CL == 0 && (T == 2 || T == 4), "a slot takes two or four chains");
  using Sums = ColSums<BR, CPL, TA>;
  constexpr int kRows = kBlock / G;
  const int lb = xcd_chunked_block(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x), kSpmvChunk);
  const int row = lb * kRows + static_cast<int>(threadIdx.x) / G;
  const int lane = static_cast<int>(threadIdx.x) % G;
  const int slot = lane / CL, cl = lane % CL;
  const int piece = cl * PER < BE - PER ? cl * PER : BE - PER;  // the lane's values of a block
  Sums sum{};
  const bool active = row < nbr;
  if (active) {
    const int k1 = rowptr[row + 1];
    const int k0 = rowptr[row] + slot;
#pragma unroll 1
    for (int h = 0; h < T / 2; ++h) {
      Sums pair{};
#pragma unroll 1
      for (int t = h; t < T; t += T / 2) {
        Sums chain{};
#pragma unroll 1
        for (int kb = k0 + t * S; kb < k1; kb += V * U) {
          TM raw[U][PER];
          TA xv[U][BC][CPL];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int k = kb + u * V;
            if (k < k1) {
              const TX* xc = x + static_cast<size_t>(colidx[k]) * (BC * 8) + cl * CPL;
              const TM* b = val + static_cast<size_t>(k) * BE + piece;
#pragma unroll
              for (int e = 0; e < PER; ++e) raw[u][e] = b[e];
#pragma unroll
              for (int j = 0; j < BC; ++j) ld_cols<TA>(xc + j * 8, xv[u][j]);
            } else {
#pragma unroll
              for (int e = 0; e < PER; ++e) raw[u][e] = TM{};
#pragma unroll
              for (int j = 0; j < BC; ++j)
#pragma unroll
                for (int q = 0; q < CPL; ++q) xv[u][j][q] = TA(0);
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            TA a[PER];
#pragma unroll
            for (int e = 0; e < PER; ++e) a[e] = ld<TA>(&raw[u][e]);
            panel_fma<0, BE, BC, CL, PER, CPL, BR, TA>(a, xv[u], chain.v);
          }
        }
        pair.add(chain);
      }
      sum.add(pair);
    }
  }
  TA (&acc)[BR][CPL] = sum.v;
#pragma unroll
  for (int off = G / 2; off >= CL; off >>= 1) {
#pragma unroll
    for (int i = 0; i < BR; ++i)
#pragma unroll
      for (int q = 0; q < CPL; ++q) acc[i][q] += __shfl_xor(acc[i][q], off, G);
  }
  if (active) epi.template apply8<BR, S, CPL>(row, slot, cl, acc);
}

// mir != nullptr selects the symmetric reads (one right-hand side, square blocks;
// ignored otherwise).  Their workgroup runs per XCD then span sym_dist / 8 rows (one
// eighth of the matrix's typical lower bandwidth, e.g. one node plane of a 3D mesh in
// natural order): run r + 8, the next run of the same XCD, holds the rows sym_dist
// further on, whose mirrored lower blocks run r has just streamed into that XCD's L2.
template <int BR, int BC, int NR, int G, int U, class TM, class TX, class TA, class Epi>
int launch_g(int nbr, const int32_t* rowptr, const int32_t* colidx, const TM* val, const TX* x, const Epi& epi,
             hipStream_t s, const int32_t* mir, int sym_dist) {
  const int grid = ceil_div(nbr, kBlock / G);
  constexpr int kRows = kBlock / G;
  const int sym_chunk =
      sym_dist > 0 ? std::max(1, std::min(1 << 16, (sym_dist + kNumXcd * kRows / 2) / (kNumXcd * kRows))) : kSpmvChunk;
  if constexpr (NR == 8) {
    static_assert(!Epi::kReduce, "reducing epilogues take one right-hand side");
    spmm8_kernel<BR, BC, G, U, TM, TX, TA, Epi><<<grid, kBlock, 0, s>>>(nbr, rowptr, colidx, val, x, epi);
  } else if constexpr (BR == BC) {
    if (mir)
      spmv_kernel<BR, BC, NR, G, U, TM, TX, TA, Epi, true><<<grid, kBlock, 0, s>>>(nbr, rowptr, colidx, val, x, epi,
                                                                                    mir, sym_chunk);
    else
      spmv_kernel<BR, BC, NR, G, U, TM, TX, TA, Epi><<<grid, kBlock, 0, s>>>(nbr, rowptr, colidx, val, x, epi);
  } else {
    spmv_kernel<BR, BC, NR, G, U, TM, TX, TA, Epi><<<grid, kBlock, 0, s>>>(nbr, rowptr, colidx, val, x, epi);
  }
  return grid;
}

// Lane configuration: G lanes per block row (power of two, <= 64), U blocks per lane
// per step.  Encoded as G * 8 + U.
inline int lane_code(int G, int U) { return G * 8 + U; }

// Every lane code launch_rows compiles.
constexpr int kLaneCodes[] = {8 * 8 + 1, 8 * 8 + 2, 16 * 8 + 1, 16 * 8 + 2, 32 * 8 + 1, 32 * 8 + 2, 64 * 8 + 1, 64 * 8 + 2};

// Launch spmv_kernel with (G, U) chosen at run time; returns the number of
// workgroups (= number of partial sums written by a reducing epilogue).
template <int BR, int BC, int NR, class TM, class TX, class TA, class Epi>
int launch_rows(int code, int nbr, const int32_t* rowptr, const int32_t* colidx, const TM* val, const TX* x,
                const Epi& epi, hipStream_t s, const int32_t* mir = nullptr, int sym_dist = 0) {
  if (nbr <= 0) return 0;
  int grid;
  switch (code) {
#define BLK_CASE(GG, UU)                                                                                        \
  case GG * 8 + UU:                                                                                             \
    grid = launch_g<BR, BC, NR, GG, UU, TM, TX, TA, Epi>(nbr, rowptr, colidx, val, x, epi, s, mir, sym_dist);   \
    break;
    BLK_CASE(8, 1)
    BLK_CASE(8, 2)
    BLK_CASE(16, 1)
    BLK_CASE(16, 2)
    BLK_CASE(32, 1)
    BLK_CASE(32, 2)
    BLK_CASE(64, 1)
    BLK_CASE(64, 2)
#undef BLK_CASE
    default:
      grid = launch_g<BR, BC, NR, 64, 2, TM, TX, TA, Epi>(nbr, rowptr, colidx, val, x, epi, s, mir, sym_dist);
      break;
  }
  HIP_CHECK(hipGetLastError());
  return grid;
}

inline int grid_for(int G, int nbr) { return ceil_div(nbr, kBlock / G); }

// Epilogues implement
//   prefetch<BR,NR,G>(active, row) -> Pre   (own-row operands, loaded early)
//   apply<BR,NR,G>(active, row, lane, acc, pre) -> contribution to a block sum
// and set kReduce when the contributions are to be summed (partial[] per block).
struct NoPre {};

template <class T, int N>
struct RowVals {
  T v[N];
};

// When the BR * NR outputs of a row fit in its lane group (BR * NR <= G), lane l < BR * NR
// owns output l: it alone loads that output's own-row operands and stores it, instead
// of every lane of the group loading all of them.
template <int N, int G>
constexpr bool lane_owned() { return N <= G; }

// y = alpha * (A x) + beta * y
template <class TY, class TA>
struct EpiAxpby {
  static constexpr bool kReduce = false;
  TY* __restrict__ y;
  TA alpha, beta;
  double* partial = nullptr;
  template <int BR, int NR, int G>
  static constexpr int pre_len() { return lane_owned<BR * NR, G>() ? 1 : BR * NR; }
  template <int BR, int NR, int G>
  __device__ __forceinline__ RowVals<TA, pre_len<BR, NR, G>()> prefetch(bool active, int row) const {
    constexpr int N = BR * NR;
    RowVals<TA, pre_len<BR, NR, G>()> p;
#pragma unroll
    for (int t = 0; t < pre_len<BR, NR, G>(); ++t) p.v[t] = TA(0);
    if (!active || beta == TA(0)) return p;
    if constexpr (lane_owned<N, G>()) {
      const int lane = min(static_cast<int>(threadIdx.x) % G, N - 1);
      p.v[0] = ld<TA>(y + static_cast<size_t>(row) * N + lane);
    } else {
#pragma unroll
      for (int t = 0; t < N; ++t) p.v[t] = ld<TA>(y + static_cast<size_t>(row) * N + t);
    }
    return p;
  }
  template <int BR, int NR, int G>
  __device__ __forceinline__ double apply(bool active, int row, int lane, const TA (&acc)[BR * NR],
                                          const RowVals<TA, pre_len<BR, NR, G>()>& pre) const {
    constexpr int N = BR * NR;
    if (!active) return 0.0;
    if constexpr (lane_owned<N, G>()) {
      if (lane < N) {
        TA v = alpha * pick<N>(acc, lane);
        if (beta != TA(0)) v = fmadd(beta, pre.v[0], v);
        st(y + static_cast<size_t>(row) * N + lane, v);
      }
    } else {
#pragma unroll
      for (int l = 0; l < N; ++l) {
        if ((l % G) != lane) continue;
        TA v = alpha * acc[l];
        if (beta != TA(0)) v = fmadd(beta, pre.v[l], v);
        st(y + static_cast<size_t>(row) * N + l, v);
      }
    }
    return 0.0;
  }
  // eight right-hand sides: columns cl * CPL .. of rows slot, slot + S, ...
  template <int BR, int S, int CPL>
  __device__ __forceinline__ void apply8(int row, int slot, int cl, const TA (&acc)[BR][CPL]) const {
#pragma unroll
    for (int i = 0; i < BR; ++i) {
      if (i % S != slot) continue;
      TY* yp = y + (static_cast<size_t>(row) * BR + i) * 8 + cl * CPL;
      TA v[CPL], old[CPL];
      if (beta != TA(0)) ld_cols<TA>(yp, old);
#pragma unroll
      for (int q = 0; q < CPL; ++q) {
        v[q] = alpha * acc[i][q];
        if (beta != TA(0)) v[q] = fmadd(beta, old[q], v[q]);
      }
      st_cols(yp, v);
    }
  }
};

}  // namespace blk
