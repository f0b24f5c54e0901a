// Galerkin product of the 3x3-blocked level in bricks (paper §2.1, §3.1, §3.5), symmetric
// mode: A P never leaves the chip.
//
// The rows whose product row in A P starts at the same coarse column form a brick (27 rows
// on a lattice of 3x3x3 aggregates); one workgroup takes a brick in batches of rows (nine,
// one layer).  Per batch it stages the rows of A and every row of P they multiply in LDS,
// forms the rows of A P the upper triangle of A_c needs, and adds P^T (A P) to the brick's
// coarse blocks, which stay in registers over the batches.  Each brick writes its coarse
// blocks once as partial sums; a last kernel adds the partial sums of every coarse block
// in a fixed order and writes the block and its mirror.
//
// Why: the two separate passes were bound by their gathers.  At 128^3 the A P pass made 27
// L1 accesses per load instruction for 144-byte blocks of P (81 % of the L1's cycles), and
// the R (A P) pass fetched every A P row 3 to 4 times from beyond L2 (17.9 GB, 5.2 TB/s).
// Here P is read once per batch in contiguous runs, A P costs no memory traffic, and the
// partial sums (86 blocks a brick on that lattice) are written and read once.
// Measured, two passes -> bricks, for 100^3 elements: FP64 4.03 -> 2.70 ms, FP32 2.64 -> 2.04,
// P in BF16 2.50 -> 1.99; 40^3: 0.30 -> 0.21, 0.20 -> 0.14, 0.20 -> 0.14; 16^3: 0.091 -> 0.061,
// 0.114 -> 0.041, 0.108 -> 0.041.  No size was found where the two passes win, so they are
// taken where the patterns do not fit (below), and for a plan used once.  The tables cost a
// plan 0.3 ms at 40^3 and 2.8 ms at 100^3, two to three products' gain.
// What bounds it now (100^3, FP64): a batch is staged, multiplied and added in turn between
// barriers; two workgroups a CU overlap, with the LDS 47 % and the VALU 44 % busy, and the
// loads of a batch wait some 560 cycles each for the L1.  A third workgroup a CU does not fit
// the registers (128), and 48 more bytes spilled a lane cost 9 %.
#include <algorithm>
#include <array>
#include <type_traits>

#include <hipcub/hipcub.hpp>

#include "ptap_plan.hpp"
#include "spmv_core.hpp"

namespace blk {
namespace {

// Four lanes (a quad) work on a 3x6 or 6x6 block: lane m < 3 takes the products over inner
// index m, and the quad's sums are added at the end.  So a contribution costs a lane nine
// values from LDS in A P (three of A, six of P) and twelve in P^T (A P).
constexpr int kQuads = 128;              // blocks of a batch, and of a brick, at most
constexpr int kThreads = 4 * kQuads;     // eight waves: two workgroups fill a CU evenly at 128 registers
constexpr int kChunk = 16;               // quads of a wave
constexpr int kBatchRows = 64;           // rows of a batch at most
constexpr int kGroupRows = 128;          // rows of a brick at most
constexpr int kGroupCand = 1024;         // contributions of a brick at most (their codes lie in LDS)
constexpr int kPiece = 7;                // P blocks one wave instruction copies (nine lanes a block)
constexpr int kPieces = kThreads;        // pieces of a batch at most: a wave holds its own ones, a lane each
constexpr int kBlk = 18;                 // values of a 3x6 block
constexpr int kLdsP = 50 * 1024;         // LDS for the rows of P: two workgroups stay on a CU

__device__ __forceinline__ int lower_bound(const int32_t* __restrict__ v, int lo, int hi, int key) {
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (v[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// ---------------------------------------------------------------------------
// symbolic
// ---------------------------------------------------------------------------
struct Patterns {
  int nrows, ncoarse, keep;
  const int32_t *a_rp, *a_ci, *p_rp, *p_ci, *ap_rp, *ap_ci;
};

// Per row: brick key (first column of its A P row; ncoarse = in no brick), first needed
// A P block (the first whose column is not below the row's first P column: the others only
// feed lower blocks of A_c), needed blocks and contributions to upper coarse blocks.
__global__ void brick_rows_kernel(Patterns t, uint32_t* __restrict__ key, int32_t* __restrict__ iota,
                                  int32_t* __restrict__ first, int32_t* __restrict__ need,
                                  int32_t* __restrict__ cand) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= t.nrows) return;
  const int s0 = t.ap_rp[i], s1 = t.ap_rp[i + 1], q0 = t.p_rp[i], q1 = t.p_rp[i + 1];
  int c = 0, f = s0;
  for (int q = q0; q < q1; ++q) {
    const int lb = lower_bound(t.ap_ci, s0, s1, t.p_ci[q]);
    if (q == q0 && !t.keep) f = lb;
    c += s1 - lb;
  }
  const bool in = s1 > s0 && (t.keep || q1 > q0);
  key[i] = in ? static_cast<uint32_t>(t.ap_ci[s0]) : static_cast<uint32_t>(t.ncoarse);
  iota[i] = i;
  first[i] = f;
  need[i] = in ? s1 - f : 0;
  cand[i] = in ? c : 0;
}

// Rows in brick order: their sizes, and where a key's rows begin.  total: rows in bricks,
// contributions to upper coarse blocks.
__global__ void brick_gather_kernel(Patterns t, const uint32_t* __restrict__ key, const int32_t* __restrict__ rows,
                                    const int32_t* __restrict__ first, const int32_t* __restrict__ need,
                                    const int32_t* __restrict__ cand, int32_t* __restrict__ first_s,
                                    int32_t* __restrict__ need_s, int32_t* __restrict__ alen_s,
                                    int32_t* __restrict__ cand_s, int32_t* __restrict__ head,
                                    unsigned long long* __restrict__ total) {
  const int pos = blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long sum = pos < t.nrows ? static_cast<unsigned long long>(cand[rows[pos]]) : 0ull;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  if ((threadIdx.x & 63) == 0 && sum) atomicAdd(total + 1, sum);
  if (pos >= t.nrows) return;
  const uint32_t nc = static_cast<uint32_t>(t.ncoarse);
  const int i = rows[pos];
  const bool in = key[pos] < nc;
  first_s[pos] = first[i];
  need_s[pos] = need[i];
  cand_s[pos] = cand[i];
  alen_s[pos] = in ? t.a_rp[i + 1] - t.a_rp[i] : 0;
  head[pos] = in && (pos == 0 || key[pos - 1] != key[pos]) ? 1 : 0;
  if (in && (pos + 1 == t.nrows || key[pos + 1] >= nc)) total[0] = static_cast<unsigned long long>(pos) + 1ull;
}

// Walk of every key's rows: a brick is split where it would exceed the limits of a brick,
// and its rows into batches.  bad = a row beyond the limits of a batch by itself.
__global__ void brick_split_kernel(int used, int a_cap, int ap_cap, const int32_t* __restrict__ key_head,
                                   const int32_t* __restrict__ need, const int32_t* __restrict__ alen,
                                   const int32_t* __restrict__ cand, int32_t* __restrict__ ghead,
                                   int32_t* __restrict__ bhead, int* __restrict__ bad) {
  const int p0 = blockIdx.x * blockDim.x + threadIdx.x;
  if (p0 >= used || !key_head[p0]) return;
  int gr = 0, gc = 0, br = 0, bn = 0, ba = 0;
  for (int p = p0; p < used && (p == p0 || !key_head[p]); ++p) {
    const int n = need[p], a = alen[p], c = cand[p];
    if (n > ap_cap || a > a_cap || c > kGroupCand) *bad = 1;
    const bool g = p == p0 || gr + 1 > kGroupRows || gc + c > kGroupCand;
    const bool b = g || br + 1 > kBatchRows || bn + n > ap_cap || ba + a > a_cap;
    if (g) gr = gc = 0;
    if (b) br = bn = ba = 0;
    ++gr;
    gc += c;
    ++br;
    bn += n;
    ba += a;
    ghead[p] = g ? 1 : 0;
    bhead[p] = b ? 1 : 0;
  }
}

// first row of every brick and batch, first batch of every brick (gid / bid: inclusive sums)
__global__ void brick_ptr_kernel(int used, const int32_t* __restrict__ ghead, const int32_t* __restrict__ bhead,
                                 const int32_t* __restrict__ gid, const int32_t* __restrict__ bid,
                                 int32_t* __restrict__ group_row, int32_t* __restrict__ batch_row,
                                 int32_t* __restrict__ group_batch) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= used) return;
  if (bhead[p]) batch_row[bid[p] - 1] = p;
  if (ghead[p]) {
    group_row[gid[p] - 1] = p;
    group_batch[gid[p] - 1] = bid[p] - 1;
  }
  if (p == used - 1) {
    batch_row[bid[p]] = used;
    group_row[gid[p]] = used;
    group_batch[gid[p]] = bid[p];
  }
}

// bitonic sort of n keys (padded to a power of two) by the whole workgroup
template <class K>
__device__ __forceinline__ void sort_lds(K* keys, int n, K pad) {
  int p2 = 1;
  while (p2 < n) p2 <<= 1;
  for (int i = n + threadIdx.x; i < p2; i += blockDim.x) keys[i] = pad;
  __syncthreads();
  for (int size = 2; size <= p2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = threadIdx.x; t < p2 / 2; t += blockDim.x) {
        const int lo = 2 * stride * (t / stride) + (t % stride), hi = lo + stride;
        const K a = keys[lo], b = keys[hi];
        if ((a > b) == ((lo & size) == 0)) {
          keys[lo] = b;
          keys[hi] = a;
        }
      }
      __syncthreads();
    }
}

// The upper coarse blocks a brick adds to, and each one's contributions in (row, P block,
// A P block) order: at out[g * max_out], blocks ordered by falling contribution count (lanes
// of a wave then run loops of similar length): {the block's index among the upper ones, its
// codes end << 16 | begin in the brick's}.  A code: row << 24 | LDS block of P << 8 | LDS
// block of A P, both in the row's batch.  Eight lanes generate a row, one per block of P.
__global__ __launch_bounds__(256) void brick_outputs_kernel(Patterns t, int max_out,
                                                            const int32_t* __restrict__ group_row,
                                                            const int32_t* __restrict__ rows,
                                                            const int32_t* __restrict__ first,
                                                            const int32_t* __restrict__ cand_off,
                                                            const int32_t* __restrict__ need_off,
                                                            const uint16_t* __restrict__ own,
                                                            const uint8_t* __restrict__ rank_of,
                                                            const int32_t* __restrict__ c_rp,
                                                            const int32_t* __restrict__ c_ci,
                                                            const int32_t* __restrict__ up_rp,
                                                            int32_t* __restrict__ n_out, int2* __restrict__ out,
                                                            uint32_t* __restrict__ codes, int* __restrict__ bad) {
  constexpr int kMax = 256;
  __shared__ uint64_t keys[kGroupCand];
  __shared__ uint32_t pay[kGroupCand];
  __shared__ int beg[kMax + 1];
  __shared__ int n_runs;
  const int g = blockIdx.x;
  const int p0 = group_row[g], p1 = group_row[g + 1];
  const int base = cand_off[p0], n = cand_off[p1] - base;
  const int sub = threadIdx.x & 7;
  for (int pb = p0; pb < p1; pb += 32) {
    const int p = min(pb + static_cast<int>(threadIdx.x >> 3), p1 - 1);
    const bool in = pb + static_cast<int>(threadIdx.x >> 3) < p1;
    const int i = rows[p], s0 = t.ap_rp[i], s1 = t.ap_rp[i + 1], f = first[p];
    const int q0 = t.p_rp[i], q1 = t.p_rp[i + 1], own_p = own[p], need_p = need_off[p];
    int at0 = cand_off[p] - base;
    for (int qb = q0; qb < q1; qb += 8) {  // the eight lanes of a row run it together
      const int q = qb + sub, a = q < q1 ? t.p_ci[q] : 0;
      const int lo = q < q1 ? lower_bound(t.ap_ci, s0, s1, a) : s1;
      int incl = s1 - lo;
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) {
        const int v = __shfl_up(incl, d, 8);
        if (sub >= d) incl += v;
      }
      if (in && lo < s1) {
        int at = at0 + incl - (s1 - lo);
        const int tail = c_rp[a + 1] - (up_rp[a + 1] - up_rp[a]);  // the upper columns end the full row
        int c = tail;
        for (int s = lo; s < s1; ++s) {
          c = lower_bound(c_ci, c, c_rp[a + 1], t.ap_ci[s]);
          const int u = up_rp[a] + c - tail;
          keys[at] = (static_cast<uint64_t>(static_cast<uint32_t>(u)) << 32) | static_cast<uint32_t>(at);
          pay[at] = (static_cast<uint32_t>(p - p0) << 24) | (static_cast<uint32_t>(own_p + q - q0) << 8) |
                    rank_of[need_p + s - f];
          ++at;
        }
      }
      at0 += __shfl(incl, 7, 8);
    }
  }
  __syncthreads();
  sort_lds<uint64_t>(keys, n, ~uint64_t{0});
  // starts of the runs of equal u, found in order by one wave
  if (threadIdx.x < 64) {
    int runs = 0;
    for (int b = 0; b < n; b += 64) {
      const int p = b + static_cast<int>(threadIdx.x);
      const bool start = p < n && (p == 0 || (keys[p] >> 32) != (keys[p - 1] >> 32));
      const uint64_t ball = __ballot(start);
      const int at = runs + __popcll(ball & ((1ull << threadIdx.x) - 1ull));
      if (start && at < kMax) beg[at] = p;
      runs += __popcll(ball);
    }
    if (threadIdx.x == 0) {
      n_runs = runs;
      beg[min(runs, kMax)] = n;
    }
  }
  __syncthreads();
  const int m = n_runs, r = threadIdx.x;
  if (r == 0) {
    n_out[g] = m;
    if (m > max_out) *bad = 1;
  }
  if (m > max_out) return;
  if (r < m) {
    const int c = beg[r + 1] - beg[r];
    int rank = 0;
    for (int o = 0; o < m; ++o) {
      const int d = beg[o + 1] - beg[o];
      rank += (d > c || (d == c && o < r)) ? 1 : 0;
    }
    out[static_cast<size_t>(g) * max_out + rank] =
        make_int2(static_cast<int32_t>(keys[beg[r]] >> 32), beg[r + 1] << 16 | beg[r]);
  }
  for (int p = r; p < n; p += 256) codes[base + p] = pay[static_cast<uint32_t>(keys[p])];
}

// The bricks' coarse blocks one after the other
__global__ __launch_bounds__(256) void brick_slots_kernel(int max_out, const int32_t* __restrict__ group_row,
                                                          const int32_t* __restrict__ cand_off,
                                                          const int32_t* __restrict__ slot_ptr,
                                                          const int2* __restrict__ out, int32_t* __restrict__ slot_u,
                                                          int32_t* __restrict__ iota, int32_t* __restrict__ slot_beg,
                                                          int32_t* __restrict__ slot_end) {
  const int g = blockIdx.x, r = threadIdx.x, at = slot_ptr[g] + r;
  if (at >= slot_ptr[g + 1]) return;
  const int2 o = out[static_cast<size_t>(g) * max_out + r];
  const int base = cand_off[group_row[g]];
  slot_u[at] = o.x;
  iota[at] = at;
  slot_beg[at] = base + (o.y & 0xFFFF);
  slot_end[at] = base + (o.y >> 16);
}

// The rows of P a batch multiplies (those of its A entries and its own rows), and where
// each one lies in LDS when they are copied one after the other.  COUNT: number of blocks
// and of pieces (up to seven consecutive blocks of P, one wave instruction each) at the
// batch's first row, and its end there (a batch counted before, with the same end, is
// passed over); otherwise the pieces (first block; blocks << 16 | LDS block), pofs of each
// A entry and own of each row.
constexpr int kMaxKeys = 1024;
template <bool COUNT>
__global__ __launch_bounds__(256) void brick_stage_kernel(Patterns t, const int32_t* __restrict__ batch_row,
                                                          const int32_t* __restrict__ rows,
                                                          const int32_t* __restrict__ a_off,
                                                          int32_t* __restrict__ n_pieces,
                                                          int32_t* __restrict__ n_blocks, int32_t* __restrict__ n_end,
                                                          const int32_t* __restrict__ piece_ptr,
                                                          int2* __restrict__ pieces, uint16_t* __restrict__ pofs,
                                                          uint16_t* __restrict__ own) {
  __shared__ int32_t key[kMaxKeys];
  __shared__ int32_t ofs[kMaxKeys];
  __shared__ uint8_t head[kMaxKeys];
  __shared__ int count, made;
  const int b = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int p0 = batch_row[b], p1 = batch_row[b + 1];
  if (COUNT && n_end[p0] == p1) return;
  const int a0 = a_off[p0], na = a_off[p1] - a0, n = na + p1 - p0;
  for (int p = p0 + wave; p < p1; p += 4) {
    const int i = rows[p], k0 = t.a_rp[i], at = a_off[p] - a0, len = a_off[p + 1] - a_off[p];
    for (int k = lane; k < len; k += 64) key[at + k] = t.a_ci[k0 + k];
  }
  for (int p = threadIdx.x; p < p1 - p0; p += 256) key[na + p] = rows[p0 + p];
  if (threadIdx.x == 0) made = 0;
  __syncthreads();
  sort_lds<int32_t>(key, n, INT32_MAX);
  // distinct rows, their offsets and the heads of runs of consecutive rows, in order by one
  // wave, in place (an entry moves to a position already read)
  if (threadIdx.x < 64) {
    int uniq = 0, off = 0;
    for (int base = 0; base < n; base += 64) {
      const int p = base + lane;
      const int j = p < n ? key[p] : 0, before = p > 0 && p < n ? key[p - 1] : -2;
      const bool start = p < n && j != before;
      const int len = start ? t.p_rp[j + 1] - t.p_rp[j] : 0;
      const uint64_t su = __ballot(start);
      int incl = len;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(incl, d, 64);
        if (lane >= d) incl += v;
      }
      __builtin_amdgcn_wave_barrier();
      if (start) {
        const int u = uniq + __popcll(su & ((1ull << lane) - 1ull));
        key[u] = j;
        ofs[u] = off + incl - len;
        head[u] = before + 1 != j;
      }
      __builtin_amdgcn_wave_barrier();
      uniq += __popcll(su);
      off += __shfl(incl, 63, 64);
    }
    if (lane == 0) {
      count = uniq;
      if (COUNT) n_blocks[p0] = off;
    }
  }
  __syncthreads();
  // pieces of the run that starts at u (in any order: each names its own place)
  const int uniq = count;
  for (int u = threadIdx.x; u < uniq; u += 256) {
    if (!head[u]) continue;
    int e = u + 1;
    while (e < uniq && !head[e]) ++e;
    const int from = t.p_rp[key[u]], blocks = t.p_rp[key[e - 1] + 1] - from;
    const int np = (blocks + kPiece - 1) / kPiece;
    const int at = atomicAdd(&made, np);
    if constexpr (!COUNT)
      for (int q = 0; q < np; ++q)
        pieces[piece_ptr[b] + at + q] =
            make_int2(from + q * kPiece, min(kPiece, blocks - q * kPiece) << 16 | (ofs[u] + q * kPiece));
  }
  if constexpr (COUNT) {
    __syncthreads();
    if (threadIdx.x == 0) {
      n_pieces[p0] = made;
      n_end[p0] = p1;
    }
    return;
  }
  for (int p = p0 + wave; p < p1; p += 4) {
    const int i = rows[p], k0 = t.a_rp[i], at = a_off[p], len = a_off[p + 1] - at;
    for (int k = lane; k < len; k += 64)
      pofs[at + k] = static_cast<uint16_t>(ofs[lower_bound(key, 0, uniq, t.a_ci[k0 + k])]);
  }
  for (int p = p0 + static_cast<int>(threadIdx.x); p < p1; p += 256)
    own[p] = static_cast<uint16_t>(ofs[lower_bound(key, 0, uniq, rows[p])]);
}

// A batch too large for LDS, or of more pieces than the waves hold (scattered rows of one P
// block each), is cut in two at its middle row (bhead set there); a single row that does not
// fit ends the attempt.
__global__ void brick_cut_kernel(int nb, int p_cap, const int32_t* __restrict__ batch_row,
                                 const int32_t* __restrict__ n_blocks, const int32_t* __restrict__ n_pieces,
                                 int32_t* __restrict__ bhead,
                                 int* __restrict__ cut, int* __restrict__ bad) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const int p0 = batch_row[b], p1 = batch_row[b + 1];
  if (n_blocks[p0] <= p_cap && n_pieces[p0] <= kPieces) return;
  if (p1 - p0 < 2) *bad = 1;
  else bhead[(p0 + p1) / 2] = 1;
  *cut = 1;
}

// Sizes by batch: pieces, chunks of A P blocks; the largest number of P blocks
__global__ void brick_sizes_kernel(int nb, const int32_t* __restrict__ batch_row, const int32_t* __restrict__ pos_pieces,
                                   const int32_t* __restrict__ pos_blocks, const int32_t* __restrict__ need_off,
                                   int32_t* __restrict__ n_pieces, int32_t* __restrict__ n_chunks,
                                   int* __restrict__ most) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  int blocks = 0;
  if (b < nb) {
    const int p0 = batch_row[b];
    n_pieces[b] = pos_pieces[p0];
    n_chunks[b] = (need_off[batch_row[b + 1]] - need_off[p0] + kChunk - 1) / kChunk;
    blocks = pos_blocks[p0];
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) blocks = max(blocks, __shfl_xor(blocks, d, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(most, blocks);
}

// Inside every batch, the needed A P blocks by falling number of contributions.  LEN:
// rank_of each, and the sizes of its 16-block chunks' code tables (a chunk's first block is
// its longest).  Otherwise the tables: code e of rank r at chunk_off + 16 e + r % 16, A entry
// of the batch << 16 | LDS block of P; count and the A P block of each rank.
template <bool LEN, class CT>
__global__ __launch_bounds__(kQuads) void brick_order_kernel(const int32_t* __restrict__ batch_row,
                                                          const int32_t* __restrict__ need_off,
                                                          const int32_t* __restrict__ a_off,
                                                          const int32_t* __restrict__ first,
                                                          const int32_t* __restrict__ pp, const CT* __restrict__ codes,
                                                          int shift, const uint16_t* __restrict__ pofs,
                                                          uint8_t* __restrict__ rank_of,
                                                          const int32_t* __restrict__ batch_chunk,
                                                          int32_t* __restrict__ chunk_len,
                                                          const int32_t* __restrict__ chunk_off,
                                                          uint32_t* __restrict__ ell, uint16_t* __restrict__ count,
                                                          int32_t* __restrict__ slot_ap) {
  __shared__ int need[kBatchRows + 1], from[kBatchRows], cnt[kQuads];
  const int b = blockIdx.x, s = threadIdx.x;
  const int p0 = batch_row[b], nr = batch_row[b + 1] - p0;
  const int n0 = need_off[p0];
  if (s <= nr) need[s] = need_off[p0 + s] - n0;
  if (s < nr) from[s] = first[p0 + s];
  __syncthreads();
  const int n = need[nr];
  if (s >= n && LEN) cnt[s] = 0;
  int row = 0, q0 = 0, len = 0;
  if (s < n) {
    for (int hi = nr; hi - row > 1;) {
      const int mid = (row + hi) >> 1;
      if (need[mid] <= s) row = mid; else hi = mid;
    }
    const int q = from[row] + s - need[row];
    q0 = pp[q];
    len = pp[q + 1] - q0;
    if constexpr (LEN) cnt[s] = len;
    else if (slot_ap) slot_ap[n0 + rank_of[n0 + s]] = q;
  }
  if constexpr (LEN) {
    __syncthreads();
    int rank = 0;
    if (s < n) {
      for (int o = 0; o < n; ++o) rank += (cnt[o] > len || (cnt[o] == len && o < s)) ? 1 : 0;
      rank_of[n0 + s] = static_cast<uint8_t>(rank);
      if (rank % kChunk == 0) chunk_len[batch_chunk[b] + rank / kChunk] = len * kChunk;
    }
  } else if (s < n) {
    const int rank = rank_of[n0 + s];
    const int a0 = a_off[p0 + row], rel = a0 - a_off[p0];
    uint32_t* o = ell + chunk_off[batch_chunk[b] + rank / kChunk] + rank % kChunk;
    for (int e = 0; e < len; ++e) {
      const uint32_t c = codes[q0 + e];
      const int k = static_cast<int>(c >> shift), lo = static_cast<int>(c & ((1u << shift) - 1u));
      o[e * kChunk] = (static_cast<uint32_t>(rel + k) << 16) | static_cast<uint32_t>(pofs[a0 + k] + lo);
    }
    count[n0 + rank] = static_cast<uint16_t>(len);
  }
}

// What the numeric kernel reads first: per brick {first row, first batch, first coarse
// block, first contribution}, per batch {first row, first needed A P block, first piece,
// first chunk}, each with one more entry for the ends; per row its first A entry.
__global__ void brick_desc_kernel(int ng, int nb, int used, const int32_t* __restrict__ group_row,
                                  const int32_t* __restrict__ group_batch, const int32_t* __restrict__ slot_ptr,
                                  const int32_t* __restrict__ cand_off, const int32_t* __restrict__ batch_row,
                                  const int32_t* __restrict__ need_off, const int32_t* __restrict__ piece_ptr,
                                  const int32_t* __restrict__ batch_chunk, const int32_t* __restrict__ rows,
                                  const int32_t* __restrict__ a_rp, int4* __restrict__ brick, int4* __restrict__ batch,
                                  int32_t* __restrict__ a_first) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i <= ng) brick[i] = make_int4(group_row[i], group_batch[i], slot_ptr[i], cand_off[group_row[i]]);
  if (i <= nb) batch[i] = make_int4(batch_row[i], need_off[batch_row[i]], piece_ptr[i], batch_chunk[i]);
  if (i < used) a_first[i] = a_rp[rows[i]];
}

// seg[u] = first position of u among the sorted keys
__global__ void brick_seg_kernel(int nu, int n, const int32_t* __restrict__ key, int32_t* __restrict__ seg) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u <= nu) seg[u] = lower_bound(key, 0, n, u);
}

// ---------------------------------------------------------------------------
// numeric
// ---------------------------------------------------------------------------
template <class TA>
__device__ __forceinline__ void ld6(const TA* __restrict__ p, TA (&v)[6]) {
  using V = typename std::conditional<sizeof(TA) == 8, double2, float2>::type;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const V x = reinterpret_cast<const V*>(p)[t];
    v[2 * t] = x.x;
    v[2 * t + 1] = x.y;
  }
}

// v of another lane of the quad (DPP quad permutation)
template <int PERM, class T>
__device__ __forceinline__ T quad_perm(T v) {
  int w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int t = 0; t < static_cast<int>(sizeof(T) / 4); ++t)
    w[t] = __builtin_amdgcn_mov_dpp(w[t], PERM, 0xf, 0xf, true);
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}
// sum over a quad, in every lane of it
template <class TA>
__device__ __forceinline__ TA quad_sum(TA v) {
  v += quad_perm<0xB1>(v);  // lanes 1 0 3 2
  v += quad_perm<0x4E>(v);  // lanes 2 3 0 1
  return v;
}

struct BrickArgs {
  int ng, a_cap, p_cap;
  const int4 *brick, *batch;
  const int32_t *a_off, *a_first, *chunk_off;
  const int2* pieces;
  const uint32_t *ell, *c_codes;
  const uint16_t* count;
  const int32_t *slot_ap, *slot_beg, *slot_end;
};

__host__ __device__ constexpr size_t up16(size_t b) { return (b + 15) & ~static_cast<size_t>(15); }

// LDS of a workgroup: rows of P; A's blocks and, after them in the same place, the batch's
// A P blocks.
template <class TX, class TA>
size_t brick_lds(int a_cap, int p_cap) {
  return up16(static_cast<size_t>(p_cap) * kBlk * sizeof(TA)) +
         std::max(up16(static_cast<size_t>(a_cap) * 9 * sizeof(TX)), static_cast<size_t>(kQuads) * kBlk * sizeof(TA));
}

// two consecutive values, element alignment
template <class T>
struct Two {
  T a, b;
};
template <class TA, class T>
__device__ __forceinline__ Two<TA> ld_two(const T* p) {
  Two<T> v;
  __builtin_memcpy(&v, p, sizeof(v));
  return {ld<TA>(&v.a), ld<TA>(&v.b)};
}

// One workgroup per brick, two on a CU: one stages a batch (all loads of a wave in flight at
// once) while the other computes.  The code tables come a batch early into registers, so
// the loops over contributions read only LDS and registers.
template <class TX, class TP, class TA>
__global__ __launch_bounds__(kThreads, 4) void brick_kernel(BrickArgs g, const TX* __restrict__ a_v,
                                                                const TP* __restrict__ p_v, TA* __restrict__ ap_out,
                                                                TA* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char brick_sh[];
  __shared__ int ra[kGroupRows + 1], rk[kGroupRows];  // A entries before a row, its first entry
  __shared__ uint32_t ccode[kGroupCand];
  TA* const ps = reinterpret_cast<TA*>(brick_sh);
  unsigned char* const sh_a = brick_sh + up16(static_cast<size_t>(g.p_cap) * kBlk * sizeof(TA));
  TX* const as = reinterpret_cast<TX*>(sh_a);
  TA* const aps = reinterpret_cast<TA*>(sh_a);
  constexpr int kT = kThreads, kWaves = kT / 64;
  constexpr int UP = 8, UA = 4, UC = 7;  // pieces of P, halves of A rows, quads of codes held in registers
  const int lb = xcd_chunked_block(static_cast<int>(blockIdx.x), g.ng, 8);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int quad = tid >> 2, m = tid & 3, mm = m < 3 ? m : 2;
  const int4 d0 = g.brick[lb], d1 = g.brick[lb + 1];
  const int row0 = d0.x, nrows = d1.x - row0, b0 = d0.y, b1 = d1.y, cbase = d0.w, ncand = d1.w - cbase;
  const int out = d0.z + quad;
  const bool has_out = out < d1.z;
  int e = has_out ? g.slot_beg[out] - cbase : 0;
  const int e_end = has_out ? g.slot_end[out] - cbase : 0;
  if (tid <= nrows) {
    const int aoff0 = g.a_off[row0];
    ra[tid] = g.a_off[row0 + tid] - aoff0;
    if (tid < nrows) rk[tid] = g.a_first[row0 + tid];
  }
  for (int t = tid; t < ncand; t += kT) ccode[t] = g.c_codes[cbase + t];
  __syncthreads();
  TA acc[9];  // three rows of A_c by three columns
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = TA(0);
  const int pblk = min(lane / 9, kPiece - 1), pval = 2 * (lane % 9);  // lane's part of a piece
  uint32_t cd[UC];
  int n = 0;
  int4 bd = g.batch[b0], be = g.batch[b0 + 1];
  auto load_piece = [&](int2 pc) {
    const int blk = min(pblk, (pc.y >> 16) - 1);
    return ld_two<TA>(p_v + (static_cast<size_t>(pc.x) + blk) * kBlk + pval);
  };
  auto store_piece = [&](int2 pc, const Two<TA>& v) {
    if (lane < 9 * (pc.y >> 16)) {
      TA* d = ps + ((pc.y & 0xFFFF) + pblk) * kBlk + pval;
      d[0] = v.a;
      d[1] = v.b;
    }
  };
  // half h of row r of A: values 128 h + 2 lane, + 1 (a row of 28 blocks has two halves)
  auto load_a = [&](int r, int h) {
    const int len = (ra[r + 1] - ra[r]) * 9;
    return ld_two<TX>(a_v + static_cast<size_t>(rk[r]) * 9 + min(128 * h + 2 * lane, len - 2));
  };
  auto store_a = [&](int r, int h, int a0, const Two<TX>& v) {
    const int len = (ra[r + 1] - ra[r]) * 9, at = 128 * h + 2 * lane;
    TX* d = as + (ra[r] - a0) * 9;
    if (at + 1 < len) {
      d[at] = v.a;
      d[at + 1] = v.b;
    } else if (at < len) {
      d[at] = v.b;  // the load was moved back by one
    }
  };
  int2 pd;  // lane u holds the wave's u-th piece (kPieces: at most 64 a wave)
  auto piece = [&](int u) {
    return make_int2(__builtin_amdgcn_readlane(pd.x, u), __builtin_amdgcn_readlane(pd.y, u));
  };
  auto load_codes = [&]() {
    pd = g.pieces[min(bd.z + wave + kWaves * lane, be.z - 1)];
    n = 0;
    if (quad < be.y - bd.y) {
      n = g.count[bd.y + quad];
      const uint32_t* ell = g.ell + g.chunk_off[bd.w + wave] + quad % kChunk;
#pragma unroll
      for (int u = 0; u < UC; ++u) cd[u] = ell[min(4 * u + m, n - 1) * kChunk];
    }
  };
  load_codes();
  for (int b = b0; b < b1; ++b) {
    const int4 cur = bd, end = be;
    const int q0 = cur.x - row0, q1 = end.x - row0, a0 = ra[q0], ns = end.y - cur.y;
    {
      Two<TA> xp[UP];
      Two<TX> xa[UA];
#pragma unroll
      for (int u = 0; u < UA; ++u) xa[u] = load_a(min(q0 + wave + kWaves * (u / 2), q1 - 1), u % 2);
#pragma unroll
      for (int u = 0; u < UP; ++u) xp[u] = load_piece(piece(u));
#pragma unroll
      for (int u = 0; u < UA; ++u)
        if (q0 + wave + kWaves * (u / 2) < q1) store_a(q0 + wave + kWaves * (u / 2), u % 2, a0, xa[u]);
#pragma unroll
      for (int u = 0; u < UP; ++u)
        if (cur.z + wave + kWaves * u < end.z) store_piece(piece(u), xp[u]);
    }
    // what the registers do not hold: more pieces, more rows, longer rows
    for (int u = UP; cur.z + wave + kWaves * u < end.z; ++u) store_piece(piece(u), load_piece(piece(u)));
    for (int r = q0 + wave; r < q1; r += kWaves) {
      const int halves = ((ra[r + 1] - ra[r]) * 9 + 127) / 128;
      for (int h = r < q0 + wave + kWaves * (UA / 2) ? 2 : 0; h < halves; ++h) store_a(r, h, a0, load_a(r, h));
    }
    __syncthreads();
    // A P: lane m adds A[:, m] P[m, :] of every contribution
    TA ap[18];
#pragma unroll
    for (int t = 0; t < 18; ++t) ap[t] = TA(0);
    {
      auto fetch = [&](uint32_t code, TA (&x)[3], TA (&y)[6]) {
        const TX* pa = as + (code >> 16) * 9 + mm;
#pragma unroll
        for (int i = 0; i < 3; ++i) x[i] = pa[3 * i];
        ld6(ps + (code & 0xFFFFu) * kBlk + 6 * mm, y);
      };
      auto add = [&](const TA (&x)[3], const TA (&y)[6]) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int c = 0; c < 6; ++c) ap[6 * i + c] = fmadd(x[i], y[c], ap[6 * i + c]);
      };
      // two codes at a time; a code past the end repeats the last one and adds nothing
      auto two = [&](uint32_t c0, uint32_t c1, int left) {
        TA x0[3], y0[6], x1[3], y1[6];
        fetch(c0, x0, y0);
        fetch(c1, x1, y1);
        __builtin_amdgcn_sched_barrier(0);
        add(x0, y0);
        if (left > 1) add(x1, y1);
      };
      for (int base = 0; base < n; base += 4 * UC) {
        if (base > 0) {
          const uint32_t* ell = g.ell + g.chunk_off[cur.w + wave] + quad % kChunk;
#pragma unroll
          for (int u = 0; u < UC; ++u) cd[u] = ell[min(base + 4 * u + m, n - 1) * kChunk];
        }
#pragma unroll
        for (int u = 0; u < UC; ++u) {
          const int left = n - base - 4 * u;
          if (left > 0) {
            two(quad_perm<0x00>(cd[u]), quad_perm<0x55>(cd[u]), left);
            if (left > 2) two(quad_perm<0xAA>(cd[u]), quad_perm<0xFF>(cd[u]), left - 2);
          }
        }
      }
    }
    if (b + 1 < b1) {
      bd = end;
      be = g.batch[b + 2];
      load_codes();
    }
    if (m == 3) {
#pragma unroll
      for (int t = 0; t < 18; ++t) ap[t] = TA(0);
    }
#pragma unroll
    for (int t = 0; t < 18; ++t) ap[t] = quad_sum(ap[t]);
    __syncthreads();  // A's blocks have been read: the A P blocks take their place
    if (quad < ns && m < 3) {
      TA row[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) row[c] = m == 0 ? ap[c] : m == 1 ? ap[6 + c] : ap[12 + c];
#pragma unroll
      for (int c = 0; c < 6; ++c) aps[quad * kBlk + 6 * m + c] = row[c];
      if (ap_out) {
        TA* o = ap_out + static_cast<size_t>(g.slot_ap[cur.y + quad]) * kBlk + 6 * m;
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = row[c];
      }
    }
    __syncthreads();
    // A_c += P_i^T (A P)_i over the batch's rows, three rows by three columns a lane
    auto fetch_c = [&](uint32_t code, TA (&x)[9], TA (&y)[9]) {
      const TA* px = ps + ((code >> 8) & 0xFFFFu) * kBlk + 3 * (m >> 1);
      const TA* py = aps + (code & 0xFFu) * kBlk + 3 * (m & 1);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        x[t] = px[6 * (t / 3) + t % 3];
        y[t] = py[6 * (t / 3) + t % 3];
      }
    };
    auto add_c = [&](const TA (&x)[9], const TA (&y)[9]) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[3 * i + c] = fmadd(x[3 * k + i], y[3 * k + c], acc[3 * i + c]);
    };
    // the code after the current one is read ahead (0xFF...: no row has that number)
    uint32_t c0 = e < e_end ? ccode[e] : ~0u, c1 = e + 1 < e_end ? ccode[e + 1] : ~0u;
    const uint32_t past = static_cast<uint32_t>(q1) << 24;
    while (c0 < past) {
      TA x0[9], y0[9];
      fetch_c(c0, x0, y0);
      if (c1 < past) {
        TA x1[9], y1[9];
        fetch_c(c1, x1, y1);
        e += 2;
        c0 = e < e_end ? ccode[e] : ~0u;
        c1 = e + 1 < e_end ? ccode[e + 1] : ~0u;
        __builtin_amdgcn_sched_barrier(0);
        add_c(x0, y0);
        add_c(x1, y1);
      } else {
        e += 1;
        c0 = ~0u;
        add_c(x0, y0);
      }
    }
    __syncthreads();  // the next batch overwrites the LDS
  }
  if (has_out) {
    TA* o = partial + static_cast<size_t>(out) * 36 + 18 * (m >> 1) + 3 * (m & 1);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) o[6 * i + c] = acc[3 * i + c];
  }
}

// Upper coarse block u = the sum of its bricks' partial sums in brick order; three values a
// thread.  The transposed block goes to its mirror (-1 on the diagonal).
template <class TA>
__global__ __launch_bounds__(256) void brick_sum_kernel(int64_t nu, const int32_t* __restrict__ seg,
                                                        const int32_t* __restrict__ perm,
                                                        const TA* __restrict__ partial,
                                                        const int32_t* __restrict__ up_idx,
                                                        const int32_t* __restrict__ mirror, TA* __restrict__ c_v) {
  const int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int64_t u = t / 12;
  if (u >= nu) return;
  const int v0 = static_cast<int>(t - u * 12) * 3;
  TA acc[3] = {TA(0), TA(0), TA(0)};
  const int s1 = seg[u + 1];
  constexpr int kU = 4;
  for (int s = seg[u]; s < s1; s += kU) {
    TA x[kU][3];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const TA* p = partial + static_cast<size_t>(perm[min(s + k, s1 - 1)]) * 36 + v0;
#pragma unroll
      for (int c = 0; c < 3; ++c) x[k][c] = p[c];
    }
#pragma unroll
    for (int k = 0; k < kU; ++k)
      if (s + k < s1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] += x[k][c];
      }
  }
  TA* o = c_v + static_cast<size_t>(up_idx[u]) * 36 + v0;
#pragma unroll
  for (int c = 0; c < 3; ++c) o[c] = acc[c];
  const int m = mirror[u];
  if (m >= 0) {
    TA* o2 = c_v + static_cast<size_t>(m) * 36;
#pragma unroll
    for (int c = 0; c < 3; ++c) o2[((v0 + c) % 6) * 6 + (v0 + c) / 6] = acc[c];
  }
}

// out[0..n] = exclusive sums of in.  tmp grows as needed.
void scan32(const int32_t* in, int32_t* out, int n, DevBuf<char>& tmp, hipStream_t s) {
  size_t bytes = 0;
  HIP_CHECK(hipMemsetAsync(out, 0, sizeof(int32_t), s));
  HIP_CHECK(hipcub::DeviceScan::InclusiveSum(nullptr, bytes, in, out + 1, n, s));
  if (tmp.n < bytes) tmp.alloc(bytes);
  HIP_CHECK(hipcub::DeviceScan::InclusiveSum(tmp.p, bytes, in, out + 1, n, s));
}

// *out += the sum of n values, in 64 bits
__global__ __launch_bounds__(256) void sum64_kernel(int n, const int32_t* __restrict__ in,
                                                    unsigned long long* __restrict__ out) {
  unsigned long long v = 0;
  for (int64_t i = blockIdx.x * 256 + static_cast<int>(threadIdx.x); i < n; i += gridDim.x * 256)
    v += static_cast<unsigned long long>(in[i]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(out, v);
}

// *out = the sum of n sizes whose offsets scan32 may not hold; read as two of fetch's values (to64)
void sum64(const int32_t* in, int n, unsigned long long* out, hipStream_t s) {
  HIP_CHECK(hipMemsetAsync(out, 0, sizeof(*out), s));
  if (n > 0) sum64_kernel<<<std::min((n + 255) / 256, 512), 256, 0, s>>>(n, in, out);
  HIP_CHECK(hipGetLastError());
}
int64_t to64(int32_t lo, int32_t hi) {
  return static_cast<int64_t>(static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32 | static_cast<uint32_t>(lo));
}

constexpr int kFetch = 8;
struct Places {
  const int32_t* p[kFetch];
};
__global__ void fetch_kernel(Places f, int32_t* __restrict__ out) {
  if (threadIdx.x < kFetch && f.p[threadIdx.x]) out[threadIdx.x] = *f.p[threadIdx.x];
}
// the values at up to kFetch places, with one copy and one wait
std::array<int32_t, kFetch> fetch(const Places& f, int32_t* out, hipStream_t s) {
  std::array<int32_t, kFetch> h{};
  fetch_kernel<<<1, 64, 0, s>>>(f, out);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipMemcpyAsync(h.data(), out, sizeof(h), hipMemcpyDeviceToHost, s));
  HIP_CHECK(hipStreamSynchronize(s));
  return h;
}

template <class TX, class TP, class TA>
void launch_brick(const PtapPlan& pl, const bsr_s* A, const bsr_s* P, bsr_s* C, hipStream_t s) {
  const BrickPlan& k = pl.brick;
  const BrickArgs g{k.ng, k.a_cap, k.p_cap, reinterpret_cast<const int4*>(k.brick.p),
                    reinterpret_cast<const int4*>(k.batch.p), k.a_off.p, k.a_first.p, k.chunk_off.p,
                    reinterpret_cast<const int2*>(k.pieces.p), k.ell.p, k.codes.p, k.count.p, k.slot_ap.p,
                    k.slot_beg.p, k.slot_end.p};
  TA* part = reinterpret_cast<TA*>(k.partial.p);
  brick_kernel<TX, TP, TA><<<k.ng, kThreads, brick_lds<TX, TA>(k.a_cap, k.p_cap), s>>>(
      g, static_cast<const TX*>(A->val), static_cast<const TP*>(P->val),
      k.keep_ap ? reinterpret_cast<TA*>(pl.ap_val.p) : nullptr, part);
  HIP_CHECK(hipGetLastError());
  const int64_t nu = pl.c_nslots;
  brick_sum_kernel<TA><<<static_cast<int>((nu * 12 + 255) / 256), 256, 0, s>>>(
      nu, k.sum_seg.p, k.sum_perm.p, part, pl.c_up_idx.p, pl.c_mirror.p, static_cast<TA*>(C->val));
  HIP_CHECK(hipGetLastError());
}

}  // namespace

void brick_numeric(const PtapPlan& pl, const bsr_s* A, const bsr_s* P, bsr_s* C, hipStream_t s) {
  if (A->dtype == BLKAMG_F64) launch_brick<double, double, double>(pl, A, P, C, s);
  else if (P->dtype == BLKAMG_F32) launch_brick<float, float, float>(pl, A, P, C, s);
  else launch_brick<float, bf16, float>(pl, A, P, C, s);
}

bool brick_symbolic(const bsr_s* A, const bsr_s* P, const bsr_s* C, PtapPlan& pl, bool keep_ap, hipStream_t s) {
  BrickPlan& k = pl.brick;
  const int n = A->nbr;
  if (!pl.sym || A->br != 3 || n == 0 || pl.ap_nslots == 0 || pl.c_nslots == 0 || !pl.ap_pairs.width) return false;
  const size_t acc = A->dtype == BLKAMG_F64 ? 8 : 4;
  const Patterns t{n, P->nbc, keep_ap ? 1 : 0, A->rowptr, A->colidx, P->rowptr, P->colidx, pl.ap_rowptr.p,
                   pl.ap_colidx.p};
  const int gn = (n + 255) / 256;
  // A entries of a batch: 18 KB of LDS, nine rows of 27 blocks in FP64
  k.a_cap = acc == 8 ? 250 : 500;
  const int ap_cap = kQuads;
  k.keep_ap = keep_ap;
  // one allocation for the arrays of a value per row that only this function reads
  const size_t each = (static_cast<size_t>(n) + 64) / 64 * 64;
  DevBuf<int32_t> work(each * 16);
  int taken = 0;
  auto take = [&]() { return work.p + each * taken++; };
  int32_t *rows = take(), *first = take(), *need_s = take(), *alen_s = take(), *cand_s = take(), *head = take();
  int32_t *need_off = take(), *cand_off = take();
  DevBuf<unsigned long long> total_d(3);
  unsigned long long* const sum_d = total_d.p + 2;
  const int32_t* const sum_w = reinterpret_cast<const int32_t*>(sum_d);
  DevBuf<int> bad(3 + kFetch);  // bad, cut, most blocks of a batch; what fetch reads
  int* const cut = bad.p + 1;
  int* const got = bad.p + 3;
  HIP_CHECK(hipMemsetAsync(total_d.p, 0, total_d.bytes(), s));
  HIP_CHECK(hipMemsetAsync(bad.p, 0, bad.bytes(), s));
  unsigned long long total[2] = {0, 0};
  DevBuf<char> tmp;
  const int spare = taken;
  {
    uint32_t *key = reinterpret_cast<uint32_t*>(take()), *key_s = reinterpret_cast<uint32_t*>(take());
    int32_t *iota = take(), *first_r = take(), *need_r = take(), *cand_r = take();
    brick_rows_kernel<<<gn, 256, 0, s>>>(t, key, iota, first_r, need_r, cand_r);
    HIP_CHECK(hipGetLastError());
    int bits = 1;
    while ((int64_t{1} << bits) <= P->nbc) ++bits;
    size_t bytes = 0;
    HIP_CHECK(hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, key, key_s, iota, rows, n, 0, bits, s));
    tmp.alloc(std::max<size_t>(bytes, 1));
    HIP_CHECK(hipcub::DeviceRadixSort::SortPairs(tmp.p, bytes, key, key_s, iota, rows, n, 0, bits, s));
    brick_gather_kernel<<<gn, 256, 0, s>>>(t, key_s, rows, first_r, need_r, cand_r, first, need_s, alen_s, cand_s,
                                           head, total_d.p);
    HIP_CHECK(hipGetLastError());
    HIP_CHECK(hipMemcpyAsync(total, total_d.p, sizeof(total), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
  }
  taken = spare;
  const int used = static_cast<int>(total[0]);
  if (used == 0 || total[1] > INT32_MAX) return false;
  k.a_off.alloc(static_cast<size_t>(used) + 1);
  const int gu = (used + 255) / 256;
  int32_t *ghead = take(), *bhead = take(), *gid = take(), *bid = take();
  int32_t *pos_pieces = take(), *pos_blocks = take(), *pos_end = take();
  uint16_t* own = reinterpret_cast<uint16_t*>(take());
  HIP_CHECK(hipMemsetAsync(pos_end, 0, sizeof(int32_t) * used, s));
  brick_split_kernel<<<gu, 256, 0, s>>>(used, k.a_cap, ap_cap, head, need_s, alen_s, cand_s, ghead, bhead, bad.p);
  HIP_CHECK(hipGetLastError());
  scan32(need_s, need_off, used, tmp, s);
  scan32(alen_s, k.a_off.p, used, tmp, s);
  scan32(cand_s, cand_off, used, tmp, s);
  scan32(ghead, gid, used, tmp, s);
  scan32(bhead, bid, used, tmp, s);
  const auto h0 = fetch({bad.p, need_off + used, k.a_off.p + used, cand_off + used, gid + used, bid + used}, got, s);
  if (h0[0]) return false;
  const int64_t n_need = h0[1], n_a = h0[2], n_cand = h0[3];
  k.ng = h0[4];
  int nb = h0[5];
  DevBuf<int32_t> n_pieces, n_chunks, batch_row, group_row, group_batch, piece_ptr, batch_chunk, slot_ptr;
  group_row.alloc(static_cast<size_t>(k.ng) + 1);
  group_batch.alloc(static_cast<size_t>(k.ng) + 1);
  // batches whose rows of P fit LDS and the waves' registers: cut in two until they do
  k.p_cap = static_cast<int>(kLdsP / (kBlk * acc));
  int64_t total_pieces = 0, chunks = 0;
  for (int round = 0;; ++round) {
    batch_row.alloc(static_cast<size_t>(nb) + 1);
    brick_ptr_kernel<<<gu, 256, 0, s>>>(used, ghead, bhead, gid + 1, bid + 1, group_row.p, batch_row.p,
                                        group_batch.p);
    HIP_CHECK(hipMemsetAsync(cut, 0, 2 * sizeof(int), s));
    brick_stage_kernel<true><<<nb, 256, 0, s>>>(t, batch_row.p, rows, k.a_off.p, pos_pieces, pos_blocks,
                                                pos_end, nullptr, nullptr, nullptr, nullptr);
    brick_cut_kernel<<<(nb + 255) / 256, 256, 0, s>>>(nb, k.p_cap, batch_row.p, pos_blocks, pos_pieces, bhead,
                                                      cut, bad.p);
    HIP_CHECK(hipGetLastError());
    // the next round's batches, and the sizes if this one was the last
    scan32(bhead, bid, used, tmp, s);
    n_pieces.alloc(nb);
    n_chunks.alloc(nb);
    piece_ptr.alloc(static_cast<size_t>(nb) + 1);
    batch_chunk.alloc(static_cast<size_t>(nb) + 1);
    brick_sizes_kernel<<<(nb + 255) / 256, 256, 0, s>>>(nb, batch_row.p, pos_pieces, pos_blocks, need_off,
                                                        n_pieces.p, n_chunks.p, cut + 1);
    HIP_CHECK(hipGetLastError());
    scan32(n_pieces.p, piece_ptr.p, nb, tmp, s);
    scan32(n_chunks.p, batch_chunk.p, nb, tmp, s);
    sum64(n_pieces.p, nb, sum_d, s);
    const auto h = fetch({bad.p, cut, cut + 1, batch_chunk.p + nb, bid + used, sum_w, sum_w + 1}, got, s);
    if (h[0]) return false;
    if (!h[1]) {
      k.p_cap = std::max(h[2], 1);
      chunks = h[3];
      total_pieces = to64(h[5], h[6]);
      break;
    }
    if (round == 8) return false;
    nb = h[4];
  }
  if (total_pieces == 0 || total_pieces > INT32_MAX) return false;
  k.pieces.alloc(static_cast<size_t>(total_pieces) * 2);
  DevBuf<uint16_t> pofs(n_a);
  brick_stage_kernel<false><<<nb, 256, 0, s>>>(t, batch_row.p, rows, k.a_off.p, nullptr, nullptr, nullptr,
                                               piece_ptr.p, reinterpret_cast<int2*>(k.pieces.p), pofs.p, own);
  HIP_CHECK(hipGetLastError());
  // code tables of the batches' A P blocks
  DevBuf<uint8_t> rank_of(std::max<int64_t>(n_need, 1));
  const PairList& pr = pl.ap_pairs;
  k.chunk_off.alloc(static_cast<size_t>(chunks) + 1);
  DevBuf<int32_t> chunk_len(std::max<int64_t>(chunks, 1));
  if (keep_ap) k.slot_ap.alloc(std::max<int64_t>(n_need, 1));
  k.count.alloc(std::max<int64_t>(n_need, 1));
  auto order = [&](auto len, auto code) {
    brick_order_kernel<decltype(len)::value, decltype(code)><<<nb, kQuads, 0, s>>>(
        batch_row.p, need_off, k.a_off.p, first, pr.ptr.p, reinterpret_cast<const decltype(code)*>(pr.codes.p),
        pr.shift, pofs.p, rank_of.p, batch_chunk.p, chunk_len.p, k.chunk_off.p, k.ell.p, k.count.p, k.slot_ap.p);
    HIP_CHECK(hipGetLastError());
  };
  order(std::true_type{}, uint8_t{});
  // a chunk is padded to 16 times its longest list, so the tables can outgrow the pair list
  // (rows of many A blocks and few A P blocks) and 32 bits
  scan32(chunk_len.p, k.chunk_off.p, static_cast<int>(chunks), tmp, s);
  sum64(chunk_len.p, static_cast<int>(chunks), sum_d, s);
  const auto h1 = fetch({sum_w, sum_w + 1}, got, s);
  const int64_t n_ell = to64(h1[0], h1[1]);
  if (n_ell > INT32_MAX) return false;
  k.ell.alloc(std::max<int64_t>(n_ell, 1));
  if (pr.width == 1) order(std::false_type{}, uint8_t{});
  else if (pr.width == 2) order(std::false_type{}, uint16_t{});
  else order(std::false_type{}, uint32_t{});
  // coarse blocks of every brick
  DevBuf<int32_t> n_out(k.ng);
  DevBuf<int2> out(static_cast<size_t>(k.ng) * ap_cap);
  k.codes.alloc(std::max<int64_t>(n_cand, 1));
  brick_outputs_kernel<<<k.ng, 256, 0, s>>>(t, ap_cap, group_row.p, rows, first, cand_off, need_off,
                                            own, rank_of.p, C->rowptr, C->colidx, pl.c_up_rp.p, n_out.p, out.p,
                                            k.codes.p, bad.p);
  HIP_CHECK(hipGetLastError());
  slot_ptr.alloc(static_cast<size_t>(k.ng) + 1);
  scan32(n_out.p, slot_ptr.p, k.ng, tmp, s);
  const auto h2 = fetch({bad.p, slot_ptr.p + k.ng}, got, s);
  if (h2[0]) return false;
  const int64_t n_slots = h2[1];
  // a partial sum is written and read (2 x 36 values) where the two passes read an 18-value
  // A P block per contribution: with fewer than four contributions a partial sum there is
  // nothing to gain
  if (n_slots == 0 || n_slots * 4 > n_cand) return false;
  DevBuf<int32_t> slot_u(n_slots), slot_s(n_slots), iota(n_slots);
  k.slot_beg.alloc(n_slots);
  k.slot_end.alloc(n_slots);
  static_assert(kQuads <= 256);
  brick_slots_kernel<<<k.ng, 256, 0, s>>>(ap_cap, group_row.p, cand_off, slot_ptr.p, out.p, slot_u.p, iota.p,
                                          k.slot_beg.p, k.slot_end.p);
  HIP_CHECK(hipGetLastError());
  // partial sums of every coarse block, bricks in order
  const int ns = static_cast<int>(n_slots), nu = static_cast<int>(pl.c_nslots);
  k.sum_perm.alloc(n_slots);
  k.sum_seg.alloc(static_cast<size_t>(nu) + 1);
  int bits = 1;
  while ((int64_t{1} << bits) <= nu) ++bits;
  size_t bytes = 0;
  HIP_CHECK(hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, slot_u.p, slot_s.p, iota.p, k.sum_perm.p, ns, 0, bits, s));
  if (tmp.n < bytes) tmp.alloc(bytes);
  HIP_CHECK(hipcub::DeviceRadixSort::SortPairs(tmp.p, bytes, slot_u.p, slot_s.p, iota.p, k.sum_perm.p, ns, 0, bits, s));
  brick_seg_kernel<<<(nu + 1 + 255) / 256, 256, 0, s>>>(nu, ns, slot_s.p, k.sum_seg.p);
  HIP_CHECK(hipGetLastError());
  k.brick.alloc((static_cast<size_t>(k.ng) + 1) * 4);
  k.batch.alloc((static_cast<size_t>(nb) + 1) * 4);
  k.a_first.alloc(used);
  brick_desc_kernel<<<(std::max(used, nb + 1) + 255) / 256, 256, 0, s>>>(
      k.ng, nb, used, group_row.p, group_batch.p, slot_ptr.p, cand_off, batch_row.p, need_off, piece_ptr.p,
      batch_chunk.p, rows, A->rowptr, reinterpret_cast<int4*>(k.brick.p), reinterpret_cast<int4*>(k.batch.p),
      k.a_first.p);
  HIP_CHECK(hipGetLastError());
  k.partial.alloc(static_cast<size_t>(n_slots) * 36 * acc);
  HIP_CHECK(hipStreamSynchronize(s));
  k.n_codes = n_cand;
  k.on = true;
  return true;
}

}  // namespace blk
