// Type-1 spreading (steps 1 and 2a of section 4.2): c_{k,i} = w_k(x_i) x_i (eq:c)
// spread onto the fine grids with the exponential-of-semicircle window.
//
// Owner-computes on sub-tiles of 64 cells (64 in 1-D, 8^2 in 2-D, 4^3 in 3-D)
// with one wavefront per sub-tile and one cell per lane.  The points whose
// window reaches a sub-tile are listed once per plan (in the order the sorted
// points are visited), so a matvec streams exactly the contributing points of
// each sub-tile.  Every cell is summed in a fixed order: the list four points at a
// time, added by one matrix instruction in fp64, while fp32 keeps four sums, of every
// fourth point each, that are joined at the end (the result is bitwise reproducible;
// no atomics, no zero-fill pass, plain stores).
#include <algorithm>
#include <limits>

#include "gp_internal.h"

namespace gp {
namespace {

template <typename T> struct V2;
template <> struct V2<double> { using type = double2; };
template <> struct V2<float> { using type = float2; };

constexpr int kSubThreads = 64;  // one wavefront per sub-tile
constexpr int kGCmax = 8;        // grid pairs per wavefront
constexpr int kSpreadBatch = 16;  // points per batch of the spreading
// A launch has fewer than 2^32 threads: one wavefront per sub-tile reaches that at
// 6.7e7 sub-tiles (3-D grids of 1625^3 cells on); launches take 2^31 threads each.
constexpr int64_t kSliceBlocks = ((int64_t)1 << 31) / kSubThreads;

// Sub-tile blk = bin * nsub + sub (sub-tiles of a bin consecutive, first
// dimension fastest): its first cell s0 and its bin's coordinates tcoord.  32-bit
// arithmetic (there are fewer than 2^30 sub-tiles): 64-bit divisions took a third
// of the time of a wavefront with few points.
__device__ __forceinline__ void sub_tile_origin(const NuArgs& a, int D, int st, unsigned blk,
                                                int* s0, int* tcoord) {
  unsigned nsub = 1;
  for (int r = 0; r < D; ++r) nsub *= (unsigned)(a.tile[r] / st);  // st divides every tile side
  unsigned tb = blk / nsub, sub = blk - tb * nsub;
  for (int r = 0; r < 3; ++r) {
    s0[r] = 0;
    tcoord[r] = 0;
  }
  for (int r = 0; r < D; ++r) {
    const unsigned per = (unsigned)(a.tile[r] / st), nb = (unsigned)a.nbins[r];
    const unsigned tq = tb / nb, sq = sub / per;
    tcoord[r] = (int)(tb - tq * nb);
    s0[r] = tcoord[r] * a.tile[r] + (int)(sub - sq * per) * st;
    tb = tq;
    sub = sq;
  }
}

// Workgroups go to the 8 XCDs round-robin by id.  Sub-tiles are dealt to the
// XCDs in groups of `grp` consecutive ones (the sub-tiles of the bins that
// share cache lines of grid rows), so each group is written through one L2,
// while the groups still alternate between XCDs (clustered points keep every
// XCD equally busy).  The grid is padded to a multiple of 8 grp workgroups;
// the map is a bijection onto [0, gridDim.x) and ids >= the sub-tile count
// have no work.
__device__ __forceinline__ unsigned xcd_grouped(unsigned bid, unsigned grp) {
  const unsigned x = bid % 8, k = bid / 8, q = k / grp;
  return (q * 8 + x) * grp + (k - q * grp);
}

// Plan time, one wavefront per sub-tile: walk the concatenated source bins
// (the tile's bin and its lower neighbours within w-1 cells, first dimension
// fastest, without the bins none of whose points reach this sub-tile: along
// dimension r the points of the bin dq >= 1 tiles below start at most at
// t0 - (dq - 1) tile - 1, so their windows end before s0 when that
// start + w - 1 < s0), keep the points whose window reaches the sub-tile in
// every dimension, and either count them (FILL = false) or write them at
// list[off[blk] ..] in visiting order (FILL = true): {sorted index, first
// window cell relative to s0 - (w - 1), 8 bits per dimension}.
template <int D, bool FILL>
__global__ __launch_bounds__(kSubThreads) void spread_list_build_kernel(
    NuArgs a, int st, int64_t blk0, const int* __restrict__ cell, const int* __restrict__ bin_start,
    int* __restrict__ cnt, const int64_t* __restrict__ off, int2* __restrict__ list) {
  extern __shared__ int ismem[];
  const int64_t blk = blk0 + blockIdx.x;
  int s0[3], tcoord[3];
  sub_tile_origin(a, D, st, blk, s0, tcoord);
  const int w = a.w;
  int nsrc_tot = 1;
  for (int r = 0; r < D; ++r) nsrc_tot *= a.nsrc;
  int* s_sb0 = ismem;              // [nsrc_tot]
  int* s_soff = s_sb0 + nsrc_tot;  // [nsrc_tot + 1]
  for (int sb = threadIdx.x; sb < nsrc_tot; sb += kSubThreads) {
    int64_t b = 0, mul = 1;
    bool ok = true;
    int q = sb;
    for (int r = 0; r < D; ++r) {
      const int dq = q % a.nsrc;
      const int br = tcoord[r] - dq;
      q /= a.nsrc;
      if (br < 0) ok = false;
      if (dq > 0 && tcoord[r] * a.tile[r] - (dq - 1) * a.tile[r] - 1 + w - 1 < s0[r]) ok = false;
      b += (int64_t)br * mul;
      mul *= a.nbins[r];
    }
    const int b0 = ok ? bin_start[b] : 0;
    s_sb0[sb] = b0;
    s_soff[sb + 1] = ok ? bin_start[b + 1] - b0 : 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s_soff[0] = 0;
    for (int sb = 0; sb < nsrc_tot; ++sb) s_soff[sb + 1] += s_soff[sb];
  }
  __syncthreads();
  const int seq_hi = s_soff[nsrc_tot];
  int64_t count = 0;
  const int64_t o = FILL ? off[blk] : 0;
  for (int base = 0; base < seq_hi; base += kSubThreads) {
    const int qpos = base + (int)threadIdx.x;
    bool keep = qpos < seq_hi;
    int idx = 0, cw = 0;
    if (keep) {
      int sb = 0;
      while (qpos >= s_soff[sb + 1]) ++sb;
      idx = s_sb0[sb] + (qpos - s_soff[sb]);
      int cr[3];
      for (int r = 0; r < D; ++r) cr[r] = cell[r * a.n + idx];
      for (int r = 0; r < D; ++r) {
        keep = keep & (cr[r] + w - 1 >= s0[r]) & (cr[r] < s0[r] + st);
        cw |= (cr[r] - s0[r] + w - 1) << (8 * r);
      }
    }
    const unsigned long long m = __ballot(keep);
    if (FILL && keep) list[o + count + __popcll(m & ((1ull << threadIdx.x) - 1ull))] = int2{idx, cw};
    count += __popcll(m);
  }
  if (!FILL && threadIdx.x == 0) cnt[blk] = (int)count;
}

// v of lane k, in scalar registers
__device__ __forceinline__ int64_t lane_value(int64_t v, int k) {
  const unsigned a = __builtin_amdgcn_readlane((int)v, k), b = __builtin_amdgcn_readlane((int)(v >> 32), k);
  return (int64_t)((uint64_t)b << 32 | a);
}

using d4 = __attribute__((ext_vector_type(4))) double;
using f4 = __attribute__((ext_vector_type(4))) float;

// A lane's element of the 4-point product that adds to 16 cells: cells along the
// columns, weights along the rows, see spread_list_kernel.
template <int NM>
struct Acc64 {
  d4 c[4];
  __device__ __forceinline__ void zero() {
    for (int j = 0; j < 4; ++j) c[j] = d4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void add(int j, double wk, double v) {
    c[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(wk, v, c[j], 0, 0, 0);
  }
};
template <int NM>
struct Acc32 {
  f4 c[4][NM];
  __device__ __forceinline__ void zero() {
    for (int j = 0; j < 4; ++j)
      for (int s = 0; s < NM; ++s) c[j][s] = f4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void add(int j, float wk, float v) {
    c[j][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(wk, v, c[j][0], 2, 0, 0);
    if constexpr (NM > 1) c[j][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(wk, v, c[j][1], 2, 1, 0);
    if constexpr (NM > 2) c[j][2] = __builtin_amdgcn_mfma_f32_4x4x1f32(wk, v, c[j][2], 2, 2, 0);
    if constexpr (NM > 3) c[j][3] = __builtin_amdgcn_mfma_f32_4x4x1f32(wk, v, c[j][3], 2, 3, 0);
  }
};
template <typename T, int NM> struct AccOf;
template <int NM> struct AccOf<double, NM> { using type = Acc64<NM>; };
template <int NM> struct AccOf<float, NM> { using type = Acc32<NM>; };

// One wavefront per item: a sub-tile (or a chunk of its list, summed into
// partial tile `slot`), gc <= 8 grid pairs.  Spreading is a product per sub-tile,
//   cells x weights += (window values, cells x points) (w_k, points x weights),
// done by matrix instructions on four points at a time.  Lane l = 16 q + n holds,
// of point q of the four, weight n (one operand) and the window value of cell
// 16 j + n for j = 0..3 (the other).
//  fp64: 16x16x4, which sums over the four points; operand row i of the weights
//        is weight 4 (i % 4) + i / 4, so that the result's four values of lane
//        (n, q), rows q + 4 r, are the weights 4 q + r of its cell.
//  fp32: 4x4x1 in 16 blocks, the four blocks of point q taking the weights
//        4 s..4 s + 3 of that point (broadcast within the four); 8 weights take
//        half the time of the 16-row form.  The four points' sums are added at
//        the end.
// The 16 lanes of a point load its row (its windows 16 values at a time, its
// weights as the matrix operand they are), one batch ahead.  The windows go
// through LDS, with st - 1 zeros on both sides in d >= 2 so that a cell outside
// the window reads zero without a test; the values along the dimensions that do
// not change with j serve all 64 cells.
// A wavefront does `per` consecutive sub-tiles (one item where lists are split):
// their lists follow each other in memory, so the batch that is fetched ahead
// may be the next sub-tile's.
//
// Before, fp64 tiles of 16^2 cells read every weight from LDS for every cell (the
// bound: 64 lanes' copies of 14 doubles per point and wavefront) and tested every
// point of the source bins, and fp32 lists staged zero-padded windows per point.
// ms per launch, before -> now: d=2 N=1e6 fp64 0.777 -> 0.544 (the grids written
// take 0.27), N=1e5 0.119 -> 0.076, 16 vectors at N=1e5 1.95 -> 0.97, fp32 N=1e6
// 0.242 -> 0.229, d=3 N=1e7 fp32 3.38 -> 2.93, d=1 N=2000 fp64 0.017 -> 0.006, N=1.6e5
// fp32 0.045 -> 0.014; d=3 N=2e5 fp64 (9 points per sub-tile) 0.71 -> 0.77.  What
// bounds it now, per batch of 16 points and CU at d=3 fp32: address and window
// arithmetic 125 cycles, LDS 145, loads 100, matrix 64, in 330.
template <typename T, int D, int NM, int KW, bool FULL, typename Off>
__global__ __launch_bounds__(kSubThreads, NM > 2 || (sizeof(T) == 8 && KW > 2) ? 3 : (sizeof(T) == 4 && KW == 1 ? 5 : 4)) void spread_list_kernel(
    NuArgs a, int lg_, int grp, unsigned bid0, unsigned nitems, int per, int64_t set_stride, const double* __restrict__ x,
    const T* __restrict__ pw, int rs, const int64_t* __restrict__ off, const int2* __restrict__ list,
    const int4* __restrict__ items, typename V2<T>::type* __restrict__ part,
    typename V2<T>::type* __restrict__ grid) {
  using V = typename V2<T>::type;
  constexpr int NU = kSpreadBatch / 4;                // groups of four points per batch
  constexpr int LGF = D == 1 ? 6 : (D == 2 ? 3 : 2);  // the side of a full sub-tile of 64 cells
  constexpr bool PAD = D > 1;
  extern __shared__ __align__(16) unsigned char smem[];
  T* s_win = reinterpret_cast<T*>(smem);  // [kSpreadBatch][S]
  const int set = blockIdx.z;
  // the last chunk of grid pairs overlaps the one before when gc does not divide
  // their number (both write the same values)
  const int g0 = min((int)blockIdx.y * a.gc, a.npair - a.gc);
  const int lane = threadIdx.x, n = lane & 15, q = lane >> 4;
  unsigned blk = xcd_grouped(bid0 + blockIdx.x, (unsigned)grp), nsub = 1;
  int slot = -1;
  int64_t lo, hi;
  int64_t ends = 0;  // lane k: end of the list of sub-tile blk + k
  if (items) {  // {sub-tile, first, last + 1 (positions in its list), slot}
    if (blk >= nitems) return;
    const int4 wk = items[blk];
    blk = wk.x;
    slot = wk.w;
    lo = off[blk] + wk.y;
    hi = off[blk] + wk.z;
  } else {
    blk *= per;
    if (blk >= nitems) return;
    nsub = min((unsigned)per, nitems - blk);
    ends = off[blk + min((unsigned)lane + 1, nsub)];
    lo = off[blk];
    hi = lane_value(ends, 0);
  }
  const int lg = FULL ? LGF : lg_;
  const int st = 1 << lg, w = a.w, dw = D * w;
  const int PS = PAD ? w + 2 * (st - 1) : w;  // one dimension's window in LDS
  const int S = (D * PS) | 1;
  // coordinates of cell 16 j + n along each dimension; those that change with j
  // are the last dimension's in a full sub-tile (x in 1-D, y in 2-D, z in 3-D)
  auto coord = [&](int j, int r) {
    const int c = 16 * j + n;
    return D == 1 ? c : (c >> (r * lg)) & (st - 1);
  };
  // the lane's weight and window values of its point's row, and their places
  const int kw = sizeof(T) == 8 ? 4 * (n % 4) + n / 4 : n;
  const bool kin = kw < 2 * a.gc;
  const Off koff = (Off)(dw + 2 * g0 + (kin ? kw : 0));
  // window value 16 k + n of the row is at dst + 16 k + (its dimension) (PS - w)
  auto wdst = [&](int k) {
    const int c = 16 * k + n;
    return q * S + c + (PAD ? st - 1 + ((c >= w) + (D > 2 && c >= 2 * w)) * (PS - w) : 0);
  };
  x += (int64_t)set * a.n;
  typename AccOf<T, NM>::type acc;
  acc.zero();
  if (PAD) {  // the zeros beside the windows (16-byte stores; the buffer's size is a multiple)
    const int nz = (int)(kSpreadBatch * S * sizeof(T) + 15) / 16;
    for (int e = lane; e < nz; e += kSubThreads) reinterpret_cast<float4*>(smem)[e] = float4{0, 0, 0, 0};
    __syncthreads();
  }
  const int64_t end = items ? hi : lane_value(ends, (int)nsub - 1), last = end - 1;

  // store the sums of sub-tile b: lane (n, q) of fp64 has weights 4 q .. 4 q + 3
  // (pairs 2 q, 2 q + 1) of the cells 16 j + n; of fp32, after adding the points'
  // sums, all weights of the cell 16 q + n
  auto flush = [&](unsigned b) {
    const int cells = 1 << (D * lg);
    int s0[3], tcoord[3];
    sub_tile_origin(a, D, st, b, s0, tcoord);
    V* out = slot >= 0 ? part + ((int64_t)(set * a.n_slots + slot) * a.npair + g0) * cells
                       : grid + set * set_stride + (int64_t)g0 * a.pair_stride + a.grid_off +
                             (int64_t)s0[0] * a.gstride[0] + (int64_t)s0[1] * a.gstride[1] +
                             (int64_t)s0[2] * a.gstride[2];
    const int64_t gs = slot >= 0 ? cells : a.pair_stride;
    auto put = [&](int c, int g, V val) {
      if ((!FULL && c >= cells) || g >= a.gc) return;
      const int64_t at = slot >= 0 ? c
                                   : (int64_t)(D == 1 ? c : c & (st - 1)) +
                                         (D > 1 ? ((c >> lg) & (st - 1)) * a.gstride[1] : 0) +
                                         (D > 2 ? ((c >> (2 * lg)) & (st - 1)) * a.gstride[2] : 0);
      out[g * gs + at] = val;
    };
    if constexpr (sizeof(T) == 8) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        put(16 * j + n, 2 * q, V{acc.c[j][0], acc.c[j][1]});
        put(16 * j + n, 2 * q + 1, V{acc.c[j][2], acc.c[j][3]});
      }
    } else {
      // exchange and add: lanes of q >= 2 keep cells j = 2, 3, the others j = 0, 1;
      // then odd q keep the odd j
#pragma unroll
      for (int s = 0; s < NM; ++s) {
        f4 r;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float keep[2], send[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            keep[h] = q >= 2 ? acc.c[2 + h][s][k] : acc.c[h][s][k];
            send[h] = q >= 2 ? acc.c[h][s][k] : acc.c[2 + h][s][k];
            keep[h] += __shfl_xor(send[h], 32);
          }
          const float kp = (q & 1) ? keep[1] : keep[0], sd = (q & 1) ? keep[0] : keep[1];
          r[k] = kp + __shfl_xor(sd, 16);
        }
        put(16 * q + n, 2 * s, V{r[0], r[1]});
        put(16 * q + n, 2 * s + 1, V{r[2], r[3]});
      }
    }
    acc.zero();
  };

  int2 ent{0, 0}, nent{0, 0};
  T xn = T(0), rv[NU][KW], wk[NU];
  auto fetch = [&](const int2& e) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const Off row = (Off)__shfl(e.x, 4 * u + q) * (Off)rs;
#pragma unroll
      for (int k = 0; k < KW; ++k) rv[u][k] = pw[row + (Off)min(16 * k + n, dw - 1)];
      wk[u] = pw[row + koff];
    }
  };
  if (lo < end) {
    ent = list[min(lo + n, last)];
    xn = (T)x[ent.x];
    fetch(ent);
  }
  unsigned sub = 0;  // current sub-tile blk + sub, its list ends at hi
  int64_t base = lo;
  while (true) {
    while (base >= hi) {  // finished, and empty ones
      flush(blk + sub);
      if (++sub == nsub) return;
      hi = lane_value(ends, (int)sub);
    }
    // the batch: positions base .. nbase of the current list
    const int64_t nbase = min(base + kSpreadBatch, hi);
    nent = list[min(nbase + n, last)];  // the batch after it
    T wx[NU];
    int cw[NU];
    xn = base + n < hi ? xn : T(0);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
#pragma unroll
      for (int k = 0; k < KW; ++k)
        if (16 * k + n < dw) s_win[4 * u * S + wdst(k)] = rv[u][k];
      const T xq = __shfl(xn, 4 * u + q);  // by all lanes, also those without a weight
      wx[u] = kin ? wk[u] * xq : T(0);
      cw[u] = __shfl(ent.y, 4 * u + q);
    }
    __syncthreads();
    // the next batch is on its way while this one is added
    ent = nent;
    if (nbase < end) {
      xn = (T)x[ent.x];
      fetch(ent);
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if (sizeof(T) == 8 && base + 4 * u >= hi) break;  // groups past the end (fp32: 0.23 -> 0.26 ms)
      const T* row = s_win + (4 * u + q) * S;
      // window place of coordinate 0 along each dimension
      const int b0 = w - 1 - (cw[u] & 255), b1 = w - 1 - ((cw[u] >> 8) & 255), b2 = w - 1 - ((cw[u] >> 16) & 255);
      T v[4];
      if constexpr (D == 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int p = coord(j, 0) + b0;
          const bool in = (unsigned)p < (unsigned)w;
          const T t = row[in ? p : 0];
          v[j] = in ? t : T(0);
        }
      } else {
        const T* w0 = row + st - 1 + b0;
        const T* w1 = row + PS + st - 1 + b1;
        const T* w2 = row + 2 * PS + st - 1 + b2;
        if (FULL) {
          if constexpr (D == 2) {
            const T p0 = w0[coord(0, 0)];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = p0 * w1[coord(0, 1) + 2 * j];
          } else {
            const T p01 = w0[coord(0, 0)] * w1[coord(0, 1)];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = p01 * w2[j];
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[j] = w0[coord(j, 0)] * w1[coord(j, 1)];
            if (D > 2) v[j] *= w2[coord(j, 2)];
          }
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) acc.add(j, wx[u], v[j]);
    }
    __syncthreads();  // the windows are overwritten next
    base = nbase;
  }
}

// Sub-tiles split into chunks: their cells are the sums of the chunks' partial
// tiles, added in list order.  One workgroup per split sub-tile {sub-tile,
// first slot, chunks}.
template <typename T, int D>
__global__ __launch_bounds__(256) void spread_reduce_kernel(
    NuArgs a, int lg, int64_t set_stride, const int4* __restrict__ red,
    const typename V2<T>::type* __restrict__ part, typename V2<T>::type* __restrict__ grid) {
  using V = typename V2<T>::type;
  const int4 wk = red[blockIdx.x];
  const int set = blockIdx.z, st = 1 << lg, cells = 1 << (D * lg);
  int s0[3], tcoord[3];
  sub_tile_origin(a, D, st, wk.x, s0, tcoord);
  for (int e = threadIdx.x; e < a.npair * cells; e += 256) {
    const int g = e / cells, t = e % cells;
    V v = V{T(0), T(0)};
    for (int j = 0; j < wk.z; ++j) {
      const V u = part[((int64_t)(set * a.n_slots + wk.y + j) * a.npair + g) * cells + t];
      v.x += u.x;
      v.y += u.y;
    }
    const int64_t gi = set * set_stride + a.grid_off + (int64_t)(s0[0] + (t & (st - 1))) * a.gstride[0] +
                       (int64_t)(s0[1] + (D > 1 ? (t >> lg) & (st - 1) : 0)) * a.gstride[1] +
                       (int64_t)(s0[2] + (D > 2 ? t >> (2 * lg) : 0)) * a.gstride[2];
    grid[(int64_t)g * a.pair_stride + gi] = v;
  }
}

// Work items of the spreading, where a list is longer than `chunk`: sub-tile b has
// nit(b) = max(1, ceil(cnt / chunk)) items (equal parts of its list), with a
// partial tile each when nit > 1.  FILL = false counts items, slots and split
// sub-tiles; FILL = true writes them at the scanned offsets.
template <bool FILL>
__global__ __launch_bounds__(256) void spread_items_kernel(
    int64_t nsub, int chunk, const int* __restrict__ cnt, int* __restrict__ nitem, int* __restrict__ nslot,
    int* __restrict__ nsplit, const int64_t* __restrict__ oitem, const int64_t* __restrict__ oslot,
    const int64_t* __restrict__ osplit, int4* __restrict__ items, int4* __restrict__ red) {
  const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (b >= nsub) return;
  const int c = cnt[b];
  const int k = c > chunk ? (c + chunk - 1) / chunk : 1;
  if (!FILL) {
    nitem[b] = k;
    nslot[b] = k > 1 ? k : 0;
    nsplit[b] = k > 1;
    return;
  }
  const int s0 = (int)oslot[b];
  for (int j = 0; j < k; ++j)
    items[oitem[b] + j] = int4{(int)b, (int)((int64_t)c * j / k), (int)((int64_t)c * (j + 1) / k),
                               k > 1 ? s0 + j : -1};
  if (k > 1) red[osplit[b]] = int4{(int)b, s0, k, 0};
}

__global__ __launch_bounds__(256) void max_count_kernel(int64_t n, const int* __restrict__ cnt,
                                                        int* __restrict__ out) {
  int m = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    m = max(m, cnt[i]);
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) atomicMax(out, m);
}

// ------------------------------------------------------------------ scan ----
// Exclusive prefix sum of counts into int64 offsets; 1024 elements per
// workgroup (4 per thread), the workgroup totals scanned the same way and
// added back.
constexpr int kScanThreads = 256, kScanPer = 4, kScanBlock = kScanThreads * kScanPer;
template <typename In>
__global__ __launch_bounds__(kScanThreads) void scan_block_kernel(const In* __restrict__ in, int64_t n,
                                                                  int64_t* __restrict__ out,
                                                                  int64_t* __restrict__ sums) {
  __shared__ int64_t s[kScanThreads];
  const int64_t b0 = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
  int64_t v[kScanPer], tsum = 0;
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = b0 + k < n ? (int64_t)in[b0 + k] : 0;
    tsum += v[k];
  }
  s[threadIdx.x] = tsum;
  __syncthreads();
  for (int d = 1; d < kScanThreads; d *= 2) {
    const int64_t add = (int)threadIdx.x >= d ? s[threadIdx.x - d] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  int64_t run = s[threadIdx.x] - tsum;  // exclusive prefix of this thread
  for (int k = 0; k < kScanPer; ++k) {
    if (b0 + k < n) out[b0 + k] = run;
    run += v[k];
  }
  if (threadIdx.x == kScanThreads - 1) sums[blockIdx.x] = s[threadIdx.x];
}
__global__ __launch_bounds__(kScanThreads) void scan_add_kernel(int64_t* __restrict__ out, int64_t n,
                                                                const int64_t* __restrict__ offs) {
  const int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x;
  if (i < n) out[i] += offs[i / kScanBlock];
}

// out[0..n) = exclusive prefix sums of in[0..n); *total = their sum (read back
// once at the end; plan time only).
template <typename In>
void exclusive_scan(const In* in, int64_t n, int64_t* out, hipStream_t s, int64_t* total) {
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  DevBuf sums, soff;
  sums.alloc((size_t)std::max<int64_t>(nb, 1) * sizeof(int64_t), s);
  if (n > 0) {
    hipLaunchKernelGGL((scan_block_kernel<In>), dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n,
                       out, sums.as<int64_t>());
    GP_CHECK_LAUNCH();
  }
  if (nb > 1) {
    soff.alloc((size_t)nb * sizeof(int64_t), s);
    int64_t sub_total = 0;
    exclusive_scan<int64_t>(sums.as<int64_t>(), nb, soff.as<int64_t>(), s, &sub_total);
    hipLaunchKernelGGL(scan_add_kernel, dim3((unsigned)((n + kScanThreads - 1) / kScanThreads)),
                       dim3(kScanThreads), 0, s, out, n, soff.as<int64_t>());
    GP_CHECK_LAUNCH();
    *total = sub_total;
    GP_HIP(hipStreamSynchronize(s));  // sums and soff are released on return
    return;
  }
  int64_t tv = 0;
  if (n > 0) GP_HIP(hipMemcpyAsync(&tv, sums.p, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  GP_HIP(hipStreamSynchronize(s));
  *total = tv;
}

template <typename T, int D>
void launch_sub(Plan* P, const Records& R, const double* xs, int nsets) {
  using V = typename V2<T>::type;
  PhaseScope ps(P, PH_SPREAD);
  NuArgs a = nu_args(P, R);
  a.n_slots = (int)R.n_slots;
  int lg = 0;
  while ((1 << lg) < R.sub_st) ++lg;
  // where lists are split, as many vectors at once as there are partial tiles for
  const int group = R.n_slots > 0 && nsets > 1 ? P->m_part : nsets;
  V* part = group > 1 ? P->mpart.as<V>() : R.part.as<V>();
  // equal chunks of grid pairs, at most kGCmax each
  const int nch = (P->npair + kGCmax - 1) / kGCmax;
  const int gc = (P->npair + nch - 1) / nch;
  // groups: the sub-tiles of one bin, or of two bins along dimension 0 in 3-D
  // (whose 8-cell rows of fp32 pairs are half a 128-byte line); longer groups gain
  // nothing or leave XCDs unevenly loaded (d=2 N=1e6 fp64, four rows of bins:
  // 0.55 -> 0.58 ms)
  int grp = 1;
  for (int r = 0; r < D; ++r) grp *= P->tile[r] / R.sub_st;
  if (D == 3 && P->nbins[0] % 2 == 0) grp *= 2;
  const bool split = R.n_sp_work > 0;
  const int64_t ni = split ? R.n_sp_work : R.n_sub;
  // four sub-tiles per wavefront where most have no or few points (a wavefront's
  // start then costs more than its points: d=2 N=2e4 fp32 0.110 -> 0.084 ms), as
  // long as thousands of wavefronts are left; else one (d=3 N=2e5 fp64 0.83 -> 0.77 ms)
  const int per = split || R.n_list >= 8 * R.n_sub || ni * nch * nsets < 4 * 4096 ? 1 : 4;
  grp = std::max(1, grp / per);
  const int64_t nw = (ni + per - 1) / per, nblk = (nw + 8 * grp - 1) / (8 * grp) * (8 * grp);
  const int64_t set_stride = (int64_t)P->npair * P->grid_elems[0];
  V* grid = static_cast<V*>(grid_a_current(P));
  a.gc = gc;
  // element offsets into the rows fit 32 bits (byte offsets 4 GiB) or not
  const bool big = (double)R.n * R.rs * sizeof(T) >= 4.0e9;
  const int win = D > 1 ? P->w + 2 * (R.sub_st - 1) : P->w;
  const size_t smem = ((size_t)kSpreadBatch * ((D * win) | 1) * sizeof(T) + 15) / 16 * 16;
  auto go = [&](auto kern) {
    for (int set = 0; set < nsets; set += group) {
      const unsigned ns = (unsigned)std::min(group, nsets - set);
      V* gset = grid + set * set_stride;
      for (int64_t b = 0; b < nblk; b += kSliceBlocks) {
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min(kSliceBlocks, nblk - b), nch, ns), dim3(kSubThreads),
                           smem, P->stream, a, lg, grp, (unsigned)b, (unsigned)ni, per, set_stride,
                           xs + set * R.n, R.pw.as<T>(), R.rs, R.sub_off.as<int64_t>(), R.sub_list.as<int2>(),
                           split ? R.sp_work.as<int4>() : nullptr, part, gset);
        GP_CHECK_LAUNCH();
      }
      if (R.n_sp_red > 0) {
        hipLaunchKernelGGL((spread_reduce_kernel<T, D>), dim3((unsigned)R.n_sp_red, 1, ns), dim3(256), 0,
                           P->stream, a, lg, set_stride, R.sp_red.as<int4>(), part, gset);
        GP_CHECK_LAUNCH();
      }
    }
  };
  // matrix instructions per 16 cells (fp32: 4 weights each) and loads of 16 window values
  const int nm = sizeof(T) == 8 ? 1 : (2 * gc + 3) / 4, kw = (D * P->w + 15) / 16;
  const bool full = (1 << (D * lg)) == kSubThreads;
#define GP_SUB_GO(N, K)                                                                                  \
  go(big    ? (full ? spread_list_kernel<T, D, N, K, true, int64_t> : spread_list_kernel<T, D, N, K, false, int64_t>) \
     : full ? spread_list_kernel<T, D, N, K, true, uint32_t>                                             \
            : spread_list_kernel<T, D, N, K, false, uint32_t>)
#define GP_SUB_KW(N)                                                        \
  do {                                                                      \
    if constexpr (D == 1) GP_SUB_GO(N, 1);                                  \
    else if constexpr (D == 2) { if (kw == 1) GP_SUB_GO(N, 1); else GP_SUB_GO(N, 2); } \
    else { if (kw == 1) GP_SUB_GO(N, 1); else if (kw == 2) GP_SUB_GO(N, 2); else GP_SUB_GO(N, 3); } \
  } while (0)
  if constexpr (sizeof(T) == 8) {
    GP_SUB_KW(1);
  } else {
    switch (nm) {
      case 1: GP_SUB_KW(1); break;
      case 2: GP_SUB_KW(2); break;
      case 3: GP_SUB_KW(3); break;
      default: GP_SUB_KW(4); break;
    }
  }
#undef GP_SUB_KW
#undef GP_SUB_GO
}

template <int D, bool FILL>
void launch_list_build(const NuArgs& a, int st, int64_t nsub, size_t smem, hipStream_t s, const Records& R,
                       int* cnt, const int64_t* off, int2* list) {
  for (int64_t b = 0; b < nsub; b += kSliceBlocks) {
    hipLaunchKernelGGL((spread_list_build_kernel<D, FILL>), dim3((unsigned)std::min(kSliceBlocks, nsub - b)),
                       dim3(kSubThreads), smem, s, a, st, b, R.cell.as<int>(), R.bin_start.as<int>(), cnt, off,
                       list);
    GP_CHECK_LAUNCH();
  }
}
template <bool FILL>
void list_build(int d, const NuArgs& a, int st, int64_t nsub, size_t smem, hipStream_t s, const Records& R,
                int* cnt, const int64_t* off, int2* list) {
  if (d == 1) launch_list_build<1, FILL>(a, st, nsub, smem, s, R, cnt, off, list);
  else if (d == 2) launch_list_build<2, FILL>(a, st, nsub, smem, s, R, cnt, off, list);
  else launch_list_build<3, FILL>(a, st, nsub, smem, s, R, cnt, off, list);
}

// Chunks of a list per work item: short enough that a launch has thousands of
// wavefronts where the points allow it, long enough that writing and adding a
// partial tile stays small beside the points.
constexpr int64_t kListItems = 8192, kMinListChunk = 128;
int64_t list_chunk(int64_t total) { return std::max(kMinListChunk, (total + kListItems - 1) / kListItems); }

}  // namespace

int spread_sub_side(const Plan* P) {
  if (P->spread_mode == GP_SPREAD_LDS_ATOMIC) return 0;
  if (P->lean && (P->d == 1 || P->precision == GP_FP64)) return 0;
  // 64 cells, at most a tile (tiles are powers of two)
  int st = P->d == 1 ? 64 : (P->d == 2 ? 8 : 4);
  for (int r = 0; r < P->d; ++r) st = std::min(st, P->tile[r]);
  return st;
}

size_t spread_list_bound_bytes(const Plan* P, int64_t n, bool split) {
  const int st = spread_sub_side(P);
  if (st == 0) return 0;
  int64_t per_point = 1, nsub = P->n_bins, cells = 1;
  for (int r = 0; r < P->d; ++r) {
    per_point *= (P->w - 2 + st) / st + 1;  // sub-tiles one window spans, at most
    nsub *= P->tile[r] / st;
    cells *= st;
  }
  const int64_t total = n * per_point, chunk = list_chunk(total);
  // items and split sub-tiles only where some list is longer than a chunk
  split = split && total > chunk;
  const int64_t slots = split ? std::min(2 * (total / chunk), total / chunk + nsub) : 0;
  const int64_t items = split ? nsub + slots : 0;
  const size_t cs = P->precision == GP_FP64 ? 16 : 8;
  return (size_t)total * sizeof(int2) + (size_t)(2 * nsub + 1) * sizeof(int64_t) +
         (size_t)(items + slots) * sizeof(int4) + (size_t)slots * cells * P->npair * cs;
}

size_t spread_partial_bytes(const Plan* P, const Records& R) {
  if (!spread_uses_sub_tiles(P)) return 0;
  size_t cells = 1;
  for (int r = 0; r < P->d; ++r) cells *= R.sub_st;
  return (size_t)R.n_slots * cells * P->npair * (P->precision == GP_FP64 ? 16 : 8);
}

// The exact source lists of sub-tile spreading, built on the device from the
// sorted points: count per sub-tile, scan, fill (both passes visit the points
// in the same order, so the lists and every later sum are deterministic); and
// the work items, where a list is long.
void build_spread_lists(Plan* P, Records& R) {
  R.n_sub = 0;
  const int st = spread_sub_side(P);
  if (st == 0) return;
  R.n_sp_work = R.n_sp_red = R.n_slots = 0;
  hipStream_t s = P->stream;
  for (int r = 0; r < P->d; ++r)
    if (P->tile[r] % st != 0) throw Error{GP_EDEVICE, "internal: sub-tile does not divide the tile"};
  int64_t nsub = P->n_bins;
  for (int r = 0; r < P->d; ++r) nsub *= P->tile[r] / st;
  if (nsub > (int64_t)std::numeric_limits<int>::max() / 2) throw Error{GP_ENOMEM, "too many sub-tiles"};
  NuArgs a = nu_args(P, R);
  int nsrc_tot = 1;
  for (int r = 0; r < P->d; ++r) nsrc_tot *= P->nsrc;
  const size_t smem = (2 * (size_t)nsrc_tot + 1) * sizeof(int);
  DevBuf cnt;
  cnt.alloc((size_t)(nsub + 1) * sizeof(int), s);  // the counts and their maximum
  int* cmax = cnt.as<int>() + nsub;
  R.sub_off.alloc((size_t)(nsub + 1) * sizeof(int64_t), s);
  GP_HIP(hipMemsetAsync(cmax, 0, sizeof(int), s));
  list_build<false>(P->d, a, st, nsub, smem, s, R, cnt.as<int>(), nullptr, nullptr);
  hipLaunchKernelGGL(max_count_kernel, dim3((unsigned)std::min<int64_t>((nsub + 255) / 256, 1024)),
                     dim3(256), 0, s, nsub, cnt.as<int>(), cmax);
  GP_CHECK_LAUNCH();
  int longest = 0;
  GP_HIP(hipMemcpyAsync(&longest, cmax, sizeof(int), hipMemcpyDeviceToHost, s));
  int64_t total = 0;
  exclusive_scan<int>(cnt.as<int>(), nsub, R.sub_off.as<int64_t>(), s, &total);  // synchronises
  GP_HIP(hipMemcpyAsync(R.sub_off.as<int64_t>() + nsub, &total, sizeof(int64_t), hipMemcpyHostToDevice, s));
  const size_t bound = spread_list_bound_bytes(P, R.n, false);
  if ((size_t)total * sizeof(int2) > bound) throw Error{GP_EDEVICE, "internal: sub-tile lists over their bound"};
  R.sub_list.alloc((size_t)std::max<int64_t>(total, 1) * sizeof(int2), s);
  list_build<true>(P->d, a, st, nsub, smem, s, R, nullptr, R.sub_off.as<int64_t>(), R.sub_list.as<int2>());
  const int64_t chunk = list_chunk(total);
  if (longest > chunk && !P->lean) {
    DevBuf n3, o3;
    n3.alloc((size_t)nsub * 3 * sizeof(int), s);
    o3.alloc((size_t)nsub * 3 * sizeof(int64_t), s);
    int* n_[3] = {n3.as<int>(), n3.as<int>() + nsub, n3.as<int>() + 2 * nsub};
    int64_t* o_[3] = {o3.as<int64_t>(), o3.as<int64_t>() + nsub, o3.as<int64_t>() + 2 * nsub};
    const dim3 g((unsigned)((nsub + 255) / 256));
    hipLaunchKernelGGL((spread_items_kernel<false>), g, dim3(256), 0, s, nsub, (int)chunk, cnt.as<int>(),
                       n_[0], n_[1], n_[2], nullptr, nullptr, nullptr, nullptr, nullptr);
    GP_CHECK_LAUNCH();
    int64_t tot[3] = {0, 0, 0};
    for (int k = 0; k < 3; ++k) exclusive_scan<int>(n_[k], nsub, o_[k], s, &tot[k]);
    R.sp_work.alloc((size_t)tot[0] * sizeof(int4), s);
    R.sp_red.alloc((size_t)tot[2] * sizeof(int4), s);
    hipLaunchKernelGGL((spread_items_kernel<true>), g, dim3(256), 0, s, nsub, (int)chunk, cnt.as<int>(),
                       nullptr, nullptr, nullptr, o_[0], o_[1], o_[2], R.sp_work.as<int4>(),
                       R.sp_red.as<int4>());
    GP_CHECK_LAUNCH();
    R.n_sp_work = tot[0];
    R.n_slots = tot[1];
    R.n_sp_red = tot[2];
    R.sub_st = st;
    R.part.alloc(spread_partial_bytes(P, R), s);
    GP_HIP(hipStreamSynchronize(s));  // n3 and o3 are released on return
  }
  GP_HIP(hipStreamSynchronize(s));  // &total is a host stack value
  R.n_sub = nsub;
  R.n_list = total;
  R.sub_st = st;
}

void exclusive_scan_counts(const int* in, int64_t n, int64_t* out, hipStream_t s, int64_t* total) {
  exclusive_scan<int>(in, n, out, s, total);
}

void spread_sub_launch(Plan* P, const Records& R, const double* xs, int nsets) {
  if (R.n_sub <= 0) throw Error{GP_EDEVICE, "internal: sub-tile lists missing"};
  const bool f64 = P->precision == GP_FP64;
  if (P->d == 1) f64 ? launch_sub<double, 1>(P, R, xs, nsets) : launch_sub<float, 1>(P, R, xs, nsets);
  else if (P->d == 2) f64 ? launch_sub<double, 2>(P, R, xs, nsets) : launch_sub<float, 2>(P, R, xs, nsets);
  else f64 ? launch_sub<double, 3>(P, R, xs, nsets) : launch_sub<float, 3>(P, R, xs, nsets);
}

}  // namespace gp
