// Type-2 interpolation and combine (steps 4b and 5 of section 4.2):
// y_i = sum_k w_k(x_i) beta_k(x_i) (+ eta^2 x_i), where beta_k is grid k summed
// over the w^d cells of the point's window.  Two kernels, chosen by how many
// points share the cells of a block:
//  interp_tile_kernel   many points per block: the block's cells and the halo of
//                       w-1 cells are staged in LDS one grid pair at a time
//  interp_wave_kernel   few points per block (and d = 1): a group of lanes reads
//                       each point's window straight from the grids
#include <algorithm>
#include <mutex>
#include <vector>

#include "gp_internal.h"
#include "gp_window.h"

namespace gp {
namespace {

// Complex grid values as native vectors (arrays of them stay in registers).
template <typename T> struct V2;
template <> struct V2<double> { using type = __attribute__((ext_vector_type(2))) double; };
template <> struct V2<float> { using type = __attribute__((ext_vector_type(2))) float; };

// Blocks go to the 8 XCDs round-robin; groups of grp consecutive items are
// dealt to one XCD each, so neighbouring items, whose windows overlap, read the
// grids through one L2.  The grid is padded to a multiple of 8 grp blocks.
__device__ __forceinline__ int64_t xcd_item(int64_t bid, int grp) {
  const int64_t x = bid % 8, k = bid / 8;
  return ((k / grp) * 8 + x) * grp + k % grp;
}
int64_t xcd_blocks(int64_t n, int grp) { return (n + 8 * grp - 1) / (8 * grp) * (8 * grp); }

// ------------------------------------------------------------------ tile ----
// One workgroup per chunk of the points of a block of bins, C0 x C1 (x C2) cells.
// RG lanes share a point: lane half rg takes the window rows (2-D) or planes
// (3-D) rg, rg + RG, ...; their sums meet in one shuffle.  The window values sit
// in registers for all grid pairs, the next pair's cells are loaded into
// registers while the current pair is summed.
//
// The kernel is bound by LDS reads (w^d cells of 8 or 16 bytes per point and
// pair), so the points of a batch are dealt to lanes by the LDS bank of their
// first cell: every read of a point is at the same distance from its first
// cell on every lane, so lanes whose first cells lie in different banks never
// conflict (against points in batch order: d=2 N=1e6 fp64 0.48 -> 0.41 ms, d=3
// N=1e7 fp32 2.92 -> 2.55 ms).
// Blocks of 2x2 bins (43^2 cells at w = 12) with two lanes per point and 256
// threads in 2-D: one lane per point 0.47, 128 threads 0.64 against 0.41 ms; 2x2x1
// bins (20 x 20 x 12 cells at w = 5) with one lane per point in 3-D: 256 threads
// 2.55, 512 threads 2.03, two lanes per point 2.46 ms (fewer threads stage the
// block more often and hold more of it in registers).  Compile-time widths keep
// the window values in registers: at w = 15 (d=2 N=1e5) 0.32 -> 0.10 ms.
template <typename T, int D, int W, int C0, int C1, int C2, int RG, int NT>
struct TileShape {
  static constexpr int PC0 = C0 + W - 1, PS0 = PC0 | 1, PC1 = C1 + W - 1;
  static constexpr int PC2 = D > 2 ? C2 + W - 1 : 1;
  static constexpr int NC = PS0 * PC1 * PC2;           // staged cells (rows padded to odd)
  static constexpr int NP = NT / RG;                   // points per batch
  static constexpr int LS = (D * W) | 1;               // stride of the staged window values
  static constexpr int TE = (NC + NT - 1) / NT;        // staged cells per thread
  static constexpr int BK = 256 / (2 * (int)sizeof(T));  // cells in one sweep of the LDS banks
  static constexpr size_t cell_bytes = (size_t)NC * 2 * sizeof(T);
  static constexpr size_t row_bytes = (size_t)NP * LS * sizeof(T);
  static constexpr size_t main_bytes = ((cell_bytes > row_bytes ? cell_bytes : row_bytes) + 15) / 16 * 16;
  static constexpr size_t smem = main_bytes + (size_t)(3 * NP + BK + 8) * sizeof(int);
};

// Waves per SIMD to compile for: fp32 in 3-D at w = 6 takes ten registers more than
// four waves leave it otherwise (d=3 N=2e6 0.54 -> 0.42 ms, one register spilled).
template <typename T, int D, int W>
constexpr int kTileWaves = sizeof(T) == 4 && D == 3 && W == 6 ? 4 : 1;

// The order of a point's sum and its measured error: window_sum (ROWS: see interp_w).
template <typename T, int D, int W, int C0, int C1, int C2, int RG, int NT, bool ROWS>
__global__ __launch_bounds__(NT, (kTileWaves<T, D, W>)) void interp_tile_kernel(
    NuArgs a, const typename V2<T>::type* __restrict__ grid, int64_t set_stride,
    const int* __restrict__ cell, const T* __restrict__ pw, int rs,
    const int* __restrict__ bin_start, const int4* __restrict__ work,
    const double* __restrict__ x, double* __restrict__ y, int64_t nwork, int grp, int nbb) {
  using V = typename V2<T>::type;
  using S = TileShape<T, D, W, C0, C1, C2, RG, NT>;
  constexpr int HP = (W + RG - 1) / RG;  // rows or planes per lane
  extern __shared__ __align__(16) unsigned char smem[];
  V* tile = reinterpret_cast<V*>(smem);
  T* s_row = reinterpret_cast<T*>(smem);  // window values, before the first tile
  int* s_slot = reinterpret_cast<int*>(smem + S::main_bytes);  // [NP] slot -> batch point (-1: none)
  int* s_over = s_slot + S::NP;                                // [NP] points whose bank is full
  int* s_org = s_over + S::NP;                                 // [NP] first cell in the tile
  int* s_cnt = s_org + S::NP;                                  // [BK] points per bank, then counters

  const int64_t item = xcd_item(blockIdx.x, grp);
  if (item >= nwork) return;
  grid += blockIdx.y * set_stride;
  x += blockIdx.y * a.n;
  y += blockIdx.y * a.n;
  const int4 wk = work[item];
  // nbb x nbb (x 1) bins per block: the block's origin and its two ranges of
  // consecutive sorted points (one when nbb = 1)
  const int nsb0 = (a.nbins[0] + nbb - 1) / nbb, nsb1 = (a.nbins[1] + nbb - 1) / nbb;
  const int sx = wk.x % nsb0, sy = (wk.x / nsb0) % nsb1, sz = D > 2 ? wk.x / (nsb0 * nsb1) : 0;
  const int t00 = sx * C0, t01 = sy * C1, t02 = sz * C2;
  int r_lo[2] = {0, 0}, r_len0 = 0;
  if (nbb == 1) {
    r_len0 = INT32_MAX;  // in_work: positions are sorted indices
  } else {
    const int bx0 = 2 * sx, bx1 = min(2 * sx + 1, a.nbins[0] - 1);
    for (int q = 0; q < 2; ++q) {
      const int by = 2 * sy + q;
      if (by >= a.nbins[1]) break;
      const int64_t rowbin = ((int64_t)sz * a.nbins[1] + by) * a.nbins[0];
      r_lo[q] = bin_start[rowbin + bx0];
      if (q == 0) r_len0 = bin_start[rowbin + bx1 + 1] - r_lo[0];
    }
  }
  // byte offsets of the thread's cells in a grid pair (cells past the active
  // box are clamped: no window reaches them)
  unsigned off[S::TE];
#pragma unroll
  for (int j = 0; j < S::TE; ++j) {
    const int e = min((int)threadIdx.x + j * NT, S::NC - 1);
    const int l12 = e / S::PS0, l0 = e - l12 * S::PS0;
    const int l1 = D > 2 ? l12 % S::PC1 : l12, l2 = D > 2 ? l12 / S::PC1 : 0;
    const int c0 = min(t00 + l0, a.na[0] - 1), c1 = min(t01 + l1, a.na[1] - 1);
    const int c2 = D > 2 ? min(t02 + l2, a.na[2] - 1) : 0;
    off[j] = (unsigned)((c2 * a.na[1] + c1) * a.na[0] + c0) * (unsigned)sizeof(V);
  }
  const char* gb = reinterpret_cast<const char*>(grid);
  const int64_t gstep = a.pair_stride * (int64_t)sizeof(V);
  // lanes: wave wv holds points wv * (64 / RG) ..; lane half rg = lane / (64 / RG)
  constexpr int PW = 64 / RG;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int slot = wv * PW + lane % PW, rg = lane / PW;

  for (int pos = wk.y; pos < wk.z; pos += S::NP) {
    const int np = min(S::NP, wk.z - pos);
    // the first pair's cells are on their way while the points are dealt
    V nxt[S::TE];
#pragma unroll
    for (int j = 0; j < S::TE; ++j) nxt[j] = *reinterpret_cast<const V*>(gb + off[j]);
    __syncthreads();  // previous batch done with LDS
    for (int e = threadIdx.x; e < S::BK + 1; e += NT) s_cnt[e] = 0;
    // the rows of window values, coalesced, and the deal of the points
    for (int e = threadIdx.x; e < np * D * W; e += NT) {
      const int p = e / (D * W), c = e - p * (D * W);
      const int q = pos + p;
      const int idx = q < r_len0 ? r_lo[0] + q : r_lo[1] + (q - r_len0);
      s_row[p * S::LS + c] = pw[(int64_t)idx * rs + c];
    }
    __syncthreads();
    int over = -1;
    if ((int)threadIdx.x < np) {
      const int q = pos + threadIdx.x;
      const int idx = q < r_len0 ? r_lo[0] + q : r_lo[1] + (q - r_len0);
      int o = cell[idx] - t00 + (cell[a.n + idx] - t01) * S::PS0;
      if (D > 2) o += (cell[2 * a.n + idx] - t02) * S::PS0 * S::PC1;
      s_org[threadIdx.x] = o;
      const int bk = o % S::BK;
      const int r = atomicAdd(&s_cnt[bk], 1);
      if (r < S::NP / S::BK)
        s_slot[r * S::BK + bk] = threadIdx.x;
      else
        over = atomicAdd(&s_cnt[S::BK], 1);
      if (over >= 0) s_over[over] = threadIdx.x;
    }
    __syncthreads();
    // wave 0 gives the k-th free slot the k-th point without one
    if (wv == 0) {
      const int nover = s_cnt[S::BK];
      int base = 0;
      for (int s0 = 0; s0 < S::NP; s0 += 64) {
        const int s = s0 + lane;
        const bool fr = s < S::NP && s / S::BK >= s_cnt[s % S::BK];
        const unsigned long long m = __ballot(fr);
        const int k = base + __popcll(m & ((1ull << lane) - 1ull));
        if (fr) s_slot[s] = k < nover ? s_over[k] : -1;
        base += __popcll(m);
      }
    }
    __syncthreads();
    const int p = s_slot[slot];
    const bool act = p >= 0;
    T p0[W], p1[D > 2 ? W : HP], p2[D > 2 ? HP : 1];
    int idx = 0, o = 0;
    {
      const int pp = act ? p : 0;
      const T* pr = s_row + pp * S::LS;
#pragma unroll
      for (int q = 0; q < W; ++q) p0[q] = pr[q];
      if constexpr (D > 2) {
#pragma unroll
        for (int q = 0; q < W; ++q) p1[q] = pr[W + q];
#pragma unroll
        for (int j = 0; j < HP; ++j) p2[j] = rg + RG * j < W ? pr[2 * W + min(rg + RG * j, W - 1)] : T(0);
      } else {
#pragma unroll
        for (int j = 0; j < HP; ++j) p1[j] = rg + RG * j < W ? pr[W + min(rg + RG * j, W - 1)] : T(0);
      }
      const int q = pos + pp;
      idx = q < r_len0 ? r_lo[0] + q : r_lo[1] + (q - r_len0);
      o = s_org[pp];
    }
    constexpr int HS = D > 2 ? S::PS0 * S::PC1 : S::PS0;  // step between rows / planes
    const V* tr0 = tile + o + rg * HS;
    // the last row of a lane may lie outside the window (odd W): it re-reads the
    // lane's first row with weight zero
    const int lastoff = rg + RG * (HP - 1) < W ? RG * (HP - 1) * HS : 0;
    const T* wrow = pw + (int64_t)idx * rs + D * W;
    double part = 0.0;
    T wa = wrow[0], wb = wrow[1];
    for (int g = 0; g < a.npair; ++g) {
      __syncthreads();  // rows in registers / previous pair's tile no longer read
#pragma unroll
      for (int j = 0; j < S::TE; ++j)
        if (j + 1 < S::TE || (int)threadIdx.x + j * NT < S::NC) tile[threadIdx.x + j * NT] = nxt[j];
      if (g + 1 < a.npair) {
        const char* gn = gb + (g + 1) * gstep;
#pragma unroll
        for (int j = 0; j < S::TE; ++j) nxt[j] = *reinterpret_cast<const V*>(gn + off[j]);
      }
      __syncthreads();
      if (act) {
        double bx, by;
        window_sum<T, V, D, W, HP, RG, S::PS0, HS, ROWS>(tr0, lastoff, p0, p1, p2, &bx, &by);
        part += (double)wa * bx + (double)wb * by;
      }
      if (g + 1 < a.npair) {
        wa = wrow[2 * g + 2];
        wb = wrow[2 * g + 3];
      }
    }
    if (RG == 2) part += __shfl_xor(part, 32);
    if (act && rg == 0) y[idx] = (a.add_noise ? a.eta2 * x[idx] : 0.0) + part;
  }
}

// ------------------------------------------------------------------ wave ----
// XL lanes along the window's first dimension, YL along its rows; a wave holds
// 64 / (XL YL) points (one in d >= 2).  Each lane sums its cells of every grid
// pair, weights the sums in fp64, and the group adds up by xor shuffles.  All of
// a pair's loads are in flight at once; rows of w cells are contiguous.  Bound by
// cache lines: d=3 N=2e5 fp64 (280^3 cells, w = 7) 6.72 -> 0.82 ms against blocks
// staged in LDS (263 KB of cells per 4.7 points), d=2 N=2e4 fp32 0.061 -> 0.021,
// d=1 N=2000 fp64 two launches of 0.009 + 0.006 -> one of 0.007.
constexpr int kWaveThreads = 256;
template <typename T, int D, int W>
__global__ __launch_bounds__(kWaveThreads) void interp_wave_kernel(
    NuArgs a, const typename V2<T>::type* __restrict__ grid, int64_t set_stride,
    const int* __restrict__ cell, const T* __restrict__ pw, int rs, const double* __restrict__ x,
    double* __restrict__ y, int grp, int64_t i0) {
  using V = typename V2<T>::type;
  constexpr int XL = W <= 4 ? 4 : (W <= 8 ? 8 : 16);
  constexpr int ROWS = D == 1 ? 1 : (D == 2 ? W : W * W);
  constexpr int YL = D == 1 ? 1 : 64 / XL;
  constexpr int PPW = 64 / (XL * YL);
  constexpr int NS = (ROWS + YL - 1) / YL;  // rows per lane
  constexpr int NU = NS < 8 ? NS : 8;
  const int lane = threadIdx.x & 63;
  int64_t wid = xcd_item(blockIdx.x, grp) * (kWaveThreads / 64);
  wid += __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t i = i0 + wid * PPW + lane / (XL * YL);
  if (i >= a.n) return;  // whole groups
  grid += blockIdx.y * set_stride;
  x += blockIdx.y * a.n;
  y += blockIdx.y * a.n;
  const int lx = lane % XL, ly = (lane / XL) % YL;
  const T* pr = pw + i * rs;
  const T p0 = lx < W ? pr[lx] : T(0);
  const int64_t base = a.grid_off + (int64_t)cell[i] * a.gstride[0] +
                       (D > 1 ? (int64_t)cell[a.n + i] * a.gstride[1] : 0) +
                       (D > 2 ? (int64_t)cell[2 * a.n + i] * a.gstride[2] : 0) + min(lx, W - 1);
  double part = 0.0;
  if constexpr (NS <= 8) {
    // all of a pair's cells in flight; row offsets and weights are shared by the pairs
    int64_t ro[NS];
    T wr[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int row = ly + YL * j, rc = min(row, ROWS - 1);
      const int q1 = D > 2 ? rc % W : rc, q2 = D > 2 ? rc / W : 0;
      ro[j] = (D > 1 ? (int64_t)q1 * a.gstride[1] : 0) + (D > 2 ? (int64_t)q2 * a.gstride[2] : 0);
      T wv = D > 1 ? pr[W + q1] : T(1);
      if (D > 2) wv *= pr[2 * W + q2];
      wr[j] = row < ROWS ? wv * p0 : T(0);
    }
#pragma unroll 2
    for (int g = 0; g < a.npair; ++g) {
      const V* gp = grid + (int64_t)g * a.pair_stride + base;
      V v[NS];
#pragma unroll
      for (int j = 0; j < NS; ++j) v[j] = gp[ro[j]];
      T sx = 0, sy = 0;
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        sx += wr[j] * v[j].x;
        sy += wr[j] * v[j].y;
      }
      part += (double)pr[D * W + 2 * g] * (double)sx + (double)pr[D * W + 2 * g + 1] * (double)sy;
    }
  } else {
    for (int g = 0; g < a.npair; ++g) {
      const V* gp = grid + (int64_t)g * a.pair_stride + base;
      double sx = 0, sy = 0;  // up to 64 rows: fp32 grids' in fp64
#pragma unroll NU
      for (int j = 0; j < NS; ++j) {
        const int row = ly + YL * j, rc = min(row, ROWS - 1);
        const int q1 = D > 2 ? rc % W : rc, q2 = D > 2 ? rc / W : 0;
        const V v = gp[(int64_t)q1 * a.gstride[1] + (D > 2 ? (int64_t)q2 * a.gstride[2] : 0)];
        T wv = pr[W + q1];
        if (D > 2) wv *= pr[2 * W + q2];
        wv = row < ROWS ? wv * p0 : T(0);
        sx += (double)wv * (double)v.x;
        sy += (double)wv * (double)v.y;
      }
      part += (double)pr[D * W + 2 * g] * sx + (double)pr[D * W + 2 * g + 1] * sy;
    }
  }
#pragma unroll
  for (int o = XL * YL / 2; o > 0; o >>= 1) part += __shfl_xor(part, o);
  if (lane % (XL * YL) == 0) y[i] = (a.add_noise ? a.eta2 * x[i] : 0.0) + part;
}

// Dynamic LDS above 64 KB needs an explicit opt-in for each kernel (each
// instantiation: kernels of one signature are distinct functions).
void allow_lds(const void* f, size_t bytes) {
  static std::mutex mu;
  static std::vector<const void*> done;
  std::lock_guard<std::mutex> lk(mu);
  if (std::find(done.begin(), done.end(), f) != done.end()) return;
  GP_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  done.push_back(f);
}

struct InterpCall {
  Plan* P;
  const Records* R;
  const double* xs;
  double* ys;
  int add_noise, nsets;
  const void* grid;
  int64_t set_stride;
};

template <typename T, int D, int W, int C0, int C1, int C2, int RG, int NT, bool ROWS = false>
void launch_tile(const InterpCall& c, bool per_bin) {
  using S = TileShape<T, D, W, C0, C1, C2, RG, NT>;
  static_assert(S::smem <= 80 * 1024, "at least two workgroups per CU");
  const Records& R = *c.R;
  const int64_t nw = per_bin ? R.n_in_work : R.n_in_work2;
  if (nw == 0) return;
  auto kern = interp_tile_kernel<T, D, W, C0, C1, C2, RG, NT, ROWS>;
  if (S::smem > 64 * 1024) allow_lds(reinterpret_cast<const void*>(kern), S::smem);
  NuArgs a = nu_args(c.P, R);
  a.add_noise = c.add_noise;
  constexpr int grp = 16;
  hipLaunchKernelGGL(kern, dim3((unsigned)xcd_blocks(nw, grp), (unsigned)c.nsets), dim3(NT), S::smem,
                     c.P->stream, a, static_cast<const typename V2<T>::type*>(c.grid), c.set_stride,
                     R.cell.as<int>(), R.pw.as<T>(), R.rs, R.bin_start.as<int>(),
                     per_bin ? R.in_work.as<int4>() : R.in_work2.as<int4>(), c.xs, c.ys, nw, grp,
                     per_bin ? 1 : 2);
  GP_CHECK_LAUNCH();
}

template <typename T, int D, int W>
void launch_wave(const InterpCall& c) {
  const Records& R = *c.R;
  if (R.n == 0) return;
  constexpr int XL = W <= 4 ? 4 : (W <= 8 ? 8 : 16);
  constexpr int PPB = kWaveThreads / (D == 1 ? XL : 64);
  constexpr int grp = 16;
  NuArgs a = nu_args(c.P, R);
  a.add_noise = c.add_noise;
  // a launch has fewer than 2^32 threads: with 16 lanes per point that is reached at 2.7e8
  // points (slices of whole groups of blocks, so that none is done twice)
  constexpr int64_t slice = ((int64_t)1 << 31) / kWaveThreads * PPB;
  static_assert(slice % (8 * grp * PPB) == 0, "slices of whole groups of blocks");
  for (int64_t i0 = 0; i0 < R.n; i0 += slice) {
    const int64_t np = std::min(slice, R.n - i0);
    hipLaunchKernelGGL((interp_wave_kernel<T, D, W>),
                       dim3((unsigned)xcd_blocks((np + PPB - 1) / PPB, grp), (unsigned)c.nsets),
                       dim3(kWaveThreads), 0, c.P->stream, a,
                       static_cast<const typename V2<T>::type*>(c.grid), c.set_stride,
                       R.cell.as<int>(), R.pw.as<T>(), R.rs, c.xs, c.ys, grp, i0);
    GP_CHECK_LAUNCH();
  }
}

// The blocks of interp_tile_kernel: 2x2 bins of 16^2 cells in 2-D, 2x2x1 bins
// of 8^3 cells in 3-D where two workgroups fit a CU's LDS, else one bin.
template <typename T, int D, int W>
constexpr bool kTile3Super = TileShape<T, 3, W, 16, 16, 8, 1, 512>::smem <= 64 * 1024;
template <typename T, int D, int W>
constexpr bool kTile3Bin = TileShape<T, 3, W, 8, 8, 8, 1, 256>::smem <= 80 * 1024;

template <typename T, int D, int W>
void interp_w(const InterpCall& c) {
  const Plan* P = c.P;
  if constexpr (D > 1) {
    const int def = D == 2 ? 16 : 8;  // the tile side the blocks are compiled for
    bool fits = (double)P->na[0] * P->na[1] * P->na[2] * 2 * sizeof(T) < 4.0e9;  // 32-bit cell offsets
    for (int r = 0; r < D; ++r) fits = fits && P->tile[r] == def;
    // The block is staged for all of its points, a point's own window costs w^d
    // cells and about as much again in partial lines: staging pays from `line` windows'
    // worth of points per block on (ms staged / by waves at the windows per block):
    //  2-D, 2: d=2 N=1e5 fp64 at 7 0.10 staged
    //  3-D, 2x2x1 bins, 1: fp32 w=5 1.06 0.34 / 0.40, 1.7 0.37 / 0.60, 3.2 0.40 / 0.99
    //  3-D, one bin, 2: fp64 w=7 1.2 0.29 / 0.18, 2.4 0.30 / 0.30, 5 0.32 / 0.57; w=4 0.6
    //  0.068 / 0.042, 2 0.075 / 0.102; w=8 3.1 0.49 / 0.42, 6.5 0.52 / 0.78; fp32 w=9 1.8 0.15 / 0.10,
    //  3.7 0.16 / 0.20.  fp64 w=9 (8) and 10 (11), where staging takes six times as long
    //  as at w=8 (why was not found): w=9 3.4 2.83 / 1.33, 7.2 2.9 / 2.7, 29 3.9 / 10.7; w=10 4.2
    //  4.4 / 1.8, 8.7 4.5 / 3.8, 12 4.6 / 5.3.  fp64 from w=11 on fits no block; waves take 0.06 to 0.54 of the
    //  per-bin kernel's time (interp = 2) from 3 to 60 points per bin (w=11, 12).
    // The average is over all blocks.  Clustered points fill few of them: there the
    // blocks that are staged count, at a line of twice (2-D: 1.5 times) as many windows, so that
    // the empty border of uniform points does not change their kernel, and from one
    // block per CU on (d=2 fp32 N=1e5 in one cluster 0.034 -> 0.016 ms, d=3 fp32 N=1e6 in
    // eight 0.56 -> 0.25; with 80 blocks, d=2 fp64 N=1e4, 0.016 staged and 0.011 by waves).
    auto dense = [&](double window, int nc, double blocks, int64_t staged, double line) {
      const double cells = (double)c.R->n * window;
      return cells > line * blocks * nc ||
             (staged >= 256 && cells > line * (D == 2 ? 1.5 : 2.0) * (double)staged * nc);
    };
    if (fits) {
      if constexpr (D == 2) {
        using S = TileShape<T, 2, W, 32, 32, 1, 2, 256>;
        if (dense(W * W, S::NC, 0.25 * P->nbins[0] * P->nbins[1], c.R->n_in_work2, 2.0)) {
          launch_tile<T, 2, W, 32, 32, 1, 2, 256>(c, false);
          return;
        }
      } else if constexpr (kTile3Super<T, D, W>) {
        using S = TileShape<T, 3, W, 16, 16, 8, 1, 512>;
        if (dense(W * W * W, S::NC, 0.25 * P->n_bins, c.R->n_in_work2, 1.0)) {
          // fp32, w = 7: rows of 26 weights on took a block of 2x2x1 bins over the LDS that
          // the former kernel had, and the per-bin one joins rows in fp64
          if constexpr (sizeof(T) == 4 && W == 7) {
            if (P->nkp >= 26) {
              launch_tile<T, 3, W, 16, 16, 8, 1, 512, true>(c, false);
              return;
            }
          }
          launch_tile<T, 3, W, 16, 16, 8, 1, 512>(c, false);
          return;
        }
      } else if constexpr (kTile3Bin<T, D, W>) {
        using S = TileShape<T, 3, W, 8, 8, 8, 1, 256>;
        constexpr double line = sizeof(T) == 4 || W < 9 ? 2.0 : (W == 9 ? 8.0 : 11.0);
        if (dense(W * W * W, S::NC, (double)P->n_bins, c.R->n_in_work, line)) {
          launch_tile<T, 3, W, 8, 8, 8, 1, 256, (W > 7)>(c, true);
          return;
        }
      }
    }
  }
  launch_wave<T, D, W>(c);
}

template <typename T, int D>
void interp_d(const InterpCall& c) {
  switch (c.P->w) {
#define GP_IW(N) case N: interp_w<T, D, N>(c); return;
    GP_IW(2) GP_IW(3) GP_IW(4) GP_IW(5) GP_IW(6) GP_IW(7) GP_IW(8) GP_IW(9) GP_IW(10) GP_IW(11)
    GP_IW(12) GP_IW(13) GP_IW(14) GP_IW(15) GP_IW(16)
#undef GP_IW
    default: throw Error{GP_EUNSUPPORTED, "window width not compiled"};
  }
}

}  // namespace

// Compiled twice (GP_INTERP_FP64 = 1 / 0) so the two precisions build in parallel.
#if GP_INTERP_FP64
#define GP_INTERP_T double
#define GP_INTERP_FN interp_fp64
#else
#define GP_INTERP_T float
#define GP_INTERP_FN interp_fp32
#endif

// ys = sum_k w_k beta_k (+ eta^2 xs) at the points of R for nsets consecutive
// vectors, whose grids lie set_stride complex elements apart.
void GP_INTERP_FN(Plan* P, const Records& R, const double* xs, double* ys, int add_noise, int nsets,
                  const void* grid, int64_t set_stride) {
  using T = GP_INTERP_T;
  PhaseScope ps(P, PH_INTERP);
  const InterpCall c{P, &R, xs, ys, add_noise, nsets, grid, set_stride};
  if (P->d == 1) interp_d<T, 1>(c);
  else if (P->d == 2) interp_d<T, 2>(c);
  else interp_d<T, 3>(c);
}

}  // namespace gp
