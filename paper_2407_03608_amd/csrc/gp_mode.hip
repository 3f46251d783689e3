// Step 3 of section 4.2: mixing of the Fourier coefficients of the N_sigma+1
// grids at every mode of the grid {-M..M}^d (rem:step3).  Two variants:
// the precomputed tensor A_k'k stored per distinct |n|^2 (default) and the
// direct sum over the t nodes.  Both fold the window deconvolution in.
#include "gp_internal.h"

namespace gp {
namespace {

template <typename T> struct V2;
template <> struct V2<double> { using type = double2; };
template <> struct V2<float> { using type = float2; };

constexpr int kThreads = 256;

// ------------------------------------------------------------------ mode ----
struct ModeArgs {
  int d;
  int64_t M, mc, F;       // mc = 2M+1, F = mc^d
  int64_t mp;             // distance of rows of modes
  int nk, npair, nt;
  int64_t pair_stride;
  int fourstep;
  int64_t nf, L1, L2;
};

__device__ __forceinline__ int64_t mode_store(const ModeArgs& a, int64_t f, const int64_t* nv) {
  if (!a.fourstep) return f % a.mc + (f / a.mc) * a.mp;
  int64_t k = nv[0] % a.nf;
  if (k < 0) k += a.nf;
  return (k % a.L2) * a.L1 + (k / a.L2);
}

// Each thread owns a mode pair (n, -n) of every complex grid: it unpacks the two
// real spectra b_2g, b_2g+1, deconvolves, applies
//   a_k'[n] = sum_j v~_j G^_k'j[n] sum_k G^_kj[n] b_k[n]     (step 3, rem:step3 direct)
// re-deconvolves and packs the result back in place.
template <typename T, int NK>
__global__ __launch_bounds__(kThreads) void mode_kernel(
    ModeArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ gtab,
    const T* __restrict__ etab, const T* __restrict__ vt, const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  const int64_t f = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t half = (a.F + 1) / 2;
  if (f >= half) return;
  const int64_t fc = a.F - 1 - f;
  int64_t nv[3] = {0, 0, 0}, nvc[3] = {0, 0, 0};
  int64_t an[3] = {0, 0, 0};
  {
    int64_t q = f;
    for (int r = 0; r < a.d; ++r) {
      nv[r] = q % a.mc - a.M;
      q /= a.mc;
      nvc[r] = -nv[r];
      an[r] = nv[r] < 0 ? -nv[r] : nv[r];
    }
  }
  const int64_t M1 = a.M + 1;
  T D = T(1);
  for (int r = 0; r < a.d; ++r) D *= dec[r * M1 + an[r]];
  const int64_t s0 = mode_store(a, f, nv), s1 = mode_store(a, fc, nvc);
  V b[NK], acc[NK];
#pragma unroll
  for (int g = 0; g < NK / 2; ++g) {
    V z = V{T(0), T(0)}, zc = V{T(0), T(0)};
    if (g < a.npair) {
      z = C[g * a.pair_stride + s0];
      zc = C[g * a.pair_stride + s1];
    }
    b[2 * g] = V{T(0.5) * (z.x + zc.x) * D, T(0.5) * (z.y - zc.y) * D};
    b[2 * g + 1] = V{T(0.5) * (z.y + zc.y) * D, T(-0.5) * (z.x - zc.x) * D};
    acc[2 * g] = V{T(0), T(0)};
    acc[2 * g + 1] = V{T(0), T(0)};
  }
  const int nk = a.nk;
  for (int j = 0; j < a.nt; ++j) {
    const T* g0 = gtab + ((int64_t)j * nk) * M1 + an[0];
    const T* e1 = etab + ((int64_t)j * nk) * M1 + an[1];
    const T* e2 = etab + ((int64_t)j * nk) * M1 + an[2];
    T gk[NK];
    V s = V{T(0), T(0)};
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      T g = T(0);
      if (k < nk) {
        g = g0[k * M1];
        if (a.d > 1) g *= e1[k * M1];
        if (a.d > 2) g *= e2[k * M1];
      }
      gk[k] = g;
      s.x += g * b[k].x;
      s.y += g * b[k].y;
    }
    const T v = vt[j];
    s.x *= v;
    s.y *= v;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      acc[k].x += gk[k] * s.x;
      acc[k].y += gk[k] * s.y;
    }
  }
#pragma unroll
  for (int g = 0; g < NK / 2; ++g) {
    if (g >= a.npair) break;
    const V p = V{acc[2 * g].x * D, acc[2 * g].y * D};
    const V q = V{acc[2 * g + 1].x * D, acc[2 * g + 1].y * D};
    C[g * a.pair_stride + s0] = V{p.x - q.y, p.y + q.x};
    if (s1 != s0) C[g * a.pair_stride + s1] = V{p.x + q.y, -p.y + q.x};
  }
}

// Step 3 with the precomputed tensor of rem:step3.  A_k'k[n] depends on n only
// through |n|^2, so it is stored once per distinct |n|^2 (upper triangle, nkp
// wide).  Each thread owns the orthant point (|n_0|, .., |n_d-1|) and the up to
// 2^(d-1) conjugate pairs (s*n, -s*n) of sign patterns s that share its row.
struct RadialArgs {
  int d;
  int64_t M, mc, Q;       // Q = (M+1)^d orthant points
  int64_t mp;             // distance of rows of modes
  int npair;
  int64_t pair_stride;
  int fourstep;
  int64_t nf, L1, L2;
  int nsets;              // vector sets (consecutive, set_stride elements apart)
  int64_t set_stride;
  const int* tiles;       // 2-D: the block -> orthant tile order (null: linear in q)
  int64_t ntx;            // tiles along n_0
};
static_assert(kModeTileX * kModeTileY == kThreads, "one orthant tile per block");

__device__ __forceinline__ int64_t radial_store(const RadialArgs& a, const int64_t* nv) {
  if (!a.fourstep) {
    int64_t f = 0, mul = 1;
    for (int r = 0; r < a.d; ++r) {
      f += (nv[r] + a.M) * mul;
      mul *= r == 0 ? a.mp : a.mc;
    }
    return f;
  }
  int64_t k = nv[0] % a.nf;
  if (k < 0) k += a.nf;
  return (k % a.L2) * a.L1 + (k / a.L2);
}

template <typename T, int NK>
__global__ __launch_bounds__(kThreads) void mode_radial_kernel(
    RadialArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ Atab,
    const int* __restrict__ rowidx, const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  constexpr int NP = NK * (NK + 1) / 2;
  const int64_t M1 = a.M + 1;
  int64_t an[3] = {0, 0, 0};
  if (a.tiles) {
    const int64_t t = a.tiles[blockIdx.x];
    an[0] = (t % a.ntx) * kModeTileX + threadIdx.x % kModeTileX;
    an[1] = (t / a.ntx) * kModeTileY + threadIdx.x / kModeTileX;
    if (an[0] > a.M || an[1] > a.M) return;
  } else {
    const int64_t tid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (tid >= a.Q) return;
    int64_t q = tid;
    for (int r = 0; r < a.d; ++r) {
      an[r] = q % M1;
      q /= M1;
    }
  }
  const int64_t s2 = an[0] * an[0] + an[1] * an[1] + an[2] * an[2];
  const int64_t row = a.d == 1 ? an[0] : (int64_t)rowidx[s2];
  const T* Ar = Atab + row * NP;
  T D = T(1);
  for (int r = 0; r < a.d; ++r) D *= dec[r * M1 + an[r]];
  int first_nz = -1;
  for (int r = 0; r < a.d; ++r)
    if (an[r] != 0) {
      first_nz = r;
      break;
    }
  // Sign patterns are processed two at a time so that one pass over the row of
  // A serves both (the row is the dominant read of this kernel); the vector
  // sets of a multi-vector application reuse the row from the caches.
  const int npat = 1 << (a.d - 1);
  for (int set = 0; set < a.nsets; ++set)
  for (int pg = 0; pg < npat; pg += 2) {
    V* __restrict__ Cs = C + set * a.set_stride;
    bool keep[2];
    int64_t st0[2], st1[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pat = pg + h;
      keep[h] = pat < npat;
      int64_t nv[3] = {0, 0, 0}, nvc[3] = {0, 0, 0};
      for (int r = 0; r < a.d; ++r) {
        const int neg = r == 0 ? 0 : ((pat >> (r - 1)) & 1);
        if (neg && (an[r] == 0 || r == first_nz)) keep[h] = false;  // duplicate pattern
        nv[r] = neg ? -an[r] : an[r];
        nvc[r] = -nv[r];
      }
      st0[h] = keep[h] ? radial_store(a, nv) : 0;
      st1[h] = keep[h] ? radial_store(a, nvc) : 0;
    }
    if (!keep[0] && !keep[1]) continue;
    V b[2][NK];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < NK / 2; ++g) {
        V z = V{T(0), T(0)}, zc = V{T(0), T(0)};
        if (keep[h] && g < a.npair) {
          z = Cs[g * a.pair_stride + st0[h]];
          zc = Cs[g * a.pair_stride + st1[h]];
        }
        b[h][2 * g] = V{T(0.5) * (z.x + zc.x) * D, T(0.5) * (z.y - zc.y) * D};
        b[h][2 * g + 1] = V{T(0.5) * (z.y + zc.y) * D, T(-0.5) * (z.x - zc.x) * D};
      }
    V acc[2][NK];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < NK; ++k) acc[h][k] = V{T(0), T(0)};
    int p = 0;
#pragma unroll
    for (int k1 = 0; k1 < NK; ++k1) {
#pragma unroll
      for (int k2 = k1; k2 < NK; ++k2) {
        const T av = Ar[p++];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          acc[h][k1].x += av * b[h][k2].x;
          acc[h][k1].y += av * b[h][k2].y;
          if (k2 != k1) {
            acc[h][k2].x += av * b[h][k1].x;
            acc[h][k2].y += av * b[h][k1].y;
          }
        }
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!keep[h]) continue;
#pragma unroll
      for (int g = 0; g < NK / 2; ++g) {
        if (g >= a.npair) break;
        const V pp = V{acc[h][2 * g].x * D, acc[h][2 * g].y * D};
        const V qq = V{acc[h][2 * g + 1].x * D, acc[h][2 * g + 1].y * D};
        Cs[g * a.pair_stride + st0[h]] = V{pp.x - qq.y, pp.y + qq.x};
        if (st1[h] != st0[h]) Cs[g * a.pair_stride + st1[h]] = V{pp.x + qq.y, -pp.y + qq.x};
      }
    }
  }
}

// Grid pair (a_2g, a_2g+1) of one mode times the deconvolution D, packed for the modes n
// and -n.  Written with explicit fma so that the kernels that call it round
// alike: a column of several vector sets has the bits of a single product.
template <typename V, typename T>
__device__ __forceinline__ void pack_pair(V p, V q, T D, V* z, V* zc) {
  const T px = p.x * D, py = p.y * D;
  *z = V{__builtin_elementwise_fma(-q.y, D, px), __builtin_elementwise_fma(q.x, D, py)};
  *zc = V{__builtin_elementwise_fma(q.y, D, px), __builtin_elementwise_fma(q.x, D, -py)};
}

// d = 2, several vector sets: one thread per (orthant point, sign pattern), the two patterns of a
// point on adjacent lanes, so each reads the same row of A in the same load
// instruction (one fetch) while holding half the registers of a thread that
// owns both patterns.  Two blocks per orthant tile (two of its rows each).
template <typename T, int NK>
__global__ __launch_bounds__(kThreads) void mode_radial2_kernel(
    RadialArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ Atab,
    const int* __restrict__ rowidx, const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  constexpr int NP = NK * (NK + 1) / 2;
  const int h = (int)(threadIdx.x & 1);
  const int lp = (int)(threadIdx.x >> 1);
  const int64_t M1 = a.M + 1;
  const int64_t t = a.tiles[blockIdx.x >> 1];
  const int64_t an0 = (t % a.ntx) * kModeTileX + lp % kModeTileX;
  const int64_t an1 = (t / a.ntx) * kModeTileY + (kModeTileY / 2) * (blockIdx.x & 1) + lp / kModeTileX;
  if (an0 > a.M || an1 > a.M) return;
  const T* Ar = Atab + (int64_t)rowidx[an0 * an0 + an1 * an1] * NP;
  const T D = dec[an0] * dec[M1 + an1];
  // pattern 1 negates n_1; it repeats pattern 0 when n_0 = 0 or n_1 = 0
  if (h == 1 && (an0 == 0 || an1 == 0)) return;
  const int64_t n1 = h ? -an1 : an1;
  const int64_t st0 = (an0 + a.M) + (n1 + a.M) * a.mp;
  const int64_t st1 = (-an0 + a.M) + (-n1 + a.M) * a.mp;
  for (int set = 0; set < a.nsets; ++set) {
    V* __restrict__ Cs = C + set * a.set_stride;
    V b[NK];
#pragma unroll
    for (int g = 0; g < NK / 2; ++g) {
      V z = V{T(0), T(0)}, zc = V{T(0), T(0)};
      if (g < a.npair) {
        z = Cs[g * a.pair_stride + st0];
        zc = Cs[g * a.pair_stride + st1];
      }
      b[2 * g] = V{T(0.5) * (z.x + zc.x) * D, T(0.5) * (z.y - zc.y) * D};
      b[2 * g + 1] = V{T(0.5) * (z.y + zc.y) * D, T(-0.5) * (z.x - zc.x) * D};
    }
    V acc[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) acc[k] = V{T(0), T(0)};
    int p = 0;
#pragma unroll
    for (int k1 = 0; k1 < NK; ++k1) {
#pragma unroll
      for (int k2 = k1; k2 < NK; ++k2) {
        const T av = Ar[p++];
        acc[k1].x += av * b[k2].x;
        acc[k1].y += av * b[k2].y;
        if (k2 != k1) {
          acc[k2].x += av * b[k1].x;
          acc[k2].y += av * b[k1].y;
        }
      }
    }
#pragma unroll
    for (int g = 0; g < NK / 2; ++g) {
      if (g >= a.npair) break;
      V z, zc;
      pack_pair(acc[2 * g], acc[2 * g + 1], D, &z, &zc);
      Cs[g * a.pair_stride + st0] = z;
      if (st1 != st0) Cs[g * a.pair_stride + st1] = zc;
    }
  }
}

// LDS accesses of the wave's lanes before it are done before those after it.  A wave's
// LDS operations complete in order, so this only binds the compiler (no instruction).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// fp64, d = 2 and 3: a wave takes 64 / 2^(d-1) orthant points, a point's sign
// patterns on adjacent lanes.  The rows of A it needs come through LDS, 128 bytes
// of every row at a time: eight lanes load one row's 128 bytes (16 each), the next
// chunk is in flight while the current one is used, and each lane then reads its
// own row (slots permuted by the row so that the lanes fall on different banks).
// In the kernels above each lane gathers its own row, at a cache-line lookup per
// lane and load: d=3 M=189 (6 grid pairs) 3.66 -> 2.60 ms, d=2 M=2047 (7 pairs) 1.27 ->
// 1.20 ms, M=805 0.211 -> 0.202.  What bounds this one is not established.  In 3-D it
// moves the mode values at 4.1 TB/s, near a copy's 4.7.  In 2-D 8.2 GB leave the L2s per
// launch (6.8 TB/s, so part of it from the cache behind them): 3.8 of mode values and
// 4.3 of table, which is every point's 8 lines of 128 bytes with no reuse.  fp32 (segments of 256 bytes instead of 512 per
// pattern) loses: d=2 M=2047 0.350 -> 0.373, d=3 M=115 0.223 -> 0.260; and so do several
// vector sets in 2-D, whose row mode_radial2_kernel keeps in registers: 16
// sets M=805 2.45 -> 2.96.  Taking the mirrored point (n_1, n_0), which shares the row,
// on the same XCD at the same time changed nothing (1.19 and 0.206).
template <typename T, int NK, int D>
__global__ __launch_bounds__(kThreads) void mode_rows_kernel(
    RadialArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ Atab,
    const int* __restrict__ rowidx, const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  constexpr int E = 16 / (int)sizeof(T);  // table elements per 16-byte piece
  typedef T Piece __attribute__((ext_vector_type(E)));
  typedef T PieceU __attribute__((ext_vector_type(E), aligned(sizeof(T))));  // rows start at any element
  constexpr int NP = NK * (NK + 1) / 2;
  constexpr int PPR = (NP + E - 1) / E;     // pieces per row (the table ends with one to spare)
  constexpr int NCH = (PPR + 7) / 8;        // chunks of 8 pieces
  constexpr int NPAT = 1 << (D - 1), PW = 64 / NPAT;  // points per wave
  constexpr int NLD = PW / 8;               // pieces loaded per lane and chunk
  __shared__ Piece stage[kThreads / 64][PW * 8];
  const int lane = (int)(threadIdx.x & 63);
  const int h = lane % NPAT, rr = lane / NPAT;
  const int lp = (int)threadIdx.x / NPAT;
  const int64_t M1 = a.M + 1;
  int64_t an[3] = {0, 0, 0};
  bool act;
  if (D == 2) {  // two blocks per orthant tile
    const int64_t t = a.tiles[blockIdx.x >> 1];
    an[0] = (t % a.ntx) * kModeTileX + lp % kModeTileX;
    an[1] = (t / a.ntx) * kModeTileY + (kModeTileY / 2) * (blockIdx.x & 1) + lp / kModeTileX;
    act = an[0] <= a.M && an[1] <= a.M;
  } else {
    int64_t q = (int64_t)blockIdx.x * (kThreads / NPAT) + lp;
    act = q < a.Q;
    an[0] = q % M1;
    q /= M1;
    an[1] = q % M1;
    an[2] = q / M1;
  }
  if (!act) an[0] = an[1] = an[2] = 0;
  const int row = rowidx[an[0] * an[0] + an[1] * an[1] + an[2] * an[2]];
  const T* src[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int r = (lane >> 3) + 8 * i;  // the row of piece lane + 64 i
    src[i] = Atab + (int64_t)__shfl(row, r * NPAT) * NP + ((lane & 7) ^ ((r >> 1) & 7)) * E;
  }
  T dd = dec[an[0]] * dec[M1 + an[1]];
  if (D == 3) dd *= dec[2 * M1 + an[2]];
  // pattern h negates the n_r whose bits are set; it repeats another pattern where
  // one of those is zero or the point's first nonzero coordinate
  int64_t nv[3];
  const int first_nz = an[0] != 0 ? 0 : (an[1] != 0 ? 1 : 2);
  nv[0] = an[0];
#pragma unroll
  for (int r = 1; r < D; ++r) {
    const bool neg = (h >> (r - 1)) & 1;
    if (neg && (an[r] == 0 || r == first_nz)) act = false;
    nv[r] = neg ? -an[r] : an[r];
  }
  int64_t st0 = 0, st1 = 0, mul = 1;
#pragma unroll
  for (int r = 0; r < D; ++r) {
    st0 += (nv[r] + a.M) * mul;
    st1 += (a.M - nv[r]) * mul;
    mul *= r == 0 ? a.mp : a.mc;
  }
  Piece* own = stage[threadIdx.x >> 6];
  const Piece* mine = own + rr * 8;
  const int swz = (rr >> 1) & 7;
  for (int set = 0; set < a.nsets; ++set) {
    V* __restrict__ Cs = C + set * a.set_stride;
    // (a value the compiler cannot see through: it would otherwise load the whole row
    // into registers ahead of the loop over sets)
    int zero = 0;
    int64_t r0 = st0, r1 = st1;
    asm volatile("" : "+s"(zero), "+v"(r0), "+v"(r1));
    Piece next[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i)
      if (8 <= PPR || (((lane & 7) ^ ((((lane >> 3) + 8 * i) >> 1) & 7)) < PPR))
        next[i] = *reinterpret_cast<const PieceU*>(src[i] + zero);
    V b[NK];
#pragma unroll
    for (int g = 0; g < NK / 2; ++g) {
      const V z = Cs[g * a.pair_stride + r0], zc = Cs[g * a.pair_stride + r1];
      b[2 * g] = V{T(0.5) * (z.x + zc.x) * dd, T(0.5) * (z.y - zc.y) * dd};
      b[2 * g + 1] = V{T(0.5) * (z.y + zc.y) * dd, T(-0.5) * (z.x - zc.x) * dd};
    }
    V acc[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) acc[k] = V{T(0), T(0)};
    int p = 0;
    Piece cur;
#pragma unroll
    for (int k1 = 0; k1 < NK; ++k1) {
#pragma unroll
      for (int k2 = k1; k2 < NK; ++k2) {
        if (p % (8 * E) == 0) {
          const int ch = p / (8 * E);
          // the sums so far are formed here: else the compiler puts them off and keeps the
          // whole row in registers
#pragma unroll
          for (int k = 0; k < NK; ++k) asm volatile("" : "+v"(acc[k].x), "+v"(acc[k].y));
          wave_lds_sync();
#pragma unroll
          for (int i = 0; i < NLD; ++i) own[lane + 64 * i] = next[i];
          wave_lds_sync();
          if (ch + 1 < NCH) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
              const int pc = (ch + 1) * 8 + ((lane & 7) ^ ((((lane >> 3) + 8 * i) >> 1) & 7));
              if ((ch + 2) * 8 <= PPR || pc < PPR)
                next[i] = *reinterpret_cast<const PieceU*>(src[i] + zero + (ch + 1) * 8 * E);
            }
          }
        }
        if (p % E == 0) cur = mine[(p / E % 8) ^ swz];
        const T av = cur[p % E];
        ++p;
        acc[k1].x += av * b[k2].x;
        acc[k1].y += av * b[k2].y;
        if (k2 != k1) {
          acc[k2].x += av * b[k1].x;
          acc[k2].y += av * b[k1].y;
        }
      }
    }
    if (!act) continue;
    // (addresses formed again, not kept in registers since the loads)
    int64_t w0 = st0, w1 = st1;
    asm volatile("" : "+v"(w0), "+v"(w1));
#pragma unroll
    for (int g = 0; g < NK / 2; ++g) {
      V z, zc;
      pack_pair(acc[2 * g], acc[2 * g + 1], dd, &z, &zc);
      Cs[g * a.pair_stride + w0] = z;
      if (w1 != w0) Cs[g * a.pair_stride + w1] = zc;
    }
  }
}

// Step 3 with the rows of A in low-rank form (rem:step3, last paragraph):
// A(|n|^2) ~ sum_a R_a R_a', rank_r = (off[r+1] - off[r]) / NK factors of NK
// entries each.  a = R (R' b): 2 rank NK multiply-adds per complex value
// instead of NK^2.  Orthant points and sign patterns as in mode_radial_kernel.
template <typename T, int NK>
__global__ __launch_bounds__(kThreads) void mode_lowrank_kernel(
    RadialArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ Rtab,
    const int64_t* __restrict__ off, const int* __restrict__ rowidx, const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  const int64_t tid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (tid >= a.Q) return;
  const int64_t M1 = a.M + 1;
  int64_t an[3] = {0, 0, 0};
  {
    int64_t q = tid;
    for (int r = 0; r < a.d; ++r) {
      an[r] = q % M1;
      q /= M1;
    }
  }
  const int64_t s2 = an[0] * an[0] + an[1] * an[1] + an[2] * an[2];
  const int64_t row = a.d == 1 ? an[0] : (int64_t)rowidx[s2];
  const T* Rr = Rtab + off[row];
  const int rank = (int)((off[row + 1] - off[row]) / NK);
  T D = T(1);
  for (int r = 0; r < a.d; ++r) D *= dec[r * M1 + an[r]];
  int first_nz = -1;
  for (int r = 0; r < a.d; ++r)
    if (an[r] != 0) {
      first_nz = r;
      break;
    }
  const int npat = 1 << (a.d - 1);
  for (int set = 0; set < a.nsets; ++set)
  for (int pg = 0; pg < npat; pg += 2) {
    V* __restrict__ Cs = C + set * a.set_stride;
    bool keep[2];
    int64_t st0[2], st1[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int pat = pg + h;
      keep[h] = pat < npat;
      int64_t nv[3] = {0, 0, 0}, nvc[3] = {0, 0, 0};
      for (int r = 0; r < a.d; ++r) {
        const int neg = r == 0 ? 0 : ((pat >> (r - 1)) & 1);
        if (neg && (an[r] == 0 || r == first_nz)) keep[h] = false;
        nv[r] = neg ? -an[r] : an[r];
        nvc[r] = -nv[r];
      }
      st0[h] = keep[h] ? radial_store(a, nv) : 0;
      st1[h] = keep[h] ? radial_store(a, nvc) : 0;
    }
    if (!keep[0] && !keep[1]) continue;
    V b[2][NK];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int g = 0; g < NK / 2; ++g) {
        V z = V{T(0), T(0)}, zc = V{T(0), T(0)};
        if (keep[h] && g < a.npair) {
          z = Cs[g * a.pair_stride + st0[h]];
          zc = Cs[g * a.pair_stride + st1[h]];
        }
        b[h][2 * g] = V{T(0.5) * (z.x + zc.x) * D, T(0.5) * (z.y - zc.y) * D};
        b[h][2 * g + 1] = V{T(0.5) * (z.y + zc.y) * D, T(-0.5) * (z.x - zc.x) * D};
      }
    V acc[2][NK];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < NK; ++k) acc[h][k] = V{T(0), T(0)};
    for (int f = 0; f < rank; ++f) {
      const T* ra = Rr + (int64_t)f * NK;
      T rv[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) rv[k] = ra[k];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        V t = V{T(0), T(0)};
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          t.x += rv[k] * b[h][k].x;
          t.y += rv[k] * b[h][k].y;
        }
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          acc[h][k].x += rv[k] * t.x;
          acc[h][k].y += rv[k] * t.y;
        }
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!keep[h]) continue;
#pragma unroll
      for (int g = 0; g < NK / 2; ++g) {
        if (g >= a.npair) break;
        const V pp = V{acc[h][2 * g].x * D, acc[h][2 * g].y * D};
        const V qq = V{acc[h][2 * g + 1].x * D, acc[h][2 * g + 1].y * D};
        Cs[g * a.pair_stride + st0[h]] = V{pp.x - qq.y, pp.y + qq.x};
        if (st1[h] != st0[h]) Cs[g * a.pair_stride + st1[h]] = V{pp.x + qq.y, -pp.y + qq.x};
      }
    }
  }
}

// d = 1: the M+1 orthant points are too few to fill the chip one per thread,
// so each point takes a group of NK lanes: lane j forms b_j, computes row j
// of A b (terms in the order k = 0..NK-1, as the per-thread kernel adds them),
// and lanes g < npair write the conjugate pair (n, -n) of grid g.
template <typename T, int NK>
__global__ __launch_bounds__(kThreads) void mode_radial_1d_kernel(
    RadialArgs a, typename V2<T>::type* __restrict__ C, const T* __restrict__ Atab,
    const T* __restrict__ dec) {
  using V = typename V2<T>::type;
  constexpr int NP = NK * (NK + 1) / 2;
  constexpr int PPB = kThreads / NK;  // points per workgroup
  __shared__ V sb[PPB][NK];
  __shared__ V sa[PPB][NK];
  const int lp = threadIdx.x / NK, j = threadIdx.x % NK;
  // Four-step grids hold mode k = k2 + L2 k1 at k2 L1 + k1: the points are dealt along k1,
  // so that neighbours in a block are neighbours in memory (the table's rows
  // are long enough to be read in any order).  In the order of n every access was a
  // line of its own: d=1 nf=49152, 12 grids 15.2 -> 11.8 us, fp32 12.9 -> 9.3.
  const int q = (int)blockIdx.x * PPB + lp;
  const int L1 = (int)a.L1, L2 = (int)a.L2, nk1 = a.fourstep ? (int)a.M / L2 + 1 : 1;
  const int k2 = a.fourstep ? q / nk1 : q, k1 = q - k2 * nk1;
  const int n0 = a.fourstep ? k2 + L2 * k1 : q;
  const bool act = lp < PPB && n0 <= (int)a.M && (!a.fourstep || k2 < L2);
  int64_t st0 = 0, st1 = 0;
  T D = T(0);
  if (act) {
    if (!a.fourstep) {
      st0 = a.M + n0;
      st1 = a.M - n0;
    } else {  // -n is mode L1 L2 - n
      st0 = (int64_t)k2 * L1 + k1;
      st1 = n0 == 0 ? 0 : (k2 > 0 ? (int64_t)(L2 - k2) * L1 + (L1 - 1 - k1) : L1 - k1);
    }
    D = dec[n0];
    const int g = j / 2;
    V z = V{T(0), T(0)}, zc = V{T(0), T(0)};
    if (g < a.npair) {
      z = C[g * a.pair_stride + st0];
      zc = C[g * a.pair_stride + st1];
    }
    sb[lp][j] = (j & 1) ? V{T(0.5) * (z.y + zc.y) * D, T(-0.5) * (z.x - zc.x) * D}
                        : V{T(0.5) * (z.x + zc.x) * D, T(0.5) * (z.y - zc.y) * D};
  }
  __syncthreads();
  if (act) {
    const T* Ar = Atab + (int64_t)n0 * NP;
    V acc = V{T(0), T(0)};
#pragma unroll 8
    for (int k = 0; k < NK; ++k) {
      const int lo = min(j, k), hi = max(j, k);
      const T av = Ar[lo * NK - lo * (lo - 1) / 2 + (hi - lo)];
      acc.x += av * sb[lp][k].x;
      acc.y += av * sb[lp][k].y;
    }
    sa[lp][j] = acc;
  }
  __syncthreads();
  if (act && j < a.npair) {
    const V pp = V{sa[lp][2 * j].x * D, sa[lp][2 * j].y * D};
    const V qq = V{sa[lp][2 * j + 1].x * D, sa[lp][2 * j + 1].y * D};
    C[j * a.pair_stride + st0] = V{pp.x - qq.y, pp.y + qq.x};
    if (st1 != st0) C[j * a.pair_stride + st1] = V{pp.x + qq.y, -pp.y + qq.x};
  }
}

template <typename T, int NK>
void launch_mode_nk(Plan* P) {
  PhaseScope ps(P, PH_MODE);
  ModeArgs a;
  a.d = P->d;
  a.M = P->M;
  a.mc = P->mcount;
  a.mp = P->mp;
  a.F = 1;
  for (int r = 0; r < P->d; ++r) a.F *= a.mc;
  a.nk = P->nk;
  a.npair = P->npair;
  a.nt = P->nt_eff;
  a.fourstep = P->fourstep;
  a.nf = P->nf[0];
  a.L1 = P->L1;
  a.L2 = P->L2;
  a.pair_stride = P->grid_elems[3];
  const int64_t half = (a.F + 1) / 2;
  for (int set = 0; set < P->gv.nsets; ++set) {
    hipLaunchKernelGGL((mode_kernel<T, NK>), dim3((unsigned)((half + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, P->stream, a,
                       static_cast<typename V2<T>::type*>(P->gv.C) + set * P->npair * a.pair_stride,
                       P->gtab.as<T>(), P->etab.as<T>(), P->vtd.as<T>(), P->dec.as<T>());
    GP_CHECK_LAUNCH();
  }
}

template <typename T, int NK>
void launch_radial_nk(Plan* P) {
  PhaseScope ps(P, PH_MODE);
  RadialArgs a;
  a.d = P->d;
  a.M = P->M;
  a.mc = P->mcount;
  a.mp = P->mp;
  a.Q = 1;
  for (int r = 0; r < P->d; ++r) a.Q *= (P->M + 1);
  a.npair = P->npair;
  a.fourstep = P->fourstep;
  a.nf = P->nf[0];
  a.L1 = P->L1;
  a.L2 = P->L2;
  a.pair_stride = P->grid_elems[3];
  a.nsets = P->gv.nsets;
  a.set_stride = P->npair * a.pair_stride;
  a.tiles = nullptr;
  a.ntx = 0;
  auto* C = static_cast<typename V2<T>::type*>(P->gv.C);
  if (P->step3 == 2) {
    hipLaunchKernelGGL((mode_lowrank_kernel<T, NK>), dim3((unsigned)((a.Q + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, P->stream, a, C, P->atab.as<T>(), P->lr_off.as<int64_t>(),
                       P->d > 1 ? P->rowidx.as<int>() : nullptr, P->dec.as<T>());
    GP_CHECK_LAUNCH();
    return;
  }
  if (P->d == 1) {
    constexpr int PPB = kThreads / NK;
    const int64_t np = a.fourstep ? a.L2 * (a.M / a.L2 + 1) : a.Q;
    for (int set = 0; set < a.nsets; ++set) {
      hipLaunchKernelGGL((mode_radial_1d_kernel<T, NK>), dim3((unsigned)((np + PPB - 1) / PPB)),
                         dim3(kThreads), 0, P->stream, a, C + set * a.set_stride,
                         P->atab.as<T>(), P->dec.as<T>());
      GP_CHECK_LAUNCH();
    }
    return;
  }
  // 2-D: orthant tiles nearest the origin first (the table rows in use then
  // form a band that stays in the caches)
  if (P->d == 2) {
    a.tiles = P->mode_tiles.as<int>();
    a.ntx = P->mode_ntx;
  }
  // lanes: threads per orthant point
  auto go = [&](auto kern, int lanes) {
    const int64_t ppb = kThreads / lanes;
    const int64_t nblk = P->d == 2 ? lanes * P->mode_ntx * (P->M / kModeTileY + 1) : (a.Q + ppb - 1) / ppb;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(kThreads), 0, P->stream, a, C, P->atab.as<T>(),
                       P->rowidx.as<int>(), P->dec.as<T>());
    GP_CHECK_LAUNCH();
  };
  // The measured sides of this rule are at mode_rows_kernel.
  if constexpr (sizeof(T) == 8) {
    if (P->d == 3) go(mode_rows_kernel<T, NK, 3>, 4);
    else if (a.nsets == 1) go(mode_rows_kernel<T, NK, 2>, 2);
    else go(mode_radial2_kernel<T, NK>, 2);
  } else {
    go(mode_radial_kernel<T, NK>, 1);
  }
}

template <typename T>
void launch_mode(Plan* P) {
  const int nk2 = 2 * P->npair;
  if (P->step3 != 1) {
    switch (nk2) {
#define GP_R(N) case N: launch_radial_nk<T, N>(P); return;
      GP_R(2) GP_R(4) GP_R(6) GP_R(8) GP_R(10) GP_R(12) GP_R(14) GP_R(16) GP_R(18) GP_R(20)
      GP_R(22) GP_R(24) GP_R(26) GP_R(28) GP_R(30) GP_R(32) GP_R(34) GP_R(36) GP_R(38) GP_R(40)
      GP_R(42) GP_R(44) GP_R(46) GP_R(48)
#undef GP_R
      default:
        throw Error{GP_EUNSUPPORTED, "too many Chebyshev nodes"};
    }
  }
  switch (nk2) {
#define GP_M(N) case N: launch_mode_nk<T, N>(P); break;
    GP_M(2) GP_M(4) GP_M(6) GP_M(8) GP_M(10) GP_M(12) GP_M(14) GP_M(16) GP_M(18) GP_M(20)
    GP_M(22) GP_M(24) GP_M(26) GP_M(28) GP_M(30) GP_M(32) GP_M(34) GP_M(36) GP_M(38) GP_M(40)
    GP_M(42) GP_M(44) GP_M(46) GP_M(48)
#undef GP_M
    default:
      throw Error{GP_EUNSUPPORTED, "too many Chebyshev nodes"};
  }
}

}  // namespace

// Compiled twice (GP_MODE_FP64 = 1 / 0) so the two precisions build in parallel.
#if GP_MODE_FP64
#define GP_MODE_T double
#define GP_MIX_FN mix_modes_fp64
#else
#define GP_MODE_T float
#define GP_MIX_FN mix_modes_fp32
#endif

void GP_MIX_FN(Plan* P) {
  launch_mode<GP_MODE_T>(P);
}

}  // namespace gp
