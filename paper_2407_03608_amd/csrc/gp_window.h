// Sum of a point's window over staged grid cells (type-2 interpolation), for the
// device and, in the tests, for the host.
#pragma once

#include <type_traits>

#ifdef __HIPCC__
#define GP_WINDOW_FN __device__ __forceinline__
#define GP_WINDOW_UNROLL _Pragma("unroll")
#else
#define GP_WINDOW_FN inline
#define GP_WINDOW_UNROLL
#endif

namespace gp {

// i-th place of a window of W values, from the ends to the middle (ON) or in order
template <bool ON, int W>
GP_WINDOW_FN constexpr int ends_first(int i) {
  return !ON ? i : (i % 2 ? W - 1 - i / 2 : i / 2);
}

// Window values p0, p1 (, p2) of a point on the cells tr: rows of W cells S1 apart,
// planes S2 apart in 3-D (2-D: S2 = S1).  The lane takes every RG-th row (2-D) or plane
// (3-D), HP of them with the values p1 or p2, the last at tr + last.
//
// fp32 grids: the sum errs no more than that of four lanes' quarters of the rows,
// each added in fp32 and joined in fp64, which this order took the place of.  2-D joins
// rows in fp64 (no slower).  3-D adds from the window's ends to its middle, the small
// values first, and joins two chains of planes (w < 4: every plane) in fp64; ROWS
// joins every row in fp64, for the widths and plans whose rows always were.  Error in
// units of 2^-24 of the result on smooth / random grids, w = 5: in order and all in
// fp32 0.97 / 1.28, quarters 0.69 / 1.16, now 0.61 / 0.87; w = 7 1.13 / 1.46, 0.81 / 1.43,
// 0.60 / 0.90.  Time at d=3 N=1e7 (w = 5): 2.03 ms, all in fp32 2.00; every plane joined in
// fp64 2.17, every row 3.06.  fp64 grids are added in order.
template <typename T, typename V, int D, int W, int HP, int RG, int S1, int S2, bool ROWS>
GP_WINDOW_FN void window_sum(const V* tr, int last, const T (&p0)[W], const T (&p1)[D > 2 ? W : HP],
                             const T (&p2)[D > 2 ? HP : 1], double* bx, double* by) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr bool S64 = D == 2 || ROWS || W < 4;
  using Plane = std::conditional_t<ROWS || W < 3, double, T>;  // sum of a plane's rows (3-D)
  using Sum = std::conditional_t<S64, double, T>;  // of rows (2-D) or planes
  constexpr int NSUM = S64 || !F32 ? 1 : 2;        // chains, joined in fp64
  Sum sx[NSUM] = {}, sy[NSUM] = {};
  GP_WINDOW_UNROLL
  for (int i = 0; i < HP; ++i) {
    const int j = ends_first<F32 && (D > 2), HP>(i);
    const V* tp = tr + (j + 1 < HP ? RG * j * S2 : last);
    if constexpr (D > 2) {
      Plane ax = 0, ay = 0;
      GP_WINDOW_UNROLL
      for (int i1 = 0; i1 < W; ++i1) {
        const int q1 = ends_first<F32, W>(i1);
        T rx = 0, ry = 0;
        GP_WINDOW_UNROLL
        for (int i0 = 0; i0 < W; ++i0) {
          const int q0 = ends_first<F32 && !ROWS, W>(i0);
          const V gv = tp[q1 * S1 + q0];
          rx += p0[q0] * gv.x;
          ry += p0[q0] * gv.y;
        }
        ax += (Plane)p1[q1] * (Plane)rx;
        ay += (Plane)p1[q1] * (Plane)ry;
      }
      sx[i % NSUM] += (Sum)p2[j] * (Sum)ax;
      sy[i % NSUM] += (Sum)p2[j] * (Sum)ay;
    } else {
      T rx = 0, ry = 0;
      GP_WINDOW_UNROLL
      for (int q0 = 0; q0 < W; ++q0) {
        const V gv = tp[q0];
        rx += p0[q0] * gv.x;
        ry += p0[q0] * gv.y;
      }
      sx[0] += (Sum)p1[j] * (Sum)rx;
      sy[0] += (Sum)p1[j] * (Sum)ry;
    }
  }
  *bx = (double)sx[0];
  *by = (double)sy[0];
  if constexpr (NSUM > 1) {
    *bx += (double)sx[1];
    *by += (double)sy[1];
  }
}

}  // namespace gp
