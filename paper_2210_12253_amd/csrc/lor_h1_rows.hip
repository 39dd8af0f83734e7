// H1 values row by row (lor_rows.hpp).
//
// What bounds it: vector issue, about 1,400 instructions per cell and row, 65% of
// the SIMD's cycles at two waves per SIMD: 0.43 us per 1,000 cells, after about 10
// us.  Triangle-split meshes, FP64, against the coloured kernel: p = 2, 384
// elements 21 us against 126; p = 4, 216 elements 21 against 146; p = 2, 30,720
// elements 135 against 179; p = 4, 7,200 elements (461,000 cells) 214 against 207.
// Four lanes per row: with eight, a wave adds to half as many rows per serial
// step (p = 4, 7,200 elements: 254 us), and two would need 32 KB of LDS per wave.
#include "lor_h1_math.hpp"
#include "lor_rows.hpp"

namespace lor {

template <int P>
struct H1Rows {
  static constexpr int LANES = 4, NE = 8, WPE = 2;
  static constexpr int Q = P + 1, NSUB = P * P * P, NLOC = Q * Q * Q, T1 = 3 * P + 1;
  // cells along one axis around lattice coordinate t
  static __device__ __forceinline__ int cells1(int t) { return t > 0 && t < P ? 2 : 1; }
  static __device__ __forceinline__ int cells(int l) {
    return cells1(l % Q) * cells1((l / Q) % Q) * cells1(l / (Q * Q));
  }
  template <typename T>
  static __device__ __forceinline__ void cell(const RowArgs& g, const T* __restrict__ kappa, int e, int l, int nth,
                                              int (&at)[NE], double (&en)[NE]) {
    const int x = l % Q, y = (l / Q) % Q, z = l / (Q * Q);
    // the nth corner u = a + 2b + 4c that leaves the cell inside the element
    const int n2 = cells1(x), n1 = cells1(y);
    const int a = n2 == 2 ? nth & 1 : (x == P);
    const int r1 = n2 == 2 ? nth >> 1 : nth;
    const int b = n1 == 2 ? r1 & 1 : (y == P);
    const int r2 = n1 == 2 ? r1 >> 1 : r1;
    const int c = z > 0 && z < P ? r2 & 1 : (z == P);
    const int u = a + 2 * b + 4 * c;
    const int sx = x - a, sy = y - b, sz = z - c;
    // entry (dx, dy, dz) of local row l in the element's rank table
    {
      const uint8_t* tab = g.tables + static_cast<int64_t>(g.elem_class[e]) * g.tab_stride;
      auto cnt = [](int t) { return t == 0 || t == P ? 2 : 3; };
      auto pre = [](int t) { return t == 0 ? 0 : 3 * t - 1; };
      const int nx = cnt(x), ny = cnt(y), nz = cnt(z);
      const int base = pre(z) * T1 * T1 + nz * pre(y) * T1 + nz * ny * pre(x) + ((z > 0 ? 1 : 0) - c) * nx * ny +
                       ((y > 0 ? 1 : 0) - b) * nx + (x > 0 ? 1 : 0) - a;
#pragma unroll
      for (int v = 0; v < 8; ++v) at[v] = tab[base + (v >> 2) * nx * ny + ((v >> 1) & 1) * nx + (v & 1)] & kRankMask;
    }
    const double kap = static_cast<double>(kappa[static_cast<int64_t>(e) * NSUB + sx + P * (sy + P * sz)]);
    double ex[2][2][3], ey[2][2][3], ez[2][2][3];
    {
      double X[8][3];
      row_corners<Q>(g, e, sx, sy, sz, X);
      h1_edges<double>(X, ex, ey, ez);
      if constexpr (sizeof(T) == 4) {
        if (g.diag && u == 0 && (g.flags & LOR_FP64_FALLBACK)) {
          float fx[2][2][3], fy[2][2][3], fz[2][2][3], dmin, dmax;
          h1_edges<float>(X, fx, fy, fz);
          h1_corner_det_range<float>(fx, fy, fz, dmin, dmax);
          if (!(dmin > 0.0f) || dmax > g.det_thresh * dmin) atomicAdd(&g.diag[0], 1);
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 8; ++v) en[v] = 0.0;
    const bool ok = h1_cell<double>(ex, ey, ez, kap, g.beta, [&](int i, double w) {
#pragma unroll
      for (int m = 0; m < 8; ++m)
#pragma unroll
        for (int v = 0; v < 8; ++v)
          if (pair_index(m, v) == i) en[v] = u == m ? w : en[v];
    });
    if (!ok && g.diag && u == 0) atomicAdd(&g.diag[1], 1);
  }
};

LOR_ROWS_DISPATCH(dispatch_h1_rows, H1Rows)

}  // namespace lor
