// H(div) values row by row (lor_rows.hpp).
//
// What bounds it: three dependent loads and about 900 vector instructions per
// cell and row, little overlapped at two waves per SIMD (192 registers; at three
// it spills 49 and is 1.7 times slower): 0.35 us per 1,000 cells after about 10 us.
// Triangle-split meshes, FP64, against the coloured kernel: p = 2, 384 elements
// 10.6 us against 27.1; p = 1, 138,240 elements 49 against 69; p = 3, 7,200
// elements (194,000 cells) 69 against 61.
#include "lor_rows.hpp"
#include "lor_rt_math.hpp"

namespace lor {

template <int P>
struct RTRows {
  static constexpr int LANES = 2, NE = 6, WPE = 2;
  static constexpr int Q = P + 1, NSUB = P * P * P, NDIR = P * P * Q, NLOC = 3 * NDIR;
  // direction and lattice position of local face l: x-faces i + q (j + p k),
  // y-faces i + p (j + q k), z-faces i + p (j + p k)
  static __device__ __forceinline__ int decode(int l, int (&pos)[3]) {
    const int d = l / NDIR, r = l - d * NDIR;
    const int n0 = d == 0 ? Q : P, n1 = d == 1 ? Q : P;
    pos[0] = r % n0;
    pos[1] = (r / n0) % n1;
    pos[2] = r / (n0 * n1);
    return d;
  }
  static __device__ __forceinline__ int along(int d, const int (&pos)[3]) {
    return d == 0 ? pos[0] : d == 1 ? pos[1] : pos[2];
  }
  static __device__ __forceinline__ int cells(int l) {
    int pos[3];
    const int d = decode(l, pos), t = along(d, pos);
    return t > 0 && t < P ? 2 : 1;
  }
  template <typename T>
  static __device__ __forceinline__ void cell(const RowArgs& g, const T* __restrict__ kappa, int e, int l, int nth,
                                              int (&at)[NE], double (&en)[NE]) {
    int pos[3];
    const int d = decode(l, pos), t = along(d, pos);
    const int side = t > 0 && t < P ? nth : (t == P);  // the face's side in the cell
    const int u = 2 * d + side;
    const int off[3] = {d == 0 ? side : 0, d == 1 ? side : 0, d == 2 ? side : 0};
    const int sx = pos[0] - off[0], sy = pos[1] - off[1], sz = pos[2] - off[2];
    // The table entries of local face l are the faces of its element's cells
    // beside it, x-faces, y-faces, z-faces, each in (z, y, x) order over per-axis
    // ranges: along d the nodes (faces along d) or cells next to the face, along
    // the others one cell, or its two nodes for the faces along that axis.
    {
      const uint8_t* tab = g.tables + static_cast<int64_t>(g.elem_class[e]) * g.tab_stride + g.st_ptr[l];
      const int lo = t > 0 ? 1 : 0, hi = t < P ? 1 : 0;
      int cn[3], cc[3], q[3];  // nodes and cells in each range; the cell's place in it
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        cn[m] = m == d ? 1 + lo + hi : 2;
        cc[m] = m == d ? lo + hi : 1;
        q[m] = m == d ? lo - side : 0;
      }
      const int off1 = cn[0] * cc[1] * cc[2], off2 = off1 + cc[0] * cn[1] * cc[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        at[s] = tab[(q[2] * cc[1] + q[1]) * cn[0] + q[0] + s] & kRankMask;
        at[2 + s] = tab[off1 + (q[2] * cn[1] + q[1] + s) * cc[0] + q[0]] & kRankMask;
        at[4 + s] = tab[off2 + ((q[2] + s) * cc[1] + q[1]) * cc[0] + q[0]] & kRankMask;
      }
    }
    unsigned neg = 0;  // bit v set if local face v is reversed
    {
      const int32_t* fm = g.elem_map + static_cast<int64_t>(e) * NLOC;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        neg |= (fm[(sx + s) + Q * (sy + P * sz)] < 0 ? 1u : 0u) << s;
        neg |= (fm[NDIR + sx + P * ((sy + s) + Q * sz)] < 0 ? 1u : 0u) << (2 + s);
        neg |= (fm[2 * NDIR + sx + P * (sy + P * (sz + s))] < 0 ? 1u : 0u) << (4 + s);
      }
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
    RTFactors<double> F;
    const bool ok = rt_factors<double>(ex, ey, ez, kap, g.beta, F);
    if (!ok && g.diag && u == 0) atomicAdd(&g.diag[1], 1);
    const unsigned sr = neg >> u & 1u;
#pragma unroll
    for (int v = 0; v < NE; ++v) {
      double w = 0.0;
#pragma unroll
      for (int r = 0; r < NE; ++r) w = u == r ? rt_entry<double>(F, r < v ? r : v, r < v ? v : r) : w;
      const uint64_t flip = static_cast<uint64_t>((neg >> v & 1u) ^ sr) << 63;
      en[v] = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, w) ^ flip);
    }
  }
};

LOR_ROWS_DISPATCH(dispatch_rt_rows, RTRows)

}  // namespace lor
