// H(curl) values row by row (lor_rows.hpp).
//
// What bounds it: about 2,000 vector instructions per cell and row at one wave per
// SIMD (the 84 factors of all 78 entries and the geometry need 400 registers; at
// two waves it spills 215): 1.85 us per 1,000 cells after about 15 us.
// Triangle-split meshes, FP64, against the coloured kernel: p = 3, 72 elements 19
// us against 118; p = 2, 384 elements 22 against 147; p = 1, 138,240 elements 284
// against 251.
#include "lor_nd_math.hpp"
#include "lor_rows.hpp"

namespace lor {

template <int P>
struct NDRows {
  static constexpr int LANES = 4, NE = 12, WPE = 1;
  static constexpr int Q = P + 1, NSUB = P * P * P, NDIR = P * Q * Q, NLOC = 3 * NDIR;
  // direction and lattice position of local edge l: x-edges i + p (j + q k),
  // y-edges i + q (j + p k), z-edges i + q (j + q k)
  static __device__ __forceinline__ int decode(int l, int (&pos)[3]) {
    const int d = l / NDIR, r = l - d * NDIR;
    const int n0 = d == 0 ? P : Q, n1 = d == 1 ? P : Q;
    pos[0] = r % n0;
    pos[1] = (r / n0) % n1;
    pos[2] = r / (n0 * n1);
    return d;
  }
  static __device__ __forceinline__ int cells1(int t) { return t > 0 && t < P ? 2 : 1; }
  static __device__ __forceinline__ int cells(int l) {
    int pos[3];
    const int d = decode(l, pos);
    return (d == 0 ? 1 : cells1(pos[0])) * (d == 1 ? 1 : cells1(pos[1])) * (d == 2 ? 1 : cells1(pos[2]));
  }
  template <typename T>
  static __device__ __forceinline__ void cell(const RowArgs& g, const T* __restrict__ kappa, int e, int l, int nth,
                                              int (&at)[NE], double (&en)[NE]) {
    int pos[3];
    const int d = decode(l, pos);
    const int t1 = d == 0 ? pos[1] : pos[0], t2 = d == 2 ? pos[1] : pos[2];  // the two other axes
    const int n1 = cells1(t1);
    const int a = n1 == 2 ? nth & 1 : (t1 == P);
    const int r1 = n1 == 2 ? nth >> 1 : nth;
    const int b = t2 > 0 && t2 < P ? r1 & 1 : (t2 == P);
    const int u = 4 * d + a + 2 * b;
    const int off[3] = {d == 0 ? 0 : a, d == 0 ? a : (d == 1 ? 0 : b), d == 2 ? 0 : b};
    const int sx = pos[0] - off[0], sy = pos[1] - off[1], sz = pos[2] - off[2];
    // The table entries of local edge l are the edges of its element's cells
    // around it, x-edges, y-edges, z-edges, each in (z, y, x) order over per-axis
    // ranges: along d one cell (edges along d) or two nodes, along the others
    // the nodes (cells, for the edges along that axis) next to the edge.
    {
      const uint8_t* tab = g.tables + static_cast<int64_t>(g.elem_class[e]) * g.tab_stride + g.st_ptr[l];
      int lo[3], cn[3], cc[3];  // steps down to the range's start; nodes and cells in it
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        lo[m] = m != d && pos[m] > 0 ? 1 : 0;
        const int hi = m != d && pos[m] < P ? 1 : 0;
        cn[m] = m == d ? 2 : 1 + lo[m] + hi;
        cc[m] = m == d ? 1 : lo[m] + hi;
      }
      // cell's lower corner in the ranges (nodes and cells start at pos - lo)
      const int qx = lo[0] - off[0], qy = lo[1] - off[1], qz = lo[2] - off[2];
      const int off1 = cc[0] * cn[1] * cn[2], off2 = off1 + cn[0] * cc[1] * cn[2];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int p0 = s & 1, p1 = s >> 1;
        at[s] = tab[((qz + p1) * cn[1] + qy + p0) * cc[0] + qx] & kRankMask;
        at[4 + s] = tab[off1 + ((qz + p1) * cc[1] + qy) * cn[0] + qx + p0] & kRankMask;
        at[8 + s] = tab[off2 + (qz * cn[1] + qy + p1) * cn[0] + qx + p0] & kRankMask;
      }
    }
    // orientations of the cell's edges: bit v set if local edge v is reversed
    unsigned neg = 0;
    {
      const int32_t* em = g.elem_map + static_cast<int64_t>(e) * NLOC;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int p0 = s & 1, p1 = s >> 1;
        neg |= (em[sx + P * ((sy + p0) + Q * (sz + p1))] < 0 ? 1u : 0u) << s;
        neg |= (em[NDIR + (sx + p0) + Q * (sy + P * (sz + p1))] < 0 ? 1u : 0u) << (4 + s);
        neg |= (em[2 * NDIR + (sx + p0) + Q * ((sy + p1) + Q * sz)] < 0 ? 1u : 0u) << (8 + s);
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
    H1Factors<double> F;
    NDCurl<double> W;
    const bool ok = nd_factors<double>(ex, ey, ez, kap, g.beta, F, W);
    if (!ok && g.diag && u == 0) atomicAdd(&g.diag[1], 1);
    // the entries of edge u
#pragma unroll
    for (int v = 0; v < NE; ++v) en[v] = 0.0;
#pragma unroll
    for (int r = 0; r < NE; ++r)
#pragma unroll
      for (int v = r; v < NE; ++v) {
        const double w = nd_entry<double>(F, W, r, v);
        en[v] = u == r ? w : en[v];
        if (v != r) en[r] = u == v ? w : en[r];
      }
    const unsigned sr = neg >> u & 1u;
#pragma unroll
    for (int v = 0; v < NE; ++v) {
      const uint64_t flip = static_cast<uint64_t>((neg >> v & 1u) ^ sr) << 63;
      en[v] = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, en[v]) ^ flip);
    }
  }
};

LOR_ROWS_DISPATCH(dispatch_nd_rows, NDRows)

}  // namespace lor
