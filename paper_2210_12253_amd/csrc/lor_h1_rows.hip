// Values of the LOR H1 matrix, one row at a time (Step S1.2, any mesh).
//
// The coloured kernel (lor_h1.hip) integrates every cell once, but needs one
// launch per colour, and on a small mesh each launch is the latency of one
// group (about 11 us): 12 colours take 130 us whatever the mesh.  This kernel
// is one launch: kRowLanes lanes sum one row, each integrating its share of the
// cells around the row's vertex, so every cell is integrated by each of its
// eight corners, and every row is stored once, whole.
//
//   * The cells around a vertex follow from its incidences (element, local
//     vertex), sorted in the schedule: within an element, the cells at the
//     vertex's lattice point minus corner u, in increasing u.  That list is
//     dealt to the lanes in turn.
//   * A lane integrates its cell (the whole symmetric matrix, so that (i, j)
//     and (j, i) have the same bits) and takes the eight entries of its corner;
//     their places in the row come from the element's rank table.
//   * The lanes then add their entries to the row in LDS one after another, in
//     the order of the list.  The order within an element is decreasing in the
//     cell's position, and increasing in the element across elements, for both
//     rows of an entry: the matrix is bitwise symmetric and repeatable.
// All arithmetic is FP64, whatever the type of the values (FP64 and unpacked
// FP32 instructions issue at the same rate), and every entry is rounded once.
//
// What bounds it: vector issue, about 1,400 instructions per cell and row, 65% of
// the SIMD's cycles at two waves per SIMD: 0.43 us per 1,000 cells, after about 10
// us.  Triangle-split meshes, FP64, against the coloured kernel: p = 2, 384
// elements 21 us against 126; p = 4, 216 elements 21 against 146; p = 2, 30,720
// elements 135 against 179; p = 4, 7,200 elements (461,000 cells) 214 against 207.
// Four lanes per row: with eight, a wave adds to half as many rows per serial
// step (p = 4, 7,200 elements: 254 us), and two would need 32 KB of LDS per wave.
#include "lor_common.hpp"
#include "lor_h1_math.hpp"

namespace lor {

constexpr int kRowLanes = 4;                      // lanes per row
constexpr int kRowThreads = 256;
constexpr int kRowsPerWg = kRowThreads / kRowLanes;
constexpr int kRowStride = LOR_MAX_ROW_NNZ;       // odd: rows start in different banks
static_assert(kRowStride % 2 == 1, "row stride in LDS");

template <int P, typename T>
__global__ __launch_bounds__(kRowThreads, 2) void k_h1_rows(
    const int32_t* __restrict__ inc_ptr, const int32_t* __restrict__ inc_list, const int32_t* __restrict__ elem_class,
    const uint8_t* __restrict__ tables, int64_t tab_stride, const int32_t* __restrict__ elem_dofs,
    const double* __restrict__ coords, const T* __restrict__ kappa, T beta, const int32_t* __restrict__ row_ptr,
    int64_t nrows, int64_t nel, int64_t nnz, T* __restrict__ values, unsigned flags, float det_thresh,
    int32_t* __restrict__ diag) {
  constexpr int Q = P + 1, NSUB = P * P * P, NLOC = Q * Q * Q, T1 = 3 * P + 1;
  __shared__ double sRow[kRowsPerWg * kRowStride];
  const int tid = threadIdx.x, k = tid % kRowLanes;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * kRowsPerWg + tid / kRowLanes;
  kappa += static_cast<int64_t>(blockIdx.y) * nel * NSUB;
  values += static_cast<int64_t>(blockIdx.y) * nnz;
  const bool live = row < nrows;
  const int32_t first = live ? inc_ptr[row] : 0, ninc = live ? inc_ptr[row + 1] - first : 0;
  const int32_t start = live ? row_ptr[row] : 0, rlen = live ? row_ptr[row + 1] - start : 0;
  const int32_t len = rlen < kRowStride ? rlen : kRowStride;
  double* const acc = sRow + (tid / kRowLanes) * kRowStride;
  for (int j = k; j < len; j += kRowLanes) acc[j] = 0.0;

  // lattice point of a local vertex, and the number of cells of the element
  // around it along one axis
  auto cells1 = [](int t) { return t > 0 && t < P ? 2 : 1; };
  for (int i0 = 0; __ballot(i0 < ninc) != 0; i0 += kRowLanes) {
    // this lane's incidence of the next kRowLanes, and the number of cells
    // before its own in the list
    const int32_t inc = i0 + k < ninc ? inc_list[first + i0 + k] : 0;
    int mine = 0;
    if (i0 + k < ninc) {
      const int l = inc % NLOC;
      mine = cells1(l % Q) * cells1((l / Q) % Q) * cells1(l / (Q * Q));
    }
    int before = mine;
#pragma unroll
    for (int m = 1; m < kRowLanes; m <<= 1) {
      const int t = __shfl_up(before, m, kRowLanes);
      if (k >= m) before += t;
    }
    const int total = __shfl(before, kRowLanes - 1, kRowLanes);
    before -= mine;
    for (int o0 = 0; __ballot(o0 < total) != 0; o0 += kRowLanes) {
      // cell number o0 + k of the list: its incidence, and its number there
      const int o = o0 + k;
      int32_t einc = 0;
      int nth = 0;
#pragma unroll
      for (int j = 0; j < kRowLanes; ++j) {
        const int32_t ij = __shfl(inc, j, kRowLanes);
        const int bj = __shfl(before, j, kRowLanes), mj = __shfl(mine, j, kRowLanes);
        if (o >= bj && o < bj + mj) {
          einc = ij;
          nth = o - bj;
        }
      }
      const bool have = o < total;
      double e8[8];
      int32_t at[8];
      if (have) {
        const int e = einc / NLOC, l = einc - e * NLOC;
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
        // places of the row's entries towards the cell's corners: entry
        // (dx, dy, dz) of local row l in the element's rank table
        {
          const uint8_t* tab = tables + static_cast<int64_t>(elem_class[e]) * tab_stride;
          auto cnt = [](int t) { return t == 0 || t == P ? 2 : 3; };
          auto pre = [](int t) { return t == 0 ? 0 : 3 * t - 1; };
          const int nx = cnt(x), ny = cnt(y), nz = cnt(z);
          const int base = pre(z) * T1 * T1 + nz * pre(y) * T1 + nz * ny * pre(x) +
                           ((z > 0 ? 1 : 0) - c) * nx * ny + ((y > 0 ? 1 : 0) - b) * nx + (x > 0 ? 1 : 0) - a;
#pragma unroll
          for (int v = 0; v < 8; ++v)
            at[v] = tab[base + (v >> 2) * nx * ny + ((v >> 1) & 1) * nx + (v & 1)] & kRankMask;
        }
        const double kap = static_cast<double>(kappa[static_cast<int64_t>(e) * NSUB + sx + P * (sy + P * sz)]);
        double ex[2][2][3], ey[2][2][3], ez[2][2][3];
        {
          const int32_t* ed = elem_dofs + static_cast<int64_t>(e) * NLOC + sx + Q * (sy + Q * sz);
          int32_t g[8];
#pragma unroll
          for (int v = 0; v < 8; ++v) g[v] = ed[(v & 1) + Q * (((v >> 1) & 1) + Q * (v >> 2))];
          double X[8][3];
#pragma unroll
          for (int v = 0; v < 8; ++v)
#pragma unroll
            for (int d = 0; d < 3; ++d) X[v][d] = coords[3 * static_cast<int64_t>(g[v]) + d];
          h1_edges<double>(X, ex, ey, ez);
          if constexpr (sizeof(T) == 4) {
            if (diag && u == 0 && (flags & LOR_FP64_FALLBACK)) {
              float fx[2][2][3], fy[2][2][3], fz[2][2][3], dmin, dmax;
              h1_edges<float>(X, fx, fy, fz);
              h1_corner_det_range<float>(fx, fy, fz, dmin, dmax);
              if (!(dmin > 0.0f) || dmax > det_thresh * dmin) atomicAdd(&diag[0], 1);
            }
          }
        }
        // the eight entries of corner u
#pragma unroll
        for (int v = 0; v < 8; ++v) e8[v] = 0.0;
        const bool ok = h1_cell<double>(ex, ey, ez, kap, static_cast<double>(beta), [&](int i, double w) {
#pragma unroll
          for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int v = 0; v < 8; ++v)
              if (pair_index(m, v) == i) e8[v] = u == m ? w : e8[v];
        });
        if (!ok && diag && u == 0) atomicAdd(&diag[1], 1);
      }
      // into the row, one lane after another
#pragma unroll 1
      for (int j = 0; j < kRowLanes; ++j) {
        if (have && k == j) {
          double t[8];
#pragma unroll
          for (int v = 0; v < 8; ++v) t[v] = acc[at[v]];
#pragma unroll
          for (int v = 0; v < 8; ++v) acc[at[v]] = t[v] + e8[v];
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  for (int j = k; j < len; j += kRowLanes) values[static_cast<int64_t>(start) + j] = static_cast<T>(acc[j]);
}

template <int P, typename T>
static int launch_rows(const lor_sched* s, int batch, const int32_t* ed, const double* x, const void* kappa,
                       double beta, const int32_t* rp, void* values, unsigned flags, double thr, int32_t* diag,
                       hipStream_t st) {
  const int64_t wgs = ceil_div(s->nrows, kRowsPerWg);
  dim3 grid(static_cast<unsigned>(wgs), static_cast<unsigned>(batch));
  k_h1_rows<P, T><<<grid, kRowThreads, 0, st>>>(
      dev_at<int32_t>(s, s->off_inc_ptr), dev_at<int32_t>(s, s->off_inc_list), dev_at<int32_t>(s, s->off_class),
      dev_at<uint8_t>(s, s->off_tables), s->tab_stride, ed, x, static_cast<const T*>(kappa), static_cast<T>(beta), rp,
      s->nrows, s->nel, s->nnz, static_cast<T*>(values), flags, static_cast<float>(thr), diag);
  LOR_LAUNCHED("k_h1_rows");
  return LOR_OK;
}

template <typename T>
int dispatch_rows(int p, const lor_sched* s, int batch, const int32_t* ed, const double* x, const void* k, double beta,
                  const int32_t* rp, void* v, unsigned f, double thr, int32_t* diag, hipStream_t st) {
  switch (p) {
    case 1: return launch_rows<1, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    case 2: return launch_rows<2, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    case 3: return launch_rows<3, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    case 4: return launch_rows<4, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    case 5: return launch_rows<5, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    case 6: return launch_rows<6, T>(s, batch, ed, x, k, beta, rp, v, f, thr, diag, st);
    default: LOR_FAIL(LOR_EUNSUPPORTED, "p = %d not compiled", p);
  }
}

template int dispatch_rows<double>(int, const lor_sched*, int, const int32_t*, const double*, const void*, double,
                                   const int32_t*, void*, unsigned, double, int32_t*, hipStream_t);
template int dispatch_rows<float>(int, const lor_sched*, int, const int32_t*, const double*, const void*, double,
                                  const int32_t*, void*, unsigned, double, int32_t*, hipStream_t);

}  // namespace lor
