// Matrix values one row at a time, on any mesh: the part that H1, H(curl) and H(div)
// share (in 3D; the 2D call has no such kernel).
//
// The coloured kernels integrate every cell once, but need one launch per
// colour, and on a small mesh each launch is the latency of one group (about
// 11 us): 12 colours take 130 us whatever the mesh.  Here one launch does it:
// S::LANES lanes sum one row, each integrating its share of the cells around
// the row's vertex, edge or face, so every cell is integrated once per dof of
// its own (8 vertices, 12 edges, 6 faces), and every row is stored once, whole.
//
//   * The cells around a dof follow from its incidences (element, local dof),
//     sorted in the schedule: within an element, in increasing number u of the
//     dof within the cell, which is decreasing position of the cell.  That list
//     is dealt to the lanes in turn.
//   * A lane integrates its cell (all unique entries of the symmetric matrix, so
//     that (i, j) and (j, i) have the same bits) and takes the entries of its dof;
//     their places in the row come from the element's rank table.
//   * The lanes then add their entries to the row in LDS one after another, in
//     the order of the list: increasing element, decreasing cell within it, for
//     both rows of an entry.  The matrix is bitwise symmetric and repeatable.
// All arithmetic is FP64, whatever the type of the values (FP64 and unpacked
// FP32 instructions issue at the same rate), and every entry is rounded once.
//
// S (one per space and degree) has
//   LANES, NE (entries of one dof in one cell), NLOC (dofs of an element), NSUB
//   cells(l)            number of the element's cells around local dof l
//   cell(a, e, l, nth, kappa, at, en)   places and values of the entries of the
//                       nth of them; returns the dof's number u in the cell
#pragma once

#include "lor_common.hpp"

namespace lor {

struct RowArgs {
  const int32_t *inc_ptr, *inc_list, *elem_class;
  const uint8_t* tables;
  int64_t tab_stride;
  const int32_t* st_ptr;     // first table entry of each local dof
  const int32_t* elem_verts;
  const int32_t* elem_map;   // signed edge or face map
  const double* coords;
  double beta;
  const int32_t* row_ptr;
  int64_t nrows, nel, nnz;
  unsigned flags;            // LOR_FP64_FALLBACK: count the cells past the threshold (FP32 form)
  float det_thresh;
  int32_t* diag;
};

constexpr int kRowThreads = 256;
constexpr size_t kRowLds = 64 * 1024;  // LDS of a workgroup, at most

// Entries between two rows in LDS: the mesh's longest row (the schedule's
// max_row_nnz; 0 if unknown), odd, so that rows start in different banks.
inline int row_stride(const lor_sched* s) { return (s->max_row_nnz > 0 ? s->max_row_nnz : LOR_MAX_ROW_NNZ) | 1; }
inline size_t row_lds(const lor_sched* s, int lanes) {
  return static_cast<size_t>(kRowThreads / lanes) * row_stride(s) * sizeof(double);
}

template <class S, typename T>
__global__ __launch_bounds__(kRowThreads, S::WPE) void k_rows(RowArgs a, int stride, const T* __restrict__ kappa,
                                                              T* __restrict__ values) {
  constexpr int LANES = S::LANES, ROWS = kRowThreads / LANES;
  static_assert(64 % LANES == 0, "a row's lanes are in one wave");
  extern __shared__ double sRow[];
  const int tid = threadIdx.x, k = tid % LANES;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * ROWS + tid / LANES;
  kappa += static_cast<int64_t>(blockIdx.y) * a.nel * S::NSUB;
  values += static_cast<int64_t>(blockIdx.y) * a.nnz;
  const bool live = row < a.nrows;
  const int32_t first = live ? a.inc_ptr[row] : 0, ninc = live ? a.inc_ptr[row + 1] - first : 0;
  const int32_t start = live ? a.row_ptr[row] : 0, rlen = live ? a.row_ptr[row + 1] - start : 0;
  const int32_t len = rlen < stride ? rlen : stride;
  double* const acc = sRow + (tid / LANES) * stride;
  for (int j = k; j < len; j += LANES) acc[j] = 0.0;

  for (int i0 = 0; __ballot(i0 < ninc) != 0; i0 += LANES) {
    // this lane's incidence of the next LANES, and the number of cells before
    // its own in the list
    const int32_t inc = i0 + k < ninc ? a.inc_list[first + i0 + k] : 0;
    const int mine = i0 + k < ninc ? S::cells(inc % S::NLOC) : 0;
    int before = mine;
#pragma unroll
    for (int m = 1; m < LANES; m <<= 1) {
      const int t = __shfl_up(before, m, LANES);
      if (k >= m) before += t;
    }
    const int total = __shfl(before, LANES - 1, LANES);
    before -= mine;
    for (int o0 = 0; __ballot(o0 < total) != 0; o0 += LANES) {
      // cell number o0 + k of the list: its incidence, and its number there
      const int o = o0 + k;
      int32_t einc = 0;
      int nth = 0;
#pragma unroll
      for (int j = 0; j < LANES; ++j) {
        const int32_t ij = __shfl(inc, j, LANES);
        const int bj = __shfl(before, j, LANES), mj = __shfl(mine, j, LANES);
        if (o >= bj && o < bj + mj) {
          einc = ij;
          nth = o - bj;
        }
      }
      const bool have = o < total;
      int at[S::NE];
      double en[S::NE];
      if (have) S::template cell<T>(a, kappa, einc / S::NLOC, einc % S::NLOC, nth, at, en);
      // into the row, one lane after another
#pragma unroll 1
      for (int j = 0; j < LANES; ++j) {
        if (have && k == j) {
          double t[S::NE];
#pragma unroll
          for (int v = 0; v < S::NE; ++v) t[v] = acc[at[v]];
#pragma unroll
          for (int v = 0; v < S::NE; ++v) acc[at[v]] = t[v] + en[v];
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  for (int j = k; j < len; j += LANES) values[static_cast<int64_t>(start) + j] = static_cast<T>(acc[j]);
}

// Corners of cell (sx, sy, sz) of element e (lattice of q = Q points per axis).
template <int Q>
__device__ __forceinline__ void row_corners(const RowArgs& a, int e, int sx, int sy, int sz, double (&X)[8][3]) {
  const int32_t* ed = a.elem_verts + static_cast<int64_t>(e) * Q * Q * Q + sx + Q * (sy + Q * sz);
  int32_t g[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) g[v] = ed[(v & 1) + Q * (((v >> 1) & 1) + Q * (v >> 2))];
#pragma unroll
  for (int v = 0; v < 8; ++v)
#pragma unroll
    for (int d = 0; d < 3; ++d) X[v][d] = a.coords[3 * static_cast<int64_t>(g[v]) + d];
}

template <class S, typename T>
static int launch_rows(const lor_sched* s, int batch, const int32_t* elem_verts, const int32_t* elem_map,
                       const double* coords, const void* kappa, double beta, const int32_t* row_ptr, void* values,
                       unsigned flags, double thr, int32_t* diag, hipStream_t st) {
  if (row_lds(s, S::LANES) > kRowLds) LOR_FAIL(LOR_EUNSUPPORTED, "rows of %d entries", row_stride(s));
  RowArgs a;
  a.inc_ptr = dev_at<int32_t>(s, s->off_inc_ptr);
  a.inc_list = dev_at<int32_t>(s, s->off_inc_list);
  a.elem_class = dev_at<int32_t>(s, s->off_class);
  a.tables = dev_at<uint8_t>(s, s->off_tables);
  a.tab_stride = s->tab_stride;
  a.st_ptr = dev_at<int32_t>(s, s->off_st_ptr);
  a.elem_verts = elem_verts;
  a.elem_map = elem_map;
  a.coords = coords;
  a.beta = static_cast<double>(static_cast<T>(beta));
  a.row_ptr = row_ptr;
  a.nrows = s->nrows;
  a.nel = s->nel;
  a.nnz = s->nnz;
  a.flags = flags;
  a.det_thresh = static_cast<float>(thr);
  a.diag = diag;
  dim3 grid(static_cast<unsigned>(ceil_div(s->nrows, kRowThreads / S::LANES)), static_cast<unsigned>(batch));
  k_rows<S, T><<<grid, kRowThreads, row_lds(s, S::LANES), st>>>(a, row_stride(s), static_cast<const T*>(kappa), static_cast<T*>(values));
  LOR_LAUNCHED("k_rows");
  return LOR_OK;
}

// dispatch over the degree: FN<P, T>(args)
#define LOR_ROWS_DISPATCH(NAME, SPACE)                                                                               \
  template <typename T>                                                                                               \
  int NAME(int p, const lor_sched* s, int batch, const int32_t* verts, const int32_t* map, const double* x,           \
           const void* k, double beta, const int32_t* rp, void* v, unsigned f, double thr, int32_t* diag,             \
           hipStream_t st) {                                                                                          \
    switch (p) {                                                                                                      \
      case 1: return launch_rows<SPACE<1>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      case 2: return launch_rows<SPACE<2>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      case 3: return launch_rows<SPACE<3>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      case 4: return launch_rows<SPACE<4>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      case 5: return launch_rows<SPACE<5>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      case 6: return launch_rows<SPACE<6>, T>(s, batch, verts, map, x, k, beta, rp, v, f, thr, diag, st);             \
      default: LOR_FAIL(LOR_EUNSUPPORTED, "p = %d not compiled", p);                                                  \
    }                                                                                                                 \
  }                                                                                                                   \
  template int NAME<double>(int, const lor_sched*, int, const int32_t*, const int32_t*, const double*, const void*,   \
                            double, const int32_t*, void*, unsigned, double, int32_t*, hipStream_t);                  \
  template int NAME<float>(int, const lor_sched*, int, const int32_t*, const int32_t*, const double*, const void*,    \
                           double, const int32_t*, void*, unsigned, double, int32_t*, hipStream_t);

}  // namespace lor
