// Adjoint of the LOR H1 assembly with respect to kappa and the coordinates.
//
// L = sum_b <Gbar_b, A_b>,  A_b = sum_s kappa_{b,s} K^s + beta M^s  (K^s at kappa = 1).
//   dL/dkappa_{b,s} = sum_{u,v} Gbar_b[pos(s,u,v)] K^s_uv,
//   dL/dX = sum_s <sum_b kappa_{b,s} Gbar_b|s, dK^s/dX> + <sum_b Gbar_b|s, dM^s/dX>.
// One lane per subelement (or two, with half of its corner pairs each)
// recomputes the geometry and K^s (nothing is stored by the forward pass),
// gathers the cotangent at the 64 CSR positions of its 8x8 block for every batch
// entry, writes dL/dkappa, and runs the reverse of the sum-factorised integration
// to get the adjoint of its 8 corner coordinates.  The corners are summed per
// element vertex in LDS in a fixed order (element E-vector), then per global
// vertex over its sorted incidences (deterministic; coordinates are shared by the
// batch, so their gradient is the sum over the batch).
#include <mutex>

#include "lor_common.hpp"
#include "lor_h1_adjoint.hpp"

namespace lor {

// Workspace of the allocation-free entry point: a file-scope device array, one
// copy per GPU, alive until the process ends.  Host code never uses its name
// as an address (on the host it is only a stand-in for the symbol): the
// device address comes from hipGetSymbolAddress, taken once per device with
// that device current, and is what the kernels receive.
constexpr size_t kBwScratchBytes = size_t(32) << 20;
__device__ __align__(256) unsigned char scratch[kBwScratchBytes];

static int bw_scratch_address(void** out) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = -1;
  LOR_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) LOR_FAIL(LOR_EDEVICE, "device index %d outside [0, 64)", dev);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* ptr = nullptr;
    LOR_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) LOR_FAIL(LOR_EDEVICE, "hipGetSymbolAddress returned NULL for the workspace array");
    addr[dev] = ptr;
  }
  *out = addr[dev];
  return LOR_OK;
}

__global__ void k_bw_zero_f64(double* __restrict__ x, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.0;
}

int check_sched(const lor_sched* s, int space, int p, int64_t nel, int64_t nrows);

// One small workgroup per group of E elements (one wave where the
// subelements allow: E p^3 <= 64 lanes), one workgroup per group, so that
// several independent workgroups share a CU and hide each other's latency
// (gathers of coordinates and cotangents, LDS round trips).
template <int P, int ELEMS>
struct BwCfg {
  static constexpr int Q = P + 1;
  static constexpr int NSUB = P * P * P;
  static constexpr int NLOC = Q * Q * Q;
  static constexpr int T1 = 3 * P + 1;
  static constexpr int NENT = T1 * T1 * T1;
  static constexpr int NENTP = (NENT + 15) / 16 * 16;
  static constexpr int E = ELEMS;
  static constexpr int LANES = (E * NSUB + 63) / 64 * 64;  // one per subelement
  static constexpr int TWE = NENTP / 4;
};

// The unique pairs (u <= v) that lane h of the H of a subelement takes: all, or those
// of 18 of 36 whose lower corner is 0, 3, 4 or 7 (or not); pair_slot: how many of
// lane 1's come before (u, v).
template <int H>
__host__ __device__ constexpr bool pair_of(int h, int u) {
  return H == 1 || (u == 0 || u == 3 || u == 4 || u == 7) == (h == 0);
}
__host__ __device__ constexpr int pair_slot(int u, int v) {
  int n = 0;
  for (int a = 0; a < u; ++a) n += pair_of<2>(1, a) ? 8 - a : 0;
  return n + v - u;
}

// What bounds the kernel at p = 4, 16^3, batch 8: HBM.  FP64 fetches 701 MB and writes
// 29 in 162 us, 4.5 TB/s or 88% of a copy's rate (FP32 404 and 29 MB in 95 us or more);
// about 200 MB of that are cotangent rows on element faces fetched again, for
// neighbouring elements run on different XCDs, which share no L2.
//
// Lanes per subelement (H) and waves per SIMD to reserve registers for (WPS).  On
// its way there it waits more than it computes (VALU issue in 36% of a wave's
// cycles), so waves are what it wants, but a lane keeps 108 accumulators
// (K, and the adjoints of K and M, per corner pair) and the next batch entry's
// gathered cotangents.  FP32: two lanes share a subelement, each with 18 of the 36
// pairs until the batch is through, and a register budget of two or three waves.
// In FP64 that spills 40 to 60 registers.  Batch 8, boxes, us with
// one lane and one wave / two lanes and two waves / two lanes and three waves:
//   FP64  p = 2, 20^3   90 / 125         p = 4, 16^3  191 / 231
//   FP32  p = 2, 20^3   74 /  57 /  60   p = 4, 16^3  152 / 121 / 104
//         p = 3, 16^3   84 /  66 /  58   p = 5, 13^3  147 / 121 / 124
// FP32, p = 6 (11^3): 179 and, two lanes, 181, but 124 with one lane and two waves;
// p = 1 (40^3) 93 and 111.
template <int P, typename R>
struct BwLanes {
  static constexpr bool F64 = sizeof(R) == 8;
  static constexpr int H = F64 || P == 1 || P == 6 ? 1 : 2;
  static constexpr int WPS = F64 || P == 1 ? 1 : P == 3 || P == 4 ? 3 : 2;
  // Elements per group.  At p = 1 not one per lane: a group's entries are gathered by
  // all lanes, 64 per element, and with 64 elements those in flight fill the
  // registers (40^3, batch 8, FP64 and FP32, us: 64 elements 136 and 92, 32 121 and
  // 88, 16 133 and 79; 60^3 376, 297, 376 and 214, 215, 204).
  static constexpr int E = P == 1 ? (F64 ? 32 : 16) : P == 2 ? 8 : P == 3 ? 2 : 1;
  // Half of that on a mesh whose groups are all resident at once even so: what a
  // group gathers in a row is then half as long (p = 1, 8^3 35 -> 29 us; p = 2, 4^3 36
  // -> 31, but 20^3 90 -> 95).  p = 3 in FP32 (two waves for 27 subelements): only up to
  // half of the chip's waves (9^3, batch 1: 21.5 us in pairs, 19.7 one by one, but 10^3
  // 20.9 and 24.3, 11^3 21.5 and 27.9).
  static constexpr int ESMALL = P == 1 ? 16 : P == 2 ? 4 : 1;
  static constexpr int SMALL_PART = P == 3 && !F64 ? 2 : 1;  // of the waves, one in so many
};

// p = 1: groups of 64 elements (one per lane) where smaller ones are the slower, with
// `round` the elements that these groups take in one round of the chip.  Us with 64
// and with 32 (FP64) or 16 (FP32):
//   a second round of smaller groups that is nearly empty, just above half a round:
//     FP64 (to two thirds) 33^3 38 and 46, 35^3 40 and 46, batch 8 75 and 85, 81 and 86;
//       37^3 59 and 48
//     FP32 (to three fifths, small batches) 33^3 36 and 41, batch 4 43 and 48; 35^3 36
//       and 37, batch 4 45 and 43
//   large meshes in FP32 with little to gather per element: 57^3 96 and 108, 93^3 421
//     and 486, batch 2 106 and 114, 462 and 506, but batch 4 129 and 128, batch 8, 79^3
//     454 and 462; 54^3 87 and 90, batch 2 99 and 95
inline bool bw_one_per_lane(bool f64, int64_t nel, int64_t round, int batch) {
  if (2 * nel > round && (f64 ? 3 * nel <= 2 * round : 5 * nel <= 3 * round)) return f64 || batch <= 4;
  return !f64 && batch <= 2 && 2 * nel > 5 * round;
}

// Compact index of stencil entry (vertex (x,y,z), offset (dx,dy,dz)) inside
// the element table: rows in lexicographic order, each row's valid offsets in
// (dz, dy, dx) lexicographic order.
template <int P>
__device__ __forceinline__ int compact_index(int x, int y, int z, int dx, int dy, int dz) {
  constexpr int T1 = 3 * P + 1;
  auto cnt = [](int t) { return (t == 0 || t == P) ? 2 : 3; };
  auto pre = [](int t) { return t == 0 ? 0 : 3 * t - 1; };
  const int nx = cnt(x), ny = cnt(y);
  const int rbase = pre(z) * T1 * T1 + cnt(z) * pre(y) * T1 + cnt(z) * ny * pre(x);
  return rbase + ((dz + (z > 0 ? 1 : 0)) * ny + (dy + (y > 0 ? 1 : 0))) * nx + (dx + (x > 0 ? 1 : 0));
}

template <int P, typename T, typename R, int H, int ELEMS>
__global__ __launch_bounds__((BwCfg<P, ELEMS>::LANES * H), (BwLanes<P, R>::WPS)) void k_h1_backward(
    int64_t nel, int32_t chunk, const int32_t* __restrict__ elem_dofs, const double* __restrict__ coords,
    const T* __restrict__ kappa, T beta, const int32_t* __restrict__ row_ptr, const uint8_t* __restrict__ tables,
    const int32_t* __restrict__ elem_class, int64_t tab_stride, const uint16_t* __restrict__ ent_row, int batch,
    int64_t nnz, const T* __restrict__ gvals, T* __restrict__ gkappa, double* __restrict__ ework) {
  using C = BwCfg<P, ELEMS>;
  constexpr int Q = C::Q, NSUB = C::NSUB, NLOC = C::NLOC, NENT = C::NENT, NENTP = C::NENTP, E = C::E;
  constexpr int LANES = C::LANES, TH = LANES * H, TWE = C::TWE;
  constexpr int NJ = (E * NENT + TH - 1) / TH;            // gathered entries per lane
  constexpr int XW = 3 * E * 8 * NSUB;                    // corner adjoints
  constexpr int HW = H > 1 ? XW + 36 * LANES : XW;        // and what lane 1 hands to lane 0
  constexpr int GW = E * NENT > HW ? E * NENT : HW;
  // coordinates by component ([d][element vertex]): lanes reading the same
  // corner of neighbouring subelements then hit consecutive words
  __shared__ double sX[3 * E * NLOC];
  __shared__ int32_t sRp[E * NLOC];
  __shared__ uint32_t sTabW[E * TWE];
  // cotangent entries in compact order, later the corner adjoints; in the
  // arithmetic's precision (both are R values), which halves this buffer in
  // the FP32 form
  __shared__ R sGX[GW];
  __shared__ R sGk[H > 1 ? LANES : 1];  // the second lane's part of dL/dkappa
  const uint8_t* sTab = reinterpret_cast<const uint8_t*>(sTabW);
  R* sG = sGX;
  R* sXb = sGX;

  const int64_t cbeg = static_cast<int64_t>(blockIdx.x) * chunk;
  const int nce = static_cast<int>(nel - cbeg < chunk ? nel - cbeg : chunk);
  const int ngr = (nce + E - 1) / E;
  for (int g = 0; g < ngr; ++g) {
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));
    __builtin_assume(tid >= 0 && tid < TH);
    const int ne = nce - g * E < E ? nce - g * E : E;
    const int64_t e0 = cbeg + static_cast<int64_t>(g) * E;  // elements e0 .. e0+ne-1
    __syncthreads();
    // staging: every load of a phase is issued before the first is used (a
    // loop that loads, waits and writes LDS per trip would pay one memory
    // round trip per trip); indices past the group are clamped, their values
    // not written
    {
      constexpr int NV = (E * NLOC + TH - 1) / TH, NW = (E * TWE + TH - 1) / TH;
      int32_t vid[NV], cls[NW];
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int i = tid + k * TH;
        const int i2 = i < ne * NLOC ? i : 0;
        vid[k] = elem_dofs[e0 * NLOC + i2];
      }
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const int i = tid + k * TH;
        cls[k] = elem_class[e0 + (i < ne * TWE ? i : 0) / TWE];
      }
      double xv[NV][3];
      int32_t rpv[NV];
      uint32_t tw[NW];
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int64_t v = vid[k];
        xv[k][0] = coords[3 * v + 0];
        xv[k][1] = coords[3 * v + 1];
        xv[k][2] = coords[3 * v + 2];
        rpv[k] = row_ptr[v];
      }
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const int i = tid + k * TH;
        const int i2 = i < ne * TWE ? i : 0;
        tw[k] = reinterpret_cast<const uint32_t*>(tables + cls[k] * tab_stride)[i2 % TWE];
      }
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int i = tid + k * TH;
        if (i < ne * NLOC) {
          sX[i] = xv[k][0];
          sX[E * NLOC + i] = xv[k][1];
          sX[2 * E * NLOC + i] = xv[k][2];
          sRp[i] = rpv[k];
        }
      }
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const int i = tid + k * TH;
        if (i < ne * TWE) sTabW[i] = tw[k];
      }
    }
    // CSR position of every compact entry of the group (row pointer + rank)
    int32_t gpos[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = tid + j * TH;
      const int i2 = i < ne * NENT ? i : 0;
      const int el = i2 / NENT;
      gpos[j] = static_cast<int32_t>(ent_row[i2 - el * NENT]);  // local row, completed below
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int i = tid + j * TH;
      const int i2 = i < ne * NENT ? i : 0;
      const int el = i2 / NENT;
      gpos[j] = sRp[el * NLOC + gpos[j]] + (sTab[el * NENTP + (i2 - el * NENT)] & kRankMask);
    }

    const int half = H > 1 ? __builtin_amdgcn_readfirstlane(tid / LANES) : 0;
    const int ct = tid - half * LANES;  // the lane's subelement
    const bool act = ct < ne * NSUB;
    const int el = act ? ct / NSUB : 0;
    const int s = act ? ct - el * NSUB : 0;
    const int64_t e = e0 + el;
    const int si = s % P, sj = (s / P) % P, sk = s / (P * P);
    auto edges = [&](R (&ex)[2][2][3], R (&ey)[2][2][3], R (&ez)[2][2][3]) {
      double X[8][3];
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const int lv = (si + (v & 1)) + Q * ((sj + ((v >> 1) & 1)) + Q * (sk + (v >> 2)));
#pragma unroll
        for (int d = 0; d < 3; ++d) X[v][d] = sX[d * E * NLOC + el * NLOC + lv];
      }
      h1_edges<R>(X, ex, ey, ez);
    };
    const int64_t kofs = e * NSUB + s;
    // everything between the staging and the vertex sums, for the pairs of lane h
    auto cells = [&](auto half_t) {
      constexpr int h = decltype(half_t)::value;
      R Kt[36], Wk[36], Wm[36];
#pragma unroll
      for (int i = 0; i < 36; ++i) Kt[i] = Wk[i] = Wm[i] = R(0);
      if (act) {
        R ex[2][2][3], ey[2][2][3], ez[2][2][3];
        edges(ex, ey, ez);
        H1Factors<R> F;
        (void)h1_factors<R>(ex, ey, ez, R(1), R(0), F);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int v = u; v < 8; ++v)
            if (pair_of<H>(h, u)) Kt[pair_index(u, v)] = h1_entry<R>(F, u, v);
      }
      // compact index of the ordered corner pairs (u, v) and (u, v + 1), v even:
      // they are neighbours in corner u's row; the same for every batch entry
      int kpair[32];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int x = si + (u & 1), y = sj + ((u >> 1) & 1), z = sk + (u >> 2);
#pragma unroll
        for (int v = 0; v < 8; v += 2)
          kpair[(u * 8 + v) / 2] = el * NENT + compact_index<P>(x, y, z, -(u & 1), ((v >> 1) & 1) - ((u >> 1) & 1),
                                                                (v >> 2) - (u >> 2));
      }
      // the group's cotangent entries in compact (row-contiguous) order and the
      // lane's coefficient: those of the next batch entry are loaded before this
      // entry's compute (unconditionally: the last entry reloads itself), so
      // that their latency is hidden behind it
      T gv[NJ];
      T kn;
#pragma unroll
      for (int j = 0; j < NJ; ++j) gv[j] = gvals[gpos[j]];
      kn = kappa[kofs];
      R gk = R(0);
      // dL/dkappa of batch entry b: this lane's part and the other's (written
      // before the last barrier)
      auto put_gk = [&](int b) {
        if (h == 0 && act)
          gkappa[static_cast<int64_t>(b) * nel * NSUB + kofs] = static_cast<T>(H > 1 ? gk + sGk[ct] : gk);
      };
      for (int b = 0; b < batch; ++b) {
        lds_barrier();  // the previous entry of the batch has been consumed
        if (b > 0) put_gk(b - 1);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int i = tid + j * TH;
          if (i < ne * NENT) sG[i] = static_cast<R>(gv[j]);
        }
        const R kb = static_cast<R>(kn);
        {
          const int bn = b + 1 < batch ? b + 1 : b;
          const T* gn = gvals + static_cast<int64_t>(bn) * nnz;
#pragma unroll
          for (int j = 0; j < NJ; ++j) gv[j] = gn[gpos[j]];
          kn = kappa[static_cast<int64_t>(bn) * nel * NSUB + kofs];
        }
        lds_barrier();
        gk = R(0);
        if (act) {
          // (u, v) and (v, u) both feed the unique entry {u, v}; the entries of a
          // corner's row and column are read ahead of their uses, so that the LDS
          // reads overlap
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (!pair_of<H>(h, u)) continue;
            R w[8], wt[8];
#pragma unroll
            for (int v = u; v < 8; ++v) {
              w[v] = sG[kpair[(u * 8 + (v & ~1)) / 2] + (v & 1)];
              if (v > u) wt[v] = sG[kpair[(v * 8 + (u & ~1)) / 2] + (u & 1)];
            }
            if constexpr (P > 1) __builtin_amdgcn_sched_barrier(0);  // (p = 1 would spill)
#pragma unroll
            for (int v = u; v < 8; ++v) {
              const int i = pair_index(u, v);
              const R t = v == u ? w[v] : w[v] + wt[v];
              gk += Kt[i] * t;
              if constexpr (std::is_same<R, double>::value) {
                Wk[i] += kb * t;
                Wm[i] += t;
              } else {  // FP32: one after the other, without the rounding of t
                Wk[i] += kb * w[v];
                Wm[i] += w[v];
                if (v > u) {
                  Wk[i] += kb * wt[v];
                  Wm[i] += wt[v];
                }
              }
            }
          }
        }
        if (h == 1) sGk[ct] = gk;
      }
      __syncthreads();  // sG is reused for the corner adjoints
      put_gk(batch - 1);
      if constexpr (H > 1) {
        // lane 0 takes the adjoint of all pairs through the geometry
        R* other = sGX + XW + ct;
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int v = u; v < 8; ++v)
            if (h == 1 && pair_of<H>(1, u)) {
              other[2 * pair_slot(u, v) * LANES] = Wk[pair_index(u, v)];
              other[(2 * pair_slot(u, v) + 1) * LANES] = Wm[pair_index(u, v)];
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int v = u; v < 8; ++v)
            if (h == 0 && pair_of<H>(1, u)) {
              Wk[pair_index(u, v)] = other[2 * pair_slot(u, v) * LANES];
              Wm[pair_index(u, v)] = other[(2 * pair_slot(u, v) + 1) * LANES];
            }
      }
      if (h == 0 && act) {
        R ex[2][2][3], ey[2][2][3], ez[2][2][3];
        edges(ex, ey, ez);
        R gx[2][2][3], gy[2][2][3], gz[2][2][3];
        h1_adjoint<R>(ex, ey, ez, Wk, Wm, static_cast<R>(beta), gx, gy, gz);
        // corner adjoints from the edge adjoints: e = X(hi) - X(lo)
        R* xb = sXb + el * 24 * NSUB + s;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
          const int a = v & 1, b2 = (v >> 1) & 1, c = v >> 2;
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            const R val = (a ? gx[b2][c][d] : -gx[b2][c][d]) + (b2 ? gy[a][c][d] : -gy[a][c][d]) +
                          (c ? gz[a][b2][d] : -gz[a][b2][d]);
            xb[(v * 3 + d) * NSUB] = val;
          }
        }
      }
    };
    if (half == 0)
      cells(std::integral_constant<int, 0>{});
    else
      cells(std::integral_constant<int, H - 1>{});
    __syncthreads();
    // per element vertex: sum its <= 8 subelement corners in a fixed order
    for (int i = tid; i < ne * NLOC; i += TH) {
      const int el2 = i / NLOC;
      const int l = i - el2 * NLOC;
      const int x = l % Q, y = (l / Q) % Q, z = l / (Q * Q);
      double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int sx = x - (u & 1), sy = y - ((u >> 1) & 1), sz = z - (u >> 2);
        if (sx >= 0 && sx < P && sy >= 0 && sy < P && sz >= 0 && sz < P) {
          const int s2 = sx + P * (sy + P * sz);
#pragma unroll
          for (int d = 0; d < 3; ++d) acc[d] += static_cast<double>(sXb[el2 * 24 * NSUB + (u * 3 + d) * NSUB + s2]);
        }
      }
      double* w = ework + ((e0 + el2) * NLOC + l) * 3;
      w[0] = acc[0];
      w[1] = acc[1];
      w[2] = acc[2];
    }
  }
}

// grad_coords[g] = sum over the sorted incidences (e, l) of g of the element
// E-vector adjoint.
__global__ void k_gather_vertices(const int32_t* __restrict__ inc_ptr, const int32_t* __restrict__ inc_list,
                                  int64_t nrows, const double* __restrict__ ework, double* __restrict__ gcoords) {
  const int64_t g = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= nrows) return;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int32_t i = inc_ptr[g]; i < inc_ptr[g + 1]; ++i) {
    const double* w = ework + 3 * static_cast<int64_t>(inc_list[i]);
    a0 += w[0];
    a1 += w[1];
    a2 += w[2];
  }
  gcoords[3 * g + 0] = a0;
  gcoords[3 * g + 1] = a1;
  gcoords[3 * g + 2] = a2;
}

static int num_cus_bw() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

template <int P, typename T, typename R>
static int launch_bw(const lor_sched* sched, int batch, const int32_t* elem_dofs, const double* coords,
                     const void* kappa, double beta, const int32_t* row_ptr, const void* gvals, void* gkappa,
                     double* gcoords, void* workspace, hipStream_t st) {
  using L = BwLanes<P, R>;
  const int64_t nel = sched->nel;
  double* ework = static_cast<double*>(workspace);
  auto launch = [&](auto elems) -> int {
    constexpr int E = decltype(elems)::value;
    using C = BwCfg<P, E>;
    if (sched->tab_stride != C::NENTP || sched->nent != C::NENT)
      LOR_FAIL(LOR_EINVAL, "schedule tables do not match p = %d", P);
    // one group of E elements per workgroup
    k_h1_backward<P, T, R, L::H, E><<<static_cast<unsigned>(ceil_div(nel, E)), C::LANES * L::H, 0, st>>>(
        nel, E, elem_dofs, coords, static_cast<const T*>(kappa), static_cast<T>(beta), row_ptr,
        dev_at<uint8_t>(sched, sched->off_tables), dev_at<int32_t>(sched, sched->off_class), sched->tab_stride,
        dev_at<uint16_t>(sched, sched->off_ent_row), batch, sched->nnz, static_cast<const T*>(gvals),
        static_cast<T*>(gkappa), ework);
    LOR_LAUNCHED("k_h1_backward");
    return LOR_OK;
  };
  const int64_t slots = static_cast<int64_t>(4 * L::WPS) * num_cus_bw();  // waves
  const int64_t small = ceil_div(nel, L::ESMALL) * (BwCfg<P, L::ESMALL>::LANES / 64 * L::H) * L::SMALL_PART;
  int rc;
  if (P == 1 && bw_one_per_lane(L::F64, nel, 64 * slots, batch))
    rc = launch(std::integral_constant<int, P == 1 ? 64 : L::E>{});
  else if (small <= slots)
    rc = launch(std::integral_constant<int, L::ESMALL>{});
  else
    rc = launch(std::integral_constant<int, L::E>{});
  if (rc) return rc;
  k_gather_vertices<<<static_cast<unsigned>(ceil_div(sched->nrows, 256)), 256, 0, st>>>(
      dev_at<int32_t>(sched, sched->off_inc_ptr), dev_at<int32_t>(sched, sched->off_inc_list), sched->nrows, ework,
      gcoords);
  LOR_LAUNCHED("k_gather_vertices");
  return LOR_OK;
}

template <typename T, typename R>
static int dispatch_bw(int p, const lor_sched* s, int batch, const int32_t* ed, const double* x, const void* k,
                       double beta, const int32_t* rp, const void* gv, void* gk, double* gx, void* ws,
                       hipStream_t st) {
  switch (p) {
    case 1: return launch_bw<1, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    case 2: return launch_bw<2, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    case 3: return launch_bw<3, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    case 4: return launch_bw<4, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    case 5: return launch_bw<5, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    case 6: return launch_bw<6, T, R>(s, batch, ed, x, k, beta, rp, gv, gk, gx, ws, st);
    default: LOR_FAIL(LOR_EUNSUPPORTED, "p = %d not compiled", p);
  }
}

}  // namespace lor

using namespace lor;

extern "C" size_t lor_backward_workspace(int p, int64_t nel, int batch, int dtype) {
  if (p < 1 || p > LOR_MAX_P || nel < 0 || batch < 1 || (dtype != LOR_F64 && dtype != LOR_F32)) return 0;
  return sizeof(double) * 3 * static_cast<size_t>(nel) * nloc_h1(p);
}

namespace lor {

// Host-side checks shared by both backward entry points (workspace excluded).
static int check_bw_args(int p, int64_t nel, int64_t ndofs, int batch, const int32_t* elem_dofs,
                         const double* coords, const void* kappa, const int32_t* row_ptr, const void* grad_values,
                         void* grad_kappa, double* grad_coords, int dtype) {
  if (p < 1 || p > LOR_MAX_P) LOR_FAIL(LOR_EINVAL, "p = %d outside [1, %d]", p, LOR_MAX_P);
  if (nel < 0 || ndofs < 1) LOR_FAIL(LOR_EINVAL, "nel < 0 or ndofs < 1");
  if (batch < 1) LOR_FAIL(LOR_EINVAL, "batch < 1");
  if (dtype != LOR_F64 && dtype != LOR_F32) LOR_FAIL(LOR_EINVAL, "dtype must be LOR_F64 or LOR_F32");
  if (!grad_coords) LOR_FAIL(LOR_EINVAL, "grad_coords is NULL");
  if (nel > 0 && (!elem_dofs || !coords || !kappa || !row_ptr || !grad_values || !grad_kappa))
    LOR_FAIL(LOR_EINVAL, "a required pointer is NULL");
  return LOR_OK;
}

static int run_bw(int p, int64_t nel, int64_t ndofs, int batch, const int32_t* elem_dofs, const double* coords,
                  const void* kappa, double beta, const int32_t* row_ptr, const lor_sched* sched,
                  const void* grad_values, void* grad_kappa, double* grad_coords, void* workspace, int dtype,
                  hipStream_t st) {
  if (nel == 0) {
    // a fill kernel rather than a memset node, so that the call can be captured
    k_bw_zero_f64<<<static_cast<unsigned>(ceil_div(3 * ndofs, 256)), 256, 0, st>>>(grad_coords, 3 * ndofs);
    LOR_LAUNCHED("k_bw_zero_f64");
    return LOR_OK;
  }
  if (dtype == LOR_F64)
    return dispatch_bw<double, double>(p, sched, batch, elem_dofs, coords, kappa, beta, row_ptr, grad_values,
                                       grad_kappa, grad_coords, workspace, st);
  return dispatch_bw<float, float>(p, sched, batch, elem_dofs, coords, kappa, beta, row_ptr, grad_values,
                                   grad_kappa, grad_coords, workspace, st);
}

}  // namespace lor

extern "C" int lor_assemble_backward(int p, int64_t nel, int64_t ndofs, int batch, const int32_t* elem_dofs,
                                     const double* coords, const void* kappa, double beta, const int32_t* row_ptr,
                                     const lor_sched* sched, const void* grad_values, void* grad_kappa,
                                     double* grad_coords, void* workspace, int dtype, void* stream) {
  clear_error();
  int rc = check_bw_args(p, nel, ndofs, batch, elem_dofs, coords, kappa, row_ptr, grad_values, grad_kappa,
                         grad_coords, dtype);
  if (rc) return rc;
  if (nel > 0 && !workspace) LOR_FAIL(LOR_EINVAL, "workspace is NULL");
  rc = check_sched(sched, LOR_H1, p, nel, ndofs);
  if (rc) return rc;
  return run_bw(p, nel, ndofs, batch, elem_dofs, coords, kappa, beta, row_ptr, sched, grad_values, grad_kappa,
                grad_coords, workspace, dtype, as_stream(stream));
}

extern "C" size_t lor_backward_noalloc_max_workspace(void) { return kBwScratchBytes; }

extern "C" int lor_assemble_backward_noalloc(int p, int64_t nel, int64_t ndofs, int batch,
                                             const int32_t* elem_dofs, const double* coords, const void* kappa,
                                             double beta, const int32_t* row_ptr, const lor_sched* sched,
                                             const void* grad_values, void* grad_kappa, double* grad_coords,
                                             int dtype, void* stream) {
  clear_error();
  int rc = check_bw_args(p, nel, ndofs, batch, elem_dofs, coords, kappa, row_ptr, grad_values, grad_kappa,
                         grad_coords, dtype);
  if (rc) return rc;
  const size_t need = lor_backward_workspace(p, nel, batch, dtype);
  if (need > kBwScratchBytes)
    LOR_FAIL(LOR_EUNSUPPORTED,
             "the backward needs %zu workspace bytes, above the %zu bytes of the built-in workspace "
             "(nel * (p+1)^3 must be at most %zu); use lor_assemble_backward with a caller workspace",
             need, kBwScratchBytes, kBwScratchBytes / (3 * sizeof(double)));
  rc = check_sched(sched, LOR_H1, p, nel, ndofs);
  if (rc) return rc;
  void* ws = nullptr;
  rc = bw_scratch_address(&ws);
  if (rc) return rc;
  return run_bw(p, nel, ndofs, batch, elem_dofs, coords, kappa, beta, row_ptr, sched, grad_values, grad_kappa,
                grad_coords, ws, dtype, as_stream(stream));
}
