// Kernels of the single-instance reverse: the scan of a pass and the edge
// gradients of its voxels (bwd_scan.h says why they are two).
#include "bwd_scan.h"
#include "edge_grid.h"

namespace ggdt {
namespace {

using namespace dev;

template <class Geo>
__global__ __launch_bounds__(Geo::NTCAP) void bwd_scan_cell_kernel(BwdDesc g, unsigned* words,
                                                                   unsigned long long limit) {
  __shared__ float2 pair[2 * Geo::NT];
  __shared__ int fail;
  if (ld_relaxed(words + kWordAbort) != 0u) return;
  run_bwd_scan_cell<Geo>(g, g.xbuf, words, limit, pair, &fail, xcd_remap(blockIdx.x, gridDim.x), gridDim.x);
}

template <bool SCANC>
__global__ __launch_bounds__(kRowLanes) void bwd_scan_row_kernel(BwdDesc g, unsigned* words,
                                                                 unsigned long long limit) {
  if (ld_relaxed(words + kWordAbort) != 0u) return;
  run_bwd_scan_row<SCANC>(g, g.xbuf, words, limit, xcd_remap(blockIdx.x, gridDim.x), gridDim.x);
}

// One voxel per thread, threads along the contiguous axis.  A voxel's children
// are found by comparing the 3 / 9 records of the child plane; the few that
// match (one on average) are then walked lane by lane, so that a wave runs the
// root and the division as often as its busiest lane needs them and not once
// per offset.  ND: axes; NCH: channels (0: g.C, known at run time only).
template <int ND, int MODE, int NCH>
__device__ __forceinline__ void edge_voxel(const BwdDesc& g, const EdgeDesc& s, const float* sA, int col,
                                           long long row) {
  constexpr int NJ = ND == 3 ? 9 : 3;
  constexpr bool USE_I = MODE != kModeLam0;
  const int C = NCH > 0 ? NCH : g.C;
  const gmem<const float> gI = to_gmem(g.image);
  const gmem<const uint8_t> gR = to_gmem(g.rec);
  const gmem<const float> gA = to_gmem(s.a);
  const long long y = row * s.d2 + col;
  // coordinates along the scan axis (array order) and the plane axes
  int k, pp, qq;
  if (ND == 3) {
    const int z = (int)(row / s.d1), r1 = (int)(row - (long long)z * s.d1);
    k = s.axis == 0 ? z : (s.axis == 1 ? r1 : col);
    pp = s.axis == 0 ? r1 : z;
    qq = s.axis == 2 ? r1 : col;
  } else {
    k = s.axis == 0 ? (int)row : col;
    pp = 0;
    qq = s.axis == 0 ? col : (int)row;
  }
  const int ry = gR[y];
  const float ay = gA[y];
  if (USE_I) {
    const int kch = k + g.sign, kpar = k - g.sign;
    const bool has_child = kch >= 0 && kch < g.Na;
    const bool has_par = kpar >= 0 && kpar < g.Na;
    const long long step = (long long)g.sign * g.sa;
    float gy[NCH > 0 ? NCH : 8], iy[NCH > 0 ? NCH : 8];
#pragma unroll
    for (int c = 0; c < (NCH > 0 ? NCH : 8); ++c) {
      if (c >= C) break;
      iy[c] = gI[c * (long long)g.N + y];
      gy[c] = s.first ? 0.0f : s.gI[c * (long long)g.N + y];
    }
    // gradient of the edge to the voxel at offset x, with coefficient a lambda / w;
    // child: y is the parent (d = I(x) - I(y), subtracted), else the child
    auto edge = [&](long long x, int j, float a, bool child) {
      float d[NCH > 0 ? NCH : 8], q = 0.0f;
#pragma unroll
      for (int c = 0; c < (NCH > 0 ? NCH : 8); ++c) {
        if (c >= C) break;
        const float ix = gI[c * (long long)g.N + x];
        d[c] = child ? ix - iy[c] : iy[c] - ix;
        q = c == 0 ? d[c] * d[c] : fmaf(d[c], d[c], q);
      }
      float w;
      if (MODE == kModeLam1C1)
        w = fabsf(d[0]);
      else
        w = general_root<MODE, NCH != 1>(fmaf(g.lam, q, sA[j]));
      if (w > 0.0f) {
        const float coef = (a * g.lam) / w;
#pragma unroll
        for (int c = 0; c < (NCH > 0 ? NCH : 8); ++c) {
          if (c >= C) break;
          gy[c] = child ? gy[c] - coef * d[c] : gy[c] + coef * d[c];
        }
      }
    };
    unsigned match = 0;
    if (has_child) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int dp = ND == 3 ? j / 3 - 1 : 0, dq = (ND == 3 ? j % 3 : j) - 1;
        const int cp = pp - dp, cq = qq - dq;  // child x_j = y - delta_j
        if (cp >= 0 && cp < g.Np && cq >= 0 && cq < g.Nq) {
          const long long x = y + step - dp * g.sp - dq * g.sq;
          match |= (gR[x] == 1 + j ? 1u : 0u) << j;
        }
      }
    }
    while (match != 0u) {
      const int j = __ffs(match) - 1;
      match &= match - 1u;
      const int dp = ND == 3 ? j / 3 - 1 : 0, dq = (ND == 3 ? j % 3 : j) - 1;
      const long long x = y + step - dp * g.sp - dq * g.sq;
      edge(x, j, gA[x], true);
    }
    // a parent outside the grid only comes from records of another schedule: skip it
    if (has_par && ry >= 1 && ry <= NJ) {
      const int j = ry - 1;
      const int dp = ND == 3 ? j / 3 - 1 : 0, dq = (ND == 3 ? j % 3 : j) - 1;
      if (pp + dp >= 0 && pp + dp < g.Np && qq + dq >= 0 && qq + dq < g.Nq)
        edge(y - step + dp * g.sp + dq * g.sq, j, ay, false);
    }
#pragma unroll
    for (int c = 0; c < (NCH > 0 ? NCH : 8); ++c) {
      if (c >= C) break;
      s.gI[c * (long long)g.N + y] = gy[c];
    }
  } else if (s.first) {
    for (int c = 0; c < C; ++c) s.gI[c * (long long)g.N + y] = 0.0f;
  }
  const float a = ry != 0 ? 0.0f : ay;
  s.out[y] = s.last ? s.v * a : a;
}

template <int ND, int NCH>
__global__ __launch_bounds__(kEdgeThreads) void bwd_edge_kernel(BwdDesc g, EdgeDesc s, const unsigned* words) {
  __shared__ float sA[9];
  if (threadIdx.x < 9) sA[threadIdx.x] = g.A[threadIdx.x];
  __syncthreads();
  const unsigned ucol = s.col0 + blockIdx.x * kEdgeCols + (threadIdx.x & (kEdgeCols - 1));
  if (ucol >= (unsigned)s.d2) return;
  const int col = (int)ucol;
  const unsigned* cls = words + kWordClass;
  const long long rows = (long long)(g.N / s.d2);
  for (long long row = (long long)blockIdx.y * kEdgeRows + (threadIdx.x / kEdgeCols); row < rows;
       row += (long long)gridDim.y * kEdgeRows) {
    if (g.mode == kModeLam0)
      edge_voxel<ND, kModeLam0, NCH>(g, s, sA, col, row);
    else if (NCH == 1 && g.mode == kModeLam1C1 && fast_mode_ok(kModeLam1C1, ld_relaxed(cls)))
      edge_voxel<ND, kModeLam1C1, NCH>(g, s, sA, col, row);
    else if (g.mode == kModeGeneral && general_n_ok(g.sqrt_normal, cls))
      edge_voxel<ND, kModeGeneralN, NCH>(g, s, sA, col, row);
    else
      edge_voxel<ND, kModeGeneral, NCH>(g, s, sA, col, row);
  }
}

using ScanKernel = void (*)(BwdDesc, unsigned*, unsigned long long);

int scan_capacity(ScanKernel fn, int threads) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)fn, threads, 0) != hipSuccess) return 0;
  return per_cu * cus;
}

template <class Geo>
hipError_t launch_scan_cell(const BwdDesc& d, unsigned* words, unsigned long long limit, hipStream_t stream) {
  static int cached = 0;
  int cap = cached;
  if (cap <= 0) cached = cap = scan_capacity(bwd_scan_cell_kernel<Geo>, Geo::NTCAP);
  if (cap <= 0) return hipErrorInvalidConfiguration;
  const int ntiles = d.ntp * d.ntq, grid = ntiles < cap ? ntiles : cap;
  hipLaunchKernelGGL(bwd_scan_cell_kernel<Geo>, dim3(grid), dim3(Geo::NT), 0, stream, d, words, limit);
  return hipGetLastError();
}

template <bool SCANC>
hipError_t launch_scan_row(const BwdDesc& d, unsigned* words, unsigned long long limit, hipStream_t stream) {
  static int cached = 0;
  int cap = cached;
  if (cap <= 0) cached = cap = scan_capacity(bwd_scan_row_kernel<SCANC>, kRowLanes);
  if (cap <= 0) return hipErrorInvalidConfiguration;
  const int grid = d.ntq < cap ? d.ntq : cap;
  hipLaunchKernelGGL(bwd_scan_row_kernel<SCANC>, dim3(grid), dim3(kRowLanes), 0, stream, d, words, limit);
  return hipGetLastError();
}

template <int ND>
hipError_t launch_edges(const BwdDesc& g, EdgeDesc s, const unsigned* words, hipStream_t stream) {
  const long long rows = (long long)(g.N / s.d2);
  auto fn = g.C == 1 ? bwd_edge_kernel<ND, 1>
                     : (g.C == 2 ? bwd_edge_kernel<ND, 2> : (g.C == 3 ? bwd_edge_kernel<ND, 3> : bwd_edge_kernel<ND, 0>));
  for (unsigned col0 = 0; col0 < (unsigned)s.d2; col0 += kEdgeLaunchCols) {
    unsigned gx, gy;
    edge_grid((unsigned)s.d2, col0, rows, &gx, &gy);
    s.col0 = col0;
    hipLaunchKernelGGL(fn, dim3(gx, gy), dim3(kEdgeThreads), 0, stream, g, s, words);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_bwd_scan(const BwdDesc& d, int ndim, unsigned* words, unsigned long long spin_limit,
                           hipStream_t stream) {
  if (ndim == 3) {
    if (d.K != kCellK) return hipErrorInvalidConfiguration;
    if (d.TP == 16 && d.TQ == 16) return launch_scan_cell<CellGeomBase>(d, words, spin_limit, stream);
    if (d.TP == 8 && d.TQ == 16) return launch_scan_cell<CellGeomMid>(d, words, spin_limit, stream);
    if (d.TP == 8 && d.TQ == 8) return launch_scan_cell<CellGeomSmall>(d, words, spin_limit, stream);
    return hipErrorInvalidConfiguration;
  }
  if (d.TP != 1 || d.TQ != kRowTQ || d.K != kRowK) return hipErrorInvalidConfiguration;
  return d.sa == 1 ? launch_scan_row<true>(d, words, spin_limit, stream)
                   : launch_scan_row<false>(d, words, spin_limit, stream);
}

hipError_t launch_bwd_edges(const BwdDesc& g, int ndim, const EdgeDesc& s, const unsigned* words, hipStream_t stream) {
  return ndim == 3 ? launch_edges<3>(g, s, words, stream) : launch_edges<2>(g, s, words, stream);
}

}  // namespace ggdt
