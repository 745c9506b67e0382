// Reverse of one directional pass in two launches: a scan along the planes that
// carries abar, and a pass over all voxels that applies the edges' gradients.
//
// For a parent plane Y of a child plane X (record 1 + j: the child took its
// value through offset j; the arithmetic and its order per voxel are those of
// run_bwd_pass in backward_device.h):
//   scan   abar(y) = abar_in(y) + sum over children x_j with record 1 + j (j ascending) of abar(x_j)
//   edges  Ibar(y) -= coef(x_j) * (I(x_j) - I(y)) for the same children, j ascending,
//          coef(x) = (abar(x) * lambda) / w(x, parent), 0 when w = 0
//          Ibar(y) += coef(y) * (I(y) - I(y'))    when y has a parent y'
//          abar_out(y) = record(y) ? 0 : abar(y)
// Only the first line depends on the plane before; the root and the division
// of every edge are taken off the serial chain of planes, where a step is bound
// by its latency, and run over all voxels at once.  The scan needs no image, so
// it is the same kernel for every channel count and lambda.
//
// The scan uses the overlapped tiling and the epoch-tagged exchange words of
// the forward passes (pass_cell.h in 3D, pass_row.h in 2D); it reads a_in and
// writes abar before zeroing to a_out.
#pragma once

#include "pass_cell.h"
#include "pass_team.h"

namespace ggdt {
namespace dev {

// The scan of a 3D pass, one thread per cell of the tile's box, by workgroup
// `wg` of G (Geo::NT threads).  A step gathers the nine possible children's
// (abar, record) from LDS.  `pair`: 2 * Geo::NT float2.  False if a bounded
// wait gave up.
template <class Geo>
__device__ __forceinline__ bool run_bwd_scan_cell(const BwdDesc& g, unsigned long long* xbuf, unsigned* words,
                                                  unsigned long long limit, float2* pair, int* failw, int wg, int G) {
  constexpr int TP = Geo::TP, TQ = Geo::TQ, K = Geo::K, BQ = Geo::BQ;
  const gmem<const uint8_t> gRec = to_gmem(g.rec);
  const gmem<const float> gAin = to_gmem(g.a_in);
  const gmem<float> gAout = to_gmem(g.a_out);
  const int tid = threadIdx.x;
  const int br = tid / BQ, bc = tid - br * BQ;
  // Chebyshev distance outside the tile; threads past the box lie further out
  // than K and take part in the barriers only
  const int e = max(max(max(K - br, br - (K + TP - 1)), max(K - bc, bc - (K + TQ - 1))), 0);
  const int own_slot = (br - K) * TQ + (bc - K);  // valid when e == 0
  const int ntiles = g.ntp * g.ntq;
  const int Na = g.Na, Np = g.Np, Nq = g.Nq;
  float2* const S0 = pair;
  float2* const S1 = pair + Geo::NT;
  if (tid == 0) *failw = 0;  // read only after a barrier

  // Last plane of the forward scan: no children.
  {
    const int kl = g.sign > 0 ? Na - 1 : 0;
    for (int tile = wg; tile < ntiles; tile += G) {
      const int tp = tile / g.ntq, tq = tile - tp * g.ntq;
      const int pp = tp * TP - K + br, qq = tq * TQ - K + bc;
      if (e == 0 && pp < Np && qq < Nq) {
        const int x = kl * g.sa + pp * g.sp + qq * g.sq;
        gAout[x] = gAin[x];
      }
    }
  }

  const int nmine = (ntiles - wg + G - 1) / G;
  const int nitems = g.nchunk * nmine;
  struct Item {
    int c, T0, kk, tile, pp, qq, xpq;
    bool in;
  };
  auto item_of = [&](int n) {
    Item it;
    it.c = n / nmine;
    it.tile = wg + (n - it.c * nmine) * G;
    it.T0 = Na - 1 - it.c * K;  // scan position of the chunk's first child plane (m = 0)
    it.kk = min(K, it.T0);
    const int tp = it.tile / g.ntq, tq = it.tile - tp * g.ntq;
    it.pp = tp * TP - K + br;
    it.qq = tq * TQ - K + bc;
    it.in = it.pp >= 0 && it.pp < Np && it.qq >= 0 && it.qq < Nq;
    it.xpq = it.in ? it.pp * g.sp + it.qq * g.sq : 0;
    return it;
  };
  // memory index of plane m of an item (scan position T0 - m)
  auto xof = [&](const Item& it, int m) {
    const int t = it.T0 - m;
    return (g.sign > 0 ? t : Na - 1 - t) * g.sa + it.xpq;
  };
  float nA[K + 1];
  int nR[K + 1];
  auto fetch = [&](const Item& it) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m <= K; ++m) {
      nA[m] = 0.0f;
      nR[m] = 0;
      if (it.in && m <= it.kk && e <= it.kk - m) {
        const int x = xof(it, m);
        if (m >= 1 || it.c == 0) nA[m] = gAin[x];
        nR[m] = gRec[x];
      }
    }
  };

  Item cur = item_of(0);
  fetch(cur);
  for (int n = 0; n < nitems; ++n) {
    const int c = cur.c, kk = cur.kk;
    const unsigned epoch_in = g.epoch_base + (unsigned)c;
    const bool has_next = n + 1 < nitems;
    const Item nxt = item_of(has_next ? n + 1 : n);
    float ain[K + 1];
    int rec[K + 1];
#pragma unroll
    for (int m = 0; m <= K; ++m) {
      ain[m] = nA[m];
      rec[m] = nR[m];
    }
    // Plane 0 of the chunk: abar_in of the pass's last plane in chunk 0, else
    // the state the previous chunk published (this tile's and its neighbours').
    float s0 = 0.0f;
    int fail = 0;
    if (cur.in && e <= kk) {
      if (c == 0) {
        s0 = ain[0];
      } else {
        const int otp = cur.pp / TP, otq = cur.qq / TQ;
        const int slot = (cur.pp - otp * TP) * TQ + (cur.qq - otq * TQ);
        s0 = wait_word(xbuf + (size_t)((c - 1) & 1) * ntiles * (TP * TQ) +
                           (size_t)(otp * g.ntq + otq) * (TP * TQ) + slot,
                       epoch_in, words, limit, &fail);
      }
    }
    // Cells outside the volume hold record 0 in both planes: never a child.
    S0[tid] = make_float2(s0, __int_as_float(rec[0]));
    if (!cur.in) S1[tid] = make_float2(0.0f, __int_as_float(0));
    if (fail) *failw = n + 1;
    step_barrier();
    if (*failw == n + 1) return false;
    if (has_next) fetch(nxt);

    float2* Sc = S0;
    float2* Sn = S1;
    unsigned long long* xout = xbuf + (size_t)(c & 1) * ntiles * (TP * TQ) + (size_t)cur.tile * (TP * TQ);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      if (i >= kk) break;
      if (cur.in && e <= kk - 1 - i) {
        float a = ain[i + 1];
        float2 ch[9];  // children x_j = y - delta_j: (abar, record)
#pragma unroll
        for (int j = 0; j < 9; ++j) ch[j] = Sc[tid - (j / 3 - 1) * BQ - (j % 3 - 1)];
#pragma unroll
        for (int j = 0; j < 9; ++j) {
          const float t = a + ch[j].x;
          a = __float_as_int(ch[j].y) == 1 + j ? t : a;
        }
        Sn[tid] = make_float2(a, __int_as_float(rec[i + 1]));
        if (e == 0) {
          gAout[xof(cur, i + 1)] = a;
          if (i == kk - 1)
            st64_relaxed(xout + own_slot, ((unsigned long long)(epoch_in + 1u) << 32) | __float_as_uint(a));
        }
      }
      step_barrier();
      float2* ts = Sc;
      Sc = Sn;
      Sn = ts;
    }
    cur = nxt;
  }
  return true;
}

// The scan of a 2D pass, one wave per 32-cell tile (see pass_row.h): the three
// possible children are the adjacent lanes, moved by whole-wave shifts.  SCANC:
// along the contiguous axis, where a full chunk moves by 16-byte pieces of each
// lane's memory row (as in pass_team.h).
template <bool SCANC>
__device__ __forceinline__ bool run_bwd_scan_row(const BwdDesc& g, unsigned long long* xbuf, unsigned* words,
                                                 unsigned long long limit, int wg, int G) {
  constexpr int K = kRowK, TQ = kRowTQ;
  const gmem<const uint8_t> gRec = to_gmem(g.rec);
  const gmem<const float> gAin = to_gmem(g.a_in);
  const gmem<float> gAout = to_gmem(g.a_out);
  const int lane = threadIdx.x;
  const int e = max(max(K - lane, lane - (K + TQ - 1)), 0);
  const int own = lane - K;
  const int ntiles = g.ntq;
  const int Na = g.Na, Nq = g.Nq;
  {
    const int kl = g.sign > 0 ? Na - 1 : 0;
    for (int tile = wg; tile < ntiles; tile += G) {
      const int q = tile * TQ + own;
      if (e == 0 && q < Nq) {
        const int x = kl * g.sa + q * g.sq;
        gAout[x] = gAin[x];
      }
    }
  }
  const int nmine = (ntiles - wg + G - 1) / G;
  const int nitems = g.nchunk * nmine;
  struct Item {
    int c, tile, T0, kk, q, xq;
    bool in;
  };
  auto item_of = [&](int n) {
    Item it;
    it.c = n / nmine;
    it.tile = wg + (n - it.c * nmine) * G;
    it.T0 = Na - 1 - it.c * K;
    it.kk = min(K, it.T0);
    it.q = it.tile * TQ - K + lane;
    it.in = it.q >= 0 && it.q < Nq;
    it.xq = it.in ? it.q * g.sq : 0;
    return it;
  };
  auto xof = [&](const Item& it, int m) {
    const int t = it.T0 - m;
    return (g.sign > 0 ? t : Na - 1 - t) * g.sa + it.xq;
  };
  // Branch-free loads, as in the team pass: an unneeded row is read from
  // a clamped, in-bounds address and dropped where consumed.
  float nA[K + 1];
  int nR[K + 1];
  unsigned nRw[4] = {0u, 0u, 0u, 0u};  // records of rows 1 .. K of a full chunk, in memory order
  bool nfull = false;
  int nlast = -1;  // the last row the lane needs
  const bool up = g.sign < 0;  // rows ascend in memory (the reverse walks against the scan)
  auto fetch = [&](const Item& it) {
    const int x0 = xof(it, 0);
    const int step = -g.sign * g.sa;
    const int last = it.in ? it.kk - e : -1;
    nlast = last;
    if constexpr (SCANC) {
      nfull = it.kk == K;
      if (nfull) {
        nA[0] = gAin[x0];
        nR[0] = gRec[x0];
        const int xk = up ? x0 + 1 : x0 - K;
#pragma unroll
        for (int m = 0; m < K; m += 4) {
          const float4_a4 v = *(gmem<const float4_a4>)(gAin + (up ? xk + m : xk + K - 4 - m));
          nA[m + 1] = up ? v.x : v.w;
          nA[m + 2] = up ? v.y : v.z;
          nA[m + 3] = up ? v.z : v.y;
          nA[m + 4] = up ? v.w : v.x;
        }
        const uint4_a1 w = *(gmem<const uint4_a1>)(gRec + xk);
        nRw[0] = w.x;
        nRw[1] = w.y;
        nRw[2] = w.z;
        nRw[3] = w.w;
        return;
      }
    }
#pragma unroll
    for (int m = 0; m <= K; ++m) {
      int x = m <= last ? x0 + m * step : 0;
      __asm__ volatile("" : "+v"(x));  // keeps the clamp from becoming a branch per row
      nA[m] = gAin[x];
      nR[m] = gRec[x];
    }
  };
  Item cur = item_of(0);
  fetch(cur);
  for (int n = 0; n < nitems; ++n) {
    const int c = cur.c, kk = cur.kk;
    const unsigned epoch_in = g.epoch_base + (unsigned)c;
    const bool has_next = n + 1 < nitems;
    const Item nxt = item_of(has_next ? n + 1 : n);
    float ain[K + 1];
    int rec[K + 1];
#pragma unroll
    for (int m = 0; m <= K; ++m) {
      ain[m] = nA[m];
      int r = nR[m];
      if (SCANC && m > 0) {
        const int lo = (m - 1) & 15, hi = (K - m) & 15;  // byte of row m, ascending or descending
        const unsigned wd = up ? nRw[lo >> 2] >> (8 * (lo & 3)) : nRw[hi >> 2] >> (8 * (hi & 3));
        r = nfull ? (int)(wd & 0xffu) : r;
      }
      rec[m] = m <= nlast ? r : 0;
    }
    float a = 0.0f;
    int fail = 0;
    if (cur.in && e <= kk) {
      if (c == 0)
        a = ain[0];
      else  // the owner's slot of cell q is q itself: tile q / TQ, slot q % TQ
        a = wait_word(xbuf + (size_t)((c - 1) & 1) * ntiles * TQ + cur.q, epoch_in, words, limit, &fail);
    }
    if (__any(fail)) return false;
    if (has_next) fetch(nxt);
    // The steps: lanes outside the image have record 0, and values outside the
    // shrinking cone are never read by a lane of the cone.
    float res[K];
    auto step = [&](int i) {
      const float al = from_left(a), ar = from_right(a);
      const int rl = __float_as_int(from_left(__int_as_float(rec[i])));
      const int rr = __float_as_int(from_right(__int_as_float(rec[i])));
      float s = ain[i + 1];  // children x_j = y - delta_j, j ascending
      s = rr == 1 ? s + ar : s;
      s = rec[i] == 2 ? s + a : s;
      s = rl == 3 ? s + al : s;
      a = s;
      res[i] = s;
    };
    if (kk == K) {
#pragma unroll
      for (int i = 0; i < K; ++i) step(i);
    } else {
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (i < kk) step(i);
    }
    if (cur.in && e == 0) {
      unsigned long long* xout = xbuf + (size_t)(c & 1) * ntiles * TQ + (size_t)cur.tile * TQ;
      st64_relaxed(xout + own, ((unsigned long long)(epoch_in + 1u) << 32) | __float_as_uint(a));
      if (SCANC && kk == K) {
        const int x1 = xof(cur, 1), xk = up ? x1 : x1 - (K - 1);
#pragma unroll
        for (int m = 0; m < K; m += 4) {
          float4_a4 v;
          v.x = up ? res[m] : res[K - 1 - m];
          v.y = up ? res[m + 1] : res[K - 2 - m];
          v.z = up ? res[m + 2] : res[K - 3 - m];
          v.w = up ? res[m + 3] : res[K - 4 - m];
          *(gmem<float4_a4>)(gAout + xk + m) = v;
        }
      } else {
#pragma unroll
        for (int i = 0; i < K; ++i)
          if (i < kk) gAout[xof(cur, i + 1)] = res[i];
      }
    }
    cur = nxt;
  }
  return true;
}

}  // namespace dev
}  // namespace ggdt
