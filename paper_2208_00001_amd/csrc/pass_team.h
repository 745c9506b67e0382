// Directional pass of a 2D image by a team of four wavefronts per tile.
//
// A row's edge costs depend on the image alone, not on the distances of the row
// before, but a lone wave runs them inside the serial chain of rows: at
// lambda in (0, 1) with three channels 50 of a row step's 75 instructions, at
// one instruction per four cycles.  Here three producer waves compute the costs
// of the next chunk's rows into LDS, each on a SIMD of its own, while the chain
// wave advances the current chunk: a step of it is three additions and minima,
// whatever the channel count.  Tiles, chunks, exchange words and the lanes'
// cells are described in pass_row.h.  ns per row at 2048 x 2048, the costs inside
// the chain / here (the mean of both axes): one channel at lambda 0.5 226 / 111, at
// 1 150 / 111, at 0 137 / 106; three channels at 0.5 283 / 119; a chunk of 16 rows
// takes 1.7 to 1.9 us, 0.5 of it the neighbours' words' latency.
#pragma once

#include "pass_cell.h"
#include "pass_row.h"

#include <type_traits>

namespace ggdt {
namespace dev {

constexpr int kTeamThreads = 4 * kRowLanes;
// costs of one chunk of K rows: [row][offset][lane]
constexpr int team_chunk(int K) { return K * 3 * kRowLanes; }

// Four elements of a row at any element's address (passes along the contiguous
// axis).
typedef float float4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned uint4_a1 __attribute__((ext_vector_type(4), aligned(1)));

// Element of a row at `lane_bytes` from its start: a wave-uniform base and a
// 32-bit lane offset, which is one addition on the scalar unit and the access
// itself where a per-lane index costs five instructions.
template <class T>
__device__ __forceinline__ gmem<T> in_row(gmem<T> row, unsigned lane_bytes) {
  using B = std::conditional_t<std::is_const<T>::value, const char, char>;
  return (gmem<T>)((gmem<B>)row + lane_bytes);
}

// One 2D pass by workgroup `wg` of G, each of NTEAM teams (kTeamThreads threads
// a team).  `costs`: two chunks per team in LDS; `failw`: one LDS word.  False
// if a bounded wait gave up.  SCANC: the scan axis is the contiguous one; every
// lane is then on another memory row, and a full chunk moves by 16-byte pieces
// of it instead of one cache-line request per lane and element.
template <int MODE, int NCH, bool REC, int FMT, bool SCANC, int K = kRowK, int NTEAM = 1>
__device__ __forceinline__ bool run_pass_team(const PassDesc* gp, unsigned long long* xbuf, unsigned* words,
                                              unsigned long long limit, float* costs, int* failw, int wg, int G) {
  constexpr int TQ = kRowLanes - 2 * K;
  static_assert(!SCANC || K == 16, "four 16-byte pieces per chunk");
  constexpr bool USE_I = MODE != kModeLam0;  // lambda 0: constant costs, the producers only meet the barriers
  const PassDesc g = *gp;
  const auto gImage = image_of<FMT>(g.image);
  const gmem<const float> gMask = to_gmem(g.mask);
  const gmem<float> gD = to_gmem(g.D);
  const gmem<uint8_t> gRec = to_gmem(g.rec);
  const int lane = threadIdx.x & (kRowLanes - 1);
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x / kRowLanes);
  // 0: the team's chain wave, else a producer.  A workgroup's waves go to the four
  // SIMDs in turn: the rotation gives every team's chain wave another SIMD.
  const int wave = (wave_id + (wave_id >> 2)) & 3;
  const int team = wg * NTEAM + (wave_id >> 2), nteam = G * NTEAM;
  costs += (wave_id >> 2) * 2 * team_chunk(K);
  const int e = max(max(K - lane, lane - (K + TQ - 1)), 0);
  const int own = lane - K;
  const int ntiles = g.ntq;
  if (wg * NTEAM >= ntiles) return true;
  const int Na = g.Na, Nq = g.Nq;
  const long long cstride = g.N;
  if (threadIdx.x == 0) *failw = 0;  // read only after a barrier

  if (wave == 0 && (g.init || REC)) {  // first row in scan order
    const int kf = g.sign > 0 ? 0 : Na - 1;
    for (int tile = team; tile < ntiles; tile += nteam) {
      const int q = tile * TQ + own;
      if (e == 0 && q < Nq) {
        const int x = kf * g.sa + q * g.sq;
        if (g.init) gD[x] = g.v * gMask[x];
        if (REC && g.rec) gRec[x] = 0;
      }
    }
  }

  const gmem<const float> dsrc0 = g.init ? gMask : (gmem<const float>)gD;
  const float vscale = g.init ? g.v : 1.0f;
  // rounds of one tile per team; a team without a tile in the last round only
  // meets the barriers
  const int nmine = (ntiles - wg * NTEAM + nteam - 1) / nteam;
  const int nitems = g.nchunk * nmine;
  struct Item {
    int c, tile, t0, kk, q, xq;
    bool in;
  };
  auto item_of = [&](int n) {
    Item it;
    it.c = n / nmine;
    it.tile = team + (n - it.c * nmine) * nteam;
    it.t0 = 1 + it.c * K;
    it.kk = min(K, Na - it.t0);
    it.q = it.tile * TQ - K + lane;
    it.in = it.q >= 0 && it.q < Nq && it.tile < ntiles;
    it.xq = it.in ? it.q * g.sq : 0;
    return it;
  };
  auto xof = [&](const Item& it, int j) {
    const int t = it.t0 - 1 + j;
    return (g.sign > 0 ? t : Na - 1 - t) * g.sa + it.xq;
  };
  const int rstep = g.sign * g.sa;
  // memory index of row j's first element (uniform)
  auto row_of = [&](const Item& it, int j) {
    const int t = it.t0 - 1 + j;
    return (long long)(g.sign > 0 ? t : Na - 1 - t) * g.sa;
  };

  if (wave != 0) {
    // Producer: rows r0 .. r0 + NR - 1 of every chunk (the last producer's rows
    // past the chunk are not stored), from image rows r0 .. r0 + NR.
    constexpr int NR = (K + 2) / 3;
    const int r0 = (wave - 1) * NR;
    using T = typename ImgElem<FMT>::T;
    T nx[NR + 1][NCH];
    // Branch-free loads at clamped, in-bounds addresses: a row past the chunk or
    // a lane outside the image gives costs that no cell uses.
    auto fetch = [&](const Item& it) {
      const int x0 = xof(it, 0);
      if constexpr (SCANC && FMT == kImgF32) {
        if (it.kk == K) {
          // rows r0 .. r0 + 3, and r0 + 4 .. (the last producer: 13 .. 16)
          const int r1 = min(r0 + 4, K - 3);
          const bool up = g.sign > 0;
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            const gmem<const float> a = gImage + c * cstride;
            const float4_a4 v = *(gmem<const float4_a4>)(a + (up ? x0 + r0 : x0 - r0 - 3));
            const float4_a4 w = *(gmem<const float4_a4>)(a + (up ? x0 + r1 : x0 - r1 - 3));
            nx[0][c] = up ? v.x : v.w;
            nx[1][c] = up ? v.y : v.z;
            nx[2][c] = up ? v.z : v.y;
            nx[3][c] = up ? v.w : v.x;
            const float w0 = up ? w.x : w.w, w3 = up ? w.w : w.x;
            nx[4][c] = r1 == r0 + 4 ? w0 : w3;
            nx[5][c] = up ? w.y : w.z;
            nx[6][c] = up ? w.z : w.y;
          }
          return;
        }
      }
      if constexpr (!SCANC) {  // along the rows' axis: q is the memory column
        const unsigned lb = it.in ? (unsigned)it.q * (unsigned)sizeof(T) : 0u;
#pragma unroll
        for (int j = 0; j <= NR; ++j) {
          const long long r = row_of(it, min(r0 + j, it.kk));
#pragma unroll
          for (int c = 0; c < NCH; ++c) nx[j][c] = *in_row(gImage + (c * cstride + r), lb);
        }
        return;
      }
#pragma unroll
      for (int j = 0; j <= NR; ++j) {
        int x = it.in ? x0 + min(r0 + j, it.kk) * rstep : 0;
        __asm__ volatile("" : "+v"(x));  // keeps the clamp from becoming a branch per row
#pragma unroll
        for (int c = 0; c < NCH; ++c) nx[j][c] = gImage[c * cstride + x];
      }
    };
    if (USE_I && nitems > 0) fetch(item_of(0));
    for (int n = 0; n <= nitems; ++n) {
      if (USE_I && n < nitems) {
        float ix[NR + 1][NCH];
#pragma unroll
        for (int j = 0; j <= NR; ++j)
#pragma unroll
          for (int c = 0; c < NCH; ++c) ix[j][c] = widen<FMT>(nx[j][c]);
        if (n + 1 < nitems) fetch(item_of(n + 1));
        float* out = costs + (n & 1) * team_chunk(K) + r0 * 3 * kRowLanes + lane;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          float iy[3][NCH];
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            iy[0][c] = from_left(ix[i][c]);
            iy[1][c] = ix[i][c];
            iy[2][c] = from_right(ix[i][c]);
          }
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const float w = row_edge<MODE, NCH>(g, j, ix[i + 1], iy[j]);
            if (r0 + i < K) out[(i * 3 + j) * kRowLanes] = w;
          }
        }
      }
      step_barrier();
      if (*failw) return false;
    }
    return true;
  }

  // Chain wave: item n - 1 in phase n.  Where teams share the SIMDs (NTEAM > 1)
  // it issues before the producers, which have a whole phase.
  if (NTEAM > 1) __builtin_amdgcn_s_setprio(3);
  float nd[K + 1];
  auto fetch = [&](const Item& it) {
    const int x0 = xof(it, 0);
    if constexpr (SCANC) {
      if (it.kk == K) {
        const bool up = g.sign > 0;
        nd[0] = dsrc0[x0];
#pragma unroll
        for (int m = 0; m < K; m += 4) {
          const float4_a4 v = *(gmem<const float4_a4>)(dsrc0 + (up ? x0 + 1 + m : x0 - 4 - m));
          nd[m + 1] = up ? v.x : v.w;
          nd[m + 2] = up ? v.y : v.z;
          nd[m + 3] = up ? v.z : v.y;
          nd[m + 4] = up ? v.w : v.x;
        }
        return;
      }
    }
    if constexpr (!SCANC) {
      // every row of the chunk, needed or not: a cell outside the cone uses none
      const unsigned lb = it.in ? (unsigned)it.q * 4u : 0u;
#pragma unroll
      for (int j = 0; j <= K; ++j) nd[j] = *in_row(dsrc0 + row_of(it, min(j, it.kk)), lb);
      return;
    }
    const int last = it.in ? it.kk - e : -1;  // the lane needs rows 0 .. last
#pragma unroll
    for (int j = 0; j <= K; ++j) {
      int x = j <= last ? x0 + j * rstep : 0;
      __asm__ volatile("" : "+v"(x));
      nd[j] = dsrc0[x];
    }
  };
  int chg = 0;  // an own cell was lowered (convergence mode)
  Item cur = item_of(0);
  if (nitems > 0) fetch(cur);
  step_barrier();
  for (int n = 0; n < nitems; ++n) {
    const int c = cur.c, kk = cur.kk;
    const unsigned epoch_in = g.epoch_base + (unsigned)c;  // published by chunk c - 1
    const bool has_next = n + 1 < nitems;
    const Item nxt = item_of(has_next ? n + 1 : n);
    float dd[K + 1];
#pragma unroll
    for (int j = 0; j <= K; ++j) dd[j] = nd[j] * vscale;  // the initialising pass reads the mask: D_old = v * M
    float dcur = __builtin_inff();
    int fail = 0;
    if (cur.in && e <= kk) {
      if (c == 0)
        dcur = dd[0];
      else  // the owner's slot of cell q is q itself: tile q / TQ, slot q % TQ
        dcur = wait_word(xbuf + (size_t)((c - 1) & 1) * ntiles * TQ + cur.q, epoch_in, words, limit, &fail);
    }
    if (__any(fail)) *failw = 1;
    if (has_next) fetch(nxt);
    const float* wc = costs + (n & 1) * team_chunk(K) + lane;
    float res[K];
    int rch[K];
    auto step = [&](int i) {
      const float dy[3] = {from_left(dcur), dcur, from_right(dcur)};
      float best = dd[i + 1];
      int choice = 0;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const float cand = dy[j] + (USE_I ? wc[(i * 3 + j) * kRowLanes] : g.W0[j]);
        if (REC) {
          choice = cand < best ? 1 + j : choice;
          best = cand < best ? cand : best;
        } else {
          best = fminf(best, cand);
        }
      }
      res[i] = best;
      rch[i] = choice;
      dcur = cur.in ? best : __builtin_inff();
    };
    if (kk == K) {
#pragma unroll
      for (int i = 0; i < K; ++i) step(i);
    } else {
#pragma unroll
      for (int i = 0; i < K; ++i)
        if (i < kk) step(i);
    }
    // The exchange word of the chunk's last row first (the neighbours wait for
    // it), then the rows.
    if (cur.in && e == 0 && !fail) {
      unsigned long long* xout = xbuf + (size_t)(c & 1) * ntiles * TQ + (size_t)cur.tile * TQ;
      st64_relaxed(xout + own, ((unsigned long long)(epoch_in + 1u) << 32) | __float_as_uint(dcur));
      bool done = false;
      if constexpr (SCANC) {
        if (kk == K) {
          const bool up = g.sign > 0;
          const int x1 = xof(cur, 1), xk = up ? x1 : x1 - (K - 1);  // the chunk's lowest element
#pragma unroll
          for (int m = 0; m < K; m += 4) {
            float4_a4 v;
            v.x = up ? res[m] : res[K - 1 - m];
            v.y = up ? res[m + 1] : res[K - 2 - m];
            v.z = up ? res[m + 2] : res[K - 3 - m];
            v.w = up ? res[m + 3] : res[K - 4 - m];
            *(gmem<float4_a4>)(gD + xk + m) = v;
          }
          if (REC && g.rec) {
            unsigned w[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              w[m] = 0u;
#pragma unroll
              for (int i = 0; i < 4; ++i)
                w[m] |= (unsigned)(up ? rch[4 * m + i] : rch[K - 1 - 4 * m - i]) << (8 * i);
            }
            *(gmem<uint4_a1>)(gRec + xk) = uint4_a1{w[0], w[1], w[2], w[3]};
          }
          done = true;
        }
      }
      if (!done) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          if (i < kk) {
            if constexpr (SCANC) {
              const int x = xof(cur, i + 1);
              gD[x] = res[i];
              if (REC && g.rec) gRec[x] = (uint8_t)rch[i];
            } else {
              const long long r = row_of(cur, i + 1);
              *in_row(gD + r, (unsigned)cur.q * 4u) = res[i];
              if (REC && g.rec) *in_row(gRec + r, (unsigned)cur.q) = (uint8_t)rch[i];
            }
          }
        }
      }
      if (g.converge) {
#pragma unroll
        for (int i = 0; i < K; ++i)
          if (i < kk) chg |= res[i] < dd[i + 1];
      }
    }
    step_barrier();
    if (*failw) return false;  // (the launch ends: every wave of it returns)
    cur = nxt;
  }
  if (NTEAM > 1) __builtin_amdgcn_s_setprio(0);
  if (g.converge && __any(chg) && lane == 0)
    __hip_atomic_store(words + kWordChanged, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// Requested mode RMODE falls back to the general formula when the image
// classification word rules the fast edge cost out.
template <int RMODE, int NCH, bool REC, int FMT, bool SCANC, int K = kRowK, int NTEAM = 1>
__device__ __forceinline__ bool run_pass_team_mode(const PassDesc* gp, unsigned long long* xbuf, unsigned* words,
                                                   const unsigned* cls_word, unsigned long long limit, float* costs,
                                                   int* failw, int wg, int G) {
  if (RMODE == kModeGeneral) {
    if (general_n_ok(gp->sqrt_normal, cls_word))
      return run_pass_team<kModeGeneralN, NCH, REC, FMT, SCANC, K, NTEAM>(gp, xbuf, words, limit, costs, failw, wg, G);
    return run_pass_team<kModeGeneral, NCH, REC, FMT, SCANC, K, NTEAM>(gp, xbuf, words, limit, costs, failw, wg, G);
  }
  if (fast_mode_ok(RMODE, ld_relaxed(cls_word)))
    return run_pass_team<RMODE, NCH, REC, FMT, SCANC, K, NTEAM>(gp, xbuf, words, limit, costs, failw, wg, G);
  return run_pass_team<kModeGeneral, NCH, REC, FMT, SCANC, K, NTEAM>(gp, xbuf, words, limit, costs, failw, wg, G);
}

}  // namespace dev
}  // namespace ggdt
