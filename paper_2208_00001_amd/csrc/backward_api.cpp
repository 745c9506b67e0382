// C ABI of the backward (single instance: one or two launches per reversed pass;
// batched: one persistent launch, tables built by ggdt_batched_plan).
#include <math.h>
#include <string.h>

#include "ggdt.h"
#include "ggdt_api_internal.h"
#include "ggdt_internal.h"

namespace ggdt {

constexpr int kMaxBwdChannels = 8;

size_t bwd_workspace_for(const Problem& pr) {
  const size_t base = workspace_for(pr, Tuning{});
  return base + ((size_t)pr.N * 4 + 255) / 256 * 256;
}

// Whether the reverse of a volume takes one launch a pass, the edges inside the
// plane step (backward_cell.h), and not a scan and a launch over all voxels for
// the edges (bwd_scan.h).  The step with the edges is longer by about 0.6 us a
// plane, for every round of 256 tiles (0.15 at lambda 0, where there are no
// edges), and more against the scan's smaller tiles where it has them; the
// second launch costs about 15 ns per 1000 voxels (3 at lambda 0, to zero abar).
// So the voxels per plane step decide.  Two launches / one, ms, two iterations at
// lambda 0, 0.5, 1: 176^3 1.47 / 1.65, 2.11 / 2.73, 2.26 / 2.68; 200^3 2.16 / 2.03,
// 3.21 / 3.28, 3.38 / 3.23; 256^3 2.88 / 2.61, 5.02 / 4.33, 5.33 / 4.26; 288^3 (two
// rounds of tiles) 5.66 / 5.34, 9.04 / 9.14, 9.48 / 8.99; 40 x 512 x 512 3.13 / 3.52,
// 4.19 / 5.99, 4.42 / 5.90.  With several channels two launches are faster
// throughout.
static bool reverse_in_one_launch(const Problem& pr, float lam) {
  if (pr.ndim != 3 || pr.C != 1 || pr.dims[2] < 2) return false;
  double steps = 0.0;
  for (int a = 0; a < 3; ++a) {
    PassDesc g;
    pass_geometry(pr, a, &g);
    int TP, TQ;
    cell_tile(g.Np, g.Nq, 1, &TP, &TQ);
    const long long tiles = (long long)((g.Np + kCellTP - 1) / kCellTP) * ((g.Nq + kCellTQ - 1) / kCellTQ);
    steps += (TP < kCellTP ? 1.3 : 1.0) * g.Na * (double)((tiles + 255) / 256);
  }
  return (double)pr.N > (lam > 0.0f && lam < 1.0f ? 15000.0 : 12300.0) * steps;
}

// The scan-major area of the reverse (after bwd_workspace_for).  In two launches:
// abar before and after the scan (fp32 volumes) and a pass's records (a byte
// volume).  In one: the image, abar twice and dL/dI, and two passes' records.
static size_t vol1_bytes(const Problem& pr) { return ((size_t)pr.N + 255) / 256 * 256; }
static size_t bwd_split_area(const Problem& pr) {
  if (pr.ndim != 3 || pr.dims[2] < 2) return 0;
  return 2 * scan_major_vol_bytes(pr) + vol1_bytes(pr);
}
static size_t bwd_fused_area(const Problem& pr) { return 4 * scan_major_vol_bytes(pr) + 2 * vol1_bytes(pr); }
size_t bwd_scan_major_bytes(const Problem& pr) {  // for any lambda
  return reverse_in_one_launch(pr, 1.0f) ? bwd_fused_area(pr) : bwd_split_area(pr);
}

// Descriptor of the reverse of forward pass p; a_in / a_out / xbuf set by the caller.
int build_bwd_pass(const Problem& pr, const float* image, const uint8_t* records, const float* spacing, float lam,
                   float* gI, int p, int K, unsigned epoch_base, BwdDesc* d) {
  PassDesc f;
  const int rc = build_pass(pr, image, nullptr, spacing, 1.0f, lam, nullptr, nullptr, p, 0, &f);
  if (rc) return rc;
  memset(d, 0, sizeof *d);
  d->image = image;
  d->rec = records + (size_t)p * pr.N;
  d->gI = gI;
  d->N = (int)pr.N;
  d->sa = f.sa;
  d->sp = f.sp;
  d->sq = f.sq;
  d->Na = f.Na;
  d->Np = f.Np;
  d->Nq = f.Nq;
  d->sign = f.sign;
  d->C = pr.C;
  d->TP = f.TP;
  d->TQ = f.TQ;
  d->K = K;
  d->ntp = f.ntp;
  d->ntq = f.ntq;
  d->nchunk = (f.Na - 1 + K - 1) / K;
  d->mode = f.mode;
  d->sqrt_normal = f.sqrt_normal;
  d->lam = lam;
  for (int j = 0; j < 9; ++j) d->A[j] = f.A[j];
  d->epoch_base = epoch_base;
  d->a_in_off = -1;
  d->a_out_off = -1;
  d->op = kOpPass;
  d->lsrc_off = d->ldst_off = d->image_off = d->rec_off = d->gi_off = -1;
  return GGDT_OK;
}

namespace {

// The reverse with a pass per launch, for the volumes that reverse_in_one_launch
// names; the words of ws are reset and the image is classified.  With room for
// them (sm: ws holds bwd_workspace_for(pr) + bwd_fused_area(pr) bytes) the passes
// along the last axis run on [W][D][H] copies of the image (moved once), of abar
// and dL/dI (moved there before each pair of those passes and back after it) and
// of the pair's records.
int reverse_passes(const Problem& pr, const float* image, const uint8_t* records, const float* grad_out,
                   const float* spacing, float v, float lam, int P, float* grad_image, float* grad_softmask, void* ws,
                   bool sm, hipStream_t stream) {
  unsigned* words = (unsigned*)ws;
  float* const scratch = (float*)((unsigned char*)ws + workspace_for(pr, Tuning{}));
  const int D0 = pr.dims[0], D1 = pr.dims[1], D2 = pr.dims[2];
  const size_t vol = scan_major_vol_bytes(pr);
  unsigned char* const area = (unsigned char*)ws + bwd_workspace_for(pr);
  float* const s_img = (float*)area;
  float* const s_a = (float*)(area + vol);
  float* const s_b = (float*)(area + 2 * vol);
  float* const s_g = (float*)(area + 3 * vol);
  uint8_t* const s_r[2] = {area + 4 * vol, area + 4 * vol + vol1_bytes(pr)};
  if (launch_reset((unsigned*)grad_image, (long long)pr.N, stream) != hipSuccess) return GGDT_ERR_HIP;
  if (sm && launch_to_scan_major(image, s_img, 4, D0, D1, D2, nullptr, stream) != hipSuccess) return GGDT_ERR_HIP;
  unsigned base = 0;
  const float* a_in = grad_out;
  for (int p = P - 1; p >= 0; --p) {
    const int k = p % 6;
    BwdDesc d;
    if (const int rc = build_bwd_pass(pr, image, records, spacing, lam, grad_image, p, kCellK, base, &d)) return rc;
    float* const a_out = p % 2 == 0 ? grad_softmask : scratch;  // P is even: the last pass writes grad_softmask
    d.a_in = a_in;
    d.a_out = a_out;
    d.xbuf = (unsigned long long*)(words + kHeaderWords);
    base += (unsigned)d.nchunk + 1u;
    if (sm && k == 5 &&  // first of the pair (2, -), (2, +) in reverse order
        (launch_to_scan_major(a_in, s_a, 4, D0, D1, D2, nullptr, stream) != hipSuccess ||
         launch_to_scan_major(grad_image, s_g, 4, D0, D1, D2, nullptr, stream) != hipSuccess ||
         launch_to_scan_major(records + (size_t)p * pr.N, s_r[0], 1, D0, D1, D2, nullptr, stream) != hipSuccess ||
         launch_to_scan_major(records + (size_t)(p - 1) * pr.N, s_r[1], 1, D0, D1, D2, nullptr, stream) !=
             hipSuccess))
      return GGDT_ERR_HIP;
    if (sm && k >= 4) {
      // planes (z, y) of the [W][D][H] copies: same tiles, offsets and constants
      d.sa = D0 * D1;
      d.sp = D1;
      d.sq = 1;
      d.image = s_img;
      d.rec = s_r[k == 5 ? 0 : 1];
      d.gI = s_g;
      d.a_in = k == 5 ? s_a : s_b;
      d.a_out = k == 5 ? s_b : s_a;
    }
    prof_before(stream);
    const hipError_t e = launch_bwd_pass(d, words, g_spin_limit, stream);
    prof_after(stream);
    if (e != hipSuccess) return GGDT_ERR_HIP;
    if (sm && k == 4 && (launch_from_scan_major(s_a, a_out, 4, D0, D1, D2, nullptr, stream) != hipSuccess ||
                         launch_from_scan_major(s_g, grad_image, 4, D0, D1, D2, nullptr, stream) != hipSuccess))
      return GGDT_ERR_HIP;
    a_in = a_out;
  }
  // dL/dM = v * abar
  return launch_scale(grad_softmask, v, grad_softmask, pr.N, stream) == hipSuccess ? GGDT_OK : GGDT_ERR_HIP;
}

int backward_entry(int ndim, const int* dims, int C, const float* image, const uint8_t* records,
                   const float* grad_out, const float* spacing, float v, float lam, int iterations, float* grad_image,
                   float* grad_softmask, void* ws, size_t wsb, hipStream_t stream) {
  if (!image || !records || !grad_out || !grad_image || !grad_softmask || !ws || !dims) return GGDT_ERR_NULL_PTR;
  Problem pr;
  int rc = make_problem(ndim, dims, C, &pr);
  if (rc) return rc;
  if (C > kMaxBwdChannels) return GGDT_ERR_BAD_SHAPE;
  rc = check_params(ndim, spacing, v, lam, iterations);
  if (rc) return rc;
  if (wsb < bwd_workspace_for(pr)) return GGDT_ERR_WORKSPACE_TOO_SMALL;
  const size_t nb = (size_t)pr.N * 4, ni = nb * C, nrec = (size_t)iterations * 2 * ndim * pr.N;
  {
    const void* ins[5] = {image, records, grad_out, ws, grad_softmask};
    const size_t nins[5] = {ni, nrec, nb, wsb, nb};
    if ((rc = check_alias(grad_image, ni, ins, nins, 5))) return rc;
    const void* ins2[4] = {image, records, grad_out, ws};
    const size_t nins2[4] = {ni, nrec, nb, wsb};
    if ((rc = check_alias(grad_softmask, nb, ins2, nins2, 4))) return rc;
  }
  if ((rc = check_device())) return rc;
  unsigned* words = (unsigned*)ws;
  const size_t fwd_ws = workspace_for(pr, Tuning{});
  unsigned long long* xbuf = (unsigned long long*)(words + kHeaderWords);
  float* scratch = (float*)((unsigned char*)ws + fwd_ws);
  if (launch_reset(words, (long long)(fwd_ws / 4), stream) != hipSuccess) return GGDT_ERR_HIP;
  if (iterations == 0) {
    if (launch_reset((unsigned*)grad_image, (long long)pr.N * C, stream) != hipSuccess) return GGDT_ERR_HIP;
    return launch_scale(grad_out, v, grad_softmask, pr.N, stream) == hipSuccess ? GGDT_OK : GGDT_ERR_HIP;
  }
  if (launch_classify(image, (long long)C * pr.N, words, stream) != hipSuccess) return GGDT_ERR_HIP;
  const int P = iterations * 2 * ndim;
  // The scans along the last axis of a volume run on [W][D][H] copies of abar
  // and of the records, where the workspace has room for them; the edges are
  // taken in the array layout.
  const size_t smb = bwd_split_area(pr), bmin = bwd_workspace_for(pr);
  const bool sm = smb > 0 && wsb >= bmin + smb;
  // (without room for any copies, the step with the edges is the faster one at
  // lambda 0 only: 256^3 two launches / one 3.65 / 3.41 ms, at 0.5 5.69 / 6.06)
  const bool room = wsb >= bmin + bwd_fused_area(pr);
  if (reverse_in_one_launch(pr, lam) && (room || (lam == 0.0f && !sm)))
    return reverse_passes(pr, image, records, grad_out, spacing, v, lam, P, grad_image, grad_softmask, ws, room,
                          stream);
  const int D0 = pr.dims[0], D1 = pr.dims[1], D2 = pr.dims[ndim - 1];
  float* const s_a = (float*)((unsigned char*)ws + bmin);
  float* const s_b = (float*)((unsigned char*)ws + bmin + scan_major_vol_bytes(pr));
  uint8_t* const s_r = (unsigned char*)ws + bmin + 2 * scan_major_vol_bytes(pr);
  unsigned base = 0;
  for (int p = P - 1; p >= 0; --p) {
    const int axis = (p % (2 * ndim)) / 2;
    const bool on_copy = sm && axis == 2;
    const float* a_in = p == P - 1 ? grad_out : grad_softmask;
    BwdDesc d;
    if ((rc = build_bwd_pass(pr, image, records, spacing, lam, grad_image, p, ndim == 3 ? kCellK : kRowK, base, &d)))
      return rc;
    d.a_in = a_in;
    d.a_out = scratch;
    d.xbuf = xbuf;
    if (ndim == 2) {
      d.TP = 1;
      d.TQ = kRowTQ;
    } else {
      cell_tile(d.Np, d.Nq, 1, &d.TP, &d.TQ);
    }
    d.ntp = (d.Np + d.TP - 1) / d.TP;
    d.ntq = (d.Nq + d.TQ - 1) / d.TQ;
    base += (unsigned)d.nchunk + 1u;
    BwdDesc scan = d;
    if (on_copy) {
      // planes (z, y) of the [W][D][H] copies: same tiles and offsets
      if (launch_to_scan_major(a_in, s_a, 4, D0, D1, D2, nullptr, stream) != hipSuccess ||
          launch_to_scan_major(d.rec, s_r, 1, D0, D1, D2, nullptr, stream) != hipSuccess)
        return GGDT_ERR_HIP;
      scan.sa = D0 * D1;
      scan.sp = D1;
      scan.sq = 1;
      scan.rec = s_r;
      scan.a_in = s_a;
      scan.a_out = s_b;
    }
    prof_before(stream);
    const hipError_t e = launch_bwd_scan(scan, ndim, words, g_spin_limit, stream);
    prof_after(stream);
    if (e != hipSuccess) return GGDT_ERR_HIP;
    if (on_copy && launch_from_scan_major(s_b, scratch, 4, D0, D1, D2, nullptr, stream) != hipSuccess)
      return GGDT_ERR_HIP;
    EdgeDesc s;
    s.a = scratch;
    s.out = grad_softmask;
    s.gI = grad_image;
    s.d1 = pr.dims[1];
    s.d2 = D2;
    s.axis = axis;
    s.first = p == P - 1;
    s.last = p == 0;  // dL/dM = v * abar
    s.v = v;
    if (launch_bwd_edges(d, ndim, s, words, stream) != hipSuccess) return GGDT_ERR_HIP;
  }
  return GGDT_OK;
}

}  // namespace
}  // namespace ggdt

using namespace ggdt;

extern "C" {

size_t ggdt_backward_workspace_bytes(int ndim, const int* dims, int C) {
  if (!dims) return 0;
  Problem pr;
  if (make_problem(ndim, dims, C, &pr) || C > kMaxBwdChannels) return 0;
  return bwd_workspace_for(pr) + bwd_scan_major_bytes(pr);
}

size_t ggdt_backward_workspace_min_bytes(int ndim, const int* dims, int C) {
  if (!dims) return 0;
  Problem pr;
  if (make_problem(ndim, dims, C, &pr) || C > kMaxBwdChannels) return 0;
  return bwd_workspace_for(pr);
}

int ggdt2d_backward(const float* image, const uint8_t* records, const float* grad_out, const float* spacing, float v,
                    float lambda, int iterations, float* grad_image, float* grad_softmask, int C, int H, int W,
                    void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const int dims[2] = {H, W};
  return backward_entry(2, dims, C, image, records, grad_out, spacing, v, lambda, iterations, grad_image,
                        grad_softmask, workspace, workspace_bytes, stream);
}

int ggdt3d_backward(const float* image, const uint8_t* records, const float* grad_out, const float* spacing, float v,
                    float lambda, int iterations, float* grad_image, float* grad_softmask, int C, int D, int H, int W,
                    void* workspace, size_t workspace_bytes, hipStream_t stream) {
  const int dims[3] = {D, H, W};
  return backward_entry(3, dims, C, image, records, grad_out, spacing, v, lambda, iterations, grad_image,
                        grad_softmask, workspace, workspace_bytes, stream);
}

}  // extern "C"
