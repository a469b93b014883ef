// Screen-space denoiser (Section 2.4.3) for gfx950: temporal accumulation of the interpolated
// irradiance over the reprojected history, then a spatial filter whose radius shrinks as the
// history grows (wider where the history is short: the dilated blur mask), edge-aware by depth
// and normal.  A separate object from the GI context: it needs only the G-buffer, the
// irradiance and the camera.
//
// Per pixel (one thread each):
//   temporal  the world position projected with the previous camera lands on a previous pixel;
//             the history is valid if that pixel held one, was not sky, lies within the
//             pixel's cell size (Algorithm 6) of its tangent plane and its normal's cosine
//             exceeds 0.9.  Valid: n = min(n_prev + 1, hist_max), value = hist + (E - hist) / n;
//             else n = 1, value = E.  A pixel without a probe (flag 2) keeps its history as it
//             is, or stays empty (n = 0).
//   radius    floor(radius_max / n) (radius_max at n = 0), 0 on sky.
//   spatial   R = the largest radius of the 3x3 neighbourhood; the mean over the (2R+1)^2 window
//             of the neighbours holding a value, weights cs / (cs + |depth difference|) times
//             max(0, normal cosine)^8, summed in row order.
// The accumulated values (before the spatial filter) and this G-buffer become the history: the
// temporal pass writes them into the other of two histories (29 + 32 us as a pass and a copy of
// its results and of the G-buffer, 36 us together).

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <new>

#include "gi.h"

namespace {

constexpr uint32_t kMiss = 0xFFFFFFFFu;

struct DnCamera {
  float pos[3], fwd[3], right[3], up[3];
  float tan_half;
};

// One of the two histories: accumulated values (rgb, n) and the G-buffer they were taken with
// (the normals' w: the view distance, so that a tap of the spatial filter is two reads)
struct DnHistory {
  float4 *acc, *pos, *nrm;
  uint32_t* prim;
};

struct DnArgs {
  const float4* pos;
  const float4* nrm;
  const uint32_t* prim;
  const float4* in;
  DnHistory h[2];
  // which history is the previous frame's: phase[0] for the temporal pass, phase[1] for the
  // spatial one.  In device memory, so that a replayed capture goes on from where it left off;
  // each pass reads its own word and writes the other's, so that no block of a launch can see
  // the change
  uint32_t* phase;
  uint32_t* rad;
  uint32_t W, H, hist_max, radius_max, has_prev;
  float kappa;
  float cam[3];
  DnCamera prev;
};

__device__ inline bool project_prev_cam(const DnCamera& pc, uint32_t W, uint32_t H, float Xx, float Xy, float Xz,
                                        uint32_t& qx, uint32_t& qy) {
  const float v0 = Xx - pc.pos[0], v1 = Xy - pc.pos[1], v2 = Xz - pc.pos[2];
  const float z = (v0 * pc.fwd[0] + v1 * pc.fwd[1]) + v2 * pc.fwd[2];
  if (!(z > 0.0f)) return false;
  const float a = ((v0 * pc.right[0] + v1 * pc.right[1]) + v2 * pc.right[2]) / z;
  const float b = ((v0 * pc.up[0] + v1 * pc.up[1]) + v2 * pc.up[2]) / z;
  const float aspect = (float)W / (float)H;
  const float sx = a / (pc.tan_half * aspect), sy = b / pc.tan_half;
  const float fx = ((sx + 1.0f) * (float)W) * 0.5f, fy = ((1.0f - sy) * (float)H) * 0.5f;
  if (!(fx >= 0.0f && fx < (float)W && fy >= 0.0f && fy < (float)H)) return false;
  qx = (uint32_t)fx;
  qy = (uint32_t)fy;
  return true;
}

__global__ __launch_bounds__(256) void k_dn_temporal(DnArgs d) {
  const uint32_t p = blockIdx.x * 256u + threadIdx.x;
  if (p >= d.W * d.H) return;
  const uint32_t ph = d.phase[0] & 1u;
  const DnHistory prev = d.h[ph], next = d.h[ph ^ 1u];
  if (p == 0) d.phase[1] = ph ^ 1u;
  const uint32_t prim = d.prim[p];
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
  uint32_t r = 0u;
  next.prim[p] = prim;
  if (prim != kMiss) {
    const float4 X = d.pos[p], n = d.nrm[p], E = d.in[p];
    next.pos[p] = X;
    next.nrm[p] = make_float4(n.x, n.y, n.z, X.w);
    bool hv = false;
    float4 Hh = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t qx, qy;
    if (d.has_prev && project_prev_cam(d.prev, d.W, d.H, X.x, X.y, X.z, qx, qy)) {
      const uint32_t q = qy * d.W + qx;
      Hh = prev.acc[q];
      if (prev.prim[q] != kMiss && Hh.w > 0.0f) {
        const float4 Xq = prev.pos[q], nq = prev.nrm[q];
        const float ex = X.x - d.cam[0], ey = X.y - d.cam[1], ez = X.z - d.cam[2];
        const float cs = d.kappa * sqrtf((ex * ex + ey * ey) + ez * ez);
        const float pd = fabsf(((Xq.x - X.x) * n.x + (Xq.y - X.y) * n.y) + (Xq.z - X.z) * n.z);
        const float nc = (nq.x * n.x + nq.y * n.y) + nq.z * n.z;
        hv = pd < cs && nc > 0.9f;
      }
    }
    if (E.w == 2.0f) {
      if (hv) a = Hh;
    } else if (hv) {
      const float np = Hh.w + 1.0f;
      const float nn = np < (float)d.hist_max ? np : (float)d.hist_max;
      a = make_float4(Hh.x + (E.x - Hh.x) / nn, Hh.y + (E.y - Hh.y) / nn, Hh.z + (E.z - Hh.z) / nn, nn);
    } else {
      a = make_float4(E.x, E.y, E.z, 1.0f);
    }
    const uint32_t nh = (uint32_t)a.w;
    r = nh == 0u ? d.radius_max : d.radius_max / nh;
  }
  next.acc[p] = a;
  d.rad[p] = r;
}

// the filtered value of pixel (x, y), R > 0
__device__ inline float4 dn_filter(const DnArgs& d, const DnHistory& h, int32_t x, int32_t y, int32_t r) {
  const int32_t W = (int32_t)d.W, H = (int32_t)d.H;
  const uint32_t p = (uint32_t)(y * W + x);
  const float4 X = d.pos[p], n = h.nrm[p];
  const float ex = X.x - d.cam[0], ey = X.y - d.cam[1], ez = X.z - d.cam[2];
  const float cs = d.kappa * sqrtf((ex * ex + ey * ey) + ez * ez);
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, ws = 0.f;
  const int32_t x0 = max(x - r, 0), x1 = min(x + r, W - 1), y0 = max(y - r, 0), y1 = min(y + r, H - 1);
  for (int32_t yy = y0; yy <= y1; ++yy) {
    uint32_t q = (uint32_t)(yy * W + x0);
    for (int32_t xx = x0; xx <= x1; ++xx, ++q) {
      const float4 aq = h.acc[q];
      if (aq.w == 0.0f) continue;             // no value: never a probe, or sky
      const float4 nq = h.nrm[q];
      const float nd = fmaxf(fmaf(n.z, nq.z, fmaf(n.y, nq.y, n.x * nq.x)), 0.0f);
      const float n2 = nd * nd, n4 = n2 * n2, n8 = n4 * n4;
      const float w = (cs / (cs + fabsf(nq.w - X.w))) * n8;
      s0 = fmaf(w, aq.x, s0);
      s1 = fmaf(w, aq.y, s1);
      s2 = fmaf(w, aq.z, s2);
      ws = ws + w;
    }
  }
  if (ws > 0.0f) return make_float4(s0 / ws, s1 / ws, s2 / ws, 0.f);
  return h.acc[p];
}

// A block filters a 16x16 square (a wave an 8x8 one).  Bound by the taps' VALU issue and L1 reads,
// and only the pixels of short history have any: they are found first and taken in dense waves,
// the wide windows before the narrow ones, where a wave of its own pixels walked the widest
// window of any of them (1080p, moving camera: 189 us in rows of 64 pixels, 158 in squares,
// 113 as now).  Wide is a radius above 2: with the line at 1 or 4 it takes 113.4 or 113.8, with
// none 115.9.
__global__ __launch_bounds__(256) void k_dn_spatial(DnArgs d, float4* out) {
  __shared__ uint32_t work[256], wide_s[4], narrow_s[4];
  const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
  const int32_t bx = (int32_t)(blockIdx.x * 16u), by = (int32_t)(blockIdx.y * 16u);
  const int32_t x = bx + (int32_t)((wv & 1u) * 8u + (t & 7u)), y = by + (int32_t)((wv >> 1) * 8u + ((t >> 3) & 7u));
  const int32_t W = (int32_t)d.W, H = (int32_t)d.H;
  const uint32_t ph = d.phase[1] & 1u;
  const DnHistory h = d.h[ph];
  uint32_t R = 0u;
  if (x < W && y < H) {
    const uint32_t p = (uint32_t)(y * W + x);
    if (p == 0) d.phase[0] = ph;
    const float E = d.in[p].w;
    if (d.prim[p] == kMiss) {
      out[p] = make_float4(0.f, 0.f, 0.f, E);
    } else {
      for (int32_t yy = max(y - 1, 0); yy <= min(y + 1, H - 1); ++yy)
        for (int32_t xx = max(x - 1, 0); xx <= min(x + 1, W - 1); ++xx) R = max(R, d.rad[yy * W + xx]);
      if (R == 0u) {
        const float4 a = h.acc[p];
        out[p] = make_float4(a.x, a.y, a.z, E);
      }
    }
  }
  const uint64_t below = (1ull << lane) - 1ull;
  const uint64_t wide = __ballot(R > 2u), narrow = __ballot(R > 0u && R <= 2u);
  if (lane == 0u) {
    wide_s[wv] = (uint32_t)__popcll(wide);
    narrow_s[wv] = (uint32_t)__popcll(narrow);
  }
  __syncthreads();
  uint32_t wide_at = 0, narrow_at = 0, total = 0;
#pragma unroll
  for (uint32_t k = 0; k < 4u; ++k) {
    if (k < wv) {
      wide_at += wide_s[k];
      narrow_at += narrow_s[k];
    }
    narrow_at += wide_s[k];
    total += wide_s[k] + narrow_s[k];
  }
  const uint32_t at = R > 2u ? wide_at + (uint32_t)__popcll(wide & below) : narrow_at + (uint32_t)__popcll(narrow & below);
  if (R > 0u) work[at] = R << 16 | (uint32_t)(y - by) << 8 | (uint32_t)(x - bx);
  __syncthreads();
  if (t >= total) return;
  const uint32_t k = work[t];
  const int32_t px = bx + (int32_t)(k & 255u), py = by + (int32_t)((k >> 8) & 255u);
  const uint32_t p = (uint32_t)(py * W + px);
  const float4 v = dn_filter(d, h, px, py, (int32_t)(k >> 16));
  out[p] = make_float4(v.x, v.y, v.z, d.in[p].w);
}

}  // namespace

struct gi_denoiser {
  uint32_t W = 0, H = 0, hist_max = 16, radius_max = 4;
  DnHistory h[2]{};
  uint32_t *phase = nullptr, *rad = nullptr;
  bool has_prev = false;
  gi_frame prev{};
};

namespace {

void dn_free(gi_denoiser* d) {
  for (const DnHistory& h : d->h)
    for (void* p : {(void*)h.acc, (void*)h.pos, (void*)h.nrm, (void*)h.prim})
      if (p) (void)hipFree(p);
  for (uint32_t* p : {d->phase, d->rad})
    if (p) (void)hipFree(p);
  delete d;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

extern "C" {

gi_status gi_denoiser_create(uint32_t width, uint32_t height, uint32_t hist_max, uint32_t radius_max,
                             gi_denoiser** out) {
  if (!out) return GI_ERR_INVALID_ARG;
  *out = nullptr;
  if (width < 8 || height < 8 || width > 8192 || height > 8192 || hist_max < 1 || hist_max > 1024 ||
      radius_max > 16)
    return GI_ERR_INVALID_ARG;
  gi_denoiser* d = new (std::nothrow) gi_denoiser();
  if (!d) return GI_ERR_OOM;
  d->W = width;
  d->H = height;
  d->hist_max = hist_max;
  d->radius_max = radius_max;
  const size_t n = (size_t)width * height;
  hipError_t e = hipSuccess;
  auto A = [&](hipError_t r) { if (e == hipSuccess) e = r; };
  for (DnHistory& h : d->h) {
    A(hipMalloc(&h.acc, 16 * n));
    A(hipMalloc(&h.pos, 16 * n));
    A(hipMalloc(&h.nrm, 16 * n));
    A(hipMalloc(&h.prim, 4 * n));
  }
  A(hipMalloc(&d->phase, 8));
  A(hipMalloc(&d->rad, 4 * n));
  if (e == hipSuccess) A(hipMemset(d->phase, 0, 8));
  if (e != hipSuccess) {
    dn_free(d);
    return e == hipErrorOutOfMemory ? GI_ERR_OOM : GI_ERR_HIP;
  }
  *out = d;
  return GI_OK;
}

void gi_denoiser_destroy(gi_denoiser* d) {
  if (d) dn_free(d);
}

gi_status gi_denoiser_reset(gi_denoiser* d) {
  if (!d) return GI_ERR_INVALID_ARG;
  d->has_prev = false;
  return GI_OK;
}

gi_status gi_denoise(gi_denoiser* d, const gi_frame* f, const float* pos, const float* nrm, const uint32_t* prim,
                     const float* irradiance, float* out, void* stream) {
  if (!d || !f || !pos || !nrm || !prim || !irradiance || !out) return GI_ERR_INVALID_ARG;
  if (!aligned16(pos) || !aligned16(nrm) || !aligned16(irradiance) || !aligned16(out)) return GI_ERR_INVALID_ARG;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  DnArgs a;
  a.pos = reinterpret_cast<const float4*>(pos);
  a.nrm = reinterpret_cast<const float4*>(nrm);
  a.prim = prim;
  a.in = reinterpret_cast<const float4*>(irradiance);
  a.h[0] = d->h[0];
  a.h[1] = d->h[1];
  a.phase = d->phase;
  a.rad = d->rad;
  a.W = d->W;
  a.H = d->H;
  a.hist_max = d->hist_max;
  a.radius_max = d->radius_max;
  a.has_prev = d->has_prev ? 1u : 0u;
  {
    // Algorithm 6's distance scale on the host in float64, rounded once
    const double x = 1.0 / (double)d->H, y = (double)d->H / ((double)d->W * (double)d->W);
    a.kappa = (float)std::tan((double)f->fov_y * 8.0 * (x > y ? x : y));
  }
  for (int k = 0; k < 3; ++k) {
    a.cam[k] = f->pos[k];
    a.prev.pos[k] = d->prev.pos[k];
    a.prev.fwd[k] = d->prev.fwd[k];
    a.prev.right[k] = d->prev.right[k];
    a.prev.up[k] = d->prev.up[k];
  }
  a.prev.tan_half = d->prev.tan_half;
  const uint32_t n = d->W * d->H, blocks = (n + 255u) / 256u;
  k_dn_temporal<<<blocks, 256, 0, s>>>(a);
  k_dn_spatial<<<dim3((d->W + 15u) / 16u, (d->H + 15u) / 16u), 256, 0, s>>>(a, reinterpret_cast<float4*>(out));
  if (hipGetLastError() != hipSuccess) return GI_ERR_HIP;
  d->prev = *f;
  d->has_prev = true;
  return GI_OK;
}

gi_status gi_denoiser_export(gi_denoiser* d, float* h_hist, uint32_t* h_radius) {
  if (!d) return GI_ERR_INVALID_ARG;
  if (hipDeviceSynchronize() != hipSuccess) return GI_ERR_HIP;
  const size_t n = (size_t)d->W * d->H;
  uint32_t phase = 0;
  if (h_hist && hipMemcpy(&phase, d->phase, 4, hipMemcpyDeviceToHost) != hipSuccess) return GI_ERR_HIP;
  if (h_hist && hipMemcpy(h_hist, d->h[phase & 1u].acc, 16 * n, hipMemcpyDeviceToHost) != hipSuccess) return GI_ERR_HIP;
  if (h_radius && hipMemcpy(h_radius, d->rad, 4 * n, hipMemcpyDeviceToHost) != hipSuccess) return GI_ERR_HIP;
  return GI_OK;
}

}  // extern "C"
