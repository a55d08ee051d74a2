// Kernels of the path-guiding hot path for gfx950.
//
// One lane per pixel.  Streaming passes (reprojection, sampling, densities,
// light field) use 64x4 blocks so that each wave reads one 256-byte row
// segment of every plane.  The training pass stages the sample records of a
// tile plus a 3-pixel halo in LDS as float4 (direction, L/p_src or 0), so the
// neighbour picks of Sec. 4.2 are LDS reads, and maps block ids to tiles so
// that each XCD works on one contiguous band of the image (its L2 then holds
// the halo rows its neighbours share).
#pragma once
#include "pg_device.hpp"

namespace pgk {

struct ViewK {
  int W, H, pitch;
  const float *n, *o, *z, *rough, *alb, *mv;
  const uint8_t *mask;
};

struct ParamsK {
  uint32_t key0, key1, frame, view;
  int k_max;
  float pi_init, pi_lo, pi_hi, eps, tau_z, tau_n, rough_min, s_d, f0;
  uint32_t flags;
  float stale_tau;
  // material constants derived on the host (FP32, as the device would round
  // them), so that kernels take them as uniform operands
  float s_d_pi, one_m_f0, one_m_sd_q;  // s_d / pi, 1 - f0, (1 - s_d) / (4 pi)
};

struct SamplesK {
  int spp;
  float *dir, *pmix, *pb, *L;
  uint8_t *strat;
};

constexpr uint32_t kNoClamp = 1u;
constexpr uint32_t kStaleReset = 4u;
constexpr int kR = 3;                       // pick radius: 7x7 window
constexpr int kSide = 2 * kR + 1;
constexpr int kCand = kSide * kSide - 1;    // 48 neighbours

// Blocks are dealt to the 8 XCDs round robin; xcd_tile gives XCD j the j-th
// contiguous run of the n tiles, so that neighbouring tiles (which share
// cache lines and halos) are fetched into the same L2.
__device__ __forceinline__ int xcd_tile(int bid, int n) {
  // blocks are dealt to the 8 XCDs round robin; give XCD j the j-th
  // contiguous run of tiles
  const int xcd = bid & 7, local = bid >> 3;
  const int base = n >> 3, rem = n & 7;
  return xcd * base + min(xcd, rem) + local;
}

// Streaming kernels: one 64x4 pixel tile per block of a 1-D grid, tiles in
// XCD bands.
__device__ __forceinline__ void stream_xy(int W, int H, int &x, int &y) {
  const int tx = (W + 63) >> 6, n = tx * ((H + 3) >> 2);
  const int t = xcd_tile((int)blockIdx.x, n);
  x = (t % tx) * 64 + (int)threadIdx.x;
  y = (t / tx) * 4 + (int)threadIdx.y;
}

__device__ __forceinline__ V3 load3(const float *p, int plane, int idx) {
  return V3{at(p, idx), at(p + plane, idx), at(p + 2 * plane, idx)};
}

__device__ __forceinline__ void gamma_reset(const ParamsK &P, float g[8]) {
  g[0] = 0.5f;
  g[1] = 0.5f;
  g[2] = 1.0f / 12.0f;
  g[3] = 0.0f;
  g[4] = 1.0f / 12.0f;
  g[5] = P.pi_init;
  g[6] = 0.0f;
  g[7] = 0.0f;
}

// Per-pixel material constants in the local frame.
__device__ __forceinline__ Pixel make_pixel(const ParamsK &P, V3 n, V3 o, float rough, float albedo) {
  Pixel px;
  px.f = make_frame(n);
  px.wo = to_local(px.f, normalized(o));
  const float alpha = rough * rough;
  px.alpha2 = alpha * alpha;
  px.albedo_pi = albedo * kInvPi;
  const float g1 = smith_g1(px.wo, px.alpha2) * frcp(2.0f * kPi * px.wo.z);
  px.f0_g1 = P.f0 * g1;
  px.omf0_g1 = P.one_m_f0 * g1;
  px.s_d = P.s_d;
  px.s_d_pi = P.s_d_pi;
  px.one_m_sd_q = P.one_m_sd_q;
  return px;
}

// ---------------------------------------------------------------------------
// Reprojection of one pixel (Sec. 3.1).  The decisions that turn FP32 inputs
// into a source address or a reset flag use explicit operation orders:
// validity and the normal test are fma(z, z', fma(y, y', x * x')), the
// address is (x + 1/2) - mv, the depth test |z - z'| > tau z.
// The G-buffer values of one pixel that both reprojection and sampling read.
struct PixelIn {
  V3 n, o;
  float rough;
};

__device__ __forceinline__ PixelIn load_pixel(const ViewK &v, int idx) {
  const int plane = v.H * v.pitch;
  return PixelIn{load3(v.n, plane, idx), load3(v.o, plane, idx), at(v.rough, idx)};
}

template <typename TG>
__device__ __forceinline__ int reproject_pixel(const ParamsK &P, const ViewK &cur, const ViewK &prev,
                                               const TG *__restrict__ gprev, bool has_prev, int x,
                                               int y, const PixelIn &pi, float g[8]) {
  const int plane = cur.H * cur.pitch;
  const int idx = y * cur.pitch + x;
  const V3 n = pi.n;
  const bool guided = dot3(n, pi.o) > 0.0f && pi.rough >= P.rough_min;
  // everything read at p, then everything read at the source q: two rounds
  // of loads whatever the tests decide
  float zp = 0.0f, mx = 0.0f, my = 0.0f;
  bool keep = has_prev && guided;
  if (keep) {
    zp = at(cur.z, idx);
    if (cur.mv) {
      mx = at(cur.mv, idx);
      my = at(cur.mv + plane, idx);
    }
    if (cur.mask != nullptr && at(cur.mask, idx) != 0) keep = false;
  }
  int qx = 0, qy = 0;
  if (keep) {
    const float fx = ((float)x + 0.5f) - mx;
    const float fy = ((float)y + 0.5f) - my;
    if (fx >= 0.0f && fy >= 0.0f && fx < (float)prev.W && fy < (float)prev.H) {
      qx = (int)floorf(fx);
      qy = (int)floorf(fy);
    } else {
      keep = false;
    }
  }
  if (keep) {
    const int pplane = prev.H * prev.pitch;
    const int qidx = qy * prev.pitch + qx;
    const float zq = at(prev.z, qidx);
    const V3 nq = load3(prev.n, pplane, qidx);
    gamma_load(gprev, pplane, qidx, g);
    if (fabsf(zp - zq) > P.tau_z * zp) keep = false;
    if (dot3(n, nq) < P.tau_n) keep = false;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (!isfinite(g[c])) keep = false;
    if (keep && !(n.x == nq.x && n.y == nq.y && n.z == nq.z)) {
      // change of hemisphere: keep the world direction of M(mu)
      const Frame fq = make_frame(nq);
      const Frame fp = make_frame(n);
      const V3 lq = sq2hemi(fminf(fmaxf(g[0], 0.0f), 1.0f), fminf(fmaxf(g[1], 0.0f), 1.0f));
      const V3 lp = to_local(fp, to_world(fq, lq));
      if (lp.z <= 0.0f) {
        keep = false;
      } else {
        hemi2sq(normalized(lp), g[0], g[1]);
      }
    }
  }
  if (!keep) {
    gamma_reset(P, g);
    return -1;
  }
  return qy * prev.W + qx;
}

// First-bounce estimate of one pixel: the mean over its samples of
// f_r L cos / D (null samples count zero), the Monte Carlo estimator of the
// reflected radiance with the mixture density of the samples.  Bound by HBM
// (21 B a record, 36 B a pixel).  A record is loaded and evaluated without a
// branch on what it holds: with its strategy tested first, its other loads
// waited for that one (1080p: 90.8 us at 8 spp, now 78: 5.4 TB/s; 19.7 and 19.0
// at 1 spp).  The records of four samples in flight cost 19 registers and, where
// there are not as many samples, loads (1 spp 20.7, 3 spp 32.7 against 30.1, 8
// spp 80.8).
__global__ __launch_bounds__(256) void k_estimate(ParamsK P, ViewK v, SamplesK S, float *__restrict__ out) {
  int x, y;
  stream_xy(v.W, v.H, x, y);
  if (x >= v.W || y >= v.H) return;
  const int plane = v.H * v.pitch;
  const int idx = row_off(y, v.pitch) + x;
  const int splane = S.spp * plane;
  const V3 n = load3(v.n, plane, idx), o = load3(v.o, plane, idx);
  const float rough = at(v.rough, idx), albedo = at(v.alb, idx);
  float acc = 0.0f;
  if (dot3(n, o) > 0.0f) {
    const Pixel px = make_pixel(P, n, o, rough, albedo);
    for (int s = 0; s < S.spp; ++s) {
      const int r = s * plane + idx;
      const uint32_t code = at(S.strat, r);
      const float D = at(S.pmix, r), L = at(S.L, r);
      const V3 l = to_local(px.f, normalized(load3(S.dir, splane, r)));
      float f, pb;
      brdf_eval(px, l, f, pb);
      const float sum = acc + f * L * l.z / D;
      acc = (code == 1 || code == 2) && D > 0.0f && !(l.z <= 0.0f) ? sum : acc;
    }
    acc /= (float)S.spp;
  }
  at(out, idx) = acc;
}

// Analytic incident radiance (stand-in for the trace).  For unit w and xi,
// w . xi - 1 = -|w - xi|^2 / 2, which has no cancellation near the axis.
struct LightsK {
  int count;
  float ambient;
  float l[8][5];
};

// exp(x) = 2^n exp2(x log2(e) - n) to about 1 ulp over FP32's whole range,
// subnormal results included: n whole, the rest formed in two fused steps (the
// second adds what log2(e) lost to FP32) and at most 1/2, where the hardware
// exp2 is accurate.  Beyond the range the rest keeps the sign and the clamp of
// n keeps inf - inf from x = +-inf: 0 and inf there, NaN for NaN.
__device__ __forceinline__ float exp_fast(float x) {
  const float n = rintf(__builtin_amdgcn_fmed3f(x * 1.44269504088896340736f, -160.0f, 160.0f));
  const float y = fmaf(x, 1.92596299e-8f, fmaf(x, 1.44269504088896340736f, -n));
  return ldexpf(__builtin_amdgcn_exp2f(y), (int)n);
}

__device__ __forceinline__ float light_radiance(const LightsK &Lt, uint32_t bits, V3 wdir) {
  const V3 w = normalized(wdir);
  float L = Lt.ambient;
  for (int k = 0; k < Lt.count; ++k) {
    const V3 a = V3{w.x - Lt.l[k][0], w.y - Lt.l[k][1], w.z - Lt.l[k][2]};
    // (every light is evaluated: with a bit per pixel and light hardly any
    // wave could skip one)
    const float with = fmaf(Lt.l[k][4], exp_fast(-0.5f * Lt.l[k][3] * dot3(a, a)), L);
    L = ((bits >> k) & 1u) ? with : L;
  }
  return L;
}

// ---------------------------------------------------------------------------
// Sampling of one pixel (Sec. 3.1, Eq. (2)).  Each strategy's own density is
// taken in its sample space (Gaussian from z, GGX from xi_1), the other
// component from the direction.
// With Lt given, the radiance of each sample is evaluated as well (the
// batched frame fuses the trace stand-in into this pass).
__device__ __forceinline__ void sample_pixel(const ParamsK &P, const ViewK &v, const SamplesK &S,
                                             int x, int y, const PixelIn &pi, const float g[8],
                                             const LightsK *Lt = nullptr, uint32_t visbits = 0) {
  const int plane = v.H * v.pitch;
  const int splane = S.spp * plane;
  const V3 n = pi.n;
  const V3 o = pi.o;
  const float rough = pi.rough;
  const bool valid = dot3(n, o) > 0.0f;
  const bool guided = valid && rough >= P.rough_min;
  const float pe = (guided && g[7] >= 1.0f) ? g[5] : 0.0f;
  const Pixel px = make_pixel(P, n, o, rough, 0.0f);
  const Gauss G = gauss_setup(g[0], g[1], g[2], g[3], g[4], P.eps);
  const uint32_t pix = (uint32_t)(y * v.W + x);
  for (int s = 0; s < S.spp; ++s) {
    const int rec = (s * v.H + y) * v.pitch + x;
    uint8_t code = 0;
    V3 l = V3{0.0f, 0.0f, 0.0f};
    float D = 0.0f, pb = 0.0f;
    if (valid) {
      const uint4 w4 = philox4x32_10(pix, P.frame, (uint32_t)s, P.view, P.key0, P.key1);
      const float zeta = u24(w4.x), xl = u24(w4.y), x1 = u24(w4.z), x2 = u24(w4.w);
      float sn, cs;
      sincospi_small(2.0f * x2, &sn, &cs);
      // the guided and the cosine draws take p_b from the direction, after
      // the branches, so that a wave whose lanes took both evaluates it once
      bool pb_dir = false;
      float pgz = 0.0f;  // the Gaussian density of a guided draw, from z
      if (zeta < pe) {
        // -2 ln(1 - x1) = -2 ln2 log2(1 - x1); 1 - x1 >= 2^-24 is normal
        const float rho = fsqrt(-1.38629436f * __builtin_amdgcn_logf(1.0f - x1));
        const float z1 = rho * cs, z2 = rho * sn;
        const float ux = fmaf(G.l11, z1, G.mx);
        const float uy = fmaf(G.l22, z2, fmaf(G.l21, z1, G.my));
        if (ux >= 0.0f && ux <= 1.0f && uy >= 0.0f && uy <= 1.0f) {
          l = sq2hemi(ux, uy);
          pgz = G.norm * __builtin_amdgcn_exp2f(-0.72134752f * fmaf(z1, z1, z2 * z2));
          pb_dir = l.z > 0.0f;
          code = 2;
        } else {
          code = 3;
        }
      } else if (xl < P.s_d) {
        const float r = fsqrt(x1);
        l = V3{r * cs, r * sn, fsqrt(1.0f - x1)};
        pb_dir = l.z > 0.0f;
        code = pb_dir ? 1 : 4;
      }
      if (pb_dir) pb = brdf_pdf_only(px, l);
      if (code == 2) {
        D = fmaf(pe, pgz, (1.0f - pe) * pb);
      } else if (code == 0) {
        // the GGX draw (the only strategy left without a code)
        // x1 <= 1 - 2^-24, so 1 - x1 and t2 (0 or >= alpha^2 2^-24) are normal
        const float t2 = px.alpha2 * x1 * frcp(1.0f - x1);
        const float ch = __builtin_amdgcn_rsqf(1.0f + t2);
        const float sh = fsqrt(t2) * ch;
        const V3 h = V3{sh * cs, sh * sn, ch};
        const float woh = dot3(px.wo, h);
        l = V3{2.0f * woh * h.x - px.wo.x, 2.0f * woh * h.y - px.wo.y, 2.0f * woh * h.z - px.wo.z};
        const bool ok = l.z > 0.0f && woh > 0.0f;
        if (ok) {
          // GGX density of the drawn normal in closed form of xi_1:
          // D(h) = (1 - xi_1 (1 - alpha^2))^2 / (pi alpha^2)
          const float q = fmaf(-x1, 1.0f - px.alpha2, 1.0f);
          const float pggx = 0.25f * kInvPi * q * q * ch * frcp(px.alpha2 * woh);
          pb = fmaf(px.s_d * kInvPi, l.z, (1.0f - px.s_d) * pggx);
        }
        code = ok ? 1 : 4;
      }
      if (code == 1) {  // a BRDF draw: the Gaussian's density from the direction
        float pg = 0.0f;
        if (pe > 0.0f) {
          float ux, uy;
          hemi2sq(l, ux, uy);
          pg = gauss_pdf_fast(G, ux, uy);
        }
        D = fmaf(pe, pg, (1.0f - pe) * pb);
      }
    }
    V3 w = V3{0.0f, 0.0f, 0.0f};
    if (code == 1 || code == 2) {
      w = to_world(px.f, l);
    } else {
      D = 0.0f;
      pb = 0.0f;
    }
    at(S.dir, rec) = w.x;
    at(S.dir + splane, rec) = w.y;
    at(S.dir + 2 * splane, rec) = w.z;
    at(S.pmix, rec) = D;
    at(S.pb, rec) = pb;
    at(S.strat, rec) = code;
    if (Lt) at(S.L, rec) = (code == 1 || code == 2) ? light_radiance(*Lt, visbits, w) : 0.0f;
  }
}

template <typename TG>
__global__ __launch_bounds__(256) void k_reproject(ParamsK P, ViewK cur, ViewK prev,
                                                   const TG *__restrict__ gprev, TG *__restrict__ gout,
                                                   int32_t *__restrict__ src_index, int has_prev) {
  int x, y;
  stream_xy(cur.W, cur.H, x, y);
  if (x >= cur.W || y >= cur.H) return;
  float g[8];
  const int idx = y * cur.pitch + x;
  const int src = reproject_pixel(P, cur, prev, gprev, has_prev != 0, x, y, load_pixel(cur, idx), g);
  gamma_store(gout, cur.H * cur.pitch, idx, g);
  if (src_index) at(src_index, idx) = src;
}

template <typename TG>
__global__ __launch_bounds__(256) void k_sample(ParamsK P, ViewK v, const TG *__restrict__ gamma,
                                                SamplesK S) {
  int x, y;
  stream_xy(v.W, v.H, x, y);
  if (x >= v.W || y >= v.H) return;
  float g[8];
  const int idx = y * v.pitch + x;
  gamma_load(gamma, v.H * v.pitch, idx, g);
  sample_pixel(P, v, S, x, y, load_pixel(v, idx), g);
}

// Reprojection and sampling of one pixel: the reprojected model stays in
// registers, the sample pass sees it exactly as stored (rounded to TG), and
// the state is stored last (after the G-buffer has been read once).
template <typename TG>
__device__ __forceinline__ void reproject_sample_pixel(const ParamsK &P, const ViewK &cur, const ViewK &prev,
                                                       const TG *__restrict__ gprev, TG *__restrict__ gout,
                                                       const SamplesK &S, bool has_prev, int x, int y,
                                                       const LightsK *Lt = nullptr,
                                                       const uint8_t *vis = nullptr) {
  const int idx = y * cur.pitch + x;
  const PixelIn pi = load_pixel(cur, idx);
  const uint32_t visbits = vis ? at(vis, idx) : 0u;
  float g[8];
  reproject_pixel(P, cur, prev, gprev, has_prev, x, y, pi, g);
  float gs[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    TG t;
    gamma_put(&t, c, g[c]);
    gs[c] = gamma_get(&t, c);
  }
  sample_pixel(P, cur, S, x, y, pi, gs, Lt, visbits);
  gamma_store(gout, cur.H * cur.pitch, idx, g);
}

template <typename TG>
__global__ __launch_bounds__(256) void k_reproject_sample(ParamsK P, ViewK cur, ViewK prev,
                                                          const TG *__restrict__ gprev,
                                                          TG *__restrict__ gout, SamplesK S,
                                                          int has_prev) {
  int x, y;
  stream_xy(cur.W, cur.H, x, y);
  if (x >= cur.W || y >= cur.H) return;
  reproject_sample_pixel(P, cur, prev, gprev, gout, S, has_prev != 0, x, y);
}

// Densities of given directions.
template <typename TG>
__global__ __launch_bounds__(256) void k_pdf(ParamsK P, ViewK v, const TG *__restrict__ gamma, int n_per_px,
                                             const float *__restrict__ dir, float *__restrict__ pmix,
                                             float *__restrict__ pguide, float *__restrict__ pbrdf) {
  int x, y;
  stream_xy(v.W, v.H, x, y);
  if (x >= v.W || y >= v.H) return;
  const int plane = v.H * v.pitch;
  const int idx = y * v.pitch + x;
  const int dplane = n_per_px * plane;
  float g[8];
  gamma_load(gamma, plane, idx, g);
  const V3 n = load3(v.n, plane, idx);
  const V3 o = load3(v.o, plane, idx);
  const float rough = at(v.rough, idx);
  const bool valid = dot3(n, o) > 0.0f;
  const bool guided = valid && rough >= P.rough_min;
  const float pe = (guided && g[7] >= 1.0f) ? g[5] : 0.0f;
  const Pixel px = make_pixel(P, n, o, rough, 0.0f);
  const Gauss G = gauss_setup(g[0], g[1], g[2], g[3], g[4], P.eps);
  for (int j = 0; j < n_per_px; ++j) {
    const int r = (j * v.H + y) * v.pitch + x;
    const V3 w = load3(dir, dplane, r);
    float pg = 0.0f, pb = 0.0f;
    const float ww = dot3(w, w);
    if (valid && ww > 0.0f) {
      const V3 l = to_local(px.f, normalized(w));
      if (l.z > 0.0f) {
        float ux, uy;
        hemi2sq(l, ux, uy);
        pg = gauss_pdf_acc(G, ux, uy);
        pb = brdf_pdf_only(px, l);
      }
    }
    at(pmix, r) = fmaf(pe, pg, (1.0f - pe) * pb);
    if (pguide) at(pguide, r) = pg;
    if (pbrdf) at(pbrdf, r) = pb;
  }
}


// The light field over the records of one sample plane per blockIdx.y.  FOUR:
// four pixels of a row a lane in blocks of 32x8 lanes (128x8 pixels): 16-byte
// loads and stores, and four independent chains of arithmetic to cover them.
// Bound by HBM: 17 B a record and 1 B a pixel.  One pixel a lane and all of its
// samples in turn took 79 us in a 1080p frame of 8 spp (now 57: 5.3 TB/s) and,
// on records that the Infinity Cache partly holds, 66 us (now 45) and at 4K and
// 1 spp 34 us (now 23).  Without FOUR one pixel a lane (64x4), a quarter of the
// work in each: the shorter chain where the lanes do not fill the chip anyway.
template <bool FOUR>
__global__ __launch_bounds__(256) void k_light(LightsK Lt, ViewK v, const uint8_t *__restrict__ vis,
                                               SamplesK S) {
  const int plane = v.H * v.pitch, splane = S.spp * plane, s = (int)blockIdx.y;
  constexpr int BW = FOUR ? 128 : 64, BH = FOUR ? 8 : 4;
  const int tx = (v.W + BW - 1) / BW, n = tx * ((v.H + BH - 1) / BH);
  const int t = xcd_tile((int)blockIdx.x, n);
  const int x = (t % tx) * BW + (FOUR ? 4 : 1) * (int)threadIdx.x, y = (t / tx) * BH + (int)threadIdx.y;
  if (x >= v.W || y >= v.H) return;
  const int idx = row_off(y, v.pitch) + x, r = s * plane + idx;
  if (FOUR && x + 4 <= v.W) {
    const uint32_t bits = vis ? load4(vis, idx) : 0u, st = load4(S.strat, r);
    const F4 dx = load4(S.dir, r), dy = load4(S.dir + splane, r), dz = load4(S.dir + 2 * splane, r);
    F4 L;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t code = (st >> (8 * j)) & 0xFFu;
      const float l = light_radiance(Lt, bits >> (8 * j), V3{dx[j], dy[j], dz[j]});
      L[j] = code == 1 || code == 2 ? l : 0.0f;
    }
    store4(S.L, r, L);
    return;
  }
  for (int j = 0; FOUR ? x + j < v.W : j < 1; ++j) {  // the end of a row, or the lane's one pixel
    const uint8_t code = at(S.strat, r + j);
    const uint32_t bits = vis ? at(vis, idx + j) : 0u;
    const V3 w = load3(S.dir, splane, r + j);
    at(S.L, r + j) = code == 1 || code == 2 ? light_radiance(Lt, bits, w) : 0.0f;
  }
}

// ---------------------------------------------------------------------------
// Training pass (Sec. 3.2, Sec. 4.2).
//
// Block = one TW x TH tile; LDS holds the records of the tile and a
// 3-pixel halo for every sample index: float4 (direction, L / p_src) with 0
// in the last slot for records that are not BRDF-strategy samples or lie
// outside the image (such records add nothing to any sum, which is the same
// as leaving them out of the training set).

// A tile's records are read four at a time: the window of TW + 8 columns from
// tx0 - 4 on (the halo of 3 and one more on either side) is whole groups of
// four, whose 16-byte loads start at multiples of 16 bytes in a plane of
// aligned rows.  One record a lane, as before, started 12 bytes off those
// multiples and split a wave over three rows: the address units spent 23
// cycles on each such load (4 on an aligned one), half of the two-pass
// kernel's time at spp 8, and the plane-by-plane rounds their latency on top.
template <int TW, int TH>
struct Window {
  static constexpr int SW = TW + 8, G = SW / 4, SH = TH + 2 * kR, NG = SH * G, NT = TW * TH;
  static_assert(TW % 4 == 0 && NG % 2 == 0, "groups of four, in pairs");
};

// Group `item` of the records of sample planes s0, s0 + 1, ... of a tile:
// four records of one row.
struct RecordGroup {
  F4 x, y, z, l, p;
  uint32_t st;  // the four strategy codes
  uint32_t in;  // bits 0-3: record j lies inside the image; from bit 8 on: the
                // records by which the loads start before the group
};

// Plane, row and group column of an item (item < 2^13: the float quotients
// floor exactly).
template <int TW, int TH>
__device__ __forceinline__ void item_place(int item, int &s, int &sy, int &g) {
  using Wn = Window<TW, TH>;
  s = (int)(((float)item + 0.5f) * (1.0f / Wn::NG));
  const int r = item - (int)__umul24((uint32_t)s, (uint32_t)Wn::NG);
  sy = (int)(((float)r + 0.5f) * (1.0f / Wn::G));
  g = r - (int)__umul24((uint32_t)sy, (uint32_t)Wn::G);
}

// Issue the loads of an item (no use of the results here): strategy and
// density (KEY) and direction and radiance (REC).  The loads take no branch:
// a group outside the image reads the planes' first records, and one that
// would cross the end of the planes (its row's end, in the last row of an
// image whose pitch is no multiple of 4) starts up to three records early.
// The planes must hold four records or more in all (stage_few otherwise).
template <int TW, int TH, bool KEY, bool REC>
__device__ __forceinline__ void load_group(const ViewK &v, const SamplesK &S, int tx0, int ty0, int s0, int item,
                                           RecordGroup &q) {
  int s, sy, g;
  item_place<TW, TH>(item, s, sy, g);
  const int plane = v.H * v.pitch, splane = S.spp * plane;
  const int gx = tx0 - 4 + 4 * g, gy = ty0 - kR + sy;
  const int n = min(v.W - gx, 4);  // records before the right edge
  const bool in = gy >= 0 && gy < v.H && gx >= 0 && n > 0;
  const int o0 = in ? (s0 + s) * plane + row_off(gy, v.pitch) + gx : 0;
  const int o = min(o0, splane - 4);
  q.in = (in ? (1u << n) - 1u : 0u) | (uint32_t)(o0 - o) << 8;
  if (KEY) q.st = load4(S.strat, o);
  q.p = load4(S.pb, o);
  if (REC) {
    q.x = load4(S.dir, o);
    q.y = load4(S.dir + splane, o);
    q.z = load4(S.dir + 2 * splane, o);
    q.l = load4(S.L, o);
  }
}

// A group at its place, once its loads have come back.  (The barrier keeps the
// compiler from testing values, and so awaiting them, right after their own
// loads, before it issues others.)
template <bool REC>
__device__ __forceinline__ void settle(RecordGroup &q) {
  asm volatile("" : "+v"(q.st), "+v"(q.p));
  for (uint32_t d = q.in >> 8; d > 0; --d) {
    q.st >>= 8;
    q.p = q.p.yzww;
    if (REC) {
      q.x = q.x.yzww;
      q.y = q.y.yzww;
      q.z = q.z.yzww;
      q.l = q.l.yzww;
    }
  }
}

// Whether record j of a group trains: a BRDF-strategy sample inside the image
// (its density is a normal number: at least s_d cos/pi of a valid draw, or
// the GGX density of the drawn normal).
__device__ __forceinline__ bool group_valid(const RecordGroup &q, int j) {
  return ((q.in >> j) & 1u) != 0u && ((q.st >> (8 * j)) & 0xFFu) == 1u && q.p[j] > 0.0f;
}
__device__ __forceinline__ float group_weight(const RecordGroup &q, int j) {
  return q.l[j] * frcp(fmaxf(q.p[j], 1.17549435e-38f));
}

// A group's records to the LDS of the single-pass tile, [spp][TH+6][TW+6]:
// L / p_src is 0 for a record that does not train (and the rest of it is
// then never read).
template <int TW, int TH>
__device__ __forceinline__ void put_group(float4 *lds, int item, RecordGroup &q) {
  constexpr int SW = TW + 2 * kR, SA = SW * (TH + 2 * kR), G = Window<TW, TH>::G;
  int s, sy, g;
  item_place<TW, TH>(item, s, sy, g);
  const int e = s * SA + (int)__umul24((uint32_t)sy, (uint32_t)SW) + 4 * g - 1;
  settle<true>(q);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if ((j > 0 || g > 0) && (j < 3 || g < G - 1))
      lds[e + j] = make_float4(q.x[j], q.y[j], q.z[j], group_valid(q, j) ? group_weight(q, j) : 0.0f);
}

// The single-pass tile's records from item `begin` on (all sample planes).
template <int TW, int TH>
__device__ __forceinline__ void stage_records(const ViewK &v, const SamplesK &S, float4 *lds, int tx0, int ty0,
                                              int begin) {
  const int n = S.spp * Window<TW, TH>::NG;
  for (int i = begin + (int)threadIdx.x; i < n; i += TW * TH) {
    RecordGroup q;
    load_group<TW, TH, true, true>(v, S, tx0, ty0, 0, i, q);
    put_group<TW, TH>(lds, i, q);
  }
}

// Sample planes of fewer than four records in all (an image of one to three
// pixels) hold no group: their records one by one.
__device__ __forceinline__ bool few_records(const ViewK &v, const SamplesK &S) { return S.spp * v.H * v.pitch < 4; }
template <int TW, int TH>
__device__ __forceinline__ void stage_few(const ViewK &v, const SamplesK &S, float4 *lds, int tx0, int ty0) {
  constexpr int SW = TW + 2 * kR, SA = SW * (TH + 2 * kR);
  const int plane = v.H * v.pitch, splane = S.spp * plane;
  for (int i = threadIdx.x; i < S.spp * SA; i += TW * TH) {
    const int s = i / SA, e = i - s * SA, gx = tx0 - kR + e % SW, gy = ty0 - kR + e / SW;
    float4 r = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (gx >= 0 && gy >= 0 && gx < v.W && gy < v.H) {
      const int o = s * plane + row_off(gy, v.pitch) + gx;
      const float p = at(S.pb, o);
      if (at(S.strat, o) == 1 && p > 0.0f)
        r = make_float4(at(S.dir, o), at(S.dir + splane, o), at(S.dir + 2 * splane, o),
                        at(S.L, o) * frcp(fmaxf(p, 1.17549435e-38f)));
    }
    lds[i] = r;
  }
}

// Running sums of one E-step: B0 = sum w, B1 = sum w gamma, and the
// weighted mean (mx, my) and normalised scatter (sxx, sxy, syy) of the
// samples' points under the weights v = w gamma, updated per sample in the
// pairwise form
//   m += (v / B1') d,   S = (B1 / B1') (S + (v / B1') d d^T),   d = r - m,
// which has no cancellation when a heavy sample follows light ones.  The
// points are r = u - mu, relative to the lobe's mean before the step (the
// value the Gaussian term needs anyway, exact near the mean); accum_to_unit
// adds the mean back once, after the last sample.  A Gaussian weight below
// FP32's normal range counts as no evidence, so the reciprocal of B1' is
// always of a normal number.
struct Accum {
  float B0, B1, mx, my, sxx, sxy, syy;
};

// The mean of the points r = u - mu back to u (the scatter is the same).
__device__ __forceinline__ void accum_to_unit(Accum &a, const LobeTerm &t) {
  a.mx += 0.5f - t.hx;
  a.my += 0.5f - t.hy;
}

// Stepwise merge of one frame's E-step sums into the state (Sec. 3.2):
// eta = 1/(k+1) and the evidence W; only ratios of evidences appear, so a
// subnormal B1 is harmless.
__device__ __forceinline__ void em_merge_online(const ParamsK &P, float g[8], const Accum &a) {
  const float eta = frcp(g[7] + 1.0f);  // k + 1 in [1, kMax + 1]
  const float sw = fmaf(1.0f - eta, g[6], eta * a.B0);
  const float so = (1.0f - eta) * g[5] * g[6];
  const float sn = eta * a.B1;
  const float sg = so + sn;
  if (sg > 0.0f && a.B1 > 0.0f) {
    float al, be;
    div2_pos(so, sn, sg, al, be);
    const float dx = g[0] - a.mx, dy = g[1] - a.my;
    const float ab = al * be;
    g[0] = fmaf(al, g[0], be * a.mx);
    g[1] = fmaf(al, g[1], be * a.my);
    g[2] = fmaf(ab * dx, dx, fmaf(al, g[2], be * a.sxx));
    g[3] = fmaf(ab * dx, dy, fmaf(al, g[3], be * a.sxy));
    g[4] = fmaf(ab * dy, dy, fmaf(al, g[4], be * a.syy));
  }
  float pn = div_pos(sg, sw);  // sg <= sw: B1 <= B0 and pi <= 1
  if (!(P.flags & kNoClamp)) pn = fminf(fmaxf(pn, P.pi_lo), P.pi_hi);
  g[5] = pn;
  g[6] = sw;
  g[7] = fminf(g[7] + 1.0f, (float)P.k_max);
}

struct EmCtx {
  Pixel px;
  LobeTerm T;  // the lobe's Gaussian term
  float pi;
};

// One training sample of a list (its staged record is never zero: lists
// hold only BRDF-strategy records inside the image).  Mean and scatter
// accumulate relative to the lobe's centre (see Accum).
__device__ __forceinline__ void em_visit(const EmCtx &c, float4 r, Accum &a) {
  const V3 l = to_local(c.px.f, V3{r.x, r.y, r.z});
  if (l.z <= 0.0f) return;
  float cx, cy, f, pb;
  hemi2sq_c(l, cx, cy);
  const float rx = cx + c.T.hx, ry = cy + c.T.hy;
  brdf_eval(c.px, l, f, pb);
  const float w = r.w * f * l.z;
  const float ga = lobe_eval(c.T, rx, ry);
  const float gb = fmaf(-c.pi, pb, pb);  // (1 - pi) p_b, one rounding
  const float gam = ga * __builtin_amdgcn_rcpf(fmaxf(ga + gb, 1.17549435e-38f));
  a.B0 += w;
  const float vw = w * gam;
  if (vw >= 1.17549435e-38f) {
    const float bn = a.B1 + vw;
    const float rb = __builtin_amdgcn_rcpf(bn);
    const float fr = vw * rb, keep = a.B1 * rb;
    a.B1 = bn;
    const float dx = rx - a.mx, dy = ry - a.my;
    a.mx = fmaf(dx, fr, a.mx);
    a.my = fmaf(dy, fr, a.my);
    const float fx = fr * dx, fy = fr * dy;
    a.sxx = keep * fmaf(fx, dx, a.sxx);
    a.sxy = keep * fmaf(fx, dy, a.sxy);
    a.syy = keep * fmaf(fy, dy, a.syy);
  }
}

// Pick table of a tile shape (records in rows of SW, planes of SA), after the
// lists in dynamic LDS: code c in [0, 48 spp) of a pick, (o, s) = (c div spp,
// c mod spp), the centre of the window skipped and (dx, dy) = (o mod 7 - 3, o
// div 7 - 3), to the offset s SA + dy SW + dx of its candidate from the
// pixel's own record of plane 0, so that a pick costs one LDS read and one
// addition.  Built once per block.
__host__ __device__ constexpr int pick_table_bytes(int spp) { return (kCand * spp * 2 + 15) & ~15; }

template <int SA, int SW>
__device__ __forceinline__ void build_pick_table(int16_t *tab, int spp) {
  // c div spp = (c ceil(2^16 / spp)) >> 16, exact for c < 48 spp
  const uint32_t inv_spp = (65536u + (uint32_t)spp - 1u) / (uint32_t)spp;
  for (int c = (int)threadIdx.x; c < kCand * spp; c += (int)blockDim.x) {
    const uint32_t o0 = __umul24((uint32_t)c, inv_spp) >> 16;
    const int s = c - (int)__umul24(o0, (uint32_t)spp);
    const uint32_t o = o0 + (o0 >= (uint32_t)(kCand / 2) ? 1u : 0u);
    const uint32_t row = __umul24(o, 37u) >> 8;  // o / 7, exact for o < 49
    tab[c] = (int16_t)(s * SA + (int)(o + __umul24(row, (uint32_t)(SW - kSide))) - (kR * SW + kR));
  }
}

// The two-pass training tile (from spp 4) holds the records of the first
// ceil(spp/2) sample planes at a time; its dynamic LDS: those records
// [PG][TH+6][TW+8] float4, a validity bit for every candidate record of all
// planes [spp][TH+6][TW+8], the lists [spp+20][w h] uint16, the pick table
// and, per pixel, the list's entries in the first pass [w h] uint8.  (Rows of
// whole groups of four: two lanes' groups are one byte of bits.)
__host__ __device__ constexpr bool em2_spp(int spp) { return spp >= 4; }  // (pmmguide.hip gives the figures)
__host__ __device__ constexpr int em2_planes(int spp) { return (spp + 1) >> 1; }
__host__ __device__ constexpr int em2_stride(int tw, int th) { return (tw + 8) * (th + 2 * kR); }
__host__ __device__ constexpr size_t em2_bits_bytes(int tw, int th, int spp) {
  return ((size_t)spp * em2_stride(tw, th) / 8 + 15) & ~(size_t)15;
}
__host__ __device__ constexpr size_t em2_lds_front(int tw, int th, int spp) {
  return (size_t)em2_stride(tw, th) * em2_planes(spp) * 16 + em2_bits_bytes(tw, th, spp) +
         (size_t)(spp + 20) * tw * th * 2 + (size_t)pick_table_bytes(spp) + (size_t)tw * th;
}

// Where a training tile's lists start in dynamic LDS (after the records, and
// in the two-pass tile after the validity bits); the pick table follows the
// lists.
template <int TW, int TH, bool TWO>
__device__ __forceinline__ uint16_t *em_lists(float4 *lds, int spp) {
  constexpr int SA = (TW + 2 * kR) * (TH + 2 * kR);
  if (TWO)
    return reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(lds + em2_planes(spp) * em2_stride(TW, TH)) +
                                        em2_bits_bytes(TW, TH, spp));
  return reinterpret_cast<uint16_t *>(lds + spp * SA);
}

// The pick table of a training tile, at its place in dynamic LDS (called by
// every thread before em_tile; em_tile's first barrier publishes it).
template <int TW, int TH, bool TWO = false>
__device__ __forceinline__ void build_em_pick_table(float4 *lds, int spp) {
  constexpr int SW = TW + (TWO ? 8 : 2 * kR), SA = SW * (TH + 2 * kR), NT = TW * TH;
  build_pick_table<SA, SW>(reinterpret_cast<int16_t *>(em_lists<TW, TH, TWO>(lds, spp) + (spp + 20) * NT), spp);
}

// Number of neighbour picks N(k) = 5 + floor(15 (kMax - k) / kMax) (Sec. 4.2).
// The quotient is at most 15, so the product with the reciprocal is off by at
// most one, which the remainder shows (an integer division is 25
// instructions).
__device__ __forceinline__ int n_picks(const ParamsK &P, int k) {
  k = min(max(k, 0), P.k_max);
  const int a = 15 * (P.k_max - k);
  int q = (int)((float)a * frcp((float)P.k_max));
  const int r = a - q * P.k_max;
  q += (r >= P.k_max ? 1 : 0) - (r < 0 ? 1 : 0);
  return 5 + q;
}

// A list entry is the byte offset of its staged record from the start of the
// records area (below 64 KiB: the area is part of one block's LDS), so that
// the record's LDS address is the entry plus a constant.
__device__ __forceinline__ float4 list_record(const float4 *lds, uint32_t off) {
  return *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(lds) + off);
}

// Calls f on the staged records of n list entries of one pixel, at rows
// j0, j0 + step, ... of its column (column `me` of the [rows][nt] list
// area).  AHEAD = 0: one record at a time (its entry's and its own LDS
// reads wait in turn); AHEAD = 1: the next record is read from LDS before
// f runs on the current one (its entry's read still waits); AHEAD = 2: the
// next record and the entry after it, so both dependent LDS reads of a
// visit pass during the previous visits' arithmetic (four more registers).
// Reads past the last entry repeat the last entry (always a staged record).
template <int AHEAD, typename F>
__device__ __forceinline__ void for_each_record(const float4 *rec, const uint16_t *list, int nt, int me, int j0,
                                                int step, int n, F &&f) {
  static_assert(AHEAD >= 0 && AHEAD <= 2, "look-ahead of at most two records");
  if (n <= 0) return;
  const uint16_t *col = list + me;
  if (AHEAD == 0) {
    for (int i = 0; i < n; ++i) f(list_record(rec, col[(j0 + step * i) * nt]));
    return;
  }
  const int last = n - 1;
  auto entry = [&](int i) { return (uint32_t)col[(j0 + step * min(i, last)) * nt]; };
  float4 r0 = list_record(rec, entry(0));
  if (AHEAD == 1) {
    for (int i = 0; i < n; ++i) {
      const float4 r1 = list_record(rec, entry(i + 1));
      f(r0);
      r0 = r1;
    }
  } else {
    uint32_t off1 = entry(1);
    for (int i = 0; i < n; ++i) {
      const uint32_t off2 = entry(i + 2);
      const float4 r1 = list_record(rec, off1);
      f(r0);
      r0 = r1;
      off1 = off2;
    }
  }
}

// Training list of one pixel: the LDS byte offsets of its kept candidates, in the
// order of the training set (own samples by sample index, then picks by pick
// index), stored in column `col` of the list area.  A candidate is kept when
// its staged record is a BRDF-strategy sample inside the image.  Candidates
// are examined eight at a time (one Philox call): their addresses are formed
// in registers and their records read together, then appended without
// branches (a rejected candidate's slot is overwritten by the next one; the
// area has room for every candidate).  Returns the list length.
template <int TW, int TH>
__device__ __forceinline__ int build_list(const ParamsK &P, const float4 *lds, const int16_t *ptab, uint16_t *list,
                                          int col, int lx, int ly, int npick, int spp, uint32_t pix) {
  constexpr int SW = TW + 2 * kR, SH = TH + 2 * kR, SA = SW * SH, NT = TW * TH;
  const uint32_t cs = (uint32_t)(kCand * spp);
  const int own = (ly + kR) * SW + (lx + kR);
  int n = 0;
  {
    float wv[kMaxSpp];
#pragma unroll
    for (int s = 0; s < kMaxSpp; ++s) wv[s] = s < spp ? lds[s * SA + own].w : 0.0f;
#pragma unroll
    for (int s = 0; s < kMaxSpp; ++s)
      if (s < spp) {
        list[n * NT + col] = (uint16_t)((s * SA + own) << 4);
        n += wv[s] != 0.0f ? 1 : 0;
      }
  }
  for (int m0 = 0; m0 < npick; m0 += 8) {
    const uint4 w4 = philox4x32_10(pix, P.frame, (1u << 16) | (uint32_t)(m0 >> 3), P.view, P.key0, P.key1);
    int e[8];
    float wv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // the 16-bit field j of the four words, scaled to a code in [0, 48 spp)
      const uint32_t word = (j >> 1) == 0 ? w4.x : (j >> 1) == 1 ? w4.y : (j >> 1) == 2 ? w4.z : w4.w;
      const uint32_t h = (j & 1) ? (word >> 16) : (word & 0xFFFFu);
      e[j] = own + ptab[__umul24(h, cs) >> 16];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) wv[j] = lds[e[j]].w;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (m0 + j < npick) {
        list[n * NT + col] = (uint16_t)(e[j] << 4);
        n += wv[j] != 0.0f ? 1 : 0;
      }
  }
  return n;
}

// Rejection of a stale history (the stronger rejection of reprojected models
// that Sec. 5 leaves open, as read here): the weighted log-likelihood of the
// pixel's training set under the model, l_m = sum w log(pi p_g + (1 - pi)
// p_b), against the one under a new model (reset lobe, pi_init), l_r; the
// history is stale when l_m - l_r < -stale_tau sum w.  A pass of its own
// over the list, so that the E-step is untouched when the test is off.
__device__ __forceinline__ bool stale_history(const ParamsK &P, const Pixel &px, const float g[8],
                                              const float4 *lds, const uint16_t *list, int me, int len, int nt) {
  const Gauss G = gauss_setup(g[0], g[1], g[2], g[3], g[4], P.eps);
  const Gauss G0 = gauss_setup(0.5f, 0.5f, 1.0f / 12.0f, 0.0f, 1.0f / 12.0f, P.eps);
  const float pi = g[5], pi0 = P.pi_init;
  float lm = 0.0f, lr = 0.0f, ws = 0.0f;
  for (int j = 0; j < len; ++j) {
    const float4 r = list_record(lds, list[j * nt + me]);
    const V3 l = to_local(px.f, V3{r.x, r.y, r.z});
    if (l.z <= 0.0f) continue;
    float ux, uy, f, pb;
    hemi2sq(l, ux, uy);
    brdf_eval(px, l, f, pb);
    const float w = r.w * f * l.z;
    const float dm = fmaf(pi, gauss_pdf_acc(G, ux, uy), (1.0f - pi) * pb);
    const float dr = fmaf(pi0, gauss_pdf_acc(G0, ux, uy), (1.0f - pi0) * pb);
    if (!(w > 0.0f) || !(dm > 0.0f) || !(dr > 0.0f)) continue;
    lm = fmaf(w, __logf(dm), lm);
    lr = fmaf(w, __logf(dr), lr);
    ws += w;
  }
  return ws > 0.0f && (lm - lr) < -P.stale_tau * ws;
}

// Counting sort of the tile's items by decreasing work `len` (0 .. kMaxLen -
// 1) so that the lanes of a wave carry nearly equal work (the order inside a
// class is irrelevant: a pixel's arithmetic does not depend on the lane that
// runs it).  The k-th heaviest group of 64 items goes to wave (k + rot) mod
// waves, so that the heavy waves of the blocks resident on a CU do not all
// land on the same SIMD.  cnt[0 .. kMaxLen) must be zero and visible to the
// block on entry.  Each thread offers `item`; returns the item this lane
// takes.
constexpr int kMaxLen = kMaxSpp + 21;
constexpr int kTrained = 128;  // flag beside a list length: the pixel trains

template <int NT>
__device__ __forceinline__ int balance(int len, int item, int *cnt, uint16_t *perm, int rot) {
  static_assert(kMaxLen <= 32, "one half-wave scans the classes");
  const int rank = atomicAdd(&cnt[len], 1);
  __syncthreads();
  if (threadIdx.x < 64) {
    // wave 0: cnt[b] <- items in the classes heavier than b (suffix scan)
    const int l = threadIdx.x;
    const int c = l < kMaxLen ? cnt[l] : 0;
    int x = c;
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
      const int y = __shfl_down(x, d, 64);
      if (l + d < 32) x += y;
    }
    if (l < kMaxLen) cnt[l] = x - c;
  }
  __syncthreads();
  constexpr int NW = NT / 64;
  const int pos = cnt[len] + rank;                                // rank in the sorted order
  const int wave = NW > 1 ? ((pos >> 6) + rot) % NW : 0;
  perm[wave * 64 + (pos & 63)] = (uint16_t)item;
  __syncthreads();
  return perm[threadIdx.x];
}

// LDS of one training tile besides the dynamic records/state/lists area.
template <int NT>
struct EmShared {
  int cnt[2][kMaxLen];
  uint16_t perm[NT];
  uint8_t work[NT];  // per pixel: candidate count, then list length
};

// Dynamic LDS of the single-lobe training kernels: the records
// [spp][h+6][w+6] float4, the lists [spp+20][w h] uint16 and the pick table
// (the block's EmShared is static).  Keeping EmShared static measured 2% faster
// than placing it after the dynamic area, where the records would start at
// LDS address 0 and the list entries could serve as addresses directly.
__host__ __device__ constexpr size_t em_lds_front(int tw, int th, int spp) {
  return (size_t)(tw + 2 * kR) * (th + 2 * kR) * spp * 16 + (size_t)(spp + 20) * tw * th * 2 +
         (size_t)pick_table_bytes(spp);
}

// What decides a pixel's candidate count (epoch, normal, view direction,
// roughness; natural order).
struct EmPixel {
  float k, rough;
  V3 n, o;
};

template <typename Op>
__device__ __forceinline__ EmPixel em_load_pixel(const ViewK &v, const Op &op, int tx0, int ty0, int tw) {
  const int plane = v.H * v.pitch;
  // clamped into the image, so that the loads need no branch (a branch made
  // the compiler await the epoch inside it, before anything else was issued);
  // the caller masks what lies outside
  const int x0 = min(tx0 + (int)threadIdx.x % tw, v.W - 1), y0 = min(ty0 + (int)threadIdx.x / tw, v.H - 1);
  const int idx0 = row_off(y0, v.pitch) + x0;
  return EmPixel{op.epoch(plane, idx0), at(v.rough, idx0), load3(v.n, plane, idx0), load3(v.o, plane, idx0)};
}

// A single-pass tile's inputs in flight: a thread's pixel and its first group
// of records.
template <int TW, int TH>
struct EmInput {
  EmPixel q;
  RecordGroup r;
};

// Issue the loads of a tile's inputs (no use of the results here).
template <typename Op, int TW, int TH>
__device__ __forceinline__ void em_load(const ViewK &v, const SamplesK &S, const Op &op, int tx0, int ty0,
                                        EmInput<TW, TH> &R) {
  R.q = em_load_pixel(v, op, tx0, ty0, TW);
  if ((int)threadIdx.x < S.spp * Window<TW, TH>::NG && !few_records(v, S))
    load_group<TW, TH, true, true>(v, S, tx0, ty0, 0, (int)threadIdx.x, R.r);
}

// What a training tile does with each pixel's training set, as a type `Op`:
//   epoch(plane, idx)        the k that decides the number of picks
//   load(plane, idx, g)      the pixel's state or parameters
//   Ctx context(P, px, g)    what a visit needs of the pixel
//   visit(ctx, record, acc)  one member of the training set
//   finish(P, ctx, acc, idx, g)  the pixel's results, in g
//   put(ch), store(plane, idx, out)  the channels of g that are results
// kEvery: the pixels with an empty training set have results of their own
// (EM leaves them as they are).  EmOp is the EM update of a state.
template <typename TG>
struct EmOp {
  using Ctx = EmCtx;
  using Acc = Accum;
  static constexpr bool kEvery = false;
  TG *gamma;
  __device__ __forceinline__ float epoch(int plane, int idx) const { return gamma_get(&at(gamma + 7 * plane, idx), 7); }
  __device__ __forceinline__ void load(int plane, int idx, float g[8]) const { gamma_load(gamma, plane, idx, g); }
  static __device__ __forceinline__ Ctx context(const ParamsK &P, const Pixel &px, const float g[8]) {
    return Ctx{px, lobe_term(gauss_setup(g[0], g[1], g[2], g[3], g[4], P.eps), g[5]), g[5]};
  }
  static __device__ __forceinline__ void visit(const Ctx &c, float4 r, Acc &a) { em_visit(c, r, a); }
  __device__ __forceinline__ void finish(const ParamsK &P, const Ctx &c, Acc &a, int, float g[8]) const {
    if (!(a.B0 > 0.0f)) return;  // no weight: the model stays as it is
    accum_to_unit(a, c.T);
    em_merge_online(P, g, a);
  }
  static constexpr bool put(int ch) { return ch < 8; }
  __device__ __forceinline__ void store(int plane, int idx, const float out[8]) const {
    gamma_store(gamma, plane, idx, out);
  }
};

// Plain batch EM of one pixel: `iterations` rounds on its training list (mu,
// Sigma and pi replaced; W and k kept).
__device__ __forceinline__ void em_batch(const ParamsK &P, const Pixel &px, const float4 *lds, const uint16_t *list,
                                         int me, int len, int nt, int iterations, float g[8]) {
  for (int it = 0; it < iterations; ++it) {
    const EmCtx c = EmOp<float>::context(P, px, g);
    Accum a = {0, 0, 0, 0, 0, 0, 0};
    // more state live than online: one record at a time
    for_each_record<0>(lds, list, nt, me, 0, 1, len, [&](float4 r) { em_visit(c, r, a); });
    if (!(a.B0 > 0.0f)) break;
    accum_to_unit(a, c.T);
    if (a.B1 > 0.0f) {
      g[0] = a.mx;
      g[1] = a.my;
      g[2] = a.sxx;
      g[3] = a.sxy;
      g[4] = a.syy;
    }
    float pn = div_pos(a.B1, a.B0);
    if (!(P.flags & kNoClamp)) pn = fminf(fmaxf(pn, P.pi_lo), P.pi_hi);
    g[5] = pn;
  }
}

// A tile's results from the sorted lanes to global memory in natural order
// (full cache lines), through LDS [channels][NT] over the dead records.
template <typename Op, int NT>
__device__ __forceinline__ void tile_write_back(const Op &op, float *wb, int me, bool me_in, const float g[8], int t,
                                                bool in_image, int plane, int idx0) {
  if (me_in) {
#pragma unroll
    for (int ch = 0; ch < 8; ++ch)
      if (Op::put(ch)) wb[ch * NT + me] = g[ch];
  }
  __syncthreads();
  if (in_image) {
    float go[8];
#pragma unroll
    for (int ch = 0; ch < 8; ++ch)
      if (Op::put(ch)) go[ch] = wb[ch * NT + t];
    op.store(plane, idx0, go);
  }
}

// One training tile.  Its inputs arrive in R (what decides each pixel's
// candidate count, natural order; records of plane 0; further planes are
// staged here): stage the records in LDS; sort the pixels by candidate count
// and build each pixel's training list; sort them again by list length, load
// each pixel's state and material in that order and run the E- and M-steps;
// write the tile's Gamma back in natural order through LDS (full cache
// lines).  Every thread of the block calls it and
// none leaves early; a block that runs several tiles synchronises between
// them (the write-back area overlaps the records).
// Dynamic LDS: records [spp][SH][SW] float4, then lists [spp + 20][NT]
// uint16, then the pick table [48 spp] int16; the write-back reuses the area
// ([8][NT] float).
template <typename Op, int TW, int TH, bool STALE = false, bool BATCH = false>
__device__ __forceinline__ void em_tile(const ParamsK &P, const ViewK &v, const SamplesK &S, const Op &op,
                                        int iterations, int tx0, int ty0, int rot, float4 *lds,
                                        EmShared<TW * TH> &sh, EmInput<TW, TH> &R) {
  constexpr int SA = (TW + 2 * kR) * (TH + 2 * kR), NT = TW * TH;
  uint16_t *list = reinterpret_cast<uint16_t *>(lds + S.spp * SA);
  float *wb = reinterpret_cast<float *>(lds);  // write-back area, once the records are no longer read
  const int plane = v.H * v.pitch;
  const int t = threadIdx.x;
  const int x0 = tx0 + t % TW, y0 = ty0 + t / TW;
  const bool in_image = x0 < v.W && y0 < v.H;
  const int16_t *ptab = reinterpret_cast<const int16_t *>(list + (S.spp + 20) * NT);
  if (t < 2 * kMaxLen) (&sh.cnt[0][0])[t] = 0;
  if (few_records(v, S)) {
    stage_few<TW, TH>(v, S, lds, tx0, ty0);
  } else {
    if (t < S.spp * Window<TW, TH>::NG) put_group<TW, TH>(lds, t, R.r);
    if (S.spp * Window<TW, TH>::NG > NT) stage_records<TW, TH>(v, S, lds, tx0, ty0, NT);
  }
  // the number of candidates of this lane's pixel (0 when it is not trained)
  int ncand = 0;
  if (in_image && dot3(R.q.n, R.q.o) > 0.0f && R.q.rough >= P.rough_min) ncand = S.spp + n_picks(P, (int)R.q.k);
  sh.work[t] = (uint8_t)ncand;
  __syncthreads();
  // lists: pixels by decreasing candidate count
  int me;
  {
    const int pa = balance<NT>(ncand, t, sh.cnt[0], sh.perm, rot);
    const int nc = sh.work[pa];
    int len = 0;
    if (nc > 0) {
      const int lx = pa % TW, ly = pa / TW;
      len = build_list<TW, TH>(P, lds, ptab, list, pa, lx, ly, nc - S.spp, S.spp,
                               (uint32_t)(row_off(ty0 + ly, v.W) + tx0 + lx));
    }
    sh.work[pa] = (uint8_t)(Op::kEvery && nc > 0 ? len | kTrained : len);
    // E- and M-steps: pixels by decreasing list length
    me = balance<NT>(len, pa, sh.cnt[1], sh.perm, rot + 1);
  }
  const int len = Op::kEvery ? sh.work[me] & (kTrained - 1) : sh.work[me];
  const bool run = Op::kEvery ? (sh.work[me] & kTrained) != 0 : len > 0;
  float g[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  // every pixel of the tile, trained or not, passes its state to the
  // natural-order write-back through LDS (the loads run for the trained
  // lanes of the wave anyway)
  const int mex = tx0 + me % TW, mey = ty0 + me / TW;
  const bool me_in = mex < v.W && mey < v.H;
  const int idx = row_off(mey, v.pitch) + mex;
  if (Op::kEvery ? run : me_in) op.load(plane, idx, g);
  Pixel px;
  if (run) {
    px = make_pixel(P, load3(v.n, plane, idx), load3(v.o, plane, idx), at(v.rough, idx), at(v.alb, idx));
    if constexpr (STALE && !BATCH)
      if (g[7] >= 1.0f && stale_history(P, px, g, lds, list, me, len, NT)) gamma_reset(P, g);
  }
  if (run) {
    if constexpr (BATCH) {
      em_batch(P, px, lds, list, me, len, NT, iterations, g);
    } else {
      const typename Op::Ctx c = Op::context(P, px, g);
      typename Op::Acc a = {};
      // at spp 1 one record at a time: 8 waves per SIMD cover the LDS
      // latency, and a look-ahead's index arithmetic measured 3% slower;
      // above, the staged records leave 4-5 waves and the reads go ahead
      if (S.spp > 1)
        for_each_record<2>(lds, list, NT, me, 0, 1, len, [&](float4 r) { Op::visit(c, r, a); });
      else
        for_each_record<0>(lds, list, NT, me, 0, 1, len, [&](float4 r) { Op::visit(c, r, a); });
      op.finish(P, c, a, idx, g);
    }
  }
  __syncthreads();  // records and lists are no longer read
  tile_write_back<Op, NT>(op, wb, me, me_in, g, t, in_image, plane, row_off(y0, v.pitch) + x0);
}

// Two-pass training tile (from spp 4).  Above spp 1 the staged records of
// every sample plane fill the LDS and few blocks share a CU (at spp 8, two).
// Here the records of the first PG = ceil(spp/2) planes are staged, with one
// validity bit per candidate record of all planes; each pixel's list is built
// once, as in em_tile, storing its entries of the first planes from the
// front of its column and those of the last planes from the back; the E-step
// runs over the first planes, the records area is restaged with the last
// planes, and the same sums continue over them.  Each pass keeps the
// training set's order, so the result does not depend on the tile shape.
// What bounds it at 1080p and 8 spp (333 to 341 us; 381 before its records were
// staged in groups and its lists kept by address): VALU issue 59% of the
// cycles at 2.6 of 3 waves per SIMD; without any visit 205 us, with records
// that hit the caches 293.  Reading the second pass's records ahead into
// registers (355), windows on whole 128-byte lines (341) and two visits side by
// side (345) gained nothing.

// A group's records (REC) and validity bits (KEY) to the LDS of the two-pass
// tile: records at their own item, bits at `bit_item` (the same unless the
// planes before are not among the items).  The lanes of a pair of groups,
// neighbours in a wave, form one byte of bits.
template <int TW, int TH, bool KEY, bool REC>
__device__ __forceinline__ void put_group2(float4 *rec, uint8_t *vb, int item, int bit_item, RecordGroup &q) {
  settle<REC>(q);
  if (KEY) {
    uint32_t b = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) b |= group_valid(q, j) ? 1u << j : 0u;
    const uint32_t hi = (uint32_t)__shfl_down((int)b, 1, 64);
    if ((item & 1) == 0) vb[bit_item >> 1] = (uint8_t)(b | (hi << 4));
  }
  if (REC) {
#pragma unroll
    for (int j = 0; j < 4; ++j)  // (a record whose bit is not set is never read)
      rec[4 * item + j] = make_float4(q.x[j], q.y[j], q.z[j], group_weight(q, j));
  }
}

// Staging of the two-pass tile: validity bits of every sample plane, and the
// records of the first `pg`; then, in their place, those of the others.  A
// first round holds two groups a thread in flight (42 registers), and with
// them two of the planes that need bits alone; what is left (16 groups of 528
// in a 16x16 tile at spp 7 and 8) follows one by one.  The first round is no
// part of the loop: at a loop's head the compiler awaits what the round before
// left in flight.
template <int TW, int TH>
__device__ __forceinline__ void stage2_first(const ViewK &v, const SamplesK &S, float4 *rec, uint8_t *vb, int tx0,
                                             int ty0, int pg) {
  constexpr int NT = TW * TH, NG = Window<TW, TH>::NG;
  const int t = threadIdx.x, n = pg * NG, m = (S.spp - pg) * NG;
  RecordGroup a, b, c, d;
  if (t < n) load_group<TW, TH, true, true>(v, S, tx0, ty0, 0, t, a);
  if (t + NT < n) load_group<TW, TH, true, true>(v, S, tx0, ty0, 0, t + NT, b);
  if (t < m) load_group<TW, TH, true, false>(v, S, tx0, ty0, pg, t, c);
  if (t + NT < m) load_group<TW, TH, true, false>(v, S, tx0, ty0, pg, t + NT, d);
  if (t < n) put_group2<TW, TH, true, true>(rec, vb, t, t, a);
  if (t + NT < n) put_group2<TW, TH, true, true>(rec, vb, t + NT, t + NT, b);
  if (t < m) put_group2<TW, TH, true, false>(rec, vb, t, n + t, c);
  if (t + NT < m) put_group2<TW, TH, true, false>(rec, vb, t + NT, n + t + NT, d);
  for (int i = t + 2 * NT; i < n; i += NT) {
    load_group<TW, TH, true, true>(v, S, tx0, ty0, 0, i, a);
    if (i < m) load_group<TW, TH, true, false>(v, S, tx0, ty0, pg, i, c);
    put_group2<TW, TH, true, true>(rec, vb, i, i, a);
    if (i < m) put_group2<TW, TH, true, false>(rec, vb, i, n + i, c);
  }
}
template <int TW, int TH>
__device__ __forceinline__ void stage2_last(const ViewK &v, const SamplesK &S, float4 *rec, int tx0, int ty0, int pg) {
  constexpr int NT = TW * TH, NG = Window<TW, TH>::NG;
  const int t = threadIdx.x, n = (S.spp - pg) * NG;
  RecordGroup a, b;
  if (t < n) load_group<TW, TH, false, true>(v, S, tx0, ty0, pg, t, a);
  if (t + NT < n) load_group<TW, TH, false, true>(v, S, tx0, ty0, pg, t + NT, b);
  if (t < n) put_group2<TW, TH, false, true>(rec, nullptr, t, t, a);
  if (t + NT < n) put_group2<TW, TH, false, true>(rec, nullptr, t + NT, t + NT, b);
  for (int i = t + 2 * NT; i < n; i += NT) {
    load_group<TW, TH, false, true>(v, S, tx0, ty0, pg, i, a);
    put_group2<TW, TH, false, true>(rec, nullptr, i, i, a);
  }
}

// Training list of one pixel for the two-pass tile: the same candidates in
// the same order as build_list, kept by their validity bit; an entry is the
// record's byte offset in its pass's records area, the first pass's entries
// from the front of column `col`, the last pass's from the back.  Returns
// the list length and the first pass's count in n0.
template <int TW, int TH>
__device__ __forceinline__ int build_list2(const ParamsK &P, const uint32_t *vb, const int16_t *ptab,
                                           uint16_t *list, int col, int lx, int ly, int npick, int spp,
                                           uint32_t pix, int &n0) {
  constexpr int SW = TW + 8, SA = em2_stride(TW, TH), NT = TW * TH;
  const int cap = spp + 20, pg = em2_planes(spp), split = pg * SA;  // the first record of the last pass
  const uint32_t cs = (uint32_t)(kCand * spp);
  const int own = (ly + kR) * SW + (lx + 4);
  // where the next entry of the first and of the last pass goes
  char *const a0 = reinterpret_cast<char *>(list + col), *const b0 = a0 + (cap - 1) * 2 * NT;
  char *a = a0, *b = b0;
#pragma unroll
  for (int s = 0; s < kMaxSpp; ++s)
    if (s < spp) {
      const int e = s * SA + own;
      const int step = (int)((vb[e >> 5] >> (e & 31)) & 1u) * (2 * NT);
      if (s < pg) {  // (a rejected entry is overwritten by the next)
        *reinterpret_cast<uint16_t *>(a) = (uint16_t)(e << 4);
        a += step;
      } else {
        *reinterpret_cast<uint16_t *>(b) = (uint16_t)((e - split) << 4);
        b -= step;
      }
    }
  for (int m0 = 0; m0 < npick; m0 += 8) {
    const uint4 w4 = philox4x32_10(pix, P.frame, (1u << 16) | (uint32_t)(m0 >> 3), P.view, P.key0, P.key1);
    int e[8];
    uint32_t wv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // the 16-bit field j of the four words, scaled to a code in [0, 48 spp)
      const uint32_t word = (j >> 1) == 0 ? w4.x : (j >> 1) == 1 ? w4.y : (j >> 1) == 2 ? w4.z : w4.w;
      const uint32_t h = (j & 1) ? (word >> 16) : (word & 0xFFFFu);
      e[j] = own + ptab[__umul24(h, cs) >> 16];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) wv[j] = vb[e[j] >> 5] >> (e[j] & 31);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (m0 + j < npick) {
        const bool last = e[j] >= split;
        *reinterpret_cast<uint16_t *>(last ? b : a) = (uint16_t)((e[j] - (last ? split : 0)) << 4);
        const int step = (int)(wv[j] & 1u) * (2 * NT), back = last ? step : 0;
        a += step - back;
        b -= back;
      }
  }
  n0 = (int)((uint32_t)(a - a0) / (2u * NT));
  return n0 + (int)((uint32_t)(b0 - b) / (2u * NT));
}

template <typename Op, int TW, int TH>
__device__ __forceinline__ void em_tile2(const ParamsK &P, const ViewK &v, const SamplesK &S, const Op &op, int tx0,
                                         int ty0, int rot, float4 *lds, EmShared<TW * TH> &sh) {
  constexpr int NT = TW * TH, SA = em2_stride(TW, TH);
  const int spp = S.spp, pg = em2_planes(spp), cap = spp + 20;
  float4 *rec = lds;
  uint32_t *vb = reinterpret_cast<uint32_t *>(lds + pg * SA);
  uint16_t *list = em_lists<TW, TH, true>(lds, spp);
  const int16_t *ptab = reinterpret_cast<const int16_t *>(list + cap * NT);
  uint8_t *work0 = reinterpret_cast<uint8_t *>(list + cap * NT) + pick_table_bytes(spp);
  float *wb = reinterpret_cast<float *>(lds);  // write-back area (records, bits, lists: all dead by then)
  const int plane = v.H * v.pitch;
  const int t = threadIdx.x;
  const int x0 = tx0 + t % TW, y0 = ty0 + t / TW;
  const bool in_image = x0 < v.W && y0 < v.H;
  if (t < 2 * kMaxLen) (&sh.cnt[0][0])[t] = 0;
  const EmPixel px0 = em_load_pixel(v, op, tx0, ty0, TW);
  stage2_first<TW, TH>(v, S, rec, reinterpret_cast<uint8_t *>(vb), tx0, ty0, pg);
  int ncand = 0;
  if (in_image && dot3(px0.n, px0.o) > 0.0f && px0.rough >= P.rough_min) ncand = spp + n_picks(P, (int)px0.k);
  sh.work[t] = (uint8_t)ncand;
  __syncthreads();
  int me;
  {
    const int pa = balance<NT>(ncand, t, sh.cnt[0], sh.perm, rot);
    const int nc = sh.work[pa];
    int len = 0, n0 = 0;
    if (nc > 0) {
      const int lx = pa % TW, ly = pa / TW;
      len = build_list2<TW, TH>(P, vb, ptab, list, pa, lx, ly, nc - spp, spp,
                                (uint32_t)(row_off(ty0 + ly, v.W) + tx0 + lx), n0);
    }
    sh.work[pa] = (uint8_t)(Op::kEvery && nc > 0 ? len | kTrained : len);
    work0[pa] = (uint8_t)n0;
    // each pass lasts as long as its longest list in the wave, so the lanes
    // are grouped by the longer of their two parts (max(n0) + max(n1) per
    // wave), not by the whole list
    me = balance<NT>(max(n0, len - n0), pa, sh.cnt[1], sh.perm, rot + 1);
  }
  const int len = Op::kEvery ? sh.work[me] & (kTrained - 1) : sh.work[me], n0 = work0[me];
  const bool run = Op::kEvery ? (sh.work[me] & kTrained) != 0 : len > 0;
  float g[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int mex = tx0 + me % TW, mey = ty0 + me / TW;
  const bool me_in = mex < v.W && mey < v.H;
  const int idx = row_off(mey, v.pitch) + mex;
  if (Op::kEvery ? run : me_in) op.load(plane, idx, g);
  typename Op::Acc a = {};
  // the pixel's context is built for each pass (its loads hit the caches):
  // across the restaging only the sums and the state stay in registers
  if (run) {
    const typename Op::Ctx c = Op::context(
        P, make_pixel(P, load3(v.n, plane, idx), load3(v.o, plane, idx), at(v.rough, idx), at(v.alb, idx)), g);
    for_each_record<2>(rec, list, NT, me, 0, 1, n0, [&](float4 r) { Op::visit(c, r, a); });
  }
  __syncthreads();  // the first planes' records are no longer read
  stage2_last<TW, TH>(v, S, rec, tx0, ty0, pg);
  __syncthreads();
  if (run) {
    const typename Op::Ctx c = Op::context(
        P, make_pixel(P, load3(v.n, plane, idx), load3(v.o, plane, idx), at(v.rough, idx), at(v.alb, idx)), g);
    for_each_record<2>(rec, list, NT, me, cap - 1, -1, len - n0, [&](float4 r) { Op::visit(c, r, a); });
    op.finish(P, c, a, idx, g);
  }
  __syncthreads();  // records and lists are no longer read
  tile_write_back<Op, NT>(op, wb, me, me_in, g, t, in_image, plane, row_off(y0, v.pitch) + x0);
}

// One tile per block (blocks are mapped to XCD bands by xcd_tile); with the
// LDS and registers of a tile, several blocks share each CU, which hides the
// loads of one block behind the arithmetic of the others better than a
// persistent loop with register prefetch.
// TWO: the two-pass tile (online EM from spp 4; em2_lds_front).
template <typename TG, int TW, int TH, bool STALE, bool TWO = false, bool BATCH = false>
__global__ __launch_bounds__(TW *TH) __attribute__((amdgpu_waves_per_eu(TWO ? 5 : 8))) void k_em(ParamsK P, ViewK v, SamplesK S, TG *__restrict__ gamma,
                                               int iterations, int tiles_x, int n_tiles) {
  extern __shared__ float4 lds[];  // records, lists and the pick table (em_lds_front, em2_lds_front)
  __shared__ EmShared<TW * TH> sh;
  const int tile = xcd_tile(blockIdx.x, n_tiles);
  const int tx0 = (tile % tiles_x) * TW, ty0 = (tile / tiles_x) * TH;
  build_em_pick_table<TW, TH, TWO>(lds, S.spp);  // before the loads: fewer live registers
  const EmOp<TG> op{gamma};
  if constexpr (TWO) {
    em_tile2<EmOp<TG>, TW, TH>(P, v, S, op, tx0, ty0, (int)blockIdx.x, lds, sh);
  } else {
    EmInput<TW, TH> R;
    em_load(v, S, op, tx0, ty0, R);
    em_tile<EmOp<TG>, TW, TH, STALE, BATCH>(P, v, S, op, iterations, tx0, ty0, (int)blockIdx.x, lds, sh, R);
  }
}

// ---------------------------------------------------------------------------
// Weighted NLL of the mixture over the training set and its adjoint.
struct NllAccum {
  float loss, gmx, gmy, gxx, gxy, gyy, gl;
};

struct NllCtx {
  Pixel px;
  LobeTerm T;
  float pi, one_m_pi, ia, ib, ic;  // ia, ib, ic: the inverse of Sigma + eps I
};

// NLL (LOSS) and its gradient (GRAD) of the pixels' parameters theta = (mu,
// Cholesky factor, logit pi, -, k).  The training tile of the EM update runs
// it: the picks of a pixel are examined once against the staged records and
// only the kept ones visited, by lanes sorted to nearly equal lists.  (One
// lane per pixel in image order visited all of its candidates: 24 visits a
// wave at spp 4, where the sorted lists need about 15.)  4K, 4 spp: 635 us for
// the loss, 710 for the gradient, 731 for both, bound by VALU issue; 922 us each
// before.
template <bool LOSS, bool GRAD>
struct NllOp {
  using Ctx = NllCtx;
  using Acc = NllAccum;
  static constexpr bool kEvery = true;
  const float *theta, *grad_out;
  float *grad, *nll;
  __device__ __forceinline__ float epoch(int plane, int idx) const { return at(theta + 7 * plane, idx); }
  __device__ __forceinline__ void load(int plane, int idx, float g[8]) const {
#pragma unroll
    for (int ch = 0; ch < 6; ++ch) g[ch] = at(theta + ch * plane, idx);
  }
  static __device__ __forceinline__ Ctx context(const ParamsK &P, const Pixel &px, const float g[8]) {
    Ctx c;
    const float l11 = g[2], l21 = g[3], l22 = g[4];
    const Gauss G = gauss_setup(g[0], g[1], l11 * l11, l11 * l21, fmaf(l21, l21, l22 * l22), P.eps);
    c.px = px;
    c.pi = 1.0f / (1.0f + expf(-g[5]));
    c.one_m_pi = 1.0f - c.pi;
    c.T = lobe_term(G, c.pi);
    // (L L^T)^-1 from the whitening z = L^-1 r, z1 = i11 rx, z2 = i22 ry + c21 z1
    const float b = c.T.c21 * G.i11;
    c.ia = fmaf(b, b, G.i11 * G.i11);
    c.ib = b * G.i22;
    c.ic = G.i22 * G.i22;
    return c;
  }
  static __device__ __forceinline__ void visit(const Ctx &c, float4 r, Acc &a) {
    if (r.w == 0.0f) return;
    const V3 l = to_local(c.px.f, V3{r.x, r.y, r.z});
    if (l.z <= 0.0f) return;
    float cx, cy, f, pb;
    hemi2sq_c(l, cx, cy);
    const float rx = cx + c.T.hx, ry = cy + c.T.hy;
    brdf_eval(c.px, l, f, pb);
    const float w = r.w * f * l.z;
    const float z1 = rx * c.T.i11;
    const float z2 = fmaf(ry, c.T.i22, z1 * c.T.c21);
    const float e = -0.72134752044448170368f * fmaf(z1, z1, z2 * z2);
    float ga = c.T.pi_norm * __builtin_amdgcn_exp2f(e);
    float D = fmaf(c.one_m_pi, pb, ga), off = 0.0f;
    // The hardware exponential gives 0 below 2^-126, and the logarithm and the
    // reciprocal take subnormals for 0: where so little is left (1 - pi is 0 or
    // at least 2^-24, so that p_b no longer counts), the Gaussian is taken 2^32
    // times larger before it is rounded, which reaches below the smallest
    // subnormal.  (e + 32 is exact for e < -32.)  One uniform branch for the
    // wave, seldom taken.
    const bool far = D < 0x1p-64f;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
      const float gs = e < -32.0f ? c.T.pi_norm * __builtin_amdgcn_exp2f(e + 32.0f) : ga * 0x1p32f;
      ga = far ? gs : ga;
      D = far ? fmaf(c.one_m_pi * 0x1p32f, pb, gs) : D;
      off = far ? 32.0f : 0.0f;
    }
    if (LOSS) a.loss = fmaf(w, 0.693147180559945309417f * (off - __builtin_amdgcn_logf(D)), a.loss);
    if (GRAD) {
      // the quotient corrected by its remainder, as a division rounds it (1
      // where the Gaussian is alone)
      const float Dn = fmaxf(D, 1.17549435e-38f), rD = __builtin_amdgcn_rcpf(Dn), q = ga * rD;
      const float gam = fmaf(fmaf(-q, Dn, ga), rD, q);
      // Sigma^-1 r = L^-T z
      const float vx = c.T.i11 * fmaf(c.T.c21, z2, z1), vy = c.T.i22 * z2;
      const float wg = w * gam, hg = -0.5f * wg;
      a.gmx = fmaf(-wg, vx, a.gmx);
      a.gmy = fmaf(-wg, vy, a.gmy);
      a.gxx = fmaf(hg, fmaf(vx, vx, -c.ia), a.gxx);
      a.gxy = fmaf(hg, fmaf(vx, vy, -c.ib), a.gxy);
      a.gyy = fmaf(hg, fmaf(vy, vy, -c.ic), a.gyy);
      a.gl = fmaf(-w, gam - c.pi, a.gl);
    }
  }
  __device__ __forceinline__ void finish(const ParamsK &, const Ctx &, const Acc &a, int idx, float g[8]) const {
    if (GRAD) {
      const float sc = grad_out ? at(grad_out, idx) : 1.0f;
      const float l11 = g[2], l21 = g[3], l22 = g[4];
      g[0] = sc * a.gmx;
      g[1] = sc * a.gmy;
      g[2] = sc * 2.0f * fmaf(a.gxx, l11, a.gxy * l21);
      g[3] = sc * 2.0f * fmaf(a.gxy, l11, a.gyy * l21);
      g[4] = sc * 2.0f * (a.gyy * l22);
      g[5] = sc * a.gl;
    }
    if (LOSS) g[6] = a.loss;
  }
  static constexpr bool put(int ch) { return (GRAD && ch < 6) || (LOSS && ch == 6); }
  __device__ __forceinline__ void store(int plane, int idx, const float out[8]) const {
    if (GRAD) {
#pragma unroll
      for (int ch = 0; ch < 8; ++ch) at(grad + ch * plane, idx) = ch < 6 ? out[ch] : 0.0f;
    }
    if (LOSS) at(nll, idx) = out[6];
  }
};

template <int TW, int TH, bool LOSS, bool GRAD, bool TWO>
__global__ __launch_bounds__(TW *TH) void k_nll(ParamsK P, ViewK v, SamplesK S, NllOp<LOSS, GRAD> op, int tiles_x,
                                                int n_tiles) {
  extern __shared__ float4 lds[];  // records, lists and the pick table (em_lds_front, em2_lds_front)
  __shared__ EmShared<TW * TH> sh;
  const int tile = xcd_tile(blockIdx.x, n_tiles);
  const int tx0 = (tile % tiles_x) * TW, ty0 = (tile / tiles_x) * TH;
  build_em_pick_table<TW, TH, TWO>(lds, S.spp);
  if constexpr (TWO) {
    em_tile2<NllOp<LOSS, GRAD>, TW, TH>(P, v, S, op, tx0, ty0, (int)blockIdx.x, lds, sh);
  } else {
    EmInput<TW, TH> R;
    em_load(v, S, op, tx0, ty0, R);
    em_tile(P, v, S, op, 1, tx0, ty0, (int)blockIdx.x, lds, sh, R);
  }
}

// ---------------------------------------------------------------------------
// Batched frame: many views of any size and spp in a sampling launch
// (reprojection + sampling + light) and a training launch per spp, which read
// everything from a table in device memory, so that one captured graph (table
// upload + kernels) replays later frames of all views once the table is re-packed.
struct BatchViewK {
  ViewK cur;
  const float *prev_n, *prev_z;
  const void *gprev;
  void *gout;
  SamplesK S;
  const uint8_t *vis;
  LightsK lights;
  uint32_t key0, key1, frame, view;
  int rs_begin, rs_tiles_x, em_begin, em_tiles_x;
};

// The views of a table are ordered by spp; the views of one spp form a class
// whose training tiles are contiguous in the tile list and run in a launch of
// their own, with the tile shape and LDS of that spp.
struct BatchClass {
  int spp, tile_w, tile_h, em_begin, em_end, pad[3];
};

struct BatchHeader {
  int n_views, rs_tiles, em_tiles, dtype, n_classes, magic, pad[2];
  ParamsK base;  // fields shared by every view (key, frame, view come per view)
  BatchClass cls[kMaxSpp];
};

constexpr int kBatchViewsOffset = (int)((sizeof(BatchHeader) + 63) / 64 * 64);

__device__ __forceinline__ const BatchViewK *batch_views(const char *table) {
  return reinterpret_cast<const BatchViewK *>(table + kBatchViewsOffset);
}

// The view owning tile t: the last one whose first tile is <= t (the tiles of
// consecutive views are contiguous).  Uniform across the block.
template <bool EM>
__device__ __forceinline__ int batch_find(const BatchViewK *vs, int n, int t) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int b = EM ? vs[mid].em_begin : vs[mid].rs_begin;
    if (b <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ ParamsK batch_params(const ParamsK &base, const BatchViewK &bv) {
  ParamsK P = base;
  P.key0 = bv.key0;
  P.key1 = bv.key1;
  P.frame = bv.frame;
  P.view = bv.view;
  return P;
}

// Pointers that a kernel reads from memory are generic ones to the compiler,
// and every access through them a FLAT one, which waits for the LDS as well as
// for memory and has no immediate offsets.  The table holds device memory
// only; these say so, which gives the batched kernels the same global loads
// as the plain ones have (pointers in kernel arguments are known to be
// global).  Eight FP16 views of 1 to 8 spp: 3.00 ms a frame, 3.09 with FLAT
// accesses.
template <typename T>
__device__ __forceinline__ T *global_ptr(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)reinterpret_cast<uintptr_t>(p);
}
__device__ __forceinline__ ViewK global_view(const ViewK &v) {
  return {v.W, v.H, v.pitch, global_ptr(v.n), global_ptr(v.o), global_ptr(v.z), global_ptr(v.rough),
          global_ptr(v.alb), global_ptr(v.mv), global_ptr(v.mask)};
}
__device__ __forceinline__ SamplesK global_samples(const SamplesK &s) {
  return {s.spp, global_ptr(s.dir), global_ptr(s.pmix), global_ptr(s.pb), global_ptr(s.L), global_ptr(s.strat)};
}

// Reprojection + sampling + light field over the 64x4 pixel tiles of all
// views, one block per tile (a persistent grid-stride loop held 72-80 VGPRs,
// this 60-62).  `dtype` is the launch's Gamma type: a table of another type,
// or with more tiles than the grid, is not processed.
template <typename TG>
__global__ __launch_bounds__(256) void k_rs_batched(const char *__restrict__ table, int dtype) {
  const BatchHeader *hd = reinterpret_cast<const BatchHeader *>(table);
  if (hd->dtype != dtype) return;
  const int n_views = hd->n_views, n_tiles = hd->rs_tiles;
  const BatchViewK *vs = batch_views(table);
  // one block per tile, in tile order: blocks are dealt to the XCDs round
  // robin, so the views (ordered by spp) are interleaved over the XCDs
  const int t = (int)blockIdx.x;
  if (n_tiles > (int)gridDim.x || t >= n_tiles) return;  // more tiles than the grid: a different table
  const BatchViewK &bv = vs[batch_find<false>(vs, n_views, t)];
  const int local = t - bv.rs_begin;
  const int x = (local % bv.rs_tiles_x) * 64 + (int)(threadIdx.x & 63);
  const int y = (local / bv.rs_tiles_x) * 4 + (int)(threadIdx.x >> 6);
  const ViewK cur = global_view(bv.cur);
  if (x >= cur.W || y >= cur.H) return;
  const ParamsK P = batch_params(hd->base, bv);
  ViewK prev = cur;
  prev.n = global_ptr(bv.prev_n);
  prev.z = global_ptr(bv.prev_z);
  reproject_sample_pixel(P, cur, prev, global_ptr((const TG *)bv.gprev), global_ptr((TG *)bv.gout),
                         global_samples(bv.S), bv.frame > 0, x, y, &bv.lights, global_ptr(bv.vis));
}

// Training over the TW x TH tiles of the views of class `cls`, one block per
// tile in XCD bands (like k_em: with no state carried from tile to tile the
// kernel fits 8 waves/SIMD; a persistent loop over tiles needed ~30 more
// VGPRs).  `spp_cap` is the spp the dynamic LDS was sized for; a table whose
// class differs from the launch (tile, one or two passes, more spp, dtype, or
// more tiles than the grid) is not processed.  (The tile alone does not tell
// the passes apart: 32x8 is the default of both.  A two-pass launch cannot
// train a class of few samples: its staging takes four records for granted.)
template <typename TG, int TW, int TH, bool TWO>
__global__ __launch_bounds__(TW *TH) __attribute__((amdgpu_waves_per_eu(TH == 2 ? 1 : (TWO ? 5 : 8)))) void k_em_batched(const char *__restrict__ table, int dtype, int cls,
                                                       int spp_cap) {
  extern __shared__ float4 lds[];  // sized for spp_cap (em_lds_front, em2_lds_front)
  __shared__ EmShared<TW * TH> sh;
  const BatchHeader *hd = reinterpret_cast<const BatchHeader *>(table);
  if (hd->dtype != dtype || cls >= hd->n_classes) return;
  const BatchClass c = hd->cls[cls];
  if (c.spp > spp_cap || em2_spp(c.spp) != TWO || c.tile_w != TW || c.tile_h != TH) return;
  const int n_views = hd->n_views;
  const BatchViewK *vs = batch_views(table);
  const int n = c.em_end - c.em_begin;
  // a class with more tiles than the grid (a replayed launch for other views)
  // differs from the launch: not processed
  if (n > (int)gridDim.x || (int)blockIdx.x >= n) return;
  const int t = c.em_begin + xcd_tile((int)blockIdx.x, n);
  const BatchViewK &bv = vs[batch_find<true>(vs, n_views, t)];
  const int l = t - bv.em_begin;
  const int tx0 = (l % bv.em_tiles_x) * TW, ty0 = (l / bv.em_tiles_x) * TH;
  const ParamsK P = batch_params(hd->base, bv);
  const ViewK v = global_view(bv.cur);
  const SamplesK S = global_samples(bv.S);
  build_em_pick_table<TW, TH, TWO>(lds, S.spp);
  const EmOp<TG> op{global_ptr((TG *)bv.gout)};
  if constexpr (TWO) {
    em_tile2<EmOp<TG>, TW, TH>(P, v, S, op, tx0, ty0, (int)blockIdx.x, lds, sh);
  } else {
    EmInput<TW, TH> R;
    em_load(v, S, op, tx0, ty0, R);
    em_tile(P, v, S, op, 1, tx0, ty0, (int)blockIdx.x, lds, sh, R);
  }
}

// Philox words for given counters (diagnostic entry).
__global__ void k_philox(int n, const uint32_t *__restrict__ ctr, uint32_t key0, uint32_t key1,
                         uint32_t *__restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint4 r = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], key0, key1);
  out[4 * i] = r.x;
  out[4 * i + 1] = r.y;
  out[4 * i + 2] = r.z;
  out[4 * i + 3] = r.w;
}

}  // namespace pgk
