// View-dependent features by spherical harmonics (paper Sec. III-B: each Gaussian's colour
// and semantic features are represented with SH). Per view v, Gaussian i and channel c,
//   f_vic = dc_ic + sum_{1 <= j < (degree+1)^2} Y_j(d_vi) k_ijc,
// d_vi = (mu_i - c_v) / |mu_i - c_v|, c_v = -R_v^T t_v the camera centre, Y_j the real
// spherical harmonics (index j = l^2 + l + m, the sign convention of the 3DGS renderer).
// The constant band is the plain feature, so degree 0 reproduces view-independent features.
//
// The forward writes one feature block per view for the render kernels (cfg.view_features).
// The backward takes the render's per-view feature gradients back to the constant band, the
// coefficients, the means (through d) and each view's pose (through c_v, which moves by
// -R^T rho under T_cw <- Exp(xi) T_cw and not with phi).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace gs {
namespace {

constexpr double kPiD = 3.14159265358979323846;
constexpr double csqrt(double x) {   // Newton's iteration, for the constants below
  double r = x > 1.0 ? x : 1.0;
  for (int k = 0; k < 100; ++k) r = 0.5 * (r + x / r);
  return r;
}
constexpr float kC1 = (float)csqrt(3.0 / (4.0 * kPiD));
constexpr float kC2a = (float)(csqrt(15.0 / kPiD) / 2.0);   // xy, -yz, -xz
constexpr float kC2b = (float)(csqrt(5.0 / kPiD) / 4.0);    // 2zz - xx - yy
constexpr float kC2c = (float)(csqrt(15.0 / kPiD) / 4.0);   // xx - yy
constexpr float kC3a = (float)(csqrt(35.0 / (2.0 * kPiD)) / 4.0);
constexpr float kC3b = (float)(csqrt(105.0 / kPiD) / 2.0);
constexpr float kC3c = (float)(csqrt(21.0 / (2.0 * kPiD)) / 4.0);
constexpr float kC3d = (float)(csqrt(7.0 / kPiD) / 4.0);
constexpr float kC3e = (float)(csqrt(105.0 / kPiD) / 4.0);

// Y_1 .. Y_{K-1} at the unit direction (x, y, z).
__device__ __forceinline__ void sh_basis(float x, float y, float z, int deg, float* Y) {
  if (deg < 1) return;
  Y[1] = -kC1 * y;
  Y[2] = kC1 * z;
  Y[3] = -kC1 * x;
  if (deg < 2) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  Y[4] = kC2a * x * y;
  Y[5] = -kC2a * y * z;
  Y[6] = kC2b * (2.0f * zz - xx - yy);
  Y[7] = -kC2a * x * z;
  Y[8] = kC2c * (xx - yy);
  if (deg < 3) return;
  Y[9] = -kC3a * y * (3.0f * xx - yy);
  Y[10] = kC3b * x * y * z;
  Y[11] = -kC3c * y * (4.0f * zz - xx - yy);
  Y[12] = kC3d * z * (2.0f * zz - 3.0f * xx - 3.0f * yy);
  Y[13] = -kC3c * x * (4.0f * zz - xx - yy);
  Y[14] = kC3e * z * (xx - yy);
  Y[15] = -kC3a * x * (xx - 3.0f * yy);
}

// sum_j a_j dY_j/dd (the polynomials' gradient in the ambient coordinates), j >= 1.
__device__ __forceinline__ void sh_grad_dot(float x, float y, float z, int deg, const float* a, float& gx, float& gy,
                                            float& gz) {
  gx = gy = gz = 0.0f;
  if (deg < 1) return;
  gy += -kC1 * a[1];
  gz += kC1 * a[2];
  gx += -kC1 * a[3];
  if (deg < 2) return;
  gx += kC2a * y * a[4];
  gy += kC2a * x * a[4];
  gy += -kC2a * z * a[5];
  gz += -kC2a * y * a[5];
  gx += -2.0f * kC2b * x * a[6];
  gy += -2.0f * kC2b * y * a[6];
  gz += 4.0f * kC2b * z * a[6];
  gx += -kC2a * z * a[7];
  gz += -kC2a * x * a[7];
  gx += 2.0f * kC2c * x * a[8];
  gy += -2.0f * kC2c * y * a[8];
  if (deg < 3) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  gx += -kC3a * 6.0f * x * y * a[9];
  gy += -kC3a * (3.0f * xx - 3.0f * yy) * a[9];
  gx += kC3b * y * z * a[10];
  gy += kC3b * x * z * a[10];
  gz += kC3b * x * y * a[10];
  gx += -kC3c * (-2.0f * x * y) * a[11];
  gy += -kC3c * (4.0f * zz - xx - 3.0f * yy) * a[11];
  gz += -kC3c * 8.0f * y * z * a[11];
  gx += kC3d * (-6.0f * x * z) * a[12];
  gy += kC3d * (-6.0f * y * z) * a[12];
  gz += kC3d * (6.0f * zz - 3.0f * xx - 3.0f * yy) * a[12];
  gx += -kC3c * (4.0f * zz - 3.0f * xx - yy) * a[13];
  gy += -kC3c * (-2.0f * x * y) * a[13];
  gz += -kC3c * 8.0f * x * z * a[13];
  gx += kC3e * 2.0f * x * z * a[14];
  gy += kC3e * (-2.0f * y * z) * a[14];
  gz += kC3e * (xx - yy) * a[14];
  gx += -kC3a * (3.0f * xx - 3.0f * yy) * a[15];
  gy += -kC3a * (-6.0f * x * y) * a[15];
}

// Up to the semantic degrees below both kernels give a wave 16 Gaussians and take the views four at a time:
//   lane 4 g + k works out the direction of Gaussian g from view k once and leaves Y_1.. in LDS
//   (a row of 64 for each function, so that one b128 read has a Gaussian's four views);
//   the semantic channels go by four Gaussians at a time, 16 lanes each, channels l16 + 16 m:
//   every load is four runs of 64 bytes, and a sum over channels stays in a row of 16 lanes;
//   rgb's 48 (Gaussian, channel) pairs have a lane each in the forward; in the backward their
//   coefficients, 16 consecutive rows, go through LDS in the order they lie in memory.
// Bound by memory, whose floor is 168 us for 200k Gaussians, 52 classes of degree 1, rgb of degree 3
// and two views: a lane per (Gaussian, channel) had every lane work out its Gaussian's directions,
// and three rgb channels' degree 3 cost the whole wave: forward 101 us, backward 377. Now 75 and 127
// (three registers a lane of the backward in scratch).
constexpr int kShG = 16, kShV = 4, kShWaves = 4, kShBwdWaves = 8;
// The largest semantic degree that goes this way; past it a step has too many coefficients for
// loads of several steps in flight, and rows are fetched again for their other channels. Measured
// with 100k Gaussians, 52 classes, two views, this way and with a lane per channel: forward, degree
// 2, 60 and 48 us; backward, degree 2, 161 and 172 us, degree 3 278 and 216 us.
constexpr int kShFwdDegree = 1, kShBwdDegree = 2;
// Steps whose loads are issued together: four of few coefficients, two of more, else the registers
// run out (the case above with one step at a time: 115 and 159 us; two: 108 and 143).
constexpr int sh_steps(int deg) { return deg <= 1 ? 4 : 2; }
constexpr int sh_rest(int deg) { return (deg + 1) * (deg + 1) - 1; }   // functions past the constant band

// A wave's steps over the semantic channels: 16 channels from c0 of four Gaussians from q0.
struct ShStep {
  int M, m, c0, q0;
  __device__ __forceinline__ explicit ShStep(int steps) : M(steps), m(0), c0(0), q0(0) {}
  __device__ __forceinline__ bool last() const { return m == M - 1; }   // of its Gaussians
  __device__ __forceinline__ void next() {
    const bool l = last();
    q0 += l ? 4 : 0;
    m = l ? 0 : m + 1;
    c0 = 16 * m;
  }
};

// The camera centre of a view, and the direction of a Gaussian from it: (d, 1 / distance).
__device__ __forceinline__ void sh_camera(const gs_view& V, float* c) {
#pragma unroll
  for (int a = 0; a < 3; ++a) c[a] = -(V.R[a] * V.t[0] + V.R[3 + a] * V.t[1] + V.R[6 + a] * V.t[2]);
}
__device__ __forceinline__ float4 sh_dir(const float* c, const float* m) {
  const float x = m[0] - c[0], y = m[1] - c[1], z = m[2] - c[2];
  const float ir = rsqrtf(x * x + y * y + z * z);
  return make_float4(x * ir, y * ir, z * ir, ir);
}

// Whether a gradient of four views has a share where the direction (bit k) does not exist.
__device__ __forceinline__ bool sh_nan(uint32_t bad, const float4 g) {
  return ((bad & 1) && g.x != 0.0f) || ((bad & 2) && g.y != 0.0f) || ((bad & 4) && g.z != 0.0f) || ((bad & 8) && g.w != 0.0f);
}

__device__ __forceinline__ float4 lds4(const float* p) { return *reinterpret_cast<const float4*>(p); }

template <int RD, int SD>
__global__ __launch_bounds__(64 * kShWaves) void k_sh_fwd(gs_gaussians g, gs_sh sh, int n_sem,
                                                          const gs_view* __restrict__ views, int n_views,
                                                          float* __restrict__ rgb_out, float* __restrict__ sem_out) {
  constexpr int JR = sh_rest(RD), JS = sh_rest(SD), D = RD > SD ? RD : SD, J = sh_rest(D), MU = sh_steps(SD);
  __shared__ __align__(16) float s_mem[kShWaves][J * 64 + 4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g4 = lane >> 4;
  float* const Y = s_mem[wave];
  const int64_t n = g.n, i0 = ((int64_t)blockIdx.x * kShWaves + wave) * kShG;
  if (i0 >= n) return;   // (nothing below is shared between waves)
  const int ng = (int)(n - i0 < kShG ? n - i0 : kShG);
  // rgb: a lane per (Gaussian, channel), its coefficients in registers over all views
  float rc[JR + 1];
  {
    const uint32_t l = min(lane, 3 * ng - 1), b = l / 3 * (3 * JR) + l % 3;
    rc[0] = (g.rgb + 3 * i0)[l];
#pragma unroll
    for (int j = 0; j < JR; ++j) rc[j + 1] = (sh.rgb_rest + 3 * JR * i0)[b + 3 * j];
  }
  float m[3] = {0.0f, 0.0f, 0.0f};
  if constexpr (J > 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) m[a] = g.mean[3 * (i0 + min(lane >> 2, ng - 1)) + a];
  }
  for (int v0 = 0; v0 < n_views; v0 += kShV) {
    const int nv = min(kShV, n_views - v0);
    if constexpr (J > 0) {
      float cam[3];
      sh_camera(views[v0 + min(lane & 3, nv - 1)], cam);
      const float4 d = sh_dir(cam, m);
      float B[J + 1];
      sh_basis(d.x, d.y, d.z, D, B);
#pragma unroll
      for (int j = 0; j < J; ++j) Y[64 * j + lane] = B[j + 1];
    }
    wave_sync();
    // (scalar bases, 32-bit lane offsets)
    const float* const dc = g.sem + n_sem * i0;
    const float* const rest = JS ? sh.sem_rest + JS * n_sem * i0 : nullptr;
    float* const out = sem_out + n_sem * (v0 * n + i0);
    const int M = (n_sem + 15) / 16;   // steps of four Gaussians; 4 M in all, a multiple of MU
#pragma unroll 1
    for (ShStep st(M); st.q0 < ng && M > 0;) {
      float f[MU], x[MU][JS + 1];
      ShStep ld = st;
#pragma unroll
      for (int u = 0; u < MU; ++u, ld.next()) {
        const uint32_t row = n_sem * min(ld.q0 + g4, ng - 1), c = min(ld.c0 + l16, n_sem - 1);
        f[u] = dc[row + c];
#pragma unroll
        for (int j = 0; j < JS; ++j) x[u][j] = (rest + j * n_sem)[JS * row + c];
      }
#pragma unroll
      for (int u = 0; u < MU; ++u, st.next()) {
        const int q = st.q0 + g4, c = st.c0 + l16;
        float4 o = make_float4(f[u], f[u], f[u], f[u]);
#pragma unroll
        for (int j = 0; j < JS; ++j) {
          const float4 y = lds4(Y + 64 * j + 4 * (q & (kShG - 1)));
          o.x = fmaf(y.x, x[u][j], o.x);
          o.y = fmaf(y.y, x[u][j], o.y);
          o.z = fmaf(y.z, x[u][j], o.z);
          o.w = fmaf(y.w, x[u][j], o.w);
        }
        if (q < ng && c < n_sem) {
          const uint32_t e = n_sem * q + c;
          out[e] = o.x;
          if (nv > 1) (out + n_sem * n)[e] = o.y;
          if (nv > 2) (out + 2 * n_sem * n)[e] = o.z;
          if (nv > 3) (out + 3 * n_sem * n)[e] = o.w;
        }
      }
    }
    {
      float4 o = make_float4(rc[0], rc[0], rc[0], rc[0]);
#pragma unroll
      for (int j = 0; j < JR; ++j) {
        const float4 y = lds4(Y + 64 * j + 4 * min(lane / 3, kShG - 1));
        o.x = fmaf(y.x, rc[j + 1], o.x);
        o.y = fmaf(y.y, rc[j + 1], o.y);
        o.z = fmaf(y.z, rc[j + 1], o.z);
        o.w = fmaf(y.w, rc[j + 1], o.w);
      }
      if (lane < 3 * ng) {
        float* d = rgb_out + 3 * (v0 * n + i0);
        d[lane] = o.x;
        if (nv > 1) (d + 3 * n)[lane] = o.y;
        if (nv > 2) (d + 6 * n)[lane] = o.z;
        if (nv > 3) (d + 9 * n)[lane] = o.w;
      }
    }
    wave_sync();   // the next views' Y overwrite these
  }
}

// The backward, persistent blocks walking the Gaussians: the constant band and the bands sum the
// feature gradient (times Y_j) over views. The direction's share needs only h_j = sum_c g_c k_jc of
// each (Gaussian, view), a sum over its channels; lane 4 g + k then takes sum_j h_j dY_j/dd through
// the normalisation to the mean (summed over the views' four lanes) and to the pose's rho
// (gpose[v][0..2] += R_v sum), which it keeps in double precision over all its Gaussians, so a block adds
// to each pose once. Every one of these atomics rounds the sum so far, and that is most of a pose
// gradient's error, so blocks are few and of eight waves. The bands of a
// later four views are added to the first four's.
// A gradient of zero has no share, whatever it would be multiplied with (a direction from the
// camera's own place, an infinite coefficient): such a Gaussian is rare, and done over by its lane.
template <int RD, int SD>
__global__ __launch_bounds__(64 * kShBwdWaves, SD <= 1 ? 4 : 2) void k_sh_bwd(
    gs_gaussians g, gs_sh sh, int n_sem, const gs_view* __restrict__ views, int n_views,
    const float* __restrict__ grgb, const float* __restrict__ gsem, float* __restrict__ gdc_rgb,
    float* __restrict__ grest_rgb, float* __restrict__ gdc_sem, float* __restrict__ grest_sem,
    float* __restrict__ gmean, float* __restrict__ gpose) {
  constexpr int JR = sh_rest(RD), JS = sh_rest(SD), D = RD > SD ? RD : SD, J = sh_rest(D), MU = sh_steps(SD);
  __shared__ __align__(16) float s_mem[kShBwdWaves][64 * J + 64 * 3 + 64 * JS + 3 * kShG * JR];
  __shared__ double s_red[kShBwdWaves][kShV][3];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g4 = lane >> 4;
  const int vk = lane & 3;   // the lane's view of the four, as the lane of Gaussian lane / 4
  float* const Y = s_mem[wave];
  float* const G = Y + 64 * J;   // rgb gradients, a row of 64 for each channel
  float* const H = G + 64 * 3;   // h of the semantics
  float* const C = H + 64 * JS;  // the rgb coefficients
  const int64_t n = g.n, step = (int64_t)gridDim.x * kShBwdWaves * kShG;
  for (int v0 = 0; v0 < n_views; v0 += kShV) {
    const int nv = min(kShV, n_views - v0);
    double us[3] = {0.0, 0.0, 0.0};   // d L/d mu of the lane's view
    const gs_view& V = views[v0 + min(vk, nv - 1)];
    float cam[3];
    sh_camera(V, cam);
    for (int64_t i0 = ((int64_t)blockIdx.x * kShBwdWaves + wave) * kShG; i0 < n; i0 += step) {
      const int ng = (int)(n - i0 < kShG ? n - i0 : kShG);
      const int64_t iq = i0 + min(lane >> 2, ng - 1);
      const bool valid = vk < nv && (lane >> 2) < ng;
      // the (Gaussian, view) lanes' inputs, and the rgb coefficients
      float gr[3], m[3], gm0 = 0.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a) gr[a] = grgb[3 * ((v0 + min(vk, nv - 1)) * n + iq) + a];
      if constexpr (J > 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) m[a] = g.mean[3 * iq + a];
        gm0 = gmean[3 * iq + min(vk, 2)];
      }
      if constexpr (JR > 0) {
        float x[(3 * kShG * JR + 63) / 64];
#pragma unroll
        for (int e0 = 0; e0 < 3 * kShG * JR; e0 += 64) x[e0 / 64] = sh.rgb_rest[3 * JR * i0 + min(e0 + lane, 3 * ng * JR - 1)];
#pragma unroll
        for (int e0 = 0; e0 < 3 * kShG * JR; e0 += 64)
          if (e0 + lane < 3 * kShG * JR) C[e0 + lane] = x[e0 / 64];
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        gr[a] = valid ? gr[a] : 0.0f;
        G[64 * a + lane] = gr[a];
      }
      float4 d = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      bool bad = false;
      uint64_t bads = 0;   // (Gaussian, view) without a direction: Y = 0 there
      if constexpr (J > 0) {
        d = sh_dir(cam, m);
        bad = !(fabsf(d.x) + fabsf(d.y) + fabsf(d.z) < 4.0f);
        bads = __ballot(bad);
        float B[J + 1];
        sh_basis(d.x, d.y, d.z, D, B);
#pragma unroll
        for (int j = 0; j < J; ++j) Y[64 * j + lane] = bad ? 0.0f : B[j + 1];
      }
      wave_sync();
      // (scalar bases, 32-bit lane offsets)
      const float* const gs = gsem + n_sem * (v0 * n + i0);
      const float* const rest = JS ? sh.sem_rest + JS * n_sem * i0 : nullptr;
      float* const odc = gdc_sem + n_sem * i0;
      float* const ore = grest_sem + JS * n_sem * i0;
      const int M = (n_sem + 15) / 16;
      float4 hs[JS + 1];
#pragma unroll
      for (int j = 0; j < JS; ++j) hs[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 1
      for (ShStep st(M); st.q0 < ng && M > 0;) {
        float x[MU][JS + 1];
        float4 gf[MU];
        ShStep ld = st;
#pragma unroll
        for (int u = 0; u < MU; ++u, ld.next()) {
          const uint32_t row = n_sem * min(ld.q0 + g4, ng - 1), c = min(ld.c0 + l16, n_sem - 1), e = row + c;
          gf[u].x = gs[e];
          gf[u].y = nv > 1 ? (gs + n_sem * n)[e] : 0.0f;
          gf[u].z = nv > 2 ? (gs + 2 * n_sem * n)[e] : 0.0f;
          gf[u].w = nv > 3 ? (gs + 3 * n_sem * n)[e] : 0.0f;
#pragma unroll
          for (int j = 0; j < JS; ++j) x[u][j] = (rest + j * n_sem)[JS * row + c];
        }
#pragma unroll
        for (int u = 0; u < MU; ++u, st.next()) {
          const int q = st.q0 + g4, c = st.c0 + l16, qy = 4 * (q & (kShG - 1));
          const uint32_t row = n_sem * q;
          const bool on = q < ng && c < n_sem;
          const float4 w = on ? gf[u] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          const bool nan = bads && sh_nan((uint32_t)(bads >> qy), w);
          if (on && gdc_sem) {
            // the first four views store, later ones add (no read before the first store)
            const float t = ((w.x + w.y) + w.z) + w.w;
            float* o = odc + (row + c);
            *o = v0 == 0 ? t : *o + t;
          }
#pragma unroll
          for (int j = 0; j < JS; ++j) {
            const float4 y = lds4(Y + 64 * j + qy);
            float t = fmaf(w.w, y.w, fmaf(w.z, y.z, fmaf(w.y, y.y, w.x * y.x)));
            t = nan ? NAN : t;
            hs[j].x = fmaf(w.x, x[u][j], hs[j].x);
            hs[j].y = fmaf(w.y, x[u][j], hs[j].y);
            hs[j].z = fmaf(w.z, x[u][j], hs[j].z);
            hs[j].w = fmaf(w.w, x[u][j], hs[j].w);
            if (on && grest_sem) {
              float* o = (ore + j * n_sem) + (JS * row + (uint32_t)c);
              *o = v0 == 0 ? t : *o + t;
            }
          }
          if constexpr (JS > 0) {
            if (st.last() && st.q0 < ng) {
#pragma unroll
              for (int j = 0; j < JS; ++j) {
                float4 t = make_float4(row_sum16(hs[j].x), 0.0f, 0.0f, 0.0f);
                if (nv > 1) t.y = row_sum16(hs[j].y);
                if (nv > 2) {
                  t.z = row_sum16(hs[j].z);
                  t.w = row_sum16(hs[j].w);
                }
                if (l16 == 0) *reinterpret_cast<float4*>(H + 64 * j + qy) = t;
                hs[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
              }
            }
          }
        }
      }
      // rgb: the lanes' h, then the bands as they lie in memory
      float h[J + 1];   // (h[0] unused, the constant band)
#pragma unroll
      for (int j = 0; j <= J; ++j) h[j] = 0.0f;
      if constexpr (JR > 0) {
#pragma unroll
        for (int j = 0; j < JR; ++j)
#pragma unroll
          for (int a = 0; a < 3; ++a) h[j + 1] = fmaf(gr[a], C[3 * JR * (lane >> 2) + 3 * j + a], h[j + 1]);
        if (grest_rgb) {
          int l = lane;
          asm volatile("" : "+v"(l));   // (else the addresses of every step stay in registers)
#pragma unroll
          for (int e0 = 0; e0 < 3 * kShG * JR; e0 += 64) {
            const int e = e0 + l, q = e / (3 * JR), j = e % (3 * JR) / 3, a = e % 3;
            if (e < 3 * ng * JR) {
              const float4 x = lds4(G + 64 * a + 4 * q), y = lds4(Y + 64 * j + 4 * q);
              float acc = fmaf(x.w, y.w, fmaf(x.z, y.z, fmaf(x.y, y.y, x.x * y.x)));
              if (bads && sh_nan((uint32_t)(bads >> (4 * q)), x)) acc = NAN;
              float* o = grest_rgb + 3 * JR * i0 + e;
              *o = v0 == 0 ? acc : *o + acc;
            }
          }
        }
      }
      if (gdc_rgb && lane < 3 * ng) {
        const float4 x = lds4(G + 64 * (lane % 3) + 4 * (lane / 3));
        const float acc = ((x.x + x.y) + x.z) + x.w;
        float* o = gdc_rgb + 3 * i0 + lane;
        *o = v0 == 0 ? acc : *o + acc;
      }
      if constexpr (J > 0) {
        wave_sync();
        if (n_sem > 0 && valid) {
#pragma unroll
          for (int j = 0; j < JS; ++j) h[j + 1] += H[64 * j + lane];
        }
        bool redo = bad;
#pragma unroll
        for (int j = 1; j <= J; ++j) redo = redo || !(fabsf(h[j]) <= 3.0e38f);
        redo = redo && valid;
        bool share = valid;
        if (redo) {
          share = false;
#pragma unroll
          for (int j = 1; j <= J; ++j) h[j] = 0.0f;
          if constexpr (JR > 0)
            for (int a = 0; a < 3; ++a)
              if (gr[a] != 0.0f) {
                share = true;
#pragma unroll
                for (int j = 0; j < JR; ++j) h[j + 1] = fmaf(gr[a], sh.rgb_rest[(JR * iq + j) * 3 + a], h[j + 1]);
              }
          if constexpr (JS > 0)
            for (int c = 0; c < n_sem; ++c) {
              const float w = gsem[((v0 + vk) * n + iq) * n_sem + c];
              if (w != 0.0f) {
                share = true;
#pragma unroll
                for (int j = 0; j < JS; ++j) h[j + 1] = fmaf(w, sh.sem_rest[(JS * iq + j) * n_sem + c], h[j + 1]);
              }
            }
        }
        float gx, gy, gz;
        sh_grad_dot(d.x, d.y, d.z, D, h, gx, gy, gz);
        const float dd = d.x * gx + d.y * gy + d.z * gz;
        float u[3] = {(gx - d.x * dd) * d.w, (gy - d.y * dd) * d.w, (gz - d.z * dd) * d.w};
#pragma unroll
        for (int a = 0; a < 3; ++a) u[a] = share ? u[a] : 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) us[a] += (double)u[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          u[a] += dpp_xor1(u[a]);
          u[a] += dpp_xor2(u[a]);
        }
        if (vk < 3 && (lane >> 2) < ng) gmean[3 * iq + vk] = gm0 + (vk == 0 ? u[0] : vk == 1 ? u[1] : u[2]);
      }
      wave_sync();   // the next Gaussians' values overwrite these
    }
    if constexpr (J > 0) {   // the rho sums: one block reduction, one atomic per (view, component)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        // rho: R_v (d L/d mu), the camera centre -R^T t moving by -R^T rho
        double S = (double)V.R[3 * a] * us[0] + (double)V.R[3 * a + 1] * us[1] + (double)V.R[3 * a + 2] * us[2];
#pragma unroll
        for (int off = 4; off < 64; off <<= 1) S += __shfl_xor(S, off, 64);
        if (lane < kShV) s_red[wave][lane][a] = S;
      }
      __syncthreads();
      const int t = threadIdx.x;
      if (t < 3 * nv) {
        double S = 0.0;
        for (int w = 0; w < kShBwdWaves; ++w) S += s_red[w][t / 3][t % 3];
        if (S != 0.0) atomicAdd(gpose + 6 * (v0 + t / 3) + t % 3, (float)S);
      }
      __syncthreads();
    }
  }
}

template <int RD, int SD>
int launch_fwd_d(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views, float* rgb_out,
                 float* sem_out, hipStream_t s) {
  hipLaunchKernelGGL((k_sh_fwd<RD, SD>), dim3((unsigned)ceil_div(g.n, kShWaves * kShG)), dim3(64 * kShWaves), 0, s, g, sh,
                     n_sem, views, n_views, rgb_out, sem_out);
  return launch_status();
}

template <int RD, int SD>
int launch_bwd_d(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views,
                 const float* grgb, const float* gsem, float* gdc_rgb, float* grest_rgb, float* gdc_sem,
                 float* grest_sem, float* gmean, float* gpose, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(ceil_div(g.n, kShBwdWaves * kShG),
                                           resident_blocks(k_sh_bwd<RD, SD>, 64 * kShBwdWaves, 512));
  hipLaunchKernelGGL((k_sh_bwd<RD, SD>), dim3((unsigned)blocks), dim3(64 * kShBwdWaves), 0, s, g, sh, n_sem, views, n_views,
                     grgb, gsem, gdc_rgb, grest_rgb, gdc_sem, grest_sem, gmean, gpose);
  return launch_status();
}

// f(rgb degree, semantic degree) as compile-time constants, degrees up to 3 and MAX (1 or 2).
template <int MAX, class F>
int with_degrees(int rd, int sd, F f) {
  auto sem = [&](auto r) {
    if constexpr (MAX > 1) {
      if (sd == 2) return f(r, std::integral_constant<int, 2>());
    }
    return sd ? f(r, std::integral_constant<int, 1>()) : f(r, std::integral_constant<int, 0>());
  };
  if (rd == 0) return sem(std::integral_constant<int, 0>());
  if (rd == 1) return sem(std::integral_constant<int, 1>());
  if (rd == 2) return sem(std::integral_constant<int, 2>());
  return sem(std::integral_constant<int, 3>());
}

// Higher semantic degrees, a lane per (Gaussian, channel): each Gaussian takes an aligned group of `gsz` lanes (the
// channel count 3 + n_sem <= 63 rounded up to a power of two), its channels on consecutive
// lanes, so loads and stores of a Gaussian's channels are contiguous and a reduction over
// them is a butterfly within the group.
__device__ __forceinline__ int group_size(int ct) {
  int g = 1;
  while (g < ct) g <<= 1;
  return g;
}

constexpr int kViewChunk = 256;   // camera centres staged in LDS per pass over the views

__device__ __forceinline__ void stage_centres(const gs_view* __restrict__ views, int v0, int nv, float* s_c) {
  for (int k = threadIdx.x; k < nv; k += blockDim.x) {
    const gs_view V = views[v0 + k];
    for (int a = 0; a < 3; ++a)
      s_c[3 * k + a] = -(V.R[a] * V.t[0] + V.R[3 + a] * V.t[1] + V.R[6 + a] * V.t[2]);
  }
}

// Channel c of Gaussian i: the constant band, the degree and the coefficient walk of its
// feature array (rgb: c < 3; semantics: c >= 3).
struct ShChan {
  const float* rest;   // first coefficient of the channel, or null
  int stride, deg;
  float dc;
};

__device__ __forceinline__ ShChan sh_chan(const gs_gaussians& g, const gs_sh& sh, int n_sem, int64_t i, int c) {
  ShChan h;
  const bool rgb = c < 3;
  const int ch = rgb ? 3 : n_sem;
  const int k = rgb ? c : c - 3;
  h.deg = rgb ? sh.rgb_degree : sh.sem_degree;
  h.dc = rgb ? g.rgb[3 * i + k] : g.sem[(int64_t)n_sem * i + k];
  const int nk = (h.deg + 1) * (h.deg + 1) - 1;
  const float* base = rgb ? sh.rgb_rest : sh.sem_rest;
  h.rest = (h.deg > 0) ? base + ((int64_t)i * nk) * ch + k : nullptr;
  h.stride = ch;
  return h;
}

__global__ __launch_bounds__(256) void k_sh_fwd_lanes(gs_gaussians g, gs_sh sh, int n_sem, const gs_view* __restrict__ views,
                                                int n_views, float* __restrict__ rgb_out, float* __restrict__ sem_out) {
  __shared__ float s_c[3 * kViewChunk];
  const int Ct = 3 + n_sem, gsz = group_size(Ct);
  const int64_t i0 = (int64_t)blockIdx.x * (256 / gsz) + threadIdx.x / gsz;
  const int c0 = (int)(threadIdx.x % gsz);
  const bool live = i0 < g.n && c0 < Ct;
  const int64_t i = live ? i0 : 0;
  const int c = live ? c0 : 0;
  ShChan h{};
  float coef[16];
  float mx = 0.0f, my = 0.0f, mz = 0.0f;
  if (live) {
    h = sh_chan(g, sh, n_sem, i, c);
    const int K = (h.deg + 1) * (h.deg + 1);
#pragma unroll
    for (int j = 1; j < 16; ++j) coef[j] = j < K ? h.rest[(int64_t)(j - 1) * h.stride] : 0.0f;
    mx = g.mean[3 * i];
    my = g.mean[3 * i + 1];
    mz = g.mean[3 * i + 2];
  }
  for (int v0 = 0; v0 < n_views; v0 += kViewChunk) {
    const int nv = min(kViewChunk, n_views - v0);
    __syncthreads();
    stage_centres(views, v0, nv, s_c);
    __syncthreads();
    if (!live) continue;
    for (int k = 0; k < nv; ++k) {
      float f = h.dc;
      if (h.deg > 0) {
        const float ux = mx - s_c[3 * k], uy = my - s_c[3 * k + 1], uz = mz - s_c[3 * k + 2];
        const float ir = rsqrtf(ux * ux + uy * uy + uz * uz);
        float Y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) Y[j] = 0.0f;
        sh_basis(ux * ir, uy * ir, uz * ir, h.deg, Y);
#pragma unroll
        for (int j = 1; j < 16; ++j) f = fmaf(Y[j], coef[j], f);
      }
      const int64_t v = v0 + k;
      if (c < 3) rgb_out[(v * g.n + i) * 3 + c] = f;
      else sem_out[(v * g.n + i) * n_sem + (c - 3)] = f;
    }
  }
}

// The backward, one lane per (Gaussian, channel), persistent blocks of 256 lanes walking the
// Gaussians: the constant band and the bands sum the feature gradient (times Y_j) over views;
// the channel's share of d L/d d, g_c sum_j k_jc dY_j/dd, goes through the normalisation
// (linear, so channels can be summed in any order) to the mean, summed over the Gaussian's
// lane group by a butterfly, and to the pose's rho (gpose[v][0..2] += R_v sum). Views are
// taken kPoseViews at a time: each lane keeps that many rho sums in registers over all its
// Gaussians, so a block adds to each pose once per chunk (a grid of few blocks keeps those
// same-address atomics few). The bands of a later chunk are added to the first chunk's.
constexpr int kPoseViews = 4;
constexpr int kShBwdThreads = 256;

// What one lane reads for one Gaussian: its channel's bands, the mean, the feature gradient
// of each view of the chunk.
struct ShIn {
  float coef[16];
  float m[3];
  float gm0[3];   // the mean gradient so far (read by the lane that adds to it, the only writer)
  float gf[kPoseViews];
};

__device__ __forceinline__ void sh_load(const gs_gaussians& g, const gs_sh& sh, int n_sem, int64_t i, int c, bool live,
                                        int v0, int nv, const float* __restrict__ grgb,
                                        const float* __restrict__ gsem, const float* gmean, ShIn& in) {
  const bool rgb = c < 3;
  const int ch = rgb ? 3 : n_sem, kc = rgb ? c : c - 3;
  const int deg = rgb ? sh.rgb_degree : sh.sem_degree;
  const int K = (deg + 1) * (deg + 1);
  const float* rest = rgb ? sh.rgb_rest : sh.sem_rest;
  const float* r = (live && deg > 0) ? rest + (int64_t)i * (K - 1) * ch + kc : nullptr;
#pragma unroll
  for (int j = 0; j < 16; ++j) in.coef[j] = (r && j >= 1 && j < K) ? r[(int64_t)(j - 1) * ch] : 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) in.m[a] = live ? g.mean[3 * i + a] : 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) in.gm0[a] = (live && c == 0 && gmean) ? gmean[3 * i + a] : 0.0f;
#pragma unroll
  for (int k = 0; k < kPoseViews; ++k) {
    const int64_t v = v0 + k;
    in.gf[k] = (live && k < nv) ? (rgb ? grgb[(v * g.n + i) * 3 + c] : gsem[(v * g.n + i) * n_sem + kc]) : 0.0f;
  }
}

__global__ __launch_bounds__(kShBwdThreads) void k_sh_bwd_lanes(gs_gaussians g, gs_sh sh, int n_sem,
                                                          const gs_view* __restrict__ views, int n_views,
                                                          const float* __restrict__ grgb,
                                                          const float* __restrict__ gsem, float* __restrict__ gdc_rgb,
                                                          float* __restrict__ grest_rgb, float* __restrict__ gdc_sem,
                                                          float* __restrict__ grest_sem, float* __restrict__ gmean,
                                                          float* __restrict__ gpose) {
  __shared__ double red[kShBwdThreads / 64][3 * kPoseViews];
  const int Ct = 3 + n_sem, gsz = group_size(Ct);
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int per_block = kShBwdThreads / gsz;          // Gaussians per block and pass
  const int64_t step = (int64_t)gridDim.x * per_block;
  const int c0 = tid % gsz;
  const int c = c0 < Ct ? c0 : 0;
  const bool rgb = c < 3;
  const int ch = rgb ? 3 : n_sem, kc = rgb ? c : c - 3;
  const int deg = rgb ? sh.rgb_degree : sh.sem_degree;
  const int nk = (deg + 1) * (deg + 1);
  const bool any_dir = sh.rgb_degree > 0 || sh.sem_degree > 0;
  for (int v0 = 0; v0 < n_views; v0 += kPoseViews) {
    const int nv = min(kPoseViews, n_views - v0);
    float pr[kPoseViews][3];
#pragma unroll
    for (int k = 0; k < kPoseViews; ++k) pr[k][0] = pr[k][1] = pr[k][2] = 0.0f;
    float Rv[kPoseViews][9], cv[kPoseViews][3];   // the chunk's rotations and camera centres
#pragma unroll
    for (int k = 0; k < kPoseViews; ++k) {
      const gs_view V = views[v0 + min(k, nv - 1)];
#pragma unroll
      for (int e = 0; e < 9; ++e) Rv[k][e] = V.R[e];
#pragma unroll
      for (int a = 0; a < 3; ++a) cv[k][a] = -(V.R[a] * V.t[0] + V.R[3 + a] * V.t[1] + V.R[6 + a] * V.t[2]);
    }
    int64_t gb = (int64_t)blockIdx.x * per_block;
    ShIn cur;
    {
      const int64_t i0 = gb + tid / gsz;
      const bool live = i0 < g.n && c0 < Ct;
      sh_load(g, sh, n_sem, live ? i0 : 0, c, live && c0 < Ct, v0, nv, grgb, gsem, any_dir ? gmean : nullptr, cur);
    }
    for (; gb < g.n; gb += step) {
      const int64_t i0 = gb + tid / gsz;
      const bool live = i0 < g.n && c0 < Ct;
      const int64_t i = live ? i0 : 0;
      ShIn nxt;                               // the next Gaussian's inputs, in flight meanwhile
      {
        const int64_t j0 = gb + step + tid / gsz;
        const bool nlive = j0 < g.n && c0 < Ct;
        sh_load(g, sh, n_sem, nlive ? j0 : 0, c, nlive, v0, nv, grgb, gsem, any_dir ? gmean : nullptr, nxt);
      }
      float acc[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
      float gm[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < kPoseViews; ++k) {
        const float gf = cur.gf[k];
        acc[0] += gf;
        if (deg == 0 || gf == 0.0f) continue;
        const float ux = cur.m[0] - cv[k][0], uy = cur.m[1] - cv[k][1], uz = cur.m[2] - cv[k][2];
        const float ir = rsqrtf(ux * ux + uy * uy + uz * uz);
        const float dx = ux * ir, dy = uy * ir, dz = uz * ir;
        float Y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) Y[j] = 0.0f;
        sh_basis(dx, dy, dz, deg, Y);
#pragma unroll
        for (int j = 1; j < 16; ++j) acc[j] = fmaf(Y[j], gf, acc[j]);
        float gx, gy, gz;   // sum_j k_jc dY_j/dd, times g_c below (linear in g_c)
        sh_grad_dot(dx, dy, dz, deg, cur.coef, gx, gy, gz);
        const float dd = dx * gx + dy * gy + dz * gz;
        const float gi = gf * ir;
        const float u0 = (gx - dx * dd) * gi, u1 = (gy - dy * dd) * gi, u2 = (gz - dz * dd) * gi;
        gm[0] += u0;
        gm[1] += u1;
        gm[2] += u2;
        // rho: R_v (d L/d mu), the camera centre -R^T t moving by -R^T rho
        pr[k][0] += Rv[k][0] * u0 + Rv[k][1] * u1 + Rv[k][2] * u2;
        pr[k][1] += Rv[k][3] * u0 + Rv[k][4] * u1 + Rv[k][5] * u2;
        pr[k][2] += Rv[k][6] * u0 + Rv[k][7] * u1 + Rv[k][8] * u2;
      }
      if (live) {
        float* gdc = rgb ? gdc_rgb : gdc_sem;
        float* grest = rgb ? grest_rgb : grest_sem;
        // the first chunk of views stores, later chunks add (no read before the first store)
        if (gdc) {
          float* o = gdc + (int64_t)ch * i + kc;
          if (v0 == 0) *o = acc[0];
          else *o += acc[0];
        }
        if (deg > 0 && grest) {
          float* o = grest + (int64_t)i * (nk - 1) * ch + kc;
          if (v0 == 0) {
#pragma unroll
            for (int j = 1; j < 16; ++j)
              if (j < nk) o[(int64_t)(j - 1) * ch] = acc[j];
          } else {
#pragma unroll
            for (int j = 1; j < 16; ++j)
              if (j < nk) o[(int64_t)(j - 1) * ch] += acc[j];
          }
        }
      }
      if (any_dir) {   // the mean's share over the Gaussian's channels, added by the group's first lane
        for (int o = 1; o < gsz; o <<= 1)
          for (int k = 0; k < 3; ++k) gm[k] += __shfl_xor(gm[k], o, 64);
        if (live && c0 == 0)
          for (int k = 0; k < 3; ++k) gmean[3 * i + k] = cur.gm0[k] + gm[k];
      }
      cur = nxt;
    }
    if (any_dir) {   // the chunk's rho sums: one block reduction, one atomic per (view, component)
#pragma unroll
      for (int k = 0; k < kPoseViews; ++k)
        for (int a = 0; a < 3; ++a) {
          const double sum = wave_sum_d((double)pr[k][a]);
          if (lane == 0) red[wid][3 * k + a] = sum;
        }
      __syncthreads();
      if (tid < 3 * nv) {
        double S = 0.0;
        for (int w = 0; w < kShBwdThreads / 64; ++w) S += red[w][tid];
        if (S != 0.0) atomicAdd(gpose + 6 * (v0 + tid / 3) + tid % 3, (float)S);
      }
      __syncthreads();
    }
  }
}

int launch_fwd_lanes(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views, float* rgb_out,
                     float* sem_out, hipStream_t s) {
  int gsz = 1;
  while (gsz < 3 + n_sem) gsz <<= 1;
  hipLaunchKernelGGL(k_sh_fwd_lanes, dim3((unsigned)ceil_div(g.n, 256 / gsz)), dim3(256), 0, s, g, sh, n_sem, views,
                     n_views, rgb_out, sem_out);
  return launch_status();
}

int launch_bwd_lanes(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views,
                     const float* grgb, const float* gsem, float* gdc_rgb, float* grest_rgb, float* gdc_sem,
                     float* grest_sem, float* gmean, float* gpose, hipStream_t s) {
  int gsz = 1;
  while (gsz < 3 + n_sem) gsz <<= 1;
  // a few blocks per CU: enough lanes in flight, few same-address atomics on the poses
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    cus = 256;
  const int64_t blocks = std::min<int64_t>(ceil_div(g.n, kShBwdThreads / gsz), 4 * (int64_t)cus);
  hipLaunchKernelGGL(k_sh_bwd_lanes, dim3((unsigned)blocks), dim3(kShBwdThreads), 0, s, g, sh, n_sem, views, n_views, grgb,
                     gsem, gdc_rgb, grest_rgb, gdc_sem, grest_sem, gmean, gpose);
  return launch_status();
}

}  // namespace

int launch_sh_fwd(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views, float* rgb_out,
                  float* sem_out, hipStream_t s) {
  if (g.n == 0 || n_views == 0) return GS_OK;
  const int sd = n_sem ? sh.sem_degree : 0;
  if (sd > kShFwdDegree) return launch_fwd_lanes(g, sh, n_sem, views, n_views, rgb_out, sem_out, s);
  return with_degrees<kShFwdDegree>(sh.rgb_degree, sd, [&](auto r, auto d) {
    return launch_fwd_d<r(), d()>(g, sh, n_sem, views, n_views, rgb_out, sem_out, s);
  });
}

int launch_sh_bwd(const gs_gaussians& g, const gs_sh& sh, int n_sem, const gs_view* views, int n_views,
                  const float* grgb, const float* gsem, float* gdc_rgb, float* grest_rgb, float* gdc_sem,
                  float* grest_sem, float* gmean, float* gpose, hipStream_t s) {
  if (g.n == 0 || n_views == 0) return GS_OK;
  const int sd = n_sem ? sh.sem_degree : 0;
  if (sd > kShBwdDegree)
    return launch_bwd_lanes(g, sh, n_sem, views, n_views, grgb, gsem, gdc_rgb, grest_rgb, gdc_sem, grest_sem, gmean,
                            gpose, s);
  return with_degrees<kShBwdDegree>(sh.rgb_degree, sd, [&](auto r, auto d) {
    return launch_bwd_d<r(), d()>(g, sh, n_sem, views, n_views, grgb, gsem, gdc_rgb, grest_rgb, gdc_sem, grest_sem,
                                  gmean, gpose, s);
  });
}

}  // namespace gs
