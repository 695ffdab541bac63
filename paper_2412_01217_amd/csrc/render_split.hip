// Tile compositing (eq. 7-9) and its reverse pass, with every dense contraction on the
// bfloat16 matrix cores of gfx950 (v_mfma_f32_16x16x32_bf16, 2.5 PFLOP/s) and single
// precision kept by splitting each operand x = hi + lo, hi = bf16(x), lo = bf16(x - hi):
//   a b ~ a_hi b_hi + a_hi b_lo + a_lo b_hi      (relative error about 2^-16)
//
// Forward, per wave of 64 pixels and per batch of 32 depth-ordered Gaussians that reach them:
//   each lane runs its pixel's transmittance recurrence, w[p][i] = alpha_i T_i, then
//   out^T[c][p] += sum_i F^T[c][i] W^T[i][p] on the matrix cores.
// Backward, per wave and per group of 16 reaching Gaussians (back to front):
//   GF^T[i][p] = sum_c F[i][c] G^T[c][p]  (g . f of every pixel-Gaussian pair; it decides
//     dL/dalpha, in which terms cancel) in single precision: three bfloat16 parts with 32 padded
//     channels, v_mfma_f32_16x16x4f32 with 64; a 4x4 block transpose across lane rows (permlane
//     swaps) hands every lane its own pixel's 16 values;
//   each lane runs the reverse recurrence (T recovered with the reciprocal of 1 - alpha)
//     and writes w[i][p] to LDS, Gaussian-major;
//   dF[i][c] = sum_p W^T[i][p] G[p][c]                       (feature gradients)
//   the 2D mean, conic and opacity gradients are summed per pair in single precision across the
//   wave: expanding them into moments about a fixed centre would lose accuracy for compact
//   Gaussians.
//
// 16x16x32 bf16 operand layout (lane l, verified on the device):
//   A[i][k]: i = l % 16, k = 8 (l / 16) + 0..7     B[k][j]: k = 8 (l / 16) + 0..7, j = l % 16
//   D[i][j]: j = l % 16, i = 4 (l / 16) + r, r = 0..3
#include <type_traits>

#include "common.h"

namespace gs {

int64_t scan_partials_needed(int64_t n);
int scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* partial, uint64_t* total, hipStream_t s);

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

constexpr int kB = 32;          // Gaussians per batch
constexpr int kWs = kB + 4;     // dword stride of a pixel-major row of 32 Gaussians
constexpr int kPs = 64 + 4;     // dword stride of a Gaussian-major row of a wave's 64 pixels

template <int NS>
struct SShape {
  static constexpr int K = 4 + NS;
  static constexpr int KP = (K + 31) / 32 * 32;   // channels padded to whole 32-wide k-steps
  static constexpr int KS = KP / 32;
  static constexpr int CB = KP / 16;              // 16-channel blocks
  static constexpr int CPT = KP / 8;              // channels staged per thread
  static constexpr int FST = KP + 4;              // dword stride of a Gaussian-major feature row
};

// x -> (bf16(x) << 16) | bf16(x - bf16(x))
__device__ __forceinline__ uint32_t pack_hl(float x) {
  const float h = (float)(__bf16)x;
  const bf2 v = __builtin_convertvector((f2){x - h, x}, bf2);
  return __builtin_bit_cast(uint32_t, v);
}

// Eight packed values -> the hi and lo bfloat16 operands.
__device__ __forceinline__ void unpack8(const uint4 a, const uint4 b, v8bf& hi, v8bf& lo) {
  const uint32_t d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint4 h, l;
  h.x = __builtin_amdgcn_perm(d[1], d[0], 0x07060302u);
  h.y = __builtin_amdgcn_perm(d[3], d[2], 0x07060302u);
  h.z = __builtin_amdgcn_perm(d[5], d[4], 0x07060302u);
  h.w = __builtin_amdgcn_perm(d[7], d[6], 0x07060302u);
  l.x = __builtin_amdgcn_perm(d[1], d[0], 0x05040100u);
  l.y = __builtin_amdgcn_perm(d[3], d[2], 0x05040100u);
  l.z = __builtin_amdgcn_perm(d[5], d[4], 0x05040100u);
  l.w = __builtin_amdgcn_perm(d[7], d[6], 0x05040100u);
  hi = __builtin_bit_cast(v8bf, h);
  lo = __builtin_bit_cast(v8bf, l);
}

__device__ __forceinline__ void load_op(const uint32_t* p, v8bf& hi, v8bf& lo) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  const uint4 b = *reinterpret_cast<const uint4*>(p + 4);
  unpack8(a, b, hi, lo);
}

// Splits eight floats into hi and lo operands, two values per conversion.
__device__ __forceinline__ void split8(const float* x, v8bf& hi, v8bf& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t hb = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){x[2 * k], x[2 * k + 1]}, bf2));
    const float h0 = __uint_as_float(hb << 16), h1 = __uint_as_float(hb & 0xffff0000u);
    h[k] = hb;
    l[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){x[2 * k] - h0, x[2 * k + 1] - h1}, bf2));
  }
  hi = __builtin_bit_cast(v8bf, make_uint4(h[0], h[1], h[2], h[3]));
  lo = __builtin_bit_cast(v8bf, make_uint4(l[0], l[1], l[2], l[3]));
}

// Splits eight floats into three bfloat16 parts, x = hi + mid + lo to about 2^-24 of x
// (each part the rounding of what the previous ones leave, every remainder exact).
__device__ __forceinline__ void split8x3(const float* x, v8bf& hi, v8bf& mid, v8bf& lo) {
  split8(x, hi, mid);
  const uint4 h = __builtin_bit_cast(uint4, hi), m = __builtin_bit_cast(uint4, mid);
  const uint32_t hw[4] = {h.x, h.y, h.z, h.w}, mw[4] = {m.x, m.y, m.z, m.w};
  uint32_t l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float r0 = (x[2 * k] - __uint_as_float(hw[k] << 16)) - __uint_as_float(mw[k] << 16);
    const float r1 = (x[2 * k + 1] - __uint_as_float(hw[k] & 0xffff0000u)) - __uint_as_float(mw[k] & 0xffff0000u);
    l[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){r0, r1}, bf2));
  }
  lo = __builtin_bit_cast(v8bf, make_uint4(l[0], l[1], l[2], l[3]));
}


// The render record as the compositing loops read it from LDS, 8 floats per Gaussian:
//   mx, my   mean2d relative to the tile's middle (the centre of its pixel (tw / 2, th / 2)),
//            so that a pixel's offset is its integer position relative to that pixel minus
//            (mx, my); a middle origin keeps |mx|, |my| (and their rounding) small for every
//            tile shape;
//   a, b, c  the conic scaled so that a dx^2 + b dx dy + c dy^2 is the exponent of eq. 4
//            in base 2: a = -A log2(e) / 2, b = -B log2(e), c = -C log2(e) / 2;
//   o        opacity (two floats of padding).
// The mean's hi + lo sum is rounded once, after the exact subtraction of the tile origin.
constexpr float kLog2e = 1.4426950408889634f;
struct LRec {
  float4 m;   // mx, my, a, b
  float2 c;   // c, o
};
// Stages half of a render record (part 0: mean hi, lo; part 1: conic, opacity).
__device__ __forceinline__ void stage_rec(float* s_rec, int q, const float4 r, int part, float ox, float oy) {
  float* d = s_rec + 8 * q;
  if (part == 0) {
    *reinterpret_cast<float2*>(d) = make_float2((r.x - ox) + r.z, (r.y - oy) + r.w);
  } else {
    *reinterpret_cast<float2*>(d + 2) = make_float2(-0.5f * kLog2e * r.x, -kLog2e * r.y);
    *reinterpret_cast<float2*>(d + 4) = make_float2(-0.5f * kLog2e * r.z, r.w);
  }
}
__device__ __forceinline__ LRec load_rec(const float* s_rec, int q) {
  LRec r;
  r.m = *reinterpret_cast<const float4*>(s_rec + 8 * q);
  r.c = *reinterpret_cast<const float2*>(s_rec + 8 * q + 4);
  return r;
}

// Base-2 footprint exponent at tile-local pixel (lx, ly), clamped at zero; dx, dy are the
// pixel's offsets from the mean and t = a dx + b dy.
__device__ __forceinline__ float local_power2(float lx, float ly, const LRec& r, float& dx, float& dy, float& t) {
  dx = lx - r.m.x;
  dy = ly - r.m.y;
  t = __builtin_fmaf(r.m.z, dx, r.m.w * dy);
  return fminf(__builtin_fmaf(t, dx, (r.c.x * dy) * dy), 0.0f);
}

// Whether the footprint can reach alpha_min anywhere in the rectangle [x0, x1] x [y0, y1]
// of tile-local positions (a wave's band of pixel centres): false only if the largest
// base-2 exponent over the continuous rectangle lies below log2(alpha_min / o) by a margin
// (0.1, far above the exponent's single-precision rounding), so a pixel of the band never
// takes the Gaussian. The exponent is concave; its maximum is 0 at the mean if the mean
// lies in the rectangle, else on an edge, at the edge's own vertex clamped to the edge.
// A degenerate record (a non-finite maximum) is never skipped.
__device__ __forceinline__ bool band_reaches(const LRec& r, float x0, float x1, float y0, float y1, float amin) {
  const float a = r.m.z, b = r.m.w, c = r.c.x;
  const float X0 = x0 - r.m.x, X1 = x1 - r.m.x, Y0 = y0 - r.m.y, Y1 = y1 - r.m.y;
  if (X0 <= 0.0f && X1 >= 0.0f && Y0 <= 0.0f && Y1 >= 0.0f) return true;
  // the vertices from approximate reciprocals: the exponent is flat there, so the value at
  // a slightly moved point differs from the maximum by far less than the margin
  const float ia = -0.5f * __builtin_amdgcn_rcpf(a), ic = -0.5f * __builtin_amdgcn_rcpf(c);
  auto along_x = [&](float Y) {   // dy = Y, dx over [X0, X1]
    const float dx = fminf(X1, fmaxf(X0, b * Y * ia));
    return (a * dx + b * Y) * dx + c * Y * Y;
  };
  auto along_y = [&](float X) {   // dx = X, dy over [Y0, Y1]
    const float dy = fminf(Y1, fmaxf(Y0, b * X * ic));
    return (c * dy + b * X) * dy + a * X * X;
  };
  const float m = fmaxf(fmaxf(along_x(Y0), along_x(Y1)), fmaxf(along_y(X0), along_y(X1)));
  return !(m < __log2f(amin) - __log2f(r.c.y) - 0.1f);
}

__device__ __forceinline__ v4f mma(v8bf a, v8bf b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v4f mma3(v8bf ah, v8bf al, v8bf bh, v8bf bl, v4f c) {
  c = mma(ah, bh, c);
  c = mma(ah, bl, c);
  c = mma(al, bh, c);
  return c;
}
// Six products of three-part operands: a b to about 2^-24 relative per product term.
__device__ __forceinline__ v4f mma6(const v8bf (&a)[3], const v8bf (&b)[3], v4f c) {
  c = mma(a[0], b[0], c);
  c = mma(a[0], b[1], c);
  c = mma(a[1], b[0], c);
  c = mma(a[0], b[2], c);
  c = mma(a[1], b[1], c);
  c = mma(a[2], b[0], c);
  return c;
}
__device__ __forceinline__ v4f zero4() { return (v4f){0.0f, 0.0f, 0.0f, 0.0f}; }

// Batch staging, double-buffered through registers: thread t stages Gaussian q = t / 8
// of the batch, channels [(t % 8) CPT, +CPT) of its features and, for t % 8 < 2, half of
// its 8-float record. The batch's Gaussian ids are loaded a batch earlier than its data
// (load_ids, then fetch_data), so that the gathers that depend on them issue without
// waiting for a load.
template <int NS>
struct SStage {
  static constexpr int CPT = SShape<NS>::CPT;
  float4 r;
  uint32_t gid, gpre;
  float f[CPT];

  __device__ __forceinline__ void load_ids(const uint32_t* __restrict__ vals, uint32_t b, int cnt) {
    const int q = threadIdx.x >> 3;
    gpre = q < cnt ? vals[b + q] : 0u;
  }
  __device__ __forceinline__ void fetch(const uint32_t* __restrict__ vals, uint32_t b, int cnt, int item, int64_t n,
                                        const float* __restrict__ rec, const float* __restrict__ depth,
                                        const float* __restrict__ rgb, const float* __restrict__ sem,
                                        const uint16_t* __restrict__ emb, int n_sem, int64_t foff) {
    load_ids(vals, b, cnt);
    fetch_data(cnt, item, n, rec, depth, rgb, sem, emb, n_sem, foff);
  }
  // gathers the data of the batch whose ids load_ids loaded (cnt Gaussians)
  __device__ __forceinline__ void fetch_data(int cnt, int item, int64_t n, const float* __restrict__ rec,
                                             const float* __restrict__ depth, const float* __restrict__ rgb,
                                             const float* __restrict__ sem, const uint16_t* __restrict__ emb,
                                             int n_sem, int64_t foff) {
    const int q = threadIdx.x >> 3, part = threadIdx.x & 7;
    const bool live = q < cnt;
    const uint32_t g = gpre;
    gid = g;
    const int64_t e = (int64_t)item * n + g;
    r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live && part < 2) r = reinterpret_cast<const float4*>(rec + kRecFloats * e)[part];
    const int Kr = 4 + n_sem;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int k = part * CPT + j;
      float v = 0.0f;
      if (live && k < Kr) {
        if (k < 3) v = rgb[3 * ((int64_t)g + foff) + k];
        else if (k == 3) v = depth[e];
        else if (emb) v = __uint_as_float((uint32_t)emb[(int64_t)n_sem * ((int64_t)g + foff) + (k - 4)] << 16);
        else v = sem[(int64_t)n_sem * ((int64_t)g + foff) + (k - 4)];
      }
      f[j] = v;
    }
  }
  // features Gaussian-major, single precision: s_f[q][c]; Gaussian ids to s_gid[q]
  __device__ __forceinline__ void commit_rows(float* s_rec, float* s_f, uint32_t* s_gid, float ox, float oy) const {
    const int q = threadIdx.x >> 3, part = threadIdx.x & 7;
    if (part < 2) stage_rec(s_rec, q, r, part, ox, oy);
    if (part == 0) s_gid[q] = gid;
    float* dst = s_f + q * SShape<NS>::FST + part * CPT;
#pragma unroll
    for (int j = 0; j < CPT; j += 4) *reinterpret_cast<float4*>(dst + j) = make_float4(f[j], f[j + 1], f[j + 2], f[j + 3]);
  }
};

// ------------------------------------------------------------------------- forward
// Long tile lists are cut into segments of seg_len(cfg) list positions. The reverse pass
// takes every segment as a work item of its own; the forward walks up to `chunk`
// consecutive segments of a list in one work item (one sequential transmittance chain),
// so that only lists longer than a chunk need a starting transmittance from a pre-pass.
// The forward state and the reverse pass's segment list are sized for the configured length
// (at most one segment per tile more than the duplicates over it); seg_len = 0 selects
// kSegDefault.
constexpr int kSegDefault = 1024;
__host__ __device__ inline int seg_len(const gs_config& cfg) { return cfg.seg_len > 0 ? cfg.seg_len : kSegDefault; }

// Segments per forward work item (cfg.fwd_chunk; 0 = the whole list).
__host__ __device__ inline int fwd_chunk(const gs_config& cfg) { return cfg.fwd_chunk > 0 ? cfg.fwd_chunk : 1 << 16; }

// Saved state of a forward that split its long lists, one slot per segment (a tile's
// slots are consecutive from tbase[tile]; the work list has an entry per slot):
//   P[slot][px]     at the first slot of a chunk: product of (1 - alpha) over the chunk's
//                   Gaussians with alpha >= alpha_min, the stop rule ignored
//                   (transmittance pre-pass; not for a list's last chunk);
//   Te[slot][px]    T at the segment's end, for pixels active in it;
//   info[slot][px]  1 + list position of the last blend in it (0 if none) | active at its
//                   start << 30 | stopped inside it << 31;
//   CS[slot][k][px] the segment's colour, then the sum of the colours of all later
//                   segments of the list, which the reverse pass turns into its starting
//                   sum of w (g . f) with one dot product.
struct FState {
  uint32_t* tcnt;    // [n_tiles] segments of the tile: 1 = whole list, no slot data
  uint32_t* tbase;   // [n_tiles] first slot of the tile
  float* P;
  float* Te;
  uint32_t* info;
  float* CS;
};
constexpr uint32_t kInfoActive = 1u << 30, kInfoStopped = 1u << 31, kInfoLast = kInfoActive - 1;

// Segments per tile: every tile is at least one item (it writes the tile's output).
__global__ __launch_bounds__(256) void k_fseg_count(const uint32_t* __restrict__ ranges, int n_tiles, int order,
                                                    uint32_t seg, uint32_t* __restrict__ cnt_ord) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_tiles) return;
  const uint32_t len = ranges[2 * (int64_t)t + 1] - ranges[2 * (int64_t)t];
  cnt_ord[order ? t : n_tiles - 1 - t] = len <= seg ? 1u : (len + seg - 1) / seg;
}

// Transmittance pre-pass: P of every chunk of a list but the last. Persistent blocks
// take work items from ctl[2].
__global__ __launch_bounds__(256) void k_fwd_trans(gs_config cfg, const float* __restrict__ rec, int64_t n,
                                                   const gs_item* __restrict__ items, int n_items,
                                                   const uint32_t* __restrict__ vals,
                                                   const uint32_t* __restrict__ ranges, const uint2* __restrict__ work,
                                                   uint32_t* __restrict__ ctl, float* __restrict__ P) {
  __shared__ __align__(16) float s_rec[8 * kB];
  __shared__ uint32_t s_wi;
  const int tid = threadIdx.x;
  const int tws = tile_shift(cfg);
  const float lx = (float)((tid & ((1 << tws) - 1)) - (1 << (tws - 1))), ly = (float)((tid >> tws) - (128 >> tws));
  const float amin = cfg.alpha_min, amax = cfg.alpha_max, tmin = cfg.t_min;
  const uint32_t n_work = ctl[0];
  for (;;) {
    if (tid == 0) s_wi = atomicAdd(&ctl[2], 1u);
    lds_barrier();
    const uint32_t wi = s_wi;
    lds_barrier();
    if (wi >= n_work) break;
    const uint2 wk = work[wi];
    const int seg = (int)(wk.y & 0xffffu), nseg = (int)(wk.y >> 16);
    const int chunk = fwd_chunk(cfg);
    if (seg % chunk != 0 || seg + chunk >= nseg) continue;
    const Ctx c = make_ctx_of(items, n_items, ranges, (int)wk.x, tws);
    int u, v;
    tile_pixel(c, tid, u, v);
    const bool inside = u < c.W && v < c.H;
    const float ox = (float)tile_mid_x(c) + 0.5f, oy = (float)tile_mid_y(c) + 0.5f;
    const int seglen = seg_len(cfg);
    const uint32_t a0 = c.start + seg * seglen;
    const uint32_t b0 = (uint32_t)min((int64_t)c.end, (int64_t)a0 + (int64_t)chunk * seglen);
    // thread t < 64 stages half (t % 2) of the record of Gaussian t / 2
    const int q = tid >> 1, part = tid & 1;
    auto fetch = [&](uint32_t b) -> float4 {
      if (tid >= 2 * kB || b + q >= b0) return make_float4(0.f, 0.f, 0.f, 0.f);
      const int64_t e = (int64_t)c.item * n + vals[b + q];
      return reinterpret_cast<const float4*>(rec + kRecFloats * e)[part];
    };
    float p = 1.0f;
    float4 r = fetch(a0);
    for (uint32_t b = a0; b < b0; b += kB) {
      // below t_min the product's exact value no longer matters
      if (__syncthreads_count(inside & (p >= tmin)) == 0) break;
      if (tid < 2 * kB) stage_rec(s_rec, q, r, part, ox, oy);
      lds_barrier();
      const int cnt = (int)min((uint32_t)kB, b0 - b);
      r = fetch(b + kB);
      // records of the next four Gaussians are read while the current four are used
      LRec R[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) R[e] = load_rec(s_rec, e);
#pragma unroll
      for (int k4 = 0; k4 < kB; k4 += 4) {
        LRec N[4];
        if (k4 + 4 < kB)
#pragma unroll
          for (int e = 0; e < 4; ++e) N[e] = load_rec(s_rec, k4 + 4 + e);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float dx, dy, t;
          const float araw = R[e].c.y * __builtin_amdgcn_exp2f(local_power2(lx, ly, R[e], dx, dy, t));
          const bool ok = (k4 + e < cnt) & (araw >= amin);
          p = ok ? p - fminf(amax, araw) * p : p;
        }
        if (k4 + 4 < kB)
#pragma unroll
          for (int e = 0; e < 4; ++e) R[e] = N[e];
      }
    }
    P[(int64_t)wi * kTilePx + tid] = p;
  }
}

// Swaps the 4x4 blocks (lane row R, register group X[pb]) -> (lane row pb, group R):
// permlane32 exchanges rows 0,1 with 2,3, permlane16 rows 0 with 1 and 2 with 3.
template <int NK>
__device__ __forceinline__ void block_transpose(uint32_t (&X)[4][NK]) {
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    auto s02 = __builtin_amdgcn_permlane32_swap(X[0][k], X[2][k], false, false);
    auto s13 = __builtin_amdgcn_permlane32_swap(X[1][k], X[3][k], false, false);
    X[0][k] = s02[0];
    X[2][k] = s02[1];
    X[1][k] = s13[0];
    X[3][k] = s13[1];
    auto s01 = __builtin_amdgcn_permlane16_swap(X[0][k], X[1][k], false, false);
    auto s23 = __builtin_amdgcn_permlane16_swap(X[2][k], X[3][k], false, false);
    X[0][k] = s01[0];
    X[1][k] = s01[1];
    X[2][k] = s23[0];
    X[3][k] = s23[1];
  }
}

// A wave's 64 pixels are a compact region of the tile: an 8x8 quad (16x4 of a 64x4 tile).
// Fewer Gaussians reach a quad than a 16x4 band (1.1-1.5 of the four regions per list entry
// against 1.2-1.6), and more of a reached quad's pixels take them.
struct Region {
  int px;                     // this lane's pixel, row-major in the tile
  float lx, ly;               // its position from the tile's middle pixel
  float x0, x1, y0, y1;       // the region's corner pixels, likewise
};
__device__ __forceinline__ Region wave_region(int tws, int r, int lane) {
  const int rws = tws == 6 ? 4 : 3, per = 1 << (tws - rws);   // regions side by side in the tile
  const int x0 = (r & (per - 1)) << rws, y0 = (r / per) * (64 >> rws);
  const int x = x0 + (lane & ((1 << rws) - 1)), y = y0 + (lane >> rws);
  const int mx = 1 << (tws - 1), my = 128 >> tws;
  Region g;
  g.px = (y << tws) + x;
  g.lx = (float)(x - mx);
  g.ly = (float)(y - my);
  g.x0 = (float)(x0 - mx);
  g.x1 = g.x0 + (float)((1 << rws) - 1);
  g.y0 = (float)(y0 - my);
  g.y1 = g.y0 + (float)((64 >> rws) - 1);
  return g;
}

// Where a Gaussian's channels come from, and how its semantic row is read (a template parameter:
// a branch between the loads would make the compiler wait for them where its sides meet).
struct FeatSrc {
  const float *rgb, *sem, *depth;
  const uint16_t* emb;
  int n_sem;
};
enum FeatMode {
  kRowVec,     // class logits, 16 bytes at a time: n_sem a multiple of 4, the array 16-byte aligned
  kEmbVec,     // embedding, 8 bytes at a time: the array 16-byte aligned (a row is 32 bytes)
  kValues      // logits or embedding, value by value
};
inline FeatMode feat_mode(const gs_gaussians& g, int n_sem) {
  if (g.emb) return (uintptr_t)g.emb % 16 == 0 ? kEmbVec : kValues;
  return n_sem > 0 && n_sem % 4 == 0 && (uintptr_t)g.sem % 16 == 0 ? kRowVec : kValues;
}
// The quads of channels k .. k + 3 (k % 4 = 0) of the rows of Gaussians g[p], into f[4 p ..]. With
// kRowVec every lane loads from a valid address, and what lies past the last channel is dropped when
// it is used. kValues has no such loads: a value's is conditional on its channel and picks logits or
// embedding, zero past the last channel, and the compiler waits where the sides meet (class counts
// that four does not divide, arrays off a 16-byte boundary).
template <int MODE, int NP>
__device__ __forceinline__ void load_quads(const FeatSrc& s, const uint32_t (&g)[NP], int64_t foff, int k, float* f) {
  if constexpr (MODE == kRowVec) {
    const float* a = s.sem + (int64_t)s.n_sem * foff + (k < s.n_sem ? k : 0);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float4 v = *reinterpret_cast<const float4*>(a + (uint64_t)(uint32_t)s.n_sem * g[p]);
      f[4 * p] = v.x;
      f[4 * p + 1] = v.y;
      f[4 * p + 2] = v.z;
      f[4 * p + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v = 0.0f;
        if (k + i < s.n_sem) {
          const int64_t at = (int64_t)s.n_sem * ((int64_t)g[p] + foff) + k + i;
          v = s.emb ? __uint_as_float((uint32_t)s.emb[at] << 16) : s.sem[at];
        }
        f[4 * p + i] = v;
      }
  }
}

// A batch's features on their way from memory to F^T in LDS. Neighbouring lanes read the
// neighbouring quads (four channels) of a row, so that a load touches few cache lines: QL
// lanes a Gaussian for plain semantics, four for an embedding (8 bytes each). Colour and depth
// come beside them: lane q < 32 Gaussian q's colour, lane 32 + q its depth.
template <int NS, int MODE>
struct Feats {
  static constexpr bool EMB = MODE == kEmbVec;
  static constexpr int KP = SShape<NS>::KP;
  static constexpr int QL = EMB ? 4 : KP / 4, NP = QL / 2;   // lanes a Gaussian, passes over 32 Gaussians
  float f[EMB ? 1 : 4 * NP];
  uint2 r[EMB ? NP : 1];
  float c0, c1, c2;

  // q-th queued Gaussian: its index at Q[8 q + 7] (0 where there is none); see load_quads
  __device__ __forceinline__ void load(const FeatSrc& s, const float* Q, int64_t foff, int64_t e0, int lane) {
    uint32_t g[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) g[p] = __float_as_uint(Q[8 * (p * (64 / QL) + lane / QL) + 7]);
    const uint32_t gc = __float_as_uint(Q[8 * (lane & 31) + 7]);
    if constexpr (EMB) {
      const uint16_t* a = s.emb + 4 * (lane % QL);
#pragma unroll
      for (int p = 0; p < NP; ++p) r[p] = *reinterpret_cast<const uint2*>(a + 16 * (uint64_t)g[p]);
    } else {
      load_quads<MODE>(s, g, foff, 4 * (lane % QL), f);
    }
    const float* a = lane < 32 ? s.rgb + 3 * ((int64_t)gc + foff) : s.depth + (e0 + gc);
    const int o = lane < 32 ? 1 : 0;   // (depth again for the lanes that have no colour to load)
    c0 = a[0];
    c1 = a[o];
    c2 = a[2 * o];
  }
  // F^T[channel][Gaussian], packed hi|lo (an embedding value is its own hi part), of cnt
  // Gaussians; zero for the rest of the batch and past the last channel
  __device__ __forceinline__ void commit(uint32_t* FT, int n_sem, int cnt, int lane) const {
    const int k = 4 * (lane % QL);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int q = p * (64 / QL) + lane / QL;
      uint32_t* d = FT + (4 + k) * kWs + q;
      // (a mask: a branch around each value's conversion would wait for the loads one by one. A quad
      // of a kRowVec row is whole or absent, one of kValues is zero past the last channel.)
      const uint32_t m = q < cnt && (EMB || k < n_sem) ? ~0u : 0u;
      if constexpr (EMB) {
        d[0] = (r[p].x << 16) & m;
        d[kWs] = (r[p].x & 0xffff0000u) & m;
        d[2 * kWs] = (r[p].y << 16) & m;
        d[3 * kWs] = (r[p].y & 0xffff0000u) & m;
      } else if (k < NS) {
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i * kWs] = pack_hl(f[4 * p + i]) & m;
      }
    }
    uint32_t* d = FT + (lane < 32 ? 0 : 3 * kWs) + (lane & 31);
    const uint32_t m = (lane & 31) < cnt ? ~0u : 0u;
    d[0] = pack_hl(c0) & m;
    if (lane < 32) {
      d[kWs] = pack_hl(c1) & m;
      d[2 * kWs] = pack_hl(c2) & m;
    }
  }
};

// The record of a list entry in the tile's frame (see LRec), from the two halves of gs_projected.rec.
__device__ __forceinline__ LRec local_rec(const float4 a, const float4 b, float ox, float oy) {
  LRec r;
  r.m = make_float4((a.x - ox) + a.z, (a.y - oy) + a.w, -0.5f * kLog2e * b.x, -kLog2e * b.y);
  r.c = make_float2(-0.5f * kLog2e * b.z, b.w);
  return r;
}

// Work items of a block whose waves do not meet at a barrier. Each wave takes the block's items in
// the same order; the first to need item j takes it from the launch's counter for all four, once
// they all hold item j - 1: a wave runs at most one item ahead of the slowest. Further ahead, the
// waves no longer find in the L1 cache what the others gathered from the same list.
struct BlockItems {
  uint32_t item, tag;           // the newest item and its number in the block's order + 1
  uint32_t claimed, taken[4];   // items claimed so far; items each wave has taken
};
__device__ __forceinline__ void items_init(BlockItems& b) {
  if (threadIdx.x < sizeof(b) / 4) reinterpret_cast<uint32_t*>(&b)[threadIdx.x] = 0u;
  __syncthreads();
}
__device__ __forceinline__ uint32_t lds_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Item j of the block, in every lane of wave `wave`. The waits end: one is for waves that have not
// taken item j - 1 (they hold an earlier one and go on to take the next), the other for the wave
// that is fetching item j. A fetched item stays until this wave has taken it too. After the last
// item every wave sees the same first number past the work and stops there.
__device__ __forceinline__ uint32_t next_item(BlockItems& b, uint32_t* counter, int wave, uint32_t j) {
  uint32_t wi = 0;
  if ((threadIdx.x & 63) == 0) {
    uint32_t want = j;
    if (__hip_atomic_compare_exchange_strong(&b.claimed, &want, j + 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP)) {
      for (int w = 0; w < 4; ++w)
        while (lds_load(&b.taken[w]) < j) __builtin_amdgcn_s_sleep(1);
      wi = atomicAdd(counter, 1u);
      lds_store(&b.item, wi);
      lds_store(&b.tag, j + 1u);
    } else {
      while (lds_load(&b.tag) != j + 1u) __builtin_amdgcn_s_sleep(1);
      wi = lds_load(&b.item);
    }
    lds_store(&b.taken[wave], j + 1u);
  }
  return __builtin_amdgcn_readfirstlane(wi);
}

// Hides a value's origin: what is computed from the copy is not hoisted out of the loop over
// work items, where the many channel masks and addresses of an item's end would hold registers.
__device__ __forceinline__ int opaque(int x) { asm volatile("" : "+s"(x)); return x; }
__device__ __forceinline__ int opaque_v(int x) { asm volatile("" : "+v"(x)); return x; }

// Compositing. A block takes a work item, a whole tile list (SEG = false, one block per tile)
// or, SEG = true, a chunk of up to cfg.fwd_chunk segments of a list (persistent blocks, items
// from ctl[1]), starting from the product of the earlier chunks' P. Each of its waves then
// walks the list for its own 64 pixels, with nothing shared and no barrier:
//   64 entries at a time, a lane each, are tested against the wave's region (band_reaches);
//   the ones that can reach alpha_min in it (27-37 % of them) are appended to the wave's queue
//   in LDS, in list order. The next 64 entries' records are on their way meanwhile.
//   Every 32 queued Gaussians make a dense batch: their features are gathered, the 64 pixels'
//   recurrence runs over them (unrolled, weights in registers), and by then the features have
//   arrived: F^T goes to LDS and F W to the matrix cores. The weights reach the operand layout
//   by a block transpose across lane rows, not through LDS.
// A split list leaves each segment's colour, end T and blend record in its slot; when the list
// is one chunk, the block also joins its segments (image, T, n_contrib, suffix colours).
// What bounds it: on a full chip vector issue and the gathers at once (16 full-HD pyramids, embedding,
// segments of 4096: vector instructions issue in 82-83 % of the cycles, and 50 GB pass the fabric in
// 9.5 ms, 5.2 TB/s, the rate of a copy; a region's Gaussian costs a line each for colour, depth and
// features); with 64 channels the wait for gathers at two waves a SIMD (54-55 % issue); one wave's chain
// of batches (about 4000 cycles of recurrence each) where the longest list sets the time. It replaces a
// block that staged 32 list entries at a time for all four waves, with two barriers a batch and
// dense products over entries that mostly miss: 16 full-HD pyramids, embedding 30.7 -> 11.0 ms;
// eight 636x476 pyramids, 20 classes 3.43 -> 1.62 ms; 1200x680 pyramid, 52 classes
// 0.39 -> 0.20 ms; a 320x240 pyramid whose longest list has 2100 entries 0.26 -> 0.13 ms.
// Three waves a SIMD with 32 channels; two with 64, since at three the compiler spills (0.39
// against 0.21 ms: scratch traffic queues between the gathers).
constexpr int kQueue = 128;     // a batch's remainder (31), 64 entries and a last batch's filling (32)

template <int NS, bool SEG, int MODE>
__global__ __launch_bounds__(256, NS <= 28 ? 3 : 2) void k_render_fwd_split(
    gs_config cfg, FeatSrc src, const float* __restrict__ rec, int64_t n, const gs_item* __restrict__ items, int n_items,
    const uint32_t* __restrict__ vals, const uint32_t* __restrict__ ranges, float* __restrict__ color,
    float* __restrict__ Tout, uint32_t* __restrict__ ncout, const uint2* __restrict__ work, uint32_t* __restrict__ ctl,
    FState fs) {
  using S = SShape<NS>;
  constexpr bool EMB = MODE == kEmbVec;
  constexpr int CB = S::CB, KP = S::KP;
  __shared__ __align__(16) float s_queue[4][8 * kQueue];    // per wave: the record's six floats, list position, Gaussian
  __shared__ __align__(16) uint32_t s_ft[4][KP * kWs];      // per wave: F^T, packed hi|lo, [channel][Gaussian]
  __shared__ uint32_t s_wi;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int Kr = 4 + src.n_sem;
  const int tws = tile_shift(cfg);
  const Region rg = wave_region(tws, wave, lane);
  const float amin = cfg.alpha_min, amax = cfg.alpha_max, tmin = cfg.t_min;
  const uint32_t n_work = SEG ? ctl[0] : 1u;
  float* const Q = s_queue[wave];
  uint32_t* const FT = s_ft[wave];
  if constexpr (EMB)   // the channels past the embedding's
    for (int i = lane; i < (KP - 20) * kWs; i += 64) FT[20 * kWs + i] = 0u;
  for (uint32_t round = 0;; ++round) {
    uint32_t wi = 0;
    int tile, seg = 0, nseg = 1;
    if constexpr (SEG) {
      if (tid == 0) s_wi = atomicAdd(&ctl[1], 1u);
      lds_barrier();
      wi = __builtin_amdgcn_readfirstlane(s_wi);   // the same in every lane: scalar registers
      lds_barrier();
      if (wi >= n_work) break;
      const uint2 wk = work[wi];
      tile = (int)__builtin_amdgcn_readfirstlane(wk.x);
      const uint32_t sg2 = __builtin_amdgcn_readfirstlane(wk.y);
      seg = (int)(sg2 & 0xffffu);
      nseg = (int)(sg2 >> 16);
      if (seg % fwd_chunk(cfg) != 0) continue;   // inside a chunk walked by another item
    } else {
      if (round > 0) break;
      tile = cfg.tile_order ? (int)blockIdx.x : (int)gridDim.x - 1 - (int)blockIdx.x;
    }
    const Ctx c = make_ctx_of(items, n_items, ranges, tile, tws);
    const int64_t foff = feature_offset(cfg, c.view, n), e0 = (int64_t)c.item * n;
    int u, v;
    tile_pixel(c, rg.px, u, v);
    const bool inside = u < c.W && v < c.H;
    const float ox = (float)tile_mid_x(c) + 0.5f, oy = (float)tile_mid_y(c) + 0.5f;
    const bool split = SEG && nseg > 1;
    const int chunk = fwd_chunk(cfg), seglen = seg_len(cfg);
    const int s_hi = split ? min(nseg, seg + chunk) : 1;   // segments [seg, s_hi) of this item
    const int64_t slot0 = (int64_t)wi - seg;                  // the tile's first slot
    v4f acc[CB][4];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) acc[cb][pb] = zero4();
    float T = 1.0f;
    if (split)
      for (int s2 = 0; s2 < seg; s2 += chunk) T *= fs.P[(slot0 + s2) * kTilePx + rg.px];
    // a pixel whose transmittance in front of the chunk is below t_min stopped earlier
    float Tw = (inside & (T >= tmin)) ? T : 0.0f;
    auto alive = [&]() { return Tw >= tmin; };
    uint32_t last = 0;

    // composites the cnt (1..32) queued Gaussians from position o of the queue on
    auto batch = [&](int o, int cnt) {
      const float* R0 = Q + 8 * o;
      Feats<NS, MODE> ft;
      ft.load(src, R0, foff, e0, lane);
      // front-to-back recurrence, branch-free; only Tw carries from one Gaussian to the next:
      // T while the pixel is active, 0 once it has stopped (so that it takes nothing more); `at`
      // is the batch position + 1 of the last Gaussian taken. The records of the next two
      // Gaussians are read while two are used.
      constexpr int kG = KP > 32 || EMB ? 4 : 2;
      float w[kB];
      int at = 0;
      auto half = [&](auto q0_) {
        constexpr int q0 = decltype(q0_)::value;
        LRec A[kG], B[kG];
#pragma unroll
        for (int e = 0; e < kG; ++e) A[e] = load_rec(R0, q0 + e);
#pragma unroll
        for (int q = q0; q < q0 + 16; q += kG) {
          if (q + kG < q0 + 16)
#pragma unroll
            for (int e = 0; e < kG; ++e) B[e] = load_rec(R0, q + kG + e);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int e = 0; e < kG; ++e) {
            float dx, dy, t;
            const float araw = A[e].c.y * __builtin_amdgcn_exp2f(local_power2(rg.lx, rg.ly, A[e], dx, dy, t));
            const bool ok = araw >= amin;
            const float wq = (ok ? fminf(amax, araw) : 0.0f) * Tw;
            const float Tn = Tw - wq;
            const bool low = Tn < tmin;
            w[q + e] = low ? 0.0f : wq;
            T = low ? T : Tn;
            Tw = low ? 0.0f : Tn;
            at = (ok & !low) ? q + e + 1 : at;
          }
#pragma unroll
          for (int e = 0; e < kG; ++e) A[e] = B[e];
        }
      };
      half(std::integral_constant<int, 0>());
      if (cnt > 16) {
        half(std::integral_constant<int, 16>());
      } else {
#pragma unroll
        for (int q = 16; q < kB; ++q) w[q] = 0.0f;
      }
      if (at > 0) last = __float_as_uint(R0[8 * at - 2]);
      wave_sync();   // the previous batch's reads of F^T come first
      ft.commit(FT, src.n_sem, cnt, lane);
      // W^T operands: X[g] = this pixel's weights of Gaussians 8 g .. 8 g + 7, hi then lo parts; the
      // transpose leaves lane (row g4, l16) with the weights 8 g4 + 0..7 of pixel 16 pb + l16 in X[pb]
      uint32_t X[4][8];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        v8bf hi, lo;
        split8(w + 8 * g, hi, lo);
        const uint4 h = __builtin_bit_cast(uint4, hi), l = __builtin_bit_cast(uint4, lo);
        X[g][0] = h.x; X[g][1] = h.y; X[g][2] = h.z; X[g][3] = h.w;
        X[g][4] = l.x; X[g][5] = l.y; X[g][6] = l.z; X[g][7] = l.w;
      }
      block_transpose(X);
      wave_sync();
      // out^T[c][p] += F^T[c][i] W^T[i][p]: A = F^T (i = channel 16 cb + l16, k = Gaussian 8 g4 + e),
      // B = W^T (k = Gaussian, j = pixel 16 pb + l16)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        v8bf ah, al;
        load_op(FT + (16 * cb + l16) * kWs + 8 * g4, ah, al);
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
          const v8bf bh = __builtin_bit_cast(v8bf, make_uint4(X[pb][0], X[pb][1], X[pb][2], X[pb][3]));
          const v8bf bl = __builtin_bit_cast(v8bf, make_uint4(X[pb][4], X[pb][5], X[pb][6], X[pb][7]));
          if (EMB && cb > 0) acc[cb][pb] = mma(ah, bl, mma(ah, bh, acc[cb][pb]));   // bfloat16 values: no lo part
          else acc[cb][pb] = mma3(ah, al, bh, bl, acc[cb][pb]);
        }
      }
    };

    for (int sg = seg; sg < s_hi; ++sg) {
      const uint32_t a0 = split ? c.start + sg * seglen : c.start;
      const uint32_t b0 = split ? min(c.end, a0 + seglen) : c.end;
      const bool active = alive();
      if (__ballot(alive()) != 0ull && a0 < b0) {
        // this lane's entry of the 64 at hand (ra, rb: its record) and the next 64 entries' ids
        // (every lane loads, past the last entry that entry again: no wait at a branch's end)
        auto load_id = [&](uint32_t b) -> uint32_t { return vals[min(b + lane, b0 - 1u)]; };
        auto load_half = [&](uint32_t g, int part) -> float4 {
          return reinterpret_cast<const float4*>(rec + kRecFloats * (e0 + g))[part];
        };
        uint32_t gid = load_id(a0);
        uint32_t gnext = load_id(a0 + 64);
        float4 ra = load_half(gid, 0), rb = load_half(gid, 1);
        int qn = 0;   // queued Gaussians
        for (uint32_t b = a0;; b += 64) {
          const LRec r = local_rec(ra, rb, ox, oy);
          const bool hit = b + lane < b0 && band_reaches(r, rg.x0, rg.x1, rg.y0, rg.y1, amin);
          const uint64_t m = __ballot(hit);
          if (hit) {
            const int at = qn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            float4* d = reinterpret_cast<float4*>(Q + 8 * at);
            d[0] = r.m;
            d[1] = make_float4(r.c.x, r.c.y, __uint_as_float(b + lane + 1 - c.start), __uint_as_float(gid));
          }
          qn += __builtin_popcountll(m);
          const bool more = b + 64 < b0;   // else the remainder is composited too
          gid = gnext;
          ra = load_half(gid, 0);
          rb = load_half(gid, 1);
          gnext = load_id(b + 128);
          // a last batch's missing entries: a negative opacity, so no alpha reaches the threshold
          if (!more) reinterpret_cast<float4*>(Q + 8 * qn)[lane] = make_float4(0.f, (lane & 1) ? -1.f : 0.f, 0.f, 0.f);
          wave_sync();
          int o = 0;
          while (qn - o >= (more ? kB : 1) && __ballot(alive()) != 0ull) {
            batch(o, min(kB, qn - o));
            o += kB;
          }
          if (!more || __ballot(alive()) == 0ull) break;
          if (o > 0 && qn > o) {   // the remainder (at most 31) moves to the front
            const float4* s4 = reinterpret_cast<const float4*>(Q + 8 * o);
            const float4 t = lane < 2 * (qn - o) ? s4[lane] : make_float4(0.f, 0.f, 0.f, 0.f);
            wave_sync();
            if (lane < 2 * (qn - o)) reinterpret_cast<float4*>(Q)[lane] = t;
          }
          qn -= o;
          wave_sync();
        }
        wave_sync();
      }
      if (split) {
        // the segment's slot; D[c][p]: lane holds pixel 16 pb + l16 of this wave, channels
        // 16 cb + 4 g4 + r
        const int64_t sl = slot0 + sg;
        const int K2 = opaque(Kr), la = opaque_v(lane), li = la & 15, gi = 4 * (la >> 4);
        float* dst = fs.CS + sl * K2 * kTilePx;
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
          const int px = wave_region(tws, wave, 16 * pb + li).px;
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int ch = 16 * cb + gi + r;
              if (ch < K2) dst[ch * kTilePx + px] = acc[cb][pb][r];
              acc[cb][pb][r] = 0.0f;
            }
        }
        const int64_t o = sl * kTilePx + rg.px;
        fs.Te[o] = T;
        const uint32_t lseg = last > (uint32_t)(sg * seglen) ? last : 0u;
        fs.info[o] = lseg | (active ? kInfoActive : 0u) | ((active && !alive()) ? kInfoStopped : 0u);
      }
    }
    if (split && nseg > chunk) continue;   // joined by k_fwd_combine
    const int64_t pix = c.pixel_base + (int64_t)v * c.W + u;
    if (inside) {
      Tout[pix] = T;
      ncout[pix] = last;
    }
    // D[c][p] (the image), or for a split list the sum of its segments' colours taken back
    // to front, each slot left holding the sum of the ones after it (acc, zero after the
    // last flush, carries the running sum; every value read here was written by this lane)
    const int K2 = opaque(Kr), la = opaque_v(lane), li = la & 15, gi = 4 * (la >> 4);
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
      const int px = wave_region(tws, wave, 16 * pb + li).px;
      if (split) {
        float* p = fs.CS + slot0 * K2 * kTilePx + px;
        for (int s2 = nseg - 1; s2 >= 0; --s2) {
          float* ps = p + (int64_t)s2 * K2 * kTilePx;
          float cs[CB][4];
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int ch = 16 * cb + gi + r;
              cs[cb][r] = ch < K2 ? ps[ch * kTilePx] : 0.0f;
            }
#pragma unroll
          for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int ch = 16 * cb + gi + r;
              if (ch < K2) ps[ch * kTilePx] = acc[cb][pb][r];
              acc[cb][pb][r] += cs[cb][r];
            }
        }
      }
      int pu, pv;
      tile_pixel(c, px, pu, pv);
      if (pu >= c.W || pv >= c.H) continue;
      const int64_t pbase = c.pixel_base * K2 + (int64_t)pv * c.W + pu;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ch = 16 * cb + gi + r;
          if (ch < K2) color[pbase + ch * c.HW] = acc[cb][pb][r];
        }
    }
  }
}

// Joins the segments of every list longer than one chunk: a pixel takes its segments in
// order up to the one in which it stopped (a later chunk that still found it active, its
// starting product being rounded differently from the stopping chain, is dropped); the
// image gets their colour sum, T and n_contrib, and each segment's colour is replaced by
// the sum of the colours of the kept segments after it. Segments are walked back to
// front with all channels of a segment loaded at once.
template <int NS>
__global__ __launch_bounds__(256) void k_fwd_combine(const gs_item* __restrict__ items, int n_items,
                                                     const uint32_t* __restrict__ ranges, int Kr, int chunk, int tws,
                                                     FState fs, float* __restrict__ color, float* __restrict__ Tout,
                                                     uint32_t* __restrict__ ncout) {
  constexpr int KP = SShape<NS>::KP;
  const int tile = blockIdx.x, tid = threadIdx.x;
  const int nseg = (int)fs.tcnt[tile];
  if (nseg <= chunk) return;
  const Ctx c = make_ctx_of(items, n_items, ranges, tile, tws);
  int u, v;
  tile_pixel(c, tid, u, v);
  if (u >= c.W || v >= c.H) return;
  const int64_t b = fs.tbase[tile];
  float T = 1.0f;
  uint32_t last = 0;
  int s_end = nseg;
  for (int s = 0; s < nseg; ++s) {
    const int64_t o = (b + s) * kTilePx + tid;
    const uint32_t inf = fs.info[o];
    if (!(inf & kInfoActive)) break;
    T = fs.Te[o];
    if (inf & kInfoLast) last = inf & kInfoLast;
    if (inf & kInfoStopped) {
      s_end = s + 1;
      break;
    }
  }
  const int64_t pix = c.pixel_base + (int64_t)v * c.W + u;
  Tout[pix] = T;
  ncout[pix] = last;
  float sum[KP];
#pragma unroll
  for (int k = 0; k < KP; ++k) sum[k] = 0.0f;
  for (int s = nseg - 1; s >= 0; --s) {
    float* p = fs.CS + (b + s) * Kr * kTilePx + tid;
    float cs[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) cs[k] = (k < Kr && s < s_end) ? p[k * kTilePx] : 0.0f;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      if (k < Kr) p[k * kTilePx] = sum[k];
      sum[k] += cs[k];
    }
  }
  float* out = color + c.pixel_base * Kr + (int64_t)v * c.W + u;
#pragma unroll
  for (int k = 0; k < KP; ++k)
    if (k < Kr) out[k * c.HW] = sum[k];
}

// ------------------------------------------------------------------------- backward
// Walking a segment of a split list backwards needs, per pixel, the transmittance after
// it and the suffix sum over every later Gaussian of w (g . f). Without the forward's
// saved state, a summary pass gives every segment s of a long list, per pixel,
//   P_s  = prod over its blended Gaussians of (1 - alpha)            (front to back)
//   GC_s = sum over its blended Gaussians of alpha T_loc (g . f),     T_loc from 1
// and then T_after(s) = prod_{s' <= s} P_s' and suffix(s) = sum_{s' > s} T_before(s') GC_s'.
// With the exponent E = a dx^2 + b dx dy + c dy^2 of the local record (E = log2(e) power),
// d power/d mean2d = -(dE/d dx, dE/d dy) / log2(e) and d power/d(A, B, C) =
// -(dx^2 / 2, dx dy, dy^2 / 2); the reverse pass sums dE/d dx, dE/d dy, dx^2, dx dy, dy^2
// (times dL/d power) and applies these factors once per Gaussian.
// The geometric sums of a group from D[Gaussian][pixel of the wave] = dL/d power: lane (g4, l16)
// takes Gaussian l16's pixels 32 ks + 8 g4 + e, two runs of eight along x, so that dy is one value a
// run and three sums over it (of D, D dx, D dx^2) give all six terms; the four lane rows' parts
// are then added with values halved at each step (permlane32 pairs rows (0, 2) and (1, 3), permlane16
// rows (0, 1) and (2, 3)). The opacity's sum is that of D over the opacity
// (an opacity of 0, which alpha_min = 0 lets through, has no gradient: its logit's is o (1 - o) times
// it). The mean's two terms are combined after the sums, 2a S(D dx) + b S(D dy), where a thin oblique
// footprint's two parts cancel as sums and not pixel by pixel. (Six terms for each pixel's
// lane and their sums over 64 lanes were a quarter of the reverse pass's instructions.)
// (x, y): position of the lane's first pixel; ys: rows from its first run to its second.
__device__ __forceinline__ void geo_sums(const float* D, const float* R, float x, float y, float ys, int l16, int g4,
                                         float& Y0, float& Y1) {
  const LRec q = load_rec(R, l16);
  float dx[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) dx[e] = (x + (float)e) - q.m.x;
  float s00 = 0.0f, s10 = 0.0f, s20 = 0.0f, s01 = 0.0f, s11 = 0.0f, s02 = 0.0f;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const float* d8 = D + l16 * kPs + 32 * ks + 8 * g4;
    const float4 d0 = *reinterpret_cast<const float4*>(d8), d1 = *reinterpret_cast<const float4*>(d8 + 4);
    const float d[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
    float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = d[e] * dx[e];
      a += d[e];
      b += t;
      c = __builtin_fmaf(t, dx[e], c);
    }
    const float dy = (y + (ks ? ys : 0.0f)) - q.m.y;
    s00 += a;
    s10 += b;
    s20 += c;
    const float t = a * dy;
    s01 += t;
    s11 = __builtin_fmaf(b, dy, s11);
    s02 = __builtin_fmaf(t, dy, s02);
  }
  // sums of D times dE/d dx = 2a dx + b dy, dE/d dy = b dx + 2c dy, dx^2, dx dy, dy^2, 1 / opacity
  const float V[6] = {__builtin_fmaf(2.0f * q.m.z, s10, q.m.w * s01), __builtin_fmaf(q.m.w, s10, 2.0f * (q.c.x * s01)),
                      s20, s11, s02, q.c.y > 1e-30f ? s00 * __builtin_amdgcn_rcpf(q.c.y) : 0.0f};
  float W[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(V[j]), __float_as_uint(V[j + 3]), false, false);
    W[j] = __uint_as_float(t[0]) + __uint_as_float(t[1]);
  }
  // lane row g4: Y0 is term 0, 1, 3, 4; Y1 term 2, 2, 5, 5
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(W[0]), __float_as_uint(W[1]), false, false);
  Y0 = __uint_as_float(t[0]) + __uint_as_float(t[1]);
  const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(W[2]), __float_as_uint(W[2]), false, false);
  Y1 = __uint_as_float(u[0]) + __uint_as_float(u[1]);
}

__constant__ float kGeoScale[6] = {-1.0f / kLog2e, -1.0f / kLog2e, -0.5f, -1.0f, -0.5f, 1.0f};

// One wave per tile: the tile's list length in use (largest n_contrib) and its segment
// count, stored in work order (coarse pyramid levels first unless tile_order = 1).
// With a forward state, a tile that the forward did not split stays one item.
// (A block per tile spent its time being launched: 174k tiles 540 us, now 93; 4270 tiles 16, now 5.)
__global__ __launch_bounds__(256) void k_seg_count(const gs_item* __restrict__ items, int n_items,
                                                   const uint32_t* __restrict__ ranges,
                                                   const uint32_t* __restrict__ ncin, int n_tiles, int order, int tws,
                                                   uint32_t seg, const uint32_t* __restrict__ ftcnt,
                                                   uint32_t* __restrict__ tile_lmax, uint32_t* __restrict__ cnt_ord) {
  const int lane = threadIdx.x & 63;
  const int tile = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (tile >= n_tiles) return;
  const int item = item_of_tile(items, n_items, tile);
  const gs_item it = items[item];
  const int lt = tile - it.tile_base;
  const int u0 = (lt % it.tiles_x) << tws, v0 = (lt / it.tiles_x) * (kTilePx >> tws);
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < kTilePx / 64; ++j) {
    const int t = 64 * j + lane, u = u0 + (t & ((1 << tws) - 1)), v = v0 + (t >> tws);
    const uint32_t c = ncin[it.pixel_base + (int64_t)min(v, it.H - 1) * it.W + min(u, it.W - 1)];
    m = u < it.W && v < it.H ? max(m, c) : m;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if (lane == 0) {
    m = min(m, ranges[2 * (int64_t)tile + 1] - ranges[2 * (int64_t)tile]);
    tile_lmax[tile] = m;
    const bool one = m <= seg || (ftcnt && ftcnt[tile] < 2);
    cnt_ord[order ? tile : n_tiles - 1 - tile] = m == 0 ? 0u : (one ? 1u : (m + seg - 1) / seg);
  }
}

// Work list: (tile, segment | segment count << 16). If the segments do not fit the
// workspace, every tile becomes a single item. Also resets the two work counters and,
// if tcnt is given, records per tile its item count and first item.
__global__ void k_seg_list(const uint32_t* __restrict__ cnt_ord, const uint32_t* __restrict__ base_ord,
                           const uint64_t* __restrict__ total, int n_tiles, int order, int64_t max_segs,
                           uint2* __restrict__ work, uint32_t* __restrict__ ctl, uint32_t* __restrict__ tcnt,
                           uint32_t* __restrict__ tbase) {
  const int o = blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t tot = *total;
  const bool fits = tot <= (uint64_t)max_segs;
  if (o == 0) {
    ctl[0] = fits ? (uint32_t)tot : (uint32_t)n_tiles;
    ctl[1] = 0;
    ctl[2] = 0;
  }
  if (o >= n_tiles) return;
  const uint32_t tile = order ? o : n_tiles - 1 - o;
  if (fits) {
    const uint32_t c = cnt_ord[o], b = base_ord[o];
    for (uint32_t k = 0; k < c; ++k) work[b + k] = make_uint2(tile, k | (c << 16));
    if (tcnt) {
      tcnt[tile] = c;
      tbase[tile] = b;
    }
  } else {
    work[o] = make_uint2(tile, 1u << 16);
    if (tcnt) {
      tcnt[tile] = 1;
      tbase[tile] = o;
    }
  }
}

// The summary pass over the segments of long lists, without a forward state: per segment and
// pixel, P and GC (above), front to back. Persistent blocks take work items from a counter.
template <int NS>
__global__ __launch_bounds__(256, 2) void k_seg_summary(gs_config cfg, const float* __restrict__ rgb,
                                                        const float* __restrict__ sem,
                                                        const uint16_t* __restrict__ emb, int n_sem,
                                                        const float* __restrict__ rec,
                                                        const float* __restrict__ depth, int64_t n,
                                                        const gs_item* __restrict__ items, int n_items,
                                                        const uint32_t* __restrict__ vals,
                                                        const uint32_t* __restrict__ ranges,
                                                        const uint32_t* __restrict__ ncin,
                                                        const float* __restrict__ gcolor,
                                                        const uint2* __restrict__ work, uint32_t* __restrict__ ctl,
                                                        const uint32_t* __restrict__ tile_lmax,
                                                        float* __restrict__ segP, float* __restrict__ segGC) {
  using S = SShape<NS>;
  constexpr int KP = S::KP, FST = S::FST;
  __shared__ __align__(16) float s_rec[8 * kB];
  __shared__ __align__(16) float s_f[kB * FST];             // F, [Gaussian][channel]
  __shared__ uint32_t s_wi;
  __shared__ uint32_t s_gid[kB];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int Kr = 4 + n_sem;
  const float amin = cfg.alpha_min, amax = cfg.alpha_max;
  const uint32_t n_work = ctl[0];
  for (;;) {
    if (tid == 0) s_wi = atomicAdd(&ctl[1], 1u);
    lds_barrier();
    const uint32_t wi = s_wi;
    lds_barrier();
    if (wi >= n_work) break;
    const uint2 wk = work[wi];
    const int tile = (int)wk.x;
    const int seg = (int)(wk.y & 0xffffu), nseg = (int)(wk.y >> 16);
    if (nseg < 2) continue;
    const Ctx c = make_ctx_of(items, n_items, ranges, tile, tile_shift(cfg));
    const int64_t foff = feature_offset(cfg, c.view, n);
    int u, v;
    tile_pixel(c, tid, u, v);
    const bool inside = u < c.W && v < c.H;
    const float lx = (float)((tid & ((1 << c.tws) - 1)) - (1 << (c.tws - 1))), ly = (float)((tid >> c.tws) - (128 >> c.tws));
    const float ox = (float)tile_mid_x(c) + 0.5f, oy = (float)tile_mid_y(c) + 0.5f;
    const int64_t pix = c.pixel_base + (int64_t)v * c.W + u;
    // n_contrib comes from the matching forward; clamp so that a mismatched call stays in range
    const uint32_t last = inside ? min(ncin[pix], c.end - c.start) : 0u;
    const int lmax = (int)tile_lmax[tile];
    const int seglen = seg_len(cfg);
    const int a0 = seg * seglen, b0 = min(lmax, a0 + seglen);
    // upstream gradient of a wave pixel (0..63) and channel, zero outside the image
    auto gval = [&](int wp, int ch) -> float {
      int pu, pv;
      tile_pixel(c, wave * 64 + wp, pu, pv);
      if (pu >= c.W || pv >= c.H || ch >= Kr) return 0.0f;
      return gcolor[c.pixel_base * Kr + (int64_t)pv * c.W + pu + ch * c.HW];
    };
    // G^T as B of GF (k = channel 4 ks + g4, j = pixel 16 pb + l16)
    float g1[4][KP / 4];
#pragma unroll
    for (int pb = 0; pb < 4; ++pb)
#pragma unroll
      for (int ks = 0; ks < KP / 4; ++ks) g1[pb][ks] = gval(16 * pb + l16, 4 * ks + g4);
    float T = 1.0f, acc = 0.0f;
    SStage<NS> st;
    if (a0 < b0) {
      st.fetch(vals, c.start + a0, min(kB, b0 - a0), c.item, n, rec, depth, rgb, sem, emb, n_sem, foff);
      if (a0 + kB < b0) st.load_ids(vals, c.start + a0 + kB, min(kB, b0 - a0 - kB));
    }
    for (int lo = a0; lo < b0; lo += kB) {
      const int cnt = min(kB, b0 - lo);
      lds_barrier();
      st.commit_rows(s_rec, s_f, s_gid, ox, oy);
      lds_barrier();
      if (lo + kB < b0) {
        st.fetch_data(min(kB, b0 - lo - kB), c.item, n, rec, depth, rgb, sem, emb, n_sem, foff);
        if (lo + 2 * kB < b0) st.load_ids(vals, c.start + lo + 2 * kB, min(kB, b0 - lo - 2 * kB));
      }
      if (__ballot((uint32_t)lo < last) == 0ull) continue;
      // GF^T[i][p] in single precision: v_mfma_f32_16x16x4_f32, A = F (i = Gaussian 16 bq + l16,
      // k = channel 4 ks + g4), B = G^T; lane row g4 holds Gaussians {4 g4 + r, 16 + 4 g4 + r} of all
      // four pixel rows, and after the transpose every lane its own pixel's values:
      // X[g][4 bq + r] = gf of Gaussian 16 bq + 4 g + r
      uint32_t X[4][8];
      v4f gfa[4][2];
#pragma unroll
      for (int pb = 0; pb < 4; ++pb) gfa[pb][0] = gfa[pb][1] = zero4();
#pragma unroll
      for (int bq = 0; bq < 2; ++bq)
#pragma unroll
        for (int ks = 0; ks < KP / 4; ++ks) {
          const float a = s_f[(16 * bq + l16) * FST + 4 * ks + g4];
#pragma unroll
          for (int pb = 0; pb < 4; ++pb)
            gfa[pb][bq] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, g1[pb][ks], gfa[pb][bq], 0, 0, 0);
        }
#pragma unroll
      for (int pb = 0; pb < 4; ++pb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          X[pb][r] = __float_as_uint(gfa[pb][0][r]);
          X[pb][4 + r] = __float_as_uint(gfa[pb][1][r]);
        }
      block_transpose(X);
#pragma unroll
      for (int q = 0; q < kB; ++q) {
        const LRec rq = load_rec(s_rec, q);
        float dx, dy, t;
        const float araw = rq.c.y * __builtin_amdgcn_exp2f(local_power2(lx, ly, rq, dx, dy, t));
        const bool act = (q < cnt) & ((uint32_t)(lo + q) < last) & (araw >= amin);
        const float w = fminf(amax, araw) * T;
        const float gf = __uint_as_float(X[(q >> 2) & 3][4 * (q >> 4) + (q & 3)]);
        acc = act ? __builtin_fmaf(w, gf, acc) : acc;
        T = act ? T - w : T;
      }
    }
    segP[(int64_t)wi * kTilePx + tid] = T;
    segGC[(int64_t)wi * kTilePx + tid] = acc;
  }
}

// ------------------------------------------------------------------------- backward, main pass
// Where the reverse pass's per-Gaussian sums go from LDS: the n_sem semantic channels and rgb in
// single precision, the record's seven components (kGradRec) in double precision. A wave adds its
// own sums, so a feature gradient is rounded some four times as often as when a block added them
// (error of all outputs against 64 bits, eight 636x476 pyramids 6.08e-6 -> 6.19e-6, a 640x480 frame
// 1.41e-6 -> 1.74e-6; two runs of one build differ by as much).
struct GradDst {
  float *grgb, *gsem;
  double* g2d;
};

// The reverse pass over one work item (a whole tile list, or one segment of it), back to front.
// Persistent blocks take work items from a counter; each wave then walks the list for its own 64
// pixels, with nothing shared and no barrier:
//   64 entries at a time, a lane each, are tested against the wave's region, from the last entry
//   that its forward used; the ones that can reach alpha_min there (27-37 %) go to the wave's ring
//   in LDS, back to front.
//   Every 16 of them make a dense group: g . f on the matrix cores, the reverse recurrence, the
//   geometric sums, dF on the matrix cores, all over Gaussians that these pixels can see.
//   A group's features are gathered while the one before is worked on, and its sums leave for
//   memory before the gather after it is issued: loads and atomics complete in order, so neither
//   is waited for until a whole group's work has passed.
// Memory takes 21 G atomic requests a second of up to 64 bytes each, however few bytes they carry
// (measured), so a group's sums go out with the lanes of a Gaussian side by side: a record's seven
// components or an embedding's row (64 bytes) are one request each.
// It replaces a block that staged 32 entries at a time for its four waves and met at two barriers a
// batch: 16 full-HD pyramids, embedding 70.3 -> 24.2 ms; eight 636x476 pyramids, 20 classes
// 6.44 -> 2.61 ms; a 1200x680 pyramid, 52 classes 1.04 -> 0.44 ms; a 320x240 pyramid 0.28 -> 0.13 ms
// (29.7, 3.14, 0.52 and 0.14 ms with a barrier per work item, sums read one by one as they go out
// and records in single precision; 27.0, 2.90, 0.48 and 0.14 with the geometric sums by pixel).
// Windows of 64 entries shared by the four waves, their sums meeting in LDS (half the atomic
// requests), took 45.9 ms and 0.88 ms on the first and third: 28 % of the cycles were waves waiting
// for the one with most entries in the window. On the first (segments of 4096), vector instructions
// now issue in 58 % of the cycles, at the two waves per SIMD that the registers allow, and 80 GB pass
// the fabric, 3.8 TB/s: regions gather and add for themselves, 42 % more than the block's 56 GB. With
// 64 channels (256 registers) they issue in 36-37 %.
constexpr int kGrp = 16, kRing = 128;   // ring: a part group (15), two groups in work, 64 new entries

template <int NS>
struct BShape {
  static constexpr int KP = SShape<NS>::KP;
  static constexpr bool kGF3 = KP == 32;                       // g . f in three bfloat16 parts
  static constexpr int FROW = kGF3 ? 3 * 16 + 4 : KP + 4;      // dwords of a feature row: 3 parts of 32 bf16, or floats
  static constexpr int AROW = KP + 8;                          // floats of a sum row: channels, then 6 geometric sums
  static constexpr int kQ = 8 * kRing, kW = kGrp * kPs, kF = kGrp * FROW, kA = kGrp * AROW;
  // dL/d power of a group [Gaussian][pixel]: with 64 channels in the features' place, which the
  // products have read by then
  static constexpr int kD = KP > 32 ? 0 : kGrp * kPs;
  static_assert(kD > 0 || kF >= kGrp * kPs, "the features' rows hold dL/d power");
  static constexpr int kStage = 32 * kPs;                      // upstream gradient staging at an item's start
  static constexpr int kSum = kQ + kW + kF + kA + kD, kWave = kSum > kStage ? kSum : kStage;
};

template <int NS, int MODE>
__global__ __launch_bounds__(256, 2) void k_render_bwd_main(
    gs_config cfg, FeatSrc src, const float* __restrict__ rec, int64_t n, const gs_item* __restrict__ items, int n_items,
    const uint32_t* __restrict__ vals, const uint32_t* __restrict__ ranges, const float* __restrict__ Tfin,
    const uint32_t* __restrict__ ncin, const float* __restrict__ gcolor, GradDst out, const uint2* __restrict__ work,
    uint32_t* __restrict__ ctl, const float* __restrict__ segP, const float* __restrict__ segGC, FState fs) {
  using B = BShape<NS>;
  constexpr bool EMB = MODE == kEmbVec;
  constexpr int KP = SShape<NS>::KP, CB = SShape<NS>::CB, FROW = B::FROW, AROW = B::AROW;
  constexpr bool kGF3 = B::kGF3;
  __shared__ __align__(16) float s_mem[4][B::kWave];
  __shared__ BlockItems s_items;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l16 = lane & 15, g4 = lane >> 4;
  const int Kr = 4 + src.n_sem;
  const int tws = tile_shift(cfg);
  const float amin = cfg.alpha_min, amax = cfg.alpha_max;
  const uint32_t n_work = ctl[0];
  // the wave's memory: ring of records {mx, my, a, b, c, o, list position, Gaussian}, W of a group
  // [Gaussian][pixel], features [Gaussian][channel], sums [Gaussian][channel, geometric]
  float* const Q = s_mem[wave];
  float* const W = Q + B::kQ;
  float* const F = W + B::kW;
  float* const A = F + B::kF;
  float* const D = B::kD ? A + B::kA : F;
  const Region rg = wave_region(tws, wave, lane);
  // the lane's two runs of eight pixels in geo_sums
  const bool wide = tws == 6;   // a region of 16x4 pixels
  const float gx = rg.x0 + (wide ? (float)(8 * (g4 & 1)) : 0.0f), gy = rg.y0 + (float)(wide ? g4 >> 1 : g4);
  items_init(s_items);
  for (uint32_t round = 0;; ++round) {
    const uint32_t wi = next_item(s_items, &ctl[2], wave, round);
    if (wi >= n_work) break;
    const uint2 wk = work[wi];
    const int tile = (int)__builtin_amdgcn_readfirstlane(wk.x);
    const uint32_t sg = __builtin_amdgcn_readfirstlane(wk.y);
    const int seg = (int)(sg & 0xffffu), nseg = (int)(sg >> 16);
    const Ctx c = make_ctx_of(items, n_items, ranges, tile, tws);
    const int64_t foff = feature_offset(cfg, c.view, n), e0 = (int64_t)c.item * n;
    int u, v;
    tile_pixel(c, rg.px, u, v);
    const bool inside = u < c.W && v < c.H;
    const float ox = (float)tile_mid_x(c) + 0.5f, oy = (float)tile_mid_y(c) + 0.5f;
    const int64_t pix = c.pixel_base + (int64_t)v * c.W + u;
    // n_contrib comes from the matching forward; clamp so that a mismatched call stays in range
    const uint32_t len = c.end - c.start;
    const uint32_t last = inside ? min(ncin[pix], len) : 0u;
    const int seglen = seg_len(cfg);
    const int a0 = nseg == 1 ? 0 : seg * seglen;
    // the last entry that one of the wave's pixels used
    uint32_t wl = last;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) wl = max(wl, (uint32_t)__shfl_xor((int)wl, off, 64));
    wl = __builtin_amdgcn_readfirstlane(wl);
    const int b0 = nseg == 1 ? (int)wl : min((int)wl, a0 + seglen);
    if (a0 >= b0) continue;   // (the same for the whole wave)

    // Upstream gradient of the wave's 64 pixels in two operand layouts, through LDS 32 channels
    // at a time: B of g . f (k = channel, j = pixel 16 pb + l16), with 32 padded channels in three
    // bfloat16 parts (single-precision products at a sixth of the 16x16x4 products' time), else
    // in single precision; B of dF (k = pixel 32 ks + 8 g4 + e, j = channel 16 cb + l16). The
    // lane's own pixel's values also give the forward state's dot product.
    float g1[4][kGF3 ? 1 : KP / 4];
    v8bf g3[kGF3 ? 4 : 1][3];
    v8bf g2h[2][CB], g2l[2][CB];
    float gdot = 0.0f;          // sum_k g_k S_k of the lane's pixel (forward state)
    {
      const bool use_state = nseg > 1 && fs.tcnt != nullptr && inside;
      const float* sc = use_state ? fs.CS + ((int64_t)fs.tbase[tile] + seg) * Kr * kTilePx + rg.px : nullptr;
      const float* gp = gcolor + c.pixel_base * Kr + (int64_t)v * c.W + u;   // this lane's pixel
      float* stg = Q;
#pragma unroll
      for (int h = 0; h < KP / 32; ++h) {
        const int K2 = opaque(Kr);
        float gl[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) gl[j] = (inside && 32 * h + j < K2) ? gp[(int64_t)(32 * h + j) * c.HW] : 0.0f;
        if (use_state) {
          // all 32 loads in flight where the registers allow it, else 8 at a time
          constexpr int kSv = KP <= 32 ? 32 : 8;
#pragma unroll
          for (int j0 = 0; j0 < 32; j0 += kSv) {
            float sv[kSv];
#pragma unroll
            for (int j = 0; j < kSv; ++j) sv[j] = 32 * h + j0 + j < K2 ? sc[(32 * h + j0 + j) * kTilePx] : 0.0f;
#pragma unroll
            for (int j = 0; j < kSv; ++j) gdot = __builtin_fmaf(gl[j0 + j], sv[j], gdot);
          }
        }
#pragma unroll
        for (int j = 0; j < 32; ++j) stg[j * kPs + lane] = gl[j];
        wave_sync();
        if constexpr (kGF3) {
#pragma unroll
          for (int pb = 0; pb < 4; ++pb) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = stg[(8 * g4 + e) * kPs + 16 * pb + l16];
            split8x3(x, g3[pb][0], g3[pb][1], g3[pb][2]);
          }
        } else {
#pragma unroll
          for (int ks = 8 * h; ks < 8 * h + 8; ++ks)
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) g1[pb][ks] = stg[(4 * ks + g4 - 32 * h) * kPs + 16 * pb + l16];
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int cb = 2 * h; cb < 2 * h + 2; ++cb) {
            const float* s8 = stg + (16 * cb + l16 - 32 * h) * kPs + 32 * ks + 8 * g4;
            const float4 x0 = *reinterpret_cast<const float4*>(s8), x1 = *reinterpret_cast<const float4*>(s8 + 4);
            const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            split8(x, g2h[ks][cb], g2l[ks][cb]);
          }
        wave_sync();   // every lane has read the stage before the next half overwrites it
      }
    }

    // per-pixel state at the segment's back end: T, and the suffix sum of w (g . f) behind it
    float T = 1.0f, acc = 0.0f;
    {
      const float tf = inside ? Tfin[pix] : 1.0f;
      if (nseg == 1 || seg == nseg - 1) T = tf;
      if (nseg > 1 && fs.tcnt) {
        // the forward's state: T at the segment's end and the suffix colour sum
        const int64_t slot = (int64_t)fs.tbase[tile] + seg, o = slot * kTilePx + rg.px;
        if (fs.info[o] & kInfoActive) T = fs.Te[o];
        acc = gdot;
      } else if (nseg > 1) {
        const int64_t w0 = (int64_t)wi - seg;
        float tb = 1.0f;   // transmittance in front of segment s
        for (int s = 0; s < nseg; ++s) {
          const float P = segP[(w0 + s) * kTilePx + rg.px], GC = segGC[(w0 + s) * kTilePx + rg.px];
          if (s > seg) acc = __builtin_fmaf(tb, GC, acc);
          tb *= P;
          if (s == seg && seg < nseg - 1) T = tb;
        }
      }
    }
    // A group's features on their way: four lanes a Gaussian for an embedding (8 bytes each) and
    // for colour and depth (a value each), QL lanes (a quad of channels each) for plain semantics.
    constexpr int QL = EMB ? 4 : KP / 4, NP = EMB ? 1 : QL / 4;
    float f[EMB ? 1 : 4 * NP], f0 = 0.0f;
    uint2 fe = make_uint2(0u, 0u);
    auto gather = [&](int grp) {
      const float* R = Q + 8 * kGrp * (grp & (kRing / kGrp - 1));
      uint32_t gq[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) gq[p] = __float_as_uint(R[8 * (p * (64 / QL) + lane / QL) + 7]);
      const uint32_t gc = __float_as_uint(R[8 * (lane >> 2) + 7]);
      const float* a0p = (lane & 3) < 3 ? src.rgb + 3 * ((int64_t)gc + foff) + (lane & 3) : src.depth + (e0 + gc);
      f0 = *a0p;
      if constexpr (EMB) fe = *reinterpret_cast<const uint2*>(src.emb + 16 * (uint64_t)gc + 4 * (lane & 3));
      else load_quads<MODE>(src, gq, foff, 4 * (lane % QL), f);
    };
    // the gathered features to their rows: three bfloat16 parts of each value, or the value. (A
    // part group's missing Gaussians have a row too, of whatever Gaussian 0 has; no sum uses it.)
    auto commit = [&]() {
      auto put4 = [&](int q, int k, const float (&x)[4]) {   // channels k .. k + 3 of Gaussian q
        if constexpr (kGF3) {
          uint32_t h[2], m[2], l[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){x[2 * i], x[2 * i + 1]}, bf2));
            const float r0 = x[2 * i] - __uint_as_float(h[i] << 16), r1 = x[2 * i + 1] - __uint_as_float(h[i] & 0xffff0000u);
            m[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){r0, r1}, bf2));
            l[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){r0 - __uint_as_float(m[i] << 16),
                                                                             r1 - __uint_as_float(m[i] & 0xffff0000u)}, bf2));
          }
          uint32_t* row = reinterpret_cast<uint32_t*>(F + q * FROW) + k / 2;
          *reinterpret_cast<uint2*>(row) = make_uint2(h[0], h[1]);
          *reinterpret_cast<uint2*>(row + 16) = make_uint2(m[0], m[1]);
          *reinterpret_cast<uint2*>(row + 32) = make_uint2(l[0], l[1]);
        } else {
          *reinterpret_cast<float4*>(F + q * FROW + k) = make_float4(x[0], x[1], x[2], x[3]);
        }
      };
      // the four lanes of a Gaussian put colour and depth together
      {
        const float x1 = dpp_xor1(f0), x2 = dpp_xor2(f0), x3 = dpp_xor2(x1);
        const float x[4] = {f0, x1, x2, x3};   // of the Gaussian's lane 0
        if ((lane & 3) == 0) put4(lane >> 2, 0, x);
      }
      if constexpr (EMB) {
        // bfloat16 values: the other parts are zero, and so are the channels past the embedding
        const int k = 4 + 4 * (lane & 3);
        uint32_t* row = reinterpret_cast<uint32_t*>(F + (lane >> 2) * FROW) + k / 2;
        const uint2 z = make_uint2(0u, 0u);
        *reinterpret_cast<uint2*>(row) = fe;
        *reinterpret_cast<uint2*>(row + 16) = z;
        *reinterpret_cast<uint2*>(row + 32) = z;
      } else {
        const int k = 4 * (lane % QL);
        const uint32_t m = k < src.n_sem ? ~0u : 0u;   // (see Feats::commit)
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          float x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(__float_as_uint(f[4 * p + i]) & m);
          if (k < NS) put4(p * (64 / QL) + lane / QL, 4 + k, x);
        }
      }
    };
    if constexpr (EMB) {   // channels 20 .. 31
      for (int i = lane; i < kGrp * 18; i += 64)
        reinterpret_cast<uint32_t*>(F)[(i / 18) * FROW + 10 + 16 * ((i % 18) / 6) + i % 6] = 0u;
    }

    // the sums of a finished group of cnt Gaussians to memory; L neighbouring lanes take the
    // values of one Gaussian
    auto flush = [&](int grp, int cnt) {
      const float* R = Q + 8 * kGrp * (grp & (kRing / kGrp - 1));
      const int n_sem = opaque(src.n_sem), total = n_sem + 10;
      const int ls = total <= 16 ? 4 : total <= 32 ? 5 : 6, L = 1 << ls;
      for (int o = lane & (L - 1); o < total; o += L) {
        char* base;
        int stride, col;
        const int k = o - n_sem - 3;   // the record's component, if any
        if (o < n_sem) {
          base = (char*)(out.gsem + n_sem * foff + o);
          stride = 4 * n_sem;
          col = 4 + o;
        } else if (k < 0) {
          base = (char*)(out.grgb + 3 * foff + (o - n_sem));
          stride = 12;
          col = o - n_sem;
        } else {
          base = (char*)(out.g2d + kGradRec * e0 + k);
          stride = 8 * kGradRec;
          col = k < 6 ? KP + k : 3;
        }
        const float scale = k >= 0 && k < 6 ? kGeoScale[k] : 1.0f;
        // eight Gaussians' values are read before the first goes out
        for (int e1 = lane >> ls; e1 < cnt; e1 += 512 >> ls) {
          float val[8];
          uint32_t g[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int e = min(e1 + i * (64 >> ls), kGrp - 1);
            val[i] = A[e * AROW + col];
            g[i] = __float_as_uint(R[8 * e + 7]);
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (e1 + i * (64 >> ls) < cnt && val[i] != 0.0f) {
              char* p = base + (int64_t)stride * g[i];
              if (k < 0) atomicAdd((float*)p, val[i]);
              else atomicAdd((double*)p, (double)(val[i] * scale));
            }
        }
      }
    };

    // this lane's entry of the 64 at hand (ra, rb: its record), list position hi - 1 - lane
    // (every lane loads, past the first entry that entry again: no wait at a branch's end)
    auto load_id = [&](int hi) -> uint32_t { return vals[c.start + max(hi - 1 - lane, a0)]; };
    auto load_half = [&](uint32_t g, int part) -> float4 {
      return reinterpret_cast<const float4*>(rec + kRecFloats * (e0 + g))[part];
    };
    uint32_t gid = load_id(b0);
    uint32_t gnext = load_id(b0 - 64);
    float4 ra = load_half(gid, 0), rb = load_half(gid, 1);
    int tail = 0, done = 0, issued = 0;   // entries in the ring so far; groups worked on, gathered
    for (int hi = b0;; hi -= 64) {
      {
        const LRec r = local_rec(ra, rb, ox, oy);
        const bool hit = hi - 1 - lane >= a0 && band_reaches(r, rg.x0, rg.x1, rg.y0, rg.y1, amin);
        const uint64_t m = __ballot(hit);
        if (hit) {
          const int at = tail + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          float4* d = reinterpret_cast<float4*>(Q + 8 * (at & (kRing - 1)));
          d[0] = r.m;
          d[1] = make_float4(r.c.x, r.c.y, __int_as_float(hi - 1 - lane), __uint_as_float(gid));
        }
        tail += __builtin_popcountll(m);
      }
      const bool fin = hi - 64 <= a0;
      gid = gnext;
      ra = load_half(gid, 0);
      rb = load_half(gid, 1);
      gnext = load_id(hi - 128);
      if (fin && lane < 2 * (-tail & (kGrp - 1))) {
        // a part group's missing entries: a negative opacity, so no alpha reaches the threshold
        reinterpret_cast<float4*>(Q + 8 * ((tail + (lane >> 1)) & (kRing - 1)))[lane & 1] =
            make_float4(0.f, (lane & 1) ? -1.f : 0.f, 0.f, 0.f);
      }
      wave_sync();
      const int ready = fin ? (tail + kGrp - 1) / kGrp : tail / kGrp;
      if (issued == done && ready > done) gather(issued++);
      while (issued > done && (fin || ready > done + 1)) {
        wave_sync();
        commit();
        if (done > 0) flush(done - 1, kGrp);
        if (ready > issued) gather(issued++);
        wave_sync();
        const float* R = Q + 8 * kGrp * (done & (kRing / kGrp - 1));
        // g . f: A = F (i = Gaussian l16 of the group, k = channel); D lane (row g4, l16): Gaussians
        // 4 g4 + r of pixel 16 pb + l16. The transpose gives every lane its own pixel's values:
        // Y4[qq / 4][qq % 4] = g . f of Gaussian qq of the group
        uint32_t Y4[4][4];
        {
          v4f gfa[4];
#pragma unroll
          for (int pb = 0; pb < 4; ++pb) gfa[pb] = zero4();
          if constexpr (kGF3) {
            v8bf fa[3];
#pragma unroll
            for (int part = 0; part < 3; ++part)
              fa[part] = *reinterpret_cast<const v8bf*>(F + l16 * FROW + 16 * part + 4 * g4);
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) gfa[pb] = mma6(fa, g3[pb], gfa[pb]);
          } else {
#pragma unroll
            for (int ks = 0; ks < KP / 4; ++ks) {
              const float a = F[l16 * FROW + 4 * ks + g4];
#pragma unroll
              for (int pb = 0; pb < 4; ++pb) gfa[pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, g1[pb][ks], gfa[pb], 0, 0, 0);
            }
          }
#pragma unroll
          for (int pb = 0; pb < 4; ++pb)
#pragma unroll
            for (int r = 0; r < 4; ++r) Y4[pb][r] = __float_as_uint(gfa[pb][r]);
        }
        block_transpose(Y4);
        // reverse recurrence over the group (T recovered with the hardware reciprocal)
#pragma unroll
        for (int qq = 0; qq < kGrp; ++qq) {
          const LRec rq = load_rec(R, qq);
          const uint32_t pos = __float_as_uint(R[8 * qq + 6]);
          float dx, dy, t;
          const float G = __builtin_amdgcn_exp2f(local_power2(rg.lx, rg.ly, rq, dx, dy, t));
          const float araw = rq.c.y * G;
          const bool act = (pos < last) & (araw >= amin);
          const float a = fminf(amax, araw);
          const float rom = __builtin_amdgcn_rcpf(1.0f - a);
          const float Tq = act ? T * rom : T;   // transmittance in front of this Gaussian
          const float wq = act ? a * Tq : 0.0f;
          const float gf = __uint_as_float(Y4[qq >> 2][qq & 3]);
          const float dalpha = Tq * gf - acc * rom;
          acc = act ? __builtin_fmaf(gf, wq, acc) : acc;
          T = Tq;
          W[qq * kPs + lane] = wq;
          // d L / d power, none through the clamp. (Selected after the product: an opacity that is NaN,
          // which no pixel takes, must leave zeros in the sums.)
          D[qq * kPs + lane] = (act & (araw < amax)) ? dalpha * araw : 0.0f;
        }
        wave_sync();
        {
          // d power / d (mean2d, A, B, C) up to the per-component factors of kGeoScale
          float Y0, Y1;
          geo_sums(D, R, gx, gy, wide ? 2.0f : 4.0f, l16, g4, Y0, Y1);
          float* a = A + l16 * AROW + KP;
          a[g4 + (g4 >> 1)] = Y0;
          if ((g4 & 1) == 0) a[2 + 3 * (g4 >> 1)] = Y1;
        }
        // dF: A = W^T (i = Gaussian l16 of the group, k = pixel 32 ks + 8 g4 + e)
        v8bf wh[2], wl2[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const float* s8 = W + l16 * kPs + 32 * ks + 8 * g4;
          const float4 w0 = *reinterpret_cast<const float4*>(s8), w1 = *reinterpret_cast<const float4*>(s8 + 4);
          const float x[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
          split8(x, wh[ks], wl2[ks]);
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          v4f d = zero4();
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) d = mma3(wh[ks], wl2[ks], g2h[ks][cb], g2l[ks][cb], d);
          // D[i][c]: Gaussian 4 g4 + r of the group, channel 16 cb + l16
#pragma unroll
          for (int r = 0; r < 4; ++r) A[(4 * g4 + r) * AROW + 16 * cb + l16] = d[r];
        }
        ++done;
      }
      if (fin) break;
    }
    wave_sync();
    if (done > 0) flush(done - 1, tail - kGrp * (done - 1));
    wave_sync();
  }
}

// Caller workspace of the reverse pass: the segment work list, sized for `cap` duplicates in
// segments of `seg` list positions (at most one more segment per tile than cap / seg).
struct SegWs {
  uint32_t *lmax, *cnt, *base, *partial, *ctl;
  uint64_t* total;
  uint2* work;
  float *P, *GC;
  int64_t max_segs;
};

size_t seg_layout(int n_tiles, int64_t cap, int seg, char* base, SegWs* w) {
  const int64_t max_segs = (int64_t)n_tiles + ceil_div(cap, seg) + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes);
    return base ? base + o : nullptr;
  };
  char* p_lmax = take(4 * (size_t)n_tiles);
  char* p_cnt = take(4 * (size_t)n_tiles);
  char* p_base = take(4 * (size_t)n_tiles);
  char* p_part = take(4 * (size_t)scan_partials_needed(n_tiles));
  char* p_tot = take(8);
  char* p_ctl = take(16);
  char* p_work = take(8 * (size_t)max_segs);
  char* p_P = take(4 * (size_t)kTilePx * max_segs);
  char* p_GC = take(4 * (size_t)kTilePx * max_segs);
  if (w) {
    w->lmax = (uint32_t*)p_lmax;
    w->cnt = (uint32_t*)p_cnt;
    w->base = (uint32_t*)p_base;
    w->partial = (uint32_t*)p_part;
    w->total = (uint64_t*)p_tot;
    w->ctl = (uint32_t*)p_ctl;
    w->work = (uint2*)p_work;
    w->P = (float*)p_P;
    w->GC = (float*)p_GC;
    w->max_segs = max_segs;
  }
  return off;
}

// Caller buffer of a splitting forward (its saved state), sized for `cap` duplicates, K
// channels and segments of `seg` list positions.
struct FLayout {
  FState fs;
  uint32_t *cnt, *base, *partial, *ctl;
  uint64_t* total;
  uint2* work;
  int64_t max_segs;
};

size_t fstate_layout(int n_tiles, int64_t cap, int K, int seg, char* base, FLayout* w) {
  const int64_t max_segs = (int64_t)n_tiles + ceil_div(cap, seg) + 1;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes);
    return base ? base + o : nullptr;
  };
  char* p_tcnt = take(4 * (size_t)n_tiles);
  char* p_tbase = take(4 * (size_t)n_tiles);
  char* p_cnt = take(4 * (size_t)n_tiles);
  char* p_base = take(4 * (size_t)n_tiles);
  char* p_part = take(4 * (size_t)scan_partials_needed(n_tiles));
  char* p_tot = take(8);
  char* p_ctl = take(16);
  char* p_work = take(8 * (size_t)max_segs);
  char* p_P = take(4 * (size_t)kTilePx * max_segs);
  char* p_Te = take(4 * (size_t)kTilePx * max_segs);
  char* p_info = take(4 * (size_t)kTilePx * max_segs);
  char* p_CS = take(4 * (size_t)kTilePx * max_segs * (size_t)K);
  if (w) {
    w->fs.tcnt = (uint32_t*)p_tcnt;
    w->fs.tbase = (uint32_t*)p_tbase;
    w->fs.P = (float*)p_P;
    w->fs.Te = (float*)p_Te;
    w->fs.info = (uint32_t*)p_info;
    w->fs.CS = (float*)p_CS;
    w->cnt = (uint32_t*)p_cnt;
    w->base = (uint32_t*)p_base;
    w->partial = (uint32_t*)p_part;
    w->total = (uint64_t*)p_tot;
    w->ctl = (uint32_t*)p_ctl;
    w->work = (uint2*)p_work;
    w->max_segs = max_segs;
  }
  return off;
}

}  // namespace

int render_seg_len(const gs_config& cfg) { return seg_len(cfg); }

size_t render_state_bytes(int n_tiles, int64_t dup_capacity, int K, int seg) {
  return fstate_layout(n_tiles, std::max<int64_t>(dup_capacity, 0), K, seg, nullptr, nullptr);
}

// Largest duplicate capacity whose forward state fits in `bytes` (-1 if none does).
int64_t render_state_capacity(int n_tiles, int K, int seg, size_t bytes) {
  if (render_state_bytes(n_tiles, 0, K, seg) > bytes) return -1;
  int64_t lo = 0, hi = 1;
  while (hi < ((int64_t)1 << 40) && render_state_bytes(n_tiles, hi, K, seg) <= bytes) hi *= 2;
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (render_state_bytes(n_tiles, mid, K, seg) <= bytes) lo = mid; else hi = mid;
  }
  return lo;
}

namespace {

// Forward state of images `im` (fs.tcnt == nullptr if there is none).
FLayout state_of(const gs_images& im, int n_tiles, int K, int seg) {
  FLayout w{};
  if (!im.state) return w;
  const int64_t cap = render_state_capacity(n_tiles, K, seg, im.state_bytes);
  if (cap >= 0) fstate_layout(n_tiles, cap, K, seg, (char*)im.state, &w);
  return w;
}

template <int NS, int MODE>
int launch_fwd_s(const gs_config& cfg, const gs_gaussians& g, const gs_projected& p, const gs_item* items, int n_items,
                 int n_tiles, const uint32_t* vals, const uint32_t* ranges, const gs_images& out, hipStream_t s) {
  const FLayout w = state_of(out, n_tiles, 4 + cfg.n_sem, seg_len(cfg));
  const FeatSrc src{g.rgb, g.sem, p.depth, g.emb, cfg.n_sem};
  if (!w.fs.tcnt) {
    hipLaunchKernelGGL((k_render_fwd_split<NS, false, MODE>), dim3(n_tiles), dim3(256), 0, s, cfg, src, p.rec, g.n, items,
                       n_items, vals, ranges, out.color, out.T, out.n_contrib, nullptr, nullptr, w.fs);
    return launch_status();
  }
  const unsigned tb = (unsigned)ceil_div(n_tiles, 256);
  hipLaunchKernelGGL(k_fseg_count, dim3(tb), dim3(256), 0, s, ranges, n_tiles, cfg.tile_order,
                     (uint32_t)seg_len(cfg), w.cnt);
  int st = launch_status();
  st = st ? st : scan_u32(w.cnt, w.base, n_tiles, w.partial, w.total, s);
  if (st) return st;
  hipLaunchKernelGGL(k_seg_list, dim3(tb), dim3(256), 0, s, w.cnt, w.base, w.total, n_tiles, cfg.tile_order,
                     w.max_segs, w.work, w.ctl, w.fs.tcnt, w.fs.tbase);
  const int grid_t = resident_blocks(k_fwd_trans, 256, 0);
  const int grid_f = resident_blocks(k_render_fwd_split<NS, true, MODE>, 256, 0);
  if (!grid_t || !grid_f) return GS_ERR_HIP;
  if (cfg.fwd_chunk > 0)
    hipLaunchKernelGGL(k_fwd_trans, dim3(grid_t), dim3(256), 0, s, cfg, p.rec, g.n, items, n_items, vals, ranges,
                       w.work, w.ctl, w.fs.P);
  hipLaunchKernelGGL((k_render_fwd_split<NS, true, MODE>), dim3(grid_f), dim3(256), 0, s, cfg, src, p.rec, g.n, items, n_items,
                     vals, ranges, out.color, out.T, out.n_contrib, w.work, w.ctl, w.fs);
  if (cfg.fwd_chunk > 0)
    hipLaunchKernelGGL(k_fwd_combine<NS>, dim3(n_tiles), dim3(256), 0, s, items, n_items, ranges, 4 + cfg.n_sem,
                       cfg.fwd_chunk, tile_shift(cfg), w.fs, out.color, out.T, out.n_contrib);
  return launch_status();
}

template <int NS, int MODE>
int launch_bwd_s(const gs_config& cfg, const gs_gaussians& g, const gs_projected& p, const gs_item* items, int n_items,
                 int n_tiles, const uint32_t* vals, const uint32_t* ranges, const gs_images& fwd,
                 const gs_images& gin, double* g2d, const gs_grads& gr, void* seg_ws, int64_t cap, hipStream_t s) {
  SegWs w;
  seg_layout(n_tiles, cap, seg_len(cfg), (char*)seg_ws, &w);
  // with the forward's saved state the segments start from it: no summary pass
  const FState fs = state_of(fwd, n_tiles, 4 + cfg.n_sem, seg_len(cfg)).fs;
  hipLaunchKernelGGL(k_seg_count, dim3((unsigned)ceil_div(n_tiles, 4)), dim3(256), 0, s, items, n_items, ranges, fwd.n_contrib, n_tiles,
                     cfg.tile_order, tile_shift(cfg), (uint32_t)seg_len(cfg), fs.tcnt, w.lmax, w.cnt);
  int st = launch_status();
  st = st ? st : scan_u32(w.cnt, w.base, n_tiles, w.partial, w.total, s);
  if (st) return st;
  hipLaunchKernelGGL(k_seg_list, dim3((unsigned)ceil_div(n_tiles, 256)), dim3(256), 0, s, w.cnt, w.base, w.total,
                     n_tiles, cfg.tile_order, w.max_segs, w.work, w.ctl, nullptr, nullptr);
  const int grid_main = resident_blocks(k_render_bwd_main<NS, MODE>, 256, 0);
  if (!grid_main) return GS_ERR_HIP;
  if (!fs.tcnt) {
    const int grid_sum = resident_blocks(k_seg_summary<NS>, 256, 0);
    if (!grid_sum) return GS_ERR_HIP;
    hipLaunchKernelGGL(k_seg_summary<NS>, dim3(grid_sum), dim3(256), 0, s, cfg, g.rgb, g.sem, g.emb, cfg.n_sem, p.rec,
                       p.depth, g.n, items, n_items, vals, ranges, fwd.n_contrib, gin.color, w.work, w.ctl, w.lmax, w.P,
                       w.GC);
  }
  const FeatSrc src{g.rgb, g.sem, p.depth, g.emb, cfg.n_sem};
  hipLaunchKernelGGL((k_render_bwd_main<NS, MODE>), dim3(grid_main), dim3(256), 0, s, cfg, src, p.rec, g.n, items, n_items,
                     vals, ranges, fwd.T, fwd.n_contrib, gin.color, GradDst{gr.rgb, gr.sem, g2d}, w.work, w.ctl, w.P,
                     w.GC, fs);
  return launch_status();
}

}  // namespace

size_t render_seg_workspace(int n_tiles, int64_t dup_capacity, int seg) {
  return seg_layout(n_tiles, std::max<int64_t>(dup_capacity, 0), seg, nullptr, nullptr);
}

// Largest duplicate capacity whose segment workspace fits in `bytes` (-1 if none does).
int64_t render_seg_capacity(int n_tiles, int seg, size_t bytes) {
  if (render_seg_workspace(n_tiles, 0, seg) > bytes) return -1;
  int64_t lo = 0, hi = 1;
  while (hi < ((int64_t)1 << 40) && render_seg_workspace(n_tiles, hi, seg) <= bytes) hi *= 2;
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (render_seg_workspace(n_tiles, mid, seg) <= bytes) lo = mid; else hi = mid;
  }
  return lo;
}

int launch_render_fwd_split(const gs_config& cfg, const gs_gaussians& g, const gs_projected& p, const gs_item* items,
                            int n_items, int n_tiles, const uint32_t* vals, const uint32_t* ranges,
                            const gs_images& out, hipStream_t s) {
  const auto launch = [&](auto f) { return f(cfg, g, p, items, n_items, n_tiles, vals, ranges, out, s); };
  const FeatMode m = feat_mode(g, cfg.n_sem);
  if (cfg.n_sem <= 28)
    return launch(m == kEmbVec ? launch_fwd_s<28, kEmbVec> : m == kRowVec ? launch_fwd_s<28, kRowVec> : launch_fwd_s<28, kValues>);
  if (cfg.n_sem <= 60) return launch(m == kRowVec ? launch_fwd_s<60, kRowVec> : launch_fwd_s<60, kValues>);
  return GS_ERR_UNSUPPORTED;
}

int launch_render_bwd_split(const gs_config& cfg, const gs_gaussians& g, const gs_projected& p, const gs_item* items,
                            int n_items, int n_tiles, const uint32_t* vals, const uint32_t* ranges,
                            const gs_images& fwd, const gs_images& gin, double* g2d, const gs_grads& gr, void* seg_ws,
                            int64_t cap, hipStream_t s) {
  if (cap < 0) return GS_ERR_WORKSPACE;
  const auto launch = [&](auto f) {
    return f(cfg, g, p, items, n_items, n_tiles, vals, ranges, fwd, gin, g2d, gr, seg_ws, cap, s);
  };
  const FeatMode m = feat_mode(g, cfg.n_sem);
  if (cfg.n_sem <= 28)
    return launch(m == kEmbVec ? launch_bwd_s<28, kEmbVec> : m == kRowVec ? launch_bwd_s<28, kRowVec> : launch_bwd_s<28, kValues>);
  if (cfg.n_sem <= 60) return launch(m == kRowVec ? launch_bwd_s<60, kRowVec> : launch_bwd_s<60, kValues>);
  return GS_ERR_UNSUPPORTED;
}

}  // namespace gs
