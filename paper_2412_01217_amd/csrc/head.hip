// Learned semantic head: logits = W2 relu(W1 E + b1) + b2 per pixel, where E is the
// composited 16-wide embedding (eq. 9 with an embedding in place of class logits),
// W1 [64][16] and W2 [C][64] bfloat16, biases float32. Forward and backward run on
// matrix cores as v_mfma_f32_32x32x16_bf16, two k-steps of 32x32x8 at a time (mfma2). Single-precision activations enter the
// bfloat16 products as a hi + lo pair (x = bf16(x) + bf16(x - bf16(x))), which keeps
// the decode within ~2^-16 of single precision; products of two single-precision
// factors (weight gradients) use hi*hi + hi*lo + lo*hi.
//
// 32x32x8 bf16 operand layout (lane l): A[i][k]: i = l % 32, k = 4 (l / 32) + 0..3;
// B[k][j]: k = 4 (l / 32) + 0..3, j = l % 32; D as the 32x32 f32 layout
// (j = l % 32, i = 8 (r / 4) + 4 (l / 32) + r % 4). Computing the transposed
// activations H^T = W1 E^T leaves, in registers 4g..4g+3 of a lane, exactly the four
// hidden units that form the B operand of the next product's k-step g, so layers chain
// without a transpose.
#include "common.h"

namespace gs {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));

constexpr int kDin = 16;
constexpr int kHid = 64;
constexpr int kHeadBlocksMax = 512;
// per-block partial of the weight gradients: dW2 [64][64], dW1 [64][32] (column 16 = db1), db2 [64]
constexpr int kPartW2 = 64 * 64;
constexpr int kPartW1 = 64 * 32;
constexpr int kPartB2 = 64;
constexpr int kPart = kPartW2 + kPartW1 + kPartB2;
constexpr int kWtStride = kHid + 8;   // bfloat16 row stride of the transposed weights in LDS (16-byte rows)

__device__ __forceinline__ int drow(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Splits four floats into hi and lo bfloat16 operands (hardware round-to-nearest-even), two
// values per conversion.
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split4(const float* x, v4s& hi, v4s& lo) {
  uint32_t h[2], l[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    h[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){x[2 * k], x[2 * k + 1]}, bf2));
    const float h0 = __uint_as_float(h[k] << 16), h1 = __uint_as_float(h[k] & 0xffff0000u);
    l[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2){x[2 * k] - h0, x[2 * k + 1] - h1}, bf2));
  }
  hi = __builtin_bit_cast(v4s, make_uint2(h[0], h[1]));
  lo = __builtin_bit_cast(v4s, make_uint2(l[0], l[1]));
}

// Two consecutive k-steps of 32x32x8 as one v_mfma_f32_32x32x16_bf16 (twice the work per
// instruction on gfx950): lane (l % 32, h = l / 32) supplies k = 8 h + 0..7 of the 16; given
// k-step pairs whose lane h holds k = 8 (2s) + 4 h + 0..3 and 8 (2s + 1) + 4 h + 0..3 (the
// layout above), the concatenation [step 2s, step 2s + 1] covers each k of the pair once in
// both operands, so the product is the same sum over the 16 k.
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
__device__ __forceinline__ v16f mfma2(v8s a, v8s b, v16f c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}
__device__ __forceinline__ v8s cat(v4s x0, v4s x1) { return __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7); }
__device__ __forceinline__ v16f mfma2(v4s a0, v4s a1, v4s b0, v4s b1, v16f c) { return mfma2(cat(a0, a1), cat(b0, b1), c); }
__device__ __forceinline__ v16f mfma2(v8s a, v4s b0, v4s b1, v16f c) { return mfma2(a, cat(b0, b1), c); }
__device__ __forceinline__ v16f mfma2(v4s a0, v4s a1, v8s b, v16f c) { return mfma2(cat(a0, a1), b, c); }

__device__ __forceinline__ v16f zero16() {
  v16f z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.0f;
  return z;
}

// Walks the 64-pixel chunks of the concatenated items in increasing order. Chunks
// never straddle two items, so every pixel of a chunk shares one item's plane layout.
struct ChunkCursor {
  int item;
  int64_t first, end;   // chunks [first, end) belong to `item`
};

__device__ __forceinline__ int64_t item_chunks(const gs_item& it) { return ((int64_t)it.W * it.H + 63) / 64; }

// Moves the cursor forward to the item holding `chunk`; false once past the last item.
__device__ __forceinline__ bool seek_chunk(const gs_item* __restrict__ items, int n_items, int64_t chunk,
                                           ChunkCursor& cur) {
  while (chunk >= cur.end && cur.item + 1 < n_items) {
    ++cur.item;
    cur.first = cur.end;
    cur.end += item_chunks(items[cur.item]);
  }
  return chunk < cur.end;
}

// Backward of the head. Each wave takes 64-pixel chunks in a grid-stride loop. It
// stages the chunk's logit gradients in LDS ([class][pixel], classes >= C stay zero),
// then, per 32-pixel half,
//  (1) recomputes the hidden pre-activations for the ReLU mask,
//  (2) forms dH^T = W2^T dlogits^T (hidden in registers, pixels across lanes),
//  (3) adds (or stores) dE^T = W1^T dH^T to the colour-gradient planes 4..19,
//  (4) recomputes H and dH with pixels in registers and hidden units across lanes --
//      the layout in which a matrix-core product contracts over pixels -- and
//  (5) accumulates dW2 = dlogits^T relu(H), db2 and dW1 = dH^T [E, 1] (column 16 is
//      db1) in registers that live across the whole loop.
// The accumulators are summed over the block's waves in LDS once at the end and written
// as one partial per block; k_head_reduce adds the partials.
constexpr int kGst = 65;   // LDS row stride of the staged logit gradients

// The block's shared state of a head backward: transposed weights and the per-wave staging.
// The transposed weights' rows are stored with the contraction index k at kperm(k) (bits 2
// and 3 of k swapped), so that the 8 values a lane supplies to a 32x32x16 product of the
// k-step pair s (k = 16 s + 4 h + 0..3 and 16 s + 8 + 4 h + 0..3, see mfma2) are contiguous
// at 16 s + 8 h: one 16-byte LDS read.
__host__ __device__ constexpr int kperm(int k) { return (k & ~12) | ((k & 4) << 1) | ((k & 8) >> 1); }

template <int ROW, int WAVES>
struct alignas(16) HeadLdsOf {
  static constexpr int kRow = ROW;
  float buf[WAVES * kHid * ROW];         // per wave [class][pixel]; the block's partial at the end
  uint16_t w2t[kHid * kWtStride];    // W2^T [hidden][kperm(class)], classes >= C zero
  uint16_t w1t[kDin * kWtStride];    // W1^T [d][kperm(hidden)]
  float b1[kHid];
};
using HeadLds = HeadLdsOf<kGst, 4>;

// Per-lane accumulators of the weight gradients over a block's chunks.
struct HeadAcc {
  v16f W2[2][2], W1[2];   // W2[cb][hb]: D[c][h]; W1[hb]: D[h][d]
  float B2[2];            // class l32 + 32 cb, this lane's pixels
};

template <class LDS>
__device__ __forceinline__ void head_setup(LDS& L, int C, const uint16_t* __restrict__ W1,
                                           const float* __restrict__ b1, const uint16_t* __restrict__ W2,
                                           HeadAcc& acc, v4s (&w1a)[2][2], float (&b1l)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
  for (int i = threadIdx.x; i < kHid * kHid; i += (int)blockDim.x) {
    const int c = i / kHid, h = i % kHid;
    L.w2t[h * kWtStride + kperm(c)] = c < C ? W2[c * kHid + h] : (uint16_t)0;
  }
  for (int i = threadIdx.x; i < kHid * kDin; i += (int)blockDim.x) {
    const int h = i / kDin, d = i % kDin;
    L.w1t[d * kWtStride + kperm(h)] = W1[h * kDin + d];
  }
  if (threadIdx.x < kHid) L.b1[threadIdx.x] = b1[threadIdx.x];
  float* sg = L.buf + wave * kHid * LDS::kRow;
  for (int i = C * LDS::kRow + lane; i < kHid * LDS::kRow; i += 64) sg[i] = 0.0f;   // rows of absent classes
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    acc.W1[i] = zero16();
    acc.W2[i][0] = zero16();
    acc.W2[i][1] = zero16();
    acc.B2[i] = 0.0f;
  }
  // W1 as A (i = hidden l32 + 32 hb, k = d 8 ks + 4 half + j), which is also W1^T as B (k = d, j = hidden)
#pragma unroll
  for (int hb = 0; hb < 2; ++hb)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j) w1a[hb][ks][j] = (short)W1[(l32 + 32 * hb) * kDin + 8 * ks + 4 * half + j];
  b1l[0] = L.b1[l32];
  b1l[1] = L.b1[l32 + 32];
}

// Steps (1)-(5) for one 64-pixel chunk whose logit gradients are staged in sg [class][pixel].
// Eb: pixel 0 of plane 0 of the chunk's embedding, plane d at Eb + d HW; dEb: the chunk's
// gradient planes, which dE is added to.
__device__ __forceinline__ void head_chunk_backward(const HeadLds& L, const float* sg, const float* Eb, float* dEb,
                                                    int64_t HW, int nlive, const v4s (&w1a)[2][2],
                                                    const float (&b1l)[2], HeadAcc& acc) {
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
#pragma unroll 1
  for (int pb = 0; pb < 2; ++pb) {
    const int q = l32 + 32 * pb;
    const bool qlive = q < nlive;
    const float* Eq = Eb + 4 * half * HW + min(q, nlive - 1);   // plane 8 ks + 4 half + j at Eq + (8 ks + j) HW
    const float* Gq = sg + 4 * half * kGst + q;                 // class 8 ks + 4 half + j at Gq + (8 ks + j) kGst
    // (1) E with d in registers, pixels across lanes; the sign of the hidden pre-activations
    v4s ehi[2], elo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      float e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = Eq[(8 * ks + j) * HW];
        e[j] = qlive ? v : 0.0f;
      }
      split4(e, ehi[ks], elo[ks]);
    }
    uint32_t on[2];   // bit r: hidden unit drow(r) + 32 hb is active at this pixel
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        v16f h;
#pragma unroll
        for (int r = 0; r < 16; ++r) h[r] = L.b1[drow(r, lane) + 32 * hb];
        h = mfma2(w1a[hb][0], w1a[hb][1], ehi[0], ehi[1], h);
        h = mfma2(w1a[hb][0], w1a[hb][1], elo[0], elo[1], h);
        uint32_t bits = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) bits |= (h[r] > 0.0f ? 1u : 0u) << r;
        on[hb] = bits;
      }

    // (2) dH^T = W2^T dlogits^T: A = W2^T (i = hidden l32 + 32 hb, k = class 8 ks + 4 half + j)
    v16f dHT[2] = {zero16(), zero16()};
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      v4s hi[2], lo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int ks = 2 * s2 + u;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = Gq[(8 * ks + j) * kGst];
        split4(x, hi[u], lo[u]);
      }
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const v8s a = *reinterpret_cast<const v8s*>(L.w2t + (l32 + 32 * hb) * kWtStride + 16 * s2 + 8 * half);
        dHT[hb] = mfma2(a, hi[0], hi[1], dHT[hb]);
        dHT[hb] = mfma2(a, lo[0], lo[1], dHT[hb]);
      }
    }
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 16; ++r) dHT[hb][r] = ((on[hb] >> r) & 1u) ? dHT[hb][r] : 0.0f;

    // (3) dE^T = W1^T dH^T: A = W1^T (i = d l32, k = hidden 8 ks + 4 half + j); B from the
    // dH^T registers 4 (ks % 4) .. +3 of block ks / 4
    {
      v16f dE = zero16();
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        v8s a = {0, 0, 0, 0, 0, 0, 0, 0};
        if (l32 < kDin) a = *reinterpret_cast<const v8s*>(L.w1t + l32 * kWtStride + 16 * s2 + 8 * half);
        v4s hi[2], lo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int ks = 2 * s2 + u;
          float x[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = dHT[ks >> 2][4 * (ks & 3) + j];
          split4(x, hi[u], lo[u]);
        }
        dE = mfma2(a, hi[0], hi[1], dE);
        dE = mfma2(a, lo[0], lo[1], dE);
      }
      // rows 0..15 = d: added to what the caller's gradient holds there
      if (qlive)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          float* dst = dEb + (int64_t)drow(r, lane) * HW + q;
          *dst += dE[r];
        }
    }

    // Reloading from LDS below is cheaper than keeping (2)'s operands alive through (3).
    asm volatile("" ::: "memory");
    // (4) H with pixels in registers: A = E (i = pixel), B = W1^T (k = d, j = hidden l32 + 32 hb)
    v16f H[2];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      H[hb] = mfma2(ehi[0], ehi[1], w1a[hb][0], w1a[hb][1], zero16());
      H[hb] = mfma2(elo[0], elo[1], w1a[hb][0], w1a[hb][1], H[hb]);
#pragma unroll
      for (int r = 0; r < 16; ++r) H[hb][r] = fmaxf(H[hb][r] + b1l[hb], 0.0f);
    }
    // (5a) dW2[c][h] += sum_p dlogits[c][p] relu(H)[p][h] over the half's pixels
    // p = 32 pb + 8 kk + 4 half + j (registers 4 kk + j): A = dlogits (i = class l32 + 32 cb, k = p)
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        v4s ahi[2], alo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int p0 = 32 * pb + 8 * (2 * k2 + u) + 4 * half;
          float x[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = sg[(l32 + 32 * cb) * kGst + p0 + j];
          acc.B2[cb] += (x[0] + x[1]) + (x[2] + x[3]);
          split4(x, ahi[u], alo[u]);
        }
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          v4s bhi[2], blo[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float y[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = H[hb][4 * (2 * k2 + u) + j];
            split4(y, bhi[u], blo[u]);
          }
          acc.W2[cb][hb] = mfma2(ahi[0], ahi[1], bhi[0], bhi[1], acc.W2[cb][hb]);
          acc.W2[cb][hb] = mfma2(ahi[0], ahi[1], blo[0], blo[1], acc.W2[cb][hb]);
          acc.W2[cb][hb] = mfma2(alo[0], alo[1], bhi[0], bhi[1], acc.W2[cb][hb]);
        }
      }
    }
    uint32_t onH[2];   // bit r: hidden unit l32 + 32 hb is active at pixel drow(r) of the half
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      uint32_t bits = 0;
#pragma unroll
      for (int r = 0; r < 16; ++r) bits |= (H[hb][r] > 0.0f ? 1u : 0u) << r;
      onH[hb] = bits;
    }
    // (4b) dH with pixels in registers: A = dlogits (i = pixel, k = class), B = W2 (j = hidden)
    v16f dH[2] = {zero16(), zero16()};
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      v4s hi[2], lo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int ks = 2 * s2 + u;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = Gq[(8 * ks + j) * kGst];
        split4(x, hi[u], lo[u]);
      }
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const v8s b = *reinterpret_cast<const v8s*>(L.w2t + (l32 + 32 * hb) * kWtStride + 16 * s2 + 8 * half);
        dH[hb] = mfma2(hi[0], hi[1], b, dH[hb]);
        dH[hb] = mfma2(lo[0], lo[1], b, dH[hb]);
      }
    }
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 16; ++r) dH[hb][r] = ((onH[hb] >> r) & 1u) ? dH[hb][r] : 0.0f;
    // (5b) dW1[h][d] += sum_p dH[p][h] [E, 1][p][d]: A = dH (i = hidden l32 + 32 hb, k = p), B = [E, 1] (j = d l32)
    const float* Ed = Eb + (int64_t)min(l32, kDin - 1) * HW;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      v4s bhi[2], blo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int p0 = 32 * pb + 8 * (2 * k2 + u) + 4 * half;
        float e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = Ed[min(p0 + j, nlive - 1)];
          e[j] = p0 + j >= nlive ? 0.0f : (l32 < kDin ? v : (l32 == kDin ? 1.0f : 0.0f));
        }
        split4(e, bhi[u], blo[u]);
      }
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        v4s ahi[2], alo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float y[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) y[j] = dH[hb][4 * (2 * k2 + u) + j];
          split4(y, ahi[u], alo[u]);
        }
        acc.W1[hb] = mfma2(ahi[0], ahi[1], bhi[0], bhi[1], acc.W1[hb]);
        acc.W1[hb] = mfma2(ahi[0], ahi[1], blo[0], blo[1], acc.W1[hb]);
        acc.W1[hb] = mfma2(alo[0], alo[1], bhi[0], bhi[1], acc.W1[hb]);
      }
    }
  }
}

// Sums the block's waves' accumulators in LDS and writes the block's partial.
template <class LDS>
__device__ __forceinline__ void head_write_partial(LDS& L, const HeadAcc& acc, float* __restrict__ partial, bool add) {
  const int lane = threadIdx.x & 63, l32 = lane & 31;
  float* s_acc = L.buf;
  __syncthreads();
  for (int i = threadIdx.x; i < kPart; i += (int)blockDim.x) s_acc[i] = 0.0f;
  __syncthreads();
  if (add) {   // (uniform over the wave: it had a chunk)
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = drow(r, lane) + 32 * cb;   // D[c][h]: h = l32 + 32 hb
          atomicAdd(&s_acc[c * 64 + l32 + 32 * hb], acc.W2[cb][hb][r]);
        }
      atomicAdd(&s_acc[kPartW2 + kPartW1 + l32 + 32 * cb], acc.B2[cb]);
    }
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int r = 0; r < 16; ++r) atomicAdd(&s_acc[kPartW2 + (drow(r, lane) + 32 * hb) * 32 + l32], acc.W1[hb][r]);
  }
  __syncthreads();
  float* out = partial + (int64_t)blockIdx.x * kPart;
  for (int i = threadIdx.x; i < kPart; i += (int)blockDim.x) out[i] = s_acc[i];
}

__global__ __launch_bounds__(256, 1) void k_head_bwd(const gs_item* __restrict__ items, int n_items, int K, int C,
                                                     const float* __restrict__ color,
                                                     const float* __restrict__ glogits,
                                                     const uint16_t* __restrict__ W1, const float* __restrict__ b1,
                                                     const uint16_t* __restrict__ W2, float* __restrict__ gcolor,
                                                     float* __restrict__ partial) {
  __shared__ HeadLds L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  HeadAcc acc;
  v4s w1a[2][2];
  float b1l[2];
  head_setup(L, C, W1, b1, W2, acc, w1a, b1l);
  float* sg = L.buf + wave * kHid * kGst;
  ChunkCursor cur;
  cur.item = 0;
  cur.first = 0;
  cur.end = item_chunks(items[0]);
  for (int64_t chunk = (int64_t)blockIdx.x * 4 + wave;; chunk += (int64_t)gridDim.x * 4) {
    if (!seek_chunk(items, n_items, chunk, cur)) break;
    const gs_item it = items[cur.item];
    const int64_t HW = (int64_t)it.W * it.H;
    const int64_t local0 = (chunk - cur.first) * 64;
    const int nlive = (int)min((int64_t)64, HW - local0);
    {
      // stage: lane = pixel, one coalesced row per class; dead pixels are zero
      // (16 rows' loads in flight per round trip)
      const bool live = lane < nlive;
      const float* g = glogits + it.pixel_base * C + local0 + min(lane, nlive - 1);
      for (int c0 = 0; c0 < C; c0 += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = c0 + k < C ? g[(int64_t)(c0 + k) * HW] : 0.0f;
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (c0 + k < C) sg[(c0 + k) * kGst + lane] = live ? v[k] : 0.0f;
      }
    }
    wave_sync();
    head_chunk_backward(L, sg, color + it.pixel_base * K + 4 * HW + local0, gcolor + it.pixel_base * K + 4 * HW + local0,
                        HW, nlive, w1a, b1l, acc);
    // every lane is past this chunk's reads of the staged rows before the next chunk writes them
    wave_sync();
  }
  head_write_partial(L, acc, partial, true);
}

// Learned-mode loss with the decode fused in (paper eq. 10-13 with the semantic term a
// cross-entropy on the head's logits): per 64-pixel chunk of one item, the L1 colour and
// depth terms (lane = pixel, as in the plain loss), the decode logits = W2 relu(W1 E + b1)
// + b2 on the matrix cores, the cross-entropy against the label and its logit gradient
// w2 (softmax - onehot) / HW, and the head's backward (steps (2)-(5) above) storing dL/dE in the colour-gradient planes 4..19 and accumulating the weight gradients.
// No logits touch global memory. Loss partial sums go to the same per-item slots as the
// plain loss's.
//
// A block is eight waves, two per SIMD, on one CU: the weights are in LDS once for all, and what
// is left of the 160 KB is a wave's half of logit gradients (9 KB) and two buffers for the 16
// embedding planes of a chunk (4 KB each): while a wave works on one chunk, direct global-to-LDS
// loads fill the other buffer with its next chunk. The buffers are two separate LDS arrays and the
// loop handles two chunks per iteration, one from each, so that the compiler's wait for a buffer's
// loads never waits for the other's. Labels come one chunk ahead in a register, colour, depth and
// their targets during the chunk. (One wave per SIMD with every input staged, logit gradients
// staged and read back as three operands, ReLU masks as bits: 2.80 ms on four full-HD pyramids with
// 52 classes; everything over classes in registers: 1.95; two waves per SIMD: 1.74, 64 bytes a lane
// of it in scratch.)
constexpr int kEst = 65;   // row stride (floats) of a staged embedding plane: lanes on rows meet no bank twice
constexpr int kFusedWaves = 8;

struct ChunkStage {        // one wave's staged chunk: 64 pixels of every embedding plane
  float E[kDin][kEst];
};

struct ChunkInfo {
  int64_t chunk, pixel_base, HW, local0;
  int item, nlive;
};

// The item table read through the constant address space: the chunk walk is wave-uniform,
// and its reads become scalar loads, which do not wait behind the vector memory queue
// (where the staging loads are in flight).
typedef const __attribute__((address_space(4))) gs_item* ConstItems;

__device__ __forceinline__ bool seek_chunk_c(ConstItems items, int n_items, int64_t chunk, ChunkCursor& cur) {
  while (chunk >= cur.end && cur.item + 1 < n_items) {
    ++cur.item;
    cur.first = cur.end;
    cur.end += ((int64_t)items[cur.item].W * items[cur.item].H + 63) / 64;
  }
  return chunk < cur.end;
}

// The chunk's place in the item table (false once past the last item).
__device__ __forceinline__ bool chunk_info(ConstItems items, int n_items, int64_t chunk, ChunkCursor& cur,
                                           ChunkInfo& ci) {
  if (!seek_chunk_c(items, n_items, chunk, cur)) return false;
  ci.chunk = chunk;
  ci.item = cur.item;
  ci.pixel_base = items[cur.item].pixel_base;
  ci.HW = (int64_t)items[cur.item].W * items[cur.item].H;
  ci.local0 = (chunk - cur.first) * 64;
  ci.nlive = (int)min((int64_t)64, ci.HW - ci.local0);
  return true;
}

// Decode of the rendered embeddings: logits W2 relu(W1 E + b1) + b2 per pixel. Persistent waves
// walk 64-pixel chunks; W1 stays in registers, W2 in LDS, and the next chunk's 16 values per lane
// are loaded before this one's are used. A half of a chunk's 32 pixels goes through
// H^T = W1 E^T and logits^T = W2 h^T with the hidden layer in registers (see the top of the file),
// split once for both class blocks. Bound by the logits' way to memory: at 52 classes 2.07 million
// pixels read 133 MB and write 431 MB, 0.12 ms at copy rate; a wave per chunk that fetched the
// weights value by value took 0.36 ms. Pixels from the P-th on (gs_images.n_pixels) are not written.
__global__ __launch_bounds__(256, 2) void k_head_fwd(const gs_item* __restrict__ items, int n_items, int64_t P, int K,
                                                     int C, const float* __restrict__ color,
                                                     const uint16_t* __restrict__ W1, const float* __restrict__ b1,
                                                     const uint16_t* __restrict__ W2, const float* __restrict__ b2,
                                                     float* __restrict__ logits) {
  __shared__ __align__(16) uint16_t w2r[kHid * kWtStride];   // W2 [class][kperm(hidden)], rows >= C zero
  __shared__ float s_b1[kHid], s_b2[kHid];
  const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < kHid * kHid; i += 256) {
    const int c = i / kHid, h = i % kHid;
    w2r[c * kWtStride + kperm(h)] = c < C ? W2[c * kHid + h] : (uint16_t)0;
  }
  if (threadIdx.x < kHid) {
    s_b1[threadIdx.x] = b1[threadIdx.x];
    s_b2[threadIdx.x] = (int)threadIdx.x < C ? b2[threadIdx.x] : 0.0f;
  }
  // A = W1 (i = hidden l32 + 32 hb, k = d 8 ks + 4 half + j)
  v4s w1a[2][2];
#pragma unroll
  for (int hb = 0; hb < 2; ++hb)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 4; ++j) w1a[hb][ks][j] = (short)W1[(l32 + 32 * hb) * kDin + 8 * ks + 4 * half + j];
  __syncthreads();
  ConstItems citems = (ConstItems)items;
  ChunkCursor cur;
  cur.item = 0;
  cur.first = 0;
  cur.end = ((int64_t)citems[0].W * citems[0].H + 63) / 64;
  const int64_t stride = (int64_t)gridDim.x * 4;
  ChunkInfo ci, cn;
  float e[2][2][4];   // embedding value 8 ks + 4 half + j of pixel 32 pb + l32
  auto load = [&](const ChunkInfo& c) {
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      const float* b = color + c.pixel_base * K + c.local0 + min(l32 + 32 * pb, c.nlive - 1) + (4 + 4 * half) * c.HW;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 4; ++j) e[pb][ks][j] = b[(8 * ks + j) * c.HW];
    }
  };
  if (!chunk_info(citems, n_items, (int64_t)blockIdx.x * 4 + wave, cur, ci)) return;
  load(ci);
  for (;;) {
    v4s ehi[2][2], elo[2][2];
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) split4(e[pb][ks], ehi[pb][ks], elo[pb][ks]);
    const bool more = chunk_info(citems, n_items, ci.chunk + stride, cur, cn);
    if (more) load(cn);
    float* out = logits + ci.pixel_base * C + ci.local0 + l32;
    const int nout = (int)max((int64_t)0, min((int64_t)ci.nlive, P - (ci.pixel_base + ci.local0)));
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      v16f H[2];
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        H[hb] = mfma2(w1a[hb][0], w1a[hb][1], ehi[pb][0], ehi[pb][1], zero16());
        H[hb] = mfma2(w1a[hb][0], w1a[hb][1], elo[pb][0], elo[pb][1], H[hb]);
#pragma unroll
        for (int r = 0; r < 16; ++r) H[hb][r] = fmaxf(H[hb][r] + s_b1[drow(r, lane) + 32 * hb], 0.0f);
      }
      v16f Lg[2] = {zero16(), zero16()};
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        v4s hi[2], lo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int ks = 2 * s2 + u;
          float x[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = H[ks >> 2][4 * (ks & 3) + j];
          split4(x, hi[u], lo[u]);
        }
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const v8s a = *reinterpret_cast<const v8s*>(w2r + (l32 + 32 * cb) * kWtStride + 16 * s2 + 8 * half);
          Lg[cb] = mfma2(a, hi[0], hi[1], Lg[cb]);
          Lg[cb] = mfma2(a, lo[0], lo[1], Lg[cb]);
        }
      }
      if (l32 + 32 * pb < nout)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = drow(r, lane) + 32 * cb;
            if (c < C) __builtin_nontemporal_store(Lg[cb][r] + s_b2[c], out + 32 * pb + c * ci.HW);
          }
    }
    if (!more) break;
    ci = cn;
  }
}

constexpr int kStageLoads = kDin;   // direct-to-LDS loads per staged chunk

// Waits until at most kStageLoads vector memory operations are in flight: those are the
// other buffer's loads, issued last, so everything before them -- this buffer's loads and
// the previous chunk's stores -- is complete. Vector memory operations complete in issue
// order. (s_waitcnt encoding: vmcnt 16 in bits 3:0 and 15:14, expcnt and lgkmcnt not
// waited for.)
__device__ __forceinline__ void wait_own_stage() {
  static_assert(kStageLoads == 16, "the wait below encodes vmcnt(16)");
  __builtin_amdgcn_s_waitcnt((1 << 14) | (0xF << 8) | (0x7 << 4) | 0);
}

// Issues the direct-to-LDS loads of chunk ci into S (lane l fills entry l of every row;
// lanes past the item's last pixel load that pixel again).
__device__ __forceinline__ void stage_chunk(ChunkStage& S, const ChunkInfo& ci, int K, const float* color) {
  const int lane = threadIdx.x & 63;
  const int64_t p = ci.local0 + min(lane, ci.nlive - 1);
  const float* cb = color + ci.pixel_base * K + p;
  // the previous chunk's reads of S are complete before the loads overwrite it
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int d = 0; d < kDin; ++d)
    __builtin_amdgcn_global_load_lds(cb + (int64_t)(4 + d) * ci.HW, &S.E[d][0], 4, 0, 0);
}
__device__ __forceinline__ int load_label(const ChunkInfo& ci, const int32_t* tlabel) {
  return tlabel[ci.pixel_base + ci.local0 + min((int)(threadIdx.x & 63), ci.nlive - 1)];
}

// A wave's loss sums over its chunks of one item, per lane.
struct LossSums {
  float rgb, depth, ce, valid;
  int item, slot;
};
// One atomic per wave and quantity.
__device__ __forceinline__ void flush_loss(LossSums& a, int n_slots, float* loss_slots, float* count_slots) {
  const float lr = wave_sum(a.rgb), ld = wave_sum(a.depth), c = wave_sum(a.ce), v = wave_sum(a.valid);
  if ((threadIdx.x & 63) == 0) {
    float* loss = loss_slots + a.slot;
    atomicAdd(&loss[(3 * a.item + 0) * n_slots], lr);
    if (v != 0.0f) {
      atomicAdd(&loss[(3 * a.item + 1) * n_slots], ld);
      atomicAdd(&count_slots[a.item * n_slots + a.slot], v);
    }
    atomicAdd(&loss[(3 * a.item + 2) * n_slots], c);
  }
  a.rgb = a.depth = a.ce = a.valid = 0.0f;
}

// Everything k_head_loss does for one staged chunk.
constexpr int kFst = 36;   // LDS row stride of a half's logit gradients (32 pixels)
using FusedLds = HeadLdsOf<kFst, kFusedWaves>;
__device__ __forceinline__ void head_loss_chunk(const FusedLds& L, const uint16_t* w2r, const ChunkStage& S,
                                                const ChunkInfo& ci, float* sg, int K, int C, float w0, float w2,
                                                bool rgb_grad, int n_slots, const float* b2s,
                                                const v4s (&w1a)[2][2], const float (&b1l)[2], HeadAcc& acc,
                                                LossSums& sums, int y_own, const float* __restrict__ color,
                                                const float* __restrict__ trgb, const float* __restrict__ tdepth,
                                                float* __restrict__ loss_slots, float* __restrict__ count_slots,
                                                float* __restrict__ gcolor) {
  const int lane = threadIdx.x & 63;
  const int64_t HW = ci.HW;
  const int nlive = ci.nlive;
  const float invp = 1.0f / (float)HW;
  if (sums.item != ci.item) {   // (uniform)
    if (sums.item >= 0) flush_loss(sums, n_slots, loss_slots, count_slots);
    sums.item = ci.item;
    sums.slot = (int)(ci.chunk % n_slots);
  }
  wait_own_stage();
  // Per half of 32 pixels, decode, cross-entropy and their backward in one go. In the D layout
  // lane l holds pixel 32 pb + l32 of hidden units (or classes) drow(r) + 32 hb, which is also the
  // operand layout of the next product over them, so the logit gradients go from the softmax to
  // the products over classes in registers, split once; only the product over pixels (5a) takes
  // them from LDS, where it finds a class's pixels side by side.
#pragma unroll 1
  for (int pb = 0; pb < 2; ++pb) {
    // (a lane number of unknown origin: the many LDS addresses formed from it are not hoisted out of
    // the loops, where they would hold the registers that the accumulators need)
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int l32 = lane & 31, half = lane >> 5;
    const int q = l32 + 32 * pb;
    const bool qlive = q < nlive;
    const int y = __shfl(y_own, q, 64);
    // E with d in registers, pixels across lanes
    v4s ehi[2], elo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      float e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = S.E[8 * ks + 4 * half + j][q];
        e[j] = qlive ? v : 0.0f;
      }
      split4(e, ehi[ks], elo[ks]);
    }
    v16f H[2];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      H[hb] = mfma2(w1a[hb][0], w1a[hb][1], ehi[0], ehi[1], zero16());
      H[hb] = mfma2(w1a[hb][0], w1a[hb][1], elo[0], elo[1], H[hb]);
#pragma unroll
      for (int r = 0; r < 16; ++r) H[hb][r] = fmaxf(H[hb][r] + L.b1[drow(r, lane) + 32 * hb], 0.0f);
    }
    __builtin_amdgcn_sched_barrier(0);
    // logits: A = W2 (i = class l32 + 32 cb, k = hidden 8 ks + 4 half + j); rows >= C are zero
    v16f Lg[2] = {zero16(), zero16()};
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      __builtin_amdgcn_sched_barrier(0);
      v4s hi[2], lo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int ks = 2 * s2 + u;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = H[ks >> 2][4 * (ks & 3) + j];
        split4(x, hi[u], lo[u]);
      }
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const v8s a = *reinterpret_cast<const v8s*>(w2r + (l32 + 32 * cb) * kWtStride + 16 * s2 + 8 * half);
        Lg[cb] = mfma2(a, hi[0], hi[1], Lg[cb]);
        Lg[cb] = mfma2(a, lo[0], lo[1], Lg[cb]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // softmax over the pixel's classes: this lane's 32, then the partner lane's. b2s is minus
    // infinity for an absent class, whose logit then leaves nothing behind.
    float m = -INFINITY;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        Lg[cb][r] += b2s[drow(r, lane) + 32 * cb];
        m = fmaxf(m, Lg[cb][r]);
      }
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    const int yl = y - 4 * half;   // class drow(r) + 32 cb is 8 (r / 4) + r % 4 + 32 cb of this lane's
    float z = 0.0f, xy = 0.0f;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        xy = yl == 8 * (r >> 2) + (r & 3) + 32 * cb ? Lg[cb][r] : xy;
        const float e = __expf(Lg[cb][r] - m);
        Lg[cb][r] = e;
        z += e;
      }
    z += __shfl_xor(z, 32, 64);
    xy += __shfl_xor(xy, 32, 64);
    const bool labelled = qlive && y >= 0 && y < C;   // outside [0, C): unlabelled, no semantic term
    if (labelled && lane < 32) sums.ce += (m + __logf(z) - xy) * invp;
    const float sc = labelled ? w2 * invp / z : 0.0f;
    const float oh = labelled ? w2 * invp : 0.0f;
    __builtin_amdgcn_sched_barrier(0);
    v4s dhi[8], dlo[8];   // dlogits as an operand over classes, k-step ks
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = 4 * g + j;
          x[j] = Lg[cb][r] * sc - (yl == 8 * (r >> 2) + (r & 3) + 32 * cb ? oh : 0.0f);
          sg[(drow(r, lane) + 32 * cb) * kFst + l32] = x[j];
        }
        split4(x, dhi[4 * cb + g], dlo[4 * cb + g]);
      }
    __builtin_amdgcn_sched_barrier(0);
    // (2) dH^T = W2^T dlogits^T: A = W2^T (i = hidden l32 + 32 hb, k = class 8 ks + 4 half + j),
    // masked by the ReLU
    v16f dHT[2];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      __builtin_amdgcn_sched_barrier(0);
      dHT[hb] = zero16();
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const v8s a = *reinterpret_cast<const v8s*>(L.w2t + (l32 + 32 * hb) * kWtStride + 16 * s2 + 8 * half);
        dHT[hb] = mfma2(a, dhi[2 * s2], dhi[2 * s2 + 1], dHT[hb]);
        dHT[hb] = mfma2(a, dlo[2 * s2], dlo[2 * s2 + 1], dHT[hb]);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) dHT[hb][r] = H[hb][r] > 0.0f ? dHT[hb][r] : 0.0f;
    }
    __builtin_amdgcn_sched_barrier(0);
    // (3) dE^T = W1^T dH^T: A = W1^T (i = d l32, k = hidden 8 ks + 4 half + j)
    {
      v16f dE = zero16();
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        v8s a = {0, 0, 0, 0, 0, 0, 0, 0};
        if (l32 < kDin) a = *reinterpret_cast<const v8s*>(L.w1t + l32 * kWtStride + 16 * s2 + 8 * half);
        v4s hi[2], lo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int ks = 2 * s2 + u;
          float x[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) x[j] = dHT[ks >> 2][4 * (ks & 3) + j];
          split4(x, hi[u], lo[u]);
        }
        dE = mfma2(a, hi[0], hi[1], dE);
        dE = mfma2(a, lo[0], lo[1], dE);
      }
      if (qlive) {   // rows 0..15 = d
        float* dst = gcolor + ci.pixel_base * K + 4 * HW + ci.local0 + q;
#pragma unroll
        for (int r = 0; r < 8; ++r) dst[(int64_t)drow(r, lane) * HW] = dE[r];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (4) dH with pixels in registers: A = dlogits (i = pixel, k = class), B = W2 (j = hidden
    // l32 + 32 hb); H likewise: A = E (i = pixel), B = W1^T (k = d)
    v16f dH[2];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      dH[hb] = zero16();
#pragma unroll
      for (int s2 = 0; s2 < 4; ++s2) {
        const v8s b = *reinterpret_cast<const v8s*>(L.w2t + (l32 + 32 * hb) * kWtStride + 16 * s2 + 8 * half);
        dH[hb] = mfma2(dhi[2 * s2], dhi[2 * s2 + 1], b, dH[hb]);
        dH[hb] = mfma2(dlo[2 * s2], dlo[2 * s2 + 1], b, dH[hb]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      H[hb] = mfma2(ehi[0], ehi[1], w1a[hb][0], w1a[hb][1], zero16());
      H[hb] = mfma2(elo[0], elo[1], w1a[hb][0], w1a[hb][1], H[hb]);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        H[hb][r] = fmaxf(H[hb][r] + b1l[hb], 0.0f);
        dH[hb][r] = H[hb][r] > 0.0f ? dH[hb][r] : 0.0f;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    wave_sync();
    // (5) over the half's pixels p = 8 kk + 4 half + j (registers 4 kk + j):
    //  dW2[c][h] += dlogits[c][p] relu(H)[p][h], A = dlogits (i = class l32 + 32 cb, k = p);
    //  dW1[h][d] += dH[p][h] [E, 1][p][d], A = dH (i = hidden l32 + 32 hb, k = p), B = [E, 1] (j = d l32)
    const float* Ed = &S.E[min(l32, kDin - 1)][32 * pb];
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      __builtin_amdgcn_sched_barrier(0);
      v4s hhi[2][2], hlo[2][2];
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float y4[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) y4[j] = H[hb][4 * (2 * k2 + u) + j];
          split4(y4, hhi[hb][u], hlo[hb][u]);
        }
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        v4s ahi[2], alo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const float4 v = *reinterpret_cast<const float4*>(sg + (l32 + 32 * cb) * kFst + 8 * (2 * k2 + u) + 4 * half);
          const float x[4] = {v.x, v.y, v.z, v.w};
          acc.B2[cb] += (x[0] + x[1]) + (x[2] + x[3]);
          split4(x, ahi[u], alo[u]);
        }
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          acc.W2[cb][hb] = mfma2(ahi[0], ahi[1], hhi[hb][0], hhi[hb][1], acc.W2[cb][hb]);
          acc.W2[cb][hb] = mfma2(ahi[0], ahi[1], hlo[hb][0], hlo[hb][1], acc.W2[cb][hb]);
          acc.W2[cb][hb] = mfma2(alo[0], alo[1], hhi[hb][0], hhi[hb][1], acc.W2[cb][hb]);
        }
      }
      v4s bhi[2], blo[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int p0 = 8 * (2 * k2 + u) + 4 * half;
        float e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = Ed[p0 + j];
          e[j] = 32 * pb + p0 + j >= nlive ? 0.0f : (l32 < kDin ? v : (l32 == kDin ? 1.0f : 0.0f));
        }
        split4(e, bhi[u], blo[u]);
      }
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        v4s ahi[2], alo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float y4[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) y4[j] = dH[hb][4 * (2 * k2 + u) + j];
          split4(y4, ahi[u], alo[u]);
        }
        acc.W1[hb] = mfma2(ahi[0], ahi[1], bhi[0], bhi[1], acc.W1[hb]);
        acc.W1[hb] = mfma2(ahi[0], ahi[1], blo[0], blo[1], acc.W1[hb]);
        acc.W1[hb] = mfma2(alo[0], alo[1], bhi[0], bhi[1], acc.W1[hb]);
      }
    }
    wave_sync();   // the half's rows are read before the next half writes them
  }
  // L1 colour and depth, lane = pixel
  const bool live = lane < nlive;
  const int64_t cbase = ci.pixel_base * K + ci.local0 + min(lane, nlive - 1);
  float col[4], tr[3];
#pragma unroll
  for (int ch = 0; ch < 4; ++ch) col[ch] = color[cbase + ch * HW];
  const int64_t tpix = ci.local0 + min(lane, nlive - 1);
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) tr[ch] = trgb[ci.pixel_base * 3 + tpix + ch * HW];
  const float td = tdepth[ci.pixel_base + tpix];
  {
    const float inv3 = 1.0f / (3.0f * (float)HW);
    float gc[3], lr = 0.0f;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float d = col[ch] - tr[ch];
      lr += fabsf(d) * inv3;
      gc[ch] = w0 * (float)((d > 0.0f) - (d < 0.0f)) * inv3;
    }
    const float dd = col[3] - td;
    const bool valid = td > 0.0f;
    const float gd = valid ? (float)((dd > 0.0f) - (dd < 0.0f)) : 0.0f;
    if (live) {
      if (rgb_grad)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) __builtin_nontemporal_store(gc[ch], &gcolor[cbase + ch * HW]);
      __builtin_nontemporal_store(gd, &gcolor[cbase + 3 * HW]);
      sums.rgb += lr;
      sums.depth += valid ? fabsf(dd) : 0.0f;
      sums.valid += valid ? 1.0f : 0.0f;
    }
  }
}

__global__ __launch_bounds__(64 * kFusedWaves, 2) void k_head_loss(const gs_item* __restrict__ items, int n_items, int K, int C,
                                                      const float* __restrict__ color, const float* __restrict__ trgb,
                                                      const float* __restrict__ tdepth,
                                                      const int32_t* __restrict__ tlabel,
                                                      const uint16_t* __restrict__ W1, const float* __restrict__ b1,
                                                      const uint16_t* __restrict__ W2, const float* __restrict__ b2,
                                                      float w0, float w2, bool rgb_grad, int n_slots, int waves,
                                                      float* __restrict__ loss_slots, float* __restrict__ count_slots,
                                                      float* __restrict__ gcolor, float* __restrict__ partial) {
  __shared__ FusedLds L;
  __shared__ __align__(16) uint16_t w2r[kHid * kWtStride];   // W2 [class][kperm(hidden)], rows >= C zero
  __shared__ float b2s[kHid];                                // b2, minus infinity for absent classes
  __shared__ ChunkStage SA[kFusedWaves];
  __shared__ ChunkStage SB[kFusedWaves];
  // wave-uniform: the chunk walk and the item table reads stay in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = threadIdx.x; i < kHid * kHid; i += 64 * kFusedWaves) {
    const int c = i / kHid, h = i % kHid;
    w2r[c * kWtStride + kperm(h)] = c < C ? W2[c * kHid + h] : (uint16_t)0;
  }
  if (threadIdx.x < kHid) b2s[threadIdx.x] = (int)threadIdx.x < C ? b2[threadIdx.x] : -INFINITY;
  HeadAcc acc;
  v4s w1a[2][2];
  float b1l[2];
  head_setup(L, C, W1, b1, W2, acc, w1a, b1l);   // ends in a block barrier: w2r is complete
  float* sg = L.buf + wave * kHid * kFst;
  LossSums sums{0.0f, 0.0f, 0.0f, 0.0f, -1, 0};
  ConstItems citems = (ConstItems)items;
  ChunkCursor cur;
  cur.item = 0;
  cur.first = 0;
  cur.end = ((int64_t)citems[0].W * citems[0].H + 63) / 64;
  const int64_t stride = (int64_t)gridDim.x * waves;
  // Every iteration issues the same loads whether or not a next chunk exists (past the end
  // the current chunk is loaded again and not used), so the number of loads in flight is
  // the same on every path and each buffer's wait covers exactly its own loads.
  ChunkInfo ca, cb;
  bool have = wave < waves && chunk_info(citems, n_items, (int64_t)blockIdx.x * waves + wave, cur, ca);
  if (!have) {
    head_write_partial(L, acc, partial, false);
    return;
  }
  int ya = load_label(ca, tlabel), yb;
  stage_chunk(SA[wave], ca, K, color);
  for (;;) {
    const bool hb = chunk_info(citems, n_items, ca.chunk + stride, cur, cb);
    if (!hb) cb = ca;
    yb = load_label(cb, tlabel);
    stage_chunk(SB[wave], cb, K, color);
    head_loss_chunk(L, w2r, SA[wave], ca, sg, K, C, w0, w2, rgb_grad, n_slots, b2s, w1a, b1l, acc, sums, ya, color,
                    trgb, tdepth, loss_slots, count_slots, gcolor);
    if (!hb) break;
    const bool ha = chunk_info(citems, n_items, cb.chunk + stride, cur, ca);
    if (!ha) ca = cb;
    ya = load_label(ca, tlabel);
    stage_chunk(SA[wave], ca, K, color);
    head_loss_chunk(L, w2r, SB[wave], cb, sg, K, C, w0, w2, rgb_grad, n_slots, b2s, w1a, b1l, acc, sums, yb, color,
                    trgb, tdepth, loss_slots, count_slots, gcolor);
    if (!ha) break;
  }
  flush_loss(sums, n_slots, loss_slots, count_slots);
  // the last iteration's loads into the unused buffer are complete before the block's LDS
  // is reused below
  __builtin_amdgcn_s_waitcnt(0);
  head_write_partial(L, acc, partial, true);
}

// Sums the per-block partials into the head's weight gradients: block = 64 columns, sixteen
// thread groups over interleaved partials, eight loads in flight each, combined in LDS.
constexpr int kReduceGroups = 16;
__global__ __launch_bounds__(64 * kReduceGroups) void k_head_reduce(const float* __restrict__ partial, int n_blocks, int C,
                                                     float* __restrict__ gW1, float* __restrict__ gb1,
                                                     float* __restrict__ gW2, float* __restrict__ gb2) {
  __shared__ float s_sum[kReduceGroups][64];
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + col;
  float s = 0.0f;
  for (int b = grp; b < n_blocks; b += 8 * kReduceGroups) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = partial[(int64_t)min(b + u * kReduceGroups, n_blocks - 1) * kPart + min(i, kPart - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += b + u * kReduceGroups < n_blocks ? v[u] : 0.0f;
  }
  s_sum[grp][col] = s;
  __syncthreads();
  if (grp != 0 || i >= kPart) return;
  s = 0.0f;
#pragma unroll
  for (int u = 0; u < kReduceGroups; u += 4) s += (s_sum[u][col] + s_sum[u + 1][col]) + (s_sum[u + 2][col] + s_sum[u + 3][col]);
  if (i < kPartW2) {
    const int c = i / 64, h = i % 64;
    if (c < C) gW2[c * kHid + h] = s;
  } else if (i < kPartW2 + kPartW1) {
    const int h = (i - kPartW2) / 32, d = (i - kPartW2) % 32;
    if (d < kDin) gW1[h * kDin + d] = s;
    else if (d == kDin) gb1[h] = s;
  } else {
    const int c = i - kPartW2 - kPartW1;
    if (c < C) gb2[c] = s;
  }
}

}  // namespace

size_t head_bwd_workspace() { return sizeof(float) * (size_t)kHeadBlocksMax * kPart; }

int head_shape_ok(const gs_head& h) { return h.d_in == kDin && h.d_hidden == kHid && h.n_classes >= 1 && h.n_classes <= 64; }

int launch_head_fwd(const gs_item* items, int n_items, int64_t P, int K, const gs_head& h, const float* color,
                    float* logits, hipStream_t s) {
  if (P == 0) return GS_OK;
  // at most one 64-pixel chunk per item is partial, so P / 64 + n_items bounds the chunk count
  const int resident = resident_blocks(k_head_fwd, 256, 512);
  const int64_t blocks = std::min<int64_t>(resident, ceil_div(ceil_div(P, 64) + n_items, 4));
  hipLaunchKernelGGL(k_head_fwd, dim3((unsigned)blocks), dim3(256), 0, s, items, n_items, P, K, h.n_classes, color,
                     h.W1, h.b1, h.W2, h.b2, logits);
  return launch_status();
}

int launch_head_bwd(const gs_item* items, int n_items, int64_t P, int K, const gs_head& h, const float* color,
                    const float* glogits, float* gcolor, float* partial, float* gW1, float* gb1, float* gW2, float* gb2,
                    hipStream_t s) {
  if (P == 0) return GS_OK;
  // at most one 64-pixel chunk per item is partial, so P / 64 + n_items bounds the chunk count;
  // the blocks walk the chunks grid-stride, so the grid is the resident count (one wave per
  // SIMD: the register file holds the weight-gradient accumulators without spilling)
  const int resident = resident_blocks(k_head_bwd, 256, kHeadBlocksMax);
  const int blocks = (int)std::min<int64_t>(std::min(kHeadBlocksMax, resident), ceil_div(ceil_div(P, 64) + n_items, 4));
  hipLaunchKernelGGL(k_head_bwd, dim3(blocks), dim3(256), 0, s, items, n_items, K, h.n_classes, color, glogits, h.W1,
                     h.b1, h.W2, gcolor, partial);
  hipLaunchKernelGGL(k_head_reduce, dim3((unsigned)ceil_div(kPart, 64)), dim3(64 * kReduceGroups), 0, s, partial, blocks, h.n_classes,
                     gW1, gb1, gW2, gb2);
  return launch_status();
}

int launch_head_loss(const gs_item* items, int n_items, int64_t P, int K, const gs_head& h, const float* color,
                     const gs_targets& t, float w0, float w2, bool rgb_grad, int n_slots, float* loss_slots,
                     float* count_slots, float* gcolor, float* partial, float* gW1, float* gb1, float* gW2, float* gb2,
                     hipStream_t s) {
  if (P == 0) return GS_OK;
  const int resident = resident_blocks(k_head_loss, 64 * kFusedWaves, kHeadBlocksMax);
  // few chunks: half of a block's waves take them, one per SIMD, on twice the blocks. (36k pixels, 13
  // classes, the whole loss: 123 us with all eight, 85 with four, no sums from idle waves and the
  // partials added with loads in flight, 18.8 -> 4.6 us of it.)
  const int64_t chunks = ceil_div(P, 64) + n_items, most = std::min(kHeadBlocksMax, resident);
  const int waves = chunks > kFusedWaves / 2 * most ? kFusedWaves : kFusedWaves / 2;
  const int blocks = (int)std::min<int64_t>(most, ceil_div(chunks, waves));
  hipLaunchKernelGGL(k_head_loss, dim3(blocks), dim3(64 * kFusedWaves), 0, s, items, n_items, K, h.n_classes, color, t.rgb, t.depth,
                     t.label, h.W1, h.b1, h.W2, h.b2, w0, w2, rgb_grad, n_slots, waves, loss_slots, count_slots, gcolor,
                     partial);
  hipLaunchKernelGGL(k_head_reduce, dim3((unsigned)ceil_div(kPart, 64)), dim3(64 * kReduceGroups), 0, s, partial, blocks, h.n_classes,
                     gW1, gb1, gW2, gb2);
  return launch_status();
}

}  // namespace gs
