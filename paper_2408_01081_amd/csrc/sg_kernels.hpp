// Kernels of the learned window surrogate: a linear U-Net on the first-order
// system's variables with FiLM gains, 3x3 convolutions as implicit GEMMs on
// gfx950 BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
//
// Activations are FP32 NHWC ([batch][y][x][channel]).  A convolution operand
// is rounded to BF16 when it is fed to the matrix core; with SPLIT = 3 each
// FP32 operand x is carried as hi = bf16(x), lo = bf16(x - hi) and the product
// is hi*hi + lo*hi + hi*lo (about 16 significant bits instead of 8).
//
// Every stored conv output z is pre-FiLM; a consumer multiplies it by the
// layer's gain gamma[b][c] when it loads it ("scale on load"), which is also
// exactly what the backward pass needs (dL/dz = gamma * dL/dy).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace sgk {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// round-to-nearest-even FP32 -> BF16 (finite inputs)
__device__ __host__ inline unsigned short bf16_bits(float x) {
  uint32_t u;
  __builtin_memcpy(&u, &x, 4);
  u = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
  return (unsigned short)u;
}
__device__ __host__ inline float bf16_value(unsigned short b) {
  const uint32_t u = (uint32_t)b << 16;
  float f;
  __builtin_memcpy(&f, &u, 4);
  return f;
}
__device__ inline bf16 as_bf16(unsigned short b) {
  bf16 r;
  __builtin_memcpy(&r, &b, 2);
  return r;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two FP32 values rounded to nearest even to BF16 in one conversion
// instruction (v_cvt_pk_bf16_f32), a0 in the low half; bitwise bf16_bits for
// every finite input, subnormal ones included
__device__ __forceinline__ uint32_t bf16_pair(float a0, float a1) {
  const f32x2 v = {a0, a1};
  const bf16x2 h = __builtin_convertvector(v, bf16x2);
  uint32_t u;
  __builtin_memcpy(&u, &h, 4);
  return u;
}
// the pair's values (exact)
__device__ __forceinline__ float pair_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float pair_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// BF16 hi and (SPLIT = 3) lo parts of 8 values: hi = bf16(a), lo = bf16(a - hi)
template <int SPLIT>
__device__ __forceinline__ void split_pairs(const float (&a)[8], uint32_t (&h)[4],
                                            uint32_t (&l)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = bf16_pair(a[2 * j], a[2 * j + 1]);
    l[j] = SPLIT == 3 ? bf16_pair(a[2 * j] - pair_lo(h[j]), a[2 * j + 1] - pair_hi(h[j])) : 0u;
  }
}

// BF16 hi (and, SPLIT = 3, lo) parts of 8 activations times their gains,
// rounded to nearest even (a zero activation gives zero parts)
template <int SPLIT>
__device__ __forceinline__ void split8(const float (&x)[8], const float (&s)[8], bool scaled,
                                       bf16x8& hi, bf16x8& lo) {
  float a[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = scaled ? x[j] * s[j] : x[j];
  uint32_t h[4], l[4];
  split_pairs<SPLIT>(a, h, l);
  __builtin_memcpy(&hi, h, 16);
  __builtin_memcpy(&lo, l, 16);
}

// ---------------------------------------------------------------------------
// 3x3 convolution, implicit GEMM.  Z[b,y,x,o] = sum_{t,i} Wt[t][o][i] * s[b,i] * X[b,y+dy,x+dx,i]
// Operand layouts of v_mfma_f32_16x16x32_bf16 (checked on gfx950 by an
// in-bounds probe): lane l holds A[l%16][8(l/16)+j], B[8(l/16)+j][l%16] for
// j = 0..7, and D[4(l/16)+j][l%16] for j = 0..3.
// One wave computes PB blocks of 16 pixels (each one row piece, W % 16 == 0)
// x 16*NB output channels, so every weight fragment feeds PB products.  The
// 4 waves of a workgroup are 4/KS pixel groups x KS slices of the reduction
// (input-channel chunks of 32 taken round robin); the KS partial sums are
// added in LDS in slice order, so the result does not depend on timing.  A
// workgroup covers 16 * PB * 4/KS pixels.  Cin % 32 == 0.
// Used for the forward pass (Wt = [9][Cout][Cin]) and, with the flipped and
// transposed weights, for the data gradient.  The input is read in FP32 and
// split into BF16 parts (split8) with its gain as it is read.
// ---------------------------------------------------------------------------
template <int SPLIT, int NB, int PB, int KS>
__global__ __launch_bounds__(256) void k_conv(const float* __restrict__ X,
                                              const float* __restrict__ xscale,
                                              const unsigned short* __restrict__ Whi,
                                              const unsigned short* __restrict__ Wlo,
                                              float* __restrict__ Z, int H, int W, int Cin,
                                              int Cout, int circular, int accumulate) {
  static_assert(KS == 1 || KS == 2 || KS == 4, "reduction slices per workgroup");
  constexpr int PG = 4 / KS;  // pixel groups per workgroup
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int pg = wave / KS, ks = wave % KS;
  const int64_t HW = (int64_t)H * W;
  const int m = lane & 15, kq = lane >> 4;
  const int co0 = blockIdx.y * 16 * NB;
  int64_t pix0[PB];
  int bb[PB], yy[PB], xx[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    pix0[pb] = ((int64_t)blockIdx.x * PG * PB + pg * PB + pb) * 16;
    bb[pb] = (int)(pix0[pb] / HW);
    const int rem = (int)(pix0[pb] - (int64_t)bb[pb] * HW);
    yy[pb] = rem / W;
    xx[pb] = rem - yy[pb] * W + m;
  }
  f32x4 acc[PB][NB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[pb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};

  for (int c0 = 32 * ks; c0 < Cin; c0 += 32 * KS) {
    // the gains of this lane's 8 input channels in each pixel block's image
    float sc[PB][8];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int j = 0; j < 8; ++j)
        sc[pb][j] = xscale ? xscale[(int64_t)bb[pb] * Cin + c0 + 8 * kq + j] : 1.f;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dy = t / 3 - 1, dx = t % 3 - 1;
      bf16x8 ahi[PB], alo[PB];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        int ys = yy[pb] + dy, xs = xx[pb] + dx;
        bool valid = true;
        if (circular) {
          ys = ys < 0 ? ys + H : (ys >= H ? ys - H : ys);
          xs = xs < 0 ? xs + W : (xs >= W ? xs - W : xs);
        } else {
          valid = ys >= 0 && ys < H && xs >= 0 && xs < W;
          ys = ys < 0 ? 0 : (ys >= H ? H - 1 : ys);
          xs = xs < 0 ? 0 : (xs >= W ? W - 1 : xs);
        }
        const int64_t xo = (((int64_t)bb[pb] * H + ys) * W + xs) * Cin + 8 * kq + c0;
        float4 u0 = {0.f, 0.f, 0.f, 0.f}, u1 = {0.f, 0.f, 0.f, 0.f};
        if (valid) {
          u0 = *reinterpret_cast<const float4*>(X + xo);
          u1 = *reinterpret_cast<const float4*>(X + xo + 4);
        }
        const float a[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        split8<SPLIT>(a, sc[pb], xscale != nullptr, ahi[pb], alo[pb]);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int64_t wo = ((int64_t)t * Cout + co0 + 16 * nb + m) * Cin + 8 * kq + c0;
        const bf16x8 bhi = *reinterpret_cast<const bf16x8*>(Whi + wo);
        bf16x8 blo;
        if (SPLIT == 3) blo = *reinterpret_cast<const bf16x8*>(Wlo + wo);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[pb], bhi, acc[pb][nb], 0, 0, 0);
          if (SPLIT == 3) {
            acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[pb], bhi, acc[pb][nb], 0, 0, 0);
            acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[pb], blo, acc[pb][nb], 0, 0, 0);
          }
        }
      }
    }
  }
  if (KS > 1) {
    // slices 1..KS-1 hand their sums to slice 0 of the same pixel group
    __shared__ f32x4 red[KS > 1 ? 4 : 1][PB * NB][64];
    if (ks > 0) {
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) red[wave][pb * NB + nb][lane] = acc[pb][nb];
    }
    __syncthreads();
    if (ks > 0) return;
#pragma unroll
    for (int k = 1; k < KS; ++k)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const f32x4 r = red[wave + k][pb * NB + nb][lane];
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[pb][nb][j] += r[j];
        }
  }
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float* zp = Z + (pix0[pb] + 4 * kq + j) * Cout + co0 + 16 * nb + m;
        *zp = accumulate ? *zp + acc[pb][nb][j] : acc[pb][nb][j];
      }
}

// ---------------------------------------------------------------------------
// The same convolution with the input tile staged in LDS.  A workgroup computes
// a block of RW rows x WT pixels of one image (WT = 64 with W % 64 == 0, or
// WT = W = 32 or 16; RW * WT = 64) x CT output channels; for every
// 32-channel chunk of the input the neighbourhood of those pixels (one pixel
// more on every side) is read from the FP32 activations, multiplied by the gain and
// split into BF16 hi and lo parts exactly as split8 does, and stored in
// LDS (20 dwords per pixel: 16 data + 4 padding, so the 16 lanes of an
// A-fragment read hit distinct banks), where all 9 taps and all waves read it.  Wave w owns 16 PB pixels (w mod WPX) x
// 16 NB output channels (w / WPX).  The products are accumulated in the same
// order as k_conv<SPLIT, NB, PB, 1> (chunks, taps, channel blocks, pixel
// blocks), so the two give bitwise identical results.  Cin % 32 == 0,
// Cout % CT == 0.
// ---------------------------------------------------------------------------
template <int SPLIT, int PB, int NB, bool WL, int WT>
__global__ __launch_bounds__(256) void k_convt(const float* __restrict__ X,
                                               const float* __restrict__ xscale,
                                               const unsigned short* __restrict__ Whi,
                                               const unsigned short* __restrict__ Wlo,
                                               float* __restrict__ Z, int H, int W, int Cin,
                                               int Cout, int circular, int accumulate) {
  // the workgroup's pixels: RW rows of WT pixels (WT = 64 for W >= 64, else W)
  constexpr int RW = 64 / WT, NPX = RW * WT;
  constexpr int WPX = NPX / (16 * PB);  // waves along the pixels
  constexpr int WCO = 4 / WPX;          // waves along the output channels
  static_assert(WPX * WCO == 4 && NPX % (16 * PB) == 0, "four waves per workgroup");
  constexpr int CT = WCO * 16 * NB;     // output channels per workgroup
  constexpr int TR = RW + 2;           // tile rows: those rows + one each side
  constexpr int TW = WT + 2;           // tile columns: WT pixels + one each side
  constexpr int PS = 20;               // dwords per tile pixel
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  // WL: the chunk's weights of the workgroup's CT channels for all 9 taps
  // are staged in LDS as well ([hi/lo][tap][channel], PS dwords per channel)
  constexpr int WS = WL ? 9 * CT * PS : 0;
  __shared__ uint4 tile4[NH * (TR * TW * PS + WS) / 4];
  uint32_t* tile = reinterpret_cast<uint32_t*>(tile4);
  uint32_t* wtile = tile + NH * TR * TW * PS;

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const int wp = wave % WPX, wc = wave / WPX;
  // the workgroup's block: rows y .. y + RW - 1, columns x0 .. x0 + WT - 1
  const int tx = W / WT, tiles = (H / RW) * tx;
  const int b = (int)(blockIdx.x / (unsigned)tiles);
  const int rem = (int)(blockIdx.x - (unsigned)b * (unsigned)tiles);
  const int y = (rem / tx) * RW, x0 = (rem - (rem / tx) * tx) * WT;
  const int cw = 16 * NB * wc;  // the wave's channels within the workgroup's CT
  const int co0 = blockIdx.y * CT + cw;
  const int px0 = 16 * PB * wp;

  f32x4 acc[PB][NB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[pb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // staging: thread t handles the items t, t + 256, ... of the tile (and of
  // the weights); 256 is a multiple of 4, so its piece q of 8 channels is
  // the same in every item.  A chunk's loads (input tile, gains, weights)
  // are all issued before the first is used, so their latencies overlap, and
  // those of the next chunk are in flight during this chunk's products.
  constexpr int NTILE = TR * TW * 4, PER = (NTILE + 255) / 256;
  constexpr int NWT = WL ? 9 * CT * 4 : 1, PERW = (NWT + 255) / 256;
  const int q = threadIdx.x & 3;
  float4 u0[PER], u1[PER];
  bool valid[PER];
  float sc[8];
  // (dword arrays: arrays of uint4 were placed in scratch memory)
  uint32_t wh[WL ? PERW : 1][4], wl[WL ? PERW : 1][4];
  auto issue = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      const int col = (i >> 2) % TW, row = (i >> 2) / TW;
      int ys = y + row - 1, xs = x0 + col - 1;
      bool v = i < NTILE;
      if (circular) {
        ys = ys < 0 ? ys + H : (ys >= H ? ys - H : ys);
        xs = xs < 0 ? xs + W : (xs >= W ? xs - W : xs);
      } else {
        v = v && ys >= 0 && ys < H && xs >= 0 && xs < W;
      }
      valid[k] = v;
      if (v) {
        const int64_t xo = (((int64_t)b * H + ys) * W + xs) * Cin + c0 + 8 * q;
        u0[k] = *reinterpret_cast<const float4*>(X + xo);
        u1[k] = *reinterpret_cast<const float4*>(X + xo + 4);
      }
    }
    if (xscale) {
      const float* sp = xscale + (int64_t)b * Cin + c0 + 8 * q;
#pragma unroll
      for (int j = 0; j < 8; ++j) sc[j] = sp[j];
    }
    if (WL) {
      // 9 taps x CT channels x 4 pieces of 8 input channels (from L2: every
      // workgroup reads the same weights)
#pragma unroll
      for (int k = 0; k < PERW; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < NWT) {
          const int co = (i >> 2) % CT, t = (i >> 2) / CT;
          const int64_t wo = ((int64_t)t * Cout + blockIdx.y * CT + co) * Cin + c0 + 8 * q;
          const uint4 a = *reinterpret_cast<const uint4*>(Whi + wo);
          wh[k][0] = a.x; wh[k][1] = a.y; wh[k][2] = a.z; wh[k][3] = a.w;
          if (SPLIT == 3) {
            const uint4 c = *reinterpret_cast<const uint4*>(Wlo + wo);
            wl[k][0] = c.x; wl[k][1] = c.y; wl[k][2] = c.z; wl[k][3] = c.w;
          }
        }
      }
    }
  };
  issue(0);
  for (int c0 = 0; c0 < Cin; c0 += 32) {
    if (c0) __syncthreads();  // every wave is done with the previous chunk
    // TR rows x TW columns x 4 pieces of 8 channels, hi (and lo)
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (k + 1 < PER || i < NTILE) {
      const int col = (i >> 2) % TW, row = (i >> 2) / TW;
      uint4 vh = {0u, 0u, 0u, 0u}, vl = {0u, 0u, 0u, 0u};
      if (valid[k]) {
        float a[8] = {u0[k].x, u0[k].y, u0[k].z, u0[k].w, u1[k].x, u1[k].y, u1[k].z, u1[k].w};
        if (xscale) {
#pragma unroll
          for (int j = 0; j < 8; ++j) a[j] *= sc[j];
        }
        uint32_t h[4], l[4];
        split_pairs<SPLIT>(a, h, l);
        vh = (uint4){h[0], h[1], h[2], h[3]};
        if (SPLIT == 3) vl = (uint4){l[0], l[1], l[2], l[3]};
      }
      const int d = (row * TW + col) * PS + 4 * q;
      *reinterpret_cast<uint4*>(tile + d) = vh;
      if (SPLIT == 3) *reinterpret_cast<uint4*>(tile + TR * TW * PS + d) = vl;
      }
    }
    if (WL) {
#pragma unroll
      for (int k = 0; k < PERW; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < NWT) {
          const int co = (i >> 2) % CT, t = (i >> 2) / CT;
          const int d = (t * CT + co) * PS + 4 * q;
          *reinterpret_cast<uint4*>(wtile + d) = (uint4){wh[k][0], wh[k][1], wh[k][2], wh[k][3]};
          if (SPLIT == 3)
            *reinterpret_cast<uint4*>(wtile + WS + d) = (uint4){wl[k][0], wl[k][1], wl[k][2], wl[k][3]};
        }
      }
    }
    if (c0 + 32 < Cin) issue(c0 + 32);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int dy = t / 3 - 1, dx = t % 3 - 1;
      bf16x8 ahi[PB], alo[PB];
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const int p = px0 + 16 * pb + m, r = p / WT, xp = p - r * WT;
        const int d = ((r + dy + 1) * TW + xp + dx + 1) * PS + 4 * kq;
        ahi[pb] = *reinterpret_cast<const bf16x8*>(tile + d);
        if (SPLIT == 3) alo[pb] = *reinterpret_cast<const bf16x8*>(tile + TR * TW * PS + d);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        bf16x8 bhi, blo;
        if (WL) {
          const int d = (t * CT + cw + 16 * nb + m) * PS + 4 * kq;
          bhi = *reinterpret_cast<const bf16x8*>(wtile + d);
          if (SPLIT == 3) blo = *reinterpret_cast<const bf16x8*>(wtile + WS + d);
        } else {
          const int64_t wo = ((int64_t)t * Cout + co0 + 16 * nb + m) * Cin + 8 * kq + c0;
          bhi = *reinterpret_cast<const bf16x8*>(Whi + wo);
          if (SPLIT == 3) blo = *reinterpret_cast<const bf16x8*>(Wlo + wo);
        }
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[pb], bhi, acc[pb][nb], 0, 0, 0);
          if (SPLIT == 3) {
            acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo[pb], bhi, acc[pb][nb], 0, 0, 0);
            acc[pb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi[pb], blo, acc[pb][nb], 0, 0, 0);
          }
        }
      }
    }
  }
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = px0 + 16 * pb + 4 * kq + j, r = p / WT, xp = p - r * WT;
        const int64_t pix = ((int64_t)b * H + y + r) * W + x0 + xp;
        float* zp = Z + pix * Cout + co0 + 16 * nb + m;
        *zp = accumulate ? *zp + acc[pb][nb][j] : acc[pb][nb][j];
      }
}

// dword of 16-byte piece q of staged row p (k_convw, k_convs)
__device__ __forceinline__ int swz(int p, int q) { return 16 * p + 4 * (q ^ ((p >> 1) & 3)); }

struct Mat {
  float cK, cm, rho;
};
__device__ inline Mat material(const float* in, int64_t HW, int64_t p) {
  const float lam = in[5 * HW + p], mu = in[6 * HW + p], rho = in[7 * HW + p];
  Mat m;
  m.cK = sqrtf((lam + mu) / rho);
  m.cm = sqrtf(mu / rho);
  m.rho = rho;
  return m;
}
__device__ inline void phys_to_U(const float* f, int64_t HW, int64_t p, const Mat& m,
                                 float U[5]) {
  const float sxx = f[2 * HW + p] / m.rho, syy = f[3 * HW + p] / m.rho,
              sxy = f[4 * HW + p] / m.rho;
  U[0] = f[p];
  U[1] = f[HW + p];
  U[2] = -(sxx + syy) / (2.f * m.cK);
  U[3] = -(sxx - syy) / (2.f * m.cm);
  U[4] = -sxy / m.cm;
}

// physical output fields of a pixel from U
__device__ inline void U_to_phys(const float U[5], float* o, int64_t HW, int64_t p, const Mat& m) {
  o[p] = U[0];
  o[HW + p] = U[1];
  o[2 * HW + p] = -m.rho * (m.cK * U[2] + m.cm * U[3]);
  o[3 * HW + p] = -m.rho * (m.cK * U[2] - m.cm * U[3]);
  o[4 * HW + p] = -m.rho * (m.cm * U[4]);
}

// ---------------------------------------------------------------------------
// Scale, Chebyshev values and FiLM gains of a sample
// ---------------------------------------------------------------------------
constexpr int NBASIS = 4;
constexpr int NLAYER = 16;
constexpr double THETA_LO = 8.0 * M_PI / 180.0;
constexpr double THETA_HI = 45.0 * M_PI / 180.0;

// partial sums per sample: a pixel per thread up to 256 workgroups
inline int stats_chunks(int64_t HW) { return (int)(HW < 65536 ? (HW + 255) / 256 : 256); }

struct SampleStats {
  const double* part;  // [B][chunks][3]: sums of |U|^2, c_K, c_mu
  int chunks, HW;
  float* s;  // [B]
  float* T;  // [B][NBASIS]
  const float* a[NLAYER];  // gain coefficients [cout][NBASIS] of the layers
  float* g[NLAYER];        // gains [B][cout]: sum_k a[c][k] T[b][k]
  int cout[NLAYER];        // <= 128
};

// the sum over a wave, in every lane
__device__ __forceinline__ double wave_total(double v) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k, 64);
  return v;
}

// sum j of sample b's partial sums, in every lane
__device__ __forceinline__ double sample_sum(const SampleStats& st, int b, int j) {
  const double* q = st.part + (int64_t)b * st.chunks * 3 + j;
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = (int)(threadIdx.x & 63) + 64 * k;
    v[k] = i < st.chunks ? q[3 * i] : 0.0;
  }
  return wave_total((v[0] + v[1]) + (v[2] + v[3]));
}

__device__ __forceinline__ float sample_scale(double u2, int HW) {
  const double s = sqrt(u2 / (5.0 * HW));
  return (float)(s > 0 ? s : 1.0);
}

// A workgroup of 256 for sample b.  A chain of latencies: the coefficients are
// loaded before the sums that T needs, and every wave forms T itself.
__device__ __forceinline__ void sample_stats(const SampleStats& st, int b) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  float a[NLAYER / 4][2][NBASIS];
#pragma unroll
  for (int i = 0; i < NLAYER / 4; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int l = wave + 4 * i, c = lane + 64 * h;
      const float* p = st.a[l] + (c < st.cout[l] ? c : 0) * NBASIS;
#pragma unroll
      for (int k = 0; k < NBASIS; ++k) a[i][h][k] = p[k];
    }
  const double u2 = sample_sum(st, b, 0), ck = sample_sum(st, b, 1), cm = sample_sum(st, b, 2);
  const double th = atan2(cm, ck);
  const double t = 2.0 * (th - THETA_LO) / (THETA_HI - THETA_LO) - 1.0;
  double Tm[NBASIS];
  Tm[0] = 1.0;
  Tm[1] = t;
#pragma unroll
  for (int k = 2; k < NBASIS; ++k) Tm[k] = 2.0 * t * Tm[k - 1] - Tm[k - 2];
  if (threadIdx.x == 0) {
    st.s[b] = sample_scale(u2, st.HW);
#pragma unroll
    for (int k = 0; k < NBASIS; ++k) st.T[b * NBASIS + k] = (float)Tm[k];
  }
#pragma unroll
  for (int i = 0; i < NLAYER / 4; ++i)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int l = wave + 4 * i, c = lane + 64 * h;
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < NBASIS; ++k) s = fmaf(a[i][h][k], (float)Tm[k], s);
      if (c < st.cout[l]) st.g[l][b * st.cout[l] + c] = s;
    }
}

// What a workgroup does with its sums besides (or instead of) writing Z: the
// 2 x 2 pooling or the up-sampled skip sum of the layer's output, or the map
// to the physical output fields, which as kernels of their own read Z back
// (batch 32, 128 x 128: 27 us of pooling, 42 of skip sums and 16 of output
// map per forward pass); one by one the operations of k_pool, k_upadd and
// k_post.  EPI_POST is the network's last layer: only its first 16 output
// channels are computed (5 are used).
// EPI_FILM (backward): Z is dL/dy of the layer before, whose FiLM gain
// gradient sum_p dL/dy z it forms per tile and channel (FP64, fixed order)
// (batch 32, 128 x 128, 32 channels: 39.0 us against 31.5 and a kernel of 16.7
// that reads both tensors).
enum { EPI_NONE = 0, EPI_POOL = 1, EPI_UP = 2, EPI_POST = 3, EPI_FILM = 4 };
struct ConvEpi {
  float* out;          // pooled [B][H/2][W/2][Cout], up-sampled [B][2H][2W][Cout] or fields
  const float* gain;   // this layer's gains [B][Cout]
  const float* skip;   // [B][2H][2W][Cout] (EPI_UP), z [B][H][W][Cout] (EPI_FILM)
  const float* sgain;  // the skip's gains [B][Cout]
  const float* in;     // the network's input (EPI_POST)
  const float* sv;     // its samples' RMS
  int store;           // write Z as well (EPI_POOL, EPI_UP)
  double* part;        // [B][H W / 256][Cout] (EPI_FILM)
};

// the value of the lane holding the other pixel of a horizontal pair (m ^ 1)
__device__ __forceinline__ float lane_pair(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xb1, 0xf, 0xf, true));
}

// A wave's sums: 4 rows from yy on, the lane's column xx, channels co + 16 nb
// .. + 3 (lane 16 kq + m: channels 4 kq .. of 16, pixel m).  PRE: the skip
// values of EPI_UP are in pre[row][pixel of 2 x 2].
template <int EPI, int NB, bool PRE = false>
__device__ __forceinline__ void conv_epilogue(const f32x4 (&acc)[4][NB], float* __restrict__ Z,
                                              const ConvEpi& E, int b, int yy, int xx, int m,
                                              int kq, int co, int H, int W, int Cout,
                                              const f32x4 (*pre)[4] = nullptr) {
  if (EPI == EPI_NONE || EPI == EPI_FILM || (EPI != EPI_POST && E.store)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* zp = Z + (((int64_t)b * H + yy + r) * W + xx) * Cout + co;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4*>(zp + 16 * nb) = acc[r][nb];
    }
  }
  if constexpr (EPI == EPI_POST) {
    // lane (m, kq) takes pixel m of row kq: channels 0 .. 3 are in lane m,
    // channel 4 in lane 16 + m
    float z[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const float v = __shfl(acc[r][0][c & 3], c < 4 ? m : 16 + m, 64);
        z[c] = kq == r ? v : z[c];
      }
    const int64_t HW = (int64_t)H * W, p = (int64_t)(yy + kq) * W + xx;
    const float* f = E.in + (int64_t)b * 8 * HW;
    const Mat mt = material(f, HW, p);
    float U[5];
    phys_to_U(f, HW, p, mt, U);
    const float* gp = E.gain + (int64_t)b * Cout;
    const float sv = E.sv[b];
#pragma unroll
    for (int c = 0; c < 5; ++c) U[c] = U[c] + sv * (gp[c] * z[c]);
    U_to_phys(U, E.out + (int64_t)b * 5 * HW, HW, p, mt);
  } else if constexpr (EPI == EPI_POOL || EPI == EPI_UP) {
    f32x4 gn[NB], sg[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      gn[nb] = *reinterpret_cast<const f32x4*>(E.gain + (int64_t)b * Cout + co + 16 * nb);
      if (EPI == EPI_UP)
        sg[nb] = *reinterpret_cast<const f32x4*>(E.sgain + (int64_t)b * Cout + co + 16 * nb);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        if constexpr (EPI == EPI_POOL) {
          if (r & 1) continue;
          const int64_t px = ((int64_t)b * (H / 2) + (yy + r) / 2) * (W / 2) + xx / 2;
          f32x4 o;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float p = acc[r][nb][j] + lane_pair(acc[r][nb][j]);
            const float q = acc[r + 1][nb][j] + lane_pair(acc[r + 1][nb][j]);
            o[j] = 0.25f * gn[nb][j] * (p + q);
          }
          if (!(m & 1)) *reinterpret_cast<f32x4*>(E.out + px * Cout + co + 16 * nb) = o;
        } else {
          const int64_t p0 = ((int64_t)b * 2 * H + 2 * (yy + r)) * 2 * W + 2 * xx;
          f32x4 k[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            k[e] = PRE ? pre[r][e]
                       : *reinterpret_cast<const f32x4*>(
                             E.skip + (p0 + (e >> 1) * 2 * W + (e & 1)) * Cout + co + 16 * nb);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            f32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              o[j] = gn[nb][j] * acc[r][nb][j] + sg[nb][j] * k[e][j];
            *reinterpret_cast<f32x4*>(E.out + (p0 + (e >> 1) * 2 * W + (e & 1)) * Cout + co +
                                      16 * nb) = o;
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same convolution for layers with many pixels: a workgroup computes RW x
// WT = 256 pixels x CT = 32 output channels, each of its 4 waves 4 rows of 16
// pixels x all CT channels, so that a weight fragment read from LDS feeds 64
// pixels and a pixel fragment CT channels of up to three taps.  Input tile
// and weights of a 32-channel chunk (9 taps x CT channels) are both in LDS,
// 16 dwords per pixel and per channel row, whose 16-byte pieces are rotated
// by the row (swz) so that fragment reads meet no bank conflicts without
// padding: 80 KB, so two workgroups share a CU and one's staging runs beside
// the other's products.  Workgroups run through their tiles (tile, chunk) by
// (tile, chunk): the next chunk's or tile's loads are in registers while this
// one's products run, and with one chunk and Cout = CT the weights are staged
// once per workgroup.  The weights are the A operand, so a lane ends up with
// 4 consecutive channels of a pixel and stores 16 bytes.  Cin % 32 == 0,
// Cout % CT == 0, H % RW == 0, W % WT == 0.
// Bound by the matrix cores: a layer of 29 GFLOP in three passes (batch 32,
// 128 x 128: 32 channels at full, 64 at half, 128 at quarter resolution)
// takes 33.7 us, 860 TFLOP/s; k_convt took 58, 52 and 77.  Measured on the
// way: one workgroup of 4 waves x 64 channels per CU 37.5 us (its waves stage,
// wait and multiply one after the other), 8 waves on 512 pixels 39.5 us.
// ---------------------------------------------------------------------------
template <int SPLIT, int WT, int EPI>
__global__ __launch_bounds__(256, 2) void k_convw(const float* __restrict__ X,
                                                  const float* __restrict__ xscale,
                                                  const unsigned short* __restrict__ Whi,
                                                  const unsigned short* __restrict__ Wlo,
                                                  float* __restrict__ Z, int H, int W, int Cin,
                                                  int Cout, int circular, int nwork, ConvEpi E) {
  constexpr int NB = EPI == EPI_POST ? 1 : 2, CT = 16 * NB;
  constexpr int RW = 256 / WT;  // rows of a tile
  constexpr int TR = RW + 2, TW = WT + 2;
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  constexpr int XS = TR * TW * 16, WS = 9 * CT * 16;  // dwords per hi/lo part
  __shared__ uint4 lds4[NH * (XS + WS) / 4];
  __shared__ double red[EPI == EPI_FILM ? 4 : 1][32];
  uint32_t* tile = reinterpret_cast<uint32_t*>(lds4);
  uint32_t* wtile = tile + NH * XS;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m = lane & 15, kq = lane >> 4;
  const int q = threadIdx.x & 3;
  // the wave's pixels: 4 rows of 16, from (wx, wy) of the tile
  const int wx = 16 * (wave % (WT / 16)), wy = 4 * (wave / (WT / 16));

  // work items (pixel tile, channel block) in runs per XCD, whose L2 then
  // serves the halo rows and the channel blocks of a pixel tile
  const int ncb = EPI == EPI_POST ? 1 : Cout / CT, tx = W / WT, tiles = (H / RW) * tx;
  const int xcd = blockIdx.x & 7, nq = nwork >> 3, nr = nwork & 7;
  const int first = xcd * nq + (xcd < nr ? xcd : nr), count = nq + (xcd < nr ? 1 : 0);
  const int stride = (gridDim.x + 7 - xcd) >> 3;  // workgroups of this XCD's run
  const bool keep_w = Cin == 32 && ncb == 1;

  constexpr int NTILE = TR * TW * 4, PER = (NTILE + 255) / 256;
  constexpr int NWT = 9 * CT * 4, PERW = (NWT + 255) / 256;
  int off[PER];   // each staged piece's place in the image, in pieces of 8 channels
  uint32_t live;  // bit k: piece k is inside the image (else zero)
  float u[PER][8];
  float sc[8];
  uint32_t wh[PERW][4], wl[SPLIT == 3 ? PERW : 1][4];

  auto place = [&](int item, int& b, int& y, int& x0, int& cb) __attribute__((always_inline)) {
    const int pt = item / ncb;
    cb = item - pt * ncb;
    b = pt / tiles;
    const int rem = pt - b * tiles;
    y = (rem / tx) * RW;
    x0 = (rem - (rem / tx) * tx) * WT;
  };
  auto offsets = [&](int y, int x0) __attribute__((always_inline)) {
    live = 0u;
    // (rows and columns recomputed for every tile: kept, they would spill)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = tid + 256 * k;
      const int row = (i >> 2) / TW, col = (i >> 2) - row * TW;
      const int yr = y + row - 1, xr = x0 + col - 1;
      // wrapped (at most one period; rows past the tile's end too)
      const int ys = yr < 0 ? yr + H : (yr >= H ? yr - H : yr);
      const int xs = xr < 0 ? xr + W : (xr >= W ? xr - W : xr);
      const bool v = i < NTILE && (circular || (ys == yr && xs == xr));
      live |= v ? 1u << k : 0u;
      off[k] = v ? (ys * W + xs) * (Cin >> 3) + q : 0;
    }
  };
  auto fetch = [&](int b, int c0) __attribute__((always_inline)) {
    const float* xb = X + (int64_t)b * H * W * Cin + c0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const float* xp = xb + 8 * (int64_t)off[k];
      const float4 a = *reinterpret_cast<const float4*>(xp);
      const float4 c = *reinterpret_cast<const float4*>(xp + 4);
      u[k][0] = a.x; u[k][1] = a.y; u[k][2] = a.z; u[k][3] = a.w;
      u[k][4] = c.x; u[k][5] = c.y; u[k][6] = c.z; u[k][7] = c.w;
    }
    if (xscale) {
      const float* sp = xscale + (int64_t)b * Cin + c0 + 8 * q;
#pragma unroll
      for (int j = 0; j < 8; ++j) sc[j] = sp[j];
    }
  };
  auto fetch_w = [&](int cb, int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < PERW; ++k) {
      const int i = (int)threadIdx.x + 256 * k;
      if (NWT % 256 == 0 || k + 1 < PERW || i < NWT) {
        const int co = (i >> 2) % CT, t = (i >> 2) / CT;
        const int wo = (t * Cout + cb * CT + co) * Cin + c0 + 8 * q;
        const uint4 a = *reinterpret_cast<const uint4*>(Whi + wo);
        wh[k][0] = a.x; wh[k][1] = a.y; wh[k][2] = a.z; wh[k][3] = a.w;
        if (SPLIT == 3) {
          const uint4 c = *reinterpret_cast<const uint4*>(Wlo + wo);
          wl[k][0] = c.x; wl[k][1] = c.y; wl[k][2] = c.z; wl[k][3] = c.w;
        }
      }
    }
  };

  f32x4 acc[4][NB];
  int k0 = blockIdx.x >> 3;
  if (k0 >= count) return;  // uniform: the whole workgroup
  int b, y, x0, cb;
  place(first + k0, b, y, x0, cb);
  offsets(y, x0);
  fetch(b, 0);
  fetch_w(cb, 0);
  bool stage_w = true;
  for (int c0 = 0;;) {
    // this chunk's operands: registers -> LDS
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = (int)threadIdx.x + 256 * k;
      if (NTILE % 256 == 0 || k + 1 < PER || i < NTILE) {
        float a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          a[j] = xscale ? u[k][j] * sc[j] : u[k][j];
          a[j] = live >> k & 1 ? a[j] : 0.f;
        }
        uint32_t h[4], l[4];
        split_pairs<SPLIT>(a, h, l);
        const int d = swz(i >> 2, q);
        *reinterpret_cast<uint4*>(tile + d) = (uint4){h[0], h[1], h[2], h[3]};
        if (SPLIT == 3) *reinterpret_cast<uint4*>(tile + XS + d) = (uint4){l[0], l[1], l[2], l[3]};
      }
    }
    if (stage_w) {
#pragma unroll
      for (int k = 0; k < PERW; ++k) {
        const int i = (int)threadIdx.x + 256 * k;
        if (NWT % 256 == 0 || k + 1 < PERW || i < NWT) {
          const int d = swz(i >> 2, q);
          *reinterpret_cast<uint4*>(wtile + d) = (uint4){wh[k][0], wh[k][1], wh[k][2], wh[k][3]};
          if (SPLIT == 3)
            *reinterpret_cast<uint4*>(wtile + WS + d) = (uint4){wl[k][0], wl[k][1], wl[k][2], wl[k][3]};
        }
      }
    }
    if (c0 == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[r][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    // the next chunk, or the first of the next tile, is fetched meanwhile
    const bool last = c0 + 32 >= Cin;
    const int kn = last ? k0 + stride : k0, cn = last ? 0 : c0 + 32;
    const bool more = kn < count;
    int bn = b, yn = y, xn = x0, cbn = cb;
    if (more) {
      if (last) {
        place(first + kn, bn, yn, xn, cbn);
        offsets(yn, xn);
      }
      fetch(bn, cn);
      stage_w = !keep_w;
      if (stage_w) fetch_w(cbn, cn);
    }
    __syncthreads();
    if constexpr (SPLIT == 1) {
      // taps in k_conv's order: with plain BF16 operands the order of a
      // layer's sums decides roundings in every layer after it
      bf16x8 x[3][6];
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int r = 0; r < 6; ++r)
          x[dx][r] = *reinterpret_cast<const bf16x8*>(
              tile + swz((wy + r) * TW + wx + dx + m, kq));
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const bf16x8 ah =
              *reinterpret_cast<const bf16x8*>(wtile + swz(t * CT + 16 * nb + m, kq));
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, x[t % 3][r + t / 3],
                                                                 acc[r][nb], 0, 0, 0);
        }
    } else {
      // tap column by tap column: the six row fragments under it serve the
      // three tap rows of all four pixel rows
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        bf16x8 xh[6], xl[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
          const int d = swz((wy + r) * TW + wx + dx + m, kq);
          xh[r] = *reinterpret_cast<const bf16x8*>(tile + d);
          xl[r] = *reinterpret_cast<const bf16x8*>(tile + XS + d);
        }
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const int d = swz((3 * dy + dx) * CT + 16 * nb + m, kq);
            const bf16x8 ah = *reinterpret_cast<const bf16x8*>(wtile + d);
#pragma unroll
            for (int r = 0; r < 4; ++r)
              acc[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, xh[r + dy], acc[r][nb], 0, 0, 0);
            if (SPLIT == 3) {
              const bf16x8 al = *reinterpret_cast<const bf16x8*>(wtile + WS + d);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                acc[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, xl[r + dy], acc[r][nb], 0, 0, 0);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                acc[r][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, xh[r + dy], acc[r][nb], 0, 0, 0);
            }
          }
        }
      }
    }
    if (last) {
      // D[row = channel 4 kq + j][col = pixel m]
      conv_epilogue<EPI, NB>(acc, Z, E, b, y + wy, x0 + wx + m, m, kq, cb * CT + 4 * kq, H, W,
                             Cout);
      if constexpr (EPI == EPI_FILM) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));  // (lane places kept across the loop spill)
        const int ml = t & 15, kl = t >> 4 & 3;
        double s[8];  // [nb][j]
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          f32x4 z[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            z[r] = *reinterpret_cast<const f32x4*>(
                E.skip + (((int64_t)b * H + y + wy + r) * W + x0 + wx + ml) * Cout + cb * CT +
                4 * kl + 16 * nb);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            s[4 * nb + j] = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) s[4 * nb + j] += (double)acc[r][nb][j] * (double)z[r][j];
          }
        }
        // over the 16 pixels: each step halves the sums a lane holds, so lane
        // m ends with sum m / 2
#pragma unroll
        for (int k = 4, bit = 8; k >= 1; k >>= 1, bit >>= 1) {
          const bool up = ml & bit;
#pragma unroll
          for (int i = 0; i < k; ++i) {
            const double give = up ? s[i] : s[i + k], own = up ? s[i + k] : s[i];
            s[i] = own + __shfl_xor(give, bit, 64);
          }
        }
        s[0] += __shfl_xor(s[0], 1, 64);
        if (!(ml & 1)) red[wave][16 * (ml >> 3) + 4 * kl + (ml >> 1 & 3)] = s[0];
        __syncthreads();
        if (t < 32)
          E.part[((int64_t)b * tiles + (y / RW) * tx + x0 / WT) * Cout + cb * CT + t] =
              (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
      }
    }
    if (!more) return;
    __syncthreads();  // every wave is done with this chunk's operands
    k0 = kn;
    c0 = cn;
    b = bn;
    y = yn;
    x0 = xn;
    cb = cbn;
  }
}

// ---------------------------------------------------------------------------
// The same convolution for layers with few pixels, where a workgroup's chain
// of latencies is the layer's time: all NG = Cin / 32 chunks at once.  A
// workgroup of 2 NG waves computes TR x 16 pixels x 32 output channels; wave
// (g, h) takes chunk g and channels 16 h .. + 15, its weights read from global
// memory (L2) straight into fragments while the chunks of the input tile are
// loaded, converted and staged; the chunks' sums are added in LDS in chunk
// order.  W % 16 == 0, H % TR == 0.
// (Batch 1, 256 x 256: a layer of 64 x 64 pixels and 128 channels takes
// 10.2 us, one of 32 x 32 9.0, one of 128 x 128 and 64 channels 9.8; with the
// chunks one after the other 11.7, 12.0 and 10.2, and 3.4 to 4.9 for the
// pooling or skip sum.  Batch 32 of 128 x 128, 16 x 16 pixels and 128 channels:
// TR = 8 14.5 us, TR = 4 19.8, one after the other 18.2.)
// ---------------------------------------------------------------------------
template <int SPLIT, int NG, int TR, int EPI>
__global__ __launch_bounds__(128 * NG) void k_convs(const float* __restrict__ X,
                                                    const float* __restrict__ xscale,
                                                    const unsigned short* __restrict__ Whi,
                                                    const unsigned short* __restrict__ Wlo,
                                                    float* __restrict__ Z, int H, int W, int Cout,
                                                    int circular, ConvEpi E) {
  constexpr int Cin = 32 * NG, NT = 128 * NG, TW = 18, NPX = (TR + 2) * TW;
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  constexpr int XS = NPX * 16;  // dwords of a chunk's hi or lo part
  constexpr int SUMS = (NG - 1) * 2 * TR * 64 * 4;  // dwords of the chunks' sums
  __shared__ uint4 lds4[(NG * NH * XS > SUMS ? NG * NH * XS : SUMS) / 4];
  uint32_t* tile = reinterpret_cast<uint32_t*>(lds4);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m = lane & 15, kq = lane >> 4, q = threadIdx.x & 3;
  const int g = wave >> 1, h = wave & 1;
  const int ncb = Cout / 32, tx = W / 16, tiles = (H / TR) * tx;
  const int nt = (int)gridDim.x, xq = nt >> 3, xr = nt & 7, xcd = blockIdx.x & 7;
  const int item = xcd * xq + (xcd < xr ? xcd : xr) + (int)(blockIdx.x >> 3);
  const int pt = item / ncb, cb = item - pt * ncb;
  const int b = pt / tiles, rem = pt - b * tiles;
  const int y = (rem / tx) * TR, x0 = (rem - (rem / tx) * tx) * 16;

  // input pieces of 8 channels: (chunk, pixel, q)
  constexpr int NTILE = NG * NPX * 4, PER = (NTILE + NT - 1) / NT;
  float u[PER][8], sc[PER][8];
  uint32_t live = 0u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = ((int)threadIdx.x + NT * k) >> 2;
    const int c = i / NPX, p = i - c * NPX, row = p / TW, col = p - row * TW;
    const int yr = y + row - 1, xr2 = x0 + col - 1;
    const int ys = yr < 0 ? yr + H : (yr >= H ? yr - H : yr);
    const int xs = xr2 < 0 ? xr2 + W : (xr2 >= W ? xr2 - W : xr2);
    const bool v = c < NG && (circular || (ys == yr && xs == xr2));
    live |= v ? 1u << k : 0u;
    const int c0 = v ? 32 * c + 8 * q : 0;
    const float* xp = X + (((int64_t)b * H + (v ? ys : 0)) * W + (v ? xs : 0)) * Cin + c0;
    const float4 a = *reinterpret_cast<const float4*>(xp), d = *reinterpret_cast<const float4*>(xp + 4);
    u[k][0] = a.x; u[k][1] = a.y; u[k][2] = a.z; u[k][3] = a.w;
    u[k][4] = d.x; u[k][5] = d.y; u[k][6] = d.z; u[k][7] = d.w;
    if (xscale) {
      const float* sp = xscale + (int64_t)b * Cin + c0;
      const float4 e = *reinterpret_cast<const float4*>(sp), f = *reinterpret_cast<const float4*>(sp + 4);
      sc[k][0] = e.x; sc[k][1] = e.y; sc[k][2] = e.z; sc[k][3] = e.w;
      sc[k][4] = f.x; sc[k][5] = f.y; sc[k][6] = f.z; sc[k][7] = f.w;
    }
  }
  bf16x8 ah[9], al[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int wo = (t * Cout + cb * 32 + 16 * h + m) * Cin + 32 * g + 8 * kq;
    ah[t] = *reinterpret_cast<const bf16x8*>(Whi + wo);
    if (SPLIT == 3) al[t] = *reinterpret_cast<const bf16x8*>(Wlo + wo);
  }
  // (the skip values too, where the registers hold them)
  constexpr bool PRE = EPI == EPI_UP && TR == 4;
  f32x4 pre[4][4] = {};
  if (PRE && g == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        pre[r][e] = *reinterpret_cast<const f32x4*>(
            E.skip + (((int64_t)b * 2 * H + 2 * (y + r) + (e >> 1)) * 2 * W + 2 * (x0 + m) +
                      (e & 1)) * Cout + cb * 32 + 16 * h + 4 * kq);
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = ((int)threadIdx.x + NT * k) >> 2;
    if (NTILE % NT != 0 && k + 1 == PER && i >= NG * NPX) continue;
    const int c = i / NPX, p = i - c * NPX;
    float a[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      a[j] = xscale ? u[k][j] * sc[k][j] : u[k][j];
      a[j] = live >> k & 1 ? a[j] : 0.f;
    }
    uint32_t hi[4], lo[4];
    split_pairs<SPLIT>(a, hi, lo);
    uint32_t* t = tile + c * NH * XS + swz(p, q);
    *reinterpret_cast<uint4*>(t) = (uint4){hi[0], hi[1], hi[2], hi[3]};
    if (SPLIT == 3) *reinterpret_cast<uint4*>(t + XS) = (uint4){lo[0], lo[1], lo[2], lo[3]};
  }
  __syncthreads();
  f32x4 acc[TR / 4][4][1];
#pragma unroll
  for (int r = 0; r < TR; ++r) acc[r >> 2][r & 3][0] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const uint32_t* mine = tile + g * NH * XS;
#pragma unroll
  for (int dx = 0; dx < 3; ++dx) {
    bf16x8 xh[TR + 2], xl[TR + 2];
#pragma unroll
    for (int r = 0; r < TR + 2; ++r) {
      const int d = swz(r * TW + dx + m, kq);
      xh[r] = *reinterpret_cast<const bf16x8*>(mine + d);
      if (SPLIT == 3) xl[r] = *reinterpret_cast<const bf16x8*>(mine + XS + d);
    }
#pragma unroll
    for (int part = 0; part < SPLIT; ++part)
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int r = 0; r < TR; ++r)
          acc[r >> 2][r & 3][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              part == 2 ? al[3 * dy + dx] : ah[3 * dy + dx], part == 1 ? xl[r + dy] : xh[r + dy],
              acc[r >> 2][r & 3][0], 0, 0, 0);
  }
  if (NG > 1) {
    f32x4* red = reinterpret_cast<f32x4*>(lds4);
    __syncthreads();  // the tile is no longer read
    if (g) {
#pragma unroll
      for (int r = 0; r < TR; ++r)
        red[(((g - 1) * 2 + h) * TR + r) * 64 + lane] = acc[r >> 2][r & 3][0];
    }
    __syncthreads();
    if (g) return;
#pragma unroll
    for (int k = 1; k < NG; ++k)
#pragma unroll
      for (int r = 0; r < TR; ++r)
        acc[r >> 2][r & 3][0] += red[(((k - 1) * 2 + h) * TR + r) * 64 + lane];
  }
  if (EPI == EPI_POST && h) return;  // (channels 16 .. 31 are not used)
#pragma unroll
  for (int r = 0; r < TR / 4; ++r)
    conv_epilogue<EPI, 1, PRE>(acc[r], Z, E, b, y + 4 * r, x0 + m, m, kq,
                               cb * 32 + 16 * h + 4 * kq, H, W, Cout, pre);
}

// ---------------------------------------------------------------------------
// The network's first layer from its physical input: the tile's pixels are
// mapped to U / s as they are staged (the operations of k_pre), 5 channels
// padded to 8, so a product of K = 32 holds 4 taps x 8 channels (lane group
// kq tap 4 s + kq of step s; taps 9 .. 11 have zero weights) and the layer
// takes 3 K steps instead of 9 and reads 32 B per pixel instead of 128.  Tile
// of 8 x 32 pixels x 32 channels per workgroup, waves as in k_convw.  Bound by
// the 128 B written per pixel (batch 32, 128 x 128: 25 us; input map and
// layer as two kernels 23 + 42, batch 1, 256 x 256: 7.0 us; with the scale
// summed here and one more workgroup per sample for the gains 28 and 8.1, in
// place of k_stats of 10 and 8).
// ---------------------------------------------------------------------------
template <int SPLIT>
__global__ __launch_bounds__(256) void k_conv_in(const float* __restrict__ in,
                                                 const unsigned short* __restrict__ Whi,
                                                 const unsigned short* __restrict__ Wlo,
                                                 float* __restrict__ Z, int H, int W,
                                                 int circular, int work, SampleStats st) {
  constexpr int WT = 32, RW = 8, TR = RW + 2, TW = WT + 2, NPX = TR * TW, CO = 32;
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  __shared__ uint4 xt[NH][NPX];      // 8 channels of a pixel
  __shared__ uint4 wt[NH][12 * CO];  // 8 input channels of (tap, output channel)
  if ((int)blockIdx.x >= work) {
    sample_stats(st, (int)blockIdx.x - work);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m = lane & 15, kq = lane >> 4;
  const int wx = 16 * (wave & 1), wy = 4 * (wave >> 1);
  const int tx = W / WT, tiles = (H / RW) * tx;
  const int nt = work, xq = nt >> 3, xr = nt & 7, xcd = blockIdx.x & 7;
  const int pt = xcd * xq + (xcd < xr ? xcd : xr) + (int)(blockIdx.x >> 3);
  const int b = pt / tiles, rem = pt - b * tiles;
  const int y = (rem / tx) * RW, x0 = (rem - (rem / tx) * tx) * WT;
  const int64_t HW = (int64_t)H * W;
  const float* f = in + (int64_t)b * 8 * HW;
  const float r = 1.f / sample_scale(sample_sum(st, b, 0), st.HW);
  for (int i = threadIdx.x; i < 12 * CO; i += 256) {
    const int t = i / CO, o = i - t * CO;
    uint4 h = {0u, 0u, 0u, 0u}, l = {0u, 0u, 0u, 0u};
    if (t < 9) {
      h = *reinterpret_cast<const uint4*>(Whi + (t * CO + o) * 32);
      if (SPLIT == 3) l = *reinterpret_cast<const uint4*>(Wlo + (t * CO + o) * 32);
    }
    // (channels 5 .. 7 meet zeros in the pixels)
    wt[0][i] = h;
    if (SPLIT == 3) wt[NH - 1][i] = l;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = (int)threadIdx.x + 256 * k;
    if (i >= NPX) continue;
    const int row = i / TW, col = i - row * TW;
    const int yr = y + row - 1, xr2 = x0 + col - 1;
    const int ys = yr < 0 ? yr + H : (yr >= H ? yr - H : yr);
    const int xs = xr2 < 0 ? xr2 + W : (xr2 >= W ? xr2 - W : xr2);
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (circular || (ys == yr && xs == xr2)) {
      const int64_t p = (int64_t)ys * W + xs;
      float U[5];
      phys_to_U(f, HW, p, material(f, HW, p), U);
#pragma unroll
      for (int c = 0; c < 5; ++c) a[c] = U[c] * r;
    }
    uint32_t h[4], l[4];
    split_pairs<SPLIT>(a, h, l);
    xt[0][i] = (uint4){h[0], h[1], h[2], h[3]};
    if (SPLIT == 3) xt[NH - 1][i] = (uint4){l[0], l[1], l[2], l[3]};
  }
  __syncthreads();
  f32x4 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) acc[i][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int t = 4 * s + kq, tt = t < 9 ? t : 0;
    bf16x8 xh[4], xl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int d = (wy + i + tt / 3) * TW + wx + tt % 3 + m;
      xh[i] = *reinterpret_cast<const bf16x8*>(&xt[0][d]);
      if (SPLIT == 3) xl[i] = *reinterpret_cast<const bf16x8*>(&xt[NH - 1][d]);
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const bf16x8 ah = *reinterpret_cast<const bf16x8*>(&wt[0][t * CO + 16 * nb + m]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, xh[i], acc[i][nb], 0, 0, 0);
      if (SPLIT == 3) {
        const bf16x8 al = *reinterpret_cast<const bf16x8*>(&wt[NH - 1][t * CO + 16 * nb + m]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, xl[i], acc[i][nb], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, xh[i], acc[i][nb], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float* zp = Z + (((int64_t)b * H + y + wy + i) * W + x0 + wx + m) * CO + 4 * kq;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) *reinterpret_cast<f32x4*>(zp + 16 * nb) = acc[i][nb];
  }
}

// ---------------------------------------------------------------------------
// Weight gradient.  dW[t][o][i] = sum_{b,p} G[b,p,o] * s_o[b,o] * X[b,p+off_t,i] * s_i[b,i]
// As a GEMM: D (16 o x 16 i) += A (16 o x 32 pixels) B (32 pixels x 16 i).
// grid: x = tap (9) * (Cout/16) * (Cin/(16 NI)), y = pixel split; each of the
// 4 waves takes every 4th chunk of 32 pixels of the split, the waves' sums are
// added in LDS in a fixed order and written to partial[split][t][o][i].
// ---------------------------------------------------------------------------
template <int SPLIT, int NI>
__global__ __launch_bounds__(256) void k_wgrad(const float* __restrict__ G,
                                               const float* __restrict__ gscale,
                                               const float* __restrict__ X,
                                               const float* __restrict__ xscale,
                                               float* __restrict__ partial, int B, int H, int W,
                                               int Cin, int Cout, int circular,
                                               int64_t pix_per_split) {
  __shared__ float red[4][16 * NI][16 + 1];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const int nib = Cin / (16 * NI), nob = Cout / 16;
  int id = blockIdx.x;
  const int t = id / (nob * nib);
  id -= t * nob * nib;
  const int ob = id / nib, ib = id - ob * nib;
  const int dy = t / 3 - 1, dx = t % 3 - 1;
  const int o = ob * 16 + m;  // A row for this lane
  const int64_t HW = (int64_t)H * W;
  const int64_t p_begin = (int64_t)blockIdx.y * pix_per_split;
  f32x4 acc[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) acc[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int64_t pc = p_begin + 32 * wave; pc < p_begin + pix_per_split; pc += 128) {
    float a[8], xv[NI][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t p = pc + 8 * kq + j;
      const int b = (int)(p / HW);
      const int r = (int)(p - (int64_t)b * HW);
      const int yy = r / W, xx = r - yy * W;
      a[j] = G[p * Cout + o] * (gscale ? gscale[(int64_t)b * Cout + o] : 1.f);
      int ys = yy + dy, xs = xx + dx;
      bool valid = true;
      if (circular) {
        ys = ys < 0 ? ys + H : (ys >= H ? ys - H : ys);
        xs = xs < 0 ? xs + W : (xs >= W ? xs - W : xs);
      } else {
        valid = ys >= 0 && ys < H && xs >= 0 && xs < W;
        ys = ys < 0 ? 0 : (ys >= H ? H - 1 : ys);
        xs = xs < 0 ? 0 : (xs >= W ? W - 1 : xs);
      }
      const float* xp = X + (((int64_t)b * H + ys) * W + xs) * Cin;
#pragma unroll
      for (int k = 0; k < NI; ++k) {
        const int i = (ib * NI + k) * 16 + m;
        float v = valid ? xp[i] : 0.f;
        if (xscale) v *= xscale[(int64_t)b * Cin + i];
        xv[k][j] = v;
      }
    }
    bf16x8 ahi, alo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned short h = bf16_bits(a[j]);
      ahi[j] = as_bf16(h);
      alo[j] = as_bf16(bf16_bits(a[j] - bf16_value(h)));
    }
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      bf16x8 bhi, blo;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned short h = bf16_bits(xv[k][j]);
        bhi[j] = as_bf16(h);
        blo[j] = as_bf16(bf16_bits(xv[k][j] - bf16_value(h)));
      }
      acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bhi, acc[k], 0, 0, 0);
      if (SPLIT == 3) {
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bhi, acc[k], 0, 0, 0);
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, blo, acc[k], 0, 0, 0);
      }
    }
  }
  // D[row = o (4kq + j)][col = i (m)]
#pragma unroll
  for (int k = 0; k < NI; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[wave][16 * k + m][4 * kq + j] = acc[k][j];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * 16 * NI; e += 256) {
    const int ii = e % (16 * NI), oo = e / (16 * NI);
    const float s = ((red[0][ii][oo] + red[1][ii][oo]) + red[2][ii][oo]) + red[3][ii][oo];
    const int i = ib * NI * 16 + ii, oabs = ob * 16 + oo;
    partial[(((int64_t)blockIdx.y * 9 + t) * Cout + oabs) * Cin + i] = s;
  }
}

// sum the pixel splits in a fixed order: grad[o][i][t] (master layout)
// The weight gradient with both operands staged in LDS, channel-major (the
// matrix core's reduction runs over pixels, which must be contiguous per
// channel): a workgroup owns a 32 x 32 (output, input channel) tile of all 9
// taps and sweeps blocks of 64 pixels, blocks blockIdx.x, blockIdx.x +
// gridDim.x, ...  A block is 64 pixels of one image row (W % 64 == 0) or
// RB = 64 / W whole rows (W = 16, 32; H % RB == 0), pixel p at row
// y + p / PW, column x0 + p % PW (PW = min(W, 64)).  Per block it stages
//   gT[h][o][p]       gamma-scaled gradient, split into hi/lo, 72 bf16 per row;
//   xT[h][d][i][r][p] the gain-scaled input at tap (r - 1, d - 1) of pixel p
//                     (three copies d = 0, 1, 2 so that every tap reads 8
//                     pixels at an aligned offset), 72 per row;
// (row strides of 36 and 108 dwords keep the 16 lanes of a fragment read on
// distinct banks).  Wave w computes the 16 x 16 sub-tile (w / 2, w mod 2) for
// all taps and writes partial[blockIdx.x][t][o][i] for k_wgrad_reduce.
template <int SPLIT>
__global__ __launch_bounds__(256) void k_wgradt(const float* __restrict__ G,
                                                const float* __restrict__ gscale,
                                                const float* __restrict__ X,
                                                const float* __restrict__ xscale,
                                                float* __restrict__ partial, int B, int H, int W,
                                                int Cin, int Cout, int circular) {
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  constexpr int RS = 72;                      // bf16 per staged row (64 + 8 padding)
  constexpr int GT = 32 * RS;                 // gT elements per hi/lo part
  constexpr int XT = 3 * 32 * 3 * RS;         // xT elements per hi/lo part
  __shared__ uint4 lds4[NH * (GT + XT) * 2 / 16];
  unsigned short* gT = reinterpret_cast<unsigned short*>(lds4);
  unsigned short* xT = gT + NH * GT;

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, kq = lane >> 4;
  const int nit = Cin / 32;
  const int o0 = (int)(blockIdx.y / (unsigned)nit) * 32, i0 = (int)(blockIdx.y % (unsigned)nit) * 32;
  const int ow = 16 * (wave >> 1), iw = 16 * (wave & 1);
  const int PW = W < 64 ? W : 64;   // pixels of a block per image row
  const int RB = 64 / PW;           // image rows per block
  const int tx = W / PW;            // blocks across a row
  const int HB = H / RB;            // block rows per image
  const int64_t nblocks = (int64_t)B * HB * tx;

  f32x4 acc[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // A block's operands pass through registers: the next block's loads are
  // issued before this block's matrix-core phase and written to LDS after
  // it, so their latency hides behind the products (one workgroup per CU).
  // Input: halo rows hr = 0 .. RB + 1 (image y - 1 + hr), halo columns
  // hc = 0 .. PW + 1 (image x0 - 1 + hc), 4 x 8 channels per element, at
  // most 4 elements per thread ((RB + 2) (PW + 2) 4 <= 1024 for 64 % W == 0
  // or W % 64 == 0); each element is tap (r - 1, d - 1) of the pixels at row
  // hr - r, column hc - d.
  const int HC = PW + 2;
  const int NIT = (RB + 2) * HC * 4;
  constexpr int MAXIT = 4;
  float gr[8], xr[MAXIT][8];
  auto fetch = [&](int64_t blk) {
    const int b = (int)(blk / ((int64_t)HB * tx));
    const int rem = (int)(blk - (int64_t)b * HB * tx);
    const int y = (rem / tx) * RB, x0 = (rem - (rem / tx) * tx) * 64;
    {
      // gradient: thread t -> pixel t mod 64, output channels 8 (t / 64) ...
      // (a wave writes one channel row at 64 consecutive pixels: no two
      // lanes on one LDS bank but the two halves of a dword)
      const int p = threadIdx.x & 63, q = threadIdx.x >> 6;
      const int64_t go = (((int64_t)b * H + y + p / PW) * W + x0 + p % PW) * Cout + o0 + 8 * q;
      const float4 u0 = *reinterpret_cast<const float4*>(G + go);
      const float4 u1 = *reinterpret_cast<const float4*>(G + go + 4);
      gr[0] = u0.x; gr[1] = u0.y; gr[2] = u0.z; gr[3] = u0.w;
      gr[4] = u1.x; gr[5] = u1.y; gr[6] = u1.z; gr[7] = u1.w;
      if (gscale) {
        const float* sc = gscale + (int64_t)b * Cout + o0 + 8 * q;
#pragma unroll
        for (int j = 0; j < 8; ++j) gr[j] *= sc[j];
      }
    }
#pragma unroll
    for (int k = 0; k < MAXIT; ++k) {
      const int it = threadIdx.x + 256 * k;
#pragma unroll
      for (int j = 0; j < 8; ++j) xr[k][j] = 0.f;
      if (it >= NIT) continue;
      // consecutive lanes take consecutive halo columns (see the gradient)
      const int hc = it % HC, hr = (it / HC) % (RB + 2), q = it / (HC * (RB + 2));
      int ys = y + hr - 1, xs = x0 + hc - 1;
      bool valid = true;
      if (circular) {
        ys = ys < 0 ? ys + H : (ys >= H ? ys - H : ys);
        xs = xs < 0 ? xs + W : (xs >= W ? xs - W : xs);
      } else {
        valid = ys >= 0 && ys < H && xs >= 0 && xs < W;
      }
      if (valid) {
        const int64_t xo = (((int64_t)b * H + ys) * W + xs) * Cin + i0 + 8 * q;
        const float4 u0 = *reinterpret_cast<const float4*>(X + xo);
        const float4 u1 = *reinterpret_cast<const float4*>(X + xo + 4);
        xr[k][0] = u0.x; xr[k][1] = u0.y; xr[k][2] = u0.z; xr[k][3] = u0.w;
        xr[k][4] = u1.x; xr[k][5] = u1.y; xr[k][6] = u1.z; xr[k][7] = u1.w;
        if (xscale) {
          const float* sc = xscale + (int64_t)b * Cin + i0 + 8 * q;
#pragma unroll
          for (int j = 0; j < 8; ++j) xr[k][j] *= sc[j];
        }
      }
    }
  };
  auto stage = [&]() {
    {
      const int p = threadIdx.x & 63, q = threadIdx.x >> 6;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned short h = bf16_bits(gr[j]);
        gT[(8 * q + j) * RS + p] = h;
        if (SPLIT == 3) gT[GT + (8 * q + j) * RS + p] = bf16_bits(gr[j] - bf16_value(h));
      }
    }
#pragma unroll
    for (int k = 0; k < MAXIT; ++k) {
      const int it = threadIdx.x + 256 * k;
      if (it >= NIT) continue;
      const int hc = it % HC, hr = (it / HC) % (RB + 2), q = it / (HC * (RB + 2));
      unsigned short hb[8], lb[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        hb[j] = bf16_bits(xr[k][j]);
        lb[j] = bf16_bits(xr[k][j] - bf16_value(hb[j]));
      }
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int pr = hr - r;
        if (pr < 0 || pr >= RB) continue;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int c = hc - d;
          if (c < 0 || c >= PW) continue;
          const int pp = pr * PW + c;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int e = ((d * 32 + 8 * q + j) * 3 + r) * RS + pp;
            xT[e] = hb[j];
            if (SPLIT == 3) xT[XT + e] = lb[j];
          }
        }
      }
    }
  };

  if ((int64_t)blockIdx.x < nblocks) fetch(blockIdx.x);
  for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    __syncthreads();  // the previous block's fragments have been read
    stage();
    if (blk + gridDim.x < nblocks) fetch(blk + gridDim.x);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int pk = 32 * ks + 8 * kq;
      const int ga = (ow + m) * RS + pk;
      const bf16x8 ahi = *reinterpret_cast<const bf16x8*>(gT + ga);
      bf16x8 alo;
      if (SPLIT == 3) alo = *reinterpret_cast<const bf16x8*>(gT + GT + ga);
#pragma unroll
      for (int t = 0; t < 9; ++t) {
        const int r = t / 3, d = t % 3;  // dy + 1, dx + 1
        const int xb = ((d * 32 + iw + m) * 3 + r) * RS + pk;
        const bf16x8 bhi = *reinterpret_cast<const bf16x8*>(xT + xb);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bhi, acc[t], 0, 0, 0);
        if (SPLIT == 3) {
          const bf16x8 blo = *reinterpret_cast<const bf16x8*>(xT + XT + xb);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bhi, acc[t], 0, 0, 0);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, blo, acc[t], 0, 0, 0);
        }
      }
    }
  }
  // D[row = o (4 kq + j)][col = i (m)]
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      partial[(((int64_t)blockIdx.x * 9 + t) * Cout + o0 + ow + 4 * kq + j) * Cin + i0 + iw + m] =
          acc[t][j];
}

// The weight gradient for layers with many pixels.  A workgroup owns a 32 x
// 32 (output, input channel) tile of all 9 taps and runs through pixel tiles
// of RW x WT = 256 pixels, group `g` of `ng` taking every ng-th; the next
// tile's loads are in registers while this one's products run.  Both operands
// are staged as the convolution stages them (pixel rows of 32 channels, BF16
// hi and lo, one copy), and the matrix core's fragments, which run along the
// pixels, come from transposing LDS reads (ds_read_b64_tr_b16: four lanes
// give the addresses of a pixel's 16 channels, lane i of a group of 16 gets
// channel i of four pixels; lane layout checked on gfx950 by an in-bounds
// probe), which take any pixel offset, so a tap is an offset and nothing is
// staged three times.
// K step s of a tile: 32 pixels, the row s (WT = 32) or the rows s and s + 8
// (WT = 16).  Wave w takes steps 4 (w / 2) .. + 3 and 16 input channels,
// w mod 2, of all 32 output channels and 9 taps (72 accumulators; all 32 input
// channels of half as many steps spilled): an input row's fragments (three
// dx) serve the steps above, at and below it.  Waves 2 and 3 hand their sums
// to 0 and 1 through LDS, which write partial[g][t][o][i].  76 KB of LDS: two
// workgroups share a CU.
// Bound by the matrix cores and the staging between them: 29 GFLOP in three
// passes (batch 32, 128 x 128: 32 channels at full, 64 at half, 128 at quarter
// resolution) 35.6 us, 810 TFLOP/s, where k_wgradt, which writes single BF16
// values of three shifted copies, took 172, 167 and 102.
template <int SPLIT, int WT>
__global__ __launch_bounds__(256, 2) void k_wgradw(const float* __restrict__ G,
                                                   const float* __restrict__ gscale,
                                                   const float* __restrict__ X,
                                                   const float* __restrict__ xscale,
                                                   float* __restrict__ partial, int H, int W,
                                                   int Cin, int Cout, int circular, int npt,
                                                   int ng) {
  constexpr int RW = 256 / WT, TR = RW + 2, TW = WT + 2;
  constexpr int NH = SPLIT == 3 ? 2 : 1;
  constexpr int XS = TR * TW * 16, GS = 256 * 16;  // dwords per hi/lo part
  constexpr int RED = 18 * 64 * 4;                 // sums of a wave
  constexpr int LDS = NH * (XS + GS) > 2 * RED ? NH * (XS + GS) : 2 * RED;
  __shared__ uint4 lds4[LDS / 4];
  uint32_t* xt = reinterpret_cast<uint32_t*>(lds4);
  uint32_t* gt = xt + NH * XS;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int m = lane & 15, kq = lane >> 4;
  const int q = threadIdx.x & 3;
  const int kh = wave >> 1, ch = wave & 1;
  // group and channel tile: the channel tiles of a pixel group on one XCD
  const int nit = Cin / 32, nct = (Cout / 32) * nit;
  int g, ct;
  if (ng % 8 == 0) {
    const int i = blockIdx.x >> 3;
    ct = i % nct;
    g = (i / nct) * 8 + (blockIdx.x & 7);
  } else {
    ct = blockIdx.x % nct;
    g = blockIdx.x / nct;
  }
  const int o0 = ct / nit * 32, i0 = ct % nit * 32;
  const int tx = W / WT, tiles = (H / RW) * tx;

  // 16-byte piece q of the pixel at column c sits at q ^ rot(c): conflict-free
  // for 8 pixels' equal pieces (staging) and for 4 pixels' piece pairs
  auto rot = [](int c) __attribute__((always_inline)) { return (c & 2) | ((c >> 2) & 1); };
  // dword offsets of this lane's 8 bytes of a transposing read (channels 0 ..
  // 15; channels 16 .. 31: ^ 8): pixel 4 h + m / 4 of its 8, 4-channel piece m % 4
  const int row8 = WT == 16 ? 8 * (kq >> 1) : 0, col8 = WT == 16 ? 8 * (kq & 1) : 8 * kq;
  auto at = [&](int tw, int col) __attribute__((always_inline)) {
    return 16 * ((row8 + 4 * kh) * tw + col) + 4 * (((m & 3) >> 1) ^ rot(col)) + 2 * (m & 1);
  };
  int ga[2], xa[3][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int col = col8 + 4 * h + (m >> 2);
    ga[h] = at(WT, col);
#pragma unroll
    for (int d = 0; d < 3; ++d) xa[d][h] = at(TW, col + d) ^ (8 * ch);
  }
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* LdsP;
  auto frag = [&](const uint32_t* base, int a0, int a1) __attribute__((always_inline)) {
    const s16x4 u = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsP)(base + a0));
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsP)(base + a1));
    bf16x8 r;
    __builtin_memcpy(&r, &u, 8);
    __builtin_memcpy(reinterpret_cast<char*>(&r) + 8, &v, 8);
    return r;
  };

  f32x4 acc[9][2];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int a = 0; a < 2; ++a) acc[t][a] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // staged pieces of 8 channels: PER of the input (with its halo), then 4 of
  // the gradient
  constexpr int NTILE = TR * TW * 4, PER = (NTILE + 255) / 256;
  float u[PER + 4][8];
  uint32_t live;  // bit k: input piece k is inside the image (else zero)
  auto fetch = [&](int pt) __attribute__((always_inline)) {
    const int b = pt / tiles, rem = pt - b * tiles;
    const int y = (rem / tx) * RW, x0 = (rem - (rem / tx) * tx) * WT;
    const float* xb = X + (int64_t)b * H * W * Cin + i0 + 8 * q;
    const float* gb = G + (int64_t)b * H * W * Cout + o0 + 8 * q;
    live = 0u;
    // (recomputed for every tile: rows and columns kept across the products
    // would spill, and a reload waits for all loads in flight)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int k = 0; k < PER + 4; ++k) {
      const float* p;
      if (k < PER) {
        const int i = tid + 256 * k;
        const int row = (i >> 2) / TW, col = (i >> 2) - row * TW;
        const int yr = y + row - 1, xr = x0 + col - 1;
        const int ys = yr < 0 ? yr + H : (yr >= H ? yr - H : yr);
        const int xs = xr < 0 ? xr + W : (xr >= W ? xr - W : xr);
        const bool v = i < NTILE && (circular || (ys == yr && xs == xr));
        live |= v ? 1u << k : 0u;
        p = xb + (v ? ((int64_t)ys * W + xs) * Cin : 0);
      } else {
        const int i = (tid >> 2) + 64 * (k - PER), row = i / WT, col = i - row * WT;
        p = gb + ((int64_t)(y + row) * W + x0 + col) * Cout;
      }
      const float4 a = *reinterpret_cast<const float4*>(p), c = *reinterpret_cast<const float4*>(p + 4);
      u[k][0] = a.x; u[k][1] = a.y; u[k][2] = a.z; u[k][3] = a.w;
      u[k][4] = c.x; u[k][5] = c.y; u[k][6] = c.z; u[k][7] = c.w;
    }
  };
  if (g < npt) fetch(g);
  for (int pt = g; pt < npt; pt += ng) {
    const int b = pt / tiles;
    float sx[8], sg[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sx[j] = xscale ? xscale[(int64_t)b * Cin + i0 + 8 * q + j] : 1.f;
      sg[j] = gscale ? gscale[(int64_t)b * Cout + o0 + 8 * q + j] : 1.f;
    }
    __syncthreads();  // the previous tile's fragments have been read
#pragma unroll
    for (int k = 0; k < PER + 4; ++k) {
      const int i = (int)threadIdx.x + 256 * (k < PER ? k : k - PER);
      if (k + 1 == PER && NTILE % 256 != 0 && i >= NTILE) continue;
      float a[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a[j] = u[k][j] * (k < PER ? sx[j] : sg[j]);
        if (k < PER) a[j] = live >> k & 1 ? a[j] : 0.f;
      }
      uint32_t h[4], l[4];
      split_pairs<SPLIT>(a, h, l);
      const int p = i >> 2, col = k < PER ? p % TW : p % WT;
      const int d = 16 * p + 4 * (q ^ rot(col));
      uint32_t* t = k < PER ? xt : gt;
      *reinterpret_cast<uint4*>(t + d) = (uint4){h[0], h[1], h[2], h[3]};
      if (SPLIT == 3)
        *reinterpret_cast<uint4*>(t + (k < PER ? XS : GS) + d) = (uint4){l[0], l[1], l[2], l[3]};
    }
    if (pt + ng < npt) fetch(pt + ng);
    __syncthreads();
    bf16x8 gh[4][2], gl[4][2];  // [step][half of the output channels]
#pragma unroll
    for (int r = 0; r < 6; ++r) {  // input row 4 kh + r of the tile
      // (plain BF16: without the barrier the fragments of all rows are read ahead of
      // the products, 256 registers and 36 B of scratch per lane; 216 and none with it)
      if (SPLIT == 1) __builtin_amdgcn_sched_barrier(0);
      if (r < 4) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const uint32_t* base = gt + r * WT * 16;
          gh[r][a] = frag(base, ga[0] ^ (8 * a), ga[1] ^ (8 * a));
          if (SPLIT == 3) gl[r][a] = frag(base + GS, ga[0] ^ (8 * a), ga[1] ^ (8 * a));
        }
      }
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const uint32_t* base = xt + r * TW * 16;
        const bf16x8 xh = frag(base, xa[dx][0], xa[dx][1]);
        bf16x8 xl = xh;  // (plain BF16 operands: not used)
        if (SPLIT == 3) xl = frag(base + XS, xa[dx][0], xa[dx][1]);
#pragma unroll
        for (int part = 0; part < SPLIT; ++part)
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
            const int s = r - dy;
            if (s < 0 || s > 3) continue;
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              f32x4& d = acc[3 * dy + dx][a];
              d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part == 1 ? gl[s][a] : gh[s][a],
                                                          part == 2 ? xl : xh, d, 0, 0, 0);
            }
          }
      }
    }
  }
  // D[row = o (4 kq + j)][col = i (m)]; the second half's steps are added to
  // the first's
  float* red = reinterpret_cast<float*>(lds4) + ch * RED;
  __syncthreads();
  if (kh) {
#pragma unroll
    for (int e = 0; e < 18; ++e)
      *reinterpret_cast<f32x4*>(red + (e * 64 + lane) * 4) = acc[e >> 1][e & 1];
  }
  __syncthreads();
  if (kh) return;
#pragma unroll
  for (int e = 0; e < 18; ++e) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(red + (e * 64 + lane) * 4);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      partial[(((int64_t)g * 9 + (e >> 1)) * Cout + o0 + 16 * (e & 1) + 4 * kq + j) * Cin + i0 +
              16 * ch + m] = acc[e >> 1][e & 1][j] + v[j];
  }
}

// Sum of the weight-gradient partials in a fixed order: 64 weights per
// workgroup as 16 x 4, 16 groups of threads summing every 16th partial, then
// the group sums in order.  One float per thread and 4 groups left a chain of
// dependent memory latencies (256 partials of a 32 x 32 layer: 19.9 us, 512:
// 37.8); 16 groups of float4 take 4.8 us for 512.
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* __restrict__ partial,
                                                      int nsplit, int Cin, int Cout,
                                                      float* __restrict__ grad) {
  __shared__ float4 sh[16][16];
  const int el = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int64_t n = (int64_t)9 * Cout * Cin;  // a multiple of 64
  const float* p = partial + (int64_t)blockIdx.x * 64 + 4 * el;
  float4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int k = g; k < nsplit; k += 16) {
    const float4 v = *reinterpret_cast<const float4*>(p + (int64_t)k * n);
    s.x += v.x;
    s.y += v.y;
    s.z += v.z;
    s.w += v.w;
  }
  sh[g][el] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const float* q = reinterpret_cast<const float*>(sh) + threadIdx.x;
  float r = q[0];
#pragma unroll
  for (int k = 1; k < 16; ++k) r += q[64 * k];
  const int64_t e = (int64_t)blockIdx.x * 64 + threadIdx.x;
  const int t = (int)(e / ((int64_t)Cout * Cin));
  const int64_t oi = e - (int64_t)t * Cout * Cin;
  const int o = (int)(oi / Cin), i = (int)(oi - (int64_t)o * Cin);
  grad[((int64_t)o * Cin + i) * 9 + t] = r;
}

// master weights [o][i][3][3] FP32 of every layer -> BF16 hi/lo in [t][o][i]
// (forward) and flipped/transposed [t][i][o] (data gradient); layer l's
// elements are e = at[l] .. at[l + 1] - 1, in one launch (a launch per layer:
// 95 us for the 16)
constexpr int MAXL = 16;
struct PrepArgs {
  int at[MAXL + 1];      // first element of each layer
  int64_t woff[MAXL];    // the layer's weights in the parameter vector
  int64_t wq_off[MAXL];  // and in the BF16 arrays
  int cin[MAXL], cout[MAXL];
  int n;
};

__global__ __launch_bounds__(256) void k_prep_weights(const float* __restrict__ param, PrepArgs a,
                                                      unsigned short* __restrict__ fhi,
                                                      unsigned short* __restrict__ flo,
                                                      unsigned short* __restrict__ bhi,
                                                      unsigned short* __restrict__ blo) {
  // (a layer's element count is a multiple of 256: one layer per workgroup)
  const int e0 = blockIdx.x * 256;
  int l = 0;
  while (l + 1 < a.n && e0 >= a.at[l + 1]) ++l;
  const int e = e0 - a.at[l] + (int)threadIdx.x;
  const int Cin = a.cin[l], Cout = a.cout[l];
  const int o = e / (9 * Cin), r = e - o * 9 * Cin, i = r / 9, t = r - i * 9;
  const float v = param[a.woff[l] + e];
  const unsigned short h = bf16_bits(v), lo = bf16_bits(v - bf16_value(h));
  const int64_t f = a.wq_off[l] + ((int64_t)t * Cout + o) * Cin + i;
  const int64_t b = a.wq_off[l] + ((int64_t)(8 - t) * Cin + i) * Cout + o;
  fhi[f] = h;
  flo[f] = lo;
  bhi[b] = h;
  blo[b] = lo;
}

// ---------------------------------------------------------------------------
// pooling / up-sampling (NHWC, scale on load); thread e handles the 4
// channels 4 (e mod C/4) .. + 3 of one pixel (C % 4 == 0), each with the
// operations written for one element
// ---------------------------------------------------------------------------
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 scale4(const float* s, int64_t i) {
  return s ? ld4(s + i) : make_float4(1.f, 1.f, 1.f, 1.f);
}

// pixel and channel of 4-channel item e of a [B][H][W][C] tensor
__device__ __forceinline__ void item4(int64_t e, int H, int W, int C, int& b, int& y, int& x,
                                      int& c) {
  const int C4 = C >> 2;
  int64_t r = e / C4;
  c = 4 * (int)(e - r * C4);
  x = (int)(r % W);
  r /= W;
  y = (int)(r % H);
  b = (int)(r / H);
}

// out[b,Y,X,c] = 1/4 sum_{2x2} s[b,c] in[b,2Y+u,2X+v,c]
__global__ __launch_bounds__(256) void k_pool(const float* __restrict__ in,
                                              const float* __restrict__ scale,
                                              float* __restrict__ out, int B, int Ho, int Wo,
                                              int C) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)B * Ho * Wo * C / 4) return;
  int b, Y, X, c;
  item4(e, Ho, Wo, C, b, Y, X, c);
  const int Wi = 2 * Wo;
  const float* p = in + (((int64_t)b * 2 * Ho + 2 * Y) * Wi + 2 * X) * C + c;
  const float4 s = scale4(scale, (int64_t)b * C + c);
  const float4 p0 = ld4(p), p1 = ld4(p + C), p2 = ld4(p + (int64_t)Wi * C),
               p3 = ld4(p + (int64_t)Wi * C + C);
  float4 o;
  o.x = 0.25f * s.x * ((p0.x + p1.x) + (p2.x + p3.x));
  o.y = 0.25f * s.y * ((p0.y + p1.y) + (p2.y + p3.y));
  o.z = 0.25f * s.z * ((p0.z + p1.z) + (p2.z + p3.z));
  o.w = 0.25f * s.w * ((p0.w + p1.w) + (p2.w + p3.w));
  *reinterpret_cast<float4*>(out + 4 * e) = o;
}

// out[b,y,x,c] = sc[b,c] coarse[b,y/2,x/2,c] + ss[b,c] skip[b,y,x,c]
__global__ __launch_bounds__(256) void k_upadd(const float* __restrict__ coarse,
                                               const float* __restrict__ sc,
                                               const float* __restrict__ skip,
                                               const float* __restrict__ ss,
                                               float* __restrict__ out, int B, int H, int W,
                                               int C) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)B * H * W * C / 4) return;
  int b, y, x, c;
  item4(e, H, W, C, b, y, x, c);
  const float4 cv = ld4(coarse + (((int64_t)b * (H / 2) + y / 2) * (W / 2) + x / 2) * C + c);
  const float4 a = scale4(sc, (int64_t)b * C + c), t = scale4(ss, (int64_t)b * C + c);
  const float4 k = ld4(skip + 4 * e);
  float4 o;
  o.x = a.x * cv.x + t.x * k.x;
  o.y = a.y * cv.y + t.y * k.y;
  o.z = a.z * cv.z + t.z * k.z;
  o.w = a.w * cv.w + t.w * k.w;
  *reinterpret_cast<float4*>(out + 4 * e) = o;
}

// backward of pooling, plus an optional addend:
// out[b,y,x,c] = 1/4 g[b,y/2,x/2,c] + (add ? add[b,y,x,c] : 0)
__global__ __launch_bounds__(256) void k_pool_back(const float* __restrict__ g,
                                                   const float* __restrict__ add,
                                                   float* __restrict__ out, int B, int H, int W,
                                                   int C) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)B * H * W * C / 4) return;
  int b, y, x, c;
  item4(e, H, W, C, b, y, x, c);
  const float4 gv = ld4(g + (((int64_t)b * (H / 2) + y / 2) * (W / 2) + x / 2) * C + c);
  float4 o = make_float4(0.25f * gv.x, 0.25f * gv.y, 0.25f * gv.z, 0.25f * gv.w);
  if (add) {
    const float4 d = ld4(add + 4 * e);
    o.x += d.x;
    o.y += d.y;
    o.z += d.z;
    o.w += d.w;
  }
  *reinterpret_cast<float4*>(out + 4 * e) = o;
}

// backward of nearest up-sampling: out[b,Y,X,c] = sum_{2x2} g[b,2Y+u,2X+v,c]
__global__ __launch_bounds__(256) void k_up_back(const float* __restrict__ g,
                                                 float* __restrict__ out, int B, int Ho, int Wo,
                                                 int C) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)B * Ho * Wo * C / 4) return;
  int b, Y, X, c;
  item4(e, Ho, Wo, C, b, Y, X, c);
  const int Wi = 2 * Wo;
  const float* p = g + (((int64_t)b * 2 * Ho + 2 * Y) * Wi + 2 * X) * C + c;
  const float4 p0 = ld4(p), p1 = ld4(p + C), p2 = ld4(p + (int64_t)Wi * C),
               p3 = ld4(p + (int64_t)Wi * C + C);
  float4 o;
  o.x = (p0.x + p1.x) + (p2.x + p3.x);
  o.y = (p0.y + p1.y) + (p2.y + p3.y);
  o.z = (p0.z + p1.z) + (p2.z + p3.z);
  o.w = (p0.w + p1.w) + (p2.w + p3.w);
  *reinterpret_cast<float4*>(out + 4 * e) = o;
}

}  // namespace sgk
