// Learned window surrogate (C ABI in include/sg.h): a linear U-Net on the
// first-order system's variables with FiLM gains, trained on windows of the
// lattice Boltzmann scheme and checked by it.  Forward, loss, backward and
// Adam all run in this file's kernels and sg_kernels.hpp's matrix-core
// convolutions; the host code only sequences launches.
//
// Input per sample: 8 physical channels [8][H][W] (v_x, v_y, sigma_xx,
// sigma_yy, sigma_xy, lambda, mu, rho).  pre: U = (v, j) through the inverse
// of Eq. sigma_num with the pixel's material, divided by the per-sample RMS s
// of U, channels 5..31 zero.  Conditioning t in [-1, 1] from theta =
// atan2(mean c_mu, mean c_K) (time step at half the CFL-like limit, so theta
// fixes both Courant numbers); FiLM gain of conv layer l, output channel c:
// gamma[b][c] = sum_m a_l[c][m] T_m(t_b), Chebyshev T_0..T_3.  post:
// U' = U + s * gamma_out * z_out[0..4], back to physical fields.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <new>
#include <string>
#include <vector>

#include "lbm_host.hpp"
#include "sg.h"
#include "sg_kernels.hpp"

using namespace sgk;
using lbmh::fail;
using lbmh::hip_check;
using lbmh::launch_check;
using lbmh::round_up;

namespace {

constexpr int CP = 32;  // padded input/output channels

struct LayerSpec {
  const char* name;
  int cin, cout, level;
};
// two convolutions per level, four levels; order = parameter order
const LayerSpec kLayers[] = {
    {"in", 32, 32, 0},    {"e0a", 32, 32, 0},   {"e0b", 32, 32, 0},   {"e1a", 32, 64, 1},
    {"e1b", 64, 64, 1},   {"e2a", 64, 128, 2},  {"e2b", 128, 128, 2}, {"e3a", 128, 128, 3},
    {"e3b", 128, 128, 3}, {"d2a", 128, 128, 2}, {"d2b", 128, 64, 2},  {"d1a", 64, 64, 1},
    {"d1b", 64, 32, 1},   {"d0a", 32, 32, 0},   {"d0b", 32, 32, 0},   {"out", 32, 32, 0}};
constexpr int NL = (int)(sizeof(kLayers) / sizeof(kLayers[0]));
static_assert(NL == NLAYER, "SampleStats size");
enum { L_IN, L_E0A, L_E0B, L_E1A, L_E1B, L_E2A, L_E2B, L_E3A, L_E3B, L_D2A, L_D2B, L_D1A,
       L_D1B, L_D0A, L_D0B, L_OUT };

constexpr int RT = 256;

// ---- per-sample statistics and pre/post -------------------------------------
__device__ inline double wg_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = RT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Per-sample statistics in two passes: stats_chunks(HW) workgroups per sample
// sum |U|^2, c_K and c_mu over their pixels (FP64), then sample_stats (the
// workgroups at the end of k_conv_in's grid, or k_stats) adds the partial sums
// in a fixed order and forms s_b, the Chebyshev values T[b][m] and the gains.
// (256 x 256, batch 1: 64 workgroups of 4 pixels per thread 6.2 us, 256 of one
// 3.7; the rest 8.3 us as a launch of its own, 4.7 with the loads ahead of the
// sums, and hidden behind the first layer.)
__global__ __launch_bounds__(RT) void k_stats_partial(const float* __restrict__ in, int HW,
                                                      double* __restrict__ part) {
  __shared__ double sh[3][RT / 64];
  const int b = blockIdx.y;
  const float* f = in + (int64_t)b * 8 * HW;
  double u2 = 0.0, ck = 0.0, cm = 0.0;
  for (int p = blockIdx.x * RT + threadIdx.x; p < HW; p += gridDim.x * RT) {
    const Mat m = material(f, HW, p);
    float U[5];
    phys_to_U(f, HW, p, m, U);
    for (int c = 0; c < 5; ++c) u2 += (double)U[c] * U[c];
    ck += m.cK;
    cm += m.cm;
  }
  u2 = wave_total(u2);
  ck = wave_total(ck);
  cm = wave_total(cm);
  if ((threadIdx.x & 63) == 0) {
    sh[0][threadIdx.x >> 6] = u2;
    sh[1][threadIdx.x >> 6] = ck;
    sh[2][threadIdx.x >> 6] = cm;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const double* q = sh[threadIdx.x];
    part[((int64_t)b * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = (q[0] + q[1]) + (q[2] + q[3]);
  }
}

__global__ __launch_bounds__(RT) void k_stats(SampleStats st) { sample_stats(st, blockIdx.x); }

// x0[b][p][c] = U_c / s_b for c < 5, 0 otherwise
__global__ __launch_bounds__(RT) void k_pre(const float* __restrict__ in, int B, int HW,
                                            const float* __restrict__ sv,
                                            float* __restrict__ x0) {
  const int64_t e = (int64_t)blockIdx.x * RT + threadIdx.x;
  if (e >= (int64_t)B * HW) return;
  const int b = (int)(e / HW);
  const int64_t p = e - (int64_t)b * HW;
  const float* f = in + (int64_t)b * 8 * HW;
  const Mat m = material(f, HW, p);
  float U[5];
  phys_to_U(f, HW, p, m, U);
  const float r = 1.f / sv[b];
  float* o = x0 + e * CP;
  for (int c = 0; c < 5; ++c) o[c] = U[c] * r;
  for (int c = 5; c < CP; ++c) o[c] = 0.f;
}

// out[b][5][H][W] physical = fields of U + s gamma z_out[0..4]
__global__ __launch_bounds__(RT) void k_post(const float* __restrict__ in,
                                             const float* __restrict__ zout,
                                             const float* __restrict__ gout,
                                             const float* __restrict__ sv, int B, int HW,
                                             float* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * RT + threadIdx.x;
  if (e >= (int64_t)B * HW) return;
  const int b = (int)(e / HW);
  const int64_t p = e - (int64_t)b * HW;
  const float* f = in + (int64_t)b * 8 * HW;
  const Mat m = material(f, HW, p);
  float U[5];
  phys_to_U(f, HW, p, m, U);
  const float* z = zout + e * CP;
  const float* g = gout + (int64_t)b * CP;
  for (int c = 0; c < 5; ++c) U[c] = U[c] + sv[b] * (g[c] * z[c]);
  float* o = out + (int64_t)b * 5 * HW;
  o[p] = U[0];
  o[HW + p] = U[1];
  o[2 * HW + p] = -m.rho * (m.cK * U[2] + m.cm * U[3]);
  o[3 * HW + p] = -m.rho * (m.cK * U[2] - m.cm * U[3]);
  o[4 * HW + p] = -m.rho * (m.cm * U[4]);
}

// loss = mean (gamma z_out[0..4] - (U_target - U)/s)^2, gradient w.r.t. y_out
// (NHWC, 32 channels, zero beyond 5); per-workgroup partial sums
__global__ __launch_bounds__(RT) void k_loss(const float* __restrict__ in,
                                             const float* __restrict__ target,
                                             const float* __restrict__ zout,
                                             const float* __restrict__ gout,
                                             const float* __restrict__ sv, int B, int HW,
                                             float inv_n, float* __restrict__ gy,
                                             double* __restrict__ partial) {
  __shared__ double sh[RT];
  const int64_t e = (int64_t)blockIdx.x * RT + threadIdx.x;
  double l = 0.0;
  if (e < (int64_t)B * HW) {
    const int b = (int)(e / HW);
    const int64_t p = e - (int64_t)b * HW;
    const float* f = in + (int64_t)b * 8 * HW;
    const Mat m = material(f, HW, p);
    float U[5], Ut[5];
    phys_to_U(f, HW, p, m, U);
    phys_to_U(target + (int64_t)b * 5 * HW, HW, p, m, Ut);
    const float* z = zout + e * CP;
    const float* g = gout + (int64_t)b * CP;
    float* o = gy + e * CP;
    const float r = 1.f / sv[b];
    for (int c = 0; c < 5; ++c) {
      const float d = g[c] * z[c] - (Ut[c] - U[c]) * r;
      l += (double)d * d;
      o[c] = 2.f * d * inv_n;
    }
    for (int c = 5; c < CP; ++c) o[c] = 0.f;
  }
  l = wg_sum(l, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = l;
}

__global__ __launch_bounds__(RT) void k_sum_partials(const double* __restrict__ p, int n,
                                                     double* __restrict__ out) {
  __shared__ double sh[RT];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += RT) s += p[i];
  s = wg_sum(s, sh);
  if (threadIdx.x == 0) *out = s;
}

// dgamma[b][c] = sum_p g[b,p,c] z[b,p,c] (FiLM gain gradient), in two passes.
// First, workgroup (b, s) takes pixel chunk s of sample b for all C channels:
// a thread 4 consecutive channels of every (4 RT / C)-th pixel, FP64 sums,
// added per channel in a fixed order.  Bound by memory (both tensors read
// once): 32 samples of 128 x 128 x 32 channels, 134 MB, took 35 us with one
// float per load and 16 chunks per sample, 17 with 16-byte loads and 64 (the
// gradient is still in the last-level cache).
__global__ __launch_bounds__(RT) void k_film_grad_part(const float* __restrict__ g,
                                                       const float* __restrict__ z, int HW, int C,
                                                       int S, double* __restrict__ part) {
  __shared__ double sh[RT][4];
  const int b = blockIdx.x / S, sidx = blockIdx.x - b * S;
  const int C4 = C / 4, G = RT / C4, c4 = threadIdx.x % C4, grp = threadIdx.x / C4;
  const int p0 = (int)((int64_t)HW * sidx / S), p1 = (int)((int64_t)HW * (sidx + 1) / S);
  const float* gp = g + (int64_t)b * HW * C + 4 * c4;
  const float* zp = z + (int64_t)b * HW * C + 4 * c4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int p = p0 + grp; p < p1; p += G) {
    const float4 x = *reinterpret_cast<const float4*>(gp + (int64_t)p * C);
    const float4 y = *reinterpret_cast<const float4*>(zp + (int64_t)p * C);
    acc[0] += (double)x.x * y.x;
    acc[1] += (double)x.y * y.y;
    acc[2] += (double)x.z * y.z;
    acc[3] += (double)x.w * y.w;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) sh[threadIdx.x][j] = acc[j];
  __syncthreads();
  if ((int)threadIdx.x < C) {
    double t = 0.0;
    for (int k = 0; k < G; ++k) t += sh[k * C4 + threadIdx.x / 4][threadIdx.x % 4];
    part[(int64_t)blockIdx.x * C + threadIdx.x] = t;
  }
}

// Then, for every layer in one launch, dgamma[b][c] = the sum over the chunks
// in order and the coefficient gradients da[c][m] = sum_b T[b][m] dgamma[b][c]
// in order of b.  A workgroup takes 32 channels of one layer, 8 samples at a
// time.  (As two launches per layer, the second a chain of B dependent reads,
// they took 250 us of a step.)
struct FilmArgs {
  const double* part[NL];  // [b][s][c]
  float* da[NL];
  int cout[NL], S[NL];
};

__global__ __launch_bounds__(RT) void k_film_grad_coef(FilmArgs a, const float* __restrict__ T,
                                                       int B) {
  __shared__ float dg[8][32];
  int blk = blockIdx.x, l = 0;
  while (blk >= a.cout[l] / 32) blk -= a.cout[l++] / 32;
  const int C = a.cout[l], S = a.S[l];
  const int c = threadIdx.x & 31, bg = threadIdx.x >> 5;
  const double* part = a.part[l] + 32 * blk + c;
  const int cc = threadIdx.x / NBASIS, m = threadIdx.x % NBASIS;
  float s = 0.f;
  for (int b0 = 0; b0 < B; b0 += 8) {
    const int b = b0 + bg;
    double t = 0.0;
    if (b < B) {
#pragma unroll 16
      for (int k = 0; k < S; ++k) t += part[((int64_t)b * S + k) * C];
    }
    dg[bg][c] = (float)t;
    __syncthreads();
    if ((int)threadIdx.x < 32 * NBASIS)
      for (int k = 0; k < 8 && b0 + k < B; ++k)
        s = fmaf(T[(b0 + k) * NBASIS + m], dg[k][cc], s);
    __syncthreads();
  }
  if ((int)threadIdx.x < 32 * NBASIS) a.da[l][(32 * blk + cc) * NBASIS + m] = s;
}

__global__ __launch_bounds__(RT) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                             float* __restrict__ mo, float* __restrict__ ve,
                                             int64_t n, float lr, float b1, float b2, float eps,
                                             float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * RT + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float m = b1 * mo[i] + (1.f - b1) * gi;
  const float v = b2 * ve[i] + (1.f - b2) * gi * gi;
  mo[i] = m;
  ve[i] = v;
  p[i] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// ---- host-side plan ----------------------------------------------------------
struct Tensor {
  float* p = nullptr;
  int H = 0, W = 0, C = 0;
};

struct Plan {
  int B, H, W, split, train;
  int64_t nparam = 0;
  int64_t woff[NL], aoff[NL];      // offsets in the parameter vector
  int64_t wq_off[NL];              // offsets in the bf16 weight arrays
  int64_t nwq = 0;
  size_t bytes = 0;
  // workspace offsets
  size_t o_param, o_grad, o_m, o_v, o_wfh, o_wfl, o_wbh, o_wbl, o_s, o_T, o_gam,
      o_part, o_spart, o_loss, o_x0, o_z[NL], o_pool[3], o_up[3], o_g[NL], o_gpool[3], o_gup[3],
      o_wpart, o_fpart[NL];
  int64_t wpart_floats = 0;
};

// pixel chunks per sample of the FiLM gradient: about 2048 workgroups, at
// least 64 pixels each
constexpr int FILM_WG = 2048;
int film_chunks(int B, int HW) {
  int S = (FILM_WG + B - 1) / B;
  if (S > HW / 64) S = HW / 64;
  return S < 1 ? 1 : S;
}

int level_h(const Plan& P, int l) { return P.H >> l; }
int level_w(const Plan& P, int l) { return P.W >> l; }

lbm_status make_plan(const sg_config* cfg, Plan* P) {
  if (!cfg) return fail(LBM_E_ARG, "null config");
  if (cfg->batch < 1 || cfg->height < 64 || cfg->width < 128)
    return fail(LBM_E_ARG, "need batch >= 1, height >= 64, width >= 128");
  if (cfg->height % 64 || cfg->width % 128)
    return fail(LBM_E_ARG, "height must be a multiple of 64 and width of 128");
  if (cfg->split != 1 && cfg->split != 3) return fail(LBM_E_ARG, "split must be 1 or 3");
  P->B = cfg->batch;
  P->H = cfg->height;
  P->W = cfg->width;
  P->split = cfg->split;
  P->train = cfg->train ? 1 : 0;
  int64_t np = 0, nq = 0;
  for (int l = 0; l < NL; ++l) {
    P->woff[l] = np;
    np += (int64_t)kLayers[l].cout * kLayers[l].cin * 9;
    P->aoff[l] = np;
    np += (int64_t)kLayers[l].cout * NBASIS;
    P->wq_off[l] = nq;
    nq += (int64_t)kLayers[l].cout * kLayers[l].cin * 9;
  }
  P->nparam = np;
  P->nwq = nq;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (size_t)round_up((int64_t)bytes, 256);
    return at;
  };
  const int64_t B = P->B;
  auto act = [&](int level, int C) { return (size_t)B * level_h(*P, level) * level_w(*P, level) * C * 4; };
  P->o_param = take(np * 4);
  P->o_wfh = take(nq * 2);
  P->o_wfl = take(nq * 2);
  P->o_wbh = take(nq * 2);
  P->o_wbl = take(nq * 2);
  P->o_s = take(B * 4);
  P->o_T = take(B * NBASIS * 4);
  P->o_gam = take((size_t)NL * B * 128 * 4);
  P->o_part = take(((size_t)B * P->H * P->W / RT + 1) * 8);
  P->o_spart = take((size_t)B * stats_chunks((int64_t)P->H * P->W) * 3 * 8);
  P->o_loss = take(8);
  P->o_x0 = take(act(0, CP));
  for (int l = 0; l < NL; ++l) P->o_z[l] = take(act(kLayers[l].level, kLayers[l].cout));
  const int pc[3] = {32, 64, 128};
  for (int k = 0; k < 3; ++k) P->o_pool[k] = take(act(k + 1, pc[k]));
  const int uc[3] = {32, 64, 128};  // u0 (level 0), u1 (level 1), u2 (level 2)
  for (int k = 0; k < 3; ++k) P->o_up[k] = take(act(k, uc[k]));
  if (P->train) {
    P->o_grad = take(np * 4);
    P->o_m = take(np * 4);
    P->o_v = take(np * 4);
    // chunk sums of any batch up to B (B S <= FILM_WG + B, or a chunk per
    // tile of k_convw)
    for (int l = 0; l < NL; ++l) {
      const size_t tiles = (size_t)B * (P->H >> kLayers[l].level) * (P->W >> kLayers[l].level) / 256;
      const size_t chunks = (size_t)FILM_WG + B;
      P->o_fpart[l] = take((chunks > tiles ? chunks : tiles) * kLayers[l].cout * 8);
    }
    for (int l = 0; l < NL; ++l) P->o_g[l] = take(act(kLayers[l].level, kLayers[l].cout));
    for (int k = 0; k < 3; ++k) P->o_gpool[k] = take(act(k + 1, pc[k]));
    for (int k = 0; k < 3; ++k) P->o_gup[k] = take(act(k, uc[k]));
    // weight-gradient partials: splits x 9 x Cout x Cin for the largest layer
    int64_t mx = 0;
    for (int l = 0; l < NL; ++l) {
      const int64_t v = (int64_t)9 * kLayers[l].cout * kLayers[l].cin;
      mx = v > mx ? v : mx;
    }
    P->wpart_floats = mx * 64;
    P->o_wpart = take(P->wpart_floats * 4);
  }
  P->bytes = o;
  return LBM_OK;
}

}  // namespace

struct sg_net {
  Plan P;
  char* ws;
  hipStream_t stream;
  float* param;
  float* grad;
  float *m, *v;
  unsigned short *wfh, *wfl, *wbh, *wbl;
  float* s;
  float* T;
  float* gam[NL];
  double* fpart[NL];  // FiLM gradient chunk sums
  int fchunks[NL];    // and their number per sample, 0 until the backward pass has them
  double* part;
  double* spart;  // per-sample statistics partials [B][stats_chunks][3]
  double* loss;
  float* x0;
  Tensor z[NL], pool[3], up[3], g[NL], gpool[3], gup[3];
  float* wpart;
  int B;          // batch of the current forward
  int circular;   // padding of the current forward
  const float* in;
  int64_t adam_step;
  bool weights_ready;
  int conv_mode;  // 0: k_convw, k_convs; 1: direct kernel only; 2: k_convt
};

namespace {

inline unsigned grid1(int64_t n) { return (unsigned)((n + RT - 1) / RT); }

template <int SPLIT, int NB, int PB, int KS>
void launch_conv(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                 const unsigned short* wl, Tensor& z, int cin, int cout, int accumulate) {
  const int64_t pixels = (int64_t)n->B * x.H * x.W;
  dim3 grid((unsigned)(pixels / (16 * PB * (4 / KS))), (unsigned)(cout / (16 * NB)));
  hipLaunchKernelGGL((k_conv<SPLIT, NB, PB, KS>), grid, dim3(256), 0, n->stream,
                     (const float*)x.p, xscale, wh, wl, z.p, x.H, x.W, cin, cout, n->circular,
                     accumulate);
}

// Tile shapes of the convolution, most work per wave first: (NB, PB, KS).
// The first one that gives at least kConvMinWG workgroups is used (else the
// one with the most workgroups), so small late layers still fill the chip.
struct ConvShape {
  int nb, pb, ks;
};
const ConvShape kConvShapes[] = {{4, 2, 1}, {4, 1, 1}, {2, 2, 1}, {2, 1, 1}, {4, 1, 2},
                                 {2, 1, 2}, {1, 1, 2}, {2, 1, 4}, {1, 1, 4}};
constexpr int64_t kConvMinWG = 1024;

int conv_shape(int64_t pixels, int cin, int cout) {
  int best = -1;
  int64_t best_wg = -1;
  for (int k = 0; k < (int)(sizeof(kConvShapes) / sizeof(kConvShapes[0])); ++k) {
    const ConvShape& c = kConvShapes[k];
    const int64_t px = 16 * c.pb * (4 / c.ks);
    if (cout % (16 * c.nb) || pixels % px || cin / 32 < c.ks) continue;
    const int64_t wg = pixels / px * (cout / (16 * c.nb));
    if (wg >= kConvMinWG) return k;
    if (wg > best_wg) best_wg = wg, best = k;
  }
  return best >= 0 ? best : 3;
}

template <int SPLIT>
void launch_conv_shape(int k, sg_net* n, const Tensor& x, const float* xscale,
                       const unsigned short* wh, const unsigned short* wl, Tensor& z, int cin,
                       int cout, int accumulate) {
  switch (k) {
    case 0: return launch_conv<SPLIT, 4, 2, 1>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 1: return launch_conv<SPLIT, 4, 1, 1>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 2: return launch_conv<SPLIT, 2, 2, 1>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 3: return launch_conv<SPLIT, 2, 1, 1>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 4: return launch_conv<SPLIT, 4, 1, 2>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 5: return launch_conv<SPLIT, 2, 1, 2>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 6: return launch_conv<SPLIT, 1, 1, 2>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    case 7: return launch_conv<SPLIT, 2, 1, 4>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
    default: return launch_conv<SPLIT, 1, 1, 4>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  }
}

template <int SPLIT, int PB, int NB, bool WL, int WT>
void launch_convt(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                  const unsigned short* wl, Tensor& z, int cin, int cout, int accumulate) {
  constexpr int CT = PB * 16 * NB;
  dim3 grid((unsigned)((int64_t)n->B * x.H * x.W / 64), (unsigned)(cout / CT));
  hipLaunchKernelGGL((k_convt<SPLIT, PB, NB, WL, WT>), grid, dim3(256), 0, n->stream,
                     (const float*)x.p, xscale, wh, wl, z.p, x.H, x.W, cin, cout, n->circular,
                     accumulate);
}

// k_convw where it has a workgroup for every CU (256 pixels x 32 channels
// each); two workgroups share a CU, each running through its share.  With
// fewer, k_convs spreads the layer over more CUs (128 x 128 pixels, 64
// channels, batch 1: 128 workgroups of k_convw 11.9 us, 512 of k_convs 9.8).
template <int SPLIT, int WT>
bool conv_wide(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
               const unsigned short* wl, Tensor& z, int cin, int cout, int epi, const ConvEpi& E) {
  const int64_t work = (int64_t)n->B * x.H * x.W / 256 * (cout / 32);
  if (x.W % WT || x.H % (256 / WT) || work < 256) return false;
  auto fn = epi == EPI_POOL   ? &k_convw<SPLIT, WT, EPI_POOL>
            : epi == EPI_UP   ? &k_convw<SPLIT, WT, EPI_UP>
            : epi == EPI_FILM ? &k_convw<SPLIT, WT, EPI_FILM>
                              : &k_convw<SPLIT, WT, EPI_NONE>;
  // (the last layer's rows are a multiple of 128 pixels)
  if constexpr (WT == 32)
    if (epi == EPI_POST) fn = &k_convw<SPLIT, WT, EPI_POST>;
  hipLaunchKernelGGL(fn, dim3((unsigned)(work < 512 ? work : 512)), dim3(256), 0, n->stream,
                     (const float*)x.p, xscale, wh, wl, z.p, x.H, x.W, cin, cout, n->circular,
                     (int)work, E);
  return true;
}

// k_convs for the layers with fewer pixels (hi/lo operands)
template <int NG, int TR>
void launch_convs(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                  const unsigned short* wl, Tensor& z, int cout, int epi, const ConvEpi& E) {
  auto fn = epi == EPI_POOL   ? &k_convs<3, NG, TR, EPI_POOL>
            : epi == EPI_UP   ? &k_convs<3, NG, TR, EPI_UP>
                              : &k_convs<3, NG, TR, EPI_NONE>;
  if constexpr (NG == 1)
    if (epi == EPI_POST) fn = &k_convs<3, NG, TR, EPI_POST>;
  hipLaunchKernelGGL(fn, dim3((unsigned)((int64_t)n->B * x.H * x.W / (16 * TR) * (cout / 32))),
                     dim3(128 * NG), 0, n->stream, (const float*)x.p, xscale, wh, wl, z.p, x.H,
                     x.W, cout, n->circular, E);
}

bool conv_small(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                const unsigned short* wl, Tensor& z, int cin, int cout, int epi,
                const ConvEpi& E) {
  if (x.W % 16 || x.H % 8) return false;
  const int64_t work = (int64_t)n->B * x.H * x.W / 64 * (cout / 32);
  switch (cin) {
    case 32: launch_convs<1, 4>(n, x, xscale, wh, wl, z, cout, epi, E); return true;
    case 64: launch_convs<2, 4>(n, x, xscale, wh, wl, z, cout, epi, E); return true;
    case 128:
      // (a workgroup fills its CU)
      if (work > 256)
        launch_convs<4, 8>(n, x, xscale, wh, wl, z, cout, epi, E);
      else
        launch_convs<4, 4>(n, x, xscale, wh, wl, z, cout, epi, E);
      return true;
  }
  return false;
}

// The 64-pixel tiled kernel, where the row is a multiple of 64 pixels or 32 or
// 16 pixels long and it gives at least 256 workgroups: 64 output channels per
// workgroup (2 x 2 waves of 32 x 32) when that still gives 512 workgroups, else
// 32 (4 waves of 16 pixels x 32 channels), or 16 where 32 gives fewer than 256
// workgroups.  In mode 0 it serves plain BF16's layers with few pixels, with
// the weights staged in LDS too (batch 1, 128 x 384: 161 us a forward call,
// 193 with the weights from global memory).
template <int SPLIT, int WT>
void conv_tiled_w(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                  const unsigned short* wl, Tensor& z, int cin, int cout, int accumulate) {
  const int64_t tiles = (int64_t)n->B * x.H * x.W / 64;
  const bool few = tiles * (cout / 32) < 256;
  if (cout % 64 == 0 && tiles * (cout / 64) >= 512)
    return launch_convt<SPLIT, 2, 2, false, WT>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  if constexpr (SPLIT == 1) {
    if (n->conv_mode == 0) {
      if (few)
        launch_convt<SPLIT, 1, 1, true, WT>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
      else
        launch_convt<SPLIT, 1, 2, true, WT>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
      return;
    }
  }
  if (few)
    launch_convt<SPLIT, 1, 1, false, WT>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  else
    launch_convt<SPLIT, 1, 2, false, WT>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
}

template <int SPLIT>
bool conv_tiled(sg_net* n, const Tensor& x, const float* xscale, const unsigned short* wh,
                const unsigned short* wl, Tensor& z, int cin, int cout, int accumulate) {
  if (n->conv_mode == 1 || cin % 32 || cout % 32 || ((int64_t)x.H * x.W) % 64) return false;
  // too few workgroups to fill the chip even with 16 output channels per
  // workgroup: the direct kernel splits the reduction over waves instead
  if ((int64_t)n->B * x.H * x.W / 64 * (cout / 16) < 256) return false;
  if (x.W % 64 == 0)
    conv_tiled_w<SPLIT, 64>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  else if (x.W == 32)
    conv_tiled_w<SPLIT, 32>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  else if (x.W == 16)
    conv_tiled_w<SPLIT, 16>(n, x, xscale, wh, wl, z, cin, cout, accumulate);
  else
    return false;
  return true;
}

// epi: what follows the layer (k_convw's epilogues); returns whether it was done
bool conv(sg_net* n, const Tensor& x, const float* xscale, int l, Tensor& z, bool backward,
          int accumulate, int epi = EPI_NONE, const ConvEpi& E = ConvEpi{}) {
  const LayerSpec& L = kLayers[l];
  const int cin = backward ? L.cout : L.cin, cout = backward ? L.cin : L.cout;
  const unsigned short* wh = (backward ? n->wbh : n->wfh) + n->P.wq_off[l];
  const unsigned short* wl = (backward ? n->wbl : n->wfl) + n->P.wq_off[l];
  const int64_t pixels = (int64_t)n->B * x.H * x.W;
  if (n->conv_mode == 0 && !accumulate) {
    if (n->P.split == 3 ? conv_wide<3, 32>(n, x, xscale, wh, wl, z, cin, cout, epi, E) ||
                              conv_wide<3, 16>(n, x, xscale, wh, wl, z, cin, cout, epi, E)
                        : conv_wide<1, 32>(n, x, xscale, wh, wl, z, cin, cout, epi, E) ||
                              conv_wide<1, 16>(n, x, xscale, wh, wl, z, cin, cout, epi, E))
      return true;
    const int e = epi == EPI_FILM ? EPI_NONE : epi;
    if (n->P.split == 3 && conv_small(n, x, xscale, wh, wl, z, cin, cout, e, E)) return e == epi;
  }
  // modes 1 and 2, and plain BF16's layers with few pixels, whose sums keep the
  // order they have there; the tiled kernel splits its input tiles itself
  if (n->P.split == 3 ? conv_tiled<3>(n, x, xscale, wh, wl, z, cin, cout, accumulate)
                      : conv_tiled<1>(n, x, xscale, wh, wl, z, cin, cout, accumulate))
    return false;
  // the direct kernel splits its input (with its gain) into BF16 hi/lo parts
  // as it reads it
  const int k = conv_shape(pixels, cin, cout);
  if (n->P.split == 3)
    launch_conv_shape<3>(k, n, x, xscale, wh, wl, z, cin, cout, accumulate);
  else
    launch_conv_shape<1>(k, n, x, xscale, wh, wl, z, cin, cout, accumulate);
  return false;
}

void pool(sg_net* n, const Tensor& in, const float* scale, Tensor& out) {
  const int64_t e = (int64_t)n->B * out.H * out.W * out.C / 4;  // 4 channels per thread
  hipLaunchKernelGGL(k_pool, dim3(grid1(e)), dim3(RT), 0, n->stream, in.p, scale, out.p, n->B,
                     out.H, out.W, out.C);
}

void upadd(sg_net* n, const Tensor& coarse, const float* sc, const Tensor& skip, const float* ss,
           Tensor& out) {
  const int64_t e = (int64_t)n->B * out.H * out.W * out.C / 4;  // 4 channels per thread
  hipLaunchKernelGGL(k_upadd, dim3(grid1(e)), dim3(RT), 0, n->stream, coarse.p, sc, skip.p, ss,
                     out.p, n->B, out.H, out.W, out.C);
}

// the input map and the first layer in one launch, with k_convw's tiles, and
// one workgroup per sample for what k_stats forms
bool conv_in(sg_net* n, const float* in, Tensor& z, const SampleStats& st) {
  const int64_t work = (int64_t)n->B * z.H * z.W / 256;
  // (its products take 4 taps at a time, another order of sums: see k_convw)
  if (n->conv_mode != 0 || n->P.split != 3 || z.W % 32 || z.H % 8 || work < 256) return false;
  hipLaunchKernelGGL(k_conv_in<3>, dim3((unsigned)(work + n->B)), dim3(256), 0, n->stream, in,
                     (const unsigned short*)n->wfh + n->P.wq_off[L_IN],
                     (const unsigned short*)n->wfl + n->P.wq_off[L_IN], z.p, z.H, z.W,
                     n->circular, (int)work, st);
  return true;
}

// layer l followed by the pooling of its output
void conv_pool(sg_net* n, const Tensor& x, const float* xscale, int l, Tensor& pooled) {
  ConvEpi E{pooled.p, n->gam[l], nullptr, nullptr, nullptr, nullptr, 1, nullptr};
  if (!conv(n, x, xscale, l, n->z[l], false, 0, EPI_POOL, E)) pool(n, n->z[l], n->gam[l], pooled);
}

// layer l followed by the skip sum up(gain y) + gain_s z_skip; keep: the
// layer's own output is needed again (the backward pass)
void conv_up(sg_net* n, const Tensor& x, const float* xscale, int l, int skip, Tensor& out,
             int keep) {
  ConvEpi E{out.p, n->gam[l], n->z[skip].p, n->gam[skip], nullptr, nullptr, keep, nullptr};
  if (!conv(n, x, xscale, l, n->z[l], false, 0, EPI_UP, E))
    upadd(n, n->z[l], n->gam[l], n->z[skip], n->gam[skip], out);
}

void prep_weights(sg_net* n) {
  static_assert(NL <= MAXL, "PrepArgs size");
  PrepArgs a;
  a.n = NL;
  a.at[0] = 0;
  for (int l = 0; l < NL; ++l) {
    a.woff[l] = n->P.woff[l];
    a.wq_off[l] = n->P.wq_off[l];
    a.cin[l] = kLayers[l].cin;
    a.cout[l] = kLayers[l].cout;
    a.at[l + 1] = a.at[l] + 9 * kLayers[l].cin * kLayers[l].cout;
  }
  hipLaunchKernelGGL(k_prep_weights, dim3((unsigned)(a.at[NL] / 256)), dim3(256), 0, n->stream,
                     (const float*)n->param, a, n->wfh, n->wfl, n->wbh, n->wbl);
  n->weights_ready = true;
}

// out: the physical output fields, or null for a training step (which keeps
// every layer's input and output for the backward pass and forms the loss
// from z_out)
lbm_status forward(sg_net* n, const float* in, int B, int circular, float* out) {
  Plan& P = n->P;
  n->B = B;
  n->circular = circular;
  n->in = in;
  if (!n->weights_ready) prep_weights(n);
  const int HW = P.H * P.W;
  SampleStats st{n->spart, stats_chunks(HW), HW, n->s, n->T, {}, {}, {}};
  for (int l = 0; l < NL; ++l) {
    st.a[l] = n->param + P.aoff[l];
    st.g[l] = n->gam[l];
    st.cout[l] = kLayers[l].cout;
  }
  hipLaunchKernelGGL(k_stats_partial, dim3(st.chunks, B), dim3(RT), 0, n->stream, in, HW,
                     n->spart);
  Tensor x0{n->x0, P.H, P.W, CP};
  Tensor* z = n->z;
  float** gm = n->gam;
  // the input map goes into the first layer and the output map into the last
  // where x0 and z_out are not needed again
  const bool fused = !out ? false : conv_in(n, in, z[L_IN], st);
  if (!fused) {
    hipLaunchKernelGGL(k_stats, dim3(B), dim3(RT), 0, n->stream, st);
    hipLaunchKernelGGL(k_pre, dim3(grid1((int64_t)B * HW)), dim3(RT), 0, n->stream, in, B, HW,
                       n->s, n->x0);
    conv(n, x0, nullptr, L_IN, z[L_IN], false, 0);
  }
  conv(n, z[L_IN], gm[L_IN], L_E0A, z[L_E0A], false, 0);
  conv_pool(n, z[L_E0A], gm[L_E0A], L_E0B, n->pool[0]);
  conv(n, n->pool[0], nullptr, L_E1A, z[L_E1A], false, 0);
  conv_pool(n, z[L_E1A], gm[L_E1A], L_E1B, n->pool[1]);
  conv(n, n->pool[1], nullptr, L_E2A, z[L_E2A], false, 0);
  conv_pool(n, z[L_E2A], gm[L_E2A], L_E2B, n->pool[2]);
  conv(n, n->pool[2], nullptr, L_E3A, z[L_E3A], false, 0);
  conv_up(n, z[L_E3A], gm[L_E3A], L_E3B, L_E2B, n->up[2], !out);
  conv(n, n->up[2], nullptr, L_D2A, z[L_D2A], false, 0);
  conv_up(n, z[L_D2A], gm[L_D2A], L_D2B, L_E1B, n->up[1], !out);
  conv(n, n->up[1], nullptr, L_D1A, z[L_D1A], false, 0);
  conv_up(n, z[L_D1A], gm[L_D1A], L_D1B, L_E0B, n->up[0], !out);
  conv(n, n->up[0], nullptr, L_D0A, z[L_D0A], false, 0);
  conv(n, z[L_D0A], gm[L_D0A], L_D0B, z[L_D0B], false, 0);
  if (!out) {
    conv(n, z[L_D0B], gm[L_D0B], L_OUT, z[L_OUT], false, 0);
    return launch_check("surrogate forward");
  }
  ConvEpi E{};
  E.out = out;
  E.gain = gm[L_OUT];
  E.in = in;
  E.sv = n->s;
  if (!conv(n, z[L_D0B], gm[L_D0B], L_OUT, z[L_OUT], false, 0, EPI_POST, E))
    hipLaunchKernelGGL(k_post, dim3(grid1((int64_t)B * HW)), dim3(RT), 0, n->stream, in,
                       (const float*)z[L_OUT].p, (const float*)gm[L_OUT], (const float*)n->s, B,
                       HW, out);
  return launch_check("surrogate forward");
}

// data gradient: conv with flipped, transposed weights of (gamma * gy).  The
// FiLM sums of layer prev go with it where the chunks they leave to add in a
// row are not more than FILM_TILES per sample (k_film_grad_part's are as many
// at batch 1 of 512 x 512).
constexpr int FILM_TILES = 1024;
void data_grad(sg_net* n, int l, const Tensor& gy, Tensor& gin, int accumulate, int prev) {
  if (!gin.p) return;
  const int tiles = gin.H * gin.W / 256;
  if (prev < 0 || tiles > FILM_TILES) {
    conv(n, gy, n->gam[l], l, gin, true, accumulate);
    return;
  }
  ConvEpi E{};
  E.skip = n->z[prev].p;
  E.part = n->fpart[prev];
  if (conv(n, gy, n->gam[l], l, gin, true, accumulate, EPI_FILM, E)) n->fchunks[prev] = tiles;
}

// backward through conv layer l: g_y (dL/dy_l) -> parameter gradients and
// dL/d(input of l) written to gin (accumulated if accumulate); prev >= 0: gin
// is dL/dy of that layer, whose FiLM sums the convolution then forms as well
void conv_back(sg_net* n, int l, const Tensor& gy, const Tensor& xin, const float* xscale,
               Tensor& gin, int accumulate, int prev = -1) {
  Plan& P = n->P;
  const LayerSpec& L = kLayers[l];
  const Tensor& zl = n->z[l];
  const int HW = zl.H * zl.W;
  // FiLM coefficients: the chunk sums now, the rest for all layers at the end
  if (!n->fchunks[l]) {
    const int S = film_chunks(n->B, HW);
    hipLaunchKernelGGL(k_film_grad_part, dim3((unsigned)(n->B * S)), dim3(RT), 0, n->stream, gy.p,
                       zl.p, HW, L.cout, S, n->fpart[l]);
    n->fchunks[l] = S;
  }
  // weights: dW = sum (gamma * gy) (x) (xscale * x)
  const int64_t pixels = (int64_t)n->B * HW;
  const int wt = zl.W % 32 == 0 && zl.H % 8 == 0 ? 32 : zl.W % 16 == 0 && zl.H % 16 == 0 ? 16 : 0;
  const int64_t ntile = pixels / 256, nct = (L.cout / 32) * (L.cin / 32);
  if (n->conv_mode != 1 && wt && ntile * nct >= 128) {
    // two workgroups per CU
    int64_t ng = 512 / nct;
    const int64_t cap = n->P.wpart_floats / ((int64_t)9 * L.cout * L.cin);
    ng = ng > cap ? cap : ng;
    ng = ng > ntile ? ntile : ng;
    auto fn = P.split == 3 ? (wt == 32 ? &k_wgradw<3, 32> : &k_wgradw<3, 16>)
                           : (wt == 32 ? &k_wgradw<1, 32> : &k_wgradw<1, 16>);
    hipLaunchKernelGGL(fn, dim3((unsigned)(ng * nct)), dim3(256), 0, n->stream, gy.p,
                       (const float*)n->gam[l], xin.p, xscale, n->wpart, zl.H, zl.W, L.cin, L.cout,
                       n->circular, (int)ntile, (int)ng);
    const int64_t nw = (int64_t)9 * L.cout * L.cin;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((nw + 63) / 64)), dim3(RT), 0, n->stream,
                       (const float*)n->wpart, (int)ng, L.cin, L.cout, n->grad + P.woff[l]);
    data_grad(n, l, gy, gin, accumulate, prev);
    return;
  }
  const bool rows_fit = zl.W % 64 == 0 || (64 % zl.W == 0 && zl.H % (64 / zl.W) == 0);
  if (n->conv_mode != 1 && rows_fit && L.cin % 32 == 0 && L.cout % 32 == 0) {
    // LDS-staged kernel: ~256 workgroups (one per CU: 92 KB of LDS), as many
    // pixel-block groups as the partials' buffer holds
    const int64_t nblocks = pixels / 64;
    const int tiles = (L.cout / 32) * (L.cin / 32);
    int64_t ng = 256 / tiles;
    const int64_t cap = n->P.wpart_floats / ((int64_t)9 * L.cout * L.cin);
    ng = ng > cap ? cap : ng;
    ng = ng > nblocks ? nblocks : ng;
    ng = ng < 1 ? 1 : ng;
    if (P.split == 3)
      hipLaunchKernelGGL((k_wgradt<3>), dim3((unsigned)ng, (unsigned)tiles), dim3(256), 0,
                         n->stream, gy.p, (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B,
                         zl.H, zl.W, L.cin, L.cout, n->circular);
    else
      hipLaunchKernelGGL((k_wgradt<1>), dim3((unsigned)ng, (unsigned)tiles), dim3(256), 0,
                         n->stream, gy.p, (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B,
                         zl.H, zl.W, L.cin, L.cout, n->circular);
    const int64_t nw = (int64_t)9 * L.cout * L.cin;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((nw + 63) / 64)), dim3(RT), 0, n->stream,
                       (const float*)n->wpart, (int)ng, L.cin, L.cout, n->grad + P.woff[l]);
    data_grad(n, l, gy, gin, accumulate, prev);
    return;
  }
  int nsplit = 1;
  while (nsplit < 64 && pixels / (nsplit * 2) >= 2048 && (pixels % (nsplit * 2 * 128)) == 0)
    nsplit *= 2;
  const int64_t pps = pixels / nsplit;
  const int ni = L.cin >= 64 ? 4 : 2;
  dim3 grid((unsigned)(9 * (L.cout / 16) * (L.cin / (16 * ni))), (unsigned)nsplit);
  if (P.split == 3) {
    if (ni == 4)
      hipLaunchKernelGGL((k_wgrad<3, 4>), grid, dim3(256), 0, n->stream, gy.p,
                         (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B, zl.H, zl.W,
                         L.cin, L.cout, n->circular, pps);
    else
      hipLaunchKernelGGL((k_wgrad<3, 2>), grid, dim3(256), 0, n->stream, gy.p,
                         (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B, zl.H, zl.W,
                         L.cin, L.cout, n->circular, pps);
  } else {
    if (ni == 4)
      hipLaunchKernelGGL((k_wgrad<1, 4>), grid, dim3(256), 0, n->stream, gy.p,
                         (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B, zl.H, zl.W,
                         L.cin, L.cout, n->circular, pps);
    else
      hipLaunchKernelGGL((k_wgrad<1, 2>), grid, dim3(256), 0, n->stream, gy.p,
                         (const float*)n->gam[l], xin.p, xscale, n->wpart, n->B, zl.H, zl.W,
                         L.cin, L.cout, n->circular, pps);
  }
  const int64_t nw = (int64_t)9 * L.cout * L.cin;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((nw + 63) / 64)), dim3(RT), 0, n->stream,
                     (const float*)n->wpart, nsplit, L.cin, L.cout, n->grad + P.woff[l]);
  data_grad(n, l, gy, gin, accumulate, prev);
}

void up_back(sg_net* n, const Tensor& g, Tensor& out) {
  const int64_t e = (int64_t)n->B * out.H * out.W * out.C / 4;  // 4 channels per thread
  hipLaunchKernelGGL(k_up_back, dim3(grid1(e)), dim3(RT), 0, n->stream, g.p, out.p, n->B, out.H,
                     out.W, out.C);
}

void pool_back(sg_net* n, const Tensor& g, const float* add, Tensor& out) {
  const int64_t e = (int64_t)n->B * out.H * out.W * out.C / 4;  // 4 channels per thread
  hipLaunchKernelGGL(k_pool_back, dim3(grid1(e)), dim3(RT), 0, n->stream, g.p, add, out.p, n->B,
                     out.H, out.W, out.C);
}

lbm_status backward(sg_net* n) {
  Tensor* z = n->z;
  Tensor* g = n->g;
  float** gm = n->gam;
  Tensor x0{n->x0, n->P.H, n->P.W, CP};
  Tensor none;
  for (int l = 0; l < NL; ++l) n->fchunks[l] = 0;
  // g[L_OUT] holds dL/dy_out from the loss kernel
  conv_back(n, L_OUT, g[L_OUT], z[L_D0B], gm[L_D0B], g[L_D0B], 0, L_D0B);
  conv_back(n, L_D0B, g[L_D0B], z[L_D0A], gm[L_D0A], g[L_D0A], 0, L_D0A);
  conv_back(n, L_D0A, g[L_D0A], n->up[0], nullptr, n->gup[0], 0);       // dL/du0
  up_back(n, n->gup[0], g[L_D1B]);                                        // dL/dy_d1b
  conv_back(n, L_D1B, g[L_D1B], z[L_D1A], gm[L_D1A], g[L_D1A], 0, L_D1A);
  conv_back(n, L_D1A, g[L_D1A], n->up[1], nullptr, n->gup[1], 0);       // dL/du1
  up_back(n, n->gup[1], g[L_D2B]);
  conv_back(n, L_D2B, g[L_D2B], z[L_D2A], gm[L_D2A], g[L_D2A], 0, L_D2A);
  conv_back(n, L_D2A, g[L_D2A], n->up[2], nullptr, n->gup[2], 0);       // dL/du2
  up_back(n, n->gup[2], g[L_E3B]);
  conv_back(n, L_E3B, g[L_E3B], z[L_E3A], gm[L_E3A], g[L_E3A], 0, L_E3A);
  conv_back(n, L_E3A, g[L_E3A], n->pool[2], nullptr, n->gpool[2], 0);   // dL/dp3
  pool_back(n, n->gpool[2], n->gup[2].p, g[L_E2B]);                      // + skip from u2
  conv_back(n, L_E2B, g[L_E2B], z[L_E2A], gm[L_E2A], g[L_E2A], 0, L_E2A);
  conv_back(n, L_E2A, g[L_E2A], n->pool[1], nullptr, n->gpool[1], 0);
  pool_back(n, n->gpool[1], n->gup[1].p, g[L_E1B]);
  conv_back(n, L_E1B, g[L_E1B], z[L_E1A], gm[L_E1A], g[L_E1A], 0, L_E1A);
  conv_back(n, L_E1A, g[L_E1A], n->pool[0], nullptr, n->gpool[0], 0);
  pool_back(n, n->gpool[0], n->gup[0].p, g[L_E0B]);
  conv_back(n, L_E0B, g[L_E0B], z[L_E0A], gm[L_E0A], g[L_E0A], 0, L_E0A);
  conv_back(n, L_E0A, g[L_E0A], z[L_IN], gm[L_IN], g[L_IN], 0, L_IN);
  conv_back(n, L_IN, g[L_IN], x0, nullptr, none, 0);
  FilmArgs a;
  int groups = 0;
  for (int l = 0; l < NL; ++l) {
    a.part[l] = n->fpart[l];
    a.da[l] = n->grad + n->P.aoff[l];
    a.cout[l] = kLayers[l].cout;
    a.S[l] = n->fchunks[l];
    groups += kLayers[l].cout / 32;
  }
  hipLaunchKernelGGL(k_film_grad_coef, dim3((unsigned)groups), dim3(RT), 0, n->stream, a,
                     (const float*)n->T, n->B);
  return launch_check("surrogate backward");
}

}  // namespace

extern "C" {

size_t sg_workspace_bytes(const sg_config* cfg) {
  Plan P;
  if (make_plan(cfg, &P) != LBM_OK) return 0;
  return P.bytes;
}

int64_t sg_param_count(void) {
  int64_t np = 0;
  for (int l = 0; l < NL; ++l) np += (int64_t)kLayers[l].cout * (kLayers[l].cin * 9 + NBASIS);
  return np;
}

lbm_status sg_create(const sg_config* cfg, void* d_ws, size_t ws_bytes, void* hip_stream,
                     sg_net** out) {
  if (!out) return fail(LBM_E_ARG, "null out");
  if (!d_ws || ((uintptr_t)d_ws & 255)) return fail(LBM_E_ARG, "workspace null or misaligned");
  sg_net* n = new (std::nothrow) sg_net();
  if (!n) return fail(LBM_E_ARG, "out of host memory");
  lbm_status s = make_plan(cfg, &n->P);
  if (s == LBM_OK && ws_bytes < n->P.bytes) s = fail(LBM_E_SPACE, "workspace too small");
  if (s) {
    delete n;
    return s;
  }
  Plan& P = n->P;
  char* w = (char*)d_ws;
  n->ws = w;
  n->stream = (hipStream_t)hip_stream;
  n->param = (float*)(w + P.o_param);
  n->wfh = (unsigned short*)(w + P.o_wfh);
  n->wfl = (unsigned short*)(w + P.o_wfl);
  n->wbh = (unsigned short*)(w + P.o_wbh);
  n->wbl = (unsigned short*)(w + P.o_wbl);
  n->s = (float*)(w + P.o_s);
  n->T = (float*)(w + P.o_T);
  for (int l = 0; l < NL; ++l) n->gam[l] = (float*)(w + P.o_gam) + (size_t)l * P.B * 128;
  n->part = (double*)(w + P.o_part);
  n->spart = (double*)(w + P.o_spart);
  n->loss = (double*)(w + P.o_loss);
  n->x0 = (float*)(w + P.o_x0);
  for (int l = 0; l < NL; ++l) {
    const int lv = kLayers[l].level;
    n->z[l] = Tensor{(float*)(w + P.o_z[l]), level_h(P, lv), level_w(P, lv), kLayers[l].cout};
  }
  const int pc[3] = {32, 64, 128};
  for (int k = 0; k < 3; ++k) {
    n->pool[k] = Tensor{(float*)(w + P.o_pool[k]), level_h(P, k + 1), level_w(P, k + 1), pc[k]};
    n->up[k] = Tensor{(float*)(w + P.o_up[k]), level_h(P, k), level_w(P, k), pc[k]};
  }
  if (P.train) {
    n->grad = (float*)(w + P.o_grad);
    n->m = (float*)(w + P.o_m);
    n->v = (float*)(w + P.o_v);
    for (int l = 0; l < NL; ++l) n->fpart[l] = (double*)(w + P.o_fpart[l]);
    for (int l = 0; l < NL; ++l) {
      const int lv = kLayers[l].level;
      n->g[l] = Tensor{(float*)(w + P.o_g[l]), level_h(P, lv), level_w(P, lv), kLayers[l].cout};
    }
    for (int k = 0; k < 3; ++k) {
      n->gpool[k] = Tensor{(float*)(w + P.o_gpool[k]), level_h(P, k + 1), level_w(P, k + 1), pc[k]};
      n->gup[k] = Tensor{(float*)(w + P.o_gup[k]), level_h(P, k), level_w(P, k), pc[k]};
    }
    n->wpart = (float*)(w + P.o_wpart);
  }
  n->adam_step = 0;
  n->weights_ready = false;
  *out = n;
  return LBM_OK;
}

lbm_status sg_set_conv_mode(sg_net* n, int32_t mode) {
  if (!n) return fail(LBM_E_ARG, "null net");
  if (mode < 0 || mode > 2) return fail(LBM_E_ARG, "conv mode must be 0, 1 or 2");
  n->conv_mode = mode;
  return LBM_OK;
}

lbm_status sg_destroy(sg_net* n) {
  delete n;
  return LBM_OK;
}

lbm_status sg_set_params(sg_net* n, const float* d_params) {
  if (!n || !d_params) return fail(LBM_E_ARG, "null argument");
  lbm_status s = hip_check(hipMemcpyAsync(n->param, d_params, n->P.nparam * 4,
                                          hipMemcpyDeviceToDevice, n->stream),
                           "set params");
  if (s) return s;
  n->weights_ready = false;
  if (n->P.train) {
    s = hip_check(hipMemsetAsync(n->m, 0, n->P.nparam * 4, n->stream), "reset adam");
    if (s == LBM_OK) s = hip_check(hipMemsetAsync(n->v, 0, n->P.nparam * 4, n->stream), "reset adam");
    n->adam_step = 0;
  }
  return s;
}

lbm_status sg_get_params(sg_net* n, float* d_params) {
  if (!n || !d_params) return fail(LBM_E_ARG, "null argument");
  return hip_check(hipMemcpyAsync(d_params, n->param, n->P.nparam * 4, hipMemcpyDeviceToDevice,
                                  n->stream),
                   "get params");
}

lbm_status sg_get_grads(sg_net* n, float* d_grads) {
  if (!n || !d_grads) return fail(LBM_E_ARG, "null argument");
  if (!n->P.train) return fail(LBM_E_STATE, "network created without training buffers");
  return hip_check(hipMemcpyAsync(d_grads, n->grad, n->P.nparam * 4, hipMemcpyDeviceToDevice,
                                  n->stream),
                   "get grads");
}

lbm_status sg_forward(sg_net* n, const float* d_in, int32_t batch, int32_t circular,
                      float* d_out) {
  if (!n || !d_in || !d_out) return fail(LBM_E_ARG, "null argument");
  if (batch < 1 || batch > n->P.B) return fail(LBM_E_ARG, "batch out of range");
  return forward(n, d_in, batch, circular ? 1 : 0, d_out);
}

lbm_status sg_train_step(sg_net* n, const float* d_in, const float* d_target, int32_t batch,
                         int32_t circular, float lr, double* h_loss) {
  if (!n || !d_in || !d_target) return fail(LBM_E_ARG, "null argument");
  if (!n->P.train) return fail(LBM_E_STATE, "network created without training buffers");
  if (batch < 1 || batch > n->P.B) return fail(LBM_E_ARG, "batch out of range");
  lbm_status s = forward(n, d_in, batch, circular ? 1 : 0, nullptr);
  if (s) return s;
  const int HW = n->P.H * n->P.W;
  const int64_t np = (int64_t)batch * HW;
  const unsigned nb = grid1(np);
  hipLaunchKernelGGL(k_loss, dim3(nb), dim3(RT), 0, n->stream, d_in, d_target,
                     (const float*)n->z[L_OUT].p, (const float*)n->gam[L_OUT],
                     (const float*)n->s, batch, HW, (float)(1.0 / (5.0 * np)), n->g[L_OUT].p,
                     n->part);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(RT), 0, n->stream, (const double*)n->part,
                     (int)nb, n->loss);
  s = backward(n);
  if (s) return s;
  if (lr > 0.f) {
    n->adam_step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)n->adam_step), c2 = 1.f - powf(b2, (float)n->adam_step);
    hipLaunchKernelGGL(k_adam, dim3(grid1(n->P.nparam)), dim3(RT), 0, n->stream, n->param,
                       (const float*)n->grad, n->m, n->v, n->P.nparam, lr, b1, b2, 1e-8f, c1, c2);
    n->weights_ready = false;
    prep_weights(n);
  }
  s = launch_check("surrogate train step");
  if (s) return s;
  if (h_loss) {
    double lsum;
    s = hip_check(hipMemcpyAsync(&lsum, n->loss, 8, hipMemcpyDeviceToHost, n->stream), "loss copy");
    if (s) return s;
    s = hip_check(hipStreamSynchronize(n->stream), "loss sync");
    if (s) return s;
    *h_loss = lsum / (5.0 * np);
  }
  return LBM_OK;
}

}  // extern "C"
