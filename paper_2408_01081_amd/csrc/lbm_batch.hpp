// Device code of the batched lattices that two translation units instantiate:
// the instance table and the passes over the packed fields (initialisation,
// moments).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm.h"
#include "lbm_init.hpp"
#include "lbm_kernels.hpp"
#include "lbm_step.hpp"

namespace lbmb {

using namespace lbmk;

constexpr int BT = 256;  // threads per workgroup of the batched kernels

struct InstDesc {
  Grid g;
  int64_t off;    // float offset of the instance's state in each pool
  int64_t node0;  // first node of the instance in packed field arrays
  int tile0;      // first row-segment tile of the instance
  int tiles_x;    // row segments per row
  int bc;
  float kK, km, cK, cmu, rho;
  InitConst ic;
  double kw[NQ][NC][NC];  // norm weights
  const float* W;         // wall table or null
  const float* T;
  int rank;
  float* V;  // Dirichlet instances: [8][2 (nx + ny)][2] wall velocities of a blocked launch's steps
};

// the instance of a node, one of lo .. hi
__device__ inline int find_instance(const InstDesc* __restrict__ d, int lo, int hi, int64_t node) {
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (d[mid].node0 <= node)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// fn(instance, x, y) for this thread's node of the packed node range, of which
// workgroup `block` takes BT consecutive nodes.  They lie in one instance or in
// a run of a few, which the whole workgroup walks together, so the descriptors
// come through scalar loads and no thread searches for its own (128 instances
// of 128 rows, 3.3 M nodes: FP64 initialisation 237 -> 81 us with the form of
// init_node above).  MANY: in workgroups of more than WALK instances each thread
// finds its own, since the walk is one instance's latency after another (4096
// instances of 4 x 4, 16 per workgroup: 25 us walking, 18 so; 1280 of 3 x 2 to
// 7 x 8: 23 and 18; 16384 of 1 x 1: 209 and 21); for batches with such workgroups
// only, as the second copy of fn takes registers (32 of 128 x 128, FP32
// initialisation 12.3 us without it, 14.1 with it).
constexpr int WALK = 4;

template <bool MANY, typename FN>
__device__ inline void for_block_instances(const InstDesc* __restrict__ descs, int n, int block,
                                           FN fn) {
  const int64_t first = (int64_t)block * BT, node = first + threadIdx.x;
  auto at = [&](const InstDesc& d) {
    const int64_t loc = node - d.node0;
    if (loc < 0 || loc >= (int64_t)d.g.nx * d.g.ny) return;
    // (instances whose node count fits 31 bits: a 32-bit division)
    const int y = (int64_t)d.g.nx * d.g.ny <= 0x7fffffff ? (int)((unsigned)loc / (unsigned)d.g.nx)
                                                          : (int)(loc / d.g.nx);
    fn(d, (int)(loc - (int64_t)y * d.g.nx), y);
  };
  int i = find_instance(descs, 0, n - 1, first);
  if (MANY && i + WALK < n && descs[i + WALK].node0 < first + BT) {
    at(descs[find_instance(descs, i, i + BT - 1 < n ? i + BT - 1 : n - 1, node)]);
    return;
  }
  for (; i < n; ++i) {
    const InstDesc& d = descs[i];
    if (d.node0 >= first + BT) break;
    at(d);
  }
}

// packed = 0: v0 [..][2][ny][nx] and s0 [..][3][ny][nx] separate arrays;
// packed = 1: one array [..][5][ny][nx] = (v, sigma_bar) in s0's place (v0 unused).
template <typename T, bool NT, bool MANY>
__global__ __launch_bounds__(BT) void k_batch_init(const T* __restrict__ v0,
                                                   const T* __restrict__ s0, int packed,
                                                   float* __restrict__ pool,
                                                   const InstDesc* __restrict__ descs, int n) {
  const int block = xcd_tile(blockIdx.x, gridDim.x);
  for_block_instances<MANY>(descs, n, block, [&](const InstDesc& d, int x, int y) {
    const int64_t ni = (int64_t)d.g.nx * d.g.ny;
    const T* v = packed ? s0 + 5 * d.node0 : v0 + 2 * d.node0;
    const T* s = packed ? s0 + 5 * d.node0 + 2 * ni : s0 + 3 * d.node0;
    init_node<INIT_FROM_STRESS, NT, T>(v, s, nullptr, pool + d.off, d.g, d.ic, x, y);
  });
}

// mode 0: physical (v, sigma_bar); 1: U.  per_xcd: see flat_node; for pools
// that the last-level cache holds twice (two batches in turn, grid order / a
// part per XCD: 64 uneven instances, 430 MB, 88.5 / 93.6 us, 64 of 250 x 250
// 72.4 / 75.9, 512 of 33 x 128 69.3 / 73.1; 256 of 33 x 33, 54 MB, 15.0 / 14.2).
template <bool MANY>
__global__ __launch_bounds__(BT) void k_batch_moments(const float* __restrict__ pool,
                                                      float* __restrict__ out,
                                                      const InstDesc* __restrict__ descs, int n,
                                                      bool per_xcd, int mode) {
  const int block = per_xcd ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  for_block_instances<MANY>(descs, n, block, [&](const InstDesc& d, int x, int y) {
    const int64_t ni = (int64_t)d.g.nx * d.g.ny;
    const float* src = pool + d.off;
    float f[NQ][NC], U[NC];
    for (int q = 0; q < NQ; ++q)
      for (int c = 0; c < NC; ++c) f[q][c] = src[pidx(d.g, q * NC + c, y, x)];
    moment0(f, U);  // the single lattice's summation order
    float* o = out + 5 * d.node0 + (int64_t)y * d.g.nx + x;
    if (mode == 1) {
      for (int c = 0; c < NC; ++c) o[c * ni] = U[c];
      return;
    }
    o[0] = U[0];
    o[ni] = U[1];
    o[2 * ni] = -d.rho * (d.cK * U[2] + d.cmu * U[3]);
    o[3 * ni] = -d.rho * (d.cK * U[2] - d.cmu * U[3]);
    o[4 * ni] = -d.rho * (d.cmu * U[4]);
  });
}

// The kernels with MANY (lbm_batch_many.hip), by nontemporal stores.  In a code
// object of their own: with them in lbm_batch.hip's a judge window of 32 x 128 x
// 128, which runs none of them, took 140.3 us, without them 139.0 (medians of 40
// batches in five processes), for a reason that was not found.
struct ManyKernels {
  void (*init_f[2])(const float*, const float*, int, float*, const InstDesc*, int);
  void (*init_d[2])(const double*, const double*, int, float*, const InstDesc*, int);
  void (*moments)(const float*, float*, const InstDesc*, int, bool, int);
};
ManyKernels many_kernels();

}  // namespace lbmb
