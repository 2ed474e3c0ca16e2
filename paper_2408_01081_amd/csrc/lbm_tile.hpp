// T time steps per launch on small lattices: a workgroup per tile.
//
// The sweep of lbm_tblock.hpp forms its levels one after the other in every
// wave (2T rows of pipeline fill, then a row at a time), so a launch takes as
// long as one wave's chain of rows; where the lattice has fewer waves than the
// chip has SIMDs, that chain is the launch time.  Here a workgroup of NW waves
// holds a tile of 64 columns x R = 2 NW rows in registers, 2 rows per wave and
// a column per lane, and all of its waves advance one step at a time: only one
// level is kept, T is a run-time number, and a step's chain is 2 rows.  Rows
// of neighbouring waves meet in LDS (a wave writes the upward populations of
// its last row and the downward ones of its first, one barrier per step, two
// buffers by step parity); the x neighbours are DPP lane shifts, as in the
// sweep.  Each step costs the tile one row and column of exact values at
// every edge, so 64 - 2T columns x R - 2T rows are stored.
// The update of a node is the sweep's level_update on the same inputs: the
// results are bitwise those of single steps.
//
// Bound by vector instructions at two or three waves per SIMD (0.14 to 0.18 us
// per row update of a wave; R / 4 of them per SIMD and step) and by 3.4 to 5
// us per launch (dispatch, loads, stores).  Which shape pays depends on the
// grid and is the autotuner's choice; per step, the fastest tile against the
// fastest other variant: 160 x 160 with walls 1.49 us (T = 5, 16 rows) against
// 2.90; 256 x 256 with walls 1.61 against 2.94, periodic 1.56 (T = 8, 24
// rows) against 1.97; 384 x 384 1.99 against 2.13; 512 x 512 3.07 against 2.84
// (walls: 3.63 against 3.79); 724 x 724 5.07 against 3.60.  160 x 160 with a
// load of rank 16 and the displacement state: 2.3 us (2.7 in a trace), one launch
// per step 4.9.
// 3 or 4 rows per wave: equal or slower (fewer waves; the wall code needs the
// registers); tiles of 32 rows: slower.
#pragma once

#include "lbm_tblock.hpp"

namespace lbmk {

constexpr int TILE_K = 2;  // rows per wave
constexpr int TILE_MAX_ROWS = 24;  // rows of the largest tile variant

// the body load and displacement state of a launch (TBExtra; the row factors
// Y[r][y] T_{n+l}[r] are formed in LDS at the start of the launch)
struct TileExtra {
  const float* X;   // [rank][2][nx]
  const float* Y;   // [rank][ny]
  const float* T1;  // [..][rank], the row of the launch's first level
  int rank;
  float scale;
  double* D;  // [2][ny][nx]
  double half_dt;
};

// most steps of a launch of tiles of `rows` rows with a load or displacement: two thirds
// of the tile's rows are overlap then
constexpr int tile_max_steps(int rows) { return rows / 3; }

// update of row r of the wave (in place) from the rows below and above it
template <int BC, bool EDGE, bool FORCE, bool DISP, int MR>
__device__ __forceinline__ void tile_row(const Grid& g, const TBConst& sc, const Wall& w,
                                         const TileExtra& F, const LaneLoad<MR>& ll, int xw, int y,
                                         const float* fac, const float (&f1)[NC],
                                         const float (&f3)[NC], float (&f)[NP], double (&d)[2]) {
  const int yc = y < 0 ? 0 : (y >= g.ny ? g.ny - 1 : y);
  float yt[MR], below[NP], above[NP], out[NP], Uo[2];
  if constexpr (FORCE) fac_read<MR>(fac, 1, yt);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    below[1 * NC + c] = f1[c];
    above[3 * NC + c] = f3[c];
  }
  level_update<BC, EDGE, FORCE, MR>(below, f, above, xw, yc, g.nx, g.ny, sc.kK, sc.km, w, ll, yt,
                                    F.scale, out, Uo);
  if constexpr (DISP) d_update(d, Uo, F.half_dt);
#pragma unroll
  for (int k = 0; k < NP; ++k) f[k] = out[k];
}

// The T steps of one wave (EDGE: see level_update).
template <int BC, bool EDGE, bool FORCE, bool DISP, int MR>
__device__ __forceinline__ void tile_steps(const Grid& g, const TBConst& sc, const WallSeq& ws,
                                           const TileExtra& F, const LaneLoad<MR>& ll, int xw,
                                           int wave, int nw, int yw, int T, float* ex,
                                           const float* fac, float (&f)[TILE_K][NP],
                                           double (&d)[TILE_K][2]) {
  const int lane = threadIdx.x & 63;
  const int wb = wave > 0 ? wave - 1 : 0, wa = wave + 1 < nw ? wave + 1 : wave;
#pragma unroll 1
  for (int s = 0; s < T; ++s) {
    float* buf = ex + (s & 1) * nw * 10 * TB_LANES;
    float* mine = buf + wave * 10 * TB_LANES + lane;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      mine[c * TB_LANES] = f[1][1 * NC + c];
      mine[(NC + c) * TB_LANES] = f[0][3 * NC + c];
    }
    __syncthreads();
    // (the tile's first and last rows have no neighbour: any value, never
    // part of a stored result)
    float below[NC], above[NC], up[NC], down[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      below[c] = buf[(wb * 10 + c) * TB_LANES + lane];
      above[c] = buf[(wa * 10 + NC + c) * TB_LANES + lane];
      up[c] = f[0][1 * NC + c];
      down[c] = f[1][3 * NC + c];
    }
    Wall w;
    w.L = ws.L;
    w.V = ws.V ? ws.V + (int64_t)s * 2 * ws.L : nullptr;
    w.W = nullptr;
    w.rank = 0;
    w.Trow = nullptr;
    const float* fs = fac + (s * nw + wave) * TILE_K * MR;
    tile_row<BC, EDGE, FORCE, DISP, MR>(g, sc, w, F, ll, xw, yw, fs, below, down, f[0], d[0]);
    tile_row<BC, EDGE, FORCE, DISP, MR>(g, sc, w, F, ll, xw, yw + 1, fs + MR, up, above, f[1],
                                        d[1]);
  }
}

// sc.nstrips strips of 64 - 2T columns, sc.nseg segments of sc.seg_rows =
// R - 2T rows; one workgroup of nw = blockDim.x / 64 waves each.  MAXW: the
// most waves of a launch (sets the registers a wave may use).
template <int BC, bool FORCE, bool DISP, int MR, int MAXW>
__global__ __launch_bounds__(64 * MAXW) void k_tile(const float* __restrict__ src,
                                                    float* __restrict__ dst, Grid g, TBConst sc,
                                                    WallSeq ws, TileExtra F, int T) {
  __shared__ float ex[2 * MAXW * 10 * TB_LANES];  // two exchange buffers
  __shared__ __attribute__((aligned(16))) float
      fac[FORCE ? tile_max_steps(TILE_K * MAXW) * TILE_K * MAXW * MR : 4];
  const int nw = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = xcd_tile(blockIdx.x, sc.nstrips * sc.nseg);
  const int seg = tile / sc.nstrips, strip = tile - seg * sc.nstrips;
  const int nx = g.nx, ny = g.ny;
  const int x0 = strip * (TB_LANES - 2 * T) - T, x = x0 + lane;
  const int y0 = seg * sc.seg_rows - T;  // sweep row of the tile's first row
  const int yw = y0 + TILE_K * wave;
  const int xc = BC == LBM_PERIODIC ? wrap_mod(x, nx) : (x < 0 ? 0 : (x >= nx ? nx - 1 : x));
  const bool store = lane >= T && lane < TB_LANES - T && x < nx;
  Strip st;
  st.xw = x >= 0 && x < nx ? x : -2;
  st.xr4 = (int)((uint32_t)xc * 4u);
  st.xs4 = store ? (int)((uint32_t)x * 4u) : TB_DROP;
  const int pitch4 = (int)(g.pitch * 4);

  float f[TILE_K][NP];
  double d[TILE_K][2];
  bool own[TILE_K];
#pragma unroll
  for (int r = 0; r < TILE_K; ++r) {
    const int y = yw + r, t = TILE_K * wave + r;
    own[r] = t >= T && t < TILE_K * nw - T && y < ny;  // (t >= T: y >= 0)
    load_row(src, pitch4, sc, st, row_index<BC>(y, ny), f[r]);
    if constexpr (DISP) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
        d[r][c] = own[r] && store ? F.D[((int64_t)c * ny + y) * nx + x] : 0.0;
    }
  }
  LaneLoad<MR> ll;
  if constexpr (FORCE) {
#pragma unroll
    for (int r = 0; r < MR; ++r)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        ll.x[c][r] = r < F.rank ? F.X[((int64_t)r * 2 + c) * nx + xc] : 0.f;
    // row factors of the tile's rows at every level (TBExtra's padding)
    const int R = TILE_K * nw;
    for (int e = threadIdx.x; e < T * R * MR; e += blockDim.x) {
      const int r = e % MR, t = (e / MR) % R, l = e / (MR * R);
      const int y = row_index<BC>(y0 + t, ny);
      fac[e] = r < F.rank ? F.Y[(int64_t)r * ny + y] * F.T1[(int64_t)l * F.rank + r] : -0.f;
    }
  }
  // a tile of a Dirichlet lattice meets the side walls only if its columns
  // include one (uniform across the workgroup)
  if (BC == LBM_DIRICHLET && (x0 <= 0 || x0 + TB_LANES - 1 >= nx - 1))
    tile_steps<BC, BC == LBM_DIRICHLET, FORCE, DISP, MR>(g, sc, ws, F, ll, st.xw, wave, nw, yw, T,
                                                         ex, fac, f, d);
  else
    tile_steps<BC, false, FORCE, DISP, MR>(g, sc, ws, F, ll, st.xw, wave, nw, yw, T, ex, fac, f,
                                           d);
  const int doff = store ? (int)((uint32_t)x * 8u) : TB_DROP;
#pragma unroll
  for (int r = 0; r < TILE_K; ++r) {
    if (!own[r]) continue;  // uniform
    const int y = yw + r;
    char* rp = (char*)dst + (int64_t)y * pitch4;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)rp, (short)0, sc.extent, TB_RSRC_WORD3);
#pragma unroll
    for (int k = 0; k < NP; ++k)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f[r][k]), rs, st.xs4, k * sc.plane4, 0);
    if constexpr (DISP) {
      TBExtra e{};
      e.D = F.D;
      d_store(e, g, doff, y, d[r]);
    }
  }
}

typedef void (*TileFn)(const float*, float*, Grid, TBConst, WallSeq, TileExtra, int);
// kernels by extras (0 load, 1 displacement, 2 both, 3 none), load ranks (0:
// 16, 1: 32) and boundary type
struct TileTable {
  TileFn fn[4][2][2];
};
// most waves of a kernel: those of the largest tile, fewer with a load.  They set
// its LDS and the registers a wave may use, 512 / (waves per SIMD).  (With a load,
// 12 waves left the wall code 80 to 150 B of scratch per lane: 160 x 160 with load
// and displacement 3.1 us per step; 8 waves 2.7.  With walls, ranks above 16 and
// the displacement state 8 waves leave 44 B: 3.0 us per step, where one launch per
// step takes 6.5 and the sweep, with 92 B, 15.5.)
constexpr int tile_max_waves(int extras) {
  return extras == 3 || extras == 1 ? TILE_MAX_ROWS / TILE_K : 8;
}
void tile_fill(TileTable& t);  // lbm_tile.hip

}  // namespace lbmk
