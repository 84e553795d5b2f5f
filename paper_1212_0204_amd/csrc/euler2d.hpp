// Euler sub-steps on 2D grids (wavefront strips, or LDS tiles on narrow grids)
// and 3D grids (LDS tiles).
#pragma once
#include "dpp.hpp"
#include "kernels.hpp"
#include "rules.hpp"
#include "slope.hpp"

namespace hofks {

// Euler sub-step on a 2D grid by wavefront strips (section 4.3.2, eq.
// (discmom) with the limited slopes of the MUSCL flux).  A wavefront holds a
// strip of 64 consecutive x cells, of which it advances the inner 60 on H
// rows (y0 .. y0 + H - 1); lane l is cell X0 - 2 + l.
//
// A limited slope is formed once, by its own cell, so a cell needs two per
// axis and moment; twice the face flux is (W+_j + W-_{j+1}) + (s+_j - s-_{j+1})/2,
// rounded as the per-cell form `euler_cell` rounds it.  Along
// x the neighbours' values come by one-lane shifts of the ALU; along y the
// wavefront marches over the rows y0 - 2 .. y0 + H + 1 and keeps the last
// fluxes and half states in registers.  No LDS and no barrier except the
// reduction of the speeds, so the blocks find room beside the kinetic
// blocks.
//
// Bound by latency on small grids (launch, loads, the chain of a strip) and
// by the FP64 issue rate from about 512^2 cells.  Measured per sub-step
// against 16 x 16 LDS tiles (four slopes per face pair, four block barriers),
// which narrow grids keep: alone 9.2 -> 5.4 us on 70 x 37 cells, 8.8 -> 6.4 on
// 256^2, 25.8 -> 12.3 on 512^2.
// The flux divergence of the H inner rows of a strip: row(q, U) gives the
// moments of strip row q (0 .. H + 3, the lane's cell) and done(k, div) takes
// twice the divergence (times dx) of inner row k as soon as it is complete.
template <int H, bool UNL, typename Row, typename Done>
__device__ __forceinline__ void strip_div(const double* alpha, Row&& row, Done&& done) {
  constexpr int NM = 4;
  // of the last rows; wsum: W+ + W- across the face before row q - 1
  double Wpp[NM] = {}, dP[NM] = {}, Wmp[NM] = {}, dM[NM] = {}, hpp[NM] = {}, wsum[NM] = {}, Fp[NM] = {};
  double div[H][NM];
#pragma unroll
  for (int q = 0; q < H + 4; ++q) {
    double U[NM], Wp[NM], Wm[NM];
    row(q, U);
    const double ir = rcp_nr(U[0]);
    if (q >= 2 && q < H + 2) {  // x faces of the row
      split_flux2(U, ir, 0, alpha[0], Wp, Wm);
#pragma unroll
      for (int r = 0; r < NM; ++r) {
        const double wn = lane_next(Wm[r]);
        const double dp = lane_next(Wp[r]) - Wp[r], dm = wn - Wm[r];
        const double hp = half_slope<UNL>(lane_prev(dp), dp);
        const double hm = half_slope<UNL>(lane_prev(dm), dm);
        const double f = (Wp[r] + wn) + (hp - lane_next(hm));
        div[q - 2][r] = f - lane_prev(f);
      }
    }
    split_flux2(U, ir, 1, alpha[1], Wp, Wm);
#pragma unroll
    for (int r = 0; r < NM; ++r) {
      const double dp = Wp[r] - Wpp[r], dm = Wm[r] - Wmp[r];
      double f = 0.0, hp = 0.0;
      if (q >= 3) {  // face between rows q - 2 and q - 1
        f = wsum[r] + (hpp[r] - half_slope<UNL>(dM[r], dm));
        if (q >= 4) div[q - 4][r] += f - Fp[r];
      }
      if (q >= 2 && q < H + 3) hp = half_slope<UNL>(dP[r], dp);  // of row q - 1
      wsum[r] = Wpp[r] + Wm[r];
      Wpp[r] = Wp[r];
      Wmp[r] = Wm[r];
      dP[r] = dp;
      dM[r] = dm;
      hpp[r] = hp;
      Fp[r] = f;
    }
    if (q >= 4) done(q - 4, div[q - 4]);
  }
}

// map_axis for a strip's cells and rows, i >= -HALO: those past N + HALO - 1
// are never used and taken as that, and an axis of HALO cells or more needs no
// division
template <int HALO>
__device__ __forceinline__ int map_near(int i, int N, int bc) {
  i = min(i, N + HALO - 1);
  if (bc == 0 && N >= HALO) return i < 0 ? i + N : (i >= N ? i - N : i);
  return map_axis(i, N, bc);
}

// speeds of row i of a 2D set: lane 4 q + d reads axis d of slot q (row 0 has
// one slot); every lane of the wavefront takes part
__device__ __forceinline__ void strip_speeds(const double* S, int i, int lane, double* alpha) {
  if (i == 0) {
    const double al = S[lane & 1];
    alpha[0] = lane_value(al, 0);
    alpha[1] = lane_value(al, 1);
    return;
  }
  double al = S[ASTR + (size_t)(i - 1) * NSLOT * ASTR + (lane & 31)];
  al = dpp_max<0x114, 0xF>(al);  // lanes 4..: max with lane - 4
  al = dpp_max<0x118, 0xF>(al);  // lanes 12..15: the row's four slots
  alpha[0] = fmax(lane_value(al, 12), lane_value(al, 28));
  alpha[1] = fmax(lane_value(al, 13), lane_value(al, 29));
}

// the largest speeds of a block of four strips into row i of the set
__device__ __forceinline__ void fold_speeds(double* S, int i, int lane, int wv, const double* mx) {
  __shared__ double wm4[2][4];
#pragma unroll
  for (int d2 = 0; d2 < 2; ++d2) {
    const double m = wave_max_dpp(mx[d2]);
    if (lane == 0) wm4[d2][wv] = m;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    const double* m = wm4[threadIdx.x];
    atomic_max_pos(speed_row(S, i, blockIdx.x % NSLOT) + threadIdx.x,
                   fmax(fmax(m[0], m[1]), fmax(m[2], m[3])));
  }
}

// One-row strips beside FP32 pieces hold 96 registers (106 and no spill
// otherwise): three wavefronts of the four-wavefront kinetic blocks on a SIMD
// leave 104, and a strip that does not fit them takes a kinetic block's place.
// FP32 256^2 x 32^2 at lambda = 0.46 0.232 -> 0.211 ms per step, 320 x 300 x 32^2
// 0.300 -> 0.271.
template <typename T, int H, bool UNL>
__global__ __launch_bounds__(256, H == 1 && sizeof(T) == 4 ? 5 : 1) void k_euler_strip(StepArgs<T> a, Geom G, int i, int nsx) {
  constexpr int NM = 4, W = STRIP_W;
  double* S = a.set_r;
  const int Nx = G.n[0], Ny = G.n[1];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // contiguous ranges of blocks per die (blocks reach the dies round-robin)
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int X0 = (tile % nsx) * W, y0 = ((tile / nsx) * 4 + wv) * H;
  const double* in = (i == 0) ? a.U_in : ((i & 1) ? a.UE1 : a.UE0);
  double* out = ((i + 1) & 1) ? a.UE1 : a.UE0;

  // every row of the strip, loaded before the speeds of the sub-step are
  // read so that the memory round trips overlap
  const int gx = map_near<2>(X0 - 2 + lane, Nx, G.bc[0]);
  double Ur[H + 4][NM];
#pragma unroll
  for (int q = 0; q < H + 4; ++q) {
    const size_t j = (size_t)map_near<2>(y0 - 2 + q, Ny, G.bc[1]) * Nx + gx;
#pragma unroll
    for (int r = 0; r < NM; ++r) Ur[q][r] = in[(size_t)r * G.nc + j];
  }
  double alpha[2];
  strip_speeds(S, i, lane, alpha);
  // the count: formed by sub-step 0, which records it for the later launches
  const int s = i == 0 ? open_substeps<2>(a, G) : a.flag[1];
  if (i >= s) return;
  const double hdts_dx = 0.5 * ((G.dt / s) / G.dx);

  bool phys = true;
  double mx[2] = {0.0, 0.0};
  const bool ownx = lane >= 2 && lane < 2 + W && X0 + lane - 2 < Nx;
  strip_div<H, UNL>(
      alpha,
      [&](int q, double* U) {
#pragma unroll
        for (int r = 0; r < NM; ++r) U[r] = Ur[q][r];
      },
      [&](int k, const double* div) {
        const int y = y0 + k;
        const double* Uc = Ur[k + 2];
        double Un[NM], sp[2];
#pragma unroll
        for (int r = 0; r < NM; ++r) Un[r] = fma(-hdts_dx, div[r], Uc[r]);
        if (!ownx || y >= Ny) return;
        phys &= i > 0 || speeds2(Uc, rcp_nr(Uc[0]), G.gam, sp);  // U^n; later inputs were checked as results
        const size_t j = (size_t)y * Nx + X0 + lane - 2;
#pragma unroll
        for (int r = 0; r < NM; ++r) out[(size_t)r * G.nc + j] = Un[r];
        if (i + 1 < s) {
          phys &= speeds2(Un, rcp_nr(Un[0]), G.gam, sp);
          mx[0] = fmax(mx[0], sp[0]);
          mx[1] = fmax(mx[1], sp[1]);
        }
      });
  if (!phys) atomicOr(a.flag, FLAG_NONPHYS);
  if (i + 1 < s) fold_speeds(S, i + 1, lane, wv, mx);
}

// The same sub-step with LDS tiles, for grids whose rows leave most lanes of
// the strips idle (see `euler_tiles`): a block loads a 16 x 16 tile of cells
// with two halo cells on every side, then for each axis in turn evaluates the
// split fluxes of the cells the faces along that axis need (x: 20 x 16, y:
// 16 x 20) into one buffer, every thread adding the difference of its cell's
// two faces along that axis; then the new value.  The same bits as the strips.
//
// Bound by its block barriers and LDS round trips on such grids (25.8 us per
// sub-step on 512^2, 8.8 on 256^2, against the strips' 12.3 and 6.4).
constexpr int EH = ET + 4;  // tile edge with two halo cells on each side

template <typename T>
__global__ __launch_bounds__(256) void k_euler_sub_tile(StepArgs<T> a, Geom G, int i, int ntx) {
  constexpr int NM = 4;
  double* S = a.set_r;
  const int Nx = G.n[0], Ny = G.n[1];
  // contiguous ranges of tiles per die (blocks reach the dies round-robin),
  // so that the halo of most tiles was written on the same die
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int X0 = (tile % ntx) * ET, Y0 = (tile / ntx) * ET;
  const int t = threadIdx.x;
  const double* in = (i == 0) ? a.U_in : ((i & 1) ? a.UE1 : a.UE0);
  double* out = ((i + 1) & 1) ? a.UE1 : a.UE0;

  __shared__ double Ut[NM][EH][EH];
  // split fluxes along one axis at a time (x, then y) in one buffer:
  // x: [+/-][r][y][x + 2] over 16 x 20 cells; y: [+/-][r][y + 2][x] over 20 x 16
  __shared__ double Wb[2][NM][ET * EH];

  // tile + halo (periodic wrap or outflow clamp, as the per-cell form),
  // loaded before the speeds of the sub-step are read so that the two
  // memory round trips overlap (both buffers exist whatever s is)
  constexpr int NQ = (EH * EH + 255) / 256;
  double Uload[NQ][NM];
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int q = t + k * 256;
    if (q < EH * EH) {
      const int hx = q % EH, hy = q / EH;
      const int gx = map_axis(X0 + hx - 2, Nx, G.bc[0]);
      const int gy = map_axis(Y0 + hy - 2, Ny, G.bc[1]);
      const size_t j = (size_t)gy * Nx + gx;
#pragma unroll
      for (int r = 0; r < NM; ++r) Uload[k][r] = in[(size_t)r * G.nc + j];
    }
  }
  double alpha[2];
  strip_speeds(S, i, t & 63, alpha);
  // the count: formed by sub-step 0, which records it for the later launches
  const int s = i == 0 ? open_substeps<2>(a, G) : a.flag[1];
  if (i >= s) return;
  const double dts_dx = (G.dt / s) / G.dx;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int q = t + k * 256;
    if (q < EH * EH) {
#pragma unroll
      for (int r = 0; r < NM; ++r) Ut[r][q / EH][q % EH] = Uload[k][r];
    }
  }
  __syncthreads();
  bool phys = true;
  const int lx = t % ET, ly = t / ET;
  const int gx = X0 + lx, gy = Y0 + ly;
  const bool own = gx < Nx && gy < Ny;
  double div[NM] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ax = 0; ax < 2; ++ax) {
    if (ax == 1) __syncthreads();  // the x faces have been read
    // fluxes along ax: x for cells (x = -2..17, y = 0..15), y for (x = 0..15, y = -2..17)
    for (int q = t; q < ET * EH; q += blockDim.x) {
      const int hx = ax == 0 ? q % EH : q % ET + 2;
      const int hy = ax == 0 ? q / EH + 2 : q / ET;
      double Uq[NM];
#pragma unroll
      for (int r = 0; r < NM; ++r) Uq[r] = Ut[r][hy][hx];
      double Wp[NM], Wm[NM];
      phys &= split_flux<2>(Uq, ax, alpha[ax], G.gam, Wp, Wm);
#pragma unroll
      for (int r = 0; r < NM; ++r) {
        Wb[0][r][q] = Wp[r];
        Wb[1][r][q] = Wm[r];
      }
    }
    __syncthreads();
    if (own) {
#pragma unroll
      for (int r = 0; r < NM; ++r) {
        // cells l-2 .. l+2 along ax: x -> entries ly*EH + lx + k, y -> (ly + k)*ET + lx
        double wp[5], wm[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          const int e = ax == 0 ? ly * EH + lx + k : (ly + k) * ET + lx;
          wp[k] = Wb[0][r][e];
          wm[k] = Wb[1][r][e];
        }
        const double spl = vl_slope(wp[1] - wp[0], wp[2] - wp[1], a.unlimited);
        const double sml = vl_slope(wm[2] - wm[1], wm[3] - wm[2], a.unlimited);
        const double spr = vl_slope(wp[2] - wp[1], wp[3] - wp[2], a.unlimited);
        const double smr = vl_slope(wm[3] - wm[2], wm[4] - wm[3], a.unlimited);
        const double psil = 0.5 * (wp[1] + wm[2]) + 0.25 * (spl - sml);
        const double psir = 0.5 * (wp[2] + wm[3]) + 0.25 * (spr - smr);
        div[r] += psir - psil;
      }
    }
  }
  double mx[2] = {0.0, 0.0};
  if (own) {
    double Un[NM];
#pragma unroll
    for (int r = 0; r < NM; ++r) Un[r] = Ut[r][ly + 2][lx + 2] - dts_dx * div[r];
    const size_t j = (size_t)gy * Nx + gx;
#pragma unroll
    for (int r = 0; r < NM; ++r) out[(size_t)r * G.nc + j] = Un[r];
    if (i + 1 < s) {
      double sp[3];
      phys &= lf_speeds<2>(Un, G.gam, sp);
      mx[0] = sp[0];
      mx[1] = sp[1];
    }
  }
  if (!phys) atomicOr(a.flag, FLAG_NONPHYS);
  if (i + 1 < s) fold_speeds(S, i + 1, t & 63, t >> 6, mx);
}

// Euler sub-step on a 3D grid with LDS tiles: one block of 256 threads
// advances an 8 x 4 x 4 tile, loaded with two halo cells on every side
// (an 12 x 8 x 8 box) into LDS; for each axis in turn the split fluxes of
// the cells the faces along that axis need are evaluated once, one per
// thread, then every cell thread forms its two faces and adds their
// difference.  Same arithmetic per face as `euler_cell`; few registers
// (at most 64), so that the sub-step blocks find room beside the blocks of
// the kinetic kernel running at the same time.
constexpr int E3X = 8, E3Y = 4, E3Z = 4;  // tile (cells)
constexpr int E3C = E3X * E3Y * E3Z;      // 128 cells
constexpr int B3X = E3X + 4, B3Y = E3Y + 4, B3Z = E3Z + 4;  // box with halo

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(64))) void k_euler_sub_tile3(StepArgs<T> a, Geom G, int i, int ntx,
                                                           int nty) {
  constexpr int NM = 5;
  double* S = a.set_r;
  const int Nx = G.n[0], Ny = G.n[1], Nz = G.n[2];
  const int tb = xcd_tile(blockIdx.x, gridDim.x);  // contiguous ranges of tiles per die
  const int X0 = (tb % ntx) * E3X, Y0 = ((tb / ntx) % nty) * E3Y, Z0 = (tb / ntx / nty) * E3Z;
  const int t = threadIdx.x;
  const double* in = (i == 0) ? a.U_in : ((i & 1) ? a.UE1 : a.UE0);
  double* out = ((i + 1) & 1) ? a.UE1 : a.UE0;

  __shared__ double Ub[NM][B3Z * B3Y * B3X];  // box: [z][y][x]
  __shared__ double Wb[2][NM][256];          // split fluxes along one axis

  // the count: formed by sub-step 0, which records it for the later launches
  const int s = i == 0 ? open_substeps<3>(a, G) : a.flag[1];
  if (i >= s) return;
  double alpha[3];
  row_speeds<3>(S, i, alpha);
  const double dts_dx = (G.dt / s) / G.dx;
  // box (periodic wrap or outflow clamp, as the per-cell form)
  for (int q = t; q < B3Z * B3Y * B3X; q += 256) {
    const int hx = q % B3X, hy = (q / B3X) % B3Y, hz = q / (B3X * B3Y);
    const int gx = map_axis(X0 + hx - 2, Nx, G.bc[0]);
    const int gy = map_axis(Y0 + hy - 2, Ny, G.bc[1]);
    const int gz = map_axis(Z0 + hz - 2, Nz, G.bc[2]);
    const size_t j = ((size_t)gz * Ny + gy) * Nx + gx;
#pragma unroll
    for (int r = 0; r < NM; ++r) Ub[r][q] = in[(size_t)r * G.nc + j];
  }
  __syncthreads();
  bool phys = true;
  const int lx = t % E3X, ly = (t / E3X) % E3Y, lz = t / (E3X * E3Y);  // cell of t < 128
  const int gx = X0 + lx, gy = Y0 + ly, gz = Z0 + lz;
  const bool own = t < E3C && gx < Nx && gy < Ny && gz < Nz;
  double div[NM] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int ax = 0; ax < 3; ++ax) {
    if (ax > 0) __syncthreads();  // the fluxes of the previous axis have been read
    // entries: the tile extended by two cells on each side along ax
    const int ex = ax == 0 ? B3X : E3X, ey = ax == 1 ? B3Y : E3Y;
    const int ne = ex * ey * (ax == 2 ? B3Z : E3Z);
    if (t < ne) {
      const int qx = t % ex, qy = (t / ex) % ey, qz = t / (ex * ey);
      const int hx = ax == 0 ? qx : qx + 2, hy = ax == 1 ? qy : qy + 2, hz = ax == 2 ? qz : qz + 2;
      const int b = (hz * B3Y + hy) * B3X + hx;
      double Uq[NM];
#pragma unroll
      for (int r = 0; r < NM; ++r) Uq[r] = Ub[r][b];
      double Wp[NM], Wm[NM];
      phys &= split_flux<3>(Uq, ax, alpha[ax], G.gam, Wp, Wm);
#pragma unroll
      for (int r = 0; r < NM; ++r) {
        Wb[0][r][t] = Wp[r];
        Wb[1][r][t] = Wm[r];
      }
    }
    __syncthreads();
    if (own) {
      // entries of the cells l-2 .. l+2 along ax
      const int e0 = ax == 0 ? (lz * E3Y + ly) * B3X + lx
                   : ax == 1 ? (lz * B3Y + ly) * E3X + lx : (lz * E3Y + ly) * E3X + lx;
      const int es = ax == 0 ? 1 : ax == 1 ? E3X : E3X * E3Y;
      // one moment at a time (few live registers)
#pragma unroll 1
      for (int r = 0; r < NM; ++r) {
        double wp[5], wm[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
          wp[k] = Wb[0][r][e0 + k * es];
          wm[k] = Wb[1][r][e0 + k * es];
        }
        const double spl = vl_slope(wp[1] - wp[0], wp[2] - wp[1], a.unlimited);
        const double sml = vl_slope(wm[2] - wm[1], wm[3] - wm[2], a.unlimited);
        const double spr = vl_slope(wp[2] - wp[1], wp[3] - wp[2], a.unlimited);
        const double smr = vl_slope(wm[3] - wm[2], wm[4] - wm[3], a.unlimited);
        const double psil = 0.5 * (wp[1] + wm[2]) + 0.25 * (spl - sml);
        const double psir = 0.5 * (wp[2] + wm[3]) + 0.25 * (spr - smr);
        div[r] += psir - psil;
      }
    }
  }
  double mx[3] = {0.0, 0.0, 0.0};
  if (own) {
    const int b = ((lz + 2) * B3Y + ly + 2) * B3X + lx + 2;
    double Un[NM];
#pragma unroll
    for (int r = 0; r < NM; ++r) Un[r] = Ub[r][b] - dts_dx * div[r];
    const size_t j = ((size_t)gz * Ny + gy) * Nx + gx;
#pragma unroll
    for (int r = 0; r < NM; ++r) out[(size_t)r * G.nc + j] = Un[r];
    if (i + 1 < s) phys &= lf_speeds<3>(Un, G.gam, mx);
  }
  if (!phys) atomicOr(a.flag, FLAG_NONPHYS);
  if (i + 1 < s) {
    __shared__ double wm4[4][ASTR];
#pragma unroll
    for (int d2 = 0; d2 < 3; ++d2) {
      const double m = wave_max(mx[d2]);
      if ((t & 63) == 0) wm4[t >> 6][d2] = m;
    }
    __syncthreads();
    if (t < 3) {
      double m = wm4[0][t];
      for (int w = 1; w < 4; ++w) m = fmax(m, wm4[w][t]);
      atomic_max_pos(speed_row(S, i + 1, blockIdx.x % NSLOT) + t, m);
    }
  }
}

}  // namespace hofks
