// euler1d.hpp -- the whole Euler solve of a 1D row of cells in one group of
// wavefronts of one block, every cell's moments in registers (section 4.3.2,
// eq. (discmom) with the limited slopes of the MUSCL flux).  Used for single
// 1D grids (`k_euler_line`) and for the tubes of a batch.
#pragma once
#include "dpp.hpp"
#include "kernels.hpp"
#include "slope.hpp"

namespace hofks {

// Flux F(U) of one 1D cell from U and 1/rho, with the expressions of
// split_flux (W+- = F +- alpha U); false if the state is not physical
__device__ __forceinline__ bool flux1(const double* U, double irho, double* F) {
  const double rho = U[0];
  const double u = U[1] * irho;
  const double usq = u * u;
  const double p = fma(-rho, usq, 2.0 * U[2]);
  F[0] = U[1];
  F[1] = fma(U[1], u, p);
  F[2] = (U[2] + p) * u;
  return (rho > 0.0) && (p > 0.0) && isfinite(rho) && isfinite(p) && isfinite(usq);
}

// Lax-Friedrichs speed |u| + sqrt(gam p / rho) of one 1D cell (p = rho
// theta) from U and 1/rho; 0 and false if the state is not physical
__device__ __forceinline__ bool speed1(const double* U, double irho, double gam, double* sp) {
  const double rho = U[0];
  const double u = U[1] * irho;
  const double usq = u * u;
  const double p = fma(-rho, usq, 2.0 * U[2]);
  const bool ok = (rho > 0.0) && (p > 0.0) && isfinite(rho) && isfinite(p) && isfinite(usq);
  *sp = ok ? fabs(u) + sqrt(gam * p * irho) : 0.0;
  return ok;
}

// W+ (w[0..2]) and W- (w[3..5]) of one cell
__device__ __forceinline__ void wsplit(const double* U, const double* F, double alpha, double* w) {
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    w[r] = fma(alpha, U[r], F[r]);
    w[3 + r] = fma(-alpha, U[r], F[r]);
  }
}

// Twice a face flux from W+ and half its slope of the left cell and W- and
// half its slope of the right cell
__device__ __forceinline__ double face2(double wp, double hp, double wm, double hm) {
  return (wp + wm) + (hp - hm);
}

// A wavefront of the group holds 64 CPT consecutive cells, CPT per lane, of
// which the first and last two are copies of its neighbours' cells, so it
// advances line_own(CPT) = 64 CPT - 4 cells.  A sub-step needs two limited slopes
// per cell and moment; the values of the neighbouring lanes (W of one cell on
// each side, a half state and a face flux) come by one-lane shifts of the ALU.
// Then every wavefront leaves its edge cells, the row's end cells and its
// largest speed in LDS (two sets, by sub-step parity), one block barrier
// follows, and the copies and alpha are read back.
//
// The form is bound by the latency of this chain while a SIMD holds one
// wavefront and by the FP64 issue rate beyond.
constexpr int LINE_SLOT = 4;  // doubles per exchanged cell: U, 1/rho
constexpr int LINE_SETS = 16 * 4 * LINE_SLOT + 4 * LINE_SLOT + 16;  // edges, row ends, speeds
constexpr int LINE_LDS = 2 * LINE_SETS;  // doubles per group
__host__ __device__ constexpr int line_own(int cpt) { return 64 * cpt - 4; }

// wv: wavefront of the group (of nwv <= 16); s sub-steps are run, and smax
// block barriers met (another group of the block may run more); U0 and out
// are 3 x Nx.  Every thread of the block calls this with the same smax > 0.
template <int CPT, bool UNL>
__device__ __forceinline__ bool euler_line(const double* __restrict__ U0, double* __restrict__ out,
                                           int Nx, int bc, int wv, int nwv, double alpha, int s,
                                           int smax, double hdts, double gam, double* L) {
  constexpr int NP = 64 * CPT;  // cells a wavefront holds
  const int lane = threadIdx.x & 63;
  const int w0 = wv * line_own(CPT) - 2;  // first cell of the wavefront
  const int c0 = w0 + lane * CPT;
  // wavefronts that hold one of the row's end cells or a copy of one
  const bool ends = w0 <= 1 || (w0 + NP > Nx - 2 && w0 < Nx + 2);
  // edge slots a lane of one or two cells writes and reads (-1: none)
  int wslot = -1, rslot = -1;
  if (CPT <= 2) {
    const int pos = lane * CPT;
    if (pos == 2 || pos == 3) wslot = wv * 4 + pos - 2;
    if (pos == NP - 4 || pos == NP - 3) wslot = wv * 4 + pos - (NP - 6);
    if (pos < 2) rslot = max(wv - 1, 0) * 4 + 2 + pos;
    if (pos >= NP - 2) rslot = min(wv + 1, nwv - 1) * 4 + pos - (NP - 2);
  }
  double U[CPT][3], ir[CPT];
  bool phys = true;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int c = map_axis(min(c0 + j, Nx + 1), Nx, bc);
#pragma unroll
    for (int r = 0; r < 3; ++r) U[j][r] = U0[(size_t)r * Nx + c];
    ir[j] = rcp_nr(U[j][0]);
  }
  auto own = [&](int j) {
    const int pos = lane * CPT + j;
    return pos >= 2 && pos < NP - 2 && c0 + j < Nx;
  };
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    double F[3];
    phys &= flux1(U[j], ir[j], F) || s == 0 || !own(j);
  }
  if (threadIdx.x % 64 < 16 && wv == 0) {  // speeds of absent wavefronts
    L[LINE_SETS - 16 + lane] = 0.0;
    L[2 * LINE_SETS - 16 + lane] = 0.0;
  }
  __syncthreads();
  for (int i = 0; i < smax; ++i) {
    if (i < s) {
      double W[CPT][6];
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        double F[3];
        (void)flux1(U[j], ir[j], F);  // U^n was checked above, later inputs as results
        wsplit(U[j], F, alpha, W[j]);
      }
      // d: differences to the left cell; hp: half the + slope of the last cell;
      // f: its left face (f0: the lane's second face)
      double d[6], hp[3], f[3], hm0[3], f0[3];
#pragma unroll
      for (int q = 0; q < 6; ++q) d[q] = W[0][q] - lane_prev(W[CPT - 1][q]);
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          const double np = j + 1 < CPT ? W[j + 1 < CPT ? j + 1 : 0][r] : lane_next(W[0][r]);
          const double nm = j + 1 < CPT ? W[j + 1 < CPT ? j + 1 : 0][3 + r] : lane_next(W[0][3 + r]);
          const double dp = np - W[j][r], dm = nm - W[j][3 + r];
          const double hm = half_slope<UNL>(d[3 + r], dm);
          if (j == 0) {
            hm0[r] = hm;
          } else {  // face between cells j - 1 and j
            const double fj = face2(W[j > 0 ? j - 1 : 0][r], hp[r], W[j][3 + r], hm);
            if (j == 1)
              f0[r] = fj;
            else
              U[j > 0 ? j - 1 : 0][r] = fma(-hdts, fj - f[r], U[j > 0 ? j - 1 : 0][r]);
            f[r] = fj;
          }
          hp[r] = half_slope<UNL>(d[r], dp);
          d[r] = dp;
          d[3 + r] = dm;
        }
      }
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double fl = face2(W[CPT - 1][r], hp[r], lane_next(W[0][3 + r]), lane_next(hm0[r]));
        const double fp = lane_prev(fl);  // first face of the lane
        U[0][r] = fma(-hdts, (CPT == 1 ? fl : f0[r]) - fp, U[0][r]);
        if (CPT > 1) U[CPT - 1][r] = fma(-hdts, fl - f[r], U[CPT - 1][r]);
      }
      if (i + 1 < s) {
        double mx = 0.0;
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          ir[j] = rcp_nr(U[j][0]);
          double sp;
          const bool ps = speed1(U[j], ir[j], gam, &sp);
          if (own(j)) {
            phys &= ps;
            mx = fmax(mx, sp);
          }
        }
        double* S = L + (i & 1) * LINE_SETS;
        double* E = S + 16 * 4 * LINE_SLOT;
        auto put = [&](double* o, int j) {
#pragma unroll
          for (int r = 0; r < 3; ++r) o[r] = U[j][r];
          o[3] = ir[j];
        };
        // cells 2 and 3 of the wavefront and those before its last two (one
        // branch where the cells have the same place in their lanes)
        if constexpr (CPT <= 2) {
          if (wslot >= 0) {
#pragma unroll
            for (int j = 0; j < CPT; ++j) put(S + (wslot + j) * LINE_SLOT, j);
          }
        } else {
#pragma unroll
          for (int k = 2; k < 4; ++k) {
            if (lane == k / CPT) put(S + (wv * 4 + k - 2) * LINE_SLOT, k % CPT);
            if (lane == 63 - k / CPT) put(S + (wv * 4 + 5 - k) * LINE_SLOT, CPT - 1 - k % CPT);
          }
        }
        if (ends) {
#pragma unroll
          for (int j = 0; j < CPT; ++j) {
            const int c = c0 + j;
            if (own(j) && (c <= 1 || c >= Nx - 2)) {
              if (c <= 1) put(E + c * LINE_SLOT, j);
              if (c >= Nx - 2) put(E + (c - Nx + 4) * LINE_SLOT, j);
            }
          }
        }
        const double wm = wave_max_dpp(mx);
        if (lane == 0) S[LINE_SETS - 16 + wv] = wm;
      }
    }
    if (i + 1 < smax) __syncthreads();
    if (i + 1 < s) {
      const double* S = L + (i & 1) * LINE_SETS;
      const double* E = S + 16 * 4 * LINE_SLOT;
      auto get = [&](const double* o, int j) {
#pragma unroll
        for (int r = 0; r < 3; ++r) U[j][r] = o[r];
        ir[j] = o[3];
      };
      double m = S[LINE_SETS - 16 + (lane & 15)];
      m = dpp_max<0x111, 0xF>(m);
      m = dpp_max<0x112, 0xF>(m);
      m = dpp_max<0x114, 0xF>(m);
      m = dpp_max<0x118, 0xF>(m);
      alpha = lane_value(m, 15);
      if constexpr (CPT <= 2) {
        if (rslot >= 0) {
#pragma unroll
          for (int j = 0; j < CPT; ++j) get(S + (rslot + j) * LINE_SLOT, j);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (lane == k / CPT) get(S + (max(wv - 1, 0) * 4 + 2 + k) * LINE_SLOT, k % CPT);
          if (lane == 63 - k / CPT)
            get(S + (min(wv + 1, nwv - 1) * 4 + 1 - k) * LINE_SLOT, CPT - 1 - k % CPT);
        }
      }
      if (ends) {
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
          const int c = c0 + j;
          if ((c < 0 && c >= -2) || c == Nx || c == Nx + 1) {
            const int k = map_axis(c, Nx, bc);  // one of the row's end cells
            get(E + (k <= 1 ? k : k - Nx + 4) * LINE_SLOT, j);
          }
        }
      }
    }
  }
  if (s > 0) {
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      if (own(j)) {
#pragma unroll
        for (int r = 0; r < 3; ++r) out[(size_t)r * Nx + c0 + j] = U[j][r];
      }
    }
  }
  return phys;
}

// The Euler solve of a step on a 1D grid whose cells fit one group: one
// launch of one block for all s sub-steps, instead of one launch for the
// first and a block that kept the state in memory for the others.
template <typename T, int CPT, bool UNL>
__global__ __launch_bounds__(1024) void k_euler_line(StepArgs<T> a, Geom G) {
  __shared__ double L[LINE_LDS];
  const int s = open_substeps<1>(a, G);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool ok = euler_line<CPT, UNL>(a.U_in, (s & 1) ? a.UE1 : a.UE0, G.nc, G.bc[0], wv,
                                       (int)(blockDim.x >> 6), a.set_r[0], s, s,
                                       0.5 * ((G.dt / s) / G.dx), G.gam, L);
  if (!ok) atomicOr(a.flag, FLAG_NONPHYS);
}

}  // namespace hofks
