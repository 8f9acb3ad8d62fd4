// sbm_leg2d.hip -- the legs of a 2D V-cycle, one launch each (FP64, Gauss-Seidel).
//
// Down: the colour half-sweeps of the pre-smoothing, the residual and its full
// weighting to the coarse load.  Up: the correction's prolongation and the
// post-smoothing.  Launch by launch these were 7 and 5 passes: on levels of up to
// some 257^2 nodes bound by launch and memory latency (3 to 5 us each whatever the
// size), above by reading and writing the iterate in each.  Here a workgroup takes
// a tile of TS x TS nodes with a halo as deep as the half-sweeps reach (one node
// per half-sweep, two more for the residual under the restriction), keeps iterate
// and psi in LDS and the load in registers, and relaxes a region that shrinks by a
// node per half-sweep: every value is that of the separate passes, the halo's
// computed again by the neighbouring tiles.  A half-sweep holds its new values in
// registers until every thread has read the old ones, which is the frozen copy of
// the separate passes.  The result goes to another buffer than the one read.
// Bound by arithmetic and barriers (the diagonal is inverted once; at 2049^2 the
// 60 B per node it moves would take 50 us).  Both legs, passes -> legs: 2049^2 500 ->
// 253 us, 1025^2 170 -> 83 us, 65^2 54 -> 19 us.
#include "sbm_internal.h"

namespace sbm {
namespace {

// The coefficients of 2D eq. K as scalars (an array captured by the stencil's
// lambda went to scratch memory).
struct Coef2 {
  double xx, xy, yx, yy, p, m;
};
__device__ __forceinline__ double coef_cd(const Coef2 &C, int i, int j) {
  return i == 0 ? (j == 0 ? C.xx : C.xy) : (j == 0 ? C.yx : C.yy);
}
__device__ __forceinline__ double coef_cp(const Coef2 &C, int) { return C.p; }
__device__ __forceinline__ double coef_cm(const Coef2 &C, int) { return C.m; }

template <bool UP, int NU, int TS>
struct LegShape {
  static constexpr int N = 2 * NU;                // half-sweeps
  static constexpr int H = UP ? N : N + 2;        // halo (even: pairs keep their parity)
  static constexpr int RS = TS + 2 * H;           // region
  static constexpr int HR = RS / 2;               // x-pairs per row
  static constexpr int NT = TS == 32 ? 512 : 256;
  static constexpr int Q = (RS * HR + NT - 1) / NT;  // x-pairs per thread
};

template <bool UP, int NU, int TS>
__global__ __launch_bounds__(TS == 32 ? 512 : 256) void k_leg2(
    Geom g, Geom gc, Coef2 C, const double *__restrict__ psi,
    const double *__restrict__ xin, const double *__restrict__ f, double *__restrict__ xout,
    const double *__restrict__ e, double *__restrict__ fc, double *__restrict__ ec, double omega,
    int c0, int ntx, int ntiles) {
  using S = LegShape<UP, NU, TS>;
  constexpr int H = S::H, RS = S::RS, HR = S::HR, NT = S::NT, Q = S::Q, RT = TS + 2;
  // rows hold the even columns first, then the odd ones: the nodes of a colour and
  // their x-neighbours are consecutive over the lanes
  __shared__ double sx[2][RS * RS];
  __shared__ double sp[RS * RS];
  __shared__ double sr[UP ? 1 : 2][UP ? 1 : RT * RT];  // residual of the tile and one node around
  const int li = xcd_block();
  if (li >= ntiles) return;
  const int ty = li / ntx, tx = li - ty * ntx;
  const int gx0 = tx * TS - H, gy0 = ty * TS - H;
  const int nn = (int)g.nn, ncn = (int)gc.nn;
  auto at = [](int lx, int ly) { return ly * RS + (lx & 1) * HR + (lx >> 1); };
  // per x-pair: [0] its node of colour c0, [1] the other (an index that is known when
  // compiled; by column the arrays went to scratch memory)
  double fv[Q][2][2];
  auto column = [&](int ly, int k) { return (c0 + ly + k) & 1; };
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = threadIdx.x + q * NT;
    const int ly = t / HR, p = t - ly * HR;
    const int gx = gx0 + 2 * p, gy = gy0 + ly;
    const bool live = t < RS * HR;
    const int yc = min(max(gy, 0), g.ny - 1), zc = min(max(gy, 0), g.cy - 1);
    double xv[2][2], pv[2], ev[2][2][2];
    bool in[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int h = column(ly, k);
      in[k] = live && gx + h >= 0 && gx + h < g.nx && gy >= 0 && gy < g.ny;
      const int id = min(max(gx + h, 0), g.nx - 1) + g.nx * yc;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        fv[q][k][c] = f[c * nn + id];
        xv[k][c] = xin ? xin[c * nn + id] : 0.0;
      }
      pv[k] = psi[min(max(gx + h, 0), g.cx - 1) + g.cx * zc];
    }
    if constexpr (UP) {
      const int I = gx >> 1, J = gy >> 1;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          const int ic = min(max(I + o, 0), gc.nx - 1) + gc.nx * min(max(J + b, 0), gc.ny - 1);
#pragma unroll
          for (int c = 0; c < 2; ++c) ev[b][o][c] = e[c * ncn + ic];
        }
    }
    if (!live) continue;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int h = column(ly, k);
      const int id = at(2 * p + h, ly);
      const bool cell = gx + h >= 0 && gx + h < g.cx && gy >= 0 && gy < g.cy;
      sp[id] = cell ? pv[k] : 0.0;
      uint32_t fb = 0;
      if constexpr (UP) fb = face_bits(g, gx + h, gy, 0);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double v = xv[k][c];
        if constexpr (UP) {
          const bool oj = gy & 1;
          double acc = ev[0][0][c];
          if (h) acc += ev[0][1][c];
          if (oj) acc += ev[1][0][c];
          if (oj && h) acc += ev[1][1][c];
          const double w = 1.0 / (double)((h ? 2 : 1) * (oj ? 2 : 1));
          v += ((g.dmask >> c) & fb) ? 0.0 : w * acc;
        }
        sx[c][id] = in[k] ? v : 0.0;
      }
    }
  }
  __syncthreads();
  // eq. K at region node (lx, ly)
  auto stencil = [&](int lx, int ly, double (&out)[3], double (&dg)[3], double (&uc)[2])
                     __attribute__((always_inline)) {
    double P[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int o = 0; o < 2; ++o) P[a][o] = sp[at(lx - 1 + o, ly - 1 + a)];
    auto U = [&](int c, int dx, int dy) -> double { return sx[c][at(lx + dx, ly + dy)]; };
    stencil2<double>(C, P, U, out, dg);
    uc[0] = U(0, 0, 0);
    uc[1] = U(1, 0, 0);
  };
  // omega over the diagonal (0 on displacement DOF and outside the box): every
  // node is relaxed NU times
  double wd[Q][2][2];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = threadIdx.x + q * NT;
    const int ly = t / HR, p = t - ly * HR, gy = gy0 + ly;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int lx = 2 * p + column(ly, k), gx = gx0 + lx;
      wd[q][k][0] = wd[q][k][1] = 0.0;
      if (t < RS * HR && lx > 0 && lx < RS - 1 && ly > 0 && ly < RS - 1 && gx >= 0 && gx < g.nx &&
          gy >= 0 && gy < g.ny) {
        double out[3], dg[3], uc[2];
        stencil(lx, ly, out, dg, uc);
        const uint32_t fb = face_bits(g, gx, gy, 0);
#pragma unroll
        for (int c = 0; c < 2; ++c) wd[q][k][c] = ((g.dmask >> c) & fb) ? 0.0 : omega / dg[c];
      }
    }
  }
#pragma unroll
  for (int s = 1; s <= S::N; ++s) {
    const int k = 1 - (s & 1);
    double nv[Q][2];
    int nid[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int t = threadIdx.x + q * NT;
      const int ly = t / HR, p = t - ly * HR;
      const int lx = 2 * p + column(ly, k);
      const int gx = gx0 + lx, gy = gy0 + ly;
      nid[q] = -1;
      if (t < RS * HR && lx >= s && lx < RS - s && ly >= s && ly < RS - s && gx >= 0 &&
          gx < g.nx && gy >= 0 && gy < g.ny) {
        double out[3], dg[3], uc[2];
        stencil(lx, ly, out, dg, uc);
        nid[q] = at(lx, ly);
#pragma unroll
        for (int c = 0; c < 2; ++c)
          nv[q][c] = uc[c] + wd[q][k][c] * (fv[q][k][c] - out[c]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (nid[q] >= 0) {
        sx[0][nid[q]] = nv[q][0];
        sx[1][nid[q]] = nv[q][1];
      }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = threadIdx.x + q * NT;
    const int ly = t / HR, p = t - ly * HR, gy = gy0 + ly;
    if (t >= RS * HR) continue;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int lx = 2 * p + column(ly, k), gx = gx0 + lx;
      const bool in = gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
      if (in && lx >= H && lx < H + TS && ly >= H && ly < H + TS) {
        const int id = gx + g.nx * gy;
#pragma unroll
        for (int c = 0; c < 2; ++c) xout[c * nn + id] = sx[c][at(lx, ly)];
      }
      if constexpr (!UP) {
        if (lx >= H - 1 && lx <= H + TS && ly >= H - 1 && ly <= H + TS) {
          double r[2] = {0.0, 0.0};
          if (in) {
            double out[3], dg[3], uc[2];
            stencil(lx, ly, out, dg, uc);
            const uint32_t fb = face_bits(g, gx, gy, 0);
#pragma unroll
            for (int c = 0; c < 2; ++c)
              r[c] = ((g.dmask >> c) & fb) ? 0.0 : fv[q][k][c] - out[c];
          }
          const int id = (ly - H + 1) * RT + lx - H + 1;
          sr[0][id] = r[0];
          sr[1][id] = r[1];
        }
      }
    }
  }
  if constexpr (!UP) {
    __syncthreads();
    const int t = threadIdx.x, cy = t / (TS / 2), cx = t - cy * (TS / 2);
    const int I = tx * (TS / 2) + cx, J = ty * (TS / 2) + cy;
    if (cy < TS / 2 && I < gc.nx && J < gc.ny) {
      double acc[2] = {0.0, 0.0};
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          const double w = (dy == 0 ? 1.0 : 0.5) * (dx == 0 ? 1.0 : 0.5);
          const int id = (2 * cy + dy + 1) * RT + 2 * cx + dx + 1;
#pragma unroll
          for (int c = 0; c < 2; ++c) acc[c] += w * sr[c][id];
        }
      const int id = I + gc.nx * J;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        fc[c * ncn + id] = is_dirichlet(gc, I, J, 0, c) ? 0.0 : acc[c] * 0.25;
        if (ec) ec[c * ncn + id] = 0.0;
      }
    }
  }
}

template <bool UP>
hipError_t launch_leg2(const Level &L, const Level &Lc, const double *xin, const double *f,
                       double *xout, const double *e, double *fc, double *ec, double omega,
                       int first_colour, int nu, hipStream_t st) {
  if (L.g.dim != 2 || nu < 1 || nu > 2 || xin == xout) return hipErrorInvalidValue;
  (void)hipGetLastError();
  const Coef<double> &K = L.c64;
  const Coef2 C{K.cd[0][0], K.cd[0][1], K.cd[1][0], K.cd[1][1], K.cp[0], K.cm[0]};
  auto go = [&](auto nuc, auto tsc) {
    constexpr int NU = decltype(nuc)::value, TS = decltype(tsc)::value;
    const int ntx = (L.g.nx + TS - 1) / TS, nty = (L.g.ny + TS - 1) / TS;
    const int n = ntx * nty;
    hipLaunchKernelGGL((k_leg2<UP, NU, TS>), dim3((n + 7) / 8 * 8), dim3(LegShape<UP, NU, TS>::NT),
                       0, st, L.g, Lc.g, C, L.psi64, xin, f, xout, e, fc, ec, omega,
                       first_colour, ntx, n);
  };
  // large tiles (less halo: 1.9 times the nodes instead of 3.1) where they leave a
  // workgroup per CU; below, more workgroups (at 513 x 385 both take the same time)
  const bool large = (int64_t)((L.g.nx + 31) / 32) * ((L.g.ny + 31) / 32) >= 256;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using T16 = std::integral_constant<int, 16>;
  using T32 = std::integral_constant<int, 32>;
  if (nu == 1 && large) go(I1{}, T32{});
  else if (nu == 1) go(I1{}, T16{});
  else if (large) go(I2{}, T32{});
  else go(I2{}, T16{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_leg2_down(const Level &L, const Level &Lc, const double *xin, const double *f,
                            double *xout, double *fc, double *ec, double omega, int first_colour,
                            int nu, hipStream_t st) {
  return launch_leg2<false>(L, Lc, xin, f, xout, nullptr, fc, ec, omega, first_colour, nu, st);
}

hipError_t launch_leg2_up(const Level &L, const Level &Lc, const double *xin, const double *f,
                          double *xout, const double *e, double omega, int first_colour, int nu,
                          hipStream_t st) {
  return launch_leg2<true>(L, Lc, xin, f, xout, e, nullptr, nullptr, omega, first_colour, nu, st);
}

}  // namespace sbm
