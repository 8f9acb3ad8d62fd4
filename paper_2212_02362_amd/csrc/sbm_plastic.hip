// sbm_plastic.hip -- plastic strain on the finest grid (Sec. 3.1, 3D): the
// load of a cell plastic strain and the J2 radial-return update of the cell
// state, the two pointwise kernels of the staggered elastic / plastic step.
//
// Stress sigma = C (grad u - eps_p) turns the equilibrium into
// K u = b - div(psi C eps_p).  The divergence is the flux form of eq. K: for
// node n, component i,
//   fp_i(n) = -(1/4) sum_j (1/h_j) sum_{b in {0,1}^3} (2 b_j - 1) S_ij(c_b),
// over the 8 cells c_b = n - 1 + b around the node, S = psi C eps_p (cells
// outside the box count 0): the half-edge stresses are the means of the four
// cells around each edge, as the edge psi of eq. K.
//
// Cell state arrays (cells, x fastest): eps_p and beta as 6 components (xx,
// yy, zz, yz, xz, xy) one array after another, alpha one array.
#include <algorithm>

#include "sbm_internal.h"

namespace sbm {
namespace {

constexpr int kVi[6] = {0, 1, 2, 1, 0, 0}, kVj[6] = {0, 1, 2, 2, 2, 1};

// fp = -div(psi C eps_p) at every node.  A thread takes kz nodes of a column and
// marches up: it evaluates the cells (i, j - 1) and (i, j) of a layer and gets
// those at i - 1 from the lane before (63 nodes per wave, the first lane only
// serves the second), and what a layer gives the node below and the node above
// it differs in the sign of the stress along z alone: 14 values loaded per node
// instead of 56, a layer ahead of their use.  Bound by memory: 168 MB at 128^3 cells,
// 85 us a thread per node, 69 marching with four cells per thread, 50 as it is.
constexpr int kSourceNodes = kBlock / 64 * 63;  // nodes of a plane per workgroup
// Columns are as long as leaves this many workgroups (128^3: 512 workgroups 56 us,
// 1024 51, 2048 50, 3000 56).
constexpr int kSourceBlocks = 1536;
__global__ __launch_bounds__(kBlock) void k_plastic_source(Geom g, double lam, double mu,
                                                          double ihx, double ihy, double ihz,
                                                          const double *__restrict__ psi,
                                                          const double *__restrict__ ep,
                                                          double *__restrict__ fp, int kz,
                                                          int nbp) {
  const int b = xcd_block();
  const int zb = b / nbp;
  const int nxy = g.nx * g.ny;
  const int k0 = zb * kz, k1 = min(k0 + kz, g.nz);
  if (k0 >= k1) return;
  const int lane = threadIdx.x & 63;
  const int pid = (b - zb * nbp) * kSourceNodes + (int)(threadIdx.x >> 6) * 63 + lane - 1;
  const uint32_t pc = (uint32_t)min(max(pid, 0), nxy - 1);
  const int j = (int)g.fnx.div(pc), i = (int)(pc - (uint32_t)j * (uint32_t)g.nx);
  const bool own = lane > 0 && pid < nxy;
  const int64_t nc = g.nc, cxy = (int64_t)g.cx * g.cy;
  // the cells (i, j - 1) and (i, j), clamped into the box; weight 0 outside
  int cq[2];
  bool in[2];
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int y = j - 1 + m;
    in[m] = i < g.cx && y >= 0 && y < g.cy;
    cq[m] = min(i, g.cx - 1) + g.cx * min(max(y, 0), g.cy - 1);
  }
  auto load = [&](int z, double (&pv)[2], double (&ev)[2][6]) __attribute__((always_inline)) {
    const int64_t zo = min(max(z, 0), g.cz - 1) * cxy;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      pv[m] = psi[zo + cq[m]];
#pragma unroll
      for (int c = 0; c < 6; ++c) ev[m][c] = ep[c * nc + zo + cq[m]];
    }
  };
  // the in-plane part (both nodes) and the z part (+ above, - below) of a layer
  auto layer = [&](int z, const double (&pv)[2], const double (&ev)[2][6], double (&B)[3],
                   double (&Z)[3]) __attribute__((always_inline)) {
    const bool zin = z >= 0 && z < g.cz;
    double S[2][3][3];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const double w = zin && in[m] ? pv[m] : 0.0;
      const double tr = ev[m][0] + ev[m][1] + ev[m][2];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const double s = w * (2.0 * mu * ev[m][c] + (c < 3 ? lam * tr : 0.0));
        S[m][kVi[c]][kVj[c]] = s;
        S[m][kVj[c]][kVi[c]] = s;
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double x = (S[0][c][0] + S[1][c][0]) * ihx, y = (S[1][c][1] - S[0][c][1]) * ihy;
      const double v = (S[0][c][2] + S[1][c][2]) * ihz;
      const double lb = __shfl_up(y - x, 1), lv = __shfl_up(v, 1);
      B[c] = x + y + (i > 0 ? lb : 0.0);
      Z[c] = v + (i > 0 ? lv : 0.0);
    }
  };
  double pv[2], ev[2][6], pn[2], en[2][6], B0[3], Z0[3], B1[3], Z1[3];
  load(k0 - 1, pv, ev);
  load(k0, pn, en);
  layer(k0 - 1, pv, ev, B0, Z0);
  for (int k = k0; k < k1; ++k) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      pv[m] = pn[m];
#pragma unroll
      for (int c = 0; c < 6; ++c) ev[m][c] = en[m][c];
    }
    load(min(k + 1, k1 - 1), pn, en);
    __builtin_amdgcn_sched_barrier(0);
    layer(k, pv, ev, B1, Z1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (own) fp[c * g.nn + pid + (int64_t)k * nxy] = -0.25 * (B0[c] + B1[c] + (Z1[c] - Z0[c]));
      B0[c] = B1[c];
      Z0[c] = Z1[c];
    }
  }
}

// Radial return (linear combined hardening) of every cell for the strain of
// u: one thread per cell.  The state is read from (ep, alpha, beta) and written
// to (epn, alphan, betan); in place (the same arrays) only where the cell yields.
// Bound by memory: 232 B per cell out of place (128^3: 108 us, 4.5 TB/s; copies of
// the state and an update in place 84 + 109 us).
// Counts the yielding cells (integer sum per block, one atomic per block).
__global__ __launch_bounds__(kBlock) void k_return_map(Geom g, double mu, double sy, double hb,
                                                      double theta, double ihx, double ihy,
                                                      double ihz, const double *__restrict__ u,
                                                      const double *ep, const double *alpha,
                                                      const double *beta, double *epn,
                                                      double *alphan, double *betan,
                                                      int *__restrict__ count) {
  __shared__ int wcount[kBlock / 64];
  const int64_t cid = (int64_t)xcd_block() * kBlock + threadIdx.x;
  bool yielded = false;
  if (cid < g.nc) {
    int cx, cy, cz;
    cell_ijk(g, cid, cx, cy, cz);
    const int64_t nc = g.nc;
    // corner nodes: un[b][c] at node (cx + b0, cy + b1, cz + b2)
    double un[8][3];
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int64_t q = (cx + (b & 1)) + (int64_t)g.nx * ((cy + ((b >> 1) & 1)) +
                                                         (int64_t)g.ny * (cz + (b >> 2)));
#pragma unroll
      for (int c = 0; c < 3; ++c) un[b][c] = u[c * g.nn + q];
    }
    double e0[6], b0[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      e0[m] = ep[m * nc + cid];
      b0[m] = beta[m * nc + cid];
    }
    const double a0 = alpha[cid];
    __builtin_amdgcn_sched_barrier(0);
    // cell gradient G[c][l]: mean over the four cell edges along l
    const double ih[3] = {ihx, ihy, ihz};
    double G[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b)
          if ((b >> l) & 1) s += un[b][c] - un[b ^ (1 << l)][c];
        G[c][l] = 0.25 * s * ih[l];
      }
    // eta_trial = 2 mu dev(eps - eps_p) - beta
    double ee[6];
#pragma unroll
    for (int m = 0; m < 6; ++m)
      ee[m] = 0.5 * (G[kVi[m]][kVj[m]] + G[kVj[m]][kVi[m]]) - e0[m];
    const double tr3 = (ee[0] + ee[1] + ee[2]) / 3.0;
    double eta[6], n2 = 0.0;
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      eta[m] = 2.0 * mu * (ee[m] - (m < 3 ? tr3 : 0.0)) - b0[m];
      n2 += (m < 3 ? 1.0 : 2.0) * eta[m] * eta[m];
    }
    const double nrm = sqrt(n2);
    const double r23 = sqrt(2.0 / 3.0);
    const double ftrial = nrm - r23 * (sy + theta * hb * a0);
    if (ftrial > 0.0) {
      yielded = true;
      const double dg = ftrial / (2.0 * mu + (2.0 / 3.0) * hb);
      const double kb = (2.0 / 3.0) * (1.0 - theta) * hb * dg;
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        const double nm = eta[m] / nrm;
        epn[m * nc + cid] = e0[m] + dg * nm;
        betan[m * nc + cid] = b0[m] + kb * nm;
      }
      alphan[cid] = a0 + r23 * dg;
    } else {
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        if (epn != ep) epn[m * nc + cid] = e0[m];
        if (betan != beta) betan[m * nc + cid] = b0[m];
      }
      if (alphan != alpha) alphan[cid] = a0;
    }
  }
  if (count) {
    const uint64_t ball = __ballot(yielded);
    if ((threadIdx.x & 63) == 0) wcount[threadIdx.x >> 6] = __popcll(ball);
    __syncthreads();
    if (threadIdx.x == 0) {
      int s = 0;
      for (int w = 0; w < kBlock / 64; ++w) s += wcount[w];
      if (s) atomicAdd(count, s);
    }
  }
}

}  // namespace

hipError_t launch_plastic_source(const Level &L, double lam, double mu, const double *eps_p,
                                 double *fp, hipStream_t st) {
  (void)hipGetLastError();
  const int nbp = (int)(((int64_t)L.g.nx * L.g.ny + kSourceNodes - 1) / kSourceNodes);
  const int kz =
      (int)std::max<int64_t>(1, std::min<int64_t>(16, (int64_t)nbp * L.g.nz / kSourceBlocks));
  const int nz = (L.g.nz + kz - 1) / kz;
  hipLaunchKernelGGL(k_plastic_source, dim3((nbp * nz + 7) / 8 * 8), dim3(kBlock), 0, st, L.g, lam,
                     mu, 1.0 / L.h[0], 1.0 / L.h[1], 1.0 / L.h[2], L.psi64, eps_p, fp, kz, nbp);
  return hipGetLastError();
}

hipError_t launch_return_map(const Level &L, double mu, double sigma_y, double hbar, double theta,
                             const double *u, const double *eps_p, const double *alpha,
                             const double *beta, double *eps_out, double *alpha_out,
                             double *beta_out, int *count, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_return_map, dim3(grid_blocks(L.g.nc)), dim3(kBlock), 0, st, L.g, mu,
                     sigma_y, hbar, theta, 1.0 / L.h[0], 1.0 / L.h[1], 1.0 / L.h[2], u, eps_p,
                     alpha, beta, eps_out, alpha_out, beta_out, count);
  return hipGetLastError();
}

}  // namespace sbm
