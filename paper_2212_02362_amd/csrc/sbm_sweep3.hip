// sbm_sweep3.hip -- a whole Gauss-Seidel sweep of a small 3D level in one launch (FP64).
//
// On levels of a few thousand to some ten thousand nodes a half-sweep takes 4 to 5
// us whatever it moves (launch and one memory round trip).  Here a workgroup takes a
// tile of 8 x 4 x 4 nodes with a halo of two, relaxes the first colour on the tile
// and one node around it and the second on the tile: every value is that of the two
// half-sweeps, the halo's computed again by the neighbouring tiles.  Each colour is
// relaxed from the state at its start (new values in registers until every thread has
// read the old ones).  The result goes to another buffer than the one read.  Bound by
// latency: one round trip for everything the tile reads, then two stencils.  A sweep,
// two half-sweeps -> one launch: 17^3 9.5 -> 5.2 us, 33^3 9.4 -> 6.9 us.
#include "sbm_tile.h"

namespace sbm {
namespace {

constexpr int BX = 8, BY = 4, BZ = 4;                  // tile (even: parities are the region's)
constexpr int RX = BX + 4, RY = BY + 4, RZ = BZ + 4;   // region
constexpr int RN = RX * RY * RZ;
constexpr int NT3 = 192;
constexpr int NA = (BX + 2) / 2 * (BY + 2) * (BZ + 2);  // first-colour nodes, one per x-pair
constexpr int NB = BX / 2 * BY * BZ;
static_assert(NA <= NT3 && BX * BY * BZ <= NT3 && RN % NT3 == 0, "a node per thread");

template <typename CO>
__global__ __launch_bounds__(NT3) void k_sweep3(Geom g, CO C, const double *__restrict__ psi,
                                                const double *__restrict__ xin,
                                                const double *__restrict__ f,
                                                double *__restrict__ xout, double omega, int c0,
                                                int ntx, int nty, int ntiles) {
  __shared__ double sx[3][RN];
  __shared__ double sp[RN];
  const int li = xcd_block();
  if (li >= ntiles) return;
  const int t = threadIdx.x, nn = (int)g.nn, nxy = g.nx * g.ny;
  const int tx = li % ntx, rest = li / ntx, ty = rest % nty, tz = rest / nty;
  const int gx0 = tx * BX - 2, gy0 = ty * BY - 2, gz0 = tz * BZ - 2;
  constexpr int Q = RN / NT3;
  auto inside = [&](int x, int y, int z) {
    return x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
  };
  // the thread's node of either colour (region coordinates): of a pair along x
  const bool isa = t < NA, isb = t < NB;
  int a[3], b[3];
  {
    constexpr int PA = (BX + 2) / 2, PB = BX / 2;
    const int ra = t / PA, rb = t / PB;
    a[1] = 1 + ra % (BY + 2);
    a[2] = 1 + ra / (BY + 2);
    a[0] = 1 + 2 * (t - ra * PA) + ((c0 + 1 + a[1] + a[2]) & 1);
    b[1] = 2 + rb % BY;
    b[2] = 2 + rb / BY;
    b[0] = 2 + 2 * (t - rb * PB) + ((1 - c0 + b[1] + b[2]) & 1);
  }
  const bool oka = isa && inside(gx0 + a[0], gy0 + a[1], gz0 + a[2]);
  const bool okb = isb && inside(gx0 + b[0], gy0 + b[1], gz0 + b[2]);
  const int qa = oka ? gx0 + a[0] + g.nx * (gy0 + a[1]) + nxy * (gz0 + a[2]) : 0;
  const int qb = okb ? gx0 + b[0] + g.nx * (gy0 + b[1]) + nxy * (gz0 + b[2]) : 0;
  double xv[Q][3], pv[Q], fa[3], fb[3];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = t + q * NT3;
    const int x = gx0 + e % RX, y = gy0 + (e / RX) % RY, z = gz0 + e / (RX * RY);
    const int id = min(max(x, 0), g.nx - 1) + g.nx * min(max(y, 0), g.ny - 1) +
                   nxy * min(max(z, 0), g.nz - 1);
#pragma unroll
    for (int c = 0; c < 3; ++c) xv[q][c] = xin ? xin[c * nn + id] : 0.0;
    pv[q] = psi[min(max(x, 0), g.cx - 1) +
                g.cx * (min(max(y, 0), g.cy - 1) + g.cy * min(max(z, 0), g.cz - 1))];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    fa[c] = f[c * nn + qa];
    fb[c] = f[c * nn + qb];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int e = t + q * NT3;
    const int x = gx0 + e % RX, y = gy0 + (e / RX) % RY, z = gz0 + e / (RX * RY);
    const bool in = inside(x, y, z);
    const bool cell = x >= 0 && x < g.cx && y >= 0 && y < g.cy && z >= 0 && z < g.cz;
#pragma unroll
    for (int c = 0; c < 3; ++c) sx[c][e] = in ? xv[q][c] : 0.0;
    sp[e] = cell ? pv[q] : 0.0;
  }
  __syncthreads();
  auto relax = [&](const int (&n)[3], const double (&fv)[3], double (&nv)[3])
                   __attribute__((always_inline)) {
    const int id = n[0] + RX * (n[1] + RY * n[2]);
    double P[2][2][2];
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
      for (int c1 = 0; c1 < 2; ++c1)
#pragma unroll
        for (int d = 0; d < 2; ++d) P[c2][c1][d] = sp[id - 1 + d + RX * (c1 - 1 + RY * (c2 - 1))];
    auto U = [&](int c, int dx, int dy, int dz) -> double {
      return sx[c][id + dx + RX * (dy + RY * dz)];
    };
    double out[3], dg[3];
    stencil3<double>(C, P, U, out, dg);
    const uint32_t bits = face_bits(g, gx0 + n[0], gy0 + n[1], gz0 + n[2]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      // (a displacement DOF may have no solid around it: a zero diagonal)
      const double uc = U(c, 0, 0, 0), upd = uc + omega * (fv[c] - out[c]) / dg[c];
      nv[c] = ((g.dmask >> c) & bits) ? uc : upd;
    }
  };
  double nv[3];
  if (oka) relax(a, fa, nv);
  __syncthreads();
  if (oka)
#pragma unroll
    for (int c = 0; c < 3; ++c) sx[c][a[0] + RX * (a[1] + RY * a[2])] = nv[c];
  __syncthreads();
  if (okb) relax(b, fb, nv);
  // the tile's first colour from LDS, its second from the threads that relaxed it
  if (okb)
#pragma unroll
    for (int c = 0; c < 3; ++c) xout[c * nn + qb] = nv[c];
  if (t < NB) {
    // the other node of the B thread's pair
    const int ox = b[0] ^ 1;
    if (inside(gx0 + ox, gy0 + b[1], gz0 + b[2])) {
      const int id = gx0 + ox + g.nx * (gy0 + b[1]) + nxy * (gz0 + b[2]);
#pragma unroll
      for (int c = 0; c < 3; ++c) xout[c * nn + id] = sx[c][ox + RX * (b[1] + RY * b[2])];
    }
  }
}

}  // namespace

hipError_t launch_sweep3(const Level &L, const double *xin, const double *f, double *xout,
                         double omega, int first_colour, hipStream_t st) {
  if (L.g.dim != 3 || L.g.hx || xin == xout) return hipErrorInvalidValue;
  const int ntx = (L.g.nx + BX - 1) / BX, nty = (L.g.ny + BY - 1) / BY;
  const int n = ntx * nty * ((L.g.nz + BZ - 1) / BZ);
  const Coef<double> &C = L.c64;
  CoefCubic<double> cc;
  const bool cubic = cubic_coef(C, cc);
  (void)hipGetLastError();
  const dim3 grid((n + 7) / 8 * 8), block(NT3);
  if (cubic)
    hipLaunchKernelGGL(k_sweep3<CoefCubic<double>>, grid, block, 0, st, L.g, cc, L.psi64, xin, f,
                       xout, omega, first_colour, ntx, nty, n);
  else
    hipLaunchKernelGGL(k_sweep3<Coef<double>>, grid, block, 0, st, L.g, C, L.psi64, xin, f, xout,
                       omega, first_colour, ntx, nty, n);
  return hipGetLastError();
}

}  // namespace sbm
