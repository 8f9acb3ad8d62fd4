// sbm_split.hip -- the colour half-sweep of the solver's wide 3D levels, whose
// vectors have split rows (sbm_device.h: even columns of a row first, then the
// odd ones, so the two colours are the two halves of every row).
//
// A workgroup owns a node column tile and marches up a chunk of z planes; four
// planes of u and three of cell psi live in an LDS ring.  What bounds it is the
// memory it moves.  Natural rows made a half-sweep read and copy both colours,
// because they interleave in every cache line: 80 B per node in FP64.  Here the
// relaxed colour goes to the other buffer and nothing is copied (u, psi, half of
// f read, half of u written: 56 B), the state of a colour being in whichever
// buffer its last half-sweep wrote: the kernel takes the buffer of the relaxed
// colour (us) and that of the other (uo).  u and psi are loaded 16 bytes per
// lane (6 loads per plane step instead of 11) into LDS planes of the same order
// (rows of one colour contiguous, so the LDS reads of a wave are consecutive),
// and every load of a step is issued without a branch before the arithmetic.
// Isolated launches, natural -> split: 257^3 FP64 339 -> 242 us (3.9 TB/s of its
// 56 B per node), FP32 205 -> 131 us; 129^3 FP64 41 -> 32, FP32 27.5 -> 22.8 us.
// One barrier per step with the fourth plane or two with three: the same.
#include "sbm_tile.h"

namespace sbm {
namespace {

constexpr int kOff = 0x7ffffff0;  // byte offset past every buffer (16-byte loads)

typedef unsigned int u32v4 __attribute__((ext_vector_type(4)));

// What a half-sweep does besides: kDot (FP64) forms the partial sums of
// f . u_out over free DOF of both colours, kZero relaxes from a state that is
// zero on the relaxed colour (us is not read: the second half-sweep from a zero
// iterate, k_zero_split being the first).
enum SplitMode { kPlain, kDot, kZero };

// Tile and LDS shape: TX x TY nodes, 256 threads, NP x-pairs per thread.  FP64:
// 64 x 8.  FP32: 128 x 8 (131 us at 257^3 where 64 x 16 takes 152 us: longer runs
// of a row per load).  Both take the same LDS bytes.
template <typename T, int MODE>
struct Shape {
  static constexpr int W = sizeof(T), NV = 16 / W;          // elements per 16-byte chunk
  static constexpr int NP = 8 / W;
  static constexpr int TX = 64 * NP, TY = 8, NT = 256;
  static constexpr int HR = (TX / 2 + NV) / NV * NV;        // entries of a half row with halo
  static constexpr int CH = HR / NV, RY = TY + 2;
  static constexpr int NCU = 3 * RY * CH;                   // chunks of one colour's plane
  static constexpr int CP = (TX + 1 + NV - 1) / NV * NV;    // cells of an LDS psi row
  static constexpr int NCP = (TY + 1) * (CP / NV);          // chunks of a psi plane
  static constexpr int OTH = MODE == kZero ? 0 : 512 * NV;  // offset of the other colour
  static constexpr int PU = OTH + NCU * NV, PP = NCP * NV;  // LDS plane sizes
  static_assert(NCU > NT && NCU <= 2 * NT && NCP > NT && NCP <= 2 * NT, "two chunks per thread");
};

template <typename T, typename CO, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_rb_split(
    TG g, CO C, const T *__restrict__ psi, const T *__restrict__ us, const T *__restrict__ uo,
    const T *__restrict__ f, T *__restrict__ u_out, T omega, int colour, TileGeom tg,
    double *__restrict__ partials) {
  using S = Shape<T, MODE>;
  constexpr int W = S::W, NV = S::NV, NP = S::NP, NT = S::NT;
  constexpr bool DOT = MODE == kDot, ZERO = MODE == kZero;
  __shared__ __attribute__((aligned(16))) T su[4][S::PU];
  __shared__ __attribute__((aligned(16))) T sp[3][S::PP];
  __shared__ double red[DOT ? NT / 64 + 1 : 1];
  const int nx = g.nx, nn = g.nn, H = g.hx, t = threadIdx.x;
  const int li = tile_or_face(tg.ntiles);
  if (li < 0) {
    // the last column / row of a 2^n + 1 level, a node per thread
    const int fb = -1 - li;
    double acc = 0.0;
    int x, y, z;
    if (face_node(g, tg, fb * NT + t, x, y, z)) {
      const int q = split_x(H, x) + nx * (y + g.ny * z);
      const bool own = ((x + y + z) & 1) == colour;
      T nv[3];
      if (own) {
        T out[3], dg[3], uc[3] = {T(0), T(0), T(0)};
        if constexpr (ZERO) {
          T P[2][2][2], E[3][2], F[3][3][2];
#pragma unroll
          for (int b = 0; b < 8; ++b) {
            const int i = x - 1 + (b & 1), j = y - 1 + ((b >> 1) & 1), k = z - 1 + (b >> 2);
            const bool in = i >= 0 && i < g.cx && j >= 0 && j < g.cy && k >= 0 && k < g.cz;
            P[b >> 2][(b >> 1) & 1][b & 1] = in ? psi[i + g.cx * (j + g.cy * k)] : T(0);
          }
#pragma unroll
          for (int b = 0; b < 6; ++b) {
            const int a = b >> 1, s = 2 * (b & 1) - 1;
            const int i = x + (a == 0 ? s : 0), j = y + (a == 1 ? s : 0), k = z + (a == 2 ? s : 0);
            const bool in = i >= 0 && i < nx && j >= 0 && j < g.ny && k >= 0 && k < g.nz;
#pragma unroll
            for (int c = 0; c < 3; ++c)
              F[c][a][b & 1] = in ? uo[c * nn + split_x(H, i) + nx * (j + g.ny * k)] : T(0);
          }
          zero_diag<T>(C, P, E, dg);
          zero_face_stencil<T>(C, P, E, F, out);
        } else {
          node_stencil<T, 3, true, TG, CO>(g, C, psi, us, x, y, z, out, dg, uc, uo);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const T upd = uc[c] + omega * (f[c * nn + q] - out[c]) / dg[c];
          nv[c] = tg_dirichlet(g, x, y, z, c) ? uc[c] : upd;
          u_out[c * nn + q] = nv[c];
        }
      } else if (DOT) {
#pragma unroll
        for (int c = 0; c < 3; ++c) nv[c] = uo[c * nn + q];
      }
      if constexpr (DOT) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          if (!tg_dirichlet(g, x, y, z, c)) acc += (double)f[c * nn + q] * (double)nv[c];
      }
    }
    if constexpr (DOT) {
      const double sum = block_sum(acc, red);
      if (t == 0) partials[tg.ntiles + fb] = sum;
    }
    return;
  }
  if (li >= tg.ntiles) return;
  const int nxy = nx * g.ny, vb = 3 * nn * W;
  const int tx = li % tg.ntx, rest = li / tg.ntx, ty = rest % tg.nty, tz = rest / tg.nty;
  const int x0 = tx * S::TX, y0 = ty * S::TY;
  int k0, k1;
  tile_chunk(tg, tz, g.nz, k0, k1);
  // (u is read up to 64 bytes past its end: workspace)
  // Byte offsets of the thread's chunks.  A half row of u starts at column x0
  // (even half) or x0 - 1 (odd half) and runs S::HR entries.  Rows outside the
  // box read 0; entries past the box in x hold whatever lies there (the row's
  // other half, whose colour may not have been written yet), so the tiles at
  // the box faces replace them by 0 (ka, kb: a bit per entry inside).
  // Relaxed-colour rows are the half of parity (colour + y + z), so the two
  // offsets of a chunk change places from plane to plane.
  int va[2], vbo[2], vp[2], ka[2], kb[2], kp[2];
  const bool edge = x0 == 0 || x0 + S::TX > nx - 1;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int e = t + NT * m;
    va[m] = vbo[m] = vp[m] = kOff;
    ka[m] = kb[m] = kp[m] = 0;
    if (e < S::NCU) {
      const int c = e / (S::RY * S::CH), r = e - c * (S::RY * S::CH);
      const int row = r / S::CH, ch = r - row * S::CH, gy = y0 - 1 + row;
      if (gy >= 0 && gy < g.ny) {
        const int base = c * nn + gy * nx + x0 / 2 + NV * ch;
        const int even = base * W, odd = (base + H - 1) * W;
        va[m] = ((colour + gy) & 1) ? odd : even;
        vbo[m] = ((colour + gy) & 1) ? even : odd;
        int ke = 0, ko = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int xe = x0 + 2 * (NV * ch + i);
          ke |= (xe < nx ? 1 : 0) << i;
          ko |= (xe > 0 && xe - 1 < nx ? 1 : 0) << i;
        }
        ka[m] = ((colour + gy) & 1) ? ko : ke;
        kb[m] = ((colour + gy) & 1) ? ke : ko;
      }
    }
    if (e < S::NCP) {
      const int row = e / (S::CP / NV), ch = e - row * (S::CP / NV), gy = y0 - 1 + row;
      // (psi - NV is readable)
      if (gy >= 0 && gy < g.cy) vp[m] = (gy * g.cx + x0 - 1 + NV + NV * ch) * W;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int x = x0 - 1 + NV * ch + i;
        kp[m] |= (x >= 0 && x < g.cx ? 1 : 0) << i;
      }
    }
  }
  const T *psim = psi - NV;
  auto fetch_u = [&](int z, u32v4 (&r)[4]) __attribute__((always_inline)) {
    const bool in = z >= 0 && z < g.nz;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(us, in ? vb + 64 : 0);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(uo, in ? vb + 64 : 0);
    const int so = z * nxy * W;
    const bool odd = z & 1;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      if constexpr (!ZERO)
        r[m] = __builtin_bit_cast(
            u32v4, __builtin_amdgcn_raw_buffer_load_b128(rs, odd ? vbo[m] : va[m], so, 0));
      r[2 + m] = __builtin_bit_cast(
          u32v4, __builtin_amdgcn_raw_buffer_load_b128(ro, odd ? va[m] : vbo[m], so, 0));
    }
  };
  auto put_u = [&](int z, u32v4 (&r)[4]) __attribute__((always_inline)) {
    T *d = su[z & 3];
    if (edge) {
      const bool odd = z & 1;
#pragma unroll
      for (int m = ZERO ? 2 : 0; m < 4; ++m) {
        const int keep = (odd != (m >= 2)) ? kb[m & 1] : ka[m & 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) r[m][i] = (keep >> (i / (4 / NV))) & 1 ? r[m][i] : 0u;
      }
    }
#pragma unroll
    for (int m = ZERO ? 2 : 0; m < 4; ++m)
      if ((m & 1) == 0 || t < S::NCU - NT)
        *(u32v4 *)(d + (m >> 1) * S::OTH + (t + NT * (m & 1)) * NV) = r[m];
  };
  auto fetch_p = [&](int z, u32v4 (&r)[2]) __attribute__((always_inline)) {
    const bool in = z >= 0 && z < g.cz;
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(psim, in ? (g.cx * g.cy * g.cz + 2 * NV) * W : 0);
    const int so = z * g.cx * g.cy * W;
#pragma unroll
    for (int m = 0; m < 2; ++m)
      r[m] = __builtin_bit_cast(u32v4, __builtin_amdgcn_raw_buffer_load_b128(rp, vp[m], so, 0));
  };
  auto put_p = [&](T *d, u32v4 (&r)[2]) __attribute__((always_inline)) {
    if (edge)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) r[m][i] = (kp[m] >> (i / (4 / NV))) & 1 ? r[m][i] : 0u;
    *(u32v4 *)(d + t * NV) = r[0];
    if (t < S::NCP - NT) *(u32v4 *)(d + (t + NT) * NV) = r[1];
  };
  // The thread's x-pairs q: columns x0 + 2 p, + 1 (p = p0 + 32 q) of row y0 + yl;
  // the pair's nodes sit at half-row position x0/2 + p of either half
  const int yl = t / 32, p0 = t % 32, gy = y0 + yl;
  const int vh = gy < g.ny ? (gy * nx + x0 / 2 + p0) * W : kOff;  // p0 of the even half
  auto node_off = [&](int q, int px) __attribute__((always_inline)) {
    return (vh != kOff && x0 + 2 * (p0 + 32 * q) + px < nx) ? vh + (32 * q + px * H) * W : kOff;
  };
  // f of the relaxed nodes of plane k (0 past the chunk); with DOT also of the
  // other node of each pair
  auto fetch_f = [&](int k, T (&r)[NP][3], T (&rc)[DOT ? NP : 1][3]) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rf = make_rsrc(f, k < k1 ? vb : 0);
    const int so = k * nxy * W, px = (colour + gy + k) & 1;
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        r[q][c] = bload<T>(rf, node_off(q, px), so + c * nn * W);
        if constexpr (DOT) rc[q][c] = bload<T>(rf, node_off(q, 1 - px), so + c * nn * W);
      }
  };
  const __amdgpu_buffer_rsrc_t rout = make_rsrc(u_out, vb);
  T FN[NP][3], FC[DOT ? NP : 1][3];
  fetch_f(k0, FN, FC);
  {
    u32v4 a0[4], a1[4], a2[4], p0[2], p1[2];
    fetch_u(k0 - 1, a0);
    fetch_u(k0, a1);
    fetch_u(k0 + 1, a2);
    fetch_p(k0 - 1, p0);
    fetch_p(k0, p1);
    put_u(k0 - 1, a0);
    put_u(k0, a1);
    put_u(k0 + 1, a2);
    put_p(sp[(k0 + 2) % 3], p0);
    put_p(sp[k0 % 3], p1);
  }
  __syncthreads();
  double acc = 0.0;
  for (int k = k0; k < k1; ++k) {
    T fr[NP][3], fc[DOT ? NP : 1][3];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        fr[q][c] = FN[q][c];
        if constexpr (DOT) fc[q][c] = FC[q][c];
      }
    u32v4 RU[4], RP[2];
    fetch_u(k + 2, RU);
    fetch_p(k + 1, RP);
    fetch_f(k + 1, FN, FC);
    const T *Lm = su[(k + 3) & 3], *L0 = su[k & 3], *L1 = su[(k + 1) & 3];
    const T *Pm = sp[(k + 2) % 3], *P0 = sp[k % 3];
    const uint32_t by = (gy == 0 ? 64u : 0u) | (gy == g.ny - 1 ? 512u : 0u) |
                        (k == 0 ? 4096u : 0u) | (k == g.nz - 1 ? 32768u : 0u);
    const int so = k * nxy * W, px = (colour + gy + k) & 1, row = (yl + 1) * S::HR;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int p = p0 + 32 * q, gx = x0 + 2 * p + px, lc = 2 * p + px;
      T P[2][2][2];
#pragma unroll
      for (int c1 = 0; c1 < 2; ++c1)
#pragma unroll
        for (int c0 = 0; c0 < 2; ++c0) {
          P[0][c1][c0] = Pm[(yl + c1) * S::CP + lc + c0];
          P[1][c1][c0] = P0[(yl + c1) * S::CP + lc + c0];
        }
      // neighbours of the node's own colour are the edge ones, of the other the
      // face ones; in a half row the node sits at p + px, its x-neighbours'
      // half has them at p and p + 1
      auto U = [&](int c, int dx, int dy, int dz) -> T {
        const T *L = (dz < 0 ? Lm : (dz > 0 ? L1 : L0)) + (((dx + dy + dz) & 1) ? S::OTH : 0);
        return L[c * S::RY * S::HR + row + dy * S::HR + p + (dx == 0 ? px : (dx > 0 ? 1 : 0))];
      };
      T out[3], dg[3];
      if constexpr (ZERO) {
        T E[3][2], F[3][3][2];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            F[c][0][s] = U(c, 2 * s - 1, 0, 0);
            F[c][1][s] = U(c, 0, 2 * s - 1, 0);
            F[c][2][s] = U(c, 0, 0, 2 * s - 1);
          }
        zero_diag<T>(C, P, E, dg);
        zero_face_stencil<T>(C, P, E, F, out);
      } else {
        stencil3<T>(C, P, U, out, dg);
      }
      const uint32_t fb = by | (gx == 0 ? 1u : 0u) | (gx == nx - 1 ? 8u : 0u);
      const int vo = node_off(q, px);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const bool fixed = ((g.dmask >> c) & fb) != 0u;
        T uc = T(0);
        if constexpr (!ZERO) uc = U(c, 0, 0, 0);
        // (a displacement DOF may have no solid around it: a zero diagonal)
        const T upd = uc + omega * (fr[q][c] - out[c]) / dg[c];
        const T nv = fixed ? uc : upd;
        bstore<T>(nv, rout, vo, so + c * nn * W);
        if constexpr (DOT) {
          // f . u_out at both nodes of the pair (a node outside the box adds nothing)
          const int gxc = gx + 1 - 2 * px;
          const uint32_t fbc = by | (gxc == 0 ? 1u : 0u) | (gxc == nx - 1 ? 8u : 0u);
          const bool ok = vo != kOff && !fixed;
          const bool okc = node_off(q, 1 - px) != kOff && !((g.dmask >> c) & fbc);
          acc += ok ? (double)fr[q][c] * (double)nv : 0.0;
          acc += okc ? (double)fc[q][c] * (double)U(c, 1 - 2 * px, 0, 0) : 0.0;
        }
      }
    }
    // the fourth plane is free: one barrier orders both the writes below before
    // the next step's reads and this step's reads before its writes
    put_u(k + 2, RU);
    put_p(sp[(k + 1) % 3], RP);
    __syncthreads();
  }
  if constexpr (DOT) {
    const double sum = block_sum(acc, red);
    if (t == 0) partials[li] = sum;
  }
}

// Tiles of a level: z chunks for about 1280 tiles
// (FP64 1280 tiles at 257^3: 241 us against 248 for 1152 and 252 for 1536), chunks of
// at least 8 planes (two more are loaded per chunk; 129^3 FP64: 32 us in 8-plane
// chunks, 33 us in 4-plane ones), or of 4 where that leaves fewer than the 512
// tiles the chip holds at once.
template <typename T>
TileGeom split_geom(const TG &g) {
  using S = Shape<T, kPlain>;
  TileGeom t{};
  t.xface = g.nx > S::TX && g.nx % S::TX == 1;
  t.yface = g.ny > S::TY && g.ny % S::TY == 1;
  t.ntx = t.xface ? g.nx / S::TX : (g.nx + S::TX - 1) / S::TX;
  t.nty = t.yface ? g.ny / S::TY : (g.ny + S::TY - 1) / S::TY;
  const int64_t per_plane = (t.xface ? g.ny : 0) + (t.yface ? g.nx - t.xface : 0);
  t.nface = (int)((per_plane * g.nz + S::NT - 1) / S::NT);
  const int cols = t.ntx * t.nty;
  int nzc = std::min(1280 / cols, g.nz / 8);
  if (nzc * cols < 512) nzc = std::min((512 + cols - 1) / cols, g.nz / 4);
  t.nzc = std::max(nzc, 1);
  t.kz = (g.nz + t.nzc - 1) / t.nzc;
  t.ntiles = cols * t.nzc;
  return t;
}

}  // namespace

bool split_level(const Level &L, bool fp32) {
  // FP64: 3D levels wider than 96 nodes (below, the 64-node tiles leave most CUs
  // idle and a launch is bound by latency).  FP32: wider than 192 nodes (129^3:
  // 25 us either way, and the node-parallel passes around it prefer natural
  // rows there).  The buffer offsets of a vector must stay below kOff.
  return L.g.dim == 3 && L.g.nx > (fp32 ? 192 : 96) && L.g.ny > 24 &&
         3 * L.g.nn * (int64_t)sizeof(double) < (int64_t)kOff - 64;
}

int rb_split_partials(const Level &L) {
  const TileGeom tg = split_geom<double>(make_tg(L.g));
  return tg.ntiles + tg.nface;
}

template <typename T>
hipError_t launch_rb_split(const Level &L, const T *psi, const Coef<T> &C, const T *us,
                           const T *uo, const T *f, T *u_out, double omega, int colour,
                           hipStream_t st, double *partials) {
  if (!L.g.hx || (partials && (sizeof(T) != 8 || !us))) return hipErrorInvalidValue;
  const TG gg = make_tg(L.g);
  const TileGeom tg = split_geom<T>(gg);
  CoefCubic<T> cc;
  const bool cubic = cubic_coef(C, cc);
  (void)hipGetLastError();
  auto go = [&](auto &&cf, auto mode) {
    hipLaunchKernelGGL((k_rb_split<T, std::decay_t<decltype(cf)>, decltype(mode)::value>),
                       dim3(tiled_grid(tg.ntiles, tg.nface)), dim3(256), 0, st, gg, cf, psi, us,
                       uo, f, u_out, (T)omega, colour, tg, partials);
  };
  auto pick = [&](auto mode) {
    if (cubic) go(cc, mode);
    else go(C, mode);
  };
  if (!us) {
    pick(std::integral_constant<int, kZero>{});
  } else if (partials) {
    if constexpr (sizeof(T) == 8) pick(std::integral_constant<int, kDot>{});
  } else {
    pick(std::integral_constant<int, kPlain>{});
  }
  return hipGetLastError();
}

#define SBM_SPLIT_INST(T)                                                                       \
  template hipError_t launch_rb_split<T>(const Level &, const T *, const Coef<T> &, const T *,  \
                                         const T *, const T *, T *, double, int, hipStream_t,   \
                                         double *);
SBM_SPLIT_INST(double)
SBM_SPLIT_INST(float)

}  // namespace sbm
