// sbm_tile.h -- pieces shared by the LDS-tiled 3D kernels (sbm_tiled.hip,
// sbm_split.hip): the level geometry, z chunks, face nodes, raw buffer access and
// the workgroup numbering.
#pragma once

#include "sbm_internal.h"

namespace sbm {

// The level geometry the tiled kernels need (3D only; fewer scalar registers
// than Geom).
struct TG {
  int nx, ny, nz, cx, cy, cz, nn;
  uint32_t dmask;
  int hx;
};

__device__ __forceinline__ int rows_hx(const TG &g) { return g.hx; }

inline TG make_tg(const GeomS &g) {
  return TG{g.nx, g.ny, g.nz, g.cx, g.cy, g.cz, (int)g.nn, g.dmask, g.hx};
}

__device__ __forceinline__ bool tg_dirichlet(const TG &g, int i, int j, int k, int comp) {
  const uint32_t m = g.dmask >> comp;
  return ((i == 0) && (m & 1u)) || ((i == g.nx - 1) && ((m >> 3) & 1u)) ||
         ((j == 0) && ((m >> 6) & 1u)) || ((j == g.ny - 1) && ((m >> 9) & 1u)) ||
         ((k == 0) && ((m >> 12) & 1u)) || ((k == g.nz - 1) && ((m >> 15) & 1u));
}

// Planes [k0, k1) of chunk tz.
__device__ __forceinline__ void tile_chunk(const TileGeom &tg, int tz, int nz, int &k0, int &k1) {
  if (tg.nzc > 0) {
    k0 = tz * nz / tg.nzc;
    k1 = (tz + 1) * nz / tg.nzc;
  } else {
    k0 = tz * tg.kz;
    k1 = min(k0 + tg.kz, nz);
  }
}

// Face node f of a launch with face blocks: the last column x = nx-1 (all
// rows) first, then the last row y = ny-1 (the other columns), plane by plane.
__device__ __forceinline__ bool face_node(const TG &g, const TileGeom &tg, int f, int &x, int &y,
                                          int &z) {
  const int per = (tg.xface ? g.ny : 0) + (tg.yface ? g.nx - tg.xface : 0);
  if (f >= per * g.nz) return false;
  z = f / per;
  const int e = f - z * per;
  if (tg.xface && e < g.ny) {
    x = g.nx - 1;
    y = e;
  } else {
    x = e - (tg.xface ? g.ny : 0);
    y = g.ny - 1;
  }
  return true;
}

// ---------------------------------------------------------------- buffers
//
// The tiled kernels address u, f, psi and the outputs through raw buffer
// descriptors: the per-thread byte offset within a plane (a VGPR computed once)
// plus the plane's offset (an SGPR) is added by the memory unit, and an offset
// at or past the buffer's size reads 0 and drops a store.  Halo entries
// outside the box therefore load as the zeros eq. K needs there, with no
// select per value, and a thread without a node stores nothing.  Offsets stay
// below 2^31 (tiled_ok limits a level's vector to that many bytes).
constexpr int kOOB = 0x7ffffff8;    // byte offset past every buffer
constexpr int kRsrcW3 = 0x00020000; // descriptor word 3: 32-bit data format, raw access

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, bytes, kRsrcW3);
}
template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
typedef unsigned int u32x2 __attribute__((__vector_size__(2 * sizeof(unsigned int))));
template <typename T>
__device__ __forceinline__ void bstore(T v, __amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
}

// The FP64 residual an FP32 half-sweep with DOT reads instead of its load:
// the load is r / s (s = sqrt(*ss)) formed as the mixed cast forms it, and the
// sum is r . (s u_out), the CG's r . z with z = s e.
struct DotSrc {
  const double *r, *ss;
};

// Hardware block b of a launch over n listed (or all) tiles: the tiles first,
// in the XCD-ordered numbering of the first n rounded up to 8 blocks (workgroup
// b runs on XCD b mod 8; each XCD gets a contiguous range of tiles); the face
// blocks of a whole-level launch last (short node-parallel blocks that fill
// the slots the last tiles leave idle).  Returns the logical tile, or -1 - fb
// for face block fb.
__device__ __forceinline__ int tile_or_face(int n) {
  const int n8 = (n + 7) / 8 * 8;
  const int b = blockIdx.x;
  if (b >= n8) return -1 - (b - n8);
  return (b & 7) * (n8 >> 3) + (b >> 3);
}

// The level's coefficients as the 4 scalars of CoefCubic when its cells are
// cubic (the same numbers, so the results are those of Coef).
template <typename T>
inline bool cubic_coef(const Coef<T> &C, CoefCubic<T> &cc) {
  cc = CoefCubic<T>{C.cd[0][0], C.cd[0][1], C.cp[0], C.cm[0]};
  for (int i = 0; i < 3; ++i) {
    if (C.cp[i] != cc.p || C.cm[i] != cc.m) return false;
    for (int j = 0; j < 3; ++j)
      if (C.cd[i][j] != (i == j ? cc.dd : cc.od)) return false;
  }
  return true;
}

// The edge sums E of the 8 cells P[c2][c1][c0] around a node and the diagonal D of
// K (stencil3's direct part).
template <typename T, typename CO>
__device__ __forceinline__ void zero_diag(const CO &C, const T (&P)[2][2][2], T (&E)[3][2],
                                          T dg[3]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    E[0][s] = P[0][0][s] + P[0][1][s] + P[1][0][s] + P[1][1][s];
    E[1][s] = P[0][s][0] + P[0][s][1] + P[1][s][0] + P[1][s][1];
    E[2][s] = P[s][0][0] + P[s][0][1] + P[s][1][0] + P[s][1][1];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
    dg[c] = coef_cd(C, c, 0) * (E[0][0] + E[0][1]) + coef_cd(C, c, 1) * (E[1][0] + E[1][1]) +
            coef_cd(C, c, 2) * (E[2][0] + E[2][1]);
}

// (K u)(n) at a node n whose centre and edge neighbours are 0: F[c][a][s] is
// component c at the face neighbour n + (2s - 1) e_a.  The expressions are
// stencil3's with the zero terms removed.
template <typename T, typename CO>
__device__ __forceinline__ void zero_face_stencil(const CO &C, const T (&P)[2][2][2],
                                                  const T (&E)[3][2], const T (&F)[3][3][2],
                                                  T out[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c)
    out[c] = -(coef_cd(C, c, 0) * (E[0][1] * F[c][0][1] + E[0][0] * F[c][0][0]) +
               coef_cd(C, c, 1) * (E[1][1] * F[c][1][1] + E[1][0] * F[c][1][0]) +
               coef_cd(C, c, 2) * (E[2][1] * F[c][2][1] + E[2][0] * F[c][2][0]));
#pragma unroll
  for (int pl = 0; pl < 3; ++pl) {
    const int a = (pl == 2) ? 1 : 0;
    const int b = (pl == 0) ? 1 : 2;
    const T cm = coef_cm(C, pl);
    T ra = T(0), rb = T(0);
#pragma unroll
    for (int qa = 0; qa < 2; ++qa)
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        const int sa = 2 * qa - 1, sb = 2 * qb - 1;
        T Fs;
        if (pl == 0) Fs = P[0][qb][qa] + P[1][qb][qa];
        else if (pl == 1) Fs = P[qb][0][qa] + P[qb][1][qa];
        else Fs = P[qb][qa][0] + P[qb][qa][1];
        const T w = (sa * sb > 0) ? Fs : -Fs;
        // u_b(n + sb e_b) - u_b(n + sa e_a) and u_a(n + sa e_a) - u_a(n + sb e_b)
        ra += w * (cm * (F[b][b][qb] - F[b][a][qa]));
        rb += w * (cm * (F[a][a][qa] - F[a][b][qb]));
      }
    out[a] -= ra;
    out[b] -= rb;
  }
}

// Workgroups of a tiled launch over n tiles: the tiles rounded up to a
// multiple of 8 (XCD order), then the face blocks of a whole-level launch.
inline int tiled_grid(int n, int nface) { return (n + 7) / 8 * 8 + nface; }

}  // namespace sbm
