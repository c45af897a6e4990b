// Discrete adjoint of the tracer step (FP64), in the variable Z = M^-1 lambda.
//
// Forward step: x^{n+1} = S P(x^n) + c with P the SSP-RK3 stages of
// L = M^-1 R and S = (M - dt A)^-1 M.  With lambda = M Z the reverse sweep is
//
//   mu       = (M - dt A^T)^-1 M Z^{n+1}                    (transposed solve)
//   dJ/dkappa_l += dt mu^T (dA/dkappa_l) x^{n+1}             (A is linear in kappa)
//   Zb2 = 2/3 (mu + dt Lt mu),  Zb1 = 1/4 (Zb2 + dt Lt Zb2)
//   Z^n = (Zb1 + dt Lt Zb1) + 1/3 mu + 3/4 Zb2                (reverse RK3 stages)
//
// where Lt = M^-1 R_lin^T is the adjoint of L in the M inner product and
// R_lin the advective residual without the exterior inflow values.  Per prism
// q, with the upwind-positive face matrices K+ of the forward kernel,
//
//   (R_lin^T y)_j = int phi_j U.grad(y_h) dV - sum_faces K+ (y_q - y_nbr),
//
// (y_nbr = 0 on open boundaries, no term on walls): the volume part reuses
// the forward kernel's contravariant contractions, the face part is the
// downwind counterpart of the forward upwind flux.
#include "internal.h"
#include "quadrature.h"

namespace sdg {
namespace {

__device__ __forceinline__ double ld(const double* __restrict__ row, uint32_t byte_off) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(row) + byte_off);
}
// Row r of a [..][6][S] nodal array at byte offset off: one uniform base per
// 6-row block and 32-bit offsets (a 6-row block is below 4 GiB).
__device__ __forceinline__ double ldr(const double* __restrict__ arr, size_t S, int r, uint32_t off) {
  return ld(arr + (size_t)(r / 6 * 6) * S, (uint32_t)(r % 6) * (uint32_t)(S * 8) + off);
}
__device__ __forceinline__ void st(double* __restrict__ row, uint32_t byte_off, double v) {
  *reinterpret_cast<double*>(reinterpret_cast<char*>(row) + byte_off) = v;
}
__device__ __forceinline__ double upos(double x) { return x > 0.0 ? x : 0.0; }

// symmetric 3x3 storage: 0:00 1:11 2:22 3:01 4:02 5:12
__device__ __forceinline__ int sidx(int a, int b) {
  return a == b ? a : (a + b == 1 ? 3 : (a + b == 2 ? 4 : 5));
}

// ---------------------------------------------------------------------------
// Adjoint stage: out = b (Y + dt M^-1 R_lin^T Y) + a1 X1 + a2 X2
// ---------------------------------------------------------------------------
struct AdjStageArgs {
  DevMesh m;
  const WgTile* tiles;
  int32_t n_tiles;
  int32_t xcd;
  const double* Y;
  const double* X1;   // may be null (then a1 is ignored)
  const double* X2;
  double* out;        // may alias X1 or X2 (element-local reads), never Y
  const double* U;
  double dt, b, a1, a2;
};

// The residuals are formed up to here, and no instruction moves across: keeps a
// term's loads and factors from being live together with another's.
template <int NF>
__device__ __forceinline__ void formed(double (&res)[NF][6]) {
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) asm volatile("" : "+v"(res[f][i]));
  __builtin_amdgcn_sched_barrier(0);
}

// One thread per prism.  No load depends on control flow: threads past their
// column's depth run on in-bounds padding slots of their cell and skip the
// store, faces without a live neighbour address the prism's own nodes.  The terms
// are taken one after the other, each term's neighbour values requested one term
// ahead: the kernel is bound by the latency of its loads at two wavefronts per
// SIMD.  Against loads behind branches per face, each waiting on its own:
// 18.8 -> 11.3 us (2 fields, 55 k prisms), 91.7 -> 84.3 us (1 field, 1.0 M prisms).
// With SH each wavefront puts its layer's Y and horizontal velocity in LDS, reads
// them again from there for each term, and with them its neighbours in the cell:
// the address unit of the loads is then no longer the bound of a large launch, where
// a neighbour gather costs it five times a row of the own prisms.
template <int NF>
constexpr int kAdjRows = 6 * NF + 12;   // LDS rows of a wavefront: Y, u, v

template <int NF, bool WZ, bool SH>
__global__ __launch_bounds__(256) void adj_stage_kernel(AdjStageArgs a) {
  // each wavefront's own rows: its LDS accesses complete in order, no barrier needed
  extern __shared__ __align__(16) char adj_lds[];
  double* sh = SH ? reinterpret_cast<double*>(adj_lds) + (threadIdx.x >> 6) * (kAdjRows<NF> * kCell) : nullptr;
  const DevMesh& m = a.m;
  const WgTile tile = a.tiles[a.xcd ? xcd_tile(blockIdx.x, a.n_tiles) : (int)blockIdx.x];
  const int lane = threadIdx.x & (kCell - 1);
  const int l = tile.layer0 + (threadIdx.x >> 6);
  const int c = tile.cell * kCell + lane;
  const int N = m.nlay[c];
  const int depth = (m.cell_base[tile.cell + 1] - m.cell_base[tile.cell]) / kCell;
  if (l >= depth) return;  // uniform per wavefront
  const size_t S = (size_t)m.n_slots;
  const size_t LS = (size_t)m.n_lslots;
  const int CS = m.n_col_slots;
  const uint32_t p = (uint32_t)m.cell_base[tile.cell] + (uint32_t)l * kCell + lane;
  const uint32_t lt = (uint32_t)m.cell_lbase[tile.cell] + (uint32_t)l * kCell + lane;
  const uint32_t rs = (uint32_t)(S * 8);
  const uint32_t po = p * 8u;
  const uint32_t co = (uint32_t)c * 8u;
  const uint32_t co4 = (uint32_t)c * 4u;
  const double* __restrict__ Y = a.Y;
  const double* __restrict__ U = a.U;
  const double* __restrict__ geo = m.geo;

  const double xxi = ld(geo + G_XXI * CS, co), xet = ld(geo + G_XET * CS, co);
  const double yxi = ld(geo + G_YXI * CS, co), yet = ld(geo + G_YET * CS, co);
  const double Jh = ld(geo + G_JH * CS, co);
  int nslots[3], metas[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    nslots[e] = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(m.nbr_slot + e * CS) + co4);
    metas[e] = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(m.nbr_meta + e * CS) + co4);
  }
  double zt[3], zb[3], dz[3];
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    zt[v] = ld(m.zl + v * LS, lt * 8u);
    zb[v] = ld(m.zl + v * LS, (lt + kCell) * 8u);
    dz[v] = zt[v] - zb[v];
  }
  double res[NF][6];
  // the prism's own velocity and Y, loaded once and reused by every term
  double u[6], v[6], w[6], yv[NF][6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    u[i] = ldr(U, S, i, po);
    v[i] = ldr(U, S, 6 + i, po);
    w[i] = WZ ? 0.0 : ldr(U, S, 12 + i, po);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) yv[f][i] = ldr(Y, S, f * 6 + i, po);

  // lateral face e: the neighbour's velocity and Y at the face nodes A top, B top,
  // A bottom, B bottom, and the face's normal and length; with SH a neighbour in the
  // cell (here) is read from LDS at the time of its use, at offsets lo
  double nu[2][4], nv[2][4], ny4[2][NF][4], fn[2][3];
  uint32_t lo[2][2];
  bool here[2];
  const uint32_t cell_base = (uint32_t)m.cell_base[tile.cell];
  auto request_face = [&](int e) {
    const int s = e & 1;
    const bool live = nslots[e] >= 0 && l < (metas[e] >> 2);
    const int kp = metas[e] & 3;
    const uint32_t nA = live ? (uint32_t)((kp + 1) % 3) : (uint32_t)e;
    const uint32_t nB = live ? (uint32_t)kp : (uint32_t)((e + 1) % 3);
    const uint32_t nl = (uint32_t)nslots[e] - cell_base;   // < 64 iff the neighbour is in this cell
    here[s] = SH && (!live || nl < (uint32_t)kCell);
    const uint32_t src = live ? nl : (uint32_t)lane;
    lo[s][0] = here[s] ? nA * kCell + src : 0u;
    lo[s][1] = here[s] ? nB * kCell + src : 0u;
    const uint32_t pno = live ? ((uint32_t)nslots[e] + (uint32_t)l * kCell) * 8u : po;
    const uint32_t no[4] = {nA * rs + pno, nB * rs + pno, (nA + 3u) * rs + pno, (nB + 3u) * rs + pno};
    fn[s][0] = ld(geo + (G_NX + e) * CS, co);
    fn[s][1] = ld(geo + (G_NY + e) * CS, co);
    fn[s][2] = ld(geo + (G_LE + e) * CS, co);
    if (!here[s]) {
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        nu[s][n] = ld(U, no[n]);
        nv[s][n] = ld(U + 6 * S, no[n]);
      }
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int n = 0; n < 4; ++n) ny4[s][f][n] = ld(Y + (size_t)(f * 6) * S, no[n]);
    }
  };
  auto resolve_face = [&](int s) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const uint32_t o = lo[s][n & 1] + (uint32_t)(n >> 1) * 3u * kCell;
      const double x = sh[6 * NF * kCell + o], y = sh[(6 * NF + 6) * kCell + o];
      nu[s][n] = here[s] ? x : nu[s][n];
      nv[s][n] = here[s] ? y : nv[s][n];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const double t = sh[f * 6 * kCell + o];
        ny4[s][f][n] = here[s] ? t : ny4[s][f][n];
      }
    }
  };
  // with SH the own values are read from LDS again for each term
  auto reread = [&]() {
    if constexpr (SH) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        u[i] = sh[(6 * NF + i) * kCell + lane];
        v[i] = sh[(6 * NF + 6 + i) * kCell + lane];
#pragma unroll
        for (int f = 0; f < NF; ++f) yv[f][i] = sh[(f * 6 + i) * kCell + lane];
      }
    }
  };
  // the layer above (side 0, its bottom nodes) or below (side 1, its top nodes)
  double nw[2][9], ny3[2][NF][3];
  auto request_layer = [&](int s) {
    const int oo = s == 0 ? 3 : 0;
    const uint32_t pno = (s == 0 ? (l > 0 ? p - kCell : p) : (l + 1 < depth ? p + kCell : p)) * 8u;
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      nw[s][n] = ldr(U, S, oo + n, pno);
      nw[s][3 + n] = ldr(U, S, 6 + oo + n, pno);
      nw[s][6 + n] = WZ ? 0.0 : ldr(U, S, 12 + oo + n, pno);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int n = 0; n < 3; ++n) ny3[s][f][n] = ldr(Y, S, f * 6 + oo + n, pno);
  };
  request_face(0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (SH) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
      for (int f = 0; f < NF; ++f) sh[(f * 6 + i) * kCell + lane] = yv[f][i];
      sh[(6 * NF + i) * kCell + lane] = u[i];
      sh[(6 * NF + 6 + i) * kCell + lane] = v[i];
    }
    asm volatile("" ::: "memory");
  }

  // ---- volume: int phi_j U.grad(y_h) ----
  // sum over the points of w_q lambda_n x y for x, y linear over the triangle, by
  // the closed form (X Y + x_n Y + X y_n + x.y + 2 x_n y_n) / 120 of the cubic
  {
    double hx[2][3], he[2][3], G[2][6];
    const double zs = dz[0] + dz[1] + dz[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const double tk = kZt[k], bk = kZb[k];
      const double z_xi = tk * (zt[1] - zt[0]) + bk * (zb[1] - zb[0]);
      const double z_et = tk * (zt[2] - zt[0]) + bk * (zb[2] - zb[0]);
      double al[3], be[3], cz[3];
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        const double ua = tk * u[n] + bk * u[n + 3];
        const double va = tk * v[n] + bk * v[n + 3];
        al[n] = yet * ua - xet * va;
        be[n] = xxi * va - yxi * ua;
        double x = -(z_xi * al[n] + z_et * be[n]);
        if (!WZ) x += Jh * (tk * w[n] + bk * w[n + 3]);
        cz[n] = (1.0 / 120.0) * x;
      }
      const double as = al[0] + al[1] + al[2], bs = be[0] + be[1] + be[2], cs = cz[0] + cz[1] + cz[2];
      const double ax = zs * as + (dz[0] * al[0] + dz[1] * al[1] + dz[2] * al[2]);
      const double bx = zs * bs + (dz[0] * be[0] + dz[1] * be[1] + dz[2] * be[2]);
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        hx[k][n] = (1.0 / 240.0) * (ax + zs * al[n] + dz[n] * (as + 2.0 * al[n]));
        he[k][n] = (1.0 / 240.0) * (bx + zs * be[n] + dz[n] * (bs + 2.0 * be[n]));
        G[k][n] = 2.0 * cs + 4.0 * cz[n];
      }
      G[k][3] = cs + cz[0] + cz[1];
      G[k][4] = cs + cz[0] + cz[2];
      G[k][5] = cs + cz[1] + cz[2];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double* y = yv[f];
      const double d0 = y[0] - y[3], d1 = y[1] - y[4], d2 = y[2] - y[5];
#pragma unroll
      for (int i = 0; i < 6; ++i) res[f][i] = 0.0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double tk = kZt[k], bk = kZb[k];
        const double yx = tk * (y[1] - y[0]) + bk * (y[4] - y[3]);
        const double ye = tk * (y[2] - y[0]) + bk * (y[5] - y[3]);
#pragma unroll
        for (int n = 0; n < 3; ++n) {
          const double gz = 0.5 * (G[k][sidx(n, 0)] * d0 + G[k][sidx(n, 1)] * d1 + G[k][sidx(n, 2)] * d2);
          const double s = hx[k][n] * yx + he[k][n] * ye + gz;
          res[f][n] += tk * s;
          res[f][n + 3] += bk * s;
        }
      }
    }
  }
  formed<NF>(res);

  // ---- lateral faces: -K+ (y_q - y_nbr), nothing at a wall, y_nbr = 0 at an open boundary ----
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    if (e < 2) request_face(e + 1);
    else request_layer(0);
    __builtin_amdgcn_sched_barrier(0);
    const int A = e, B = (e + 1) % 3, s2 = e & 1;
    if constexpr (SH) resolve_face(s2);
    reread();
    const bool interior = nslots[e] >= 0;
    const bool wall = interior && l >= (metas[e] >> 2);
    const double nx = fn[s2][0], ny = fn[s2][1];
    const double Le = wall ? 0.0 : fn[s2][2];
    const int oi[4] = {A, B, A + 3, B + 3};      // the face's own nodes
    double un[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const double own = nx * u[oi[n]] + ny * v[oi[n]];
      const double avg = 0.5 * (own + nx * nu[s2][n] + ny * nv[s2][n]);
      un[n] = interior ? avg : own;
    }
    double gp[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double s = kS[j], s1 = 1.0 - kS[j];
      const double dS = kSw[j] * Le * 0.5 * (s1 * dz[A] + s * dz[B]);
      double qp[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double q = (s1 * (kZt[k] * un[0] + kZb[k] * un[2]) + s * (kZt[k] * un[1] + kZb[k] * un[3])) * dS;
        qp[k] = upos(q);
      }
      gp[j][0] = kZt[0] * kZt[0] * qp[0] + kZt[1] * kZt[1] * qp[1];
      gp[j][1] = kZt[0] * kZb[0] * qp[0] + kZt[1] * kZb[1] * qp[1];
      gp[j][2] = kZb[0] * kZb[0] * qp[0] + kZb[1] * kZb[1] * qp[1];
    }
    double Kp[3][3];
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int y = 0; y < 3; ++y) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const double sj = kS[j], s1j = 1.0 - kS[j];
          acc += (x == 0 ? s1j * s1j : (x == 1 ? s1j * sj : sj * sj)) * gp[j][y];
        }
        Kp[x][y] = acc;
      }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double d[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        d[n] = yv[f][oi[n]] - (interior ? ny4[s2][f][n] : 0.0);
        d[n] = wall ? 0.0 : d[n];
      }
      res[f][A] -= Kp[0][0] * d[0] + Kp[1][0] * d[1] + Kp[0][1] * d[2] + Kp[1][1] * d[3];
      res[f][B] -= Kp[1][0] * d[0] + Kp[2][0] * d[1] + Kp[1][1] * d[2] + Kp[2][1] * d[3];
      res[f][A + 3] -= Kp[0][1] * d[0] + Kp[1][1] * d[1] + Kp[0][2] * d[2] + Kp[1][2] * d[3];
      res[f][B + 3] -= Kp[1][1] * d[0] + Kp[2][1] * d[1] + Kp[1][2] * d[2] + Kp[2][2] * d[3];
    }
    formed<NF>(res);
  }

  // ---- top and bottom faces ----
  double x1[NF][6], x2[NF][6];
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    if (side == 0) request_layer(1);
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        if (side == 0) x1[f][i] = a.X1 ? ldr(a.X1, S, f * 6 + i, po) : 0.0;
        else x2[f][i] = a.X2 ? ldr(a.X2, S, f * 6 + i, po) : 0.0;
      }
    __builtin_amdgcn_sched_barrier(0);
    reread();
    const int o = side == 0 ? 0 : 3;
    const bool has_nb = side == 0 ? (l > 0) : (l < N - 1);
    const double* zf = side == 0 ? zt : zb;
    const double zxi = zf[1] - zf[0], zet = zf[2] - zf[0];
    const double jzx = zxi * yet - zet * yxi;
    const double jzy = zet * xxi - zxi * xet;
    const double sg = side == 0 ? 1.0 : -1.0;
    double un[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      double own = -(u[o + n] * jzx + v[o + n] * jzy);
      if (!WZ) own += Jh * w[o + n];
      double nb = -(nw[side][n] * jzx + nw[side][3 + n] * jzy);
      if (!WZ) nb += Jh * nw[side][6 + n];
      un[n] = has_nb ? 0.5 * (own + nb) : own;
    }
    double Kp[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const double fq = sg * kTw[q] * (kL0[q] * un[0] + kL1[q] * un[1] + kL2[q] * un[2]);
      const double qp = upos(fq);
      Kp[0] += kL0[q] * kL0[q] * qp;
      Kp[1] += kL1[q] * kL1[q] * qp;
      Kp[2] += kL2[q] * kL2[q] * qp;
      Kp[3] += kL0[q] * kL1[q] * qp;
      Kp[4] += kL0[q] * kL2[q] * qp;
      Kp[5] += kL1[q] * kL2[q] * qp;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double d[3];
#pragma unroll
      for (int n = 0; n < 3; ++n) d[n] = yv[f][o + n] - (has_nb ? ny3[side][f][n] : 0.0);
      res[f][o] -= Kp[0] * d[0] + Kp[3] * d[1] + Kp[4] * d[2];
      res[f][o + 1] -= Kp[3] * d[0] + Kp[1] * d[1] + Kp[5] * d[2];
      res[f][o + 2] -= Kp[4] * d[0] + Kp[5] * d[1] + Kp[2] * d[2];
    }
    formed<NF>(res);
  }
  if (l >= N) return;

  // ---- M^-1 and the combination ----
  reread();
  const double m00 = 3.0 * dz[0] + dz[1] + dz[2];
  const double m11 = dz[0] + 3.0 * dz[1] + dz[2];
  const double m22 = dz[0] + dz[1] + 3.0 * dz[2];
  const double m01 = dz[0] + dz[1] + 0.5 * dz[2];
  const double m02 = dz[0] + dz[2] + 0.5 * dz[1];
  const double m12 = dz[1] + dz[2] + 0.5 * dz[0];
  const double c00 = m11 * m22 - m12 * m12, c01 = m02 * m12 - m01 * m22, c02 = m01 * m12 - m02 * m11;
  const double c11 = m00 * m22 - m02 * m02, c12 = m01 * m02 - m00 * m12, c22 = m00 * m11 - m01 * m01;
  const double sc = 120.0 / (Jh * (m00 * c00 + m01 * c01 + m02 * c02));
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const double ht[3] = {2.0 * res[f][0] - res[f][3], 2.0 * res[f][1] - res[f][4], 2.0 * res[f][2] - res[f][5]};
    const double hb[3] = {2.0 * res[f][3] - res[f][0], 2.0 * res[f][4] - res[f][1], 2.0 * res[f][5] - res[f][2]};
    double L[6];
    L[0] = sc * (c00 * ht[0] + c01 * ht[1] + c02 * ht[2]);
    L[1] = sc * (c01 * ht[0] + c11 * ht[1] + c12 * ht[2]);
    L[2] = sc * (c02 * ht[0] + c12 * ht[1] + c22 * ht[2]);
    L[3] = sc * (c00 * hb[0] + c01 * hb[1] + c02 * hb[2]);
    L[4] = sc * (c01 * hb[0] + c11 * hb[1] + c12 * hb[2]);
    L[5] = sc * (c02 * hb[0] + c12 * hb[1] + c22 * hb[2]);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      double o = a.b * (yv[f][i] + a.dt * L[i]);
      if (a.X1) o += a.a1 * x1[f][i];
      if (a.X2) o += a.a2 * x2[f][i];
      st(a.out + (size_t)(f * 6 + i) * S, po, o);
    }
  }
}

// ---------------------------------------------------------------------------
// Per-prism geometry shared by the transposed solve and the kappa gradient
// ---------------------------------------------------------------------------
struct LayerGeo {
  double dz[3];
  double hbar;
};

__device__ __forceinline__ void load_layer(const DevMesh& m, size_t lt, LayerGeo& g) {
  const size_t LS = (size_t)m.n_lslots;
#pragma unroll
  for (int v = 0; v < 3; ++v) g.dz[v] = m.zl[v * LS + lt] - m.zl[v * LS + lt + kCell];
  g.hbar = (g.dz[0] + g.dz[1] + g.dz[2]) * (1.0 / 3.0);
}

__device__ __forceinline__ void vertical_stiffness(const LayerGeo& g, double Jh, double kv[6]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) kv[i] = 0.0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const double l0 = kL0[q], l1 = kL1[q], l2 = kL2[q];
    const double inv = kTw[q] / (l0 * g.dz[0] + l1 * g.dz[1] + l2 * g.dz[2]);
    kv[0] += l0 * l0 * inv;
    kv[1] += l1 * l1 * inv;
    kv[2] += l2 * l2 * inv;
    kv[3] += l0 * l1 * inv;
    kv[4] += l0 * l2 * inv;
    kv[5] += l1 * l2 * inv;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) kv[i] *= Jh;
}

__device__ __forceinline__ void mass_z(const LayerGeo& g, double Jh, double mz[6]) {
  const double s = Jh * (1.0 / 120.0);
  const double* dz = g.dz;
  mz[0] = s * (3.0 * dz[0] + dz[1] + dz[2]);
  mz[1] = s * (dz[0] + 3.0 * dz[1] + dz[2]);
  mz[2] = s * (dz[0] + dz[1] + 3.0 * dz[2]);
  mz[3] = s * (dz[0] + dz[1] + 0.5 * dz[2]);
  mz[4] = s * (dz[0] + dz[2] + 0.5 * dz[1]);
  mz[5] = s * (dz[1] + dz[2] + 0.5 * dz[0]);
}

__device__ __forceinline__ double penalty(double eta, double ka, double kb, double ha, double hb) {
  return eta * 0.5 * (ka + kb) / fmin(ha, hb);
}

// ---------------------------------------------------------------------------
// Transposed column solve: (M - dt A^T) mu = M Z
// ---------------------------------------------------------------------------
// The transposed column matrix has diagonal blocks D_l^T = [TT BT; TB BB]
// (the 3x3 sub-blocks of D_l are symmetric), the block left of the diagonal
// Lo_l = C_{l-1}^T (only columns of the bottom nodes of l-1 nonzero) and the
// block right of it Up_l = B_{l+1}^T (only columns of the top nodes of l+1):
//   Lo_l = dt [kappa_l Kv_l/2 - sig_u S ; -kappa_l Kv_l/2]          (6 x 3)
//   Up_l = dt [-kappa_l Kv_l/2 ; kappa_l Kv_l/2 - sig_d S]          (6 x 3)
// Block Thomas: D'_l = D_l^T - Lo_l G_{l-1}[3:6, :] (columns 0..2 only),
// G_l = D'_l^-1 Up_l and y_l = D'_l^-1 (r_l - Lo_l y_{l-1}[3:6]); back
// substitution mu_l = y_l - G_l mu_{l+1}[0:3].  As in the forward solve, G_l
// depends only on the mesh, kappa, dt and the penalty: a sweep without fields
// (NF = 0) keeps it in its own array, each solve's forward sweep recomputes it
// in registers and stores y_l into the output rows, and the back
// substitution reads the kept G_l and overwrites y_l with mu_l.
struct TSolveArgs {
  DevMesh m;
  const double* Z;     // may be the same array as mu
  double* mu;
  const double* kappa;
  double* gfac;        // [18][n_slots]: the kept G_l
  double dt, eta;
};

template <int NF>
__global__ __launch_bounds__(64) void tsolve_kernel(TSolveArgs a) {
  constexpr int kF = NF > 0 ? NF : 1;   // array extent (the factor sweep has no fields)
  const DevMesh& m = a.m;
  const int cell = m.cell_order[blockIdx.x];   // deepest cells first
  const int lane = threadIdx.x;
  const int c = cell * kCell + lane;
  const int N = m.nlay[c];
  if (N == 0) return;
  const size_t SL = (size_t)m.n_slots;
  const size_t p0 = (size_t)m.cell_base[cell] + lane;
  const size_t lt0 = (size_t)m.cell_lbase[cell] + lane;
  const double Jh = m.geo[G_JH * m.n_col_slots + c];
  const double dt = a.dt, eta = a.eta;
  const double* __restrict__ kap = a.kappa;
  double* __restrict__ Gsc = a.gfac;
  const double sd = Jh * (1.0 / 12.0), so = Jh * (1.0 / 24.0);

  // Each layer's loads are issued one layer ahead of their use (the next
  // layer's Z and the geometry two layers down), so that a column's serial
  // sweep does not wait a memory round trip per layer.
  LayerGeo gc, gn, gp;
  load_layer(m, lt0, gc);
  double kvc[6];
  vertical_stiffness(gc, Jh, kvc);
  double Gp[6][3];
  double yp[kF][6];
  double kp = 0.0;
  gp = gc;
  double zc[kF][6];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) zc[f][i] = a.Z[(size_t)(f * 6 + i) * SL + p0];
  double kn = 0.0;
  if (N > 1) {
    load_layer(m, lt0 + (size_t)kCell, gn);
    kn = kap[1];
  }
  for (int l = 0; l < N; ++l) {
    const size_t p = p0 + (size_t)l * kCell;
    const double kc = kap[l];
    const bool below = l < N - 1;
    double zx[kF][6];
    if (below) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) zx[f][i] = a.Z[(size_t)(f * 6 + i) * SL + p + kCell];
    }
    LayerGeo gnn = gn;
    double knn = 0.0;
    if (l + 2 < N) {
      load_layer(m, lt0 + (size_t)(l + 2) * kCell, gnn);
      knn = kap[l + 2];
    }
    double mz[6];
    mass_z(gc, Jh, mz);
    const double sig_u = l > 0 ? penalty(eta, kp, kc, gp.hbar, gc.hbar) : 0.0;
    const double sig_d = below ? penalty(eta, kc, kn, gc.hbar, gn.hbar) : 0.0;
    // forward sub-blocks TT, TB, BT, BB of D_l, then D_l^T = [TT BT; TB BB]
    double d[6][6];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const double mm = mz[sidx(i, j)], kk = dt * kc * kvc[sidx(i, j)], hk = 0.5 * kk;
        const double s_ij = (i == j ? sd : so);
        double TT = (2.0 / 3.0) * mm + kk, TB = (1.0 / 3.0) * mm - kk;
        double BT = (1.0 / 3.0) * mm - kk, BB = (2.0 / 3.0) * mm + kk;
        if (l > 0) {
          TT += -hk + dt * sig_u * s_ij;
          TB += hk;
        }
        if (below) {
          BT += hk;
          BB += -hk + dt * sig_d * s_ij;
        }
        d[i][j] = TT;
        d[i][j + 3] = BT;
        d[i + 3][j] = TB;
        d[i + 3][j + 3] = BB;
      }
    // right-hand sides r = M Z
    double r[kF][6];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double* t = zc[f];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        double at = 0.0, ab = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          at += mz[sidx(i, j)] * t[j];
          ab += mz[sidx(i, j)] * t[j + 3];
        }
        r[f][i] = (2.0 / 3.0) * at + (1.0 / 3.0) * ab;
        r[f][i + 3] = (1.0 / 3.0) * at + (2.0 / 3.0) * ab;
      }
    }
    if (l > 0) {
      double Lo[6][3];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const double hk = 0.5 * dt * kc * kvc[sidx(i, j)];
          Lo[i][j] = hk - dt * sig_u * (i == j ? sd : so);
          Lo[i + 3][j] = -hk;
        }
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          double acc = 0.0;
#pragma unroll
          for (int k = 0; k < 3; ++k) acc += Lo[i][k] * Gp[k + 3][j];
          d[i][j] -= acc;
        }
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          double acc = 0.0;
#pragma unroll
          for (int k = 0; k < 3; ++k) acc += Lo[i][k] * yp[f][k + 3];
          r[f][i] -= acc;
        }
    }
    // LU of d without pivoting
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const double inv = 1.0 / d[k][k];
#pragma unroll
      for (int i = k + 1; i < 6; ++i) {
        const double li = d[i][k] * inv;
        d[i][k] = li;
#pragma unroll
        for (int j = k + 1; j < 6; ++j) d[i][j] -= li * d[k][j];
      }
    }
    // G = d^-1 Up (only needed when there is a layer below)
    double Gc[6][3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      double z[6];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        double hk = 0.5 * dt * kc * kvc[sidx(i, q)];
        z[i] = below ? -hk : 0.0;
        z[i + 3] = below ? hk - dt * sig_d * (i == q ? sd : so) : 0.0;
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        double acc = z[i];
#pragma unroll
        for (int k = 0; k < i; ++k) acc -= d[i][k] * z[k];
        z[i] = acc;
      }
#pragma unroll
      for (int i = 5; i >= 0; --i) {
        double acc = z[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) acc -= d[i][k] * z[k];
        z[i] = acc / d[i][i];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) Gc[i][q] = z[i];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double z[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        double acc = r[f][i];
#pragma unroll
        for (int k = 0; k < i; ++k) acc -= d[i][k] * z[k];
        z[i] = acc;
      }
#pragma unroll
      for (int i = 5; i >= 0; --i) {
        double acc = z[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) acc -= d[i][k] * z[k];
        z[i] = acc / d[i][i];
      }
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        yp[f][i] = z[i];
        a.mu[(size_t)(f * 6 + i) * SL + p] = z[i];   // Z_l has been read: y_l may overwrite it
      }
    }
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        Gp[i][q] = Gc[i][q];
        if (NF == 0) Gsc[(size_t)(i * 3 + q) * SL + p] = Gc[i][q];
      }
    kp = kc;
    gp = gc;
    if (below) {
      gc = gn;
      vertical_stiffness(gc, Jh, kvc);
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) zc[f][i] = zx[f][i];
    }
    gn = gnn;
    kn = knn;
  }
  if (NF == 0) return;
  // back substitution
  double xn[kF][6];
  {
    const size_t p = p0 + (size_t)(N - 1) * kCell;
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        xn[f][i] = yp[f][i];
        a.mu[(size_t)(f * 6 + i) * SL + p] = yp[f][i];
      }
  }
  // G_l and y_l one layer ahead of their use, as in the forward sweep
  double G[6][3], yl[kF][6];
  if (N > 1) {
    const size_t p = p0 + (size_t)(N - 2) * kCell;
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int q = 0; q < 3; ++q) G[i][q] = Gsc[(size_t)(i * 3 + q) * SL + p];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int i = 0; i < 6; ++i) yl[f][i] = a.mu[(size_t)(f * 6 + i) * SL + p];
  }
  for (int l = N - 2; l >= 0; --l) {
    const size_t p = p0 + (size_t)l * kCell;
    double Gx[6][3], yx[kF][6];
    if (l > 0) {
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q) Gx[i][q] = Gsc[(size_t)(i * 3 + q) * SL + p - kCell];
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) yx[f][i] = a.mu[(size_t)(f * 6 + i) * SL + p - kCell];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double xt[3] = {xn[f][0], xn[f][1], xn[f][2]};
#pragma unroll
      for (int i = 0; i < 6; ++i)
        xn[f][i] = yl[f][i] - (G[i][0] * xt[0] + G[i][1] * xt[1] + G[i][2] * xt[2]);
#pragma unroll
      for (int i = 0; i < 6; ++i) a.mu[(size_t)(f * 6 + i) * SL + p] = xn[f][i];
    }
    if (l > 0) {
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q) G[i][q] = Gx[i][q];
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) yl[f][i] = yx[f][i];
    }
  }
}

// ---------------------------------------------------------------------------
// kappa gradient: g_l = sum_f mu_f^T (dA/dkappa_l) x_f per column and layer.
// A depends on kappa_l through the volume term of prism l and, on the faces
// above and below it, through {kappa dT/dz} (kappa/2 per side) and the
// penalty (d sigma / d kappa = s' = eta / (2 min(hbar_up, hbar_dn))).  With
// [v] = v_up,bottom - v_dn,top across a face and S = M_h:
//   volume of l:                -(mu_t - mu_b)^T Kv_l (x_t - x_b)
//   each face touching l:       -[mu]^T (s' S [x] + Kv_l (x_l,t - x_l,b) / 2)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double quad3(const double K[6], const double a[3], const double b[3]) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) s += a[i] * K[sidx(i, j)] * b[j];
  return s;
}

__device__ __forceinline__ double quadS(double sd, double so, const double a[3], const double b[3]) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) s += a[i] * (i == j ? sd : so) * b[j];
  return s;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// One thread per prism over the 2-layer tile table, one wavefront per layer
// of a cell: each prism evaluates every term of its own g (its volume and
// both faces touching it; the penalty of a face is evaluated by the prisms on
// both sides), so no column is walked and the loads of all layers are in
// flight at once.  The 64 columns of a cell are summed with a fixed
// butterfly, cells per layer with a fixed tree (kgrad_reduce_kernel).
struct KGradTileArgs {
  DevMesh m;
  const WgTile* tiles;
  const double* mu;
  const double* x;
  double* partial;   // [max_layers][n_cells]
  double eta;
};

template <int NF>
__global__ __launch_bounds__(128) void kgrad_tile_kernel(KGradTileArgs a) {
  const DevMesh& m = a.m;
  const WgTile tile = a.tiles[blockIdx.x];
  const int lane = threadIdx.x & (kCell - 1);
  const int l = tile.layer0 + (threadIdx.x >> 6);
  const int cell = tile.cell;
  const int depth = (m.cell_base[cell + 1] - m.cell_base[cell]) / kCell;
  if (l >= depth) return;                      // uniform per wavefront
  const int c = cell * kCell + lane;
  const int N = m.nlay[c];
  const bool live = l < N;
  const bool up = live && l > 0, dn = live && l + 1 < N;
  const size_t SL = (size_t)m.n_slots;
  const size_t p = (size_t)m.cell_base[cell] + (size_t)l * kCell + lane;
  const size_t pu = up ? p - kCell : p, pd = dn ? p + kCell : p;
  const size_t lt = (size_t)m.cell_lbase[cell] + (size_t)l * kCell + lane;
  double g = 0.0;
  if (live) {
    const double Jh = m.geo[G_JH * m.n_col_slots + c];
    const double sd = Jh * (1.0 / 12.0), so = Jh * (1.0 / 24.0);
    LayerGeo gl, gu, gd;
    load_layer(m, lt, gl);
    load_layer(m, up ? lt - kCell : lt, gu);
    load_layer(m, dn ? lt + kCell : lt, gd);
    double kv[6];
    vertical_stiffness(gl, Jh, kv);
    const double spu = up ? a.eta / (2.0 * fmin(gu.hbar, gl.hbar)) : 0.0;
    const double spd = dn ? a.eta / (2.0 * fmin(gl.hbar, gd.hbar)) : 0.0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      double mt[3], mb[3], xt[3], xb[3], dm[3], dx[3];
      double mub[3], xub[3], mdt[3], xdt[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const size_t rt = (size_t)(f * 6 + i) * SL, rb = (size_t)(f * 6 + i + 3) * SL;
        mt[i] = a.mu[rt + p];
        mb[i] = a.mu[rb + p];
        xt[i] = a.x[rt + p];
        xb[i] = a.x[rb + p];
        mub[i] = a.mu[rb + pu];
        xub[i] = a.x[rb + pu];
        mdt[i] = a.mu[rt + pd];
        xdt[i] = a.x[rt + pd];
        dm[i] = mt[i] - mb[i];
        dx[i] = xt[i] - xb[i];
      }
      g -= quad3(kv, dm, dx);
      if (up) {                                 // the face above: kappa_l below it
        double jm[3], jx[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          jm[i] = mub[i] - mt[i];
          jx[i] = xub[i] - xt[i];
        }
        g -= quadS(spu * sd, spu * so, jm, jx) + 0.5 * quad3(kv, jm, dx);
      }
      if (dn) {                                 // the face below: kappa_l above it
        double jm[3], jx[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          jm[i] = mb[i] - mdt[i];
          jx[i] = xb[i] - xdt[i];
        }
        g -= quadS(spd * sd, spd * so, jm, jx) + 0.5 * quad3(kv, jm, dx);
      }
    }
  }
  const double v = wave_sum(g);
  if (lane == 0) a.partial[(size_t)l * m.n_cells + cell] = v;
}

// dkappa[l] += dt * sum over cells deeper than l of partial[l][cell]
__global__ __launch_bounds__(256) void kgrad_reduce_kernel(DevMesh m, const double* partial, double dt,
                                                            double* dkappa) {
  const int l = blockIdx.x;
  __shared__ double red[256];
  double acc = 0.0;
  for (int k = threadIdx.x; k < m.n_cells; k += 256) {
    const int depth = (m.cell_base[k + 1] - m.cell_base[k]) / kCell;
    if (l < depth) acc += partial[(size_t)l * m.n_cells + k];
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) dkappa[l] += dt * red[0];
}

// ---------------------------------------------------------------------------
// Mass operator: Y = M X or M^-1 X per prism; column partials of X^T M Y.
// ---------------------------------------------------------------------------
// One thread per prism, four layers of a cell a block: a walk down each column by one
// thread left the launch at a few wavefronts per CU with one layer's loads in flight
// (whole call, new result included: 2 fields of 55 k prisms 16.6 -> 11.4 us, float 2
// fields of 0.71 M 46 -> 22, 4 fields of 2.6 M ragged prisms 419 -> 350).  Shallower
// meshes take a block of as many wavefronts as they have layers (180,000 columns of one
// layer, 4 fields: 13.5 us with four, 13.1 with one).
constexpr int kMassLayers = 4;
template <typename R>
__global__ __launch_bounds__(kCell * kMassLayers) void mass_apply_kernel(DevMesh m, const R* X, R* Y, int nf,
                                                                         int inverse) {
  const int cell = blockIdx.x;
  const int lane = threadIdx.x % kCell;
  const int l = (blockIdx.y * blockDim.x + threadIdx.x) / kCell;
  const int c = cell * kCell + lane;
  if (l >= m.nlay[c]) return;
  const size_t SL = (size_t)m.n_slots;
  const double Jh = m.geo[G_JH * m.n_col_slots + c];
  const size_t p = (size_t)m.cell_base[cell] + (size_t)l * kCell + lane;
  LayerGeo g;
  load_layer(m, (size_t)m.cell_lbase[cell] + (size_t)l * kCell + lane, g);
  double mz[6];
  mass_z(g, Jh, mz);
  double inv[6];
  if (inverse) {
    const double c00 = mz[1] * mz[2] - mz[5] * mz[5], c01 = mz[4] * mz[5] - mz[3] * mz[2];
    const double c02 = mz[3] * mz[5] - mz[4] * mz[1], c11 = mz[0] * mz[2] - mz[4] * mz[4];
    const double c12 = mz[3] * mz[4] - mz[0] * mz[5], c22 = mz[0] * mz[1] - mz[3] * mz[3];
    const double det = mz[0] * c00 + mz[3] * c01 + mz[4] * c02;
    inv[0] = c00 / det; inv[1] = c11 / det; inv[2] = c22 / det;
    inv[3] = c01 / det; inv[4] = c02 / det; inv[5] = c12 / det;
  }
  for (int f = 0; f < nf; ++f) {
    double t[6], o[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) t[i] = (double)X[(size_t)(f * 6 + i) * SL + p];
    // M = [2 1; 1 2]/3 (x) Mz, M^-1 = [2 -1; -1 2] (x) Mz^-1
    double ht[3], hb[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ht[i] = inverse ? 2.0 * t[i] - t[i + 3] : (2.0 * t[i] + t[i + 3]) * (1.0 / 3.0);
      hb[i] = inverse ? 2.0 * t[i + 3] - t[i] : (t[i] + 2.0 * t[i + 3]) * (1.0 / 3.0);
    }
    const double* K = inverse ? inv : mz;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      o[i] = K[sidx(i, 0)] * ht[0] + K[sidx(i, 1)] * ht[1] + K[sidx(i, 2)] * ht[2];
      o[i + 3] = K[sidx(i, 0)] * hb[0] + K[sidx(i, 1)] * hb[1] + K[sidx(i, 2)] * hb[2];
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) Y[(size_t)(f * 6 + i) * SL + p] = (R)o[i];
  }
}

// Per column and field X^T M Y.  A block of column_waves() wavefronts takes a cell; wave
// k adds the layers k, k + waves, ... in this order, and the waves' sums are added in
// theirs, so the result is the same on every call (whole call, one thread per column ->
// now: 1 field of 1.0 M prisms 100 -> 47 us, 4 fields of 6.0 M 491 -> 331).
template <typename R>
__global__ __launch_bounds__(kCell * kColumnWaves) void mdot_column_kernel(DevMesh m, const R* X, const R* Y, int nf,
                                                                           double* out) {
  __shared__ double part[kColumnWaves][kMaxFields][kCell];
  const int cell = blockIdx.x;
  const int lane = threadIdx.x % kCell, wave = threadIdx.x / kCell, waves = blockDim.x / kCell;
  const int c = cell * kCell + lane;
  const int N = m.nlay[c];
  const int CS = m.n_col_slots;
  const size_t SL = (size_t)m.n_slots;
  double acc[kMaxFields] = {0.0, 0.0, 0.0, 0.0};
  const double Jh = m.geo[G_JH * CS + c];
  for (int l = wave; l < N; l += waves) {
    const size_t p = (size_t)m.cell_base[cell] + (size_t)l * kCell + lane;
    LayerGeo g;
    load_layer(m, (size_t)m.cell_lbase[cell] + (size_t)l * kCell + lane, g);
    double mz[6];
    mass_z(g, Jh, mz);
    for (int f = 0; f < nf; ++f) {
      double x[6], y[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        x[i] = (double)X[(size_t)(f * 6 + i) * SL + p];
        y[i] = (double)Y[(size_t)(f * 6 + i) * SL + p];
      }
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const double mm = mz[sidx(i, j)];
          s += mm * ((2.0 / 3.0) * (x[i] * y[j] + x[i + 3] * y[j + 3]) +
                     (1.0 / 3.0) * (x[i] * y[j + 3] + x[i + 3] * y[j]));
        }
      acc[f] += s;
    }
  }
#pragma unroll
  for (int f = 0; f < kMaxFields; ++f) part[wave][f][lane] = acc[f];
  __syncthreads();
  // wave f adds field f
  if (wave < nf) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kColumnWaves; ++k) s += k < waves ? part[k][wave][lane] : 0.0;
    out[(size_t)wave * CS + c] = s;
  }
}

template <int NF>
hipError_t launch_adj_stage_nf(const AdjStageArgs& a, bool w_zero, int tile_layers, int n_cu, hipStream_t s) {
  // no wavefronts for layers that no cell has, as in the forward stages
  const int layers = tile_layers < a.m.max_layers ? tile_layers : a.m.max_layers;
  const dim3 grid(a.n_tiles), block(kCell * layers);
  // more than 16 wavefronts per CU, with four fields 28: neighbours in the cell through
  // LDS.  Reverse step (three of these kernels and a solve), 1 to 4 fields, without ->
  // with LDS:
  //    1469 wavefronts   46.5  59.1  80.8  93.5 ->  44.3  57.7  74.3  95.6 us
  //    3000              75.2  97.0   136   160 ->  73.7  98.2   131   170
  //    4140              91.1   121   165   200 ->  87.8   119   161   213
  //    6210               125   167   239   312 ->   120   164   240   319
  //    8100               151   204   342   429 ->   143   205   302   420
  //   15602               317   492     -   851 ->   288   437     -   808
  constexpr int kLine = NF == 4 ? 28 : 16;
  if ((int64_t)a.n_tiles * layers > kLine * (int64_t)n_cu) {
    const size_t lds = block.x * kAdjRows<NF> * sizeof(double);
    if (w_zero) hipLaunchKernelGGL((adj_stage_kernel<NF, true, true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((adj_stage_kernel<NF, false, true>), grid, block, lds, s, a);
  } else {
    if (w_zero) hipLaunchKernelGGL((adj_stage_kernel<NF, true, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((adj_stage_kernel<NF, false, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint_stage(const DevMesh& m, const WgTile* tiles, int n_tiles, int tile_layers, int xcd,
                                int n_cu, int n_fields, bool w_zero, const double* Y, const double* X1, const double* X2,
                                double* out, const double* U, double dt, double b, double a1, double a2,
                                hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  AdjStageArgs a{};
  a.m = m;
  a.tiles = tiles;
  a.n_tiles = n_tiles;
  a.xcd = xcd;
  a.Y = Y;
  a.X1 = X1;
  a.X2 = X2;
  a.out = out;
  a.U = U;
  a.dt = dt;
  a.b = b;
  a.a1 = a1;
  a.a2 = a2;
  switch (n_fields) {
    case 1: return launch_adj_stage_nf<1>(a, w_zero, tile_layers, n_cu, s);
    case 2: return launch_adj_stage_nf<2>(a, w_zero, tile_layers, n_cu, s);
    case 3: return launch_adj_stage_nf<3>(a, w_zero, tile_layers, n_cu, s);
    case 4: return launch_adj_stage_nf<4>(a, w_zero, tile_layers, n_cu, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tsolve(const DevMesh& m, int n_fields, const double* Z, double* mu, const double* kappa,
                         double* gfac, double dt, double eta, bool factor, hipStream_t s) {
  if (m.n_cells == 0) return hipSuccess;
  TSolveArgs a{};
  a.m = m;
  a.Z = Z;
  a.mu = mu;
  a.kappa = kappa;
  a.gfac = gfac;
  a.dt = dt;
  a.eta = eta;
  dim3 grid(m.n_cells), block(kCell);
  if (factor) {
    hipLaunchKernelGGL((tsolve_kernel<0>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  switch (n_fields) {
    case 1: hipLaunchKernelGGL((tsolve_kernel<1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((tsolve_kernel<2>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((tsolve_kernel<3>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((tsolve_kernel<4>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_kappa_gradient(const DevMesh& m, const WgTile* tiles2, int n_tiles2, int n_fields,
                                 const double* mu, const double* x, double* partial, double eta, double dt,
                                 double* dkappa, hipStream_t s) {
  if (m.n_cells == 0) return hipSuccess;
  KGradTileArgs a{};
  a.m = m;
  a.tiles = tiles2;
  a.mu = mu;
  a.x = x;
  a.partial = partial;
  a.eta = eta;
  const dim3 grid(n_tiles2), block(2 * kCell);
  switch (n_fields) {
    case 1: hipLaunchKernelGGL((kgrad_tile_kernel<1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((kgrad_tile_kernel<2>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((kgrad_tile_kernel<3>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((kgrad_tile_kernel<4>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kgrad_reduce_kernel, dim3(m.max_layers), dim3(256), 0, s, m, partial, dt, dkappa);
  return hipGetLastError();
}

hipError_t launch_mass_apply(const DevMesh& m, const void* X, void* Y, int n_fields, bool fp32, bool inverse,
                             hipStream_t s) {
  const int rows = m.max_layers < kMassLayers ? m.max_layers : kMassLayers;
  const dim3 grid(m.n_cells, (m.max_layers + rows - 1) / rows), block(kCell * rows);
  if (fp32)
    hipLaunchKernelGGL(mass_apply_kernel<float>, grid, block, 0, s, m,
                       static_cast<const float*>(X), static_cast<float*>(Y), n_fields, (int)inverse);
  else
    hipLaunchKernelGGL(mass_apply_kernel<double>, grid, block, 0, s, m,
                       static_cast<const double*>(X), static_cast<double*>(Y), n_fields, (int)inverse);
  return hipGetLastError();
}

hipError_t launch_mdot_columns(const DevMesh& m, const void* X, const void* Y, int n_fields, bool fp32,
                               double* col_out, hipStream_t s) {
  if (fp32)
    hipLaunchKernelGGL(mdot_column_kernel<float>, dim3(m.n_cells), dim3(kCell * column_waves(m, n_fields)), 0, s, m,
                       static_cast<const float*>(X), static_cast<const float*>(Y), n_fields, col_out);
  else
    hipLaunchKernelGGL(mdot_column_kernel<double>, dim3(m.n_cells), dim3(kCell * column_waves(m, n_fields)), 0, s, m,
                       static_cast<const double*>(X), static_cast<const double*>(Y), n_fields, col_out);
  return hipGetLastError();
}

}  // namespace sdg
