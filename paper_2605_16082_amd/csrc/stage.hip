// Explicit DG operator and SSP-RK3 stage on extruded linear prisms.
//
// Per prism and field:
//
//   R_i = int_K T U.grad(phi_i) dV - sum_faces int_f phi_i Fhat dS
//   L   = M^-1 R                          (block-diagonal mass matrix)
//   out = a Tn + b (Ts + dt L)            (SSP-RK3, Shu-Osher form)
//
// with the quadrature that defines the operator: 6-point degree-4 triangle
// rule x 2-point Gauss in zeta for the volume and horizontal faces, 3-point
// Gauss along edges x 2-point in zeta for lateral faces; upwind flux per
// quadrature point, Fhat dS = max(u_n dS, 0) T_in + min(u_n dS, 0) T_out
// with u_n the average of the two velocity traces.
//
// The volume term uses contravariant fluxes: with alpha = y_eta u - x_eta v
// and beta = x_xi v - y_xi u, the integrand T U.(|J| grad phi_i) equals
// T (dphi_i/dxi z_zeta alpha + dphi_i/deta z_zeta beta
//    + dphi_i/dzeta (J_h w - z_xi alpha - z_eta beta)),
// so the geometric work is shared by all fields.  The mass matrix of a prism
// is H (x) Mz with H = [2 1; 1 2]/3 and Mz_ab = J_h int lambda_a lambda_b
// z_zeta, so M^-1 = [2 -1; -1 2] (x) Mz^-1 and only a symmetric 3x3 inverse
// is needed.
//
// Two kernels compute the same arithmetic (bitwise: they share every device
// function below and accumulate in the same order):
//
//  * stage_kernel: one thread per prism; a workgroup covers 1, 2 or 4 layers
//    of one cell of 64 columns (one wavefront per layer), so each wavefront
//    reads 64 consecutive slots of every nodal array (the paper's section
//    2.1.1 cell layout, with wavefront-sized cells).  No load depends on
//    control flow: lanes past their column's depth compute on in-bounds
//    padding slots and skip the store, and faces without a neighbour address
//    the prism's own nodes and select the exterior value.
//    On launches of more than one wavefront per SIMD each wavefront reads its
//    neighbours in the cell from its layer's rows in LDS.
//
//  * walk_kernel: one wavefront walks down a segment of a cell's layers.
//    The next layer's stage input, velocity, bottom level heights (and Tn,
//    where it fits) are copied global -> LDS by the wavefront's own 16-byte
//    direct loads while the current layer computes, so the HBM latency of
//    the streamed data is hidden by the pipeline rather than by occupancy,
//    and the loads take no registers.  The horizontal face between layers l
//    and l+1 is computed once and its contribution to layer l+1's top nodes
//    carried in registers.  Lateral neighbours are read from L2.
#include <atomic>

#include "internal.h"
#include "quadrature.h"

// Multiply-adds are fused only within one expression, never across
// statements, so the shared device functions below round the same way in
// both kernels whatever the surrounding code.
#pragma clang fp contract(on)

namespace sdg {
namespace {

template <typename R> __device__ __forceinline__ const R* geo_of(const DevMesh& m);
template <> __device__ __forceinline__ const double* geo_of<double>(const DevMesh& m) { return m.geo; }
template <> __device__ __forceinline__ const float* geo_of<float>(const DevMesh& m) { return m.geo32; }
template <typename R> __device__ __forceinline__ const R* zl_of(const DevMesh& m);
template <> __device__ __forceinline__ const double* zl_of<double>(const DevMesh& m) { return m.zl; }
template <> __device__ __forceinline__ const float* zl_of<float>(const DevMesh& m) { return m.zl32; }

// Load from a row whose base pointer is wavefront-uniform, at a 32-bit byte
// offset: lets the compiler use the scalar-base + vector-offset load form
// instead of per-lane 64-bit address arithmetic.
template <typename T>
__device__ __forceinline__ T ldb(const T* __restrict__ row, uint32_t byte_off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(row) + byte_off);
}
template <typename T>
__device__ __forceinline__ void stb(T* __restrict__ row, uint32_t byte_off, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(row) + byte_off) = v;
}
// Row r of a [..][6][S] nodal array at byte offset off: the address is the base of
// the row's 6-row block plus a 32-bit offset (r mod 6) S + off, so there is one
// uniform base per block instead of one per row; the kernels keep far fewer 64-bit
// row addresses in scalar registers, which they otherwise spill to vector lanes
// (double stages 2% faster; the float walk of 4 fields executes 5% fewer
// instructions).  A 6-row block is below 4 GiB (checked at mesh upload).
template <typename T>
__device__ __forceinline__ T ldr(const T* __restrict__ arr, size_t S, int r, uint32_t off) {
  return ldb(arr + (size_t)(r / 6 * 6) * S, (uint32_t)(r % 6) * (uint32_t)(S * sizeof(T)) + off);
}
template <typename T>
__device__ __forceinline__ void str(T* __restrict__ arr, size_t S, int r, uint32_t off, T v) {
  stb(arr + (size_t)(r / 6 * 6) * S, (uint32_t)(r % 6) * (uint32_t)(S * sizeof(T)) + off, v);
}

template <typename R>
__device__ __forceinline__ R upos(R x) { return x > R(0) ? x : R(0); }
template <typename R>
__device__ __forceinline__ R uneg(R x) { return x < R(0) ? x : R(0); }

// Per-column map derivatives and J_h = 2 area.
template <typename R>
struct ColGeo {
  R xxi, xet, yxi, yet, Jh;
};

template <typename R>
__device__ __forceinline__ ColGeo<R> load_colgeo(const DevMesh& m, uint32_t co) {
  const R* __restrict__ geo = geo_of<R>(m);
  const int CS = m.n_col_slots;
  ColGeo<R> g;
  g.xxi = ldb(geo + G_XXI * CS, co);
  g.xet = ldb(geo + G_XET * CS, co);
  g.yxi = ldb(geo + G_YXI * CS, co);
  g.yet = ldb(geo + G_YET * CS, co);
  g.Jh = ldb(geo + G_JH * CS, co);
  return g;
}

// ===========================================================================
// Term by term, all fields: a prism's residuals res[NF][6] are carried through
// the volume term, the lateral faces 0, 1, 2, the top and the bottom face, in
// this order.  Of the field-independent factors only one term's are live at a
// time, and each term's end is a point that the compiler may not reorder over
// (formed); the one-thread-per-prism kernel requests a term's neighbour values
// one term ahead.  What bounds the kernels is the latency of their loads at the
// one to three wavefronts per SIMD that their registers allow.  Before, all
// factors were formed first, the fields went one at a time, and the compiler
// placed the loads; registers of the third stage before and after: FP64 2 fields
// 304 -> 237 (one thread per prism: two wavefronts for one), FP32 2 fields
// 184 -> 142 (three for two), FP64 column walk of 4 fields 462 -> 413.  Third
// stage of sigma-grid boxes, 64 columns a cell, before and after:
//   one thread per prism  FP64 4 fields, 6.0 M prisms   1.87 -> 1.49 ms
//                         FP64 3 fields with w, 0.35 M  82   -> 66 us
//                         FP32 2 fields, 0.71 M         56   -> 47 us
//                         FP64 1 field, 1.0 M           100  -> 97 us
//   column walk, 12       FP64 4 fields, 6.0 M prisms   1.20 -> 1.14 ms
//                         FP64 4 fields, 2.6 M          546  -> 506 us
//                         FP32 4 fields, 6.0 M          0.64 -> 0.64 ms
// own(f, i) gives the prism's nodal value i of field f.
// ===========================================================================

// No instruction moves across this point.
__device__ __forceinline__ void phase() { __builtin_amdgcn_sched_barrier(0); }

// The residuals are formed up to here: without it the compiler sinks the whole
// arithmetic of a prism into the branch around its stores, behind all of its
// loads, whose values then all wait in registers.
template <typename R, int NF>
__device__ __forceinline__ void formed(R (&res)[NF][6]) {
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) asm volatile("" : "+v"(res[f][i]));
  phase();
}

// Volume term: with alpha = y_eta u - x_eta v, beta = x_xi v - y_xi u at
// volume point (k, q), each field takes, with ta_k its three nodal values
// interpolated to zeta_k, ta_k . Px_k, ta_k . Pe_k and G_k ta_k, where
//   Px_k[a] = sum_q w_q lambda_a z_zeta alpha,  Pe_k[a] = sum_q w_q lambda_a z_zeta beta,
//   G_k[n][a] = sum_q w_q lambda_n lambda_a (J_h w - z_xi alpha - z_eta beta).
// z_zeta, alpha, beta and the bracket are linear over the triangle and the
// degree-4 rule is exact on the cubics, so with nodal values x_b, y_c
//   sum_q w_q lambda_a x y = (X Y + x_a Y + X y_a + x.y + 2 x_a y_a) / 120
// (X, Y the sums over the nodes), and the same with x = lambda_n: about 150
// multiply-adds for both k where the sums over the points take 400.
template <typename R, int NF, bool WZ, typename Own>
__device__ __forceinline__ void volume_term(const ColGeo<R>& g, const R zt[3], const R zb[3], const R dz[3],
                                            const R u[6], const R v[6], const R w[6], Own own, R (&res)[NF][6]) {
  const R xxi = g.xxi, xet = g.xet, yxi = g.yxi, yet = g.yet, Jh = g.Jh;
  R Px[2][3], Pe[2][3], G[2][6];   // G: symmetric 3x3, entries 00 11 22 01 02 12
  const R zs = dz[0] + dz[1] + dz[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const R tk = R(kZt[k]), bk = R(kZb[k]);
    const R z_xi = tk * (zt[1] - zt[0]) + bk * (zb[1] - zb[0]);
    const R z_et = tk * (zt[2] - zt[0]) + bk * (zb[2] - zb[0]);
    R al[3], be[3], c[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      const R ua = tk * u[n] + bk * u[n + 3];
      const R va = tk * v[n] + bk * v[n + 3];
      al[n] = yet * ua - xet * va;
      be[n] = xxi * va - yxi * ua;
      R x = -(z_xi * al[n] + z_et * be[n]);
      if (!WZ) x += Jh * (tk * w[n] + bk * w[n + 3]);
      c[n] = R(1.0 / 120.0) * x;
    }
    const R as = al[0] + al[1] + al[2], bs = be[0] + be[1] + be[2], cs = c[0] + c[1] + c[2];
    const R ax = zs * as + (dz[0] * al[0] + dz[1] * al[1] + dz[2] * al[2]);
    const R bx = zs * bs + (dz[0] * be[0] + dz[1] * be[1] + dz[2] * be[2]);
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      Px[k][n] = R(1.0 / 240.0) * (ax + zs * al[n] + dz[n] * (as + R(2) * al[n]));
      Pe[k][n] = R(1.0 / 240.0) * (bx + zs * be[n] + dz[n] * (bs + R(2) * be[n]));
      G[k][n] = R(2) * cs + R(4) * c[n];
    }
    G[k][3] = cs + c[0] + c[1];
    G[k][4] = cs + c[0] + c[2];
    G[k][5] = cs + c[1] + c[2];
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    R sx[2], se[2], sz[3];
    R T[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) T[i] = own(f, i);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const R tk = R(kZt[k]), bk = R(kZb[k]);
      R ta[3];
#pragma unroll
      for (int n = 0; n < 3; ++n) ta[n] = tk * T[n] + bk * T[n + 3];
      sx[k] = ta[0] * Px[k][0] + ta[1] * Px[k][1] + ta[2] * Px[k][2];
      se[k] = ta[0] * Pe[k][0] + ta[1] * Pe[k][1] + ta[2] * Pe[k][2];
      const R g[3][3] = {{G[k][0], G[k][3], G[k][4]}, {G[k][3], G[k][1], G[k][5]}, {G[k][4], G[k][5], G[k][2]}};
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        if (k == 0)
          sz[n] = g[n][0] * ta[0];
        else
          sz[n] += g[n][0] * ta[0];
        sz[n] += g[n][1] * ta[1];
        sz[n] += g[n][2] * ta[2];
      }
    }
    // dphi/dxi = dlambda/dxi * (t or b), dphi/dzeta = +-lambda/2
    const R sxt = R(kZt[0]) * sx[0] + R(kZt[1]) * sx[1];
    const R sxb = R(kZb[0]) * sx[0] + R(kZb[1]) * sx[1];
    const R set = R(kZt[0]) * se[0] + R(kZt[1]) * se[1];
    const R seb = R(kZb[0]) * se[0] + R(kZb[1]) * se[1];
    res[f][0] = -sxt - set + R(0.5) * sz[0];
    res[f][1] = sxt + R(0.5) * sz[1];
    res[f][2] = set + R(0.5) * sz[2];
    res[f][3] = -sxb - seb - R(0.5) * sz[0];
    res[f][4] = sxb - R(0.5) * sz[1];
    res[f][5] = seb - R(0.5) * sz[2];
  }
}

// Lateral face e (edge A = e -> B = e+1) of a column: neighbour slot and
// edge, outward normal and length (the same for every layer).
template <typename R>
struct LatMeta {
  int nslot, meta;
  R nx, ny, Le;
};

template <typename R>
__device__ __forceinline__ void lat_meta(const DevMesh& m, int e, uint32_t co, LatMeta<R>& M) {
  const int CS = m.n_col_slots;
  const uint32_t co4 = co / (uint32_t)sizeof(R) * 4u;
  const R* __restrict__ geo = geo_of<R>(m);
  M.nslot = ldb(m.nbr_slot + e * CS, co4);
  M.meta = ldb(m.nbr_meta + e * CS, co4);
  M.nx = ldb(geo + (G_NX + e) * CS, co);
  M.ny = ldb(geo + (G_NY + e) * CS, co);
  M.Le = ldb(geo + (G_LE + e) * CS, co);
}

// At layer l (prism byte offset po): the byte offsets (within a field block)
// of the neighbour's face nodes A top, B top, A bottom, B bottom, and its
// velocity there.  A wall (neighbour shallower than l) or an open boundary
// has no live neighbour: the offsets then point at the prism's own nodes
// (in bounds, unused) so the loads need no branch.
template <typename R>
struct LatNb {
  uint32_t no[4];
  R uo[4], vo[4];
  bool lds;          // no[] are offsets into the layer's rows in LDS (the neighbour is in the cell)
};

template <typename R>
__device__ __forceinline__ void lat_nb(const StageArgs& a, const LatMeta<R>& M, int e, int l, uint32_t po,
                                       LatNb<R>& nb) {
  const size_t S = (size_t)a.m.n_slots;
  const uint32_t rs = (uint32_t)(S * sizeof(R));     // bytes per node row
  const R* __restrict__ U = static_cast<const R*>(a.U);
  const int A = e, B = (e + 1) % 3;
  const bool live = M.nslot >= 0 && l < (M.meta >> 2);
  const int kp = M.meta & 3;
  const uint32_t nA = live ? (uint32_t)((kp + 1) % 3) : (uint32_t)A;
  const uint32_t nB = live ? (uint32_t)kp : (uint32_t)B;
  const uint32_t pno = live ? ((uint32_t)M.nslot + (uint32_t)l * kCell) * (uint32_t)sizeof(R) : po;
  nb.no[0] = nA * rs + pno;
  nb.no[1] = nB * rs + pno;
  nb.no[2] = nb.no[0] + 3u * rs;
  nb.no[3] = nb.no[1] + 3u * rs;
  nb.lds = false;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    nb.uo[j] = ldb(U, nb.no[j]);
    nb.vo[j] = ldb(U + 6 * S, nb.no[j]);
  }
}

template <typename R>
__device__ __forceinline__ R lds_at(const R* slot, uint32_t byte_off) {
  return *reinterpret_cast<const R*>(reinterpret_cast<const char*>(slot) + byte_off);
}

// Keeps later LDS reads below a just-issued copy or store (compiler barrier only).
__device__ __forceinline__ void mem_order() { asm volatile("" ::: "memory"); }

// The request of the one-thread-per-prism kernel: the neighbour's velocity and stage
// input, ahead of their use.  With SH a neighbour in the cell is not requested: the
// wavefront holds its layer's rows of all 64 columns in LDS (stage input from row 0,
// u from row 6 NF, v after it), and lat_resolve reads them from there at the time of
// their use.  A face without a live neighbour then points at the own rows.
template <typename R, int NF, bool SH>
__device__ __forceinline__ void lat_request(const StageArgs& a, const LatMeta<R>& M, int e, int l, uint32_t po,
                                            int lane, uint32_t cell_base, LatNb<R>& nb, R (&to)[NF][4]) {
  const size_t S = (size_t)a.m.n_slots;
  const R* __restrict__ Ts = static_cast<const R*>(a.Ts);
  if constexpr (!SH) {
    lat_nb<R>(a, M, e, l, po, nb);
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) to[f][j] = ldb(Ts + (size_t)(f * 6) * S, nb.no[j]);
  } else {
    const bool live = M.nslot >= 0 && l < (M.meta >> 2);
    const int kp = M.meta & 3;
    const uint32_t nl = (uint32_t)M.nslot - cell_base;   // < 64 iff the neighbour is in this cell
    nb.lds = !live || nl < (uint32_t)kCell;
    const uint32_t nA = live ? (uint32_t)((kp + 1) % 3) : (uint32_t)e;
    const uint32_t nB = live ? (uint32_t)kp : (uint32_t)((e + 1) % 3);
    const uint32_t src = live && nb.lds ? nl : (uint32_t)lane;
    constexpr uint32_t row = kCell * sizeof(R);
    nb.no[0] = nA * row + src * (uint32_t)sizeof(R);
    nb.no[1] = nB * row + src * (uint32_t)sizeof(R);
    nb.no[2] = nb.no[0] + 3u * row;
    nb.no[3] = nb.no[1] + 3u * row;
    if (!nb.lds) {
      const uint32_t rs = (uint32_t)(S * sizeof(R));     // bytes per node row
      const R* __restrict__ U = static_cast<const R*>(a.U);
      const uint32_t pno = ((uint32_t)M.nslot + (uint32_t)l * kCell) * (uint32_t)sizeof(R);
      const uint32_t go[4] = {nA * rs + pno, nB * rs + pno, (nA + 3u) * rs + pno, (nB + 3u) * rs + pno};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        nb.uo[j] = ldb(U, go[j]);
        nb.vo[j] = ldb(U + 6 * S, go[j]);
      }
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) to[f][j] = ldb(Ts + (size_t)(f * 6) * S, go[j]);
    }
  }
}

template <typename R, int NF>
__device__ __forceinline__ void lat_resolve(const R* sh, LatNb<R>& nb, R (&to)[NF][4]) {
  constexpr uint32_t row = kCell * sizeof(R);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const R x = lds_at(sh, 6 * NF * row + nb.no[j]), y = lds_at(sh, (6 * NF + 6) * row + nb.no[j]);
    nb.uo[j] = nb.lds ? x : nb.uo[j];
    nb.vo[j] = nb.lds ? y : nb.vo[j];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const R t = lds_at(sh, f * 6 * row + nb.no[j]);
      to[f][j] = nb.lds ? t : to[f][j];
    }
  }
}

// Face weights q = u_n dS at the 3 x 2 face points (edge point j, zeta_k), u_n
// the normal component of the average of the two velocity traces (a wall
// carries no flux): the flux is q times the inner trace where q > 0, else the
// outer one.
template <typename R>
struct LatQ {
  R q[3][2];
};

template <typename R>
__device__ __forceinline__ void lat_weights(const LatMeta<R>& M, const LatNb<R>& nb, int e, int l, const R dz[3],
                                            const R u[6], const R v[6], LatQ<R>& F) {
  const int A = e, B = (e + 1) % 3;
  const bool interior = M.nslot >= 0;
  const bool wall = interior && l >= (M.meta >> 2);
  const bool live = interior && !wall;
  const R nx = M.nx, ny = M.ny;
  const R Le = wall ? R(0) : M.Le;
  R un[4] = {nx * u[A] + ny * v[A], nx * u[B] + ny * v[B], nx * u[A + 3] + ny * v[A + 3],
             nx * u[B + 3] + ny * v[B + 3]};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const R avg = R(0.5) * (un[j] + nx * nb.uo[j] + ny * nb.vo[j]);
    un[j] = live ? avg : un[j];
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const R s = R(kS[j]), s1 = R(1) - R(kS[j]);
    const R dS = R(kSw[j]) * Le * R(0.5) * (s1 * dz[A] + s * dz[B]);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const R tk = R(kZt[k]), bk = R(kZb[k]);
      F.q[j][k] = (s1 * (tk * un[0] + bk * un[2]) + s * (tk * un[1] + bk * un[3])) * dS;
    }
  }
}

// The neighbour's face-node value (stage input), or the exterior value on an
// open boundary.
template <typename R>
__device__ __forceinline__ R lat_trace(const StageArgs& a, const LatMeta<R>& M, int f, R x) {
  return M.nslot >= 0 ? x : R(a.t_ext[f]);
}

// res[f][i] -= int_face phi_i Fhat dS of all fields; to[f]: the outer traces.
// In float with two fields or more the sums over the points are contracted
// first, for inflow and outflow, over zeta then along the edge, into the 4 x 4
// matrices of the face nodes (9 distinct entries each), so a field takes 32
// multiply-adds instead of about 80.  In double that is 2% faster for four
// fields too, but the point form picks the upwind trace by the sign of q, and
// so keeps a non-finite value out of the prisms upwind of it.
template <typename R, int NF, typename Own>
__device__ __forceinline__ void lat_apply(int e, const LatQ<R>& F, Own own, const R (&to)[NF][4], R (&res)[NF][6]) {
  const int A = e, B = (e + 1) % 3;
  if constexpr (NF == 1 || sizeof(R) == 8) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const R TA = own(f, A), TB = own(f, B), TA3 = own(f, A + 3), TB3 = own(f, B + 3);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const R s = R(kS[j]), s1 = R(1) - R(kS[j]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const R tk = R(kZt[k]), bk = R(kZb[k]);
          const R ti = s1 * (tk * TA + bk * TA3) + s * (tk * TB + bk * TB3);
          const R tq = s1 * (tk * to[f][0] + bk * to[f][2]) + s * (tk * to[f][1] + bk * to[f][3]);
          const R fl = F.q[j][k] * (F.q[j][k] > R(0) ? ti : tq);
          res[f][A] -= s1 * tk * fl;
          res[f][B] -= s * tk * fl;
          res[f][A + 3] -= s1 * bk * fl;
          res[f][B + 3] -= s * bk * fl;
        }
      }
    }
  } else {
    // K[x][y]: x = AA, AB, BB along the edge, y = top-top, top-bottom, bottom-bottom
    R Kp[3][3], Km[3][3];
    R gp[3][3], gm[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const R p0 = upos(F.q[j][0]), p1 = upos(F.q[j][1]), m0 = uneg(F.q[j][0]), m1 = uneg(F.q[j][1]);
      gp[j][0] = R(kZt[0] * kZt[0]) * p0 + R(kZt[1] * kZt[1]) * p1;
      gp[j][1] = R(kZt[0] * kZb[0]) * p0 + R(kZt[1] * kZb[1]) * p1;
      gp[j][2] = R(kZb[0] * kZb[0]) * p0 + R(kZb[1] * kZb[1]) * p1;
      gm[j][0] = R(kZt[0] * kZt[0]) * m0 + R(kZt[1] * kZt[1]) * m1;
      gm[j][1] = R(kZt[0] * kZb[0]) * m0 + R(kZt[1] * kZb[1]) * m1;
      gm[j][2] = R(kZb[0] * kZb[0]) * m0 + R(kZb[1] * kZb[1]) * m1;
    }
#pragma unroll
    for (int y = 0; y < 3; ++y) {
      constexpr double s0 = kS[0], s2 = kS[2];
      // edge points at s0, 1/2 and s2 = 1 - s0
      Kp[0][y] = R(s2 * s2) * gp[0][y] + R(0.25) * gp[1][y] + R(s0 * s0) * gp[2][y];
      Kp[1][y] = R(s0 * s2) * gp[0][y] + R(0.25) * gp[1][y] + R(s0 * s2) * gp[2][y];
      Kp[2][y] = R(s0 * s0) * gp[0][y] + R(0.25) * gp[1][y] + R(s2 * s2) * gp[2][y];
      Km[0][y] = R(s2 * s2) * gm[0][y] + R(0.25) * gm[1][y] + R(s0 * s0) * gm[2][y];
      Km[1][y] = R(s0 * s2) * gm[0][y] + R(0.25) * gm[1][y] + R(s0 * s2) * gm[2][y];
      Km[2][y] = R(s0 * s0) * gm[0][y] + R(0.25) * gm[1][y] + R(s2 * s2) * gm[2][y];
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const R TA = own(f, A), TB = own(f, B), TA3 = own(f, A + 3), TB3 = own(f, B + 3);
      const R* o = to[f];
      const R Ti[4] = {TA, TB, TA3, TB3};
      R* r = res[f];
      // one multiply-add a product (FP32 2 fields 0.71 M prisms 41.1 -> 39.0 us, the walk
      // of 8 layers with 4 fields 634 -> 623)
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int x = n & 1, y = n >> 1;
        r[A] -= Kp[x][y] * Ti[n];
        r[B] -= Kp[1 + x][y] * Ti[n];
        r[A + 3] -= Kp[x][1 + y] * Ti[n];
        r[B + 3] -= Kp[1 + x][1 + y] * Ti[n];
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int x = n & 1, y = n >> 1;
        r[A] -= Km[x][y] * o[n];
        r[B] -= Km[1 + x][y] * o[n];
        r[A + 3] -= Km[x][1 + y] * o[n];
        r[B + 3] -= Km[1 + x][1 + y] * o[n];
      }
    }
  }
}

// Horizontal face between an upper prism (its bottom nodes 3..5) and a lower
// prism (its top nodes 0..2) of one column, at level heights zf:
//   F_q = w_q lambda(q).un      upward flux (un: upward normal velocity times
//                               J_h at the 3 face nodes, averaged over the
//                               two sides where both exist)
//   h_q = max(F_q, 0) T_lower(q) + min(F_q, 0) T_upper(q)
//   g_n = sum_q lambda_n(q) h_q
// The upper prism adds g to its bottom nodes' residual, the lower prism
// subtracts it from its top nodes'.  A missing side (surface, bottom) takes
// the exterior value and does not enter the velocity average.
// As in the volume term, the sums over q are contracted once per face into
//   Gp[n][a] = sum_q lambda_n(q) lambda_a(q) max(F_q, 0),
//   Gm[n][a] = sum_q lambda_n(q) lambda_a(q) min(F_q, 0)   (both symmetric),
// so g = Gp T_lower + Gm T_upper per field (18 multiply-adds instead of 66).
template <typename R>
struct HorF {
  R gp[6], gm[6];   // symmetric 3x3, entries 00 11 22 01 02 12
  bool has_up, has_lo;
};

template <typename R, bool WZ>
__device__ __forceinline__ void hface_factors(const ColGeo<R>& cg, const R zf[3], bool has_up, const R uu[3],
                                              const R vu[3], const R wu[3], bool has_lo, const R ul[3],
                                              const R vl[3], const R wl[3], HorF<R>& F) {
  const R zxi = zf[1] - zf[0], zet = zf[2] - zf[0];
  const R jzx = zxi * cg.yet - zet * cg.yxi;
  const R jzy = zet * cg.xxi - zxi * cg.xet;
  R un[3];
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    R x = -(uu[n] * jzx + vu[n] * jzy);
    if (!WZ) x += cg.Jh * wu[n];
    R y = -(ul[n] * jzx + vl[n] * jzy);
    if (!WZ) y += cg.Jh * wl[n];
    const R avg = R(0.5) * (x + y);
    un[n] = has_up ? (has_lo ? avg : x) : y;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) F.gp[i] = F.gm[i] = R(0);
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const R Fq = R(kTw[q]) * (R(kL0[q]) * un[0] + R(kL1[q]) * un[1] + R(kL2[q]) * un[2]);
    const R fp = upos(Fq), fm = uneg(Fq);
    const R c[6] = {R(kL0[q] * kL0[q]), R(kL1[q] * kL1[q]), R(kL2[q] * kL2[q]),
                    R(kL0[q] * kL1[q]), R(kL0[q] * kL2[q]), R(kL1[q] * kL2[q])};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      F.gp[i] += c[i] * fp;
      F.gm[i] += c[i] * fm;
    }
  }
  F.has_up = has_up;
  F.has_lo = has_lo;
}

template <typename R>
__device__ __forceinline__ void hface_field(const HorF<R>& F, R te, const R Tu[3], const R Tl[3], R g[3]) {
  R tu[3], tl[3];
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    tu[n] = F.has_up ? Tu[n] : te;
    tl[n] = F.has_lo ? Tl[n] : te;
  }
  const R gp[3][3] = {{F.gp[0], F.gp[3], F.gp[4]}, {F.gp[3], F.gp[1], F.gp[5]}, {F.gp[4], F.gp[5], F.gp[2]}};
  const R gm[3][3] = {{F.gm[0], F.gm[3], F.gm[4]}, {F.gm[3], F.gm[1], F.gm[5]}, {F.gm[4], F.gm[5], F.gm[2]}};
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    g[n] = gp[n][0] * tl[0];
    g[n] += gp[n][1] * tl[1];
    g[n] += gp[n][2] * tl[2];
    g[n] += gm[n][0] * tu[0];
    g[n] += gm[n][1] * tu[1];
    g[n] += gm[n][2] * tu[2];
  }
}

// Mz = J_h/120 * m with m_aa = 3 dz_a + dz_b + dz_c, m_ab = dz_a + dz_b + dz_c/2;
// Mz^-1 = sc * cofactors.
template <typename R>
struct MinvF {
  R c00, c01, c02, c11, c12, c22, sc;
};

template <typename R>
__device__ __forceinline__ void minv_factors(const ColGeo<R>& cg, const R dz[3], MinvF<R>& F) {
  const R m00 = R(3) * dz[0] + dz[1] + dz[2];
  const R m11 = dz[0] + R(3) * dz[1] + dz[2];
  const R m22 = dz[0] + dz[1] + R(3) * dz[2];
  const R m01 = dz[0] + dz[1] + R(0.5) * dz[2];
  const R m02 = dz[0] + dz[2] + R(0.5) * dz[1];
  const R m12 = dz[1] + dz[2] + R(0.5) * dz[0];
  F.c00 = m11 * m22 - m12 * m12;
  F.c01 = m02 * m12 - m01 * m22;
  F.c02 = m01 * m12 - m02 * m11;
  F.c11 = m00 * m22 - m02 * m02;
  F.c12 = m01 * m02 - m00 * m12;
  F.c22 = m00 * m11 - m01 * m01;
  const R det = m00 * F.c00 + m01 * F.c01 + m02 * F.c02;
  F.sc = R(120) / (cg.Jh * det);
}

// L = M^-1 res (M^-1 = [2 -1; -1 2] (x) Mz^-1), then out = a Tn + b (T + dt L)
// (or L alone), stored at row f of the output for an active prism.
template <typename R, bool RHS, bool READ_TN, bool OUT2>
__device__ __forceinline__ void finish_field(const StageArgs& a, const MinvF<R>& F, int f, const R T[6],
                                             const R res[6], const R tn[6], uint32_t po, bool active) {
  const R ht[3] = {R(2) * res[0] - res[3], R(2) * res[1] - res[4], R(2) * res[2] - res[5]};
  const R hb[3] = {R(2) * res[3] - res[0], R(2) * res[4] - res[1], R(2) * res[5] - res[2]};
  R L[6];
  L[0] = F.sc * (F.c00 * ht[0] + F.c01 * ht[1] + F.c02 * ht[2]);
  L[1] = F.sc * (F.c01 * ht[0] + F.c11 * ht[1] + F.c12 * ht[2]);
  L[2] = F.sc * (F.c02 * ht[0] + F.c12 * ht[1] + F.c22 * ht[2]);
  L[3] = F.sc * (F.c00 * hb[0] + F.c01 * hb[1] + F.c02 * hb[2]);
  L[4] = F.sc * (F.c01 * hb[0] + F.c11 * hb[1] + F.c12 * hb[2]);
  L[5] = F.sc * (F.c02 * hb[0] + F.c12 * hb[1] + F.c22 * hb[2]);
  const size_t S = (size_t)a.m.n_slots;
  R* __restrict__ Out = static_cast<R*>(a.Tout);
  R* __restrict__ Out2 = static_cast<R*>(a.Tout2);
  const R dt = R(a.dt), ca = R(a.a), cb = R(a.b);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    R out;
    if (RHS) {
      out = L[i];
    } else {
      out = cb * (T[i] + dt * L[i]);
      if (READ_TN) out += ca * tn[i];
    }
    if (active) {
      str(Out, S, f * 6 + i, po, out);
      // second output T - 2 Tout (the split-IMEX first step)
      if (OUT2) str(Out2, S, f * 6 + i, po, T[i] - R(2) * out);
    }
  }
}

// Which tiles workgroup b processes: one tile, or (a.persistent) a grid sized
// to what the chip holds at once, each workgroup walking tiles with a stride.
// With the XCD remap, tiles are split into 8 contiguous parts and workgroup
// b, which the dispatcher places on XCD b mod 8, takes part b mod 8, so tiles
// that share faces are processed on one XCD and its L2 (the persistent grid is
// a multiple of 8).
struct TileRange {
  int t, end, step;
};

__device__ __forceinline__ TileRange tile_range(const StageArgs& a) {
  const int b = (int)blockIdx.x;
  TileRange r;
  if (!a.persistent) {
    r.t = a.xcd ? xcd_tile(b, a.n_tiles) : b;
    r.end = r.t + 1;
    r.step = 1;
  } else if (a.xcd) {
    const int q = a.n_tiles >> 3, rem = a.n_tiles & 7, x = b & 7;
    const int lo = x * q + (x < rem ? x : rem);
    r.t = lo + (b >> 3);
    r.end = lo + q + (x < rem ? 1 : 0);
    r.step = (int)gridDim.x >> 3;
  } else {
    r.t = b;
    r.end = a.n_tiles;
    r.step = (int)gridDim.x;
  }
  return r;
}

// ===========================================================================
// stage_kernel: one thread per prism.
// ===========================================================================
// With SH each wavefront puts its layer's stage input and horizontal velocity in LDS,
// reads them again from there for each term, and with them its neighbours in the
// cell.  Without, the kernel is bound by the address unit of the loads, busy for 0.8
// of the time: a neighbour gather touches about 45 lines where a row of the own
// prisms touches 8.  With, four fields in double take 247 registers for 372 (two
// wavefronts per SIMD for one).  Third stage, without -> with: FP64 4 fields 6.0 M
// prisms 1.49 -> 1.22 ms, FP32 4 fields 0.80 -> 0.66 ms, FP64 1 field 1.0 M 93 ->
// 79 us, FP64 3 fields with w 0.35 M 68 -> 61 us.
// A launch of at most one wavefront per SIMD has only its own chain of latencies, to
// which LDS adds: launch_mode draws the line there.  Third stage in blocks of two
// layers, without -> with LDS (without: one wavefront per SIMD, see stage_kernel):
//   904 wavefronts   FP64 1-4 fields  7.5 9.6 12.2 13.4 -> 9.9 12.7 15.7 17.8 us
//                    FP32             5.6 7.1  8.4 10.2 -> 5.9  7.5  8.7 10.2
// and on the line's other side, where more than one wavefront has to fit a SIMD:
//   1130 wavefronts  FP64            10.3 12.9 18.5 21.0 -> 10.9 13.8 17.0 19.6
//                    FP32             6.9  8.6 10.5 12.6 ->  6.2  7.8  9.4 11.4
//   1400 wavefronts  FP64            12.0 15.9 22.2 25.3 -> 12.4 15.3 20.0 22.0
template <int NF>
constexpr int kStageRows = 6 * NF + 12;   // LDS rows of a wavefront: stage input, u, v

template <typename R, int NF, bool WZ, bool RHS, bool READ_TN, bool OUT2, bool SH>
__device__ __forceinline__ void stage_tile(const StageArgs& a, const WgTile tile, R* sh) {
  const DevMesh& m = a.m;
  const int lane = threadIdx.x & (kCell - 1);
  const int l = tile.layer0 + (threadIdx.x >> 6);
  const int c = tile.cell * kCell + lane;
  // Threads past their column's depth still run (on in-bounds padding slots
  // of their cell) so that no load waits on nlay; only the store is masked.
  const int N = m.nlay[c];
  const int depth = (m.cell_base[tile.cell + 1] - m.cell_base[tile.cell]) / kCell;
  if (l >= depth) return;  // uniform per wavefront
  const bool active = l < N;

  const size_t S = (size_t)m.n_slots;
  const size_t LS = (size_t)m.n_lslots;
  const uint32_t p = (uint32_t)m.cell_base[tile.cell] + (uint32_t)l * kCell + lane;
  const uint32_t lt = (uint32_t)m.cell_lbase[tile.cell] + (uint32_t)l * kCell + lane;
  const uint32_t po = p * (uint32_t)sizeof(R);       // this prism's byte offset in a row
  const uint32_t co = (uint32_t)c * (uint32_t)sizeof(R);
  const R* __restrict__ Ts = static_cast<const R*>(a.Ts);
  const R* __restrict__ U = static_cast<const R*>(a.U);
  const R* __restrict__ Tn = static_cast<const R*>(a.Tn);
  const R* __restrict__ zl = zl_of<R>(m);
  // neighbour layers above and below; the address only needs the
  // (wavefront-uniform) cell depth, the value select the column's own depth
  const uint32_t pup = (l > 0 ? p - kCell : p) * (uint32_t)sizeof(R);
  const uint32_t plo = (l + 1 < depth ? p + kCell : p) * (uint32_t)sizeof(R);

  const ColGeo<R> cg = load_colgeo<R>(m, co);
  R zt[3], zb[3], dz[3];
#pragma unroll
  for (int v3 = 0; v3 < 3; ++v3) {
    zt[v3] = ldb(zl + v3 * LS, lt * (uint32_t)sizeof(R));
    zb[v3] = ldb(zl + v3 * LS, (lt + kCell) * (uint32_t)sizeof(R));
    dz[v3] = zt[v3] - zb[v3];
  }
  R T[NF][6], res[NF][6];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) T[f][i] = ldr(Ts, S, f * 6 + i, po);
  auto held = [&](int f, int i) { return T[f][i]; };
  auto own = [&](int f, int i) { return SH ? sh[(f * 6 + i) * kCell + lane] : T[f][i]; };
  R u[6], v[6], w[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    u[i] = ldr(U, S, 0 * 6 + i, po);
    v[i] = ldr(U, S, 1 * 6 + i, po);
    w[i] = WZ ? R(0) : ldr(U, S, 2 * 6 + i, po);
  }
  LatMeta<R> M[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) lat_meta<R>(m, e, co, M[e]);
  // the velocity again for the next term
  auto reread = [&]() {
    if constexpr (SH) {
      mem_order();
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        u[i] = sh[(6 * NF + i) * kCell + lane];
        v[i] = sh[(6 * NF + 6 + i) * kCell + lane];
      }
    }
  };
  // A term's neighbour values are requested one term ahead of their use.
  LatNb<R> nb[2];
  R to[2][NF][4];
  const uint32_t cell_base = (uint32_t)m.cell_base[tile.cell];
  auto request = [&](int e) {
    lat_request<R, NF, SH>(a, M[e], e, l, po, lane, cell_base, nb[e & 1], to[e & 1]);
  };
  R ut[2][9], Tx[2][NF][3];   // above (bottom nodes) and below (top nodes): velocity, stage input
  auto request_layer = [&](int s, uint32_t pn) {
    const int n0 = s == 0 ? 3 : 0;
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      ut[s][n] = ldr(U, S, 0 * 6 + n0 + n, pn);
      ut[s][3 + n] = ldr(U, S, 1 * 6 + n0 + n, pn);
      ut[s][6 + n] = WZ ? R(0) : ldr(U, S, 2 * 6 + n0 + n, pn);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int n = 0; n < 3; ++n) Tx[s][f][n] = ldr(Ts, S, f * 6 + n0 + n, pn);
  };
  request(0);
  phase();
  if constexpr (SH) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
      for (int f = 0; f < NF; ++f) sh[(f * 6 + i) * kCell + lane] = T[f][i];
      sh[(6 * NF + i) * kCell + lane] = u[i];
      sh[(6 * NF + 6 + i) * kCell + lane] = v[i];
    }
    mem_order();
  }
  volume_term<R, NF, WZ>(cg, zt, zb, dz, u, v, w, held, res);
  formed<R, NF>(res);
  if constexpr (SH) mem_order();
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    if (e < 2) request(e + 1);
    else request_layer(0, pup);
    phase();
    if constexpr (SH) lat_resolve<R, NF>(sh, nb[e & 1], to[e & 1]);
    LatQ<R> F;
    reread();
    lat_weights<R>(M[e], nb[e & 1], e, l, dz, u, v, F);
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) to[e & 1][f][j] = lat_trace<R>(a, M[e], f, to[e & 1][f][j]);
    lat_apply<R, NF>(e, F, own, to[e & 1], res);
    formed<R, NF>(res);
  }
  request_layer(1, plo);
  R tn[NF][6];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) tn[f][i] = READ_TN ? ldr(Tn, S, f * 6 + i, po) : R(0);
  phase();
  HorF<R> hf;
  reread();
  hface_factors<R, WZ>(cg, zt, l > 0, ut[0], ut[0] + 3, ut[0] + 6, true, u, v, w, hf);
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const R To[3] = {own(f, 0), own(f, 1), own(f, 2)};
    R g[3];
    hface_field<R>(hf, R(a.t_ext[f]), Tx[0][f], To, g);
#pragma unroll
    for (int n = 0; n < 3; ++n) res[f][n] -= g[n];
  }
  formed<R, NF>(res);
  reread();
  hface_factors<R, WZ>(cg, zb, true, u + 3, v + 3, w + 3, l < N - 1, ut[1], ut[1] + 3, ut[1] + 6, hf);
  MinvF<R> mf;
  minv_factors<R>(cg, dz, mf);
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    R g[3], To[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) To[i] = own(f, i);
    hface_field<R>(hf, R(a.t_ext[f]), To + 3, Tx[1][f], g);
#pragma unroll
    for (int n = 0; n < 3; ++n) res[f][3 + n] += g[n];
    finish_field<R, RHS, READ_TN, OUT2>(a, mf, f, To, res[f], tn[f], po, active);
  }
}

// Without SH the launch has at most one wavefront per SIMD.  In double with one or two
// fields the kernel then reserves more than half of a SIMD's registers, as with three
// and four fields it needs: of two blocks of two wavefronts the dispatcher puts the
// second on the SIMDs of the first while others idle, where both fit.  Third stage of
// 640 wavefronts in blocks of two, both fitting -> reserved: 1 field 9.0 -> 7.3 us, 2
// fields 11.5 -> 9.2.  In float it gains less (4 fields 10.0 -> 9.1), and steps of four
// streams side by side lose (904 wavefronts each, 20 -> 22 us a step).
template <typename R, int NF, bool WZ, bool RHS, bool READ_TN, bool OUT2, bool SH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, !SH && sizeof(R) == 8 && NF <= 2 ? 1 : 8)))
void stage_kernel(StageArgs a) {
  // each wavefront's own rows: the LDS accesses of a wavefront complete in order, so
  // they need no barrier, neither within a tile nor from one tile to the next
  extern __shared__ __align__(16) char stage_lds[];
  R* sh = SH ? reinterpret_cast<R*>(stage_lds) + (threadIdx.x >> 6) * (kStageRows<NF> * kCell) : nullptr;
  TileRange r = tile_range(a);
  for (; r.t < r.end; r.t += r.step) stage_tile<R, NF, WZ, RHS, READ_TN, OUT2, SH>(a, a.tiles[r.t], sh);
}

// ===========================================================================
// walk_kernel: one wavefront walks a cell's layers l0 .. l0 + nlay - 1 of its tile.
// ===========================================================================
constexpr int kWalkLdsBytes = 40960;   // two layer slots; 4 wavefronts per CU

// LDS slot of one layer: [row][64 lanes] values of type R, in sections
// (stage input, velocity, bottom level heights, Tn where it fits), each
// padded to whole 1 KiB loads.
template <typename R, int NF, bool WZ, bool READ_TN>
struct WalkLayout {
  static constexpr int kPerLoad = 1024 / (kCell * (int)sizeof(R));   // rows per 16 B/lane load
  static constexpr int pad(int r) { return (r + kPerLoad - 1) / kPerLoad * kPerLoad; }
  static constexpr int kNU = WZ ? 12 : 18;            // u 0..5, v 0..5 (, w 0..5)
  static constexpr int kTs = 0;
  static constexpr int kU = pad(6 * NF);
  static constexpr int kZ = kU + pad(kNU);
  static constexpr int kBase = kZ + pad(3);
  // Tn joins the layer copy only where two slots with it stay within one
  // wavefront's share of the CU's LDS: 40 KB in FP64 (one wavefront per
  // SIMD), 20 KB in FP32 (two).  In FP32 with 4 fields it would not, and
  // holding it there cut the residency to five wavefronts per CU (stages 1
  // and 2: 0.94 against 0.72 ms with Tn read from global memory).
  static constexpr bool kTnLds =
      READ_TN && 2 * (kBase + pad(6 * NF)) * kCell * (int)sizeof(R) <= kWalkLdsBytes / (sizeof(R) == 8 ? 1 : 2);
  static constexpr int kTn = kBase;
  static constexpr int kRows = kBase + (kTnLds ? pad(6 * NF) : 0);
  static constexpr int kSlot = kRows * kCell;         // values of type R per slot
  static constexpr int kBytes = 2 * kSlot * (int)sizeof(R);
  static_assert(kBytes <= 65536, "walk LDS above the workgroup limit");
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Copy `count` rows (row stride rowb bytes) starting at `base` + lane offset
// `voff` into LDS rows from `dst`: each 16-byte-per-lane load moves kPerLoad
// rows of kCell values, lane i writing LDS bytes [16 i, 16 i + 16) of the
// load's 1 KiB block; rows past `count` in the last load repeat the last row.
template <typename R, int kPerLoad>
__device__ __forceinline__ void fetch_rows(const char* base, uint32_t rowb, int count, uint32_t voff, int sub,
                                           R* dst) {
#pragma unroll
  for (int k = 0; k < (count + kPerLoad - 1) / kPerLoad; ++k) {
    const int left = count - 1 - k * kPerLoad;
    const uint32_t j = (uint32_t)(sub < left ? sub : left);
    __builtin_amdgcn_global_load_lds(base + (size_t)(k * kPerLoad) * rowb + (j * rowb + voff),
                                     (lds_ptr_t)(dst + k * kPerLoad * kCell), 16, 0, 0);
  }
}

struct WalkCell {
  int cell, N, depth;
  uint32_t base, lbase;
};
// One layer L of this cell into an LDS slot.
template <typename R, int NF, bool WZ, bool READ_TN>
__device__ __forceinline__ void walk_fetch(const StageArgs& a, const WalkCell& wc, int L, R* slot, int lane) {
  using Ly = WalkLayout<R, NF, WZ, READ_TN>;
  constexpr int kLanesPerRow = kCell / Ly::kPerLoad;
  const DevMesh& m = a.m;
  const int sub = lane / kLanesPerRow;
  const uint32_t chunk = (uint32_t)(lane % kLanesPerRow) * 16u;
  const uint32_t rowb = (uint32_t)((size_t)m.n_slots * sizeof(R));
  const uint32_t lrowb = (uint32_t)((size_t)m.n_lslots * sizeof(R));
  const uint32_t pb = (wc.base + (uint32_t)L * kCell) * (uint32_t)sizeof(R) + chunk;
  const uint32_t zb = (wc.lbase + (uint32_t)(L + 1) * kCell) * (uint32_t)sizeof(R) + chunk;
  fetch_rows<R, Ly::kPerLoad>(static_cast<const char*>(a.Ts), rowb, 6 * NF, pb, sub, slot + Ly::kTs * kCell);
  fetch_rows<R, Ly::kPerLoad>(static_cast<const char*>(a.U), rowb, Ly::kNU, pb, sub, slot + Ly::kU * kCell);
  fetch_rows<R, Ly::kPerLoad>(reinterpret_cast<const char*>(zl_of<R>(m)), lrowb, 3, zb, sub, slot + Ly::kZ * kCell);
  if (Ly::kTnLds)
    fetch_rows<R, Ly::kPerLoad>(static_cast<const char*>(a.Tn), rowb, 6 * NF, pb, sub, slot + Ly::kTn * kCell);
}

// vmcnt(0) / lgkmcnt(0) alone (gfx9 s_waitcnt encoding), each also a
// compiler memory barrier so no LDS read is moved above the wait that makes
// its data valid, nor a copy into LDS above the reads it must follow.
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lgkm() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
}
// Column-walk form of lat_nb.  The layer's stage input and velocity of all
// 64 columns of the cell are already in the LDS slot `cur`, so a neighbour
// column of the same cell (most lateral faces of a locality-ordered mesh) is
// read from there; only a neighbour in another cell is read from global
// memory.  A face without a live neighbour points at the column's own nodes
// in LDS (in bounds, unused).
template <typename R, int kURow>
__device__ __forceinline__ void lat_nb_walk(const StageArgs& a, const LatMeta<R>& M, int e, int l, uint32_t po,
                                            int lane, uint32_t cell_base, const R* cur, LatNb<R>& nb) {
  const size_t S = (size_t)a.m.n_slots;
  const uint32_t rs = (uint32_t)(S * sizeof(R));
  const R* __restrict__ U = static_cast<const R*>(a.U);
  const int A = e, B = (e + 1) % 3;
  const bool live = M.nslot >= 0 && l < (M.meta >> 2);
  const int kp = M.meta & 3;
  const uint32_t nlane = (uint32_t)M.nslot - cell_base;   // < 64 iff the neighbour is in this cell
  nb.lds = !live || nlane < (uint32_t)kCell;
  const uint32_t nA = live ? (uint32_t)((kp + 1) % 3) : (uint32_t)A;
  const uint32_t nB = live ? (uint32_t)kp : (uint32_t)B;
  if (nb.lds) {
    constexpr uint32_t row = kCell * sizeof(R);
    const uint32_t ln = (live ? nlane : (uint32_t)lane) * (uint32_t)sizeof(R);
    nb.no[0] = nA * row + ln;
    nb.no[1] = nB * row + ln;
    nb.no[2] = nb.no[0] + 3u * row;
    nb.no[3] = nb.no[1] + 3u * row;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      nb.uo[j] = lds_at(cur, (uint32_t)kURow * row + nb.no[j]);
      nb.vo[j] = lds_at(cur, (uint32_t)(kURow + 6) * row + nb.no[j]);
    }
  } else {
    const uint32_t pno = ((uint32_t)M.nslot + (uint32_t)l * kCell) * (uint32_t)sizeof(R);
    (void)po;
    nb.no[0] = nA * rs + pno;
    nb.no[1] = nB * rs + pno;
    nb.no[2] = nb.no[0] + 3u * rs;
    nb.no[3] = nb.no[1] + 3u * rs;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      nb.uo[j] = ldb(U, nb.no[j]);
      nb.vo[j] = ldb(U + 6 * S, nb.no[j]);
    }
  }
}

// Column-walk form of the neighbour traces of field f: from the LDS slot or from
// global memory, as lat_nb_walk decided.
template <typename R, int kTsRow>
__device__ __forceinline__ void lat_traces_walk(const StageArgs& a, const LatNb<R>& nb, int f, const R* cur, R to[4]) {
  const R* fb = static_cast<const R*>(a.Ts) + (size_t)(f * 6) * (size_t)a.m.n_slots;
  constexpr uint32_t row = kCell * sizeof(R);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (nb.lds)
      to[j] = lds_at(cur, (uint32_t)(kTsRow + f * 6) * row + nb.no[j]);
    else
      to[j] = ldb(fb, nb.no[j]);
  }
}

// State a wavefront carries from one layer of its walk to the next.
template <typename R, int NF>
struct WalkCarry {
  R zt[3];          // heights of the layer's top level
  R gtop[NF][3];    // horizontal-face contribution to the layer's top nodes
};

// One layer l of the walk.  `cur` holds layer l (complete), `nxt` receives
// layer l+1.  cur and nxt are distinct __shared__ arrays, so the compiler
// sees that reading cur does not wait for the copy into nxt.  Loads complete
// in order, so the layer's loads are issued in the order of their use, all of
// them before its arithmetic: the prism's own values (LDS), the neighbours'
// velocities and traces, the next layer's copy, Tn.  Nothing but the bottom
// face and the update then waits on the copy.
template <typename R, int NF, bool WZ, bool RHS, bool READ_TN, bool OUT2>
__device__ __forceinline__ void walk_layer(const StageArgs& a, const ColGeo<R>& cg, const LatMeta<R> (&lm)[3],
                                           const WalkCell& wc, int lane, int l, const R* cur, R* nxt,
                                           WalkCarry<R, NF>& cs) {
  const int N = wc.N, depth = wc.depth;
  using Ly = WalkLayout<R, NF, WZ, READ_TN>;
  const DevMesh& m = a.m;
  const size_t S = (size_t)m.n_slots;
  const uint32_t p = wc.base + (uint32_t)l * kCell + lane;
  const uint32_t po = p * (uint32_t)sizeof(R);
  const bool below = l + 1 < depth;   // wavefront-uniform
  const bool active = l < N;
  auto at = [&](int row) { return cur[row * kCell + lane]; };
  auto next = [&](int row, R fallback) { return below ? nxt[row * kCell + lane] : fallback; };

  R T[NF][6], u[6], v[6], w[6], zb[3], dz[3];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < 6; ++i) T[f][i] = at(Ly::kTs + f * 6 + i);
  auto held = [&](int f, int i) { return T[f][i]; };
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    u[i] = at(Ly::kU + i);
    v[i] = at(Ly::kU + 6 + i);
    w[i] = WZ ? R(0) : at(Ly::kU + 12 + i);
  }
#pragma unroll
  for (int v3 = 0; v3 < 3; ++v3) {
    zb[v3] = at(Ly::kZ + v3);
    dz[v3] = cs.zt[v3] - zb[v3];
  }
  // the neighbour reads below are flat loads, which count against both wait
  // counters: an LDS read still in flight would make its user wait for them too
  wait_lgkm();
  phase();
  LatNb<R> nb[3];
  R to[3][NF][4];
#pragma unroll
  for (int e = 0; e < 3; ++e) lat_nb_walk<R, Ly::kU>(a, lm[e], e, l, po, lane, wc.base, cur, nb[e]);
#pragma unroll
  for (int e = 0; e < 3; ++e)
#pragma unroll
    for (int f = 0; f < NF; ++f) lat_traces_walk<R, Ly::kTs>(a, nb[e], f, cur, to[e][f]);
  phase();
  if (below) walk_fetch<R, NF, WZ, READ_TN>(a, wc, l + 1, nxt, lane);
  mem_order();
  phase();

  R res[NF][6];
  volume_term<R, NF, WZ>(cg, cs.zt, zb, dz, u, v, w, held, res);
  formed<R, NF>(res);
  // from here on the prism's own values are read from LDS again: the first use
  // of a neighbour value waits for all of them, and LDS reads no longer wait
  mem_order();
  auto own = [&](int f, int i) { return at(Ly::kTs + f * 6 + i); };
  const R* __restrict__ Tn = static_cast<const R*>(a.Tn);
  R tn[NF][6];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    LatQ<R> F;
    lat_weights<R>(lm[e], nb[e], e, l, dz, u, v, F);
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) to[e][f][j] = lat_trace<R>(a, lm[e], f, to[e][f][j]);
    lat_apply<R, NF>(e, F, own, to[e], res);
    formed<R, NF>(res);
    if (e == 1) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) tn[f][i] = (READ_TN && !Ly::kTnLds) ? ldr(Tn, S, f * 6 + i, po) : R(0);
      phase();
    }
  }
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int n = 0; n < 3; ++n) res[f][n] -= cs.gtop[f][n];
  MinvF<R> mf;
  minv_factors<R>(cg, dz, mf);
  phase();
  wait_vm();   // layer l+1 has arrived
  HorF<R> bot;
  {
    R ul[3], vl[3], wl[3];
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      ul[n] = next(Ly::kU + n, u[3 + n]);
      vl[n] = next(Ly::kU + 6 + n, v[3 + n]);
      wl[n] = WZ ? R(0) : next(Ly::kU + 12 + n, w[3 + n]);
    }
    hface_factors<R, WZ>(cg, zb, true, u + 3, v + 3, w + 3, l < N - 1, ul, vl, wl, bot);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    phase();
    R Tl[3], Tf[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) Tf[i] = own(f, i);
#pragma unroll
    for (int n = 0; n < 3; ++n) Tl[n] = next(Ly::kTs + f * 6 + n, Tf[3 + n]);
    hface_field<R>(bot, R(a.t_ext[f]), Tf + 3, Tl, cs.gtop[f]);
#pragma unroll
    for (int n = 0; n < 3; ++n) res[f][3 + n] += cs.gtop[f][n];
    if (Ly::kTnLds) {
#pragma unroll
      for (int i = 0; i < 6; ++i) tn[f][i] = at(Ly::kTn + f * 6 + i);
    }
    finish_field<R, RHS, READ_TN, OUT2>(a, mf, f, Tf, res[f], tn[f], po, active);
  }
#pragma unroll
  for (int v3 = 0; v3 < 3; ++v3) cs.zt[v3] = zb[v3];
}

template <typename R, int NF, bool WZ, bool RHS, bool READ_TN, bool OUT2>
__global__ __launch_bounds__(64) void walk_kernel(StageArgs a) {
  using Ly = WalkLayout<R, NF, WZ, READ_TN>;
  __shared__ __align__(16) R slot0[Ly::kSlot];
  __shared__ __align__(16) R slot1[Ly::kSlot];
  const DevMesh& m = a.m;
  const int lane = threadIdx.x;
  TileRange r = tile_range(a);
  for (; r.t < r.end; r.t += r.step) {
    const WgTile tile = a.tiles[r.t];
    const int cell = tile.cell;
    const int c = cell * kCell + lane;
    WalkCell wc;
    wc.cell = cell;
    wc.N = m.nlay[c];
    wc.base = (uint32_t)m.cell_base[cell];
    wc.lbase = (uint32_t)m.cell_lbase[cell];
    wc.depth = (int)(((uint32_t)m.cell_base[cell + 1] - wc.base) / kCell);
    const int l0 = tile.layer0;
    const int l1 = l0 + tile.nlay;
    const size_t S = (size_t)m.n_slots;
    const size_t LS = (size_t)m.n_lslots;
    const uint32_t pc = wc.base + lane;
    const R* __restrict__ Ts = static_cast<const R*>(a.Ts);
    const R* __restrict__ U = static_cast<const R*>(a.U);
    const R* __restrict__ zl = zl_of<R>(m);
    const uint32_t co = (uint32_t)c * (uint32_t)sizeof(R);
    const ColGeo<R> cg = load_colgeo<R>(m, co);
    LatMeta<R> lm[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) lat_meta<R>(m, e, co, lm[e]);

    // layer l0 into slot0; the top face of l0 from the layer above (global)
    wait_lgkm();
    walk_fetch<R, NF, WZ, READ_TN>(a, wc, l0, slot0, lane);
    WalkCarry<R, NF> cs;
    {
      const uint32_t lt = wc.lbase + (uint32_t)l0 * kCell + lane;
#pragma unroll
      for (int v3 = 0; v3 < 3; ++v3) cs.zt[v3] = ldb(zl + v3 * LS, lt * (uint32_t)sizeof(R));
      const uint32_t pup = (l0 > 0 ? pc + (uint32_t)(l0 - 1) * kCell : pc) * (uint32_t)sizeof(R);
      R uu[3], vu[3], wu[3], ul[3], vl[3], wl[3];
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        uu[n] = ldr(U, S, 0 * 6 + 3 + n, pup);
        vu[n] = ldr(U, S, 1 * 6 + 3 + n, pup);
        wu[n] = WZ ? R(0) : ldr(U, S, 2 * 6 + 3 + n, pup);
      }
      // the layer above's bottom values, requested with its velocity before the wait
      R Tu[NF][3];
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int n = 0; n < 3; ++n) Tu[f][n] = ldr(Ts, S, f * 6 + 3 + n, pup);
      wait_vm();
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        ul[n] = slot0[(Ly::kU + n) * kCell + lane];
        vl[n] = slot0[(Ly::kU + 6 + n) * kCell + lane];
        wl[n] = WZ ? R(0) : slot0[(Ly::kU + 12 + n) * kCell + lane];
      }
      HorF<R> top;
      hface_factors<R, WZ>(cg, cs.zt, l0 > 0, uu, vu, wu, true, ul, vl, wl, top);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        R Tl[3];
#pragma unroll
        for (int n = 0; n < 3; ++n) Tl[n] = slot0[(Ly::kTs + f * 6 + n) * kCell + lane];
        hface_field<R>(top, R(a.t_ext[f]), Tu[f], Tl, cs.gtop[f]);
      }
    }
    // layers in pairs so that each half names its slots statically
    for (int l = l0; l < l1; l += 2) {
      walk_layer<R, NF, WZ, RHS, READ_TN, OUT2>(a, cg, lm, wc, lane, l, slot0, slot1, cs);
      if (l + 1 < l1) walk_layer<R, NF, WZ, RHS, READ_TN, OUT2>(a, cg, lm, wc, lane, l + 1, slot1, slot0, cs);
    }
    // the last layer may have started a copy into a slot the next tile reuses
    wait_vm();
  }
}

// ---------------------------------------------------------------------------
// Launch.
// ---------------------------------------------------------------------------
// Workgroups of one kernel instance and block size that fit on one CU at once,
// queried once.
template <typename Kern>
hipError_t resident_per_cu(Kern kern, int threads, size_t lds, std::atomic<int>* cache, int* out) {
  int v = cache->load(std::memory_order_relaxed);
  if (v == 0) {
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, reinterpret_cast<const void*>(kern), threads,
                                                                 lds);
    if (e != hipSuccess) return e;
    if (v < 1) v = 1;
    cache->store(v, std::memory_order_relaxed);
  }
  *out = v;
  return hipSuccess;
}

// Launches one kernel over the tiles.
template <typename Kern>
hipError_t launch_tiles(Kern kern, const StageArgs& a, int threads, size_t lds, std::atomic<int>* cache,
                        hipStream_t s) {
  int grid = a.n_tiles;
  if (a.persistent) {
    int per_cu = 1;
    hipError_t e = resident_per_cu(kern, threads, lds, cache, &per_cu);
    if (e != hipSuccess) return e;
    grid = (per_cu * a.n_cu) & ~7;
    if (grid < 8) grid = 8;
    const int need = (a.n_tiles + 7) & ~7;
    if (grid > need) grid = need;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, s, a);
  return hipGetLastError();
}

template <typename R, int NF, bool WZ, bool RHS, bool READ_TN, bool OUT2>
hipError_t launch_mode(const StageArgs& a, hipStream_t s) {
  // one entry per block size: a walk is always one wavefront
  static std::atomic<int> walk_cache, lds_cache[kWalkMinLayers], cache[kWalkMinLayers];
  if (a.tile_layers >= kWalkMinLayers)
    return launch_tiles(&walk_kernel<R, NF, WZ, RHS, READ_TN, OUT2>, a, kCell, 0, &walk_cache, s);
  // no wavefronts for layers that no cell has: they would hold LDS (1,250 cells of one
  // layer in tiles of four, FP32 4 fields: 17.4 -> 11.7 us, FP64 1 field 13.6 -> 11.3)
  const int layers = a.tile_layers < a.m.max_layers ? a.tile_layers : a.m.max_layers;
  const int threads = kCell * layers;
  // more than one wavefront per SIMD (4 per CU): neighbours in the cell through LDS
  if ((int64_t)a.n_tiles * layers > 4 * (int64_t)a.n_cu)
    return launch_tiles(&stage_kernel<R, NF, WZ, RHS, READ_TN, OUT2, true>, a, threads,
                        (size_t)threads * kStageRows<NF> * sizeof(R), &lds_cache[layers], s);
  return launch_tiles(&stage_kernel<R, NF, WZ, RHS, READ_TN, OUT2, false>, a, threads, 0, &cache[layers], s);
}

template <typename R, int NF>
hipError_t launch_nf(const StageArgs& a, bool w_zero, bool rhs_only, bool read_tn, hipStream_t s) {
  if (rhs_only)
    return w_zero ? launch_mode<R, NF, true, true, false, false>(a, s) : launch_mode<R, NF, false, true, false, false>(a, s);
  if (read_tn)
    return w_zero ? launch_mode<R, NF, true, false, true, false>(a, s) : launch_mode<R, NF, false, false, true, false>(a, s);
  if (a.Tout2)
    return w_zero ? launch_mode<R, NF, true, false, false, true>(a, s) : launch_mode<R, NF, false, false, false, true>(a, s);
  return w_zero ? launch_mode<R, NF, true, false, false, false>(a, s) : launch_mode<R, NF, false, false, false, false>(a, s);
}

template <typename R>
hipError_t launch_r(const StageArgs& a, bool w_zero, bool rhs_only, bool read_tn, hipStream_t s) {
  switch (a.n_fields) {
    case 1: return launch_nf<R, 1>(a, w_zero, rhs_only, read_tn, s);
    case 2: return launch_nf<R, 2>(a, w_zero, rhs_only, read_tn, s);
    case 3: return launch_nf<R, 3>(a, w_zero, rhs_only, read_tn, s);
    case 4: return launch_nf<R, 4>(a, w_zero, rhs_only, read_tn, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_stage(const StageArgs& a, bool fp32, bool w_zero, bool rhs_only, bool read_tn,
                        hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  if (a.Tout2 && (rhs_only || read_tn)) return hipErrorInvalidValue;
  return fp32 ? launch_r<float>(a, w_zero, rhs_only, read_tn, s)
              : launch_r<double>(a, w_zero, rhs_only, read_tn, s);
}

}  // namespace sdg
