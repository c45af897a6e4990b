// Layer-parallel column solves: (M - dt A) x = M T* (forward, see vsolve.hip)
// and (M - dt A)^T mu = M Z (the adjoint's), one thread per prism.
//
// The block-Thomas recurrences of a column are nonlinear only in the pivots
// D'_l.  With B_l and C_l the 3x6 couplings to the layers above and below and
// P_l = B_l D'_{l-1}^-1 [:, bottom] (3x3) kept from one factor sweep per
// (kappa, dt, eta), every thread rebuilds its own D'_l (the Schur term is
// P_l C_{l-1} on the top rows) and inverts it in registers, and what is left
// of the recurrences is affine in three values per field:
//   down:  u_l = B_{l+1} y_l     = c_l - K_l u_{l-1}
//   up:    v_l = C_{l-1} x_l     = d_l - H_l v_{l+1}
//   x_l = D'_l^-1 (M T*_l - [u_{l-1}; 0] - [0; v_{l+1}])
// A block holds a group of columns over all their layers; (K, c) and (H, d)
// go through LDS, where a quad of lanes per (column, field) runs the two 3x3 chains,
// a lane per component.
// The transposed system has the same pivots (its block LU factors are the
// transposes): with q the forward intermediate, the chains carry q_l's bottom
// and mu_l's top values with K = H_fwd^T and H = K_fwd^T, so both systems use
// the same kept P.
//
// Against one lane per column walking its layers (vsolve.hip), which is left
// for deeper columns: that sweep moves 114 values per prism and field set of
// four (y_l makes a round trip through memory, E_l is read) and repeats an LU
// per layer in one serial chain; here a prism moves its right-hand side, its
// solution, the 9 kept values and its heights (60 values), and the serial part is a
// chain of three multiply-adds and a lane exchange a layer, twice.  One solve before ->
// now: 199,712 x 30 prisms, 4 fields, double 1158 -> 800 us (2.9 GB at 3.6 TB/s; 714 to
// 764 on other cards; some 70 us less without the two chains, 90 without the stores: a
// block's loads all come at its start, so memory idles while it computes), float state
// 1033 -> 606, float 586 -> 480; 68,220 ragged columns to 60 layers, 4 fields 1106 -> 452;
// 49,928 x 20, 1 field 115 -> 64; 1,800 x 10, 1 field 32 -> 7.
#include "internal.h"
#include "quadrature.h"

namespace sdg {
namespace {

template <typename C>
struct alignas(2 * sizeof(C)) CPair {
  C lo, hi;
};

// symmetric 3x3 storage: 0:00 1:11 2:22 3:01 4:02 5:12
__device__ __forceinline__ constexpr int sx(int a, int b) {
  return a == b ? a : (a + b == 1 ? 3 : (a + b == 2 ? 4 : 5));
}

template <typename C>
struct M3 {
  C m[3][3];
};

// 1/x to rounding: the hardware estimate and two Newton steps (x is a sum of
// layer thicknesses or a determinant of the column's mass-like blocks, far
// from the ends of the exponent range).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float recip(float x) { return 1.0f / x; }

// Inverse by cofactors.
template <typename C>
__device__ __forceinline__ M3<C> inv3(const M3<C>& a) {
  M3<C> r;
  r.m[0][0] = a.m[1][1] * a.m[2][2] - a.m[1][2] * a.m[2][1];
  r.m[1][0] = a.m[1][2] * a.m[2][0] - a.m[1][0] * a.m[2][2];
  r.m[2][0] = a.m[1][0] * a.m[2][1] - a.m[1][1] * a.m[2][0];
  r.m[0][1] = a.m[0][2] * a.m[2][1] - a.m[0][1] * a.m[2][2];
  r.m[1][1] = a.m[0][0] * a.m[2][2] - a.m[0][2] * a.m[2][0];
  r.m[2][1] = a.m[0][1] * a.m[2][0] - a.m[0][0] * a.m[2][1];
  r.m[0][2] = a.m[0][1] * a.m[1][2] - a.m[0][2] * a.m[1][1];
  r.m[1][2] = a.m[0][2] * a.m[1][0] - a.m[0][0] * a.m[1][2];
  r.m[2][2] = a.m[0][0] * a.m[1][1] - a.m[0][1] * a.m[1][0];
  const C s = recip(a.m[0][0] * r.m[0][0] + a.m[0][1] * r.m[1][0] + a.m[0][2] * r.m[2][0]);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.m[i][j] *= s;
  return r;
}

// a b, and base - a b
template <typename C>
__device__ __forceinline__ M3<C> mul3(const M3<C>& a, const M3<C>& b) {
  M3<C> r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.m[i][j] = a.m[i][0] * b.m[0][j] + a.m[i][1] * b.m[1][j] + a.m[i][2] * b.m[2][j];
  return r;
}
template <typename C>
__device__ __forceinline__ M3<C> sub_mul3(const M3<C>& base, const M3<C>& a, const M3<C>& b) {
  M3<C> r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      r.m[i][j] = base.m[i][j] - a.m[i][0] * b.m[0][j] - a.m[i][1] * b.m[1][j] - a.m[i][2] * b.m[2][j];
  return r;
}
template <typename C>
__device__ __forceinline__ M3<C> neg3(const M3<C>& a) {
  M3<C> r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.m[i][j] = -a.m[i][j];
  return r;
}
// Q (x - y) - t (2D mass) z, the products of the couplings:
// rows i: sum_k Q_ik (x_kj - y_kj) - t (sum_k z_kj + z_ij)
template <typename C>
__device__ __forceinline__ M3<C> couple3(const C Q[6], const M3<C>& x, const M3<C>& y, C t, const M3<C>& z) {
  M3<C> r;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const C e0 = x.m[0][j] - y.m[0][j], e1 = x.m[1][j] - y.m[1][j], e2 = x.m[2][j] - y.m[2][j];
    const C s = z.m[0][j] + z.m[1][j] + z.m[2][j];
#pragma unroll
    for (int i = 0; i < 3; ++i)
      r.m[i][j] = Q[sx(i, 0)] * e0 + Q[sx(i, 1)] * e1 + Q[sx(i, 2)] * e2 - t * (s + z.m[i][j]);
  }
  return r;
}
template <typename C>
__device__ __forceinline__ void couple_v(const C Q[6], const C x[3], const C y[3], C t, const C z[3], C out[3]) {
  const C e0 = x[0] - y[0], e1 = x[1] - y[1], e2 = x[2] - y[2];
  const C s = z[0] + z[1] + z[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) out[i] = Q[sx(i, 0)] * e0 + Q[sx(i, 1)] * e1 + Q[sx(i, 2)] * e2 - t * (s + z[i]);
}

// Q = scale sum_q w lambda lambda / D(q), D the thickness at the triangle rule's points.
template <typename C>
__device__ __forceinline__ void coupling_q(C scale, const C dz[3], C Q[6]) {
#pragma unroll
  for (int i = 0; i < 6; ++i) Q[i] = (C)0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const C inv = (C)kTw[q] * recip((C)kL0[q] * dz[0] + (C)kL1[q] * dz[1] + (C)kL2[q] * dz[2]);
    Q[0] += (C)(kL0[q] * kL0[q]) * inv;
    Q[1] += (C)(kL1[q] * kL1[q]) * inv;
    Q[2] += (C)(kL2[q] * kL2[q]) * inv;
    Q[3] += (C)(kL0[q] * kL1[q]) * inv;
    Q[4] += (C)(kL0[q] * kL2[q]) * inv;
    Q[5] += (C)(kL1[q] * kL2[q]) * inv;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) Q[i] *= scale;
}
// Mz / (3 J_h)
template <typename C>
__device__ __forceinline__ void mass_third(const C dz[3], C mz[6]) {
  const C s = (C)(1.0 / 360.0);
  mz[0] = s * ((C)3 * dz[0] + dz[1] + dz[2]);
  mz[1] = s * (dz[0] + (C)3 * dz[1] + dz[2]);
  mz[2] = s * (dz[0] + dz[1] + (C)3 * dz[2]);
  mz[3] = s * (dz[0] + dz[1] + (C)0.5 * dz[2]);
  mz[4] = s * (dz[0] + dz[2] + (C)0.5 * dz[1]);
  mz[5] = s * (dz[1] + dz[2] + (C)0.5 * dz[0]);
}

// y -= D'^-T g with g = [Q s - t S s; -Q s] (above: the coupling C_{l-1}^T s) or
// [-Q s; Q s - t S s] (below: B_{l+1}^T s).
template <typename C>
__device__ __forceinline__ void sub_transposed(const M3<C>& TT, const M3<C>& TB, const M3<C>& BT, const M3<C>& BB,
                                               const C Q[6], const C s[3], C t, bool above, C y[6]) {
  const C sum = s[0] + s[1] + s[2];
  C q[3], g[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    q[i] = Q[sx(i, 0)] * s[0] + Q[sx(i, 1)] * s[1] + Q[sx(i, 2)] * s[2];
    g[i] = q[i] - t * (sum + s[i]);
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    C s0 = (C)0, s1 = (C)0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      s0 += above ? TT.m[j][i] * g[j] - BT.m[j][i] * q[j] : BT.m[j][i] * g[j] - TT.m[j][i] * q[j];
      s1 += above ? TB.m[j][i] * g[j] - BB.m[j][i] * q[j] : BB.m[j][i] * g[j] - TB.m[j][i] * q[j];
    }
    y[i] -= s0;
    y[i + 3] -= s1;
  }
}

// The value of the quad's lane (lane + Q) mod 3; lane 3 gets what lane 2 gets.
template <int Q>
__device__ __forceinline__ int quad_rot(int x) {
  constexpr int perm = Q == 1 ? (1 | 2 << 2 | 0 << 4 | 0 << 6) : (2 | 0 << 2 | 1 << 4 | 1 << 6);
  return __builtin_amdgcn_mov_dpp(x, perm, 0xf, 0xf, true);
}
template <int Q>
__device__ __forceinline__ float quad_rot(float x) {
  return __int_as_float(quad_rot<Q>(__float_as_int(x)));
}
template <int Q>
__device__ __forceinline__ double quad_rot(double x) {
  return __hiloint2double(quad_rot<Q>(__double2hiint(x)), quad_rot<Q>(__double2loint(x)));
}

template <typename T>
__device__ __forceinline__ T ldo(const T* row, uint32_t byte_off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(row) + byte_off);
}
__device__ __forceinline__ void phase() { __builtin_amdgcn_sched_barrier(0); }

// LDS of a block of BT prisms: first the staged right-hand sides, a wave's rows
// [kRows][64] after another; then, over them, K or H as [9][kRow] and c or d as
// [3][NF][kRow].
template <typename S, typename C, int NF, int BT>
struct ColLds {
  static constexpr int kPer = 16 / (int)sizeof(S);              // prisms a lane copies at once
  static constexpr int kRows = (6 * NF + kPer - 1) / kPer * kPer;
  // the pad puts the rows that the chains' quads read together on different banks
  static constexpr int kRow = BT + 16 / (int)sizeof(C);
  static constexpr bool kThrough = NF >= 2 && sizeof(C) == 8;
  // a wavefront's part: room for its prisms' right-hand sides, or their y
  static constexpr int kWave = 64 * (kThrough && 6 * NF * sizeof(C) > kRows * sizeof(S) ? 6 * NF * (int)sizeof(C) : kRows * (int)sizeof(S));
  static constexpr int kStage = kWave * (BT / 64);
  static constexpr int kChain = (9 + 3 * NF) * kRow * (int)sizeof(C);
  static constexpr int kBytes = kStage > kChain ? kStage : kChain;
};

// w_e <- c_e - K_e w_(previous e) down or up a column: n values from slot e on
// with stride st.  A quad runs one chain: its lanes 0..2 hold the three
// components (lane 3 repeats lane 2), each with its row of K rotated so that its own
// component comes first and only two values a step cross lanes.  K and c are read
// NB - 1 steps ahead.
template <typename C, int NF, int kRow, int NB>
__device__ __forceinline__ void run_chain(const C* K, C* cc, int e, int f, int comp, int n, int st) {
  const int i = comp < 3 ? comp : 2;
  const C* k0 = K + (3 * i + i) * kRow + e;
  const C* k1 = K + (3 * i + (i + 1) % 3) * kRow + e;
  const C* k2 = K + (3 * i + (i + 2) % 3) * kRow + e;
  C* cr = cc + (i * NF + f) * kRow + e;
  C w = (C)0;
  C k[NB][3], c[NB];
  auto load = [&](int b, int j) {
    const int o = (j < n ? j : n - 1) * st;
    k[b][0] = k0[o];
    k[b][1] = k1[o];
    k[b][2] = k2[o];
    c[b] = cr[o];
  };
  auto step = [&](int b, int j) {
    const C r1 = quad_rot<1>(w), r2 = quad_rot<2>(w);
    w = c[b] - k[b][0] * w - k[b][1] * r1 - k[b][2] * r2;
    cr[j * st] = w;
  };
#pragma unroll
  for (int b = 0; b + 1 < NB; ++b) load(b, b);
  int j = 0;
  for (; j + NB - 1 < n; j += NB) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      load((b + NB - 1) % NB, j + b + NB - 1);
      step(b, j + b);
    }
  }
#pragma unroll
  for (int b = 0; b + 1 < NB; ++b)
    if (j + b < n) step(b, j + b);
}

template <typename C, int NF, int kRow>
__device__ __forceinline__ void clear_chain(C* K, C* cc, int slot) {
#pragma unroll
  for (int i = 0; i < 9; ++i) K[i * kRow + slot] = (C)0;
#pragma unroll
  for (int i = 0; i < 3 * NF; ++i) cc[i * kRow + slot] = (C)0;
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;
// 16 bytes a lane, global to LDS: lane i fills bytes [16 i, 16 i + 16) from dst (uniform).
__device__ __forceinline__ void copy16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)dst, 16, 0, 0);
}
// vmcnt(0): the wavefront's own copies have arrived.
__device__ __forceinline__ void wait_copies() {
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");
}

// A block's prisms, thread = (layer, column) with the columns fastest.  At least MW and
// at most MX wavefronts a SIMD.
template <typename S, typename C, int NF, bool TR, int BT, int MW, int MX>
__global__ __attribute__((amdgpu_flat_work_group_size(1, BT), amdgpu_waves_per_eu(MW, MX))) void
column_solve_kernel(ColSolveArgs a) {
  extern __shared__ __align__(16) char smem[];
  using Lds = ColLds<S, C, NF, BT>;
  constexpr int kRow = Lds::kRow;
  constexpr int kAhead = sizeof(C) == 8 && NF > 3 ? 2 : 3;   // three spill with four fields in double
  const DevMesh& m = a.m;
  const ColTile tile = a.tiles[xcd_tile((int)blockIdx.x, a.n_tiles)];
  const int tid = threadIdx.x;
  const int g = tile.log2cols;
  const int G = 1 << g;
  const int l = tid >> g;
  const int col = tid & (G - 1);
  const size_t SL = (size_t)m.n_slots;
  const S* Tst = static_cast<const S*>(a.Tstar);
  S* Tout = static_cast<S*>(a.Tout);

  // every wavefront copies its own prisms' right-hand sides to LDS; layers past the
  // cell's depth repeat the last (in bounds, unused)
  const int lane = tid & 63;
  char* wave = smem + __builtin_amdgcn_readfirstlane(tid >> 6) * Lds::kWave;
  S* stage = reinterpret_cast<S*>(wave + Lds::kWave) - Lds::kRows * 64;   // at the end of the wavefront's part
  // two fields or more in double: the y of a field waits in LDS, over right-hand sides
  // already read, until P is no longer held (held in registers, 13 of them spilled:
  // 860 us for 199,712 x 30 columns, 4 fields)
  constexpr bool kThrough = Lds::kThrough;
  C* yst = reinterpret_cast<C*>(wave) + lane;
  {
    constexpr int kPer = Lds::kPer, kLanes = 64 / kPer;
    const int q = (tid & ~63) + (lane & (kLanes - 1)) * kPer;
    const int ql = q >> g;
    const uint32_t src = (uint32_t)tile.base + (uint32_t)(ql < tile.depth ? ql : tile.depth - 1) * kCell + (uint32_t)(q & (G - 1));
    const int sub = lane / kLanes;
    if (a.aligned) {
#pragma unroll
      for (int k = 0; k < Lds::kRows / kPer; ++k) {
        const int r = k * kPer + sub < 6 * NF ? k * kPer + sub : 6 * NF - 1;
        copy16(Tst + (size_t)r * SL + src, stage + k * kPer * 64);
      }
    } else {
      const uint32_t own = (uint32_t)tile.base + (uint32_t)(l < tile.depth ? l : tile.depth - 1) * kCell + (uint32_t)col;
      for (int r = 0; r < 6 * NF; ++r) stage[r * 64 + lane] = Tst[(size_t)r * SL + own];
    }
  }

  const int cs = tile.col + col;
  const int N = m.nlay[cs];
  const bool live = l < N;
  C* chK = reinterpret_cast<C*>(smem);   // over the staged right-hand sides, once they are read
  C* chC = chK + 9 * kRow;
  const uint32_t p = (uint32_t)tile.base + (uint32_t)l * kCell + (uint32_t)col;
  const uint32_t po = p * (uint32_t)sizeof(S);

  // every block of the system carries J_h: it is left out
  C Q[6];                      // dt kappa_l Kv_l / 2
  C tu = (C)0, td = (C)0;     // dt sigma / 24 of the faces above and below
  M3<C> TT, TB, BT_, BB;     // D'_l^-1
  C mz[6];                      // mass block Mz / 3
  M3<C> P;                      // the kept P_l (zero in the surface layer)
  bool weak = false;            // a weak diffusion over dt (below)
  constexpr bool kCorrect = sizeof(S) == sizeof(C);
  if (live) {
    const size_t LS = (size_t)m.n_lslots;
    const uint32_t lt = (uint32_t)tile.lbase + (uint32_t)l * kCell + (uint32_t)col;
    const bool up = l > 0, dn = l + 1 < N;
    const uint32_t lu = up ? lt - kCell : lt, ld = dn ? lt + 2 * kCell : lt + kCell;
    C dz[3], hu = (C)0, hd = (C)0;
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      const double* zr = m.zl + v * LS;
      const double zt = ldo(zr, lt * 8u), zb = ldo(zr, (lt + kCell) * 8u);
      dz[v] = (C)(zt - zb);
      hu += (C)(ldo(zr, lu * 8u) - zt);
      hd += (C)(zb - ldo(zr, ld * 8u));
    }
    CPair<C> pp[5] = {};
    if (up) {
      const CPair<C>* __restrict__ Pk = reinterpret_cast<const CPair<C>*>(a.fac);
#pragma unroll
      for (int k = 0; k < 5; ++k) pp[k] = (Pk + (size_t)k * SL)[p];
    }
    const C dt = (C)a.dt, eta = (C)a.eta;
    const C kc = (C)a.kappa[l];
    const C third = (C)(1.0 / 3.0);
    const C h = (dz[0] + dz[1] + dz[2]) * third;
    hu *= third;
    hd *= third;
    const C pen = dt * eta * (C)(0.5 / 24.0);
    if (up) tu = pen * ((C)a.kappa[l - 1] + kc) * recip(hu < h ? hu : h);
    if (dn) td = pen * (kc + (C)a.kappa[l + 1]) * recip(h < hd ? h : hd);
    coupling_q((C)0.5 * dt * kc, dz, Q);
    weak = kCorrect && tu + td + (C)8 * Q[0] < (C)0.2 * h;
    mass_third(dz, mz);
    {
      // D'_l = [tt tb; bt bb]
      M3<C> tt, tb, bt, bb;
      const C fu = up ? (C)1 : (C)2, fd = dn ? (C)1 : (C)2;
      P = {{{(C)pp[0].lo, (C)pp[0].hi, (C)pp[1].lo}, {(C)pp[1].hi, (C)pp[2].lo, (C)pp[2].hi},
            {(C)pp[3].lo, (C)pp[3].hi, (C)pp[4].lo}}};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const C ps = (C)1 + (P.m[i][0] + P.m[i][1] + P.m[i][2]);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const C mm = mz[sx(i, j)], q = Q[sx(i, j)];
          const C pq = P.m[i][0] * Q[sx(0, j)] + P.m[i][1] * Q[sx(1, j)] + P.m[i][2] * Q[sx(2, j)];
          const C e = i == j ? (C)1 : (C)0;
          tt.m[i][j] = (C)2 * mm + fu * q - pq + tu * (ps + P.m[i][j] + e);
          tb.m[i][j] = mm - fu * q + pq;
          bt.m[i][j] = mm - fd * q;
          bb.m[i][j] = (C)2 * mm + fd * q + td * ((C)1 + e);
        }
      }
      const M3<C> ai = inv3(tt);
      const M3<C> x1 = mul3(ai, tb);
      const M3<C> y1 = mul3(bt, ai);
      BB = inv3(sub_mul3(bb, bt, x1));
      TB = neg3(mul3(x1, BB));
      BT_ = neg3(mul3(BB, y1));
      TT = sub_mul3(ai, x1, BT_);
    }
  }
  wait_copies();
  // y = D'^-1 M T* (its transpose times M Z).  Where the diffusion over dt is
  // weak (kappa dt / dz^2 below about 0.3 at the usual penalty) it is formed as
  // T* + D'^-1 (M - D') T*, whose products are small against T*: 3 to 5 times
  // nearer to the exact solution than D'^-1 (M T*); in stiff layers the second
  // rounds like an LU and the first up to 10 times worse.  A float result of the
  // double solve rounds far above either.
  C y[NF][6];
  if (live) {
    const C fu = l > 0 ? (C)1 : (C)2, fd = l + 1 < N ? (C)1 : (C)2;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C t[6], r[6], h[3], q[3];
      phase();
#pragma unroll
      for (int i = 0; i < 6; ++i) t[i] = (C)stage[(f * 6 + i) * 64 + lane];
      if (!kCorrect || !weak) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const C at = mz[sx(i, 0)] * t[0] + mz[sx(i, 1)] * t[1] + mz[sx(i, 2)] * t[2];
          const C ab = mz[sx(i, 0)] * t[3] + mz[sx(i, 1)] * t[4] + mz[sx(i, 2)] * t[5];
          r[i] = (C)2 * at + ab;
          r[i + 3] = at + (C)2 * ab;
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) t[i] = (C)0;
      } else if (TR) {
        // h = P^T t_top; [-q - tu S (t_top + h); q - td S t_bottom], q = Q (fu t_top - fd t_bottom - h)
#pragma unroll
        for (int i = 0; i < 3; ++i) h[i] = P.m[0][i] * t[0] + P.m[1][i] * t[1] + P.m[2][i] * t[2];
        const C e0 = fu * t[0] - fd * t[3] - h[0], e1 = fu * t[1] - fd * t[4] - h[1], e2 = fu * t[2] - fd * t[5] - h[2];
        const C su = (t[0] + h[0]) + (t[1] + h[1]) + (t[2] + h[2]), sd = t[3] + t[4] + t[5];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          q[i] = Q[sx(i, 0)] * e0 + Q[sx(i, 1)] * e1 + Q[sx(i, 2)] * e2;
          r[i] = -q[i] - tu * (su + (t[i] + h[i]));
          r[i + 3] = q[i] - td * (sd + t[i + 3]);
        }
      } else {
        // [-(fu q + tu S t_top) + P (q - tu S t_top); fd q - td S t_bottom], q = Q (t_top - t_bottom)
        const C e0 = t[0] - t[3], e1 = t[1] - t[4], e2 = t[2] - t[5];
        const C su = t[0] + t[1] + t[2], sd = t[3] + t[4] + t[5];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          q[i] = Q[sx(i, 0)] * e0 + Q[sx(i, 1)] * e1 + Q[sx(i, 2)] * e2;
          const C g = tu * (su + t[i]);
          h[i] = q[i] - g;
          r[i] = -fu * q[i] - g;
          r[i + 3] = fd * q[i] - td * (sd + t[i + 3]);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) r[i] += P.m[i][0] * h[0] + P.m[i][1] * h[1] + P.m[i][2] * h[2];
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        C s0 = (C)0, s1 = (C)0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          s0 += (TR ? TT.m[j][i] : TT.m[i][j]) * r[j];
          s1 += (TR ? TB.m[j][i] : BT_.m[i][j]) * r[j];
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          s0 += (TR ? BT_.m[j][i] : TB.m[i][j]) * r[j + 3];
          s1 += (TR ? BB.m[j][i] : BB.m[i][j]) * r[j + 3];
        }
        y[f][i] = t[i] + s0;
        y[f][i + 3] = t[i + 3] + s1;
      }
      if constexpr (kThrough) {
#pragma unroll
        for (int i = 0; i < 6; ++i) yst[(f * 6 + i) * 64] = y[f][i];
        asm volatile("" ::: "memory");
      }
    }
    if constexpr (kThrough) {
      phase();
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 6; ++i) y[f][i] = yst[(f * 6 + i) * 64];
    }
  }
  auto store = [&](int f) {
#pragma unroll
    for (int i = 0; i < 6; ++i)
      *reinterpret_cast<S*>(reinterpret_cast<char*>(Tout + (size_t)(f * 6 + i) * SL) + po) = (S)y[f][i];
  };
  // a block of one wavefront holds columns of one layer: x = y (without the rest, FP64,
  // 512 such columns of 1 field 4.8 -> 3.9 us, 51,200 of 4 fields 7.8 -> 7.0)
  if constexpr (BT == kCell) {
    if (live)
#pragma unroll
      for (int f = 0; f < NF; ++f) store(f);
    return;
  }
  phase();
  __syncthreads();   // the chain arrays take the staging space
  // prisms that feed no other get K = 0 and c = 0 (below a column's seabed for
  // good), so that all chains run over the cell's depth
  if (live && l + 1 < N) {
    const M3<C> K = TR ? couple3(Q, TB, BB, tu, TB) : couple3(Q, BT_, TT, td, BT_);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) chK[(i * 3 + j) * kRow + tid] = TR ? K.m[j][i] : K.m[i][j];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C cc[3];
      phase();
      if (!TR) couple_v(Q, y[f] + 3, y[f], td, y[f] + 3, cc);
#pragma unroll
      for (int i = 0; i < 3; ++i) chC[(i * NF + f) * kRow + tid] = TR ? y[f][i + 3] : cc[i];
    }
  } else {
    clear_chain<C, NF, kRow>(chK, chC, tid);
  }
  phase();
  __syncthreads();
  // w <- c - K w from the surface down; slot l then holds layer l + 1's input
  const int nch = tile.depth - 1;
  if (nch > 0)
    for (int q = tid >> 2; q < G * NF; q += BT / 4)
      run_chain<C, NF, kRow, kAhead>(chK, chC, q / NF, q % NF, tid & 3, nch, G);
  __syncthreads();
  phase();
  if (live && l > 0) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C u[3];
      phase();
#pragma unroll
      for (int i = 0; i < 3; ++i) u[i] = chC[(i * NF + f) * kRow + tid - G];
      if (TR) sub_transposed(TT, TB, BT_, BB, Q, u, tu, true, y[f]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if (!TR) {
          y[f][i] -= TT.m[i][0] * u[0] + TT.m[i][1] * u[1] + TT.m[i][2] * u[2];
          y[f][i + 3] -= BT_.m[i][0] * u[0] + BT_.m[i][1] * u[1] + BT_.m[i][2] * u[2];
        }
      }
    }
  }
  __syncthreads();
  phase();
  if (live && l > 0) {
    const M3<C> H = TR ? couple3(Q, BT_, TT, td, BT_) : couple3(Q, TB, BB, tu, TB);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) chK[(i * 3 + j) * kRow + tid] = TR ? H.m[j][i] : H.m[i][j];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      C d[3];
      phase();
      if (!TR) couple_v(Q, y[f], y[f] + 3, tu, y[f], d);
#pragma unroll
      for (int i = 0; i < 3; ++i) chC[(i * NF + f) * kRow + tid] = TR ? y[f][i] : d[i];
    }
  }
  phase();
  __syncthreads();
  // the same from the seabed up; slot l then holds layer l - 1's input
  if (nch > 0)
    for (int q = tid >> 2; q < G * NF; q += BT / 4)
      run_chain<C, NF, kRow, kAhead>(chK, chC, q / NF + nch * G, q % NF, tid & 3, nch, -G);
  __syncthreads();
  phase();
  if (live) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if (l + 1 < N) {
        C v[3];
        phase();
#pragma unroll
        for (int i = 0; i < 3; ++i) v[i] = chC[(i * NF + f) * kRow + tid + G];
        if (TR) sub_transposed(TT, TB, BT_, BB, Q, v, td, false, y[f]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          if (!TR) {
            y[f][i] -= TB.m[i][0] * v[0] + TB.m[i][1] * v[1] + TB.m[i][2] * v[2];
            y[f][i + 3] -= BB.m[i][0] * v[0] + BB.m[i][1] * v[1] + BB.m[i][2] * v[2];
          }
        }
      }
      store(f);
    }
  }
}

// The kept P_l = B_l D'_{l-1}^-1 [:, bottom] of all layers, one lane per column and one
// wavefront per cell of 64 columns: the recurrence is serial, and bound by the chain
// of its some 450 operations a layer at one wavefront per SIMD or less.  The pivots
// are inverted by 3x3 blocks as in the solve above and only the blocks that P needs
// are formed; against a sweep with the LU of the 6x6 pivots (vsolve.hip's), double,
// 49,928 x 20 columns 62 -> 43 us, 4,418 x 13 24.7 -> 14.5, 199,712 x 30 211 -> 139;
// float, 60 ragged layers, 93 -> 92.
template <typename C>
struct FactorLayer {
  C dz[3], h;
};

template <typename C>
__global__ __launch_bounds__(64) void column_factor_kernel(ColFactorArgs a) {
  const DevMesh& m = a.m;
  const int cell = m.cell_order[blockIdx.x];   // deepest cells first
  const int lane = threadIdx.x;
  const int N = m.nlay[cell * kCell + lane];
  if (N == 0) return;
  const size_t SL = (size_t)m.n_slots, LS = (size_t)m.n_lslots;
  const size_t p0 = (size_t)m.cell_base[cell] + lane, lt0 = (size_t)m.cell_lbase[cell] + lane;
  CPair<C>* __restrict__ Pk = reinterpret_cast<CPair<C>*>(a.fac);
  const C dt = (C)a.dt;
  const C pen = dt * (C)a.eta * (C)(0.5 / 24.0);
  auto load = [&](int l, FactorLayer<C>& g) {
    const size_t lt = lt0 + (size_t)(l < N ? l : N - 1) * kCell;
#pragma unroll
    for (int v = 0; v < 3; ++v) g.dz[v] = (C)(m.zl[v * LS + lt] - m.zl[v * LS + lt + kCell]);
  };
  auto mean = [](FactorLayer<C>& g) { g.h = (g.dz[0] + g.dz[1] + g.dz[2]) * (C)(1.0 / 3.0); };
  FactorLayer<C> g0, g1, g2;       // layers l, l + 1, l + 2
  load(0, g0);
  load(1, g1);
  mean(g0);
  M3<C> P = {};
  C tu = (C)0;
  // the heights and kappa are read two layers ahead
  auto kap = [&](int l) { return (C)a.kappa[l < N ? l : N - 1]; };
  C kc = kap(0), kn = kap(1);
  for (int l = 0; l + 1 < N; ++l) {
    load(l + 2, g2);
    const C kn2 = kap(l + 2);
    mean(g1);
    const C td = pen * (kc + kn) * recip(g0.h < g1.h ? g0.h : g1.h);
    C Q[6], mz[6];
    coupling_q((C)0.5 * dt * kc, g0.dz, Q);
    mass_third(g0.dz, mz);
    // D'_l = [tt tb; bt bb] (a layer below exists); its inverse's right blocks
    const C fu = l > 0 ? (C)1 : (C)2;
    M3<C> tt, tb, bt, bb;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const C ps = (C)1 + (P.m[i][0] + P.m[i][1] + P.m[i][2]);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const C mm = mz[sx(i, j)], q = Q[sx(i, j)];
        const C pq = P.m[i][0] * Q[sx(0, j)] + P.m[i][1] * Q[sx(1, j)] + P.m[i][2] * Q[sx(2, j)];
        const C e = i == j ? (C)1 : (C)0;
        tt.m[i][j] = (C)2 * mm + fu * q - pq + tu * (ps + P.m[i][j] + e);
        tb.m[i][j] = mm - fu * q + pq;
        bt.m[i][j] = mm - q;
        bb.m[i][j] = (C)2 * mm + q + td * ((C)1 + e);
      }
    }
    const M3<C> x1 = mul3(inv3(tt), tb);
    const M3<C> BB = inv3(sub_mul3(bb, bt, x1));
    const M3<C> TB = neg3(mul3(x1, BB));
    P = couple3(Q, BB, TB, td, BB);
    const size_t p = p0 + (size_t)(l + 1) * kCell;
#pragma unroll
    for (int k = 0; k < 5; ++k)
      Pk[(size_t)k * SL + p] =
          CPair<C>{P.m[(2 * k) / 3][(2 * k) % 3], k < 4 ? P.m[(2 * k + 1) / 3][(2 * k + 1) % 3] : (C)0};
    tu = td;
    kc = kn;
    kn = kn2;
    g0 = g1;
    g1 = g2;
  }
}

template <typename S, typename C, int NF, bool TR, int BT>
hipError_t launch_block(const ColSolveArgs& a, hipStream_t s) {
  // three wavefronts per SIMD (168 registers): at two the solve of 2,454,178 prisms
  // with three fields takes 413 us against 322; at four it spills (49,928 x 20 columns,
  // one field: 93 us against 64).  The float solve fits five.
  constexpr int MW = 3;
  constexpr size_t lds = ColLds<S, C, NF, BT>::kBytes;
  // Columns of two layers, and no more wavefronts than SIMDs: one wavefront a SIMD, as
  // the dispatcher would put a CU's second block of two on the SIMDs of its first
  // (22,050 x 2 columns, FP64 4 fields 13.2 -> 10.7 us, 1 field 7.5 -> 6.3).  Blocks of four
  // wavefronts spread by themselves.
  if constexpr (BT == 2 * kCell && !TR) {
    if (a.n_tiles * (BT / kCell) <= 4 * a.n_cu) {
      hipLaunchKernelGGL((column_solve_kernel<S, C, NF, TR, BT, 1, 1>), dim3(a.n_tiles), dim3(BT), lds, s, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((column_solve_kernel<S, C, NF, TR, BT, MW, 8>), dim3(a.n_tiles), dim3(BT), lds, s, a);
  return hipGetLastError();
}

// Blocks of the fewest wavefronts that hold the mesh's largest column group.
template <typename S, typename C, int NF, bool TR>
hipError_t launch_block(const ColSolveArgs& a, hipStream_t s) {
  if (a.max_np <= 64) return launch_block<S, C, NF, TR, 64>(a, s);
  if (a.max_np <= 128) return launch_block<S, C, NF, TR, 128>(a, s);
  if (a.max_np <= 192) return launch_block<S, C, NF, TR, 192>(a, s);
  return launch_block<S, C, NF, TR, 256>(a, s);
}

template <typename S, typename C, bool TR>
hipError_t launch_nf(const ColSolveArgs& a, hipStream_t s) {
  switch (a.n_fields) {
    case 1: return launch_block<S, C, 1, TR>(a, s);
    case 2: return launch_block<S, C, 2, TR>(a, s);
    case 3: return launch_block<S, C, 3, TR>(a, s);
    case 4: return launch_block<S, C, 4, TR>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_column_factor(const ColFactorArgs& a, bool fp32_solve, hipStream_t s) {
  if (a.m.n_cells == 0) return hipSuccess;
  if (fp32_solve) hipLaunchKernelGGL(column_factor_kernel<float>, dim3(a.m.n_cells), dim3(kCell), 0, s, a);
  else hipLaunchKernelGGL(column_factor_kernel<double>, dim3(a.m.n_cells), dim3(kCell), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_column_solve(const ColSolveArgs& a, bool fp32_state, bool fp32_solve, bool transposed,
                               hipStream_t s) {
  if (a.n_tiles == 0) return hipSuccess;
  if (a.max_np > kColSolveMaxPrisms) return hipErrorInvalidValue;
  if (transposed) return fp32_state ? hipErrorInvalidValue : launch_nf<double, double, true>(a, s);
  if (!fp32_state) return launch_nf<double, double, false>(a, s);
  return fp32_solve ? launch_nf<float, float, false>(a, s) : launch_nf<float, double, false>(a, s);
}

}  // namespace sdg
