// Device code of the line kernels (see tc_line.hip for the layout and the
// rule that selects them): one wave's lane layout, the banded substitution
// over a line, and the three kernels built on it.  Included once per number
// of lanes per slot (tc_line_*.hip), each compiled by itself.
#pragma once
#include <atomic>

#include "tc_internal.h"
#include "tc_solve_dev.h"

namespace tc {
namespace {

constexpr int NLANE = 64;  // lanes per wave
// Waves per workgroup: four, one per SIMD, share the stencil table; one on
// grids of few waves, which then have a CU's LDS and L1 each to themselves.
constexpr int WAVES = 4;
constexpr int LINE_SPREAD_WAVES = 512;

typedef double dbl2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ cd z0() { return cd{0.0, 0.0}; }
__device__ __forceinline__ cd fmac(cd acc, double w, cd v) { return cd{fma(w, v.x, acc.x), fma(w, v.y, acc.y)}; }
__device__ __forceinline__ cd nfmac(cd acc, double w, cd v) { return cd{fma(-w, v.x, acc.x), fma(-w, v.y, acc.y)}; }
__device__ __forceinline__ cd scl(cd v, double w) { return cd{v.x * w, v.y * w}; }
// i * w * v
__device__ __forceinline__ cd imul(cd v, double w) { return cd{-w * v.y, w * v.x}; }

// ------------------------------------------------------------------ moves between the lanes of a line
// A slot's LPS lanes are consecutive and aligned, so up to 16 lanes they lie
// within one DPP row and every move is a VALU instruction; 32 lanes go
// through ds_bpermute.
template <int CTRL> __device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
// value of the lane DIST before (DIR > 0) or after (DIR < 0) this one
// (garbage where that is outside the line)
template <int LPS, int DIR, int DIST> __device__ __forceinline__ double from(double v) {
  if constexpr (LPS <= 16) return dpp<(DIR > 0 ? 0x110 : 0x100) + DIST>(v);  // row_shr, row_shl
  else if constexpr (DIR > 0) return __shfl_up(v, DIST, NLANE);
  else return __shfl_down(v, DIST, NLANE);
}
template <int LPS, int DIR, int DIST> __device__ __forceinline__ cd from(cd v) {
  return cd{from<LPS, DIR, DIST>(v.x), from<LPS, DIR, DIST>(v.y)};
}
// Copies a workgroup's per-row table to LDS, all loads issued before any is
// used (COUNT loads per lane serve a workgroup of one wave).
template <int COUNT> struct TableCopy {
  double v[(COUNT + NLANE - 1) / NLANE];
  __device__ __forceinline__ void load(const double* __restrict__ src) {
#pragma unroll
    for (int k = 0; k < (COUNT + NLANE - 1) / NLANE; ++k) {
      const int i = threadIdx.x + k * blockDim.x;
      if (i < COUNT) v[k] = src[i];
    }
  }
  __device__ __forceinline__ void store(double* dst) const {
#pragma unroll
    for (int k = 0; k < (COUNT + NLANE - 1) / NLANE; ++k) {
      const int i = threadIdx.x + k * blockDim.x;
      if (i < COUNT) dst[i] = v[k];
    }
    __syncthreads();
  }
};
// Orders this wave's LDS accesses where one lane reads what another wrote.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ one line
template <int LPS, int RPL> struct Line {
  static constexpr int BLK = LPS * RPL * NFAC;  // doubles of one (operator, mode) block of flin
  using Coef = double[RPL][4];
  using Rows = cd[RPL];

  // Window of a field around the lane's rows: w[i] holds row RPL k - 4 + i
  // of the lane's slot, zero outside the line.
  static __device__ __forceinline__ void halo(const Rows& x, cd (&w)[RPL + 2 * HW], int ch) {
#pragma unroll
    for (int i = 0; i < HW; ++i) {
      const cd lo = from<LPS, 1, 1>(x[RPL - HW + i]);
      const cd hi = from<LPS, -1, 1>(x[i]);
      w[i] = ch == 0 ? z0() : lo;
      w[RPL + HW + i] = ch == LPS - 1 ? z0() : hi;
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) w[HW + r] = x[r];
  }

  // D1 (or its transpose, by the table) of a windowed field at the lane's row r
  static __device__ __forceinline__ cd d1_at(const double* tab, int ch, int r, const cd (&w)[RPL + 2 * HW]) {
    cd s = z0();
#pragma unroll
    for (int m = 0; m < NB9; ++m) s = fmac(s, tab[(r * LINE_TAB_F + m) * LPS + ch], w[r + m]);
    return s;
  }

  // Coefficients of kind 0 (L) or 1 (U scaled by the inverse pivots), and
  // the inverse pivots, of one block
  static __device__ __forceinline__ void load_coef(const double* blk, int kind, Coef& m) {
    const double* base = blk + kind * RPL * 4 * LPS;
#pragma unroll
    for (int p = 0; p < RPL; ++p)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const dbl2 v = *reinterpret_cast<const dbl2*>(base + (2 * p + h) * 2 * LPS);
        m[p][2 * h] = v.x;
        m[p][2 * h + 1] = v.y;
      }
  }

  // one level of the scan of sweep(): distance DIST
  template <int DIR, int DIST>
  static __device__ __forceinline__ void scan(cd (&g)[4], double (&T)[4][4], int pos) {
    if constexpr (DIST < LPS) {
      constexpr bool last = 2 * DIST >= LPS;
      cd gs[4];
      double Ts[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) gs[i] = from<LPS, DIR, DIST>(g[i]);
      if constexpr (!last) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) Ts[i][e] = from<LPS, DIR, DIST>(T[i][e]);
      }
      if (pos >= DIST) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < 4; ++c) g[i] = fmac(g[i], T[i][c], gs[c]);
        if constexpr (!last) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            double t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              t[e] = T[i][0] * Ts[0][e];
#pragma unroll
              for (int c = 1; c < 4; ++c) t[e] = fma(T[i][c], Ts[c][e], t[e]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) T[i][e] = t[e];
          }
        }
      }
      scan<DIR, 2 * DIST>(g, T, pos);
    }
  }

  // One substitution along the line, y_i = f_i - sum_{c<4} m_i[c] y_{i-1-c},
  // rows ascending (DIR > 0) or descending; f is overwritten.
  template <int DIR> static __device__ __forceinline__ void sweep(const Coef& m, Rows& f, int ch) {
    const int pos = DIR > 0 ? ch : LPS - 1 - ch;
    // local pass from a zero incoming state: g = last 4 outputs (newest
    // first), T[i][e] = their dependence on incoming value e
    cd g[4] = {z0(), z0(), z0(), z0()};
    double T[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) T[i][e] = (i == e) ? 1.0 : 0.0;
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int p = DIR > 0 ? q : RPL - 1 - q;
      cd v = f[p];
      double w[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 3; c >= 0; --c) {
        if (c < q) v = nfmac(v, m[p][c], g[c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // outputs older than the lane's first row are the incoming values themselves
          if (c >= q) w[e] = (e == c - q) ? w[e] - m[p][c] : w[e];
          else w[e] = fma(-m[p][c], T[c][e], w[e]);
        }
      }
#pragma unroll
      for (int c = 3; c >= 1; --c) {
        g[c] = g[c - 1];
#pragma unroll
        for (int e = 0; e < 4; ++e) T[c][e] = T[c - 1][e];
      }
      g[0] = v;
#pragma unroll
      for (int e = 0; e < 4; ++e) T[0][e] = w[e];
    }
    // inclusive scan of the maps over the line: after the level of distance
    // d a lane holds the composition over itself and the 2d - 1 lanes before it
    scan<DIR, 1>(g, T, pos);
    // incoming state: the outputs of the preceding lane; then the lane's rows
    cd y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const cd t = from<LPS, DIR, 1>(g[i]);
      y[i] = pos == 0 ? z0() : t;
    }
#pragma unroll
    for (int q = 0; q < RPL; ++q) {
      const int p = DIR > 0 ? q : RPL - 1 - q;
      cd v = f[p];
#pragma unroll
      for (int c = 3; c >= 0; --c) v = nfmac(v, m[p][c], y[c]);
#pragma unroll
      for (int c = 3; c >= 1; --c) y[c] = y[c - 1];
      y[0] = v;
      f[p] = v;
    }
  }

  // Coefficients of the transposed recurrence in direction DIR from those of
  // the rows before in it, the nearest rows of the preceding lane included.
  template <int DIR> static __device__ __forceinline__ void transpose(const Coef& m, Coef& t, int ch) {
    const bool first = ch == (DIR > 0 ? 0 : LPS - 1);
#pragma unroll
    for (int p = 0; p < RPL; ++p)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int q = DIR > 0 ? p - 1 - c : p + 1 + c;
        if (q >= 0 && q < RPL) {
          t[p][c] = m[q][c];
        } else {
          const double v = from<LPS, DIR, 1>(m[DIR > 0 ? RPL + q : q - RPL][c]);
          t[p][c] = first ? 0.0 : v;
        }
      }
  }

  // Solves with operators in turn, f in the operator's own row order (that
  // of its factorisation: ascending for P, descending, i.e. mirrored, for
  // the Helmholtz operators).  The first sweep's coefficients load while the
  // operator before runs its second sweep, the second's during the first.
  struct Solver {
    Coef first;
    const double* fl;  // the lane's mode in flin, operator 0
    int64_t fop;       // doubles between operators
    int ch;
    template <bool TR> __device__ __forceinline__ void prefetch(int op) {
      load_coef(fl + op * fop, TR ? 1 : 0, first);
    }
    // A x = f (TR: A^T x = f up to the row scale of P), f in place; nop: the
    // operator of the next call (< 0: none)
    template <bool TR> __device__ __forceinline__ void solve(int op, int nop, Rows& f) {
      Coef second;
      double piv[RPL];
      load_coef(fl + op * fop, TR ? 0 : 1, second);
#pragma unroll
      for (int p = 0; p < RPL; ++p) piv[p] = fl[op * fop + 8 * RPL * LPS - ch + p * LPS];
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (TR) {
        Coef t;
        transpose<1>(first, t, ch);
        sweep<1>(t, f, ch);
      } else {
        sweep<1>(first, f, ch);
      }
#pragma unroll
      for (int p = 0; p < RPL; ++p) f[p] = scl(f[p], piv[p]);
      __builtin_amdgcn_sched_barrier(0);
      if (nop >= 0) prefetch<TR>(nop);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (TR) {
        Coef t;
        transpose<-1>(second, t, ch);
        sweep<-1>(t, f, ch);
      } else {
        sweep<-1>(second, f, ch);
      }
    }
  };
};

// Lane of a wave: the slot's mode and the rows RPL ch .. RPL ch + RPL - 1.
// Tiles of 16 SPW distinct modes x 2 axial signs (32 waves) are dispatched
// consecutively to one XCD, so the two slots of a mode, which
// read the same factors, go through the same L2.
template <int LPS, int RPL> struct LineLane {
  static constexpr int SPW = NLANE / LPS;  // slots (distinct modes) per wave
  int lane, wv, ch, dmc, n, labs, sign, j0;
  bool reg, nyq, zero_mode;
  int64_t o, onyq;
  double a, b;
  __device__ __forceinline__ bool make(const Dims& d, int ntile, int per) {
    lane = threadIdx.x % NLANE;
    wv = threadIdx.x / NLANE;
    ch = lane % LPS;
    const int nw = blockDim.x / NLANE, wgs = 32 / nw;  // workgroups per tile
    const int x = blockIdx.x % 8, rr = blockIdx.x / 8;
    const int t = x * per + rr / wgs, q = rr % wgs;
    if (t >= ntile) return false;
    sign = q & 1;
    const int dm = (t * 16 + (q >> 1) * nw + wv) * SPW + lane / LPS;
    const bool active = dm < d.ndm;
    if (__ballot(active) == 0) return false;
    dmc = active ? dm : d.ndm - 1;
    labs = dmc / d.mt;
    n = dmc - labs * d.mt;
    // a lane of sign -1 at |l| = 0 keeps the empty axial slot (l = -m_z/2) of
    // its n at zero; it and the lanes past the last mode compute on slot 0's
    // data (the wave's moves need every lane) and store nothing else
    nyq = active && sign == 1 && labs == 0;
    reg = active && !nyq;
    const int s = sign ? d.mz - labs : labs;
    o = reg ? (int64_t)s * d.mt + n : 0;
    onyq = (int64_t)d.nyq * d.mt + n;
    a = n * d.kt;
    b = (sign ? -labs : labs) * d.kz;
    zero_mode = labs == 0 && n == 0;
    j0 = RPL * ch;
    return true;
  }
  // plane offset of row r, clamped to the last node: rows past it carry
  // zero coefficients everywhere and are never stored
  __device__ __forceinline__ int64_t row(const Dims& d, int r) const {
    const int j = j0 + r, M = d.n_r - 1;
    return (int64_t)(j < M ? j : M) * d.S;
  }
};

}  // namespace

// Predictor-corrector of one step with the line on chip.  What bounds it: one
// wave per SIMD (its four fields fill the LDS and the coefficients of two
// sweeps the registers), so on small grids the chain of loads and
// substitutions, and on larger ones the state and factors, 19 fields and 36
// doubles per distinct mode-row: 64 x 64 x 128 moves 235 MB in 55 us, 4.3 TB/s.
template <int LPS, int RPL>
__global__ __launch_bounds__(WAVES * NLANE) void k_pcl(const double* __restrict__ rc, const double* __restrict__ flin,
                                                      const double* __restrict__ ltab, Dims d, const cd* __restrict__ u, const cd* up,
                                                      const cd* __restrict__ N, const cd* __restrict__ Np, cd* un,
                                                      cd* p, int want_p, cd* omg, int ntile, int per) {
  using L = Line<LPS, RPL>;
  // each wave's lines: Helmholtz right-hand sides, then u*, then u^{i+1}
  // (3 fields), and p*; each lane touches only its own entries
  extern __shared__ __align__(16) unsigned char lds_raw[];
  cd* const fld = reinterpret_cast<cd*>(lds_raw);
  double* const tab = reinterpret_cast<double*>(fld + (blockDim.x / NLANE) * 4 * RPL * NLANE);
  const int M = d.n_r - 1;
  TableCopy<RPL * LINE_TAB_F * LPS> tc;
  tc.load(ltab);
  tc.store(tab);
  LineLane<LPS, RPL> q;
  if (!q.make(d, ntile, per)) return;
  const int ch = q.ch, j0 = q.j0;
  const int64_t F = d.F, S = d.S, o = q.o;
  const double a = q.a, b = q.b;
  auto TAB = [&](int f, int r) { return tab[(r * LINE_TAB_F + f) * LPS + ch]; };
  auto V = [&](int c, int r) -> cd& { return fld[((q.wv * 4 + c) * RPL + r) * NLANE + q.lane]; };
  // row r of the line from its other end
  const int mlane = q.lane - ch + LPS - 1 - ch;
  auto VM = [&](int c, int r) -> cd& { return fld[((q.wv * 4 + c) * RPL + RPL - 1 - r) * NLANE + mlane]; };
  typename L::Solver sv;
  sv.fl = flin + (int64_t)q.dmc * L::BLK + 2 * q.ch;
  sv.fop = (int64_t)d.ndm * L::BLK;
  sv.ch = ch;
  if (q.nyq) {
    for (int j = j0; j < j0 + RPL && j <= M; ++j) {
      const int64_t oj = j * S + q.onyq;
      un[oj] = un[F + oj] = un[2 * F + oj] = z0();
      if (want_p) p[oj] = z0();
      if (omg) omg[oj] = omg[F + oj] = omg[2 * F + oj] = z0();
    }
  }
  cd w[RPL + 2 * HW];
  typename L::Rows f;

  // 1. Ne = 2 N^i - N^{i-1}; the pressure right-hand side -D(Ne) with the
  //    consistent Neumann rows at the walls, V_r(2 u^i - u^{i-1}) there with
  //    V_r = (L+ u+ + L- u-)/2; the part of the Helmholtz right-hand sides
  //    that does not hold p* (in fld)
  {
    const double c_dt = 1.0 / (2.0 * d.dt);
    typename L::Rows er, l;
    cd bc0 = z0(), bcM = z0();
    // the loads of N, then of u, are issued together: a lane waits for
    // memory twice, not once per row
    cd xv[RPL][3], yv[RPL][3];
    auto load2 = [&](const cd* x, const cd* y) {
#pragma unroll
      for (int r = 0; r < RPL; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int64_t oj = q.row(d, r) + o + c * F;
          xv[r][c] = x[oj];
          yv[r][c] = y[oj];
        }
    };
    load2(N, Np);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      cd e3[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        e3[c] = csub(scl(xv[r][c], 2.0), yv[r][c]);
        V(c, r) = e3[c];
      }
      const double ir = TAB(LINE_TAB_IR, r);
      er[r] = scl(cadd(e3[0], e3[1]), 0.5);
      cd lr = scl(er[r], ir);
      lr = fmac(lr, 0.5 * a * ir, csub(e3[0], e3[1]));
      l[r] = cadd(lr, imul(e3[2], b));
    }
    __builtin_amdgcn_sched_barrier(0);
    load2(u, up);
    sv.template prefetch<false>(OP_P);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = j0 + r;
      const cd sum = csub(scl(cadd(xv[r][0], xv[r][1]), 2.0), cadd(yv[r][0], yv[r][1]));
      bc0 = fmac(bc0, TAB(LINE_TAB_W0, r), sum);
      bcM = fmac(bcM, TAB(LINE_TAB_WM, r), sum);
      if (j == 0 || j == M) {
        const cd dif = csub(csub(scl(xv[r][0], 2.0), yv[r][0]), csub(scl(xv[r][1], 2.0), yv[r][1]));
        const double ir2 = rc[(int64_t)j * RC_N + RC_IR2];
        cd t = scl(sum, 0.5 * (-(a * a + 1.0) * ir2 - b * b));
        t = fmac(t, -a * ir2, dif);
        if (j == 0) bc0 = cadd(bc0, t);
        else bcM = cadd(bcM, t);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const cd ut = csub(scl(xv[r][c], 4.0), yv[r][c]);
        const cd e = V(c, r);
        V(c, r) = cd{e.x - ut.x * c_dt, e.y - ut.y * c_dt};
      }
    }
    // the 5 rows next to the outer wall may begin in the lane before
    const cd bp = from<LPS, 1, 1>(bcM);
    bcM = ch == 0 ? bcM : cadd(bcM, bp);
    L::halo(er, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = j0 + r;
      const cd acc = cadd(L::d1_at(tab, ch, r, w), l[r]);
      f[r] = cd{-acc.x, -acc.y};
      if (j == 0) f[r] = scl(csub(bc0, er[r]), d.s0);
      if (j == M) f[r] = q.zero_mode ? z0() : scl(csub(bcM, er[r]), d.sM);
    }
  }

  // 2.-4. the five solves in turn: p* (P), u* (H+, H-, H_z), phi (P); one
  //    copy of the code, which fits the instruction cache
#pragma unroll 1
  for (int k = 0; k < 5; ++k) {
    if (k == 4) {
      // P phi = D(u*), homogeneous Neumann rows
      typename L::Rows ur, l;
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const cd x0 = V(0, r), x1 = V(1, r), x2 = V(2, r);
        const double ir = TAB(LINE_TAB_IR, r);
        ur[r] = scl(cadd(x0, x1), 0.5);
        cd lr = scl(ur[r], ir);
        lr = fmac(lr, 0.5 * a * ir, csub(x0, x1));
        l[r] = cadd(lr, imul(x2, b));
      }
      L::halo(ur, w, ch);
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        f[r] = cadd(L::d1_at(tab, ch, r, w), l[r]);
        if (j0 + r == 0 || j0 + r == M) f[r] = z0();
      }
    } else if (k > 0) {
#pragma unroll
      for (int r = 0; r < RPL; ++r) f[r] = VM(k - 1, r);
    }
    sv.template solve<false>(k < 4 ? k : OP_P, k < 3 ? k + 1 : (k == 3 ? OP_P : -1), f);
    if (k == 0) {
      // p* (kept for the update) and its gradient in the Helmholtz
      // right-hand sides; their wall rows hold the boundary values
      L::halo(f, w, ch);
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const int j = j0 + r;
        const double ir = TAB(LINE_TAB_IR, r);
        const cd d1 = L::d1_at(tab, ch, r, w);
        const cd pi = f[r];
        V(3, r) = pi;
        cd h0 = cadd(V(0, r), nfmac(d1, a * ir, pi));
        cd h1 = cadd(V(1, r), fmac(d1, a * ir, pi));
        cd h2 = cadd(V(2, r), imul(pi, b));
        if (j == 0 || j == M) {
          const double Re = j == 0 ? d.Re_i : d.Re_o;
          h0 = q.zero_mode ? cd{0.0, Re} : z0();
          h1 = q.zero_mode ? cd{0.0, -Re} : z0();
          h2 = z0();
        }
        V(0, r) = h0;
        V(1, r) = h1;
        V(2, r) = h2;
      }
    } else if (k < 4) {
#pragma unroll
      for (int r = 0; r < RPL; ++r) VM(k - 1, r) = f[r];
    }
    wave_lds_fence();
  }

  // 5. correction u^{i+1} = u* - grad phi, p = p* + 3 phi / (2 dt)
  //    (mode (0,0): the correction removes u*_r, the exact solution of the
  //    correction equation for that mode)
  {
    const double c_p = 1.5 / d.dt;
    L::halo(f, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int64_t oj = q.row(d, r) + o;
      const double ir = TAB(LINE_TAB_IR, r);
      const cd d1 = L::d1_at(tab, ch, r, w);
      const cd ph = f[r];
      const cd x0 = V(0, r), x1 = V(1, r), x2 = V(2, r);
      cd v0 = csub(x0, nfmac(d1, a * ir, ph));
      cd v1 = csub(x1, fmac(d1, a * ir, ph));
      const cd v2 = csub(x2, imul(ph, b));
      if (q.zero_mode) {
        v0 = scl(csub(x0, x1), 0.5);
        v1 = cd{-v0.x, -v0.y};
      }
      if (q.reg && j0 + r <= M) {
        un[oj] = v0;
        un[F + oj] = v1;
        un[2 * F + oj] = v2;
        if (want_p) p[oj] = fmac(V(3, r), c_p, ph);
      }
      V(0, r) = v0;
      V(1, r) = v1;
      V(2, r) = v2;
    }
  }

  // 6. omega = curl u^{i+1} for the next step's nonlinear term
  if (omg) {
    typename L::Rows xr, dp, dmn;
#pragma unroll
    for (int r = 0; r < RPL; ++r) xr[r] = V(0, r);
    L::halo(xr, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) dp[r] = L::d1_at(tab, ch, r, w);
#pragma unroll
    for (int r = 0; r < RPL; ++r) xr[r] = V(1, r);
    L::halo(xr, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) dmn[r] = L::d1_at(tab, ch, r, w);
#pragma unroll
    for (int r = 0; r < RPL; ++r) xr[r] = V(2, r);
    L::halo(xr, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int64_t oj = q.row(d, r) + o;
      const double ir = TAB(LINE_TAB_IR, r);
      const cd dz = L::d1_at(tab, ch, r, w);
      const cd upv = V(0, r), umv = V(1, r), uzv = xr[r];
      // omega+ = i (a/r uz - D1 uz) - b u+ ;  omega- = i (a/r uz + D1 uz) + b u-
      const cd tp = {a * ir * uzv.x - dz.x, a * ir * uzv.y - dz.y};
      const cd tm = {a * ir * uzv.x + dz.x, a * ir * uzv.y + dz.y};
      const cd op = {-tp.y - b * upv.x, tp.x - b * upv.y};
      const cd om = {-tm.y + b * umv.x, tm.x + b * umv.y};
      // omega_z = -(i/2) [ (D1 + (1+a)/r) u+ - (D1 + (1-a)/r) u- ]
      const cd qz = {dp[r].x + (1.0 + a) * ir * upv.x - dmn[r].x - (1.0 - a) * ir * umv.x,
                     dp[r].y + (1.0 + a) * ir * upv.y - dmn[r].y - (1.0 - a) * ir * umv.y};
      if (q.reg && j0 + r <= M) {
        omg[oj] = op;
        omg[F + oj] = om;
        omg[2 * F + oj] = cd{0.5 * qz.y, -0.5 * qz.x};
      }
    }
  }
}

// Solves A x = rhs (or, transposed, A^T x = rhs) on their own: operators
// op0 .. op0 + nop - 1 on fields rhs + k F -> x + k F (x may alias rhs: each
// lane reads its rows before it writes them).
template <int LPS, int RPL>
__global__ __launch_bounds__(WAVES * NLANE) void k_solve_l(const double* __restrict__ flin, Dims d, int op0, int nop,
                                                          int transposed, const cd* rhs, cd* x, int ntile, int per) {
  using L = Line<LPS, RPL>;
  LineLane<LPS, RPL> q;
  if (!q.make(d, ntile, per)) return;
  const int M = d.n_r - 1;
  typename L::Solver sv;
  sv.fl = flin + (int64_t)q.dmc * L::BLK + 2 * q.ch;
  sv.fop = (int64_t)d.ndm * L::BLK;
  sv.ch = q.ch;
#pragma unroll 1
  for (int k = 0; k < nop; ++k) {
    const int op = op0 + k;
    typename L::Rows f;
    // f holds the line in the operator's row order: node of row r
    auto node = [&](int r) { return op == OP_P ? q.j0 + r : RPL * LPS - 1 - (q.j0 + r); };
    // the Neumann rows 0 and M of P are scaled (row M of mode (0,0) is
    // Dirichlet): A = S^-1 L U, so rhs is scaled before a solve and x after
    // a transposed one
    auto scale_walls = [&]() {
      if (op != OP_P) return;
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        if (q.j0 + r == 0) f[r] = scl(f[r], d.s0);
        if (q.j0 + r == M && !q.zero_mode) f[r] = scl(f[r], d.sM);
      }
    };
    const cd* src = rhs + k * d.F + q.o;
#pragma unroll
    for (int r = 0; r < RPL; ++r) f[r] = src[(int64_t)(node(r) < M ? node(r) : M) * d.S];
    if (transposed) {
      sv.template prefetch<true>(op);
      sv.template solve<true>(op, -1, f);
      scale_walls();
    } else {
      sv.template prefetch<false>(op);
      scale_walls();
      sv.template solve<false>(op, -1, f);
    }
    cd* dst = x + k * d.F;
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      if (node(r) > M) continue;
      if (q.reg) dst[node(r) * d.S + q.o] = f[r];
      if (q.nyq) dst[node(r) * d.S + q.onyq] = z0();
    }
  }
}

// Backward error of the line solves: k_factor_check (tc_solve.hip) with the
// copy of the factors and the sweeps across lanes that the other kernels here
// use.  The right-hand side and the residual are formed on chip, so the kernel
// reads the copy and little else.
template <int LPS, int RPL>
__global__ __launch_bounds__(WAVES * NLANE) void k_check_l(const double* __restrict__ rc, const double* __restrict__ flin,
                                                          Dims d, unsigned long long* worst, int ntile, int per) {
  using L = Line<LPS, RPL>;
  extern __shared__ double x0s[];
  const int M = d.n_r - 1;
  for (int j = threadIdx.x; j <= M; j += blockDim.x) x0s[j] = 1.0 + 0.5 * sin(0.7 * j);
  __syncthreads();
  LineLane<LPS, RPL> q;
  if (!q.make(d, ntile, per) || q.sign) return;  // the slots +l and -l share their factors
  typename L::Solver sv;
  sv.fl = flin + (int64_t)q.dmc * L::BLK + 2 * q.ch;
  sv.fop = (int64_t)d.ndm * L::BLK;
  sv.ch = q.ch;
  double err = 0.0;
  bool bad = false;
#pragma unroll 1
  for (int op = 0; op < NOPS; ++op) {
    auto node = [&](int r) { return op == OP_P ? q.j0 + r : RPL * LPS - 1 - (q.j0 + r); };
    typename L::Rows f;
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = node(r);
      double s = 0.0;
      if (j <= M) {
        double row[NB9];
        operator_row(rc, d, op, j, q.a, q.b, row);
#pragma unroll
        for (int k = 0; k < NB9; ++k) {
          const int i = j + k - HW;
          if (i >= 0 && i <= M) s = fma(row[k], x0s[i], s);
        }
      }
      f[r] = cd{s, 0.0};
    }
    double rhs[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) rhs[r] = f[r].x;
    sv.template prefetch<false>(op);
    sv.template solve<false>(op, -1, f);
    cd w[RPL + 2 * HW];
    L::halo(f, w, q.ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = node(r);
      if (j > M) continue;
      double row[NB9];
      operator_row(rc, d, op, j, q.a, q.b, row);
      double s = 0.0, den = 0.0;
#pragma unroll
      for (int k = 0; k < NB9; ++k) {
        const double x = op == OP_P ? w[r + k].x : w[r + 2 * HW - k].x;
        s = fma(row[k], x, s);
        den = fma(fabs(row[k]), fabs(x), den);
      }
      den += fabs(rhs[r]);
      const double e = den > 0.0 ? fabs(s - rhs[r]) / den : 0.0;
      bad = bad || !(e <= 1.0);
      err = fmax(err, e);
    }
  }
  if (bad) err = 1.0;  // a non-finite residual counts as the worst
  for (int off = 32; off > 0; off >>= 1) err = fmax(err, __shfl_xor(err, off));
  if (q.lane == 0) atomicMax(worst, (unsigned long long)__double_as_longlong(err));
}

// Adjoint of the predictor-corrector on the line layout: the chain of the
// adjoint step (tc_adjoint.hip) from the cotangent u_bar' of u^{i+1} and
// N_bar of N^i to the cotangents of u^i, u^{i-1}, N^{i-1} and the total
// cotangent of N(u^i), with every intermediate on chip:
//   phi_bar = -grad^H u_bar' (0 for mode (0,0))      r_phi = P^-T phi_bar
//   u*_bar = u_bar' + div^H(I r_phi)                 r_u = H^-T u*_bar
//   p_bar = grad^H(I r_u)                            r_p = P^-T p_bar
//   Ne_bar = I r_u - div^H(I r_p) - (W r_p)/2
//   u_bar = -(2/dt) I r_u + 2 V,  u_prev_bar = I r_u/(2dt) - V,
//   V = (L+^T W r_p, L-^T W r_p)/2 (zero past HW rows from the walls)
//   N_prev_bar = -Ne_bar,  N_tot = 2 Ne_bar + N_bar
// (I: interior rows, W: the wall rows of the consistent Neumann condition,
// not the outer row of mode (0,0)).  D1^T sums, for row k, the D1 weights
// of rows k-4 .. k+4 in column k, in that order; the per-row table holds
// those transposed weights.
template <int LPS, int RPL>
__global__ __launch_bounds__(WAVES * NLANE) void k_pcl_adj(const double* __restrict__ rc,
                                                          const double* __restrict__ flin,
                                                          const double* __restrict__ ltab, Dims d,
                                                          const cd* __restrict__ ub, const cd* __restrict__ nin,
                                                          cd* __restrict__ out_u, cd* __restrict__ out_up,
                                                          cd* __restrict__ out_np, cd* __restrict__ ntot, int ntile,
                                                          int per) {
  using L = Line<LPS, RPL>;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  cd* const fld = reinterpret_cast<cd*>(lds_raw);
  double* const tab = reinterpret_cast<double*>(fld + (blockDim.x / NLANE) * 3 * RPL * NLANE);
  const int M = d.n_r - 1;
  TableCopy<RPL * LINE_TAB_F * LPS> tc;
  tc.load(ltab);
  tc.store(tab);
  LineLane<LPS, RPL> q;
  if (!q.make(d, ntile, per)) return;
  const int ch = q.ch, j0 = q.j0;
  const int64_t F = d.F, S = d.S, o = q.o;
  const double a = q.a, b = q.b;
  auto IR = [&](int r) { return tab[(r * LINE_TAB_F + LINE_TAB_IR) * LPS + ch]; };
  auto V = [&](int c, int r) -> cd& { return fld[((q.wv * 3 + c) * RPL + r) * NLANE + q.lane]; };
  // row r of the line from its other end
  const int mlane = q.lane - ch + LPS - 1 - ch;
  auto VM = [&](int c, int r) -> cd& { return fld[((q.wv * 3 + c) * RPL + RPL - 1 - r) * NLANE + mlane]; };
  auto interior = [&](int r) { return j0 + r != 0 && j0 + r < M; };
  typename L::Solver sv;
  sv.fl = flin + (int64_t)q.dmc * L::BLK + 2 * q.ch;
  sv.fop = (int64_t)d.ndm * L::BLK;
  sv.ch = ch;
  sv.template prefetch<true>(OP_P);
  if (q.nyq) {
    for (int j = j0; j < j0 + RPL && j <= M; ++j)
      for (int c = 0; c < 3; ++c) {
        const int64_t oj = c * F + j * S + q.onyq;
        out_u[oj] = out_up[oj] = out_np[oj] = ntot[oj] = z0();
      }
  }
  cd w[RPL + 2 * HW];
  typename L::Rows f;
#pragma unroll
  for (int r = 0; r < RPL; ++r) {
    const int64_t oj = q.row(d, r) + o;
#pragma unroll
    for (int c = 0; c < 3; ++c) V(c, r) = ub[c * F + oj];
  }
  // r_phi (P), r_u (H+, H-, H_z), r_p (P) in turn
#pragma unroll 1
  for (int k = 0; k < 5; ++k) {
    if (k == 0 || k == 4) {
      // grad^H v = D1^T (v+ + v-) - (a/r) v+ + (a/r) v- - i b v_z, of u_bar'
      // (negated: phi_bar) and of I r_u (p_bar)
      typename L::Rows sm;
#pragma unroll
      for (int r = 0; r < RPL; ++r) sm[r] = cadd(V(0, r), V(1, r));
      L::halo(sm, w, ch);
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        cd g = L::d1_at(tab, ch, r, w);
        g = cadd(g, scl(csub(V(1, r), V(0, r)), a * IR(r)));
        g = csub(g, imul(V(2, r), b));
        if (k == 0) g = q.zero_mode ? z0() : cd{-g.x, -g.y};
        f[r] = g;
      }
    } else {
#pragma unroll
      for (int r = 0; r < RPL; ++r) f[r] = VM(k - 1, r);
    }
    sv.template solve<true>(k < 4 ? k : OP_P, k < 3 ? k + 1 : (k == 3 ? OP_P : -1), f);
    if (k == 0) {
      // u*_bar = u_bar' + div^H(I r_phi) (mode (0,0): the transpose of
      // u^{i+1}+- = u*+- - u*_r maps (v+, v-) to ((v+ - v-)/2, (v- - v+)/2))
#pragma unroll
      for (int r = 0; r < RPL; ++r)
        if (!interior(r)) f[r] = z0();
      L::halo(f, w, ch);
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const double ir = IR(r);
        const cd dt = scl(L::d1_at(tab, ch, r, w), 0.5);
        const cd v0 = V(0, r), v1 = V(1, r);
        cd vp = v0, vm = v1;
        if (q.zero_mode) {
          vp = scl(csub(v0, v1), 0.5);
          vm = cd{-vp.x, -vp.y};
        }
        V(0, r) = cadd(vp, cadd(dt, scl(f[r], 0.5 * (1.0 + a) * ir)));
        V(1, r) = cadd(vm, cadd(dt, scl(f[r], 0.5 * (1.0 - a) * ir)));
        V(2, r) = csub(V(2, r), imul(f[r], b));
      }
    } else if (k < 4) {
#pragma unroll
      for (int r = 0; r < RPL; ++r) {  // I r_u
        const int j = RPL * LPS - 1 - (j0 + r);
        VM(k - 1, r) = (j != 0 && j < M) ? f[r] : z0();
      }
    }
    wave_lds_fence();
  }
  // Ne_bar, the cotangents of u^i, u^{i-1}, N^{i-1} and N_tot
  {
    const double c_dt = 1.0 / d.dt;
    // W r_p: the wall rows of r_p, scaled like x = S v (not row M of mode
    // (0,0)), known to the lanes whose rows lie in the wall rows' stencils
    cd w0 = z0(), wM = z0();
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      if (j0 + r == 0) w0 = scl(f[r], d.s0);
      if (j0 + r == M && !q.zero_mode) wM = scl(f[r], d.sM);
    }
    const cd wn = from<LPS, -1, 1>(wM);
    if (ch < LPS - 1 && j0 + RPL <= M) wM = wn;
#pragma unroll
    for (int r = 0; r < RPL; ++r)
      if (!interior(r)) f[r] = z0();
    L::halo(f, w, ch);
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int j = j0 + r;
      if (j > M) continue;
      const int64_t oj = (int64_t)j * S + o;
      const double ir = IR(r);
      const cd dt = scl(L::d1_at(tab, ch, r, w), 0.5);
      cd ne[3] = {V(0, r), V(1, r), V(2, r)};  // I r_u
      cd ou[3], oup[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ou[c] = scl(ne[c], -2.0 * c_dt);
        oup[c] = scl(ne[c], 0.5 * c_dt);
      }
      ne[0] = csub(ne[0], cadd(dt, scl(f[r], 0.5 * (1.0 + a) * ir)));
      ne[1] = csub(ne[1], cadd(dt, scl(f[r], 0.5 * (1.0 - a) * ir)));
      ne[2] = cadd(ne[2], imul(f[r], b));
      if (j <= HW || j >= M - HW) {
        const cd wj = j == 0 ? w0 : (j == M ? wM : z0());
        ne[0] = csub(ne[0], scl(wj, 0.5));
        ne[1] = csub(ne[1], scl(wj, 0.5));
        // L+-^T w = D2^T w + D1^T(w / r) - (a^2/r^2 + b^2 + (1 +- 2a)/r^2) w
        cd base = z0();
#pragma unroll
        for (int ws = 0; ws < 2; ++ws) {
          const int jw = ws ? M : 0, kk = j - jw + HW;  // place of row j in the wall row's stencil
          if (kk < 0 || kk >= NB9) continue;
          const double* Rw = rc + (int64_t)jw * RC_N;
          const cd wv = ws ? wM : w0;
          base = fmac(base, Rw[RC_W2 + kk], wv);
          base = fmac(base, Rw[RC_W1 + kk], scl(wv, Rw[RC_IR]));
        }
        const double ir2 = rc[(int64_t)j * RC_N + RC_IR2];
        const double dd = a * a * ir2 + b * b;
        const cd vp = scl(csub(base, scl(wj, dd + (1.0 + 2.0 * a) * ir2)), 0.5);
        const cd vm = scl(csub(base, scl(wj, dd + (1.0 - 2.0 * a) * ir2)), 0.5);
        ou[0] = cadd(ou[0], scl(vp, 2.0));
        ou[1] = cadd(ou[1], scl(vm, 2.0));
        oup[0] = csub(oup[0], vp);
        oup[1] = csub(oup[1], vm);
      }
      if (q.reg) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          out_u[c * F + oj] = ou[c];
          out_up[c * F + oj] = oup[c];
          out_np[c * F + oj] = cd{-ne[c].x, -ne[c].y};
          ntot[c * F + oj] = cadd(scl(ne[c], 2.0), nin[c * F + oj]);
        }
      }
    }
  }
}

namespace {

struct LineGrid {
  dim3 grid, block;
  int ntile, per, nw;
};
template <int LPS> LineGrid line_grid(const Dims& d) {
  constexpr int SPW = NLANE / LPS;
  const int ntile = (d.ndm + 16 * SPW - 1) / (16 * SPW);
  const int per = (ntile + 7) / 8;
  const int nw = ntile * 32 <= LINE_SPREAD_WAVES ? 1 : WAVES;
  return {dim3(8 * per * (32 / nw)), dim3(nw * NLANE), ntile, per, nw};
}

// LDS of a workgroup holding nf fields of each of its waves' lines
template <int LPS, int RPL> size_t line_lds(int nw, int nf) {
  return (size_t)nw * nf * RPL * NLANE * sizeof(cd) + (size_t)RPL * LINE_TAB_F * LPS * sizeof(double);
}
// lets the kernel take that much LDS, once per device
template <int LPS, int RPL, int NF, typename K> hipError_t lds_limit(K kernel, std::atomic<uint64_t>& devices, int dev) {
  const uint64_t bit = (uint64_t)1 << (dev & 63);
  if (devices.load(std::memory_order_relaxed) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)line_lds<LPS, RPL>(WAVES, NF));
  if (e == hipSuccess) devices.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

template <int LPS, int RPL> hipError_t run_pcl(tc_ctx* c, const LineArgs& x) {
  const LineGrid g = line_grid<LPS>(c->d);
  static std::atomic<uint64_t> pc_devices{0}, adj_devices{0};
  hipError_t e = hipSuccess;
  switch (x.what) {
    case LINE_PC:
      e = lds_limit<LPS, RPL, 4>(&k_pcl<LPS, RPL>, pc_devices, c->device);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((k_pcl<LPS, RPL>), g.grid, g.block, (line_lds<LPS, RPL>(g.nw, 4)), c->stream, c->rc_dev, c->flin,
                         c->ltab, c->d, x.in[0], x.in[1], x.in[2], x.in[3], x.out[0], x.out[1], x.flag, x.out[2], g.ntile, g.per);
      break;
    case LINE_SOLVE:
      hipLaunchKernelGGL((k_solve_l<LPS, RPL>), g.grid, g.block, 0, c->stream, c->flin, c->d, x.op0, x.nop, x.flag,
                         x.in[0], x.out[0], g.ntile, g.per);
      break;
    case LINE_CHECK:
      hipLaunchKernelGGL((k_check_l<LPS, RPL>), g.grid, g.block, c->d.n_r * sizeof(double), c->stream, c->rc_dev, c->flin,
                         c->d, x.worst, g.ntile, g.per);
      break;
    case LINE_ADJ:
      e = lds_limit<LPS, RPL, 3>(&k_pcl_adj<LPS, RPL>, adj_devices, c->device);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((k_pcl_adj<LPS, RPL>), g.grid, g.block, (line_lds<LPS, RPL>(g.nw, 3)), c->stream, c->rc_dev,
                         c->flin, c->ltab + (size_t)RPL * LINE_TAB_F * LPS, c->d, x.in[0], x.in[1], x.out[0], x.out[1], x.out[2],
                         x.out[3], g.ntile, g.per);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int LPS> hipError_t run_rpl(tc_ctx* c, const LineArgs& x) {
  switch (line_shape(c->d).rpl) {
    case 5: return run_pcl<LPS, 5>(c, x);
    case 6: return run_pcl<LPS, 6>(c, x);
    case 7: return run_pcl<LPS, 7>(c, x);
    case 8: return run_pcl<LPS, 8>(c, x);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace tc
