// Predictor-corrector of one step with every radial line held on chip
// (Sec. 3.2, steps 2-5): the solves, stencils and update of the four-sweep
// kernels of tc_solve.hip, with a slot's line spread over LPS lanes (a power
// of two), RPL consecutive rows (5 to 8) on each.  The four-sweep kernels
// have one lane per mode: on small and medium grids too few to hide the
// latency of their radial chains, and everywhere they pass the step's
// intermediates through HBM.
//
// Work decomposition: LPS lanes per axial slot of a distinct mode (|l|, n),
// 64 / LPS slots of consecutive distinct modes per wave.  Lane k of a slot
// holds rows RPL k .. RPL k + RPL - 1 of every radial field of that slot, in
// registers and LDS, so the step's intermediates (Ne, p*, the Helmholtz
// right-hand sides, u*, phi) never leave the chip: the kernel reads u^i,
// u^{i-1}, N^i, N^{i-1} and the factors once and writes u^{i+1}, p and, when
// asked, the curl of u^{i+1} that the next step's nonlinear term needs.  A
// load of one row across a wave reads 64 / LPS consecutive slots: whole
// cache lines from LPS = 8 down.  Rows past the last node (RPL LPS > n_r)
// have zero coefficients and are never stored.
//
// Banded substitutions across lanes: a sweep of the unpivoted LU factors is
// a linear recurrence of order 4 along the rows (each output depends on the
// 4 previous ones in the sweep's order).  Each lane runs the recurrence over
// its rows from a zero incoming state, which gives the affine map (T, g)
// from the 4 values it receives to the 4 it passes on; a Kogge-Stone scan of
// these maps over the slot's lanes (log2 LPS levels of DPP moves) gives
// every lane its true incoming state, and the lane runs its rows again from
// it.  The rows a lane finally computes are the sequential sweep's, up to
// the rounding of the incoming state.
//
// One copy of the sweeps: the factors are held as L D U^ (U^ = D^-1 U, unit
// diagonal), so every sweep, either factor's, is y_i = f_i - sum m_i[c]
// y_{i-1-c}, first up, then down the operator's own row order (a Helmholtz
// operator's line is read mirrored), and a transposed one takes its
// coefficients from the rows before.  The ten sweeps of a step then run one loop
// body of two sweeps, and a sweep's coefficients load while the one before it
// runs.
// (Written out, operator by operator, with the loads of each in front of it
// and the moves through LDS, a wave took 126 000 cycles for 64 rows on a
// small grid; it takes 79 000 now, 34 000 of them in the sweeps, whose
// instructions issue back to back.  k_pcl on 32 x 16 x 32: 43.5 -> 30 us; on
// 64 x 64 x 128, where it moves 235 MB, 61 -> 55 us.)
//
// Stencils (D1 over +-4 rows) take their 4 halo rows from the neighbouring
// lanes; the per-row stencil weights sit in LDS.
//
// The factors are a second, lane-contiguous copy of the ones the other
// solves use (flin, tc_internal.h).
#include "tc_internal.h"

namespace tc {

// Where the line kernels run, from the predictor-corrector group of both
// forms, with the curl, timed by events (about 3 us above the kernels' own
// times) over n_r = 16 .. 256 and planes of 16 x 32 to 512 x 1024 modes (us,
// line against four sweeps):
//   to 64 rows (8 lanes) everywhere: 32 against 150 (64 x 16 x 32), 58
//     against 222 (64 x 64 x 128), 4090 against 4700 to 5370 (64 x 512 x 1024);
//   to 128 rows (16 lanes) to 65536 distinct modes: 116 against 336
//     (100 x 64 x 128), 1920 against 2030 (100 x 256 x 512), but 7510
//     against 7070 (100 x 512 x 1024), where the sweeps stream whole cache
//     lines from HBM and have lanes enough to hide their chains;
//   to 256 rows (32 lanes) below 16384 distinct modes: 312 against 671
//     (200 x 64 x 128), 1330 against 1510 (256 x 96 x 320), but 5040 against
//     2980 (160 x 256 x 512): a wave's load of one row is two slots, 32
//     bytes, wide.
// Grids whose waves, of 64 lanes, are at most one for each SIMD with twice
// the lanes per slot take that many lanes of fewer rows, where it saves two
// rows or more (one saves nothing: 31.7 against 33.0 on 48 x 32 x 64) and the
// moves stay within 16 lanes: a wave then has 5 rows in the place of 8 to go
// through, and there are CUs enough.  8 -> 5 rows: 34.5 -> 26.8 (32 x 16 x
// 32), 38.6 -> 31.6 (64 x 16 x 32), 44.9 -> 40.6 (64 x 32 x 128); with two
// waves for each SIMD 55 -> 78 (64 x 64 x 128), with 32 lanes 51 -> 60 (128 x
// 32 x 64).
LineShape line_shape(const Dims& d) {
  LineShape s{0, 0};
  for (int lps = 2; lps <= LINE_LPS_MAX; lps *= 2)
    if (8 * lps >= d.n_r) {
      if ((lps == 16 && d.ndm > 65536) || (lps == 32 && d.ndm >= 16384)) return s;
      s.lps = lps;
      s.rpl = std::max(HW + 1, (d.n_r + lps - 1) / lps);
      if (lps <= 8 && (int64_t)d.ndm * 4 * lps <= 1024 * 64) {
        const int rpl = std::max(HW + 1, (d.n_r + 2 * lps - 1) / (2 * lps));
        if (rpl + 2 <= s.rpl) s = {2 * lps, rpl};
      }
      break;
    }
  return s;
}

std::vector<double> line_tables(const Dims& d, const std::vector<double>& rc) {
  const LineShape ln = line_shape(d);
  const int M = d.n_r - 1;
  std::vector<double> t((size_t)2 * ln.rpl * LINE_TAB_F * ln.lps, 0.0);
  auto R = [&](int j) { return &rc[(size_t)j * RC_N]; };
  for (int j = 0; j <= M; ++j) {
    const int k = j / ln.rpl, r = j % ln.rpl;
    auto put = [&](int which, int f, double x) {
      t[((size_t)(which * ln.rpl + r) * LINE_TAB_F + f) * ln.lps + k] = x;
    };
    for (int m = 0; m < NB9; ++m) {
      put(0, m, R(j)[RC_W1 + m]);
      // D1^T: entry m of row j multiplies row i = j + m - 4 and is D1[i][j]
      const int i = j + m - HW;
      if (i >= 0 && i <= M) put(1, m, R(i)[RC_W1 + (NB9 - 1 - m)]);
    }
    for (int which = 0; which < 2; ++which) put(which, LINE_TAB_IR, R(j)[RC_IR]);
    for (int w = 0; w < 2; ++w) {
      const int jw = w ? M : 0, m = j - jw + HW;
      if (m >= 0 && m < NB9)
        put(0, w ? LINE_TAB_WM : LINE_TAB_W0, 0.5 * (R(jw)[RC_W2 + m] + R(jw)[RC_W1 + m] * R(jw)[RC_IR]));
    }
  }
  return t;
}

static hipError_t run_line(tc_ctx* c, const LineArgs& x) {
  if (!c->flin_captured) {
    hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &s) != hipSuccess) (void)hipGetLastError();
    c->flin_captured = s != hipStreamCaptureStatusNone;
  }
  switch (line_shape(c->d).lps) {
    case 2: return run_line_2(c, x);
    case 4: return run_line_4(c, x);
    case 8: return run_line_8(c, x);
    case 16: return run_line_16(c, x);
    case 32: return run_line_32(c, x);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_pc_line(tc_ctx* c, const cd* u, const cd* u_prev, const cd* N, const cd* N_prev, cd* u_next,
                          cd* p, int want_p, cd* omg) {
  return run_line(c, LineArgs{LINE_PC, want_p, 0, 0, {u, u_prev, N, N_prev}, {u_next, p, omg, nullptr}});
}

hipError_t launch_solve_line(tc_ctx* c, int op0, int nop, int transposed, const cd* rhs, cd* x) {
  return run_line(c, LineArgs{LINE_SOLVE, transposed, op0, nop, {rhs}, {x}});
}

hipError_t launch_line_check(tc_ctx* c, unsigned long long* worst) {
  LineArgs x{};
  x.what = LINE_CHECK;
  x.worst = worst;
  return run_line(c, x);
}

hipError_t launch_pc_adj_line(tc_ctx* c, const cd* ub, const cd* nin, cd* out_u, cd* out_up, cd* out_np, cd* ntot) {
  return run_line(c, LineArgs{LINE_ADJ, 0, 0, 0, {ub, nin}, {out_u, out_up, out_np, ntot}});
}

}  // namespace tc
