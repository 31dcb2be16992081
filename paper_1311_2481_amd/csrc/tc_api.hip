// C-ABI entry points of libtc: context set-up (radial grid, FD weights,
// factorisation), state handling, the time-step driver and diagnostics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "tc_internal.h"

using namespace tc;

namespace tc {

tc_status fail(tc_ctx* c, tc_status s, const std::string& msg) {
  if (c) c->err = msg;
  return s;
}

tc_status hip_check(tc_ctx* c, hipError_t e, const char* what) {
  if (e == hipSuccess) return TC_OK;
  return fail(c, TC_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

bool no_room(const char* what) {
  const char* e = std::getenv("TC_NO_ROOM");
  return e && std::strcmp(e, what) == 0;
}

hipError_t make_flin(tc_ctx* c) {
  const LineShape ln = line_shape(c->d);
  const char* off = std::getenv("TC_PC_LINE");
  if (ln.lps == 0 || (off && std::atoi(off) == 0) || no_room("lines")) return hipSuccess;
  const size_t fac = (size_t)NOPS * ln.lps * ln.rpl * NFAC * c->d.ndm;
  const size_t bytes = (fac + (size_t)2 * ln.rpl * LINE_TAB_F * ln.lps) * sizeof(double);
  void* p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return hipSuccess;
  }
  c->flin = static_cast<double*>(p);
  c->ltab = c->flin + fac;
  c->flin_bytes = bytes;
  c->bytes += bytes;
  const std::vector<double> tab = line_tables(c->d, c->rc);
  hipError_t e = hipMemcpyAsync(c->ltab, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = launch_factor_lines(c);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);  // tab ends here
  return e;
}

bool drop_flin(tc_ctx* c) {
  if (!c->flin || c->flin_captured) return false;
  if (hipStreamSynchronize(c->stream) != hipSuccess || hipFree(c->flin) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  c->flin = c->ltab = nullptr;
  c->bytes -= c->flin_bytes;
  return true;
}

void timer_begin(tc_ctx* c, int which) {
  if (!c->timing) return;
  KernelTimer& t = c->timers[which];
  t.open = false;
  if ((size_t)(t.used + 2) > t.ev.size()) {
    hipEvent_t a = nullptr, b = nullptr;
    if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
      if (a) (void)hipEventDestroy(a);
      (void)hipGetLastError();
      return;  // this launch goes untimed
    }
    t.ev.push_back(a);
    t.ev.push_back(b);
  }
  if (hipEventRecord(t.ev[t.used], c->stream) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  t.open = true;
}

void timer_end(tc_ctx* c, int which) {
  if (!c->timing) return;
  KernelTimer& t = c->timers[which];
  if (!t.open) return;
  t.open = false;
  if (hipEventRecord(t.ev[t.used + 1], c->stream) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  t.used += 2;
}

}  // namespace tc

namespace {

thread_local std::string g_init_error;

// ---------------------------------------------------------------- radial grid
// Nodes of eq. nodeDist with j = 0..M:  r_j = (1+eta)/(2(1-eta)) +
// asin(-alpha cos(pi j / M)) / (2 asin alpha), alpha -> 0 the Chebyshev
// limit.  -cos(pi j/M) is evaluated as sin(pi (j - M/2) / M), exact at the
// walls and odd about mid-gap.
std::vector<double> radial_nodes(int n_r, double eta, double alpha) {
  std::vector<double> r(n_r);
  const int M = n_r - 1;
  const long double centre = (1.0L + eta) / (2.0L * (1.0L - eta));
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int j = 0; j < n_r; ++j) {
    const long double x = std::sin(pi * ((long double)j - 0.5L * M) / (long double)M);
    long double v;
    if (alpha == 0.0)
      v = centre + 0.5L * x;
    else
      v = centre + std::asin((long double)alpha * x) / (2.0L * std::asin((long double)alpha));
    r[j] = (double)v;
  }
  return r;
}

// Finite-difference weights by Fornberg's recursion (Math. Comp. 51, 1988):
// delta[m][k][v] is the weight of node v for the m-th derivative using
// nodes 0..k; built up one node at a time.  Returns weights for m = 1, 2
// at z from the nodes x[0..n-1].
void fd_weights(double z, const double* x, int n, double* w1, double* w2) {
  const int MD = 2;
  std::vector<long double> delta((size_t)(MD + 1) * n * n, 0.0L);
  auto D = [&](int m, int k, int v) -> long double& { return delta[((size_t)m * n + k) * n + v]; };
  D(0, 0, 0) = 1.0L;
  long double c1 = 1.0L;
  for (int k = 1; k < n; ++k) {
    long double c2 = 1.0L;
    for (int v = 0; v < k; ++v) {
      const long double c3 = (long double)x[k] - x[v];
      c2 *= c3;
      for (int m = 0; m <= std::min(k, MD); ++m) {
        const long double prev = D(m, k - 1, v);
        const long double prevm = m > 0 ? D(m - 1, k - 1, v) : 0.0L;
        D(m, k, v) = (((long double)x[k] - z) * prev - m * prevm) / c3;
      }
    }
    for (int m = 0; m <= std::min(k, MD); ++m) {
      const long double prev = D(m, k - 1, k - 1);
      const long double prevm = m > 0 ? D(m - 1, k - 1, k - 1) : 0.0L;
      D(m, k, k) = c1 / c2 * (m * prevm - ((long double)x[k - 1] - z) * prev);
    }
    c1 = c2;
  }
  for (int v = 0; v < n; ++v) {
    w1[v] = (double)D(1, n - 1, v);
    w2[v] = (double)D(2, n - 1, v);
  }
}

template <typename T>
T* dev_alloc(tc_ctx* c, size_t bytes, tc_status& st) {
  void* p = nullptr;
  if (st != TC_OK) return nullptr;
  if (bytes == 0) bytes = 16;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    st = fail(c, TC_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    return nullptr;
  }
  c->bytes += bytes;
  return reinterpret_cast<T*>(p);
}

void dev_free(void* p) {
  if (p) (void)hipFree(p);
}

template <typename T>
void twiddles(int L, std::vector<C2<T>>& out) {
  out.resize(L);
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int e = 0; e < L; ++e) {
    const long double ang = -2.0L * pi * (long double)e / (long double)L;
    out[e] = C2<T>{(T)std::cos(ang), (T)std::sin(ang)};
  }
}

void free_ctx(tc_ctx* c) {
  if (!c) return;
  void* ptrs[] = {c->rc_dev, c->fac, c->flin, c->tw_t, c->tw_z, c->twf_t, c->twf_z, c->u, c->u_prev, c->N_prev,
                  c->N_cur, c->p, c->omega, c->aux, c->inter, c->zmax, c->diag_wr, c->diag_uc, c->red};
  for (void* p : ptrs) dev_free(p);
  for (auto& t : c->timers)
    for (auto e : t.ev) (void)hipEventDestroy(e);
  delete c;
}

// One evaluation of the nonlinear term in the convective form: the radial
// derivatives of u, then per plane batch the axial, azimuthal and forward
// axial passes over the 9-field intermediate.
tc_status nonlinear_conv(tc_ctx* c, const cd* u, cd* N) {
  hipError_t e = hipSuccess;
  c->omega_fresh = false;  // the curl buffer holds D1 u here
  timer_begin(c, TK_CURL);
  e = launch_dr(c, u, c->omega);
  timer_end(c, TK_CURL);
  if (e != hipSuccess) return hip_check(c, e, "radial derivatives");
  for (int p0 = 0; p0 < c->d.n_r; p0 += c->batch) {
    const int np = std::min(c->batch, c->d.n_r - p0);
    timer_begin(c, TK_ZINV);
    e = launch_zinv_conv(c, p0, np, u, c->omega);
    timer_end(c, TK_ZINV);
    if (e != hipSuccess) return hip_check(c, e, "axial inverse transform");
    timer_begin(c, TK_THETA);
    e = launch_theta_conv(c, p0, np);
    timer_end(c, TK_THETA);
    if (e != hipSuccess) return hip_check(c, e, "azimuthal transforms");
    timer_begin(c, TK_ZFWD);
    e = launch_zfwd(c, p0, np, N);
    timer_end(c, TK_ZFWD);
    if (e != hipSuccess) return hip_check(c, e, "axial forward transform");
  }
  return TC_OK;
}

// One evaluation of the nonlinear term: u -> N (both 3 fields).
tc_status nonlinear(tc_ctx* c, const cd* u, cd* N) {
  if (c->d.form == TC_CONVECTIVE) return nonlinear_conv(c, u, N);
  hipError_t e = hipSuccess;
  // the previous step's last sweep may already have formed curl(u)
  if (!(u == c->u && c->omega_fresh)) {
    timer_begin(c, TK_CURL);
    e = launch_curl(c, u, c->omega);
    timer_end(c, TK_CURL);
    if (e != hipSuccess) return hip_check(c, e, "curl");
  }
  c->omega_fresh = (u == c->u);
  for (int p0 = 0; p0 < c->d.n_r; p0 += c->batch) {
    const int np = std::min(c->batch, c->d.n_r - p0);
    timer_begin(c, TK_ZINV);
    e = launch_zinv(c, p0, np, u, c->omega);
    timer_end(c, TK_ZINV);
    if (e != hipSuccess) return hip_check(c, e, "axial inverse transform");
    timer_begin(c, TK_THETA);
    e = launch_theta(c, np);
    timer_end(c, TK_THETA);
    if (e != hipSuccess) return hip_check(c, e, "azimuthal transforms");
    timer_begin(c, TK_ZFWD);
    e = launch_zfwd(c, p0, np, N);
    timer_end(c, TK_ZFWD);
    if (e != hipSuccess) return hip_check(c, e, "axial forward transform");
  }
  return TC_OK;
}

size_t field_bytes(const tc_ctx* c) { return (size_t)c->d.F * sizeof(cd); }

}  // namespace

// ---------------------------------------------------------------- diagnostics kernels
namespace tc {

// Per-block partial sums of sum_j w_j r_j sum_{s,n} c_n e(j,s,n), where e is
// the energy density of u.
__global__ void k_energy(Dims d, const cd* __restrict__ u, const double* __restrict__ wr,
                         double* __restrict__ partial) {
  __shared__ double red[256];
  double acc = 0.0;
  const int64_t total = d.F;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(idx / d.S);
    const int64_t rem = idx - (int64_t)j * d.S;
    const int s = (int)(rem / d.mt), n = (int)(rem - (int64_t)s * d.mt);
    if (s == d.nyq) continue;
    const cd p = u[idx], m = u[d.F + idx], z = u[2 * d.F + idx];
    const double e = 0.5 * (p.x * p.x + p.y * p.y + m.x * m.x + m.y * m.y) + z.x * z.x + z.y * z.y;
    acc += (n == 0 ? 1.0 : 2.0) * wr[j] * e;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Partial results of the diagnostics, in one array of doubles: per
// workgroup (blocks along the slots, one per DIAG_ROWS radial nodes) the
// sums of the energy and the perturbation energy and the maximum of |div u|;
// the wall slip's sums of the workgroups at the inner wall; per node and block
// the three CFL mode sums; the theta-z mean of u_theta on every node.
// 32 blocks, doubled while they leave slots for a second round and the
// workgroups are fewer than 512 (two for each CU): with 32 throughout, 9 x 512
// x 1024 ran on 64 workgroups and took 640 us, 129 now (to 1024: 113, but 128 x
// 96 x 320 104 -> 107).  The partials are then
// those of fewer than 2 DIAG_GROUPS workgroups, with 32 blocks 109 n_r doubles
// at most.
constexpr int DIAG_BLOCKS = 32, DIAG_ROWS = 8, DIAG_THREADS = 256, DIAG_GROUPS = 512;
struct DiagLayout {
  int blocks, groups;
  size_t e, ep, dv, sl, cfl, mean, total;
};

__host__ __device__ inline DiagLayout diag_layout(const Dims& d) {
  DiagLayout L;
  const int rows = (d.n_r + DIAG_ROWS - 1) / DIAG_ROWS;
  L.blocks = DIAG_BLOCKS;
  while ((int64_t)L.blocks * DIAG_THREADS < d.S && L.blocks * rows < DIAG_GROUPS) L.blocks *= 2;
  L.groups = L.blocks * rows;
  L.e = 0;
  L.ep = L.e + L.groups;
  L.dv = L.ep + L.groups;
  L.sl = L.dv + L.groups;
  L.cfl = L.sl + L.blocks;
  L.mean = L.cfl + (size_t)d.n_r * L.blocks * 3;
  L.total = L.mean + d.n_r;
  return L;
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// All diagnostics of u in one pass: a thread takes DIAG_ROWS nodes of a slot,
// all its loads (those rows and the 4 on either side for D1) issued together,
// so u comes from HBM once.  (As separate kernels, the divergence one lane per
// slot down the whole radius, a call took 390 us on 128 x 96 x 320.)
__global__ __launch_bounds__(DIAG_THREADS) void k_diag(const double* __restrict__ rc, Dims d, const cd* __restrict__ u,
                                                       const double* __restrict__ wr, const double* __restrict__ Uc,
                                                       double* __restrict__ part) {
  constexpr int R = DIAG_ROWS, NW = DIAG_THREADS / 64;
  __shared__ double rows[NW][R][3];
  __shared__ double red[4][NW];
  const int M = d.n_r - 1, j0 = blockIdx.y * R, wv = threadIdx.x / 64, lane = threadIdx.x & 63;
  const int64_t F = d.F, S = d.S;
  if (lane < R)
    for (int k = 0; k < 3; ++k) rows[wv][lane][k] = 0.0;
  __syncthreads();  // lane 0 adds to what other lanes cleared
  const DiagLayout L = diag_layout(d);
  double E = 0.0, Ep = 0.0, sl = 0.0, dv = 0.0;
  for (int64_t base = (int64_t)blockIdx.x * DIAG_THREADS; base < S; base += (int64_t)L.blocks * DIAG_THREADS) {
    const int64_t idx = base + threadIdx.x;
    const int s = (int)(idx / d.mt), n = (int)(idx - (int64_t)s * d.mt);
    const bool in = idx < S && s != d.nyq;
    const double a = n * d.kt, b = (s < d.half ? s : s - d.mz) * d.kz, c = n == 0 ? 1.0 : 2.0;
    const bool zero = s == 0 && n == 0;
    cd p[R + 2 * HW], m[R + 2 * HW], z[R];
#pragma unroll
    for (int r = 0; r < R + 2 * HW; ++r) {
      const int j = j0 + r - HW, jj = j < 0 ? 0 : (j > M ? M : j);
      const int64_t o = jj * S + (in ? idx : 0);
      p[r] = u[o];
      m[r] = u[F + o];
      if (r >= HW && r < R + HW) z[r - HW] = u[2 * F + o];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = j0 + r;
      if (j > M) continue;
      const double* Rj = rc + (int64_t)j * RC_N;
      const cd pj = p[r + HW], mj = m[r + HW], zj = z[r];
      double s0 = 0.0, s1 = 0.0, s2 = 0.0;
      if (in) {
        const double w = c * wr[j];
        const double ez = zj.x * zj.x + zj.y * zj.y;
        E += w * (0.5 * (pj.x * pj.x + pj.y * pj.y + mj.x * mj.x + mj.y * mj.y) + ez);
        const double U = zero ? Uc[j] : 0.0, py = pj.y - U, my = mj.y + U;
        Ep += w * (0.5 * (pj.x * pj.x + py * py + mj.x * mj.x + my * my) + ez);
        // mode sums of |u_r|, |u_theta|, |u_z|: bounds of their plane maxima
        s0 = c * 0.5 * hypot(pj.x + mj.x, pj.y + mj.y);  // u_r = (u+ + u-)/2
        s1 = c * 0.5 * hypot(pj.x - mj.x, pj.y - mj.y);  // |u_theta| = |u+ - u-|/2
        s2 = c * hypot(zj.x, zj.y);
        if (j > 0 && j < M) {
          cd dr = {0.0, 0.0};
#pragma unroll
          for (int k = 0; k < NB9; ++k) {
            const double q = 0.5 * Rj[RC_W1 + k];
            dr.x = fma(q, p[r + k].x + m[r + k].x, dr.x);
            dr.y = fma(q, p[r + k].y + m[r + k].y, dr.y);
          }
          const double ir = Rj[RC_IR];
          const double vx = dr.x + 0.5 * (pj.x + mj.x) * ir + 0.5 * a * ir * (pj.x - mj.x) - b * zj.y;
          const double vy = dr.y + 0.5 * (pj.y + mj.y) * ir + 0.5 * a * ir * (pj.y - mj.y) + b * zj.x;
          dv = fmax(dv, sqrt(vx * vx + vy * vy));
        }
        if (j == 0) {
          // u_theta = -i (u+ - u-) / 2
          const double tx = 0.5 * (pj.y - mj.y) - (zero ? d.Re_i : 0.0), ty = -0.5 * (pj.x - mj.x);
          sl += c * (tx * tx + ty * ty + zj.x * zj.x + zj.y * zj.y);
        }
        // theta-z mean of u_theta: Re(-i (u+ - u-) / 2) of mode (0, 0)
        if (zero) part[L.mean + j] = 0.5 * (pj.y - mj.y);
      }
      s0 = wave_sum(s0);
      s1 = wave_sum(s1);
      s2 = wave_sum(s2);
      if (lane == 0) {
        rows[wv][r][0] += s0;
        rows[wv][r][1] += s1;
        rows[wv][r][2] += s2;
      }
    }
  }
  E = wave_sum(E);
  Ep = wave_sum(Ep);
  sl = wave_sum(sl);
  for (int off = 32; off > 0; off >>= 1) dv = fmax(dv, __shfl_xor(dv, off));
  if (lane == 0) {
    red[0][wv] = E;
    red[1][wv] = Ep;
    red[2][wv] = sl;
    red[3][wv] = dv;
  }
  __syncthreads();
  if (threadIdx.x < 3 * R) {
    const int r = threadIdx.x / 3, k = threadIdx.x % 3, j = j0 + r;
    double v = 0.0;
    for (int q = 0; q < NW; ++q) v += rows[q][r][k];
    if (j <= M) part[L.cfl + ((size_t)j * L.blocks + blockIdx.x) * 3 + k] = v;
  }
  if (threadIdx.x == 0) {
    const int g = blockIdx.y * L.blocks + blockIdx.x;
    for (int q = 1; q < NW; ++q) {
      red[0][0] += red[0][q];
      red[1][0] += red[1][q];
      red[2][0] += red[2][q];
      red[3][0] = fmax(red[3][0], red[3][q]);
    }
    part[L.e + g] = red[0][0];
    part[L.ep + g] = red[1][0];
    if (blockIdx.y == 0) part[L.sl + blockIdx.x] = red[2][0];
    part[L.dv + g] = red[3][0];
  }
}

// The eight diagnostics from the partials, by one workgroup.
constexpr int FINISH_THREADS = 1024;
__global__ __launch_bounds__(FINISH_THREADS) void k_diag_finish(Dims d, const double* __restrict__ part,
                                                                const double* __restrict__ rc, double eta,
                                                                double* __restrict__ out) {
  constexpr int NW = FINISH_THREADS / 64;
  __shared__ double red[4][NW];
  __shared__ double v[4096];  // n_r <= 4096
  __shared__ int nan_row[NW];
  const DiagLayout L = diag_layout(d);
  const int tid = threadIdx.x, wv = tid / 64, lane = tid & 63, M = d.n_r - 1;
  const double pi = 3.14159265358979323846;
  double E = 0.0, Ep = 0.0, sl = 0.0, dv = 0.0;
  for (int i = tid; i < L.groups; i += FINISH_THREADS) {
    E += part[L.e + i];
    Ep += part[L.ep + i];
    dv = fmax(dv, part[L.dv + i]);
  }
  for (int i = tid; i < L.blocks && wv == 0; i += 64) sl += part[L.sl + i];
  // CFL bound: dt max_j (B_r/dr_j + B_theta/(r_j dtheta) + B_z/dz) on the
  // physical grid (2 m_theta, m_z), dr_j the distance to the nearer neighbour;
  // a node that is not a number hides those before it
  const double dth = 2.0 * pi / (d.kt * 2.0 * d.mt), dz = 2.0 * pi / (d.kz * d.mz);
  auto r_of = [&](int j) { return rc[(size_t)j * RC_N + RC_R]; };
  int last = -1;
  static_assert(DIAG_BLOCKS % 32 == 0, "a half wave adds up one node's partials");
  for (int j = tid / 32; j <= M; j += FINISH_THREADS / 32) {
    double B[3] = {0.0, 0.0, 0.0};
    for (int q = tid & 31; q < L.blocks; q += 32)
      for (int k = 0; k < 3; ++k) B[k] += part[L.cfl + ((size_t)j * L.blocks + q) * 3 + k];
    for (int off = 16; off > 0; off >>= 1)
      for (int k = 0; k < 3; ++k) B[k] += __shfl_xor(B[k], off);
    double dr = HUGE_VAL;
    if (j > 0) dr = fmin(dr, r_of(j) - r_of(j - 1));
    if (j < M) dr = fmin(dr, r_of(j + 1) - r_of(j));
    const double vj = B[0] / dr + B[1] / (r_of(j) * dth) + B[2] / dz;
    if ((tid & 31) == 0) v[j] = vj;
    if (isnan(vj)) last = j;
  }
  E = wave_sum(E);
  Ep = wave_sum(Ep);
  sl = wave_sum(sl);
  for (int off = 32; off > 0; off >>= 1) {
    dv = fmax(dv, __shfl_xor(dv, off));
    last = max(last, __shfl_xor(last, off));
  }
  if (lane == 0) {
    red[0][wv] = E;
    red[1][wv] = Ep;
    red[2][wv] = dv;
    nan_row[wv] = last;
  }
  if (tid == 0) out[3] = sqrt(sl) / fabs(d.Re_i == 0.0 ? 1.0 : d.Re_i);
  __syncthreads();
  for (int q = 0; q < NW; ++q) last = max(last, nan_row[q]);
  double cfl = 0.0;
  for (int j = tid; j <= M; j += FINISH_THREADS)
    if (j > last) cfl = fmax(cfl, v[j]);
  for (int off = 32; off > 0; off >>= 1) cfl = fmax(cfl, __shfl_xor(cfl, off));
  if (lane == 0) red[3][wv] = cfl;
  __syncthreads();
  if (tid > 0) return;
  const double area = (2.0 * pi / d.kt) * (2.0 * pi / d.kz);
  for (int q = 1; q < NW; ++q) {
    red[0][0] += red[0][q];
    red[1][0] += red[1][q];
    red[2][0] = fmax(red[2][0], red[2][q]);
    red[3][0] = fmax(red[3][0], red[3][q]);
  }
  out[0] = 0.5 * area * red[0][0];
  out[1] = 0.5 * area * red[1][0];
  out[2] = red[2][0];
  out[4] = d.dt * (last == M ? NAN : red[3][0]);
  out[5] = 0.0;  // the step count is filled in by the caller
  // Quasi-Nusselt numbers: r^3 d<omega>/dr at each wall over its Couette
  // value -2 C2, <omega> = <u_theta>/r, d/dr by the wall rows of D1
  const double C2 = eta * (d.Re_i - eta * d.Re_o) / ((1.0 - eta) * (1.0 - eta * eta));
  for (int w = 0; w < 2; ++w) {
    const int j = w ? M : 0;
    const int lo = j - HW < 0 ? 0 : j - HW, hi = j + HW > M ? M : j + HW;
    double dw = 0.0;
    for (int k = lo; k <= hi; ++k) dw += rc[(size_t)j * RC_N + RC_W1 + (k - j + HW)] * (part[L.mean + k] / r_of(k));
    out[6 + w] = C2 == 0.0 ? NAN : r_of(j) * r_of(j) * r_of(j) * dw / (-2.0 * C2);
  }
}

// Gradient of E_pert = 1/2 int |u - U_c|^2 dV (trapezoid rule in r, Parseval
// in theta and z) with respect to the stored coefficients under
// <x, y> = sum Re(conj(x) y):  g+- = (A/2) w_j r_j c_n (u+- - U_c+-),
// g_z = A w_j r_j c_n u_z, A = (2 pi / k_theta)(2 pi / k_z).
__global__ void k_egrad(const double* __restrict__ rc, Dims d, double C1, double C2, double area,
                        const cd* __restrict__ u, cd* __restrict__ g) {
  // (area carries the seed's scale factor)
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= d.S) return;
  const int s = (int)(idx / d.mt), n = (int)(idx - (int64_t)s * d.mt);
  const int M = d.n_r - 1;
  for (int j = 0; j <= M; ++j) {
    const int64_t o = j * d.S + idx;
    if (s == d.nyq) {
      g[o] = g[d.F + o] = g[2 * d.F + o] = cd{0, 0};
      continue;
    }
    const double r = rc[(int64_t)j * RC_N + RC_R];
    double w = 0.0;
    if (j > 0) w += 0.5 * (r - rc[(int64_t)(j - 1) * RC_N + RC_R]);
    if (j < M) w += 0.5 * (rc[(int64_t)(j + 1) * RC_N + RC_R] - r);
    const double k = area * w * r * (n == 0 ? 1.0 : 2.0);
    cd p = u[o], m = u[d.F + o];
    if (s == 0 && n == 0) {
      const double U = C1 * r + C2 / r;
      p.y -= U;
      m.y += U;
    }
    const cd z = u[2 * d.F + o];
    g[o] = cd{0.5 * k * p.x, 0.5 * k * p.y};
    g[d.F + o] = cd{0.5 * k * m.x, 0.5 * k * m.y};
    g[2 * d.F + o] = cd{k * z.x, k * z.y};
  }
}

__global__ void k_finite(int64_t count, const double* __restrict__ x, int* __restrict__ flag) {
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    if (!isfinite(x[i])) bad = 1;
  if (bad) atomicOr(flag, 1);
}

}  // namespace tc


namespace {

// The eight diagnostics of the context's velocity into out_host; part:
// diag_layout().total + 8 doubles of device memory.  Synchronous.
tc_status diag_of(tc_ctx* c, double* part, double* out_host, const char* what) {
  const Dims& d = c->d;
  const DiagLayout L = diag_layout(d);
  hipLaunchKernelGGL(k_diag, dim3(L.blocks, (d.n_r + DIAG_ROWS - 1) / DIAG_ROWS), dim3(DIAG_THREADS), 0, c->stream,
                     c->rc_dev, d, c->u, c->diag_wr, c->diag_uc, part);
  hipLaunchKernelGGL(k_diag_finish, dim3(1), dim3(FINISH_THREADS), 0, c->stream, d, part, c->rc_dev, c->eta,
                     part + L.total);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = hipMemcpyAsync(out_host, part + L.total, 8 * sizeof(double), hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_check(c, e, what);
  out_host[5] = (double)c->steps;
  return TC_OK;
}

// Scratch of tc_get_diag_noalloc: one array per GPU, from module load to
// process end.  Host code takes its device address per device from
// hipGetSymbolAddress (tc_init, with the context's device current) and
// never uses the array's name.
static __device__ __align__(256) double scratch[TC_DIAG_SCRATCH_DOUBLES];

constexpr int MAX_DEVICES = 64;
double* g_scratch[MAX_DEVICES] = {};

// Device address of the scratch on the current device (looked up once per
// device); nullptr if the lookup fails.
double* scratch_address(int dev) {
  static std::mutex m;
  std::lock_guard<std::mutex> lk(m);
  if (dev < 0 || dev >= MAX_DEVICES) return nullptr;
  if (!g_scratch[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch[dev] = static_cast<double*>(ptr);
  }
  return g_scratch[dev];
}

double* diag_scratch(const tc_ctx* c) {
  return (c->device >= 0 && c->device < MAX_DEVICES) ? g_scratch[c->device] : nullptr;
}

}  // namespace

namespace tc {

hipError_t energy_of(tc_ctx* c, const cd* u, double& E) {
  const int nb = 1024;
  std::lock_guard<std::mutex> lk(c->red_mutex);
  hipLaunchKernelGGL(k_energy, dim3(nb), dim3(256), 0, c->stream, c->d, u, c->diag_wr, c->red);
  hipError_t e = hipGetLastError();
  std::vector<double> h(nb, 0.0);
  if (e == hipSuccess) e = hipMemcpyAsync(h.data(), c->red, nb * sizeof(double), hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  double sum = 0.0;
  for (int i = 0; i < nb; ++i) sum += h[i];
  const double area = (2.0 * M_PI / c->d.kt) * (2.0 * M_PI / c->d.kz);
  E = 0.5 * area * sum;
  return e;
}

}  // namespace tc

// ================================================================== C ABI
extern "C" {

const char* tc_last_error(const tc_ctx* ctx) {
  if (!ctx) return g_init_error.c_str();
  return ctx->err.c_str();
}

// smallest supported transform length >= L (0 if there is none)
static int fft_length_at_least(int L) {
  for (int x = L < 1 ? 1 : L; x <= 2048; ++x)
    if (fft_length_supported(x)) return x;
  return 0;
}

tc_status tc_init(const tc_grid* g, double eta, double Re_i, double Re_o, double dt, void* hip_stream,
                  tc_ctx** out) {
  g_init_error.clear();
  if (!out) {
    g_init_error = "out is NULL";
    return TC_EINVAL;
  }
  *out = nullptr;
  if (!g) {
    g_init_error = "grid is NULL";
    return TC_EINVAL;
  }
  tc_grid G = *g;
  // default dealiased grid: the smallest supported length that meets the
  // 3/2 rule (0 when the rule asks for more than the longest one, which the
  // length check below then rejects)
  if (G.p_theta == 0) G.p_theta = fft_length_at_least(3 * G.m_theta - 2);
  if (G.p_z == 0) G.p_z = fft_length_at_least(3 * G.m_z / 2 - 2);
  std::string why;
  if (G.n_r < 9 || G.n_r > 4096) why = "n_r must be in [9, 4096]";
  else if (G.m_theta < 1 || G.m_z < 2 || (G.m_z % 2)) why = "m_theta >= 1 and even m_z >= 2 required";
  else if (G.n_s != 9) why = "only n_s = 9 is supported";
  else if (G.precision != TC_FP64 && G.precision != TC_FP32_BULK) why = "unknown precision";
  else if (G.form != TC_ROTATIONAL && G.form != TC_CONVECTIVE) why = "unknown form of the nonlinear term";
  else if (G.form == TC_CONVECTIVE && G.precision != TC_FP64) why = "the convective form runs in FP64 only";
  else if (G.p_theta < 3 * G.m_theta - 2 || G.p_z < 3 * G.m_z / 2 - 2) why = "dealiased grid below the 3/2 rule";
  else if (!fft_length_supported(G.p_theta) || !fft_length_supported(G.p_z)) why = "unsupported transform length";
  else if (!(eta > 0.0 && eta < 1.0)) why = "eta must be in (0, 1)";
  else if (!(dt > 0.0) || !std::isfinite(dt)) why = "dt must be positive";
  else if (!(G.k_theta > 0.0) || !(G.k_z > 0.0)) why = "k_theta, k_z must be positive";
  else if (!(G.alpha >= 0.0 && G.alpha <= 1.0)) why = "alpha must be in [0, 1]";
  else if (!std::isfinite(Re_i) || !std::isfinite(Re_o)) why = "Reynolds numbers must be finite";
  if (!why.empty()) {
    g_init_error = why;
    return TC_EINVAL;
  }

  tc_ctx* c = new (std::nothrow) tc_ctx();
  if (!c) {
    g_init_error = "out of host memory";
    return TC_ENOMEM;
  }
  c->g = G;
  c->eta = eta;
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  c->r_i = eta / (1.0 - eta);
  c->r_o = 1.0 / (1.0 - eta);
  Dims& d = c->d;
  d.n_r = G.n_r;
  d.mt = G.m_theta;
  d.mz = G.m_z;
  d.pt = G.p_theta;
  d.pz = G.p_z;
  d.half = G.m_z / 2;
  d.nyq = G.m_z / 2;
  d.ndm = G.m_theta * (G.m_z / 2);
  d.S = (int64_t)G.m_z * G.m_theta;
  d.F = (int64_t)G.n_r * d.S;
  d.kt = G.k_theta;
  d.kz = G.k_z;
  d.dt = dt;
  d.Re_i = Re_i;
  d.Re_o = Re_o;
  d.form = G.form;

  // radial grid and per-node constants
  c->r = radial_nodes(d.n_r, eta, G.alpha);
  const int M = d.n_r - 1;
  c->rc.assign((size_t)d.n_r * RC_N, 0.0);
  for (int j = 0; j < d.n_r; ++j) {
    double* R = &c->rc[(size_t)j * RC_N];
    R[RC_R] = c->r[j];
    R[RC_IR] = 1.0 / c->r[j];
    R[RC_IR2] = 1.0 / (c->r[j] * c->r[j]);
    const int lo = std::max(0, j - HW), hi = std::min(M, j + HW);
    double w1[NB9], w2[NB9];
    fd_weights(c->r[j], &c->r[lo], hi - lo + 1, w1, w2);
    for (int k = lo; k <= hi; ++k) {
      R[RC_W1 + (k - j + HW)] = w1[k - lo];
      R[RC_W2 + (k - j + HW)] = w2[k - lo];
    }
  }
  // Neumann rows of P scaled to the size of the adjacent Laplacian rows
  auto rowmax = [&](int j, int off) {
    double m = 0.0;
    for (int k = 0; k < NB9; ++k) m = std::max(m, std::fabs(c->rc[(size_t)j * RC_N + off + k]));
    return m;
  };
  d.s0 = rowmax(1, RC_W2) / rowmax(0, RC_W1);
  d.sM = rowmax(M - 1, RC_W2) / rowmax(M, RC_W1);

  tc_status st = TC_OK;
  const size_t FB = field_bytes(c);
  c->rc_dev = dev_alloc<double>(c, c->rc.size() * sizeof(double), st);
  c->fac = dev_alloc<double>(c, (size_t)NOPS * d.n_r * NFAC * d.ndm * sizeof(double), st);
  // the curl adjoint as one radial sweep per slot where there are enough
  // slots for the GPU (at least 2048 waves); TC_ADJ_CURL_SWEEP=0 or 1 at
  // this call chooses the grouped or the sweep form on any grid
  {
    const char* e = std::getenv("TC_ADJ_CURL_SWEEP");
    c->adj_curl_sweep = e ? std::atoi(e) != 0 : d.S >= 131072;
  }
  c->tw_t = dev_alloc<cd>(c, (size_t)d.pt * sizeof(cd), st);
  c->tw_z = dev_alloc<cd>(c, (size_t)d.pz * sizeof(cd), st);
  c->twf_t = dev_alloc<cf>(c, (size_t)d.pt * sizeof(cf), st);
  c->twf_z = dev_alloc<cf>(c, (size_t)d.pz * sizeof(cf), st);
  c->u = dev_alloc<cd>(c, 3 * FB, st);
  c->u_prev = dev_alloc<cd>(c, 3 * FB, st);
  c->N_prev = dev_alloc<cd>(c, 3 * FB, st);
  c->N_cur = dev_alloc<cd>(c, 3 * FB, st);
  c->p = dev_alloc<cd>(c, FB, st);
  c->omega = dev_alloc<cd>(c, 3 * FB, st);
  c->zmax = dev_alloc<unsigned int>(c, (size_t)ZMAX_WORDS * d.n_r * sizeof(unsigned int), st);
  c->diag_wr = dev_alloc<double>(c, (size_t)d.n_r * sizeof(double), st);
  c->diag_uc = dev_alloc<double>(c, (size_t)d.n_r * sizeof(double), st);
  c->red = dev_alloc<double>(c, (TC_RED_DOUBLES + diag_layout(d).total + 8) * sizeof(double), st);
  // plane batch of the nonlinear term: all planes when they fit a budget
  {
    const size_t per = inter_bytes_per_plane(c);
    size_t budget = (size_t)48 << 30;
    if (const char* e = std::getenv("TC_BATCH_PLANES")) c->batch = std::max(1, std::atoi(e));
    else c->batch = (int)std::max<size_t>(1, std::min<size_t>((size_t)d.n_r, budget / std::max<size_t>(per, 1)));
    c->batch = std::min(c->batch, d.n_r);
    c->inter = dev_alloc<void>(c, per * (size_t)c->batch, st);
  }
  if (st != TC_OK) {
    g_init_error = c->err;
    free_ctx(c);
    return st;
  }
  hipError_t e = hipSuccess;
  auto up = [&](void* dst, const void* src, size_t n) {
    if (e == hipSuccess) e = hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, c->stream);
  };
  up(c->rc_dev, c->rc.data(), c->rc.size() * sizeof(double));
  // energy weights w_j r_j (trapezoid rule) and the Couette profile, for
  // the diagnostics
  std::vector<double> wr(d.n_r, 0.0), Uc(d.n_r);
  {
    for (int j = 0; j + 1 < d.n_r; ++j) {
      const double h = c->r[j + 1] - c->r[j];
      wr[j] += 0.5 * h;
      wr[j + 1] += 0.5 * h;
    }
    const double C1 = (d.Re_o - eta * d.Re_i) / (1.0 + eta);
    const double C2 = eta * (d.Re_i - eta * d.Re_o) / ((1.0 - eta) * (1.0 - eta * eta));
    for (int j = 0; j < d.n_r; ++j) {
      wr[j] *= c->r[j];
      Uc[j] = C1 * c->r[j] + C2 / c->r[j];
    }
  }
  up(c->diag_wr, wr.data(), wr.size() * sizeof(double));
  up(c->diag_uc, Uc.data(), Uc.size() * sizeof(double));
  // twiddle tables (separate host vectors: the copies are asynchronous)
  std::vector<cd> tw_t, tw_z;
  std::vector<cf> twf_t, twf_z;
  twiddles<double>(d.pt, tw_t);
  twiddles<double>(d.pz, tw_z);
  twiddles<float>(d.pt, twf_t);
  twiddles<float>(d.pz, twf_z);
  up(c->tw_t, tw_t.data(), tw_t.size() * sizeof(cd));
  up(c->tw_z, tw_z.data(), tw_z.size() * sizeof(cd));
  up(c->twf_t, twf_t.data(), twf_t.size() * sizeof(cf));
  up(c->twf_z, twf_z.data(), twf_z.size() * sizeof(cf));
  if (e == hipSuccess) e = hipMemsetAsync(c->u, 0, 3 * FB, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->u_prev, 0, 3 * FB, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->N_prev, 0, 3 * FB, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->N_cur, 0, 3 * FB, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->p, 0, FB, c->stream);
  if (e == hipSuccess) e = hipMemsetAsync(c->zmax, 0, (size_t)ZMAX_WORDS * d.n_r * sizeof(unsigned int), c->stream);
  // (the factorisation's flag and the check's result and work space lie in
  // buffers that hold nothing yet: the check needs a field's size)
  int* const bad = reinterpret_cast<int*>(c->red);
  if (e == hipSuccess) e = hipMemsetAsync(bad, 0, sizeof(int), c->stream);
  if (e == hipSuccess) e = launch_factor(c, bad);
  int hbad = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) {
    g_init_error = std::string("HIP error during set-up: ") + hipGetErrorString(e);
    free_ctx(c);
    return TC_EHIP;
  }
  if (hbad) {
    g_init_error = "zero or non-finite pivot in the banded factorisation";
    free_ctx(c);
    return TC_ESINGULAR;
  }
  // the line kernels' copy of the factors, where the grid allows them
  // (TC_PC_LINE=0 selects the four-sweep kernels instead): the last allocation,
  // left out where the device has no room for it
  if (e = make_flin(c); e != hipSuccess) {
    g_init_error = std::string("HIP error during set-up: ") + hipGetErrorString(e);
    free_ctx(c);
    return TC_EHIP;
  }
  // the factors are unpivoted: check their backward error on one solve per
  // operator and mode before accepting them, by the kernels that the steps use;
  // a copy that failed would be given up and the factors themselves checked
  for (;;) {
    unsigned long long* const worst = reinterpret_cast<unsigned long long*>(c->red);
    unsigned long long hw = 0;
    static_assert(NOPS * sizeof(double) <= 2 * sizeof(cd), "the check's work space fits one field of m_z = 2 |l| slots");
    e = hipMemsetAsync(worst, 0, sizeof(*worst), c->stream);
    if (e == hipSuccess)
      e = c->flin ? launch_line_check(c, worst) : launch_factor_check(c, reinterpret_cast<double*>(c->omega), worst);
    if (e == hipSuccess) e = hipMemcpyAsync(&hw, worst, sizeof(hw), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
      g_init_error = std::string("HIP error during the factor check: ") + hipGetErrorString(e);
      free_ctx(c);
      return TC_EHIP;
    }
    std::memcpy(&c->factor_error, &hw, sizeof(double));
    if (c->factor_error <= TC_FACTOR_CHECK_MAX) break;
    if (drop_flin(c)) continue;
    g_init_error = "the unpivoted factors fail the backward-error check (" + std::to_string(c->factor_error) + ")";
    free_ctx(c);
    return TC_ESINGULAR;
  }
  // the allocation-free diagnostics' scratch address on this device
  if (hipGetDevice(&c->device) != hipSuccess || !scratch_address(c->device)) {
    (void)hipGetLastError();
    g_init_error = "cannot look up the diagnostics scratch on this device";
    free_ctx(c);
    return TC_EHIP;
  }
  *out = c;
  return TC_OK;
}

tc_status tc_destroy(tc_ctx* ctx) {
  if (!ctx) return TC_EINVAL;
  (void)hipStreamSynchronize(ctx->stream);
  free_ctx(ctx);
  return TC_OK;
}

tc_status tc_radial_nodes(const tc_ctx* ctx, double* r_host) {
  if (!ctx || !r_host) return TC_EINVAL;
  std::memcpy(r_host, ctx->r.data(), ctx->r.size() * sizeof(double));
  return TC_OK;
}

tc_status tc_set_state(tc_ctx* c, const void* u, const void* u_prev, const void* N_prev) {
  if (!c) return TC_EINVAL;
  if (!u) return fail(c, TC_EINVAL, "u is NULL");
  const size_t B3 = 3 * field_bytes(c);
  c->omega_fresh = false;
  hipError_t e = hipMemcpyAsync(c->u, u, B3, hipMemcpyDeviceToDevice, c->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(c->u_prev, u_prev ? u_prev : u, B3, hipMemcpyDeviceToDevice, c->stream);
  if (e != hipSuccess) return hip_check(c, e, "tc_set_state copy");
  if (N_prev) {
    e = hipMemcpyAsync(c->N_prev, N_prev, B3, hipMemcpyDeviceToDevice, c->stream);
    if (e != hipSuccess) return hip_check(c, e, "tc_set_state copy");
  } else {
    tc_status s = nonlinear(c, c->u_prev, c->N_prev);
    if (s != TC_OK) return s;
  }
  e = hipMemsetAsync(c->p, 0, field_bytes(c), c->stream);
  if (e != hipSuccess) return hip_check(c, e, "tc_set_state");
  c->steps = 0;
  c->have_p = false;
  return TC_OK;
}

tc_status tc_get_state(const tc_ctx* cc, void* u, void* p) {
  tc_ctx* c = const_cast<tc_ctx*>(cc);
  if (!c) return TC_EINVAL;
  if (!u && !p) return fail(c, TC_EINVAL, "nothing to copy");
  hipError_t e = hipSuccess;
  if (u) e = hipMemcpyAsync(u, c->u, 3 * field_bytes(c), hipMemcpyDeviceToDevice, c->stream);
  if (e == hipSuccess && p) e = hipMemcpyAsync(p, c->p, field_bytes(c), hipMemcpyDeviceToDevice, c->stream);
  return hip_check(c, e, "tc_get_state copy");
}

tc_status tc_get_history(const tc_ctx* cc, void* u_prev, void* N_prev) {
  tc_ctx* c = const_cast<tc_ctx*>(cc);
  if (!c) return TC_EINVAL;
  hipError_t e = hipSuccess;
  if (u_prev) e = hipMemcpyAsync(u_prev, c->u_prev, 3 * field_bytes(c), hipMemcpyDeviceToDevice, c->stream);
  if (e == hipSuccess && N_prev)
    e = hipMemcpyAsync(N_prev, c->N_prev, 3 * field_bytes(c), hipMemcpyDeviceToDevice, c->stream);
  return hip_check(c, e, "tc_get_history copy");
}

tc_status tc_step(tc_ctx* c, int32_t nsteps) {
  if (!c) return TC_EINVAL;
  if (nsteps < 0) return fail(c, TC_EINVAL, "nsteps must be >= 0");
  if (c->timing)
    for (auto& t : c->timers) t.used = 0;
  for (int32_t k = 0; k < nsteps; ++k) {
    tc_status s = nonlinear(c, c->u, c->N_cur);
    if (s != TC_OK) return s;
    timer_begin(c, TK_PC);
    hipError_t e = launch_pc(c, c->u, c->u_prev, c->N_cur, c->N_prev, c->u_prev, c->p, k == nsteps - 1, c->omega);
    timer_end(c, TK_PC);
    if (e != hipSuccess) return hip_check(c, e, "predictor-corrector");
    std::swap(c->u, c->u_prev);
    std::swap(c->N_cur, c->N_prev);
    c->omega_fresh = pc_fuses_curl(c);  // then omega = curl(u^{i+1})
    ++c->steps;
    c->have_p = true;
  }
  return TC_OK;
}

tc_status tc_nonlinear(tc_ctx* c, const void* u, void* N) {
  if (!c) return TC_EINVAL;
  if (!u || !N) return fail(c, TC_EINVAL, "NULL array");
  const char* a = static_cast<const char*>(u);
  const char* b = static_cast<const char*>(N);
  const size_t B3 = 3 * field_bytes(c);
  if (a < b + B3 && b < a + B3) return fail(c, TC_EINVAL, "u and N overlap");
  return nonlinear(c, static_cast<const cd*>(u), static_cast<cd*>(N));
}

static int op_of(tc_solve_kind k) {
  switch (k) {
    case TC_SOLVE_P:
    case TC_SOLVE_PHI: return OP_P;
    case TC_SOLVE_UPLUS: return OP_HP;
    case TC_SOLVE_UMINUS: return OP_HM;
    case TC_SOLVE_UZ: return OP_HZ;
  }
  return -1;
}

tc_status tc_helmholtz_solve(tc_ctx* c, tc_solve_kind k, const void* rhs, void* x) {
  if (!c) return TC_EINVAL;
  const int op = op_of(k);
  if (op < 0) return fail(c, TC_EINVAL, "unknown solve kind");
  if (!rhs || !x) return fail(c, TC_EINVAL, "NULL array");
  return hip_check(c, launch_solve(c, op, 0, static_cast<const cd*>(rhs), static_cast<cd*>(x)), "solve");
}

tc_status tc_helmholtz_solve_transposed(tc_ctx* c, tc_solve_kind k, const void* rhs, void* x) {
  if (!c) return TC_EINVAL;
  const int op = op_of(k);
  if (op < 0) return fail(c, TC_EINVAL, "unknown solve kind");
  if (!rhs || !x) return fail(c, TC_EINVAL, "NULL array");
  if (rhs == x) return fail(c, TC_EINVAL, "the transposed solve needs x != rhs");
  return hip_check(c, launch_solve(c, op, 1, static_cast<const cd*>(rhs), static_cast<cd*>(x)), "solve");
}

tc_status tc_get_diag(tc_ctx* c, double* out) {
  if (!c || !out) return TC_EINVAL;
  std::lock_guard<std::mutex> lk(c->red_mutex);
  return diag_of(c, c->red + TC_RED_DOUBLES, out, "tc_get_diag");
}

tc_status tc_get_diag_noalloc(tc_ctx* c, double* out) {
  if (!c || !out) return TC_EINVAL;
  // the documented limit (partials that an earlier layout needed; those of any
  // grid within it fit)
  const size_t need = 4 * (size_t)std::max<int64_t>(1024, (c->d.S + 255) / 256) + 97 * (size_t)c->d.n_r + 8;
  static_assert((size_t)(3 * DIAG_BLOCKS / DIAG_ROWS + 3 * DIAG_BLOCKS + 1) * 4096 + 4 * DIAG_BLOCKS + 8 <=
                    TC_DIAG_SCRATCH_DOUBLES, "the partials of the largest n_r must fit the scratch");
  static_assert((size_t)2 * DIAG_GROUPS * (3 + 1 + 3 * DIAG_ROWS + DIAG_ROWS) + 8 <= TC_DIAG_SCRATCH_DOUBLES,
                "the partials of the most workgroups must fit the scratch");
  if (need > TC_DIAG_SCRATCH_DOUBLES)
    return fail(c, TC_EINVAL, "tc_get_diag_noalloc: the grid is past the limit of the scratch (" + std::to_string(need) +
                                  " of " + std::to_string(TC_DIAG_SCRATCH_DOUBLES) + ")");
  double* part = diag_scratch(c);
  if (!part) return fail(c, TC_EHIP, "tc_get_diag_noalloc: no scratch address for this device");
  return diag_of(c, part, out, "tc_get_diag_noalloc");
}

tc_status tc_adjoint_seed(tc_ctx* c, const void* u, double scale, void* g) {
  if (!c) return TC_EINVAL;
  if (!u || !g) return fail(c, TC_EINVAL, "NULL array");
  if (!std::isfinite(scale)) return fail(c, TC_EINVAL, "scale must be finite");
  const Dims& d = c->d;
  const double C1 = (d.Re_o - c->eta * d.Re_i) / (1.0 + c->eta);
  const double C2 = c->eta * (d.Re_i - c->eta * d.Re_o) / ((1.0 - c->eta) * (1.0 - c->eta * c->eta));
  const double area = scale * (2.0 * M_PI / d.kt) * (2.0 * M_PI / d.kz);
  hipLaunchKernelGGL(k_egrad, dim3((unsigned)((d.S + 255) / 256)), dim3(256), 0, c->stream, c->rc_dev, d, C1, C2,
                     area, static_cast<const cd*>(u), static_cast<cd*>(g));
  return hip_check(c, hipGetLastError(), "tc_adjoint_seed");
}

tc_status tc_perturbation_energy_gradient(tc_ctx* c, const void* u, void* g) {
  if (!c) return TC_EINVAL;
  if (!u || !g) return fail(c, TC_EINVAL, "NULL array");
  const Dims& d = c->d;
  const double C1 = (d.Re_o - c->eta * d.Re_i) / (1.0 + c->eta);
  const double C2 = c->eta * (d.Re_i - c->eta * d.Re_o) / ((1.0 - c->eta) * (1.0 - c->eta * c->eta));
  const double area = (2.0 * M_PI / d.kt) * (2.0 * M_PI / d.kz);
  hipLaunchKernelGGL(k_egrad, dim3((unsigned)((d.S + 255) / 256)), dim3(256), 0, c->stream, c->rc_dev, d, C1, C2,
                     area, static_cast<const cd*>(u), static_cast<cd*>(g));
  return hip_check(c, hipGetLastError(), "tc_perturbation_energy_gradient");
}

tc_status tc_check_finite(tc_ctx* c) {
  if (!c) return TC_EINVAL;
  std::lock_guard<std::mutex> lk(c->red_mutex);
  int* flag = reinterpret_cast<int*>(c->red);
  int h = 0;
  hipError_t e = hipMemsetAsync(flag, 0, sizeof(int), c->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_finite, dim3(2048), dim3(256), 0, c->stream, (int64_t)6 * c->d.F,
                       reinterpret_cast<const double*>(c->u), flag);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_check(c, e, "tc_check_finite");
  return h ? fail(c, TC_ENONFINITE, "non-finite value in the velocity") : TC_OK;
}

tc_status tc_set_timing(tc_ctx* c, int32_t enable) {
  if (!c) return TC_EINVAL;
  c->timing = enable != 0;
  for (auto& t : c->timers) t.used = 0;
  return TC_OK;
}

tc_status tc_kernel_time(tc_ctx* c, int32_t which, double* ms_out, int32_t* launches_out) {
  if (!c || !ms_out || which < 0 || which >= TK_N) return TC_EINVAL;
  KernelTimer& t = c->timers[which];
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_check(c, e, "tc_kernel_time");
  double tot = 0.0;
  int n = 0;
  for (int i = 0; i + 1 < t.used; i += 2) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.ev[i], t.ev[i + 1]) == hipSuccess) {
      tot += ms;
      ++n;
    }
  }
  *ms_out = n ? tot / n : 0.0;
  if (launches_out) *launches_out = n;
  return TC_OK;
}

tc_status tc_factor_backward_error(const tc_ctx* c, double* out) {
  if (!c || !out) return TC_EINVAL;
  *out = c->factor_error;
  return TC_OK;
}

tc_status tc_memory_bytes(const tc_ctx* c, uint64_t* out) {
  if (!c || !out) return TC_EINVAL;
  *out = c->bytes;
  return TC_OK;
}

tc_status tc_line_copy_bytes(const tc_ctx* c, uint64_t* out) {
  if (!c || !out) return TC_EINVAL;
  *out = c->flin ? c->flin_bytes : 0;
  return TC_OK;
}

}  // extern "C"
