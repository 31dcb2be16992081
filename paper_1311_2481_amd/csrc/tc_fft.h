// Mixed-radix Stockham FFT for gfx950 (radices 8, 4, 2, 3, 5, 6, 10), registers
// plus LDS exchanges.
//
// A workgroup transforms NF sequences of length L at once, TPF threads per
// sequence; thread (t, f) has t in [0, TPF), f in [0, NF).
//
// Pass with radix R after the radices already applied (their product NS):
// butterfly j in [0, L/R) reads x[j + q L/R], q = 0..R-1, multiplies input q
// by w^(q k L/(NS R)) with k = j mod NS and w = exp(SIGN 2 pi i / L), takes
// the R-point DFT and writes output s to (j / NS) NS R + k + s NS.  After
// the last pass the data is in natural order (Stockham autosort).
// Butterfly j of every pass belongs to thread t = j mod TPF.
//
// The first pass takes its inputs from registers filled by the caller
// (element j + q L/R0 in slot [k][q], j = t + k TPF), the last pass leaves
// its outputs in registers (element j + s L/RN in slot [k][s]): only the
// exchanges between passes go through LDS.  A transform run with the radix
// order reversed starts exactly where a transform in natural order ends
// (its first-pass inputs are the other's last-pass outputs in the same
// slots), so a pointwise product between an inverse and a forward
// transform never leaves registers.
//
// LDS layout: element e of sequence f at (e + e/8) * NF + f; the pad word
// every 8 elements spreads the stride-8 writes of the early passes over
// the banks.  SIGN = +1 is the unnormalised inverse transform of eq.
// fourier, SIGN = -1 the forward one (scaling is left to the caller).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace tc {

// Aligned to its full size so that LDS and global accesses are single
// 128-bit (double) or 64-bit (float) operations: split 64-bit accesses of
// interleaved complex data would hit the LDS banks two-way.
template <typename T> struct alignas(2 * sizeof(T)) C2 { T x, y; };

template <typename T> __device__ __forceinline__ C2<T> cadd(C2<T> a, C2<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T> __device__ __forceinline__ C2<T> csub(C2<T> a, C2<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T> __device__ __forceinline__ C2<T> cmul(C2<T> a, C2<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T> __device__ __forceinline__ C2<T> cscale(C2<T> a, T s) { return {a.x * s, a.y * s}; }
// multiply by SIGN * i
template <int SIGN, typename T> __device__ __forceinline__ C2<T> mul_si(C2<T> a) {
  return SIGN > 0 ? C2<T>{-a.y, a.x} : C2<T>{a.y, -a.x};
}
template <typename T> __device__ __forceinline__ C2<T> cconj(C2<T> a) { return {a.x, -a.y}; }

struct RadixList {
  int n;
  int r[24];
};

// Radices of a length 2^a 3^b 5^c: as many 8s as fit; a 2 left over goes into
// a 6 or a 10, two into 6 6 or 6 10, so that few passes (and exchanges) are
// left: 48 = 8 6, 144 = 8 3 6, 288 = 8 6 6, 480 = 8 10 6.  A 3 or 6 comes
// last, where there is none an 8: with L / 6 or L / 8 threads a thread then
// holds 6 or 8 points at the end.  SIX: an 8
// and a 3 as 4 6 (1536 = 8 8 4 6 instead of 8 8 8 3), which leaves every
// thread one butterfly in the last pass.
constexpr RadixList make_radices(int L, bool SIX = false) {
  RadixList rl{0, {}};
  int a = 0, b = 0, c = 0;
  while (L % 2 == 0) { ++a; L /= 2; }
  while (L % 3 == 0) { ++b; L /= 3; }
  while (L % 5 == 0) { ++c; L /= 5; }
  int six = 0, ten = 0;
  if (SIX && a % 3 == 0 && a >= 6 && b >= 1) { six = 1; --a; --b; }
  for (; a >= 3; a -= 3) rl.r[rl.n++] = 8;
  if (a == 2 && b >= 2 && !six) { six = 2; a = 0; b -= 2; }
  if (a == 2 && b >= 1 && c >= 1 && !six) { six = 1; ten = 1; a = 0; --b; --c; }
  if (a == 1 && b >= 1) { six = 1; a = 0; --b; }
  if (a == 1 && c >= 1) { ten = 1; a = 0; --c; }
  if (a == 2) rl.r[rl.n++] = 4;
  if (a == 1) rl.r[rl.n++] = 2;
  for (; ten > 0; --ten) rl.r[rl.n++] = 10;
  for (; c > 0; --c) rl.r[rl.n++] = 5;
  for (; b > 0; --b) rl.r[rl.n++] = 3;
  for (; six > 0; --six) rl.r[rl.n++] = 6;
  if (rl.r[rl.n - 1] % 3 != 0 && rl.r[0] == 8 && !(rl.n == 2 && rl.r[1] == 2)) {
    for (int i = 1; i < rl.n; ++i) rl.r[i - 1] = rl.r[i];
    rl.r[rl.n - 1] = 8;
  }
  if (L != 1) rl.n = -1;
  return rl;
}

constexpr int radix_product(const RadixList& rl, int upto) {
  int p = 1;
  for (int i = 0; i < upto; ++i) p *= rl.r[i];
  return p;
}

// R-point DFT in registers, y_s = sum_q v_q exp(SIGN 2 pi i q s / R).
template <int R, int SIGN, typename T> struct Butterfly;

template <int SIGN, typename T> struct Butterfly<2, SIGN, T> {
  static __device__ __forceinline__ void run(C2<T>* v) {
    C2<T> a = cadd(v[0], v[1]), b = csub(v[0], v[1]);
    v[0] = a; v[1] = b;
  }
};

template <int SIGN, typename T> struct Butterfly<4, SIGN, T> {
  static __device__ __forceinline__ void run(C2<T>* v) {
    C2<T> t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    C2<T> t2 = cadd(v[1], v[3]), t3 = mul_si<SIGN>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2); v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3); v[3] = csub(t1, t3);
  }
};

template <int SIGN, typename T> struct Butterfly<8, SIGN, T> {
  static __device__ __forceinline__ void run(C2<T>* v) {
    C2<T> e[4] = {v[0], v[2], v[4], v[6]};
    C2<T> o[4] = {v[1], v[3], v[5], v[7]};
    Butterfly<4, SIGN, T>::run(e);
    Butterfly<4, SIGN, T>::run(o);
    const T h = T(0.70710678118654752440084436210484903928);
    // o_k *= exp(SIGN 2 pi i k / 8)
    C2<T> o1 = {h * (o[1].x - T(SIGN) * o[1].y), h * (o[1].y + T(SIGN) * o[1].x)};
    C2<T> o2 = mul_si<SIGN>(o[2]);
    C2<T> o3 = {h * (-o[3].x - T(SIGN) * o[3].y), h * (-o[3].y + T(SIGN) * o[3].x)};
    v[0] = cadd(e[0], o[0]); v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);   v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);   v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);   v[7] = csub(e[3], o3);
  }
};

template <int SIGN, typename T> struct Butterfly<3, SIGN, T> {
  static __device__ __forceinline__ void run(C2<T>* v) {
    const T s3 = T(0.86602540378443864676372317075293618347);
    C2<T> a = cadd(v[1], v[2]);
    C2<T> d = csub(v[1], v[2]);
    C2<T> t = {v[0].x - T(0.5) * a.x, v[0].y - T(0.5) * a.y};
    C2<T> s = mul_si<SIGN>(cscale(d, s3));
    v[0] = cadd(v[0], a);
    v[1] = cadd(t, s);
    v[2] = csub(t, s);
  }
};

template <int SIGN, typename T> struct Butterfly<5, SIGN, T> {
  static __device__ __forceinline__ void run(C2<T>* v) {
    const T c1 = T(0.30901699437494742410229341718281905886);
    const T c2 = T(-0.80901699437494742410229341718281905886);
    const T s1 = T(0.95105651629515357211643933337938214340);
    const T s2 = T(0.58778525229247312916870595463907276860);
    C2<T> a1 = cadd(v[1], v[4]), a2 = cadd(v[2], v[3]);
    C2<T> b1 = csub(v[1], v[4]), b2 = csub(v[2], v[3]);
    C2<T> t1 = {v[0].x + c1 * a1.x + c2 * a2.x, v[0].y + c1 * a1.y + c2 * a2.y};
    C2<T> t2 = {v[0].x + c2 * a1.x + c1 * a2.x, v[0].y + c2 * a1.y + c1 * a2.y};
    C2<T> u1 = mul_si<SIGN>(C2<T>{s1 * b1.x + s2 * b2.x, s1 * b1.y + s2 * b2.y});
    C2<T> u2 = mul_si<SIGN>(C2<T>{s2 * b1.x - s1 * b2.x, s2 * b1.y - s1 * b2.y});
    v[0] = cadd(v[0], cadd(a1, a2));
    v[1] = cadd(t1, u1); v[4] = csub(t1, u1);
    v[2] = cadd(t2, u2); v[3] = csub(t2, u2);
  }
};

// 2 M points, M = 3 or 5: the prime-factor form, two M-point transforms and M
// pairs, input M n1 + 2 n2 and output M k1 + (M + 1) k2 (mod 2 M), no twiddles
template <int M, int SIGN, typename T> struct ButterflyPair {
  static __device__ __forceinline__ void run(C2<T>* v) {
    C2<T> e[M], o[M];
#pragma unroll
    for (int n = 0; n < M; ++n) {
      e[n] = v[(2 * n) % (2 * M)];
      o[n] = v[(M + 2 * n) % (2 * M)];
    }
    Butterfly<M, SIGN, T>::run(e);
    Butterfly<M, SIGN, T>::run(o);
#pragma unroll
    for (int k = 0; k < M; ++k) {
      v[((M + 1) * k) % (2 * M)] = cadd(e[k], o[k]);
      v[(M + (M + 1) * k) % (2 * M)] = csub(e[k], o[k]);
    }
  }
};
template <int SIGN, typename T> struct Butterfly<6, SIGN, T> : ButterflyPair<3, SIGN, T> {};
template <int SIGN, typename T> struct Butterfly<10, SIGN, T> : ButterflyPair<5, SIGN, T> {};

constexpr RadixList reversed(RadixList rl) {
  RadixList o{rl.n, {}};
  for (int i = 0; i < rl.n; ++i) o.r[i] = rl.r[rl.n - 1 - i];
  return o;
}

// LDS slot of element e.  SWZ = false: one pad word every 8 elements.
// SWZ = true (lengths that are multiples of 16): no padding; the slots of
// each 16-element block are permuted by bits 3-6 and 9-12 of e, which
// removes the bank conflicts of the strided exchanges at the cost of a few
// integer operations per access.
template <int L, bool SWZ> __host__ __device__ constexpr int lds_slot(int e) {
  if constexpr (SWZ) {
    static_assert(L % 16 == 0, "swizzled layout needs L % 16 == 0");
    return (e & ~15) | ((e ^ (e >> 3) ^ (e >> 9)) & 15);
  } else {
    return e + (e >> 3);
  }
}
template <int L, bool SWZ> __host__ __device__ constexpr int lds_len() {
  if constexpr (SWZ) return L;
  else return lds_slot<L, false>(L - 1) + 1;
}

// Mean square, over the outputs of all passes but the first (which has no
// twiddles), of the factor by which the rounding of the one twiddle read grows
// in the powers w^q formed from it: q by a chain of products, less where w^3
// is read as well (w^4 = w^3 w, w^5 = w^3 w^2, w^6 = w^3 w^3, ...): level 1
// reads it in the passes between the first and the last, whose registers have
// room for it, level 2 in the last too (radices from 6 on).
constexpr bool twiddle_cubed(const RadixList& rl, int pass, int level) {
  return pass > 0 && rl.r[pass] >= 6 && level >= (pass < rl.n - 1 ? 1 : 2);
}
constexpr double twiddle_growth(const RadixList& rl, int level) {
  constexpr int cubed[10] = {0, 1, 4, 1, 2, 5, 4, 5, 8, 9};
  double sum = 0.0;
  for (int i = 1; i < rl.n; ++i) {
    double pass = 0.0;
    for (int q = 1; q < rl.r[i]; ++q) pass += twiddle_cubed(rl, i, level) ? cubed[q] : q * q;
    sum += pass / rl.r[i];
  }
  return sum;
}

// The plain factorisation (8s, a 4 or 2, 3s, 5s) is the measure of accuracy:
// a list of other radices or in another order reads w^3 where its powers
// would be worse.  (With w alone the error of omega x u, in double, was 1.57
// times that of the plain passes at 16 points, 1.44 at 32 and 40, 1.51 at 480,
// 1.38 at 640, 1.11 at 1152; it is 0.8 to 1.03 times at every length now, for
// at most 7% of k_theta's time, at 288 points.)
constexpr RadixList plain_radices(int L) {
  RadixList rl{0, {}};
  for (int R : {8, 4, 2, 3, 5})
    for (; L % R == 0; L /= R) rl.r[rl.n++] = R;
  return rl;
}
constexpr int twiddle_level(const RadixList& rl, const RadixList& plain) {
  for (int level = 0; level < 2; ++level)
    if (twiddle_growth(rl, level) <= twiddle_growth(plain, 0) + 1e-9) return level;
  return 2;
}

// Twiddles w^q, q = 1..R-1, of one butterfly, w = W[base] (conjugated for
// SIGN > 0).  load() reads the few that are kept, some time before apply()
// needs them: their latency then passes during the exchange before.  In
// double w is read, with CUBE w^3 too, and the other powers are formed by
// products as they are needed, so that few twiddles are live: register
// pressure decides the occupancy of the long transforms.  In float w, w^2 (and
// w^4 from radix 6 on) are read and the other powers formed by products.
template <int R, int SIGN, typename T, bool CUBE> struct Twiddle {
  static constexpr bool F64 = sizeof(T) == 8;
  static constexpr int N = F64 ? (CUBE ? 2 : 1) : (R >= 6 ? 3 : (R == 2 || R == 3 ? 1 : 2));
  C2<T> w[N];
  __device__ __forceinline__ void load(const C2<T>* __restrict__ W, int base) {
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = W[(k == 0 ? 1 : F64 ? 3 : 1 << k) * base];
  }
  // v[q] *= w^q, q = 1..R-1
  __device__ __forceinline__ void apply(C2<T>* v) const {
    C2<T> u[N];
#pragma unroll
    for (int k = 0; k < N; ++k) u[k] = SIGN > 0 ? cconj(w[k]) : w[k];
    v[1] = cmul(v[1], u[0]);
    if constexpr (F64 && CUBE) {
      static_assert(R >= 6, "w^3 is a power of its own from radix 6 on");
      C2<T> p = cmul(u[0], u[0]);
      v[2] = cmul(v[2], p);
      v[5] = cmul(v[5], cmul(u[1], p));
      v[3] = cmul(v[3], u[1]);
      v[4] = cmul(v[4], cmul(u[1], u[0]));
      if constexpr (R >= 8) {
        const C2<T> w6 = cmul(u[1], u[1]);
        v[6] = cmul(v[6], w6);
        v[7] = cmul(v[7], cmul(w6, u[0]));
        if constexpr (R == 10) {
          v[8] = cmul(v[8], cmul(w6, p));
          v[9] = cmul(v[9], cmul(w6, u[1]));
        }
      }
    } else if constexpr (F64) {
      C2<T> wq = u[0];
#pragma unroll
      for (int q = 2; q < R; ++q) {
        wq = cmul(wq, u[0]);
        v[q] = cmul(v[q], wq);
      }
    } else if constexpr (R == 3) {
      v[2] = cmul(v[2], cmul(u[0], u[0]));
    } else if constexpr (R > 3) {
      const C2<T> w3 = cmul(u[0], u[1]);
      v[2] = cmul(v[2], u[1]);
      v[3] = cmul(v[3], w3);
      if constexpr (R == 5) v[4] = cmul(v[4], cmul(u[1], u[1]));
      if constexpr (R >= 6) {
        const C2<T> w5 = cmul(u[0], u[2]);
        v[4] = cmul(v[4], u[2]);
        v[5] = cmul(v[5], w5);
        if constexpr (R >= 8) {
          v[6] = cmul(v[6], cmul(u[1], u[2]));
          v[7] = cmul(v[7], cmul(w3, u[2]));
        }
        if constexpr (R == 10) {
          v[8] = cmul(v[8], cmul(u[2], u[2]));
          v[9] = cmul(v[9], cmul(w5, u[2]));
        }
      }
    }
  }
};

template <typename T, int L, int TPF, int SIGN, bool REV, bool SWZ = false, bool SIX = false, bool EARLY = (L < 1024),
          int MAX_LEVEL = 2, bool PLAIN = false>
struct Fft {
  static constexpr RadixList LIST = PLAIN ? plain_radices(L) : make_radices(L, SIX);
  static constexpr RadixList RL = REV ? reversed(LIST) : LIST;
  static_assert(RL.n > 0, "unsupported transform length");
  static constexpr int P = RL.n;
  static constexpr int R0 = RL.r[0];
  static constexpr int RN = RL.r[P - 1];
  static constexpr int PER0 = (L / R0 + TPF - 1) / TPF;
  static constexpr int PERN = (L / RN + TPF - 1) / TPF;
  using In = C2<T>[PER0][R0];
  using Out = C2<T>[PERN][RN];

  // twiddles of one butterfly of pass PP
  static constexpr int LEVEL_BEST = twiddle_level(RL, REV ? reversed(plain_radices(L)) : plain_radices(L));
  static constexpr int LEVEL = LEVEL_BEST < MAX_LEVEL ? LEVEL_BEST : MAX_LEVEL;
  template <int PP>
  using Tw = Twiddle<RL.r[PP < P ? PP : P - 1], SIGN, T, twiddle_cubed(RL, PP < P ? PP : P - 1, LEVEL)>;

  // twiddles of this thread's butterflies of pass PP
  template <int PP, int PER>
  static __device__ __forceinline__ void load_twiddles(Tw<PP> (&tw)[PER], const C2<T>* __restrict__ W, int t) {
    constexpr int R = RL.r[PP], NS = radix_product(RL, PP), NB = L / R;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = t + k * TPF;
      // (past the last butterfly: any place of the table)
      tw[k].load(W, (NB % TPF == 0 || j < NB ? j % NS : 0) * (L / (NS * R)));  // q (j % NS) L/(NS R) < L
    }
  }

  // EARLY: a pass's twiddles are read before the exchange in front of it; the
  // long transforms, whose registers are capped for occupancy, read them at
  // their use.

  // Pass PP and those after it.  v: the inputs of pass PP (element j + q
  // L/R, j = t + k TPF), tw: its twiddles (none for the first pass).  Each
  // exchange goes through buf (lds_len<L>() * NF elements), whole elements
  // at a time, or, SPLIT, one component at a time through a buffer of T
  // (half the bytes, twice the barriers): the real parts are written in this
  // pass's output order and read in the next pass's input order, then the
  // imaginary parts.
  template <int NF, bool SPLIT, int PP, int PER, int R>
  static __device__ __forceinline__ void pass(C2<T> (&v)[PER][R], Tw<PP> (&tw)[PER], Out& vn, void* buf,
                                              const C2<T>* __restrict__ W, int t, int f) {
    constexpr int NS = radix_product(RL, PP);
    constexpr int NB = L / R;
    if constexpr (PP > 0 && !EARLY) load_twiddles<PP, PER>(tw, W, t);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = t + k * TPF;
      if (NB % TPF == 0 || j < NB) {
        if constexpr (PP > 0) tw[k].apply(v[k]);
        Butterfly<R, SIGN, T>::run(v[k]);
      }
    }
    if constexpr (PP == P - 1) {
#pragma unroll
      for (int k = 0; k < PER; ++k)
#pragma unroll
        for (int s = 0; s < R; ++s) vn[k][s] = v[k][s];
    } else {
      constexpr int R2 = RL.r[PP + 1];
      constexpr int NB2 = L / R2;
      constexpr int PER2 = (NB2 + TPF - 1) / TPF;
      C2<T> nx[PER2][R2];
      Tw<PP + 1> tw2[PER2];
      if constexpr (EARLY) load_twiddles<PP + 1, PER2>(tw2, W, t);
      using E = typename std::conditional<SPLIT, T, C2<T>>::type;
      E* b = reinterpret_cast<E*>(buf);
#pragma unroll
      for (int comp = 0; comp < (SPLIT ? 2 : 1); ++comp) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const int j = t + k * TPF;
          if (NB % TPF == 0 || j < NB) {
            const int base = (j / NS) * NS * R + j % NS;
#pragma unroll
            for (int s = 0; s < R; ++s) {
              E& x = b[lds_slot<L, SWZ>(base + s * NS) * NF + f];
              if constexpr (SPLIT) x = comp ? v[k][s].y : v[k][s].x;
              else x = v[k][s];
            }
          }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER2; ++k) {
          const int j = t + k * TPF;
          if (NB2 % TPF == 0 || j < NB2) {
#pragma unroll
            for (int q = 0; q < R2; ++q) {
              const E x = b[lds_slot<L, SWZ>(j + q * NB2) * NF + f];
              if constexpr (SPLIT) (comp ? nx[k][q].y : nx[k][q].x) = x;
              else nx[k][q] = x;
            }
          }
        }
        __syncthreads();
      }
      pass<NF, SPLIT, PP + 1, PER2, R2>(nx, tw2, vn, buf, W, t, f);
    }
  }

  // Full transform.  buf: LDS, lds_len<L>() * NF elements of C2<T> (T when
  // SPLIT).  Every exchange ends with a barrier, so buf may be reused at once.
  template <int NF, bool SPLIT = false>
  static __device__ __forceinline__ void run(In& v0, Out& vn, void* buf, const C2<T>* __restrict__ W, int t, int f) {
    Tw<0> none[PER0];
    pass<NF, SPLIT, 0, PER0, R0>(v0, none, vn, buf, W, t, f);
  }

  // element index held in register slot [k][q] before / after the transform
  static __device__ __forceinline__ int in_index(int t, int k, int q) { return t + k * TPF + q * (L / R0); }
  static __device__ __forceinline__ int out_index(int t, int k, int s) { return t + k * TPF + s * (L / RN); }
  static __device__ __forceinline__ bool in_valid(int t, int k) { return (L / R0) % TPF == 0 || t + k * TPF < L / R0; }
  static __device__ __forceinline__ bool out_valid(int t, int k) { return (L / RN) % TPF == 0 || t + k * TPF < L / RN; }
};

}  // namespace tc
