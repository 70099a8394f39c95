// Rosenbrock-Wanner (Rodas4) step for one trajectory per lane, and its
// reverse.  Paper references: the Rosenbrock replay with the mesh frozen and
// the transposed linear solve plus the Jacobian's own derivative in the
// reverse sweep (Section 3.2).
//
// Everything lives in registers with compile-time indexing: the d x d
// matrix W = I/(gamma h) - J is factored in place with partial pivoting,
// the row interchanges done by selects, and the pivot row of each column
// kept so that a right-hand side is permuted by the same interchanges in
// the same order (and in reverse order for the transposed solve).
//
// Structural zeros: a system may declare the pattern of its Jacobian
// (JAC_ROWS).  From it the factorisation's possible fill is found at
// compile time, over every pivot order partial pivoting could choose, and
// the factorisation and the solves leave out the operations on entries that
// are zero whatever the values: the rows that cannot hold a column's pivot
// are neither compared nor interchanged, rows with a zero in the pivot
// column are not eliminated, and the solves skip the zeros of L and U.
// Each skipped operation would have added or moved an exact zero, so the
// results are those of the dense factorisation (up to the sign of a zero
// that no result reads).
namespace ens {

// c ? a : b for the values the factorisation moves by selects (a separate
// function so that a scalar type made of several parts can select them part
// by part).
template <class T>
__device__ __forceinline__ T pick(bool c, T a, T b) {
  return c ? a : b;
}

// 1 / x.  In FP64 the hardware estimate, two Newton steps, the second rounding
// a value good to 2^-96, and the fix-up of zeros, infinities and NaN: six
// instructions for the general division's eleven, of which a step has D + 2.
// The same as the division's to the bit over the whole range, subnormal
// arguments and results, overflow and the special values included
// (tests/test_gpu_inverse.py; over 2^32 arguments in each of five ranges of the
// normal numbers up to 2^1021 none differed either).
template <class T>
__device__ __forceinline__ T inverse(T x) {
  return T(1.0) / x;
}
__device__ __forceinline__ double inverse(double x) {
  double q = __builtin_amdgcn_rcp(x);
  q = fmaT(q, fmaT(-x, q, 1.0), q);
  q = fmaT(q, fmaT(-x, q, 1.0), q);
  return __builtin_amdgcn_div_fixup(q, x, 1.0);
}

// The nonzero pattern of row i of the Jacobian, bit j for column j: the
// system's JAC_ROWS if it declares one, else every column.
template <class S>
constexpr auto jac_row_of(int i, int) -> decltype(S::JAC_ROWS[0], 0u) {
  return S::JAC_ROWS[i];
}
template <class S>
constexpr unsigned jac_row_of(int, long) {
  return (1u << S::D) - 1u;
}

// The one interchange that the factorisation without the general ones still
// makes: in column SWAP[0], of that row and row SWAP[1], where the system
// declares it, else none.  (HIRES: column 1 holds 8.75 + 1 / (gamma h) less a
// little in row 1 and 8.32 in row 3, so rows 1 and 3 change places once h is
// large; of 430 interchanges in 128 trajectories at rtol 1e-6 354 are this one,
// and it makes one more entry of U and one of L possible.)
struct SwapAt {
  int col, row;
};
// (built-in systems only: a registered one's members are its own)
template <class S>
constexpr auto swap_of(int) -> decltype(SwapAt{S::SWAP[0], S::SWAP[1]}) {
  return S::ID < 1000 ? SwapAt{S::SWAP[0], S::SWAP[1]} : SwapAt{-1, -1};
}
template <class S>
constexpr SwapAt swap_of(long) {
  return SwapAt{-1, -1};
}

// What partial pivoting can make of W's pattern, step by step.  Rows are
// bitmasks of the columns that may be nonzero.  Step k: the rows at or
// below k with a possibly nonzero column-k entry are the pivot candidates;
// the interchange may give row k any candidate's pattern and a candidate
// row k's; then each row below k with a possibly nonzero column-k entry is
// eliminated, taking on the pivot row's pattern right of column k.  PIV
// false: the pattern where nothing but the system's SWAP is interchanged (row
// k is the only other candidate of column k).
template <int D>
struct LuPattern {
  unsigned cand[D];    // step k: candidate pivot rows (bit i), row k included
  unsigned before[D][D];  // step k: row patterns before the interchange
  unsigned pivrow[D];  // step k: the pivot row's pattern after the interchange
  unsigned elim[D];    // step k: rows below k that are eliminated
  unsigned fin[D];     // the factors: L below the diagonal, U and 1/U_kk on and above
};

template <class Sys, bool PIV = true>
constexpr LuPattern<Sys::D> lu_pattern() {
  constexpr int D = Sys::D;
  LuPattern<D> P{};
  unsigned M[D] = {};
  for (int i = 0; i < D; ++i) M[i] = jac_row_of<Sys>(i, 0) | (1u << i);
  for (int k = 0; k < D; ++k) {
    for (int i = 0; i < D; ++i) P.before[k][i] = M[i];
    unsigned cand = 1u << k, any = M[k];
    for (int i = k + 1; i < D; ++i)
      if ((PIV || (k == swap_of<Sys>(0).col && i == swap_of<Sys>(0).row)) &&
          ((M[i] >> k) & 1u)) {
        cand |= 1u << i;
        any |= M[i];
      }
    const unsigned mk = M[k];
    for (int i = k + 1; i < D; ++i)
      if ((cand >> i) & 1u) M[i] |= mk;
    M[k] = any;
    P.cand[k] = cand;
    P.pivrow[k] = any;
    const unsigned right = any & ~((2u << k) - 1u);
    unsigned el = 0;
    for (int i = k + 1; i < D; ++i)
      if ((M[i] >> k) & 1u) {
        el |= 1u << i;
        M[i] |= right;
      }
    P.elim[k] = el;
  }
  for (int i = 0; i < D; ++i) P.fin[i] = M[i];
  return P;
}

constexpr bool has(unsigned mask, int j) { return ((mask >> j) & 1u) != 0u; }

// W = I/(gamma h) - J(y) factored as P W = L U (unit L below the diagonal,
// U above it).  The pivot of column k is the first row i >= k with the
// largest |W_ik|; piv[k] records it.  The column is scaled by the pivot's
// reciprocal r_k = 1/U_kk (as LAPACK's getf2 does), and the diagonal keeps
// r_k, which the triangular solves multiply by: one division per pivot.
template <class Sys, class Tab, class T>
__device__ __forceinline__ void ros_factor(const T* y, const T* p, T h, T (&W)[Sys::D * Sys::D],
                                           int (&piv)[Sys::D]) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys>();
  Sys::jac(y, p, W);
  const T dg = inverse(T(T(Tab::GAMMA) * h));
#pragma unroll
  for (int i = 0; i < D * D; ++i) W[i] = -W[i];
#pragma unroll
  for (int i = 0; i < D; ++i) W[i * D + i] = W[i * D + i] + dg;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    int pk = k;
    T best = fabs(W[k * D + k]);
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.cand[k], i)) continue;  // a zero never beats |W_kk| >= 0
      const T v = fabs(W[i * D + k]);
      const bool gt = v > best;
      best = pick(gt, v, best);
      pk = gt ? i : pk;
    }
    piv[k] = pk;
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.cand[k], i)) continue;
      const bool sw = (pk == i);
#pragma unroll
      for (int j = 0; j < D; ++j) {
        if (!has(P.before[k][k] | P.before[k][i], j)) continue;  // both zero
        const T a = W[k * D + j], b = W[i * D + j];
        W[k * D + j] = pick(sw, b, a);
        W[i * D + j] = pick(sw, a, b);
      }
    }
    const T r = inverse(W[k * D + k]);
    W[k * D + k] = r;
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.elim[k], i)) continue;  // its multiplier is zero
      const T l = W[i * D + k] * r;
      W[i * D + k] = l;
#pragma unroll
      for (int j = k + 1; j < D; ++j)
        if (has(P.pivrow[k], j)) W[i * D + j] = fmaT(-l, W[k * D + j], W[i * D + j]);
    }
  }
}

// The factors without the general interchanges, indexed as the register array
// they are in; the solves take them with the smaller pattern.
template <class Sys, class T>
struct PlainMat {
  T w[Sys::D * Sys::D];
  bool sw;  // whether the system's SWAP was made
  __device__ __forceinline__ T operator[](int e) const { return w[e]; }
};

// Rows a and b of a vector interchanged where sw.
template <class T>
__device__ __forceinline__ void swap_where(bool sw, T& a, T& b) {
  const T t = a;
  a = pick(sw, b, a);
  b = pick(sw, t, b);
}

// The factorisation where every column's pivot is on the diagonal, or is the
// system's SWAP: the same operations as ros_factor's on a lane that makes no
// other interchange (what that does on the fill of other pivot orders adds
// exact zeros).  Returns whether the lane would have made one, in which case
// the factors are not ros_factor's.
template <class Sys, class Tab, class T>
__device__ __forceinline__ bool ros_factor_plain(const T* y, const T* p, T h,
                                                 PlainMat<Sys, T>& F) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys, false>();
  constexpr SwapAt SW = swap_of<Sys>(0);
  T(&W)[D * D] = F.w;
  Sys::jac(y, p, W);
  const T dg = inverse(T(T(Tab::GAMMA) * h));
#pragma unroll
  for (int i = 0; i < D * D; ++i) W[i] = -W[i];
#pragma unroll
  for (int i = 0; i < D; ++i) W[i * D + i] = W[i * D + i] + dg;
  bool other = false;
  F.sw = false;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    T best = fabs(W[k * D + k]);
    if constexpr (SW.col >= 0) {
      if (k == SW.col) {
        const T v = fabs(W[SW.row * D + k]);
        F.sw = v > best;
        best = pick(F.sw, v, best);
        // the first of the largest is the pivot
#pragma unroll
        for (int i = k + 1; i < D; ++i)
          if (has(P.elim[k], i) && i != SW.row) {
            const T o = fabs(W[i * D + k]);
            other |= o > best || (i < SW.row && F.sw && o == best);
          }
#pragma unroll
        for (int j = 0; j < D; ++j)
          if (has(P.before[k][k] | P.before[k][SW.row], j))
            swap_where(F.sw, W[k * D + j], W[SW.row * D + j]);
      }
    }
    const T r = inverse(W[k * D + k]);
    W[k * D + k] = r;
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.elim[k], i)) continue;  // its multiplier is zero
      if (k != SW.col) other |= fabs(W[i * D + k]) > best;
      const T l = W[i * D + k] * r;
      W[i * D + k] = l;
#pragma unroll
      for (int j = k + 1; j < D; ++j)
        if (has(P.pivrow[k], j)) W[i * D + j] = fmaT(-l, W[k * D + j], W[i * D + j]);
    }
  }
  return other;
}

template <class Mat>
struct Pivoted {
  static constexpr bool value = true;
};
template <class Sys, class T>
struct Pivoted<PlainMat<Sys, T>> {
  static constexpr bool value = false;
};

// Apply the interchanges of the factorisation to v, first to last (only
// the candidate rows of each step can have been interchanged).
template <class Sys, class T>
__device__ __forceinline__ void permute_fwd(const int (&piv)[Sys::D], T* v) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys>();
#pragma unroll
  for (int k = 0; k < D; ++k) {
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.cand[k], i)) continue;
      const bool sw = (piv[k] == i);
      const T a = v[k], b = v[i];
      v[k] = pick(sw, b, a);
      v[i] = pick(sw, a, b);
    }
  }
}

// Undo them (last to first): the permutation's transpose.
template <class Sys, class T>
__device__ __forceinline__ void permute_bwd(const int (&piv)[Sys::D], T* v) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys>();
#pragma unroll
  for (int k = D - 1; k >= 0; --k) {
#pragma unroll
    for (int i = k + 1; i < D; ++i) {
      if (!has(P.cand[k], i)) continue;
      const bool sw = (piv[k] == i);
      const T a = v[k], b = v[i];
      v[k] = pick(sw, b, a);
      v[i] = pick(sw, a, b);
    }
  }
}

// x = W^{-1} b in place: L z = P b forward, then U x = z backward (the
// diagonal holds 1/U_kk); the zeros of L and U skipped.
template <class Sys, class T, class Mat>
__device__ __forceinline__ void lu_solve(const Mat& W, const int (&piv)[Sys::D], T* x) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys, Pivoted<Mat>::value>();
  constexpr SwapAt SW = swap_of<Sys>(0);
  if constexpr (Pivoted<Mat>::value)
    permute_fwd<Sys, T>(piv, x);
  else if constexpr (SW.col >= 0)
    swap_where(W.sw, x[SW.col], x[SW.row]);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    T acc = x[i];
#pragma unroll
    for (int j = 0; j < i; ++j)
      if (has(P.fin[i], j)) acc = fmaT(-W[i * D + j], x[j], acc);
    x[i] = acc;
  }
#pragma unroll
  for (int i = D - 1; i >= 0; --i) {
    T acc = x[i];
#pragma unroll
    for (int j = i + 1; j < D; ++j)
      if (has(P.fin[i], j)) acc = fmaT(-W[i * D + j], x[j], acc);
    x[i] = acc * W[i * D + i];
  }
}

// z = W^{-T} b in place: U^T v = b forward, L^T w = v backward, z = P^T w.
// W: the factors (a register array, or a PlainMat).
template <class Sys, class T, class Mat>
__device__ __forceinline__ void lu_solve_t(const Mat& W, const int (&piv)[Sys::D], T* z) {
  constexpr int D = Sys::D;
  constexpr LuPattern<D> P = lu_pattern<Sys, Pivoted<Mat>::value>();
#pragma unroll
  for (int i = 0; i < D; ++i) {
    T acc = z[i];
#pragma unroll
    for (int j = 0; j < i; ++j)
      if (has(P.fin[j], i)) acc = fmaT(-W[j * D + i], z[j], acc);
    z[i] = acc * W[i * D + i];
  }
#pragma unroll
  for (int i = D - 1; i >= 0; --i) {
    T acc = z[i];
#pragma unroll
    for (int j = i + 1; j < D; ++j)
      if (has(P.fin[j], i)) acc = fmaT(-W[j * D + i], z[j], acc);
    z[i] = acc;
  }
  constexpr SwapAt SW = swap_of<Sys>(0);
  if constexpr (Pivoted<Mat>::value)
    permute_bwd<Sys, T>(piv, z);
  else if constexpr (SW.col >= 0)
    swap_where(W.sw, z[SW.col], z[SW.row]);
}

// Stage input Y_i = y + sum_{j<i} A_ij u_j (index order, first term a
// product, the rest fmas).
template <class Tab, int D, class T>
__device__ __forceinline__ void ros_input(int i, const T* y, const T (&u)[Tab::S][D], T* Yi) {
#pragma unroll
  for (int c = 0; c < D; ++c) {
    T acc = T(0);
    bool first = true;
#pragma unroll
    for (int j = 0; j < Tab::S; ++j) {
      if (j < i && Tab::A[i][j] != 0.0) {
        acc = first ? cmul(Tab::A[i][j], u[j][c]) : cfma(Tab::A[i][j], u[j][c], acc);
        first = false;
      }
    }
    Yi[c] = first ? y[c] : y[c] + acc;
  }
}

// The increments u_1..u_NSC of one step from y with step h (h != 0), the
// factors left in W/piv for the reverse, and y_new: Y_s + u_s, or the last
// stage input Y_s (NEW_AT_INPUT).  NSC = S forms every stage (a trial step
// needs the last for its error estimate); NSC = SU only those that enter
// y_new (a replay).  W: the factors (a register array, or a PlainMat).
template <class Sys, class Tab, class T, class Mat, int NSC = Tab::S>
__device__ __forceinline__ void ros_stages(const T* y, const T* p, T h, const Mat& W,
                                           const int (&piv)[Sys::D], T (&u)[Tab::S][Sys::D],
                                           T* ynew) {
  constexpr int D = Sys::D, NS = Tab::S;
  static_assert(NSC == NS || (NSC == Tab::SU && Tab::NEW_AT_INPUT),
                "a step that stops short of the last stage needs y_new at its input");
  const T hinv = inverse(h);
  T Yi[D];
#pragma unroll
  for (int i = 0; i < NSC; ++i) {
    ros_input<Tab, D, T>(i, y, u, Yi);
    T F[D];
    Sys::rhs(Yi, p, F);
#pragma unroll
    for (int c = 0; c < D; ++c) {
      T acc = T(0);
      bool first = true;
#pragma unroll
      for (int j = 0; j < i; ++j) {
        if (Tab::C[i][j] != 0.0) {
          acc = first ? cmul(Tab::C[i][j], u[j][c]) : cfma(Tab::C[i][j], u[j][c], acc);
          first = false;
        }
      }
      u[i][c] = first ? F[c] : fmah(acc, hinv, F[c]);
    }
    lu_solve<Sys, T, Mat>(W, piv, u[i]);
  }
  if constexpr (Tab::NEW_AT_INPUT) {
    ros_input<Tab, D, T>(NS - 1, y, u, ynew);
  } else {
#pragma unroll
    for (int c = 0; c < D; ++c) ynew[c] = Yi[c] + u[NS - 1][c];
  }
}

template <class Sys, class Tab, class T, int NSC = Tab::S>
__device__ __forceinline__ void ros_step(const T* y, const T* p, T h, T (&W)[Sys::D * Sys::D],
                                         int (&piv)[Sys::D], T (&u)[Tab::S][Sys::D], T* ynew) {
  ros_factor<Sys, Tab, T>(y, p, h, W, piv);
  ros_stages<Sys, Tab, T, T[Sys::D * Sys::D], NSC>(y, p, h, W, piv, u, ynew);
}

// Error estimate e = sum_j E_j u_j (Rodas4: u_6 itself).
template <class Tab, int D, class T>
__device__ __forceinline__ void ros_errvec(const T (&u)[Tab::S][D], T* e) {
#pragma unroll
  for (int c = 0; c < D; ++c) {
    T acc = T(0);
    bool first = true;
#pragma unroll
    for (int j = 0; j < Tab::S; ++j) {
      if (Tab::E[j] != 0.0) {
        acc = first ? cmul(Tab::E[j], u[j][c]) : cfma(Tab::E[j], u[j][c], acc);
        first = false;
      }
    }
    e[c] = acc;
  }
}

// Whether a wavefront tries the factorisation without interchanges.  A
// registered system of d >= 6 that changes rows in step after step would pay
// for it in vain each time (an 8 x 8 dense one in nearly every step, 16,384
// trajectories, record / replay: always tried 4.51 / 4.15 ms, so 3.16 / 2.94,
// always general 3.86 / 3.41); so after five failures in a row it is tried in
// every ninth step only, until it succeeds.  With d <= 5 the vain attempt costs
// less than the shorter general step gains (d = 5, the same way: 1.21 / 1.14
// ms, always general 1.27 / 1.15), and for the built-in systems it hardly ever
// fails, so those always try.  Either way gives the same values.
struct RosTry {
  static constexpr int FAILS = 5, WAIT = 8;
  int failed = 0;  // in a row (the same in every lane of the wavefront)
  int wait = 0;    // steps until the next attempt
};

// One step: y_new and, if ERR, the error estimate e.  Where no lane of the
// wavefront interchanges rows, but for the system's SWAP (every trip of the
// Robertson workloads, 96 % of the HIRES ones at rtol 1e-6 and 81 % at 1e-4;
// 83 % and 58 % without the SWAP), the factorisation and the solves without
// the general interchanges and their fill serve, with the same values;
// otherwise the whole wavefront takes the general ones, at three to five times
// the instructions (HIRES, 2^17: the SWAP takes the record from 3.31 to 2.93
// ms, the sweep from 6.39 to 5.61).  The branch is marked unlikely, so that what the
// general path has no registers for moves inside it.
template <class Sys, class Tab, class T, int NSC, bool ERR>
__device__ __forceinline__ void ros_eval(const T* y, const T* p, T h, T* ynew, T* e,
                                         RosTry& rt) {
  constexpr int D = Sys::D;
  constexpr bool ALWAYS = Sys::ID < 1000 || D < 6;
  if (ALWAYS || __builtin_amdgcn_readfirstlane(rt.wait) == 0) {
    PlainMat<Sys, T> F;
    if (__builtin_expect(!__any(ros_factor_plain<Sys, Tab, T>(y, p, h, F)), 1)) {
      T u[Tab::S][D];
      int piv[D];
      ros_stages<Sys, Tab, T, PlainMat<Sys, T>, NSC>(y, p, h, F, piv, u, ynew);
      if constexpr (ERR) ros_errvec<Tab, D, T>(u, e);
      if constexpr (!ALWAYS) rt.failed = 0;
      return;
    }
    if constexpr (!ALWAYS) {
      rt.failed = __builtin_amdgcn_readfirstlane(rt.failed) + 1;
      rt.wait = rt.failed < RosTry::FAILS ? 0 : RosTry::WAIT;
    }
  } else {
    rt.wait = __builtin_amdgcn_readfirstlane(rt.wait) - 1;
  }
  T W[D * D], u[Tab::S][D];
  int piv[D];
  ros_step<Sys, Tab, T, NSC>(y, p, h, W, piv, u, ynew);
  if constexpr (ERR) ros_errvec<Tab, D, T>(u, e);
}

// The increments u_1..u_SU as the reverse reads them: a register array, or
// the lane's LDS slots (entry (q, c) at base[(q D + c) * 256 + lane]).  From LDS
// each stage reads what it needs afresh (fetch is a compiler memory barrier);
// a read costs half an instruction a double, the moves to and from the
// accumulation registers, where the array would wait, four.
template <class T, int D>
struct RegIncr {
  const T (*u)[D];
  __device__ __forceinline__ T operator()(int q, int c) const { return u[q][c]; }
  __device__ __forceinline__ void fetch() const {}
};
template <class T, int D>
struct LdsIncr {
  T* base;
  __device__ __forceinline__ T operator()(int q, int c) const {
    return base[(q * D + c) * 256 + threadIdx.x];
  }
  __device__ __forceinline__ void put(int q, const T* v) const {
#pragma unroll
    for (int c = 0; c < D; ++c) base[(q * D + c) * 256 + threadIdx.x] = v[c];
  }
  __device__ __forceinline__ void fetch() const { __asm__ __volatile__("" ::: "memory"); }
};

template <class Tab>
constexpr bool m_nonzero_below_su() {
  for (int i = 0; i < Tab::SU; ++i)
    if (Tab::M[i] == 0.0) return false;
  return true;
}

// Reverse of one step (W, piv, u from ros_step or ros_factor_plain and
// ros_stages at the same y, h): with the
// output cotangent w, lam_in = d(y_new)/dy^T w and gp += d(y_new)/dp^T w.
//   ubar_i = M_i w + sum_{l>i} (A_li Ybar_l + C_li rbar_l / h)   (l from s down)
//   rbar_i = W^{-T} ubar_i,  Ybar_i = f_y(Y_i)^T rbar_i,  gp += f_p(Y_i)^T rbar_i
//   lam_in = w + sum_i Ybar_i + d/dy sum_i rbar_i^T J(y) u_i,
// the last term (and its p part, into gp) from each stage in turn.  Stage
// cotangents are pushed into running sums as they are formed.  Only the SU
// stages that enter y_new are reversed (a stage that serves the error
// estimate alone has a zero cotangent).
template <class Sys, class Tab, class T, class Mat, class Incr>
__device__ __forceinline__ void ros_step_vjp(const T* y, const T* p, T h, const Mat& W,
                                             const int (&piv)[Sys::D], const Incr& u,
                                             const T* w, T* lam_in, T* gp) {
  constexpr int D = Sys::D, NS = Tab::SU;
  static_assert(m_nonzero_below_su<Tab>(), "every stage sum starts with its M term");
  // Stages from KEEP up are pulled: their Ybar and rbar / h are kept until
  // stage KEEP is done, and only then pushed into the sums of the stages
  // below, which take later ones as they come.  Each sum gets its terms in
  // the same order either way; with all of them pushed at once, 6 x D sums
  // and 6 x D increments are live together at the last stage, with this at
  // most 4 of each (or the kept two stages).
  constexpr int KEEP = NS >= 4 ? NS - 2 : NS;
  const T hinv = inverse(h);
  T ub[NS][D], gJ[D], kY[NS][D], kt[NS][D];
#pragma unroll
  for (int c = 0; c < D; ++c) {
    lam_in[c] = w[c];
    gJ[c] = T(0);
  }
  auto open = [&](int i) {  // ub_i = M_i w and the kept stages' terms
#pragma unroll
    for (int c = 0; c < D; ++c) {
      T acc = T(Tab::M[i]) * w[c];
#pragma unroll
      for (int l = NS - 1; l >= KEEP; --l) {
        if (l <= i) continue;
        if (Tab::A[l][i] != 0.0) acc = fmaT(T(Tab::A[l][i]), kY[l][c], acc);
        if (Tab::C[l][i] != 0.0) acc = fmaT(T(Tab::C[l][i]), kt[l][c], acc);
      }
      ub[i][c] = acc;
    }
  };
  if constexpr (KEEP == NS) {
#pragma unroll
    for (int i = 0; i < NS; ++i) open(i);
  }
#pragma unroll
  for (int i = NS - 1; i >= 0; --i) {
    if (i >= KEEP) open(i);
    T rb[D], tb[D], Yi[D], Yb[D], ui[D];
    u.fetch();
#pragma unroll
    for (int c = 0; c < D; ++c) {
      rb[c] = ub[i][c];
      ui[c] = u(i, c);
    }
    lu_solve_t<Sys, T, Mat>(W, piv, rb);
#pragma unroll
    for (int c = 0; c < D; ++c) tb[c] = hinv * rb[c];
#pragma unroll
    for (int c = 0; c < D; ++c) {
      T acc = T(0);
      bool first = true;
#pragma unroll
      for (int j = 0; j < i; ++j) {
        if (Tab::A[i][j] != 0.0) {
          acc = first ? T(Tab::A[i][j]) * u(j, c) : fmaT(T(Tab::A[i][j]), u(j, c), acc);
          first = false;
        }
      }
      Yi[c] = first ? y[c] : y[c] + acc;
    }
    Sys::vjp(Yi, p, rb, Yb, gp);
#pragma unroll
    for (int c = 0; c < D; ++c) lam_in[c] = lam_in[c] + Yb[c];
    Sys::jac_vjp(y, p, rb, ui, gJ, gp);
    if (i >= KEEP) {
#pragma unroll
      for (int c = 0; c < D; ++c) {
        kY[i][c] = Yb[c];
        kt[i][c] = tb[c];
      }
      if (i == KEEP) {
#pragma unroll
        for (int j = 0; j < i; ++j) open(j);
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < i; ++j) {
#pragma unroll
      for (int c = 0; c < D; ++c) {
        if (Tab::A[i][j] != 0.0) ub[j][c] = fmaT(T(Tab::A[i][j]), Yb[c], ub[j][c]);
        if (Tab::C[i][j] != 0.0) ub[j][c] = fmaT(T(Tab::C[i][j]), tb[c], ub[j][c]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < D; ++c) lam_in[c] = lam_in[c] + gJ[c];
}

// One step from yb recomputed and reversed from its factors: cot(ys, w) gives
// the cotangent w of the state ys it reaches; lin = d(ys)/dyb^T w,
// g += d(ys)/dp^T w.  U_LDS (d >= 6): between the two the increments wait in
// the lane's LDS slots sU.
template <class Sys, class Tab, class T, bool U_LDS, class Mat, class Cot>
__device__ __forceinline__ void ros_reverse_of(const T* yb, const T* p, T h, const Mat& W,
                                               const int (&piv)[Sys::D], T* sU, Cot& cot, T* lin,
                                               T* g) {
  constexpr int D = Sys::D;
  T u[Tab::S][D], ys[D], w[D];
  ros_stages<Sys, Tab, T, Mat, Tab::SU>(yb, p, h, W, piv, u, ys);
  if constexpr (U_LDS) {
    const LdsIncr<T, D> ul{sU};
#pragma unroll
    for (int q = 0; q < Tab::SU; ++q) ul.put(q, u[q]);
    cot(ys, w);
    ros_step_vjp<Sys, Tab, T>(yb, p, h, W, piv, ul, w, lin, g);
  } else {
    cot(ys, w);
    ros_step_vjp<Sys, Tab, T>(yb, p, h, W, piv, RegIncr<T, D>{u}, w, lin, g);
  }
}

// Without interchanges in the wavefront as ros_eval; otherwise the general
// factorisation.
template <class Sys, class Tab, class T, bool U_LDS, class Cot>
__device__ __forceinline__ void ros_reverse(const T* yb, const T* p, T h, T* sU, Cot& cot, T* lin,
                                            T* g) {
  constexpr int D = Sys::D;
  int piv[D];
  PlainMat<Sys, T> F;
  if (__builtin_expect(!__any(ros_factor_plain<Sys, Tab, T>(yb, p, h, F)), 1)) {
    ros_reverse_of<Sys, Tab, T, U_LDS>(yb, p, h, F, piv, sU, cot, lin, g);
  } else {
    T W[D * D];
    ros_factor<Sys, Tab, T>(yb, p, h, W, piv);
    ros_reverse_of<Sys, Tab, T, U_LDS>(yb, p, h, W, piv, sU, cot, lin, g);
  }
}

// Mean square (the RMS norm squared) of the scaled error estimate against
// atol + rtol max(|y|, |y_new|); the reciprocal of each scale as the
// explicit pairs' recip (the hardware estimate and one Newton step).
template <int D, class T>
__device__ __forceinline__ double ros_ms(const T* y, const T* ynew, const T* e, double rtol,
                                         double atol) {
  double ss = 0.0;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double sc = fmaT(rtol, (double)max_abs(y[c], ynew[c]), atol);
    const double q0 = __builtin_amdgcn_rcp(sc);
    const double q = fmaT(q0, fmaT(-sc, q0, 1.0), q0);
    const double r = (double)e[c] * q;
    ss = c == 0 ? r * r : fmaT(r, r, ss);
  }
  return ss * (1.0 / (double)D);
}

}  // namespace ens
