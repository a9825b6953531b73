// 1D level step of ARK-based RIDC and of RIDC with a nonlinear stiff term, for gfx950.
//
// One workgroup advances one (instance, level) work item by one pipeline step: it computes the
// level's value at t_{n+1} from its value at t_n with the s stages of the level's IMEX pair
// (section II):
//   Y_i = y_n + I_i + dt sum_{l<i} (AS_il K^S_l + AN_il K^N_l) + dt AS_ii K^S_i,
//   K^S_i = f^S(Y_i) - f^S(eta(t_n + c_i dt)),  K^N_i = f^N(Y_i) - f^N(eta(t_n + c_i dt)),
// where, for a corrector (section III-A, the integral form of the error equation), eta is the
// previous level interpolated through its S stored nodes (the section III-C window widened to
// S nodes) and I_i = int_{t_n}^{t_n + c_i dt} f(eta); for the predictor I_i and the subtracted
// terms are zero.  Every pair is stiffly accurate, so y_{n+1} = Y_s.  Stage 0 is explicit with
// c_0 = 0 (Y_0 = y_n); every other stage solves y - tau f^S(y) = rhs, tau = dt AS_ii:
//  - f^S = nu Lap_h: one tridiagonal solve (I - tau nu D2) y = rhs;
//  - f^S = nu Lap_h + kappa g: Newton's method (section III-B), each iterate solving the
//    Jacobian system (I - tau (nu D2 + kappa diag g'(y))) delta = rhs - (y - tau f^S(y)) and
//    stopping when the update reaches rounding.
// The implicit stage derivative is taken from the stage equation, f^S(Y_i) = (Y_i - rhs)/tau.
// The new value and f = f^S + f^N of it (read by the next level's window) go to the level's
// rings.
//
// Layout.  Thread t of T owns the M consecutive rows g0 = t M .. g0 + M - 1 in registers; rows
// at or past n are padding (identity rows, value 0).  Stencil neighbours come from global memory
// (loaded vectors) or from the adjacent lanes and, between waves, LDS (computed values).
//
// Every implicit solve is a correction (the FP64 residual of the value so far on the right), a linear
// stage's as well as a Newton iterate's, so the rounding of the solver scales with the correction and
// not with the value; solves follow until that rounding is below the value's own (stage_solve).
//
// Tridiagonal solve (a partition method in three levels, one workgroup barrier):
//  1. each thread eliminates its block, so that every row couples to the last unknown of the block
//     before and of its own; substituting the next block's first row leaves one tridiagonal row
//     per thread, in the blocks' last unknowns;
//  2. parallel cyclic reduction with DPP moves inside the rows of 16 lanes, whose last lane stays
//     an unknown: two equations per 16 threads (its first and its last unknown) go to LDS;
//  3. every wave reads all of them (at most 32 groups, one per lane), joins them into a
//     tridiagonal system of the groups' last unknowns, reduces its rows of 16 lanes the same way and
//     eliminates the last unknowns of the two rows in order.
// The unknowns come back the same way: by registers, lane moves and no further barrier.
// Periodic grids (cyclic systems) take the Sherman-Morrison correction: the cyclic matrix is a
// tridiagonal one plus a rank-one term, so one solve with two right-hand sides and a scalar
// combination give the cyclic solution.
//
// Bound: latency and FP64 issue inside one compute unit per level (a solve is some 720 FP64 and 700
// other instructions a lane with 16 rows; the level's vectors cross its L2 port once a stage).
// Reducing all 2 T block rows through LDS, one barrier per stage, with every vector in grid order
// and re-read per stage, took 180 us per step of ARK3 + FBE and 181 us of RIDC4 with the cubic
// reaction (9 Newton iterates) at n = 8192; this form takes 63 and 71.
#include "ridc_internal.h"

namespace ridc {

namespace {

// Global-memory views of descriptor pointers.  Pointers read from a table carry no address space,
// so the compiler would emit flat instructions, which also count against the LDS wait counter.
typedef __attribute__((address_space(1))) double gdbl;
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) dbl2 gdbl2;
__device__ __forceinline__ gdbl* gp(double* p) { return (gdbl*)p; }
__device__ __forceinline__ const gdbl* gp(const double* p) { return (const gdbl*)p; }

// g and g' of the stiff reaction, by selects (fs is uniform; a branch per row would cut the row
// loops into blocks that cannot overlap)
__device__ __forceinline__ double react(int fs, double u) {
  const double q = u * (1.0 - u), c = u - u * u * u;
  return fs == RIDC_FS_CUBIC ? c : (fs == RIDC_FS_LOGISTIC ? q : 0.0);
}
__device__ __forceinline__ double react_prime(int fs, double u) {
  const double q = 1.0 - 2.0 * u, c = 1.0 - 3.0 * u * u;
  return fs == RIDC_FS_CUBIC ? c : (fs == RIDC_FS_LOGISTIC ? q : 0.0);
}

// f_E of M rows: u[0] .. u[M+1] are rows g0-1 .. g0+M (the kind is branched on once)
template <int M>
__device__ __forceinline__ void fe_rows(int fe, double ce, const double (&u)[M + 2],
                                        double (&out)[M]) {
  auto all = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < M; ++i) out[i] = f(u[i], u[i + 1], u[i + 2]);
  };
  if (fe == RIDC_FE_ADVECT_C2) all([&](double a, double, double b) { return -ce * (b - a); });
  else if (fe == RIDC_FE_LOGISTIC) all([](double, double x, double) { return x * (1.0 - x); });
  else if (fe == RIDC_FE_ADVECT_UPWIND && ce >= 0.0)
    all([&](double a, double x, double) { return -ce * (x - a); });
  else if (fe == RIDC_FE_ADVECT_UPWIND) all([&](double, double x, double b) { return -ce * (b - x); });
  else if (fe == RIDC_FE_BURGERS)
    all([&](double a, double, double b) { return -ce * (b * b - a * a); });
  else all([](double, double, double) { return 0.0; });
}

// Per-workgroup state: problem data, thread position and the LDS regions.  A region has two
// buffers used alternately, so that one barrier per use keeps readers and writers apart (pointer
// arithmetic, not an indexed array, so that the context stays in registers).
struct Ctx {
  int n, T, t, g0, lane, wave, fe, fs;
  double ce, nu_h2, kappa;
  double* grp;     // group equations: (3 + NR - 1) + (3 + NR - 1) values x kGroups, per buffer
  double* ex;      // wave edges: first and last rows (16 waves each), rows 0 and n-1, maxima
  double* rhs;     // stage right-hand side (M >= 16): row i of thread t at i T + t
  int gk, xk;      // buffer toggles
};
constexpr int kGroups = kImexMaxThreads / 16;
constexpr int kGroupRows = kGroups / 16;         // rows of 16 lanes that hold one group a lane
static_assert(kGroups % 16 == 0 && kGroups <= 64, "one group per lane of a wave");
constexpr int kWaves = kImexMaxThreads / 64;
// values of one edge buffer: per right-hand side 2 per wave and 2 rows; then 2 maxima per wave
__host__ __device__ constexpr int ex_doubles(int NR) { return NR * (2 * kWaves + 2) + 2 * kWaves; }
__host__ __device__ constexpr int grp_doubles(int NR) { return 2 * (2 + NR) * kGroups; }

// LDS doubles of a workgroup of T threads (layout as in imex_step)
inline size_t lds_doubles(int NR, int M, int T) {
  return 2 * (size_t)grp_doubles(NR) + 2 * (size_t)ex_doubles(NR) + (M >= 16 ? (size_t)M * T : 0);
}

// v of another lane, moved as two 32-bit halves by DPP; lanes without a source take `old`.  All
// lanes of the wave are active.  kUp/kDown + k: the lane k below / above in the same row of 16;
// kWaveUp / kWaveDown: the adjacent lane of the wave.
constexpr int kUp = 0x110, kDown = 0x100, kWaveUp = 0x138, kWaveDown = 0x130;
template <int CTRL>
__device__ __forceinline__ double move0(double v) {   // lanes without a source take 0
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ double move(double v, double old) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, 0xF, 0xF,
                                             false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, 0xF, 0xF,
                                             false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// 1 / b (b of moderate size) from the hardware estimate (2^-24) and two Newton steps, about an
// ulp.  Used in the solves only, whose results are corrections.  (With one step, 2^-48, in the solves
// of a stiff reaction, the cubic one's steps took 2-3 % less and ended 1.5 times as far from the
// exact solution: a last update of some 1e-15 is not exact enough then.)
__device__ __forceinline__ double recip(double b) {
  double x = __builtin_amdgcn_rcp(b);
  x = __builtin_fma(__builtin_fma(-b, x, 1.0), x, x);
  return __builtin_fma(__builtin_fma(-b, x, 1.0), x, x);
}

// The largest v of the wave: of doubles (NaN passed over), or of non-negative ints.
__device__ __forceinline__ double larger(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ int larger(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, move<0x121>(v, v));
  v = fmax(v, move<0x122>(v, v));
  v = fmax(v, move<0x124>(v, v));
  v = fmax(v, move<0x128>(v, v));
  return fmax(fmax(lane_value(v, 0), lane_value(v, 16)),
              fmax(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ int wave_max(int v) {
  v = larger(v, __builtin_amdgcn_update_dpp(v, v, 0x121, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(v, v, 0x122, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(v, v, 0x124, 0xF, 0xF, false));
  v = larger(v, __builtin_amdgcn_update_dpp(v, v, 0x128, 0xF, 0xF, false));
  return larger(larger(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                larger(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Publish the wave's first and last rows (and rows 0 and n-1 from their owners), then read the
// neighbours of the block: xl = row g0-1, xr = row g0+M (0 past either end), w0 = row 0, wn = row
// n-1 (periodic grids only).  With `mx`, also the largest mx[0] and mx[1] over the workgroup.
template <int M, int NR, bool PER, typename Max = double>
__device__ __forceinline__ void exchange(Ctx& c, const double (&x)[NR][M], double (&xl)[NR],
                                         double (&xr)[NR], double (&w0)[NR], double (&wn)[NR],
                                         Max* mx = nullptr) {
  double* e = c.ex + (c.xk & 1) * ex_doubles(NR);
  c.xk++;
  double* ends = e + NR * 2 * kWaves;
  Max* red = reinterpret_cast<Max*>(e + NR * (2 * kWaves + 2));
  if (mx) {
#pragma unroll
    for (int k = 0; k < 2; ++k) mx[k] = wave_max(mx[k]);
  }
  if (c.lane == 0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) e[2 * (r * kWaves + c.wave)] = x[r][0];
    if (mx) {
      red[2 * c.wave] = mx[0];
      red[2 * c.wave + 1] = mx[1];
    }
  }
  if (c.lane == 63) {
#pragma unroll
    for (int r = 0; r < NR; ++r) e[2 * (r * kWaves + c.wave) + 1] = x[r][M - 1];
  }
  if constexpr (PER) {
    if (c.t == 0) {
#pragma unroll
      for (int r = 0; r < NR; ++r) ends[2 * r] = x[r][0];
    }
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (c.g0 + i == c.n - 1) {
#pragma unroll
        for (int r = 0; r < NR; ++r) ends[2 * r + 1] = x[r][i];
      }
  }
  __syncthreads();
  const int nw = c.T >> 6;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const double below = c.wave > 0 ? e[2 * (r * kWaves + c.wave - 1) + 1] : 0.0;
    const double above = c.wave + 1 < nw ? e[2 * (r * kWaves + c.wave + 1)] : 0.0;
    xl[r] = move<kWaveUp>(x[r][M - 1], below);
    xr[r] = move<kWaveDown>(x[r][0], above);
    if constexpr (PER) {
      w0[r] = ends[2 * r];
      wn[r] = ends[2 * r + 1];
    } else {
      w0[r] = wn[r] = 0.0;
    }
  }
  if (mx) {
    // all waves' values at once (a missing wave's read the last one's)
    Max a[kWaves], b[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      a[w] = red[2 * (w < nw ? w : nw - 1)];
      b[w] = red[2 * (w < nw ? w : nw - 1) + 1];
    }
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      a[0] = larger(a[0], a[w]);
      b[0] = larger(b[0], b[w]);
    }
    mx[0] = a[0];
    mx[1] = b[0];
  }
}

// Vectors in global memory (rings and workspace) keep their rows in block order: row i of thread t
// at i T + t, padding rows zero, so that a wave's access is contiguous whatever M is (with rows in
// grid order every lane of a load touches a line of its own: 80 against 102 us per step, ARK3 + FBE
// at n = 8192, M = 16).

// This thread's rows.
template <int M>
__device__ __forceinline__ void load_rows(const Ctx& c, const gdbl* __restrict__ v,
                                          double (&out)[M]) {
#pragma unroll
  for (int i = 0; i < M; ++i) out[i] = (v + i * c.T)[(unsigned)c.t];
}
template <int M>
__device__ __forceinline__ void store_rows(const Ctx& c, gdbl* __restrict__ v,
                                           const double (&x)[M]) {
#pragma unroll
  for (int i = 0; i < M; ++i) (v + i * c.T)[(unsigned)c.t] = x[i];
}
// The same, zero in the padding rows.
template <int M>
__device__ __forceinline__ void store_real(const Ctx& c, gdbl* __restrict__ v,
                                           const double (&x)[M]) {
#pragma unroll
  for (int i = 0; i < M; ++i) (v + i * c.T)[(unsigned)c.t] = c.g0 + i < c.n ? x[i] : 0.0;
}

// Rows g0-1 .. g0+M: zero ghosts (Dirichlet), or wrapped (periodic).
template <int M, bool PER>
__device__ __forceinline__ void load_halo(const Ctx& c, const gdbl* __restrict__ v,
                                          double (&out)[M + 2]) {
  const unsigned lt = c.t > 0 ? c.t - 1 : 0, rt = c.t + 1 < c.T ? c.t + 1 : c.T - 1;
  const double l = (v + (M - 1) * c.T)[lt], r = v[rt];
#pragma unroll
  for (int i = 0; i < M; ++i) out[i + 1] = (v + i * c.T)[(unsigned)c.t];
  out[0] = c.t > 0 ? l : 0.0;
  out[M + 1] = c.t + 1 < c.T ? r : 0.0;
  if constexpr (PER) {
    const int q = (c.n - 1) / M, k = (c.n - 1) % M;           // row n-1 sits in thread q, row k
    const double first = v[0], last = v[k * c.T + q];
    if (c.t == 0) out[0] = last;
#pragma unroll
    for (int i = 1; i <= M; ++i)
      if (c.g0 + i == c.n) out[i + 1] = first;
  }
}

// f^S = nu Lap_h u + kappa g(u) and f^N at one row.
__device__ __forceinline__ double fstiff(const Ctx& c, double um, double u0, double up) {
  return c.nu_h2 * (up - 2.0 * u0 + um) + c.kappa * react(c.fs, u0);
}

// One stage of parallel cyclic reduction over the lanes of a row of 16, stride S: row q,
// a x_{q-S} + x_q + c x_{q+S} = d, takes rows q -+ S.  Past the row's ends the coupling stays (to
// the unknown before or after the row): a missing row reads as (a, c, d) = (-1, 0, 0) below and
// (0, -1, 0) above.
template <int S, int NR>
__device__ __forceinline__ void reduce_stage(double& a, double& c, double (&d)[NR]) {
  const double am = move<kUp + S>(a, -1.0), cm = move0<kUp + S>(c);
  const double ap = move0<kDown + S>(a), cp = move<kDown + S>(c, -1.0);
  double dm[NR], dp[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    dm[k] = move0<kUp + S>(d[k]);
    dp[k] = move0<kDown + S>(d[k]);
  }
  const double inv = recip(__builtin_fma(-a, cm, __builtin_fma(-c, ap, 1.0)));
#pragma unroll
  for (int k = 0; k < NR; ++k)
    d[k] = __builtin_fma(-a, dm[k], __builtin_fma(-c, dp[k], d[k])) * inv;
  a = -a * am * inv;
  c = -c * cp * inv;
}
template <int NR>
__device__ __forceinline__ void reduce_row(double& a, double& c, double (&d)[NR]) {
  reduce_stage<1, NR>(a, c, d);
  reduce_stage<2, NR>(a, c, d);
  reduce_stage<4, NR>(a, c, d);
  reduce_stage<8, NR>(a, c, d);
}

// Solve the tridiagonal system with off-diagonals -r (zero at Dirichlet ends; periodic: cyclic
// with corners -r) whose diagonal b_g and right-hand side d_g this thread's rows get from
// rows(i, b, d).  x receives this thread's rows of the solution (padding rows: 0).
// Periodic (PER): d0 is the diagonal of row 0; the second right-hand side is the rank-one
// correction's vector.
template <int M, bool PER, typename Rows>
__device__ __forceinline__ void tri_solve(Ctx& c, double r, double d0, Rows rows,
                                          double (&x)[M]) {
  constexpr int NR = PER ? 2 : 1;
  const int n = c.n, g0 = c.g0;
  // Down the block: x_i = D_i - A_i x_{-1} + E_i x_{i+1}, x_{-1} the last row of the block before.
  // Only E = r / pivot and D are kept: A_i = E_i A_{i-1}, and the block's first row in terms of
  // x_{-1} and x_{M-1}, x_0 = d0 - a0 x_{-1} - c0 x_{M-1}, is summed on the way (w = E_0 .. E_{i-1}).
  // Padding rows have E = D = 0: their value 0 is the ghost row after row n-1.
  double E[M], D[NR][M], a0 = 0.0, d0s[NR], w = 1.0, A = 0.0;
#pragma unroll
  for (int q = 0; q < NR; ++q) d0s[q] = 0.0;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int g = g0 + i;
    double b, d[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) d[q] = 0.0;
    rows(i, b, d[0]);
    if (PER) {
      if (g == 0) {
        b += d0;            // b - gamma, gamma = -d0
        d[NR - 1] = -d0;    // u_0 = gamma
      }
      if (g == n - 1) {
        b += r * r / d0;    // b - a_0 c_{n-1} / gamma
        d[NR - 1] = -r;     // u_{n-1} = c_{n-1}
      }
    }
    if (i > 0) b = __builtin_fma(-r, E[i - 1], b);
    double inv = recip(b);
    inv = g < n ? inv : 0.0;
    E[i] = r * inv;
#pragma unroll
    for (int q = 0; q < NR; ++q)
      D[q][i] = (i > 0 ? __builtin_fma(r, D[q][i - 1], d[q]) : d[q]) * inv;
    A = i > 0 ? E[i] * A : (g == 0 ? 0.0 : -E[0]);
    if (i < M - 1) {
      a0 = __builtin_fma(w, A, a0);
#pragma unroll
      for (int q = 0; q < NR; ++q) d0s[q] = __builtin_fma(w, D[q][i], d0s[q]);
      w *= E[i];
    }
  }
  const double A0 = g0 == 0 ? 0.0 : -E[0], c0 = -w, Cl = -E[M - 1];
  // one row per thread: the next block's first row replaces its unknown.  The last lane of a row
  // of 16 keeps its equation for later and stands as the unknown after the others (0, -1, 0).
  const bool tail = (c.lane & 15) == 15;
  double ra, rc, rd[NR];
  {
    const double an = move0<kDown + 1>(a0), cn = move0<kDown + 1>(c0);
    const double inv = recip(__builtin_fma(-Cl, an, 1.0));
    ra = tail ? 0.0 : A * inv;
    rc = tail ? -1.0 : -Cl * cn * inv;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const double dn = move0<kDown + 1>(d0s[q]);
      rd[q] = tail ? 0.0 : __builtin_fma(-Cl, dn, D[q][M - 1]) * inv;
    }
  }
  reduce_row<NR>(ra, rc, rd);
  // the group's equations: its last unknown L + a XL + c F' = d (XL: the last unknown of the group
  // before, F': the first row of the next group), its first row F + a XL + c L = d
  double* gr = c.grp + (c.gk & 1) * grp_doubles(NR);
  double* gf = gr + (2 + NR) * kGroups;
  c.gk++;
  const int grp = c.t >> 4;
  {
    const double a14 = move0<kUp + 1>(ra), c14 = move0<kUp + 1>(rc);
    double d14[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) d14[q] = move0<kUp + 1>(rd[q]);
    if (tail) {
      const double inv = recip(__builtin_fma(-A, c14, 1.0));
      gr[grp] = -A * a14 * inv;
      gr[kGroups + grp] = Cl * inv;
#pragma unroll
      for (int q = 0; q < NR; ++q)
        gr[(2 + q) * kGroups + grp] = __builtin_fma(-A, d14[q], D[q][M - 1]) * inv;
    }
    if ((c.lane & 15) == 0) {
      gf[grp] = __builtin_fma(-c0, ra, a0);
      gf[kGroups + grp] = -c0 * rc;
#pragma unroll
      for (int q = 0; q < NR; ++q)
        gf[(2 + q) * kGroups + grp] = __builtin_fma(-c0, rd[q], d0s[q]);
    }
  }
  __syncthreads();
  // all groups' last unknowns, one per lane of every wave
  const int G = c.T >> 4, q0 = c.lane;
  double ga = 0.0, gc = 0.0, gd[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) gd[q] = 0.0;
  if (q0 < G) {
    const bool nx = q0 + 1 < G;
    const double af = nx ? gf[q0 + 1] : 0.0, cf = nx ? gf[kGroups + q0 + 1] : 0.0;
    const double cl = gr[kGroups + q0];
    const double inv = recip(__builtin_fma(-cl, af, 1.0));
    ga = gr[q0] * inv;
    gc = -cl * cf * inv;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const double df = nx ? gf[(2 + q) * kGroups + q0 + 1] : 0.0;
      gd[q] = __builtin_fma(-cl, df, gr[(2 + q) * kGroups + q0]) * inv;
    }
  }
  reduce_row<NR>(ga, gc, gd);
  double X[NR];                                  // group q0's last unknown
  if (G <= 16) {
#pragma unroll
    for (int q = 0; q < NR; ++q) X[q] = gd[q];
  } else {
    // the rows of 16 groups in order: F_r = y - z F_{r+1} and L_r = al - be F_{r+1} for their first
    // and last unknowns
    double be = 0.0, y[NR][kGroupRows], z[kGroupRows], al[NR][kGroupRows], bl[kGroupRows];
#pragma unroll
    for (int s = 0; s < kGroupRows; ++s) {
      const double aF = lane_value(ga, 16 * s), cF = lane_value(gc, 16 * s);
      const double aL = lane_value(ga, 16 * s + 15), cL = lane_value(gc, 16 * s + 15);
      const double inv = recip(__builtin_fma(-aF, be, 1.0));
      z[s] = cF * inv;
      bl[s] = __builtin_fma(aL * be, z[s], cL);
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const double ap = s > 0 ? al[q][s - 1] : 0.0;
        y[q][s] = __builtin_fma(-aF, ap, lane_value(gd[q], 16 * s)) * inv;
        al[q][s] = __builtin_fma(aL * be, y[q][s],
                                 __builtin_fma(-aL, ap, lane_value(gd[q], 16 * s + 15)));
      }
      be = bl[s];
    }
    const int row = c.lane >> 4;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      double F = 0.0, before = 0.0, after = 0.0;
#pragma unroll
      for (int s = kGroupRows - 1; s >= 0; --s) {
        const double L = __builtin_fma(-bl[s], F, al[q][s]);
        if (row == s) after = F;
        if (row == s + 1) before = L;
        F = __builtin_fma(-z[s], F, y[q][s]);
      }
      X[q] = __builtin_fma(-ga, before, __builtin_fma(-gc, after, gd[q]));
    }
  }
  // back: the last unknowns of this group and of the one before, of this block and of the one
  // before, then the rows
  const int w4 = __builtin_amdgcn_readfirstlane(c.wave) * 4, row = c.lane >> 4;
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const double l0 = lane_value(X[q], w4), l1 = lane_value(X[q], w4 + 1);
    const double l2 = lane_value(X[q], w4 + 2), l3 = lane_value(X[q], w4 + 3);
    const double lb = w4 > 0 ? lane_value(X[q], w4 - 1) : 0.0;
    const double L = row == 0 ? l0 : (row == 1 ? l1 : (row == 2 ? l2 : l3));
    const double XL = row == 0 ? lb : (row == 1 ? l0 : (row == 2 ? l1 : l2));
    const double xl = __builtin_fma(-ra, XL, __builtin_fma(-rc, L, rd[q]));
    const double xp = move<kUp + 1>(xl, XL);
    double p = A0 * xp;
#pragma unroll
    for (int i = 0; i < M - 1; ++i) {
      D[q][i] -= p;
      p *= E[i + 1];
    }
    D[q][M - 1] = xl;
#pragma unroll
    for (int i = M - 2; i >= 0; --i) D[q][i] = __builtin_fma(E[i], D[q][i + 1], D[q][i]);
  }
  if constexpr (PER) {
    // x = y - z (v.y) / (1 + v.z),  v = (1, 0, .., 0, r/d0)
    double xl[NR], xr[NR], w0[NR], wn[NR];
    exchange<M, NR, true>(c, D, xl, xr, w0, wn);
    const double v1 = r / d0;
    const double f = (w0[0] + v1 * wn[0]) / (1.0 + w0[NR - 1] + v1 * wn[NR - 1]);
#pragma unroll
    for (int i = 0; i < M; ++i) x[i] = D[0][i] - f * D[NR - 1][i];
  } else {
#pragma unroll
    for (int i = 0; i < M; ++i) x[i] = D[0][i];
  }
}

constexpr int kMaxCorrections = 4;

// Neighbours of a register block of values (one right-hand side).
template <int M>
struct Edges {
  double l, r, w0, wn;
};

template <int M, bool PER, typename Max = double>
__device__ __forceinline__ Edges<M> edges(Ctx& c, const double (&x)[M], Max* mx = nullptr) {
  constexpr int NR = PER ? 2 : 1;       // the edge buffers have this layout
  double xx[NR][M];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int i = 0; i < M; ++i) xx[r][i] = x[i];
  double xl[NR], xr[NR], w0[NR], wn[NR];
  exchange<M, NR, PER, Max>(c, xx, xl, xr, w0, wn, mx);
  return Edges<M>{xl[0], xr[0], w0[0], wn[0]};
}

// Rows g0-1 .. g0+M of a register block as its stencils see them (a periodic grid wraps rows 0 and
// n-1: the block's row before row 0 is row n-1; a row after row n-1 is row 0).
template <int M, bool PER>
__device__ __forceinline__ void with_halo(const Ctx& c, const double (&x)[M], const Edges<M>& e,
                                          double (&out)[M + 2]) {
  out[0] = PER && c.g0 == 0 ? e.wn : e.l;
#pragma unroll
  for (int i = 0; i < M; ++i) out[i + 1] = PER && c.g0 + i == c.n ? e.w0 : x[i];
  out[M + 1] = PER && c.g0 + M == c.n ? e.w0 : e.r;
}

// Solve y - tau f^S(y) = rhs for this thread's rows (guess in y on entry) and leave the solution's
// neighbours in e.  Linear f^S: y += solve(FP64 residual of y), until what the last solve lost is
// below eps / 64 of y.  A solve loses some eps cond / 8 of its correction (the diagonal's 1 rounds
// away beside 2 r; cond: the condition number), the same way in every row and step: one solve alone
// left 1e-10 of y at r = 6.7e5 (two: 5e-14) and 4e-16 at r = 25 (two: 1.6e-16).  Correctors,
// whose guess is the level below, take one; predictors two while r times the guess's error shows
// (ARK3 + FBE at n = 8192, r = 34: one solve 59 us a step, this rule 63).
// Otherwise Newton's method with the stopping rule: the largest update is below 1e-15 max(1,
// max|y|), or below 1e-11 max(1, max|y|) and above half the previous one (rounding noise); after
// maxit iterates without stopping, y becomes NaN.  rhs_at(i): the right-hand side of local row i.
template <int M, bool PER, typename Rhs>
__device__ __forceinline__ void stage_solve(Ctx& c, double tau, int maxit, Rhs rhs_at,
                                            double (&y)[M], Edges<M>& e) {
  const double r = tau * c.nu_h2;
  const double b0 = 1.0 + 2.0 * r;
  e = edges<M, PER>(c, y);
  if (PER || c.fs == RIDC_FS_DIFFUSION) {    // a stiff reaction comes on Dirichlet grids only
    const double np = c.n + 1.0;
    const double cond = (1.0 + 4.0 * r) / (PER ? 1.0 : 1.0 + 9.8 * r / (np * np));
    for (int it = 0; it < kMaxCorrections; ++it) {
      double delta[M], yh[M + 2];
      with_halo<M, PER>(c, y, e, yh);
      tri_solve<M, PER>(
          c, r, b0,
          [&](int i, double& b, double& d) __attribute__((always_inline)) {
            d = rhs_at(i) - (y[i] - tau * c.nu_h2 * (yh[i + 2] - 2.0 * y[i] + yh[i]));
            b = b0;
          },
          delta);
      // the largest correction and value, by the high words of their magnitudes (padding rows hold
      // no correction, and zero or row 0's value)
      int mx[2] = {0, 0};
#pragma unroll
      for (int i = 0; i < M; ++i) {
        y[i] += delta[i];
        mx[0] = larger(mx[0], __double2hiint(delta[i]) & 0x7fffffff);
        mx[1] = larger(mx[1], __double2hiint(y[i]) & 0x7fffffff);
      }
      e = edges<M, PER>(c, y, mx);
      const double dmax = __hiloint2double(__builtin_amdgcn_readfirstlane(mx[0]), 0);
      const double ymax = __hiloint2double(__builtin_amdgcn_readfirstlane(mx[1]), 0);
      if (8.0 * cond * dmax <= ymax) break;
    }
    return;
  }
  double last = __builtin_inf();
  bool done = false;
  for (int it = 0; it < maxit && !done; ++it) {
    double delta[M], yh[M + 2];
    with_halo<M, PER>(c, y, e, yh);
    tri_solve<M, PER>(
        c, r, b0,
        [&](int i, double& b, double& d) __attribute__((always_inline)) {
          d = rhs_at(i) - (y[i] - tau * fstiff(c, yh[i], y[i], yh[i + 2]));
          b = b0 - tau * c.kappa * react_prime(c.fs, y[i]);
        },
        delta);
    double mx[2] = {0.0, 0.0};          // largest update, largest value
#pragma unroll
    for (int i = 0; i < M; ++i) {
      y[i] += delta[i];
      const bool real = c.g0 + i < c.n;
      mx[0] = real ? fmax(mx[0], fabs(delta[i])) : mx[0];
      mx[1] = real ? fmax(mx[1], fabs(y[i])) : mx[1];
    }
    e = edges<M, PER>(c, y, mx);
    const double scale = fmax(1.0, mx[1]);
    done = mx[0] <= 1e-15 * scale || (mx[0] <= 1e-11 * scale && mx[0] > 0.5 * last);
    last = mx[0];
  }
  if (!done) {
#pragma unroll
    for (int i = 0; i < M; ++i) y[i] = __builtin_nan("");
    e = edges<M, PER>(c, y);
  }
}

// m mod R (a step's index fits 32 bits in all but the longest runs)
__device__ __forceinline__ int ring_slot(int64_t m, int R) {
  const int s = (uint64_t)m >> 32 == 0 ? (int)((uint32_t)m % (uint32_t)R) : (int)(m % R);
  return __builtin_amdgcn_readfirstlane(s);    // uniform: addresses built from it stay scalar
}

template <int M, bool PER>
__device__ __forceinline__ void imex_step(const ImexLvl& L, int64_t sigma, bool init, double* lds) {
  constexpr int NR = PER ? 2 : 1;
  Ctx c;
  c.n = L.n;
  c.T = blockDim.x;
  c.t = threadIdx.x;
  c.g0 = c.t * M;
  c.fe = L.fe;
  c.fs = L.fs;
  c.ce = L.ce;
  c.nu_h2 = L.nu_h2;
  c.kappa = L.kappa;
  c.lane = c.t & 63;
  c.wave = c.t >> 6;
  c.grp = lds;
  c.ex = lds + 2 * grp_doubles(NR);
  c.rhs = c.ex + 2 * ex_doubles(NR);
  c.gk = c.xk = 0;
  const int64_t V = (int64_t)M * c.T;    // doubles per vector
  if (init) {
    // f of the initial value (slot 0), read by the next level's window at node t_0
    if (!L.ownF) return;
    double u[M + 2];
    load_halo<M, PER>(c, gp(L.own), u);
    double f[M];
    fe_rows<M>(c.fe, c.ce, u, f);
#pragma unroll
    for (int i = 0; i < M; ++i) f[i] += fstiff(c, u[i], u[i + 1], u[i + 2]);
    store_real<M>(c, gp(L.ownF), f);
    return;
  }
  const int64_t m = sigma - L.sigma0 - L.delay;   // this step computes t_m from t_{m-1}
  if (m < 1 || m > L.nt) return;
  const int64_t tn = m - 1;
  const double dt = L.dt;
  const int s = L.s, S = L.S;
  const bool corr = L.prev != nullptr;
  const gdbl* yn_p = gp(L.own) + ring_slot(tn, L.R_own) * V;
  // corrector window: S nodes t_start .. t_{start+S-1}; t_n sits at position rpos
  int64_t start = 0;
  int rpos = 0, slot0 = 0;
  if (corr) {
    start = tn >= S - 2 ? tn + 2 - S : 0;
    rpos = (int)(tn - start);
    slot0 = ring_slot(start, L.R_prev);
  }
  gdbl* const ks = gp(L.ks);
  gdbl* const ss_p = ks + 2 * (s - 1) * V;     // f^S(eta(t_n + c_i dt)) during a solve
  gdbl* const sn_p = ss_p + V;                 // f^N(eta(t_n + c_i dt)) during a solve
  // does a later stage take K^S_i, K^N_i ?
  auto taken = [&](int i, bool* S_i, bool* N_i) {
    *S_i = *N_i = false;
    for (int l = i + 1; l < s; ++l) {
      *S_i = *S_i || L.AS[l][i] != 0.0;
      *N_i = *N_i || L.AN[l][i] != 0.0;
    }
  };
  bool useS, useN;
  {
    // stage 0: explicit, c = 0, so Y_0 = y_n and eta is the node at t_n
    taken(0, &useS, &useN);
    double y[M + 2], v[M + 2], k[M], f[M];
    load_halo<M, PER>(c, yn_p, y);
    if (corr) load_halo<M, PER>(c, gp(L.prev) + ring_slot(tn, L.R_prev) * V, v);
    if (useS) {
#pragma unroll
      for (int x = 0; x < M; ++x) {
        k[x] = fstiff(c, y[x], y[x + 1], y[x + 2]);
        if (corr) k[x] -= fstiff(c, v[x], v[x + 1], v[x + 2]);
      }
      store_rows<M>(c, ks, k);
    }
    if (useN) {
      fe_rows<M>(c.fe, c.ce, y, k);
      if (corr) {
        fe_rows<M>(c.fe, c.ce, v, f);
#pragma unroll
        for (int x = 0; x < M; ++x) k[x] -= f[x];
      }
      store_rows<M>(c, ks + V, k);
    }
  }
  double Y[M], rhs[M];
  Edges<M> edge;     // neighbours of this thread's block of Y_i
  for (int i = 1; i < s; ++i) {
    const double tau = dt * L.AS[i][i];
    // rhs = y_n + I_i - tau f^S(eta) + dt sum_{l<i} (AS K^S_l + AN K^N_l)
    load_rows<M>(c, yn_p, rhs);
    if (corr) {
      const gdbl* w = gp(L.wt) + ((int64_t)rpos * s + i) * 2 * S;
      {
        // eta; nodes of weight zero are not read (a stage at a node takes that node alone)
        double e[M + 2], f[M];
#pragma unroll
        for (int k = 0; k < M + 2; ++k) e[k] = 0.0;
        int at = slot0;
        for (int k = 0; k < S; ++k) {
          const double lk = w[k];
          if (lk != 0.0) {
            double v[M + 2];
            load_halo<M, PER>(c, gp(L.prev) + at * V, v);
#pragma unroll
            for (int x = 0; x < M + 2; ++x) e[x] += lk * v[x];
          }
          at = at + 1 == L.R_prev ? 0 : at + 1;
        }
        if (i < s - 1) {
          fe_rows<M>(c.fe, c.ce, e, f);
          store_rows<M>(c, sn_p, f);
        }
#pragma unroll
        for (int x = 0; x < M; ++x) {
          f[x] = fstiff(c, e[x], e[x + 1], e[x + 2]);
          rhs[x] -= tau * f[x];
          Y[x] = e[x + 1];
        }
        if (i < s - 1) store_rows<M>(c, ss_p, f);
      }
      double q[M];
#pragma unroll
      for (int k = 0; k < M; ++k) q[k] = 0.0;
      int at = slot0;
      for (int k = 0; k < S; ++k) {
        const double qk = w[S + k];
        double fv[M];
        load_rows<M>(c, gp(L.prevF) + at * V, fv);
#pragma unroll
        for (int x = 0; x < M; ++x) q[x] += qk * fv[x];
        at = at + 1 == L.R_prev ? 0 : at + 1;
      }
#pragma unroll
      for (int x = 0; x < M; ++x) rhs[x] = rhs[x] + dt * q[x];
    } else if (i > 1 && (PER || c.fs == RIDC_FS_DIFFUSION)) {
      // the guess follows the line through y_n and the stage before: of the third-order pair's four
      // solves only the first is off by O(dt), which saves most of the second solves (68 -> 65 us a
      // step, n = 8192).  A stiff reaction's stages start from y_n, on the branch the value is on
      const double f = L.c[i] / L.c[i - 1];
#pragma unroll
      for (int x = 0; x < M; ++x) Y[x] = __builtin_fma(f, Y[x] - rhs[x], rhs[x]);
    } else {
#pragma unroll
      for (int x = 0; x < M; ++x) Y[x] = rhs[x];
    }
    // the two terms of a stage are added up before the value, whose size sets the rounding: once a
    // stage and not twice
    for (int l = 0; l < i; ++l) {
      const double as = dt * L.AS[i][l], an = dt * L.AN[i][l];
      if (as == 0.0 && an == 0.0) continue;
      double k[M];
#pragma unroll
      for (int x = 0; x < M; ++x) k[x] = 0.0;
      if (as != 0.0) {
        load_rows<M>(c, ks + 2 * l * V, k);
#pragma unroll
        for (int x = 0; x < M; ++x) k[x] *= as;
      }
      if (an != 0.0) {
        double kn[M];
        load_rows<M>(c, ks + (2 * l + 1) * V, kn);
#pragma unroll
        for (int x = 0; x < M; ++x) k[x] += an * kn[x];
      }
#pragma unroll
      for (int x = 0; x < M; ++x) rhs[x] += k[x];
    }
    // the largest blocks keep the right-hand side in LDS during the solve
    constexpr bool kMem = M >= 16;
    if constexpr (kMem) {
#pragma unroll
      for (int x = 0; x < M; ++x) c.rhs[x * c.T + c.t] = rhs[x];
      stage_solve<M, PER>(c, tau, L.maxit, [&](int x) __attribute__((always_inline)) { return c.rhs[x * c.T + c.t]; }, Y, edge);
    } else {
      stage_solve<M, PER>(c, tau, L.maxit, [&](int x) __attribute__((always_inline)) { return rhs[x]; }, Y, edge);
    }
    if (i < s - 1) {
      // K^S_i = (Y_i - rhs) / tau - f^S(eta), K^N_i = f^N(Y_i) - f^N(eta), where taken
      taken(i, &useS, &useN);
      if (useS) {
        double k[M];
#pragma unroll
        for (int x = 0; x < M; ++x)
          k[x] = (Y[x] - (kMem ? c.rhs[x * c.T + c.t] : rhs[x])) / tau;
        if (corr) {
          double v[M];
          load_rows<M>(c, ss_p, v);
#pragma unroll
          for (int x = 0; x < M; ++x) k[x] -= v[x];
        }
        store_rows<M>(c, ks + 2 * i * V, k);
      }
      if (useN) {
        double k[M], yh[M + 2];
        with_halo<M, PER>(c, Y, edge, yh);
        fe_rows<M>(c.fe, c.ce, yh, k);
        if (corr) {
          double v[M];
          load_rows<M>(c, sn_p, v);
#pragma unroll
          for (int x = 0; x < M; ++x) k[x] -= v[x];
        }
        store_rows<M>(c, ks + (2 * i + 1) * V, k);
      }
    }
  }
  const int64_t slot = ring_slot(m, L.R_own) * V;
  store_real<M>(c, gp(L.own) + slot, Y);
  if (L.ownF) {
    double f[M], yh[M + 2];
    with_halo<M, PER>(c, Y, edge, yh);
    fe_rows<M>(c.fe, c.ce, yh, f);
#pragma unroll
    for (int x = 0; x < M; ++x) f[x] += fstiff(c, yh[x], yh[x + 1], yh[x + 2]);
    store_real<M>(c, gp(L.ownF) + slot, f);
  }
}

template <int M, bool PER>
__global__ __launch_bounds__(kImexMaxThreads) void k_imex1d(const ImexLvl* __restrict__ items,
                                                            int64_t sigma, int init) {
  extern __shared__ double lds[];
  imex_step<M, PER>(items[blockIdx.x], sigma, init != 0, lds);
}

// Slot 0 of every level's ring from the initial data (block order, zero padding).
__global__ void k_imex_load(const double* __restrict__ u0, ImexRings rings, int n, int M, int T) {
  double* __restrict__ dst = rings.ring[blockIdx.y];
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < M * T; e += gridDim.x * blockDim.x) {
    const int g = (e % T) * M + e / T;
    dst[e] = g < n ? u0[g] : 0.0;
  }
}

// A vector in block order to grid order; *flag set to 1 when a value is not finite.
__global__ void k_imex_read(const double* __restrict__ src, double* __restrict__ dst, int n, int M,
                            int T, int* flag) {
  int bad = 0;
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < n; g += gridDim.x * blockDim.x) {
    const double v = src[(g % M) * T + g / M];
    dst[g] = v;
    if (!(v - v == 0.0)) bad = 1;      // NaN or Inf
  }
  if (flag && __any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

template <int M, bool PER>
hipError_t launch_t(const ImexLvl* items, int count, int threads, int64_t sigma, bool init,
                    hipStream_t stream) {
  const size_t lds = sizeof(double) * lds_doubles(PER ? 2 : 1, M, threads);
  static size_t allowed = 65536;
  if (lds > allowed) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_imex1d<M, PER>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    allowed = lds;
  }
  hipLaunchKernelGGL((k_imex1d<M, PER>), dim3(count), dim3(threads), lds, stream, items, sigma,
                     init ? 1 : 0);
  return hipGetLastError();
}

template <bool PER>
hipError_t launch_m(int M, const ImexLvl* items, int count, int threads, int64_t sigma,
                    bool init, hipStream_t stream) {
  switch (M) {
    case 2: return launch_t<2, PER>(items, count, threads, sigma, init, stream);
    case 4: return launch_t<4, PER>(items, count, threads, sigma, init, stream);
    case 8: return launch_t<8, PER>(items, count, threads, sigma, init, stream);
    case 16: return launch_t<16, PER>(items, count, threads, sigma, init, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

void imex_shape(int64_t n, int* M, int* threads) {
  // The fewest rows per thread that keep the workgroup within one wave per SIMD (256 threads), 8
  // rows at most up to n = 4096.  Steps of RIDC4 with the cubic reaction, us, at 2 / 4 / 8 / 16 rows:
  // n = 500 21.5 / 23.0 / 27.2 / 42.8, 999 32.0 / 24.0 / 28.7 / 42.9, 2000 - / 36.5 / 29.9 / 44.9, 4000
  // - / - / 46.0 / 47.9 (two waves on a SIMD take turns; a longer block is a longer chain).
  int m = 2;
  while (m < 8 && (n + m - 1) / m > 256) m *= 2;
  while (m < kImexMaxRows && (n + m - 1) / m > kImexMaxThreads) m *= 2;
  const int64_t t = (n + m - 1) / m;
  *M = m;
  *threads = (int)((t + 63) / 64 * 64);
}

hipError_t launch_imex_load(const double* u0, const ImexRings& rings, int P, int n, int M, int T,
                            hipStream_t stream) {
  hipLaunchKernelGGL(k_imex_load, dim3((M * T + 255) / 256, P), dim3(256), 0, stream, u0, rings, n,
                     M, T);
  return hipGetLastError();
}

hipError_t launch_imex_read(const double* src, double* dst, int n, int M, int T, int* flag,
                            hipStream_t stream) {
  hipLaunchKernelGGL(k_imex_read, dim3((n + 255) / 256), dim3(256), 0, stream, src, dst, n, M, T,
                     flag);
  return hipGetLastError();
}

hipError_t launch_imex1d(const ImexLvl* d_items, int count, int M, int threads, bool periodic,
                         int64_t sigma, bool init, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  if (threads < 64 || threads > kImexMaxThreads || threads % 64) return hipErrorInvalidValue;
  return periodic ? launch_m<true>(M, d_items, count, threads, sigma, init, stream)
                  : launch_m<false>(M, d_items, count, threads, sigma, init, stream);
}

}  // namespace ridc
