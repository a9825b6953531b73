// 2D (n x n, zero Dirichlet) part of the RIDC pipeline for gfx950.
//
// Every level step is taken in increment form, which is algebraically the step of the paper:
//   predictor (section II, eq. imex_diffusion):
//     (I - dt L) d = dt (f_E + L)(eta[0]_n),               eta[0]_{n+1} = eta[0]_n + d
//   corrector (section III-C, eq. corr, with the (j+1)-node quadrature Q of f along level j-1):
//     (I - dt L) e = eta[j]_n - eta[j-1]_{n+1} + dt Q + dt [f_E(eta[j]_n) - f_E(eta[j-1]_n)],
//     eta[j]_{n+1} = eta[j-1]_{n+1} + e
// (subtract (I - dt L) eta[j-1]_{n+1}, resp. (I - dt L) eta[0]_n, from both sides of the
// paper's equation).  The right-hand side is small (O(dt) resp. O(dt^j)), so the rounding of
// the transforms scales with the increment, not with u; the sums and level differences are
// FP64 in every precision.
//
// Solve: diagonalisation along the rows only.  With the orthonormal type-I sine matrix Q
// (symmetric, Q_{ik} = sqrt(2/(n+1)) sin(pi (i+1)(k+1)/(n+1))) and mu_k = (4/h^2) sin^2(pi (k+1) /
// (2(n+1))), T = B Q turns (I - dt nu Lap_h) X = B into one constant tridiagonal system down each
// column j of T, (1 + dt nu mu_j) x - dt nu D2 x = T_j, and X is the solutions times Q.
// Diagonalising the columns as well would take two more products by Q, the cost of a pass each
// (75 us at 1024^2 over four levels in FP64); the line solves read and write each vector once
// (k_lines2d, 14 us there; the step went from 305 to 180 us).
// Each product by Q is one pass C = A Q, a GEMM on the matrix cores (v_mfma_f64_16x16x4f64,
// v_mfma_f32_16x16x4_f32, or three v_mfma_f32_16x16x32_bf16 products of hi/lo BF16 splits),
// batched over every active level of every instance in one launch; the final update is fused
// into the epilogue of the second pass.  Sides that are multiples of 64 fold Q by its reflection
// symmetry, Q_{n-1-k, j} = (-1)^j Q_{k, j}, which halves the contraction (k_pass2d): a pass folds
// its operand while staging it; the operand of a folded split-BF16 pass arrives folded and split
// (store_split).
//
// Reduced precision (FP32 or split BF16) adds one FP64 residual refinement:
//   x1 = S~(b),  rho = b - (x1 - dt nu Lap_h x1)  (FP64 5-point),  x = x1 + S~(rho);
// x1 is held in FP32: the pass that produces it accumulates in FP32, so x1 is an FP32 value and
// storing it in FP32 loses nothing.  The line solves compute in FP64 and store FP32.
#include <hip/hip_bf16.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>

#include "ridc2d.h"
#include "ridc_internal.h"

namespace ridc {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16;

enum { PREC_F64 = 0, PREC_F32 = 1, PREC_BF16 = 2 };
enum { OUT_F64 = 0, OUT_F32 = 1, OUT_FINAL = 3 };

// One (instance, level) of the 2D pipeline: static for a handle.
struct Lvl2D {
  double* own;          // ring of this level (R_own slots of n*n)
  const double* prev;   // ring of level j-1 (null for j = 0)
  const double* W;      // weights, j rows x (j+1)
  double* b64;          // FP64 right-hand side (kept for the residual)
  double* x64;          // FP64 sine coefficients, or (refined paths) the FP32 first solve
  float* lo0;           // reduced precision: the right-hand side or residual the solve takes
  float* lo1;           // reduced precision: its sine coefficients
                        // (split-BF16 folded systems: both as split operands, store_split, lo1
                        // between its pass and the line solves in paired column order)
  const double* col;    // line-solve constants of every column: lambda, g, kappa (n each)
  int64_t nt, sigma0;
  int32_t n, j, R_own, R_prev, fe, prec;
  double dt, nu_h2;
};

// One batch entry of a transform pass: entry e of a pass belongs to entry e of the level table (so
// that a block reads both at once).
struct Pass2D {
  const void* A;        // input: row-major n x n (FP64, or FP32 in the reduced-precision paths)
  void* C;              // output (unless final)
  const float* add;     // final epilogue: extra term (x1 of the refinement, FP32), nullable
  const void* Q;        // transform matrix in the input precision (BF16: hi, lo at +n*n)
  int64_t paired;       // C takes its columns in paired order (paired_col)
};

struct Plan2D {
  ridc_problem p{};
  int P = 1, prec = 0;
  int64_t n = 0;
  double h = 0;
  std::vector<Lvl2D> levels;        // host copy (nt filled at arm)
  Lvl2D* d_levels = nullptr;
  // pass tables: npass passes x P entries, device
  int npass = 0;
  std::vector<Pass2D> passes;
  Pass2D* d_passes = nullptr;
  // transform data (shared per n)
  const double* Q64 = nullptr;
  const float* Q32 = nullptr;
  const u16* Qbf = nullptr;         // hi then lo
  double* col = nullptr;            // line-solve constants (Lvl2D::col)
  hipStream_t stream = nullptr;
  int tile = 0;                     // pass launch shape: kPassWide64 | kPassNarrowK (results
                                    // are bitwise the same for every shape)
};

// ---------------------------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ bool level_active(const Lvl2D& L, int64_t sigma, int64_t* m_out) {
  const int64_t m = sigma - L.sigma0 - (int64_t)L.j * (L.j + 1) / 2;
  *m_out = m;
  return m >= 1 && m <= L.nt;
}

// m mod R.  A step's index fits 32 bits in all but the longest runs, and a 64-bit remainder is some
// hundred dependent instructions at the head of every kernel.
__device__ __forceinline__ int ring_slot(int64_t m, int R) {
  if ((uint64_t)m >> 32 == 0) return (int)((uint32_t)m % (uint32_t)R);
  return (int)(m % R);
}

__device__ __forceinline__ double fe2(int fe, double u) {
  return fe == RIDC_FE_LOGISTIC ? u * (1.0 - u) : 0.0;
}

// Loads and stores through pointers read from the launch tables.  The compiler cannot tell
// their address space and would emit flat instructions, which also count against the LDS wait
// counter (every LDS wait would then wait for the outstanding global loads too); these name the
// global space.
template <typename V>
__device__ __forceinline__ V gld(const void* p) {
  return *(const __attribute__((address_space(1))) V*)p;
}
template <typename V>
__device__ __forceinline__ void gst(void* p, V v) {
  *(__attribute__((address_space(1))) V*)p = v;
}

// The FP32 copy of a right-hand side or residual that the first pass of an FP32 solve (or of a
// split-BF16 one that does not fold) reads: row-major; that pass folds or splits it while staging.
__device__ __forceinline__ void store_lo(float* base, int64_t idx, double v) {
  gst<float>(base + idx, (float)v);
}

// FP32 -> BF16 hi (round to nearest) in the low half, BF16 lo (of the remainder) in the high half
__device__ __forceinline__ unsigned split_bf16(float v) {
  const __bf16 b = (__bf16)v;
  return (unsigned)__builtin_bit_cast(unsigned short, b) |
         ((unsigned)__builtin_bit_cast(unsigned short, (__bf16)(v - (float)b)) << 16);
}

// The operand of a folded split-BF16 pass, 4 n bytes a row like the FP32 values it stands for: for
// every 8 k < n/2 the BF16 hi and lo of the sums a_k + a_{n-1-k}, then of the differences a_k -
// a_{n-1-k}, 16 bytes each.  Folding and splitting where the values are made costs each of them once;
// in the pass every column tile did it again.  At 1024^2, four levels: a pass 24.3 -> 22.4 us (20.6 with
// the LDS rows of ROW_PAD and a second slice on its way), the right-hand side 24.3 -> 26.2, the line
// solves 9.5 -> 11.3; a whole step 153.7 -> 144.
// A lane holds x = a_k and y = a_{n-1-k} (low) or the two exchanged and writes two k of one plane:
// lanes l and l ^ 1 hold neighbouring k and exchange halves.
__device__ __forceinline__ void store_split(void* row, int k, bool low, float x, float y) {
  const unsigned own = split_bf16(low ? x + y : y - x);
  const unsigned oth = (unsigned)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xF, 0xF, false);
  const unsigned a = k & 1 ? oth : own, b = k & 1 ? own : oth;      // of the even k, of the odd one
  const bool hi = (threadIdx.x & 1) == 0;
  const unsigned w = hi ? (a & 0xffffu) | (b << 16) : (a >> 16) | (b & 0xffff0000u);
  gst<unsigned>((char*)row + (k >> 3) * 64 + (low ? 0 : 32) + (hi ? 0 : 16) + (k & 6) * 2, w);
}

// Paired column order: position p of a row holds, sixteen at a time, 8 columns and the 8 that
// mirror them, so that a block of the line solves owns both halves of the sums and differences it
// writes (n a multiple of 64).
__device__ __forceinline__ int paired_col(int p, int n) {
  const int g = p >> 4, o = p & 15;
  return o < 8 ? 8 * g + o : n - 16 - 8 * g + o;
}

// ---------------------------------------------------------------------------------------------
// stencil kernels: a wave owns 64 columns of RY consecutive rows and walks down them, keeping
// the rows above and below in registers, so each stencil vector is read once per point.  Column
// neighbours come from the adjacent lanes (DPP wave shifts); the columns just outside the wave's
// 64, which lanes 0 and 63 take, come from one load per half-wave at one address.  Columns at or
// beyond n hold zero, which is also the Dirichlet ghost value, so a wave that straddles the last
// column needs no special case.  SPLIT (operands for a folded split-BF16 pass): the wave owns 32
// columns and the 32 that mirror them, lane l and lane 63 - l mirrored, and has four outside columns,
// a quarter-wave each.
// ---------------------------------------------------------------------------------------------
constexpr int ST_WAVES = 4;  // waves per block, stacked in rows

__device__ __forceinline__ double lane_below(double v) {   // lane l gets lane l-1's v (lane 0: 0)
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_above(double v) {   // lane l gets lane l+1's v (lane 63: 0)
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_below(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_above(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, false));
}

// The block a workgroup runs: column strip bx, block row by, level bz.  Workgroups go to the 8
// XCDs round-robin by linear id.  When the block rows of all levels (grid y times z) are a
// multiple of 8, block row R = 8k + x runs whole on XCD x, so the strips beside a block, whose
// edge columns it reads, sit in the same L2; the levels still spread over every XCD.
struct StBlock {
  unsigned x, y, z;
};
__device__ __forceinline__ StBlock stencil_block() {
  const unsigned gx = gridDim.x, rows = gridDim.y * gridDim.z;
  if (rows % 8 != 0) return StBlock{blockIdx.x, blockIdx.y, blockIdx.z};
  const unsigned id = blockIdx.x + gx * (blockIdx.y + gridDim.y * blockIdx.z);
  const unsigned r = id / 8;
  const unsigned row = (r / gx) * 8 + id % 8;
  return StBlock{r % gx, row % gridDim.y, row / gridDim.y};
}

// Where a block's wave sits: the first row and column it owns, or false when it owns none.
template <int RY>
__device__ __forceinline__ bool stencil_tile(int n, const StBlock& b, int* iy0, int* ix0) {
  *ix0 = (int)b.x * 64;
  *iy0 = ((int)b.y * ST_WAVES + (int)(threadIdx.x >> 6)) * RY;
  return *ix0 < n && *iy0 < n;
}

// The column of this lane in the strip at ix0, and the column just outside that lanes 0 (west) and 63
// (east), or with SPLIT also 32 (west) and 31 (east), take from `outside`.
template <bool SPLIT>
__device__ __forceinline__ int strip_col(int lane, int ix0, int n) {
  return SPLIT && lane >= 32 ? n - ix0 / 2 - 64 + lane : (SPLIT ? ix0 / 2 : ix0) + lane;
}
template <bool SPLIT>
__device__ __forceinline__ int strip_outside(int lane, int ix0, int n) {
  if constexpr (SPLIT) {
    const int k0 = ix0 / 2;
    return lane < 32 ? (lane < 16 ? k0 - 1 : k0 + 32) : (lane < 48 ? n - k0 - 33 : n - k0);
  } else {
    return lane < 32 ? ix0 - 1 : ix0 + 64;
  }
}
template <bool SPLIT>
__device__ __forceinline__ bool strip_west(int lane) {
  return lane == 0 || (SPLIT && lane == 32);
}
template <bool SPLIT>
__device__ __forceinline__ bool strip_east(int lane) {
  return lane == 63 || (SPLIT && lane == 31);
}

// ---------------------------------------------------------------------------------------------
// right-hand side (increment form), FP64; also writes the low-precision copy.  The quadrature
// of f along level j-1 is taken as sum_i w_i f_E(v_i) + nu Lap_h (sum_i w_i v_i): the stencil
// is linear, so one stencil of the weighted window replaces j+1 stencils.
// ---------------------------------------------------------------------------------------------
// The values of one grid row that the right-hand side needs at a column.
struct RhsRow {
  double V;     // sum_i w_i v_i (level 0: the own value u)
  double fq;    // sum_i w_i f_E(v_i) (level 0: f_E(u))
  double fen;   // f_E(v at node n)
  double vn1;   // v at node n+1
  double u;     // own value at node n
};

// JT = the number of window vectors j + 1 when it is fixed at compile time (0 for the
// predictor), or -1: any j, up to the largest order.  This kernel uses no LDS, and its plain
// (flat) loads measured faster than global ones (31.2 against 33.2 us per launch at 1024^2,
// FP64).
template <int JT, int RY, bool SPLIT>
__device__ __forceinline__ void rhs_level(const Lvl2D& L, int64_t m, int iy0, int ix0) {
  constexpr int JN = JT < 0 ? RIDC_MAX_ORDER : (JT == 0 ? 1 : JT);
  const int n = L.n;
  const int ix = strip_col<SPLIT>(threadIdx.x & 63, ix0, n);
  const bool col = SPLIT || ix < n;
  const int64_t nn = (int64_t)n * n;
  const int64_t nidx = m - 1;
  const double* __restrict__ u = L.own + ring_slot(nidx, L.R_own) * nn;
  const int nv = JT < 0 ? L.j + 1 : JT;        // window vectors
  const double* __restrict__ vp[JN];
  double w[JN];
  int rn = 0;                                  // window index of node n (node n+1 is rn + 1)
  if (JT == 0) {
    vp[0] = u;
    w[0] = 1.0;
  } else {
    const int64_t s = m - L.j > 0 ? m - L.j : 0;
    rn = (int)(nidx - s);
    int slot = ring_slot(s, L.R_prev);
#pragma unroll
    for (int i = 0; i < JN; ++i) {
      if (i < nv) {
        vp[i] = L.prev + slot * nn;
        slot = slot + 1 == L.R_prev ? 0 : slot + 1;
        w[i] = gld<double>(L.W + (nidx - s) * (L.j + 1) + i);
      }
    }
  }
  auto window_sum = [&](int64_t c) {           // sum_i w_i v_i at one point
    if (JT == 0) return u[c];
    double V = 0.0;
#pragma unroll
    for (int i = 0; i < JN; ++i)
      if (i < nv) V += w[i] * vp[i][c];
    return V;
  };
  // The walk down the strip goes RG rows at a time, each group unrolled and without a branch,
  // so that the loads of a group's rows are issued together: lanes past n and rows outside the
  // grid load a clamped in-range address and take zero instead, lanes 0 and 63 take their edge
  // column by a select, and the stores follow each group.  Every wave has RY rows (n is a
  // multiple of 32).  Measured at 1024^2, FP64: 29.1 us per launch with a branch per row and
  // edge, 22.6 us with RG = 2 (114 registers), 22.8 with 1, 26.5 with 4 (148), 27.7 with 8
  // (228), 38.5 with the whole strip unrolled (388 registers, one wave per SIMD).
  const int ixc = col ? ix : n - 1;
  auto load = [&](int iy) {
    const bool in = iy >= 0 && iy < n && col;
    const int64_t c = (int64_t)(iy < 0 ? 0 : (iy < n ? iy : n - 1)) * n + ixc;
    RhsRow r{0.0, 0.0, 0.0, 0.0, 0.0};
    if (JT == 0) {
      r.u = u[c];
      r.V = r.u;
      r.fq = fe2(L.fe, r.u);
    } else {
      r.u = u[c];
#pragma unroll
      for (int i = 0; i < JN; ++i) {
        if (i < nv) {
          const double v = vp[i][c];
          const double f = fe2(L.fe, v);
          r.V += w[i] * v;
          r.fq += w[i] * f;
          if (i == rn) r.fen = f;
          if (i == rn + 1) r.vn1 = v;
        }
      }
    }
    const RhsRow z{0.0, 0.0, 0.0, 0.0, 0.0};
    return in ? r : z;
  };
  // the column just outside the strip that lane 0 (west) or lane 63 (east) takes: every lane
  // of a half reads that one address (zero outside the grid, the Dirichlet ghost value)
  const int lane = threadIdx.x & 63;
  const int xo = strip_outside<SPLIT>(lane, ix0, n);
  const bool xok = xo >= 0 && xo < n;
  const int xoc = xok ? xo : ixc;
  const double dt = L.dt;
  double up = load(iy0 - 1).V;
  RhsRow mid = load(iy0);
  constexpr int RG = RY == 4 ? 4 : 2;      // short strips: every row at once
#pragma unroll
  for (int q = 0; q < RY; q += RG) {
    double bs[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) {
      const int iy = iy0 + q + r;
      const RhsRow dn = load(iy + 1);
      const double ev = window_sum((int64_t)iy * n + xoc);
      double vw = lane_below(mid.V), ve = lane_above(mid.V);
      vw = strip_west<SPLIT>(lane) ? (xok ? ev : 0.0) : vw;
      ve = strip_east<SPLIT>(lane) ? (xok ? ev : 0.0) : ve;
      const double lap = ((vw + ve) + (up + dn.V)) - 4.0 * mid.V;
      const double quad = mid.fq + L.nu_h2 * lap;
      bs[r] = JT == 0 ? dt * quad
                      : (mid.u - mid.vn1) + dt * quad + dt * (fe2(L.fe, mid.u) - mid.fen);
      up = mid.V;
      mid = dn;
    }
    if (col) {
#pragma unroll
      for (int r = 0; r < RG; ++r) {
        const int64_t c = (int64_t)(iy0 + q + r) * n + ix;
        L.b64[c] = bs[r];
        if constexpr (SPLIT) {
          const float x = (float)bs[r];
          store_split(L.lo0 + (int64_t)(iy0 + q + r) * n, lane < 32 ? ix : n - 1 - ix, lane < 32, x,
                      __shfl_xor(x, 63));
        } else if (L.prec != PREC_F64) {
          store_lo(L.lo0, c, bs[r]);
        }
      }
    }
  }
}

template <int RY, bool SPLIT>
__global__ __launch_bounds__(256) void k_rhs2d(const Lvl2D* __restrict__ levels, int64_t sigma) {
  const StBlock blk = stencil_block();
  const Lvl2D& L = levels[blk.z];
  int64_t m;
  if (!level_active(L, sigma, &m)) return;
  int iy0, ix0;
  if (!stencil_tile<RY>(L.n, blk, &iy0, &ix0)) return;
  switch (L.j) {
    case 0: rhs_level<0, RY, SPLIT>(L, m, iy0, ix0); break;
    case 1: rhs_level<2, RY, SPLIT>(L, m, iy0, ix0); break;
    case 2: rhs_level<3, RY, SPLIT>(L, m, iy0, ix0); break;
    case 3: rhs_level<4, RY, SPLIT>(L, m, iy0, ix0); break;
    default: rhs_level<-1, RY, SPLIT>(L, m, iy0, ix0); break;
  }
}

// rho = b - (x1 - dt nu Lap_h x1), FP64, written in low precision.  The first solve x1 is held in
// FP32 (in the x64 buffer; it leaves an FP32 accumulator, so nothing is lost).  Every row of the
// wave's column strip is loaded before any is used, so all of a wave's loads are in flight at
// once.
template <int RY, bool SPLIT>
__global__ __launch_bounds__(256) void k_resid2d(const Lvl2D* __restrict__ levels, int64_t sigma) {
  const StBlock blk = stencil_block();
  const Lvl2D& L = levels[blk.z];
  int64_t m;
  if (!level_active(L, sigma, &m)) return;
  const int n = L.n;
  int iy0, ix0;
  if (!stencil_tile<RY>(n, blk, &iy0, &ix0)) return;
  const int lane = threadIdx.x & 63;
  const int ix = strip_col<SPLIT>(lane, ix0, n);
  const bool col = SPLIT || ix < n;
  const float* __restrict__ x1 = (const float*)L.x64;
  // No load sits behind a branch, so that all of them issue back to back: lanes past n and the
  // rows beyond the grid read a clamped in-range address and take zero instead, and the column
  // just outside the strip, which lane 0 (west) or 63 (east) takes, is read by every lane of
  // its half at that one address.  Every wave has RY rows (n is a multiple of 32).
  const int ixc = col ? ix : n - 1;
  const int xo = strip_outside<SPLIT>(lane, ix0, n);
  const bool xok = xo >= 0 && xo < n;
  const int xoc = xok ? xo : ixc;
  float xr[RY + 2], xe[RY];
  double br[RY];
#pragma unroll
  for (int r = 0; r < RY + 2; ++r) {
    const int iy = iy0 - 1 + r;
    const int iyc = iy < 0 ? 0 : (iy < n ? iy : n - 1);
    const float v = gld<float>(x1 + (int64_t)iyc * n + ixc);
    xr[r] = iy >= 0 && iy < n && col ? v : 0.0f;
  }
#pragma unroll
  for (int r = 0; r < RY; ++r) {
    const int64_t row = (int64_t)(iy0 + r) * n;
    const double b = gld<double>(L.b64 + row + ixc);
    const float e = gld<float>(x1 + row + xoc);
    br[r] = col ? b : 0.0;
    xe[r] = xok ? e : 0.0f;
  }
  double res[RY];
#pragma unroll
  for (int r = 0; r < RY; ++r) {
    double xw = (double)lane_below(xr[r + 1]), xa = (double)lane_above(xr[r + 1]);
    xw = strip_west<SPLIT>(lane) ? (double)xe[r] : xw;
    xa = strip_east<SPLIT>(lane) ? (double)xe[r] : xa;
    const double x = (double)xr[r + 1];
    const double lap = ((xw + xa) + ((double)xr[r] + (double)xr[r + 2])) - 4.0 * x;
    res[r] = br[r] - (x - L.dt * L.nu_h2 * lap);
  }
  if (col) {
#pragma unroll
    for (int r = 0; r < RY; ++r) {
      if constexpr (SPLIT) {
        const float v = (float)res[r];
        store_split(L.lo0 + (int64_t)(iy0 + r) * n, lane < 32 ? ix : n - 1 - ix, lane < 32, v,
                    __shfl_xor(v, 63));
      } else {
        store_lo(L.lo0, (int64_t)(iy0 + r) * n + ix, res[r]);
      }
    }
  }
}

// One launch of a stencil kernel over `cnt` levels of sides up to nmax.  Rows per wave: 16 when
// that gives every SIMD two waves or more, else 4, so that a small grid's loads spread over more
// compute units and a wave's walk down its rows is a quarter as long (the bits are the same).
template <int RY>
static dim3 stencil_grid(int cnt, int64_t nmax) {
  return dim3((unsigned)((nmax + 63) / 64), (unsigned)((nmax + RY * ST_WAVES - 1) / (RY * ST_WAVES)),
              cnt);
}
static bool short_strips(int cnt, int64_t nmax) {
  return (nmax + 63) / 64 * (nmax / 16) * cnt < 2048;
}
// split: the systems' passes take split operands (split_operands)
static void launch_rhs(const Lvl2D* lv, int cnt, int64_t nmax, int64_t sigma, bool split,
                       hipStream_t st) {
  auto go = [&](auto kern, dim3 grid) {
    hipLaunchKernelGGL(kern, grid, dim3(64 * ST_WAVES), 0, st, lv, sigma);
  };
  if (short_strips(cnt, nmax))
    split ? go(k_rhs2d<4, true>, stencil_grid<4>(cnt, nmax))
          : go(k_rhs2d<4, false>, stencil_grid<4>(cnt, nmax));
  else
    split ? go(k_rhs2d<16, true>, stencil_grid<16>(cnt, nmax))
          : go(k_rhs2d<16, false>, stencil_grid<16>(cnt, nmax));
}
static void launch_resid(const Lvl2D* lv, int cnt, int64_t nmax, int64_t sigma, bool split,
                         hipStream_t st) {
  auto go = [&](auto kern, dim3 grid) {
    hipLaunchKernelGGL(kern, grid, dim3(64 * ST_WAVES), 0, st, lv, sigma);
  };
  if (short_strips(cnt, nmax))
    split ? go(k_resid2d<4, true>, stencil_grid<4>(cnt, nmax))
          : go(k_resid2d<4, false>, stencil_grid<4>(cnt, nmax));
  else
    split ? go(k_resid2d<16, true>, stencil_grid<16>(cnt, nmax))
          : go(k_resid2d<16, false>, stencil_grid<16>(cnt, nmax));
}

// ---------------------------------------------------------------------------------------------
// line solves: (1 + lam_j + 2r) x_y - r (x_{y-1} + x_{y+1}) = T_y down every column j
//
// The matrix is constant along a column, so up to its first row it is (1/g)(1 - lambda E^-1)
// (1 - lambda E) (E: the shift by a row; lambda = 2r / (b + sqrt(b^2 - 4r^2)) < 1, b = 1 + lam_j +
// 2r, g = lambda / r): a first-order recurrence down the column, one back up, and a factor.  The
// upward recurrence starts from zero past the last row, the zero ghost there; the downward one
// starts from c_0 = -kappa z_0, kappa = lambda (1 - lambda^2) / (1 - lambda^{2n+2}), which makes the
// value at the other ghost row zero (z_0: what the two recurrences leave in the first row when
// c_0 = 0).  Every term of a recurrence has lambda's sign, so nothing cancels.
//
// A thread holds M consecutive rows of one column (a segment) in registers and runs both
// recurrences over them from zero; two numbers per segment (its last value going down and its
// first value coming back up) go through LDS, a wave chains them over a column's
// segments (line_chain), and the recurrences run again from the true carries.  A block is 16 columns (128
// bytes of a row, a cache line in FP64) of the whole height: 64 segments of M = 16 rows at
// n = 1024, one block per compute unit for four levels.  Bound: HBM, one read and one write of
// each vector; the arithmetic is FP64 also where the coefficients are stored in FP32.
// ---------------------------------------------------------------------------------------------
constexpr int LS_COLS = 16;   // columns per block
constexpr int LS_SEGS = 64;   // segments in registers at a time
constexpr int LS_STRIDE = LS_COLS + 1;   // LDS row of a segment's values over the columns

// Blocks go to the 8 XCDs round-robin by linear id; each XCD takes a contiguous run of column
// blocks, so that two blocks sharing a 128-byte line (FP32 columns) share its L2.
__device__ __forceinline__ unsigned xcd_run(unsigned id, unsigned total) {
  return total % 8 == 0 ? (id % 8) * (total / 8) + id / 8 : id;
}

// The recurrences over one segment from zero: its last value going down (t) and the first value
// coming back up (h); v keeps the downward values.
template <int M>
__device__ __forceinline__ void line_down(double lam, double (&v)[M], double* t, double* h) {
#pragma unroll
  for (int k = 1; k < M; ++k) v[k] = __builtin_fma(lam, v[k - 1], v[k]);
  double up = v[M - 1];
#pragma unroll
  for (int k = M - 2; k >= 0; --k) up = __builtin_fma(lam, up, v[k]);
  *t = v[M - 1];
  *h = up;
}

// Add the true downward carry c and come back up from the true upward carry z, storing g z_k (SPLIT:
// as the split operand, 64 bytes per row where the block's 16 columns, in paired order, stood).
template <typename T, int M, bool SPLIT>
__device__ __forceinline__ void line_up(double lam, double g, double (&v)[M], double c, double z,
                                        T* __restrict__ col, int n) {
  const int cl = threadIdx.x % LS_COLS;
#pragma unroll
  for (int k = 0; k < M; ++k) {
    c *= lam;
    v[k] += c;
  }
#pragma unroll
  for (int k = M - 1; k >= 0; --k) {
    z = __builtin_fma(lam, z, v[k]);
    if constexpr (SPLIT) {
      const float x = (float)(g * z);
      const float y = __int_as_float(
          __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, false));
      store_split(col - cl + (int64_t)k * n, cl < 8 ? cl : 15 - cl, cl < 8, x, y);
    } else {
      gst<T>(col + (int64_t)k * n, (T)(g * z));
    }
  }
}

// P = lambda^M and G = sum_{k<M} lambda^(2k+1) = lambda (1 + lambda^2)(1 + lambda^4) .. (1 +
// lambda^M), M a power of two: what a carry becomes over a segment, down, and down and back up.
template <int M>
__device__ __forceinline__ void line_powers(double lam, double* P, double* G) {
  double p = lam, g = lam;
#pragma unroll
  for (int k = 1; k < M; k *= 2) {
    p *= p;
    g = __builtin_fma(g, p, g);
  }
  *P = p;
  *G = g;
}

// The value of lane l - N or l + N of the same row of 16 lanes, 0 past the row's end.
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Chain the segments of a column over the lanes of a wave: lane s holds t and h of segment s (t,
// h and G zero past the last), and leaves with its carries (the downward value before, the upward value after
// the segment).  The two recurrences over the lanes are scans with the weights P, P^2, P^4, P^8
// inside the rows of 16 lanes; WIDE carries them from row to row (one column of up to 64 segments
// per wave), otherwise each row is a column of its own.
template <bool WIDE>
__device__ __forceinline__ void line_chain(int lane, double P, double G, double kappa, double* t,
                                           double* h) {
  const int r = lane & 15;
  const double P2 = P * P, P4 = P2 * P2, P8 = P4 * P4, P16 = P8 * P8;
  const double up = (r & 1 ? P : 1.0) * (r & 2 ? P2 : 1.0) * ((r & 4 ? P4 : 1.0) * (r & 8 ? P8 : 1.0));
  const int q = 15 - r;
  const double dn = (q & 1 ? P : 1.0) * (q & 2 ? P2 : 1.0) * ((q & 4 ? P4 : 1.0) * (q & 8 ? P8 : 1.0));
  // sum_{k <= s} P^(s-k) t_k, then the carry before each segment (c_0 = 0)
  double c = *t;
  c = __builtin_fma(P, row_move<0x111>(c), c);
  c = __builtin_fma(P2, row_move<0x112>(c), c);
  c = __builtin_fma(P4, row_move<0x114>(c), c);
  c = __builtin_fma(P8, row_move<0x118>(c), c);
  double first = 1.0;                                // P^s
  if constexpr (WIDE) {
    const double c1 = lane_value(c, 15), c2 = __builtin_fma(P16, c1, lane_value(c, 31));
    const double c3 = __builtin_fma(P16, c2, lane_value(c, 47));
    const double cr = lane < 16 ? 0.0 : (lane < 32 ? c1 : (lane < 48 ? c2 : c3));
    c = __builtin_fma(up * P, cr, c);
    c = lane_below(c);
    first = up * (lane < 16 ? 1.0 : (lane < 32 ? P16 : (lane < 48 ? P16 * P16 : P16 * P16 * P16)));
  } else {
    c = row_move<0x111>(c);
    first = up;
  }
  // sum_{k >= s} P^(k-s) x_k
  auto sums_above = [&](double x) {
    x = __builtin_fma(P, row_move<0x101>(x), x);
    x = __builtin_fma(P2, row_move<0x102>(x), x);
    x = __builtin_fma(P4, row_move<0x104>(x), x);
    x = __builtin_fma(P8, row_move<0x108>(x), x);
    if constexpr (WIDE) {
      const double d2 = lane_value(x, 48), d1 = __builtin_fma(P16, d2, lane_value(x, 32));
      const double d0 = __builtin_fma(P16, d1, lane_value(x, 16));
      const double dr = lane < 16 ? d0 : (lane < 32 ? d1 : (lane < 48 ? d2 : 0.0));
      x = __builtin_fma(dn * P, dr, x);
    }
    return x;
  };
  const double z = sums_above(__builtin_fma(c, G, *h));
  const double z0 = WIDE ? lane_value(z, 0) : __shfl(z, lane & 48, 64);
  c = __builtin_fma(-kappa * z0, first, c);
  const double v = sums_above(__builtin_fma(c, G, *h));
  *t = c;
  *h = WIDE ? lane_above(v) : row_move<0x101>(v);
}

// ns = blockDim.x / 16 segments of M rows: n = ns M.
template <typename T, int M, bool SPLIT>
__global__ __launch_bounds__(LS_COLS * LS_SEGS) void k_lines2d(const Lvl2D* __restrict__ levels,
                                                               int64_t sigma) {
  __shared__ double ex[2][LS_SEGS * LS_STRIDE], pw[3][LS_COLS];
  const unsigned q = xcd_run(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const Lvl2D& L = levels[q / gridDim.x];
  int64_t m;
  if (!level_active(L, sigma, &m)) return;
  const int n = L.n, cl = threadIdx.x % LS_COLS;
  const int at = (int)(q % gridDim.x) * LS_COLS + cl, j = SPLIT ? paired_col(at, n) : at;
  const int seg = threadIdx.x / LS_COLS, ns = blockDim.x / LS_COLS;
  T* __restrict__ col =
      (sizeof(T) == 8 ? (T*)L.x64 : (T*)L.lo1) + (int64_t)seg * M * n + at;
  double v[M];
#pragma unroll
  for (int k = 0; k < M; ++k) v[k] = (double)gld<T>(col + (int64_t)k * n);
  const double lam = gld<double>(L.col + j), g = gld<double>(L.col + n + j);
  const double kappa = gld<double>(L.col + 2 * n + j);
  double t, h, P, G;
  line_down<M>(lam, v, &t, &h);
  line_powers<M>(lam, &P, &G);
  ex[0][seg * LS_STRIDE + cl] = t;
  ex[1][seg * LS_STRIDE + cl] = h;
  if (seg == 0) {
    pw[0][cl] = P;
    pw[1][cl] = G;
    pw[2][cl] = kappa;
  }
  __syncthreads();
  // the waves share the block's 16 columns: a column of more than 16 segments takes a wave's 64
  // lanes, four shorter ones take its four rows of 16
  {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (wave >= nw) {
      // the last wave may be a part of one: it takes no column (its lanes cannot all move)
    } else if (ns > 16) {
      for (int cc = wave; cc < LS_COLS; cc += nw) {
        const bool in = lane < ns;
        double a = in ? ex[0][lane * LS_STRIDE + cc] : 0.0, b = in ? ex[1][lane * LS_STRIDE + cc] : 0.0;
        line_chain<true>(lane, pw[0][cc], in ? pw[1][cc] : 0.0, pw[2][cc], &a, &b);
        if (in) {
          ex[0][lane * LS_STRIDE + cc] = a;
          ex[1][lane * LS_STRIDE + cc] = b;
        }
      }
    } else {
      for (int c4 = wave; c4 < LS_COLS / 4; c4 += nw) {
        const int cc = c4 * 4 + (lane >> 4), sg = lane & 15;
        const bool in = sg < ns;
        double a = in ? ex[0][sg * LS_STRIDE + cc] : 0.0, b = in ? ex[1][sg * LS_STRIDE + cc] : 0.0;
        line_chain<false>(lane, pw[0][cc], in ? pw[1][cc] : 0.0, pw[2][cc], &a, &b);
        if (in) {
          ex[0][sg * LS_STRIDE + cc] = a;
          ex[1][sg * LS_STRIDE + cc] = b;
        }
      }
    }
  }
  __syncthreads();
  line_up<T, M, SPLIT>(lam, g, v, ex[0][seg * LS_STRIDE + cl], ex[1][seg * LS_STRIDE + cl], col, n);
}

// Columns of more than 64 segments of 32 rows (n > 2048): the block walks its columns 2048 rows
// at a time, twice (the second walk reads the rows again instead of keeping them); t and h of
// all n / 32 segments stay in LDS (at most 128 KB), where one thread per column turns them into
// the segments' carries.
template <typename T, bool SPLIT>
__global__ __launch_bounds__(LS_COLS * LS_SEGS) void k_lines2d_long(const Lvl2D* __restrict__ levels,
                                                                    int64_t sigma) {
  constexpr int M = 32;
  extern __shared__ double exl[];
  const unsigned q = xcd_run(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const Lvl2D& L = levels[q / gridDim.x];
  int64_t m;
  if (!level_active(L, sigma, &m)) return;
  const int n = L.n, cl = threadIdx.x % LS_COLS, ns = n / M;
  const int at = (int)(q % gridDim.x) * LS_COLS + cl, j = SPLIT ? paired_col(at, n) : at;
  T* __restrict__ col0 = (sizeof(T) == 8 ? (T*)L.x64 : (T*)L.lo1) + at;
  double* tt = exl;
  double* hh = exl + ns * LS_COLS;
  const double lam = gld<double>(L.col + j), g = gld<double>(L.col + n + j);
  const double kappa = gld<double>(L.col + 2 * n + j);
  double v[M];
  for (int seg = threadIdx.x / LS_COLS; seg < ns; seg += LS_SEGS) {
    const T* __restrict__ col = col0 + (int64_t)seg * M * n;
#pragma unroll
    for (int k = 0; k < M; ++k) v[k] = (double)gld<T>(col + (int64_t)k * n);
    line_down<M>(lam, v, &tt[seg * LS_COLS + cl], &hh[seg * LS_COLS + cl]);
  }
  __syncthreads();
  if (threadIdx.x < LS_COLS) {
    double P, G, c = 0.0, z = 0.0, w = 1.0;
    line_powers<M>(lam, &P, &G);
    for (int s = 0; s < ns; ++s) {
      z = __builtin_fma(w, __builtin_fma(c, G, hh[s * LS_COLS + cl]), z);
      c = __builtin_fma(P, c, tt[s * LS_COLS + cl]);
      w *= P;
    }
    c = -kappa * z;
    for (int s = 0; s < ns; ++s) {           // tt: the carry before a segment; hh: its first value
      const double t = tt[s * LS_COLS + cl];
      hh[s * LS_COLS + cl] = __builtin_fma(c, G, hh[s * LS_COLS + cl]);
      tt[s * LS_COLS + cl] = c;
      c = __builtin_fma(P, c, t);
    }
    z = 0.0;
    for (int s = ns - 1; s >= 0; --s) {      // hh: the carry after a segment
      const double h = hh[s * LS_COLS + cl];
      hh[s * LS_COLS + cl] = z;
      z = __builtin_fma(P, z, h);
    }
  }
  __syncthreads();
  for (int seg = threadIdx.x / LS_COLS; seg < ns; seg += LS_SEGS) {
    T* __restrict__ col = col0 + (int64_t)seg * M * n;
#pragma unroll
    for (int k = 0; k < M; ++k) v[k] = (double)gld<T>(col + (int64_t)k * n);
    double t, h;
    line_down<M>(lam, v, &t, &h);
    line_up<T, M, SPLIT>(lam, g, v, tt[seg * LS_COLS + cl], hh[seg * LS_COLS + cl], col, n);
  }
}

// Rows per segment: the fewest (8, 16 or 32) that keep a column within 64 segments; n is a
// multiple of 32.
template <typename T, bool SPLIT>
static void launch_lines(const Lvl2D* lv, int cnt, int64_t n, int64_t sigma, hipStream_t st) {
  const dim3 grid((unsigned)(n / LS_COLS), (unsigned)cnt);
  const unsigned t8 = (unsigned)(n / 8 * LS_COLS);
  if (n <= 8 * LS_SEGS)
    hipLaunchKernelGGL((k_lines2d<T, 8, SPLIT>), grid, dim3(t8), 0, st, lv, sigma);
  else if (n <= 16 * LS_SEGS)
    hipLaunchKernelGGL((k_lines2d<T, 16, SPLIT>), grid, dim3(t8 / 2), 0, st, lv, sigma);
  else if (n <= 32 * LS_SEGS)
    hipLaunchKernelGGL((k_lines2d<T, 32, SPLIT>), grid, dim3(t8 / 4), 0, st, lv, sigma);
  else
    hipLaunchKernelGGL((k_lines2d_long<T, SPLIT>), grid, dim3(LS_COLS * LS_SEGS),
                       2 * (size_t)(n / 32) * LS_COLS * sizeof(double), st, lv, sigma);
}

// ---------------------------------------------------------------------------------------------
// transform pass C = A Q along the rows, on the matrix cores
//   block tile BT x BT (128: 8 waves of 64 x 32 or 4 of 64 x 64; 64: 4 waves of 32 x 32; 32: 2
//   waves of 32 x 16), each wave a grid of 16 x 16 MFMA tiles; k staged through LDS in slices of
//   BK with 16-byte global loads
// ---------------------------------------------------------------------------------------------
constexpr int BT0 = 128;     // largest block tile (rows of A x columns of Q)
// Rows per wave, and threads per block of waves of WC columns.  WC = 32 at BT = 128 puts two
// waves on a SIMD; WC = 64 one, with the whole register file and fewer LDS reads per MFMA.
template <int BT>
constexpr int wave_rows() {
  return BT == 128 ? 64 : 32;
}
template <int BT, int WC>
constexpr int pass_threads() {
  return (BT / wave_rows<BT>()) * (BT / WC) * 64;
}

template <int PREC>
struct Tr;

template <>
struct Tr<PREC_F64> {
  typedef double T;
  static constexpr int BK = 16;
  typedef dbl4 Acc;
};
template <>
struct Tr<PREC_F32> {
  typedef float T;
  static constexpr int BK = 32;
  typedef flt4 Acc;
};
template <>
struct Tr<PREC_BF16> {
  typedef u16 T;
  static constexpr int BK = 32;
  typedef flt4 Acc;
};

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef float flt2 __attribute__((ext_vector_type(2)));

// Folding by the reflection symmetry of the sine matrix, Q_{n-1-k, j} = (-1)^j Q_{k, j}:
//   (A Q)_{ij} = sum_{k < n/2} (A_{ik} + (-1)^j A_{i, n-1-k}) Q_{kj},
// so the even output columns take the sums and the odd ones the differences of mirrored columns
// of A, against half of Q.  a holds columns k .. k+e-1 of a row, m the mirrored chunk
// n-k-e .. n-k-1 (its elements in reverse order pair with a's).
__device__ __forceinline__ void fold_f64(u32x4 a, u32x4 m, u32x4* sum, u32x4* dif) {
  const dbl2 x = __builtin_bit_cast(dbl2, a), y = __builtin_bit_cast(dbl2, m);
  *sum = __builtin_bit_cast(u32x4, dbl2{x[0] + y[1], x[1] + y[0]});
  *dif = __builtin_bit_cast(u32x4, dbl2{x[0] - y[1], x[1] - y[0]});
}
__device__ __forceinline__ void fold_f32(u32x4 a, u32x4 m, u32x4* sum, u32x4* dif) {
  const flt4 x = __builtin_bit_cast(flt4, a), y = __builtin_bit_cast(flt4, m);
  *sum = __builtin_bit_cast(u32x4, flt4{x[0] + y[3], x[1] + y[2], x[2] + y[1], x[3] + y[0]});
  *dif = __builtin_bit_cast(u32x4, flt4{x[0] - y[3], x[1] - y[2], x[2] - y[1], x[3] - y[0]});
}
// 4 FP32 values -> BF16 hi and lo, 8 bytes each
__device__ __forceinline__ void split4_bf16(flt4 v, uint2* hi, uint2* lo) {
  unsigned w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = split_bf16(v[e]);
  *hi = uint2{(w[0] & 0xffffu) | (w[1] << 16), (w[2] & 0xffffu) | (w[3] << 16)};
  *lo = uint2{(w[0] >> 16) | (w[1] & 0xffff0000u), (w[2] >> 16) | (w[3] & 0xffff0000u)};
}

// Instruction order of one pipelined k-slice step (a single basic block): NR LDS reads, then
// NW LDS writes and global loads, each placed after one of the step's NM MFMAs, and the rest of
// the MFMAs after them.  Groups with no instruction left to take stay empty.
template <int NM, int NR, int NW>
__device__ __forceinline__ void interleave_step() {
  static_assert(NR + NW <= NM, "one MFMA per memory instruction");
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
    __builtin_amdgcn_sched_group_barrier(0x210, 1, 0);   // LDS write or global load
  }
  __builtin_amdgcn_sched_group_barrier(0x008, NM - NR - NW, 0);
}

// FOLD (n a multiple of 64): the contraction runs over k < n/2 with the folded A operands and
// E.Q the folded transform: row j' (n rows) holds Q_{k, perm(j')} for k < n/2, perm(j') = 2j'
// for j' < n/2 and 2(j' - n/2) + 1 above.  A block takes BT consecutive output columns, its
// first BT/2 local columns the even ones (against the sums), the others the odd ones (against
// the differences); a wave's columns are all of one parity.
// A folded split-BF16 pass takes a split operand (store_split): its 16-byte chunks go to LDS as they
// are, four planes (sums hi, lo, differences hi, lo) whose LDS starts are 32 bytes apart modulo the 128
// of all banks, so that the four chunks of 8 k and the next four meet no bank twice.
// KX = 2 doubles the k-slice (split BF16: one slice in flight instead of two).  A k-slice has
// two LDS stages (the next slice is stored while the current one feeds the matrix cores, one
// barrier per slice), except the wide split-BF16 slices, whose operands fill one stage's worth of
// the LDS twice over.  Most variants need more than 64 KB, so every variant takes its LDS
// dynamically (pass_lds_bytes).
template <int PREC, int KX>
constexpr int lds_stages() {
  return PREC == PREC_BF16 && KX == 2 ? 1 : 2;
}
// Bytes between the LDS rows of an operand: a slice's row is a multiple of 64 bytes, and rows at a
// stride of 32 modulo 64 are what 16 lanes reading 16 bytes each of 16 rows need to meet all 64 banks
// once (4 cycles a fragment; 8 at a padding of 16, and a write at either takes 8).
constexpr int ROW_PAD = 32;
template <int PREC, int FOLD>
constexpr bool split_a() {
  return PREC == PREC_BF16 && FOLD;
}
template <int PREC, int KX, int BT>
constexpr size_t pass_lds_bytes(int fold) {
  typedef typename Tr<PREC>::T T;
  typedef typename std::conditional<PREC == PREC_F64, double, float>::type ST;
  constexpr int BK = Tr<PREC>::BK * KX;
  constexpr int LDE = (BK * (int)sizeof(T) + ROW_PAD) / (int)sizeof(T);
  constexpr int NSPLIT = PREC == PREC_BF16 ? 2 : 1;
  const size_t pad = PREC == PREC_BF16 && fold ? 4 * 32 : 0;
  const size_t k = (size_t)lds_stages<PREC, KX>() *
                   (((fold ? 2 : 1) * NSPLIT + NSPLIT) * BT * LDE * sizeof(T) + pad);
  const size_t ep = (size_t)(PREC == PREC_F64 && BT == 128 ? 32 : BT) * (BT * sizeof(ST) + 16);
  return k > ep ? k : ep;
}

// DEEP (small tiles, a multiple of four slices): four slices' loads in flight instead of two.
template <int PREC, int OUT, int FOLD, int KX, int BT, int WC, bool DEEP = false>
__global__ __launch_bounds__((pass_threads<BT, WC>())) void k_pass2d(
    const Pass2D* __restrict__ passes, const Lvl2D* __restrict__ levels, int64_t sigma) {
  constexpr int NTHR = pass_threads<BT, WC>();
  constexpr int WM = wave_rows<BT>();
  constexpr int MT = WM / 16, NB = WC / 16;           // 16 x 16 MFMA tiles per wave
  typedef Tr<PREC> TR;
  typedef typename TR::T T;
  typedef typename TR::Acc Acc;
  constexpr int BK = TR::BK * KX;
  constexpr int ROWB = BK * (int)sizeof(T) + ROW_PAD;   // LDS row stride in bytes
  constexpr int LDE = ROWB / (int)sizeof(T);          // ... in elements
  constexpr int CH = BK * (int)sizeof(T) / 16;        // 16-byte chunks per row
  constexpr int NSPLIT = PREC == PREC_BF16 ? 2 : 1;
  constexpr int CPT = BT * CH / NTHR;                 // chunks per thread per operand and split
  constexpr int NA = FOLD ? 2 : 1;                    // A operands in LDS (sums, differences)
  static_assert(BT * CH % NTHR == 0, "whole chunks per thread");
  extern __shared__ __attribute__((aligned(16))) unsigned char pass_smem[];
  // LDS stage b of a k-slice: the A operands, then Q
  constexpr bool SPLITA = split_a<PREC, FOLD>();
  constexpr int APL = BT * LDE + (SPLITA ? 16 : 0);   // elements of an A plane
  constexpr size_t A_BYTES = (size_t)NA * NSPLIT * APL * sizeof(T);
  constexpr size_t STAGE_BYTES = A_BYTES + (size_t)NSPLIT * BT * LDE * sizeof(T);
  auto stage_a = [&](int b) {
    return reinterpret_cast<T (*)[NSPLIT][APL]>(pass_smem + b * STAGE_BYTES);
  };
  auto stage_b = [&](int b) {
    return reinterpret_cast<T (*)[BT * LDE]>(pass_smem + b * STAGE_BYTES + A_BYTES);
  };

  // XCD-aware tile order: each XCD takes a contiguous run of tiles, and the column tiles of one
  // row tile of A meet in one L2
  unsigned bx, by, bz;
  {
    const unsigned t = gridDim.x;
    const unsigned q = xcd_run(blockIdx.x + t * (blockIdx.y + gridDim.y * blockIdx.z),
                               t * gridDim.y * gridDim.z);
    bx = q % t;
    by = (q / t) % gridDim.y;
    bz = q / (t * gridDim.y);
  }
  const Pass2D& E = passes[bz];
  const Lvl2D& L = levels[bz];
  int64_t m;
  if (!level_active(L, sigma, &m)) return;
  const int n = L.n;
  const int row0 = by * BT, col0 = bx * BT;
  if (row0 >= n || col0 >= n) return;
  const int64_t nn = (int64_t)n * n;
  const int half = n >> 1;
  // A arrives row-major in FP64 or FP32 (the split-BF16 pass splits it while staging); Q in T
  typedef typename std::conditional<PREC == PREC_BF16, float, T>::type TA;
  constexpr int EA = 16 / (int)sizeof(TA);          // A elements per 16-byte chunk
  constexpr int CHA = BK * (int)sizeof(TA) * (SPLITA ? 2 : 1) / 16;   // A chunks per row
  constexpr int NAC = BT * CHA / NTHR;              // A chunks per thread
  static_assert(BT * CHA % NTHR == 0, "whole A chunks per thread");
  const TA* A = (const TA*)E.A;
  const T* Q = (const T*)E.Q;
  const int K = FOLD ? half : n;                    // contraction length
  const int64_t qsplit = (int64_t)n * K;            // BF16: lo part of the transform
  constexpr int E16 = 16 / (int)sizeof(T);          // elements per 16-byte chunk
  // row of Q of local column c (rows past n read a row in range; their columns are never stored)
  auto q_row = [&](int c) {
    if constexpr (FOLD) {
      if (SPLITA && E.paired) {
        const int p = col0 + (c < BT / 2 ? 2 * c : 2 * (c - BT / 2) + 1);
        const int j = paired_col(p < n ? p : n - 1, n);
        return (j & 1 ? half : 0) + (j >> 1);
      }
      const int e = (col0 >> 1) + (c < BT / 2 ? c : c - BT / 2);
      return (c < BT / 2 ? 0 : half) + (e < half ? e : half - 1);
    } else {
      return col0 + c < n ? col0 + c : n - 1;
    }
  };

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = (wave / (BT / WC)) * WM;    // wave tile origin inside the block
  const int wn = (wave % (BT / WC)) * WC;

  // The FP32 accumulators go to the accumulation registers (the empty asm asks for the class):
  // left among the vector registers, the allocator renamed some of them through registers that
  // the next fragment loads write, which the build rejects.
  Acc acc[MT][NB];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      Acc z = Acc{0, 0, 0, 0};
      if constexpr (PREC != PREC_F64) asm volatile("" : "+a"(z));
      acc[a][b] = z;
    }

  // global -> register staging of one k-slice (A, its mirrored columns when folding, Q); a
  // slice's loads are issued one MFMA phase before they are stored into LDS.  Rows past n (a
  // partial block tile) read row n-1 instead: they only reach output rows past n, which the
  // epilogue never stores, and no select on the loaded values makes a step wait for its loads.
  // row of Q chunk id: in order, but the 8 lanes of a write that hold two rows of 64 bytes hold rows r
  // and r + 2, which are 64 bytes apart modulo the 128 that a cycle writes
  auto q_chunk_row = [](int id) {
    const int r = id / CH;
    return CH == 4 ? (r & ~3) | ((r & 1) << 1) | ((r >> 1) & 1) : r;
  };
  struct Slice {
    u32x4 ra[NAC], rm[FOLD && !SPLITA ? NAC : 1], rb[NSPLIT][CPT];
  };
  auto gload = [&](Slice& S, int k0) {
#pragma unroll
    for (int c = 0; c < NAC; ++c) {
      const int id = tid + c * NTHR;
      const int r = id / CHA, q = id % CHA;
      const int ga = row0 + r;
      const int64_t ko = k0 + q * EA;
      const TA* arow = A + (int64_t)(ga < n ? ga : n - 1) * n;
      if constexpr (SPLITA) {
        S.ra[c] = gld<u32x4>(arow + 2 * k0 + q * EA);
        continue;
      }
      S.ra[c] = gld<u32x4>(arow + ko);
      if constexpr (FOLD && !SPLITA) S.rm[c] = gld<u32x4>(arow + (n - ko - EA));
    }
#pragma unroll
    for (int s = 0; s < NSPLIT; ++s)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int id = tid + c * NTHR;
        const int r = q_chunk_row(id), q = id % CH;
        const int64_t ko = k0 + q * E16;
        S.rb[s][c] = gld<u32x4>(Q + s * qsplit + (int64_t)q_row(r) * K + ko);
      }
  };
  // Rows keep a slice's k in order.  A lane of an FP32/FP64 fragment takes every fourth 16-byte chunk
  // of its row, from chunk l / 16, so that MFMA (v, e) of the slice multiplies k = EV (4v + l / 16) + e
  // (the same for every shape), EV elements a chunk.
  constexpr int KQ = BK / 4;
  auto put = [&](T* row_base, int q, u32x4 v) { *(u32x4*)((char*)row_base + q * 16) = v; };
  auto sstore = [&](const Slice& S, int stage) {
    T (*As)[NSPLIT][APL] = stage_a(stage);
    T (*Bs)[BT * LDE] = stage_b(stage);
#pragma unroll
    for (int c = 0; c < NAC; ++c) {
      const int id = tid + c * NTHR;
      const int r = id / CHA, q = id % CHA;
      const int ro = r * LDE;                        // row start, in elements
      if constexpr (SPLITA) {
        put(As[(q >> 1) & 1][q & 1] + ro, q >> 2, S.ra[c]);
        continue;
      }
      u32x4 su = S.ra[c], di = S.ra[c];
      if constexpr (FOLD && !SPLITA) {
        if constexpr (PREC == PREC_F64)
          fold_f64(S.ra[c], S.rm[c], &su, &di);
        else
          fold_f32(S.ra[c], S.rm[c], &su, &di);
      }
      if constexpr (PREC == PREC_BF16) {
        // 4 FP32 values -> BF16 hi and lo at elements 4q .. 4q+3
        auto put4 = [&](int a, u32x4 v) {
          uint2 hi, lo;
          split4_bf16(__builtin_bit_cast(flt4, v), &hi, &lo);
          *(uint2*)(As[a][0] + ro + q * 4) = hi;
          *(uint2*)(As[a][1] + ro + q * 4) = lo;
        };
        put4(0, su);
      } else {
        put(As[0][0] + ro, q, su);
        if constexpr (FOLD) put(As[1][0] + ro, q, di);
      }
    }
#pragma unroll
    for (int s = 0; s < NSPLIT; ++s)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int id = tid + c * NTHR;
        const int r = q_chunk_row(id), q = id % CH;
        put(Bs[s] + r * LDE, q, S.rb[s][c]);
      }
  };

  // the A operand of this wave's columns: sums (0) for even output columns, differences (1) for
  // odd ones
  const int pa0 = FOLD && wn >= BT / 2 ? 1 : 0;
  const int KT = K / BK;
  const int r16 = lane & 15;
  // FP32/FP64: a lane's KQ values of a slice, read 16 bytes at a time
  constexpr int EV = 16 / (int)sizeof(T);
  struct Frag {
    T x[KQ];
  };
  auto frag = [&](const T* row) {
    Frag f;
    const int k4 = lane >> 4;
#pragma unroll
    for (int v = 0; v < KQ / EV; ++v) {
      const u32x4 w = *(const u32x4*)(row + (v * 4 + k4) * EV);
      struct Ev {
        T x[EV];
      };
      const Ev ev = __builtin_bit_cast(Ev, w);
#pragma unroll
      for (int e = 0; e < EV; ++e) f.x[v * EV + e] = ev.x[e];
    }
    return f;
  };
  // this wave's fragments of the slice in LDS stage `stage`: MT tiles of A rows, NB of Q rows
  auto read_frags = [&](int stage, Frag (&fa)[MT], Frag (&fb)[NB]) {
    T (*As)[NSPLIT][APL] = stage_a(stage);
    T (*Bs)[BT * LDE] = stage_b(stage);
#pragma unroll
    for (int t = 0; t < MT; ++t) fa[t] = frag(As[pa0][0] + (wm + t * 16 + r16) * LDE);
#pragma unroll
    for (int t = 0; t < NB; ++t) fb[t] = frag(Bs[0] + (wn + t * 16 + r16) * LDE);
  };
  auto mfma_frags = [&](const Frag (&fa)[MT], const Frag (&fb)[NB]) {
    if constexpr (PREC != PREC_BF16) {
#pragma unroll
      for (int i = 0; i < KQ; ++i)
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            if constexpr (PREC == PREC_F64)
              acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a].x[i], fb[b].x[i],
                                                               acc[a][b], 0, 0, 0);
            else
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a].x[i], fb[b].x[i],
                                                               acc[a][b], 0, 0, 0);
          }
    }
  };
  // split BF16: the hi/lo fragments of one 32-wide k-step ks of a slice (lane holds 8
  // consecutive k of row l % 16, k offset 8 (l / 16)), and its three products: each accumulator
  // takes lo*hi, hi*lo, hi*hi in that order; the accumulators are independent, so one kind of
  // product is issued over all of them before the next
  struct FragB {
    bf16x8 ahi[MT], alo[MT], bhi[NB], blo[NB];
  };
  auto read_frags_bf = [&](int stage, int ks, FragB& f) {
    T (*As)[NSPLIT][APL] = stage_a(stage);
    T (*Bs)[BT * LDE] = stage_b(stage);
    const int kb = (lane >> 4) * 16 + ks * 64;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int ro = (wm + t * 16 + r16) * ROWB + kb;
      f.ahi[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)((const char*)As[pa0][0] + ro));
      f.alo[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)((const char*)As[pa0][NSPLIT - 1] + ro));
    }
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int ro = (wn + t * 16 + r16) * ROWB + kb;
      f.bhi[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)((const char*)Bs[0] + ro));
      f.blo[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)((const char*)Bs[NSPLIT - 1] + ro));
    }
  };
  auto mfma_bf = [&](const FragB& f) {
    if constexpr (PREC == PREC_BF16) {
#pragma unroll
      for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.alo[a], f.bhi[b], acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.ahi[a], f.blo[b], acc[a][b], 0, 0, 0);
#pragma unroll
      for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.ahi[a], f.bhi[b], acc[a][b], 0, 0, 0);
    }
  };
  // the epilogue's geometry: the block tile goes through LDS at once, the large FP64 one in rounds of
  // a tile row of every wave (at 1024^2, four levels, a pass takes 78.0 us in rounds, 79.0 at once;
  // split BF16 20.7 and 20.6)
  constexpr int ROUNDS = PREC == PREC_F64 && BT == 128 ? MT : 1;
  constexpr int AG = MT / ROUNDS;                             // tile rows of a wave per round
  constexpr int RW = 16 * AG;                                 // ... in rows
  typedef typename std::conditional<PREC == PREC_F64, double, float>::type ST;
  constexpr int SS = BT + 16 / (int)sizeof(ST);               // LDS row stride, 16-byte rows
  constexpr int EC = OUT == OUT_F32 ? 4 : 2;                  // elements per chunk
  constexpr int CPR = BT / EC;                                // chunks per row
  constexpr int NC = BT * CPR / NTHR;                         // chunks per thread
  constexpr int GC = BT < 128 ? NC : (NC + 3) / 4;            // ... per group (below)
  constexpr int NG = NC / GC, GR = NG / ROUNDS;               // groups, and groups per round
  static_assert(NC % GC == 0 && NG % ROUNDS == 0, "whole groups");
  static_assert(BT * CPR % NTHR == 0, "whole chunks per thread");
  ST* stg = reinterpret_cast<ST*>(pass_smem);
  double* out64 = nullptr;
  const double* base = nullptr;
  if constexpr (OUT == OUT_FINAL) {
    out64 = L.own + ring_slot(m, L.R_own) * nn;
    base = L.j == 0 ? L.own + ring_slot(m - 1, L.R_own) * nn : L.prev + ring_slot(m, L.R_prev) * nn;
  }
  // output row of accumulator element r: FP32 tiles hold rows 4(l/16) + r, FP64 tiles hold
  // rows (l/16) + 4r (measured lane layouts of the two instructions)
  const int i_base = PREC == PREC_F64 ? (lane >> 4) : 4 * (lane >> 4);
  constexpr int i_step = PREC == PREC_F64 ? 4 : 1;
  auto chunk_at = [&](int g, int c, int* lr, int* lc, int64_t* o) {   // chunk c of group g
    const int id = tid + (g % GR * GC + c) * NTHR;
    *lr = id / CPR;                                  // LDS row: the round's rows of every wave row
    *lc = (id % CPR) * EC;
    const int row = row0 + *lr / RW * WM + g / GR * RW + *lr % RW;
    *o = (int64_t)row * n + col0 + *lc;
    return row < n && col0 + *lc < n;                // n is a multiple of 32: whole chunks
  };
  // the final update's FP64 operands (base, add) of this thread's chunks, in groups of GC: all of them
  // before the k-loop of the small tiles, under which they arrive; in the large ones a group ahead,
  // the first under the last slices
  constexpr int SLOTS = OUT == OUT_FINAL ? (NG > 1 ? 2 : 1) : 1;
  dbl2 bq[SLOTS][GC];
  flt2 aq[SLOTS][GC];
  auto fetch = [&](int g) {
    if constexpr (OUT == OUT_FINAL) {
#pragma unroll
      for (int c = 0; c < GC; ++c) {
        int lr, lc;
        int64_t o;
        if (!chunk_at(g, c, &lr, &lc, &o)) continue;
        bq[g % SLOTS][c] = gld<dbl2>(base + o);
        aq[g % SLOTS][c] = PREC != PREC_F64 && E.add ? gld<flt2>(E.add + o) : flt2{0.0f, 0.0f};
      }
    }
  };
  if constexpr (BT < 128) fetch(0);
  auto kslice = [&](int k) { return (k < KT ? k : KT - 1) * BK; };
  if constexpr (PREC == PREC_BF16 && lds_stages<PREC, KX>() == 1) {
    // wide slices: one in flight, its loads cover a whole MFMA phase of twice the length
    Slice sl;
    gload(sl, 0);
    for (int kt = 0; kt < KT; ++kt) {
      __syncthreads();
      sstore(sl, 0);
      __syncthreads();
      if (kt + 1 < KT) gload(sl, (kt + 1) * BK);
      else fetch(0);
#pragma unroll
      for (int ks = 0; ks < KX; ++ks) {
        FragB f;
        read_frags_bf(0, ks, f);
        mfma_bf(f);
      }
    }
  } else if constexpr (BT < 128) {
    // small tiles: a pass is a few slices long and bound by the latency of its loads, so the
    // loads of two slices, or of four (DEEP), are in flight from the start
    auto multiply = [&](int kt) {
      if constexpr (PREC == PREC_BF16) {
        FragB f;
        read_frags_bf(kt & 1, 0, f);
        mfma_bf(f);
      } else {
        Frag fa[MT], fb[NB];
        read_frags(kt & 1, fa, fb);
        mfma_frags(fa, fb);
      }
    };
    Slice s0, s1;
    if constexpr (DEEP) {
      Slice s2, s3;
      gload(s0, 0);
      gload(s1, BK);
      gload(s2, 2 * BK);
      gload(s3, 3 * BK);
      sstore(s0, 0);
      __syncthreads();
      // `mine` held slice kt, `next` holds slice kt + 1
      auto step = [&](int kt, Slice& mine, Slice& next) {
        gload(mine, (kt + 4) * BK);
        multiply(kt);
        sstore(next, (kt + 1) & 1);
        __syncthreads();
      };
      auto last = [&](int kt, Slice& next) {
        multiply(kt);
        sstore(next, (kt + 1) & 1);
        __syncthreads();
      };
      int kt = 0;
      for (; kt + 4 < KT; kt += 4) {
        step(kt, s0, s1);
        step(kt + 1, s1, s2);
        step(kt + 2, s2, s3);
        step(kt + 3, s3, s0);
      }
      last(kt, s1);
      last(kt + 1, s2);
      last(kt + 2, s3);
      multiply(kt + 3);
    } else {
      gload(s0, 0);
      if (KT > 1) gload(s1, BK);
      sstore(s0, 0);
      __syncthreads();
      auto step = [&](int kt, Slice& mine, Slice& next) {
        if (kt + 2 < KT) gload(mine, (kt + 2) * BK);
        multiply(kt);
        if (kt + 1 < KT) sstore(next, (kt + 1) & 1);
        __syncthreads();
      };
      for (int kt = 0; kt < KT; kt += 2) {
        step(kt, s0, s1);
        if (kt + 1 < KT) step(kt + 1, s1, s0);
      }
    }
  } else {
    // Two LDS stages and two register sets of fragments.  Step kt issues the MFMAs of slice kt from
    // registers while the fragments of slice kt+1 are read from LDS, slice kt+2 is stored into the
    // stage slice kt came from (read into registers before the previous barrier) and slice kt+3
    // (TWO: and kt+4, where the registers hold two slices) is loading: one barrier per slice.  A step
    // is one basic block (loads past the end re-read the last slice and are never used), so that
    // its LDS and global memory instructions can be issued one between each pair of MFMAs
    // (interleave_step): the memory work runs under the matrix cores instead of between them.
    // The last two slices have nothing left to load, and a final update's first operands come in
    // under them (not in FP64, whose registers are full).
    auto run = [&](auto read, auto mfma, auto& f0, auto& f1, auto interleave) {
      constexpr bool TWO = PREC == PREC_BF16 && OUT != OUT_FINAL;
      Slice s0, s1;
      gload(s0, 0);
      gload(s1, kslice(1));
      sstore(s0, 0);
      gload(s0, kslice(2));
      __syncthreads();
      read(0, f0);
      sstore(s1, 1);
      if constexpr (TWO) gload(s1, kslice(3));
      __syncthreads();
      auto step = [&](int kt, Slice& sl, const auto& cur, auto& next) {
        read((kt + 1) & 1, next);
        sstore(sl, kt & 1);
        gload(sl, kslice(kt + (TWO ? 4 : 3)));
        mfma(cur);
        interleave();
        __syncthreads();
      };
      Slice& odd = TWO ? s1 : s0;
      if constexpr (PREC == PREC_F64) {
        for (int kt = 0; kt < KT; kt += 2) {
          step(kt, s0, f0, f1);
          if (kt + 1 < KT) step(kt + 1, s0, f1, f0);
        }
        fetch(0);
        return;
      }
      int kt = 0;
      for (; kt + 3 < KT; kt += 2) {
        step(kt, s0, f0, f1);
        step(kt + 1, odd, f1, f0);
      }
      if (kt + 3 == KT) {
        step(kt, s0, f0, f1);
        fetch(0);
        read((kt + 2) & 1, f0);
        mfma(f1);
        mfma(f0);
      } else {
        fetch(0);
        if (kt + 2 == KT) read((kt + 1) & 1, f1);
        mfma(f0);
        if (kt + 2 == KT) mfma(f1);
      }
    };
    if constexpr (PREC == PREC_BF16) {
      FragB f0, f1;
      run([&](int st, FragB& f) { read_frags_bf(st, 0, f); }, [&](const FragB& f) { mfma_bf(f); },
          f0, f1, [] { interleave_step<3 * MT * NB, 2 * (MT + NB), MT * NB * 3 - 2 * (MT + NB)>(); });
    } else {
      struct Fr {
        Frag a[MT], b[NB];
      };
      Fr f0, f1;
      constexpr int NM = KQ * MT * NB, NR = KQ / EV * (MT + NB);   // MFMAs, 16-byte reads
      run([&](int st, Fr& f) { read_frags(st, f.a, f.b); },
          [&](const Fr& f) { mfma_frags(f.a, f.b); }, f0, f1,
          [] { interleave_step<NM, NR, (NM - NR < 24 ? NM - NR : 24)>(); });
    }
  }

  // epilogue: acc[a][b] holds the 16 x 16 tile at local rows wm + 16a, local columns wn + 16b
  // (column l%16 of lane l).  A round goes through LDS, the columns put back in their natural
  // order; each thread then finishes and writes 16-byte chunks, consecutive threads consecutive
  // chunks of a row.
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (g % GR == 0) {
      __syncthreads();                                // the buffer is free
#pragma unroll
      for (int ar = 0; ar < AG; ++ar)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int c = wn + 16 * b + r16;
          const int nat = FOLD ? (c < BT / 2 ? 2 * c : 2 * (c - BT / 2) + 1) : c;
          ST* dst = stg + (wm / WM * RW + 16 * ar + i_base) * SS + nat;
#pragma unroll
          for (int r = 0; r < 4; ++r) dst[i_step * r * SS] = acc[g / GR * AG + ar][b][r];
        }
      __syncthreads();
    }
    if (g + 1 < NG) fetch(g + 1);
#pragma unroll
    for (int c = 0; c < GC; ++c) {
      int lr, lc;
      int64_t o;
      if (!chunk_at(g, c, &lr, &lc, &o)) continue;
      const ST* src = stg + lr * SS + lc;
      if constexpr (OUT == OUT_F64) {
        gst<dbl2>((double*)E.C + o, *(const dbl2*)src);
      } else if constexpr (OUT == OUT_F32) {
        gst<flt4>((float*)E.C + o, *(const flt4*)src);
      } else {
        const dbl2 bs = bq[g % SLOTS][c];
        if constexpr (PREC == PREC_F64) {
          gst<dbl2>(out64 + o, dbl2{bs[0] + src[0], bs[1] + src[1]});
        } else {
          const flt2 ad = aq[g % SLOTS][c];
          gst<dbl2>(out64 + o, dbl2{bs[0] + ((double)ad[0] + (double)src[0]),
                                    bs[1] + ((double)ad[1] + (double)src[1])});
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
namespace {

// Systems whose side is a multiple of 64 use the folded transform (their plans hold it).
bool folded(int64_t n) { return n % 64 == 0; }

struct Transform {
  double* q64 = nullptr;
  float* q32 = nullptr;
  u16* qbf = nullptr;
};
std::mutex g_tf_mu;
std::map<int64_t, Transform> g_tf;  // per n, per device id in the high bits; kept until exit

int get_transform(int64_t n, int prec, Transform* out) {
  int dev = 0;
  RIDC_HIP_TRY(hipGetDevice(&dev));
  const int64_t key = ((int64_t)dev << 40) | n;
  std::lock_guard<std::mutex> lk(g_tf_mu);
  Transform& t = g_tf[key];
  const int64_t nn = n * n;
  if ((prec == PREC_F64 && !t.q64) || (prec == PREC_F32 && !t.q32) ||
      (prec == PREC_BF16 && !t.qbf)) {
    // Q_{ik} = sqrt(2/(n+1)) sin(pi (i+1)(k+1)/(n+1)), argument reduced exactly mod 2(n+1)
    std::vector<double> q(nn);
    const long double scale = std::sqrt(2.0L / (long double)(n + 1));
    const long double pi = 3.141592653589793238462643383279502884L;
    const int64_t period = 2 * (n + 1);
    std::vector<long double> s(period);
    for (int64_t k = 0; k < period; ++k) s[k] = scale * std::sin(pi * (long double)k / (n + 1));
    for (int64_t i = 0; i < n; ++i)
      for (int64_t k = 0; k < n; ++k) q[i * n + k] = (double)s[((i + 1) * (k + 1)) % period];
    // folded systems keep rows j' of Q_{k, perm(j')}, k < n/2 (see k_pass2d); others all of Q
    int64_t cnt = nn;
    if (folded(n)) {
      const int64_t K = n / 2;
      std::vector<double> qh(n * K);
      for (int64_t jp = 0; jp < n; ++jp) {
        const int64_t j = jp < K ? 2 * jp : 2 * (jp - K) + 1;
        for (int64_t k = 0; k < K; ++k) qh[jp * K + k] = q[k * n + j];
      }
      q.swap(qh);
      cnt = n * K;
    }
    if (prec == PREC_F64) {
      if (hipMalloc(&t.q64, cnt * sizeof(double)) != hipSuccess) return fail(RIDC_E_NOMEM, "Q64");
      RIDC_HIP_TRY(hipMemcpy(t.q64, q.data(), cnt * sizeof(double), hipMemcpyHostToDevice));
    } else if (prec == PREC_F32) {
      std::vector<float> qf(cnt);
      for (int64_t i = 0; i < cnt; ++i) qf[i] = (float)q[i];
      if (hipMalloc(&t.q32, cnt * sizeof(float)) != hipSuccess) return fail(RIDC_E_NOMEM, "Q32");
      RIDC_HIP_TRY(hipMemcpy(t.q32, qf.data(), cnt * sizeof(float), hipMemcpyHostToDevice));
    } else {
      std::vector<u16> qb(2 * cnt);
      for (int64_t i = 0; i < cnt; ++i) {
        // round to nearest even BF16 of the FP32 value, then of the FP32 remainder
        auto to_bf = [](float f) -> u16 {
          uint32_t u = __builtin_bit_cast(uint32_t, f);
          u += 0x7fff + ((u >> 16) & 1);
          return (u16)(u >> 16);
        };
        auto from_bf = [](u16 b) -> float { return __builtin_bit_cast(float, (uint32_t)b << 16); };
        const float f = (float)q[i];
        const u16 hi = to_bf(f);
        const u16 lo = to_bf(f - from_bf(hi));
        qb[i] = hi;
        qb[cnt + i] = lo;
      }
      if (hipMalloc(&t.qbf, 2 * cnt * sizeof(u16)) != hipSuccess) return fail(RIDC_E_NOMEM, "Qbf");
      RIDC_HIP_TRY(hipMemcpy(t.qbf, qb.data(), 2 * cnt * sizeof(u16), hipMemcpyHostToDevice));
    }
  }
  *out = t;
  return RIDC_OK;
}

int prec_of(const ridc_problem* p) {
  return p->prec == RIDC_PREC_FP64 ? PREC_F64 : (p->prec == RIDC_PREC_FP32_REFINE ? PREC_F32 : PREC_BF16);
}

size_t level_ws_bytes(int64_t n, int prec) {
  const size_t nn = (size_t)n * n;
  if (prec == PREC_F64) return 2 * nn * sizeof(double);             // b64, x64 (intermediate)
  return 2 * nn * sizeof(double) + 2 * nn * sizeof(float);          // b64, x64, lo0, lo1
}

// Whether the passes of a system take split operands (store_split).
bool split_operands(int prec, int64_t n) { return prec == PREC_BF16 && folded(n); }

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Wide k-slices for the split-BF16 pass are possible when the folded contraction is a multiple of twice
// the slice.  An untuned handle takes narrow ones: whole steps, us, wide / narrow, order 4: 1024^2 155.6 /
// 144.2, 768^2 115.3 / 103.1, 512^2 60.2 / 60.5 (no 128-tiles).
template <int PREC>
bool wide_slices(int64_t n) {
  return PREC == PREC_BF16 && folded(n) && (n / 2) % (2 * Tr<PREC>::BK) == 0;
}

// 64-column waves (tile bit kPassWide64) are possible when the fold cannot split a wave's
// columns between sums and differences (n/2 a multiple of 64, or no fold), for the FP32 and
// FP64 passes; the split-BF16 pass takes 64-wide k-slices unless tile bit kPassNarrowK asks for
// 32-wide ones.  Every shape issues the same MFMA sequence for every output element.
template <int PREC>
bool wide_waves(int64_t n, int tile) {
  return PREC != PREC_BF16 && (tile & kPassWide64) && (!folded(n) || n % 128 == 0);
}

// Block tile of a pass over `cnt` levels of side n: 128 while that fills half of the 256 compute
// units, then 64 while that gives every unit more than one block (split BF16: one, its blocks
// being bound by LDS work and not by latency), else 32, so that a small grid is not left to a few
// units.  Whole steps, us, for tiles of 32 / 64 / 128: 256^2 FP64 order 4 25.3 / 32.8 / 54.9, 512^2
// FP32 order 2 57.4 / 60.0 / 108, 512^2 order 4 FP64 53.1 / 54.0 / 91.2 and split BF16 64.5 / 63.0 /
// 80.3, 768^2 split BF16 order 3 120 / 94.4 / 106 and FP64 order 4 141 / 148 / 134, 1024^2 FP64
// order 4 285 / 237 / 178 and order 1 79.6 / 81.7 / 149.  The tile does not change an output
// element's MFMA sequence, hence no bit of it.
template <int PREC>
int block_tile(int64_t n, int cnt) {
  auto blocks = [&](int64_t t) { return ((n + t - 1) / t) * ((n + t - 1) / t) * cnt; };
  if (blocks(128) >= 128) return 128;
  return blocks(64) >= (PREC == PREC_BF16 ? 256 : 257) ? 64 : 32;
}

// One transform pass.
template <int PREC, int OUT>
void launch_pass(const Pass2D* d, const Lvl2D* lv, int count, int64_t n, int64_t sigma, int tile,
                 hipStream_t st) {
  auto go = [&](auto kern, int bt, unsigned threads, size_t lds) {
    const unsigned t = (unsigned)((n + bt - 1) / bt);
    hipLaunchKernelGGL(kern, dim3(t, t, count), dim3(threads), lds, st, d, lv, sigma);
  };
  const int bt = block_tile<PREC>(n, count);
  const bool fold = folded(n);
  if (bt == 128) {
    constexpr size_t full = pass_lds_bytes<PREC, 1, 128>(0), half = pass_lds_bytes<PREC, 1, 128>(1);
    if constexpr (PREC != PREC_BF16) {
      if (wide_waves<PREC>(n, tile)) {
        if (fold) go(k_pass2d<PREC, OUT, 1, 1, 128, 64>, 128, pass_threads<128, 64>(), half);
        else go(k_pass2d<PREC, OUT, 0, 1, 128, 64>, 128, pass_threads<128, 64>(), full);
        return;
      }
    } else if (wide_slices<PREC>(n) && !(tile & kPassNarrowK)) {
      go(k_pass2d<PREC, OUT, 1, 2, 128, 32>, 128, pass_threads<128, 32>(),
         pass_lds_bytes<PREC, 2, 128>(1));
      return;
    }
    if (fold) go(k_pass2d<PREC, OUT, 1, 1, 128, 32>, 128, pass_threads<128, 32>(), half);
    else go(k_pass2d<PREC, OUT, 0, 1, 128, 32>, 128, pass_threads<128, 32>(), full);
  } else {
    // Whole steps, us, with two slices / four in flight: 256^2 FP64 order 4 26.1 / 24.0, 512^2 order 2 FP64
    // 44.5 / 41.4, FP32 57.1 / 55.5 and split BF16 49.6 / 46.1, 768^2 order 2 FP32 116 / 104; split BF16
    // in 64-tiles 1024^2 order 1 (256 blocks) 80.2 / 67.0, 512^2 order 4 (256) 61.0 / 55.7 and order 6
    // (384) 79.9 / 79.3, 768^2 order 2 (288) 78.7 / 76.4 and order 3 (432) 86.6 / 86.0.
    // Slices that are not a multiple of four need a test at every load (1-2 % slower at 64^2..384^2).
    const bool deep = fold && n / 2 / Tr<PREC>::BK % 4 == 0;
    if (bt == 64) {
      constexpr size_t half = pass_lds_bytes<PREC, 1, 64>(1);
      if (deep) go(k_pass2d<PREC, OUT, 1, 1, 64, 32, true>, 64, pass_threads<64, 32>(), half);
      else if (fold) go(k_pass2d<PREC, OUT, 1, 1, 64, 32>, 64, pass_threads<64, 32>(), half);
      else go(k_pass2d<PREC, OUT, 0, 1, 64, 32>, 64, pass_threads<64, 32>(), pass_lds_bytes<PREC, 1, 64>(0));
    } else {
      constexpr size_t half = pass_lds_bytes<PREC, 1, 32>(1);
      if (deep) go(k_pass2d<PREC, OUT, 1, 1, 32, 16, true>, 32, pass_threads<32, 16>(), half);
      else if (fold) go(k_pass2d<PREC, OUT, 1, 1, 32, 16>, 32, pass_threads<32, 16>(), half);
      else go(k_pass2d<PREC, OUT, 0, 1, 32, 16>, 32, pass_threads<32, 16>(), pass_lds_bytes<PREC, 1, 32>(0));
    }
  }
}

// Allow every variant launch_pass<PREC, OUT> can launch its LDS (host call, outside any stream
// capture).
template <int PREC, int OUT>
hipError_t allow_lds() {
  hipError_t e = hipSuccess;
  auto add = [&](auto kern, size_t lds) {
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  };
  add(&k_pass2d<PREC, OUT, 0, 1, 128, 32>, pass_lds_bytes<PREC, 1, 128>(0));
  add(&k_pass2d<PREC, OUT, 1, 1, 128, 32>, pass_lds_bytes<PREC, 1, 128>(1));
  add(&k_pass2d<PREC, OUT, 0, 1, 64, 32>, pass_lds_bytes<PREC, 1, 64>(0));
  add(&k_pass2d<PREC, OUT, 1, 1, 64, 32>, pass_lds_bytes<PREC, 1, 64>(1));
  add(&k_pass2d<PREC, OUT, 1, 1, 64, 32, true>, pass_lds_bytes<PREC, 1, 64>(1));
  add(&k_pass2d<PREC, OUT, 0, 1, 32, 16>, pass_lds_bytes<PREC, 1, 32>(0));
  add(&k_pass2d<PREC, OUT, 1, 1, 32, 16>, pass_lds_bytes<PREC, 1, 32>(1));
  add(&k_pass2d<PREC, OUT, 1, 1, 32, 16, true>, pass_lds_bytes<PREC, 1, 32>(1));
  if constexpr (PREC == PREC_BF16) {
    add(&k_pass2d<PREC, OUT, 1, 2, 128, 32>, pass_lds_bytes<PREC, 2, 128>(1));
  } else {
    add(&k_pass2d<PREC, OUT, 0, 1, 128, 64>, pass_lds_bytes<PREC, 1, 128>(0));
    add(&k_pass2d<PREC, OUT, 1, 1, 128, 64>, pass_lds_bytes<PREC, 1, 128>(1));
  }
  return e;
}
template <int PREC>
hipError_t allow_pass() {
  typedef typename std::conditional<PREC == PREC_F64, double, float>::type T;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lines2d_long<T, false>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     2 * (16384 / 32) * LS_COLS * (int)sizeof(double));
  if constexpr (PREC == PREC_BF16)
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_lines2d_long<T, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              2 * (16384 / 32) * LS_COLS * (int)sizeof(double));
  if (e == hipSuccess) e = allow_lds<PREC, PREC == PREC_F64 ? OUT_F64 : OUT_F32>();
  if (e == hipSuccess) e = allow_lds<PREC, OUT_FINAL>();
  return e;
}

// Once per device and precision (the attributes stay; setting them costs 50 us a plan).
hipError_t prepare_pass_kernels(int prec) {
  static std::atomic<unsigned> done[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool known = dev >= 0 && dev < 64;
  if (known && (done[dev].load(std::memory_order_acquire) >> prec & 1u)) return hipSuccess;
  e = prec == PREC_BF16  ? allow_pass<PREC_BF16>()
      : prec == PREC_F32 ? allow_pass<PREC_F32>()
                         : allow_pass<PREC_F64>();
  if (e == hipSuccess && known) done[dev].fetch_or(1u << prec, std::memory_order_release);
  return e;
}

// transform passes of one step: two per solve, two solves on the refined paths
int passes_of(int prec) { return prec == PREC_F64 ? 2 : 4; }

}  // namespace

int plan2d_validate(const ridc_problem* p) {
  if (p->n % 32 != 0) return fail(RIDC_E_UNSUPPORTED, "2D n must be a multiple of 32");
  if (p->n > 16384) return fail(RIDC_E_UNSUPPORTED, "2D n above 16384");
  return RIDC_OK;
}

size_t plan2d_workspace_bytes(const ridc_problem* p) {
  const int P = p->order;
  const int prec = prec_of(p);
  size_t b = 0;
  b += align256(sizeof(Lvl2D) * P);
  b += align256(sizeof(Pass2D) * P * passes_of(prec));
  b += align256(3 * sizeof(double) * (size_t)p->n);                 // line-solve constants
  b += (size_t)P * align256(level_ws_bytes(p->n, prec));
  return b;
}

int plan2d_create(const ridc_problem* p, double h, double* const* ring, const int* R,
                  const double* W, const int64_t* woff, char* ws, size_t ws_bytes,
                  hipStream_t stream, Plan2D** out) {
  auto* pl = new Plan2D();
  pl->p = *p;
  pl->P = p->order;
  pl->prec = prec_of(p);
  pl->n = p->n;
  pl->h = h;
  pl->stream = stream;
  const int P = pl->P;
  const int64_t n = p->n, nn = n * n;
  Transform tf;
  int rc = get_transform(n, pl->prec, &tf);
  if (rc == RIDC_OK && prepare_pass_kernels(pl->prec) != hipSuccess)
    rc = fail(RIDC_E_HIP, "the transform kernels need more LDS than the device allows");
  if (rc != RIDC_OK) {
    delete pl;
    return rc;
  }
  pl->Q64 = tf.q64;
  pl->Q32 = tf.q32;
  pl->Qbf = tf.qbf;
  char* cur = ws;
  pl->d_levels = (Lvl2D*)cur;
  cur += align256(sizeof(Lvl2D) * P);
  pl->npass = passes_of(pl->prec);
  pl->d_passes = (Pass2D*)cur;
  cur += align256(sizeof(Pass2D) * P * pl->npass);
  pl->col = (double*)cur;
  cur += align256(3 * sizeof(double) * n);
  // line-solve constants of column k (k_lines2d), lam_k = dt nu (4/h^2) sin^2(pi (k+1) / (2(n+1)))
  {
    std::vector<double> col(3 * n);
    const long double pi = 3.141592653589793238462643383279502884L;
    const long double r = (long double)p->dt * p->nu / ((long double)h * h);
    for (int64_t k = 0; k < n; ++k) {
      const long double s = std::sin(pi * (long double)(k + 1) / (2.0L * (n + 1)));
      const long double d = 1.0L + 4.0L * r * s * s;                // 1 + lam_k
      const long double g = 2.0L / (d + 2.0L * r + std::sqrt(d * (d + 4.0L * r)));
      const long double lam = r * g;
      // kappa = lambda (1 - lambda^2) / (1 - lambda^{2n+2})
      col[k] = (double)lam;
      col[n + k] = (double)g;
      long double e = lam > 0.0L ? (2 * n + 2) * std::log(lam) : -100.0L;   // below e^-50: nothing
      e = e < -50.0L ? 0.0L : std::exp(e);
      col[2 * n + k] = (double)(lam * (1.0L - lam * lam) / (1.0L - e));
    }
    RIDC_HIP_TRY(hipMemcpy(pl->col, col.data(), col.size() * sizeof(double), hipMemcpyHostToDevice));
  }
  pl->levels.assign(P, Lvl2D{});
  const size_t lws = align256(level_ws_bytes(n, pl->prec));
  for (int j = 0; j < P; ++j) {
    Lvl2D& L = pl->levels[j];
    L.own = ring[j];
    L.prev = j > 0 ? ring[j - 1] : nullptr;
    L.W = j > 0 ? W + woff[j] : nullptr;
    char* lw = cur + j * lws;
    L.b64 = (double*)lw;
    L.x64 = (double*)(lw + nn * sizeof(double));
    if (pl->prec != PREC_F64) {
      L.lo0 = (float*)(lw + 2 * nn * sizeof(double));
      L.lo1 = L.lo0 + nn;
    }
    L.col = pl->col;
    L.nt = 0;
    L.sigma0 = 0;
    L.n = (int32_t)n;
    L.j = j;
    L.R_own = R[j];
    L.R_prev = j > 0 ? R[j - 1] : 1;
    L.fe = p->fe_kind;
    L.prec = pl->prec;
    L.dt = p->dt;
    L.nu_h2 = p->nu / (h * h);
  }
  cur += P * lws;
  if ((size_t)(cur - ws) > ws_bytes) {
    delete pl;
    return fail(RIDC_E_NOMEM, "2D workspace layout overflow");
  }
  // pass tables: pass k, level j at passes[k * P + j]
  pl->passes.assign(pl->npass * P, Pass2D{});
  for (int j = 0; j < P; ++j) {
    Lvl2D& L = pl->levels[j];
    for (int k = 0; k < pl->npass; ++k) {
      Pass2D& E = pl->passes[k * P + j];
      // even passes: the right-hand side or residual to its sine coefficients; odd ones back, to
      // the level's new value or (first solve of a refined path) to x1, kept in FP32
      if (pl->prec == PREC_F64) {
        E.Q = pl->Q64;
        E.A = k == 0 ? L.b64 : L.x64;
        E.C = k == 0 ? L.x64 : nullptr;
      } else {
        E.Q = pl->prec == PREC_F32 ? (const void*)pl->Q32 : (const void*)pl->Qbf;
        E.A = k % 2 == 0 ? L.lo0 : L.lo1;
        E.C = k % 2 == 0 ? (void*)L.lo1 : k == 1 ? (void*)L.x64 : nullptr;
        E.paired = k % 2 == 0 && split_operands(pl->prec, n);
        if (k == 3) E.add = (const float*)L.x64;   // x = x1 + S~(rho)
      }
    }
  }
  RIDC_HIP_TRY(hipMemcpy(pl->d_passes, pl->passes.data(), sizeof(Pass2D) * pl->passes.size(),
                         hipMemcpyHostToDevice));
  {
    // the pass shape recorded for this (n, precision), if the tuning table has one
    int tile = 0;
    if (!tune_get_2d(p->n, p->prec, &tile) || plan2d_set_tile(pl, tile) != RIDC_OK)
      pl->tile = plan2d_default_tile(pl);
    set_error("");
  }
  *out = pl;
  return RIDC_OK;
}

void plan2d_destroy(Plan2D* pl) { delete pl; }

int plan2d_tile(const Plan2D* pl) { return pl->tile; }

void plan2d_tile_candidates(const Plan2D* pl, std::vector<int>* out) {
  out->clear();
  out->push_back(0);
  if (pl->prec != PREC_BF16 && (!folded(pl->n) || pl->n % 128 == 0)) out->push_back(kPassWide64);
  if (pl->prec == PREC_BF16 && wide_slices<PREC_BF16>(pl->n)) out->push_back(kPassNarrowK);
}

// Narrow k-slices where they are a choice: whole steps at n = 1024, order 4, 144 us against 156.
int plan2d_default_tile(const Plan2D* pl) {
  return pl->prec == PREC_BF16 && wide_slices<PREC_BF16>(pl->n) ? kPassNarrowK : 0;
}

bool plan2d_tile_matters(const Plan2D* pl) {
  const int bt = pl->prec == PREC_F64   ? block_tile<PREC_F64>(pl->n, pl->P)
                 : pl->prec == PREC_F32 ? block_tile<PREC_F32>(pl->n, pl->P)
                                        : block_tile<PREC_BF16>(pl->n, pl->P);
  return bt == BT0;
}

int plan2d_set_tile(Plan2D* pl, int tile) {
  std::vector<int> c;
  plan2d_tile_candidates(pl, &c);
  const int shape = pl->n % 256 == 0 ? tile & ~kPassPlainA : tile;
  if (std::find(c.begin(), c.end(), shape) == c.end())
    return fail(RIDC_E_INVAL, "launch shape not available for this side and precision");
  pl->tile = shape;          // (plans are grouped by it)
  return RIDC_OK;
}

int plan2d_arm(Plan2D* pl, int64_t nt, hipStream_t stream) {
  for (auto& L : pl->levels) {
    L.nt = nt;
    L.sigma0 = 0;
  }
  RIDC_HIP_TRY(hipMemcpyAsync(pl->d_levels, pl->levels.data(), sizeof(Lvl2D) * pl->levels.size(),
                              hipMemcpyHostToDevice, stream));
  return RIDC_OK;
}

namespace {

// One solve (passes d[0], d[cnt]): to sine coefficients along the rows, line solves down the
// columns, and back; the last pass writes LAST.
template <int PREC, int LAST>
void run_solve(const Lvl2D* lv, const Pass2D* d, int cnt, int64_t n, int64_t s, int tile,
               hipStream_t st) {
  constexpr int OWN = PREC == PREC_F64 ? OUT_F64 : OUT_F32;
  typedef typename std::conditional<PREC == PREC_F64, double, float>::type T;
  launch_pass<PREC, OWN>(d, lv, cnt, n, s, tile, st);
  if constexpr (PREC == PREC_BF16)
    split_operands(PREC, n) ? launch_lines<T, true>(lv, cnt, n, s, st)
                            : launch_lines<T, false>(lv, cnt, n, s, st);
  else
    launch_lines<T, false>(lv, cnt, n, s, st);
  launch_pass<PREC, LAST>(d + cnt, lv, cnt, n, s, tile, st);
}

// Every stage of one pipeline step for `cnt` (plan, level) entries of one precision: the
// right-hand side, the solve and (reduced precision) the residual and a second solve.
// passes is pass-major: passes[k * cnt + e].
void run_stages(int prec, const Lvl2D* lv, const Pass2D* d, int cnt, int64_t n, int64_t s,
                int tile, hipStream_t st) {
  launch_rhs(lv, cnt, n, s, split_operands(prec, n), st);
  if (prec == PREC_F64) {
    run_solve<PREC_F64, OUT_FINAL>(lv, d, cnt, n, s, tile, st);
  } else if (prec == PREC_F32) {
    run_solve<PREC_F32, OUT_F32>(lv, d, cnt, n, s, tile, st);
    launch_resid(lv, cnt, n, s, false, st);
    run_solve<PREC_F32, OUT_FINAL>(lv, d + 2 * cnt, cnt, n, s, tile, st);
  } else {
    run_solve<PREC_BF16, OUT_F32>(lv, d, cnt, n, s, tile, st);
    launch_resid(lv, cnt, n, s, split_operands(prec, n), st);
    run_solve<PREC_BF16, OUT_FINAL>(lv, d + 2 * cnt, cnt, n, s, tile, st);
  }
}

// Launch tables of grouped plans (one set per calling thread and device).  `done` follows the
// upload of the pinned staging copy (the host waits for it before rewriting the staging);
// `used` follows the last launch that read the device tables, and an upload on another stream
// waits for it on the device, so the tables are never rewritten under a running kernel.
struct Arena2D {
  int device = -1;
  Lvl2D* d_lv = nullptr;
  Pass2D* d_ps = nullptr;
  Lvl2D* h_lv = nullptr;
  Pass2D* h_ps = nullptr;
  size_t cap_lv = 0, cap_ps = 0;
  hipEvent_t done = nullptr;
  bool pending = false;
  hipEvent_t used = nullptr;
  hipStream_t used_stream = nullptr;
  bool in_use = false;
};
thread_local Arena2D g_a2;

int arena2d_reserve(size_t nlv, size_t nps, hipStream_t stream) {
  int dev = 0;
  RIDC_HIP_TRY(hipGetDevice(&dev));
  if (g_a2.device != dev) {
    g_a2 = Arena2D{};
    g_a2.device = dev;
  }
  if (!g_a2.done) RIDC_HIP_TRY(hipEventCreateWithFlags(&g_a2.done, hipEventDisableTiming));
  if (!g_a2.used) RIDC_HIP_TRY(hipEventCreateWithFlags(&g_a2.used, hipEventDisableTiming));
  if (g_a2.pending) {
    RIDC_HIP_TRY(hipEventSynchronize(g_a2.done));
    g_a2.pending = false;
  }
  if (g_a2.in_use && g_a2.used_stream != stream)
    RIDC_HIP_TRY(hipStreamWaitEvent(stream, g_a2.used, 0));
  if (g_a2.in_use && (nlv > g_a2.cap_lv || nps > g_a2.cap_ps)) {
    RIDC_HIP_TRY(hipEventSynchronize(g_a2.used));   // a table is about to be freed
    g_a2.in_use = false;
  }
  if (nlv > g_a2.cap_lv) {
    if (g_a2.d_lv) (void)hipFree(g_a2.d_lv);
    if (g_a2.h_lv) (void)hipHostFree(g_a2.h_lv);
    g_a2.d_lv = nullptr;
    g_a2.h_lv = nullptr;
    const size_t cap = std::max(nlv, 2 * g_a2.cap_lv);
    if (hipMalloc(&g_a2.d_lv, cap * sizeof(Lvl2D)) != hipSuccess) return fail(RIDC_E_NOMEM, "2D level table");
    if (hipHostMalloc(&g_a2.h_lv, cap * sizeof(Lvl2D), hipHostMallocDefault) != hipSuccess)
      return fail(RIDC_E_NOMEM, "2D level staging");
    g_a2.cap_lv = cap;
  }
  if (nps > g_a2.cap_ps) {
    if (g_a2.d_ps) (void)hipFree(g_a2.d_ps);
    if (g_a2.h_ps) (void)hipHostFree(g_a2.h_ps);
    g_a2.d_ps = nullptr;
    g_a2.h_ps = nullptr;
    const size_t cap = std::max(nps, 2 * g_a2.cap_ps);
    if (hipMalloc(&g_a2.d_ps, cap * sizeof(Pass2D)) != hipSuccess) return fail(RIDC_E_NOMEM, "2D pass table");
    if (hipHostMalloc(&g_a2.h_ps, cap * sizeof(Pass2D), hipHostMallocDefault) != hipSuccess)
      return fail(RIDC_E_NOMEM, "2D pass staging");
    g_a2.cap_ps = cap;
  }
  return RIDC_OK;
}

// Side streams that run groups beside the caller's stream: three of the calling thread's own for the
// device it used last.  The caller's stream waits for them before a call returns, so to the caller
// everything stays in its stream's order.  A thread that ends (or goes to another device) may leave
// work on them that has not run yet, so they are not destroyed then but kept for the next thread, whose
// work queues up behind; of more than kSpare idle sets one is drained and given back.
struct SideStreams {
  static constexpr int N = 3;
  int device = -1;
  hipStream_t s[N] = {};
  hipEvent_t fork = nullptr, join[N] = {};
  void destroy() {
    for (auto& x : s)
      if (x) {
        (void)hipStreamSynchronize(x);
        (void)hipStreamDestroy(x);
      }
    for (auto& x : join)
      if (x) (void)hipEventDestroy(x);
    if (fork) (void)hipEventDestroy(fork);
    *this = SideStreams{};
  }
  bool create(int dev) {
    bool ok = hipEventCreateWithFlags(&fork, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; i < N && ok; ++i)
      ok = hipStreamCreateWithFlags(&s[i], hipStreamNonBlocking) == hipSuccess &&
           hipEventCreateWithFlags(&join[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();
      destroy();
      return false;
    }
    device = dev;
    return true;
  }
};
struct SpareStreams {
  static constexpr size_t kSpare = 8;
  std::mutex mu;
  std::vector<SideStreams> sets;
  bool take(int dev, SideStreams* out) {
    std::lock_guard<std::mutex> lk(mu);
    for (size_t i = 0; i < sets.size(); ++i)
      if (sets[i].device == dev) {
        *out = sets[i];
        sets.erase(sets.begin() + i);
        return true;
      }
    return false;
  }
  void give(SideStreams* in) {
    if (in->device < 0) return;
    SideStreams old;
    {
      std::lock_guard<std::mutex> lk(mu);
      if (sets.size() >= kSpare) {
        old = sets.front();
        sets.erase(sets.begin());
      }
      sets.push_back(*in);
    }
    *in = SideStreams{};
    old.destroy();
  }
};
SpareStreams& spare_streams() {
  static auto* p = new SpareStreams();   // outlives the threads that end at exit
  return *p;
}
struct SideStreamsOwner {
  SideStreams v;
  ~SideStreamsOwner() { spare_streams().give(&v); }
  // the streams of the current device; false when they cannot be had
  bool reserve() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (v.device == dev) return true;
    spare_streams().give(&v);
    return spare_streams().take(dev, &v) || v.create(dev);
  }
};
thread_local SideStreamsOwner g_side;

}  // namespace

// Advance plans by `steps` pipeline steps.  A single plan uses its own tables.  Several plans
// are grouped by (precision, n): each group runs every stage of a step as one launch with one
// grid z-slice per (plan, level), with the same tile shapes as a single plan, so a plan's bits
// do not depend on its company.  Plan i's own step during launch step s is sigma_before[i] + s.
// Groups do not depend on each other: the largest keeps the caller's stream and the others run beside
// it (except under capture), so that the short launches of small grids, which leave most of the chip
// idle, fill the gaps of the large ones'.
int plan2d_advance(Plan2D* const* pls, int count, const int64_t* sigma_before, int64_t steps,
                   hipStream_t stream) {
  if (count <= 0 || steps <= 0) return RIDC_OK;
  if (count == 1) {
    Plan2D* pl = pls[0];
    for (int64_t s = 1; s <= steps; ++s)
      run_stages(pl->prec, pl->d_levels, pl->d_passes, pl->P, pl->n, sigma_before[0] + s, pl->tile,
                 stream);
    RIDC_HIP_TRY(hipGetLastError());
    return RIDC_OK;
  }
  // groups keyed by (prec, n, launch shape), in first-seen order
  std::vector<std::pair<std::pair<int, int64_t>, std::vector<int>>> groups;
  size_t nlv = 0, nps = 0;
  for (int i = 0; i < count; ++i) {
    const auto key = std::make_pair(pls[i]->prec | (pls[i]->tile << 8), pls[i]->n);
    auto it = std::find_if(groups.begin(), groups.end(), [&](auto& g) { return g.first == key; });
    if (it == groups.end()) {
      groups.push_back({key, {}});
      it = groups.end() - 1;
    }
    it->second.push_back(i);
    nlv += pls[i]->P;
    nps += (size_t)pls[i]->P * pls[i]->npass;
  }
  int rc = arena2d_reserve(nlv, nps, stream);
  if (rc != RIDC_OK) return rc;
  struct G {
    int prec, cnt;
    int64_t n;
    size_t lv_off, ps_off;
    int tile;
  };
  std::vector<G> gs;
  size_t lo = 0, po = 0;
  for (auto& g : groups) {
    const int prec = g.first.first & 0xff;
    const int npass = passes_of(prec);
    int cnt = 0;
    for (int i : g.second) cnt += pls[i]->P;
    G gg{prec, cnt, g.first.second, lo, po, g.first.first >> 8};
    int e = 0;
    for (int i : g.second) {
      Plan2D* pl = pls[i];
      for (int j = 0; j < pl->P; ++j) {
        Lvl2D L = pl->levels[j];
        L.sigma0 = -sigma_before[i];
        g_a2.h_lv[lo + e + j] = L;
        for (int k = 0; k < npass; ++k) {
          g_a2.h_ps[po + (size_t)k * cnt + e + j] = pl->passes[k * pl->P + j];
        }
      }
      e += pl->P;
    }
    lo += cnt;
    po += (size_t)cnt * npass;
    gs.push_back(gg);
  }
  RIDC_HIP_TRY(hipMemcpyAsync(g_a2.d_lv, g_a2.h_lv, lo * sizeof(Lvl2D), hipMemcpyHostToDevice, stream));
  RIDC_HIP_TRY(hipMemcpyAsync(g_a2.d_ps, g_a2.h_ps, po * sizeof(Pass2D), hipMemcpyHostToDevice, stream));
  RIDC_HIP_TRY(hipEventRecord(g_a2.done, stream));
  g_a2.pending = true;
  // lanes: 0 the caller's stream, then the side streams
  hipStream_t lane[1 + SideStreams::N] = {stream};
  int nl = 1;
  if (gs.size() > 1) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(stream, &cap) == hipSuccess;
    if (!known) (void)hipGetLastError();
    if (known && cap == hipStreamCaptureStatusNone && g_side.reserve()) {
      nl = (int)std::min<size_t>(gs.size(), 1 + SideStreams::N);
      RIDC_HIP_TRY(hipEventRecord(g_side.v.fork, stream));
      for (int i = 1; i < nl; ++i) {
        lane[i] = g_side.v.s[i - 1];
        RIDC_HIP_TRY(hipStreamWaitEvent(lane[i], g_side.v.fork, 0));
      }
    }
  }
  std::stable_sort(gs.begin(), gs.end(), [](const G& a, const G& b) {
    return a.n * a.n * a.n * a.cnt > b.n * b.n * b.n * b.cnt;
  });
  for (int64_t s = 1; s <= steps; ++s)
    for (size_t k = 0; k < gs.size(); ++k) {
      const G& g = gs[k];
      run_stages(g.prec, g_a2.d_lv + g.lv_off, g_a2.d_ps + g.ps_off, g.cnt, g.n, s, g.tile,
                 lane[k % nl]);
    }
  const hipError_t launched = hipGetLastError();
  for (int i = 1; i < nl; ++i) {
    RIDC_HIP_TRY(hipEventRecord(g_side.v.join[i - 1], lane[i]));
    RIDC_HIP_TRY(hipStreamWaitEvent(stream, g_side.v.join[i - 1], 0));
  }
  RIDC_HIP_TRY(launched);
  RIDC_HIP_TRY(hipEventRecord(g_a2.used, stream));
  g_a2.used_stream = stream;
  g_a2.in_use = true;
  return RIDC_OK;
}

int plan2d_time_pass(Plan2D* pl, int64_t sigma, int reps, hipStream_t stream, double* us) {
  const int P = pl->P;
  const int64_t n = pl->n;
  const int tile = pl->tile;
  // the right-hand side of this step, then `reps` back-to-back launches of its first pass, which
  // rewrite the sine coefficients only
  launch_rhs(pl->d_levels, P, n, sigma, split_operands(pl->prec, n), stream);
  auto pass = [&] {
    if (pl->prec == PREC_F64)
      launch_pass<PREC_F64, OUT_F64>(pl->d_passes, pl->d_levels, P, n, sigma, tile, stream);
    else if (pl->prec == PREC_F32)
      launch_pass<PREC_F32, OUT_F32>(pl->d_passes, pl->d_levels, P, n, sigma, tile, stream);
    else
      launch_pass<PREC_BF16, OUT_F32>(pl->d_passes, pl->d_levels, P, n, sigma, tile, stream);
  };
  hipEvent_t a, b;
  RIDC_HIP_TRY(hipEventCreate(&a));
  RIDC_HIP_TRY(hipEventCreate(&b));
  pass();
  (void)hipEventRecord(a, stream);
  for (int r = 0; r < reps; ++r) pass();
  (void)hipEventRecord(b, stream);
  hipError_t e = hipEventSynchronize(b);
  float ms = 0;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (e != hipSuccess) return fail(RIDC_E_HIP, std::string("pass timing: ") + hipGetErrorString(e));
  *us = 1e3 * (double)ms / reps;
  return RIDC_OK;
}

int plan2d_time_rhs(Plan2D* pl, int64_t sigma, int reps, hipStream_t stream, double* us,
                    double* bytes) {
  const int P = pl->P;
  const int64_t n = pl->n;
  // the right-hand side of this step, launched repeatedly (it rewrites the same values)
  launch_rhs(pl->d_levels, P, n, sigma, split_operands(pl->prec, n), stream);
  hipEvent_t a, b;
  RIDC_HIP_TRY(hipEventCreate(&a));
  RIDC_HIP_TRY(hipEventCreate(&b));
  (void)hipEventRecord(a, stream);
  for (int r = 0; r < reps; ++r)
    launch_rhs(pl->d_levels, P, n, sigma, split_operands(pl->prec, n), stream);
  (void)hipEventRecord(b, stream);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipEventSynchronize(b);
  float ms = 0;
  if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (e != hipSuccess) return fail(RIDC_E_HIP, std::string("rhs timing: ") + hipGetErrorString(e));
  *us = 1e3 * (double)ms / reps;
  // algorithmic bytes per point: level 0 reads its value (a 5-point stencil of one vector),
  // level j > 0 its value and j+1 window vectors; every level writes the FP64 right-hand side
  // and, in the mixed paths, its 4-byte low-precision copy
  const double lo = pl->prec == PREC_F64 ? 0.0 : 4.0;
  double per = 0.0;
  for (int j = 0; j < P; ++j) per += 8.0 * (j == 0 ? 1 : j + 2) + 8.0 + lo;
  *bytes = per * (double)n * (double)n;
  return RIDC_OK;
}

void plan2d_cost(const Plan2D* pl, double* bytes, double* flops) {
  const double n = (double)pl->n;
  // algorithmic flops of the transforms at steady state: P level solves of 2 (or 4) n^3 GEMMs
  *flops = 2.0 * n * n * n * passes_of(pl->prec) * pl->P;
  (void)bytes;
}

}  // namespace ridc
