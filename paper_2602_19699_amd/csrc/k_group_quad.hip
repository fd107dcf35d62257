// Workgroup-per-instance iLQR for the 37-state synthetic quadruped
// (q in R^19, v in R^18, u in R^12; paper Sec. II eq. 1 and Sec. IV).
//
// One 256-thread workgroup owns one instance.  The backward Riccati sweep
// keeps P, [f_x | f_u], P [f_x | f_u], the gains and Q_ux in LDS and forms the
// products as 16 x 16 output tiles on the matrix cores (FP32 MFMA for the
// mixed form, FP64 MFMA for the plain one), the tiles spread over the four
// waves (see backward); Q_uu is factored in FP64 (one wave, rows held by
// lanes) in both precisions.  The dynamics step needs a Cholesky of the 18 x
// 18 mass matrix M(q) = A^T A + diag(1 + 0.1 sin q); a wave does it with its
// lanes holding the rows.  The dynamics Jacobians do not depend on P, so the
// sweep evaluates them ahead of the recursion, CH steps at a time with every
// wave taking its own steps, into per-slot blocks in HBM that the recursion
// then reads back.  Line-search trials run one per wave: in round r wave w
// tries alpha_j with j = 4 r + w, and the first accepted j is taken, as in the
// sequential rule.  Trajectories and gains use the same step-major workspace
// as the lane schedule.
#include "lane_launch.hpp"

namespace cbic {
namespace quad {

constexpr int NQ = 19, NV = 18, N = 37, M = 12;
constexpr int LD = 40;   // length of a state vector in LDS
constexpr int NT = 256;  // threads per workgroup
constexpr int NW = NT / 64;
// A matrix operand of a product with inner size 37 is kept row by row with the
// inner index k at kpos(k), the indices that one lane group of the matrix
// instruction takes (k = lk, lk + 4, ...) side by side, so that a lane reads
// its ten values of a row in three (FP64: five) wide loads; places past 36
// that are read hold zeros.  kq: the same for inner size 12.
constexpr int KG = 12, KROW = 4 * KG;  // places per lane group and row
__host__ __device__ constexpr int kpos(int k) { return (k & 3) * KG + (k >> 2); }
__host__ __device__ constexpr int kq(int t) { return (t & 3) * 4 + (t >> 2); }
// row strides in LDS: sixteen rows read by 16-byte pieces start on sixteen
// different groups of banks
template <class R> struct Stride { static constexpr int k = 52; };
template <> struct Stride<double> { static constexpr int k = 50; };
constexpr int SQ = 20;
constexpr int BROW = 48;                // first LDS row of f_u^T behind f_x^T's three 16-row blocks
constexpr int DB = (N + M) * KROW;      // derivative block: the 49 columns of [f_x | f_u] as operand rows
// steps per chunk of precomputed derivative blocks, a multiple of the four
// waves; 8, 12, 16 and 24 measured within 2 % of each other at every batch size,
// and the chunk is what a slot's workspace holds beyond its trajectories
constexpr int CH = 12;

// device block: [dt, w_u, w_T, w_q, w_v, M0 = A^T A (18x18), W1, W2, e(18), x_nom(37)]
constexpr int O_DT = 0, O_WU = 1, O_WT = 2, O_WQ = 3, O_WV = 4, O_M0 = 5, O_W1 = O_M0 + 324,
              O_W2 = O_W1 + 324, O_E = O_W2 + 324, O_XN = O_E + 18, NPRM = O_XN + 37;

constexpr int LR = 20;  // row stride of 18-wide LDS matrices: whole 16-byte pieces
template <class R>
struct WaveScratch {
  alignas(16) R L[NV][LR];  // Cholesky factor of M(q), lower, row-major, zero above
  alignas(16) R Li[LR];     // reciprocals of its diagonal
  alignas(16) R s[LR], c[LR];  // sin, cos of q[0:18]
  R x[LD];                  // state of this wave's rollout
  R xn[LD];                 // next state
  R u[16];                  // control
  R dx[LD];
  R a[NV];                  // acceleration M^-1 (S u - b)
  R w2c[NV];                // W2 cos q
};

template <class R>
struct Smem {
  using real = R;
  alignas(16) R M0[NV][LR];
  alignas(16) R W1[NV][LR];
  alignas(16) R W2[NV][LR];
  R e[NV];
  R xnom[LD];
  alignas(16) R P[48][Stride<R>::k];       // value Hessian (operand rows; symmetric), row 37: its gradient p
  alignas(16) R AT[2][64][Stride<R>::k];   // [f_x | f_u]^T of this and the next step: rows 0..36 and BROW..BROW+11
  alignas(16) R PAT[64][Stride<R>::k];     // (P [f_x | f_u])^T, the same rows; scratch of the update
  alignas(16) R QuxT[48][SQ], KT[48][SQ];  // Q_ux^T and the feedback gain's transpose (places kq)
  alignas(16) R Lr[M][16];                 // factor of Q_uu in R
  alignas(16) R Lri[M];                    // reciprocals of its diagonal
  R Qg[N + M];                             // f_x^T p, f_u^T p
  R xs[2][LD], us[2][16];                  // state and control of this and the next step
  alignas(16) R Qu[16], kk[16];
  double Quu[M][M + 1];
  // the bounded step's face factor
  double Lq[M][M + 1], Lqi[M], Li[M];
  double wJ[NW];
  int wok[NW];
  int flag;     // Q_uu did not factor (then the bounded step's state)
  int nonfin;   // the gains are not finite
  unsigned Hq_held;  // components held at a bound by the bounded step
  WaveScratch<R> wv[NW];
};

// Shared memory of the kernels that need only the constants, one vector and
// the scratch of NWV waves (the initial rollout, the finalize): small enough
// for every instance of a CU's share of the batch to be resident at once
template <class R, int NWV>
struct WaveSmem {
  using real = R;
  alignas(16) R M0[NV][LR];
  alignas(16) R W1[NV][LR];
  alignas(16) R W2[NV][LR];
  R e[NV];
  R xnom[LD];
  R p[LD];  // the finalize's costate
  WaveScratch<R> wv[NWV];
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v, opaque to the compiler: what is derived from it (addresses, lane masks) is
// formed where it is used.  Derived from the lane number itself, they are
// invariant over the whole solve, and the compiler keeps hundreds of them
// through it, in scratch memory (145 registers of the mixed kernel for two
// instances per CU, 173 of the FP64 one): a quarter more time for 1024 mixed
// instances, a fifth more for 100 in FP64.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// c ? a : b with both values formed first: left to itself the compiler turns
// a chain of lane selects into branches around the arithmetic of each
template <class R>
__device__ __forceinline__ R pick(bool c, R a, R b) {
  asm("" : "+v"(a), "+v"(b));
  return c ? a : b;
}

// value of v in lane j (j uniform), read through a scalar register
__device__ __forceinline__ float bcast(float v, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
// 1/sqrt(d) from the hardware estimate and Newton steps y <- y (3 - d y^2) / 2,
// each squaring the relative error: two in FP64, one in FP32 (the pivots of
// the Cholesky factors below are then d * (1/sqrt(d)), without a division)
__device__ __forceinline__ double rsqrt_nr(double d) {
  double y = __builtin_amdgcn_rsq(d);
  y = y * (1.5 - 0.5 * d * y * y);
  return y * (1.5 - 0.5 * d * y * y);
}
__device__ __forceinline__ float rsqrt_nr(float d) {
  const float y = __builtin_amdgcn_rsqf(d);
  return y * (1.5f - 0.5f * d * y * y);
}

__device__ __forceinline__ double bcast(double v, int j) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, j);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), j);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The value of the lane whose number differs in bit `O`, given that the lanes
// that differ in higher bits hold the same value already (a sum over the wave
// from the highest bit down): register swaps between half waves and rows, then
// rotations within a row (rotating by 4 reaches lane ^ 4 or its copy at ^ 8).
template <int O>
__device__ __forceinline__ int lane_other(int v, int lane) {
  if constexpr (O == 32) {
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return lane & 32 ? p[0] : p[1];
  } else if constexpr (O == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return lane & 16 ? p[0] : p[1];
  } else {
    constexpr int ctrl = O == 8 ? 0x128 : (O == 4 ? 0x124 : (O == 2 ? 0x4E : 0xB1));
    return __builtin_amdgcn_mov_dpp(v, ctrl, 0xF, 0xF, true);
  }
}
template <int O>
__device__ __forceinline__ float lane_other(float v, int lane) {
  return __int_as_float(lane_other<O>(__float_as_int(v), lane));
}
template <int O>
__device__ __forceinline__ double lane_other(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = unsigned(lane_other<O>(int(b), lane)), hi = unsigned(lane_other<O>(int(b >> 32), lane));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <class R>
__device__ __forceinline__ R wave_sum(R v, int lane) {
  v += lane_other<32>(v, lane);
  v += lane_other<16>(v, lane);
  v += lane_other<8>(v, lane);
  v += lane_other<4>(v, lane);
  v += lane_other<2>(v, lane);
  v += lane_other<1>(v, lane);
  return v;
}

// ------------------------------------------------------------------ constants
template <class S>
__device__ __forceinline__ void stage_constants(S& sm, const double* __restrict__ prm, int tid, int nt = NT) {
  using R = typename S::real;
  for (int i = tid; i < NV * NV; i += nt) {
    const int r = i / NV, c = i % NV;
    sm.M0[r][c] = R(prm[O_M0 + i]);
    sm.W1[r][c] = R(prm[O_W1 + i]);
    sm.W2[r][c] = R(prm[O_W2 + i]);
  }
  if (tid < NV) sm.e[tid] = R(prm[O_E + tid]);
  if (tid < N) sm.xnom[tid] = R(prm[O_XN + tid]);
}

// ------------------------------------------------------------------ wave-level dynamics
// an 18-wide row (or vector) in LDS, by 16-byte pieces
template <class R>
__device__ __forceinline__ void ld_row(R (&v)[NV], const R* p) {
  struct alignas(16) Piece { R v[16 / sizeof(R)]; };
  constexpr int E = 16 / int(sizeof(R));
#pragma unroll
  for (int i = 0; i < NV; i += E) {
    const Piece q = *reinterpret_cast<const Piece*>(p + i);
#pragma unroll
    for (int j = 0; j < E; ++j)
      if (i + j < NV) v[i + j] = q.v[j];
  }
}
template <class R>
__device__ __forceinline__ void st_row(R* p, const R (&v)[NV]) {
  struct alignas(16) Piece { R v[16 / sizeof(R)]; };
  constexpr int E = 16 / int(sizeof(R));
#pragma unroll
  for (int i = 0; i < NV; i += E) {
    Piece q;
#pragma unroll
    for (int j = 0; j < E; ++j) q.v[j] = i + j < NV ? v[i + j < NV ? i + j : 0] : R(0);
    *reinterpret_cast<Piece*>(p + i) = q;
  }
}
// one step of the forward (lanes past j) and backward (lanes before j)
// substitution, entry j of the right-hand side in lane j: without branches,
// which the chain of eighteen would wait on one by one
template <class R>
__device__ __forceinline__ R forward_step(R y, R l, R inv, int j, int lane) {
  const R yj = bcast(y, j) * inv;
  return pick(lane == j, yj, pick(lane > j, y - l * yj, y));
}
template <class R>
__device__ __forceinline__ R backward_step(R y, R l, R inv, int j, int lane) {
  const R zj = bcast(y, j) * inv;
  return pick(lane == j, zj, pick(lane < j, y - l * zj, y));
}

// One semi-implicit Euler step for wave scratch ws: reads ws.x and ws.u,
// writes ws.xn; leaves L (factor of M), a, sin/cos and W2 cos q in ws.  A
// serial chain (eighteen pivots, eighteen entries of the back substitution;
// the forward one runs along with the factor); everything a lane needs of LDS
// is loaded in wide pieces ahead of the chains.  A step of a line-search trial
// takes 9.3 thousand cycles alone on its SIMD (17.9 with a branch per entry,
// single loads inside the chains and shuffle sums); solve of 1024 mixed
// instances 2.3 ms shorter, of 100 in FP64 2.1 ms (of 8.8 and 9.3 ms).
template <class R, class S>
__device__ __forceinline__ void wave_dyn(const S& sm, WaveScratch<R>& ws, R dt, int lane_) {
  const int lane = fresh(lane_);
  const bool row = lane < NV;
  const int ri = row ? lane : 0;
  R m[NV], w1[NV], w2[NV];
  ld_row(m, sm.M0[ri]);
  ld_row(w1, sm.W1[ri]);
  ld_row(w2, sm.W2[ri]);
  const R xq = ws.x[ri], xv = ws.x[NQ + ri], er = sm.e[ri], x18 = ws.x[NV];
  const R ua = ws.u[ri >= 6 ? ri - 6 : 0];
  R sn = R(0);
  if (row) {
    R cs;
    dsincos_lib(xq, &sn, &cs);
    ws.s[lane] = sn;
    ws.c[lane] = cs;
  }
  wave_sync();
  // bias forces and right-hand side r = S u - b
  R y = R(0);
  {
    R sv[NV], cv[NV], b1 = R(0), b2 = R(0);
    ld_row(sv, ws.s);
    ld_row(cv, ws.c);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      b1 += w1[j] * sv[j];
      b2 += w2[j] * cv[j];
    }
    const R b = b1 + b2 * xv;
    if (row) {
      ws.w2c[ri] = b2;
      y = (ri >= 6 ? ua : R(0)) - b;
    }
  }
  // M = A^T A + diag(1 + 0.1 sin q); Cholesky with the rows on lanes, the
  // pivot column broadcast from its lane, and L z = r along with it
  {
    const R d = R(1) + R(0.1) * sn;
#pragma unroll
    for (int j = 0; j < NV; ++j) m[j] = pick(j == lane, m[j] + d, m[j]);
  }
  R inv[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const R piv = bcast(m[j], j);
    inv[j] = rsqrt_nr(piv);
    const R ljj = piv * inv[j];
    const R lij = pick(lane == j, ljj, pick(lane > j && row, m[j] * inv[j], R(0)));
    m[j] = lij;
#pragma unroll
    for (int k = j + 1; k < NV; ++k) m[k] -= lij * bcast(lij, k);
    y = forward_step(y, lij, inv[j], j, lane);
  }
  if (row) st_row(ws.L[ri], m);
  if (lane == 0) st_row(ws.Li, inv);
  wave_sync();
  // L^T a = z
#pragma unroll
  for (int j = 0; j < NV; ++j) m[j] = ws.L[j][ri];
#pragma unroll
  for (int j = NV - 1; j >= 0; --j) y = backward_step(y, m[j], inv[j], j, lane);
  const R vn = xv + dt * y;
  const R ev = wave_sum(row ? er * vn : R(0), lane);
  if (row) {
    ws.a[ri] = y;
    ws.xn[NQ + ri] = vn;
    ws.xn[ri] = xq + dt * vn;
  }
  if (lane == 0) ws.xn[NV] = x18 + dt * ev;
  wave_sync();
}

// running cost l(x, u) of the wave's (x, u); the same value in every lane
template <class R, class S>
__device__ __forceinline__ R wave_cost(const S& sm, const R* x, const R* u, const double* __restrict__ prm, int lane,
                       bool terminal) {
  R v = R(0);
  if (lane < N) {
    const R d = x[lane] - sm.xnom[lane];
    v = (lane < NQ ? R(prm[O_WQ]) : R(prm[O_WV])) * d * d;
    if (terminal) v *= R(prm[O_WT]);
  } else if (!terminal && lane < N + M) {
    const R uu = u[lane - N];
    v = R(prm[O_WU]) * uu * uu;
  }
  return wave_sum(v, lane);
}

// ------------------------------------------------------------------ MFMA tiles
// A 16 x 16 output tile C += A B by one wave with 16x16x4 matrix-core
// instructions: FP32 for the mixed form, FP64 for the plain one.  Lane l
// supplies A(i0 + l % 16, k0 + l / 16) and B(k0 + l / 16, j0 + l % 16) per step
// of 4; its result register r holds C(i0 + 4 (l / 16) + r, j0 + l % 16) in FP32
// and C(i0 + l / 16 + 4 r, j0 + l % 16) in FP64.  With the operands swapped a
// lane gets the transposed product's entries, the same sums of the same
// products.
typedef float mf_f4 __attribute__((ext_vector_type(4)));
typedef double mf_d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ mf_f4 mfma16(float a, float b, mf_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ mf_d4 mfma16(double a, double b, mf_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <class R> struct MfAcc;
template <> struct MfAcc<float> {
  using type = mf_f4;
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};
template <> struct MfAcc<double> {
  using type = mf_d4;
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
};

// a lane's ten values of an operand row of inner size 37 (p: the row at its
// lane group's place)
template <class R>
__device__ __forceinline__ void ld_op(R (&v)[10], const R* p) {
  if constexpr (sizeof(R) == 4) {
    const mf_f4 a = *reinterpret_cast<const mf_f4*>(p), b = *reinterpret_cast<const mf_f4*>(p + 4);
    const float2 c = *reinterpret_cast<const float2*>(p + 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = a[i];
      v[4 + i] = b[i];
    }
    v[8] = c.x;
    v[9] = c.y;
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const double2 a = *reinterpret_cast<const double2*>(p + 2 * i);
      v[2 * i] = a.x;
      v[2 * i + 1] = a.y;
    }
  }
}
// a row of twelve, by 16-byte pieces
template <class R>
__device__ __forceinline__ void ld12(R (&v)[M], const R* p) {
  struct alignas(16) Piece { R v[16 / sizeof(R)]; };
  constexpr int E = 16 / int(sizeof(R));
#pragma unroll
  for (int i = 0; i < M; i += E) {
    const Piece q = *reinterpret_cast<const Piece*>(p + i);
#pragma unroll
    for (int j = 0; j < E; ++j) v[i + j] = q.v[j];
  }
}
// its three values of an operand row of inner size 12
template <class R>
__device__ __forceinline__ void ld_op12(R (&v)[3], const R* p) {
  if constexpr (sizeof(R) == 4) {
    const mf_f4 a = *reinterpret_cast<const mf_f4*>(p);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = a[i];
  } else {
    const double2 a = *reinterpret_cast<const double2*>(p);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = p[2];
  }
}

// ------------------------------------------------------------------ wave Jacobians
// [f_x | f_u] at (ws.x, ws.u) by one wave, after wave_dyn on that point (L, its
// reciprocal diagonal, a, sin/cos and W2 cos q in ws), written to dst column by
// column as operand rows (kpos order, KROW places each).  Lane c < 48 owns
// column c of the right-hand sides (0..17 -dD/dq with a and v held, 18..35
// -dD/dv, 36..47 the actuation S), solves it with M = L L^T in registers and
// writes the output column that depends on it: c for c < 18, c + 1 otherwise.
// Lane 48 writes column 18 (q_18 does not enter the dynamics; only the
// identity).
template <class R>
__device__ __forceinline__ void put_op(R* __restrict__ dst, const R (&v)[N]) {
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int q = 0; q < 10; ++q) dst[g * KG + q] = g + 4 * q < N ? v[g + 4 * q < N ? g + 4 * q : 0] : R(0);
}
template <class R>
__device__ __forceinline__ void wave_jac(const Smem<R>& sm, const WaveScratch<R>& ws, R dt, int lane_,
                                         R* __restrict__ dst) {
  const int lane = fresh(lane_);
  if (lane < 48) {
    const int c = lane, cq = c < NV ? c : 0;
    R y[NV], av[NV], w2c[NV], l[NV][NV], li[NV];
    const R sc = ws.s[cq], cc = ws.c[cq];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      av[i] = ws.a[i];
      w2c[i] = ws.w2c[i];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      R v = -(sm.W1[i][cq] * cc - ws.x[NQ + i] * sm.W2[i][cq] * sc);
      if (i == c) v -= R(0.1) * ws.c[i] * av[i];
      const R vv = (c - NV == i) ? -w2c[i] : R(0);
      const R vu = (c - 2 * NV + 6 == i) ? R(1) : R(0);
      y[i] = c < NV ? v : (c < 2 * NV ? vv : vu);
    }
    ld_row(li, ws.Li);
#pragma unroll
    for (int i = 0; i < NV; ++i) ld_row(l[i], ws.L[i]);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      R v0 = y[i], v1 = R(0);
#pragma unroll
      for (int k = 0; k < i; ++k) {
        if (k & 1) v1 += l[i][k] * y[k];
        else v0 -= l[i][k] * y[k];
      }
      y[i] = (v0 - v1) * li[i];
    }
#pragma unroll
    for (int i = NV - 1; i >= 0; --i) {
      R v0 = y[i], v1 = R(0);
#pragma unroll
      for (int k = i + 1; k < NV; ++k) {
        if (k & 1) v1 += l[k][i] * y[k];
        else v0 -= l[k][i] * y[k];
      }
      y[i] = (v0 - v1) * li[i];
    }
    // d v+_i / d (x, u)_col = [col is the velocity column i] + dt y_i; rows:
    // v+ (19..36), q+ = q + dt v+ (0..17), q_18+ = q_18 + dt e . v+
    const int col = c < NV ? c : c + 1;
    R se = R(0), out[N];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const R d = ((c >= NV && c < 2 * NV && c - NV == i) ? R(1) : R(0)) + dt * y[i];
      se += sm.e[i] * d;
      out[NQ + i] = d;
      out[i] = ((col == i) ? R(1) : R(0)) + dt * d;
    }
    out[NV] = dt * se;
    put_op(dst + col * KROW, out);
  } else if (lane == 48) {
    R out[N];
#pragma unroll
    for (int r = 0; r < N; ++r) out[r] = (r == NV) ? R(1) : R(0);
    put_op(dst + NV * KROW, out);
  }
}

// ------------------------------------------------------------------ FP64 Cholesky of Q_uu and the gains
// Both by one wave.  factor_quu: Q_uu (rows on lanes 0..11; the pivot column
// reaches the other lanes by row broadcasts, which the subtraction reads as an
// operand) to its factor in R (the mixed form's gain solves run in FP32 on the
// FP64 factor rounded to FP32, as in the lane kernels).
//
// row_fnma_past<J>: m[k] -= l l_k (l_k: lane k's l) for the columns k past J,
// in one statement with the wait states that a DPP read of l needs after the
// write of it: in statements of their own the compiler may place a copy or a
// reload of l between the two.
#define CBIC_FNMA(K) "v_fmac_f64_dpp %[m" #K "], -%[l], %[l] row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n\t"
#define CBIC_FNMA_IO(K) [m##K] "+&v"(m[K])
#define CBIC_FNMA_11 CBIC_FNMA(11)
#define CBIC_FNMA_10 CBIC_FNMA(10) CBIC_FNMA_11
#define CBIC_FNMA_9 CBIC_FNMA(9) CBIC_FNMA_10
#define CBIC_FNMA_8 CBIC_FNMA(8) CBIC_FNMA_9
#define CBIC_FNMA_7 CBIC_FNMA(7) CBIC_FNMA_8
#define CBIC_FNMA_6 CBIC_FNMA(6) CBIC_FNMA_7
#define CBIC_FNMA_5 CBIC_FNMA(5) CBIC_FNMA_6
#define CBIC_FNMA_4 CBIC_FNMA(4) CBIC_FNMA_5
#define CBIC_FNMA_3 CBIC_FNMA(3) CBIC_FNMA_4
#define CBIC_FNMA_2 CBIC_FNMA(2) CBIC_FNMA_3
#define CBIC_FNMA_1 CBIC_FNMA(1) CBIC_FNMA_2
#define CBIC_FNMA_IO_11 CBIC_FNMA_IO(11)
#define CBIC_FNMA_IO_10 CBIC_FNMA_IO(10), CBIC_FNMA_IO_11
#define CBIC_FNMA_IO_9 CBIC_FNMA_IO(9), CBIC_FNMA_IO_10
#define CBIC_FNMA_IO_8 CBIC_FNMA_IO(8), CBIC_FNMA_IO_9
#define CBIC_FNMA_IO_7 CBIC_FNMA_IO(7), CBIC_FNMA_IO_8
#define CBIC_FNMA_IO_6 CBIC_FNMA_IO(6), CBIC_FNMA_IO_7
#define CBIC_FNMA_IO_5 CBIC_FNMA_IO(5), CBIC_FNMA_IO_6
#define CBIC_FNMA_IO_4 CBIC_FNMA_IO(4), CBIC_FNMA_IO_5
#define CBIC_FNMA_IO_3 CBIC_FNMA_IO(3), CBIC_FNMA_IO_4
#define CBIC_FNMA_IO_2 CBIC_FNMA_IO(2), CBIC_FNMA_IO_3
#define CBIC_FNMA_IO_1 CBIC_FNMA_IO(1), CBIC_FNMA_IO_2
template <int J>
__device__ __forceinline__ void row_fnma_past(double (&m)[M], double l) {
  static_assert(M == 12, "one statement per column of a 12-wide factor");
  if constexpr (J == 0) asm("s_nop 1\n\t" CBIC_FNMA_1 : CBIC_FNMA_IO_1 : [l] "v"(l));
  if constexpr (J == 1) asm("s_nop 1\n\t" CBIC_FNMA_2 : CBIC_FNMA_IO_2 : [l] "v"(l));
  if constexpr (J == 2) asm("s_nop 1\n\t" CBIC_FNMA_3 : CBIC_FNMA_IO_3 : [l] "v"(l));
  if constexpr (J == 3) asm("s_nop 1\n\t" CBIC_FNMA_4 : CBIC_FNMA_IO_4 : [l] "v"(l));
  if constexpr (J == 4) asm("s_nop 1\n\t" CBIC_FNMA_5 : CBIC_FNMA_IO_5 : [l] "v"(l));
  if constexpr (J == 5) asm("s_nop 1\n\t" CBIC_FNMA_6 : CBIC_FNMA_IO_6 : [l] "v"(l));
  if constexpr (J == 6) asm("s_nop 1\n\t" CBIC_FNMA_7 : CBIC_FNMA_IO_7 : [l] "v"(l));
  if constexpr (J == 7) asm("s_nop 1\n\t" CBIC_FNMA_8 : CBIC_FNMA_IO_8 : [l] "v"(l));
  if constexpr (J == 8) asm("s_nop 1\n\t" CBIC_FNMA_9 : CBIC_FNMA_IO_9 : [l] "v"(l));
  if constexpr (J == 9) asm("s_nop 1\n\t" CBIC_FNMA_10 : CBIC_FNMA_IO_10 : [l] "v"(l));
  if constexpr (J == 10) asm("s_nop 1\n\t" CBIC_FNMA_11 : CBIC_FNMA_IO_11 : [l] "v"(l));
}
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_bit_cast(double, dpp_update_i64(0L, __builtin_bit_cast(long, v), 0x150 + J, 0xF, 0xF, true));
}
template <int J>
__device__ __forceinline__ void factor_col(double (&m)[M], double (&invs)[M], bool& ok, int lane) {
  if constexpr (J < M) {
    const double piv = row_bcast<J>(m[J]);
    ok = ok && (piv > 0.0) && isfinite(piv);
    const double inv = rsqrt_nr(piv);
    const double ljj = piv * inv;
    invs[J] = inv;
    const double lij = pick(lane == J, ljj, pick(lane > J && lane < M, m[J] * inv, 0.0));
    m[J] = lij;
    row_fnma_past<J>(m, lij);
    factor_col<J + 1>(m, invs, ok, lane);
  }
}
template <class R>
__device__ __forceinline__ void factor_quu(Smem<R>& sm, int lane_) {
  const int lane = fresh(lane_);
  const bool row = lane < M;
  const int ri = row ? lane : 0;
  double m[M];
#pragma unroll
  for (int j = 0; j < M; ++j) m[j] = row ? sm.Quu[min(ri, j)][max(ri, j)] : 0.0;
  bool ok = true;
  double invs[M];
  factor_col<0>(m, invs, ok, lane);
  if (row)
#pragma unroll
    for (int j = 0; j < M; ++j) sm.Lr[ri][j] = R(m[j]);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < M; ++j) sm.Lri[j] = R(invs[j]);
    sm.flag = ok ? 0 : 1;
  }
}

// Column `lane` (< 38) of [K | k] from that of [Q_ux | Q_u], in registers;
// a non-finite gain sets nonfin (lanes past 37 repeat the last column).
template <class R>
__device__ __forceinline__ void solve_gains(Smem<R>& sm, int lane) {
  R l[M][M], li[M], qc[M], kc[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    ld12(l[i], sm.Lr[i]);
    qc[i] = lane < N ? sm.QuxT[lane < N ? lane : 0][kq(i)] : sm.Qu[i];
  }
  ld12(li, sm.Lri);
#pragma unroll
  for (int i = 0; i < M; ++i) {
    R v0 = qc[i], v1 = R(0);
#pragma unroll
    for (int k = 0; k < i; ++k) {
      if (k & 1) v1 += l[i][k] * kc[k];
      else v0 -= l[i][k] * kc[k];
    }
    kc[i] = (v0 - v1) * li[i];
  }
#pragma unroll
  for (int i = M - 1; i >= 0; --i) {
    R v0 = kc[i], v1 = R(0);
#pragma unroll
    for (int k = i + 1; k < M; ++k) {
      if (k & 1) v1 += l[k][i] * kc[k];
      else v0 -= l[k][i] * kc[k];
    }
    kc[i] = (v0 - v1) * li[i];
  }
  bool fin = true;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    fin = fin && isfinite(kc[i]);
    kc[i] = -kc[i];
  }
  if (lane < N) {
#pragma unroll
    for (int i = 0; i < M; ++i) sm.KT[lane][kq(i)] = kc[i];
  }
  if (lane == N) {
#pragma unroll
    for (int i = 0; i < M; ++i) sm.kk[i] = kc[i];
  }
  if (!fin) sm.nonfin = 1;
}

// ------------------------------------------------------------------ bounded control step (eq. 1)
// Wave-parallel Cholesky (rows on lanes, the pivot column broadcast from its
// lane) of the face of H with the components in W held: their rows and
// columns become identity.  Lane i < M keeps row i of the factor in f and
// stores it to Lf[i]; the reciprocal pivots go to Li (lane 0 writes).  False
// when a pivot is not positive or not finite.
__device__ __forceinline__ bool face_factor(const double* H, unsigned W, int lane, double (&f)[M],
                                            double (*Lf)[M + 1], double* Li) {
  const bool row = lane < M;
  const int ri = row ? lane : 0;
  const bool hr = (W >> ri) & 1u;
#pragma unroll
  for (int j = 0; j < M; ++j)
    f[j] = !row ? 0.0 : (hr || ((W >> j) & 1u)) ? (ri == j ? 1.0 : 0.0) : H[min(ri, j) * (M + 1) + max(ri, j)];
  bool ok = true;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const double piv = bcast(f[j], j);
    ok = ok && (piv > 0.0) && isfinite(piv);
    const double inv = rsqrt_nr(piv);
    if (lane == 0) Li[j] = inv;
    const double lij = (lane == j) ? piv * inv : (lane > j && row ? f[j] * inv : 0.0);
    f[j] = lij;
#pragma unroll
    for (int k = j + 1; k < M; ++k) f[k] -= lij * bcast(lij, k);
  }
  if (row)
#pragma unroll
    for (int j = 0; j < M; ++j) Lf[ri][j] = f[j];
  wave_sync();
  return ok;
}

// (L L^T) y = b for the factor (rows on lanes in f, all rows in Lf) and its
// reciprocal pivots Li; lane i < M holds b_i on entry and y_i on return.
__device__ __forceinline__ double face_solve(const double (&f)[M], const double (*Lf)[M + 1], const double* Li,
                                             double y, int lane) {
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const double yj = bcast(y, j) * Li[j];
    if (lane == j) y = yj;
    else if (lane > j && lane < M) y -= f[j] * yj;
  }
  const int ri = lane < M ? lane : 0;
#pragma unroll
  for (int j = M - 1; j >= 0; --j) {
    const double zj = bcast(y, j) * Li[j];
    if (lane == j) y = zj;
    else if (lane < j) y -= Lf[j][ri] * zj;
  }
  return y;
}

// The control step under the bound (paper eq. 1) once solve_gains has formed the
// unconstrained gains: when the step k_k lies in the box [-umax - u_k,
// umax - u_k] it stands (so a bound that never binds changes nothing).
// Otherwise wave 0 minimises 0.5 d'Hd + Q_u'd over the box exactly in FP64 by
// the primal active-set method of the lane kernels (box_qp in dev_common.hpp):
// start from the clamped unconstrained minimiser, holding the clamped
// components; move towards the current face's minimiser until a free
// component meets a bound (smallest step, lowest index on ties), or at the
// face's minimiser release the held component with the most negative
// multiplier (lowest index on ties); at most 4 M + 4 steps.  The feedback rows
// of the held components are zero and the free ones come from the final
// face's factor: K = -[face factor]^-1 Q_ux with the held rows of Q_ux zeroed.
// Returns 0 or the status bit that freezes the instance.
template <class R>
__device__ uint32_t box_step(Smem<R>& sm, const R* uk, double umax, int tid) {
  const double* H = &sm.Quu[0][0];
  double* Li = sm.Li;
  if (tid < 64) {
    const int lane = tid;
    const bool row = lane < M;
    const int ri = row ? lane : 0;
    const double u = double(uk[ri]);
    const double lo = -umax - u, hi = umax - u;
    const double kk = double(sm.kk[ri]);
    const bool inside = !row || (kk >= lo && kk <= hi);
    unsigned W = 0, up = 0;
    bool ok = true;
    if (__ballot(!inside)) {
      constexpr unsigned ALL = (1u << M) - 1u;
      const double g = double(sm.Qu[ri]);
      // the unconstrained minimiser -H^-1 g in FP64 from the factor of H
      double f[M];
      ok = face_factor(H, 0u, lane, f, sm.Lq, Li);
      double d = face_solve(f, sm.Lq, Li, row ? -g : 0.0, lane);
      const bool dl = row && d < lo, dh = row && d > hi;
      d = dl ? lo : (dh ? hi : d);
      W = unsigned(__ballot(dl || dh)) & ALL;
      up = unsigned(__ballot(dh)) & ALL;
      bool at_min = false;
      for (int it = 0; it < 4 * M + 4 && ok; ++it) {
        if (!at_min) {
          if (W == ALL) {
            at_min = true;
            continue;
          }
          ok = face_factor(H, W, lane, f, sm.Lq, Li);
          if (!ok) break;
          const bool held = (W >> ri) & 1u;
          double v = g;
#pragma unroll
          for (int j = 0; j < M; ++j) {
            const double dj = bcast(d, j);
            if ((W >> j) & 1u) v += H[min(ri, j) * (M + 1) + max(ri, j)] * dj;
          }
          const double y = face_solve(f, sm.Lq, Li, (row && !held) ? -v : 0.0, lane);
          // ratio test over the free components
          const double pdir = y - d;
          double t = __builtin_inf();
          if (row && !held) {
            if (pdir < 0.0) t = (lo - d) / pdir;
            else if (pdir > 0.0) t = (hi - d) / pdir;
          }
          double alpha = 1.0;
          int blk = -1;
#pragma unroll
          for (int j = 0; j < M; ++j) {
            const double tj = bcast(t, j);
            if (tj < alpha) {
              alpha = tj;
              blk = j;
            }
          }
          if (blk < 0) {
            if (row && !held) d = y;
            at_min = true;
          } else {
            const bool bup = bcast(pdir, blk) > 0.0;
            if (row && !held)
              d = lane == blk ? (bup ? hi : lo) : clamp_nan2(d + alpha * (y - d), lo, hi);
            W |= 1u << blk;
            up = bup ? (up | (1u << blk)) : (up & ~(1u << blk));
          }
        } else {
          double gr = g;
#pragma unroll
          for (int j = 0; j < M; ++j) gr += H[min(ri, j) * (M + 1) + max(ri, j)] * bcast(d, j);
          const double lam = ((up >> ri) & 1u) ? -gr : gr;
          double lmin = 0.0;
          int rel = -1;
#pragma unroll
          for (int j = 0; j < M; ++j) {
            const double lj = bcast(lam, j);
            if (((W >> j) & 1u) && lj < lmin) {
              lmin = lj;
              rel = j;
            }
          }
          if (rel < 0) break;
          W &= ~(1u << rel);
          at_min = false;
        }
      }
      // the final face's factor (to Lq, Lqi) and the step
      if (ok) ok = face_factor(H, W, lane, f, sm.Lq, Li);
      if (row) sm.kk[ri] = R(d);
      if (lane < M) sm.Lqi[lane] = Li[lane];
      if (lane == 0) sm.flag = ok ? 3 : 1;  // 3: the feedback rows are recomputed below
    } else if (lane == 0) {
      sm.flag = 0;
    }
    if (lane == 0) sm.Hq_held = W;
  }
  __syncthreads();
  if (sm.flag == 1) return ST_CHOL_FAIL;
  if (sm.flag == 0) return 0u;
  // feedback rows from the face factor (FP64), the held rows zero
  if (tid < N) {
    const unsigned W = sm.Hq_held;
    double y[M];
#pragma unroll
    for (int i = 0; i < M; ++i) y[i] = ((W >> i) & 1u) ? 0.0 : double(sm.QuxT[tid][kq(i)]);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      double v = y[i];
#pragma unroll
      for (int k = 0; k < i; ++k) v -= sm.Lq[i][k] * y[k];
      y[i] = v * sm.Lqi[i];
    }
#pragma unroll
    for (int i = M - 1; i >= 0; --i) {
      double v = y[i];
#pragma unroll
      for (int k = i + 1; k < M; ++k) v -= sm.Lq[k][i] * y[k];
      y[i] = v * sm.Lqi[i];
    }
    bool fin = true;
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const R kv = R(-y[i]);
      sm.KT[tid][kq(i)] = kv;
      fin = fin && isfinite(kv);
    }
    if (tid < M) fin = fin && isfinite(sm.kk[tid]);
    if (!fin) sm.flag = 2;
  }
  __syncthreads();
  return sm.flag == 2 ? ST_NONFINITE : 0u;
}

template <class R>
struct QW {  // workspace accessors (the lane schedule's slot-major layout)
  static __device__ __forceinline__ R* xp(const LaneState<R>& w, int buf, int k, int s) {
    return w.X + (size_t(buf) * w.Bcap + s) * w.xs + k * N;
  }
  static __device__ __forceinline__ R* up(const LaneState<R>& w, int buf, int k, int s) {
    return w.U + (size_t(buf) * w.Bcap + s) * w.us + k * M;
  }
  static __device__ __forceinline__ R* Kp(const LaneState<R>& w, int k, int s) {
    return w.K + size_t(s) * w.Ks + k * (M * N);
  }
  static __device__ __forceinline__ R* kp(const LaneState<R>& w, int k, int s) {
    return w.kf + size_t(s) * w.ks + k * M;
  }
};

// ------------------------------------------------------------------ backward sweep
// BOX: the bounded control step of eq. 1 (umax); mu: the Levenberg-Marquardt
// shift of Q_uu (zero for the clipped form).
//
// A step is a chain of four phases between barriers, each spread over the
// four waves (16 x 16 tiles; all operands as rows in kpos order):
//   1. (P [f_x | f_u])^T, wave w the columns of block w (three of f_x, one of
//      f_u) against P's three row blocks; P's row 37 holds p, so the same
//      tiles give f_x^T p and f_u^T p;
//   2. waves 0..2: the Q_xx tiles (w, w), (w, w + 1) and the transpose of
//      (w + 1, w), kept in registers, and Q_ux's tile of block w; wave 3: Q_uu
//      and its factor, the phase's longest chain;
//   3. wave 3: the gains; waves 0..2 put the next step's derivative block,
//      which they loaded during phase 2, into the other buffer;
//   4. waves 0..2: C = Q_xx + Q_ux^T K on their tiles and P = sym(C): a pair
//      of tiles is symmetrised in registers, a diagonal tile through the
//      wave's own scratch; wave 3: the gains' store and p.
// Bound: this chain (latency of the dependent matrix instructions, of the
// factor's twelve pivots and of LDS), of which two resident instances hide
// each other's.  Before, with scalar operand loads under bounds checks and
// Q_xx, C and its symmetrised form through LDS, a step took six barriers and
// 1024 mixed instances 13.0 ms per solve, 100 in FP64 13.9; now 5.9 and 5.9,
// with wave_dyn's share (a step's phases take 2.4, 5.6, 2.6 and 2.7 thousand
// cycles with two instances per CU).
template <class R, bool BOX>
__device__ __forceinline__ uint32_t backward(Smem<R>& sm, const double* __restrict__ prm, const LaneState<R>& w, int s, int T,
                             int buf, R eps, int tid, R* __restrict__ blk, double mu, double umax) {
  using Q = QW<R>;
  using V = typename MfAcc<R>::type;
  constexpr int S = Stride<R>::k;
  const R dt = R(prm[O_DT]);
  const R wq = R(prm[O_WQ]), wv = R(prm[O_WV]), wu = R(prm[O_WU]), wT = R(prm[O_WT]);
  // terminal: P = clip(l_T,xx) (diagonal), p = l_T,x
  for (int i = tid; i < (N + 1) * S; i += NT) (&sm.P[0][0])[i] = R(0);
  __syncthreads();
  if (tid < N) {
    const R xv = Q::xp(w, buf, T, s)[tid];
    const R wi = (tid < NQ ? wq : wv) * wT;
    sm.P[N][kpos(tid)] = R(2) * wi * (xv - sm.xnom[tid]);
    sm.P[tid][kpos(tid)] = dmax(R(2) * wi, eps);
  }
  __syncthreads();
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  // derivative blocks are copied by 16-byte pieces
  typedef float Piece __attribute__((ext_vector_type(4)));
  constexpr int PR = KROW * int(sizeof(R)) / 16, NP = (N + M) * PR;  // pieces per row, per block
  auto block_of = [&](int kk) { return blk + ((T - 1 - kk) % CH) * DB; };
  auto put_piece = [&](int kk, int i, const Piece& v) {
    const int r = i / PR, c = i - r * PR;
    *reinterpret_cast<Piece*>(&sm.AT[kk & 1][r < N ? r : BROW + r - N][c * (16 / int(sizeof(R)))]) = v;
  };
  constexpr int NS = NT - 64, PP = (NP + NS - 1) / NS;  // staging threads of a step, pieces of each
  for (int k = T - 1; k >= 0; --k) {
    const int q = (T - 1 - k) % CH;
    const int cb = k & 1;
    if (q == 0) {
      const int lane = fresh(tid & 63);
      // derivative blocks of the next CH steps, wave wid taking every fourth
      // step (they do not depend on P)
      WaveScratch<R>& wsw = sm.wv[wid];
      for (int qq = wid; qq < CH && k - qq >= 0; qq += NW) {
        if (lane < N) wsw.x[lane] = Q::xp(w, buf, k - qq, s)[lane];
        if (lane < M) wsw.u[lane] = Q::up(w, buf, k - qq, s)[lane];
        wave_sync();
        wave_dyn(sm, wsw, dt, lane);
        wave_jac(sm, wsw, dt, lane, blk + qq * DB);
        wave_sync();
      }
      __syncthreads();
      const Piece* src = reinterpret_cast<const Piece*>(block_of(k));
      for (int i = tid; i < NP; i += NT) put_piece(k, i, src[i]);
      if (tid < N) sm.xs[cb][tid] = Q::xp(w, buf, k, s)[tid];
      if (tid < M) sm.us[cb][tid] = Q::up(w, buf, k, s)[tid];
      __syncthreads();
    }
    // ---- phase 1
    {
      const int lane = fresh(tid & 63), li = lane & 15, lk = lane >> 4;
      R at[10], pr[3][10];
      ld_op(at, &sm.AT[cb][16 * wid + li][lk * KG]);
#pragma unroll
      for (int b = 0; b < 3; ++b) ld_op(pr[b], &sm.P[16 * b + li][lk * KG]);
      V acc[3] = {};
#pragma unroll
      for (int t = 0; t < 10; ++t)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc[b] = mfma16(pr[b][t], at[t], acc[b]);
      R* dst = sm.PAT[16 * wid + li];
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * b + MfAcc<R>::row(lk, r);
          dst[kpos(i)] = i < N ? acc[b][r] : R(0);
        }
      // row 37 of the products
      if (lk == 1) {
        const int j = wid < 3 ? 16 * wid + li : N + li;
        if (wid < 3 ? j < N : li < M) sm.Qg[j] = acc[2][1];
      }
    }
    __syncthreads();
    // ---- phase 2
    const int lane = fresh(tid & 63), li = lane & 15, lk = lane >> 4, ltid = 64 * wid + lane;
    V cxy = {}, cyx = {}, cd = {};  // tiles (x, y), (y, x)^T and (x, x) of Q_xx
    const int x0 = 16 * wid, y0 = wid == 2 ? 0 : 16 * (wid + 1);
    const bool ahead = k >= 1 && q + 1 < CH;
    Piece nxt[PP];
    R xn = R(0), un = R(0);
    if (wid < 3) {
      if (ahead) {
        // (all loads without a condition, so that none is waited for here)
        const Piece* src = reinterpret_cast<const Piece*>(block_of(k - 1));
#pragma unroll
        for (int i = 0; i < PP; ++i) nxt[i] = src[min(ltid + i * NS, NP - 1)];
        xn = Q::xp(w, buf, k - 1, s)[min(ltid, N - 1)];
        un = Q::up(w, buf, k - 1, s)[min(ltid, M - 1)];
      }
      R ax[10], ay[10], px[10], py[10], bt[10];
      ld_op(ax, &sm.AT[cb][x0 + li][lk * KG]);
      ld_op(px, &sm.PAT[x0 + li][lk * KG]);
      ld_op(bt, &sm.AT[cb][BROW + li][lk * KG]);
      ld_op(ay, &sm.AT[cb][y0 + li][lk * KG]);
      ld_op(py, &sm.PAT[y0 + li][lk * KG]);
      V cu = {};
#pragma unroll
      for (int t = 0; t < 10; ++t) {
        cu = mfma16(bt[t], px[t], cu);
        cd = mfma16(ax[t], px[t], cd);
        cxy = mfma16(ax[t], py[t], cxy);
        cyx = mfma16(px[t], ay[t], cyx);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sm.QuxT[x0 + li][kq(MfAcc<R>::row(lk, r))] = cu[r];
        // the clipped diagonal Hessian
        const int i = x0 + MfAcc<R>::row(lk, r);
        if (MfAcc<R>::row(lk, r) == li && i < N) cd[r] += dmax(R(2) * (i < NQ ? wq : wv), eps);
      }
    } else {
      // Q_uu = clip(l_uu) + B^T (P B) (+ mu I, the Levenberg-Marquardt shift,
      // zero otherwise: adding it changes no bit) in FP64
      R bt[10], pb[10];
      ld_op(bt, &sm.AT[cb][BROW + li][lk * KG]);
      ld_op(pb, &sm.PAT[BROW + li][lk * KG]);
      V cq = {};
#pragma unroll
      for (int t = 0; t < 10; ++t) cq = mfma16(bt[t], pb[t], cq);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = MfAcc<R>::row(lk, r);
        if (i < M && li < M) {
          double v = double(cq[r]) + (i == li ? double(dmax(R(2) * wu, eps)) : 0.0);
          if (i == li) v += mu;
          sm.Quu[i][li] = v;
        }
      }
      if (lane < M) sm.Qu[lane] = R(2) * wu * sm.us[cb][lane] + sm.Qg[N + lane];
      if (lane == 0) sm.nonfin = 0;
      wave_sync();
      factor_quu(sm, lane);
    }
    __syncthreads();
    if (sm.flag) return ST_CHOL_FAIL;
    // ---- phase 3
    if (wid == 3) {
      solve_gains(sm, lane);
    } else if (ahead) {
#pragma unroll
      for (int i = 0; i < PP; ++i)
        if (ltid + i * NS < NP) put_piece(k - 1, ltid + i * NS, nxt[i]);
      if (ltid < N) sm.xs[cb ^ 1][ltid] = xn;
      if (ltid < M) sm.us[cb ^ 1][ltid] = un;
    }
    __syncthreads();
    if (sm.nonfin) return ST_NONFINITE;
    if constexpr (BOX) {
      const uint32_t b = box_step(sm, sm.us[cb], umax, tid);
      if (b) return b;
    }
    // ---- phase 4: C = Q_xx + Q_ux^T K, P = sym(C), p = Q_x + Q_ux^T k
    if (wid < 3) {
      R qx[3], qy[3], kx[3], ky[3];
      ld_op12(qx, &sm.QuxT[x0 + li][lk * 4]);
      ld_op12(kx, &sm.KT[x0 + li][lk * 4]);
      ld_op12(qy, &sm.QuxT[y0 + li][lk * 4]);
      ld_op12(ky, &sm.KT[y0 + li][lk * 4]);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        cd = mfma16(qx[t], kx[t], cd);
        cxy = mfma16(qx[t], ky[t], cxy);
        cyx = mfma16(kx[t], qy[t], cyx);
      }
      R* sc = sm.PAT[x0];  // the wave's sixteen rows
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[MfAcc<R>::row(lk, r) * S + li] = cd[r];
      const int j = y0 + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = x0 + MfAcc<R>::row(lk, r);
        if (i < N && j < N) {
          const R v = R(0.5) * (cxy[r] + cyx[r]);
          sm.P[i][kpos(j)] = v;
          sm.P[j][kpos(i)] = v;
        }
      }
      wave_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = MfAcc<R>::row(lk, r);
        const R v = R(0.5) * (cd[r] + sc[li * S + i]);
        if (x0 + i < N && x0 + li < N) sm.P[x0 + i][kpos(x0 + li)] = v;
      }
    } else {
      R* dK = Q::Kp(w, k, s);
      R kb[M], kc[M], qc[M];
      ld12(kb, sm.kk);
      const int row = lane < N ? lane : 0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        R a[3], b[3];
        ld_op12(a, &sm.KT[row][4 * g]);
        ld_op12(b, &sm.QuxT[row][4 * g]);
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          kc[g + 4 * t] = a[t];
          qc[g + 4 * t] = b[t];
        }
      }
      if (lane < N) {
        R v = R(2) * (lane < NQ ? wq : wv) * (sm.xs[cb][lane] - sm.xnom[lane]) + sm.Qg[lane];
#pragma unroll
        for (int t = 0; t < M; ++t) {
          dK[t * N + lane] = kc[t];
          v += qc[t] * kb[t];
        }
        sm.P[N][kpos(lane)] = v;
      }
      if (lane < M) Q::kp(w, k, s)[lane] = sm.kk[lane];
    }
    __syncthreads();
  }
  return 0;
}

// ------------------------------------------------------------------ line-search trial (one wave)
// Closed-loop rollout of wave `wid` with step alpha; writes the trajectory
// when `write`; early stop once the partial cost reaches Jcur (costs >= 0).
// With BOX the trial's controls are clamped into [-umax, umax] (eq. 1).
template <class R, bool BOX>
__device__ __forceinline__ double wave_trial(Smem<R>& sm, const double* __restrict__ prm, const LaneState<R>& w, int s, int T,
                             int buf, R alpha, double Jcur, bool write, int lane_, int wid, int& steps, R umax) {
  using Q = QW<R>;
  const int lane = fresh(lane_);
  WaveScratch<R>& ws = sm.wv[wid];
  const R dt = R(prm[O_DT]);
  const int nb = buf ^ 1;
  if (lane < N) ws.x[lane] = Q::xp(w, buf, 0, s)[lane];
  wave_sync();
  double Jh = 0.0;
  steps = T;
  // the iterate's step data (x_k; lane (c, part): entries part, part + 4, ...
  // of row c of K_k; u_k and k_k for c) are loaded one step ahead of their use
  constexpr int KQ = (N + 3) / 4;
  R xq = R(0), uq = R(0), kq = R(0), Kq[KQ];
  auto load = [&](int k) {
    const int lane = fresh(lane_), c = lane >> 2, part = lane & 3;
    if (lane < N) xq = Q::xp(w, buf, k, s)[lane];
    if (c < M) {
      const R* Kr = Q::Kp(w, k, s) + c * N;
#pragma unroll
      for (int q = 0; q < KQ; ++q) Kq[q] = part + 4 * q < N ? Kr[part + 4 * q] : R(0);
      if (part == 0) {
        uq = Q::up(w, buf, k, s)[c];
        kq = Q::kp(w, k, s)[c];
      }
    }
  };
  load(0);
  for (int k = 0; k < T; ++k) {
    const int lane = fresh(lane_), c = lane >> 2, part = lane & 3;
    const R xk = xq, uk = uq, kk = kq;
    R Kc[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) Kc[q] = Kq[q];
    if (k + 1 < T) load(k + 1);
    if (lane < N) ws.dx[lane] = ws.x[lane] - xk;
    wave_sync();
    {
      R acc = R(0);
      if (c < M) {
#pragma unroll
        for (int q = 0; q < KQ; ++q)
          if (part + 4 * q < N) acc += Kc[q] * ws.dx[part + 4 * q];
      }
      acc += lane_other<1>(acc, lane);
      acc += lane_other<2>(acc, lane);
      if (c < M && part == 0) {
        const R v = uk + alpha * kk + acc;
        ws.u[c] = BOX ? clamp_nan(v, umax) : v;
      }
    }
    wave_sync();
    Jh += double(wave_cost(sm, ws.x, ws.u, prm, lane, false));
    wave_dyn(sm, ws, dt, lane);
    if (write) {
      if (lane < M) Q::up(w, nb, k, s)[lane] = ws.u[lane];
      if (lane < N) Q::xp(w, nb, k + 1, s)[lane] = ws.xn[lane];
    }
    if (lane < N) ws.x[lane] = ws.xn[lane];
    wave_sync();
    if (!(Jh < Jcur)) {
      steps = k + 1;
      return Jh;
    }
  }
  Jh += double(wave_cost(sm, ws.x, ws.u, prm, lane, true));
  return Jh;
}

// ------------------------------------------------------------------ kernels
// Initial rollout: one wave per instance, a serial chain of T dynamics steps
template <class R>
__global__ void __launch_bounds__(64) quad_init(const double* __restrict__ prm, LaneState<R> w, int nthreads,
                                                 const int32_t* __restrict__ slots, int Tmax,
                                                 const int32_t* __restrict__ Tin, const int32_t* __restrict__ perm,
                                                 const double* __restrict__ x0, const double* __restrict__ U0,
                                                 int max_iter, double* __restrict__ trace, double umax) {
  using Q = QW<R>;
  __shared__ WaveSmem<R, 1> sm;
  const int g = blockIdx.x, tid = threadIdx.x;
  if (g >= nthreads) return;
  const int s = slots ? slots[g] : g;
  const int b = perm ? perm[g] : g;
  const int Tr = Tin ? Tin[b] : Tmax;
  const bool badT = Tr < 1 || Tr > Tmax || Tr > w.Tcap;
  const int T = badT ? 0 : Tr;
  stage_constants(sm, prm, tid, 64);
  __syncthreads();
  const int lane = tid;
  WaveScratch<R>& ws = sm.wv[0];
  const R dt = R(prm[O_DT]);
  if (lane < N) {
    const R v = R(x0[size_t(b) * N + lane]);
    ws.x[lane] = v;
    Q::xp(w, 0, 0, s)[lane] = v;
    Q::xp(w, 1, 0, s)[lane] = v;
  }
  wave_sync();
  double J = 0.0;
  for (int k = 0; k < T; ++k) {
    if (lane < M) {
      // the warm start is clamped into the box of eq. 1 (umax infinite: none)
      const R v = clamp_nan(U0 ? R(U0[(size_t(b) * Tmax + k) * M + lane]) : R(0), R(umax));
      ws.u[lane] = v;
      Q::up(w, 0, k, s)[lane] = v;
    }
    wave_sync();
    J += double(wave_cost(sm, ws.x, ws.u, prm, lane, false));
    wave_dyn(sm, ws, dt, lane);
    if (lane < N) {
      ws.x[lane] = ws.xn[lane];
      Q::xp(w, 0, k + 1, s)[lane] = ws.xn[lane];
    }
    wave_sync();
  }
  J += double(wave_cost(sm, ws.x, ws.u, prm, lane, true));
  if (lane == 0) {
    uint32_t st = isfinite(J) ? 0u : ST_NONFINITE;
    if (st == 0 && max_iter <= 0) st = ST_MAX_ITER;
    if (badT) {
      st = ST_BAD_INPUT;
      J = __builtin_nan("");
    }
    w.T[s] = T;
    w.inst[s] = slots ? s : b;
    w.J[s] = J;
    w.okey[s] = order_key(Tin != nullptr, T, J, 0.f, Tmax);  // no non-convex share: J^0 alone
    w.iters[s] = 0;
    w.status[s] = st;
    w.cur[s] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) w.work[4 * s + i] = 0;
    if (trace) trace[size_t(slots ? s : b) * (max_iter + 1)] = J;
  }
}

template <class R, bool BOX, bool LM, int OCC>
// OCC: workgroups resident per CU the registers are sized for.  With 1 the
// kernel keeps its values in registers (one wave per SIMD); with 2 the
// registers are capped at 256 and some values spill (28 B of scratch, 304 with
// the bound), but the per-step chain is latency-bound and a second resident
// instance per CU hides most of it once the batch fills every CU (mixed, 50
// steps, four iterations, one / two per CU: 512 instances 6.13 / 4.15 ms, 64
// instances 3.22 / 3.24).  FP64 is built for one: its 145 KB of LDS fit a CU
// once.
// BOX: the variant with the control bound of eq. 1 (sp.umax finite).  LM: the
// Levenberg-Marquardt variant (sp.reg = 1), in which a failed Cholesky or line search
// multiplies mu by mu_fac and retries the sweep while mu stays within mu_max;
// an accepted step divides it (not below mu0); mu carries over between launches.
__global__ void __launch_bounds__(NT, OCC) quad_iterate(const double* __restrict__ prm, LaneState<R> w, int nslots,
                                                    const int32_t* __restrict__ slots, SolveParams sp,
                                                    int iters_this_launch, IterTrace tr,
                                                    R* __restrict__ dblk) {
  __shared__ Smem<R> sm;
  const int g = blockIdx.x, tid = threadIdx.x;
  if (g >= nslots) return;
  const int s = slots ? slots[g] : g;
  uint32_t st = w.status[s];
  if (st) return;  // uniform over the workgroup
  const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  stage_constants(sm, prm, tid);
  __syncthreads();
  const int T = w.T[s];
  const int b = w.inst[s];
  double J = w.J[s];
  int iters = w.iters[s];
  int buf = w.cur[s];
  int nsweep = w.work[4 * s], npass = w.work[4 * s + 1], nread = w.work[4 * s + 2], nwrite = w.work[4 * s + 3];
  const R eps = R(sp.eps);
  constexpr bool lm = LM;
  double mu = lm ? (nsweep == 0 ? sp.mu0 : w.mu[s]) : 0.0;
  for (int it = 0; it < iters_this_launch && st == 0; ++it) {
    if (iters >= sp.max_iter) {
      st = ST_MAX_ITER;
      break;
    }
    int acc = -1;
    double Jn = J;
    uint32_t fail = 0;
    for (;;) {
      ++nsweep;
      const uint32_t bad = backward<R, BOX>(sm, prm, w, s, T, buf, eps, tid, dblk + size_t(s) * CH * DB, mu, sp.umax);
      if (bad) {
        if (lm && bad == ST_CHOL_FAIL && mu * sp.mu_fac <= sp.mu_max) {
          mu *= sp.mu_fac;
          continue;
        }
        fail = bad;
        break;
      }
      // line search: rounds of NW parallel trials, then (if the accepted step
      // is not alpha = 1, which wave 0 wrote while trying it) one commit
      // rollout; a single call site keeps the kernel's register footprint down
      acc = -1;
      Jn = J;
      bool commit = false;
      for (int j0 = 0;;) {
        const int j = commit ? acc : j0 + wid;
        const bool run = commit ? (wid == 0) : (j < sp.ls_trials);
        double Jh = __builtin_nan("");
        int steps = 0;
        if (run) {
          double alpha = 1.0;
          for (int q = 0; q < j; ++q) alpha *= sp.beta;
          Jh = wave_trial<R, BOX>(sm, prm, w, s, T, buf, R(alpha), commit ? __builtin_inf() : J, commit || j == 0,
                                  lane, wid, steps, R(sp.umax));
        }
        if (lane == 0) {
          sm.wJ[wid] = Jh;
          sm.wok[wid] = steps;
        }
        __syncthreads();
        ++npass;
        if (commit) {
          Jn = sm.wJ[0];
          nread += T;
          nwrite += T;
          __syncthreads();
          break;
        }
        int longest = 0;
        for (int q = 0; q < NW; ++q) {
          longest = max(longest, sm.wok[q]);
          const double v = sm.wJ[q];
          if (acc < 0 && j0 + q < sp.ls_trials && isfinite(v) && v < J) {
            acc = j0 + q;
            Jn = v;
          }
        }
        if (j0 == 0) nwrite += sm.wok[0];
        nread += longest;
        __syncthreads();
        j0 += NW;
        if (acc == 0 || (acc < 0 && j0 >= sp.ls_trials)) break;
        if (acc > 0) commit = true;
      }
      if (acc < 0) {
        if (lm && mu * sp.mu_fac <= sp.mu_max) {
          mu *= sp.mu_fac;
          continue;
        }
        fail = ST_LS_FAILED;
      }
      break;
    }
    if (tr.j && tid == 0) tr.j[size_t(b) * sp.max_iter + iters] = fail ? -1 : acc;
    if (fail) {
      st = fail;
      break;
    }
    if (lm) mu = fmax(mu / sp.mu_fac, sp.mu0);
    buf ^= 1;
    const double Jold = J;
    J = Jn;
    ++iters;
    if (tr.J && tid == 0) tr.J[size_t(b) * (sp.max_iter + 1) + iters] = J;
    if (sp.stop_mode == 1 && (Jold - J) <= sp.rtol * fabs(Jold)) {
      st = ST_CONVERGED;
      break;
    }
    if (iters >= sp.max_iter) st = ST_MAX_ITER;
  }
  if (tid == 0) {
    w.J[s] = J;
    w.iters[s] = iters;
    w.status[s] = st;
    w.cur[s] = buf;
    w.work[4 * s] = nsweep;
    w.work[4 * s + 1] = npass;
    w.work[4 * s + 2] = nread;
    w.work[4 * s + 3] = nwrite;
    if (lm) w.mu[s] = mu;
  }
}

template <class R>
__global__ void __launch_bounds__(NT, 2) quad_final(const double* __restrict__ prm, LaneState<R> w, int nslots,
                                                  const int32_t* __restrict__ slots, int Tmax, int max_iter,
                                                  int lookahead, FinalOut o, R* __restrict__ dblk) {
  using Q = QW<R>;
  __shared__ WaveSmem<R, NW> sm;
  const int g = blockIdx.x, tid = threadIdx.x;
  if (g >= nslots) return;
  const int s = slots ? slots[g] : g;
  const int b = w.inst[s];
  const int buf = w.cur[s];
  uint32_t st = w.status[s];
  if (st == 0) st = ST_MAX_ITER;
  const int T = (st & ST_BAD_INPUT) ? -1 : w.T[s];
  const double J = w.J[s];
  const int iters = w.iters[s];
  if (tid == 0) {
    o.J[b] = J;
    o.iters[b] = iters;
    o.status[b] = st;
    if (o.work)
      for (int i = 0; i < 4; ++i) o.work[4 * b + i] = w.work[4 * s + i];
  }
  if (o.trace)
    for (int i = iters + 1 + tid; i <= max_iter; i += NT) o.trace[size_t(b) * (max_iter + 1) + i] = J;
  double* Xo = o.X + size_t(b) * (Tmax + 1) * N;
  double* Uo = o.U + size_t(b) * Tmax * M;
  for (int idx = tid; idx < (Tmax + 1) * N; idx += NT) {
    const int k = idx / N, i = idx % N;
    Xo[idx] = k <= T ? double(Q::xp(w, buf, k, s)[i]) : 0.0;
  }
  for (int idx = tid; idx < Tmax * M; idx += NT) {
    const int k = idx / M, i = idx % M;
    Uo[idx] = k < T ? double(Q::up(w, buf, k, s)[i]) : 0.0;
  }
  const int K = lookahead <= 0 ? T : lookahead;
  if (o.xK) {
    double* xo = o.xK + size_t(b) * (Tmax + 1) * N;
    for (int idx = tid; idx < (Tmax + 1) * N; idx += NT) {
      const int k = idx / N, i = idx % N;
      xo[idx] = k <= T ? double(Q::xp(w, buf, (k + K < T ? k + K : T), s)[i]) : 0.0;
    }
  }
  double* Vo = o.Vbar ? o.Vbar + size_t(b) * (Tmax + 1) : nullptr;
  double* Lo = o.Vx ? o.Vx + size_t(b) * (Tmax + 1) * N : nullptr;
  if (T < 0) {
    if (Vo)
      for (int k = tid; k <= Tmax; k += NT) Vo[k] = 0.0;
    if (Lo)
      for (int idx = tid; idx < (Tmax + 1) * N; idx += NT) Lo[idx] = 0.0;
    return;
  }
  if (!Vo && !Lo) return;
  stage_constants(sm, prm, tid);
  __syncthreads();
  const R dt = R(prm[O_DT]);
  const R wq = R(prm[O_WQ]), wv = R(prm[O_WV]), wT = R(prm[O_WT]);
  WaveScratch<R>& w0 = sm.wv[0];
  // lambda_T = d l_T / dx
  if (tid < N) {
    w0.x[tid] = Q::xp(w, buf, T, s)[tid];
    const R wi = (tid < NQ ? wq : wv) * wT;
    sm.p[tid] = R(2) * wi * (w0.x[tid] - sm.xnom[tid]);
    if (Lo) Lo[size_t(T) * N + tid] = double(sm.p[tid]);
  }
  __syncthreads();
  if (Vo && tid < 64) {
    const double cT = double(wave_cost(sm, w0.x, w0.u, prm, tid, true));
    if (tid == 0) Vo[T] = cT;
  }
  __syncthreads();
  // costate lambda_k = l_x + f_x^T lambda_{k+1} through the adjoint of the
  // semi-implicit step instead of f_x itself: with
  // mu = lambda_v+ + dt E^T lambda_q+ and nu = M^-1 mu (M's factor from the
  // dynamics at (x_k, u_k); M is symmetric),
  //   f_x^T lambda+ = [lambda_q+ + dt g ; mu - dt (W2 cos q) . nu],
  //   g_j = -cos q_j (W1^T nu)_j + sin q_j (W2^T (nu . v))_j - 0.1 cos q_j a_j nu_j  (j < 18),
  // and nothing from the dynamics for q_18: one solve per step instead of the
  // 48 columns of [f_x | f_u].
  // The dynamics at a step (M's factor, accelerations, sin/cos) do not depend
  // on lambda: the four waves evaluate them for four steps at once (wave w
  // for step kc - w, with that step's stage cost), then wave 0 walks the four
  // steps.
  (void)dblk;
  {
    const int wid = tid >> 6, lane = tid & 63;
    const bool row = lane < NV;
    const int ri = row ? lane : 0;
    for (int kc = T - 1; kc >= 0; kc -= NW) {
      {
        const int k = kc - wid;
        WaveScratch<R>& ws = sm.wv[wid];
        if (k >= 0) {
          if (lane < N) ws.x[lane] = Q::xp(w, buf, k, s)[lane];
          if (lane < M) ws.u[lane] = Q::up(w, buf, k, s)[lane];
          wave_sync();
          if (Vo) {
            const double c = double(wave_cost(sm, ws.x, ws.u, prm, lane, false));
            if (lane == 0) Vo[k] = c;
          }
          if (Lo) wave_dyn(sm, ws, dt, lane);
        }
      }
      __syncthreads();
      if (Lo && wid == 0) {
        for (int q = 0; q < NW && kc - q >= 0; ++q) {
          const int k = kc - q;
          WaveScratch<R>& ws = sm.wv[q];
          // nu = M^-1 mu: L z = mu, then L^T nu = z (rows on lanes)
          R y = row ? sm.p[NQ + ri] + dt * (sm.p[ri] + sm.e[ri] * sm.p[NV]) : R(0);
          R l[NV], lt[NV], inv[NV];
          ld_row(l, ws.L[ri]);
          ld_row(inv, ws.Li);
#pragma unroll
          for (int j = 0; j < NV; ++j) lt[j] = ws.L[j][ri];
#pragma unroll
          for (int j = 0; j < NV; ++j) y = forward_step(y, l[j], inv[j], j, lane);
#pragma unroll
          for (int j = NV - 1; j >= 0; --j) y = backward_step(y, lt[j], inv[j], j, lane);
          if (row) ws.dx[ri] = y;
          wave_sync();
          R ln = R(0);
          if (lane < N) {
            ln = R(2) * (lane < NQ ? wq : wv) * (ws.x[lane] - sm.xnom[lane]);
            if (lane < NV) {
              R g1 = R(0), g2 = R(0);
#pragma unroll
              for (int i = 0; i < NV; ++i) {
                g1 += sm.W1[i][lane] * ws.dx[i];
                g2 += sm.W2[i][lane] * (ws.dx[i] * ws.x[NQ + i]);
              }
              const R gq = -ws.c[lane] * g1 + ws.s[lane] * g2 - R(0.1) * ws.c[lane] * ws.a[lane] * ws.dx[lane];
              ln += sm.p[lane] + dt * gq;
            } else if (lane == NV) {
              ln += sm.p[NV];
            } else {
              const int i = lane - NQ;
              const R mu = sm.p[lane] + dt * (sm.p[i] + sm.e[i] * sm.p[NV]);
              ln += mu - dt * ws.w2c[i] * ws.dx[i];
            }
          }
          wave_sync();  // every read of lambda_{k+1} is done before it is replaced
          if (lane < N) {
            sm.p[lane] = ln;
            Lo[size_t(k) * N + lane] = double(ln);
          }
          wave_sync();
        }
      }
      __syncthreads();
    }
  }
  __syncthreads();
  if (Vo && tid == 0) {
    const double cT = Vo[T];
    if (K >= T) {
      double acc = cT;
      for (int k = T - 1; k >= 0; --k) {
        acc = Vo[k] + acc;
        Vo[k] = acc;
      }
    } else {
      for (int k = 0; k < T; ++k) {
        const int end = k + K < T ? k + K : T;
        double v = 0.0;
        for (int j = k; j < end; ++j) v += Vo[j];
        if (k + K >= T) v += cT;
        Vo[k] = v;
      }
    }
    for (int k = T + 1; k <= Tmax; ++k) Vo[k] = 0.0;
  }
  if (Lo)
    for (int idx = (T + 1) * N + tid; idx < (Tmax + 1) * N; idx += NT) Lo[idx] = 0.0;
}

template <class R>
struct QuadLaunch {
  // the lane layout, then per slot CH derivative blocks
  static size_t ws_bytes(int Bcap, int Tcap) {
    return lane_layout(N, M, int(sizeof(R)), Bcap, Tcap).total + size_t(Bcap) * CH * DB * sizeof(R);
  }
  static R* blocks(void* base, int Bcap, int Tcap) {
    return reinterpret_cast<R*>(static_cast<char*>(base) + lane_layout(N, M, int(sizeof(R)), Bcap, Tcap).total);
  }

  static hipError_t init(const double* prm, void* base, int Bcap, int Tcap, int nthreads, const int32_t* slots,
                         int Tmax, const int32_t* Tin, const int32_t* perm, const double* x0, const double* U0,
                         int max_iter, double* trace, double umax, hipStream_t st) {
    if (nthreads <= 0) return hipSuccess;
    auto w = lane_state<R>(base, N, M, Bcap, Tcap, 2);
    // one wave per instance (quad_init is built for 64-thread workgroups)
    hipLaunchKernelGGL(quad_init<R>, dim3(nthreads), dim3(64), 0, st, prm, w, nthreads, slots, Tmax, Tin, perm,
                       x0, U0, max_iter, trace, umax);
    return hipGetLastError();
  }

  // the bounded and Levenberg-Marquardt variants are kernels of their own, so
  // that the plain one keeps its register allocation and shared-memory footprint
  template <int OCC>
  static void launch_forms(bool box, bool lm, const double* prm, const LaneState<R>& w, int nthreads,
                           const int32_t* slots, const SolveParams& d, int G, const IterTrace& tr, R* blk,
                           hipStream_t st) {
    if (box && lm)
      hipLaunchKernelGGL((quad_iterate<R, true, true, OCC>), dim3(nthreads), dim3(NT), 0, st, prm, w, nthreads,
                         slots, d, G, tr, blk);
    else if (box)
      hipLaunchKernelGGL((quad_iterate<R, true, false, OCC>), dim3(nthreads), dim3(NT), 0, st, prm, w, nthreads,
                         slots, d, G, tr, blk);
    else if (lm)
      hipLaunchKernelGGL((quad_iterate<R, false, true, OCC>), dim3(nthreads), dim3(NT), 0, st, prm, w, nthreads,
                         slots, d, G, tr, blk);
    else
      hipLaunchKernelGGL((quad_iterate<R, false, false, OCC>), dim3(nthreads), dim3(NT), 0, st, prm, w, nthreads,
                         slots, d, G, tr, blk);
  }

  static hipError_t iterate(const double* prm, void* base, int Bcap, int Tcap, int nthreads,
                            const int32_t* slots, const SolveParamsH& sp, int G, int group, const IterTrace& tr,
                            hipStream_t st) {
    if (nthreads <= 0) return hipSuccess;
    auto w = lane_state<R>(base, N, M, Bcap, Tcap, 2);
    const SolveParams d = to_dev(sp);
    R* blk = blocks(base, Bcap, Tcap);
    const bool box = __builtin_isfinite(sp.umax), lm = sp.reg == 1;
    // group: workgroups per CU (2 only in FP32; FP64 always runs one per CU)
    if constexpr (sizeof(R) == 4) {
      if (group == 2) {
        launch_forms<2>(box, lm, prm, w, nthreads, slots, d, G, tr, blk, st);
        return hipGetLastError();
      }
    }
    launch_forms<1>(box, lm, prm, w, nthreads, slots, d, G, tr, blk, st);
    return hipGetLastError();
  }

  static hipError_t finalize(const double* prm, void* base, int Bcap, int Tcap, int nthreads,
                             const int32_t* slots, int Tmax, int max_iter, int lookahead, const FinalOutH& o,
                             hipStream_t st) {
    if (nthreads <= 0) return hipSuccess;
    auto w = lane_state<R>(base, N, M, Bcap, Tcap, 2);
    FinalOut fo{o.X, o.U, o.J, o.iters, o.status, o.Vbar, o.Vx, o.xK, o.trace, o.work};
    hipLaunchKernelGGL(quad_final<R>, dim3(nthreads), dim3(NT), 0, st, prm, w, nthreads, slots, Tmax, max_iter,
                       lookahead, fo, blocks(base, Bcap, Tcap));
    return hipGetLastError();
  }

  static const Launcher* get() {
    static const Launcher L{N, M, int(sizeof(R)), CBIC_SCHED_GROUP, &ws_bytes, &init, &iterate, &finalize,
                            size_t(CH) * DB * sizeof(R)};
    return &L;
  }
};

}  // namespace quad

const Launcher* launcher_quad(int precision) {
  return precision ? quad::QuadLaunch<float>::get() : quad::QuadLaunch<double>::get();
}

}  // namespace cbic
