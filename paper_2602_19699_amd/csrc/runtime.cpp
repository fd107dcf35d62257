// Host runtime: error reporting, workspace layouts, per-system device
// parameter blocks, the launcher table and the batched solve entry point.
#include "runtime.hpp"

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <atomic>
#include <climits>

namespace cbic {

const Launcher* launcher_point_mass(int precision);
const Launcher* launcher_lq(int n, int m, int precision);
const Launcher* launcher_arm(int precision);
const Launcher* launcher_quad(int precision);

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
}

const char* last_error() { return g_err; }

static size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

LaneLayout lane_layout(int N, int M, int elem, int Bcap, int Tcap, int nbuf) {
  LaneLayout L{};
  size_t o = 0;
  const size_t B = size_t(Bcap);
  L.T = o; o = align256(o + 4 * B);
  L.inst = o; o = align256(o + 4 * B);
  L.J = o; o = align256(o + 8 * B);
  L.iters = o; o = align256(o + 4 * B);
  L.status = o; o = align256(o + 4 * B);
  L.cur = o; o = align256(o + 4 * B);
  L.work = o; o = align256(o + 16 * B);
  L.mu = o; o = align256(o + 8 * B);
  L.okey = o; o = align256(o + 4 * B);
  // slot-major, each slot's block padded to whole cache lines
  L.X = o; o = align256(o + size_t(elem) * nbuf * B * lane_stride((Tcap + 1) * N, elem));
  L.U = o; o = align256(o + size_t(elem) * nbuf * B * lane_stride(Tcap * M, elem));
  L.K = o; o = align256(o + size_t(elem) * B * lane_stride(Tcap * M * N, elem));
  L.kf = o; o = align256(o + size_t(elem) * B * lane_stride(Tcap * M, elem));
  L.total = o;
  return L;
}

const Launcher* find_launcher(int kind, int n, int m, int precision, int schedule) {
  const Launcher* L = nullptr;
  switch (kind) {
    case CBIC_SYS_POINT_MASS: L = launcher_point_mass(precision); break;
    case CBIC_SYS_PLANAR3: L = launcher_arm(precision); break;
    case CBIC_SYS_LQ: L = launcher_lq(n, m, precision); break;
    case CBIC_SYS_QUAD_SYNTH: L = launcher_quad(precision); break;
    default: break;
  }
  if (L && schedule != 0 && L->schedule != schedule) return nullptr;
  return L;
}

int cu_count(int device) {
  static std::atomic<int> cache[64];
  if (device < 0 || device >= 64) return 256;
  int v = cache[device].load(std::memory_order_relaxed);
  if (v > 0) return v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || v <= 0) v = 256;
  cache[device].store(v, std::memory_order_relaxed);
  return v;
}

// Lane schedule: a line-search round tries as many steps as fill the chip's
// SIMDs once (65536 lanes), for every instance, so that the work counters of a
// batch do not depend on what follows (rounds as wide as the groups would be
// shorter for some: point mass, mixed, tolerance 1e-4, 16384 instances 530 us
// with 8 lanes and 8 trials, 560 with the 4 trials taken here; cbic_autotune
// tries them).  The other work of a group, the
// derivative blocks and the arm's columns, shares out over more lanes than
// that, which shortens each instance's chain and costs the chip more waves.  It
// pays while the chip has room: where the instances end at different times
// (horizons of their own, a tolerance stop, a fixed budget long enough that
// converged ones freeze on the way) far more often than where all run the same
// steps, and less where a wave needs many registers or much LDS time (FP64, the
// arm's bound).  Time of groups as wide as their rounds / of 8 / of 16 lanes, ms,
// 50 or 60 steps, ragged horizons from a quarter of those on:
//   arm, mixed, one horizon, 6 iterations: B 8192 .99 / - / .84, 9700 1.32 / 1.33 / 1.31,
//     16384 1.30 / 1.43 / 1.65, 32768 2.73 / 3.28 / -; ragged: 16384 1.18 / 1.03 / 1.04,
//     65536 4.39 / 4.24 / -; with a bound: 32768 2.83 / 5.65 / -, ragged 2.64 / 3.75 / -
//   arm, FP64, one horizon, 6 iterations: B 4900 1.29 / - / 1.60, 16384 2.14 / 2.78 / -;
//     ragged: 8192 1.25 / - / 1.10, 38800 5.28 / 5.18 / -, 46400 5.46 / 6.05 / -
//   point mass, mixed, one horizon, 6 iterations: B 8192 .40 / - / .44, 16384 .66 / .62
//     / -, 19400 1.26 / 1.32 / -, 32768 1.38 / 1.64 / -; ragged: 46400 2.29 / 2.25 / -, 55200
//     2.47 / 2.64 / -; with a tolerance: 32768 2.07 / 1.95 / -, 65536 4.90 / 4.30 / -
// and relative to narrow groups with 50 iterations: arm, mixed, one horizon,
// 16 lanes: B 4097 .57, 11600 .95, 16384 1.11, 8 lanes: 16385 .72, 23200 1.08, ragged 65536
// .69; FP64, 16 lanes, one: 4097 .63, 5800 1.26, 8 lanes, ragged: 46400 .93, 65536 1.2;
// point mass, 8 lanes, one: mixed 65536 .83, FP64 65536 .66.
// The linear-quadratic kernels have nothing to share and are slower in wider
// groups (6 states, FP64, B 16384: 4 / 8 lanes 2176 / 3090 us).
struct WideLimits {
  long w16, w8;  // the most lanes of a batch in groups of 16, of 8
  long from8;    // lanes in groups of 8 up to which those do not pay either
};
static WideLimits wide_limits(const Launcher* L, const cbic_solve_opts* o, bool ragged) {
  constexpr long S = 65536, ANY = LONG_MAX;
  const bool f32 = L->elem == 4, bound = std::isfinite(o->u_max), lm = o->regularization == CBIC_REG_LM,
             stop = o->stop_mode == 1;
  // (a budget of up to 12 iterations, 13 to 32, more)
  const bool more = o->max_iter > 32, mid = !stop && !more && o->max_iter > 12;
  if (L->N == 4) {  // point mass: converges in 4 iterations (median), 8 (99 %)
    if (stop) return {2 * S, ANY, 0};
    if (lm && (mid || more)) return {2 * S, f32 ? (ragged ? ANY : 8 * S) : (ragged ? 6 : 3) * S, 0};
    if (mid || more) return {2 * S, f32 && mid && !ragged ? 5 * S : ANY, 0};
    if (ragged) return {2 * S, (f32 ? 6 : 4) * S, 0};
    return {lm ? 2 * S : S, f32 ? 9 * S / 4 : S, 0};
  }
  // arm: converges in 56 (median)
  if (ragged) {
    if (f32 && bound) return {4 * S, more ? 8 * S : 5 * S / 2, 0};
    if (f32) return {4 * S, mid && !lm ? 7 * S : ANY, 0};
    if (lm && !bound && (mid || more)) return {2 * S, ANY, 0};
    return {2 * S, more ? 6 * S : (bound || lm ? 5 * S / 2 : 5 * S), 0};
  }
  if (lm && !bound) return f32 ? WideLimits{4 * S, ANY, 0} : WideLimits{2 * S, mid || more ? ANY : S, 0};
  if (!stop && !more) return {f32 ? 5 * S / 2 : S, S, 0};
  return {f32 ? 3 * S : 5 * S / 4, bound ? S : 5 * S / 2, 2 * S};
}

int default_group(const Launcher* L, int B, const cbic_solve_opts* o, bool ragged, int device) {
  if (L->schedule == CBIC_SCHED_GROUP) return (o->precision == CBIC_FP64 || B <= cu_count(device)) ? 1 : 2;
  int trials = 1;
  while (trials < 16 && long(B) * trials * 2 <= 65536) trials *= 2;
  if (L->wide_lanes == 0) return trials;
  const WideLimits w = wide_limits(L, o, ragged);
  int lanes = trials;
  if (long(B) * 16 <= std::min(w.w16, L->wide_lanes)) lanes = 16;
  else if (long(B) * 8 > w.from8 && long(B) * 8 <= w.w8) lanes = 8;
  return group_code(std::max(lanes, trials), trials);
}

int requested_group(const Launcher* L, const cbic_solve_opts* o) {
  return L->schedule == CBIC_SCHED_GROUP ? o->wg_per_cu : o->group_lanes;
}

// ------------------------------------------------------------------ host Jacobi (LQ Hessians)
// Symmetric eigen-decomposition by cyclic Jacobi rotations; used once per LQ
// system to clip its constant Hessians.
static void host_clip(int n, const double* H, double eps, double* out) {
  std::vector<double> a(n * n), v(n * n, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) a[i * n + j] = 0.5 * (H[i * n + j] + H[j * n + i]);
  if (eps < 0.0) {  // no clipping (the Levenberg-Marquardt variant): symmetric part only
    for (int i = 0; i < n * n; ++i) out[i] = a[i];
    return;
  }
  for (int i = 0; i < n; ++i) v[i * n + i] = 1.0;
  for (int sweep = 0; sweep < 60; ++sweep) {
    double off = 0.0, dia = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) (i == j ? dia : off) += a[i * n + j] * a[i * n + j];
    if (!(off > 1e-32 * dia)) break;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const double apq = a[p * n + q];
        if (apq == 0.0) continue;
        const double th = (a[q * n + q] - a[p * n + p]) / (2.0 * apq);
        const double t = (th >= 0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(1.0 + th * th));
        const double c = 1.0 / std::sqrt(1.0 + t * t), s = t * c;
        for (int k = 0; k < n; ++k) {
          const double x = a[k * n + p], y = a[k * n + q];
          a[k * n + p] = c * x - s * y;
          a[k * n + q] = s * x + c * y;
        }
        for (int k = 0; k < n; ++k) {
          const double x = a[p * n + k], y = a[q * n + k];
          a[p * n + k] = c * x - s * y;
          a[q * n + k] = s * x + c * y;
        }
        for (int k = 0; k < n; ++k) {
          const double x = v[k * n + p], y = v[k * n + q];
          v[k * n + p] = c * x - s * y;
          v[k * n + q] = s * x + c * y;
        }
      }
  }
  for (int i = 0; i < n; ++i)
    for (int j = i; j < n; ++j) {
      double s = 0.0;
      for (int k = 0; k < n; ++k) s += v[i * n + k] * std::max(a[k * n + k], eps) * v[j * n + k];
      out[i * n + j] = s;
      out[j * n + i] = s;
    }
}

// ------------------------------------------------------------------ device parameter blocks
static bool all_finite(const double* p, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!std::isfinite(p[i])) return false;
  return true;
}

bool build_device_block(const cbic_system* s, double eps, std::vector<double>& d) {
  const std::vector<double>& p = s->params;
  d.clear();
  switch (s->kind) {
    case CBIC_SYS_POINT_MASS: {
      d = {p[0], p[1], p[2], p[3], p[4], p[5], p[6]};
      for (int i = 0; i < 3; ++i) {
        d.push_back(p[7 + 3 * i]);
        d.push_back(p[8 + 3 * i]);
        d.push_back(1.0 / (p[9 + 3 * i] * p[9 + 3 * i]));
      }
      return true;
    }
    case CBIC_SYS_PLANAR3: {
      const double m1 = p[1], m2 = p[2], m3 = p[3], l1 = p[4], l2 = p[5], l3 = p[6];
      const double I1 = m1 * l1 * l1 / 12.0, I2 = m2 * l2 * l2 / 12.0, I3 = m3 * l3 * l3 / 12.0;
      const double h11 = m1 * l1 * l1 / 4.0 + (m2 + m3) * l1 * l1;
      const double h22 = m2 * l2 * l2 / 4.0 + m3 * l2 * l2;
      const double h33 = m3 * l3 * l3 / 4.0;
      const double h12 = (0.5 * m2 + m3) * l1 * l2;
      const double h13 = 0.5 * m3 * l1 * l3;
      const double h23 = 0.5 * m3 * l2 * l3;
      d = {p[0], h11 + I1, h22 + I2, h33 + I3, h12, h13, h23, l1, l2, l3,
           p[7], p[8], p[9], p[10], p[11], p[12], p[13], p[14], 1.0 / (p[15] * p[15])};
      return true;
    }
    case CBIC_SYS_LQ: {
      const int n = s->n, m = s->m;
      const double* A = p.data() + 2;
      const double* B = A + n * n;
      const double* Q = B + n * m;
      const double* R = Q + n * n;
      const double* QT = R + m * m;
      const double* xr = QT + n * n;
      std::vector<double> Qs(n * n), Rs(m * m), QTs(n * n), Qc(n * n), Rc(m * m), QTc(n * n);
      for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) {
          Qs[i * n + j] = Q[i * n + j] + Q[j * n + i];
          QTs[i * n + j] = QT[i * n + j] + QT[j * n + i];
        }
      for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) Rs[i * m + j] = R[i * m + j] + R[j * m + i];
      host_clip(n, Qs.data(), eps, Qc.data());
      host_clip(m, Rs.data(), eps, Rc.data());
      host_clip(n, QTs.data(), eps, QTc.data());
      d.insert(d.end(), A, A + n * n);
      d.insert(d.end(), B, B + n * m);
      d.insert(d.end(), Qs.begin(), Qs.end());
      d.insert(d.end(), Rs.begin(), Rs.end());
      d.insert(d.end(), QTs.begin(), QTs.end());
      d.insert(d.end(), xr, xr + n);
      d.insert(d.end(), Qc.begin(), Qc.end());
      d.insert(d.end(), Rc.begin(), Rc.end());
      d.insert(d.end(), QTc.begin(), QTc.end());
      return true;
    }
    case CBIC_SYS_QUAD_SYNTH: {
      // same layout as the user's vector with A replaced by the constant part
      // of the mass matrix, A^T A
      d = p;
      const double* A = p.data() + 5;
      for (int a = 0; a < 18; ++a)
        for (int b = 0; b < 18; ++b) {
          double v = 0.0;
          for (int k = 0; k < 18; ++k) v += A[k * 18 + a] * A[k * 18 + b];
          d[5 + a * 18 + b] = v;
        }
      return true;
    }
    default:
      return false;
  }
}

bool make_device_block(cbic_system* s, double eps) { return build_device_block(s, eps, s->dev); }

bool validate_params(int kind, const double* p, size_t np, int* n, int* m) {
  if (!p) {
    set_error("params is NULL");
    return false;
  }
  if (!all_finite(p, np)) {
    set_error("params contain a non-finite value");
    return false;
  }
  switch (kind) {
    case CBIC_SYS_POINT_MASS:
      if (np != 16) { set_error("point mass needs 16 parameters, got %zu", np); return false; }
      if (!(p[0] > 0)) { set_error("dt must be > 0"); return false; }
      for (int i = 0; i < 3; ++i)
        if (!(p[9 + 3 * i] > 0)) { set_error("obstacle radius must be > 0"); return false; }
      *n = 4; *m = 2;
      return true;
    case CBIC_SYS_PLANAR3:
      if (np != 16) { set_error("planar arm needs 16 parameters, got %zu", np); return false; }
      if (!(p[0] > 0)) { set_error("dt must be > 0"); return false; }
      for (int i = 1; i < 7; ++i)
        if (!(p[i] > 0)) { set_error("link masses and lengths must be > 0"); return false; }
      if (!(p[15] > 0)) { set_error("obstacle radius must be > 0"); return false; }
      *n = 6; *m = 3;
      return true;
    case CBIC_SYS_QUAD_SYNTH:
      if (np != 5 + 3 * 324 + 18 + 37) { set_error("quadruped needs 1032 parameters, got %zu", np); return false; }
      if (!(p[0] > 0)) { set_error("dt must be > 0"); return false; }
      *n = 37; *m = 12;
      return true;
    case CBIC_SYS_LQ: {
      if (np < 2) { set_error("LQ parameter vector too short"); return false; }
      const double dn = p[0], dm = p[1];
      if (dn != std::floor(dn) || dm != std::floor(dm) || dn < 1 || dm < 1 || dn > 64 || dm > 64) {
        set_error("LQ dims must be integers in 1..64");
        return false;
      }
      const int nn = int(dn), mm = int(dm);
      const size_t need = 2 + 3 * size_t(nn) * nn + size_t(nn) * mm + size_t(mm) * mm + nn;
      if (np != need) { set_error("LQ with n=%d m=%d needs %zu parameters, got %zu", nn, mm, need, np); return false; }
      *n = nn; *m = mm;
      return true;
    }
    default:
      set_error("unknown system kind %d", kind);
      return false;
  }
}

}  // namespace cbic
