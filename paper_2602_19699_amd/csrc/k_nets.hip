// Biased initial-state selection and the actor warm start (paper Sec. II,
// III-C/D): std-critic scoring of candidate initial states, selection of the
// N highest scores, and closed-loop rollouts of the system under the actor.
#include <hip/hip_ext.h>

#include <cmath>
#include <cstring>
#include <mutex>

#include "dev_systems.hpp"
#include "nets.hpp"
#include "runtime.hpp"

namespace cbic {

namespace {

#define HIP_TRY(expr)                                                   \
  do {                                                                  \
    hipError_t e_ = (expr);                                             \
    if (e_ != hipSuccess) {                                             \
      set_error("%s failed: %s", #expr, hipGetErrorString(e_));         \
      return CBIC_E_HIP;                                                \
    }                                                                   \
  } while (0)

constexpr int kNetWG = 256;  // four waves of 16 samples

// Dynamic LDS beyond 64 KiB (the largest networks take up to 79 KiB of the
// CU's 160 KiB) has to be allowed per kernel before the launch.
template <class K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(bytes));
}

// blocks of `per` that hold n (without the overflow of rounding n up first: n
// goes up to 2^31 - 1)
__host__ __device__ constexpr int blocks_of(int n, int per) { return n / per + (n % per != 0); }

__device__ __forceinline__ void sel_clear(uint32_t* __restrict__ sc, int N);

// score[b] = net(x_b, tau_b), tau_b = (T_max - T_b) / T_max (FP64 inputs
// rounded to FP32, as the network computes in FP32); without T the network
// takes the state alone.  16 candidates per wave.
template <int W, int ACT>
__global__ void __launch_bounds__(kNetWG) mlp_score(MlpDev net, MlpLds L, int B, int n,
                                                    const double* __restrict__ x, const int32_t* __restrict__ T,
                                                    int Tmax, float* __restrict__ score, uint32_t* __restrict__ sc,
                                                    int N) {
  // the selection's scratch, for the launches after this one
  if (sc && blockIdx.x == 0) sel_clear(sc, N);
  extern __shared__ float lds[];
  mlp_stage(net, L, lds);
  const int lane = threadIdx.x & 63;
  const int b = (blockIdx.x * (kNetWG / 64) + (threadIdx.x >> 6)) * 16 + (lane & 15);
  const bool valid = b < B;
  const double* xb = x + size_t(valid ? b : 0) * n;
  const float tau = (T && valid) ? float(Tmax - T[b]) * (1.0f / float(Tmax)) : 0.0f;
  const nf4 y = mlp_tile<W, 0, ACT>(net, L, lds, [&](int s, int g) {
    const int f = 4 * s + g;
    return !valid ? 0.0f : (f < n ? float(xb[f]) : (f == n && T ? tau : 0.0f));
  });
  if (valid && lane < 16) score[b] = y[0];
}

// out[b][:] = net(in[b][:]) for FP32 rows, 16 rows per wave.
template <int W, int ACT>
__global__ void __launch_bounds__(kNetWG) mlp_rows(MlpDev net, MlpLds L, int B, const float* __restrict__ in,
                                                   float* __restrict__ out) {
  extern __shared__ float lds[];
  mlp_stage(net, L, lds);
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int b = (blockIdx.x * (kNetWG / 64) + (threadIdx.x >> 6)) * 16 + (lane & 15);
  const bool valid = b < B;
  const float* ib = in + size_t(valid ? b : 0) * net.in_dim;
  const nf4 y = mlp_tile<W, 0, ACT>(net, L, lds, [&](int s, int gg) {
    const int f = 4 * s + gg;
    return valid && f < net.in_dim ? ib[f] : 0.0f;
  });
  if (valid)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * g + r < net.out_dim) out[size_t(b) * net.out_dim + 4 * g + r] = y[r];
}

// mlp_score and mlp_rows with the weights in registers (MlpRegs), for networks
// of one or two hidden layers and 5..8 inputs: a wave loads them once and
// takes every nwaves-th tile of 16 samples.  Bound by issue: 88 MFMA of 32
// cycles and about 340 vector instructions (half of them the activations) per
// tile of a 64-64 network.  163840 candidates: 27 us (68 TFLOP/s with the
// padding), 47 us with the weights staged in LDS by every workgroup of four
// tiles; 3000 candidates 5.6 us against 13.6.
template <int W, int ACT, int DEPTH>
__global__ void __launch_bounds__(kNetWG, 3) mlp_score_r(MlpDev net, int B, int n, const double* __restrict__ x,
                                                         const int32_t* __restrict__ T, int Tmax,
                                                         float* __restrict__ score, uint32_t* __restrict__ sc, int N) {
  // the selection's scratch, for the launches after this one
  if (sc && blockIdx.x == 0) sel_clear(sc, N);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int nwaves = gridDim.x * (kNetWG / 64), tiles = blocks_of(B, 16);
  MlpRegs<W, DEPTH> w;
  w.load(net, lane);
  const float inv_T = 1.0f / float(Tmax);
  for (int tile = blockIdx.x * (kNetWG / 64) + (threadIdx.x >> 6); tile < tiles; tile += nwaves) {
    const int b = tile * 16 + c;
    const bool valid = b < B;
    const double* xb = x + size_t(valid ? b : 0) * n;
    const float tau = (T && valid) ? float(Tmax - T[b]) * inv_T : 0.0f;
    float f[kRegIn4 / 4];
#pragma unroll
    for (int s = 0; s < kRegIn4 / 4; ++s) {
      const int i = 4 * s + g;
      f[s] = !valid ? 0.0f : (i < n ? float(xb[i]) : (i == n && T ? tau : 0.0f));
    }
    const nf4 y = w.template eval<ACT>(f, net.out_act, net.out_scale);
    if (valid && lane < 16) score[b] = y[0];
  }
}

template <int W, int ACT, int DEPTH>
__global__ void __launch_bounds__(kNetWG, 3) mlp_rows_r(MlpDev net, int B, const float* __restrict__ in,
                                                        float* __restrict__ out) {
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int nwaves = gridDim.x * (kNetWG / 64), tiles = blocks_of(B, 16);
  MlpRegs<W, DEPTH> w;
  w.load(net, lane);
  for (int tile = blockIdx.x * (kNetWG / 64) + (threadIdx.x >> 6); tile < tiles; tile += nwaves) {
    const int b = tile * 16 + c;
    const bool valid = b < B;
    const float* ib = in + size_t(valid ? b : 0) * net.in_dim;
    float f[kRegIn4 / 4];
#pragma unroll
    for (int s = 0; s < kRegIn4 / 4; ++s) f[s] = valid && 4 * s + g < net.in_dim ? ib[4 * s + g] : 0.0f;
    const nf4 y = w.template eval<ACT>(f, net.out_act, net.out_scale);
    if (valid)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (4 * g + r < net.out_dim) out[size_t(b) * net.out_dim + 4 * g + r] = y[r];
  }
}

// whether the register kernels take a network: their loops are unrolled for
// eight padded inputs, and a third hidden layer would leave one wave per SIMD
bool regs_take(const MlpDev& d) { return (d.in_dim + 3) / 4 * 4 == kRegIn4 && d.depth <= 2; }
// blocks for B samples: three waves per SIMD at most, then several tiles a wave
int reg_blocks(int B, int device) {
  const int want = blocks_of(B, kNetWG / 4), most = 3 * cu_count(device);
  return want < most ? want : most;
}

// ------------------------------------------------------------------ selection
// Order-preserving key of a score: a larger score has a larger key; -0 and +0
// share a key; NaN gets the smallest key.
__device__ __forceinline__ uint32_t score_key(float s) {
  if (!(s == s)) return 0u;
  if (s == 0.0f) s = 0.0f;
  const uint32_t u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix sum of v over the workgroup's WG threads (in thread
// order) and the workgroup's total; `wtot` holds one slot per wave.
template <int WG>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* wtot, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  if (lane == 63) wtot[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < WG / 64; ++w) {
    const uint32_t t = wtot[w];
    before += w < wave ? t : 0u;
    total += t;
  }
  __syncthreads();
  return before + inc - v;
}

// The N highest scores of Bc, in ascending index order (equal scores: lower
// index first): a radix select of the N-th largest key (11 + 11 + 10 bits)
// and an order-preserving compaction that also gathers the selected rows of
// x (n wide) and T.  Up to kSelSmall keys one workgroup does it all with the
// keys in registers (sel_small).  Larger sets are spread over blocks of
// kSelChunk keys, and the block that finishes a pass last does the pass's
// one-block part, so that a pass is one launch; the scoring kernel before them
// clears the scratch.  Scratch (uint32): hist [2048], state {prefix, mask, left,
// blocks done} at kSelState, then per block: greater count, equal count,
// output base, tie base.  Launch- and latency-bound: 163840 keys take five
// launches and 41 us, 3000 keys one launch and 13 us; with a launch of its own
// for every part it was ten launches, 59 and 45 us.  16384 keys (the most that
// 1024 threads keep in registers) still take less in one workgroup than 16385
// over the chip: scoring and selection of a tenth 28 against 48 us, of half 40
// against 52.
constexpr int kSelWG = 256, kSelE = 8, kSelChunk = kSelWG * kSelE;
constexpr int kSelState = 2048, kSelBlocks = 2056;
constexpr int kSmallWG = 1024, kSmallE = 16, kSelSmall = kSmallWG * kSmallE;

// cleared scratch for a selection of N, by one block of any size
__device__ __forceinline__ void sel_clear(uint32_t* __restrict__ sc, int N) {
  for (int i = threadIdx.x; i < kSelBlocks; i += blockDim.x) sc[i] = i == kSelState + 2 ? uint32_t(N) : 0u;
}

// The digit of the left-th largest key from the histogram h[0..nb) of the
// remaining keys' digits (WG threads; nb a multiple of WG): *bin, and in *rest
// the keys still to take within that bin.  The keys in the bins above a
// thread's own come from a suffix sum over the threads.
template <int WG>
__device__ __forceinline__ void sel_digit(const uint32_t* h, uint32_t nb, uint32_t left, uint32_t* wtot,
                                          uint32_t* bin, uint32_t* rest) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int per = int(nb) / WG;
  uint32_t mine = 0;
  for (int j = 0; j < per; ++j) mine += h[per * t + j];
  uint32_t inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_down(inc, o, 64);
    if (lane + o < 64) inc += u;
  }
  if (lane == 0) wtot[wave] = inc;
  if (t == 0) {
    *bin = 0u;
    *rest = left;
  }
  __syncthreads();
  uint32_t above = inc - mine;
#pragma unroll
  for (int w = 0; w < WG / 64; ++w) above += w > wave ? wtot[w] : 0u;
  for (int j = per - 1; j >= 0; --j) {
    const uint32_t c = h[per * t + j];
    if (above < left && left <= above + c) {
      *bin = uint32_t(per * t + j);
      *rest = left - above;
    }
    above += c;
  }
  __syncthreads();
}

// What the blocks of a pass tell the last one passes through device-scope
// atomics alone: an update returns a value that the thread waits for (so it
// has taken place, at the one point all dies of the chip share, before the
// block counts itself done), and the last block reads with atomic loads.  A
// fence instead would write back and invalidate the die's whole L2 for every
// block (a pass over 163840 keys 14 us; with the returned values 9 us).
__device__ __forceinline__ uint32_t sel_add(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t sel_put(uint32_t* p, uint32_t v) {
  return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t sel_read(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// whether this block is the last of the grid's G to come here; `seen` gathers
// the values its updates returned
__device__ __forceinline__ bool sel_last(uint32_t* sc, int G, uint32_t* flag, uint32_t seen) {
  asm volatile("" ::"v"(seen) : "memory");  // the returned values have arrived
  __syncthreads();
  if (threadIdx.x == 0)
    *flag = __hip_atomic_fetch_add(&sc[kSelState + 3], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == uint32_t(G) - 1u;
  __syncthreads();
  return *flag != 0u;
}

// One pass: the digits of the keys that match the prefix so far; the last
// block finds the next digit and clears the histogram for the next pass.
__global__ void __launch_bounds__(kSelWG) sel_hist(const float* __restrict__ score, int Bc, uint32_t* __restrict__ sc,
                                                   int shift, uint32_t nb) {
  __shared__ uint32_t h[2048];
  __shared__ uint32_t wtot[kSelWG / 64], s_bin, s_left, s_flag;
  const int t = threadIdx.x;
  for (uint32_t i = t; i < nb; i += kSelWG) h[i] = 0u;
  const uint32_t prefix = sc[kSelState], mask = sc[kSelState + 1], left = sc[kSelState + 2];
  __syncthreads();
  const int base = blockIdx.x * kSelChunk;
  uint32_t k[kSelE];
#pragma unroll
  for (int j = 0; j < kSelE; ++j) {
    const int i = base + j * kSelWG + t;
    k[j] = i < Bc ? score_key(score[i]) : 0u;
  }
#pragma unroll
  for (int j = 0; j < kSelE; ++j)
    if (base + j * kSelWG + t < Bc && (k[j] & mask) == prefix) atomicAdd(&h[(k[j] >> shift) & (nb - 1u)], 1u);
  __syncthreads();
  uint32_t got[2048 / kSelWG] = {}, seen = 0;  // (all issued before the first is waited for)
#pragma unroll
  for (int j = 0; j < 2048 / kSelWG; ++j) {
    const uint32_t i = j * kSelWG + t;
    if (i < nb && h[i]) got[j] = sel_add(&sc[i], h[i]);
  }
#pragma unroll
  for (int j = 0; j < 2048 / kSelWG; ++j) seen |= got[j];
  if (!sel_last(sc, int(gridDim.x), &s_flag, seen)) return;
  for (uint32_t i = t; i < nb; i += kSelWG) {
    h[i] = sel_read(&sc[i]);
    sc[i] = 0u;
  }
  __syncthreads();
  sel_digit<kSelWG>(h, nb, left, wtot, &s_bin, &s_left);
  if (t == 0) {
    sc[kSelState] = prefix | (s_bin << shift);
    sc[kSelState + 1] = mask | ((nb - 1u) << shift);
    sc[kSelState + 2] = s_left;
    sc[kSelState + 3] = 0u;
  }
}

// Per block: keys above the threshold key and keys equal to it; the last
// block forms each block's first output position and first tie rank.
__global__ void __launch_bounds__(kSelWG) sel_count(const float* __restrict__ score, int Bc,
                                                    uint32_t* __restrict__ sc) {
  __shared__ uint32_t wtot[kSelWG / 64], s_flag;
  const int t = threadIdx.x, G = int(gridDim.x);
  const uint32_t thr = sc[kSelState], left = sc[kSelState + 2];
  const int base = blockIdx.x * kSelChunk;
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < kSelE; ++j) {
    const int i = base + j * kSelWG + t;
    const uint32_t k = i < Bc ? score_key(score[i]) : 0u;
    gt += (i < Bc && k > thr) ? 1u : 0u;
    eq += (i < Bc && k == thr) ? 1u : 0u;
  }
  uint32_t tg, te, tt;
  block_scan<kSelWG>(gt, wtot, tg);
  block_scan<kSelWG>(eq, wtot, te);
  uint32_t seen = 0;
  if (t == 0) {
    const uint32_t a = sel_put(&sc[kSelBlocks + blockIdx.x], tg), b = sel_put(&sc[kSelBlocks + G + blockIdx.x], te);
    seen = a | b;
  }
  if (!sel_last(sc, G, &s_flag, seen)) return;
  uint32_t out_run = 0, tie_run = 0;
  for (int c = 0; c < G; c += kSelWG) {
    const int b = c + t;
    const uint32_t bg = b < G ? sel_read(&sc[kSelBlocks + b]) : 0u, be = b < G ? sel_read(&sc[kSelBlocks + G + b]) : 0u;
    const uint32_t tie0 = tie_run + block_scan<kSelWG>(be, wtot, te);
    const uint32_t ties_taken = tie0 >= left ? 0u : min(be, left - tie0);
    const uint32_t out0 = out_run + block_scan<kSelWG>(bg + ties_taken, wtot, tt);
    if (b < G) {
      sc[kSelBlocks + 2 * G + b] = out0;
      sc[kSelBlocks + 3 * G + b] = tie0;
    }
    out_run += tt;
    tie_run += te;
  }
}

// The rows of the selected indices sel[p0..p1) (written by this block before
// a barrier), by the block's threads, element by element.
__device__ __forceinline__ void sel_gather(const int32_t* sel, int p0, int p1, int n, const double* __restrict__ x,
                                           const int32_t* __restrict__ T, double* __restrict__ xs,
                                           int32_t* __restrict__ Ts) {
  if (xs)
    for (long e = long(p0) * n + threadIdx.x; e < long(p1) * n; e += blockDim.x) {
      const int p = int(e / n), q = int(e - long(p) * n);
      xs[e] = x[size_t(sel[p]) * n + q];
    }
  if (Ts)
    for (int p = p0 + threadIdx.x; p < p1; p += blockDim.x) Ts[p] = T[sel[p]];
}

// The selected among a thread's E consecutive keys from i0: bit j of `gt`
// for a key above the threshold, of `eq` for one equal to it.
template <int E>
__device__ __forceinline__ void sel_flags(const uint32_t (&k)[E], int i0, int Bc, uint32_t thr, uint32_t& gt,
                                          uint32_t& eq) {
  gt = 0;
  eq = 0;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    if (i0 + j < Bc && k[j] > thr) gt |= 1u << j;
    if (i0 + j < Bc && k[j] == thr) eq |= 1u << j;
  }
}
// of those flags the ones taken: all above, and the ties whose rank (from
// `rank` on) is below `left`
template <int E>
__device__ __forceinline__ uint32_t sel_take(uint32_t gt, uint32_t eq, uint32_t rank, uint32_t left) {
  uint32_t take = gt;
#pragma unroll
  for (int j = 0; j < E; ++j)
    if ((eq >> j) & 1u) {
      if (rank < left) take |= 1u << j;
      ++rank;
    }
  return take;
}

// Per block: write the selected indices (and rows) in ascending index order;
// thread t handles keys [base + E t, base + E t + E).
__global__ void __launch_bounds__(kSelWG) sel_scatter(const float* __restrict__ score, int Bc, int N,
                                                      int32_t* __restrict__ sel, int n, const double* __restrict__ x,
                                                      const int32_t* __restrict__ T, double* __restrict__ xs,
                                                      int32_t* __restrict__ Ts, const uint32_t* __restrict__ sc,
                                                      int G) {
  __shared__ uint32_t wtot[kSelWG / 64];
  const int t = threadIdx.x;
  const uint32_t thr = sc[kSelState], left = sc[kSelState + 2];
  const int i0 = blockIdx.x * kSelChunk + kSelE * t;
  uint32_t k[kSelE], gt, eq, te, tt;
#pragma unroll
  for (int j = 0; j < kSelE; ++j) k[j] = i0 + j < Bc ? score_key(score[i0 + j]) : 0u;
  sel_flags<kSelE>(k, i0, Bc, thr, gt, eq);
  const uint32_t rank = sc[kSelBlocks + 3 * G + blockIdx.x] + block_scan<kSelWG>(__popc(eq), wtot, te);
  const uint32_t take = sel_take<kSelE>(gt, eq, rank, left);
  const uint32_t first = sc[kSelBlocks + 2 * G + blockIdx.x];
  uint32_t pos = first + block_scan<kSelWG>(__popc(take), wtot, tt);
#pragma unroll
  for (int j = 0; j < kSelE; ++j)
    if ((take >> j) & 1u) {
      if (pos < uint32_t(N)) sel[pos] = i0 + j;
      ++pos;
    }
  __syncthreads();
  sel_gather(sel, int(first), min(int(first + tt), N), n, x, T, xs, Ts);
}

// The whole selection in one workgroup for Bc <= kSelSmall.
__global__ void __launch_bounds__(kSmallWG) sel_small(const float* __restrict__ score, int Bc, int N,
                                                      int32_t* __restrict__ sel, int n, const double* __restrict__ x,
                                                      const int32_t* __restrict__ T, double* __restrict__ xs,
                                                      int32_t* __restrict__ Ts) {
  __shared__ uint32_t h[2048];
  __shared__ uint32_t wtot[kSmallWG / 64], s_bin, s_left;
  const int t = threadIdx.x, i0 = kSmallE * t;
  uint32_t k[kSmallE];
#pragma unroll
  for (int j = 0; j < kSmallE; ++j) k[j] = i0 + j < Bc ? score_key(score[i0 + j]) : 0u;
  uint32_t prefix = 0, mask = 0, left = uint32_t(N);
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
    const uint32_t nb = pass < 2 ? 2048u : 1024u;
    for (uint32_t i = t; i < nb; i += kSmallWG) h[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallE; ++j)
      if (i0 + j < Bc && (k[j] & mask) == prefix) atomicAdd(&h[(k[j] >> shift) & (nb - 1u)], 1u);
    __syncthreads();
    sel_digit<kSmallWG>(h, nb, left, wtot, &s_bin, &s_left);
    prefix |= s_bin << shift;
    mask |= (nb - 1u) << shift;
    left = s_left;
    __syncthreads();
  }
  uint32_t gt, eq, te, tt;
  sel_flags<kSmallE>(k, i0, Bc, prefix, gt, eq);
  const uint32_t take = sel_take<kSmallE>(gt, eq, block_scan<kSmallWG>(__popc(eq), wtot, te), left);
  uint32_t pos = block_scan<kSmallWG>(__popc(take), wtot, tt);
#pragma unroll
  for (int j = 0; j < kSmallE; ++j)
    if ((take >> j) & 1u) {
      if (pos < uint32_t(N)) sel[pos] = i0 + j;
      ++pos;
    }
  __syncthreads();
  sel_gather(sel, 0, N, n, x, T, xs, Ts);
}

// ------------------------------------------------------------------ actor rollout
// Sixteen instances per workgroup of W / 16 waves: wave v evaluates the
// neurons 16 v .. 16 v + 15 of every hidden layer for all sixteen and keeps
// those weights in registers; a layer's activations pass through LDS.  One
// wave (another one from block to block) also evaluates the output layer,
// keeps the instances' states (four lanes per instance, redundantly), steps
// the FP64 dynamics and publishes the next inputs.  The block runs until its
// longest horizon, so ragged batches are taken in horizon order (perm, longest
// first) and a block holds similar horizons.  Outputs are zero past each
// horizon (all zero for a horizon outside 1..T_max).
//
// Bound: the serial chain of one step (the matrix products of the layers, 16
// dependent MFMA each, the activations between them and the dynamics), which
// the split over waves shortens to a quarter of its products and activations;
// the products are those of one wave evaluating the network alone, in the same
// order.  64-64 network, horizons up to 100: a step alone takes 0.87 us (2.0 us
// with one wave per 16 instances and the weights read from LDS every step);
// 16384 point-mass instances, horizons 1..100: 172 us against 278.
template <class Sys, int W, int ACT>
__global__ void __launch_bounds__(4 * W) actor_rollout(const double* __restrict__ prm, MlpDev net, int B, int Tmax,
                                                       const int32_t* __restrict__ Tin,
                                                       const int32_t* __restrict__ perm,
                                                       const double* __restrict__ x0, double* __restrict__ U,
                                                       double* __restrict__ X) {
  constexpr int N = Sys::N, M = Sys::M;
  constexpr int IN4 = (N + 1 + 3) & ~3;
  constexpr int NW = W / 16, KS = W / 4, HL = 3;  // waves, K steps of a hidden layer, hidden layers beyond the first
  static_assert(M <= 4, "outputs of lane group 0");
  __shared__ nf4 hb[2][NW][64];
  __shared__ float feat[IN4][16];
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15, wv = threadIdx.x >> 6;
  // blocks 256 apart share a compute unit, whose SIMDs take a wave of each: the
  // leads, with the output layer and the dynamics on top, go to different ones
  const bool lead = wv == int(blockIdx.x + blockIdx.x / 256) % NW;
  // this wave's weights: neuron 16 wv + c (output c for the output layer) by
  // the K rows of lane group g
  float w0[IN4 / 4], wh[HL][KS], wo[KS];
  nf4 b0, bh[HL], bo;
  {
    const int in = net.in_dim, out = net.out_dim;
    const float* p = net.p;
#pragma unroll
    for (int s = 0; s < IN4 / 4; ++s) w0[s] = 4 * s + g < in ? p[(4 * s + g) * W + 16 * wv + c] : 0.0f;
    p += in * W;
#pragma unroll
    for (int r = 0; r < 4; ++r) b0[r] = p[16 * wv + 4 * g + r];
    p += W;
#pragma unroll
    for (int l = 0; l < HL; ++l)
      if (l + 1 < net.depth) {
#pragma unroll
        for (int s = 0; s < KS; ++s) wh[l][s] = p[(16 * (s >> 2) + 4 * g + (s & 3)) * W + 16 * wv + c];
        p += W * W;
#pragma unroll
        for (int r = 0; r < 4; ++r) bh[l][r] = p[16 * wv + 4 * g + r];
        p += W;
      }
#pragma unroll
    for (int s = 0; s < KS; ++s) wo[s] = c < out ? p[(16 * (s >> 2) + 4 * g + (s & 3)) * out + c] : 0.0f;
    p += W * out;
#pragma unroll
    for (int r = 0; r < 4; ++r) bo[r] = 4 * g + r < out ? p[4 * g + r] : 0.0f;
  }
  const int slot = blockIdx.x * 16 + c;
  const bool valid = slot < B;
  const int b = valid ? (perm ? perm[slot] : slot) : 0;
  const typename Sys::template Model<double> mdl{prm};
  const int Tr = valid ? (Tin ? Tin[b] : Tmax) : 0;
  const int T = (Tr < 1 || Tr > Tmax) ? 0 : Tr;
  int Tw = T;  // the block's longest horizon (every wave holds the same sixteen)
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) Tw = max(Tw, __shfl_xor(Tw, o, 64));
  // zeros past the horizons, a wave per instance
  for (int i = wv; i < 16; i += NW) {
    if (int(blockIdx.x) * 16 + i >= B) break;
    const int bi = __shfl(b, i, 64), Ti = __shfl(T, i, 64);
    double* u = U + size_t(bi) * Tmax * M;
    for (int q = Ti * M + lane; q < Tmax * M; q += 64) u[q] = 0.0;
    if (X) {
      double* xx = X + size_t(bi) * (Tmax + 1) * N;
      for (int q = (Ti + 1) * N + lane; q < (Tmax + 1) * N; q += 64) xx[q] = 0.0;
    }
  }
  const bool writer = lead && valid && g == 0;
  double* Ub = U + size_t(b) * Tmax * M;
  double* Xb = X ? X + size_t(b) * (Tmax + 1) * N : nullptr;
  double x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = T > 0 ? x0[size_t(b) * N + i] : 0.0;
  if (writer && Xb)
#pragma unroll
    for (int i = 0; i < N; ++i) Xb[i] = x[i];
  const float inv_T = 1.0f / float(Tmax);
  // the inputs of step k: lane group g publishes features g, g + 4, ...
  auto publish = [&](int k) {
#pragma unroll
    for (int s = 0; s < IN4 / 4; ++s) {
      float f[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * s + q;
        f[q] = i < N ? float(x[i < N ? i : 0]) : (i == N ? float(Tmax - T + k) * inv_T : 0.0f);
      }
      feat[4 * s + g][c] = g == 0 ? f[0] : (g == 1 ? f[1] : (g == 2 ? f[2] : f[3]));
    }
  };
  if (lead) publish(0);
  __syncthreads();
  for (int k = 0; k < Tw; ++k) {
    nf4 h = b0;
#pragma unroll
    for (int s = 0; s < IN4 / 4; ++s) h = mfma_f32_16x16x4(w0[s], feat[4 * s + g][c], h);
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = mlp_act<ACT>(h[r]);
    hb[0][wv][lane] = h;
    __syncthreads();
#pragma unroll
    for (int l = 0; l < HL; ++l)
      if (l + 1 < net.depth) {
        nf4 o = bh[l], hin[NW];
#pragma unroll
        for (int t = 0; t < NW; ++t) hin[t] = hb[l & 1][t][lane];
#pragma unroll
        for (int s = 0; s < KS; ++s) o = mfma_f32_16x16x4(wh[l][s], hin[s >> 2][s & 3], o);
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = mlp_act<ACT>(o[r]);
        hb[(l + 1) & 1][wv][lane] = o;
        __syncthreads();
      }
    if (lead) {
      nf4 y = bo, hin[NW];
#pragma unroll
      for (int t = 0; t < NW; ++t) hin[t] = hb[(net.depth - 1) & 1][t][lane];
#pragma unroll
      for (int s = 0; s < KS; ++s) y = mfma_f32_16x16x4(wo[s], hin[s >> 2][s & 3], y);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = mlp_out(y[r], net.out_act, net.out_scale);
      // outputs 0..M-1 of instance c sit in lane c (group 0), registers 0..M-1
      double u[M];
#pragma unroll
      for (int o = 0; o < M; ++o) u[o] = double(__shfl(y[o], c, 64));
      if (k < T) {
        double xn[N];
        mdl.dyn(x, u, xn);
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = xn[i];
        if (writer) {
#pragma unroll
          for (int i = 0; i < M; ++i) Ub[size_t(k) * M + i] = u[i];
          if (Xb)
#pragma unroll
            for (int i = 0; i < N; ++i) Xb[size_t(k + 1) * N + i] = x[i];
        }
      }
      publish(k + 1);
    }
    __syncthreads();
  }
}

// The same rollout with a whole network per wave: 16 instances per wave, four
// waves per workgroup, the weights read from LDS every step; bit for bit the
// results of actor_rollout.  A step of a wave alone takes longer (one wave
// issues the whole network), but a batch needs a quarter of the waves (half of
// them with 32 neurons) and no barriers, which wins once the chip is full of
// waves (wave_per_tile).
template <class Sys, int W, int ACT>
__global__ void __launch_bounds__(kNetWG) actor_rollout_wave(const double* __restrict__ prm, MlpDev net, MlpLds L,
                                                             int B, int Tmax, const int32_t* __restrict__ Tin,
                                                             const int32_t* __restrict__ perm,
                                                             const double* __restrict__ x0, double* __restrict__ U,
                                                             double* __restrict__ X) {
  constexpr int N = Sys::N, M = Sys::M;
  constexpr int IN4 = (N + 1 + 3) & ~3;
  static_assert(M <= 4, "outputs of lane group 0");
  extern __shared__ float lds[];
  mlp_stage(net, L, lds);
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  const int slot = (blockIdx.x * (kNetWG / 64) + (threadIdx.x >> 6)) * 16 + c;
  const bool valid = slot < B;
  const int b = valid ? (perm ? perm[slot] : slot) : 0;
  const typename Sys::template Model<double> mdl{prm};
  const int Tr = valid ? (Tin ? Tin[b] : Tmax) : 0;
  const int T = (Tr < 1 || Tr > Tmax) ? 0 : Tr;
  int Tw = T;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) Tw = max(Tw, __shfl_xor(Tw, o, 64));
  const bool writer = valid && g == 0;
  double* Ub = U + size_t(valid ? b : 0) * Tmax * M;
  double* Xb = X ? X + size_t(valid ? b : 0) * (Tmax + 1) * N : nullptr;
  double x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = T > 0 ? x0[size_t(b) * N + i] : 0.0;
  if (writer && Xb)
#pragma unroll
    for (int i = 0; i < N; ++i) Xb[i] = x[i];
  const float inv_T = 1.0f / float(Tmax);
  for (int k = 0; k < Tw; ++k) {
    float f[IN4];
#pragma unroll
    for (int i = 0; i < IN4; ++i) f[i] = i < N ? float(x[i < N ? i : 0]) : (i == N ? float(Tmax - T + k) * inv_T : 0.0f);
    const nf4 y = mlp_tile<W, IN4, ACT>(net, L, lds, [&](int s, int gg) {
      return gg == 0 ? f[4 * s] : (gg == 1 ? f[4 * s + 1] : (gg == 2 ? f[4 * s + 2] : f[4 * s + 3]));
    });
    // outputs 0..M-1 of instance c sit in lane c (group 0), registers 0..M-1
    double u[M];
#pragma unroll
    for (int o = 0; o < M; ++o) u[o] = double(__shfl(y[o], c, 64));
    if (k < T) {
      double xn[N];
      mdl.dyn(x, u, xn);
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] = xn[i];
      if (writer) {
#pragma unroll
        for (int i = 0; i < M; ++i) Ub[size_t(k) * M + i] = u[i];
        if (Xb)
#pragma unroll
          for (int i = 0; i < N; ++i) Xb[size_t(k + 1) * N + i] = x[i];
      }
    }
  }
  if (writer) {
    for (int k = T; k < Tmax; ++k)
#pragma unroll
      for (int i = 0; i < M; ++i) Ub[size_t(k) * M + i] = 0.0;
    if (Xb)
      for (int k = T + 1; k <= Tmax; ++k)
#pragma unroll
        for (int i = 0; i < N; ++i) Xb[size_t(k) * N + i] = 0.0;
  }
}

// Which of the two: with one horizon the wave kernel takes a step's time for
// every 16384 instances begun (one wave per SIMD), the other one grows with the
// batch, so it is taken while less than a share of the last 16384 is filled.
// Ragged batches empty as they go, and the split pays up to larger ones.  The
// lines lie where the two measured alike at horizons up to 60; the arm's
// dynamics, which one wave of a block steps while the others wait, bring them
// down.  us, split / wave: 64-64 network, point mass, one horizon: B 8192 93 /
// 164, 16384 184 / 165, 20480 211 / 261, 32768 331 / 264; ragged: 16384 113 / 177, 32768 292 /
// 306, 65536 550 / 515; arm, one horizon: 16384 263 / 209, 65536 918 / 601; one layer of
// 32, arm: 4096 80 / 86, 8192 115 / 87.
bool wave_per_tile(bool arm, int W, int depth, int B, bool ragged) {
  const int d = depth < 4 ? depth - 1 : 3, w = W == 64;
  if (ragged) {
    static constexpr int most[2][2][4] = {{{1, 8, 16, 16}, {5, 8, 12, 12}}, {{1, 3, 6, 6}, {5, 6, 10, 12}}};  // of 4096
    return B > 4096 * most[arm][w][d];
  }
  static constexpr int share[2][2][4] = {{{25, 25, 70, 75}, {50, 75, 80, 85}}, {{25, 25, 25, 25}, {50, 70, 75, 80}}};  // %
  const int rounds = blocks_of(B, 16384);
  return long(B) * 100 > long(share[arm][w][d]) * 16384 * rounds;
}

template <class Sys, int W, int ACT>
hipError_t launch_actor_k(const double* prm, const MlpDev& net, const MlpLds& L, int B, int Tmax, const int32_t* d_T,
                          const int32_t* perm, const double* x0, double* U, double* X, hipStream_t st) {
  if (wave_per_tile(Sys::kSemiImplicit, W, net.depth, B, d_T != nullptr)) {
    const size_t lds = size_t(L.total()) * sizeof(float);
    hipError_t e = allow_lds(actor_rollout_wave<Sys, W, ACT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((actor_rollout_wave<Sys, W, ACT>), dim3(blocks_of(B, kNetWG / 4)), dim3(kNetWG), lds,
                       st, prm, net, L, B, Tmax, d_T, perm, x0, U, X);
  } else {
    hipLaunchKernelGGL((actor_rollout<Sys, W, ACT>), dim3(blocks_of(B, 16)), dim3(4 * W), 0, st, prm, net, B, Tmax, d_T,
                       perm, x0, U, X);
  }
  return hipGetLastError();
}

template <class Sys>
hipError_t launch_actor(const double* prm, const MlpDev& net, const MlpLds& L, int B, int Tmax, const int32_t* d_T,
                        const int32_t* perm, const double* x0, double* U, double* X, hipStream_t st) {
#define CBIC_ACTOR(WW, AA) launch_actor_k<Sys, WW, AA>(prm, net, L, B, Tmax, d_T, perm, x0, U, X, st)
  if (L.W == 32) return net.act == 0 ? CBIC_ACTOR(32, 0) : (net.act == 1 ? CBIC_ACTOR(32, 1) : CBIC_ACTOR(32, 2));
  return net.act == 0 ? CBIC_ACTOR(64, 0) : (net.act == 1 ? CBIC_ACTOR(64, 1) : CBIC_ACTOR(64, 2));
#undef CBIC_ACTOR
}

int64_t param_count(const cbic_mlp& m) {
  const int64_t W = m.width;
  return m.in_dim * W + W + (m.depth - 1) * (W * W + W) + W * m.out_dim + m.out_dim;
}

cbic_status check_mlp(const cbic_mlp* m) {
  if (!m) {
    set_error("network description is NULL");
    return CBIC_E_INVALID;
  }
  if (m->in_dim < 1 || m->in_dim > 64 || (m->width != 32 && m->width != 64) || m->depth < 1 || m->depth > 4 ||
      m->out_dim < 1 || m->out_dim > 16 || m->act < CBIC_ACT_TANH || m->act > CBIC_ACT_RELU ||
      m->out_act < CBIC_OUT_LINEAR || m->out_act > CBIC_OUT_SOFTPLUS || !std::isfinite(m->out_scale)) {
    set_error("network must have in_dim 1..64, width 32 or 64, depth 1..4, out_dim 1..16, known activations "
              "and a finite out_scale");
    return CBIC_E_INVALID;
  }
  return CBIC_OK;
}

MlpDev dev_mlp(const cbic_mlp& m) {
  return MlpDev{m.params, m.in_dim, m.depth, m.out_dim, m.act, m.out_act, float(m.out_scale)};
}

}  // namespace
}  // namespace cbic

using namespace cbic;

extern "C" {

cbic_status cbic_mlp_param_count(const cbic_mlp* net, int64_t* count) {
  if (cbic_status st = check_mlp(net)) return st;
  if (!count) {
    set_error("count is NULL");
    return CBIC_E_INVALID;
  }
  *count = param_count(*net);
  return CBIC_OK;
}

cbic_status cbic_mlp_forward(cbic_context* ctx, const cbic_mlp* net, int32_t B, const float* d_in, float* d_out,
                             void* stream) {
  if (cbic_status st = check_mlp(net)) return st;
  if (!ctx || !net->params || (B > 0 && (!d_in || !d_out)) || B < 0) {
    set_error("ctx, params, d_in and d_out are required and B >= 0");
    return CBIC_E_INVALID;
  }
  if (B == 0) return CBIC_OK;
  HIP_TRY(hipSetDevice(ctx->device));
  (void)hipGetLastError();  // launch errors below are this call's, not a stale one
  hipStream_t st = static_cast<hipStream_t>(stream);
  const MlpDev d = dev_mlp(*net);
  const MlpLds L = mlp_lds(net->in_dim, net->width, net->depth, net->out_dim);
  const dim3 grid(blocks_of(B, kNetWG / 4)), rgrid(reg_blocks(B, ctx->device)), block(kNetWG);
  const bool regs = regs_take(d);
  const size_t lds = size_t(L.total()) * sizeof(float);
#define CBIC_ROWS(WW, AA)                                                                                    \
  do {                                                                                                       \
    if (regs && d.depth == 1) hipLaunchKernelGGL((mlp_rows_r<WW, AA, 1>), rgrid, block, 0, st, d, B, d_in, d_out); \
    else if (regs) hipLaunchKernelGGL((mlp_rows_r<WW, AA, 2>), rgrid, block, 0, st, d, B, d_in, d_out);      \
    else {                                                                                                   \
      HIP_TRY(allow_lds(mlp_rows<WW, AA>, lds));                                                             \
      hipLaunchKernelGGL((mlp_rows<WW, AA>), grid, block, lds, st, d, L, B, d_in, d_out);                    \
    }                                                                                                        \
  } while (0)
  if (net->width == 32) {
    if (net->act == 0) CBIC_ROWS(32, 0);
    else if (net->act == 1) CBIC_ROWS(32, 1);
    else CBIC_ROWS(32, 2);
  } else {
    if (net->act == 0) CBIC_ROWS(64, 0);
    else if (net->act == 1) CBIC_ROWS(64, 1);
    else CBIC_ROWS(64, 2);
  }
#undef CBIC_ROWS
  HIP_TRY(hipGetLastError());
  return CBIC_OK;
}

cbic_status cbic_bic_select(cbic_context* ctx, const cbic_mlp* net, int32_t Bc, int32_t n, const double* d_x,
                            const int32_t* d_T, int32_t T_max, int32_t N, float* d_score, int32_t* d_sel,
                            double* d_x_sel, int32_t* d_T_sel, void* stream) {
  if (cbic_status st = check_mlp(net)) return st;
  if (!ctx || !net->params || Bc < 1 || n < 1 || N < 0 || N > Bc || !d_x || !d_score || (N > 0 && !d_sel) ||
      (d_T && T_max < 1) || (d_T_sel && !d_T)) {
    set_error("ctx, params, d_x, d_score and d_sel are required (d_T with d_T_sel, T_max >= 1 with d_T); "
              "Bc >= 1, n >= 1, 0 <= N <= Bc");
    return CBIC_E_INVALID;
  }
  if (net->in_dim != n + (d_T ? 1 : 0) || net->out_dim != 1) {
    set_error("the std-critic must take %d inputs and give one output", n + (d_T ? 1 : 0));
    return CBIC_E_INVALID;
  }
  HIP_TRY(hipSetDevice(ctx->device));
  (void)hipGetLastError();  // launch errors below are this call's, not a stale one
  hipStream_t st = static_cast<hipStream_t>(stream);
  const MlpDev d = dev_mlp(*net);
  const MlpLds L = mlp_lds(net->in_dim, net->width, net->depth, net->out_dim);
  const dim3 grid(blocks_of(Bc, kNetWG / 4)), rgrid(reg_blocks(Bc, ctx->device)), block(kNetWG);
  const bool regs = regs_take(d);
  const size_t lds = size_t(L.total()) * sizeof(float);
  // scratch of the selection beyond one workgroup's; with or without it a
  // selection is ordered after the context's previous call on another stream,
  // and the next such call after it (a captured one that needs no scratch takes
  // its place in its graph alone)
  const int G = blocks_of(Bc, kSelChunk);
  uint32_t* sc = nullptr;
  std::unique_lock<std::mutex> lk(ctx->mu, std::defer_lock);
  bool ordered = N > 0;
  if (ordered && Bc <= kSelSmall) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess) (void)hipGetLastError();
    ordered = cs == hipStreamCaptureStatusNone;
  }
  if (ordered) {
    lk.lock();
    if (Bc > kSelSmall) {
      void* aux = nullptr;
      if (cbic_status e = context_aux(ctx, (size_t(kSelBlocks) + 4 * size_t(G)) * sizeof(uint32_t), &aux)) return e;
      sc = static_cast<uint32_t*>(aux);
    }
    if (ctx->have_last && ctx->last_stream != st) HIP_TRY(hipStreamWaitEvent(st, ctx->done_ev, 0));
  }
#define CBIC_SCORE(WW, AA)                                                                                      \
  do {                                                                                                          \
    if (regs && d.depth == 1)                                                                                   \
      hipLaunchKernelGGL((mlp_score_r<WW, AA, 1>), rgrid, block, 0, st, d, Bc, n, d_x, d_T, T_max, d_score, sc, N); \
    else if (regs)                                                                                              \
      hipLaunchKernelGGL((mlp_score_r<WW, AA, 2>), rgrid, block, 0, st, d, Bc, n, d_x, d_T, T_max, d_score, sc, N); \
    else {                                                                                                      \
      HIP_TRY(allow_lds(mlp_score<WW, AA>, lds));                                                               \
      hipLaunchKernelGGL((mlp_score<WW, AA>), grid, block, lds, st, d, L, Bc, n, d_x, d_T, T_max, d_score, sc, N); \
    }                                                                                                           \
  } while (0)
  if (net->width == 32) {
    if (net->act == 0) CBIC_SCORE(32, 0);
    else if (net->act == 1) CBIC_SCORE(32, 1);
    else CBIC_SCORE(32, 2);
  } else {
    if (net->act == 0) CBIC_SCORE(64, 0);
    else if (net->act == 1) CBIC_SCORE(64, 1);
    else CBIC_SCORE(64, 2);
  }
#undef CBIC_SCORE
  HIP_TRY(hipGetLastError());
  if (N > 0 && !sc) {
    // the event goes with the kernel's own completion: recorded after it, it
    // took 2.8 us of a 17.7 us call, so 0.9
    if (ordered)
      hipExtLaunchKernelGGL(sel_small, dim3(1), dim3(kSmallWG), 0, st, nullptr, ctx->done_ev, 0, d_score, Bc, N, d_sel,
                            n, d_x, d_T, d_x_sel, d_T_sel);
    else
      hipLaunchKernelGGL(sel_small, dim3(1), dim3(kSmallWG), 0, st, d_score, Bc, N, d_sel, n, d_x, d_T, d_x_sel,
                         d_T_sel);
  } else if (sc) {
    for (int pass = 0; pass < 3; ++pass)
      hipLaunchKernelGGL(sel_hist, dim3(G), dim3(kSelWG), 0, st, d_score, Bc, sc, pass == 0 ? 21 : (pass == 1 ? 10 : 0),
                         pass < 2 ? 2048u : 1024u);
    hipLaunchKernelGGL(sel_count, dim3(G), dim3(kSelWG), 0, st, d_score, Bc, sc);
    hipLaunchKernelGGL(sel_scatter, dim3(G), dim3(kSelWG), 0, st, d_score, Bc, N, d_sel, n, d_x, d_T, d_x_sel,
                       d_T_sel, sc, G);
  }
  HIP_TRY(hipGetLastError());
  if (ordered) {
    if (sc) HIP_TRY(hipEventRecord(ctx->done_ev, st));
    ctx->last_stream = st;
    ctx->have_last = true;
  }
  return CBIC_OK;
}

cbic_status cbic_actor_rollout(cbic_context* ctx, const cbic_system* sys, const cbic_mlp* actor, int32_t B,
                               int32_t T_max, const int32_t* d_T, const double* d_x0, double* d_U, double* d_X,
                               void* stream) {
  if (cbic_status st = check_mlp(actor)) return st;
  if (!ctx || !sys || !actor->params || B < 1 || T_max < 1 || !d_x0 || !d_U) {
    set_error("ctx, sys, params, d_x0 and d_U are required; B, T_max >= 1");
    return CBIC_E_INVALID;
  }
  if (actor->in_dim != sys->n + 1 || actor->out_dim != sys->m) {
    set_error("the actor must take n + 1 = %d inputs and give m = %d outputs", sys->n + 1, sys->m);
    return CBIC_E_INVALID;
  }
  HIP_TRY(hipSetDevice(ctx->device));
  (void)hipGetLastError();  // launch errors below are this call's, not a stale one
  hipStream_t st = static_cast<hipStream_t>(stream);
  const MlpDev d = dev_mlp(*actor);
  const MlpLds w = mlp_lds(actor->in_dim, actor->width, actor->depth, actor->out_dim);
  const bool known = sys->kind == CBIC_SYS_POINT_MASS || sys->kind == CBIC_SYS_PLANAR3 ||
                     (sys->kind == CBIC_SYS_LQ && ((sys->n == 2 && sys->m == 1) || (sys->n == 4 && sys->m == 2) ||
                                                   (sys->n == 6 && sys->m == 3)));
  if (!known) {
    set_error("no actor rollout for system kind %d (n=%d, m=%d)", sys->kind, sys->n, sys->m);
    return CBIC_E_UNSUPPORTED;
  }
  // a ragged batch is taken in horizon order (sorted on the device)
  std::lock_guard<std::mutex> lk(ctx->mu);
  int32_t* perm = nullptr;
  if (d_T) {
    const size_t hb = (size_t(T_max) + 1) * 4, hb_al = (hb + 255) / 256 * 256;
    void* aux = nullptr;
    if (cbic_status e = context_aux(ctx, hb_al + size_t(B) * 4, &aux)) return e;
    if (ctx->have_last && ctx->last_stream != st) HIP_TRY(hipStreamWaitEvent(st, ctx->done_ev, 0));
    int32_t* hist = static_cast<int32_t*>(aux);
    perm = reinterpret_cast<int32_t*>(static_cast<char*>(aux) + hb_al);
    HIP_TRY(launch_horizon_sort(d_T, B, T_max, hist, perm, st));
  }
  hipError_t e;
  if (sys->kind == CBIC_SYS_POINT_MASS) {
    e = launch_actor<PointMass>(sys->d_prm, d, w, B, T_max, d_T, perm, d_x0, d_U, d_X, st);
  } else if (sys->kind == CBIC_SYS_PLANAR3) {
    e = launch_actor<Arm3>(sys->d_prm, d, w, B, T_max, d_T, perm, d_x0, d_U, d_X, st);
  } else if (sys->kind == CBIC_SYS_LQ && sys->n == 2 && sys->m == 1) {
    e = launch_actor<LinQuad<2, 1>>(sys->d_prm, d, w, B, T_max, d_T, perm, d_x0, d_U, d_X, st);
  } else if (sys->kind == CBIC_SYS_LQ && sys->n == 4 && sys->m == 2) {
    e = launch_actor<LinQuad<4, 2>>(sys->d_prm, d, w, B, T_max, d_T, perm, d_x0, d_U, d_X, st);
  } else {
    e = launch_actor<LinQuad<6, 3>>(sys->d_prm, d, w, B, T_max, d_T, perm, d_x0, d_U, d_X, st);
  }
  HIP_TRY(e);
  if (perm) {
    HIP_TRY(hipEventRecord(ctx->done_ev, st));
    ctx->last_stream = st;
    ctx->have_last = true;
  }
  return CBIC_OK;
}

}  // extern "C"
