// Causal depthwise convolution over compact rows with true-ancestor context
// (HARTS, Sec. 4.2, "KDA state reuse and causal convolution"), for gfx950.
//
// Along every trajectory, y_t[c] = sum_{i < w} W[c, i] x_{t-i}[c], zero
// before the trajectory's first token.  In the compact layout a row's i-th
// predecessor on its trajectory is unique (a row has one ancestor path): the
// row i above it inside its segment, else a row of an ancestor segment,
// never a row of an adjacent packed sequence.  harts_conv_context (host,
// semantic.cpp) writes that predecessor table once per plan, and the
// transposed table of consumers, which the backward walks to gather each
// row's gradient.
//   k_conv_fwd      one thread per (4 channels, sub-run of 16 rows);
//   k_conv_bwd      the same threads, four sub-runs to a run of 64 rows: dx
//                   of each row (its own term plus every consumer's, in
//                   (tap, row) order) and the run's tap sums
//                   x[pred_i(r)] dy[r], in row order within a sub-run, the
//                   sub-runs added in order;
//   k_conv_dw_sum   per (channel, tap), the runs' partials in a fixed order.
// Arithmetic in float32; no atomics, so reruns are bitwise identical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <new>
#include <string>
#include <vector>

#include "harts.h"
#include "plan.hpp"

namespace harts {
namespace {

typedef __bf16 bf16;
constexpr int CV_THR = 256;
constexpr int CV_MAXW = 8;
constexpr int CV_SUB = 4;                     // sub-runs (waves) of a workgroup
constexpr int CV_RT = 16;                     // rows of a sub-run
constexpr int CV_RUN = CV_SUB * CV_RT;        // rows of a run (one partial dW per run)
constexpr int CV_G = 4;                       // rows taken at a time
constexpr int CV_SUCC = 1024;                 // consumer entries of a run staged in LDS
static_assert(CV_SUB * 64 == CV_THR && CV_RUN == 64 && CV_RT % CV_G == 0 && CV_RT <= 32, "one wave per sub-run, one bit per row");

template <typename T> struct CV;
template <> struct CV<bf16> {
  static constexpr int N = 4;  // 8-byte pieces: half the registers of 16-byte ones
  static constexpr int B = 4;  // consumer entries of a row taken at a time (as many as the registers hold)
  static constexpr int waves(int w) { return w <= 3 ? 4 : (w == 4 ? 3 : 2); }  // a SIMD, in the backward
  using Raw = uint2;           // a piece as loaded, widened where it is used
  __device__ static inline Raw raw(const bf16* p) { return *reinterpret_cast<const uint2*>(p); }
  __device__ static inline void cvt(const Raw u, float* x) {
    x[0] = __uint_as_float(u.x << 16);
    x[1] = __uint_as_float(u.x & 0xffff0000u);
    x[2] = __uint_as_float(u.y << 16);
    x[3] = __uint_as_float(u.y & 0xffff0000u);
  }
  __device__ static inline void store(bf16* p, const float* x) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    bf16x4 b;
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = static_cast<bf16>(x[i]);
    *reinterpret_cast<bf16x4*>(p) = b;
  }
};
template <> struct CV<float> {
  static constexpr int N = 4;
  static constexpr int B = 2;
  static constexpr int waves(int w) { return w == 2 ? 4 : (w <= 4 ? 3 : 2); }
  using Raw = float4;
  __device__ static inline Raw raw(const float* p) { return *reinterpret_cast<const float4*>(p); }
  __device__ static inline void cvt(const Raw u, float* x) {
    x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w;
  }
  __device__ static inline void store(float* p, const float* x) {
    *reinterpret_cast<float4*>(p) = float4{x[0], x[1], x[2], x[3]};
  }
};

// A workgroup takes a run of 64 rows for 64 vectors of 4 channels: wave s the
// rows of sub-run s, lane l vector l of the block (a row of a wave is one
// contiguous piece of 512 or 1024 bytes), the W taps in registers.  These
// kernels only stream, so what bounds them is how many bytes a CU has in
// flight: a wave requests the next CV_G rows before it uses the present ones,
// and short sub-runs give a small call enough waves.  Measured against one
// thread per whole run (64 rows backward, 32 forward), every row through the
// tables: backward of 68,161 x 6,144 bf16, w = 4: 792 -> 518 us (4.9 TB/s of
// x, dy and dx), of 3,001 x 1,000 float32, w = 3 (47 workgroups before):
// 53.9 -> 12.1 us; forward 325 -> 310 and 14.4 -> 8.0 us.  Sub-runs of 32 rows
// (the forward): 315 us, but 41.9 us instead of 43.2 for 16,000 x 2,048
// float32, which the cache holds; of 8 rows, or two rows at a time, the
// backward took longer.
//
// The windows over x and dy stay in registers.  A row whose predecessors are
// the row above it and that row's own needs no table, whatever segments they
// lie in: the window moves by one.  At any other row (in the forests of trees:
// a segment's first) the window is gathered through the table, its W - 1 loads
// together.  In the backward a row whose consumers are exactly the W - 1 rows
// below it needs no table either; any other row takes its consumers in table
// order, those in the window from registers, the rest a few requests at a
// time.  Groups of CV_G rows without either have no branches.  Every row adds
// in the same order on every path.  With every tap and consumer of a segment's
// first and last W - 1 rows loaded one by one, forests of short segments took
// up to three times as long: 65,536 x 6,144 bf16, forward and backward, w = 4:
// segments of 1 to 200 rows 307 + 630 -> 310 + 532 us, of 8 371 + 1,276 -> 317
// + 737, of 3 570 + 1,779 -> 333 + 1,016; w = 8, of 1 to 200 rows 489 + 2,552
// -> 346 + 1,011 us.
template <typename T, int W>
__device__ inline void load_taps(const float* __restrict__ Wt, int c0, float (&wt)[W][CV<T>::N]) {
#pragma unroll
  for (int e = 0; e < CV<T>::N; ++e) {
    const float4* src = reinterpret_cast<const float4*>(Wt + (c0 + e) * W);
    if constexpr (W % 4 == 0) {
#pragma unroll
      for (int q = 0; q < W / 4; ++q) {
        const float4 u = src[q];
        wt[4 * q][e] = u.x; wt[4 * q + 1][e] = u.y; wt[4 * q + 2][e] = u.z; wt[4 * q + 3][e] = u.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < W; ++i) wt[i][e] = Wt[(c0 + e) * W + i];
    }
  }
}

// The row's predecessors are the W - 1 rows just above it.
template <int W>
__device__ inline bool regular_pred(const int32_t* pr, int64_t r) {
  bool ok = r >= W - 1;
#pragma unroll
  for (int i = 1; i < W; ++i) ok &= pr[i - 1] == r - i;
  return ok;
}

// Bit i of the result: row rs + i of a wave's sub-run (n rows, their table
// entries at pr) does not follow from the row above it, i.e. its predecessors
// are not that row and then that row's own (at the sub-run's first row: not
// the W - 1 rows just above it, which the window starts with).
template <int W>
__device__ inline uint32_t window_breaks(const int32_t* pr, int64_t rs, int n, int lane) {
  bool brk = false;
  if (lane < n) {
    const int32_t* p = pr + lane * (W - 1);
    if (lane == 0) {
      brk = !regular_pred<W>(p, rs);
    } else {
      brk = p[0] != rs + lane - 1;
#pragma unroll
      for (int i = 2; i < W; ++i) brk |= p[i - 1] != p[i - 2 - (W - 1)];
    }
  }
  return static_cast<uint32_t>(__ballot(brk));
}

// The window over x at a break: xw[-i] <- x[pred_i] (zero before the trajectory
// start or for an invalid entry), all of them requested together.
template <typename T, int W>
__device__ inline void gather_window(typename CV<T>::Raw* xw, const T* __restrict__ x, int64_t C, int Cch, int c0,
                                     const int32_t* pr) {
  int32_t p[W - 1];
#pragma unroll
  for (int i = 1; i < W; ++i) p[i - 1] = __builtin_amdgcn_readfirstlane(pr[i - 1]);
#pragma unroll
  for (int i = 1; i < W; ++i)
    xw[-i] = CV<T>::raw(x + (p[i - 1] >= 0 && p[i - 1] < C ? static_cast<int64_t>(p[i - 1]) : 0) * Cch + c0);
#pragma unroll
  for (int i = 1; i < W; ++i)
    if (!(p[i - 1] >= 0 && p[i - 1] < C)) xw[-i] = typename CV<T>::Raw{};
}

template <typename T, int W>
__global__ __launch_bounds__(CV_THR) void k_conv_fwd(int64_t C, int Cch, const T* __restrict__ x,
                                                     const float* __restrict__ Wt,
                                                     const int32_t* __restrict__ pred, T* __restrict__ y) {
  using V = CV<T>;
  using Raw = typename V::Raw;
  const int lane = threadIdx.x & 63, sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int vec = blockIdx.x * 64 + lane;
  const int c0 = vec * V::N;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * CV_RUN;
  const int64_t r1 = r0 + CV_RUN < C ? r0 + CV_RUN : C;
  // the run's predecessor table, staged in LDS (one global round trip per
  // workgroup instead of one per row)
  __shared__ int32_t s_pred[CV_RUN * (W - 1)];
  for (int j = threadIdx.x; j < (r1 - r0) * (W - 1); j += CV_THR) s_pred[j] = pred[r0 * (W - 1) + j];
  __syncthreads();
  const int64_t rs = r0 + sub * CV_RT;
  const int n = static_cast<int>(r1 - rs < CV_RT ? r1 - rs : CV_RT);
  if (n <= 0) return;
  const int32_t* sp = s_pred + sub * CV_RT * (W - 1);
  const uint32_t brk = window_breaks<W>(sp, rs, n, lane);
  if (vec >= Cch / V::N) return;
  float wt[W][V::N];
  load_taps<T, W>(Wt, c0, wt);
  // xw[j] = x[row - (W - 1) + j] as loaded; requests past either end are
  // clamped and never used (a window that reaches past the start is gathered)
  Raw xw[W - 1 + CV_G];
#pragma unroll
  for (int j = 0; j < W - 1 + CV_G; ++j) {
    const int64_t r = rs - (W - 1) + j;
    xw[j] = V::raw(x + (r < 0 ? 0 : (r < C ? r : C - 1)) * Cch + c0);
  }
  for (int g = 0; CV_G * g < n; ++g) {
    const int64_t r = rs + CV_G * g;
    // (guarded, the loads past a sub-run's end cost 5% of the forward;
    // guarding them in the backward made it 4% slower)
    Raw xn[CV_G];
#pragma unroll
    for (int q = 0; q < CV_G; ++q)
      if (CV_G * (g + 1) < n) xn[q] = V::raw(x + (r + CV_G + q < C ? r + CV_G + q : C - 1) * Cch + c0);
    const auto row = [&](int q) __attribute__((always_inline)) {
      float v[V::N], acc[V::N];
      V::cvt(xw[W - 1 + q], v);
#pragma unroll
      for (int e = 0; e < V::N; ++e) acc[e] = wt[0][e] * v[e];
#pragma unroll
      for (int i = 1; i < W; ++i) {
        V::cvt(xw[W - 1 + q - i], v);
#pragma unroll
        for (int e = 0; e < V::N; ++e) acc[e] += wt[i][e] * v[e];
      }
      V::store(y + (r + q) * Cch + c0, acc);
    };
    const uint32_t gb = brk >> (CV_G * g) & ((1u << CV_G) - 1u);
    if (gb == 0 && CV_G * (g + 1) <= n) {
#pragma unroll
      for (int q = 0; q < CV_G; ++q) row(q);
    } else {
#pragma unroll
      for (int q = 0; q < CV_G; ++q) {
        if (CV_G * g + q >= n) break;
        if (gb >> q & 1u) gather_window<T, W>(xw + W - 1 + q, x, C, Cch, c0, sp + (CV_G * g + q) * (W - 1));
        row(q);
      }
    }
#pragma unroll
    for (int j = 0; j < W - 1; ++j) xw[j] = xw[CV_G + j];
#pragma unroll
    for (int q = 0; q < CV_G; ++q) xw[W - 1 + q] = xn[q];
  }
}

// dx of a run of rows, and the run's partial weight gradient:
// part[run][i][c] = sum over the run's rows r of x[pred_i(r)][c] dy[r][c].
template <typename T, int W>
__global__ __launch_bounds__(CV_THR, CV<T>::waves(W)) void k_conv_bwd(int64_t C, int Cch, const T* __restrict__ x,
                                                     const float* __restrict__ Wt,
                                                     const int32_t* __restrict__ pred,
                                                     const int64_t* __restrict__ succ_off,
                                                     const int32_t* __restrict__ succ, int64_t n_succ,
                                                     const T* __restrict__ dy, T* __restrict__ dx,
                                                     float* __restrict__ part) {
  using V = CV<T>;
  using Raw = typename V::Raw;
  const int lane = threadIdx.x & 63, sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int vec = blockIdx.x * 64 + lane;
  const int c0 = vec * V::N;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * CV_RUN;
  const int64_t r1 = r0 + CV_RUN < C ? r0 + CV_RUN : C;
  // the run's tables, staged in LDS: predecessors, consumer offsets
  // (relative to the run's first entry) and up to CV_SUCC consumer entries;
  // entries beyond that (rows feeding very many children) are read from
  // global memory
  __shared__ int32_t s_pred[CV_RUN * (W - 1)];
  __shared__ int32_t s_off[CV_RUN + 1];
  __shared__ int32_t s_succ[CV_SUCC];
  __shared__ float4 s_gw[CV_SUB][W][64];
  const int64_t nr = r1 - r0;
  const int64_t b0 = succ_off[r0] < 0 ? 0 : (succ_off[r0] > n_succ ? n_succ : succ_off[r0]);
  for (int j = threadIdx.x; j < nr * (W - 1); j += CV_THR) s_pred[j] = pred[r0 * (W - 1) + j];
  for (int j = threadIdx.x; j <= nr; j += CV_THR) {
    int64_t o = succ_off[r0 + j];
    o = o < b0 ? b0 : (o > n_succ ? n_succ : o);
    s_off[j] = static_cast<int32_t>(o - b0 < INT32_MAX ? o - b0 : INT32_MAX);
  }
  __syncthreads();
  const int32_t n_run_succ = s_off[nr];
  for (int j = threadIdx.x; j < n_run_succ && j < CV_SUCC; j += CV_THR) s_succ[j] = succ[b0 + j];
  __syncthreads();
  const int64_t rs = r0 + sub * CV_RT;
  const int n = static_cast<int>(r1 - rs < CV_RT ? r1 - rs : CV_RT);
  const bool live = vec < Cch / V::N;
  const int32_t* sp = s_pred + sub * CV_RT * (W - 1);
  const uint32_t brk = window_breaks<W>(sp, rs, n, lane);
  // rows whose consumers are not exactly the W - 1 rows just below them
  bool far = false;
  if (lane < n) {
    const int64_t r = rs + lane;
    const int32_t jb = s_off[sub * CV_RT + lane];
    far = r + W - 1 >= C || s_off[sub * CV_RT + lane + 1] != jb + W - 1 || jb + W - 1 > CV_SUCC;
    if (!far) {
#pragma unroll
      for (int i = 1; i < W; ++i) far |= s_succ[jb + i - 1] != (r + i) * 8 + i;
    }
  }
  const uint32_t fars = static_cast<uint32_t>(__ballot(far));
  float gw[W][V::N];
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int e = 0; e < V::N; ++e) gw[i][e] = 0.f;
  if (live && n > 0) {
    float wt[W][V::N];
    load_taps<T, W>(Wt, c0, wt);
    // windows as loaded: xw[j] = x[row - (W - 1) + j], dw[j] = dy[row + j];
    // requests past either end are clamped and never used (a window over x
    // that reaches past the start is gathered, no consumer is past the end)
    Raw xw[W - 1 + CV_G], dw[W - 1 + CV_G];
#pragma unroll
    for (int j = 0; j < W - 1 + CV_G; ++j) {
      const int64_t rx = rs - (W - 1) + j, rd = rs + j;
      xw[j] = V::raw(x + (rx < 0 ? 0 : (rx < C ? rx : C - 1)) * Cch + c0);
      dw[j] = V::raw(dy + (rd < C ? rd : C - 1) * Cch + c0);
    }
    for (int g = 0; CV_G * g < n; ++g) {
      const int64_t r = rs + CV_G * g;
      Raw xn[CV_G], dn[CV_G];
#pragma unroll
      for (int q = 0; q < CV_G; ++q) {
        const int64_t rx = r + CV_G + q, rd = rx + W - 1;
        xn[q] = V::raw(x + (rx < C ? rx : C - 1) * Cch + c0);
        dn[q] = V::raw(dy + (rd < C ? rd : C - 1) * Cch + c0);
      }
      // the row's tap sums and its own term of dx
      const auto own = [&](int q, float (&acc)[V::N]) __attribute__((always_inline)) {
        float d0[V::N], v[V::N];
        V::cvt(dw[q], d0);
#pragma unroll
        for (int i = 0; i < W; ++i) {
          V::cvt(xw[W - 1 + q - i], v);
#pragma unroll
          for (int e = 0; e < V::N; ++e) gw[i][e] += v[e] * d0[e];
        }
#pragma unroll
        for (int e = 0; e < V::N; ++e) acc[e] = wt[0][e] * d0[e];
      };
      // the terms of the W - 1 rows below
      const auto below = [&](int q, float (&acc)[V::N]) __attribute__((always_inline)) {
        float v[V::N];
#pragma unroll
        for (int i = 1; i < W; ++i) {
          V::cvt(dw[q + i], v);
#pragma unroll
          for (int e = 0; e < V::N; ++e) acc[e] += wt[i][e] * v[e];
        }
      };
      const uint32_t gb = brk >> (CV_G * g) & ((1u << CV_G) - 1u);
      const uint32_t gf = fars >> (CV_G * g) & ((1u << CV_G) - 1u);
      if ((gb | gf) == 0 && CV_G * (g + 1) <= n) {
#pragma unroll
        for (int q = 0; q < CV_G; ++q) {
          float acc[V::N];
          own(q, acc);
          below(q, acc);
          V::store(dx + (r + q) * Cch + c0, acc);
        }
      } else {
#pragma unroll
        for (int q = 0; q < CV_G; ++q) {
          const int lr = CV_G * g + q;   // row of the sub-run
          if (lr >= n) break;
          if (gb >> q & 1u) gather_window<T, W>(xw + W - 1 + q, x, C, Cch, c0, sp + lr * (W - 1));
          float acc[V::N];
          own(q, acc);
          if (!(gf >> q & 1u)) {
            below(q, acc);
          } else {
            // consumers in table order, V::B at a time: the staged entries
            // from LDS, any beyond them from global memory (two loops, so that
            // neither read goes through a flat address, which would wait for
            // every outstanding load)
            const auto consume = [&](int32_t j, int32_t je, auto entry) __attribute__((always_inline)) {
              Raw rb[V::B];
              int tap[V::B];      // 0: none
              bool low[V::B];     // the row tap below: in the window
#pragma unroll
              for (int u = 0; u < V::B; ++u) {
                const int32_t code = j + u < je ? __builtin_amdgcn_readfirstlane(entry(j + u)) : -1;
                const int32_t sr = code >> 3, i = code & 7;  // consumer row, tap
                tap[u] = sr < 0 || sr >= C || i < 1 || i >= W ? 0 : i;
                low[u] = sr == r + q + i;
                if (tap[u] != 0 && !low[u]) rb[u] = V::raw(dy + static_cast<int64_t>(sr) * Cch + c0);
              }
#pragma unroll
              for (int u = 0; u < V::B; ++u)
#pragma unroll
                for (int k = 1; k < W; ++k)
                  if (tap[u] == k) {
                    float v[V::N];
                    V::cvt(low[u] ? dw[q + k] : rb[u], v);
#pragma unroll
                    for (int e = 0; e < V::N; ++e) acc[e] += wt[k][e] * v[e];
                  }
            };
            const int32_t jb = __builtin_amdgcn_readfirstlane(s_off[sub * CV_RT + lr]);
            const int32_t je = __builtin_amdgcn_readfirstlane(s_off[sub * CV_RT + lr + 1]);
            const int32_t jl = je < CV_SUCC ? je : CV_SUCC;
            for (int32_t j = jb; j < jl; j += V::B) consume(j, jl, [&](int32_t k) { return s_succ[k]; });
            for (int32_t j = jb > CV_SUCC ? jb : CV_SUCC; j < je; j += V::B)
              consume(j, je, [&](int32_t k) { return succ[b0 + k]; });
          }
          V::store(dx + (r + q) * Cch + c0, acc);
        }
      }
#pragma unroll
      for (int j = 0; j < W - 1; ++j) {
        xw[j] = xw[CV_G + j];
        dw[j] = dw[CV_G + j];
      }
#pragma unroll
      for (int q = 0; q < CV_G; ++q) {
        xw[W - 1 + q] = xn[q];
        dw[W - 1 + q] = dn[q];
      }
    }
  }
  // the sub-runs' tap sums, added in order; the waves share the taps
#pragma unroll
  for (int i = 0; i < W; ++i) s_gw[sub][i][lane] = float4{gw[i][0], gw[i][1], gw[i][2], gw[i][3]};
  __syncthreads();
  // partials tap-major ([run][tap][channel]): every store is a coalesced
  // piece of one tap's channel row
  float* out = part + static_cast<int64_t>(blockIdx.y) * Cch * W;
  for (int i = sub; i < W && live; i += CV_SUB) {
    float4 a = s_gw[0][i][lane];
#pragma unroll
    for (int k = 1; k < CV_SUB; ++k) {
      const float4 b = s_gw[k][i][lane];
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    *reinterpret_cast<float4*>(out + static_cast<int64_t>(i) * Cch + c0) = a;
  }
}

// dW[c][i] = sum over runs of part[run][i][c]: a workgroup takes 32
// consecutive (tap, channel) entries; its 8 groups of 32 threads sum every
// 8th run (group g takes runs g, g + 8, ...), and the 8 group sums are
// added in group order: a fixed association, independent of scheduling.
constexpr int DW_K = 32, DW_G = CV_THR / DW_K;
__global__ __launch_bounds__(CV_THR) void k_conv_dw_sum(int64_t n_run, int Cch, int W,
                                                        const float* __restrict__ part,
                                                        float* __restrict__ dW) {
  __shared__ float red[DW_G][DW_K];
  const int lk = threadIdx.x % DW_K, g = threadIdx.x / DW_K;
  const int64_t n = static_cast<int64_t>(Cch) * W;
  const int64_t k = static_cast<int64_t>(blockIdx.x) * DW_K + lk;  // i * Cch + c
  float acc = 0.f;
  if (k < n) {
    // eight partials requested together: 59 -> 27 us for the 1,066 runs of a
    // 68,161 x 6,144 call, w = 4 (105 MB)
#pragma unroll 8
    for (int64_t b = g; b < n_run; b += DW_G) acc += part[b * n + k];
  }
  red[g][lk] = acc;
  __syncthreads();
  if (g == 0 && k < n) {
    float sum = red[0][lk];
#pragma unroll
    for (int j = 1; j < DW_G; ++j) sum += red[j][lk];
    const int64_t i = k / Cch, c = k % Cch;
    dW[c * W + i] = sum;
  }
}

int conv_status(const char* where) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(where) + ": " + hipGetErrorString(e));
    return HARTS_EHIP;
  }
  return HARTS_OK;
}

int check_conv(int32_t dtype, int64_t C, int32_t Cch, int32_t w, const char* where) {
  const std::string s(where);
  if (dtype != HARTS_F32 && dtype != HARTS_BF16) { set_error(s + ": unknown dtype"); return HARTS_EUNSUPPORTED; }
  if (w < 2 || w > CV_MAXW) { set_error(s + ": width must be in [2, 8]"); return HARTS_EUNSUPPORTED; }
  if (Cch < 8 || Cch % 8 || Cch > (1 << 20)) {
    set_error(s + ": channels must be a positive multiple of 8, at most 2^20");
    return HARTS_EUNSUPPORTED;
  }
  if (C < 0 || C >= (int64_t{1} << 28)) { set_error(s + ": need 0 <= C < 2^28 rows"); return HARTS_EUNSUPPORTED; }
  return HARTS_OK;
}

bool a16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

template <typename T>
int launch_fwd(int w, int64_t C, int Cch, const void* x, const float* Wt, const int32_t* pred, void* y,
               hipStream_t s) {
  const int nvec = Cch / CV<T>::N;
  const dim3 grid(static_cast<uint32_t>((nvec + 63) / 64),
                  static_cast<uint32_t>((C + CV_RUN - 1) / CV_RUN));
  const T* xx = static_cast<const T*>(x);
  T* yy = static_cast<T*>(y);
  switch (w) {
#define HARTS_CONV_FWD(WW) \
  case WW: hipLaunchKernelGGL((k_conv_fwd<T, WW>), grid, dim3(CV_THR), 0, s, C, Cch, xx, Wt, pred, yy); break;
    HARTS_CONV_FWD(2) HARTS_CONV_FWD(3) HARTS_CONV_FWD(4) HARTS_CONV_FWD(5)
    HARTS_CONV_FWD(6) HARTS_CONV_FWD(7) HARTS_CONV_FWD(8)
#undef HARTS_CONV_FWD
  }
  return conv_status("k_conv_fwd");
}

template <typename T>
int launch_bwd(int w, int64_t C, int Cch, const void* x, const float* Wt, const int32_t* pred,
               const int64_t* succ_off, const int32_t* succ, int64_t n_succ, const void* dy, void* dx,
               float* dW, float* part, hipStream_t s) {
  const int nvec = Cch / CV<T>::N;
  const int64_t n_run = (C + CV_RUN - 1) / CV_RUN;
  const dim3 grid(static_cast<uint32_t>((nvec + 63) / 64), static_cast<uint32_t>(n_run));
  const T* xx = static_cast<const T*>(x);
  const T* gy = static_cast<const T*>(dy);
  T* gx = static_cast<T*>(dx);
  switch (w) {
#define HARTS_CONV_BWD(WW)                                                                            \
  case WW:                                                                                            \
    hipLaunchKernelGGL((k_conv_bwd<T, WW>), grid, dim3(CV_THR), 0, s, C, Cch, xx, Wt, pred, succ_off, \
                       succ, n_succ, gy, gx, part);                                                   \
    break;
    HARTS_CONV_BWD(2) HARTS_CONV_BWD(3) HARTS_CONV_BWD(4) HARTS_CONV_BWD(5)
    HARTS_CONV_BWD(6) HARTS_CONV_BWD(7) HARTS_CONV_BWD(8)
#undef HARTS_CONV_BWD
  }
  if (int rc = conv_status("k_conv_bwd")) return rc;
  const int64_t n = static_cast<int64_t>(Cch) * w;
  hipLaunchKernelGGL(k_conv_dw_sum, dim3(static_cast<uint32_t>((n + DW_K - 1) / DW_K)), dim3(CV_THR), 0,
                     s, n_run, Cch, w, part, dW);
  return conv_status("k_conv_dw_sum");
}

}  // namespace
}  // namespace harts

using namespace harts;

extern "C" int harts_conv_workspace_size(int64_t C, int32_t Cch, int32_t w, size_t* bytes) {
  if (int rc = check_conv(HARTS_F32, C, Cch, w, "harts_conv_workspace_size")) return rc;
  if (!bytes) { set_error("harts_conv_workspace_size: NULL bytes"); return HARTS_EINVAL; }
  const int64_t n_run = (C + CV_RUN - 1) / CV_RUN;
  *bytes = static_cast<size_t>(std::max<int64_t>(n_run, 1)) * Cch * w * sizeof(float);
  return HARTS_OK;
}

extern "C" int harts_conv_fwd(int32_t dtype, int64_t C, int32_t Cch, int32_t w, const void* x, const float* Wt,
                              const int32_t* pred, void* y, void* stream) {
  if (int rc = check_conv(dtype, C, Cch, w, "harts_conv_fwd")) return rc;
  if (C == 0) return HARTS_OK;
  if (!x || !Wt || !pred || !y || !a16(x) || !a16(y) || !a16(Wt)) {
    set_error("harts_conv_fwd: NULL or misaligned (16 bytes) pointer");
    return HARTS_EINVAL;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  return dtype == HARTS_BF16 ? launch_fwd<bf16>(w, C, Cch, x, Wt, pred, y, s)
                             : launch_fwd<float>(w, C, Cch, x, Wt, pred, y, s);
}

extern "C" int harts_conv_bwd(int32_t dtype, int64_t C, int32_t Cch, int32_t w, const void* x, const float* Wt,
                              const int32_t* pred, const int64_t* succ_off, const int32_t* succ,
                              int64_t n_succ, const void* dy, void* dx, float* dW, void* ws,
                              size_t ws_bytes, void* stream) {
  if (int rc = check_conv(dtype, C, Cch, w, "harts_conv_bwd")) return rc;
  if (C == 0) return HARTS_OK;
  if (!x || !Wt || !pred || !succ_off || (!succ && n_succ > 0) || n_succ < 0 || !dy || !dx || !dW || !ws ||
      !a16(x) || !a16(dy) || !a16(dx) || !a16(Wt)) {
    set_error("harts_conv_bwd: NULL or misaligned (16 bytes) pointer, or n_succ < 0");
    return HARTS_EINVAL;
  }
  size_t need = 0;
  harts_conv_workspace_size(C, Cch, w, &need);
  if (ws_bytes < need) {
    set_error("harts_conv_bwd: workspace too small (see harts_conv_workspace_size)");
    return HARTS_EINVAL;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* part = static_cast<float*>(ws);
  return dtype == HARTS_BF16
             ? launch_bwd<bf16>(w, C, Cch, x, Wt, pred, succ_off, succ, n_succ, dy, dx, dW, part, s)
             : launch_bwd<float>(w, C, Cch, x, Wt, pred, succ_off, succ, n_succ, dy, dx, dW, part, s);
}
