// Compact-to-semantic log-probabilities for gfx950 (HARTS, Sec. 3.5).
//
// Vocabulary-wide work runs once per compact logit row, scalar work once
// per semantic position (eq. mapped-logp):
//   k_logp_lse     one workgroup per compact row c streams z[c, :] and keeps
//                  a running (max, sum of exponentials) per thread, then
//                  combines them: lse_c = log sum_v exp z[c, v];
//   k_logp_gather  one thread per position s: lambda_s = z[m(s), y_s] - lse.
// Backward (eq. mapped-logp-grad), for upstream gradients g_s:
//   k_logp_grad    one workgroup per row: G_c = sum of g_s over the row's
//                  positions, in the row's (target, position) order; then
//                  dz[c, v] = -G_c p_{c,v}, p = exp(z - lse), over the whole
//                  vocabulary; then the row's target columns again,
//                  dz[c, y] = -G_c p_{c,y} + (sum of g_s over the row's
//                  positions with y_s = y), one rounding from float32.
// Rows are streamed as 16-byte vectors (8 bf16 or 4 float32 logits per
// load, four loads in flight per thread); exponentials are base 2 of
// log2(e)-scaled logits.  No atomics, every sum in a fixed order.
//
// Both row kernels are bound by the bytes of the logits: the forward reads
// them at 6.5 TB/s, the backward reads and writes at 5.4 (17,640 rows of
// 157,184 bf16: 858 and 2,040 us; a large copy moves 5.0 TB/s).  What is left
// to save is launches (the row sums and the target columns were kernels of
// their own: a pass over 481 rows of 32,008 float32 went from 53 to 40 us).
// A row without a gradient (G = 0) is read all the same: lse passes over
// vectors of NaN and -inf, so only the logits tell where 0 times p is NaN.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "harts.h"
#include "plan.hpp"

namespace harts {
namespace {

typedef __bf16 bf16;
constexpr int LP_THR = 256;   // threads per row workgroup (and per workgroup of positions)
// A row of at least LP_WIDE vectors takes 1,024 threads instead of 256: fewer
// rows are open at a time for the same loads in flight.  Backward of 17,640
// rows of 157,184 bf16 2,200 -> 2,040 us (its forward the same within the
// runs, 790 at best); forward of 481 rows of 32,008 float32 14.7 -> 13.6 us.
// A shorter row would leave most of the 1,024 threads without a vector.
constexpr int64_t LP_WIDE = 2048;
constexpr int LP_THR_W = 1024;
constexpr int LP_UNROLL = 4;  // 16-byte loads in flight per thread
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Logits of more than LP_STREAM bytes are not in the 256 MB last-level cache
// when the next kernel comes: the forward then reads and the backward writes
// them non-temporally.  5.5 GB of bf16 logits: forward 941 -> 858 us, backward
// 2,101 -> 2,040 us (2,006 with non-temporal reads as well); on 62 MB, which
// the backward finds in the cache, neither is faster.
constexpr int64_t LP_STREAM = int64_t{256} << 20;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__device__ inline u32x4 load16(const void* p) {
  const u32x4* q = static_cast<const u32x4*>(p);
  return NT ? __builtin_nontemporal_load(q) : *q;
}
template <bool NT>
__device__ inline void store16(void* p, const u32x4 v) {
  u32x4* q = static_cast<u32x4*>(p);
  if (NT) __builtin_nontemporal_store(v, q);
  else *q = v;
}

template <typename T> struct LV;
template <> struct LV<bf16> {
  static constexpr int N = 8;
  template <bool NT>
  __device__ static inline void load(const bf16* p, float* x) {
    const u32x4 w = load16<NT>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(w[i] << 16);
      x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  template <bool NT>
  __device__ static inline void store(bf16* p, const float* x) {
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = static_cast<bf16>(x[i]);  // round to nearest even
    store16<NT>(p, __builtin_bit_cast(u32x4, b));
  }
  __device__ static inline float one(const bf16* p) { return static_cast<float>(*p); }
  __device__ static inline void put(bf16* p, float x) { *p = static_cast<bf16>(x); }
};
template <> struct LV<float> {
  static constexpr int N = 4;
  template <bool NT>
  __device__ static inline void load(const float* p, float* x) {
    const u32x4 w = load16<NT>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(w[i]);
  }
  template <bool NT>
  __device__ static inline void store(float* p, const float* x) {
    store16<NT>(p, u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])});
  }
  __device__ static inline float one(const float* p) { return *p; }
  __device__ static inline void put(float* p, float x) { *p = x; }
};

__device__ inline float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// (m, s) with s = sum 2^(x - m): merge two partial results
__device__ inline void lse_merge(float& m, float& s, float m2, float s2) {
  const float n = fmaxf(m, m2);
  s = (m == -INFINITY ? 0.f : s * ex2(m - n)) + (m2 == -INFINITY ? 0.f : s2 * ex2(m2 - n));
  m = n;
}

template <typename T, int THR, bool NT>
__global__ __launch_bounds__(THR) void k_logp_lse(const T* __restrict__ z, int64_t V,
                                                     float* __restrict__ lse) {
  using L = LV<T>;
  const int64_t c = blockIdx.x;
  const int t = threadIdx.x;
  const T* row = z + c * V;
  const int64_t nvec = V / L::N;
  float m = -INFINITY, s = 0.f;
  for (int64_t i0 = t; i0 < nvec; i0 += static_cast<int64_t>(THR) * LP_UNROLL) {
    float x[LP_UNROLL][L::N];
#pragma unroll
    for (int u = 0; u < LP_UNROLL; ++u) {
      const int64_t i = i0 + static_cast<int64_t>(u) * THR;
      if (i < nvec) {
        L::template load<NT>(row + i * L::N, x[u]);
      } else {
#pragma unroll
        for (int e = 0; e < L::N; ++e) x[u][e] = -INFINITY;
      }
    }
#pragma unroll
    for (int u = 0; u < LP_UNROLL; ++u) {
      float vm = -INFINITY;
#pragma unroll
      for (int e = 0; e < L::N; ++e) {
        x[u][e] *= kLog2e;
        vm = fmaxf(vm, x[u][e]);
      }
      if (vm == -INFINITY) continue;  // past the row's end, or nothing but -inf and NaN
      const float n = fmaxf(m, vm);
      float acc = m == -INFINITY ? 0.f : s * ex2(m - n);
#pragma unroll
      for (int e = 0; e < L::N; ++e) acc += ex2(x[u][e] - n);
      m = n;
      s = acc;
    }
  }
  // wave, then workgroup
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const float m2 = __shfl_xor(m, off);
    const float s2 = __shfl_xor(s, off);
    lse_merge(m, s, m2, s2);
  }
  __shared__ float ms[THR / 64], ss[THR / 64];
  if ((t & 63) == 0) {
    ms[t >> 6] = m;
    ss[t >> 6] = s;
  }
  __syncthreads();
  if (t == 0) {
    float mm = ms[0], sa = ss[0];
    for (int w = 1; w < THR / 64; ++w) lse_merge(mm, sa, ms[w], ss[w]);
    lse[c] = (mm + log2f(sa)) * kLn2;
  }
}

template <typename T>
__global__ __launch_bounds__(LP_THR) void k_logp_gather(const T* __restrict__ z, int64_t C, int64_t V,
                                                        const float* __restrict__ lse,
                                                        const int32_t* __restrict__ m,
                                                        const int32_t* __restrict__ y, int64_t n_pos,
                                                        float* __restrict__ logp) {
  const int64_t s = static_cast<int64_t>(blockIdx.x) * LP_THR + threadIdx.x;
  if (s >= n_pos) return;
  const int32_t c = m[s], v = y[s];
  // an index outside the logits yields NaN instead of a read out of bounds
  if (c < 0 || c >= C || v < 0 || v >= V) {
    logp[s] = __builtin_nanf("");
    return;
  }
  logp[s] = LV<T>::one(z + static_cast<int64_t>(c) * V + v) - lse[c];
}

template <typename T, int THR, bool NT>
__global__ __launch_bounds__(THR) void k_logp_grad(const T* __restrict__ z, int64_t V,
                                                   const float* __restrict__ lse,
                                                   const int64_t* __restrict__ row_off,
                                                   const int32_t* __restrict__ row_pos,
                                                   const int32_t* __restrict__ y, const float* __restrict__ g,
                                                   int64_t n_pos, float* __restrict__ G, T* __restrict__ dz) {
  using L = LV<T>;
  const int64_t c = blockIdx.x;
  const int t = threadIdx.x;
  const T* row = z + c * V;
  T* out = dz + c * V;
  const int64_t nvec = V / L::N;
  const int64_t b = row_off[c] < 0 ? 0 : row_off[c];
  const int64_t e = row_off[c + 1] > n_pos ? n_pos : row_off[c + 1];
  const float l2 = lse[c] * kLog2e;
  const auto valid = [n_pos](int32_t s) { return s >= 0 && s < n_pos; };
  // G: the positions' gradients are requested together and added in order by
  // every thread from LDS (an invalid entry adds nothing)
  __shared__ float sg[THR];
  float Gc = 0.f;
  for (int64_t j0 = b; j0 < e; j0 += THR) {
    if (j0 > b) __syncthreads();
    if (j0 + t < e) {
      const int32_t s = row_pos[j0 + t];
      sg[t] = valid(s) ? g[s] : 0.f;
    }
    __syncthreads();
    const int n = static_cast<int>(e - j0 < THR ? e - j0 : THR);
    for (int k = 0; k < n; ++k) Gc += sg[k];
  }
  if (t == 0) G[c] = Gc;
  const float ng = -Gc;
  for (int64_t i0 = t; i0 < nvec; i0 += static_cast<int64_t>(THR) * LP_UNROLL) {
    float x[LP_UNROLL][L::N];
#pragma unroll
    for (int u = 0; u < LP_UNROLL; ++u) {
      const int64_t i = i0 + static_cast<int64_t>(u) * THR;
      if (i < nvec) L::template load<false>(row + i * L::N, x[u]);
    }
#pragma unroll
    for (int u = 0; u < LP_UNROLL; ++u) {
      const int64_t i = i0 + static_cast<int64_t>(u) * THR;
      if (i < nvec) {
#pragma unroll
        for (int k = 0; k < L::N; ++k) x[u][k] = ng * ex2(x[u][k] * kLog2e - l2);
        L::template store<NT>(out + i * L::N, x[u]);
      }
    }
  }
  if (e <= b) return;
  __syncthreads();   // the target columns are written after the row
  // a thread per run of positions with one target (the list is in target
  // order): the thread of its first entry adds the run in order
  for (int64_t j0 = b + t; j0 < e; j0 += THR) {
    const int32_t s0 = row_pos[j0];
    if (!valid(s0)) continue;                 // an invalid entry: skipped
    const int32_t v = y[s0];
    if (j0 > b) {
      const int32_t sp = row_pos[j0 - 1];
      if (valid(sp) && y[sp] == v) continue;  // inside a run
    }
    if (v < 0 || v >= V) continue;            // a target outside the vocabulary: skipped
    float acc = 0.f;
    int64_t j = j0;
    for (; j < e; ++j) {
      const int32_t s = row_pos[j];
      if (!valid(s) || y[s] != v) break;
      acc += g[s];
    }
    // of runs of one target that only invalid entries part, the last is kept
    while (j < e && !valid(row_pos[j])) ++j;
    if (j < e && y[row_pos[j]] == v) continue;
    const float p = ex2(LV<T>::one(row + v) * kLog2e - l2);
    LV<T>::put(out + v, ng * p + acc);
  }
}

int hip_status(const char* where) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(where) + ": " + hipGetErrorString(e));
    return HARTS_EHIP;
  }
  return HARTS_OK;
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_logits(int32_t dtype, int64_t C, int64_t V, const char* where) {
  const std::string w(where);
  if (dtype != HARTS_F32 && dtype != HARTS_BF16) {
    set_error(w + ": unknown dtype");
    return HARTS_EUNSUPPORTED;
  }
  if (C < 0 || C > INT32_MAX) { set_error(w + ": need 0 <= C <= 2^31 - 1"); return HARTS_EINVAL; }
  if (V < 8 || V % 8 != 0 || V > INT32_MAX) {
    set_error(w + ": the vocabulary size must be a positive multiple of 8, below 2^31");
    return HARTS_EUNSUPPORTED;
  }
  return HARTS_OK;
}

// Rows of a grid of one workgroup each: a launch holds fewer than 2^32 threads,
// so from 2^22 rows on long ones take 256 threads as well.
template <typename T>
bool wide_rows(int64_t C, int64_t V) {
  return V / LV<T>::N >= LP_WIDE && C < (int64_t{1} << 32) / LP_THR_W;
}

template <typename T>
int launch_lse(int64_t C, int64_t V, const void* z, float* lse, hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>(C));
  const T* zz = static_cast<const T*>(z);
  const bool wide = wide_rows<T>(C, V);
  if (C > LP_STREAM / static_cast<int64_t>(sizeof(T)) / V) {
    if (wide) hipLaunchKernelGGL((k_logp_lse<T, LP_THR_W, true>), grid, dim3(LP_THR_W), 0, s, zz, V, lse);
    else hipLaunchKernelGGL((k_logp_lse<T, LP_THR, true>), grid, dim3(LP_THR), 0, s, zz, V, lse);
  } else {
    if (wide) hipLaunchKernelGGL((k_logp_lse<T, LP_THR_W, false>), grid, dim3(LP_THR_W), 0, s, zz, V, lse);
    else hipLaunchKernelGGL((k_logp_lse<T, LP_THR, false>), grid, dim3(LP_THR), 0, s, zz, V, lse);
  }
  return hip_status("k_logp_lse");
}

template <typename T, int THR, bool NT>
void launch_grad_as(int64_t C, int64_t V, const void* z, const float* lse, const int64_t* row_off,
                    const int32_t* row_pos, const int32_t* y, const float* g, int64_t n_pos, float* G, void* dz,
                    hipStream_t s) {
  hipLaunchKernelGGL((k_logp_grad<T, THR, NT>), dim3(static_cast<uint32_t>(C)), dim3(THR), 0, s,
                     static_cast<const T*>(z), V, lse, row_off, row_pos, y, g, n_pos, G, static_cast<T*>(dz));
}

template <typename T>
int launch_grad(int64_t C, int64_t V, const void* z, const float* lse, const int64_t* row_off, const int32_t* row_pos,
                const int32_t* y, const float* g, int64_t n_pos, float* G, void* dz, hipStream_t s) {
  const bool wide = wide_rows<T>(C, V);
  const auto f = C > LP_STREAM / static_cast<int64_t>(sizeof(T)) / V
                     ? (wide ? launch_grad_as<T, LP_THR_W, true> : launch_grad_as<T, LP_THR, true>)
                     : (wide ? launch_grad_as<T, LP_THR_W, false> : launch_grad_as<T, LP_THR, false>);
  f(C, V, z, lse, row_off, row_pos, y, g, n_pos, G, dz, s);
  return hip_status("k_logp_grad");
}

}  // namespace
}  // namespace harts

using namespace harts;

extern "C" int harts_logp_fwd(int32_t dtype, int64_t C, int64_t V, const void* logits, int64_t n_pos,
                              const int32_t* m, const int32_t* y, float* lse, float* logp,
                              void* stream) {
  if (int rc = check_logits(dtype, C, V, "harts_logp_fwd")) return rc;
  if (n_pos < 0 || (C > 0 && (!logits || !lse)) || (n_pos > 0 && (!m || !y || !logp))) {
    set_error("harts_logp_fwd: NULL required pointer or n_pos < 0");
    return HARTS_EINVAL;
  }
  if (!al16(logits)) { set_error("harts_logp_fwd: logits must be 16-byte aligned"); return HARTS_EINVAL; }
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (C > 0) {
    const int rc = dtype == HARTS_BF16 ? launch_lse<bf16>(C, V, logits, lse, s) : launch_lse<float>(C, V, logits, lse, s);
    if (rc) return rc;
  }
  if (n_pos > 0) {
    const dim3 grid(static_cast<uint32_t>((n_pos + LP_THR - 1) / LP_THR));
    if (dtype == HARTS_BF16)
      hipLaunchKernelGGL((k_logp_gather<bf16>), grid, dim3(LP_THR), 0, s,
                         static_cast<const bf16*>(logits), C, V, lse, m, y, n_pos, logp);
    else
      hipLaunchKernelGGL((k_logp_gather<float>), grid, dim3(LP_THR), 0, s,
                         static_cast<const float*>(logits), C, V, lse, m, y, n_pos, logp);
    if (int rc = hip_status("k_logp_gather")) return rc;
  }
  return HARTS_OK;
}

extern "C" int harts_logp_bwd(int32_t dtype, int64_t C, int64_t V, const void* logits,
                              const float* lse, int64_t n_pos, const int64_t* row_off,
                              const int32_t* row_pos, const int32_t* y, const float* dlogp,
                              float* row_g, void* dlogits, void* stream) {
  if (int rc = check_logits(dtype, C, V, "harts_logp_bwd")) return rc;
  if (n_pos < 0 || (C > 0 && (!logits || !lse || !row_off || !row_g || !dlogits)) ||
      (n_pos > 0 && (!row_pos || !y || !dlogp))) {
    set_error("harts_logp_bwd: NULL required pointer or n_pos < 0");
    return HARTS_EINVAL;
  }
  if (!al16(logits) || !al16(dlogits)) {
    set_error("harts_logp_bwd: logits and dlogits must be 16-byte aligned");
    return HARTS_EINVAL;
  }
  if (C == 0) return HARTS_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  return dtype == HARTS_BF16
             ? launch_grad<bf16>(C, V, logits, lse, row_off, row_pos, y, dlogp, n_pos, row_g, dlogits, s)
             : launch_grad<float>(C, V, logits, lse, row_off, row_pos, y, dlogp, n_pos, row_g, dlogits, s);
}
