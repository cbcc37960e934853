// Full attention over compact rows through asymmetric packed Q/KV views
// (HARTS, Sec. 4.2, eqs. asymmetric-qkv and bottom-right), bf16 on gfx950.
//
// A view is one input sequence of the plan: its query row holds its l own
// rows (contiguous physical compact rows), its key/value row the h ancestor
// positions of its trajectory followed by the same l rows, gathered into a
// packed KV buffer.  Query i sees keys j <= h + i (bottom-right alignment).
// Outputs go straight back to the queries' compact rows (a row is an own row
// of exactly one view); key/value gradients of the views are summed into
// the compact rows they were gathered from, in a fixed order.
//
// Flash-style kernels: a workgroup of 4 waves owns 128 rows of one view and
// head (queries in the forward and dq, keys in dk/dv), a wave 32 of them as
// two 16-row halves (64 and 16 where the call is too small to fill the chip
// with those), and steps over the other side 32 or 64 rows at a time; bf16
// MFMA 16x16x32 with float32 accumulation.  Each step's tiles are loaded
// straight into one of two LDS buffers while the step before it computes, so
// a step has one barrier, no LDS writes (but the zeros of rows past a view's
// end) and no prefetch registers; every fragment read from LDS feeds both halves of the wave.  Every product is
// issued with the operand roles chosen so that the row the wave owns is the
// accumulator column (lane % 16): per-row softmax statistics, rescales and
// outputs then stay in one lane, and a score tile in accumulators is already
// the B operand of the next product (two 16-key tiles form one 32-deep
// operand).  Steps that no row of a wave can see are skipped by that wave;
// masks are evaluated only on steps that cross the causal diagonal.
//   k_attn_fwd   per (query tile, head): S = Q K^T, online softmax, O = P V;
//                writes o and the row log-sum-exp;
//   k_attn_dq    per (query tile, head): P from the stored log-sum-exp,
//                dP = dO V^T, dS = P (dP - delta) with delta = dO . O,
//                dQ = scale dS K; further workgroups write delta of all rows
//                for k_attn_dkdv;
//   k_attn_dkdv  per (key tile, head): over the query tiles that see it,
//                dV = P^T dO and dK = scale dS^T Q (float32 view rows);
//   k_attn_gather / k_attn_scatter: compact rows to view rows and back.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <new>
#include <string>
#include <vector>

#include "harts.h"
#include "la_common.hpp"
#include "lds_load.hpp"
#include "plan.hpp"

namespace harts {
namespace {

constexpr int AT_THR = 256;          // 4 waves
constexpr int AT_TQ = 32;            // queries of a step (dk/dv)
constexpr int AT_WT = 128;           // rows of a table tile (queries in fwd/dq, keys in dk/dv)
constexpr float AT_LOG2E = 1.4426950408889634f;
constexpr float AT_NEG = -1.0e30f;   // masked score (finite: no inf - inf)
// The forward keeps a row's reference maximum until a score exceeds it by
// more than this (base 2): weights then stay below 2^8, and the rescale of
// the accumulators is skipped on most steps.
constexpr float AT_SLACK = 8.f;

// view table: 4 int32 per view
enum { V_QROW = 0, V_L = 1, V_KVOFF = 2, V_H = 3 };

// LDS tile of rows x D bf16, unpadded (the layout a load straight into LDS
// can write: 16 bytes a lane, lanes contiguous).  Row r keeps its 16-byte
// piece p at slot p ^ swz(r), chosen for the lanes that gfx950 serves
// together.  A 16-byte read takes 16 lanes a clock, lanes 0-3, 12-15 and
// 20-27 first, then 4-11, 16-19 and 28-31: in a k-contiguous fragment (lane
// (g, i): row i, piece g) two sets of rows, r and r ^ 12 in the same one, at
// neighbouring pieces; so swz differs over the 16 rows and pairs r with
// r ^ 12.  A transposed read takes 32 lanes, 8 rows of two neighbouring
// pieces: swz / 2 differs over each 8.  (At D = 64 two rows share the 64
// banks, and the same holds for the rows of one parity.)  Measured without a
// conflict; with r paired to r + 8 each 16-byte read took 8 clocks instead of 4.
template <int D>
struct AtTile {
  static constexpr int PPR = D / 8;       // pieces per row
  __device__ static inline int swz(int r) {
    const int hi = (r >> 3) & 1;
    if (D == 128) return (((r & 7) ^ (hi << 2)) << 1) | hi;
    return ((r & 6) ^ (hi << 2)) | hi;
  }
  // k-contiguous fragment of 16 rows from r0 (a multiple of 16), k = 32 s ..:
  // lane (g, i) holds row r0 + i, k = 32 s + 8 g .. + 7 (both operands of a
  // product read this way, so the order of k does not matter)
  __device__ static inline bf16x8 kc(const bf16* t, int r0, int s, int lane) {
    typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    const int i = lane & 15, g = lane >> 4;
    return *(const lds_bf16x8*)(t + r0 * D + i * D + (((4 * s + g) ^ swz(i)) << 3));
  }
  // transposed fragment of 32 rows (the contraction index) from r0, columns
  // c0 .. c0 + 15: lane (g, i) holds column c0 + i, rows r0 + {4g .. 4g + 3}
  // and r0 + 16 + {4g .. 4g + 3}
  __device__ static inline bf16x8 km(const bf16* t, int r0, int c0, int lane) {
    typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
    const int r = (lane >> 4) * 4 + ((lane & 15) >> 2), c = lane & 3;
    const bf16* p = t + r0 * D + r * D + ((((c0 >> 3) + (c >> 1)) ^ swz(r)) << 3) + 4 * (c & 1);
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 16 * D));
    return Frag<bf16>::join(__builtin_bit_cast(bf16x4, lo), __builtin_bit_cast(bf16x4, hi));
  }
};

// Rows row0 .. row0 + NR - 1 of head h of a [rows, H, D] tensor (the first n of
// them, zeros past those), requested straight into an LDS tile (lds_load.hpp):
// the 16-byte pieces of a wave's request land in consecutive LDS slots, so the
// lane picks the piece that belongs there.  (Zeros, because a masked weight is
// 0 and 0 times another row's infinity would not be.)
template <int D>
struct AtRequest {
  static constexpr int PPR = AtTile<D>::PPR;
  static constexpr int RPE = AT_THR / PPR;    // rows of one request of the workgroup (16 or 32)
  uint32_t rowb;                              // bytes of a row, < 2^24
  uint32_t off;                               // the lane's offset in a whole request
  int r0, p16, w;                             // its row, its piece (bytes), its wave
  __device__ inline AtRequest(int H, int wave, int lane) {
    const int slot = 64 * wave + lane;
    w = wave;
    rowb = static_cast<uint32_t>(H) * D * 2;
    r0 = slot / PPR;
    p16 = 16 * ((slot % PPR) ^ AtTile<D>::swz(r0));   // (every request starts at a multiple of 16 rows)
    off = r0 * rowb + p16;
  }
  template <int NR>
  __device__ inline void rows(const bf16* __restrict__ src, int64_t row0, int n, int h, const bf16* tile) const {
    static_assert(NR % RPE == 0 && RPE % 16 == 0, "whole requests");
    const char* base = reinterpret_cast<const char*>(src + static_cast<int64_t>(h) * D) + row0 * rowb;
    if (n >= NR) {
#pragma unroll
      for (int e = 0; e < NR / RPE; ++e)
        lds_load16(base + e * RPE * static_cast<int64_t>(rowb), off, tile + (e * AT_THR + 64 * w) * 8);
    } else {
      // (the zeros in 8-byte pieces take 6 registers fewer, which at d = 64
      // keep the forward at four waves a SIMD; rolled, the loop cost 1% of a
      // 2,000-row pass)
#pragma unroll
      for (int e = 0; e < NR / RPE; ++e) {
        const bf16* dst = tile + (e * AT_THR + 64 * w) * 8;
        if (r0 + RPE * e < n) {
          lds_load16(base, off + static_cast<uint32_t>(RPE * e) * rowb, dst);   // n < 128: below 2^31
        } else {
          typedef __attribute__((address_space(3))) volatile uint64_t lds_u64;
          lds_u64* z = (lds_u64*)(dst + 8 * (threadIdx.x & 63));
          z[0] = 0;
          z[1] = 0;
        }
      }
    }
  }
};
// The fragments of 16 rows of a [rows, H, D] tensor from row0 (rows clamped to
// last), straight from global memory into registers.
template <int D>
__device__ inline void at_frags(bf16x8 (&f)[D / 32], const bf16* __restrict__ src, int64_t row0, int last, int H,
                                int h, int lane) {
  const bf16* p = src + ((row0 + min(lane & 15, last)) * H + h) * D + 8 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < D / 32; ++s) f[s] = *reinterpret_cast<const bf16x8*>(p + 32 * s);
}

// 2^x with the hardware instruction (results below 2^-126 flush to zero,
// which a softmax weight can afford).
__device__ inline float at_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ inline float row_max4(float x) {  // over the 4 lane groups (same lane % 16)
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ inline float row_sum4(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

// Rows of a workgroup and of a wave: NH halves of 16 rows a wave, 4 waves.
// A table tile (AT_WT rows) is split over AT_WT / (64 NH) workgroups.
template <int NH>
struct AtRows {
  static constexpr int WR = 16 * NH;        // rows a wave owns
  static constexpr int WG = 4 * WR;         // rows a workgroup owns
  static constexpr int SUB = AT_WT / WG;    // workgroups per table tile
  static_assert(NH == 1 || NH == 2, "one or two 16-row halves a wave");
};

// Decode blockIdx.x = (table tile * SUB + sub) * H + h.
template <int NH>
__device__ inline void at_block(int H, int& tile, int& sub, int& h) {
  const int b = blockIdx.x / H;
  h = blockIdx.x % H;
  tile = b / AtRows<NH>::SUB;
  sub = b % AtRows<NH>::SUB;
}

// ---------------------------------------------------------------------------
// forward: workgroup = 64 NH queries of one view and head; wave w owns
// 16 NH of them (halves a).  Per step of T keys, every K fragment read from
// LDS feeds all halves, and so does every V fragment.  The next step's tiles
// are requested into the other pair of LDS tiles before this step computes.
// 128-query workgroups of d = 128 take 32 keys a step: three of them fit a CU
// then, and a step's softmax and LDS waits hide behind the products of two
// other waves (the 64k call: 2,634 us against 2,870 with 64 keys and two
// workgroups).  At d = 64 three and more fit with 64 keys too (30,000 rows, 16
// heads: 598 us with 32 keys, 574 with 64; held to the registers of four
// workgroups neither was faster).
// 64-query ones, used where the chip is not full, take 64 (11.7 us against
// 13.6 for 2,000 rows of 6 heads of 64).
// ---------------------------------------------------------------------------
template <int D, int NH>
__global__ __launch_bounds__(AT_THR, NH == 2 ? 3 : 2) void k_attn_fwd(const int32_t* __restrict__ views,
                                                        const int32_t* __restrict__ qtiles, int H, float scale,
                                                        const bf16* __restrict__ q, const bf16* __restrict__ kv_k,
                                                        const bf16* __restrict__ kv_v, bf16* __restrict__ o,
                                                        float* __restrict__ lse) {
  using F = Frag<bf16>;
  using L = AtTile<D>;
  using R = AtRows<NH>;
  constexpr int NS = D / 32;  // 32-deep steps over d
  constexpr int NJ = D / 16;  // 16-column output tiles
  constexpr int T = D == 128 && NH == 2 ? 32 : 64;   // keys of a step
  __shared__ __align__(16) bf16 sT[2][2][T * D];   // [buffer][K, V]
  int tile, sub, h;
  at_block<NH>(H, tile, sub, h);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int v = qtiles[2 * tile], t0 = qtiles[2 * tile + 1] + R::WG * sub;
  const int32_t* vw = views + 4 * v;
  const int64_t qrow0 = vw[V_QROW];
  const int l = vw[V_L], hh = vw[V_H];
  const int64_t kvoff = vw[V_KVOFF];
  const int nq = min(R::WG, l - t0);
  if (nq <= 0) return;                      // the view ends in an earlier workgroup of the tile
  const int kv_end = hh + t0 + nq;          // keys the workgroup's last query sees
  const AtRequest<D> req(H, w, lane);
  req.template rows<T>(kv_k, kvoff, kv_end, h, sT[0][0]);
  req.template rows<T>(kv_v, kvoff, kv_end, h, sT[0][1]);
  const int i = lane & 15, g = lane >> 4;
  const int wq0 = t0 + R::WR * w;           // the wave's first query (within the view)
  const bool wave_live = R::WR * w < nq;
  bf16x8 qf[NH][NS];
#pragma unroll
  for (int a = 0; a < NH; ++a) {
    const int r = min(R::WR * w + 16 * a, nq - 1);      // (halves past the view read its last row)
    at_frags<D>(qf[a], q, qrow0 + t0 + r, nq - 1 - r, H, h, lane);
  }
  const int wave_end = min(kv_end, hh + wq0 + R::WR);   // keys the wave's last query sees
  const float c2 = scale * AT_LOG2E;        // scores in base 2
  float m[NH], lsum[NH];
  f32x4 acc[NH][NJ];
#pragma unroll
  for (int a = 0; a < NH; ++a) {
    m[a] = AT_NEG;
    lsum[a] = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int buf = 0;
  for (int k0 = 0; k0 < kv_end; k0 += T, buf ^= 1) {
    lds_landed();                            // this step's tiles are here, the other pair's readers are done
    if (k0 + T < kv_end) {
      req.template rows<T>(kv_k, kvoff + k0 + T, kv_end - k0 - T, h, sT[buf ^ 1][0]);
      req.template rows<T>(kv_v, kvoff + k0 + T, kv_end - k0 - T, h, sT[buf ^ 1][1]);
    }
    if (!wave_live || k0 >= wave_end) continue;      // wave-uniform
    const bf16 *sK = sT[buf][0], *sV = sT[buf][1];
    // S^T tiles: lane (g, i) of half a gets S[q = wq0 + 16 a + i][key = k0 + 16 j + 4 g + r]
    f32x4 sc[NH][T / 16];
#pragma unroll
    for (int j = 0; j < T / 16; ++j)
#pragma unroll
      for (int a = 0; a < NH; ++a) sc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the product blocks run at raised wave priority, so that the SIMD's
    // other waves do their softmax work while this one feeds the matrix core
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int j = 0; j < T / 16; ++j) {
        const bf16x8 kf = L::kc(sK, 16 * j, s, lane);
#pragma unroll
        for (int a = 0; a < NH; ++a) F::mma(sc[a][j], kf, qf[a][s]);
      }
    __builtin_amdgcn_s_setprio(0);
    // steps that cross the diagonal: keys past a query's last visible key
    if (k0 + T > hh + wq0 + 1) {
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        const int lim = hh + wq0 + 16 * a + i - k0 - 4 * g;
#pragma unroll
        for (int j = 0; j < T / 16; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * j + r > lim) sc[a][j][r] = AT_NEG;
      }
    }
    // online softmax in base 2 against a reference maximum m per row: it is
    // raised (and the accumulators rescaled) only when some score of the
    // wave exceeds its row's m by more than the slack, and until it is the
    // maximum of the first 64 keys: of 32 it is less often the row's own, whose
    // weight, the heaviest, then is 1 and not rounded to bf16
    float tmx[NH];
    bool raise = T < 64 && k0 == T;
#pragma unroll
    for (int a = 0; a < NH; ++a) {
      float x = sc[a][0][0];
#pragma unroll
      for (int j = 0; j < T / 16; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) x = fmaxf(x, sc[a][j][r]);
      tmx[a] = x * c2;
      raise |= tmx[a] > m[a] + AT_SLACK;
    }
    if (__ballot(raise) != 0ull) {
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        const float mn = fmaxf(m[a], row_max4(tmx[a]));
        const float corr = at_exp2(m[a] - mn);
        m[a] = mn;
        lsum[a] *= corr;
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[a][j] *= corr;
      }
    }
#pragma unroll
    for (int a = 0; a < NH; ++a) {
      const float nm = -m[a];
#pragma unroll
      for (int j = 0; j < T / 16; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = at_exp2(fmaf(sc[a][j][r], c2, nm));
          sc[a][j][r] = p;
          lsum[a] += p;          // this lane's share of the row sum
        }
    }
    // O^T += V^T P^T: lane (g, i) of half a gets O[q = wq0 + 16 a + i][d = 16 jn + 4 g + r]
#pragma unroll
    for (int s2 = 0; s2 < T / 32; ++s2) {
      bf16x8 pf[NH];
#pragma unroll
      for (int a = 0; a < NH; ++a) pf[a] = RegB<bf16>::pack(sc[a] + 2 * s2);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        const bf16x8 vf = L::km(sV, 32 * s2, 16 * jn, lane);
#pragma unroll
        for (int a = 0; a < NH; ++a) F::mma(acc[a][jn], vf, pf[a]);
      }
      __builtin_amdgcn_s_setprio(0);
    }
  }
#pragma unroll
  for (int a = 0; a < NH; ++a) lsum[a] = row_sum4(lsum[a]);
#pragma unroll
  for (int a = 0; a < NH; ++a) {
    if (R::WR * w + 16 * a + i < nq) {
      const float inv = lsum[a] > 0.f ? 1.f / lsum[a] : 0.f;
      const int64_t row = qrow0 + wq0 + 16 * a + i;
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn)
        Vec4<bf16>::store(o + (row * H + h) * D + 16 * jn + 4 * g, acc[a][jn] * inv);
      if (g == 0) lse[row * H + h] = (m[a] + log2f(lsum[a])) / AT_LOG2E;   // natural log of sum exp(scale s)
    }
  }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// delta = dO . o of 256 (row, head) entries from e0, D / 8 lanes an entry.
template <int D>
__device__ inline void at_delta(int64_t e0, int64_t n, const bf16* __restrict__ o, const bf16* __restrict__ dO,
                                float* __restrict__ delta) {
  constexpr int LPE = D / 8, EPI = AT_THR / LPE;   // lanes an entry, entries a round
  const int c = threadIdx.x % LPE;
#pragma unroll 2
  for (int k0 = 0; k0 < AT_THR / EPI; ++k0) {
    const int64_t r = e0 + EPI * k0 + threadIdx.x / LPE;
    float x = 0.f;
    if (r < n) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(o + r * D + 8 * c);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(dO + r * D + 8 * c);
#pragma unroll
      for (int k = 0; k < 8; ++k) x = fmaf(static_cast<float>(a[k]), static_cast<float>(b[k]), x);
    }
#pragma unroll
    for (int m = LPE / 2; m >= 1; m >>= 1) x += __shfl_xor(x, m);
    if (c == 0 && r < n) delta[r] = x;
  }
}

// dq: workgroup = 64 NH queries of one view and head, wave w owns 16 NH of
// them; delta = dO . o of its rows first; per 64-key step S and dP from the K
// and V tiles (each fragment feeding all halves), dS = P (dP - delta),
// dQ += dS K.  The workgroups past the tiles' write delta of all C rows for
// the dk/dv kernel: as a kernel of their own (one thread an entry) they took
// 215 us of an 11.8 ms backward and a launch of every small one.  Where dq is
// written over o they go first, in a launch of their own, and the tiles read
// delta and not o (have_delta).
template <int D, int NH>
__global__ __launch_bounds__(AT_THR, D == 64 && NH == 2 ? 4 : 2) void k_attn_dq(
    const int32_t* __restrict__ views, const int32_t* __restrict__ qtiles, int H, float scale,
    const bf16* __restrict__ q, const bf16* __restrict__ kv_k, const bf16* __restrict__ kv_v,
    const bf16* __restrict__ o, const bf16* __restrict__ dO, const float* __restrict__ lse, uint32_t n_tile_wg,
    int64_t n_rows, int have_delta, float* __restrict__ delta, bf16* __restrict__ dq) {
  using F = Frag<bf16>;
  using L = AtTile<D>;
  using R = AtRows<NH>;
  constexpr int NS = D / 32, NJ = D / 16;
  constexpr int T = D == 64 && NH == 2 ? 32 : 64;   // keys of a step
  __shared__ __align__(16) bf16 sT[2][2][T * D];   // [buffer][K, V]
  if (blockIdx.x >= n_tile_wg) {
    at_delta<D>(static_cast<int64_t>(blockIdx.x - n_tile_wg) * AT_THR, n_rows, o, dO, delta);
    return;
  }
  int tile, sub, h;
  at_block<NH>(H, tile, sub, h);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int v = qtiles[2 * tile], t0 = qtiles[2 * tile + 1] + R::WG * sub;
  const int32_t* vw = views + 4 * v;
  const int64_t qrow0 = vw[V_QROW];
  const int l = vw[V_L], hh = vw[V_H];
  const int64_t kvoff = vw[V_KVOFF];
  const int nq = min(R::WG, l - t0);
  if (nq <= 0) return;
  const int kv_end = hh + t0 + nq;
  const AtRequest<D> req(H, w, lane);
  req.template rows<T>(kv_k, kvoff, kv_end, h, sT[0][0]);
  req.template rows<T>(kv_v, kvoff, kv_end, h, sT[0][1]);
  const int i = lane & 15, g = lane >> 4;
  const int wq0 = t0 + R::WR * w;
  bf16x8 qf[NH][NS], df[NH][NS];
  float l2[NH], dl[NH];
#pragma unroll
  for (int a = 0; a < NH; ++a) {
    const int r = min(R::WR * w + 16 * a, nq - 1), last = nq - 1 - r;
    const bool live = R::WR * w + 16 * a + i < nq;
    const int64_t row = qrow0 + (live ? wq0 + 16 * a + i : t0);
    at_frags<D>(qf[a], q, qrow0 + t0 + r, last, H, h, lane);
    at_frags<D>(df[a], dO, qrow0 + t0 + r, last, H, h, lane);
    if (have_delta) {
      dl[a] = delta[row * H + h];
    } else {
      bf16x8 of[NS];
      at_frags<D>(of, o, qrow0 + t0 + r, last, H, h, lane);
      float x = 0.f;
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) x = fmaf(static_cast<float>(of[s][e]), static_cast<float>(df[a][s][e]), x);
      dl[a] = row_sum4(x);
    }
    l2[a] = live ? lse[row * H + h] * AT_LOG2E : 0.f;
  }
  const bool wave_live = R::WR * w < nq;
  const int wave_end = min(kv_end, hh + wq0 + R::WR);
  const float c2 = scale * AT_LOG2E;
  f32x4 acc[NH][NJ];
#pragma unroll
  for (int a = 0; a < NH; ++a)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int buf = 0;
  for (int k0 = 0; k0 < kv_end; k0 += T, buf ^= 1) {
    lds_landed();
    if (k0 + T < kv_end) {
      req.template rows<T>(kv_k, kvoff + k0 + T, kv_end - k0 - T, h, sT[buf ^ 1][0]);
      req.template rows<T>(kv_v, kvoff + k0 + T, kv_end - k0 - T, h, sT[buf ^ 1][1]);
    }
    if (!wave_live || k0 >= wave_end) continue;
    const bf16 *sK = sT[buf][0], *sV = sT[buf][1];
    // per 16-key group j: S and dP over d, then dS = P (dP - delta) with
    // P = exp(scale s - lse), so that dP lives for one group only
    f32x4 sc[NH][T / 16];
#pragma unroll
    for (int j = 0; j < T / 16; ++j) {
      f32x4 dp[NH];
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        sc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        dp[a] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bf16x8 kf = L::kc(sK, 16 * j, s, lane);
#pragma unroll
        for (int a = 0; a < NH; ++a) F::mma(sc[a][j], kf, qf[a][s]);
        const bf16x8 vf = L::kc(sV, 16 * j, s, lane);
#pragma unroll
        for (int a = 0; a < NH; ++a) F::mma(dp[a], vf, df[a][s]);
      }
#pragma unroll
      for (int a = 0; a < NH; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = at_exp2(fmaf(sc[a][j][r], c2, -l2[a]));
          sc[a][j][r] = p * (dp[a][r] - dl[a]);
        }
    }
    // steps that cross the diagonal, or hold rows past the view: zero what
    // the row cannot see
    if (k0 + T > hh + wq0 + 1 || R::WR * (w + 1) > nq) {
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        const int lim = R::WR * w + 16 * a + i < nq ? hh + wq0 + 16 * a + i - k0 - 4 * g : -T;
#pragma unroll
        for (int j = 0; j < T / 16; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * j + r > lim) sc[a][j][r] = 0.f;
      }
    }
    // dQ^T += K^T dS^T: lane (g, i) of half a gets dQ[q = wq0 + 16 a + i][d = 16 jn + 4 g + r]
#pragma unroll
    for (int s2 = 0; s2 < T / 32; ++s2) {
      bf16x8 sf[NH];
#pragma unroll
      for (int a = 0; a < NH; ++a) sf[a] = RegB<bf16>::pack(sc[a] + 2 * s2);
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        const bf16x8 kt = L::km(sK, 32 * s2, 16 * jn, lane);
#pragma unroll
        for (int a = 0; a < NH; ++a) F::mma(acc[a][jn], kt, sf[a]);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < NH; ++a) {
    if (R::WR * w + 16 * a + i < nq) {
      const int64_t row = qrow0 + wq0 + 16 * a + i;
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn)
        Vec4<bf16>::store(dq + (row * H + h) * D + 16 * jn + 4 * g, acc[a][jn] * scale);
    }
  }
}

// dk, dv: workgroup = 64 NH keys of one view row and head, wave w owns
// 16 NH of them (halves b); per 32-query step over the queries that see
// them, P and dS from the Q and dO tiles, dV += P^T dO and dK += scale dS^T Q,
// each Q and dO fragment feeding all halves.  The keys' K fragments stay in
// registers, their V rows in LDS: with both in registers, and the next step's
// tiles on their way through registers, two halves of keys did not fit beside
// their 128 accumulator registers, and one half read every Q and dO fragment
// for one product (64k call, 16 heads of 128: 8,021 -> 6,250 us, 624 -> 805
// TFLOP/s).  What bounds it now: two waves a SIMD, each with a chain of LDS
// reads, products, exponentials and products a step (MFMA busy 40%, LDS 28%).
// Three waves of one half each: 7,176 us.  Raised priority around the products
// adds 1% to the backward (10,080 -> 10,170 us; nothing at d = 64, and 10% with
// one half a wave).  At d = 64 the two halves fit three waves a SIMD (30,000
// rows, 16 heads: 1,545 -> 1,355 us).
template <int D, int NH>
__global__ __launch_bounds__(AT_THR, D == 64 ? 3 : 2) void k_attn_dkdv(
    const int32_t* __restrict__ views, const int32_t* __restrict__ kvtiles, int H, float scale,
    const bf16* __restrict__ q, const bf16* __restrict__ kv_k, const bf16* __restrict__ kv_v,
    const bf16* __restrict__ dO, const float* __restrict__ lse, const float* __restrict__ delta,
    float* __restrict__ dk_view, float* __restrict__ dv_view) {
  using F = Frag<bf16>;
  using L = AtTile<D>;
  using R = AtRows<NH>;
  constexpr int NS = D / 32, NJ = D / 16;
  constexpr int TQ = AT_TQ * D;
  // the requested tiles first (they have to lie in the first 64 KB):
  // [buffer][Q, dO], then the keys' V rows; then lse and delta of a step
  __shared__ __align__(16) bf16 sT[4 * TQ + R::WG * D + 2 * 2 * AT_TQ * 2];
  bf16* const sV = sT + 4 * TQ;
  float* const sL = reinterpret_cast<float*>(sV + R::WG * D);    // [buffer][lse, delta][AT_TQ]
  int tile, sub, h;
  at_block<NH>(H, tile, sub, h);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int v = kvtiles[2 * tile], k0 = kvtiles[2 * tile + 1] + R::WG * sub;
  const int32_t* vw = views + 4 * v;
  const int64_t qrow0 = vw[V_QROW];
  const int l = vw[V_L], hh = vw[V_H];
  const int64_t kvoff = vw[V_KVOFF];
  const int nk = min(R::WG, hh + l - k0);
  if (nk <= 0) return;
  const int i = lane & 15, g = lane >> 4;
  const int wk0 = k0 + R::WR * w;           // the wave's first key (within the view row)
  // queries that see key k0 or later: qi >= k0 - hh
  const int q_first = max(0, k0 - hh);
  const int tq0 = (q_first / AT_TQ) * AT_TQ;
  const AtRequest<D> req(H, w, lane);
  req.template rows<R::WG>(kv_v, kvoff + k0, nk, h, sV);
  req.template rows<AT_TQ>(q, qrow0 + tq0, l - tq0, h, sT);
  req.template rows<AT_TQ>(dO, qrow0 + tq0, l - tq0, h, sT + TQ);
  bf16x8 kf[NH][NS];
#pragma unroll
  for (int b = 0; b < NH; ++b) {
    const int r = min(R::WR * w + 16 * b, nk - 1);
    at_frags<D>(kf[b], kv_k, kvoff + k0 + r, nk - 1 - r, H, h, lane);
  }
  // lse and delta of a step's queries (threads 0..63): step 0's into LDS
  // now, the next step's waits in a register until its buffer is free
  const auto stat = [&](int s0) __attribute__((always_inline)) {
    const int r = min(s0 + (t & (AT_TQ - 1)), l - 1);   // (past the view: never used)
    const float* src = (t & AT_TQ) == 0 ? lse : delta;
    return src[(qrow0 + r) * H + h];
  };
  if (t < 2 * AT_TQ) sL[t] = stat(tq0);
  float pl = stat(tq0 + AT_TQ);
  const bool wave_live = R::WR * w < nk;
  f32x4 dk[NH][NJ], dv[NH][NJ];
#pragma unroll
  for (int b = 0; b < NH; ++b)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      dk[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      dv[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  const float c2 = scale * AT_LOG2E;
  int buf = 0;
  for (int t0 = tq0; t0 < l; t0 += AT_TQ, buf ^= 1) {
    const int nq = min(AT_TQ, l - t0);
    lds_landed();
    if (t0 + AT_TQ < l) {
      // (before the requests: the wait for pl must not become one for them)
      if (t < 2 * AT_TQ) sL[(buf ^ 1) * 2 * AT_TQ + t] = pl;
      bf16* nt = sT + (buf ^ 1) * 2 * TQ;
      req.template rows<AT_TQ>(q, qrow0 + t0 + AT_TQ, l - t0 - AT_TQ, h, nt);
      req.template rows<AT_TQ>(dO, qrow0 + t0 + AT_TQ, l - t0 - AT_TQ, h, nt + TQ);
      pl = stat(t0 + 2 * AT_TQ);
    }
    // no query of the step sees the wave's first key: skip (wave-uniform)
    if (!wave_live || wk0 > hh + t0 + nq - 1) continue;
    const bf16 *sQ = sT + buf * 2 * TQ, *sD = sQ + TQ;
    const float* sl = sL + buf * 2 * AT_TQ;
    // lane (g, i) of half b gets S[q = t0 + 16 j + 4 g + r][key = wk0 + 16 b + i]
    f32x4 sc[NH][2], dp[NH][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int b = 0; b < NH; ++b) {
        sc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        dp[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 qa = L::kc(sQ, 16 * j, s, lane);
#pragma unroll
        for (int b = 0; b < NH; ++b) F::mma(sc[b][j], qa, kf[b][s]);
      }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      bf16x8 vf[NH];
#pragma unroll
      for (int b = 0; b < NH; ++b) vf[b] = L::kc(sV, R::WR * w + 16 * b, s, lane);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 da = L::kc(sD, 16 * j, s, lane);
#pragma unroll
        for (int b = 0; b < NH; ++b) F::mma(dp[b][j], da, vf[b]);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 lq = *reinterpret_cast<const f32x4*>(sl + 16 * j + 4 * g) * AT_LOG2E;
      const f32x4 dq4 = *reinterpret_cast<const f32x4*>(sl + AT_TQ + 16 * j + 4 * g);
#pragma unroll
      for (int b = 0; b < NH; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = at_exp2(fmaf(sc[b][j][r], c2, -lq[r]));
          sc[b][j][r] = p;                            // P
          dp[b][j][r] = p * (dp[b][j][r] - dq4[r]);   // dS
        }
    }
    // steps where some query does not see some key of the wave (the
    // diagonal, rows past the view, keys past the view row): zero those
    if (!(wk0 + R::WR - 1 <= hh + t0 && nq == AT_TQ && R::WR * (w + 1) <= nk)) {
#pragma unroll
      for (int b = 0; b < NH; ++b) {
        const int key = wk0 + 16 * b + i;
        const int kl = key < hh + l ? key - hh - t0 : INT32_MAX;   // visible iff kl <= query row
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int qr = 16 * j + 4 * g + r;        // query row within the step
            if (qr >= nq || kl > qr) {
              sc[b][j][r] = 0.f;
              dp[b][j][r] = 0.f;
            }
          }
      }
    }
    // dV^T += dO^T P, dK^T += Q^T dS: lane (g, i) of half b gets [key][d = 16 jn + 4 g + r]
    bf16x8 pf[NH], sf[NH];
#pragma unroll
    for (int b = 0; b < NH; ++b) {
      pf[b] = RegB<bf16>::pack(sc[b]);
      sf[b] = RegB<bf16>::pack(dp[b]);
    }
#pragma unroll
    for (int jn = 0; jn < NJ; ++jn) {
      const bf16x8 dt = L::km(sD, 0, 16 * jn, lane);
#pragma unroll
      for (int b = 0; b < NH; ++b) F::mma(dv[b][jn], dt, pf[b]);
      const bf16x8 qt = L::km(sQ, 0, 16 * jn, lane);
#pragma unroll
      for (int b = 0; b < NH; ++b) F::mma(dk[b][jn], qt, sf[b]);
    }
  }
#pragma unroll
  for (int b = 0; b < NH; ++b) {
    if (R::WR * w + 16 * b + i < nk) {
      const int64_t e = (kvoff + wk0 + 16 * b + i) * H + h;
#pragma unroll
      for (int jn = 0; jn < NJ; ++jn) {
        *reinterpret_cast<f32x4*>(dk_view + e * D + 16 * jn + 4 * g) = dk[b][jn] * scale;
        *reinterpret_cast<f32x4*>(dv_view + e * D + 16 * jn + 4 * g) = dv[b][jn];
      }
    }
  }
}

// view rows <- compact rows (bf16, 16-byte pieces): a thread moves the same
// piece of AT_GR consecutive view rows, their loads in flight together
constexpr int AT_GR = 4;
__global__ __launch_bounds__(AT_THR) void k_attn_gather(const bf16* __restrict__ src,
                                                        const int32_t* __restrict__ rows, int64_t n_kv,
                                                        int64_t C, int row_elems, bf16* __restrict__ dst) {
  const int vpr = row_elems / 8;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * AT_THR + threadIdx.x;
  const int64_t e0 = (idx / vpr) * AT_GR;
  if (e0 >= n_kv) return;
  const int c = static_cast<int>(idx % vpr) * 8;
  int32_t r[AT_GR];
#pragma unroll
  for (int q = 0; q < AT_GR; ++q) r[q] = e0 + q < n_kv ? rows[e0 + q] : -1;
  uint4 v[AT_GR];
#pragma unroll
  for (int q = 0; q < AT_GR; ++q) {
    v[q] = uint4{0u, 0u, 0u, 0u};
    if (r[q] >= 0 && r[q] < C) v[q] = *reinterpret_cast<const uint4*>(src + static_cast<int64_t>(r[q]) * row_elems + c);
  }
#pragma unroll
  for (int q = 0; q < AT_GR; ++q)
    if (e0 + q < n_kv) *reinterpret_cast<uint4*>(dst + (e0 + q) * row_elems + c) = v[q];
}

// compact rows <- sum of their view rows, in the row's (fixed) entry order;
// the entries are taken AT_GR at a time, their indices and then their rows
// requested together (an entry past the row's last, or invalid, adds zero)
__global__ __launch_bounds__(AT_THR) void k_attn_scatter(const float* __restrict__ src,
                                                         const int64_t* __restrict__ row_off,
                                                         const int32_t* __restrict__ ent, int64_t C,
                                                         int64_t n_kv, int row_elems, bf16* __restrict__ dst) {
  const int vpr = row_elems / 4;
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * AT_THR + threadIdx.x;
  const int64_t r = idx / vpr;
  if (r >= C) return;
  const int c = static_cast<int>(idx % vpr) * 4;
  const int64_t b = row_off[r] < 0 ? 0 : row_off[r];
  const int64_t e_end = row_off[r + 1] > n_kv ? n_kv : row_off[r + 1];
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int64_t j = b; j < e_end; j += AT_GR) {
    int32_t e[AT_GR];
#pragma unroll
    for (int q = 0; q < AT_GR; ++q) {
      e[q] = j + q < e_end ? ent[j + q] : -1;
      if (e[q] >= n_kv) e[q] = -1;
    }
    f32x4 v[AT_GR];
#pragma unroll
    for (int q = 0; q < AT_GR; ++q) {
      v[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (e[q] >= 0) v[q] = *reinterpret_cast<const f32x4*>(src + static_cast<int64_t>(e[q]) * row_elems + c);
    }
#pragma unroll
    for (int q = 0; q < AT_GR; ++q)
      if (e[q] >= 0) acc += v[q];
  }
  Vec4<bf16>::store(dst + r * row_elems + c, acc);
}

int at_status(const char* where) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(where) + ": " + hipGetErrorString(e));
    return HARTS_EHIP;
  }
  return HARTS_OK;
}

bool at16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Whether 128-row workgroups (two 16-row halves a wave) give every CU two;
// fewer take 64-row ones, whose chains of steps are as long but twice as many
// (2,000 rows, 6 heads of 64, about 120 workgroups of 128 rows: forward 16.0
// -> 11.5 us, dq 19.0 -> 15.2 us).
bool at_fills(int64_t tiles, int32_t H) { return tiles * H >= 512; }

int check_attn(int32_t H, int32_t d, const char* where) {
  if (H < 1 || H > 65535 || (d != 64 && d != 128)) {
    set_error(std::string(where) + ": need 1 <= H <= 65535 and d in {64, 128}");
    return HARTS_EUNSUPPORTED;
  }
  return HARTS_OK;
}

}  // namespace
}  // namespace harts

using namespace harts;

extern "C" int harts_attn_fwd(const int32_t* views, const int32_t* qtiles, int64_t n_qtiles, int32_t H,
                              int32_t d, float scale, const void* q, const void* kv_k, const void* kv_v,
                              void* o, float* lse, void* stream) {
  if (int rc = check_attn(H, d, "harts_attn_fwd")) return rc;
  if (n_qtiles < 0 || n_qtiles * 2 * H > INT32_MAX) { set_error("harts_attn_fwd: bad tile count"); return HARTS_EINVAL; }
  if (n_qtiles == 0) return HARTS_OK;
  if (!views || !qtiles || !q || !kv_k || !kv_v || !o || !lse || !at16(q) || !at16(kv_k) || !at16(kv_v) ||
      !at16(o)) {
    set_error("harts_attn_fwd: NULL or misaligned pointer");
    return HARTS_EINVAL;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const auto* bq = static_cast<const bf16*>(q);
  const auto* bk = static_cast<const bf16*>(kv_k);
  const auto* bv = static_cast<const bf16*>(kv_v);
  auto* bo = static_cast<bf16*>(o);
  const auto launch = [&](auto kernel, int sub) {
    hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(n_qtiles * sub * H)), dim3(AT_THR), 0, s, views, qtiles, H,
                       scale, bq, bk, bv, bo, lse);
  };
  if (at_fills(n_qtiles, H)) {
    if (d == 128) launch(k_attn_fwd<128, 2>, AtRows<2>::SUB);
    else launch(k_attn_fwd<64, 2>, AtRows<2>::SUB);
  } else {
    if (d == 128) launch(k_attn_fwd<128, 1>, AtRows<1>::SUB);
    else launch(k_attn_fwd<64, 1>, AtRows<1>::SUB);
  }
  return at_status("k_attn_fwd");
}

extern "C" int harts_attn_bwd(const int32_t* views, const int32_t* qtiles, int64_t n_qtiles,
                              const int32_t* kvtiles, int64_t n_kvtiles, int64_t C, int32_t H, int32_t d,
                              float scale, const void* q, const void* kv_k, const void* kv_v, const void* o,
                              const float* lse, const void* dO, float* delta, void* dq, float* dk_view,
                              float* dv_view, void* stream) {
  if (int rc = check_attn(H, d, "harts_attn_bwd")) return rc;
  if (n_qtiles < 0 || n_kvtiles < 0 || C < 0 || n_qtiles * 2 * H > INT32_MAX || n_kvtiles * 2 * H > INT32_MAX) {
    set_error("harts_attn_bwd: bad sizes");
    return HARTS_EINVAL;
  }
  if (C == 0) return HARTS_OK;
  if (!views || !qtiles || !kvtiles || !q || !kv_k || !kv_v || !o || !lse || !dO || !delta || !dq || !dk_view ||
      !dv_view || !at16(q) || !at16(kv_k) || !at16(kv_v) || !at16(o) || !at16(dO) || !at16(dq) ||
      !at16(dk_view) || !at16(dv_view)) {
    set_error("harts_attn_bwd: NULL or misaligned pointer");
    return HARTS_EINVAL;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const auto* bq = static_cast<const bf16*>(q);
  const auto* bk = static_cast<const bf16*>(kv_k);
  const auto* bv = static_cast<const bf16*>(kv_v);
  const auto* bo = static_cast<const bf16*>(o);
  const auto* bd = static_cast<const bf16*>(dO);
  auto* bdq = static_cast<bf16*>(dq);
  const int64_t n = C * H;
  // dq over o: a workgroup's delta would read what another's dq has written
  const uintptr_t o0 = reinterpret_cast<uintptr_t>(o), q0 = reinterpret_cast<uintptr_t>(dq);
  const bool over = (o0 < q0 ? q0 - o0 : o0 - q0) < static_cast<uintptr_t>(n) * d * sizeof(bf16);
  const auto launch_dq = [&](auto kernel, int sub) {
    const uint32_t tiles = static_cast<uint32_t>(n_qtiles * sub * H);
    const uint32_t rows = static_cast<uint32_t>((n + AT_THR - 1) / AT_THR);
    const auto go = [&](uint32_t t, uint32_t r, int have_delta) {
      if (t + r > 0)
        hipLaunchKernelGGL(kernel, dim3(t + r), dim3(AT_THR), 0, s, views, qtiles, H, scale, bq, bk, bv, bo, bd, lse,
                           t, n, have_delta, delta, bdq);
    };
    if (over) go(0, rows, 0);
    go(tiles, over ? 0 : rows, over);
  };
  if (at_fills(n_qtiles, H)) {
    if (d == 128) launch_dq(k_attn_dq<128, 2>, AtRows<2>::SUB);
    else launch_dq(k_attn_dq<64, 2>, AtRows<2>::SUB);
  } else {
    if (d == 128) launch_dq(k_attn_dq<128, 1>, AtRows<1>::SUB);
    else launch_dq(k_attn_dq<64, 1>, AtRows<1>::SUB);
  }
  if (int rc = at_status("k_attn_dq")) return rc;
  if (n_kvtiles > 0) {
    const auto launch = [&](auto kernel, int sub) {
      hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(n_kvtiles * sub * H)), dim3(AT_THR), 0, s, views, kvtiles,
                         H, scale, bq, bk, bv, bd, lse, delta, dk_view, dv_view);
    };
    if (at_fills(n_kvtiles, H)) {
      if (d == 128) launch(k_attn_dkdv<128, 2>, AtRows<2>::SUB);
      else launch(k_attn_dkdv<64, 2>, AtRows<2>::SUB);
    } else {
      if (d == 128) launch(k_attn_dkdv<128, 1>, AtRows<1>::SUB);
      else launch(k_attn_dkdv<64, 1>, AtRows<1>::SUB);
    }
    if (int rc = at_status("k_attn_dkdv")) return rc;
  }
  return HARTS_OK;
}

extern "C" int harts_attn_gather(const void* src, const int32_t* kv_rows, int64_t n_kv, int64_t C, int32_t H,
                                 int32_t d, void* dst, void* stream) {
  if (int rc = check_attn(H, d, "harts_attn_gather")) return rc;
  if (n_kv < 0 || C < 0) { set_error("harts_attn_gather: bad sizes"); return HARTS_EINVAL; }
  if (n_kv == 0) return HARTS_OK;
  if (!src || !kv_rows || !dst || !at16(src) || !at16(dst)) {
    set_error("harts_attn_gather: NULL or misaligned pointer");
    return HARTS_EINVAL;
  }
  const int row_elems = H * d;
  const int64_t threads = (n_kv + AT_GR - 1) / AT_GR * (row_elems / 8);
  hipLaunchKernelGGL(k_attn_gather, dim3(static_cast<uint32_t>((threads + AT_THR - 1) / AT_THR)), dim3(AT_THR),
                     0, static_cast<hipStream_t>(stream), static_cast<const bf16*>(src), kv_rows, n_kv, C,
                     row_elems, static_cast<bf16*>(dst));
  return at_status("k_attn_gather");
}

extern "C" int harts_attn_scatter(const float* src, const int64_t* row_off, const int32_t* ent, int64_t C,
                                  int64_t n_kv, int32_t H, int32_t d, void* dst, void* stream) {
  if (int rc = check_attn(H, d, "harts_attn_scatter")) return rc;
  if (n_kv < 0 || C < 0) { set_error("harts_attn_scatter: bad sizes"); return HARTS_EINVAL; }
  if (C == 0) return HARTS_OK;
  if (!src || !row_off || (!ent && n_kv > 0) || !dst || !at16(src) || !at16(dst)) {
    set_error("harts_attn_scatter: NULL or misaligned pointer");
    return HARTS_EINVAL;
  }
  const int row_elems = H * d;
  const int64_t threads = C * (row_elems / 4);
  hipLaunchKernelGGL(k_attn_scatter, dim3(static_cast<uint32_t>((threads + AT_THR - 1) / AT_THR)), dim3(AT_THR),
                     0, static_cast<hipStream_t>(stream), src, row_off, ent, C, n_kv, row_elems,
                     static_cast<bf16*>(dst));
  return at_status("k_attn_scatter");
}
