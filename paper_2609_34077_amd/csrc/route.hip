// Router logits + softmax + hard-mask / soft-prior Top-K + gates, fused in one kernel.
//
// Section 3.1 (Eq. 1): z = W x, p = softmax(z), A = Top-K(p), gates g_i = p_i or
// p_i / sum_{j in A} p_j. Section 3.2, Stage 1 (Eq. 2): A = Top-K(p * m) with a binary
// mask m; the gates computed from p * m equal those of p on A. Section 3.2, inference
// (Eq. 4): A = Top-K(p * pi) with a prior pi > 0; gates stay those of p.
//
// Experts are ranked on log-domain keys z_i + c_i, with c_i = 0 (plain), 0 or -inf
// (mask), log pi_i (prior); softmax is monotone with a shared normaliser, so these order
// experts exactly as the products do and avoid ties from exp underflow. Equal keys go to
// the lower expert index.
//
// bf16 logits use v_mfma_f32_16x16x32_bf16 (route_bf16_kernel): a workgroup computes a tile of
// (16*MB tokens) x (16*NB*WN outputs), where outputs are the rows of [L*E, d] router
// weights of whole layers; its WN*WK waves split the outputs (WN) and the k-steps (WK)
// and the WK partial tiles are summed in LDS in a fixed order. Small token counts
// (decode) use WK = 8..16 so all of d is in flight at once; large token counts stream x.
// Many tokens routed through many layers at once use tiles staged through LDS instead
// (route_mid_kernel, route_gemm_kernel, route_wide_kernel, route_tile_kernel).
// The selection reads the fp32 logits from LDS: up to 16 experts one 16-lane row per token (one layer)
// or one thread per (token, layer), above that one wavefront per pair where few share it (wave_selects).

#include <limits.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"
#include "permute_block.hpp"

namespace maskmoe {
namespace {

constexpr int kMaxRouteK = 16;
constexpr int kMaxK = kMaxRouteK;
constexpr int kMaxModeParams = 512;
// Selection by one thread per (token, layer) pair up to this many experts, by one wavefront
// (a lane per expert) above it when E <= 64. The softmax normaliser over all E experts (g = p)
// is summed in expert order for E <= kSelThreadE and E > 64; for kSelThreadE < E <= 64 in the
// order of a 64-lane butterfly: lane e with lane e ^ 32, then ^ 16, ..., ^ 1, experts past E
// counting as 0. The wavefront selection sums that way in six steps (a serial sum over the
// lanes took ~5 us of the 4096-token selection kernel), the per-thread selection replays the
// same tree, so every path gives the same bits.
constexpr int kSelThreadE = 16;
// Launches that the tile kernels (route_mid_kernel, route_gemm_kernel, route_wide_kernel,
// route_tile_kernel) can take: they all sum a logit in ascending order of k, as the 32-token tiles of
// route_bf16_kernel do, so that split and fused routing of the same call give the same bits whichever of
// them each takes. Their 32-bit offsets reach over a tile's rows.
inline bool route_tiles(int T, int d, int E, int L) {
  return d % 64 == 0 && d <= (1 << 20) && T >= kRouteSplitMinT && L * E > 64;
}
// Of these, launches with selection that take the 32-token tiles of route_bf16_kernel (`groups` of
// outputs): until they are more than one per CU, or two where short rows or many experts make the selection
// the longer part, they hide it better than the tile GEMMs. 9 and 32 layers of 8 experts, d 4096, 32-token
// tiles / tile GEMM: 600 tokens 54 / 64 and 100 / 130 us, 8192 tokens 55 / 65 and 103 / 132, 12000 tokens
// 101 / 66 and 187 / 134; 13 layers of 5 experts, d 1024, 16000 tokens 31 / 38, 33000 66 / 45; one layer of
// 100 experts, d 2048, 9000 tokens 137 / 155, 40000 251 / 177; of 256, 8192 tokens 171 / 384.
inline bool route_small_tiles(int T, int d, int E, int groups) {
  return (T + 31) / 32 * groups <= (d < 2048 || E > kWave ? 512 : 256);
}
constexpr int kRouteWideT = 32768;

struct RouteParams {
  const void* x;
  const void* w;       // [L, E, d] router weights of this launch's first layer
  int32_t* idx;        // [L, T, K]
  float* gate;         // [L, T, K]
  float* margin;       // [L, T] or null
  float* logits;       // [L, T, E] fp32 router logits or null
  int T, d, E, K, L, lpw, mode, gate_mode;
  PermBuffers pb;               // fused permutation (single-workgroup launches only)
  int n_shared, tile_rows;
  float modep[kMaxModeParams];  // [L, E]: mask (0/1) or prior values of this launch
};

__device__ __forceinline__ float key_offset(int mode, float v) {
  if (mode == 1) return v != 0.0f ? 0.0f : -INFINITY;  // hard mask
  if (mode == 2) return logf(v);                        // soft prior
  return 0.0f;                                          // plain
}

// Selection, gates and outputs of one (token, layer) pair: z the E fp32 logits, o the E key
// offsets, obase the pair's index in the [L, T] outputs. write_logits: also store z in p.logits.
// EC, KC: the expert and selection counts when known at compile time (0: p.E, p.K); the arithmetic
// is the same. The (K+1)-th pick is looked for only when the margin is asked for.
template <int EC = 0, int KC = 0>
__device__ __forceinline__ void select_pair(const RouteParams& p, const float* z, const float* o, size_t obase,
                                            bool write_logits) {
  constexpr int kMaxK = KC ? KC : kMaxRouteK;
  const int E = EC ? EC : p.E, K = KC ? KC : p.K;
  uint64_t tk0 = 0, tk1 = 0, tk2 = 0, tk3 = 0;
  int sel[kMaxK];
  float selz[kMaxK];
  float kth = -INFINITY, nxt = -INFINITY;
#pragma unroll
  for (int j = 0; j <= kMaxK; ++j) {
    if (j < K || (j == K && p.margin)) {
      float best = -INFINITY;
      int bi = -1;
#pragma unroll
      for (int e = 0; e < (EC ? EC : E); ++e) {
        const uint64_t word = e < 64 ? tk0 : e < 128 ? tk1 : e < 192 ? tk2 : tk3;
        if ((word >> (e & 63)) & 1ull) continue;
        const float key = z[e] + o[e];
        if (key > best) {
          best = key;
          bi = e;
        }
      }
      if (j < K) {
        if (bi < 0) {  // only reachable with non-finite logits: keep the output well formed
          for (int e = 0; e < E && bi < 0; ++e) {
            const uint64_t word = e < 64 ? tk0 : e < 128 ? tk1 : e < 192 ? tk2 : tk3;
            if (!((word >> (e & 63)) & 1ull)) bi = e;
          }
        }
        const uint64_t bit = 1ull << (bi & 63);
        if (bi < 64) tk0 |= bit; else if (bi < 128) tk1 |= bit; else if (bi < 192) tk2 |= bit; else tk3 |= bit;
        sel[j] = bi;
        selz[j] = z[bi];
        kth = best;
      } else {
        nxt = best;
      }
    }
  }

  float zref, norm = 0.0f;
  if (p.gate_mode == 0) {  // g = p_i: full softmax over all E experts
    zref = z[0];
    for (int e = 1; e < E; ++e) zref = fmaxf(zref, z[e]);
    if (E > kSelThreadE && E <= kWave) {   // the butterfly's tree (kSelThreadE)
      float a[kWave / 2];
#pragma unroll
      for (int i = 0; i < kWave / 2; ++i)
        a[i] = (i < E ? expf(z[i] - zref) : 0.0f) + (i + kWave / 2 < E ? expf(z[i + kWave / 2] - zref) : 0.0f);
#pragma unroll
      for (int w = kWave / 4; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) a[i] = a[i] + a[i + w];
      norm = a[0];
    } else {
      for (int e = 0; e < E; ++e) norm += expf(z[e] - zref);
    }
  } else {  // g = p_i / sum_{j in A} p_j
    zref = selz[0];
#pragma unroll
    for (int j = 1; j < kMaxK; ++j)
      if (j < K) zref = fmaxf(zref, selz[j]);
#pragma unroll
    for (int j = 0; j < kMaxK; ++j)
      if (j < K) norm += expf(selz[j] - zref);
  }
  const float inv = 1.0f / norm;
#pragma unroll
  for (int j = 0; j < kMaxK; ++j) {
    if (j < K) {
      p.idx[obase * K + j] = sel[j];
      p.gate[obase * K + j] = expf(selz[j] - zref) * inv;
    }
  }
  if (p.margin) p.margin[obase] = (nxt == -INFINITY) ? INFINITY : (kth - nxt);
  if (write_logits && p.logits)
    for (int e = 0; e < E; ++e) p.logits[obase * E + e] = z[e];
}

// Selection and gates for every (token, layer) pair of the tile. logits[tt * ld + lw*E + e]
// are the fp32 router logits, lo[lw*E + e] the key offsets. TOKEN_FASTEST: consecutive threads
// take consecutive tokens of one layer (conflict-free LDS reads when ld is odd, coalesced
// stores); otherwise consecutive layers of one token.
template <bool TOKEN_FASTEST = false>
__device__ void route_finalize(const RouteParams& p, const float* logits, int ld, const float* lo,
                               int t0, int TT, int lg0, int nl, int nthreads) {
  const int E = p.E;
  for (int pi = threadIdx.x; pi < TT * nl; pi += nthreads) {
    const int tt = TOKEN_FASTEST ? pi % TT : pi / nl;
    const int lw = TOKEN_FASTEST ? pi / TT : pi - tt * nl;
    const int t = t0 + tt;
    if (t >= p.T) continue;
    const float* z = logits + tt * ld + lw * E;
    const float* o = lo + lw * E;
    const size_t obase = (static_cast<size_t>(lg0 + lw) * p.T + t);

    select_pair(p, z, o, obase, true);
  }
}

// Split routing: the logits of every (token, layer) pair are first written to p.logits
// ([L, T, E] fp32, the caller's output or workspace) by the logit kernels, then selected here at
// full occupancy (the selection otherwise runs after the logit GEMM at the GEMM's occupancy).
// Pairs are taken token-fastest: pair q is (layer q / T, token q % T), its logits at q * E.
constexpr int kSelThreads = 256;

// E <= kSelThreadE: one thread per pair, the block's logits staged in LDS (odd row stride) so
// the per-pair selection reads them without bank conflicts. With E and K known at compile time the
// picks unroll without their runtime guards (4.2 M pairs of 8 experts, top-2: 65 -> 35 us; 30 us are
// the memory traffic).
template <int EC, int KC = 0>
__global__ __launch_bounds__(kSelThreads) void route_select_kernel(const RouteParams p) {
  constexpr int EMAX = EC ? EC : kSelThreadE;
  __shared__ float zs[kSelThreads * (EMAX + 1)];
  __shared__ float lo[kMaxModeParams];
  const int E = EC ? EC : p.E;
  const uint32_t pairs = static_cast<uint32_t>(p.L) * p.T;   // < 2^31
  const uint32_t q0 = blockIdx.x * kSelThreads;
  for (int i = threadIdx.x; i < p.L * E; i += kSelThreads) lo[i] = key_offset(p.mode, p.modep[i]);
  const int rows = pairs - q0 < kSelThreads ? static_cast<int>(pairs - q0) : kSelThreads;
  const float* src = p.logits + static_cast<size_t>(q0) * E;
  if ((E & 3) == 0) {   // 16-byte loads; a 4-float unit never straddles two rows
    for (int i = threadIdx.x; i < rows * E / 4; i += kSelThreads) {
      const f32x4 v = reinterpret_cast<const f32x4*>(src)[i];
      const int r = (4 * i) / E, c = 4 * i - r * E;
      float* d = zs + r * (E + 1) + c;
      d[0] = v[0];
      d[1] = v[1];
      d[2] = v[2];
      d[3] = v[3];
    }
  } else {
    for (int i = threadIdx.x; i < rows * E; i += kSelThreads) {
      const int r = i / E;
      zs[r * (E + 1) + i - r * E] = src[i];
    }
  }
  __syncthreads();
  const uint32_t q = q0 + threadIdx.x;
  if (q >= pairs) return;
  const int l = static_cast<int>(q / static_cast<uint32_t>(p.T));
  select_pair<EC, KC>(p, zs + threadIdx.x * (E + 1), lo + l * E, q, false);
}

// Lane exchanges within a 16-lane row (DPP): lane e of the row receives lane (e - R) mod 16.
template <int R>
__device__ __forceinline__ int row_ror(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x120 + R, 0xF, 0xF, false);
}

// Adds to `rank` the number of the row's keys src_key (of experts src_idx, one per lane,
// rotated by R .. 15 lanes within the row; R = 0 is the lane's own source) that rank above
// (key, idx): valid (above -inf, not NaN) and larger, or equal with a lower index. Branch-free.
template <int R>
__device__ __forceinline__ void rank_from_row(float src_key, int src_idx, float key, int idx, int& rank) {
  if constexpr (R < 16) {
    const float kf = R == 0 ? src_key : __int_as_float(row_ror<R == 0 ? 1 : R>(__float_as_int(src_key)));
    const int f = R == 0 ? src_idx : row_ror<R == 0 ? 1 : R>(src_idx);
    rank += static_cast<int>(kf > -INFINITY) &
            (static_cast<int>(kf > key) | (static_cast<int>(kf == key) & static_cast<int>(f < idx)));
    rank_from_row<R + 1>(src_key, src_idx, key, idx, rank);
  }
}

// One (token, layer) pair on one wavefront, lane e holding expert e (E <= 64): z its logit,
// key its log-domain key (z + offset). Each expert's rank (the number of valid keys larger, or
// equal with a lower index; -inf and NaN keys are not valid) is its position in the successive
// picks of select_pair, so both give the same selection, margin and gate bits (the normalisers
// are summed in the same order). Writes the pair's outputs at obase; returns, in lanes j < K,
// pick j.
__device__ __forceinline__ int wave_select_pair(const RouteParams& p, float z, float key, bool in, size_t obase) {
  const int lane = threadIdx.x & 63;
  const int E = p.E, K = p.K;
  const bool valid = in && key > -INFINITY;   // false for NaN too
  // rank over the 64 lanes (lanes past E hold -inf): the lane's own row by DPP rotations, the
  // other three rows through one lane exchange each
  int rank = 0;
  rank_from_row<1>(key, lane, key, lane, rank);
#pragma unroll
  for (int ro = 16; ro < 64; ro += 16) rank_from_row<0>(__shfl_xor(key, ro, kWave), lane ^ ro, key, lane, rank);
  const uint64_t vmask = __ballot(valid);
  const int n_valid = __popcll(vmask);
  // picks in order: valid experts by rank, then (fewer than K valid keys) the lowest others
  uint64_t taken = 0;
  int my_sel = 0;
  float my_selz = 0.0f, kth = -INFINITY, nxt = -INFINITY;
  for (int j = 0; j < K; ++j) {
    int e;
    if (j < n_valid) {
      e = __ffsll(static_cast<unsigned long long>(__ballot(valid && rank == j))) - 1;
      kth = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), e));
    } else {
      e = __ffsll(static_cast<unsigned long long>(~taken & (E == 64 ? ~0ull : ((1ull << E) - 1)))) - 1;
      kth = -INFINITY;
    }
    taken |= 1ull << e;
    const float ze = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), e));
    if (lane == j) {
      my_sel = e;
      my_selz = ze;
    }
  }
  if (K < n_valid) {
    const int e = __ffsll(static_cast<unsigned long long>(__ballot(valid && rank == K))) - 1;
    nxt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(key), e));
  }
  float zref, norm = 0.0f;
  if (p.gate_mode == 0) {   // softmax over all E
    // the largest logit: fmaxf drops NaN operands (lanes past E hold NaN), so the reduction
    // order does not change the value (the largest non-NaN logit, NaN if all are NaN)
    zref = in ? z : __builtin_nanf("");
#pragma unroll
    for (int m = kWave / 2; m >= 1; m >>= 1) zref = fmaxf(zref, __shfl_xor(zref, m, kWave));
    float ex = in ? expf(z - zref) : 0.0f;
    if (E > kSelThreadE) {   // the butterfly's tree (kSelThreadE)
#pragma unroll
      for (int m = kWave / 2; m >= 1; m >>= 1) ex += __shfl_xor(ex, m, kWave);
      norm = ex;
    } else {   // expert order, as the per-thread selection for E <= kSelThreadE
      for (int e = 0; e < E; ++e) norm += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ex), e));
    }
  } else {   // renormalised over the picks, in pick order
    zref = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_selz), 0));
    for (int j = 1; j < K; ++j) zref = fmaxf(zref, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_selz), j)));
    for (int j = 0; j < K; ++j)
      norm += expf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_selz), j)) - zref);
  }
  const float inv = 1.0f / norm;
  if (lane < K) {
    p.idx[obase * K + lane] = my_sel;
    p.gate[obase * K + lane] = expf(my_selz - zref) * inv;
  }
  if (lane == 0 && p.margin) p.margin[obase] = (nxt == -INFINITY) ? INFINITY : (kth - nxt);
  return my_sel;
}

// kSelThreadE < E <= 64: one wavefront per pair (wave_select_pair).
__global__ __launch_bounds__(kSelThreads) void route_select_wave_kernel(const RouteParams p) {
  const int lane = threadIdx.x & 63;
  const int E = p.E, T = p.T;
  const uint32_t q = blockIdx.x * (kSelThreads / 64) + (threadIdx.x >> 6);
  if (q >= static_cast<uint32_t>(p.L) * T) return;   // the whole wavefront leaves (L * T < 2^31)
  const int l = static_cast<int>(q / static_cast<uint32_t>(T));
  const bool in = lane < E;
  const float z = in ? p.logits[static_cast<size_t>(q) * E + lane] : 0.0f;
  const float key = in ? z + key_offset(p.mode, p.modep[l * E + lane]) : -INFINITY;
  wave_select_pair(p, z, key, in, q);
}

// The same selection and gates for E > kSelThreadE, one wavefront per (token, layer) pair of the
// tile (tokens t0 .. t0 + TT - 1, layers lg0 .. lg0 + nl - 1; consecutive layers of one token): lane
// e holds the keys of experts e, e + 64, ...; each of the K + 1 picks is a wave reduction
// (largest key, then lowest index), and the softmax normaliser is summed in expert order
// (selection order for the renormalised rule), as in route_finalize, so both give the same bits.
// A thread per pair leaves most of a 16-token tile's threads idle behind K + 1 serial passes
// over E keys: 333 tokens, 64 experts, top-6: 57 us, this way 20 (with many pairs: wave_selects). The selections are also left in
// sel_lds [T, K] for the permutation when given (one layer).
__device__ void route_finalize_wave(const RouteParams& p, const float* logits, int ld, const float* lo, int t0, int TT,
                                    int lg0, int nl, int32_t* sel_lds, int nwaves) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int E = p.E, K = p.K;
  const int pairs = min(TT, p.T - t0) * nl;
  if (E <= 64) {   // one expert per lane: rank-based picks, no cross-lane reductions
    for (int pi = wave; pi < pairs; pi += nwaves) {
      const int t = pi / nl, lw = pi - t * nl;
      const size_t obase = static_cast<size_t>(lg0 + lw) * p.T + t0 + t;
      const bool in = lane < E;
      const float z = in ? logits[t * ld + lw * E + lane] : 0.0f;
      const float key = in ? z + lo[lw * E + lane] : -INFINITY;
      const int my_sel = wave_select_pair(p, z, key, in, obase);
      if (sel_lds && lane < K) sel_lds[t * K + lane] = my_sel;
      if (p.logits && in) p.logits[obase * E + lane] = z;
    }
    return;
  }
  constexpr int Q = 4;   // experts per lane, E <= 256
  for (int pi = wave; pi < pairs; pi += nwaves) {
    const int t = pi / nl, lw = pi - t * nl;
    const size_t obase = static_cast<size_t>(lg0 + lw) * p.T + t0 + t;
    const float* z = logits + t * ld + lw * E;
    float key[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int e = lane + 64 * q;
      key[q] = e < E ? z[e] + lo[lw * E + e] : -INFINITY;
    }
    uint32_t taken = 0;   // bit q: expert lane + 64 q is selected
    int my_sel = 0;
    float my_selz = 0.0f, kth = -INFINITY, nxt = -INFINITY;
    for (int j = 0; j <= K; ++j) {
      float bv = -INFINITY;
      int bi = -1;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int e = lane + 64 * q;
        if (e < E && !((taken >> q) & 1u) && key[q] > bv) {
          bv = key[q];
          bi = e;
        }
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) {
        const float ov = __shfl_xor(bv, m, kWave);
        const int oi = __shfl_xor(bi, m, kWave);
        if (oi >= 0 && (bi < 0 || ov > bv || (ov == bv && oi < bi))) {
          bv = ov;
          bi = oi;
        }
      }
      if (j < K) {
        if (bi < 0) {   // only reachable with non-finite logits: the lowest expert not taken
          int lowest = INT_MAX;
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int e = lane + 64 * q;
            if (e < E && !((taken >> q) & 1u)) lowest = min(lowest, e);
          }
          bi = wave_min_int(lowest);
        }
        if (lane == (bi & 63)) taken |= 1u << (bi >> 6);
        const float zb = z[bi];
        if (lane == j) {
          my_sel = bi;
          my_selz = zb;
        }
        kth = bv;
      } else {
        nxt = bv;
      }
    }
    float zref, norm = 0.0f;
    if (p.gate_mode == 0) {   // g = p_i: softmax over all E experts
      float m = -INFINITY;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (lane + 64 * q < E) m = fmaxf(m, z[lane + 64 * q]);
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
      zref = m;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float ex = lane + 64 * q < E ? expf(z[lane + 64 * q] - zref) : 0.0f;
        const int n_q = min(64, E - 64 * q);
        for (int l = 0; l < n_q; ++l) norm += __shfl(ex, l, kWave);   // expert order
      }
    } else {   // g = p_i / sum_{j in A} p_j, in selection order
      zref = __shfl(my_selz, 0, kWave);
      for (int j = 1; j < K; ++j) zref = fmaxf(zref, __shfl(my_selz, j, kWave));
      for (int j = 0; j < K; ++j) norm += expf(__shfl(my_selz, j, kWave) - zref);
    }
    const float inv = 1.0f / norm;
    if (lane < K) {
      p.idx[obase * K + lane] = my_sel;
      p.gate[obase * K + lane] = expf(my_selz - zref) * inv;
      if (sel_lds) sel_lds[t * K + lane] = my_sel;
    }
    if (lane == 0 && p.margin) p.margin[obase] = (nxt == -INFINITY) ? INFINITY : (kth - nxt);
    if (p.logits)
      for (int e = lane; e < E; e += 64) p.logits[obase * E + e] = z[e];
  }
}

// Whether route_finalize_wave selects a workgroup's `pairs` pairs sooner than route_finalize (a thread per
// pair), in key comparisons of the latter (about 0.13 us each: a thread walks E keys K + 1 times): a
// wavefront's pair costs about 38 of them with up to 64 experts, top-6, 121 with 256, top-8. Workgroups of
// four wavefronts and 32 tokens, 600 tokens, a thread / a wavefront per pair: 24 experts, top-4, 6 layers
// 46 / 207 us; 64 experts, top-6, 4 layers 96 / 167; 256 experts, top-8, one layer 391 / 165. With more
// workgroups than CUs the threads' waits overlap and the wavefronts' work does not: 24 experts, one layer,
// 16000 tokens 39 / 50.
__device__ __forceinline__ bool wave_selects(int E, int K, int pairs, int nthreads) {
  if (gridDim.x * gridDim.y > 256) return false;
  const int nwaves = nthreads / kWave;
  const int wave_cost = 4 * (K + 1) + (E <= kWave ? 10 : E / 3);
  return (pairs + nwaves - 1) / nwaves * wave_cost < (pairs + nthreads - 1) / nthreads * (K + 1) * E;
}

// fmaxf over the 16 lanes of the row, in every lane. fmaxf drops NaN operands, so any order
// of the reduction gives the same value (the largest non-NaN, NaN if all are NaN).
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, __int_as_float(row_ror<8>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(row_ror<4>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(row_ror<2>(__float_as_int(v))));
  v = fmaxf(v, __int_as_float(row_ror<1>(__float_as_int(v))));
  return v;
}

// E <= 16 experts, a 16-token tile of one layer from token t0 (4 per wavefront, every wavefront
// calls this: it holds a barrier): token t0 + t is selected by 16-lane row t % 4 of wavefront t / 4,
// lane e of the row holding expert e. An expert's rank among the valid keys (larger, or equal
// with a lower index; -inf and NaN keys are not valid) is its position in select_pair's
// successive picks; with fewer than K valid keys the lowest other experts follow in index
// order. Each picked lane writes its own outputs. The maxima are order-free; the normalisers
// are summed through LDS (`sc`, [16 tokens][16]) in select_pair's order (picks for the
// renormalised rule, experts for the softmax), so both give the same bits. The picks are also
// left in sel_lds [T, K] for the permutation when given (t0 = 0). obase: the tile's first pair in
// the [L, T] outputs.
__device__ void route_select_rows(const RouteParams& p, const float* logits, int ld, const float* lo, float* sc,
                                  int t0, size_t obase, int32_t* sel_lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int E = p.E, K = p.K, rb = lane & 48, e = lane & 15;
  const int t = 4 * wave + (lane >> 4);
  const int nt = min(16, p.T - t0);
  const bool act = 4 * wave < nt;    // wavefronts without tokens only take part in the barrier
  const bool live = t < nt;
  const bool in = live && e < E;
  const bool soft_all = p.gate_mode == 0;   // g = p_i (softmax over all E), else renormalised over the picks
  float z = 0.0f, key = -INFINITY, ex = 0.0f, zref = 0.0f, kth = -INFINITY, nxt = -INFINITY;
  int pos = 0;
  bool pick = false;
  if (act) {
    z = in ? logits[t * ld + e] : 0.0f;
    key = in ? z + lo[e] : -INFINITY;
    const bool valid = key > -INFINITY;   // false for NaN too
    int rank = 0;
    rank_from_row<1>(key, e, key, e, rank);
    const uint32_t vbits = static_cast<uint32_t>(__ballot(valid) >> rb) & 0xffffu;
    const uint32_t ibits = static_cast<uint32_t>(__ballot(in && !valid) >> rb) & 0xffffu;
    pos = valid ? rank : __popc(vbits) + __popc(ibits & ((1u << e) - 1u));
    pick = in && pos < K;
    kth = row_max(pick && valid && pos == K - 1 ? key : -INFINITY);
    nxt = row_max(valid && rank == K ? key : -INFINITY);
    const bool term = soft_all ? in : pick;
    zref = row_max(term ? z : __builtin_nanf(""));
    ex = expf(z - zref);
    if (term) sc[t * 16 + (soft_all ? e : pos)] = ex;
  }
  lds_sync();
  if (!act) return;
  float norm = 0.0f;
  const int nterms = soft_all ? E : K;
  if (live)
    for (int i = 0; i < nterms; ++i) norm += sc[t * 16 + i];
  const float inv = 1.0f / norm;
  if (pick) {
    p.idx[(obase + t) * K + pos] = e;
    p.gate[(obase + t) * K + pos] = ex * inv;
    if (sel_lds) sel_lds[t * K + pos] = e;
  }
  if (live && e == 0 && p.margin) p.margin[obase + t] = (nxt == -INFINITY) ? INFINITY : (kth - nxt);
  if (in && p.logits) p.logits[(obase + t) * E + e] = z;
}

// FUSE: the grid is one workgroup holding every token of one layer; after the selection it
// also groups the (token, slot) pairs by expert (permute_wave for few entries, else
// permute_block).
// SPLIT (not with FUSE): the tile's logits go to p.logits and route_select_kernel selects.
// Kernel parameters not needed before the epilogue, read at the start so that their loads
// share the first memory round trip: the argument block is fetched from memory at each
// launch, and a parameter first read after the k-loop would cost a round trip of its own.
template <typename V>
__device__ __forceinline__ void load_now(V v) {
  asm volatile("" ::"s"(v));
}

template <int MB, int NB, int WN, int WK, bool FUSE, bool SPLIT = false>
__global__ __launch_bounds__(64 * WN * WK) void route_bf16_kernel(const RouteParams p) {
  constexpr int TT = 16 * MB, NO = 16 * NB * WN, NT = 64 * WN * WK;
  // FUSE with one 16-wide output tile: the E <= 16 key parameters of the single layer are
  // loaded as scalars with the others.
  constexpr bool kScalarModep = FUSE && NO <= 16;
  __shared__ float red[WK * TT * NO];
  __shared__ float lo[NO];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % WN, wk = wave / WN;
  const int t0 = blockIdx.x * TT;
  const int lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0);
  const int nout = nl * p.E;
  const uint16_t* x = static_cast<const uint16_t*>(p.x);
  const uint16_t* w = static_cast<const uint16_t*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d;
  const int ksteps = p.d >> 5;
  const int kg = (lane >> 4) * 8;
  float mp[16];
  if (FUSE) {
    load_now(p.idx); load_now(p.gate); load_now(p.logits);
    load_now(p.K); load_now(p.mode); load_now(p.gate_mode); load_now(p.n_shared); load_now(p.tile_rows);
    load_now(p.pb.offsets); load_now(p.pb.tile_off); load_now(p.pb.active); load_now(p.pb.n_active);
    load_now(p.pb.perm); load_now(p.pb.inv); load_now(p.pb.row_tok);
  }
  if (kScalarModep) {   // lg0 == 0; 16 <= kMaxModeParams
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mp[i] = p.modep[i];
      load_now(mp[i]);
    }
  }

  // Rows past the last token / output are clamped onto valid rows and not loaded (zeros):
  // their results are never written, and MFMA rows and columns do not mix.
  const uint16_t* ap[MB];
  const uint16_t* bp[NB];
  bool arow[MB], brow[NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int t = min(t0 + mb * 16 + (lane & 15), p.T - 1);
    ap[mb] = x + static_cast<size_t>(t) * p.d + kg;
    arow[mb] = t0 + mb * 16 + (lane & 15) < p.T;
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int o = min((wn * NB + nb) * 16 + (lane & 15), nout - 1);
    bp[nb] = w + static_cast<size_t>(o) * p.d + kg;
    brow[nb] = (wn * NB + nb) * 16 + (lane & 15) < nout;
  }
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // k-steps wk, wk+WK, ...; groups of U steps are loaded before any is multiplied. Each wave
  // accumulates its steps in increasing order on every path below.
  constexpr int U = (MB + NB) <= 2 ? 8 : 4;
  int s = wk;
  // Few tokens in the fused launch: their rows are read once into LDS (all lanes of a row
  // tile share them) and the A operands come from there, which halves the load instructions;
  // the first group's weight loads are issued before the rows are stored.
  constexpr bool kStageX = FUSE && NO <= 16 && MB == 1 && NB == 1;
  constexpr int kXsUnits = kStageX ? 2 * NT : 1;   // 16-byte units: 32 KB
  __shared__ u32x4 xs[kXsUnits];
  if (kStageX && p.T * p.d <= kXsUnits * 8) {
    const int units = p.T * p.d / 8;
    const int tr = lane & 15;   // token row of this lane's A operand (loaded when tr < T)
    u32x4 xr[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = threadIdx.x + i * NT;
      xr[i] = c < units ? reinterpret_cast<const u32x4*>(x)[c] : zero4;
    }
    u32x4 bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int st = s + u * WK;
      bv[u] = brow[0] && st < ksteps ? *reinterpret_cast<const u32x4*>(bp[0] + (st << 5)) : zero4;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = threadIdx.x + i * NT;
      if (c < units) xs[c] = xr[i];
    }
    lds_sync();
    const u32x4* xa = xs + (tr * p.d + kg) / 8;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int st = s + u * WK;
      if (st < ksteps) acc[0][0] = mfma_16x16x32(arow[0] ? xa[st * 4] : zero4, bv[u], acc[0][0]);
    }
    for (s += U * WK; s < ksteps; s += WK) {
      const u32x4 b = brow[0] ? *reinterpret_cast<const u32x4*>(bp[0] + (s << 5)) : zero4;
      acc[0][0] = mfma_16x16x32(arow[0] ? xa[s * 4] : zero4, b, acc[0][0]);
    }
  }
  for (; s + (U - 1) * WK < ksteps; s += U * WK) {
    u32x4 av[U][MB], bv[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (s + u * WK) << 5;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) av[u][mb] = arow[mb] ? *reinterpret_cast<const u32x4*>(ap[mb] + k) : zero4;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) bv[u][nb] = brow[nb] ? *reinterpret_cast<const u32x4*>(bp[nb] + k) : zero4;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma_16x16x32(av[u][mb], bv[u][nb], acc[mb][nb]);
  }
  for (; s < ksteps; s += WK) {
    const int k = s << 5;
    u32x4 av[MB], bv[NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) av[mb] = arow[mb] ? *reinterpret_cast<const u32x4*>(ap[mb] + k) : zero4;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) bv[nb] = brow[nb] ? *reinterpret_cast<const u32x4*>(bp[nb] + k) : zero4;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma_16x16x32(av[mb], bv[nb], acc[mb][nb]);
  }

  float* r = red + wk * TT * NO;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        r[(mb * 16 + (lane >> 4) * 4 + i) * NO + (wn * NB + nb) * 16 + (lane & 15)] = acc[mb][nb][i];
  if (kScalarModep) {
    if (wave == 0) {   // lane i: expert i
      float v = mp[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) v = lane == i ? mp[i] : v;
      if (lane < nout) lo[lane] = key_offset(p.mode, v);
    }
  } else {
    for (int i = threadIdx.x; i < nout; i += NT) lo[i] = key_offset(p.mode, p.modep[lg0 * p.E + i]);
  }
  lds_sync();
  if (WK > 1) {
    for (int i = threadIdx.x; i < TT * NO; i += NT) {
      float s = red[i];
#pragma unroll
      for (int q = 1; q < WK; ++q) s += red[q * TT * NO + i];
      red[i] = s;
    }
    lds_sync();
  }
  if (SPLIT) {   // [TT, nl * E] tile -> p.logits [L, T, E], consecutive threads on consecutive floats
    for (int i = threadIdx.x; i < TT * nout; i += NT) {
      const int lw = i / (TT * p.E), rem = i - lw * TT * p.E;
      const int tt = rem / p.E, e = rem - tt * p.E;
      if (t0 + tt < p.T)
        p.logits[(static_cast<size_t>(lg0 + lw) * p.T + t0 + tt) * p.E + e] = red[tt * NO + lw * p.E + e];
    }
  } else if (FUSE) {
    __shared__ PermLds plds;
    __shared__ int32_t sel_lds[kRouteOneBlockT * kMaxK];
    if (NO <= 16) {   // E <= 16
      static_assert(!FUSE || NO > 16 || (TT == 16 && NT >= 4 * 64), "four wavefronts of 4 rows hold the 16 tokens");
      __shared__ float sc[16 * 16];
      route_select_rows(p, red, NO, lo, sc, 0, 0, sel_lds);
    } else
      route_finalize_wave(p, red, NO, lo, 0, TT, 0, 1, sel_lds, NT / 64);
    lds_sync();   // the selections left in sel_lds are read by other threads
    if (p.T * p.K <= kWave && p.E + p.n_shared < kWave) {
      if (wave == 0) permute_wave(sel_lds, p.T, p.K, p.E, p.n_shared, p.tile_rows, p.pb);
    } else {
      permute_block<1>(sel_lds, p.T, p.K, p.E, p.n_shared, p.tile_rows, p.pb, plds, NT);
    }
  } else if (p.E > kSelThreadE && wave_selects(p.E, p.K, TT * nl, NT)) {
    route_finalize_wave(p, red, NO, lo, t0, TT, lg0, nl, nullptr, NT / 64);
  } else if (TT == 16 && NT >= 4 * 64 && nl == 1 && p.E <= kSelThreadE) {   // one layer: four tokens per wavefront
    __shared__ float sc[16 * 16];
    route_select_rows(p, red, NO, lo, sc, t0, static_cast<size_t>(lg0) * p.T + t0, nullptr);
  } else {
    route_finalize(p, red, NO, lo, t0, TT, lg0, nl, NT);
  }
}

// Logits of token t at outputs o .. o + 3 of the layers from lg0 (o % 4 == 0; outputs at or past nout
// are not there) to p.logits [L, T, E].
__device__ __forceinline__ void store_logits4(const RouteParams& p, int lg0, int nout, int o, int t, float v0, float v1,
                                              float v2, float v3) {
  if (o >= nout) return;
  const int E = p.E;
  if ((E & 3) == 0) {   // four outputs of one layer, 16-byte aligned
    const int lw = o / E;
    *reinterpret_cast<f32x4*>(p.logits + (static_cast<size_t>(lg0 + lw) * p.T + t) * E + o - lw * E) =
        f32x4{v0, v1, v2, v3};
    return;
  }
  const float v[4] = {v0, v1, v2, v3};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (o + e < nout) {
      const int l = (o + e) / E;
      p.logits[(static_cast<size_t>(lg0 + l) * p.T + t) * E + o + e - l * E] = v[e];
    }
}

// Many tokens and many router outputs (tens of layers routed from the same tokens): a tile of
// 128 tokens x BN outputs (128 or 256) of whole layers per workgroup of four wavefronts (2 along
// tokens x 2 along outputs), 64-wide k-tiles of both operands staged through LDS, accumulated on
// v_mfma_f32_32x32x16_bf16 with the router rows as the row operand: a lane then holds four
// neighbouring outputs of one token. Every token row is read from HBM once, the router rows are
// shared by all workgroups through L2. One LDS buffer (48 KB) and two workgroups per CU: while one
// stores a k-tile or waits at a barrier, the other multiplies; the tokens of two k-tiles and the
// router rows of one travel in registers meanwhile.
constexpr int kRgBM = 128, kRgMaxBN = 256, kRgBK = 64, kRgThreads = 256;

template <int BN, bool SPLIT>
__global__ __launch_bounds__(kRgThreads, 2) void route_gemm_kernel(const RouteParams p) {
  constexpr int BM = kRgBM, BK = kRgBK, NT = kRgThreads;
  constexpr int TM = 2, TN = BN / 64;          // 32-token and 32-output fragments per wavefront
  constexpr int UA = BM * 8 / NT, UB = BN * 8 / NT;   // 16-byte units per thread and k-tile
  constexpr int HALF = BM / 2;                 // token rows per selection phase (one wave row)
  constexpr int LD = BN + 1;                   // logits row stride: odd, so token rows fall on distinct banks
  constexpr int STAGING = (BM + BN) * BK * 2, LOGITS = SPLIT ? 0 : HALF * LD * 4;
  __shared__ __attribute__((aligned(16))) unsigned char smem[STAGING > LOGITS ? STAGING : LOGITS];
  __shared__ float lo[SPLIT ? 1 : BN];
  u32x4* lds_a = reinterpret_cast<u32x4*>(smem);    // [BM * 8]
  u32x4* lds_b = lds_a + BM * 8;                    // [BN * 8]
  float* logits = reinterpret_cast<float*>(smem);   // [HALF][LD], after the k-loop

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int t0 = blockIdx.x * BM;
  const int lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0);
  const int nout = nl * p.E;
  const uint16_t* x = static_cast<const uint16_t*>(p.x);
  const uint16_t* w = static_cast<const uint16_t*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d;

  // Thread tid loads rows (tid >> 3) + 32 i of each operand; rows past the last token or
  // output are clamped onto valid rows and their results never written. Buffer loads: 32-bit
  // offsets within the tile's rows, the k-tile in a scalar.
  const int r0 = tid >> 3, rows = min(BM, p.T - t0);
  const int dst = r0 * 8 + ((tid & 7) ^ lds_swizzle(r0));   // unit i: + NT * i
  const __amdgpu_buffer_rsrc_t ar = make_rsrc(x + static_cast<size_t>(t0) * p.d, 2u * rows * p.d);
  const __amdgpu_buffer_rsrc_t br = make_rsrc(w, 2u * nout * p.d);
  uint32_t asrc[UA], bsrc[UB];
#pragma unroll
  for (int i = 0; i < UA; ++i) asrc[i] = 2u * (min(r0 + 32 * i, rows - 1) * p.d + (tid & 7) * 8);
#pragma unroll
  for (int i = 0; i < UB; ++i) bsrc[i] = 2u * (min(r0 + 32 * i, nout - 1) * p.d + (tid & 7) * 8);
  const int sw = lds_swizzle(lane & 31);   // fragment rows are a multiple of 32 plus (lane & 31)

  f32x16 acc[TN][TM];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.0f;

  const int nk = p.d / BK;
  auto k_bytes = [&](int kt) { return min(kt, nk - 1) * (2 * BK); };   // past the end: the last k-tile again, not used
  u32x4 ra[2][UA], rb[UB];
  constexpr int kNt = 2;   // the load's non-temporal bit: token rows are read once
  auto load_a = [&](int kt, u32x4 (&r)[UA]) {
    const int k = k_bytes(kt);
#pragma unroll
    for (int i = 0; i < UA; ++i) r[i] = __builtin_amdgcn_raw_buffer_load_b128(ar, asrc[i], k, kNt);
  };
  auto load_b = [&](int kt) {
    const int k = k_bytes(kt);
#pragma unroll
    for (int i = 0; i < UB; ++i) rb[i] = __builtin_amdgcn_raw_buffer_load_b128(br, bsrc[i], k, 0);
  };
  // k-tile kt: registers to LDS, then the router rows of kt + 1 and the tokens of kt + 2 on
  // their way (in this order: waiting for router rows, which come from L2, leaves the youngest
  // tokens, which come from HBM, in flight), then the products.
  auto tile = [&](int kt, auto set_c) {
    constexpr int set = decltype(set_c)::value;
#pragma unroll
    for (int i = 0; i < UA; ++i) lds_a[dst + NT * i] = ra[set][i];
#pragma unroll
    for (int i = 0; i < UB; ++i) lds_b[dst + NT * i] = rb[i];
    __builtin_amdgcn_sched_barrier(0);
    load_b(kt + 1);
    __builtin_amdgcn_sched_barrier(0);
    load_a(kt + 2, ra[set]);
    __builtin_amdgcn_sched_barrier(0);
    lds_sync();
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int ch = (kk * 2 + (lane >> 5)) ^ sw;
      u32x4 af[TM], bf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = lds_a[(wm * HALF + i * 32 + (lane & 31)) * 8 + ch];
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[j] = lds_b[(wn * (BN / 2) + j * 32 + (lane & 31)) * 8 + ch];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = mfma_32x32x16(bf[j], af[i], acc[j][i]);
    }
    lds_sync();   // the buffer is read
  };
  load_a(0, ra[0]);
  __builtin_amdgcn_sched_barrier(0);
  load_b(0);
  __builtin_amdgcn_sched_barrier(0);
  load_a(1, ra[1]);
  __builtin_amdgcn_sched_barrier(0);
  int kt = 0;
  for (; kt + 1 < nk; kt += 2) {
    tile(kt, std::integral_constant<int, 0>{});
    tile(kt + 1, std::integral_constant<int, 1>{});
  }
  if (kt < nk) tile(kt, std::integral_constant<int, 0>{});

  // acc[j][i][4 q + e] is output wn*BN/2 + j*32 + 8 q + 4 (lane >> 5) + e of token
  // t0 + wm*64 + i*32 + (lane & 31).
  if (SPLIT) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int t = t0 + wm * HALF + i * 32 + (lane & 31);
      if (t >= p.T) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          store_logits4(p, lg0, nout, wn * (BN / 2) + j * 32 + 8 * q + 4 * (lane >> 5), t, acc[j][i][4 * q],
                        acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]);
    }
    return;
  }
  // Phase h: the waves of token half h write their logits to LDS (the last barrier of the loop
  // ended every read of the staging buffer), then every thread selects for those tokens.
  for (int i = tid; i < nout; i += NT) lo[i] = key_offset(p.mode, p.modep[lg0 * p.E + i]);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (wm == h) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            logits[(i * 32 + (lane & 31)) * LD + wn * (BN / 2) + j * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] =
                acc[j][i][r];
    }
    lds_sync();
    route_finalize<true>(p, logits, LD, lo, t0 + h * HALF, HALF, lg0, nl, NT);
    lds_sync();   // the next phase overwrites the logits
  }
}

// Selection with the logits, more than 128 outputs and more than kRouteWideT tokens: 256 tokens x 256
// outputs per workgroup of eight wavefronts, double-buffered k-tiles, one workgroup per CU; the selection
// as in route_gemm_kernel, on 128 tokens at a time. (32 layers of 8 experts, d 4096, 128-token tiles /
// this: 20000 tokens 137 / 143 us, 33000 181 / 157, 64000 215 / 192.)
constexpr int kRwBM = 256, kRwThreads = 512;

__global__ __launch_bounds__(kRwThreads) void route_wide_kernel(const RouteParams p) {
  constexpr int BM = kRwBM, BN = kRgMaxBN, BK = kRgBK, NT = kRwThreads;
  constexpr int WN = 4;                        // waves: 2 along tokens x 4 along outputs
  constexpr int TM = 4, TN = 2;                // 32x32 fragments per wave: 128 tokens x 64 outputs
  constexpr int HALF = BM / 2;                 // token rows per selection phase (one wave row)
  constexpr int UA = BM * 8 / NT, UB = BN * 8 / NT;   // 16-byte units per thread and stage
  constexpr int SA = BM * 8, SB = BN * 8;             // 16-byte slots per stage
  constexpr int STAGING = 2 * (SA + SB) * 16;
  constexpr int LD = BN + 1;                   // logits row stride: odd, so token rows fall on distinct banks
  constexpr int LOGITS = HALF * LD * 4;
  __shared__ __attribute__((aligned(16))) unsigned char smem[STAGING > LOGITS ? STAGING : LOGITS];
  __shared__ float lo[BN];
  u32x4* lds_a = reinterpret_cast<u32x4*>(smem);   // [2][SA]
  u32x4* lds_b = lds_a + 2 * SA;                    // [2][SB]
  float* logits = reinterpret_cast<float*>(smem);   // [HALF][LD], after the k-loop

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int t0 = blockIdx.x * BM;
  const int lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0);
  const int nout = nl * p.E;
  const uint16_t* x = static_cast<const uint16_t*>(p.x);
  const uint16_t* w = static_cast<const uint16_t*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d;

  // Thread tid loads rows (tid >> 3) + 64 i of each operand; rows past the last token or
  // output are clamped onto valid rows and their results never written.
  const int r0 = tid >> 3;
  const int chunk = ((tid & 7) ^ lds_swizzle(r0)) * 8;
  const uint16_t* asrc[UA];
  const uint16_t* bsrc[UB];
#pragma unroll
  for (int i = 0; i < UA; ++i) asrc[i] = x + static_cast<size_t>(min(t0 + r0 + 64 * i, p.T - 1)) * p.d + chunk;
#pragma unroll
  for (int i = 0; i < UB; ++i) bsrc[i] = w + static_cast<size_t>(min(r0 + 64 * i, nout - 1)) * p.d + chunk;
  int aoff[TM], boff[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) aoff[i] = (wm * 128 + i * 32 + (lane & 31)) * 8;
#pragma unroll
  for (int j = 0; j < TN; ++j) boff[j] = (wn * 64 + j * 32 + (lane & 31)) * 8;
  const int sw = lds_swizzle(lane);   // fragment rows are a multiple of 32 plus (lane & 31)

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  u32x4 ra[UA], rb[UB];
  auto gload = [&](int kt) {
#pragma unroll
    for (int i = 0; i < UA; ++i) ra[i] = *reinterpret_cast<const u32x4*>(asrc[i] + kt * BK);
#pragma unroll
    for (int i = 0; i < UB; ++i) rb[i] = *reinterpret_cast<const u32x4*>(bsrc[i] + kt * BK);
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < UA; ++i) lds_a[buf * SA + tid + NT * i] = ra[i];
#pragma unroll
    for (int i = 0; i < UB; ++i) lds_b[buf * SB + tid + NT * i] = rb[i];
  };
  u32x4 af[2][TM], bf[2][TN];
  auto read_frags = [&](int buf, int kk, int slot) {
    const int ch = (kk * 2 + (lane >> 5)) ^ sw;
#pragma unroll
    for (int i = 0; i < TM; ++i) af[slot][i] = lds_a[buf * SA + aoff[i] + ch];
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[slot][j] = lds_b[buf * SB + boff[j] + ch];
  };

  // k-tile kt sits in LDS buffer kt & 1 and tile kt + 1 in registers; after the first k16 step
  // of tile kt the registers go to the other buffer and are refilled with tile kt + 2.
  // Branch-free body, interleaved by LLVM's MFMA/DS strategy as in the expert GEMM: past the end
  // the last tile is loaded again into the idle buffer, which nothing reads.
  const int nk = p.d / BK;
  gload(0);
  lstore(0);
  gload(min(1, nk - 1));
  __syncthreads();
  read_frags(0, 0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    __builtin_amdgcn_iglp_opt(0);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int cur = kk & 1;
      if (kk + 1 < BK / 16) read_frags(buf, kk + 1, cur ^ 1);
      if (kk == 0) {
        lstore(buf ^ 1);
        gload(min(kt + 2, nk - 1));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma_32x32x16(af[cur][i], bf[cur][j], acc[i][j]);
    }
    __syncthreads();
    read_frags(buf ^ 1, 0, 0);
  }

  // The last barrier of the loop ends every read of the staging buffers. Phase h: the waves
  // of token half h write their logits, then every thread selects for those tokens.
  // acc[i][j][4 jj + ii] is token row wm*128 + i*32 + 8 jj + 4 (lane >> 5) + ii, output
  // column wn*64 + j*32 + (lane & 31).
  for (int i = tid; i < nout; i += NT) lo[i] = key_offset(p.mode, p.modep[lg0 * p.E + i]);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (wm == h) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            logits[row * LD + wn * 64 + j * 32 + (lane & 31)] = acc[i][j][r];
          }
    }
    lds_sync();
    route_finalize<true>(p, logits, LD, lo, t0 + h * HALF, HALF, lg0, nl, NT);
    lds_sync();   // the next phase overwrites the logits
  }
}

// Split routing with more than 128 outputs: 256 tokens x 256 outputs per workgroup on the expert
// GEMM's ping-pong tile (gemm_tile.hpp), the router rows as its A operand and the token rows, two
// k-tiles ahead and non-temporal, as its B operand; the logits go straight to p.logits. Bound by the
// token stream: 131072 tokens, 32 layers, 1.07 GB: 306 us before (register-staged 256 x 256 tiles),
// 255 to 290 us now. Starting the k-loop of neighbouring workgroups at different k-tiles, so that
// they do not read the same columns at once, took it to 262 us, but sums each logit from another
// k on: near-tied experts change places, so it is not done.
__global__ __launch_bounds__(kTileThreads) void route_tile_kernel(const RouteParams p) {
  __shared__ TileLds lds;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave >> 2, wn = wave & 3;
  const int t0 = blockIdx.x * kTileN, lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0), nout = nl * p.E, rows = min(kTileN, p.T - t0);
  const int nk = p.d / kTileK;
  TileOps ops;
  ops.a = reinterpret_cast<const char*>(static_cast<const uint16_t*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d);
  ops.b = reinterpret_cast<const char*>(static_cast<const uint16_t*>(p.x) + static_cast<size_t>(t0) * p.d);
  ops.b_step = kTileK * 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {   // rows past the end are clamped, their results never stored
    const int r = tile_dma_row(i), c = tile_dma_chunk(i) * 8;
    ops.aoff[i] = 2u * static_cast<uint32_t>(min(r, nout - 1) * p.d + c);
    ops.boff[i] = 2u * static_cast<uint32_t>(min(r, rows - 1) * p.d + c);
  }
  int bfrag[kTileTN];
#pragma unroll
  for (int j = 0; j < kTileTN; ++j) bfrag[j] = wn * 64 + j * 32 + (lane & 31);
  f32x16 acc[kTileTM][kTileTN];
#pragma unroll
  for (int i = 0; i < kTileTM; ++i)
#pragma unroll
    for (int j = 0; j < kTileTN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  gemm_tile_mainloop<false, false, false, true>(ops, nk, bfrag, acc, lds);
  // acc[i][j][4 q + e]: output wm*128 + i*32 + 8 q + 4 (lane >> 5) + e of token t0 + bfrag[j]
#pragma unroll
  for (int i = 0; i < kTileTM; ++i)
#pragma unroll
    for (int j = 0; j < kTileTN; ++j) {
      const int t = t0 + bfrag[j];
      if (t >= p.T) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        store_logits4(p, lg0, nout, wm * 128 + i * 32 + 8 * q + 4 * (lane >> 5), t, acc[i][j][4 * q], acc[i][j][4 * q + 1],
                      acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    }
}

// Split routing of fewer tokens than fill the chip with 256 x 256 tiles: 64 tokens x BN outputs (64
// or 128) per workgroup of four wavefronts (2 along tokens x 2 along outputs), 64-wide k-tiles
// staged through LDS, four of them in flight in registers: with about one workgroup per CU the time
// is the chain of memory latencies along the reduction. 32 layers of 8 experts, d 4096, whole call:
// 600 tokens 100 -> 28 us, 1500 88 -> 27, 5000 85 -> 42; 16 layers, 2000 tokens 85 -> 26.
constexpr int kRmBM = 64, kRmThreads = 256, kRmDepth = 4;

template <int BN>
__global__ __launch_bounds__(kRmThreads, 2) void route_mid_kernel(const RouteParams p) {
  constexpr int BK = 64, NT = kRmThreads, ROWS = kRmBM + BN;
  constexpr int PER = ROWS * 8 / NT, PB = BN * 8 / NT;   // 16-byte pieces per thread, the first PB of the router
  constexpr int TN = BN / 64;                            // 32-output fragments per wavefront
  __shared__ u32x4 lds[2][ROWS * 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
  const int t0 = blockIdx.x * kRmBM, lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0), nout = nl * p.E, rows = min(kRmBM, p.T - t0);
  const int nk = p.d / BK, r0 = tid >> 3;
  const __amdgpu_buffer_rsrc_t ar =
      make_rsrc(static_cast<const uint16_t*>(p.x) + static_cast<size_t>(t0) * p.d, 2u * rows * p.d);
  const __amdgpu_buffer_rsrc_t br =
      make_rsrc(static_cast<const uint16_t*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d, 2u * nout * p.d);
  uint32_t off[PER];   // rows past the end are clamped, their results never stored
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int r = i < PB ? min(r0 + 32 * i, nout - 1) : min(r0 + 32 * (i - PB), rows - 1);
    off[i] = 2u * static_cast<uint32_t>(r * p.d + (tid & 7) * 8);
  }
  const int dst = r0 * 8 + ((tid & 7) ^ lds_swizzle(r0));   // piece i: + NT * i
  u32x4 reg[kRmDepth][PER];
  auto load = [&](int c, u32x4 (&r)[PER]) {   // past the end: the last k-tile again, not used
    const int k = min(c, nk - 1) * (2 * BK);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      r[i] = i < PB ? __builtin_amdgcn_raw_buffer_load_b128(br, off[i], k, 0)
                    : __builtin_amdgcn_raw_buffer_load_b128(ar, off[i], k, 0);
  };
  auto store = [&](int buf, const u32x4 (&r)[PER]) {
#pragma unroll
    for (int i = 0; i < PER; ++i) lds[buf][dst + NT * i] = r[i];
  };
  f32x16 acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
  const int l32 = lane & 31, sw = lds_swizzle(l32);
  int c = 0;
  auto step = [&](auto ph) {   // k-tile c in LDS buffer c & 1, its registers (set c & 3) take k-tile c + 4
    constexpr int PH = decltype(ph)::value;
    load(c + kRmDepth, reg[PH]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int ch = (kk * 2 + (lane >> 5)) ^ sw;
      const u32x4 t = lds[PH & 1][(BN + wm * 32 + l32) * 8 + ch];
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[j] = mfma_32x32x16(lds[PH & 1][(wn * (BN / 2) + j * 32 + l32) * 8 + ch], t, acc[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
    store((PH & 1) ^ 1, reg[(PH + 1) & 3]);
    lds_sync();
    return ++c < nk;
  };
#pragma unroll
  for (int i = 0; i < kRmDepth; ++i) {
    load(i, reg[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
  store(0, reg[0]);
  lds_sync();
  while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{}) &&
         step(std::integral_constant<int, 2>{}) && step(std::integral_constant<int, 3>{})) {
  }
  // acc[j][4 q + e]: output wn*BN/2 + j*32 + 8 q + 4 (lane >> 5) + e of token t0 + wm*32 + l32
  const int t = t0 + wm * 32 + l32;
  if (t >= p.T) return;
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      store_logits4(p, lg0, nout, wn * (BN / 2) + j * 32 + 8 * q + 4 * (lane >> 5), t, acc[j][4 * q], acc[j][4 * q + 1],
                    acc[j][4 * q + 2], acc[j][4 * q + 3]);
}

// fp32 router: 16 tokens x up to 256 outputs (whole layers) per workgroup on
// v_mfma_f32_16x16x4_f32, operands straight from memory, four k per lane and 16-byte load. With
// up to four 16-wide output tiles the wavefronts split the reduction and their partial sums are
// added in LDS in wavefront order; with more they split the tiles. (One thread per (token,
// output) that walked its two rows alone took 30 us for 64 tokens, d 256, 8 experts.)
constexpr int kF32TT = 16, kF32Waves = 4, kF32Outs = 256;

// Four values of a row at k .. k + 3, zeros past d; VEC: d % 4 == 0 (16-byte loads).
template <bool VEC>
__device__ __forceinline__ f32x4 load_row4(const float* row, int k, int d) {
  f32x4 r;
  if (VEC) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(row + min(k, d - 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = k < d ? v[e] : 0.0f;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = row[min(k + e, d - 1)];
      r[e] = k + e < d ? v : 0.0f;
    }
  }
  return r;
}

template <bool VEC>
__global__ __launch_bounds__(64 * kF32Waves) void route_f32_kernel(const RouteParams p) {
  constexpr int NT = 64 * kF32Waves;
  __shared__ float logits[kF32TT * kF32Outs];   // split reduction: [wavefront][16][64]
  __shared__ float lo[kF32Outs];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, lg = lane >> 4;
  const int t0 = blockIdx.x * kF32TT;
  const int lg0 = blockIdx.y * p.lpw;
  const int nl = min(p.lpw, p.L - lg0);
  const int nout = nl * p.E, ntiles = (nout + 15) / 16;
  const float* w = static_cast<const float*>(p.w) + static_cast<size_t>(lg0) * p.E * p.d;
  const float* xr = static_cast<const float*>(p.x) + static_cast<size_t>(min(t0 + l16, p.T - 1)) * p.d;
  for (int i = threadIdx.x; i < nout; i += NT) lo[i] = key_offset(p.mode, p.modep[lg0 * p.E + i]);
  const int ksteps = (p.d + 15) / 16;
  // acc += tokens x outputs 16 ot .. + 15 over k-steps [s0, s1): rows past the ends are clamped
  auto tile = [&](int ot, int s0, int s1) {
    const float* wr = w + static_cast<size_t>(min(16 * ot + l16, nout - 1)) * p.d;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int U = 4;   // k-steps loaded together
    for (int s = s0; s < s1; s += U) {
      f32x4 a[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = s + u < s1 ? 16 * (s + u) + 4 * lg : p.d;   // zeros past the range
        a[u] = load_row4<VEC>(xr, k, p.d);
        b[u] = load_row4<VEC>(wr, k, p.d);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], acc, 0, 0, 0);
    }
    return acc;   // acc[i]: token 4 lg + i, output 16 ot + l16
  };
  int ld = kF32Outs;
  if (ntiles <= 4) {
    ld = 64;
    const int per = (ksteps + kF32Waves - 1) / kF32Waves;
    const int s0 = min(wave * per, ksteps), s1 = min(s0 + per, ksteps);
    for (int ot = 0; ot < ntiles; ++ot) {
      const f32x4 acc = tile(ot, s0, s1);
#pragma unroll
      for (int i = 0; i < 4; ++i) logits[(wave * kF32TT + 4 * lg + i) * 64 + 16 * ot + l16] = acc[i];
    }
    lds_sync();
    for (int i = threadIdx.x; i < kF32TT * 64; i += NT) {
      if ((i & 63) >= nout) continue;
      float s = logits[i];
#pragma unroll
      for (int q = 1; q < kF32Waves; ++q) s += logits[q * kF32TT * 64 + i];
      logits[i] = s;
    }
  } else {
    for (int ot = wave; ot < ntiles; ot += kF32Waves) {
      const f32x4 acc = tile(ot, 0, ksteps);
#pragma unroll
      for (int i = 0; i < 4; ++i) logits[(4 * lg + i) * kF32Outs + 16 * ot + l16] = acc[i];
    }
  }
  lds_sync();
  if (p.E > kSelThreadE && wave_selects(p.E, p.K, kF32TT * nl, NT))
    route_finalize_wave(p, logits, ld, lo, t0, kF32TT, lg0, nl, nullptr, kF32Waves);
  else route_finalize(p, logits, ld, lo, t0, kF32TT, lg0, nl, NT);
}

template <int MB, int NB, int WN, int WK, bool FUSE = false, bool SPLIT = false>
hipError_t launch_bf16(RouteParams& p, hipStream_t stream) {
  constexpr int TT = 16 * MB, NO = 16 * NB * WN;
  p.lpw = NO / p.E < 1 ? 1 : NO / p.E;
  if (p.lpw > p.L) p.lpw = p.L;
  dim3 grid((p.T + TT - 1) / TT, (p.L + p.lpw - 1) / p.lpw);
  if (FUSE && (grid.x != 1 || grid.y != 1)) return hipErrorInvalidValue;  // needs one workgroup
  hipLaunchKernelGGL((route_bf16_kernel<MB, NB, WN, WK, FUSE, SPLIT>), grid, dim3(64 * WN * WK), 0, stream, p);
  return hipGetLastError();
}

void fill_params(RouteParams& p, const void* x, const void* w_router, int T, int d, int E, int K, int L, int l0,
                 int mode, int gate_mode, const uint8_t* mask, const float* prior, int32_t* idx, float* gate,
                 float* margin, float* logits, size_t esz) {
  p.x = x;
  p.w = static_cast<const char*>(w_router) + static_cast<size_t>(l0) * E * d * esz;
  p.idx = idx + static_cast<size_t>(l0) * T * K;
  p.gate = gate + static_cast<size_t>(l0) * T * K;
  p.margin = margin ? margin + static_cast<size_t>(l0) * T : nullptr;
  p.logits = logits ? logits + static_cast<size_t>(l0) * T * E : nullptr;
  p.T = T; p.d = d; p.E = E; p.K = K;
  p.L = L;
  p.mode = mode; p.gate_mode = gate_mode;
  p.pb = PermBuffers{};
  p.n_shared = 0;
  p.tile_rows = 1;
  for (int i = 0; i < p.L * E; ++i) {
    const size_t gi = static_cast<size_t>(l0) * E + i;
    p.modep[i] = mode == 1 ? (mask[gi] ? 1.0f : 0.0f) : mode == 2 ? prior[gi] : 1.0f;
  }
}

}  // namespace

hipError_t launch_route(bool bf16, const void* x, const void* w_router, int T, int d, int E, int K,
                        int L, int mode, int gate_mode, const uint8_t* mask, const float* prior,
                        int32_t* idx, float* gate, float* margin, float* logits, float* split_ws,
                        hipStream_t stream) {
  if (T == 0 || L == 0) return hipSuccess;
  // Split routing needs an [L, T, E] fp32 buffer: the caller's logits output, else split_ws.
  float* zbuf = logits ? logits : split_ws;
  const bool split = route_splits(bf16, T, E) && zbuf;
  // Layers are processed in launches whose (layer, expert) parameters fit in the kernel
  // arguments; every launch covers whole layers.
  const int max_layers = kMaxModeParams / E;
  const size_t esz = bf16 ? 2 : 4;
  for (int l0 = 0; l0 < L; l0 += max_layers) {
    RouteParams p;
    fill_params(p, x, w_router, T, d, E, K, L - l0 < max_layers ? L - l0 : max_layers, l0, mode, gate_mode, mask,
                prior, idx, gate, margin, split ? zbuf : logits, esz);
    hipError_t err;
    if (!bf16) {
      p.lpw = kF32Outs / E < 1 ? 1 : kF32Outs / E;
      if (p.lpw > p.L) p.lpw = p.L;
      dim3 grid((T + kF32TT - 1) / kF32TT, (p.L + p.lpw - 1) / p.lpw);
      if (d % 4 == 0) hipLaunchKernelGGL(route_f32_kernel<true>, grid, dim3(64 * kF32Waves), 0, stream, p);
      else hipLaunchKernelGGL(route_f32_kernel<false>, grid, dim3(64 * kF32Waves), 0, stream, p);
      err = hipGetLastError();
    } else if (split && route_tiles(T, d, E, p.L)) {
      // The tile by how many workgroups it gives (the 256 CUs need about one each; beyond two
      // each the larger tile's fewer loads win). 32 layers of 8 experts, d 4096, whole call with
      // 64-output, 128-output and 256 x 256 tiles: 2000 tokens 29 / 37 / 79 us, 5000 49 / 42 / 81,
      // 12000 82 / 61 / 86, 30000 188 / 145 / 105, 131072 973 / 613 / 311. 16 layers: 30000 tokens,
      // 128-output tiles of 64 / 128 tokens 82 / 77, 131072 tokens 310 / 293 (262 non-temporal).
      const int outs = p.L * E;
      const int mt = (T + kRmBM - 1) / kRmBM;
      auto layers = [&](int bn) { return std::max(std::min(bn / E, p.L), 1); };   // whole layers per workgroup
      auto cover = [&](int bn) { return (p.L + layers(bn) - 1) / layers(bn); };     // column blocks
      if (mt * cover(64) <= 256) {
        p.lpw = layers(64);
        hipLaunchKernelGGL(route_mid_kernel<64>, dim3(mt, cover(64)), dim3(kRmThreads), 0, stream, p);
      } else if (mt * cover(128) <= 512) {
        p.lpw = layers(128);
        hipLaunchKernelGGL(route_mid_kernel<128>, dim3(mt, cover(128)), dim3(kRmThreads), 0, stream, p);
      } else if (outs <= 128) {
        p.lpw = layers(128);
        hipLaunchKernelGGL((route_gemm_kernel<128, true>), dim3((T + kRgBM - 1) / kRgBM, cover(128)), dim3(kRgThreads),
                           0, stream, p);
      } else {
        p.lpw = layers(256);
        hipLaunchKernelGGL(route_tile_kernel, dim3((T + kTileN - 1) / kTileN, cover(256)), dim3(kTileThreads), 0,
                           stream, p);
      }
      err = hipGetLastError();
    } else if (!split && route_tiles(T, d, E, p.L) && !route_small_tiles(T, d, E, (p.L + 256 / E - 1) / (256 / E))) {
      const bool narrow = p.L * E <= 128;   // one 128-output tile holds every layer
      const bool wide = !narrow && T > kRouteWideT;
      p.lpw = std::min((narrow ? 128 : kRgMaxBN) / E, p.L);
      const int bm = wide ? kRwBM : kRgBM;
      const dim3 grid((T + bm - 1) / bm, (p.L + p.lpw - 1) / p.lpw);
      if (narrow) hipLaunchKernelGGL((route_gemm_kernel<128, false>), grid, dim3(kRgThreads), 0, stream, p);
      else if (wide) hipLaunchKernelGGL(route_wide_kernel, grid, dim3(kRwThreads), 0, stream, p);
      else hipLaunchKernelGGL((route_gemm_kernel<kRgMaxBN, false>), grid, dim3(kRgThreads), 0, stream, p);
      err = hipGetLastError();
    } else {
      const int need = p.L * E < 256 ? p.L * E : 256;
      const bool small = T <= 128;
      if (split) {   // T >= kRouteSplitMinT
        if (need <= 16) err = launch_bf16<1, 1, 1, 8, false, true>(p, stream);
        else if (need <= 64) err = launch_bf16<1, 4, 1, 8, false, true>(p, stream);
        else err = launch_bf16<2, 4, 4, 1, false, true>(p, stream);
      } else if (need <= 16) {   // the split launch's logit tiles for many tokens: the same bits
        err = small ? launch_bf16<1, 1, 1, 16>(p, stream) : launch_bf16<1, 1, 1, 8>(p, stream);
      } else if (need <= 64) {
        err = launch_bf16<1, 4, 1, 8>(p, stream);
      } else {
        err = small ? launch_bf16<1, 4, 4, 2>(p, stream) : launch_bf16<2, 4, 4, 1>(p, stream);
      }
    }
    if (err != hipSuccess) return err;
    if (split) {
      const size_t pairs = static_cast<size_t>(p.L) * T;
      if (E <= kSelThreadE) {
        dim3 grid(static_cast<unsigned>((pairs + kSelThreads - 1) / kSelThreads));
        if (E == 8 && K == 2) hipLaunchKernelGGL((route_select_kernel<8, 2>), grid, dim3(kSelThreads), 0, stream, p);
        else if (E == 8) hipLaunchKernelGGL(route_select_kernel<8>, grid, dim3(kSelThreads), 0, stream, p);
        else if (E == 16) hipLaunchKernelGGL(route_select_kernel<16>, grid, dim3(kSelThreads), 0, stream, p);
        else hipLaunchKernelGGL(route_select_kernel<0>, grid, dim3(kSelThreads), 0, stream, p);
      } else {
        constexpr int per_block = kSelThreads / 64;
        dim3 grid(static_cast<unsigned>((pairs + per_block - 1) / per_block));
        hipLaunchKernelGGL(route_select_wave_kernel, grid, dim3(kSelThreads), 0, stream, p);
      }
      err = hipGetLastError();
      if (err != hipSuccess) return err;
    }
  }
  return hipSuccess;
}

hipError_t launch_route_permute(const void* x, const void* w_router, int T, int d, int E, int K, int mode,
                                int gate_mode, const uint8_t* mask, const float* prior, int32_t* idx,
                                float* gate, float* logits, int n_shared, int tile_rows, const PermBuffers& pb,
                                hipStream_t stream) {
  if (T == 0) return hipSuccess;
  if (T > kRouteOneBlockT) return hipErrorInvalidValue;
  RouteParams p;
  fill_params(p, x, w_router, T, d, E, K, 1, 0, mode, gate_mode, mask, prior, idx, gate, nullptr, logits, 2);
  p.pb = pb;
  p.n_shared = n_shared;
  p.tile_rows = tile_rows;
  if (E <= 16) return launch_bf16<1, 1, 1, 16, true>(p, stream);
  if (E <= 64) return launch_bf16<1, 4, 1, 8, true>(p, stream);
  return launch_bf16<1, 4, 4, 2, true>(p, stream);
}

}  // namespace maskmoe
