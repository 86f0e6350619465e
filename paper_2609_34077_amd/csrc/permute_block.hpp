// Token permutation by expert, run by one workgroup of `nthreads` threads (the launch's block
// size, a multiple of 64, <= 1024).
//
// The combine of Eq. 1 (Section 3.1) sums, for every token, the outputs of the experts it
// selected. To run each expert as one dense GEMM over the tokens that chose it, the T*K
// (token, slot) entries j = t*K + k are grouped by expert, keeping entry order inside a
// group (a stable counting sort), and n_shared groups holding every token are appended
// for the shared experts (Section 3.1). Outputs, with G = E + n_shared groups:
//   offsets[g]   first row of group g (offsets[G] = T*(K + n_shared))
//   tile_off[g]  first row-tile of group g in units of `tile_rows` (tile_off[G] = total)
//   active[i]    the i-th non-empty group, n_active[0] their count
//   perm[pos]    entry j placed at row pos (routed rows only), inv[j] = pos
//   row_tok[pos] token of row pos (routed and shared rows)
// Every wavefront owns a contiguous run of entries: it counts them per expert in LDS, the counts
// become each wavefront's first rank per expert (a prefix over wavefronts) and one wavefront's
// prefix sums the group offsets; then each wavefront places its entries in order, an entry's
// rank among equal experts of its 64 coming from ballots on the expert id bits. Four barriers,
// however many entries. Integer only, deterministic. `idx` may have been written by this workgroup
// just before the call, after a barrier that orders it (lds_sync for LDS, __syncthreads for
// global memory). The threads exchange data through LDS only; the outputs are written, never
// read back.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace maskmoe {

constexpr int kPermMaxWaves = 16;
constexpr int kPermMaxGroups = 256 + 8;

struct PermLds {
  int total[kPermMaxGroups];   // entries of each expert, then its first row
  int wcnt[kPermMaxWaves][kPermMaxGroups];
};

// Inclusive prefix sum over the 64 lanes with DPP lane shifts: within each 16-lane row by
// shifts of 1, 2, 4, 8 (lanes shifted in from outside the row add 0), then the last lane of
// rows 0 and 2 is added to rows 1 and 3 (row_bcast:15) and lane 31 to rows 2 and 3
// (row_bcast:31).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2, 3
  return v;
}

// Group offsets, row-tile offsets and the active list from the experts' entry counts total[0, E)
// (LDS), by the first wavefront of the workgroup; lane l takes PG groups in order. total[g]
// becomes the first row of expert g.
__device__ __forceinline__ void permute_scan_groups(int* total, int T, int E, int n_shared, int tile_rows,
                                                    const PermBuffers& pb) {
  const int lane = threadIdx.x & 63, G = E + n_shared;
  constexpr int kMaxPG = (kPermMaxGroups + kWave - 1) / kWave;
  const int PG = G / kWave + 1, g0 = lane * PG;   // lanes cover groups 0 .. G (the totals)
  int cnt[kMaxPG], til[kMaxPG], sc = 0, st = 0, sa = 0;
#pragma unroll
  for (int i = 0; i < kMaxPG; ++i) {
    const int g = g0 + i;
    cnt[i] = i < PG && g < G ? (g < E ? total[g] : T) : 0;
    til[i] = (cnt[i] + tile_rows - 1) / tile_rows;
    sc += cnt[i];
    st += til[i];
    sa += cnt[i] > 0 ? 1 : 0;
  }
  int off = wave_inclusive_sum(sc) - sc, toff = wave_inclusive_sum(st) - st, na = wave_inclusive_sum(sa) - sa;
#pragma unroll
  for (int i = 0; i < kMaxPG; ++i) {
    const int g = g0 + i;
    if (i < PG && g <= G) {
      pb.offsets[g] = off;
      pb.tile_off[g] = toff;
      if (g < E) total[g] = off;
      if (g < G && cnt[i] > 0) pb.active[na++] = g;
    }
    off += cnt[i];
    toff += til[i];
  }
  if (lane == kWave - 1) pb.n_active[0] = na;
  if (!pb.wide_off) return;
  int sw = 0;
#pragma unroll
  for (int i = 0; i < kMaxPG; ++i) sw += (cnt[i] + kGemmBM - 1) / kGemmBM;
  int woff = wave_inclusive_sum(sw) - sw;
#pragma unroll
  for (int i = 0; i < kMaxPG; ++i) {
    if (i < PG && g0 + i <= G) pb.wide_off[g0 + i] = woff;
    woff += (cnt[i] + kGemmBM - 1) / kGemmBM;
  }
}

// Orders LDS accesses of the lanes of one wavefront (which execute them in order) for the compiler.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Lanes of the wavefront that hold the same expert e (valid lanes only).
__device__ __forceinline__ uint64_t same_expert(int e, bool valid) {
  uint64_t same = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 9; ++b) {
    const uint64_t bb = __ballot(valid && ((e >> b) & 1));
    same &= ((e >> b) & 1) ? bb : ~bb;
  }
  return same;
}

// IT: entries per thread, T * K <= IT * nthreads.
template <int IT>
__device__ inline void permute_block(const int32_t* idx, int T, int K, int E, int n_shared, int tile_rows,
                                     const PermBuffers& pb, PermLds& s, int nthreads) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = T * K;
  const int per = (n + nthreads - 1) / nthreads;              // 64-entry rounds of a wavefront
  const int nact = (n + 64 * per - 1) / (64 * per);           // wavefronts with entries
  const int j0 = wave * 64 * per + lane;
  int e[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int j = j0 + 64 * i;
    e[i] = i < per && j < n ? idx[j] : -1;
    if (e[i] >= E) e[i] = -1;
  }
  if (wave < nact) {
    for (int g = lane; g < E; g += kWave) s.wcnt[wave][g] = 0;
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (e[i] >= 0) atomicAdd(&s.wcnt[wave][e[i]], 1);   // LDS integer counts: order-independent
  }
  lds_sync();
  for (int g = tid; g < E; g += nthreads) {   // counts -> each wavefront's first rank
    int run = 0;
    for (int w = 0; w < nact; ++w) {
      const int c = s.wcnt[w][g];
      s.wcnt[w][g] = run;
      run += c;
    }
    s.total[g] = run;
  }
  lds_sync();
  if (wave == 0) permute_scan_groups(s.total, T, E, n_shared, tile_rows, pb);
  // shared-expert rows: token t of shared expert s sits at row n + s*T + t
  for (int r = tid; r < n_shared * T; r += nthreads) pb.row_tok[n + r] = r % T;
  lds_sync();
  if (wave >= nact) return;
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    if (i >= per) break;
    const bool valid = e[i] >= 0;
    const uint64_t same = same_expert(e[i], valid);
    const uint64_t lower = same & lanemask_lt(lane);
    const int before = valid ? s.wcnt[wave][e[i]] : 0;
    wave_lds_order();
    if (valid && lower == 0) s.wcnt[wave][e[i]] = before + __popcll(same);   // one lane per expert
    wave_lds_order();
    if (valid) {
      const int j = j0 + 64 * i;
      const int pos = s.total[e[i]] + before + __popcll(lower);
      pb.perm[pos] = j;
      pb.inv[j] = pos;
      pb.row_tok[pos] = j / K;
    }
  }
}

// The same layout computed by one wavefront, for n = T*K <= 64 entries and G = E + n_shared < 64
// groups: lane j holds entry j and lane g group g. Group sizes come from a pass over the
// entries, first rows and row-tiles from lane prefix sums, the rank of an entry among equal
// experts from ballots on the expert id bits; no LDS passes and no barriers. Same outputs as
// permute_block (and the same contract for `idx`).
__device__ inline void permute_wave(const int32_t* idx, int T, int K, int E, int n_shared, int tile_rows,
                                    const PermBuffers& pb) {
  const int lane = threadIdx.x & 63;
  const int n = T * K, G = E + n_shared;
  const int e = lane < n ? idx[lane] : -1;
  const bool valid = e >= 0 && e < E;
  uint64_t same = __ballot(valid);   // as same_expert, six id bits (E < 64)
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    const uint64_t bb = __ballot(valid && ((e >> b) & 1));
    same &= ((e >> b) & 1) ? bb : ~bb;
  }
  int c = 0;   // entries of expert `lane` (an invalid entry matches no lane below E)
  for (int j = 0; j < n; ++j) c += __builtin_amdgcn_readlane(e, j) == lane ? 1 : 0;
  if (lane >= E) c = lane < G ? T : 0;   // shared groups hold every token; none past G
  const int tiles = (c + tile_rows - 1) / tile_rows;
  int off = wave_inclusive_sum(c), toff = wave_inclusive_sum(tiles);
  off -= c;   // first row and row-tile of group `lane`; lane G: the totals
  toff -= tiles;
  if (lane <= G) {
    pb.offsets[lane] = off;
    pb.tile_off[lane] = toff;
  }
  const uint64_t act = __ballot(lane < G && c > 0);
  if (lane < G && c > 0) pb.active[__popcll(act & lanemask_lt(lane))] = lane;
  if (lane == 0) pb.n_active[0] = __popcll(act);
  // shared-expert rows: token t of shared expert s sits at row n + s*T + t
  for (int r = lane; r < n_shared * T; r += kWave) pb.row_tok[n + r] = r % T;
  const int first = __shfl(off, valid ? e : 0);
  if (valid) {
    const int pos = first + __popcll(same & lanemask_lt(lane));
    pb.perm[pos] = lane;
    pb.inv[lane] = pos;
    pb.row_tok[pos] = lane / K;
  }
}

}  // namespace maskmoe
