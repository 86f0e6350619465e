// Low-rank adapters of the experts (Stage 2 of the fine-tuning, Section 3.2; rank 8, alpha 16
// in Appendix B; routed and shared experts): an adapted projection computes
// W x + s B (A x), s = alpha / r, for the gate, up and down projections of every expert.
//
// The adapter term rides in the expert GEMMs as one more 64-wide k-tile (gemm_tile.hpp):
// A' = [U | rows] with U = rows A^T (r or 2r values, zero-padded to 64, bf16) and
// B' = [s B | W] (the matching s B row, zero-padded, bf16). For gate/up, U holds A_gate x in
// columns 0..r-1 and A_up x in r..2r-1, and a gate row of B' carries s B_gate in columns
// 0..r-1, an up row s B_up in r..2r-1, so the two adapters stay apart in one product.
// lora_prepare_kernel builds B' and computes U (gate/up: from the gathered token rows),
// lora_hidden_kernel V = h A_down^T (down: from the SwiGLU rows), with v_mfma_f32_16x16x32_bf16,
// 16 rows per workgroup, per expert group.

#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace maskmoe {
namespace {

constexpr int kLoraThreads = 256;

// B' rows: [G, rows, 64] from b [G, rows, r] (shared groups from bs), scaled by s and padded;
// one thread per 8 columns of a row (one 16-byte store).
// gate_up (UPSPLIT): rows < F carry columns 0..r-1, rows >= F columns r..2r-1.
// WHOLE: r % 8 == 0 and 16-byte aligned matrices, so that a piece is eight adapter values (one load)
// or zeros; otherwise values are taken one by one.
template <bool UPSPLIT, bool WHOLE>
__device__ __forceinline__ void lora_pack(const uint16_t* __restrict__ b, const uint16_t* __restrict__ bs, int g, int E,
                                          int rows, int F, int r, float s, uint16_t* __restrict__ out, int first,
                                          int stride) {
  const uint16_t* src = g < E ? b + static_cast<size_t>(g) * rows * r : bs + static_cast<size_t>(g - E) * rows * r;
  u32x4* dst = reinterpret_cast<u32x4*>(out + static_cast<size_t>(g) * rows * 64);
  const int n = rows * 8;
#pragma unroll 4
  for (int i = first; i < n; i += stride) {
    const int row = i >> 3, c8 = (i & 7) * 8;
    const int c0 = (UPSPLIT && row >= F) ? r : 0;   // first column of this row's adapter
    const uint16_t* v = src + static_cast<size_t>(row) * r - c0;   // + c: the value of column c
    u32x4 w = {0u, 0u, 0u, 0u};
    if (WHOLE) {
      if (c8 >= c0 && c8 < c0 + r) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(v + c8);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[j] = f32x2_to_bf16x2(s * __uint_as_float(x[j] << 16), s * __uint_as_float(x[j] & 0xffff0000u));
      }
    } else if (c8 + 8 > c0 && c8 < c0 + r) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = c8 + 2 * j + h;
          const float e = c >= c0 && c < c0 + r ? s * bf16_to_f32(v[c]) : 0.0f;
          w[j] |= static_cast<uint32_t>(f32_to_bf16(e)) << (16 * h);
        }
    }
    dst[i] = w;
  }
}

// out[row, 0..63] = bf16(src_row . A_g[q]) for q < nq (A_g the [nq, K] adapter matrix of the
// row's group), 0 for q >= nq. One workgroup per 16 rows of a group (`block`: tile_rows / 16 per row tile
// of the permutation); its 4 wavefronts take contiguous quarters of K, 8 k-steps of loads in flight,
// and their partial sums are added in LDS in wave order.
constexpr int kLoraRows = 16, kLoraWaves = kLoraThreads / 64, kLoraUnroll = 8;
__device__ __forceinline__ void lora_down(const uint16_t* __restrict__ src, const int32_t* __restrict__ row_tok, int K,
                                          const uint16_t* __restrict__ a, const uint16_t* __restrict__ as, int nq,
                                          int G, int E, const int32_t* __restrict__ offsets,
                                          const int32_t* __restrict__ tile_off, int tile_rows,
                                          uint16_t* __restrict__ out, int block) {
  __shared__ float part[kLoraWaves][kLoraRows][32];
  const int kSub = tile_rows / kLoraRows;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mt = block / kSub, sub = block % kSub;
  // The group with tile_off[g] <= mt < tile_off[g + 1], one group per lane: a workgroup is short, and
  // each step of a binary search is a round trip to memory (DeepSeek-shaped, 2000 tokens, gate/up:
  // 40.8 -> 35.4 us at the least).
  int g = -1, mt0 = 0, row0 = 0, row_end = 0;
  for (int base = 0; base < G && g < 0; base += 64) {
    const int q = min(base + lane, G - 1);
    const int m0 = tile_off[q], m1 = tile_off[q + 1], r0 = offsets[q], r1 = offsets[q + 1];
    const uint64_t hit = __ballot(m0 <= mt && mt < m1);
    if (hit) {
      const int l = __builtin_ctzll(hit);
      g = min(base + l, G - 1);
      mt0 = __builtin_amdgcn_readlane(m0, l);
      row0 = __builtin_amdgcn_readlane(r0, l);
      row_end = __builtin_amdgcn_readlane(r1, l);
    }
  }
  if (g < 0) return;   // past the last tile
  row0 += (mt - mt0) * tile_rows + sub * kLoraRows;
  if (row0 >= row_end) return;   // the whole workgroup leaves together
  const int rr = min(row0 + (lane & 15), row_end - 1);
  const uint16_t* xrow = src + static_cast<size_t>(row_tok ? row_tok[rr] : rr) * K + (lane >> 4) * 8;
  const uint16_t* la = g < E ? a + static_cast<size_t>(g) * nq * K : as + static_cast<size_t>(g - E) * nq * K;
  const int n0 = lane & 15, n1 = n0 + 16;
  const uint16_t* b0 = la + static_cast<size_t>(min(n0, nq - 1)) * K + (lane >> 4) * 8;
  const uint16_t* b1 = la + static_cast<size_t>(min(n1, nq - 1)) * K + (lane >> 4) * 8;
  const bool two = nq > 16, has0 = n0 < nq, has1 = n1 < nq;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  const int steps = K / 32, per = (steps + kLoraWaves - 1) / kLoraWaves;
  const int s0 = min(wave * per, steps), s1 = min(s0 + per, steps);
  for (int s = s0; s < s1; s += kLoraUnroll) {   // all loads of kLoraUnroll k-steps first; zeros past s1
    u32x4 av[kLoraUnroll], bv0[kLoraUnroll], bv1[kLoraUnroll];
#pragma unroll
    for (int u = 0; u < kLoraUnroll; ++u) {
      const bool in = s + u < s1;
      const int k = (s + u) * 32;
      av[u] = in ? *reinterpret_cast<const u32x4*>(xrow + k) : zero;
      bv0[u] = in && has0 ? *reinterpret_cast<const u32x4*>(b0 + k) : zero;
      bv1[u] = in && has1 ? *reinterpret_cast<const u32x4*>(b1 + k) : zero;
    }
#pragma unroll
    for (int u = 0; u < kLoraUnroll; ++u)
      if (s + u < s1) {
        acc0 = mfma_16x16x32(av[u], bv0[u], acc0);
        if (two) acc1 = mfma_16x16x32(av[u], bv1[u], acc1);
      }
  }
  // acc[i] is row 4 (lane >> 4) + i, column lane & 15 (second tile: + 16)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    part[wave][4 * (lane >> 4) + i][n0] = acc0[i];
    part[wave][4 * (lane >> 4) + i][n1] = acc1[i];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kLoraRows * 64; e += kLoraThreads) {
    const int r = e / 64, c = e % 64, row = row0 + r;
    if (row >= row_end) continue;
    float v = 0.0f;
    if (c < 32) {
#pragma unroll
      for (int w = 0; w < kLoraWaves; ++w) v += part[w][r][c];
    }
    out[static_cast<size_t>(row) * 64 + c] = f32_to_bf16(v);
  }
}

constexpr int kPackPer = 8;   // rounds of a packing workgroup

struct PrepareArgs {
  LoraArgs l;
  const uint16_t* x;
  PermBuffers pb;
  int d, F, E, G, tile_rows, u_blocks;
  int gu_blocks, dn_blocks;   // packing workgroups of one expert's gate/up and down adapters
  bool whole;
};

// U = A x of every row (workgroups 0 .. u_blocks - 1) beside the packing of both scaled B matrices
// (the rest), in one launch instead of three. DeepSeek-shaped, 2000 tokens: 59 -> 53 us (the gather of x
// by 64-byte pieces bounds it); Mixtral-shaped, 300 tokens: 50 -> 17 us.
__global__ __launch_bounds__(kLoraThreads) void lora_prepare_kernel(const PrepareArgs p) {
  const int b = static_cast<int>(blockIdx.x);
  if (b < p.u_blocks) {
    lora_down(p.x, p.pb.row_tok, p.d, p.l.a_gate_up, p.l.as_gate_up, 2 * p.l.rank, p.G, p.E, p.pb.offsets, p.pb.tile_off,
              p.tile_rows, p.l.u, b);
    return;
  }
  const int per = p.gu_blocks + p.dn_blocks;
  const int q = b - p.u_blocks, g = q / per, w = q % per;
  const bool gu = w < p.gu_blocks;
  const int first = (gu ? w : w - p.gu_blocks) * kLoraThreads + threadIdx.x;
  const int stride = (gu ? p.gu_blocks : p.dn_blocks) * kLoraThreads;
  auto pack = [&](auto whole) {
    constexpr bool W = decltype(whole)::value;
    if (gu) lora_pack<true, W>(p.l.b_gate_up, p.l.bs_gate_up, g, p.E, 2 * p.F, p.F, p.l.rank, p.l.scale, p.l.bp_gate_up, first, stride);
    else lora_pack<false, W>(p.l.b_down, p.l.bs_down, g, p.E, p.d, p.F, p.l.rank, p.l.scale, p.l.bp_down, first, stride);
  };
  if (p.whole) pack(std::true_type{});
  else pack(std::false_type{});
}

// V = A h of every row.
__global__ __launch_bounds__(kLoraThreads) void lora_hidden_kernel(const PrepareArgs p, const uint16_t* __restrict__ h) {
  lora_down(h, nullptr, p.F, p.l.a_down, p.l.as_down, p.l.rank, p.G, p.E, p.pb.offsets, p.pb.tile_off, p.tile_rows, p.l.v,
            static_cast<int>(blockIdx.x));
}

PrepareArgs prepare_args(const LoraArgs& l, const ExpertArgs& a, const PermBuffers& pb, int tile_rows, int max_tiles) {
  PrepareArgs p;
  p.l = l;
  p.x = static_cast<const uint16_t*>(a.x);
  p.pb = pb;
  p.d = a.d; p.F = a.F; p.E = a.E; p.G = a.E + a.n_shared;
  p.tile_rows = tile_rows;
  p.u_blocks = tile_rows / kLoraRows * max_tiles;
  constexpr int kItems = kPackPer * kLoraThreads;
  p.gu_blocks = (2 * a.F * 8 + kItems - 1) / kItems;
  p.dn_blocks = (a.d * 8 + kItems - 1) / kItems;
  p.whole = l.rank % 8 == 0;
  for (const uint16_t* m : {l.b_gate_up, l.b_down, l.bs_gate_up, l.bs_down})
    p.whole = p.whole && reinterpret_cast<uintptr_t>(m) % 16 == 0;
  return p;
}

}  // namespace

hipError_t launch_lora_prepare(const LoraArgs& l, const ExpertArgs& a, const PermBuffers& pb, int tile_rows,
                               int max_tiles, hipStream_t stream) {
  const PrepareArgs p = prepare_args(l, a, pb, tile_rows, max_tiles);
  hipLaunchKernelGGL(lora_prepare_kernel, dim3(p.u_blocks + p.G * (p.gu_blocks + p.dn_blocks)), dim3(kLoraThreads), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_lora_hidden(const LoraArgs& l, const ExpertArgs& a, const PermBuffers& pb, int tile_rows,
                              int max_tiles, const uint16_t* h, hipStream_t stream) {
  const PrepareArgs p = prepare_args(l, a, pb, tile_rows, max_tiles);
  hipLaunchKernelGGL(lora_hidden_kernel, dim3(p.u_blocks), dim3(kLoraThreads), 0, stream, p, h);
  return hipGetLastError();
}

}  // namespace maskmoe
