// Expert FFNs of fp32 layers: grouped GEMMs on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (fp32 products and sums, 256 FLOP per clock and CU, twice the vector
// rate), replacing one thread per output element that walked its weight row alone, a different
// cache line per lane and load. A workgroup of four wavefronts (2 token blocks x 2 weight
// blocks of 16) owns 32 rows of one expert and 32 output columns (gate/up: 32 gate and the 32
// matching up rows of the weights); 64-column chunks of both operands pass through registers
// (two in flight) into LDS. Small output tiles, since one instruction takes 32 cycles: 1.4 LDS
// bytes per matrix FLOP suffice, and a small layer still fills the chip. A lane's 16-byte LDS
// read of four neighbouring k feeds four instructions, so instruction i sums the k = 4 g + i of
// the lane groups g. Weight rows are the row operand: a lane then holds four neighbouring
// output columns of one token. Measured, 64 tokens, d 256, F 512, 8 experts, top-2: the layer 237 ->
// 32 us, this pair of kernels 208 -> about 12 us; its error against 64 bits is unchanged (6e-7).

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace maskmoe {
namespace {

constexpr int kThreads = 256;
constexpr int kTM = kF32TileRows;   // token rows per workgroup
constexpr int kTN = 32;             // output columns per workgroup
constexpr int kCK = 64;             // reduction values per chunk: 16 16-byte units per row
static_assert(kTM == 32, "two 16-row token blocks");

struct F32Args {
  const float* a;           // EPI 0: x [T, d] (rows via row_tok); EPI 1: H [rows, F]
  const int32_t* row_tok;
  const float* w;           // routed weights: EPI 0 [E, 2F, d], EPI 1 [E, d, F]
  const float* ws;          // shared weights
  const int32_t* offsets;   // [G+1]
  const int32_t* tile_off;  // [G+1], tiles of kTM rows
  float* out;               // EPI 0: H [rows, F]; EPI 1: O [rows, d]
  int G, E, N, K;           // N: output columns (F or d), K: reduction length
  int n_tiles;
};

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// KMODE: 0 whole chunks (K % 64 == 0), 1 rows of whole 16-byte units (K % 4 == 0), 2 any K.
template <int EPI, int KMODE>
__global__ __launch_bounds__(kThreads) void f32_gemm_kernel(const F32Args p) {
  constexpr int NF = EPI == 0 ? 2 : 1;         // weight fragments per wavefront: gate and up, or down
  constexpr int WR = NF * kTN, ROWS = WR + kTM;
  constexpr int PW = WR / 16, PER = ROWS / 16; // 16-byte pieces per thread and chunk, the first PW of weights
  __shared__ f32x4 lds[2][ROWS * 16];

  const int live = p.tile_off[p.G] * p.n_tiles;
  if (static_cast<int>(blockIdx.x) >= live) return;
  const int lid = xcd_tile_id(live);
  int lo = 0, hi = p.G;                        // tile_off[lo] <= lid / n_tiles < tile_off[hi]
  const int mt = lid / p.n_tiles;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.tile_off[mid] <= mt) lo = mid; else hi = mid;
  }
  const int g = lo, mtiles = p.tile_off[g + 1] - p.tile_off[g];
  const int within = lid - p.tile_off[g] * p.n_tiles;
  const int m = within % mtiles, n0 = within / mtiles * kTN;   // a group's row tiles share weights: neighbours
  const int row0 = p.offsets[g] + m * kTM, row_end = p.offsets[g + 1];
  const int nc = (p.K + kCK - 1) / kCK;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const size_t mat = static_cast<size_t>(NF) * p.N * p.K;
  const float* wg = g < p.E ? p.w + g * mat : p.ws + (g - p.E) * mat;

  // Piece i of this thread: stage row 16 i + tid / 16 (weight rows, then token rows), floats
  // 4 (tid % 16) .. + 3 of the chunk. Rows past the end are clamped: their products are never
  // stored.
  const int pr = tid >> 4, pk = (tid & 15) * 4;
  const float* src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int r = 16 * i + pr;
    if (i < PW) {
      const int n = min(n0 + r % kTN, p.N - 1);
      src[i] = wg + static_cast<size_t>(r < kTN ? n : p.N + n) * p.K;
    } else {
      const int t = min(row0 + r - WR, row_end - 1);
      src[i] = p.a + static_cast<size_t>(EPI == 0 ? p.row_tok[t] : t) * p.K;
    }
  }
  f32x4 reg[2][PER];
  auto load = [&](int c, f32x4 (&r)[PER]) {   // chunks past the last one reload it and are not used
    const int k = min(c, nc - 1) * kCK + pk;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (KMODE == 0) {
        r[i] = *reinterpret_cast<const f32x4*>(src[i] + k);
      } else if (KMODE == 1) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(src[i] + min(k, p.K - 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) r[i][e] = k < p.K ? v[e] : 0.0f;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = src[i][min(k + e, p.K - 1)];
          r[i][e] = k + e < p.K ? v : 0.0f;
        }
      }
    }
  };
  // LDS rows of 256 bytes; unit u of row r at u ^ (r % 16): 16 rows read at one unit, or one row
  // written, touch every bank once
  const int dst = pr * 16 + ((tid & 15) ^ pr);
  auto store = [&](int buf, const f32x4 (&r)[PER]) {
#pragma unroll
    for (int i = 0; i < PER; ++i) lds[buf][dst + kThreads * i] = r[i];
  };
  const int l16 = lane & 15, lg = lane >> 4;
  f32x4 acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < kCK / 16; ++kk) {
      const int u = (4 * kk + lg) ^ l16;
      const f32x4 t = lds[buf][(WR + 16 * wm + l16) * 16 + u];
      f32x4 w[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) w[f] = lds[buf][(kTN * f + 16 * wn + l16) * 16 + u];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = mfma_f32(w[f][e], t[e], acc[f]);
    }
  };
  int c = 0;
  auto step = [&](auto buf_c) {   // chunk c in LDS buffer and register set c & 1, as in batch.hip
    constexpr int buf = decltype(buf_c)::value;
    load(c + 2, reg[buf]);
    compute(buf);
    store(buf ^ 1, reg[buf ^ 1]);
    lds_sync();
    return ++c < nc;
  };
  load(0, reg[0]);
  load(1, reg[1]);
  store(0, reg[0]);
  lds_sync();
  while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
  }

  // acc[f][i]: weight row 16 wn + 4 lg + i, token row 16 wm + l16
  const int row = row0 + 16 * wm + l16, col = n0 + 16 * wn + 4 * lg;
  if (row >= row_end || col >= p.N) return;
  float v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = EPI == 0 ? (acc[0][i] / (1.0f + expf(-acc[0][i]))) * acc[NF - 1][i] : acc[0][i];
  float* out = p.out + static_cast<size_t>(row) * p.N + col;
  if (p.N % 4 == 0) {   // rows of the output start on 16 bytes
    *reinterpret_cast<f32x4*>(out) = f32x4{v[0], v[1], v[2], v[3]};
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (col + i < p.N) out[i] = v[i];
  }
}

template <int EPI>
hipError_t launch(const F32Args& p, int max_tiles, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(max_tiles) * p.n_tiles), block(kThreads);
  if (p.K % kCK == 0) hipLaunchKernelGGL((f32_gemm_kernel<EPI, 0>), grid, block, 0, s, p);
  else if (p.K % 4 == 0) hipLaunchKernelGGL((f32_gemm_kernel<EPI, 1>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((f32_gemm_kernel<EPI, 2>), grid, block, 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_experts_f32(const ExpertArgs& a, const PermBuffers& pb, float* H, float* O,
                              void* y, hipStream_t stream, hipEvent_t* marks) {
  const int64_t TK = static_cast<int64_t>(a.T) * a.K;
  const int max_tiles = static_cast<int>(TK / kTM + std::min<int64_t>(TK, a.E)) +
                        a.n_shared * ((a.T + kTM - 1) / kTM);
  F32Args p;
  p.row_tok = pb.row_tok;
  p.offsets = pb.offsets;
  p.tile_off = pb.tile_off;
  p.E = a.E; p.G = a.E + a.n_shared;
  p.a = static_cast<const float*>(a.x);
  p.w = static_cast<const float*>(a.w_gate_up);
  p.ws = static_cast<const float*>(a.ws_gate_up);
  p.out = H;
  p.N = a.F; p.K = a.d;
  p.n_tiles = (p.N + kTN - 1) / kTN;
  hipError_t err = launch<0>(p, max_tiles, stream);
  if (err != hipSuccess) return err;
  record_mark(marks, 0, stream);
  p.a = H;
  p.w = static_cast<const float*>(a.w_down);
  p.ws = static_cast<const float*>(a.ws_down);
  p.out = O;
  p.N = a.d; p.K = a.F;
  p.n_tiles = (p.N + kTN - 1) / kTN;
  err = launch<1>(p, max_tiles, stream);
  if (err != hipSuccess) return err;
  record_mark(marks, 1, stream);
  err = launch_combine_f32(a, pb, O, y, stream);
  record_mark(marks, 2, stream);
  return err;
}

}  // namespace maskmoe
