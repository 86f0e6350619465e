// Expert FFNs of a serving-sized batch (bf16): more tokens than the few-token kernels take, but
// few enough rows per expert that the time is still the stream of the experts' weights from HBM.
//
// The 256 x 256 tiles of the many-token path (gemm_tile.hpp) keep about one k-tile of weights in
// flight per CU behind a matrix pipeline that multiplies mostly padding there (4.1 TB/s). Here a
// workgroup of four wavefronts owns 128 weight rows of one expert and BM token rows (64 or 128)
// and streams 64-column chunks of both: chunks c + 1 and c + 2 travel in registers while chunk c
// is multiplied from LDS on v_mfma_f32_32x32x16_bf16, so the 3 (BM 64) or 2 (BM 128) workgroups
// of a CU keep 96 or 64 KB of weights in flight. Weight rows are the MFMA's row operand: a lane
// then holds four neighbouring output columns of one token and stores them at once, and the gate
// and up values of a column meet in one lane.
// Workgroups that share weight rows (a group's row tiles) are neighbours on one XCD and read them
// through its L2; weights that one workgroup alone reads are loaded non-temporally.
// Measured against the 256-row tiles, Mixtral-shaped layer, packed, soft prior: 17 tokens 668 -> 433 us
// (gate/up 271 us = 6.9 TB/s), 96 tokens 664 -> 452, 200 tokens 675 -> 526; DeepSeek-shaped, 333 tokens:
// 395 -> 267 (gate/up 189 -> 141, down 131 -> 78). Three or four chunks in flight changed nothing, and
// 256 token rows (one workgroup per CU) lost 15-60%: its loads, LDS accesses and products no
// longer overlap.
// Adapted experts (LORA) take the adapters' term as one more chunk, as the many-token path does.
// Every sum is formed in the many-token path's order, so that a layer gives the same bits on either
// (and as its training forward): chunks in ascending order, and a down projection whose 256 x 256
// tile that path would split (tile_slices) in the same slices, which batch_fixup_kernel adds in order
// (5.6 us at 96 tokens). Starting neighbouring column tiles at different chunks, so that they do not read
// the same columns at once, was 2 to 3% of a layer with row-major weights (none packed; 10% of the GEMMs at
// d 2048, F 4096) and changed the bits: not done.

#include "common.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <type_traits>

namespace maskmoe {
namespace {

constexpr int kW = 128;           // weight rows per workgroup (one packed group)
constexpr int kCK = kPackCols;    // reduction values per chunk
// Byte offset of a token row that is not there: past any operand (fewer than 2^31 elements of whole
// 128-byte pieces, so at most 2^32 - 128 bytes); the load returns zeros without touching memory.
constexpr uint32_t kNoRow = 0xfffffff0u;

struct BatchArgs {
  const uint16_t* a;        // EPI 0: x [T, d] (rows via row_tok); EPI 1: H [rows, F]
  const int32_t* row_tok;
  const uint16_t* w;        // routed weights: EPI 0 [E, 2F, d], EPI 1 [E, d, F]
  const uint16_t* ws;       // shared weights
  const int32_t* offsets;   // [G+1]
  const int32_t* tile_off;  // [G+1], tiles of BM rows
  uint16_t* out;            // EPI 0: H [rows, F]; EPI 1: O [rows, d]
  const int32_t* wide_off;  // [G+1], tiles of kGemmBM rows
  float* part;              // EPI 1: partial tiles, kTailSlots x [256 rows][256 columns] fp32
  int G, E, N, K, F, rows;  // N: output columns (F or d), K: reduction length
  const uint16_t* lora_u;   // LORA: rank projections of a's rows, bf16 [rows, 64]
  const uint16_t* lora_b;   // LORA: the scaled adapter rows beside the weight rows, bf16 [G, weight rows, 64]
  int n_tiles, split, a_rows;   // split: workgroups that share a tile's slices; a_rows: rows of a (T or rows)
  int cu_xcd;
  int skew;                 // batch_skewed: the many-token path's tiles are taken instead
};

constexpr int kThreads = 256, kRowsPerPiece = kThreads / 8;
constexpr int kPW = kW / kRowsPerPiece;   // 16-byte pieces of weights per thread and chunk
template <int BM>
constexpr int kPieces = kPW + BM / kRowsPerPiece;

// The stream of one tile: acc += W X^T over nc chunks. off[]: this thread's 16-byte pieces of a
// chunk (the first PW are weights, in w from byte w0 + chunk * wstep; then tokens, in a from a0 + 128 chunk).
// NT: non-temporal weight loads. LORA: with `extra`, one more chunk goes
// first, the adapters' term [s B] U^T (weight pieces in xw at xoff[], token pieces in xu).
template <int BM, bool NT, bool LORA>
__device__ __forceinline__ void stream_tile(const void* w, uint32_t wbytes, uint32_t w0, uint32_t wstep,
                                            const void* a, uint32_t abytes, uint32_t a0, int nc,
                                            const uint32_t (&off)[kPieces<BM>], u32x4 (*lds)[(kW + BM) * 8], int wrow0,
                                            int wrow1, int trow, f32x16 (&acc)[2][BM / 64], bool extra,
                                            const void* xw, uint32_t xwbytes, const void* xu, uint32_t xubytes,
                                            const uint32_t (&xoff)[kPieces<BM>]) {
  constexpr int TN = BM / 64, PER = kPieces<BM>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int dst = (tid >> 3) * 8 + ((tid & 7) ^ lds_swizzle(tid >> 3));   // piece i: + kThreads * i
  const int sw = lds_swizzle(lane & 31);
  u32x4 reg[2][PER];
  // Past the last chunk the buffers are empty and the scalar offset is 0 (the range check compares with
  // the size less that offset, which must not wrap): the loads return zeros without touching memory, and
  // every step has the same loads behind the ones its stores wait for.
  constexpr int kNt = 2;   // the load's non-temporal bit
  const int x = LORA && extra ? 1 : 0, steps = nc + x;
  auto load = [&](int ci, u32x4 (&r)[PER]) {
    const int c = LORA ? ci - x : ci;
    const bool in = c < nc;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(w, in ? wbytes : 0), ar = make_rsrc(a, in ? abytes : 0);
    const uint32_t ws = in ? w0 + static_cast<uint32_t>(c) * wstep : 0;
    const uint32_t as = in ? a0 + static_cast<uint32_t>(c) * (2 * kCK) : 0;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      r[i] = i < kPW ? __builtin_amdgcn_raw_buffer_load_b128(wr, off[i], ws, NT ? kNt : 0)
                    : __builtin_amdgcn_raw_buffer_load_b128(ar, off[i], as, 0);
  };
  auto store = [&](int buf, const u32x4 (&r)[PER]) {
#pragma unroll
    for (int i = 0; i < PER; ++i) lds[buf][dst + kThreads * i] = r[i];
  };
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < kCK / 16; ++kk) {
      const int ch = (kk * 2 + (lane >> 5)) ^ sw;
      const u32x4 w0 = lds[buf][wrow0 * 8 + ch], w1 = lds[buf][wrow1 * 8 + ch];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const u32x4 t = lds[buf][(trow + 32 * j) * 8 + ch];
        acc[0][j] = mfma_32x32x16(w0, t, acc[0][j]);
        acc[1][j] = mfma_32x32x16(w1, t, acc[1][j]);
      }
    }
  };
  // Chunk c sits in LDS buffer c & 1 and came from register set c & 1 (a compile-time index, so
  // that the sets stay in registers), which takes chunk c + 2. The loads come first, the LDS
  // stores of chunk c + 1 last. Returns whether another chunk follows.
  int c = 0;
  auto step = [&](auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    load(c + 2, reg[buf]);
    __builtin_amdgcn_sched_barrier(0);
    compute(buf);
    __builtin_amdgcn_sched_barrier(0);
    store(buf ^ 1, reg[buf ^ 1]);
    lds_sync();
    return ++c < steps;
  };
  if (LORA && extra) {
    const __amdgpu_buffer_rsrc_t br = make_rsrc(xw, xwbytes), ur = make_rsrc(xu, xubytes);
#pragma unroll
    for (int i = 0; i < PER; ++i) reg[0][i] = __builtin_amdgcn_raw_buffer_load_b128(i < kPW ? br : ur, xoff[i], 0, 0);
  } else {
    load(0, reg[0]);
  }
  load(1, reg[1]);
  store(0, reg[0]);
  lds_sync();
  while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
  }
}

// EPI 0: gate/up with SwiGLU; EPI 1: down. PACKED: weights in the packed layout.
template <int EPI, int BM, bool PACKED, bool LORA>
__global__ __launch_bounds__(kThreads, BM == 64 ? 3 : 2) void batch_gemm_kernel(const BatchArgs p) {
  constexpr int TN = BM / 64;                  // 32-token fragments per wavefront
  __shared__ u32x4 lds[2][(kW + BM) * 8];

  const int per = p.n_tiles * p.split;         // jobs per row tile
  const int live = p.tile_off[p.G] * per;
  if (static_cast<int>(blockIdx.x) >= live || batch_skewed(p.tile_off[p.G], p.wide_off[p.G], p.skew)) return;
  const int lid = xcd_tile_id(live);
  int lo = 0, hi = p.G;                        // tile_off[lo] <= lid / per < tile_off[hi]
  const int mt = lid / per;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.tile_off[mid] <= mt) lo = mid; else hi = mid;
  }
  const int g = lo;
  const int mtiles = p.tile_off[g + 1] - p.tile_off[g];
  const int within = lid - p.tile_off[g] * per;
  const int m = within % mtiles, nz = within / mtiles;
  const int nt = nz / p.split;
  const int row0 = p.offsets[g] + m * BM, row_end = p.offsets[g + 1];
  TileSlices sl{1, -1};
  if (EPI == 1 && tail_can_split(1, p.K / kCK)) {
    const int wide_live = p.wide_off[p.G], wide_tiles = (p.N + kTileN - 1) / kTileN;
    sl = tile_slices(grouped_tile_lid(p.wide_off[g] + m * BM / kTileM, nt * kW / kTileN, wide_live, wide_tiles),
                     wide_live * wide_tiles, p.cu_xcd, p.K / kCK, true);
  }
  const int nc = p.K / kCK / sl.s;             // chunks of a slice

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;     // token part, weight half
  const int n0 = nt * (EPI == 0 ? kW / 2 : kW);
  const size_t mat = static_cast<size_t>(EPI == 0 ? 2 * p.F : p.N) * p.K;
  const uint16_t* wg = g < p.E ? p.w + g * mat : p.ws + (g - p.E) * mat;
  const uint32_t wbytes = static_cast<uint32_t>(2 * mat), abytes = 2u * static_cast<uint32_t>(p.a_rows) * p.K;

  // Piece i of this thread: row 32 i + tid / 8 of the stage (weight rows, then token rows), 16
  // bytes at column chunk tid % 8. Weight rows past the end are clamped and token rows past it
  // read as zeros: their products land in columns and rows that are never stored.
  const int pr = tid >> 3, pc = tid & 7;
  uint32_t off[kPieces<BM>];
#pragma unroll
  for (int i = 0; i < kPieces<BM>; ++i) {
    if (i < kPW) {
      const int r = kRowsPerPiece * i + pr;
      int elem;
      if (PACKED) elem = r * kPackCols;
      else if (EPI == 0) elem = (r < kW / 2 ? n0 + r : p.F + n0 + r - kW / 2) * p.K;
      else elem = min(n0 + r, p.N - 1) * p.K;
      off[i] = static_cast<uint32_t>(elem + pc * 8) * 2u;
    } else {
      const int r = row0 + kRowsPerPiece * (i - kPW) + pr;
      off[i] = r < row_end ? static_cast<uint32_t>((EPI == 0 ? p.row_tok[r] : r) * p.K + pc * 8) * 2u : kNoRow;
    }
  }

  // fragment rows of the stage: weights (EPI 0: gate rows and the matching up rows), tokens
  const int l32 = lane & 31;
  const int wrow0 = (EPI == 0 ? wn * 32 : wn * 64) + l32, wrow1 = wrow0 + (EPI == 0 ? kW / 2 : 32);
  const int trow = kW + wm * 32 * TN + l32;
  constexpr int wstep = 2 * (PACKED ? kPackBlock : kCK);
  // the adapters' chunk, in the first slice: weight rows of lora_b, token rows of U
  uint32_t xoff[kPieces<BM>];
  const void* xw = nullptr;
  const uint32_t wrows = EPI == 0 ? 2 * p.F : p.N;
  if (LORA) {
    xw = p.lora_b + static_cast<size_t>(g) * wrows * 64;
#pragma unroll
    for (int i = 0; i < kPieces<BM>; ++i) {
      if (i < kPW) {
        const int r = kRowsPerPiece * i + pr;
        const int row = EPI == 0 ? (r < kW / 2 ? n0 + r : p.F + n0 + r - kW / 2) : min(n0 + r, p.N - 1);
        xoff[i] = static_cast<uint32_t>(row * 64 + pc * 8) * 2u;
      } else {
        const int r = row0 + kRowsPerPiece * (i - kPW) + pr;
        xoff[i] = r < row_end ? static_cast<uint32_t>(r * 64 + pc * 8) * 2u : kNoRow;
      }
    }
  }

  for (int z = nz % p.split; z < sl.s; z += p.split) {   // this workgroup's slices (EPI 0: one)
    const int c0 = z * nc;
    // byte offsets of chunk c0 within the expert's matrix (below 2^32: 2 F d < 2^31 elements)
    const uint32_t w0 = PACKED ? 2u * (static_cast<uint32_t>(nt) * kW * p.K + static_cast<uint32_t>(c0) * kPackBlock)
                               : 2u * static_cast<uint32_t>(c0) * kCK;
    const uint32_t a0 = 2u * static_cast<uint32_t>(c0) * kCK;
    const bool extra = LORA && z == 0;
    f32x16 acc[2][TN];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    if (mtiles == 1)
      stream_tile<BM, true, LORA>(wg, wbytes, w0, wstep, p.a, abytes, a0, nc, off, lds, wrow0, wrow1, trow, acc, extra, xw,
                                  wrows * 128u, p.lora_u, static_cast<uint32_t>(p.rows) * 128u, xoff);
    else
      stream_tile<BM, false, LORA>(wg, wbytes, w0, wstep, p.a, abytes, a0, nc, off, lds, wrow0, wrow1, trow, acc, extra, xw,
                                   wrows * 128u, p.lora_u, static_cast<uint32_t>(p.rows) * 128u, xoff);

    // acc[i][j][4 q + e]: weight row 8 q + 4 (lane >> 5) + e of fragment i, token row lane & 31 of
    // fragment j
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int row = row0 + wm * 32 * TN + 32 * j + l32;
      if (row >= row_end) continue;
      if (EPI == 0) {
        uint16_t* dsth = p.out + static_cast<size_t>(row) * p.F + n0 + wn * 32 + 4 * (lane >> 5);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = silu(acc[0][j][4 * q + e]) * acc[1][j][4 * q + e];
          uint2 v;
          v.x = f32x2_to_bf16x2(h[0], h[1]);
          v.y = f32x2_to_bf16x2(h[2], h[3]);
          *reinterpret_cast<uint2*>(dsth + 8 * q) = v;
        }
      } else {
        float* slot = sl.s > 1 ? p.part + static_cast<size_t>(sl.slot + z) * kTailTileFloats : nullptr;
        const int wrow = m * BM % kTileM + row - row0, wcol = n0 % kTileN;           // within the 256 x 256 tile
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = wn * 64 + 32 * i + 8 * q + 4 * (lane >> 5);
            if (n0 + c >= p.N) continue;   // N % 64 == 0: four columns are all inside or all outside
            const f32x16& a = acc[i][j];
            if (sl.s > 1) {
              *reinterpret_cast<float4*>(slot + wrow * kTileN + wcol + c) =
                  make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
            } else {
              uint2 v;
              v.x = f32x2_to_bf16x2(a[4 * q], a[4 * q + 1]);
              v.y = f32x2_to_bf16x2(a[4 * q + 2], a[4 * q + 3]);
              *reinterpret_cast<uint2*>(p.out + static_cast<size_t>(row) * p.N + n0 + c) = v;
            }
          }
      }
    }
  }
}

// Adds the slices of the down projection's split tiles in slice order and stores their rows of O:
// kFixRows rows of one tile per workgroup, tail tile t of XCD xcd at workgroup 8 (t * parts + part) + xcd.
constexpr int kFixRows = 16;
__global__ __launch_bounds__(kThreads) void batch_fixup_kernel(const BatchArgs p, int parts) {
  const int b = blockIdx.x, xcd = b & 7, t = (b >> 3) / parts, part = (b >> 3) % parts;
  const int mt_live = p.wide_off[p.G], n_tiles = (p.N + kTileN - 1) / kTileN;
  const XcdShare x = xcd_share(xcd, mt_live * n_tiles, p.cu_xcd, p.K / kCK, true);
  if (x.s == 1 || t >= x.r) return;
  int mt, nt;
  grouped_tile_coords(x.base + x.full + t, mt_live, n_tiles, mt, nt);
  int lo = 0, hi = p.G;                        // wide_off[lo] <= mt < wide_off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.wide_off[mid] <= mt) lo = mid; else hi = mid;
  }
  const int row0 = p.offsets[lo] + (mt - p.wide_off[lo]) * kTileM, row_end = min(p.offsets[lo + 1], row0 + kTileM);
  const float* src = p.part + static_cast<size_t>(xcd * kTailSlotsPerXcd + t * x.s) * kTailTileFloats;
  auto sum = [&](int off) {   // four values at float offset off of every slice
    float4 v[kTailMaxSplit];
#pragma unroll
    for (int z = 0; z < kTailMaxSplit; ++z)
      if (z < x.s) v[z] = *reinterpret_cast<const float4*>(src + static_cast<size_t>(z) * kTailTileFloats + off);
    float4 a = v[0];
#pragma unroll
    for (int z = 1; z < kTailMaxSplit; ++z)
      if (z < x.s) {
        a.x += v[z].x; a.y += v[z].y; a.z += v[z].z; a.w += v[z].w;
      }
    return a;
  };
  if (batch_skewed(p.tile_off[p.G], mt_live, p.skew)) {   // tail_store_partial's layout: four rows of a column
    const int c = threadIdx.x, col = nt * kTileN + c;
    if (col >= p.N) return;
#pragma unroll
    for (int i = 0; i < kFixRows / 4; ++i) {
      const int r = part * kFixRows + 4 * i;
      if (row0 + r >= row_end) break;
      const int e = ((r >> 5 & 3) * kTileTN + (c >> 5 & 1)) * 4 + (r >> 3 & 3);
      const float4 a = sum((e * kTileThreads + ((r >> 7) * 4 + (c >> 6)) * kWave + 32 * (r >> 2 & 1) + (c & 31)) * 4);
      const float v[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (row0 + r + u < row_end) p.out[static_cast<size_t>(row0 + r + u) * p.N + col] = f32_to_bf16(v[u]);
    }
    return;
  }
  const int c = (threadIdx.x & 63) * 4, col = nt * kTileN + c;
  if (col >= p.N) return;
#pragma unroll
  for (int i = 0; i < kFixRows / 4; ++i) {
    const int r = part * kFixRows + 4 * i + (threadIdx.x >> 6);
    if (row0 + r >= row_end) break;
    const float4 a = sum(r * kTileN + c);
    uint2 o;
    o.x = f32x2_to_bf16x2(a.x, a.y);
    o.y = f32x2_to_bf16x2(a.z, a.w);
    *reinterpret_cast<uint2*>(p.out + static_cast<size_t>(row0 + r) * p.N + col) = o;
  }
}

template <int EPI, int BM>
void launch_bm(bool packed, int grid, const BatchArgs& p, hipStream_t s) {
  const dim3 g(grid), b(kThreads);
  if (p.lora_b) {
    if (packed) hipLaunchKernelGGL((batch_gemm_kernel<EPI, BM, true, true>), g, b, 0, s, p);
    else hipLaunchKernelGGL((batch_gemm_kernel<EPI, BM, false, true>), g, b, 0, s, p);
  } else {
    if (packed) hipLaunchKernelGGL((batch_gemm_kernel<EPI, BM, true, false>), g, b, 0, s, p);
    else hipLaunchKernelGGL((batch_gemm_kernel<EPI, BM, false, false>), g, b, 0, s, p);
  }
}

template <int EPI>
hipError_t launch(int bm, bool packed, int grid, const BatchArgs& p, hipStream_t s) {
  if (bm == 64) launch_bm<EPI, 64>(packed, grid, p, s);
  else launch_bm<EPI, 128>(packed, grid, p, s);
  return hipGetLastError();
}

}  // namespace

// By the rows an expert gets, since the time goes with the passes over the weights (row tiles).
// Layer times with 64-row and 128-row tiles here and on the many-token path (256-row tiles whose
// last one multiplies only its own 64-row pieces), by the average rows of a selectable expert:
// Mixtral-shaped, plain routing, 24 rows 446 / 456 / 539 us, 75 rows 700 / 534 / 563, 100 rows
// 708 / 579 / 574, 150 rows 917 / 888 / 612; hard mask over 4 experts, 75 rows 342 / 288 / 308,
// 104 rows 361 / 311 / 314, 150 rows 471 / 447 / 332. A prior sends more rows to some experts, whose
// second 128-row tile is another pass over their weights: `peak` is its largest entry over a uniform
// one's; soft prior over 4 of 8 experts (peak 1.5), 36 rows 469 / 478 / 545, 50 rows 565 / 508 / 554, 71
// rows 584 / 541 / 561. With dozens of experts the tiles of neighbouring experts hide such passes and the
// line lies at the average: DeepSeek-shaped, soft (peak 2.1), 31 rows 247 / 255 / 281, 66 rows
// 300 / 284 / 299, 84 rows 336 / 319 / 308, 113 rows 399 / 351 / 325; over its 12-expert set, 32 rows
// 81 / 86 / 83, 100 rows 96 / 97 / 99, 200 rows 139 / 124 / 108. What the rows really are is known on the
// device only (batch_skewed, below).
int batch_tile_rows(int T, int K, int pool, float peak) {
  const double avg = static_cast<double>(T) * K / pool;
  if (avg <= 36) return 64;
  return (pool >= 32 ? avg <= 75 : avg * peak <= 104) ? 128 : 0;
}

hipError_t launch_experts_batch(const ExpertArgs& a, const PermBuffers& pb, int bm, int pool, uint16_t* H, uint16_t* O,
                                float* part, void* y, hipStream_t stream, hipEvent_t* marks, const LoraArgs* lora) {
  const int64_t TK = static_cast<int64_t>(a.T) * a.K;
  const int nonempty = static_cast<int>(std::min<int64_t>(TK, a.E));
  const int shared_tiles = a.n_shared * ((a.T + bm - 1) / bm);
  const int max_tiles = static_cast<int>(TK / bm) + nonempty + shared_tiles;
  const int max_wide = static_cast<int>(TK / kTileM) + nonempty + a.n_shared * ((a.T + kTileM - 1) / kTileM);
  BatchArgs p{};
  // The rule above knows the average and the prior, not the routing: tokens that all choose the same
  // few experts make groups of many row tiles, and every one is another pass over its expert's weights.
  // So the counts decide on the device: with more than skew / 8 row tiles for each 256-row one, the
  // many-token path's GEMMs, launched beside these, do the work and these leave (batch_skewed).
  // Mixtral-shaped, plain routing, every token to the same two experts, many-token path before its tail
  // pieces / 64- or 128-row tiles / this way: 144 tokens (3 tiles for 1) 206 / 266 / 196 us, 208 (2 for
  // 1) 216 / 272 / 217, 400 (4 for 2) 326 / 450 / 313; DeepSeek-shaped, to twelve experts, 333 tokens (5
  // for 2) 148 / 129 / 108, 900 193 / 225 / 183. The launches that leave cost a layer about 4 us (333
  // tokens 247 -> 251). Not made up to 128 tokens, where a group is at most two tiles of 64 rows (120
  // tokens to the same two experts 217 / 220).
  p.skew = bm == 64 ? 15 : pool >= 32 ? 11 : 9;
  const bool may_skew = a.T > 128;
  if (!may_skew) p.skew = 1 << 16;
  p.row_tok = pb.row_tok;
  p.offsets = pb.offsets;
  p.tile_off = pb.tile_off;
  p.wide_off = pb.wide_off;
  p.part = part;
  p.cu_xcd = device_cus_per_xcd();
  p.G = a.E + a.n_shared; p.E = a.E; p.F = a.F;
  p.rows = a.T * (a.K + a.n_shared);

  p.a = static_cast<const uint16_t*>(a.x);
  p.w = static_cast<const uint16_t*>(a.w_gate_up);
  p.ws = static_cast<const uint16_t*>(a.ws_gate_up);
  p.out = H;
  p.N = a.F; p.K = a.d; p.a_rows = a.T;
  p.n_tiles = a.F / (kW / 2);
  p.split = 1;
  hipError_t err;
  if (lora) {
    err = launch_lora_prepare(*lora, a, pb, bm, max_tiles, stream);
    if (err != hipSuccess) return err;
    p.lora_u = lora->u;
    p.lora_b = lora->bp_gate_up;
  }
  err = launch<0>(bm, a.packed, max_tiles * p.n_tiles, p, stream);
  if (err != hipSuccess) return err;
  if (may_skew) {
    err = launch_grouped_skewed(0, a, pb, max_wide, p.skew, H, O, part, lora, stream);
    if (err != hipSuccess) return err;
  }
  record_mark(marks, 0, stream);
  if (lora) {
    err = launch_lora_hidden(*lora, a, pb, bm, max_tiles, H, stream);
    if (err != hipSuccess) return err;
    p.lora_u = lora->v;
    p.lora_b = lora->bp_down;
  }

  p.a = H;
  p.w = static_cast<const uint16_t*>(a.w_down);
  p.ws = static_cast<const uint16_t*>(a.ws_down);
  p.out = O;
  p.N = a.d; p.K = a.F; p.a_rows = p.rows;
  p.n_tiles = (a.d + kW - 1) / kW;
  // One workgroup per slice of the likely number of tiles (fewer experts chosen, in more slices: a
  // workgroup takes several in turn).
  const bool sliced = tail_can_split(1, a.F / kCK);
  const int wide_tiles = (a.d + kTileN - 1) / kTileN;
  if (sliced) {
    const int active = static_cast<int>(std::min<int64_t>(pool, TK));
    const int mt = static_cast<int>(std::max<int64_t>(active, TK / kTileM)) + a.n_shared * ((a.T + kTileM - 1) / kTileM);
    p.split = xcd_share(0, mt * wide_tiles, p.cu_xcd, a.F / kCK, true).s;
  }
  err = launch<1>(bm, a.packed, max_tiles * p.n_tiles * p.split, p, stream);
  if (err != hipSuccess) return err;
  if (may_skew) {
    err = launch_grouped_skewed(1, a, pb, max_wide, p.skew, H, O, part, lora, stream);
    if (err != hipSuccess) return err;
  }
  if (sliced) {
    const int tails = static_cast<int>(std::min<int64_t>((static_cast<int64_t>(max_wide) * wide_tiles + 7) / 8, kTailSlotsPerXcd));
    const int parts = (std::min(a.T, kTileM) + kFixRows - 1) / kFixRows;   // a group holds at most T rows
    hipLaunchKernelGGL(batch_fixup_kernel, dim3(8 * tails * parts), dim3(kThreads), 0, stream, p, parts);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  record_mark(marks, 1, stream);
  err = launch_combine(a, pb, O, true, 1, y, stream);
  record_mark(marks, 2, stream);
  return err;
}

}  // namespace maskmoe
