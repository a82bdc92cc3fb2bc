// Merge and compaction (Eq. 6) for images with many pruned tokens
// (R > kTiledMinPruned), where out = T_kept + alpha P T_prop is a real GEMM
// (M x R times R x D) and belongs on the matrix cores.
//
// The plan is fp32 and must not lose precision to bf16 (one rounding would put
// 2e-3 alpha |T| on every merged feature), so every entry is split on the fly
// into two bf16 numbers, P = hi + lo with |P - hi - lo| <= 2^-18 |P|, and each
// product is two v_mfma_f32_16x16x32_bf16, accumulated in fp32 like the vector
// kernel's sum.  The pruned token rows are bf16 already; the matrix instruction
// wants eight consecutive pruned rows of one feature per lane: they lie in LDS as
// they lie in memory and are turned by its transposing reads.
//
// Workgroup = 4 waves as 2 x 2 on a tile of 128 kept rows x 256 features (128 in small
// batches, which then have tiles for twice as many workgroups, and at widths of which the last tile would leave
// much unused), 32
// pruned rows per step, LDS double-buffered, two workgroups per compute unit; a wave owns 64 rows x half of the features.  P's LDS
// rows are 64 bytes of payload on a pitch of 80.  The finished tile
// goes through LDS once more so that the kept rows are read and the merged rows
// written 16 bytes per lane.
//
// What bounds it: 16 pages of 4512 tokens take 0.552 ms, 357 useful TFLOP/s and twice that executed (the matrix
// cores are at work 32 % of the time, counted; LDS conflicts 39 % of its cycles, waits for it 1.5 % of the waves'); a step's plan entries (16 four-byte loads a thread, their rows being 4-byte aligned) and
// their split are paid once per 256 features.  Before, with 128 features and the pruned rows turned
// by 4-byte LDS writes on their way from registers: 0.847 ms (0.577 with the change, before an image's tiles were on one
// XCD); 32 pages of 2137 tokens 0.422 -> 0.305 -> 0.287, 64 of 1083 0.274 -> 0.202 -> 0.180.  One page of 4512 tokens: 0.118 with 256 features a tile, 0.100 with 128 (0.104 before).
#pragma once
#include "common.hpp"
#include "scores_mfma.hpp"
#include "scores_tiled.hpp"
#include "sinkhorn_team.hpp"

namespace rtp {

constexpr int kMergeTileRows = 128;    // kept rows per workgroup tile
constexpr int kMergeTileCols = 256;    // features per workgroup tile (a width of 128 (2 k + 1) leaves half of the last)
constexpr int kMergeThinCols = 128;    // of small batches
constexpr int kMergeTileStep = 32;     // pruned rows per step
constexpr int kMergeTilePitch = 80;    // LDS bytes per staged row of P (32 bf16 + padding)
constexpr int kMergeTiledThreads = 256;
constexpr int kMergeOperandBytes = kMergeTileRows * kMergeTilePitch;      // P hi or P lo of a step
// merge_tile's LDS buffer: its staging tiles (P hi, P lo, pruned rows, twice); the output tile fits too
constexpr int merge_tiled_lds(int cols) { return 2 * (2 * kMergeOperandBytes + kMergeTileStep * cols * 2); }
constexpr int kMergeTiledLdsBytes = merge_tiled_lds(kMergeTileCols);

// What both launch forms of the kernel pass on.
struct MergeTiledArgs {
  const bf16_t* tokens;
  const int32_t* offsets;
  int D;
  const int32_t* sel_idx;
  const int32_t* keep;
  const int32_t* out_offsets;
  const float* plan;
  const long long* plan_offsets;
  float alpha;
  int max_tokens, tiles_d;
  bf16_t* out;
  int xcd_images;   // tile_of_grid (the grid form)
};

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
// A transposing read: lanes 16 g .. 16 g + 15 each read four consecutive values of a 4 x 16 block (lane i: row i / 4,
// columns 4 (i % 4) .. + 3); lane n of them gets column n, the four rows in order.
__device__ __forceinline__ s16x4_t read_turned(const unsigned char* at) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(const_cast<unsigned char*>(at)));
}

// Tile `tile` (kept-row tile major, feature tile minor) of image b.
template <int COLS>
__device__ __forceinline__ void merge_tile(const MergeTiledArgs& A, int b, int tile, unsigned char* lds) {
  const bf16_t* __restrict__ tokens = A.tokens;
  const int32_t* __restrict__ offsets = A.offsets;
  const int D = A.D;
  const int32_t* __restrict__ sel_idx = A.sel_idx;
  const int32_t* __restrict__ out_offsets = A.out_offsets;
  const float* __restrict__ plan = A.plan;
  const long long* __restrict__ plan_offsets = A.plan_offsets;
  const float alpha = A.alpha;
  const int max_tokens = A.max_tokens, tiles_d = A.tiles_d;
  bf16_t* __restrict__ out = A.out;
  const int lo = offsets[b];
  const int n = offsets[b + 1] - lo;
  if (lo < 0 || n <= 0 || n > max_tokens) return;
  const int m = min(max(A.keep[b], 0), n), r = n - m;
  if (r <= kTiledMinPruned) return;                  // k_merge_lds
  const int ti = tile / tiles_d, td = tile - ti * tiles_d;
  const int i0 = ti * kMergeTileRows, d0 = td * COLS;
  if (i0 >= m) return;
  const int32_t* sel = sel_idx + lo;
  const float* __restrict__ P = plan + plan_offsets[b];
  const size_t obase = static_cast<size_t>(out_offsets[b]);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;

  constexpr int kOperand = kMergeOperandBytes;
  constexpr int kRowBytes = 2 * COLS, kBuffer = 2 * kOperand + kMergeTileStep * kRowBytes;   // [P hi, P lo, T_prop]
  constexpr int kOutPitch = COLS + 4;                                 // floats per row of the output tile, half of which:
  static_assert(merge_tiled_lds(COLS) == 2 * kBuffer && 2 * kBuffer >= 64 * kOutPitch * 4, "the caller's LDS buffer");
  constexpr int kUnits = COLS / 32;                                   // matrix tiles across a wave's half of the features
  constexpr int kPieces = COLS / 8, kReqRows = 64 / kPieces, kReqs = 8 / kReqRows;   // 16-byte pieces of a row; a request's rows; a wave's requests
  const int features = min(D - d0, COLS);                             // 256 or 128

  // staging of P: thread t takes entries 4 (t % 8) .. + 3 of the step for rows t / 8 + 32 q
  const int pj = 4 * (tid & 7), prow = tid >> 3;
  const float* pptr[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) pptr[q] = P + static_cast<long long>(min(i0 + prow + 32 * q, m - 1)) * r;
  // staging of T_prop: request q of a wave brings the step's rows 8 wave + kReqRows q and on, a row being kPieces pieces
  // of 16 bytes that go to slots of blocks of two: block ^ (row % 4 + 4 (row / 8)), as far as there are blocks.  A
  // transposing read's 16 rows of one block then lie in 16 (8) different blocks, all banks twice; in place
  // they would share one.
  const int trow = 8 * wave + lane / kPieces;
  auto block_of = [](int row) { return ((row & 3) | ((row >> 3 & 3) << 2)) & (COLS / 16 - 1); };
  const bf16_t* tbase = tokens + static_cast<size_t>(lo) * D + d0;
  int trows[kReqs];                                    // of the step fetched next
  auto find = [&](int j0) {
#pragma unroll
    for (int q = 0; q < kReqs; ++q) trows[q] = sel[m + min(j0 + trow + kReqRows * q, r - 1)];
  };
  const uint32_t lds_at = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)lds)) + 2 * kOperand);
  float pv[4][4];
  auto fetch = [&](int buf, int j0) {
#pragma unroll
    for (int q = 0; q < kReqs; ++q) {
      const int piece = (lane & 1) + 2 * ((lane % kPieces >> 1) ^ block_of(trow + kReqRows * q));
      load_to_lds_16(tbase + static_cast<size_t>(clamp_index(trows[q], n)) * D + min(8 * piece, features - 8),
                     lds_at + buf * kBuffer + (8 * wave + kReqRows * q) * kRowBytes);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[q][e] = pptr[q][min(j0 + pj + e, r - 1)];
  };
  auto stage = [&](int buf, int j0) {
    unsigned char* base = lds + buf * kBuffer;
    // only the last step can reach past the last pruned row: there, what lies past it is zero
    if (j0 + kMergeTileStep > r) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (j0 + pj + e >= r) pv[q][e] = 0.f;
#pragma unroll
      for (int q = 0; q < kReqs; ++q)
        if (j0 + trow + kReqRows * q >= r)
          *reinterpret_cast<uint4*>(base + 2 * kOperand + (8 * wave + kReqRows * q) * kRowBytes + 16 * lane) = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint2 h2, l2;
      h2.x = pack_bf16x2(pv[q][0], pv[q][1]);
      h2.y = pack_bf16x2(pv[q][2], pv[q][3]);
      l2.x = pack_bf16x2(pv[q][0] - __uint_as_float(h2.x << 16), pv[q][1] - __uint_as_float(h2.x & 0xffff0000u));
      l2.y = pack_bf16x2(pv[q][2] - __uint_as_float(h2.y << 16), pv[q][3] - __uint_as_float(h2.y & 0xffff0000u));
      const int off = (prow + 32 * q) * kMergeTilePitch + 2 * pj;
      *reinterpret_cast<uint2*>(base + off) = h2;
      *reinterpret_cast<uint2*>(base + kOperand + off) = l2;
    }
  };

  floatx4_t acc[4][kUnits];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int u = 0; u < kUnits; ++u) acc[t][u] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  // fragments.  P: lane l reads the 16 bytes (eight consecutive pruned rows 8 (l / 16) .. + 7) of row l % 16.
  // T_prop: read h of block u reads the four rows 8 g + 4 h .. + 3 of the 16 features for lanes 16 g .. 16 g + 15
  // (lane: row (l % 16) / 4, features 4 (l % 4) .. + 3) and hands lane l feature l % 16 of all four.
  const int frag_off = (lane & 15) * kMergeTilePitch + 16 * (lane >> 4);
  const int krow = 8 * (lane >> 4) + (lane >> 2 & 3);                  // of read 0
  const int tr_row = 2 * kOperand + krow * kRowBytes + 8 * (lane & 3), tr_block = block_of(krow);
  const bool mine = COLS / 2 * wn < features;                             // (the other half of the last tile does not exist)
  const int steps = (r + kMergeTileStep - 1) / kMergeTileStep;
  find(0);
  fetch(0, 0);
  find(kMergeTileStep);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  stage(0, 0);
  __syncthreads();
  for (int s = 0; s < steps; ++s) {
    const int buf = s & 1;
    if (s + 1 < steps) {
      fetch(buf ^ 1, (s + 1) * kMergeTileStep);
      find((s + 2) * kMergeTileStep);
    }
    const unsigned char* base = lds + buf * kBuffer;
    if (mine) {
      uint4 fh[4], fl[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        fh[t] = *reinterpret_cast<const uint4*>(base + (64 * wm + 16 * t) * kMergeTilePitch + frag_off);
        fl[t] = *reinterpret_cast<const uint4*>(base + kOperand + (64 * wm + 16 * t) * kMergeTilePitch + frag_off);
      }
#pragma unroll
      for (int u = 0; u < kUnits; ++u) {
        const unsigned char* at = base + tr_row + 32 * ((kUnits * wn + u) ^ tr_block);
        const s16x4_t b0 = read_turned(at), b1 = read_turned(at + 4 * kRowBytes);
        const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, s16x8_t{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]});
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fh[t]), fb, acc[t][u], 0, 0, 0);
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fl[t]), fb, acc[t][u], 0, 0, 0);
        }
      }
    }
    if (s + 1 < steps) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      stage(buf ^ 1, (s + 1) * kMergeTileStep);
    }
    __syncthreads();
  }

  // accumulator element v of lane l is (kept row 4 (l / 16) + v, feature l % 16) of its tile.
  // Half of the tile (64 kept rows) at a time: through LDS as fp32, then each
  // thread adds eight features of one kept row and writes them as 16 bytes.
  // The thread's kept rows' pieces of it are requested first (their indices together, then
  // the rows together): two trips to memory instead of sixteen one after the other.
  float* ot = reinterpret_cast<float*>(lds);
  constexpr int kOutRows = kMergeTiledThreads / kPieces, kOutPasses = 64 / kOutRows;
  const int dd = 8 * (tid % kPieces), orow = tid / kPieces;
  const bool there = dd < features;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    int krows[kOutPasses];
#pragma unroll
    for (int k = 0; k < kOutPasses; ++k) krows[k] = sel[min(i0 + 64 * half + orow + kOutRows * k, m - 1)];
    uint4 kept[kOutPasses];
#pragma unroll
    for (int k = 0; k < kOutPasses; ++k)
      kept[k] = *reinterpret_cast<const uint4*>(tokens + static_cast<size_t>(lo + clamp_index(krows[k], n)) * D + d0 + min(dd, features - 8));
    __syncthreads();                                   // the previous use of this LDS is over
    if (wm == half && mine) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < kUnits; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            ot[(16 * t + 4 * (lane >> 4) + v) * kOutPitch + COLS / 2 * wn + 16 * u + (lane & 15)] = acc[t][u][v];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kOutPasses; ++q) {
      const int row = orow + kOutRows * q;              // 0 .. 63
      const int i = i0 + 64 * half + row;
      if (i >= m || !there) continue;
      const uint32_t kw[4] = {kept[q].x, kept[q].y, kept[q].z, kept[q].w};
      const float* src = ot + row * kOutPitch + dd;
      uint32_t ow[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x0 = __uint_as_float(kw[e] << 16), x1 = __uint_as_float(kw[e] & 0xffff0000u);
        ow[e] = pack_bf16x2(fmaf(alpha, src[2 * e], x0), fmaf(alpha, src[2 * e + 1], x1));
      }
      store_stream(out + (obase + i) * D + d0 + dd, make_uint4(ow[0], ow[1], ow[2], ow[3]));
    }
  }
}

// One workgroup per (tile, image): the staged call, and fused calls whose images
// are known to be large.
template <int COLS>
__global__ __launch_bounds__(kMergeTiledThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_merge_tiled(
    MergeTiledArgs A, const int32_t* __restrict__ status) {
  if (status && status[0]) return;
  __shared__ __attribute__((aligned(16))) unsigned char lds[merge_tiled_lds(COLS)];
  int image, tile;
  tile_of_grid(A.xcd_images, image, tile);
  merge_tile<COLS>(A, image, tile, lds);
}

}  // namespace rtp
