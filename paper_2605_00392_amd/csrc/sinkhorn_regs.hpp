// The work lists of the Sinkhorn kernels, and the launch of the images that a workgroup or less holds in registers.
#pragma once
#include "common.hpp"
#include "sinkhorn_grid.hpp"
#include "sinkhorn_quad.hpp"
#include "sinkhorn_team.hpp"
#include "sinkhorn_wave.hpp"
#include "splice.hpp"
#include "stage1.hpp"

namespace rtp {

constexpr int kRegsThreads = 64 * kSinkhornBlockWaves;   // of a workgroup of k_sinkhorn_regs

// The list that an image is on: its variant's, but all images of one wave share kVariantA's.  (A
// workgroup's two-wave images meet a barrier an iteration, at which they wait for every wave of it that has not ended: beside
// images of one wave, which meet none, they would not start before those have ended.  40 of 100 x 15 beside 40 of
// 300 x 15, 2500 iterations: 1.11 and 1.66 ms alone, 2.74 together in the same workgroups.)
// Its entry there says which of the two shapes it takes.
constexpr int kListSmallFlag = 1 << 30;
__device__ __forceinline__ int sinkhorn_list(int m, int r, int mode) {
  return WaveSmallShape::fits(m, r) ? kVariantA : sinkhorn_variant(m, r, mode);
}

// Work lists for the register-resident kernels: `work` holds kWorkLists counts
// (one per shape, indexed by variant id) followed by as many lists of B image
// indices each.  One workgroup; list order follows image order.
// `strip`: the strip kernels' words (null: the call does not launch any).
constexpr int kClassifyLdsBytes = (kWorkLists + kStripShapes + 1) * 256 * 4;   // LDS classify_images works in
__device__ __forceinline__ void classify_images(const int32_t* __restrict__ offsets,
                                                const int32_t* __restrict__ keep, int B,
                                                int32_t* __restrict__ work, int32_t* __restrict__ strip, int mode,
                                                void* lds) {
  constexpr int NV = kWorkLists, NM = NV + kStripShapes, NS = NM + 1;   // (the strip kernels' behind the lists, then the work
                                                                        // of kMergeMidPays, which a thread's share stops at)
  int (*cnt)[256] = static_cast<int (*)[256]>(lds);   // [NS][256]
  const int tid = threadIdx.x;
  const int span = (B + 255) / 256;
  const int b0 = min(B, tid * span), b1 = min(B, b0 + span);
  int c[NS];
#pragma unroll
  for (int v = 0; v < NS; ++v) c[v] = 0;
  __shared__ unsigned long long sweep_cells;      // entries of the sweep kernels' matrices, padding included
  __shared__ int strip_tops[kStripShapes];        // workgroups of the strip image that takes most of them
  if (tid == 0) sweep_cells = 0;
  if (tid < kStripShapes) strip_tops[tid] = 0;
  __syncthreads();
  unsigned long long cells = 0;
  for (int b = b0; b < b1; ++b) {
    const int n = offsets[b + 1] - offsets[b];
    const int m = min(max(keep[b], 0), max(n, 0));
    const int v = sinkhorn_list(m, n - m, mode);
    if (n > 0 && v < kGeneralVariant) {
#pragma unroll
      for (int u = 0; u < NV; ++u) c[u] += (u == v);
    }
    if (n > 0 && v == kVariantStrip) {
      const int shape = strip_shape(n - m, mode);
#pragma unroll
      for (int u = 0; u < kStripShapes; ++u) c[NV + u] += u + 1 == shape;
      atomicMax(&strip_tops[shape - 1], strip_groups(shape, m, mode));
    }
    if (n > 0 && v == kVariantSweep) cells += static_cast<unsigned long long>(m) * k32_pitch(n - m);
    if (n > 0 && n - m > kTiledMinPruned) c[kListTiled] += 1;
    if (n > 0 && merge_is_mid(n - m)) c[kListMid] += 1;
    if (n - m > kMergeMidMin) c[NM] = min(c[NM] + min(n * (n - m), kMergeMidPays), kMergeMidPays);
  }
#pragma unroll
  for (int v = 0; v < NS; ++v) cnt[v][tid] = c[v];
  if (cells) atomicAdd(&sweep_cells, cells);
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    int add[NS];
#pragma unroll
    for (int v = 0; v < NS; ++v) add[v] = tid >= o ? cnt[v][tid - o] : 0;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NS; ++v) cnt[v][tid] += add[v];
    __syncthreads();
  }
  int at[NS];
#pragma unroll
  for (int v = 0; v < NS; ++v) at[v] = cnt[v][tid] - c[v];
#pragma unroll
  for (int u = 1; u < kStripShapes; ++u)
#pragma unroll
    for (int w = 0; w < u; ++w) at[NV + u] += cnt[NV + w][255];   // (one list, shape after shape)
  for (int b = b0; b < b1; ++b) {
    const int n = offsets[b + 1] - offsets[b];
    const int m = min(max(keep[b], 0), max(n, 0));
    const int v = sinkhorn_list(m, n - m, mode);
    if (n > 0 && v < kGeneralVariant) {
#pragma unroll
      for (int u = 0; u < NV; ++u)
        if (u == v) work[NV + u * B + at[u]++] = u == kVariantA && !WaveShape::fits(m, n - m) ? b | kListSmallFlag : b;
    }
    if (strip && n > 0 && v == kVariantStrip) {
      const int shape = strip_shape(n - m, mode);
#pragma unroll
      for (int u = 0; u < kStripShapes; ++u)
        if (u + 1 == shape) strip[kStripList + at[NV + u]++] = b;
    }
    if (n > 0 && n - m > kTiledMinPruned) work[NV + kListTiled * B + at[kListTiled]++] = b;
    if (n > 0 && merge_is_mid(n - m)) work[NV + kListMid * B + at[kListMid]++] = b;
  }
  if (tid == 255) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      work[v] = cnt[v][255] | (v == kListMid && cnt[NM][255] >= kMergeMidPays ? kMergeMidPaysFlag : 0);
  }
  if (strip && tid < kStripShapes) {
    int32_t* words = strip + tid * kStripShapeWords;
    int first = 0;
    for (int w = 0; w < tid; ++w) first += cnt[NV + w][255];
    words[kStripCount] = cnt[NV + tid][255];
    words[kStripTop] = strip_tops[tid];
    words[kStripFirst] = first;
    for (int e = kStripCounters; e < kStripShapeWords; ++e) words[e] = 0;
  }
  // the cluster kernel's arrival counters and give-up word start at zero
  if (tid < kWorkStreamWord) work[NV * (1 + B) + tid] = 0;
  if (tid == kWorkStreamWord) {
    // (the matrices are fp32 when the range allows and the sweep kernels run, else fp64)
    const double bytes = static_cast<double>(sweep_cells) * (((mode & kModeF32) && (mode & kModeSweep)) ? 4.0 : 8.0);
    const double over = bytes > static_cast<double>(kSweepResidentBytes)
                            ? 1.0 - static_cast<double>(kSweepResidentBytes) / bytes : 0.0;
    work[NV * (1 + B) + kWorkStreamWord] = static_cast<int>(ceil(16.0 * over));
  }
}

// The lists for the merge alone (staged calls), after a check of the ragged layout.
__global__ __launch_bounds__(256) void k_classify(const int32_t* __restrict__ offsets,
                                                  const int32_t* __restrict__ keep, int B, long long total_tokens,
                                                  int max_tokens, int32_t* __restrict__ work, int32_t* __restrict__ status) {
  if (validate_offsets(offsets, B, total_tokens, max_tokens, status)) return;
  __shared__ __align__(16) unsigned char lds[kClassifyLdsBytes];
  classify_images(offsets, keep, B, work, nullptr, 0, lds);
}

// The two- and one-wave images, the shortest-running roles: workgroup `blk` of theirs.  `others`: how
// many workgroups the launch's other roles have.
// Two-wave images: four per workgroup, one-wave images: eight - or, when the whole launch then still has
// no more workgroups than the chip has CUs (a workgroup of these kernels fills a
// CU's registers, so a surplus one waits for a CU to come free), two and four, on the
// first four waves, so that each wave has a SIMD to itself: a wave alone issues an instruction in 5.2
// clocks, one of two in 9.  Two-wave iterations 1.3 -> 0.7 us.  The two-wave images, which take longer, come
// first.  Waves without an image end at once; a wave that has ended no longer counts at the workgroup's barriers.
__device__ __forceinline__ void sinkhorn_short_block(const SinkhornArgs& A, const int32_t* __restrict__ work, int B,
                                                     int cus, int others, int blk) {
  constexpr int NV = kWorkLists;
  constexpr int kWavesPerBlock = kRegsThreads / 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nA = work[kVariantA];
  const int nP = work[kVariantPair];
  const bool alone = others + (nP + 1) / 2 + (nA + 3) / 4 <= cus;
  const int per_block = alone || others + (nP + 1) / 2 + (nA + kWavesPerBlock - 1) / kWavesPerBlock <= cus
                            ? 2 : kWavesPerBlock / PairShape::kWaves;
  const int ones = alone ? 4 : kWavesPerBlock;
  int cnt = (nP + per_block - 1) / per_block;
  if (blk < cnt) {
    const int slot = wave / PairShape::kWaves, idx = blk * per_block + slot;
    if (slot >= per_block || idx >= nP) return;
    const int img = __builtin_amdgcn_readfirstlane(work[NV + kVariantPair * B + idx]);
    sinkhorn_waves_image<PairShape>(A, img, slot, wave % PairShape::kWaves, lane);
    return;
  }
  blk -= cnt;
  // one-wave images: the shortest-running role, handed out last
  cnt = (nA + ones - 1) / ones;
  if (blk < cnt) {
    const int idx = blk * ones + wave;
    if (wave >= ones || idx >= nA) return;
    const int entry = __builtin_amdgcn_readfirstlane(work[NV + kVariantA * B + idx]);
    if (entry & kListSmallFlag) sinkhorn_waves_image<WaveSmallShape>(A, entry & (kListSmallFlag - 1), wave, 0, lane);
    else sinkhorn_waves_image<WaveShape>(A, entry, wave, 0, lane);
  }
}

// All register-resident Sinkhorn work of a batch in one launch.  Workgroups are
// handed out longest-running role first: the wide teams, team C, 64, 48 and 32 columns
// (sinkhorn_grid.hpp), two-wave (two or four images per workgroup), one-wave (eight
// images per workgroup).  `cus`: compute units of the device.
// `c32`: list kVariantC32 is this launch's too.  Workgroups from B on: X.
__global__ __launch_bounds__(kRegsThreads) void k_sinkhorn_regs(SinkhornArgs A,
                                                               const int32_t* __restrict__ work, int B, int cus, int c32,
                                                               SpliceText X, const int32_t* __restrict__ status) {
  if (status[0]) return;
  if (static_cast<int>(blockIdx.x) >= B) {
    splice_text(X, blockIdx.x - B);
    return;
  }
  constexpr int NV = kWorkLists;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int blk = blockIdx.x;
  int cnt = work[kVariantWideC];
  if (blk < cnt) { sinkhorn_team_image<TeamWideC, float>(A, work[NV + kVariantWideC * B + blk], wave, lane); return; }
  blk -= cnt;
  cnt = work[kVariantWideB];
  if (blk < cnt) { sinkhorn_team_image<TeamWideB, float>(A, work[NV + kVariantWideB * B + blk], wave, lane); return; }
  blk -= cnt;
  cnt = work[kVariantWideA];
  if (blk < cnt) { sinkhorn_team_image<TeamWideA, float>(A, work[NV + kVariantWideA * B + blk], wave, lane); return; }
  blk -= cnt;
  cnt = work[kVariantC];
  if (blk < cnt) { sinkhorn_team_image<TeamC>(A, work[NV + kVariantC * B + blk], wave, lane); return; }
  blk -= cnt;
  __shared__ __align__(16) GridLds<8> lds;
  static_assert(sizeof(QuadLds<4>) <= sizeof(lds), "an image of list kVariantC32 works in it");
  const int of_c32 = c32 ? work[kVariantC32] : 0;
  if (blk < of_c32) { sinkhorn_c32_image<8>(A, work[NV + kVariantC32 * B + blk], &lds); return; }
  blk -= of_c32;
  cnt = work[kVariantGrid64];
  if (blk < cnt) { sinkhorn_grid_image<GridShape<8, 8, double>>(A, work[NV + kVariantGrid64 * B + blk], lds); return; }
  blk -= cnt;
  cnt = work[kVariantGrid48];
  if (blk < cnt) { sinkhorn_grid_image<GridShape<8, 6, double>>(A, work[NV + kVariantGrid48 * B + blk], lds); return; }
  blk -= cnt;
  cnt = work[kVariantGrid32];
  if (blk < cnt) { sinkhorn_grid_image<GridShape<8, 4, double>>(A, work[NV + kVariantGrid32 * B + blk], lds); return; }
  blk -= cnt;
  sinkhorn_short_block(A, work, B, cus,
                       work[kVariantWideA] + work[kVariantWideB] + work[kVariantWideC] + work[kVariantC] + of_c32 +
                           work[kVariantGrid64] + work[kVariantGrid48] + work[kVariantGrid32],
                       blk);
}

// The images of one workgroup or less in a batch with tall ones, the longest-running role first:
// workgroup `blk` of that part of k_sinkhorn_large's launch (sinkhorn_cluster.hpp).  The tall
// shapes (more than 512 rows), then, when `all` is set, the shorter images, which are then all of
// k_sinkhorn_regs's 32-column, two-wave and one-wave shapes.
__device__ __forceinline__ void sinkhorn_tall_block(const SinkhornArgs& A, const int32_t* __restrict__ work, int B,
                                                    int cus, int blk, bool all) {
  constexpr int NV = kWorkLists;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int cnt = work[kVariantTeamTall];
  if (blk < cnt) {
    const int img = work[NV + kVariantTeamTall * B + blk];
    const int n_img = A.offsets[img + 1] - A.offsets[img];
    const int r_img = n_img - min(max(A.keep[img], 0), max(n_img, 0));
    __shared__ __align__(16) unsigned char lds[sizeof(GridLds<8>) > sizeof(QuadLds<8>) ? sizeof(GridLds<8>) : sizeof(QuadLds<8>)];
    if (r_img + 1 <= GridTallShape::kMaxCols) sinkhorn_grid_tall_image(A, img, *reinterpret_cast<GridLds<8>*>(lds));
    else if (r_img <= QuadTall32::kMaxR) sinkhorn_quad_image<QuadTall32>(A, img, *reinterpret_cast<QuadLds<8>*>(lds));
    else if (r_img <= QuadTall48::kMaxR) sinkhorn_quad_image<QuadTall48>(A, img, *reinterpret_cast<QuadLds<8>*>(lds));
    else sinkhorn_team_image<TeamTall, float>(A, img, wave, lane);
    return;
  }
  blk -= cnt;
  cnt = work[kVariantTall];
  if (blk < cnt) { sinkhorn_waves_image<TallShape>(A, work[NV + kVariantTall * B + blk], 0, wave, lane); return; }
  if (!all) return;
  blk -= cnt;
  cnt = work[kVariantGrid32];
  if (blk < cnt) {
    __shared__ __align__(16) GridLds<8> lds;
    sinkhorn_grid_image<GridShape<8, 4, double>>(A, work[NV + kVariantGrid32 * B + blk], lds);
    return;
  }
  sinkhorn_short_block(A, work, B, cus, work[kVariantTeamTall] + work[kVariantTall] + cnt, blk - cnt);
}

}  // namespace rtp
