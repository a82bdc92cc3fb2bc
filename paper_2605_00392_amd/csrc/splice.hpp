// Sequence splice: the pruned, merged visual tokens go straight into the
// language model's prefill input (the pruning runs before the prefill stage,
// Sec. 4.3) - per image: text embeddings before the image, the kept visual
// tokens, text embeddings after it - with a position id per token.
//
//   text_flags      validates the two text-span offset arrays (the norm pass's first workgroup, with the ragged layout)
//   splice_scan     seq_offsets[b] = sum_{b' < b} (P + M + S), and the row at which
//                   image b's visual tokens start (what the merge kernel writes to; an extra workgroup of the score pass)
//   splice_text     copies the text rows and writes every position id (workgroups of a Sinkhorn launch)
#pragma once
#include "common.hpp"
#include "stage1.hpp"

namespace rtp {

// (of batches without tokens, which have no norm pass)
__global__ __launch_bounds__(256) void k_splice_check(TextSpans t, int B, int32_t* __restrict__ status) {
  const int flags = text_flags(t, B);
  if (flags) atomicOr(status, flags);
}

// Image order, on one workgroup of 256 threads with kSpliceScanLdsBytes of LDS.
constexpr int kSpliceScanLdsBytes = 256 * 8;
__device__ __forceinline__ void splice_scan(const TextSpans& t, const int32_t* __restrict__ keep, int B,
                                            int32_t* __restrict__ seq_offsets, int32_t* __restrict__ visual_start, void* lds) {
  long long* sm = static_cast<long long*>(lds);
  const int tid = threadIdx.x;
  const int span = (B + 255) / 256;
  const int b0 = min(B, tid * span), b1 = min(B, b0 + span);
  long long c = 0;
  for (int b = b0; b < b1; ++b) c += span_len(t.prefix_offsets, b) + keep[b] + span_len(t.suffix_offsets, b);
  sm[tid] = c;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const long long v = tid >= o ? sm[tid - o] : 0;
    __syncthreads();
    sm[tid] += v;
    __syncthreads();
  }
  long long at = sm[tid] - c;
  for (int b = b0; b < b1; ++b) {
    seq_offsets[b] = static_cast<int32_t>(at);
    visual_start[b] = static_cast<int32_t>(at + span_len(t.prefix_offsets, b));
    at += span_len(t.prefix_offsets, b) + keep[b] + span_len(t.suffix_offsets, b);
  }
  if (tid == 255) seq_offsets[B] = static_cast<int32_t>(sm[255]);
}
__global__ __launch_bounds__(256) void k_splice_scan(TextSpans t, const int32_t* __restrict__ keep, int B,
                                                     int32_t* __restrict__ seq_offsets,
                                                     int32_t* __restrict__ visual_start,
                                                     const int32_t* __restrict__ status) {
  if (status[0]) return;
  __shared__ __align__(16) unsigned char lds[kSpliceScanLdsBytes];
  splice_scan(t, keep, B, seq_offsets, visual_start, lds);
}

// Text rows and position ids, by `blocks` workgroups.  They depend on the kept counts and the selection
// only, so they go at the end of a Sinkhorn launch, which is bound by latency and leaves memory, and in smaller batches
// compute units, idle: 128 tiled pages, 24 us less a call than as a launch of their own behind the merge.
// A wave takes its share of the rows of all images' text together, and of all sequences' positions, so it does not matter
// whose they are (dealt image by image, all 20480 rows of 128 pages before the first of them took a call 1071 us; spread
// evenly 64).
struct SpliceText {
  TextSpans t;
  int B;
  const int32_t* offsets;
  const int32_t* keep;
  const int32_t* sel_idx;
  const int32_t* seq_offsets;
  void* seq;
  int32_t* position_ids;       // may be null
  int row_pieces;              // 16-byte pieces of a row (the library's width limits make that exact)
  int mode;
  int blocks;                  // 0: not in this launch
};
constexpr int kSpliceTextThreads = 512;
constexpr int kSpliceTextRows = 64;            // text rows to a workgroup,
constexpr int kSpliceTextPositions = 4096;     // and positions
inline int splice_text_blocks(long long text_rows, long long positions) {
  const long long blocks = (text_rows + kSpliceTextRows - 1) / kSpliceTextRows + (positions + kSpliceTextPositions - 1) / kSpliceTextPositions;
  return static_cast<int>(blocks < 65536 ? blocks : 65536);
}

// The span that position `at` is in, of spans b and later (span i: start[i] .. start[i + 1] - 1; some are empty).
__device__ __forceinline__ int span_of(const int32_t* __restrict__ start, int b, int B, int at) {
  int last = B - 1;
  while (b < last) {
    const int mid = (b + last) >> 1;
    if (start[mid + 1] > at) last = mid;
    else b = mid + 1;
  }
  return b;
}
// Rows k0 .. k1 - 1 of the text before (or after) the images, the same for every lane of the wave.
__device__ __forceinline__ void splice_rows(const SpliceText& X, const void* text, const int32_t* __restrict__ start, bool after,
                                            int k0, int k1) {
  const int lane = threadIdx.x & 63;
  for (int k = k0, b = 0; k < k1;) {
    b = __builtin_amdgcn_readfirstlane(span_of(start, b, X.B, k));
    const int end = min(start[b + 1], k1);
    const size_t to = after ? static_cast<size_t>(X.seq_offsets[b + 1]) - (start[b + 1] - k)
                            : static_cast<size_t>(X.seq_offsets[b]) + (k - start[b]);
    const uint4* src = static_cast<const uint4*>(text) + static_cast<size_t>(k) * X.row_pieces;
    uint4* dst = static_cast<uint4*>(X.seq) + to * X.row_pieces;
    const long long pieces = static_cast<long long>(end - k) * X.row_pieces;
    long long g = lane;
    for (; g + 3 * 64 < pieces; g += 4 * 64) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = src[g + 64 * u];
#pragma unroll
      for (int u = 0; u < 4; ++u) store_stream(dst + g + 64 * u, v[u]);
    }
    for (; g < pieces; g += 64) store_stream(dst + g, src[g]);
    k = end;
  }
}
__device__ __forceinline__ void splice_text(const SpliceText& X, int block) {
  const TextSpans& t = X.t;
  const int waves = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long long share = static_cast<long long>(block) * waves + wave, shares = static_cast<long long>(X.blocks) * waves;
  auto part = [&](long long rows, long long i) { return static_cast<int>(rows * i / shares); };
  splice_rows(X, t.prefix, t.prefix_offsets, false, part(t.prefix_rows, share), part(t.prefix_rows, share + 1));
  splice_rows(X, t.suffix, t.suffix_offsets, true, part(t.suffix_rows, share), part(t.suffix_rows, share + 1));
  if (!X.position_ids) return;
  const int positions = X.seq_offsets[X.B];
  const int k1 = part(positions, share + 1);
  int b = 0, from = 0, end = 0, P = 0, M = 0, n = 0, lo = 0;
  for (int k = part(positions, share) + lane; k < k1; k += 64) {
    if (k >= end) {
      b = span_of(X.seq_offsets, b, X.B, k);
      from = X.seq_offsets[b];
      end = X.seq_offsets[b + 1];
      lo = X.offsets[b];
      n = X.offsets[b + 1] - lo;
      P = span_len(t.prefix_offsets, b);
      M = min(max(X.keep[b], 0), n);
    }
    const int i = k - from;
    X.position_ids[k] = X.mode == 0 || i < P ? i : i < P + M ? P + clamp_index(X.sel_idx[lo + i - P], n) : P + n + (i - P - M);
  }
}
// (of calls whose Sinkhorn launches are others)
__global__ __launch_bounds__(kSpliceTextThreads) void k_splice_text(SpliceText X, const int32_t* __restrict__ status) {
  if (!status[0]) splice_text(X, blockIdx.x);
}

}  // namespace rtp
