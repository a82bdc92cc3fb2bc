// Merge and compaction (Eq. 6) on the matrix cores for images with a middling
// number of pruned tokens (kMergeMidMin < R <= kTiledMinPruned = 64): too many for
// the vector kernel, which is then bound by its multiply-adds (1.3 ms for 1024
// pages with 63 pruned tokens each), too few for the LDS-tiled kernel to repay
// its staging of both operands and of the result.  Here the kept rows and the
// result never touch LDS, and the kernel is a stream over the kept rows again.
//
//   out = T_kept + alpha P T_prop      (kept rows x features)
//
// v_mfma_f32_16x16x32_bf16 contracts 32 pruned rows at a time.  Its second
// operand is a 32 x 16 block of P transposed: a lane's eight consecutive pruned
// rows of one kept row are eight consecutive floats of a plan row; each is split
// into three bf16 numbers, P = hi + mid + lo exactly (eight bits each, the fp32
// entry has 24), so each product is three matrix instructions accumulated in fp32,
// and nothing but the order of its additions tells this kernel from the vector one
// (for finite features: 0 times infinity is not 0).  The first operand is 16 features
// of 32 pruned rows, which lie in LDS as they lie in memory and are turned by its
// transposing reads.  The accumulator holds, per lane, four features of one kept
// row; the rows of two instructions stand for features 8 g + 4 h .. + 3 (g the
// lane's group of 16, h the instruction), so that a lane ends up with eight
// adjacent features: one 16-byte read of T_kept and one 16-byte store.
//
// A wave owns 16 RB kept rows (their blocks of P split once and kept in
// registers) and walks the features 128 at a time, the two stages after the one it
// computes in flight: the kept rows in registers, the pruned rows, which a workgroup's
// four waves share, straight into one of three LDS buffers.
//
// What bounds it: the stream over the rows (1.8 GB per 1024 pages of 400 tokens, 337 kept).  That call took 1455 us with
// one stage ahead, the pruned rows turned by 2-byte LDS writes on their way from registers, and takes 1414 (this kernel
// 472 -> 430 us, 5.0 TB/s counted; 442 with three terms, the matrix cores at work 23 % of the time); with 64-byte
// pieces of 16 rows an access instead of whole lines (merge_mid_swap) 1527 to 1569, with the pieces exchanged for the stores only 1441,
// with plain instead of non-temporal stores 1445.
// With two terms of P (18 bits of it) 1024 pages with 63 pruned tokens took 1286 us a call and take 1294, 32 pages of 256 with
// 40 pruned, of which a wave has a SIMD to itself and waits for the matrix cores, 102 and 105 (the vector kernel: 108).  With the terms' products in turn for
// both halves of the features a register is spilled: 107.
#pragma once
#include "common.hpp"
#include "scores_mfma.hpp"
#include "sinkhorn_team.hpp"
#include "merge_tiled.hpp"

namespace rtp {

static_assert(kTiledMinPruned == 64, "two operand blocks of 32 pruned rows");
constexpr int kMergeMidFeatures = 64;                 // the width is a multiple of this
constexpr int kMergeMidStage = 2 * kMergeMidFeatures; // features per stage (the last may have half)
constexpr int kMergeMidRB = 2;                        // 16-row blocks per wave
constexpr int kMergeMidWaveRows = 16 * kMergeMidRB;
constexpr int kMergeMidBlockRows = 4 * kMergeMidWaveRows;
static_assert(kMergeMidPays == 2048 * kMergeMidBlockRows, "as its comment says");
constexpr int kMergeMidThreads = 256;
constexpr int kMergeMidRowBytes = 2 * kMergeMidStage;
constexpr int kMergeMidBuffer = kTiledMinPruned * kMergeMidRowBytes;   // a stage's pruned rows
constexpr uint32_t kMergeMidBeyond = 0x40000000;      // an offset outside every descriptor
constexpr int kMergeMidStream = 2;                    // a buffer store's cache policy: non-temporal
constexpr int kMergeMidLdsBytes = 3 * kMergeMidBuffer;

// What is loaded in the place of pruned rows past the last (T_prop may hold infinities: 0 times another row's is not 0).
__device__ const uint4 kMergeMidNothing = {0u, 0u, 0u, 0u};

struct MergeMidArgs {
  const bf16_t* tokens;
  const int32_t* offsets;
  int D;
  const int32_t* sel_idx;
  const int32_t* keep;
  const int32_t* out_offsets;
  const float* plan;
  const long long* plan_offsets;
  float alpha;
  int max_tokens;
  bf16_t* out;
};

// A wave's requests but the latest NEWEST are done, its LDS reads are over, and, after the meeting, those of the
// workgroup's other waves.  (Written out: a workgroup-scope fence would wait for every request.  The wavefront-scope
// fences emit nothing.  The scheduling barrier keeps arithmetic on rows requested for a later stage, and with it the wait
// for them, behind that stage's meeting.)
template <int NEWEST>
__device__ __forceinline__ void merge_mid_wait() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NEWEST) : "memory");
}
__device__ __forceinline__ void merge_mid_meet() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_sched_barrier(0);
}

// Between what the matrix instructions want and what memory does: a = the first, b = the second 64 bytes of a lane's row
// of a 128-byte line, on all 16 rows at once, become, on neighbouring lanes c and c + 1 (c even), the first and second
// half of row c (in a) and of row c + 1 (in b), so that an access covers whole lines.  Its own inverse.
__device__ __forceinline__ void merge_mid_swap(bool odd, u32x4_t& a, u32x4_t& b) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t got = __builtin_amdgcn_mov_dpp(odd ? a[e] : b[e], 0xB1, 0xf, 0xf, true);   // lane ^ 1
    if (odd) a[e] = got;
    else b[e] = got;
  }
}

// Rows i0 .. i0 + kMergeMidBlockRows - 1 of image b, which has r <= 32 KB pruned rows of n, m kept.
//
// An LDS row is a pruned row's 256 bytes of the stage, its 64-byte blocks exchanged: block x lies at x ^ (row % 4), so
// the four rows that 16 lanes of a transposing read want at once lie in different banks.
template <int KB>
__device__ __forceinline__ void merge_mid_rows(const MergeMidArgs& A, int b, int lo, int n, int m, int r, int i0,
                                               unsigned char* lds) {
  constexpr int RB = kMergeMidRB, kReqs = 2 * KB;      // a wave's requests for a stage's pruned rows, four rows each
  constexpr int kPieces = 4 * RB;                      // 16-byte pieces of the kept rows a lane reads (and writes) per stage
  const int D = A.D;
  const int stages = (D + kMergeMidStage - 1) / kMergeMidStage;
  const bool half = D % kMergeMidStage != 0;           // the last stage has 64 features
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int iw = i0 + kMergeMidWaveRows * wave;        // the wave's first kept row
  const bool active = iw < m;                          // else the wave only helps to fetch
  const int32_t* sel = A.sel_idx + lo;
  const float* __restrict__ P = A.plan + A.plan_offsets[b];
  const int c = lane & 15, g = lane >> 4;

  const char* tbase = reinterpret_cast<const char*>(A.tokens + static_cast<size_t>(lo) * D);
  char* obase = reinterpret_cast<char*>(A.out + (static_cast<size_t>(A.out_offsets[b]) + i0) * D);
  const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(tbase), 0, n * D * 2, 0x00020000);
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(obase, 0, (m - i0) * D * 2, 0x00020000);
  // byte offsets within the image (at most 8192 rows of 8 KB): kept row iw + 16 rb + c rounded down to even + k, its 16 bytes g of the line's
  // half c % 2 (merge_mid_swap);
  // pruned row 16 q + 4 wave + g, the 16 bytes that go to the lane's place of it (row % 4 = g)
  const bool odd = c & 1;
  uint32_t koff[RB][2], poff[kReqs];
  bool there[kReqs];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      koff[rb][k] = static_cast<uint32_t>(clamp_index(sel[min(iw + 16 * rb + (c & 14) + k, m - 1)], n) * D + 8 * g) * 2u + 64 * (c & 1);
#pragma unroll
  for (int q = 0; q < kReqs; ++q) {
    const int k = 16 * q + 4 * wave + g;
    there[q] = k < r;
    poff[q] = static_cast<uint32_t>(clamp_index(sel[m + min(k, r - 1)], n) * D) * 2u;
  }
  const int piece = c ^ (4 * g);
  // the plan entries of kept row iw + 16 rb + c, pruned rows 32 kb + 8 g .. + 7
  float pv[RB][KB][8];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const float* prow = P + static_cast<long long>(min(iw + 16 * rb + c, m - 1)) * r;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[rb][kb][e] = prow[min(32 * kb + 8 * g + e, r - 1)];
  }

  const uint32_t lds_at = __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)lds)) +
      4 * wave * kMergeMidRowBytes);
  // In a half last stage whatever lies 64 features on is read 64 features back instead (and not used).
  auto request = [&](int s, int buf, u32x4_t (&kept)[RB][4], bool keep) {
    const uint32_t at = static_cast<uint32_t>(s) * kMergeMidRowBytes;
    const bool short_stage = half && s == stages - 1;
    if (keep) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          kept[rb][u] = __builtin_amdgcn_raw_buffer_load_b128(rows, koff[rb][u & 1] + (u >= 2 && !short_stage ? 128 : 0), at, 0);
    }
    const uint32_t pat = at + 16 * (short_stage ? piece & 7 : piece);
#pragma unroll
    for (int q = 0; q < kReqs; ++q) {
      const void* src = there[q] ? static_cast<const void*>(tbase + poff[q] + pat) : static_cast<const void*>(&kMergeMidNothing);
      load_to_lds_16(src, lds_at + buf * kMergeMidBuffer + 16 * q * kMergeMidRowBytes);
    }
  };
  u32x4_t k0[RB][4], k1[RB][4], k2[RB][4];
  merge_mid_wait<0>();
  merge_mid_meet();                                    // the previous tile's last LDS reads are over
  if (!active) {
    request(0, 0, k0, false);
    if (stages > 1) request(1, 1, k1, false);
    for (int s = 0, buf = 0; s < stages; ++s, buf = buf == 2 ? 0 : buf + 1) {
      if (s + 1 < stages) merge_mid_wait<kReqs>();
      else merge_mid_wait<0>();
      merge_mid_meet();
      if (s + 2 < stages) request(s + 2, buf ? buf - 1 : 2, k2, false);
    }
    return;
  }
  // Stores past the last kept row (and past a half last stage) fall outside the descriptor and are dropped.  So every
  // stage of an active wave issues kPieces of them, and as many stand for each of the two stages before the first:
  // the waits below have the same counts from there on.
  auto no_stores = [&]() {
#pragma unroll
    for (int k = 0; k < kPieces; ++k)                  // (to different places: of equal stores the compiler keeps one)
      __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{0u, 0u, 0u, 0u}, rsrc, kMergeMidBeyond + 64 * k, 0, kMergeMidStream);
  };
  request(0, 0, k0, true);
  no_stores();
  request(min(1, stages - 1), 1, k1, true);
  no_stores();

  bf16x8_t phi[RB][KB], pmid[RB][KB], plo[RB][KB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      uint32_t h[4], d[4], l[4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const int k = 32 * kb + 8 * g + e;
        const float v0 = k < r ? pv[rb][kb][e] : 0.f, v1 = k + 1 < r ? pv[rb][kb][e + 1] : 0.f;
        h[e >> 1] = pack_bf16x2(v0, v1);
        const float w0 = v0 - __uint_as_float(h[e >> 1] << 16), w1 = v1 - __uint_as_float(h[e >> 1] & 0xffff0000u);
        d[e >> 1] = pack_bf16x2(w0, w1);
        l[e >> 1] = pack_bf16x2(w0 - __uint_as_float(d[e >> 1] << 16), w1 - __uint_as_float(d[e >> 1] & 0xffff0000u));
      }
      phi[rb][kb] = __builtin_bit_cast(bf16x8_t, make_uint4(h[0], h[1], h[2], h[3]));
      pmid[rb][kb] = __builtin_bit_cast(bf16x8_t, make_uint4(d[0], d[1], d[2], d[3]));
      plo[rb][kb] = __builtin_bit_cast(bf16x8_t, make_uint4(l[0], l[1], l[2], l[3]));
    }

  uint32_t ooff[RB][2];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int k = 0; k < 2; ++k)
      ooff[rb][k] = static_cast<uint32_t>((kMergeMidWaveRows * wave + 16 * rb + (c & 14) + k) * D + 8 * g) * 2u + 64 * (c & 1);
  // transposing reads: lane -> pruned row 8 g + (lane % 16) / 4, features 8 (lane % 4) + 4 h .. + 3 of a block of 32
  const int krow = lane >> 2 & 3;
  const unsigned char* tr_at = lds + (8 * g + krow) * kMergeMidRowBytes + 16 * (lane & 3);

  // Stage s from buffer `buf`, its kept rows in `cur`; with `more` (constant in the long loop: the compiler's own waits
  // for `cur` then count all that was issued after it) stage s + 2 is requested into `nxt`.
  // After the stage's own requests were issued: the stores of stage s - 2, the requests of stage s + 1, the stores of
  // stage s - 1.
  auto step = [&](int s, int buf, bool more, const u32x4_t (&cur)[RB][4], u32x4_t (&nxt)[RB][4]) {
    if (more || s + 1 < stages) merge_mid_wait<3 * kPieces + kReqs>();
    else merge_mid_wait<2 * kPieces>();
    merge_mid_meet();                                  // the stage's pruned rows are in LDS; nobody reads stage s - 1's
    if (more) request(s + 2, buf ? buf - 1 : 2, nxt, true);
    const unsigned char* base = tr_at + buf * kMergeMidBuffer;
    const uint32_t at = static_cast<uint32_t>(s) * kMergeMidRowBytes;
    const bool short_stage = half && s == stages - 1;
#pragma unroll
    for (int pair = 0; pair < 2; ++pair) {             // 64 features
      u32x4_t o[RB][2];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int k = 0; k < 2; ++k) o[rb][k] = cur[rb][2 * pair + k];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) merge_mid_swap(odd, o[rb][0], o[rb][1]);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        bf16x8_t t[2][KB];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            const unsigned char* p = base + 32 * kb * kMergeMidRowBytes + 64 * ((2 * pair + k) ^ krow) + 8 * h;
            const s16x4_t b0 = read_turned(p), b1 = read_turned(p + 4 * kMergeMidRowBytes);
            t[h][kb] = __builtin_bit_cast(bf16x8_t, s16x8_t{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]});
          }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          floatx4_t acc[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            acc[h] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
              acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[h][kb], phi[rb][kb], acc[h], 0, 0, 0);
              acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[h][kb], pmid[rb][kb], acc[h], 0, 0, 0);
              acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t[h][kb], plo[rb][kb], acc[h], 0, 0, 0);
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t w = o[rb][k][e];
            const float x0 = __uint_as_float(w << 16), x1 = __uint_as_float(w & 0xffff0000u);
            const int v = 2 * (e & 1);
            o[rb][k][e] = pack_bf16x2(fmaf(A.alpha, acc[e >> 1][v], x0), fmaf(A.alpha, acc[e >> 1][v + 1], x1));
          }
        }
      }
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        merge_mid_swap(odd, o[rb][0], o[rb][1]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          // The stage's offset goes into the vector register.  With a scalar one the compiler lets the very next
          // instruction write over the stored registers, and its values were what the store wrote.  (Forgotten, it
          // stays there, and the two places of a store stay one store.)
          uint32_t to = pair && short_stage ? kMergeMidBeyond + 1024 * rb + 64 * k : ooff[rb][k] + at;
          forget_origin(to);
          __builtin_amdgcn_raw_buffer_store_b128(o[rb][k], rsrc, to + 128 * pair, 0, kMergeMidStream);
        }
      }
    }
  };
  int s = 0;
  for (; s + 4 < stages; s += 3) {
    step(s, 0, true, k0, k2);
    step(s + 1, 1, true, k1, k0);
    step(s + 2, 2, true, k2, k1);
  }
  // one to four stages are left
  step(s, 0, s + 2 < stages, k0, k2);
  if (s + 1 < stages) step(s + 1, 1, s + 3 < stages, k1, k0);
  if (s + 2 < stages) step(s + 2, 2, false, k2, k1);
  if (s + 3 < stages) step(s + 3, 0, false, k0, k2);
}

__device__ __forceinline__ void merge_mid_tile(const MergeMidArgs& A, int b, int i0, unsigned char* lds) {
  const int lo = A.offsets[b];
  const int n = A.offsets[b + 1] - lo;
  if (lo < 0 || n <= 0 || n > A.max_tokens) return;    // (these are the same for the whole workgroup)
  const int m = min(max(A.keep[b], 0), n), r = n - m;
  if (!merge_is_mid(r) || i0 >= m) return;
  if (r > 32) merge_mid_rows<2>(A, b, lo, n, m, r, i0, lds);
  else merge_mid_rows<1>(A, b, lo, n, m, r, i0, lds);
}

// The tiles of the images on the tiled list, `tile_rows` rows of them to an image.
template <int COLS>
__device__ __forceinline__ void merge_tiled_list(MergeTiledArgs A, int tile_rows, const int32_t* __restrict__ work, int B,
                                                 unsigned char* lds) {
  A.tiles_d = (A.D + COLS - 1) / COLS;
  const int tiles = tile_rows * A.tiles_d;
  const long long items = static_cast<long long>(work[kListTiled]) * tiles;
  for (long long item = blockIdx.x; item < items; item += gridDim.x) {
    __syncthreads();   // the previous tile's last LDS reads
    const int k = static_cast<int>(item / tiles);
    merge_tile<COLS>(A, work[kWorkLists + kListTiled * B + k], static_cast<int>(item - static_cast<long long>(k) * tiles), lds);
  }
}

// The list forms of both matrix-core merge kernels in one launch (the sizes of the
// pruned sets were decided on the device): a fixed number of workgroups, a multiple
// of eight, first walk the tiles of the images on the tiled list (more than 64
// pruned tokens; merge_tiled.hpp), then the row tiles of the images on this file's
// list.  For the latter, workgroups being dealt to the eight XCDs in turn, item q
// runs on XCD q % 8: the tiles of one image are given items of one residue, and
// its pruned rows are fetched into one L2 only.  `tile_rows` / `tiles_m` = 0: that
// role is not wanted.  Fewer than `thin_below` wide tiles in all: narrow ones (merge_thin_below).  Both roles
// use the same LDS buffer.
__global__ __launch_bounds__(kMergeMidThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_merge_lists(
    MergeTiledArgs TA, int tile_rows, int thin_below, MergeMidArgs A, int tiles_m, const int32_t* __restrict__ work, int B, MergeMidRule mid_rule,
    const int32_t* __restrict__ status) {
  if (status[0]) return;
  static_assert(kMergeTiledThreads == kMergeMidThreads, "one workgroup shape for both roles");
  constexpr int kLdsBytes = kMergeTiledLdsBytes > kMergeMidLdsBytes ? kMergeTiledLdsBytes : kMergeMidLdsBytes;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kLdsBytes];
  if (tile_rows > 0) {
    const long long rows = static_cast<long long>(work[kListTiled]) * tile_rows;
    if (rows * ((TA.D + kMergeTileCols - 1) / kMergeTileCols) < thin_below) merge_tiled_list<kMergeThinCols>(TA, tile_rows, work, B, lds);
    else merge_tiled_list<kMergeTileCols>(TA, tile_rows, work, B, lds);
  }
  if (tiles_m > 0 && merge_mid_runs(work[kListMid], mid_rule)) {
    const int count = work[kListMid] & kMergeMidCount;
    const long long items = static_cast<long long>((count + 7) / 8) * 8 * tiles_m;
    for (long long q = blockIdx.x; q < items; q += gridDim.x) {
      const long long s = q >> 3;
      const int k = static_cast<int>(s / tiles_m) * 8 + static_cast<int>(q & 7);
      if (k >= count) continue;
      merge_mid_tile(A, work[kWorkLists + kListMid * B + k], kMergeMidBlockRows * static_cast<int>(s % tiles_m), lds);
    }
  }
}

}  // namespace rtp
