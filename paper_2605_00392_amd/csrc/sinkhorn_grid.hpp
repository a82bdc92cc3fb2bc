// Sinkhorn (Appendix C) for images of up to 511 kept and 63 pruned tokens beyond the one- and two-wave
// shapes: the kernel matrix in fp64 registers, once, a workgroup of eight or four waves per image.
//
// The dustbin row and column are ordinary entries of the augmented kernel ((M+1) x (R+1), kz on the last row
// and column), so neither scaling needs a sum of its own.  A wave is eight column slots (cs: lane bits 0, 1 and 3) x
// eight row slots (rs: bits 2, 4 and 5); a lane holds columns 2 cs, 2 cs + 1, 16 + 2 cs, ... (CPT of them) of the
// rows it owns.  Rows come in batches of four: batch q of row group p (0 to 3) is rows 8 p + rs + 32 (4 q + u),
// u < 4.  Even batches are one part of the column sums, odd ones another ("parts", eight in all: four groups x
// two), whoever holds them:
//   eight waves (GridShape<8, ...>)  a wave per part, up to two batches each: M + 1 <= 512
//   four waves  (GridShape<4, ...>)  both parts of a group, the odd batch first: M + 1 <= 352 (the
//                                    last batch of three rows: registers), two workgroups to a compute unit
// so both add up the same numbers in the same order and give the same bits: eight waves for as many images
// as the chip has compute units, where an iteration's latency decides, four for more, where the
// instructions of all of them do.
//
// Per batch the four rows' sums over the column slots meet in two halving exchanges and an addition, one
// reciprocal serves four rows, and quad permutes hand the four x to the column slots; the entries are used where
// they lie (held as fp32 they cost a conversion each per iteration).  The column sums of a wave's row slots meet
// in halving exchanges as well (swap instructions), after which a lane owns one column: what goes through LDS is 512
// bytes a part, one workgroup barrier an iteration.
//
// What bounds it: a wave alone on its SIMD issues an fp64 instruction every 5.2 clocks, dependent or not, two waves one
// every 4.5 together (with all compute units at work the clock drops, 6.0 at 2.4 GHz); then the exchange.  Column
// sums added up through LDS instead, 4 KB a wave each way, are slower than the instructions they save: of
// 3070 clocks an iteration of eight waves 2066 went there.  Measured, 100 iterations that do not settle, against the
// copy held as fp32 (sinkhorn_quad.hpp) and two fp64 copies, one for each direction: 1024 pages of 400 tokens
// with 63 pruned 510 -> 453 us, 256 such 154 -> 126; calls: one such page 194 -> 120, 32 pages of 256 with 40 pruned
// 137 -> 107.
#pragma once
#include "common.hpp"
#include "sinkhorn_quad.hpp"
#include "sinkhorn_team.hpp"

namespace rtp {

// W waves, CPT columns a lane, entries read from memory as KT (fp32: kKernelRowsF32).
template <int W_, int CPT_, typename KT_>
struct GridShape {
  typedef KT_ KT;
  static constexpr int W = W_, CPT = CPT_, kThreads = 64 * W, kBatches = W == 8 ? 2 : 3;
  static constexpr int kMaxRows = W == 8 ? 512 : 352, kMaxCols = 8 * CPT;       // augmented
  static constexpr int rows_of(int k) { return W == 4 && k == 2 ? 3 : 4; }      // of the k-th batch that a wave takes
  static_assert((W == 8 || W == 4) && CPT % 2 == 0 && CPT <= 8, "eight parts; whole pairs of columns; a lane per column");
};
constexpr int kGridParts = 8;
template <int W>
struct GridLds {
  static constexpr int kPitch = 72;            // doubles
  double sum[2][kGridParts][64];               // the parts' column sums by owner lane, by iteration parity
  double y[W][64];                             // every wave's copy
  double stage[W][8][kPitch];                  // rows of the plan and pairing keys, at the end
  int moved;                                   // 1 + the last iteration in which an x changed
};
typedef double f64x2g_t __attribute__((ext_vector_type(2)));

// a + (the partner's a) on lanes whose bit is clear, b + (the partner's b) on the others.
template <int CTRL>                            // 0xB1: bit 0, 0x4E: bit 1
__device__ __forceinline__ double halve_quad(double a, double b, bool set) {
  const double keep = set ? b : a, send = set ? a : b;
  return keep + dpp_move<CTRL>(send);
}

// The wave's column sums of t, scattered: lane l ends up with that of entry grid_entry<CPT>(l) of its own columns.
template <int CPT>
__device__ __forceinline__ int grid_entry(int lane) {
  const int b5 = lane >> 5, b4 = (lane >> 4) & 1, b2 = (lane >> 2) & 1;
  return CPT == 8 ? 4 * b5 + 2 * b4 + b2 : CPT == 6 ? 3 * b5 + (b2 ? 1 : 2 * b4) : 2 * b5 + b4;
}
template <int CPT>
__device__ __forceinline__ double grid_scatter(const double (&t)[CPT]) {
  static_assert(CPT == 8 || CPT == 6 || CPT == 4, "three shapes");
  double h[CPT / 2];
#pragma unroll
  for (int c = 0; c < CPT / 2; ++c) h[c] = halve32(t[c], t[c + CPT / 2]);
  if constexpr (CPT == 8) return halve4(halve16(h[0], h[2]), halve16(h[1], h[3]));
  else if constexpr (CPT == 6) return halve4(halve16(h[0], h[2]), add_xor_lane<16>(h[1]));
  else return add_xor_lane4(halve16(h[0], h[1]));
}

template <typename S>
__device__ __forceinline__ void sinkhorn_grid_image(const SinkhornArgs& A, int b, GridLds<S::W>& L) {
  constexpr int W = S::W, CPT = S::CPT, kB = S::kBatches;
  typedef typename S::KT KT;
  constexpr bool kNarrow = std::is_same<KT, float>::value;
  const DevParams& p = A.p;
  const int tt = threadIdx.x, tw = __builtin_amdgcn_readfirstlane(tt >> 6), lane = tt & 63;
  const int cs = (lane & 3) + ((lane >> 1) & 4), rs = ((lane >> 4) & 3) + (lane & 4);
  const int lo = __builtin_amdgcn_readfirstlane(A.offsets[b]);
  const int n = __builtin_amdgcn_readfirstlane(A.offsets[b + 1]) - lo;
  if (n <= 0) return;
  const int m = min(max(__builtin_amdgcn_readfirstlane(A.keep[b]), 0), n), r = n - m;
  if (m + 1 > S::kMaxRows || r + 1 > S::kMaxCols) return;    // uniform over the workgroup
  int32_t* __restrict__ pair_out = A.pair_out;
  if (pair_out)
    for (int i = tt; i < m; i += S::kThreads) pair_out[lo + i] = i;
  if (r <= 0 || m <= 0) return;
  const long long po = A.plan_offsets[b];
  if (!plan_fits(po, m, r, A.plan_cap)) return;
  const KT* Kg;
  int pitch;
  if constexpr (kNarrow) { Kg = k32_base(A.kmat, po); pitch = k32_pitch(r); }
  else { Kg = A.kmat + po; pitch = r; }
  const double kz = exp((p.z - p.shift) / p.eps);

  // the batches of this wave, in the order in which it takes them, and the part each belongs to
  const int group = tw & 3, odd = tw >> 2;                   // (four waves: odd = 0)
  auto batch_of = [&](int k) { return W == 8 ? 2 * k + odd : k == 0 ? 1 : 2 * (k - 1); };
  const int row0 = 8 * group + rs;
  auto row_of = [&](int k, int u) { return row0 + 32 * (4 * batch_of(k) + u); };
  auto col_of = [&](int c) { return 2 * cs + 16 * (c >> 1) + (c & 1); };
  const int last = m >> 7;                                   // the batch of the dustbin row: the last one there is

  // (loads from clamped positions, all of a batch in flight together.  Rows past the dustbin hold a single 1 and
  // get a zero marginal, so that their x is an ordinary 0.)
  double K[kB][4][CPT];
#pragma unroll
  for (int k = 0; k < kB; ++k) {
    KT v[4][CPT];
#pragma unroll
    for (int u = 0; u < S::rows_of(k); ++u) {
      const KT* row = Kg + static_cast<long long>(min(row_of(k, u), m - 1)) * pitch;
#pragma unroll
      for (int c = 0; c < CPT; ++c) v[u][c] = row[min(col_of(c), r - 1)];
    }
#pragma unroll
    for (int u = 0; u < S::rows_of(k); ++u)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const int i = row_of(k, u), j = col_of(c);
        K[k][u][c] = i < m && j < r ? static_cast<double>(v[u][c]) : i <= m && j <= r ? kz : i > m && j == 0 ? 1.0 : 0.0;
        forget_origin(K[k][u][c]);
      }
  }

  const double x_init = exp(p.shift / p.eps);                // T = 0 leaves u = 0
  const int u_own = lane & 3;                                // the row of a batch this lane finishes
  const bool bit0 = (lane & 1) != 0, bit1 = (lane & 2) != 0;
  const int own = col_of(grid_entry<CPT>(lane));             // the column this lane finishes
  auto spread = [](double v, double (&x)[4]) {               // the x of a batch's four rows, from the lanes that own them
    x[0] = dpp_move<0x00>(v);
    x[1] = dpp_move<0x55>(v);
    x[2] = dpp_move<0xAA>(v);
    x[3] = dpp_move<0xFF>(v);
  };
  const double b_col = own < r ? 1.0 : static_cast<double>(m);
  const int i_last = row0 + 32 * (4 * last + u_own);
  const double a_last = i_last < m ? 1.0 : i_last == m ? static_cast<double>(r) : 0.0;
  constexpr bool kKeepY = W == 8;                            // (four waves have no registers for it)
  double y[CPT], x_own[kB];
  auto read_y = [&] {
    int at = 2 * cs;
    forget_origin(at);                                       // (anew every time)
#pragma unroll
    for (int c = 0; c < CPT; c += 2) {
      const f64x2g_t v = *static_cast<const f64x2g_t*>(__builtin_assume_aligned(&L.y[tw][at + 8 * c], 16));
      y[c] = v[0];
      y[c + 1] = v[1];
    }
  };
  L.y[tw][own] = own <= r ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < kB; ++k) x_own[k] = row_of(k, 0) + 32 * u_own <= m ? x_init : 0.0;
  if (tt == 0) L.moved = 0;
  // (sums of parts without rows are never written again)
  for (int e = tt; e < 2 * kGridParts * 64; e += S::kThreads) (&L.sum[0][0][0])[e] = 0.0;
  __syncthreads();
  read_y();

  int stop_at = p.iters;
  for (int it = 0; it < stop_at; ++it) {
    bool differs = false;
    double t[CPT];
    auto put = [&](int part) { L.sum[it & 1][part][lane] = grid_scatter<CPT>(t); };
#pragma unroll
    for (int c = 0; c < CPT; ++c) t[c] = 0.0;
#pragma unroll
    for (int k = 0; k < kB; ++k) {
      if (batch_of(k) <= last) {                             // (the same for every lane of the wave)
        double s[4];
        if constexpr (!kKeepY) read_y();
#pragma unroll
        for (int u = 0; u < 4; ++u) s[u] = u < S::rows_of(k) ? K[k][u < S::rows_of(k) ? u : 0][0] * y[0] : 1.0;
#pragma unroll
        for (int c = 1; c < CPT; ++c)
#pragma unroll
          for (int u = 0; u < S::rows_of(k); ++u) s[u] = fma(K[k][u][c], y[c], s[u]);
        double xv = rcp64_tight(add_xor_lane<8>(
            halve_quad<0x4E>(halve_quad<0xB1>(s[0], s[1], bit0), halve_quad<0xB1>(s[2], s[3], bit0), bit1)));
        if (batch_of(k) == last) xv *= a_last;
        differs |= __double_as_longlong(xv) != __double_as_longlong(x_own[k]);
        x_own[k] = xv;
        double x[4];
        spread(xv, x);
#pragma unroll
        for (int u = 0; u < S::rows_of(k); ++u)
#pragma unroll
          for (int c = 0; c < CPT; ++c) t[c] = fma(K[k][u][c], x[u], t[c]);
        if (W == 4 && k == 0) {
          put(4 + group);
#pragma unroll
          for (int c = 0; c < CPT; ++c) t[c] = 0.0;
        }
        if constexpr (W == 4) __builtin_amdgcn_sched_barrier(0);
      }
    }
    put(tw);
    if (differs) L.moved = it + 1;
    __syncthreads();
    const int moved = __builtin_amdgcn_readfirstlane(L.moved);
    const double (*part)[64] = L.sum[it & 1];
    const double total = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) +
                         ((part[4][lane] + part[5][lane]) + (part[6][lane] + part[7][lane]));
    L.y[tw][own] = own <= r ? b_col * rcp64_tight(total) : 0.0;
    wave_lds_fence();
    if constexpr (kKeepY) read_y();
    // (the same in every wave: a later number is of a wave that has gone on, which it has not if nothing moved)
    stop_at = settled_stop(stop_at, it, moved >= it + 1);
  }

  // ---- plan and pairing (row m is the dustbin) ----
  read_y();
  float* P = A.plan_out ? A.plan_out + po : nullptr;
  float bv[CPT];
  int bi[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) { bv[c] = -1.f; bi[c] = 0x7fffffff; }
  float* rows = reinterpret_cast<float*>(&L.stage[tw][0][0]);  // the wave's eight rows of the plan, turned to whole rows
  constexpr int kRowPitch = 2 * GridLds<W>::kPitch;
#pragma unroll
  for (int k = 0; k < kB; ++k) {
    if (batch_of(k) > last) continue;
    double x[4];
    spread(x_own[k], x);
#pragma unroll
    for (int u = 0; u < S::rows_of(k); ++u) {
      int i = row_of(k, u);
      forget_origin(i);
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const float v = static_cast<float>(x[u] * K[k][u][c] * y[c]);
        rows[rs * kRowPitch + col_of(c)] = v;
        if (i <= m && (v > bv[c] || (v == bv[c] && i < bi[c]))) { bv[c] = v; bi[c] = i; }   // (four waves: not in ascending order)
      }
      wave_lds_fence();
      if (P && lane < r) {
#pragma unroll
        for (int l = 0; l < 8; ++l) {
          const int il = i - rs + l;
          if (il < m) P[il * r + lane] = rows[l * kRowPitch + lane];
        }
      }
      wave_lds_fence();
    }
  }
  if (!pair_out) return;
  // a column's best as a key (value bits, then the lower row): plan entries are >= 0, so their bit
  // patterns order like their values; "no row" (-1) is below all
  long long (*keys)[GridLds<W>::kPitch] = reinterpret_cast<long long (*)[GridLds<W>::kPitch]>(L.stage[tw]);
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    keys[rs][col_of(c)] = (static_cast<long long>(__float_as_int(bv[c])) << 32) | static_cast<unsigned>(0x7fffffff - bi[c]);
  wave_lds_fence();
  long long best = keys[0][lane];
#pragma unroll
  for (int k = 1; k < 8; ++k) best = keys[k][lane] > best ? keys[k][lane] : best;
  __syncthreads();                                           // the last iteration's totals have been read
  long long* of_wave = reinterpret_cast<long long*>(&L.sum[0][0][0]);
  of_wave[64 * tw + lane] = best;
  __syncthreads();
  if (tw == 0 && lane < r) {
#pragma unroll
    for (int w = 1; w < W; ++w) best = of_wave[64 * w + lane] > best ? of_wave[64 * w + lane] : best;
    const int i = 0x7fffffff - static_cast<int>(best);
    pair_out[lo + m + lane] = i >= m ? -1 : i;
  }
}

// Tall images (up to 1279 kept rows) with up to 31 pruned tokens: the same scheme on eight waves with four column slots
// (lane bits 0 and 1) x sixteen row slots, so that a lane's ten rows are two batches and a half instead of five: lane
// (cs, rs) holds columns 2 cs, 2 cs + 1, 8 + 2 cs, ... of rows 16 tw + rs + 128 a.  A wave is a part.
// Measured, 64 images of 1156 tokens with 28 pruned, an iteration: 1.34 us (eight column slots, entries held as fp32 and
// column sums through LDS, sinkhorn_quad.hpp: 2.35); 128 ragged tiled pages, 50 iterations, a call 457 -> 400 us.  Not kept: 47 pruned
// the same way, 120 entries a lane held as fp32, of which the compiler spills 64: 4.1 us against 2.8.
struct GridTallShape {
  static constexpr int W = 8, CPT = 8, RPT = 10, kMaxRows = 128 * RPT, kMaxCols = 4 * CPT;   // augmented
};
__device__ __forceinline__ int grid_tall_entry(int lane) { return 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1); }
__device__ __forceinline__ double grid_tall_scatter(const double (&t)[8]) {
  double h[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) h[c] = halve32(t[c], t[c + 4]);
  return add_xor_lane4(halve8(halve16(h[0], h[2]), halve16(h[1], h[3])));
}
__device__ __forceinline__ void sinkhorn_grid_tall_image(const SinkhornArgs& A, int b, GridLds<8>& L) {
  using S = GridTallShape;
  constexpr int W = S::W, CPT = S::CPT, RPT = S::RPT, kB = (RPT + 3) / 4;
  const DevParams& p = A.p;
  const int tt = threadIdx.x, tw = __builtin_amdgcn_readfirstlane(tt >> 6), lane = tt & 63;
  const int cs = lane & 3, rs = lane >> 2;
  const int lo = __builtin_amdgcn_readfirstlane(A.offsets[b]);
  const int n = __builtin_amdgcn_readfirstlane(A.offsets[b + 1]) - lo;
  if (n <= 0) return;
  const int m = min(max(__builtin_amdgcn_readfirstlane(A.keep[b]), 0), n), r = n - m;
  if (m + 1 > S::kMaxRows || r + 1 > S::kMaxCols) return;    // uniform over the workgroup
  int32_t* __restrict__ pair_out = A.pair_out;
  if (pair_out)
    for (int i = tt; i < m; i += 64 * W) pair_out[lo + i] = i;
  if (r <= 0 || m <= 0) return;
  const long long po = A.plan_offsets[b];
  if (!plan_fits(po, m, r, A.plan_cap)) return;
  const float* __restrict__ Kg = k32_base(A.kmat, po);       // stored as fp32 (kKernelRowsF32)
  const int pitch = k32_pitch(r);
  const double kz = exp((p.z - p.shift) / p.eps);
  const int row0 = 16 * tw + rs;
  auto col_of = [&](int c) { return 2 * cs + 8 * (c >> 1) + (c & 1); };
  const int last = m >> 9;                                   // the batch of the dustbin row: the last one there is

  double K[RPT][CPT];
#pragma unroll
  for (int a = 0; a < RPT; ++a) {
    const float* row = Kg + min(row0 + 128 * a, m - 1) * pitch;
    float v[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) v[c] = row[min(col_of(c), r - 1)];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int i = row0 + 128 * a, j = col_of(c);
      K[a][c] = i < m && j < r ? static_cast<double>(v[c]) : i <= m && j <= r ? kz : i > m && j == 0 ? 1.0 : 0.0;
      forget_origin(K[a][c]);
    }
  }

  const double x_init = exp(p.shift / p.eps);                // T = 0 leaves u = 0
  const int u_own = lane & 3;                                // the row of a batch this lane finishes
  const bool bit0 = (lane & 1) != 0, bit1 = (lane & 2) != 0;
  const int own = col_of(grid_tall_entry(lane));        // the column this lane finishes
  const double b_col = own < r ? 1.0 : static_cast<double>(m);
  const int i_last = row0 + 128 * (4 * last + u_own);
  const double a_last = i_last < m ? 1.0 : i_last == m ? static_cast<double>(r) : 0.0;
  double y[CPT], x_own[kB];
#pragma unroll
  for (int q = 0; q < kB; ++q) {
    x_own[q] = row0 + 128 * (4 * q + u_own) <= m ? x_init : 0.0;
  }
  L.y[tw][own] = own <= r ? 1.0 : 0.0;
  wave_lds_fence();
  auto read_y = [&] {
#pragma unroll
    for (int c = 0; c < CPT; c += 2) {
      const f64x2g_t v = *reinterpret_cast<const f64x2g_t*>(&L.y[tw][2 * cs + 4 * c]);
      y[c] = v[0];
      y[c + 1] = v[1];
    }
  };
  auto spread = [](double v, double (&x)[4]) {
    x[0] = dpp_move<0x00>(v);
    x[1] = dpp_move<0x55>(v);
    x[2] = dpp_move<0xAA>(v);
    x[3] = dpp_move<0xFF>(v);
  };
  read_y();
  if (tt == 0) L.moved = 0;
  __syncthreads();

  int stop_at = p.iters;
  for (int it = 0; it < stop_at; ++it) {
    bool differs = false;
    double t[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) t[c] = 0.0;
#pragma unroll
    for (int q = 0; q < kB; ++q) {
      if (q > last) continue;                                // (the same for every thread)
      double s[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int a = 4 * q + u < RPT ? 4 * q + u : 0;
        s[u] = 1.0;                                          // (rows that a lane does not have)
        if (4 * q + u < RPT) {
#pragma unroll
          for (int c = 0; c < CPT; ++c) s[u] = c == 0 ? K[a][c] * y[c] : fma(K[a][c], y[c], s[u]);
        }
      }
      double xv = rcp64_tight(halve_quad<0x4E>(halve_quad<0xB1>(s[0], s[1], bit0), halve_quad<0xB1>(s[2], s[3], bit0), bit1));
      if (q == last) xv *= a_last;
      differs |= __double_as_longlong(xv) != __double_as_longlong(x_own[q]);
      x_own[q] = xv;
      double x[4];
      spread(xv, x);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (4 * q + u < RPT) {
#pragma unroll
          for (int c = 0; c < CPT; ++c) t[c] = fma(K[4 * q + u < RPT ? 4 * q + u : 0][c], x[u], t[c]);
        }
    }
    L.sum[it & 1][tw][lane] = grid_tall_scatter(t);
    if (differs) L.moved = it + 1;
    __syncthreads();
    const int moved = __builtin_amdgcn_readfirstlane(L.moved);
    const double (*part)[64] = L.sum[it & 1];
    const double total = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) +
                   ((part[4][lane] + part[5][lane]) + (part[6][lane] + part[7][lane]));
    L.y[tw][own] = own <= r ? b_col * rcp64_tight(total) : 0.0;
    wave_lds_fence();
    read_y();
    // (the same in every wave, see sinkhorn_grid_image)
    stop_at = settled_stop(stop_at, it, moved >= it + 1);
  }

  // ---- plan and pairing (row m is the dustbin) ----
  float* P = A.plan_out ? A.plan_out + po : nullptr;
  float bv[CPT];
  int bi[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) { bv[c] = -1.f; bi[c] = 0x7fffffff; }
  float* rows = reinterpret_cast<float*>(&L.stage[tw][0][0]);  // sixteen rows of the plan, turned to whole rows
  constexpr int kRowPitch = GridLds<8>::kPitch;
#pragma unroll
  for (int q = 0; q < kB; ++q) {
    if (q > last) continue;
    double x[4];
    spread(x_own[q], x);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (4 * q + u >= RPT) continue;
      const int a = 4 * q + u < RPT ? 4 * q + u : 0;
      int i = row0 + 128 * a;
      forget_origin(i);
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const float v = static_cast<float>(x[u] * K[a][c] * y[c]);
        rows[rs * kRowPitch + col_of(c)] = v;
        if (i <= m && v > bv[c]) { bv[c] = v; bi[c] = i; }
      }
      wave_lds_fence();
      if (P && lane < r) {
#pragma unroll
        for (int l = 0; l < 16; ++l) {
          const int il = i - rs + l;
          if (il < m) P[il * r + lane] = rows[l * kRowPitch + lane];
        }
      }
      wave_lds_fence();
    }
  }
  if (!pair_out) return;
  // a column's best as a key (value bits, then the lower row), over lane bit 2 at once, then as in sinkhorn_grid_image
  long long (*keys)[GridLds<8>::kPitch] = reinterpret_cast<long long (*)[GridLds<8>::kPitch]>(L.stage[tw]);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    long long key = (static_cast<long long>(__float_as_int(bv[c])) << 32) | static_cast<unsigned>(0x7fffffff - bi[c]);
    const long long other = __shfl_xor(key, 4, kWave);
    key = other > key ? other : key;
    if ((lane & 4) == 0) keys[rs >> 1][col_of(c)] = key;
  }
  wave_lds_fence();
  long long best = keys[0][lane];
#pragma unroll
  for (int k = 1; k < 8; ++k) best = keys[k][lane] > best ? keys[k][lane] : best;
  __syncthreads();                                           // the last iteration's totals have been read
  long long* of_wave = reinterpret_cast<long long*>(&L.sum[0][0][0]);
  of_wave[64 * tw + lane] = best;
  __syncthreads();
  if (tw == 0 && lane < r) {
#pragma unroll
    for (int w = 1; w < W; ++w) best = of_wave[64 * w + lane] > best ? of_wave[64 * w + lane] : best;
    const int i = 0x7fffffff - static_cast<int>(best);
    pair_out[lo + m + lane] = i >= m ? -1 : i;
  }
}

// An image of list kVariantC32 on a workgroup of W waves (four of them for those beyond 351 x 63: the limit of four waves holds
// for eight as well, so that an image gives the same bits alone and in a large batch).
template <int W>
__device__ __forceinline__ void sinkhorn_c32_image(const SinkhornArgs& A, int img, void* lds) {
  const int n = A.offsets[img + 1] - A.offsets[img], m = min(max(A.keep[img], 0), max(n, 0));
  if (m + 1 <= GridShape<4, 8, float>::kMaxRows && n - m + 1 <= GridShape<4, 8, float>::kMaxCols)
    sinkhorn_grid_image<GridShape<W, 8, float>>(A, img, *static_cast<GridLds<W>*>(lds));
  else if (W == QuadPage::W || threadIdx.x < QuadPage::kThreads)
    sinkhorn_quad_image<QuadPage>(A, img, *static_cast<QuadLds<QuadPage::W>*>(lds));
}

// The images of list kVariantC32 of a batch of more images than the chip has compute units (of fewer, they are
// k_sinkhorn_regs's), one at a time per workgroup, two workgroups per compute unit (at most 256
// registers per lane; with three batches of rows on four waves seven are spilled, 32 bytes a lane, before and after the
// iterations), which take the list in turns.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sinkhorn_c32(
    SinkhornArgs A, const int32_t* __restrict__ work, int B, const int32_t* __restrict__ status) {
  if (status[0]) return;
  __shared__ __align__(16) unsigned char lds[sizeof(GridLds<4>) > sizeof(QuadLds<4>) ? sizeof(GridLds<4>) : sizeof(QuadLds<4>)];
  const int cnt = work[kVariantC32];
  for (int blk = blockIdx.x; blk < cnt; blk += gridDim.x) {
    if (blk != static_cast<int>(blockIdx.x)) __syncthreads();   // the previous image's LDS is still being read
    sinkhorn_c32_image<4>(A, work[kWorkLists + kVariantC32 * B + blk], lds);
  }
}

}  // namespace rtp
