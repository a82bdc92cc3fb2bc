// Sinkhorn (Appendix C) for images with more than 128 pruned tokens, or more kept rows than the
// shapes of sinkhorn_cluster.hpp hold (the page sizes of other OCR models): the kernel matrix is
// held as fp32 in the registers of several workgroups for all T iterations.
//
// The workgroups of all slots are resident together (one per compute unit and no more are
// launched: each fills a compute unit's registers), a slot being as many workgroups as the
// largest of the launch's images needs (the list's builder counts them: a host that only knows the
// parameters does not know them when the kept counts are the caller's), and a slot works through its
// share of the list with all its workgroups in step.  Slots of up to sixteen keep to one XCD.
//
// Who waits for whom.  Calls on other streams may hold compute units with workgroups that wait for
// their own slots, so that no slot gets complete: three calls with 10 + 11 + 11 workgroups of slots of
// sixteen fill an XCD, and slots across XCDs can each lack workgroups that another's keep out.  So no
// slot waits for ever to be complete: before a slot's workgroups touch anything they meet, and one that
// has waited too long (C.form_limit, some 30 ms) gives the slot up, for good and for all its workgroups,
// which leave.  The images of slots given up are done by the launch's last `groups` workgroups,
// which nobody else of the launch waits for and which do wait until they are all there.  They have
// consecutive numbers, at most kStripMaxGroups / 8 = 8 of them on an XCD, so of four such calls (one per
// hardware queue) at most 7 + 3 * 8 = 31 of an XCD's 32 compute units are held by workgroups that
// wait for others of theirs (slots of sinkhorn_cluster.hpp: 7 each): the next always finds a place.
//
// A workgroup's eight waves hold RPT whole rows each, a lane the columns lane, lane + 64, ...  An
// iteration is two passes over the registers, widening every entry at both uses:
//   rows     a lane's share of the row sums of eight rows at a time; the 64 lanes' shares go
//            through a reduce-scatter (halving exchanges) that leaves eight lanes with one row's
//            total, so that the exchanges and the reciprocal are paid once for eight rows, and
//            the x travel back through scalar registers;
//   columns  sum_i x_i K_ij over the wave's rows, lane-local; the eight waves meet in LDS.
// What bounds it: vector instruction issue in the two passes (two conversions and two multiply-adds
// per entry, 3.7 us of an iteration), then the exchange (2 us in one trip, 6 in two).  Measured for
// 100 iterations: 64 pages of 1083 tokens (four workgroups of 144 x 576 each) 0.91 -> 0.60 ms, 32
// pages of 2137 (sixteen of 80 x 960) 2.48 -> 1.46 ms against strips that gave every row a reduction
// of its own over the 64 lanes and a reciprocal in all of them (28 instructions a row beside 27 for
// its nine columns' arithmetic); 16 pages of 4512 tokens (58 of 48 x 1792) 6.72 -> 3.92 ms against
// streaming the matrices from memory every iteration.
//
// The exchange.  A few workgroups publish their column sums and everybody adds everybody's in
// rank order.  With more of them (strip_direct) that means groups x (r + 1) doubles read by each
// workgroup and iteration, so the columns are dealt out instead: a workgroup receives all the
// others' sums for its share of the columns, adds them in a fixed order, takes the reciprocal and
// publishes the finished y; everybody reads all y.  Two trips through memory instead of one, but
// 2 (r + 1) values read instead of groups (r + 1).
// Values travel as device-scope relaxed atomics, and a place holds a "not yet" pattern until its
// value is there, so no counters and no barriers across workgroups; four buffers in turn (they lie
// in the image's own kernel-matrix slot, see strip_exchange_doubles), cleared before the image:
//   direct   a workgroup that publishes iteration i has seen everybody's sums of i - 1, whose
//            owners had by then finished reading i - 2, so its place in the buffer of i - 2
//            (= i + 2 modulo four) gets its "not yet" back now; the store is acknowledged (the
//            wait before the next publication) before the sums of i + 1 go out, and nobody looks
//            at the buffer of i + 2 before having seen those.
//   shares   the only reader of a place in the sums' buffer i is the owner of the columns, which
//            puts "not yet" back as soon as it has read it; that is acknowledged before the
//            owner publishes the y of i + 1, without which nobody gets to iteration i + 2, let
//            alone to the next use of the buffer, i + 4.  The y of i are put back by their owner
//            once it has all the sums of i + 1, which every workgroup publishes after reading
//            the y of i; acknowledged before the y of i + 2 go out, while the places are polled
//            again for the y of i + 4, after those of i + 3 have been seen.
#pragma once
#include "common.hpp"
#include "sinkhorn_team.hpp"

namespace rtp {

constexpr int kStripThreads = 512;
// what a value's place holds until the value has been published: no sum has this bit pattern (a NaN)
constexpr long long kStripNotYet = -1;

struct StripArgs {
  SinkhornArgs S;
  int32_t* words;           // the shape's words, prepared by the kernel that built the lists
  int cus;                  // compute units the slots may take
  int slot_blocks;          // workgroups of the launch that make up slots; the others are the last ones
  int form_limit;           // polls for a slot to be complete (0: every slot is given up at once, for tests)
  int spin_limit;
  int32_t* status;
};

__device__ __forceinline__ void ex_store(double* at, double v) {
  __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ex_not_yet(double* at) {
  __hip_atomic_store(reinterpret_cast<long long*>(at), kStripNotYet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ex_load(const double* at) {
  return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool ex_missing(double v) { return __double_as_longlong(v) == kStripNotYet; }

// Whether a poll that has failed `spin` times goes on (false: gave up, here or elsewhere).
__device__ __forceinline__ bool ex_wait(const StripArgs& C, int spin) {
  if (spin >= C.spin_limit) return false;
  if ((spin & 63) == 63 && __hip_atomic_load(C.words + kStripGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    return false;
  __builtin_amdgcn_s_sleep(1);
  return true;
}

// Meeting of workgroups of a slot: this one arrives (if `join`) and waits until the slot's counter has
// reached `arrived` (every workgroup keeps the same running total).  A workgroup that has no strip of
// the current image waits for the image's meeting without joining: if it went on to the slot's next
// image at once, its arrival there would be counted into this one.  False: gave up.
__device__ __forceinline__ bool strip_meet(const StripArgs& C, int32_t* counter, int arrived, bool join, int* s_flag) {
  // This thread's published values must have been acknowledged before anybody is told that the
  // workgroup has arrived.  A workgroup-scope release does not wait for stores to be acknowledged
  // (waves of a workgroup share their caches), so the store counter is waited for explicitly.
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t* gave_up = C.words + kStripGaveUp;
    if (join) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int ok = 0;
    for (int spin = 0; spin < C.spin_limit; ++spin) {
      if (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= arrived) { ok = 1; break; }
      if (__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      __builtin_amdgcn_s_sleep(2);
    }
    if (!ok) {
      __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      atomicOr(C.status, RTP_DEV_SYNC_TIMEOUT);
    }
    *s_flag = ok;
  }
  __syncthreads();
  return *s_flag != 0;
}

// Whether a slot is complete (all its workgroups resident) or has been given up: neither changes any
// more.  `join`: this workgroup is one of the slot's.  Nothing has been touched yet, so a workgroup of
// a slot given up just leaves.
constexpr int kStripGivenUp = 1 << 30;     // in the slot's arrival counter (which stays below it: 65 535 images x 128)
__device__ __forceinline__ bool strip_complete(int32_t* counter, int per_slot, int limit, bool join, int* s_flag) {
  __syncthreads();                                     // the flag's last value has been read
  if (threadIdx.x == 0) {
    if (join && limit > 0) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int seen;
    for (int spin = 0;; ++spin) {
      seen = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((seen & kStripGivenUp) || seen >= per_slot) break;
      if (spin >= limit) {                             // (a failed exchange: another arrival, or given up by another)
        if (__hip_atomic_compare_exchange_strong(counter, &seen, seen | kStripGivenUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT)) {
          seen |= kStripGivenUp;
          break;
        }
        continue;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    *s_flag = !(seen & kStripGivenUp);
  }
  __syncthreads();
  return *s_flag != 0;
}

// Where image `b`'s workgroups exchange their values: the upper end of its kernel-matrix slot
// (strip_exchange_fits).  The sums' buffers first, then those of y (shares only), then the
// pairing keys, groups x r of them.
__device__ __forceinline__ double* strip_area(const SinkhornArgs& A, int shape, long long po, int m, int r, int groups) {
  const long long at = po + static_cast<long long>(m) * r - strip_exchange_doubles(shape, r, groups);
  return const_cast<double*>(A.kmat) + (at - at % kStripAlign);
}

// "Not yet" into workgroup `rank`'s part of image `b`'s exchange area, when it is a strip image.
template <typename S>
__device__ __forceinline__ void strip_clear(const StripArgs& C, int b, int rank) {
  const SinkhornArgs& A = C.S;
  const int n = A.offsets[b + 1] - A.offsets[b];
  const int m = min(max(A.keep[b], 0), max(n, 0)), r = max(n, 0) - m;
  if (m <= 0 || r <= 0 || sinkhorn_variant(m, r, A.p.mode) != kVariantStrip) return;
  if (!plan_fits(A.plan_offsets[b], m, r, A.plan_cap)) return;
  const int groups = strip_groups(S::kShape, m, A.p.mode);
  if (groups <= 1 || rank >= groups) return;
  double* area = strip_area(A, S::kShape, A.plan_offsets[b], m, r, groups);
  const int total = static_cast<int>(strip_exchange_doubles(S::kShape, r, groups) - static_cast<long long>(groups) * r);
  const int each = (total + groups - 1) / groups;
  const int e1 = min(total, (rank + 1) * each);
  for (int e = rank * each + threadIdx.x; e < e1; e += kStripThreads) ex_not_yet(area + e);
}

// LDS of a strip workgroup: the waves' column sums (reused for the pairing's candidates), their
// sums of x, the y (and the sum of x behind them), the received sums of the own columns; flags, and the
// slot's loop over its images while one is worked on.
template <typename S> constexpr int strip_lds_of() {
  return 8 * (8 * S::kCols + 8 + S::kCols + 2 + S::kCols + 258) + 64;
}
// Workgroup barrier that orders LDS accesses only: published values still on their way are not
// waited for, as __syncthreads would.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Row sums of eight rows (q[u]: this lane's share of row u): the total of row strip_row8(lane).
__device__ __forceinline__ double strip_reduce8(const double (&q)[8], int lane) {
  double h[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) h[k] = halve32(q[k], q[k + 4]);
  const double g0 = halve16(h[0], h[2]), g1 = halve16(h[1], h[3]);
  const bool b3 = (lane & 8) != 0;
  const double keep = b3 ? g1 : g0, send = b3 ? g0 : g1;
  return group_sum<3>(keep + dpp_move<0x128>(send));                 // (lane ^ 8)
}
__device__ __forceinline__ int strip_row8(int lane) { return 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1); }
constexpr int strip_lane8(int u) { return 32 * (u >> 2) + 16 * ((u >> 1) & 1) + 8 * (u & 1); }
// The same for four rows.
__device__ __forceinline__ double strip_reduce4(const double (&q)[8]) {
  return group_sum<4>(halve16(halve32(q[0], q[2]), halve32(q[1], q[3])));
}
__device__ __forceinline__ int strip_row4(int lane) { return 2 * (lane >> 5) + ((lane >> 4) & 1); }
constexpr int strip_lane4(int u) { return 32 * (u >> 1) + 16 * (u & 1); }

// The compiler forgets that it has seen rows a0 .. a0 + 7 (it would keep their entries' widened
// copies otherwise).
template <int RPT, int CPT>
__device__ __forceinline__ void forget_rows(float (&K)[RPT][CPT], int a0) {
#pragma unroll
  for (int a = 0; a < RPT; ++a)
#pragma unroll
    for (int c = 0; c < CPT; ++c)
      if (a >= a0 && a < a0 + 8) forget_origin(K[a][c]);
}

// One image on `groups` workgroups of a slot; this one is `rank` < groups.  `arrived`: the slot's
// arrival count once they have all met at the image's end.  False: a wait was given up, leave the kernel.
template <typename S>
__device__ __forceinline__ bool sinkhorn_strip_image(const StripArgs& C, int b, int rank, int groups, int32_t* counter,
                                                     int arrived, void* lds, int* s_flag) {
  constexpr int RPT = S::RPT, CPT = S::CPT, kCols = S::kCols, T = kStripThreads;
  constexpr int kChunks = (RPT + 7) / 8, kLast = RPT - 8 * (kChunks - 1);
  constexpr bool kKeepY = CPT <= 9;          // y in registers across the chunks of rows (else re-read from LDS)
  const SinkhornArgs& A = C.S;
  const DevParams& p = A.p;
  const int tt = threadIdx.x, tw = __builtin_amdgcn_readfirstlane(tt >> 6), lane = tt & 63;
  const int lo = A.offsets[b];
  const int n = A.offsets[b + 1] - lo;
  const int m = min(max(A.keep[b], 0), n), r = n - m;        // (the list holds images with n > 0, r > 0 only)
  const long long po = A.plan_offsets[b];
  const float* __restrict__ Kg = k32_base(A.kmat, po);        // stored as fp32 (kKernelRowsF32)
  const int pitch = k32_pitch(r);
  int32_t* __restrict__ pair_out = A.pair_out;
  const int rows_per = (m + groups - 1) / groups;            // the rows dealt evenly
  const int row_base = rank * rows_per;
  const int m_loc = min(m - row_base, rows_per);             // >= 1: groups = ceil(m / rows per strip)
  constexpr bool kMayDirect = strip_direct(S::kShape, 1);    // (the wider shapes never are)
  const bool direct = kMayDirect && strip_direct(S::kShape, groups);
  const int cw = strip_share(r, groups);                     // columns (the sum of x counted as column r) a workgroup owns
  const int own0 = rank * cw, own = max(0, min(cw, r + 1 - own0));
  double* area = groups > 1 ? strip_area(A, S::kShape, po, m, r, groups) : nullptr;
  const int sums_buf = direct ? groups * (r + 1) : groups * groups * cw;   // doubles of one buffer of sums
  double* ybufs = area + kStripBufs * sums_buf;
  long long* keys = reinterpret_cast<long long*>(direct ? ybufs : ybufs + kStripBufs * groups * cw);
  if (pair_out)
    for (int i = tt; i < m_loc; i += T) pair_out[lo + row_base + i] = row_base + i;

  double* xw = static_cast<double*>(lds);                    // [8][kCols]
  double* xsum = xw + 8 * kCols;                             // [8]
  double* ys = xsum + 8;                                     // [kCols] and the sum of x
  double* red = ys + kCols + 2;                              // [groups][cw]
  int* seen_words = reinterpret_cast<int*>(red + kCols + 258);   // [2]

  float K[RPT][CPT];
#pragma unroll
  for (int a = 0; a < RPT; ++a) {
    const float* row = Kg + static_cast<long long>(row_base + min(8 * a + tw, m_loc - 1)) * pitch;
#pragma unroll
    for (int c = 0; c < CPT; ++c) K[a][c] = row[min(64 * c + lane, r - 1)];
  }
#pragma unroll
  for (int a = 0; a < RPT; ++a)
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      K[a][c] = (8 * a + tw < m_loc && 64 * c + lane < r) ? K[a][c] : 0.f;
      forget_origin(K[a][c]);
    }

  const double kz = exp((p.z - p.shift) / p.eps);
  const double x_init = exp(p.shift / p.eps);      // T = 0 leaves u = 0
  for (int e = tt; e <= kCols; e += T) ys[e] = e < r ? 1.0 : 0.0;
  double x_dust = x_init, y_dust = 1.0;
  double xv[kChunks];                              // lanes strip_lane8(u) (last four or fewer rows: strip_lane4(u)): row 8 ch + u
#pragma unroll
  for (int ch = 0; ch < kChunks; ++ch) xv[ch] = x_init;
  const float inv_cw = 1.0f / static_cast<float>(cw);
  __syncthreads();

  for (int it = 0; it < p.iters; ++it) {
    const double row_dust = kz * y_dust;
    double xs = 0.0, ly = 0.0;
    double t[kChunks > 1 ? CPT : 1];
    double y[kKeepY ? CPT : 1];
    if constexpr (kKeepY) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) y[c] = ys[64 * c + lane];
    }
    if constexpr (kChunks > 1) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) t[c] = 0.0;
    }
#pragma unroll
    for (int ch = 0; ch < kChunks; ++ch) {
      if (ch > 0 && 64 * ch >= m_loc) continue;                // no row of this chunk exists (the same for every thread)
      const bool four = ch == kChunks - 1 && kLast <= 4;       // (known when unrolled, like the bounds below)
      double q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = 0.0;
      forget_rows(K, 8 * ch);
      // (y from LDS comes in kAhead columns at a time, one group ahead)
      constexpr int kAhead = CPT > 15 && CPT <= 22 ? 4 : 2;       // (what fits the registers)
      double yn[kAhead];
      if constexpr (!kKeepY) {
#pragma unroll
        for (int c = 0; c < kAhead; ++c) yn[c] = ys[64 * c + lane];
      }
#pragma unroll
      for (int c0 = 0; c0 < CPT; c0 += kAhead) {
        double yc[kAhead];
#pragma unroll
        for (int c = 0; c < kAhead; ++c) {
          yc[c] = kKeepY ? y[kKeepY && c0 + c < CPT ? c0 + c : 0] : yn[c];
          if constexpr (!kKeepY) {
            if (c0 + kAhead + c < CPT) yn[c] = ys[64 * (c0 + kAhead + c) + lane];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < kAhead; ++c)
          if (c0 + c < CPT) {
            if (ch == 0) ly += yc[c];
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (8 * ch + u < RPT)
                q[u] = fma(static_cast<double>(K[8 * ch + u < RPT ? 8 * ch + u : 0][c0 + c < CPT ? c0 + c : 0]), yc[c], q[u]);
          }
      }
      const double sum = four ? strip_reduce4(q) : strip_reduce8(q, lane);
      const int u_own = four ? strip_row4(lane) : strip_row8(lane);
      xv[ch] = 8 * (8 * ch + u_own) + tw < m_loc ? rcp64(sum + row_dust) : 0.0;
      double x[8];                                               // the same in every lane (scalar registers)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (8 * ch + u < RPT) {
          x[u] = read_lane(xv[ch], four ? strip_lane4(u & 3) : strip_lane8(u));
          xs += x[u];
        }
      forget_rows(K, 8 * ch);                                    // (entries are widened again, not kept widened)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        double acc = kChunks > 1 ? t[kChunks > 1 ? c : 0] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int a = 8 * ch + u;
          if (a < RPT) acc = fma(static_cast<double>(K[a < RPT ? a : 0][c]), x[u], acc);
        }
        if constexpr (kChunks > 1) t[c] = acc;
        else xw[tw * kCols + 64 * c + lane] = acc;
        if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (kChunks > 1) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) xw[tw * kCols + 64 * c + lane] = t[c];
    }
    if (lane == 0) xsum[tw] = xs;
    int& seen_all = seen_words[it & 1];                // (two words in turn: the next write of one is a whole iteration away)
    if (tt == 0) seen_all = 1;
    lds_barrier();
    // this workgroup's sums: column e (the sum of x as column r) by thread e, e + 512, ...
    constexpr int kE = (kCols + T) / T;                // r + 1 <= kCols + 1 columns
    int te = tt;
    forget_origin(te);                                 // (the places' addresses are worked out anew: registers)
    double part[kE];
#pragma unroll
    for (int l = 0; l < kE; ++l) {
      const int e = te + T * l;
      const double* col = e < r ? xw + min(e, kCols - 1) : xsum;
      const int step = e < r ? kCols : 1;
      double acc = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) acc += col[w * step];
      part[l] = acc;
    }
    const int buf = it & 3;
    double* sums = area + buf * sums_buf;
    if (groups > 1) {
      __builtin_amdgcn_s_waitcnt(0);                   // what was put back last iteration has been acknowledged
#pragma unroll
      for (int l = 0; l < kE; ++l) {
        const int e = te + T * l;
        const int o = static_cast<int>((static_cast<float>(e) + 0.5f) * inv_cw);   // e / cw
        if (e <= r) ex_store(sums + (direct ? rank * (r + 1) + e : (o * groups + rank) * cw + (e - o * cw)), part[l]);
      }
      if (direct) {
        double* ahead = area + ((it + 2) & 3) * sums_buf + rank * (r + 1);
#pragma unroll
        for (int l = 0; l < kE; ++l)
          if (te + T * l <= r) ex_not_yet(ahead + te + T * l);
      }
    }
    // (while the sums travel) the dustbins' scalings from the previous y
    x_dust = static_cast<double>(r) * rcp64(kz * (wave_sum_dpp(ly) + y_dust));
    const double col_dust = kz * x_dust;
    bool seen = true;
    if (kMayDirect && groups > 1 && direct) {
      // everybody's sums of the own columns, four workgroups at a time, added in rank order
#pragma unroll
      for (int l = 0; l < kE; ++l) part[l] = 0.0;
      for (int g0 = 0; g0 < groups; g0 += 4) {
        double v[kE][4];
        for (int spin = 0;; ++spin) {
          bool ready = true;
#pragma unroll
          for (int l = 0; l < kE; ++l)
#pragma unroll
            for (int g = 0; g < 4; ++g) v[l][g] = ex_load(sums + min(g0 + g, groups - 1) * (r + 1) + min(te + T * l, r));
#pragma unroll
          for (int l = 0; l < kE; ++l)
#pragma unroll
            for (int g = 0; g < 4; ++g) ready = ready && !ex_missing(v[l][g]);
          if (ready) break;
          if (!seen || !ex_wait(C, spin)) { seen = false; break; }
        }
#pragma unroll
        for (int l = 0; l < kE; ++l)
#pragma unroll
          for (int g = 0; g < 4; ++g) part[l] += g0 + g < groups ? v[l][g] : 0.0;
      }
    }
    if (groups > 1 && !direct) {
      constexpr int kLoads = (kCols + 256 + T - 1) / T;      // groups cw <= r + groups values
      {
        double* in = sums + rank * groups * cw;
        double v[kLoads];
        bool mine[kLoads];
#pragma unroll
        for (int l = 0; l < kLoads; ++l) {
          const int e = te + T * l, g = static_cast<int>((static_cast<float>(e) + 0.5f) * inv_cw);
          mine[l] = e < groups * cw && e - g * cw < own;
        }
        for (int spin = 0;; ++spin) {
          bool ready = true;
#pragma unroll
          for (int l = 0; l < kLoads; ++l) v[l] = ex_load(in + (mine[l] ? te + T * l : 0));
#pragma unroll
          for (int l = 0; l < kLoads; ++l) ready = ready && !(mine[l] && ex_missing(v[l]));
          if (ready) break;
          if (!ex_wait(C, spin)) { seen = false; break; }
        }
#pragma unroll
        for (int l = 0; l < kLoads; ++l)
          if (mine[l]) red[te + T * l] = v[l];
        lds_barrier();
        // sixteen lanes add up a column
        double* yout = ybufs + buf * groups * cw + own0;
        for (int k = te >> 4; k < own; k += T / 16) {
          double acc = 0.0;
          for (int g = te & 15; g < groups; g += 16) acc += red[g * cw + k];
          acc = group_sum<4>(acc);
          if ((te & 15) == 0) ex_store(yout + k, own0 + k < r ? rcp64(acc + col_dust) : acc);
        }
        // put back: the sums just read, and the previous iteration's y (all the sums of this
        // iteration are here, so everybody has read those)
#pragma unroll
        for (int l = 0; l < kLoads; ++l)
          if (mine[l]) ex_not_yet(in + te + T * l);
        double* ylast = ybufs + ((it + 3) & 3) * groups * cw + own0;
        for (int k = te; k < own; k += T) ex_not_yet(ylast + k);
      }
      const double* yin = ybufs + buf * groups * cw;
      for (int spin = 0;; ++spin) {
        bool ready = true;
#pragma unroll
        for (int l = 0; l < kE; ++l) part[l] = ex_load(yin + min(te + T * l, r));
#pragma unroll
        for (int l = 0; l < kE; ++l) ready = ready && !ex_missing(part[l]);
        if (ready) break;
        if (!seen || !ex_wait(C, spin)) { seen = false; break; }
      }
    }
    const bool finished = groups > 1 && !direct;       // `part` holds y already
#pragma unroll
    for (int l = 0; l < kE; ++l) {
      const int e = te + T * l;
      const double v = finished || e >= r ? part[l] : rcp64(part[l] + col_dust);
      if (e <= r) ys[e < r ? e : kCols] = v;
    }
    if (!seen) seen_all = 0;
    lds_barrier();
    if (!seen_all) {                                   // a wait was given up (here or elsewhere): everybody leaves
      if (tt == 0) {
        __hip_atomic_store(C.words + kStripGaveUp, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicOr(C.status, RTP_DEV_SYNC_TIMEOUT);
      }
      return false;
    }
    y_dust = static_cast<double>(m) * rcp64(kz * (ys[kCols] + x_dust));
  }
  __syncthreads();

  // ---- plan and this workgroup's best partner per column ----
  float* P = A.plan_out ? A.plan_out + po : nullptr;
  float* pv = static_cast<float*>(lds);                        // [8][kCols], where the sums were
  int* pi = reinterpret_cast<int*>(pv + 8 * kCols);            // [8][kCols]
  int lane_p = lane, row_p = row_base + tw;
  forget_origin(lane_p);                                       // (keeps the entries' offsets out of the loop's registers)
  forget_origin(row_p);
  double x[RPT];
#pragma unroll
  for (int a = 0; a < RPT; ++a)
    x[a] = read_lane(xv[a / 8], a / 8 == kChunks - 1 && kLast <= 4 ? strip_lane4(a & 3) : strip_lane8(a & 7));
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int j = 64 * c + lane_p;
    const double yj = ys[64 * c + lane];
    float bv = -1.f;
    int bi = 0x7fffffff;
#pragma unroll
    for (int a = 0; a < RPT; ++a) {
      const int i = row_p + 8 * a;
      if (8 * a + tw < m_loc && j < r) {
        const float v = static_cast<float>(x[a] * static_cast<double>(K[a][c]) * yj);
        if (P) P[static_cast<long long>(i) * r + j] = v;
        if (v > bv) { bv = v; bi = i; }
      }
    }
    pv[tw * kCols + 64 * c + lane] = bv;
    pi[tw * kCols + 64 * c + lane] = bi;
  }
  __syncthreads();
  // each column's best of the workgroup's rows as a key (value bits, then the lower row): plan
  // entries are >= 0, so their bit patterns order like their values; "no row" (-1) is below all
  if (pair_out) {
    for (int e = tt; e < r; e += T) {
      float bv = -1.f;
      int bi = 0x7fffffff;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const float ov = pv[w * kCols + e];
        const int oi = pi[w * kCols + e];
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      if (groups == 1)
        pair_out[lo + m + e] = static_cast<float>(x_dust * kz * ys[e]) > bv ? -1 : bi;
      else
        __hip_atomic_store(keys + static_cast<long long>(rank) * r + e,
                           (static_cast<long long>(__float_as_int(bv)) << 32) | static_cast<unsigned>(0x7fffffff - bi),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (!strip_meet(C, counter, arrived, true, s_flag)) return false;
  if (pair_out && groups > 1) {
    // every workgroup picks the best of its share of the columns, eight lanes to a column
    for (int k = tt >> 3; k < own; k += T / 8) {
      const int e = own0 + k;
      if (e >= r) break;
      long long best = static_cast<long long>(__float_as_int(-1.f)) << 32;
      for (int g = tt & 7; g < groups; g += 8) {
        const long long key = __hip_atomic_load(keys + static_cast<long long>(g) * r + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        best = key > best ? key : best;
      }
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {
        const long long other = __shfl_xor(best, o, kWave);
        best = other > best ? other : best;
      }
      if ((tt & 7) == 0)
        pair_out[lo + m + e] =
            static_cast<float>(x_dust * kz * ys[e]) > __int_as_float(static_cast<int>(best >> 32)) ? -1 : 0x7fffffff - static_cast<int>(best);
    }
  }
  return true;
}

// Slot s takes images s, s + slots, ... of the list.  The slot's arrival counter runs on through all
// its meetings: one when the slot is complete, one of all its workgroups before each image (the image's
// exchange area cleared), one of the image's workgroups at its end (the pairing keys out).  The last
// workgroups take the slots given up, one after another, with a counter of their own.
template <typename S>
__global__ __launch_bounds__(kStripThreads) void k_sinkhorn_strips(StripArgs C) {
  __shared__ __align__(16) unsigned char lds[strip_lds_of<S>()];
  int* flag = reinterpret_cast<int*>(lds + strip_lds_of<S>()) - 2;
  // (all waves or none: a slot that gives up writes the word while the last workgroups may be starting)
  if (threadIdx.x == 0) *flag = C.status[0];
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*flag)) return;
  int count = C.words[kStripCount], per_slot = C.words[kStripTop];
  if (count == 0) return;
  const int block = blockIdx.x;
  bool last = block >= C.slot_blocks;
  int slots = strip_slots(per_slot, C.cus), slot, rank;
  if (per_slot <= kStripXcdGroups) {                   // one XCD per slot
    slots = min(slots, (count + 7) / 8 * 8);
    slot = (block & 7) * (slots >> 3) + (block >> 3) / per_slot;
    rank = (block >> 3) % per_slot;
  } else {
    slots = min(slots, count);
    slot = block / per_slot;
    rank = block % per_slot;
  }
  if (last) {
    slot = 0;
    rank = block - C.slot_blocks;
    if (rank >= per_slot) return;
    const int seen = static_cast<int>(threadIdx.x) < min(slots, count)   // (the slots that have images)
                         ? __hip_atomic_load(C.words + kStripCounters + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                         : per_slot;
    if (!__syncthreads_or((seen & kStripGivenUp) || seen < per_slot)) return;   // all complete: the usual case
  } else if (block >= slots * per_slot || slot >= count) {
    return;
  }
  const SinkhornArgs& A = C.S;
  int arrived = last ? 0 : per_slot, form_limit = C.form_limit;
  // the loop's state, in LDS while an image is worked on: in registers it makes the kernels spill
  // (4512-token pages 5.75 -> 5.90 ms a call)
  int* at = reinterpret_cast<int*>(lds + strip_lds_of<S>()) - 12;
  for (;;) {
    if (strip_complete(C.words + kStripCounters + slot, per_slot, form_limit, !last, flag) != last) {
      for (int k = slot; k < count; k += slots) {
        const int b = C.words[kStripList - (S::kShape - 1) * kStripShapeWords + C.words[kStripFirst] + k];
        const int n = A.offsets[b + 1] - A.offsets[b];
        const int m = min(max(A.keep[b], 0), max(n, 0)), r = max(n, 0) - m;
        // (every workgroup of the slot takes the same decisions: they read the same words)
        if (m <= 0 || r <= 0 || sinkhorn_variant(m, r, A.p.mode) != kVariantStrip) continue;
        if (!plan_fits(A.plan_offsets[b], m, r, A.plan_cap)) continue;
        const int groups = strip_groups(S::kShape, m, A.p.mode);   // (at most per_slot: the list's builder has counted)
        int32_t* counter = C.words + (last ? kStripLast : kStripCounters + slot);
        strip_clear<S>(C, b, rank);
        arrived += per_slot;
        if (!strip_meet(C, counter, arrived, true, flag)) return;
        arrived += groups;
        if (rank < groups) {
          if (threadIdx.x == 0) {
            at[0] = slot, at[1] = k, at[2] = arrived, at[3] = slots, at[4] = count, at[5] = per_slot, at[6] = rank, at[7] = last, at[8] = form_limit;
          }
          if (!sinkhorn_strip_image<S>(C, b, rank, groups, counter, arrived, lds, flag)) return;
          slot = __builtin_amdgcn_readfirstlane(at[0]);
          k = __builtin_amdgcn_readfirstlane(at[1]);
          arrived = __builtin_amdgcn_readfirstlane(at[2]);
          slots = __builtin_amdgcn_readfirstlane(at[3]);
          count = __builtin_amdgcn_readfirstlane(at[4]);
          per_slot = __builtin_amdgcn_readfirstlane(at[5]);
          rank = __builtin_amdgcn_readfirstlane(at[6]);
          last = __builtin_amdgcn_readfirstlane(at[7]) != 0;
          form_limit = __builtin_amdgcn_readfirstlane(at[8]);
        } else if (!strip_meet(C, counter, arrived, false, flag)) {
          return;
        }
      }
    }
    if (!last || ++slot >= min(slots, count)) return;
  }
}

}  // namespace rtp
