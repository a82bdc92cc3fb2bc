// Sinkhorn (Appendix C) for images with more than 128 pruned tokens, or more kept rows than the
// shapes of sinkhorn_cluster.hpp hold (the page sizes of other OCR models): the kernel matrix is
// held as fp32 in the registers of several workgroups for all T iterations.
//
// The workgroups of all slots are resident together (two per compute unit and no more are
// launched: they fill its registers), a slot being as many compute units' as the
// largest of the launch's images needs (the list's builder counts them: a host that only knows the
// parameters does not know them when the kept counts are the caller's), and a slot works through its
// share of the list with all its workgroups in step.  Slots of up to sixteen compute units keep to one XCD.
//
// Who waits for whom.  Calls on other streams may hold compute units with workgroups that wait for
// their own slots, so that no slot gets complete: three calls with slots of 10, 11 and 11 of sixteen
// compute units fill an XCD, and slots across XCDs can each lack workgroups that another's keep out.  Nor is a
// compute unit always good for two: registers and LDS are taken as ranges, and a workgroup that was put
// above another kernel's waves leaves no 256 registers on either side when those have gone.  So no
// slot waits for ever to be complete: before a slot's workgroups touch anything they meet, and one that
// has waited too long (C.form_limit, some 30 ms) gives the slot up, for good and for all its workgroups,
// which leave.  The images of slots given up are done by a launch of their own behind this one
// (k_sinkhorn_strips_left), whose workgroups do wait until they are all there.  They are twice as large, the work of
// two, and fill a compute unit: at most kStripMaxGroups / 8 = 8 of them on an XCD, so of four such calls (one per
// hardware queue) at most 7 + 3 * 8 = 31 of an XCD's 32 compute units are held by workgroups that
// wait for others of theirs (slots of sinkhorn_cluster.hpp: 7 each), and the next finds a place on the last as soon as
// those that wait for nobody have left it.
//
// A workgroup's four waves hold RPT whole rows each, a lane the columns lane, lane + 64, ...; two workgroups
// share a compute unit, as a rule of different images, so that one's exchange runs beside the other's
// arithmetic.  An iteration is two passes over the registers, widening every entry at both uses:
//   rows     a lane's share of the row sums of eight rows at a time; the 64 lanes' shares go
//            through a reduce-scatter (halving exchanges) that leaves eight lanes with one row's
//            total, so that the exchanges and the reciprocal are paid once for eight rows, and
//            the x travel back through scalar registers;
//   columns  sum_i x_i K_ij over the wave's rows, lane-local; the waves meet in LDS.
// What bounds it: of an iteration's 12 100 clocks on 64 pages of 1083 tokens (two workgroups of 72 x 576 to a
// compute unit) 5 100 are the two passes (two conversions and two multiply-adds per entry), the others the
// exchange: sums to LDS and out 1 300, the trip 1 800, adding up and out again 1 100, the second trip
// 2 900.  16 pages of 4512 tokens (116 workgroups an image, across the XCDs): 21 000, 4 800 in the passes, the trips
// 4 200 and 7 900.  Against one workgroup of eight waves to a compute unit, with one trip among up to sixteen workgroups
// and places put back to a "not yet" pattern (100 iterations): 32 pages of 2137 tokens 1.46 -> 1.21 ms, 16 pages of
// 4512 3.90 -> 3.67, 64 pages of 1083 0.59 -> 0.58.
// Before those, strips that gave every row a reduction of its own: 0.91 (1083 tokens) and 2.48 ms (2137);
// streaming the matrices from memory every iteration: 6.72 ms (4512).
//
// The exchange.  While it is not much to read (strip_direct: 18 KB), everybody adds everybody's column sums in
// rank order.  With more workgroups or columns than that, groups x (r + 1) doubles a
// workgroup and iteration, the columns are dealt out instead: a workgroup receives all the
// others' sums for its share of the columns, adds them in a fixed order, takes the reciprocal and
// publishes the finished y; everybody reads all y.  Two trips through memory instead of one, but
// 2 (r + 1) values read instead of groups (r + 1).  (Eight workgroups of 523 columns, 64 images: 0.88 ms
// with one trip, 0.81 with two, with the protocol of the time; up to six of 280: 0.540 and 0.577.)
// Values travel as device-scope stores and loads past the caches, the loads straight into LDS, and carry in
// their sign, which is theirs to spare (sums of products of positive numbers, and reciprocals of such), which use of
// their place they belong to (the uses alternate), so no counters, no barriers across workgroups, nothing put back and
// all 53 bits.
// The places lie in the image's own kernel-matrix slot, see strip_exchange_doubles, and are zero (of no use
// yet) before the image:
//   direct   two buffers in turn: a workgroup that publishes iteration i has seen everybody's sums of
//            i - 1, whose owners had by then finished reading i - 2, which it overwrites.
//   shares   one: the only reader of a sum is the owner of its column, who publishes the y of i after
//            reading the sums of i, and nobody publishes sums of i + 1 before having read all y of i.
//            The y of i are overwritten by their owner once it has all the sums of i + 1, which every
//            workgroup publishes after reading the y of i.
// A place is read by the same lane every iteration, so it is never seen to go back to an older use.
#pragma once
#include "common.hpp"
#include "sinkhorn_team.hpp"

namespace rtp {

constexpr int kStripThreads = 256, kStripWaves = kStripThreads / 64, kStripTeams = 2;   // workgroups to a compute unit
// (A workgroup of k_sinkhorn_strips_left has two teams of kStripThreads, each with the part of a workgroup of
// k_sinkhorn_strips and its own LDS.)
__device__ __forceinline__ int strip_thread() { return threadIdx.x & (kStripThreads - 1); }

struct StripArgs {
  SinkhornArgs S;
  int32_t* words;           // the shape's words, prepared by the kernel that built the lists
  int cus;                  // compute units the slots may take, two workgroups on each
  int form_limit;           // polls for a slot to be complete (0: every slot is given up at once, for tests)
  int spin_limit;
  int32_t* status;
};

// Two places at once, `at` (even) doubles into an image's exchange area: device-scope stores of 16 bytes, of which
// every 8 arrive whole (a lane's aligned 16 bytes lie in one request, written and read).  A value's sign says which use of its place it belongs to (`use`: 0 or kExOdd).
constexpr uint32_t kExOdd = 0x80000000u;
__host__ __device__ inline uint32_t ex_mark(uint32_t high, uint32_t use) { return (high & ~kExOdd) | use; }   // (a NaN may have either sign)
__host__ __device__ inline bool ex_is_of(uint32_t high, uint32_t use) { return ((high ^ use) & kExOdd) == 0; }
__host__ __device__ inline double ex_value(double marked) { return fabs(marked); }
typedef double f64x2_t __attribute__((ext_vector_type(2)));
constexpr int kExAgent = 16;   // (sc1: as far as all XCDs see it)
__device__ __forceinline__ auto ex_resource(double* area) { return __builtin_amdgcn_make_buffer_rsrc(area, 0, 0x7fffffff, 0x00020000); }
template <typename R>
__device__ __forceinline__ void ex_store2(R ex, int at, double v0, double v1, uint32_t use) {
  u32x4_t w = __builtin_bit_cast(u32x4_t, f64x2_t{v0, v1});
  w[1] = ex_mark(w[1], use);
  w[3] = ex_mark(w[3], use);
  __builtin_amdgcn_raw_buffer_store_b128(w, ex, 8 * at, 0, kExAgent);
}

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
  if (strip_thread() == 0) {
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

// Whether this workgroup's slot is complete (all its workgroups resident) or has been given up: neither changes any
// more.  Nothing has been touched yet, so a workgroup of a slot given up just leaves.
constexpr int kStripGivenUp = 1 << 30;     // in the slot's arrival counter (which stays below it: 65 535 images x 2 x 128)
__device__ __forceinline__ bool strip_complete(int32_t* counter, int per_slot, int limit, int* s_flag) {
  __syncthreads();                                     // the flag's last value has been read
  if (threadIdx.x == 0) {
    if (limit > 0) __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
// (strip_exchange_fits).  The sums first, then the y (shares only).
__device__ __forceinline__ double* strip_area(const SinkhornArgs& A, int shape, long long po, int m, int r, int groups) {
  const long long at = po + static_cast<long long>(m) * r - strip_exchange_doubles(shape, r, groups);
  return const_cast<double*>(A.kmat) + (at - at % kStripAlign);
}

// Zeros (of no use yet) into workgroup `rank`'s part of image `b`'s exchange area, when it is a strip image.
template <typename S>
__device__ __forceinline__ void strip_clear(const StripArgs& C, int b, int rank) {
  const SinkhornArgs& A = C.S;
  const int n = A.offsets[b + 1] - A.offsets[b];
  const int m = min(max(A.keep[b], 0), max(n, 0)), r = max(n, 0) - m;
  if (m <= 0 || r <= 0 || sinkhorn_variant(m, r, A.p.mode) != kVariantStrip) return;
  if (!plan_fits(A.plan_offsets[b], m, r, A.plan_cap)) return;
  const int groups = strip_teams(S::kShape, m, A.p.mode);
  if (groups <= 1 || rank >= groups) return;
  double* area = strip_area(A, S::kShape, A.plan_offsets[b], m, r, groups);
  const int total = static_cast<int>(strip_exchange_doubles(S::kShape, r, groups));
  const int each = (total + groups - 1) / groups;
  const int e1 = min(total, (rank + 1) * each);
  for (int e = rank * each + strip_thread(); e < e1; e += kStripThreads)
    __hip_atomic_store(area + e, 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS of a strip workgroup.  First the waves' column sums, which the values received from the others (whole
// pieces of 128 doubles, at most kReceive at a time) and in the end the pairing's candidates take the place of;
// then the y with the sum of x behind them, the image's constants; flags, and the slot's loop over its images
// while one is worked on.  Half a compute unit's 160 KB holds it.
constexpr int kStripPiece = 128;
template <typename S> struct StripLds {
  static constexpr int kPitch = S::kCols + 2;          // of a wave's column sums: with its sum of x behind them, and a zero
  static constexpr int kDirect = strip_direct(S::kShape, 1, 1) ? kStripDirectDoubles : 0;
  static constexpr int kShares = (S::kCols + 16 * kStripMaxGroups + kStripPiece - 1) / kStripPiece * kStripPiece;   // sums; behind them y
  static constexpr int kReceive = kDirect > 2 * kShares ? kDirect : 2 * kShares;
  static constexpr int kWaves = kStripWaves * kPitch;
  static constexpr int kFirst = ((kReceive > kWaves ? kReceive : kWaves) + kStripPiece - 1) / kStripPiece * kStripPiece;
  static constexpr int kBytes = 8 * (kFirst + S::kCols + 6) + 72;
  static_assert(kBytes <= 160 * 1024 / kStripTeams, "a compute unit's workgroups share its LDS");
};
template <typename S> constexpr int strip_lds_of() { return StripLds<S>::kBytes; }
// Workgroup barrier that orders LDS accesses only: published values still on their way are not
// waited for, as __syncthreads would.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Before a first look, about as long as the values take to get here (64 clocks a unit; up to sixteen workgroups, up
// to 32, which an XCD holds, and more).  A look at places that are being written costs more than the wait.  Calls of
// 100 iterations, us, after (sums, y) units: 64 pages of 1083 tokens, eight workgroups an image, (0, 0) 1008, (0, 4) 1004,
// (0, 8) 1005, (0, 12) 972, (0, 16) 952, (0, 20) 948, (4, 16) 959; 32 pages of 2137 tokens, 31 an image, (0, 16) 1786,
// (4, 8) 1890, (4, 12) 1805, (4, 16) 1769, (8, 16) 1782; 16 pages of 4512 tokens, 116 an image, (4, 20) 4875,
// (12, 16) 4835, (12, 20) 4797, (16, 24) 4723 (which one page of 4512 tokens takes 12 longer with).
__device__ __forceinline__ void ex_pause(int units) {
  for (int k = 0; k < units; k += 4) __builtin_amdgcn_s_sleep(4);
}

// `n` (even) published doubles from `src` into `rx`, straight from memory into LDS: wave `tw` takes every
// kStripWaves-th piece of 128, requests them all, and asks again for a piece until all of it is of use
// `use`; then `take(e, v0, v1)` gets values e and e + 1 of it.  No wave looks at another's pieces
// (a barrier makes rx readable for all).  False: gave up.
template <typename F>
__device__ __forceinline__ bool strip_receive(const StripArgs& C, const double* src, int n, uint32_t use, double* rx, int tw,
                                              int lane, F take) {
  const int pieces = (n + kStripPiece - 1) / kStripPiece, last = n - 2;
  auto request = [&](int k) {
    const double* at = src + min(kStripPiece * k + 2 * lane, last);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)at,
                                     (__attribute__((address_space(3))) void*)(rx + kStripPiece * k), 16, 0, kExAgent);
  };
#pragma unroll 1
  for (int k = tw; k < pieces; k += kStripWaves) request(k);
  int spin = 0;
  bool seen = true;
#pragma unroll 1
  for (int k = tw; k < pieces; k += kStripWaves) {
    f64x2_t v;
    for (;;) {
      __builtin_amdgcn_s_waitcnt(0);
      asm volatile("" ::: "memory");
      v = *reinterpret_cast<const f64x2_t*>(rx + kStripPiece * k + 2 * lane);
      const u32x4_t w = __builtin_bit_cast(u32x4_t, v);
      if (__ballot(!(ex_is_of(w[1], use) && ex_is_of(w[3], use))) == 0) break;
      if (!seen || !ex_wait(C, spin++)) { seen = false; break; }
      request(k);
    }
    take(kStripPiece * k + 2 * lane, ex_value(v[0]), ex_value(v[1]));
  }
  return seen;
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

// A strip's entries in a lane's registers, two to an aligned pair of them.  (One by one the allocator
// leaves no aligned pairs between them for the fp64 values and spills.)
template <int RPT, int CPT>
struct StripEntries {
  static_assert(RPT * CPT % 2 == 0, "whole pairs");
  floatx2_t pair[RPT * CPT / 2];
  __device__ __forceinline__ float get(int a, int c) const { return pair[(a * CPT + c) / 2][(a * CPT + c) % 2]; }
  __device__ __forceinline__ void set(int a, int c, float v) { pair[(a * CPT + c) / 2][(a * CPT + c) % 2] = v; }
  // The compiler forgets that it has seen rows a0 .. a1 - 1 (it would keep their entries' widened
  // copies otherwise).
  __device__ __forceinline__ void forget(int a0, int a1) {
#pragma unroll
    for (int k = 0; k < RPT * CPT / 2; ++k)
      if (k >= a0 * CPT / 2 && k < (a1 * CPT + 1) / 2) asm volatile("" : "+v"(pair[k]));
  }
};

// One image on `groups` workgroups of a slot; this one is `rank` < groups.  `arrived`: the slot's
// arrival count once they have all met at the image's end.  False: a wait was given up, leave the kernel.
// PAIRED: on a workgroup of two teams, of which this is one; both take the same barriers, also the second team
// that `groups` leaves without rows and columns (rank == groups), which publishes and writes nothing.
template <typename S, bool PAIRED>
__device__ __forceinline__ bool sinkhorn_strip_image(const StripArgs& C, int b, int rank, int groups, int32_t* counter,
                                                     int arrived, bool first, void* lds, int* s_flag) {
  constexpr int RPT = S::RPT, CPT = S::CPT, kCols = S::kCols, T = kStripThreads;
  constexpr int kChunks = (RPT + 7) / 8, kLast = RPT - 8 * (kChunks - 1);
  constexpr bool kKeepY = CPT <= 9;          // y in registers across the chunks of rows (else re-read from LDS)
  const SinkhornArgs& A = C.S;
  const DevParams& p = A.p;
  const int tt = strip_thread(), tw = __builtin_amdgcn_readfirstlane(tt >> 6), lane = tt & 63;
  const bool here = !PAIRED || rank < groups;
  // (in scalar registers: the compiler does not see that these loads' values are the same in all lanes)
  const int lo = __builtin_amdgcn_readfirstlane(A.offsets[b]);
  const int n = __builtin_amdgcn_readfirstlane(A.offsets[b + 1]) - lo;
  const int m = min(max(__builtin_amdgcn_readfirstlane(A.keep[b]), 0), n), r = n - m;   // (the list holds images with n > 0, r > 0 only)
  const long long po_at = A.plan_offsets[b];
  const long long po = static_cast<long long>((static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(po_at >> 32)))) << 32) |
                                              static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(po_at))));
  const float* __restrict__ Kg = k32_base(A.kmat, po);        // stored as fp32 (kKernelRowsF32)
  const int pitch = k32_pitch(r);
  int32_t* __restrict__ pair_out = A.pair_out;
  const int rows_per = (m + groups - 1) / groups;            // the rows dealt evenly
  const int row_base = rank * rows_per;
  const int rows = min(m - row_base, rows_per), m_loc = rows;   // >= 1: groups = ceil(m / rows per strip)
  constexpr bool kMayDirect = strip_direct(S::kShape, 1, 1);    // (the wider shapes never are)
  const bool direct = kMayDirect && strip_direct(S::kShape, r, groups);
  const int cw = strip_share(r, groups);                     // columns (the sum of x counted as column r) a workgroup owns
  const int own0 = rank * cw;
  double* area = groups > 1 ? strip_area(A, S::kShape, po, m, r, groups) : nullptr;
  const int owned = strip_owned(r, cw);                      // doubles of y, and of a buffer of sums:
  const int own = own0 < owned ? cw : 0;                     // (columns past the sum of x are zeros)
  const int row = strip_row(r), sums_buf = groups * (direct ? row : owned);
  // the pairing keys, `row` places to a workgroup: in a buffer of sums that everybody has read at the end
  long long* keys = reinterpret_cast<long long*>(area + (direct ? p.iters % 2 * sums_buf : 0));
  if (pair_out)
    for (int i = tt; i < m_loc; i += T) pair_out[lo + row_base + i] = row_base + i;

  constexpr int W = kStripWaves;
  constexpr int kPitch = StripLds<S>::kPitch;
  double* xw = static_cast<double*>(lds);                    // [W][kPitch]
  double* ys = xw + StripLds<S>::kFirst;                     // [kCols] and the sum of x
  double* rx = xw;                                           // received: [teams at a time][row], [groups][cw] or [owned]
  int* seen_words = reinterpret_cast<int*>(ys + kCols + 6);  // [2]

  // (buffer loads: a row that the workgroup does not have, or a column past the last one, reads as zero,
  // with no mask and no address of its own in registers)
  StripEntries<RPT, CPT> K;
#pragma unroll
  for (int a = 0; a < RPT; ++a) {
    const bool there = W * a + tw < m_loc;
    const float* at = Kg + static_cast<long long>(row_base + (there ? W * a + tw : 0)) * pitch;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(at), 0, there ? 4 * r : 0, 0x00020000);
#pragma unroll
    for (int c = 0; c < CPT; ++c) K.set(a, c, __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, 4 * lane + 256 * c, 0, 0)));
  }
  K.forget(0, RPT);

  const double kz = exp((p.z - p.shift) / p.eps);
  const double x_init = exp(p.shift / p.eps);      // T = 0 leaves u = 0
  for (int e = tt; e <= kCols; e += T) ys[e] = e < r ? 1.0 : 0.0;
  double x_dust = x_init, y_dust = 1.0;
  double xv[kChunks];                              // lanes strip_lane8(u) (last four or fewer rows: strip_lane4(u)): row 8 ch + u
#pragma unroll
  for (int ch = 0; ch < kChunks; ++ch) xv[ch] = x_init;
  if (tt == 0) {
    ys[kCols + 2] = kz;
    ys[kCols + 3] = static_cast<double>(r);
    ys[kCols + 4] = static_cast<double>(m);
    ys[kCols + 5] = static_cast<double>(1.0f / static_cast<float>(cw));
  }
  __syncthreads();

  for (int it = 0; it < p.iters; ++it) {
    if (first) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    int fixed = kCols + 2;                             // (the image's constants are read anew: registers)
    forget_origin(fixed);
    int m_loc = rows;                                  // (and what is compared with it: else the results are held, and spilled)
    forget_scalar(m_loc);
    const double row_dust = ys[fixed] * y_dust;
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
      if (ch > 0 && 8 * W * ch >= m_loc) continue;                // no row of this chunk exists (the same for every thread)
      const bool four = ch == kChunks - 1 && kLast <= 4;       // (known when unrolled, like the bounds below)
      double q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = 0.0;
      K.forget(8 * ch, min(8 * ch + 8, RPT));
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
                q[u] = fma(static_cast<double>(K.get(8 * ch + u < RPT ? 8 * ch + u : 0, c0 + c < CPT ? c0 + c : 0)), yc[c], q[u]);
          }
      }
      if (ch == 0) forget_origin(ly);       // (else the additions are put off to where ly is needed, with all y in registers until then)
      const double sum = four ? strip_reduce4(q) : strip_reduce8(q, lane);
      const int u_own = four ? strip_row4(lane) : strip_row8(lane);
      xv[ch] = W * (8 * ch + u_own) + tw < m_loc ? rcp64(sum + row_dust) : 0.0;
      double x[8];                                               // the same in every lane (scalar registers)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (8 * ch + u < RPT) {
          x[u] = read_lane(xv[ch], four ? strip_lane4(u & 3) : strip_lane8(u));
          xs += x[u];
        }
      K.forget(8 * ch, min(8 * ch + 8, RPT));                    // (entries are widened again, not kept widened)
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        double acc = kChunks > 1 ? t[kChunks > 1 ? c : 0] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int a = 8 * ch + u;
          if (a < RPT) acc = fma(static_cast<double>(K.get(a < RPT ? a : 0, c)), x[u], acc);
        }
        if constexpr (kChunks > 1) t[c] = acc;
        else xw[tw * kPitch + 64 * c + lane] = acc;
        if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (kChunks > 1) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) xw[tw * kPitch + 64 * c + lane] = t[c];
    }
    __builtin_amdgcn_s_setprio(3);
    int te = tt;                                       // (comparisons and addresses are worked out anew: registers)
    forget_origin(te);
    if ((te & 63) < 2) xw[tw * kPitch + kCols + (te & 63)] = 0.0;
    if ((te & 63) == 0) xw[tw * kPitch + r] = xs;   // (the columns past the last one are zero: this one is the sum of x)
    int& seen_all = seen_words[it & 1];                // (two words in turn: the next write of one is a whole iteration away)
    if (te == 0) seen_all = 1;
    lds_barrier();
    // this workgroup's sums: columns 2 k and 2 k + 1 (the sum of x as column r) by thread k, k + T, ...
    const float inv_cw = static_cast<float>(ys[fixed + 3]);
    auto own_sums = [&](int e) {
      const f64x2_t* col = reinterpret_cast<const f64x2_t*>(xw + min(e, kCols));
      f64x2_t acc = col[0];
#pragma unroll
      for (int w = 1; w < W; ++w) {
        const f64x2_t v = col[w * (kPitch / 2)];
        acc[0] += v[0];
        acc[1] += v[1];
      }
      return acc;
    };
    const int sums = direct ? (it & 1) * sums_buf : 0; // (places are counted from `area`)
    const uint32_t use = (direct ? ~(it >> 1) : ~it) & 1 ? kExOdd : 0u;
    const auto ex = ex_resource(area);
    if (groups > 1 && here) {
      const int published = direct ? row : owned;
#pragma unroll 1
      for (int e = 2 * te; e < published; e += 2 * T) {
        const int o = static_cast<int>((static_cast<float>(e) + 0.5f) * inv_cw);   // e / cw
        const f64x2_t v = own_sums(e);
        ex_store2(ex, sums + (direct ? rank * row + e : (o * groups + rank) * cw + (e - o * cw)),
                  e <= r ? v[0] : 0.0, e < r ? v[1] : 0.0, use);
      }
    }
    // (while the sums travel) the dustbins' scalings from the previous y
    x_dust = ys[fixed + 1] * rcp64(ys[fixed] * (wave_sum_dpp(ly) + y_dust));
    const double col_dust = ys[fixed] * x_dust;
    bool seen = true;
    auto keep = [&](int e, double v0, double v1) {     // y (and the sum of x) of columns e and e + 1
      if (e <= r) ys[e < r ? e : kCols] = v0;
      if (e + 1 <= r) ys[e + 1 < r ? e + 1 : kCols] = v1;
    };
    auto finish = [&](int e, double sum) { return e < r ? rcp64(sum + col_dust) : sum; };
    if (groups == 1) {
      for (int e = 2 * te; e <= r; e += 2 * T) {
        const f64x2_t v = own_sums(e);
        keep(e, finish(e, v[0]), finish(e + 1, v[1]));
      }
    } else if (kMayDirect && direct) {
      // everybody's sums, added in rank order
      lds_barrier();                                   // (the waves' column sums have been read)
      seen = strip_receive(C, area + sums, groups * row, use, rx, tw, te & 63, [](int, double, double) {});
      lds_barrier();
      for (int e = 2 * te; e < row; e += 2 * T) {
        f64x2_t acc = *reinterpret_cast<const f64x2_t*>(rx + e);
        acc = f64x2_t{ex_value(acc[0]), ex_value(acc[1])};
        for (int g = 1; g < groups; ++g) {
          const f64x2_t v = *reinterpret_cast<const f64x2_t*>(rx + g * row + e);
          acc[0] += ex_value(v[0]);
          acc[1] += ex_value(v[1]);
        }
        keep(e, finish(e, acc[0]), finish(e + 1, acc[1]));
      }
    } else {
      // the others' sums of the own columns
      const int in = sums + rank * groups * cw;
      lds_barrier();                                   // (the waves' column sums have been read)
      ex_pause(groups <= kStripXcdGroups ? 0 : groups <= kStripTeams * kStripXcdGroups ? 4 : 12);
      if (own > 0) seen = strip_receive(C, area + in, groups * cw, use, rx, tw, te & 63, [](int, double, double) {});
      lds_barrier();
      // 4, 16 or 32 lanes add up two columns: about all threads at work, each on as few workgroups' as that allows
      const int yout = sums_buf + own0;
      const int wide = cw <= 16 ? 5 : cw <= 32 ? 4 : 2, lanes = 1 << wide;
      for (int k = 2 * (te >> wide); k < own; k += 2 * (T >> wide)) {
        f64x2_t acc = {0.0, 0.0};
#pragma unroll 4
        for (int g = te & (lanes - 1); g < groups; g += lanes) {
          const f64x2_t v = *reinterpret_cast<const f64x2_t*>(rx + g * cw + k);
          acc[0] += ex_value(v[0]);
          acc[1] += ex_value(v[1]);
        }
        double v0 = group_sum<2>(acc[0]), v1 = group_sum<2>(acc[1]);
        if (wide >= 4) {
          v0 += dpp_move<0x141>(v0);
          v1 += dpp_move<0x141>(v1);
          v0 += dpp_move<0x140>(v0);
          v1 += dpp_move<0x140>(v1);
        }
        if (wide == 5) {
          v0 = add_xor_lane<16>(v0);
          v1 = add_xor_lane<16>(v1);
        }
        if ((te & (lanes - 1)) == 0) ex_store2(ex, yout + k, finish(own0 + k, v0), finish(own0 + k + 1, v1), use);
      }
      ex_pause(groups <= kStripTeams * kStripXcdGroups ? 16 : 20);
      if (!strip_receive(C, area + sums_buf, owned, use, rx + StripLds<S>::kShares, tw, te & 63, keep)) seen = false;
    }
    if (!seen) seen_all = 0;
    lds_barrier();
    if (!seen_all) {                                   // a wait was given up (here or elsewhere): everybody leaves
      if (te == 0) {
        __hip_atomic_store(C.words + kStripGaveUp, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        atomicOr(C.status, RTP_DEV_SYNC_TIMEOUT);
      }
      return false;
    }
    y_dust = ys[fixed + 2] * rcp64(ys[fixed] * (ys[kCols] + x_dust));
  }
  __syncthreads();

  // ---- plan and this workgroup's best partner per column ----
  float* P = A.plan_out ? A.plan_out + po : nullptr;
  float* pv = static_cast<float*>(lds);                        // [W][kCols], where the sums were
  int* pi = reinterpret_cast<int*>(pv + W * kCols);            // [W][kCols]
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
      const int i = row_p + W * a;
      if (W * a + tw < m_loc && j < r) {
        const float v = static_cast<float>(x[a] * static_cast<double>(K.get(a, c)) * yj);
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
  if (pair_out && here) {
    for (int e = tt; e < r; e += T) {
      float bv = -1.f;
      int bi = 0x7fffffff;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float ov = pv[w * kCols + e];
        const int oi = pi[w * kCols + e];
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
      }
      if (groups == 1)
        pair_out[lo + m + e] = static_cast<float>(x_dust * ys[kCols + 2] * ys[e]) > bv ? -1 : bi;
      else
        __hip_atomic_store(keys + rank * row + e,
                           (static_cast<long long>(__float_as_int(bv)) << 32) | static_cast<unsigned>(0x7fffffff - bi),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (!strip_meet(C, counter, arrived, here, s_flag)) return false;
  if (pair_out && groups > 1) {
    // every workgroup picks the best of its share of the columns, eight lanes to a column
    for (int k = tt >> 3; k < own; k += T / 8) {
      const int e = own0 + k;
      if (e >= r) break;
      long long best = static_cast<long long>(__float_as_int(-1.f)) << 32;
      for (int g = tt & 7; g < groups; g += 8) {
        const long long key = __hip_atomic_load(keys + g * row + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        best = key > best ? key : best;
      }
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) {
        const long long other = __shfl_xor(best, o, kWave);
        best = other > best ? other : best;
      }
      if ((tt & 7) == 0)
        pair_out[lo + m + e] =
            static_cast<float>(x_dust * ys[kCols + 2] * ys[e]) > __int_as_float(static_cast<int>(best >> 32)) ? -1 : 0x7fffffff - static_cast<int>(best);
    }
  }
  return true;
}

// Slots of a launch: as many as are complete at once, and no more than have images (those that keep to an XCD: whole
// eights).
__device__ __forceinline__ int strip_slots_used(int units, int count, int cus) {
  return min(strip_slots(units, cus), units <= kStripXcdGroups ? (count + 7) / 8 * 8 : count);
}

// The images slot, slot + slots, ... of the list on the slot's `per_slot` teams; this one is `rank`.  They meet before
// each image (its exchange area cleared), and the image's at its end (the pairing keys out); `arrived`: the
// counter's total so far.  False: a wait was given up, leave the kernel.
template <typename S, bool PAIRED>
__device__ __forceinline__ bool strip_images(const StripArgs& C, int slot, int slots, int count, int rank, int per_slot,
                                             int& arrived, unsigned char* lds) {
  const SinkhornArgs& A = C.S;
  int* flag = reinterpret_cast<int*>(lds + strip_lds_of<S>()) - 2;
  // the loop's state, in LDS while an image is worked on: in registers it makes the kernels spill
  // (4512-token pages 5.75 -> 5.90 ms a call)
  int* at = reinterpret_cast<int*>(lds + strip_lds_of<S>()) - 12;
  // (Once round.  Without a loop that the compiler takes for one, it keeps entries of the matrix in two places and moves
  // them from one to the other each iteration.)
  for (int again = 0;;) {
    for (int k = slot; k < count; k += slots) {
      const int b = C.words[kStripList - (S::kShape - 1) * kStripShapeWords + C.words[kStripFirst] + k];
      const int n = A.offsets[b + 1] - A.offsets[b];
      const int m = min(max(A.keep[b], 0), max(n, 0)), r = max(n, 0) - m;
      // (every workgroup of the slot takes the same decisions: they read the same words)
      if (m <= 0 || r <= 0 || sinkhorn_variant(m, r, A.p.mode) != kVariantStrip) continue;
      if (!plan_fits(A.plan_offsets[b], m, r, A.plan_cap)) continue;
      const int groups = strip_teams(S::kShape, m, A.p.mode);   // (at most per_slot: the list's builder has counted)
      int32_t* counter = C.words + (PAIRED ? kStripLast : kStripCounters + slot);
      strip_clear<S>(C, b, rank);
      arrived += per_slot;
      if (!strip_meet(C, counter, arrived, true, flag)) return false;
      arrived += groups;
      if ((PAIRED ? rank & ~1 : rank) < groups) {                // (a workgroup's two teams decide alike)
        if (strip_thread() == 0) {
          at[0] = slot, at[1] = k, at[2] = arrived, at[3] = slots, at[4] = count, at[5] = per_slot, at[6] = rank;
        }
        if (!sinkhorn_strip_image<S, PAIRED>(C, b, rank, groups, counter, arrived, 2 * slot < slots, lds, flag)) return false;
        slot = __builtin_amdgcn_readfirstlane(at[0]);
        k = __builtin_amdgcn_readfirstlane(at[1]);
        arrived = __builtin_amdgcn_readfirstlane(at[2]);
        slots = __builtin_amdgcn_readfirstlane(at[3]);
        count = __builtin_amdgcn_readfirstlane(at[4]);
        per_slot = __builtin_amdgcn_readfirstlane(at[5]);
        rank = __builtin_amdgcn_readfirstlane(at[6]);
      } else if (!strip_meet(C, counter, arrived, false, flag)) {
        return false;
      }
    }
    forget_scalar(again);
    if (!again) return true;
  }
}

// Slot s takes images s, s + slots, ... of the list.  The slot's arrival counter runs on through all
// its meetings, the first of which is when the slot is complete.
template <typename S>
__global__ __launch_bounds__(kStripThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sinkhorn_strips(StripArgs C) {
  __shared__ __align__(16) unsigned char lds[strip_lds_of<S>()];
  int* flag = reinterpret_cast<int*>(lds + strip_lds_of<S>()) - 2;
  // (all waves or none: a slot that gives up writes the word while others may be starting)
  if (threadIdx.x == 0) *flag = C.status[0];
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*flag)) return;
  const int count = C.words[kStripCount];
  if (count == 0) return;
  const int units = C.words[kStripTop], per_slot = kStripTeams * units;
  const int block = blockIdx.x;
  const int slots = strip_slots_used(units, count, C.cus);
  int slot, rank;
  if (units <= kStripXcdGroups) {                   // one XCD per slot
    slot = (block & 7) * (slots >> 3) + (block >> 3) / per_slot;
    rank = (block >> 3) % per_slot;
  } else {
    slot = block / per_slot;
    rank = block % per_slot;
  }
  if (block >= slots * per_slot || slot >= count) return;
  if (!strip_complete(C.words + kStripCounters + slot, per_slot, C.form_limit, flag)) return;
  int arrived = per_slot;
  strip_images<S, false>(C, slot, slots, count, rank, per_slot, arrived, lds);
}

// The slots given up, one after another, with a counter of their own.  Behind k_sinkhorn_strips on its stream, with as
// many workgroups as a slot has compute units; none given up, the usual case, costs a call 1 to 4 us.
template <typename S>
__global__ __launch_bounds__(kStripTeams * kStripThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sinkhorn_strips_left(StripArgs C) {
  constexpr int kTeamLds = (strip_lds_of<S>() + 15) & ~15;
  __shared__ __align__(16) unsigned char lds[kStripTeams * kTeamLds];
  int* flag = reinterpret_cast<int*>(lds);
  // (all waves or none: one that gives up writes the word while others may be starting)
  if (threadIdx.x == 0) *flag = C.status[0];
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*flag)) return;
  const int count = C.words[kStripCount];
  const int units = C.words[kStripTop], per_slot = kStripTeams * units;
  if (count == 0 || static_cast<int>(blockIdx.x) >= units) return;
  const int slots = strip_slots_used(units, count, C.cus), with_images = min(slots, count);
  auto left = [&](int slot) {
    return (__hip_atomic_load(C.words + kStripCounters + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kStripGivenUp) != 0;
  };
  if (!__syncthreads_or(static_cast<int>(threadIdx.x) < with_images && left(threadIdx.x))) return;
  const int team = __builtin_amdgcn_readfirstlane(threadIdx.x / kStripThreads);
  int arrived = 0;
  for (int slot = 0; slot < with_images; ++slot)
    if (left(slot) && !strip_images<S, true>(C, slot, slots, count, kStripTeams * blockIdx.x + team, per_slot, arrived, lds + team * kTeamLds))
      return;
}

}  // namespace rtp
