// select.hip — support selection and CSR schedule construction on gfx950.
//
// Paper Section 5.1, eq. (block_working_set): per query block, the smallest
// set of admissible key blocks whose mass reaches the threshold, i.e. the
// heaviest k* blocks with k* the first prefix of the descending order that
// reaches tau * total.  The schedule is a device-resident CSR (Appendix B,
// "Sparse-kernel implementation") plus a longest-support-first row order.
//
//   select_rows_kernel   one wave per row: the cut of the masses ordered by
//                        (mass desc, block asc) and summed in that order in
//                        fp64, forced blocks added, a bitmask and a count
//   csr_kernel           counts -> row_ptr (exclusive scan), bitmask ->
//                        ascending col_idx, and per (batch, head) its rows by
//                        count descending (ties by row id)
//
// The paper's own working set (Section 5.1, eq. block_working_set) is the
// union over the discovery window of per-step sets B_q^(t, eta).  For it the
// per-row kernel runs on one step's masses with no forced blocks and leaves
// the step's bitmask with the caller; union_rows_kernel ORs any number of
// such masks, adds the forced blocks, and feeds the same csr kernel.  Two diagnostics close the file: the (intersection, union)
// sizes of two masks (the adjacent rolling-set Jaccard of Appendix C,
// "Stability of the Deployed Working Set") and the attention mass a support
// retains from one step's block masses (Section 7.1 and Appendix B, the
// retained future full-attention mass).
#include <algorithm>
#include <mutex>

#include "csr_entries.hpp"
#include "wise.h"
#include "wise_device.hpp"
#include "wise_kernels.hpp"

namespace wise {

constexpr int kSelWaves = 4;        // rows per work-group in the per-row kernels

// Orderable 32-bit image of a float: unsigned order == float order.
__device__ __forceinline__ uint32_t float_key(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Order LDS traffic within one wave (each wave of the per-row kernel works on
// its own row and its own LDS, so the group needs no barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Lane l's x from another lane by DPP, 0 where the pattern gives none.
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, kCtrl, kRows, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), kCtrl, kRows, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Inclusive sums over the wave's lanes, on the VALU (a shuffle per step goes
// through LDS): shifts within rows of 16, then the row ends broadcast.
__device__ __forceinline__ double wave_scan(double x) {
  x += dpp_f64<0x111, 0xF>(x);   // row_shr 1
  x += dpp_f64<0x112, 0xF>(x);
  x += dpp_f64<0x114, 0xF>(x);
  x += dpp_f64<0x118, 0xF>(x);
  x += dpp_f64<0x142, 0xA>(x);   // row_bcast 15 into rows 1 and 3
  x += dpp_f64<0x143, 0xC>(x);   // row_bcast 31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ double read_lane(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double wave_sum(double x) { return read_lane(wave_scan(x), 63); }

// LDS bytes of one row's wave: 256 digit sums, or nb keys and nb sorted masses.
constexpr int kDigitBins = 256;
__host__ __device__ constexpr size_t select_row_lds(int nb) {
  return (size_t)(2 * nb > kDigitBins ? 2 * nb : kDigitBins) * 8;
}

// k* of one row by definition: rank every candidate, add the ordered masses
// one by one in fp64.  keys[e] / rank[e]: candidate lane + 64 e.
template <int E>
__device__ int cut_by_rank(const float x[E], int cnt, double tau, uint64_t* lds, int nb, int lane,
                           int rank[E]) {
  uint64_t* keys = lds;                                 // [nb] sort keys, later prefixes
  double* sv = (double*)(lds + nb);                     // [nb] masses in sorted order
  uint64_t key[E];
  // composite keys: mass descending, then block index ascending
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int b = lane + 64 * e;
    key[e] = 0;
    rank[e] = 0;
    if (b < cnt) {
      key[e] = ((uint64_t)float_key(x[e]) << 32) | (uint32_t)(~(uint32_t)b);
      keys[b] = key[e];
    }
  }
  wave_sync();
  // rank = number of candidates ordered before this one
  for (int c = 0; c < cnt; ++c) {
    const uint64_t kc = keys[c];
#pragma unroll
    for (int e = 0; e < E; ++e) rank[e] += (kc > key[e]) ? 1 : 0;
  }
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (lane + 64 * e < cnt) sv[rank[e]] = (double)x[e];
  wave_sync();
  // sequential fp64 prefix sums in sorted order (identical in every lane)
  double* pre = (double*)keys;
  double run = 0.0;
  for (int r = 0; r < cnt; ++r) {
    run += sv[r];
    if (lane == 0) pre[r] = run;
  }
  wave_sync();
  // k* = min{k >= 0 : c_k >= tau * total}, c_0 = 0
  const double thr = tau * run;
  int kstar = cnt;
  if (thr <= 0.0) {
    kstar = 0;
  } else {
    for (int r = lane; r < cnt; r += 64)
      if (pre[r] >= thr) { kstar = min(kstar, r + 1); break; }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) kstar = min(kstar, __shfl_xor(kstar, off, 64));
  }
  wave_sync();
  return kstar;
}

// The same cut without sorting, for the masses attention gives.  fp64 sums of
// fp32 masses are exact, whatever their order, while every mass is a multiple
// of 2^-53 times a power of two above their sum: so for the heavy masses
// (exponent at most 28 below the total's) the ordered prefix sums are plain
// sums, and the cut is found digit by digit of the mass bits from sums per digit.  The light
// masses only follow the heavy ones in the order; they matter for the total,
// which the ordered sum rounds at each of up to 1024 of them: it is within 1050
// roundings (2^-53 each) of a sum in any order, and a cut that is the same at
// both ends of that range (here 2^-42) is the cut.  Returns false (nothing decided) for
// negative, infinite or NaN masses, a cut among the light ones, or one that
// the range leaves open: cut_by_rank then does the row.  On success sel[e] tells
// whether candidate lane + 64 e is among the first k*.
// Bound by instruction issue: about four passes of E LDS adds and one 64-lane
// scan, where ranking takes nb / 2 comparisons per candidate and a serial sum.
// wise_select_step, every row ranked / so: 28160 rows of 128 blocks 69.7 / 18.7
// us on uniform masses, 69.6 / 12.8 on one heavy mass and light ones (70.4
// where such rows were ranked to round their total); 8192 rows of 1024 blocks
// 481 / 47 and 480 / 26.
template <int E>
__device__ bool cut_by_digits(const float x[E], int cnt, double tau, uint64_t* lds, int lane,
                              bool sel[E]) {
  uint32_t u[E];
  bool plain = true;
  double part = 0.0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    u[e] = lane + 64 * e < cnt ? __builtin_bit_cast(uint32_t, x[e]) : 0u;
    plain = plain && u[e] < 0x7f800000u;
    part += (double)__builtin_bit_cast(float, u[e]);
    sel[e] = false;
  }
  if (__builtin_amdgcn_ballot_w64(!plain)) return false;
  const double about = wave_sum(part);                  // the total but for its rounding
  if (about == 0.0) return true;                        // k* = 0
  // about < 2^(et + 1): masses with biased exponent >= et - 29 + 127 are heavy.
  const int et = (int)((__builtin_bit_cast(uint64_t, about) >> 52) & 0x7ff) - 1023;
  const int e0 = max(et + 127 - 28, 0);
  const uint32_t heavy = (uint32_t)e0 << 23;            // smallest heavy mass bits
  double hp = 0.0;
  bool light = false;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (u[e] >= heavy) hp += (double)__builtin_bit_cast(float, u[e]);
    else light = light || u[e] > 0;
  }
  const double big = wave_sum(hp);
  double low = tau * big, thr = low;                    // the threshold is in low .. thr
  if (__builtin_amdgcn_ballot_w64(light)) {
    low = tau * (about * (1.0 - 0x1p-42));
    thr = tau * (about * (1.0 + 0x1p-42));
  }
  if (thr > big) return false;
  double* bins = (double*)lds;
  uint32_t head = 0;                                    // leading bits of the cut's mass
  double above = 0.0;                                   // sum of all masses with larger leading bits
  uint32_t cut = 0;
  bool found = false;
#pragma unroll
  for (int pass = 0; pass < 4 && !found; ++pass) {
    constexpr int kShift[4] = {23, 15, 7, 0};
    const int shift = kShift[pass], width = pass < 3 ? 8 : 7;
    const uint32_t mask = (1u << width) - 1u;
    double2* own4 = (double2*)bins + 2 * (63 - lane);     // digits 252 - 4 l .. 255 - 4 l
    own4[0] = own4[1] = double2{0.0, 0.0};
    wave_sync();
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (u[e] >= heavy && u[e] > 0 && (u[e] >> shift >> width) == head)
        __hip_atomic_fetch_add(&bins[(u[e] >> shift) & mask], (double)__builtin_bit_cast(float, u[e]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    wave_sync();
    // lane l holds the four digits 255 - 4 l downwards
    const double2 low2 = own4[0], high2 = own4[1];
    wave_sync();
    const double d[4] = {high2.y, high2.x, low2.y, low2.x};
    const double own = d[0] + d[1] + d[2] + d[3];
    const double c = wave_scan(own);
    const uint64_t hit = __builtin_amdgcn_ballot_w64(above + c >= thr);
    const int first = __builtin_ctzll(hit);             // thr <= big: some lane reaches it
    double before = above + (c - own);
    int digit = 0;
    bool done = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!done && before + d[i] >= thr) {
        digit = kDigitBins - 1 - 4 * lane - i;
        done = true;
      }
      if (!done) before += d[i];
    }
    digit = __builtin_amdgcn_readlane(digit, first);
    above = read_lane(before, first);
    head = (head << width) | (uint32_t)digit;
    int members = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint64_t b = __builtin_amdgcn_ballot_w64(u[e] > 0 && (u[e] >> shift) == head);
      members += __builtin_popcountll(b);
      if (b) cut = __builtin_amdgcn_readlane(u[e], __builtin_ctzll(b));
    }
    found = members == 1 || pass == 3;                  // all members equal `cut`
  }
  // Everything heavier, and of the masses equal to the cut as many, lowest
  // blocks first, as reach the threshold.
  const double val = (double)__builtin_bit_cast(float, cut);
  int need = 0;
  double shorter = above;                               // the sum without the last of them
  for (double c = above; c < thr; c += val) {
    shorter = c;
    ++need;
  }
  if (shorter >= low) return false;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint64_t b = __builtin_amdgcn_ballot_w64(u[e] == cut);
    const int ahead = __builtin_popcountll(b & ((1ull << lane) - 1ull));
    sel[e] = u[e] > cut || (u[e] == cut && ahead < need);
    need -= min(need, __builtin_popcountll(b));
  }
  return true;
}

// Candidates up to which a row is ranked at once: that many comparisons cost
// less than the digits' passes.  wise_select_step, digits / ranked: 4096 heads
// of 8 blocks 14.3 / 12.3 us, 2048 of 12 11.5 / 10.2, 2048 of 16 15.3 / 15.9
// (all rows digits / rows of up to 8, 12 and 16 ranked).
constexpr int kRankRows = 12;

// E = candidates per lane (ceil(nb / 64) rounded up to a power of two).  One
// wave per row, four rows per group, no barriers.
template <int E>
__global__ void __launch_bounds__(kSelWaves * 64)
select_rows_kernel(const float* __restrict__ acc, int rows, int nb, double tau, uint32_t flags,
                   int32_t* __restrict__ counts, uint64_t* __restrict__ masks, int words) {
  extern __shared__ __attribute__((aligned(16))) uint64_t sel_smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * kSelWaves + wave;
  if (row >= rows) return;
  uint64_t* lds = sel_smem + (size_t)wave * (select_row_lds(nb) / 8);
  const int qb = row % nb;
  const int cnt = qb + 1;
  const float* v = acc + (size_t)row * nb;
  float x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) x[e] = lane + 64 * e < cnt ? v[lane + 64 * e] : 0.f;
  bool sel[E];
  if (cnt <= kRankRows || !cut_by_digits<E>(x, cnt, tau, lds, lane, sel)) {
    int rank[E];
    const int kstar = cut_by_rank<E>(x, cnt, tau, lds, nb, lane, rank);
#pragma unroll
    for (int e = 0; e < E; ++e) sel[e] = rank[e] < kstar;
  }
  // selection bitmask, forced blocks, empty -> diagonal
  int total = 0;
  uint64_t mword[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int b = lane + 64 * e;
    bool s = false;
    if (b < cnt) s = sel[e] || (b == 0 && (flags & 1u)) || (b == qb && (flags & 2u));
    mword[e] = __builtin_amdgcn_ballot_w64(s);
    total += __builtin_popcountll(mword[e]);
  }
  if (total == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e == qb >> 6) mword[e] |= 1ull << (qb & 63);
    total = 1;
  }
  if (lane == 0) {
    if (counts != nullptr) counts[row] = total;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e < words) masks[(size_t)row * words + e] = mword[e];
  }
}

// Inclusive scan of one value per thread over a 1024-thread block.
__device__ __forceinline__ int block_scan_1024(int x, int* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  if (wave == 0) {
    int w = lane < 16 ? wsum[lane] : 0;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
      const int y = __shfl_up(w, off, 64);
      if (lane >= off) w += y;
    }
    if (lane < 16) wsum[lane] = w;
  }
  __syncthreads();
  const int add = wave > 0 ? wsum[wave - 1] : 0;
  __syncthreads();
  return x + add;
}

// row_ptr[0] = 0, row_ptr[r+1] = counts[0] + ... + counts[r], by one group.
// Only where the csr groups would read too much (kSumReads).
__global__ void __launch_bounds__(1024)
scan_kernel(const int32_t* __restrict__ counts, int rows, int32_t* __restrict__ row_ptr) {
  __shared__ int wsum[16];
  __shared__ int carry;
  if (threadIdx.x == 0) {
    carry = 0;
    row_ptr[0] = 0;
  }
  __syncthreads();
  for (int base = 0; base < rows; base += 1024) {
    const int r = base + threadIdx.x;
    const int x = r < rows ? counts[r] : 0;
    const int inc = block_scan_1024(x, wsum);
    const int c0 = carry;
    if (r < rows) row_ptr[r + 1] = c0 + inc;
    __syncthreads();
    if (threadIdx.x == 1023) carry = c0 + inc;
    __syncthreads();
  }
}

// Counts and bitmasks -> row_ptr, col_idx and row order.  One group takes
// kCsrRows rows of one head, or as many whole heads as kCsrRows rows hold at
// most (per of the bh heads; grid: groups of heads x chunks of a head):
//   its first entry   the sum of every earlier row's count (read again by each
//                     group, from L2: kSumReads), or row_ptr
//                     where the scan has run
//   row_ptr           the scan of its own rows' counts from there
//   col_idx           one wave per row at a time: set bits of the mask, ascending
//   order             row r of a head lands at rank(r) = #{rows with a larger
//                     count} + #{earlier rows with the same count}, eight
//                     lanes per row over the head's counts in LDS
// Latency bound (6 us for 28160 rows, where a one-group scan, a scatter and an
// order kernel took about 45); 16 waves per group put eight rows' masks of
// each wave in flight at once.  Short heads share a group because a group's
// own cost, 1024 threads and the sum before it, does not shrink with its rows:
// CSR from masks, a group per head -> shared: 4096 heads of 8 blocks 29.1 ->
// 9.1 us, 8192 of 16 151 -> 24.4 us (the three kernels: 39.9 and 135).
constexpr int kCsrRows = 128;

template <bool kScanned>
__global__ void __launch_bounds__(1024)
csr_kernel(const int32_t* __restrict__ counts, const uint64_t* __restrict__ masks, int bh, int per,
           int nb, int words, int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx,
           int32_t* __restrict__ order) {
  __shared__ int head[1024];             // counts of the group's heads: max(kCsrRows, nb) at most
  __shared__ int start[kCsrRows];
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h0 = blockIdx.x * per, base = h0 * nb;         // the group's first head and its first row
  const int rows = min(per, bh - h0) * nb;                 // of its heads
  const int r0 = blockIdx.y * kCsrRows, nr = min(kCsrRows, rows - r0);
  const int first = base + r0;
  // Up to eight rows' masks per wave, loaded before the sums they wait for.
  constexpr int kRowsPerWave = kCsrRows / 16;
  uint64_t m[kRowsPerWave];
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    const int r = wave + 16 * i;
    m[i] = r < nr && lane < words ? masks[(size_t)(first + r) * words + lane] : 0ull;
  }
  if (tid < rows) head[tid] = counts[base + tid];
  int before = 0;
  if constexpr (!kScanned) {
    const int4* c4 = (const int4*)counts;                  // 256-byte aligned
    const int n4 = first >> 2;
    int sum = 0;
#pragma unroll 4
    for (int i = tid; i < n4; i += 1024) {
      const int4 c = c4[i];
      sum += c.x + c.y + c.z + c.w;
    }
    if (tid < (first & 3)) sum += counts[4 * n4 + tid];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == 0) wsum[wave] = sum;
  }
  __syncthreads();
  if constexpr (kScanned) {
    before = row_ptr[first];
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) before += wsum[i];
  }
  // Exclusive scan of the chunk's counts: two waves, the second adds the
  // first's total.
  if (tid < kCsrRows) {
    const int x = tid < nr ? head[r0 + tid] : 0;
    int inc = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(inc, off, 64);
      if (lane >= off) inc += y;
    }
    if (wave == 1) {
      int low = head[r0 + lane];                           // rows 0 .. 63 of the chunk: nr > 64 or unused
      if (r0 + lane >= rows) low = 0;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) low += __shfl_xor(low, off, 64);
      inc += low;
    }
    if (tid < nr) {
      start[tid] = before + inc - x;
      if constexpr (!kScanned) row_ptr[first + tid + 1] = before + inc;
    }
  }
  if (!kScanned && first == 0 && tid == 0) row_ptr[0] = 0;
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    const int r = wave + 16 * i;
    if (r >= nr) break;
    int pos = start[r];
    for (int e = 0; e < words; ++e) {
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)m[i], e);
      const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(m[i] >> 32), e);
      const uint64_t w = ((uint64_t)hi << 32) | lo;
      if ((w >> lane) & 1ull) col_idx[pos + __builtin_popcountll(w & below)] = 64 * e + lane;
      pos += __builtin_popcountll(w);
    }
  }
  if (order != nullptr) {
    const int r = r0 + (tid >> 3), part = tid & 7;         // row of the group's heads, eighth of its head
    const bool live = (tid >> 3) < nr;
    const int h = per > 1 ? r / nb * nb : 0;               // its head's first row
    const int* own = head + h;
    const int at = r - h, c = live ? own[at] : 0;
    int rank = 0;
    if (live)
      for (int t = part; t < nb; t += 8) {
        const int ct = own[t];
        rank += (ct > c || (ct == c && t < at)) ? 1 : 0;
      }
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1) rank += __shfl_xor(rank, off, 64);
    if (live && part == 0) order[base + h + rank] = base + r;
  }
}

// Workspace layout: counts | masks, each 256-B aligned.
struct SelectWs {
  size_t counts, masks, total;
  int words;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int mask_words(const Dims& s) { return (s.nb + 63) / 64; }

static SelectWs select_ws(const Dims& s) {
  SelectWs w;
  const size_t rows = (size_t)s.bh * s.nb;
  w.words = mask_words(s);
  w.counts = 0;
  w.masks = align256(w.counts + rows * 4);
  w.total = align256(w.masks + rows * w.words * 8);
  return w;
}

size_t select_workspace_bytes(const Dims& s) { return select_ws(s).total; }

// HIP refuses a grid of 2^32 threads or more in one dimension.  The kernels of
// a call read what the ones before them wrote (the CSR kernel writes col_idx
// where the counts say), so a call launches all of its kernels or none.
static bool grid_fits(int64_t groups, int threads) { return groups * threads < (int64_t)1 << 32; }

static int64_t row_groups(const Dims& s) { return ((int64_t)s.bh * s.nb + kSelWaves - 1) / kSelWaves; }

// Per-row selection of every row: counts (may be null) and bitmasks.
static void launch_rows(const Dims& s, const float* acc, float tau, uint32_t flags,
                        int32_t* counts, uint64_t* masks, hipStream_t st) {
  const int rows = s.bh * s.nb, words = mask_words(s);
  const size_t smem = kSelWaves * select_row_lds(s.nb);
  const dim3 sg((unsigned)row_groups(s)), sb(kSelWaves * 64);
  const double dtau = (double)tau;
  if (s.nb <= 64)
    hipLaunchKernelGGL(select_rows_kernel<1>, sg, sb, smem, st, acc, rows, s.nb, dtau, flags, counts, masks, words);
  else if (s.nb <= 128)
    hipLaunchKernelGGL(select_rows_kernel<2>, sg, sb, smem, st, acc, rows, s.nb, dtau, flags, counts, masks, words);
  else if (s.nb <= 256)
    hipLaunchKernelGGL(select_rows_kernel<4>, sg, sb, smem, st, acc, rows, s.nb, dtau, flags, counts, masks, words);
  else if (s.nb <= 512)
    hipLaunchKernelGGL(select_rows_kernel<8>, sg, sb, smem, st, acc, rows, s.nb, dtau, flags, counts, masks, words);
  else
    hipLaunchKernelGGL(select_rows_kernel<16>, sg, sb, smem, st, acc, rows, s.nb, dtau, flags, counts, masks, words);
}

// counts + masks (in the workspace) -> row_ptr, col_idx, row_order.
// Each csr group adds up the counts before its rows itself while all groups
// together read little, groups x rows / 2 counts from L2; past that one group
// scans them first, 0.95 us per 1024 rows.  Both ways, CSR from masks: 131072
// rows in 1024 groups (2^26 reads) 29 against 146 us, 1048576 in 8192 (2^32)
// 553 against 1000, in 16256 groups of 129-block heads (2^33) 1071 against 1097.
constexpr int64_t kSumReads = (int64_t)1 << 33;

// While the heads are fewer than the 1024-thread groups the chip holds, each
// has a group of its own: its rows then share no wave.
constexpr int kCsrGroups = 512;

struct CsrGrid {
  int per;                                              // heads per group
  int64_t groups;                                       // x; the chunks of a head in y
  int chunks;
};
static CsrGrid csr_grid(const Dims& s) {
  const int fit = s.nb < kCsrRows ? kCsrRows / s.nb : 1;
  const int per = (int)std::min<int64_t>(fit, ((int64_t)s.bh + kCsrGroups - 1) / kCsrGroups);
  return {per, ((int64_t)s.bh + per - 1) / per, (s.nb + kCsrRows - 1) / kCsrRows};
}
static bool csr_fits(const Dims& s) { return grid_fits(csr_grid(s).groups, 1024); }

static void launch_csr(const Dims& s, const int32_t* counts, const uint64_t* masks,
                       int32_t* row_ptr, int32_t* col_idx, int32_t* row_order, hipStream_t st) {
  const int rows = s.bh * s.nb;
  const CsrGrid g = csr_grid(s);
  const dim3 grid((unsigned)g.groups, g.chunks);
  if (g.groups * g.chunks * rows / 2 <= kSumReads) {
    hipLaunchKernelGGL(csr_kernel<false>, grid, dim3(1024), 0, st, counts, masks, s.bh, g.per, s.nb,
                       mask_words(s), row_ptr, col_idx, row_order);
  } else {
    hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, st, counts, rows, row_ptr);
    hipLaunchKernelGGL(csr_kernel<true>, grid, dim3(1024), 0, st, counts, masks, s.bh, g.per, s.nb,
                       mask_words(s), row_ptr, col_idx, row_order);
  }
}

hipError_t launch_select(const Dims& s, const float* acc, float tau, uint32_t flags,
                         int32_t* row_ptr, int32_t* col_idx, int32_t* row_order, void* ws,
                         hipStream_t st) {
  if (!grid_fits(row_groups(s), kSelWaves * 64) || !csr_fits(s)) return hipErrorInvalidConfiguration;
  const SelectWs w = select_ws(s);
  char* base = (char*)ws;
  auto* counts = (int32_t*)(base + w.counts);
  auto* masks = (uint64_t*)(base + w.masks);
  launch_rows(s, acc, tau, flags, counts, masks, st);
  launch_csr(s, counts, masks, row_ptr, col_idx, row_order, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Selection with no caller workspace (wise_select_support_noalloc): the
// per-row counts and bitmasks live in `scratch`, a file-scope device array of
// WISE_NOALLOC_SCRATCH_BYTES that every GPU the library runs on holds until
// the process ends.  In host code `scratch` names a host-side stand-in, not
// device memory, so kernels only ever receive the address the runtime
// reports for the current device, looked up once per device.  Every row's
// count and mask words are written before they are read, so nothing in the
// array needs clearing; calls that overlap on one device share it and race.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[WISE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static void* scratch_addr[kMaxDevices];

static hipError_t device_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (scratch_addr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    scratch_addr[dev] = p;
  }
  *out = scratch_addr[dev];
  return hipSuccess;
}

hipError_t launch_select_noalloc(const Dims& s, const float* acc, float tau, uint32_t flags,
                                 int32_t* row_ptr, int32_t* col_idx, int32_t* row_order,
                                 hipStream_t st) {
  if (select_workspace_bytes(s) > (size_t)WISE_NOALLOC_SCRATCH_BYTES) return hipErrorInvalidValue;
  void* ws = nullptr;
  const hipError_t e = device_scratch(&ws);
  if (e != hipSuccess) return e;
  return launch_select(s, acc, tau, flags, row_ptr, col_idx, row_order, ws, st);
}

// ---------------------------------------------------------------------------
// Temporal union of per-step supports
// ---------------------------------------------------------------------------

hipError_t launch_select_step(const Dims& s, const float* r, float tau, uint64_t* mask,
                              hipStream_t st) {
  launch_rows(s, r, tau, 0u, nullptr, mask, st);
  return hipGetLastError();
}

constexpr int kMaskThreads = 256;

// One thread per row: OR of the row's words over every mask, bits past the
// diagonal dropped, forced blocks added, an empty row given its diagonal.
__global__ void __launch_bounds__(kMaskThreads)
union_rows_kernel(const uint64_t* __restrict__ masks, int n_masks, size_t slab, int rows, int nb,
                  int words, uint32_t flags, int32_t* __restrict__ counts,
                  uint64_t* __restrict__ out) {
  const int row = blockIdx.x * kMaskThreads + threadIdx.x;
  if (row >= rows) return;
  const int qb = row % nb;
  const size_t base = (size_t)row * words;
  int total = 0;
  for (int w = 0; w < words; ++w) {
    uint64_t m = 0;
    for (int i = 0; i < n_masks; ++i) m |= masks[(size_t)i * slab + base + w];
    const int lo = 64 * w;
    const uint64_t keep = qb < lo ? 0ull : (qb - lo >= 63 ? ~0ull : (~0ull >> (63 - (qb - lo))));
    m &= keep;
    if (w == 0 && (flags & 1u)) m |= 1ull;
    if (w == (qb >> 6) && (flags & 2u)) m |= 1ull << (qb & 63);
    out[base + w] = m;
    total += __builtin_popcountll(m);
  }
  if (total == 0) {
    out[base + (qb >> 6)] = 1ull << (qb & 63);
    total = 1;
  }
  counts[row] = total;
}

hipError_t launch_support_from_masks(const Dims& s, const uint64_t* masks, int n_masks,
                                     uint32_t flags, int32_t* row_ptr, int32_t* col_idx,
                                     int32_t* row_order, void* ws, hipStream_t st) {
  const int64_t groups = ((int64_t)s.bh * s.nb + kMaskThreads - 1) / kMaskThreads;
  if (!grid_fits(groups, kMaskThreads) || !csr_fits(s)) return hipErrorInvalidConfiguration;
  const SelectWs w = select_ws(s);
  char* base = (char*)ws;
  auto* counts = (int32_t*)(base + w.counts);
  auto* umask = (uint64_t*)(base + w.masks);
  const int rows = s.bh * s.nb;
  const size_t slab = (size_t)rows * w.words;
  hipLaunchKernelGGL(union_rows_kernel, dim3((unsigned)groups), dim3(kMaskThreads), 0, st, masks,
                     n_masks, slab, rows, s.nb, w.words, flags, counts, umask);
  launch_csr(s, counts, umask, row_ptr, col_idx, row_order, st);
  return hipGetLastError();
}

// out[x] = OR over i of masks[i * slab + x]; out may be one of the masks.
__global__ void __launch_bounds__(kMaskThreads)
mask_union_kernel(const uint64_t* masks, int n_masks, size_t slab, uint64_t* out) {
  for (size_t x = (size_t)blockIdx.x * kMaskThreads + threadIdx.x; x < slab;
       x += (size_t)gridDim.x * kMaskThreads) {
    uint64_t m = 0;
    for (int i = 0; i < n_masks; ++i) m |= masks[(size_t)i * slab + x];
    out[x] = m;
  }
}

hipError_t launch_mask_union(const Dims& s, const uint64_t* masks, int n_masks, uint64_t* out,
                             hipStream_t st) {
  const size_t slab = (size_t)s.bh * s.nb * mask_words(s);
  const size_t blocks = (slab + kMaskThreads - 1) / kMaskThreads;
  hipLaunchKernelGGL(mask_union_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)),
                     dim3(kMaskThreads), 0, st, masks, n_masks, slab, out);
  return hipGetLastError();
}

// Sum over a 1024-thread block; the result is valid in thread 0.
template <typename T>
__device__ __forceinline__ T block_sum_1024(T x, T* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  if (lane == 0) wsum[wave] = x;
  __syncthreads();
  T t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < 16; ++i) t += wsum[i];
  return t;
}

// counts[0] = |A & B|, counts[1] = |A | B| (set bits), one work-group.
__global__ void __launch_bounds__(1024)
mask_overlap_kernel(const uint64_t* __restrict__ a, const uint64_t* __restrict__ b, size_t slab,
                    int64_t* __restrict__ counts) {
  __shared__ long long wsum[16];
  long long inter = 0, uni = 0;
  for (size_t x = threadIdx.x; x < slab; x += 1024) {
    const uint64_t p = a[x], q = b[x];
    inter += __builtin_popcountll(p & q);
    uni += __builtin_popcountll(p | q);
  }
  const long long ti = block_sum_1024(inter, wsum);
  __syncthreads();
  const long long tu = block_sum_1024(uni, wsum);
  if (threadIdx.x == 0) {
    counts[0] = ti;
    counts[1] = tu;
  }
}

hipError_t launch_mask_overlap(const Dims& s, const uint64_t* a, const uint64_t* b,
                               int64_t* counts, hipStream_t st) {
  const size_t slab = (size_t)s.bh * s.nb * mask_words(s);
  hipLaunchKernelGGL(mask_overlap_kernel, dim3(1), dim3(1024), 0, st, a, b, slab, counts);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Retained attention mass of a support
// ---------------------------------------------------------------------------

// One wave per row: row_mass[row] = (sum of r over the row's CSR blocks
// kb <= qb, sum of r over kb <= qb), in fp64, lane-strided then a fixed
// butterfly, so the result is bitwise reproducible.
__global__ void __launch_bounds__(kSelWaves * 64)
row_mass_kernel(const float* __restrict__ r, const int32_t* __restrict__ row_ptr,
                const int32_t* __restrict__ col_idx, int rows, int nb,
                double* __restrict__ row_mass) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kSelWaves + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int qb = row % nb;
  const float* v = r + (size_t)row * nb;
  double inside = 0.0, total = 0.0;
  for (int kb = lane; kb <= qb; kb += 64) total += (double)v[kb];
  for (Entries e(row_ptr[row], row_ptr[row + 1]); e.holds(lane); e.advance(64)) {
    const int kb = col_idx[e.at + lane];
    if (kb >= 0 && kb <= qb) inside += (double)v[kb];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    inside += __shfl_xor(inside, off, 64);
    total += __shfl_xor(total, off, 64);
  }
  if (lane == 0) {
    row_mass[2 * (size_t)row] = inside;
    row_mass[2 * (size_t)row + 1] = total;
  }
}

__global__ void __launch_bounds__(1024)
mass_total_kernel(const double* __restrict__ row_mass, int rows, double* __restrict__ totals) {
  __shared__ double wsum[16];
  double inside = 0.0, total = 0.0;
  for (int x = threadIdx.x; x < rows; x += 1024) {
    inside += row_mass[2 * (size_t)x];
    total += row_mass[2 * (size_t)x + 1];
  }
  const double ti = block_sum_1024(inside, wsum);
  __syncthreads();
  const double tt = block_sum_1024(total, wsum);
  if (threadIdx.x == 0) {
    totals[0] = ti;
    totals[1] = tt;
  }
}

hipError_t launch_support_mass(const Dims& s, const float* r, const int32_t* row_ptr,
                               const int32_t* col_idx, double* row_mass, double* totals,
                               hipStream_t st) {
  const int rows = s.bh * s.nb;
  if (!grid_fits(row_groups(s), kSelWaves * 64)) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(row_mass_kernel, dim3((unsigned)row_groups(s)), dim3(kSelWaves * 64), 0, st,
                     r, row_ptr, col_idx, rows, s.nb, row_mass);
  if (totals != nullptr)
    hipLaunchKernelGGL(mass_total_kernel, dim3(1), dim3(1024), 0, st, row_mass, rows, totals);
  return hipGetLastError();
}

}  // namespace wise
