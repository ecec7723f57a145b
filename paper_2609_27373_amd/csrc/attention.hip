// attention.hip — the attention kernels of libwise on gfx950:
//
//   dense_attn_kernel   causal flash attention, O and natural-log LSE
//                       (paper Section 3, eq. recurrent_attention), and
//                       optionally the block-pooled attention mass
//                       (Section 5.1, eq. block_attention_mass)
//   sparse_attn_kernel  attention restricted to a CSR block support
//   sparse_group_kernel (Section 5.2, eq. wise_attention): one work-group
//   sparse_row32_kernel per row (64- and 128-key blocks); groups of
//   sparse_row16_kernel consecutive rows over the union of their supports
//                       (the same outputs, for dense supports); one wave per
//                       row of 32- or 16-key blocks
//
// Shared tile engine (all but the 16-key kernel).  A wave owns 32 consecutive
// queries.  For each tile of 64 keys (32 for 32-key blocks) it computes S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16 (A = K from
// LDS, B = Q^T held in registers for the whole row), so every lane ends up
// holding 32 scores of ONE query.  The row max needs one cross-lane step
// (lanes l and l^32 share a query), the row sum none until the end, and the
// probabilities are already in the B-operand layout of O^T = V^T P^T: they are
// packed to bf16 in place and fed straight to the second MFMA chain.  V stays
// row-major in LDS and its A-operand fragments are read transposed with
// ds_read_b64_tr_b16; row pads (2-wave dense and grouped kernels, which stage
// tiles through registers) or permuted rows (Swizzle, the others) make those
// reads, like the 128-bit K reads, free of bank conflicts.  Softmax is
// online in base 2 with the exact running max (so the largest probability of
// a row is exactly 1 in bf16); the O rescale is skipped, wave-uniformly, on
// tiles that raise no row's max.
//
// Work order: see sched_slot and row_slot (heaviest items of every head first,
// heads grouped per XCD).
#include <algorithm>
#include <type_traits>

#include "csr_entries.hpp"
#include "wise_device.hpp"
#include "wise_kernels.hpp"
namespace wise {

// ---------------------------------------------------------------------------
// Global -> register -> LDS staging of one tile of 64 keys (K rows permuted so
// the S^T accumulator comes out in PV operand order; V rows in natural order).  Loads for the next tile are
// issued before the current one is computed, so the memory latency hides
// behind the MFMA work; stores go to an LDS tile no wave still reads: after
// the barrier that retires it, or, in the 8-wave grouped late step, into its
// second buffer.  Used by that kernel's groups and the 2-wave dense group.
// ---------------------------------------------------------------------------
template <int D, int NT>
struct TileStage {
  using G = Geo<D>;
  static constexpr int kRowChunks = D / 8;                    // 16-B chunks per key row
  static constexpr int kChunks = kKeyTile * kRowChunks;       // per tensor
  static constexpr int kPer = (kChunks + NT - 1) / NT;

  u32x4_t kr[kPer];
  u32x4_t vr[kPer];

  // Chunk i of this thread: key row ch / kRowChunks, column (ch % kRowChunks) * 8.
  __device__ __forceinline__ static int chunk(int tid, int i) { return tid + i * NT; }
  __device__ __forceinline__ static bool live(int tid, int i) {
    return kChunks % NT == 0 || chunk(tid, i) < kChunks;
  }

  // rk, rv: the head's K and V; key0: this tile's first key row (uniform,
  // a scalar byte offset), per-lane offsets constant across tiles.
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rk, __amdgpu_buffer_rsrc_t rv,
                                       int key0, int tid) {
    const uint32_t soff = (uint32_t)key0 * (D * 2);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (live(tid, i)) {
        const int ch = chunk(tid, i);
        const uint32_t off = (uint32_t)((ch / kRowChunks) * D + (ch % kRowChunks) * 8) * 2;
        kr[i] = buffer_load16(rk, off, soff);
        vr[i] = buffer_load16(rv, off, soff);
      }
    }
  }

  __device__ __forceinline__ void store(uint16_t* ks, uint16_t* vs, int tid) const {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (live(tid, i)) {
        const int ch = chunk(tid, i);
        const int key = ch / kRowChunks, c8 = (ch % kRowChunks) * 8;
        *(u32x4_t*)(ks + k_lds_row(key) * G::kKStride + c8) = kr[i];
        *(u32x4_t*)(vs + key * G::kVStride + c8) = vr[i];
      }
    }
  }
};

// Global -> LDS copies of one 64-key tile by NW waves into the swizzled layout:
// copy i of wave w fills 1 KB at (w * kPer + i) * 1024.
template <int D, int NW>
struct TileCopy {
  using S = Swizzle<D>;
  static constexpr int kPer = S::kTile / 1024 / NW;
  static_assert(S::kTile % (1024 * NW) == 0, "whole copies per wave");
  uint32_t ko[kPer], vo[kPer];                        // this lane's source bytes in a tile

  __device__ __forceinline__ void init(int wave, int lane) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int at = (wave * kPer + i) * 1024 + lane * 16;
      const int row = at / S::kRow, slot = at % S::kRow / 16;
      ko[i] = k_lds_row(row) * S::kRow + S::k_chunk(row, slot) * 16;
      vo[i] = row * S::kRow + (S::v_block(row, slot >> 2) * 4 + (slot & 3)) * 16;
    }
  }
  // One copy of tile `tile`'s K (V) into the buffer at LDS address `lds`.
  __device__ __forceinline__ void k1(u32x4_t r, int tile, uint32_t lds, int wave, int i) const {
    copy16_to_lds(r, ko[i], (uint32_t)tile * S::kTile, lds + (uint32_t)(wave * kPer + i) * 1024);
  }
  __device__ __forceinline__ void v1(u32x4_t r, int tile, uint32_t lds, int wave, int i) const {
    copy16_to_lds(r, vo[i], (uint32_t)tile * S::kTile, lds + (uint32_t)(wave * kPer + i) * 1024);
  }
  __device__ __forceinline__ void k(u32x4_t r, int tile, uint32_t lds, int wave) const {
#pragma unroll
    for (int i = 0; i < kPer; ++i) k1(r, tile, lds, wave, i);
  }
  __device__ __forceinline__ void v(u32x4_t r, int tile, uint32_t lds, int wave) const {
#pragma unroll
    for (int i = 0; i < kPer; ++i) v1(r, tile, lds, wave, i);
  }
};

// LDS byte offsets of a lane's operand reads in a swizzled tile: K fragment
// (chunk c, half u) at k[c] + u * 32 rows, V fragment (k-step, dims 32 t) at
// v[t] + 16 ks rows (and 4 rows further).
template <int D>
struct ReadAddr {
  using S = Swizzle<D>;
  uint32_t k[D / 16], v[D / 32];
  __device__ __forceinline__ void init(int lane) {
    const int m = lane & 31, h = lane >> 5, r = 8 * h + ((lane >> 2) & 3);
#pragma unroll
    for (int c = 0; c < D / 16; ++c) k[c] = m * S::kRow + S::k_chunk(m, 2 * c + h) * 16;
#pragma unroll
    for (int t = 0; t < D / 32; ++t)
      v[t] = r * S::kRow + S::v_block(r, t) * 64 + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
  }
};

// Tile-local key held by register r of S^T tile t in a lane of half-wave h.
__device__ __forceinline__ int score_key(int t, int r, int h) {
  const int j = r >> 2, i = r & 3;
  return 32 * t + 16 * (j >> 1) + 8 * h + 4 * (j & 1) + i;
}

// ---------------------------------------------------------------------------
// Per-wave state and steps of the tile engine.
// ---------------------------------------------------------------------------
template <int D>
struct WaveRows {
  using G = Geo<D>;
  u32x4_t qf[G::kDChunks];   // Q^T B-operand fragments, one per 16-dim chunk
  f32x16_t o[G::kDTiles];    // O^T accumulator, 32 dims x 32 queries per tile
  float m;                   // running max of scale*log2(e)*s (per query)
  float l;                   // running sum over this lane's half of the keys
  float hs[4];               // last tile's per-part sums (softmax_pv<H, P>, P > 0)

  __device__ __forceinline__ void load_q(const uint16_t* qg, int q0, int lane) {
    const uint16_t* row = qg + (size_t)(q0 + (lane & 31)) * D + 8 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < G::kDChunks; ++c) qf[c] = *(const u32x4_t*)(row + 16 * c);
  }

  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int t = 0; t < G::kDTiles; ++t) o[t] = f32x16_t{};
    m = -INFINITY;
    l = 0.f;
  }

  // S^T of one LDS tile of 32*H keys: s[t] covers LDS rows 32t..32t+31.
  template <int H>
  __device__ __forceinline__ void scores(const uint16_t* ks, int lane, f32x16_t s[H]) const {
    const uint16_t* a0 = ks + (lane & 31) * G::kKStride + 8 * (lane >> 5);
    const uint16_t* a1 = a0 + 32 * G::kKStride;
    f32x16_t s0{}, s1{};
#pragma unroll
    for (int c = 0; c < G::kDChunks; ++c) {
      s0 = mfma32x32x16(*(const u32x4_t*)(a0 + 16 * c), qf[c], s0);
      if constexpr (H == 2) s1 = mfma32x32x16(*(const u32x4_t*)(a1 + 16 * c), qf[c], s1);
    }
    s[0] = s0;
    if constexpr (H == 2) s[1] = s1;
  }

  // Causal mask inside a tile: key0 + local key > query -> -inf.
  template <int H>
  __device__ __forceinline__ static void mask(f32x16_t s[H], int key0, int qi, int lane) {
    const int h = lane >> 5;
#pragma unroll
    for (int t = 0; t < H; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key0 + score_key(t, r, h) > qi) s[t][r] = -INFINITY;
  }

  // Online softmax of one tile: the probabilities packed in pb, O and l
  // rescaled.  With kParts = 2 (4) the sums of this lane's probabilities over
  // each 32-key half (16-key quarter) of the tile are kept in hs[] (the row
  // sum then adds the parts).
  template <int H, int kParts = 0>
  __device__ __forceinline__ void softmax(f32x16_t s[H], u32x4_t pb[2 * H], float c) {
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < H; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    mx = pair_max(mx) * c;
    const bool grow = mx > m;
    if (__builtin_amdgcn_ballot_w64(grow)) {
      const float mn = grow ? mx : m;
      const float alpha = (mn == m) ? 1.f : fast_exp2(m - mn);
      l *= alpha;
      // In-place multiply: keeps O in the same registers on both sides of the
      // branch (a plain `*=` lets the allocator rename O and copy all of it
      // back on the path that skips the rescale).
#pragma unroll
      for (int t = 0; t < G::kDTiles; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) asm volatile("v_mul_f32 %0, %0, %1" : "+v"(o[t][r]) : "v"(alpha));
      m = mn;
    }
    const float mb = (m == -INFINITY) ? 0.f : m;
    // The tile's probabilities are summed on their own and added to the row
    // sum once per tile: a long row (16K keys per lane at 32K) then carries
    // rounding error ~ tiles * eps instead of ~ keys * eps.
    float ts = 0.f;
#pragma unroll
    for (int t = 0; t < H; ++t) {
      float th = 0.f, tq[2] = {0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(__builtin_fmaf(s[t][r], c, -mb));
        s[t][r] = p;
        if constexpr (kParts == 4) tq[r >> 3] += p;
        else if constexpr (kParts == 2) th += p;
        else ts += p;
      }
      if constexpr (kParts == 4) {
        hs[2 * t] = tq[0];
        hs[2 * t + 1] = tq[1];
        ts += tq[0] + tq[1];
      } else if constexpr (kParts == 2) {
        hs[t] = th;
        ts += th;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          pb[2 * t + u][e] = pack_bf16x2(s[t][8 * u + 2 * e], s[t][8 * u + 2 * e + 1]);
    }
    l += ts;
  }

  // Softmax of one tile and O^T += V^T P^T.  A = V^T fragment: lane L needs
  // V[16ks + 8(L/32) + e][32t + L%32], e = 0..7, fetched as two transpose
  // reads of 4 keys each (see lds_read_tr16).
  template <int H, int kParts = 0>
  __device__ __forceinline__ void softmax_pv(f32x16_t s[H], const uint16_t* vt, int lane, float c) {
    u32x4_t pb[2 * H];
    softmax<H, kParts>(s, pb, c);
    const uint16_t* a = vt + (8 * (lane >> 5) + ((lane >> 2) & 3)) * G::kVStride +
                        16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int ks = 0; ks < 2 * H; ++ks)
#pragma unroll
      for (int t = 0; t < G::kDTiles; ++t) {
        const u32x2_t lo = lds_read_tr16(a + (16 * ks) * G::kVStride + 32 * t);
        const u32x2_t hi = lds_read_tr16(a + (16 * ks + 4) * G::kVStride + 32 * t);
        o[t] = mfma32x32x16(u32x4_t{lo[0], lo[1], hi[0], hi[1]}, pb[ks], o[t]);
      }
  }

  // One tile: S^T, the causal mask when the tile reaches past this wave's
  // first query (only ever on diagonal tiles, and only instantiated for
  // them), online softmax and PV.
  template <bool kMask, int H = 2, int kParts = 0>
  __device__ __forceinline__ void attend(const uint16_t* ks, const uint16_t* vt, int lane,
                                         float c, int key0, int q0) {
    f32x16_t s[H];
    scores<H>(ks, lane, s);
    if constexpr (kMask) {
      if (key0 + 32 * H - 1 > q0) mask<H>(s, key0, q0 + (lane & 31), lane);
    }
    softmax_pv<H, kParts>(s, vt, lane, c);
  }

  // S^T of a swizzled 64-key tile, and O^T += V^T P^T from one.
  __device__ __forceinline__ void scores_swizzled(const char* kt, const ReadAddr<D>& ra, f32x16_t s[2]) const {
#pragma unroll
    for (int i = 0; i < G::kDChunks; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        s[t] = mfma32x32x16(*(const u32x4_t*)(kt + ra.k[i] + 32 * t * Swizzle<D>::kRow), qf[i], s[t]);
  }
  __device__ __forceinline__ void pv_swizzled(const char* vt, const ReadAddr<D>& ra, const u32x4_t pb[4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int t = 0; t < G::kDTiles; ++t) {
        const char* p = vt + ra.v[t] + 16 * ks * Swizzle<D>::kRow;
        const u32x2_t lo = lds_read_tr16((const uint16_t*)p);
        const u32x2_t hi = lds_read_tr16((const uint16_t*)(p + 4 * Swizzle<D>::kRow));
        o[t] = mfma32x32x16(u32x4_t{lo[0], lo[1], hi[0], hi[1]}, pb[ks], o[t]);
      }
  }

  // New running max from a tile's max mx; true (wave-uniform) when some
  // query's max grew: alpha then holds the factor of O, l is rescaled here.
  __device__ __forceinline__ bool raise_max(float mx, float& alpha) {
    const bool grow = mx > m;
    if (!__builtin_amdgcn_ballot_w64(grow)) return false;
    const float mn = grow ? mx : m;
    alpha = (mn == m) ? 1.f : fast_exp2(m - mn);
    l *= alpha;
    m = mn;
    return true;
  }

  static constexpr int kAhead = 4;               // LDS fragments in flight

  // One step of the software pipeline of the dense groups: S^T of the
  // next tile (kQk: into sn, from its K tile kn, masked by maskn) and online
  // softmax and PV of the current one (kPv: its masked scores s, their max mx,
  // its V tile vt).  The same operations in the same order as attend(), so the
  // same bits.  It is laid out in 2 kN slots of one MFMA each, the LDS reads
  // kAhead slots before their use and the exponentials, sums, packing and the
  // next tile's max spread between the MFMAs, because two waves per SIMD in
  // step leave nothing else to fill a wave's waits; mid(n, j) runs in slot j
  // (the copies).  The wave's priority falls through the step, so of the two
  // waves of a SIMD the one behind issues first and they reach the barrier
  // together.  VALU and matrix cores are then both close to full.
  template <int H, bool kQk, bool kPv, int kParts, class Mid, class Mask>
  __device__ __forceinline__ void step(const char* kn, const char* vt, const ReadAddr<D>& ra, int lane, float c,
                                       f32x16_t s[H], f32x16_t sn[H], float& mx, Mid mid, Mask maskn) {
    constexpr int kN = G::kDChunks * H;          // MFMAs of S^T; PV has as many
    constexpr int kPairs = 8 * H;
    u32x4_t kf[kN], vf[kN], pb[2 * H];
    auto read_k = [&](int j) {
      kf[j] = *(const u32x4_t*)(kn + ra.k[j / H] + (j % H) * 32 * Swizzle<D>::kRow);
    };
    auto read_v = [&](int j) {
      const int ks = j / G::kDTiles, t = j % G::kDTiles;
      const char* p = vt + ra.v[t] + 16 * ks * Swizzle<D>::kRow;
      const u32x2_t lo = lds_read_tr16((const uint16_t*)p);
      const u32x2_t hi = lds_read_tr16((const uint16_t*)(p + 4 * Swizzle<D>::kRow));
      vf[j] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
    };
    float mb = 0.f, ts = 0.f, tp[4] = {0.f, 0.f, 0.f, 0.f};
    // Pair k: probabilities 2k, 2k + 1 of this lane, exponentials first, sums
    // and packing a slot later.  The empty asm keeps each in its slot.
    float pv[2 * kPairs];
    auto pair_exp = [&](int k) {
      if (k >= kPairs) return;
      const int t = k / 8, r = 2 * (k % 8);
      float p0 = fast_exp2(__builtin_fmaf(s[t][r], c, -mb));
      float p1 = fast_exp2(__builtin_fmaf(s[t][r + 1], c, -mb));
      asm volatile("" : "+v"(p0), "+v"(p1));
      pv[2 * k] = p0;
      pv[2 * k + 1] = p1;
    };
    auto pair_fin = [&](int k) {
      if (k < 0 || k >= kPairs) return;
      const int t = k / 8, r = 2 * (k % 8);
      float& a = kParts == 0 ? ts : kParts == 4 ? tp[2 * t + (r >> 3)] : tp[t];
      a += pv[2 * k];
      a += pv[2 * k + 1];
      uint32_t w = pack_bf16x2(pv[2 * k], pv[2 * k + 1]);
      asm volatile("" : "+v"(a), "+v"(w));
      pb[2 * t + (r >> 3)][(r & 7) >> 1] = w;
    };
    // Slot of the exponentials of pair k: slots 0 .. kN-1 hold the MFMAs of
    // S^T, kN .. 2 kN - 1 those of PV.
    constexpr int kS0 = 3;                        // S^T MFMAs issued before the new max is needed
    auto pairs_before = [](int slot) {           // pairs whose exponentials are done before it
      const int first = kS0, last = 2 * kN - kN / 4 - 1;   // first slot used, first slot past them
      const int x = slot <= first ? 0 : (slot - first) * kPairs / (last - first);
      return x > kPairs ? kPairs : x;
    };
    constexpr int kM0 = kN + 2;                  // first slot of the next tile's max
    auto maxes_before = [](int slot) {
      const int x = slot <= kM0 ? 0 : ((slot - kM0) * kPairs + 2 * kN - kM0 - 1) / (2 * kN - kM0);
      return x > kPairs ? kPairs : x;
    };
    if constexpr (kQk) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) read_k(j);
    }
    __builtin_amdgcn_s_setprio(3);
    float alpha = 1.f;
    bool grew = false;
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      if constexpr (kQk) {
        if (j + kAhead < kN) read_k(j + kAhead);
        sn[j % H] = mfma32x32x16(kf[j], qf[j / H], j < H ? f32x16_t{} : sn[j % H]);
      }
      if constexpr (kPv) {
        if (j == kS0) {
          __builtin_amdgcn_sched_barrier(0);
          grew = raise_max(mx, alpha);
          mb = (m == -INFINITY) ? 0.f : m;
        }
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (k >= pairs_before(j) && k < pairs_before(j + 1)) pair_exp(k);
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (k >= pairs_before(j - 1) && k < pairs_before(j)) pair_fin(k);
        // O rescaled in place, a tile of 32 dims at a time between the MFMAs
        // (a plain `*=` lets the allocator rename O and copy all of it back on
        // the path that skips the rescale).
        constexpr int kGap = (kN - kS0) / G::kDTiles;
        if (j >= kS0 && (j - kS0) % kGap == 0 && (j - kS0) / kGap < G::kDTiles) {
          const int t = (j - kS0) / kGap;
          if (grew) {
#pragma unroll
            for (int r = 0; r < 16; ++r) asm volatile("v_mul_f32 %0, %0, %1" : "+v"(o[t][r]) : "v"(alpha));
          }
        }
        if (j + kAhead >= kN) read_v(j + kAhead - kN);
      }
      mid(std::integral_constant<int, 2 * kN>{}, j);
      if (j == kN / 2) __builtin_amdgcn_s_setprio(2);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(1);
    if constexpr (kQk) maskn(sn);
    __builtin_amdgcn_sched_barrier(0);
    float mn = -INFINITY;
#pragma unroll
    for (int j = kN; j < 2 * kN; ++j) {
      if constexpr (kPv) {
        const int i = j - kN;
        if (i + kAhead < kN) read_v(i + kAhead);
        o[i % G::kDTiles] = mfma32x32x16(vf[i], pb[i / G::kDTiles], o[i % G::kDTiles]);
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (k >= pairs_before(j) && k < pairs_before(j + 1)) pair_exp(k);
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (k >= pairs_before(j - 1) && k < pairs_before(j)) pair_fin(k);
      }
      if constexpr (kQk) {
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (k >= maxes_before(j) && k < maxes_before(j + 1)) {
            mn = fmaxf(fmaxf(mn, sn[k / 8][2 * (k % 8)]), sn[k / 8][2 * (k % 8) + 1]);
            asm volatile("" : "+v"(mn));
          }
      }
      mid(std::integral_constant<int, 2 * kN>{}, j);
      if (j == kN + kN / 2) __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kPv) {
      if constexpr (kParts == 4) {
#pragma unroll
        for (int t = 0; t < H; ++t) {
          hs[2 * t] = tp[2 * t];
          hs[2 * t + 1] = tp[2 * t + 1];
          ts += tp[2 * t] + tp[2 * t + 1];
        }
      } else if constexpr (kParts == 2) {
#pragma unroll
        for (int t = 0; t < H; ++t) {
          hs[t] = tp[t];
          ts += tp[t];
        }
      }
      l += ts;
    }
    if constexpr (kQk) mx = pair_max(mn) * c;
  }

  // log2 of the last tile's probability mass per query, unnormalised (taken
  // against the running max m): entries 0..3 for the four 16-key quarters
  // (E = 16), 0 and 1 for the two 32-key halves (E = 32) or entry 0 for the
  // whole tile (E = 64).  -inf for no mass.
  template <int E>
  __device__ __forceinline__ void tile_log_mass(float out[4]) const {
    if constexpr (E == 16) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const float x = pair_sum(hs[t]);
        out[t] = x > 0.f ? m + __builtin_log2f(x) : -INFINITY;
      }
    } else if constexpr (E == 32) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float x = pair_sum(hs[t]);
        out[t] = x > 0.f ? m + __builtin_log2f(x) : -INFINITY;
      }
    } else {
      const float x = pair_sum(hs[0] + hs[1]);
      out[0] = x > 0.f ? m + __builtin_log2f(x) : -INFINITY;
    }
  }

  // log2 of the row normaliser: lse / ln 2.
  __device__ __forceinline__ float lse2() const { return m + __builtin_log2f(pair_sum(l)); }

  // O = O^T / l written as bf16 rows; lse in natural log.  Only the first
  // nq of the wave's 32 query columns are written.
  __device__ __forceinline__ void finish(uint16_t* og, float* lse, int q0, int lane,
                                         int nq = 32) const {
    const float lt = pair_sum(l);
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const int q = q0 + (lane & 31), h = lane >> 5;
    if ((lane & 31) >= nq) return;
    uint16_t* row = og + (size_t)q * D + 4 * h;
#pragma unroll
    for (int t = 0; t < G::kDTiles; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u32x2_t w;
        w[0] = pack_bf16x2(o[t][4 * j] * inv, o[t][4 * j + 1] * inv);
        w[1] = pack_bf16x2(o[t][4 * j + 2] * inv, o[t][4 * j + 3] * inv);
        *(u32x2_t*)(row + 32 * t + 8 * j) = w;
      }
    if (lse != nullptr && h == 0) lse[q] = lt > 0.f ? (m + __builtin_log2f(lt)) * kLn2 : -INFINITY;
  }
};

// ---------------------------------------------------------------------------
// Dense causal attention.  A work-group of NW waves owns 32*NW consecutive
// queries of one (batch, head); heavier (later) query tiles are issued first.
//
// With BM > 0 the kernel also pools the attention mass into blocks of BM keys
// and BM queries (Section 5.1, eq. block_attention_mass):
//   acc[qb][kb] += (1/BM) sum_{i in qb} sum_{j in kb, j <= i} A_ij.
// A_ij = 2^(s_ij - lse2_i) needs the row normaliser, known only after the
// row's last tile, so every tile leaves per query the log2 of its
// unnormalised mass (against the running max of that moment) in a workspace
// entry of E = min(BM, 64) keys (only spans up to the query tile's end are
// stored), and the epilogue, once lse2 is known, turns
// each entry into 2^(entry - lse2), sums it over the wave's 32 queries and
// then over the waves and entries of each (query block, key block).  The
// group owns the acc rows of its query blocks: no atomics, and the sums run
// in a fixed order, so the result is bitwise reproducible.
// ---------------------------------------------------------------------------
constexpr int kMassChunk = 256;   // workspace entries reduced per epilogue pass
constexpr int kMassBatch = 16;    // entry loads in flight per half-wave in the epilogue

// Tiles in each LDS ring of the dense group (0: one tile, staged through
// registers).  An 8-wave group fills its CU alone, so its copies get two steps
// to land; two 4-wave groups (three at d 64) share a CU and cover each
// other's waits, and four tiles each would leave one (d 96: 1242 us instead of
// 796 at 8192 x 55 heads).  Rings against the staged loop, 4-wave groups: d 96,
// 4096 x 220 heads 825 -> 790 us, with 32-key masses 943 -> 886, 1024 x 32
// grouped heads 24.0 -> 21.4; d 64, 4096 x 192 grouped heads 493 -> 467, with
// 32-key masses 590 -> 574; d 128, 640 x 4 heads 18.1 -> 15.7.  2-wave groups
// (lengths 128 does not divide) stay staged: eight copies per wave and tile cost
// its two waves more than the staging (1216 x 15 heads of 64: 24.0 against 22.0).
constexpr int dense_ring(int nw) { return nw == 8 ? 4 : nw == 4 ? 2 : 0; }

template <int D, int NW, int BM>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
dense_attn_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                  const uint16_t* __restrict__ V, uint16_t* __restrict__ O,
                  float* __restrict__ lse, int n, int heads, int gq, Sched sc, float c,
                  float* __restrict__ acc, float* __restrict__ mws) {
  using G = Geo<D>;
  constexpr int kNT = NW * 64, kQT = NW * 32;
  constexpr bool kMass = BM > 0;
  constexpr int kE = BM > 0 && BM < 64 ? BM : 64;   // keys per workspace entry
  constexpr int kEPT = kKeyTile / kE;               // entries per 64-key tile
  constexpr int kParts = kMass ? (kE == 16 ? 4 : 2) : 0;
  constexpr int R = dense_ring(NW);
  __shared__ __attribute__((aligned(1024))) char smem[R > 0 ? 2 * R * Swizzle<D>::kTile : 1];   // rings
  // The staged tile: two arrays, so that the compiler need not order one's
  // stores and the other's reads (1088 x 12 heads of 128: 26.0 us, 29.8 in one).
  __shared__ __attribute__((aligned(16))) uint16_t ks[R > 0 ? 1 : G::kKElems], vt[R > 0 ? 1 : G::kVElems];
  int bh, item;
  if (!sched_slot(sc, bh, item)) return;
  const int qt = sc.items - 1 - item;
  const size_t hoff = (size_t)bh * n * D;
  const size_t kvoff = (size_t)kv_head(bh, heads, gq) * n * D;
  const int tid = threadIdx.x, lane = tid & 63;
  // scalar for the copies' addresses; the staged loop has none (1216 x 15 heads
  // of 64 with masses: 23.7 us with it, 23.6 without)
  const int wave = R > 0 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int qbase = qt * kQT, q0 = qbase + 32 * wave;
  // Workspace: per head, per query tile qt, (qt+1)*kQT/kE entries of kQT
  // queries each (only the spans up to the tile's last query), query-minor.
  const int nq = sc.items;
  const size_t per_tile = (size_t)kQT * (kQT / kE);
  float* ew = kMass ? mws + per_tile * ((size_t)bh * nq * (nq + 1) / 2 + (size_t)qt * (qt + 1) / 2) +
                          32 * wave + (lane & 31)
                    : nullptr;

  WaveRows<D> w;
  w.load_q(Q + hoff, q0, lane);
  w.reset();
  // Per-tile mass entries of this lane's query (lanes 0..31 write them).
  auto put_mass = [&](int it) {
    if constexpr (kMass) {
      float lm[4];
      w.template tile_log_mass<kE>(lm);
      if (lane < 32) {
#pragma unroll
        for (int t = 0; t < kEPT; ++t) ew[(size_t)(it * kEPT + t) * kQT] = lm[t];
      }
    }
  };
  // Tiles 0 .. nfull-1 lie wholly below every query of the group; the last
  // kQT/64 tiles hold the diagonal and are masked per wave.
  const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(K + kvoff), rv = buffer_rsrc(V + kvoff);
  const int ntiles = (qbase + kQT) / kKeyTile;
  const int nfull = qbase / kKeyTile;
  TileStage<D, kNT> st;
  if constexpr (R == 0) st.load(rk, rv, 0, tid);
  if constexpr (R > 0) {
    // Software pipeline: in step `it` a wave computes S^T of tile it+1 and
    // softmax and PV of tile it, while K(it+R) and V(it+R-1) are copied into
    // rings of R K and R V tiles.  At d 128, R = 4 (128 KB of LDS; registers
    // already limit a CU to one 8-wave group), copies have two steps to land:
    // one step is less than the latency of a tile from HBM (16K: 1.01x instead
    // of 1.06x of the unpipelined loop).  Against that loop (S^T, softmax and PV
    // one after the other, tiles staged through registers): 4096 x 32 heads 148.7
    // -> 137.9 us, 16384 x 64 heads 4069 -> 3827 us (1081 -> 1149 TFLOP/s).
    constexpr int kT = Swizzle<D>::kTile;
    const u32x4_t bk = buffer_words(K + kvoff), bv = buffer_words(V + kvoff);
    TileCopy<D, NW> cp;
    ReadAddr<D> ra;
    cp.init(wave, lane);
    ra.init(lane);
    const uint32_t lk = lds_address(smem), lv = lk + R * kT;
    const char* sk = smem;
    const char* sv = smem + R * kT;
    constexpr int kC = TileCopy<D, NW>::kPer;     // copies per tile and tensor
    // The compiler waits for Q with nothing left in flight, so only what the
    // first steps need is issued before Q's first use.
    cp.k(bk, 0, lk, wave);
    cp.v(bv, 0, lv, wave);
    if (ntiles > 1) cp.k(bk, 1, lk + kT, wave);
#pragma unroll
    for (int cc = 0; cc < G::kDChunks; ++cc) asm volatile("" : "+v"(w.qf[cc]));
    wait_copies<0>();
    __syncthreads();
#pragma unroll
    for (int u = 1; u < R - 1; ++u) {
      if (u < ntiles) cp.v(bv, u, lv + u * kT, wave);
      if (u + 1 < ntiles) cp.k(bk, u + 1, lk + (u + 1) * kT, wave);
    }
    const int ntw = q0 / kKeyTile + 1;            // this wave's tiles; the last holds its diagonal
    f32x16_t s0[2], s1[2];
    float mx = 0.f;
    auto mask_last = [&](f32x16_t sn[2]) {
      int lastk = (ntw - 1) * kKeyTile;
      asm volatile("" : "+s"(lastk));
      WaveRows<D>::template mask<2>(sn, lastk, q0 + (lane & 31), lane);
    };
    w.template step<2, true, false, kParts>(sk, sv, ra, lane, c, s1, s0, mx, [](auto, int) {},
                                            [&](f32x16_t sn[2]) { if (ntw == 1) mask_last(sn); });
    __syncthreads();                              // K(0) read by every wave: K(R) may take its place
    // End of step it: K(it+2) and V(it+1) have landed for every wave.  Copies
    // land in order; those issued after them may stay in flight, and in the ring
    // of two the step's `stores` last operations, its mass entries (dwords kQT
    // floats apart, a store each).  Waiting for those too cost every step their
    // round trip: d 64, 64-key masses, 2048 x 32 heads 40.1 us instead of 37.2,
    // 16384 x 4 269 instead of 250.
    auto advance = [&](int it, auto stores) {
      if (it + 1 == ntiles) return;               // nothing left in flight, no tile to replace
      if constexpr (R == 4) {
        if (it + 4 < ntiles) wait_copies<4 * kC>();
        else if (it + 4 == ntiles) wait_copies<3 * kC>();
        else if (it + 3 == ntiles) wait_copies<kC>();
        else wait_copies<0>();
      } else {
        wait_copies<decltype(stores)::value>();
      }
      __syncthreads();
    };
    using Stores = std::integral_constant<int, kMass ? kEPT : 0>;
    // Step it reads K(it+1) and V(it); V(it+R-1) and K(it+R) go where V(it-1)
    // and K(it) were, last read in the step before.  b = it % R.
    auto copy = [&](int it, int b, int i) {
      if (i < kC) {
        if (it + R - 1 < ntiles) cp.v1(bv, it + R - 1, lv + ((b + R - 1) % R) * kT, wave, i);
      } else {
        if (it + R < ntiles) cp.k1(bk, it + R, lk + b * kT, wave, i - kC);
      }
    };
    auto fused = [&](int it, int b, f32x16_t sc[2], f32x16_t sn[2]) {
      w.template step<2, true, true, kParts>(
          sk + ((b + 1) % R) * kT, sv + b * kT, ra, lane, c, sc, sn, mx,
          [&](auto n, int j) {
            // from the third slot on, over the first five eighths of the step
            constexpr int kGap = std::max(1, (decltype(n)::value * 5 / 8 - 2) / (2 * kC));
            if (j >= 2 && (j - 2) % kGap == 0 && (j - 2) / kGap < 2 * kC) copy(it, b, (j - 2) / kGap);
          },
          [&](f32x16_t x[2]) { if (it + 2 == ntw) mask_last(x); });
      put_mass(it);
      advance(it, Stores{});
    };
    int it = 0;
    if constexpr (R == 4) {
      for (; it + 4 < ntw; it += 4) {
        fused(it, 0, s0, s1);
        fused(it + 1, 1, s1, s0);
        fused(it + 2, 2, s0, s1);
        fused(it + 3, 3, s1, s0);
      }
    } else {
      for (; it + 2 < ntw; it += 2) {
        fused(it, 0, s0, s1);
        fused(it + 1, 1, s1, s0);
      }
    }
    for (; it + 1 < ntw; ++it) {
      fused(it, it % R, s0, s1);
      s0[0] = s1[0];
      s0[1] = s1[1];
    }
    auto copies = [&](int it) {
#pragma unroll
      for (int i = 0; i < 2 * kC; ++i) copy(it, it % R, i);
    };
    copies(it);
    w.template step<2, false, true, kParts>(sk, sv + (it % R) * kT, ra, lane, c, s0, s1, mx,
                                            [](auto, int) {}, [](f32x16_t*) {});
    put_mass(it);
    advance(it, Stores{});
    for (++it; it < ntiles; ++it) {
      copies(it);
      advance(it, std::integral_constant<int, 0>{});
    }
  } else {
    for (int it = 0; it < nfull; ++it) {
      st.store(ks, vt, tid);
      __syncthreads();
      st.load(rk, rv, (it + 1) * kKeyTile, tid);
      w.template attend<false, 2, kParts>(ks, vt, lane, c, it * kKeyTile, q0);
      put_mass(it);
      __syncthreads();
    }
    for (int it = nfull; it < ntiles; ++it) {
      st.store(ks, vt, tid);
      __syncthreads();
      if (it + 1 < ntiles) st.load(rk, rv, (it + 1) * kKeyTile, tid);
      if (it * kKeyTile <= q0) {
        w.template attend<true, 2, kParts>(ks, vt, lane, c, it * kKeyTile, q0);
        put_mass(it);
      }
      __syncthreads();
    }
  }
  w.finish(O + hoff, lse ? lse + (size_t)bh * n : nullptr, q0, lane);
  if constexpr (kMass) {
    // Epilogue: entries 0 .. elast of this wave were written above (the
    // tiles it attended); later ones hold no mass for its queries.  A
    // 16-query block is half of a wave's queries: its sums run over 16-lane
    // rows, and each wave feeds two query blocks.
    constexpr int kSub = BM < 32 ? 32 / BM : 1;     // query blocks per wave
    constexpr int kWPB = BM < 32 ? 1 : BM / 32;     // waves (or wave halves) per query block
    constexpr int kQB = kQT / BM;                   // query blocks of the group
    constexpr int kBE = BM / kE;                    // entries per key block
    static_assert(kQB >= 1 && kQT % BM == 0, "mass block larger than the group");
    __shared__ float red[NW * kSub][kMassChunk];
    const float l2 = w.lse2();
    const int elast = (q0 + 31) / kE;
    const int nb = n / BM;
    const int eend = (qbase + kQT - 1) / kE + 1;    // entries any wave of the group wrote
    const int hsel = lane >> 5;                     // each half-wave takes every other entry
    for (int c0 = 0; c0 < eend; c0 += kMassChunk) {
      const int cend = min(c0 + kMassChunk, eend);
      for (int e0 = c0; e0 < cend; e0 += 2 * kMassBatch) {
        float x[kMassBatch];
#pragma unroll
        for (int u = 0; u < kMassBatch; ++u) {      // all loads first, then the sums
          const int e = e0 + 2 * u + hsel;
          x[u] = e < cend && e <= elast ? ew[(size_t)e * kQT] : -INFINITY;
        }
#pragma unroll
        for (int u = 0; u < kMassBatch; ++u) {
          const int e = e0 + 2 * u + hsel;
          if constexpr (kSub == 2) {
            const float y = row16_sum(fast_exp2(x[u] - l2));
            if ((lane & 15) == 0 && e < cend) red[2 * wave + ((lane >> 4) & 1)][e - c0] = y;
          } else {
            const float y = half_wave_sum(fast_exp2(x[u] - l2));
            if ((lane & 31) == 0 && e < cend) red[wave][e - c0] = y;
          }
        }
      }
      __syncthreads();
      const int b0 = c0 / kBE, b1 = (min(c0 + kMassChunk, eend) + kBE - 1) / kBE;
      for (int x = tid; x < kQB * (b1 - b0); x += kNT) {
        const int j = x / (b1 - b0), kb = b0 + x % (b1 - b0);
        const int qb = qbase / BM + j;
        if (kb > qb) continue;
        float sum = 0.f;
#pragma unroll
        for (int wv = 0; wv < kWPB; ++wv)
#pragma unroll
          for (int u = 0; u < kBE; ++u) sum += red[j * kWPB + wv][kb * kBE + u - c0];
        acc[((size_t)bh * nb + qb) * nb + kb] += sum * (1.f / BM);
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// A support row's valid ids (0..qb) in order, 64 read at a time; ids outside
// are skipped.  Everything but `ids` is wave-uniform.
// ---------------------------------------------------------------------------
struct RowIds {
  const int32_t* col_idx;
  Entries e;
  int qb, ids;
  uint64_t left;
  __device__ __forceinline__ RowIds(const int32_t* row_ptr, const int32_t* ci, int row, int qb_)
      : col_idx(ci), e(row_ptr[row], row_ptr[row + 1]), qb(qb_), ids(0), left(0) {}
  __device__ __forceinline__ int next(int lane) {    // -1: no more
    while (left == 0) {
      if (!e.more()) return -1;
      ids = e.holds(lane) ? col_idx[e.at + lane] : -1;
      left = __builtin_amdgcn_ballot_w64((unsigned)ids <= (unsigned)qb);
      e.advance(64);
    }
    const int at = __builtin_ctzll(left);
    left &= left - 1;
    return (int)__builtin_amdgcn_readlane(ids, at);
  }
};

// ---------------------------------------------------------------------------
// Block-sparse attention over a CSR support.  One work-group per (batch,
// head, query block) row of 64- or 128-key blocks, NW = block/32 waves, in
// tiles of 64 keys.
// Schedule slot s (a logical id, contiguous per XCD) runs row order[s];
// wise_select_support writes the rows of each head together, longest support
// first, so an XCD works through a few heads at a time and their K/V tiles
// stay in its L2.
//
// Bound by the round trip of a tile to L2 and beyond: what counts is how many
// copies are in flight on a CU and how long they have to land.  K and V are
// copied straight into LDS without row pads, no tile waits in registers (133,
// 160 and 191 VGPRs at d 64, 96 and 128: 3, 3 and 2 waves per SIMD).
//   kBufs 1   one tile each, 32 KB at d 128: the next K is copied after S^T,
//             the next V after PV, each with half a tile of work to land, and
//             four barriers a tile.  Registers, not LDS, limit the groups of a
//             CU (six 2-wave groups, four at d 128).
//   kBufs 2   two tiles each: both copies have a whole tile to land and one
//             barrier is enough.  4-wave groups (128-key blocks) still fit
//             four, three and two to a CU; of 2-wave groups LDS then holds
//             five, three and two, so they take it in small grids only
//             (kSmallGrid).
// us, tiles staged through registers / one tile / two: 64-key blocks at density
// 0.3 (about 0.3 of the causal blocks, drawn at random), 2048 x 4 heads of 64
// 15.8 / 16.8 / 14.5, 4096 x 16 heads of 96 43.0 / 41.6 / 38.8, 4096 x 55 of 96
// 106 / 95 / 108, 4096 x 32 of 128 73.9 / 71.0 / 88; 128-key blocks, 2048 x 16
// grouped heads of 64 (density 1) 33.3 / 36.9 / 28.9, 4096 x 32 of 128 (0.7)
// 130 / 124 / 118, 4096 x 55 of 96 (0.3) 103 / 98.5 / 95.1.  Same bits.
// ---------------------------------------------------------------------------
template <int D, int NW, int kBufs>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3)))
sparse_attn_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                   const uint16_t* __restrict__ V, const int32_t* __restrict__ row_ptr,
                   const int32_t* __restrict__ col_idx, const int32_t* __restrict__ order,
                   uint16_t* __restrict__ O, float* __restrict__ lse, int n, int nb, int rows,
                   int heads, int gq, RowSched sc, float c) {
  using G = Geo<D>;
  constexpr int kB = NW * 32, kTPB = kB / kKeyTile;
  constexpr int kRow = Swizzle<D>::kRow, kTile = Swizzle<D>::kTile;   // bytes
  constexpr int kP = D / 32;                        // 1 KB copies per 16 rows
  constexpr int kU = 4 / NW, kC = kU * kP;          // a wave's 16-row pieces and copies of a tile
  static_assert(kTPB >= 1 && kB % kKeyTile == 0 && 4 % NW == 0, "block / key tile");
  extern __shared__ __attribute__((aligned(1024))) char tiles[];   // kBufs K tiles, kBufs V tiles
  const char* const kt = tiles;
  const char* const vt = tiles + kBufs * kTile;
  int sh, sit;
  if (!row_slot(sc, sh, sit)) return;
  const int row = order ? order[sh * nb + sit] : sh * nb + (nb - 1 - sit);
  if ((unsigned)row >= (unsigned)rows) return;
  const int bh = row / nb, qb = row % nb;
  const size_t hoff = (size_t)bh * n * D;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q0 = qb * kB + 32 * wave;
  const size_t kvoff = (size_t)kv_head(bh, heads, gq) * n * D;
  const u32x4_t bk = buffer_words(K + kvoff), bv = buffer_words(V + kvoff);
  const uint32_t lk = lds_address(kt), lv = lds_address(vt);
  RowIds ids(row_ptr, col_idx, row, qb);

  WaveRows<D> w;
  w.load_q(Q + hoff, q0, lane);
  w.reset();
  ReadAddr<D> ra;
  ra.init(lane);
  uint32_t ko[kP], vo[kP];                          // source bytes of this lane's copies in 16 rows
#pragma unroll
  for (int i = 0; i < kP; ++i) {
    const int at = 1024 * i + 16 * lane, r = at / kRow, ch = at % kRow / 16;
    ko[i] = k_lds_row(r) * kRow + Swizzle<D>::k_chunk(r, ch) * 16;
    vo[i] = r * kRow + (Swizzle<D>::v_block(r, ch >> 2) * 4 + (ch & 3)) * 16;
  }
  auto copy = [&](u32x4_t r, const uint32_t off[kP], int key0, uint32_t lds) {
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int i = 0; i < kP; ++i) {
        const int at = wave * kU + u;
        copy16_to_lds(r, off[i], (uint32_t)(key0 + 16 * at) * kRow, lds + 1024 * (at * kP + i));
      }
  };
  // The row's 64-key tiles: the first key of the next one, -1 past the last.
  int blk = -1, sub = kTPB - 1;
  auto next_key = [&] {
    if (sub + 1 < kTPB) {
      ++sub;
    } else {
      blk = ids.next(lane);
      sub = 0;
    }
    return blk < 0 ? -1 : blk * kB + sub * kKeyTile;
  };
  int key0 = next_key();
#pragma unroll
  for (int i = 0; i < G::kDChunks; ++i) asm volatile("" : "+v"(w.qf[i]));   // Q has landed: only copies count below
  if (key0 >= 0) {
    copy(bk, ko, key0, lk);
    copy(bv, vo, key0, lv);
  }
  if constexpr (kBufs == 2) {
    auto step = [&](auto buf) {                     // the tile in buffer buf; true: there is another
      constexpr int kOther = 1 - decltype(buf)::value;
      const int next = next_key();
      wait_copies<0>();
      __syncthreads();                              // it has landed and the one before is read, for every wave
      if (next >= 0) {
        copy(bk, ko, next, lk + kOther * kTile);
        copy(bv, vo, next, lv + kOther * kTile);
      }
      if (key0 <= q0) {                             // else the tile lies past this wave's queries
        f32x16_t s[2] = {f32x16_t{}, f32x16_t{}};
        u32x4_t pb[4];
        w.scores_swizzled(kt + decltype(buf)::value * kTile, ra, s);
        if (key0 + kKeyTile - 1 > q0) WaveRows<D>::template mask<2>(s, key0, q0 + (lane & 31), lane);
        w.template softmax<2>(s, pb, c);
        w.pv_swizzled(vt + decltype(buf)::value * kTile, ra, pb);
      }
      key0 = next;
      return next >= 0;
    };
    if (key0 >= 0)
      while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {}
  } else {
    while (key0 >= 0) {
      const int next = next_key();
      const bool mine = key0 <= q0;                 // else the tile lies past this wave's queries
      wait_copies<kC>();                            // this tile's K; its V may be in flight
      __syncthreads();
      f32x16_t s[2] = {f32x16_t{}, f32x16_t{}};
      if (mine) w.scores_swizzled(kt, ra, s);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();                              // K read: its place is free
      if (next >= 0) copy(bk, ko, next, lk);
      u32x4_t pb[4];
      if (mine) {
        if (key0 + kKeyTile - 1 > q0) WaveRows<D>::template mask<2>(s, key0, q0 + (lane & 31), lane);
        w.template softmax<2>(s, pb, c);
      }
      if (next >= 0) wait_copies<kC>();             // this tile's V; the next K may be in flight
      else wait_copies<0>();
      __syncthreads();
      if (mine) w.pv_swizzled(vt, ra, pb);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();                              // V read: its place is free
      if (next >= 0) copy(bv, vo, next, lv);
      key0 = next;
    }
  }
  w.finish(O + hoff, lse ? lse + (size_t)bh * n : nullptr, q0, lane);
}

// ---------------------------------------------------------------------------
// Block-sparse attention over groups of consecutive rows of BR-key blocks:
// a work-group of the dense kernel's size (NW waves, 32 NW queries: 4 rows of 64 or 2
// of 128 keys at head_dim 128, 2 rows of 64 otherwise) walks the ascending
// union of its rows' supports in 64-key tiles, staging each tile once for all
// its waves, and each wave attends only the tiles its own row holds (its
// diagonal block masked, tiles wholly past its queries skipped), so every row
// gets exactly its own attention, in the one-row kernel's tile order.  Where
// consecutive rows' supports nearly coincide (dense supports) the union adds
// few tiles and every staged tile feeds 2-4 times the queries of the one-row
// group; where they differ, the union walk costs more than it saves.  The
// membership of each row and the union are built in LDS as bitmasks (up to
// 1024 key blocks).
// ---------------------------------------------------------------------------
constexpr int kGroupMaskWords = 16;

template <int D, int NW, int BR>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
sparse_group_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                    const uint16_t* __restrict__ V, const int32_t* __restrict__ row_ptr,
                    const int32_t* __restrict__ col_idx, uint16_t* __restrict__ O,
                    float* __restrict__ lse, int n, int nb, int heads, int gq, Sched sc,
                    float c) {
  using G = Geo<D>;
  constexpr int kNT = NW * 64, kQT = NW * 32, kR = kQT / BR;   // rows per group
  constexpr int kTPB = BR / kKeyTile, kWR = BR / 32;           // tiles per block, waves per row
  static_assert(kR >= 2 && kQT % BR == 0 && BR % kKeyTile == 0, "group of rows");
  constexpr int kW = kGroupMaskWords;
  constexpr int kBufs = NW == 8 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) uint16_t ks[kBufs * G::kKElems];
  __shared__ __attribute__((aligned(16))) uint16_t vt[kBufs * G::kVElems];
  __shared__ unsigned long long rmask[kR][kW];   // membership per row of the group
  __shared__ unsigned long long umask[kW];       // their union
  int bh, item;
  if (!sched_slot(sc, bh, item)) return;
  const int qt = sc.items - 1 - item;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qbase = qt * kQT, q0 = qbase + 32 * wave;
  const int qb0 = qt * kR, mine = wave / kWR;     // the group's first row; this wave's row
  const size_t hoff = (size_t)bh * n * D;
  const size_t kvoff = (size_t)kv_head(bh, heads, gq) * n * D;
  const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(K + kvoff), rv = buffer_rsrc(V + kvoff);
  const int words = (nb + 63) >> 6;

  WaveRows<D> w;
  w.load_q(Q + hoff, q0, lane);
  // The group's first tile is its union's lowest block: block 0 wherever a
  // row holds the sink block, so that tile's loads start before the
  // supports are read (and are reissued for another first block).
  TileStage<D, kNT> st;
  st.load(rk, rv, 0, tid);
  w.reset();
  // The group's rows are consecutive CSR rows: their entries form one range,
  // read in one pass.
  const int row0 = bh * nb + qb0;
  int bound[kR + 1];
#pragma unroll
  for (int r = 0; r <= kR; ++r) bound[r] = row_ptr[row0 + r];
  for (int i = tid; i < (kR + 1) * kW; i += kNT) {
    if (i < kR * kW) rmask[i / kW][i % kW] = 0ull;
    else umask[i - kR * kW] = 0ull;
  }
  __syncthreads();
  // Valid ids (0..qb) of every row of the group into the bitmasks.
  for (Entries all(bound[0], bound[kR]); all.more(); all.advance(kNT)) {
    if (!all.holds(tid)) break;
    const int e = all.at + tid, kb = col_idx[e];
    int r = 0;
#pragma unroll
    for (int j = 1; j < kR; ++j) r += e >= bound[j];
    if ((unsigned)kb <= (unsigned)(qb0 + r)) {
      const unsigned long long bit = 1ull << (kb & 63);
      atomicOr(&rmask[r][kb >> 6], bit);
      atomicOr(&umask[kb >> 6], bit);
    }
  }
  __syncthreads();
  // The 64-key tiles of the union's blocks in ascending order (the same
  // sequence in every wave; block cb's tiles are cb * kTPB + 0 .. kTPB - 1),
  // each with this wave's membership.  The walk holds the union's and its
  // row's current 64-block words as wave-uniform values and reads LDS only
  // when it moves on to the next word, so no tile waits on an LDS read for
  // its membership between the barrier and its MFMAs.
  auto uniform64 = [](unsigned long long x) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)x);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
  };
  int wi = 0, cb = 0, sub = kTPB - 1;
  unsigned long long cur = uniform64(umask[0]), mw = uniform64(rmask[mine][0]);
  bool cm = false;                                  // this wave's row holds block cb
  auto next = [&](int& tile, bool& mem) {
    if (sub + 1 < kTPB) {
      tile = cb * kTPB + ++sub;
      mem = cm;
      return true;
    }
    while (cur == 0ull) {
      if (++wi >= words) return false;
      cur = uniform64(umask[wi]);
      mw = uniform64(rmask[mine][wi]);
    }
    const int bit = __builtin_ctzll(cur);
    cb = (wi << 6) + bit;
    cur &= cur - 1ull;
    cm = (mw >> bit) & 1ull;
    sub = 0;
    tile = cb * kTPB;
    mem = cm;
    return true;
  };
  // One instance of the tile step for every tile (it masks only a tile that
  // reaches past the wave's first query): a second, unmasked instance for
  // the tiles below the diagonal costs registers and code for nothing.
  auto attend = [&](const uint16_t* kt, const uint16_t* vv, int tile, bool mem) {
    const int key0 = tile * kKeyTile;
    if (!mem || key0 > q0) return;
    w.template attend<true>(kt, vv, lane, c, key0, q0);
  };

  int kb = 0, kb1 = 0, kb2 = 0;     // tiles: current, next, the one after
  bool m0 = false, m1 = false, m2 = false;
  bool have = next(kb, m0);
  if (have && kb != 0) st.load(rk, rv, kb * kKeyTile, tid);
  if constexpr (kBufs == 2) {
    // Double-buffered (an 8-wave group fills its CU alone): tile i+1 is stored into the
    // idle buffer right after tile i is computed, one barrier per tile.
    if (have) {
      st.store(ks, vt, tid);
      bool h1 = next(kb1, m1);
      if (h1) st.load(rk, rv, kb1 * kKeyTile, tid);
      __syncthreads();
      for (int it = 0;; ++it) {
        const int cu = it & 1;
        attend(ks + cu * G::kKElems, vt + cu * G::kVElems, kb, m0);
        bool h2 = false;
        if (h1) {
          const int nx = (it + 1) & 1;
          st.store(ks + nx * G::kKElems, vt + nx * G::kVElems, tid);
          h2 = next(kb2, m2);
          if (h2) st.load(rk, rv, kb2 * kKeyTile, tid);
        }
        __syncthreads();
        if (!h1) break;
        kb = kb1;
        m0 = m1;
        kb1 = kb2;
        m1 = m2;
        h1 = h2;
      }
    }
  } else {
    while (have) {
      st.store(ks, vt, tid);
      __syncthreads();
      const bool more = next(kb1, m1);
      if (more) st.load(rk, rv, kb1 * kKeyTile, tid);
      attend(ks, vt, kb, m0);
      __syncthreads();
      kb = kb1;
      m0 = m1;
      have = more;
    }
  }
  w.finish(O + hoff, lse ? lse + (size_t)bh * n : nullptr, q0, lane);
}

// ---------------------------------------------------------------------------
// Block-sparse attention for 32-key blocks: one one-wave work-group per
// (batch, head, query block) row, a tile per block.  K and V are copied
// straight into LDS, one tile each (12 KB at d 96): the next tile's K as soon
// as this one's is in registers, its V after PV, so each has half a tile of
// work to land, and no registers hold tiles in flight.  LDS decides how many
// waves fit a CU at d 96 (13) and 128 (10), registers at d 64 (102: 16 waves).
// The online softmax groups keys in 32s, so a full support does not reproduce
// the dense kernel's bits.
//
// Every row reads its own K and V through L2: 80 million 128-byte requests (10.3
// GB, 90% hits) at 4096 x 220 heads, d 96, density 0.40, 506 us or 20 TB/s; bound
// by that and by the round trip, of which a wave hides half a tile's work.
// Against tiles staged through registers (one more tile of 48 VGPRs in flight,
// LDS written by the wave): 545 -> 506 us there, 305 -> 288 at 192 grouped heads
// of 64 (45 million requests), 182 -> 153 at 32 heads of 128; rows of about five
// blocks are slower (d 128, 4096 x 220 heads at density 0.05 230 -> 250 us): their
// first tile, and what the round trip is longer than half a tile, weigh more.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : D == 96 ? 3 : 2)))
sparse_row32_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                    const uint16_t* __restrict__ V, const int32_t* __restrict__ row_ptr,
                    const int32_t* __restrict__ col_idx, const int32_t* __restrict__ order,
                    uint16_t* __restrict__ O, float* __restrict__ lse, int n, int nb, int rows,
                    int heads, int gq, RowSched sc, float c) {
  using G = Geo<D>;
  constexpr int kC = D / 32;                        // 1 KB copies per 16 rows
  constexpr int kRow = 2 * D, kTile = 32 * kRow;    // bytes
  __shared__ __attribute__((aligned(1024))) char kt[kTile], vt[kTile];
  int sh, sit;
  if (!row_slot(sc, sh, sit)) return;
  const int row = order ? order[sh * nb + sit] : sh * nb + (nb - 1 - sit);
  if ((unsigned)row >= (unsigned)rows) return;
  const int bh = row / nb, qb = row % nb;
  const size_t hoff = (size_t)bh * n * D;
  const int lane = threadIdx.x, q0 = 32 * qb;
  const size_t kvoff = (size_t)kv_head(bh, heads, gq) * n * D;
  const u32x4_t bk = buffer_words(K + kvoff), bv = buffer_words(V + kvoff);
  const uint32_t lk = lds_address(kt), lv = lds_address(vt);
  RowIds ids(row_ptr, col_idx, row, qb);

  WaveRows<D> w;
  w.load_q(Q + hoff, q0, lane);
  w.reset();
  ReadAddr<D> ra;
  ra.init(lane);
  uint32_t ko[kC], vo[kC];                          // source bytes of this lane's copies in 16 rows
#pragma unroll
  for (int i = 0; i < kC; ++i) {
    const int at = 1024 * i + 16 * lane, r = at / kRow, ch = at % kRow / 16;
    ko[i] = k_lds_row(r) * kRow + Swizzle<D>::k_chunk(r, ch) * 16;
    vo[i] = r * kRow + (Swizzle<D>::v_block(r, ch >> 2) * 4 + (ch & 3)) * 16;
  }
  auto copy = [&](u32x4_t r, const uint32_t off[kC], int kb, uint32_t lds) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < kC; ++i)
        copy16_to_lds(r, off[i], (uint32_t)(2 * kb + u) * 16 * kRow, lds + 1024 * (u * kC + i));
  };
  int kb = ids.next(lane);
#pragma unroll
  for (int i = 0; i < G::kDChunks; ++i) asm volatile("" : "+v"(w.qf[i]));   // Q has landed: only copies count below
  if (kb >= 0) {
    copy(bk, ko, kb, lk);
    copy(bv, vo, kb, lv);
  }
  while (kb >= 0) {
    const int next = ids.next(lane);
    wait_copies<2 * kC>();                          // this tile's K; its V may be in flight
    u32x4_t kf[G::kDChunks];
#pragma unroll
    for (int i = 0; i < G::kDChunks; ++i) kf[i] = *(const u32x4_t*)(kt + ra.k[i]);
    f32x16_t s[1] = {f32x16_t{}};
#pragma unroll
    for (int i = 0; i < G::kDChunks; ++i) s[0] = mfma32x32x16(kf[i], w.qf[i], s[0]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // K read: its place is free
    if (next >= 0) copy(bk, ko, next, lk);
    if (kb == qb) WaveRows<D>::template mask<1>(s, q0, q0 + (lane & 31), lane);
    u32x4_t pb[2];
    w.template softmax<1>(s, pb, c);
    if (next >= 0) wait_copies<2 * kC>();           // this tile's V; the next K may be in flight
    else wait_copies<0>();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int t = 0; t < G::kDTiles; ++t) {
        const char* p = vt + ra.v[t] + 16 * ks * kRow;
        const u32x2_t lo = lds_read_tr16((const uint16_t*)p);
        const u32x2_t hi = lds_read_tr16((const uint16_t*)(p + 4 * kRow));
        w.o[t] = mfma32x32x16(u32x4_t{lo[0], lo[1], hi[0], hi[1]}, pb[ks], w.o[t]);
      }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // V read: its place is free
    if (next >= 0) copy(bv, vo, next, lv);
    kb = next;
  }
  w.finish(O + hoff, lse ? lse + (size_t)bh * n : nullptr, q0, lane);
}

// ---------------------------------------------------------------------------
// Block-sparse attention for 16-key blocks.  One one-wave work-group per
// (batch, head, query block) row on v_mfma_f32_16x16x32_bf16, whose 16 columns
// are the row's 16 queries.  A tile is any two consecutive blocks of the row's
// support.  S^T = K Q^T block by block, so lane 16 g + n holds keys
// 4 g .. 4 g + 3 of either block for query n: the two fours are the 8
// consecutive B entries of O^T = V^T P^T with the tile's keys taken in the
// order 4 g of a, 4 g of b, g = 0 .. 3, which the rows of the transposing V
// reads follow.  K and V are copied straight into LDS, one tile each (12 KB at
// d 96): the next tile's K as soon as this one's is in registers, its V after
// PV, so each has half a tile of work to land and 13 waves fit a CU.  A last
// tile with one block takes it twice and masks the copy.
//
// Bound by the L2: every row reads its own K and V, 99 million 128-byte requests
// (12.7 GB, 94% hits) at 4096 x 220 heads, d 96, density 0.28, 549 us or 23 TB/s.
// 840 -> 549 us there and 348 -> 262 us at 192 grouped heads of 64, against
// 32x32x16 MFMAs with the queries held twice and
// tiles staged through registers; K read straight into registers (64-byte
// pieces of rows, half the L2 rate) took 664 and 400 us.
// ---------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(D == 128 ? 3 : 4)))
sparse_row16_kernel(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                    const uint16_t* __restrict__ V, const int32_t* __restrict__ row_ptr,
                    const int32_t* __restrict__ col_idx, const int32_t* __restrict__ order,
                    uint16_t* __restrict__ O, float* __restrict__ lse, int n, int nb, int rows,
                    int heads, int gq, RowSched sc, float c) {
  constexpr int kC = D / 32;                        // MFMAs of a block's S^T; 1 KB copies of its V
  constexpr int kT = D / 16;                        // MFMAs of PV
  constexpr int kRow = 2 * D, kBlock = 16 * kRow;   // bytes
  __shared__ __attribute__((aligned(1024))) char kt[2 * kBlock], vt[2 * kBlock];
  int sh, sit;
  if (!row_slot(sc, sh, sit)) return;
  const int row = order ? order[sh * nb + sit] : sh * nb + (nb - 1 - sit);
  if ((unsigned)row >= (unsigned)rows) return;
  const int bh = row / nb, qb = row % nb;
  const size_t hoff = (size_t)bh * n * D;
  const int lane = threadIdx.x, g = lane >> 4, ln = lane & 15;
  const int q0 = 16 * qb;
  const size_t kvoff = (size_t)kv_head(bh, heads, gq) * n * D;
  const u32x4_t bk = buffer_words(K + kvoff), bv = buffer_words(V + kvoff);
  const uint32_t lk = lds_address(kt), lv = lds_address(vt);

  RowIds ids(row_ptr, col_idx, row, qb);            // the last valid id can be the diagonal
  auto next_tile = [&](int& a, int& b) {            // b < 0: a alone
    a = ids.next(lane);
    b = a < 0 ? -1 : ids.next(lane);
    return a >= 0;
  };

  u32x4_t qf[kC];
  const uint16_t* qr = Q + hoff + (size_t)(q0 + ln) * D + 8 * g;
#pragma unroll
  for (int i = 0; i < kC; ++i) qf[i] = *(const u32x4_t*)(qr + 32 * i);
  f32x4_t o[kT];
#pragma unroll
  for (int t = 0; t < kT; ++t) o[t] = f32x4_t{};
  float m = -INFINITY, l = 0.f;

  // V rows in LDS: 32-byte pieces permuted by row, so that the 8 rows a half
  // wave reads 32 bytes of fall on distinct banks.
  auto piece = [](int r, int p) {
    return D == 128 ? p ^ (r & 7) : D == 96 ? p ^ ((r >> 2) & 1) : p ^ ((r >> 1) & 3);
  };
  uint32_t ko[kC], vo[kC];                          // source bytes of this lane's copies in a block
#pragma unroll
  for (int i = 0; i < kC; ++i) {
    const int at = 1024 * i + 16 * lane, r = at / kRow, ch = at % kRow / 16;
    ko[i] = r * kRow + Swizzle<D>::k_chunk(r, ch) * 16;
    vo[i] = r * kRow + piece(r, ch >> 1) * 32 + (ch & 1) * 16;
  }
  const int vr = 4 * g + ((lane >> 2) & 3);         // row of this lane's transposing reads
  uint32_t ka[kC], va[kT];
#pragma unroll
  for (int i = 0; i < kC; ++i) ka[i] = ln * kRow + Swizzle<D>::k_chunk(ln, 4 * i + g) * 16;
#pragma unroll
  for (int t = 0; t < kT; ++t) va[t] = vr * kRow + piece(vr, t) * 32 + 8 * (lane & 3);

  auto copy = [&](u32x4_t r, const uint32_t off[kC], int x, int y, uint32_t lds) {
    const uint32_t sx = (uint32_t)x * kBlock, sy = (uint32_t)(y < 0 ? x : y) * kBlock;
#pragma unroll
    for (int i = 0; i < kC; ++i) copy16_to_lds(r, off[i], sx, lds + 1024 * i);
#pragma unroll
    for (int i = 0; i < kC; ++i) copy16_to_lds(r, off[i], sy, lds + kBlock + 1024 * i);
  };

  int a = -1, b = -1, an = -1, bn = -1;
  bool have = next_tile(a, b);
#pragma unroll
  for (int i = 0; i < kC; ++i) asm volatile("" : "+v"(qf[i]));   // Q has landed: only copies count below
  if (have) {
    copy(bk, ko, a, b, lk);
    copy(bv, vo, a, b, lv);
  }
  const int qi = q0 + ln;
  while (have) {
    const bool more = next_tile(an, bn);
    wait_copies<2 * kC>();                          // this tile's K; its V may be in flight
    u32x4_t kf[2][kC];
#pragma unroll
    for (int i = 0; i < kC; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) kf[u][i] = *(const u32x4_t*)(kt + ka[i] + u * kBlock);
    f32x4_t s[2] = {f32x4_t{}, f32x4_t{}};
#pragma unroll
    for (int i = 0; i < kC; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) s[u] = mfma16x16x32(kf[u][i], qf[i], s[u]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // K read: its place is free
    if (more) copy(bk, ko, an, bn, lk);
    if (!more) {   // the last tile: the diagonal block (if present) and a masked copy
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int blk = u ? b : a;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (blk < 0 || 16 * blk + 4 * g + i > qi) s[u][i] = -INFINITY;
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[u][i]);
    mx = quad_max(mx) * c;
    const bool grow = mx > m;
    if (__builtin_amdgcn_ballot_w64(grow)) {
      const float mn = grow ? mx : m;
      const float alpha = (mn == m) ? 1.f : fast_exp2(m - mn);
      l *= alpha;
#pragma unroll
      for (int t = 0; t < kT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("v_mul_f32 %0, %0, %1" : "+v"(o[t][i]) : "v"(alpha));
      m = mn;
    }
    const float mb = (m == -INFINITY) ? 0.f : m;
    u32x4_t pb;
    float ts = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[u][i] = fast_exp2(__builtin_fmaf(s[u][i], c, -mb));
        ts += s[u][i];
      }
      pb[2 * u] = pack_bf16x2(s[u][0], s[u][1]);
      pb[2 * u + 1] = pack_bf16x2(s[u][2], s[u][3]);
    }
    l += ts;
    if (more) wait_copies<2 * kC>();                // this tile's V; the next K may be in flight
    else wait_copies<0>();
#pragma unroll
    for (int t = 0; t < kT; ++t) {
      const u32x2_t lo = lds_read_tr16((const uint16_t*)(vt + va[t]));
      const u32x2_t hi = lds_read_tr16((const uint16_t*)(vt + va[t] + kBlock));
      o[t] = mfma16x16x32(u32x4_t{lo[0], lo[1], hi[0], hi[1]}, pb, o[t]);
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // V read: its place is free
    if (more) copy(bv, vo, an, bn, lv);
    a = an;
    b = bn;
    have = more;
  }
  const float lt = quad_sum(l);
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  uint16_t* orow = O + hoff + (size_t)qi * D + 4 * g;
#pragma unroll
  for (int t = 0; t < kT; ++t) {
    u32x2_t w;
    w[0] = pack_bf16x2(o[t][0] * inv, o[t][1] * inv);
    w[1] = pack_bf16x2(o[t][2] * inv, o[t][3] * inv);
    *(u32x2_t*)(orow + 16 * t) = w;
  }
  if (lse != nullptr && g == 0)
    lse[(size_t)bh * n + qi] = lt > 0.f ? (m + __builtin_log2f(lt)) * kLn2 : -INFINITY;
}

// ---------------------------------------------------------------------------
// Launchers (shapes already validated by the C ABI layer).
// ---------------------------------------------------------------------------
template <int D, int NW, int BM>
static void launch_dense_nw(const Dims& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                            uint16_t* O, float* lse, float* acc, float* ws, hipStream_t st) {
  const Sched sc = make_sched(s.bh, s.n / (NW * 32), (size_t)s.n * D * 4 / s.gq);
  hipLaunchKernelGGL((dense_attn_kernel<D, NW, BM>), dim3(sched_grid(sc)), dim3(NW * 64), 0, st,
                     Q, K, V, O, lse, s.n, s.heads, s.gq, sc, s.scale * kLog2e, acc, ws);
}

template <int D, int NW>
static void launch_dense_bm(const Dims& s, const uint16_t* Q, const uint16_t* K,
                            const uint16_t* V, uint16_t* O, float* lse, float* acc, float* ws,
                            hipStream_t st) {
  if (acc == nullptr) return launch_dense_nw<D, NW, 0>(s, Q, K, V, O, lse, acc, ws, st);
  if (s.block == 16) return launch_dense_nw<D, NW, 16>(s, Q, K, V, O, lse, acc, ws, st);
  if (s.block == 32) return launch_dense_nw<D, NW, 32>(s, Q, K, V, O, lse, acc, ws, st);
  if (s.block == 64) return launch_dense_nw<D, NW, 64>(s, Q, K, V, O, lse, acc, ws, st);
  if constexpr (NW >= 4) launch_dense_nw<D, NW, 128>(s, Q, K, V, O, lse, acc, ws, st);
}

template <int D>
static hipError_t launch_dense_d(const Dims& s, const void* q, const void* k, const void* v,
                                 void* o, float* lse, float* acc, float* ws, hipStream_t st) {
  const auto* Q = (const uint16_t*)q;
  const auto* K = (const uint16_t*)k;
  const auto* V = (const uint16_t*)v;
  // Queries per group (dense_query_tile): 256 for d 128 (each staged K/V tile
  // then feeds twice the MFMA work; 6-8% faster at 4K-32K, slower at d 64
  // and 96), else 128 when they divide n (always so for 128-key blocks).
  //
  // A grid of 8-wave groups that leaves CUs without a second group lasts as
  // long as its longest group, whose two waves per SIMD take turns at the
  // matrix cores: groups of 4 waves walk the same tiles with one.  256 CUs;
  // dense time in groups of 256 and of 128 queries, by the former's count: 16
  // (4096 x 1 head) 92 / 68 us, 64 (16384 x 1) 336 / 247, 128 (2048 x 16) 53.9
  // / 40.8, 192 (4096 x 12) 96.9 / 82.9, 256 (8192 x 8) 192 / 174, 320 (4096 x
  // 20) 110.9 / 104.2, 384 (8192 x 12) 223 / 217, 512 (16384 x 8) 500 / 504;
  // with 64-key masses 320: 116.7 / 114.1, 384: 122.1 / 124.9.  The same bits;
  // the mass workspace of 256-query tiles is the larger one.
  int qt = dense_query_tile(s);
  if (qt == 256 && (int64_t)s.bh * (s.n / 256) <= 320) qt = 128;
  if constexpr (D == 128) {
    if (qt == 256) {
      launch_dense_bm<D, 8>(s, Q, K, V, (uint16_t*)o, lse, acc, ws, st);
      return hipGetLastError();
    }
  }
  if (qt == 128) launch_dense_bm<D, 4>(s, Q, K, V, (uint16_t*)o, lse, acc, ws, st);
  else launch_dense_bm<D, 2>(s, Q, K, V, (uint16_t*)o, lse, acc, ws, st);
  return hipGetLastError();
}

hipError_t launch_dense(const Dims& s, const void* q, const void* k, const void* v, void* o,
                        float* lse, float* acc, void* ws, hipStream_t st) {
  switch (s.d) {
    case 64: return launch_dense_d<64>(s, q, k, v, o, lse, acc, (float*)ws, st);
    case 96: return launch_dense_d<96>(s, q, k, v, o, lse, acc, (float*)ws, st);
    default: return launch_dense_d<128>(s, q, k, v, o, lse, acc, (float*)ws, st);
  }
}

int dense_query_tile(const Dims& s) {
  if (s.d == 128 && s.n % 256 == 0) return 256;
  return s.n % 128 == 0 ? 128 : 64;
}

size_t mass_workspace_bytes(const Dims& s) {
  // Enough for dense_attn_kernel: tiles of T = dense_query_tile queries (fewer
  // need less), entries of E keys, tile qt holding (qt+1)*T/E entries of T
  // queries.
  const size_t e = s.block < 64 ? s.block : 64;
  const size_t qt = (size_t)dense_query_tile(s);
  const size_t nq = s.n / qt;
  return (size_t)s.bh * qt * (qt / e) * (nq * (nq + 1) / 2) * sizeof(float);
}

// 64-key-block rows up to which a group holds two tiles of each (sparse_attn_kernel).
// us with one / two, 4096 tokens, every block kept: d 64, 16 heads (1024 rows)
// 67.4 / 64.5, 17 heads at density 0.3 35.7 / 38.7; d 96, 20 heads 96.1 / 93.6,
// 24 heads 107 / 111; d 128, 12 heads 93.9 / 90.0, 14 heads 97.4 / 109.
template <int D>
constexpr int kSmallGrid = D == 64 ? 1024 : D == 96 ? 1280 : 768;

// LDS that a group leaves unused, so that four and not six groups of 64-key
// rows of d 96 share a CU.  With fewer than 2048 rows (8 groups a CU) six at once
// leave too few to even out what the first ones differ by.  us with six / four,
// 4096 tokens at density 0.3 and 1: 22 heads 60.8 / 54.5 and 136 / 125, 30 heads
// 64.5 / 58.3 and 148 / 142; 32 heads at 0.3 55.0 / 58.4.
template <int D>
static unsigned idle_lds(int rows) {
  return D == 96 && rows < 2048 ? 40960 - 2 * Swizzle<D>::kTile : 0;
}

template <int D, int NW, int kBufs>
static void launch_rows_of(const Dims& s, const RowSched& sc, unsigned idle, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                           const int32_t* rp, const int32_t* ci, const int32_t* order, uint16_t* o, float* lse, hipStream_t st) {
  hipLaunchKernelGGL((sparse_attn_kernel<D, NW, kBufs>), dim3(row_grid(sc)), dim3(NW * 64), 2 * kBufs * Swizzle<D>::kTile + idle, st,
                     Q, K, V, rp, ci, order, o, lse, s.n, s.nb, s.bh * s.nb, s.heads, s.gq, sc, s.scale * kLog2e);
}

template <int D>
static hipError_t launch_sparse_d(const Dims& s, const void* q, const void* k, const void* v,
                                  const int32_t* rp, const int32_t* ci, const int32_t* order,
                                  void* o, float* lse, hipStream_t st) {
  const float c = s.scale * kLog2e;
  const auto* Q = (const uint16_t*)q;
  const auto* K = (const uint16_t*)k;
  const auto* V = (const uint16_t*)v;
  const int rows = s.bh * s.nb;
  const RowSched sc = make_row_sched(s.bh, s.nb, (size_t)s.n * D * 4 / s.gq, s.block < 64);
  const dim3 grid(row_grid(sc));
  if (s.block == 16)
    hipLaunchKernelGGL((sparse_row16_kernel<D>), grid, dim3(64), 0, st, Q, K, V, rp, ci, order,
                       (uint16_t*)o, lse, s.n, s.nb, rows, s.heads, s.gq, sc, c);
  else if (s.block == 32)
    hipLaunchKernelGGL((sparse_row32_kernel<D>), grid, dim3(64), 0, st, Q, K, V, rp, ci, order,
                       (uint16_t*)o, lse, s.n, s.nb, rows, s.heads, s.gq, sc, c);
  else if (s.block == 128)
    launch_rows_of<D, 4, 2>(s, sc, 0, Q, K, V, rp, ci, order, (uint16_t*)o, lse, st);
  else if (rows <= kSmallGrid<D>)
    launch_rows_of<D, 2, 2>(s, sc, 0, Q, K, V, rp, ci, order, (uint16_t*)o, lse, st);
  else
    launch_rows_of<D, 2, 1>(s, sc, idle_lds<D>(rows), Q, K, V, rp, ci, order, (uint16_t*)o, lse, st);
  return hipGetLastError();
}

template <int D, int NW, int BR = 64>
static void launch_group_nw(const Dims& s, const void* q, const void* k, const void* v,
                            const int32_t* rp, const int32_t* ci, void* o, float* lse,
                            hipStream_t st) {
  const Sched sc = make_sched(s.bh, s.n / (NW * 32), (size_t)s.n * D * 4 / s.gq);
  hipLaunchKernelGGL((sparse_group_kernel<D, NW, BR>), dim3(sched_grid(sc)), dim3(NW * 64), 0, st,
                     (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, rp, ci,
                     (uint16_t*)o, lse, s.n, s.nb, s.heads, s.gq, sc, s.scale * kLog2e);
}

int sparse_group_rows(const Dims& s) {
  if (s.nb > 64 * kGroupMaskWords) return 0;
  const int qt = dense_query_tile(s);
  if (s.block == 64) return qt >= 128 ? qt / 64 : 0;
  if (s.block == 128) return qt == 256 ? 2 : 0;
  return 0;
}

hipError_t launch_sparse_grouped(const Dims& s, const void* q, const void* k, const void* v,
                                 const int32_t* rp, const int32_t* ci, void* o, float* lse,
                                 hipStream_t st) {
  const int rows = sparse_group_rows(s);
  if (s.block == 128) {
    if (rows == 2 && s.d == 128) launch_group_nw<128, 8, 128>(s, q, k, v, rp, ci, o, lse, st);
    else return launch_sparse(s, q, k, v, rp, ci, nullptr, o, lse, st);
  } else if (rows == 4 && s.d == 128) launch_group_nw<128, 8>(s, q, k, v, rp, ci, o, lse, st);
  else if (rows == 2 && s.d == 128) launch_group_nw<128, 4>(s, q, k, v, rp, ci, o, lse, st);
  else if (rows == 2 && s.d == 96) launch_group_nw<96, 4>(s, q, k, v, rp, ci, o, lse, st);
  else if (rows == 2 && s.d == 64) launch_group_nw<64, 4>(s, q, k, v, rp, ci, o, lse, st);
  else return launch_sparse(s, q, k, v, rp, ci, nullptr, o, lse, st);
  return hipGetLastError();
}

hipError_t launch_sparse(const Dims& s, const void* q, const void* k, const void* v,
                         const int32_t* rp, const int32_t* ci, const int32_t* order, void* o,
                         float* lse, hipStream_t st) {
  switch (s.d) {
    case 64: return launch_sparse_d<64>(s, q, k, v, rp, ci, order, o, lse, st);
    case 96: return launch_sparse_d<96>(s, q, k, v, rp, ci, order, o, lse, st);
    default: return launch_sparse_d<128>(s, q, k, v, rp, ci, order, o, lse, st);
  }
}

}  // namespace wise
