// Internal: tiled matrix product of one group of four waves: 64 * NC rows of a factor in operand tiles times 128 token
// positions, contracted over the rank (the rebuild K^T = B_k^T C_k^T or V^T = B_v^T C_v^T of two cached pages) or over the
// model dimension (the down-projection C^T = A^T X^T of 128 tokens).
#ifndef LORC_TILE_PRODUCT_H_
#define LORC_TILE_PRODUCT_H_

#include "lorc_device.h"

namespace lorc {

// Both operands pass through an LDS ring of NS slots of two k-steps each (NC = 4: 16 KiB of factor + 8 KiB of positions per
// slot), filled NS - 1 slots ahead of their use by direct global -> LDS copies.  Every factor operand read from LDS feeds two
// matrix-core ops, every position operand NC.
template <int NC, int NS, int KT = 2>
constexpr int rt_ring_bytes() { return NS * KT * (2 * NC + 4) * 1024; }

// Column block (of 32 columns) number q of a workgroup: wave w multiplies the blocks q = (w & 1) * NC + c, c < NC, with
// the positions of page w >> 1.  The blocks c and c + NC / 2 (head_dim 128) or c and c + 1 (64) of a wave are RoPE
// partners in the rebuild, so NC = 2 and head_dim 128 deals the blocks of a head to the waves as (0, 2) and (1, 3).
template <int HD, int NC>
__device__ __forceinline__ constexpr int rt_col_block(int q) { return HD == 128 && NC == 2 ? (q >> 1) + 2 * (q & 1) : q; }

// How the positions' operand lies in memory.
enum TileSource {
  kPageKeys,    // K part of a page: 1 KiB operand blocks
  kPageValues,  // V part of a page: a lane holds 8 positions of one latent index.  The operand is transposed on the way
                // from LDS to registers (ds_read_b64_tr_b16); the 16-byte pieces of a block are permuted as they are copied
                // (a lane may fetch any piece), which puts those that a transposed read touches together in different banks
  kRows         // row-major tokens, `row_bytes` apart: 64 bytes of a row per k-tile, pieces permuted likewise
};

// acc[c][pb] += factor block c x operand of position block pb, over n_kt k-tiles of two k-steps.
//   factor   : descriptor of the factor tiles, nks k-steps per column block;  cb0: first column block of the workgroup,
//              ncb: blocks in all (a block past the last repeats it; its results are not to be used)
//   source   : descriptor of the K (or V) part of page w >> 1 (size zero: a page that is not cached reads as zeros), or of
//              the tile's token rows (rows past its size read as zeros)
//   setup    : called once the first copies are on their way; its LDS writes outside the ring are visible afterwards
// SWAP: the operands change places, so that a lane owns a factor column and its registers walk the positions.
struct NoSetup { __device__ __forceinline__ void operator()() const {} };
template <int HD, int NC, int NS, TileSource SRC, bool SWAP, int KT = 2, class Setup = NoSetup>
__device__ __forceinline__ void tile_product(f32x16 (&acc)[NC][2], unsigned char* ring, u32x4 factor, u32x4 source, int cb0, int ncb,
                                             int nks, int w, int lane, int n_kt, uint32_t row_bytes = 0, Setup setup = Setup{}) {
  static_assert(KT == 2 || (KT == 4 && SRC == kRows), "k-steps per slot");
  constexpr int FC = NC * KT / 2, COPIES = FC + KT;  // copies per wave and slot
  const int hf = lane >> 5;
  const uint32_t ring_off = (uint32_t)(uintptr_t)ring, lane16 = (uint32_t)lane * 16u;
  uint32_t fsrc[NC / 2];  // source of this wave's factor copies (byte offset of k-step 0)
#pragma unroll
  for (int j = 0; j < NC / 2; ++j) {
    const int q = w * (NC / 2) + j, cb = cb0 + rt_col_block<HD, NC>(q);
    fsrc[j] = (uint32_t)((cb < ncb ? cb : ncb - 1) * nks) * 1024u;
  }
  uint32_t vlane[KT];
#pragma unroll
  for (int i = 0; i < KT; ++i) {
    // V block s16 = 2 (w & 1) + i: LDS piece l holds source piece (j ^ 4 hi ^ 8 (s16 & 1)) + 32 hi, j = l % 32, hi = l / 32
    if constexpr (SRC == kPageValues) vlane[i] = (uint32_t)((((lane & 31) ^ (4 * hf) ^ (8 * i)) + 32 * hf) * 16);
    // token rows 32 w + 16 i + l / 4: LDS piece l holds the row's piece (l % 4) ^ (row / 4 % 4) of the k-tile
    if constexpr (SRC == kRows && KT == 2) vlane[i] = (uint32_t)(32 * w + 16 * i + (lane >> 2)) * row_bytes + (uint32_t)((lane & 3) ^ (lane >> 4)) * 16u;
    // token rows 32 w + 8 i + l / 8: LDS piece l holds the row's piece (l % 8) ^ (row % 8)
    if constexpr (SRC == kRows && KT == 4) vlane[i] = (uint32_t)(32 * w + 8 * i + (lane >> 3)) * row_bytes + (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;
  }
  const unsigned char* fbase = ring + (size_t)(w & 1) * NC * KT * 1024 + lane16;
  const unsigned char* lbase;
  uint32_t tr1 = 0;  // kPageValues: distance from the first to the second transposed read of an operand; kRows: of k-step 0 to 1
  if constexpr (SRC == kRows && KT == 4) {
    lbase = ring + (size_t)(2 * NC * KT + 2 * KT * (w >> 1)) * 1024 + (lane & 31) * 128;
  } else if constexpr (SRC == kRows) {
    const int piece = hf ^ ((lane >> 2) & 3);  // of row l32 of a position block (two blocks of 16 rows); k-step 1: piece ^ 2
    lbase = ring + (size_t)(4 * NC + 4 * (w >> 1)) * 1024 + (lane & 31) * 64 + piece * 16;
    tr1 = piece & 2 ? -32u : 32u;
  } else if constexpr (SRC == kPageValues) {
    // 16-lane group: positions 16 (group & 1) .. + 15 of the block, latent indices 16 ks + 8 hf + 4 r .. + 3 (read r);
    // lane i of it addresses index i / 4, positions 4 (i % 4) .. + 3
    const int i = lane & 15, s = (lane >> 4) & 1, hi = (i >> 1) & 1;
    const int j0 = (8 * hf + (i >> 2)) ^ (4 * hi) ^ (8 * s);
    lbase = ring + (size_t)(4 * NC + 4 * (w >> 1) + s) * 1024 + (j0 + 32 * hi) * 16 + (i & 1) * 8;
    tr1 = hi ? -64u : 64u;  // bit 2 of the index flips
  } else {
    lbase = ring + (size_t)(4 * NC + 4 * (w >> 1)) * 1024 + lane16;
  }
  auto factor_at = [&](const unsigned char* fs, int ks, int c) { return load_frag(reinterpret_cast<const uint16_t*>(fs + (c * KT + ks) * 1024)); };
  auto source_at = [&](const unsigned char* ls, int ks, int pb) {
    if constexpr (SRC == kRows && KT == 4) {
      return load_frag(reinterpret_cast<const uint16_t*>(ls + pb * 4096 + (((2 * ks + hf) ^ (lane & 7)) * 16)));
    } else if constexpr (SRC == kRows) {
      return load_frag(reinterpret_cast<const uint16_t*>(ls + pb * 2048 + (int)(ks ? tr1 : 0u)));
    } else if constexpr (SRC == kPageValues) {
      typedef __attribute__((ext_vector_type(4))) short s16x4;
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      const unsigned char* src = ls + pb * 2048 + ks * 256;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + (int)tr1));
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, both);
    } else {
      return load_frag(reinterpret_cast<const uint16_t*>(ls + (pb * 2 + ks) * 1024));
    }
  };
  // k-tiles past the last one are asked for with descriptors of size zero: the number of copies in flight stays fixed and
  // nothing is fetched
  u32x4 factor_kt = factor, source_kt = source;
  auto select_tile = [&](int kt) {
    factor_kt[2] = kt < n_kt ? factor[2] : 0u;
    source_kt[2] = kt < n_kt ? source[2] : 0u;
  };
  auto copy_one = [&](int kt, uint32_t slot, int i) {
    if (i < FC) {
      const int j = i / KT, ks = i % KT;
      dma_1k(factor_kt, ring_off + slot + (uint32_t)((w * (NC / 2) + j) * KT + ks) * 1024u, lane16, fsrc[j] + (uint32_t)(KT * kt + ks) * 1024u);
    } else {
      const int u = i - FC;
      const uint32_t dst = ring_off + slot + (uint32_t)(2 * NC * KT + KT * w + u) * 1024u;
      if constexpr (SRC == kPageValues) dma_1k(source_kt, dst, vlane[u], (uint32_t)(4 * kt + 2 * (w & 1) + u) * 1024u);
      else if constexpr (SRC == kRows) dma_1k(source_kt, dst, vlane[u], (uint32_t)kt * (KT * 32u));
      else dma_1k(source_kt, dst, lane16, (uint32_t)((w & 1) * nks + 2 * kt + u) * 1024u);
    }
  };
  constexpr int SLOT = rt_ring_bytes<NC, 1, KT>();
  bf16x8 a[2][KT][NC], b[2][KT][2];  // operands of the k-tile that is multiplied and of the next one: [set][k-step]
  constexpr int READS = KT * (NC + 2), PRODUCTS = 2 * KT * NC;
  auto read_one = [&](auto set_c, const unsigned char* fs, const unsigned char* ls, auto i_c) {  // in the order of use
    constexpr int SET = decltype(set_c)::value, ks = decltype(i_c)::value / (NC + 2), i = decltype(i_c)::value % (NC + 2);
    if constexpr (i < 2) b[SET][ks][i] = source_at(ls, ks, i);
    else a[SET][ks][i - 2] = factor_at(fs, ks, i - 2);
  };
  uint32_t s_cur = 0, s_next = SLOT;  // slots of k-tiles kt and kt + 1
  // Products of k-tile kt, in a pinned order; between them the operand reads of k-tile kt + 1 (a whole k-tile ahead of
  // their use: an in-order wave that asks LDS for an operand shortly before its product waits for it) and the copies of
  // k-tile kt + NS into the slot that k-tile kt, all in registers by now, has left.
  auto k_tile = [&](auto set_c, int kt) {
    constexpr int SET = decltype(set_c)::value;
    dma_barrier<(NS - 2) * COPIES>();  // k-tile kt + 1 has landed, younger ones may be in flight
    const int k_new = kt + NS;
    select_tile(k_new);
    const unsigned char *fs = fbase + s_next, *ls = lbase + s_next;
    static_for<PRODUCTS>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value, ks = i / (2 * NC), c = (i % (2 * NC)) >> 1, pb = i & 1;
      acc[c][pb] = SWAP ? mfma32(b[SET][ks][pb], a[SET][ks][c], acc[c][pb]) : mfma32(a[SET][ks][c], b[SET][ks][pb], acc[c][pb]);
      if constexpr (i < READS) read_one(std::integral_constant<int, SET ^ 1>{}, fs, ls, i_c);
      if constexpr (i % 2 == 1 && i / 2 < COPIES) copy_one(k_new, s_cur, i / 2);
      __builtin_amdgcn_sched_barrier(0);
    });
    s_cur = s_next;
    s_next = s_next == (NS - 1) * SLOT ? 0u : s_next + SLOT;
  };
  static_assert(READS <= PRODUCTS && 2 * COPIES <= PRODUCTS, "one read per product, one copy per two");
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    select_tile(t);
#pragma unroll
    for (int i = 0; i < COPIES; ++i) copy_one(t, t * SLOT, i);
  }
  setup();
  dma_barrier<(NS - 1) * COPIES>();
  static_for<READS>([&](auto i_c) { read_one(std::integral_constant<int, 0>{}, fbase, lbase, i_c); });
  for (int kt = 0; kt < n_kt; kt += 2) {
    k_tile(std::integral_constant<int, 0>{}, kt);
    if (kt + 1 < n_kt) k_tile(std::integral_constant<int, 1>{}, kt + 1);
  }
  __builtin_amdgcn_s_waitcnt(0);  // the copies past the end have written their zeros before the ring is reused
}

}  // namespace lorc
#endif  // LORC_TILE_PRODUCT_H_
