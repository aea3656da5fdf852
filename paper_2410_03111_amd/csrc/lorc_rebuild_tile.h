// Internal: the rank-r rebuild K^T = B_k^T C_k^T (or V^T = B_v^T C_v^T) as a tiled matrix product: one workgroup of four
// waves takes two cached pages (128 positions) times 64 * NC output columns and walks the rank.  Shared by the prefill
// rebuild and by the scores of the three-launch decode.
#ifndef LORC_REBUILD_TILE_H_
#define LORC_REBUILD_TILE_H_

#include "lorc_device.h"

namespace lorc {

// Both operands pass through an LDS ring of three slots of two k-steps (32 latent indices) each, filled two slots ahead
// by direct global -> LDS copies: NC = 4: 16 KiB of factor + 8 KiB of latents per slot, 72 KiB, so two workgroups share
// a CU and one multiplies while the other waits at a barrier or runs its epilogue.  Every factor operand read from LDS
// feeds two matrix-core ops, every latent operand NC.
constexpr int kRtSlots = 3;
template <int NC>
constexpr int rt_slot_bytes() { return (4 * NC + 8) * 1024; }
template <int NC>
constexpr int rt_ring_bytes() { return kRtSlots * rt_slot_bytes<NC>(); }

// Column block (of 32 columns) number q of a workgroup: wave w multiplies the blocks q = (w & 1) * NC + c, c < NC, with
// the positions of page w >> 1.  The blocks c and c + NC / 2 (head_dim 128) or c and c + 1 (64) of a wave are RoPE
// partners, so NC = 2 and head_dim 128 deals the blocks of a head to the waves as (0, 2) and (1, 3).
template <int HD, int NC>
__device__ __forceinline__ constexpr int rt_col_block(int q) { return HD == 128 && NC == 2 ? (q >> 1) + 2 * (q & 1) : q; }

// acc[c][pb] += factor block c x latents of position block pb, over all nks k-steps (nks even).
//   factor   : descriptor of the packed factor tiles;  cb0: first column block of the workgroup, ncb: blocks in all
//              (a block past the last repeats it; its results are not to be used)
//   latents  : descriptor of the K (or V) part of page w >> 1 (size zero: a page that is not cached reads as zeros)
// VALUES: the latents are in the V tiling (a lane holds 8 positions of one latent index): they are transposed on the
// way from LDS to registers (ds_read_b64_tr_b16), and the operands change places, so that a lane owns an output column
// and its registers walk the positions.  The 16-byte pieces of a V block are permuted as they are copied (a lane may
// fetch any piece of the block), which puts the pieces that a transposed read touches together in different banks.
template <int HD, int NC, bool VALUES>
__device__ __forceinline__ void rebuild_tile(f32x16 (&acc)[NC][2], unsigned char* ring, u32x4 factor, u32x4 latents, int cb0, int ncb,
                                             int nks, int w, int lane) {
  constexpr int COPIES = NC + 2;  // per wave and slot
  const int hf = lane >> 5;
  const uint32_t ring_off = (uint32_t)(uintptr_t)ring, lane16 = (uint32_t)lane * 16u;
  const int n_kt = nks >> 1;
  uint32_t fsrc[NC / 2];  // source of this wave's factor copies (byte offset of k-step 0)
#pragma unroll
  for (int j = 0; j < NC / 2; ++j) {
    const int q = w * (NC / 2) + j, cb = cb0 + rt_col_block<HD, NC>(q);
    fsrc[j] = (uint32_t)((cb < ncb ? cb : ncb - 1) * nks) * 1024u;
  }
  // V block s16 = 2 (w & 1) + i: LDS piece l holds source piece (j ^ 4 hi ^ 8 (s16 & 1)) + 32 hi, j = l % 32, hi = l / 32
  uint32_t vlane[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) vlane[i] = (uint32_t)((((lane & 31) ^ (4 * hf) ^ (8 * i)) + 32 * hf) * 16);
  auto issue = [&](int kt, uint32_t slot) {
#pragma unroll
    for (int j = 0; j < NC / 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        dma_1k(factor, ring_off + slot + (uint32_t)((w * (NC / 2) + j) * 2 + ks) * 1024u, lane16, fsrc[j] + (uint32_t)(2 * kt + ks) * 1024u);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t dst = ring_off + slot + (uint32_t)(4 * NC + 2 * w + i) * 1024u;
      if constexpr (VALUES) dma_1k(latents, dst, vlane[i], (uint32_t)(4 * kt + 2 * (w & 1) + i) * 1024u);
      else dma_1k(latents, dst, lane16, (uint32_t)((w & 1) * nks + 2 * kt + i) * 1024u);
    }
  };
  const unsigned char* fbase = ring + (size_t)(w & 1) * NC * 2048 + lane16;
  const unsigned char* lbase;
  uint32_t tr1 = 0;  // distance from the first to the second transposed read of an operand
  if constexpr (VALUES) {
    // 16-lane group: positions 16 (group & 1) .. + 15 of the block, latent indices 16 ks + 8 hf + 4 r .. + 3 (read r);
    // lane i of it addresses index i / 4, positions 4 (i % 4) .. + 3
    const int i = lane & 15, s = (lane >> 4) & 1, hi = (i >> 1) & 1;
    const int j0 = (8 * hf + (i >> 2)) ^ (4 * hi) ^ (8 * s);
    lbase = ring + (size_t)(4 * NC + 4 * (w >> 1) + s) * 1024 + (j0 + 32 * hi) * 16 + (i & 1) * 8;
    tr1 = hi ? -64u : 64u;  // bit 2 of the index flips
  } else {
    lbase = ring + (size_t)(4 * NC + 4 * (w >> 1)) * 1024 + lane16;
  }
  issue(0, 0);
  if (n_kt > 1) issue(1, rt_slot_bytes<NC>());
  uint32_t slot = 0;
  for (int kt = 0; kt < n_kt; ++kt) {
    // this k-tile's copies have landed (the next one's may be in flight), and every wave is through the previous
    // k-tile, whose slot takes the copies of k-tile kt + 2
    if (kt + 1 < n_kt) dma_barrier<COPIES>();
    else dma_barrier<0>();
    if (kt + 2 < n_kt) issue(kt + 2, slot == 0 ? 2 * rt_slot_bytes<NC>() : slot - rt_slot_bytes<NC>());
    const unsigned char* fs = fbase + slot;
    const unsigned char* ls = lbase + slot;
    bf16x8 a[2][NC], b[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int pb = 0; pb < 2; ++pb) {
        if constexpr (VALUES) {
          typedef __attribute__((ext_vector_type(4))) short s16x4;
          typedef __attribute__((ext_vector_type(8))) short s16x8;
          const unsigned char* src = ls + pb * 2048 + ks * 256;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(src + (int)tr1));
          const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          b[ks][pb] = __builtin_bit_cast(bf16x8, both);
        } else {
          b[ks][pb] = load_frag(reinterpret_cast<const uint16_t*>(ls + (pb * 2 + ks) * 1024));
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) a[ks][c] = load_frag(reinterpret_cast<const uint16_t*>(fs + (c * 2 + ks) * 1024));
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int pb = 0; pb < 2; ++pb)
          acc[c][pb] = VALUES ? mfma32(b[ks][pb], a[ks][c], acc[c][pb]) : mfma32(a[ks][c], b[ks][pb], acc[c][pb]);
    slot = slot == 2 * rt_slot_bytes<NC>() ? 0 : slot + rt_slot_bytes<NC>();
  }
}

}  // namespace lorc
#endif  // LORC_REBUILD_TILE_H_
