// Causal prefill attention over the latent cache (Eq. 1 with the mask j <= i; GQA of Section 4.3; RoPE applied
// to rebuilt keys as in the Appendix on the adjusted position embedding).
//
// Two launches per call:
//   rebuild : a tiled matrix product over (two pages) x (64 NC columns), keys and values alike (lorc_tile_product.h).
//             Keys are rotated in registers and written once to scratch as fp16; values likewise, transposed.
//   attend  : flash-style causal attention.  One workgroup per (sequence, 64-query block, KV head); each wave
//             owns one query head of the group.  S^T = K Q^T so that a lane owns one query column: row maxima
//             and sums need a single cross-lane exchange, the P^T accumulators are re-used in place as the
//             B operand of O^T += V^T P^T, and rescaling is a per-lane scalar.
// The scratch is laid out in the attention kernel's operand order (krot_block, vt_block below), so that both launches
// move whole KiB blocks: one store instruction of the rebuild = one operand of the attention.
#include <type_traits>

#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_rebuild.h"
#include "lorc_tile_product.h"

namespace lorc {

constexpr float kNegInfP = -__builtin_huge_valf();


// Scratch layout, in 1 KiB operand blocks of 64 lanes x 8 fp16; page = sequence * tiles_per_seq + page of the sequence.
// Keys: block (page, KV head, pb, u): lane (l32, hf) holds position 32 pb + l32 and, as element e, head-dim coordinate
// 16 u + 8 (e >> 2) + 4 hf + (e & 3).  Values: block (page, KV head, db, v): lane (l32, hf) holds coordinate 32 db + l32
// and, as element e, position 16 v + 8 (e >> 2) + 4 hf + (e & 3).  Both orders are those in which a 32x32 accumulator
// block lies in registers (eight consecutive registers = one lane's 16 bytes), and the V order is also the one in which
// the attention kernel's P accumulators serve as operands.
template <int HD>
__device__ __forceinline__ size_t krot_block(int page, int h_kv, int g, int pb, int u) {
  return ((((size_t)page * h_kv + g) * 2 + pb) * (HD / 16) + u) * 512;
}
template <int HD>
__device__ __forceinline__ size_t vt_block(int page, int h_kv, int g, int db, int v) {
  return ((((size_t)page * h_kv + g) * (HD / 32) + db) * 4 + v) * 512;
}

// Positions of a sequence, as far as its scratch reaches: the launch is sized by the host's max_seqlen, and a longer entry of
// cu_seqlens, which only the device sees, must not lead past the sequence's pages (rows beyond them are left as they are).
__device__ __forceinline__ int prompt_len(const PrefillParams& p, int seq) {
  const int len = p.cu_seqlens[seq + 1] - p.cu_seqlens[seq];
  return len < p.lp ? len : p.lp;
}

// ------------------------------------------------------------------------------------------------ rebuild
// One workgroup per (two pages of a sequence, 64 NC columns of K or of V).  At large sizes two workgroups per CU keep the matrix
// cores busy 42 % (rank 512) to 54 % (rank 2048) of the time at the 1.75 and 1.93 GHz that the power limit leaves (counters;
// 2 (r_k + r_v) n flop per position: 800 and 1030 TFLOP/s), the rest is prologue, rotation and stores; at small ones the chip's
// width decides, which is why the columns are dealt to workgroups of their own: before, one workgroup per page walked all
// columns, and the 8B shape's 53-page batch ran on 53 of 256 CUs, a rank-2048 layer copied its latents to LDS once for every
// eight heads.
//   8B, rank 512, 4 x 8192 positions: 114 -> 82 us.  8B, rank 576, 3116 positions in 6 prompts: 59 -> 18 us.
//   13B, rank 2048, 3378 positions in 3 prompts (142 GFLOP): 1277 -> 137 us.
// NC = 4 unless its workgroups do not cover the CUs twice; NC = 2 then doubles their number.
constexpr int kRebuildColGroups = 8;  // column groups whose workgroups run side by side on an XCD
constexpr int kRebuildFewTiles = 64;
__host__ __device__ inline bool rebuild_by_column(int n_pt, int ncg) { return n_pt < kRebuildFewTiles && 2 * ncg >= 8; }

template <int HD, int NC>
__global__ __launch_bounds__(256, 2) void prefill_rebuild_kernel(PrefillParams p) {
  constexpr int HALF = HD / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Block id -> (position tile, column group of K or V); an XCD takes the block ids of one residue mod 8.
  //  * many position tiles: an XCD takes every eighth tile; on it, the column groups run kRebuildColGroups at a time over
  //    all of its tiles, so that the workgroups in flight share a few factor slices and latent tiles in the XCD's L2;
  //  * fewer than kRebuildFewTiles: an XCD takes every eighth column group and all tiles.  Its share then does not depend
  //    on which tiles the prompts' lengths leave empty (13B, prompts of 1500, 688 and 1190: 227 -> 160 us).
  const int ncb = p.h_kv * HD / 32, ncg = (ncb + 2 * NC - 1) / (2 * NC);  // column blocks of 32; groups of K (and of V)
  const int tps2 = (p.tiles_per_seq + 1) >> 1, n_pt = p.b * tps2;
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  int pt, cgi;
  if (rebuild_by_column(n_pt, ncg)) {
    pt = idx % n_pt;
    cgi = idx / n_pt * 8 + xcd;
    if (cgi >= 2 * ncg) return;
  } else {
    const int t8 = (n_pt + 7) >> 3, chunk = idx / (t8 * kRebuildColGroups), rest = idx - chunk * t8 * kRebuildColGroups;
    const int left = 2 * ncg - chunk * kRebuildColGroups, width = left < kRebuildColGroups ? left : kRebuildColGroups;
    pt = (rest / width) * 8 + xcd;
    cgi = chunk * kRebuildColGroups + rest % width;
  }
  if (pt >= n_pt) return;
  const int seq = pt / tps2, page0 = (pt - seq * tps2) * 2;
  const int len = prompt_len(p, seq);
  if (page0 * kPage >= len) return;
  const bool values = cgi >= ncg;
  const int cb0 = (values ? cgi - ncg : cgi) * 2 * NC;

  const int my_page = page0 + (w >> 1), pos0 = my_page * kPage;  // the wave's page of the sequence
  const bool live = pos0 < len;
  const int id = live ? p.block_table[(size_t)seq * p.max_pages + my_page] : -1;
  const bool page_ok = id >= 0 && id < p.n_pages;
  const uint16_t* page = p.cache + (size_t)(page_ok ? id : 0) * p.page_elems;
  const int n = p.h_kv * HD, spage = seq * p.tiles_per_seq + my_page;

  f32x16 acc[NC][2];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[c][pb][j] = 0.f;

  if (!values) {
    // Rotations of the four position blocks' first positions (angles reduced in fp64).  A key's rotation is its block's times
    // that of its offset inside the block, from the packed table.  (One fp32 angle per key in the hardware sine and cosine takes
    // 0.1 to 0.5 us less per call -- 8B rank 576, six prompts: 106.4 against 107.0 -- but rounds a fifth to a third more keys to the
    // wrong fp16 value.)
    float2* cs_base = reinterpret_cast<float2*>(smem + rt_ring_bytes<NC, 3>());
    const double theta = p.rope_tab[tid % HALF];
    float2 cl[16];  // offsets of pair pr; NC = 2 has the registers to ask for them ahead of the product
    auto offsets = [&](int pr) {
      const int fbase = 32 * ((cb0 + rt_col_block<HD, NC>((w & 1) * NC + (HD == 128 ? pr : 2 * pr))) % (HD / 32));
#pragma unroll
      for (int j = 0; j < 16; ++j) cl[j] = p.lane_cs[l32 * HALF + fbase + acc_row(j, hf)];
    };
    if constexpr (NC == 2) offsets(0);
    __builtin_amdgcn_sched_barrier(0);  // (asked for behind the copies, either would wait for them)
    auto setup = [&]() {  // behind the product's first copies
      if (tid < 4 * HALF) cs_base[tid] = cos_sin_reduced((double)(page0 * kPage + 32 * (tid / HALF)) * theta);
    };
    tile_product<HD, NC, 3, kPageKeys, false>(acc, smem, dma_rsrc(p.bk, (uint32_t)n * p.r_k * 2u), dma_rsrc(page, page_ok ? (uint32_t)kPage * p.r_k * 2u : 0u),
                                cb0, ncb, p.r_k >> 4, w, lane, p.r_k >> 5, 0, setup);
    if (!live) return;
#pragma unroll
    for (int pr = 0; pr < NC / 2; ++pr) {  // pairs of RoPE partner blocks
      const int ca = HD == 128 ? pr : 2 * pr, cc = HD == 128 ? pr + NC / 2 : 2 * pr + 1;
      const int cb = cb0 + rt_col_block<HD, NC>((w & 1) * NC + ca);
      if (cb >= ncb) continue;
      const int g = cb / (HD / 32), fbase = 32 * (cb % (HD / 32));
      if constexpr (NC != 2) offsets(pr);
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          f16x8 lo, hi;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int j = 8 * u + e;
            const float2 bt = cs_base[(2 * (w >> 1) + pb) * HALF + fbase + acc_row(j, hf)];
            const float cs = bt.x * cl[j].x - bt.y * cl[j].y, sn = bt.y * cl[j].x + bt.x * cl[j].y;
            const float x = acc[ca][pb][j], y = acc[cc][pb][j];
            lo[e] = static_cast<_Float16>(x * cs - y * sn);
            hi[e] = static_cast<_Float16>(y * cs + x * sn);
          }
          *reinterpret_cast<f16x8*>(p.krot + krot_block<HD>(spage, p.h_kv, g, pb, fbase / 16 + u) + lane * 8) = lo;
          *reinterpret_cast<f16x8*>(p.krot + krot_block<HD>(spage, p.h_kv, g, pb, (fbase + HALF) / 16 + u) + lane * 8) = hi;
        }
    }
  } else {
    const unsigned char* vpart = reinterpret_cast<const unsigned char*>(page) + (page_ok ? (size_t)kPage * p.r_k * 2 : 0);
    tile_product<HD, NC, 3, kPageValues, true>(acc, smem, dma_rsrc(p.bv, (uint32_t)n * p.r_v * 2u), dma_rsrc(vpart, page_ok ? (uint32_t)kPage * p.r_v * 2u : 0u),
                               cb0, ncb, p.r_v >> 4, w, lane, p.r_v >> 5);
    if (!live) return;
    const bool ragged = !page_ok || pos0 + kPage > len;  // slots past the sequence hold anything: written as zeros
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int cb = cb0 + rt_col_block<HD, NC>((w & 1) * NC + c);
      if (cb >= ncb) continue;
      const int g = cb / (HD / 32), db = cb % (HD / 32);
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          f16x8 v;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int j = 8 * u + e;
            float x = acc[c][pb][j];
            if (ragged && (!page_ok || pos0 + 32 * pb + acc_row(j, hf) >= len)) x = 0.f;
            v[e] = static_cast<_Float16>(x);
          }
          *reinterpret_cast<f16x8*>(p.vt + vt_block<HD>(spage, p.h_kv, g, db, 2 * pb + u) + lane * 8) = v;
        }
    }
  }
}

// ------------------------------------------------------------------------------------------------ uncompressed layers
// The rebuild launch for a layer whose pages hold the keys and values themselves (rank = n, no read-side factors):
// nothing to multiply.  One workgroup per (sequence, page); wave w takes position block w % 2 and the KV heads of
// parity w / 2.  Keys: a lane of a K operand block holds one position and 8 consecutive head-dim coordinates, its
// rotation partner the same lane and element four blocks further; rotated (angles reduced in fp64, hardware sine /
// cosine in turns) and rounded to fp16.  Values: a lane of a V operand block holds one column and 8 consecutive
// positions.  Both blocks differ from the scratch's only in which half of the wave holds which four of sixteen
// elements (permute_halves).  Slots past the sequence and pages that are not cached are written as zeros.

__global__ __launch_bounds__(256, 2) void prefill_plain_gather_kernel(PrefillParams p) {
  constexpr int HD = 128, T = 64;
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seq = blockIdx.x / p.tiles_per_seq, tile = blockIdx.x % p.tiles_per_seq;
  const int len = prompt_len(p, seq);
  const int pos0 = tile * T;
  if (pos0 >= len) return;
  const int n = p.h_kv * HD, pb = w & 1;
  const int id = p.block_table[(size_t)seq * p.max_pages + tile];
  const bool page_ok = id >= 0 && id < p.n_pages;
  const uint16_t* page = uniform_ptr(p.cache + (size_t)(page_ok ? id : 0) * p.page_elems);
  const __amdgpu_buffer_rsrc_t pr = make_rsrc(page, page_ok ? (uint32_t)kPage * 2u * n * 2u : 0u);  // K part, then V part

  float cs_c[4][8], cs_s[4][8];
  {
    const double pos = (double)(pos0 + 32 * pb + l32);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double turns = pos * p.rope_tab[16 * kb + 8 * hf + e] * 0.15915494309189533576888;
        const float fr = (float)(turns - rint(turns));
        cs_c[kb][e] = __builtin_amdgcn_cosf(fr);
        cs_s[kb][e] = __builtin_amdgcn_sinf(fr);
      }
  }
  const int blocks_per_row = n >> 4;
  const bool k_live = pos0 + 32 * pb + l32 < len;
  const int spage = seq * p.tiles_per_seq + tile;
  for (int g = w >> 1; g < p.h_kv; g += 2) {
    u32x4 raw[8];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
      raw[kb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(pr, lane * 16, (pb * blocks_per_row + g * 8 + kb) * 1024, 0));
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      uint16_t lo[8], hi[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = bf16_to_float((uint16_t)(raw[kb][e >> 1] >> (16 * (e & 1))));
        const float y = bf16_to_float((uint16_t)(raw[kb + 4][e >> 1] >> (16 * (e & 1))));
        lo[e] = k_live ? f16_bits(x * cs_c[kb][e] - y * cs_s[kb][e]) : (uint16_t)0;
        hi[e] = k_live ? f16_bits(y * cs_c[kb][e] + x * cs_s[kb][e]) : (uint16_t)0;
      }
      u32x4 plo, phi;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        plo[c] = (uint32_t)lo[2 * c] | ((uint32_t)lo[2 * c + 1] << 16);
        phi[c] = (uint32_t)hi[2 * c] | ((uint32_t)hi[2 * c + 1] << 16);
      }
      *reinterpret_cast<u32x4*>(p.krot + krot_block<HD>(spage, p.h_kv, g, pb, kb) + lane * 8) = permute_halves(plo);
      *reinterpret_cast<u32x4*>(p.krot + krot_block<HD>(spage, p.h_kv, g, pb, kb + 4) + lane * 8) = permute_halves(phi);
    }
  }
  // values: operand block (jb, kp) = columns 32 jb .. +31, positions 16 kp .. +15; wave w takes the blocks jb = w mod 4
  const uint32_t v_base = (uint32_t)kPage * n * 2u;
  for (int jb = w; jb < (n >> 5); jb += 4) {
    u32x4 raw[4];
#pragma unroll
    for (int kp = 0; kp < 4; ++kp)
      raw[kp] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(pr, lane * 16, v_base + (jb * 4 + kp) * 1024, 0));
#pragma unroll
    for (int kp = 0; kp < 4; ++kp) {
      uint16_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool live = pos0 + kp * 16 + 8 * hf + e < len;
        h[e] = live ? f16_bits(bf16_to_float((uint16_t)(raw[kp][e >> 1] >> (16 * (e & 1))))) : (uint16_t)0;
      }
      const u32x4 v = {(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                       (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
      *reinterpret_cast<u32x4*>(p.vt + vt_block<HD>(spage, p.h_kv, jb >> 2, jb & 3, kp) + lane * 8) = permute_halves(v);
    }
  }
}

// ------------------------------------------------------------------------------------------------ attend
// Four waves per workgroup, each with one 32-query block of one query head, two workgroups per CU (each hides the
// other's softmax behind its matrix-core work).  The waves are dealt as (query sub-block, head of the group): groups
// of 4 or more heads take 4 heads x 1 sub-block (32 queries per workgroup), 2 heads x 2 sub-blocks, 1 head x 4
// sub-blocks (128 queries), so that every wave has work whatever the grouping and a K/V tile copied to LDS serves 128
// query rows.  (Eight waves and 256 rows per tile, which halves the copies from L2, measured 7 % slower.)
constexpr int kAttnWaves = 4;
__host__ __device__ inline int attn_heads_per_pass(int G) { return G >= 4 ? 4 : (G >= 2 ? 2 : 1); }

template <int HD>
__global__ __launch_bounds__(64 * kAttnWaves, kAttnWaves == 4 ? 2 : 1) void prefill_attn_kernel(PrefillParams p) {
  constexpr int KS = HD / 16, ND = HD / 32, BK = 64, NW = kAttnWaves;
  constexpr int NKF = 2 * KS, NVF = 4 * ND;  // K and V operand fragments per tile
  constexpr int RING = 8;                    // fragments in flight from LDS
  static_assert(NKF % RING == 0 && NVF % RING == 0, "fragment ring");
  constexpr int KINS = 4 * KS / 2, VINS = 4 * ND;               // 1 KiB operand blocks per K and V tile
  constexpr int KELE = KINS * 512, VELE = VINS * 512;           // elements per stage
  extern __shared__ __align__(16) unsigned char smem_attn[];
  uint16_t* const sK = reinterpret_cast<uint16_t*>(smem_attn);          // [2][KELE]
  uint16_t* const sV = sK + 2 * KELE;                                   // [2][VELE]
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = p.h_kv * HD, G = p.G;
  const int NH = attn_heads_per_pass(G), BQW = 32 * (NW / NH);  // heads per pass; queries per workgroup
  const int wh = w % NH, wq = w / NH;                            // this wave's head of the pass and query sub-block
  const int g = blockIdx.x % p.h_kv;
  const int rest = blockIdx.x / p.h_kv;
  const int nqb = (p.lp + BQW - 1) / BQW;       // query blocks per sequence
  const int qb = nqb - 1 - rest % nqb;          // longest blocks first
  const int seq = rest / nqb;
  const int tok0 = p.cu_seqlens[seq];
  const int len = prompt_len(p, seq);
  if (qb * BQW >= len) return;
  const int q_last = qb * BQW + BQW - 1 < p.lp - 1 ? qb * BQW + BQW - 1 : p.lp - 1;
  const int t_wg = q_last / BK;                 // the last tile any wave of the workgroup needs
  const int qw0 = qb * BQW + wq * 32;           // this wave's first query
  const int t_w = qw0 / BK;                     // the tile that holds this wave's diagonal
  const int dq = qw0 - t_w * BK;                // offset of the wave's first query inside that tile
  // One K/V tile = one page's blocks of this KV head, global -> LDS as they lie (an operand read is 1 KiB of consecutive
  // LDS: no conflicts).  Wave w copies the blocks w, w + 4, ...
  constexpr int KI = KINS / NW, VI = VINS / NW;
  static_assert(KINS % NW == 0 && VINS % NW == 0 && KI + VI <= NKF, "one copy per score MFMA");
  const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(p.krot + (size_t)seq * p.lp * n, (uint32_t)((size_t)p.lp * n * 2));
  const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(p.vt + (size_t)seq * p.lp * n, (uint32_t)((size_t)p.lp * n * 2));
  auto tile_dma_one = [&](int t, int buf, int i) {  // copy i < KI + VI of this wave's share
    const uint32_t src = ((uint32_t)t * p.h_kv + g) * (BK * HD * 2u);
    if (i < KI) {
      const int blk = i * NW + w;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (__attribute__((address_space(3))) void*)(sK + (size_t)buf * KELE + (size_t)blk * 512), 16,
                                               lane * 16, (int)(src + blk * 1024u), 0, 0);
    } else {
      const int blk = (i - KI) * NW + w;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (__attribute__((address_space(3))) void*)(sV + (size_t)buf * VELE + (size_t)blk * 512), 16,
                                               lane * 16, (int)(src + blk * 1024u), 0, 0);
    }
  };
  auto tile_dma = [&](int t, int buf) {
#pragma unroll
    for (int i = 0; i < KI + VI; ++i) tile_dma_one(t, buf, i);
  };

  for (int hc = 0; hc < G; hc += NH) {
    const int hq = hc + wh;
    const bool active = hq < G && qw0 < len;
    const int h = g * G + hq;

    // Q operands (B operand: n = query, k = head-dim coordinate), rotated at the query's position and scaled.
    // The angle is reduced in fp64 turns and evaluated by the hardware sine and cosine (which take turns).
    f16x8 qf[KS];
    {
      const int qpos = qw0 + l32;
      const bool ok = active && qpos < len;
      const uint16_t* qrow = p.q + ((size_t)(tok0 + (ok ? qpos : 0)) * p.h_q + (active ? h : 0)) * HD;
      bf16x8 raw[KS];  // coordinates in the order of the key blocks
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x4 a = *reinterpret_cast<const bf16x4*>(qrow + ks * 16 + 4 * hf), b = *reinterpret_cast<const bf16x4*>(qrow + ks * 16 + 8 + 4 * hf);
        raw[ks] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      }
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double turns = (double)qpos * p.rope_tab[ks * 16 + acc_row(e, hf)] * 0.15915494309189533576888;
          const float fr = (float)(turns - rint(turns));
          const float c = __builtin_amdgcn_cosf(fr), sn = __builtin_amdgcn_sinf(fr);
          const float lo = (float)raw[ks][e], hi = (float)raw[ks + KS / 2][e];
          qf[ks][e] = static_cast<_Float16>(ok ? (lo * c - hi * sn) * p.q_scale : 0.f);
          qf[ks + KS / 2][e] = static_cast<_Float16>(ok ? (hi * c + lo * sn) * p.q_scale : 0.f);
        }
    }
    f32x16 o[ND];
#pragma unroll
    for (int a = 0; a < ND; ++a)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[a][j] = 0.f;
    // running maximum of the query's row (both halves of the wave agree on it) and this half's share of its sum
    float m_run = kNegInfP, l_half = 0.f;

    __syncthreads();  // previous head chunk is done with both stages
    tile_dma(0, 0);
    // One tile.  An in-order wave that asks LDS for an operand right before the MFMA that takes it pays the whole
    // LDS latency every time, so the operand reads run RING fragments ahead of the MFMAs: K fragment i + RING is
    // requested behind MFMA i, the first V fragments behind the last score MFMAs (they land under the softmax),
    // the rest behind the first value MFMAs.  The softmax itself touches no LDS (the row maximum crosses the
    // wave's halves on the vector ALU; the row sum is kept per half until the end).  The wave's share of the next
    // tile's copies is issued one copy per score MFMA rather than as a burst (a burst holds the wave, and its MFMAs,
    // in the issue of the loads); past the workgroup's last tile the copies repeat that tile into the idle stage.
    auto tile_step = [&](int t, auto diag_c) {  // the wave's diagonal tile is the only one that needs the mask
      const int buf = t & 1;
      const uint16_t* const kt = sK + buf * KELE + lane * 8;
      const uint16_t* const vtile = sV + buf * VELE + lane * 8;
      auto k_at = [&](int i) { return load_frag_f16(kt + ((i & 1) * KS + (i >> 1)) * 512); };         // i = 2 ks + mb
      auto v_at = [&](int j) { return load_frag_f16(vtile + ((j % ND) * 4 + j / ND) * 512); };      // j = ND k4 + db
      f16x8 fr[RING];
#pragma unroll
      for (int i = 0; i < RING; ++i) fr[i] = k_at(i);
      __builtin_amdgcn_sched_barrier(0);
      f32x16 s[2];
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const int tn = t + 1 <= t_wg ? t + 1 : t_wg;  // (clamped: the copies are unconditional)
#pragma unroll
      for (int i = 0; i < NKF; ++i) {
        s[i & 1] = mfma32_f16(fr[i % RING], qf[i >> 1], i < 2 ? zero : s[i & 1]);
        fr[i % RING] = i + RING < NKF ? k_at(i + RING) : v_at(i + RING - NKF);
        if (i < KI + VI) tile_dma_one(tn, buf ^ 1, i);
      }
#pragma unroll
      for (int i = 0; i < NKF; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
        if (i < KI + VI) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(diag_c)::value) {  // diagonal tile: key position must not exceed the query position
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int jj = 0; jj < 16; ++jj)
            if (mb * 32 + acc_row(jj, hf) > dq + l32) s[mb][jj] = kNegInfP;
      }
      float mx = kNegInfP;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) mx = fmaxf(mx, s[mb][jj]);
      {
        const float2 both = half_pair(mx);
        mx = fmaxf(both.x, both.y);
      }
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      f16x8 pf[4];
      float sum = 0.f;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
          const float pv = __builtin_amdgcn_exp2f(s[mb][jj] - m_new);
          sum += pv;
          pf[mb * 2 + (jj >> 3)][jj & 7] = static_cast<_Float16>(pv);
        }
      l_half = l_half * alpha + sum;
      const bool moved = m_new > m_run;
      m_run = m_new;
      if (__builtin_amdgcn_ballot_w64(moved) != 0) {  // some row's maximum moved
#pragma unroll
        for (int db = 0; db < ND; ++db)
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) o[db][jj] *= alpha;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NVF; ++j) {
        o[j % ND] = mfma32_f16(fr[j % RING], pf[j / ND], o[j % ND]);
        if (j + RING < NVF) fr[j % RING] = v_at(j + RING);
      }
#pragma unroll
      for (int j = 0; j < NVF - RING; ++j) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // Every wave passes every hand-over of the workgroup's tiles; it computes on the tiles up to its own diagonal
    // (waves of the earlier sub-blocks are done before the workgroup's last tiles).
    const int t_mine = active ? t_w : -1;
    auto hand_over = [&](int t) {
      __builtin_amdgcn_s_waitcnt(0);   // this wave's part of tile t has landed (LDS-bound loads count as vector memory)
      __syncthreads();                 // tile t visible; everyone is done with the other stage
      if (t > t_mine && t + 1 <= t_wg) tile_dma(t + 1, (t + 1) & 1);  // a wave with no work on tile t: as a burst
    };
    for (int t = 0; t < t_mine; ++t) {
      hand_over(t);
      tile_step(t, std::false_type{});
    }
    if (active) {
      hand_over(t_w);
      tile_step(t_w, std::true_type{});
    }
    for (int t = t_mine + 1; t <= t_wg; ++t) hand_over(t);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): no LDS-bound copy is left in flight when the wave ends

    if (active) {
      const int qpos = qw0 + l32;
      const float2 l_both = half_pair(l_half);
      const float l_run = l_both.x + l_both.y;
      if (qpos < len) {
        const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
        uint16_t* orow = p.out + ((size_t)(tok0 + qpos) * p.h_q + h) * HD;
#pragma unroll
        for (int db = 0; db < ND; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            uint16_t v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = bf16_bits(o[db][4 * q4 + i] * inv);
            const u32x2 pk = {(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16)};
            *reinterpret_cast<u32x2*>(orow + db * 32 + 8 * q4 + 4 * hf) = pk;
          }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------ host
static size_t align256p(size_t x) { return (x + 255) & ~(size_t)255; }

PrefillPlan make_prefill_plan(const lorc_layer_desc& d, int b, int max_seqlen) {
  PrefillPlan pl;
  pl.tiles_per_seq = (max_seqlen + kPage - 1) / kPage;
  if (pl.tiles_per_seq < 1) pl.tiles_per_seq = 1;
  pl.lp = pl.tiles_per_seq * kPage;
  const size_t n = (size_t)d.n_kv_heads * d.head_dim;
  size_t off = 0;
  pl.off_rope = off;
  off = align256p(off + 64 * sizeof(double));
  pl.off_krot = off;
  off = align256p(off + (size_t)b * pl.lp * n * 2);
  pl.off_vt = off;
  off = align256p(off + (size_t)b * pl.lp * n * 2);
  pl.total_bytes = off;
  return pl;
}

static size_t attn_lds_bytes(int hd) { return (size_t)2 * 2 * 64 * hd * 2; }  // two stages of a K and a V tile

static int attn_grid(const PrefillParams& p) {  // one workgroup per (sequence, block of queries, KV head)
  const int bqw = 32 * (kAttnWaves / attn_heads_per_pass(p.G));
  return p.b * ((p.lp + bqw - 1) / bqw) * p.h_kv;
}

template <int HD, int NC>
static int launch_rebuild(const PrefillParams& p, hipStream_t s) {
  const int ncg = (p.h_kv * HD / 32 + 2 * NC - 1) / (2 * NC), n_pt = p.b * ((p.tiles_per_seq + 1) / 2);
  const size_t lds = (size_t)rt_ring_bytes<NC, 3>() + (size_t)4 * (HD / 2) * 8;
  const int grid = rebuild_by_column(n_pt, ncg) ? (2 * ncg + 7) / 8 * 8 * n_pt : (n_pt + 7) / 8 * 8 * 2 * ncg;
  return launch_kernel(prefill_rebuild_kernel<HD, NC>, dim3(grid), dim3(256), lds, s, p);
}

int set_kernel_attributes_prefill() {
  const void* kernels[] = {reinterpret_cast<const void*>(prefill_attn_kernel<128>),
                           reinterpret_cast<const void*>(prefill_attn_kernel<64>),
                           reinterpret_cast<const void*>(prefill_rebuild_kernel<128, 4>),
                           reinterpret_cast<const void*>(prefill_rebuild_kernel<128, 2>),
                           reinterpret_cast<const void*>(prefill_rebuild_kernel<64, 4>),
                           reinterpret_cast<const void*>(prefill_rebuild_kernel<64, 2>)};
  for (const void* k : kernels)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return LORC_EHIP;
  return LORC_OK;
}

int launch_prefill(const PrefillParams& p, int n_cus, hipStream_t s, bool plain) {
  const bool d128 = p.head_dim == 128;
  int rc;
  if (plain) {  // uncompressed layer: keys and values are gathered from the pages, then the same attention kernel
    if (!d128) return LORC_EUNSUPPORTED;
    rc = launch_kernel(prefill_plain_gather_kernel, dim3(p.b * p.tiles_per_seq), dim3(256), 0, s, p);
  } else {
    const long wgs4 = (long)p.b * ((p.tiles_per_seq + 1) / 2) * 2 * ((p.h_kv * p.head_dim + 255) / 256);
    if (wgs4 >= 2L * n_cus) rc = d128 ? launch_rebuild<128, 4>(p, s) : launch_rebuild<64, 4>(p, s);
    else rc = d128 ? launch_rebuild<128, 2>(p, s) : launch_rebuild<64, 2>(p, s);
  }
  if (rc != LORC_OK) return rc;
  const dim3 grid_a(attn_grid(p));
  if (d128) return launch_kernel(prefill_attn_kernel<128>, grid_a, dim3(64 * kAttnWaves), attn_lds_bytes(128), s, p);
  return launch_kernel(prefill_attn_kernel<64>, grid_a, dim3(64 * kAttnWaves), attn_lds_bytes(64), s, p);
}

}  // namespace lorc
