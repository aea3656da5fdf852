// Decode attention in two or three launches, for the shapes the single-pass split kernels do not take:
//   * wide layers: ranks above 1024 (Table 2's LLaMA-2-13B row: MHA, 40 heads, n = 5120 compressed to 2048).  A tile's
//     K latents no longer fit LDS and the latent-space output of all heads no longer fits one workgroup's registers,
//     so the rank is walked through a ring and o_lat in column chunks;
//   * layers that Algorithm 1's threshold leaves uncompressed (Section 6.2): the cache pages hold the un-rotated
//     keys and the values themselves (rank = n, identity read-side factors that are never stored or multiplied).
//
//   scores : S[seq][h][t] = softmax_scale * log2(e) * <R(q_pos) q_h, R(t) k_t>   (Eq. 1; the Appendix on the adjusted
//            position embedding: keys are rotated when they are read).  Wide layers rebuild k_t = c_t B_k on the matrix
//            cores, the rank walked through an LDS ring; uncompressed layers read k_t.
//   values : per (sequence, context split, column chunk): row maxima of the split's scores, P = exp2(S - m), row
//            sums, o = P C_v for the chunk's columns on the matrix cores; written as split partials (m, l, o / l) in
//            the format of the single-pass kernels.  Wide layers: all heads x 512 latent columns per workgroup (the
//            latent is joint across heads, Section 4.1).  Uncompressed layers: one KV head's group x its 128 columns.
//   merge  : the common merge kernel (wide: softmax-merge of the splits, then B_v; uncompressed: the merge alone).
// Uncompressed layers of eight KV heads (or a multiple) take scores and values in one launch (decode_plain_kernel).
#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_rebuild.h"
#include "lorc_tile_product.h"

namespace lorc {

namespace {
constexpr float kNegInfW = -__builtin_huge_valf();
constexpr int kWideT = 64;           // positions per tile of the value kernel = one page
constexpr int kWideMaxG = 8;
constexpr int kScoreNC = 4;          // column blocks per wave of the scores kernel: the 128 columns of one KV head
constexpr int kScorePairs = 8;       // head pairs whose workgroups run side by side on an XCD
constexpr int kScoreFewTiles = 64;

constexpr int kScoreSlots = 3;       // ring of 3 x 24 KiB: two workgroups share a CU
constexpr int kScorePages = 2;       // pages per workgroup
// ring, rotation bases of the four position blocks, rotated and scaled queries of two KV heads (fp16)
constexpr int kScoreLdsBytes = rt_ring_bytes<kScoreNC, kScoreSlots>() + 4 * 64 * 8 + 2 * kWideMaxG * 128 * 2;
__host__ __device__ inline bool scores_by_pair(int n_pt, int n_pairs) { return n_pt < kScoreFewTiles && n_pairs >= 8; }
// Block ids of the scores launch (the kernel's mapping, below): eight XCDs' shares of equal length.
inline unsigned scores_grid(int n_pt, int n_pairs) {
  if (scores_by_pair(n_pt, n_pairs)) return 8u * n_pt * ((n_pairs + 7) / 8);
  return 8u * ((n_pt + 7) / 8) * n_pairs;
}
}  // namespace

// ------------------------------------------------------------------------------------------------ scores, compressed
// One workgroup per (pair of KV heads, two cached pages of a sequence): the rebuild K^T = B_k^T C_k^T of 256 columns x 128
// positions as a tiled matrix product (lorc_tile_product.h).  A wave's accumulators hold whole keys (one KV head, one page):
// they are rotated in registers and multiplied with the group's query rows (fp16 matrix-core op), and the scores are
// complete without an exchange between waves.  Bound by the matrix cores (2 r_k n flop per position): busy 73 % of the time at the
// 1.6 GHz that the power limit leaves.
//   13B layer, rank 2048, 16 x 4096 positions, whole call with append: 1684 -> 1245 us (1.1 to 1.2 PFLOP/s).  Before, a wave
//   streamed its factor operands from L2, two products per operand, and copied a page's latents twice.
//   Tried: 256 positions per workgroup (256 accumulators per lane, one workgroup per CU, two products per operand read):
//   no faster there (1238 against 1247 us), 592 against 539 at rank 768 (8B layer, 32 x 8192) and 62 against 55 at one short sequence: with one
//   workgroup per CU nothing runs under another's prologue and rotation.
__global__ __launch_bounds__(256, 2) void wide_scores_kernel(DecodeParams p) {
  constexpr int HD = 128, HALF = 64, NC = kScoreNC, NS = kScoreSlots, PB = 2;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Block id -> (position tile, head pair); an XCD takes the block ids of one residue mod 8: every eighth position tile,
  // kScorePairs head pairs at a time over all of them, so that the workgroups in flight share factor slices and latents in
  // the XCD's L2; with few position tiles every eighth head pair and all tiles.
  const int pages = p.score_stride / kPage, tps = (pages + kScorePages - 1) / kScorePages, n_pt = p.b * tps, n_pairs = (p.h_kv + 1) >> 1;
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  int pt, pair;
  if (scores_by_pair(n_pt, n_pairs)) {
    pt = idx % n_pt;
    pair = idx / n_pt * 8 + xcd;
    if (pair >= n_pairs) return;
  } else {
    const int t8 = (n_pt + 7) >> 3, chunk = idx / (t8 * kScorePairs), rest = idx - chunk * t8 * kScorePairs;
    const int left = n_pairs - chunk * kScorePairs, width = left < kScorePairs ? left : kScorePairs;
    pt = (rest / width) * 8 + xcd;
    pair = chunk * kScorePairs + rest % width;
  }
  if (pt >= n_pt) return;
  const int seq = pt / tps, page0 = (pt - seq * tps) * kScorePages, pos0 = page0 * kPage;
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  if (pos0 >= ctx) return;  // whole workgroup: nothing of this tile is attended to
  const int G = p.G, r_k = p.r_k, ncb = p.h_kv * (HD / 32);

  // the wave's page; one that is not cached, or past the context, reads as zeros (nothing is fetched)
  const int cpage = page0 + (w >> 1);
  const int id = cpage * kPage < ctx ? p.block_table[(size_t)seq * p.max_pages + cpage] : -1;
  const bool page_ok = id >= 0 && id < p.n_pages;
  const u32x4 page = dma_rsrc(p.cache + (size_t)(page_ok ? id : 0) * p.page_elems, page_ok ? (uint32_t)kPage * r_k * 2u : 0u);

  float2* const cs_base = reinterpret_cast<float2*>(smem + rt_ring_bytes<NC, NS>());  // [4 position blocks][HALF]
  _Float16* const qrot = reinterpret_cast<_Float16*>(cs_base + 4 * HALF);               // [2 heads x G][HD]
  // rotation bases of the position blocks, and the two groups' query rows rotated at q_pos and scaled
  auto setup = [&]() {
    cs_base[tid] = cos_sin_reduced((double)(pos0 + 32 * (tid / HALF)) * p.rope_tab[tid % HALF]);  // 4 x HALF = 256
    const int q_pos = p.q_pos[seq];
    for (int i = tid; i < 2 * G * HALF; i += 256) {
      const int hl = i / HALF, f = i % HALF, h = pair * 2 * G + hl;
      if (h < p.h_q) {
        const float2 cs = cos_sin_reduced((double)q_pos * p.rope_tab[f]);
        const uint16_t* qs = p.q + ((size_t)seq * p.h_q + h) * HD;
        const float lo = bf16_to_float(qs[f]) * p.q_scale, hi = bf16_to_float(qs[f + HALF]) * p.q_scale;
        qrot[hl * HD + f] = static_cast<_Float16>(lo * cs.x - hi * cs.y);
        qrot[hl * HD + f + HALF] = static_cast<_Float16>(hi * cs.x + lo * cs.y);
      }
    }
  };
  f32x16 acc[NC][PB];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int pb = 0; pb < PB; ++pb)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[c][pb][j] = 0.f;
  tile_product<HD, NC, NS, kPageKeys, false>(acc, smem, dma_rsrc(p.bk, (uint32_t)p.h_kv * HD * r_k * 2u), page, pair * 2 * NC, ncb,
                                                    r_k >> 4, w, lane, r_k >> 5, 0, setup);
  const int gl = w & 1, g = pair * 2 + gl;
  if (g >= p.h_kv) return;
  const bool qreal = l32 < G;
  const _Float16* qh = qrot + (size_t)(gl * G + (qreal ? l32 : 0)) * HD + 4 * hf;
  f32x16 S[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int j = 0; j < 16; ++j) S[pb][j] = 0.f;
#pragma unroll
  for (int wh = 0; wh < 2; ++wh) {  // halves of the head's rotation pairs: columns [32 wh, 32 wh + 32) and their partners
    // Query operands (m = query head of the group, k = 16 head-dim coordinates) in the order in which the rotated K^T
    // accumulators serve as B operands: element e of operand s4 is coordinate 16 (s4 & 1) + 8 (e >> 2) + 4 hf + (e & 3) of
    // half s4 >> 1 of the head, + 32 wh.
    f16x8 qf[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const _Float16* src = qh + 32 * wh + HALF * (s4 >> 1) + 16 * (s4 & 1);
      const u32x2 lo = *reinterpret_cast<const u32x2*>(src), hi = *reinterpret_cast<const u32x2*>(src + 8);
      const u32x4 v = {qreal ? lo[0] : 0u, qreal ? lo[1] : 0u, qreal ? hi[0] : 0u, qreal ? hi[1] : 0u};
      qf[s4] = __builtin_bit_cast(f16x8, v);
    }
    float2 cl[16];  // rotation by the lane's offset inside a position block, the same for all blocks (at most 5 turns)
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) cl[jj] = p.lane_cs[l32 * HALF + 32 * wh + acc_row(jj, hf)];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      f16x8 kf[4];
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        const float2 cb = cs_base[((w >> 1) * PB + pb) * HALF + 32 * wh + acc_row(jj, hf)];
        const float cA = cb.x * cl[jj].x - cb.y * cl[jj].y;
        const float sA = cb.y * cl[jj].x + cb.x * cl[jj].y;
        const float x = acc[wh][pb][jj], y = acc[wh + 2][pb][jj];
        kf[jj >> 3][jj & 7] = static_cast<_Float16>(x * cA - y * sA);
        kf[2 + (jj >> 3)][jj & 7] = static_cast<_Float16>(y * cA + x * sA);
      }
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) S[pb] = mfma32_f16(qf[s4], kf[s4], S[pb]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int jr = 0; jr < 4; ++jr) {  // rows 0 .. 7 of the score block hold the group's (at most eight) heads
    const int m = acc_row(jr, hf);
    if (m < G) {
      float* row = p.scores + ((size_t)seq * p.h_q + g * G + m) * p.score_stride;
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        const int pos = pos0 + kPage * (w >> 1) + 32 * pb;
        if (pos < p.score_stride) row[pos + l32] = S[pb][jr];
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------ scores, uncompressed
// One workgroup per (sequence, 64-position tile).  Wave w takes position block w % 2 and the KV heads of parity
// w / 2.  A lane of a K operand block holds one position and 8 consecutive head-dim coordinates, and the rotation
// partner of a block sits four blocks further in the same lane and element: the keys are rotated in registers
// (angles per position and frequency worked out once per tile and shared by all heads; reduced in fp64, evaluated
// by the hardware sine / cosine, which take turns), rounded to fp16 and multiplied with the group's query rows.
__global__ __launch_bounds__(256, 2) void plain_scores_kernel(DecodeParams p) {
  constexpr int HD = 128, HALF = 64, T = kWideT;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = p.score_stride / T;
  const int seq = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int pos0 = tile * T;
  if (pos0 >= ctx) return;
  const int G = p.G, n = p.h_kv * HD;
  _Float16* qrot = reinterpret_cast<_Float16*>(smem);  // [h_q][HD]

  const int id = p.block_table[(size_t)seq * p.max_pages + tile];
  const bool page_ok = id >= 0 && id < p.n_pages;
  const uint16_t* page = uniform_ptr(p.cache + (size_t)(page_ok ? id : 0) * p.page_elems);
  // a page that is not cached reads as zeros through a descriptor of size zero
  const __amdgpu_buffer_rsrc_t kr = make_rsrc(page, page_ok ? (uint32_t)kPage * n * 2u : 0u);
  const int q_pos = p.q_pos[seq];

  for (int idx = tid; idx < p.h_q * HALF; idx += 256) {
    const int h = idx / HALF, i = idx % HALF;
    const float2 cs = cos_sin_reduced((double)q_pos * p.rope_tab[i]);
    const uint16_t* qs = p.q + ((size_t)seq * p.h_q + h) * HD;
    const float lo = bf16_to_float(qs[i]) * p.q_scale, hi = bf16_to_float(qs[i + HALF]) * p.q_scale;
    qrot[h * HD + i] = static_cast<_Float16>(lo * cs.x - hi * cs.y);
    qrot[h * HD + i + HALF] = static_cast<_Float16>(hi * cs.x + lo * cs.y);
  }
  const int pb = w & 1;
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
  __syncthreads();

  const int blocks_per_row = n >> 4;  // 1 KiB operand blocks per 32 positions
  for (int g = w >> 1; g < p.h_kv; g += 2) {
    u32x4 raw[8];
#pragma unroll
    for (int kb = 0; kb < 8; ++kb)
      raw[kb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(kr, lane * 16, (pb * blocks_per_row + g * 8 + kb) * 1024, 0));
    f16x8 kf[8];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = bf16_to_float((uint16_t)(raw[kb][e >> 1] >> (16 * (e & 1))));
        const float y = bf16_to_float((uint16_t)(raw[kb + 4][e >> 1] >> (16 * (e & 1))));
        kf[kb][e] = static_cast<_Float16>(x * cs_c[kb][e] - y * cs_s[kb][e]);
        kf[kb + 4][e] = static_cast<_Float16>(y * cs_c[kb][e] + x * cs_s[kb][e]);
      }
    f32x16 S;
#pragma unroll
    for (int j = 0; j < 16; ++j) S[j] = 0.f;
    const bool qreal = l32 < G;
    const _Float16* qh = qrot + (size_t)(g * G + (qreal ? l32 : 0)) * HD + 8 * hf;
#pragma unroll
    for (int kb = 0; kb < 8; ++kb) {
      const u32x4 qv = *reinterpret_cast<const u32x4*>(qh + 16 * kb);
      const u32x4 v = {qreal ? qv[0] : 0u, qreal ? qv[1] : 0u, qreal ? qv[2] : 0u, qreal ? qv[3] : 0u};
      S = mfma32_f16(__builtin_bit_cast(f16x8, v), kf[kb], S);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int m = acc_row(j, hf);
      if (m < G) p.scores[((size_t)seq * p.h_q + g * G + m) * p.score_stride + pos0 + 32 * pb + l32] = S[j];
    }
  }
}

// ------------------------------------------------------------------------------------------------ uncompressed, one pass
// Decode of an uncompressed layer with eight KV heads (or a multiple; the groups then have at most eight query heads, which fill
// half of a 16-wide operand) in one pass over the pages: one workgroup per (eight KV heads, split, sequence), wave w owns the KV
// heads w and w + 4 of the eight and walks the split's positions 32 at a time with online softmax; the waves exchange nothing.  Bound by the page stream.  A wave keeps
// one step of keys and one of values (16 KiB each) in flight: the next keys are requested when the scores have used the
// current ones, the next values when the weighted sum has.  16x16x32 products throughout:
//   S^T = K Q^T: row r = 4 q + j of block b (lane group q = lane / 16) is position 8 q + 4 b + j of the step, so that a lane's
//   eight weights are those of eight consecutive positions, which is what it holds of V^T as an operand of O^T = V^T P^T.
// Keys are rotated in registers: the lane's offset inside a step (constant) times the step's base angle (64 frequencies, one
// per lane, handed round through LDS); base and query angles are reduced in fp64 and evaluated by the hardware sine and cosine
// (sincosf for both changes the outputs' error by less than 0.4 %).  Error of the outputs against fp64 over 1 to 64 sequences of 100
// to 20000 positions: 1.78e-3 to 2.36e-3 in the 2-norm, 1.90e-3 to 2.38e-3 for scores, values and merge.
//   8B layer (n = 1024), 16 x 4096 positions, call with append: 82 us as scores, values and merge -> 68 (268 MB of pages);
//   64 x 8192, ragged: 344 -> 278; 1 x 2000: 31 -> 24; 4 x 1000: 32 -> 25.
constexpr int kPlainHeads = 8, kPlainStep = 32;
__global__ __launch_bounds__(256, 1) void decode_plain_kernel(DecodeParams p) {
  constexpr int HD = 128, HALF = 64;
  __shared__ __align__(16) float2 base_cs[4][HALF];  // per wave: rotation of the step's first position
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_hg = p.h_kv / kPlainHeads, hg = blockIdx.x % n_hg, ss = blockIdx.x / n_hg;
  const int split = ss % p.n_splits, seq = ss / p.n_splits;
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int G = p.G, n = p.h_kv * HD, blocks_per_row = n >> 4;
  const int t_begin = split * p.tiles_per_split * kPage;
  int t_end = t_begin + p.tiles_per_split * kPage;
  if (t_end > ctx) t_end = ctx;
  const int n_steps = t_end > t_begin ? (t_end - t_begin + kPlainStep - 1) / kPlainStep : 0;
  const int g0 = hg * kPlainHeads + w;  // the wave's KV heads: g0, g0 + 4

  // lane offsets of the operands inside a page (bytes)
  const int po[2] = {8 * (m >> 2) + (m & 3), 8 * (m >> 2) + 4 + (m & 3)};  // position of key row m, block b
  uint32_t koff[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) koff[b] = (uint32_t)(q >> 1) * 1024u + (uint32_t)(po[b] + 32 * (q & 1)) * 16u;
  const uint32_t voff = (uint32_t)(q >> 1) * 1024u + (uint32_t)(m + 32 * (q & 1)) * 16u;
  const uint32_t part_bytes = (uint32_t)kPage * n * 2u;
  u32x4 kraw[2][2][4], vraw[2][8];
  // Requests of step i; past the last one nothing is fetched (descriptor of size zero, as for a page that is not cached).
  auto page_of = [&](int i, bool& ok) {
    const int tile = i < n_steps ? (t_begin + i * kPlainStep) / kPage : 0;
    const int id = __builtin_amdgcn_readfirstlane(i < n_steps ? p.block_table[(size_t)seq * p.max_pages + tile] : -1);
    ok = id >= 0 && id < p.n_pages;
    return uniform_ptr(p.cache + (size_t)(ok ? id : 0) * p.page_elems);
  };
  auto k_request = [&](int i) {
    bool ok;
    const uint16_t* page = page_of(i, ok);
    const __amdgpu_buffer_rsrc_t r = make_rsrc(page, ok ? part_bytes : 0u);
    const int row = (i & 1) * blocks_per_row;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          kraw[h][b][kk] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, koff[b], (row + (g0 + 4 * h) * 8 + 2 * kk) * 1024, 0));
  };
  auto v_request = [&](int i) {
    bool ok;
    const uint16_t* page = page_of(i, ok);
    const __amdgpu_buffer_rsrc_t r = make_rsrc(page + (size_t)kPage * n, ok ? part_bytes : 0u);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int mb = 0; mb < 8; ++mb)
        vraw[h][mb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                    r, voff, (((g0 + 4 * h) * 4 + (mb >> 1)) * 4 + 2 * (i & 1)) * 1024 + (mb & 1) * 256, 0));
  };
  k_request(0);
  v_request(0);

  // query operands (n = query head of the group, k = 32 coordinates), rotated at q_pos and scaled; rows past the group: zeros
  f16x8 qf[2][4];
  {
    const double q_pos = (double)p.q_pos[seq];
    float qc[2][8], qs[2][8];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double turns = q_pos * p.rope_tab[32 * kk + 8 * q + e] * 0.15915494309189533576888;
        const float fr = (float)(turns - rint(turns));
        qc[kk][e] = __builtin_amdgcn_cosf(fr);
        qs[kk][e] = __builtin_amdgcn_sinf(fr);
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float scale = m < G ? p.q_scale : 0.f;
      const uint16_t* row = p.q + ((size_t)seq * p.h_q + (size_t)(g0 + 4 * h) * G + (m < G ? m : 0)) * HD + 8 * q;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 lo = load_frag(row + 32 * kk), hi = load_frag(row + 32 * kk + HALF);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = m < G ? (float)lo[e] * scale : 0.f, y = m < G ? (float)hi[e] * scale : 0.f;
          qf[h][kk][e] = static_cast<_Float16>(x * qc[kk][e] - y * qs[kk][e]);
          qf[h][kk + 2][e] = static_cast<_Float16>(y * qc[kk][e] + x * qs[kk][e]);
        }
      }
    }
  }
  float2 cl[2][2][8];  // rotation of the lane's offset inside a step
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) cl[b][kk][e] = p.lane_cs[po[b] * HALF + 32 * kk + 8 * q + e];
  const double theta = p.rope_tab[lane] * 0.15915494309189533576888;  // turns per position

  // finite from the start: while every score so far is -inf, the weights and the rescaling are exp2(-inf) and exp2(0)
  float m_run[2] = {kNoWeight, kNoWeight}, l_run[2] = {0.f, 0.f};
  f32x4 o[2][8];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[h][mb][j] = 0.f;

  for (int i = 0; i < n_steps; ++i) {
    const int pos0 = t_begin + i * kPlainStep;
    {
      const double turns = (double)pos0 * theta;
      const float fr = (float)(turns - rint(turns));
      base_cs[w][lane] = make_float2(__builtin_amdgcn_cosf(fr), __builtin_amdgcn_sinf(fr));
      __builtin_amdgcn_wave_barrier();  // a wave's LDS operations run in order
    }
    // ---- scores
    f32x4 S[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) S[h][b][j] = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        float c[8], s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float2 bs = base_cs[w][32 * kk + 8 * q + e], l = cl[b][kk][e];
          c[e] = bs.x * l.x - bs.y * l.y;
          s[e] = bs.y * l.x + bs.x * l.y;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f16x8 lo, hi;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = bf16_to_float((uint16_t)(kraw[h][b][kk][e >> 1] >> (16 * (e & 1))));
            const float y = bf16_to_float((uint16_t)(kraw[h][b][kk + 2][e >> 1] >> (16 * (e & 1))));
            lo[e] = static_cast<_Float16>(x * c[e] - y * s[e]);
            hi[e] = static_cast<_Float16>(y * c[e] + x * s[e]);
          }
          S[h][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, qf[h][kk], S[h][b], 0, 0, 0);
          S[h][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, qf[h][kk + 2], S[h][b], 0, 0, 0);
        }
      }
    __builtin_amdgcn_wave_barrier();
    k_request(i + 1);
    // ---- online softmax: a lane holds eight positions of query head m; the four lane groups meet in the maximum
    bf16x8 pf[2];
    float alpha[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float sv[8], mx = kNegInfW;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sv[e] = pos0 + 8 * q + e < t_end ? S[h][e >> 2][e & 3] : kNegInfW;
        mx = fmaxf(mx, sv[e]);
      }
      const float2 a = row_pair(mx);
      mx = fmaxf(a.x, a.y);
      const float2 c = half_pair(mx);
      mx = fmaxf(c.x, c.y);
      const float m_new = fmaxf(m_run[h], mx);
      alpha[h] = exp2f(m_run[h] - m_new);
      m_run[h] = m_new;
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pe = pos0 + 8 * q + e < t_end ? exp2f(sv[e] - m_new) : 0.f;
        pf[h][e] = static_cast<__bf16>(pe);
        sum += (float)pf[h][e];  // the weights as they are multiplied: they add up to one whatever their rounding
      }
      l_run[h] = l_run[h] * alpha[h] + sum;
    }
    // ---- o += V^T P^T
    if (pos0 + kPlainStep > t_end) {
      // slots past the context hold whatever the pool held before (possibly NaN patterns) and 0 * NaN is not zero
      int nv = t_end - pos0 - 8 * q;
      nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            vraw[h][mb][c] &= (2 * c < nv ? 0x0000ffffu : 0u) | (2 * c + 1 < nv ? 0xffff0000u : 0u);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[h][mb][j] *= alpha[h];
        o[h][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vraw[h][mb]), pf[h], o[h][mb], 0, 0, 0);
      }
    v_request(i + 1);
  }

  // ---- partials: O^T has columns along the accumulator rows (16 mb + 4 q + j) and query head m
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float2 a = row_pair(l_run[h]);
    const float2 c = half_pair(a.x + a.y);
    const float l = c.x + c.y, inv = l > 0.f ? 1.f / l : 0.f;
    if (m < G) {
      const size_t row = ((size_t)seq * p.n_splits + split) * p.h_q + (size_t)(g0 + 4 * h) * G + m;
      if (q == 0) {
        p.part_ml[row * 2] = n_steps > 0 ? m_run[h] : kNegInfW;
        p.part_ml[row * 2 + 1] = l;
      }
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) {
        const f32x4 v = o[h][mb];
        const u32x2 pk = {(uint32_t)f16_bits(v[0] * inv) | ((uint32_t)f16_bits(v[1] * inv) << 16),
                          (uint32_t)f16_bits(v[2] * inv) | ((uint32_t)f16_bits(v[3] * inv) << 16)};
        *reinterpret_cast<u32x2*>(p.part_o + row * HD + 16 * mb + 4 * q) = pk;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------ scores, absorbed query
// Models without positional rotation (Section 4.1, Eq. 7): S[h][t] = scale * <q_lat[h], c_k[t]> on the cached K
// latents themselves.  One workgroup per (sequence, 64-position tile).  Wave w takes position block w % 2 and the
// k-steps of parity w / 2, for all QB blocks of 32 heads: a K operand block (k = 16 latent indices, n = 32 positions:
// the page tiling) is read once, by one wave; the query operands (m = head, k = 16 latent indices: 16 contiguous
// bytes of a q_lat row per lane) come from L2.  The two parities meet in LDS.
template <int QB>
__global__ __launch_bounds__(256, 2) void absorbed_scores_kernel(DecodeParams p) {
  constexpr int T = kWideT, U = 4;
  __shared__ float xs[2][QB][16][64];  // [position block][row block][accumulator register][lane]
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = p.score_stride / T;
  const int seq = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int pos0 = tile * T;
  if (pos0 >= ctx) return;
  const int r_k = p.r_k, nks = r_k >> 4, pb = w & 1, par = w >> 1;
  const int id = p.block_table[(size_t)seq * p.max_pages + tile];
  const bool page_ok = id >= 0 && id < p.n_pages;
  const uint16_t* page = uniform_ptr(p.cache + (size_t)(page_ok ? id : 0) * p.page_elems);
  const __amdgpu_buffer_rsrc_t kr = make_rsrc(page, page_ok ? (uint32_t)kPage * r_k * 2u : 0u);  // not cached: zeros
  // rows past the last head read row 0 and are not written
  const __amdgpu_buffer_rsrc_t qr = make_rsrc(p.q + (size_t)seq * p.h_q * r_k, (uint32_t)p.h_q * r_k * 2u);
  uint32_t qoff[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int h = qb * 32 + l32;
    qoff[qb] = (uint32_t)((h < p.h_q ? h : 0) * r_k + 8 * hf) * 2u;
  }
  f32x16 S[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int j = 0; j < 16; ++j) S[qb][j] = 0.f;
  const int my_steps = (nks - par + 1) >> 1;  // k-steps par, par + 2, ...
  for (int i0 = 0; i0 < my_steps; i0 += U) {
    bf16x8 kf[U], qf[U][QB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u < my_steps ? i0 + u : my_steps - 1;  // clamped: the repeats are not multiplied
      const int ks = par + 2 * i;
      kf[u] = buf_frag(kr, (uint32_t)lane * 16u, (uint32_t)(pb * nks + ks) * 1024u);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) qf[u][qb] = buf_frag(qr, qoff[qb], (uint32_t)ks * 32u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u < my_steps)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) S[qb] = mfma32(qf[u][qb], kf[u], S[qb]);
  }
  if (par == 1) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int j = 0; j < 16; ++j) xs[pb][qb][j][lane] = S[qb][j];
  }
  __syncthreads();
  if (par == 0) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int h = qb * 32 + acc_row(j, hf);
        if (h < p.h_q)
          p.scores[((size_t)seq * p.h_q + h) * p.score_stride + pos0 + 32 * pb + l32] = (S[qb][j] + xs[pb][qb][j][lane]) * p.q_scale;
      }
  }
}

// ------------------------------------------------------------------------------------------------ values
// QB: blocks of 32 score rows; NB: blocks of 32 output columns per wave.
//   wide  (PLAIN = false): rows = all query heads, columns = latent indices [512 chunk, 512 chunk + 512) of C_v;
//   plain (PLAIN = true) : rows = the G heads of KV head `chunk`, columns = that head's 128 value coordinates.
// Grid: (sequence, split, chunk).  The split's row maxima are taken first (the scores are there already), so the
// weights need no rescaling afterwards; P goes to LDS in A-operand order (bf16), the value operands come straight
// from the page tiling (a wave-wide 1 KiB block is one B operand: k = 16 positions, n = 32 columns).
template <int QB, int NB, bool PLAIN>
__global__ __launch_bounds__(256, QB == 1 ? 2 : 1) void latent_pv_kernel(DecodeParams p) {
  constexpr int T = kWideT, KP = T / 16;
  __shared__ __align__(16) uint16_t pbuf[2][QB * KP * 512];
  __shared__ float m_s[QB * 32], l_s[QB * 32];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nc = PLAIN ? p.h_kv : p.v_chunks;
  const int chunk = blockIdx.x % nc, ss = blockIdx.x / nc;
  const int split = ss % p.n_splits, seq = ss / p.n_splits;
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int R = PLAIN ? p.G : p.h_q;                        // real rows
  const int head0 = PLAIN ? chunk * p.G : 0;                // head of row 0
  const int r_k = p.r_k, r_v = p.r_v;
  const int t_begin = split * p.tiles_per_split * T;
  int t_end = t_begin + p.tiles_per_split * T;
  if (t_end > ctx) t_end = ctx;
  const int out_w = PLAIN ? 128 : r_v;                      // width of a partial row
  const int nblk = r_v >> 5;                                // 32-column blocks of the value part
  const size_t part_row0 = ((size_t)seq * p.n_splits + split) * p.h_q + head0;

  // this thread's share of a tile's scores: row tid / 4, sixteen positions
  const int prow = tid >> 2, pseg = tid & 3;
  const bool prow_real = prow < QB * 32 && prow < R;
  const float* srow = p.scores + ((size_t)seq * p.h_q + head0 + (prow_real ? prow : 0)) * p.score_stride;
  const int tile_begin = t_begin / T, tile_end = (t_end + T - 1) / T;  // empty split: tile_end <= tile_begin

  // ---- 1. row maxima over the split (same thread layout as the weights below; the loads of several tiles are
  //         independent and in flight together)
  {
    float mx = kNegInfW;
    if (prow_real) {
#pragma unroll 4
      for (int tile = tile_begin; tile < tile_end; ++tile) {
        const int tb = tile * T + pseg * 16;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x4 s4 = *reinterpret_cast<const f32x4*>(srow + tb + q4 * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) mx = fmaxf(mx, tb + q4 * 4 + e < t_end ? s4[e] : kNegInfW);
        }
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 1));
    mx = fmaxf(mx, __shfl_xor(mx, 2));
    if (tid < QB * 32 * 4 && pseg == 0) m_s[prow] = mx;
  }
  __syncthreads();

  f32x16 o[QB][NB];
#pragma unroll
  for (int a = 0; a < QB; ++a)
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[a][i][j] = 0.f;

  const float pm = prow < QB * 32 ? m_s[prow] : 0.f;
  float lsum = 0.f;

  // column blocks of this wave (clamped: blocks past the rank are computed on repeated data and never written)
  int jb[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b_ = PLAIN ? chunk * 4 + w : chunk * 16 + w * NB + i;
    jb[i] = b_ < nblk ? b_ : nblk - 1;
  }
  // Page ids are fetched two tiles ahead and a tile's value operands one tile ahead, and inside a tile the scores
  // are requested before the next tile's operands: the in-order load counter then lets the weights wait for the
  // scores alone while the operands (the HBM stream) stay in flight across the tile's work.
  auto page_id = [&](int tile) {
    const int tc = tile < tile_end ? tile : tile_end - 1;
    return p.block_table[(size_t)seq * p.max_pages + (tc > 0 ? tc : 0)];
  };
  auto v_load = [&](bf16x8 (&v)[NB][KP], int id_raw) {
    const int id = __builtin_amdgcn_readfirstlane(id_raw);
    const bool ok = id >= 0 && id < p.n_pages;
    const uint16_t* vpart = uniform_ptr(p.cache + (size_t)(ok ? id : 0) * p.page_elems + (size_t)kPage * r_k);
    const __amdgpu_buffer_rsrc_t vr = make_rsrc(vpart, ok ? (uint32_t)kPage * r_v * 2u : 0u);  // not cached: zeros, nothing fetched
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int kp = 0; kp < KP; ++kp) v[i][kp] = buf_frag(vr, (uint32_t)lane * 16u, (uint32_t)(jb[i] * KP + kp) * 1024u);
  };

  bf16x8 v[NB][KP], v_next[NB][KP];
  int id_next = 0;
  if (tile_begin < tile_end) {
    const int id0 = page_id(tile_begin);
    id_next = page_id(tile_begin + 1);
    v_load(v_next, id0);
  }
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    const int pos0 = tile * T, buf = (tile - tile_begin) & 1;
    f32x4 s4[4];  // threads without a row read row 0 (unconditional: a fixed number of loads in flight)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) s4[q4] = *reinterpret_cast<const f32x4*>(srow + pos0 + pseg * 16 + q4 * 4);
    const int id_after = page_id(tile + 2);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int kp = 0; kp < KP; ++kp) v[i][kp] = v_next[i][kp];
    v_load(v_next, id_next);  // tile + 1 (past the end: the last page again, never multiplied)
    id_next = id_after;
    if (pos0 + T > t_end) {
      // Ragged last tile: slots past the context hold whatever the pool held before (possibly NaN patterns); P is
      // zero there, but 0 * NaN is not, so those elements of the value operands are cleared.  Element e of operand
      // kp is position 16 kp + 8 hf + e.
#pragma unroll
      for (int kp = 0; kp < KP; ++kp) {
        int nv = t_end - pos0 - kp * 16 - 8 * hf;
        nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
        const uint32_t vmask = (1u << nv) - 1u;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          u32x4 raw = __builtin_bit_cast(u32x4, v[i][kp]);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const uint32_t two = (vmask >> (2 * c)) & 3u;
            raw[c] &= (two & 1u ? 0x0000ffffu : 0u) | (two & 2u ? 0xffff0000u : 0u);
          }
          v[i][kp] = __builtin_bit_cast(bf16x8, raw);
        }
      }
    }
    // ---- 2. weights of the tile
    if (tid < QB * 32 * 4) {
      float pv[16];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int t = pos0 + pseg * 16 + q4 * 4 + e;
          const float pe = (prow_real && t < t_end) ? exp2f(s4[q4][e] - pm) : 0.f;
          pv[q4 * 4 + e] = pe;
          lsum += pe;
        }
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        u32x4 pk;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          pk[c] = (uint32_t)bf16_bits(pv[half * 8 + 2 * c]) | ((uint32_t)bf16_bits(pv[half * 8 + 2 * c + 1]) << 16);
        const int qb = prow >> 5, m = prow & 31;
        *reinterpret_cast<u32x4*>(&pbuf[buf][(size_t)((qb * KP + pseg) * 64 + m + 32 * half) * 8]) = pk;
      }
    }
    __syncthreads();  // P of this tile is complete; the buffer of the tile before the previous one is free again
    // ---- 3. o += P V
#pragma unroll
    for (int kp = 0; kp < KP; ++kp) {
      bf16x8 a[QB];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) a[qb] = load_frag(&pbuf[buf][(size_t)((qb * KP + kp) * 64 + lane) * 8]);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int i = 0; i < NB; ++i) o[qb][i] = mfma32(a[qb], v[i][kp], o[qb][i]);
    }
  }

  // ---- 4. row sums, partials
  lsum += __shfl_xor(lsum, 1);
  lsum += __shfl_xor(lsum, 2);
  if (tid < QB * 32 * 4 && pseg == 0) l_s[prow] = lsum;
  __syncthreads();
  if ((PLAIN || chunk == 0) && tid < QB * 32 && tid < R) {
    float* ml = p.part_ml + (part_row0 + tid) * 2;
    ml[0] = m_s[tid];
    ml[1] = l_s[tid];
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int b_ = PLAIN ? chunk * 4 + w : chunk * 16 + w * NB + i;
      if (b_ >= nblk) continue;
      const int col = (PLAIN ? w * 32 : b_ * 32) + l32;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int r = qb * 32 + acc_row(j, hf);
        if (r < R) {
          const float l = l_s[r];
          p.part_o[(part_row0 + r) * out_w + col] = f16_bits(l > 0.f ? o[qb][i][j] / l : 0.f);
        }
      }
    }
}

// ------------------------------------------------------------------------------------------------ host
static size_t align256w(size_t x) { return (x + 255) & ~(size_t)255; }

bool wide_shape_ok(const lorc_layer_desc& d) {
  const int G = d.n_q_heads / d.n_kv_heads;
  return d.head_dim == 128 && G <= kWideMaxG && d.n_q_heads <= 64 && d.rank_k <= kWideMaxRank && d.rank_v <= kWideMaxRank;
}

bool plain_shape_ok(const lorc_layer_desc& d) {
  const int n = d.n_kv_heads * d.head_dim, G = d.n_q_heads / d.n_kv_heads;
  return d.head_dim == 128 && d.rank_k == n && d.rank_v == n && G <= 32 && d.n_q_heads <= 64;
}

// Uncompressed layers in one pass: all eight KV heads of a workgroup are real.  (Its sixteen operand columns hold any group
// then: 64 query heads at most.)  Other counts stay with scores and values: 16 x 4096 positions with append, 4 KV heads 48.5 us,
// 10 KV heads 100 us (eight in one pass: 68 us for 268 MB of pages, against 134 and 336 MB).
static bool plain_one_pass(int h_kv) { return h_kv % kPlainHeads == 0; }

// Splits for the value kernel: enough workgroups for about two per CU, each walking at least four tiles (uncompressed layers) or, while
// every split has a compute unit, one (the others); for the one-pass kernel of uncompressed layers see below.
DecodePlan make_wide_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, bool plain, int max_splits) {
  DecodePlan pl{};
  pl.tile = kWideT;
  pl.occupancy = 1;
  pl.stationary = 0;
  pl.wide = plain ? 2 : 1;
  const bool one_pass = plain && plain_one_pass(d.n_kv_heads);
  int n_tiles = (max_ctx + kWideT - 1) / kWideT;
  if (n_tiles < 1) n_tiles = 1;
  pl.score_stride = n_tiles * kWideT;
  pl.v_chunks = plain ? d.n_kv_heads : (d.rank_v + 511) / 512;
  const int cus = n_cus > 0 ? n_cus : 256;
  if (one_pass) {
    // The cheapest of one to eight tiles per split (more would let sequences of different lengths leave CUs idle) by an
    // estimate in microseconds: rounds of one workgroup per CU, 5 per tile and 5 to start and end, and the merge's walk over
    // the splits.  With four tiles at least 1 x 2000 positions take 38 us instead of 24, 4 x 1000 39 instead of 25.
    pl.v_chunks = d.n_kv_heads / kPlainHeads;
    const int first = (n_tiles + 511) / 512;  // at most 512 splits
    double best = 0;
    for (int tps = first; tps <= 8 || tps == first; ++tps) {
      const long ns = (n_tiles + tps - 1) / tps, rounds = ((long)b * pl.v_chunks * ns + cus - 1) / cus;
      const double cost = 5.0 * rounds * (tps + 1) + 0.09 * ns;
      if (tps == first || cost < best) {
        best = cost;
        pl.tiles_per_split = tps;
      }
    }
  } else {
    // uncompressed layers: a workgroup streams only one head's 16 KiB per tile, so many more of them are kept in flight
    const long want = (plain ? 8L : 2L) * cus;
    long ns = (want + (long)b * pl.v_chunks - 1) / ((long)b * pl.v_chunks);
    // four tiles per split at least, fewer while every split still has a compute unit (and the merge at most 64 splits): values of
    // one sequence of 1000 positions at rank 2048 24 -> 18 us, of 2 x 1000 (64 heads, rank 768) 27 -> 22
    long tps_min = 4;
    if (!plain) {
      tps_min = 1;
      while (tps_min < 4 && (long)b * pl.v_chunks * ((n_tiles + tps_min - 1) / tps_min) > cus) ++tps_min;
      if (tps_min < 4 && tps_min < (n_tiles + 63) / 64) tps_min = (n_tiles + 63) / 64;
    }
    if (ns > (n_tiles + tps_min - 1) / tps_min) ns = (n_tiles + tps_min - 1) / tps_min;
    if (ns > 512) ns = 512;
    if (ns > max_splits) ns = max_splits;
    if (ns < 1) ns = 1;
    pl.tiles_per_split = (int)((n_tiles + ns - 1) / ns);
  }
  pl.n_splits = (n_tiles + pl.tiles_per_split - 1) / pl.tiles_per_split;
  const int out_w = plain ? d.head_dim : d.rank_v;
  // A loop that sizes its workspace once, for its longest context and largest batch, calls with less of either, and the cheapest
  // split often takes more splits for fewer tiles (16 x 1024 positions: 16 splits, 16 x 1088: 9).  So the one-pass kernel's
  // partials are given room for a number that no call with fewer tiles or sequences exceeds: with P = b x head groups, a choice
  // of t tiles costs at least 5 P (n_tiles + splits) / cus + 0.09 splits, and no more than eight tiles per split, which cost at
  // most 45 (P (n_tiles / 8 + 1) / cus + 1) + 0.09 (n_tiles / 8 + 1).
  size_t room = pl.n_splits;
  if (one_pass) {
    const double P = (double)b * pl.v_chunks;
    room = (size_t)(n_tiles / 8.0 + (45.0 * (P + cus) + 0.09 * cus) / (5.0 * P + 0.09 * cus)) + 1;
    if (room > (size_t)n_tiles) room = n_tiles;
    if (room > 512) room = 512;
    if (room < (size_t)pl.n_splits) room = pl.n_splits;  // (rounding in the estimates)
  }
  size_t off = 0;
  pl.off_ml = off;
  off = align256w(off + (size_t)b * room * d.n_q_heads * 2 * 4);
  pl.off_o = off;
  off = align256w(off + (size_t)b * room * d.n_q_heads * out_w * 2);
  pl.off_scores = off;
  if (!one_pass) off = align256w(off + (size_t)b * d.n_q_heads * pl.score_stride * 4);
  pl.total_bytes = off;
  return pl;
}

int set_kernel_attributes_decode_wide() {
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(wide_scores_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kScoreLdsBytes) != hipSuccess)
    return LORC_EHIP;
  return LORC_OK;
}

bool wide_absorbed_shape_ok(const lorc_layer_desc& d) {
  return d.n_q_heads <= 64 && d.rank_v <= kWideMaxRank;
}

// The two streaming launches; the caller records its events around them and runs the merge.
int launch_decode_wide(const DecodeParams& p, const DecodePlan& plan, hipStream_t s) {
  const int tiles = plan.score_stride / kWideT;
  const int qb = (p.h_q + 31) / 32;
  if (plan.wide == 3) {  // absorbed query: scores on the latents, then the same value kernel
    const dim3 grid(p.b * p.n_splits * p.v_chunks);
    if (qb == 1) {
      if (int rc = launch_kernel(absorbed_scores_kernel<1>, dim3(p.b * tiles), dim3(256), 0, s, p)) return rc;
      return launch_kernel(latent_pv_kernel<1, 4, false>, grid, dim3(256), 0, s, p);
    }
    if (int rc = launch_kernel(absorbed_scores_kernel<2>, dim3(p.b * tiles), dim3(256), 0, s, p)) return rc;
    return launch_kernel(latent_pv_kernel<2, 4, false>, grid, dim3(256), 0, s, p);
  }
  if (plan.wide == 2 && plain_one_pass(p.h_kv))
    return launch_kernel(decode_plain_kernel, dim3(p.b * p.n_splits * (p.h_kv / kPlainHeads)), dim3(256), 0, s, p);
  if (plan.wide == 2) {
    const size_t lds = (size_t)p.h_q * 128 * 2;
    if (int rc = launch_kernel(plain_scores_kernel, dim3(p.b * tiles), dim3(256), lds, s, p)) return rc;
    return launch_kernel(latent_pv_kernel<1, 1, true>, dim3(p.b * p.n_splits * p.h_kv), dim3(256), 0, s, p);
  }
  if (p.G > kWideMaxG) return LORC_EUNSUPPORTED;
  const int n_pairs = (p.h_kv + 1) / 2;
  const int n_pt = p.b * ((tiles + kScorePages - 1) / kScorePages);
  if (int rc = launch_kernel(wide_scores_kernel, dim3(scores_grid(n_pt, n_pairs)), dim3(256), kScoreLdsBytes, s, p)) return rc;
  const dim3 grid(p.b * p.n_splits * p.v_chunks);
  if (qb == 1) return launch_kernel(latent_pv_kernel<1, 4, false>, grid, dim3(256), 0, s, p);
  return launch_kernel(latent_pv_kernel<2, 4, false>, grid, dim3(256), 0, s, p);
}

}  // namespace lorc
