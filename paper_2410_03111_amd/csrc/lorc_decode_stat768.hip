// Decode attention over the latent cache with the key factor held stationary, ranks 544 to 768: the form of
// lorc_decode_stat.hip for factors that take most of a workgroup's registers.
//
// Same division of work: one workgroup of eight waves (two per SIMD) owns two KV heads, every wave the factor of 16 coordinates
// of a head and their RoPE partners, and walks the context of one (sequence, context split).  At rank 768 the factor would take 192
// of a lane's 256 registers, so what is left of them decides the rest:
//   * 16x16x32 products: accumulators, keys and scores of 16 positions take 4 registers each;
//   * a tile is 32 positions (half a page: K and V latents are 48 KiB each in LDS) and its accumulators are not doubled: a
//     tile's keys are rotated at the head of the next tile's stream, one half before the products that overwrite it;
//   * FL of the NK k-steps (32 latent indices each) take their factor operands from LDS (rank 768: three of 24, 48 KiB);
//   * up to eight query heads fill half of the 16 rows of o_lat: two latent blocks share an accumulator, P entering the
//     product in the upper or the lower rows (PACK).
// Per tile: three hand-overs.  At each, one third of the K tile is released for the next tile's copies and the following third
// has landed; the second also hands over the previous tile's P and its V latents, the third releases them.  The stream of a
// tile carries the previous tile's scores, softmax and P C_v.  Rotation (queries take the base of 16 positions, keys their offset),
// softmax reference, copies and partials are those of lorc_decode_stat.hip.
// Bound by issue and hand-overs: matrix cores busy 49 % of the time at 1.94 GHz, 448 us for 32 x 8192 positions at rank 768 (0.49 of
// it their operations).  Before, the streaming kernel of lorc_decode.hip: one workgroup per (sequence, split) for all heads, factor
// operands from L2 for two products each, 586 us.  us per layer-step of the 8B shape, streaming / this: 32 x 8192 rank 768 668 / 550, rank
// 672 546 / 430, rank 544 467 / 371; 16 x 4096 rank 704 178 / 140; 1 x 700 rank 768 61 / 36; 60 x 300 rank 608 126 / 75.
#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_stationary.h"

namespace lorc {

namespace {
constexpr int kHalfT = 32;  // positions per tile

// query heads per workgroup at most, rows of a KV head's score block, 1 KiB blocks of a V tile
template <bool PACK> constexpr int kHeads = PACK ? 8 : 16;
template <int NK> constexpr int kVBlocks = (NK + 3) / 4 * 8;

template <int NK, int FL, bool PACK>
constexpr size_t stat768_fixed_lds() {
  size_t b = (size_t)(2 * NK + kVBlocks<NK>) * 1024 + (size_t)16 * FL * 1024;  // K and V tile, factor operands
  b += 1024;                                                 // sink for copies and stores that must not land anywhere
  b += (size_t)4 * kHeads<PACK> * kHalfT * 4;                // partial scores of the four quarters of a head
  b += (size_t)(PACK ? 2 : 1) * 1024;                        // P operands: heads in rows 0 .. ; PACK: and in rows 8 .. 15
  b += (size_t)2 * kHeads<PACK> * kStatQPitch * 4;           // scaled queries (fp16 pairs), rotated for the tile's two halves
  b += (size_t)3 * kStatMaxHeads * 4;                        // alpha; running max and sum at the end
  b += (size_t)64 * 8;                                       // rotation frequencies in turns per position
  return b;
}
}  // namespace

// NK: k-steps the rank is padded to;  FL: how many of them, from kF on, have their factor operands in LDS;  PACK: at most eight
// query heads per workgroup.
template <int NK, int FL, bool PACK>
__global__ __launch_bounds__(kStatThreads, 2) void decode_split_kernel(DecodeParams p) {
  constexpr int HD = 128, HALF = 64, NW = kStatWaves, NT = kStatThreads, T = kHalfT;
  constexpr int NV = kVBlocks<NK> / 8, NH = kHeads<PACK>, GR = NH / 2;  // V copies per wave and tile (also its 16-wide latent blocks of o_lat); heads; rows per KV head
  constexpr int NO = PACK ? (NV + 1) / 2 : NV;     // accumulators of o_lat
  constexpr int QW = PACK ? 1 : 2;                 // query heads a wave rotates
  constexpr int C1 = (NK + 2) / 3, C2 = 2 * C1;    // thirds of the K tile: k-steps 0 .. C1 - 1, C1 .. C2 - 1, C2 .. NK - 1
  constexpr int kBar1 = C1 - 1, kBar2 = C2 - 1, kBar3 = NK - 1;
  constexpr int kF = 4;                            // first k-step with factor operands in LDS
  static_assert(NK % 3 == 0 && C1 <= 8 && C1 >= 6, "thirds: two copies per wave, room for the softmax; ring of three operands");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, n16 = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int NQ = p.h_kv >> 1;
  const int grp = blockIdx.x / (8 * NQ), rem = blockIdx.x % (8 * NQ);
  const int hp = rem >> 3, unit = grp * 8 + (rem & 7);
  if (unit >= p.b * p.n_splits) return;
  const int seq = unit / p.n_splits, split = unit % p.n_splits;
  const int G = p.G, r_k = p.r_k, r_v = p.r_v, nk = r_k >> 5;
  const int n_heads = 2 * G, h0 = hp * n_heads;

  unsigned char* kbuf = smem;
  unsigned char* vbuf = kbuf + (size_t)2 * NK * 1024;
  unsigned char* fbuf = vbuf + (size_t)kVBlocks<NK> * 1024;
  unsigned char* sink = fbuf + (size_t)16 * FL * 1024;
  float* sbuf = reinterpret_cast<float*>(sink + 1024);
  uint16_t* pbuf = reinterpret_cast<uint16_t*>(sbuf + 4 * NH * T);
  uint32_t* qrot = reinterpret_cast<uint32_t*>(pbuf + (PACK ? 1024 : 512));
  float* alpha = reinterpret_cast<float*>(qrot + 2 * NH * kStatQPitch);
  float* m_fin = alpha + kStatMaxHeads;
  float* l_fin = m_fin + kStatMaxHeads;
  double* theta_rev_tab = reinterpret_cast<double*>(l_fin + kStatMaxHeads);
  int* ids = reinterpret_cast<int*>(theta_rev_tab + HALF);
  const uint32_t kbuf_off = (uint32_t)(uintptr_t)kbuf, vbuf_off = (uint32_t)(uintptr_t)vbuf, sink_off = (uint32_t)(uintptr_t)sink;

  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int page_begin = split * p.tiles_per_split;
  int pos_end = (page_begin + p.tiles_per_split) * kPage;
  if (pos_end > ctx) pos_end = ctx;
  const int pos_begin = page_begin * kPage;
  const int nt = pos_end > pos_begin ? (pos_end - pos_begin + T - 1) / T : 0, n_pages_here = (nt + 1) >> 1;
  const int q_pos = p.q_pos[seq];
  for (int i = tid; i < n_pages_here; i += NT) {
    const int id = p.block_table[(size_t)seq * p.max_pages + page_begin + i];
    ids[i] = id >= 0 && id < p.n_pages ? id : -1;
  }
  if (tid < (PACK ? 128 : 64)) reinterpret_cast<u32x4*>(pbuf)[tid] = u32x4{0u, 0u, 0u, 0u};
  if (tid < kStatMaxHeads) {
    alpha[tid] = 1.f;
    l_fin[tid] = 0.f;
  }
  __syncthreads();  // page ids

  // ---- latent copies (1 KiB each, lane order).  A descriptor of size zero delivers zeros, on which this kernel relies for all that
  // has to be finite before or without a copy of latents: the K tile's padding (multiplied by zero factors), the V tile of the tile
  // before the first one and of pages that are not cached (multiplied by zero weights).  Clearing both tiles by hand costs 0.4 us per
  // call, and at rank 768 registers: 32 x 4096 positions 233 -> 244 us.
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto tile_page = [&](int t) {  // page id of tile t of the split, -1 outside
    const bool in = t >= 0 && t < nt;
    const int id = __builtin_amdgcn_readfirstlane(ids[in ? t >> 1 : 0]);
    return in ? id : -1;
  };
  auto k_rsrc = [&](int id, int t) {
    const bool ok = id >= 0;
    const uint16_t* base = p.cache + (ok ? (size_t)id * p.page_elems + (size_t)(t & 1) * T * r_k : 0);
    return dma_rsrc(base, ok ? (uint32_t)T * r_k * 2u : 0u);
  };
  auto v_rsrc = [&](int id, int t) {
    const bool ok = id >= 0;
    const uint16_t* base = p.cache + (ok ? (size_t)id * p.page_elems + (size_t)kPage * r_k + (size_t)(t & 1) * 1024 : 0);
    return dma_rsrc(base, ok ? (uint32_t)kPage * r_v * 2u - (uint32_t)(t & 1) * 2048u : 0u);
  };
  // copy j (of 2) of third c of a K tile: blocks of 16 latent indices; blocks past the rank are zeros
  auto issue_k = [&](u32x4 kr, int c, int j) {
    const int first = c == 0 ? 0 : (c == 1 ? 2 * C1 : 2 * C2), count = c < 2 ? 2 * C1 : 2 * (NK - C2);
    const int i = w + NW * j, blk = first + i;
    if (i >= count || blk >= 2 * nk) kr[2] = 0u;
    dma_1k(kr, i < count ? kbuf_off + (uint32_t)blk * 1024u : sink_off, lane16, (uint32_t)blk * 1024u);
  };
  // copy j (of NV) of a V tile: 16 positions x 32 latent indices
  auto issue_v = [&](u32x4 vr, int j) {
    const int blk = w + NW * j;
    if ((blk >> 1) * 32 >= r_v) vr[2] = 0u;
    dma_1k(vr, vbuf_off + (uint32_t)blk * 1024u, lane16, (uint32_t)((blk >> 1) * 4 + (blk & 1)) * 1024u);
  };

  // ---- factor operands: column 16 wq + n16 of the wave's head (x) and its partner (y), 8 latent indices per lane
  const int kvh = w >> 2, wq = w & 3, g = 2 * hp + kvh;
  bf16x8 fx[NK], fy[NK];
  // Lane index rebuilt where it is used: registers are what this kernel is short of, not vector instructions.
  auto my_lane = [&]() {
    int l = lane_id();
    asm volatile("" : "+v"(l));
    return l;
  };
  auto f_lds = [&]() { return reinterpret_cast<uint16_t*>(fbuf) + (size_t)w * FL * 1024 + (size_t)my_lane() * 8; };
  int id_cur = tile_page(0), id_next = tile_page(1);
  {
    const u32x4 kr0 = k_rsrc(id_cur, 0);
    issue_k(kr0, 0, 0);
    issue_k(kr0, 0, 1);
    issue_k(kr0, 1, 0);
    issue_k(kr0, 1, 1);
  }
  {
    const uint32_t bk_bytes = (uint32_t)p.h_kv * HD * r_k * 2u;
    const uint32_t lane_off = (uint32_t)((kq >> 1) * 64 + 16 * (wq & 1) + n16 + 32 * (kq & 1)) * 16u;
    const uint32_t sx = (uint32_t)((g * 4 + (wq >> 1)) * 2 * nk) * 1024u, sy = (uint32_t)((g * 4 + (wq >> 1) + 2) * 2 * nk) * 1024u;
    auto load_one = [&](int ks, bf16x8& x, bf16x8& y) {  // k-steps past the rank: zeros
      const __amdgpu_buffer_rsrc_t r = make_rsrc(p.bk, ks < nk ? bk_bytes : 0u);
      x = buf_frag(r, lane_off, sx + (uint32_t)ks * 2048u);
      y = buf_frag(r, lane_off, sy + (uint32_t)ks * 2048u);
    };
    if constexpr (FL > 0) {  // (the wave's operands in LDS are its own: no hand-over)
      uint16_t* const dst = f_lds();
#pragma unroll
      for (int i = 0; i < FL; ++i) {
        bf16x8 x, y;
        load_one(kF + i, x, y);
        *reinterpret_cast<bf16x8*>(dst + (2 * i) * 512) = x;
        *reinterpret_cast<bf16x8*>(dst + (2 * i + 1) * 512) = y;
      }
    }
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
      if (ks < kF || ks >= kF + FL) load_one(ks, fx[ks], fy[ks]);
  }
  // rotation of the lane's four frequencies by its position's offset in 16
  float rc[4], rs[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float2 cs = p.lane_cs[n16 * HALF + 16 * wq + 4 * kq + j];
    rc[j] = cs.x;
    rs[j] = cs.y;
  }
  uint32_t q_raw[QW];
#pragma unroll
  for (int u = 0; u < QW; ++u) {
    const int hl = w + NW * u < n_heads ? w + NW * u : n_heads - 1;
    const uint16_t* qsrc = p.q + ((size_t)seq * p.h_q + h0 + hl) * HD + lane;
    q_raw[u] = (uint32_t)qsrc[0] | ((uint32_t)qsrc[HALF] << 16);
  }
  if (tid < HALF) theta_rev_tab[tid] = p.rope_tab[tid] * kInvTwoPi;
  for (int i = tid; i < 2 * NH * kStatQPitch; i += NT) qrot[i] = 0u;  // read before the first tile's queries are there
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  // ---- lane bases of what the stream addresses
  const uint16_t* kl = reinterpret_cast<const uint16_t*>(kbuf) + (size_t)((kq >> 1) * 64 + n16 + 32 * (kq & 1)) * 8;
  const unsigned char* v_src = vbuf + (size_t)(((w >> 1) * 2 + (kq >> 1)) * 64 + 16 * (w & 1) + n16 + 32 * (kq & 1)) * 16;
  const uint32_t* q_src = qrot + (size_t)(kvh * G + (n16 < G ? n16 : 0)) * kStatQPitch + 16 * wq + 4 * kq;
  float* s_dst = 4 * kq < GR ? sbuf + (size_t)((wq * 2 + kvh) * GR + 4 * kq) * T + n16 : reinterpret_cast<float*>(sink) + n16;
  auto sm_head = [&](int ln) {
    const int h = PACK ? w : 2 * w + (ln >> 5);
    return h < n_heads ? h : n_heads - 1;
  };
  f32x4s o[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) o[i] = f32x4s{0.f, 0.f, 0.f, 0.f};
  float m_run = kNegInfS, m_high = kNegInfS, l_run = 0.f;
  f32x4s ax[2], ay[2];
  const f32x4s zero4 = {0.f, 0.f, 0.f, 0.f};
  ax[0] = ax[1] = ay[0] = ay[1] = zero4;

  auto rotate = [&](f16x8& kf, const f32x4s& x, const f32x4s& y) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      kf[2 * j] = static_cast<_Float16>(x[j] * rc[j] - y[j] * rs[j]);
      kf[2 * j + 1] = static_cast<_Float16>(y[j] * rc[j] + x[j] * rs[j]);
    }
    asm volatile("" : "+v"(kf));  // here, not where it is first used
  };
  auto score = [&](const f16x8& q, const f16x8& kf) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(q, kf, zero4, 0, 0, 0); };
  auto score_load = [&](int sb) { return __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(q_src + sb * NH * kStatQPitch)); };
  auto score_store = [&](const f32x4s& sa, int sb) {
#pragma unroll
    for (int j = 0; j < 4; ++j) s_dst[j * T + sb * 16] = sa[j];
  };
  struct Query {
    double turns;
    float fr, cs, sn;
  };
  auto query_reduce = [&](Query& qr) { qr.fr = (float)(qr.turns - rint(qr.turns)); };
  auto query_angle = [&](Query& qr) {
    qr.cs = __builtin_amdgcn_cosf(qr.fr);
    qr.sn = __builtin_amdgcn_sinf(qr.fr);
  };
  auto query_store = [&](const Query& qr, int sb) {
#pragma unroll
    for (int u = 0; u < QW; ++u) {
      const int hl = w + NW * u < n_heads ? w + NW * u : n_heads - 1;
      const float x = __uint_as_float(q_raw[u] << 16) * p.q_scale, y = __uint_as_float(q_raw[u] & 0xffff0000u) * p.q_scale;
      f16x2 v;
      v[0] = static_cast<_Float16>(x * qr.cs - y * qr.sn);
      v[1] = static_cast<_Float16>(y * qr.cs + x * qr.sn);
      qrot[(sb * NH + hl) * kStatQPitch + my_lane()] = __builtin_bit_cast(uint32_t, v);
    }
  };
  struct Softmax {
    float a[4], s, mx, pv, al;
  };
  auto softmax_a = [&](Softmax& sm) {
    const int ln = my_lane(), h = sm_head(ln);
    const float* src = sbuf + (size_t)(h < G ? h : GR + h - G) * T + (ln & 31);
#pragma unroll
    for (int q = 0; q < 4; ++q) sm.a[q] = src[q * NH * T];
  };
  auto softmax_b1 = [&](Softmax& sm, int valid_, bool page_ok_, float fill_) {
    sm.s = page_ok_ ? (sm.a[0] + sm.a[1]) + (sm.a[2] + sm.a[3]) : fill_;
    if (valid_ < T && (my_lane() & 31) >= valid_) sm.s = kNegInfS;
  };
  auto softmax_b2 = [&](Softmax& sm) {
    sm.mx = row_max_step<0>(sm.s);
    sm.mx = row_max_step<1>(sm.mx);
    sm.mx = row_max_step<2>(sm.mx);
  };
  auto softmax_b3 = [&](Softmax& sm) {
    sm.mx = row_max_step<3>(sm.mx);
    const float2 rows = row_pair(sm.mx);
    sm.mx = fmaxf(rows.x, rows.y);
  };
  auto softmax_c = [&](Softmax& sm) {
    m_high = fmaxf(m_high, sm.mx);
    const float m_new = fmaxf(sm.mx, m_high - kBelow);
    const float m_ref = fmaxf(m_new, -1e30f);
    sm.pv = __builtin_amdgcn_exp2f(sm.s - m_ref);
    sm.al = __builtin_amdgcn_exp2f(m_run - m_ref);
    m_run = m_new;
  };
  auto softmax_d = [&](const Softmax& sm, bool page_ok_) {
    const int ln = my_lane(), h = sm_head(ln), pos = ln & 31;
    alpha[h] = sm.al;
    // P operand: position 8 kg + e of head h sits in lane h + 16 kg, element e; PACK: the upper half of the wave (the same head) files
    // it for the rows 8 .. 15
    const int row = PACK ? h + 8 * (ln >> 5) : h;
    uint16_t* p_dst = pbuf + (PACK ? 512 * (ln >> 5) : 0) + (row + 16 * (pos >> 3)) * 8 + (pos & 7);
    const uint32_t bits = bf16_bits(sm.pv);
    l_run = l_run * sm.al + sm.pv;
    *p_dst = page_ok_ ? (uint16_t)bits : (uint16_t)0;
  };
  struct PV {
    f32x4s al;
    bf16x8 pa;
  };
  auto p_load = [&](int rows) { return load_frag(pbuf + rows * 512 + (size_t)my_lane() * 8); };
  auto pv_prep = [&](PV& pv) {
    pv.al = *reinterpret_cast<const f32x4s*>(alpha + 4 * (PACK ? kq & 1 : kq));
    pv.pa = p_load(0);
  };
  // The wave's latent blocks w + 8 i in the order in which they are taken: with PACK those that go to the lower rows first
  constexpr auto block = [](int k) constexpr { return PACK ? (k < (NV + 1) / 2 ? 2 * k : 2 * (k - (NV + 1) / 2) + 1) : k; };
  auto v_load = [&](int i) { return *reinterpret_cast<const u32x4*>(v_src + i * NW * 1024); };
  auto pv_mfma = [&](const PV& pv, const u32x4& v, auto k_c) {
    constexpr int K = decltype(k_c)::value, I = block(K), oi = PACK ? I / 2 : I;
    if constexpr (!PACK || (I & 1) == 0) o[oi] *= pv.al;
    o[oi] = mfma16(pv.pa, __builtin_bit_cast(bf16x8, v), o[oi]);
  };

  int id_prev = -1;
  bool page_ok_prev = false;
  float fill = kNegInfS;
  bf16x8 c[3];  // latent operands (k-step, half) in the order of use, two ahead
  c[0] = load_frag(kl);
  c[1] = load_frag(kl + 128);

  for (int t = 0; t < nt; ++t) {
    const int pos0 = pos_begin + t * T;
    const bool page_ok = id_cur >= 0;
    const u32x4 kr_cur = k_rsrc(id_cur, t), kr_next = k_rsrc(id_next, t + 1), v_prev = v_rsrc(id_prev, t - 1);
    int id_after_raw = -1, id_after = -1;
    f16x8 kf[2], sq;
    f32x4s sa;
    Softmax sm;
    PV pv;
    u32x4 vv;
    Query qr;
    double theta_rev = 0.0;
    bf16x8 fl[2];
    static_for<NK>([&](auto s_c) {
      constexpr int s = decltype(s_c)::value, nx = (s + 1) % NK;
      // -- hand-overs: third 1 has landed, third 0 is free (also: scores are complete); third 2 and the previous tile's V have landed,
      // third 1 is free (also: P, this tile's queries); the next tile's third 0 has landed, third 2 and the V tile are free
      if constexpr (s == kBar1) dma_barrier<2 + NV>();
      if constexpr (s == kBar2) dma_barrier<2>();
      if constexpr (s == kBar3) dma_barrier<2>();
      // -- copies: this tile's third 2 and the previous tile's V right at the start, the next tile's thirds as they become free
      if constexpr (s == 0) {
        issue_k(kr_cur, 2, 0);
        issue_k(kr_cur, 2, 1);
      }
      static_for<NV>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        if constexpr (s == 1 + j / 2) issue_v(v_prev, j);
      });
      if constexpr (s == kBar1 || s == kBar1 + 2) issue_k(kr_next, 0, (s - kBar1) / 2);
      if constexpr (s == kBar2 || s == kBar2 + 2) issue_k(kr_next, 1, (s - kBar2) / 2);
      auto read_ahead = [&](auto f_c) {  // operand f + 2 of the tile (or the first ones of the next)
        constexpr int f = (decltype(f_c)::value + 2) % (2 * NK);
        c[(decltype(f_c)::value + 2) % 3] = load_frag(kl + (f >> 1) * 1024 + (f & 1) * 128);
      };
      bf16x8 a_x, a_y;
      if constexpr (s >= kF && s < kF + FL) {
        a_x = fl[0];
        a_y = fl[1];
      } else {
        a_x = fx[s];
        a_y = fy[s];
      }
      // -- the products; the previous tile's keys leave the accumulators before they are overwritten
      if constexpr (s == 0) {
        sq = score_load(0);
        rotate(kf[0], ax[0], ay[0]);
      }
      read_ahead(std::integral_constant<int, 2 * s>{});
      ax[0] = mfma16(a_x, c[2 * s % 3], s == 0 ? zero4 : ax[0]);
      ay[0] = mfma16(a_y, c[2 * s % 3], s == 0 ? zero4 : ay[0]);
      if constexpr (s == 0) rotate(kf[1], ax[1], ay[1]);
      read_ahead(std::integral_constant<int, 2 * s + 1>{});
      ax[1] = mfma16(a_x, c[(2 * s + 1) % 3], s == 0 ? zero4 : ax[1]);
      ay[1] = mfma16(a_y, c[(2 * s + 1) % 3], s == 0 ? zero4 : ay[1]);
      if constexpr (FL > 0 && nx >= kF && nx < kF + FL) {
        const uint16_t* src = f_lds();
        fl[0] = load_frag(src + 2 * (nx - kF) * 512);
        fl[1] = load_frag(src + (2 * (nx - kF) + 1) * 512);
      }
      // -- scores of the previous tile
      if constexpr (s == 1) {
        sa = score(sq, kf[0]);
        sq = score_load(1);
      }
      if constexpr (s == 2) {
        score_store(sa, 0);
        sa = score(sq, kf[1]);
      }
      if constexpr (s == 3) score_store(sa, 1);
      // -- page id of the tile after the next
      if constexpr (s == 2) id_after_raw = ids[t + 2 < nt ? (t + 2) >> 1 : 0];
      if constexpr (s == 4) id_after = t + 2 < nt ? __builtin_amdgcn_readfirstlane(id_after_raw) : -1;
      // -- softmax of the previous tile
      if constexpr (s == kBar1) softmax_a(sm);
      if constexpr (s == kBar1 + 1) softmax_b1(sm, T, page_ok_prev, fill);
      if constexpr (s == kBar1 + 2) softmax_b2(sm);
      if constexpr (s == kBar1 + 3) softmax_b3(sm);
      if constexpr (s == kBar1 + 4) softmax_c(sm);
      if constexpr (s == kBar1 + 5) softmax_d(sm, page_ok_prev);
      // -- this tile's queries
      if constexpr (s == kBar1) theta_rev = theta_rev_tab[lane_id()];
      if constexpr (s == kBar1 + 1) qr.turns = (double)(q_pos - pos0) * theta_rev;
      if constexpr (s == kBar1 + 2) query_reduce(qr);
      if constexpr (s == kBar1 + 3) {
        query_angle(qr);
        query_store(qr, 0);
      }
      if constexpr (s == kBar1 + 4) {
        qr.turns = __builtin_fma(-16.0, theta_rev, qr.turns);
        query_reduce(qr);
      }
      if constexpr (s == kBar1 + 5) {
        query_angle(qr);
        query_store(qr, 1);
      }
      // -- P C_v of the previous tile
      if constexpr (s == kBar2) pv_prep(pv);
      static_for<NV>([&](auto i_c) {
        constexpr int k = decltype(i_c)::value;
        if constexpr (s == kBar2 + 2 + k) {
          pv_mfma(pv, vv, i_c);
          if constexpr (PACK && k == (NV + 1) / 2 - 1) pv.pa = p_load(1);
        }
      });
      static_for<NV>([&](auto i_c) {
        if constexpr (s == kBar2 + 1 + decltype(i_c)::value) vv = v_load(block(decltype(i_c)::value));
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    static_assert(kBar1 + 5 < kBar2 && kBar2 + 1 + NV - 1 < kBar3 && kBar2 + 2 + NV - 1 <= kBar3 && 1 + (NV - 1) / 2 < kBar1 && kF + FL <= kBar1 + 1, "stream schedule");
    page_ok_prev = page_ok;
    fill = 0.f;
    asm volatile("" : "+s"(fill));  // (the compiler would peel the first tile, a second copy of the stream)
    id_prev = id_cur;
    id_cur = id_next;
    id_next = id_after;
  }

  // ---- the last tile's scores, softmax and P C_v (only the last tile of a context can be ragged)
  if (nt > 0) {
    const int valid = pos_end - (pos_begin + (nt - 1) * T);
    const u32x4 vr = v_rsrc(id_prev, nt - 1);
    static_for<NV>([&](auto j_c) { issue_v(vr, decltype(j_c)::value); });
    f16x8 kf[2];
    rotate(kf[0], ax[0], ay[0]);
    rotate(kf[1], ax[1], ay[1]);
    score_store(score(score_load(0), kf[0]), 0);
    score_store(score(score_load(1), kf[1]), 1);
    lds_barrier();
    Softmax sm;
    PV pv;
    softmax_a(sm);
    softmax_b1(sm, valid, page_ok_prev, 0.f);
    softmax_b2(sm);
    softmax_b3(sm);
    softmax_c(sm);
    softmax_d(sm, page_ok_prev);
    dma_barrier<0>();
    pv_prep(pv);
    int nv = valid - 8 * kq;  // slots past the context hold anything
    nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
    const uint32_t vmask = (1u << nv) - 1u;
    static_for<NV>([&](auto i_c) {
      if constexpr (PACK && decltype(i_c)::value == (NV + 1) / 2) pv.pa = p_load(1);
      u32x4 v = v_load(block(decltype(i_c)::value));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t two = (vmask >> (2 * e)) & 3u;
        v[e] &= (two & 1u ? 0x0000ffffu : 0u) | (two & 2u ? 0xffff0000u : 0u);
      }
      pv_mfma(pv, v, i_c);
    });
  }

  // ---- partials of this split (format of lorc_decode.hip); the staging area reuses the K tile
  __builtin_amdgcn_s_waitcnt(0);
  l_run += half_wave_peer<0>(l_run);
  l_run += half_wave_peer<1>(l_run);
  l_run += half_wave_peer<2>(l_run);
  l_run += half_wave_peer<3>(l_run);
  const float2 l_rows = row_pair(l_run);
  const int sm_h = sm_head(lane);
  m_fin[sm_h] = m_run;
  l_fin[sm_h] = l_rows.x + l_rows.y;
  __syncthreads();
  const size_t pbase = (size_t)seq * p.n_splits + split;
  if (tid < n_heads) {
    p.part_ml[(pbase * p.h_q + h0 + tid) * 2 + 0] = m_fin[tid];
    p.part_ml[(pbase * p.h_q + h0 + tid) * 2 + 1] = l_fin[tid];
  }
  const int pitch = r_v * 2 + 16;
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int blk = PACK ? 2 * i + (kq >> 1) : i, jb = w + NW * blk;
    if (blk < NV && jb * 16 < r_v) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = 4 * (PACK ? kq & 1 : kq) + j;
        const float l = l_fin[row], inv = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
        *reinterpret_cast<uint16_t*>(smem + (size_t)row * pitch + (jb * 16 + n16) * 2) = f16_bits(o[i][j] * inv);
      }
    }
  }
  lds_barrier();
  uint16_t* dst_rows = p.part_o + (pbase * p.h_q + h0) * r_v;
  const int cpr = r_v >> 3, n_chunks = n_heads * cpr;  // 16-byte chunks
  for (int i = tid; i < n_chunks; i += NT) {
    const int h = i / cpr, cc = i - h * cpr;
    *reinterpret_cast<u32x4*>(dst_rows + (size_t)i * 8) = *reinterpret_cast<const u32x4*>(smem + (size_t)h * pitch + cc * 16);
  }
}

// ------------------------------------------------------------------------------------------------ host
namespace {
using Stat768Kernel = void (*)(DecodeParams);
struct Stat768Form {
  Stat768Kernel kernel;
  size_t lds;
  const char* symbol;
};
Stat768Form stat768_form(int rank, bool pack) {
  if (!pack) return rank <= 576 ? Stat768Form{decode_split_kernel<18, 0, false>, stat768_fixed_lds<18, 0, false>(), "decode_split_kernel<18, 0, false>"}
                                : Stat768Form{decode_split_kernel<21, 3, false>, stat768_fixed_lds<21, 3, false>(), "decode_split_kernel<21, 3, false>"};
  if (rank <= 576) return {decode_split_kernel<18, 0, true>, stat768_fixed_lds<18, 0, true>(), "decode_split_kernel<18, 0, true>"};
  if (rank <= 672) return {decode_split_kernel<21, 1, true>, stat768_fixed_lds<21, 1, true>(), "decode_split_kernel<21, 1, true>"};
  return {decode_split_kernel<24, 3, true>, stat768_fixed_lds<24, 3, true>(), "decode_split_kernel<24, 3, true>"};
}
}  // namespace

// Groups of more than four heads need twice the accumulators of o_lat, which leaves room for 672 latent indices; beyond, they take
// the three launches of lorc_decode_wide.hip.  70B shape, us per layer-step, three launches / this: 32 x 8192 rank 640 549 / 439, rank 544
// 515 / 382; 1 x 1000 rank 640 62 / 27; 16 x 2000 rank 672 112 / 81.
bool stationary768_shape_ok(const lorc_layer_desc& d) {
  const int G = d.n_q_heads / d.n_kv_heads, rank = d.rank_k > d.rank_v ? d.rank_k : d.rank_v;
  return d.head_dim == 128 && d.n_kv_heads % 2 == 0 && G <= 8 && rank > 512 && rank <= (G <= 4 && d.n_q_heads <= 32 ? 768 : 672) && d.rank_k > 128;
}

const char* stationary768_kernel_symbol(const lorc_layer_desc& d) {
  return stat768_form(d.rank_k > d.rank_v ? d.rank_k : d.rank_v, 2 * (d.n_q_heads / d.n_kv_heads) <= 8).symbol;
}

int set_kernel_attributes_decode_stationary768() {
  for (bool pack : {true, false})
    for (int rank : {576, 672, 768})
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(stat768_form(rank, pack).kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024) != hipSuccess) return LORC_EHIP;
  return LORC_OK;
}

int launch_decode_stationary768_split(const DecodeParams& p, const DecodePlan& plan, hipStream_t s) {
  const int rank = p.r_k > p.r_v ? p.r_k : p.r_v;
  const Stat768Form f = stat768_form(rank, 2 * p.G <= 8);
  const size_t lds = (f.lds + (size_t)plan.tiles_per_split * 4 + 15) & ~(size_t)15;
  if (lds > 160 * 1024 || plan.tiles_per_split > kStatMaxTiles || p.G > 8 || rank > (p.G <= 4 ? 768 : 672)) return LORC_EUNSUPPORTED;
  const int units = p.b * p.n_splits, nq = p.h_kv / 2;
  return launch_kernel(f.kernel, dim3(((units + 7) / 8) * 8 * nq), dim3(kStatThreads), lds, s, p);
}

}  // namespace lorc
