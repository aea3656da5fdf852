// Decode attention over the latent cache with the key factor held stationary in registers (Eq. 1 on cached
// latents; GQA of Section 4.3; RoPE applied at read time to the rebuilt keys, as the cache holds un-rotated latents).
//
// The rebuild K^T = B_k^T C_k^T is a [n x r_k] x [r_k x positions] product whose left operand never changes.  One
// workgroup (eight waves, two per SIMD, 256 registers each) owns two KV heads: every wave keeps the 32 columns of
// B_k it is responsible for (16 coordinates of a head and their RoPE partners) in registers for the whole kernel, 128
// registers at rank 512, and walks the context of one (sequence, context split).  The only operand that moves is
// the latent tile: it is copied global -> LDS once per workgroup and read from there by the eight waves, 1 KiB per
// matrix-core op; the factor causes no traffic at all.  The h_kv / 2 workgroups that share a (sequence, split) are dealt
// to the same XCD, so that the latent tile they all read comes out of that XCD's L2 after the first of them has fetched it.
//
// Per 64-position tile: rebuild the wave's 32 x 64 block of K^T (position block 0, then 1), rotate it in
// registers, score it against the group's query heads (fp16 operands), leave the four quarter-head partial scores in
// LDS; then one softmax pass over the workgroup's 2 G heads x 64 positions, and o_lat += P C_v on 16x16x32
// matrix-core ops with the V latents read from their LDS copy.  Split partials and the merge are those of
// lorc_decode.hip.
//
// Rotation: R(base + l) k against R(q_pos) q is R(l) k against R(q_pos - base) q.  The keys therefore only take the
// angles of their offset l < 32 in the position block, which are the same for every tile (sixteen registers per lane, from
// the packed table), and the base goes to the queries, 2 G rows per position block instead of 32 keys per head.
//
// Why two waves per SIMD and this rotation: with one wave of 64 columns per SIMD and per-key angles the matrix cores were
// busy 46 % of the time, because vector instructions of any wave add to the matrix-core ops of a SIMD instead of hiding under them;
// a tile took 10.2 k cycles, 302 vector instructions per wave once split over eight waves still 8.2 k.  Now 144 of them (addresses are
// lane bases plus immediates, angles constants, the running sum stays per lane): 7.3 k cycles, busy 64 %; the rebuild alone with its copies
// takes 5.2 k.  What is left is power: the clock falls from 1.79 to 1.43 GHz under the counters as the matrix cores get busier, and the same
// stream without the latent copies runs a quarter faster.  Per layer-step, append and merge included: 70B shape, 64 x 32768 positions, rank 512:
// 2559 -> 2243 us; 8B shape, 16 x 4096: 96.5 -> 87.8; 1 x 1337: 27.0 -> 23.7.
//
// Latent copies are direct global -> LDS loads issued from inline assembly, on purpose: the compiler would make
// every LDS read that follows such a load in program order wait for it, which forbids refilling one part of the K
// tile while another is being read.  Their completion is tracked by hand (fixed number of loads per wave between
// any two waits, s_waitcnt vmcnt(N) immediates).  The K tile is a ring of four chunks, each refilled for the next
// tile as soon as all waves have consumed it, so every chunk has a whole tile time to arrive.
#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_rebuild.h"
#include "lorc_stationary.h"

namespace lorc {

constexpr int kStatTile = 64;          // positions per tile = one cache page
constexpr int kStatVLoads = 64 / kStatWaves;  // 1 KiB V copies per wave and tile (r_v <= 512)
constexpr int kStatMaxNks = 32;        // k-steps (of 16 latent indices) whose factor operands a wave holds at most

__host__ __device__ inline size_t stat_lds_bytes(int nks_pad, int tiles_per_split) {
  size_t b = (size_t)2 * nks_pad * 1024;                  // K tile, padded to nks_pad k-steps per position block
  b += 64 * 1024;                                         // V tile (page order), padded to 512 latent indices
  b += 1024;                                              // sink for copies that must not land anywhere
  b += (size_t)4 * kStatMaxHeads * kStatTile * 4;         // partial scores of the four quarters of a head
  b += (size_t)2 * 1024;                                  // P operands
  b += (size_t)2 * kStatMaxHeads * kStatQPitch * 4;       // scaled queries (fp16 pairs), rotated for the tile's two position blocks
  b += (size_t)3 * kStatMaxHeads * 4;                     // alpha; running max and sum at the end
  b += (size_t)64 * 8;                                    // rotation frequencies in turns per position
  b += (size_t)tiles_per_split * 4;                       // page ids of the split
  return (b + 15) & ~(size_t)15;
}

// Where the latent copies of a tile sit in its rebuild stream (compile-time table).  The stream has NG = 4 H k-steps;
// chunk c of the K tile holds k-steps [c H, (c + 1) H).  A copy may only be issued once every wave is through the
// data it overwrites: chunks 0 / 1 / 2 of the next tile after the barriers kB2 / kB3 / kB4, chunk 3 and the V tile
// after kB0 (their copies wrap around into the next tile's stream).  Copies are spread, at most a few per k-step:
// each costs issue time next to the matrix-core stream, and a burst fills the memory pipeline's queue.
template <int NKS>
struct CopySched {
  static constexpr int H = NKS / 2, NG = 4 * H, D = 3, KI = (H + kStatWaves - 1) / kStatWaves, NV = kStatVLoads, MAXI = 4;
  static constexpr int kB0 = NG - D, kB1 = H - D, kB2 = 2 * H - D, kB3 = 3 * H - D, kB4 = 3 * H + H / 2;
  int n[NG];            // copies issued in k-step gi (after the step's barrier, if it has one)
  int kind[NG][MAXI];   // 0 .. 3: chunk of the K tile, 4: V tile
  int idx[NG][MAXI];    // which of the wave's copies of that kind
  constexpr void put(int step, int k, int j) {
    kind[step][n[step]] = k;
    idx[step][n[step]] = j;
    ++n[step];
  }
  constexpr void place(int k, int count, int first) {  // one copy every 4 H / 16 k-steps from `first` on
    for (int j = 0; j < count; ++j) put((first + (j * 4 * H) / 16) % NG, k, j);
  }
  constexpr CopySched() : n{}, kind{}, idx{} {
    place(4, NV, kB0);
    place(3, KI, kB0 + 1);
    place(0, KI, kB2 + 1);
    place(1, KI, kB3 + 1);
    for (int j = 0; j < KI; ++j) put(kB4 + j, 2, j);
  }
  // Copies issued after the last one of kind k and before the barrier of k-step gb (which precedes that step's own
  // copies), walking back around the stream: the vmcnt that guarantees kind k has landed.
  constexpr int younger(int k, int gb) const {
    int count = 0;
    for (int back = 1; back <= NG; ++back) {
      const int s = ((gb - back) % NG + NG) % NG;
      for (int i = n[s] - 1; i >= 0; --i) {
        if (kind[s][i] == k) return count;
        ++count;
      }
    }
    return count;
  }
};

// NKS: k-steps (of 16 latent indices) the K tile is padded to; ranks up to 16 * NKS.  Padding k-steps multiply zero
// factor operands with a zeroed part of the tile.  PPL: positions of a tile that one lane takes through the softmax: a
// wave for each of up to eight query heads (1), or half a wave for each of up to sixteen (2).
template <int NKS, int PPL>
__device__ __forceinline__ void stationary_split(const DecodeParams& p) {
  constexpr int HD = 128, HALF = 64, T = kStatTile, NW = kStatWaves, NT = kStatThreads;
  static_assert(NKS % 4 == 0 && NKS <= 32, "chunks of the K ring");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // workgroup -> (sequence, split, head pair): the head pairs of one (sequence, split) are 8 workgroup ids apart,
  // i.e. on one XCD, and next to each other in dispatch order
  const int NQ = p.h_kv >> 1;
  const int grp = blockIdx.x / (8 * NQ), rem = blockIdx.x % (8 * NQ);
  const int hp = rem >> 3, unit = grp * 8 + (rem & 7);
  if (unit >= p.b * p.n_splits) return;
  const int seq = unit / p.n_splits, split = unit % p.n_splits;
  const int G = p.G, r_k = p.r_k, r_v = p.r_v, nks = r_k >> 4;
  const int n_heads = 2 * G;               // query heads of this workgroup
  const int h0 = hp * n_heads;             // its first query head

  // Lane index rebuilt where it is used (two VALU ops), so that nothing derived from it stays in a register across the
  // rebuild stream.
  auto my_lane = [&]() {
    int l = lane_id();
    asm volatile("" : "+v"(l));
    return l;
  };

  unsigned char* kbuf = smem;
  unsigned char* vbuf = kbuf + (size_t)2 * NKS * 1024;
  unsigned char* sink = vbuf + 64 * 1024;
  float* sbuf = reinterpret_cast<float*>(sink + 1024);
  uint16_t* pbuf = reinterpret_cast<uint16_t*>(sbuf + 4 * kStatMaxHeads * T);
  uint32_t* qrot = reinterpret_cast<uint32_t*>(pbuf + 1024);
  float* alpha = reinterpret_cast<float*>(qrot + 2 * kStatMaxHeads * kStatQPitch);
  float* m_fin = alpha + kStatMaxHeads;
  float* l_fin = m_fin + kStatMaxHeads;
  double* theta_rev_tab = reinterpret_cast<double*>(l_fin + kStatMaxHeads);  // turns per position of frequency i
  int* ids = reinterpret_cast<int*>(theta_rev_tab + HALF);
  const uint32_t kbuf_off = (uint32_t)(uintptr_t)kbuf, vbuf_off = (uint32_t)(uintptr_t)vbuf, sink_off = (uint32_t)(uintptr_t)sink;

  // ---- what the set-up needs from memory
  int ctx = p.ctx_len[seq];
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  const int tile_begin = split * p.tiles_per_split;
  int tile_end = tile_begin + p.tiles_per_split;
  const int n_tiles = (ctx + T - 1) / T;
  if (tile_end > n_tiles) tile_end = n_tiles;
  const int nt = tile_end > tile_begin ? tile_end - tile_begin : 0;
  const int q_pos = p.q_pos[seq];

  const int kvh = w >> 2, wq = w & 3;  // this wave's KV head of the pair; its frequencies are 16 wq .. 16 wq + 15
  bf16x8 bk[NKS];                      // stationary factor operands, loaded below while the first latent chunks travel
  // page ids of the split (validated here: -1 = not cached)
  for (int i = tid; i < nt; i += NT) {
    const int id = p.block_table[(size_t)seq * p.max_pages + tile_begin + i];
    ids[i] = id >= 0 && id < p.n_pages ? id : -1;
  }
  // the K tile's padding, the V tile (read under a zero P before its first copy lands) and the P operands start as zeros
  {
    const u32x4 z = {0u, 0u, 0u, 0u};
    if (nks < NKS)
      for (int i = tid; i < (2 * NKS * 1024) / 16; i += NT) reinterpret_cast<u32x4*>(kbuf)[i] = z;
    for (int i = tid; i < 64 * 1024 / 16; i += NT) reinterpret_cast<u32x4*>(vbuf)[i] = z;
    if (tid < 128) reinterpret_cast<u32x4*>(pbuf)[tid] = z;
    if (tid < kStatMaxHeads) {
      alpha[tid] = 1.f;
      l_fin[tid] = 0.f;
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();  // page ids and zeroed tiles in place: the copies may start

  // ---- latent copies.  Wave w moves blocks w, w + 8, ... of whatever is copied.
  constexpr CopySched<NKS> sched{};
  constexpr int H = sched.H, NG = sched.NG, D = sched.D;
  constexpr int kB0 = sched.kB0, kB1 = sched.kB1, kB2 = sched.kB2, kB3 = sched.kB3, kB4 = sched.kB4;
  // descriptor of one part of a cached page (id < 0: not cached, or no such tile: a descriptor of size zero, whose
  // copies fetch nothing and deliver zeros)
  auto page_rsrc = [&](int id, uint32_t part_off, uint32_t part_bytes) {
    const bool ok = id >= 0 && id < p.n_pages;
    const uint16_t* base = p.cache + (ok ? (size_t)id * p.page_elems : 0);
    return dma_rsrc(reinterpret_cast<const unsigned char*>(base) + (ok ? part_off : 0u), ok ? part_bytes : 0u);
  };
  auto k_rsrc = [&](int id) { return page_rsrc(id, 0u, (uint32_t)T * r_k * 2u); };
  auto v_rsrc = [&](int id) { return page_rsrc(id, (uint32_t)T * r_k * 2u, (uint32_t)T * r_v * 2u); };
  auto tile_id = [&](int t_local) {  // page id of tile t_local of the split, -1 outside [0, nt)
    const bool in_split = t_local >= 0 && t_local < nt;
    const int id = __builtin_amdgcn_readfirstlane(ids[in_split ? t_local : 0]);
    return in_split ? id : -1;
  };
  // copy j (of KI) of chunk c of a K tile: position block c / 2, k-step (c % 2) H + w + 8 j; k-steps past the rank
  // go to the sink
  // the one lane-derived value that stays in a register for the whole kernel: every copy needs it (16 per tile)
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto issue_k_copy = [&](const u32x4& kr, int c, int j) {
    const int pb = c >> 1, ks = (c & 1) * H + w + NW * j;
    const bool real = ks < nks && w + NW * j < H;
    dma_1k(kr, real ? kbuf_off + (uint32_t)(pb * NKS + ks) * 1024u : sink_off, lane16, real ? (uint32_t)(pb * nks + ks) * 1024u : 0u);
  };
  // copy j of a V tile: block w + 8 j (1 KiB: 16 positions x 32 latent indices)
  auto issue_v_copy = [&](const u32x4& vr, int j) {
    const int blk = w + NW * j;
    const bool real = blk * 8 < r_v;
    dma_1k(vr, real ? vbuf_off + (uint32_t)blk * 1024u : sink_off, lane16, real ? (uint32_t)blk * 1024u : 0u);
  };
  // The copies the schedule places in k-step gi.  kr_cur / kr_next: K parts of the current and the next tile's page,
  // v_prev / v_cur: V parts of the previous and the current tile's page.  Chunks 0 .. 2 are the next tile's; chunk 3
  // and the V tile are released at kB0, their copies wrap around into the next tile's stream.
  auto issue_step = [&](auto gi_c, const u32x4& kr_cur, const u32x4& kr_next, const u32x4& v_prev, const u32x4& v_cur) {
    constexpr int gi = decltype(gi_c)::value;
    static_for<sched.MAXI>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      if constexpr (i < sched.n[gi]) {
        constexpr int kind = sched.kind[gi][i], j = sched.idx[gi][i];
        if constexpr (kind < 3) issue_k_copy(kr_next, kind, j);
        else if constexpr (kind == 3) issue_k_copy(gi >= kB0 ? kr_next : kr_cur, 3, j);
        else issue_v_copy(gi >= kB0 ? v_cur : v_prev, j);
      }
    });
  };

  constexpr int NB = 32 / NW;  // 16-wide latent blocks of o_lat per wave
  f32x4s o[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o[i] = f32x4s{0.f, 0.f, 0.f, 0.f};

  // Addresses inside the stream are these lane-derived bases plus immediates: next to the matrix cores every vector
  // instruction of both waves of a SIMD costs its issue time.
  const uint16_t* kl = reinterpret_cast<const uint16_t*>(kbuf) + (size_t)lane * 8;   // (also the P operands': same lane offset)

  f32x16 zero16;
#pragma unroll
  for (int j = 0; j < 16; ++j) zero16[j] = 0.f;

  // The wave's K^T block: rows 0 .. 15 are the coordinates 16 wq + row of the head, rows 16 .. 31 their partners (+ 64), so
  // that a lane holds both of a pair (registers j and j + 8), for position l32 of the block.
  // Rotation of rows [J0, J1) of a block into fp16 score operands: (x, y) pairs, element order = row order.
  float rc[8], rs[8];  // (cos, sin)(l32 theta) of the lane's eight frequencies
  auto rotate_rows = [&](const f32x16& acc, f16x8 (&kf)[2], auto j0_c, auto j1_c) {
    constexpr int J0 = decltype(j0_c)::value, J1 = decltype(j1_c)::value;
    static_for<J1 - J0>([&](auto d_c) {
      constexpr int j = J0 + decltype(d_c)::value;
      const float x = acc[j], y = acc[j + 8];
      kf[j >> 2][2 * (j & 3)] = static_cast<_Float16>(x * rc[j] - y * rs[j]);
      kf[j >> 2][2 * (j & 3) + 1] = static_cast<_Float16>(y * rc[j] + x * rs[j]);
    });
    if constexpr (J1 % 4 == 0) {  // the rotation happens here, not where its result is first used
      f16x8& done = kf[J1 / 4 - 1];
      asm volatile("" : "+v"(done));
    }
  };
  // Queries of the workgroup's heads for a position block: rotated by the distance to the block's base, fp16, in LDS as
  // (x, y) pairs.  Lane = frequency; wave w takes head w (and w + 8); waves past the last head repeat it (same values to the
  // same words).  In stages of few vector instructions, like everything that rides in the stream.
  float qx[PPL], qy[PPL];  // scaled (softmax scale x log2 e)
  uint32_t* q_dst = qrot + (size_t)(w < n_heads ? w : n_heads - 1) * kStatQPitch + lane;
  const int q_dst2 = ((w + NW < n_heads ? w + NW : n_heads - 1) - (w < n_heads ? w : n_heads - 1)) * kStatQPitch;  // PPL 2: the second head
  struct Query {
    double turns;
    float fr, cs, sn;
  };
  auto query_reduce = [&](Query& qr) { qr.fr = (float)(qr.turns - rint(qr.turns)); };
  auto query_angle = [&](Query& qr) {
    qr.cs = __builtin_amdgcn_cosf(qr.fr);
    qr.sn = __builtin_amdgcn_sinf(qr.fr);
  };
  auto query_store = [&](const Query& qr, auto pb_c) {
    constexpr int PB = decltype(pb_c)::value;
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
      f16x2 v;
      v[0] = static_cast<_Float16>(qx[u] * qr.cs - qy[u] * qr.sn);
      v[1] = static_cast<_Float16>(qy[u] * qr.cs + qx[u] * qr.sn);
      q_dst[PB * kStatMaxHeads * kStatQPitch + (u ? q_dst2 : 0)] = __builtin_bit_cast(uint32_t, v);
    }
  };
  // Scores of a position block against the group's heads, in steps that the stream puts apart (a step only consumes what
  // an earlier one requested or issued).  Rows of the A operand = heads; rows past G repeat the first head, their
  // results are never read.  k order of both operands: (x, y) pairs of the rows 8 s + 4 hf + 0 .. 3.
  struct ScoreOps {
    f16x8 q[2];
  };
  const uint32_t* q_src = qrot + (size_t)(kvh * G + (l32 < G ? l32 : 0)) * kStatQPitch + 16 * wq + 4 * hf;
  auto score_load = [&](ScoreOps& so, auto pb_c) {
    constexpr int PB = decltype(pb_c)::value;
    const uint32_t* src = q_src + PB * kStatMaxHeads * kStatQPitch;
    so.q[0] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(src));
    so.q[1] = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(src + 8));
  };
  // rows 4 hf + j (j < 4) of the score block are heads of the group (or rows past G: filed, not read); this wave holds a
  // quarter of the head-dim sum.  [quarter][KV head][8 rows][64 positions]
  float* s_dst = sbuf + (size_t)((wq * 2 + kvh) * 8 + 4 * hf) * T + l32;
  auto score_store = [&](const f32x16& sa, auto pb_c) {
    constexpr int PB = decltype(pb_c)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j) s_dst[j * T + PB * 32] = sa[j];
  };

  // ---- softmax of one tile over the workgroup's heads, in stages that the rebuild stream spreads over consecutive
  // k-steps (each stage only consumes what the one before requested): 64 / PPL lanes per head, PPL positions per lane; waves
  // past the workgroup's last head repeat it (same values to the same words).  The reference is the tile's own maximum (its
  // largest weight is then 1, which bf16 holds exactly), but at most 2^kBelow below the largest so far.  A reference that only moves
  // up by large steps leaves the largest weights rounded and costs the outputs 10 to 20 % of error against fp64 (8 x 4096 positions of the 8B shape at
  // rank 512: 2.39e-3, 1.97e-3 with the tile's own).  The sum is of the weights in fp32 and stays per lane until the end.
  const int sm_h_raw = PPL == 1 ? w : 2 * w + hf;
  const int sm_h = sm_h_raw < n_heads ? sm_h_raw : n_heads - 1;
  const int sm_pos = PPL == 1 ? lane : 2 * l32;
  const float* s_src = sbuf + (size_t)(sm_h < G ? sm_h : 8 + sm_h - G) * T + sm_pos;
  // P operand of the 16x16x32 product: position 32 ph + 8 kg + e of head h sits in lane h + 16 kg, element e
  uint16_t* p_dst = pbuf + ((size_t)((sm_pos >> 5) * 64 + sm_h + 16 * ((sm_pos & 31) >> 3)) * 8 + (sm_pos & 7));
  float m_run = kNegInfS, m_high = kNegInfS, l_run = 0.f;  // of head sm_h: reference, largest score, and this lane's share of the sum
  struct Softmax {
    float a[4][PPL], s[PPL], mx, pv[PPL], al;
  };
  auto softmax_a = [&](Softmax& sm) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int i = 0; i < PPL; ++i) sm.a[q][i] = s_src[q * kStatMaxHeads * T + i];
    }
  };
  // fill: what a position counts as whose page is not cached (zero latents: score 0), or of the tile before the first (none)
  auto softmax_b1 = [&](Softmax& sm, int valid_, bool page_ok_, float fill) {
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      sm.s[i] = page_ok_ ? (sm.a[0][i] + sm.a[1][i]) + (sm.a[2][i] + sm.a[3][i]) : fill;
      if (valid_ < T && sm_pos + i >= valid_) sm.s[i] = kNegInfS;
      sm.mx = i == 0 ? sm.s[0] : fmaxf(sm.mx, sm.s[i]);
    }
  };
  auto softmax_b2 = [&](Softmax& sm) {
    sm.mx = row_max_step<0>(sm.mx);
    sm.mx = row_max_step<1>(sm.mx);
  };
  auto softmax_b3 = [&](Softmax& sm) {
    sm.mx = row_max_step<2>(sm.mx);
    sm.mx = row_max_step<3>(sm.mx);
  };
  auto softmax_b4 = [&](Softmax& sm) {
    const float2 rows = row_pair(sm.mx);
    sm.mx = fmaxf(rows.x, rows.y);
    if constexpr (PPL == 1) {
      const float2 halves = half_pair(sm.mx);
      sm.mx = fmaxf(halves.x, halves.y);
    }
  };
  auto softmax_c = [&](Softmax& sm) {
    m_high = fmaxf(m_high, sm.mx);
    const float m_new = fmaxf(sm.mx, m_high - kBelow);
    const float m_ref = fmaxf(m_new, -1e30f);
#pragma unroll
    for (int i = 0; i < PPL; ++i) sm.pv[i] = __builtin_amdgcn_exp2f(sm.s[i] - m_ref);
    sm.al = __builtin_amdgcn_exp2f(m_run - m_ref);  // (0 while there is no reference: nothing to scale)
    m_run = m_new;
  };
  auto softmax_d = [&](const Softmax& sm, bool page_ok_) {
    alpha[sm_h] = sm.al;  // all lanes of a head hold the same value and store it to the same word (no branch in the stream)
    // A page that is not cached counts in the sums (zero keys) but adds nothing to o_lat (zero values): its P is filed as zero, and
    // whatever finite data the V tile holds is multiplied by it.
    uint32_t bits[PPL];
    l_run *= sm.al;
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      bits[i] = bf16_bits(sm.pv[i]);
      l_run += sm.pv[i];
    }
    if constexpr (PPL == 1) *p_dst = page_ok_ ? (uint16_t)bits[0] : (uint16_t)0;
    else *reinterpret_cast<uint32_t*>(p_dst) = page_ok_ ? bits[0] | (bits[PPL - 1] << 16) : 0u;
  };

  // ---- o_lat = alpha o_lat + P C_v of one tile: wave w owns the 16-wide latent blocks w, w + 8, ...
  struct PV {
    f32x4s al;
    bf16x8 pa0, pa1;
    u32x4 v0[NB], v1[NB];
  };
  auto pv_prep = [&](PV& pv) {
    pv.al = *reinterpret_cast<const f32x4s*>(alpha + 4 * (my_lane() >> 4));
    pv.pa0 = load_frag(kl + (pbuf - reinterpret_cast<const uint16_t*>(kbuf)));
    pv.pa1 = load_frag(kl + (pbuf - reinterpret_cast<const uint16_t*>(kbuf)) + 64 * 8);
  };
  // (unconditional: a branch around the four products would cost the LDS operations in flight at its join)
  auto pv_rescale = [&](const PV& pv, auto i_c) { o[decltype(i_c)::value] *= pv.al; };
  // V operand of block I (positions 32 ph + 8 kg .. + 7, latent 16 jb + n16, jb = w + 8 I) out of the page tiling of the V
  // tile; blocks past r_v read the padding
  const unsigned char* v_src = vbuf + (size_t)((((w >> 1) * 4 + (lane >> 5)) * 64 + 16 * (w & 1) + (lane & 15) + 32 * ((lane >> 4) & 1)) * 16);
  auto pv_load = [&](PV& pv, auto i_c) {
    constexpr int I = decltype(i_c)::value;
    pv.v0[I] = *reinterpret_cast<const u32x4*>(v_src + I * NW * 2048);
    pv.v1[I] = *reinterpret_cast<const u32x4*>(v_src + I * NW * 2048 + 2 * 1024);
  };
  // inside the stream: whole tiles only (a ragged tile is the last of its split and is finished after the loop), a
  // block past r_v multiplies the padding into an accumulator that is never written out
  auto pv_mfma_plain = [&](const PV& pv, auto i_c) {
    constexpr int I = decltype(i_c)::value;
    o[I] = mfma16(pv.pa0, __builtin_bit_cast(bf16x8, pv.v0[I]), o[I]);
    o[I] = mfma16(pv.pa1, __builtin_bit_cast(bf16x8, pv.v1[I]), o[I]);
  };
  auto pv_mfma = [&](PV& pv, auto i_c, int valid_, bool page_ok_) {
    constexpr int I = decltype(i_c)::value;
    const int jb = w + NW * I;
    if (jb * 16 < r_v) {
      if (!page_ok_ || valid_ < T) {  // wave-uniform: slots past the context (or a page that is not cached) hold anything
        const int kg = my_lane() >> 4;
#pragma unroll
        for (int ph = 0; ph < 2; ++ph) {
          int nv = valid_ - 32 * ph - 8 * kg;
          nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
          const uint32_t vmask = page_ok_ ? (1u << nv) - 1u : 0u;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const uint32_t two = (vmask >> (2 * c)) & 3u;
            const uint32_t keep = (two & 1u ? 0x0000ffffu : 0u) | (two & 2u ? 0xffff0000u : 0u);
            if (ph == 0) pv.v0[I][c] &= keep;
            else pv.v1[I][c] &= keep;
          }
        }
      }
      o[I] = mfma16(pv.pa0, __builtin_bit_cast(bf16x8, pv.v0[I]), o[I]);
      o[I] = mfma16(pv.pa1, __builtin_bit_cast(bf16x8, pv.v1[I]), o[I]);
    }
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I8 = std::integral_constant<int, 8>;
  // Schedule of a tile's stream (k-step indices; the copies have their own table).  Besides its own rebuild, the
  // stream of tile t carries the rest of tile t - 1 (rotation and scores of its second position block, its softmax,
  // its P C_v product) and the queries, rotation and scores of tile t's first position block, each placed where its inputs
  // are certainly there.  Barriers: kB1 / kB2 / kB3 = chunk 1 / 2 / 3 of the tile has landed (D steps before its first
  // k-step, where its first operand is requested), kB4 = chunk 2 is free, kB0 = the next tile's chunk 0 has landed
  // and every wave is through this tile's reads of chunk 3 and of the V tile.
  constexpr int kRotPer = (16 + H - 1) / H;                // rows rotated per k-step
  constexpr int kRotSteps = 8 / kRotPer;                   // k-steps one block's rotation takes
  constexpr int kIdRead = 2, kIdUse = 4;                   // page id of the tile after the next: LDS read, then its use
  // rotation and scores of a block: rotation from two steps after the block's last product on, query operands, products,
  // results filed.  This tile's first block waits with its scores until the previous tile's P C_v is through (registers; and
  // the softmax of the previous tile has read its scores then).
  constexpr int kRot1 = 2, kSc1 = kRot1 + kRotSteps, kRot0 = 2 * H + 2, kSc0 = kB0 - 2;
  constexpr int kQuery = kB1 - 2;                          // this tile's queries: nine stages, the fifth and the last file them
  auto sm_at = [](int stage) constexpr { return kB2 + (stage * (H - 1)) / 6; };  // the seven softmax stages, between kB2 and kB3
  constexpr int kPvPrep = kB3, kPvFirst = kB3 + 1, kPvSpan = kB0 - 2 - kPvFirst;  // block I: operands at kPvFirst + I kPvSpan / NB, product two steps later
  static_assert(kSc1 + 4 < kB2 && kRot0 + kRotSteps <= kSc0 && kSc0 + 4 < NG && kSc1 - 2 < kB1, "stream schedule: scores");
  static_assert(kQuery + 4 > kB1 && kQuery + 8 < kB2 && kPvSpan >= NB && NG % (D + 1) == 0 && kIdUse < NG && sm_at(6) < kB3, "stream schedule");

  f32x16 acc[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[b][j] = 0.f;
  int valid_prev = 0;          // the tile before the first one: no positions, everything it contributes is zero
  bool page_ok_prev = false;
  float fill = kNegInfS;
  bf16x8 c[D + 1];                        // latent operands read ahead; carried from one tile's stream into the next

  // ---- what a tile before the first one would have left in flight: the first tile's K chunks, in the order and
  // at the places of the schedule (the waits of the first stream count copies exactly like those of any other)
  int id_prev = -1, id_cur = -1, id_next = tile_id(0);
  {
    const u32x4 none = k_rsrc(-1), kr0 = k_rsrc(id_next);
    static_for<kB0 - kB2>([&](auto d_c) { issue_step(std::integral_constant<int, kB2 + decltype(d_c)::value>{}, none, kr0, none, none); });
    // While the first chunks travel: the factor operands, the queries, the rotation constants.  Their loads are
    // younger than the copies, so the wait below covers both, once.
    // stationary factor operands: row m of the operand is column 16 wq + m (m < 16) or its RoPE partner (+ 64 - 16)
    {
      const int g = 2 * hp + kvh;
      const int col = 16 * wq + l32 + (l32 < 16 ? 0 : HALF - 16);
      const uint32_t lane_off = (uint32_t)((col >> 5) * nks * 64 + (col & 31) + 32 * hf) * 16u;
      const __amdgpu_buffer_rsrc_t bk_rsrc = make_rsrc(p.bk, (uint32_t)p.h_kv * HD * r_k * 2u);
      const uint32_t s0 = (uint32_t)(g * 4 * nks) * 1024u;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks < nks) bk[ks] = buf_frag(bk_rsrc, lane_off, s0 + (uint32_t)ks * 1024u);
        else bk[ks] = zero_frag();
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float2 cs = p.lane_cs[l32 * HALF + 16 * wq + acc_row(j, hf)];
      rc[j] = cs.x;
      rs[j] = cs.y;
    }
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
      const int hl = w + NW * u < n_heads ? w + NW * u : n_heads - 1;
      const uint16_t* qsrc = p.q + ((size_t)seq * p.h_q + h0 + hl) * HD + lane;
      qx[u] = bf16_to_float(qsrc[0]) * p.q_scale;
      qy[u] = bf16_to_float(qsrc[HALF]) * p.q_scale;
    }
    if (tid < HALF) theta_rev_tab[tid] = p.rope_tab[tid] * 0.15915494309189533576888;
    for (int i = tid; i < 2 * kStatMaxHeads * kStatQPitch; i += NT) qrot[i] = 0u;  // read before the first tile's queries are there
    // Every load of the set-up has to be back here: a wait for one of them placed inside the tile loop would be a
    // wait for the latent copies issued after it (one in-order counter), on every tile.
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    static_for<NG - kB0>([&](auto d_c) {
      constexpr int gi = kB0 + decltype(d_c)::value;
      issue_step(std::integral_constant<int, gi>{}, none, kr0, none, none);
      c[(gi + D - NG) % (D + 1)] = load_frag(kl + (size_t)(gi + D - NG) * 512);
    });
  }
  id_cur = id_next;
  id_next = tile_id(1);

  for (int t = 0; t < nt; ++t) {
    const int pos0 = (tile_begin + t) * T;
    const int valid = (ctx - pos0) < T ? (ctx - pos0) : T;
    const bool page_ok = id_cur >= 0;
    const u32x4 kr_cur = k_rsrc(id_cur), kr_next = k_rsrc(id_next), v_prev = v_rsrc(id_prev), v_cur = v_rsrc(id_cur);
    int id_after_raw = -1, id_after = -1;

    f16x8 kf[2];
    ScoreOps so;
    f32x16 sa;
    Softmax sm;
    PV pv;
    double theta_rev = 0.0;
    Query qr0, qr1;
    static_for<NG>([&](auto gi_c) {
      constexpr int gi = decltype(gi_c)::value, nx = gi + D;
      // -- barriers and latent copies
      if constexpr (gi == kB0) dma_barrier<sched.younger(0, kB0)>();
      if constexpr (gi == kB1) dma_barrier<sched.younger(1, kB1)>();
      if constexpr (gi == kB2) dma_barrier<sched.younger(2, kB2)>();   // also: the previous tile's scores and this tile's queries are complete
      if constexpr (gi == kB3) dma_barrier<(sched.younger(3, kB3) < sched.younger(4, kB3) ? sched.younger(3, kB3) : sched.younger(4, kB3))>();  // also: its P is visible
      if constexpr (gi == kB4) lds_barrier();
      issue_step(gi_c, kr_cur, kr_next, v_prev, v_cur);
      // -- LDS read-ahead (past the end of the stream: the next tile's first k-steps) and the matrix-core op
      {
        constexpr int nxw = nx % NG, pbn = nxw / (2 * H), ksn = nxw % (2 * H);
        c[nx % (D + 1)] = load_frag(kl + (size_t)(pbn * NKS + ksn) * 512);
      }
      constexpr int pb = gi / (2 * H), ks = gi % (2 * H);
      acc[pb] = mfma32(bk[ks], c[gi % (D + 1)], ks == 0 ? zero16 : acc[pb]);
      // -- this tile's queries, rotated for its two position blocks
      if constexpr (gi == kQuery) theta_rev = theta_rev_tab[my_lane()];
      if constexpr (gi == kQuery + 1) qr0.turns = (double)(q_pos - pos0) * theta_rev;
      if constexpr (gi == kQuery + 2) query_reduce(qr0);
      if constexpr (gi == kQuery + 3) query_angle(qr0);
      if constexpr (gi == kQuery + 4) query_store(qr0, I0{});
      if constexpr (gi == kQuery + 5) qr1.turns = __builtin_fma(-32.0, theta_rev, qr0.turns);
      if constexpr (gi == kQuery + 6) query_reduce(qr1);
      if constexpr (gi == kQuery + 7) query_angle(qr1);
      if constexpr (gi == kQuery + 8) query_store(qr1, I1{});
      // -- page id of the tile after the next
      if constexpr (gi == kIdRead) id_after_raw = ids[t + 2 < nt ? t + 2 : 0];
      if constexpr (gi == kIdUse) id_after = t + 2 < nt ? __builtin_amdgcn_readfirstlane(id_after_raw) : -1;
      // -- rotation and scores: the previous tile's second position block, this tile's first
      static_for<2>([&](auto b_c) {
        constexpr int r = gi - (decltype(b_c)::value ? kRot0 : kRot1), sc = gi - (decltype(b_c)::value ? kSc0 : kSc1);
        using Blk = std::integral_constant<int, 1 - decltype(b_c)::value>;
        if constexpr (r >= 0 && r < kRotSteps)
          rotate_rows(acc[Blk::value], kf, std::integral_constant<int, r * kRotPer>{}, std::integral_constant<int, (r + 1) * kRotPer>{});
        if constexpr (sc == -2) score_load(so, Blk{});
        if constexpr (sc == 0) sa = mfma32_f16(so.q[0], kf[0], zero16);
        if constexpr (sc == 1) sa = mfma32_f16(so.q[1], kf[1], sa);
        if constexpr (sc == 4) score_store(sa, Blk{});
      });
      // -- the previous tile's softmax
      if constexpr (gi == sm_at(0)) softmax_a(sm);
      if constexpr (gi == sm_at(1)) softmax_b1(sm, T, page_ok_prev, fill);  // (a ragged tile is the last one: after the loop)
      if constexpr (gi == sm_at(2)) softmax_b2(sm);
      if constexpr (gi == sm_at(3)) softmax_b3(sm);
      if constexpr (gi == sm_at(4)) softmax_b4(sm);
      if constexpr (gi == sm_at(5)) softmax_c(sm);
      if constexpr (gi == sm_at(6)) softmax_d(sm, page_ok_prev);
      // -- the previous tile's P C_v
      if constexpr (gi == kPvPrep) pv_prep(pv);
      static_for<NB>([&](auto i_c) {
        constexpr int I = decltype(i_c)::value, at = kPvFirst + I * kPvSpan / NB;
        if constexpr (gi == at + 1) pv_rescale(pv, i_c);
        if constexpr (gi == at + 2) pv_mfma_plain(pv, i_c);
      });
      static_for<NB>([&](auto i_c) {
        constexpr int I = decltype(i_c)::value, at = kPvFirst + I * kPvSpan / NB;
        if constexpr (gi == at) pv_load(pv, i_c);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    valid_prev = valid;
    page_ok_prev = page_ok;
    fill = 0.f;
    asm volatile("" : "+s"(fill));  // (known from the second tile on: the compiler would peel the first, a second copy of the stream)
    id_prev = id_cur;
    id_cur = id_next;
    id_next = id_after;
  }

  // ---- the last tile's second half: the rest of its V tile, rotation and scores of position block 1, softmax,
  // P C_v (with the masks a ragged tile needs: only the last tile of a context can be one)
  if (nt > 0) {
    {
      const u32x4 vr = v_rsrc(id_prev);
      static_for<kB0>([&](auto gi_c) {  // the copies of the V tile that the schedule leaves to the next stream
        constexpr int gi = decltype(gi_c)::value;
        static_for<sched.MAXI>([&](auto i_c) {
          constexpr int i = decltype(i_c)::value;
          if constexpr (i < sched.n[gi]) {
            if constexpr (sched.kind[gi][i] == 4) issue_v_copy(vr, sched.idx[gi][i]);
          }
        });
      });
    }
    f16x8 kf[2];
    ScoreOps so;
    score_load(so, I1{});
    rotate_rows(acc[1], kf, I0{}, I8{});
    f32x16 sa = mfma32_f16(so.q[0], kf[0], zero16);
    sa = mfma32_f16(so.q[1], kf[1], sa);
    score_store(sa, I1{});
    lds_barrier();
    Softmax sm;
    PV pv;
    softmax_a(sm);
    softmax_b1(sm, valid_prev, page_ok_prev, 0.f);
    softmax_b2(sm);
    softmax_b3(sm);
    softmax_b4(sm);
    softmax_c(sm);
    softmax_d(sm, page_ok_prev);
    dma_barrier<0>();  // P and alpha visible; the V tile (and every other copy) has landed
    pv_prep(pv);
    static_for<NB>([&](auto i_c) {
      pv_rescale(pv, i_c);
      pv_load(pv, i_c);
    });
    static_for<NB>([&](auto i_c) { pv_mfma(pv, i_c, valid_prev, page_ok_prev); });
  }

  // ---- partials of this split (format of lorc_decode.hip): every copy still in flight has to land first, the
  // staging area reuses the K tile
  __builtin_amdgcn_s_waitcnt(0);
  {  // the lanes' shares of the sums
    l_run += half_wave_peer<0>(l_run);
    l_run += half_wave_peer<1>(l_run);
    l_run += half_wave_peer<2>(l_run);
    l_run += half_wave_peer<3>(l_run);
    const float2 rows = row_pair(l_run);
    l_run = rows.x + rows.y;
    if constexpr (PPL == 1) {
      const float2 halves = half_pair(l_run);
      l_run = halves.x + halves.y;
    }
  }
  m_fin[sm_h] = m_run;
  l_fin[sm_h] = l_run;
  __syncthreads();
  const size_t pbase = (size_t)seq * p.n_splits + split;
  if (tid < n_heads) {
    p.part_ml[(pbase * p.h_q + h0 + tid) * 2 + 0] = m_fin[tid];
    p.part_ml[(pbase * p.h_q + h0 + tid) * 2 + 1] = l_fin[tid];
  }
  const int pitch = r_v * 2 + 16;  // bytes per staged row
  {
    const int n16 = lane & 15, kg = lane >> 4;
    float inv_l[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float l = l_fin[4 * kg + j];
      inv_l[j] = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int jb = w + NW * i;
      if (jb * 16 < r_v) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<uint16_t*>(smem + (size_t)(4 * kg + j) * pitch + (jb * 16 + n16) * 2) = f16_bits(o[i][j] * inv_l[j]);
      }
    }
  }
  lds_barrier();
  uint16_t* dst_rows = p.part_o + (pbase * p.h_q + h0) * r_v;
  const int cpr = r_v >> 3, n_chunks = n_heads * cpr;  // 16-byte chunks
  for (int c = tid; c < n_chunks; c += NT) {
    const int h = c / cpr, cc = c - h * cpr;
    *reinterpret_cast<u32x4*>(dst_rows + (size_t)c * 8) = *reinterpret_cast<const u32x4*>(smem + (size_t)h * pitch + cc * 16);
  }
}

// The two names under which the kernel runs: ranks above 384, and the smaller ranks of what decode_split_kernel serves.
template <int NKS, int PPL>
__global__ __launch_bounds__(kStatThreads, 2) void decode_stationary_kernel(DecodeParams p) {
  stationary_split<NKS, PPL>(p);
}
template <int NKS, int PPL>
__global__ __launch_bounds__(kStatThreads, 2) void decode_split_kernel(DecodeParams p) {
  stationary_split<NKS, PPL>(p);
}

// ------------------------------------------------------------------------------------------------ host
// Shapes the kernel is built for.  Up to rank 128 the streaming kernel of lorc_decode.hip, which does not pad the rank to 256, is
// faster on large problems (8B shape, 32 x 8192 positions, us per layer-step, streaming / this: rank 64 160 / 182, 128 173 / 174,
// 192 201 / 190, 256 243 / 223, 320 273 / 243, 384 294 / 259; one sequence of 700 positions at rank 256 31.3 / 18.6, of 12000 at rank 384 58 / 29) and
// keeps those of up to 32 query heads; beyond 32 it would need two score blocks, and the other way is three launches (64 heads, 32 x 8192: rank
// 64 246 / 184, rank 384 405 / 277).
bool stationary_shape_ok(const lorc_layer_desc& d) {
  const int G = d.n_q_heads / d.n_kv_heads;
  return d.head_dim == 128 && d.n_kv_heads % 2 == 0 && G <= 8 && d.rank_k <= 16 * kStatMaxNks && d.rank_v <= 512 &&
         (d.rank_k > 128 || d.n_q_heads > 32);
}

// Rounds of workgroups over the eight XCDs (the head pairs of a (sequence, split) sit on one) x (tiles per workgroup + the fixed cost of
// a workgroup, about two tiles' worth: factor load, first tile, write-out).
static double stationary_cost(const lorc_layer_desc& d, int b, int n_splits, int tiles_per_split, int n_cus) {
  const long per_xcd = ((long)b * n_splits + 7) / 8 * (d.n_kv_heads / 2), xcd_cus = ((n_cus > 0 ? n_cus : 256) + 7) / 8;
  return (double)((per_xcd + xcd_cus - 1) / xcd_cus) * (tiles_per_split + 2.0);
}

double stationary_overhead(const lorc_layer_desc& d, int b, int max_ctx, const DecodePlan& pl, int n_cus, double* share) {
  const int n_tiles = max_ctx > 0 ? (max_ctx + kStatTile - 1) / kStatTile : 1;
  *share = (double)b * n_tiles * (d.n_kv_heads / 2) / (n_cus > 0 ? n_cus : 256);
  return stationary_cost(d, b, pl.n_splits, pl.tiles_per_split, n_cus) - *share;
}

DecodePlan make_stationary_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, int max_splits) {
  DecodePlan pl{};
  pl.tile = kStatTile;
  pl.occupancy = 1;
  pl.stationary = 1;
  int n_tiles = (max_ctx + kStatTile - 1) / kStatTile;
  if (n_tiles < 1) n_tiles = 1;
  // Context splits: the count of least cost.  Rounds are an XCD's: with 20 pairs two (sequences, splits) are 40 workgroups for 32 CUs,
  // three 60 for 64.  us per layer-step of 40 / 40 heads, rounds of the whole device / of an XCD: 4 x 4000 rank 256 113 / 71, rank 512
  // 165 / 107, rank 544 208 / 126; 2 x 1000 rank 384 38.7 / 29.1.
  int min_splits = (n_tiles + kStatMaxTiles - 1) / kStatMaxTiles;
  int best = min_splits;
  double best_cost = 0;
  if (max_splits > 64) max_splits = 64;  // the group merge's limit
  for (int ns = min_splits; ns <= n_tiles && (ns == min_splits || ns <= max_splits); ++ns) {
    const int tps = (n_tiles + ns - 1) / ns;
    const int ns_eff = (n_tiles + tps - 1) / tps;
    const double cost = stationary_cost(d, b, ns_eff, tps, n_cus);
    if (ns == min_splits || cost < best_cost * 0.999) {
      best = ns_eff;
      best_cost = cost;
    }
  }
  pl.tiles_per_split = (n_tiles + best - 1) / best;
  pl.n_splits = (n_tiles + pl.tiles_per_split - 1) / pl.tiles_per_split;
  size_t off = 0;
  pl.off_ml = off;
  off = ((off + (size_t)b * pl.n_splits * d.n_q_heads * 2 * 4) + 255) & ~(size_t)255;
  pl.off_o = off;
  off = ((off + (size_t)b * pl.n_splits * d.n_q_heads * d.rank_v * 2) + 255) & ~(size_t)255;
  pl.total_bytes = off;
  return pl;
}

namespace {
using StatKernel = void (*)(DecodeParams);
// k-steps the rank is padded to: 16 to 32 in steps of 4 (64 latent indices)
int stat_nks(int r_k) { return r_k <= 256 ? 16 : (r_k + 63) / 64 * 4; }
template <int PPL>
StatKernel stat_kernel(int nks_pad) {
  switch (nks_pad) {
    case 16: return decode_split_kernel<16, PPL>;
    case 20: return decode_split_kernel<20, PPL>;
    case 24: return decode_split_kernel<24, PPL>;
    case 28: return decode_stationary_kernel<28, PPL>;
    default: return decode_stationary_kernel<32, PPL>;
  }
}
}  // namespace

const char* stationary_kernel_symbol(const lorc_layer_desc& d) {
  const bool one = 2 * (d.n_q_heads / d.n_kv_heads) <= 8;
  switch (stat_nks(d.rank_k)) {
    case 16: return one ? "decode_split_kernel<16, 1>" : "decode_split_kernel<16, 2>";
    case 20: return one ? "decode_split_kernel<20, 1>" : "decode_split_kernel<20, 2>";
    case 24: return one ? "decode_split_kernel<24, 1>" : "decode_split_kernel<24, 2>";
    case 28: return one ? "decode_stationary_kernel<28, 1>" : "decode_stationary_kernel<28, 2>";
    default: return one ? "decode_stationary_kernel<32, 1>" : "decode_stationary_kernel<32, 2>";
  }
}

int set_kernel_attributes_decode_stationary() {
  for (int nks_pad = 16; nks_pad <= kStatMaxNks; nks_pad += 4)
    for (StatKernel k : {stat_kernel<1>(nks_pad), stat_kernel<2>(nks_pad)})
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
        return LORC_EHIP;
  return LORC_OK;
}

int launch_decode_stationary_split(const DecodeParams& p, const DecodePlan& plan, hipStream_t s) {
  const int nks_pad = stat_nks(p.r_k);
  const size_t lds = stat_lds_bytes(nks_pad, plan.tiles_per_split);
  if (lds > 160 * 1024 || plan.tiles_per_split > kStatMaxTiles || 2 * p.G > kStatMaxHeads || p.r_k > 16 * kStatMaxNks) return LORC_EUNSUPPORTED;
  const int units = p.b * p.n_splits, nq = p.h_kv / 2;
  const dim3 grid(((units + 7) / 8) * 8 * nq), block(kStatThreads);
  return launch_kernel(2 * p.G <= 8 ? stat_kernel<1>(nks_pad) : stat_kernel<2>(nks_pad), grid, block, lds, s, p);
}

}  // namespace lorc
