// Decode attention over the latent cache (Eq. 1 on cached latents; GQA of Section 4.3; RoPE applied at read
// time to the rebuilt keys, as the cache holds un-rotated latents).
//
// Two launches per call:
//   split    : one workgroup per (sequence, context split).  Per tile of T positions it copies the K latents
//              into LDS once, and for every KV head rebuilds K^T = B_k^T C_k^T on the matrix cores (B_k tiles
//              stream from L2, the latent tile is reused by all heads), rotates it in registers, takes
//              scores against the group's query heads, keeps an online softmax per head, and accumulates
//              o_lat += P C_v in latent space with the V latents loaded straight from the cache
//   merge    : combine the splits' (m, l, o_lat) and apply the value up-projection o = o_lat B_v
#include <type_traits>

#include <stdio.h>

#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_rebuild.h"

namespace lorc {

constexpr float kNegInf = -__builtin_huge_valf();

// N independent reductions over the 32 lanes of each wavefront half, walked step by step together so that their
// dependency chains overlap.
template <int N, class Op>
__device__ __forceinline__ void half_wave_reduce(float (&v)[N], Op op) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = op(v[i], half_wave_peer<0>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = op(v[i], half_wave_peer<1>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = op(v[i], half_wave_peer<2>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = op(v[i], half_wave_peer<3>(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) {  // the half's two rows
    const float2 rows = row_pair(v[i]);
    v[i] = op(rows.x, rows.y);
  }
}

__host__ __device__ inline size_t decode_lds_bytes(int T, int QB, int G, int r_k, int half) {
  size_t b = (size_t)T * r_k * 2;        // K latent tile
  b += (size_t)2 * G * T * 4;            // partner exchange of partial scores
  b += (size_t)QB * 32 * T * 2 + 128;    // P operands + one scrap element per lane
  b += (size_t)3 * QB * 32 * 4;          // alpha, running max, running sum
  b += (size_t)(T / 32) * half * 8;      // per-tile rotation bases
  b += (size_t)QB * 32 * half * 2 * 2;   // rotated, scaled queries of the sequence (fp16)
  return b;
}


// ------------------------------------------------------------------------------------------------ split
// JR = accumulator registers of a score block that can hold real query heads (rows 4*hf + j, j < JR <= 4
// covers G <= 8; JR = 16 covers G <= 32).
template <int HD, int NPB, int QB, int NBW, int JR, int OCC>
__global__ __launch_bounds__(256, OCC) void decode_split_kernel(DecodeParams p) {
  constexpr int T = 32 * NPB, HALF = HD / 2, KP = T / 16, PAGES = T / kPage;
  constexpr int PF = 4;  // B_k operand prefetch depth (k-steps)
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index as a scalar: keeps per-wave addresses in SGPRs
  const int seq = blockIdx.x / p.n_splits, split = blockIdx.x % p.n_splits;
  const int r_k = p.r_k, r_v = p.r_v, G = p.G, nks = r_k >> 4;
  auto my_tid = [&]() {
    int l = lane_id();
    asm volatile("" : "+v"(l));
    return l + (w << 6);
  };

  uint16_t* ck = reinterpret_cast<uint16_t*>(smem);
  float* xbuf = reinterpret_cast<float*>(smem + (size_t)T * r_k * 2);
  uint16_t* pbuf = reinterpret_cast<uint16_t*>(xbuf + 2 * G * T);
  float* alpha = reinterpret_cast<float*>(pbuf + QB * 32 * T + 64);  // 64 scrap elements follow the P operands
  float* m_run = alpha + QB * 32;
  float* l_run = m_run + QB * 32;
  float2* cs_base = reinterpret_cast<float2*>(l_run + QB * 32);
  _Float16* qrot = reinterpret_cast<_Float16*>(cs_base + NPB * HALF);  // [h_q][HD]
  // Everything the set-up needs from memory is requested here, before any of it is used, so that it costs one
  // round trip: the context length, the page ids of the split's first tile (speculatively: whether the tile
  // exists depends on the context length), the query position and this thread's share of the query rows, the
  // rotation tables.
  const int tile_begin = split * p.tiles_per_split;
  const int ctx_raw = p.ctx_len[seq];
  int ids0[PAGES];
#pragma unroll
  for (int pg = 0; pg < PAGES; ++pg) {
    const int pi = (tile_begin * T) / kPage + pg;
    ids0[pg] = pi < p.max_pages ? p.block_table[(size_t)seq * p.max_pages + pi] : -1;
  }
  const int q_pos = p.q_pos[seq];
  const double theta_t = p.rope_tab[tid % HALF];
  constexpr int QI = QB * 32 * HALF / 256;  // (head, frequency) pairs of the query per thread
  uint16_t q_lo[QI], q_hi[QI];
  {
    const uint16_t* qsrc = p.q + (size_t)seq * p.h_q * HD;
#pragma unroll
    for (int u = 0; u < QI; ++u) {
      const int idx = tid + 256 * u, h = idx / HALF, i = idx % HALF;
      const int hc = h < p.h_q ? h : p.h_q - 1;  // unconditional loads (rows past the last head repeat it, unused)
      q_lo[u] = qsrc[hc * HD + i];
      q_hi[u] = qsrc[hc * HD + i + HALF];
    }
  }
  // Per-lane rotation constants: (cos, sin)((lane % 32) * theta_i) for the 16 frequencies this lane's
  // accumulator rows carry.  The wave's half of the head (HD = 128) is fixed: task % 2 == wave % 2.
  const int fbase = HD == 128 ? 32 * (w & 1) : 0;
  float cl[16], sl[16];
#pragma unroll
  for (int jj = 0; jj < 16; ++jj) {
    const float2 t = p.lane_cs[l32 * HALF + fbase + acc_row(jj, hf)];
    cl[jj] = t.x;
    sl[jj] = t.y;
  }

  // All of the above has to be here before the first tile is requested: the tile's loads are counted in the same
  // in-order counter and their number is not known at compile time, so any later wait for one of the values
  // above would turn into a wait for the whole tile.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  int ctx = ctx_raw;
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  int tile_end = tile_begin + p.tiles_per_split;
  const int n_tiles = (ctx + T - 1) / T;
  if (tile_end > n_tiles) tile_end = n_tiles;

  // Pages of a tile (nullptr = not cached) and the copy of their K latents into LDS.  The copy is made of direct
  // global -> LDS loads, 1 KiB per instruction, the LDS image being the page's own tiling; it is issued while the
  // previous tile still has its softmax and P C_v phases to run, and waited for at the top of the tile.
  // Page ids of a tile are fetched one tile ahead (a vector load: its latency hides behind the tile's work) and
  // turned into pointers when the tile's K latents are requested.
  auto fetch_ids = [&](int tile_, int (&ids)[PAGES]) {
    const int valid_ = ctx - tile_ * T;
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg) {
      ids[pg] = -1;
      if (tile_ < tile_end && pg * kPage < valid_) ids[pg] = p.block_table[(size_t)seq * p.max_pages + (tile_ * T) / kPage + pg];
    }
  };
  auto ids_to_pages = [&](const int (&ids)[PAGES], const uint16_t* (&pp)[PAGES]) {
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg) {
      const int id = __builtin_amdgcn_readfirstlane(ids[pg]);
      pp[pg] = id >= 0 && id < p.n_pages ? p.cache + (size_t)id * p.page_elems : nullptr;
    }
  };
  // Waves blk0, blk0 + stride, ... of the issuing set each take every stride-th KiB block.
  auto issue_k_tile = [&](int tile_, const uint16_t* const (&pp)[PAGES], int blk0, int stride) {
    const int valid_ = ctx - tile_ * T;
    const int n_kib = r_k >> 3;  // 64 * r_k * 2 bytes per page / 1024
    int lo = lane_id(), zero = 0;  // recomputed / opaque: nothing derived from them is carried in registers
    asm volatile("" : "+v"(lo), "+v"(zero));
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg) {
      uint16_t* dst = ck + (size_t)pg * kPage * r_k;
      if (pp[pg] != nullptr) {
        const __amdgpu_buffer_rsrc_t pr = make_rsrc(pp[pg], (uint32_t)kPage * r_k * 2u);
        for (int blk = blk0; blk < n_kib; blk += stride)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(pr, (__attribute__((address_space(3))) void*)(dst + (size_t)blk * 512), 16, lo * 16,
                                                   blk * 1024, 0, 2);
      } else if (pg * kPage < valid_) {
        const u32x4 z = {(uint32_t)zero, (uint32_t)zero, (uint32_t)zero, (uint32_t)zero};
        for (int c = blk0 * 64 + lo; c < 8 * r_k; c += stride * 64) reinterpret_cast<u32x4*>(dst)[c] = z;
      }
    }
  };

  // One 1 KiB operand block of a page's V latents (used once: streamed past the caches).  For a page that is not
  // cached the load is still issued, through a descriptor of size zero: it fetches nothing and returns zeros; the
  // caller masks what it reads all the same.
  auto v_operand = [&](const uint16_t* page, int kib, int lane_) {
    const __amdgpu_buffer_rsrc_t vr = make_rsrc((page != nullptr ? page : p.cache) + (size_t)kPage * r_k, page != nullptr ? (uint32_t)kPage * r_v * 2u : 0u);
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vr, lane_ * 16, kib * 1024, 2));
  };

  // One-page tiles: the first tile's K latents are requested into registers right here (sixteen 1 KiB blocks per
  // wave, a fixed count; blocks past the rank and pages that are not cached come back as zeros without a fetch),
  // travel while the set-up below runs, and are written to LDS where the set-up's own LDS traffic is over.
  // Later tiles come by direct global -> LDS loads, which the set-up's LDS reads would have to wait for.
  constexpr int KST = PAGES == 1 ? 16 : 1;
  static_assert(PAGES != 1 || kStreamMaxRank / 8 <= 4 * 16 * 2, "blocks per page against the staging registers");
  const uint16_t* page_ptr[PAGES];
#pragma unroll
  for (int pg = 0; pg < PAGES; ++pg) page_ptr[pg] = nullptr;
  u32x4 kstage[KST];
  const bool stage_first = PAGES == 1 && (r_k >> 3) <= 4 * KST;  // every block of the page has a register
  if (stage_first && tile_begin < tile_end) {
    if (0 >= ctx - tile_begin * T) ids0[0] = -1;
    ids_to_pages(ids0, page_ptr);
    const __amdgpu_buffer_rsrc_t pr = make_rsrc(page_ptr[0] != nullptr ? page_ptr[0] : p.cache, page_ptr[0] != nullptr ? (uint32_t)kPage * r_k * 2u : 0u);
    int lo = lane_id();
    asm volatile("" : "+v"(lo));
#pragma unroll
    for (int u = 0; u < KST; ++u) kstage[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(pr, lo * 16, (w + 4 * u) * 1024, 2));
  }

  // Set-up work that needs the thread index comes before the first tile is requested, so that nothing derived
  // from it has to be kept (or reloaded, which would wait for the tile) across the request.
  const int tq = my_tid();
  if (tq < QB * 32) {
    alpha[tq] = 0.f;
    m_run[tq] = kNegInf;
    l_run[tq] = 0.f;
  }
  for (int i = tq; i < QB * 32 * T / 2; i += 256) reinterpret_cast<uint32_t*>(pbuf)[i] = 0u;
  // Queries of this sequence: rotated at q_pos, scaled (softmax scale x log2 e) and rounded to fp16 once, kept in
  // LDS; the score operands of every pass are gathered from there.  cs_base is free until the first tile.
  if (tq < HALF) {
    double a = (double)q_pos * theta_t;
    a -= kTwoPi * rint(a / kTwoPi);
    float sn, cs;
    sincosf((float)a, &sn, &cs);
    cs_base[tq] = make_float2(cs, sn);
  }
  int q_dst[QI], q_cs[QI];  // where this thread's query pairs go, and which rotation they take
  float q_lf[QI], q_hf[QI];  // the pairs, scaled (their first use is here, before the tile request, on purpose)
#pragma unroll
  for (int u = 0; u < QI; ++u) {
    const int idx = tq + 256 * u, h = idx / HALF, i = idx % HALF;
    q_dst[u] = h < p.h_q ? h * HD + i : -1;
    q_cs[u] = i;
    q_lf[u] = bf16_to_float(q_lo[u]) * p.q_scale;
    q_hf[u] = bf16_to_float(q_hi[u]) * p.q_scale;
    asm volatile("" : "+v"(q_lf[u]), "+v"(q_hf[u]));  // pins the computation (and its wait) here
  }

  lds_barrier();
#pragma unroll
  for (int u = 0; u < QI; ++u) {
    if (q_dst[u] >= 0) {
      const float2 cs = cs_base[q_cs[u]];
      qrot[q_dst[u]] = static_cast<_Float16>(q_lf[u] * cs.x - q_hf[u] * cs.y);
      qrot[q_dst[u] + HALF] = static_cast<_Float16>(q_hf[u] * cs.x + q_lf[u] * cs.y);
    }
  }
  lds_barrier();

  // First tile.  By direct-to-LDS loads it is requested only now: an LDS read that follows such a load in program
  // order waits for it (the compiler cannot tell the two apart), so the set-up's LDS traffic has to be over first.
  if (stage_first) {
    if (tile_begin < tile_end) {
      int lo = lane_id();
      asm volatile("" : "+v"(lo));
#pragma unroll
      for (int u = 0; u < KST; ++u)
        if (w + 4 * u < (r_k >> 3)) reinterpret_cast<u32x4*>(ck)[(size_t)(w + 4 * u) * 64 + lo] = kstage[u];
    }
  } else if (tile_begin < tile_end) {
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg)
      if (pg * kPage >= ctx - tile_begin * T) ids0[pg] = -1;  // page past the context: not part of the tile
    ids_to_pages(ids0, page_ptr);
    issue_k_tile(tile_begin, page_ptr, w, 4);
  }

  f32x16 o[QB][NBW];
#pragma unroll
  for (int a = 0; a < QB; ++a)
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[a][b][j] = 0.f;

  const int n_pass = (p.n_tasks + 3) >> 2;
  const __amdgpu_buffer_rsrc_t bk_rsrc = make_rsrc(p.bk, (uint32_t)p.h_kv * HD * r_k * 2u);

  for (int tile = tile_begin; tile < tile_end; ++tile) {
    const int pos0 = tile * T;
    const int valid = (ctx - pos0) < T ? (ctx - pos0) : T;
    const uint16_t* next_ptr[PAGES];
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg) next_ptr[pg] = nullptr;
    int next_ids[PAGES];
    fetch_ids(tile + 1, next_ids);

    // ---- 1. rotation bases of the tile; the tile's K latents (requested earlier) must have landed
    const int tt = my_tid();
    if (tt < NPB * HALF) {
      double a = (double)(pos0 + 32 * (tt / HALF)) * p.rope_tab[tt % HALF];
      a -= kTwoPi * rint(a / kTwoPi);
      float s, c;
      sincosf((float)a, &s, &c);
      cs_base[tt] = make_float2(c, s);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    lds_barrier();

    // The V operands of the first group of latent blocks and the next tile's K latents are requested as soon as
    // the last head has been rebuilt (the K tile in LDS is dead from then on), and arrive while the softmax and
    // the P C_v product of this tile run.
    constexpr int NG = NBW < 4 ? NBW : 4;
    u32x4 vraw0[NG][KP];
    auto request_ahead = [&]() {
      if (tile + 1 < tile_end) {
        ids_to_pages(next_ids, next_ptr);
        // HD = 128: the odd waves have no softmax to run, they issue the whole tile
        if (HD != 128) issue_k_tile(tile + 1, next_ptr, w, 4);
        else if (w & 1) issue_k_tile(tile + 1, next_ptr, w >> 1, 2);
      }
      int lo = lane_id();
      asm volatile("" : "+v"(lo));
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        const int nb = w + 4 * i;
        const int nbc = nb * 32 < r_v ? nb : w;  // clamp: blocks past r_v are loaded but never used
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) vraw0[i][kp] = v_operand(page_ptr[kp >> 2], nbc * 4 + (kp & 3), lo);
      }
    };

    // ---- 2. per KV head: rebuild K^T, rotate, score, softmax bookkeeping
    auto head_pass = [&](int ps, auto last_tag) {
      constexpr bool kLast = decltype(last_tag)::value;  // the tile's last pass: peeled, it starts the loads ahead
      const int task = ps * 4 + w;
      const bool active = task < p.n_tasks;
      const int g = HD == 128 ? task >> 1 : task;
      const int wh = HD == 128 ? task & 1 : 0;
      float sr[NPB][JR];  // scores of the real query-head rows

      if (active) {
        const int cb0 = HD == 128 ? g * 4 + wh : g * 2;
        const int cb1 = cb0 + (HD == 128 ? 2 : 1);

        f32x16 acc[2][NPB];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[a][pb][j] = 0.f;

        rebuild_pair<NPB, PF>(acc, bk_rsrc, (uint32_t)(cb0 * nks) * 1024u, (uint32_t)(cb1 * nks) * 1024u, (uint32_t)lane * 16u, ck + (size_t)lane * 8, nks);
        __builtin_amdgcn_sched_barrier(0);
        // rotate (pair = same register of the two accumulator blocks), round to fp16, score
        // Score A operands (m = query head of the group, k = 16 head-dim coordinates), in the order in which
        // the rotated K^T accumulators are re-used as B operands: element e of operand s4 is coordinate
        // 16*(s4 & 1) + 8*(e >> 2) + 4*hf + (e & 3) of half s4 >> 1 of the head (+ 32*wh for HD = 128).
        f16x8 qf[4];
        {
          const bool qreal = l32 < G;
          const _Float16* qh = qrot + (size_t)(g * G + (qreal ? l32 : 0)) * HD + (HD == 128 ? 32 * wh : 0) + 4 * hf;
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) {
            const _Float16* src = qh + HALF * (s4 >> 1) + 16 * (s4 & 1);
            const u32x2 lo = *reinterpret_cast<const u32x2*>(src), hi = *reinterpret_cast<const u32x2*>(src + 8);
            const u32x4 v = {qreal ? lo[0] : 0u, qreal ? lo[1] : 0u, qreal ? hi[0] : 0u, qreal ? hi[1] : 0u};
            qf[s4] = __builtin_bit_cast(f16x8, v);
          }
        }
#pragma unroll
        for (int pb = 0; pb < NPB; ++pb) {
          f16x8 kf[4];
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) {
            const float2 cb = cs_base[pb * HALF + fbase + acc_row(jj, hf)];
            const float cA = cb.x * cl[jj] - cb.y * sl[jj];
            const float sA = cb.y * cl[jj] + cb.x * sl[jj];
            const float x = acc[0][pb][jj], y = acc[1][pb][jj];
            kf[jj >> 3][jj & 7] = static_cast<_Float16>(x * cA - y * sA);
            kf[2 + (jj >> 3)][jj & 7] = static_cast<_Float16>(y * cA + x * sA);
          }
          f32x16 sa;
#pragma unroll
          for (int j = 0; j < 16; ++j) sa[j] = 0.f;
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) sa = mfma32_f16(qf[s4], kf[s4], sa);
#pragma unroll
          for (int jr = 0; jr < JR; ++jr) sr[pb][jr] = sa[jr];
          __builtin_amdgcn_sched_barrier(0);  // keep one position block in flight: bounds live registers
        }
      }
      if (HD == 128) {
        // the two waves of a head each hold half of the head-dim contraction
        float* xb = xbuf + (size_t)(w >> 1) * G * T;
        if (active && wh == 1) {
#pragma unroll
          for (int jr = 0; jr < JR; ++jr) {
            const int m = acc_row(jr, hf);
            if (m < G) {
#pragma unroll
              for (int pb = 0; pb < NPB; ++pb) xb[m * T + pb * 32 + l32] = sr[pb][jr];
            }
          }
        }
        __syncthreads();
        if constexpr (kLast) request_ahead();
        if (active && wh == 0) {
#pragma unroll
          for (int jr = 0; jr < JR; ++jr) {
            const int m = acc_row(jr, hf);
            if (m < G) {
#pragma unroll
              for (int pb = 0; pb < NPB; ++pb) sr[pb][jr] += xb[m * T + pb * 32 + l32];
            }
          }
        }
      }
      if (active && wh == 0) {
        // Online softmax for the JR head rows this lane may hold; the rows are walked together so that their
        // cross-lane reductions (independent dependency chains) overlap instead of running back to back.
        // Lanes whose register is not a query head of the group do the same arithmetic on harmless values and
        // store to a scrap slot: no per-row branches.  The lane index is recomputed here, so that the LDS addresses
        // below are rebuilt on the spot instead of being carried (spilled) across the rebuild loop.
        int lid = lane_id();
        asm volatile("" : "+v"(lid));
        const int lq = lid & 31, hq = lid >> 5;
        const int lane_t = (lq >> 4) * 512 + ((lq >> 3) & 1) * 256 + (lq & 7);  // position part of the P operand index
        float mx[JR], m_old[JR], sum[JR];
        int hterm[JR];
        bool real[JR];
#pragma unroll
        for (int jr = 0; jr < JR; ++jr) {
          const int row = 8 * (jr >> 2) + 4 * hq + (jr & 3);
          real[jr] = row < G;
          const int h = real[jr] ? g * G + row : 0;
          hterm[jr] = (h >> 5) * (KP * 512) + (h & 31) * 8 + lane_t;
          mx[jr] = kNegInf;
#pragma unroll
          for (int pb = 0; pb < NPB; ++pb) {
            if (pb * 32 + lq >= valid) sr[pb][jr] = kNegInf;
            mx[jr] = fmaxf(mx[jr], sr[pb][jr]);
          }
          const float mo = m_run[h];
          m_old[jr] = real[jr] ? mo : 0.f;
        }
        half_wave_reduce<JR>(mx, [](float x, float y) { return fmaxf(x, y); });
        const int scrap = QB * 32 * T + (hq * 32 + lq);  // past the P operands: one element per lane
#pragma unroll
        for (int jr = 0; jr < JR; ++jr) {
          const float m_new = fmaxf(m_old[jr], mx[jr]);
          mx[jr] = m_new;
          sum[jr] = 0.f;
#pragma unroll
          for (int pb = 0; pb < NPB; ++pb) {
            const float pv = __builtin_amdgcn_exp2f(sr[pb][jr] - m_new);  // arguments <= 0: no range fix-up needed
            sum[jr] += pv;
            pbuf[real[jr] ? hterm[jr] + pb * 1024 : scrap] = bf16_bits(pv);
          }
        }
        half_wave_reduce<JR>(sum, [](float x, float y) { return x + y; });
        // lane jr of each half files the running state of register jr's row
        float s_new = mx[0], s_old = m_old[0], s_sum = sum[0];
#pragma unroll
        for (int jr = 1; jr < JR; ++jr) {
          s_new = lq == jr ? mx[jr] : s_new;
          s_old = lq == jr ? m_old[jr] : s_old;
          s_sum = lq == jr ? sum[jr] : s_sum;
        }
        const int srow = 8 * (lq >> 2) + 4 * hq + (lq & 3);
        if (lq < JR && srow < G) {
          const int h = g * G + srow;
          const float a = __builtin_amdgcn_exp2f(s_old - s_new);
          m_run[h] = s_new;
          l_run[h] = l_run[h] * a + s_sum;
          alpha[h] = a;
        }
      }
      if (HD == 128) lds_barrier();
    };
    for (int ps = 0; ps + 1 < n_pass; ++ps) head_pass(ps, std::false_type{});
    head_pass(n_pass - 1, std::true_type{});
    lds_barrier();
    if (HD != 128) request_ahead();  // no barrier inside the passes: only here is the K tile known to be dead

    // ---- 3. o_lat = alpha * o_lat + P C_v : wave w owns latent blocks w, w+4, ... of the V latent
    {
      float al[QB][16];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) al[qb][jj] = alpha[qb * 32 + acc_row(jj, hf)];
      // Slots past the context hold whatever the pool held before: P is zero there, but 0 * NaN is not,
      // so the V operand is masked.  vmask[kp] = bit e set when position kp*16 + 8*hf + e is cached.
      // Loads are unconditional (for a page that is not cached they return zeros and are fully masked) so that
      // all of a block's operands are in flight together.
      uint32_t vmask[KP];
#pragma unroll
      for (int kp = 0; kp < KP; ++kp) {
        int nv = valid - kp * 16 - 8 * hf;
        nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
        vmask[kp] = page_ptr[kp >> 2] != nullptr ? (1u << nv) - 1u : 0u;
      }
      // The V operands of up to four latent blocks (all positions of the tile) are requested before any is
      // used: the loads are the only HBM traffic of this phase and need that much in flight to stream.  The
      // first group was requested ahead.
#pragma unroll
      for (int n0 = 0; n0 < NBW; n0 += NG) {
        u32x4 vraw[NG][KP];
#pragma unroll
        for (int i = 0; i < NG; ++i) {
          const int nb = w + 4 * (n0 + i);
          const int nbc = nb * 32 < r_v ? nb : w;  // clamp: blocks past r_v are loaded but never used
#pragma unroll
          for (int kp = 0; kp < KP; ++kp) {
            if (n0 == 0) {
              vraw[i][kp] = vraw0[i][kp];
            } else {
              vraw[i][kp] = v_operand(page_ptr[kp >> 2], nbc * 4 + (kp & 3), lane);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
          const int nbw = n0 + i;
          const int nb = w + 4 * nbw;
          if (nb * 32 < r_v) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
              for (int jj = 0; jj < 16; ++jj) o[qb][nbw][jj] *= al[qb][jj];
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) {
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const uint32_t two = (vmask[kp] >> (2 * c)) & 3u;
                vraw[i][kp][c] &= (two & 1u ? 0x0000ffffu : 0u) | (two & 2u ? 0xffff0000u : 0u);
              }
              const bf16x8 vb = __builtin_bit_cast(bf16x8, vraw[i][kp]);
#pragma unroll
              for (int qb = 0; qb < QB; ++qb) {
                const bf16x8 pa = load_frag(pbuf + ((size_t)(qb * KP + kp) * 64 + lane) * 8);
                o[qb][nbw] = mfma32(pa, vb, o[qb][nbw]);
              }
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier();
#pragma unroll
    for (int pg = 0; pg < PAGES; ++pg) page_ptr[pg] = next_ptr[pg];
  }

  // ---- partials of this split
  const size_t pbase = (size_t)seq * p.n_splits + split;
  __syncthreads();
  const int te = my_tid();
  if (te < p.h_q) {
    p.part_ml[(pbase * p.h_q + te) * 2 + 0] = m_run[te];
    p.part_ml[(pbase * p.h_q + te) * 2 + 1] = l_run[te];
  }
  // The split's latent-space output is stored normalised by its own sum (so that it is bounded by the value
  // latents and fits fp16, half the bytes of fp32); always written (zeros for a split past the context) so that
  // the merge can read without guards.  The workgroup's rows [h_q][r_v] are one contiguous range of the
  // workspace: when they fit into the (now dead) K tile they are staged there and written as whole 16-byte
  // chunks, a full row per wave and store, instead of as two-byte elements.
  const int pitch = r_v * 2 + 16;  // bytes; the +16 puts the two half-wave rows of an accumulator on different banks
  const bool staged = (size_t)QB * 32 * pitch <= (size_t)T * r_k * 2;
  unsigned char* stage = smem;
  uint16_t* dst_rows = p.part_o + pbase * p.h_q * r_v;
  float inv_l[QB][16];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const float l = l_run[qb * 32 + acc_row(jj, hf)];
      inv_l[qb][jj] = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
    }
  if (staged) {  // one branch around the whole write-out: the element loops below are straight-line code
    unsigned char* lane_base = stage + (size_t)(4 * hf) * pitch + l32 * 2 + w * 64;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int nbw = 0; nbw < NBW; ++nbw) {
        if ((w + 4 * nbw) * 32 < r_v) {
#pragma unroll
          for (int jj = 0; jj < 16; ++jj)
            *reinterpret_cast<uint16_t*>(lane_base + (qb * 32 + 8 * (jj >> 2) + (jj & 3)) * pitch + nbw * 256) =
                f16_bits(o[qb][nbw][jj] * inv_l[qb][jj]);
        }
      }
    lds_barrier();
    const int cpr = r_v >> 3;  // 16-byte chunks per row
    const int n_chunks = p.h_q * cpr;
    for (int c = te; c < n_chunks; c += 256) {
      const int h = c / cpr, cc = c - h * cpr;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stage + (size_t)h * pitch + cc * 16);
      *reinterpret_cast<u32x4*>(dst_rows + (size_t)c * 8) = v;
    }
  } else {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int nbw = 0; nbw < NBW; ++nbw) {
        const int nb = w + 4 * nbw;
        if (nb * 32 < r_v) {
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) {
            const int h = qb * 32 + acc_row(jj, hf);
            if (h < p.h_q) dst_rows[(size_t)h * r_v + nb * 32 + l32] = f16_bits(o[qb][nbw][jj] * inv_l[qb][jj]);
          }
        }
      }
  }
}

// ------------------------------------------------------------------------------------------------ merge
// One workgroup per (sequence, query head): softmax-merge the splits' (m, l, o_lat), then the value
// up-projection o = o_lat B_v^g with the 256 threads laid out as head_dim columns x latent slices.
constexpr int kMaxSplits = 512;

template <int HD>
__global__ __launch_bounds__(256) void decode_merge_kernel(DecodeParams p) {
  constexpr int NS = 256 / HD;  // latent slices reduced through LDS
  __shared__ float olat[kWideMaxRank];
  __shared__ float wgt[kMaxSplits];
  __shared__ float red[NS][HD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int seq = blockIdx.x / p.h_q, h = blockIdx.x % p.h_q, g = h / p.G;
  const int r_v = p.r_v, ns = p.n_splits;
  if (tid < 64) {  // first wave: weights of the splits
    const float* ml = p.part_ml + ((size_t)seq * ns * p.h_q + h) * 2;
    const size_t st = (size_t)p.h_q * 2;
    float M = kNegInf;
    for (int s = lane; s < ns; s += 64) M = fmaxf(M, ml[s * st]);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
    float L = 0.f;
    for (int s = lane; s < ns; s += 64) {
      const float ms = ml[s * st];
      const float e = (ms == kNegInf ? 0.f : exp2f(ms - M)) * ml[s * st + 1];  // partials are stored normalised
      L += e;
      wgt[s] = e;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) L += __shfl_xor(L, off);
    const float invL = L > 0.f ? 1.f / L : (M == kNoWeight ? __builtin_nanf("") : 0.f);
    for (int s = lane; s < ns; s += 64) wgt[s] *= invL;
  }
  __syncthreads();
  {
    const uint16_t* po = p.part_o + ((size_t)seq * ns * p.h_q + h) * r_v;
    const size_t st = (size_t)p.h_q * r_v;
    for (int j = tid; j < r_v; j += 256) {
      float a = 0.f;
      int s = 0;
      for (; s + 8 <= ns; s += 8) {
        uint16_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = po[(size_t)(s + u) * st + j];
#pragma unroll
        for (int u = 0; u < 8; ++u) a += wgt[s + u] * (float)__builtin_bit_cast(_Float16, v[u]);
      }
      for (; s < ns; ++s) a += wgt[s] * (float)__builtin_bit_cast(_Float16, po[(size_t)s * st + j]);
      olat[j] = a;
    }
  }
  __syncthreads();
  if (p.latent_out) {  // o_lat / l itself is the result: the caller applies B_v (or a matrix that absorbed it)
    for (int j = tid; j < r_v; j += 256) p.out[((size_t)seq * p.h_q + h) * r_v + j] = bf16_bits(olat[j]);
    return;
  }
  const int c = tid % HD, sl = tid / HD;
  const int cg = g * HD + c;
  const int per = ((r_v / 8 + NS - 1) / NS) * 8;  // latent indices per slice (multiple of 8)
  const int j_begin = sl * per, j_end = (j_begin + per) < r_v ? (j_begin + per) : r_v;
  float acc = 0.f;
  int j = j_begin;
  for (; j + 32 <= j_end; j += 32) {
    bf16x8 bv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) bv[u] = load_frag(p.bv + b_tile_index(r_v, j + 8 * u, cg));
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc += olat[j + 8 * u + e] * (float)bv[u][e];
  }
  for (; j < j_end; j += 8) {
    const bf16x8 bv = load_frag(p.bv + b_tile_index(r_v, j, cg));
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += olat[j + e] * (float)bv[e];
  }
  red[sl][c] = acc;
  __syncthreads();
  if (tid < HD) {
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) v += red[i][tid];
    p.out[((size_t)seq * p.h_q + h) * HD + tid] = bf16_bits(v);
  }
}

// ------------------------------------------------------------------------------------------------ merge, common shapes
// One workgroup of sixteen waves per (sequence, KV head): the G query heads of the group share the factor block
// B_v^g, which is read once, as matrix-core operands.  The split partials are requested first (eight fp16 columns per thread; up
// to eight sets of threads share the splits), then the factor operands; the split weights are worked out while both travel.
// The up-projection runs on the matrix cores with o_lat split into bf16 terms: a head and a remainder up to rank 512 (16 bits), above a
// third one, with which they hold all 24 bits of the fp32 sum, as the scalar products of decode_merge_kernel take it.
// Shapes: G <= 8, at most 64 splits, r_v <= 1024.  Bound by latency: launch, one round trip
// for both operands, the product's chain.  Value ranks above 512 before, a workgroup per query head and scalar products: 14.5 us
// for one sequence at rank 768, whole call 36.5 -> 25.2; 1 x 1337 at rank 512 (four columns per thread, all splits in one): 23.0 -> 22.1.
constexpr int kMgMaxG = 8, kMgMaxSplits = 64, kMgMaxRank = 1024, kMgMaxRankG1 = 2048;
// HS: workgroups that share a group's heads;  CS: workgroups that share the head's columns (each works out the weighted sums of its
// heads for itself);  MAXR: largest value rank;  MAXG: heads of a workgroup;  TERMS: bf16 terms of o_lat.
template <int HD, int HS, int CS, int MAXR, int MAXG = kMgMaxG / HS, int TERMS = (MAXR <= 512 ? 2 : 3)>
__global__ __launch_bounds__(1024 / HS) void decode_merge_group_kernel(DecodeParams p) {
  constexpr int NCB = HD / 32 / CS, NKQ = (16 / HS) / NCB, MAXKS = (MAXR / 16 + NKQ - 1) / NKQ;
  constexpr int PITCH = MAXR + 8, COLS = 32 * NCB;
  constexpr int BATCH = HS == 2 ? 16 : (MAXR == 1024 && CS == 1 ? 4 : 8);  // partials a thread has in flight (16 bytes each)
  __shared__ float wgt[MAXG][kMgMaxSplits];
  __shared__ __align__(16) uint16_t o_terms[TERMS][MAXG][PITCH];
  constexpr int SHARE = 512;               // threads that share the splits at most
  // Weighted sums of a thread's splits; later the parts of the product.  Three terms: their parts take three times the columns and meet
  // where the terms were.
  constexpr bool PACK = TERMS == 3;
  constexpr int RC = PACK ? 3 * MAXG : MAXG, PARTS = NKQ * COLS * RC;
  constexpr int SCRATCH = PACK || SHARE * 8 > PARTS ? SHARE * 8 : PARTS;
  static_assert(!PACK || (PARTS * 4 <= (int)sizeof(o_terms) && 3 * MAXG <= 32), "parts of the product; columns of an operand");
  __shared__ __align__(16) float scratch[SCRATCH];
  float (*const part)[8] = reinterpret_cast<float (*)[8]>(scratch);
  float (*const red)[COLS][RC] = reinterpret_cast<float (*)[COLS][RC]>(PACK ? reinterpret_cast<float*>(&o_terms[0][0][0]) : scratch);
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cs = blockIdx.x % CS, sg = blockIdx.x / (CS * HS), seq = sg / p.h_kv, g = sg % p.h_kv;
  const int G = p.G / HS, r_v = p.r_v, ns = p.n_splits, nks = r_v >> 4;  // G: heads of this workgroup
  const int h0 = g * p.G + (blockIdx.x / CS % HS) * G;                   // its first query head

  // ---- partials: 8 columns of a head per thread; as many sets of threads as there are share the splits
  const int per_set = G * (r_v >> 3), most = ns < 8 ? ns : 8;
  const int sets = per_set * most <= SHARE ? most : (2 * per_set <= SHARE ? SHARE / per_set : 1);
  const int set = tid / per_set, in_set = tid - set * per_set;
  const bool owner = set < sets;
  const int oh = owner ? in_set / (r_v >> 3) : 0, oj = owner ? (in_set % (r_v >> 3)) * 8 : 0;
  const uint16_t* po = p.part_o + (((size_t)seq * ns) * p.h_q + (size_t)h0 + oh) * r_v + oj;
  const size_t pst = (size_t)p.h_q * r_v;
  u32x4 pre[BATCH];
  auto load_batch = [&](int u0) {
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int s_ = set + (u0 + u) * sets;  // clamped: the tail is loaded again and weighted zero
      pre[u] = *reinterpret_cast<const u32x4*>(po + (size_t)(s_ < ns ? s_ : ns - 1) * pst);
    }
  };
  if (owner) load_batch(0);

  // ---- factor operands of this wave: column block cb of the head, k-steps [ks0, ks1)
  const int cb = cs * NCB + w % NCB, kq = w / NCB;
  const int ks_per = (nks + NKQ - 1) / NKQ;
  const int ks0 = kq * ks_per, ks1 = ks0 + ks_per < nks ? ks0 + ks_per : nks;
  bf16x8 bvf[MAXKS];
  if (!p.latent_out) {
    const uint16_t* bp = p.bv + ((size_t)(g * (HD / 32) + cb) * nks * 64 + lane) * 8;
#pragma unroll
    for (int u = 0; u < MAXKS; ++u) {
      const int ks = ks0 + u < nks ? ks0 + u : nks - 1;
      bvf[u] = load_frag(bp + (size_t)ks * 512);
    }
  }

  // ---- split weights: wave h < G handles head h, one split per lane
  if (w < G) {
    const int h = h0 + w;
    const float* ml = p.part_ml + (((size_t)seq * ns) * p.h_q + h) * 2;
    const size_t st = (size_t)p.h_q * 2;
    const float ms = lane < ns ? ml[lane * st] : kNegInf;
    const float ls = lane < ns ? ml[lane * st + 1] : 0.f;
    float M = ms;
    M = fmaxf(M, half_wave_peer<0>(M));
    M = fmaxf(M, half_wave_peer<1>(M));
    M = fmaxf(M, half_wave_peer<2>(M));
    M = fmaxf(M, half_wave_peer<3>(M));
    const float2 mr = row_pair(M);
    M = fmaxf(mr.x, mr.y);
    const float2 mh = half_pair(M);
    M = fmaxf(mh.x, mh.y);
    const float e = (ms == kNegInf ? 0.f : exp2f(ms - M)) * ls;  // partials are stored normalised
    float L = e;
    L += half_wave_peer<0>(L);
    L += half_wave_peer<1>(L);
    L += half_wave_peer<2>(L);
    L += half_wave_peer<3>(L);
    const float2 lr = row_pair(L);
    L = lr.x + lr.y;
    const float2 lh = half_pair(L);
    L = lh.x + lh.y;
    if (lane < ns) wgt[w][lane] = L > 0.f ? e / L : 0.f;
  }
  __syncthreads();

  // ---- o_lat = sum over splits of weight * partial
  float a[8];
  if (owner) {
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = 0.f;
    const int count = (ns - set + sets - 1) / sets;  // splits of this set
    for (int u0 = 0; u0 < count; u0 += BATCH) {
      if (u0 != 0) load_batch(u0);
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int s_ = set + (u0 + u) * sets;
        const float wv = s_ < ns ? wgt[oh][s_] : 0.f;
        typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_;
        const f16x8_ hv = __builtin_bit_cast(f16x8_, pre[u]);
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] += wv * (float)hv[i];
      }
    }
    if (sets > 1) {
      *reinterpret_cast<f32x4*>(&part[tid][0]) = f32x4{a[0], a[1], a[2], a[3]};
      *reinterpret_cast<f32x4*>(&part[tid][4]) = f32x4{a[4], a[5], a[6], a[7]};
    }
  }
  if (sets > 1) __syncthreads();
  if (set == 0) {
    for (int o_ = 1; o_ < sets; ++o_) {
      const f32x4 b0 = *reinterpret_cast<const f32x4*>(&part[tid + o_ * per_set][0]), b1 = *reinterpret_cast<const f32x4*>(&part[tid + o_ * per_set][4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] += b0[i];
        a[4 + i] += b1[i];
      }
    }
    uint32_t term[TERMS][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float x = a[2 * i], y = a[2 * i + 1];
#pragma unroll
      for (int k = 0; k < TERMS; ++k) {  // (every remainder is exact in fp32)
        const uint16_t bx = bf16_bits(x), by = bf16_bits(y);
        term[k][i] = (uint32_t)bx | ((uint32_t)by << 16);
        x -= bf16_to_float(bx);
        y -= bf16_to_float(by);
      }
    }
    if (p.latent_out) {
      *reinterpret_cast<u32x4*>(p.out + ((size_t)seq * p.h_q + (size_t)h0 + oh) * r_v + oj) = u32x4{term[0][0], term[0][1], term[0][2], term[0][3]};
    } else {
#pragma unroll
      for (int k = 0; k < TERMS; ++k) *reinterpret_cast<u32x4*>(&o_terms[k][oh][oj]) = u32x4{term[k][0], term[k][1], term[k][2], term[k][3]};
    }
  }
  if (p.latent_out) return;
  __syncthreads();

  // ---- out^T[c][h] = sum_j B_v[j][c] o_lat[h][j]: A operand = factor tile (m = column), B operand = o_lat^T.  Three terms are columns of
  // one operand (24 of 32 at most), two have a product and an accumulator each.
  f32x16 acc, acc_lo;
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = acc_lo[j] = 0.f;
  const int term = l32 < G ? 0 : (l32 < 2 * G ? 1 : 2), cols = PACK ? 3 * G : G;
  const uint16_t* const o_src = &o_terms[PACK && l32 < cols ? term : 0][PACK && l32 < cols ? l32 - term * G : (l32 < G ? l32 : 0)][8 * hf];
#pragma unroll
  for (int u = 0; u < MAXKS; ++u) {
    if (ks0 + u < ks1) {
      const int j0 = (ks0 + u) * 16;
      acc = mfma32(bvf[u], l32 < cols ? load_frag(o_src + j0) : zero_frag(), acc);
      if constexpr (!PACK) acc_lo = mfma32(bvf[u], l32 < G ? load_frag(o_src + MAXG * PITCH + j0) : zero_frag(), acc_lo);
    }
  }
  if constexpr (PACK) __syncthreads();
  if (l32 < cols) {
#pragma unroll
    for (int j = 0; j < 16; ++j) red[kq][(w % NCB) * 32 + acc_row(j, hf)][l32] = PACK ? acc[j] : acc[j] + acc_lo[j];
  }
  __syncthreads();
  if (tid < COLS * G) {
    const int c = tid % COLS, h = tid / COLS;
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < NKQ; ++i) {
      if constexpr (PACK) v += red[i][c][h] + (red[i][c][G + h] + red[i][c][2 * G + h]);
      else v += red[i][c][h];
    }
    p.out[((size_t)seq * p.h_q + (size_t)h0 + h) * HD + cs * COLS + c] = bf16_bits(v);
  }
}

// ------------------------------------------------------------------------------------------------ absorbed split
// Decode without positional rotation (Section 4.1, Eq. 7): the key factor is folded into the query, scores are
// taken in latent space, s[h][j] = q_lat[h] . c_K[j], and nothing is rebuilt.  32 flop per byte of latent: the
// kernel is a stream over the cache.  One workgroup per (sequence, context split), two per CU.  Every wave owns
// 16 of a tile's 64 positions for all heads (16x16x32 matrix-core products); a K operand block (16 positions x 32
// latent indices) is therefore used by exactly one wave and needs no staging in LDS: it goes from the cache
// straight into registers as the B operand, read out of the page's own tiling.  What sits in LDS is the absorbed
// query (A operands, tiled in operand order).  Softmax: row statistics inside the wave by DPP, one exchange of
// (max, sum) between the four waves through LDS, running statistics in LDS.  P C_v, the partials and the merge
// are those of the rotary path.  All loads are plain buffer loads of fixed count (also past the last tile, from a
// page nobody reads), so the compiler's partial waits are exact; 204 registers, no scratch.
constexpr int kAbsMaxRankK = 512;  // sixteen K operands per wave and tile, one register ring

__host__ __device__ inline size_t absorbed_lds_bytes(int r_k, int r_v) {
  const size_t qb = (size_t)32 * r_k * 2, st = (size_t)32 * (r_v * 2 + 16);
  return (qb > st ? qb : st) + (size_t)32 * kPage * 2 + 128 + (size_t)(2 * 32 * 4 + 32 + 32 + 32) * 4;
}

template <int NBW>
__global__ __launch_bounds__(256, 2) void decode_absorbed_kernel(DecodeParams p) {
  constexpr int T = kPage, KP = T / 16, NK32 = kAbsMaxRankK / 32;
  static_assert(NBW * KP == NK32, "K and V operands of a tile share one register ring");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31, n16 = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seq = blockIdx.x / p.n_splits, split = blockIdx.x % p.n_splits;
  const int r_k = p.r_k, r_v = p.r_v, nks = r_k >> 4, nk32 = r_k >> 5;
  const size_t qbytes = (size_t)32 * r_k * 2, stbytes = (size_t)32 * (r_v * 2 + 16);
  uint16_t* qlds = reinterpret_cast<uint16_t*>(smem);                           // [2 head blocks][nk32][64 lanes][8]
  uint16_t* pbuf = reinterpret_cast<uint16_t*>(smem + (qbytes > stbytes ? qbytes : stbytes));  // P operands (+ scrap)
  float* xm = reinterpret_cast<float*>(pbuf + 32 * T + 64);                     // [32 heads][4 waves] wave-local maxima
  float* xs = xm + 32 * 4;
  float* alpha = xs + 32 * 4;
  float* l_fin = alpha + 32;   // running sums (final after the last tile)
  float* m_fin = l_fin + 32;   // running maxima

  const int tile_begin = split * p.tiles_per_split;
  int ctx = __builtin_amdgcn_readfirstlane(p.ctx_len[seq]);
  ctx = ctx < 0 ? 0 : (ctx > p.max_ctx ? p.max_ctx : ctx);
  int tile_end = tile_begin + p.tiles_per_split;
  const int n_tiles = (ctx + T - 1) / T;
  if (tile_end > n_tiles) tile_end = n_tiles;

  // Set-up order: the page ids, the absorbed query and the first tile's K operands are three round trips to
  // memory; they are requested back to back (ids, query chunks into registers, then -- as soon as the ids are
  // back -- the K operands) and the query goes to LDS while the K operands travel.
  auto fetch_id = [&](int tile_) { return p.block_table[(size_t)seq * p.max_pages + (tile_ < p.max_pages ? tile_ : p.max_pages - 1)]; };
  const int id0 = fetch_id(tile_begin), id1 = fetch_id(tile_begin + 1);
  int id_nn = fetch_id(tile_begin + 2);
  // absorbed query: chunk c (8 latent indices) of head h goes to lane (h % 16) + 16 (c % 4) of operand
  // (h / 16, c / 4); heads past h_q are zero.  Unconditional loads of a fixed count (clamped, masked afterwards).
  constexpr int QCH = 32 * (kAbsMaxRankK / 8) / 256;
  const int cpr = r_k >> 3;
  u32x4 qv[QCH];
  {
    const uint16_t* qsrc = p.q + (size_t)seq * p.h_q * r_k;
#pragma unroll
    for (int u = 0; u < QCH; ++u) {
      const int c = tid + 256 * u < 32 * cpr ? tid + 256 * u : 32 * cpr - 1;
      const int h = c / cpr, cc = c - h * cpr;
      qv[u] = *reinterpret_cast<const u32x4*>(qsrc + (size_t)(h < p.h_q ? h : p.h_q - 1) * r_k + cc * 8);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if (tid < 32) {
    alpha[tid] = 0.f;
    l_fin[tid] = 0.f;
    m_fin[tid] = kNegInf;
  }
  // Page ids are fetched a tile before they are needed and turned into wave-uniform pointers then; nullptr = not
  // cached or past the split's last tile: the loads are still issued (their count stays fixed) through a
  // descriptor of size zero, so they fetch nothing and return zeros, and everything read is masked as well.
  auto to_page = [&](int id_raw, int tile_) -> const uint16_t* {
    const int id = __builtin_amdgcn_readfirstlane(id_raw);
    return tile_ < tile_end && id >= 0 && id < p.n_pages ? p.cache + (size_t)id * p.page_elems : nullptr;
  };
  // K operand (positions 16 w .. 16 w + 15 of the page, latent indices 32 ks .. 32 ks + 31) straight from the page
  // tiling: lane (n, kg) takes the 16 bytes of position n, indices 8 kg .. 8 kg + 7.
  const uint32_t k_lane = (uint32_t)((((w >> 1) * nks + (kg >> 1)) * 64 + (w & 1) * 16 + n16 + 32 * (kg & 1)) * 16);
  auto k_frag = [&](const uint16_t* page, int ks) {
    const __amdgpu_buffer_rsrc_t pr = make_rsrc(uniform_ptr(page != nullptr ? page : p.cache), page != nullptr ? (uint32_t)kPage * r_k * 2u : 0u);
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(pr, k_lane, (ks < nk32 ? ks : nk32 - 1) * 2048, 2));
  };
  auto v_frag = [&](const uint16_t* page, int idx) {  // V operand idx = 4 * (block slot i) + kp of this wave
    const __amdgpu_buffer_rsrc_t vr = make_rsrc(uniform_ptr(page != nullptr ? page : p.cache) + (size_t)kPage * r_k, page != nullptr ? (uint32_t)kPage * r_v * 2u : 0u);
    const int nb = w + 4 * (idx >> 2);
    const int nbc = nb * 32 < r_v ? nb : w;  // clamp: blocks past r_v are loaded but never used
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vr, lane * 16, (nbc * 4 + (idx & 3)) * 1024, 2));
  };

  f32x16 o[NBW];
#pragma unroll
  for (int b = 0; b < NBW; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[b][j] = 0.f;

  const uint16_t* page_cur = to_page(id0, tile_begin);
  const uint16_t* page_nxt = to_page(id1, tile_begin + 1);
  // One ring of sixteen operand registers per wave carries the whole stream: slot j holds K operand j of a tile until
  // the scores have used it, then V operand j of the same tile until P C_v has used it, then K operand j of the
  // next tile.  Every slot is re-requested the moment it is consumed, so a workgroup always has one tile's K or V
  // latents (64 KiB) on their way.
  u32x4 ring[NK32];
#pragma unroll
  for (int u = 0; u < NK32; ++u) ring[u] = k_frag(page_cur, u);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < QCH; ++u) {
    const int c = tid + 256 * u;
    if (c < 32 * cpr) {
      const int h = c / cpr, cc = c - h * cpr;
      const u32x4 z = {0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(qlds + ((size_t)((h >> 4) * nk32 + (cc >> 2)) * 64 + (h & 15) + 16 * (cc & 3)) * 8) = h < p.h_q ? qv[u] : z;
    }
  }
  __syncthreads();  // absorbed query in place
  const uint16_t* qa_lane = qlds + (size_t)lane * 8;

  for (int tile = tile_begin; tile < tile_end; ++tile) {
    const int valid = (ctx - tile * T) < T ? (ctx - tile * T) : T;
    // ---- scores; every K operand consumed is replaced by the request for the V operand of the same slot
    f32x4 sacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < NK32; ++ks) {
      // straight-line: a step past the rank re-reads the last query block and is switched off by zeroing that operand
      const int kc = ks < nk32 ? ks : nk32 - 1;
      const uint32_t keep = ks < nk32 ? 0xffffffffu : 0u;
      u32x4 a0 = *reinterpret_cast<const u32x4*>(qa_lane + (size_t)kc * 512), a1 = *reinterpret_cast<const u32x4*>(qa_lane + (size_t)(nk32 + kc) * 512);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a0[c] &= keep;
        a1[c] &= keep;
      }
      const bf16x8 kf = __builtin_bit_cast(bf16x8, ring[ks]);
      sacc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), kf, sacc[0], 0, 0, 0);
      sacc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), kf, sacc[1], 0, 0, 0);
      ring[ks] = v_frag(page_cur, ks);
      __builtin_amdgcn_sched_barrier(0);  // keeps the query operand reads of later steps from being hoisted (and spilled)
    }
    // ---- wave-local softmax statistics (rows of 16 lanes share a head), exchanged once between the waves
    float pv[2][4], m_loc[2][4], s_loc[2][4];
    const bool in_ctx = page_cur != nullptr && 16 * w + n16 < valid;
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        pv[hb][j] = in_ctx ? sacc[hb][j] * p.q_scale : kNegInf;
        float m = pv[hb][j];
        m = fmaxf(m, half_wave_peer<0>(m));
        m = fmaxf(m, half_wave_peer<1>(m));
        m = fmaxf(m, half_wave_peer<2>(m));
        m = fmaxf(m, half_wave_peer<3>(m));
        m_loc[hb][j] = m;
        const float e = __builtin_amdgcn_exp2f(pv[hb][j] - fmaxf(m, -1e30f));  // all masked: exp2(-inf) = 0
        pv[hb][j] = e;
        float su = e;
        su += half_wave_peer<0>(su);
        su += half_wave_peer<1>(su);
        su += half_wave_peer<2>(su);
        su += half_wave_peer<3>(su);
        s_loc[hb][j] = su;
      }
    lds_barrier();  // the previous tile's readers of pbuf, alpha and the exchange arrays are done
    if (n16 == 0) {
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int h = hb * 16 + 4 * kg + j;
          xm[h * 4 + w] = m_loc[hb][j];
          xs[h * 4 + w] = s_loc[hb][j];
        }
    }
    lds_barrier();
    float lnew[2][4], mnew[2][4];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int h = hb * 16 + 4 * kg + j;
        const f32x4 wm = *reinterpret_cast<const f32x4*>(xm + h * 4);
        const f32x4 wsu = *reinterpret_cast<const f32x4*>(xs + h * 4);
        const float m_old = m_fin[h];
        const float m_new = fmaxf(fmaxf(m_old, fmaxf(wm[0], wm[1])), fmaxf(wm[2], wm[3]));
        const float m_ref = fmaxf(m_new, -1e30f);
        if (w == 0 && n16 == 0) {  // one lane per head keeps the running state (read by everyone before the barrier below)
          float lsum = 0.f;
#pragma unroll
          for (int u = 0; u < 4; ++u) lsum += wsu[u] * __builtin_amdgcn_exp2f(wm[u] - m_ref);
          const float a = __builtin_amdgcn_exp2f(m_old - m_ref);
          alpha[h] = a;
          lnew[hb][j] = l_fin[h] * a + lsum;
        }
        mnew[hb][j] = m_new;
        pbuf[((size_t)w * 64 + h + 32 * (n16 >> 3)) * 8 + (n16 & 7)] = bf16_bits(pv[hb][j] * __builtin_amdgcn_exp2f(m_loc[hb][j] - m_ref));
      }
    lds_barrier();  // every lane has read the old running maxima: they can be replaced
    if (w == 0 && n16 == 0) {
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          m_fin[hb * 16 + 4 * kg + j] = mnew[hb][j];
          l_fin[hb * 16 + 4 * kg + j] = lnew[hb][j];
        }
    }
    // ---- o_lat = alpha * o_lat + P C_v : wave w owns latent blocks w, w + 4, ...
    {
      const bool ragged = page_cur == nullptr || valid < T;  // wave-uniform: only then the V operand needs masking
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        if ((w + 4 * i) * 32 < r_v) {
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) o[i][jj] *= alpha[acc_row(jj, hf)];
          if (!ragged) {
#pragma unroll
            for (int kp = 0; kp < KP; ++kp)
              o[i] = mfma32(load_frag(pbuf + ((size_t)kp * 64 + lane) * 8), __builtin_bit_cast(bf16x8, ring[i * KP + kp]), o[i]);
          } else {
#pragma unroll
            for (int kp = 0; kp < KP; ++kp) {
              int nv = valid - kp * 16 - 8 * hf;
              nv = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
              const uint32_t vmask = page_cur != nullptr ? (1u << nv) - 1u : 0u;
              u32x4 vv = ring[i * KP + kp];
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const uint32_t two = (vmask >> (2 * c)) & 3u;
                vv[c] &= (two & 1u ? 0x0000ffffu : 0u) | (two & 2u ? 0xffff0000u : 0u);
              }
              o[i] = mfma32(load_frag(pbuf + ((size_t)kp * 64 + lane) * 8), __builtin_bit_cast(bf16x8, vv), o[i]);
            }
          }
        }
        // the slots of this block now take the next tile's K operands (past the last tile: a page nobody reads)
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) ring[i * KP + kp] = k_frag(page_nxt, i * KP + kp);
      }
    }
    page_cur = page_nxt;
    page_nxt = to_page(id_nn, tile + 2);
    id_nn = fetch_id(tile + 3);
  }

  // ---- partials of this split (same format as the rotary path)
  const size_t pbase = (size_t)seq * p.n_splits + split;
  __syncthreads();  // every wave is done with the query operands: their memory becomes the staging area
  if (tid < p.h_q) {
    p.part_ml[(pbase * p.h_q + tid) * 2 + 0] = m_fin[tid];
    p.part_ml[(pbase * p.h_q + tid) * 2 + 1] = l_fin[tid];
  }
  __syncthreads();
  float inv_l[16];
#pragma unroll
  for (int jj = 0; jj < 16; ++jj) {
    const float l = l_fin[acc_row(jj, hf)];
    inv_l[jj] = l > 0.f ? __builtin_amdgcn_rcpf(l) : 0.f;
  }
  const int pitch = r_v * 2 + 16;
  unsigned char* lane_base = smem + (size_t)(4 * hf) * pitch + l32 * 2 + w * 64;
#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    if ((w + 4 * i) * 32 < r_v) {
#pragma unroll
      for (int jj = 0; jj < 16; ++jj)
        *reinterpret_cast<uint16_t*>(lane_base + (8 * (jj >> 2) + (jj & 3)) * pitch + i * 256) = f16_bits(o[i][jj] * inv_l[jj]);
    }
  }
  lds_barrier();
  uint16_t* dst_rows = p.part_o + pbase * p.h_q * r_v;
  const int cpv = r_v >> 3, n_chunks = p.h_q * cpv;
  for (int c = tid; c < n_chunks; c += 256) {
    const int h = c / cpv, cc = c - h * cpv;
    *reinterpret_cast<u32x4*>(dst_rows + (size_t)c * 8) = *reinterpret_cast<const u32x4*>(smem + (size_t)h * pitch + cc * 16);
  }
}

// ------------------------------------------------------------------------------------------------ host
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Context splits: about one tile-walk per workgroup slot of the device, never more than kMaxSplits per sequence.
// A context of zero positions still gets one split (it writes empty partials, which the merge turns into zeros).
static void plan_splits(DecodePlan& pl, int b, int max_ctx, int slots, int max_splits) {
  int n_tiles = (max_ctx + pl.tile - 1) / pl.tile;
  if (n_tiles < 1) n_tiles = 1;
  long tps = (long)b * n_tiles / slots;
  if (tps < 1) tps = 1;
  if (tps > n_tiles) tps = n_tiles;
  const int most = max_splits < kMaxSplits ? max_splits : kMaxSplits;
  if ((n_tiles + tps - 1) / tps > most) tps = (n_tiles + most - 1) / most;
  pl.tiles_per_split = (int)tps;
  pl.n_splits = (int)((n_tiles + tps - 1) / tps);
}

static void plan_workspace(DecodePlan& pl, const lorc_layer_desc& d, int b) {
  size_t off = 0;
  pl.off_ml = off;
  off = align256(off + (size_t)b * pl.n_splits * d.n_q_heads * 2 * 4);
  pl.off_o = off;
  off = align256(off + (size_t)b * pl.n_splits * d.n_q_heads * d.rank_v * 2);
  pl.total_bytes = off;
}

// The plan of every shape that the stationary kernel does not take (and of those that it does, had it not been there).
static DecodePlan make_streaming_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, int max_splits) {
  const int qb_ = (d.n_q_heads + 31) / 32;
  // More than 32 query heads: the streaming kernel needs two score blocks per wave and spills; scores + values + merge
  // as three launches is 1.1x (rank 256) to 1.6x (rank 1024) faster at 64 heads, b 32, context 8192.
  if (qb_ > 1 && wide_shape_ok(d)) return make_wide_plan(d, b, max_ctx, n_cus, false, max_splits);
  if (d.rank_k > kStreamMaxRank || d.rank_v > kStreamMaxRank ||
      decode_lds_bytes(64, qb_, d.n_q_heads / d.n_kv_heads, d.rank_k, d.head_dim / 2) > 160 * 1024) {
    // no single-pass kernel holds this shape: the three-launch path, or nothing (total_bytes = 0: unsupported)
    if (wide_shape_ok(d)) return make_wide_plan(d, b, max_ctx, n_cus, false, max_splits);
    return DecodePlan{};
  }
  DecodePlan pl{};
  pl.stationary = 0;
  // Two shapes: a 128-position tile with one workgroup per CU (each B_k operand is reused over 128 positions), or
  // 64-position tiles with two co-resident workgroups (the second hides the first one's loads and VALU phases)
  // when two latent tiles fit LDS together and the per-wave state fits 256 registers.
  const int G = d.n_q_heads / d.n_kv_heads;
  const bool two_wg = d.rank_k <= 512 && d.rank_v <= 512 && d.n_q_heads <= 32 && G <= 8 &&
                      2 * ((decode_lds_bytes(64, 1, G, d.rank_k, d.head_dim / 2) + 1023) & ~(size_t)1023) <= 160 * 1024;
  // the 128-position tile only where its LDS image fits (64 query heads at rank 512 do not: they take the
  // 64-position tile with one workgroup per CU)
  const int qb = (d.n_q_heads + 31) / 32;
  const bool fits128 = decode_lds_bytes(128, qb, G, d.rank_k, d.head_dim / 2) <= 160 * 1024;
  pl.tile = (d.rank_k <= 512 && !two_wg && fits128) ? 128 : 64;
  pl.occupancy = two_wg ? 2 : 1;
  plan_splits(pl, b, max_ctx, (n_cus > 0 ? n_cus : 256) * pl.occupancy, max_splits);
  plan_workspace(pl, d, b);
  return pl;
}

static DecodePlan make_any_stationary_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, int max_splits) {
  DecodePlan pl = make_stationary_plan(d, b, max_ctx, n_cus, max_splits);
  if (!stationary_shape_ok(d)) pl.stationary = 2;
  return pl;
}

// Groups of one or two heads leave a stationary workgroup little work per factor load, and layers of them have many head pairs: many
// short sequences, or pairs that do not divide an XCD's CUs, are then faster elsewhere.  us per layer-step, three launches / stationary,
// overhead (and even share where it decides) in brackets: 64 / 64 heads rank 544 16 x 1000 [4] 199 / 192, 16 x 4000 [4] 663 / 631, 32 x 1000 [8]
// 362 / 390, 64 x 100 [16] 143 / 246; 40 / 40 heads rank 544 12 x 1000 [5] 112 / 106, 8 x 2000 [6] 134 / 134, 16 x 1000 [10] 132 / 149; 40 / 40
// heads rank 64 (padded to 256) 12 x 1000 [5] 61 / 57, 32 x 1000 [10] 114 / 133, rank 128 32 x 1000 [10] 138 / 137.  Groups of two: 40 / 20 heads
// rank 544 16 x 1000 [8 of 10] 89 / 85, 32 x 1000 [10 of 20] 138 / 147, 200 x 300 [17 of 39] 349 / 297; 36 / 18 heads rank 640 64 x 500 [12 of 18]
// 155 / 173; 64 / 32 heads rank 544 64 x 500 [8 of 32] 218 / 214.  Groups of three and more gain (48 / 16 heads rank 544 128 x 100 [8] 115 / 114,
// 200 x 300 [18] 324 / 281).  Up to 32 heads, streaming / stationary: 32 / 32 heads 200 x 300 [28] rank 160 246 / 301, rank 384 352 / 385,
// 128 x 100 [16] rank 160 136 / 135.
static bool stationary_loses(const lorc_layer_desc& d, int b, int max_ctx, const DecodePlan& pl, int n_cus) {
  const int G = d.n_q_heads / d.n_kv_heads;
  double share;
  const double overhead = stationary_overhead(d, b, max_ctx, pl, n_cus, &share);
  if (G == 1 && d.n_q_heads > 32) return overhead >= 6 && (pl.stationary == 2 || d.rank_k <= 96);
  if (G == 1) return pl.stationary == 1 && d.rank_k <= 384 && overhead >= 18;
  return G == 2 && d.n_q_heads > 32 && pl.stationary == 2 && overhead >= 9.5 && overhead >= 0.5 * share;
}

DecodePlan make_decode_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, int max_splits) {
  if (stationary_shape_ok(d) || stationary768_shape_ok(d)) {
    const DecodePlan pl = make_any_stationary_plan(d, b, max_ctx, n_cus, kAnySplits);
    if (!stationary_loses(d, b, max_ctx, pl, n_cus)) return max_splits >= kAnySplits ? pl : make_any_stationary_plan(d, b, max_ctx, n_cus, max_splits);
  }
  return make_streaming_plan(d, b, max_ctx, n_cus, max_splits);
}

// A plan of at most as many splits as a workspace of `bytes` holds, or, if there is none, the one without that limit.
template <typename Make>
static DecodePlan plan_within(const lorc_layer_desc& d, int b, size_t bytes, Make make) {
  const DecodePlan pl = make(kAnySplits);
  if (pl.total_bytes <= bytes) return pl;
  const size_t per_split = (size_t)b * d.n_q_heads * (8 + 2 * (size_t)d.rank_v);
  const size_t scores = pl.wide ? pl.total_bytes - pl.off_scores : 0;
  size_t most = bytes > scores ? (bytes - scores) / per_split : 0;
  if (most >= (size_t)pl.n_splits) most = pl.n_splits - 1;
  for (; most >= 1; --most) {  // (a few steps: what the alignment of the parts takes)
    const DecodePlan fewer = make((int)most);
    if (fewer.total_bytes <= bytes) return fewer;
    if (fewer.n_splits > (int)most) break;  // the fewest that the kernel can walk
  }
  return pl;
}

DecodePlan make_decode_plan_within(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, size_t bytes) {
  const DecodePlan pl = plan_within(d, b, bytes, [&](int most) { return make_decode_plan(d, b, max_ctx, n_cus, most); });
  if (pl.total_bytes <= bytes || !(stationary_shape_ok(d) || stationary768_shape_ok(d))) return pl;
  // Shapes of two kernels: the other one's plan.  The stationary kernels have no scores to keep, a split of the streaming one may walk
  // more than their 512 pages.
  const DecodePlan other = plan_within(d, b, bytes, [&](int most) {
    return pl.stationary ? make_streaming_plan(d, b, max_ctx, n_cus, most) : make_any_stationary_plan(d, b, max_ctx, n_cus, most);
  });
  return other.total_bytes != 0 && other.total_bytes <= bytes ? other : pl;
}

template <int HD, int NPB, int QB, int NBW, int JR, int OCC>
static const char* split_symbol() {
  struct Text {
    char s[64];
    Text() { snprintf(s, sizeof(s), "decode_split_kernel<%d, %d, %d, %d, %d, %d>", HD, NPB, QB, NBW, JR, OCC); }
  };
  static const Text text;
  return text.s;
}

template <int HD, int NPB, int QB, int NBW, int JR, int OCC>
static int launch_split(const DecodeParams& p, hipStream_t s, bool attr_only, const char** symbol) {
  auto kern = decode_split_kernel<HD, NPB, QB, NBW, JR, OCC>;
  if (symbol) {
    *symbol = split_symbol<HD, NPB, QB, NBW, JR, OCC>();
    return LORC_OK;
  }
  if (attr_only)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess
               ? LORC_OK : LORC_EHIP;
  const size_t lds = decode_lds_bytes(32 * NPB, QB, p.G, p.r_k, HD / 2);
  if (lds > 160 * 1024) return LORC_EUNSUPPORTED;
  return launch_kernel(kern, dim3(p.b * p.n_splits), dim3(256), lds, s, p);
}

// Picks the instantiation for a shape and launches it; with attr_all it walks every instantiation instead and
// sets its LDS attribute, with symbol it only names it (nothing is launched).
template <int HD, int NPB>
static int dispatch_split(const DecodeParams& p, const DecodePlan& plan, hipStream_t s, bool attr_all = false, const char** symbol = nullptr) {
  const int qb = (p.h_q + 31) / 32;
  const int nbw = (p.r_v / 32 + 3) / 4;  // V latent blocks per wave
  int rc = LORC_OK;
  if (attr_all || (NPB == 2 && plan.occupancy == 2 && p.G <= 8 && qb == 1 && nbw <= 4)) {
    rc = launch_split<HD, 2, 1, 4, 4, 2>(p, s, attr_all, symbol);
    if (!attr_all || rc) return rc;
  }
  if (attr_all || p.G <= 8) {
    if (attr_all || (qb == 1 && nbw <= 4)) { rc = launch_split<HD, NPB, 1, 4, 4, 1>(p, s, attr_all, symbol); if (!attr_all || rc) return rc; }
    if (attr_all || qb == 1) { rc = launch_split<HD, NPB, 1, 8, 4, 1>(p, s, attr_all, symbol); if (!attr_all || rc) return rc; }
    if (attr_all || nbw <= 4) { rc = launch_split<HD, NPB, 2, 4, 4, 1>(p, s, attr_all, symbol); if (!attr_all || rc) return rc; }
    rc = launch_split<HD, NPB, 2, 8, 4, 1>(p, s, attr_all, symbol);
    if (!attr_all || rc) return rc;
  }
  // large query groups (G > 8): one generic instantiation per query-block count
  if (attr_all || qb == 1) { rc = launch_split<HD, NPB, 1, 8, 16, 1>(p, s, attr_all, symbol); if (!attr_all || rc) return rc; }
  return launch_split<HD, NPB, 2, 8, 16, 1>(p, s, attr_all, symbol);
}

static bool merge_group_ok(const DecodeParams& p) {
  return p.G <= kMgMaxG && p.n_splits <= kMgMaxSplits && p.r_v <= kMgMaxRank;
}

template <int HD, int HS, int CS, int MAXR, int MAXG = kMgMaxG / HS>
static int launch_merge_form(const DecodeParams& p, hipStream_t s) {
  return launch_kernel(decode_merge_group_kernel<HD, HS, CS, MAXR, MAXG>, dim3(p.b * p.h_kv * HS * CS), dim3(1024 / HS), 0, s, p);
}

template <int HD, int CS>
static int launch_merge_1024(const DecodeParams& p, hipStream_t s) {
  if (p.G == 1) return launch_merge_form<HD, 1, CS, 1024, 1>(p, s);
  if (p.G <= 4) return launch_merge_form<HD, 1, CS, 1024, 4>(p, s);
  return launch_merge_form<HD, 1, CS, 1024, 8>(p, s);
}

// Workgroups per group of heads, as many as add CUs (the figures are of 256 of them): us per call, one / more.
template <int HD>
static int launch_merge_group(const DecodeParams& p, hipStream_t s) {
  const int groups = p.b * p.h_kv, even = p.G % 2 == 0;
  // Two halves of the heads x blocks of 32 columns, up to 32 groups: 1 x 1337 23.0 / 22.1, 4 x 2000 at rank 544 30.4 / 28.5, but 8 x 2000
  // at rank 384 33.7 / 36.1, 16 x 4096 97 / 105 (the partials are fetched once per column block).
  const bool columns = even && p.latent_out == 0 && groups <= p.n_cus / 8;
  if (p.r_v <= 512) {
    if (columns) return launch_merge_form<HD, 2, HD / 32, 512>(p, s);
    return even && groups <= p.n_cus ? launch_merge_form<HD, 2, 1, 512>(p, s) : launch_merge_form<HD, 1, 1, 512>(p, s);
  }
  // Value ranks above 512.  Up to four heads: both to 16 groups (8B shape rank 1024, 32 groups 62.7, halves of the columns 60.6).  More, in
  // even number: both to 32 (70B shape rank 576 4 x 2000 29.7, halves of the columns 30.8), halves of both to 64 (7 x 546 25.1 / 26.7).
  // Then halves of the columns up to 128 groups (rank 768, 64 groups 44.0 / 42.3, 128 68.0 / 66.6, 256 70.2 / 72.9; 40 KV heads rank 640, 40
  // groups 39.9 / 38.0, 160 87.0 / 89.2).
  if (columns && groups <= p.n_cus / (p.G > 4 ? 8 : 16)) return launch_merge_form<HD, 2, HD / 32, 1024>(p, s);
  if (even && p.G > 4 && p.latent_out == 0 && groups <= p.n_cus / 4) return launch_merge_form<HD, 2, 2, 1024>(p, s);
  return groups <= p.n_cus / 2 && p.latent_out == 0 ? launch_merge_1024<HD, 2>(p, s) : launch_merge_1024<HD, 1>(p, s);
}

// The merge launch that follows every split kernel.
static int launch_merge(const DecodeParams& p, hipStream_t s) {
  // Groups of one head: every head reads a factor block of its own for every sequence, so that beyond a row or two per CU the kernel
  // below, four rows to a CU, is as fast or faster.  40 heads, us per layer-step, generic merge / this: rank 2048 1 x 700 84 / 54 (merge
  // alone 37 / 8), 4 x 700 134 / 120, 6 x 300 108 / 98, 8 x 500 143 / 146, 16 x 300 188 / 212; rank 704 8 x 2000 149.4 / 149.3, 16 x 1000
  // 151 / 157, 64 x 500 278 / 304; rank 1024 4 x 1000 87.6 / 79.6, 8 x 2000 194 / 192, 16 x 1000 196 / 200, 64 x 500 368 / 392; 32 heads
  // rank 800 16 x 1000 150.9 / 149.5, 64 x 500 288 / 302.
  if (p.G == 1 && p.r_v > kMgMaxRank && p.head_dim == 128 && p.latent_out == 0 && p.r_v <= kMgMaxRankG1 && p.n_splits <= kMgMaxSplits &&
      p.b * p.h_q <= p.n_cus)
    return launch_merge_form<128, 1, 4, kMgMaxRankG1, 1>(p, s);
  // Groups of two likewise: 64 / 32 heads, rank 544 64 x 100 104 / 114, 64 x 500 213 / 224, rank 768 128 x 100 200 / 224; 32 / 16 heads, 512
  // groups, rank 544 40.7 / 41.0, rank 768 47.4 / 46.6.  (Three: 48 / 16 heads, 2048 groups, rank 768 135 / 132.)
  if (!merge_group_ok(p) || (p.G <= 2 && p.r_v > 512 && p.b * p.h_kv > 2 * p.n_cus)) {
    if (p.head_dim == 128) return launch_kernel(decode_merge_kernel<128>, dim3(p.b * p.h_q), dim3(256), 0, s, p);
    return launch_kernel(decode_merge_kernel<64>, dim3(p.b * p.h_q), dim3(256), 0, s, p);
  }
  return p.head_dim == 128 ? launch_merge_group<128>(p, s) : launch_merge_group<64>(p, s);
}

DecodePlan make_absorbed_plan(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, int max_splits) {
  if (d.n_q_heads > 32 || d.rank_k > kAbsMaxRankK || d.rank_v > 512) {
    // beyond the single-pass kernel (one register ring per wave): scores, values in column chunks, merge
    if (!wide_absorbed_shape_ok(d)) return DecodePlan{};
    DecodePlan pl = make_wide_plan(d, b, max_ctx, n_cus, false, max_splits);
    pl.wide = 3;
    return pl;
  }
  DecodePlan pl{};
  pl.stationary = 0;
  pl.tile = kPage;
  pl.occupancy = 2;
  plan_splits(pl, b, max_ctx, 2 * (n_cus > 0 ? n_cus : 256), max_splits);  // two workgroups per CU
  plan_workspace(pl, d, b);
  return pl;
}

DecodePlan make_absorbed_plan_within(const lorc_layer_desc& d, int b, int max_ctx, int n_cus, size_t bytes) {
  return plan_within(d, b, bytes, [&](int most) { return make_absorbed_plan(d, b, max_ctx, n_cus, most); });
}

const char* decode_kernel_symbol(const lorc_layer_desc& d, const DecodePlan& plan, bool absorbed) {
  if (plan.wide == 3) return d.n_q_heads <= 32 ? "absorbed_scores_kernel<1>" : "absorbed_scores_kernel<2>";
  if (absorbed) return "decode_absorbed_kernel<4>";
  if (plan.wide) return "wide_scores_kernel";
  if (plan.stationary) return plan.stationary == 2 ? stationary768_kernel_symbol(d) : stationary_kernel_symbol(d);
  DecodeParams p{};
  p.h_q = d.n_q_heads;
  p.G = d.n_q_heads / d.n_kv_heads;
  p.r_v = d.rank_v;
  const char* symbol = nullptr;
  if (d.head_dim == 128) plan.tile == 128 ? dispatch_split<128, 4>(p, plan, nullptr, false, &symbol) : dispatch_split<128, 2>(p, plan, nullptr, false, &symbol);
  else plan.tile == 128 ? dispatch_split<64, 4>(p, plan, nullptr, false, &symbol) : dispatch_split<64, 2>(p, plan, nullptr, false, &symbol);
  return symbol;
}

int set_kernel_attributes_decode() {
  const DecodeParams none{};
  const DecodePlan plan{};
  if (int rc = dispatch_split<128, 4>(none, plan, nullptr, true)) return rc;
  if (int rc = dispatch_split<128, 2>(none, plan, nullptr, true)) return rc;
  if (int rc = dispatch_split<64, 4>(none, plan, nullptr, true)) return rc;
  if (int rc = dispatch_split<64, 2>(none, plan, nullptr, true)) return rc;
  if (int rc = set_kernel_attributes_decode_stationary()) return rc;
  if (int rc = set_kernel_attributes_decode_stationary768()) return rc;
  if (int rc = set_kernel_attributes_decode_wide()) return rc;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(decode_absorbed_kernel<4>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             160 * 1024) == hipSuccess ? LORC_OK : LORC_EHIP;
}

static int record(hipEvent_t ev, hipStream_t s) {
  return ev == nullptr || hipEventRecord(ev, s) == hipSuccess ? LORC_OK : LORC_EHIP;
}

int launch_decode_absorbed(const DecodeParams& p, const DecodePlan& plan, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end) {
  if (plan.total_bytes == 0) return LORC_EUNSUPPORTED;
  if (plan.wide) {
    if (int rc = record(ev_begin, s)) return rc;
    if (int rc = launch_decode_wide(p, plan, s)) return rc;
    if (int rc = record(ev_end, s)) return rc;
    if (p.head_dim == 128) return launch_kernel(decode_merge_kernel<128>, dim3(p.b * p.h_q), dim3(256), 0, s, p);
    return launch_kernel(decode_merge_kernel<64>, dim3(p.b * p.h_q), dim3(256), 0, s, p);
  }
  if (p.h_q > 32 || p.r_k > kAbsMaxRankK || p.r_v > 512) return LORC_EUNSUPPORTED;
  const size_t lds = absorbed_lds_bytes(p.r_k, p.r_v);
  if (lds > 160 * 1024) return LORC_EUNSUPPORTED;
  if (int rc = record(ev_begin, s)) return rc;
  if (int rc = launch_kernel(decode_absorbed_kernel<4>, dim3(p.b * p.n_splits), dim3(256), lds, s, p)) return rc;  // up to 16 V latent blocks, four per wave
  if (int rc = record(ev_end, s)) return rc;
  return launch_merge(p, s);
}

int launch_decode(const DecodeParams& p, const DecodePlan& plan, hipStream_t s, hipEvent_t ev_begin, hipEvent_t ev_end) {
  // shapes no instantiation covers are refused before anything (the begin event included) is put on the stream
  const int npb = plan.tile / 32, qb = (p.h_q + 31) / 32;
  if (plan.total_bytes == 0) return LORC_EUNSUPPORTED;
  if (!plan.stationary && !plan.wide && decode_lds_bytes(32 * npb, qb, p.G, p.r_k, p.head_dim / 2) > 160 * 1024) return LORC_EUNSUPPORTED;
  if (plan.wide == 1 && p.latent_out == 0 && p.r_v > kWideMaxRank) return LORC_EUNSUPPORTED;
  if (int rc = record(ev_begin, s)) return rc;
  int rc;
  if (plan.wide) {
    rc = launch_decode_wide(p, plan, s);
    if (rc != LORC_OK) return rc;
    if (int rc2 = record(ev_end, s)) return rc2;
    // the generic merge: softmax-merge of the splits; wide layers then apply B_v, uncompressed layers have none
    // (their partial rows are head_dim wide and are written out as they are)
    if (plan.wide == 2) {
      DecodeParams pm = p;
      pm.r_v = p.head_dim;
      pm.latent_out = 1;
      return launch_kernel(decode_merge_kernel<128>, dim3(pm.b * pm.h_q), dim3(256), 0, s, pm);
    }
    return launch_merge(p, s);  // the group merge where its limits hold, the generic one otherwise
  }
  if (plan.stationary == 2) rc = launch_decode_stationary768_split(p, plan, s);
  else if (plan.stationary) rc = launch_decode_stationary_split(p, plan, s);
  else if (p.head_dim == 128) rc = plan.tile == 128 ? dispatch_split<128, 4>(p, plan, s) : dispatch_split<128, 2>(p, plan, s);
  else rc = plan.tile == 128 ? dispatch_split<64, 4>(p, plan, s) : dispatch_split<64, 2>(p, plan, s);
  if (rc != LORC_OK) return rc;
  if (int rc2 = record(ev_end, s)) return rc2;
  return launch_merge(p, s);
}

}  // namespace lorc
