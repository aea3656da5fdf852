// Factor packing and the cache write (down-projection GEMM + paged scatter).
//
// lorc_append: C^T[j, t] = sum_k At[j, k] X[t, k]  (the compressed key/value x A of Section 4.1), bf16
// operands, fp32 accumulation on the 32x32x16 matrix-core op, RNE to bf16, scattered into the tiled pages.
#include "lorc_device.h"
#include "lorc_kernels.h"
#include "lorc_rebuild.h"
#include "lorc_tile_product.h"

namespace lorc {

// ------------------------------------------------------------------------------------------------ packing
__global__ void pack_factors_kernel(const uint16_t* __restrict__ A_k, const uint16_t* __restrict__ A_v,
                                    const uint16_t* __restrict__ B_k, const uint16_t* __restrict__ B_v,
                                    uint16_t* __restrict__ packed, int D, int r_k, int r_v, int n, int head_dim,
                                    float rope_base) {
  if (blockIdx.x == 0) {  // rotation tables: theta_i, and (cos, sin)(l * theta_i) in the arithmetic of the kernels
    const int half = head_dim / 2;
    double* theta = reinterpret_cast<double*>(packed + packed_off_rope(D, r_k, r_v, n));
    float2* lane_cs = reinterpret_cast<float2*>(theta + 64);
    for (int i = threadIdx.x; i < half; i += blockDim.x) theta[i] = rope_theta(i, head_dim, rope_base);
    for (int idx = threadIdx.x; idx < 32 * half; idx += blockDim.x) {
      const float th = (float)rope_theta(idx % half, head_dim, rope_base);
      float sn, cs;
      sincosf((float)(idx / half) * th, &sn, &cs);
      lane_cs[idx] = make_float2(cs, sn);
    }
  }
  const size_t n_at = packed_at_elems(D, r_k, r_v);
  const size_t n_bk = packed_b_elems(r_k, n);
  const size_t n_bv = packed_b_elems(r_v, n);
  const size_t total = n_at + n_bk + n_bv;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    if (i < n_at) {  // i = j * D + k  (output order: coalesced writes)
      const int j = (int)(i / D), k = (int)(i % D);
      const uint16_t v = j < r_k ? A_k[(size_t)k * r_k + j] : A_v[(size_t)k * r_v + (j - r_k)];
      packed[i] = v;
      packed[total + at_tile_index(D, j, k)] = v;
    } else if (B_k == nullptr) {  // uncompressed layer: no read-side factors
    } else if (i < n_at + n_bk) {  // source order: i' = j * n + c
      const size_t s = i - n_at;
      const int j = (int)(s / n), c = (int)(s % n);
      packed[n_at + b_tile_index(r_k, j, c)] = B_k[s];
    } else {
      const size_t s = i - n_at - n_bk;
      const int j = (int)(s / n), c = (int)(s % n);
      packed[n_at + n_bk + b_tile_index(r_v, j, c)] = B_v[s];
    }
  }
}

// ------------------------------------------------------------------------------------------------ append
// Short prompts.  Block tile: 64 latent rows x 64 tokens, k-tile 64, 4 waves as 2x2; or 32 x 32, each wave a k-step of the k-tile.
// LDS rows are 64 bf16 = 8 chunks of 16 B; chunk c of row r is stored at c ^ (r & 7) so that the 32 rows a
// fragment load touches spread over all banks.  With so few workgroups the walk over the model dimension is a
// chain of memory latencies, so every thread keeps PF k-tiles of both operands in flight in registers (buffer
// loads: rows past the end of either operand read as zero).
constexpr int kApBK = 64;

__device__ __forceinline__ int swz(int row, int chunk) { return (row * 8 + (chunk ^ (row & 7))) * 8; }

template <int BM>
__global__ __launch_bounds__(256) void append_kernel(AppendParams p) {
  constexpr int PF = 8, BN = BM, NB = 1, LD = BM / 32;  // accumulator blocks per wave and side; 16-byte loads per thread, operand and k-tile
  static_assert(PF % 2 == 0, "the LDS buffer of a k-tile is chosen by its stage's parity");
  __shared__ __align__(16) uint16_t sA[4][BM * kApBK];  // two buffers of each operand
  uint16_t (*const sB)[BM * kApBK] = sA + 2;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
  const int hf = lane >> 5, l32 = lane & 31;
  const int j0 = blockIdx.y * BM, t0 = blockIdx.x * BN;
  const int rt = p.r_k + p.r_v;
  const int D = p.D, nkt = D / kApBK;

  f32x16 acc[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[a][b][j] = 0.f;

  auto rows_rsrc = [&](const uint16_t* base, long long rows) {  // raw buffer over `rows` rows of D elements
    const long long bytes = rows * (long long)D * 2;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, bytes > 0x7fffffffLL ? 0x7fffffff : (int)bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t at_rsrc = rows_rsrc(p.at + (size_t)j0 * D, rt - j0);
  const __amdgpu_buffer_rsrc_t x_rsrc = rows_rsrc(p.x + (size_t)t0 * D, p.T - t0);
  uint32_t off[LD];
#pragma unroll
  for (int i = 0; i < LD; ++i) {
    const int c = tid + 256 * i, row = c >> 3, ch = c & 7;
    off[i] = (uint32_t)((row * D + ch * 8) * 2);
  }
  u32x4 ra[PF][LD], rb[PF][LD];
  auto request = [&](int st, int kt) {  // k-tile kt (the last one again past the end: never used, keeps the count fixed)
    const uint32_t koff = (uint32_t)((kt < nkt ? kt : nkt - 1) * (kApBK * 2));
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      ra[st][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(at_rsrc, (int)(off[i] + koff), 0, 0));
      rb[st][i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, (int)(off[i] + koff), 0, 0));
    }
  };
  auto to_lds = [&](int st) {  // stage st's registers into the LDS buffer of its parity
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int c = tid + 256 * i, row = c >> 3, ch = c & 7;
      *reinterpret_cast<u32x4*>(sA[st & 1] + swz(row, ch)) = ra[st][i];
      *reinterpret_cast<u32x4*>(sB[st & 1] + swz(row, ch)) = rb[st][i];
    }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < kApBK / 16; ++ks) {
      if constexpr (BM == 32) {  // wave w takes k-step w of the k-tile for the whole tile
        if (ks == 0)
          acc[0][0] = mfma32(load_frag(sA[buf] + swz(l32, w * 2 + hf)), load_frag(sB[buf] + swz(l32, w * 2 + hf)), acc[0][0]);
        continue;
      }
      bf16x8 a[NB], b[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        a[i] = load_frag(sA[buf] + swz(wm * (BM / 2) + i * 32 + l32, ks * 2 + hf));
        b[i] = load_frag(sB[buf] + swz(wn * (BN / 2) + i * 32 + l32, ks * 2 + hf));
      }
#pragma unroll
      for (int mi = 0; mi < NB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) acc[mi][ni] = mfma32(a[mi], b[ni], acc[mi][ni]);
    }
  };
  // k-tile kt lives in stage kt % PF; while it is multiplied out of one LDS buffer, tile kt + 1 is written into
  // the other and tile kt + PF is requested into the registers tile kt left: one barrier per k-tile.
#pragma unroll
  for (int st = 0; st < PF; ++st) request(st, st);
  to_lds(0);
  __syncthreads();
  int kt0 = 0;
  for (; kt0 + PF <= nkt; kt0 += PF) {
#pragma unroll
    for (int st = 0; st < PF; ++st) {
      request(st, kt0 + st + PF);
      to_lds((st + 1) % PF);  // past the last k-tile: a copy of the last one, never multiplied
      multiply(st & 1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int st = 0; st < PF; ++st) {
    if (kt0 + st < nkt) {  // same for the whole workgroup
      if (st + 1 < PF) to_lds(st + 1);
      multiply(st & 1);
      __syncthreads();
    }
  }

  // 32 x 32 tiles: the waves' sums meet in LDS; wave w adds and files the rows 8 w + 4 hf .. + 3.
  f32x4 mine = {0.f, 0.f, 0.f, 0.f};
  if constexpr (BM == 32) {
    static_assert(BM != 32 || 4 * BM * kApBK * 2 >= 16 * 1024, "room for sixteen KiB of sums in sA and sB");
    f32x4* const meet = reinterpret_cast<f32x4*>(&sA[0][0]);  // [quarter][wave][64 lanes]
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      meet[(q4 * 4 + w) * 64 + lane] = f32x4{acc[0][0][4 * q4], acc[0][0][4 * q4 + 1], acc[0][0][4 * q4 + 2], acc[0][0][4 * q4 + 3]};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) mine += meet[(w * 4 + i) * 64 + lane];
  }
  // Epilogue: lane holds token column l32 of each block and 16 latent rows; 4 consecutive rows per group.
#pragma unroll
  for (int ni = 0; ni < NB; ++ni) {
    const int t = t0 + (BM == 32 ? 0 : wn * (BN / 2) + ni * 32) + l32;
    if (t >= p.T) continue;
    const int seq = p.slot_seq[t], pos = p.slot_pos[t];
    if (seq < 0 || seq >= p.n_seqs || pos < 0 || pos >= p.max_pages * kPage) continue;
    const int page = p.block_table[(size_t)seq * p.max_pages + pos / kPage];
    if (page < 0 || page >= p.n_pages) continue;
    const int slot = pos % kPage;
    uint16_t* base = p.cache + (size_t)page * p.page_elems;
#pragma unroll
    for (int mi = 0; mi < NB; ++mi) {
      const int jb = j0 + (BM == 32 ? 0 : wm * (BM / 2) + mi * 32);
      if (jb >= rt) continue;
#pragma unroll
      for (int q = 0; q < (BM == 32 ? 1 : 4); ++q) {
        const int j = jb + 8 * (BM == 32 ? w : q) + 4 * hf;
        uint16_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = bf16_bits(BM == 32 ? mine[i] : acc[mi][ni][4 * q + i]);
        if (j < p.r_k) {
          u32x2 pk = {(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16)};
          *reinterpret_cast<u32x2*>(base + k_index(p.r_k, slot, j)) = pk;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) base[v_index(p.r_k, slot, j - p.r_k + i)] = v[i];
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------ append, tiled
// 64 NC latent rows (of K or of V) x 128 tokens per workgroup (lorc_tile_product.h).  A CU takes 64 bytes per clock through
// its vector memory path, so 32 of the model dimension cannot be faster than 256 cycles at NC = 2 (16 KiB for 256
// matrix-core cycles) or 384 at NC = 4 (24 KiB for 512); with barrier and operand reads one workgroup alone needs about
// 500 and 850, two on a CU overlap.  Forms (NC, NS, KT): (2, 5, 4) all of LDS, for at most one workgroup per CU;
// (2, 2, 4) and (4, 3, 2) leave room for two.
// Epilogue: lanes own tokens in K row blocks and latent indices in V row blocks (operands swapped), so that after
// permute_halves a lane holds one 16-byte piece of a page's tiling: eight latent indices of a token, or eight
// consecutive slots of a latent index.
template <int NC, int NS, int KT>
__global__ __launch_bounds__(256, 2) void append_tile_kernel(AppendParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Block id -> tile.  An XCD (block id mod 8) takes a contiguous eighth of the tiles in an order whose inner index runs
  // over the operand with fewer bytes, so that its L2 holds a slice of the larger operand and streams the smaller.
  const int ncg_k = (p.r_k + 64 * NC - 1) / (64 * NC), ncg_v = (p.r_v + 64 * NC - 1) / (64 * NC), ncg = ncg_k + ncg_v;
  const int n_t = (p.T + 127) >> 7, total = ncg * n_t, per_xcd = (total + 7) >> 3;
  const int lin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || lin >= total) return;
  const bool rows_inner = p.T > p.r_k + p.r_v;
  const int cg = rows_inner ? lin % ncg : lin / n_t, t0 = (rows_inner ? lin / ncg : lin % n_t) * 128;
  const bool v_rows = cg >= ncg_k;
  const int rank = v_rows ? p.r_v : p.r_k, cb0 = (v_rows ? cg - ncg_k : cg) * 2 * NC, ncb = rank >> 5, nks = p.D >> 4;

  // where the tile's tokens go (looked up now: the latency hides behind the product)
  long long my_page = -1;
  int my_slot = 0;
  if (tid < 128 && t0 + tid < p.T) {
    const int seq = p.slot_seq[t0 + tid], pos = p.slot_pos[t0 + tid];
    if (seq >= 0 && seq < p.n_seqs && pos >= 0 && pos < p.max_pages * kPage) {
      const int page = p.block_table[(size_t)seq * p.max_pages + pos / kPage];
      if (page >= 0 && page < p.n_pages) {
        my_page = (long long)page * (long long)p.page_elems;
        my_slot = pos % kPage;
      }
    }
  }
  f32x16 acc[NC][2];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[c][pb][j] = 0.f;
  const u32x4 at = dma_rsrc(p.at_tiled + (v_rows ? (size_t)p.r_k * p.D : 0), (uint32_t)rank * (uint32_t)p.D * 2u);
  const int left = p.T - t0 < 128 ? p.T - t0 : 128;
  const u32x4 x = dma_rsrc(p.x + (size_t)t0 * p.D, (uint32_t)left * (uint32_t)p.D * 2u);
  const int n_kt = p.D / (16 * KT);
  if (v_rows) tile_product<64, NC, NS, kRows, true, KT>(acc, smem, at, x, cb0, ncb, nks, w, lane, n_kt, (uint32_t)p.D * 2u);
  else tile_product<64, NC, NS, kRows, false, KT>(acc, smem, at, x, cb0, ncb, nks, w, lane, n_kt, (uint32_t)p.D * 2u);
  __syncthreads();
  long long* tok_page = reinterpret_cast<long long*>(smem);
  int* tok_slot = reinterpret_cast<int*>(tok_page + 128);
  if (tid < 128) {
    tok_page[tid] = my_page;
    tok_slot[tid] = my_slot;
  }
  __syncthreads();
  auto pack8 = [&](const f32x16& a, int u) {
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)bf16_bits(a[8 * u + 2 * i]) | ((uint32_t)bf16_bits(a[8 * u + 2 * i + 1]) << 16);
    return permute_halves(v);
  };
#pragma unroll
  for (int pb = 0; pb < 2; ++pb) {
    const int tl = 64 * (w >> 1) + 32 * pb;  // first token (of the tile) of the position block
    if (!v_rows) {
      const long long page = tok_page[tl + l32];
      const int slot = tok_slot[tl + l32];
      uint16_t* dst = p.cache + (page < 0 ? 0 : page) + ((size_t)(slot >> 5) * (p.r_k >> 4) * 64 + (slot & 31) + 32 * hf) * 8;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int cb = cb0 + (w & 1) * NC + c;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const u32x4 v = pack8(acc[c][pb], u);
          if (cb < ncb && page >= 0) *reinterpret_cast<u32x4*>(dst + (size_t)(2 * cb + u) * 512) = v;
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int t8 = tl + 16 * u + 8 * hf;  // this lane's eight tokens
        const long long page0 = tok_page[t8];
        const int s0 = tok_slot[t8];
        bool run = page0 >= 0 && (s0 & 7) == 0;  // eight consecutive slots of one page: one piece of the V tiling
#pragma unroll
        for (int i = 1; i < 8; ++i) run = run && tok_page[t8 + i] == page0 && tok_slot[t8 + i] == s0 + i;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const int cb = cb0 + (w & 1) * NC + c;
          const u32x4 v = pack8(acc[c][pb], u);
          if (cb >= ncb) continue;
          if (run) {
            *reinterpret_cast<u32x4*>(p.cache + page0 + v_index(p.r_k, s0, 32 * cb + l32)) = v;
          } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const long long page = tok_page[t8 + i];
              if (page >= 0) p.cache[page + v_index(p.r_k, tok_slot[t8 + i], 32 * cb + l32)] = (uint16_t)(v[i >> 1] >> (16 * (i & 1)));
            }
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------ append, large T
// Prefill down-projection: 256 latent rows x 256 tokens per workgroup, four waves of 128 x 128 (16 accumulator
// blocks each: eight LDS operand reads per sixteen MFMAs).  Both operands go through a five-slot LDS ring (k-tile
// 64, 32 KiB per slot = all 160 KiB of the CU) filled by direct global -> LDS loads; the only other loads in the
// loop are LDS reads, so the in-order memory counter measures exactly the ring.
// Row blocks of the V latent are computed with the operands swapped (tokens along accumulator rows), which puts
// four consecutive cache slots of one latent index in one lane: 8-byte stores into the V tiling.
constexpr int kGmBM = 256, kGmBN = 256, kGmBK = 64, kGmSlots = 5;
constexpr int kGmSlotElems = 256 * kGmBK;  // one operand tile: 256 rows x 64 = 32 KiB
constexpr int kGmLdsBytes = kGmSlots * kGmSlotElems * 2;

// Slot ring: operand tiles are filled in the order X0 A0 X1 A1 ... into slots 0 1 2 3 4 0 1 ...; k-tile kt uses
// fills 2kt (tokens) and 2kt+1 (weights).  The refills are spread over the k-steps, four loads per wave and
// k-step: once k-tile kt has been handed over, its two slots take the weights of k-tile kt+2 (half in the last
// k-step of kt, half in the first of kt+1) and the tokens of k-tile kt+3 (second and third k-step of kt+1).
// Rows are 128 B = one cache line per row and k-tile (8 chunks of 16 B, chunk c of row r at c ^ (r & 7)): every
// line fetched is fully used, and operand reads stay conflict-free with per-lane bases.
template <bool SWAP>
__device__ __forceinline__ void gemm_mainloop(f32x16 (&acc)[4][4], uint16_t* lds, __amdgpu_buffer_rsrc_t at, __amdgpu_buffer_rsrc_t x,
                                              const uint32_t (&aoff)[8], const uint32_t (&xoff)[8], int nkt, int w, int wm,
                                              int wn, int hf, int l32) {
  int ra[4], rb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int phys = (2 * ks + hf) ^ (l32 & 7);
    ra[ks] = ((wm * 128 + l32) * 8 + phys) * 8;
    rb[ks] = ((wn * 128 + l32) * 8 + phys) * 8;
  }
  auto fill_part = [&](int f, int half) {  // half of fill number f: operand f & 1 (0 = X, 1 = At) of k-tile f >> 1
    const int kt = f >> 1, k = kt < nkt ? kt : nkt - 1;  // clamped refills keep the loads in flight constant
    uint16_t* base = lds + (size_t)(f % kGmSlots) * kGmSlotElems;
#pragma unroll
    for (int i = 4 * half; i < 4 * half + 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds((f & 1) ? at : x, (__attribute__((address_space(3))) void*)(base + (size_t)(i * 4 + w) * 512), 16,
                                               (f & 1) ? aoff[i] : xoff[i], k * (kGmBK * 2), 0, 0);
  };
  auto fill = [&](int f) { fill_part(f, 0); fill_part(f, 1); };
  // Operand fragments are double-buffered in registers: the LDS reads of k-step s+1 are issued among the MFMAs
  // of k-step s, so no MFMA waits on an LDS round trip.  The barrier that hands over the next k-tile therefore
  // sits inside the last k-step of the current one.
  bf16x8 fa[2][4], fb[2][4];
  auto frags = [&](int buf, int kt, int ks) {
    const uint16_t* sa = lds + (size_t)((2 * kt + 1) % kGmSlots) * kGmSlotElems;
    const uint16_t* sb = lds + (size_t)((2 * kt) % kGmSlots) * kGmSlotElems;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[buf][i] = load_frag(sa + ra[ks] + i * 32 * 8 * 8);
      fb[buf][i] = load_frag(sb + rb[ks] + i * 32 * 8 * 8);
    }
  };
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
#pragma unroll
      for (int ni = 0; ni < 4; ++ni)
        acc[mi][ni] = SWAP ? mfma32(fb[buf][ni], fa[buf][mi], acc[mi][ni]) : mfma32(fa[buf][mi], fb[buf][ni], acc[mi][ni]);
  };
  // The refills are spread evenly over the k-steps, four loads per k-step and wave: a burst of sixteen at the
  // hand-over asks for more than the L2 -> CU path sustains, the queue backs up and the wave -- in-order, one per
  // SIMD -- stalls in the issue of a load with its MFMAs behind it.
  fill(0);
  fill(1);
  fill(2);
  fill_part(3, 0);
  __builtin_amdgcn_s_waitcnt(0x0F7C);  // vmcnt(12): fills 0 and 1 landed
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  frags(0, 0, 0);
  for (int kt = 0; kt < nkt; ++kt) {
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      frags((ks + 1) & 1, kt, ks + 1);
      // ks 0: second half of the weights of k-tile kt+1;  ks 1, 2: the tokens of k-tile kt+2
      if (ks == 0) fill_part(2 * kt + 3, 1);
      else fill_part(2 * kt + 4, ks - 1);
      mfmas(ks & 1);
      // the ring writes may alias the fragment reads as far as the compiler knows, so the reads go first
#pragma unroll
      // an MFMA leads: the wait in front of it then covers only the previous k-step's reads, long since back
      for (int g = 0; g < 8; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // two MFMAs
        __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);  // one global -> LDS load
      }
    }
    // Last k-step.  Its fragments are in registers, so once every wave is here k-tile kt's two slots are free;
    // fills 2kt+2 and 2kt+3 (k-tile kt+1) must have landed, fill 2kt+4 (8 loads per wave, issued in this
    // k-tile's second and third k-step) may still be in flight.
    __builtin_amdgcn_s_waitcnt(0x0078);  // vmcnt(8) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();  // bare: a fence would make the compiler drain every LDS-bound load in flight
    asm volatile("" ::: "memory");
    frags(0, kt + 1, 0);
    fill_part(2 * kt + 5, 0);  // first half of the weights of k-tile kt+2, into the slot of k-tile kt's tokens
    mfmas(1);
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // drain the clamped tail loads before LDS is reused
  __syncthreads();
}

__global__ __launch_bounds__(256, 1) void append_gemm_kernel(AppendParams p) {
  extern __shared__ __align__(16) unsigned char smem_gemm[];
  uint16_t* const lds = reinterpret_cast<uint16_t*>(smem_gemm);
  // after the main loop the ring's memory holds, per token of the tile, the element offset of its page in the
  // pool (or -1) and its slot
  long long* const tok_page = reinterpret_cast<long long*>(smem_gemm);
  int* const tok_slot = reinterpret_cast<int*>(tok_page + kGmBN);
  long long* const grp_page = reinterpret_cast<long long*>(tok_slot + kGmBN);  // per aligned group of 4 tokens
  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
  // Workgroups are dealt round-robin over the 8 XCDs (each with its own L2).  The row blocks that share a token
  // tile get consecutive turns on ONE XCD, so that the tile comes from HBM once and is an L2 hit for the others.
  const int ny = (p.r_k + p.r_v + kGmBM - 1) / kGmBM;
  const int n_virtual = (((p.T + kGmBN - 1) / kGmBN + 7) / 8) * 8 * ny;
  // Persistent: the grid is one workgroup per CU (a multiple of 8, so that a workgroup stays on its XCD's turn
  // sequence) and every workgroup walks its tiles; a tile's stores drain while the next tile's ring fills.
  for (int vb = blockIdx.x; vb < n_virtual; vb += gridDim.x) {
  const int xcd = vb & 7, turn = vb >> 3;
  const int bx = (turn / ny) * 8 + xcd, by = turn % ny;
  if (bx * kGmBN >= p.T) continue;
  const int j0 = by * kGmBM, t0 = bx * kGmBN;
  const int rt = p.r_k + p.r_v, D = p.D;
  const int nkt = D / kGmBK;

  // The workgroup's 256 latent rows; at the matrix edge the window is slid back so that every row is real,
  // and rows outside a wave's own share are skipped by the epilogue.
  const int j0_eff = j0 + kGmBM <= rt ? j0 : (rt - kGmBM > 0 ? rt - kGmBM : 0);
  const int jw_eff = j0_eff + wm * 128;
  // This lane's eight source chunks per operand, as byte offsets from the tile's first row (rows past the matrices
  // are clamped, never stored).  The copies are buffer loads -- a descriptor of the tile's rows, a 32-bit lane
  // offset, the k-tile as scalar offset: next to a saturated MFMA stream they issue in a few cycles, where a
  // load with 64-bit lane addresses holds the wave, and its MFMAs, for about thirty.
  uint32_t aoff[8], xoff[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int L = (i * 4 + w) * 64 + lane, row = L >> 3, c = (L & 7) ^ (row & 7);
    const int ja = j0_eff + row < rt ? row : rt - 1 - j0_eff;
    const int tb = t0 + row < p.T ? row : p.T - 1 - t0;
    aoff[i] = (uint32_t)((ja * D + c * 8) * 2);
    xoff[i] = (uint32_t)((tb * D + c * 8) * 2);
  }
  auto rows_rsrc = [&](const uint16_t* base, long long rows) {  // raw buffer over `rows` rows of D elements
    const long long bytes = rows * D * 2;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, bytes > 0x7fffffffLL ? 0x7fffffff : (int)bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t at_rsrc = rows_rsrc(p.at + (size_t)j0_eff * D, rt - j0_eff);
  const __amdgpu_buffer_rsrc_t x_rsrc = rows_rsrc(p.x + (size_t)t0 * D, p.T - t0);
  // this thread's token of the tile: where it goes (looked up now, its latency hides behind the main loop)
  long long my_page_off = -1;
  int my_slot = 0;
  if (t0 + tid < p.T) {
    const int seq = p.slot_seq[t0 + tid], pos = p.slot_pos[t0 + tid];
    if (seq >= 0 && seq < p.n_seqs && pos >= 0 && pos < p.max_pages * kPage) {
      const int page = p.block_table[(size_t)seq * p.max_pages + pos / kPage];
      if (page >= 0 && page < p.n_pages) {
        my_page_off = (long long)page * (long long)p.page_elems;
        my_slot = pos % kPage;
      }
    }
  }
  f32x16 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[a][b][j] = 0.f;
  const bool all_v = jw_eff >= p.r_k;  // every block of this wave lies in the V latent: swapped operands
  if (all_v) gemm_mainloop<true>(acc, lds, at_rsrc, x_rsrc, aoff, xoff, nkt, w, wm, wn, hf, l32);
  else gemm_mainloop<false>(acc, lds, at_rsrc, x_rsrc, aoff, xoff, nkt, w, wm, wn, hf, l32);
  tok_page[tid] = my_page_off;
  tok_slot[tid] = my_slot;
  __syncthreads();
  if (tid < kGmBN / 4) {  // aligned groups of four tokens that sit in four consecutive slots of one page
    const long long pg0 = tok_page[4 * tid];
    const int s0 = tok_slot[4 * tid];
    bool run = pg0 >= 0 && (s0 & 3) == 0;
#pragma unroll
    for (int i = 1; i < 4; ++i) run = run && tok_page[4 * tid + i] == pg0 && tok_slot[4 * tid + i] == s0 + i;
    grp_page[tid] = run ? pg0 : -1;
  }
  __syncthreads();

  // ---------------- epilogue
  // Index arithmetic is hoisted: a destination is (page, slot)-dependent part + (latent block)-dependent part, the
  // first computed once per token (group), the second wave-uniform.
  auto pack4 = [&](const f32x16& a, int q4) {
    uint16_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = bf16_bits(a[4 * q4 + i]);
    return u32x2{(uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16)};
  };
  if (!all_v) {
    // accumulator rows = latent index, lane = token: 4 consecutive latent indices per register group
    const int nks = p.r_k >> 4;
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
      const int tl = wn * 128 + ni * 32 + l32;
      const long long page_off = tok_page[tl];
      if (page_off < 0) continue;
      const int slot = tok_slot[tl];
      uint16_t* base = p.cache + page_off;
      // K tiling: k_index(slot, jb + 8 q4 + 4 hf) = [slot part] + 4 hf + 32 jb + 256 q4   (jb a multiple of 32)
      uint16_t* kdst = base + ((size_t)(slot >> 5) * nks * 512 + (slot & 31) * 8 + 4 * hf);
#pragma unroll
      for (int mi = 0; mi < 4; ++mi) {
        const int jb = jw_eff + mi * 32;
        if (jb < j0 || jb >= rt) continue;  // rows of the slid-back window that belong to the previous workgroup
        if (jb + 32 <= p.r_k) {             // wave-uniform: the whole block is K latent
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) *reinterpret_cast<u32x2*>(kdst + (size_t)jb * 32 + q4 * 256) = pack4(acc[mi][ni], q4);
        } else {
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int j = jb + 8 * q4 + 4 * hf;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint16_t v = bf16_bits(acc[mi][ni][4 * q4 + i]);
              if (j + i < p.r_k) base[k_index(p.r_k, slot, j + i)] = v;
              else base[v_index(p.r_k, slot, j + i - p.r_k)] = v;
            }
          }
        }
      }
    }
  } else {
    // swapped: accumulator rows = token, lane = latent index; 4 consecutive tokens per register group
#pragma unroll
    for (int ni = 0; ni < 4; ++ni) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int tl = wn * 128 + ni * 32 + 8 * q4 + 4 * hf;
        const long long pg0 = grp_page[tl >> 2];
        const int s0 = tok_slot[tl];
        if (pg0 >= 0) {  // four consecutive slots of one page: contiguous in the V tiling
          // v_index(s0, jv) = 64 r_k + [slot part] + 8 (jv % 32) + 2048 (jv / 32),  jv = jb - r_k + l32
          uint16_t* vdst = p.cache + pg0 + ((size_t)kPage * p.r_k + (size_t)(s0 >> 4) * 512 + ((s0 & 15) >> 3) * 256 + (s0 & 7) + l32 * 8);
#pragma unroll
          for (int mi = 0; mi < 4; ++mi) {
            const int jb = jw_eff + mi * 32;
            if (jb < j0 || jb >= rt) continue;
            *reinterpret_cast<u32x2*>(vdst + (size_t)((jb - p.r_k) >> 5) * 2048) = pack4(acc[mi][ni], q4);
          }
        } else {
#pragma unroll
          for (int mi = 0; mi < 4; ++mi) {
            const int jb = jw_eff + mi * 32;
            if (jb < j0 || jb >= rt) continue;
            const int jv = jb + l32 - p.r_k;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const long long pg = tok_page[tl + i];
              if (pg >= 0) p.cache[pg + v_index(p.r_k, tok_slot[tl + i], jv)] = bf16_bits(acc[mi][ni][4 * q4 + i]);
            }
          }
        }
      }
    }
  }
  __syncthreads();  // the token arrays in the ring's memory have been read by everyone: the next tile may fill it
  }
}

// ------------------------------------------------------------------------------------------- append, small T
// Decode-time append: up to 64 tokens against the whole down-projection in one pass over the weights (8 MiB for the 8B shape).
// The rows are dealt evenly to all CUs: `rows` of them (at most 16) per workgroup of sixteen waves; wave w owns the lines (64 of
// the model dimension) w, w + 16, ... of all of them: 16x16x32 products, A = the workgroup's rows, B = 16 tokens; the waves'
// partial sums meet in LDS.  Bound by one load latency and the reduction for a few tokens (about 4 us), and then by the tokens,
// which every CU reads whole: 48 bytes per ns and CU past the L1 whatever the order of the lines, the rows per workgroup or the
// number of requests in flight (0.17 us per token at D = 4096, 0.34 at 8192).  A request costs its 16 cycles of address work
// even where it fetches nothing, hence a form per number of tokens, and rows past eight only where there are any.
//   us, weights cold (dot products over 4 rows, 16 tokens a pass / this kernel with 32 tokens a pass, a wave on consecutive
//   lines, slots looked up behind the products / now):
//   8B rank 512, T = 1: 7.4 / 5.6 / 4.1;  16: 7.9 / 7.7 / 7.0;  48: 17.0 / 18.9 / 14.2;  64: 21.6 / 21.3 / 17.7
//   70B rank 512, T = 1: 10.3 / 8.6 / 5.7;  16: 11.2 / 13.0 / 11.6;  48: 25.2 / 33.6 / 25.6;  64: 32.0 / 38.7 / 32.7
//   13B rank 2048, T = 16: 24.2 / 15.1 / 14.9;  64: 75.6 / 39.4 / 29.1;  tiny layer, T = 1: 5.5 / 3.0 / 2.4
constexpr int kSkWaves = 16, kSkMaxRows = 16;

// Rows x 64 of the contraction (a 128-byte line of each row) as the operands of two k-steps: lane m + 16 q holds the pieces q
// and 4 + q (of eight, 16 bytes each) of row m.  Sixteen rows take two requests of 64 bytes per row; eight rows take one request
// of whole lines -- lane m + 16 q fetches piece q + 4 (m / 8) of row m % 8 -- and the second k-step has the halves of each row of
// lanes changed round (rows 8 .. 15 of the operands then repeat and are not to be used).
template <bool SIXTEEN>
struct RowLines {
  u32x4 v[SIXTEEN ? 2 : 1];
  static __device__ __forceinline__ uint32_t lane_offset(int lane, uint32_t row_bytes) {
    const int m = lane & 15, q = lane >> 4;
    return SIXTEEN ? (uint32_t)m * row_bytes + (uint32_t)q * 16u : (uint32_t)(m & 7) * row_bytes + (uint32_t)(q + 4 * (m >> 3)) * 16u;
  }
  template <int AUX>  // cache policy bits of the load
  __device__ __forceinline__ void request(__amdgpu_buffer_rsrc_t r, uint32_t at) {
    v[0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, AUX));
    if constexpr (SIXTEEN) v[1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at + 64u, 0, AUX));
  }
  __device__ __forceinline__ bf16x8 step(int s) const {
    if constexpr (SIXTEEN) return __builtin_bit_cast(bf16x8, v[s]);
    if (s == 0) return __builtin_bit_cast(bf16x8, v[0]);
    u32x4 r;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t x = v[0][c];
      r[c] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xF, 0xF, false);  // row_ror:8
    }
    return __builtin_bit_cast(bf16x8, r);
  }
};

// TG: groups of 16 tokens, all of the call's (0: at most eight tokens);  R16: more than eight rows
template <int TG, bool R16>
__global__ __launch_bounds__(64 * kSkWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void append_skinny_kernel(AppendParams p, int rows) {
  constexpr int NG = TG > 0 ? TG : 1, PF = 2;  // lines in flight (four: no faster, and more requests past a wave's share)
  __shared__ float red[kSkWaves][NG][16][16];  // [wave][token group][row][token]
  const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rt = p.r_k + p.r_v, j0 = blockIdx.x * rows, n_rows = rt - j0 < rows ? rt - j0 : rows;
  // Output (row o / 16 NG, token o % 16 NG) is thread o's: its token's slot is asked for before the operands, and its page
  // behind them, so that neither look-up is waited for.
  const int orow = tid / (16 * NG), ot = tid % (16 * NG);
  const bool out = orow < n_rows && ot < p.T;
  const int seq = out ? p.slot_seq[ot] : -1, pos = out ? p.slot_pos[ot] : -1;
  __builtin_amdgcn_sched_barrier(0);

  const int n_mine = ((p.D >> 6) - w + kSkWaves - 1) / kSkWaves;  // this wave's lines: w, w + 16, ...
  const uint32_t row_bytes = (uint32_t)p.D * 2u;
  const __amdgpu_buffer_rsrc_t ar = make_rsrc(uniform_ptr(p.at + (size_t)j0 * p.D), (uint32_t)n_rows * row_bytes);
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, (uint32_t)p.T * row_bytes);
  using Rows = RowLines<R16>;
  using Tokens = RowLines<(TG > 0)>;
  const uint32_t a_off = Rows::lane_offset(lane, row_bytes), b_off = Tokens::lane_offset(lane, row_bytes);
  f32x4 acc[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[g][j] = 0.f;
  Rows a[PF];
  Tokens b[PF][NG];
  // rows past the descriptors read as zeros and fetch nothing; so do lines past the wave's share (offset past 2 GiB)
  auto request = [&](int u, int i) {
    const uint32_t at = i < n_mine ? (uint32_t)(w + kSkWaves * i) * 128u : 0x80000000u;
    a[u].template request<2>(ar, a_off + at);  // (non-temporal: a row is one workgroup's alone)
#pragma unroll
    for (int g = 0; g < NG; ++g) b[u][g].template request<0>(xr, b_off + (uint32_t)(16 * g) * row_bytes + at);
  };
  auto multiply = [&](int u) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u].step(s), b[u][g].step(s), acc[g], 0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < PF; ++u) request(u, u);
  __builtin_amdgcn_sched_barrier(0);  // every request before the first product
  const bool in_table = seq >= 0 && seq < p.n_seqs && pos >= 0 && pos < p.max_pages * kPage;
  const int page = in_table ? p.block_table[(size_t)seq * p.max_pages + pos / kPage] : -1;
  __builtin_amdgcn_sched_barrier(0);
  for (int i0 = 0; i0 + PF < n_mine; i0 += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      multiply(u);
      request(u, i0 + PF + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < PF; ++u) multiply(u);
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[w][g][4 * q + j][m] = acc[g][j];  // accumulator: row 4 q + j, token m
  __syncthreads();
  if (page >= 0 && page < p.n_pages) {
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < kSkWaves; ++i) v += red[i][ot >> 4][orow][ot & 15];
    const int j = j0 + orow, slot = pos % kPage;
    uint16_t* dst = p.cache + (size_t)page * p.page_elems;
    dst[j < p.r_k ? k_index(p.r_k, slot, j) : v_index(p.r_k, slot, j - p.r_k)] = bf16_bits(v);
  }
}

// ------------------------------------------------------------------------------------------------ probe
__global__ void stream_read_kernel(const u32x4* __restrict__ src, size_t n16, uint32_t* sink) {
  uint32_t acc = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x) {
    const u32x4 v = __builtin_nontemporal_load(src + i);
    acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
  }
  if (acc == 0x9e3779b9u) sink[0] = acc;  // practically never true: keeps the loads alive without a store
}

// Matrix-core rate probe: every wave issues `iters` x 8 independent 32x32x16 bf16 MFMAs on operands held in registers
// (no memory traffic in the loop).  What it sustains is what the board's power management leaves of the nominal
// peak for this operand data: 0 = pseudo-random sign and mantissa, 1 = zeros, 2 = ones.
__global__ __launch_bounds__(256, 1) void mfma_rate_kernel(float* sink, int iters, int operands) {
  bf16x8 a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u32x4 va, vb;
    uint32_t sa = (uint32_t)threadIdx.x * 9781u + (uint32_t)i * 7u + 1u, sb = (uint32_t)threadIdx.x * 6271u + (uint32_t)i * 13u + 5u + blockIdx.x;
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // xorshift; |x| in [2^-5, 2^-4)
      sa ^= sa << 13; sa ^= sa >> 17; sa ^= sa << 5;
      sb ^= sb << 13; sb ^= sb >> 17; sb ^= sb << 5;
      va[c] = operands == 0 ? ((sa & 0x807f807fu) | 0x3d003d00u) : (operands == 2 ? 0x3f803f80u : 0u);
      vb[c] = operands == 0 ? ((sb & 0x807f807fu) | 0x3d003d00u) : (operands == 2 ? 0x3f803f80u : 0u);
    }
    a[i] = __builtin_bit_cast(bf16x8, va);
    b[i] = __builtin_bit_cast(bf16x8, vb);
  }
  f32x16 acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;
  for (int it = 0; it < iters; ++it)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = mfma32(a[i & 3], b[(i >> 1) & 3], acc[i]);
  float r = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) r += acc[i][j];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = r;
}

int launch_mfma_probe(float* sink, int workgroups, int iters, int operands, hipStream_t s) {
  return launch_kernel(mfma_rate_kernel, dim3(workgroups), dim3(256), 0, s, sink, iters, operands);
}

int launch_pack(const lorc_layer_desc& d, const void* A_k, const void* A_v, const void* B_k, const void* B_v,
                void* packed, hipStream_t s) {
  const int n = d.n_kv_heads * d.head_dim;
  return launch_kernel(pack_factors_kernel, dim3(2048), dim3(256), 0, s, (const uint16_t*)A_k, (const uint16_t*)A_v,
                       (const uint16_t*)B_k, (const uint16_t*)B_v, (uint16_t*)packed, d.d_model, d.rank_k, d.rank_v, n,
                       d.head_dim, d.rope_base);
}

int set_kernel_attributes_append() {
  const void* kernels[] = {reinterpret_cast<const void*>(append_gemm_kernel), reinterpret_cast<const void*>(append_tile_kernel<4, 3, 2>),
                           reinterpret_cast<const void*>(append_tile_kernel<2, 5, 4>), reinterpret_cast<const void*>(append_tile_kernel<2, 2, 4>)};
  for (const void* k : kernels)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return LORC_EHIP;
  return LORC_OK;
}

// Which kernel takes which batch.  Up to 64 tokens the one-pass kernel (at T = 64, against the 64-tile GEMM: 8B rank 512 17.7
// and 23.7 us, 13B rank 2048 29.1 and 32.5, 70B rank 512 32.7 and 40.3).  Beyond, the cheapest of four tile sizes by the
// estimates below: microseconds per 32 of the model dimension, fitted to D 4096 .. 8192, ranks 256 .. 5120, T 65 .. 32768
// (460 sizes measured with every tile, weights in HBM, 130 of them also with weights the caches still hold: the choice is 0.5 %
// behind the best on average).  The 64-tile GEMM needs 0.16 to 0.19 while every CU has at most one workgroup.  Just beyond, it
// depends on the number of token tiles: block ids go to the XCDs in turn, so a multiple of eight gives an XCD the same tokens
// for every row tile (0.28), another number spreads them over all XCDs (0.29 to 0.33).  With up to two per CU, a multiple of
// eight is 10 % faster than 128 x 128 tiles on weights from HBM and 10 % slower on cached ones (8B rank 768, 1000 tokens: 37
// and 41 us, 36 and 34), and another number slower on both, so that the line is drawn at 1.125.  Measured, us, 64 x 64 /
// 128 x 128 / 256 x 128 / 256 x 256 tiles, weights in HBM:
//   8B rank 576: T = 777: 24.5 / 33 / 66 / 102,  900: 37 / 33 / 65 / 102,  1500: 36 / 41 / 77 / 103,  1700: 48 / 36 / 69 / 102,
//     3116: - / 40 / 58 / 98,  6002: - / 67 / 101 / 105,  12288: - / - / 158 / 110,  16384: - / - / 185 / 199;
//   13B rank 2048: T = 300: 56 / 44 / 84 / 130,  777: 64 / 43 / 80 / 128,  3000: - / 144 / 133 / 155,  6002: - / 274 / 246 / 273,
//     8192: - / - / 325 / 278;   13B uncompressed: T = 777: 233 / 136 / 112 / 240,  1500: 327 / 171 / 166 / 241.
// (Sequences whose tokens do not start at a multiple of eight slots store V latents one by one, which costs the 256 x 256 tiles
// up to 15 %; where tokens go is not known here.)
constexpr int kSkinnyMaxT = 64, kSkinnyMinTiles = 32;

static double append_tile_cost(AppendForm form, int rows_k, int rows_v, int T, int n_cus) {
  auto up = [](int x, int y) { return (x + y - 1) / y; };
  if (form == AppendForm::kTile64) {
    const int token_tiles = up(T, 64);
    const double load = (double)token_tiles * up(rows_k + rows_v, 64) / n_cus;  // tiles per CU, here and below
    if (load <= 1) return 0.18;
    if (load > 1.125) return 1e9;
    return token_tiles % 8 == 0 ? 0.285 : 0.34;
  }
  if (form == AppendForm::kTile256) {
    // One workgroup per CU walks rounds of block ids, 0.55 and up to 0.35 more each, by how full it is.  Token tiles come in
    // eights (one per XCD): whole eights first, then ny turns of the `odd` ones.
    const int slots = n_cus / 8 * 8, ny = up(rows_k + rows_v, 256), nx = up(T, 256), odd = nx % 8;
    const long whole = (long)(nx - odd) * ny;
    double cost = 0.9 * (whole / slots);
    long here = whole % slots, left = (long)odd * ny;
    do {
      const long room = (slots - here) / 8 * odd, n = here + (left < room ? left : room);
      if (n > 0) cost += 0.55 + 0.35 * n / slots;
      left -= n - here;
      here = 0;
    } while (left > 0);
    return cost;
  }
  const int rows = form == AppendForm::kTile128 ? 128 : 256;
  const double load = (double)(up(rows_k, rows) + up(rows_v, rows)) * up(T, 128) / n_cus;
  if (form == AppendForm::kTile128) return load <= 1 ? 0.31 : (load <= 2 ? 0.24 + 0.155 * load : (load <= 3.14 ? 0.88 : 0.28 * load));
  return load <= 1 ? 0.36 + 0.18 * load : (load <= 1.58 ? 0.82 : 0.52 * load);
}

// 32 x 32 tiles while there are no more than CUs.  A CU takes about 52 bytes of these operands per ns, with 32 workgroups on the chip
// as with 256, so what counts is the bytes per workgroup: 64 rows of the model dimension instead of 128, or of all tokens in the one-pass
// kernel, which keeps up to 32 tokens (equal there).  us, weights from HBM, before -> now: 8B rank 512 T = 48 14.2 -> 10.3, 64 18.3 -> 10.4, 100
// 20.3 -> 10.4, 256 20.8 -> 13.0; rank 256 T = 500 20.8 -> 11.2; 70B rank 512 T = 64 32.6 -> 17.7; 13B rank 2048 T = 64 28.6 -> 16.9.
// Tried without gain: four groups of waves over the model dimension in a 64 x 64 workgroup (22.3 -> 23.1 at 777 tokens), two in a 128 x 128
// one (28 -> 35 at 900), another first k-tile per workgroup (22.4 -> 28.6).
static bool append_small_tiles(int rows, int T, int n_cus) { return (long)((rows + 31) / 32) * ((T + 31) / 32) <= n_cus; }

AppendForm append_form(int D, int rows_k, int rows_v, int T, int n_cus) {
  const bool small = append_small_tiles(rows_k + rows_v, T, n_cus);
  if (T <= kSkinnyMaxT) {
    // Rows 4 KiB apart (D 2048) cost the 32 x 32 tiles, which read 32 of them side by side, more than the one-pass kernel with few tokens for
    // many rows.  us, one pass / tiles: 4096 rows T = 33 8.6 / 10.9, 48 9.9 / 11.0, 56 11.1 / 11.0; 3072 rows T = 40 8.7 / 9.0, 48 9.4 / 9.2; 2560
    // rows T = 36 8.1 / 8.2, 40 8.5 / 8.2; 2048 rows T = 36 7.5 / 7.4.  4096 rows, T = 33 elsewhere: D 1024 6.8 / 6.3, 3072 12.9 / 10.4, 4096
    // 14.4 / 14.9, 5120 19.5 / 15.4, 8192 25.8 / 29.4.
    const bool few = D == 2048 && 5 * T * n_cus < 70 * n_cus + 12 * (rows_k + rows_v);
    return T > kSkinnyMinTiles && D >= 1024 && small && !few ? AppendForm::kTile64 : AppendForm::kSkinny;
  }
  if (small) return AppendForm::kTile64;
  AppendForm best = AppendForm::kTile64;
  double best_cost = append_tile_cost(best, rows_k, rows_v, T, n_cus);
  for (AppendForm f : {AppendForm::kTile128, AppendForm::kTile256x128, AppendForm::kTile256}) {
    if (f == AppendForm::kTile256 && D / kGmBK < 2) continue;  // its ring wants two k-tiles
    const double cost = append_tile_cost(f, rows_k, rows_v, T, n_cus);
    if (cost < best_cost) best = f, best_cost = cost;
  }
  return best;
}

static unsigned tile_grid(int rows_k, int rows_v, int T, int rows) {  // of append_tile_kernel: eight XCDs' equal shares
  const int tiles = ((rows_k + rows - 1) / rows + (rows_v + rows - 1) / rows) * ((T + 127) / 128);
  return (tiles + 7) / 8 * 8;
}

const char* append_kernel_name(int D, int rows_k, int rows_v, int T, int n_cus) {
  switch (append_form(D, rows_k, rows_v, T, n_cus)) {
    case AppendForm::kSkinny: return "append_skinny_kernel";
    case AppendForm::kTile64: return "append_kernel";
    case AppendForm::kTile128:
      return (int)tile_grid(rows_k, rows_v, T, 128) <= n_cus ? "append_tile_kernel<2, 5, 4>" : "append_tile_kernel<2, 2, 4>";
    case AppendForm::kTile256x128: return "append_tile_kernel<4, 3, 2>";
    default: return "append_gemm_kernel";
  }
}

const char* append_kernel_symbol(int D, int rows_k, int rows_v, int T, int n_cus) {
  if (append_form(D, rows_k, rows_v, T, n_cus) != AppendForm::kTile64) return append_kernel_name(D, rows_k, rows_v, T, n_cus);
  return append_small_tiles(rows_k + rows_v, T, n_cus) ? "append_kernel<32>" : "append_kernel<64>";
}

template <bool R16>
static int launch_skinny(const AppendParams& p, int rows, hipStream_t s) {
  const dim3 grid((p.r_k + p.r_v + rows - 1) / rows), block(64 * kSkWaves);
  if (p.T <= 8) return launch_kernel(append_skinny_kernel<0, R16>, grid, block, 0, s, p, rows);
  if (p.T <= 16) return launch_kernel(append_skinny_kernel<1, R16>, grid, block, 0, s, p, rows);
  if (p.T <= 32) return launch_kernel(append_skinny_kernel<2, R16>, grid, block, 0, s, p, rows);
  if (p.T <= 48) return launch_kernel(append_skinny_kernel<3, R16>, grid, block, 0, s, p, rows);
  return launch_kernel(append_skinny_kernel<4, R16>, grid, block, 0, s, p, rows);
}

int launch_append(const AppendParams& p, int n_cus, hipStream_t s) {
  const int rt = p.r_k + p.r_v;
  switch (append_form(p.D, p.r_k, p.r_v, p.T, n_cus)) {
    case AppendForm::kSkinny: {
      int rows = (rt + n_cus - 1) / n_cus;  // one workgroup per CU while 16 rows each suffice
      if (rows > kSkMaxRows) rows = kSkMaxRows;
      return rows > 8 ? launch_skinny<true>(p, rows, s) : launch_skinny<false>(p, rows, s);
    }
    case AppendForm::kTile64:
    {
      if (append_small_tiles(rt, p.T, n_cus)) return launch_kernel(append_kernel<32>, dim3((p.T + 31) / 32, (rt + 31) / 32), dim3(256), 0, s, p);
      return launch_kernel(append_kernel<64>, dim3((p.T + 63) / 64, (rt + 63) / 64), dim3(256), 0, s, p);
    }
    case AppendForm::kTile128: {
      const dim3 grid(tile_grid(p.r_k, p.r_v, p.T, 128));
      if ((int)grid.x <= n_cus) return launch_kernel(append_tile_kernel<2, 5, 4>, grid, dim3(256), rt_ring_bytes<2, 5, 4>(), s, p);
      return launch_kernel(append_tile_kernel<2, 2, 4>, grid, dim3(256), rt_ring_bytes<2, 2, 4>(), s, p);
    }
    case AppendForm::kTile256x128:
      return launch_kernel(append_tile_kernel<4, 3, 2>, dim3(tile_grid(p.r_k, p.r_v, p.T, 256)), dim3(256), rt_ring_bytes<4, 3, 2>(), s, p);
    default: {
      const int nx = (p.T + kGmBN - 1) / kGmBN, ny = (rt + kGmBM - 1) / kGmBM;
      const int n_virtual = ((nx + 7) / 8) * 8 * ny, slots = (n_cus / 8) * 8;
      return launch_kernel(append_gemm_kernel, dim3(n_virtual < slots ? n_virtual : slots), dim3(256), kGmLdsBytes, s, p);
    }
  }
}

int launch_stream_probe(const void* src, size_t bytes, void* sink, hipStream_t s) {
  return launch_kernel(stream_read_kernel, dim3(256 * 8), dim3(256), 0, s, (const u32x4*)src, bytes / 16, (uint32_t*)sink);
}

}  // namespace lorc

