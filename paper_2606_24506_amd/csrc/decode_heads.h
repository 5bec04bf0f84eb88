// Matrix-core decode path for 64 or 128 query heads per KV head with separate
// K and V rows (MQA / GQA groups, head_dim 128). Per KV byte there are 64 to
// 128 flops, a quarter to a half of what the matrix cores deliver at HBM
// speed, so the kernel must keep both busy: what it avoids is any exchange
// between waves inside the tile loop.
//
// Each of the NW = 8 waves owns 16 query heads from the scores to the output:
// its P values never leave its registers (the two 16-token score accumulators
// are the B operand of the P.V product as they stand, with the token index
// ordered {4q..4q+3, 16+4q..16+4q+3} for lane group q), and its softmax
// state and its 16 x 128 outputs are its own. HW = G / 16 waves form a token
// stream that shares a ring of NSLOT tiles of T = 32 tokens, filled by direct
// non-temporal loads NSLOT - 2 tiles ahead; one barrier per two tiles frees
// their slots. With fewer than 128 heads several streams run side by side: each
// takes KV heads of its own when the model's KV heads are a multiple of the
// stream count, and interleaved tiles otherwise (their softmax states are
// then merged through LDS at the end of the piece).
//
// K and V rows (256 bytes) lie unpadded in LDS with 16-byte chunk g of row r
// at g ^ (2r mod 16), which the direct loads apply through their per-lane
// source addresses: both the K operand reads (16 rows x 16 bytes per lane
// group) and the V transpose reads are then free of bank conflicts.
//
// Measured on 13 MQA-128 and 3 GQA-128:2 requests of 1K-64K tokens (183 MB of
// KV): 42.7 us in one launch (4.3 TB/s; 45.1 with a barrier and a softmax
// update per tile; another 1.6 us less with the two group sizes sharing the
// launch by time), where a workgroup of four waves that
// split scores by heads and P.V by columns, with P and the rescale factors
// going through LDS and two barriers per tile, took 66.5 and 37.4 us in a
// launch per group size (about 4,300 cycles per tile, 512 of them products).
#pragma once

#include "decode_mfma.h"

namespace cp {

typedef unsigned int u32x4h __attribute__((ext_vector_type(4)));

template <int G, int D>
struct HeadsCfg {
  static constexpr int NW = 8, T = 32;
  static constexpr int HW = G / 16;                  // waves of a stream
  static constexpr int NSTREAM = NW / HW;
  static constexpr int ROW = D * 2;                  // bytes of one K or V row
  static constexpr int TILE = 2 * T * ROW;           // K rows, then V rows
  static constexpr int LPW = TILE / 1024 / HW;       // 1 KiB direct loads per wave and tile
  static constexpr int NSLOT = 8 / NSTREAM;          // ring depth of a stream (128 KiB in all)
  static constexpr int KSTEPS = D / 32, NBLK = D / 16;
  static constexpr int OPITCH = D + 8;               // merge area row pitch (floats)
  static constexpr int RING = NSTREAM * NSLOT * TILE;
  static constexpr int MERGE = NSTREAM == 1 ? 0 : NSTREAM * G * OPITCH * 4 + 2 * NSTREAM * G * 4;
  static constexpr int LDS = RING > MERGE ? RING : MERGE;
  static_assert(G == 64 || G == 128, "whole head blocks, one per wave");
  static_assert(D == 128, "rows of 16 chunks");
  static_assert(LPW == 2 || LPW % 4 == 0, "direct loads in groups");
  static_assert(NSLOT >= 4 && NSLOT % 2 == 0 && LDS <= 163840 - 64, "ring depth and LDS budget");
};

// One unit: tokens [sg.tok_begin, sg.tok_end) of a request for KV head sg.hblk
// (or NSTREAM consecutive KV heads, one per stream).
template <int G, int D>
__device__ __forceinline__ void heads_unit(const DecodeArgs &a, const GeomK &gm, const DecReq &rq, const Seg &sg,
                                           char *lds) {
  using C = HeadsCfg<G, D>;
  constexpr int T = C::T;
  const int lane = lane_ids().lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stream = wave / C::HW, hw = wave % C::HW;
  const int col = lane & 15, quad = lane >> 4;
  const int P = gm.page_tokens;  // the host routes only pages of a multiple of 32 tokens here
  const int tpp = P / T;
  const uint32_t slot = sg.slot;
  const bool head_par = gm.hkv % C::NSTREAM == 0;
  const int kvh = head_par ? C::NSTREAM * (int)sg.hblk + stream : (int)sg.hblk;
  const int h0 = kvh * G + 16 * hw;  // first query head of this wave

  const uint32_t tok_begin = sg.tok_begin, tok_end = sg.tok_end;
  const uint32_t pg0 = tok_begin / (uint32_t)P;  // the piece may start inside a page:
  const int off = (int)(tok_begin - pg0 * (uint32_t)P) / T;  // ... by this many tiles
  const int ntiles = (int)((tok_end - tok_begin + T - 1) / T);
  const int first = head_par ? 0 : stream, step = head_par ? 1 : C::NSTREAM;  // this stream's tiles
  const int mine = ntiles > first ? (ntiles - first + step - 1) / step : 0;
  const int most = head_par ? ntiles : (ntiles + C::NSTREAM - 1) / C::NSTREAM;  // tiles of any stream
  const uint64_t kv_head_bytes = (uint64_t)2 * P * C::ROW;
  char *const ring = lds + stream * (C::NSLOT * C::TILE);
  const int npg = (int)((tok_end + P - 1) / P) - (int)pg0;

  // page-table entries of the unit, 64 at a time (lane i: page 64 b + i)
  uint32_t pte_lane = 0;
  int pte_batch = -1;
  auto load_ptes = [&](int batch) {
    const int sp = batch * 64 + lane;
    pte_lane = sp < npg ? a.pte[rq.pte_base + pg0 + (uint32_t)sp] : 0u;
    pte_batch = batch;
    // a visible wait: the tile loads are inline asm the compiler cannot
    // count, so its own wait at the first use would drain them every tile
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  };
  // Direct loads LPW hw .. LPW hw + LPW - 1 of a tile's 16 are this wave's:
  // load j covers four rows, K for j < 8 and V above.
  uint32_t voff[C::LPW];
#pragma unroll
  for (int j = 0; j < C::LPW; ++j) {
    const int ld = C::LPW * hw + j, row = 4 * (ld & 7) + (lane >> 4);
    voff[j] = (uint32_t)((ld < 8 ? 0 : P * C::ROW) + row * C::ROW + 16 * ((lane & 15) ^ ((2 * row) & 15))) + kDmaBias -
              1024u * (j & 3);
  }
  auto issue = [&](int i) {
    const int tl = off + first + step * i, sp = tl / tpp;  // tile, from the unit's first page on, and page
    if ((sp >> 6) != pte_batch) load_ptes(sp >> 6);
    const uint32_t pte = __builtin_amdgcn_readlane(pte_lane, sp & 63);
    const uint64_t sb = uniform_ptr(a.pool + ((uint64_t)pte << 8) + (uint64_t)kvh * kv_head_bytes +
                                    (uint64_t)(tl % tpp) * T * C::ROW - kDmaBias);
    const uint32_t lb = lds_addr(ring + (i % C::NSLOT) * C::TILE) + 1024 * (C::LPW * hw);
    if constexpr (C::LPW == 2) {
      const uint32_t v[4] = {voff[0], voff[1], 0u, 0u};
      dma_group<2>(sb, v, lb);
    } else {
#pragma unroll
      for (int g = 0; g < C::LPW / 4; ++g) {
        const uint32_t v[4] = {voff[4 * g], voff[4 * g + 1], voff[4 * g + 2], voff[4 * g + 3]};
        dma_group<4>(sb, v, lb + 4096 * g);
      }
    }
  };

  // Q^T operand fragments: lane holds head h0 + col, dims 32 c + 8 quad .. +7
  bf16x8 qf[C::KSTEPS];
  {
    const uint16_t *qrow = a.q + rq.q_off + (uint32_t)(h0 + col) * D + 8 * quad;
#pragma unroll
    for (int c = 0; c < C::KSTEPS; ++c) qf[c] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * c);
  }
  float m = -INFINITY, lsum = 0.f;
  f32x4 o[C::NBLK];
#pragma unroll
  for (int nb = 0; nb < C::NBLK; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sl2 = gm.scale_log2;

  load_ptes(0);  // its wait covers the query loads too
  for (int i = 0; i < C::NSLOT - 2 && i < mine; ++i) issue(i);

  // LDS byte offsets within a tile. K fragment of slice u, k-step c: row 16 u
  // + col, chunk 4 c + quad; V^T fragment of column block nb: rows 4 quad +
  // (col >> 2) and 16 more, chunk 2 nb + ((col >> 1) & 1), half col & 1.
  const uint32_t krow = (uint32_t)(col * C::ROW), ksw = (2 * col) & 15;
  const int vr = 4 * quad + (col >> 2);
  const uint32_t vrow = (uint32_t)(T * C::ROW + vr * C::ROW + 8 * (col & 1)), vsw = (2 * vr) & 15;

  // Two tiles (64 tokens) per iteration: one barrier, one softmax update, and
  // twice the independent products and LDS reads to cover their latencies.
#pragma unroll 1
  for (int i = 0; i < most; i += 2) {
    // own loads of tiles i and i + 1 have landed once at most those of the
    // later tiles issued so far (up to tile i + NSLOT - 3) remain
    const int later = mine - 2 - i;
    if (later >= C::NSLOT - 4) wait_vm<C::LPW *(C::NSLOT - 4)>();
    else if (C::NSLOT > 5 && later == 1) wait_vm<C::LPW>();
    else if (C::NSLOT > 6 && later == 2) wait_vm<2 * C::LPW>();
    else if (C::NSLOT > 7 && later == 3) wait_vm<3 * C::LPW>();
    else wait_vm<0>();
    __syncthreads();  // both tiles are visible to the stream; the slots of tiles i-2 and i-1 are free
    if (i + C::NSLOT - 2 < mine) issue(i + C::NSLOT - 2);
    if (i + C::NSLOT - 1 < mine) issue(i + C::NSLOT - 1);
    if (i >= mine) continue;
    // tokens of the two tiles; the second is absent (0) at an odd end
    int valid[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) valid[k] = i + k < mine ? min(T, (int)(tok_end - tok_begin) - (first + step * (i + k)) * T) : 0;

    // ---- scores of the four 16-token slices; each tile's V^T fragments are
    // read behind its K fragments, so that they arrive during the products
    f32x4 s[4];
    bf16x8 vf[2][C::NBLK];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const char *tb = ring + ((i + k) % C::NSLOT) * C::TILE;
      bf16x8 kf[2][C::KSTEPS];
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          kf[u][c] = *reinterpret_cast<const bf16x8 *>(tb + krow + u * 16 * C::ROW + 16 * ((4 * c + quad) ^ ksw));
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb) {
        const char *p0 = tb + vrow + 16 * ((2 * nb + ((col >> 1) & 1)) ^ vsw);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p0);
        const s16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p0 + 16 * C::ROW));
        vf[k][nb] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u) s[2 * k + u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          s[2 * k + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][c], qf[c], s[2 * k + u], 0, 0, 0);
    }

    // ---- online softmax (lane: head col, tokens 16 u + 4 quad + r of a
    // tile). Scores stay unscaled: the positive scale goes onto the maximum
    // and into the exponent's fma. The reference moves when some lane's own
    // maximum passes it by kLazy; only then is the head's maximum taken
    // across lanes.
    if (valid[0] + valid[1] < 2 * T) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (16 * u + 4 * quad + r >= valid[k]) s[2 * k + u][r] = -INFINITY;
        // V rows past the context may hold stale bytes: their p is 0, and the
        // operand's elements are zeroed so that 0 * V stays 0
        u32x4h mask;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int t = 16 * (w >> 1) + 4 * quad + 2 * (w & 1);
          mask[w] = (t < valid[k] ? 0xFFFFu : 0u) | (t + 1 < valid[k] ? 0xFFFF0000u : 0u);
        }
#pragma unroll
        for (int nb = 0; nb < C::NBLK; ++nb)
          vf[k][nb] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4h, vf[k][nb]) & mask);
      }
    }
    float x = s[0][0];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) x = __builtin_fmaxf(x, s[u][r]);
    if (__builtin_amdgcn_ballot_w64(x * sl2 > m + kLazy)) {
      const float mt = xor_max_16_32(x) * sl2;
      const float mn = mt > m + kLazy ? mt : m;
      const float al = fast_exp2(m - mn);
      m = mn;
      lsum *= al;
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb) o[nb] *= al;
    }
    // ---- P (fp32 into the row sum, bf16 as the operand) and O^T += V^T P^T
    float ps = 0.f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      bf16x8 pf;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p = fast_exp2(__builtin_fmaf(s[2 * k + u][r], sl2, -m));
          ps += p;
          pf[4 * u + r] = (__bf16)p;
        }
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb)
        o[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[k][nb], pf, o[nb], 0, 0, 0);
    }
    lsum += ps;
  }

  // ---- unit end
  lsum = xor_sum_16_32(lsum);
  const bool split = rq.ws_base != kNoWs;
  auto write_out = [&](uint32_t head, int d, const f32x4 &v) {
    uint16_t *dst = split ? a.ws_o + ((uint64_t)rq.ws_orow + (uint64_t)slot * gm.hq + head) * D + d
                          : a.out + rq.o_off + head * D + d;
    *reinterpret_cast<uint2 *>(dst) = bf16x4_bits(v[0], v[1], v[2], v[3]);
  };
  auto write_lse = [&](uint32_t head, float lse) {
    if (split)
      a.ws_l[(uint64_t)rq.ws_base + (uint64_t)slot * gm.hq + head] = lse;
    else
      a.lse[rq.lse_off + head] = lse;
  };
  if (C::NSTREAM == 1 || head_par) {
    const float inv = 1.0f / lsum;
    const uint32_t head = (uint32_t)(h0 + col);
#pragma unroll
    for (int nb = 0; nb < C::NBLK; ++nb) write_out(head, 16 * nb + 4 * quad, o[nb] * inv);
    if (quad == 0) write_lse(head, (m + fast_log2(lsum)) * kLn2);
  } else {
    // tiles were split over the streams: merge their softmax states
    float *const macc = reinterpret_cast<float *>(lds);     // [NSTREAM][G][OPITCH]
    float *const m_x = macc + C::NSTREAM * G * C::OPITCH;   // [NSTREAM][G]
    float *const l_x = m_x + C::NSTREAM * G;                // [NSTREAM][G]
    __syncthreads();  // every stream is done with its ring
    const int hh = 16 * hw + col;
    if (quad == 0) {
      m_x[stream * G + hh] = m;
      l_x[stream * G + hh] = lsum;
    }
    __syncthreads();
    float M = -INFINITY;
#pragma unroll
    for (int s2 = 0; s2 < C::NSTREAM; ++s2) M = fmaxf(M, m_x[s2 * G + hh]);
    // a stream without tiles has m = -inf and contributes nothing
    const float f = m == -INFINITY ? 0.f : fast_exp2(m - M);
#pragma unroll
    for (int nb = 0; nb < C::NBLK; ++nb)
      *reinterpret_cast<f32x4 *>(macc + (stream * G + hh) * C::OPITCH + 16 * nb + 4 * quad) = o[nb] * f;
    __syncthreads();
    // normalise and write: thread t takes head t / TPH and the 16-byte
    // column chunks t % TPH + TPH j
    constexpr int TPH = 64 * C::NW / G, NCH = D / 4 / TPH;
    const int wh = threadIdx.x / TPH, ci = threadIdx.x % TPH;
    float Mw = -INFINITY, L = 0.f;
#pragma unroll
    for (int s2 = 0; s2 < C::NSTREAM; ++s2) Mw = fmaxf(Mw, m_x[s2 * G + wh]);
#pragma unroll
    for (int s2 = 0; s2 < C::NSTREAM; ++s2) {
      const float ms = m_x[s2 * G + wh];
      const float l = l_x[s2 * G + wh];
      L += ms == -INFINITY ? (l != l ? l : 0.f) : l * fast_exp2(ms - Mw);  // (all-NaN scores leave m = -inf)
    }
    const float inv = 1.0f / L;
    const uint32_t head = (uint32_t)(kvh * G + wh);
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int d = 4 * (ci + TPH * j);
      f32x4 v = *reinterpret_cast<const f32x4 *>(macc + wh * C::OPITCH + d);
#pragma unroll
      for (int r = 1; r < C::NSTREAM; ++r) v += *reinterpret_cast<const f32x4 *>(macc + (r * G + wh) * C::OPITCH + d);
      write_out(head, d, v * inv);
    }
    if (ci == 0) write_lse(head, (Mw + fast_log2(L)) * kLn2);
  }
  __syncthreads();  // LDS is reused by the next unit
}

}  // namespace cp
