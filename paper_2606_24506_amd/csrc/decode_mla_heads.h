// Matrix-core decode path for MLA models (512 + 64 wide latent rows) with 17
// to 64 query heads, or any other number above that in units of up to 64:
// shards of a 128-head model, and head counts that are no power of two.
// At 32 to 64 heads the work is 60 to 120 flops per KV byte: a quarter to a
// half of the matrix cores' rate at HBM speed.
//
// The eight waves work in pairs: a pair owns 16 query heads, both of its
// waves compute their scores (so P stays in the registers it is computed in
// and nothing crosses waves inside the loop) and each accumulates P.V for
// half of the 512 value columns. HS pairs (HS = 2: up to 32 heads, HS = 4: up
// to 64) share one token stream, a ring of NSLOT tiles of T = 32 tokens that
// direct non-temporal loads fill NSLOT - 1 tiles ahead; one barrier per tile
// frees a slot. With HS = 2 two streams take alternate tiles and are merged
// through LDS at the end of the unit. Scoring twice costs matrix time that is
// free here; splitting the scores instead would put P through LDS behind a
// second barrier.
//
// P stays a 32-bit quantity: P.V takes it as the exact sum of three bf16 operands
// (split_bf16), because these head counts otherwise run on the vector kernel,
// which multiplies in fp32.
//
// LDS rows are unpadded: 16-byte chunk g of row r at g ^ (2r mod 16) in a
// value row (1024 bytes) and at g ^ (r & 6) in a rotary row (128 bytes), free
// of bank conflicts for the K operand reads and the V transpose reads.
//
// Measured (whole decode calls, 16 requests of 1K-32K tokens, 160 MB of KV):
// 20 heads 44 us, 32 heads 49 us (two units of 16 heads reading the KV twice:
// 73 us), 64 heads 66 us (2.4 TB/s); the generic vector kernel took 1,650 us
// with 20 heads and 3,380 us with 64. With two operands for P (2^-16 of it left
// out, which shows where V cancels) 43, 47 and 61 us.
#pragma once

#include "decode_mla.h"

namespace cp {

typedef unsigned int u32x4m __attribute__((ext_vector_type(4)));

template <int HS>
struct MlaHeadsCfg {
  static constexpr int NW = 8, T = 32, HEADS = 16 * HS;
  static constexpr int DK = 576, DV = 512;
  static constexpr int KROW = DK * 2, MROW = DV * 2, RROW = KROW - MROW;
  static constexpr int WPS = 2 * HS;                  // waves of a stream
  static constexpr int NSTREAM = NW / WPS;
  static constexpr int NSLOT = 4 / NSTREAM;
  static constexpr int TILE = T * KROW;               // value rows, then rotary rows: 36 KiB
  static constexpr int VLW = T / WPS;                 // value rows (1 KiB loads) per wave and tile
  static constexpr int LPT = VLW + 1;                 // ... and one rotary load
  static constexpr int KMAIN = DV / 32, KSTEPS = DK / 32;
  static constexpr int NBW = DV / 16 / 2;             // value column blocks per wave
  static constexpr int OPITCH = DV + 8;               // merge area row pitch (floats)
  static constexpr int RING = NSTREAM * NSLOT * TILE;
  static constexpr int MERGE = NSTREAM == 1 ? 0 : NSTREAM * HEADS * OPITCH * 4 + 2 * NSTREAM * HEADS * 4;
  static constexpr int LDS = RING > MERGE ? RING : MERGE;
  static_assert(HS == 2 || HS == 4, "two streams or one");
  static_assert(VLW % 4 == 0 && LDS <= 163840 - 64, "load groups and LDS budget");
};

// One unit: up to HEADS query heads (block sg.hblk) over the pages of one KV
// range.
template <int HS>
__device__ __forceinline__ void mla_heads_unit(const DecodeArgs &a, const GeomK &gm, const DecReq &rq, const Seg &sg,
                                               char *lds) {
  using C = MlaHeadsCfg<HS>;
  constexpr int T = C::T;
  const int lane = lane_ids().lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stream = wave % C::NSTREAM, wis = wave / C::NSTREAM;  // wave within the stream
  const int member = wis & 1, pair = wis >> 1;
  const int col = lane & 15, quad = lane >> 4;
  const int P = gm.page_tokens;  // the host routes only pages of a multiple of 32 tokens here
  const int tpp = P / T;
  const int u0 = (int)sg.hblk * C::HEADS;            // first query head of the unit
  const int uv = min(C::HEADS, gm.g - u0);           // ... and how many it has
  const int h0 = u0 + 16 * pair;                     // first head of this wave
  const int hv = min(16, gm.g - h0);                 // its valid heads (none or fewer when padded)
  const int nb0 = member * C::NBW;                   // first value column block of this wave

  const uint32_t tok_begin = sg.tok_begin, tok_end = sg.tok_end;
  const uint32_t pg0 = tok_begin / (uint32_t)P;  // the piece may start inside a page:
  const int off = (int)(tok_begin - pg0 * (uint32_t)P) / T;  // ... by this many tiles
  const int ntok = (int)(tok_end - tok_begin);
  const int ntiles = (ntok + T - 1) / T;
  const int mine = ntiles > stream ? (ntiles - stream + C::NSTREAM - 1) / C::NSTREAM : 0;
  const int iters = (ntiles + C::NSTREAM - 1) / C::NSTREAM;  // the same in every wave
  const int npg = (int)((tok_end + P - 1) / P) - (int)pg0;
  char *const ring = lds + stream * (C::NSLOT * C::TILE);

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
  // This wave loads value rows VLW wis .. + VLW - 1 of a tile (a KiB each) and
  // as many rotary rows (one load; half its lanes when VLW = 4).
  auto issue = [&](int i) {
    const int tl = off + stream + C::NSTREAM * i, sp = tl / tpp;  // tile, from the unit's first page on, and page
    if ((sp >> 6) != pte_batch) load_ptes(sp >> 6);
    const uint32_t pte = __builtin_amdgcn_readlane(pte_lane, sp & 63);
    const uint64_t sb = uniform_ptr(a.pool + ((uint64_t)pte << 8) + (uint64_t)(tl % tpp) * T * C::KROW - kDmaBias);
    const uint32_t lb = lds_addr(ring + (i % C::NSLOT) * C::TILE);
    const int lane = lane_ids().lane;  // counted afresh: the offsets are formed here, not kept through the loop
#pragma unroll
    for (int g = 0; g < C::VLW / 4; ++g) {
      uint32_t vo[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = C::VLW * wis + 4 * g + q;
        vo[q] = (uint32_t)(r * C::KROW + 16 * (lane ^ mla_vswz(r))) + kDmaBias - 1024u * q;
      }
      dma_group<4>(sb, vo, lb + (uint32_t)(C::VLW * wis + 4 * g) * C::MROW);
    }
    if (lane < C::VLW * 8) {
      const int r = C::VLW * wis + (lane >> 3);
      const uint32_t vo[4] = {(uint32_t)(r * C::KROW + C::MROW + 16 * ((lane & 7) ^ mla_rswz(r))) + kDmaBias, 0u, 0u,
                              0u};
      dma_group<1>(sb, vo, lb + T * C::MROW + (uint32_t)(C::VLW * wis) * C::RROW);
    }
  };

  // Q^T operand fragments: lane holds head h0 + col, dims 32 c + 8 quad .. +7
  bf16x8 qf[C::KSTEPS];
  {
    const uint16_t *qrow = a.q + rq.q_off + (uint32_t)(col < hv ? h0 + col : u0) * C::DK + 8 * quad;
#pragma unroll
    for (int c = 0; c < C::KSTEPS; ++c) qf[c] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * c);
  }
  load_ptes(0);  // its wait covers the query loads too
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c) {
    if (col >= hv) qf[c] = bf16x8{};
    // kept in the accumulation registers, which the matrix cores read as they are
    asm volatile("" : "+a"(qf[c]));
  }
  for (int i = 0; i < C::NSLOT - 1 && i < mine; ++i) issue(i);

  float m = -INFINITY, lsum = 0.f;
  f32x4 o[C::NBW];
#pragma unroll
  for (int nb = 0; nb < C::NBW; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sl2 = gm.scale_log2;

  // LDS byte offsets within a slot: the K fragment of slice half u, value
  // k-step 4a + b sits at kva[b] + 256 a + u 16 MROW, rotary k-step c at kra ^
  // (64 c) + u 16 RROW; the V^T fragment of column block nb at vrow + 16 ((2
  // nb + ((col >> 1) & 1)) ^ vsw), and 16 rows further.
  uint32_t kva[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
    kva[b] = (uint32_t)(col * C::MROW + 64 * (b ^ (mla_vswz(col) >> 2)) + 16 * (quad ^ (mla_vswz(col) & 3)));
  const uint32_t kra = (uint32_t)(col * C::RROW + 64 * (mla_rswz(col) >> 2) + 16 * (quad ^ (mla_rswz(col) & 3)));
  const int vr = 4 * quad + (col >> 2);
  const uint32_t vrow = (uint32_t)(vr * C::MROW + 8 * (col & 1)), vsw = (uint32_t)mla_vswz(vr);

#pragma unroll 1
  for (int i = 0; i < iters; ++i) {
    // own loads of tile i have landed once at most the later tiles' remain
    const int later = mine - 1 - i;
    if (later >= C::NSLOT - 2) wait_vm<C::LPT *(C::NSLOT - 2)>();
    else if (C::NSLOT > 3 && later == 1) wait_vm<C::LPT>();
    else wait_vm<0>();
    __syncthreads();  // tile i is visible to the stream; the slot of tile i-1 is free
    if (i + C::NSLOT - 1 < mine) issue(i + C::NSLOT - 1);
    if (i >= mine) continue;
    char *tb = ring + (i % C::NSLOT) * C::TILE;
    const int valid = ntok - (stream + C::NSTREAM * i) * T;
    if (valid < T) {
      // value rows past the context may hold stale bytes: this wave zeroes
      // the columns it multiplies (other waves write the same zeros), so that
      // 0 * V stays 0; the scores of those rows are masked below
      constexpr int CH = C::NBW * 2;
      for (int z = lane; z < (T - valid) * CH; z += 64) {
        const int row = valid + z / CH, g = 2 * nb0 + z % CH;
        *reinterpret_cast<uint4 *>(tb + row * C::MROW + 16 * (g ^ mla_vswz(row))) = make_uint4(0, 0, 0, 0);
      }
    }

    // ---- scores of both 16-token halves: fragments read KD k-steps ahead
    f32x4 s[2];
    s[0] = s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
      constexpr int KD = 3;
      bf16x8 kf[KD + 1][2];
      auto kread = [&](int c, int u) -> bf16x8 {
        const uint32_t ad = c < C::KMAIN ? kva[c & 3] + 256 * (c >> 2) + u * 16 * C::MROW
                                         : T * C::MROW + (kra ^ (64 * (c - C::KMAIN))) + u * 16 * C::RROW;
        return *reinterpret_cast<const bf16x8 *>(tb + ad);
      };
#pragma unroll
      for (int c = 0; c < KD; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u) kf[c][u] = kread(c, u);
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c) {
        if (c + KD < C::KSTEPS) {
#pragma unroll
          for (int u = 0; u < 2; ++u) kf[(c + KD) % (KD + 1)][u] = kread(c + KD, u);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 2; ++u)
          s[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c % (KD + 1)][u], qf[c], s[u], 0, 0, 0);
      }
    }
    // V^T fragments in batches of VB column blocks, the next batch read while
    // this one feeds the matrix cores; the first arrives during the softmax
    constexpr int VB = 4;
    bf16x8 vf[2][VB];
    auto vread = [&](int nb) -> bf16x8 {
      const char *p0 = tb + vrow + 16 * ((2 * (nb0 + nb) + ((col >> 1) & 1)) ^ vsw);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p0);
      const s16x4 hi =
          __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p0 + 16 * C::MROW));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
#pragma unroll
    for (int j = 0; j < VB; ++j) vf[0][j] = vread(j);
    __builtin_amdgcn_sched_barrier(0);

    // ---- online softmax (lane: head col, tokens 16 u + 4 quad + r); the
    // reference moves when some lane's own maximum passes it by kLazy
    if (valid < T) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (16 * u + 4 * quad + r >= valid) s[u][r] = -INFINITY;
    }
    float x = s[0][0];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) x = __builtin_fmaxf(x, s[u][r]);
    if (__builtin_amdgcn_ballot_w64(x * sl2 > m + kLazy)) {
      const float mt = xor_max_16_32(x) * sl2;
      const float mn = mt > m + kLazy ? mt : m;
      const float al = fast_exp2(m - mn);
      m = mn;
      lsum *= al;
#pragma unroll
      for (int nb = 0; nb < C::NBW; ++nb) o[nb] *= al;
    }
    // ---- P = hi + mid + lo (bf16 each), O^T += V^T hi^T + V^T mid^T + V^T lo^T,
    // with the token index ordered {4q..4q+3, 16+4q..16+4q+3} for lane group q
    u32x4m pw[3];
    float ps = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        Bf16Parts x[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float p = fast_exp2(__builtin_fmaf(s[u][r + e], sl2, -m));
          ps += p;
          x[e] = split_bf16(p);
        }
        pw[0][2 * u + r / 2] = upper_halves(x[0].hi, x[1].hi);
        pw[1][2 * u + r / 2] = upper_halves(x[0].mid, x[1].mid);
        pw[2][2 * u + r / 2] = upper_halves(x[0].lo, x[1].lo);
      }
    lsum += ps;
#pragma unroll
    for (int b = 0; b < C::NBW / VB; ++b) {
      if (b + 1 < C::NBW / VB) {
#pragma unroll
        for (int j = 0; j < VB; ++j) vf[(b + 1) & 1][j] = vread((b + 1) * VB + j);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < 3; ++h)
#pragma unroll
        for (int j = 0; j < VB; ++j)
          o[b * VB + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[b & 1][j], __builtin_bit_cast(bf16x8, pw[h]),
                                                                  o[b * VB + j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- unit end
  lsum = xor_sum_16_32(lsum);
  const bool split = rq.ws_base != kNoWs;
  const uint32_t slot = sg.slot;
  auto write_out = [&](uint32_t head, int d, const f32x4 &v) {
    uint16_t *dst = split ? a.ws_o + ((uint64_t)rq.ws_orow + (uint64_t)slot * gm.hq + head) * C::DV + d
                          : a.out + rq.o_off + head * C::DV + d;
    *reinterpret_cast<uint2 *>(dst) = bf16x4_bits(v[0], v[1], v[2], v[3]);
  };
  auto write_lse = [&](uint32_t head, float lse) {
    if (split)
      a.ws_l[(uint64_t)rq.ws_base + (uint64_t)slot * gm.hq + head] = lse;
    else
      a.lse[rq.lse_off + head] = lse;
  };
  if constexpr (C::NSTREAM == 1) {
    if (col < hv) {
      const float inv = 1.0f / lsum;
#pragma unroll
      for (int nb = 0; nb < C::NBW; ++nb) write_out((uint32_t)(h0 + col), 16 * (nb0 + nb) + 4 * quad, o[nb] * inv);
      if (member == 0 && quad == 0) write_lse((uint32_t)(h0 + col), (m + fast_log2(lsum)) * kLn2);
    }
  } else {
    // tiles were split over the streams: merge their softmax states
    float *const macc = reinterpret_cast<float *>(lds);          // [NSTREAM][HEADS][OPITCH]
    float *const m_x = macc + C::NSTREAM * C::HEADS * C::OPITCH; // [NSTREAM][HEADS]
    float *const l_x = m_x + C::NSTREAM * C::HEADS;              // [NSTREAM][HEADS]
    __syncthreads();  // every stream is done with its ring
    const int hh = 16 * pair + col;
    if (member == 0 && quad == 0) {
      m_x[stream * C::HEADS + hh] = m;
      l_x[stream * C::HEADS + hh] = lsum;
    }
    if (col < hv) {
#pragma unroll
      for (int nb = 0; nb < C::NBW; ++nb)
        *reinterpret_cast<f32x4 *>(macc + (stream * C::HEADS + hh) * C::OPITCH + 16 * (nb0 + nb) + 4 * quad) = o[nb];
    }
    __syncthreads();
    constexpr int CH = C::DV / 4;  // 16-byte column chunks of a head
    for (int t = threadIdx.x; t < uv * CH; t += 64 * C::NW) {
      const int h = t / CH, d = 4 * (t % CH);
      float M = -INFINITY, L = 0.f;
#pragma unroll
      for (int s2 = 0; s2 < C::NSTREAM; ++s2) M = fmaxf(M, m_x[s2 * C::HEADS + h]);
      f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2 = 0; s2 < C::NSTREAM; ++s2) {
        const float ms = m_x[s2 * C::HEADS + h];
        const float f = ms == -INFINITY ? 0.f : fast_exp2(ms - M);  // a stream without tiles adds nothing
        L += l_x[s2 * C::HEADS + h] * f;
        v += *reinterpret_cast<const f32x4 *>(macc + (s2 * C::HEADS + h) * C::OPITCH + d) * f;
      }
      write_out((uint32_t)(u0 + h), d, v * (1.0f / L));
      if (d == 0) write_lse((uint32_t)(u0 + h), (M + fast_log2(L)) * kLn2);
    }
  }
  __syncthreads();  // LDS is reused by the next unit
}

}  // namespace cp
