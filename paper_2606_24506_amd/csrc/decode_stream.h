// Matrix-core decode path for the GQA / MHA geometries outside the other
// matrix kernels: any number of query heads per KV head (in units of up to
// 16) with head_dim 64 or 128. At up to 16 heads per KV byte the work is far
// below the matrix cores' rate even padded to 16 head columns, so the kernel
// is all about keeping loads in flight and spending few instructions per
// byte.
//
// Each of the NW = 8 waves is a token stream of its own with a private ring
// of two LDS slots of 8 KiB (K and V of TW tokens), filled by direct
// non-temporal loads, so the loop has no barrier: a wave waits for its slice,
// moves the operand fragments to registers, refills the slot with the slice
// after next, and computes. Two slices per wave, 128 KiB per CU, are in
// flight all the time but for that short read.
//
// HP = min(8, largest power of two dividing the KV heads) KV heads run side
// by side, NT = 8 / HP waves each; the NT waves of a KV head take interleaved
// slices and are merged through LDS at the end of the unit (HP = 8: no
// merge).
//
// P stays a 32-bit quantity: the P.V product takes it as the exact sum of three
// bf16 operands (split_bf16), so the result carries no more rounding than the
// vector kernels (decode_small.h, valu_unit), which multiply in fp32. The further
// products read no further LDS.
//
// LDS rows lie unpadded, 16-byte chunk g of row r at g ^ (2r mod 16) (256-byte
// rows) or g ^ (r & 6) (128-byte rows): the K operand reads and the V
// transpose reads are then free of bank conflicts.
//
// Measured (whole decode calls, KV bytes over time): 16 requests of 32 heads
// on 8 KV heads, 512-32K tokens, 458 MB: 80 us (5.7 TB/s), with the
// small-group vector kernel 122 us (3.8 TB/s; half of its time went to vector
// instructions, about 110 per 32 bytes and lane). 32 requests of four models
// with groups of 1 to 4 heads, head_dim 64 and 128, 235 MB: 45 against 116
// us. The third operand of P costs 0.2% of either.
#pragma once

#include "decode_mfma.h"

namespace cp {

typedef unsigned int u32x4s __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2s __attribute__((ext_vector_type(2)));

template <int D>
struct StreamCfg {
  static constexpr int NW = 8, HEADS = 16;
  static constexpr int ROW = D * 2;              // bytes of one K or V row
  static constexpr int CPR = ROW / 16;           // 16-byte chunks per row
  static constexpr int TW = 4096 / ROW;          // tokens per slice: 16 (D = 128) or 32 (D = 64)
  static constexpr int SLICE = 2 * TW * ROW;     // K rows, then V rows: 8 KiB
  static constexpr int LOADS = SLICE / 1024;     // direct loads per slice
  static constexpr int RPL = 1024 / ROW;         // rows per direct load
  static constexpr int NSLOT = 2;
  static constexpr int KSTEPS = D / 32, NBLK = D / 16, NSL = TW / 16;
  static constexpr int OPITCH = D + 8;           // merge area row pitch (floats)
  static constexpr int RING = NW * NSLOT * SLICE;
  static constexpr int MERGE = NW * HEADS * OPITCH * 4 + 2 * NW * HEADS * 4;
  static constexpr int LDS = RING > MERGE ? RING : MERGE;
  static_assert(D == 64 || D == 128, "head_dim 64 or 128");
  static_assert(SLICE == 8192 && LOADS == 8, "two groups of four loads per slice");
};

// KV heads a workgroup takes side by side.
__host__ __device__ constexpr int stream_heads(int hkv) {
  const int low = hkv & -hkv;
  return low < 8 ? low : 8;
}

// One unit: up to 16 query heads (block hblk % nb) of each of HP consecutive
// KV heads over the pages of one KV range.
template <int D>
__device__ __forceinline__ void stream_unit(const DecodeArgs &a, const GeomK &gm, const DecReq &rq, const Seg &sg,
                                            char *lds) {
  using C = StreamCfg<D>;
  constexpr int TW = C::TW;
  const int lane = lane_ids().lane;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, quad = lane >> 4;
  const int P = gm.page_tokens;  // the host routes only pages of a multiple of TW tokens here
  const int spp = P / TW;
  const int HP = stream_heads(gm.hkv), NT = C::NW / HP;
  const int hp = wave / NT, ts = wave % NT;  // KV head of the unit, token stream of that head
  const int sub = (int)sg.hblk % gm.nb;
  const int kvh = ((int)sg.hblk / gm.nb) * HP + hp;
  const int h0 = kvh * gm.g + sub * C::HEADS;           // first query head of this wave
  const int hv = min(C::HEADS, gm.g - sub * C::HEADS);  // ... and how many it has

  const uint32_t tok_begin = sg.tok_begin, tok_end = sg.tok_end;
  const uint32_t pg0 = tok_begin / (uint32_t)P;  // the piece may start inside a page:
  const int off = (int)(tok_begin - pg0 * (uint32_t)P) / TW;  // ... by this many slices
  const int ntok = (int)(tok_end - tok_begin);
  const int nslices = (ntok + TW - 1) / TW;
  const int mine = nslices > ts ? (nslices - ts + NT - 1) / NT : 0;
  const int npg = (int)((tok_end + P - 1) / P) - (int)pg0;
  char *const ring = lds + wave * (C::NSLOT * C::SLICE);

  // page-table entries of the unit, 64 at a time (lane i: page 64 b + i)
  uint32_t pte_lane = 0;
  int pte_batch = -1;
  auto load_ptes = [&](int batch) {
    const int sp = batch * 64 + lane;
    pte_lane = sp < npg ? a.pte[rq.pte_base + pg0 + (uint32_t)sp] : 0u;
    pte_batch = batch;
    // a visible wait: the slice loads are inline asm the compiler cannot
    // count, so its own wait at the first use would drain them every slice
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
  };
  // per-lane source offsets of the four loads of K (and, P rows further, V)
  uint32_t voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = C::RPL * j + lane / C::CPR, sw = D == 128 ? (2 * row) & 15 : row & 6;
    voff[j] = (uint32_t)(row * C::ROW + 16 * ((lane % C::CPR) ^ sw)) + kDmaBias - 1024u * j;
  }
  auto issue = [&](int i) {
    const int sl = off + ts + NT * i, sp = sl / spp;  // slice, from the unit's first page on, and page
    if ((sp >> 6) != pte_batch) load_ptes(sp >> 6);
    const uint32_t pte = __builtin_amdgcn_readlane(pte_lane, sp & 63);
    const uint64_t sb = uniform_ptr(a.pool + ((uint64_t)pte << 8) + (uint64_t)kvh * (2u * (uint32_t)P * C::ROW) +
                                    (uint64_t)(sl % spp) * TW * C::ROW - kDmaBias);
    const uint32_t lb = lds_addr(ring + (i & 1) * C::SLICE);
    dma_group<4>(sb, voff, lb);
    dma_group<4>(sb + (uint64_t)P * C::ROW, voff, lb + TW * C::ROW);
  };

  // Q^T operand fragments: lane holds head h0 + col, dims 32 c + 8 quad .. +7
  bf16x8 qf[C::KSTEPS];
  {
    const uint16_t *qrow = a.q + rq.q_off + (uint32_t)(h0 + (col < hv ? col : 0)) * D + 8 * quad;
#pragma unroll
    for (int c = 0; c < C::KSTEPS; ++c) qf[c] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * c);
  }
  load_ptes(0);  // its wait covers the query loads too
#pragma unroll
  for (int c = 0; c < C::KSTEPS; ++c)
    if (col >= hv) qf[c] = bf16x8{};
  if (mine > 0) issue(0);
  if (mine > 1) issue(1);

  float m = -INFINITY, lsum = 0.f;
  f32x4 o[C::NBLK];
#pragma unroll
  for (int nb = 0; nb < C::NBLK; ++nb) o[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sl2 = gm.scale_log2;

  // LDS byte offsets within a slot: K fragment of slice half u, k-step c: row
  // 16 u + col, chunk 4 c + quad; V^T fragment of column block nb: row 4 quad
  // + (col >> 2) (and 16 more), chunk 2 nb + ((col >> 1) & 1), half col & 1.
  const uint32_t krow = (uint32_t)(col * C::ROW), ksw = D == 128 ? (2 * col) & 15 : col & 6;
  const int vr = 4 * quad + (col >> 2);
  const uint32_t vrow = (uint32_t)(TW * C::ROW + vr * C::ROW + 8 * (col & 1)), vsw = D == 128 ? (2 * vr) & 15 : vr & 6;

#pragma unroll 1
  for (int i = 0; i < mine; ++i) {
    // own loads of slice i have landed once at most slice i+1's remain
    if (i + 1 < mine) wait_vm<C::LOADS>();
    else wait_vm<0>();
    const char *tb = ring + (i & 1) * C::SLICE;
    bf16x8 kf[C::NSL][C::KSTEPS];
#pragma unroll
    for (int u = 0; u < C::NSL; ++u)
#pragma unroll
      for (int c = 0; c < C::KSTEPS; ++c)
        kf[u][c] = *reinterpret_cast<const bf16x8 *>(tb + krow + u * 16 * C::ROW + 16 * ((4 * c + quad) ^ ksw));
    s16x4 vf[C::NSL][C::NBLK];
#pragma unroll
    for (int nb = 0; nb < C::NBLK; ++nb)
#pragma unroll
      for (int u = 0; u < C::NSL; ++u)
        vf[u][nb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(
            tb + vrow + u * 16 * C::ROW + 16 * ((2 * nb + ((col >> 1) & 1)) ^ vsw)));
    // the fragments are in registers: the slot takes the slice after next
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (i + 2 < mine) issue(i + 2);

    // ---- scores
    f32x4 s[C::NSL];
#pragma unroll
    for (int u = 0; u < C::NSL; ++u) s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C::KSTEPS; ++c)
#pragma unroll
      for (int u = 0; u < C::NSL; ++u) s[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][c], qf[c], s[u], 0, 0, 0);

    // ---- online softmax (lane: head col, tokens 16 u + 4 quad + r). Scores
    // stay unscaled: the positive scale goes onto the maximum and into the
    // exponent's fma. The reference moves when some lane's own maximum
    // passes it by kLazy; only then is the head's maximum taken across lanes.
    const int valid = ntok - (ts + NT * i) * TW;
    if (valid < TW) {
      // rows past the context may hold stale bytes: their p is 0, and their
      // V elements are zeroed so that 0 * V stays 0
#pragma unroll
      for (int u = 0; u < C::NSL; ++u) {
        const int t = 16 * u + 4 * quad;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t + r >= valid) s[u][r] = -INFINITY;
        const u32x2s mask = {(t < valid ? 0xFFFFu : 0u) | (t + 1 < valid ? 0xFFFF0000u : 0u),
                             (t + 2 < valid ? 0xFFFFu : 0u) | (t + 3 < valid ? 0xFFFF0000u : 0u)};
#pragma unroll
        for (int nb = 0; nb < C::NBLK; ++nb)
          vf[u][nb] = __builtin_bit_cast(s16x4, __builtin_bit_cast(u32x2s, vf[u][nb]) & mask);
      }
    }
    float x = s[0][0];
#pragma unroll
    for (int u = 0; u < C::NSL; ++u)
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
    // ---- P = hi + mid + lo (bf16 each), O^T += V^T hi^T + V^T mid^T + V^T lo^T
    float ps = 0.f;
    uint32_t pw[3][2 * C::NSL];  // two values each
#pragma unroll
    for (int u = 0; u < C::NSL; ++u)
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
    if constexpr (C::NSL == 1) {
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const s16x4 ph = __builtin_bit_cast(s16x4, u32x2s{pw[h][0], pw[h][1]});
#pragma unroll
        for (int nb = 0; nb < C::NBLK; ++nb)
          o[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[0][nb], ph, o[nb], 0, 0, 0);
      }
    } else {
      // token index ordered {4q..4q+3, 16+4q..16+4q+3} for lane group q
      constexpr int N1 = 2 * C::NSL - 2;
      bf16x8 vv[C::NBLK];
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb)
        vv[nb] = __builtin_bit_cast(
            bf16x8, __builtin_shufflevector(vf[0][nb], vf[C::NSL - 1][nb], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4s{pw[h][0], pw[h][1], pw[h][N1], pw[h][N1 + 1]});
#pragma unroll
        for (int nb = 0; nb < C::NBLK; ++nb) o[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv[nb], ph, o[nb], 0, 0, 0);
      }
    }
  }

  // ---- unit end
  lsum = xor_sum_16_32(lsum);
  const bool split = rq.ws_base != kNoWs;
  const uint32_t slot = sg.slot;
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
  if (NT == 1) {
    // the wave owns its KV head
    if (col < hv) {
      const float inv = 1.0f / lsum;
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb) write_out((uint32_t)(h0 + col), 16 * nb + 4 * quad, o[nb] * inv);
      if (quad == 0) write_lse((uint32_t)(h0 + col), (m + fast_log2(lsum)) * kLn2);
    }
  } else {
    float *const macc = reinterpret_cast<float *>(lds);       // [NW][HEADS][OPITCH]
    float *const m_x = macc + C::NW * C::HEADS * C::OPITCH;   // [NW][HEADS]
    float *const l_x = m_x + C::NW * C::HEADS;                // [NW][HEADS]
    __syncthreads();  // every wave is done with its ring
    if (quad == 0) {
      m_x[wave * C::HEADS + col] = m;
      l_x[wave * C::HEADS + col] = lsum;
    }
    if (col < hv) {
#pragma unroll
      for (int nb = 0; nb < C::NBLK; ++nb)
        *reinterpret_cast<f32x4 *>(macc + (wave * C::HEADS + col) * C::OPITCH + 16 * nb + 4 * quad) = o[nb];
    }
    __syncthreads();
    // item: (KV head of the unit, query head, 16-byte column chunk)
    constexpr int CH = D / 4;
    for (int t = threadIdx.x; t < HP * hv * CH; t += 64 * C::NW) {
      const int d = 4 * (t % CH), h = (t / CH) % hv, k = t / (CH * hv);
      float M = -INFINITY, L = 0.f;
      for (int w = k * NT; w < (k + 1) * NT; ++w) M = fmaxf(M, m_x[w * C::HEADS + h]);
      f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int w = k * NT; w < (k + 1) * NT; ++w) {
        const float mw = m_x[w * C::HEADS + h];
        const float f = mw == -INFINITY ? 0.f : fast_exp2(mw - M);  // a wave without slices adds nothing
        L += l_x[w * C::HEADS + h] * f;
        v += *reinterpret_cast<const f32x4 *>(macc + (w * C::HEADS + h) * C::OPITCH + d) * f;
      }
      const uint32_t head = (uint32_t)((((int)sg.hblk / gm.nb) * HP + k) * gm.g + sub * C::HEADS + h);
      write_out(head, d, v * (1.0f / L));
      if (d == 0) write_lse(head, (M + fast_log2(L)) * kLn2);
    }
  }
  __syncthreads();  // LDS is reused by the next unit
}

}  // namespace cp
