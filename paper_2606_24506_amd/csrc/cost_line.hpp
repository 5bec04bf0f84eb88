// The balanced schedule's plan of one launch: its requests' KV laid on one
// cost line, which is cut into equal shares, one per workgroup. Host only.
// The kernels find their pieces from the same numbers (next_balanced in
// schedule.h).
#pragma once

#include <algorithm>
#include <cstdint>

#include "kargs.h"

namespace cp {

// One request of a launch.
struct LineReq {
  int64_t tokens;        // attended context, >= 1
  int32_t page_tokens;
  int32_t step_tokens;   // tokens its kernel works through in one step, 0: whole pages only
  int32_t kappa;         // KV bytes per token
  int32_t rereads;       // times every KV byte is read (head blocks)
  int32_t weight;        // time per KiB, in units of 1 / kTimeWeightUnit
  uint32_t out_elems;    // outputs: a range of a split request writes as many partial ones
};
constexpr int32_t kTimeWeightUnit = 8;

// Ranges cut inside pages hold no less than this (one MLA page of 64
// tokens), or a page of models with smaller ones.
constexpr uint64_t kMinRangeKib = 72;

// The requests of a launch (its arguments hold no more).
struct LineReqs {
  LineReq r[kMaxReqPerLaunch];
  int n = 0;
};

// A cut line: block j of request i (blk_tokens[i] tokens, blocks[i] of them)
// sits at cost position begin[i] + j blk_cost[i]; share w of `workers` is
// [floor(w total / workers), floor((w + 1) total / workers)). first, ranges:
// the first share a request meets, and how many. Arrays, not vectors: a line
// is laid on the path of every call, for small batches twice.
struct Line {
  int32_t blk_tokens[kMaxReqPerLaunch], blk_cost[kMaxReqPerLaunch], first[kMaxReqPerLaunch], ranges[kMaxReqPerLaunch];
  uint32_t blocks[kMaxReqPerLaunch];
  uint64_t begin[kMaxReqPerLaunch];
  uint64_t total = 0;
  uint32_t workers = 0;
  bool finer = false;  // cut inside pages, or shared by time
};

// Lays out blocks of the given sizes and costs. Every workgroup pays the
// fixed cost of its first piece, so the line charges `fixed` only where a
// request boundary falls inside a workgroup's share (that workgroup runs a
// second piece): not before the first request, and not at a boundary that
// coincides with a share boundary of the line without fixed costs (equal
// requests over a multiple of their count of workgroups). `least`: no share
// is smaller, and it is at least every block's cost, so that no request has
// an empty share between its first and last one.
inline void lay_line(int n, uint64_t fixed, uint64_t least, uint64_t slots, Line *ln) {
  uint64_t T0 = 0;
  for (int i = 0; i < n; ++i) T0 += (uint64_t)ln->blocks[i] * (uint64_t)ln->blk_cost[i];
  const uint64_t W0 = std::max<uint64_t>(1, std::min(slots, T0 / least));
  uint64_t T = 0, pre0 = 0;
  for (int i = 0; i < n; ++i) {
    const bool straddled = i > 0 && (pre0 * W0) % T0 != 0;
    T += straddled ? fixed : 0;
    ln->begin[i] = T;
    T += (uint64_t)ln->blocks[i] * (uint64_t)ln->blk_cost[i];
    pre0 += (uint64_t)ln->blocks[i] * (uint64_t)ln->blk_cost[i];
  }
  const uint64_t W = std::max<uint64_t>(1, std::min(slots, T / least));
  auto owner = [&](uint64_t x) { return (int32_t)(((x + 1) * W - 1) / T); };
  for (int i = 0; i < n; ++i) {
    ln->first[i] = owner(ln->begin[i]);
    ln->ranges[i] = owner(ln->begin[i] + (uint64_t)(ln->blocks[i] - 1) * (uint64_t)ln->blk_cost[i]) - ln->first[i] + 1;
  }
  ln->total = T;
  ln->workers = (uint32_t)W;
}

// Ranges of whole pages, shared by bytes. The line counts units of 8 KiB where
// every page is a multiple of that, else KiB (in units of 8 a 36 KiB page would
// count 11% too much beside one of 32). Shares are floored at whole units, so
// the unit decides which page a share ends at, and with it the bits of the
// results: it stays what it is for the pages of 64 tokens of every model.
inline void whole_page_line(const LineReqs &rs, uint64_t slots, Line *ln) {
  int64_t unit = 8192;
  for (int i = 0; i < rs.n; ++i)
    if ((int64_t)rs.r[i].page_tokens * rs.r[i].kappa % unit) unit = 1024;
  uint64_t least = 1;
  for (int i = 0; i < rs.n; ++i) {
    const LineReq &r = rs.r[i];
    ln->blk_tokens[i] = r.page_tokens;
    ln->blocks[i] = (uint32_t)((r.tokens + r.page_tokens - 1) / r.page_tokens);
    ln->blk_cost[i] = (int32_t)(((int64_t)r.page_tokens * r.kappa + unit - 1) / unit * r.rereads);
    least = std::max(least, (uint64_t)ln->blk_cost[i]);
  }
  ln->finer = false;
  lay_line(rs.n, kPieceFixedCost * 1024 / (uint64_t)unit, least, slots, ln);
}

// Pages of more than 128 KiB are cut where the kernel ends a step (six
// requests of groups of 1 to 4 heads, 128-1024 tokens, 64-token pages of 128
// and 256 KiB: 14.4 us a call against 19.4 with whole pages; cutting 32 to 128
// KiB pages too gained nothing and cost 1 to 4% on batches that small, by more
// partials).
inline bool cut_inside_pages(const LineReq &r) {
  return (int64_t)r.page_tokens * r.kappa > (128 << 10) && r.step_tokens > 0 && r.page_tokens % r.step_tokens == 0 &&
         r.step_tokens < r.page_tokens;
}

// Ranges that end inside large pages; the line counts KiB. Where models of
// different time per KiB share a launch that fills every workgroup, it counts
// time; smaller launches are bound by their ranges' latency and stay cut as
// finely as the blocks allow. False where the line would not fit.
inline bool fine_line(const LineReqs &rs, uint64_t slots, Line *ln) {
  uint64_t least = 1, least_w = 1, Tw = 0, T = 0;
  int32_t wmin = 1 << 30, wmax = 0;
  for (int i = 0; i < rs.n; ++i) {
    const LineReq &r = rs.r[i];
    const int32_t blk = cut_inside_pages(r) ? r.step_tokens : r.page_tokens;
    const uint64_t c = (uint64_t)(((int64_t)blk * r.kappa + 1023) / 1024 * r.rereads);
    const uint64_t page = c * (uint64_t)(r.page_tokens / blk);
    // a range spans at least a block of every model, and a page of those
    // whose pages are smaller than kMinRangeKib (splitting further makes
    // more partials without shortening the launch)
    const uint64_t l = std::max(c, std::min<uint64_t>(page, kMinRangeKib));
    ln->blk_tokens[i] = blk;
    ln->blocks[i] = (uint32_t)((r.tokens + blk - 1) / blk);
    ln->blk_cost[i] = (int32_t)c;
    least = std::max(least, l);
    least_w = std::max(least_w, l * (uint64_t)r.weight);
    T += ln->blocks[i] * c;
    Tw += ln->blocks[i] * c * (uint64_t)r.weight;
    wmin = std::min(wmin, r.weight);
    wmax = std::max(wmax, r.weight);
  }
  uint64_t fixed = kPieceFixedCost;
  if (wmin != wmax && Tw / least_w >= slots && Tw < (1ull << 31)) {
    for (int i = 0; i < rs.n; ++i) ln->blk_cost[i] *= rs.r[i].weight;
    fixed *= kTimeWeightUnit;
    least = least_w;
  } else if (T >= (1ull << 31)) {
    return false;
  }
  ln->finer = true;
  lay_line(rs.n, fixed, least, slots, ln);
  return true;
}

// What a line's launch is expected to take: the longest share, in byte-times
// (a byte of a model of weight kTimeWeightUnit takes that many), with the fixed
// cost of every piece; the outputs of its split requests, and their partials.
struct LineTime {
  uint64_t longest = 0, partials = 0, split = 0;
};
inline LineTime line_time(const LineReqs &rs, const Line &ln) {
  LineTime t;
  const uint64_t q = ln.total / ln.workers, rm = ln.total % ln.workers;
  uint64_t share = 0;  // of share `at`; requests lie on the line in order
  uint64_t end = q, acc = rm;  // its end: floor((at + 1) total / workers), and the remainder
  int32_t at = 0;
  auto next = [&] {
    ++at;
    end += q;
    acc += rm;
    if (acc >= ln.workers) {
      acc -= ln.workers;
      ++end;
    }
  };
  for (int i = 0; i < rs.n; ++i) {
    const LineReq &r = rs.r[i];
    const uint64_t tok_time = (uint64_t)r.kappa * (uint64_t)r.rereads * (uint64_t)r.weight;
    // x / blk_cost by multiplication: exact for x below 2^32, but for a cost of 1
    const uint64_t c = (uint64_t)ln.blk_cost[i], inv = ~0ull / c + 1;
    uint32_t j = 0;
    for (int32_t k = 0; k < ln.ranges[i]; ++k) {
      if (ln.first[i] + k != at) {
        t.longest = std::max(t.longest, share);
        share = 0;
        while (ln.first[i] + k != at) next();
      }
      uint32_t je = ln.blocks[i];
      if (k + 1 < ln.ranges[i]) {
        const uint64_t x = end - ln.begin[i] + c - 1;
        je = (uint32_t)(c == 1 ? x : ((unsigned __int128)x * inv) >> 64);
      }
      const int64_t toks = std::min<int64_t>(r.tokens, (int64_t)je * ln.blk_tokens[i]) - (int64_t)j * ln.blk_tokens[i];
      share += (uint64_t)toks * tok_time + (uint64_t)kPieceFixedCost * 1024 * kTimeWeightUnit;
      j = je;
    }
    if (ln.ranges[i] > 1) {
      t.partials += (uint64_t)ln.ranges[i] * r.out_elems;
      t.split += r.out_elems;
    }
  }
  t.longest = std::max(t.longest, share);
  return t;
}

// The line of a launch: of whole pages, unless some model's pages can be cut or
// the models' times per KiB differ and the finer line is the better one: its
// longest share shorter by more than its further partials cost a workgroup
// (two bytes each, written and read back by the merge). Where blocks are half
// a page and a workgroup has less than a page, finer ranges only add partials
// or leave some workgroups two pieces: MLA-16, 128-token pages (144 KiB; us a
// call of whole pages, always finer): 30 requests of 32K tokens in all 22.1,
// 26.0; 16 of 18K 17.8, 19.0; but 16 of 32K 22.4, 21.1. GQA-64:8, 8 requests of
// 16K tokens: 25.5, 27.4. In each the shorter longest share is the faster call.
//
// Partial outputs are bf16. A request in one range is summed in fp32 throughout,
// one in several is rounded twice, however many they are (2.3e-3 relative
// instead of 1.7e-3). More ranges are therefore not taken where they split
// requests that whole pages leave in one piece, counted by outputs. (With as
// many ranges it is chance which requests straddle a boundary.)
inline void plan_line(const LineReqs &rs, uint64_t slots, bool whole_pages, Line *ln) {
  whole_page_line(rs, slots, ln);
  bool finer = false;
  for (int i = 0; i < rs.n; ++i) finer = finer || cut_inside_pages(rs.r[i]) || rs.r[i].weight != rs.r[0].weight;
  if (!finer || whole_pages || ln->total > 0xFFFFFFFFull) return;
  Line f;
  if (!fine_line(rs, slots, &f)) return;
  const LineTime tw = line_time(rs, *ln), tf = line_time(rs, f);
  const uint64_t more = tf.partials > tw.partials ? (tf.partials - tw.partials) * 4 * kTimeWeightUnit / f.workers : 0;
  const bool rounds_more = f.workers > ln->workers && tf.split > tw.split;
  if (tf.longest + more < tw.longest && !rounds_more) *ln = f;
}

}  // namespace cp
