// The balanced schedule's plan of one launch: its requests' KV laid on one
// cost line, which is cut into equal shares, one per workgroup. Host only.
// The kernels find their pieces from the same numbers (next_balanced in
// schedule.h).
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

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
};
constexpr int32_t kTimeWeightUnit = 8;

// Ranges cut inside pages hold no less than this (one MLA page of 64
// tokens), or a page of models with smaller ones.
constexpr uint64_t kMinRangeKib = 72;

// A cut line: block j of request i (blk_tokens[i] tokens) sits at cost
// position begin[i] + j blk_cost[i]; share w of `workers` is [floor(w total /
// workers), floor((w + 1) total / workers)).
struct Line {
  std::vector<int32_t> blk_tokens, blk_cost, first, ranges;  // first share of a request, and how many it meets
  std::vector<uint64_t> begin;
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
inline void lay_line(const std::vector<LineReq> &reqs, uint64_t fixed, uint64_t least, uint64_t slots, Line *ln) {
  const size_t n = reqs.size();
  auto blocks = [&](size_t i) { return (uint64_t)((reqs[i].tokens + ln->blk_tokens[i] - 1) / ln->blk_tokens[i]); };
  uint64_t T0 = 0;
  for (size_t i = 0; i < n; ++i) T0 += blocks(i) * (uint64_t)ln->blk_cost[i];
  const uint64_t W0 = std::max<uint64_t>(1, std::min(slots, T0 / least));
  uint64_t T = 0, pre0 = 0;
  ln->begin.resize(n);
  for (size_t i = 0; i < n; ++i) {
    const bool straddled = i > 0 && (pre0 * W0) % T0 != 0;
    T += straddled ? fixed : 0;
    ln->begin[i] = T;
    T += blocks(i) * (uint64_t)ln->blk_cost[i];
    pre0 += blocks(i) * (uint64_t)ln->blk_cost[i];
  }
  const uint64_t W = std::max<uint64_t>(1, std::min(slots, T / least));
  auto owner = [&](uint64_t x) { return (int32_t)(((x + 1) * W - 1) / T); };
  ln->first.resize(n);
  ln->ranges.resize(n);
  for (size_t i = 0; i < n; ++i) {
    const uint64_t C = ln->begin[i];
    ln->first[i] = owner(C);
    ln->ranges[i] = owner(C + (blocks(i) - 1) * (uint64_t)ln->blk_cost[i]) - ln->first[i] + 1;
  }
  ln->total = T;
  ln->workers = (uint32_t)W;
}

// Ranges of whole pages, shared by bytes. The line counts units of 8 KiB where
// every page is a multiple of that, else KiB (in units of 8 a 36 KiB page would
// count 11% too much beside one of 32). Shares are floored at whole units, so
// the unit decides which page a share ends at, and with it the bits of the
// results: it stays what it is for the pages of 64 tokens of every model.
inline Line whole_page_line(const std::vector<LineReq> &reqs, uint64_t slots) {
  Line ln;
  int64_t unit = 8192;
  for (const LineReq &r : reqs)
    if ((int64_t)r.page_tokens * r.kappa % unit) unit = 1024;
  uint64_t least = 1;
  for (const LineReq &r : reqs) {
    ln.blk_tokens.push_back(r.page_tokens);
    ln.blk_cost.push_back((int32_t)(((int64_t)r.page_tokens * r.kappa + unit - 1) / unit * r.rereads));
    least = std::max(least, (uint64_t)ln.blk_cost.back());
  }
  lay_line(reqs, kPieceFixedCost * 1024 / (uint64_t)unit, least, slots, &ln);
  return ln;
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
// finely as the blocks allow. workers is 0 where the line would not fit.
inline Line fine_line(const std::vector<LineReq> &reqs, uint64_t slots) {
  Line ln;
  uint64_t least = 1, least_w = 1, Tw = 0, T = 0;
  int32_t wmin = 1 << 30, wmax = 0;
  for (const LineReq &r : reqs) {
    const int32_t blk = cut_inside_pages(r) ? r.step_tokens : r.page_tokens;
    const uint64_t c = (uint64_t)(((int64_t)blk * r.kappa + 1023) / 1024 * r.rereads);
    const uint64_t page = c * (uint64_t)(r.page_tokens / blk);
    // a range spans at least a block of every model, and a page of those
    // whose pages are smaller than kMinRangeKib (splitting further makes
    // more partials without shortening the launch)
    const uint64_t l = std::max(c, std::min<uint64_t>(page, kMinRangeKib));
    const uint64_t nb = (uint64_t)((r.tokens + blk - 1) / blk);
    ln.blk_tokens.push_back(blk);
    ln.blk_cost.push_back((int32_t)c);
    least = std::max(least, l);
    least_w = std::max(least_w, l * (uint64_t)r.weight);
    T += nb * c;
    Tw += nb * c * (uint64_t)r.weight;
    wmin = std::min(wmin, r.weight);
    wmax = std::max(wmax, r.weight);
  }
  uint64_t fixed = kPieceFixedCost;
  if (wmin != wmax && Tw / least_w >= slots && Tw < (1ull << 31)) {
    for (size_t i = 0; i < reqs.size(); ++i) ln.blk_cost[i] *= reqs[i].weight;
    fixed *= kTimeWeightUnit;
    least = least_w;
  } else if (T >= (1ull << 31)) {
    return ln;
  }
  lay_line(reqs, fixed, least, slots, &ln);
  ln.finer = true;
  return ln;
}

// The line of a launch: of whole pages unless some model's pages are cut or
// the models' times per KiB differ.
inline Line plan_line(const std::vector<LineReq> &reqs, uint64_t slots, bool whole_pages) {
  bool finer = false;
  for (const LineReq &r : reqs) finer = finer || cut_inside_pages(r) || r.weight != reqs[0].weight;
  if (finer && !whole_pages) {
    Line f = fine_line(reqs, slots);
    if (f.workers) return f;
  }
  return whole_page_line(reqs, slots);
}

}  // namespace cp
