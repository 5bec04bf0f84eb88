// The balanced schedule's plan of one launch behind a C function, for
// test_cost_line.py. out: per request {blk_tokens, blk_cost, begin, first,
// ranges}; returns workers, and the line's total in *total.
#include "cost_line.hpp"

extern "C" int64_t cost_line(int32_t n, const int64_t *tokens, const int32_t *page_tokens, const int32_t *step_tokens,
                             const int32_t *kappa, const int32_t *rereads, const int32_t *weight,
                             const int32_t *out_elems, int32_t slots, int32_t whole_pages, int64_t *out,
                             int64_t *total) {
  cp::LineReqs rs;
  for (rs.n = 0; rs.n < n; ++rs.n) {
    const int i = rs.n;
    rs.r[i] = cp::LineReq{tokens[i], page_tokens[i], step_tokens[i], kappa[i], rereads[i], weight[i], (uint32_t)out_elems[i]};
  }
  cp::Line ln;
  cp::plan_line(rs, (uint64_t)slots, whole_pages != 0, &ln);
  for (int32_t i = 0; i < n; ++i) {
    const int64_t v[5] = {ln.blk_tokens[i], ln.blk_cost[i], (int64_t)ln.begin[i], ln.first[i], ln.ranges[i]};
    std::copy(v, v + 5, out + 5 * i);
  }
  *total = (int64_t)ln.total;
  return ln.workers;
}
