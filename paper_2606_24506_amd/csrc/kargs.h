// Kernel-argument records shared by the host launcher (api.cpp) and the
// kernels (kernels.hip). Everything a launch needs travels by value in the
// kernel-argument segment, so a decode step costs no host-to-device copy.
// Sizes stay well under the 4 KiB argument limit.
#pragma once
#include <stdint.h>

namespace cp {

constexpr int kMaxLaunchModels = 4;   // distinct models in one decode launch
constexpr int kMaxReqPerLaunch = 64;  // requests in one launch (at most one per lane of a wave)
constexpr uint32_t kNoWs = 0xFFFFFFFFu;
// Fixed split workspace of cp_attn_decode_noalloc, per GPU, in bytes.
constexpr uint64_t kNoAllocScratchBytes = 40ull << 20;
constexpr int kMaxScratchDevices = 64;
// Device free-page stacks (pools created with device_pages): entries per
// model; model m's stack is DecodeArgs::stack[m * kStackCap ...].
constexpr int32_t kStackCap = 8192;
// The host refills a stack with up to this many pages (a chunk's worth at
// most) when a step needs more than it holds.
constexpr int32_t kStackRefill = 1024;
enum : int32_t { kSchedBalanced = 0, kSchedQueue = 1, kSchedGrid = 2 };
// Balanced schedule (cost_line.hpp). A request's stretch of the launch's cost line
// is cut between blocks of GeomK::blk_tokens tokens: pages, or for large pages
// the tokens that the model's kernel works through in one step of its loop.
// The fixed work of one piece (page-table and query loads, the latency of its
// first pages under a loaded memory system, the end merge and the partial
// write) is charged as this many KiB: measured at about 23K cycles per piece
// on the narrow kernel, which streams about 600 cycles per 8 KiB. A request
// boundary that falls inside a workgroup's share is preceded by that much cost
// on the cost line, so the workgroup that runs a second piece there takes
// correspondingly less KV. DecReq::unit_begin is the cost position of the
// request's first block.
constexpr uint32_t kPieceFixedCost = 320;

// Decode code paths (GeomK::variant), chosen per model by the host.
//   Vector path (0-7): wavefront reductions; heads per block (16 or 8) and
//     V values per lane (8, 4, 2, 1); any geometry.
//   Small-group vector path (8-13): wavefront reductions for GQA/MHA with
//     1, 2 or 4 query heads per KV head and head_dim 64 or 128 (the forced
//     vector path, and pages the stream path does not tile).
//   Narrow matrix path (16, 17, 19, 20, 23): 8, 16 or 32 query heads per KV
//     head (MLA latent head, or head_dim 128); 17 is MLA in units of up to
//     16 heads with P as three bf16 operands (whole).
//   Head-owner matrix path (21, 22): 64 or 128 query heads per KV head with
//     head_dim 128.
//   Stream matrix path (24, 25): any other GQA / MHA group, head_dim 64 or
//     128, in units of up to 16 heads; P whole.
//   MLA head-pair path (26, 27): MLA with 17 to 32 heads, or in units of up
//     to 64; P whole.
//   128-head MLA (18): its own kernel (score waves and P.V waves).
enum : int32_t {
  kV16x8 = 0, kV16x4, kV16x2, kV16x1, kV8x8, kV8x4, kV8x2, kV8x1,
  kS_G1_D64 = 8, kS_G2_D64, kS_G4_D64, kS_G1_D128, kS_G2_D128, kS_G4_D128,
  kM_MLA_G16 = 16, kM_MLA_G16S, kM_MLA_G128, kM_D128_G16, kM_D128_G32, kM_D128_G64, kM_D128_G128, kM_D128_G8,
  kT_D64 = 24, kT_D128,
  kM_MLA_H32 = 26, kM_MLA_H64
};
constexpr bool is_stream(int v) { return v == kT_D64 || v == kT_D128; }
constexpr bool is_mla_wide(int v) { return v == kM_MLA_G128; }
// Variants with 64 or more heads per KV head, whose partials are large.
constexpr bool is_many_heads(int v) { return v == kM_MLA_G128 || v == kM_D128_G64 || v == kM_D128_G128; }

// One piece of decode work: tokens [tok_begin, tok_end) of a request (whole
// blocks, but for the last one of the context), for one
// head block, writing partial slot `slot` when the request is split; model
// is the request's index into DecodeArgs::geom.
struct Seg {
  uint32_t tok_begin, tok_end, slot, hblk, model;
};

// Per-model geometry as the kernels see it.
struct GeomK {
  int32_t kind;        // 0 MLA, 1 GQA
  int32_t hq, hkv, g;  // g = hq / hkv
  int32_t d_k, d_v, row_elems, page_tokens;
  int32_t page_bytes;
  int32_t variant;     // kernel code path chosen by the host
  float scale_log2;    // softmax scale * log2(e)
  int32_t nb;          // head blocks per KV head (vector path)
  int32_t blk_tokens;  // balanced schedule: tokens of one block (divides page_tokens)
  int32_t blk_cost;    // ... and its relative work
  int32_t pool_model;  // the model's id in the pool (its device page stack)
  int32_t layers;      // KV planes of a request of this model
};

// One request of a decode launch.
struct DecReq {
  uint32_t pte_base;  // first page-table entry of the request
  uint32_t ctx_len;   // tokens to attend over (>= 1)
  uint32_t q_off;     // bf16 element offset of the request's queries
  uint32_t o_off;     // bf16 element offset of its outputs
  uint32_t lse_off;   // float offset of its log-sum-exp values
  uint32_t ws_base;   // first partial lse row (kNoWs when the request is not split)
  uint32_t ws_orow;   // partial outputs start at element offset ws_orow * d_v
  uint32_t unit_begin;   // queue/grid: first unit; balanced: cost position of the request's first block
  uint16_t chunk_pages;  // queue/grid: pages per KV range; balanced: first worker of the request
  uint16_t n_chunks;     // KV ranges = partial slots
  uint8_t model;         // index into DecodeArgs::geom
  uint8_t app_flags;     // fused append: kAppRow (the last context token is a new row at
                         // DecodeArgs::rows + app_off), kAppPage (its page is new: app_pte),
                         // kAppPop (its page is new and comes from the model's device
                         // stack, one page per plane; app_pte is then the request id)
  uint16_t n_hblk;       // head blocks per KV range
  uint32_t app_off;      // element offset of the new row in DecodeArgs::rows
  uint32_t app_pte;      // page-table entry of the new row's page when kAppPage is set
};
enum : uint8_t { kAppRow = 1, kAppPage = 2, kAppPop = 4 };

struct DecodeArgs {
  uint8_t *pool;          // written only by the fused append
  uint32_t *pte;          // written only by the fused append (a new page's entry)
  const uint16_t *rows;   // fused append: new logical rows, packed in call order
  const uint16_t *q;
  uint16_t *out;
  float *lse;
  uint16_t *ws_o;     // partial outputs, [row][d_v] bf16, normalised
  float *ws_l;        // partial log-sum-exp, [row], natural log
  uint32_t *queue;    // queue schedule: {next unit, finished workgroups}
  // device page stacks (kAppPop): entries and per-model counts, per-request
  // pop state ((epoch << 1) | done) and per request id {first page-table
  // entry, entries per plane}
  const uint32_t *stack;
  int32_t *stack_top;
  uint32_t *pop_state;
  const uint32_t *req_geo;
  uint32_t epoch;  // this launch's pop epoch (>= 1)
  uint32_t pad0;
  // All-layer launches (cp_attn_decode_layers): a request's layer cursor
  // and the tokens its cursor has carried through every layer (both at
  // index 2 * request id), and per launch entry the pieces finished so far
  // (reset by the last one). ent_tag[r] is request id | layers << 20 for an
  // entry whose completion moves a cursor, 0 otherwise.
  uint32_t *layer_cursor;
  uint32_t *layer_tokens;
  uint32_t *entry_done;
  int32_t n_req, n_units;
  int32_t schedule;     // kSchedBalanced, kSchedQueue or kSchedGrid
  uint32_t total_cost;  // balanced: length of the launch's cost line
  GeomK geom[kMaxLaunchModels];
  DecReq req[kMaxReqPerLaunch];
  uint32_t ent_tag[kMaxReqPerLaunch];
};
constexpr uint32_t kTagLayerShift = 20;

// V columns one merge workgroup covers: 64 lanes of up to four columns
// (d_v is 64, 128, 256 or 512).
constexpr uint32_t merge_block_cols(uint32_t d_v) { return d_v >= 256 ? 256u : d_v; }

struct MergeReq {
  uint32_t block_begin;  // first merge workgroup of this request
  uint32_t hq, d_v, n_chunks;
  uint32_t ws_base, ws_orow, o_off, lse_off;
};

struct MergeArgs {
  const uint16_t *ws_o;
  const float *ws_l;
  uint16_t *out;
  float *lse;
  int32_t n_req, n_blocks, pad0, pad1;  // n_blocks: merge workgroups
  MergeReq req[kMaxReqPerLaunch];
};

// Append and gather: a workgroup of kCopyThreads copies up to kCopyUnroll
// 16-byte segments per thread, and so this many rows (a power of two, so that a
// workgroup seldom meets two pages of a power of two of tokens). At least 10 KiB,
// whatever the page holds: a launch has less than 2^32 threads, and 2^24
// workgroups of a row of 256 bytes each would bound a call to 4 GiB.
constexpr int kCopyThreads = 256, kCopyUnroll = 5;
constexpr uint32_t copy_rows_per_block(uint32_t row_elems) {
  const uint32_t fit = (uint32_t)(kCopyThreads * kCopyUnroll) / (row_elems / 8);
  uint32_t r = 1;
  while (2 * r <= fit) r *= 2;
  return r;
}

struct AppReq {
  uint64_t src_off;      // bf16 element offset of the request's first row in the input
  uint32_t block_begin;  // first workgroup of this request in the launch
  uint32_t n_new;
  uint32_t old_len;
  uint32_t pte_base;
  uint16_t model;
  uint16_t ent;  // index in AppendArgs::ent of its first new page's entry (kNoEnt: in the page table)
  uint32_t pad;
};
constexpr uint16_t kNoEnt = 0xFFFFu;
// New page-table entries one append launch carries; appends that open more
// pages copy theirs to the device first.
constexpr int kAppEntMax = 352;

struct AppendArgs {
  uint8_t *pool;
  uint32_t *pte;  // written only where a new page's entry comes with the launch
  const uint16_t *rows;
  int32_t n_req, n_blocks, n_ent, pad1;
  GeomK geom[kMaxLaunchModels];
  AppReq req[kMaxReqPerLaunch];
  uint32_t ent[kAppEntMax];
};

struct GatherArgs {
  const uint8_t *pool;
  const uint32_t *pte;
  uint16_t *dst;
  uint32_t pte_base, plane, start, n_tok;  // plane: page-table entries from one KV plane to the next
  GeomK geom;
};

// Refill of a device page stack: n entries written at dst[0..n), then the
// model's count set to new_top. The entries travel in the arguments, so the
// host keeps no staging copy alive.
constexpr int32_t kStackPushMax = 640;
struct StackPushArgs {
  uint32_t *dst;
  int32_t *top;
  int32_t n, new_top;
  uint32_t ent[kStackPushMax];
};

static_assert(kMaxReqPerLaunch <= 64, "request lookups search one key per lane");
static_assert(sizeof(StackPushArgs) <= 3072, "stack push arguments too large");
// the argument segment (with the runtime's hidden arguments) stays under 4 KiB
static_assert(sizeof(DecodeArgs) <= 3776, "decode kernel arguments too large");
static_assert(sizeof(MergeArgs) <= 3072, "merge kernel arguments too large");
static_assert(sizeof(AppendArgs) <= 3776, "append kernel arguments too large");

}  // namespace cp
