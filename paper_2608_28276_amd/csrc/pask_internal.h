// Internal declarations shared by the C ABI (pask_api.cpp) and the gfx950
// kernels (pask_append.hip, pask_attn.hip).  Not part of the public interface.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime_api.h>

#include "pask.h"

namespace pask {

enum Store { kHi = 0, kLo = 1 };
enum Counter { kCntHi = 0, kCntLo = 1, kCntPos = 2, kCntDrop = 3, kCntForced = 4, kCntLost = 5,
               kCntBudget = 6 };   // int64 remaining budget R in words 6, 7
constexpr int kCounterStride = 8;
constexpr int kPage = 16;          // tokens per page
constexpr int kQGroup = 32;        // elements per fp16 scale of a RETAIN-LOW vector
// Stream-K workers (single waves) per workgroup of the attention kernel for
// calls with more than kAlignedSegments segments: 2,048 single-wave workgroups
// took 4.5 us to dispatch; two waves per workgroup measured as four on HIGH
// pages and 5% slower on LOW pages (112.7 against 107.2 us at 87% LOW).
#ifndef PASK_ATTN_WPB
#define PASK_ATTN_WPB 4
#endif
#ifndef PASK_UNIT_TOKENS
#define PASK_UNIT_TOKENS 128
#endif
constexpr int kUnitTokens = PASK_UNIT_TOKENS;   // slots per attention work unit (multiple of 16)
constexpr uint32_t kKeepAll = 1u;

// The online controller's inputs (Alg. 2; Eq. 9-10), one copy per cache.
// `loaded` holds kBudgetLoaded once pask_budget_init has written the rest.
constexpr uint32_t kBudgetLoaded = 0x42554447u;
struct BudgetTable {
  uint32_t loaded;
  uint32_t n_tags, n_groups, n_states, n_sink;
  uint32_t pad[3];
  int64_t m[PASK_MAX_GROUPS][3];      // bytes a token persists in group c under action a
  int64_t gamma[PASK_MAX_STATES];     // reserve Gamma(s), bytes (Eq. 9)
  uint8_t crit[PASK_MAX_STATES];      // critical or lookahead-critical state
  uint8_t action[PASK_MAX_TAGS][PASK_MAX_GROUPS];
  uint8_t floor_[PASK_MAX_TAGS][PASK_MAX_GROUPS];
  float rho_up[PASK_MAX_TAGS][PASK_MAX_GROUPS][2];   // Eq. 7: R->L, L->H
};
static_assert(sizeof(BudgetTable) % 16 == 0, "BudgetTable is copied in 16-byte words");

// Device-side view of one cache buffer.
struct CacheView {
  uint32_t* status;       // [0] status word, [2] HI cursor, [3] LO cursor
  int32_t* counters;      // [max_batch][n_layers][8]
  int32_t* block_table;   // [max_batch][n_layers][2][max_pages]
  int32_t* index_list;    // [max_batch][n_layers][2][max_tokens]
  int32_t* staging;       // [max_batch][staging_stride]: a bulk append's scratch (the last four words)
  BudgetTable* budget;
  uint8_t* ring_act;      // [max_batch][n_layers][window]: action | forced << 2
  uint8_t* hi_pool;       // recent-window pages first, then the HIGH store
  uint8_t* lo_pool;
  int32_t n_layers, n_kv_heads, head_dim, max_tokens, max_pages, lo_pages;
  int32_t hi_pages;       // pool pages including the recent windows
  int32_t hi_base;        // first page of the HIGH store (= recent-window pages)
  int32_t window;         // W
  int32_t ring_pp;        // pages of one (sequence, layer) window: ceil(W / 16)
  int32_t staging_stride; // max_tokens + W + 4: the last four are the append's HIGH and LOW
                          // store counts before it, its first position p0 and n_fit
  uint32_t hi_page_bytes, lo_page_bytes;
};

// Lambda's column for one layer group: selected action a0 and floor a- per tag.
struct TableColumn {
  uint8_t a0[64];
  uint8_t amin[64];
  uint32_t n_tags;
  uint32_t n_sink;
  uint32_t group;           // the layer's group c
};

struct AppendArgs {
  CacheView cv;
  TableColumn tab;
  const int32_t* n_new;     // [batch] or null (all max_new)
  const uint8_t* tags;      // [batch][max_new] or null (KEEP_ALL)
  const uint8_t* states;    // [batch][max_new] parser states, or null (Eq. 10 alone)
  const uint16_t* k;        // bf16 bits [batch][max_new][Hkv][D]
  const uint16_t* v;
  int32_t layer, batch, max_new;
  uint32_t flags;
};

struct AttnArgs {
  CacheView cv;
  const uint16_t* q;        // bf16 bits [batch][Hq][D]
  uint16_t* out;            // bf16 bits [batch][Hq][D]
  float* lse;               // [batch][Hq] or null
  float* ws_o;              // [batch][Hkv][splits][G4 * D], G4 = max(G, 4) heads
  float* ws_ml;             // [batch][Hkv][splits][G4][2]  (max, sum) in log2 units
  // The step's new entry, persisted by the call itself (kFusedMaxBatch
  // sequences at most, no recent window, no parser states): the attention
  // kernel decides it, writes it into its page and attends it; the merge
  // kernel enters it in the counters, lists and block tables.  Null when the
  // call persists nothing or the one-token append kernel ran before it.
  const uint8_t* tags_new;  // [batch]
  const uint16_t* k_new;    // bf16 bits [batch][Hkv][D]
  const uint16_t* v_new;
  int32_t* ws_seq;          // [batch][8]: 8 u16 piece counts (one per KV head), then the entry's outcome (distortion: arrivals)
  TableColumn tab;          // Lambda's column of the layer (with tags_new)
  float scale_log2;         // softmax_scale * log2(e)
  int32_t layer, batch, n_q_heads, splits;   // splits: partials per (b, g) the workspace holds
  int32_t attn_blocks;      // stream-K workers (waves) of the attention kernel, set at launch
  int32_t min_pages;        // fewest pages a worker takes, set at launch
};

// The workspace of calls with at most kSmallSegments (sequence, KV head)
// segments holds pieces down to one page, up to kSmallPartials partials in all.
constexpr int kSmallSegments = 64;
constexpr int kSmallPartials = 4096;
// Calls with at most kAlignedSegments segments (and at most 64 sequences) cut
// every segment by itself and merge its pieces with several thread groups at
// once (small_units in pask_plan.h).  At 256 segments the cuts are too coarse
// to even out ragged ones: 32 sequences of 1,000-8,000 entries take 106.7 us
// so, 98.0 by ranges over the whole list; 16 take 54.4 and 55.0, 9 of 4,064
// 30.6 and 34.8.
constexpr int kAlignedSegments = 128;
// Calls that persist their step's entry themselves: every workgroup decides
// the entries of all sequences, 64 at a time (one per lane of a wave), and
// keeps their counts and outcomes in LDS (32 bytes per sequence, two
// workgroups per compute unit).
constexpr int kFusedMaxBatch = 1024;

// The library-owned scratch of pask_decode_attn_noalloc: a device array of
// kScratchBytes in pask_attn.hip, one copy per GPU.  scratch_workspace gives
// the current device's address of it (hipGetSymbolAddress, taken once per
// device with that device current, then cached).
constexpr size_t kScratchBytes = PASK_NOALLOC_SCRATCH_BYTES;
hipError_t scratch_workspace(void** ptr);

// Launchers (pask_append.hip: reset, budget init, append; pask_attn.hip:
// attention, distortion).  Return hipSuccess or the launch error.
hipError_t launch_reset(const CacheView& cv, int32_t max_batch, hipStream_t s);
hipError_t launch_append(const AppendArgs& a, hipStream_t s);        // chooses the windowed kernels when W > 0
hipError_t launch_append_step(const AppendArgs& a, hipStream_t s);
hipError_t launch_budget_init(const CacheView& cv, int32_t batch, int64_t r0, hipStream_t s);
hipError_t launch_attention(const AttnArgs& a, int group_size, hipStream_t s);
// Attention over two caches with the same queries (partials in ref.ws_* and itv.ws_*), then
// dist[b] += max over heads of the squared distance of the two outputs (Eq. 4).
hipError_t launch_distortion(const AttnArgs& ref, const AttnArgs& itv, int group_size, const uint8_t* in_s,
                             float* dist, hipStream_t s);

}  // namespace pask
