// Internal launch-side structures shared by the host API and the kernels.
// Not part of the public ABI (include/recguide.h is).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace rg {

constexpr int kPageSize = 16;
constexpr int kMaxReqPerLaunch = 128;  // equals RG_ATTN_MAX_REQS_PER_LAUNCH
constexpr int kKeyTile = 128;          // keys per LDS buffer; chunks are multiples of it
constexpr int kNarrowCols = 128;       // query columns of a narrow attention work group
constexpr int kFullThreads = 768;      // threads of a full attention work group; a narrow one has half
constexpr int kCombThreads = 128;      // ... of a merge work group at least
// Threads of one launch at most: at 2^32 its grid wraps, and the rest of the
// work is left out with or without an error.
constexpr int64_t kMaxLaunchThreads = (int64_t(1) << 32) - 1;
constexpr int kMaxChunkKeys = 1 << 16;  // keys per work item at most
constexpr int kSyncHeader = 4;          // queue head, exit count, give-up flag, report word
// Combine items of one launch the one-launch kernel can count (two counters
// each); launches with more use the main kernel plus the combine kernel.
constexpr int kMaxSyncComb = 16384;
// The synchronisation words open every attention workspace at a fixed place
// and size, so calls with different layouts can share a workspace: the words
// one call leaves at zero are never another call's partials.
constexpr int kSyncWords = kSyncHeader + 2 * kMaxSyncComb;

// Per-request data of one attention launch.  Everything a work group needs
// about its request travels in the kernel arguments, so no table has to be
// copied to the device before the kernels run.
struct AttnReq {
  int32_t q_start;     // first query row (token) of the request
  int32_t ctx;         // cached context tokens L
  int32_t nv;          // n (low 16 bits) | n_verify << 16, both unsigned 16-bit fields
  int32_t page_start;  // offset of the request's pages in page_indices
  int32_t item_start;  // first main-kernel work item
  int32_t part_start;  // first partial column in the workspace (split requests)
  int32_t comb_start;  // first combine work item (split requests)
};

// A request of a launch with overlap branches: its rows after the verify
// rows are branches, described by up to three words, each packed as rows
// (bits 0-15) | prefix verify rows kept (bits 16-27) | committed lead rows
// (bits 28-31), and `rep`: the word at index rep >> 28 stands for
// rep & 0xffff branches of its shape whose prefixes grow by
// (rep >> 16) & 0xfff each (a regular family, e.g. one draft block per
// hypothetical accepted length); the other words for one branch each.
// br[0] = 0 means no branch list (the rows after the verify rows are one
// continuation block that keeps every verify row).
struct AttnReqBr : AttnReq {
  int32_t br[3];
  int32_t rep;
};
constexpr int kMaxReqPerLaunchBr = 64;  // equals RG_BRANCH_MAX_REQS_PER_LAUNCH

// The same in 7 words, for requests whose keys are one work item and whose
// numbers fit the fields: two plans' requests then share one launch.
struct AttnReqBrPacked {
  uint32_t q_n;        // q_start (low 20 bits) | n << 20
  uint32_t ctx_nv;     // ctx (low 20 bits) | n_verify << 20
  int32_t page_start;
  int32_t item_start;
  uint32_t br[3];      // rows (bits 0-9) | prefix (10-19) | lead (20-23); bits 24-31: the
                       // fields of `rep`: count, prefix step, index

  bool pack(const AttnReqBr& r) {
    const uint32_t n = r.nv & 0xffff, nv = (uint32_t)r.nv >> 16;
    const uint32_t f[3] = {(uint32_t)r.rep & 0xffff, ((uint32_t)r.rep >> 16) & 0xfff, (uint32_t)r.rep >> 28};
    if ((uint32_t)r.q_start >> 20 || (uint32_t)r.ctx >> 20 || n >> 12 || nv >> 12) return false;
    q_n = (uint32_t)r.q_start | n << 20;
    ctx_nv = (uint32_t)r.ctx | nv << 20;
    page_start = r.page_start;
    item_start = r.item_start;
    for (int b = 0; b < 3; ++b) {
      const uint32_t w = (uint32_t)r.br[b], rows = w & 0xffff, prefix = (w >> 16) & 0xfff, lead = w >> 28;
      if (rows >> 10 || prefix >> 10 || f[b] >> 8) return false;
      br[b] = rows | prefix << 10 | lead << 20 | f[b] << 24;
    }
    return true;
  }
  __host__ __device__ AttnReqBr unpack() const {
    AttnReqBr r;
    r.q_start = (int32_t)(q_n & 0xfffff);
    r.ctx = (int32_t)(ctx_nv & 0xfffff);
    r.nv = (int32_t)(q_n >> 20 | (ctx_nv >> 20) << 16);
    r.page_start = page_start;
    r.item_start = item_start;
    r.part_start = r.comb_start = 0;
    for (int b = 0; b < 3; ++b)
      r.br[b] = (int32_t)((br[b] & 0x3ff) | ((br[b] >> 10) & 0x3ff) << 16 | ((br[b] >> 20) & 0xf) << 28);
    r.rep = (int32_t)(br[0] >> 24 | (br[1] >> 24) << 16 | (br[2] >> 24) << 28);
    return r;
  }
};

template <typename Req, int MaxReq>
struct AttnPlanT {
  int32_t num_req;         // requests in this launch
  int32_t chunk;           // keys per work item, multiple of kKeyTile
  int32_t total_items;     // main-kernel work items
  int32_t total_comb;      // combine work items
  int32_t grid_items;      // total_items rounded up to a multiple of 8
  int32_t grid_comb;       // total_comb rounded up to a multiple of 8
  int32_t cols_per_group;  // query columns one work group covers (256)
  int32_t max_chunks;      // most chunks of one split request (picks the combine variant)
  int32_t persist_grid;    // 0: main kernel + combine kernel; else the work groups of the
                           // one-launch work-queue kernel (main items, then combine items)
  Req req[MaxReq + 1];     // entry num_req holds the end sentinels
  int32_t narrow;          // 1: narrow work groups (no request has more than 128 columns)
};
using AttnPlan = AttnPlanT<AttnReq, kMaxReqPerLaunch>;
using AttnPlanBr = AttnPlanT<AttnReqBr, kMaxReqPerLaunchBr>;
using AttnPlanBrPacked = AttnPlanT<AttnReqBrPacked, 2 * kMaxReqPerLaunchBr>;
static_assert(sizeof(AttnPlan) <= 3700, "attention plan must fit the kernel argument block");
static_assert(sizeof(AttnPlanBr) <= 3700, "attention plan must fit the kernel argument block");
static_assert(sizeof(AttnPlanBrPacked) <= 3700, "attention plan must fit the kernel argument block");

struct AttnArgs {
  const uint16_t* q;
  const uint16_t* k_cache;
  const uint16_t* v_cache;
  uint16_t* out;
  float* lse;
  const int32_t* page_indices;
  uint16_t* part_o;  // per 32-column tile: 32 x D bf16 normalised partial outputs, MFMA fragment order
  float* part_ml;  // [partial columns][2] fp32 (running max of raw scores, sum)
  int32_t* sync;   // kSyncWords words, zero between calls: queue head, exit count, give-up
                   // flag, report word (nonzero after a call whose wait gave up, until
                   // read), then finished-tile counts (indexed by a column group's first
                   // combine item) and, kMaxSyncComb words on, started-combine counts
  int32_t hq, hkv, g;
  float sm_scale;    // natural-log domain scale
  float scale_log2;   // sm_scale * log2(e)
  float rescale_gap;  // raw-score margin before the running maximum moves
};

// Attention launchers (attention.hip).  `plan` is one launch's plan.
hipError_t launch_attention(const AttnArgs& args, const AttnPlan& plan, int head_dim,
                            hipStream_t stream);
hipError_t launch_attention(const AttnArgs& args, const AttnPlanBr& plan, int head_dim,
                            hipStream_t stream);
hipError_t launch_attention(const AttnArgs& args, const AttnPlanBrPacked& plan, int head_dim,
                            hipStream_t stream);

// Calls launch(args) for consecutive slices of `groups` work groups of
// `threads` threads, args.first and args.grid telling the slice: one up to
// 2^23 - 8 requests or 2^24 - 8 row chunks of the logit passes and 2^26 - 32
// requests of the branch plan.  Slices are whole multiples of 8 groups
// (xcd_item).  The slice travels in the argument structs' padding: as two
// more kernel arguments it cost 1 % of a logit pass over 2000 rows of 128256.
template <typename Args, typename Launch>
hipError_t sliced(Args args, int64_t groups, int threads, Launch launch) {
  const int64_t most = kMaxLaunchThreads / threads / 8 * 8;
  for (int64_t first = 0; first < groups; first += most) {
    args.first = (int32_t)(uint32_t)first;
    args.grid = (int32_t)std::min(most, groups - first);
    launch(args);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Logit-row reductions (logits.hip).
constexpr int kLogitThreads = 256;
constexpr int kLogitChunk = 8192;  // vocab entries per work group

struct VerifyArgs {
  const uint16_t* logits;
  int64_t row_stride;
  int32_t vocab, num_req, rows, nchunk;
  uint32_t cmul;       // item / nchunk = item * cmul >> cshift (chunk_divisor)
  int32_t cshift;
  const int32_t* row_indptr;
  const int32_t* tokens;
  int32_t* row_argmax;
  int32_t* accept_len;
  int32_t* next_token;
  float* row_entropy;
  float* accept_entropy;
  float4* chunk_st;    // workspace [rows * nchunk] (max, bits(argmax), Z', S)
  int32_t grid, first;  // work groups of this launch, and the first one's item (set by the launch)
};

struct DraftArgs {
  const uint16_t* logits;
  int64_t row_stride;
  int32_t vocab, rows, nchunk;
  uint32_t cmul;         // as in VerifyArgs
  int32_t cshift;
  int32_t* top1;
  int32_t* top2;
  float* p1;
  float* p2;
  float* margin;
  float* entropy;
  float4* chunk_a;       // workspace [rows * nchunk] (max, bits(i1), v2, bits(i2))
  float2* chunk_b;       // [rows * nchunk] (Z', S)
  int32_t grid, first;   // as in VerifyArgs
};

inline int32_t logit_chunks(int32_t vocab) { return (vocab + kLogitChunk - 1) / kLogitChunk; }
// log2 of the smallest power of two >= a row's chunks: with it the accepted
// sizes are bounded (rows << shift fits 30 bits).
inline int32_t logit_chunk_shift(int32_t vocab) {
  int32_t s = 0;
  while ((1 << s) < logit_chunks(vocab)) ++s;
  return s;
}
// Division of an item index (below 2^31) by the chunks per row: with
// l = logit_chunk_shift, mul = ceil(2^(31 + l) / nchunk) fits 32 bits, and
// item * mul >> (31 + l) is exact, since mul * nchunk exceeds 2^(31 + l) by
// less than nchunk <= 2^l, so the product is off by less than 2^(31 + l).  A
// row work group thus finds its row and chunk with one scalar multiply and
// no work groups are launched for slots past a row's last chunk.
inline void chunk_divisor(int32_t vocab, uint32_t& mul, int32_t& shift) {
  const uint64_t n = (uint64_t)logit_chunks(vocab);
  shift = 31 + logit_chunk_shift(vocab);
  mul = (uint32_t)(((uint64_t(1) << shift) + n - 1) / n);
}
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

hipError_t launch_verify(const VerifyArgs& a, hipStream_t stream);
hipError_t launch_draft(const DraftArgs& a, hipStream_t stream);
// Verify and draft passes of one round together: two launches in all.
hipError_t launch_round(const VerifyArgs& v, const DraftArgs& d, hipStream_t stream);

// Static device scratch of the allocation-free logit round (logits.hip):
// its size, and this device's address of it (looked up on first use).
constexpr size_t kNoAllocScratchBytes = size_t(4) << 20;  // equals RG_NOALLOC_SCRATCH_BYTES
hipError_t noalloc_scratch(void** ptr);

// Branch planning and matching (branches.hip).
struct PlanBranchArgs {
  const float* margin;
  const int32_t* top2;
  const int32_t* row_indptr;
  int32_t num_req;
  float delta;
  int32_t* n_risky;
  int32_t* n_corr;
  int32_t* corr_pos;
  int32_t* corr_tok;
  int32_t* continuation;
  int32_t grid, first;  // as in VerifyArgs
};
struct MatchBranchArgs {
  const int32_t* accept_len;
  const int32_t* next_token;
  const int32_t* block_len;
  const int32_t* n_corr;
  const int32_t* corr_pos;
  const int32_t* corr_tok;
  const int32_t* continuation;
  const int32_t* cont_first;
  int32_t num_req;
  int32_t* reused;
};
hipError_t launch_plan_branches(const PlanBranchArgs& a, hipStream_t stream);
hipError_t launch_match_branches(const MatchBranchArgs& a, hipStream_t stream);

// Verification-guided block sizing and bucketing (Sec. 5.2, Sec. 5.3).
constexpr int kMaxBlockCandidates = 8;
constexpr int kMaxSBins = 64;
constexpr int kMaxBucketRequests = 65536;
struct BlockSizeArgs {
  int32_t nb, ns;                       // candidates, s bins
  int32_t cand[kMaxBlockCandidates];    // ascending block sizes
  float edges[kMaxSBins - 1];           // ascending s-bin edges
  float cost[kMaxBlockCandidates];      // T_C(B)
  float rho;
  const float* value;                   // [nb][ns][nb][2]
  const int32_t* accept_len;
  const float* accept_entropy;
  const int32_t* prev_block;
  float* entropy_hist;
  int32_t num_req;
  int32_t* next_block;
  int32_t* order;                       // NULL when not grouping or when num_req == 0
  int32_t* bucket_offsets;              // NULL: no grouping
};
hipError_t launch_plan_block_sizes(const BlockSizeArgs& a, hipStream_t stream);

}  // namespace rg
