// Host-side declarations shared by the C-ABI layer and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/msa.h"

namespace msa {

// Validated, derived view of msa_config_t.
struct Dims {
  int N, G, P, C, Hq, Hkv, r, d;
  int cos;        // 1 = cosine, 0 = dot
  int scope_all;  // 1 = head mean over every head, one selection for all KV heads (literal Eq. 2)
  int token_pool; // 1 = document score is the max over the M tokens of a batch row (literal Eq. 2)
  float base;
  const int32_t* lens;  // device [N] document lengths, or null (every document holds G tokens)
  hipEvent_t prof_start, prof_stop;  // the caller's events around the dominant kernel of this call, or null
  int64_t NC;     // N * C routing keys per KV head
  int64_t tiles;  // ceil(NC / 16) tiles of 16 keys per KV head
};

// Work split of the MFMA-bound scoring path for many query tokens (msa_score_gemm.hip).
struct GemmPlan {
  int n_qblocks;         // blocks of tokens_per_wg query tokens (two-pass form)
  int tb1, n_qblocks1;   // one-pass form: 32-token blocks per wave (1, 2), blocks of 128 * tb1 query tokens
  int n_splits;          // key-range splits per (head, token block)
  int stages_per_split;  // 64-key stages per split
  size_t off_lists;      // byte offset of the candidate lists (after the folded fp32 queries)
  // One-pass filter (cosine, d = 128, eight chunks per document, one selection per KV group): the product runs on
  // the bf16 hi parts of the folded queries alone; every document whose one-pass score lies within twice the error
  // bound of the k-th best one-pass score is scored again exactly, and token blocks whose per-lane lists overflow
  // inside that band are redone by the two-pass kernel.
  int filter;            // 1: the filter applies
  int list_len;          // entries per per-lane list of the one-pass product (8: k <= 8, else 16)
  int tokens_per_wg;     // query tokens per workgroup = per fallback flag
  size_t off_eps;        // fp32 [BM][Hkv]: bound on |one-pass score - exact score| per (token, KV group)
  size_t off_flags;      // int32 [Hkv][n_qblocks]: 1 = this token block is redone by the two-pass kernel
  size_t off_flists;     // 64-bit keys [Hkv][BM][n_splits][2][list_len]: the per-lane lists of the one-pass product
                         // (the two-pass kernel's lists, off_lists, reuse this memory afterwards)
  size_t ws_bytes;
};
constexpr int kFilterMaxCand = 64;
bool gemm_path_applies(const Dims& dm, int BM, int k);
bool gemm_path_of_two_passes(const Dims& dm, int BM, int k);
GemmPlan plan_score_gemm(const Dims& dm, int BM, int k);
// Enqueues the scoring kernels.  Without the filter the per-split lists are left for score_merge_kernel.  With it
// the exact winners of every token are written to out_idx / out_score (or out_key: sorted 64-bit keys, token pooling),
// and the lists of the flagged token blocks are left for a merge that is gated by *gate_flags (device int32
// [Hkv][n_qblocks], null without the filter).
int launch_score_gemm_scan(const Dims& dm, const GemmPlan& pl, const void* q_route, int BM,
                           const void* KR, const float* inv_norm, int k, void* ws, hipStream_t st,
                           int32_t* out_idx, float* out_score, unsigned long long* out_key, const int** gate_flags);

// Folds the heads of BM tokens: qf fp32 [BM][Hkv][d], and where not null eps, flags, qop (see fold_queries_kernel; every M
// tokens take m_rows operand rows).
int launch_fold_queries(const Dims& dm, const void* q_route, int BM, float* qf, float* eps, int* flags, int n_flags,
                        uint4* qop, int n_rt, int pair, int M, int m_rows, hipStream_t st);

// Head mean over every head for many query tokens (msa_score_wide.hip): passes of tokens, segments of the bank.
struct WidePlan {
  int pair;              // 1: hi and lo rows, 32 tokens per workgroup; 0: hi rows alone, 64
  int pass_tokens;       // query tokens per pass
  int n_tb;              // token blocks (64 operand rows) of a whole pass
  int seg_docs;          // documents per segment (one score matrix)
  size_t off_qf, off_qop, off_eps, off_best, off_mat;
  size_t ws_bytes;
  size_t list_bytes;     // several segments, one pass: candidate lists of the tokens of a pass
  size_t off_list;       // ... where they are; 0: the workspace has no room for them
};
// Token pooling behind it without a selection per token: the best score of a block of a batch row's tokens per document,
// exact scores of the documents that can be among the k best.
struct WidePoolPlan {
  int applies;           // 1: this shape, and the buffers fit where those of WidePlan lie
  int nt, m_tiles, m_blocks;  // operand tiles of a token block; operand tiles and token blocks of a batch row
  int part_docs, n_parts;     // documents of a part, parts of the bank
  size_t off_qf, off_qop, off_eps, off_mat, off_parts, off_band, off_cnt, off_cand, off_keys;
};
WidePoolPlan plan_score_wide_pool(const Dims& dm, const WidePlan& pl, int B, int M, int k);
int launch_score_wide_pool(const Dims& dm, const WidePoolPlan& pp, const void* q_route, int B, int M, const void* KR,
                           const float* inv_norm, int k, void* ws, hipStream_t st, int32_t* out_idx, float* out_score);

// Streaming loads of the routing index; cold: of one that the caches do not hold, or do and the kernel loses little.
bool stream_index_of(const Dims& dm, bool cold);

bool wide_path_applies(const Dims& dm, int BM);
WidePlan plan_score_wide(const Dims& dm, int BM, int k);
int launch_score_wide(const Dims& dm, const WidePlan& pl, const void* q_route, int BM, const void* KR,
                      const float* inv_norm, int k, void* ws, hipStream_t st, int32_t* out_idx, float* out_score,
                      unsigned long long* out_key);

// Bytes of the workspace that msa_score_topk_noalloc brings along.
constexpr size_t kNoAllocScratchBytes = (size_t)32 << 20;

// Work split of the routing scan (depends only on the problem size, so the workspace size is a
// pure function of the arguments).
struct ScorePlan {
  int n_splits;          // blocks per KV head
  int q_per_pass;        // queries scored per launch (8 or 16)
  int n_pass;
  int mode;              // scan mode: 0 filter, 1 dense lists, 2 score matrix + row top-k (all heads: always 2)
  int tiles_per_wave;    // mode 2: contiguous tiles per wave
  size_t off_mat;        // mode 2: byte offset of the fp32 score matrix [Hkv][BM][N]
  int exchange;          // 1: waves exchange running maxima to tighten their thresholds
  int it_publish, it_adopt;
  size_t off_gmax;       // byte offset of the exchange buffer inside the workspace
  size_t off_qop;        // byte offset of the prepared query operands
  int n_qtiles;          // 8-query operand tiles (padded to whole passes)
  int all_heads;         // 1: score_scan_all_kernel (scope ALL with more than one KV head)
  int seg_docs;          // all heads: documents per segment of the bank (one score matrix each)
  int part_docs;         // all heads: documents per part of a matrix row (n_splits parts per query in all)
  int window_parts;      // all heads: parts whose lists the buffer at the workspace's start holds
  int n_windows;         // > 1: a list per query and window at off_windows
  size_t off_windows;
  int n_sel;             // selections per query token: Hkv, or 1 for scope ALL
  size_t off_tok;        // byte offset of the per-token winner keys (token pooling)
  int merge_parts;       // > 1: two-level merge, first level over merge_lpp lists per block
  int merge_lpp;
  size_t off_part;       // byte offset of the first-level winners
  int nan_docs;          // 1: a query without a score that is a number selects the first k documents (the GEMM in the place of
                         // a scan of mode 2; its lists alone would have no entry)
  int use_wide;          // 1: all heads, more tokens than one pass of the scan -> msa_score_wide.hip
  WidePlan wide;
  int use_gemm;          // 1: many query tokens, a selection per KV group -> msa_score_gemm.hip
  GemmPlan gemm;
  size_t ws_bytes;       // the least that is accepted
  size_t ws_best;        // what is asked for
};
// The plan for a workspace of this size (0: whatever is asked for).
ScorePlan plan_score(const Dims& dm, int BM, int k, size_t workspace_bytes = 0);

// record the caller's per-call events (msa_config_t.profile_*_event) around the dominant kernel; null = off
inline void profile_mark(const Dims& dm, bool stop, hipStream_t st) {
  hipEvent_t e = stop ? dm.prof_stop : dm.prof_start;
  if (e != nullptr) (void)hipEventRecord(e, st);
}

// Many tokens with selections of their own, document by document (msa_attend_docs.hip).
constexpr size_t kDocsBytes = (size_t)256 << 20;  // per-token buffers of a window (partials above all)
constexpr int kDocsItems = 2048;                  // fewer items than this: documents in parts
struct DocsPlan {
  int parts, part_steps;  // parts of a document's rows, 32-row steps of each
  int chain;              // documents of one token that share a partial, at most, where hardly any are shared
  int tokens;             // query tokens per window; 0: the workspace is too small for this path
  size_t bytes;           // workspace asked for
};
bool docs_path_applies(const Dims& dm, int B, int M, int k);
DocsPlan plan_docs(const Dims& dm, int B, int M, int k, size_t bytes);

struct AttendPlan {
  int steps_mem;         // 32-key steps over the selected documents, ceil(k * G / 32)
  int steps_total;       // + ceil(Lloc / 32)
  int steps_per_split;
  int n_splits;
  int lin_per, lin_blocks;  // > 0: linear split of the decode kernel, steps per workgroup and workgroups (n_splits then
                            // is the most workgroups that can meet in one (query, KV head) pair)
  int prefill;           // 1: shared selection and many tokens -> attend_prefill_kernel
  int split_local;       // 1: per-token selections and many tokens: the selected documents go through the decode
                         //    kernel, the local context (shared by the tokens) through attend_prefill_kernel
  int mem_splits, mem_steps_per_split;  // split_local: decode kernel over the documents
  int loc_splits, loc_steps_per_split;  // split_local: tiled kernel over the local context
  int tpw, n_ttiles;     // prefill: tokens per wave (32 / r), token tiles (4 waves each) per batch row
  size_t off_ml;         // byte offset of the (m, l) pairs inside the workspace
  int fused_merge;       // 1: the decode kernel's last-arriving workgroup of a (query, KV head) merges the splits
  size_t off_tickets;    // byte offset of the arrival counters [B*M][Hkv] (64-bit)
  size_t off_krot;       // tiled kernel: byte offset of the once-rotated keys (0 = none)
  int krot_steps;        // steps per (batch row, KV head) held there
  size_t ws_bytes;       // the least that is accepted
  int docs;              // 1: split_local, and the documents go through attend_docs_kernel if the workspace holds ...
  size_t off_docs;       // ... its buffers from here on (ws_best bytes in all hold them as planned)
  size_t ws_best;
  DocsPlan dp;
};
AttendPlan plan_attend(const Dims& dm, int B, int M, int k, int Lloc, int bank_keys_rotated,
                       size_t workspace_bytes = 0);

int launch_build(const Dims& dm, const void* K, int doc_begin, int doc_count, void* KR,
                 float* inv_norm, hipStream_t st);
int launch_score(const Dims& dm, const ScorePlan& pl, const void* q_route, int B, int M, const void* KR,
                 const float* inv_norm, int k, int32_t* out_idx, float* out_score, void* ws,
                 hipStream_t st);
int launch_attend(const Dims& dm, const AttendPlan& pl, const void* q, int B, int M, const void* K,
                  const void* V, const int32_t* idx, int k, const void* Kloc, const void* Vloc,
                  int Lloc, int pos0, const int32_t* q_pos, void* out, float* lse, void* ws,
                  int bank_keys_rotated, hipStream_t st);
int launch_pool_kv(const Dims& dm, const void* K, const void* V, int doc_begin, int doc_count,
                   void* Kbar, void* Vbar, int32_t* pooled_lens, hipStream_t st);

int launch_fetch(const Dims& dm, const void* K_dev_view, const void* V_dev_view, const int32_t* idx,
                 long long n_rows, int k, void* K_stage, void* V_stage, int32_t* idx_stage,
                 int32_t* lens_stage, hipStream_t st);

inline size_t round_up256(size_t x) { return (x + 255) & ~(size_t)255; }

// A 48-bit non-zero value that differs from call to call (clock ticks through a 64-bit mixer): the tag of the
// arrival counters of one launch (arrive_at in msa_device.h).  It only has to differ from whatever the
// caller's workspace happens to hold.
unsigned long long launch_nonce48();

}  // namespace msa
