// Types shared by the attention kernels (decode: msa_attend.hip, shared-selection prefill:
// msa_attend_prefill.hip).
#pragma once
#include "msa_device.h"
#include "msa_host.h"

namespace msa {

constexpr int kAttWaves = 4;
constexpr int kMaxHalf = 64;  // d/2 <= 64

struct RopeTheta {
  double th[kMaxHalf];   // theta_u = base^(-2u/d), computed on the host in double
  float2 e1[kMaxHalf];   // (cos, sin)(theta_u), rounded from double on the host
  float2 e16[kMaxHalf];  // (cos, sin)(16 theta_u)
};

struct AttendArgs {
  const uint16_t* q;     // [BM][Hq][D]
  const uint16_t* K;     // [N][Hkv][G][D]
  const uint16_t* V;
  const int32_t* idx;    // [BM or B][Hkv or 1][k] (see idx_rows_per_b, idx_sel)
  const uint16_t* Kloc;  // [B][Hkv][Lloc][D]
  const uint16_t* Vloc;
  const int32_t* q_pos;  // [BM]
  const int32_t* lens;   // [N] document lengths (rows of a bank slot that exist), or null = G everywhere
  uint16_t* out;         // tiled kernel with a single split: the final output and (or null) log-sum-exp,
  float* lse;            // written directly instead of partials; null = partials
  const uint16_t* Krot;  // tiled kernel: keys of every step, rotated once, [B][Hkv][steps_total][D/8][32][8]; or null
  float* part_o;         // [BM][Hq][n_splits][D]   unnormalised partial outputs
  float2* part_ml;       // [BM][Hq][n_splits]      (running max in log2 units, sum)
  int M, Hq, Hkv, r, G, k, Lloc, pos0, N;
  int gshift;            // log2(G) when G < 32 (MODE 2)
  int idx_sel;           // selections per idx row: Hkv (one per KV group) or 1 (shared by all heads)
  int idx_rows_per_b;    // idx rows per batch row: M (one per query token) or 1 (shared by the M tokens)
  int steps_mem, steps_total, steps_per_split, n_splits;
  int ph_splits, split0;  // partial slots per (query, head) in the workspace, and this launch's first slot
  float qscale;          // log2(e) / sqrt(d)
  unsigned long long* tickets;  // decode kernel: arrival counters [BM][Hkv], or null = a separate merge launch
  unsigned long long nonce;     // this launch's tag of the counters (48 bits, non-zero)
  uint16_t* final_out;          // with tickets: the merged output [BM][Hq][D] and (or null) log-sum-exp
  float* final_lse;
  int lin_per, lin_total;  // decode kernel, linear split: steps per workgroup, steps in all; 0: the grid says it
};

// Many tokens with selections of their own, document by document (msa_attend_docs.hip): one window of tokens.
struct DocsArgs {
  unsigned long long* base;  // [S][N] first item << 32 | first entry of a document
  int* cnt;                  // [S][N] pairs of a document
  int* n_items;              // [S], and [S] 1 where the list is taken in chains
  uint4* qrot;               // [tokens][Hq][D/8][hi, lo] rotated, scaled queries, 8 bf16 each
  int4* items;               // [S][cap] (document, first entry, tokens, 1 if the document's only item) or, a chain,
                             // (token << 6 | number, first entry, documents, 2; the token's last 3)
  int* entries;              // [S][cap] token << 6 | slot, by document; of a chain its documents
  int* rank;                 // [S][tokens << kshift] place of a pair among its document's
  float* part_o;             // [tokens][Hq][k][parts][D] unnormalised partial outputs
  float2* part_ml;           // [tokens][Hq][k][parts]    (running max in log2 units, sum)
  int cap;                   // entries of a list at most
  int tile_tok;              // tokens per item at most, 16 / r
  int parts, part_steps;     // parts of a document's rows, 32-row steps of each
  int kshift;                // 2^kshift >= k
  int chain, n_chains;       // documents of a chain, chains of a token at most
  int tok0, n_tok, n_all;    // this window; tokens of the call
};
int launch_attend_docs(const Dims& dm, const DocsPlan& pl, const AttendArgs& a0, const RopeTheta& th, int BM, void* ws,
                       int bank_keys_rotated, const float* loc_o, const float2* loc_ml, int n_loc, void* out, float* lse,
                       hipStream_t st);

// Merge of many rows: n1 partials of rows [row0, row0 + rows) counted from row0 and n2 of all rows.  Of heads whose list
// (per_list heads of the Hq each) is chained the first n_chained of the n1 only.
int launch_merge2(int d, const float* o1, const float2* ml1, int n1, const float* o2, const float2* ml2, int n2, uint16_t* out,
                  float* lse, long long row0, long long rows, hipStream_t st, const int* chained = nullptr, int n_chained = 0,
                  int Hq = 1, int per_list = 1);

// Shared-selection prefill: unnormalised partials of every (token, head, split) in the layout the
// decode path writes, merged by the same attend_merge_kernel.
int launch_attend_prefill_partial(const Dims& dm, const AttendPlan& pl, const AttendArgs& a,
                                  const RopeTheta& th, int B, hipStream_t st, bool dominant);

}  // namespace msa
