// msa_score_topk with the head mean over EVERY head (select_scope = ALL, Eq. 2 of the paper as printed) for more query
// tokens than one pass of the all-heads scan takes (B*M > 32): the chunk score is the mean over the KV groups g of
//     inv_norm_g(key) * (qf_g(token) . key_g),
// qf_g the folded routing query of the group.  Every group has its own keys and reciprocal norms, so the groups'
// products cannot share an accumulator: each is scaled and added to a running total, eight groups of matrix work per
// score.  With one selection per token the scores themselves are few (4 B per token and document against
// 2 * Hkv * C * d flops), so they go to a score matrix and the selection is a kernel of its own.
//
//   fold_queries_kernel   folds the heads of every (token, group) into one fp32 query, and stores its bf16 hi part (or
//                         hi and lo parts) as MFMA operands.
//   score_wide_kernel     a workgroup holds the operands of 64 operand rows and all groups in LDS (128 KiB at Hkv = 8,
//                         d = 128) for its whole life; eight waves stream units of 64 keys straight into registers
//                         (the index is stored in operand order), multiply them with all 64 rows, group after group,
//                         and write the document maxima.  The waves never synchronise after the operands are in.
//   score_wide_rows_kernel    the same for up to 160 rows at once, one group's operands in LDS at a time.
//   score_wide_select_kernel  per token: the candidates of the matrix row and their exact scores.
//   pool_*_kernel             the same per batch row where the tokens are pooled.
//
// One pass (cosine, d = 128, eight chunks per document): only the hi parts are multiplied, 64 tokens per workgroup.  The
// matrix then holds scores within the bound eps that fold_queries_kernel writes; every document within 2 eps of the
// k-th best is scored again in fp32 from the folded fp32 query.  The bound takes |key| * inv_norm for one, which the
// interface asks of an index of that shape alone.  Otherwise, and for the dot product (keys of any length), hi and lo
// parts are neighbouring rows (32 tokens per workgroup), and the matrix holds the scores to ~16 bits of the query, as
// the scan's.
//
// Bound: the matrix cores, then LDS (every operand read feeds four products: 64 of 128 B per cycle and CU at the full
// matrix rate) and the L2 (a key is read once per 64 rows: 64 B per cycle and CU).  The workgroups of all token blocks
// that read the same keys sit on one XCD and walk them together, so the index comes from memory once per XCD-resident
// group of blocks. Measured: 150 tokens, k = 32, 97656 documents: kernel 3 x 142 us (three
// segments; 192 padded rows, 0.72 PFLOP/s), selection 18 + 18 + 46 us; the call 4.87 ms as 19 passes of the scan -> 0.50
// ms, before score_wide_rows_kernel and the pooling by document took that shape (0.31).  2048 tokens, 32768 documents, k = 8: 2.4 ms (a GEMM that reloaded its operands at every group switch) -> 1.47 ms.
#include "msa_device.h"
#include "msa_host.h"

#include <type_traits>

namespace msa {

constexpr int kWideWaves = 8;
constexpr int kWideRows = 64;    // operand rows per workgroup: four tiles of 16
constexpr int kWideTiles = 4;    // 16-key tiles per unit
constexpr int kWideGroups = 256; // workgroups: one per CU (LDS)
constexpr int kWidePass = 1024;  // query tokens per pass: bounds the workspace
constexpr size_t kWideMat = (size_t)20 << 20;  // bytes of the score matrix: bounds the workspace, stays in cache

struct WideArgs {
  const uint4* qop;        // [Hkv][n_rt][d/32][64] operand tiles of 16 rows
  const uint16_t* KR;
  const float* inv_norm;   // null: dot product
  float* mat;              // [tokens of the pass][mat_stride]
  long long mat_stride;
  int n_rt;                // operand tiles in all (a multiple of 4)
  int n_tb;                // token blocks (of 64 rows)
  int n_streams;           // key streams: n_tb * n_streams workgroups
  int nq;                  // tokens of the pass
  int C;
  long long tiles;         // tiles per head in the index
  long long tile0;         // first tile of the segment
  int seg_tiles, seg_docs; // tiles and documents of the segment
  int Hkv;
  int M;                   // pooled: tokens of a batch row ...
  int m_tiles, m_blocks;   // ... its operand tiles, its token blocks (not pooled: n_rt, n_tb)
};

// Head mean, document maxima (every lane of a document's C lanes gets it), scores of unit u to the matrix; tok0: token of the
// first operand row.
template <int NT, bool PAIR, int KT>
__device__ __forceinline__ void wide_store(const WideArgs& a, const float (&tot)[NT][KT][4], int u, int tok0, float inv_heads,
                                           int lane) {
  const int dpt = 16 / a.C;
  constexpr int NR = PAIR ? 2 : 4;  // tokens per lane and tile
  int le = lane;  // (opaque: worked out ahead of the caller's loop, what follows from it would take registers)
  asm volatile("" : "+v"(le));
  const int rr = le >> 4, n = le & 15;
#pragma unroll
  for (int tq = 0; tq < NT; ++tq) {
    float m[NR][KT];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) m[i][kt] = PAIR ? tot[tq][kt][2 * i] + tot[tq][kt][2 * i + 1] : tot[tq][kt][i];
    // one instruction per maximum (fmaxf of an exchanged value takes three: the exchange, and a canonicalising
    // maximum first); the exchange reads its operand two wait states after the write at the earliest
#define MSA_LEVEL(CTRL) \
  do { \
    for (int j = 0; j < NR * KT; j += 4) \
      asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 " CTRL " row_mask:0xf bank_mask:0xf\n\t" \
          "v_max_f32_dpp %1, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf\n\t" \
          "v_max_f32_dpp %2, %2, %2 " CTRL " row_mask:0xf bank_mask:0xf\n\t" \
          "v_max_f32_dpp %3, %3, %3 " CTRL " row_mask:0xf bank_mask:0xf" \
          : "+v"(m[j / KT][j % KT]), "+v"(m[(j + 1) / KT][(j + 1) % KT]), "+v"(m[(j + 2) / KT][(j + 2) % KT]), \
            "+v"(m[(j + 3) / KT][(j + 3) % KT])); \
  } while (0)
    static_assert((KT == 2 || KT == 4) && NR * KT % 4 == 0, "four values per statement");
    if (a.C >= 2) MSA_LEVEL("quad_perm:[1,0,3,2]");
    if (a.C >= 4) MSA_LEVEL("quad_perm:[2,3,0,1]");
    if (a.C >= 8) MSA_LEVEL("row_half_mirror");
    if (a.C >= 16) MSA_LEVEL("row_mirror");
#undef MSA_LEVEL
    // The C lanes of a document take the unit's tiles in turn, up to four at once: one store then writes up to
    // 4 dpt documents of a token (a run of 32 bytes at C = 8).
    const int par = a.C < KT ? a.C : KT;   // tiles per store
    for (int k0 = 0; k0 < KT; k0 += par) {  // wave-uniform
      const int kt = k0 + (n & (par - 1));
      const int doc = (u * KT + kt) * dpt + n / a.C;
      const bool on = (n & (a.C - 1)) < par && doc < a.seg_docs;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int tok = tok0 + tq * (PAIR ? 8 : 16) + rr * NR + i;
        // (through empty asm: as selects between elements of the array they would become an indexed load of it)
        float c0 = m[i][0], c1 = m[i][1], c2 = m[i][KT - 2], c3 = m[i][KT - 1];
        asm volatile("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
        const float lo = (kt & 1) ? c1 : c0, hi = (kt & 1) ? c3 : c2;
        if (on && tok < a.nq) a.mat[tok * a.mat_stride + doc] = fmaxf(((kt & 2) ? hi : lo) * inv_heads, -INFINITY);  // (not a number: last)
      }
    }
  }
}

// STREAM: streaming loads of the keys (a single token block: nobody else reads them).
template <int D, int HKV, bool PAIR, bool COS, bool STREAM>
__global__ __launch_bounds__(64 * kWideWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void score_wide_kernel(WideArgs a) {
  constexpr int NS = D / 32;
  constexpr int NT = kWideRows / 16;
  constexpr int KT = kWideTiles;
  constexpr int TILE_ELEMS = 16 * D;
  constexpr int NOP = HKV * NT * NS;  // KiB of operands
  static_assert(NOP % kWideWaves == 0 && HKV % 2 == 0, "whole copies per wave; ring of two entries");

  __shared__ uint4 Aop[HKV][NT][NS][64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups go to the eight XCDs in turn (blockIdx % 8); each XCD takes a run of (stream, token block) pairs, so the
  // token blocks of a key stream share an XCD.
  const int total = a.n_tb * a.n_streams;
  const int vb = (blockIdx.x & 7) * ((total + 7) / 8) + (blockIdx.x >> 3);
  if (vb >= total) return;  // the grid is rounded up to whole XCDs
  const int tb = vb % a.n_tb;
  const int stream = vb / a.n_tb;

  // ---- operands: global -> LDS, requested first; the keys requested next stay in flight across their wait ---------
  const uint32_t op_lds = lds_addr_of(&Aop[0][0][0][0]);
#pragma unroll
  for (int i = 0; i < NOP / kWideWaves; ++i) {
    const int e = i * kWideWaves + wave;  // (group, tile, slice)
    const int g = e / (NT * NS), rest = e % (NT * NS);
    const uint4* src = a.qop + (((long long)g * a.n_rt + tb * NT) * NS + rest) * 64;
    copy16_to_lds_async_at(src, lane * 16, op_lds + e * 1024);
  }

  const int W = a.n_streams * kWideWaves;
  const int w = stream * kWideWaves + wave;
  const int units = (a.seg_tiles + KT - 1) / KT;
  // Addresses: a base that is the same in every lane (scalar registers) plus the lane's own 32-bit offset, which is
  // worked out from an opaque copy of the lane number every time: known ahead of the loop it would be added to the bases
  // there, and the sums would need registers the loop does not have.
  typedef const __attribute__((address_space(1))) char* gptr_t;
  const gptr_t kr0 = (gptr_t)a.KR + a.tile0 * (TILE_ELEMS * 2);
  const gptr_t in0 = (gptr_t)a.inv_norm + a.tile0 * 64;  // (COS only)
  const int last_tile = a.seg_tiles - 1;

  u32x4_t buf[2][KT][NS];
  float binv[2][KT];
  // unit u, group g into ring slot: always issued, past the end the last tile again
  auto request = [&](int u, int g, u32x4_t (&b)[KT][NS], float (&bi)[KT]) __attribute__((always_inline)) {
    uint32_t ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      int t = u * KT + kt;
      t = t < last_tile ? t : last_tile;
      const long long at = g * a.tiles + t;
      const gptr_t p = kr0 + at * (TILE_ELEMS * 2);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const auto from = (const __attribute__((address_space(1))) u32x4_t*)(p + s * 1024 + (size_t)(ln * 16));
        b[kt][s] = STREAM ? __builtin_nontemporal_load(from) : *from;
      }
      if constexpr (COS) bi[kt] = *(const __attribute__((address_space(1))) float*)(in0 + at * 64 + (size_t)((ln & 15) * 4));
    }
  };
  request(w, 0, buf[0], binv[0]);
  request(w, 1, buf[1], binv[1]);
  wait_copies_but<2 * KT * (NS + (COS ? 1 : 0))>();  // the operands are older than the keys
  lds_barrier();

  const float inv_heads = 1.0f / (float)HKV;
  // The operand reads run two ahead of the products (a ring of four slices that goes on from group to group): four
  // products of 16 cycles each per read, so a read has about 128 cycles to land.  The order is the one written here:
  // left to itself the scheduler reads every slice right before its products.
  constexpr int NA = NT * NS;  // slices per group
  bf16x8_t ar[4];
  const uint4* const A0 = &Aop[0][0][0][0] + lane;
  ar[0] = as_bf16x8(A0[0]);
  ar[1] = as_bf16x8(A0[64]);
  for (int u = w; u < units; u += W) {
    float tot[NT][KT][4];
#pragma unroll
    for (int g = 0; g < HKV; ++g) {
      const int slot = g & 1;
      // the entry is awaited HERE: its uses pass through volatile asm, so that no use of a later entry (and the wait
      // for it) moves up ahead of the requests in between
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
        for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(buf[slot][kt][s]));
        if constexpr (COS) asm volatile("" : "+v"(binv[slot][kt]));
      }
#pragma unroll
      for (int tq = 0; tq < NT; ++tq) {
        f32x4_t acc[KT];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int i = tq * NS + s;
          static_assert(NA % 4 == 0, "ring slots must be compile-time");
          ar[(i + 2) & 3] = as_bf16x8(A0[((g * NA + i + 2) % (HKV * NA)) * 64]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int kt = 0; kt < KT; ++kt)
            acc[kt] = mfma16(ar[i & 3], __builtin_bit_cast(bf16x8_t, buf[slot][kt][s]),
                             s == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[kt]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (COS)
              tot[tq][kt][i] = g == 0 ? acc[kt][i] * binv[slot][kt] : fmaf(acc[kt][i], binv[slot][kt], tot[tq][kt][i]);
            else
              tot[tq][kt][i] = g == 0 ? acc[kt][i] : tot[tq][kt][i] + acc[kt][i];
          }
        // the totals are formed HERE (deferred, the accumulators of all tiles would be live together)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
          asm volatile("" : "+v"(tot[tq][kt][0]), "+v"(tot[tq][kt][1]), "+v"(tot[tq][kt][2]), "+v"(tot[tq][kt][3]));
        __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("" ::: "memory");  // every product of the entry is issued before its slot is requested again
      request(g + 2 < HKV ? u : u + W, (g + 2) % HKV, buf[slot], binv[slot]);
      __builtin_amdgcn_sched_barrier(0);
    }

    wide_store<NT, PAIR, KT>(a, tot, u, tb * (kWideRows / (PAIR ? 2 : 1)), inv_heads, lane);
  }
}

// ---- more than 64 operand rows: a key is read once for up to 160 ----------------------------------------------------
// score_wide_kernel with NT tiles of 16 rows (cosine, d = 128, one-pass): the operands of one group at a time lie in LDS,
// 4 NT KiB, two groups in turn; the next group's are copied there (from the L2, all workgroups read the same ones) while this
// one's are multiplied.  Eight waves, two per SIMD: 32 keys and all rows each, totals of 8 NT registers, the keys of two
// groups 64.  The waves meet once per group, 8 NT products each.  Bound by the index (1.6 GB: 232 us) and, with 160 rows, the
// operand reads from LDS, as many cycles as the products take.  (Four waves of 64 keys would halve the reads; their totals
// and keys need the accumulation half of the register file, and the copies in and out of it cost as much.)
constexpr int kRowsWaves = 8;
constexpr int kRowsTiles = 2;   // 16-key tiles per unit
constexpr int kRowsMost = 10;   // tiles of 16 rows

// The best score of a block's tokens (the first n_rows operand rows) for the documents of unit u.
template <int NT, int KT>
__device__ __forceinline__ void wide_store_pooled(const WideArgs& a, const float (&tot)[NT][KT][4], int u, int tb, int n_rows,
                                                  float inv_heads, int lane) {
  int le = lane;  // (opaque, see wide_store)
  asm volatile("" : "+v"(le));
  const int rr = le >> 4, n = le & 15;
  float best[KT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) best[kt] = -INFINITY;
#pragma unroll
  for (int tq = 0; tq < NT; ++tq) {
    if (16 * tq + 16 <= n_rows) {  // wave-uniform
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) best[kt] = fmaxf(best[kt], tot[tq][kt][i]);
    } else if (16 * tq < n_rows) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) best[kt] = fmaxf(best[kt], 16 * tq + 4 * rr + i < n_rows ? tot[tq][kt][i] : -INFINITY);
    }
  }
  float mine = -INFINITY;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    best[kt] = fmaxf(best[kt], __shfl_xor(best[kt], 16, 64));
    best[kt] = fmaxf(best[kt], __shfl_xor(best[kt], 32, 64));
    best[kt] = group_max<8>(best[kt]);  // the eight chunks of a document
    mine = (n & 7) == kt ? best[kt] : mine;
  }
  const int doc = 2 * (u * KT + (n & 7)) + (n >> 3);
  if (rr == 0 && (n & 7) < KT && doc < a.seg_docs) a.mat[tb * a.mat_stride + doc] = fmaxf(mine * inv_heads, -INFINITY);  // (not a number: last)
}

// POOL: token pooling, the matrix holds the best score of a block's tokens.  STREAM: streaming loads of the keys, with pooling where
// the scans have them too (stream_index_of; index cold / again and again, whole call, 150 tokens: 9000 documents 73.8 / 67.7 -> 71.9 /
// 71.7 us, 15600 76.6 / 69.7 -> 74.6 / 73.7, 20000 97.0 / 95.3 -> 93.0 / 91.0), without from 300 MB on only: below, little is gained
// (9000 documents 82.2 / 75.4 -> 82.0 / 79.8, 13000 86.0 / 79.9 -> 85.5 / 83.9; 20000 113.5 / 109.8 -> 112.1 / 110.2, 70 tokens 99.1 /
// 97.4 -> 96.3 / 93.6).
template <int NT, bool POOL, bool STREAM>
__global__ __launch_bounds__(64 * kRowsWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void score_wide_rows_kernel(WideArgs a) {
  constexpr int D = 128;
  constexpr int NS = D / 32;
  constexpr int KT = kRowsTiles;
  constexpr int TILE_ELEMS = 16 * D;
  constexpr int NOP = NT * NS;              // KiB of operands of a group
  constexpr int OPW = NOP / kRowsWaves;     // copies of a wave
  static_assert(NOP % kRowsWaves == 0, "whole copies per wave");

  __shared__ uint4 Aop[2][NT][NS][64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int total = a.n_tb * a.n_streams;
  const int vb = (blockIdx.x & 7) * ((total + 7) / 8) + (blockIdx.x >> 3);  // (see score_wide_kernel)
  if (vb >= total) return;  // block-uniform: the grid is rounded up to whole XCDs
  const int tb = vb % a.n_tb;
  const int stream = vb / a.n_tb;
  const int Hkv = a.Hkv;

  const uint32_t op_lds = lds_addr_of(&Aop[0][0][0][0]);
  const int tile_0 = tb / a.m_blocks * a.m_tiles + tb % a.m_blocks * NT;  // first operand tile
  const int tile_n = (tb / a.m_blocks + 1) * a.m_tiles - 1;                // last one of the batch row
  // operands of group g -> place g & 1; row tiles past the last one: that one again (their scores are not stored)
  auto copy_operands = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < OPW; ++i) {
      const int e = i * kRowsWaves + wave;  // (tile, slice)
      int t = tile_0 + e / NS;
      t = t < tile_n ? t : tile_n;
      const uint4* src = a.qop + (((long long)g * a.n_rt + t) * NS + e % NS) * 64;
      copy16_to_lds_async_at(src, lane * 16, op_lds + (g & 1) * (NOP * 1024) + e * 1024);
    }
  };

  const int W = a.n_streams * kRowsWaves;
  const int units = (a.seg_tiles + KT - 1) / KT;
  typedef const __attribute__((address_space(1))) char* gptr_t;
  const gptr_t kr0 = (gptr_t)a.KR + a.tile0 * (TILE_ELEMS * 2);
  const gptr_t in0 = (gptr_t)a.inv_norm + a.tile0 * 64;
  const int last_tile = a.seg_tiles - 1;

  u32x4_t buf[2][KT][NS];
  float binv[2][KT];
  constexpr int kLoads = KT * (NS + 1);  // of a request
  // unit u, group g into ring slot: always issued, past the end the last tile again
  auto request = [&](int u, int g, u32x4_t (&b)[KT][NS], float (&bi)[KT]) __attribute__((always_inline)) {
    uint32_t ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      int t = u * KT + kt;
      t = t < last_tile ? t : last_tile;
      const long long at = g * a.tiles + t;
      const gptr_t p = kr0 + at * (TILE_ELEMS * 2);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const auto from = (const __attribute__((address_space(1))) u32x4_t*)(p + s * 1024 + (size_t)(ln * 16));
        b[kt][s] = STREAM ? __builtin_nontemporal_load(from) : *from;
      }
      bi[kt] = *(const __attribute__((address_space(1))) float*)(in0 + at * 64 + (size_t)((ln & 15) * 4));
    }
  };
  const int u_first = stream * kRowsWaves;
  copy_operands(0);
  request(u_first + wave, 0, buf[0], binv[0]);
  request(u_first + wave, 1, buf[1], binv[1]);

  const float inv_heads = 1.0f / (float)Hkv;
  constexpr int NA = NT * NS;  // slices of a group
  constexpr int kAhead = 6;    // slices read ahead of their products: two products of 16 cycles each, an LDS read takes over 100
  float tot[NT][KT][4];
  // One group: products of its keys with all rows, into the totals; PAR: its place.
  auto group = [&](auto par_c, int u, int g) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par_c)::value;
    // This group's keys and operands have landed (the next group's keys, the youngest, may be on their way); behind the
    // barrier everyone's part of the operands has, and everyone is done with the place of the group before.
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(buf[PAR][kt][s]));
      asm volatile("" : "+v"(binv[PAR][kt]));
    }
    wait_copies_but<kLoads>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    copy_operands(g + 1 < Hkv ? g + 1 : 0);
    const uint4* const A0 = &Aop[PAR][0][0][0] + lane;
    bf16x8_t ar[8];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) ar[i] = as_bf16x8(A0[i * 64]);
#pragma unroll
    for (int tq = 0; tq < NT; ++tq) {
      f32x4_t acc[KT];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = tq * NS + s;
        if (i + kAhead < NA) ar[(i + kAhead) & 7] = as_bf16x8(A0[(i + kAhead) * 64]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
          acc[kt] = mfma16(ar[i & 7], __builtin_bit_cast(bf16x8_t, buf[PAR][kt][s]),
                           s == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : acc[kt]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[tq][kt][i] = fmaf(acc[kt][i], binv[PAR][kt], tot[tq][kt][i]);
    }
    asm volatile("" ::: "memory");  // every product of the entry is issued before its slot is requested again
    request(g + 2 < Hkv ? u : u + W, g + 2 < Hkv ? g + 2 : g + 2 - Hkv, buf[PAR], binv[PAR]);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int ub = u_first; ub < units; ub += W) {  // block-uniform
    const int u = ub + wave;
#pragma unroll
    for (int tq = 0; tq < NT; ++tq)
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[tq][kt][i] = 0.f;
    for (int g = 0; g < Hkv; g += 2) {
      group(std::integral_constant<int, 0>{}, u, g);
      group(std::integral_constant<int, 1>{}, u, g + 1);
    }
    if (u < units) {
      if constexpr (POOL) wide_store_pooled<NT, KT>(a, tot, u, tb, a.M - tb % a.m_blocks * (NT * 16), inv_heads, lane);
      else wide_store<NT, false, KT>(a, tot, u, tb * NT * 16, inv_heads, lane);
    }
  }
  wait_copies_but<0>();  // (requests past the end)
}

// ---- selection -------------------------------------------------------------------------------------------------
// One workgroup per token.  Input: the token's matrix row of a segment (scores s~ within eps of the exact scores s;
// eps = 0: the exact scores), and the k best of the segments before, as sorted keys with exact scores.  Let t~ be the
// k-th largest s~ of the segment.  k documents have s >= t~ - eps, so a document of the exact k best has
// s~ >= s - eps >= t~ - 2 eps; and it is none of the k best if s~ + eps is below the k-th best exact score so far.
//   1. a lower bound theta of t~ (kth_best_bound); the documents with s~ >= theta - 2 eps go to LDS;
//   2. t~ by rank counting among them; what is left of them after the two conditions are the candidates;
//   3. the candidates' exact scores: Eq. 2 in fp32 from the folded fp32 query and the bf16 keys, eight lanes per key;
//   4. the k best of candidates and earlier winners by rank counting on the full key.
// With several segments and room for the lists (WideSelArgs::list) the exact scores wait for the last one: a segment leaves
// its candidates, as keys of matrix scores, in the token's list of up to kWideList, t~ is the k-th largest of list and
// segment, and what falls below t~ - 2 eps is dropped.  Step 3, a gather of 16 KiB per document, is then done for the
// candidates of the whole bank and not of each segment (150 tokens, k = 32, 97656 documents, three segments: selection 57 + 51 + 30 us -> 18 + 18 + 46).  A list
// that would grow longer (copies of a few documents) is scored, and the token goes on with exact winners.
// If more survive than LDS holds (ties), topk_of_ties takes the k best where the matrix holds the exact scores; else
// the row is taken in windows of kWideSurv documents: step 3 and 4 for those of a window that can still be among the k
// best.  (150 tokens, 50 of them zeros, k = 32, 97656 documents: through the windows the call took 57 ms, now 0.57; 100
// tokens whose best 4000 documents are copies of two, of 8192: 2.2 ms, bound by the exact scores of the copies.)
constexpr int kWideSel = 512;      // threads
constexpr int kWideSurv = 2048;
constexpr int kWideList = 160;     // candidates that wait for the last segment
constexpr int kWideRegs = 64;      // scores a thread keeps in registers (16: short rows)

struct WideSelArgs {
  const float* mat;
  long long mat_stride;
  const float* eps;        // BAND: [tokens][Hkv]
  const float* qf;         // BAND: [tokens][Hkv][d]
  const uint16_t* KR;
  const float* inv_norm;
  unsigned long long* best;  // [tokens][k] keys of the segments so far
  unsigned long long* list;  // BAND: [tokens][kWideList] candidates of the segments so far; null: exact winners in best
  uint2* list_n;             // [tokens] (entries, image of the k-th largest; 0: fewer than k); (~0, ..): winners in best
  int first, last;           // first segment: nothing in best yet; last: the result goes out
  int32_t* out_idx;
  float* out_score;
  unsigned long long* out_key;
  int Hkv, k;
  int n_docs, doc0;        // documents of the segment, number of the first
  int tok0;                // token number of the pass's first token
  long long tiles;
};

// BAND: the matrix holds the one-pass scores (d = 128, eight chunks per document).
template <bool BAND, int REGS>
__global__ __launch_bounds__(kWideSel) void score_wide_select_kernel(WideSelArgs a) {
  constexpr int NW = kWideSel / 64;
  constexpr int D = 128, C = 8;
  constexpr int kMost = kWideSurv + (BAND ? kWideList : 0);  // candidates at a time
  __shared__ unsigned long long surv[kMost + MSA_MAX_TOPK + 8];
  __shared__ float qs[BAND ? 8 * D : 1];
  __shared__ unsigned long long best_s[MSA_MAX_TOPK];
  __shared__ uint32_t theta_w[2][NW];
  __shared__ uint32_t kth_s;
  __shared__ int cnt_s[NW];
  __shared__ int n_surv;
  const int tid = threadIdx.x;
  const int tok = blockIdx.x;
  const int k = a.k, N = a.n_docs;
  const float* __restrict__ row = a.mat + (long long)tok * a.mat_stride;
  float eps = 0.f;
  if constexpr (BAND) {
    for (int g = 0; g < a.Hkv; ++g) eps += a.eps[(long long)tok * a.Hkv + g];
    eps /= (float)a.Hkv;
    for (int i = tid; i < a.Hkv * D; i += kWideSel) qs[i] = a.qf[(long long)tok * a.Hkv * D + i];
  }
  int n_best = 0;  // earlier winners
  int n_list = 0;  // earlier candidates
  uint32_t list_kth = 0u;
  bool listed = BAND && a.list != nullptr;
  if (listed && !a.first) {
    const uint2 l = a.list_n[tok];
    listed = l.x != ~0u;
    n_list = listed ? (int)l.x : 0;
    list_kth = l.y;
  }
  unsigned long long* const list = listed ? a.list + (long long)tok * kWideList : nullptr;
  if (!a.first && !listed) {
    n_best = k;
    if (tid < k) best_s[tid] = a.best[(long long)tok * k + tid];
  }
  if (tid == 0) n_surv = 0;

  // exact scores of the documents surv[0 .. ns), in place of their keys; eight lanes per (document, chunk)
  auto rescore = [&](int ns) {
    if constexpr (!BAND) return;
    const int part = tid & 7;
    constexpr int per = kWideSel / 8 / C;    // documents per round: one per wave
    const int ch = (tid >> 3) & (C - 1);
    const float inv_g = 1.0f / (float)a.Hkv;
    for (int j0 = 0; j0 < ns; j0 += per) {   // block-uniform
      const int j = j0 + (tid >> 3) / C;
      const uint32_t doc = key_doc(surv[j < ns ? j : ns - 1]);
      const long long key = (long long)doc * C + ch;
      const uint16_t* kp = a.KR + (key >> 4) * (16 * D) + (part * (D / 64) * 16 + (int)(key & 15)) * 8;
      float tot = 0.f;
      for (int g0 = 0; g0 < a.Hkv; g0 += 4) {  // the loads of four groups in flight (Hkv = 2: the last one again, dropped)
        uint4 kv[4][D / 64];
        float inv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int g = g0 + u < a.Hkv ? g0 + u : a.Hkv - 1;
          const uint16_t* p = kp + (long long)g * a.tiles * (16 * D);
#pragma unroll
          for (int x = 0; x < D / 64; ++x)   // dims (D/8) part .. + D/8: pieces of 8, 128 elements apart in a tile
            kv[u][x] = *reinterpret_cast<const uint4*>(p + x * 128);
          inv[u] = a.inv_norm[(long long)g * a.tiles * 16 + key];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (g0 + u >= a.Hkv) break;  // block-uniform
          float acc = 0.f;
#pragma unroll
          for (int x = 0; x < D / 64; ++x) {
            const float* q = &qs[(g0 + u) * D + part * (D / 8) + 8 * x];
            const uint4 w = kv[u][x];
            acc = fmaf(q[0], bf16_lo(w.x), acc);
            acc = fmaf(q[1], bf16_hi(w.x), acc);
            acc = fmaf(q[2], bf16_lo(w.y), acc);
            acc = fmaf(q[3], bf16_hi(w.y), acc);
            acc = fmaf(q[4], bf16_lo(w.z), acc);
            acc = fmaf(q[5], bf16_hi(w.z), acc);
            acc = fmaf(q[6], bf16_lo(w.w), acc);
            acc = fmaf(q[7], bf16_hi(w.w), acc);
          }
          acc += dpp_f<kDppXor1>(acc);
          acc += dpp_f<kDppXor2>(acc);
          acc += dpp_f<kDppHalfMirror>(acc);   // the key's dot product, in its eight lanes
          tot += acc * inv[u];
        }
      }
      float sc = tot * inv_g;
#pragma unroll
      for (int off = 8; off < 8 * C; off <<= 1) sc = fmaxf(sc, __shfl_xor(sc, off, 64));
      __syncthreads();  // every lane has read its document
      if (part == 0 && ch == 0 && j < ns) surv[j] = make_key(sc, doc);
    }
    __syncthreads();
  };
  // surv[0 .. ns) and best_s[0 .. n_best): the k best, sorted, into best_s
  auto merge = [&](int ns) {
    __syncthreads();
    if (tid < n_best) surv[ns + tid] = best_s[tid];
    if (tid < 8) surv[ns + n_best + tid] = 0ull;  // read eight at a time below (zero: greater than no key)
    __syncthreads();
    const int all = ns + n_best;
    for (int i = tid; i < all; i += kWideSel) {
      const unsigned long long x = surv[i];
      int rank = 0;
      for (int j = 0; j < all; j += 8) {
        unsigned long long y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = surv[j + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (y[u] > x) ? 1 : 0;
      }
      if (rank < k && x != 0ull) best_s[rank] = x;
    }
    n_best = all < k ? all : k;  // (documents are distinct, so are their keys)
    __syncthreads();
  };
  // lowest matrix value that can still be among the k best, as the order-preserving image of a score
  auto floor_of = [&](float t, float width) { return orderable(t - width); };

  // ---- 1. theta ------------------------------------------------------------------------------------------------
  float v[REGS];
#pragma unroll
  for (int u = 0; u < REGS; ++u) {
    const int i = u * kWideSel + tid;
    v[u] = (i < N) ? row[i] : -INFINITY;
  }
  // the rest of a row longer than the registers hold, eight loads in flight
  auto rest_of_row = [&](auto use) {
    for (int i0 = REGS * kWideSel + tid; i0 < N; i0 += 8 * kWideSel) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = (i0 + u * kWideSel < N) ? row[i0 + u * kWideSel] : -INFINITY;
#pragma unroll
      for (int u = 0; u < 8; ++u) use(i0 + u * kWideSel, x[u]);
    }
  };
  uint32_t ob = 0u;  // the best score of this lane (0: no document)
  auto best_of = [&](int i, float x) {
    const uint32_t o = i < N ? orderable(x) : 0u;
    ob = o > ob ? o : ob;
  };
#pragma unroll
  for (int u = 0; u < REGS; ++u) best_of(u * kWideSel + tid, v[u]);
  rest_of_row(best_of);
  const uint32_t theta = kth_best_bound<NW>(ob, k, theta_w);
  uint32_t lim = theta ? floor_of(unorderable(theta), 2.f * eps) : 0u;
  if (listed) {
    const uint32_t l2 = list_kth ? floor_of(unorderable(list_kth), 2.f * eps) : 0u;
    lim = l2 > lim ? l2 : lim;
  } else if (!a.first) {  // the k-th best so far (0: fewer than k)
    const unsigned long long kb = best_s[k - 1];
    // (a tie loses to the documents of earlier segments)
    const uint32_t l2 = kb ? floor_of(key_score(kb), eps) + 1u : 0u;
    lim = l2 > lim ? l2 : lim;
  }
  auto keep = [&](int i, float s) {
    if (i < N && orderable(s) >= lim) {
      const int slot = atomicAdd(&n_surv, 1);
      if (slot < kWideSurv) surv[slot] = make_key(s, (uint32_t)(a.doc0 + i));
    }
  };
#pragma unroll
  for (int u = 0; u < REGS; ++u) keep(u * kWideSel + tid, v[u]);
  rest_of_row(keep);
  __syncthreads();
  int ns = n_surv;
  __syncthreads();
  const bool over = ns > kWideSurv;  // block-uniform, as all below
  if (n_list > 0) {
    const int at = over ? 0 : ns;
    if (tid < n_list) surv[at + tid] = list[tid];
    ns += n_list;
    __syncthreads();
    if (over) {  // exact winners of those before
      rescore(n_list);
      merge(n_list);
    }
  }
  if (over) listed = false;
  if (!over) {
    // ---- 2. t~, candidates -----------------------------------------------------------------------------------------
    if (BAND && ns > k) {
      if (tid < 8) surv[ns + tid] = 0ull;
      __syncthreads();
      constexpr int kMine = (kMost + kWideSel - 1) / kWideSel;
      unsigned long long mine[kMine];
#pragma unroll
      for (int u = 0; u < kMine; ++u) {
        const int i = u * kWideSel + tid;
        mine[u] = i < ns ? surv[i] : 0ull;
        if (u * kWideSel < ns) {  // block-uniform
          int rank = 0;
          for (int j = 0; j < ns; j += 8) {
            unsigned long long y[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) y[q] = surv[j + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) rank += (y[q] > mine[u]) ? 1 : 0;
          }
          if (i < ns && rank == k - 1) kth_s = (uint32_t)(mine[u] >> 32);
        }
      }
      if (tid == 0) n_surv = 0;
      __syncthreads();
      list_kth = kth_s;
      const uint32_t l2 = floor_of(unorderable(list_kth), 2.f * eps);
      lim = l2 > lim ? l2 : lim;
#pragma unroll
      for (int u = 0; u < kMine; ++u)
        if (mine[u] != 0ull && (uint32_t)(mine[u] >> 32) >= lim) surv[atomicAdd(&n_surv, 1)] = mine[u];
      __syncthreads();
      ns = n_surv;
    }
    if (listed && !a.last && ns <= kWideList) {
      if (tid < ns) a.list[(long long)tok * kWideList + tid] = surv[tid];
      if (tid == 0) a.list_n[tok] = make_uint2((uint32_t)ns, list_kth);
      return;
    }
    // ---- 3., 4. ------------------------------------------------------------------------------------------------------
    rescore(ns);
    merge(ns);
  } else if (eps == 0.f) {  // block-uniform: the matrix holds the exact scores (and those of a query of zeros)
    topk_of_ties<REGS, NW>(v, row, N, (uint32_t)a.doc0, k, theta, ob, surv, &n_surv, cnt_s);
    merge(k);
  } else {
    for (int w0 = 0; w0 < N; w0 += kWideSurv) {  // block-uniform
      if (tid == 0) n_surv = 0;
      const unsigned long long kb = n_best == k ? best_s[k - 1] : 0ull;
      const uint32_t l2 = kb ? floor_of(key_score(kb), eps) + 1u : 0u;
      __syncthreads();
      for (int i = w0 + tid; i < w0 + kWideSurv && i < N; i += kWideSel) {
        const uint32_t o = orderable(row[i]);
        if (o >= lim && o >= l2) surv[atomicAdd(&n_surv, 1)] = make_key(row[i], (uint32_t)(a.doc0 + i));
      }
      __syncthreads();
      ns = n_surv;
      __syncthreads();
      rescore(ns);
      merge(ns);
    }
  }
  if (BAND && tid == 0 && a.list != nullptr) a.list_n[tok] = make_uint2(~0u, 0u);
  if (tid < k) {
    const unsigned long long x = tid < n_best ? best_s[tid] : 0ull;
    const long long o = (long long)(a.tok0 + tok) * k + tid;
    if (!a.last) {
      a.best[(long long)tok * k + tid] = x;
    } else if (a.out_key != nullptr) {
      a.out_key[o] = x;
    } else {
      a.out_idx[o] = x ? (int32_t)key_doc(x) : -1;
      if (a.out_score != nullptr) a.out_score[o] = x ? key_score(x) : -INFINITY;
    }
  }
}


// ---- token pooling -------------------------------------------------------------------------------------------------
// The score of a document is its best over the tokens of a batch row, so no token needs a selection of its own.  The scoring
// kernel leaves, per document, the best matrix score P~ of every block of tokens (within E, the largest of the tokens' bounds, of
// the best exact score P); then, all per batch row:
//   pool_parts_kernel   the best P~ of each of up to 512 parts of the bank, and E
//   pool_cand_kernel    theta, a lower bound on the k-th best P~ from the parts' (kth_best_bound); the documents with
//                       P~ >= theta - 2 E: the k best by P are among them (k documents have P >= theta - E)
//   pool_score_kernel   their exact scores with every token, Eq. 2 in fp32 as in score_wide_select_kernel, and the best of them
//   pool_best_kernel    the k best candidates
// Where E is zero (queries of zeros) P~ is P, and of the documents that tie with theta a workgroup lists the first k at most, less
// the parts ahead of it that reach theta (a question of 150 zeros, 8192 documents, k = 32: with the first k of every workgroup, more
// than pool_best_kernel holds, whole call 99 us, now 45).
// 150 tokens, k = 32, 97656 documents: a selection for every token (matrix of 58 MB in three segments) and their pooling, whole
// call 435 us, this way 325; 600 tokens, 30000 documents 503 -> 336, 150 over 300 48.8 -> 46.9.
constexpr int kPoolParts = 512;
constexpr int kPoolMost = 1024;  // tokens of a batch row
constexpr int kPoolTok = 4;      // tokens per workgroup of pool_score_kernel

struct WidePoolArgs {
  const float* mat;        // [B * m_blocks][N]
  const float* eps;        // [B * M][Hkv]
  const float* qf;         // [B * M][Hkv][128]
  const uint16_t* KR;
  const float* inv_norm;
  float* parts;            // [B][kPoolParts]
  float* band;             // [B] E
  int* cnt;                // [B] candidates
  int* cand;               // [B][N]
  unsigned long long* keys;  // [B][N] best exact score of a candidate
  int32_t* out_idx;
  float* out_score;
  int N, M, Hkv, k, m_blocks, part_docs, n_parts;
  int block_tokens;        // tokens of a block
  long long tiles;
};

// ranks below every number
__device__ __forceinline__ float not_a_number() { return __uint_as_float(0xffc00000u); }

__device__ __forceinline__ float pooled_of(const WidePoolArgs& a, int b, int doc) {
  const float* p = a.mat + (long long)b * a.m_blocks * a.N + doc;
  float x = p[0];
  for (int i = 1; i < a.m_blocks; ++i) x = fmaxf(x, p[(long long)i * a.N]);
  return x;
}

// a wave per part; the last workgroup of a batch row: E
__global__ __launch_bounds__(256) void pool_parts_kernel(WidePoolArgs a) {
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y;
  float best = -INFINITY;
  bool listed = false;  // a token that is not a number and lists documents all the same, as a selection per token has it
  if (blockIdx.x == gridDim.x - 1) {  // block-uniform
    best = 0.f;
    for (int m = tid; m < a.M; m += 256) {
      float e = 0.f;
      for (int g = 0; g < a.Hkv; ++g) e += a.eps[((long long)b * a.M + m) * a.Hkv + g];
      best = fmaxf(best, e / (float)a.Hkv);
      listed = listed || (e != e && __float_as_int(e) < 0);
    }
  } else {
    const int part = blockIdx.x * 4 + wave;
    const int d0 = part * a.part_docs, d1 = d0 + a.part_docs < a.N ? d0 + a.part_docs : a.N;
    for (int d = d0 + lane; d < d1; d += 64) best = fmaxf(best, pooled_of(a, b, d));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
  if (blockIdx.x == gridDim.x - 1) {
    if (lane == 0) red[wave] = best;
    const bool any = __syncthreads_or(listed);
    if (tid == 0) {
      best = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
      a.band[b] = best == 0.f && any ? -0.f : best;
      a.cnt[b] = 0;
    }
  } else if (lane == 0 && blockIdx.x * 4 + wave < a.n_parts) {
    a.parts[(long long)b * kPoolParts + blockIdx.x * 4 + wave] = best;
  }
}

__global__ __launch_bounds__(256) void pool_cand_kernel(WidePoolArgs a) {
  __shared__ uint32_t theta_w[2][4];
  __shared__ int tie_w[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y;
  uint32_t part_o[kPoolParts / 256], ob = 0u;
#pragma unroll
  for (int i = 0; i < kPoolParts / 256; ++i) {
    const int p = i * 256 + tid;
    part_o[i] = p < a.n_parts ? orderable(a.parts[(long long)b * kPoolParts + p]) : 0u;
    ob = part_o[i] > ob ? part_o[i] : ob;
  }
  const float band = a.band[b];
  const uint32_t theta = kth_best_bound<4>(ob, a.k, theta_w);
  const uint32_t lim = theta ? orderable(unorderable(theta) - 2.f * band) : 0u;
  const int d0 = blockIdx.x * 4 * a.part_docs, d1 = d0 + 4 * a.part_docs < a.N ? d0 + 4 * a.part_docs : a.N;
  // A question without a score that is a number selects the first k documents if one of its tokens does, else nothing.
  const bool nothing = theta <= orderable(-INFINITY) && !__syncthreads_or(ob > orderable(-INFINITY));  // (theta: block-uniform)
  const bool first_docs = band > 0.f || __float_as_int(band) < 0;  // -0
  int ties = 0;  // documents so far that tie with the limit or are above it, at least
  if (band == 0.f && !nothing) {  // block-uniform: one in every earlier part that reaches the limit
    int n = 0;
#pragma unroll
    for (int i = 0; i < kPoolParts / 256; ++i)
      n += __popcll(__ballot(i * 256 + tid < 4 * (int)blockIdx.x && part_o[i] >= lim));
    if (lane == 0) tie_w[wave] = n;
    __syncthreads();
    ties = tie_w[0] + tie_w[1] + tie_w[2] + tie_w[3];
  }
  for (int i0 = d0; i0 < d1; i0 += 256) {  // block-uniform
    const int d = i0 + tid;
    const float x = d < d1 ? pooled_of(a, b, d) : -INFINITY;
    const uint32_t o = orderable(x);
    bool take = d < d1 && (nothing ? first_docs && d < a.k : o >= lim);
    if (band == 0.f && !nothing) {  // block-uniform: the scores are exact; documents that tie with the limit in their order
      const bool tie = d < d1 && o == lim;
      const unsigned long long m = __ballot(tie);
      __syncthreads();
      if (lane == 0) tie_w[wave] = __popcll(m);
      __syncthreads();
      int before = ties + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        before += w < wave ? tie_w[w] : 0;
        ties += tie_w[w];
      }
      take = take && !(tie && before >= a.k);
    }
    if (take) {
      const int slot = atomicAdd(&a.cnt[b], 1);
      a.cand[(long long)b * a.N + slot] = d;
      a.keys[(long long)b * a.N + slot] = band == 0.f ? make_key(nothing ? not_a_number() : x, (uint32_t)d) : 0ull;
    }
  }
}

// A workgroup takes kPoolTok tokens and four candidates, one per wave: the folded queries of the tokens lie in LDS, the keys of a
// candidate, already fp32, in registers (lane: 16 dims of a chunk's key of every group).  A candidate passes over the blocks of
// tokens whose best matrix score is too far below its best to hold its exact best.  Bound by latency and the reads of the
// queries: with eight tokens of one candidate per wave and the queries from memory it took 37 us of the call of 150 tokens above
// and 82 of 1000 tokens over 2000 documents, now 18 and 30.
template <int HKV>
__global__ __launch_bounds__(256) void pool_score_kernel(WidePoolArgs a) {
  constexpr int D = 128, C = 8;
  __shared__ float4 qs[kPoolTok][HKV][D / 4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y;
  const float band = a.band[b];
  if (band == 0.f) return;  // block-uniform: the keys are there
  const int nc = a.cnt[b], quads = (nc + 3) / 4, chunks = (a.M + kPoolTok - 1) / kPoolTok;
  const int part = lane & 7, ch = lane >> 3;
  const int block_rows = a.block_tokens;
  for (long long it = blockIdx.x; it < (long long)quads * chunks; it += gridDim.x) {  // block-uniform
    const int quad = (int)(it / chunks), m0 = (int)(it % chunks) * kPoolTok;
    const int blk = m0 / block_rows;  // (kPoolTok divides a block)
    int doc = 0;
    unsigned need = 0u;  // the candidates that these tokens matter to (the same in every wave)
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int ci = 4 * quad + w;
      const int d = a.cand[(long long)b * a.N + (ci < nc ? ci : nc - 1)];
      doc = w == wave ? d : doc;
      const float here = a.mat[((long long)b * a.m_blocks + blk) * a.N + d];
      if (ci < nc && (a.m_blocks == 1 || here >= pooled_of(a, b, d) - 2.f * band)) need |= 1u << w;
    }
    need = __builtin_amdgcn_readfirstlane(need);
    if (need == 0u) continue;
    const int nt = a.M - m0 < kPoolTok ? a.M - m0 : kPoolTok;
    __syncthreads();  // the queries of the item before are done with
    {
      const float4* src = reinterpret_cast<const float4*>(a.qf + ((long long)b * a.M + m0) * (HKV * D));
      float4* dst = &qs[0][0][0];
      for (int i = tid; i < nt * (HKV * D / 4); i += 256) dst[i] = src[i];
    }
    float kf[HKV][16], inv[HKV];
    if ((need >> wave) & 1u) {
      const long long key = (long long)doc * C + ch;
      const uint16_t* kp = a.KR + (key >> 4) * (16 * D) + (part * (D / 64) * 16 + (int)(key & 15)) * 8;
#pragma unroll
      for (int g = 0; g < HKV; ++g) {
        const uint16_t* p = kp + (long long)g * a.tiles * (16 * D);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const uint4 w = *reinterpret_cast<const uint4*>(p + 128 * x);
          const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            kf[g][8 * x + 2 * i] = bf16_lo(v[i]);
            kf[g][8 * x + 2 * i + 1] = bf16_hi(v[i]);
          }
        }
        inv[g] = a.inv_norm[(long long)g * a.tiles * 16 + key];
      }
    }
    __syncthreads();
    if (((need >> wave) & 1u) == 0u) continue;  // wave-uniform; the next item's barriers come for every wave
    float best = not_a_number();  // (dropped by the first score that is one)
    for (int t = 0; t < nt; ++t) {  // block-uniform
      float tot = 0.f;
#pragma unroll
      for (int g = 0; g < HKV; ++g) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 q = qs[t][g][part * 4 + i];
          acc = fmaf(q.x, kf[g][4 * i], acc);
          acc = fmaf(q.y, kf[g][4 * i + 1], acc);
          acc = fmaf(q.z, kf[g][4 * i + 2], acc);
          acc = fmaf(q.w, kf[g][4 * i + 3], acc);
        }
        acc += dpp_f<kDppXor1>(acc);
        acc += dpp_f<kDppXor2>(acc);
        acc += dpp_f<kDppHalfMirror>(acc);  // the key's dot product, in its eight lanes
        tot += acc * inv[g];
      }
      best = fmaxf(best, tot * (1.0f / (float)HKV));
    }
#pragma unroll
    for (int off = 8; off < 8 * C; off <<= 1) best = fmaxf(best, __shfl_xor(best, off, 64));  // document max over its chunks
    if (best != best) best = not_a_number();
    if (lane == 0) atomicMax(&a.keys[(long long)b * a.N + 4 * quad + wave], make_key(best, (uint32_t)doc));
  }
}

constexpr int kPoolBest = 2048;  // candidates that LDS holds

__global__ __launch_bounds__(512) void pool_best_kernel(WidePoolArgs a) {
  __shared__ unsigned long long surv[kPoolBest];
  __shared__ unsigned long long red[8];
  __shared__ uint32_t theta_w[2][8];
  __shared__ int n_surv;
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const unsigned long long* keys = a.keys + (long long)b * a.N;
  const int nc = a.cnt[b];
  if (tid == 0) n_surv = 0;
  uint32_t ob = 0u;
  for (int i = tid; i < nc; i += 512) {
    const uint32_t o = (uint32_t)(keys[i] >> 32);
    ob = o > ob ? o : ob;
  }
  const uint32_t theta = kth_best_bound<8>(ob, a.k, theta_w);  // (a barrier inside)
  for (int i = tid; i < nc; i += 512) {
    const unsigned long long x = keys[i];
    if ((uint32_t)(x >> 32) >= theta) {
      const int slot = atomicAdd(&n_surv, 1);
      if (slot < kPoolBest) surv[slot] = x;
    }
  }
  __syncthreads();
  const int ns = n_surv;
  auto emit = [&](int rank, unsigned long long x) {
    const long long o = (long long)b * a.k + rank;
    a.out_idx[o] = x ? (int32_t)key_doc(x) : -1;
    if (a.out_score != nullptr) a.out_score[o] = x ? key_score(x) : -INFINITY;
  };
  if (ns <= kPoolBest) {
    for (int i = tid; i < ns; i += 512) {
      const unsigned long long x = surv[i];
      int rank = 0;
      for (int j = 0; j < ns; j += 8) {  // eight at a time, past the end whatever is there
        unsigned long long y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = surv[j + u < kPoolBest ? j + u : 0];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (j + u < ns && y[u] > x) ? 1 : 0;
      }
      if (rank < a.k) emit(rank, x);
    }
    for (int i = ns + tid; i < a.k; i += 512) emit(i, 0ull);
    return;
  }
  // more (copies of the best documents): k rounds of the largest key below the one before
  unsigned long long prev = ~0ull;
  for (int round = 0; round < a.k; ++round) {
    unsigned long long best = 0ull;
    for (int i = tid; i < nc; i += 512) {
      const unsigned long long x = keys[i];
      if (x < prev && x > best) best = x;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long y = __shfl_xor(best, off, 64);
      best = y > best ? y : best;
    }
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = best;
    __syncthreads();
    best = red[0];
#pragma unroll
    for (int w = 1; w < 8; ++w) best = red[w] > best ? red[w] : best;
    if (tid == 0) emit(round, best);
    prev = best;
  }
}

#define MSA_WIDE_ROWS(NN, PP) \
  do { \
    if (stream_index_of(dm, PP)) hipLaunchKernelGGL((score_wide_rows_kernel<NN, PP, true>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((score_wide_rows_kernel<NN, PP, false>), grid, block, 0, st, a); \
  } while (0)

// ---- host side -----------------------------------------------------------------------------------------------------
// More tokens than one pass of the all-heads scan takes.
bool wide_path_applies(const Dims& dm, int BM) { return dm.scope_all && dm.Hkv > 1 && BM > 32; }

WidePlan plan_score_wide(const Dims& dm, int BM, int k) {
  WidePlan p;
  p.pair = (dm.cos && dm.d == 128 && dm.C == 8) ? 0 : 1;
  const int n_pass = (BM + kWidePass - 1) / kWidePass;
  p.pass_tokens = (BM + n_pass - 1) / n_pass;
  const int per_wg = kWideRows / (p.pair ? 2 : 1);
  p.n_tb = (p.pass_tokens + per_wg - 1) / per_wg;
  // segments of whole units (64 documents are whole units for every C), all alike
  long long seg = (long long)(kWideMat / sizeof(float)) / p.pass_tokens;
  if (seg < 64) seg = 64;
  const long long n_seg = (dm.N + seg - 1) / seg;
  seg = ((dm.N + n_seg - 1) / n_seg + 63) / 64 * 64;
  p.seg_docs = (int)(seg < dm.N ? seg : dm.N);
  size_t end = 0;
  p.off_qf = end;
  end += round_up256((size_t)p.pass_tokens * dm.Hkv * dm.d * sizeof(float));
  p.off_qop = end;
  end += round_up256((size_t)dm.Hkv * p.n_tb * (kWideRows / 16) * (dm.d / 32) * 64 * 16);
  p.off_eps = end;
  end += round_up256((size_t)p.pass_tokens * dm.Hkv * sizeof(float));
  p.off_best = end;
  end += round_up256((size_t)BM * k * sizeof(unsigned long long));  // (each pass has its own tokens')
  p.off_mat = end;
  end += round_up256((size_t)p.pass_tokens * p.seg_docs * sizeof(float));
  p.ws_bytes = end;
  p.list_bytes = !p.pair && p.seg_docs < dm.N
                     ? round_up256((size_t)p.pass_tokens * kWideList * 8) + round_up256((size_t)p.pass_tokens * sizeof(uint2))
                     : 0;
  p.off_list = 0;
  return p;
}

WidePoolPlan plan_score_wide_pool(const Dims& dm, const WidePlan& pl, int B, int M, int k) {
  WidePoolPlan p = {};
  if (!dm.token_pool || pl.pair || M <= 32 || M > kPoolMost || B * M > kWidePass) return p;
  p.m_blocks = (M + 16 * kRowsMost - 1) / (16 * kRowsMost);
  // Every block reads the index: not where the blocks of the batch rows are more than those of 64 of all tokens (3 questions of
  // 40 tokens over 60000 documents 277 -> 348 us).
  if (B * p.m_blocks > (B * M + kWideRows - 1) / kWideRows) return p;
  p.nt = ((M + p.m_blocks - 1) / p.m_blocks + 31) / 32 * 2;
  // Next to no documents: the launches are what counts, and the most rows in a workgroup the longest (k = 9, selection per token ->
  // here: 5 documents, 60 tokens 31.1 -> 32.8 us, 10 36.8 -> 34.0; 148 tokens, one block of ten tiles, 26 38.1 -> 43.4, 64 42.8 -> 43.0;
  // 300, two blocks, 10 44.9 -> 44.0).
  if (dm.tiles < (p.m_blocks == 1 && p.nt > 6 ? 32 : 5)) return p;
  // ... and for few winners, whose selection per token is short, that longest workgroup counts up to 2000 documents (148 tokens, index
  // again and again: k = 2, 500 documents 38.8 -> 41.4 us, 2000 39.6 -> 42.8, cold the same; k = 9 44.2 -> 45.2, 45.4 -> 44.8; k = 32
  // over 300 60 -> 50).
  if (p.m_blocks == 1 && p.nt > 8 && k < 16 && dm.tiles < 1000) return p;
  p.m_tiles = (M + 15) / 16;
  p.part_docs = (dm.N + kPoolParts - 1) / kPoolParts;
  p.n_parts = (dm.N + p.part_docs - 1) / p.part_docs;
  size_t end = 0;
  auto take = [&](size_t bytes) {
    const size_t at = end;
    end += round_up256(bytes);
    return at;
  };
  p.off_qf = take((size_t)B * M * dm.Hkv * dm.d * sizeof(float));
  p.off_qop = take((size_t)dm.Hkv * B * p.m_tiles * (dm.d / 32) * 64 * 16);
  p.off_eps = take((size_t)B * M * dm.Hkv * sizeof(float));
  p.off_mat = take((size_t)B * p.m_blocks * dm.N * sizeof(float));
  p.off_parts = take((size_t)B * kPoolParts * sizeof(float));
  p.off_band = take((size_t)B * sizeof(float));
  p.off_cnt = take((size_t)B * sizeof(int));
  p.off_cand = take((size_t)B * dm.N * sizeof(int));
  p.off_keys = take((size_t)B * dm.N * sizeof(unsigned long long));
  p.applies = end <= pl.ws_bytes ? 1 : 0;  // (the bytes that a call has always been asked for)
  return p;
}

int launch_score_wide_pool(const Dims& dm, const WidePoolPlan& pp, const void* q_route, int B, int M, const void* KR,
                           const float* inv_norm, int k, void* ws, hipStream_t st, int32_t* out_idx, float* out_score) {
  char* const w = (char*)ws;
  const int n_rt = B * pp.m_tiles;
  const int rc = launch_fold_queries(dm, q_route, B * M, (float*)(w + pp.off_qf), (float*)(w + pp.off_eps), nullptr, 0,
                                     (uint4*)(w + pp.off_qop), n_rt, 0, M, 16 * pp.m_tiles, st);
  if (rc != MSA_OK) return rc;
  WideArgs a = {};
  a.qop = (const uint4*)(w + pp.off_qop);
  a.KR = (const uint16_t*)KR;
  a.inv_norm = inv_norm;
  a.mat = (float*)(w + pp.off_mat);
  a.mat_stride = dm.N;
  a.n_rt = n_rt;
  a.n_tb = B * pp.m_blocks;
  a.nq = B * M;
  a.C = dm.C;
  a.tiles = dm.tiles;
  a.seg_tiles = (int)dm.tiles;
  a.seg_docs = dm.N;
  a.Hkv = dm.Hkv;
  a.M = M;
  a.m_tiles = pp.m_tiles;
  a.m_blocks = pp.m_blocks;
  const int units = (a.seg_tiles + kRowsTiles - 1) / kRowsTiles, most = (units + kRowsWaves - 1) / kRowsWaves;
  a.n_streams = kWideGroups / a.n_tb;
  if (a.n_streams < 1) a.n_streams = 1;
  if (a.n_streams > most) a.n_streams = most;
  const dim3 grid((unsigned)((a.n_tb * a.n_streams + 7) / 8 * 8)), block(64 * kRowsWaves);
  profile_mark(dm, false, st);
  if (pp.nt <= 4) MSA_WIDE_ROWS(4, true);
  else if (pp.nt == 6) MSA_WIDE_ROWS(6, true);
  else if (pp.nt == 8) MSA_WIDE_ROWS(8, true);
  else MSA_WIDE_ROWS(10, true);
  profile_mark(dm, true, st);
  if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
  WidePoolArgs p;
  p.mat = a.mat;
  p.eps = (const float*)(w + pp.off_eps);
  p.qf = (const float*)(w + pp.off_qf);
  p.KR = a.KR;
  p.inv_norm = inv_norm;
  p.parts = (float*)(w + pp.off_parts);
  p.band = (float*)(w + pp.off_band);
  p.cnt = (int*)(w + pp.off_cnt);
  p.cand = (int*)(w + pp.off_cand);
  p.keys = (unsigned long long*)(w + pp.off_keys);
  p.out_idx = out_idx;
  p.out_score = out_score;
  p.N = dm.N;
  p.M = M;
  p.Hkv = dm.Hkv;
  p.k = k;
  p.m_blocks = pp.m_blocks;
  p.block_tokens = 16 * pp.nt;
  p.part_docs = pp.part_docs;
  p.n_parts = pp.n_parts;
  p.tiles = dm.tiles;
  const unsigned quads = (unsigned)((pp.n_parts + 3) / 4);
  hipLaunchKernelGGL(pool_parts_kernel, dim3(quads + 1, (unsigned)B), dim3(256), 0, st, p);
  hipLaunchKernelGGL(pool_cand_kernel, dim3(quads, (unsigned)B), dim3(256), 0, st, p);
  const dim3 sgrid(512, (unsigned)B);  // (150 tokens, about 100 candidates: 25 quads and 38 chunks of tokens, two items each)
  if (dm.Hkv == 2) hipLaunchKernelGGL(pool_score_kernel<2>, sgrid, dim3(256), 0, st, p);
  else if (dm.Hkv == 4) hipLaunchKernelGGL(pool_score_kernel<4>, sgrid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL(pool_score_kernel<8>, sgrid, dim3(256), 0, st, p);
  hipLaunchKernelGGL(pool_best_kernel, dim3((unsigned)B), dim3(512), 0, st, p);
  return hipGetLastError() == hipSuccess ? MSA_OK : MSA_ERR_HIP;
}

// More rows per key for 65 to 160 tokens of eight groups, whose blocks of 64 rows are two or three times the reads of a key, the
// third half empty (150 tokens, 97656 documents 496 -> 430 us; 80 401 -> 354; 70 over 300 41 -> 38).  Up to 192 three blocks are full
// (190 over 20000 124 -> 124, on another card 127 -> 136).  More tokens are bound by the products, and these by the operand reads
// (600 tokens, 30000 documents 483 -> 494, 2048 over 32768 1477 -> 1714); with four groups the resident operands leave room for
// two workgroups per CU (100 tokens, 60000 documents 157 -> 160).
// A wave's unit here is half as many keys with all rows, so the line follows the rounds of units that both take over a segment
// (index cold / again and again, blocks of 64 rows -> here):
//   six tiles of rows: as fast in a round at any size (8300 documents 76 / 64 -> 71 / 63, 10500 79 / 69 -> 74 / 69, 21500 111 / 106 -> 101);
//   eight: faster in one round (2000 50 / 42 -> 46 / 42, 8100 56 / 50 -> 55 / 51), then slower (8300 77 / 65 -> 78 / 69, 13000 82 / 73
//   -> 82 / 76) until the index is too large for the cache (19000 107 / 101 -> 105 / 103, 21500 111 / 107 -> 107 / 105);
//   next to no documents: slower (96 tokens, 26 documents 31.6 -> 33.1, 64 36.1 -> 33.2; 128 31.8 -> 36.3, 36.2 -> 36.5);
//   ten: faster with a round less (5600 68 / 58 -> 53 / 49, 11300 95 / 78 -> 82 / 77, 16800 115 / 105 -> 110 / 108), else not (300
//   documents 42 -> 45, 5300 52 / 47 -> 52 / 48, 8300 75 / 66 -> 83 / 75).
static bool rows_kernel_pays(int nq, int seg_tiles) {
  if (nq <= kWideRows || nq > 16 * kRowsMost || seg_tiles < 32) return false;
  const int blocks = (nq + kWideRows - 1) / kWideRows, waves = kWideGroups / blocks * kWideWaves;
  const int rounds = ((seg_tiles + kWideTiles - 1) / kWideTiles + waves - 1) / waves;
  const int rows_waves = kWideGroups * kRowsWaves;
  const int rows_rounds = ((seg_tiles + kRowsTiles - 1) / kRowsTiles + rows_waves - 1) / rows_waves;
  if (nq <= 96) return true;
  if (nq <= 128) return rows_rounds == 1 || seg_tiles >= 10000;
  return rows_rounds < rounds;
}

int launch_score_wide(const Dims& dm, const WidePlan& pl, const void* q_route, int BM, const void* KR,
                      const float* inv_norm, int k, void* ws, hipStream_t st, int32_t* out_idx, float* out_score,
                      unsigned long long* out_key) {
  char* const w = (char*)ws;
  WideArgs a;
  a.qop = (const uint4*)(w + pl.off_qop);
  a.KR = (const uint16_t*)KR;
  a.inv_norm = dm.cos ? inv_norm : nullptr;
  a.mat = (float*)(w + pl.off_mat);
  a.mat_stride = pl.seg_docs;
  a.C = dm.C;
  a.tiles = dm.tiles;
  WideSelArgs s;
  s.mat = a.mat;
  s.mat_stride = pl.seg_docs;
  s.eps = pl.pair ? nullptr : (const float*)(w + pl.off_eps);
  s.qf = (const float*)(w + pl.off_qf);
  s.KR = a.KR;
  s.inv_norm = a.inv_norm;
  s.out_idx = out_idx;
  s.out_score = out_score;
  s.out_key = out_key;
  s.Hkv = dm.Hkv;
  s.k = k;
  s.tiles = dm.tiles;
  s.list = pl.off_list != 0 ? (unsigned long long*)(w + pl.off_list) : nullptr;
  s.list_n = pl.off_list != 0 ? (uint2*)(w + pl.off_list + round_up256((size_t)pl.pass_tokens * kWideList * 8)) : nullptr;
  const int per_wg = kWideRows / (pl.pair ? 2 : 1);
  for (int tok0 = 0; tok0 < BM; tok0 += pl.pass_tokens) {
    const int nq = BM - tok0 < pl.pass_tokens ? BM - tok0 : pl.pass_tokens;
    a.nq = nq;
    a.n_rt = pl.n_tb * (kWideRows / 16);
    a.Hkv = dm.Hkv;
    a.M = nq;
    a.m_tiles = a.n_rt;
    const int rc = launch_fold_queries(dm, (const uint16_t*)q_route + (size_t)tok0 * dm.Hq * dm.d, nq,
                                       (float*)(w + pl.off_qf), pl.pair ? nullptr : (float*)(w + pl.off_eps), nullptr, 0,
                                       (uint4*)(w + pl.off_qop), a.n_rt, pl.pair, nq, nq, st);
    if (rc != MSA_OK) return rc;
    for (int doc0 = 0; doc0 < dm.N; doc0 += pl.seg_docs) {
      const int n_docs = dm.N - doc0 < pl.seg_docs ? dm.N - doc0 : pl.seg_docs;
      a.tile0 = (long long)doc0 * dm.C / 16;  // doc0 is a multiple of 64 (or 0)
      a.seg_docs = n_docs;
      a.seg_tiles = (int)(((long long)n_docs * dm.C + 15) / 16);
      const bool rows = !pl.pair && dm.Hkv == 8 && rows_kernel_pays(nq, a.seg_tiles);
      const int units = (a.seg_tiles + (rows ? kRowsTiles : kWideTiles) - 1) / (rows ? kRowsTiles : kWideTiles);
      const int waves = rows ? kRowsWaves : kWideWaves;
      int nt = kWideRows / 16;
      if (rows) nt = (nq + 31) / 32 * 2;
      a.n_tb = rows ? (nq + 16 * nt - 1) / (16 * nt) : (nq + per_wg - 1) / per_wg;
      int streams = kWideGroups / a.n_tb;
      if (streams < 1) streams = 1;
      const int most = (units + waves - 1) / waves;
      if (streams > most) streams = most;
      a.n_streams = streams;
      a.m_blocks = a.n_tb;
      // Streaming loads where one token block reads the keys and the cache behind the L2s keeps none of them: 40 tokens, 97656
      // documents 357 -> 321 us, 64 over 20000 106 -> 101 (102.4 -> 98.1 again and again).  A smaller index gains nothing when it
      // is cold and loses when it is not (50 over 8000 56.8, 57.9; again and again 49.6, 56.2).
      const bool stream = a.n_tb == 1 && stream_index_of(dm, false);
      dim3 grid((unsigned)((a.n_tb * streams + 7) / 8 * 8)), block(64 * waves);
      if (tok0 == 0 && doc0 == 0) profile_mark(dm, false, st);
#define MSA_WIDE(DD, HH) \
  do { \
    if (!pl.pair && stream) hipLaunchKernelGGL((score_wide_kernel<128, HH, false, true, true>), grid, block, 0, st, a); \
    else if (!pl.pair) hipLaunchKernelGGL((score_wide_kernel<128, HH, false, true, false>), grid, block, 0, st, a); \
    else if (dm.cos) hipLaunchKernelGGL((score_wide_kernel<DD, HH, true, true, false>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((score_wide_kernel<DD, HH, true, false, false>), grid, block, 0, st, a); \
  } while (0)
      if (rows) {
        if (nt == 6) MSA_WIDE_ROWS(6, false);
        else if (nt == 8) MSA_WIDE_ROWS(8, false);
        else MSA_WIDE_ROWS(10, false);
      } else if (dm.d == 128) {
        if (dm.Hkv == 2) MSA_WIDE(128, 2); else if (dm.Hkv == 4) MSA_WIDE(128, 4); else MSA_WIDE(128, 8);
      } else {
        if (dm.Hkv == 2) MSA_WIDE(64, 2); else if (dm.Hkv == 4) MSA_WIDE(64, 4); else MSA_WIDE(64, 8);
      }
#undef MSA_WIDE
      if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
      if (tok0 + nq == BM && doc0 + n_docs == dm.N) profile_mark(dm, true, st);
      s.best = (unsigned long long*)(w + pl.off_best) + (size_t)tok0 * k;
      s.first = doc0 == 0;
      s.last = doc0 + n_docs == dm.N;
      s.n_docs = n_docs;
      s.doc0 = doc0;
      s.tok0 = tok0;
#define MSA_WIDE_SELECT(BB) \
  do { \
    if (n_docs <= 16 * kWideSel) \
      hipLaunchKernelGGL((score_wide_select_kernel<BB, 16>), dim3((unsigned)nq), dim3(kWideSel), 0, st, s); \
    else \
      hipLaunchKernelGGL((score_wide_select_kernel<BB, kWideRegs>), dim3((unsigned)nq), dim3(kWideSel), 0, st, s); \
  } while (0)
      if (pl.pair) MSA_WIDE_SELECT(false); else MSA_WIDE_SELECT(true);
#undef MSA_WIDE_SELECT
      if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
    }
  }
  return MSA_OK;
}

}  // namespace msa
