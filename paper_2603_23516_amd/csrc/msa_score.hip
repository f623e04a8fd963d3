// msa_score_topk: relevance scores (paper, Eq. 2), document max and top-k (Section 3.2.1), fused so
// that chunk scores never leave the chip.  The routing index is streamed from HBM exactly once per
// group of up to 16 queries; this is the O(M L / P) term that dominates online cost (Section 5.1).
//
// Algebra.  With cosine similarity the head mean of Eq. 2 for KV group g is
//     (1/r) sum_h  q_h . key / (|q_h| |key|)  =  ( (1/r) sum_h q_h/|q_h| ) . key * (1/|key|),
// so the r heads of a group fold into ONE fp32 routing query per (token, group) and the scan is a
// thin GEMM  [queries x d] * [d x keys]  followed by a multiply with the stored 1/|key|.
//
// Mapping.  One 16x16x32 bf16 MFMA tile = 16 query rows x 16 keys.  The folded query is carried as
// a bf16 (hi, lo) pair in two adjacent rows (row 2i = hi, row 2i+1 = lo), so one MFMA tile serves 8
// queries at ~16 significant bits and the two halves of a score land in the same lane.  The index is
// stored in tiles of 16 keys already in B-operand order, so a wave reads a tile with d/32 coalesced
// 1 KiB loads and no LDS staging.
//
// Work split.  One wavefront = one stream of tiles of one KV head (wave s of S takes tiles s, s + S, ...),
// with a ring of kPrefetch tiles in flight; a workgroup holds four such streams that never synchronise.  Document max = DPP
// max over the C lanes of a document.  Top-k = threshold filter + per-(wave, query) candidate list in
// LDS: accepted lanes get their slots from a ballot and a population count (no atomics, counters live
// in registers), lists are pruned to the k best by rank counting on 64-bit (score, ~doc) keys, and
// the sorted per-wave lists are combined by a second, small kernel.
#include "msa_device.h"
#include "msa_host.h"

#include <type_traits>

namespace msa {

constexpr int kPrefetch = 4;         // tiles in flight per wave
constexpr int kListBytes = 16384;    // LDS per wave for candidate lists

struct ScoreArgs {
  const uint4* qop;         // [Hkv][n_qtiles][D/32][64] A operands (bf16 hi/lo rows) of 8-query tiles, prepared by
                            // prep_scan_operands_kernel (all-heads scan; per-group scan with the threshold exchange)
  int n_qtiles;
  const uint16_t* q_route;  // [BM][Hq][D] routing queries: a per-group scan without the exchange folds them itself
  const uint16_t* KR;       // tiled
  const float* inv_norm;    // may be null (dot)
  unsigned long long* ws;   // [Hkv][BM][n_splits][k] candidate keys, each list sorted descending
  int BM, q0;               // total queries, first query of this pass
  int Hq, Hkv, r;
  int N, C, cos;
  long long tiles;
  int n_splits, k;
  float* mat;               // MODE 2: document scores [Hkv][BM][N]
  int tiles_per_wave;       // MODE 2: contiguous tiles per wave
  float* gmax;              // [Hkv][BM][n_splits] running per-wave maxima (threshold exchange), or null
  int it_publish, it_adopt; // iterations at which a wave publishes its maxima / adopts the bound
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ float group_max_rt(float x, int C) {
  if (C >= 2) x = fmaxf(x, dpp_f<kDppXor1>(x));
  if (C >= 4) x = fmaxf(x, dpp_f<kDppXor2>(x));
  if (C >= 8) x = fmaxf(x, dpp_f<kDppHalfMirror>(x));
  if (C >= 16) x = fmaxf(x, dpp_f<kDppMirror>(x));
  return x;
}

// Keep the k largest of the c (<= CAP) distinct keys of one list, sorted descending, by rank
// counting.  Executed by one whole wave.  Returns the new count min(c, k).  UNR candidates are read
// (LDS broadcasts) per round: the final sort of a stream keeps 16 reads in flight (their latency is
// what it waits for: 15.5 -> 9.7 us per wave on the 50M-token bank), the in-stream prunes 4 to keep the
// loop body small.
template <int CAP, int UNR = 4>
__device__ __forceinline__ int prune_list(unsigned long long* cl, int c, int k, int lane) {
  constexpr int PER = CAP / 64;
  unsigned long long key[PER];
  int rank[PER];
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    key[p] = (lane + 64 * p < c) ? cl[lane + 64 * p] : 0ull;
    rank[p] = 0;
  }
  int j = 0;
  for (; j + UNR <= c; j += UNR) {
    unsigned long long x[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) x[u] = cl[j + u];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      if (64 * p < c) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) rank[p] += (x[u] > key[p]) ? 1 : 0;
      }
    }
  }
  for (; j < c; ++j) {
    const unsigned long long x = cl[j];
#pragma unroll
    for (int p = 0; p < PER; ++p) rank[p] += (x > key[p]) ? 1 : 0;
  }
  wave_sync();
#pragma unroll
  for (int p = 0; p < PER; ++p)
    if (lane + 64 * p < c && rank[p] < k) cl[rank[p]] = key[p];
  wave_sync();
  return c < k ? c : k;
}

// Sum over aligned groups of W consecutive lanes (W a power of two <= 64); every lane gets the sum.
template <int W>
__device__ __forceinline__ float group_sum(float x) {
  if (W >= 2) x += dpp_f<kDppXor1>(x);
  if (W >= 4) x += dpp_f<kDppXor2>(x);
  if (W >= 8) x += dpp_f<kDppHalfMirror>(x);
  if (W >= 16) x += dpp_f<kDppMirror>(x);
  if (W >= 32) x += __shfl_xor(x, 16, 64);
  if (W >= 64) x += __shfl_xor(x, 32, 64);
  return x;
}

// Independent streams (waves) per workgroup: measured 3-5 % faster than single-wave workgroups.
constexpr int kScanWaves = 4;

// One wave folds the r heads of KV group g of the 8 queries of tile qt into one fp32 routing query per token,
//     qf = (1/r) sum_h q_h / max(|q_h|, 1e-12)        (plain mean for the dot product),
// splits it into bf16 hi + lo and leaves the MFMA A operands of the tile in aop[s][lane]: lane 16q + n holds row n
// (query n/2, hi for even n, lo for odd n), dims 32s + 8q .. +8 of slice s.  qf: 8 * D floats of the wave's own LDS.
// Two steps, so that a caller can put other loads between the request for the queries and their use:
// fold_query_load asks for the queries, fold_query_tile folds them.
// Lane = (query lane / LPH, 16-byte piece lane % LPH): a lane loads the same piece of all r heads of
// its query, so the head sum stays in the lane and the norms need only DPP sums over LPH <= 16 lanes.
template <int D>
struct FoldRegs {
  static constexpr int LPH = D / 8, HPL = 64 / LPH, PASSES = 8 / HPL;
  uint4 v[PASSES][8];
};

template <int D>
__device__ __forceinline__ void fold_query_load(const uint16_t* __restrict__ q_route, long long qt, int g, int BM,
                                                int Hq, int r, FoldRegs<D>& fr, int lane) {
  constexpr int LPH = FoldRegs<D>::LPH, HPL = FoldRegs<D>::HPL;
  const int piece = lane % LPH;
  // No branch around a load (rows past the end re-read the last query, heads past r the last head; the fold
  // ignores both): the loads then sit in straight-line code and the wait before the fold can leave the loads
  // that were issued after them in flight.
#pragma unroll
  for (int pass = 0; pass < FoldRegs<D>::PASSES; ++pass) {
    long long qg = qt * 8 + pass * HPL + lane / LPH;
    if (qg > BM - 1) qg = BM - 1;
#pragma unroll
    for (int hh = 0; hh < 8; ++hh) {
      const int hc = hh < r ? hh : r - 1;
      fr.v[pass][hh] = *reinterpret_cast<const uint4*>(q_route + (qg * Hq + g * r + hc) * D + piece * 8);
    }
  }
}

template <int D>
__device__ __forceinline__ void fold_query_tile(const FoldRegs<D>& fr, long long qt, int BM, int r, int cos, float* qf,
                                                uint4 (*aop)[64], int lane) {
  constexpr int NS = D / 32, LPH = FoldRegs<D>::LPH, HPL = FoldRegs<D>::HPL;
  const int piece = lane % LPH;
#pragma unroll
  for (int pass = 0; pass < FoldRegs<D>::PASSES; ++pass) {
    const int qi = pass * HPL + lane / LPH;
    if (qt * 8 + pass * HPL >= BM) {  // wave-uniform: none of these queries exists
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[qi * D + piece * 8 + e] = 0.f;
      continue;
    }
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = 0.f;
#pragma unroll
    for (int hh = 0; hh < 8; ++hh) {
      if (hh < r) {  // wave-uniform
        const uint4 v = fr.v[pass][hh];
        const float x[8] = {bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y),
                            bf16_lo(v.z), bf16_hi(v.z), bf16_lo(v.w), bf16_hi(v.w)};
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += x[e] * x[e];
        ss = group_sum<LPH>(ss);
        const float w = cos ? 1.0f / fmaxf(sqrtf(ss), 1e-12f) : 1.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] += x[e] * w;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[qi * D + piece * 8 + e] = (qt * 8 + qi < BM) ? f[e] / (float)r : 0.f;
  }
  wave_sync();
  const int rr = lane >> 4, n = lane & 15;
  uint32_t w[NS][4];  // (all of qf is read before the operands are written: they may lie in the same place)
#pragma unroll
  for (int s = 0; s < NS; ++s) {
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      float h0, l0, h1, l1;
      split_bf16(qf[(n >> 1) * D + 32 * s + 8 * rr + 2 * jj], h0, l0);
      split_bf16(qf[(n >> 1) * D + 32 * s + 8 * rr + 2 * jj + 1], h1, l1);
      w[s][jj] = (n & 1) ? pack_bf16(l0, l1) : pack_bf16(h0, h1);
    }
  }
  wave_sync();
#pragma unroll
  for (int s = 0; s < NS; ++s) aop[s][lane] = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
  wave_sync();
}

// MODE 0  filter: thresholds, candidate lists, pruning (long streams).
// MODE 1  dense lists: a wave's whole stream holds no more documents than a list has slots, so every
//         document score goes straight to slot (iteration, document-in-tile) of its query's list and
//         the lists are sorted once at the end; no thresholds, ballots or counters in the stream.
// MODE 2  score matrix: like MODE 1 but the wave owns a CONTIGUOUS range of tiles and, instead of
//         sorting, writes the fp32 document scores of every query as one coalesced run of the row
//         mat[g][query][:]; topk_rows_kernel then selects per row.  For short streams (small banks,
//         many queries) the per-wave sorts and the list merge cost more than the stream itself.
// FOLD: the workgroup folds its queries into MFMA operands itself (wave t folds tile t, one workgroup barrier) instead
//       of reading operands that prep_scan_operands_kernel prepared: one launch less, which is what short streams
//       are made of.  Scans with the threshold exchange keep the prepared operands: that launch also resets the
//       exchange buffer, and their waves never synchronise.
// STREAM: streaming loads of the index (load_stream16; see stream_index_of).
// LATE: with FOLD, one tile is requested ahead of the folding and the others behind it, else all ahead (see late_requests).
template <int D, int NQT, bool COS, int MODE, bool FOLD, bool STREAM, bool LATE>
__global__ __launch_bounds__(64 * kScanWaves) __attribute__((amdgpu_waves_per_eu(2)))
void score_scan_kernel(ScoreArgs a) {
  constexpr bool DENSE = MODE != 0;
  constexpr int NS = D / 32;   // MFMA k-slices per key
  constexpr int NQ = 8 * NQT;  // queries per pass
  constexpr int CAP = kListBytes / (8 * NQ);
  constexpr int CAPF = kListBytes / (4 * NQ);  // MODE 2: fp32 scores per query
  constexpr int TILE_ELEMS = 16 * D;

  __shared__ __attribute__((aligned(16))) unsigned char smem[kScanWaves][kListBytes];
  __shared__ int cnt_all[kScanWaves][NQ];
  __shared__ float thr_all[kScanWaves][NQ];
  const int wave = threadIdx.x >> 6;
  unsigned long long* cand = reinterpret_cast<unsigned long long*>(smem[wave]);  // [NQ][CAP]
  float* candf = reinterpret_cast<float*>(smem[wave]);                            // MODE 2: [NQ][CAPF]
  int* cnt_s = cnt_all[wave];
  float* thr_s = thr_all[wave];

  const int lane = threadIdx.x & 63;
  const int rr = lane >> 4;  // MFMA k-group / D row-group
  const int n = lane & 15;   // A row / B column / D column
  const int sp = blockIdx.x * kScanWaves + wave;
  const int g = blockIdx.y;
  // wave-uniform; with FOLD a wave without a stream (the tail of the last workgroup) still takes part in the
  // workgroup barriers of the prologue, otherwise the waves of a workgroup never synchronise
  const bool active = sp < a.n_splits;
  if (!FOLD && !active) return;

  // ---- the queries this wave folds are requested first: a wave's loads return in order, and behind the first tiles
  // of every wave of the grid (tens of MB at once) they would arrive only when that burst has been served ----
  FoldRegs<D> fr;
  bf16x8_t A[NQT][NS];
  typedef uint4 aop_tile_t[64];
  if constexpr (FOLD) {
    if (wave < NQT) fold_query_load<D>(a.q_route, a.q0 / 8 + wave, g, a.BM, a.Hq, a.r, fr, lane);
  } else {
    // prepared operands: row n of query tile t is query 8t + n/2, hi (even n) or lo (odd n) half of the folded
    // fp32 routing query
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
      const long long qt = a.q0 / 8 + t;
#pragma unroll
      for (int s = 0; s < NS; ++s)
        A[t][s] = as_bf16x8(a.qop[(((long long)g * a.n_qtiles + qt) * NS + s) * 64 + lane]);
    }
  }

  // ---- start streaming at once: the first kPrefetch tiles are requested in the prologue ----
  // Wave sp takes tiles sp, sp + n_splits, sp + 2 n_splits, ...: at any moment the waves of a head
  // read one contiguous window of the index.  Loads past the end re-read the last tile: they are
  // always issued, so the number of loads in flight is the same on every path.
  const long long S = a.n_splits;
  const long long t0 = (long long)sp * a.tiles_per_wave;  // MODE 2: first tile of this wave
  const long long n_it = !active ? 0
                         : (MODE == 2) ? ((a.tiles - t0 < a.tiles_per_wave) ? a.tiles - t0 : a.tiles_per_wave)
                                       : (a.tiles - sp + S - 1) / S;  // >= 1 by construction of n_splits
  const long long i_last = n_it - 1;
  // MODE 2: the wave walks its range starting rot tiles in and wraps around, so that waves that run in step do
  // not all ask for the same 4 KB position of their 16-tile ranges (the same memory channels) at the same moment
  const long long rot = (MODE == 2 && n_it > 0) ? sp % n_it : 0;
  auto tile_at = [&](long long it) {
    if (MODE != 2) return sp + it * S;
    const long long x = it + rot;
    return t0 + (x >= n_it ? x - n_it : x);
  };
  const uint16_t* KRg = a.KR + (long long)g * a.tiles * TILE_ELEMS + lane * 8;
  const float* ing = COS ? a.inv_norm + (long long)g * a.tiles * 16 + n : nullptr;
  auto load_tile16 = [](const uint16_t* p) {
    return STREAM ? load_stream16(p) : *reinterpret_cast<const uint4*>(p);
  };
  uint4 buf[kPrefetch][NS];
  float binv[kPrefetch];
  auto first_tile = [&](int u) __attribute__((always_inline)) {
    // a wave without a stream loads tile 0 and drops it: no branch around the loads
    const long long t = active ? tile_at((u < n_it) ? u : i_last) : 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) buf[u][s] = load_tile16(KRg + t * TILE_ELEMS + s * 512);
    binv[u] = COS ? ing[t * 16] : 1.0f;
  };
  constexpr int kAheadOfFold = LATE ? 1 : kPrefetch;
#pragma unroll
  for (int u = 0; u < kAheadOfFold; ++u) first_tile(u);
  // Wave t folds tile t.  It asks for one tile ahead of that and for the others behind it: with all of them ahead, the
  // wave is held up until the memory system has taken the first requests of every wave (3 to 6 us where the grid fills the
  // chip), and the operands are ready after the first tiles have come and the memory has had nothing to do in between (one
  // query over 2048 documents, whole call: 15.1 -> 14.3 us); with none, a grid of a few workgroups waits for its tiles.
  if constexpr (FOLD) {
    // the operands pass through the candidate areas, which are free until the stream starts: tile t in the second half of
    // area t, the folding wave's scratch in the first half of its own
    static_assert(NQT <= kScanWaves && 8 * D * 4 <= kListBytes / 2 && NS * 64 * 16 <= kListBytes / 2, "prologue scratch");
    if (wave < NQT)
      fold_query_tile<D>(fr, a.q0 / 8 + wave, a.BM, a.r, COS ? 1 : 0, reinterpret_cast<float*>(smem[wave]),
                         reinterpret_cast<aop_tile_t*>(smem[wave] + kListBytes / 2), lane);
  }
#pragma unroll
  for (int u = kAheadOfFold; u < kPrefetch; ++u) first_tile(u);

  // ---- A operands: row n of query tile t is query 8t + n/2, hi (even n) or lo (odd n) half of the folded fp32
  // routing query ------------------------------------------------------------------------------------------
  if constexpr (FOLD) {
    lds_barrier();
#pragma unroll
    for (int t = 0; t < NQT; ++t)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        A[t][s] = as_bf16x8(reinterpret_cast<const aop_tile_t*>(smem[t] + kListBytes / 2)[s][lane]);
    lds_barrier();  // every wave has its operands: the candidate areas are the streams' from here on
    if (!active) return;
  } else {
    // The operands were requested ahead of the tiles; they are awaited HERE, ahead of the loop.  A wait that is
    // first needed inside the loop sits in the loop's first block and is paid on every round: there it has to
    // cover the entry from here too, where the operands are the youngest loads, so it would wait for everything,
    // i.e. drain the prefetch at the head of every round.
#pragma unroll
    for (int t = 0; t < NQT; ++t)
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(A[t][s]));
  }

  // This lane sees queries 8t + 2rr + e (e = 0, 1) of every tile; all 16 lanes of a row keep
  // identical copies of their counters and thresholds.
  float thr[NQT][2];
  int cnt[NQT][2];
#pragma unroll
  for (int t = 0; t < NQT; ++t)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      thr[t][e] = (a.q0 + 8 * t + 2 * rr + e < a.BM) ? -INFINITY : INFINITY;
      cnt[t][e] = 0;
    }
  int limit = 2 * a.k < 32 ? 32 : 2 * a.k;  // prune a list when it grows past this
  if (limit > CAP - 16) limit = CAP - 16;

  // ---- stream this wave's tiles -----------------------------------------------------------------
  const int dpt = 16 / a.C;  // documents per tile
  const int ndoc = n / a.C;  // this lane's document inside a tile
  const bool lead_lane = (n & (a.C - 1)) == 0;
  const uint32_t below = (1u << n) - 1u;
  float qmax[NQT][2];        // running maximum of this lane's document scores, per query
#pragma unroll
  for (int t = 0; t < NQT; ++t) qmax[t][0] = qmax[t][1] = -INFINITY;
  // One 8-query tile per pass: the published maxima are requested kPrefetch iterations before they
  // are used, all queries at once, so their latency hides behind that many tiles of the stream.
  constexpr bool kEarlyFetch = (NQT == 1);
  constexpr int kFetchLead = 1;  // in groups of kPrefetch iterations
  float exq[kEarlyFetch ? NQ : 1][4];
  {
    for (long long base = 0; base < n_it; base += kPrefetch) {
      // ---- threshold exchange (long streams only): every wave publishes the best score it has
      // seen per query; a little later it adopts theta = the k-th largest of all published maxima.
      // The maxima belong to distinct documents, so at least k documents score >= theta: a valid
      // lower bound on the k-th best score whatever the other waves have written so far.  The maxima
      // are published with device-scope stores and read with device-scope loads: the waves of a head sit on all
      // eight XCDs, each with its own L2, and a plainly stored maximum becomes visible elsewhere only when its
      // line happens to be evicted.  With plain index loads flooding the L2 that happened soon enough; the
      // streaming loads used here leave the L2 alone, and the bound then came from one XCD's maxima only (the
      // k-th largest of 32 instead of 256: scan 272 -> 283 us on the 50M-token index, 256 with these accesses).
      if (!DENSE && kEarlyFetch && a.gmax != nullptr && base == a.it_adopt - kFetchLead * kPrefetch) {
#pragma unroll
        for (int qi = 0; qi < (kEarlyFetch ? NQ : 1); ++qi) {
          const int qg = a.q0 + qi < a.BM ? a.q0 + qi : a.BM - 1;
          const float* src = a.gmax + ((long long)g * a.BM + qg) * a.n_splits;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            exq[qi][j] = (lane + 64 * j < a.n_splits) ? load_dev(src + lane + 64 * j) : -INFINITY;
        }
      }
      if (!DENSE && a.gmax != nullptr && (base == a.it_publish || base == a.it_adopt)) {
        if (base == a.it_publish) {
#pragma unroll
          for (int tq = 0; tq < NQT; ++tq)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float mrow = group_max<16>(qmax[tq][e]);
              const int qg = a.q0 + 8 * tq + 2 * rr + e;
              if (n == 0 && qg < a.BM) store_dev(&a.gmax[((long long)g * a.BM + qg) * a.n_splits + sp], mrow);
            }
        } else {
          // theta = k-th largest of the published maxima of one query: bitwise search on the
          // order-preserving integer image, 4 values per lane
          auto kth_largest = [&](const uint32_t (&ord)[4]) -> float {
            uint32_t prefix = 0u;
            for (int bit = 31; bit >= 12; --bit) {
              const uint32_t cnd = prefix | (1u << bit);
              int ge = 0;
#pragma unroll
              for (int j = 0; j < 4; ++j) ge += __popcll(__ballot(ord[j] >= cnd));
              if (ge >= a.k) prefix = cnd;  // wave-uniform
            }
            return prefix ? unorderable(prefix) : -INFINITY;
          };
          if constexpr (kEarlyFetch) {
#pragma unroll
            for (int qi = 0; qi < NQ; ++qi) {
              uint32_t ord[4];
#pragma unroll
              for (int j = 0; j < 4; ++j) ord[j] = orderable(exq[qi][j]);
              const float th = kth_largest(ord);
              if (lane == 0) thr_s[qi] = th;
            }
          } else {
            for (int qi = 0; qi < NQ; ++qi) {
              const int qg = a.q0 + qi;
              if (qg >= a.BM) break;  // wave-uniform
              const float* src = a.gmax + ((long long)g * a.BM + qg) * a.n_splits;
              uint32_t ord[4];
#pragma unroll
              for (int j = 0; j < 4; ++j)
                ord[j] = (lane + 64 * j < a.n_splits) ? orderable(load_dev(src + lane + 64 * j)) : 0u;
              const float th = kth_largest(ord);
              if (lane == 0) thr_s[qi] = th;
            }
          }
          wave_sync();
#pragma unroll
          for (int tq = 0; tq < NQT; ++tq)
#pragma unroll
            for (int e = 0; e < 2; ++e)
              if (a.q0 + 8 * tq + 2 * rr + e < a.BM)
                thr[tq][e] = fmaxf(thr[tq][e], thr_s[8 * tq + 2 * rr + e]);
          wave_sync();
          // Candidates accepted before the bound was known and now below it can never be among the k best: drop
          // them at once.  What is left is a handful of entries per list, so the final sort of the stream (which
          // every wave runs while the memory system idles) has next to nothing to do.
          if (n == 0) {
#pragma unroll
            for (int tq = 0; tq < NQT; ++tq)
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                cnt_s[8 * tq + 2 * rr + e] = cnt[tq][e];
                thr_s[8 * tq + 2 * rr + e] = thr[tq][e];
              }
          }
          wave_sync();
          for (int qi = 0; qi < NQ; ++qi) {
            constexpr int PER = (CAP + 63) / 64;
            const int c = cnt_s[qi];
            const float th = thr_s[qi];
            unsigned long long* cl = cand + qi * CAP;
            unsigned long long x[PER];
            bool kp[PER];
#pragma unroll
            for (int p = 0; p < PER; ++p) {
              const int j = lane + 64 * p;
              x[p] = (j < c) ? cl[j] : 0ull;
              kp[p] = j < c && key_score(x[p]) >= th;
            }
            wave_sync();  // every entry is in a register before the list is rewritten
            int kept = 0;
#pragma unroll
            for (int p = 0; p < PER; ++p) {
              const unsigned long long m = __ballot(kp[p]);
              if (kp[p]) cl[kept + __popcll(m & ((1ull << lane) - 1ull))] = x[p];
              kept += __popcll(m);
            }
            if (lane == 0) cnt_s[qi] = kept;
          }
          wave_sync();
#pragma unroll
          for (int tq = 0; tq < NQT; ++tq) {
            cnt[tq][0] = cnt_s[8 * tq + 2 * rr];
            cnt[tq][1] = cnt_s[8 * tq + 2 * rr + 1];
          }
          wave_sync();
        }
      }
#pragma unroll
      for (int u = 0; u < kPrefetch; ++u) {
        const long long it = base + u;
        const long long t = tile_at(it);
        // The products read the tile (and the scores its reciprocal norms) where they landed, and only then is
        // the next tile of this slot requested into the same registers.  (Requested earlier, while this tile is
        // still needed, the new tile would have to land in other registers; the slots would wander from one round
        // of the loop to the next and be copied back at its end, and a copy of a register with a load in flight
        // waits for that load, i.e. drains the prefetch.)
        float sraw[NQT][2];
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
          f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < NS; ++s) acc = mfma16(A[tq][s], as_bf16x8(buf[u][s]), acc);
          sraw[tq][0] = (acc[0] + acc[1]) * binv[u];
          sraw[tq][1] = (acc[2] + acc[3]) * binv[u];
          // pinned here: left alone, the compiler sinks one of the two products below the requests (and hoists the
          // requests above them), which keeps the old reciprocal norm alive and sends the new one elsewhere
          asm volatile("" : "+v"(sraw[tq][0]), "+v"(sraw[tq][1])::"memory");
        }
        {
          const long long tn = tile_at((it + kPrefetch < n_it) ? it + kPrefetch : i_last);
#pragma unroll
          for (int s = 0; s < NS; ++s)
            buf[u][s] = load_tile16(KRg + tn * TILE_ELEMS + s * 512);
          binv[u] = COS ? ing[tn * 16] : 1.0f;
        }

        const long long doc = t * dpt + ndoc;
        const bool lead = lead_lane && it < n_it && doc < a.N;
        bool over = false;
        // scores first; the slot arithmetic runs only for tiles in which some lane passes its threshold
        float scv[NQT][2];
        bool any_pred = false;
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float sc = group_max_rt(sraw[tq][e], a.C);
            if (MODE == 2) {
              if (lead) candf[(8 * tq + 2 * rr + e) * CAPF + (int)(t - t0) * dpt + ndoc] = sc;
            } else if (MODE == 1) {
              if (lead) cand[(8 * tq + 2 * rr + e) * CAP + (int)it * dpt + ndoc] = make_key(sc, (uint32_t)doc);
            } else {
              scv[tq][e] = sc;
              if (lead) qmax[tq][e] = fmaxf(qmax[tq][e], sc);
              any_pred = any_pred || (lead && sc >= thr[tq][e]);
            }
          }
        }
        if (!DENSE && __any(any_pred)) {
#pragma unroll
          for (int tq = 0; tq < NQT; ++tq) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const float sc = scv[tq][e];
              const bool pred = lead && sc >= thr[tq][e];
              const unsigned long long m = __ballot(pred);
              const uint32_t half = (rr & 2) ? (uint32_t)(m >> 32) : (uint32_t)m;
              const uint32_t row = (half >> ((rr & 1) * 16)) & 0xffffu;
              if (pred) {
                const int qi = 8 * tq + 2 * rr + e;
                cand[qi * CAP + cnt[tq][e] + __popc(row & below)] = make_key(sc, (uint32_t)doc);
              }
              cnt[tq][e] += __popc(row);
              over = over || cnt[tq][e] > limit;
            }
          }
        }
        if (__any(over)) {
          // rare path: publish the counters, prune the lists that are too long, reload
          if (n == 0) {
#pragma unroll
            for (int tq = 0; tq < NQT; ++tq) {
              cnt_s[8 * tq + 2 * rr] = cnt[tq][0];
              cnt_s[8 * tq + 2 * rr + 1] = cnt[tq][1];
              thr_s[8 * tq + 2 * rr] = thr[tq][0];
              thr_s[8 * tq + 2 * rr + 1] = thr[tq][1];
            }
          }
          wave_sync();
          for (int qi = 0; qi < NQ; ++qi) {
            const int c = cnt_s[qi];
            if (c > limit) {  // wave-uniform
              unsigned long long* cl = cand + qi * CAP;
              const int nc = prune_list<CAP>(cl, c, a.k, lane);
              if (lane == 0) {
                cnt_s[qi] = nc;
                thr_s[qi] = key_score(cl[a.k - 1]);
              }
            }
          }
          wave_sync();
#pragma unroll
          for (int tq = 0; tq < NQT; ++tq) {
            cnt[tq][0] = cnt_s[8 * tq + 2 * rr];
            cnt[tq][1] = cnt_s[8 * tq + 2 * rr + 1];
            thr[tq][0] = thr_s[8 * tq + 2 * rr];
            thr[tq][1] = thr_s[8 * tq + 2 * rr + 1];
          }
          wave_sync();
        }
      }
    }
  }

  // ---- sort every list and hand the k best to the merge kernel --------------------------------
  if (n == 0) {
#pragma unroll
    for (int tq = 0; tq < NQT; ++tq) {
      cnt_s[8 * tq + 2 * rr] = cnt[tq][0];
      cnt_s[8 * tq + 2 * rr + 1] = cnt[tq][1];
    }
  }
  wave_sync();
  // MODE 1, 2: every list holds the same documents, those of the wave's tiles in order; only the
  // last tile of the index can end early
  int c_dense = 0;
  if (DENSE) {
    const long long left = (long long)a.N - ((MODE == 2) ? t0 + i_last : tile_at(i_last)) * dpt;
    c_dense = (int)i_last * dpt + (int)(left < dpt ? (left < 0 ? 0 : left) : dpt);
  }
  if (MODE == 2) {
    const long long doc0 = t0 * dpt;  // the wave's documents are doc0 .. doc0 + c_dense - 1
    int pw = 1;
    while (pw < c_dense) pw <<= 1;  // wave-uniform
    if (pw <= 64) {
      // 64 / pw queries per wave-wide access (lane = query-in-group * pw + document), eight accesses read from
      // LDS before the first is stored: the runs of one query are short, a loop over single queries would spend
      // its time on one dependent LDS read after the other
      const int qpi = 64 / pw;
      const int j = lane & (pw - 1), qo = lane / pw;
      for (int i0 = 0; i0 < NQ; i0 += 8 * qpi) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int qi = i0 + u * qpi + qo;
          v[u] = (qi < NQ && j < c_dense) ? candf[qi * CAPF + j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int qi = i0 + u * qpi + qo;
          if (qi < NQ && a.q0 + qi < a.BM && j < c_dense)
            a.mat[((long long)g * a.BM + a.q0 + qi) * a.N + doc0 + j] = v[u];
        }
      }
      return;
    }
    for (int qi = 0; qi < NQ; ++qi) {
      const int qg = a.q0 + qi;
      if (qg >= a.BM) break;  // wave-uniform
      float* row = a.mat + ((long long)g * a.BM + qg) * a.N + doc0;
      for (int j = lane; j < c_dense; j += 64) row[j] = candf[qi * CAPF + j];
    }
    return;
  }
  for (int qi = 0; qi < NQ; ++qi) {
    const int qg = a.q0 + qi;
    if (qg >= a.BM) break;  // wave-uniform
    const int c = DENSE ? c_dense : cnt_s[qi];
    unsigned long long* cl = cand + qi * CAP;
    const int nc = prune_list<CAP, 16>(cl, c, a.k, lane);
    unsigned long long* dst = a.ws + (((long long)g * a.BM + qg) * a.n_splits + sp) * a.k;
    if (lane < a.k) dst[lane] = (lane < nc) ? cl[lane] : 0ull;
  }
}

// Literal Eq. 2 head mean (select_scope = ALL): the chunk score is the mean over EVERY query head of
// the similarity with the routing key of that head's KV group, i.e. the mean over the Hkv groups of
// the per-group scores above, so one selection serves all heads.  A wave's stream interleaves the
// heads: entry e = (tile e / HKV, head e % HKV) through the same ring of kPrefetch loads; the
// per-head partial scores are scaled by that head's 1/|key| and summed, and after the last head the
// document maxima go to the score matrix mat[query of the pass][document of the segment], from which
// topk_rows_kernel selects.
//
// Bound: the stream of the index (every key once per pass).  A pass therefore takes up to 32 queries (NQT tiles of
// 8): their A operands, HKV x NS x NQT x 1 KiB, lie in LDS once per workgroup and every wave re-reads the slices of
// the head at hand, NQT bytes of LDS per byte of index, a third of the LDS rate at NQT = 4.  With one selection per
// token the matrix is 4 B per (query, document) beside the HKV * C * 2 d B of index behind it: under 1 % at 32
// queries, and it needs no thresholds, lists, sorts or merges of the streams' lists (24 queries over 8192 documents:
// three 8-query passes 88 us + list merge 59 us -> 24 us + row top-k 8 us).
//
// Eight streams per workgroup: the operands of 32 queries leave room for one workgroup per CU, and eight waves of
// four 4 KiB tiles are what keeps the memory system busy.  A wave takes UNITS of 2^ushift tiles (at most 16
// documents), unit w, w + W, ...: at any moment the waves read one contiguous window of the index, and a unit's
// scores leave as one run of up to 64 bytes per query.  HKV in {2, 4, 8} (one group: the plain kernel computes this).
constexpr int kAllWaves = 8;
constexpr int kAllRun = 16;  // documents a wave collects per query before it writes them

constexpr int kAllGroups = 256;  // workgroups: one per CU
// (head, 8 queries) tiles that a workgroup of the all-heads scan folds itself: one for each of its waves, which takes less than
// the launch that would prepare them (4 queries over 13401 documents 18.1 -> 16.4 us, one over 2048 14.5 -> 12.7, 8 over 8192
// 30.3 -> 28.8); with two for each it takes longer (14 queries over 2048, 8 heads: 16.1 -> 18.2).
// Every workgroup reads all queries, so not more than kAllFoldElems of them (88 KiB) over a short index (again and again, prepared ->
// folded: 32 queries of 2 groups of 8 heads, 128 KiB, 1000 documents 13.9 -> 14.3 us, 3000 14.5 -> 15.4, 5500 15.8 -> 16.4, 7000 the
// same; 16 of 4 groups 3000 14.0 -> 14.3, 7000 19.6 -> 18.6; 10 of 4 groups, 80 KiB, 2048 13.7 -> 12.5, 4500 16.4 -> 15.9); from
// kAllFoldTilesIdx tiles of all heads on, 49 MB, they fold more too.
constexpr int kAllFoldTiles = 8;
// (Eight groups, where every wave folds: less than 80 KiB; five queries of 64 heads 13.4 -> 14.2 us, four 13.2 -> 12.3.)
constexpr long long kAllFoldElems = 45056, kAllFoldElems8 = 40959, kAllFoldTilesIdx = 12000;

static bool all_heads_folds(const Dims& dm, const ScorePlan& pl, int BM) {
  return pl.q_per_pass / 8 * dm.Hkv <= kAllFoldTiles &&
         ((long long)BM * dm.Hq * dm.d <= (dm.Hkv == 8 ? kAllFoldElems8 : kAllFoldElems) || (long long)dm.Hkv * dm.tiles >= kAllFoldTilesIdx);
}

// log2(tiles per unit): the unit that keeps the longest stream shortest (whole units per wave), of equals the largest
static int scan_all_ushift(long long seg_tiles, int C) {
  const long long waves = (long long)kAllGroups * kAllWaves;
  int best = 0;
  long long best_len = 0;
  for (int us = 0; (1 << us) <= C; ++us) {  // a unit holds at most kAllRun = 16 documents: 16 / C per tile
    const long long units = (seg_tiles + (1 << us) - 1) >> us;
    const long long len = ((units + waves - 1) / waves) << us;
    if (us == 0 || len <= best_len) {
      best = us;
      best_len = len;
    }
  }
  return best;
}

struct ScanAllArgs {
  const uint4* qop;       // [HKV][n_qtiles][NS][64] prepared A operands (prep_scan_operands_kernel)
  const uint16_t* q_route;  // FOLD: the queries themselves
  int BM, Hq, r;            // FOLD: queries of the call (one pass)
  const uint16_t* KR;     // tiled
  const float* inv_norm;  // null: dot product
  float* mat;             // [queries][mat_stride]
  long long mat_stride;   // documents per row
  int n_qtiles;           // operand tiles
  int nq;                 // queries (<= 8 NQT)
  int C;
  long long tiles;        // tiles per head in the index
  long long tile0;        // first tile of this segment
  long long seg_tiles;    // tiles of this segment
  int seg_docs;           // documents of this segment
  int ushift;             // log2(tiles per unit)
};

// STREAM: streaming loads of the index (see stream_index_of).
// FOLD: the workgroup folds the queries of every head itself, a wave per (head, tile of 8 queries): one launch less.
template <int D, int HKV, int NQT, bool STREAM, bool FOLD>
__global__ __launch_bounds__(64 * kAllWaves) void score_scan_all_kernel(ScanAllArgs a) {
  constexpr int NS = D / 32;
  constexpr int NQ = 8 * NQT;
  constexpr int TILE_ELEMS = 16 * D;
  constexpr int UT = HKV >= kPrefetch ? 1 : kPrefetch / HKV;  // tiles per unrolled group of entries
  static_assert((UT * HKV) % kPrefetch == 0, "ring slots must be compile-time");
  constexpr int NOP = HKV * NQT * NS;                        // KiB of operands
  constexpr int OPW = (NOP + kAllWaves - 1) / kAllWaves;     // copies per wave

  __shared__ uint4 Aop[HKV][NQT][NS][64];
  __shared__ float run_s[kAllWaves][NQ][kAllRun];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float (*run)[kAllRun] = run_s[wave];
  const int rr = lane >> 4;
  const int n = lane & 15;

  // ---- operands: global -> LDS, requested first; the tiles requested next stay in flight across their wait -------
  FoldRegs<D> fr;
  if constexpr (FOLD) {
    if (wave < HKV * NQT) fold_query_load<D>(a.q_route, wave / HKV, wave % HKV, a.BM, a.Hq, a.r, fr, lane);
  } else {
    const uint32_t op_lds = lds_addr_of(&Aop[0][0][0][0]);
#pragma unroll
    for (int i = 0; i < OPW; ++i) {
      int e = i * kAllWaves + wave;  // (head, tile, slice)
      e = e < NOP ? e : NOP - 1;     // past the end: the last piece again (the same bytes to the same place)
      const int h = e / (NQT * NS), rest = e % (NQT * NS);
      const uint4* src = a.qop + ((long long)h * a.n_qtiles * NS + rest) * 64;
      copy16_to_lds_async_at(src, lane * 16, op_lds + e * 1024);
    }
  }

  const long long W = (long long)gridDim.x * kAllWaves;
  const long long w = (long long)blockIdx.x * kAllWaves + wave;
  const int umask = (1 << a.ushift) - 1;
  const long long units = (a.seg_tiles + umask) >> a.ushift;
  const long long n_it = w < units ? ((units - w + W - 1) / W) << a.ushift : 0;  // tiles of this wave
  const uint16_t* KRl = a.KR + lane * 8;
  // dot product: the loads of the reciprocal norms run all the same (from the first bytes of the index, always the
  // same), so that the loads in flight are the same on every path, and a one takes their place
  const bool cos = a.inv_norm != nullptr;
  const float* inl = (cos ? a.inv_norm : reinterpret_cast<const float*>(a.KR)) + n;
  const long long inv_stride = cos ? 16 : 0;
  // tile number inside the segment; past the wave's end or the segment's: see clamp below
  auto tile_at = [&](long long it) { return ((w + (it >> a.ushift) * W) << a.ushift) + (it & umask); };
  auto load_at = [&](long long it) {  // always a tile of the index
    const long long t = tile_at(it);
    return a.tile0 + (t < a.seg_tiles ? t : a.seg_tiles - 1);
  };
  auto load_tile16 = [](const uint16_t* p) {
    const u32x4_t* v = reinterpret_cast<const u32x4_t*>(p);
    return STREAM ? __builtin_nontemporal_load(v) : *v;
  };
  u32x4_t buf[kPrefetch][NS];  // whole vectors throughout: element-wise uses would be put back together with copies
  float binv[kPrefetch];
  auto first_entry = [&](int u) __attribute__((always_inline)) {
    const int h = u % HKV;
    const long long t = load_at(u / HKV);
#pragma unroll
    for (int s = 0; s < NS; ++s)
      buf[u][s] = load_tile16(KRl + ((long long)h * a.tiles + t) * TILE_ELEMS + s * 512);
    binv[u] = inl[((long long)h * a.tiles + t) * inv_stride];
  };
  if constexpr (FOLD) {
    // (the folding behind one request, not behind all of them: see score_scan_kernel)
    first_entry(0);
    static_assert(HKV * NQT <= kAllWaves, "a tile per wave");
    static_assert(8 * D * 4 == NS * 64 * 16, "the folded queries take the place of their operands");
    if (wave < HKV * NQT) {
      const int h = wave % HKV, t = wave / HKV;
      fold_query_tile<D>(fr, t, a.BM, a.r, cos ? 1 : 0, reinterpret_cast<float*>(&Aop[h][t][0][0]), Aop[h][t], lane);
    }
#pragma unroll
    for (int u = 1; u < kPrefetch; ++u) first_entry(u);
  } else {
#pragma unroll
    for (int u = 0; u < kPrefetch; ++u) first_entry(u);
    wait_copies_but<kPrefetch * (NS + 1)>();  // the operands are older than the tiles
  }
  lds_barrier();
  if (n_it == 0) return;  // wave-uniform; no workgroup barrier follows

  const int dpt = 16 / a.C;
  const int ndoc = n / a.C;
  const bool lead = (n & (a.C - 1)) == 0;
  const float inv_heads = 1.0f / (float)HKV;
  const int dshift = a.ushift + 4 - (31 - __clz(a.C));  // log2(documents per unit): dpt << ushift <= kAllRun
  const int du = 1 << dshift;

  for (long long base = 0; base < n_it; base += UT) {
#pragma unroll
    for (int ut = 0; ut < UT; ++ut) {
      const long long it = base + ut;
      float tot[NQT][2];
#pragma unroll
      for (int tq = 0; tq < NQT; ++tq) tot[tq][0] = tot[tq][1] = 0.f;
#pragma unroll
      for (int h = 0; h < HKV; ++h) {
        const int slot = (ut * HKV + h) % kPrefetch;
        // products first, where the tile landed; the next tile of the slot is requested into the same registers
        // afterwards (see score_scan_kernel)
        float part[NQT][2];
        // the entry is awaited HERE: its uses pass through volatile asm, so that no use of a later entry (and the
        // wait for it) moves up ahead of the requests in between
#pragma unroll
        for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(buf[slot][s]));
        asm volatile("" : "+v"(binv[slot]));
        const float inv = cos ? binv[slot] : 1.0f;
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
          f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < NS; ++s) acc = mfma16(as_bf16x8(Aop[h][tq][s][lane]), __builtin_bit_cast(bf16x8_t, buf[slot][s]), acc);
          part[tq][0] = acc[0] + acc[1];
          part[tq][1] = acc[2] + acc[3];
          asm volatile("" : "+v"(part[tq][0]), "+v"(part[tq][1]));
        }
        asm volatile("" ::: "memory");
        {  // the entry kPrefetch ahead of this one takes over the slot (always issued)
          const int en = ut * HKV + h + kPrefetch;
          const int hn = en % HKV;
          const long long tn = load_at(base + en / HKV);
#pragma unroll
          for (int s = 0; s < NS; ++s)
            buf[slot][s] = load_tile16(KRl + ((long long)hn * a.tiles + tn) * TILE_ELEMS + s * 512);
          binv[slot] = inl[((long long)hn * a.tiles + tn) * inv_stride];
        }
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
          tot[tq][0] = fmaf(part[tq][0], inv, tot[tq][0]);
          tot[tq][1] = fmaf(part[tq][1], inv, tot[tq][1]);
        }
      }
      if (UT > 1 && it >= n_it) break;  // wave-uniform
      const int in_unit = (int)(it & umask);
      // document maxima, one level of the exchange at a time for all scores (the branches are wave-uniform)
#pragma unroll
      for (int tq = 0; tq < NQT; ++tq) {
        tot[tq][0] *= inv_heads;
        tot[tq][1] *= inv_heads;
      }
      auto level = [&](auto ctrl) {
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
          tot[tq][0] = fmaxf(tot[tq][0], dpp_f<decltype(ctrl)::value>(tot[tq][0]));
          tot[tq][1] = fmaxf(tot[tq][1], dpp_f<decltype(ctrl)::value>(tot[tq][1]));
        }
      };
      if (a.C >= 2) level(std::integral_constant<int, kDppXor1>{});
      if (a.C >= 4) level(std::integral_constant<int, kDppXor2>{});
      if (a.C >= 8) level(std::integral_constant<int, kDppHalfMirror>{});
      if (a.C >= 16) level(std::integral_constant<int, kDppMirror>{});
      if (lead) {
#pragma unroll
        for (int tq = 0; tq < NQT; ++tq) {
          run[8 * tq + 2 * rr][in_unit * dpt + ndoc] = tot[tq][0];
          run[8 * tq + 2 * rr + 1][in_unit * dpt + ndoc] = tot[tq][1];
        }
      }
      if (in_unit == umask) {  // the unit is complete: one run of du documents per query
        wave_sync();
        const long long doc0 = (tile_at(it) - umask) * dpt;  // document inside the segment
        const int j = lane & (du - 1), qo = lane >> dshift, qpi = 64 >> dshift;
        if (doc0 + j < a.seg_docs) {
          for (int qi = qo; qi < a.nq; qi += qpi) a.mat[qi * a.mat_stride + doc0 + j] = fmaxf(run[qi][j], -INFINITY);  // (not a number: last)
        }
        wave_sync();
      }
    }
  }
}

// Literal Eq. 2 token pooling (token_pool = 1): the document score of a question is the max over its
// M query tokens.  The k best documents under that score are all contained in the union of the
// per-token top-k lists: if document D is among them and token m* attains its maximum, every document
// ahead of D in token m*'s ranking is also ahead of D in the pooled ranking, so fewer than k are, and
// D is in m*'s list with exactly its pooled score.  Ranking the union by (best listed score desc,
// index asc) therefore reproduces the pooled top-k exactly.  One block per (batch row, scope slot):
// the listed entries at or above a floor go through a hash table in LDS that keeps the best entry per document (rounds
// of arg-max that skip the documents taken pay two barriers per selected document: 150 tokens, k = 32: 58 -> 8 us), and
// of its documents those that reach a lower bound on the k-th best are ranked by counting (1877 tokens, k = 15: all
// documents of the table 469 us, those 31).  More documents than the table takes: k rounds of a block-wide arg-max over the M*k
// listed keys, skipping documents already taken.
constexpr int kPoolThreads = 1024;
constexpr int kPoolSlots = 8192;                  // hash table
constexpr int kPoolDocs = kPoolSlots / 2;         // documents it takes (every thread can be one insertion past it)

__global__ __launch_bounds__(kPoolThreads) void pool_tokens_kernel(const unsigned long long* __restrict__ tok_keys,
                                                          int32_t* __restrict__ out_idx,
                                                          float* __restrict__ out_score, int M, int S,
                                                          int k) {
  __shared__ unsigned long long slots[kPoolSlots];
  __shared__ unsigned long long surv[kPoolDocs + 8];
  __shared__ unsigned long long red[kPoolThreads / 64];
  __shared__ uint32_t taken[MSA_MAX_TOPK];
  __shared__ uint32_t theta_w[2][kPoolThreads / 64];
  __shared__ int n_docs, n_surv;
  const int tid = threadIdx.x;
  const int b = blockIdx.x / S;
  const int sl = blockIdx.x % S;
  const long long o_base = ((long long)b * S + sl) * k;
  const int T = M * k;
  auto key_at = [&](int i) {
    const int m = i / k, j = i - m * k;
    return tok_keys[(((long long)b * M + m) * S + sl) * k + j];
  };
  auto block_max = [&](unsigned long long best) {
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
    for (int w = 1; w < kPoolThreads / 64; ++w) best = red[w] > best ? red[w] : best;
    return best;
  };
  for (int i = tid; i < kPoolSlots; i += kPoolThreads) slots[i] = 0ull;
  if (tid == 0) n_docs = n_surv = 0;
  // 1. A floor: one token's k listed documents already have pooled scores >= its k-th listed score,
  //    so the pooled k-th best score is at least the largest such k-th score; lower entries drop out.
  unsigned long long fl = 0ull;
  for (int m = tid; m < M; m += kPoolThreads) {
    const unsigned long long x = tok_keys[(((long long)b * M + m) * S + sl) * k + (k - 1)];
    fl = x > fl ? x : fl;
  }
  fl = block_max(fl);  // (its barriers also order the cleared table)
  const uint32_t floor_bits = (uint32_t)(fl >> 32);  // score bits only: entries that tie with the floor stay
  // 2. The best entry of every document.  A slot belongs to one document once it is filled (the low half of a key);
  //    the table is never full, so every search ends.
  for (int i = tid; i < T; i += kPoolThreads) {
    const unsigned long long x = key_at(i);
    if (x == 0ull || (uint32_t)(x >> 32) < floor_bits) continue;
    if (*(volatile int*)&n_docs > kPoolDocs) break;  // too many documents: the rounds below take over
    uint32_t h = ((uint32_t)x * 2654435761u) >> 19;  // 13 bits: kPoolSlots
    static_assert(kPoolSlots == 1 << 13, "hash width");
    for (;;) {
      const unsigned long long old = atomicCAS(&slots[h], 0ull, x);
      if (old == 0ull) {
        atomicAdd(&n_docs, 1);
        break;
      }
      if ((uint32_t)old == (uint32_t)x) {
        atomicMax(&slots[h], x);
        break;
      }
      h = (h + 1) & (kPoolSlots - 1);
    }
  }
  __syncthreads();
  if (n_docs <= kPoolDocs) {
    // 3. The documents that reach a lower bound on the k-th best, side by side, ranked by counting.
    unsigned long long mine[kPoolSlots / kPoolThreads];
    uint32_t ob = 0u;
#pragma unroll
    for (int u = 0; u < kPoolSlots / kPoolThreads; ++u) {
      mine[u] = slots[u * kPoolThreads + tid];
      const uint32_t o = (uint32_t)(mine[u] >> 32);
      ob = o > ob ? o : ob;
    }
    const uint32_t theta = kth_best_bound<kPoolThreads / 64>(ob, k, theta_w);
#pragma unroll
    for (int u = 0; u < kPoolSlots / kPoolThreads; ++u)
      if (mine[u] != 0ull && (uint32_t)(mine[u] >> 32) >= theta) surv[atomicAdd(&n_surv, 1)] = mine[u];
    __syncthreads();
    const int ns = n_surv;
    if (tid < 8) surv[ns + tid] = 0ull;  // the rank count reads eight at a time (zero: greater than no key)
    __syncthreads();
    for (int i = tid; i < ns; i += kPoolThreads) {
      const unsigned long long x = surv[i];
      int rank = 0;
      for (int j = 0; j < ns; j += 8) {
        unsigned long long y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = surv[j + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (y[u] > x) ? 1 : 0;
      }
      if (rank < k) {
        out_idx[o_base + rank] = (int32_t)key_doc(x);
        if (out_score) out_score[o_base + rank] = key_score(x);
      }
    }
    for (int i = ns + tid; i < k; i += kPoolThreads) {  // fewer than k documents
      out_idx[o_base + i] = -1;
      if (out_score) out_score[o_base + i] = -INFINITY;
    }
    return;
  }
  // Fallback (more documents than the table takes): rounds over the lists in memory, skipping taken documents.
  unsigned long long prev = ~0ull;
  for (int round = 0; round < k; ++round) {
    unsigned long long best = 0ull;
    for (int i = tid; i < T; i += kPoolThreads) {
      const unsigned long long x = key_at(i);
      if (x == 0ull || x >= prev || x <= best) continue;  // keys of one document differ in the score bits only
      const uint32_t doc = key_doc(x);
      bool dup = false;
      for (int w = 0; w < round; ++w) dup = dup || taken[w] == doc;
      if (!dup) best = x;
    }
    best = block_max(best);
    if (tid == 0) {
      out_idx[o_base + round] = best ? (int32_t)key_doc(best) : -1;
      if (out_score) out_score[o_base + round] = best ? key_score(best) : -INFINITY;
      taken[round] = best ? key_doc(best) : 0xffffffffu;
    }
    __syncthreads();
    prev = best ? best : 0ull;
  }
}

// Top-k of the rows of a document score matrix (MODE 2 of the scan, all-heads scan).  One workgroup per (row, part
// of the row).
//   1. every thread takes the best score of its strided share of the part, and kth_best_bound gives a lower bound theta
//      on the k-th best score of the part;
//   2. every document scoring >= theta goes to LDS (a few k of them) and is ranked by counting on the full
//      key.
// Exact, ties included (keys are (score, ~doc): a total order; theta compares scores only, so equal scores
// survive together).  If more survive than LDS holds (ties), topk_of_ties takes over.
constexpr int kRowSurv = 2048;
constexpr int kRowRegs = 32;        // scores a thread keeps in registers between the two passes (8: short rows)
constexpr int kRowPart = 8192;      // documents per part of a long row: what 32 registers per thread of four waves hold, or
                                    // 16 of eight

struct RowsArgs {
  const float* mat;           // [selections][BM][stride]
  long long stride;           // documents per matrix row
  int BM;                     // queries
  int n_sel;                  // selections per query
  int n_docs, doc0;           // documents of a row and the number of its first one
  int parts, part_docs;       // parts of a row
  int part0, parts_total;     // part lists: number of this launch's first part, parts per (selection, query)
  int k;
  int32_t* out_idx;           // whole rows: the final selection ...
  float* out_score;
  unsigned long long* out_key;   // ... or (not null) its sorted keys [BM][n_sel][k]
  unsigned long long* part_keys; // not null: sorted keys per part, [n_sel][BM][parts_total][k]
};

template <int REGS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void topk_rows_kernel(RowsArgs a) {
  __shared__ unsigned long long surv[kRowSurv + 8];
  __shared__ uint32_t theta_w[2][WAVES];
  __shared__ int cnt_s[WAVES];
  __shared__ int n_surv;
  constexpr int THREADS = 64 * WAVES;
  const int tid = threadIdx.x;
  const int k = a.k;
  const int part = blockIdx.x % a.parts;
  const int row_no = blockIdx.x / a.parts;
  const int qg = row_no % a.BM;
  const int g = row_no / a.BM;
  const int first = part * a.part_docs;
  const int N = a.n_docs - first < a.part_docs ? a.n_docs - first : a.part_docs;  // documents of this part
  const float* __restrict__ row = a.mat + (long long)row_no * a.stride + first;
  const uint32_t doc0 = (uint32_t)(a.doc0 + first);
  if (tid == 0) n_surv = 0;
  float v[REGS];
#pragma unroll
  for (int u = 0; u < REGS; ++u) {
    const int i = u * THREADS + tid;
    v[u] = (i < N) ? row[i] : 0.f;
  }
  // the rest of a row longer than the registers hold, eight loads in flight
  auto rest_of_row = [&](auto use) {
    for (int i0 = REGS * THREADS + tid; i0 < N; i0 += 8 * THREADS) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = (i0 + u * THREADS < N) ? row[i0 + u * THREADS] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) use(i0 + u * THREADS, x[u]);
    }
  };
  uint32_t ob = 0u;
  auto best_of = [&](int i, float x) {
    const uint32_t o = i < N ? orderable(x) : 0u;
    ob = o > ob ? o : ob;
  };
#pragma unroll
  for (int u = 0; u < REGS; ++u) best_of(u * THREADS + tid, v[u]);
  rest_of_row(best_of);
  const uint32_t theta = kth_best_bound<WAVES>(ob, k, theta_w);
  auto keep = [&](int i, float x) {
    if (i < N && orderable(x) >= theta) {
      const int slot = atomicAdd(&n_surv, 1);
      if (slot < kRowSurv) surv[slot] = make_key(x, doc0 + i);
    }
  };
#pragma unroll
  for (int u = 0; u < REGS; ++u) keep(u * THREADS + tid, v[u]);
  rest_of_row(keep);
  __syncthreads();
  const int ns = n_surv;
  const long long o_base = a.part_keys
                               ? (((long long)g * a.BM + qg) * a.parts_total + a.part0 + part) * k
                               : ((long long)qg * a.n_sel + g) * k;
  auto emit = [&](int rank, unsigned long long x) {
    if (a.part_keys) {
      a.part_keys[o_base + rank] = x;
    } else if (a.out_key) {
      a.out_key[o_base + rank] = x;
    } else {
      a.out_idx[o_base + rank] = x ? (int32_t)key_doc(x) : -1;
      if (a.out_score) a.out_score[o_base + rank] = x ? key_score(x) : -INFINITY;
    }
  };
  if (ns <= kRowSurv) {
    if (tid < 8) surv[ns + tid] = 0ull;  // the rank count below reads eight at a time (zero: greater than no key)
    __syncthreads();
    for (int i = tid; i < ns; i += THREADS) {
      const unsigned long long x = surv[i];
      int rank = 0;
      for (int j = 0; j < ns; j += 8) {
        unsigned long long y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = surv[j + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (y[u] > x) ? 1 : 0;
      }
      if (rank < k) emit(rank, x);
    }
    for (int i = ns + tid; i < k; i += THREADS) emit(i, 0ull);  // fewer than k documents (a short part)
    return;
  }
  topk_of_ties<REGS, WAVES>(v, row, N, doc0, k, theta, ob, surv, &n_surv, cnt_s);
  if (tid < k) {
    const unsigned long long x = surv[tid];
    int rank = 0;
    for (int j = 0; j < k; ++j) rank += (surv[j] > x) ? 1 : 0;
    emit(rank, x);
  }
}

// Streaming loads of the index: always from 300 MB on, of which the 256 MB of cache behind the L2s keep nothing until it is read again
// (index cold / again and again, whole call, 8 queries: 20000 documents, 328 MB, 73.3 / 69.0 -> 66.0 / 64.8 us, 32768 110 / 106 -> 99 /
// 95.5; 50 tokens over all heads 16600, 272 MB, 98.6 / 85 -> 93.7 / 89.7, 20000 104.8 / 101.5 -> 99.2 / 96.5), and from 128 MB on in one
// pass of a scan.  A program reads more than that cache holds between two scans of an index (the selected documents of its
// streams, the indexes of its other layers, its weights), so the scan finds it cold, and plain loads spend their time on caching
// what nobody reads again; where the cache holds what was written just before, they wait for that to go to memory.  An index of
// 128 to 300 MB that is routed over again and again with nothing read in between is what they are better at (cold / behind 640 MB
// that were written / again and again):
//   8 queries: 7900 documents, 129 MB, 34.6 / 54.7 / 29.5 -> 32.8 / 36.4 / 29.6 us, 9000 41.8 / 65.3 / 35.6 -> 38.9 / 43.8 / 36.5, 13000
//   52.5 / 80.8 / 45.0 -> 49.0 / 55.6 / 46.6, 15600, 256 MB, 60.0 / 87.8 / 52.0 -> 55.8 / 62.4 / 53.9; one query the same;
//   32 queries: 9000 53.6 / 76.4 / 47.3 -> 52.3 / 54.8 / 49.6, 13000 66.6 / 93.4 / 57.3 -> 62.8 / 68.1 / 60.9; from 290 MB on faster in all
//   three (18000 80.2 / 121.6 / 75.8 -> 73.9 / 83.2 / 72.2);
//   all heads, 24 queries, cold / again and again: 7900 36.1 / 31.8 -> 33.8 / 31.6, 11000 49.1 / 42.6 -> 44.9 / 42.6, 13000 55.2 / 47.0 ->
//   50.3 / 48.5, 15600 62.6 / 54.0 -> 56.1 / 54.2; 22000 of 64 dims 51.1 / 42.4 -> 45.8 / 44.4; but more than eight queries of one or two
//   chunks per document gained 2 to 7 % and lost 4 to 12 % (13 over 79101 documents of one chunk, 8 heads of 128 dims, 50.1 / 42.8 ->
//   47.9 / 44.8; 26 over 52734 of two 67.6 / 56.1 -> 63.1 / 59.6; 957 drawn calls 0.97 / 1.08 times) and keep plain loads.
// Four layers of 134 MB in turn, 8 queries: 214 -> 194 us with the other changes of the scan; the first step after the indexes
// were written 692 -> 675, in its spread.
// Below 128 MB an index may well be in the cache still when it is read again (5000 documents, 82 MB, 8 queries 24.6 / 21.5 -> 23.7 /
// 22.6, 6800, 111 MB, 29.9 / 25.8 -> 28.3 / 27.4); so it may for the second pass of a call.
bool stream_index_of(const Dims& dm, bool cold) {
  const size_t bytes = (size_t)dm.Hkv * dm.tiles * 16 * dm.d * 2;
  return bytes >= 300000000 || (cold && bytes >= 128000000);
}

// Scans of four query tiles fold in every wave, so nobody requests tiles meanwhile; a stream of more than a few tiles per wave then
// loses more than the operands that are ready earlier give (index again and again, all ahead -> one: 32 queries over 2048
// documents, 4 tiles per wave, 18.4 -> 17.4 us, 3500, 7 tiles, 25.6 -> 26.2, 9000, 18 tiles, 44.3 -> 45.8, 13000 53.8 -> 56.4; 24
// queries, whose last tile is empty, 4000, 8 tiles, 24.8 -> 24.3, 6000 30.6 -> 30.7, 13000 53.0 -> 54.1; index cold about half of
// each).
static bool late_requests(const ScorePlan& pl, int BM) {
  return pl.q_per_pass < 32 || pl.tiles_per_wave <= (BM <= 24 ? 8 : 6);
}

// Waves per workgroup: sixteen where the rows leave the chip idle anyway (one round of 256 workgroups or fewer) and a row
// is longer than four waves hold in registers: 32768 scores at once.  One workgroup then takes a row that went in parts
// with a merge launch behind: 30000 documents of 64 dims, 2 queries, whole call 27.4 -> 24.6 us; 20000 of 128, one query,
// 71.8 -> 68.  Eight waves for rows of 2049 to 8192 documents: a thread's share is 16 scores, not 32 (64 rows of 8192: 7.2 -> 5.9
// us, 24 rows 6.5 -> 5.1; sixteen waves 6.0 and 5.4).  Shorter rows gain nothing (8 rows of 2048: call 12.3 us with four
// waves, 12.1 with eight, 12.8 with sixteen; 24 of 700 11.0, 11.3, 14.1).
static void launch_topk_rows(const RowsArgs& ra, hipStream_t st) {
  const unsigned blocks = (unsigned)(ra.BM * ra.n_sel * ra.parts);
  const int n = ra.n_docs < ra.part_docs ? ra.n_docs : ra.part_docs;
#define MSA_TOPK_ROWS(RR, WW) \
  hipLaunchKernelGGL((topk_rows_kernel<RR, WW>), dim3(blocks), dim3(64 * WW), 0, st, ra)
  if (n <= 8 * 256) MSA_TOPK_ROWS(8, 4);
  else if (blocks > 256) MSA_TOPK_ROWS(kRowRegs, 4);
  else if (n <= kRowPart) MSA_TOPK_ROWS(kRowPart / 512, 8);
  else MSA_TOPK_ROWS(kRowRegs, 16);
#undef MSA_TOPK_ROWS
}

// Combine the n_lists sorted lists (k entries each, zero-padded) of one (query, group).
//   1. A lower bound theta on the k-th best score: the first j+1 entries of every list, with
//      n_lists*(j+1) >= k, are that many distinct candidates; kth_best_bound of their scores.  Where several of them tie with
//      it, or differ in the bits only that it leaves out, or more than kFewSurv entries reach it, their k-th best key instead.
//   2. Survivors (key >= theta) are compacted into LDS and ranked by counting.
//   3. If more than kMaxSurv survive (k > 32: the best of every list in a few lists), fall back to k rounds of block-wide argmax.
constexpr int kMaxSub = 1152;
constexpr int kMaxSurv = 2048;
constexpr int kFewSurv = 256;  // one entry per thread to rank
constexpr int kFewTies = 8;

// out_key != null: the winners are written as 64-bit keys instead (input of pool_tokens_kernel).
// out_parts > 1: first level of a two-level merge for very many lists.  Block (g, qg, part), part < parts, combines
// lists [part * lpp, (part + 1) * lpp) and writes its k winners as a sorted list of keys to
// out_key[g][qg][part0 + part][k], the input layout of a second call with n_lists = out_parts.
// nan_docs: a query without a candidate takes the first k documents, as the selection from a matrix row does, with the score that
// the products of the scan have then (it ranks below all others in token pooling).
__global__ __launch_bounds__(256) void score_merge_kernel(const unsigned long long* __restrict__ ws,
                                                          int32_t* __restrict__ out_idx,
                                                          float* __restrict__ out_score,
                                                          unsigned long long* __restrict__ out_key,
                                                          int BM, int Hkv, int n_lists_total, int k,
                                                          int lpp, int parts, int part0, int out_parts,
                                                          const int* __restrict__ gate, int gate_tokens,
                                                          int gate_blocks, int nan_docs) {
  __shared__ unsigned long long sub[kMaxSub + 8];
  __shared__ unsigned long long surv[kMaxSurv];
  __shared__ unsigned long long red[4];
  __shared__ unsigned long long theta_s;
  __shared__ uint32_t theta_w[2][4];
  __shared__ int n_surv;
  const int tid = threadIdx.x;
  const int part = blockIdx.x % parts;
  const int qg = (blockIdx.x / parts) % BM;
  const int g = blockIdx.x / parts / BM;
  // behind the one-pass filter of the scoring GEMM: only the token blocks it flagged have lists to merge
  if (gate != nullptr && gate[g * gate_blocks + qg / gate_tokens] == 0) return;
  const int l0 = part * lpp;
  const int n_lists = (n_lists_total - l0 < lpp) ? n_lists_total - l0 : lpp;
  const int T = n_lists * k;
  const unsigned long long* src = ws + (((long long)g * BM + qg) * n_lists_total + l0) * k;
  const long long o_base =
      (out_parts > 1) ? (((long long)g * BM + qg) * out_parts + part0 + part) * k : ((long long)qg * Hkv + g) * k;

  const int depth = (k + n_lists - 1) / n_lists;  // entries taken from the head of every list
  // k <= P < k + n_lists; any kMaxSub >= k heads of lists bound the k-th best key just as well
  const int P = (n_lists * depth <= kMaxSub) ? n_lists * depth : kMaxSub;
  for (int i = tid; i < P; i += 256) sub[i] = src[(i / depth) * k + (i % depth)];
  if (tid < 8) sub[P + tid] = 0ull;  // read eight at a time below (zero: greater than no key)
  if (tid == 0) {
    n_surv = 0;
    theta_s = 0ull;
  }
  __syncthreads();
  // (Ranking the heads one against the other for their exact k-th took 2 us of this kernel's 7.5 with 256 lists.  Up to 64 are
  // ranked sooner than bounded: 16384 merges of the GEMM's few lists, k = 16, whole call 352 -> 343 us, 6464 of 65 documents
  // 108 -> 103.)
  bool exact = P <= 64;
  unsigned long long theta = 0ull;
  if (!exact) {  // block-uniform
    uint32_t ob = 0u;
    for (int i = tid; i < P; i += 256) {
      const uint32_t o = (uint32_t)(sub[i] >> 32);
      ob = o > ob ? o : ob;
    }
    const uint32_t bound = kth_best_bound<4>(ob, k, theta_w);
    theta = (unsigned long long)bound << 32;
    // A query of zeros (an empty slot of a batch) ties with every document, copies of the best documents with each other: all
    // entries of all lists may reach a bound of score bits, and every list would be walked to its end (8 queries, 2 of them zeros,
    // 97656 documents, k = 32, whole call 428 us, with their exact k-th key 291; 3000 copies of the best document 405, 270).
    int ties = 0;  // heads in the interval of scores that starts with the bound (the same in every wave)
    for (int i0 = 0; i0 < P; i0 += 64) {
      const uint32_t o = i0 + (tid & 63) < P ? (uint32_t)(sub[i0 + (tid & 63)] >> 32) : 0u;
      ties += __popcll(__ballot(o != 0u && (o & ~0xfffu) == bound));
    }
    exact = ties > kFewTies;
  }
  auto kth_head = [&]() -> unsigned long long {  // the k-th best of the heads (0: fewer); a barrier inside
    for (int i = tid; i < P; i += 256) {
      const unsigned long long x = sub[i];
      int rank = 0;
      for (int j = 0; j < P; j += 8) {
        unsigned long long y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) y[u] = sub[j + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (y[u] > x) ? 1 : 0;
      }
      if (rank == k - 1 && x != 0ull) theta_s = x;  // keys are distinct, zeros are padding
    }
    __syncthreads();
    return theta_s;
  };
  int S;
  for (;;) {  // once or twice
    if (exact) theta = kth_head();
    if (n_lists * depth <= kMaxSub) {
      // The heads of all lists are in LDS already, and the lists are sorted: a list holds further survivors only if
      // the last entry seen of it is still >= theta, and then only as far as its entries stay >= theta.  After the
      // streams' thresholds have converged that is a handful of entries per (query, head) instead of n_lists * k.
      for (int l = tid; l < n_lists; l += 256) {
        bool more = true;
        for (int j = 0; j < depth; ++j) {
          const unsigned long long x = sub[l * depth + j];
          more = x != 0ull && x >= theta;
          if (!more) break;
          const int slot = atomicAdd(&n_surv, 1);
          if (slot < kMaxSurv) surv[slot] = x;
        }
        for (int j = depth; more && j < k; ++j) {
          const unsigned long long x = src[l * k + j];
          more = x != 0ull && x >= theta;
          if (more) {
            const int slot = atomicAdd(&n_surv, 1);
            if (slot < kMaxSurv) surv[slot] = x;
          }
        }
      }
    } else {
      for (int i0 = 0; i0 < T; i0 += 256 * 8) {  // eight independent loads per thread in flight
        unsigned long long x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = i0 + u * 256 + tid;
          x[u] = (i < T) ? src[i] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (x[u] != 0ull && x[u] >= theta) {
            const int slot = atomicAdd(&n_surv, 1);
            if (slot < kMaxSurv) surv[slot] = x[u];
          }
        }
      }
    }
    __syncthreads();
    S = n_surv;
    if (exact || S <= kFewSurv) break;  // block-uniform
    exact = true;
    if (S <= kMaxSurv) {  // what survived is in LDS: no second walk
      unsigned long long x[kMaxSurv / 256];
#pragma unroll
      for (int u = 0; u < kMaxSurv / 256; ++u) x[u] = u * 256 + tid < S ? surv[u * 256 + tid] : 0ull;
      theta = kth_head();  // (a barrier inside)
      if (tid == 0) n_surv = 0;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kMaxSurv / 256; ++u)
        if (x[u] != 0ull && x[u] >= theta) surv[atomicAdd(&n_surv, 1)] = x[u];
      __syncthreads();
      S = n_surv;
      break;
    }
    __syncthreads();
    if (tid == 0) n_surv = 0;
  }
  if (S <= kMaxSurv) {
    for (int i = tid; i < S; i += 256) {
      const unsigned long long x = surv[i];
      int rank = 0;
      for (int j = 0; j < S; ++j) rank += (surv[j] > x) ? 1 : 0;
      if (rank < k) {
        if (out_key) {
          out_key[o_base + rank] = x;
        } else {
          out_idx[o_base + rank] = (int32_t)key_doc(x);
          if (out_score) out_score[o_base + rank] = key_score(x);
        }
      }
    }
    for (int i = S + tid; i < k; i += 256) {  // fewer than k candidates: no score of the query is a number
      const bool nan = nan_docs && S == 0;
      const float sc = __uint_as_float(0xffc00000u);
      if (out_key) {
        out_key[o_base + i] = nan ? make_key(sc, (uint32_t)i) : 0ull;
      } else {
        out_idx[o_base + i] = nan ? i : -1;
        if (out_score) out_score[o_base + i] = nan ? sc : -INFINITY;
      }
    }
    return;
  }
  // fallback: k rounds of "largest key below the previous winner"
  unsigned long long prev = ~0ull;
  for (int round = 0; round < k; ++round) {
    unsigned long long best = 0ull;
    for (int i = tid; i < T; i += 256) {
      const unsigned long long x = src[i];
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
    for (int w = 1; w < 4; ++w) best = red[w] > best ? red[w] : best;
    if (tid == 0) {
      if (out_key) {
        out_key[o_base + round] = best;
      } else {
        out_idx[o_base + round] = best ? (int32_t)key_doc(best) : -1;
        if (out_score) out_score[o_base + round] = best ? key_score(best) : -INFINITY;
      }
    }
    prev = best ? best : 0ull;
  }
}

// One workgroup per (tile of 8 queries, KV head), a wave per 512 / D of its queries: fold the r heads of the group into one fp32 routing
// query per token,  qf = (1/r) sum_h q_h / max(|q_h|, 1e-12)  (plain mean for the dot product), split it
// into bf16 hi + lo and store the MFMA A operands of the tile: lane 16q + n holds row n (query n/2,
// hi for even n, lo for odd n), dims 32s + 8q .. +8 of slice s.  Also resets the threshold-exchange
// buffer of the scan to -inf.
template <int D>
__global__ __launch_bounds__(64 * (D / 64)) void prep_scan_operands_kernel(const uint16_t* __restrict__ q_route,
                                                                uint4* __restrict__ qop, int BM, int Hq,
                                                                int Hkv, int r, int cos, int n_qtiles,
                                                                float* __restrict__ gmax, long long n_gmax) {
  constexpr int NS = D / 32, LPH = D / 8, HPL = 64 / LPH, WAVES = 8 / HPL;
  __shared__ float qf[8][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qt = blockIdx.x % n_qtiles;
  const int g = blockIdx.x / n_qtiles;
  if (gmax != nullptr) {
    for (long long i = (long long)blockIdx.x * (64 * WAVES) + threadIdx.x; i < n_gmax;
         i += (long long)gridDim.x * (64 * WAVES))
      gmax[i] = -INFINITY;
  }
  // Lane = (query lane / LPH, 16-byte piece lane % LPH): a lane loads the same piece of all r heads of
  // its query, so the head sum stays in the lane and the norms need only DPP sums over LPH <= 16 lanes.
  const int piece = lane % LPH;
  {
    const int qi = wave * HPL + lane / LPH;
    const bool live = (long long)qt * 8 + qi < BM;
    const long long qg = live ? (long long)qt * 8 + qi : BM - 1;
    // no branch around a load (rows past the end re-read the last query, heads past r the last head): all are in
    // flight together
    uint4 v[8];
#pragma unroll
    for (int hh = 0; hh < 8; ++hh) {
      const int hc = hh < r ? hh : r - 1;
      v[hh] = *reinterpret_cast<const uint4*>(q_route + (qg * Hq + g * r + hc) * D + piece * 8);
    }
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = 0.f;
#pragma unroll
    for (int hh = 0; hh < 8; ++hh) {
      if (hh < r) {  // wave-uniform
        const float x[8] = {bf16_lo(v[hh].x), bf16_hi(v[hh].x), bf16_lo(v[hh].y), bf16_hi(v[hh].y),
                            bf16_lo(v[hh].z), bf16_hi(v[hh].z), bf16_lo(v[hh].w), bf16_hi(v[hh].w)};
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += x[e] * x[e];
        ss = group_sum<LPH>(ss);
        const float w = cos ? 1.0f / fmaxf(sqrtf(ss), 1e-12f) : 1.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] += x[e] * w;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[qi][piece * 8 + e] = live ? f[e] / (float)r : 0.f;
  }
  __syncthreads();
  const int rr = lane >> 4, n = lane & 15;
#pragma unroll
  for (int sw = 0; sw < NS / WAVES; ++sw) {
    const int s = sw * WAVES + wave;
    uint32_t w[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      float h0, l0, h1, l1;
      split_bf16(qf[n >> 1][32 * s + 8 * rr + 2 * jj], h0, l0);
      split_bf16(qf[n >> 1][32 * s + 8 * rr + 2 * jj + 1], h1, l1);
      w[jj] = (n & 1) ? pack_bf16(l0, l1) : pack_bf16(h0, h1);
    }
    qop[(((long long)g * n_qtiles + qt) * NS + s) * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Appends the buffers of the merge stage to a finished plan: the first-level winners of a two-level
// merge (very many lists) and the per-token winner keys of the token-pooling pass.
static void add_token_pool(const Dims& dm, int BM, int k, ScorePlan* p) {
  p->merge_lpp = 64;
  p->merge_parts = ((long long)p->n_splits * k > 16384) ? (p->n_splits + p->merge_lpp - 1) / p->merge_lpp : 1;
  p->off_part = p->ws_bytes;
  if (p->merge_parts > 1)
    p->ws_bytes += round_up256((size_t)p->n_sel * BM * p->merge_parts * k * sizeof(unsigned long long));
  p->off_tok = p->ws_bytes;
  if (dm.token_pool)
    p->ws_bytes += round_up256((size_t)BM * p->n_sel * k * sizeof(unsigned long long));
}

// All-heads scan: one pass of up to 32 queries (more take the wide kernel) over segments of the bank; the score matrix
// of one segment stays under 24 MB, which bounds the workspace and keeps the matrix in the cache behind the L2s between
// the scan that writes it and the selection that reads it.  Rows beyond 32768 documents are selected from in parts (one
// workgroup each) whose lists the merge kernel combines; up to there one workgroup per row, without the merge launch,
// is the faster way.  The lists of very long banks (more than kListsBytes: 16 queries, k = 32, from 50 million documents
// on) go through their buffer in windows of whole segments, each merged to one list per query when it is full: with a
// matrix of 20 MB the workspace then stays within the built-in scratch for any bank that fits the card.
static void plan_all_heads(const Dims& dm, int BM, int k, ScorePlan* p) {
  constexpr long long kListsBytes = (long long)6 << 20;
  p->mode = 2;
  p->tiles_per_wave = 0;
  p->exchange = p->it_publish = p->it_adopt = 0;
  p->off_gmax = 0;
  p->n_pass = 1;
  p->q_per_pass = BM <= 8 ? 8 : (BM <= 16 ? 16 : 32);
  // five segments or more: parts of 32768, which sixteen waves hold in registers, a quarter of the lists (32 queries, 4
  // million documents, k = 64: 727 -> 619 us); fewer: the short ones are 1 to 3 % faster (24 queries, 40000 documents: 124, 127)
  const bool many = (long long)dm.N * 4 * p->q_per_pass >= 5 * ((long long)24 << 20);
  p->part_docs = dm.N <= 4 * kRowPart ? dm.N : (many ? 4 * kRowPart : kRowPart);
  p->n_splits = (int)(((long long)dm.N + p->part_docs - 1) / p->part_docs);  // parts of a row = lists per query
  const long long lists = kListsBytes / ((long long)BM * k * 8);             // ... that the buffer holds (384 or more)
  const bool windows = p->n_splits > lists;
  const long long mat_bytes = (long long)(windows ? 20 : 24) << 20;
  long long seg = mat_bytes / (4 * p->q_per_pass) / p->part_docs * p->part_docs;
  if (seg > dm.N || dm.N <= 4 * kRowPart) seg = dm.N;
  p->seg_docs = (int)seg;
  const int seg_parts = (p->seg_docs + p->part_docs - 1) / p->part_docs;
  p->window_parts = windows ? (int)(lists / seg_parts * seg_parts) : p->n_splits;
  p->n_windows = (p->n_splits + p->window_parts - 1) / p->window_parts;
  size_t end = p->n_splits > 1 ? round_up256((size_t)BM * p->window_parts * k * sizeof(unsigned long long)) : 0;
  p->off_windows = end;
  if (windows) end += round_up256((size_t)BM * p->n_windows * k * sizeof(unsigned long long));
  p->n_qtiles = p->q_per_pass / 8;
  p->off_qop = end;
  end += round_up256((size_t)dm.Hkv * p->n_qtiles * (dm.d / 32) * 64 * 16);
  p->off_mat = end;
  end += round_up256((size_t)p->q_per_pass * p->seg_docs * sizeof(float));
  p->ws_bytes = end;
}

static ScorePlan plan_score_least(const Dims& dm, int BM, int k, bool two_passes = false) {
  ScorePlan p;
  p.nan_docs = 0;
  // one selection per KV group, or (literal Eq. 2 head mean, more than one group) one for all heads
  p.all_heads = (dm.scope_all && dm.Hkv > 1) ? 1 : 0;
  p.n_sel = dm.scope_all ? 1 : dm.Hkv;
  p.use_wide = wide_path_applies(dm, BM) ? 1 : 0;
  p.use_gemm = !p.use_wide && (two_passes || gemm_path_applies(dm, BM, k)) ? 1 : 0;
  if (p.use_wide) {
    p.wide = plan_score_wide(dm, BM, k);
    p.n_splits = 1;
    p.ws_bytes = p.wide.ws_bytes;
    add_token_pool(dm, BM, k, &p);
    return p;
  }
  if (p.use_gemm) {
    p.gemm = plan_score_gemm(dm, BM, k);
    p.n_splits = p.gemm.n_splits;
    p.q_per_pass = BM;
    p.n_pass = 1;
    p.exchange = 0;
    p.mode = 0;
    p.tiles_per_wave = 0;
    p.off_mat = 0;
    p.it_publish = p.it_adopt = 0;
    p.off_gmax = 0;
    p.off_qop = 0;
    p.n_qtiles = 0;
    p.ws_bytes = p.gemm.ws_bytes;
    add_token_pool(dm, BM, k, &p);
    return p;
  }
  if (p.all_heads) {
    plan_all_heads(dm, BM, k, &p);
    const int parts = p.n_splits;
    if (p.n_windows > 1) p.n_splits = p.n_windows;  // what the last merge combines
    add_token_pool(dm, BM, k, &p);
    p.n_splits = parts;
    return p;
  }
  p.q_per_pass = BM <= 8 ? 8 : ((BM <= 16 || k > 24) ? 16 : 32);
  p.n_pass = (BM + p.q_per_pass - 1) / p.q_per_pass;
  long long ns = 2048 / dm.Hkv;  // ~8 waves per CU on 256 CUs
  if (ns < 1) ns = 1;
  // streams of at least kPrefetch tiles; with 32 queries per pass the lists (64 entries each) must
  // also hold every document of the stream without pruning, so streams stay short there
  const long long min_len = kPrefetch;
  const long long by_tiles = (dm.tiles + min_len - 1) / min_len;
  if (ns > by_tiles) ns = by_tiles;
  if (ns > 1024) ns = 1024;
  if (ns < 1) ns = 1;
  const long long tiles_per_split = (dm.tiles + ns - 1) / ns;
  p.n_splits = (int)((dm.tiles + tiles_per_split - 1) / tiles_per_split);
  const size_t list_bytes = round_up256((size_t)p.n_sel * BM * p.n_splits * k * sizeof(unsigned long long));
  // threshold exchange between waves: worth it (and sound) only for long streams with >= k waves per head
  const long long n_it_min = dm.tiles / p.n_splits;
  // Short streams: nothing to filter.  MODE 2 (score matrix + row top-k) when its fp32 rows fit the
  // lists' LDS and the matrix stays small; else MODE 1 (dense lists) when the lists hold the stream.
  p.mode = 0;
  p.tiles_per_wave = 0;
  {
    const long long dpt = 16 / dm.C;
    const long long n_it_max = (dm.tiles + p.n_splits - 1) / p.n_splits;
    const long long cap = kListBytes / (8 * p.q_per_pass), capf = kListBytes / (4 * p.q_per_pass);
    const size_t mat_bytes = (size_t)dm.Hkv * BM * dm.N * sizeof(float);
    const long long L = n_it_max < kPrefetch ? kPrefetch : n_it_max;
    if (L * dpt <= capf && L <= 64 && mat_bytes <= ((size_t)256 << 20)) {
      p.mode = 2;
      p.tiles_per_wave = (int)L;
      p.n_splits = (int)((dm.tiles + L - 1) / L);
    } else if (n_it_max * dpt <= cap) {
      p.mode = 1;
    }
  }
  p.exchange = (p.mode == 0 && n_it_min >= 64 && p.n_splits >= k && p.n_splits <= 256) ? 1 : 0;
  // exchange events sit at the head of a group of kPrefetch iterations
  p.it_publish = (int)(n_it_min / 12) / kPrefetch * kPrefetch;
  p.it_adopt = p.it_publish + 3 * kPrefetch;
  p.off_gmax = list_bytes;
  p.off_qop = list_bytes + (p.exchange ? round_up256((size_t)dm.Hkv * BM * p.n_splits * sizeof(float)) : 0);
  p.n_qtiles = p.n_pass * (p.q_per_pass / 8);
  p.ws_bytes = p.off_qop + round_up256((size_t)dm.Hkv * p.n_qtiles * (dm.d / 32) * 64 * 16);
  p.off_mat = p.ws_bytes;
  if (p.mode == 2) p.ws_bytes += round_up256((size_t)dm.Hkv * BM * dm.N * sizeof(float));
  add_token_pool(dm, BM, k, &p);
  return p;
}

ScorePlan plan_score(const Dims& dm, int BM, int k, size_t workspace_bytes) {
  ScorePlan p = plan_score_least(dm, BM, k);
  p.ws_best = p.ws_bytes;
  if (!p.use_wide && !p.use_gemm && gemm_path_of_two_passes(dm, BM, k)) {
    ScorePlan g = plan_score_least(dm, BM, k, true);
    if (g.ws_bytes <= p.ws_bytes) {  // (in the workspace that the scan asks for)
      g.ws_bytes = g.ws_best = p.ws_bytes;
      g.nan_docs = p.mode == 2 ? 1 : 0;
      return g;
    }
  }
  if (p.use_wide && p.wide.list_bytes > 0) {
    // (asked for only where the built-in scratch, if it serves the call, still does)
    const size_t with = p.ws_bytes + p.wide.list_bytes;
    if (with <= kNoAllocScratchBytes || p.ws_bytes > kNoAllocScratchBytes) {
      p.ws_best = with;
      if (workspace_bytes == 0 || workspace_bytes >= with) p.wide.off_list = p.ws_bytes;
    }
  }
  return p;
}

int launch_score(const Dims& dm, const ScorePlan& pl, const void* q_route, int B, int M, const void* KR,
                 const float* inv_norm, int k, int32_t* out_idx, float* out_score, void* ws,
                 hipStream_t st) {
  const int BM = B * M;
  // with token pooling the per-token winners go to the workspace as keys and are pooled at the end
  unsigned long long* tok_keys = dm.token_pool ? (unsigned long long*)((char*)ws + pl.off_tok) : nullptr;
  auto pool_tokens = [&]() -> int {
    if (!dm.token_pool) return MSA_OK;
    hipLaunchKernelGGL(pool_tokens_kernel, dim3(B * pl.n_sel), dim3(kPoolThreads), 0, st,
                       (const unsigned long long*)tok_keys, out_idx, out_score, M, pl.n_sel, k);
    return hipGetLastError() == hipSuccess ? MSA_OK : MSA_ERR_HIP;
  };
  // combine the per-split lists of every (query, selection): one level, or two for very many lists
  const int* gate = nullptr;  // scoring GEMM with its one-pass filter: the token blocks whose lists are to be merged
  const int gate_tokens = pl.use_gemm ? (pl.gemm.tokens_per_wg > 0 ? pl.gemm.tokens_per_wg : 1) : 1;
  const int gate_blocks = pl.use_gemm ? pl.gemm.n_qblocks : 0;
  auto merge = [&](const unsigned long long* lists, int n_lists) -> int {
    if (pl.merge_parts > 1) {
      unsigned long long* part_keys = (unsigned long long*)((char*)ws + pl.off_part);
      hipLaunchKernelGGL(score_merge_kernel, dim3(BM * pl.n_sel * pl.merge_parts), dim3(256), 0, st, lists,
                         (int32_t*)nullptr, (float*)nullptr, part_keys, BM, pl.n_sel, n_lists, k,
                         pl.merge_lpp, pl.merge_parts, 0, pl.merge_parts, gate, gate_tokens, gate_blocks, pl.nan_docs);
      if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
      lists = part_keys;
      n_lists = pl.merge_parts;
    }
    hipLaunchKernelGGL(score_merge_kernel, dim3(BM * pl.n_sel), dim3(256), 0, st, lists, out_idx, out_score,
                       tok_keys, BM, pl.n_sel, n_lists, k, n_lists, 1, 0, 1, gate, gate_tokens, gate_blocks, pl.nan_docs);
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
    return pool_tokens();
  };
  if (pl.use_wide) {
    const WidePoolPlan pp = plan_score_wide_pool(dm, pl.wide, B, M, k);
    if (pp.applies) return launch_score_wide_pool(dm, pp, q_route, B, M, KR, inv_norm, k, ws, st, out_idx, out_score);
    const int rc = launch_score_wide(dm, pl.wide, q_route, BM, KR, inv_norm, k, ws, st, out_idx, out_score, tok_keys);
    if (rc != MSA_OK) return rc;
    return pool_tokens();
  }
  if (pl.use_gemm) {
    const int rc = launch_score_gemm_scan(dm, pl.gemm, q_route, BM, KR, inv_norm, k, ws, st, out_idx, out_score,
                                          tok_keys, &gate);
    if (rc != MSA_OK) return rc;
    return merge((const unsigned long long*)((const char*)ws + pl.gemm.off_lists), pl.gemm.n_splits);
  }
  ScoreArgs a;
  a.KR = (const uint16_t*)KR;
  a.inv_norm = dm.cos ? inv_norm : nullptr;
  a.ws = (unsigned long long*)ws;
  a.BM = BM;
  a.Hq = dm.Hq;
  a.Hkv = dm.Hkv;
  a.r = dm.r;
  a.N = dm.N;
  a.C = dm.C;
  a.cos = dm.cos;
  a.tiles = dm.tiles;
  a.n_splits = pl.n_splits;
  a.k = k;
  a.gmax = pl.exchange ? (float*)((char*)ws + pl.off_gmax) : nullptr;
  a.it_publish = pl.it_publish;
  a.it_adopt = pl.it_adopt;
  a.qop = (const uint4*)((char*)ws + pl.off_qop);
  a.mat = (pl.mode == 2) ? (float*)((char*)ws + pl.off_mat) : nullptr;
  a.tiles_per_wave = pl.tiles_per_wave;
  a.n_qtiles = pl.n_qtiles;
  a.q_route = (const uint16_t*)q_route;
  const bool fold_in_scan = pl.all_heads ? all_heads_folds(dm, pl, BM) : !pl.exchange;
  if (!fold_in_scan) {
    const long long n_gmax = pl.exchange ? (long long)dm.Hkv * BM * pl.n_splits : 0;
    const unsigned blocks = (unsigned)(pl.n_qtiles * dm.Hkv);
    if (dm.d == 128)
      hipLaunchKernelGGL(prep_scan_operands_kernel<128>, dim3(blocks), dim3(128), 0, st,
                         (const uint16_t*)q_route, (uint4*)((char*)ws + pl.off_qop), BM, dm.Hq, dm.Hkv,
                         dm.r, dm.cos, pl.n_qtiles, a.gmax, n_gmax);
    else
      hipLaunchKernelGGL(prep_scan_operands_kernel<64>, dim3(blocks), dim3(64), 0, st,
                         (const uint16_t*)q_route, (uint4*)((char*)ws + pl.off_qop), BM, dm.Hq, dm.Hkv,
                         dm.r, dm.cos, pl.n_qtiles, a.gmax, n_gmax);
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
  }
  const bool cold = pl.n_pass == 1 && !(pl.all_heads && dm.C <= 2 && BM > 8);
  const bool stream_index = stream_index_of(dm, cold);
  RowsArgs ra;
  ra.mat = (const float*)((char*)ws + pl.off_mat);
  ra.BM = BM;
  ra.n_sel = pl.n_sel;
  ra.k = k;
  ra.out_idx = out_idx;
  ra.out_score = out_score;
  ra.out_key = tok_keys;
  if (pl.all_heads) {
    ScanAllArgs sa;
    sa.qop = (const uint4*)((char*)ws + pl.off_qop);
    sa.q_route = (const uint16_t*)q_route;
    sa.BM = BM;
    sa.Hq = dm.Hq;
    sa.r = dm.r;
    sa.KR = (const uint16_t*)KR;
    sa.inv_norm = a.inv_norm;
    sa.mat = (float*)((char*)ws + pl.off_mat);
    sa.mat_stride = pl.seg_docs;
    sa.n_qtiles = pl.n_qtiles;
    sa.C = dm.C;
    sa.tiles = dm.tiles;
    ra.stride = pl.seg_docs;
    ra.part_docs = pl.part_docs;
    ra.part_keys = pl.n_splits > 1 ? (unsigned long long*)ws : nullptr;
    unsigned long long* const window_keys = (unsigned long long*)((char*)ws + pl.off_windows);
    const int nqt = pl.q_per_pass / 8;  // 1, 2 or 4
    profile_mark(dm, false, st);
    for (long long seg0 = 0; seg0 < dm.N; seg0 += pl.seg_docs) {
      const int doc0 = (int)seg0;
      const int n_docs = dm.N - doc0 < pl.seg_docs ? dm.N - doc0 : pl.seg_docs;
      sa.nq = BM;
      sa.tile0 = (long long)doc0 * dm.C / 16;  // doc0 is a multiple of 8192 (or 0)
      sa.seg_docs = n_docs;
      sa.seg_tiles = ((long long)n_docs * dm.C + 15) / 16;
      sa.ushift = scan_all_ushift(sa.seg_tiles, dm.C);
      const long long units = (sa.seg_tiles + (1 << sa.ushift) - 1) >> sa.ushift;
      const long long wgs = (units + kAllWaves - 1) / kAllWaves;
      dim3 grid((unsigned)(wgs < kAllGroups ? wgs : kAllGroups)), block(64 * kAllWaves);
#define MSA_SCAN_ALL(DD, HH, QQ) \
do { \
  constexpr bool FF = HH * QQ <= kAllFoldTiles; /* can fold */ \
  if (FF && !fold_in_scan) hipLaunchKernelGGL((score_scan_all_kernel<DD, HH, QQ, false, false>), grid, block, 0, st, sa); \
  else if (stream_index) hipLaunchKernelGGL((score_scan_all_kernel<DD, HH, QQ, true, FF>), grid, block, 0, st, sa); \
  else hipLaunchKernelGGL((score_scan_all_kernel<DD, HH, QQ, false, FF>), grid, block, 0, st, sa); \
} while (0)
#define MSA_SCAN_ALL_Q(DD, HH) \
do { \
  if (nqt == 1) MSA_SCAN_ALL(DD, HH, 1); else if (nqt == 2) MSA_SCAN_ALL(DD, HH, 2); else MSA_SCAN_ALL(DD, HH, 4); \
} while (0)
      if (dm.d == 128) {
        if (dm.Hkv == 2) MSA_SCAN_ALL_Q(128, 2); else if (dm.Hkv == 4) MSA_SCAN_ALL_Q(128, 4); else MSA_SCAN_ALL_Q(128, 8);
      } else {
        if (dm.Hkv == 2) MSA_SCAN_ALL_Q(64, 2); else if (dm.Hkv == 4) MSA_SCAN_ALL_Q(64, 4); else MSA_SCAN_ALL_Q(64, 8);
      }
#undef MSA_SCAN_ALL_Q
#undef MSA_SCAN_ALL
      if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
      if (doc0 + n_docs == dm.N) profile_mark(dm, true, st);
      ra.n_docs = n_docs;
      ra.doc0 = doc0;
      ra.parts = (n_docs + pl.part_docs - 1) / pl.part_docs;
      const int part = doc0 / pl.part_docs, window = part / pl.window_parts;
      const int last = pl.n_splits - window * pl.window_parts;  // parts from this window's first to the bank's last
      ra.parts_total = last < pl.window_parts ? last : pl.window_parts;
      ra.part0 = part - window * pl.window_parts;
      launch_topk_rows(ra, st);
      if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
      if (pl.n_windows > 1 && ra.part0 + ra.parts == ra.parts_total) {
        hipLaunchKernelGGL(score_merge_kernel, dim3(BM), dim3(256), 0, st, (const unsigned long long*)ws,
                           (int32_t*)nullptr, (float*)nullptr, window_keys, BM, 1, ra.parts_total, k, ra.parts_total, 1,
                           window, pl.n_windows, (const int*)nullptr, 1, 0, 0);
        if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
      }
    }
    if (pl.n_windows > 1) return merge(window_keys, pl.n_windows);
    if (pl.n_splits > 1) return merge((const unsigned long long*)ws, pl.n_splits);
    return pool_tokens();
  }
  dim3 grid((pl.n_splits + kScanWaves - 1) / kScanWaves, dm.Hkv), block(64 * kScanWaves);
  profile_mark(dm, false, st);
  for (int pass = 0; pass < pl.n_pass; ++pass) {
    a.q0 = pass * pl.q_per_pass;
    const int nqt = pl.q_per_pass / 8;  // 1, 2 or 4
    const bool late = late_requests(pl, BM);
#define MSA_SCAN_2(DD, QQ, CC, SS) \
  do { \
    if (late) hipLaunchKernelGGL((score_scan_kernel<DD, QQ, CC, 2, true, SS, true>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((score_scan_kernel<DD, QQ, CC, 2, true, SS, QQ != 4>), grid, block, 0, st, a); \
  } while (0)
#define MSA_SCAN(DD, QQ, CC) \
  do { \
    if (pl.mode == 2 && stream_index) MSA_SCAN_2(DD, QQ, CC, true); \
    else if (pl.mode == 2) MSA_SCAN_2(DD, QQ, CC, false); \
    else if (pl.mode == 1) hipLaunchKernelGGL((score_scan_kernel<DD, QQ, CC, 1, true, false, true>), grid, block, 0, st, a); \
    else if (fold_in_scan) hipLaunchKernelGGL((score_scan_kernel<DD, QQ, CC, 0, true, true, true>), grid, block, 0, st, a); \
    else hipLaunchKernelGGL((score_scan_kernel<DD, QQ, CC, 0, false, true, true>), grid, block, 0, st, a); \
  } while (0)
    if (dm.d == 128) {
      if (dm.cos) {
        if (nqt == 1) MSA_SCAN(128, 1, true); else if (nqt == 2) MSA_SCAN(128, 2, true); else MSA_SCAN(128, 4, true);
      } else {
        if (nqt == 1) MSA_SCAN(128, 1, false); else if (nqt == 2) MSA_SCAN(128, 2, false); else MSA_SCAN(128, 4, false);
      }
    } else {
      if (dm.cos) {
        if (nqt == 1) MSA_SCAN(64, 1, true); else if (nqt == 2) MSA_SCAN(64, 2, true); else MSA_SCAN(64, 4, true);
      } else {
        if (nqt == 1) MSA_SCAN(64, 1, false); else if (nqt == 2) MSA_SCAN(64, 2, false); else MSA_SCAN(64, 4, false);
      }
    }
#undef MSA_SCAN
#undef MSA_SCAN_2
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
  }
  profile_mark(dm, true, st);
  if (pl.mode == 2) {
    ra.stride = dm.N;
    ra.n_docs = ra.part_docs = dm.N;
    ra.doc0 = ra.part0 = 0;
    ra.parts = ra.parts_total = 1;
    ra.part_keys = nullptr;
    launch_topk_rows(ra, st);
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
    return pool_tokens();
  }
  return merge((const unsigned long long*)ws, pl.n_splits);
}

}  // namespace msa
