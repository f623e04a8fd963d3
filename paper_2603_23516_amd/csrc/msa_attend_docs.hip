// msa_sparse_attend for MANY query tokens with selections of their OWN: the selected documents are taken
// document by document instead of token by token.
//
// The tokens of a prompt have a topic in common, so a document is selected by several of them (and with many
// tokens over few documents by many whatever the topic is).  The decode kernel reads it once per token: 512
// tokens of 8 documents of 512 rows gather 8.6 GB of which 3.4 GB are distinct.  Here
//   group_kernel         sorts the (token, slot) pairs of every selection list by document (counting sort; one
//                        workgroup per list) into ITEMS of up to 16 / r tokens of one document, and, in its
//                        other workgroups, rotates and scales the queries once, bf16 (hi, lo) in the order of
//                        the matrix operand.  Where the pairs hardly share a document an item is a CHAIN instead, up
//                        to four documents of one token.
//   attend_docs_kernel   one WAVE per item (or per part of an item's rows where there are few): the columns of
//                        the score product are the item's (token, head) pairs, so one pass over the document's
//                        rows serves all of them.  A wave walks its items as one stream of 32-row steps; keys and
//                        values of the next item are in flight while the last steps of this one are worked on.  At the
//                        end of an item they are awaited together with the next queries, the one drain per item.
//                        No barrier after the prologue.
// An item leaves one partial (max, sum, output) per token, part and head; attend_merge2_kernel combines them with
// those of the local context (tiled kernel).  What a column holds does not depend on the columns beside it, so the
// order in which the sort places the pairs changes no bit of the result; a token's chains are its slots in order.
//
// Bound: memory (every document and KV head once, then again from the L2 for every 16 / r tokens beyond the first), two
// waves per SIMD with 24 KiB of requests in flight each.  One item per WAVE: four waves on one item would have to merge
// their outputs through LDS once per 256 KiB read.  512 tokens of 8 of 4096 documents (512 rows, 8 heads of 128), half of
// them among 32 of a topic: 1067 us token by token, 710 (sort 12, documents 650, local context 26, merge 28); selections
// drawn at random 1332, 983; 300 of 16 of 200 documents 1210, 315; 1024 of 32 of 500 9.0 ms, 1.96.
// Partials are written between the reads, and that costs more than their bytes: 67 MB of them among 8.6 GB 92 us, whichever
// way they are stored, and 45 for the instructions.  So with no document shared at all (the same sizes) items of one document
// took 1480 us, chains 1372, token by token 1367.  Documents in parts cost more than they spread (a part pays for the chain
// item - pairs - queries): 64 tokens of 4 of 8192 86 us whole, 94 in halves, so parts are for very few items only.
//
// Arithmetic per step is the decode kernel's (msa_attend.hip: keys rotated in fp32 by a recurrence, rounded to
// bf16; queries and weights as bf16 hi and lo parts; online softmax) with hi and lo as two products into one
// accumulator instead of neighbouring columns.
#include "msa_attend.h"

namespace msa {

constexpr int kGroupThreads = 1024;
constexpr int kLdsDocs = 12288;     // 147456 bytes
constexpr int kSeenDocs = 1 << 19;  // bits in LDS
constexpr int kMaxChain = 4;        // documents of a chain (entries per item: 1 << 2 at least)
constexpr int kPairs = 4;  // (token, slot) pairs of a thread at a time

// ---- sort by document, rotated queries ----------------------------------------------------------------------
// LDS: a document's counters fit there (N <= kLdsDocs).  WHOLE: the call is one window (a form of its own: with the code for
// several in it 512 tokens of 8 of 4096 documents take 759 us, else 752).
template <int D, bool LDS, bool WHOLE>
__global__ __launch_bounds__(kGroupThreads) void group_kernel(AttendArgs a, DocsArgs da, RopeTheta th) {
  constexpr int HALF = D / 2;
  const int tid = threadIdx.x;
  auto selection = [&](int t, int s) {  // of a token of the call: where list s begins in idx
    return ((long long)(a.idx_rows_per_b == 1 ? t / a.M : t) * a.idx_sel + s) * a.k;
  };
  if ((int)blockIdx.x >= a.idx_sel) {  // ---- queries of up to four tokens
    __shared__ float2 cs[4][HALF];
    const int t0 = ((int)blockIdx.x - a.idx_sel) * 4;
    if (tid < 4 * HALF) {
      const int t = t0 + tid / HALF;
      cs[tid / HALF][tid % HALF] = cis_pos(t < da.n_tok ? a.q_pos[da.tok0 + t] : 0, th.th[tid % HALF]);
    }
    __syncthreads();
    // empty partials where a slot holds no document: the maximum alone, the merge does not look at their outputs
    for (int x = tid; x < 4 * a.Hq * a.k; x += kGroupThreads) {
      const int slot = x % a.k, row = x / a.k, t = t0 + row / a.Hq;
      if (t >= da.n_tok) break;
      const int d = a.idx[selection(da.tok0 + t, a.idx_sel == 1 ? 0 : row % a.Hq / a.r) + slot];
      if (d >= 0 && d < a.N) continue;
      float2* ml = da.part_ml + ((long long)t0 * a.Hq * a.k + x) * da.parts;
      for (int p = 0; p < da.parts; ++p) ml[p] = make_float2(-INFINITY, 0.f);
    }
    constexpr int PPH = HALF / 8;  // 16-byte pieces per half row
    for (int e = tid; e < 4 * a.Hq * PPH; e += kGroupThreads) {
      const int pc = e % PPH, head = e / PPH % a.Hq, t4 = e / PPH / a.Hq;
      const int t = t0 + t4;
      if (t >= da.n_tok) break;
      const long long row = (long long)t * a.Hq + head;
      const uint16_t* qp = a.q + ((long long)da.tok0 * a.Hq + row) * D + pc * 8;
      const uint4 r1 = *reinterpret_cast<const uint4*>(qp);
      const uint4 r2 = *reinterpret_cast<const uint4*>(qp + HALF);
      const uint32_t w1[4] = {r1.x, r1.y, r1.z, r1.w}, w2[4] = {r2.x, r2.y, r2.z, r2.w};
      uint32_t h1[4], l1[4], h2[4], l2[4];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        float y1[2], y2[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float x1 = i ? bf16_hi(w1[jj]) : bf16_lo(w1[jj]);
          const float x2 = i ? bf16_hi(w2[jj]) : bf16_lo(w2[jj]);
          const float2 c = cs[t4][8 * pc + 2 * jj + i];
          y1[i] = (x1 * c.x - x2 * c.y) * a.qscale;
          y2[i] = (x2 * c.x + x1 * c.y) * a.qscale;
        }
        split_pack_bf16(y1[0], y1[1], h1[jj], l1[jj]);
        split_pack_bf16(y2[0], y2[1], h2[jj], l2[jj]);
      }
      uint4* o = da.qrot + row * (D / 4);  // [piece][hi, lo]
      o[2 * pc] = make_uint4(h1[0], h1[1], h1[2], h1[3]);
      o[2 * pc + 1] = make_uint4(l1[0], l1[1], l1[2], l1[3]);
      o[2 * (pc + PPH)] = make_uint4(h2[0], h2[1], h2[2], h2[3]);
      o[2 * (pc + PPH) + 1] = make_uint4(l2[0], l2[1], l2[2], l2[3]);
    }
    return;
  }
  // ---- one list of selections: pair e = (token e >> kshift, slot e & (2^kshift - 1)).  A phase's results are in LDS, or in
  // memory that this workgroup alone touches, at workgroup scope: the atomics and the barrier order them for its waves, and
  // nothing has to reach the other XCDs before the end of the launch.  (Device scope, i.e. memory: 40 us for 4096 pairs per
  // list.)  A thread takes up to kPairs pairs at a time, their loads together.
  __shared__ unsigned long long base_s[LDS ? kLdsDocs : 1];
  __shared__ int cnt_s[LDS ? kLdsDocs : 1];
  __shared__ int n_entries_s, n_items_s, n_valid_s, n_docs_s;
  __shared__ unsigned seen_s[LDS || WHOLE ? 1 : kSeenDocs / 32];
  const int s = blockIdx.x, lane = tid & 63;
  const int sh = da.kshift, E = da.n_tok << sh, T = da.tile_tok;
  int* const cnt = LDS ? cnt_s : da.cnt + (long long)s * a.N;
  unsigned long long* const base = LDS ? base_s : da.base + (long long)s * a.N;
  int* const rank = da.rank + (long long)s * (da.n_tok << sh);
  int* const entries = da.entries + (long long)s * da.cap;
  int4* const items = da.items + (long long)s * da.cap;
  auto phase = [&]() {  // stores and atomics of the phase are complete for everyone
    wait_stores_done();
    __syncthreads();
  };
  if (tid == 0) n_entries_s = n_items_s = n_valid_s = n_docs_s = 0;
  int d[kPairs], rk[kPairs];  // document (-1: past the end, a pad, or no document of the bank), place among its pairs
  auto docs_at = [&](int e0, int tok_from, int pairs_to) {  // (no branch around a load)
    int x[kPairs];
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      const int e = e0 + i * kGroupThreads + tid, slot = e & ((1 << sh) - 1);
      const bool ok = e < pairs_to && slot < a.k;
      x[i] = a.idx[selection(tok_from + (ok ? e >> sh : 0), s) + (ok ? slot : 0)];
      d[i] = ok ? 0 : -1;
    }
#pragma unroll
    for (int i = 0; i < kPairs; ++i) d[i] = d[i] == 0 && x[i] >= 0 && x[i] < a.N ? x[i] : -1;
  };
  auto add = [](auto* p, auto v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto read = [](auto* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  const unsigned long long below = (1ull << lane) - 1ull;
  int have_from = -1, have_to = 0;  // the tokens whose documents and places are in registers
  // the places of the pairs of [tok_from, tok_to) among those of their documents; `decide` counts pairs and documents
  auto count_pairs = [&](int tok_from, int tok_to, bool decide) {
    const int to = (tok_to - tok_from) << sh;
    for (int e0 = 0; e0 < to; e0 += kPairs * kGroupThreads) {
      docs_at(e0, tok_from, to);
#pragma unroll
      for (int i = 0; i < kPairs; ++i)
        if (d[i] >= 0) __hip_atomic_store(cnt + d[i], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    phase();
    const bool keep = to <= kPairs * kGroupThreads;
    int n_valid = 0, n_docs = 0;
    for (int e0 = 0; e0 < to; e0 += kPairs * kGroupThreads) {
      if (!keep) docs_at(e0, tok_from, to);
#pragma unroll
      for (int i = 0; i < kPairs; ++i) rk[i] = d[i] >= 0 ? add(cnt + d[i], 1) : 1;
      if (!keep && to == E) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i)
          if (d[i] >= 0) rank[e0 + i * kGroupThreads + tid] = rk[i];
      }
      if (decide) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
          n_valid += __popcll(__ballot(d[i] >= 0));
          n_docs += __popcll(__ballot(d[i] >= 0 && rk[i] == 0));
        }
      }
    }
    if (decide && lane == 0) {
      atomicAdd(&n_valid_s, n_valid);
      atomicAdd(&n_docs_s, n_docs);
    }
    phase();
    have_from = keep ? tok_from : -1;
    have_to = tok_to;
  };
  // Where hardly a document has a second token the pairs are taken as they come: chains of up to `chain` documents of one
  // token, one partial each.  Decided over all tokens of the call, so that its windows change no bit: where there are several
  // by a bit per document in LDS (counting all tokens in every window took 134 us for 2048 tokens of 8 of 32768, 85 without).
  const int t1 = da.tok0 + da.n_tok;
  if (WHOLE || a.N > (LDS ? 32 * kLdsDocs : kSeenDocs)) {
    count_pairs(0, da.n_all, true);
  } else {
    unsigned* const seen = LDS ? reinterpret_cast<unsigned*>(cnt_s) : seen_s;
    for (int i = tid; i <= (a.N - 1) / 32; i += kGroupThreads) seen[i] = 0u;
    __syncthreads();
    const int to = da.n_all << sh;
    int n_valid = 0, n_docs = 0;
    for (int e0 = 0; e0 < to; e0 += kPairs * kGroupThreads) {
      docs_at(e0, 0, to);
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        const unsigned bit = 1u << (d[i] & 31);
        const bool first = d[i] >= 0 && (atomicOr(seen + (d[i] >> 5), bit) & bit) == 0;
        n_valid += __popcll(__ballot(d[i] >= 0));
        n_docs += __popcll(__ballot(first));
      }
    }
    if (lane == 0) {
      atomicAdd(&n_valid_s, n_valid);
      atomicAdd(&n_docs_s, n_docs);
    }
    __syncthreads();
  }
  const bool chains = 10ll * n_valid_s < 11ll * n_docs_s;
  if (!WHOLE && !chains) count_pairs(da.tok0, t1, false);
  const bool once = have_from == da.tok0 && have_to == t1;  // documents and ranks of all pairs stay in registers
  if (chains) {
    const unsigned long long mine = (sh == 6 ? ~0ull : (1ull << (1 << sh)) - 1ull) << (lane & ~((1 << sh) - 1) & 63);
    for (int e0 = 0; e0 < E; e0 += kPairs * kGroupThreads) {
      if (!once) docs_at(e0, da.tok0, E);
      unsigned long long valid[kPairs], lead[kPairs];
      int be = 0, bi = 0;
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        valid[i] = __ballot(d[i] >= 0);
        lead[i] = __ballot(d[i] >= 0 && __popcll(valid[i] & mine & below) % da.chain == 0);
        be += __popcll(valid[i]);
        bi += __popcll(lead[i]);
      }
      if (lane == 0) {
        be = atomicAdd(&n_entries_s, be);
        bi = atomicAdd(&n_items_s, bi);
      }
      be = __shfl(be, 0, 64);
      bi = __shfl(bi, 0, 64);
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        if (d[i] >= 0) {
          const int at = be + __popcll(valid[i] & below);
          entries[at] = d[i];
          if ((lead[i] >> lane) & 1) {
            const int before = __popcll(valid[i] & mine & below), left = __popcll(valid[i] & mine & ~below);
            const int t = (e0 + i * kGroupThreads + tid) >> sh;
            items[bi + __popcll(lead[i] & below)] =
                make_int4((t << 6) | before / da.chain, at, left < da.chain ? left : da.chain, left <= da.chain ? 3 : 2);
          }
        }
        be += __popcll(valid[i]);
        bi += __popcll(lead[i]);
      }
    }
    __syncthreads();
    if (tid == 0) {
      da.n_items[s] = n_items_s;
      da.n_items[a.idx_sel + s] = 1;
    }
    return;
  }
  // the first pair of a document reserves its places; a wave adds up its documents first
  for (int e0 = 0; e0 < E; e0 += kPairs * kGroupThreads) {
    if (!once) {
      docs_at(e0, da.tok0, E);
#pragma unroll
      for (int i = 0; i < kPairs; ++i) rk[i] = d[i] >= 0 ? rank[e0 + i * kGroupThreads + tid] : 1;
    }
    int c[kPairs], pc = 0, pt = 0;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) c[i] = rk[i] == 0 ? read(cnt + d[i]) : 0;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      pc += c[i];
      pt += (c[i] + T - 1) / T;
    }
    const int mine_c = pc, mine_t = pt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {  // inclusive sums over the lanes
      const int x = __shfl_up(pc, off, 64), y = __shfl_up(pt, off, 64);
      if (lane >= off) {
        pc += x;
        pt += y;
      }
    }
    int be = 0, bi = 0;
    if (lane == 63) {
      be = atomicAdd(&n_entries_s, pc);
      bi = atomicAdd(&n_items_s, pt);
    }
    be = __shfl(be, 63, 64) + pc - mine_c;
    bi = __shfl(bi, 63, 64) + pt - mine_t;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      if (c[i] == 0) continue;
      __hip_atomic_store(base + d[i], ((unsigned long long)(unsigned)bi << 32) | (unsigned)be, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_WORKGROUP);
      be += c[i];
      bi += (c[i] + T - 1) / T;
    }
  }
  phase();
  for (int e0 = 0; e0 < E; e0 += kPairs * kGroupThreads) {
    if (!once) {
      docs_at(e0, da.tok0, E);
#pragma unroll
      for (int i = 0; i < kPairs; ++i) rk[i] = d[i] >= 0 ? rank[e0 + i * kGroupThreads + tid] : 1;
    }
    unsigned long long b[kPairs];
    int c[kPairs];
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      b[i] = d[i] >= 0 ? read(base + d[i]) : 0ull;
      c[i] = d[i] >= 0 && rk[i] % T == 0 ? read(cnt + d[i]) : 0;
    }
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      if (d[i] < 0) continue;
      const int e = e0 + i * kGroupThreads + tid;
      const int at = (int)(unsigned)b[i] + rk[i];
      entries[at] = (e >> sh << 6) | (e & ((1 << sh) - 1));
      if (c[i] > 0) {
        const int left = c[i] - rk[i];
        items[(int)(b[i] >> 32) + rk[i] / T] = make_int4(d[i], at, left < T ? left : T, c[i] > T ? 0 : 1);
      }
    }
  }
  if (tid == 0) {
    da.n_items[s] = n_items_s;
    da.n_items[a.idx_sel + s] = 0;
  }
}

constexpr int kFetch = 32, kFetchPairs = 192;  // items looked up at a time, at most: 32 of up to four entries, 12 of sixteen

// ---- attention, document by document -------------------------------------------------------------------------
template <int D, bool ROT>  // ROT: raw bank keys, rotated here with positions 0..G-1; else used as stored
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attend_docs_kernel(AttendArgs a, DocsArgs da, RopeTheta th) {
  constexpr int NS = D / 32;          // contraction slices of the score product
  constexpr int HALF = D / 2;
  constexpr int NU = (NS / 2) * 8;    // rotation pairs per lane
  constexpr int NCB = D / 16;         // output row blocks
  constexpr int VBYTES = 32 * D * 2;  // the 32 value rows of a step in LDS
  constexpr int NVL = VBYTES / 1024;  // wave-wide 16-byte copies covering them
  constexpr int PPR = D / 8;          // 16-byte pieces per row

  __shared__ float2 base0[16][HALF];  // e^{i n theta_u}: positions 0..15
  __shared__ float2 step16[HALF];     // e^{i 16 theta_u}
  __shared__ float2 estart[kAttWaves][HALF];
  __shared__ double theta_s[HALF];
  __shared__ int4 desc[kAttWaves][kFetch];  // items to come, and their entries
  __shared__ int entry[kAttWaves][kFetchPairs];
  __shared__ __attribute__((aligned(16))) unsigned char stage[kAttWaves][2 * VBYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rr = lane >> 4;
  const int n = lane & 15;

  // rotation tables, as in the decode kernel
  if (ROT) {
    if (tid < 4 * HALF) {
      const int u = tid % HALF, n4 = tid / HALF;
      const float2 w = th.e1[u];
      const float2 w2 = cmul(w, w);
      const float2 w4 = cmul(w2, w2);
      float2 cur = make_float2(1.f, 0.f);
      for (int i = 0; i < n4; ++i) cur = cmul(cur, w4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        base0[4 * n4 + i][u] = cur;
        cur = cmul(cur, w);
      }
    }
    if (tid < HALF) {
      step16[tid] = th.e16[tid];
      theta_s[tid] = th.th[tid];
    }
    lds_barrier();
  }

  // ---- this wave's share of the items: [g][item][part] in one line, an eighth of it per XCD (workgroups go round the
  // XCDs in turn), so that the tiles of a document that many tokens selected meet in one L2
  auto items_upto = [&]() {  // lane g: items of the KV heads up to g
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    int upto = lane < a.Hkv ? da.n_items[a.idx_sel == 1 ? 0 : lane] : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int x = __builtin_amdgcn_ds_bpermute((lane - off) * 4, upto);  // (from the opaque number, see head_row)
      if (lane >= off) upto += x;
    }
    return upto;
  };
  const long long all = (long long)__builtin_amdgcn_readlane(items_upto(), 63) * da.parts;
  const int xcd = blockIdx.x & 7, per_xcd = gridDim.x >> 3;  // (the grid is a multiple of 8)
  const int lo = (int)(all * xcd >> 3), hi = (int)(all * (xcd + 1) >> 3);
  const int stride = per_xcd * kAttWaves;
  const int first_x = lo + (int)(blockIdx.x >> 3) * kAttWaves + wave;
  if (first_x >= hi) return;  // (no barrier below)

  // Descriptors of the next items of this wave: document and its rows, or a chain's token << 6 | number; tokens | part << 8 |
  // the token's last chain << 14 | nobody else reads its rows << 15 | KV head << 16; documents of a chain, or 0.  And their
  // entries: the (token, slot) of each of the item's tokens, or each of a chain's documents (the last one again past their
  // number).
  // In LDS: the stream below has no registers for them.
  // (r, T, the entries per item and the parts are powers of two: shifts, since a division's reciprocal would be kept across
  // the stream, spill, and be reloaded with everything in flight awaited)
  const int T = da.tile_tok, rshift = 31 - __clz(a.r), pshift = 31 - __clz(da.parts);
  const int eshift = T < kMaxChain ? 2 : 31 - __clz(T);
  const int n_fetch = (kFetchPairs >> eshift) < kFetch ? kFetchPairs >> eshift : kFetch;
  auto fetch_items = [&](int x0) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int x = x0 + ln * stride;
    const int upto = items_upto();
    const int xi = x >> pshift, part = x - (xi << pshift);
    int g = 0, before = 0;
    for (int i = 0; i < a.Hkv; ++i) {
      const int u = __builtin_amdgcn_readlane(upto, i);
      if (u <= xi) {
        g = i + 1;
        before = u;
      }
    }
    int first = 0, cnt = 0;
    if (x < hi && ln < n_fetch) {
      const int list = a.idx_sel == 1 ? 0 : g;
      const int4 it = da.items[(long long)list * da.cap + (xi - before)];
      const bool chain = it.w >= 2;
      int len = a.G;
      if (a.lens != nullptr && !chain) {
        len = a.lens[it.x];
        len = len < 1 ? 1 : (len > a.G ? a.G : len);
      }
      desc[wave][ln] = make_int4(it.x, len, (chain ? 1 : it.z) | (part << 8) | (it.w == 3 ? 0x4000 : 0) | (it.w != 0 ? 0x8000 : 0) | (g << 16),
                                 chain ? it.z : 0);
      first = list * da.cap + it.y;
      cnt = it.z;
    }
    for (int p0 = 0; p0 < n_fetch << eshift; p0 += 64) {
      const int p = p0 + ln, of = p >> eshift, i = p - (of << eshift);
      const int f = __shfl(first, of & 63, 64), c = __shfl(cnt, of & 63, 64);
      if (of < n_fetch && c > 0) entry[wave][p] = da.entries[f + (i < c ? i : c - 1)];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  // One step of the stream (wave-uniform).
  struct Step {
    long long off;  // element offset of its first row in K and V
    int rows;       // rows of its item from there on, 32 or more: a whole step (0: an empty part of a short document)
    int p_first;    // position of the first row
    int left;       // steps of its document after this one, + kGoesOn if others of the chain follow
    int what;       // the item
    int pair;       // token << 6 | slot of the partial of this lane's column
  };
  constexpr int kGoesOn = 1 << 30;
  int c_x = first_x, c_lane = 0;  // the cursor's item
  int c_doc = 0, c_docs = 0;      // ... and document of a chain
  auto open_rows = [&](Step& s, int doc, int len) {
    const int part = (s.what >> 8) & 0x3f, g = s.what >> 16;
    const int most = da.part_steps * 32;
    int p0 = part * most;
    int rows = len - p0;  // rows of the document from this part on
    rows = rows < most ? rows : most;
    if (rows <= 0) p0 = rows = 0;
    s.left = rows > 0 ? (rows - 1) >> 5 : 0;
    s.p_first = p0;
    s.rows = rows;
    s.off = (((long long)doc * a.Hkv + g) * a.G + p0) * D;
  };
  auto open_of_chain = [&](Step& s) {
    const int doc = __builtin_amdgcn_readfirstlane(entry[wave][(c_lane << eshift) + c_doc]);
    int len = a.G;
    if (a.lens != nullptr) {  // (a scalar load: a vector load would be awaited with everything in flight)
      len = ((const __attribute__((address_space(4))) int32_t*)a.lens)[doc];
      len = len < 1 ? 1 : (len > a.G ? a.G : len);
    }
    open_rows(s, doc, len);
    if (++c_doc < c_docs) s.left += kGoesOn;
  };
  auto open_item = [&](Step& s) {
    const int4 d = desc[wave][c_lane];
    const int x = __builtin_amdgcn_readfirstlane(d.x);
    s.what = __builtin_amdgcn_readfirstlane(d.z);
    c_docs = __builtin_amdgcn_readfirstlane(d.w);
    c_doc = 0;
    if (c_docs > 0) {
      s.pair = x;
      open_of_chain(s);
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      s.pair = entry[wave][(c_lane << eshift) + ((ln & 15) >> rshift)];  // (that is under T)
      open_rows(s, x, __builtin_amdgcn_readfirstlane(d.y));
    }
  };
  auto advance = [&](Step& s) -> bool {  // false: the stream has ended, s stays
    if ((s.left & ~kGoesOn) > 0) {
      s.off += 32 * D;
      s.p_first += 32;
      s.rows -= 32;
      --s.left;
      return true;
    }
    if (s.left != 0) {
      open_of_chain(s);
      return true;
    }
    if (c_x + stride >= hi) return false;
    c_x += stride;
    if (++c_lane == n_fetch) {
      c_lane = 0;
      fetch_items(c_x);
    }
    open_item(s);
    return true;
  };

  typedef const __attribute__((address_space(1))) char* gptr_t;
  typedef const __attribute__((address_space(1))) u32x4_t* gvec_t;
  auto uni64 = [](unsigned long long v) {
    const unsigned lo32 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi32 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return ((unsigned long long)hi32 << 32) | (unsigned long long)lo32;
  };
  // (requests as in the decode kernel: one form for whole and ragged steps; rows past the last one repeat it)
  auto issue_keys = [&](const Step& s, uint4 (&kr)[2][NS]) {
    gptr_t kb = (gptr_t)uni64((unsigned long long)(a.K + s.off));
    const int last = s.rows > 0 ? s.rows - 1 : 0;
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int row = 16 * h + (ln & 15);
      row = row < last ? row : last;
#pragma unroll
      for (int sl = 0; sl < NS; ++sl) {
        const u32x4_t v = *(gvec_t)(kb + (unsigned)(row * D * 2 + 16 * (ln >> 4) + sl * 64));
        kr[h][sl] = make_uint4(v.x, v.y, v.z, v.w);
      }
    }
  };
  auto issue_values = [&](const Step& s, int into) {
    int ln = lane, wv = wave;
    asm volatile("" : "+v"(ln), "+v"(wv));
    const uint32_t dst = lds_addr_of(&stage[0][0]) +
                         (uint32_t)__builtin_amdgcn_readfirstlane(wv) * (2 * VBYTES) + into * VBYTES;
    const void* vb = reinterpret_cast<const void*>(uni64((unsigned long long)(a.V + s.off)));
    const int last = s.rows > 0 ? s.rows - 1 : 0;
    constexpr int RPC = 64 / PPR;
    const int lrow = (ln & 63) / PPR;
    const int poff = (((ln & 63) % PPR) ^ (2 * (lrow & 3))) * 16;
    // a document of several items is read by several waves of this XCD at about the same time: its lines stay in the L2;
    // the others, read once, are not kept (with the hint everywhere 1024 tokens over 500 documents take 2301 us, without
    // 1955; 512 over 4096 759 and 796)
    if (s.what & 0x8000) {
#pragma unroll
      for (int i = 0; i < NVL; ++i) {
        const int row = i * RPC + lrow;
        const int src_row = row < last ? row : last;
        copy16_to_lds_async_stream(vb, (uint32_t)(src_row * D * 2 + poff), dst + i * 1024);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NVL; ++i) {
        const int row = i * RPC + lrow;
        const int src_row = row < last ? row : last;
        copy16_to_lds_async_at(vb, (uint32_t)(src_row * D * 2 + poff), dst + i * 1024);
      }
    }
  };
  const int vt_lane = (4 * rr + (n >> 2)) * (D * 2) + (n >> 2) * 32 + ((n >> 1) & 1) * 16 + (n & 1) * 8;

  // ---- the item at hand: queries (B operands, column n = (token n / r, head n % r)), running softmax -------------
  bf16x8_t bqh[NS], bql[NS];
  float m_run = -INFINITY, l_run = 0.f;
  int cur_p = -1;  // position of key 0 of the sub-tile the rotation state is valid for; -1 = invalid
  f32x4_t o[NCB];
  // What follows is worked out from an opaque copy of the lane number, here and in end_item: kept across the stream it would
  // spill, and a reload is awaited with everything in flight.
  auto head_row = [&](const Step& s, int ln) {  // (token, head) of the lane's column, inside the window
    return (s.pair >> 6) * a.Hq + (s.what >> 16) * a.r + (ln & (a.r - 1));
  };
  auto issue_queries = [&](const Step& s) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    gptr_t qb = (gptr_t)uni64((unsigned long long)da.qrot);
    const unsigned at = (unsigned)head_row(s, ln) * (D * 4) + 32 * (ln >> 4);  // (a window's buffers stay under 4 GB)
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      const u32x4_t h = *(gvec_t)(qb + (at + 128 * sl)), l = *(gvec_t)(qb + (at + 128 * sl + 16));
      bqh[sl] = as_bf16x8(make_uint4(h.x, h.y, h.z, h.w));
      bql[sl] = as_bf16x8(make_uint4(l.x, l.y, l.z, l.w));
    }
  };
  auto begin_item = [&]() {
    // the queries are awaited here: left to the next turn, its waits would be placed for this path, i.e. drain every request
    // in flight
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) asm volatile("" : "+v"(bqh[sl]), "+v"(bql[sl]));
    m_run = -INFINITY;
    l_run = 0.f;
    cur_p = -1;  // the angles start afresh: no bit of the result depends on the item before
#pragma unroll
    for (int c = 0; c < NCB; ++c) o[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  // The outputs of the item's columns go through the stage whose values have been used, so that a store writes whole rows
  // (an empty partial, maximum -inf, may hold anything: the merge does not look at it).
  auto end_item = [&](const Step& s, int cur_stage) {
    int ln = lane, wv = wave;
    asm volatile("" : "+v"(ln), "+v"(wv));
    const int cols = (s.what & 0xff) * a.r, part = (s.what >> 8) & 0x3f, col = ln & 15;
    const unsigned ph = (unsigned)(head_row(s, ln) * a.k + (s.pair & 63)) * (unsigned)da.parts + part;
    float l = l_run;
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    unsigned char* const st = &stage[wv][0] + cur_stage * VBYTES;
#pragma unroll
    for (int c = 0; c < NCB; ++c)
      *reinterpret_cast<f32x4_t*>(st + col * (D * 4) + ((4 * c + (ln >> 4)) ^ col) * 16) = o[c];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    typedef __attribute__((address_space(1))) char* gout_t;
    gout_t ob = (gout_t)uni64((unsigned long long)da.part_o);
    gout_t mb = (gout_t)uni64((unsigned long long)da.part_ml);
    const float m = m_run;
    begin_item();
    if (ln < cols)
      *(__attribute__((address_space(1))) unsigned long long*)(mb + ph * 8u) =
          __builtin_bit_cast(unsigned long long, make_float2(m, l));
    if (s.what & 0x4000) {  // the partials that the merge looks at behind a token's last chain: empty
      const unsigned at = (unsigned)((s.pair >> 6) * a.Hq + (s.what >> 16) * a.r) * a.k;
      const int next = (s.pair & 63) + 1 + ln;
      if (next < da.n_chains)
        for (int h = 0; h < a.r; ++h)
          for (int p = 0; p < da.parts; ++p)
            *(__attribute__((address_space(1))) unsigned long long*)(mb + ((at + h * a.k + next) * da.parts + p) * 8u) =
                __builtin_bit_cast(unsigned long long, make_float2(-INFINITY, 0.f));
    }
    constexpr int CPS = 1024 / (D * 4);  // columns of a wave-wide store
    for (int c0 = 0; c0 < cols; c0 += CPS) {  // wave-uniform
      const int c = c0 + ln / (64 / CPS), piece = ln % (64 / CPS);
      const unsigned pc = (unsigned)__shfl((int)ph, c, 64);
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(st + c * (D * 4) + (piece ^ c) * 16);
      if (c < cols) *(__attribute__((address_space(1))) u32x4_t*)(ob + (pc * (D * 4) + piece * 16)) = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  fetch_items(c_x);
  Step s0, s1, s2;  // the step worked on, the next two
  open_item(s0);
  issue_queries(s0);
  s1 = s0;
  bool more1 = advance(s1), more2 = false;  // s1, s2 are steps of the stream (else repeats whose requests go unused)
  s2 = s1;
  if (more1) more2 = advance(s2);
  uint4 kA[2][NS], kB[2][NS];
  issue_keys(s0, kA);
  issue_values(s0, 0);
  issue_keys(s1, kB);
  begin_item();

  float2 cs[NU];  // (cos, sin)((cur_p + n) * theta_u), u = 32s' + 8rr + j at index 8s' + j
  bool live = true;

  auto turn = [&](uint4 (&kraw)[2][NS], const int cur_stage) __attribute__((always_inline)) {
    const int rows_valid = live ? s0.rows : 0;
    const int p_first = s0.p_first;
#pragma unroll
    for (int h = 0; h < 2; ++h)  // this step's keys are awaited here, ahead of the value request (see the decode kernel)
#pragma unroll
      for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(kraw[h][s].x), "+v"(kraw[h][s].y), "+v"(kraw[h][s].z), "+v"(kraw[h][s].w));
    issue_values(s1, cur_stage ^ 1);

    if (ROT && live && cur_p != p_first) {
      int ln = lane, wv = wave;
      asm volatile("" : "+v"(ln), "+v"(wv));
      const int n_ = ln & 15, rr_ = ln >> 4;
      if (p_first == 0) {
#pragma unroll
        for (int s2i = 0; s2i < NS / 2; ++s2i)
#pragma unroll
          for (int j = 0; j < 8; ++j) cs[8 * s2i + j] = base0[n_][32 * s2i + 8 * rr_ + j];
      } else {
        if (ln < HALF) estart[wv][ln] = cis_pos(p_first, theta_s[ln]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s2i = 0; s2i < NS / 2; ++s2i)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int u = 32 * s2i + 8 * rr_ + j;
            cs[8 * s2i + j] = cmul(estart[wv][u], base0[n_][u]);
            if (j & 1) __builtin_amdgcn_sched_barrier(0);  // (all 64 reads ahead of the products would spill the stream)
          }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      cur_p = p_first;
    }

    float sc[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t y1[NS / 2][4], y2[NS / 2][4];
#pragma unroll
      for (int s2i = 0; s2i < NS / 2; ++s2i) {
        const uint4 a1 = kraw[h][s2i], a2 = kraw[h][s2i + NS / 2];
        const uint32_t w1[4] = {a1.x, a1.y, a1.z, a1.w};
        const uint32_t w2[4] = {a2.x, a2.y, a2.z, a2.w};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          if (ROT) {
            const float2 c0 = cs[8 * s2i + 2 * jj], c1 = cs[8 * s2i + 2 * jj + 1];
            const float p0 = bf16_lo(w1[jj]), p1 = bf16_hi(w1[jj]);
            const float q0 = bf16_lo(w2[jj]), q1 = bf16_hi(w2[jj]);
            y1[s2i][jj] = pack_bf16(p0 * c0.x - q0 * c0.y, p1 * c1.x - q1 * c1.y);
            y2[s2i][jj] = pack_bf16(q0 * c0.x + p0 * c0.y, q1 * c1.x + p1 * c1.y);
          } else {
            y1[s2i][jj] = w1[jj];
            y2[s2i][jj] = w2[jj];
          }
        }
      }
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2i = 0; s2i < NS / 2; ++s2i) {
        const bf16x8_t k1 = as_bf16x8(make_uint4(y1[s2i][0], y1[s2i][1], y1[s2i][2], y1[s2i][3]));
        const bf16x8_t k2 = as_bf16x8(make_uint4(y2[s2i][0], y2[s2i][1], y2[s2i][2], y2[s2i][3]));
        acc = mfma16(k1, bqh[s2i], acc);
        acc = mfma16(k1, bql[s2i], acc);
        acc = mfma16(k2, bqh[s2i + NS / 2], acc);
        acc = mfma16(k2, bql[s2i + NS / 2], acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[h][i] = 16 * h + 4 * rr + i < rows_valid ? acc[i] : -INFINITY;
      if (ROT) {  // advance the rotation state by 16 positions
#pragma unroll
        for (int s2i = 0; s2i < NS / 2; ++s2i)
#pragma unroll
          for (int j = 0; j < 8; ++j) cs[8 * s2i + j] = cmul(cs[8 * s2i + j], step16[32 * s2i + 8 * rr + j]);
      }
    }
    if (ROT) cur_p += 32;
    // the keys of the step after next (this step's are in the scores now); on an item's last step as many requests for the
    // queries of the next one, whose keys then follow behind the outputs
    const bool last = live && s0.left == 0;
    issue_keys(s2, kraw);

    // ---- online softmax (exp2 domain) ---------------------------------------------------------------------
    float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                     fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const bool bump = mx > m_run;
    if (__any(bump)) {
      const float m_new = bump ? mx : m_run;
      const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < NCB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[c][i] *= alpha;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float psum = 0.f;
    uint32_t pwh[4], pwl[4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float p0 = __builtin_amdgcn_exp2f(sc[h][2 * i] - m_use);
        const float p1 = __builtin_amdgcn_exp2f(sc[h][2 * i + 1] - m_use);
        psum += p0 + p1;
        split_pack_bf16(p0, p1, pwh[2 * h + i], pwl[2 * h + i]);
      }
    l_run += psum;
    const bf16x8_t pbh = as_bf16x8(make_uint4(pwh[0], pwh[1], pwh[2], pwh[3]));
    const bf16x8_t pbl = as_bf16x8(make_uint4(pwl[0], pwl[1], pwl[2], pwl[3]));

    // ---- second product (requests younger than this step's values: keys of the next two steps or, for the second, the next
    // queries; the next values) ---
    wait_copies_but<NVL + 4 * NS>();
    {
      const unsigned char* vt = &stage[wave][0] + cur_stage * VBYTES;
      int vl = vt_lane;
      asm volatile("" : "+v"(vl));
#pragma unroll
      for (int c = 0; c < NCB; ++c) {
        const unsigned char* vp = vt + (vl ^ (32 * c));
        const s16x4_t v0 = lds_read_tr16(vp);                 // keys 4 rr .. + 3
        const s16x4_t v1 = lds_read_tr16(vp + 16 * (D * 2));  // keys 16 + 4 rr .. + 3
        const bf16x8_t av = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        o[c] = mfma16(av, pbh, o[c]);
        o[c] = mfma16(av, pbl, o[c]);
      }
    }
    // ---- next turn -------------------------------------------------------------------------------------------
    if (last) {  // the item is complete (behind the last one s1 repeats it, and the queries go unused)
      issue_queries(s1);
      end_item(s0, cur_stage);
    }
    live = more1;
    s0 = s1;
    s1 = s2;
    more1 = more2;
    if (more2) more2 = advance(s2);
  };
  do {  // always two turns per trip (the key registers have fixed names); the spare one works on masked rows
    turn(kA, 0);
    turn(kB, 1);
  } while (live);
  wait_copies_but<0>();  // the repeated requests of the last turns still write into the stages
}

// Partials of two kinds for every (token, head): n1 of its selected documents, tokens counted from tok0, and n2 of the
// local context, all tokens.  One wave per (token, head), four per workgroup; a lane owns D / 64 adjacent outputs.  The first
// eight partials are requested together with the (max, sum) pairs: where there are no more, a row is one round trip
// (32000 rows of two partials, one workgroup each: 19.3 us, so 14).
template <int D>
__global__ __launch_bounds__(256) void attend_merge2_kernel(const float* __restrict__ o1, const float2* __restrict__ ml1,
                                                            int n1, const float* __restrict__ o2,
                                                            const float2* __restrict__ ml2, int n2, uint16_t* __restrict__ out,
                                                            float* __restrict__ lse, long long row0, long long rows,
                                                            const int* __restrict__ chained, int n_chained, int Hq, int per_list) {
  constexpr int V = D / 64;
  constexpr int U = 8;
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= rows) return;
  const float2* m1 = ml1 + row * n1;
  const float* p1 = o1 + row * n1 * D + lane * V;
  if (chained != nullptr && chained[(int)(row % Hq) / per_list] != 0) n1 = n_chained;
  const int ns = n1 + n2;
  const float2* m2 = ml2 + (row0 + row) * n2;
  typedef float vec_t __attribute__((ext_vector_type(V)));
  const float* p2 = o2 + (row0 + row) * n2 * D + lane * V;
  vec_t v[U];
  auto fetch = [&](int s0) {  // (past the end: the last one again)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + u < ns ? s0 + u : ns - 1;
      v[u] = *reinterpret_cast<const vec_t*>(s < n1 ? p1 + (long long)s * D : p2 + (long long)(s - n1) * D);
    }
  };
  float2 ml[4];  // 256 partials at most
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s = lane + 64 * i;
    ml[i] = make_float2(-INFINITY, 0.f);
    if (64 * i < ns && s < ns) ml[i] = s < n1 ? m1[s] : m2[s - n1];
  }
  fetch(0);
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) mx = fmaxf(mx, ml[i].x);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  float lsum = 0.f, w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool empty = ml[i].x == -INFINITY;  // (its sum and outputs may be anything)
    w[i] = empty ? -1.f : __builtin_amdgcn_exp2f(ml[i].x - mx);
    lsum += empty ? 0.f : w[i] * ml[i].y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
  float acc[V] = {};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (64 * i >= ns) break;
    const int top = ns - 64 * i < 64 ? ns - 64 * i : 64;
    for (int j0 = 0; j0 < top; j0 += U) {
      if (i + j0 > 0) fetch(64 * i + j0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (j0 + u >= top) break;
        const float f = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w[i]), j0 + u));
        if (f < 0.f) continue;  // wave-uniform
#pragma unroll
        for (int c = 0; c < V; ++c) acc[c] += f * v[u][c];
      }
    }
  }
  const long long qh = row0 + row;
  float res[V];
#pragma unroll
  for (int c = 0; c < V; ++c) res[c] = lsum > 0.f ? acc[c] / lsum : 0.f;
  if constexpr (V == 2)
    reinterpret_cast<uint32_t*>(out + qh * D)[lane] = pack_bf16(res[0], res[1]);
  else
    out[qh * D + lane] = (uint16_t)(pack_bf16(res[0], 0.f) & 0xffffu);
  if (lse != nullptr && lane == 0) lse[qh] = lsum > 0.f ? (mx + log2f(lsum)) * 0.6931471805599453f : -INFINITY;
}

int launch_merge2(int d, const float* o1, const float2* ml1, int n1, const float* o2, const float2* ml2, int n2, uint16_t* out,
                  float* lse, long long row0, long long rows, hipStream_t st, const int* chained, int n_chained, int Hq,
                  int per_list) {
  const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  if (d == 128) hipLaunchKernelGGL(attend_merge2_kernel<128>, grid, block, 0, st, o1, ml1, n1, o2, ml2, n2, out, lse, row0, rows, chained, n_chained, Hq, per_list);
  else hipLaunchKernelGGL(attend_merge2_kernel<64>, grid, block, 0, st, o1, ml1, n1, o2, ml2, n2, out, lse, row0, rows, chained, n_chained, Hq, per_list);
  return hipGetLastError() == hipSuccess ? MSA_OK : MSA_ERR_HIP;
}

// Bytes of the fixed buffers and of those that grow with the tokens of a window.
static size_t docs_fixed_bytes(const Dims& dm) {
  const size_t S = dm.scope_all ? 1 : dm.Hkv;
  return round_up256(S * dm.N * 8) + round_up256(S * dm.N * 4) + round_up256(S * 8);
}
static int slot_bits(int k) {  // the least power of two that holds k slots
  int b = 0;
  while ((1 << b) < k) ++b;
  return b;
}
static size_t docs_window_bytes(const Dims& dm, int k, int slots, size_t tokens) {  // slots: partials per (token, head)
  const size_t S = dm.scope_all ? 1 : dm.Hkv, e = S * tokens * k;
  return round_up256(tokens * dm.Hq * dm.d * 4) + round_up256(e * 16) + round_up256(e * 4) + round_up256((S * tokens << slot_bits(k)) * 4) +
         round_up256(tokens * dm.Hq * slots * dm.d * 4) + round_up256(tokens * dm.Hq * slots * 8);
}

// Parts of a document where the items (at most one per token, slot and KV head) are few.
static int docs_parts(const Dims& dm, long long BM, int k) {
  const long long steps = dm.G / 32;
  int parts = 1;
  while (parts < 4 && 2 * parts * k <= 128 && BM * k * dm.Hkv * parts < kDocsItems && steps / (2 * parts) >= 4 && steps % (2 * parts) == 0) parts *= 2;
  return parts;
}

// Where the documents are certain to be shared (twice as many pairs as documents) or the pairs are many, and the rows that
// the decode kernel would gather are worth three launches more.  Against that kernel, us, selections of which half are among
// 4 k documents of a topic / drawn at random / without a document in common (512 rows, 8 heads of 128 and r = 4 unless said):
//   512 tokens of 8 of 4096 documents   1067 -> 710   1332 -> 983   1367 -> 1372
//   64 of 32 of 8192                     589 -> 463    681 -> 715    691 -> 712
//   40 of 16 of 8192                     251 -> 183    286 -> 250    289 -> 254
//   100 of 16 of 4000 (128 rows)         147 -> 119    174 -> 185    192 -> 208
//   64 of 12 of 2000 (256 rows)          117 -> 107    143 -> 161    158 -> 168
//   300 of 16 of 8192, r = 8             716 -> 588    842 -> 806    860 -> 960
// and 16 tokens of 16 of 64 documents 91 -> 71.  On the other side of the lines: 64 of 4 of 8192 82 -> 86, 32 of 20 of 2000
// (two heads of 64) 45 -> 67, 64 of 4 of 128 (64 rows of 64) 27 -> 31.  Sharing grows with the tokens of a topic: 16 tokens
// under 2.5 GiB (16 of 8000, 1024 rows) 174 -> 178, 200 -> 218, 202 -> 220, (64 of 8000) 333 -> 318, 353 -> 380, 357 -> 387,
// where 20 of 32 of 8192 (1024 rows) go 490 -> 360, 515 -> 469, 519 -> 471; and with r = 8, where an item takes two tokens, 32
// (32 of 8192) 180 -> 182, 191 -> 211, 196 -> 216, and 2 x 64 (16 of 4096, 128 rows) 95 -> 93, 107 -> 115, 108 -> 128.
bool docs_path_applies(const Dims& dm, int B, int M, int k) {
  const long long S = dm.scope_all ? 1 : dm.Hkv, pairs = (long long)B * M * k, items = pairs * dm.Hkv;
  const long long bytes = items * dm.G * dm.d * 4;
  if (dm.G % 32 != 0 || dm.Hkv > 64 || S * dm.N > (8 << 20)) return false;
  const bool certain = pairs >= 2ll * dm.N;
  if (!certain && dm.r == 8 && M < 128) return false;
  return bytes >= (certain || M >= 32 ? 1ll << 30 : 5ll << 29) || (items >= 3072 && bytes >= (96ll << 20) && (certain || M >= 32)) ||
         (certain && bytes >= (256ll << 20));
}

DocsPlan plan_docs(const Dims& dm, int B, int M, int k, size_t bytes) {
  DocsPlan p = {};
  const long long BM = (long long)B * M, steps = dm.G / 32;
  p.parts = docs_parts(dm, BM, k);
  p.part_steps = (int)(steps / p.parts);
  // documents of a chain: the fewest steps of the busiest wave, two for what a chain costs besides its documents
  p.chain = 1;
  for (long long c = 2, best = (BM * k * dm.Hkv + 2047) / 2048 * (steps + 2); c <= kMaxChain && p.parts == 1; ++c) {
    const long long cost = (BM * dm.Hkv * ((k + c - 1) / c) + 2047) / 2048 * (c * steps + 2);
    if (cost <= best) {
      best = cost;
      p.chain = (int)c;
    }
  }
  // Parts become fewer as k grows; the size to ask for is that of the most partials which a call of no more documents uses.
  int slots = 0;
  for (int kk = 1; kk <= k; ++kk) {
    const int s = kk * docs_parts(dm, BM, kk);
    slots = s > slots ? s : slots;
  }
  const size_t fixed = docs_fixed_bytes(dm);
  // tokens whose partials fit: in all at most kDocsBytes, but 64 tokens at least
  size_t least = BM < 64 ? BM : 64;
  size_t window = kDocsBytes;
  const size_t whole = docs_window_bytes(dm, k, slots, BM), few = docs_window_bytes(dm, k, slots, least);
  if (whole < window) window = whole;
  if (few > window) window = few;
  p.bytes = fixed + window;
  const size_t have = bytes < p.bytes ? bytes : p.bytes;
  if (have < fixed + docs_window_bytes(dm, k, k * p.parts, least)) return p;  // tokens = 0: the workspace is too small for this path
  long long lo = least, hi = BM;
  while (lo < hi) {
    const long long mid = (lo + hi + 1) / 2;
    if (fixed + docs_window_bytes(dm, k, k * p.parts, mid) <= have)
      lo = mid;
    else
      hi = mid - 1;
  }
  const long long windows = (BM + lo - 1) / lo;
  p.tokens = (int)((BM + windows - 1) / windows);
  return p;
}

int launch_attend_docs(const Dims& dm, const DocsPlan& pl, const AttendArgs& a0, const RopeTheta& th, int BM, void* ws,
                       int bank_keys_rotated, const float* loc_o, const float2* loc_ml, int n_loc, void* out, float* lse,
                       hipStream_t st) {
  const int S = a0.idx_sel;
  DocsArgs da = {};
  char* at = (char*)ws;
  auto take = [&](size_t bytes) {
    char* p = at;
    at += round_up256(bytes);
    return p;
  };
  const size_t W = pl.tokens, e = (size_t)S * W * a0.k, parts = (size_t)W * dm.Hq * a0.k * pl.parts;
  da.base = (unsigned long long*)take((size_t)S * dm.N * 8);
  da.cnt = (int*)take((size_t)S * dm.N * 4);
  da.n_items = (int*)take((size_t)S * 8);
  da.qrot = (uint4*)take(W * dm.Hq * dm.d * 4);
  da.items = (int4*)take(e * 16);
  da.entries = (int*)take(e * 4);
  da.rank = (int*)take((size_t)S * W * 4 << slot_bits(a0.k));
  da.part_o = (float*)take(parts * dm.d * 4);
  da.part_ml = (float2*)take(parts * 8);
  da.cap = (int)(W * a0.k);
  da.tile_tok = 16 / dm.r;
  da.parts = pl.parts;
  da.part_steps = pl.part_steps;
  da.kshift = slot_bits(a0.k);
  da.chain = pl.chain;
  da.n_chains = (a0.k + pl.chain - 1) / pl.chain;
  da.n_all = BM;
  AttendArgs a = a0;
  profile_mark(dm, false, st);
  for (int t0 = 0; t0 < BM; t0 += pl.tokens) {
    da.tok0 = t0;
    da.n_tok = BM - t0 < pl.tokens ? BM - t0 : pl.tokens;
    const dim3 ggrid(S + (da.n_tok + 3) / 4);
    // two workgroups per CU, and no more of them than there can be items
    long long wgs = ((long long)da.n_tok * a.k * dm.Hkv * pl.parts + kAttWaves - 1) / kAttWaves;
    wgs = wgs < 512 ? (wgs + 7) / 8 * 8 : 512;
    const long long rows = (long long)da.n_tok * dm.Hq;
#define MSA_GROUP(DD, LL) \
  do { \
    if (pl.tokens >= BM) hipLaunchKernelGGL((group_kernel<DD, LL, true>), ggrid, dim3(kGroupThreads), 0, st, a, da, th); \
    else hipLaunchKernelGGL((group_kernel<DD, LL, false>), ggrid, dim3(kGroupThreads), 0, st, a, da, th); \
  } while (0)
#define MSA_DOCS(DD) \
  do { \
    if (dm.N <= kLdsDocs) MSA_GROUP(DD, true); else MSA_GROUP(DD, false); \
    if (bank_keys_rotated) hipLaunchKernelGGL((attend_docs_kernel<DD, false>), dim3((unsigned)wgs), dim3(256), 0, st, a, da, th); \
    else hipLaunchKernelGGL((attend_docs_kernel<DD, true>), dim3((unsigned)wgs), dim3(256), 0, st, a, da, th); \
  } while (0)
    if (dm.d == 128) MSA_DOCS(128);
    else MSA_DOCS(64);
#undef MSA_DOCS
#undef MSA_GROUP
    const int rc = launch_merge2(dm.d, da.part_o, da.part_ml, a.k * pl.parts, loc_o, loc_ml, n_loc, (uint16_t*)out, lse,
                                 (long long)t0 * dm.Hq, rows, st, da.n_items + S, da.n_chains * pl.parts, dm.Hq, dm.Hq / S);
    if (rc != MSA_OK) return rc;
  }
  profile_mark(dm, true, st);
  return hipGetLastError() == hipSuccess ? MSA_OK : MSA_ERR_HIP;
}

}  // namespace msa
