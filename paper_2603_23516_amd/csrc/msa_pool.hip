// msa_pool_kv: the pooled memory bank of the offline encoding stage (paper, Section 3.4.1, Stage 1):
// every document is position-encoded on its own, positions 0..G-1 (Section 3.2.2), and the keys and
// values are chunk-mean pooled (phi of Section 3.2.1) into the K-bar, V-bar that Eq. 3 concatenates.
// A pure HBM stream like the routing-key build: each K and V element is read once, 1/P of it written.
//
// One wavefront owns one chunk of one tensor.  RoPE pairs element u with u + d/2, so a lane loads
// the 16-byte piece `pc` of a row together with piece pc + d/16 (the partner half): d/16 lanes
// cover a row and a wave-wide pair of loads covers 1024/d rows.  The angles of the lane's first row,
// (cos, sin)(p theta_u), come from a double-precision range reduction; the rows a constant stride apart
// are summed by Horner's rule.  With the vector work of the angles shared by a workgroup and halved per row the keys
// stream as fast as the values: 4.3 GB at d = 128 781 -> 704 us, 0.5 GB at d = 64 150 -> 114 us, P = 32 378 -> 295 us.  Both
// end at what reading together with writing allows: 685 and 668 us for 4.3 GB and 1/64 of it (read alone 620).
#include "msa_device.h"
#include "msa_host.h"

namespace msa {

struct PoolTheta {
  double th[64];     // theta_u = base^(-2u/d)
  float2 estep[64];  // (cos, sin)(RPL * theta_u), RPL = rows per wave-wide load
};

// HUGE: chunks of 2^31 elements or more, whose offsets need 64 bits.  A form of its own, since in 64 bits the kernel loses 2 to
// 3 % where a chunk is a single batch (4.3 GB in chunks of 32 rows of 128: the encoding 2286 us, 2322; 0.5 GB, 64 of 64: 276,
// 285).
template <int D, bool ROT, int NB, bool HUGE>
__global__ __launch_bounds__(256) void pool_chunks_kernel(const uint16_t* __restrict__ X,
                                                          uint16_t* __restrict__ Xbar,
                                                          const int32_t* __restrict__ lens,
                                                          int32_t* __restrict__ pooled_lens, int doc_begin,
                                                          uint32_t n_pairs, int Hkv, int G, int P,
                                                          int C, PoolTheta th) {
  constexpr int LPR = D / 16;    // lanes per row (each holds a piece and its partner half)
  constexpr int RPL = 64 / LPR;  // rows per wave-wide load pair
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Keys: a workgroup takes the same chunk of four (document, head) pairs (they share their angles), neighbouring
  // workgroups neighbouring chunks.  Values: chunks in order.
  const uint32_t bq = blockIdx.x / (uint32_t)C, br = blockIdx.x % (uint32_t)C;
  const uint32_t in_row = 4 * br + wave;  // values: chunk 4 blockIdx + wave = 4 bq C + in_row
  const uint32_t j = ROT ? br : in_row % (uint32_t)C;
  const uint32_t t = 4 * bq + (ROT ? wave : in_row / (uint32_t)C);
  const bool live = t < n_pairs;  // wave-uniform
  const int g = (int)(t % (uint32_t)Hkv);
  const long long doc = live ? doc_begin + t / (uint32_t)Hkv : doc_begin;
  const uint16_t* src = X + ((doc * Hkv + g) * (long long)G + (long long)j * P) * D;
  const int pc = lane % LPR;
  const int rowoff = lane / LPR;
  // tokens of this chunk (wave-uniform): a tail chunk is short, a chunk past the end has none and pools to zero
  int n_rows = live ? P : 0;
  if (lens != nullptr && live) {
    int len = lens[doc];
    len = len < 1 ? 1 : (len > G ? G : len);
    n_rows = len - (int)j * P;
    n_rows = n_rows < 0 ? 0 : (n_rows > P ? P : n_rows);
    if (pooled_lens != nullptr && g == 0 && j == 0 && lane == 0) pooled_lens[doc] = (len + P - 1) / P;
  }

  // NB load pairs per batch: with the rotation four (eight cost it too many registers: 704 -> 705 us at d = 128, 114 ->
  // 132 at d = 64), without it eight (703 -> 684 us), where a chunk has more than four (P = 8, d = 128, 0.5 GB: 222 us with
  // eight, 162 with four)
  uint4 v1[NB], v2[NB];
  auto load = [&](int it0) __attribute__((always_inline)) {
    const uint16_t* rp = HUGE ? src + (long long)it0 * (RPL * D) + (rowoff * D + pc * 8) : src + (it0 * RPL + rowoff) * D + pc * 8;
    if (HUGE ? NB * RPL <= n_rows - it0 * RPL : (it0 + NB) * RPL <= n_rows) {  // wave-uniform: whole batch, no condition on a load
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        v1[u] = load_stream16(rp + u * RPL * D);
        v2[u] = load_stream16(rp + u * RPL * D + D / 2);
      }
    } else {
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        v1[u] = v2[u] = make_uint4(0, 0, 0, 0);
        if (HUGE ? u * RPL + rowoff < n_rows - it0 * RPL : (it0 + u) * RPL + rowoff < n_rows) {
          v1[u] = load_stream16(rp + u * RPL * D);
          v2[u] = load_stream16(rp + u * RPL * D + D / 2);
        }
      }
    }
  };
  // batches that hold tokens; they run from the last to the first (see below)
  const int iters = n_rows > 0 ? __builtin_amdgcn_readfirstlane(HUGE ? (n_rows - 1) / RPL + 1 : (n_rows + RPL - 1) / RPL) : 1;
  const int last0 = (iters - 1) / NB * NB;
  load(last0);  // on its way while the angles are worked out
  __shared__ float2 cs_s[ROT ? 8 : 1][64];
  float2 stp[8];
  if (ROT) {
    // The four waves have the same chunk number and so the same angles: each works out a quarter of them.
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int e = 2 * wave + i;
      cs_s[e][lane] = cis_pos((int)j * P + rowoff, th.th[8 * pc + e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) stp[e] = th.estep[8 * pc + e];
    lds_barrier();
  }
  if (!live) return;  // wave-uniform, behind the only barrier
  float a1[8], a2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) a1[e] = a2[e] = 0.f;

  // The sum of the rotated rows of a lane, rows RPL apart, is evaluated from its last row to its first (Horner's rule on
  // the pairs as complex numbers): z = x + z e^{i RPL theta}, and the angle of the lane's first row comes in once, at
  // the end.  That is four multiply-adds per pair and row, where rotating every row takes four more for the next angle.
  for (int it0 = last0; it0 >= 0; it0 -= NB) {
    if (it0 < last0) load(it0);
#pragma unroll
    for (int u = NB - 1; u >= 0; --u) {
      const uint32_t w1[4] = {v1[u].x, v1[u].y, v1[u].z, v1[u].w};
      const uint32_t w2[4] = {v2[u].x, v2[u].y, v2[u].z, v2[u].w};
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const float p0 = bf16_lo(w1[jj]), p1 = bf16_hi(w1[jj]);
        const float q0 = bf16_lo(w2[jj]), q1 = bf16_hi(w2[jj]);
        if (ROT) {
          const float2 w0 = stp[2 * jj], w1s = stp[2 * jj + 1];
          const float z0 = a1[2 * jj], z1 = a1[2 * jj + 1];
          a1[2 * jj] = fmaf(z0, w0.x, fmaf(-a2[2 * jj], w0.y, p0));
          a1[2 * jj + 1] = fmaf(z1, w1s.x, fmaf(-a2[2 * jj + 1], w1s.y, p1));
          a2[2 * jj] = fmaf(a2[2 * jj], w0.x, fmaf(z0, w0.y, q0));
          a2[2 * jj + 1] = fmaf(a2[2 * jj + 1], w1s.x, fmaf(z1, w1s.y, q1));
        } else {
          a1[2 * jj] += p0;
          a1[2 * jj + 1] += p1;
          a2[2 * jj] += q0;
          a2[2 * jj + 1] += q1;
        }
      }
    }
  }
  if (ROT) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float2 z = cmul(make_float2(a1[e], a2[e]), cs_s[e][lane]);
      a1[e] = z.x;
      a2[e] = z.y;
    }
  }
  // combine the RPL row groups that hold the same columns
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    a1[e] = add_row_groups<LPR>(a1[e]);
    a2[e] = add_row_groups<LPR>(a2[e]);
  }
  if (rowoff == 0) {
    mean_of(a1, n_rows > 0 ? n_rows : 1);
    mean_of(a2, n_rows > 0 ? n_rows : 1);
    uint16_t* dst = Xbar + (((doc * Hkv + g) * (long long)C + j) * D) + pc * 8;
    const uint4 o1 = make_uint4(pack_bf16(a1[0], a1[1]), pack_bf16(a1[2], a1[3]), pack_bf16(a1[4], a1[5]), pack_bf16(a1[6], a1[7]));
    const uint4 o2 = make_uint4(pack_bf16(a2[0], a2[1]), pack_bf16(a2[2], a2[3]), pack_bf16(a2[4], a2[5]), pack_bf16(a2[6], a2[7]));
    // past the L2 where a store is a whole line and every chunk has its rows (0.5 GB at d = 64, whose stores are half
    // lines: the encoding 274 us, with the hint 288; documents of different lengths 1493 and 1510)
    if (D == 128 && lens == nullptr) {
      store_stream16(dst, o1);
      store_stream16(dst + D / 2, o2);
    } else {
      *reinterpret_cast<uint4*>(dst) = o1;
      *reinterpret_cast<uint4*>(dst + D / 2) = o2;
    }
  }
}

int launch_pool_kv(const Dims& dm, const void* K, const void* V, int doc_begin, int doc_count,
                   void* Kbar, void* Vbar, int32_t* pooled_lens, hipStream_t st) {
  const long long pairs = (long long)doc_count * dm.Hkv;
  if (pairs == 0) return MSA_OK;
  const long long blocks = (pairs + 3) / 4 * dm.C;  // keys; values: four chunks each, no more than that
  if (blocks > 0x7fffffffLL || pairs > 0xfffffff0LL) return MSA_ERR_UNSUPPORTED;
  const uint32_t n_pairs = (uint32_t)pairs;
  PoolTheta th;
  const int rpl = 64 / (dm.d / 16);
  for (int u = 0; u < 64; ++u) {
    th.th[u] = (u < dm.d / 2) ? pow((double)dm.base, -2.0 * (double)u / (double)dm.d) : 0.0;
    th.estep[u] = make_float2((float)cos(rpl * th.th[u]), (float)sin(rpl * th.th[u]));
  }
  dim3 grid((unsigned)blocks), block(256);
#define MSA_POOL_AS(DD, RR, BB, HH, X, OUT, LENS_OUT) \
  hipLaunchKernelGGL((pool_chunks_kernel<DD, RR, BB, HH>), grid, block, 0, st, (const uint16_t*)X, (uint16_t*)OUT, dm.lens, \
                     LENS_OUT, doc_begin, n_pairs, dm.Hkv, dm.G, dm.P, dm.C, th)
#define MSA_POOL(DD, RR, BB, X, OUT, LENS_OUT) \
  do { \
    if (huge) MSA_POOL_AS(DD, RR, 4, true, X, OUT, LENS_OUT); else MSA_POOL_AS(DD, RR, BB, false, X, OUT, LENS_OUT); \
  } while (0)
  const bool huge = (long long)dm.P * dm.d > 0x7fffffffLL;
  if (Kbar != nullptr) {
    if (dm.d == 128) MSA_POOL(128, true, 4, K, Kbar, pooled_lens);
    else MSA_POOL(64, true, 4, K, Kbar, pooled_lens);
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
  }
  if (Vbar != nullptr) {
    int32_t* const lens_out = Kbar == nullptr ? pooled_lens : nullptr;
    const bool long_chunk = dm.P > 4 * rpl;
    if (dm.d == 128) {
      if (long_chunk) MSA_POOL(128, false, 8, V, Vbar, lens_out); else MSA_POOL(128, false, 4, V, Vbar, lens_out);
    } else {
      if (long_chunk) MSA_POOL(64, false, 8, V, Vbar, lens_out); else MSA_POOL(64, false, 4, V, Vbar, lens_out);
    }
    if (hipGetLastError() != hipSuccess) return MSA_ERR_HIP;
  }
#undef MSA_POOL
#undef MSA_POOL_AS
  return MSA_OK;
}

}  // namespace msa
