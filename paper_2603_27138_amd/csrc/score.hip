// Digest construction and block-importance scoring.
//
// Digest: channel-wise min/max pooling over the keys of a block (Sec. 2.2).
// Score: query against the digest (Sec. 2.2, Sec. 3.2, Alg. 1 TopK argument);
// for a min/max digest each channel contributes max(q*min, q*max), summed over
// channels and over the G query heads of the KV head.  Because the sum over
// heads commutes with the sum over channels, the group folds into two
// coefficient vectors  P_c = sum_h max(q_hc, 0),  N_c = sum_h min(q_hc, 0)  and
// score(j) = sum_c (P_c * max_j[c] + N_c * min_j[c]):  two FMAs per channel
// whatever G is.  The pass is a pure stream over the digest cache (HBM-bound);
// accumulation is binary64 so the binary32 result is the correctly rounded
// score except for ties of the last binary64 bit.
#include "score_tile.h"

namespace scout {

// ------------------------------------------------------------------ digest

// Every key is read once, so the pass is a stream bound by HBM, and what decides its rate is which bytes a wave asks for
// together: a wave takes whole blocks (tiles of S x d elements, contiguous), one at a time or as many as make eight
// 16-byte requests per lane, all of them out before the first is used.  With 16 lanes of a wave on one block and the
// next 16 lanes on the next (four pieces 8 KiB apart per request, one row in flight per lane) 8 sequences x 8 KV heads
// of 16k to 32k tokens (bf16, d = 128, blocks of 32; 400 MB) took 99 us, with whole blocks per wave 76 us (5.8 TB/s; a bare
// read of 512 MiB reaches 6.3).  NT: see launch_digest.
//
// The rows of a block are dealt to the wave's groups of lanes (ROWB / 16 lanes per row) in contiguous ranges, and the
// groups' results are joined in token order with strict comparisons, so that the result is that of one thread that
// walks through the block's valid tokens: of equal elements (zeros of either sign) the first one stays, a NaN in the
// first token stays, later ones are passed over.
template <int DT, int DH, int S>
struct DigestTile {
  static constexpr int ES = DT == SCOUT_BF16 ? 2 : 4, EPL = 16 / ES;  // element bytes, elements per 16-byte request
  static constexpr int LPR = DH * ES / 16;                            // lanes per token row
  static constexpr int RPG = S * LPR / kWave;                         // token rows per group of lanes
  static constexpr int NBLK = RPG >= 8 ? 1 : 8 / RPG;                 // blocks per wave
};

// lower: the value of the group with the earlier tokens
__device__ __forceinline__ float first_min(float lower, float higher) { return higher < lower ? higher : lower; }
__device__ __forceinline__ float first_max(float lower, float higher) { return higher > lower ? higher : lower; }

// Whether the batch holds more keys than the 256 MiB memory-side cache (see launch_digest): the lengths of eight sequences,
// evenly spread, against the sum of theirs at which it does.  Scalar loads, all under way before the first is used: a
// vector load of all lengths would put its latency in front of every wave's keys.
__device__ __forceinline__ bool keys_exceed_cache(const Dims& D, int limit) {
  const int cap = D.max_blocks * D.S;
  int len[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) len[i] = D.ctx_len[(i * D.B) >> 3];
  asm volatile("" ::"s"(len[0]), "s"(len[1]), "s"(len[2]), "s"(len[3]), "s"(len[4]), "s"(len[5]), "s"(len[6]), "s"(len[7]));
  int sum = 0;  // below 8 * 2^20
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int tokens = len[i] < cap ? len[i] : cap;
    sum += tokens > 0 ? tokens : 0;
  }
  return sum > limit;
}

// In front of and behind loads of one side of a branch: the compiler takes plain and non-temporal loads of one address for
// the same and merges the two sides into plain ones.
__device__ __forceinline__ void only_here() { asm volatile(""); }

// MAY_NT: the rows could hold that many keys; nt_limit: see keys_exceed_cache.
template <int DT, int DH, int S, bool MAY_NT>
__global__ __launch_bounds__(256) void digest_kernel(Dims D, const void* __restrict__ k_blocks, void* __restrict__ digest,
                                                     int nt_limit) {
  using L = DigestTile<DT, DH, S>;
  const int pair = grid_pair();  // grid (x, Hkv, B)
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int j0 = (blockIdx.x * 4 + wave) * L::NBLK;
  const int ctx = D.ctx_len[blockIdx.z];
  const int nb = num_blocks(D, ctx);
  if (j0 >= nb) return;
  const int grp = lane / L::LPR;
  const u32x4* tile = static_cast<const u32x4*>(k_blocks) + ((size_t)pair * D.max_blocks + j0) * (S * L::LPR) +
                      grp * L::RPG * L::LPR + lane % L::LPR;
  u32x4 raw[L::NBLK][L::RPG];
  const bool nt = MAY_NT && keys_exceed_cache(D, nt_limit);
#pragma unroll
  for (int n = 0; n < L::NBLK; ++n) {
    if (j0 + n < nb) {  // wave-uniform
      const u32x4* p = tile + (size_t)n * (S * L::LPR);
      if (nt) {
        only_here();
#pragma unroll
        for (int i = 0; i < L::RPG; ++i) raw[n][i] = __builtin_nontemporal_load(p + i * L::LPR);
        only_here();
      } else {
#pragma unroll
        for (int i = 0; i < L::RPG; ++i) raw[n][i] = p[i * L::LPR];
      }
    }
  }
#pragma unroll
  for (int n = 0; n < L::NBLK; ++n) {
    const int j = j0 + n;
    if (j >= nb) break;
    const int valid = ctx - j * S;
    float mn[L::EPL], mx[L::EPL];
    auto element = [&](int i, int e) {
      if constexpr (DT == SCOUT_BF16) return (e & 1) ? bf16_hi(raw[n][i][e >> 1]) : bf16_lo(raw[n][i][e >> 1]);
      else return __uint_as_float(raw[n][i][e]);
    };
    // group 0 starts with the first token itself, the others with values that give way to any number
#pragma unroll
    for (int e = 0; e < L::EPL; ++e) {
      mn[e] = grp == 0 ? element(0, e) : INFINITY;
      mx[e] = grp == 0 ? element(0, e) : -INFINITY;
    }
    if (valid >= S) {  // wave-uniform
#pragma unroll
      for (int i = 0; i < L::RPG; ++i)
#pragma unroll
        for (int e = 0; e < L::EPL; ++e) {
          const float x = element(i, e);
          mn[e] = first_min(mn[e], x);
          mx[e] = first_max(mx[e], x);
        }
    } else {  // the sequence's last block, partly filled
#pragma unroll
      for (int i = 0; i < L::RPG; ++i)
        if (grp * L::RPG + i < valid) {
#pragma unroll
          for (int e = 0; e < L::EPL; ++e) {
            const float x = element(i, e);
            mn[e] = first_min(mn[e], x);
            mx[e] = first_max(mx[e], x);
          }
        }
    }
#pragma unroll
    for (int e = 0; e < L::EPL; ++e) {
      if constexpr (L::LPR == 8) {
        const float pn = __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(mn[e]), 0x128, 0xf, 0xf, false));  // row_ror:8
        const float px = __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(mx[e]), 0x128, 0xf, 0xf, false));
        mn[e] = (lane & 8) ? first_min(pn, mn[e]) : first_min(mn[e], pn);
        mx[e] = (lane & 8) ? first_max(px, mx[e]) : first_max(mx[e], px);
      }
      // a swap of a value with itself leaves the lower row's (half's) value in the first result, the higher one's in
      // the second, in all lanes
      if constexpr (L::LPR <= 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(mn[e]), __float_as_uint(mn[e]), false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx[e]), __float_as_uint(mx[e]), false, false);
        mn[e] = first_min(__uint_as_float(a[0]), __uint_as_float(a[1]));
        mx[e] = first_max(__uint_as_float(b[0]), __uint_as_float(b[1]));
      }
      const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(mn[e]), __float_as_uint(mn[e]), false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx[e]), __float_as_uint(mx[e]), false, false);
      mn[e] = first_min(__uint_as_float(a[0]), __uint_as_float(a[1]));
      mx[e] = first_max(__uint_as_float(b[0]), __uint_as_float(b[1]));
    }
    // the entry's min row from the first LPR lanes, its max row from the next
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (DT == SCOUT_BF16) {  // the values came out of bf16 storage, so the upper halves are exact
        const float lo = lane < L::LPR ? mn[2 * i] : mx[2 * i], hi = lane < L::LPR ? mn[2 * i + 1] : mx[2 * i + 1];
        w[i] = (__float_as_uint(lo) >> 16) | (__float_as_uint(hi) & 0xffff0000u);
      } else {
        w[i] = __float_as_uint(lane < L::LPR ? mn[i] : mx[i]);
      }
    }
    if (lane < 2 * L::LPR)
      __builtin_nontemporal_store(w, static_cast<u32x4*>(digest) + ((size_t)pair * D.max_blocks + j) * 2 * L::LPR + lane);
  }
}

// A thread takes 8 channels of a block and walks through its tokens, ROWS of them requested at a time (bf16 sums of
// 400 MB of keys: 92 us instead of 104 with one; fp32 one: d = 128, blocks of 64, 64 MB of keys take 19.6 us with one, 20.5 with two,
// 16.2 with four, but 256 MB in blocks of 16 take 44.1, 44.3 and 47.2, and 128 MB, d = 64, 21.2, 21.3 and 24.3).  This is how
// the sums of mean pooling are made (Sec. 2.2 names mean pooling next to min/max pooling): the digest of a block is the
// sum of its valid keys in binary32, added in token order, one rounding per token, so that the append of a token
// is one addition and gives the bits a rebuild would give; the mean is sum / count where it is used.  And it is how
// the min/max digests of 2 KiB tiles are made: there the join of eight groups of lanes costs digest_kernel more than
// its order of requests gains (bf16, d = 64, blocks of 16, 8 x 8 pairs
// of 16k to 32k tokens: 65 us there, 39 us here).
template <int DT, bool SUM, int ROWS, bool MAY_NT>
__global__ __launch_bounds__(256) void digest_rows_kernel(Dims D, const void* __restrict__ k_blocks, void* __restrict__ digest,
                                                          int nt_limit) {
  constexpr int W = DT == SCOUT_BF16 ? 1 : 2;  // 16-byte words per 8 elements
  const int pair = grid_pair();  // grid (x, Hkv, B)
  const int cpt = D.d / 8;       // 8-channel chunks per token row
  const int j = blockIdx.x * (blockDim.x / cpt) + threadIdx.x / cpt;
  const int c0 = (threadIdx.x % cpt) * 8;
  const int ctx = D.ctx_len[blockIdx.z];
  const bool nt = MAY_NT && keys_exceed_cache(D, nt_limit);
  if (j >= num_blocks(D, ctx)) return;
  const int valid = ctx - j * D.S;
  const u32x4* p = static_cast<const u32x4*>(k_blocks) + (((size_t)pair * D.max_blocks + j) * D.S * cpt + c0 / 8) * W;
  float lo[8], hi[8];  // SUM: lo is the sum
  for (int t0 = 0; t0 < D.S && t0 < valid; t0 += ROWS) {  // ROWS divides S
    u32x4 raw[ROWS][W];  // rows beyond `valid` lie inside the block and are not used
    if (nt) {
      only_here();
#pragma unroll
      for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int w = 0; w < W; ++w) raw[i][w] = __builtin_nontemporal_load(p + (size_t)(t0 + i) * cpt * W + w);
      only_here();
    } else {
#pragma unroll
      for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int w = 0; w < W; ++w) raw[i][w] = p[(size_t)(t0 + i) * cpt * W + w];
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      float x[8];
      load8<DT>(raw[i], 0, x);
      if (t0 + i < valid) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (SUM) {
            lo[e] = t0 + i == 0 ? x[e] : lo[e] + x[e];
          } else {
            lo[e] = t0 + i == 0 ? x[e] : first_min(lo[e], x[e]);
            hi[e] = t0 + i == 0 ? x[e] : first_max(hi[e], x[e]);
          }
        }
      }
    }
  }
  const size_t entry = (size_t)pair * D.max_blocks + j;
  if constexpr (SUM) {
    float4* out = reinterpret_cast<float4*>(static_cast<float*>(digest) + entry * D.d + c0);
    out[0] = make_float4(lo[0], lo[1], lo[2], lo[3]);
    out[1] = make_float4(lo[4], lo[5], lo[6], lo[7]);
  } else {
    static_assert(SUM || DT == SCOUT_BF16, "layout");
    u32x4 a, c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // the values came out of bf16 storage, so the upper halves are exact
      a[i] = (__float_as_uint(lo[2 * i]) >> 16) | (__float_as_uint(lo[2 * i + 1]) & 0xffff0000u);
      c[i] = (__float_as_uint(hi[2 * i]) >> 16) | (__float_as_uint(hi[2 * i + 1]) & 0xffff0000u);
    }
    u32x4* out = static_cast<u32x4*>(digest) + entry * 2 * cpt + c0 / 8;
    __builtin_nontemporal_store(a, out);
    __builtin_nontemporal_store(c, out + cpt);
  }
}

// ------------------------------------------------------------------- score

constexpr int kScoreWaves = 4;      // waves per workgroup

// The score of a block is sum_c P_c*max_j[c] + N_c*min_j[c], with P_c (N_c) the sum over the group's
// query heads of the positive (negative) parts of q[c]: the group is folded before the stream.
//
// Stream layout: ScoreTile.  A lane adds the products of the NL loads of an entry into one partial sum, and only the 8 lanes of an entry remain to be added
// across lanes: three DPP steps.  Where a batch of kScoreBatch loads holds several 8-entry groups,
// the first steps exchange half of the remaining sums each instead of adding all of them everywhere.
// A wave takes one batch, all of it requested at once: many small waves (8192 at 128 pairs x 1024
// blocks, 8 KiB each) measured faster than fewer waves that walk over several batches (13.5 vs 14.5 us
// for 64 MiB).  The loads go through a buffer
// descriptor that ends at the pair's last valid block: blocks beyond it read as zero without touching
// memory, so the issue path has no branches.
//
// The fold of the query group is done once per workgroup (one channel and one sign per thread) and
// handed to the lanes through LDS, while the first digest loads are in flight.  The pointers are
// deliberately not marked restrict: loads that the compiler knows to be invariant float freely, and
// here the order of issue matters (queries first, then batch by batch), because a wait for one load
// is a wait for every load issued before it.
//
// MEAN: the digest entry is one row of binary32 sums of the block's keys (mean pooling) whatever the
// element type of the queries; the score is (sum over heads of q) . sums / count, so there is one
// coefficient vector instead of two and a division by the block's token count at the end.
// AHEAD: the first `ahead` workgroups of a row (ahead_groups) ask for their digests without waiting for the sequence's length,
// a trip to memory in which it would have nothing to do; what lies beyond the last block is dropped afterwards.
//
// NH: query rows that a thread asks for, the group's and, up to 4, 8 or 16, its last one again: narrow loads in front of the
// digests'.  Sixteen for whatever group: 8 sequences x 8 heads of 64 channels, groups of four, 79.4 us a step instead of 78.5, one sequence
// 64.7 and 64.25.  The launch alone, us, sixteen rows and eight: groups of five, bf16, d = 64, 8 pairs x 1024 blocks 3.09 and 2.98,
// 64 x 1024 3.87 and 3.67, d = 128 5.15 and 4.88; groups of eight 3.90 and 3.71, 5.40 and 5.20, fp32, d = 128 11.89 and 11.88.
template <int DT, int DH, bool MEAN, int NH>
__global__ __launch_bounds__(kScoreWaves* kWave) void score_kernel(
    Dims D, const void* q, const void* digest, float* scores, uint32_t* arrived, int ahead) {
  using T = ScoreTile<DT, DH, MEAN>;
  constexpr int ESZ = (DT == SCOUT_BF16) ? 2 : 4;  // bytes per query element
  constexpr int EB = T::EB, BLK_PER_WAVE = T::BLOCKS;
  constexpr int NT = kScoreWaves * kWave;
  static_assert(2 * DH <= NT, "layout");

  __shared__ __align__(16) double coef_lds[2][DH];  // [0]: N_c (goes with the min row), [1]: P_c

  const int pair = grid_pair();  // grid (x, Hkv, B)
  const int b = blockIdx.z, g = blockIdx.y;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  auto clear_counter = [&]() { if (arrived != nullptr && blockIdx.x == 0 && threadIdx.x == 0) arrived[pair] = 0; };  // see launch_score
  const int j_wave = (blockIdx.x * kScoreWaves + wave) * BLK_PER_WAVE;
  const bool active = j_wave < D.max_blocks;  // a wave past the row still helps with the fold

  const uint32_t ctx = request_ctx(D, b);  // ahead of the queries: who waits for it does not wait for them
  // the group's queries first: thread t takes channel t % DH, negative (t < DH) or positive parts
  const int fc = threadIdx.x % DH;
  const bool fpos = threadIdx.x >= DH;
  const char* qbase = static_cast<const char*>(q) + (((size_t)b * D.Hq + g * D.G) * DH + fc) * ESZ;
  float qv[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {  // rows beyond the group re-read its last row and are ignored below
    const int hs = h < D.G ? h : D.G - 1;
    if (DT == SCOUT_BF16)
      qv[h] = __uint_as_float((uint32_t) * reinterpret_cast<const uint16_t*>(qbase + (size_t)hs * DH * ESZ) << 16);
    else
      qv[h] = *reinterpret_cast<const float*>(qbase + (size_t)hs * DH * ESZ);
  }

  // (the query loads above do not wait for the sequence's length; this is the first thing that does)
  const bool blind = (int)blockIdx.x < ahead;
  int nb = D.max_blocks;
  if (!blind) nb = num_blocks(D, arrived_ctx(ctx));
  if ((int)blockIdx.x * kScoreWaves * BLK_PER_WAVE >= nb) {
    // the whole workgroup lies beyond the sequence's last block (a ragged batch has many of these):
    // nothing to read, only the row's tail to mark
    const int j = (int)blockIdx.x * kScoreWaves * BLK_PER_WAVE + threadIdx.x;
    if (threadIdx.x < kScoreWaves * BLK_PER_WAVE && j < D.max_blocks) scores[(size_t)pair * D.max_blocks + j] = -INFINITY;
    clear_counter();
    return;
  }
  const char* dpair = static_cast<const char*>(digest) + (size_t)kv_row(D, pair) * D.max_blocks * EB;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(dpair), 0, active ? nb * EB : 0, 0x00020000);
  u32x4 raw[kScoreBatch];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int it = 0; it < kScoreBatch; ++it)
    raw[it] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, j_wave * EB + T::offset(lane, it), 0, 0));
  __builtin_amdgcn_sched_barrier(0);
  if (blind) nb = num_blocks(D, arrived_ctx(ctx));

  {
    double f = 0.0;
#pragma unroll
    for (int h = 0; h < NH; ++h)
      if (h < D.G) f += MEAN ? (double)qv[h] : (double)(fpos ? fmaxf(qv[h], 0.0f) : fminf(qv[h], 0.0f));
    if (threadIdx.x < 2 * DH) coef_lds[fpos ? 1 : 0][fc] = f;  // MEAN: both rows hold the plain sum
  }
  __syncthreads();
  clear_counter();
  double coef[T::NL][T::EPL];
  T::coefficients(coef, coef_lds[0], lane);
  double sc = T::scores(raw, coef, lane);
  const int j = j_wave + T::entry(lane);
  if (T::writer(lane) && j < D.max_blocks) {
    const bool kept = j < D.n_sink || j >= nb - D.n_tail;  // always-kept blocks rank above every score
    if (MEAN) {  // sums -> means: the block's token count (the last block may be partly filled)
      int cnt = arrived_ctx(ctx) - j * D.S;
      cnt = cnt > D.S ? D.S : (cnt < 1 ? 1 : cnt);
      sc = sc / (double)cnt;
    }
    scores[(size_t)pair * D.max_blocks + j] = j < nb ? (kept ? INFINITY : (float)sc) : -INFINITY;
  }
}

// The same stream with an estimate per head instead of their sum: for the maximum over the group's heads, and for a
// selection per query head.  The fold of the group is not possible then: a head's estimate is the sum over channels of
// the larger of q*min and q*max, which is P_h . max + N_h . min with the positive and negative parts of that head's
// queries, a contraction over 2 d elements of an entry, and the binary64 matrix instructions take it: heads are rows,
// digest entries are columns.  On the vector ALU every multiply-add needs a coefficient of its own in a register
// (1 KiB of LDS reads per four of them) and every sum is spread over 8 lanes; here an operand of four heads' coefficients
// serves 16 entries, and a lane ends up with whole sums.
//  * an entry belongs to lane % 16, and lane / 16 says which 16 bytes of each 64-byte piece of it the lane holds: element s
//    of the four lanes is the contraction index of one instruction (any labelling does if both operands agree);
//  * up to eight heads go four at a time (4x4x4, four blocks: the same four heads times four entries each), more than
//    eight through 16x16x4; either leaves the estimate of head 4 * quad + lane / 16 for entry lane % 16 in acc[.][quad];
//  * the coefficients are made once per workgroup, as binary64 in LDS, in the order of use.
// A wave takes 16 entries.  Bound by the matrix cores behind the head of the stream: 64 pairs x 1024 blocks, bf16, d = 128,
// eight heads: the multiply-adds take 4.0 us at the rate of the 4x4x4 (7.9 ns per instruction and SIMD; 16x16x4: 28 ns for
// four times the work).  The launch, us, digests from memory (on the vector ALU in brackets): 10.8 (13.1); 12 heads, through 16x16x4
// with four of its rows repeated, 14.1 (17.4), 4 heads 9.4 (10.2); 8 pairs x 600 blocks 4.4 (6.4), 12 heads 5.4 (8.8); 256 x 1024,
// 12 heads 48.3 (55.0); d = 64, 12 heads 8.6 (10.5), 4 heads 6.0 (6.4); fp32, d = 128, 12 heads 16.8 (21.2), 4 heads 14.7 (15.4); fp32, d = 64,
// 4 heads 8.3 (9.1).  Only where up to four heads find the digests in the caches, as a model of one or two layers may, the vector ALU was
// faster: bf16, d = 128, 64 x 1024 7.9 (7.5), fp32, d = 64 6.7 (5.4), fp32, d = 128, 8 x 600 4.3 (4.0).  32 entries per wave, which
// halves the reads of coefficients, lengthen the chain behind a wave's last load: 10.6 at 64 pairs, 6.2 at 8.
//
// ROWS: every head's estimate goes to a row of its own, scores[B][Hq][max_blocks] (a selection per query head:
// one pass over the KV head's digests serves its G query heads), instead of their maximum into the KV head's row.
typedef __attribute__((ext_vector_type(2))) double f64x2;
typedef __attribute__((ext_vector_type(4))) double f64x4;

template <int DT, int DH>
struct HeadTile {
  static constexpr int ESZ = (DT == SCOUT_BF16) ? 2 : 4;
  static constexpr int EPL = 16 / ESZ;              // elements per 16-byte load
  static constexpr int EB = 2 * DH * ESZ;           // bytes per digest entry
  static constexpr int NU = EB / 64;                // 64-byte pieces per entry: min row, then max row
  static constexpr int BLOCKS = 16;                 // entries per wave
  static constexpr int STEPS = NU * EPL;            // instructions of a contraction
};

// NQ: quads of heads (1, 2, 4); heads beyond G repeat head G - 1, which leaves the maximum as it is.
template <int DT, int DH, int NQ, bool ROWS>
__global__ __launch_bounds__(kScoreWaves* kWave) void score_heads_kernel(Dims D, const void* q, const void* digest,
                                                                         float* scores, uint32_t* arrived, int ahead) {
  using T = HeadTile<DT, DH>;
  constexpr int EPL = T::EPL, EB = T::EB, NU = T::NU, STEPS = T::STEPS;
  constexpr int NT = kScoreWaves * kWave, HEADS = 4 * NQ;
  constexpr bool WIDE = NQ == 4;

  // [step / 2][operand][lane of the operand][step % 2]; an operand of 4x4x4 is the same in its four blocks: 16 lanes
  __shared__ __align__(16) double coef_lds[STEPS * HEADS * 4];
  auto coef_at = [](int h, int u, int kk, int s) {  // head h, piece u, element s of lane / 16 == kk
    const int lane16 = WIDE ? kk * 16 + h : (h >> 2) * 16 + kk * 4 + (h & 3);
    return ((u * EPL + s) / 2 * (HEADS * 4) + lane16) * 2 + (s & 1);
  };

  const int pair = grid_pair();  // grid (x, Hkv, B)
  const int b = blockIdx.z, g = blockIdx.y;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t ctx = request_ctx(D, b);
  const bool blind = (int)blockIdx.x < ahead;  // see score_kernel
  int nb = D.max_blocks;
  if (!blind) nb = num_blocks(D, arrived_ctx(ctx));
  const int j_wave = (blockIdx.x * kScoreWaves + wave) * T::BLOCKS;
  const bool active = j_wave < D.max_blocks;
  const int n_rows = ROWS ? D.G : 1;  // rows of `scores` per pair
  auto clear_counters = [&]() {
    if (arrived != nullptr && blockIdx.x == 0 && (int)threadIdx.x < n_rows) arrived[pair * n_rows + threadIdx.x] = 0;
  };
  if ((int)blockIdx.x * kScoreWaves * T::BLOCKS >= nb) {  // as in score_kernel: only the rows' tails to mark
    for (int t = threadIdx.x; t < kScoreWaves * T::BLOCKS; t += NT) {
      const int j = (int)blockIdx.x * kScoreWaves * T::BLOCKS + t;
      if (j < D.max_blocks)
        for (int r = 0; r < n_rows; ++r) scores[((size_t)pair * n_rows + r) * D.max_blocks + j] = -INFINITY;
    }
    clear_counters();
    return;
  }

  // queries first (see score_kernel for why the order of issue matters); a thread's elements are dealt so that the
  // coefficients a wave writes together lie side by side in LDS
  constexpr int QPT = HEADS * DH / NT;
  static_assert(HEADS * DH % NT == 0 && 4 * EPL * (NU / 2) == DH, "layout");
  auto q_elem = [](int e, int& h, int& p, int& kk, int& s) {
    const int x = e >> 5, s_hi = x % (EPL / 2);
    s = s_hi * 2 + ((e >> 2) & 1);
    kk = (e >> 3) & 3;
    p = x / (EPL / 2) % (NU / 2);  // piece of the row
    h = (x / (EPL / 2) / (NU / 2)) * 4 + (e & 3);
  };
  float qreg[QPT];
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    int h, p, kk, s;
    q_elem(threadIdx.x + i * NT, h, p, kk, s);
    const int hs = h < D.G ? h : D.G - 1;
    qreg[i] = load1<DT>(q, ((size_t)b * D.Hq + g * D.G + hs) * DH + (p * 4 + kk) * EPL + s);
  }
  const char* dpair = static_cast<const char*>(digest) + (size_t)kv_row(D, pair) * D.max_blocks * EB;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(dpair), 0, active ? nb * EB : 0, 0x00020000);
  const int voff0 = (j_wave + (lane & 15)) * EB + (lane >> 4) * 16;
  u32x4 raw[NU];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NU; ++u)  // requested in the order of use
    raw[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff0 + u * 64, 0, 0));
  __builtin_amdgcn_sched_barrier(0);
  if (blind) nb = num_blocks(D, arrived_ctx(ctx));
#pragma unroll
  for (int i = 0; i < QPT; ++i) {
    int h, p, kk, s;
    q_elem(threadIdx.x + i * NT, h, p, kk, s);
    coef_lds[coef_at(h, p, kk, s)] = (double)fminf(qreg[i], 0.0f);
    coef_lds[coef_at(h, p + NU / 2, kk, s)] = (double)fmaxf(qreg[i], 0.0f);
  }
  __syncthreads();
  clear_counters();

  f64x4 acc = (f64x4){0.0, 0.0, 0.0, 0.0};
  const f64x2* coef = reinterpret_cast<const f64x2*>(coef_lds) + (WIDE ? lane : (lane >> 4) * 4 + (lane & 3));
#pragma unroll
  for (int u = 0; u < NU; ++u) {
#pragma unroll
    for (int s2 = 0; s2 < EPL / 2; ++s2) {
      f64x2 cf[WIDE ? 1 : NQ];
#pragma unroll
      for (int o = 0; o < (WIDE ? 1 : NQ); ++o) cf[o] = coef[(u * (EPL / 2) + s2) * (HEADS * 4) + o * 16];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        double x;
        if (DT == SCOUT_BF16) x = (double)(e ? bf16_hi(raw[u][s2 % 4]) : bf16_lo(raw[u][s2 % 4]));
        else x = (double)__uint_as_float(raw[u][(s2 * 2 + e) % 4]);
        if constexpr (WIDE) {
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(cf[0][e], x, acc, 0, 0, 0);
        } else {
#pragma unroll
          for (int o = 0; o < NQ; ++o) acc[o] = __builtin_amdgcn_mfma_f64_4x4x4f64(cf[o][e], x, acc[o], 0, 0, 0);
        }
      }
    }
  }

  const int kk = lane >> 4;  // the head of its quad
  const int j = j_wave + (lane & 15);
  auto value = [&](double est) {  // always-kept blocks rank above every score
    return j < nb ? (j < D.n_sink || j >= nb - D.n_tail ? INFINITY : (float)est) : -INFINITY;
  };
  if constexpr (ROWS) {
#pragma unroll
    for (int o = 0; o < NQ; ++o) {
      const int h = o * 4 + kk;
      if (h < D.G && j < D.max_blocks) scores[((size_t)pair * D.G + h) * D.max_blocks + j] = value(acc[o]);
    }
  } else {
    double best = -INFINITY;
#pragma unroll
    for (int o = 0; o < NQ; ++o) best = acc[o] > best ? acc[o] : best;
    const double o16 = partner_f64<4>(best);
    best = o16 > best ? o16 : best;
    const double o32 = partner_f64<5>(best);
    best = o32 > best ? o32 : best;
    if (kk == 0 && j < D.max_blocks) scores[(size_t)pair * D.max_blocks + j] = value(best);
  }
}

// ------------------------------------------------------------ host launchers

int launch_digest(const Dims& D, int dtype, const void* k_blocks, void* digest, hipStream_t st) {
  if (D.max_blocks == 0 || D.Hkv == 0 || D.B == 0) return SCOUT_OK;
  // Keys beyond what the 256 MiB memory-side cache holds pass by it (non-temporal loads): 400 MB 76 us instead of 85; of
  // 200 MB a part may still be there, and loads that pass by miss it (bf16, d = 64: 44 us instead of 39).  The lengths
  // decide, on the device: rows of 1 GiB that hold 128 MB of keys took 48 us for their sums with loads that pass by, 31 with
  // plain ones.  Rows below the line cannot exceed it and are not looked at.
  constexpr long long kCacheBytes = 256ll << 20;
  const long long token_bytes = (long long)D.B * D.Hkv * D.d * (dtype == SCOUT_BF16 ? 2 : 4);  // one token in every sequence
  const bool nt = token_bytes * D.max_blocks * D.S > kCacheBytes;
  const int nt_limit = (int)(8 * kCacheBytes / token_bytes);  // below 2^24
  // 128-byte token rows are eight groups of lanes to join for each small block: a thread per row chunk is faster
  // (bf16, d = 64: 39.2 against 65 us for blocks of 16, 39.0 against 40.8 us for blocks of 32; blocks of 64 are whole waves' work).
  const bool small_tile = dtype == SCOUT_BF16 && D.d == 64 && D.S <= 32;
  if (D.digest_kind == 1 || small_tile) {
    const int per_wg = 256 / (D.d / 8);
    dim3 grid((D.max_blocks + per_wg - 1) / per_wg, D.Hkv, D.B);
#define SCOUT_DIGEST_ROWS(DT, SUM, ROWS, MAY_NT)                                                                  \
  do {                                                                                                            \
    if (MAY_NT && nt) hipLaunchKernelGGL((digest_rows_kernel<DT, SUM, ROWS, MAY_NT>), grid, dim3(256), 0, st, D, k_blocks, digest, nt_limit); \
    else hipLaunchKernelGGL((digest_rows_kernel<DT, SUM, ROWS, false>), grid, dim3(256), 0, st, D, k_blocks, digest, nt_limit);   \
  } while (0)
    if (D.digest_kind == 0) SCOUT_DIGEST_ROWS(SCOUT_BF16, false, 8, true);
    else if (dtype == SCOUT_BF16) SCOUT_DIGEST_ROWS(SCOUT_BF16, true, 8, true);
    else SCOUT_DIGEST_ROWS(SCOUT_F32, true, 1, false);
#undef SCOUT_DIGEST_ROWS
    return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
  }
#define SCOUT_DIGEST(DT, DH, S_)                                                                                  \
  do {                                                                                                            \
    constexpr int per_wg = 4 * DigestTile<DT, DH, S_>::NBLK;                                                      \
    const dim3 grid((D.max_blocks + per_wg - 1) / per_wg, D.Hkv, D.B);                                            \
    if (nt) hipLaunchKernelGGL((digest_kernel<DT, DH, S_, true>), grid, dim3(256), 0, st, D, k_blocks, digest, nt_limit);   \
    else hipLaunchKernelGGL((digest_kernel<DT, DH, S_, false>), grid, dim3(256), 0, st, D, k_blocks, digest, nt_limit);     \
  } while (0)
#define SCOUT_DIGEST_S(DT, DH)                     \
  do {                                             \
    if (D.S == 16) SCOUT_DIGEST(DT, DH, 16);       \
    else if (D.S == 32) SCOUT_DIGEST(DT, DH, 32);  \
    else SCOUT_DIGEST(DT, DH, 64);                 \
  } while (0)
  if (dtype == SCOUT_BF16 && D.d == 128) SCOUT_DIGEST_S(SCOUT_BF16, 128);
  else if (dtype == SCOUT_BF16) SCOUT_DIGEST(SCOUT_BF16, 64, 64);
  else if (D.d == 128) SCOUT_DIGEST_S(SCOUT_F32, 128);
  else SCOUT_DIGEST_S(SCOUT_F32, 64);
#undef SCOUT_DIGEST_S
#undef SCOUT_DIGEST
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

// Workgroups of each row that ask for their digests before they know the row's length: 128 in all, rounded up to whole ones per row,
// so that at most 256 do (254 of 127 pairs, one per row of 129 to 256 pairs), of 32 KiB each, 64 KiB in score_heads_kernel with fp32, d = 128:
// rows that are much shorter than max_blocks read 8 (16) MiB for nothing at the most.  None beyond 256 pairs, whose launches the trip
// is a small part of.  Steps of four layers: 16 sequences x 8 heads x 1024 blocks 135.9 -> 134.5 us, 8 x 8 104.5 -> 103.4, one sequence 65.7 -> 64.8, 4 x 8 x 4096 111.3 -> 110.5; 256 ragged pairs (two layers) 125.6 -> 125.2.
static int ahead_groups(const Dims& D) {
  const int pairs = D.B * D.Hkv;
  return pairs <= 256 ? (128 + pairs - 1) / pairs : 0;
}

template <bool ROWS>
static int launch_score_heads(const Dims& D, int dtype, const void* q, const void* digest, float* scores,
                              uint32_t* arrived, hipStream_t st) {
  if (D.max_blocks == 0 || D.Hkv == 0 || D.B == 0) return SCOUT_OK;
#define SCOUT_SCORE_HEADS_NQ(DT, DH, NQ)                                                                                    \
  do {                                                                                                                      \
    constexpr int per_wg = HeadTile<DT, DH>::BLOCKS * kScoreWaves;                                                          \
    hipLaunchKernelGGL((score_heads_kernel<DT, DH, NQ, ROWS>), dim3((D.max_blocks + per_wg - 1) / per_wg, D.Hkv, D.B),      \
                       dim3(kScoreWaves * kWave), 0, st, D, q, digest, scores, arrived, ahead_groups(D));                   \
  } while (0)
#define SCOUT_SCORE_HEADS(DT, DH)                              \
  do {                                                         \
    if (D.G <= 4) SCOUT_SCORE_HEADS_NQ(DT, DH, 1);             \
    else if (D.G <= 8) SCOUT_SCORE_HEADS_NQ(DT, DH, 2);        \
    else SCOUT_SCORE_HEADS_NQ(DT, DH, 4);                      \
  } while (0)
  if (dtype == SCOUT_BF16 && D.d == 128) SCOUT_SCORE_HEADS(SCOUT_BF16, 128);
  else if (dtype == SCOUT_BF16) SCOUT_SCORE_HEADS(SCOUT_BF16, 64);
  else if (D.d == 128) SCOUT_SCORE_HEADS(SCOUT_F32, 128);
  else SCOUT_SCORE_HEADS(SCOUT_F32, 64);
#undef SCOUT_SCORE_HEADS
#undef SCOUT_SCORE_HEADS_NQ
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

// A selection per query head (D describes every query head as a pair of its own that shares its KV head's
// rows): the same kernel over the KV heads, every head's estimate to its own row.
static int launch_score_rows(const Dims& D, int dtype, const void* q, const void* digest, float* scores,
                             uint32_t* arrived, hipStream_t st) {
  Dims K = D;
  K.G = D.share;
  K.Hkv = D.Hkv / D.share;
  K.share = 1;
  K.share_magic = 0;
  return launch_score_heads<true>(K, dtype, q, digest, scores, arrived, st);
}

template <bool MEAN>
static int launch_score_sum(const Dims& D, int dtype, const void* q, const void* digest, float* scores,
                            uint32_t* arrived, hipStream_t st) {
  const int entry_bytes = MEAN ? D.d * 4 : 2 * D.d * (dtype == SCOUT_BF16 ? 2 : 4);
  const int lines = entry_bytes / 128;  // 128-byte lines per digest entry
  const int blocks_per_wg = kScoreBatch / lines * 8 * kScoreWaves;
  dim3 grid((D.max_blocks + blocks_per_wg - 1) / blocks_per_wg, D.Hkv, D.B);
  dim3 block(kScoreWaves * kWave);
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return SCOUT_OK;
#define SCOUT_SCORE_NH(DT, DH, NH) \
  hipLaunchKernelGGL((score_kernel<DT, DH, MEAN, NH>), grid, block, 0, st, D, q, digest, scores, arrived, ahead_groups(D))
#define SCOUT_SCORE(DT, DH)                      \
  do {                                           \
    if (D.G <= 4) SCOUT_SCORE_NH(DT, DH, 4);     \
    else if (D.G <= 8) SCOUT_SCORE_NH(DT, DH, 8); \
    else SCOUT_SCORE_NH(DT, DH, 16);             \
  } while (0)
  if (dtype == SCOUT_BF16 && D.d == 128) SCOUT_SCORE(SCOUT_BF16, 128);
  else if (dtype == SCOUT_BF16 && D.d == 64) SCOUT_SCORE(SCOUT_BF16, 64);
  else if (dtype == SCOUT_F32 && D.d == 128) SCOUT_SCORE(SCOUT_F32, 128);
  else if (dtype == SCOUT_F32 && D.d == 64) SCOUT_SCORE(SCOUT_F32, 64);
  else return SCOUT_EUNSUPPORTED;
#undef SCOUT_SCORE
#undef SCOUT_SCORE_NH
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

// arrived: null, or a word per pair that the launch leaves at zero, for the launch that attends to these scores
// (Partials::arrived).
int launch_score(const Dims& D, int dtype, const void* q, const void* digest, float* scores, uint32_t* arrived,
                 hipStream_t st) {
  if (D.digest_kind == 1) return D.group_max ? SCOUT_EUNSUPPORTED : launch_score_sum<true>(D, dtype, q, digest, scores, arrived, st);
  if (D.group_max) return launch_score_heads<false>(D, dtype, q, digest, scores, arrived, st);
  if (D.share > 1) return launch_score_rows(D, dtype, q, digest, scores, arrived, st);
  return launch_score_sum<false>(D, dtype, q, digest, scores, arrived, st);
}

}  // namespace scout
