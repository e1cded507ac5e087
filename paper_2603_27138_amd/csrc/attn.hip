// Block-sparse paged decode attention over the selected GPU-resident blocks
// (Sec. 3.2; Alg. 1 GPUAttn) and the merge of partial results (Alg. 1 Merge).
//
// A partial result of a token set is (o, m, l): m the largest logit, l the sum
// of exp(logit - m), o the weighted value sum.  Partials of disjoint sets
// combine exactly (FlashAttention rescaling), which is used three times: across
// the blocks a wave walks through, across the waves / workgroups that split a
// pair's block list, and finally with the host's partial.
//
// Inside the kernels logits are kept in base-2 units (x * log2(e)), so the
// exponentials are v_exp_f32; m is converted back to natural-log units
// where it leaves the library.
//
// Two kernel families write the same per-split partials into the workspace, both for every supported
// (dtype, d, S):
//   attn_mfma_kernel  the G query heads of a KV head form one MFMA operand (bf16, or fp32 on the fp32
//                     matrix instructions), K and V rows go from HBM straight into MFMA operand
//                     registers (no LDS), in units of 16 tokens.
//   attn_valu_kernel  plain vector ALU; only where the caller asks for it (scout_set_attn_mode).
// combine_kernel folds the splits (and optionally the host partial) together.
#include <type_traits>

#include "score_tile.h"
#include "select.h"

namespace scout {

// bare v_exp_f32: results below 2^-126 flush to zero, which rescaling factors and rounded weights can afford
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float exp2_diff(float a, float b) {
  // 2^(a-b) with the convention 2^(-inf - anything) = 0
  return a == -INFINITY ? 0.0f : fast_exp2(a - b);
}

// ---------------------------------------------------------------- MFMA family

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Pack the low (sel = 0) or high (sel = 1) bf16 of two dwords into one dword:
// result.lo = half(a), result.hi = half(b).  One v_perm_b32: its selector bytes
// 0-3 address the second source operand, 4-7 the first.
__device__ __forceinline__ uint32_t pack_halves(uint32_t a, uint32_t b, int sel) {
  return sel ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
}

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// two binary32 -> one dword of two bf16 (round to nearest even), x in the low half
__device__ __forceinline__ uint32_t cvt_pk_bf16(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
}

// N consecutive channels of a head.  The arrays may start anywhere that an element of theirs may.
template <int N>
struct Channels {
  typedef __attribute__((ext_vector_type(N))) float f;
  typedef f f_any __attribute__((aligned(4)));
  typedef __attribute__((ext_vector_type(N))) uint16_t h;
  typedef h h_any __attribute__((aligned(2)));
};
// Channels per thread in the epilogues of the attention: the weights of the two partials are made once for them.  Two: of four, the
// divisions are a chain that few threads run; of one, every thread makes weights of its own.
constexpr int CH = 2;
typedef Channels<CH>::f fch;

// The host's partial for a thread's channels (mode 2 only); loaded ahead of the point of use so
// that its latency hides behind the fold.
template <int N>
struct HostPart {
  typename Channels<N>::f o;
  float m, l;
};

template <int N>
__device__ __forceinline__ HostPart<N> load_host(const Dims& D, const Epilogue& E, int bh, int c) {
  HostPart<N> hp{};
  hp.m = -INFINITY;
  if (E.mode == 2 && E.host_o != nullptr) {
    hp.m = E.host_m[bh];
    hp.l = E.host_l[bh];
    hp.o = *reinterpret_cast<const typename Channels<N>::f_any*>(E.host_o + (size_t)bh * D.d + c);
  }
  return hp;
}

// Merge of the partial (oa, ma, la) of head bh, channels c on, with the other one: `at` is the place of the channels in `out`.
template <int N>
__device__ __forceinline__ void merge_channels(void* out, int dtype_out, float* lse, size_t at, int bh, int c,
                                               typename Channels<N>::f oa, float ma, float la, const HostPart<N>& other) {
  const float mb = other.m, lb = other.l;
  float ms = -INFINITY;
  if (la > 0.0f) ms = fmaxf(ms, ma);
  if (lb > 0.0f) ms = fmaxf(ms, mb);
  const float wa = la > 0.0f ? la * expf(ma - ms) : 0.0f;
  const float wb = lb > 0.0f ? lb * expf(mb - ms) : 0.0f;
  const float ls = wa + wb;
  typename Channels<N>::f r;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float x = 0.0f;
    if (wa > 0.0f) x += wa * oa[i];
    if (wb > 0.0f) x += wb * other.o[i];
    r[i] = ls > 0.0f ? x / ls : 0.0f;
  }
  if (dtype_out == SCOUT_BF16) {
    typename Channels<N>::h w;
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = (uint16_t)f32_to_bf16_bits(r[i]);
    *reinterpret_cast<typename Channels<N>::h_any*>(static_cast<uint16_t*>(out) + at) = w;
  } else {
    *reinterpret_cast<typename Channels<N>::f_any*>(static_cast<float*>(out) + at) = r;
  }
  if (lse != nullptr && c == 0) lse[bh] = ls > 0.0f ? ms + logf(ls) : -INFINITY;
}

// acc: unnormalised weighted value sums of the channels, l: weight sum, M2: base-2 maximum
template <int N>
__device__ __forceinline__ void finish(const Dims& D, const Epilogue& E, int bh, int c, typename Channels<N>::f acc, float l, float M2,
                                       const HostPart<N>& hp) {
  const float m_nat = M2 * kLn2;  // -inf stays -inf
  typename Channels<N>::f r;
#pragma unroll
  for (int i = 0; i < N; ++i) r[i] = l > 0.0f ? acc[i] / l : 0.0f;
  const size_t at = (size_t)bh * D.d + c;
  if (E.mode == 1) {
    *reinterpret_cast<typename Channels<N>::f_any*>(E.o + at) = r;
    if (c == 0) {
      E.m[bh] = m_nat;
      E.l[bh] = l;
    }
    return;
  }
  merge_channels<N>(E.out, E.dtype_out, E.lse, at, bh, c, r, m_nat, l, hp);
}

// The work of a pair is cut into units of 16 tokens (a block of S tokens is S/16 units; a unit's K
// rows and V rows are contiguous, 4 KiB each at bf16, d = 128).  The pair's units are dealt to the waves that share
// the pair (all waves of all its workgroups) in contiguous ranges whose lengths differ by at most
// one, so no wave waits for a neighbour that got a whole block more.  For each unit:
//   logits^T[token][head] = K[token][:] . Q[head][:]            bf16: d/32 x mfma 16x16x32, fp32: d/4 x mfma 16x16x4
//   online softmax per head (heads live in lane % 16)
//   out^T[dim][head]    += V^T[dim][token] . P^T[token][head]   bf16: d/16 x mfma 16x16x16 per term of a weight (kWeights32),
//                                                               fp32: d/4 x mfma 16x16x4
// Operand layout of the 16x16 MFMAs: lane L supplies, for A, row L%16 and for B, column L%16, the
// contraction elements of group L/16 (8 of them for x32, 4 for x16, 1 for x4); the result has column L%16 and
// rows 4*(L/16)+i.  The contraction index may be labelled freely as long as A and B agree, which
// lets the logits leave the first product in exactly the registers the second one needs: lane L
// ends up with the logits of head L%16 for tokens 4*(L/16) + i (i = 0..3), so the value rows are
// loaded in that same token order.  Element e of a lane's value chunk c feeds product r = c * CPC + e, whose
// output row index R then means channel CPC * (R + 16 * c) + e.
//
// fp32 goes through the fp32 matrix instructions (products and sums in binary32, as on the vector ALU,
// and the softmax weights are not rounded): 2048 matrix cycles per unit of 16 KiB at d = 128 are 8 bytes
// per cycle and SIMD, 2.5 times what HBM delivers, so the pass stays bandwidth-bound.
//
// The waves of a workgroup fold their partials through LDS; with one split per pair the workgroup
// finishes the pair itself (Epilogue modes 1 and 2), so the whole attention is one launch and
// nothing goes through the workspace.

constexpr int kUnitTokens = 16;

typedef __attribute__((ext_vector_type(4))) short s16x4;

// How a unit of (element type DT, head dim DH) lies in the lanes.
template <int DT, int DH>
struct Tile {
  static constexpr int ES = DT == SCOUT_BF16 ? 2 : 4;  // bytes per element
  static constexpr int ROWB = DH * ES;                 // bytes per token row
  static constexpr int UNITB = kUnitTokens * ROWB;     // bytes of K, and of V, per unit
  static constexpr int KL = ROWB / 64;                 // 16-byte K loads per lane: chunk 4 * s + kg of row ln
  static constexpr int CB = ROWB / 16 < 16 ? ROWB / 16 : 16;  // bytes of a lane's value chunk
  static constexpr int VC = ROWB / 16 / CB;            // value chunks per lane and row: chunk ln + 16 * c
  static constexpr int CPC = CB / ES;                  // channels per value chunk
  static constexpr int NR = DH / 16;                   // products (accumulator tiles) of the second contraction
  // channel of accumulator tile r, row index R
  static __device__ __forceinline__ constexpr int channel(int r, int R) { return CPC * (R + 16 * (r / CPC)) + r % CPC; }
};

// Whether the softmax weights enter the second product in binary32: for fp32, and for bf16 with d = 64 (bf16 with d = 128
// rounds them to bf16).  With bf16 values a binary32 weight goes as the sum of three bf16 terms, 24 bits, each multiplied
// with the values on the bf16 matrix instructions.  8 sequences x 8 KV heads with 128 blocks of 16 tokens listed: the
// attention takes 8.7 us, 8.5 with weights of one term, 9.8 through the fp32 matrix instructions, 30 on the vector ALU.
// Error of the outputs against binary64 (2-norm, lists of 64 to 2048 tokens, logits of standard deviation 0.3, 1, 2), three
// terms and vector ALU: 1.07 and 1.34e-7, 1.42 and 1.60e-7, 2.05 and 2.12e-7; one term: 3e-4 to 1.5e-3.  A term may be zero or negative, which
// makes a NaN of an infinite value, so a wave whose sums hold a NaN starts over with the weights whole, through the fp32
// matrix instructions (EXACT): infinite values give what they give everywhere.
template <int DT, int DH>
constexpr bool kWeights32 = DT == SCOUT_F32 || DH == 64;

// The group's queries as operand registers: 16-byte chunk 4 * s + kg of head ln.
template <int DT, int DH>
using QRegs = u32x4[Tile<DT, DH>::KL];

// K and V rows of one unit in MFMA operand registers.
template <int DT, int DH>
struct UnitRegs {
  u32x4 k[Tile<DT, DH>::KL];     // contraction step s: row = token ln, 16-byte chunk 4*s + kg
  u32x4 v[4][Tile<DT, DH>::VC];  // row = token 4*kg + i, chunk ln + 16*c (8-byte chunks use half the register)
};

// One unit, checked: where it starts in the pools (element offset) and how many of its tokens
// count (0 = nothing to read).
struct Entry {
  size_t elem_off;
  int valid;
};

// sel / slot_list point at the pair's list (global memory or LDS); u is wave-uniform.
template <int DH>
__device__ __forceinline__ Entry read_entry(const int32_t* sel, const int32_t* slot_list, int u, int u_end,
                                            int ush, int S, int ctx, long long n_slots, int tile_stride) {
  Entry e{0, 0};
  if (u < u_end) {
    const int i = u >> ush, sub = u - (i << ush);  // ush = log2(units per block)
    const int j = __builtin_amdgcn_readfirstlane(sel[i]);
    const long long slot = __builtin_amdgcn_readfirstlane(slot_list[i]);
    int valid = ctx - j * S - sub * kUnitTokens;
    valid = valid > kUnitTokens ? kUnitTokens : valid;
    if (j >= 0 && valid > 0 && slot >= 0 && slot < n_slots) {
      e.elem_off = (size_t)slot * tile_stride + sub * kUnitTokens * DH;
      e.valid = valid;
    }
  }
  return e;
}

// Request a unit.  The loads go through a buffer descriptor that covers exactly the unit, or nothing
// when the entry is void: then every lane gets zeros without touching memory.  That keeps the issue
// path free of branches, so the compiler can count outstanding loads exactly and a wave can wait for
// one unit while the next ones are still in flight.
template <int DT, int DH>
__device__ __forceinline__ void issue_unit(UnitRegs<DT, DH>& T, const void* __restrict__ k_pool,
                                           const void* __restrict__ v_pool, const Entry& e, int ln, int kg) {
  using L = Tile<DT, DH>;
  const int bytes = e.valid > 0 ? L::UNITB : 0;
  char* kp = static_cast<char*>(const_cast<void*>(k_pool)) + e.elem_off * L::ES;
  char* vp = static_cast<char*>(const_cast<void*>(v_pool)) + e.elem_off * L::ES;
  // Both descriptors stand before the first request.  Left to itself the compiler made the second one between the K and
  // the V requests and spread these over the matrix instructions in front of them: a selection per query head of 512 pairs
  // (64 listed blocks each) took 35.1 us for the attention instead of 33.2, inside a step 37.9 instead of 37.0; 256 ragged pairs 27.6 and 27.2.
  // Other types and head dims gain nothing from it.
  constexpr bool TOGETHER = DT == SCOUT_BF16 && DH == 128;
  if constexpr (TOGETHER) asm volatile("" : "+s"(kp), "+s"(vp));
  const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(kp, 0, bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(vp, 0, bytes, 0x00020000);
  const int koff = ln * L::ROWB + kg * 16;           // row ln, 16-byte chunk 4*s + kg
  const int voff = kg * 4 * L::ROWB + ln * L::CB;    // row 4*kg + i, chunk ln + 16*c
  if constexpr (TOGETHER) __builtin_amdgcn_sched_barrier(0x00A);  // only vector and matrix instructions may pass
#pragma unroll
  for (int s = 0; s < L::KL; ++s)
    T.k[s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(kr, koff + s * 64, 0, 0));
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int c = 0; c < L::VC; ++c) {
      const int off = voff + i * L::ROWB + c * 16 * L::CB;
      if constexpr (L::CB == 16) {
        T.v[i][c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vr, off, 0, 0));
      } else {
        const u32x2 w = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(vr, off, 0, 0));
        T.v[i][c][0] = w[0];
        T.v[i][c][1] = w[1];
      }
    }
}

// Online-softmax state of one wave: head ln, channel Tile::channel(r, 4*kg + i) in acc[r][i].
template <int NR>
struct WaveState {
  f32x4 acc[NR];
  float m, l;
};

// Fold one unit into the wave's state.  `valid` tokens of the unit count (0: the unit is void and
// leaves the state as it is), so this too runs without a data-dependent branch around loads.
// EXACT: see kWeights32.
template <int DT, int DH, bool EXACT>
__device__ __forceinline__ void consume_unit(WaveState<DH / 16>& W, UnitRegs<DT, DH>& T,
                                             const QRegs<DT, DH>& qreg, int valid, float scale2, int kg) {
  using L = Tile<DT, DH>;
  constexpr bool W32 = kWeights32<DT, DH>;
  f32x4 st = (f32x4){0.f, 0.f, 0.f, 0.f};
  if constexpr (DT == SCOUT_BF16) {
    if constexpr (W32) {
      static_assert(L::KL == 2, "layout");
      const f32x4 z = (f32x4){0.f, 0.f, 0.f, 0.f};
      st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.k[0]), as_bf16x8(qreg[0]), z, 0, 0, 0) +
           __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.k[1]), as_bf16x8(qreg[1]), z, 0, 0, 0);
    } else {
#pragma unroll
    for (int s = 0; s < L::KL; ++s)
      st = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.k[s]), as_bf16x8(qreg[s]), st, 0, 0, 0);
    }
  } else {
    // a chain per 8 channels, joined pairwise, as on the vector ALU: of one chain over all channels a large logit's error
    // is what the outputs' error shows (d = 128, logits of standard deviation 2: 6e-7 instead of 2.3e-7, vector ALU 2.4e-7)
    f32x4 part[L::KL];
#pragma unroll
    for (int s = 0; s < L::KL; ++s) {
      f32x4 half[2];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e % 2 == 0) half[e / 2] = (f32x4){0.f, 0.f, 0.f, 0.f};
        half[e / 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(T.k[s][e]), __uint_as_float(qreg[s][e]), half[e / 2], 0, 0, 0);
      }
      part[s] = half[0] + half[1];
    }
#pragma unroll
    for (int n = L::KL / 2; n > 0; n /= 2)
#pragma unroll
      for (int s = 0; s < n; ++s) part[s] += part[s + n];
    st = part[0];
  }
  // st[i] = logit of head ln, token 4*kg + i
  float x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = W32 ? st[i] : st[i] * scale2;
  if (valid < kUnitTokens) {  // wave-uniform and rare: a void unit, or the partly filled last block
                              // of a sequence; tokens beyond `valid` are dropped, their value rows zeroed
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (4 * kg + i >= valid) {
        x[i] = -INFINITY;
#pragma unroll
        for (int c = 0; c < L::VC; ++c) T.v[i][c] = (u32x4){0, 0, 0, 0};
      }
    }
  }
  float bm = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
  bm = max_xor32(max_xor16(bm));  // over the four lanes that share the head
  if (W32) bm *= scale2;
  const float m_new = fmaxf(W.m, bm);
  const float m_sub = m_new == -INFINITY ? 0.0f : m_new;  // nothing seen yet: weights are 2^-inf = 0
  float p[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)  // W32: scaled and shifted in one rounding, and weights below 2^-126 count, as on the vector ALU
    p[i] = W32 ? exp2f(fmaf(x[i], scale2, -m_sub)) : fast_exp2(x[i] - m_sub);
  if (__ballot(m_new != W.m) != 0) {  // some head's maximum moved: rescale what has been gathered
    const float alpha = exp2_diff(W.m, m_new);
    W.l *= alpha;
#pragma unroll
    for (int r = 0; r < L::NR; ++r) W.acc[r] *= alpha;
    W.m = m_new;
  }
  if constexpr (!W32) {
    // weights go into the second product as bf16; sum what is actually used
    const uint32_t p01 = cvt_pk_bf16(p[0], p[1]), p23 = cvt_pk_bf16(p[2], p[3]);
    W.l += (bf16_lo(p01) + bf16_hi(p01)) + (bf16_lo(p23) + bf16_hi(p23));
    const s16x4 preg = __builtin_bit_cast(s16x4, (uint2){p01, p23});
#pragma unroll
    for (int r = 0; r < L::NR; ++r) {
      const uint32_t a01 = pack_halves(T.v[0][0][r >> 1], T.v[1][0][r >> 1], r & 1);
      const uint32_t a23 = pack_halves(T.v[2][0][r >> 1], T.v[3][0][r >> 1], r & 1);
      W.acc[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, (uint2){a01, a23}), preg,
                                                           W.acc[r], 0, 0, 0);
    }
  } else {
    W.l += (p[0] + p[1]) + (p[2] + p[3]);
    if constexpr (DT == SCOUT_BF16 && !EXACT) {
      s16x4 term[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const uint32_t p01 = cvt_pk_bf16(p[0], p[1]), p23 = cvt_pk_bf16(p[2], p[3]);
        term[t] = __builtin_bit_cast(s16x4, (uint2){p01, p23});
        p[0] -= bf16_lo(p01);  // exact
        p[1] -= bf16_hi(p01);
        p[2] -= bf16_lo(p23);
        p[3] -= bf16_hi(p23);
      }
#pragma unroll
      for (int r = 0; r < L::NR; ++r) {
        const uint32_t a01 = pack_halves(T.v[0][0][r >> 1], T.v[1][0][r >> 1], r & 1);
        const uint32_t a23 = pack_halves(T.v[2][0][r >> 1], T.v[3][0][r >> 1], r & 1);
        const s16x4 v = __builtin_bit_cast(s16x4, (uint2){a01, a23});
#pragma unroll
        for (int t = 2; t >= 0; --t) W.acc[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(v, term[t], W.acc[r], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < L::NR; ++r) {
          float v;
          if constexpr (DT == SCOUT_BF16) v = (r & 1) ? bf16_hi(T.v[i][0][r >> 1]) : bf16_lo(T.v[i][0][r >> 1]);
          else v = __uint_as_float(T.v[i][r / 4][r % 4]);
          W.acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, p[i], W.acc[r], 0, 0, 0);
        }
    }
  }
}

// B operand of the first product: Q^T, column = head ln, zero beyond G
template <int DT, int DH>
__device__ __forceinline__ void load_q(QRegs<DT, DH>& qreg, const Dims& D, const void* __restrict__ q, int b,
                                       int g, int ln, int kg) {
  using L = Tile<DT, DH>;
  const int G = D.G;
  const int hsafe = ln < G ? ln : G - 1;
  const char* qrow = static_cast<const char*>(q) + ((size_t)b * D.Hq + g * G + hsafe) * L::ROWB + kg * 16;
#pragma unroll
  for (int s = 0; s < L::KL; ++s) qreg[s] = *reinterpret_cast<const u32x4*>(qrow + s * 64);
  const uint32_t keep = ln < G ? 0xffffffffu : 0u;
#pragma unroll
  for (int s = 0; s < L::KL; ++s) qreg[s] &= keep;
}

// Units in flight per wave: one where a unit is 4 KiB or more of K and of V each; two of the 2 KiB units of
// bf16 with d = 64, which ask for as many bytes.
template <int DT, int DH>
constexpr int unit_depth() { return Tile<DT, DH>::UNITB >= 4096 ? 1 : 2; }

// ---- The fold of a pair's splits by the workgroup that arrives last.
//
// The splits of a pair run on compute units of different XCDs, each with an L2 of its own, so what one leaves for
// another is written through to device memory and read past the caches (agent scope), and a workgroup counts itself as
// arrived only when its stores have been acknowledged.  Nobody waits for anybody: the workgroup that finds itself the
// last one does the rest, the others end.  A launch of its own (combine_kernel) costs a kernel boundary and the trip
// that reads the partials: a step of one sequence (8 pairs x 16 splits, 4 heads) takes 16.1 us with it and 14.0 without, 4
// sequences of 131k tokens (32 x 8, 8 heads) 34.6 and 33.7, 8 of 32k (64 x 4, 4 heads) 23.1 and 22.7.  Where it pays: see
// fold_pays.
constexpr int kAgentScope = 16;  // cache policy sc1 of the buffer instructions

struct SharedPartials {
  __amdgpu_buffer_rsrc_t o, m, l;  // the pair's rows: (split * G + h) * d floats of o, split * G + h of m and l
};

template <int DH>
__device__ __forceinline__ SharedPartials shared_partials(const Partials& P, int pair, int G) {
  const size_t row0 = (size_t)pair * P.nsplit * G;
  const int rows = P.nsplit * G;
  return SharedPartials{__builtin_amdgcn_make_buffer_rsrc(P.o + row0 * DH, 0, rows * DH * 4, 0x00020000),
                        __builtin_amdgcn_make_buffer_rsrc(P.m + row0, 0, rows * 4, 0x00020000),
                        __builtin_amdgcn_make_buffer_rsrc(P.l + row0, 0, rows * 4, 0x00020000)};
}

// CH channels from c on of row `row`; the thread with the first channels stores m and l too.
typedef __attribute__((ext_vector_type(CH))) uint32_t uch;
__device__ __forceinline__ void store_split(const SharedPartials& R, int row, int c, int dh, fch o, float m, float l) {
  static_assert(CH == 2, "one 8-byte store");
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uch, o), R.o, (row * dh + c) * 4, 0, kAgentScope);
  if (c == 0) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m), R.m, row * 4, 0, kAgentScope);
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(l), R.l, row * 4, 0, kAgentScope);
  }
}

// Splits s0, s0 + step, ... of head h, channels c on: four requested at a time.
template <int DH>
__device__ __forceinline__ void gather_splits(const Partials& P, const SharedPartials& R, int G, int h, int c, int s0, int step, fch& o,
                                              float& l, float& M) {
  constexpr int GROUP = 4;
  M = -INFINITY;
  l = 0.0f;
  o = fch{};
  for (; s0 < P.nsplit; s0 += GROUP * step) {
    fch w[GROUP];
    float ms[GROUP], ls[GROUP];
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {  // rows beyond the last split lie outside the descriptors and read as zeros
      const int row = (s0 + j * step) * G + h;
      w[j] = __builtin_bit_cast(fch, __builtin_amdgcn_raw_buffer_load_b64(R.o, (row * DH + c) * 4, 0, kAgentScope));
      ms[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(R.m, row * 4, 0, kAgentScope));
      ls[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(R.l, row * 4, 0, kAgentScope));
    }
    float Mn = M;
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {
      if (s0 + j * step >= P.nsplit) ms[j] = -INFINITY;
      Mn = fmaxf(Mn, ms[j]);
    }
    const float f0 = exp2_diff(M, Mn);
    o *= f0;
    l *= f0;
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {
      if (s0 + j * step < P.nsplit) {
        const float f = exp2_diff(ms[j], Mn);
#pragma unroll
        for (int i = 0; i < CH; ++i) o[i] += f * w[j][i];
        l += f * ls[j];
      }
    }
    M = Mn;
  }
}

// Every thread of the workgroup calls this after its store_split calls.  `flag`: a word of LDS outside smem.
// A thread takes CH channels of a head.  Up to four splits it takes all of them, one trip, and finishes its channels; of more, the
// workgroup's threads take them in `parts`, as many as it has threads and smem areas for (part i: splits i, i + parts, ...), which
// meet in LDS.  hp: the host's partial for the thread's first channels.
template <int DH, int WAVES>
__device__ __forceinline__ void fold_splits(const Dims& D, int b, int g, int pair, const Partials& P, const Epilogue& E,
                                            const HostPart<CH>& hp, float* smem, int* flag) {
  constexpr int ROW = DH + 4, Q = DH / CH;  // Q: threads per head
  constexpr int NT = WAVES * kWave;
  const int G = D.G, wstride = G * ROW + 32, bh0 = b * D.Hq + g * G;
  __builtin_amdgcn_s_waitcnt(0);  // the partial's stores have been acknowledged
  __syncthreads();
  if (threadIdx.x == 0)
    *flag = (int)__hip_atomic_fetch_add(P.arrived + pair, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*flag) != P.nsplit - 1) return;

  const SharedPartials R = shared_partials<DH>(P, pair, G);
  int parts = (int)(((uint32_t)(NT / Q) * P.g_magic) >> 16);  // NT / Q / G
  parts = parts < WAVES ? parts : WAVES;
  parts = parts < P.nsplit ? parts : P.nsplit;
  if (parts <= 1 || P.nsplit <= 4) {
    for (int item = threadIdx.x; item < G * Q; item += NT) {
      const int h = item / Q, c = (item % Q) * CH;
      float M, l;
      fch o;
      gather_splits<DH>(P, R, G, h, c, 0, 1, o, l, M);
      finish<CH>(D, E, bh0 + h, c, o, l, M, item < NT ? hp : load_host<CH>(D, E, bh0 + h, c));
    }
    return;
  }
  const int slab = threadIdx.x / Q;                              // below 16
  const int part = (int)(((uint32_t)slab * P.g_magic) >> 16);    // slab / G
  const int h = slab - part * G, c = (threadIdx.x % Q) * CH;
  float M, l;
  fch o;
  if (part < parts) {
    gather_splits<DH>(P, R, G, h, c, part, parts, o, l, M);
    float* area = smem + (size_t)part * wstride;
    *reinterpret_cast<fch*>(area + h * ROW + c) = o;
    if (c == 0) {
      area[G * ROW + h] = M;
      area[G * ROW + 16 + h] = l;
    }
  }
  __syncthreads();
  if (slab >= G) return;
  M = -INFINITY;
  l = 0.0f;
  o = fch{};
  for (int w = 0; w < parts; ++w) M = fmaxf(M, smem[(size_t)w * wstride + G * ROW + h]);
  for (int w = 0; w < parts; ++w) {
    const float* base = smem + (size_t)w * wstride;
    const float f = exp2_diff(base[G * ROW + h], M);
    const fch x = *reinterpret_cast<const fch*>(base + h * ROW + c);
#pragma unroll
    for (int i = 0; i < CH; ++i) o[i] += f * x[i];
    l += f * base[G * ROW + 16 + h];
  }
  finish<CH>(D, E, bh0 + h, c, o, l, M, hp);
}

// The attention of one workgroup: its share (split) of the pair's list, folded over the waves
// through LDS, then the epilogue.  sel / slot_list: the pair's list in global memory or LDS.
// PRIVATE: the wave holds its own list entries in registers instead (lane j: the entry of the wave's
// j-th unit, units dealt to the pair's waves in stride: v, v + waves, ...), fetched by the wave
// itself in the same trip as the count: no staging through LDS and no barrier before the first tile
// request.  At most 64 units per wave; sel / slot_list are not read.
// FOLD: P.nsplit > 1, and the workgroup of a pair that finishes last folds the pair's partials and applies E itself
// (fold_splits); `flag` is a word of LDS outside smem.
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};

// after_gather: called once the wave has consumed its units, for stores that should not hold up its first request.
template <int DT, int DH, int WAVES, int DEPTH, bool PRIVATE = false, bool FOLD = false, bool STRIDE = false, class After = Nothing>
__device__ __forceinline__ void attend_pair(const Dims& D, int b, int g, int split,
                                            const QRegs<DT, DH>& qreg,
                                            const void* __restrict__ k_pool,
                                            const void* __restrict__ v_pool, long long n_slots,
                                            const int32_t* sel, const int32_t* slot_list, int n, int ctx,
                                            const Partials& P, const Epilogue& E, float* smem, int my_sel = -1,
                                            int my_slot = -1, int* flag = nullptr, After after_gather = After{}) {
  // per wave: [G][DH + 4] floats of o (padded rows), then m[16], l[16]
  using L = Tile<DT, DH>;
  constexpr int ROW = DH + 4;
  const int pair = b * D.Hkv + g;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int ln = lane & 15, kg = lane >> 4;
  const int G = D.G;
  const int wstride = G * ROW + 32;  // floats of LDS per wave

  n = n < 0 ? 0 : (n > D.k ? D.k : n);
  if (n_slots <= 0) n = 0;
  // ctx (the sequence's length) is handed in: read here, after the caller's barrier and its stores, it
  // would be a fresh trip to memory in front of the first tile request
  const float scale2 = D.sm_scale * kLog2e;
  const int S = D.S, ush = D.s_shift - 4;  // a block is 2^ush units of 16 tokens

  // this wave's contiguous share of the pair's units: the first (units mod waves) waves take one unit
  // more than the others.  The quotient comes from a multiplication with a reciprocal made on the host
  // (at most 4096 units over at most 1024 waves: exact); an integer division here delays the first
  // tile request by a noticeable fraction of a microsecond.
  const int n_units = n << ush, n_waves = P.nsplit * WAVES, v = split * WAVES + wave;
  // STRIDE: units v, v + n_waves, ... instead.
  int u0 = v, u1 = n_units, step = n_waves;
  if constexpr (!STRIDE) {
    const int per = P.waves_magic ? (int)__umulhi((uint32_t)n_units, P.waves_magic) : n_units;
    const int extra = n_units - per * n_waves;
    u0 = v * per + (v < extra ? v : extra);
    u1 = u0 + per + (v < extra ? 1 : 0);
    step = 1;
  }

  WaveState<L::NR> W;
  // DEPTH units are kept in flight per wave: the loads of the next ones are issued before a unit is
  // consumed.  Measured at the benchmark shapes, one unit in flight per wave with eight waves per
  // workgroup (64 KiB requested per compute unit at any time) beats two, three and four (17.0, 17.4,
  // 17.7 and 19.0 us for 64.5 MiB of tiles).
  auto gather = [&](auto exact) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < L::NR; ++r) W.acc[r] = (f32x4){0.f, 0.f, 0.f, 0.f};
    W.m = -INFINITY;
    W.l = 0.0f;
    if constexpr (PRIVATE) {
      // unit v + j * n_waves of the pair is this wave's j-th; its list entry sits in lane j
      auto entry = [&](int j, int u) {
        Entry e{0, 0};
        if (u < n_units) {
          const int bj = __builtin_amdgcn_readlane(my_sel, j);
          const long long slot = __builtin_amdgcn_readlane(my_slot, j);
          const int sub = u & ((1 << ush) - 1);
          int valid = ctx - bj * S - sub * kUnitTokens;
          valid = valid > kUnitTokens ? kUnitTokens : valid;
          if (bj >= 0 && valid > 0 && slot >= 0 && slot < n_slots) {
            e.elem_off = (size_t)slot * D.tile_stride + sub * kUnitTokens * DH;
            e.valid = valid;
          }
        }
        return e;
      };
      UnitRegs<DT, DH> buf[DEPTH];
      Entry ent[DEPTH];
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        ent[d] = entry(d, v + d * n_waves);
        issue_unit<DT, DH>(buf[d], k_pool, v_pool, ent[d], ln, kg);
      }
      int j = DEPTH;
      for (int u = v; u < n_units; u += DEPTH * n_waves) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
          const Entry nx = entry(j, u + (d + DEPTH) * n_waves);
          ++j;
          consume_unit<DT, DH, decltype(exact)::value>(W, buf[d], qreg, ent[d].valid, scale2, kg);
          ent[d] = nx;
          issue_unit<DT, DH>(buf[d], k_pool, v_pool, nx, ln, kg);
        }
      }
    } else {
      UnitRegs<DT, DH> buf[DEPTH];
      Entry ent[DEPTH];
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        ent[d] = read_entry<DH>(sel, slot_list, u0 + d * step, u1, ush, S, ctx, n_slots, D.tile_stride);
        issue_unit<DT, DH>(buf[d], k_pool, v_pool, ent[d], ln, kg);
      }
      for (int u = u0; u < u1; u += DEPTH * step) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
          const Entry nx = read_entry<DH>(sel, slot_list, u + (d + DEPTH) * step, u1, ush, S, ctx, n_slots, D.tile_stride);
          consume_unit<DT, DH, decltype(exact)::value>(W, buf[d], qreg, ent[d].valid, scale2, kg);
          ent[d] = nx;
          issue_unit<DT, DH>(buf[d], k_pool, v_pool, nx, ln, kg);
        }
      }
    }
  };
  gather(std::false_type{});
  if constexpr (DT == SCOUT_BF16 && kWeights32<DT, DH>) {
    bool nan = false;
#pragma unroll
    for (int r = 0; r < L::NR; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) nan |= W.acc[r][i] != W.acc[r][i];
    if (__ballot(nan) != 0) gather(std::true_type{});  // see kWeights32
  }
  after_gather();
  f32x4(&acc)[L::NR] = W.acc;
  float m_run = W.m, l_run = W.l;

  // lanes kg = 0..3 of a head saw disjoint tokens under a common maximum
  l_run = sum_xor32(sum_xor16(l_run));

  // CH channels of a head per thread, as many times over as it takes.  The host's partial for the first of them is requested
  // now and used after the fold.
  constexpr int Q = DH / CH, NT = WAVES * kWave;
  const int bh0 = b * D.Hq + g * G;
  const HostPart<CH> hp = load_host<CH>(D, E, bh0 + ((int)threadIdx.x < G * Q ? threadIdx.x / Q : 0), (threadIdx.x % Q) * CH);

  // fold the waves of the workgroup through LDS
  float* wo = smem + (size_t)wave * wstride;
  float* wm = wo + G * ROW;
  float* wl = wm + 16;
  if (ln < G) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // four consecutive accumulator tiles are four consecutive channels
#pragma unroll
      for (int r = 0; r < L::NR; r += 4)
        *reinterpret_cast<float4*>(wo + ln * ROW + L::channel(r, 4 * kg + i)) =
            make_float4(acc[r][i], acc[r + 1][i], acc[r + 2][i], acc[r + 3][i]);
    }
    if (kg == 0) {
      wm[ln] = m_run;
      wl[ln] = l_run;
    }
  }
  __syncthreads();
  const size_t pbase = (size_t)pair * P.nsplit + split;
  for (int item = threadIdx.x; item < G * Q; item += NT) {
    const int h = item / Q, c = (item % Q) * CH;
    float mw[WAVES];
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      mw[w] = smem[(size_t)w * wstride + G * ROW + h];
      M = fmaxf(M, mw[w]);
    }
    fch o{};
    float l = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const float* base = smem + (size_t)w * wstride;
      const float f = exp2_diff(mw[w], M);
      const fch x = *reinterpret_cast<const fch*>(base + h * ROW + c);
#pragma unroll
      for (int i = 0; i < CH; ++i) o[i] += f * x[i];
      l += f * base[G * ROW + 16 + h];
    }
    if constexpr (FOLD) {
      store_split(shared_partials<DH>(P, pair, G), split * G + h, c, DH, o, M, l);
    } else if (E.mode == 0) {
      *reinterpret_cast<fch*>(P.o + (pbase * G + h) * DH + c) = o;
      if (c == 0) {
        P.m[pbase * G + h] = M;
        P.l[pbase * G + h] = l;
      }
    } else {
      finish<CH>(D, E, bh0 + h, c, o, l, M, item < NT ? hp : load_host<CH>(D, E, bh0 + h, c));
    }
  }
  if constexpr (FOLD) fold_splits<DH, WAVES>(D, b, g, pair, P, E, hp, smem, flag);
}

// Which (sequence, KV head, pair, split) a workgroup of the attention kernels works on.  Normally the grid
// is (splits, KV heads, sequences).  With a selection per query head and one workgroup per head, the launcher
// asks for a grid of one dimension instead (REMAP, a kernel instance of its own so that the usual path keeps its
// short head): the heads of a KV head choose overlapping blocks,
// so they get workgroup ids 8 apart, which the dispatcher hands to the same XCD one after the other: what one
// head reads from memory the others find in that XCD's L2 (a layer-step with per-head selection at config 3's
// shape: 96 us instead of 111 us).
template <bool REMAP>
__device__ __forceinline__ void which_pair(const Dims& D, int& b, int& g, int& pair, int& split) {
  b = blockIdx.z;
  g = blockIdx.y;
  pair = grid_pair();
  split = blockIdx.x;
  if constexpr (REMAP) {
    const int L = blockIdx.x, t = L >> 3;
    const int row = ((t / D.share) << 3) | (L & 7);  // the KV head's row; its heads are t % share
    pair = row * D.share + t % D.share;
    b = pair / D.Hkv;
    g = pair - b * D.Hkv;
    split = 0;
  }
}

// True, and the grid to launch, if the pairs that share a row can be placed on one XCD (see which_pair).
static bool xcd_grid(const Dims& D, int nsplit, dim3& grid) {
  const int pairs = D.B * D.Hkv;
  if (D.share > 1 && nsplit == 1 && (pairs / D.share) % 8 == 0) {
    grid = dim3(pairs, 1, 1);
    return true;
  }
  return false;
}

template <int DT, int DH, int WAVES, int DEPTH>
__global__ __launch_bounds__(WAVES* kWave) void attn_mfma_kernel(
    Dims D, const void* __restrict__ q, const void* __restrict__ k_pool,
    const void* __restrict__ v_pool, long long n_slots, const int32_t* __restrict__ sel_gpu,
    const int32_t* __restrict__ slot_gpu, const int32_t* __restrict__ n_gpu, Partials P, Epilogue E) {
  extern __shared__ float smem[];
  int b, g, pair, split;
  which_pair<false>(D, b, g, pair, split);
  const int lane = lane_id();
  // The pair's whole list is copied to LDS by all threads at once, in the same round trip that
  // brings the count and the queries: which entries a wave needs depends on the count, and a
  // second, dependent trip to memory would cost more than the few hundred bytes read in vain.
  int* l_sel = reinterpret_cast<int*>(smem + WAVES * (D.G * (DH + 4) + 32));
  int* l_slot = l_sel + D.k;
  const size_t list0 = (size_t)pair * D.k;
  const int n = n_gpu[pair];
  const int ctx = D.ctx_len[b];
  for (int t = threadIdx.x; t < D.k; t += WAVES * kWave) {
    l_sel[t] = sel_gpu[list0 + t];
    l_slot[t] = slot_gpu[list0 + t];
  }
  QRegs<DT, DH> qreg;
  load_q<DT, DH>(qreg, D, q, b, g, lane & 15, lane >> 4);
  __syncthreads();
  attend_pair<DT, DH, WAVES, DEPTH>(D, b, g, split, qreg, k_pool, v_pool, n_slots, l_sel, l_slot, n, ctx, P, E, smem);
}

// The same attention with the list entries fetched by the waves themselves (see attend_pair, PRIVATE):
// used when no wave can have more than 64 units.  Without the staging of the list through LDS and its
// barrier the first tile request leaves one trip to memory after the wave started: 16.4 us against
// 17.0 us for config 3's 64.5 MiB of tiles (config 2: 10.4 against 10.9, config 5: 30.0 against 30.6).
template <int DT, int DH, int WAVES, bool REMAP>
__global__ __launch_bounds__(WAVES* kWave) void attn_mfma_private_kernel(
    Dims D, const void* __restrict__ q, const void* __restrict__ k_pool,
    const void* __restrict__ v_pool, long long n_slots, const int32_t* __restrict__ sel_gpu,
    const int32_t* __restrict__ slot_gpu, const int32_t* __restrict__ n_gpu, Partials P, Epilogue E) {
  extern __shared__ float smem[];
  int b, g, pair, split;
  which_pair<REMAP>(D, b, g, pair, split);
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const size_t list0 = (size_t)pair * D.k;
  const int n_waves = P.nsplit * WAVES, v = split * WAVES + wave;
  const int e = (v + lane * n_waves) >> (D.s_shift - 4);  // the block of this wave's unit number `lane`
  int my_sel = -1, my_slot = -1;
  if (e < D.k) {
    my_sel = sel_gpu[list0 + e];
    my_slot = slot_gpu[list0 + e];
  }
  const int n = n_gpu[pair];
  const int ctx = D.ctx_len[b];
  QRegs<DT, DH> qreg;
  load_q<DT, DH>(qreg, D, q, b, g, lane & 15, lane >> 4);
  attend_pair<DT, DH, WAVES, unit_depth<DT, DH>(), true>(D, b, g, split, qreg, k_pool, v_pool, n_slots, nullptr, nullptr, n, ctx, P, E, smem,
                              my_sel, my_slot);
}

// A hint from the lists as the caller left them (in a decode loop: the previous step's lists of this
// layer; adjacent decode tokens attend to highly overlapping sets of blocks, Sec. 1).  While the waves of
// a workgroup select, they ask memory for nothing; the unit a wave would start with under the old lists
// is touched just before, one dword of every 64 bytes, so that its rows are on their way from HBM into
// the caches meanwhile (one unit per wave is what memory delivers in that time: touching two measured
// no gain).  A hint is only ever a slot number inside [0, n_slots): whatever the arrays hold, the touch
// stays inside the pools, and its value is never used.  Budgets above 128 blocks take no hint.  (Not in
// step_kernel: its workgroups are at different stages at any time, memory is never idle there, and the
// touch measured no gain: 65.5 against 65.2 us at 256 ragged pairs.)
struct Hint {
  int n_old, s_lo, s_hi;  // the old count; lane l: old slot entries l and 64 + l
};

// Requested in the same trip as whatever else the kernel asks for first.
__device__ __forceinline__ Hint load_hint(const Dims& D, int pair, int lane, const int32_t* slot_gpu,
                                          const int32_t* n_gpu) {
  Hint h{0, -1, -1};
  if (D.k <= 2 * kWave) {
    const size_t row = (size_t)pair * D.k;
    h.n_old = n_gpu[pair];
    h.s_lo = slot_gpu[row + (lane < D.k ? lane : D.k - 1)];
    h.s_hi = slot_gpu[row + (kWave + lane < D.k ? kWave + lane : D.k - 1)];
  }
  return h;
}

// Wave v of the pair's P.nsplit * WAVES waves touches the first unit of its share of the old list.  To be
// issued when the loads whose values are needed next have returned (a wave's loads return in the order
// they were issued, and a touch takes a loaded memory system's full latency).  The touch goes through a
// buffer descriptor that covers the unit, or nothing: no branch, so nothing ever waits for its value.
// The caller keeps tk and tv alive (an empty asm that names them) until its own later loads have returned.
template <int DT, int DH, int WAVES, bool STRIDE>
__device__ __forceinline__ void touch_hint(const Dims& D, const Hint& h, const Partials& P, int v, int lane,
                                           const void* k_pool, const void* v_pool, long long n_slots,
                                           uint32_t& tk, uint32_t& tv) {
  int n = __builtin_amdgcn_readfirstlane(h.n_old);
  n = n < 0 ? 0 : (n > D.k ? D.k : n);
  const int ush = D.s_shift - 4;
  const int n_units = D.k <= 2 * kWave ? n << ush : 0;
  int u0 = v;  // the first unit of this wave's share of the old list
  if constexpr (!STRIDE) {
    const int per = P.waves_magic ? (int)__umulhi((uint32_t)n_units, P.waves_magic) : n_units;
    const int extra = n_units - per * (P.nsplit * WAVES);
    u0 = v * per + (v < extra ? v : extra);
  }
  const int uc = u0 < n_units ? u0 : 0;
  const int e = uc >> ush, sub = uc & ((1 << ush) - 1);
  long long slot = e < kWave ? __builtin_amdgcn_readlane(h.s_lo, e & (kWave - 1))
                             : __builtin_amdgcn_readlane(h.s_hi, e & (kWave - 1));
  const bool ok = u0 < n_units && slot >= 0 && slot < n_slots;
  slot = ok ? slot : 0;
  const size_t off = (size_t)slot * D.tile_stride + sub * kUnitTokens * DH;
  using L = Tile<DT, DH>;
  const int bytes = ok ? L::UNITB : 0;
  char* kp = static_cast<char*>(const_cast<void*>(k_pool)) + off * L::ES;
  char* vp = static_cast<char*>(const_cast<void*>(v_pool)) + off * L::ES;
  const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(kp, 0, bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(vp, 0, bytes, 0x00020000);
  constexpr int kStep = L::UNITB / kWave;  // one dword of every 64 bytes of a 4 KiB unit
  tk = __builtin_amdgcn_raw_buffer_load_b32(kr, lane * kStep, 0, 0);
  tv = __builtin_amdgcn_raw_buffer_load_b32(vr, lane * kStep, 0, 0);
}

// A pair's lists between the selection and the stores: in LDS.  The resident part is what the attention reads; everything
// leaves behind the tiles (after_gather).  Stored in front of the first request the lists held up the workgroup that writes
// them, and with it its pair, by a microsecond.
struct Lists {
  int *sel, *slot, *all, *host;  // D.k words each
  int ng, nh;

  __device__ __forceinline__ Lists(int* lds, int kpad) : sel(lds), slot(lds + kpad), all(lds + 2 * kpad), host(lds + 3 * kpad), ng(0), nh(0) {}

  // of the key array's element r of each lane, as the Selector has them
  template <int WAVES, int KPL>
  __device__ __forceinline__ void fill(Selector<WAVES, KPL>& S, const uint32_t (&key)[KPL], const int (&slots)[KPL], int k_eff) {
    Mask<KPL> chosen{}, gpu;
    if (k_eff > 0) chosen = S.best(key, k_eff, false);
#pragma unroll
    for (int r = 0; r < KPL; ++r) gpu.m[r] = chosen.m[r] & __ballot(slots[r] >= 0);
    ng = S.emit(chosen, gpu, [&](int r, int i, int at, int at_gpu, bool resident) __attribute__((always_inline)) {
      if (resident) {
        sel[at_gpu] = i;
        slot[at_gpu] = slots[r];
      } else {
        host[at - at_gpu] = i;
      }
      all[at] = i;
    });
    nh = k_eff - ng;
  }

  __device__ __forceinline__ void store(const Dims& D, int pair, int k_eff, int n_threads, int32_t* sel_all, int32_t* sel_gpu,
                                        int32_t* slot_gpu, int32_t* n_gpu, int32_t* sel_host, int32_t* n_host) const {
    const size_t out0 = (size_t)pair * D.k;
    for (int t = threadIdx.x; t < D.k; t += n_threads) {
      sel_all[out0 + t] = t < k_eff ? all[t] : -1;
      sel_gpu[out0 + t] = t < ng ? sel[t] : -1;
      slot_gpu[out0 + t] = t < ng ? slot[t] : -1;
      sel_host[out0 + t] = t < nh ? host[t] : -1;
    }
    if (threadIdx.x == 0) {
      n_gpu[pair] = ng;
      n_host[pair] = nh;
    }
  }
};
__host__ __device__ constexpr int lists_lds_ints(int kpad) { return 4 * kpad; }

// Selection and attention of a pair in one launch (the non-pipelined description of Sec. 3.2:
// identify the top-k blocks, then attend to the resident ones).  Every workgroup of the pair
// repeats the cheap selection from the scores (integer work on a few KiB of keys), keeps the
// resident list in LDS and goes straight on to its share of the units; split 0 also writes the
// lists out, because the host needs to know which selected blocks are its own.
// FOLD: several splits per pair, folded in this launch (P.arrived).
// STRIDE: how the units are dealt to the waves (attend_pair).
template <int DT, int DH, int KPL, bool REMAP, bool FOLD, bool STRIDE>
__global__ __launch_bounds__(8 * kWave) void select_attend_kernel(
    Dims D, const void* __restrict__ q, const float* __restrict__ scores,
    const int32_t* __restrict__ table, const void* __restrict__ k_pool,
    const void* __restrict__ v_pool, long long n_slots, int32_t* __restrict__ sel_all,
    int32_t* __restrict__ sel_gpu, int32_t* __restrict__ slot_gpu, int32_t* __restrict__ n_gpu,
    int32_t* __restrict__ sel_host, int32_t* __restrict__ n_host, Partials P, Epilogue E) {
  constexpr int WAVES = 8;
  extern __shared__ float smem[];
  int b, g, pair, split;
  which_pair<REMAP>(D, b, g, pair, split);
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // LDS after the fold area: the lists, the selector's exchange words, the word that fold_splits uses
  const int kpad = (D.k + 3) & ~3;  // keeps what follows 16-byte aligned
  int* l_lists = reinterpret_cast<int*>(smem + WAVES * (D.G * (DH + 4) + 32));
  Lists lists(l_lists, kpad);
  int* l_x = l_lists + lists_lds_ints(kpad);
  int* l_n = l_x + selector_lds_ints<WAVES>();

  const int ctx = D.ctx_len[b];  // once, here: the attention below must not wait for it again
  QRegs<DT, DH> qreg;
  uint32_t touched_k = 0, touched_v = 0;
  int k_eff;

  float sc[KPL];
  int slot[KPL];
  // In the order of use, because a wait for one load is a wait for those before it: what is selected from, the hint, the queries
  // (which the attention needs).  With the queries and the hint in front: 16 sequences of 32k tokens 131.7 us a step instead of 130.2, 8 sequences
  // 101.8 instead of 99.7.
  load_scores<WAVES, KPL>(D, scores, table, pair, wave, lane, sc, slot);
  __builtin_amdgcn_sched_barrier(0);
  const Hint hint = load_hint(D, pair, lane, slot_gpu, n_gpu);
  __builtin_amdgcn_sched_barrier(0);
  load_q<DT, DH>(qreg, D, q, b, g, lane & 15, lane >> 4);
  __builtin_amdgcn_sched_barrier(0);
  Selector<WAVES, KPL> S{l_x, 0, wave};
  S.prepare();
  int nb = (ctx < 0 ? 0 : ctx + D.S - 1) >> D.s_shift;
  nb = nb < D.max_blocks ? nb : D.max_blocks;
  k_eff = D.k < nb ? D.k : nb;
  uint32_t key[KPL];
  mask_keys<WAVES, KPL>(nb, wave, lane, sc, key, slot);
  __builtin_amdgcn_sched_barrier(0);
  touch_hint<DT, DH, WAVES, STRIDE>(D, hint, P, split * WAVES + wave, lane, k_pool, v_pool, n_slots, touched_k, touched_v);
  __builtin_amdgcn_sched_barrier(0);
  lists.fill(S, key, slot, k_eff);
  __syncthreads();
  auto write_lists = [&]() __attribute__((always_inline)) {
    if (split == 0) lists.store(D, pair, k_eff, WAVES * kWave, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host);
  };
  attend_pair<DT, DH, WAVES, unit_depth<DT, DH>(), false, FOLD, STRIDE>(D, b, g, split, qreg, k_pool, v_pool, n_slots, lists.sel, lists.slot, lists.ng, ctx, P,
                                                                       E, smem, -1, -1, l_n, write_lists);
  asm volatile("" ::"v"(touched_k), "v"(touched_v));  // the touches stay loads, their registers reserved until they have returned
}

constexpr int kSmallDigestBytes = 128 << 10, kSmallTokens = 512, kSmallBytes = 288 << 10, kSmallPairs = 1024;  // see step_kernel_small

// The whole layer-step of a pair in one launch (the non-pipelined sequence of Sec. 3.2: score every
// block against its digest, keep the top-k, attend to the resident ones, merge with the host's
// partial), one workgroup per pair, nothing to combine afterwards: where the pairs alone fill the chip, and where a
// pair has so little to read that a second launch costs more than it brings (see step_kernel_supported).
// The workgroup streams the pair's digest rows, keeps the scores as selection
// keys in LDS (they go to global memory only if the caller wants them), selects, and goes on to the
// attention without a second launch or a trip of the scores through HBM.  Min/max
// digests, the group's heads summed.
//
// Scoring is ScoreTile's, as in score_kernel, so a score has the same bits whichever
// kernel made it.  A wave keeps one batch (8 KiB) in flight, the next requested as soon
// as one is scored (two or four in flight measured the same: 62.8, 62.0 against 62.2 us at batch 32).
template <int DT, int DH, int KPL>
__global__ __launch_bounds__(8 * kWave) void step_kernel(
    Dims D, const void* q, const char* digest, const int32_t* __restrict__ table,
    const void* __restrict__ k_pool, const void* __restrict__ v_pool, long long n_slots,
    float* scores, int32_t* __restrict__ sel_all, int32_t* __restrict__ sel_gpu,
    int32_t* __restrict__ slot_gpu, int32_t* __restrict__ n_gpu, int32_t* __restrict__ sel_host,
    int32_t* __restrict__ n_host, Partials P, Epilogue E) {
  using T = ScoreTile<DT, DH, false>;
  constexpr int WAVES = 8;
  extern __shared__ float smem[];
  const int b = blockIdx.z, g = blockIdx.y, pair = grid_pair();
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int kpad = (D.k + 3) & ~3;
  int* l_lists = reinterpret_cast<int*>(smem + WAVES * (D.G * (DH + 4) + 32));
  Lists lists(l_lists, kpad);
  int* l_x = l_lists + lists_lds_ints(kpad);
  uint32_t* l_key = reinterpret_cast<uint32_t*>(l_x + selector_lds_ints<WAVES>());  // [WAVES * 64 * KPL]
  double* coef_lds = reinterpret_cast<double*>(l_key + WAVES * kWave * KPL);    // [2][DH]: N_c, P_c

  // table entries of the elements this thread will hold in the selection: requested first, used last
  const size_t trow = (size_t)kv_row(D, pair) * D.max_blocks;
  int slot[KPL];
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    const int i = (wave * KPL + r) * kWave + lane;
    slot[r] = table[trow + (i < D.max_blocks ? i : D.max_blocks - 1)];
  }
  // the group's queries: thread t < 2 * DH folds channel t % DH, negative (t < DH) or positive parts
  const int fc = threadIdx.x & (DH - 1);
  const bool fpos = threadIdx.x >= DH;
  const size_t q0 = ((size_t)b * D.Hq + g * D.G) * DH + fc;
  float qv[16];
  if (threadIdx.x < 2 * DH) {
#pragma unroll
    for (int h = 0; h < 16; ++h) qv[h] = load1<DT>(q, q0 + (size_t)(h < D.G ? h : D.G - 1) * DH);
  }
  const char* dpair = digest + trow * T::EB;
  auto load_batch = [&](u32x4(&dst)[kScoreBatch], int batch, int limit) {  // of the row's first `limit` entries; beyond: reads zeros
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(dpair), 0, limit * T::EB, 0x00020000);
    const int base = (batch * T::BLOCKS < limit ? batch * T::BLOCKS : limit) * T::EB;
#pragma unroll
    for (int it = 0; it < kScoreBatch; ++it)
      dst[it] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, base + T::offset(lane, it), 0, 0));
  };
  // In short rows the first batch does not wait for the sequence's length, a trip to memory (entries beyond the last block are
  // dropped when they are scored): a step of 16 pairs of 64 fp32 blocks with an append 17.65 -> 17.4 us a layer.  Long rows, and
  // rows of many pairs, might be read for nothing, and gain nothing: 64.2 and 64.2 us for 256 pairs of 2048 blocks, 512 pairs
  // of up to 250 blocks 82.9 and 83.3.
  u32x4 raw[kScoreBatch];
  int limit = D.max_blocks;
  if (D.max_blocks * T::EB > kSmallDigestBytes || D.B * D.Hkv > 256) limit = num_blocks_of(D, b);
  load_batch(raw, wave, limit);
  Selector<WAVES, KPL> S{l_x, 0, wave};
  S.prepare();

  if (threadIdx.x < 2 * DH) {
    double f = 0.0;
#pragma unroll
    for (int h = 0; h < 16; ++h)
      if (h < D.G) f += (double)(fpos ? fmaxf(qv[h], 0.0f) : fminf(qv[h], 0.0f));
    coef_lds[(fpos ? DH : 0) + fc] = f;
  }
  const int ctx = D.ctx_len[b], nb = num_blocks(D, ctx);
  const int n_batches = (nb + T::BLOCKS - 1) / T::BLOCKS;
  // rows of the key array that no batch will write
  for (int i = n_batches * T::BLOCKS + threadIdx.x; i < WAVES * kWave * KPL; i += WAVES * kWave) l_key[i] = 0u;
  __syncthreads();
  double coef[T::NL][T::EPL];
  T::coefficients(coef, coef_lds, lane);

  const size_t srow = (size_t)pair * D.max_blocks;
  // scores of the blocks of one batch from its eight loads; a batch beyond the last one holds zeros
  // and only marks rows beyond the sequence
  auto score_batch = [&](const u32x4(&cur)[kScoreBatch], int batch) {
    const double sc = T::scores(cur, coef, lane);
    const int j = batch * T::BLOCKS + T::entry(lane);
    if (T::writer(lane)) {
      const bool kept = j < D.n_sink || j >= nb - D.n_tail;  // always-kept blocks rank above every score
      const float val = j < nb ? (kept ? INFINITY : (float)sc) : -INFINITY;
      if (j < WAVES * kWave * KPL) l_key[j] = j < nb ? score_key(val) : 0u;
      if (scores != nullptr && j < D.max_blocks) scores[srow + j] = val;
    }
  };
  for (int batch = wave; batch < n_batches; batch += WAVES) {
    score_batch(raw, batch);
    load_batch(raw, batch + WAVES, nb);
  }
  if (scores != nullptr)  // the row's tail beyond the last batch
    for (int j = n_batches * T::BLOCKS + threadIdx.x; j < D.max_blocks; j += WAVES * kWave) scores[srow + j] = -INFINITY;

  QRegs<DT, DH> qreg;
  load_q<DT, DH>(qreg, D, q, b, g, lane & 15, lane >> 4);
  __syncthreads();

  const int k_eff = D.k < nb ? D.k : nb;
  uint32_t key[KPL];
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    const int i = (wave * KPL + r) * kWave + lane;
    key[r] = l_key[i];  // 0 beyond nb
    slot[r] = i < nb ? slot[r] : -1;
  }
  lists.fill(S, key, slot, k_eff);
  __syncthreads();
  auto write_lists = [&]() __attribute__((always_inline)) {
    lists.store(D, pair, k_eff, WAVES * kWave, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host);
  };
  attend_pair<DT, DH, WAVES, unit_depth<DT, DH>()>(D, b, g, 0, qreg, k_pool, v_pool, n_slots, lists.sel, lists.slot, lists.ng, ctx, P, E,
                                                   smem, -1, -1, nullptr, write_lists);
}

// ---------------------------------------------------------------- VALU family

constexpr int kValuHeads = 4;  // query heads per wave

// One wave per (pair, split, chunk of kValuHeads heads).  A token row is spread
// over LPT = DH/8 lanes (8 channels each); the 64/LPT lane groups take different
// tokens of a block and each keeps an online-softmax stream of its own, so the
// block loop needs no cross-group traffic; the streams are folded at the end.
template <int DT, int DH>
__global__ __launch_bounds__(kWave) void attn_valu_kernel(
    Dims D, const void* __restrict__ q, const void* __restrict__ k_pool,
    const void* __restrict__ v_pool, long long n_slots, const int32_t* __restrict__ sel_gpu,
    const int32_t* __restrict__ slot_gpu, const int32_t* __restrict__ n_gpu, Partials P) {
  constexpr int LPT = DH / 8;      // lanes per token
  constexpr int TPW = kWave / LPT; // tokens per wave pass
  const int pair = blockIdx.y, split = blockIdx.x, h0 = blockIdx.z * kValuHeads;
  const int b = pair / D.Hkv, g = pair % D.Hkv;
  const int lane = lane_id();
  const int tl = lane / LPT, c0 = (lane % LPT) * 8;
  const int G = D.G;
  const int nh = (G - h0) < kValuHeads ? (G - h0) : kValuHeads;

  int n = n_gpu[pair];
  n = n < 0 ? 0 : (n > D.k ? D.k : n);
  const int ctx = D.ctx_len[b];
  const float scale2 = D.sm_scale * kLog2e;

  float qv[kValuHeads][8];
#pragma unroll
  for (int h = 0; h < kValuHeads; ++h) {
    if (h < nh) {
      load8<DT>(q, ((size_t)b * D.Hq + g * G + h0 + h) * DH + c0, qv[h]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) qv[h][i] = 0.0f;
    }
  }
  float m_run[kValuHeads], l_run[kValuHeads], o[kValuHeads][8];
#pragma unroll
  for (int h = 0; h < kValuHeads; ++h) {
    m_run[h] = -INFINITY;
    l_run[h] = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[h][i] = 0.0f;
  }

  for (int i = split; i < n; i += P.nsplit) {
    const int j = sel_gpu[(size_t)pair * D.k + i];
    const long long slot = slot_gpu[(size_t)pair * D.k + i];
    int valid = ctx - j * D.S;
    valid = valid > D.S ? D.S : valid;
    if (j < 0 || valid <= 0 || slot < 0 || slot >= n_slots) continue;
    const size_t tile = (size_t)slot * D.tile_stride;
    for (int t0 = 0; t0 < D.S; t0 += TPW) {
      const int t = t0 + tl;
      const bool live = t < valid;
      float kx[8], vx[8];
      if (live) {
        load8<DT>(k_pool, tile + (size_t)t * DH + c0, kx);
        load8<DT>(v_pool, tile + (size_t)t * DH + c0, vx);
      } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) kx[c] = vx[c] = 0.0f;
      }
#pragma unroll
      for (int h = 0; h < kValuHeads; ++h) {
        float dot = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) dot = fmaf(qv[h][c], kx[c], dot);
#pragma unroll
        for (int off = 1; off < LPT; off <<= 1) dot += __shfl_xor(dot, off);
        if (live) {
          const float x = dot * scale2;
          const float m_new = fmaxf(m_run[h], x);
          const float a = exp2_diff(m_run[h], m_new);
          const float pw = exp2f(x - m_new);
          l_run[h] = l_run[h] * a + pw;
#pragma unroll
          for (int c = 0; c < 8; ++c) o[h][c] = fmaf(pw, vx[c], o[h][c] * a);
          m_run[h] = m_new;
        }
      }
    }
  }

  // fold the TPW token streams of the wave
#pragma unroll
  for (int h = 0; h < kValuHeads; ++h) {
#pragma unroll
    for (int off = LPT; off < kWave; off <<= 1) {
      const float m2 = __shfl_xor(m_run[h], off), l2 = __shfl_xor(l_run[h], off);
      const float M = fmaxf(m_run[h], m2);
      const float fa = exp2_diff(m_run[h], M), fb = exp2_diff(m2, M);
      l_run[h] = l_run[h] * fa + l2 * fb;
#pragma unroll
      for (int c = 0; c < 8; ++c) o[h][c] = o[h][c] * fa + __shfl_xor(o[h][c], off) * fb;
      m_run[h] = M;
    }
  }
  if (tl == 0) {
    const size_t pbase = (size_t)pair * P.nsplit + split;
#pragma unroll
    for (int h = 0; h < kValuHeads; ++h) {
      if (h < nh) {
        float* dst = P.o + (pbase * G + h0 + h) * DH + c0;
        *reinterpret_cast<float4*>(dst) = make_float4(o[h][0], o[h][1], o[h][2], o[h][3]);
        *reinterpret_cast<float4*>(dst + 4) = make_float4(o[h][4], o[h][5], o[h][6], o[h][7]);
        if (c0 == 0) {
          P.m[pbase * G + h0 + h] = m_run[h];
          P.l[pbase * G + h0 + h] = l_run[h];
        }
      }
    }
  }
}

// ------------------------------------------------------- combine and merge

// Fold the nsplit partials of every (sequence, query head), then export the GPU
// partial or go straight on to the merge with the host's partial (Epilogue modes
// 1 and 2).  One workgroup of d threads per head.
template <int GROUP>
__global__ void combine_kernel(Dims D, Partials P, Epilogue E) {
  // grid (G, Hkv, B): head within the group, KV head, sequence
  const int h = blockIdx.x;
  const int pair = grid_pair(), bh = pair * D.G + h;
  const int c = threadIdx.x;
  const size_t p0 = (size_t)pair * P.nsplit;
  const HostPart<1> hp = load_host<1>(D, E, bh, c);
  // one pass with a running maximum, GROUP splits at a time: every load of a group is independent
  // of the others, so a group costs one trip to memory (GROUP covers the split count where it can)
  float M = -INFINITY, acc = 0.0f, l = 0.0f;
  for (int s0 = 0; s0 < P.nsplit; s0 += GROUP) {
    float ms[GROUP], ls[GROUP], os[GROUP];
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {
      const int sp = s0 + j < P.nsplit ? s0 + j : P.nsplit - 1;
      const size_t r = (p0 + sp) * D.G + h;
      ms[j] = P.m[r];
      ls[j] = P.l[r];
      os[j] = P.o[r * D.d + c];
    }
    float Mn = M;
#pragma unroll
    for (int j = 0; j < GROUP; ++j)
      if (s0 + j < P.nsplit) Mn = fmaxf(Mn, ms[j]);
    const float f0 = exp2_diff(M, Mn);
    acc *= f0;
    l *= f0;
#pragma unroll
    for (int j = 0; j < GROUP; ++j) {
      if (s0 + j < P.nsplit) {
        const float f = exp2_diff(ms[j], Mn);
        acc += f * os[j];
        l += f * ls[j];
      }
    }
    M = Mn;
  }
  finish<1>(D, E, bh, c, acc, l, M, hp);
}

// Stand-alone merge of two partials given in natural-log units (Alg. 1 Merge).
template <int DT_OUT>
__global__ void merge_kernel(Dims D, const float* __restrict__ o_a, const float* __restrict__ m_a,
                             const float* __restrict__ l_a, const float* __restrict__ o_b,
                             const float* __restrict__ m_b, const float* __restrict__ l_b,
                             void* __restrict__ out, float* __restrict__ lse) {
  const int bh = blockIdx.x, c = threadIdx.x;
  const size_t at = (size_t)bh * D.d + c;
  HostPart<1> b{};
  b.m = -INFINITY;
  if (o_b != nullptr) {
    b.m = m_b[bh];
    b.l = l_b[bh];
    b.o = o_b[at];
  }
  merge_channels<1>(out, DT_OUT, lse, at, bh, c, o_a[at], m_a[bh], l_a[bh], b);
}

// ------------------------------------------------------------ host launchers

size_t mfma_smem_bytes(const Dims& D, int waves) {
  return (size_t)waves * (D.G * (D.d + 4) + 32) * sizeof(float);
}

// RUN(DT, DH) for the problem's element type and head dim
#define SCOUT_BY_TYPE(dtype, d, RUN)                              \
  do {                                                            \
    if ((dtype) == SCOUT_BF16 && (d) == 128) RUN(SCOUT_BF16, 128);     \
    else if ((dtype) == SCOUT_BF16 && (d) == 64) RUN(SCOUT_BF16, 64);  \
    else if ((dtype) == SCOUT_F32 && (d) == 128) RUN(SCOUT_F32, 128);  \
    else if ((dtype) == SCOUT_F32 && (d) == 64) RUN(SCOUT_F32, 64);    \
    else return SCOUT_EUNSUPPORTED;                               \
  } while (0)

// family 2: MFMA kernel with `waves` waves per workgroup (8 or 16); family 1: vector ALU.
// E.mode != 0 requires P.nsplit == 1 and family 2 (the workgroup finishes the pair itself).
int launch_attn(const Dims& D, int dtype, int family, int waves, const void* q, const void* k_pool,
                const void* v_pool, long long n_slots, const int32_t* sel_gpu,
                const int32_t* slot_gpu, const int32_t* n_gpu, Partials P, Epilogue E, hipStream_t st) {
  const int pairs = D.B * D.Hkv;
  if (pairs == 0) return SCOUT_OK;
  if (family == 2) {
    dim3 grid(P.nsplit, D.Hkv, D.B), block(waves * kWave);
    const size_t lds = mfma_smem_bytes(D, waves) + 2 * (size_t)D.k * sizeof(int);
    // units in flight per wave: few.  Requests that only queue in the memory system buy nothing (a
    // compute unit's loads return in the order they were issued), and fewer registers leave room for
    // the next workgroup to start its head while this one folds.
    const long long units_per_wave = (((long long)D.k * (D.S / kUnitTokens)) + P.nsplit * waves - 1) / (P.nsplit * waves);
    const bool few = waves == 8 && units_per_wave <= 64;
    const bool remap = few && xcd_grid(D, P.nsplit, grid);
    if (waves != 4 && waves != 8 && waves != 16) return SCOUT_EINVAL;
#define SCOUT_ATTN(KERNEL, LDS)                                                                                     \
  hipLaunchKernelGGL(KERNEL, grid, block, LDS, st, D, q, k_pool, v_pool, n_slots, sel_gpu, slot_gpu, n_gpu, P, E)
#define SCOUT_ATTN_TYPE(DT, DH)                                                            \
  do {                                                                                     \
    if (remap) SCOUT_ATTN((attn_mfma_private_kernel<DT, DH, 8, true>), mfma_smem_bytes(D, 8));     \
    else if (few) SCOUT_ATTN((attn_mfma_private_kernel<DT, DH, 8, false>), mfma_smem_bytes(D, 8)); \
    else if (waves == 16) SCOUT_ATTN((attn_mfma_kernel<DT, DH, 16, 1>), lds);              \
    else if (waves == 8) SCOUT_ATTN((attn_mfma_kernel<DT, DH, 8, 1>), lds);                \
    else SCOUT_ATTN((attn_mfma_kernel<DT, DH, 4, 2>), lds);                                \
  } while (0)
    SCOUT_BY_TYPE(dtype, D.d, SCOUT_ATTN_TYPE);
#undef SCOUT_ATTN_TYPE
#undef SCOUT_ATTN
  } else {
    if (E.mode != 0) return SCOUT_EINVAL;
    dim3 grid(P.nsplit, pairs, (D.G + kValuHeads - 1) / kValuHeads), block(kWave);
#define SCOUT_VALU(DT, DH)                                                                                             \
  hipLaunchKernelGGL((attn_valu_kernel<DT, DH>), grid, block, 0, st, D, q, k_pool, v_pool, n_slots, sel_gpu, slot_gpu, \
                     n_gpu, P)
    SCOUT_BY_TYPE(dtype, D.d, SCOUT_VALU);
#undef SCOUT_VALU
  }
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

// Whether the last workgroup of a pair folds its splits, or a launch of its own does.  One workgroup folds nsplit * G * d
// floats where combine_kernel has one per head, so it does not pay for many heads and few splits.  A step of two layers, us, fold in the launch
// and in one of its own, pairs x splits of 512 blocks: bf16, d = 128, 4 heads 184 x 2 78.2 and 79.6; 8 heads 64 x 4 34.65 and 37.3,
// 96 x 3 53.4 and 54.3, 184 x 2 80.3 and 82.0; 16 heads 64 x 4 39.9 and 40.0, 96 x 3 58.5 and 58.2, 128 x 2 57.3 and 57.0, 184 x 2 87.1 and
// 85.4.  d = 64, 16 heads: 128 x 2 36.5 and 39.0, 184 x 2 49.5 and 51.2.  fp32, d = 128, 256 blocks: 8 heads 128 x 2 90.7 and 94.0, 184 x 2 146.7 and
// 147.2; 16 heads 64 x 4 59.8 and 60.8.
bool fold_pays(const Dims& D, int nsplit) { return D.G * D.d <= 1024 || nsplit >= 4; }

bool select_attend_supported(const Dims& D) { return D.max_blocks <= 8 * kWave * 16; }

// Selection fused into the head of the MFMA attention kernel (8 waves per workgroup).
int launch_select_attend(const Dims& D, int dtype, const void* q, const float* scores, const int32_t* table,
                         const void* k_pool, const void* v_pool, long long n_slots, int32_t* sel_all,
                         int32_t* sel_gpu, int32_t* slot_gpu, int32_t* n_gpu, int32_t* sel_host,
                         int32_t* n_host, Partials P, Epilogue E, hipStream_t st) {
  const int pairs = D.B * D.Hkv;
  if (pairs == 0) return SCOUT_OK;
  dim3 grid(P.nsplit, D.Hkv, D.B);
  const bool remap = xcd_grid(D, P.nsplit, grid);
  // In stride where heads that share blocks run side by side, so that they ask for a shared block at about the same time
  // (512 heads: 137 instead of 172 MB from HBM, 125 distinct), and from 8 splits on, where a wave has a unit or two: which units
  // a workgroup touches and takes then hardly depends on the list's length, so the hint lands in the right L2 (4 sequences of
  // 131k tokens, 8 splits: 113.5 -> 111.5 us a step of four layers; one sequence, 16 splits: 66.5 -> 66.0).  With fewer splits neighbouring units
  // stay with one wave: 4 splits 105.0, in stride 105.4; 2 splits 136.3 to 137.2 and 136.6 to 137.9 (box to box).
  const bool stride = P.nsplit >= 8;
  const size_t lds = mfma_smem_bytes(D, 8) + (lists_lds_ints((D.k + 3) & ~3) + selector_lds_ints<8>() + (size_t)4) * sizeof(int);
#define SCOUT_SA_RUN(DT, DH, KPL, REMAP, FOLD, STRIDE)                                                                      \
  hipLaunchKernelGGL((select_attend_kernel<DT, DH, KPL, REMAP, FOLD, STRIDE>), grid, dim3(8 * kWave), lds, st, D, q, scores, \
                     table, k_pool, v_pool, n_slots, sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, P, E)
#define SCOUT_SA(DT, DH, KPL)                                                                \
  do {                                                                                       \
    if (remap) SCOUT_SA_RUN(DT, DH, KPL, true, false, true);                                 \
    else if (P.arrived != nullptr && stride) SCOUT_SA_RUN(DT, DH, KPL, false, true, true);   \
    else if (P.arrived != nullptr) SCOUT_SA_RUN(DT, DH, KPL, false, true, false);            \
    else SCOUT_SA_RUN(DT, DH, KPL, false, false, false);                                     \
  } while (0)
  // All eight waves share the keys: measured faster than one wave selecting alone while seven wait
  // (46.9 vs 44.1 us per step at 1024 blocks per pair), a lone wave issues too slowly.  Eight more waves that leave after the
  // selection cost more than they bring (32 pairs x 8 of 4096 blocks: 30.0 us a step instead of 29.3).  Sizes in between
  // because a key costs whether it is there or not, and a growing sequence has one block more than a power of two.  A step of groups
  // of four, us, without the sizes in between and with them: 3 keys, 64 pairs of 1025 blocks 18.5 and 18.3, of 1500 20.5 and 20.1; 6 keys, 8
  // of 2500 14.6 and 14.1, 64 of 2500 26.6 and 26.0; 12 keys, 8 of 5000 17.9 and 16.2, 32 of 4097 26.5 and 25.4, 64 of 6100 45.9 and 44.9; 192 pairs
  // of 1500, one workgroup each, 34.9 and 35.1.
  const int per_lane = (D.max_blocks + 8 * kWave - 1) / (8 * kWave);
#define SCOUT_SA_TYPE(DT, DH)                      \
  do {                                             \
    if (per_lane <= 2) SCOUT_SA(DT, DH, 2);        \
    else if (per_lane <= 3) SCOUT_SA(DT, DH, 3);   \
    else if (per_lane <= 4) SCOUT_SA(DT, DH, 4);   \
    else if (per_lane <= 6) SCOUT_SA(DT, DH, 6);   \
    else if (per_lane <= 8) SCOUT_SA(DT, DH, 8);   \
    else if (per_lane <= 12) SCOUT_SA(DT, DH, 12); \
    else if (per_lane <= 16) SCOUT_SA(DT, DH, 16); \
    else return SCOUT_EUNSUPPORTED;                \
  } while (0)
  SCOUT_BY_TYPE(dtype, D.d, SCOUT_SA_TYPE);
#undef SCOUT_SA_TYPE
#undef SCOUT_SA
#undef SCOUT_SA_RUN
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

static bool step_kernel_takes(const Dims& D) {
  // (with a selection per query head the scoring pass of its own serves the G heads of a row in one reading)
  return D.digest_kind == 0 && D.group_max == 0 && D.share == 1;
}

// Pairs that alone fill the chip.  One workgroup streams its pair's whole digest row: worth it while a row is short
// enough that one long sequence among short ones cannot hold the launch up for long (2048 blocks = 1 MiB of digest:
// 256 ragged pairs 63.7 us against 65.4 in two launches, 256 equal ones 79.7 and 81.0; of 2049 blocks, which need the next
// size of the key array, 66 and 63).  Pairs beyond one per compute unit start when others end, and a long row then ends
// last: 384 ragged pairs of 1024 blocks 69.0 against 73.7, of 2048 blocks 105.0 against 96.6 (equal ones 127.6 and 120.2).
bool step_kernel_supported(const Dims& D, int dtype) {
  return step_kernel_takes(D) && dtype == SCOUT_BF16 && D.d == 128 && D.max_blocks <= (D.B * D.Hkv <= 256 ? 2048 : 1024);
}

// Pairs with so little to read that one workgroup is done with it before the second launch of a split pair has begun:
// at most 128 KiB of digests, 512 listed tokens (four units per wave) and 288 KiB of both.
// Measured, a layer, one launch against scoring plus split attention, three quarters of the list resident: fp32, d = 64,
// 1 pair of 128 blocks of 16 with k = 16: 9.2 against 11.3 us; bf16, d = 64, 64 pairs of 512 blocks with k = 32: 12.3 against 13.6; bf16,
// d = 128, 64 pairs of 256 blocks of 16 with k = 16 (256 KiB): 12.9 against 13.7; with 32 units per pair (16 KiB of
// digests, 272 KiB) 11.2 against 12.8, 64 KiB of digests (320 KiB) 13.6 against 13.7, 128 KiB 14.9 against 14.2; fp32,
// d = 128, 16 units (288 KiB) 13.2 against 14.4, 32 units 16.1 against 16.1 and 18.8 against 16.7.  Up to 1024 pairs this
// holds throughout (1024 pairs: 32.4 and 39.8, 41.9 and 47.0, 43.8 and 50.2, 55.9 and 56.3).  With more the workgroups come in many
// rounds and the attention's part has fewer waves in flight than in a kernel of its own, so it is right only where the digests are
// half of the tiles or more (2 * max_blocks >= k * S): fp32, d = 128, 32 blocks and 16 units, 1536 pairs 92.1 against 86.3; bf16,
// d = 64, 128 blocks and 32 units, 4096 pairs 140.6 and 133.4; 512 blocks and 32 units 188.9 and 202.2; 256 and 16 133.9 and 138.9.
bool step_kernel_small(const Dims& D, int dtype) {
  const int row_bytes = 2 * D.d * (dtype == SCOUT_BF16 ? 2 : 4);  // of a token's K and V, and of a digest entry
  return step_kernel_takes(D) && D.max_blocks * row_bytes <= kSmallDigestBytes && D.k * D.S <= kSmallTokens &&
         (D.max_blocks + D.k * D.S) * row_bytes <= kSmallBytes && (D.B * D.Hkv <= kSmallPairs || 2 * D.max_blocks >= D.k * D.S);
}

// Scoring, selection, attention and merge of every pair in one launch, one workgroup per pair
// (P.nsplit must be 1, E.mode 2).  `scores` may be null.
int launch_step(const Dims& D, int dtype, const void* q, const void* digest, const int32_t* table, const void* k_pool,
                const void* v_pool, long long n_slots, float* scores, int32_t* sel_all, int32_t* sel_gpu,
                int32_t* slot_gpu, int32_t* n_gpu, int32_t* sel_host, int32_t* n_host, Partials P, Epilogue E,
                hipStream_t st) {
  if (D.B * D.Hkv == 0) return SCOUT_OK;
  if (P.nsplit != 1 || E.mode != 2) return SCOUT_EINVAL;
  dim3 grid(1, D.Hkv, D.B), block(8 * kWave);
  const int per_lane = (D.max_blocks + 8 * kWave - 1) / (8 * kWave);
  const int kpl = per_lane <= 2 ? 2 : 4;  // longer rows: see step_kernel_supported
  if (per_lane > 4) return SCOUT_EUNSUPPORTED;
  const size_t lds = mfma_smem_bytes(D, 8) +
                     (lists_lds_ints((D.k + 3) & ~3) + selector_lds_ints<8>() + 8 * kWave * (size_t)kpl) * sizeof(int) +
                     2 * D.d * sizeof(double);
  const char* dg = static_cast<const char*>(digest);
#define SCOUT_STEP(DT, DH, KPL)                                                                              \
  hipLaunchKernelGGL((step_kernel<DT, DH, KPL>), grid, block, lds, st, D, q, dg, table, k_pool, v_pool, n_slots, scores, \
                     sel_all, sel_gpu, slot_gpu, n_gpu, sel_host, n_host, P, E)
#define SCOUT_STEP_TYPE(DT, DH)                \
  do {                                         \
    if (kpl != 2) return SCOUT_EUNSUPPORTED;   \
    SCOUT_STEP(DT, DH, 2);                     \
  } while (0)
  if (kpl == 4 && dtype == SCOUT_BF16 && D.d == 128)  // rows of 1025 to 2048 blocks: only these take them
    SCOUT_STEP(SCOUT_BF16, 128, 4);
  else
    SCOUT_BY_TYPE(dtype, D.d, SCOUT_STEP_TYPE);
#undef SCOUT_STEP_TYPE
#undef SCOUT_STEP
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

int launch_combine(const Dims& D, Partials P, Epilogue E, hipStream_t st) {
  dim3 grid(D.G, D.Hkv, D.B), block(D.d);
  if (grid.z == 0) return SCOUT_OK;
  if (P.nsplit <= 2)
    hipLaunchKernelGGL(combine_kernel<2>, grid, block, 0, st, D, P, E);
  else if (P.nsplit <= 4)
    hipLaunchKernelGGL(combine_kernel<4>, grid, block, 0, st, D, P, E);
  else
    hipLaunchKernelGGL(combine_kernel<8>, grid, block, 0, st, D, P, E);
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

int launch_merge(const Dims& D, int dtype_out, const float* o_a, const float* m_a, const float* l_a,
                 const float* o_b, const float* m_b, const float* l_b, void* out, float* lse,
                 hipStream_t st) {
  dim3 grid(D.B * D.Hq), block(D.d);
  if (grid.x == 0) return SCOUT_OK;
  if (dtype_out == SCOUT_BF16)
    hipLaunchKernelGGL(merge_kernel<SCOUT_BF16>, grid, block, 0, st, D, o_a, m_a, l_a, o_b, m_b, l_b, out,
                       lse);
  else
    hipLaunchKernelGGL(merge_kernel<SCOUT_F32>, grid, block, 0, st, D, o_a, m_a, l_a, o_b, m_b, l_b, out,
                       lse);
  return hipGetLastError() == hipSuccess ? SCOUT_OK : SCOUT_EHIP;
}

}  // namespace scout
