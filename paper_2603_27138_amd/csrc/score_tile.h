// One batch of the scoring stream: which bytes of consecutive digest entries a wave asks for, and the sums over them.
// Shared by the scoring pass and by the kernel that scores in front of its own selection, so that a score has the same
// bits whichever of them made it.
//
// A wave-wide load takes one 128-byte line from each of 8 consecutive digest entries (8 lanes x 16 bytes per entry), and
// NL such loads cover the entries whole; a batch of kScoreBatch loads holds NG such groups of entries.
#pragma once
#include "common.h"

namespace scout {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kScoreBatch = 8;  // wave-wide loads per batch

// MEAN: the entry is one row of binary32 sums whatever the element type of the queries.
template <int DT, int DH, bool MEAN>
struct ScoreTile {
  static constexpr bool DIG16 = DT == SCOUT_BF16 && !MEAN;  // digest elements are bf16
  static constexpr int EPL = DIG16 ? 8 : 4;                 // digest elements per 16-byte load
  static constexpr int DSZ = DIG16 ? 2 : 4;                 // bytes per digest element
  static constexpr int EB = (MEAN ? 1 : 2) * DH * DSZ;      // bytes per digest entry
  static constexpr int NL = EB / 128;                       // 128-byte lines per entry
  static constexpr int NG = kScoreBatch / NL;               // 8-entry groups per batch
  static constexpr int BLOCKS = NG * 8;                     // entries per batch
  static constexpr int LPR = MEAN ? NL : NL / 2;            // lines per digest row
  static_assert(NL >= 2 && NL <= kScoreBatch, "layout");

  // byte offset, from the batch's first entry, of a lane's part of load `it`
  static __device__ __forceinline__ int offset(int lane, int it) {
    return ((lane >> 3) + (it / NL) * 8) * EB + (lane & 7) * 16 + (it % NL) * 128;
  }

  // A lane's coefficients from lds[0]: N_c (min row), lds[1]: P_c (max row; MEAN: both hold the plain sum).
  // Line u of an entry: min row for u < NL/2, max row after (MEAN: the one row of sums);
  // channels (u % lines per row) * 128/DSZ + 8 lanes x EPL
  static __device__ __forceinline__ void coefficients(double (&coef)[NL][EPL], const double* lds, int lane) {
#pragma unroll
    for (int u = 0; u < NL; ++u)
#pragma unroll
      for (int i = 0; i < EPL; ++i)
        coef[u][i] = lds[(u >= LPR ? DH : 0) + (u % LPR) * (128 / DSZ) + (lane & 7) * EPL + i];
  }

  // The entry of the batch whose sum a lane holds after scores(), and whether it is the one lane to write it.
  static __device__ __forceinline__ int entry(int lane) {
    const bool hi2 = (lane >> 2) & 1, hi1 = (lane >> 1) & 1;
    const int my_g = NG == 4 ? (hi2 ? 2 : 0) + (hi1 ? 1 : 0) : NG == 2 ? (hi2 ? 1 : 0) : 0;
    return my_g * 8 + (lane >> 3);
  }
  static __device__ __forceinline__ bool writer(int lane) {
    return NG == 4 ? (lane & 1) == 0 : NG == 2 ? (lane & 3) == 0 : (lane & 7) == 0;
  }

  // sum_c P_c * max_j[c] + N_c * min_j[c] of entry(lane), in binary64
  static __device__ __forceinline__ double scores(const u32x4 (&cur)[kScoreBatch], const double (&coef)[NL][EPL], int lane) {
    const bool hi2 = (lane >> 2) & 1, hi1 = (lane >> 1) & 1;
    double a[NG];
#pragma unroll
    for (int gq = 0; gq < NG; ++gq) {
      double acc = 0.0;
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const u32x4 w = cur[gq * NL + u];
        if (DIG16) {
          acc = fma(coef[u][0], (double)bf16_lo(w[0]), acc);
          acc = fma(coef[u][1], (double)bf16_hi(w[0]), acc);
          acc = fma(coef[u][2 % EPL], (double)bf16_lo(w[1]), acc);
          acc = fma(coef[u][3 % EPL], (double)bf16_hi(w[1]), acc);
          acc = fma(coef[u][4 % EPL], (double)bf16_lo(w[2]), acc);
          acc = fma(coef[u][5 % EPL], (double)bf16_hi(w[2]), acc);
          acc = fma(coef[u][6 % EPL], (double)bf16_lo(w[3]), acc);
          acc = fma(coef[u][7 % EPL], (double)bf16_hi(w[3]), acc);
        } else {
          acc = fma(coef[u][0], (double)__uint_as_float(w[0]), acc);
          acc = fma(coef[u][1], (double)__uint_as_float(w[1]), acc);
          acc = fma(coef[u][2], (double)__uint_as_float(w[2]), acc);
          acc = fma(coef[u][3], (double)__uint_as_float(w[3]), acc);
        }
      }
      a[gq] = acc;
    }
    // add across the 8 lanes of an entry; with several groups the first steps exchange and halve
    if constexpr (NG == 4) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double keep = hi2 ? a[i + 2] : a[i], send = hi2 ? a[i] : a[i + 2];
        a[i] = keep + partner_f64<2>(send);
      }
      const double keep = hi1 ? a[1] : a[0], send = hi1 ? a[0] : a[1];
      a[0] = keep + partner_f64<1>(send);
    } else if constexpr (NG == 2) {
      const double keep = hi2 ? a[1] : a[0], send = hi2 ? a[0] : a[1];
      a[0] = keep + partner_f64<2>(send);
      a[0] += partner_f64<1>(a[0]);
    } else {
      a[0] += partner_f64<2>(a[0]);
      a[0] += partner_f64<1>(a[0]);
    }
    return a[0] + partner_f64<0>(a[0]);
  }
};

}  // namespace scout
