// One row of a sparse matrix followed slot by slot, M = 1: what the generic kernel does with every row, and the kernel of
// exact codes (egt_mfma_codes.hip) with rows that the matrix instructions do not take.
#ifndef EGT_GENERIC_BODY_H
#define EGT_GENERIC_BODY_H

#include "egt_device.h"

namespace egt {

// floor(j / d) for 1 <= d and j * d < 2^32 by a multiplication: inv = ceil(2^32 / d), and
// d = 1 (whose reciprocal does not fit) passes j through.
__device__ __forceinline__ uint32_t div_by(uint32_t j, uint32_t d, uint32_t inv) {
  return d == 1 ? j : __umulhi(j, inv);
}

// Where column c of x sits in LDS, in halves.  A lane reads the columns of eight consecutive slots
// (8, 16 or 32 columns apart from its neighbour's), which unswizzled puts every 4th to 16th lane
// on one bank; folding bits 7..10 of the column into bits 1..4 spreads them over all banks and
// keeps each pair of halves together.
__device__ __forceinline__ uint32_t x_swizzle(uint32_t c) { return c ^ (((c >> 7) & 15u) << 1); }

// What one lane requests for one word of eight slots: the index word, the codes or FP16 values,
// and the {scale, zero} pairs of the quantisation groups of its first and of its last slot.
struct SlotWord {
  uint32_t iw, nib, p_first, p_last;
  uint4 hv;
};

// One lane's share of one row's dot product with x, for the M = 1 kernels (x_at(c, c4): the activation of column c, c4 a
// 4-group whose columns share bits 7 and up with c).  N (kept entries
// per 4 columns of this row) is a compile-time constant, so the 4-group of slot k of word w is
// (8 w + k) / N with one division per word at most (N = 3; the others shift), and TWO says
// that no word of eight slots reaches into more than two quantisation groups ((N + 6) / N <=
// group / 4), so that the two {scale, zero} pairs requested with the index and value words
// cover every slot; ONE that every word lies inside one group (8 / N divides group / 4), where
// the pair is applied once per word: s (sum q x - z sum x).  With neither, each slot requests
// its own pair.  A lane requests U words (64 words apart) before it uses the first.
enum { Q_EACH = 0, Q_TWO = 1, Q_ONE = 2 };
template <int VAL_KIND, int N, int QMODE, int U = 1, class X>
__device__ __forceinline__ float row_dot(const uint8_t *__restrict__ values, const uint16_t *__restrict__ idx,
                                         const uint32_t *__restrict__ qrow, uint32_t t_row, uint32_t words,
                                         uint32_t g4, uint32_t inv_g4, int lane,
                                         const X &x_at) {
  constexpr bool INT4 = VAL_KIND != EGT_VAL_FP16, paired = VAL_KIND == EGT_VAL_INT4_PAIRED;
  constexpr bool TWO = QMODE == Q_TWO, ONE = QMODE == Q_ONE;
  float acc = 0.f;
  for (uint32_t w0 = lane; w0 < words; w0 += 64 * U) {
    SlotWord in[U];
    uint32_t c4_first[U], rem_first[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t w = w0 + 64 * u;
      in[u] = SlotWord{0, 0, 0, 0, {0, 0, 0, 0}};
      c4_first[u] = N == 3 ? __umulhi(8 * w, 0x55555556u) : 8 * w / N;      // 4-group of the word's first slot
      rem_first[u] = N == 3 ? 8 * w - 3 * c4_first[u] : 0;                  // (8 w is a multiple of 1, 2 and 4)
      if (w < words) {
        const uint32_t t0 = t_row + 8 * w;
        in[u].iw = idx[t0 >> 3];
        if (INT4) {
          in[u].nib = *(const uint32_t *)(values + (t0 >> 1));
          if (ONE) in[u].p_first = qrow[div_by(c4_first[u], g4, inv_g4)];
          if (TWO) {
            // (v * 11) >> 5 = v / 3 for v < 16
            const uint32_t c4_7 = c4_first[u] + (N == 3 ? ((rem_first[u] + 7) * 11u) >> 5 : 7u / N);
            in[u].p_first = qrow[div_by(c4_first[u], g4, inv_g4)];
            in[u].p_last = qrow[div_by(c4_7, g4, inv_g4)];
          }
        } else {
          in[u].hv = *(const uint4 *)(values + 2ull * t0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (w0 + 64 * u >= words) break;
      const uint32_t c4_0 = c4_first[u], rem = rem_first[u], iw = in[u].iw, nib = in[u].nib;
      // first 4-group past the first slot's quantisation group
      const uint32_t b_first = TWO ? (div_by(c4_0, g4, inv_g4) + 1) * g4 : 0;
      const float s_first = __half2float(__ushort_as_half((uint16_t)(in[u].p_first & 0xFFFFu)));
      const float z_first = __half2float(__ushort_as_half((uint16_t)(in[u].p_first >> 16)));
      const float s_last = __half2float(__ushort_as_half((uint16_t)(in[u].p_last & 0xFFFFu)));
      const float z_last = __half2float(__ushort_as_half((uint16_t)(in[u].p_last >> 16)));
      const uint32_t hw[4] = {in[u].hv.x, in[u].hv.y, in[u].hv.z, in[u].hv.w};
      float sum_qx = 0.f, sum_x = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t c4 = c4_0 + (N == 3 ? ((rem + k) * 11u) >> 5 : (uint32_t)k / N);
        // (for N = 1, 2, 4 a word's columns share bits 7 and up)
        const float xk = x_at(4 * c4 + ((iw >> (2 * k)) & 3u), N == 3 ? c4 : c4_0);
        float wv;
        if (INT4 && ONE) {
          const int q = (nib >> (paired ? 4 * ((k >> 1) + 4 * (k & 1)) : 4 * k)) & 15;
          sum_qx = fmaf((float)q, xk, sum_qx);
          sum_x += xk;
          continue;
        }
        if (INT4) {
          const int q = (nib >> (paired ? 4 * ((k >> 1) + 4 * (k & 1)) : 4 * k)) & 15;
          float sc, zp;
          if (TWO) {
            sc = c4 < b_first ? s_first : s_last;
            zp = c4 < b_first ? z_first : z_last;
          } else {
            const uint32_t p = qrow[div_by(c4, g4, inv_g4)];
            sc = __half2float(__ushort_as_half((uint16_t)(p & 0xFFFFu)));
            zp = __half2float(__ushort_as_half((uint16_t)(p >> 16)));
          }
          wv = sc * ((float)q - zp);
        } else {
          wv = __half2float(__ushort_as_half((uint16_t)(hw[k >> 1] >> (16 * (k & 1)))));
        }
        acc = fmaf(wv, xk, acc);
      }
      if (INT4 && ONE) acc = fmaf(s_first, sum_qx - z_first * sum_x, acc);
    }
  }
  return acc;
}

// The whole row, the same for all lanes: n_keep is 1..4, `words` index words; every lane returns its share.
template <int VAL_KIND, class X>
__device__ __forceinline__ float row_dot_any(int n_keep, const uint8_t *__restrict__ values, const uint16_t *__restrict__ idx,
                                             const uint32_t *__restrict__ qrow, uint32_t t_row, uint32_t words, uint32_t g4, uint32_t inv_g4,
                                             int lane, const X &x_at) {
  const uint32_t n = (uint32_t)n_keep;
  const bool one = n != 3 && g4 % (8u / n) == 0, two = (n + 6) / n <= g4;
#define EGT_ROW(N, Q) row_dot<VAL_KIND, N, Q>(values, idx, qrow, t_row, words, g4, inv_g4, lane, x_at)
#define EGT_ROW_N(N) (one ? EGT_ROW(N, Q_ONE) : two ? EGT_ROW(N, Q_TWO) : EGT_ROW(N, Q_EACH))
  switch (n_keep) {
    case 1: return EGT_ROW_N(1);
    case 2: return EGT_ROW_N(2);
    case 3: return two ? EGT_ROW(3, Q_TWO) : EGT_ROW(3, Q_EACH);
    default: return EGT_ROW_N(4);
  }
#undef EGT_ROW_N
#undef EGT_ROW
}

}  // namespace egt
#endif
