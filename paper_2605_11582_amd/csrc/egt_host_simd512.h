// Forms of the host encoder's row loops with 512-bit registers (AVX-512 with VBMI2, chosen at run time; egt_host_simd.h
// holds the AVX2 forms for other machines and for the rows that these leave out).  They give the same bits:
//
//  - Masks of 64 columns are one 64-bit register; the codes and offsets of the chosen columns come together with a
//    byte compression, and pairs of codes and fours of offsets with a multiplication and addition of neighbours.
//  - Extrema are taken of the binary16 numbers themselves, as integers in their order (bits of negative ones reversed).
//  - v / s is a product with 1 / s, corrected once by the remainder v - q s, which a fused multiplication and addition gives
//    exactly.  What matters of it is which side of a half-integer it lies on: a quotient that is a half-integer below 32 is a
//    binary32 number, and the corrected value, off by less than 2^-40 of itself before it is rounded to binary32, rounds
//    to it; any other is at least 2^-13 away from one (see egt_host_simd.h).
//
// One core of a Zen 5 on rows in its L2, ns for 64 columns of 2:4, AVX2 -> here: pruning 5.6 -> 2.5, validation 3.3 -> 1.3,
// extrema 3.1 -> 1.7, codes and offsets 11.6 -> 6.0, dense codes 8.1 -> 3.8.  With 16 threads, us of whole calls, medians of 60
// in turn: 4096 x 4096, groups of 128, pruning and packing 886 -> 786 (quartiles 3 percent apart; pruning 222 -> 156), dense quantisation
// 500 -> 382; 2048 x 4096 pruning and packing 483 -> 408; 256 x 4096 220 -> 211.
#ifndef EGT_HOST_SIMD512_H
#define EGT_HOST_SIMD512_H

#include "egt_host_simd.h"

#if defined(EGT_HOST_SIMD) && !defined(EGT_HOST_AVX2_ONLY)
#define EGT_HOST_SIMD512 1
#define EGT_V5 __attribute__((target("avx2,f16c,bmi,bmi2,fma,popcnt,avx512f,avx512bw,avx512vl,avx512dq,avx512vbmi,avx512vbmi2")))

namespace egt_simd512 {

inline bool available() {
  static const bool yes = egt_simd::available() && __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512bw") &&
                          __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("avx512dq") &&
                          __builtin_cpu_supports("avx512vbmi") && __builtin_cpu_supports("avx512vbmi2");
  return yes;
}

EGT_V5 inline uint64_t kept64(const uint8_t *m) {
  const __m512i v = _mm512_loadu_si512((const void *)m);
  return _mm512_test_epi8_mask(v, v);
}

// N:4 mask of one row by magnitude; cols a multiple of 64.
template <int n>
EGT_V5 inline void prune_row(const uint16_t *w, int cols, uint8_t *mask) {
  const __m512i low15 = _mm512_set1_epi16(0x7FFF);
  // the group rotated by one, two, three places; a rival that lies below its column (the rotation wraps) wins a tie
  const __m512i rot1 = _mm512_broadcast_i32x4(_mm_setr_epi8(2, 3, 4, 5, 6, 7, 0, 1, 10, 11, 12, 13, 14, 15, 8, 9));
  const __m512i rot2 = _mm512_broadcast_i32x4(_mm_setr_epi8(4, 5, 6, 7, 0, 1, 2, 3, 12, 13, 14, 15, 8, 9, 10, 11));
  const __m512i rot3 = _mm512_broadcast_i32x4(_mm_setr_epi8(6, 7, 0, 1, 2, 3, 4, 5, 14, 15, 8, 9, 10, 11, 12, 13));
  const __m512i tie1 = _mm512_set1_epi64(0x0001000000000000ll), tie2 = _mm512_set1_epi64(0x0001000100000000ll),
                tie3 = _mm512_set1_epi64(0x0001000100010000ll);
  for (int c = 0; c < cols; c += 64) {
    uint64_t keep = 0;
    for (int h = 0; h < 2; ++h) {
      const __m512i m = _mm512_and_si512(_mm512_loadu_si512((const void *)(w + c + 32 * h)), low15);
      const uint32_t g1 = _mm512_cmpgt_epu16_mask(_mm512_add_epi16(_mm512_shuffle_epi8(m, rot1), tie1), m);
      const uint32_t g2 = _mm512_cmpgt_epu16_mask(_mm512_add_epi16(_mm512_shuffle_epi8(m, rot2), tie2), m);
      const uint32_t g3 = _mm512_cmpgt_epu16_mask(_mm512_add_epi16(_mm512_shuffle_epi8(m, rot3), tie3), m);
      const uint32_t k = n == 1 ? ~(g1 | g2 | g3) : n == 2 ? ~((g1 & g2) | (g3 & (g1 | g2))) : n == 3 ? ~(g1 & g2 & g3) : ~0u;
      keep |= (uint64_t)k << (32 * h);
    }
    _mm512_storeu_si512((void *)(mask + c), _mm512_maskz_set1_epi8(keep, 1));
  }
}

// As egt_simd::row_valid; cols a multiple of 64.
EGT_V5 inline bool row_valid(const uint16_t *w, const uint8_t *mask, int cols, int n) {
  const __m512i expo = _mm512_set1_epi16(0x7C00);
  const uint64_t add = 0x1111111111111111ull * (uint64_t)(7 - n);
  uint64_t bad = 0;
  for (int c = 0; c < cols; c += 64) {
    const uint64_t k = kept64(mask + c);
    const uint64_t p = (k & 0x5555555555555555ull) + ((k >> 1) & 0x5555555555555555ull);
    const uint64_t q = (p & 0x3333333333333333ull) + ((p >> 2) & 0x3333333333333333ull);
    const __m512i x0 = _mm512_loadu_si512((const void *)(w + c)), x1 = _mm512_loadu_si512((const void *)(w + c + 32));
    bad |= ((q + add) & 0x8888888888888888ull) |
           _mm512_mask_cmpeq_epi16_mask((__mmask32)k, _mm512_and_si512(x0, expo), expo) |
           _mm512_mask_cmpeq_epi16_mask((__mmask32)(k >> 32), _mm512_and_si512(x1, expo), expo);
  }
  return bad == 0;
}

// As egt_simd::extrema; n a multiple of 32.
EGT_V5 inline void extrema(const uint16_t *w, const uint8_t *mask, int n, float &lo, float &hi) {
  const __m512i low15 = _mm512_set1_epi16(0x7FFF);
  __m512i mn = _mm512_setzero_si512(), mx = _mm512_setzero_si512();
  for (int c = 0; c < n; c += 32) {
    __mmask32 k = ~(__mmask32)0;
    if (mask) {
      const __m256i m = _mm256_loadu_si256((const __m256i *)(mask + c));
      k = _mm256_test_epi8_mask(m, m);
    }
    const __m512i v = _mm512_maskz_loadu_epi16(k, (const void *)(w + c));
    const __m512i o = _mm512_xor_si512(v, _mm512_and_si512(_mm512_srai_epi16(v, 15), low15));
    mn = _mm512_min_epi16(mn, o);
    mx = _mm512_max_epi16(mx, o);
  }
  const __m256i a = _mm256_min_epi16(_mm512_castsi512_si256(mn), _mm512_extracti64x4_epi64(mn, 1));
  const __m256i b = _mm256_max_epi16(_mm512_castsi512_si256(mx), _mm512_extracti64x4_epi64(mx, 1));
  // (the smallest of eight unsigned words in one instruction: a minimum is at or below 0, a maximum at or above)
  const __m128i a8 = _mm_min_epi16(_mm256_castsi256_si128(a), _mm256_extracti128_si256(a, 1));
  const __m128i b8 = _mm_max_epi16(_mm256_castsi256_si128(b), _mm256_extracti128_si256(b, 1));
  const int16_t l = (int16_t)(_mm_extract_epi16(_mm_minpos_epu16(_mm_xor_si128(a8, _mm_set1_epi16((short)0x8000))), 0) ^ 0x8000);
  const int16_t h = (int16_t)(0x7FFF - _mm_extract_epi16(_mm_minpos_epu16(_mm_sub_epi16(_mm_set1_epi16(0x7FFF), b8)), 0));
  lo = egt_simd::half_to_float((uint16_t)(l < 0 ? l ^ 0x7FFF : l));
  hi = egt_simd::half_to_float((uint16_t)h);
}

// Codes of sixteen columns, one per byte.  r: 1 / s.
EGT_V5 inline __m128i codes16(__m256i w, __m512 s, __m512 r, __m512 z) {
  const __m512 v = _mm512_cvtph_ps(w);
  __m512 q = _mm512_mul_ps(v, r);
  q = _mm512_fmadd_ps(_mm512_fnmadd_ps(q, s, v), r, q);
  q = _mm512_roundscale_ps(q, _MM_FROUND_TO_NEAREST_INT | _MM_FROUND_NO_EXC);
  q = _mm512_min_ps(_mm512_max_ps(_mm512_add_ps(q, z), _mm512_setzero_ps()), _mm512_set1_ps(15.0f));
  return _mm512_cvtepi32_epi8(_mm512_cvtps_epi32(q));
}
struct Scale {
  __m512 s, r, z;
  int zi;
};
EGT_V5 inline Scale scale_of(egt_simd::Pair p) {
  const __m512 s = _mm512_set1_ps(p.s);
  return {s, _mm512_div_ps(_mm512_set1_ps(1.0f), s), _mm512_set1_ps((float)p.z), p.z};
}
EGT_V5 inline __m512i join(const __m128i (&v)[4]) {
  const __m256i a = _mm256_inserti128_si256(_mm256_castsi128_si256(v[0]), v[1], 1);
  const __m256i b = _mm256_inserti128_si256(_mm256_castsi128_si256(v[2]), v[3], 1);
  return _mm512_inserti64x4(_mm512_castsi256_si512(a), b, 1);
}
// two codes to a byte, the first in the low half
EGT_V5 inline __m256i nibbles(__m512i codes) {
  return _mm512_cvtepi16_epi8(_mm512_maddubs_epi16(codes, _mm512_set1_epi16(0x1001)));
}

// The chosen columns of sixteen 4-groups: the kept ones and, where a group keeps fewer than n, the smallest other offsets.
template <int n>
EGT_V5 inline uint64_t chosen64(uint64_t kept) {
  if (_mm_popcnt_u64(kept) == 16 * n) return kept;    // (no group keeps more than n: all are full)
  uint64_t out = 0;
  for (int g = 0; g < 64; g += 4) {
    uint32_t k = (uint32_t)(kept >> g) & 15u;
    for (int j = 0; j < 4 && (int)_mm_popcnt_u32(k) < n; ++j) k |= 1u << j;
    out |= (uint64_t)k << g;
  }
  return out;
}
// Index words of the chosen columns: 4 n bytes.
template <int n>
EGT_V5 inline void store_offsets(uint64_t chosen, uint8_t *idx) {
  const __m512i o = _mm512_maskz_compress_epi8(chosen, _mm512_set1_epi32(0x03020100));
  const __m512i d = _mm512_madd_epi16(_mm512_maddubs_epi16(o, _mm512_set1_epi16(0x0401)), _mm512_set1_epi32(0x00100001));
  const __m128i b = _mm512_cvtepi32_epi8(d);
  if (n == 4) _mm_storeu_si128((__m128i *)idx, b);
  else _mm_mask_storeu_epi8((void *)idx, (__mmask16)((1u << (4 * n)) - 1), b);
}

// As egt_simd::pack_row_int4; cols a multiple of 64, group of 16.
template <int n>
EGT_V5 inline void pack_row_int4(const uint16_t *w, const uint8_t *mask, int cols, int group, const uint16_t *qp, bool paired,
                                 uint8_t *values, uint8_t *idx) {
  int g = 0, left = group;                            // group of the next sixteen columns, columns left in it
  if (cols == 0) return;
  Scale p = scale_of(egt_simd::pair_of(qp, 0));
  const __m512i order = _mm512_broadcast_i32x4(_mm_setr_epi8(0, 2, 4, 6, 1, 3, 5, 7, 8, 10, 12, 14, 9, 11, 13, 15));
  for (int c = 0; c < cols; c += 64) {
    const uint64_t kept = kept64(mask + c), chosen = chosen64<n>(kept);
    __m128i q[4], z[4];
#pragma GCC unroll 4
    for (int k = 0; k < 4; ++k) {
      const int cc = c + 16 * k;
      q[k] = codes16(_mm256_loadu_si256((const __m256i *)(w + cc)), p.s, p.r, p.z);
      z[k] = _mm_set1_epi8((char)p.zi);
      if ((left -= 16) == 0 && cc + 16 < cols) { p = scale_of(egt_simd::pair_of(qp, ++g)); left = group; }
    }
    __m512i codes = _mm512_maskz_compress_epi8(chosen, _mm512_mask_blend_epi8(kept, join(z), join(q)));
    if (paired) codes = _mm512_shuffle_epi8(codes, order);
    const __m256i b = nibbles(codes);
    if (n == 4) _mm256_storeu_si256((__m256i *)values, b);
    else _mm256_mask_storeu_epi8((void *)values, (__mmask32)((1ull << (8 * n)) - 1), b);
    store_offsets<n>(chosen, idx);
    values += 8 * n;
    idx += 4 * n;
  }
}

// As egt_simd::pack_row_fp16; cols a multiple of 64.
template <int n>
EGT_V5 inline void pack_row_fp16(const uint16_t *w, const uint8_t *mask, int cols, uint8_t *values, uint8_t *idx) {
  for (int c = 0; c < cols; c += 64) {
    const uint64_t kept = kept64(mask + c), chosen = chosen64<n>(kept);
    for (int h = 0; h < 2; ++h) {
      const __m512i v = _mm512_maskz_loadu_epi16((__mmask32)(kept >> (32 * h)), (const void *)(w + c + 32 * h));
      const __m512i x = _mm512_maskz_compress_epi16((__mmask32)(chosen >> (32 * h)), v);
      if (n == 4) _mm512_storeu_si512((void *)values, x);
      else _mm512_mask_storeu_epi16((void *)values, (__mmask32)((1ull << (8 * n)) - 1), x);
      values += 16 * n;
    }
    store_offsets<n>(chosen, idx);
    idx += 4 * n;
  }
}

// As egt_simd::quant_group; n a multiple of 64.
EGT_V5 inline void quant_group(const uint16_t *w, int n, float s, int z, uint8_t *q) {
  const Scale p = scale_of({s, z});
  for (int c = 0; c < n; c += 64) {
    __m128i v[4];
#pragma GCC unroll 4
    for (int k = 0; k < 4; ++k) v[k] = codes16(_mm256_loadu_si256((const __m256i *)(w + c + 16 * k)), p.s, p.r, p.z);
    _mm256_storeu_si256((__m256i *)(q + c / 2), nibbles(join(v)));
  }
}

}  // namespace egt_simd512
#endif
#endif
