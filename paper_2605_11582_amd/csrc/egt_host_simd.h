// Vector forms of the host encoder's row loops (AVX2, F16C and BMI2, chosen at run time; the
// plain loops of egt_host.cpp remain for other machines and for groups that are no multiple
// of eight columns).  They give the bits of the plain loops:
//
//  - Extrema and codes in binary32 instead of binary64.  v and s are binary16 numbers, a / b
//    times a power of two with integers a, b < 2^11.  A quotient that is no half-integer, but
//    below 32 in magnitude, is at least 2^-13 away from every half-integer (the difference to
//    (2m + 1) / 2 is a non-zero multiple of 1 / (2 b 2^j), and b 2^j < 2^12 for quotients of a
//    half and more), and a division in binary32 is off by at most 2^-20 there; a quotient that
//    is a half-integer is exact in both.  Quotients of 32 and more are clamped either way.
//  - A decoded value s (q - z) with an integer z in 0..15 is exact in binary32 (11 + 5 bits)
//    and rounds once to binary16.
//  - PEXT gathers the codes, offsets or values of the chosen columns of a 4-group in ascending
//    order, PDEP puts them back: one instruction per eight columns instead of a loop over
//    slots.
//
// A 4096 x 4096 matrix, 2:4, groups of 128, 16 threads: pruning and packing took 16 ms with a
// double-precision conversion, division and rounding call per column and a byte write per
// code.
#ifndef EGT_HOST_SIMD_H
#define EGT_HOST_SIMD_H

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define EGT_HOST_SIMD 1
#include <immintrin.h>

#include <cstdint>
#include <cstring>

#define EGT_V __attribute__((target("avx2,f16c,bmi,bmi2,fma,popcnt")))

namespace egt_simd {

inline bool available() {
  static const bool yes = __builtin_cpu_supports("avx2") && __builtin_cpu_supports("f16c") && __builtin_cpu_supports("bmi2");
  return yes;
}

typedef unsigned __int128 u128;

// 0xFF in every byte of m that is not zero
EGT_V inline __m128i kept_bytes(const uint8_t *m) {
  const __m128i v = _mm_loadu_si128((const __m128i *)m);
  return _mm_xor_si128(_mm_cmpeq_epi8(v, _mm_setzero_si128()), _mm_set1_epi8(-1));
}

// N:4 mask of one row by magnitude: column j of a 4-group is kept if fewer than n others beat
// it (a lower column wins a tie).  Eight 4-groups at a time: the rivals of every column are
// the group rotated by one, two and three places.
EGT_V inline void prune_row(const uint16_t *w, int cols, int n, uint8_t *mask) {
  const __m256i low15 = _mm256_set1_epi16(0x7FFF), limit = _mm256_set1_epi16((short)-n), one = _mm256_set1_epi8(1);
  // rival (j + r) & 3 lies below column j where j + r wraps
  const __m256i wrap1 = _mm256_set1_epi64x((long long)0xFFFF000000000000ull), wrap2 = _mm256_set1_epi64x((long long)0xFFFFFFFF00000000ull),
                wrap3 = _mm256_set1_epi64x((long long)0xFFFFFFFFFFFF0000ull), ones = _mm256_set1_epi16(-1);
  int c = 0;
  for (; c + 32 <= cols; c += 32) {
    __m256i keep[2];
    for (int h = 0; h < 2; ++h) {
      const __m256i m = _mm256_and_si256(_mm256_loadu_si256((const __m256i *)(w + c + 16 * h)), low15);
      __m256i beats = _mm256_setzero_si256();        // minus the number of columns that beat this one
#define EGT_RIVAL(SHUF, WRAP)                                                                                       \
  {                                                                                                                 \
    const __m256i r = _mm256_shufflehi_epi16(_mm256_shufflelo_epi16(m, SHUF), SHUF);                                \
    const __m256i gt = _mm256_cmpgt_epi16(r, m), ge = _mm256_xor_si256(_mm256_cmpgt_epi16(m, r), ones);             \
    beats = _mm256_add_epi16(beats, _mm256_blendv_epi8(gt, ge, WRAP));                                              \
  }
      EGT_RIVAL(_MM_SHUFFLE(0, 3, 2, 1), wrap1)
      EGT_RIVAL(_MM_SHUFFLE(1, 0, 3, 2), wrap2)
      EGT_RIVAL(_MM_SHUFFLE(2, 1, 0, 3), wrap3)
#undef EGT_RIVAL
      keep[h] = _mm256_cmpgt_epi16(beats, limit);    // -beats < n
    }
    const __m256i bytes = _mm256_permute4x64_epi64(_mm256_packs_epi16(keep[0], keep[1]), _MM_SHUFFLE(3, 1, 2, 0));
    _mm256_storeu_si256((__m256i *)(mask + c), _mm256_and_si256(bytes, one));
  }
  for (; c < cols; c += 4) {                          // (the mask of a matrix whose columns are no multiple of 32)
    int mag[4];
    for (int j = 0; j < 4; ++j) mag[j] = w[c + j] & 0x7FFF;
    for (int j = 0; j < 4; ++j) {
      int beats = 0;
      for (int i = 0; i < 4; ++i)
        if (i != j) beats += i < j ? (mag[i] >= mag[j]) : (mag[i] > mag[j]);
      mask[c + j] = beats < n ? 1 : 0;
    }
  }
}

// Whether a row (cols a multiple of 16) is free of 4-groups that keep more than n columns and
// of kept columns that are NaN or infinite.
EGT_V inline bool row_valid(const uint16_t *w, const uint8_t *mask, int cols, int n) {
  const __m256i expo = _mm256_set1_epi16(0x7C00);
  const uint32_t add = 0x1111u * (uint32_t)(7 - n);
  for (int c = 0; c < cols; c += 16) {
    const __m128i kept = kept_bytes(mask + c);
    const uint32_t b = (uint32_t)_mm_movemask_epi8(kept);
    const uint32_t p = (b & 0x5555u) + ((b >> 1) & 0x5555u), q = (p & 0x3333u) + ((p >> 2) & 0x3333u);
    const __m256i x = _mm256_loadu_si256((const __m256i *)(w + c));
    const __m256i bad = _mm256_and_si256(_mm256_cmpeq_epi16(_mm256_and_si256(x, expo), expo), _mm256_cvtepi8_epi16(kept));
    if (((q + add) & 0x8888u) || !_mm256_testz_si256(bad, bad)) return false;
  }
  return true;
}

EGT_V inline bool all_finite(const uint16_t *w, int cols) {
  const __m256i expo = _mm256_set1_epi16(0x7C00);
  __m256i bad = _mm256_setzero_si256();
  int c = 0;
  for (; c + 16 <= cols; c += 16) {
    const __m256i x = _mm256_loadu_si256((const __m256i *)(w + c));
    bad = _mm256_or_si256(bad, _mm256_cmpeq_epi16(_mm256_and_si256(x, expo), expo));
  }
  bool ok = _mm256_testz_si256(bad, bad);
  for (; c < cols; ++c) ok &= (w[c] & 0x7C00) != 0x7C00;
  return ok;
}

// Extrema of the kept columns [0, n) of a group together with 0 (n a multiple of eight;
// mask == nullptr: all are kept).
EGT_V inline void extrema(const uint16_t *w, const uint8_t *mask, int n, float &lo, float &hi) {
  __m256 mn = _mm256_setzero_ps(), mx = _mm256_setzero_ps();
  for (int c = 0; c < n; c += 8) {
    __m256 v = _mm256_cvtph_ps(_mm_loadu_si128((const __m128i *)(w + c)));
    if (mask) {
      const __m256i drop = _mm256_cmpeq_epi32(_mm256_cvtepu8_epi32(_mm_loadl_epi64((const __m128i *)(mask + c))), _mm256_setzero_si256());
      v = _mm256_andnot_ps(_mm256_castsi256_ps(drop), v);
    }
    mn = _mm256_min_ps(mn, v);
    mx = _mm256_max_ps(mx, v);
  }
  __m128 a = _mm_min_ps(_mm256_castps256_ps128(mn), _mm256_extractf128_ps(mn, 1));
  __m128 b = _mm_max_ps(_mm256_castps256_ps128(mx), _mm256_extractf128_ps(mx, 1));
  a = _mm_min_ps(a, _mm_movehl_ps(a, a));
  b = _mm_max_ps(b, _mm_movehl_ps(b, b));
  lo = _mm_cvtss_f32(_mm_min_ss(a, _mm_movehdup_ps(a)));
  hi = _mm_cvtss_f32(_mm_max_ss(b, _mm_movehdup_ps(b)));
}

EGT_V inline float half_to_float(uint16_t h) { return _mm_cvtss_f32(_mm_cvtph_ps(_mm_cvtsi32_si128(h))); }

// A stored {scale, zero} pair: the zero point is an integer in 0..15.
struct Pair { float s; int z; };
EGT_V inline Pair pair_of(const uint16_t *qp, int g) { return {half_to_float(qp[2 * g]), (int)half_to_float(qp[2 * g + 1])}; }

// Zero point of a group whose extrema (0 among them) start at `lo`, for the scale s.
EGT_V inline int zero_point(float lo, float s) {
  const __m128 q = _mm_div_ss(_mm_set_ss(-lo), _mm_set_ss(s));
  const float z = _mm_cvtss_f32(_mm_round_ss(q, q, _MM_FROUND_TO_NEAREST_INT | _MM_FROUND_NO_EXC));
  return (int)(z < 0.0f ? 0.0f : z > 15.0f ? 15.0f : z);
}

// Codes of eight columns, one per byte.
EGT_V inline uint64_t codes8(const uint16_t *w, float s, int z) {
  const __m256 v = _mm256_cvtph_ps(_mm_loadu_si128((const __m128i *)w));
  __m256 q = _mm256_round_ps(_mm256_div_ps(v, _mm256_set1_ps(s)), _MM_FROUND_TO_NEAREST_INT | _MM_FROUND_NO_EXC);
  // (clamped before the conversion to integers: a quotient may be larger than an integer holds)
  q = _mm256_add_ps(q, _mm256_set1_ps((float)z));
  q = _mm256_min_ps(_mm256_max_ps(q, _mm256_setzero_ps()), _mm256_set1_ps(15.0f));
  const __m256i i = _mm256_cvtps_epi32(q);
  const __m128i h = _mm_packus_epi32(_mm256_castsi256_si128(i), _mm256_extracti128_si256(i, 1));
  return (uint64_t)_mm_cvtsi128_si64(_mm_packus_epi16(h, h));
}

// 0xFF in the bytes of the chosen columns of eight (two 4-groups): the kept ones and, where a
// group keeps fewer than n, the smallest other offsets.
template <int n>
EGT_V inline uint64_t chosen8(uint64_t kept) {
  if (_mm_popcnt_u64(kept) == 16 * n) return kept;    // (no group keeps more than n: both are full)
  for (int half = 0; half < 64; half += 32)
    for (int j = 0; j < 4 && _mm_popcnt_u64((kept >> half) & 0xFFFFFFFFull) < 8 * n; ++j) kept |= 0xFFull << (half + 8 * j);
  return kept;
}
EGT_V inline uint64_t kept8(const uint8_t *mask) {
  const __m128i v = _mm_loadl_epi64((const __m128i *)mask);
  return ~(uint64_t)_mm_cvtsi128_si64(_mm_cmpeq_epi8(v, _mm_setzero_si128()));
}

// One row of INT4 values at N:4, 32 columns = n index words at a time.  qp: the row's
// {scale, zero} pairs.  values and idx: the row's first byte and word (whole words: 4 n bytes of values per step).
template <int n>
EGT_V inline void pack_row_int4(const uint16_t *w, const uint8_t *mask, int cols, int group, const uint16_t *qp, bool paired,
                                uint8_t *values, uint8_t *idx) {
  int g = 0, left = group;                            // group of the next eight columns, columns left in it
  Pair p = cols > 0 ? pair_of(qp, 0) : Pair{};
  for (int c = 0; c < cols; c += 32) {
    u128 val = 0;
    uint64_t off = 0;
#pragma GCC unroll 4
    for (int k = 0; k < 4; ++k) {
      const int cc = c + 8 * k;
      const uint64_t kept = kept8(mask + cc), chosen = chosen8<n>(kept);
      const uint64_t q = (codes8(w + cc, p.s, p.z) & kept) | ((0x0101010101010101ull * (uint64_t)p.z) & ~kept);
      val |= (u128)_pext_u64(q, chosen & 0x0F0F0F0F0F0F0F0Full) << (8 * n * k);
      off |= _pext_u64(0x0302010003020100ull, chosen & 0x0303030303030303ull) << (4 * n * k);
      if ((left -= 8) == 0 && cc + 8 < cols) { p = pair_of(qp, ++g); left = group; }
    }
    if (paired) {
      u128 v = 0;
      for (int k = 0; k < n; ++k) {
        const uint32_t word = (uint32_t)(val >> (32 * k));
        v |= (u128)(_pext_u32(word, 0x0F0F0F0Fu) | (_pext_u32(word, 0xF0F0F0F0u) << 16)) << (32 * k);
      }
      val = v;
    }
    std::memcpy(values, &val, 4 * (size_t)n);
    std::memcpy(idx, &off, 2 * (size_t)n);
    values += 4 * n;
    idx += 2 * n;
  }
}

// The same for FP16 values: 64 n bits of values per 4-group of four, +0 in padding slots.
template <int n>
EGT_V inline void pack_row_fp16(const uint16_t *w, const uint8_t *mask, int cols, uint8_t *values, uint8_t *idx) {
  for (int c = 0; c < cols; c += 32) {
    uint64_t off = 0;
#pragma GCC unroll 4
    for (int k = 0; k < 4; ++k) {
      const int cc = c + 8 * k;
      const uint64_t kept = kept8(mask + cc), chosen = chosen8<n>(kept);
      off |= _pext_u64(0x0302010003020100ull, chosen & 0x0303030303030303ull) << (4 * n * k);
      for (int h = 0; h < 2; ++h) {
        const __m128i wide = _mm_cvtepi8_epi16(_mm_cvtsi64_si128((long long)((kept >> (32 * h)) & 0xFFFFFFFFull)));
        const __m128i pick = _mm_cvtepi8_epi16(_mm_cvtsi64_si128((long long)((chosen >> (32 * h)) & 0xFFFFFFFFull)));
        uint64_t v;
        std::memcpy(&v, w + cc + 4 * h, 8);
        v = _pext_u64(v & (uint64_t)_mm_cvtsi128_si64(wide), (uint64_t)_mm_cvtsi128_si64(pick));
        std::memcpy(values, &v, 2 * (size_t)n);
        values += 2 * n;
      }
    }
    std::memcpy(idx, &off, 2 * (size_t)n);
    idx += 2 * n;
  }
}

// Codes of one group of a dense row (n a multiple of eight columns), two to a byte.
EGT_V inline void quant_group(const uint16_t *w, int n, float s, int z, uint8_t *q) {
  for (int c = 0; c < n; c += 8) {
    const uint32_t v = (uint32_t)_pext_u64(codes8(w + c, s, z), 0x0F0F0F0F0F0F0F0Full);
    std::memcpy(q + c / 2, &v, 4);
  }
}

// 4-group index bits (n offsets of two bits) -> 0xFF in the bytes of the columns, 0 where the
// offsets do not ascend.
struct GroupMasks {
  uint32_t m[5][256];
  GroupMasks() {
    for (int n = 0; n <= 4; ++n)
      for (int b = 0; b < 256; ++b) {
        uint32_t v = 0;
        int prev = -1;
        bool ok = n > 0 && (b >> (2 * n)) == 0;
        for (int k = 0; k < n && ok; ++k) {
          const int off = (b >> (2 * k)) & 3;
          ok = off > prev;
          prev = off;
          v |= 0xFFu << (8 * off);
        }
        m[n][b] = ok ? v : 0u;
      }
  }
};
inline const GroupMasks &group_masks() {
  static const GroupMasks t;
  return t;
}
template <int n>
inline uint64_t columns8(const uint32_t *tab, uint64_t bits) {        // bits: 4 n of two 4-groups
  const uint64_t one = (1ull << (2 * n)) - 1;
  return (uint64_t)tab[bits & one] | ((uint64_t)tab[(bits >> (2 * n)) & one] << 32);
}
// Whether every 4-group of a row has ascending offsets.
template <int n>
inline bool offsets_ascend(const uint8_t *idx, int cols) {
  const uint32_t *tab = group_masks().m[n];
  const uint64_t one = (1ull << (2 * n)) - 1;
  bool ok = true;
  for (int c = 0; c < cols; c += 32, idx += 2 * n) {
    uint64_t off = 0;
    std::memcpy(&off, idx, 2 * (size_t)n);
    for (int k = 0; k < 8; ++k) ok &= tab[(off >> (2 * n * k)) & one] != 0;
  }
  return ok;
}
// Decodes one row: w (may be null) and mask (may be null) of `cols` columns.  qp: the row's
// {scale, zero} pairs (INT4; group a multiple of eight), FP16 values otherwise (nullptr).
template <int n>
EGT_V inline void unpack_row(const uint8_t *values, const uint8_t *idx, int cols, int group, const uint16_t *qp, bool paired,
                             uint16_t *w, uint8_t *mask) {
  const uint32_t *tab = group_masks().m[n];
  int g = 0, left = group;
  Pair p = qp && cols > 0 ? pair_of(qp, 0) : Pair{};
  for (int c = 0; c < cols; c += 32) {
    uint64_t off = 0;
    std::memcpy(&off, idx, 2 * (size_t)n);
    idx += 2 * n;
    u128 val = 0;
    if (qp && w) {
      std::memcpy(&val, values, 4 * (size_t)n);
      values += 4 * n;
      if (paired) {
        u128 v = 0;
        for (int k = 0; k < n; ++k) {
          const uint32_t word = (uint32_t)(val >> (32 * k));
          v |= (u128)(_pdep_u32(word, 0x0F0F0F0Fu) | _pdep_u32(word >> 16, 0xF0F0F0F0u)) << (32 * k);
        }
        val = v;
      }
    }
#pragma GCC unroll 4
    for (int k = 0; k < 4; ++k) {
      const int cc = c + 8 * k;
      const uint64_t cols8 = columns8<n>(tab, off >> (4 * n * k));
      if (mask) {
        const uint64_t ones = cols8 & 0x0101010101010101ull;
        std::memcpy(mask + cc, &ones, 8);
      }
      if (!w) continue;
      const __m128i in = _mm_cvtsi64_si128((long long)cols8);
      const __m128i lanes = _mm_cvtepi8_epi16(in);
      if (qp) {
        const uint64_t q = _pdep_u64((uint64_t)(val >> (8 * n * k)), cols8 & 0x0F0F0F0F0F0F0F0Full);
        const __m256 f = _mm256_cvtepi32_ps(_mm256_sub_epi32(_mm256_cvtepu8_epi32(_mm_cvtsi64_si128((long long)q)), _mm256_set1_epi32(p.z)));
        const __m128i h = _mm256_cvtps_ph(_mm256_mul_ps(f, _mm256_set1_ps(p.s)), _MM_FROUND_TO_NEAREST_INT | _MM_FROUND_NO_EXC);
        _mm_storeu_si128((__m128i *)(w + cc), _mm_and_si128(h, lanes));
        if ((left -= 8) == 0 && cc + 8 < cols) { p = pair_of(qp, ++g); left = group; }
      } else {
        for (int h = 0; h < 2; ++h) {
          uint64_t v = 0;
          std::memcpy(&v, values, 2 * (size_t)n);
          values += 2 * n;
          v = _pdep_u64(v, (uint64_t)(h ? _mm_extract_epi64(lanes, 1) : _mm_cvtsi128_si64(lanes)));
          std::memcpy(w + cc + 4 * h, &v, 8);
        }
      }
    }
  }
}

// f(a constant n) for n in 1..4
template <int V>
struct N { static constexpr int n = V; };
template <class F>
inline auto with_n(int n, F &&f) {
  switch (n) {
    case 1: return f(N<1>{});
    case 2: return f(N<2>{});
    case 3: return f(N<3>{});
    default: return f(N<4>{});
  }
}

}  // namespace egt_simd
#endif
#endif
