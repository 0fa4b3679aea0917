// M = 1 products of INT4 matrices whose rows fill no tile of the row-per-wave kernels, on the matrix
// cores: 2:4 (either nibble order), 1:4, rows of different lengths, dense.
//
// The weights stay whole numbers: the instruction multiplies the exact FP16 integers q - z, its
// sum over a quantisation group is FP32, and the group's scale is applied to that sum in FP32.  So
// no weight is rounded (the row-per-wave kernels round s (q - z) to FP16 first), none has to lie in FP16's
// range, and the error against 64 bits is that of the slot-by-slot kernels which took these
// shapes before (20000 x 2816 2:4, dense 5003 x 2880, half of 11008 x 4096 at 1:4: 2.08e-4, the rounding of y).
//
// For that a sum must not leave its group.  The mapping is the diagonal one: a tile has UNITS units, the 64 / UNITS
// lanes (i, kb) = i + UNITS kb of unit i take its chunks, column n of B carries the activations of unit n, and
// D[i][i] is unit i's share of its row.  A unit lies inside one group: sparse rows use the 32 x 32 instruction
// with units of two chunks of 64 columns (groups of 128 and more; 32 for groups of 64, 16 for 32), dense rows the
// 16 x 16 one with units of four chunks of 32 columns, for groups of 64 and 32 the 32 x 32 one.  So a lane requests up to 16 bytes
// of codes at a time (with the 16 x 16 instruction a sparse unit would be four chunks of 32 columns, twice the requests
// for the same rows: 2:4 11008 x 3968 6.6 us).  A row takes ceil(cols / unit) units: `rpt` whole
// rows lie in a tile, or a row lies in `phases` tiles.
//
//  - 1:4: a slot becomes {q - z, q - z} with its offset in both index fields, and the scale is halved:
//    only kept columns are multiplied, so an infinity in another column reaches nothing.
//  - Rows of different lengths: the chunk of a row that keeps one of four spans the same columns
//    as that of a row that keeps two, so both use the same B operand; a tile is one row.  A chunk is requested in halves, the
//    second out of range for a row that keeps one (a branch around the requests would be waited behind).  Rows that
//    keep three or four are left to the vector units, dealt to all waves of their workgroup (codes_wide_rows).
//  - One shot, as the row-per-wave kernels: a wave requests its four tiles (of one phase) at once, the phases of a row
//    are different waves, whose sums meet in LDS; small workgroups, so that one set of rows waits for no other.  (A walk over
//    more tiles with two sets of registers, and a loop over row sets under one staged x, were slower on all but the longest rows:
//    requests out of range at the end of a walk are not free.)
//  - x goes from global memory straight into LDS, its pieces swizzled as in egt_rows.hip.
//
// Measured, us per launch slot by slot and now (weights in the last-level cache): half of 11008 x 4096's rows at 1:4 11.6, 6.1;
// dense 5003 x 2880 groups of 64 5.6, 4.3; 2:4 20000 x 2816 14.5, 7.0; 2000 x 3072 5.8, 2.8; 50000 x 512 14.4, 3.9; 1:4 4096 x 3072 5.3,
// 3.2; dense 60000 x 384 11.6, 4.2; 512 x 14400 8.5, 4.4.  What bounds it: the launch for a few megabytes, then vector issue (a wave
// of four tiles 460 instructions at 2:4, 590 where rows differ, of two dense ones 240) and memory (20000 x 2816: 42 MB at 6.0 TB/s).
#include "egt_mfma_common.h"
#include "egt_tune.h"

#include <algorithm>

namespace egt {

enum { CODES_24 = 0, CODES_14 = 1, CODES_MIXED = 2, CODES_DENSE = 3, CODES_24P = 4 };    // 24P: paired nibble order
constexpr int CODES_TPI = 4;                          // tiles of a wave at most (a tile has up to 16 rows, so a wave 64 at most)
constexpr int CODES_WAVES = 16;                       // waves of a workgroup at most

struct CodesGeom {
  int rows;
  int nchunks;         // chunks of a row (whole units)
  int upr, upr_inv;    // units of a row inside a tile; ceil(65536 / upr)
  int rpt;             // rows of a tile (1 where a row takes several, and where rows differ)
  int phases;          // tiles of a row, each a wave's
  int wpp, wpp_inv;    // row sets of a workgroup, which has wpp * phases waves; ceil(65536 / wpp)
  int red_stride;      // floats from one unit's sums to the next's: the rows of a workgroup, odd
  int split;           // log2 of the threads that add up a row
  int gshift;          // group = unit << gshift columns
  int groups_per_row;
  int npieces;         // 16-byte pieces of x
  int units;           // units of x in LDS
  int blocks;          // CODES_MIXED: blocks of 64 spans of 32 columns of a row
  int span_shift;      // and log2 of the lanes a row has in a block
  uint32_t val_row, idx_row;                          // bytes of a row (uniform rows)
  uint32_t slots_row;                                 // slots of a row; CODES_MIXED: of a row that keeps one of four
  uint32_t total_slots;                               // CODES_MIXED
  uint32_t val_bytes, idx_bytes, qp_bytes;            // extents of the arrays
  uint32_t nib_mask, nib_magic, nib_magic2;
};
struct CodesPtrs {
  const uint32_t *row_ptr;
  const uint8_t *values, *idx, *qparams;
  const __half *x;
  __half *y;
};

// bytes of codes and of index words that a lane fetches for a chunk of CPL columns
constexpr int codes_vb(int form, int cpl) { return form == CODES_DENSE ? cpl / 2 : form == CODES_14 ? cpl / 8 : cpl / 4; }
constexpr int codes_ib(int form, int cpl) { return form == CODES_DENSE ? 0 : form == CODES_14 ? cpl / 16 : cpl / 8; }

constexpr int codes_units(int form, int cpl, int unit) { return form == CODES_DENSE && 4 * cpl == unit ? 16 : 32; }
typedef float f16v __attribute__((ext_vector_type(16)));

template <int FORM, int CPL>
struct CodesTile {
  static constexpr int VW = (codes_vb(FORM, CPL) + 3) / 4, IW = FORM == CODES_DENSE ? 1 : (codes_ib(FORM, CPL) + 3) / 4;
  uint32_t v[VW], iw[IW], qp;
};

// B bytes at lane offset `lane` + uniform offset `uni`, zero-extended
template <int B, int VW>
__device__ __forceinline__ void codes_fetch(uint32_t (&v)[VW], __amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t uni) {
  if constexpr (B == 16) {
    const u4 t = __builtin_amdgcn_raw_buffer_load_b128(r, lane, uni, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = t[j];
  } else if constexpr (B == 8) {
    const u2 t = __builtin_amdgcn_raw_buffer_load_b64(r, lane, uni, 0);
    v[0] = t[0];
    v[1] = t[1];
  } else if constexpr (B == 4) {
    v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, lane, uni, 0);
  } else if constexpr (B == 2) {
    v[0] = __builtin_amdgcn_raw_buffer_load_b16(r, lane, uni, 0);
  } else {
    v[0] = __builtin_amdgcn_raw_buffer_load_b8(r, lane, uni, 0);
  }
}

// {slot 2 p, slot 2 p + 1} of a word of eight codes as the FP16 integers q - z; off: {1024 + z, 64 + z}
__device__ __forceinline__ uint32_t codes_pair(uint32_t d, int p, uint32_t off, uint32_t mask, uint32_t magic) {
  return pk_sub_f16(and_or(__builtin_amdgcn_perm(d, d, 0x0c000c00u + (uint32_t)p * 0x00010001u), mask, magic), off);
}

// 32 columns of a row that keeps N of four: its N words of codes and of indices, its parameter pair and its activations (half2
// registers): s sum (q - z) x, of the kept columns alone.
struct CodesSpan {
  uint32_t v[4], iw[3], qp;
};
template <int N>
__device__ __forceinline__ float codes_span_dot(const CodesSpan &in, const u4 (&x)[4], uint32_t nib_mask, uint32_t nib_magic, uint32_t magic) {
  const uint32_t off = pk_add_f16(__builtin_amdgcn_perm(in.qp, in.qp, 0x03020302u), nib_magic);
  float sum = 0.f;
#pragma unroll
  for (int p = 0; p < 4 * N; ++p) {
    const h2 v = __builtin_bit_cast(h2, codes_pair(in.v[p / 4], p % 4, off, nib_mask, magic));
#pragma unroll
    for (int k = 2 * p; k < 2 * p + 2; ++k) {          // slot k, of 4-group k / N
      const uint32_t x01 = x[k / N / 2][2 * (k / N % 2)], x23 = x[k / N / 2][2 * (k / N % 2) + 1];
      _Float16 xk;
      if constexpr (N == 4) {
        xk = __builtin_bit_cast(h2, k & 2 ? x23 : x01)[k & 1];                                   // (all four: the offsets of a 4-group ascend)
      } else {
        const uint32_t o = (in.iw[k / 8 < 3 ? k / 8 : 0] >> (2 * (k % 8))) & 3u;
        xk = __builtin_bit_cast(h2, __builtin_amdgcn_perm(x23, x01, 0x0100u + 0x0202u * o))[0];
      }
      sum = fmaf((float)v[k & 1], (float)xk, sum);
    }
  }
  return __half2float(__ushort_as_half((uint16_t)(in.qp & 0xFFFFu))) * sum;
}

// Rows of a workgroup that the matrix cores do not take (the bits of `wide`), on the vector units, a span of 32 columns a lane (one
// quantisation group, one unit of x).  A row is cut into blocks of 64 spans; PACKED: rows of 32 spans and fewer, of which a block
// holds two or four.  Blocks are dealt to the waves, which request two before they use the first.  `kept`, lane j: row j's first
// slot and in the low bits what it keeps.  Every sixteen lanes leave a sum.
// Measured, us, 11008 x 4096 with a half, a quarter and a tenth of rows that keep three or four: 11.4, 9.4 and 7.6, slot by slot 18.3, 14.4
// and 13.9; where these rows were followed slot by slot beside the others, a wave a row, 28.2, 18.3 and 18.0.
template <int UNIT, bool PACKED>
__device__ __forceinline__ void codes_wide_rows(const uint8_t *xs, float *part, uint64_t wide, uint32_t kept, __amdgpu_buffer_rsrc_t r_val,
                                                __amdgpu_buffer_rsrc_t r_idx, __amdgpu_buffer_rsrc_t r_qp, const CodesGeom &g, int wave, int nw, int lane, uint32_t magic) {
  constexpr uint32_t OUT = 0x7FFFFFF0u;
  constexpr int QM = UNIT / 8 > 16 ? 15 : UNIT / 8 - 1;
  const int spans = g.npieces / 4, rows_of_block = PACKED ? 64 >> g.span_shift : 1, group = PACKED ? lane >> g.span_shift : 0;
  const int lane_of_row = PACKED ? lane & ((1 << g.span_shift) - 1) : lane;
  uint64_t left = wide;                               // the block in turn: of the row of the lowest bit, or of the lowest bits
  int block = 0;
  auto advance = [&](int by) {
    for (block += by; block >= g.blocks && left != 0; block -= g.blocks)
      for (int k = 0; k < rows_of_block; ++k) left &= left - 1;
  };
  advance(wave);
  while (left != 0) {
    CodesSpan in[2];
    int in_n[2], in_row[2], in_block[2];
    bool any[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t from = 0;                              // of this lane's row: uniform unless PACKED
      int row = 0;
      if constexpr (PACKED) {
        uint64_t rest = left;
        for (int k = 0; k < rows_of_block && rest != 0; ++k, rest &= rest - 1) {
          const int r = __builtin_ctzll(rest);
          const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)kept, r);
          from = group == k ? f : from;
          row = group == k ? r : row;
        }
      } else if (left != 0) {
        row = __builtin_ctzll(left);
        from = (uint32_t)__builtin_amdgcn_readlane((int)kept, row);
      }
      const int n = (int)(from & 7u), span = 64 * block + lane_of_row;
      const uint32_t word = (from >> 3) + (uint32_t)(n * span);
      const bool on = span < spans;
      in_n[u] = n;
      in_row[u] = row;
      in_block[u] = block;
      any[u] = left != 0;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        in[u].v[d] = __builtin_amdgcn_raw_buffer_load_b32(r_val, on && d < n ? 4 * (word + d) : OUT, 0u, 0);
        if (d < 3) in[u].iw[d] = __builtin_amdgcn_raw_buffer_load_b16(r_idx, on && d < n && n < 4 ? 2 * (word + d) : OUT, 0u, 0);
      }
      in[u].qp = __builtin_amdgcn_raw_buffer_load_b32(r_qp, on && n != 0 ? 4 * (uint32_t)(row * g.groups_per_row + (32 * span / UNIT >> g.gshift)) : OUT, 0u, 0);
      advance(nw);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (!any[u]) break;
      const int span = 64 * in_block[u] + lane_of_row;
      const bool on = span < spans && in_n[u] != 0;
      float sum = 0.f;
      if (on) {
        const uint32_t at = (uint32_t)(64 * span) ^ (uint32_t)(16 * ((32 * span / UNIT) & QM));  // (the swizzle of its unit)
        u4 x[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) x[d] = *(const u4 *)(xs + (at ^ (uint32_t)(16 * d)));
        if (in_n[u] == 1) sum = codes_span_dot<1>(in[u], x, g.nib_mask, g.nib_magic, magic);
        if (in_n[u] == 2) sum = codes_span_dot<2>(in[u], x, g.nib_mask, g.nib_magic, magic);
        if (in_n[u] == 3) sum = codes_span_dot<3>(in[u], x, g.nib_mask, g.nib_magic, magic);
        if (in_n[u] == 4) sum = codes_span_dot<4>(in[u], x, g.nib_mask, g.nib_magic, magic);
      }
      sum += row_shl<8>(sum);
      sum += row_shl<4>(sum);
      sum += row_shl<2>(sum);
      sum += row_shl<1>(sum);
      if ((lane & 15) == 0 && on) part[4 * (in_row[u] * g.blocks + in_block[u]) + (lane_of_row >> 4)] = sum;
    }
  }
}

// FORM: CODES_*.  CPL: columns of a chunk.  UNITS: of a tile.  MP: a row takes several tiles.
template <int FORM, int CPL, int UNITS, int TPI, bool MP>
__device__ __forceinline__ void codes_body(const CodesPtrs &P, const CodesGeom &g) {
  extern __shared__ __align__(16) uint8_t xs[];       // x, then the quads' sums of the workgroup's rows
  constexpr bool DENSE = FORM == CODES_DENSE, MIXED = FORM == CODES_MIXED, PAIRED = FORM == CODES_24P;
  constexpr int LOADS = DENSE ? 2 : MIXED ? 5 : 3;        // (requests of a tile)
  constexpr int VB = codes_vb(FORM, CPL), IB = codes_ib(FORM, CPL);
  constexpr uint32_t OUT = 0x7FFFFFF0u;               // past every buffer (they are below 2 GiB): zeros, no traffic
  constexpr int L = 64 / UNITS, QB = 2 * L * CPL, QP = QB / 16, QM = QP > 16 ? 15 : QP - 1;   // chunks of a unit; a unit of x: bytes, pieces, and the bits of its number that move them
  typedef CodesTile<FORM, CPL> Tile;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  const int ps = (wave * g.wpp_inv) >> 16, slot = wave - ps * g.wpp;       // phase, row set
  const int i = lane % UNITS, kb = lane / UNITS;
  // ---- this wave's rows: TPI row groups; this workgroup's from wg_row0 on
  const int rpw = MP ? TPI : TPI * g.rpt;
  const int wg_row0 = (int)blockIdx.x * g.wpp * rpw, row0 = wg_row0 + slot * rpw;
  // The wave's buffers begin at its first row and end with the matrix (for a wave past the last row they are empty), and a
  // request's place in them lies in its lane offset as a whole: a row past the last one lies past the buffer.  (A uniform
  // offset is only added where it is below the buffer's size: the range check subtracts it from the size.)  Buffers begin on
  // four bytes; rows of index words at 1:4 in groups of 32 on two, the rest goes into the lane offset.
  const uint32_t row_base = (uint32_t)min(MIXED ? wg_row0 : row0, g.rows), i_row = MIXED ? 0u : row_base * g.idx_row, i_rest = IB == 1 ? i_row & 3u : 0u;
  const uint32_t v_base = MIXED ? 0u : row_base * g.val_row, i_base = i_row - i_rest, q_base = 4u * row_base * (uint32_t)g.groups_per_row;
  const __amdgpu_buffer_rsrc_t r_val = make_rsrc(P.values + v_base, g.val_bytes - v_base), r_idx = make_rsrc(P.idx + i_base, g.idx_bytes - i_base);
  const __amdgpu_buffer_rsrc_t r_qp = make_rsrc(P.qparams + q_base, g.qp_bytes - q_base), r_x = make_rsrc(P.x, 16u * (uint32_t)g.npieces);
  uint32_t rp = 0, rp_end = 0;                        // rows differ: lane j holds the row pointers of row wg_row0 + j and the next
  const int own = MIXED ? slot * TPI : 0;             // (of which this wave's begin here; a workgroup has at most 64 rows)
  if constexpr (MIXED) {
    if (wg_row0 + lane < g.rows) {
      rp = P.row_ptr[wg_row0 + lane];
      rp_end = P.row_ptr[wg_row0 + lane + 1];
    }
  }

  // ---- x: one request per kilobyte; lane l delivers to byte 16 l
  const int kib = (g.units * QB + 1023) >> 10;
  asm volatile("" ::: "memory");
  for (int u = wave; u < kib; u += nw) {
    const int Q = (64 / QP) * u + lane / QP, s = lane % QP;
    const int piece = QP * Q + (s ^ (Q & QM));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(xs + 1024 * u), 16,
                                             piece < g.npieces ? 16u * (uint32_t)piece : OUT, 0u, 0, 0);
  }
  asm volatile("" ::: "memory");

  const int rs = MP ? 0 : (i * g.upr_inv) >> 16, ui = MP ? i : i - rs * g.upr;   // row inside the tile, unit inside the row
  const int cl = L * ui + kb;                         // chunk inside the row (of phase 0)
  const bool lane_on = rs < g.rpt;

  constexpr uint32_t ALIGN = CPL == 64 ? 15u : 7u;    // (chunks of 64 columns: 8 bytes of codes at a time)
  // Rows differ: entries per 4-group that a row between two row pointers keeps; 0: nothing of it may be read.
  auto lane_n = [&](uint32_t start, uint32_t end) -> int {
    const uint32_t len = end - start, q = g.slots_row;
    int n = len == q ? 1 : len == 2 * q ? 2 : len == 3 * q ? 3 : len == 4 * q ? 4 : 0;
    if ((start & 7u) != 0 || start > g.total_slots || len > g.total_slots - start) n = 0;
    return n;
  };
  // rows that keep three or four, and rows whose requests would not be aligned
  auto slot_by_slot = [&](int n, uint32_t start) { return n > 2 || (n != 0 && (start & ALIGN) != 0); };
  // Lane j: where row wg_row0 + j begins (whole words of eight slots), and in the low bits what it keeps; which rows the matrix cores
  // do not take.
  uint32_t kept = 0;
  uint64_t wide = 0;
  if constexpr (MIXED) {
    const int n = wg_row0 + lane < g.rows ? lane_n(rp, rp_end) : 0;
    kept = n ? rp | (uint32_t)n : 0u;
    wide = __ballot(lane < g.wpp * rpw && slot_by_slot(n, rp));
  }
  auto row_n = [&](int row) { return __builtin_amdgcn_readlane((int)kept, row) & 7; };

  auto load = [&](Tile (&t)[TPI], int p) {
    const bool on = lane_on & (cl < g.nchunks - (MP ? 64 * p : 0));
    const uint32_t v_lane = on ? (uint32_t)rs * g.val_row + (uint32_t)(VB * cl) + (uint32_t)(64 * VB * p) : OUT;
    const uint32_t i_lane = on ? (uint32_t)rs * g.idx_row + (uint32_t)(IB * cl) + (uint32_t)(64 * IB * p) + i_rest : OUT;
    const uint32_t grp = (uint32_t)((ui + (MP ? UNITS * p : 0)) >> g.gshift);
    const uint32_t q_lane = on ? 4u * ((uint32_t)rs * (uint32_t)g.groups_per_row + grp) : OUT;
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const uint32_t r = (uint32_t)(MIXED ? own + k : k * g.rpt);       // from the buffers' first row on
      if constexpr (MIXED) {
        const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)kept, own + k) & ~7u;
        const int n = (wide >> (own + k)) & 1 ? 0 : row_n(own + k);
        // the halves of a chunk at 2:4, of which a chunk at 1:4 is the first (a branch would be waited behind)
        constexpr int VH = VB / 2, IH = IB / 2;
        const uint32_t s_v = n ? (start >> 1) + (uint32_t)(64 * VH * n) * (uint32_t)p : 0u, s_i = s_v >> 1;
        const uint32_t lc = (uint32_t)(n * cl);
        const bool on1 = on & (n != 0), on2 = on & (n == 2);
        uint32_t h[2][(VH + 3) / 4], j[2][1];
        codes_fetch<VH>(h[0], r_val, on1 ? VH * lc : OUT, s_v);
        codes_fetch<VH>(h[1], r_val, on2 ? VH * lc + VH : OUT, s_v);
        codes_fetch<IH>(j[0], r_idx, on1 ? IH * lc : OUT, s_i);
        codes_fetch<IH>(j[1], r_idx, on2 ? IH * lc + IH : OUT, s_i);
        if constexpr (VH >= 4) {
#pragma unroll
          for (int d = 0; d < VB / 4; ++d) t[k].v[d] = h[d / (VB / 8)][d % (VB / 8)];
        } else {
          t[k].v[0] = h[0][0] | (h[1][0] << 16);
        }
        t[k].iw[0] = IB == 8 ? j[0][0] : j[0][0] | (j[1][0] << (4 * IB));
        t[k].iw[IB == 8] = IB == 8 ? j[1][0] : t[k].iw[0];
      } else {
        codes_fetch<VB>(t[k].v, r_val, v_lane + r * g.val_row, 0u);
        if constexpr (!DENSE) codes_fetch<IB>(t[k].iw, r_idx, i_lane + r * g.idx_row, 0u);
      }
      t[k].qp = __builtin_amdgcn_raw_buffer_load_b32(r_qp, q_lane + 4u * r * (uint32_t)g.groups_per_row, 0u, 0);
    }
  };

  // ---- B operand of a phase.  Sparse: lane (n, b) supplies the k-octets b and L + b of instruction d, that
  //      is columns 16 d + 8 (b & 1) of the chunks b >> 1 and L / 2 + (b >> 1) of unit n.  Dense: columns 8 d of chunk b.
  constexpr int NB = DENSE ? CPL / 8 : CPL / 16;      // instructions of a tile
  constexpr int CP = CPL / 8;                         // pieces of a chunk
  const int b_piece = DENSE ? CP * kb : CP * (kb >> 1) + (kb & 1);
  const uint32_t b0 = (uint32_t)(QB * ui + 16 * (b_piece ^ (ui & QM)));
  u8v bs[DENSE ? 1 : NB];
  u4 bd[DENSE ? NB : 1];
  auto read_b = [&](int p) {
    const uint8_t *at = xs + (MP ? UNITS * QB * p : 0);
#pragma unroll
    for (int d = 0; d < NB; ++d) {
      if constexpr (DENSE) {
        bd[d] = *(const u4 *)(at + (b0 ^ (uint32_t)(16 * d)));
      } else {
        const uint32_t q = b0 ^ (uint32_t)(32 * d);
        const u4 lo = *(const u4 *)(at + q), hi = *(const u4 *)(at + (q ^ (uint32_t)(8 * L * CP)));
        bs[d] = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
    }
  };

  const uint32_t magic = in_vgpr(g.nib_magic), magic2 = PAIRED ? in_vgpr(g.nib_magic2) : 0u;
  const uint32_t magic1 = in_vgpr(0x64006400u), magic6 = in_vgpr(0x54005400u);                  // FP16 {1024, 1024}, {64, 64}
  float val[TPI];
  auto consume = [&](const Tile (&t)[TPI]) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const uint32_t qp = t[k].qp;
      const uint32_t zz = __builtin_amdgcn_perm(qp, qp, 0x03020302u);                            // {z, z}
      const uint32_t off = pk_add_f16(zz, g.nib_magic), off2 = PAIRED ? pk_add_f16(zz, g.nib_magic2) : 0u;
      float scale = __half2float(__ushort_as_half((uint16_t)(qp & 0xFFFFu)));
      typedef float D __attribute__((ext_vector_type(UNITS == 16 ? 4 : 16)));
      D acc = 0.f;
      if constexpr (DENSE) {
#pragma unroll
        for (int d = 0; d < NB; ++d) {
          u4 a;
#pragma unroll
          for (int q = 0; q < 4; ++q) a[q] = codes_pair(t[k].v[d], q, off, g.nib_mask, magic);
          if constexpr (UNITS == 16) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, bd[d]), acc, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, bd[d]), acc, 0, 0, 0);
        }
      } else {
        auto multiply = [&](const u4 &a, int d, uint32_t iw) {
          if (d & 1) acc = __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bs[DENSE ? 0 : d]), acc, (int)iw, 0, 1);
          else acc = __builtin_amdgcn_smfmac_f32_32x32x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bs[DENSE ? 0 : d]), acc, (int)iw, 0, 0);
        };
        auto one_of_four = [&] {
          const uint32_t off1 = __builtin_amdgcn_perm(off, off, 0x01000100u);                    // {1024 + z, 1024 + z}
          const uint32_t off6 = __builtin_amdgcn_perm(off, off, 0x03020302u);                    // {64 + z, 64 + z}
          scale *= 0.5f;
          uint32_t iw = 0;
#pragma unroll
          for (int d = 0; d < NB; ++d) {
            if (d % 2 == 0) {
              iw = d ? spread_idx<1>(t[k].iw[0], 0x0F0F0F0Fu, 0x33333333u) : spread_idx<0>(t[k].iw[0], 0x0F0F0F0Fu, 0x33333333u);
              iw |= iw << 2;
            }
            u4 a;                                     // slot 4 d + q in both halves
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint32_t w = __builtin_amdgcn_perm(t[k].v[d / 2], t[k].v[d / 2], 0x0c000c00u + (uint32_t)(2 * (d & 1) + (q >> 1)) * 0x00010001u);
              a[q] = q & 1 ? pk_sub_f16(and_or(w, 0x00F000F0u, magic6), off6) : pk_sub_f16(and_or(w, 0x000F000Fu, magic1), off1);
            }
            multiply(a, d, iw);
          }
        };
        auto two_of_four = [&] {
#pragma unroll
          for (int d = 0; d < NB; ++d) {
            const uint32_t w = t[k].v[d < Tile::VW ? d : 0];
            u4 a;
            if constexpr (PAIRED) {
              const uint32_t w8 = w >> 8;
              a[0] = pk_sub_f16(and_or(w, g.nib_mask, magic), off);
              a[1] = pk_sub_f16(and_or(w, g.nib_mask << 4, magic2), off2);
              a[2] = pk_sub_f16(and_or(w8, g.nib_mask, magic), off);
              a[3] = pk_sub_f16(and_or(w8, g.nib_mask << 4, magic2), off2);
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) a[q] = codes_pair(w, q, off, g.nib_mask, magic);
            }
            multiply(a, d, t[k].iw[d / 2 < Tile::IW ? d / 2 : 0]);
          }
        };
        if constexpr (FORM == CODES_14) {
          one_of_four();
        } else if constexpr (MIXED) {
          if (row_n(own + k) == 1) one_of_four();           // (the same for all lanes; a row of neither kind is zeros)
          else two_of_four();
        } else {
          two_of_four();
        }
      }
      // diagonal i: UNITS = 16 lane i + 16 (i / 4), register i % 4; UNITS = 32 lane i + 32 (i / 4 % 2), register 4 (i / 8) + i % 4
      float d[UNITS / 8];
#pragma unroll
      for (int q = 0; q < UNITS / 16; ++q) d[q] = select4(lane & 3, acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
      if constexpr (UNITS == 32) {
#pragma unroll
        for (int q = 2; q < 4; ++q) d[q] = select4(lane & 3, acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        d[0] = select4(i >> 3, d[0], d[1], d[2], d[3]);
      }
      val[k] = scale * d[0];
    }
  };

  // ---- the tiles are requested, then x of this wave's requests is waited for (requests return in order)
  Tile t[TPI];
  load(t, ps);
  wait_vmem<TPI * LOADS>();
  // (2^split threads add up a row; the first of them stores it, and asks for its row pointers now)
  const int out_k = (int)threadIdx.x >> g.split, out_part = (int)threadIdx.x & ((1 << g.split) - 1), out_row = wg_row0 + out_k;
  const bool in_wg = out_k < g.wpp * rpw;
  bool out_on = in_wg && out_part == 0 && out_row < g.rows;
  uint32_t out_rp = 0, out_end = 0;
  if (!DENSE && out_on) {
    out_rp = P.row_ptr[out_row];
    if (MIXED) out_end = P.row_ptr[out_row + 1];
  }
  for (int pc = g.npieces + (int)threadIdx.x; pc < (kib << 10) / 16; pc += (int)blockDim.x) {   // pieces past the end of x
    const int Q = pc / QP, s = pc % QP;
    *(u4 *)(xs + QB * Q + 16 * (s ^ (Q & QM))) = u4{0, 0, 0, 0};
  }
  lds_barrier();
  read_b(ps);
  consume(t);

  // [phase][unit of a row][row of the workgroup]; rows differ: then four sums for each [row of the workgroup][block]
  float *red = (float *)(xs + (size_t)kib * 1024);
  if (kb == ((i >> 2) & (L - 1)) && lane_on) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) red[(ps * g.upr + ui) * g.red_stride + slot * rpw + k * g.rpt + rs] = val[k];
  }
  lds_barrier();
  float v = 0.f;
  if (in_wg) {
#pragma unroll 4
    for (int k = out_part; k < g.phases * g.upr; k += 1 << g.split) v += red[k * g.red_stride + out_k];
  }
  if (g.split > 3) v += row_shl<8>(v);
  if (g.split > 2) v += row_shl<4>(v);
  if (g.split > 1) v += row_shl<2>(v);
  if (g.split > 0) v += row_shl<1>(v);
  bool ok = true;
  if constexpr (!DENSE && !MIXED) ok = out_rp == (uint32_t)out_row * g.slots_row;
  if constexpr (MIXED) {
    const int n = lane_n(out_rp, out_end);
    ok = n != 0;
    if (slot_by_slot(n, out_rp)) out_on = false;      // (below)
  }
  if (out_on) P.y[out_row] = ok ? __float2half(v) : __ushort_as_half((uint16_t)0x7E00);

  if constexpr (MIXED) {
    // The other rows of the workgroup.  (Rows of several tiles have more than 1024 columns, rows of one in groups of 32 as many at most.)
    if (wide == 0) return;
    float *part = red + g.phases * g.upr * g.red_stride;
    const bool packed = !MP && (CPL == 16 || g.span_shift < 6);
    if (packed) {
      if constexpr (!MP) codes_wide_rows<L * CPL, true>(xs, part, wide, kept, r_val, r_idx, r_qp, g, wave, nw, lane, magic);
    } else {
      if constexpr (MP || CPL > 16) codes_wide_rows<L * CPL, false>(xs, part, wide, kept, r_val, r_idx, r_qp, g, wave, nw, lane, magic);
    }
    lds_barrier();
    if (threadIdx.x < 64 && ((wide >> lane) & 1)) {
      float v = 0.f;
      for (int k = 0; k < (g.npieces / 4 + 15) / 16; ++k) v += part[4 * lane * g.blocks + k];
      P.y[wg_row0 + lane] = __float2half(v);
    }
  }
}

template <int FORM, int CPL, int UNITS, int TPI, bool MP>
__global__ __launch_bounds__(1024) void k_codes(const uint32_t *__restrict__ row_ptr, const uint8_t *__restrict__ values,
                                                  const uint8_t *__restrict__ idx, const uint8_t *__restrict__ qparams,
                                                  const __half *__restrict__ x, __half *__restrict__ y, const CodesGeom g) {
  const CodesPtrs P{row_ptr, values, idx, qparams, x, y};
  codes_body<FORM, CPL, UNITS, TPI, MP>(P, g);
}
// Up to four identically shaped matrices, blockIdx.y names the member.
template <int FORM, int CPL, int UNITS, int TPI, bool MP>
__global__ __launch_bounds__(1024) void k_codes_batch(const GemvBatch b, const CodesGeom g) {
  const unsigned k = blockIdx.y;
  const CodesPtrs P{pick4(b.row_ptr, k), pick4(b.values, k), pick4(b.idx, k), pick4(b.qparams, k), pick4(b.x, k), pick4(b.y, k)};
  codes_body<FORM, CPL, UNITS, TPI, MP>(P, g);
}

namespace {

// Everything but the pointers and the launch shape.  Rows are whole units: a group is a multiple of one and divides the row.
bool codes_geometry(int form, int rows, int cols, int n_keep, int group, uint32_t total_slots, CodesGeom &g, int &cpl) {
  const bool dense = form == CODES_DENSE, mixed = form == CODES_MIXED;
  if (rows < 1 || cols < 32 || cols > 24576 || cols % group != 0) return false;   // (x in LDS: 48 KB)
  const int unit = group >= 128 ? 128 : group == 64 || group == 32 ? group : 0;
  if (unit == 0) return false;
  cpl = dense && unit == 128 ? 32 : unit / 2;
  const int per_tile = codes_units(form, cpl, unit);
  g.gshift = 0;
  while ((unit << g.gshift) < group) ++g.gshift;
  if (unit << g.gshift != group) return false;
  g.rows = rows;
  g.nchunks = cols / cpl;
  const int units = cols / unit;
  g.phases = (units + per_tile - 1) / per_tile;
  if (g.phases > CODES_WAVES) return false;
  if (g.phases > 1 && (form == CODES_24 || form == CODES_24P) && cpl == 64) return false;   // (4096 columns and more: egt_mfma_m1.hip)
  if (g.phases > 1 && dense && unit == 128) return false;                                   // (2048 columns and more: egt_mfma_dense.hip)
  g.upr = g.phases > 1 ? per_tile : units;
  g.upr_inv = (65536 + g.upr - 1) / g.upr;
  g.rpt = g.phases > 1 || mixed ? 1 : std::min(per_tile / g.upr, 16);
  g.groups_per_row = cols / group;
  g.npieces = cols / 8;
  g.blocks = (cols + 2047) / 2048;
  g.span_shift = cols <= 512 ? 4 : cols <= 1024 ? 5 : 6;
  g.units = g.phases > 1 ? per_tile * g.phases : units;
  const int n = n_keep ? n_keep : 1;
  g.val_row = dense ? (uint32_t)cols / 2 : mixed ? 0u : (uint32_t)(n * (cols / 8));
  g.idx_row = dense || mixed ? 0u : (uint32_t)(n * (cols / 16));
  g.slots_row = (uint32_t)(n * (cols / 4));
  g.total_slots = total_slots;
  const uint64_t vb = mixed ? total_slots / 2 : (uint64_t)rows * g.val_row, qb = 4ull * (uint64_t)rows * (uint64_t)g.groups_per_row;
  if (vb >= 0x7FFF0000ull || qb >= 0x7FFF0000ull) return false;            // (see OUT)
  g.val_bytes = (uint32_t)vb;
  g.idx_bytes = dense ? 0u : mixed ? total_slots / 4 : (uint32_t)((uint64_t)rows * g.idx_row);
  g.qp_bytes = (uint32_t)qb;
  const bool paired = form == CODES_24P;
  g.nib_mask = paired ? 0x000F000Fu : 0x00F0000Fu;
  g.nib_magic = paired ? 0x64006400u : 0x54006400u;
  g.nib_magic2 = 0x54005400u;
  return true;
}

// The waves of a workgroup are the phases of `wpp` row sets.
void codes_shape(CodesGeom &g, int unit, int form, int count, int &tpi, dim3 &grid, dim3 &block, size_t &lds) {
  const size_t x_bytes = ((size_t)g.units * (size_t)(2 * unit) + 1023) & ~(size_t)1023;
  const int nrg = (g.rows + g.rpt - 1) / g.rpt;       // row groups
  // Few tiles: one or two to a wave, since the launch then lasts as long as a wave's instructions.  Us with 1, 2, 4 tiles a wave,
  // on either side of the lines: 2:4 2000 x 3072 2.9, 2.8, 3.2; 3000 3.1, 3.1, 3.3; 5000 3.8, 3.6, 4.0; 6000 4.05, 3.7, 4.1; 7000 4.4, 4.1, 4.1;
  // 11000 5.5, 5.1, 5.0 (1:4 and the paired order alike); rows that differ 5000 x 4096 4.4, 4.3, 5.0, 7000 5.3, 4.9, 5.1, 11000 6.9, 6.3, 6.1;
  // dense 1050 x 2880, two tiles a row, 2.9, 2.9, 3.1, 4000 4.3, 3.9, 3.8, 5000 4.8, 4.2, 4.4, 5200 5.0, 4.5, 4.4, 8000 6.3, 5.4, 5.1; dense 10000 x
  // 1664 4.3, 3.75, 4.0, 12000 4.8, 4.05, 4.1.  (Sparse rows of 5120 to 6500 tiles would gain up to a tenth with two.)
  const int64_t tiles = (int64_t)nrg * g.phases * count;
  tpi = tiles <= 2048 ? 1 : tiles <= (form == CODES_DENSE ? 10240 : 5120) ? 2 : 4;
  int waves = 4;                                      // (2, 6 and 8 waves: 1.1 to 1.5 times the time on 20000 x 2816 and 11008 x 4096)
  tune_pair("EGT_CODES_TUNE", waves, tpi);
  if (tpi != 1 && tpi != 2) tpi = 4;

  waves = waves < 1 ? 1 : waves > CODES_WAVES ? CODES_WAVES : waves;
  g.wpp = std::max(1, waves / g.phases);
  g.wpp_inv = (65536 + g.wpp - 1) / g.wpp;
  const int rows_wg = g.wpp * tpi * g.rpt, sets = (nrg + tpi - 1) / tpi;
  g.red_stride = rows_wg | 1;
  g.split = 0;
  // (the threads of a row fix the order of its additions, so they follow from the row alone, as if every wave had its four tiles:
  // a member of a batch has the bits of its own call)
  while (g.split < 4 && ((CODES_TPI * g.rpt) << (g.split + 1)) <= 64 * g.phases) ++g.split;
  lds = x_bytes + (size_t)g.phases * (size_t)g.upr * (size_t)g.red_stride * sizeof(float);
  if (form == CODES_MIXED) lds += (size_t)rows_wg * (size_t)(4 * g.blocks) * sizeof(float);   // (rows on the vector units)
  grid = dim3((unsigned)((sets + g.wpp - 1) / g.wpp));
  block = dim3(64u * (unsigned)(g.wpp * g.phases));
}

int codes_form(const egt_2bitcsr &w) {
  return w.val_kind == EGT_VAL_INT4_PAIRED ? CODES_24P : w.n_keep == 2 ? CODES_24 : w.n_keep == 1 ? CODES_14 : CODES_MIXED;
}

}  // namespace

// Where the slot-by-slot kernels are not the faster ones (their time over this kernel's, weights in the last-level cache).
//  - Groups of 64 and 32 make a tile 2048 and 1024 columns: a workgroup that stages a long row of x for four rows.  Two phases
//    at 1:4 and where rows differ, four otherwise, always win (30000 x 2592 groups of 32: dense 0.80, paired 0.81; 30000 x 2624
//    groups of 64: 1:4 0.90, rows differ 0.83), but for 1:4 in groups of 32 with many rows (1696 columns: 16000 rows 0.94, 30000 1.03,
//    60000 1.13).  More phases while their waves are resident at a time (1:4 groups of 32: 5000 x 2592 0.78, 8000 0.93, 16000 1.05; 2:4 5000
//    x 5152 0.79, 8000 1.02); of long rows fewer: 1:4 and rows that
//    differ from five phases on up to 2048 rows (2000 and 3200 rows: 1:4 4128 columns 0.87, 1.13; 8256, groups of 64, 0.77, 1.27; rows that
//    differ 0.66, 1.20), 2:4 from nine phases on the same (8224 columns 0.78, 1.10; 12320 0.74, 1.14), dense 1024 (1000 and 2000 rows: 8224 columns
//    0.74, 1.14; 12320 0.69, 1.04).  Dense rows with groups of 64 win throughout (0.37 to 0.97), and groups of 128 and more.
//  - Dense rows of few columns: staging x costs what it saves (300 x 384 1.17, 1000 x 896 1.11, 2000 x 896 1.09; 4000 x 896 0.97,
//    300 x 1600 0.98).
//  - Rows of different lengths: a row that keeps three or four costs up to a third more than one of both other kinds together
//    and less than slot by slot (its time over slot by slot with half of the rows at three and four: 11008 x 4096 0.67, 20000 x 1024
//    0.95), on rows shorter than 768 columns more (20000 x 640 1.13, x 512 1.13, 3000 x 512 1.14).  What the rows keep is known here as an
//    average only: short rows half of which keep one, the others two, are at 1.5 (0.80 to 0.88), and up to 1.55 few keep three or four.
static bool codes_pay(int form, const CodesGeom &g, int unit) {
  const bool dense = form == CODES_DENSE;
  const int64_t cols = 8 * (int64_t)g.npieces;
  if (tune_flag("EGT_CODES_ALL")) return true;
  if (dense && cols < 1536 && g.rows * cols < 3500000) return false;
  if (form == CODES_MIXED && cols < 768 && 20 * (uint64_t)g.total_slots > 31 * (uint64_t)g.rows * g.slots_row) return false;
  if (unit == 128 || (dense && unit == 64)) return true;
  const bool one = form == CODES_14 || form == CODES_MIXED;
  if (form == CODES_14 && unit == 32 && g.phases == 2 && g.rows > 20000) return false;
  if (g.phases >= (one ? 5 : 9) && g.rows > (dense ? 1024 : 2048)) return false;
  return g.phases <= (one ? 2 : 4) || (int64_t)g.phases * ((g.rows + CODES_TPI - 1) / CODES_TPI) <= (one ? 4096 : 8192);
}

// INT4 rows of up to 24576 columns and sixteen tiles, groups of 32 << j: 2:4 (either nibble order), 1:4, rows of different
// lengths (canonical order), dense.
bool sparse_codes_supported(const egt_2bitcsr &w) {
  CodesGeom g;
  int cpl;
  if (w.val_kind == EGT_VAL_INT4 ? w.n_keep > 2 : w.val_kind != EGT_VAL_INT4_PAIRED || w.n_keep != 2) return false;
  return codes_geometry(codes_form(w), w.rows, w.cols, w.n_keep, w.group_size, w.total_slots, g, cpl) && codes_pay(codes_form(w), g, 2 * cpl);
}
bool int4_codes_supported(int rows, int cols, int group) {
  CodesGeom g;
  int cpl;
  return codes_geometry(CODES_DENSE, rows, cols, 0, group, 0, g, cpl) && codes_pay(CODES_DENSE, g, std::min(group, 128));
}

template <int FORM, int CPL, int UNITS>
static hipError_t go(const GemvBatch &b, CodesGeom &g, int count, hipStream_t stream) {
  dim3 grid, block;
  size_t lds;
  int tpi;
  codes_shape(g, CPL * (64 / UNITS), FORM, count, tpi, grid, block, lds);
  grid.y = (unsigned)count;
#define EGT_C(TPI, MP)                                                                                                       \
  (FORM != CODES_MIXED && count > 1 ? launch(k_codes_batch<FORM == CODES_MIXED ? CODES_14 : FORM, CPL, UNITS, TPI, MP>, grid, block, lds, stream, b, g) \
             : launch(k_codes<FORM, CPL, UNITS, TPI, MP>, grid, block, lds, stream, b.row_ptr[0], b.values[0], b.idx[0], b.qparams[0], b.x[0], b.y[0], g))
#define EGT_T(MP) (tpi == 1 ? EGT_C(1, MP) : tpi == 2 ? EGT_C(2, MP) : EGT_C(4, MP))
  // (not of several tiles: sparse rows of whole 128s from 4096 columns on, dense rows of whole 128s from 2048 columns on, which are the
  // row-per-wave kernels'; dense rows of one tile in groups of 32 are 3400 tiles at least, see codes_pay)
  constexpr bool dense = FORM == CODES_DENSE, several = dense ? UNITS == 32 : !((FORM == CODES_24 || FORM == CODES_24P) && CPL == 64);
  if constexpr (several)
    if (g.phases > 1) return EGT_T(true);
  if constexpr (dense && CPL == 16) return tpi <= 2 ? EGT_C(2, false) : EGT_C(4, false);
  else return EGT_T(false);
#undef EGT_T
#undef EGT_C
}

// `count` identically shaped matrices, for rows of different lengths one.
hipError_t launch_sparse_codes(const egt_2bitcsr *ws, const uint16_t *const *xs, uint16_t *const *ys, int count, hipStream_t stream) {
  const egt_2bitcsr &w = ws[0];
  const int form = codes_form(w);
  CodesGeom g;
  int cpl;
  if (!codes_geometry(form, w.rows, w.cols, w.n_keep, w.group_size, w.total_slots, g, cpl) || (form == CODES_MIXED && count != 1)) return hipErrorInvalidValue;
  GemvBatch b = {};
  for (int k = 0; k < count; ++k) {
    b.row_ptr[k] = ws[k].row_ptr; b.values[k] = (const uint8_t *)ws[k].values; b.idx[k] = (const uint8_t *)ws[k].idx;
    b.qparams[k] = (const uint8_t *)ws[k].qparams; b.x[k] = (const __half *)xs[k]; b.y[k] = (__half *)ys[k];
  }
#define EGT_F(FORM) (cpl == 64 ? go<FORM, 64, 32>(b, g, count, stream) : cpl == 32 ? go<FORM, 32, 32>(b, g, count, stream) : go<FORM, 16, 32>(b, g, count, stream))
  switch (form) {
    case CODES_24: return EGT_F(CODES_24);
    case CODES_24P: return EGT_F(CODES_24P);
    case CODES_14: return EGT_F(CODES_14);
    default: return EGT_F(CODES_MIXED);
  }
#undef EGT_F
}

hipError_t launch_int4_codes(const uint8_t *const *qs, const uint16_t *const *qps, int rows, int cols, int group, const uint16_t *const *xs,
                             uint16_t *const *ys, int count, hipStream_t stream) {
  CodesGeom g;
  int cpl;
  if (!codes_geometry(CODES_DENSE, rows, cols, 0, group, 0, g, cpl)) return hipErrorInvalidValue;
  GemvBatch b = {};
  for (int k = 0; k < count; ++k) {
    b.values[k] = qs[k]; b.qparams[k] = (const uint8_t *)qps[k]; b.x[k] = (const __half *)xs[k]; b.y[k] = (__half *)ys[k];
  }
  if (cpl == 16) return go<CODES_DENSE, 16, 32>(b, g, count, stream);
  return group >= 128 ? go<CODES_DENSE, 32, 16>(b, g, count, stream) : go<CODES_DENSE, 32, 32>(b, g, count, stream);
}

}  // namespace egt
