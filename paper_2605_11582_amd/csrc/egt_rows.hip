// M = 1 products of matrices of any row length, on the matrix cores: 2:4, 1:4, rows of
// different lengths, dense INT4; 2:4 and 1:4 with FP16 values.
//
// The row-per-wave kernels (egt_mfma_m1.hip, egt_mfma_m1_n1.hip, egt_mfma_dense.hip) want
// rows that fill their tiles: 1024, 2048 or 4096 columns and more at 2:4.  Any other row used
// to be followed slot by slot - about seven vector instructions and an LDS gather per slot,
// 5 to 10 times what the matrix cores need.  Here a tile is 16 quads of four chunks (a chunk:
// 64 columns of a sparse INT4 row, 32 of a dense one, 16 bytes of FP16 values), and a row takes
// ceil(chunks / 4) of them: `rpt` whole rows lie in a tile, or a row lies in `phases` tiles.  Between a half and
// all of the lanes carry weights then; the rest ask out of range of the buffers (zeros, no
// traffic) and have scale 0.
//
// The mapping is the diagonal one: lane (i, kb) = i + 16 kb takes chunk kb of quad i, column n
// of B carries the activations of quad n, and D[i][i] is quad i's share of its row.  The 16
// diagonals of a tile are left in LDS; at the end of a wave one lane per row adds those of its
// quads (added tile by tile they were a chain of LDS latencies that 4 waves per SIMD did not hide).
//
//  - 1:4 rows keep the chunk of 64 columns (8 B of codes, 4 B of offsets) and with it the B
//    operand of 2:4 rows: a slot becomes the pair {value, 0}.  A matrix whose rows keep one or
//    two of four is so walked row by row, one branch per tile; a row that keeps three or four
//    is followed slot by slot.
//  - A wave owns up to 64 consecutive rows and walks them TPI tiles at a time with two sets of
//    registers, each requested again as soon as its tiles are used: sixteen waves per compute
//    unit keep up to 115 KB in flight.
//  - x goes from global memory straight into LDS (no registers, requested before the first
//    weights).  Piece s (16 bytes) of quad Q lies in slot s ^ (Q & 15) of its quad, so the
//    sixteen lanes of a B read, one quad each, fall into different banks (smaller quads: Q & 7).
//
// Measured, us per launch against the slot-by-slot kernels (weights in the last-level cache):
// 2:4 20000 x 2816 7.3 (24.7), 65536 x 2560 16.4, dense 31994 x 2304 12.3 (37), 5003 x 2880 4.9 (5.9),
// half of 11008 x 4096's rows at 1:4 7.4 (11.8), FP16 20000 x 2048 9.0 (the old form for 1024 and
// 2048 columns: 15.9).  What bounds it: vector issue at about 80 instructions a tile of at most
// 64 chunks, and memory beyond some 100 MB.  Shapes that fill the row-per-wave kernels' tiles
// stay with those (11008 x 4096: 5.1 against 6.0), which know tiles per row at compile time and
// request everything they need at once.
#include "egt_mfma_common.h"

#include "egt_dense_body.h"
#include "egt_tune.h"

#include <algorithm>

namespace egt {

enum { ROWS_24 = 0, ROWS_14 = 1, ROWS_MIXED = 2, ROWS_DENSE = 3, ROWS_F24 = 4, ROWS_F14 = 5 };
// columns of a chunk
constexpr int rows_chunk(int form) { return form == ROWS_DENSE || form == ROWS_F14 ? 32 : form == ROWS_F24 ? 16 : 64; }
// tiles in work at a time (a tile of FP16 values is a kilobyte and one or two instructions)
constexpr int rows_tpi(int form) { return form >= ROWS_F24 ? 4 : 2; }
constexpr int ROWS_PER_WAVE = 64;                     // rows a wave owns at most (a row pointer per lane)

struct RowsGeom {
  int rows;
  int nchunks;         // chunks of a row, the last one perhaps half empty (2:4)
  int qpr, qpr_inv;    // quads of a row inside a tile; ceil(65536 / qpr)
  int rpt;             // rows of a tile (1 where a row takes several)
  int phases;          // tiles of a row
  int nrg;             // row groups: ceil(rows / rpt)
  int batches;         // batches of TPI row groups a wave walks
  int red_stride;      // floats from one quad's sums to the next's: the rows of a wave, odd
  int gshift;          // columns of a quantisation group = chunk << gshift (sparse, groups of 64 and more); dense: 128 << gshift or 32 << gshift
  int groups_per_row;
  int npieces;         // 16-byte pieces of x
  int quads;           // quads of x in LDS
  uint32_t val_row, idx_row;                          // bytes of a row (uniform rows)
  uint32_t slots_row;                                 // slots of a row; ROWS_MIXED: of a row that keeps one of four
  uint32_t total_slots;                               // ROWS_MIXED
  uint32_t val_bytes, idx_bytes, qp_bytes;            // extents of the arrays
  uint32_t nib_mask, nib_magic, nib_magic2;
  uint32_t m8, m4, m2;
};
struct RowsPtrs {
  const uint32_t *row_ptr;
  const uint8_t *values, *idx, *qparams;
  const __half *x;
  __half *y;
};

template <int FORM, int QW>
struct RowsTile {
  u4 nib;                                             // 1:4: the low half
  u2 iw;                                              // 1:4: the low word
  uint32_t qp[QW];
};

// Four instructions of a sparse tile.
template <int QW, bool PAIRED>
__device__ __forceinline__ f4 rows_mfma_24(const u4 &nib, const u2 &iw, const uint32_t (&s2)[QW], const uint32_t (&off)[QW],
                                           const uint32_t (&off2)[QW], const u8v (&bx)[4], f4 acc, const RowsGeom &g, uint32_t magic,
                                           uint32_t magic2) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const u4 a = PAIRED ? dequant8_paired(nib[d], off[d * QW / 4], off2[d * QW / 4], s2[d * QW / 4], g.nib_mask, g.nib_mask << 4, magic, magic2)
                        : dequant8(nib[d], off[d * QW / 4], s2[d * QW / 4], g.nib_mask, magic);
    const int iword = (int)iw[d >> 1];
    if (d & 1) acc = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bx[d]), acc, iword, 0, 1);
    else acc = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bx[d]), acc, iword, 0, 0);
  }
  return acc;
}
// 1:4: instruction d takes slots 4 d .. 4 d + 3 of the chunk, bytes 2 (d & 1) and the next of dword d >> 1
template <int QW>
__device__ __forceinline__ f4 rows_mfma_14(const u4 &nib, uint32_t iw, const uint32_t (&s2)[QW], const uint32_t (&off)[QW],
                                           const u8v (&bx)[4], f4 acc, const RowsGeom &g, uint32_t magic) {
  const uint32_t sp[2] = {spread_idx(iw & 0xFFFFu, g.m8, g.m4, g.m2), spread_idx(iw >> 16, g.m8, g.m4, g.m2)};
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t dw = nib[d >> 1];
    u4 a;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint32_t t = __builtin_amdgcn_perm(dw, dw, 0x0c000c00u + (uint32_t)(2 * (d & 1) + p) * 0x00010001u);
      const uint32_t pair = pk_mul_f16(pk_sub_f16(and_or(t, g.nib_mask, magic), off[d * QW / 4]), s2[d * QW / 4]);
      a[2 * p] = pair & 0xFFFFu;
      a[2 * p + 1] = pair >> 16;
    }
    const int iword = (int)sp[d >> 1];
    if (d & 1) acc = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bx[d]), acc, iword, 0, 1);
    else acc = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h16, bx[d]), acc, iword, 0, 0);
  }
  return acc;
}

// FORM: ROWS_*.  QW: {scale, zero} pairs per sparse chunk (2: groups of 32); dense: 2 where the
// weights are scaled before the instruction (groups of 32 and 64), 1 where the sums are after it.
// MP: a row takes several tiles.  ODD: 2:4 rows of an odd number of 32 columns.  PAIRED: the
// paired nibble order.
template <int FORM, int QW, bool MP, bool ODD, bool PAIRED>
__device__ __forceinline__ void rows_body(const RowsPtrs &P, const RowsGeom &g) {
  extern __shared__ __align__(16) uint8_t xs[];       // x, then the quads' sums of every wave
  constexpr bool DENSE = FORM == ROWS_DENSE, MIXED = FORM == ROWS_MIXED, PRE = DENSE && QW == 2, F16 = FORM >= ROWS_F24;
  constexpr int TPI = rows_tpi(FORM), NQ = DENSE ? 1 : QW;   // NQ: parameter registers per tile
  // past every buffer (they are below 2 GiB), also with a uniform offset added: zeros, no traffic
  constexpr uint32_t OUT = 0x7FFFFFF0u;
  constexpr int QB = 8 * rows_chunk(FORM);            // bytes of a quad of x
  constexpr int QP = QB / 16, QM = QP > 16 ? 15 : QP - 1;   // its pieces, and the bits of Q that move them
  typedef RowsTile<FORM, NQ> Tile;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  const int i = lane & 15, kb = lane >> 4;
  const __amdgpu_buffer_rsrc_t r_val = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(P.values), 0, (int)g.val_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_idx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(P.idx), 0, (int)g.idx_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_qp = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(P.qparams), 0, (int)g.qp_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(P.x), 0, 16 * g.npieces, 0x00020000);

  // ---- this wave's rows: row groups [rg0, rg0 + batches * TPI)
  const int rg0 = ((int)blockIdx.x * nw + wave) * g.batches * TPI;
  const int rg_end = rg0 + g.batches * TPI;
  const int row0 = rg0 * g.rpt;
  // lane j: the row pointer of row row0 + j (and of the next one)
  uint32_t rp = 0, rp_end = 0;
  if constexpr (!DENSE) {
    const int r = row0 + lane;
    if (r < g.rows) {
      rp = P.row_ptr[r];
      if (MIXED) rp_end = P.row_ptr[r + 1];
    }
  }

  // ---- x: one request per kilobyte; lane l delivers to byte 16 l
  const int kib = (g.quads * QB + 1023) >> 10;
  asm volatile("" ::: "memory");
  for (int u = wave; u < kib; u += nw) {
    const int Q = (64 / QP) * u + lane / QP, slot = lane % QP;
    const int piece = QP * Q + (slot ^ (Q & QM));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(xs + 1024 * u), 16,
                                             piece < g.npieces ? 16u * (uint32_t)piece : OUT, 0u, 0, 0);
  }
  asm volatile("" ::: "memory");

  const int rs = MP ? 0 : (i * g.qpr_inv) >> 16, qi = MP ? i : i - rs * g.qpr;   // row inside the tile, quad inside the row
  const int cl = 4 * qi + kb;                         // chunk inside the row (of phase 0)
  const bool lane_on = rs < g.rpt;
  const uint32_t v_lane = (uint32_t)rs * g.val_row + (uint32_t)(FORM == ROWS_14 ? 8 : 16) * (uint32_t)cl;
  const uint32_t i_lane = (uint32_t)rs * g.idx_row + (uint32_t)(F16 ? 2 : FORM == ROWS_14 ? 4 : 8) * (uint32_t)cl;
  // dense, scaled after the instruction: the pair of quad (lane & 15), whose diagonal the lane may hold
  const uint32_t q_lane = 4u * ((uint32_t)rs * (uint32_t)g.groups_per_row);

  // ROWS_MIXED: entries that a row between two row pointers keeps; 0: nothing of it may be read
  auto lane_n = [&](uint32_t start, uint32_t end) -> int {
    const uint32_t len = end - start, q = g.slots_row;
    int n = len == q ? 1 : len == 2 * q ? 2 : len == 3 * q ? 3 : len == 4 * q ? 4 : 0;
    if (q == 0 || (start & 7u) != 0 || start > g.total_slots || len > g.total_slots - start) n = 0;
    return n;
  };
  // (of row k of this wave)
  auto row_n = [&](int k, uint32_t &start) -> int {
    start = (uint32_t)__builtin_amdgcn_readlane((int)rp, k);
    return lane_n(start, (uint32_t)__builtin_amdgcn_readlane((int)rp_end, k));
  };

  auto load = [&](Tile (&t)[TPI], int rg, int p) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const int left = rg + k < rg_end ? g.rows - (rg + k) * g.rpt : 0;      // uniform; rows from this group on
      const bool on = lane_on && rs < left && cl < g.nchunks - (MP ? 64 * p : 0);
      const uint32_t r = (uint32_t)((rg + k) * g.rpt);
      if constexpr (MIXED) {
        uint32_t start;
        const int n = row_n(min(rg + k - rg0, ROWS_PER_WAVE - 1), start);
        // (both ways two requests, so that the waits stay exact)
        if (n == 1) {
          const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r_val, on ? 8u * (uint32_t)cl : OUT, (start >> 1) + 512u * (uint32_t)p, 0);
          t[k].nib = u4{v[0], v[1], 0, 0};
          t[k].iw[0] = __builtin_amdgcn_raw_buffer_load_b32(r_idx, on ? 4u * (uint32_t)cl : OUT, (start >> 2) + 256u * (uint32_t)p, 0);
          t[k].iw[1] = 0;
        } else {
          const bool on2 = on && n == 2;
          t[k].nib = __builtin_amdgcn_raw_buffer_load_b128(r_val, on2 ? 16u * (uint32_t)cl : OUT, on2 ? (start >> 1) + 1024u * (uint32_t)p : 0u, 0);
          t[k].iw = __builtin_amdgcn_raw_buffer_load_b64(r_idx, on2 ? 8u * (uint32_t)cl : OUT, on2 ? (start >> 2) + 512u * (uint32_t)p : 0u, 0);
        }
      } else if constexpr (F16) {
        t[k].nib = __builtin_amdgcn_raw_buffer_load_b128(r_val, on ? v_lane : OUT, left > 0 ? r * g.val_row + 1024u * (uint32_t)p : 0u, 0);
        t[k].iw[0] = __builtin_amdgcn_raw_buffer_load_b16(r_idx, on ? i_lane : OUT, left > 0 ? r * g.idx_row + 128u * (uint32_t)p : 0u, 0);
        continue;
      } else if constexpr (FORM == ROWS_14) {
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r_val, on ? v_lane : OUT, left > 0 ? r * g.val_row + 512u * (uint32_t)p : 0u, 0);
        t[k].nib = u4{v[0], v[1], 0, 0};
        t[k].iw[0] = __builtin_amdgcn_raw_buffer_load_b32(r_idx, on ? i_lane : OUT, left > 0 ? r * g.idx_row + 256u * (uint32_t)p : 0u, 0);
        t[k].iw[1] = 0;
      } else {
        // ODD: the half chunk at the end of a row is fetched with the half before it, so that the
        // last row of the matrix stays inside its buffers
        const bool half = ODD && cl == g.nchunks - 1 - (MP ? 64 * p : 0);
        // (it may be the first of its phase: the lane's offset then holds the phase's)
        const uint32_t v_p = 1024u * (uint32_t)p, i_p = 512u * (uint32_t)p;
        const uint32_t s = left > 0 ? r * g.val_row + (ODD ? 0u : v_p) : 0u;
        t[k].nib = __builtin_amdgcn_raw_buffer_load_b128(r_val, on ? (ODD ? v_lane + v_p - (half ? 8u : 0u) : v_lane) : OUT, s, 0);
        if constexpr (!DENSE) {
          const uint32_t s_i = left > 0 ? r * g.idx_row + (ODD ? 0u : i_p) : 0u;
          t[k].iw = __builtin_amdgcn_raw_buffer_load_b64(r_idx, on ? (ODD ? i_lane + i_p - (half ? 4u : 0u) : i_lane) : OUT, s_i, 0);
        }
      }
      const uint32_t s_q = left > 0 ? 4u * r * (uint32_t)g.groups_per_row : 0u;
      if constexpr (DENSE && !PRE) {
        const uint32_t grp = (uint32_t)((qi + (MP ? 16 * p : 0)) >> g.gshift);
        const bool on_q = lane_on && rs < left && 4 * qi < g.nchunks - (MP ? 64 * p : 0);
        t[k].qp[0] = __builtin_amdgcn_raw_buffer_load_b32(r_qp, on_q ? q_lane + 4u * grp : OUT, s_q, 0);
      } else if constexpr (NQ == 2) {
        const bool half = ODD && cl == g.nchunks - 1 - (MP ? 64 * p : 0);
        const u2 v = __builtin_amdgcn_raw_buffer_load_b64(r_qp, on ? q_lane + 8u * (uint32_t)(cl + (MP ? 64 * p : 0)) - (half ? 4u : 0u) : OUT, s_q, 0);
        t[k].qp[0] = v[0];
        t[k].qp[NQ - 1] = v[1];
      } else {
        const uint32_t grp = (uint32_t)((cl + (MP ? 64 * p : 0)) >> g.gshift);
        t[k].qp[0] = __builtin_amdgcn_raw_buffer_load_b32(r_qp, on ? q_lane + 4u * grp : OUT, s_q, 0);
      }
    }
  };

  // ---- B operand of a phase.  Sparse: lane (n, b) supplies the k-octets b and 4 + b of instruction
  //      d: pieces 8 (2 h + (b >> 1)) + 2 d + (b & 1) of quad n.  Dense: piece 4 b + d.
  //      FP16 values, 2:4: pieces 4 h + b; 1:4: pieces 8 h + 4 (b >> 1) + 2 e + (b & 1) of instruction e.
  const int xq = qi & QM;
  const int b_piece = DENSE ? 4 * kb : FORM == ROWS_F24 ? kb : FORM == ROWS_F14 ? 4 * (kb >> 1) + (kb & 1) : 8 * (kb >> 1) + (kb & 1);
  const uint32_t b0 = (uint32_t)(QB * qi + 16 * (b_piece ^ xq));
  constexpr int NB = FORM == ROWS_F24 ? 1 : FORM == ROWS_F14 ? 2 : 4;     // instructions of a tile
  u8v bs[DENSE ? 1 : NB];
  u4 bd[DENSE ? 4 : 1];
  auto read_b = [&](int p) {
    const uint8_t *at = xs + (MP ? 16 * QB * p : 0);
#pragma unroll
    for (int d = 0; d < NB; ++d) {
      if constexpr (F16) {
        const uint32_t q = b0 ^ (uint32_t)(32 * d);
        const u4 lo = *(const u4 *)(at + q), hi = *(const u4 *)(at + (q ^ (FORM == ROWS_F24 ? 64u : 128u)));
        bs[d] = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      } else if constexpr (DENSE) {
        bd[d] = *(const u4 *)(at + (b0 ^ (uint32_t)(16 * d)));
      } else {
        const uint8_t *q = at + (b0 ^ (uint32_t)(32 * d));
        const u4 lo = *(const u4 *)q, hi = *(const u4 *)(q + 256);
        bs[d] = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
    }
  };

  const uint32_t magic = in_vgpr(g.nib_magic), magic2 = PAIRED ? in_vgpr(g.nib_magic2) : 0u;
  float *red = (float *)(xs + (size_t)kib * 1024) + wave * (g.qpr * g.red_stride);   // [quad of a row][row of this wave]
  // The first two items of the walk are requested; then x of this wave's requests is waited for (requests
  // return in order, and LOADS of them fetch a tile, on or off).
  const int mine = min(g.batches, (g.nrg - rg0 + TPI - 1) / TPI);
  const int total = MP ? mine * g.phases : mine;
  constexpr int LOADS = DENSE || F16 ? 2 : 3;
  Tile ta[TPI], tb[TPI];
  load(ta, rg0, 0);
  load(tb, MP ? rg0 : rg0 + TPI, MP ? 1 : 0);
  wait_vmem<2 * TPI * LOADS>();
  for (int pc = g.npieces + (int)threadIdx.x; pc < (kib << 10) / 16; pc += (int)blockDim.x) {   // pieces past the end of x
    const int Q = pc / QP, s = pc % QP;
    *(u4 *)(xs + QB * Q + 16 * (s ^ (Q & QM))) = u4{0, 0, 0, 0};
  }
  lds_barrier();
  if (row0 >= g.rows) return;                         // (no barrier follows)
  if (!MP) read_b(0);

  f4 acc[TPI];
  float val[TPI];                                     // dense, scaled after the instruction
#pragma unroll
  for (int k = 0; k < TPI; ++k) {
    acc[k] = f4{0.f, 0.f, 0.f, 0.f};
    val[k] = 0.f;
  }

  auto consume = [&](const Tile (&t)[TPI], int rg, int p) {
    if (MP) read_b(p);
    float xsum = 0.f;
    if constexpr (DENSE && !PRE) {
      const u4 ones = {0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u};
      f4 xq4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < 4; ++d)
        xq4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, ones), __builtin_bit_cast(h8, bd[d]), xq4, 0, 0, 0);
      xsum = xq4[0];                                  // of quad (lane & 15)
    }
    const bool half = ODD && cl == g.nchunks - 1 - (MP ? 64 * p : 0);
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      u4 nib = t[k].nib;
      u2 iw = t[k].iw;
      if constexpr (FORM == ROWS_F24) {
        acc[k] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, nib), __builtin_bit_cast(h16, bs[0]), acc[k], (int)iw[0], 0, 0);
      } else if constexpr (FORM == ROWS_F14) {
        // slots 4 e .. 4 e + 3, each as {value, 0}
        const int sp = (int)spread_idx(iw[0], g.m8, g.m4, g.m2);
        const u4 lo = {nib[0] & 0xFFFFu, nib[0] >> 16, nib[1] & 0xFFFFu, nib[1] >> 16}, hi = {nib[2] & 0xFFFFu, nib[2] >> 16, nib[3] & 0xFFFFu, nib[3] >> 16};
        acc[k] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, lo), __builtin_bit_cast(h16, bs[0]), acc[k], sp, 0, 0);
        acc[k] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, hi), __builtin_bit_cast(h16, bs[NB - 1]), acc[k], sp, 0, 1);
      } else {
      uint32_t qp[NQ];
#pragma unroll
      for (int j = 0; j < NQ; ++j) qp[j] = t[k].qp[j];
      if (ODD && half) {
        nib = u4{nib[2], nib[3], 0, 0};
        iw = u2{iw[1], 0};
        qp[0] = qp[NQ - 1];
        qp[NQ - 1] = 0;
      }
      if constexpr (DENSE) {
        uint32_t s2 = 0, off = 0;
        if (PRE) {
          s2 = __builtin_amdgcn_perm(qp[0], qp[0], 0x01000100u);
          off = pk_add_f16(__builtin_amdgcn_perm(qp[0], qp[0], 0x03020302u), g.nib_magic);
        }
        f4 a4 = PRE ? acc[k] : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          u4 a = nibbles_to_f16(nib[d], g.nib_mask, magic);
          if (PRE) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = pk_mul_f16(pk_sub_f16(a[j], off), s2);
          }
          a4 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, bd[d]), a4, 0, 0, 0);
        }
        if (PRE) acc[k] = a4;
        else val[k] += dense_finish(select4(lane & 3, a4[0], a4[1], a4[2], a4[3]), qp[0], xsum);
      } else {
        uint32_t s2[NQ], off[NQ], off2[NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
          s2[j] = __builtin_amdgcn_perm(qp[j], qp[j], 0x01000100u);
          const uint32_t zz = __builtin_amdgcn_perm(qp[j], qp[j], 0x03020302u);
          off[j] = pk_add_f16(zz, g.nib_magic);
          off2[j] = PAIRED ? pk_add_f16(zz, g.nib_magic2) : 0u;
        }
        if constexpr (FORM == ROWS_14) {
          acc[k] = rows_mfma_14<NQ>(nib, iw[0], s2, off, bs, acc[k], g, magic);
        } else if constexpr (MIXED) {
          uint32_t start;
          const int n = row_n(min(rg + k, g.nrg - 1) - rg0, start);
          if (n == 1) acc[k] = rows_mfma_14<NQ>(nib, iw[0], s2, off, bs, acc[k], g, magic);
          else if (n == 2) acc[k] = rows_mfma_24<NQ, false>(nib, iw, s2, off, off2, bs, acc[k], g, magic, magic2);
        } else {
          acc[k] = rows_mfma_24<NQ, PAIRED>(nib, iw, s2, off, off2, bs, acc[k], g, magic, magic2);
        }
      }
      }
    }
  };

  // ---- diagonal i of tile k sits in lane i + 16 (i / 4), register i % 4: quad qi of row rs of its row group
  auto leave = [&](int rg) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const float d = (DENSE && !PRE) ? val[k] : select4(lane & 3, acc[k][0], acc[k][1], acc[k][2], acc[k][3]);
      if (kb == (i >> 2) && lane_on) red[qi * g.red_stride + (rg + k - rg0) * g.rpt + rs] = d;
      acc[k] = f4{0.f, 0.f, 0.f, 0.f};
      val[k] = 0.f;
    }
  };

  // ---- (batch, phase) one after the other; an item's registers are filled again, for the item after
  // the next, as soon as it has been used
  int rg = rg0, p = 0;
  auto advance = [&](int &r, int &q) {
    if (!MP || ++q == g.phases) { q = 0; r += TPI; }
  };
  auto step = [&](Tile (&cur)[TPI], int it) {
    consume(cur, rg, p);
    int r2 = rg, p2 = p;
    advance(r2, p2);
    advance(r2, p2);
    if (it + 2 < total) load(cur, r2, p2);
    if (!MP || p + 1 == g.phases) leave(rg);
    advance(rg, p);
  };
  for (int it = 0; it < total; it += 2) {
    step(ta, it);
    if (it + 1 < total) step(tb, it + 1);
  }

  // ---- lane j finishes row row0 + j
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int row = row0 + lane;
  const bool have = lane < g.batches * TPI * g.rpt && row < g.rows;
  float v = 0.f;
  if (have) {
    const float *q = red + lane;
#pragma unroll 4
    for (int k = 0; k < g.qpr; ++k) v += q[k * g.red_stride];
  }
  bool ok = true;
  if constexpr (!DENSE && !MIXED) ok = rp == (uint32_t)row * g.slots_row;
  if constexpr (MIXED) {
    const int n = lane_n(rp, rp_end);
    ok = n != 0;
    for (uint64_t wide = __ballot(have && n >= 3); wide; wide &= wide - 1) {
      // a row that keeps three or four, slot by slot: lane l takes its index words l, l + 64, ...
      const int k = __builtin_ctzll(wide);
      uint32_t start;
      const int nk = row_n(k, start);
      float sum = 0.f;
      const uint32_t words = ((uint32_t)nk * g.slots_row) >> 3;
      for (uint32_t wd = (uint32_t)lane; wd < words; wd += 64) {
        const uint32_t iw = *(const uint16_t *)(P.idx + (start >> 2) + 2 * wd), nb = *(const uint32_t *)(P.values + (start >> 1) + 4 * wd);
        for (uint32_t t = 0; t < 8; ++t) {
          const uint32_t c4 = nk == 4 ? (8 * wd + t) >> 2 : (8 * wd + t) / 3, col = 4 * c4 + ((iw >> (2 * t)) & 3u);
          const uint32_t grp = NQ == 2 ? col >> 5 : (col >> 6) >> g.gshift;
          const uint32_t pr = *(const uint32_t *)(P.qparams + 4 * ((size_t)(row0 + k) * (size_t)g.groups_per_row + grp));
          const float sc = __half2float(__ushort_as_half((uint16_t)(pr & 0xFFFFu))), zp = __half2float(__ushort_as_half((uint16_t)(pr >> 16)));
          const uint32_t Q = col >> 8;
          const __half xv = *(const __half *)(xs + 512 * Q + 16 * (((col >> 3) & 31u) ^ (Q & 15u)) + 2 * (col & 7u));
          sum = fmaf(sc * ((float)((nb >> (4 * t)) & 15u) - zp), __half2float(xv), sum);
        }
      }
      for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
      if (lane == k) v = sum;
    }
  }
  if (have) P.y[row] = ok ? __float2half(v) : __ushort_as_half((uint16_t)0x7E00);
}

template <int FORM, int QW, bool MP, bool ODD, bool PAIRED>
__global__ __launch_bounds__(512, 4) void k_rows(const uint32_t *__restrict__ row_ptr, const uint8_t *__restrict__ values,
                                                 const uint8_t *__restrict__ idx, const uint8_t *__restrict__ qparams,
                                                 const __half *__restrict__ x, __half *__restrict__ y, const RowsGeom g) {
  const RowsPtrs P{row_ptr, values, idx, qparams, x, y};
  rows_body<FORM, QW, MP, ODD, PAIRED>(P, g);
}
// up to four identically shaped matrices, blockIdx.y names the member
template <int FORM, int QW, bool MP>
__global__ __launch_bounds__(512, 4) void k_rows_batch(const GemvBatch b, const RowsGeom g) {
  const unsigned k = blockIdx.y;
  const RowsPtrs P{pick4(b.row_ptr, k), pick4(b.values, k), pick4(b.idx, k), pick4(b.qparams, k), pick4(b.x, k), pick4(b.y, k)};
  rows_body<FORM, QW, MP, false, false>(P, g);
}

namespace {

bool group_shift(int group, int unit, int &shift) {
  shift = 0;
  while ((unit << shift) < group) ++shift;
  return (unit << shift) == group;
}

// Everything but the pointers; `wide`: several {scale, zero} pairs (or scaling before the instruction).
bool rows_geometry(int form, int rows, int cols, int n_keep, int group, uint32_t total_slots, RowsGeom &g, int &qw) {
  if (rows < 1 || cols < 32 || cols % 32 != 0 || cols > 24576 || group % 32 != 0) return false;
  const bool dense = form == ROWS_DENSE, f16 = form >= ROWS_F24;
  if ((form == ROWS_14 || form == ROWS_MIXED) && cols % 64 != 0) return false;
  if (form == ROWS_24 && cols < 64) return false;     // (the half chunk of an odd row is fetched with the half before it)
  g.rows = rows;
  const int chunk = rows_chunk(form);
  g.nchunks = (cols + chunk - 1) / chunk;
  const int quads = (g.nchunks + 3) / 4;
  g.phases = (quads + 15) / 16;
  g.qpr = g.phases > 1 ? 16 : quads;
  g.qpr_inv = (65536 + g.qpr - 1) / g.qpr;
  g.rpt = (g.phases > 1 || form == ROWS_MIXED) ? 1 : 16 / g.qpr;
  g.nrg = (rows + g.rpt - 1) / g.rpt;
  g.groups_per_row = f16 ? 0 : cols / group;
  g.gshift = 0;
  qw = 1;
  if (f16) {
  } else if (dense) {
    qw = group < 128 ? 2 : 1;
    if (!group_shift(group, group < 128 ? 32 : 128, g.gshift)) return false;
  } else {
    qw = group == 32 ? 2 : 1;
    if (group != 32 && !group_shift(group, 64, g.gshift)) return false;
  }
  g.npieces = cols / 8;
  g.quads = 16 * g.phases > quads && g.phases > 1 ? 16 * g.phases : quads;
  const int n = n_keep ? n_keep : 1;
  g.val_row = dense ? (uint32_t)cols / 2 : f16 ? (uint32_t)(n * (cols / 2)) : (uint32_t)(n * (cols / 8));
  g.idx_row = (uint32_t)(n * (cols / 16));
  g.slots_row = (uint32_t)(n * (cols / 4));
  g.total_slots = total_slots;
  const uint64_t vb = form == ROWS_MIXED ? total_slots / 2 : (uint64_t)rows * g.val_row, qb = 4ull * (uint64_t)rows * (uint64_t)g.groups_per_row;
  if (vb >= 0x7FFF0000ull || qb >= 0x7FFF0000ull) return false;            // (see OUT)
  g.val_bytes = (uint32_t)vb; g.idx_bytes = dense ? 0u : form == ROWS_MIXED ? total_slots / 4 : (uint32_t)((uint64_t)rows * g.idx_row);
  g.qp_bytes = (uint32_t)qb;
  g.nib_mask = dense ? 0x00F000F0u : 0x00F0000Fu;
  g.nib_magic = dense ? 0x54005400u : 0x54006400u;
  g.nib_magic2 = 0;
  g.m8 = 0x00FF00FFu; g.m4 = 0x0F0F0F0Fu; g.m2 = 0x33333333u;
  return true;
}

// Waves and workgroups: as many waves as are resident at a time (by their registers: twenty per
// compute unit, sixteen where rows differ) if the rows allow it, more rows per wave beyond that -
// one wave more than are resident and the launch ends on a second, nearly empty round (20000 x
// 2816: 7.3 us with 5000 waves of two batches, 8.7 with 3334 of three; 11008 x 4096: 6.0 with
// 2752, 6.5 with 5504).
void rows_shape(RowsGeom &g, int form, dim3 &grid, dim3 &block, size_t &lds) {
  const int tpi = rows_tpi(form), nb = (g.nrg + tpi - 1) / tpi;   // batches of the matrix
  const size_t x_bytes = ((size_t)g.quads * (size_t)(8 * rows_chunk(form)) + 1023) & ~(size_t)1023;
  int waves = x_bytes <= 8192 ? 4 : 8, per_cu = (form == ROWS_24 || form == ROWS_14) ? 20 : form == ROWS_F24 ? 24 : 16;   // (a larger x is shared by more waves)
  tune_pair("EGT_ROWS_TUNE", waves, per_cu);
  waves = waves < 1 ? 1 : waves > 8 ? 8 : waves;
  per_cu = per_cu < 1 ? 1 : per_cu > 64 ? 64 : per_cu;
  g.batches = (nb + 256 * per_cu - 1) / (256 * per_cu);
  g.batches = std::max(1, std::min(g.batches, ROWS_PER_WAVE / (tpi * g.rpt)));
  auto red_bytes = [&] {
    g.red_stride = (g.batches * tpi * g.rpt) | 1;
    return (size_t)waves * (size_t)g.qpr * (size_t)g.red_stride * sizeof(float);
  };
  while (x_bytes + red_bytes() > 64 * 1024 && g.batches > 1) --g.batches;
  const int nwaves = (nb + g.batches - 1) / g.batches;
  grid = dim3((unsigned)((nwaves + waves - 1) / waves));
  block = dim3(64u * (unsigned)waves);
  lds = x_bytes + red_bytes();
}

}  // namespace

// 2:4 and 1:4 matrices, INT4 (either nibble order at 2:4) or FP16, and INT4 matrices whose rows differ; any row length
// up to 24576 columns (x fits LDS) that is a multiple of 32 - of 64 for INT4 at 1:4 and where rows differ; groups of 32 << j.
static int rows_form(const egt_2bitcsr &w) {
  if (w.val_kind == EGT_VAL_FP16) return w.n_keep == 2 ? ROWS_F24 : ROWS_F14;
  return w.n_keep == 2 ? ROWS_24 : w.n_keep == 1 ? ROWS_14 : ROWS_MIXED;
}
bool sparse_rows_supported(const egt_2bitcsr &w) {
  RowsGeom g;
  int qw;
  if ((w.n_keep != 1 && w.n_keep != 2 && w.n_keep != 0) || (w.n_keep == 0 && w.val_kind != EGT_VAL_INT4)) return false;
  if (w.val_kind == EGT_VAL_INT4_PAIRED && w.n_keep != 2) return false;
  return rows_geometry(rows_form(w), w.rows, w.cols, w.n_keep, w.group_size, w.total_slots, g, qw);
}
bool int4_rows_supported(int rows, int cols, int group) {
  RowsGeom g;
  int qw;
  return cols % group == 0 && rows_geometry(ROWS_DENSE, rows, cols, 0, group, 0, g, qw);
}

hipError_t launch_sparse_rows(const egt_2bitcsr *ws, const uint16_t *const *xv, uint16_t *const *yv, int count, hipStream_t stream) {
  const egt_2bitcsr &w = ws[0];
  if (w.rows == 0 || count == 0) return hipSuccess;
  const int form = rows_form(w);
  const bool paired = w.val_kind == EGT_VAL_INT4_PAIRED;
  RowsGeom g;
  int qw;
  if (!rows_geometry(form, w.rows, w.cols, w.n_keep, w.group_size, w.total_slots, g, qw)) return hipErrorInvalidValue;
  if (paired) { g.nib_mask = 0x000F000Fu; g.nib_magic = 0x64006400u; g.nib_magic2 = 0x54005400u; }
  dim3 grid, block;
  size_t lds;
  rows_shape(g, form, grid, block, lds);
  const bool odd = form == ROWS_24 && w.cols % 64 != 0, mp = g.phases > 1;
  if (count > 1 && !odd && !paired && (form == ROWS_24 || form == ROWS_14)) {
    GemvBatch b = {};
    for (int k = 0; k < count; ++k) {
      b.row_ptr[k] = ws[k].row_ptr; b.values[k] = (const uint8_t *)ws[k].values; b.idx[k] = (const uint8_t *)ws[k].idx;
      b.qparams[k] = (const uint8_t *)ws[k].qparams; b.x[k] = (const __half *)xv[k]; b.y[k] = (__half *)yv[k];
    }
    grid.y = (unsigned)count;
#define EGT_B(FORM) (qw == 2 ? (mp ? launch(k_rows_batch<FORM, 2, true>, grid, block, lds, stream, b, g) : launch(k_rows_batch<FORM, 2, false>, grid, block, lds, stream, b, g)) \
                             : (mp ? launch(k_rows_batch<FORM, 1, true>, grid, block, lds, stream, b, g) : launch(k_rows_batch<FORM, 1, false>, grid, block, lds, stream, b, g)))
    return form == ROWS_24 ? EGT_B(ROWS_24) : EGT_B(ROWS_14);
#undef EGT_B
  }
  for (int k = 0; k < count; ++k) {
    const egt_2bitcsr &m = ws[k];
    g.total_slots = m.total_slots;
    hipError_t e;
#define EGT_R(FORM, QW, MP, ODD, PAIRED)                                                                                       \
  launch(k_rows<FORM, QW, MP, ODD, PAIRED>, grid, block, lds, stream, m.row_ptr, (const uint8_t *)m.values, (const uint8_t *)m.idx, \
         (const uint8_t *)m.qparams, (const __half *)xv[k], (__half *)yv[k], g)
#define EGT_RM(FORM, QW, ODD, PAIRED) (mp ? EGT_R(FORM, QW, true, ODD, PAIRED) : EGT_R(FORM, QW, false, ODD, PAIRED))
#define EGT_RQ(FORM) (qw == 2 ? EGT_RM(FORM, 2, false, false) : EGT_RM(FORM, 1, false, false))
    if (form == ROWS_F24) e = EGT_RM(ROWS_F24, 1, false, false);
    else if (form == ROWS_F14) e = EGT_RM(ROWS_F14, 1, false, false);
    else if (form == ROWS_14) e = EGT_RQ(ROWS_14);
    else if (form == ROWS_MIXED) e = EGT_RQ(ROWS_MIXED);
    else if (odd) e = paired ? EGT_RM(ROWS_24, 2, true, true) : EGT_RM(ROWS_24, 2, true, false);   // (an odd number of 32 columns: groups of 32)
    else if (paired) e = qw == 2 ? EGT_RM(ROWS_24, 2, false, true) : EGT_RM(ROWS_24, 1, false, true);
    else e = EGT_RQ(ROWS_24);
#undef EGT_RQ
#undef EGT_RM
#undef EGT_R
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_int4_rows(const uint8_t *const *qs, const uint16_t *const *qps, int rows, int cols, int group, const uint16_t *const *xv,
                            uint16_t *const *yv, int count, hipStream_t stream) {
  if (rows == 0 || count == 0) return hipSuccess;
  RowsGeom g;
  int qw;
  if (!rows_geometry(ROWS_DENSE, rows, cols, 0, group, 0, g, qw)) return hipErrorInvalidValue;
  dim3 grid, block;
  size_t lds;
  rows_shape(g, ROWS_DENSE, grid, block, lds);
  const bool mp = g.phases > 1;
  if (count > 1) {
    GemvBatch b = {};
    for (int k = 0; k < count; ++k) {
      b.values[k] = qs[k]; b.qparams[k] = (const uint8_t *)qps[k]; b.x[k] = (const __half *)xv[k]; b.y[k] = (__half *)yv[k];
    }
    grid.y = (unsigned)count;
    return qw == 2 ? (mp ? launch(k_rows_batch<ROWS_DENSE, 2, true>, grid, block, lds, stream, b, g) : launch(k_rows_batch<ROWS_DENSE, 2, false>, grid, block, lds, stream, b, g))
                   : (mp ? launch(k_rows_batch<ROWS_DENSE, 1, true>, grid, block, lds, stream, b, g) : launch(k_rows_batch<ROWS_DENSE, 1, false>, grid, block, lds, stream, b, g));
  }
#define EGT_D(QW, MP)                                                                                                              \
  launch(k_rows<ROWS_DENSE, QW, MP, false, false>, grid, block, lds, stream, nullptr, qs[0], nullptr, (const uint8_t *)qps[0], \
         (const __half *)xv[0], (__half *)yv[0], g)
  return qw == 2 ? (mp ? EGT_D(2, true) : EGT_D(2, false)) : (mp ? EGT_D(1, true) : EGT_D(1, false));
#undef EGT_D
}

}  // namespace egt
