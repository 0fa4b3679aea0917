// M = 1 products of 2:4 matrices with FP16 values and short rows on the sparse matrix cores.
//
// The row-per-wave kernel (egt_mfma_m1.hip) wants FP16 rows of 4096 columns and more in whole 64s.
// Shorter ones used to be followed slot by slot, or, at 1024 and 2048 columns, by a form of that
// kernel with several rows to a tile.  Here a tile is 16 quads of four chunks (a chunk: 16 bytes of
// values, 16 columns), and a row takes ceil(chunks / 4) quads: `rpt` whole rows lie in a tile, or a
// row lies in `phases` tiles.  Between a half and all of the lanes carry weights then; the rest ask
// out of range of the buffers (zeros, no traffic).
//
// The mapping is the diagonal one: lane (i, kb) = i + 16 kb takes chunk kb of quad i, column n
// of B carries the activations of quad n, and D[i][i] is quad i's share of its row.  The 16
// diagonals of a tile are left in LDS; at the end of a wave one lane per row adds those of its
// quads (added tile by tile they were a chain of LDS latencies that 4 waves per SIMD did not hide).
// Only kept columns are multiplied and the products are summed in FP32, as slot by slot: the two
// differ in the order of the additions (20000 x 2816: error against 64 bits 2.0777e-4 either way,
// all of it the rounding of y).
//
// Only FP16 values at 2:4 (INT4 rows: egt_mfma_codes.hip): a row of FP16 values that keeps one of four would
// multiply a second column of its 4-groups by zero, which an infinity there turns into NaN.
//
//  - A wave owns up to 64 consecutive rows and walks them TPI tiles at a time with two sets of
//    registers.
//  - x goes from global memory straight into LDS (no registers, requested before the first
//    weights).  Piece s (16 bytes) of quad Q lies in slot s ^ (Q & 7) of its quad, so the
//    sixteen lanes of a B read, one quad each, fall into different banks.
//
// Measured, us per launch before and now (weights in the last-level cache): 20000 x 2816 13.5,
// 11.6; 5003 x 2880 5.6, 4.3; 2000 x 2048 5.0, 3.1; 4096 x 1024 5.8, 2.9; 60000 x 512 13.3, 5.9.
// What bounds it: the launch for a few megabytes, the memory beyond (20000 x 2816: 64 MB at 5.5 TB/s, the
// vector units 8 % busy).
#include "egt_mfma_common.h"

#include "egt_tune.h"

#include <algorithm>

namespace egt {

constexpr int ROWS_CHUNK = 16;                        // columns of a chunk: eight values, one index word
constexpr int ROWS_TPI = 4;                           // tiles in work at a time (a tile is a kilobyte and one instruction)
constexpr int ROWS_PER_WAVE = 64;                     // rows a wave owns at most (a row pointer per lane)
constexpr int ROWS_QUAD = 8 * ROWS_CHUNK;             // bytes of a quad of x

struct RowsGeom {
  int rows;
  int nchunks;         // chunks of a row
  int qpr, qpr_inv;    // quads of a row inside a tile; ceil(65536 / qpr)
  int rpt;             // rows of a tile (1 where a row takes several)
  int phases;          // tiles of a row
  int nrg;             // row groups: ceil(rows / rpt)
  int batches;         // batches of TPI row groups a wave walks
  int red_stride;      // floats from one quad's sums to the next's: the rows of a wave, odd
  int npieces;         // 16-byte pieces of x
  int quads;           // quads of x in LDS
  uint32_t val_row, idx_row, slots_row;               // bytes and slots of a row
  uint32_t val_bytes, idx_bytes;                      // extents of the arrays
};
struct RowsPtrs {
  const uint32_t *row_ptr;
  const uint8_t *values, *idx;
  const __half *x;
  __half *y;
};

struct RowsTile {
  u4 val;
  uint32_t iw;
};

// MP: a row takes several tiles.
template <bool MP>
__device__ __forceinline__ void rows_body(const RowsPtrs &P, const RowsGeom &g) {
  extern __shared__ __align__(16) uint8_t xs[];       // x, then the quads' sums of every wave
  constexpr int TPI = ROWS_TPI, LOADS = 2;            // (requests of a tile)
  // past every buffer (they are below 2 GiB), also with a uniform offset added: zeros, no traffic
  constexpr uint32_t OUT = 0x7FFFFFF0u;
  constexpr int QP = ROWS_QUAD / 16, QM = QP - 1;     // pieces of a quad, and the bits of Q that move them
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  const int i = lane & 15, kb = lane >> 4;
  const __amdgpu_buffer_rsrc_t r_val = make_rsrc(P.values, g.val_bytes), r_idx = make_rsrc(P.idx, g.idx_bytes);
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc(P.x, 16u * (uint32_t)g.npieces);

  // ---- this wave's rows: row groups [rg0, rg0 + batches * TPI)
  const int rg0 = ((int)blockIdx.x * nw + wave) * g.batches * TPI;
  const int rg_end = rg0 + g.batches * TPI;
  const int row0 = rg0 * g.rpt;
  uint32_t rp = 0;                                    // lane j: the row pointer of row row0 + j
  if (row0 + lane < g.rows) rp = P.row_ptr[row0 + lane];

  // ---- x: one request per kilobyte; lane l delivers to byte 16 l
  const int kib = (g.quads * ROWS_QUAD + 1023) >> 10;
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
  const uint32_t v_lane = (uint32_t)rs * g.val_row + 16u * (uint32_t)cl, i_lane = (uint32_t)rs * g.idx_row + 2u * (uint32_t)cl;

  auto load = [&](RowsTile (&t)[TPI], int rg, int p) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const int left = rg + k < rg_end ? g.rows - (rg + k) * g.rpt : 0;      // uniform; rows from this group on
      const bool on = lane_on && rs < left && cl < g.nchunks - (MP ? 64 * p : 0);
      const uint32_t r = (uint32_t)((rg + k) * g.rpt);
      t[k].val = __builtin_amdgcn_raw_buffer_load_b128(r_val, on ? v_lane : OUT, left > 0 ? r * g.val_row + 1024u * (uint32_t)p : 0u, 0);
      t[k].iw = __builtin_amdgcn_raw_buffer_load_b16(r_idx, on ? i_lane : OUT, left > 0 ? r * g.idx_row + 128u * (uint32_t)p : 0u, 0);
    }
  };

  // ---- B operand of a phase: lane (n, b) supplies the k-octets b and 4 + b, pieces b and 4 + b of quad n
  const uint32_t b0 = (uint32_t)(ROWS_QUAD * qi + 16 * (kb ^ (qi & QM)));
  u8v bx;
  auto read_b = [&](int p) {
    const uint8_t *at = xs + (MP ? 16 * ROWS_QUAD * p : 0);
    const u4 lo = *(const u4 *)(at + b0), hi = *(const u4 *)(at + (b0 ^ 64u));
    bx = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  };

  float *red = (float *)(xs + (size_t)kib * 1024) + wave * (g.qpr * g.red_stride);   // [quad of a row][row of this wave]
  // The first two items of the walk are requested; then x of this wave's requests is waited for (requests
  // return in order, and LOADS of them fetch a tile, on or off).
  const int mine = min(g.batches, (g.nrg - rg0 + TPI - 1) / TPI);
  const int total = MP ? mine * g.phases : mine;
  RowsTile ta[TPI], tb[TPI];
  load(ta, rg0, 0);
  load(tb, MP ? rg0 : rg0 + TPI, MP ? 1 : 0);
  wait_vmem<2 * TPI * LOADS>();
  for (int pc = g.npieces + (int)threadIdx.x; pc < (kib << 10) / 16; pc += (int)blockDim.x) {   // pieces past the end of x
    const int Q = pc / QP, s = pc % QP;
    *(u4 *)(xs + ROWS_QUAD * Q + 16 * (s ^ (Q & QM))) = u4{0, 0, 0, 0};
  }
  lds_barrier();
  if (row0 >= g.rows) return;                         // (no barrier follows)
  if (!MP) read_b(0);

  f4 acc[TPI];
#pragma unroll
  for (int k = 0; k < TPI; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};

  auto consume = [&](const RowsTile (&t)[TPI], int p) {
    if (MP) read_b(p);
#pragma unroll
    for (int k = 0; k < TPI; ++k)
      acc[k] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, t[k].val), __builtin_bit_cast(h16, bx), acc[k], (int)t[k].iw, 0, 0);
  };

  // ---- diagonal i of tile k sits in lane i + 16 (i / 4), register i % 4: quad qi of row rs of its row group
  auto leave = [&](int rg) {
#pragma unroll
    for (int k = 0; k < TPI; ++k) {
      const float d = select4(lane & 3, acc[k][0], acc[k][1], acc[k][2], acc[k][3]);
      if (kb == (i >> 2) && lane_on) red[qi * g.red_stride + (rg + k - rg0) * g.rpt + rs] = d;
      acc[k] = f4{0.f, 0.f, 0.f, 0.f};
    }
  };

  // ---- (batch, phase) one after the other; an item's registers are requested again, for the item after
  // the next, as soon as it has been used (under a condition, behind which the compiler waits for both sets)
  int rg = rg0, p = 0;
  auto advance = [&](int &r, int &q) {
    if (!MP || ++q == g.phases) { q = 0; r += TPI; }
  };
  auto step = [&](RowsTile (&cur)[TPI], int it) {
    consume(cur, p);
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
  if (lane < g.batches * TPI * g.rpt && row < g.rows) {
    float v = 0.f;
    const float *q = red + lane;
#pragma unroll 4
    for (int k = 0; k < g.qpr; ++k) v += q[k * g.red_stride];
    P.y[row] = rp == (uint32_t)row * g.slots_row ? __float2half(v) : __ushort_as_half((uint16_t)0x7E00);
  }
}

template <bool MP>
__global__ __launch_bounds__(512, 4) void k_rows(const uint32_t *__restrict__ row_ptr, const uint8_t *__restrict__ values,
                                                 const uint8_t *__restrict__ idx, const __half *__restrict__ x, __half *__restrict__ y,
                                                 const RowsGeom g) {
  const RowsPtrs P{row_ptr, values, idx, x, y};
  rows_body<MP>(P, g);
}
// Up to four identically shaped matrices, blockIdx.y names the member (1734 x 1024, three of them: 3.5 us; the
// row-per-wave kernel's batch took 5.7).
template <bool MP>
__global__ __launch_bounds__(512, 4) void k_rows_batch(const GemvBatch b, const RowsGeom g) {
  const unsigned k = blockIdx.y;
  const RowsPtrs P{pick4(b.row_ptr, k), pick4(b.values, k), pick4(b.idx, k), pick4(b.x, k), pick4(b.y, k)};
  rows_body<MP>(P, g);
}

// Everything but the pointers.
static bool rows_geometry(const egt_2bitcsr &w, RowsGeom &g) {
  if (w.n_keep != 2 || w.val_kind != EGT_VAL_FP16 || w.rows < 1 || w.cols < 32 || w.cols % 32 != 0 || w.cols >= 4096) return false;
  g.rows = w.rows;
  g.nchunks = w.cols / ROWS_CHUNK;
  const int quads = (g.nchunks + 3) / 4;
  g.phases = (quads + 15) / 16;
  g.qpr = g.phases > 1 ? 16 : quads;
  g.qpr_inv = (65536 + g.qpr - 1) / g.qpr;
  g.rpt = g.phases > 1 ? 1 : 16 / g.qpr;
  g.nrg = (w.rows + g.rpt - 1) / g.rpt;
  g.npieces = w.cols / 8;
  g.quads = g.phases > 1 ? 16 * g.phases : quads;
  g.val_row = (uint32_t)w.cols;
  g.idx_row = (uint32_t)(w.cols / 8);
  g.slots_row = (uint32_t)(w.cols / 2);
  const uint64_t vb = (uint64_t)w.rows * g.val_row;
  if (vb >= 0x7FFF0000ull) return false;              // (see OUT)
  g.val_bytes = (uint32_t)vb;
  g.idx_bytes = (uint32_t)(vb / 8);
  return true;
}

// Waves and workgroups: as many waves as are resident at a time (by their registers twenty-four per
// compute unit) if the rows allow it, more rows per wave beyond that - one wave more than are
// resident and the launch ends on a second, nearly empty round.
static void rows_shape(RowsGeom &g, dim3 &grid, dim3 &block, size_t &lds) {
  const int nb = (g.nrg + ROWS_TPI - 1) / ROWS_TPI;   // batches of the matrix
  const size_t x_bytes = ((size_t)g.quads * ROWS_QUAD + 1023) & ~(size_t)1023;
  int waves = 4, per_cu = 24;
  tune_pair("EGT_ROWS_TUNE", waves, per_cu);
  waves = waves < 1 ? 1 : waves > 8 ? 8 : waves;
  per_cu = per_cu < 1 ? 1 : per_cu > 64 ? 64 : per_cu;
  g.batches = (nb + 256 * per_cu - 1) / (256 * per_cu);
  g.batches = std::max(1, std::min(g.batches, ROWS_PER_WAVE / (ROWS_TPI * g.rpt)));
  g.red_stride = (g.batches * ROWS_TPI * g.rpt) | 1;
  const int nwaves = (nb + g.batches - 1) / g.batches;
  grid = dim3((unsigned)((nwaves + waves - 1) / waves));
  block = dim3(64u * (unsigned)waves);
  lds = x_bytes + (size_t)waves * (size_t)g.qpr * (size_t)g.red_stride * sizeof(float);   // (at most 8 KB and 17 KB)
}

// 2:4, FP16 values, rows of fewer than 4096 columns in whole index words (and values below 2 GiB: 32-bit offsets).  Longer ones are a chain of
// five and more tiles a row in one wave: below the line 0.76 to 0.95 times the time of the slot-by-slot kernel
// (64 ... 32000 rows x 3104 ... 4064), above it few rows lose 1.15 to 1.4 times (256 x 4128 4.6 -> 5.5 us, 256 x 16416
// 9.8 -> 13.4) and many gain a tenth at most.
bool sparse_rows_supported(const egt_2bitcsr &w) {
  RowsGeom g;
  return rows_geometry(w, g);
}

hipError_t launch_sparse_rows_batch(const egt_2bitcsr *ws, const uint16_t *const *xs, uint16_t *const *ys, int count, hipStream_t stream) {
  const egt_2bitcsr &w = ws[0];
  RowsGeom g;
  if (!rows_geometry(w, g)) return hipErrorInvalidValue;
  dim3 grid, block;
  size_t lds;
  rows_shape(g, grid, block, lds);
  if (count == 1) {
#define EGT_R(MP) launch(k_rows<MP>, grid, block, lds, stream, w.row_ptr, (const uint8_t *)w.values, (const uint8_t *)w.idx, (const __half *)xs[0], (__half *)ys[0], g)
    return g.phases > 1 ? EGT_R(true) : EGT_R(false);
#undef EGT_R
  }
  GemvBatch b = {};
  for (int k = 0; k < count; ++k) {
    b.row_ptr[k] = ws[k].row_ptr; b.values[k] = (const uint8_t *)ws[k].values; b.idx[k] = (const uint8_t *)ws[k].idx;
    b.x[k] = (const __half *)xs[k]; b.y[k] = (__half *)ys[k];
  }
  grid.y = (unsigned)count;
  return g.phases > 1 ? launch(k_rows_batch<true>, grid, block, lds, stream, b, g) : launch(k_rows_batch<false>, grid, block, lds, stream, b, g);
}
hipError_t launch_sparse_rows(const egt_2bitcsr &w, const uint16_t *x, uint16_t *y, hipStream_t stream) {
  return launch_sparse_rows_batch(&w, &x, &y, 1, stream);
}

}  // namespace egt
