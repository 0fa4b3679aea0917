// Small-M products with the activations held in registers: INT4, 2 to 32 tokens, rows of at
// most as many K-steps as a workgroup of the kernel in egt_mfma_smallm.hip has waves (2:4: 4096
// columns, above 16 tokens 2048; 1:4: 4096, up to 16 tokens).
//
// In the kernel of egt_mfma_smallm.hip a wave owns a K-step of up to three or four row tiles;
// where a workgroup has more of them it starts anew - X from the L2 into LDS, B operands out of
// LDS, tiles requested, waited for, summed over the waves - for every round.  When the waves
// cover all of K in one go, a wave's B operand is the same for every row tile, so here it is read
// once and stays in registers (32 per token group at 2:4, 64 at 1:4), the LDS that X came
// through becomes room for the waves' sums, and the row tiles of a workgroup - all of them, of
// several matrices if these run under one X - are a stream: RING tiles of a wave are on their
// way, a tile's registers are requested again as soon as its products are out, and the
// sums of one set of tiles are added up and stored while the next set is multiplied.
//
// What bounds it: the start (a launch, X and the first tiles from memory, 3 to 4 us) for a few
// tiles per workgroup, instructions and the memory beyond (65536 x 4096 at 5 tokens: 22.0 us, 5.1 TB/s).
// A wave adds up a whole tile of a set, four rows of a token a lane; an output per lane took four times the
// reads, compares and selects: 65536 x 4096 at 5 tokens 23.7, 22.0; 11008 x 4096 at 16 7.06, 6.70; 20000 x 1024
// at 8 5.5, 5.1; 11008 x 2048 at 32 7.1, 6.6 (with one address per lane for all tiles; 1:4 alike or up to 8 % less).
// Before and now, in microseconds: 4096 x 4096 at 5 tokens 5.0, 3.9; 22016 x 4096 at 16 tokens 14.2,
// 11.8; 65536 x 4096 39.5, 26.4; 20000 x 1024 at 8 tokens 8.6, 5.2; two 1:4 matrices of 11008 x
// 4096 under one X 13.7, 11.8.
//
// Rows of at most half as many K-steps as there are waves: `streams` groups of waves share the
// K-steps and take the tiles in turn.
//
// The sum of a row: each K-step's products by the matrix instructions, then the K-steps in
// ascending order.  The other kernel adds the K-steps of a wave first; with a wave for every
// K-step the two give the same bits, so that a product may take either, alone or in a batch.
#include "egt_mfma_common.h"

#include "egt_tune.h"

#include <algorithm>

namespace egt {

struct SmallMHoldGeom {
  int rows, M;
  int nchunks;         // cols / 64 (2:4) or cols / 128 (1:4)
  int nsteps;          // ceil(nchunks / 4)
  int kpieces;         // cols / 8
  int gshift, groups_per_row;
  int vec_store;
  uint32_t val_bytes, idx_bytes, qp_bytes, x_bytes;
  int64_t ldx, ldy;
  uint32_t nib_mask, nib_magic, m4, m2;
  int nw;              // waves: streams * nsteps
  int streams, stream_shift, step_inv;      // wave = stream * nsteps + step; ceil(65536 / nsteps)
  int sets, sets_more; // sets of a workgroup of tiles_q and of one of tiles_q + 1 row tiles
  int wave_stride, slot_stride;   // LDS bytes from a wave's sums to the next wave's, from one of its slots to the next
  int flags_at;        // LDS offset of the row flags
  int blocks, tiles_q, tiles_r;   // workgroup b owns tiles_q + (b < tiles_r) row tiles: b, b + blocks, ...
  int mtiles;          // row tiles of one member (several matrices under one X), or of the matrix
};

constexpr int HOLD_PAIR = 1024 + 32;                  // 2:4: LDS bytes of a pair of tokens of a K-step (512 B each)
constexpr int HOLD_TOKEN_N1 = 1024 + 16;              // 1:4: of a token (1 KiB)

template <int QW>
struct HoldTile {
  u4 nib;
  u2 iw;
  uint32_t qp[QW];
};

// QW: {scale, zero} pairs per chunk.  N1: 1:4.  NG: token groups of 16.  RING: row tiles of a wave on
// their way and of a set.  ONE: one stream; X of a K-step is then its wave's own business, the wave's sums
// go over it, and no barrier stands before the first of them.
template <int QW, bool N1, int NG, int RING, bool ONE, bool JOINT>
__device__ __forceinline__ void smallm_hold_body(const SmallMBatch &b, const SmallMHoldGeom &g) {
  extern __shared__ __align__(16) uint8_t xs[];       // X, then the waves' sums; flags behind
  constexpr int NM = N1 ? 8 : 4;                      // matrix instructions per step
  constexpr int PIECES = N1 ? 64 : 32;                // 16-byte pieces of a token row in a step
  constexpr int REQ = N1 ? 16 : 8;                    // requests of X per step and token group
  constexpr int REGION = N1 ? 16 * HOLD_TOKEN_N1 : 8 * HOLD_PAIR;
  constexpr uint32_t OUT = 0x7FFFFFF0u;               // past every buffer (all below 2 GiB), also with a uniform offset added
  typedef HoldTile<QW> Tile;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = g.nw, S = ONE ? 1 : g.streams;
  const int stream = ONE ? 0 : (wave * g.step_inv) >> 16, step = wave - stream * g.nsteps;
  const int i = lane & 15, kb = lane >> 4;
  const int li = lane >> 2, lc = lane & 3;            // row, chunk this lane fetches
  const int from = 4 * (4 * i + kb);                  // lane that fetched the chunk of lane (i, kb), as a byte address
  const int mytiles = g.tiles_q + ((int)blockIdx.x < g.tiles_r ? 1 : 0);
  const int nsets = (int)blockIdx.x < g.tiles_r ? g.sets_more : g.sets;
  const uint32_t S_row = (uint32_t)g.nchunks * 32u;
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc(b.X[0], g.x_bytes);

  // ---- row tile k of this workgroup: tile blockIdx.x + k * blocks of the launch
  auto member = [&](int &v) {
    if constexpr (!JOINT) return 0;
    const int k = (v >= g.mtiles) + (v >= 2 * g.mtiles) + (v >= 3 * g.mtiles);
    v -= k * g.mtiles;
    return k;
  };
  // row pointers of a set are requested a set ahead by the threads that check them
  auto flag_row = [&](int set, int &k) {
    const int t = set * RING * S + (int)(threadIdx.x >> 4);
    int v = (int)blockIdx.x + t * g.blocks;
    k = member(v);
    return t < mytiles ? 16 * v + (int)(threadIdx.x & 15) : g.rows;
  };
  auto load_rp = [&](int set) -> uint32_t {
    int k;
    const int r = flag_row(set, k);
    if ((int)threadIdx.x >= 16 * RING * S || r >= g.rows) return 0u;
    return (JOINT ? pick4(b.row_ptr, (unsigned)k) : b.row_ptr[0])[r];
  };
  uint32_t rp = load_rp(0);                            // (first of all: the furthest away, where nothing is cached)

  // ---- X: the waves of all streams share the requests of their K-step
  const int xtl = lane >> 5;
  const int slot_piece = N1 ? lane : ((lane & 31) ^ xtl);
  const int vp = min(PIECES, g.kpieces - PIECES * step);     // pieces of the step inside K
  {
    const uint32_t off_lo = 16u * (uint32_t)min(slot_piece, vp - 1);
    const uint32_t off_hi = off_lo + (uint32_t)xtl * (uint32_t)(2 * g.ldx);
    asm volatile("" ::: "memory");
    for (int q = stream; q < NG * REQ; q += S) {
      const int t0 = N1 ? q : 2 * q;                  // first token of the request
      if (t0 < g.M)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(xs + (step * NG * REQ + q) * (REGION / REQ)), 16,
                                                 (N1 || t0 + 1 >= g.M) ? off_lo : off_hi,
                                                 (uint32_t)(16 * PIECES) * (uint32_t)step + (uint32_t)t0 * (uint32_t)(2 * g.ldx), 0, 0);
    }
    asm volatile("" ::: "memory");
  }

  const bool chunk_on = 4 * step + lc < g.nchunks;
  const uint32_t c_lane = (uint32_t)li * (uint32_t)g.nchunks + (uint32_t)(4 * step + lc);
  const uint32_t q_lane = (uint32_t)li * (uint32_t)g.groups_per_row +
                          (QW > 1 ? (uint32_t)QW * (uint32_t)(4 * step + lc) : (uint32_t)((4 * step + lc) >> g.gshift));
  const uint32_t at_val = chunk_on ? 16u * c_lane : OUT, at_idx = chunk_on ? 8u * c_lane : OUT, at_qp = chunk_on ? 4u * q_lane : OUT;
  // A tile's buffers begin at its first row and end with the matrix, so that rows past the last one lie past the
  // buffer: one address per lane for all tiles.  (With a test per lane and request the compiler made two requests
  // under opposite masks of each.)
  auto load = [&](Tile &t, int k) {
    const bool have = k < mytiles;                    // uniform
    int v = have ? (int)blockIdx.x + k * g.blocks : 0;
    if constexpr (JOINT) asm volatile("" : "+s"(v));  // (the member's resources are worked out per request: kept, they would spill)
    const unsigned m = (unsigned)member(v);
    const uint32_t cu = (uint32_t)(16 * v) * (uint32_t)g.nchunks, qu = 4u * (uint32_t)(16 * v) * (uint32_t)g.groups_per_row;
    const __amdgpu_buffer_rsrc_t r_val = make_rsrc((JOINT ? pick4(b.values, m) : b.values[0]) + 16u * cu, have ? g.val_bytes - 16u * cu : 0u);
    const __amdgpu_buffer_rsrc_t r_idx = make_rsrc((JOINT ? pick4(b.idx, m) : b.idx[0]) + 8u * cu, have ? g.idx_bytes - 8u * cu : 0u);
    const __amdgpu_buffer_rsrc_t r_qp = make_rsrc((JOINT ? pick4(b.qparams, m) : b.qparams[0]) + qu, have ? g.qp_bytes - qu : 0u);
    t.iw = __builtin_amdgcn_raw_buffer_load_b64(r_idx, at_idx, 0, 0);
    t.nib = __builtin_amdgcn_raw_buffer_load_b128(r_val, at_val, 0, 0);
    if constexpr (QW == 4) {
      const u4 q = __builtin_amdgcn_raw_buffer_load_b128(r_qp, at_qp, 0, 0);
#pragma unroll
      for (int j = 0; j < QW; ++j) t.qp[j] = q[j];
    } else if constexpr (QW == 2) {
      const u2 q = __builtin_amdgcn_raw_buffer_load_b64(r_qp, at_qp, 0, 0);
#pragma unroll
      for (int j = 0; j < QW; ++j) t.qp[j] = q[j];
    } else {
      t.qp[0] = __builtin_amdgcn_raw_buffer_load_b32(r_qp, at_qp, 0, 0);
    }
  };
  Tile ring[RING];
#pragma unroll
  for (int u = 0; u < RING; ++u) load(ring[u], u * S + stream);
  wait_vmem<3 * RING>();                         // requests return in order: this wave's part of X has landed
  if (vp < PIECES && slot_piece >= vp) {              // the pieces of the last step that lie past K become zeros
    for (int q = stream; q < NG * REQ; q += S) *(u4 *)(xs + (step * NG * REQ + q) * (REGION / REQ) + 16 * lane) = u4{0, 0, 0, 0};
  }
  if (ONE) wait_lds(); else lds_barrier();
  u8v bx[NG][NM];
#pragma unroll
  for (int grp = 0; grp < NG; ++grp) {
    const uint8_t *region = xs + (step * NG + grp) * REGION;
    const int n = lane & 15, o = lane >> 4;
    const uint8_t *base0 = N1 ? region + HOLD_TOKEN_N1 * n + 16 * (16 * (o >> 1) + (o & 1))
                              : region + HOLD_PAIR * (n >> 1) + 512 * (n & 1) + 16 * (8 * (o >> 1) + ((o ^ n) & 1));
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const u4 lo = *(const u4 *)(base0 + 32 * m), hi = *(const u4 *)(base0 + (N1 ? 512 : 256) + 32 * m);
      bx[grp][m] = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
  }
  if (!ONE) lds_barrier();                            // the LDS of X is free

  const uint32_t magic = in_vgpr(g.nib_magic);
  // sums of a wave: a kilobyte for every (set parity, tile of the set, token group)
  uint8_t *mine = xs + wave * g.wave_stride;
  uint32_t *flags = (uint32_t *)(xs + g.flags_at);

  auto do_set = [&](int set, auto last_set) {
    constexpr bool LAST = decltype(last_set)::v != 0;
    const int slot0 = (set & 1) * RING * NG;
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      Tile &t = ring[u];
      const int k = (set * RING + u) * S + stream;
      u4 nib;
#pragma unroll
      for (int d = 0; d < 4; ++d) nib[d] = lane_perm(from, t.nib[d]);
      const uint32_t iw0 = lane_perm(from, t.iw[0]), iw1 = lane_perm(from, t.iw[1]);
      uint32_t qp[QW];
#pragma unroll
      for (int q = 0; q < QW; ++q) qp[q] = lane_perm(from, t.qp[q]);
      if constexpr (!LAST) load(t, k + RING * S);     // (whether or not there is such a tile: the waits stay exact)
      if (k < mytiles) {                              // uniform
        uint32_t s2[QW], off[QW];
#pragma unroll
        for (int q = 0; q < QW; ++q) {
          s2[q] = __builtin_amdgcn_perm(qp[q], qp[q], 0x01000100u);
          off[q] = pk_add_f16(__builtin_amdgcn_perm(qp[q], qp[q], 0x03020302u), g.nib_magic);
        }
        f4 acc[NG];
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) acc[grp] = f4{0.f, 0.f, 0.f, 0.f};
        uint32_t sp[4];
        if constexpr (N1) {
          sp[0] = spread_idx<0>(iw0, g.m4, g.m2); sp[1] = spread_idx<1>(iw0, g.m4, g.m2);
          sp[2] = spread_idx<0>(iw1, g.m4, g.m2); sp[3] = spread_idx<1>(iw1, g.m4, g.m2);
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          u4 av;
          int iword;
          if constexpr (N1) {
            const uint32_t d = nib[m >> 1], of = off[m * QW / 8], sc = s2[m * QW / 8];
            av = m & 1 ? dequant4_14<1>(d, of, sc, g.nib_mask, magic) : dequant4_14<0>(d, of, sc, g.nib_mask, magic);
            iword = (int)sp[m >> 1];
          } else {
            av = dequant8(nib[m], off[m * QW / 4], s2[m * QW / 4], g.nib_mask, magic);
            iword = (int)(m < 2 ? iw0 : iw1);
          }
#pragma unroll
          for (int grp = 0; grp < NG; ++grp) {
            if (m & 1)
              acc[grp] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, av), __builtin_bit_cast(h16, bx[grp][m]), acc[grp], iword, 0, 1);
            else
              acc[grp] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, av), __builtin_bit_cast(h16, bx[grp][m]), acc[grp], iword, 0, 0);
          }
        }
#pragma unroll
        for (int grp = 0; grp < NG; ++grp)
          *(f4 *)(mine + (slot0 + u * NG + grp) * g.slot_stride + 16 * lane) = acc[grp];
      }
    }
    if (64 * wave < 16 * RING * S) {                  // uniform
      int k;
      const int r = flag_row(set, k);
      if ((int)threadIdx.x < 16 * RING * S) flags[(set & 1) * 16 * RING * S + (int)threadIdx.x] = (r < g.rows && rp == (uint32_t)r * S_row) ? 1u : 0u;
      if constexpr (!LAST) rp = load_rp(set + 1);
    }
    lds_barrier();
    // ---- outputs of the set: a wave takes a tile's kilobyte, four rows of a token a lane: float 4 l + v of it is
    // D[row 4 (l >> 4) + v][token l & 15].  The waves take turns from set to set.
    int first = wave - (set * RING * S * NG) % nw;
    first += first < 0 ? nw : 0;
    for (int tg = first; tg < RING * S * NG; tg += nw) {
      const int ts = tg / NG, grp = tg % NG;          // tile of the set, token group
      const int t = set * RING * S + ts;
      if (t >= mytiles) break;                        // (later tg are later tiles)
      const int u = ONE ? ts : ts >> g.stream_shift, str = ONE ? 0 : ts & (S - 1);
      const uint8_t *src = xs + str * g.nsteps * g.wave_stride + (slot0 + u * NG + grp) * g.slot_stride + 16 * lane;
      const u4 ok = *(const u4 *)(flags + (set & 1) * 16 * RING * S + 16 * ts + 4 * (lane >> 4));
      // (several requested before the first is added, fewer where B, still needed, leaves few registers; in ascending order of the K-steps)
      constexpr int PARTS = LAST ? 8 : N1 ? 2 : NG > 1 ? 4 : 8;
      f4 sum = f4{0.f, 0.f, 0.f, 0.f};
      int st = 0;
      for (; st + PARTS <= g.nsteps; st += PARTS) {
        f4 part[PARTS];
#pragma unroll
        for (int q = 0; q < PARTS; ++q) part[q] = *(const f4 *)(src + (st + q) * g.wave_stride);
#pragma unroll
        for (int q = 0; q < PARTS; ++q) sum += part[q];
      }
      for (; st < g.nsteps; ++st) sum += *(const f4 *)(src + st * g.wave_stride);
      int v = (int)blockIdx.x + t * g.blocks;
      const int k = member(v);
      const int row0 = 16 * v + 4 * (lane >> 4), tok = 16 * grp + (lane & 15);
      uint32_t hv[4];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) hv[rr] = ok[rr] ? __half_as_ushort(__float2half(sum[rr])) : 0x7E00u;
      if (tok < g.M) {
        __half *dst = (JOINT ? pick4(b.Y, (unsigned)k) : b.Y[0]) + (int64_t)tok * g.ldy + row0;
        if (g.vec_store && row0 + 3 < g.rows) {
          *(u2 *)dst = u2{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16)};
        } else {
#pragma unroll
          for (int rr = 0; rr < 4; ++rr)
            if (row0 + rr < g.rows) dst[rr] = __ushort_as_half((uint16_t)hv[rr]);
        }
      }
    }
  };
  for (int set = 0; set + 1 < nsets; ++set) do_set(set, IC<0>());
  do_set(nsets - 1, IC<1>());
}

template <int QW, bool N1, int NG, int RING, bool ONE, bool JOINT>
__global__ __launch_bounds__(1024) void k_smallm_hold(const SmallMBatch b, const SmallMHoldGeom g) {
  smallm_hold_body<QW, N1, NG, RING, ONE, JOINT>(b, g);
}

// Fills the geometry; false where the form does not apply.
static bool hold_plan(const egt_2bitcsr &w, int64_t ldx, int64_t ldy, int M, int count, SmallMHoldGeom &g, int &qw, int &ng, int &ring, size_t &lds) {
  if (w.val_kind != EGT_VAL_INT4 || (w.n_keep != 1 && w.n_keep != 2) || w.rows < 1 || M < 2 || M > 32) return false;
  const bool n1 = w.n_keep == 1;
  const int chunk = n1 ? 128 : 64;
  if (w.cols < chunk || w.cols % chunk != 0 || ldx % 2 != 0) return false;
  const int gm = w.group_size / 32;
  if (w.group_size % 32 != 0 || (gm & (gm - 1)) != 0) return false;
  ng = M <= 16 ? 1 : 2;
  if (n1 && ng > 1) return false;                     // (twice the registers of B)
  g.rows = w.rows; g.M = M;
  g.nchunks = w.cols / chunk;
  g.nsteps = (g.nchunks + 3) / 4;
  if (g.nsteps > (n1 || M > 16 ? 8 : 16)) return false;     // (see the sum of a row)
  g.kpieces = w.cols / 8;
  qw = w.group_size < chunk ? chunk / w.group_size : 1;
  g.gshift = 0;
  while ((chunk << g.gshift) < w.group_size) ++g.gshift;
  g.groups_per_row = w.cols / w.group_size;
  const uint64_t chunks = (uint64_t)w.rows * (uint64_t)g.nchunks, xb = ((uint64_t)(M - 1) * (uint64_t)ldx + (uint64_t)w.cols) * 2,
                 qb = 4ull * (uint64_t)w.rows * (uint64_t)g.groups_per_row;
  if (16 * chunks >= 0x7FFF0000ull || qb >= 0x7FFF0000ull || xb >= 0xFFFF0000ull) return false;
  g.val_bytes = (uint32_t)(16 * chunks); g.idx_bytes = (uint32_t)(8 * chunks); g.qp_bytes = (uint32_t)qb; g.x_bytes = (uint32_t)xb;
  g.ldx = ldx; g.ldy = ldy;
  g.nib_mask = 0x00F0000Fu; g.nib_magic = 0x54006400u;
  g.m4 = 0x0F0F0F0Fu; g.m2 = 0x33333333u;
  g.mtiles = (w.rows + 15) / 16;
  const int ntiles = g.mtiles * count;
  g.blocks = std::min(256, ntiles);
  g.tiles_q = ntiles / g.blocks; g.tiles_r = ntiles % g.blocks;
  // streams: as many as the waves allow, no more than a workgroup has tiles for, a power of two
  const int max_tiles = g.tiles_q + (g.tiles_r ? 1 : 0);
  g.streams = 1; g.stream_shift = 0;
  while (2 * g.streams * g.nsteps <= 16 && g.streams < max_tiles && g.streams < 8) { g.streams *= 2; ++g.stream_shift; }
  g.nw = g.streams * g.nsteps;
  g.step_inv = (65536 + g.nsteps - 1) / g.nsteps;
  // Two row tiles of a wave on their way, which for sixteen waves a compute unit is all the memory takes; more
  // only queue (22016 x 4096, 5 tokens, from HBM: one 12.5 us, two 12.3, three 14.2, four 15.4).  Three where
  // that is all there are, since it saves a set (three times 4096 x 4096: 8.1 us, with sets of two 9.3).
  const int stream_tiles = (max_tiles + g.streams - 1) / g.streams;
  ring = stream_tiles == 3 && g.streams == 1 && ng == 1 && !n1 ? 3 : std::min(stream_tiles, 2);
  const int per_set = ring * g.streams;
  g.sets = (g.tiles_q + per_set - 1) / per_set; g.sets_more = (g.tiles_q + per_set) / per_set;
  const size_t region = (size_t)ng * (n1 ? 16 * HOLD_TOKEN_N1 : 8 * HOLD_PAIR), x_lds = (size_t)g.nsteps * region;
  const size_t slots = (size_t)(2 * ring * ng);
  size_t sums;
  if (g.streams == 1) {                               // over the wave's own part of X
    g.wave_stride = (int)region; g.slot_stride = 1024;
    if (slots * 1024 > region) return false;
    sums = x_lds;
  } else {
    g.wave_stride = 1024; g.slot_stride = g.nw * 1024;
    sums = slots * (size_t)g.nw * 1024;
  }
  g.flags_at = (int)std::max(x_lds, sums);
  // 1:4 rows of more than 2048 columns, where a workgroup has two to four tiles: two streams of at most two
  // tiles each do not pay for the longer start (8192 x 4096, 5 tokens: 5.2 us in the other kernel, 5.6 here; 16384 x 4096: 7.7, 8.7)
  if (n1 && g.nsteps > 4 && max_tiles >= 2 && max_tiles <= 4) return false;
  // Several members whose workgroups in the other kernel do one full round, three row tiles each, where the waves here are all
  // in use (11008 x 2048, 2 tokens, two members: 7.8 us there, 9.3 here; 11008 x 1024, three: 7.4, 9.0; with 500 or
  // 780 tiles a member 0.9 and 0.8 times the time here); and 1:4 members of two tiles a workgroup in all (3259 x 512: 4.1, 4.6)
  if (count > 1 && !n1 && M <= 16 && g.mtiles > 512 && g.mtiles <= 768 && g.nsteps >= 4 && g.nsteps <= 8 && g.nw >= 14) return false;
  if (count > 1 && n1 && max_tiles == 2) return false;
  if (16 * per_set > 64 * g.nw) return false;         // (a thread per row of a set)
  lds = (size_t)g.flags_at + sizeof(uint32_t) * 2 * 16 * (size_t)per_set;
  return lds <= 160 * 1024 - 1024;
}

bool sparse_smallm_hold_supported(const egt_2bitcsr &w, int64_t ldx, int M, int count) {
  SmallMHoldGeom g;
  int qw, ng, ring;
  size_t lds;
  if (tune_flag("EGT_SM_NOHOLD")) return false;
  return hold_plan(w, ldx, w.rows, M, count, g, qw, ng, ring, lds);
}

template <int QW, bool N1, int NG, int RING, bool ONE, bool JOINT>
static hipError_t go_hold1(const SmallMBatch &b, const SmallMHoldGeom &g, size_t lds, hipStream_t stream) {
  // more than 64 KB of dynamic LDS has to be asked for once per kernel and device
  static thread_local int asked_dev = -1;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (asked_dev != dev) {
    e = hipFuncSetAttribute((const void *)k_smallm_hold<QW, N1, NG, RING, ONE, JOINT>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 1024);
    if (e != hipSuccess) return e;
    asked_dev = dev;
  }
  return launch(k_smallm_hold<QW, N1, NG, RING, ONE, JOINT>, dim3(g.blocks), dim3(64 * g.nw), lds, stream, b, g);
}

template <int QW, bool N1, int NG, bool JOINT>
static hipError_t go_hold(const SmallMBatch &b, const SmallMHoldGeom &g, int ring, size_t lds, hipStream_t stream) {
  if (g.streams > 1)
    return ring == 1 ? go_hold1<QW, N1, NG, 1, false, JOINT>(b, g, lds, stream) : go_hold1<QW, N1, NG, 2, false, JOINT>(b, g, lds, stream);
  if constexpr (NG == 1 && !N1)
    if (ring == 3) return go_hold1<QW, N1, NG, 3, true, JOINT>(b, g, lds, stream);
  return ring == 1 ? go_hold1<QW, N1, NG, 1, true, JOINT>(b, g, lds, stream) : go_hold1<QW, N1, NG, 2, true, JOINT>(b, g, lds, stream);
}

// `count` members under one X (the caller has checked that).
hipError_t launch_sparse_smallm_hold(const egt_2bitcsr *ws, const uint16_t *X, int64_t ldx, uint16_t *const *Ys, int64_t ldy, int M, int count,
                                     hipStream_t stream) {
  SmallMHoldGeom g;
  int qw, ng, ring;
  size_t lds;
  if (!hold_plan(ws[0], ldx, ldy, M, count, g, qw, ng, ring, lds)) return hipErrorInvalidValue;
  SmallMBatch b;
  g.vec_store = ldy % 4 == 0;
  for (int k = 0; k < EGT_MAX_BATCH; ++k) {
    const int j = k < count ? k : 0;
    b.row_ptr[k] = ws[j].row_ptr; b.values[k] = (const uint8_t *)ws[j].values; b.idx[k] = (const uint8_t *)ws[j].idx;
    b.qparams[k] = (const uint8_t *)ws[j].qparams; b.X[k] = (const __half *)X; b.Y[k] = (__half *)Ys[j];
    if ((uintptr_t)Ys[j] % 8 != 0) g.vec_store = 0;
  }
  const bool n1 = ws[0].n_keep == 1;
#define EGT_HOLD(QW, N1, NG) (count > 1 ? go_hold<QW, N1, NG, true>(b, g, ring, lds, stream) : go_hold<QW, N1, NG, false>(b, g, ring, lds, stream))
  if (n1) return qw == 4 ? EGT_HOLD(4, true, 1) : qw == 2 ? EGT_HOLD(2, true, 1) : EGT_HOLD(1, true, 1);
  if (ng == 2) return qw == 2 ? EGT_HOLD(2, false, 2) : EGT_HOLD(1, false, 2);
  return qw == 2 ? EGT_HOLD(2, false, 1) : EGT_HOLD(1, false, 1);
#undef EGT_HOLD
}

}  // namespace egt
