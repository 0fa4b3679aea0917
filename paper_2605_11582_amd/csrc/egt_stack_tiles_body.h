// Body of the verification-stack kernel with operands and parameters through LDS of the wave's own (included by
// egt_mfma_smallm.hip, which holds the geometry, the table and the launch).
//
// The work is k_smallm_rows': a workgroup of 8 waves owns 8 T consecutive row tiles for all of K, T a wave, in rounds of
// two K-steps, the token rows of a round staged once a workgroup.  The sums run in the same order, so a product has the
// same bits in either.  What differs is what bound that kernel (sixteen 2:4 layers of a 7B stack, 16 tokens, 341 us; with the
// requests of the weights out of range, that is everything but the memory, 206):
//  - Lane permutations took 80 of the 206 us (fourteen and seven selects a K-step).  Here a wave writes what it
//    fetched to 2 KB of LDS and reads it back in operand form: six writes and four reads for two K-steps.
//  - Parameters are a 13th of the bytes and took 40 of the 341 us: 16 bytes a row and round, of lines that were gone from
//    the caches before the next round.  Here a window of QW bytes of each row is fetched into LDS at once, whole lines
//    with QW = 128.
//  - The compiler waited for all requests at the top of every other round: a request under a condition, and a round of
//    the loop under one, make its count of what is pending the smallest of all paths.  Here rounds past the last one are requested
//    too (out of range: no traffic), and a loop turn is two rounds, the odd last round behind it.
// us before, now (bits the same; another clock than the 341 above, both sides of it in turn): 2:4 344 -> 303 at 16 tokens, 322 ->
// 274 at 4, 531 -> 511 at 64, 419 -> 365 at 32 (two tiles a wave); 1:4 (eleven layers) 174 -> 158 at 16, 165 -> 151 at 4, 225 -> 215 at 32.
// What bounds it now: HBM and the L2 (the weights and token rows alone take 260 us at 16 tokens, 178 without weights).
#ifndef EGT_STACK_TILES_BODY_H
#define EGT_STACK_TILES_BODY_H

namespace egt {

constexpr int ST_WAVES = 8, ST_Q = 2;
// LDS bytes of a workgroup: two rounds of token rows; a wave's place for operands; QW bytes of each of its rows
constexpr int st_wave_bytes(int t, int qw, bool narrow) { return (narrow ? 1024 : 2048) + t * 16 * qw; }
constexpr int st_lds_bytes(int ng, int t, int qw, bool narrow, bool n1) { return 2 * ng * ST_Q * rs_step_bytes(n1) + ST_WAVES * st_wave_bytes(t, qw, narrow); }

// NG token groups of 16, T row tiles a wave, QW bytes of parameters a row at a time, N1: 1:4.
template <int NG, int T, int QW, bool NARROW, bool N1>
__device__ __forceinline__ void stack_tiles_body(const uint8_t *__restrict__ table, int count) {
  constexpr int W = ST_WAVES, Q = ST_Q, STEP = rs_step_bytes(N1), REGION = NG * Q * STEP;
  constexpr int XREQ = N1 ? 16 : 8;                   // requests of X per K-step and token group
  constexpr int NM = N1 ? 8 : 4;                      // matrix instructions per K-step
  constexpr int PIECES = N1 ? 64 : 32;                // 16-byte pieces of a token row in a K-step
  constexpr int REQ = NG * Q * XREQ / W;              // requests of X a wave issues per round
  constexpr int LPT = 4;                              // requests of a tile's round: index words and nibbles of either half of the rows
  static_assert(REQ * W == NG * Q * XREQ, "the waves share the requests of a round evenly");
  static_assert(QW == 128 || QW == 64 || QW == 32, "parameters of a row");
  extern __shared__ __align__(16) uint8_t xs[];       // two regions of token rows, then the waves' own parts
  typedef __attribute__((address_space(1))) const uint32_t *g_u32;
  typedef __attribute__((address_space(1))) const uint8_t *g_u8;
  typedef __attribute__((address_space(1))) const __half *g_h;
  typedef __attribute__((address_space(1))) __half *g_hw;
  // the list behind the descriptors names the matrix (high half) and the workgroup's place in it (low half)
  const uint32_t where = ((const uint32_t *)(table + (size_t)count * EGT_STACK_ENTRY_BYTES))[blockIdx.x];
  const int wg = (int)(where & 0xFFFFu);
  const SmallMStackEntry *e = (const SmallMStackEntry *)(table + (size_t)(where >> 16) * EGT_STACK_ENTRY_BYTES);
  const SmallMKsGeom g = e->g;
  const uint32_t *row_ptr = (const uint32_t *)(g_u32)e->row_ptr;
  __half *Y = (__half *)(g_hw)e->Y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, kb = lane >> 4;            // operand form: row i of the tile, chunk kb of the step
  // this wave's row tiles (a wave past the last tile has none, but still stages its share of X and meets the barriers)
  const int tile0 = T * (wg * W + wave);
  const int ntiles = min(max(g.ntiles - tile0, 0), T);                      // uniform
  const int nsteps = g.nsteps, nrounds = (nsteps + Q - 1) / Q;
  const int last_row = max(g.rows - 1 - 16 * tile0, 0);                     // of the matrix, from the wave's first
  const uint32_t magic = in_vgpr(g.nib_magic);
  const uint32_t S_row = (uint32_t)g.nchunks * 32u;
  // row pointers first, checked at the end: a row whose pointer is not r * S yields NaN
  const int frow = 16 * tile0 + lane;
  const bool fchecked = lane < 16 * ntiles && frow < g.rows;
  const uint32_t frp = fchecked ? row_ptr[frow] : 0u;

  const __amdgpu_buffer_rsrc_t r_val = make_rsrc((const uint8_t *)(g_u8)e->values, g.val_bytes);
  const __amdgpu_buffer_rsrc_t r_idx = make_rsrc((const uint8_t *)(g_u8)e->idx, g.idx_bytes);
  const __amdgpu_buffer_rsrc_t r_qp = make_rsrc((const uint8_t *)(g_u8)e->qparams, g.qp_bytes);
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc((const __half *)(g_h)e->X, g.x_bytes);
  const uint32_t off_range = 0xFFFFFFF0u;             // past every buffer: such a request returns zeros and moves no data

  // ---- requests of the weights: a round of a tile is 16 rows x 8 chunks, a request 8 rows x 8 chunks, 128 contiguous
  // bytes of nibbles a row: lane (r, c) = (lane >> 3, lane & 7) fetches chunk c of row 8 h + r
  struct RoundRegs {
    u4 nib[2];
    u2 iw[2];
  };
  // (NARROW: 16 rows x 4 chunks, a K-step a request, 64 bytes of nibbles a row)
  const int r8 = NARROW ? lane >> 2 : lane >> 3, c8 = NARROW ? lane & 3 : lane & 7;
  auto load = [&](RoundRegs (&a)[T], int round) {
    const int c0 = 4 * Q * round;                                             // first chunk of the round
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const bool on = t < ntiles && round < nrounds;                          // uniform
      const uint32_t cu = on ? (uint32_t)(16 * (tile0 + t)) * (uint32_t)g.nchunks + (uint32_t)c0 : 0u;   // uniform part of the chunk number
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t lcc = (uint32_t)min((int)in_vgpr((uint32_t)c8) + (NARROW ? 4 * h : 0), g.nchunks - 1 - c0);   // chunk inside it (clamped)
        const uint32_t rel = (uint32_t)min(NARROW ? r8 : 8 * h + r8, max(last_row - 16 * t, 0));       // row inside the tile (clamped)
        const uint32_t cl = rel * (uint32_t)g.nchunks + lcc;                  // lane part
        a[t].iw[h] = __builtin_amdgcn_raw_buffer_load_b64(r_idx, on ? 8u * cl : off_range, 8u * cu, 0);
        a[t].nib[h] = __builtin_amdgcn_raw_buffer_load_b128(r_val, on ? 16u * cl : off_range, 16u * cu, 0);
      }
    }
  };
  // ---- fetched form -> operand form: lane (i, kb) takes chunk 4 q + kb of row i for K-step q of the round.  Row r keeps its
  // eight chunks in the order c ^ (r >> 1), so that the sixteen rows that are read at a time lie on different
  // banks.  (A wave's LDS operations run in order: no barrier, but the compiler must keep them in order too.)
  uint8_t *scr = xs + 2 * REGION + wave * st_wave_bytes(T, QW, NARROW);
  const int w8 = NARROW ? 4 * r8 + (c8 ^ ((r8 >> 2) & 3)) : 8 * r8 + (c8 ^ (r8 >> 1)), w8h = 8 * (8 + r8) + (c8 ^ ((8 + r8) >> 1));
  const int o0 = NARROW ? 4 * i + (kb ^ (i >> 2)) : 8 * i + (kb ^ (i >> 1)), o1 = 8 * i + ((4 + kb) ^ (i >> 1));
  struct Operands {
    u4 nib;
    u2 iw;
    uint32_t qp;
  };
  auto exchange = [&](const RoundRegs &a, Operands &q0, Operands &q1) {
    asm volatile("" ::: "memory");
    if constexpr (NARROW) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        Operands &o = q ? q1 : q0;
        *(u4 *)(scr + 16 * w8) = a.nib[q];
        asm volatile("" ::: "memory");
        o.nib = *(const u4 *)(scr + 16 * o0);
        asm volatile("" ::: "memory");
        *(u2 *)(scr + 8 * w8) = a.iw[q];
        asm volatile("" ::: "memory");
        o.iw = *(const u2 *)(scr + 8 * o0);
        asm volatile("" ::: "memory");
      }
      return;
    }
    *(u4 *)(scr + 16 * w8) = a.nib[0];
    *(u4 *)(scr + 16 * w8h) = a.nib[1];
    asm volatile("" ::: "memory");
    q0.nib = *(const u4 *)(scr + 16 * o0);
    q1.nib = *(const u4 *)(scr + 16 * o1);
    asm volatile("" ::: "memory");
    *(u2 *)(scr + 8 * w8) = a.iw[0];
    *(u2 *)(scr + 8 * w8h) = a.iw[1];
    asm volatile("" ::: "memory");
    q0.iw = *(const u2 *)(scr + 8 * o0);
    q1.iw = *(const u2 *)(scr + 8 * o1);
    asm volatile("" ::: "memory");
  };
  // ---- parameters: a window of QW bytes of each row (QW / 4 pairs), in 16-byte pieces; row r keeps piece p at place p ^
  // q_swizzle(r).  A request fetches 64 pieces: some rows of a tile, or (QW = 32) all rows of both tiles.  What of a
  // piece lies past a row's end belongs to the next row, or past the buffer: it is not read.
  uint8_t *scq = scr + (NARROW ? 1024 : 2048);
  constexpr int QPIECES = QW / 16, QROWS = 64 / QPIECES;
  auto q_swizzle = [&](int r) { return QW == 128 ? (r >> 1) & 7 : QW == 64 ? (r >> 2) & 3 : (r >> 3) & 1; };
  const int q_sw = q_swizzle(i);
  auto load_q = [&](int window) {
#pragma unroll
    for (int n = 0; n < (T * QW + 63) / 64; ++n) {
      if (T * QW < 64 && lane >= T * QW) break;       // (a request of fewer pieces: the other lanes would write zeros past them)
      const int r = QROWS * n + lane / QPIECES, piece = (lane % QPIECES) ^ q_swizzle(r & 15);
      const bool on = ntiles > 0;                     // uniform
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r_qp, (__attribute__((address_space(3))) void *)(scq + 1024 * n), 16,
                                               on ? 4u * (uint32_t)min(r, last_row) * (uint32_t)g.groups_per_row + 16u * (uint32_t)piece + (uint32_t)(QW * window) : off_range,
                                               on ? 4u * (uint32_t)(16 * tile0) * (uint32_t)g.groups_per_row : 0u, 0, 0);   // (the tile's first row: inside the buffer)
    }
  };
  auto get_q = [&](int step, int t) {                 // (a chunk past the end of K takes the last one's: it enters with scale 0)
    const int x = (min(4 * step + kb, g.nchunks - 1) >> g.gshift) & (QW / 4 - 1);
    return *(const uint32_t *)(scq + t * 16 * QW + QW * i + 16 * ((x >> 2) ^ q_sw) + 4 * (x & 3));
  };
  const int window_mask = ((QW / 16) << g.gshift) - 1;      // K-steps of a window, less one: QW / 4 pairs of 1 << gshift chunks

  // ---- X of a round, as in k_smallm_rows: one request per token group, K-step and pair of tokens (1:4: token), each landing in
  // one kilobyte of the region; every wave issues the same number, a pair past M or a step past K asks out of range
  const int xtl = lane >> 5;
  const int slot_piece = N1 ? lane : ((lane & 31) ^ xtl);   // piece of X this lane delivers
  auto dma_x = [&](int round, int buf) {
    asm volatile("" ::: "memory");                    // the requests stay together, in program order
#pragma unroll
    for (int k = 0; k < REQ; ++k) {
      const int r = wave * REQ + k, gq = r / XREQ, u = r % XREQ;
      const int grp = gq / Q, t0 = 16 * grp + (N1 ? u : 2 * u);
      const int step = Q * round + gq % Q;
      const int vp = max(1, min(PIECES, g.kpieces - PIECES * step));   // pieces of the step inside K
      const uint32_t off_lo = 16u * (uint32_t)min(slot_piece, vp - 1);
      const uint32_t off_hi = N1 ? off_lo : off_lo + (uint32_t)xtl * (uint32_t)(2 * g.ldx);
      const bool on = t0 < g.M && step < nsteps;      // uniform
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(xs + buf * REGION + gq * STEP + (N1 ? KS_TOKEN_N1 : KS_PAIR) * u), 16,
                                               on ? (t0 + 1 < g.M ? off_hi : off_lo) : off_range,
                                               on ? (uint32_t)(16 * PIECES) * (uint32_t)step + (uint32_t)t0 * (uint32_t)(2 * g.ldx) : 0u, 0, 0);
    }
    asm volatile("" ::: "memory");
  };
  // the pieces of a partly filled step that lie past K become zeros (the issuing wave's own requests)
  auto zero_tail = [&](int round, int buf) {
#pragma unroll
    for (int k = 0; k < REQ; ++k) {
      const int r = wave * REQ + k;
      const int vp = g.kpieces - PIECES * (Q * round + (r / XREQ) % Q);
      if (vp > 0 && vp < PIECES && slot_piece >= vp)
        *(u4 *)(xs + buf * REGION + (r / XREQ) * STEP + (N1 ? KS_TOKEN_N1 : KS_PAIR) * (r % XREQ) + 16 * lane) = u4{0, 0, 0, 0};
    }
  };
  // B operand of instruction m of a K-step: lane (n, b) holds token n, k-octets b and 4 + b of the instruction's 16-column group
  const int b_off = N1 ? KS_TOKEN_N1 * (lane & 15) + 16 * (16 * (lane >> 5) + ((lane >> 4) & 1))
                       : KS_PAIR * ((lane & 15) >> 1) + 512 * (lane & 1) + 16 * (8 * (lane >> 5) + (((lane >> 4) ^ lane) & 1));
  auto read_b = [&](const uint8_t *region, int m) {
    const u4 lo = *(const u4 *)(region + b_off + 32 * m), hi = *(const u4 *)(region + b_off + (N1 ? 512 : 256) + 32 * m);
    return u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  };

  f4 acc[T][NG];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int grp = 0; grp < NG; ++grp) acc[t][grp] = f4{0.f, 0.f, 0.f, 0.f};
  // Requests in a round, in this order: X(j + 1), a window of parameters where the next round begins one, the
  // weights of round j + 2 - so that at the top of a round those of round j + 1, T * LPT, may be pending and everything older
  // has arrived.  The barrier is issued with its own wait counts: a fence would wait for every pending request.
  RoundRegs raw0[T], raw1[T];
  load_q(0);
  load(raw0, 0);
  dma_x(0, 0);
  load(raw1, 1);
  // (The last round of an odd number requests nothing and waits for everything: the compiler drops or moves requests whose
  //  registers are not read on the way there, so none may be counted on.)
  auto round = [&](RoundRegs (&cur)[T], int j, int buf, auto last_round) {
    constexpr bool LAST = decltype(last_round)::v != 0;
    // the weights of the round and this wave's share of X(j) have arrived
    if constexpr (LAST) wait_vmem<0>();
    else wait_vmem<T * LPT>();
    zero_tail(j, buf);
    // X(j) of every wave has landed; nobody reads the region of round j - 1 any more
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (!LAST) dma_x(j + 1, buf ^ 1);
    Operands ops[Q][T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      exchange(cur[t], ops[0][t], ops[1][t]);
#pragma unroll
      for (int q = 0; q < Q; ++q) ops[q][t].qp = get_q(Q * j + q, t);
    }
    const int next = Q * (j + 1);
    if (!LAST && (next & window_mask) == 0 && next < nsteps) { // uniform: the next round begins a window
      wait_lds();                                     // this one has been read
      load_q(next / (window_mask + 1));
    }
    if constexpr (!LAST) load(cur, j + 2);            // (the fetch registers are free again)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      // (a step past K, a wave without a tile: requested out of range, zeros with scale 0)
      const bool live = 4 * (Q * j + q) + kb < g.nchunks;   // false: a chunk past the end of K
      // the operands of the step's instructions serve every token group
      u4 av[T][NM];
      uint32_t iwv[T][NM / 2];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const Operands &o = ops[q][t];
        const uint32_t s2 = live ? __builtin_amdgcn_perm(o.qp, o.qp, 0x01000100u) : 0u;
        const uint32_t off = pk_add_f16(__builtin_amdgcn_perm(o.qp, o.qp, 0x03020302u), g.nib_magic);
        if constexpr (N1) {
          // every slot becomes the pair {value, 0} with its offset in the even index field; instruction m takes
          // slots 4 m .. 4 m + 3 of the chunk: bytes 2 (m & 1), 2 (m & 1) + 1 of dword m >> 1
          iwv[t][0] = spread_idx<0>(o.iw[0], g.m4, g.m2);
          iwv[t][1] = spread_idx<1>(o.iw[0], g.m4, g.m2);
          iwv[t][2] = spread_idx<0>(o.iw[1], g.m4, g.m2);
          iwv[t][3] = spread_idx<1>(o.iw[1], g.m4, g.m2);
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const uint32_t d = o.nib[m >> 1];
            av[t][m] = m & 1 ? dequant4_14<1>(d, off, s2, g.nib_mask, magic) : dequant4_14<0>(d, off, s2, g.nib_mask, magic);
          }
        } else {
          iwv[t][0] = o.iw[0];
          iwv[t][1] = o.iw[1];
#pragma unroll
          for (int m = 0; m < NM; ++m) av[t][m] = dequant8(o.nib[m], off, s2, g.nib_mask, magic);
        }
      }
#pragma unroll
      for (int grp = 0; grp < NG; ++grp) {
        if (NG > 1 && 16 * grp >= g.M) continue;      // uniform
        const uint8_t *bregion = xs + buf * REGION + (grp * Q + q) * STEP;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const u8v bx = read_b(bregion, m);          // (read per instruction: 8 registers of B at a time)
#pragma unroll
          for (int t = 0; t < T; ++t) {
            const int iword = (int)iwv[t][m >> 1];
            f4 &sum = acc[t][grp];
            if (m & 1)
              sum = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, av[t][m]), __builtin_bit_cast(h16, bx), sum, iword, 0, 1);
            else
              sum = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, av[t][m]), __builtin_bit_cast(h16, bx), sum, iword, 0, 0);
          }
        }
      }
    }
  };
  int j = 0;
  for (; j + 2 <= nrounds; j += 2) {
    round(raw0, j, 0, IC<0>());
    round(raw1, j + 1, 1, IC<0>());
  }
  if (j < nrounds) round(raw0, j, 0, IC<1>());
  wait_vmem<0>();                                     // (no request for LDS outlives the workgroup)
  // register v of lane l = D[row 4 (l >> 4) + v][token l & 15]: four consecutive rows of one token
  const uint64_t good = __builtin_amdgcn_ballot_w64(fchecked && frp == (uint32_t)frow * S_row);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (t >= ntiles) return;
    const int row0 = 16 * (tile0 + t) + 4 * (lane >> 4);
#pragma unroll
    for (int grp = 0; grp < NG; ++grp) {
      const int tok = 16 * grp + (lane & 15);
      if (tok >= g.M) continue;
      uint32_t hv[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        hv[v] = ((good >> (16 * t + 4 * (lane >> 4) + v)) & 1) ? (uint32_t)__half_as_ushort(__float2half(acc[t][grp][v])) : 0x7E00u;
      __half *dst = Y + (int64_t)tok * g.ldy + row0;
      if (g.vec_store && row0 + 3 < g.rows) {
        *(u2 *)dst = u2{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16)};
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (row0 + v < g.rows) dst[v] = __ushort_as_half((uint16_t)hv[v]);
      }
    }
  }
}

// (one workgroup of 8 waves takes the LDS of a compute unit with two tiles a wave, two share it with one)
template <int NG, int T, int QW, bool NARROW, bool N1>
__global__ __launch_bounds__(64 * ST_WAVES, T == 1 ? 4 : 2) void k_stack_tiles(const uint8_t *__restrict__ table, int count) {
  stack_tiles_body<NG, T, QW, NARROW, N1>(table, count);
}

}  // namespace egt
#endif
