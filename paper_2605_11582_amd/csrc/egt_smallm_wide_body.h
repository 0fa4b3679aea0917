// Body of the small-M product for 33 to 64 tokens (2:4, INT4, a pair of quantisation parameters for every chunk or more),
// included by egt_mfma_smallm.hip.  K is split over the waves and the sums are added in wave order, as in
// k_sparse_smallm_ks: the bits of Y are the same.
//
// That kernel takes two token groups a pass: at more than 32 tokens it walks its rows twice, and the operands are
// fetched (from the caches), exchanged between lanes and dequantised twice.  Here a K-step of the row tiles is
// dequantised once, stays in registers (16 a tile) and serves all token groups.  What bounds it then is X: every
// workgroup pulls all of X through the L2 (11008 x 4096, 64 tokens: 134 MB beside 18 MB of weights).  So X comes in units
// of one token group of one K-step, into two regions of a wave's own: the unit after the next is requested as soon as a
// region has been read, across K-steps, and there is always one on its way.  The number of token groups is the
// compiler's: counted in the kernel, its branches cost 0.5 to 1 us a product.
//
// Requests return in order.  A wave asks for X(0) A(0) X(1) A(1) first (X by unit, A by phase), then within a phase p,
// after unit 0 has been read, X(next but one) A(p + 2), and after every other unit X(next but one).  The waits below
// count what is newer than the unit that is needed.  The odd last phase (LAST) asks for no tiles and counts none: the
// compiler leaves out requests whose registers nothing reads any more.
//
// Matrices from memory, us, before -> now, 64 tokens: 11008 x 4096 20.1 -> 16.4, 13824 x 5120 27.0 -> 21.6, 4096 x 4096
// 11.7 -> 11.4, 4096 x 11008 25.0 -> 22.5, 4096 x 512 7.7 -> 5.9, two of 11008 x 4096 37.9 -> 30.8; 48 tokens: 4096 x 4096
// 10.7 -> 10.2, three of 8192 x 2048 28.1 -> 18.4; 33 tokens: 4096 x 4096 9.9 -> 9.9, 5120 x 5120 18.7 -> 12.5.
#ifndef EGT_SMALLM_WIDE_BODY_H
#define EGT_SMALLM_WIDE_BODY_H

namespace egt {

constexpr int WIDE_WAVES = 8, WIDE_REGION = 8 * KS_PAIR;

// NG: token groups of 16 (3 or 4).  NIT: row tiles of a workgroup at a time.  JOINT: several matrices under one X as one,
// row tile v of the launch is tile v - k * mtiles of member k = v / mtiles.
template <int NG, int NIT, bool JOINT = false>
__device__ __forceinline__ void smallm_wide_body(const uint32_t *row_ptr, const uint8_t *values, const uint8_t *idx, const uint8_t *qparams,
                                                 const __half *X, __half *Y, const SmallMKsLaunch &g, const SmallMBatch *b = nullptr) {
  extern __shared__ __align__(16) uint8_t xs[];       // two regions of X for each wave, later its sums; row flags
  constexpr int XREQ = 8;                             // requests of a unit of X
  typedef ATile<EGT_VAL_INT4, 1> Tile;
  constexpr int NA = NIT * Tile::LOADS;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = g.nw, nblocks = g.blocks;
  const int i = lane & 15, kb = lane >> 4;
  const int li = lane >> 2, lc = lane & 3;            // row, chunk this lane fetches
  const int from = 4 * (4 * i + kb);                  // lane that fetched the chunk of lane (i, kb), as a byte address
  const int mytiles = g.tiles_q + ((int)blockIdx.x < g.tiles_r ? 1 : 0);
  const uint32_t magic = in_vgpr(g.nib_magic);
  const uint32_t S_row = (uint32_t)g.nchunks * 32u;
  uint8_t *mine = xs + wave * (2 * WIDE_REGION);
  uint32_t *flags = (uint32_t *)(xs + nw * (2 * WIDE_REGION));
  const int myphases = (g.nsteps - wave + nw - 1) / nw;
  auto member = [&](int &v) {                         // v: tile of the launch -> of its member, which is returned
    if constexpr (!JOINT) return 0u;
    const int k = (v >= g.mtiles) + (v >= 2 * g.mtiles) + (v >= 3 * g.mtiles);
    v -= k * g.mtiles;
    return (unsigned)k;
  };
  auto flag_row = [&](int t0, unsigned &k) {
    const int t = t0 + (int)(threadIdx.x >> 4);
    int v = (int)blockIdx.x + t * nblocks;
    k = member(v);
    return t < mytiles ? 16 * v + (int)(threadIdx.x & 15) : g.rows;
  };
  auto load_rp = [&](int t0) -> uint32_t {
    unsigned k;
    const int r = flag_row(t0, k);
    if ((int)threadIdx.x >= 16 * NIT || r >= g.rows) return 0u;
    if constexpr (JOINT) return pick4(b->row_ptr, k)[r];
    else return row_ptr[r];
  };
  uint32_t frp = load_rp(0);
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc(X, g.x_bytes);
  const uint32_t off_range = 0xFFFFFFF0u;

  // X of a unit: token group u % ngroups of the wave's K-step u / ngroups; always eight requests
  const int xtl = lane >> 5, slot_piece = (lane & 31) ^ xtl;
  auto dma_x = [&](int p, int grp, int region) {
    // (pinned: worked out ahead for every group and request, the uniform offsets and conditions would spill)
    int step = p * nw + wave, left = p < myphases ? g.M - 16 * grp : 0;
    uint32_t at = 512u * (uint32_t)step + (uint32_t)grp * 32u * (uint32_t)g.ldx;
    asm volatile("" : "+s"(step), "+s"(left), "+s"(at) : : "memory");
    const int vp = max(1, min(32, g.kpieces - 32 * step));
    const uint32_t off_lo = 16u * (uint32_t)min(slot_piece, vp - 1), off_hi = off_lo + (uint32_t)xtl * (uint32_t)(2 * g.ldx);
#pragma unroll
    for (int q = 0; q < XREQ; ++q) {
      const bool on = 2 * q < left;                   // uniform
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(mine + region * WIDE_REGION + KS_PAIR * q), 16,
                                               on ? (2 * q + 1 < left ? off_hi : off_lo) : off_range, on ? at : 0u, 0, 0);
      at += 4u * (uint32_t)g.ldx;
    }
    asm volatile("" ::: "memory");
  };
  auto zero_tail = [&](int step, int region) {
    const int vp = g.kpieces - 32 * step;
    if (vp < 32 && slot_piece >= vp) {
#pragma unroll
      for (int q = 0; q < XREQ; ++q) *(u4 *)(mine + region * WIDE_REGION + KS_PAIR * q + 16 * lane) = u4{0, 0, 0, 0};
    }
  };
  const int b_off = KS_PAIR * ((lane & 15) >> 1) + 512 * (lane & 1) + 16 * (8 * (lane >> 5) + (((lane >> 4) ^ lane) & 1));

  for (int t0 = 0; t0 < mytiles; t0 += NIT) {
    const int nit = min(NIT, mytiles - t0);
    auto load_a = [&](Tile (&a)[NIT], int p) {
      const int step = p * nw + wave;
      const bool in = p < myphases;                   // uniform
      const uint32_t lcc = (uint32_t)min((int)in_vgpr((uint32_t)lc), in ? g.nchunks - 1 - 4 * step : 0);
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const bool on = in && it < nit;               // uniform
        int v = on ? (int)blockIdx.x + (t0 + it) * nblocks : 0;
        asm volatile("" : "+s"(v));
        const unsigned k = member(v);
        __amdgpu_buffer_rsrc_t r_val, r_idx, r_qp;
        if constexpr (JOINT) {
          r_val = make_rsrc(pick4(b->values, k), g.val_bytes); r_idx = make_rsrc(pick4(b->idx, k), g.idx_bytes);
          r_qp = make_rsrc(pick4(b->qparams, k), g.qp_bytes);
        } else {
          r_val = make_rsrc(values, g.val_bytes); r_idx = make_rsrc(idx, g.idx_bytes); r_qp = make_rsrc(qparams, g.qp_bytes);
        }
        const uint32_t rel = (uint32_t)min(li, g.rows - 1 - 16 * v);
        const uint32_t cl = rel * (uint32_t)g.nchunks + lcc;
        const uint32_t cu = on ? (uint32_t)(16 * v) * (uint32_t)g.nchunks + (uint32_t)(4 * step) : 0u;
        a[it].iw = __builtin_amdgcn_raw_buffer_load_b64(r_idx, on ? 8u * cl : off_range, 8u * cu, 0);
        a[it].nib[0] = __builtin_amdgcn_raw_buffer_load_b128(r_val, on ? 16u * cl : off_range, 16u * cu, 0);
        const uint32_t qrow_l = rel * (uint32_t)g.groups_per_row, qrow_u = on ? (uint32_t)(16 * v) * (uint32_t)g.groups_per_row : 0u;
        a[it].qp[0] = __builtin_amdgcn_raw_buffer_load_b32(r_qp, on ? 4u * (qrow_l + (lcc >> g.gshift)) : off_range,
                                                           on ? 4u * (qrow_u + (uint32_t)((4 * step) >> g.gshift)) : 0u, 0);
      }
    };
    f4 acc[NIT][NG];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int grp = 0; grp < NG; ++grp) acc[it][grp] = f4{0.f, 0.f, 0.f, 0.f};
    Tile raw0[NIT], raw1[NIT];
    dma_x(0, 0, 0);
    load_a(raw0, 0);
    dma_x(0, 1, 1);
    load_a(raw1, 1);
    int reg = 0;                                      // region of the unit
    auto phase = [&](Tile (&raw)[NIT], int p, auto last) {
      constexpr bool LAST = decltype(last)::value;
      const int step = p * nw + wave;
      u4 held[NIT][4];
      uint32_t hiw[NIT][2];
#pragma unroll
      for (int grp = 0; grp < NG; ++grp) {
        // newer than this unit: the next one and, where they were asked for since, tiles
        if (LAST || grp == 3) wait_vmem<XREQ>();
        else if (grp == 2) wait_vmem<XREQ + NA>();
        else if (p == 0 && grp == 1) wait_vmem<XREQ + 2 * NA>();
        else if (p == 0 || grp == 1) wait_vmem<XREQ + NA>();
        else wait_vmem<XREQ>();
        zero_tail(step, reg);
        u8v bx[4];
        const uint8_t *at = mine + reg * WIDE_REGION + b_off;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const u4 lo = *(const u4 *)(at + 32 * m), hi = *(const u4 *)(at + 256 + 32 * m);
          bx[m] = u8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        if (grp == 0) {
          const bool live = 4 * step + kb < g.nchunks;
#pragma unroll
          for (int it = 0; it < NIT; ++it) {
            u4 nib;
#pragma unroll
            for (int d = 0; d < 4; ++d) nib[d] = lane_perm(from, raw[it].nib[0][d]);
            hiw[it][0] = lane_perm(from, raw[it].iw[0]);
            hiw[it][1] = lane_perm(from, raw[it].iw[1]);
            const uint32_t qp = lane_perm(from, raw[it].qp[0]);
            const uint32_t s2 = live ? __builtin_amdgcn_perm(qp, qp, 0x01000100u) : 0u;
            const uint32_t off = pk_add_f16(__builtin_amdgcn_perm(qp, qp, 0x03020302u), g.nib_magic);
#pragma unroll
            for (int m = 0; m < 4; ++m) held[it][m] = dequant8(nib[m], off, s2, g.nib_mask, magic);
          }
        }
        wait_lds();                                   // the region and the fetch registers are free
        // the unit after the next
        const int n2 = grp + 2, over = n2 >= NG ? 1 : 0;
        dma_x(p + over, over ? n2 - NG : n2, reg);
        if (!LAST && grp == 0) load_a(raw, p + 2);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          if (it < nit) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const int iword = (int)hiw[it][m >> 1];
              f4 &sum = acc[it][grp];
              if (m & 1)
                sum = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, held[it][m]), __builtin_bit_cast(h16, bx[m]), sum, iword, 0, 1);
              else
                sum = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(h8, held[it][m]), __builtin_bit_cast(h16, bx[m]), sum, iword, 0, 0);
            }
          }
        }
        reg ^= 1;
      }
    };
    int p = 0;
    for (; p + 2 <= myphases; p += 2) {
      phase(raw0, p, std::false_type());
      phase(raw1, p + 1, std::false_type());
    }
    if (p < myphases) phase(raw0, p, std::true_type());
    wait_vmem<0>();                                   // (nothing more is on its way into the regions)
    if ((int)threadIdx.x < 16 * NIT) {
      unsigned k;
      const int r = flag_row(t0, k);
      flags[threadIdx.x] = (r < g.rows && frp == (uint32_t)r * S_row) ? 1u : 0u;
    }
    if (t0 + NIT < mytiles) frp = load_rp(t0 + NIT);
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int grp = 0; grp < NG; ++grp)
        if (it < nit) *(f4 *)(mine + (it * NG + grp) * 1024 + 16 * lane) = acc[it][grp];
    lds_barrier();
    // a wave takes a tile's kilobyte, four rows of a token a lane: float 4 l + v of it is D[row 4 (l >> 4) + v][token l & 15]
    for (int tg = wave; tg < nit * NG; tg += nw) {
      const int it = tg / NG, grp = tg - it * NG;
      const uint8_t *src = xs + (it * NG + grp) * 1024 + 16 * lane;
      const u4 ok = *(const u4 *)(flags + 16 * it + 4 * (lane >> 4));
      f4 part[WIDE_WAVES];
#pragma unroll
      for (int w = 0; w < WIDE_WAVES; ++w) part[w] = *(const f4 *)(src + min(w, nw - 1) * (2 * WIDE_REGION));
      f4 sum = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < WIDE_WAVES; ++w)
        if (w < nw) sum += part[w];                   // (uniform)
      int v = (int)blockIdx.x + (t0 + it) * nblocks;
      const unsigned k = member(v);
      __half *out = Y;
      if constexpr (JOINT) out = pick4(b->Y, k);
      const int row0 = 16 * v + 4 * (lane >> 4), tok = 16 * grp + (lane & 15);
      uint32_t hv[4];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) hv[rr] = ok[rr] ? __half_as_ushort(__float2half(sum[rr])) : 0x7E00u;
      if (tok < g.M) {
        __half *dst = out + (int64_t)tok * g.ldy + row0;
        if (g.vec_store && row0 + 3 < g.rows) {
          *(u2 *)dst = u2{hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16)};
        } else {
#pragma unroll
          for (int rr = 0; rr < 4; ++rr)
            if (row0 + rr < g.rows) dst[rr] = __ushort_as_half((uint16_t)hv[rr]);
        }
      }
    }
    if (t0 + NIT < mytiles) lds_barrier();            // the next round writes the regions
  }
}

template <int NG, int NIT>
__global__ __launch_bounds__(64 * WIDE_WAVES) void k_smallm_wide(const uint32_t *row_ptr, const uint8_t *values, const uint8_t *idx,
                                                                 const uint8_t *qparams, const __half *X, __half *Y, const SmallMKsLaunch g) {
  smallm_wide_body<NG, NIT>(row_ptr, values, idx, qparams, X, Y, g);
}
// (members of their own tokens: blockIdx.y names the member)
template <int NG, int NIT>
__global__ __launch_bounds__(64 * WIDE_WAVES) void k_smallm_wide_batch(const SmallMBatch b, const SmallMKsLaunch g) {
  const unsigned k = blockIdx.y;
  smallm_wide_body<NG, NIT>(pick4(b.row_ptr, k), pick4(b.values, k), pick4(b.idx, k), pick4(b.qparams, k), pick4(b.X, k), pick4(b.Y, k), g);
}
template <int NG, int NIT>
__global__ __launch_bounds__(64 * WIDE_WAVES) void k_smallm_wide_ks_joint(const SmallMBatch b, const SmallMKsLaunch g) {
  smallm_wide_body<NG, NIT, true>(nullptr, nullptr, nullptr, nullptr, b.X[0], nullptr, g, &b);
}

template <int NG, int NIT>
static hipError_t go_wide(const egt_2bitcsr &w, const uint16_t *X, uint16_t *Y, const SmallMKsLaunch &g, int nblocks, hipStream_t stream,
                          const SmallMBatch *batch, int count) {
  const size_t lds = (size_t)g.nw * 2 * WIDE_REGION + 64 * 4;
  if constexpr (NIT > 2)                              // (members as one matrix: three tiles a workgroup and more)
    if (batch && g.mtiles) return launch(k_smallm_wide_ks_joint<NG, NIT>, dim3(nblocks), dim3(64 * g.nw), lds, stream, *batch, g);
  if (batch) return launch(k_smallm_wide_batch<NG, NIT>, dim3(nblocks, count), dim3(64 * g.nw), lds, stream, *batch, g);
  return launch(k_smallm_wide<NG, NIT>, dim3(nblocks), dim3(64 * g.nw), lds, stream, w.row_ptr, (const uint8_t *)w.values,
                (const uint8_t *)w.idx, (const uint8_t *)w.qparams, (const __half *)X, (__half *)Y, g);
}

}  // namespace egt
#endif
