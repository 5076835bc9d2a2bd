// Causal block-centric attention with several heads per KV head: each row's
// first, previous and own blocks (App. B's forced set, as far as the row
// selected them), and the merge of the partials that the block-centric kernel
// wrote for the row's other slots.
//
// A tile is T = 128 / G consecutive rows of one (batch, KV head); its columns
// are the (row, head) pairs, two 16-column groups of
// v_mfma_f32_16x16x32_bf16 per wavefront, four wavefronts per workgroup, so
// that a block is staged once for every head.  The blocks are known from the
// rows' positions alone (block 0 and the rows' previous and own ones), so the
// first block's loads leave with the tile's slot indices and queries, and the
// log-sums of the other slots arrive while the blocks are attended: a tile
// waits for memory about five times in a row where a union of its selected
// blocks, built first, made it eight.  Bound by those waits and the partials'
// bytes.  32 heads on 2 KV heads, 131072 rows, d = 64, K = 8:
// 1.58 -> 1.07 ms (1.33 with the partials in natural order, 8-byte loads).
#pragma once

#include <algorithm>

#include "attn_shared.h"

namespace pisa {

constexpr int kMergeBatch = 4;  // partials requested together

// KB: registers per lane and column group for the slots that are read ahead
// (a column's four lanes hold KB slots each).  TAIL: budgets above 4 KB, whose
// further slots are read in the merge; without it nothing of theirs is kept.
// The two staged blocks of 96 or more keys of 128 values leave room in the LDS
// for one workgroup per CU, which may then have all of its registers.
template <int D, int CT, int G, int KB, bool TAIL>
__global__ __launch_bounds__(kTileWaves * 64, CT * D > 256 ? 1 : 2) void attn_tile_kernel(
    AttnBlockArgs a, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ idx, uint16_t* __restrict__ o, float* __restrict__ lse,
    const uint16_t* __restrict__ part_o, const float* __restrict__ part_lse, int ltiles, int lcount) {
  constexpr int NW = kTileWaves, NG = kUnionGroups;
  constexpr int RW = 16 * NG / G, T = NW * RW;  // rows per wavefront, per tile
  constexpr int KS = D / 32;
  constexpr int C = CT * 32;
  constexpr int MT = C / 16;
  constexpr int MC = (D == 128 && MT > 4) ? 2 : (MT <= 6 ? MT : 4);  // 16-key tiles per softmax chunk
  static_assert(MT % MC == 0 && MC % 2 == 0, "blocks of 32, 64, 96 or 128 keys");
  constexpr int DT = D / 16;
  constexpr int NCH = D / 8;   // 16-byte chunks per key row
  constexpr int RPI = 64 / NCH;  // key rows per direct-to-LDS load instruction
  constexpr int BLK = C * D;   // elements of one staged K (or V) block
  static_assert(D == 64 || D == 128, "head dimension 64 or 128");
  // Two stages of [K block, V block], swizzled as in the union kernel.
  extern __shared__ __align__(16) uint16_t lds[];
  const uint16_t* stage = lds;
  const uint32_t stage_addr = lds_addr(lds);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int rend = min(a.Nq, a.row0 + a.nrows);
  const int first = a.N - a.Nq;
  // operand offsets of this lane (elements within a block)
  int koff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = col * D + ((4 * ks + grp) ^ union_swz<NCH>(col)) * 8;
  const int vr0 = 4 * grp + col / 4;
  int voff[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
    voff[dt] = vr0 * D + ((2 * dt + (col & 3) / 2) ^ union_swz<NCH>(vr0)) * 8 + (col & 1) * 4;

  // persistent workgroups over the tiles
  for (int li = blockIdx.x; li < lcount; li += gridDim.x) {
    const int bh = li / ltiles;
    const int tile = a.row0 / T + (li - bh * ltiles);
    // the union kernel's tiles (T divides its tile rows)
    if (a.skip && a.skip[static_cast<int64_t>(bh) * a.skip_tiles + ((tile * T) >> a.skip_shift)]) continue;
    const int b = bh / a.Hkv, h = bh - b * a.Hkv;
    const int r0 = tile * T;
    const int c_lo = (first + r0) / C, c_hi = (first + min(r0 + T, rend) - 1) / C;
    const int p0 = max(1, c_lo - 1);          // blocks 0 and p0 .. c_hi, ascending
    const int nu = 1 + max(0, c_hi - p0 + 1);
    auto block_of = [&](int u) { return u == 0 ? 0 : p0 + u - 1; };
    auto issue = [&](int blk, int buf) __attribute__((always_inline)) {
      const int rb = blk * C;
      const int last = min(C, a.N - rb) - 1;
      const uint16_t* kb = k + (static_cast<int64_t>(bh) * a.Nkv + rb) * D;
      const uint16_t* vb = v + (static_cast<int64_t>(bh) * a.Nkv + rb) * D;
      for (int ins = wave; ins < C / RPI; ins += NW) {
        const int row = ins * RPI + lane / NCH;
        const int64_t src = static_cast<int64_t>(min(row, last)) * D + ((lane % NCH) ^ union_swz<NCH>(row)) * 8;
        const uint32_t dk = stage_addr + static_cast<uint32_t>(buf * 2 * BLK + ins * RPI * D) * 2u;
        lds_dma16(kb + src, dk);
        lds_dma16(vb + src, dk + BLK * 2);
      }
    };

    // this lane's columns: group cg holds row j = wave * RW + (cg * 16 + col) / G,
    // head (cg * 16 + col) % G
    int rowc[NG], cr[NG], xs[NG][KB];
    bool vrow[NG];
    bf16x8a qb[NG][KS];
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) {
      const int cc = cg * 16 + col;
      const int row = r0 + wave * RW + cc / G;
      vrow[cg] = row < rend;
      rowc[cg] = vrow[cg] ? row : r0;
      cr[cg] = (first + rowc[cg]) / C;
      const int32_t* sl = idx + (static_cast<int64_t>(bh) * a.Nq + rowc[cg]) * a.K;
#pragma unroll
      for (int i = 0; i < KB; ++i) xs[cg][i] = 4 * i + grp < a.K ? sl[4 * i + grp] : -1;
      const uint16_t* qrow = q + ((static_cast<int64_t>(b) * a.H + h * G + cc % G) * a.Nq + rowc[cg]) * D + grp * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qb[cg][ks] = u4_as_bf16x8(*reinterpret_cast<const uint4*>(qrow + ks * 32));
    }
    __syncthreads();  // the previous tile's readers of the LDS are done
    issue(0, 0);

    // which of its three blocks each column's row selected (bits 0: block 0,
    // 1: previous, 2: own), and the log-sums of the other slots
    auto far = [&](int x, int c) { return x >= 0 && x < a.M1 && x != 0 && x != c && x != c - 1; };
    uint32_t sel[NG];
    float lsv[NG][KB];
    float m[NG], l[NG];
    f32x4a oacc[NG][DT];
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) {
      const int64_t pb = (static_cast<int64_t>(bh) * a.nrows + (rowc[cg] - a.row0)) * a.K;
      const int hq = (cg * 16 + col) % G;
      auto bits = [&](int x) {
        return (x == 0 ? 1u : 0u) | (x >= 0 && x == cr[cg] - 1 ? 2u : 0u) | (x == cr[cg] ? 4u : 0u);
      };
      uint32_t f = 0;
#pragma unroll
      for (int i = 0; i < KB; ++i) {
        f |= bits(xs[cg][i]);
        lsv[cg][i] = far(xs[cg][i], cr[cg]) ? part_lse[(pb + 4 * i + grp) * G + hq] : -INFINITY;
      }
      if constexpr (TAIL) {
        const int32_t* sl = idx + (static_cast<int64_t>(bh) * a.Nq + rowc[cg]) * a.K;
        for (int s0 = 4 * KB; s0 < a.K; s0 += 4) {
          const int x = sl[min(s0 + grp, a.K - 1)];  // (the last slot twice does no harm)
          f |= bits(x);
        }
      }
      f |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(f), 16));
      f |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(f), 32));
      sel[cg] = vrow[cg] ? f : 0u;
      m[cg] = -INFINITY;
      l[cg] = 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) oacc[cg][dt] = f32x4a{0.f, 0.f, 0.f, 0.f};
    }

    for (int u = 0; u < nu; ++u) {
      const int blk = block_of(u);
      const int rb = blk * C;
      const int nkeys = min(C, a.N - rb);
      __builtin_amdgcn_s_waitcnt(0);  // this wavefront's loads of block u have landed
      __syncthreads();                // every wavefront's have, and block u - 1 is done
      if (u + 1 < nu) issue(block_of(u + 1), (u + 1) & 1);
      const uint16_t* klds = stage + (u & 1) * 2 * BLK;
      const uint16_t* vlds = klds + BLK;
      int kmax[NG];
      bool any = false, full = true;
#pragma unroll
      for (int cg = 0; cg < NG; ++cg) {
        const bool in = ((sel[cg] & 1u) && blk == 0) || ((sel[cg] & 2u) && blk == cr[cg] - 1) ||
                        ((sel[cg] & 4u) && blk == cr[cg]);
        kmax[cg] = !in ? 0 : max(0, min(nkeys, first + rowc[cg] - rb + 1));  // keys the column sees
        any = any || kmax[cg] > 0;
        full = full && kmax[cg] == C;
      }
      if (__ballot(any) == 0) continue;  // no column of the wavefront sees a key of the block
      const bool wfull = __ballot(!full) == 0;
#pragma unroll
      for (int k0 = 0; k0 < MT; k0 += MC) {
        f32x4a sa[NG][MC];
#pragma unroll
        for (int mt = 0; mt < MC; ++mt) {
          f32x4a acc[NG];
#pragma unroll
          for (int cg = 0; cg < NG; ++cg) acc[cg] = f32x4a{0.f, 0.f, 0.f, 0.f};
          const uint16_t* arow = klds + (k0 + mt) * 16 * D;
          bf16x8a av[KS];
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) av[ks] = u4_as_bf16x8(*reinterpret_cast<const uint4*>(arow + koff[ks]));
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int cg = 0; cg < NG; ++cg)
              acc[cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ks], qb[cg][ks], acc[cg], 0, 0, 0);
#pragma unroll
          for (int cg = 0; cg < NG; ++cg) {
            if (!wfull) {
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int key = (k0 + mt) * 16 + 4 * grp + i;
                acc[cg][i] = key < kmax[cg] ? acc[cg][i] : -INFINITY;
              }
            }
            sa[cg][mt] = acc[cg];
          }
        }
        // online softmax with a lazily raised reference (see the union kernel)
        float lm[NG];
        bool over = false;
#pragma unroll
        for (int cg = 0; cg < NG; ++cg) {
          float bm = -INFINITY;
#pragma unroll
          for (int mt = 0; mt < MC; ++mt)
            bm = fmaxf(bm, fmaxf(fmaxf(sa[cg][mt][0], sa[cg][mt][1]), fmaxf(sa[cg][mt][2], sa[cg][mt][3])));
          lm[cg] = bm * a.qscale2;
          over = over || lm[cg] > m[cg] + kUnionSlack;
        }
        if (__ballot(over) != 0) {
#pragma unroll
          for (int cg = 0; cg < NG; ++cg) {
            float bm = lm[cg];
            bm = fmaxf(bm, __shfl_xor(bm, 16));
            bm = fmaxf(bm, __shfl_xor(bm, 32));
            const float nm = bm > m[cg] + kUnionSlack ? bm : m[cg];
            const float scl = nm != m[cg] ? fast_exp2(m[cg] - nm) : 1.f;
            l[cg] *= scl;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[cg][dt] *= scl;
            m[cg] = nm;
          }
        }
        float nms[NG];  // -m, or 0 while no key was seen (then every logit is -inf)
#pragma unroll
        for (int cg = 0; cg < NG; ++cg) nms[cg] = m[cg] == -INFINITY ? 0.f : -m[cg];
#pragma unroll
        for (int s2 = 0; s2 < MC / 2; ++s2) {
          bf16x8a pb[NG];
#pragma unroll
          for (int cg = 0; cg < NG; ++cg) {
            float pv[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              pv[i] = fast_exp2(fmaf(sa[cg][2 * s2][i], a.qscale2, nms[cg]));
              pv[4 + i] = fast_exp2(fmaf(sa[cg][2 * s2 + 1][i], a.qscale2, nms[cg]));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) l[cg] += pv[i];
            uint4 uu;
            uu.x = pack2_bf16(pv[0], pv[1]);
            uu.y = pack2_bf16(pv[2], pv[3]);
            uu.z = pack2_bf16(pv[4], pv[5]);
            uu.w = pack2_bf16(pv[6], pv[7]);
            pb[cg] = u4_as_bf16x8(uu);
          }
          const uint16_t* vr = vlds + (k0 + 2 * s2) * 16 * D;  // keys of tiles 2 s2, 2 s2 + 1 of the chunk
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            const v4s16 lo = lds_read_tr16x4(vr + voff[dt]);
            const v4s16 hi = lds_read_tr16x4(vr + 16 * D + voff[dt]);
            const bf16x8a avv = __builtin_bit_cast(bf16x8a, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int cg = 0; cg < NG; ++cg)
              oacc[cg][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(avv, pb[cg], oacc[cg][dt], 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int cg = 0; cg < NG; ++cg) {
      float ll = l[cg];
      ll += __shfl_xor(ll, 16);
      ll += __shfl_xor(ll, 32);
      float mm = m[cg];
      const int hq = (cg * 16 + col) % G;
      // Merge the partials (o normalised, log2-sum) of the row's other slots,
      // four slots at a time; slot 4 i + u's log-sum is in lane col + 16 u.
      const int64_t pb = (static_cast<int64_t>(bh) * a.nrows + (rowc[cg] - a.row0)) * a.K;
      const uint16_t* pcol = part_o + (pb * G + hq) * D + 8 * grp;  // slot s at pcol + s * G * D
      auto merge = [&](int s0, const float (&ls)[kMergeBatch]) __attribute__((always_inline)) {
        uint4 xo[kMergeBatch][DT / 2];  // of d tiles 2 j (x, y) and 2 j + 1 (z, w)
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
          const uint16_t* pr = pcol + static_cast<int64_t>(ls[u] != -INFINITY ? s0 + u : 0) * G * D;
#pragma unroll
          for (int j = 0; j < DT / 2; ++j) xo[u][j] = *reinterpret_cast<const uint4*>(pr + j * 32);
        }
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
          if (ls[u] == -INFINITY) continue;
          const float mn = fmaxf(mm, ls[u]);
          const float c0 = fast_exp2(mm - mn), c1 = fast_exp2(ls[u] - mn);
          ll = ll * c0 + c1;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            const uint32_t x0 = dt & 1 ? xo[u][dt / 2].z : xo[u][dt / 2].x;
            const uint32_t x1 = dt & 1 ? xo[u][dt / 2].w : xo[u][dt / 2].y;
            oacc[cg][dt][0] = oacc[cg][dt][0] * c0 + __uint_as_float(x0 << 16) * c1;
            oacc[cg][dt][1] = oacc[cg][dt][1] * c0 + __uint_as_float(x0 & 0xFFFF0000u) * c1;
            oacc[cg][dt][2] = oacc[cg][dt][2] * c0 + __uint_as_float(x1 << 16) * c1;
            oacc[cg][dt][3] = oacc[cg][dt][3] * c0 + __uint_as_float(x1 & 0xFFFF0000u) * c1;
          }
          mm = mn;
        }
      };
#pragma unroll
      for (int i = 0; i < KB; ++i) {
        if (4 * i >= a.K) break;
        float ls[kMergeBatch];
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) ls[u] = __shfl(lsv[cg][i], col | (u << 4));
        merge(4 * i, ls);
      }
      if constexpr (TAIL) {
        const int32_t* sl = idx + (static_cast<int64_t>(bh) * a.Nq + rowc[cg]) * a.K;
        for (int s0 = 4 * KB; s0 < a.K; s0 += kMergeBatch) {  // budgets above 4 KB
          float ls[kMergeBatch];
#pragma unroll
          for (int u = 0; u < kMergeBatch; ++u) {
            const int sx = s0 + u;
            const int x = sx < a.K ? sl[sx] : -1;
            ls[u] = far(x, cr[cg]) ? part_lse[(pb + sx) * G + hq] : -INFINITY;
          }
          merge(s0, ls);
        }
      }
      if (!vrow[cg]) continue;
      // oacc[cg][dt][i] = O[d = dt*16 + 4*grp + i][this column]
      const int64_t orow = (static_cast<int64_t>(b) * a.H + h * G + hq) * a.Nq + rowc[cg];
      const float inv = ll > 0.f ? 1.0f / ll : 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        uint2 w;
        w.x = pack2_bf16(oacc[cg][dt][0] * inv, oacc[cg][dt][1] * inv);
        w.y = pack2_bf16(oacc[cg][dt][2] * inv, oacc[cg][dt][3] * inv);
        *reinterpret_cast<uint2*>(o + orow * D + dt * 16 + 4 * grp) = w;
      }
      if (lse && grp == 0) lse[orow] = ll > 0.f ? (mm + fast_log2(ll)) * kLn2 : -INFINITY;
    }
  }
}

template <int D>
hipError_t launch_attn_tiles(const AttnBlockArgs& a, int BH, const uint16_t* q, const uint16_t* k, const uint16_t* v,
                             const int32_t* idx, uint16_t* o, float* lse, const uint16_t* part_o,
                             const float* part_lse, hipStream_t st) {
  const int T = attn_tile_rows(a.G);
  const int ltiles = (a.row0 + a.nrows + T - 1) / T - a.row0 / T;
  const int lcount = BH * ltiles;
  const size_t lds = static_cast<size_t>(4) * a.C * D * 2;
  auto go = [&](auto kern) {
    if (lds > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kTileWaves * 64, lds) != hipSuccess || per_cu < 1)
      per_cu = 1;
    const unsigned grid = static_cast<unsigned>(std::min(lcount, per_cu * kDeviceCUs));
    kern<<<grid, kTileWaves * 64, lds, st>>>(a, q, k, v, idx, o, lse, part_o, part_lse, ltiles, lcount);
  };
// Budgets from 17 to 32 read all of their slots ahead too (2 heads, 8192 rows,
// 30000 keys, d = 64, K = 32: 160 -> 148 us for the whole call; 16 heads on 4 KV
// heads, 4096 rows, d = 128, K = 32: 344 -> 336).
#define PISA_TILE_KB(CT, GG) \
  do { \
    if (a.K <= 8) go(attn_tile_kernel<D, CT, GG, 2, false>); \
    else if (a.K <= 16) go(attn_tile_kernel<D, CT, GG, 4, false>); \
    else if (a.K <= 32) go(attn_tile_kernel<D, CT, GG, 8, false>); \
    else go(attn_tile_kernel<D, CT, GG, 8, true>); \
  } while (0)
#define PISA_TILE_G(CT) \
  do { \
    if (a.G == 2) PISA_TILE_KB(CT, 2); \
    else if (a.G == 4) PISA_TILE_KB(CT, 4); \
    else if (a.G == 8) PISA_TILE_KB(CT, 8); \
    else PISA_TILE_KB(CT, 16); \
  } while (0)
  if (a.C == 32) PISA_TILE_G(1);
  else if (a.C == 64) PISA_TILE_G(2);
  else if (a.C == 96) PISA_TILE_G(3);
  else PISA_TILE_G(4);
#undef PISA_TILE_G
#undef PISA_TILE_KB
  return hipGetLastError();
}

}  // namespace pisa
