// Flat block selection (bf16, matrix cores): every eligible leaf mean scored,
// the Top-K taken without a running list.
//
// The blocks a query ranks fall into classes (one per accumulator register
// and lane that holds its scores).  The keepn-th best of the class bests, T,
// has keepn blocks at or above it, so the keepn best blocks all reach T; with
// 64 or 128 classes only one or two more than keepn blocks do.  A scan for
// the class bests costs one maximum per score, and what reaches T is a list
// short enough to be sorted in a lane's registers.
//
// bsa_scan_kernel (one head per KV head, K <= 16): two scans, the second
// collects what reaches T.  bsa_group_kernel (several heads): the scores cost
// an exponential per head, so its one ranking scan keeps each class's best
// three blocks instead, and collects from those.
//
// Rows that this does not decide (a list that runs over, NaN) are marked
// kBsaRedo in the output and ranked by the exact list kernel afterwards, a
// launch that otherwise reads one mark per 32 rows (6 us).  That costs more than
// the list kernel alone only where nearly every tile is marked: 32 heads on 8 KV
// heads, 131072 rows, d = 128, K = 16: 15.9 -> 6.0 ms without marks, 15.7 -> 8.3
// with the tiles of one KV head marked (all of its keys equal), 10.7 -> 17.3 with
// all of them.
//
// Measured (MI355X, the list kernel alone -> scan kernels and that launch):
// one head, 8 x 131072 rows, d = 128, K = 16: 5.04 -> 1.19 ms; 16 heads,
// 2 x 131072 rows, d = 64, K = 8: 7.31 -> 2.38 ms; 4 heads, 2 x 262144 rows,
// 128-key blocks, d = 128, K = 32: 15.6 -> 2.8 ms.
#include <algorithm>
#include <type_traits>

#include "bsa.h"
#include "common.h"
#include "kernels.h"
#include "launch_grid.h"
#include "sort32.h"
#include "sortnet.h"

namespace pisa {

namespace {

typedef __bf16 bf16x8s __attribute__((ext_vector_type(8)));
typedef float f32x16s __attribute__((ext_vector_type(16)));

__device__ __forceinline__ bf16x8s as_bf16x8(uint4 r) { return __builtin_bit_cast(bf16x8s, r); }

// The next float above x (finite x).
__device__ __forceinline__ float next_up(float x) {
  const int b = __float_as_int(x);
  return __int_as_float(b >= 0 ? b + 1 : (b == static_cast<int>(0x80000000u) ? 1 : b - 1));
}

// What one lane of the 32x32 tile knows of its query: its own leaf block c and
// the number of eligible blocks.
struct RowBlocks {
  int c, elig;
};

__device__ __forceinline__ RowBlocks row_blocks(const BsaArgs& a, int row) {
  RowBlocks r;
  r.c = (a.N - a.Nq + min(row, a.Nq - 1)) / a.C;
  r.elig = a.causal ? min(r.c + 1, a.M1) : a.M1;
  return r;
}

__device__ __forceinline__ bool rankable(const BsaArgs& a, const RowBlocks& r, int blk) {
  return (blk < r.elig) & !((a.causal != 0) & ((blk == 0) | (blk >= r.c - 1)));
}

// Block of accumulator register r in tile `ch`: v_mfma_f32_32x32x16 leaves row
// 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile in register r.
__device__ __forceinline__ int tile_block(int ch, int half, int r) { return ch * 32 + 8 * (r >> 2) + 4 * half + (r & 3); }

// The workgroup's row tile in a head_grid launch.
__device__ __forceinline__ int grid_tile() { return static_cast<int>(blockIdx.z * gridDim.y + blockIdx.y); }

// Writes one row's ascending selection: the best blocks (keepn of them, any
// order, in id[0..16)) and the forced ones.
__device__ __forceinline__ void emit_row16(const BsaArgs& a, int32_t* __restrict__ out, const RowBlocks& r, int keepn,
                                           int (&id)[16]) {
  if (r.elig <= a.K) {
#pragma unroll
    for (int i = 0; i < 16; ++i) id[i] = i < r.elig ? i : -1;
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i >= keepn) id[i] = 0x7fffffff;
      if (a.causal) {  // ranked rows have c >= K >= 3: three distinct forced blocks
        if (i == keepn) id[i] = 0;
        if (i == keepn + 1) id[i] = r.c - 1;
        if (i == keepn + 2) id[i] = r.c;
      }
    }
    oddeven_sort<16>([&](int i, int j) __attribute__((always_inline)) { cx_asc(id[i], id[j]); });
  }
  if ((a.K & 3) == 0) {
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
      if (i < a.K) *reinterpret_cast<int4*>(out + i) = make_int4(id[i], id[i + 1], id[i + 2], id[i + 3]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < a.K) out[i] = id[i];
    }
  }
}

}  // namespace

// ----------------------------------------------------------------------------
// One head per KV head, K <= 16.  A workgroup of four wavefronts takes 128 QT
// consecutive rows; each wavefront holds QT tiles of 32 queries as the B
// operand in registers and every wavefront scores every 32-block tile of
// leaf means, staged once per workgroup as bf16 hi and lo rows (double
// buffered, one barrier per tile, the next tile's loads in flight meanwhile).
// QT = 2 reads each staged operand for two products, which keeps the LDS at
// half its rate while the matrix cores are busy.  Bound by the products: at
// 8 x 131072 rows scan 1 takes 0.44 ms for 550 GFLOP (hi and lo), 1.25 PFLOP/s
// where a large library GEMM reaches 1.3 to 1.5; scan 2 as much again, and
// 0.23 ms for the collected blocks.
// ----------------------------------------------------------------------------
constexpr int kScanCap = 28;  // collected blocks per query: two workgroups fit a CU

template <int D, int QT>
__global__ __launch_bounds__(256, 2) void bsa_scan_kernel(BsaArgs a, const uint16_t* __restrict__ phi,
                                                          const uint16_t* __restrict__ plo) {
  constexpr int KS = D / 16;
  constexpr int ROW = D + 8;
  constexpr int PRE = 32 * (D / 8) / 256;  // 16-byte staging loads per thread, plane and tile
  constexpr int NQ = 128 * QT;
  __shared__ __align__(16) uint16_t stage[2][2][32 * ROW];
  __shared__ float ls[NQ * (kScanCap + 1)];
  __shared__ uint16_t li[NQ * (kScanCap + 2)];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  // longest rows first; a head's tiles on every BH-th workgroup
  const int ntx = (a.Nq + NQ - 1) / NQ;
  const int tx = grid_tile();
  if (tx >= ntx) return;
  const int bh = blockIdx.x;
  const int wg0 = (ntx - 1 - tx) * NQ;
  const int b = bh / a.Hkv, h = bh - b * a.Hkv;
  const int row0 = wg0 + wave * 32 * QT;
  const int first = a.N - a.Nq;
  const int nblk = a.causal ? min((first + min(wg0 + NQ, a.Nq) - 1) / a.C + 1, a.M1) : a.M1;
  const int ntile = (nblk + 31) / 32;
  const int keepn = a.causal ? a.K - 3 : a.K;  // of the rows that are ranked
  // the wavefront's rows: tiles past the last row's own block are not scored,
  // tiles before the first row's previous block need no masks
  const int c_lo = min(first + row0, a.N - 1) / a.C;
  const int c_hi = (first + min(row0 + 32 * QT, a.Nq) - 1) / a.C;
  const bool live = row0 < a.Nq && keepn > 0 && (a.causal ? min(c_hi + 1, a.M1) : a.M1) > a.K;
  RowBlocks rb[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) rb[t] = row_blocks(a, row0 + t * 32 + col);

  bf16x8s qB[QT][KS];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int row = min(row0 + t * 32 + col, a.Nq - 1);
    const uint16_t* qrow =
        static_cast<const uint16_t*>(a.q) + ((static_cast<int64_t>(b) * a.H + h) * a.Nq + row) * D + half * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qB[t][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qrow + ks * 16));
  }

  const uint16_t* hbase = phi + static_cast<int64_t>(bh) * a.M1 * D;
  const uint16_t* lbase = plo + static_cast<int64_t>(bh) * a.M1 * D;
  // (named values: as arrays they ended in scratch memory)
  static_assert(PRE == 1 || PRE == 2, "rows of 64 or 128");
  uint4 ph0, ph1, pl0, pl1;
  constexpr int RPK = 256 / (D / 8);  // rows per 256 threads
  const int er = threadIdx.x / (D / 8), ec = (threadIdx.x % (D / 8)) * 8;
  auto fetch = [&](int ch) __attribute__((always_inline)) {  // rows past the last block: masked
    const int64_t o0 = static_cast<int64_t>(min(ch * 32 + er, a.M1 - 1)) * D + ec;
    ph0 = *reinterpret_cast<const uint4*>(hbase + o0);
    pl0 = *reinterpret_cast<const uint4*>(lbase + o0);
    if constexpr (PRE == 2) {
      const int64_t o1 = static_cast<int64_t>(min(ch * 32 + er + RPK, a.M1 - 1)) * D + ec;
      ph1 = *reinterpret_cast<const uint4*>(hbase + o1);
      pl1 = *reinterpret_cast<const uint4*>(lbase + o1);
    }
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
    *reinterpret_cast<uint4*>(&stage[buf][0][er * ROW + ec]) = ph0;
    *reinterpret_cast<uint4*>(&stage[buf][1][er * ROW + ec]) = pl0;
    if constexpr (PRE == 2) {
      *reinterpret_cast<uint4*>(&stage[buf][0][(er + RPK) * ROW + ec]) = ph1;
      *reinterpret_cast<uint4*>(&stage[buf][1][(er + RPK) * ROW + ec]) = pl1;
    }
  };
  // raw scores of tile ch (in buffer buf); blocks that are not ranked: -inf
  auto score = [&](int ch, int buf, f32x16s (&acc)[QT]) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    }
    const uint16_t* sh = &stage[buf][0][col * ROW + half * 8];
    const uint16_t* sl = &stage[buf][1][col * ROW + half * 8];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8s ah = as_bf16x8(*reinterpret_cast<const uint4*>(sh + ks * 16));
      const bf16x8s al = as_bf16x8(*reinterpret_cast<const uint4*>(sl + ks * 16));
#pragma unroll
      for (int t = 0; t < QT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, qB[t][ks], acc[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < QT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, qB[t][ks], acc[t], 0, 0, 0);
    }
    const bool whole = a.causal ? (ch > 0 && ch * 32 + 32 < c_lo) : (ch * 32 + 32 <= a.M1);
    if (!whole) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = rankable(a, rb[t], tile_block(ch, half, r)) ? acc[t][r] : -INFINITY;
      }
    }
  };
  auto scan = [&](auto&& use) __attribute__((always_inline)) {
    __syncthreads();
    fetch(0);
    store(0);
    if (ntile > 1) fetch(1);
    __syncthreads();
    auto step = [&](int ch, auto par) __attribute__((always_inline)) {
      constexpr int P = decltype(par)::value;  // ch & 1
      if (ch + 1 < ntile) store(P ^ 1);  // its readers passed the last barrier
      if (ch + 2 < ntile) fetch(ch + 2);
      if (live && (!a.causal || ch * 32 <= c_hi)) {
        f32x16s acc[QT];
        score(ch, P, acc);
        use(ch, acc, par);
      }
      __syncthreads();
    };
    for (int ch = 0; ch < ntile; ch += 2) {
      step(ch, std::integral_constant<int, 0>{});
      if (ch + 1 < ntile) step(ch + 1, std::integral_constant<int, 1>{});
    }
  };

  // Scan 1: the best score of 64 classes per query (register, half, tile parity).
  float best[2][QT][16];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int t = 0; t < QT; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) best[s][t][r] = -INFINITY;
    }
  }
  const bool any_live = keepn > 0 && nblk > a.K;  // the same in the whole workgroup
  if (any_live) {
    scan([&](int, f32x16s (&acc)[QT], auto par) __attribute__((always_inline)) {
      constexpr int P = decltype(par)::value;
#pragma unroll
      for (int t = 0; t < QT; ++t) {
#pragma unroll
        for (int r = 0; r < 16; ++r) best[P][t][r] = sel_max(acc[t][r], best[P][t][r]);
      }
    });
  }
  // T: the keepn-th best class best (both halves of a query's lanes agree).
  float T[QT], lim[QT];
  int cnt[QT], tie[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    sort_desc<16>(best[0][t]);
    sort_desc<16>(best[1][t]);
    merge_top_desc<16>(best[0][t], best[1][t]);
    float other[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) other[r] = __shfl_xor(best[0][t][r], 32);
    merge_top_desc<16>(best[0][t], other);
    T[t] = pick_uniform<16>(best[0][t], max(keepn - 1, 0));
    lim[t] = T[t];
    cnt[t] = tie[t] = 0;
  }
  // Scan 2: what reaches T.  Scores above T fill a query's list from the
  // front, scores of exactly T from the back.  Equal scores go to the smaller
  // block, so once the list holds keepn blocks the limit moves up past T; and
  // where the two ends meet, the latest equal scores give way: at most keepn
  // minus the front's are needed, in the order they came but for the 8-block
  // runs of a tile, and kScanCap - 16 >= 8.
  if (any_live) {
    scan([&](int ch, f32x16s (&acc)[QT], auto) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const int base = (wave * 32 * QT + t * 32 + col);
        float* lsq = ls + base * (kScanCap + 1);
        uint16_t* liq = li + base * (kScanCap + 2);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float u = acc[t][r];
          const uint64_t m = __ballot(u >= lim[t]);
          if (m != 0) {
            const bool gt = u > T[t];
            const uint64_t mg = __ballot(gt), mt = m & ~mg;
            {
              const int p0 = __builtin_amdgcn_ubfe(static_cast<uint32_t>(mg), col, 1);
              const int p1 = __builtin_amdgcn_ubfe(static_cast<uint32_t>(mg >> 32), col, 1);
              const int at = cnt[t] + (half ? p0 : 0);
              cnt[t] += p0 + p1;
              if (gt && at < kScanCap) {
                lsq[at] = u;
                liq[at] = static_cast<uint16_t>(tile_block(ch, half, r));
              }
            }
            if (mt != 0) {
              const int p0 = __builtin_amdgcn_ubfe(static_cast<uint32_t>(mt), col, 1);
              const int p1 = __builtin_amdgcn_ubfe(static_cast<uint32_t>(mt >> 32), col, 1);
              const int at = kScanCap - 1 - (tie[t] + (half ? p0 : 0));
              tie[t] += p0 + p1;
              if ((half ? p1 : p0) && at >= cnt[t]) {
                lsq[at] = u;
                liq[at] = static_cast<uint16_t>(tile_block(ch, half, r));
              }
            }
          }
        }
        lim[t] = cnt[t] + tie[t] >= keepn ? next_up(T[t]) : T[t];
      }
    });
  }
  if (row0 >= a.Nq) return;
  // A lane per query: the list sorted by (score desc, block asc), the best
  // keepn and the forced blocks written in ascending order.
  wave_sync();
  const int t_of = QT == 2 ? half : 0;
  // (counts are the same in both halves of a wavefront)
  const int n_list = t_of == 0 ? cnt[0] : cnt[QT - 1];
  const int n_tie = t_of == 0 ? tie[0] : tie[QT - 1];
  const float T_list = t_of == 0 ? T[0] : T[QT - 1];
  const bool mine = (QT == 2 || half == 0) && row0 + t_of * 32 + col < a.Nq;
  const RowBlocks r_list = t_of == 0 ? rb[0] : rb[QT - 1];
  const bool ranked = r_list.elig > a.K;
  const bool redo = mine && ranked && keepn > 0 && !(n_list + n_tie >= keepn && n_list <= kScanCap && T_list > -INFINITY);
  const bool redo_any = __any(redo);
  int id[16];
  {
    const int base = wave * 32 * QT + t_of * 32 + col;
    const float* lsq = ls + base * (kScanCap + 1);
    const uint16_t* liq = li + base * (kScanCap + 2);
    uint64_t key[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      key[j] = ~static_cast<uint64_t>(0);
      if (j < kScanCap) {
        const uint64_t e = (static_cast<uint64_t>(desc_bits(lsq[j])) << 32) | liq[j];
        key[j] = ((j < n_list) | (j >= kScanCap - n_tie)) ? e : key[j];
      }
    }
    oddeven_sort<32>([&](int i, int j) __attribute__((always_inline)) { cx_asc(key[i], key[j]); });
#pragma unroll
    for (int i = 0; i < 16; ++i) id[i] = static_cast<int>(static_cast<uint32_t>(key[i]));
  }
  if (mine) {
    const int row = row0 + t_of * 32 + col;
    if (redo_any && (row & 31) == 0) {
      a.idx[(static_cast<int64_t>(bh) * a.Nq + row) * a.K] = kBsaRedo;
    } else {
      emit_row16(a, a.idx + (static_cast<int64_t>(bh) * a.Nq + row) * a.K, r_list, keepn, id);
    }
  }
}

// ----------------------------------------------------------------------------
// Several heads per KV head (scores: the heads' softmax probabilities over the
// eligible non-forced blocks, summed), K <= KP.  A workgroup of four wavefronts
// takes 32 rows, whose queries (every head) sit in LDS; wavefront w scores the
// 32-block tiles w, w + 4, ..., each tile's hi and lo means read once from L2
// into registers and used for every head, so the scans have no barriers.
// Bound by the exponentials (one per head and score and scan, a quarter of
// the vector rate) beside the products.
// ----------------------------------------------------------------------------
template <int KP>
constexpr int kGroupCap = KP == 16 ? 40 : 64;  // collected blocks per query

// LDS: the queries and their normalisers, then what the phases after each
// other need: the normalisers' merge, the class bests, the lists.
template <int KP>
size_t group_lds(int G, int D) {
  const size_t merge = 4 * 4 * 32 * 2 * 4, bests = static_cast<size_t>(4) * KP * 32 * 4;
  const size_t lists = 32 * (kGroupCap<KP> + 1) * 8 + 32 * 4 + 256 * 4;
  return static_cast<size_t>(G) * 32 * (D * 2 + 4) + std::max({merge, bests, lists});
}

template <int D, int GM, int KP>
__global__ __launch_bounds__(256, 2) void bsa_group_kernel(BsaArgs a, const uint16_t* __restrict__ phi,
                                                           const uint16_t* __restrict__ plo) {
  constexpr int KS = D / 16;
  constexpr int CH = D / 8;  // 16-byte chunks of a row
  extern __shared__ __align__(16) uint16_t lds[];
  constexpr int CAP = kGroupCap<KP>;
  uint16_t* sq = lds;                                               // [G][32][D], chunks swizzled
  float* lnorm = reinterpret_cast<float*>(lds + a.G * 32 * D);      // [G][32]
  float* red = lnorm + a.G * 32;                                    // [4 waves][4 heads][32][2]
  float* tl = red;                                                  // [4 waves][KP][32]
  float* ls = red;                                                  // [32][CAP + 1]
  int* li = reinterpret_cast<int*>(ls + 32 * (CAP + 1));            // [32][CAP + 1]
  int* cnt = li + 32 * (CAP + 1);                                   // [32]
  int* outl = cnt + 32;                                             // [4 waves][2][32]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int ntx = (a.Nq + 31) / 32;
  const int tx = grid_tile();
  if (tx >= ntx) return;
  const int bh = blockIdx.x;
  const int row0 = (ntx - 1 - tx) * 32;
  const int b = bh / a.Hkv, h = bh - b * a.Hkv;
  const int first = a.N - a.Nq;
  const int c_lo = (first + row0) / a.C;
  const int nblk = a.causal ? min((first + min(row0 + 32, a.Nq) - 1) / a.C + 1, a.M1) : a.M1;
  const int ntile = (nblk + 31) / 32;
  const int keepn = a.causal ? a.K - 3 : a.K;
  const bool live = keepn > 0 && nblk > a.K;  // some row is ranked
  const RowBlocks rb = row_blocks(a, row0 + col);
  const float sc = a.qscale2;
  // chunk c8 of row r sits at place c8 ^ swz(r): 16-byte reads of 8 consecutive rows meet 8 bank groups
  auto swz = [&](int r) __attribute__((always_inline)) { return D == 128 ? (r & 15) : ((r >> 1) & 7); };

  const uint16_t* hbase = phi + static_cast<int64_t>(bh) * a.M1 * D + half * 8;
  const uint16_t* lbase = plo + static_cast<int64_t>(bh) * a.M1 * D + half * 8;
  bf16x8s ah[KS], al[KS];
  auto fetch = [&](int ch) __attribute__((always_inline)) {
    const int64_t off = static_cast<int64_t>(min(ch * 32 + col, a.M1 - 1)) * D;  // past the last block: masked
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      ah[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(hbase + off + ks * 16));
      al[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(lbase + off + ks * 16));
    }
  };
  auto score = [&](int hh, f32x16s& acc) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const uint16_t* qr = sq + (hh * 32 + col) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8s qb = as_bf16x8(*reinterpret_cast<const uint4*>(qr + (((2 * ks + half) ^ swz(col)) * 8)));
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[ks], qb, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[ks], qb, acc, 0, 0, 0);
    }
  };
  auto whole = [&](int ch) __attribute__((always_inline)) {
    return a.causal ? (ch > 0 && ch * 32 + 32 < c_lo) : (ch * 32 + 32 <= a.M1);
  };
  // the wavefront's tiles: use(tile, summed probabilities; blocks that are not ranked: -inf)
  auto scan_scores = [&](auto&& use) __attribute__((always_inline)) {
    for (int ch = wave; ch < ntile; ch += 4) {
      fetch(ch);
      float u[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
      for (int hh = 0; hh < GM; ++hh) {
        if (hh < a.G) {
          f32x16s acc;
          score(hh, acc);
          const float ln = lnorm[hh * 32 + col];
#pragma unroll
          for (int r = 0; r < 16; ++r) u[r] += fast_exp2(fmaf(acc[r], sc, -ln));
        }
      }
      if (!whole(ch)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) u[r] = rankable(a, rb, tile_block(ch, half, r)) ? u[r] : -INFINITY;
      }
      use(ch, u);
    }
  };

  float s1[16], s2[16], s3[16];
  int i1[16], i2[16], i3[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    s1[r] = s2[r] = s3[r] = -INFINITY;
    i1[r] = i2[r] = i3[r] = 0;
  }
  if (live) {
    for (int e = threadIdx.x; e < a.G * 32 * CH; e += 256) {
      const int hh = e / (32 * CH), rem = e % (32 * CH);
      const int r = rem / CH, c8 = rem % CH;
      const int row = min(row0 + r, a.Nq - 1);
      const uint4 x = *reinterpret_cast<const uint4*>(
          static_cast<const uint16_t*>(a.q) + ((static_cast<int64_t>(b) * a.H + h * a.G + hh) * a.Nq + row) * D + c8 * 8);
      *reinterpret_cast<uint4*>(sq + (hh * 32 + r) * D + ((c8 ^ swz(r)) * 8)) = x;
    }
    __syncthreads();
    // Scan 1: each head's normaliser.
    float hm[GM], hs[GM];
#pragma unroll
    for (int hh = 0; hh < GM; ++hh) {
      hm[hh] = -INFINITY;
      hs[hh] = 0.f;
    }
    for (int ch = wave; ch < ntile; ch += 4) {
      fetch(ch);
      const bool w = whole(ch);
#pragma unroll
      for (int hh = 0; hh < GM; ++hh) {
        if (hh < a.G) {
          f32x16s acc;
          score(hh, acc);
          if (!w) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = rankable(a, rb, tile_block(ch, half, r)) ? acc[r] : -INFINITY;
          }
          float m = hm[hh];
#pragma unroll
          for (int r = 0; r < 16; ++r) m = sel_max(acc[r], m);
          const float ref = m == -INFINITY ? 0.f : m * sc;
          float s = hs[hh] * fast_exp2(fmaf(hm[hh], sc, -ref));
#pragma unroll
          for (int r = 0; r < 16; ++r) s += fast_exp2(fmaf(acc[r], sc, -ref));
          hm[hh] = m;
          hs[hh] = s;
        }
      }
    }
    // merged over the two halves, then over the wavefronts, four heads at a time
#pragma unroll
    for (int h0 = 0; h0 < GM; h0 += 4) {
      if (h0 < a.G) {
#pragma unroll
        for (int hh = h0; hh < h0 + 4 && hh < GM; ++hh) {
          const float m2 = __shfl_xor(hm[hh], 32), q2 = __shfl_xor(hs[hh], 32);
          const float m = sel_max(m2, hm[hh]);
          const float ref = m == -INFINITY ? 0.f : m * sc;
          const float s = hs[hh] * fast_exp2(fmaf(hm[hh], sc, -ref)) + q2 * fast_exp2(fmaf(m2, sc, -ref));
          if (half == 0) {
            red[((wave * 4 + hh - h0) * 32 + col) * 2 + 0] = m;
            red[((wave * 4 + hh - h0) * 32 + col) * 2 + 1] = s;
          }
        }
        __syncthreads();
        if (threadIdx.x < 128 && h0 + static_cast<int>(threadIdx.x >> 5) < a.G) {
          const int hq = threadIdx.x >> 5;
          float m = -INFINITY;
          for (int w = 0; w < 4; ++w) m = sel_max(red[((w * 4 + hq) * 32 + col) * 2], m);
          const float ref = m == -INFINITY ? 0.f : m * sc;
          float s = 0.f;
          for (int w = 0; w < 4; ++w)
            s += red[((w * 4 + hq) * 32 + col) * 2 + 1] * fast_exp2(fmaf(red[((w * 4 + hq) * 32 + col) * 2], sc, -ref));
          lnorm[(h0 + hq) * 32 + col] = ref + fast_log2(s);
        }
        __syncthreads();
      }
    }
    // Scan 2: the summed probabilities, each class's best three blocks.
    scan_scores([&](int ch, float (&u)[16]) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool g1 = u[r] > s1[r], g2 = u[r] > s2[r], g3 = u[r] > s3[r];
        i3[r] = g2 ? i2[r] : (g3 ? ch : i3[r]);
        s3[r] = g2 ? s2[r] : (g3 ? u[r] : s3[r]);
        i2[r] = g1 ? i1[r] : (g2 ? ch : i2[r]);
        s2[r] = g1 ? s1[r] : (g2 ? u[r] : s2[r]);
        i1[r] = g1 ? ch : i1[r];
        s1[r] = g1 ? u[r] : s1[r];
      }
    });
  }
  __syncthreads();
  float T = INFINITY;
  if (live) {
    float v[KP];
    {
      float x[16], y[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = s1[r];
      sort_desc<16>(x);
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = __shfl_xor(x[r], 32);
      if constexpr (KP == 16) {
        merge_top_desc<16>(x, y);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = x[r];
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          v[r] = x[r];
          v[KP - 1 - r] = y[r];
        }
        bitonic_merge_desc<KP>(v);
      }
    }
    if (half == 0) {
#pragma unroll
      for (int r = 0; r < KP; ++r) tl[(wave * KP + r) * 32 + col] = v[r];
    }
    __syncthreads();
    for (int w = 1; w < 4; ++w) {
      const int o = (wave + w) & 3;
      float y[KP];
#pragma unroll
      for (int r = 0; r < KP; ++r) y[r] = tl[(o * KP + r) * 32 + col];
      merge_top_desc<KP>(v, y);
    }
    T = pick_uniform<KP>(v, keepn - 1);
  }
  __syncthreads();
  if (threadIdx.x < 32) cnt[threadIdx.x] = 0;
  __syncthreads();
  const bool ranked = live && rb.elig > a.K;
  if (ranked) {
    int n = 0;
    bool over = !(T > -INFINITY);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      n += (s1[r] >= T ? 1 : 0) + (s2[r] >= T ? 1 : 0) + (s3[r] >= T ? 1 : 0);
    }
    over |= n > CAP;
    int at = over ? atomicAdd(&cnt[col], 0x10000) : (n > 0 ? atomicAdd(&cnt[col], n) : 0);
    if (!over && n > 0 && at + n <= CAP) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        auto put = [&](float s, int tile) __attribute__((always_inline)) {
          if (s >= T) {
            ls[col * (CAP + 1) + at] = s;
            li[col * (CAP + 1) + at] = tile_block(tile, half, r);
            ++at;
          }
        };
        put(s1[r], i1[r]);
        put(s2[r], i2[r]);
        put(s3[r], i3[r]);
      }
    }
  }
  // A class whose third block reaches T may hold more that do: its wavefront
  // scores its tiles again for those, unless the list ran over already.
  __syncthreads();
  uint32_t more = 0;
  if (ranked && T > -INFINITY && cnt[col] <= CAP) {
#pragma unroll
    for (int r = 0; r < 16; ++r) more |= s3[r] >= T ? 1u << r : 0u;
  }
  if (__any(more != 0)) {
    scan_scores([&](int ch, float (&u)[16]) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if ((more >> r & 1) && u[r] >= T && ch != i1[r] && ch != i2[r] && ch != i3[r]) {
          const int at = atomicAdd(&cnt[col], 1);
          if (at < CAP) {
            ls[col * (CAP + 1) + at] = u[r];
            li[col * (CAP + 1) + at] = tile_block(ch, half, r);
          }
        }
      }
    });
  }
  __syncthreads();
  // Two queries per wavefront and step (four steps): ranked, then written.
  const bool redo = ranked && row0 + col < a.Nq && keepn > 0 && (cnt[col] < keepn || cnt[col] > CAP);
  const bool redo_any = __any(redo);
  for (int step = 0; step < 4; ++step) {
    const int qw = wave * 8 + step * 2 + half;  // this half's query
    const int row = row0 + qw;
    const RowBlocks r = row_blocks(a, row);
    const bool rk = r.elig > a.K;
    const int n = rk && live ? min(cnt[qw], CAP) : 0;
    float key = col < n ? ls[qw * (CAP + 1) + col] : -INFINITY;
    int blk = col < n ? li[qw * (CAP + 1) + col] : 0x7fffffff;
    sort32(key, blk, col);
    if (__any(n > 32)) {  // the other half of a longer list: sorted the other way round, the better of each pair kept
      float k2 = 32 + col < n ? ls[qw * (CAP + 1) + 32 + col] : -INFINITY;
      int b2 = 32 + col < n ? li[qw * (CAP + 1) + 32 + col] : 0x7fffffff;
      sort32(k2, b2, col);
      k2 = __shfl_xor(k2, 31);
      b2 = __shfl_xor(b2, 31);
      const bool take = (k2 > key) | ((k2 == key) & (b2 < blk));
      key = take ? k2 : key;
      blk = take ? b2 : blk;
      sort32(key, blk, col);
    }
    int x = 0x7fffffff;
    if (rk) {
      if (col < keepn) x = blk;
      if (a.causal) {
        if (col == keepn) x = 0;
        if (col == keepn + 1) x = r.c - 1;
        if (col == keepn + 2) x = r.c;
      }
    }
    int* sx = outl + (wave * 2 + half) * 32;
    sx[col] = x;
    wave_sync();
    int rank = 0;
    for (int y = 0; y < a.K; ++y) rank += sx[y] < x ? 1 : 0;
    wave_sync();
    if (row < a.Nq && col < a.K) {
      int32_t* out = a.idx + (static_cast<int64_t>(bh) * a.Nq + row) * a.K;
      if (!rk) {
        out[col] = col < r.elig ? col : -1;
      } else if (!redo_any) {
        out[rank] = x;
      }
    }
  }
  if (redo_any && threadIdx.x == 0) a.idx[(static_cast<int64_t>(bh) * a.Nq + row0) * a.K] = kBsaRedo;
}

// One head: a lane sorts 16 results; several heads: 32-lane sorts.
bool bsa_scan_path(int G, int K) {
  return G == 1 ? K <= 16 : K <= 32;
}

static dim3 tile_grid(int tiles, int BH) {
  const HeadGrid g = head_grid(tiles, BH);
  return dim3(g.x, g.y, g.z);
}

hipError_t launch_bsa_scan(const BsaArgs& a, int BH, int D, const uint16_t* phi, const uint16_t* plo, hipStream_t st) {
  if (a.G == 1) {
    // 256 rows per workgroup once that gives every CU its two workgroups, 128
    // below (8 heads: 25 vs 36 us at 4097 rows, 63 either way at 16384, 153
    // vs 136 at 32768)
    const bool wide = static_cast<int64_t>((a.Nq + 255) / 256) * BH >= 512;
    const dim3 grid = tile_grid((a.Nq + (wide ? 255 : 127)) / (wide ? 256 : 128), BH);
    if (D == 128) {
      if (wide)
        bsa_scan_kernel<128, 2><<<grid, 256, 0, st>>>(a, phi, plo);
      else
        bsa_scan_kernel<128, 1><<<grid, 256, 0, st>>>(a, phi, plo);
    } else {
      if (wide)
        bsa_scan_kernel<64, 2><<<grid, 256, 0, st>>>(a, phi, plo);
      else
        bsa_scan_kernel<64, 1><<<grid, 256, 0, st>>>(a, phi, plo);
    }
    return hipGetLastError();
  }
  const int KP = a.K <= 16 ? 16 : 32;
  const size_t lds = KP == 16 ? group_lds<16>(a.G, D) : group_lds<32>(a.G, D);
  const dim3 grid = tile_grid((a.Nq + 31) / 32, BH);
  auto go = [&](auto kern) {
    if (lds > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    kern<<<grid, 256, lds, st>>>(a, phi, plo);
  };
  if (D == 128) {
    if (a.G <= 4)
      KP == 16 ? go(bsa_group_kernel<128, 4, 16>) : go(bsa_group_kernel<128, 4, 32>);
    else
      KP == 16 ? go(bsa_group_kernel<128, 16, 16>) : go(bsa_group_kernel<128, 16, 32>);
  } else {
    if (a.G <= 4)
      KP == 16 ? go(bsa_group_kernel<64, 4, 16>) : go(bsa_group_kernel<64, 4, 32>);
    else
      KP == 16 ? go(bsa_group_kernel<64, 16, 16>) : go(bsa_group_kernel<64, 16, 32>);
  }
  return hipGetLastError();
}

}  // namespace pisa
