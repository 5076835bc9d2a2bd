// Shared by the block-centric attention kernels (attn.hip, attn_tiles.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"
#include "kernels.h"

namespace pisa {

typedef __bf16 bf16x8a __attribute__((ext_vector_type(8)));
typedef float f32x4a __attribute__((ext_vector_type(4)));

struct AttnBlockArgs {
  int H, Hkv, G, Nq, N, C, K, causal, M1;
  int row0, nrows;  // row chunk handled by this launch
  float qscale2;
  int Nkv;          // rows per (batch, KV head) in k and v
  // rows attended by the row-tile union kernel (flag per tile of
  // 1 << skip_shift rows); the block-centric kernels leave them alone
  const uint8_t* skip = nullptr;
  int skip_shift = 0, skip_tiles = 0;
  // partial rows for the row-tile kernel: within each 32 values the order is
  // [grp 0..3][d tile 0..1][4 values], so that a lane of its layout (values
  // 4 grp .. 4 grp + 3 of every 16-wide d tile) reads 16 bytes at a time
  bool tile_order = false;
};

__device__ __forceinline__ bool union_row(const AttnBlockArgs& a, int bh, int row) {
  return a.skip && a.skip[static_cast<int64_t>(bh) * a.skip_tiles + (row >> a.skip_shift)];
}

__device__ __forceinline__ bf16x8a u4_as_bf16x8(uint4 r) { return __builtin_bit_cast(bf16x8a, r); }

constexpr int kUnionGroups = 2;   // 16-column groups per wavefront of the row-tile kernels
constexpr float kUnionSlack = 8.f;  // log2 units the running maximum may lag behind
constexpr size_t kUnionMaxLds = 160 * 1024;  // LDS of one CU
constexpr int kDeviceCUs = 256;

// LDS byte address of a pointer into dynamic shared memory, made wave-uniform.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane(
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p)));
}
// 16 bytes per lane from global memory straight into LDS at lds + 16 * lane.
// Issued from inline assembly so that the compiler does not make the next
// LDS read wait for it (it cannot tell the two stages apart); the consumer
// waits for it with an explicit vmcnt wait and a barrier.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds) : "memory", "m0");
}
// Chunk-position swizzle of a staged key row (NCH 16-byte chunks per row):
// the 16 rows of a K operand read get 16 distinct bank positions.
template <int NCH>
__device__ __forceinline__ int union_swz(int r) {
  return NCH == 16 ? (r & 15) : ((r >> 1) & 7);
}
// The row-tile kernel for the forced blocks of G > 1 rows (attn_tiles.h):
// rows [a.row0, a.row0 + a.nrows) that the union kernel did not take.
constexpr int kTileWaves = 4;  // wavefronts per workgroup
inline int attn_tile_rows(int G) { return kTileWaves * kUnionGroups * 16 / G; }
template <int D>
hipError_t launch_attn_tiles(const AttnBlockArgs& a, int BH, const uint16_t* q, const uint16_t* k, const uint16_t* v,
                             const int32_t* idx, uint16_t* o, float* lse, const uint16_t* part_o,
                             const float* part_lse, hipStream_t st);

}  // namespace pisa
