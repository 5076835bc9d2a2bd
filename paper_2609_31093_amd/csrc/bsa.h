// Shared by the flat-BSA kernels (bsa.hip, bsa_scan.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pisa {

struct BsaArgs {
  const void* q;
  const float* pyr;
  int32_t* idx;
  int H, Hkv, G, Nq, N, C, K, causal, M1;
  int64_t R;
  float qscale2;
};

// Marks, in the first index of rows 64 i or 64 i + 32, a 64-row tile that the
// scan kernels leave to the exact list kernel.
constexpr int kBsaRedo = -2;

// The scan kernels: every row's selection, or kBsaRedo marks.  phi, plo: the
// leaf means' bf16 hi and lo planes [BH][M1][D].
bool bsa_scan_path(int G, int K);
hipError_t launch_bsa_scan(const BsaArgs& a, int BH, int D, const uint16_t* phi, const uint16_t* plo, hipStream_t st);

}  // namespace pisa
