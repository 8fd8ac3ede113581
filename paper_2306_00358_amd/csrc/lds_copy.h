// Copies of K-contiguous operand slabs into LDS, shared by the FP64 tile kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace hotrg {

typedef __attribute__((address_space(3))) void lds_void;

// Chunk position of a row's 16-byte chunks: c ^ swz(r) puts the 16 rows that one
// 16-lane group of an MFMA fragment reads into 16 different bank groups.
template <int BK>
__device__ __forceinline__ int swz(int r) {
  // rows per 256-byte LDS line: BK=32 -> 1, BK=16 -> 2
  constexpr int L = 256 / (BK * 8);
  constexpr int CH = BK / 2;
  return (r / L) % CH;
}

// Copy rows [0, R) x K-slab of a K-contiguous operand into swizzled LDS.
// One wave instruction moves 1 KB = 1024 / (BK*8) rows.
template <int R, int BK, int NW>
__device__ __forceinline__ void load_kcontig(const double* __restrict__ G, long long ld, int row0,
                                             int rows_valid, int k0, char* lds, int wave,
                                             int lane) {
  constexpr int RPI = 1024 / (BK * 8);
  constexpr int CH = BK / 2;
  constexpr int INSTS = R / RPI;
  static_assert(INSTS % NW == 0, "instructions must split over waves");
#pragma unroll
  for (int q = 0; q < INSTS / NW; ++q) {
    const int inst = wave + q * NW;
    const int r = inst * RPI + lane / CH;
    const int c = lane % CH;
    int gr = row0 + r;
    gr = gr < rows_valid ? gr : rows_valid - 1;
    const double* src = G + (long long)gr * ld + k0 + 2 * (c ^ swz<BK>(r));
    __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)(lds + inst * 1024), 16, 0, 0);
  }
}

// The same for rows aligned to 8 bytes only: 4 bytes a lane, two rows of BK = 16 an
// instruction, into the same places.
template <int R>
__device__ __forceinline__ void load_kcontig_any(const double* __restrict__ G, long long ld,
                                                 int row0, int rows_valid, int k0, char* lds,
                                                 int lane) {
#pragma unroll
  for (int q = 0; q < R / 2; ++q) {
    const int r = 2 * q + (lane >> 5), p = lane & 31;
    int gr = row0 + r;
    gr = gr < rows_valid ? gr : rows_valid - 1;
    const int* src = (const int*)(G + (long long)gr * ld + k0) + 4 * ((p >> 2) ^ swz<16>(r)) + (p & 3);
    __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)(lds + q * 256), 4, 0, 0);
  }
}

}  // namespace hotrg
