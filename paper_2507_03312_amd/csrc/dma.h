// Shared by the tiled GEMM kernels (half and float32): direct global-to-LDS
// copies and the order of the output tiles.  Internal; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mpx {

// Output tile of this workgroup.  Workgroups are dealt to the 8 XCDs
// round-robin (workgroup w runs on XCD w % 8); they are renumbered so that
// each XCD works through one contiguous range of tiles, and that range is
// walked in groups of 8 tile rows, column by column, so the tiles an XCD
// runs at the same time form a compact block: their A row panels and B
// column panels are shared through that XCD's L2 instead of each B panel
// being fetched again for every tile row.
template <int BM, int BN>
__device__ __forceinline__ void tile_origin_of(uint32_t tile, uint32_t ntiles, int64_t M, int64_t N,
                                               int64_t& m0, int64_t& n0) {
  // 32-bit index arithmetic (tile counts stay far below 2^32; a 64-bit
  // division is a long software sequence)
  constexpr uint32_t GM = 8;
  const uint32_t tiles_m = (uint32_t)((M + BM - 1) / BM), tiles_n = (uint32_t)((N + BN - 1) / BN);
  const uint32_t xcd = tile % 8, local = tile / 8;
  const uint32_t t = xcd * (ntiles / 8) + min(xcd, ntiles % 8) + local;
  const uint32_t first = (t / (GM * tiles_n)) * GM;
  const uint32_t gm = min(tiles_m - first, GM);
  const uint32_t r = t - first * tiles_n;
  m0 = (int64_t)(first + r % gm) * BM;
  n0 = (int64_t)(r / gm) * BN;
}

template <int BM, int BN>
__device__ __forceinline__ void tile_origin(int64_t M, int64_t N, int64_t& m0, int64_t& n0) {
  tile_origin_of<BM, BN>(blockIdx.x, gridDim.x, M, N, m0, n0);
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane from base + off (bytes) into LDS at lds + 16 * lane
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

}  // namespace mpx
