// Device helper shared by the kernel sources.
#pragma once
#include <hip/hip_runtime.h>

// Workgroups are handed to the 8 XCDs of the chip round-robin (workgroup b on XCD b % 8), and each
// XCD has its own L2.  xcd_block() renumbers the grid so that XCD x works through one contiguous
// range of blocks: element tiles that are neighbours in y (one mesh row apart) are then processed
// by the same XCD shortly after each other, and the face data they share hit in that XCD's L2.
// It is a bijection of [0, gridDim.x), so results never depend on the dispatch order.
__device__ __forceinline__ long xcd_block() {
  const long nb = gridDim.x, b = blockIdx.x;
  const long q = nb >> 3, r = nb & 7, x = b & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

// Tile (tx, ty) of block b of an ntx x nty grid of tiles: the blocks walk strips of TILE_STRIP tile columns,
// row by row, so that a tile's lower neighbour ran TILE_STRIP blocks before it and its border is still in the
// L2 (at 1024 x 1024 elements, N = 4, a whole row of 5 x 4 tiles is 4 MB, an L2's size).
constexpr int TILE_STRIP = 16;
__device__ __forceinline__ void tile_of(int b, int ntx, int nty, int& tx, int& ty) {
  const int s = b / (TILE_STRIP * nty), r = b - s * (TILE_STRIP * nty);
  const int w = ntx - s * TILE_STRIP < TILE_STRIP ? ntx - s * TILE_STRIP : TILE_STRIP;
  ty = r / w;
  tx = s * TILE_STRIP + (r - ty * w);
}

// Run-table launches: one launch covers several independent runs, whose blocks are consecutive
// ranges; boff[r] is the first block of run r and boff[nr] the grid size.  Returns the run of the
// calling block (the same for all its threads) by bisection.  The result is declared wave-uniform
// (readfirstlane), so that the run's argument struct is fetched with scalar loads into scalar
// registers; a compiler that did not find that by itself would keep its pointers and constants in vector
// registers of every lane (ROCm 7.2's finds it for the kernels here: their registers are the same without).
__device__ __forceinline__ int rt_run(const int* __restrict__ boff, int nr) {
  const int b = (int)blockIdx.x;
  int lo = 0, hi = nr;  // boff[lo] <= b < boff[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (boff[mid] <= b) lo = mid;
    else hi = mid;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Run-table argument structs hold their array pointers as plain (generic) pointers.  Read through
// gl() they are loaded as global-memory pointers, so that a kernel body inlined into a run-table
// kernel addresses its arrays with global rather than flat memory instructions, as it does with
// kernel arguments (at N = 4, k = 3 with flat ones the J reconstruction needs 112 VGPRs instead of 80, 4 waves per SIMD
// instead of 6, the line-task map 157 instead of 124, 3 instead of 4).  Fields that are not pointers pass through
// unchanged.
#ifndef MHD_GLOBAL_AS
#define MHD_GLOBAL_AS __attribute__((address_space(1)))
#endif
template <class T>
__device__ __forceinline__ T* gl(T* const& field) {
  typedef MHD_GLOBAL_AS T* gptr;
  return (T*)(*reinterpret_cast<const gptr*>(&field));
}
template <class T>
__device__ __forceinline__ const T& gl(const T& field) {
  return field;
}

// The instruction scheduler moves nothing across this point.  Unrolled blocks of independent work
// otherwise get interleaved until their operands no longer fit the registers.
#if __has_builtin(__builtin_amdgcn_sched_barrier)
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#else
#define SCHED_FENCE()
#endif
