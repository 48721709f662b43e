// The LDS tiles of the bf16 GEMMs, filled by direct global-to-LDS loads, and
// the order in which output tiles are handed out (shared with the fp32 GEMMs
// on fp16 pairs).
#pragma once

#include "lds_dma.h"

namespace hfk {
namespace {

// ------------------------------------------------------------ tile loading
// A ROWS x BK tile kept in LDS as [row][k]; the CH 16-byte chunks of a row
// are XOR-swizzled by (row / RPB) % CH, RPB being the number of rows that
// span the 64 banks.  Chunk position P of the tile (P = row * CH + pos, 64
// chunks per direct-load instruction) holds global chunk pos ^ swz(row).
template <int ROWS, int BK, int NW>
struct Tile16 {
  static constexpr int CH = BK / 8;
  static constexpr int RPB = 128 / BK;
  static constexpr int SIZE = ROWS * BK;             // 16-bit elements
  static constexpr int INSTR = ROWS * CH / 64 / NW;  // direct loads per wave
  static_assert(INSTR >= 1 && ROWS * CH % (64 * NW) == 0, "tile does not split over the waves");

  __device__ static __forceinline__ int swz(int row) { return (row / RPB) % CH; }
  // element offset, within an operand of leading dimension ld, of the chunk
  // that lane `lane` of wave `wave` fetches with its instruction j
  __device__ static __forceinline__ uint32_t src(int ld, int wave, int lane, int j) {
    const int P = (wave * INSTR + j) * 64 + lane;
    const int row = P / CH, pos = P % CH;
    return (uint32_t)row * (uint32_t)ld + 8u * (uint32_t)(pos ^ swz(row));
  }
  // LDS element offset of the 64 chunks written by instruction j of a wave
  __device__ static __forceinline__ int dst(int wave, int j) {
    return (wave * INSTR + j) * 512;
  }
  // operand of MFMA step q (k = 16 q .. 16 q + 15) for lane (row, h)
  template <class V>
  __device__ static __forceinline__ V frag(const uint16_t* __restrict__ s, int row,
                                           int h, int q) {
    const int c = 2 * q + h;
    return *(const V*)(s + row * BK + ((c ^ swz(row)) * 8));
  }
};

// ------------------------------------------------------------- tile order
// The tile (tn, tm) and split tz this workgroup computes.  Linear dispatch
// index L goes to XCD L % 8; when the grid is a multiple of 8, XCD x gets
// the x-th contiguous eighth of the logical order.  Within a split, the
// logical order walks groups of 8 tile rows, column by column.
__device__ __forceinline__ void tile_of(int& tn, int& tm, int& tz) {
  const int gx = gridDim.x, gy = gridDim.y;
  const int T = gx * gy * gridDim.z;
  const int L = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int Lg = (T % 8 == 0) ? (L % 8) * (T / 8) + L / 8 : L;
  tz = Lg / (gx * gy);
  const int r = Lg % (gx * gy);
  constexpr int G = 8;
  const int g = r / (G * gx);
  const int first = g * G;
  const int rows = min(G, gy - first);
  const int w = r - g * G * gx;
  tm = first + w % rows;
  tn = w / rows;
}

}  // namespace
}  // namespace hfk
