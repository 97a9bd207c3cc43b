// terra_tile.h - LDS tiles of 64 window tokens for the 16-bit attention
// kernels: rows of HD channels, unpadded, their 16-byte chunks permuted by
// an XOR of the row index, filled by direct-to-LDS loads whose row addresses
// come from a per-window table.
#pragma once

#include "terra_common.h"

namespace terra {

// Chunk permutation of row r (HD / 8 chunks a row).  Two reads set it:
// * straight operands (16 consecutive rows at one chunk) cover all banks
//   because the 16 rows take 16 different (bank half, chunk) places;
// * transposed operands (4 consecutive rows x 64 bytes) cover the 256 bytes
//   of the banks because the two low row bits select the 64-byte span.
template <int HD>
__device__ inline int tile_swz(int r) {
  if (HD == 32) return (r >> 2) & 3;
  if (HD == 64) return ((r >> 1) & 1) * 4 + ((r >> 2) & 1) * 2 + ((r >> 3) & 1);
  return ((r & 3) << 2) | ((r >> 2) & 3);
}
template <int HD>
__device__ inline int tile_off(int row, int ch) {   // element offset of (row, channel)
  return row * HD + 8 * ((ch >> 3) ^ tile_swz<HD>(row)) + (ch & 7);
}

// Addresses (bytes inside a tile) of a lane's operand reads.  The chunk
// permutation is an XOR below the row bits, so one lane constant serves
// every chunk:
// * straight operand, chunk c of rows r0 + l % 32 (lane l receives channels
//   16c + 8 (l / 32) .. + 7): (row ^ 32c) + r0 rows;
// * transposed operand of channel block eb, rows 32 rb + 16 c2 .. + 15 in
//   the slot order of the 32x32 result registers (see lds_tr_op), its second
//   eight rows (hi): (tr ^ 64 eb ^ kHiXor hi) + (32 rb + 16 c2 + 8 hi) rows.
template <int HD>
struct TileAddr {
  static constexpr uint32_t kRow = HD * 2;
  static constexpr uint32_t kHiXor = HD == 64 ? 16 : 32;
  uint32_t row, tr;
  __device__ explicit TileAddr(int lane) {
    const int col = lane & 31, G = lane >> 4, x = (lane >> 2) & 3, m = lane & 3;
    row = (uint32_t)tile_off<HD>(col, 8 * (lane >> 5)) * 2;
    tr = (uint32_t)tile_off<HD>(4 * (G >> 1) + x, 16 * (G & 1) + 4 * m) * 2;
  }
  // Keeps the compiler from holding every XORed address in registers.
  __device__ void opaque() { asm volatile("" : "+v"(row), "+v"(tr)); }
};
template <typename T, int HD>
__device__ inline typename Operand<T>::type tile_row_op(const char* t, const TileAddr<HD>& a, int r0, int c) {
  return *reinterpret_cast<const typename Operand<T>::type*>(t + (a.row ^ (32u * c)) + r0 * a.kRow);
}
template <typename T, int HD>
__device__ inline typename Operand<T>::type tile_tr_op(const char* t, const TileAddr<HD>& a, int rb, int c2, int eb) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) v4s lds_v4s;
  const uint32_t r = (32u * rb + 16u * c2) * a.kRow;
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(t + (a.tr ^ (64u * eb)) + r));
  const v4s hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(t + (a.tr ^ (64u * eb) ^ a.kHiXor) + r + 8 * a.kRow));
  const v8s o = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(typename Operand<T>::type, o);
}

// Pairs of tile buffers of a workgroup: two, one being filled while the other
// is read; one for windows of a single tile, whose LDS plan then fits a CU
// four times at 128 channels instead of twice (16-token windows, 2 x 128 x 256
// tokens of 3 heads: forward 120 -> 68 us, backward 395 -> 328; 64 tokens,
// 256 x 540 of 8 heads, a step 1133 -> 1020).
__device__ __host__ inline int tile_pairs(int nP) { return nP > 64 ? 2 : 1; }

// Row address of a tile row past the window's n tokens: one token past the
// image (ibytes, below 2^32), where the load reads zeros.  The row's weights
// are zero, and zero times a token's infinity would not be.  An image that
// ends within two rows of 2^32 bytes has no room for that address and takes a
// row of its last token.
template <int HD>
__device__ inline uint32_t tile_pad_row(uint32_t ibytes) { return min(ibytes, 0u - 4u * HD); }

// Moves rows r0 .. r0 + 63 of one tensor into a tile: NT threads, each
// 16-byte chunk written by the load itself (DIRECT) or, for tensors that do
// not start at a multiple of 16 bytes, loaded into registers and stored: what
// a direct-to-LDS load does with an address that is not a multiple of its
// element size is not documented.  tokb[r] is the byte offset of token r's
// channels from the resource's base (tile_pad_row from the window's end to a
// multiple of 64 rows).
template <int HD, int NT, bool DIRECT>
__device__ inline void tile_load(const i32x4& rs, char* tile, const uint32_t* tokb, int r0) {
  constexpr int kChunks = 64 * HD / 8;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int u = 0; u < (kChunks + NT - 1) / NT; ++u) {
    if (kChunks % NT != 0 && u * NT + wave * 64 >= kChunks) break;    // whole waves
    const int q = u * NT + threadIdx.x;
    const int row = q / (HD / 8), p = q % (HD / 8);
    const uint32_t voff = tokb[r0 + row] + 16u * (uint32_t)(p ^ tile_swz<HD>(row));
    if constexpr (DIRECT) {
      buffer_load_lds16(rs, tile + 16 * (u * NT + wave * 64), (int)voff);
    } else {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      typedef u32x4 u32x4_2 __attribute__((aligned(2)));
      const char* base = reinterpret_cast<const char*>((uint64_t)(uint32_t)rs[1] << 32 | (uint32_t)rs[0]);
      u32x4 x = {};
      if (voff < (uint32_t)rs[2]) x = *reinterpret_cast<const u32x4_2*>(base + voff);
      *reinterpret_cast<u32x4*>(tile + 16 * q) = x;
    }
  }
}

}  // namespace terra
