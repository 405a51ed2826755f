// Tiles of 64 bf16 columns in LDS and the 32 x 32 x 16 MFMA fragments read
// from them, shared by the kernels whose second product takes a score tile
// straight from registers (attention and the field coupling).
#pragma once

#include "hcmix_internal.h"
#include "device_common.h"

namespace hcmix {

constexpr int HD = 64;          // columns of a tile

// LDS tile [rows][64] bf16: 16-byte piece p of row r at piece p ^ sw(r), with
// sw a 3-bit rotation of (r / 2) % 8.  16 consecutive rows reading one piece
// (128-bit fragment reads) cover 256 distinct bytes, and 4 rows aligned to 4
// x 64 bytes (a 32-lane transposed read) do as well: rows r and r + 2 differ
// in bit 2 of sw, so they use different 64-byte halves of the 128-byte row.
__device__ __forceinline__ int att_sw(int r) {
  const int u = (r >> 1) & 7;
  return ((u << 2) | (u >> 1)) & 7;
}
__device__ __forceinline__ int att_off(int r, int col) {
  return r * HD + ((((col >> 3) ^ att_sw(r))) << 3) + (col & 7);
}

// 32 x 16 fragment of a [rows][64] tile as an MFMA operand with the row
// index as the fragment row and 8 contiguous columns per lane: lane l gets
// row r0 + l % 32, columns c0 + 8 (l / 32) .. + 8.
__device__ __forceinline__ bf16x8 att_frag(const bf16* t, int r0, int c0, int lane) {
  return *(const bf16x8*)(t + att_off(r0 + (lane & 31), c0 + 8 * (lane >> 5)));
}

// Transposed fragment for the second product: lane l gets column c0 + l % 32
// of rows {k0 + 4h + 0..3} then {k0 + 8 + 4h + 0..3}, h = l / 32 (the key
// order of a score tile's registers 8m .. 8m + 7 when k0 = 32 kt + 16 m).
__device__ __forceinline__ bf16x8 att_trfrag(const bf16* t, int k0, int c0, int lane) {
  const int g = lane >> 4, j = lane & 15;
  const int row = k0 + 4 * (g >> 1) + (j >> 2);
  const int col = c0 + 16 * (g & 1) + 4 * (j & 3);
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(t + att_off(row, col)));
  const bf16x4 hi =
      __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(t + att_off(row + 8, col)));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Registers 8m .. 8m + 7 of a score tile as a bf16 MFMA operand.
__device__ __forceinline__ bf16x8 att_pack(const f32x16& s, int m) {
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; e++) v[e] = to_bf16(s[8 * m + e]);
  return v;
}

// Store of a 32 x 32 result tile whose rows are lanes (register e of lane l:
// row l % 32, column 8 (e / 4) + 4 (l / 32) + e % 4) to `tile`, rows `stride`
// elements apart, the first `rows` of them; 16-byte aligned.  Lanes l and l ^ 32
// hold alternating runs of four columns of one row: a swap of two of them gives
// each eight, and a swap with l ^ 16 brings a row's four eights to one
// instruction, which then writes 64 bytes of each of 16 rows instead of 16 of
// 32.  Every lane of the wave must call it.
// us, against 8-byte stores of the registers as they are, 64 windows of 256:
// attention forward 19.0 to 17.3 and backward 30.0 + 24.4 to 26.7 + 23.3 (8 heads),
// field readout 12.4 to 10.1, its dx with the coordinates 19.2 to 16.9 (512 columns).
__device__ __forceinline__ void att_store(bf16* tile, size_t stride, const f32x16& o, float scale,
                                          int lane, int rows = 32) {
  u32x4 v[2];
#pragma unroll
  for (int pr = 0; pr < 2; pr++) {
    bf16x4 a, b;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      a[e] = to_bf16(o[8 * pr + e] * scale);
      b[e] = to_bf16(o[8 * pr + 4 + e] * scale);
    }
    const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
    const auto s0 = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
    v[pr] = u32x4{s0[0], s1[0], s0[1], s1[1]};   // columns 16 pr + 8 (l / 32) .. + 8
  }
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const auto s = __builtin_amdgcn_permlane16_swap(v[0][k], v[1][k], false, false);
    v[0][k] = s[0];
    v[1][k] = s[1];
  }
  const int r = lane & 15, col = (lane & 16) + 8 * (lane >> 5);
#pragma unroll
  for (int u = 0; u < 2; u++)
    if (r + 16 * u < rows) *(u32x4*)(tile + (size_t)(r + 16 * u) * stride + col) = v[u];
}

// The query tiles (of 32 positions) of wave w: w and 7 - w, so that every wave
// has the same causal work (w + 1 and 8 - w key tiles) at n = 256.
__device__ __forceinline__ int att_tile(int wave, int which) { return which ? 7 - wave : wave; }

// Causal mask of a diagonal score tile: register e of lane l holds key
// 8 (e / 4) + 4 (l / 32) + e % 4 for query l % 32.
__device__ __forceinline__ bool att_masked(int e, int lane) {
  return 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3) > (lane & 31);
}

}  // namespace hcmix
