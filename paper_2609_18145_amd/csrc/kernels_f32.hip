// fp32 path of the mixing layer on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums, nothing rounded
// below 32 bits), for any width, alignment and row count.
//
// What bounds it: the matrix cores, which do 256 flop per clock and CU in fp32
// (a 8192^3 library product reaches 154 TFLOP/s), twice what one FMA per lane
// and clock gives.  The tiles are 64 x 64 with 32-wide contraction slices: 16
// flop per byte moved into the CU, 16 B/clk at full matrix rate, which L2
// serves; two slices sit in LDS and the next one travels through registers
// meanwhile.  Measured at 4096 rows x 256, 8 layers, forward and backward: 255
// us (76 TFLOP/s), against 6998 us with 4 x 4 FMAs per thread and a launch of
// one block per weight-gradient tile for every layer.
#include "hcmix_internal.h"

namespace hcmix {

namespace {

constexpr int BM = 64;    // rows per block (hypercube layers: 32 lower rows, then their partners)
constexpr int BN = 64;    // output columns per block, 16 per wave
constexpr int KC = 32;    // contraction slice
constexpr int NT = 512;   // two groups of four waves, one k16 step of a slice each
// LDS row strides in floats.  A [row][k] tile is read 16 bytes per lane, 16
// rows at a time: 144-byte rows put them in 16 distinct bank groups.  A
// [k][column] tile is read 4 bytes per lane, 4 k-rows of 16 columns: the k-rows
// a lane group reads lie 4 apart (weights, LDT) or 1 apart (gradients: the
// tile's width + 16), and must fall 16 banks apart.
constexpr int LDK = KC + 4;
constexpr int LDT = BN + 4;
constexpr int MAX_TILES_X = 1 << 22;   // row tiles along a launch's x (NT threads each)

__device__ __forceinline__ f32x4 mfma4(float a, float b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Columns col .. col + 3 of a row (zero outside the width, or if !valid).
// VEC: width a multiple of 4 and 16-byte aligned rows, so a piece of four is
// wholly inside or outside.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* __restrict__ row, int col, int width,
                                       bool valid) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (valid && col < width) v = *(const f32x4*)(row + col);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (valid && col + e < width) v[e] = row[col + e];
  }
  return v;
}

template <bool VEC>
__device__ __forceinline__ void put4(float* __restrict__ dst, int col, int width, const f32x4& v,
                                     bool add) {
  if constexpr (VEC) {
    if (col < width) {
      f32x4* p = (f32x4*)(dst + col);
      *p = add ? *p + v : v;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (col + e < width) dst[col + e] = add ? dst[col + e] + v[e] : v[e];
  }
}

// out[r][j] = sum_k A[r][k] W1(j,k) + m(r) sum_k A[p(r)][k] W2(j,k)
// Hypercube layer: p(r) = r ^ 2^d, m(r) = partner_upper / partner_lower by bit
// d of r; the block's rows are 32 lower rows and their 32 partners, so a row's
// partner is the other half's row of the same tile and causal blocks do no
// product for the half that takes none.  Local layer (NEAR): p(r) = r + shift
// with shift = -1 (forward; m = 0 at a window's first row) or +1 (dX; m = 0 at
// its last row); the partners are a tile of their own.
// Each wave takes all 64 rows and 16 columns, so every wave has the same work,
// and one of a slice's two k16 steps, so that a SIMD has two waves to hide
// staging and fragment reads (4096 x 256, 256 blocks: 13.6 -> 11.9 us).
// The weights are the first MFMA operand: a lane ends with four consecutive
// columns of one row.  Contraction order within a slice: lane group g holds
// k = 16 i + 4 g + e in the e-th product of step i, for both operands.
template <bool VEC, bool TRANSPOSE_W, bool NEAR>
__global__ __launch_bounds__(NT) void mix_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ W1, const float* __restrict__ W2,
    float* __restrict__ out, int rows, int width, int d, int partner_lower, int partner_upper,
    int n, int shift) {
  constexpr int A_SZ = BM * LDK, W_SZ = TRANSPOSE_W ? KC * LDT : BN * LDK;
  constexpr int STAGE = (NEAR ? 2 : 1) * A_SZ + 2 * W_SZ;
  __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (tid >> 6) & 3, group = tid >> 8;
  const int l15 = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.y * BN;
  // (tiles past the rows, where the launch's z does not divide them: every
  // row_of is -1, so they load nothing and store nothing)
  const int row_tile = blockIdx.x + blockIdx.z * gridDim.x;
  const int s = NEAR ? 0 : 1 << d;
  const int pairs = rows / 2;
  // tile row m -> row of the tensor (-1: outside)
  auto row_of = [&](int m) {
    if constexpr (NEAR) {
      const int r = row_tile * BM + m;
      return r < rows ? r : -1;
    }
    const int q = row_tile * (BM / 2) + (m & 31);
    return q < pairs ? lower_row(q, d) + (m >= 32 ? s : 0) : -1;
  };

  // this thread's 16-byte piece of each tile
  const int r_mine = row_of(tid >> 3);
  const bool a_ok = r_mine >= 0;
  const float* a_row = A + (size_t)(a_ok ? r_mine : 0) * width;
  bool p_ok = false;
  const float* p_row = A;
  if constexpr (NEAR) {
    const int pos = r_mine & (n - 1);
    p_ok = a_ok && (shift < 0 ? pos != 0 : pos != n - 1);
    if (p_ok) p_row = A + (size_t)(r_mine + shift) * width;
  }
  struct Regs { f32x4 a, p, w1, w2; } regs[2];
  auto fetch = [&](int k0, Regs& f) {
    const int col = k0 + (tid & 7) * 4;
    f.a = load4<VEC>(a_row, col, width, a_ok);
    if constexpr (NEAR) f.p = load4<VEC>(p_row, col, width, p_ok);
    if constexpr (TRANSPOSE_W) {   // rows are k, contiguous along the output columns
      const int k = k0 + (tid >> 4);
      const size_t off = (size_t)(k < width ? k : 0) * width;
      f.w1 = load4<VEC>(W1 + off, j0 + (tid & 15) * 4, width, k < width);
      f.w2 = load4<VEC>(W2 + off, j0 + (tid & 15) * 4, width, k < width);
    } else {
      const int o = j0 + (tid >> 3);
      const size_t off = (size_t)(o < width ? o : 0) * width;
      f.w1 = load4<VEC>(W1 + off, col, width, o < width);
      f.w2 = load4<VEC>(W2 + off, col, width, o < width);
    }
  };
  auto stage = [&](float* b, const Regs& f) {
    float* w1 = b + (NEAR ? 2 : 1) * A_SZ;
    const int ka = (tid >> 3) * LDK + (tid & 7) * 4, kt = (tid >> 4) * LDT + (tid & 15) * 4;
    *(f32x4*)(b + ka) = f.a;
    if constexpr (NEAR) *(f32x4*)(b + A_SZ + ka) = f.p;
    *(f32x4*)(w1 + (TRANSPOSE_W ? kt : ka)) = f.w1;
    *(f32x4*)(w1 + W_SZ + (TRANSPOSE_W ? kt : ka)) = f.w2;
  };

  f32x4 acc[4] = {};
  auto compute = [&](const float* b) {
    const float* w1 = b + (NEAR ? 2 : 1) * A_SZ;
    const float* w2 = w1 + W_SZ;
    {
      const int k = 16 * group + 4 * g;
      f32x4 b1, b2, a[4], pv[4];
      if constexpr (TRANSPOSE_W) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
          b1[e] = w1[(k + e) * LDT + 16 * wave + l15];
          b2[e] = w2[(k + e) * LDT + 16 * wave + l15];
        }
      } else {
        b1 = *(const f32x4*)(w1 + (16 * wave + l15) * LDK + k);
        b2 = *(const f32x4*)(w2 + (16 * wave + l15) * LDK + k);
      }
#pragma unroll
      for (int t = 0; t < 4; t++) {
        a[t] = *(const f32x4*)(b + (16 * t + l15) * LDK + k);
        if constexpr (NEAR) pv[t] = *(const f32x4*)(b + A_SZ + (16 * t + l15) * LDK + k);
      }
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int t = 0; t < 4; t++) acc[t] = mfma4(b1[e], a[t][e], acc[t]);
      if constexpr (NEAR) {
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int t = 0; t < 4; t++) acc[t] = mfma4(b2[e], pv[t][e], acc[t]);
      } else {
        if (partner_upper) {
#pragma unroll
          for (int e = 0; e < 4; e++)
#pragma unroll
            for (int t = 2; t < 4; t++) acc[t] = mfma4(b2[e], a[t - 2][e], acc[t]);
        }
        if (partner_lower) {
#pragma unroll
          for (int e = 0; e < 4; e++)
#pragma unroll
            for (int t = 0; t < 2; t++) acc[t] = mfma4(b2[e], a[t + 2][e], acc[t]);
        }
      }
    }
  };

  // two slices in LDS, two on the way in registers: a slice's products take
  // 0.7 us, a load past L2 up to twice that
  const int nk = (width + KC - 1) / KC;
  fetch(0, regs[0]);
  if (nk > 1) fetch(KC, regs[1]);
  stage(smem, regs[0]);
  __syncthreads();
  auto step = [&](int kt, Regs& far, const Regs& near_) {
    if (kt + 2 < nk) fetch((kt + 2) * KC, far);
    compute(smem + (kt & 1) * STAGE);
    if (kt + 1 < nk) stage(smem + ((kt + 1) & 1) * STAGE, near_);
    __syncthreads();
  };
  for (int kt = 0; kt < nk; kt += 2) {
    step(kt, regs[0], regs[1]);
    if (kt + 1 < nk) step(kt + 1, regs[1], regs[0]);
  }
  // the second group's sums, added to the first's
  f32x4* hand = (f32x4*)smem + wave * 256 + lane;
  if (group == 1)
#pragma unroll
    for (int t = 0; t < 4; t++) hand[64 * t] = acc[t];
  __syncthreads();
  if (group == 1) return;
#pragma unroll
  for (int t = 0; t < 4; t++) {
    acc[t] += hand[64 * t];
    const int r = row_of(16 * t + l15);
    if (r >= 0) put4<VEC>(out + (size_t)r * width, j0 + 16 * wave + 4 * g, width, acc[t], false);
  }
}

// Weight gradients of the layers of a stack in one launch:
//   dws[o][c] (+)= sum_r dY[r][o] X[r][c],  dwo[o][c] (+)= sum_r m(r) dY[r][o] X[p(r)][c].
// Block -> (layer, row range, matrix, tile); the off-diagonal matrix of
// a causal hypercube layer walks the receiving rows only.  Rows are walked in
// order, so the sums do not depend on the launch.  With one range per layer
// the tile goes straight to dws / dwo, otherwise to partial[layer][range][2].
// T x T tiles (128, or 64 where those are too few): a row of both operands moves 8 T
// bytes into the CU for 2 T^2 flop, so that 64 x 64 tiles were bound by L2
// (8 layers of 4096 x 256: 89 -> 70 us, with the order of the blocks below).  Four waves of (T / 2) x (T / 2).
template <bool VEC, int T>
__global__ __launch_bounds__(256) void dw_f32_kernel(DwBatchArgsF32 a) {
  constexpr int LD = T + 16, T_SZ = KC * LD, P4 = T / 4;   // row stride; pieces of a row
  constexpr int PER = KC * P4 / 256, H = T / 32;           // pieces per thread; 16-blocks per wave
  __shared__ __attribute__((aligned(16))) float smem[4 * T_SZ];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l15 = lane & 15, g = lane >> 4;
  const int wo = (wave & 1) * (T / 2), wc = (wave >> 1) * (T / 2);
  const int width = a.width, te = (width + T - 1) / T, tiles = te * te;
  int lin = blockIdx.x;
  const int tile = lin % tiles;
  lin /= tiles;
  // all diagonal matrices first: with two blocks per CU each then gets one long
  // and one short one (next to each other they go to different XCDs)
  const int per_matrix = a.num_layers * a.splits;
  const int off = lin >= per_matrix;
  lin -= off * per_matrix;
  const int split = lin % a.splits, layer = lin / a.splits;
  const int o0 = (tile / te) * T, c0 = (tile % te) * T;
  const int d = a.dim[layer];
  const int s = d < 0 ? 0 : 1 << d;
  const float* X = a.x[layer];
  const float* dY = a.dy[layer];
  const bool half = off && d >= 0 && !a.bidir;     // receiving (upper) rows only
  const int units = half ? a.rows / 2 : a.rows;
  const int per = ((units + KC - 1) / KC + a.splits - 1) / a.splits * KC;
  const int beg = min(units, split * per), end = min(units, beg + per);

  f32x4 rg[PER], rx[PER];
  auto fetch = [&](int u0) {
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int p = tid + 256 * j;
      const int u = u0 + p / P4, col = (p % P4) * 4;
      const int r = half ? lower_row(u, d) + s : u;
      bool take = u < end;
      int pr = r;
      if (off) {
        if (d < 0) {
          take = take && (r & (a.n - 1)) != 0;
          pr = r - 1;
        } else {
          pr = r ^ s;
        }
      }
      rg[j] = load4<VEC>(dY + (size_t)(u < end ? r : 0) * width, o0 + col, width, u < end);
      rx[j] = load4<VEC>(X + (size_t)(take ? pr : 0) * width, c0 + col, width, take);
    }
  };
  auto stage = [&](float* b) {
#pragma unroll
    for (int j = 0; j < PER; j++) {
      const int p = tid + 256 * j, at = p / P4 * LD + (p % P4) * 4;
      *(f32x4*)(b + at) = rg[j];
      *(f32x4*)(b + T_SZ + at) = rx[j];
    }
  };
  f32x4 acc[H][H] = {};
  auto compute = [&](const float* b) {
#pragma unroll
    for (int k = 0; k < KC; k += 4) {
      const float* gr = b + (k + g) * LD + l15;
      float gv[H], xv[H];
#pragma unroll
      for (int i = 0; i < H; i++) {
        gv[i] = gr[wo + 16 * i];
        xv[i] = gr[T_SZ + wc + 16 * i];
      }
#pragma unroll
      for (int i = 0; i < H; i++)
#pragma unroll
        for (int t = 0; t < H; t++) acc[i][t] = mfma4(xv[t], gv[i], acc[i][t]);
    }
  };
  const int nk = (end - beg + KC - 1) / KC;
  if (nk > 0) {
    fetch(beg);
    stage(smem);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; kt++) {
    if (kt + 1 < nk) fetch(beg + (kt + 1) * KC);
    compute(smem + (kt & 1) * 2 * T_SZ);
    if (kt + 1 < nk) stage(smem + ((kt + 1) & 1) * 2 * T_SZ);
    __syncthreads();
  }
  // lane: output row o0 + wo + 16 i + l15, columns c0 + wc + 16 t + 4 g + 0..3
  const size_t ww = (size_t)width * width;
  float* dst = a.splits == 1 ? (off ? a.dwo[layer] : a.dws[layer])
                             : a.partial + (((size_t)layer * a.splits + split) * 2 + off) * ww;
#pragma unroll
  for (int i = 0; i < H; i++) {
    const int o = o0 + wo + 16 * i + l15;
    if (o >= width) continue;
#pragma unroll
    for (int t = 0; t < H; t++)
      put4<VEC>(dst + (size_t)o * width, c0 + wc + 16 * t + 4 * g, width, acc[i][t],
                a.splits == 1 && a.accumulate);
  }
}

// dW[l] (+)= sum over ranges of partial[l][range], in range order.
__global__ __launch_bounds__(256) void dw_f32_reduce_kernel(DwBatchArgsF32 a) {
  const size_t ww = (size_t)a.width * a.width;
  const int l = blockIdx.y;
  const float* part = a.partial + (size_t)l * a.splits * 2 * ww;
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < 2 * ww; i += (size_t)gridDim.x * 256) {
    float acc = 0.f;
    for (int sp = 0; sp < a.splits; sp++) acc += part[(size_t)sp * 2 * ww + i];
    float* dst = i < ww ? a.dws[l] + i : a.dwo[l] + (i - ww);
    *dst = a.accumulate ? *dst + acc : acc;
  }
}

bool vec16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

hipError_t launch_mix_f32(const float* A, const float* W1, const float* W2, float* out, int rows,
                          int width, int d, int partner_lower, int partner_upper, int n, int shift,
                          bool transpose_w, hipStream_t st) {
  // a launch takes fewer than 2^32 threads along x: from 2^28 rows the row
  // tiles go over z as well
  const int tiles = d < 0 ? (rows + BM - 1) / BM : (rows / 2 + BM / 2 - 1) / (BM / 2);
  const int nz = (tiles + MAX_TILES_X - 1) / MAX_TILES_X;
  const dim3 grid((tiles + nz - 1) / nz, (width + BN - 1) / BN, nz);
  // fp32 tensors need only be 4-byte aligned
  const bool vec = width % 4 == 0 && vec16(A) && vec16(W1) && vec16(W2) && vec16(out);
#define HCMIX_MF(V, T, N)                                                                    \
  mix_f32_kernel<V, T, N><<<grid, NT, 0, st>>>(A, W1, W2, out, rows, width, d, partner_lower, \
                                               partner_upper, n, shift)
#define HCMIX_MFN(V, T) (d < 0 ? HCMIX_MF(V, T, true) : HCMIX_MF(V, T, false))
  if (vec) {
    if (transpose_w) HCMIX_MFN(true, true);
    else HCMIX_MFN(true, false);
  } else {
    if (transpose_w) HCMIX_MFN(false, true);
    else HCMIX_MFN(false, false);
  }
#undef HCMIX_MFN
#undef HCMIX_MF
  return hipGetLastError();
}

// Row ranges per layer: two rounds of blocks per CU over the launch (the causal
// off-diagonal tiles are half as long), each range at least 512 rows.
int dw_f32_splits(int rows, int width, int num_layers) {
  const int64_t te = (width + 127) / 128;
  const int64_t blocks = (int64_t)num_layers * 2 * te * te;
  int64_t splits = (512 + blocks - 1) / blocks;
  if (splits > rows / 512) splits = rows / 512;
  return splits < 1 ? 1 : (int)splits;
}

hipError_t launch_dw_f32(const DwBatchArgsF32& a, hipStream_t st) {
  // 128 x 128 tiles where they give most CUs a block (the tile does not change
  // the order of the sums); a single layer has too few of them
  const int64_t wide = (a.width + 127) / 128;
  const int tile = a.width > 64 && a.num_layers * a.splits * 2 * wide * wide >= 192 ? 128 : 64;
  const int te = (a.width + tile - 1) / tile;
  const size_t blocks = (size_t)a.num_layers * a.splits * 2 * te * te;
  bool vec = a.width % 4 == 0;
  for (int l = 0; l < a.num_layers; l++) vec = vec && vec16(a.x[l]) && vec16(a.dy[l]);
  if (tile == 128) {
    if (vec) dw_f32_kernel<true, 128><<<(unsigned)blocks, 256, 0, st>>>(a);
    else dw_f32_kernel<false, 128><<<(unsigned)blocks, 256, 0, st>>>(a);
  } else {
    if (vec) dw_f32_kernel<true, 64><<<(unsigned)blocks, 256, 0, st>>>(a);
    else dw_f32_kernel<false, 64><<<(unsigned)blocks, 256, 0, st>>>(a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return e;
  const size_t ww2 = (size_t)2 * a.width * a.width;
  const unsigned per = (unsigned)((ww2 + 255) / 256 < 256 ? (ww2 + 255) / 256 : 256);
  dw_f32_reduce_kernel<<<dim3(per, a.num_layers), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace hcmix
