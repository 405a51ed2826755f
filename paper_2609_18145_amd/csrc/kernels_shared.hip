// Channel-shared mixing stack: Eq. (1) with both maps reduced to per-position
// scalars shared by every channel, taken from an n x n table per layer:
//   y[t][i][c] = A_l[i] x[t][i][c] + B_l[i] x[t][p(i)][c],
//   A_l[i] = T_l[i][i],  B_l[i] = m(i) T_l[i][p(i)].
// Every channel is independent, so a block owns one window and one slice of
// channels (8 pieces of 16 bytes in memory: 64 bf16 or 32 fp32 channels) and
// keeps that tile in registers, in fp32, through every layer of the stack: the
// forward reads x_0 once and writes each layer's output once (rounded to the
// storage type; the chain itself goes on in fp32), and the backward reads dy
// once and each saved input once, and writes dx once.  The work is a handful
// of FMAs per element, so HBM bandwidth bounds it, and what a layer adds on
// top (exchanging partners, barriers, waiting for its coefficients) has to
// stay out of the stream's way.
//
// Thread mapping: thread tid of T (256 or 512) owns memory piece k = tid % 8 of
// the positions tid / 8 + (T / 8) j.  A wave covers 8 consecutive positions, and
// its global accesses are 128 contiguous bytes per position.  So the partner
// along dimension d is
//   d = 0, 1, 2: in another lane of the wave (lane ^ 8, 16, 32: lane moves);
//   d = 3, 4 (5 too with 512 threads) and the local layer's neighbour: in
//     another wave (through LDS);
//   the dimensions above: in another register of the same thread.
// Only the middle case needs LDS and barriers.  The coefficients are read ahead
// into LDS for many layers at once (shared_ring): read layer by layer, each
// layer waited for them (a gather of one line per position).
// Measured at 64 windows x 256 x 512 bf16, 16 layers, us per launch: forward
// 57.4 (62.6 with the tile in LDS), backward 82.9 (94.0); 285 and 306 MB at a
// device copy's 5.2 TB/s are 55 and 59.  The forward takes 512 threads from n =
// 128 (two or four positions each: 57 against 65 us), the backward 256, whose
// gradients and prefetched inputs do not fit 128 registers.
#include "device_common.h"
#include "hcmix_internal.h"

#include <type_traits>

namespace hcmix {

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int SH_PIECES = 8;   // 16-byte pieces of a row that one block owns

// 16 bytes of E as floats.
template <typename E>
struct Piece {
  static constexpr int V = 16 / (int)sizeof(E);
  float v[V];
};

template <typename E>
__device__ __forceinline__ Piece<E> unpack(const u32x4& u) {
  Piece<E> p;
  if constexpr (sizeof(E) == 2) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      p.v[2 * q] = __uint_as_float(u[q] << 16);
      p.v[2 * q + 1] = __uint_as_float(u[q] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; q++) p.v[q] = __uint_as_float(u[q]);
  }
  return p;
}

template <typename E>
__device__ __forceinline__ u32x4 pack(const Piece<E>& p) {
  u32x4 u;
  if constexpr (sizeof(E) == 2) {
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const bf16 lo = to_bf16(p.v[2 * q]), hi = to_bf16(p.v[2 * q + 1]);
      u[q] = (unsigned)__builtin_bit_cast(unsigned short, lo) |
             ((unsigned)__builtin_bit_cast(unsigned short, hi) << 16);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; q++) u[q] = __float_as_uint(p.v[q]);
  }
  return u;
}

// Partner of position i and whether i takes it (forward), for dimension d
// (d < 0: the local layer, partner i - 1).  The partner is always a valid row
// (i itself where there is none), so reads stay in the tile.
__device__ __forceinline__ int fwd_partner(int i, int d, int bidir, bool* takes) {
  if (d < 0) {
    *takes = i >= 1;
    return i >= 1 ? i - 1 : i;
  }
  *takes = bidir || ((i >> d) & 1);
  return i ^ (1 << d);
}

// The position that i sends to (whose output takes i's value), if any.
__device__ __forceinline__ int receiver(int i, int d, int n, int bidir, bool* sends) {
  if (d < 0) {
    *sends = i + 1 < n;
    return i + 1 < n ? i + 1 : i;
  }
  *sends = bidir || !((i >> d) & 1);
  return i ^ (1 << d);
}

// Sum over the 8 lanes of an aligned group (the 8 pieces of one position):
// within quads by swapping neighbours and pairs, then across the two quads of
// the group by mirroring it, all in DPP lane moves; every lane ends with the
// same value, (q0 + q1) with q the two quad sums, added in a fixed order.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

__device__ __forceinline__ float sum8(float v) {
  v += dpp_move<0xb1>(v);          // quad_perm [1,0,3,2]
  v += dpp_move<0x4e>(v);          // quad_perm [2,3,0,1]
  return v + dpp_move<0x141>(v);   // row_half_mirror: lane l of 8 <- lane 7 - l
}

// (A_l[i], B_l[i]) of every position of layers l0 .. l0 + count - 1 (at most
// `ring`, a power of two) into coef[l % ring][i], U layers' loads in flight.
// Four ahead of the first layer: with sixteen a stack of one layer read its
// lines sixteen times over (64 x 256 x 512 fp32, forward: 19.1 us, now 10.3).
template <int U>
__device__ __forceinline__ void load_coefs(const float* const* tabs, const int* dims, int l0,
                                           int count, int ring, int n, int bidir, float2* coef) {
  const int i = threadIdx.x;
  if (i >= n) return;
#pragma unroll 1
  for (int u0 = 0; u0 < count; u0 += U) {
    float ca[U], cb[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      ca[u] = cb[u] = 0.f;
      if (u0 + u >= count) continue;    // uniform
      const int l = l0 + u0 + u;
      bool takes;
      const int p = fwd_partner(i, dims[l], bidir, &takes);
      const float* row = tabs[l] + (size_t)i * n;
      ca[u] = row[i];
      cb[u] = takes ? row[p] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; u++)
      if (u0 + u < count) coef[((l0 + u0 + u) & (ring - 1)) * n + i] = make_float2(ca[u], cb[u]);
  }
}

// Per-thread view of a slice: V channels per memory piece, LP 16-byte LDS
// pieces (fp32) per memory piece, 8 * LP LDS pieces per row.
template <typename E>
struct Slice {
  static constexpr int V = Piece<E>::V;
  static constexpr int LP = V / 4;
  static constexpr int ROW = SH_PIECES * LP;
  // LDS piece h (< LP) of memory piece k of row i
  __device__ static int at(int i, int k, int h) {
    return i * ROW + ((k * LP + h) ^ (LP == 2 ? (i & 1) : 0));
  }
};

template <typename E>
__device__ __forceinline__ void lds_put(f32x4* tile, int i, int k, const Piece<E>& p) {
  using S = Slice<E>;
#pragma unroll
  for (int h = 0; h < S::LP; h++)
    tile[S::at(i, k, h)] = f32x4{p.v[4 * h], p.v[4 * h + 1], p.v[4 * h + 2], p.v[4 * h + 3]};
}

template <typename E>
__device__ __forceinline__ Piece<E> lds_get(const f32x4* tile, int i, int k) {
  using S = Slice<E>;
  Piece<E> p;
#pragma unroll
  for (int h = 0; h < S::LP; h++) {
    const f32x4 q = tile[S::at(i, k, h)];
    p.v[4 * h] = q[0];
    p.v[4 * h + 1] = q[1];
    p.v[4 * h + 2] = q[2];
    p.v[4 * h + 3] = q[3];
  }
  return p;
}

// Value of lane ^ (8 << D), D = 0, 1, 2.
template <int D>
__device__ __forceinline__ float lane_partner(float x) {
  if constexpr (D == 0) return dpp_move<0x128>(x);   // row_ror:8 of 16 lanes
  const unsigned u = __float_as_uint(x);
  const bool up = (threadIdx.x >> (3 + D)) & 1;
  // the swap leaves the lower halves' values in [0], the upper halves' in [1]
  if constexpr (D == 1) {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(up ? r[0] : r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(up ? r[0] : r[1]);
  }
}

// Rows exchanged through LDS at a time (32 KB of bf16 slices; four positions
// per thread of 256, two of 512), and one row beyond them for the local layer.
constexpr int SH_ROWS = 128;
template <typename E>
constexpr size_t shared_exchange_bytes(int n) {
  return (size_t)((n < SH_ROWS ? n : SH_ROWS) + 1) * SH_PIECES * Slice<E>::V * 4;
}

// Calls f(j, p) once for every position i0 + PJ j of this thread, p being the
// row of its partner as it was before any of these calls (f may change s[j]):
// XOR 2^d for d >= 0, i + near for the local layer (near = -1 or 1; the row
// itself where that leaves the window).  `tile` is the LDS exchange buffer;
// every thread of the block calls this with the same d.
template <typename E, int NJ, int PJ, typename F>
__device__ __forceinline__ void for_partners(const Piece<E> (&s)[NJ], int d, int near, int n, int i0,
                                             int k, f32x4* tile, F f) {
  constexpr int V = Slice<E>::V;
#define HCMIX_REGS(B)                                                       \
  if (d >= 0 && NJ > (1 << B) && (1 << d) == (PJ << B)) {                                        \
    _Pragma("unroll") for (int j = 0; j < NJ; j++) {                        \
      constexpr int M = 1 << B;                                             \
      if (j & M) continue;                                                  \
      const Piece<E> lo = s[j], hi = s[(j + M) % NJ];                       \
      f(j, hi);                                                             \
      f((j + M) % NJ, lo);                                                  \
    }                                                                       \
    return;                                                                 \
  }
#define HCMIX_LANES(D)                                                      \
  if (d == D) {                                                             \
    _Pragma("unroll") for (int j = 0; j < NJ; j++) {                        \
      Piece<E> p;                                                           \
      _Pragma("unroll") for (int v = 0; v < V; v++)                         \
          p.v[v] = lane_partner<D>(s[j].v[v]);                              \
      f(j, p);                                                              \
    }                                                                       \
    return;                                                                 \
  }
  HCMIX_REGS(0)
  HCMIX_REGS(1)
  HCMIX_REGS(2)
  HCMIX_LANES(0)
  HCMIX_LANES(1)
  HCMIX_LANES(2)
#undef HCMIX_LANES
#undef HCMIX_REGS
  // through LDS, G positions per thread at a time; the local layer takes
  // the group first whose outer neighbour belongs to the other
  constexpr int G = NJ < SH_ROWS / PJ ? NJ : SH_ROWS / PJ;
  const int rows = min(n, PJ * G);
  auto group = [&](auto at_group) {
    constexpr int j0 = decltype(at_group)::value * G;
    const int base = PJ * j0;
    __syncthreads();    // every read of the buffer is done
    if (i0 < n) {
#pragma unroll
      for (int j = 0; j < G; j++) lds_put<E>(tile, i0 + PJ * j, k, s[j0 + j]);
      if (j0 > 0 && d < 0 && near < 0 && i0 == PJ - 1) lds_put<E>(tile, rows, k, s[(j0 + NJ - 1) % NJ]);
      if (j0 + G < NJ && d < 0 && near > 0 && i0 == 0) lds_put<E>(tile, rows, k, s[(j0 + G) % NJ]);
    }
    __syncthreads();
    if (i0 < n)
#pragma unroll
      for (int j = 0; j < G; j++) {
        const int i = base + i0 + PJ * j;
        int q = i;
        if (d >= 0) q = i ^ (1 << d);
        else if (i + near >= 0 && i + near < n) q = i + near;
        const int at = q - base;
        f(j0 + j, lds_get<E>(tile, at < 0 || at >= rows ? rows : at, k));
      }
  };
  if constexpr (NJ == G) {
    group(std::integral_constant<int, 0>{});
  } else if (near < 0) {
    group(std::integral_constant<int, 1>{});
    group(std::integral_constant<int, 0>{});
  } else {
    group(std::integral_constant<int, 0>{});
    group(std::integral_constant<int, 1>{});
  }
}

template <typename E, int NJ, int T>
__global__ __launch_bounds__(T, T / 128) void shared_fwd_kernel(SharedFwdArgs a, int ring) {
  using S = Slice<E>;
  constexpr int V = S::V, PJ = T / SH_PIECES;
  const int n = a.n, width = a.width;
  const int chunks = width / (SH_PIECES * V);
  const int t = blockIdx.x / chunks;
  const int c0 = (blockIdx.x % chunks) * SH_PIECES * V;
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* tile = (f32x4*)smem;
  float2* coef = (float2*)(smem + shared_exchange_bytes<E>(n));   // [ring][n]
  const int k = threadIdx.x % SH_PIECES;
  const int i0 = threadIdx.x / SH_PIECES;
  const bool mine = i0 < n;
  const size_t at0 = ((size_t)t * n + i0) * width + c0 + k * V;
  const size_t step = (size_t)PJ * width;
  const E* x0 = (const E*)a.x0;

  u32x4 first[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++)
    first[j] = mine ? *(const u32x4*)(x0 + at0 + j * step) : u32x4{0u, 0u, 0u, 0u};
  load_coefs<4>(a.tab, a.dim, 0, min(ring, a.num_layers), ring, n, a.bidir, coef);
  __syncthreads();
  Piece<E> x[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++) x[j] = unpack<E>(first[j]);
  // The tile is there from here on.  The compiler counts no store_wt16 and
  // would wait for the loads where the loop first uses them, and with them for
  // the stores of the layer before, in every layer.
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)

  for (int l = 0; l < a.num_layers; l++) {
    if (l > 0 && (l & (ring - 1)) == 0) {
      __syncthreads();
      load_coefs<8>(a.tab, a.dim, l, min(ring, a.num_layers - l), ring, n, a.bidir, coef);
      __syncthreads();
    }
    const float2* cf = coef + (l & (ring - 1)) * n;
    const int d = a.dim[l];
    E* out = (E*)a.xs[l];
    for_partners<E, NJ, PJ>(x, d, -1, n, i0, k, tile, [&](int j, const Piece<E>& p) {
      if (!mine) return;
      const int i = i0 + PJ * j;
      bool takes;
      fwd_partner(i, d, a.bidir, &takes);
      const float2 ab = cf[i];
#pragma unroll
      for (int v = 0; v < V; v++)
        x[j].v[v] = takes ? fmaf(ab.y, p.v[v], ab.x * x[j].v[v]) : ab.x * x[j].v[v];
      store_wt16(out + at0 + j * step, pack<E>(x[j]));
    });
  }
}

// NT: dy and the inputs are read non-temporally (shared_bwd_streams).
template <typename E, int NJ, int T, bool NT>
__global__ __launch_bounds__(T, T / 128) void shared_bwd_kernel(SharedBwdArgs a, int ring) {
  using S = Slice<E>;
  constexpr int V = S::V, PJ = T / SH_PIECES;
  const int n = a.n, width = a.width;
  const int chunks = width / (SH_PIECES * V);
  const int t = blockIdx.x / chunks;
  const int c0 = (blockIdx.x % chunks) * SH_PIECES * V;
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* tile = (f32x4*)smem;
  float2* coef = (float2*)(smem + shared_exchange_bytes<E>(n));
  const int k = threadIdx.x % SH_PIECES;
  const int i0 = threadIdx.x / SH_PIECES;
  const bool mine = i0 < n;
  const size_t at0 = ((size_t)t * n + i0) * width + c0 + k * V;
  const size_t step = (size_t)PJ * width;
  const int L = a.num_layers;
  const E* dy = (const E*)a.dy;

  // g: the gradient of the layer's output; x_l rows are loaded a layer ahead.
  // Only the thread's own rows: the partner term of dT, sum over c of
  // g[r][c] x[i][c] for the receiver r of i, is formed by i's thread, which
  // holds x[i] and needs g[r] for dX anyway.
  Piece<E> g[NJ];
  u32x4 xo[NJ];
  auto fetch = [&](const E* src, int j) {
    const u32x4 none = {0u, 0u, 0u, 0u};
    if constexpr (NT)
      return mine ? __builtin_nontemporal_load((const u32x4*)(src + at0 + j * step)) : none;
    else
      return mine ? *(const u32x4*)(src + at0 + j * step) : none;
  };
#pragma unroll
  for (int j = 0; j < NJ; j++) xo[j] = fetch(dy, j);
  {
    const int lo = (L - 1) & -ring;
    load_coefs<4>(a.tab, a.dim, lo, L - lo, ring, n, a.bidir, coef);
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < NJ; j++) g[j] = unpack<E>(xo[j]);
#pragma unroll
  for (int j = 0; j < NJ; j++) xo[j] = fetch((const E*)a.xs[L - 1], j);

  for (int l = L - 1; l >= 0; l--) {
    if (l < L - 1 && (l & (ring - 1)) == ring - 1) {
      __syncthreads();
      // few at a time where the tile fills the registers
      load_coefs<NJ == 8 ? 2 : 8>(a.tab, a.dim, l - (ring - 1), ring, ring, n, a.bidir, coef);
      __syncthreads();
    }
    const E* xnext = (const E*)a.xs[l > 0 ? l - 1 : 0];
    const float2* cf = coef + (l & (ring - 1)) * n;
    const int d = a.dim[l];
    float keep_d = 0.f, keep_o = 0.f;
    for_partners<E, NJ, PJ>(g, d, 1, n, i0, k, tile, [&](int j, const Piece<E>& p) {
      if (!mine) return;
      const int i = i0 + PJ * j;
      bool sends;
      const int r = receiver(i, d, n, a.bidir, &sends);
      const float ai = cf[i].x;
      const float cr = sends ? cf[r].y : 0.f;
      const Piece<E> xi = unpack<E>(xo[j]);
      if (l > 0) xo[j] = fetch(xnext, j);     // the next layer's, once this one's is taken
      float sd = 0.f, so = 0.f;
#pragma unroll
      for (int v = 0; v < V; v++) {
        sd = fmaf(g[j].v[v], xi.v[v], sd);
        so = fmaf(p.v[v], xi.v[v], so);
        g[j].v[v] = sends ? fmaf(cr, p.v[v], ai * g[j].v[v]) : ai * g[j].v[v];
      }
      // the 8 pieces of position i sit in an aligned group of 8 lanes:
      // fixed-order sum, kept by lane j of the group
      sd = sum8(sd);
      so = sum8(so);
      keep_d = k == j ? sd : keep_d;
      keep_o = k == (NJ == SH_PIECES / 2 ? j + NJ : j) ? so : keep_o;
    });
    if (!mine) continue;
    // both sums of every position: dT[i][i] and, where i sends, dT[r][i].  One
    // store per lane and layer, of the same number every layer, so that
    // waiting for the next layer's x does not wait for the stores too.
    float* part = a.partial + (((size_t)l * gridDim.x + blockIdx.x) * n + i0) * 2;
    if constexpr (NJ == SH_PIECES)
      *(__attribute__((address_space(1))) f32x2*)(part + 2 * PJ * k) = f32x2{keep_d, keep_o};
    else if constexpr (NJ == SH_PIECES / 2)
      *(__attribute__((address_space(1))) float*)(part + 2 * PJ * (k % NJ) + k / NJ) = k < NJ ? keep_d : keep_o;
    else if (k < NJ)
      *(__attribute__((address_space(1))) f32x2*)(part + 2 * PJ * k) = f32x2{keep_d, keep_o};
  }
  if (!mine) return;
#pragma unroll
  for (int j = 0; j < NJ; j++)
    *(global_u32x4*)((E*)a.dx + at0 + j * step) = pack<E>(g[j]);
}

// dT_l: the two sums of every position i over all blocks (window x channel
// slice), then the table gradient: dT[i][i], dT[r][i] for the receiver r that
// i sends to, and zeros over the rest of i's row (unless accumulating; the
// entry of i's own partner is written by the partner's block).  Block = (layer, 16 positions: 128 contiguous bytes of
// every block's partials), 512 threads = 32 sums (16 positions x 2) x 16
// block classes: thread (q, v) adds the blocks b = q, q + 16, ... in order,
// and the 16 class sums are added in a fixed tree.
constexpr int SH_RED_ROWS = 16;
constexpr int SH_RED_CLASSES = 16;
constexpr int SH_RED_THREADS = 2 * SH_RED_ROWS * SH_RED_CLASSES;

__global__ __launch_bounds__(SH_RED_THREADS) void shared_dt_reduce_kernel(SharedReduceArgs a) {
  const int n = a.n;
  const int rows = n < SH_RED_ROWS ? n : SH_RED_ROWS;
  const int groups = n / rows;
  const int l = blockIdx.x / groups;
  const int i_base = (blockIdx.x % groups) * rows;
  const int v = threadIdx.x % (2 * SH_RED_ROWS);    // (position, which sum)
  const int q = threadIdx.x / (2 * SH_RED_ROWS);    // block class
  __shared__ float cls[SH_RED_CLASSES][2 * SH_RED_ROWS];
  __shared__ float sums[2 * SH_RED_ROWS];
  float acc = 0.f;
  if (v < 2 * rows) {
    // eight loads in flight, added in block order
    const float* src = a.partial + (size_t)l * a.blocks * n * 2 + 2 * i_base + v;
    for (int b0 = q; b0 < a.blocks; b0 += 8 * SH_RED_CLASSES) {
      float t[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int b = b0 + u * SH_RED_CLASSES;
        t[u] = b < a.blocks ? src[(size_t)b * n * 2] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; u++) acc += t[u];
    }
  }
  cls[q][v] = acc;
  __syncthreads();
  if (threadIdx.x < 2 * SH_RED_ROWS) {
    float t[SH_RED_CLASSES];
#pragma unroll
    for (int c = 0; c < SH_RED_CLASSES; c++) t[c] = cls[c][threadIdx.x];
#pragma unroll
    for (int h = SH_RED_CLASSES / 2; h >= 1; h /= 2)
#pragma unroll
      for (int c = 0; c < h; c++) t[c] += t[c + h];
    sums[threadIdx.x] = t[0];
  }
  __syncthreads();
  float* dt = a.dt[l];
  const int d = a.dim[l];
  if (!a.accumulate)
    for (int e = threadIdx.x; e < rows * n; e += SH_RED_THREADS) {
      const int row = i_base + e / n, j = e % n;
      bool takes;
      const int p = fwd_partner(row, d, a.bidir, &takes);
      if (j != row && !(takes && j == p)) dt[(size_t)row * n + j] = 0.f;
    }
  if (threadIdx.x < 2 * rows) {
    const int i = i_base + threadIdx.x / 2, off = threadIdx.x & 1;
    bool sends;
    const int r = receiver(i, d, n, a.bidir, &sends);
    if (!off || sends) {
      float* o = dt + (size_t)(off ? r : i) * n + i;
      *o = a.accumulate ? *o + sums[threadIdx.x] : sums[threadIdx.x];
    }
  }
}

}  // namespace

bool shared_stack_eligible(int64_t n, int64_t width, int32_t num_layers, int32_t elem_bytes) {
  const int64_t c = SH_PIECES * (16 / elem_bytes);
  return n >= 2 && n <= kSharedMaxN && (n & (n - 1)) == 0 && width % c == 0 && num_layers >= 1 &&
         num_layers <= kSharedMaxLayers;
}

// Layers whose coefficients are in LDS at a time: as many as the stack has, in
// 32 KB (bf16) or 16 KB (fp32, whose exchange buffer is half as large: four
// blocks per CU then, where 32 KB left three for the four of 64 x 256 x 512, a
// round and a third: 17 layers forward 132 us, now 125).
constexpr int SH_MAX_LDS = (int)shared_exchange_bytes<bf16>(kSharedMaxN) + (32 << 10);
template <typename E>
static int shared_ring(int n, int num_layers) {
  constexpr int room = (sizeof(E) == 4 ? 16 : 32) << 10;
  int ring = 1;
  while (ring < num_layers && 2 * ring * n * (int)sizeof(float2) <= room) ring *= 2;
  return ring;
}

static int shared_blocks(int batch, int width, int elem_bytes) {
  return batch * (width / (SH_PIECES * (16 / elem_bytes)));
}

size_t shared_partial_bytes(int64_t batch, int64_t n, int64_t width, int32_t num_layers,
                            int32_t elem_bytes) {
  return (size_t)num_layers * shared_blocks((int)batch, (int)width, elem_bytes) * n * 2 *
         sizeof(float);
}

// The saved inputs do not fit the 256 MB Infinity Cache, so most of what the
// forward left there is gone when the backward comes to it: better read past
// the cache.  Backward after forward, us, non-temporal against ordinary loads:
// 64 x 256 x 512 bf16, 16 layers (268 MB) 96.6 | 101, 12 layers (201 MB) 70.9 |
// 68.7; fp32, 10 layers 104 | 140, 4 layers 52 | 47 (and the forward 43 | 30).
static bool shared_bwd_streams(const SharedBwdArgs& a, int batch, int elem_bytes) {
  return (size_t)a.num_layers * batch * a.n * a.width * elem_bytes >= (size_t)256 << 20;
}

template <typename K, typename A>
static hipError_t shared_launch(K k, int threads, const A& a, int ring, int blocks, size_t lds,
                                std::atomic<unsigned long long>& lds_set, hipStream_t st) {
  // the limit is set once per kernel: the most that any n and depth asks for
  const hipError_t attr = lds_limit_once(lds_set, (const void*)k, SH_MAX_LDS);
  if (attr != hipSuccess) return attr;
  k<<<blocks, threads, lds, st>>>(a, ring);
  return hipGetLastError();
}

// Threads and positions per thread (NJ) by n; KERNEL(E, NJ, T) names the instance.
#define HCMIX_SHARED_CASES(KERNEL, E, T128, T256, ARGS, BLOCKS)                                   \
  {                                                                                               \
    static std::atomic<unsigned long long> lds_set[4];                                            \
    const int ring = shared_ring<E>(a.n, a.num_layers);                                           \
    const size_t lds = shared_exchange_bytes<E>(a.n) + (size_t)ring * a.n * sizeof(float2);       \
    auto go = [&](auto k, int threads, int c) {                                                   \
      return shared_launch(k, threads, ARGS, ring, BLOCKS, lds, lds_set[c], st);                  \
    };                                                                                            \
    switch (a.n <= 32 ? 1 : a.n / 32) {                                                           \
      case 1: e = go(KERNEL(E, 1, 256), 256, 0); break;                                           \
      case 2: e = go(KERNEL(E, 2, 256), 256, 1); break;                                           \
      case 4: e = go(KERNEL(E, 1024 / T128, T128), T128, 2); break;                               \
      default: e = go(KERNEL(E, 2048 / T256, T256), T256, 3);                                     \
    }                                                                                             \
  }
#define HCMIX_SHARED_FWD(E, NJ, T) shared_fwd_kernel<E, NJ, T>
#define HCMIX_SHARED_BWD(E, NJ, T) shared_bwd_kernel<E, NJ, T, false>
#define HCMIX_SHARED_BWD_NT(E, NJ, T) shared_bwd_kernel<E, NJ, T, true>

hipError_t launch_shared_forward(const SharedFwdArgs& a, int batch, int elem_bytes, hipStream_t st) {
  // A launch takes fewer than 2^32 threads along x, up to 512 of them a block:
  // more windows than that take a launch more (128 GiB per tensor and above).
  const int most = ((1 << 23) - 1) / shared_blocks(1, a.width, elem_bytes);
  if (batch > most) {
    const hipError_t first = launch_shared_forward(a, most, elem_bytes, st);
    if (first != hipSuccess) return first;
    const size_t skip = (size_t)most * a.n * a.width * elem_bytes;
    SharedFwdArgs rest = a;
    rest.x0 = (const char*)a.x0 + skip;
    for (int l = 0; l < a.num_layers; l++) rest.xs[l] = (char*)a.xs[l] + skip;
    return launch_shared_forward(rest, batch - most, elem_bytes, st);
  }
  const int blocks = shared_blocks(batch, a.width, elem_bytes);
  hipError_t e;
  if (elem_bytes == 2) HCMIX_SHARED_CASES(HCMIX_SHARED_FWD, bf16, 512, 512, a, blocks)
  else HCMIX_SHARED_CASES(HCMIX_SHARED_FWD, float, 512, 512, a, blocks)
  return e;
}

hipError_t launch_shared_backward(const SharedBwdArgs& a, const SharedReduceArgs& r, int batch,
                                  int elem_bytes, hipStream_t st) {
  const int blocks = shared_blocks(batch, a.width, elem_bytes);
  hipError_t e;
  if (shared_bwd_streams(a, batch, elem_bytes)) {
    if (elem_bytes == 2) HCMIX_SHARED_CASES(HCMIX_SHARED_BWD_NT, bf16, 256, 256, a, blocks)
    else HCMIX_SHARED_CASES(HCMIX_SHARED_BWD_NT, float, 256, 256, a, blocks)
  } else {
    if (elem_bytes == 2) HCMIX_SHARED_CASES(HCMIX_SHARED_BWD, bf16, 256, 256, a, blocks)
    else HCMIX_SHARED_CASES(HCMIX_SHARED_BWD, float, 256, 256, a, blocks)
  }
  if (e != hipSuccess) return e;
  SharedReduceArgs rr = r;
  rr.blocks = blocks;
  const int groups = a.n / (a.n < SH_RED_ROWS ? a.n : SH_RED_ROWS);
  shared_dt_reduce_kernel<<<a.num_layers * groups, SH_RED_THREADS, 0, st>>>(rr);
  return hipGetLastError();
}
#undef HCMIX_SHARED_BWD_NT
#undef HCMIX_SHARED_BWD
#undef HCMIX_SHARED_FWD
#undef HCMIX_SHARED_CASES

}  // namespace hcmix
