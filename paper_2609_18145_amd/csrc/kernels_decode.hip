// Decode step: one new position `pos` of every window through every layer.
// All windows are at the same position, so each layer is one small dense
// product over the batch:
//   y[b] = W_self x[b] + m(pos) W_off x_partner[b]
// with the partner's layer input read from the cache.  The kernel of layer l
// reads its input at `pos` (from the caller's x or the buffer the previous
// layer wrote), the partner's from that layer's ring of earlier inputs, may
// record its own input into the ring for a later position, and writes its
// output to the other pass-on buffer (or to y after the last layer); the
// buffers a launch writes are never ones it reads.
#include "device_common.h"
#include "hcmix_internal.h"

namespace hcmix {

namespace {

// One block per 16 output columns x 16 windows (128 blocks at width 512 and 64
// windows), 16x16 MFMAs with the weights as the A operand, so the result is
// C[o][b]; bf16 on 16x16x32, fp32 on four 16x16x4 (fp32 products and sums) per
// step of 16.  The 4 waves split the contraction in steps (wave w takes steps
// w, w + 4, ...); each wave loads the self and partner operands of CH steps
// before any of their MFMAs, so at width 512 (bf16) every load of the block is
// in flight at once and a layer costs one memory latency.  The wave partials
// are summed through LDS in wave order.  Against 32 x 32 blocks of 8 waves (32
// blocks at that shape) this spreads the loads over four times as many CUs:
// 6.3 -> 4.1 us per layer launch in a graph, with partners.
// RAG: a width that does not fill steps of 64 (bf16: a multiple of 8; fp32: any
// width and alignment), whose last pieces and columns are zero.  fp32 at width
// 384 and 64 windows took 91 us per layer with a thread per output, reading
// a weight row each, against 5.7 us.
constexpr int DEC_WAVES = 4;

template <typename E> struct DecPiece;   // what a lane loads of one operand and step
template <> struct DecPiece<bf16> { typedef bf16x8 T; static constexpr int V = 8; };
template <> struct DecPiece<float> { typedef f32x4 T; static constexpr int V = 4; };

__device__ __forceinline__ f32x4 dec_mma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return mfma16(a, b, c);
}
__device__ __forceinline__ f32x4 dec_mma(const f32x4& a, const f32x4& b, f32x4 c) {
#pragma unroll
  for (int e = 0; e < 4; e++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
  return c;
}

// V elements from column k of a row (zero past the width)
template <typename E, bool RAG>
__device__ __forceinline__ typename DecPiece<E>::T dec_load(const E* row, int k, int w) {
  typedef typename DecPiece<E>::T T;
  if constexpr (!RAG) return *(const T*)(row + k);
  T v = {};
  if constexpr (sizeof(E) == 2) {
    if (k < w) v = *(const T*)(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (k + e < w) v[e] = row[k + e];
  }
  return v;
}

__device__ __forceinline__ bf16 dec_round(float v, bf16) { return to_bf16(v); }
__device__ __forceinline__ float dec_round(float v, float) { return v; }

template <typename E, typename Args, int CH, bool RAG>
__global__ __launch_bounds__(64 * DEC_WAVES) void decode_kernel(Args a) {
  typedef typename DecPiece<E>::T T;
  constexpr int V = DecPiece<E>::V, STEP = 4 * V;
  __shared__ f32x4 part[DEC_WAVES][64];
  // `wave` and `has_partner` are wave-uniform and must be known so: an MFMA
  // under a lane mask (EXEC) still writes its whole result, so every MFMA
  // guard below has to be a scalar branch.
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool has_partner = a.x_partner != nullptr;
  const int o0 = blockIdx.x * 16, b0 = blockIdx.y * 16;
  const int w = a.width;
  const int b = min(b0 + (lane & 15), a.batch - 1);      // clamped; stores are masked
  const int orow = RAG ? min(o0 + (lane & 15), w - 1) : o0 + (lane & 15);
  const int q = lane >> 4;                               // K piece V q .. V q + V - 1 of a step
  const E* xin = a.x_in + (size_t)b * a.in_stride;
  const E* xp = has_partner ? a.x_partner + (size_t)b * a.partner_stride : a.x_in;
  const E* ws = a.w_self + (size_t)orow * w;
  const E* wo = a.w_off + (size_t)orow * w;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int ksteps = RAG ? (w + STEP - 1) / STEP : w / STEP;
  for (int kb = wave; kb < ksteps; kb += DEC_WAVES * CH) {
    T sw[CH], sx[CH], pw[CH], px[CH];
#pragma unroll
    for (int j = 0; j < CH; j++) {
      const int k = kb + DEC_WAVES * j;
      const int k0 = (k < ksteps ? k : 0) * STEP + V * q;   // clamped; the MFMA is skipped
      sw[j] = dec_load<E, RAG>(ws, k0, w);
      sx[j] = dec_load<E, RAG>(xin, k0, w);
      if (has_partner) {
        pw[j] = dec_load<E, RAG>(wo, k0, w);
        px[j] = dec_load<E, RAG>(xp, k0, w);
      }
    }
#pragma unroll
    for (int j = 0; j < CH; j++) {
      if (kb + DEC_WAVES * j >= ksteps) continue;
      acc = dec_mma(sw[j], sx[j], acc);
      if (has_partner) acc = dec_mma(pw[j], px[j], acc);
    }
  }
  part[wave][lane] = acc;
  // the layer records its input for a later position: this block's 16 columns
  if (a.record && wave == 0 && b0 + (lane & 15) < a.batch) {
    const int c = o0 + 4 * q;
    E* rec = a.record + (size_t)b * a.rec_stride;
    if constexpr (RAG) {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (c + e < w) rec[c + e] = xin[c + e];
    } else {
      typedef E E4 __attribute__((ext_vector_type(4)));
      *(E4*)(rec + c) = *(const E4*)(xin + c);
    }
  }
  __syncthreads();
  if (wave != 0) return;
  f32x4 s = part[0][lane];
#pragma unroll
  for (int v = 1; v < DEC_WAVES; v++) s += part[v][lane];
  if (b0 + (lane & 15) >= a.batch) return;
  // C[o][b]: lane l holds window b0 + l%16 and outputs o0 + 4 (l/16) + 0..3
  E* out = a.out + (size_t)b * a.out_stride + o0 + 4 * q;
  if constexpr (RAG) {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (o0 + 4 * q + e < w) out[e] = dec_round(s[e], E());
  } else {
    typedef E E4 __attribute__((ext_vector_type(4)));
    *(E4*)out = E4{dec_round(s[0], E()), dec_round(s[1], E()), dec_round(s[2], E()),
                   dec_round(s[3], E())};
  }
}

}  // namespace

// CH: steps per wave per round, as many as cover the width (no clamped
// duplicate loads) up to 4 (the whole of a bf16 width of 512 in one round).
template <typename E, bool RAG, typename Args>
static hipError_t decode_launch(const Args& a, hipStream_t st) {
  constexpr int STEP = 4 * DecPiece<E>::V;
  const dim3 grid((a.width + 15) / 16, (a.batch + 15) / 16);
  const int ksteps = (a.width + STEP - 1) / STEP;
  if (ksteps <= DEC_WAVES) decode_kernel<E, Args, 1, RAG><<<grid, 64 * DEC_WAVES, 0, st>>>(a);
  else if (ksteps <= 2 * DEC_WAVES) decode_kernel<E, Args, 2, RAG><<<grid, 64 * DEC_WAVES, 0, st>>>(a);
  else decode_kernel<E, Args, 4, RAG><<<grid, 64 * DEC_WAVES, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_decode_bf16(const DecodeLayerArgs& a, hipStream_t st) {
  return a.width % 64 == 0 ? decode_launch<bf16, false>(a, st) : decode_launch<bf16, true>(a, st);
}

hipError_t launch_decode_f32(const DecodeLayerArgsF32& a, hipStream_t st) {
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };   // (null: aligned)
  const bool whole = a.width % 16 == 0 && a.in_stride % 4 == 0 && a.partner_stride % 4 == 0 &&
                     a.out_stride % 4 == 0 && a.rec_stride % 4 == 0 && al(a.x_in) &&
                     al(a.x_partner) && al(a.w_self) && al(a.w_off) && al(a.out) && al(a.record);
  return whole ? decode_launch<float, false>(a, st) : decode_launch<float, true>(a, st);
}

}  // namespace hcmix
