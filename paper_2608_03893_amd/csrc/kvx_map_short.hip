// Map kernel for short bf16 calls at head dimension 64 (which: short_call in
// kvx_map_tile.hip).
//
// One workgroup per (target layer, head, K|V) task and 64 tokens, 18 KB of LDS, so
// that a CU holds several and their loads cover each other's latency: gather a
// source layer's rows, strip the source RoPE (Sec. 3.3) into an LDS operand tile,
// transpose its map beside it, contract on v_mfma_f32_32x32x16_bf16 (Eq. ridge_kv,
// Sec. 3.1); after the last source layer bias, target RoPE and store.  Bound by the
// latency of a source layer's loads, k in a row, and by the scalar LDS writes of
// the transposed map (8 heads, 80 layers, k = 4, 64 tokens: 23.0 us a call, 29.3
// with the tile kernel, whose workgroup has a CU to itself).
//
// Operand layout: lane L supplies operand row / column L % 32 and the reduction
// indices 8 (L / 32) .. + 7 of a 16-wide step.  Accumulator register r of lane L
// holds output row 8 (r / 4) + 4 (L / 32) + r % 4, column L % 32.
#include "kvx_bf16.h"
#include "kvx_internal.h"

namespace kvx {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int D = 64, HALF = D / 2;
constexpr int BM = 64;            // tokens per tile
constexpr int XS = D + 8;         // LDS row stride of the operands (elements)
constexpr int CS = D + 4;         // row stride of the fp32 results
constexpr int LDS = 2 * BM * XS * 2;
static_assert(BM == D && BM * CS * 4 <= LDS, "LDS");

// 8 consecutive elements as floats, and back.
__device__ __forceinline__ uint4 load16(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ void unpack8(const uint4& u, float (&v)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[2 * q] = lo_bf16(w[q]);
    v[2 * q + 1] = hi_bf16(w[q]);
  }
}
__device__ __forceinline__ uint4 pack8(const float (&v)[8]) {
  return make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
}
__device__ __forceinline__ void store8(uint16_t* p, const float (&v)[8]) { *reinterpret_cast<uint4*>(p) = pack8(v); }

// Rotate plane (u, v), by minus the angle when INVERSE; then 8 half-split planes
// (u[q], v[q]) or 4 interleaved ones by the (cos, sin) at p.
template <bool INVERSE>
__device__ __forceinline__ void rot(float& u, float& v, float2 cs) {
  const float u0 = u, v0 = v, s = INVERSE ? -cs.y : cs.y;
  u = u0 * cs.x - v0 * s;
  v = v0 * cs.x + u0 * s;
}
template <bool INVERSE>
__device__ __forceinline__ void rot_halfsplit(const float2* p, float (&u)[8], float (&v)[8]) {
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const float4 f = reinterpret_cast<const float4*>(p)[n];
    rot<INVERSE>(u[2 * n], v[2 * n], make_float2(f.x, f.y));
    rot<INVERSE>(u[2 * n + 1], v[2 * n + 1], make_float2(f.z, f.w));
  }
}
template <bool INVERSE>
__device__ __forceinline__ void rot_interleaved(const float2* p, float (&x)[8]) {
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const float4 f = reinterpret_cast<const float4*>(p)[n];
    rot<INVERSE>(x[4 * n], x[4 * n + 1], make_float2(f.x, f.y));
    rot<INVERSE>(x[4 * n + 2], x[4 * n + 3], make_float2(f.z, f.w));
  }
}

template <int STYLE, bool SLOTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6)))
void map_short_kernel(const MapArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];
  uint16_t* Xs = reinterpret_cast<uint16_t*>(smem);
  uint16_t* Ws = Xs + BM * XS;
  float* Cs = reinterpret_cast<float*>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * BM;
  const int task = blockIdx.y;
  const int kv = task & 1;
  const int h = (task >> 1) % a.H;
  const int ll = (task >> 1) / a.H;
  const int l = a.l0 + ll;
  const int64_t T = a.T;
  const int k = a.k;
  const int mb = wave & 1, nb = wave >> 1;   // the wave's 32 tokens and 32 outputs

  f32x16_t acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  const uint16_t* W = reinterpret_cast<const uint16_t*>(kv ? a.wv : a.wk) +
                      ((int64_t)l * a.H + h) * (int64_t)k * D * D;

  for (int i = 0; i < k; ++i) {
    const uint16_t* X = reinterpret_cast<const uint16_t*>(a.src) +
                        (((int64_t)a.idx[ll * k + i] * 2 + kv) * a.H + h) * T * D;
    // the map's loads first: their latency passes under the rows'
    uint4 wr[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) wr[n] = load16(W + (int64_t)i * D * D + 8 * (tid + 256 * n));
    // ---- the operand tile: rows past the end are zero
    if (kv == 0 && STYLE == 0) {
      const int r = tid / (HALF / 8), g = tid % (HALF / 8);
      const int64_t t = t0 + r;
      float u[8] = {}, v[8] = {};
      if (t < T) {
        unpack8(load16(X + t * D + 8 * g), u);
        unpack8(load16(X + t * D + HALF + 8 * g), v);
        rot_halfsplit<true>(a.cs_src + t * HALF + 8 * g, u, v);
      }
      store8(Xs + r * XS + 8 * g, u);
      store8(Xs + r * XS + HALF + 8 * g, v);
    } else {
#pragma unroll
      for (int it = tid; it < BM * (D / 8); it += 256) {
        const int r = it / (D / 8), g = it % (D / 8);
        const int64_t t = t0 + r;
        uint4 w = make_uint4(0, 0, 0, 0);
        if (t < T) {
          w = load16(X + t * D + 8 * g);
          if (kv == 0) {
            float x[8];
            unpack8(w, x);
            rot_interleaved<true>(a.cs_src + t * HALF + 4 * g, x);
            w = pack8(x);
          }
        }
        *reinterpret_cast<uint4*>(Xs + r * XS + 8 * g) = w;
      }
    }
    // ---- the map, transposed: Ws[n][kk] = W[i * D + kk][n]
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int it = tid + 256 * n, kk = it / (D / 8), ng = it % (D / 8);
      const uint32_t w4[4] = {wr[n].x, wr[n].y, wr[n].z, wr[n].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        Ws[(8 * ng + 2 * q) * XS + kk] = (uint16_t)(w4[q] & 0xffffu);
        Ws[(8 * ng + 2 * q + 1) * XS + kk] = (uint16_t)(w4[q] >> 16);
      }
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const int kof = ks * 16 + 8 * (lane >> 5);
      const bf16x8_t av = *reinterpret_cast<const bf16x8_t*>(Xs + (32 * mb + (lane & 31)) * XS + kof);
      const bf16x8_t bv = *reinterpret_cast<const bf16x8_t*>(Ws + (32 * nb + (lane & 31)) * XS + kof);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
    }
    __syncthreads();
  }

  // ---- accumulators to LDS, then bias, target RoPE and rounded store
#pragma unroll
  for (int r = 0; r < 16; ++r)
    Cs[(32 * mb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * CS + 32 * nb + (lane & 31)] = acc[r];
  __syncthreads();

  uint16_t* out = reinterpret_cast<uint16_t*>(a.tgt) + (((int64_t)l * 2 + kv) * a.H + h) * a.tgt_rows * D;
  const uint16_t* bias = reinterpret_cast<const uint16_t*>(kv ? a.bv : a.bk);   // NULL: zero
  if (bias != nullptr) bias += ((int64_t)l * a.H + h) * D;
  // output row of token t, or -1
  auto out_row = [&](int64_t t) -> int64_t {
    if (t >= T) return -1;
    if (!SLOTS) return t;
    const int64_t sl = a.slots[t];
    return sl < a.tgt_rows ? sl : -1;
  };
  auto result8 = [&](int r, int c0, float (&y)[8]) {
    float b[8] = {};
    if (bias != nullptr) unpack8(load16(bias + c0), b);
#pragma unroll
    for (int q = 0; q < 8; ++q) y[q] = Cs[r * CS + c0 + q] + b[q];
  };
  if (kv == 0 && STYLE == 0) {
    const int r = tid / (HALF / 8), g = tid % (HALF / 8);
    const int64_t t = t0 + r, orow = out_row(t);
    if (orow < 0) return;
    float u[8], v[8];
    result8(r, 8 * g, u);
    result8(r, HALF + 8 * g, v);
    rot_halfsplit<false>(a.cs_tgt + t * HALF + 8 * g, u, v);
    store8(out + orow * D + 8 * g, u);
    store8(out + orow * D + HALF + 8 * g, v);
  } else {
#pragma unroll
    for (int it = tid; it < BM * (D / 8); it += 256) {
      const int r = it / (D / 8), g = it % (D / 8);
      const int64_t t = t0 + r, orow = out_row(t);
      if (orow < 0) continue;
      float x[8];
      result8(r, 8 * g, x);
      if (kv == 0) rot_interleaved<false>(a.cs_tgt + t * HALF + 4 * g, x);
      store8(out + orow * D + 8 * g, x);
    }
  }
}

template <int STYLE>
hipError_t launch_short(const MapArgs& a, hipStream_t stream) {
  const dim3 grid((unsigned)((a.T + BM - 1) / BM), (unsigned)(a.nl * a.H * 2));
  if (a.slots != nullptr)
    hipLaunchKernelGGL((map_short_kernel<STYLE, true>), grid, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((map_short_kernel<STYLE, false>), grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_map_short(const MapArgs& a, int style, hipStream_t stream) {
  return style == 0 ? launch_short<0>(a, stream) : launch_short<1>(a, stream);
}

}  // namespace kvx
