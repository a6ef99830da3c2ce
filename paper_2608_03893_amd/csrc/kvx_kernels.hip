// HIP kernels of the KV-cache mapper for CDNA4 (gfx950).
//
// Two kernels make one mapping call:
//   rope_table_kernel  cos/sin of every (token, plane) for the source and the
//                      target RoPE (Sec. 3.3), angle p * w_j reduced in float64
//                      and stored as float32 [T][d/2] (cos, sin) pairs;
//   map_kernel         fp32 calls: for one (target layer, head, K|V) task and
//                      one tile of 64 tokens: gather the k selected source
//                      layers, strip the source RoPE from keys (Sec. 3.3) into
//                      an LDS operand tile, contract with the layer's [k*d, d]
//                      map on the matrix cores (Eq. ridge_kv, Sec. 3.1), add
//                      the bias in content space, re-apply the target RoPE and
//                      store.
//
// Matrix-core use: v_mfma_f32_32x32x2_f32.  Lane L of a wave holds operand
// row/column (L % 32) and reduction index L/32 of a 2-wide step.  Accumulator
// register r of lane L holds output row 8*(r/4) + 4*(L/32) + (r%4), column
// L % 32.
#include "kvx_internal.h"

namespace kvx {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- RoPE table

__device__ __forceinline__ uint32_t half2_bits(double c, double s) {
  // (cos, sin) rounded once from float64 to fp16, cos in the low half
  const _Float16 hc = (_Float16)c, hs = (_Float16)s;
  return (uint32_t)__builtin_bit_cast(uint16_t, hc) |
         ((uint32_t)__builtin_bit_cast(uint16_t, hs) << 16);
}

__global__ __launch_bounds__(256) void rope_table_kernel(
    const int32_t* __restrict__ pos, int T, int half, const InvFreq fs,
    const InvFreq ft, int both, float2* __restrict__ cs_src,
    float2* __restrict__ cs_tgt, uint32_t* __restrict__ cs16,
    uint32_t* __restrict__ cs16_tgt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)T * half) return;
  const int t = (int)(i / half);
  const int j = (int)(i - (int64_t)t * half);
  const double p = (double)pos[t];
  double s, c;
  sincos(p * fs.w[j], &s, &c);
  cs_src[i] = make_float2((float)c, (float)s);
  cs16[i] = half2_bits(c, s);
  if (both) {
    sincos(p * ft.w[j], &s, &c);
    cs_tgt[i] = make_float2((float)c, (float)s);
    cs16_tgt[i] = half2_bits(c, s);
  }
}

// ------------------------------------------------------------ element access

// 8 consecutive floats at p (16-byte aligned).
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = reinterpret_cast<const float4*>(p)[0];
  const float4 b = reinterpret_cast<const float4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
  reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}

__device__ __forceinline__ void load_cs8(const float2* p, float (&c)[8], float (&s)[8]) {
  const float4* q = reinterpret_cast<const float4*>(p);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const float4 f = q[n];
    c[2 * n] = f.x; s[2 * n] = f.y; c[2 * n + 1] = f.z; s[2 * n + 1] = f.w;
  }
}

__device__ __forceinline__ void load_cs4(const float2* p, float (&c)[4], float (&s)[4]) {
  const float4* q = reinterpret_cast<const float4*>(p);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const float4 f = q[n];
    c[2 * n] = f.x; s[2 * n] = f.y; c[2 * n + 1] = f.z; s[2 * n + 1] = f.w;
  }
}

// Rotate plane (u, v) by +a (forward) or -a (inverse) given cos a, sin a.
template <bool INVERSE>
__device__ __forceinline__ void rot(float& u, float& v, float c, float s) {
  const float u0 = u, v0 = v;
  if constexpr (INVERSE) {
    u = u0 * c + v0 * s;
    v = v0 * c - u0 * s;
  } else {
    u = u0 * c - v0 * s;
    v = v0 * c + u0 * s;
  }
}

// ------------------------------------------------------------------ map tile

template <int D>
struct Tile {
  static constexpr int BM = 64;                         // tokens per tile
  static constexpr int HALF = D / 2;
  static constexpr int XS = D + 4;                      // LDS row stride of the operand tile (floats)
  static constexpr int CS = D + 4;                      // fp32 result stride
  static constexpr int X_BYTES = BM * XS * 4;
  static constexpr int W_BYTES = D * D * 4;
  static constexpr int C_BYTES = BM * CS * 4;
  static constexpr int LDS = (X_BYTES + W_BYTES) > C_BYTES ? (X_BYTES + W_BYTES) : C_BYTES;
  static constexpr int MB = BM / 32;                    // 32-row blocks
  static constexpr int NBW = (D / 32) * MB / 4;         // 32-col blocks per wave
  static constexpr int NB_STRIDE = 4 / MB;              // wave's blocks: nb0 + q*NB_STRIDE
  static constexpr int XP = BM * D / 8 / 256;           // 8-float pieces of the tile per thread
  static constexpr int WP = D * D / 4 / 256;            // 4-float pieces of the map per thread
};

// Reduction order within 8 indices: step j takes index j in lanes 0..31 and
// 4 + j in lanes 32..63, so that a lane reads its four steps of an operand row
// as 16 bytes.  The map stays as given, [reduction][output], its 32-column runs
// exchanged on the rows of lanes 32..63: both halves of a wave read distinct banks.
// The next source layer's rows and map are in flight, in registers, while the
// current one is multiplied.  Bound by the fp32 matrix rate and the two barriers
// per source layer: 40 -> 64 layers, 8 heads, d = 128, k = 4, T = 2048: 3.26 ms (84
// of 152 TFLOP/s; 5.93 ms with the map transposed by scalar LDS writes and no
// loads ahead).
template <int D, int STYLE, bool SLOTS>
__global__ __launch_bounds__(256) void map_kernel(const MapArgs a) {
  using G = Tile<D>;
  constexpr int BM = G::BM, HALF = G::HALF, XS = G::XS, CS = G::CS;
  __shared__ __attribute__((aligned(16))) unsigned char smem[G::LDS];
  float* Xs = reinterpret_cast<float*>(smem);
  float* Ws = reinterpret_cast<float*>(smem + G::X_BYTES);
  float* Cs = reinterpret_cast<float*>(smem);

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int t0 = blockIdx.x * BM;
  const int task = blockIdx.y;
  const int kv = task & 1;
  const int h = (task >> 1) % a.H;
  const int ll = (task >> 1) / a.H;
  const int l = a.l0 + ll;
  const int64_t T = a.T;
  const int k = a.k;
  const int mb = wave % G::MB;
  const int nb0 = wave / G::MB;

  f32x16_t acc[G::NBW];
#pragma unroll
  for (int q = 0; q < G::NBW; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[q][r] = 0.0f;

  const float* W = reinterpret_cast<const float*>(kv ? a.wv : a.wk) +
                ((int64_t)l * a.H + h) * (int64_t)k * D * D;

  // Piece n of the tile for this thread: 8 channels at c0 of row r; a half-split
  // key's pieces come in pairs, HALF apart, in one thread.
  auto piece = [&](int n, int& r, int& c0) __attribute__((always_inline)) {
    if (STYLE == 0) {
      const int it = tid + 256 * (n >> 1);
      r = it / (HALF / 8);
      c0 = 8 * (it % (HALF / 8)) + HALF * (n & 1);
    } else {
      const int it = tid + 256 * n;
      r = it / (D / 8);
      c0 = 8 * (it % (D / 8));
    }
  };
  static_assert(G::XP % 2 == 0 && G::WP >= 1, "pieces");
  float xr[G::XP][8];
  f32x4_t wr[G::WP];   // a native vector: arrays of float4 end up in scratch memory
  auto load_layer = [&](int i) __attribute__((always_inline)) {
    const float* X = reinterpret_cast<const float*>(a.src) +
                     (((int64_t)a.idx[ll * k + i] * 2 + kv) * a.H + h) * T * D;
#pragma unroll
    for (int n = 0; n < G::XP; ++n) {
      int r, c0;
      piece(n, r, c0);
      const int64_t t = t0 + r < T ? t0 + r : T - 1;   // a clamped row feeds only its own output row
      load8(X + t * D + c0, xr[n]);
    }
#pragma unroll
    for (int n = 0; n < G::WP; ++n)
      wr[n] = reinterpret_cast<const f32x4_t*>(W + (int64_t)i * D * D)[tid + 256 * n];
  };
  load_layer(0);

  for (int i = 0; i < k; ++i) {
    if (i > 0) __syncthreads();   // the previous layer's operands are read
    // ---- strip the source RoPE (keys) and stage the operand tile and the map
    if (kv == 0) {
#pragma unroll
      for (int n = 0; n < G::XP; n += STYLE == 0 ? 2 : 1) {
        int r, c0;
        piece(n, r, c0);
        const int64_t t = t0 + r < T ? t0 + r : T - 1;
        if (STYLE == 0) {
          float c[8], sn[8];
          load_cs8(a.cs_src + t * HALF + c0, c, sn);
#pragma unroll
          for (int q = 0; q < 8; ++q) rot<true>(xr[n][q], xr[n + 1][q], c[q], sn[q]);
        } else {   // interleaved planes (2j, 2j+1)
          float c[4], sn[4];
          load_cs4(a.cs_src + t * HALF + c0 / 2, c, sn);
#pragma unroll
          for (int q = 0; q < 4; ++q) rot<true>(xr[n][2 * q], xr[n][2 * q + 1], c[q], sn[q]);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < G::XP; ++n) {
      int r, c0;
      piece(n, r, c0);
      store8(Xs + r * XS + c0, xr[n]);
    }
#pragma unroll
    for (int n = 0; n < G::WP; ++n) {
      const int e = 4 * (tid + 256 * n), kk = e / D, c0 = e % D;
      *reinterpret_cast<f32x4_t*>(Ws + kk * D + (c0 ^ (32 * ((kk >> 2) & 1)))) = wr[n];
    }
    if (i + 1 < k) load_layer(i + 1);
    __syncthreads();
    // ---- contraction on the matrix cores
    const int hi = lane >> 5, col = lane & 31;
    const float* xrow = Xs + (mb * 32 + col) * XS + 4 * hi;
    const float* wrow = Ws + 4 * hi * D;
#pragma unroll 4
    for (int m = 0; m < D / 8; ++m) {
      const float4 av = *reinterpret_cast<const float4*>(xrow + 8 * m);
      const float x4[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < G::NBW; ++q) {
          const int n = ((nb0 + q * G::NB_STRIDE) * 32 ^ (32 * hi)) + col;
          acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(x4[j], wrow[(8 * m + j) * D + n], acc[q], 0, 0, 0);
        }
    }
  }
  __syncthreads();

  // ---- accumulators to LDS (fp32), then bias + target RoPE + rounded store
#pragma unroll
  for (int q = 0; q < G::NBW; ++q) {
    const int col = (nb0 + q * G::NB_STRIDE) * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = mb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      Cs[row * CS + col] = acc[q][r];
    }
  }
  __syncthreads();

  float* out = reinterpret_cast<float*>(a.tgt) + (((int64_t)l * 2 + kv) * a.H + h) * a.tgt_rows * D;
  // NULL bias means zero; K and V biases are independent.
  const float* bias = reinterpret_cast<const float*>(kv ? a.bv : a.bk);
  if (bias != nullptr) bias += ((int64_t)l * a.H + h) * D;

  auto out_row = [&](int64_t t) -> int64_t {
    if constexpr (SLOTS) {
      const int64_t sl = a.slots[t];
      return (sl < 0 || sl >= a.tgt_rows) ? -1 : sl;
    } else {
      return t;
    }
  };
  auto bias8 = [&](int c0, float (&b)[8]) {
    if (bias != nullptr) {
      load8(bias + c0, b);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) b[q] = 0.0f;
    }
  };

  if (kv == 0 && STYLE == 0) {
    for (int it = tid; it < BM * (HALF / 8); it += 256) {
      const int r = it / (HALF / 8), g = it % (HALF / 8);
      const int64_t t = t0 + r;
      if (t >= T) continue;
      const int64_t orow = out_row(t);
      if (orow < 0) continue;
      float u[8], v[8], bu[8], bv[8], c[8], sn[8];
      bias8(8 * g, bu);
      bias8(HALF + 8 * g, bv);
      load_cs8(a.cs_tgt + t * HALF + 8 * g, c, sn);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        u[q] = Cs[r * CS + 8 * g + q] + bu[q];
        v[q] = Cs[r * CS + HALF + 8 * g + q] + bv[q];
        rot<false>(u[q], v[q], c[q], sn[q]);
      }
      store8(out + orow * D + 8 * g, u);
      store8(out + orow * D + HALF + 8 * g, v);
    }
  } else {
    for (int it = tid; it < BM * (D / 8); it += 256) {
      const int r = it / (D / 8), g = it % (D / 8);
      const int64_t t = t0 + r;
      if (t >= T) continue;
      const int64_t orow = out_row(t);
      if (orow < 0) continue;
      float x[8], b[8];
      bias8(8 * g, b);
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = Cs[r * CS + 8 * g + q] + b[q];
      if (kv == 0) {  // interleaved keys
        float c[4], sn[4];
        load_cs4(a.cs_tgt + t * HALF + 4 * g, c, sn);
#pragma unroll
        for (int q = 0; q < 4; ++q) rot<false>(x[2 * q], x[2 * q + 1], c[q], sn[q]);
      }
      store8(out + orow * D + 8 * g, x);
    }
  }
}

template <int D, int STYLE, bool SLOTS>
hipError_t launch_one(const MapArgs& a, hipStream_t stream) {
  using G = Tile<D>;
  const dim3 grid((unsigned)((a.T + G::BM - 1) / G::BM), (unsigned)(a.nl * a.H * 2));
  hipLaunchKernelGGL((map_kernel<D, STYLE, SLOTS>), grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

template <int D, int STYLE>
hipError_t launch_style(const MapArgs& a, hipStream_t stream) {
  return a.slots != nullptr ? launch_one<D, STYLE, true>(a, stream)
                            : launch_one<D, STYLE, false>(a, stream);
}

template <int D>
hipError_t launch_d(const MapArgs& a, int style, hipStream_t stream) {
  return style == 0 ? launch_style<D, 0>(a, stream) : launch_style<D, 1>(a, stream);
}

}  // namespace

hipError_t launch_rope_tables(const int32_t* positions, int T, int d,
                              const InvFreq& src, const InvFreq& tgt, bool same,
                              float2* cs_src, float2* cs_tgt, void* cs16,
                              void* cs16_tgt, hipStream_t stream) {
  const int half = d / 2;
  const int64_t n = (int64_t)T * half;
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(rope_table_kernel, dim3(blocks), dim3(256), 0, stream,
                     positions, T, half, src, tgt, same ? 0 : 1, cs_src, cs_tgt,
                     reinterpret_cast<uint32_t*>(cs16), reinterpret_cast<uint32_t*>(cs16_tgt));
  return hipGetLastError();
}

hipError_t launch_map(const MapArgs& a, int dtype, int d, int style, hipStream_t stream) {
  if (a.T == 0 || a.nl == 0) return hipSuccess;
  if (dtype == 0) return launch_map_tile(a, d, style, stream);
  if (d == 128) return launch_d<128>(a, style, stream);
  if (d == 64) return launch_d<64>(a, style, stream);
  return hipErrorInvalidValue;
}

}  // namespace kvx
