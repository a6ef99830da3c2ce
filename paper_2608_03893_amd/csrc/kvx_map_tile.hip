// Map kernels for bf16 calls outside the packed-map kernels: more than four
// source layers, or head dimension 64.
//
// Both compute one (target layer, head, K|V) task on a tile of 256 tokens, 8
// waves of 32 tokens, as C^T = W^T X^T on v_mfma_f32_16x16x32_bf16 (Eq.
// ridge_kv, Sec. 3.1).  A wave loads its tokens' rows of each selected source
// layer straight into registers, one source layer ahead, strips the source
// RoPE from keys there (Sec. 3.3, fp32 coefficients, one rounding) and feeds
// each row fragment to all D / 16 output blocks.  W is read as given and
// transposed on its way into LDS (4 input rows x 8 output channels per
// thread), so no packed copy of it is needed.
//
// Operand layout: lane L = 16 c + r supplies map row / token r and reduction
// indices 8 c .. 8 c + 7 of a 32-wide step.  Map row 16 b + 4 c + i holds
// output channel 32 (b / 2) + 8 c + 4 (b % 2) + i, so that a lane ends with
// channels 32 x + 8 c .. + 7: both members of every RoPE plane it touches, and
// 16-byte stores of which the four lanes of a token cover 64 bytes.
#include "kvx_bf16.h"
#include "kvx_internal.h"
#include "kvx_wload.h"

#include <type_traits>

namespace kvx {
namespace {

constexpr int NTHR = 512;      // threads per workgroup
constexpr int TB = 2;          // 16-token blocks per wave
constexpr int BT = 8 * 16 * TB;   // tokens per tile

template <int D>
struct TileGeo {
  static constexpr int S = D / 32;             // reduction steps per source layer
  static constexpr int NB = D / 16;            // output blocks
  static constexpr int HALF = D / 2;
  static constexpr int PL = D / 8;             // RoPE planes of a token in a lane
  static constexpr int ROWB = 2 * D;           // bytes of a map row in LDS
  static constexpr int SLOTB = D * ROWB;       // bytes of one source layer's map
  static constexpr int PIECES = (D / 4) * (D / 8);   // 4 x 8 pieces of a source layer's map
};

__device__ __forceinline__ void rot_inv32(float& u, float& v, float2 cs) {
  const float u0 = u, v0 = v;
  u = u0 * cs.x + v0 * cs.y;
  v = v0 * cs.x - u0 * cs.y;
}

__device__ __forceinline__ void rot_fwd32(float& u, float& v, float2 cs) {
  const float u0 = u, v0 = v;
  u = u0 * cs.x - v0 * cs.y;
  v = v0 * cs.x + u0 * cs.y;
}

// (cos, sin) of the planes of one token that a lane touches: half-split planes
// 32 x + 8 c + e in cs[8 x + e], interleaved planes 16 x + 4 c + e in cs[4 x + e].
template <int D, int STYLE>
__device__ __forceinline__ void load_planes(const float2* __restrict__ table, int64_t t, int c,
                                            float2 (&cs)[TileGeo<D>::PL]) {
  using G = TileGeo<D>;
  constexpr int RUN = STYLE == 0 ? 8 : 4;
  const float4* p = reinterpret_cast<const float4*>(table + t * G::HALF + RUN * c);
#pragma unroll
  for (int n = 0; n < G::PL / 2; ++n) {
    const float4 f = p[(2 * n / RUN) * 2 * RUN + (2 * n % RUN) / 2];
    cs[2 * n] = make_float2(f.x, f.y);
    cs[2 * n + 1] = make_float2(f.z, f.w);
  }
}

template <int D, int STYLE>
__device__ __forceinline__ void strip_row(u32x4_t (&x)[TileGeo<D>::S], const float2 (&cs)[TileGeo<D>::PL]) {
  constexpr int S = TileGeo<D>::S;
  if (STYLE == 0) {
#pragma unroll
    for (int s = 0; s < S / 2; ++s)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t& a = reinterpret_cast<uint32_t*>(&x[s])[w];
        uint32_t& b = reinterpret_cast<uint32_t*>(&x[s + S / 2])[w];
        float u0 = lo_bf16(a), u1 = hi_bf16(a), v0 = lo_bf16(b), v1 = hi_bf16(b);
        rot_inv32(u0, v0, cs[8 * s + 2 * w]);
        rot_inv32(u1, v1, cs[8 * s + 2 * w + 1]);
        a = pack2(u0, u1);
        b = pack2(v0, v1);
      }
  } else {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t& a = reinterpret_cast<uint32_t*>(&x[s])[w];
        float u = lo_bf16(a), v = hi_bf16(a);
        rot_inv32(u, v, cs[4 * s + w]);
        a = pack2(u, v);
      }
  }
}

// Bias, target RoPE (keys), rounding and store of one token's outputs.
template <int D, int STYLE, bool KEYS>
__device__ __forceinline__ void finish_row(const f32x4_t (&acc)[TileGeo<D>::NB],
                                           const uint16_t* __restrict__ bias,
                                           const float2* __restrict__ table, int64_t t, int c,
                                           uint16_t* __restrict__ out, bool store) {
  using G = TileGeo<D>;
  float y[G::S][8];
#pragma unroll
  for (int x = 0; x < G::S; ++x)
#pragma unroll
    for (int e = 0; e < 8; ++e) y[x][e] = acc[2 * x + (e >> 2)][e & 3];
  if (bias != nullptr) {
#pragma unroll
    for (int x = 0; x < G::S; ++x) {
      const uint4 b = *reinterpret_cast<const uint4*>(bias + 32 * x + 8 * c);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        y[x][2 * w] += lo_bf16((&b.x)[w]);
        y[x][2 * w + 1] += hi_bf16((&b.x)[w]);
      }
    }
  }
  if (KEYS) {
    float2 cs[G::PL];
    load_planes<D, STYLE>(table, t, c, cs);
    if (STYLE == 0) {
#pragma unroll
      for (int x = 0; x < G::S / 2; ++x)
#pragma unroll
        for (int e = 0; e < 8; ++e) rot_fwd32(y[x][e], y[x + G::S / 2][e], cs[8 * x + e]);
    } else {
#pragma unroll
      for (int x = 0; x < G::S; ++x)
#pragma unroll
        for (int e = 0; e < 8; e += 2) rot_fwd32(y[x][e], y[x][e + 1], cs[4 * x + e / 2]);
    }
  }
  if (store) {
#pragma unroll
    for (int x = 0; x < G::S; ++x)
      *reinterpret_cast<uint4*>(out + 32 * x + 8 * c) =
          make_uint4(pack2(y[x][0], y[x][1]), pack2(y[x][2], y[x][3]), pack2(y[x][4], y[x][5]),
                     pack2(y[x][6], y[x][7]));
  }
}

// ------------------------------------------------------- streamed maps
//
// One workgroup per CU; the maps stream through two LDS stages, one source
// layer at a time, and the pipeline runs on from item to item.  The 32 CUs of
// an XCD work on 32 target layers of one (head, K|V) and token tile, so that
// the tile's source rows are read into its L2 once.  Bound by the operand reads
// from LDS (each map fragment feeds two matrix instructions) and by the loads
// that share the vector memory pipe.  Qwen3-14B->32B shapes with k = 8, T =
// 8191: 4.35 ms (0.51 PFLOP/s); the 64-token tiles that staged rows and maps
// through LDS without a pipeline took 16.95 ms.

// The items (head, token tile, K|V, target layer; layers fastest) are cut into
// eight contiguous ranges, one per XCD.
struct TilePlan {
  int64_t items, per_xcd;
  int32_t tiles, len;   // token tiles (ranges) and their length
};

struct Item {
  int h, kv, ll;
  int64_t t0;
};

__device__ __forceinline__ Item item_of(const MapArgs& a, const TilePlan& p, int64_t n) {
  Item it;
  it.ll = (int)(n % a.nl);
  n /= a.nl;
  it.kv = (int)(n & 1);
  n >>= 1;
  it.t0 = (n % p.tiles) * p.len;
  it.h = (int)(n / p.tiles);
  return it;
}

template <int D, int STYLE, bool SLOTS>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(2, 2)))
void map_kernel(const MapArgs a, const TilePlan p) {
  using G = TileGeo<D>;
  constexpr int S = G::S, NB = G::NB;
  __shared__ __attribute__((aligned(256))) char smem[2 * G::SLOTB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane >> 4, row = lane & 15;
  const int64_t T = a.T;
  const int k = a.k;

  const int64_t x0 = (int64_t)(blockIdx.x & 7) * p.per_xcd;
  const int64_t end = x0 + p.per_xcd < p.items ? x0 + p.per_xcd : p.items;
  const int cus = gridDim.x >> 3;
  int64_t n = x0 + (blockIdx.x >> 3);
  if (n >= end) return;   // same decision in every thread

  auto w_of = [&](const Item& it, int i) __attribute__((always_inline)) -> const uint16_t* {
    return reinterpret_cast<const uint16_t*>(it.kv ? a.wv : a.wk) +
           (((int64_t)(a.l0 + it.ll) * a.H + it.h) * k + i) * (int64_t)(D * D);
  };
  auto x_of = [&](const Item& it, int i) __attribute__((always_inline)) -> const uint16_t* {
    return reinterpret_cast<const uint16_t*>(a.src) +
           (((int64_t)a.idx[it.ll * k + i] * 2 + it.kv) * a.H + it.h) * T * D;
  };
  // token row of block tb of this lane, clamped so that every load is in
  // bounds; a clamped row only feeds its own (discarded) output column
  auto row_of = [&](int64_t t0, int tb) __attribute__((always_inline)) -> int64_t {
    const int64_t t = t0 + 16 * (TB * wave + tb) + row;
    return t < T ? t : T - 1;
  };
  auto load_x = [&](const Item& it, int i, u32x4_t (&x)[TB][S]) __attribute__((always_inline)) {
    const uint16_t* X = x_of(it, i);
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const uint16_t* q = X + row_of(it.t0, tb) * D + 8 * c;
#pragma unroll
      for (int s = 0; s < S; ++s) x[tb][s] = *reinterpret_cast<const u32x4_t*>(q + 32 * s);
    }
  };
  const bool stager = tid < G::PIECES;

  Item cur = item_of(a, p, n);
  u32x4_t nx[TB][S];
  uint4 wr[4];
  float2 cs[TB][G::PL];
  int64_t cs_t0 = -1;
  if (stager) load_piece<D>(w_of(cur, 0), tid, wr);
  load_x(cur, 0, nx);
  if (stager) store_piece<D, G::ROWB>(smem, tid, wr);
  // positions one and two source layers ahead; past the end they repeat the last
  Item i1 = cur;
  int k1 = 0;
  int64_t n1 = n;
  auto advance = [&](Item& it, int& i, int64_t& m) __attribute__((always_inline)) {
    if (i + 1 < k) {
      ++i;
    } else if (m + cus < end) {
      m += cus;
      i = 0;
      it = item_of(a, p, m);
    }
  };
  advance(i1, k1, n1);
  if (stager) load_piece<D>(w_of(i1, k1), tid, wr);
  __syncthreads();

  int st = 0;
  for (; n < end; n += cus) {
    if (cur.kv == 0 && cs_t0 != cur.t0) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) load_planes<D, STYLE>(a.cs_src, row_of(cur.t0, tb), c, cs[tb]);
      cs_t0 = cur.t0;
    }
    f32x4_t acc[TB][NB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[tb][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    for (int i = 0; i < k; ++i) {
      u32x4_t x[TB][S];
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int s = 0; s < S; ++s) x[tb][s] = nx[tb][s];
      // the next source layer's map into the stage of the previous one, then
      // the loads after it
      if (stager) store_piece<D, G::ROWB>(smem + (st ^ 1) * G::SLOTB, tid, wr);
      load_x(i1, k1, nx);
      advance(i1, k1, n1);
      if (stager) load_piece<D>(w_of(i1, k1), tid, wr);
      __builtin_amdgcn_sched_barrier(0);
      if (cur.kv == 0) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) strip_row<D, STYLE>(x[tb], cs[tb]);
      }
      const char* wl = smem + st * G::SLOTB + row * G::ROWB;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const char* ws = wl + 16 * chunk_pos<D>(4 * s + c, row);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const bf16x8_t wa = *reinterpret_cast<const bf16x8_t*>(ws + b * 16 * G::ROWB);
#pragma unroll
          for (int tb = 0; tb < TB; ++tb)
            acc[tb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                wa, __builtin_bit_cast(bf16x8_t, x[tb][s]), acc[tb][b], 0, 0, 0);
        }
      }
      __syncthreads();
      st ^= 1;
    }

    const int64_t lh = (int64_t)(a.l0 + cur.ll) * a.H + cur.h;
    const uint16_t* bias = reinterpret_cast<const uint16_t*>(cur.kv ? a.bv : a.bk);
    if (bias != nullptr) bias += lh * D;
    uint16_t* out = reinterpret_cast<uint16_t*>(a.tgt) +
                    (((int64_t)(a.l0 + cur.ll) * 2 + cur.kv) * a.H + cur.h) * a.tgt_rows * D;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int64_t t = row_of(cur.t0, tb);
      const int64_t orow = SLOTS ? (int64_t)a.slots[t] : t;
      const bool store = cur.t0 + 16 * (TB * wave + tb) + row < T &&
                         (!SLOTS || (orow >= 0 && orow < a.tgt_rows));
      if (cur.kv == 0) finish_row<D, STYLE, true>(acc[tb], bias, a.cs_tgt, t, c, out + orow * D, store);
      else finish_row<D, STYLE, false>(acc[tb], bias, a.cs_tgt, t, c, out + orow * D, store);
    }
    if (n + cus < end) cur = item_of(a, p, n + cus);
  }
}

template <int D, int STYLE>
hipError_t launch_streamed(const MapArgs& a, hipStream_t stream) {
  TilePlan p;
  p.len = BT;
  p.tiles = (int32_t)(((int64_t)a.T + BT - 1) / BT);
  p.items = (int64_t)a.H * 2 * p.tiles * a.nl;
  p.per_xcd = (p.items + 7) / 8;
  if (a.slots != nullptr)
    hipLaunchKernelGGL((map_kernel<D, STYLE, true>), dim3(256), dim3(NTHR), 0, stream, a, p);
  else
    hipLaunchKernelGGL((map_kernel<D, STYLE, false>), dim3(256), dim3(NTHR), 0, stream, a, p);
  return hipGetLastError();
}

// ------------------------------------------------------- resident maps

constexpr int RES_K = 8;       // source layers whose maps stay in LDS (head dimension 64)

// One workgroup per (head, token range, K|V, target layer): the task's whole
// map in LDS (8 KB per source layer), then the range's tiles without a barrier;
// two workgroups a CU.  Bound by the row reads and stores: 16 -> 28 layers, 8
// heads, k = 4, T = 8192: 0.415 ms (1.8 TB/s of the bytes it cannot do
// without), 0.667 ms with the 64-token tiles that restaged the map per tile.
template <int D, int STYLE, bool SLOTS>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(4, 4)))
void map_resident_kernel(const MapArgs a, const TilePlan p) {
  using G = TileGeo<D>;
  constexpr int S = G::S, NB = G::NB;
  extern __shared__ __attribute__((aligned(256))) char wsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane >> 4, row = lane & 15;
  const int64_t T = a.T;
  const int k = a.k;
  const int64_t n = (int64_t)(blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
  if ((int64_t)(blockIdx.x >> 3) >= p.per_xcd || n >= p.items) return;
  Item it = item_of(a, p, n);
  const int64_t t_begin = it.t0;
  const int64_t t_end = t_begin + p.len < T ? t_begin + p.len : T;
  const int64_t lh = (int64_t)(a.l0 + it.ll) * a.H + it.h;

  {
    const uint16_t* w = reinterpret_cast<const uint16_t*>(it.kv ? a.wv : a.wk) + lh * k * (int64_t)(D * D);
    for (int m = tid; m < k * G::PIECES; m += NTHR) {
      const int i = m / G::PIECES, q = m % G::PIECES;
      uint4 r[4];
      load_piece<D>(w + i * (int64_t)(D * D), q, r);
      store_piece<D, G::ROWB>(wsm + i * G::SLOTB, q, r);
    }
  }
  const uint16_t* bias = reinterpret_cast<const uint16_t*>(it.kv ? a.bv : a.bk);
  if (bias != nullptr) bias += lh * D;
  uint16_t* out = reinterpret_cast<uint16_t*>(a.tgt) +
                  (((int64_t)(a.l0 + it.ll) * 2 + it.kv) * a.H + it.h) * a.tgt_rows * D;
  auto row_of = [&](int64_t t0, int tb) __attribute__((always_inline)) -> int64_t {
    const int64_t t = t0 + 16 * (TB * wave + tb) + row;
    return t < t_end ? t : t_end - 1;
  };
  auto load_x = [&](int i, int64_t t0, u32x4_t (&x)[TB][S]) __attribute__((always_inline)) {
    const uint16_t* X = reinterpret_cast<const uint16_t*>(a.src) +
                        (((int64_t)a.idx[it.ll * k + i] * 2 + it.kv) * a.H + it.h) * T * D;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const uint16_t* q = X + row_of(t0, tb) * D + 8 * c;
#pragma unroll
      for (int s = 0; s < S; ++s) x[tb][s] = *reinterpret_cast<const u32x4_t*>(q + 32 * s);
    }
  };

  u32x4_t nx[TB][S];
  load_x(0, t_begin, nx);
  __syncthreads();

  auto sweep = [&](auto keys) __attribute__((always_inline)) {
    constexpr bool KEYS = decltype(keys)::value;
    for (int64_t t0 = t_begin; t0 < t_end; t0 += BT) {
      float2 cs[TB][G::PL];
      if (KEYS) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) load_planes<D, STYLE>(a.cs_src, row_of(t0, tb), c, cs[tb]);
      }
      f32x4_t acc[TB][NB];
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[tb][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
      for (int i = 0; i < k; ++i) {
        u32x4_t x[TB][S];
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
          for (int s = 0; s < S; ++s) x[tb][s] = nx[tb][s];
        // the next source layer's rows, or the next tile's first (the last
        // tile loads its own again)
        if (i + 1 < k) load_x(i + 1, t0, nx);
        else load_x(0, t0 + BT < t_end ? t0 + BT : t0, nx);
        __builtin_amdgcn_sched_barrier(0);
        if (KEYS) {
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) strip_row<D, STYLE>(x[tb], cs[tb]);
        }
        const char* wl = wsm + i * G::SLOTB + row * G::ROWB;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const char* ws = wl + 16 * chunk_pos<D>(4 * s + c, row);
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const bf16x8_t wa = *reinterpret_cast<const bf16x8_t*>(ws + b * 16 * G::ROWB);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb)
              acc[tb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  wa, __builtin_bit_cast(bf16x8_t, x[tb][s]), acc[tb][b], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) {
        const int64_t t = row_of(t0, tb);
        const int64_t orow = SLOTS ? (int64_t)a.slots[t] : t;
        const bool store = t0 + 16 * (TB * wave + tb) + row < t_end &&
                           (!SLOTS || (orow >= 0 && orow < a.tgt_rows));
        finish_row<D, STYLE, KEYS>(acc[tb], bias, a.cs_tgt, t, c, out + orow * D, store);
      }
    }
  };
  if (it.kv == 0) sweep(std::true_type{});
  else sweep(std::false_type{});
}

template <int D, int STYLE>
hipError_t launch_resident(const MapArgs& a, hipStream_t stream) {
  // Token range of a workgroup: long enough to amortise staging the map (at
  // 1024 tokens it is 6% of the rows read), short enough for four rounds of
  // the 512 workgroups that fit the chip.
  const int64_t tasks = (int64_t)a.H * 2 * a.nl;
  int64_t len = (tasks * a.T / 2048 + BT - 1) / BT * BT;
  len = len < BT ? BT : len > 1024 ? 1024 : len;
  TilePlan p;
  p.len = (int32_t)len;
  p.tiles = (int32_t)(((int64_t)a.T + len - 1) / len);
  p.items = tasks * p.tiles;
  p.per_xcd = (p.items + 7) / 8;
  if (p.per_xcd * 8 > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(p.per_xcd * 8));
  const size_t lds = (size_t)a.k * TileGeo<D>::SLOTB;
  if (a.slots != nullptr)
    hipLaunchKernelGGL((map_resident_kernel<D, STYLE, true>), grid, dim3(NTHR), lds, stream, a, p);
  else
    hipLaunchKernelGGL((map_resident_kernel<D, STYLE, false>), grid, dim3(NTHR), lds, stream, a, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_map_tile(const MapArgs& a, int d, int style, hipStream_t stream) {
  if (a.T == 0 || a.nl == 0) return hipSuccess;
  if (d == 128) return style == 0 ? launch_streamed<128, 0>(a, stream) : launch_streamed<128, 1>(a, stream);
  if (d == 64 && a.k <= RES_K)
    return style == 0 ? launch_resident<64, 0>(a, stream) : launch_resident<64, 1>(a, stream);
  if (d == 64) return style == 0 ? launch_streamed<64, 0>(a, stream) : launch_streamed<64, 1>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace kvx
