// Map kernel for bf16 calls outside the packed-map kernels: more than four
// source layers, or head dimension 64.
//
// One workgroup per CU works through its items, each one (target layer, head,
// K|V) task on a tile of 256 tokens, 8 waves of 32 tokens, as C^T = W^T X^T on
// v_mfma_f32_16x16x32_bf16 (Eq. ridge_kv, Sec. 3.1).  Rows and maps stream
// through LDS in positions of 64 reduction channels (two steps, whole RoPE
// planes of a source layer), loaded straight into LDS three positions ahead,
// across items.  Rows are private to their wave, which strips the source RoPE
// from its fragments (Sec. 3.3, fp32 coefficients, one rounding) and feeds each
// to all D / 16 output blocks.  W is read as given: transposed LDS reads give
// the map fragments.  Outputs go through LDS, so that stores cover whole rows.
//
// Why rows go through LDS: fragments loaded straight into registers (16 rows x
// 64 bytes per instruction, neighbouring lanes in different rows) run at 18
// bytes per clock and CU even out of L2 (9.7 TB/s over the chip); with 64
// contiguous bytes per four neighbouring lanes the same loads reach 33 TB/s.
// Bound at k = 8 by traffic beyond L2 (14.7 GB a launch, 4.3 TB/s: the maps are
// read again for every 256 tokens), the key strip and the waits around the position
// barrier (matrix pipe busy about 30%).  Qwen3-14B->32B shapes, k = 8, T = 8191:
// 3.43 ms (0.64 PFLOP/s; 4.35 ms with rows straight into registers and barriers per
// source layer, 16.95 ms with 64-token tiles staged without a pipeline); one layer
// of it, 512 tokens 29 us and 2048 tokens 33 us (50 and 75 with 64-token tiles); head
// dimension 64, 16 -> 28 layers, k = 4, T = 8192: 0.368 ms (0.415 and 0.667).
//
// Operand layout: lane L = 16 c + r supplies map row / token r and reduction
// indices 8 c .. 8 c + 7 of a 32-wide step.  Map row 16 b + 4 c + i holds output
// channel 16 b + 4 c + i: blocks b and b + D / 32 (half-split) or neighbouring
// elements (interleaved) hold the members of a RoPE plane in one lane.
#include "kvx_bf16.h"
#include "kvx_internal.h"
#include "kvx_wload.h"

#include <type_traits>

namespace kvx {
namespace {

constexpr int NTHR = 512;      // threads per workgroup
constexpr int TB = 2;          // 16-token blocks per wave
constexpr int WT = 16 * TB;    // tokens per wave
constexpr int BT = 8 * WT;     // tokens per tile

template <int D>
struct TileGeo {
  static constexpr int S = D / 32;             // reduction steps per source layer
  static constexpr int PPS = S / 2;            // positions per source layer
  static constexpr int NB = D / 16;            // output blocks
  static constexpr int HALF = D / 2;
  static constexpr int PL = D / 8;             // RoPE planes of a token in a lane
  static constexpr int ROWB = 2 * D;           // bytes of a row of rows, maps and outputs
  static constexpr int XB = WT * 128;          // a wave's rows of one position
  static constexpr int WB = 64 * ROWB;         // the map rows of one position
  static constexpr int XD = XB / 1024;         // loads of a wave per position: rows
  static constexpr int WD = WB / 8192;         // and maps
  static constexpr int NX = 3, NW = 4;         // positions in LDS: rows and maps
  static constexpr int LDS = NX * 8 * XB + NW * WB;
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

// Place of the 32-byte runs of map row m (see the map loads): rows 0..3 and
// 8..11 of a fragment read differ in it (D = 64: beside the row's own half of
// the banks).
template <int D>
__device__ __forceinline__ int map_swz(int m) {
  return D == 128 ? (m & 3) + 4 * ((m >> 3) & 1) : ((m >> 1) & 1) + 2 * ((m >> 3) & 1);
}

// Strip the source RoPE from a token's fragments of position X.
template <int D, int STYLE, int X>
__device__ __forceinline__ void strip_pos(u32x4_t& x0, u32x4_t& x1, const float2 (&cs)[TileGeo<D>::PL]) {
  constexpr int S = TileGeo<D>::S;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float u0 = lo_bf16(x0[w]), u1 = hi_bf16(x0[w]), v0 = lo_bf16(x1[w]), v1 = hi_bf16(x1[w]);
    if (STYLE == 0) {
      rot_inv32(u0, v0, cs[8 * X + 2 * w]);
      rot_inv32(u1, v1, cs[8 * X + 2 * w + 1]);
    } else {
      rot_inv32(u0, u1, cs[4 * X + w]);
      rot_inv32(v0, v1, cs[4 * (X + S / 2) + w]);
    }
    x0[w] = pack2(u0, u1);
    x1[w] = pack2(v0, v1);
  }
}

// Bias, target RoPE (keys) and rounding of one token's outputs: channels
// 16 b + 4 c .. + 3 in o[b].
template <int D, int STYLE, bool KEYS>
__device__ __forceinline__ void finish_row(const f32x4_t (&acc)[TileGeo<D>::NB],
                                           const uint16_t* __restrict__ bias,
                                           const float2* __restrict__ table, int64_t t, int c,
                                           uint2 (&o)[TileGeo<D>::NB]) {
  using G = TileGeo<D>;
  constexpr int NB = G::NB;
  float y[NB][4];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) y[b][e] = acc[b][e];
  if (bias != nullptr) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const uint2 v = *reinterpret_cast<const uint2*>(bias + 16 * b + 4 * c);
      y[b][0] += lo_bf16(v.x);
      y[b][1] += hi_bf16(v.x);
      y[b][2] += lo_bf16(v.y);
      y[b][3] += hi_bf16(v.y);
    }
  }
  if (KEYS) {
    // half-split: planes 16 b + 4 c + e of blocks b and b + NB / 2;
    // interleaved: planes 8 b + 2 c + e / 2
    const float4* q = reinterpret_cast<const float4*>(table + t * G::HALF);
    if (STYLE == 0) {
#pragma unroll
      for (int b = 0; b < NB / 2; ++b)
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
          const float4 f = q[8 * b + 2 * c + e / 2];
          rot_fwd32(y[b][e], y[b + NB / 2][e], make_float2(f.x, f.y));
          rot_fwd32(y[b][e + 1], y[b + NB / 2][e + 1], make_float2(f.z, f.w));
        }
    } else {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float4 f = q[4 * b + c];
        rot_fwd32(y[b][0], y[b][1], make_float2(f.x, f.y));
        rot_fwd32(y[b][2], y[b][3], make_float2(f.z, f.w));
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) o[b] = make_uint2(pack2(y[b][0], y[b][1]), pack2(y[b][2], y[b][3]));
}

// The items (head, token group, K|V, tile, target layer; layers fastest) are cut
// into eight contiguous ranges, one per XCD.  The 32 CUs of an XCD then work on
// 32 target layers of one (head, K|V) and tile, whose source rows its L2 holds,
// and the maps that the tiles read again and again are those of keys or of
// values, which the last-level cache holds where it does not hold both (268 MB
// at 64 layers, 8 heads, k = 8; 2% slower with K|V inside the tiles).
// Token groups, 8 / gcd(8, heads) of them, give every XCD keys and values.
struct TilePlan {
  int64_t items, per_xcd;
  int32_t tiles, per_group;   // 256-token tiles, and of a token group
};

struct Item {
  int h, g, kv, t, ll;   // t: tile within token group g
};

__device__ __forceinline__ int group_tiles(const TilePlan& p, int g) {
  const int left = p.tiles - g * p.per_group;
  return left < p.per_group ? left : p.per_group;
}
__device__ __forceinline__ Item item_of(const MapArgs& a, const TilePlan& p, int64_t n) {
  Item it;
  const int64_t per_h = (int64_t)p.tiles * 2 * a.nl;
  it.h = (int)(n / per_h);
  n -= it.h * per_h;
  const int64_t per_g = (int64_t)p.per_group * 2 * a.nl;
  it.g = (int)(n / per_g);
  n -= it.g * per_g;
  const int64_t per_kv = (int64_t)group_tiles(p, it.g) * a.nl;
  it.kv = n >= per_kv;
  n -= it.kv ? per_kv : 0;
  it.t = (int)(n / a.nl);
  it.ll = (int)(n - (int64_t)it.t * a.nl);
  return it;
}
// The item `step` places on (no division: it runs between matrix instructions).
__device__ __forceinline__ void item_add(const MapArgs& a, const TilePlan& p, Item& it, int step) {
  it.ll += step;
  while (it.ll >= a.nl) {
    it.ll -= a.nl;
    if (++it.t == group_tiles(p, it.g)) {
      it.t = 0;
      it.kv ^= 1;
      if (it.kv == 0 && ++it.g * p.per_group >= p.tiles) {
        it.g = 0;
        ++it.h;
      }
    }
  }
}

template <int D, int STYLE, bool SLOTS>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(2, 2)))
void map_tile_kernel(const MapArgs a, const TilePlan p) {
  using G = TileGeo<D>;
  constexpr int NB = G::NB, NX = G::NX, NW = G::NW, ND = G::XD + G::WD;
  static_assert(G::LDS <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char smem[G::LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane >> 4, row = lane & 15;
  const int64_t T = a.T;
  const int k = a.k;

  const int64_t x0 = (int64_t)(blockIdx.x & 7) * p.per_xcd;
  const int64_t end = x0 + p.per_xcd < p.items ? x0 + p.per_xcd : p.items;
  const int cus = gridDim.x >> 3;
  int64_t n = x0 + (blockIdx.x >> 3);
  if (n >= end) return;   // same decision in every thread

  // LDS: [stage][wave] rows, then [stage] maps
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_u32(smem));
  const uint32_t xl = lds0 + (uint32_t)(wave * G::XB), wl = lds0 + (uint32_t)(NX * 8 * G::XB);
  char* const xp = smem + wave * G::XB;

  // Row loads: load g of a position fetches this wave's tokens 8 g .. 8 g + 7,
  // 64 contiguous bytes per four lanes; 16-byte chunk q of token r (0..3: the
  // step's channels, 4..7: those D / 2 later) at position q ^ (r / 2 % 8).
  uint32_t vx[G::XD];
#pragma unroll
  for (int g = 0; g < G::XD; ++g) {
    const int q = (lane & 7) ^ ((4 * g + (lane >> 4)) & 7);
    vx[g] = (uint32_t)((WT * wave + 8 * g + (lane >> 3)) * G::ROWB + (q >> 2) * D + 16 * (q & 3));
  }
  // Map loads: the wave's WD kilobytes of a position's 64 map rows, row m at
  // 2 D m bytes, 16-byte chunk q at position q ^ 2 f(m): the 32 bytes that half
  // a wave reads of each of eight rows fall on distinct banks.
  uint32_t vw[G::WD];
#pragma unroll
  for (int g = 0; g < G::WD; ++g) {
    constexpr int RPL = 1024 / G::ROWB;    // rows per load
    const int m = RPL * (8 * g + wave) + lane / (64 / RPL);
    const int q = (lane % (64 / RPL)) ^ (2 * map_swz<D>(m));
    vw[g] = (uint32_t)(((m & 31) + (m >> 5) * G::HALF) * G::ROWB + 16 * q);
  }
  // A position: source layer i of an item and 64 of its channels.
  struct Pos {
    int64_t n;
    Item it;
    int i, x;
  };
  // The index list is read by words: bytes of the kernel arguments come by
  // vector loads, whose wait drains the loads in flight (k = 8: 4.0 ms).
  const uint32_t* const idx4 = reinterpret_cast<const uint32_t*>(a.idx);
  auto t0_of = [&](const Item& it) __attribute__((always_inline)) -> int64_t {
    return ((int64_t)it.g * p.per_group + it.t) * BT;
  };
  auto issue = [&](const Pos& q, int sx, int sw) __attribute__((always_inline)) {
    const int64_t t0 = t0_of(q.it);
    const int64_t rows = T - t0 < BT ? T - t0 : BT;
    const int at = q.it.ll * k + q.i;
    const int sl = (int)((idx4[at >> 2] >> (8 * (at & 3))) & 0xff);
    const i32x4_t rx = make_rsrc(
        static_cast<const char*>(a.src) + ((((int64_t)sl * 2 + q.it.kv) * a.H + q.it.h) * T + t0) * G::ROWB,
        (uint32_t)rows * G::ROWB);
    const i32x4_t rw = make_rsrc(
        static_cast<const char*>(q.it.kv ? a.wv : a.wk) +
            (((int64_t)(a.l0 + q.it.ll) * a.H + q.it.h) * k + q.i) * (int64_t)(D * G::ROWB),
        D * G::ROWB);
#pragma unroll
    for (int g = 0; g < G::WD; ++g)
      dma16z(wl + (uint32_t)(sw * G::WB + (8 * g + wave) * 1024), vw[g] + (uint32_t)(q.x * 32 * G::ROWB), rw);
#pragma unroll
    for (int g = 0; g < G::XD; ++g)
      dma16z(xl + (uint32_t)(sx * 8 * G::XB + g * 1024), vx[g] + (uint32_t)(q.x * 64), rx);
  };
  // past the end the last position repeats, so that the wait counts hold
  auto advance = [&](Pos& q) __attribute__((always_inline)) {
    if (q.x + 1 < G::PPS) {
      ++q.x;
    } else if (q.i + 1 < k) {
      q.x = 0;
      ++q.i;
    } else if (q.n + cus < end) {
      q.x = q.i = 0;
      q.n += cus;
      item_add(a, p, q.it, cus);
    }
  };
  auto row_of = [&](int64_t t0, int r) __attribute__((always_inline)) -> int64_t {
    const int64_t t = t0 + WT * wave + r;
    return t < T ? t : T - 1;
  };

  Item cur = item_of(a, p, n);
  Pos next = {n, cur, 0, 0};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    issue(next, j, j);
    advance(next);
  }

  // lane offsets of the fragment reads
  uint32_t fx[2];   // rows, by step of the position
#pragma unroll
  for (int e = 0; e < 2; ++e) fx[e] = (uint32_t)(row * 128 + 16 * ((4 * e + c) ^ ((row >> 1) & 7)));
  uint32_t fw[NB];   // maps, by output block
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int m = 8 * c + (row >> 2);
    fw[b] = (uint32_t)(m * G::ROWB + 32 * (b ^ map_swz<D>(m)) + 8 * (row & 3));
  }

  auto read_x = [&](int sx, u32x4_t (&x)[TB][2]) __attribute__((always_inline)) {
    const char* xs = xp + sx * 8 * G::XB;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int e = 0; e < 2; ++e) x[tb][e] = *reinterpret_cast<const u32x4_t*>(xs + tb * 2048 + fx[e]);
  };
  auto read_w = [&](int sw, int e, int b) __attribute__((always_inline)) -> u32x4_t {
    const uint32_t wa = wl + (uint32_t)(sw * G::WB + e * 32 * G::ROWB) + fw[b];
    return tr_read8(wa, wa + 4 * G::ROWB);
  };
  float2 cs[TB][G::PL];
  int64_t cs_t0 = -1;

  // Position p (rows in stage sx, maps in sw).  Its rows and first map
  // fragments are in registers when it starts.  In its middle, this wave's
  // loads of p + 1 have landed (only those of p + 2 may be outstanding) and its
  // reads of p - 1 are long done; with the barrier that holds for every wave:
  // p + 1 can be read, its first reads arriving behind the second half's matrix
  // instructions, and the loads of p + 3 go to the stages of p (rows, the wave's
  // own) and p - 1 (maps).
  // map fragments read ahead: one more spills in the loop whose loads are counted
  constexpr int NPRE = D == 64 ? 4 : STYLE == 0 ? 2 : 1;
  u32x4_t xf[TB][2], wpre[NPRE];
  int sx = 0, sw = 0;
  vm_wait<2 * ND>();
  asm volatile("s_barrier" ::: "memory");
  read_x(0, xf);
#pragma unroll
  for (int b = 0; b < NPRE; ++b) wpre[b] = read_w(0, 0, b);
  for (; n < end; n += cus) {
    const int64_t t0 = t0_of(cur);
    if (cur.kv == 0 && cs_t0 != t0) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) load_planes<D, STYLE>(a.cs_src, row_of(t0, 16 * tb + row), c, cs[tb]);
      cs_t0 = t0;
      // a wait the compiler knows of: without it, it waits at each use, in
      // every position, and drains the loads into LDS
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    }
    f32x4_t acc[TB][NB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[tb][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    auto position = [&](auto xc) __attribute__((always_inline)) {
      constexpr int X = decltype(xc)::value;
      if (cur.kv == 0) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) strip_pos<D, STYLE, X>(xf[tb][0], xf[tb][1], cs[tb]);
      }
      auto mma = [&](const u32x4_t& w, int e, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
          acc[tb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, xf[tb][e]), acc[tb][b], 0, 0, 0);
      };
#pragma unroll
      for (int b = 0; b < NB; ++b) mma(b < NPRE ? wpre[b] : read_w(sw, 0, b), 0, b);
      u32x4_t w1[NPRE];
#pragma unroll
      for (int b = 0; b < NPRE; ++b) w1[b] = read_w(sw, 1, b);
      vm_wait<ND>();
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const int sx1 = sx + 1 == NX ? 0 : sx + 1, sw1 = (sw + 1) & (NW - 1);
      issue(next, sx, (sw + 3) & (NW - 1));
      advance(next);
      u32x4_t xn[TB][2];
      read_x(sx1, xn);
#pragma unroll
      for (int b = 0; b < NPRE; ++b) wpre[b] = read_w(sw1, 0, b);
#pragma unroll
      for (int b = 0; b < NB; ++b) mma(b < NPRE ? w1[b] : read_w(sw, 1, b), 1, b);
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int e = 0; e < 2; ++e) xf[tb][e] = xn[tb][e];
      sx = sx1;
      sw = sw1;
    };
    for (int i = 0; i < k; ++i) {
      position(std::integral_constant<int, 0>{});
      if constexpr (G::PPS == 2) position(std::integral_constant<int, 1>{});
    }

    // The outputs go through the wave's rows of the next position, which are in
    // registers, so that stores cover whole rows.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const int64_t lh = (int64_t)(a.l0 + cur.ll) * a.H + cur.h;
    const uint16_t* bias = reinterpret_cast<const uint16_t*>(cur.kv ? a.bv : a.bk);
    if (bias != nullptr) bias += lh * D;
    char* out = static_cast<char*>(a.tgt) +
                (((int64_t)(a.l0 + cur.ll) * 2 + cur.kv) * a.H + cur.h) * a.tgt_rows * G::ROWB;
    char* os = xp + sx * 8 * G::XB;
    constexpr int CPR = D / 8;              // 16-byte chunks of a row
    constexpr int RPS = 64 / CPR;           // rows per store instruction
    auto swz = [](int r) { return D == 128 ? r & 15 : (r >> 1) & 7; };
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int64_t t = row_of(t0, 16 * tb + row);
      uint2 o[NB];
      if (cur.kv == 0) finish_row<D, STYLE, true>(acc[tb], bias, a.cs_tgt, t, c, o);
      else finish_row<D, STYLE, false>(acc[tb], bias, a.cs_tgt, t, c, o);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        *reinterpret_cast<uint2*>(os + row * G::ROWB + 16 * ((2 * b + (c >> 1)) ^ swz(row)) + 8 * (c & 1)) = o[b];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own writes
#pragma unroll
      for (int g = 0; g < 16 / RPS; ++g) {
        const int r = RPS * g + lane / CPR, q = lane % CPR;
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(os + r * G::ROWB + 16 * q);
        const int64_t tr = t0 + WT * wave + 16 * tb + r;
        const int64_t orow = SLOTS ? (int64_t)a.slots[tr < T ? tr : T - 1] : tr;
        if (tr < T && (!SLOTS || (orow >= 0 && orow < a.tgt_rows)))
          *reinterpret_cast<u32x4_t*>(out + orow * G::ROWB + 16 * (q ^ swz(r))) = v;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // reads done before the next block's writes
    }
    item_add(a, p, cur, cus);
  }
  vm_wait<0>();   // no load may land in LDS after the workgroup has gone
}

template <int D, int STYLE>
hipError_t launch_tile(const MapArgs& a, hipStream_t stream) {
  TilePlan p;
  p.tiles = (int32_t)(((int64_t)a.T + BT - 1) / BT);
  int groups = 8;
  while (groups > 1 && a.H * (groups / 2) % 8 == 0) groups /= 2;
  p.per_group = (p.tiles + groups - 1) / groups;
  p.items = (int64_t)a.H * 2 * p.tiles * a.nl;
  p.per_xcd = (p.items + 7) / 8;
  const dim3 grid((unsigned)(8 * (p.per_xcd < 32 ? p.per_xcd : 32)));
  if (a.slots != nullptr)
    hipLaunchKernelGGL((map_tile_kernel<D, STYLE, true>), grid, dim3(NTHR), 0, stream, a, p);
  else
    hipLaunchKernelGGL((map_tile_kernel<D, STYLE, false>), grid, dim3(NTHR), 0, stream, a, p);
  return hipGetLastError();
}

// Whether a call at d = 64 takes map_short_kernel (64-token workgroups, several on
// a CU) and not the tile kernel: where the latter's rounds of 256 items, each for
// 256 tokens however few there are, cost more than the former's workgroups (with
// interleaved planes 8 of those fit a CU, with half-split ones 6).
// Measured in whole calls, us, map_tile_kernel / map_short_kernel, with caches
// warm where the host does not bound the call, else evicted before (e):
//   k = 1   64 layers, 8 heads     32 tokens  20.6 / 15.4 e    256 tokens  21.9 / 23.9
//           30 layers, 8 heads   1100 tokens  42.2 / 35.7
//           32 layers, 8 heads   2500 tokens  93.5 / 84.6     8192 tokens   284 / 294
//           the same interleaved 2500 tokens  94.0 / 73.4     8192 tokens   287 / 247
//           one layer, 8 heads   4100 tokens  22.1 / 17.5 e
//   k = 2   80 layers, 8 heads     64 tokens  21.9 / 17.1      100 tokens  23.1 / 23.4
//           one layer, 8 heads   4100 tokens  25.9 / 21.1 e
//   k = 4   80 layers, 8 heads     64 tokens  29.3 / 23.0      100 tokens  30.4 / 36.4
//           16 layers, 8 heads     64 tokens  18.4 / 21.0 e
//   k = 8   64 layers, 8 heads     64 tokens  35.9 / 30.8      100 tokens  36.7 / 52.6
bool short_call(const MapArgs& a, int style) {
  const int64_t tasks = (int64_t)a.nl * a.H * 2, T = a.T;
  const int64_t tiles = tasks * ((T + 63) / 64);
  const int64_t rounds = (tasks * ((T + BT - 1) / BT) + 255) / 256;
  if (a.k == 1) {
    const int64_t most = style == 1 ? (tasks <= 640 ? 65536 : 36000) : tasks <= 512 ? 32000 : tasks <= 832 ? 20000 : 0;
    return tiles <= 700 * rounds || tiles <= most;
  }
  if (a.k == 2) {
    const int64_t most = style == 1 ? (tasks <= 128 ? 3000 : 1700) : 1280, per = style == 1 ? 550 : 400;
    return tiles <= most || tiles <= per * rounds || (tasks <= 32 && tiles <= 4096);
  }
  return T <= 64 && tasks > 256;
}

}  // namespace

hipError_t launch_map_tile(const MapArgs& a, int d, int style, hipStream_t stream) {
  if (a.T == 0 || a.nl == 0) return hipSuccess;
  if (d == 64 && short_call(a, style)) return launch_map_short(a, style, stream);
  if (d == 128) return style == 0 ? launch_tile<128, 0>(a, stream) : launch_tile<128, 1>(a, stream);
  if (d == 64) return style == 0 ? launch_tile<64, 0>(a, stream) : launch_tile<64, 1>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace kvx
