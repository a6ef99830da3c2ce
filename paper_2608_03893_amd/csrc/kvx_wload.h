// Maps read as given ([k * 128, 128] row-major, the reduction index in the
// rows) into matrix operands, which need the reduction index contiguous per
// output channel (device code only).
#pragma once

#include "kvx_asm.h"

namespace kvx {
namespace {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wint-to-pointer-cast"   // LDS addresses; the host pass sees wider pointers

// One 4 x 8 piece of a source layer's map: input rows 4 kg .. + 3, output
// channels 8 ng .. + 7.  The lanes of half a wave take 8 kg and 4 ng, whose
// 8-byte LDS writes of one channel fall on distinct banks; the wave reads
// whole 128-byte lines.
__device__ __forceinline__ void piece_of(int n, int& kg, int& ng) {
  kg = (n & 7) | ((n >> 7) << 3);
  ng = ((n >> 3) & 3) | (((n >> 5) & 3) << 2);
}

__device__ __forceinline__ void load_piece(const uint16_t* __restrict__ w, int n, uint4 (&r)[4]) {
  int kg, ng;
  piece_of(n, kg, ng);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    r[j] = *reinterpret_cast<const uint4*>(w + (4 * kg + j) * 128 + 8 * ng);
}

// Into LDS at row stride ROWB, 16-byte chunk q of map row rho at position q ^
// (rho % 16): the 16 rows of a fragment read fall on distinct banks.
template <int ROWB>
__device__ __forceinline__ void store_piece(char* lds, int n, const uint4 (&r)[4]) {
  int kg, ng;
  piece_of(n, kg, ng);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int rho = 16 * (2 * (ng >> 2) + (e >> 2)) + 4 * (ng & 3) + (e & 3);
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (&r[j].x)[e >> 1];
    const uint2 v = make_uint2(__builtin_amdgcn_perm(w[1], w[0], sel),
                               __builtin_amdgcn_perm(w[3], w[2], sel));
    *reinterpret_cast<uint2*>(lds + rho * ROWB + 16 * ((kg >> 1) ^ (rho & 15)) + 8 * (kg & 1)) = v;
  }
}

constexpr int kWStep = 8192;          // bytes of one reduction step: 32 map rows
constexpr int kWRing = 4 * kWStep;    // staging bytes of a wave

// Eight consecutive reduction indices of this lane's channel: two transposed
// reads of four map rows each.  In each group of 16 lanes, lane i addresses 8
// bytes (four channels) of row i / 4 and receives channel i's four rows.
__device__ __forceinline__ u32x4_t tr_read8(uint32_t a0, uint32_t a1) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v0 = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a0));
  const u32x2 v1 = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)a1));
  return (u32x4_t){v0[0], v0[1], v1[0], v1[1]};
}

// Keep a map fragment in AGPRs from here on.
__device__ __forceinline__ void pin_a(u32x4_t& v) { asm volatile("" : "+a"(v)); }

// Map rows of reduction steps Z0 .. Z0 + ZH - 1 (four per source layer) into
// the A-fragments wf[b][z] of one wave: lane (c, row) takes output channel
// 32 (b / 2) + 8 (row / 4) + 4 (b % 2) + row % 4 and, of step s of a source
// layer, rows 32 s + 8 c .. + 7, or (SPLIT) 16 s + 4 c .. + 3 and 64 + 16 s +
// 4 c .. + 3.  The rows go straight into this wave's staging ring in LDS,
// four steps ahead, with 16-byte chunk q of a row at position q ^ 4 (row % 4),
// so that the four rows of a transposed read fall on distinct banks; a
// ds_read_b64_tr_b16 then gives each lane four consecutive rows of its channel.
// w: the task's map (k * 32 KB, map_bytes in all).
// One pass over the map instead of the three of a separate packing kernel (read,
// write, read): 40 target layers of 8 heads at k = 4 (84 MB), 333 tokens, 107
// us with the packing kernel (34 us of it its own).
template <bool SPLIT, int Z0, int ZH>
__device__ __forceinline__ void load_map_raw(u32x4_t (&wf)[8][ZH], const void* w, uint32_t map_bytes,
                                             uint32_t lds, int lane) {
  // an opaque copy: the per-lane offsets are rebuilt here, not kept live
  asm volatile("" : "+v"(lane));
  const i32x4_t rs = make_rsrc(w, map_bytes);
  const int r4 = lane >> 4;
  const uint32_t vo = (uint32_t)(r4 * 256 + 16 * ((lane & 15) ^ (4 * r4)));
  // load n of step z fetches its staged rows 4 n .. 4 n + 3
  auto stage = [&](int z) __attribute__((always_inline)) {
    const int u = (Z0 + z) >> 2, s = (Z0 + z) & 3;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int r0 = SPLIT ? (n < 4 ? 16 * s + 4 * n : 64 + 16 * s + 4 * (n - 4)) : 32 * s + 4 * n;
      dma16z(lds + (uint32_t)((z & 3) * kWStep + n * 1024), vo + (uint32_t)((u * 128 + r0) * 256), rs);
    }
  };
  const int i = lane & 15, c = lane >> 4;
  uint32_t pos[4];   // by b / 2
#pragma unroll
  for (int b2 = 0; b2 < 4; ++b2)
    pos[b2] = lds + (uint32_t)(((SPLIT ? 4 : 8) * c + (i >> 2)) * 256 +
                               16 * (4 * (b2 ^ (i >> 2)) + (i & 3)));
#pragma unroll
  for (int z = 0; z < 4 && z < ZH; ++z) stage(z);
#pragma unroll
  for (int z = 0; z < ZH; ++z) {
    // step z has landed: only the loads of the (at most three) steps after it
    // may be outstanding
    constexpr int L = 8;
    switch (ZH - 1 - z < 3 ? ZH - 1 - z : 3) {
      case 0: vm_wait<0>(); break;
      case 1: vm_wait<L>(); break;
      case 2: vm_wait<2 * L>(); break;
      default: vm_wait<3 * L>(); break;
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint32_t at = pos[b >> 1] + (uint32_t)((z & 3) * kWStep + 8 * (b & 1));
      wf[b][z] = tr_read8(at, at + (SPLIT ? 4096 : 1024));
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) pin_a(wf[b][z]);
    if (z + 4 < ZH) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the step's reads, before its ring place is refilled
      stage(z + 4);
    }
  }
}

// The fragments of load_map_raw into the task's packed image: [128 map rows
// 16 b + row][k * 128 reduction columns] bf16, 16-byte chunk u of a row at
// chunk position u ^ row.
template <bool SPLIT, int Z0, int ZH, int K>
__device__ __forceinline__ void store_map_image(const u32x4_t (&wf)[8][ZH], uint16_t* img, int lane) {
  asm volatile("" : "+v"(lane));
  const int row = lane & 15, c = lane >> 4;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    uint16_t* r0 = img + (int64_t)(16 * b + row) * (K * 128);
#pragma unroll
    for (int z = 0; z < ZH; ++z) {
      const int u = (Z0 + z) >> 2, s = (Z0 + z) & 3;
      if (SPLIT) {
        const int q1 = 16 * u + 2 * s + (c >> 1);
        *reinterpret_cast<uint2*>(r0 + 8 * (q1 ^ row) + 4 * (c & 1)) = make_uint2(wf[b][z][0], wf[b][z][1]);
        *reinterpret_cast<uint2*>(r0 + 8 * ((q1 + 8) ^ row) + 4 * (c & 1)) = make_uint2(wf[b][z][2], wf[b][z][3]);
      } else {
        *reinterpret_cast<u32x4_t*>(r0 + 8 * ((4 * (Z0 + z) + c) ^ row)) = wf[b][z];
      }
    }
  }
}

#pragma clang diagnostic pop

}  // namespace
}  // namespace kvx
