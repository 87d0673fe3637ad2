// K1, direct variant: the fused output-layer projection for states of fewer
// than 32 elements, vocabularies narrower than a tile and the widest ones
// (direct_shape), in bf16 and in float32.
//
// Operands go from memory straight into the matrix instructions' registers:
// with so few states there is nothing to stage ahead for, and a tile costs
// what its epilogue costs (bf16 640 x 16 x 30,001: 32 us a step against 239 of
// 32 x 128 tiles staged element by element, 76 of the earlier guarded staging;
// 3,000 x 1,024 x 96 in float32 40 against 63 and 50).  Every load stays in bounds by its own address (a
// state past H is read at the last one and taken as zero in both operands, a
// word past V at the last one and masked by the epilogue), so no shape needs a
// special case.  float32 uses the float32 matrix instruction, whose products
// are exact and which takes infinities as they are.
#pragma once

#include "k1_common.hpp"

namespace kb {

typedef uint32_t stage16 __attribute__((ext_vector_type(4)));
#define KB_GLOBAL __attribute__((address_space(1)))

// Element types of the register-staged and the direct kernels.
template <bool F32>
struct StageTy;
template <>
struct StageTy<false> {
  using E = uint16_t;
  typedef stage16 V16 __attribute__((aligned(2)));  // 16 bytes at any element
  static constexpr int EPC = 8, PIECES = 1, PRODS = 1;
};
template <>
struct StageTy<true> {
  using E = float;
  typedef stage16 V16 __attribute__((aligned(4)));
  static constexpr int EPC = 4, PIECES = 3, PRODS = 6;
};

// acc = the products of the tile of L::BV words from v0 and the rows from h0,
// this wave's blocks of it.  16 states at a time; a lane holds 8 of them, of
// one word and of one row per block: bf16 8 half + j, float32 8 (j / 4) + 4
// half + j % 4 (so that a row's 16 bytes are consecutive states; step j of the
// products pairs the same states of both operands).  AHEAD: the next 32 states are on
// their way during the products of these.
template <class L, bool F32, bool AHEAD>
__device__ __forceinline__ void direct_products(f32x16 (&acc)[L::WV][L::WH], const K1Args& a, int h0, int v0) {
  using T = StageTy<F32>;
  using E = typename T::E;
  using GP = const KB_GLOBAL E*;
  constexpr int WV = L::WV, WH = L::WH;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave % L::NWV, wh = wave / L::NWV;
  const int half = lane >> 5, col = lane & 31;
  const int H = a.H;
  const size_t V = a.V;
  constexpr int HS = F32 ? 4 : 8;  // states between the two halves' first
  auto state = [](int j) { return F32 ? 8 * (j >> 2) + (j & 3) : j; };  // of the first half

  GP wp[WV], hp[WH];
#pragma unroll
  for (int vb = 0; vb < WV; ++vb) {
    const uint32_t v = min((uint32_t)v0 + (wv * WV + vb) * 32 + col, (uint32_t)a.V - 1);
    wp[vb] = (GP)(const KB_GLOBAL void*)a.W + v;
  }
#pragma unroll
  for (int hb = 0; hb < WH; ++hb) {
    const int n = min(h0 + (wh * WH + hb) * 32 + col, a.N - 1);
    hp[hb] = (GP)(const KB_GLOBAL void*)a.h + (size_t)n * H;
  }
  struct Chunk {
    E w[WV][8], h[WH][8];
  };
  // 16 whole states from k0
  auto load = [&](int k0, Chunk& c) __attribute__((always_inline)) {
    const size_t kl = k0 + HS * half;
#pragma unroll
    for (int hb = 0; hb < WH; ++hb)
#pragma unroll
      for (int q = 0; q < 8; q += T::EPC) {
        const stage16 x = *(const KB_GLOBAL typename T::V16*)(hp[hb] + kl + state(q));
        __builtin_memcpy(&c.h[hb][q], &x, 16);
      }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int vb = 0; vb < WV; ++vb) c.w[vb][j] = wp[vb][(kl + state(j)) * V];
  };
  auto load_tail = [&](int k0, Chunk& c) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + HS * half + state(j), kk = min(k, H - 1);
#pragma unroll
      for (int hb = 0; hb < WH; ++hb) {
        const E x = hp[hb][kk];
        c.h[hb][j] = k < H ? x : E(0);
      }
#pragma unroll
      for (int vb = 0; vb < WV; ++vb) {
        const E x = wp[vb][(size_t)kk * V];
        c.w[vb][j] = k < H ? x : E(0);
      }
    }
  };
  auto products = [&](const Chunk& c) __attribute__((always_inline)) {
    if constexpr (F32) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int vb = 0; vb < WV; ++vb)
#pragma unroll
          for (int hb = 0; hb < WH; ++hb)
            acc[vb][hb] = __builtin_amdgcn_mfma_f32_32x32x2f32(c.w[vb][j], c.h[hb][j], acc[vb][hb], 0, 0, 0);
    } else {
      bf16x8 fb[WH];
#pragma unroll
      for (int hb = 0; hb < WH; ++hb) __builtin_memcpy(&fb[hb], c.h[hb], 16);
#pragma unroll
      for (int vb = 0; vb < WV; ++vb) {
        bf16x8 fa;
        __builtin_memcpy(&fa, c.w[vb], 16);
#pragma unroll
        for (int hb = 0; hb < WH; ++hb)
          acc[vb][hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb[hb], acc[vb][hb], 0, 0, 0);
      }
    }
  };

#pragma unroll
  for (int vb = 0; vb < WV; ++vb)
#pragma unroll
    for (int hb = 0; hb < WH; ++hb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[vb][hb][r] = 0.f;
  const int whole = H / 16;
  if constexpr (!AHEAD) {
    Chunk c;
    if (H % 16 != 0) {
      load_tail(16 * whole, c);
      products(c);
    }
    for (int i = 0; i < whole; ++i) {
      load(16 * i, c);
      products(c);
    }
    return;
  }
  Chunk c0, c1, c2;
  auto chunk = [&](int c) { return 16 * min(c, whole - 1); };  // past the last: that one again, unused
  if (H % 16 != 0) load_tail(16 * whole, c0);
  if (whole > 0) load(0, c1);
  if (whole > 1) load(16, c2);
  if (H % 16 != 0) products(c0);
  if (whole == 1) {  // (in the loop it would be loaded three times)
    products(c1);
    return;
  }
  for (int c = 0; c < whole; c += 3) {
    load(chunk(c + 2), c0);
    products(c1);
    if (c + 1 >= whole) break;
    load(chunk(c + 3), c1);
    products(c2);
    if (c + 2 >= whole) break;
    load(chunk(c + 4), c2);
    products(c0);
  }
}

// A whole cell: every tile of the split against the rows from h0.
template <class L, int KC, bool F32, bool AHEAD>
__device__ __forceinline__ void direct_cell(SmemEpi<L, KC>& ep, const K1Args& a, int h0, int split) {
  constexpr int BV = L::BV;
  const int tid = threadIdx.x;
  Epilogue<L, KC> epi;
  epi.init(ep, a.k);
  // the split's tiles are split, split + P, split + 2 P, ... (as in the other kernels)
  for (int vt = split; vt < a.n_vtiles; vt += a.P) {
    const int v0 = vt * BV;
    uint32_t tg[L::WH];
    epi.load_shared_thr(a, h0, tg);
    f32x16 acc[L::WV][L::WH];
    direct_products<L, F32, AHEAD>(acc, a, h0, v0);
    // (the tile before has been through with its bias since its first barrier)
    for (int i = tid; i < BV; i += 256) ep.bias[0][i] = a.b[min((uint32_t)v0 + i, (uint32_t)a.V - 1)];
    lds_barrier();
    epi.tile(acc, ep, a, h0, v0, v0, vt == split, tg, ep.bias[0]);
  }
  epi.finish(ep, a, h0, split);
}

template <class L, int KC, bool F32>
__global__ __launch_bounds__(256) void k1_direct(K1Args a) {
  __shared__ __attribute__((aligned(16))) SmemEpi<L, KC> ep;
  int row_tile, split;
  k1_cell(a, blockIdx.x, row_tile, split);
  direct_cell<L, KC, F32, true>(ep, a, row_tile * L::BH, split);
}

template <class L, bool F32>
hipError_t launch_k1_direct(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  const dim3 block(256);
  switch (kc) {
    case 4: k1_direct<L, 4, F32><<<grid, block, 0, st>>>(a); break;
    case 8: k1_direct<L, 8, F32><<<grid, block, 0, st>>>(a); break;
    case 12: k1_direct<L, 12, F32><<<grid, block, 0, st>>>(a); break;
    case 16: k1_direct<L, 16, F32><<<grid, block, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace kb
