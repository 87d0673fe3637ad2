// K1, register-staged variant: the fused output-layer projection for shapes of
// every alignment, in bf16 and in float32, all on the bf16 matrix cores.
//
// Operands go global -> registers -> LDS -> fragments, each step one or more
// stages ahead of the products:
//   * 16-byte loads at the elements' own alignment (rows of an odd V or H
//     start anywhere), in registers for the next NSET stages.  No load needs a
//     guard: the last stage of an H that is no multiple of a stage starts
//     early enough to end at H, and its states that earlier stages have had
//     are made zero in h; the last tile of a ragged V starts early enough to
//     end at V, and the epilogue masks the words that the tile before has had.
//     (H below a stage, V below a tile or beyond 2^25: the direct kernel);
//   * a stage in LDS is GROUPS groups of 16 states.  bf16: 32 states, two
//     groups.  float32: 16 states (the smallest tile 32), three groups for
//     each 16, the pieces of the split below.  W keeps its V-contiguous rows
//     (16-byte chunks XOR-swizzled by the row, fragments through the transpose
//     read ds_read_b64_tr_b16); an h row holds its groups side by side, padded
//     so that 16 rows' fragments fall on distinct banks;
//   * two LDS buffers: the fragments of stage g + 1 are read, and stage g + 2
//     is written to the buffer that stage g left, between the products of
//     stage g, so a stage has one barrier and waits for nothing it has just
//     asked for.
//
// float32: each operand is split into three bf16 pieces (8 + 8 + 8 significant
// bits, the first two rounded to nearest, the third what is left), whose sum
// is the operand exactly from 2^-109 up; below, where the third piece nears
// bf16's smallest subnormal of 2^-133, it is off by up to that.  A product
// is the six piece products of weight 2^-16 and above, each exact, accumulated
// in float32.  The three left out are below 2^-24 of the product together,
// with signs that do not lean either way.  Against 64 bits, relative to the
// root of the sum of squares of the products, the error is 2.6e-8 up to 16
// states (at most 1.5e-7), where the float32 matrix instruction, which rounds
// its sum every two states, has 2.5e-8 for one or two (at most 6e-8 and 8e-8),
// 3.1e-8 for four, 5.4e-8 (4.0e-7) for 16: no less precise from three states
// on.  (A first piece cut off, not rounded, left out up to 2^-22: 3.4e-8, at
// most 2.4e-7.)  An operand that rounds to infinity, within 2^-9 of FLT_MAX,
// counts as infinite below.  Six bf16 products of 32 cycles replace eight
// float32 ones of 64.
#pragma once

#include <type_traits>

#include "k1_direct.hpp"

namespace kb {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// (W piece, h piece) of product p
__device__ constexpr int prod_w(int p) {
  constexpr int w[6] = {2, 0, 1, 1, 0, 0};
  return w[p];
}
__device__ constexpr int prod_h(int p) {
  constexpr int h[6] = {0, 2, 1, 0, 1, 0};
  return h[p];
}

// The three bf16 pieces of two floats, each pair packed, in two parts of five
// and six instructions: the first piece and what it leaves, then the other two.
__device__ __forceinline__ void split_first(uint32_t u0, uint32_t u1, uint32_t& p0, f32x2& rest) {
  const f32x2 x{__uint_as_float(u0), __uint_as_float(u1)};
  p0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
  rest = f32x2{x[0] - __uint_as_float(p0 << 16), x[1] - __uint_as_float(p0 & 0xFFFF0000u)};
}
__device__ __forceinline__ void split_rest(f32x2 r, uint32_t& p1, uint32_t& p2) {
  p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
  const float t0 = r[0] - __uint_as_float(p1 << 16), t1 = r[1] - __uint_as_float(p1 & 0xFFFF0000u);
  p2 = __builtin_amdgcn_perm(__float_as_uint(t1), __float_as_uint(t0), 0x07060302u);
}

template <class L, bool F32>
struct StageGeom {
  using T = StageTy<F32>;
  // blocks of 16 states per stage: two, or one of float32, whose three pieces
  // fill LDS and registers otherwise; the smallest float32 tile, whose stages
  // are little but barrier and latency, takes two (12 rows, H = 1024,
  // V = 11,280: 37 -> 30 us; the next larger tile lost 3%, bf16's smallest
  // spilled)
  static constexpr int KS = F32 && !(L::BH == 32 && L::BV == 128) ? 1 : 2;
  static constexpr int BK = 16 * KS, GROUPS = KS * T::PIECES;
  // elements of an h row in LDS: its groups, padded so that the rows a read
  // takes at once (8 of 16 bytes) fall on distinct banks
  static constexpr int HS = F32 ? (KS == 1 ? 48 : 112) : 40;
  static constexpr int CPR = BK / T::EPC;               // chunks of a stage per h row
  static constexpr int WCH = L::BV / T::EPC;            // 16-byte chunks per W row
  static constexpr int W_OPS = BK * WCH / 256;          // chunks of W per thread and stage
  static constexpr int H_SLOTS = L::BH * CPR;
  static constexpr int H_OPS = (H_SLOTS + 255) / 256;
  static constexpr int OPS = W_OPS + H_OPS;
  // Register sets, i.e. stages between a load and its use, which have to cover
  // a memory round trip (about 1.2 us): 2 for float32 tiles of 128 rows and
  // more (1,536 cycles of products a stage), else 4, or 8 for the bf16 tiles
  // of few products a stage.
  static constexpr int NSET = F32 ? (L::BH >= 128 ? 2 : 4) : (OPS <= 5 ? 8 : 4);
  static constexpr int WG = 16 * L::BV;                 // elements of a W group
  static constexpr int WE = GROUPS * WG, HE = L::BH * HS;
  static_assert(BK * WCH % 256 == 0, "whole chunks per thread");
  // (32 rows: two threads load, split and write the same chunk, which costs
  // less than a branch)
  static_assert(H_SLOTS % 256 == 0 || H_SLOTS == 128, "whole waves load h");
  static_assert(256 % CPR == 0, "a thread's chunks are of the same states");
  static_assert(L::BV / 8 >= 16, "the swizzle permutes 16 chunks");
};

// Waves per SIMD the compiler must leave registers for: two for the tiles
// planned at two workgroups per CU.
template <class L, int KC>
constexpr int stage_waves() {
  return L::BV == 128 && (L::BH == 32 || (L::BH == 64 && KC <= 8)) ? 2 : 1;
}

template <class L, int KC, bool F32>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(stage_waves<L, KC>())))
void k1_stage(K1Args a) {
  using T = StageTy<F32>;
  using G = StageGeom<L, F32>;
  using E = typename T::E;
  constexpr int BV = L::BV, BH = L::BH, WV = L::WV, WH = L::WH, NWV = L::NWV;
  constexpr int BK = G::BK, EPC = T::EPC, PIECES = T::PIECES, GROUPS = G::GROUPS, NSET = G::NSET, HS = G::HS;
  constexpr int ESZ = sizeof(E);
  __shared__ __attribute__((aligned(16))) uint16_t S[2][G::WE + G::HE];
  __shared__ __attribute__((aligned(16))) SmemEpi<L, KC> ep;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wave % NWV, wh = wave / NWV;
  const int half = lane >> 5, col = lane & 31;
  int row_tile, split;
  k1_cell(a, blockIdx.x, row_tile, split);
  const int h0 = row_tile * BH;
  const int H = a.H, V = a.V;
  // stages of a tile, rounded up to whole register sets; those past H meet states of zero
  const int nk = (H + BK - 1) / BK;
  const int nkp = (nk + NSET - 1) / NSET * NSET;

  Epilogue<L, KC> epi;
  epi.init(ep, a.k);

  // ---- loads: chunk i of this thread is W row wr(i), words wc(i).., or, past
  // the W chunks, states kc.. of h row hslot(i).  Byte offsets from
  // the stage's first W row and h column, which are uniform.
  auto wr = [&](int i) { return (tid + 256 * i) / G::WCH; };
  auto wc = [&](int i) { return (tid + 256 * i) % G::WCH * EPC; };
  const int kc = (tid % G::CPR) * EPC;
  auto hslot = [&](int i) { return (tid + 256 * i) % G::H_SLOTS / G::CPR; };
  auto hrow = [&](int i) { return min(h0 + hslot(i), a.N - 1); };  // rows >= N: never written
  const KB_GLOBAL char* const Wg = (const KB_GLOBAL char*)(const KB_GLOBAL void*)a.W;
  const KB_GLOBAL char* const Hg = (const KB_GLOBAL char*)(const KB_GLOBAL void*)a.h;
  const KB_GLOBAL float* const Bg = (const KB_GLOBAL float*)a.b;
  uint32_t woff[G::W_OPS], hoff[G::H_OPS];
#pragma unroll
  for (int i = 0; i < G::W_OPS; ++i) woff[i] = ((uint32_t)wr(i) * (uint32_t)V + (uint32_t)wc(i)) * ESZ;
#pragma unroll
  for (int i = 0; i < G::H_OPS; ++i) hoff[i] = ((uint32_t)hrow(i) * (uint32_t)H + (uint32_t)kc) * ESZ;
  auto tile_v0 = [&](int vt) { return min(vt * BV, V - BV); };

  stage16 R[NSET][G::OPS];
  // the split's tiles are split, split + P, split + 2 P, ... (as in the DMA kernel)
  int ivt = split, ik0 = 0;  // the next stage to load; past the end, the last one again (never used)
  const KB_GLOBAL char *wb, *hb;  // its first W row and h column
  auto set_base = [&]() {
    const int k = min(ik0, H - BK);
    wb = Wg + ((size_t)k * V + tile_v0(ivt)) * ESZ;
    hb = Hg + (size_t)k * ESZ;
  };
  set_base();
  // (one path for every stage: a branch around the loads would make the
  // compiler wait for younger ones than it needs)
  auto load = [&](stage16 (&r)[G::OPS], int i) __attribute__((always_inline)) {
    const bool w = i < G::W_OPS;
    r[i] = *(const KB_GLOBAL typename T::V16*)(w ? wb + woff[i] : hb + hoff[i - G::W_OPS]);
  };
  auto next_stage = [&]() {
    const bool next = ik0 + BK >= nkp * BK;
    const bool end = next && ivt + a.P >= a.n_vtiles;
    ik0 = end ? ik0 : (next ? 0 : ik0 + BK);
    ivt += next && !end ? a.P : 0;
    set_base();
  };

  // stage k2 >= nk - 1 of a tile: states that earlier stages have had, the
  // first z of it, become zero
  auto zero_tail = [&](stage16 (&r)[G::OPS], int k2) __attribute__((always_inline)) {
    if ((k2 + 1) * BK <= H) return;
    const int z = (k2 + 1) * BK - H;
#pragma unroll
    for (int i = G::W_OPS; i < G::OPS; ++i)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t m;
        if constexpr (F32)
          m = kc + d >= z ? ~0u : 0u;
        else
          m = (kc + 2 * d >= z ? 0xFFFFu : 0u) | (kc + 2 * d + 1 >= z ? 0xFFFF0000u : 0u);
        r[i][d] &= m;
      }
  };

  // ---- registers -> LDS -> the registers' next load, in steps that fit
  // between products (seven VALU instructions hide behind one): per chunk of
  // 16 bytes two splits of two parts each, the write of three pieces, the load
  // (float32), or the write and the load (bf16)
  constexpr int STEPS = F32 ? 6 : 2, UNITS = STEPS * G::OPS;
  uint32_t piece[3][2];
  f32x2 rest;
  auto unit = [&](stage16 (&r)[G::OPS], uint16_t* buf, int u) __attribute__((always_inline)) {
    const int i = u / STEPS, step = u % STEPS;
    if (step == STEPS - 1) {
      load(r, i);
      return;
    }
    if (F32 && step < 4) {
      const int e = step >> 1;
      if ((step & 1) == 0)
        split_first(r[i][2 * e], r[i][2 * e + 1], piece[0][e], rest);
      else
        split_rest(rest, piece[1][e], piece[2][e]);
      return;
    }
    const bool w = i < G::W_OPS;
    int at;
    if (w) {
      const int rr = wr(i), c = wc(i);
      at = rr / 16 * PIECES * G::WG + rr % 16 * BV + (((c >> 3) ^ wswz(rr)) << 3) + (c & 7);
    } else {
      at = G::WE + hslot(i - G::W_OPS) * HS + kc / 16 * PIECES * 16 + kc % 16;
    }
    if constexpr (F32) {
      const int gs = w ? G::WG : 16;
#pragma unroll
      for (int p = 0; p < PIECES; ++p) *reinterpret_cast<u32x2*>(buf + at + p * gs) = u32x2{piece[p][0], piece[p][1]};
    } else {
      *reinterpret_cast<stage16*>(buf + at) = r[i];
    }
  };

  // ---- LDS -> fragments
  struct Frag {
    s16x4 lo[GROUPS][WV], hi[GROUPS][WV];
    bf16x8 b[GROUPS][WH];
  };
  Frag F[2];
  constexpr int RPG = 2 * WV + WH;     // reads per group
  constexpr int READS = GROUPS * RPG;
  auto read = [&](const uint16_t* buf, int u, Frag& f) __attribute__((always_inline)) {
    const int g = u / RPG, x = u % RPG;
    if (x < WH) {
      const int n = (wh * WH + x) * 32 + col;
      f.b[g][x] = *reinterpret_cast<const bf16x8*>(buf + G::WE + n * HS + g * 16 + half * 8);
    } else {
      const int vb = (x - WH) >> 1, hi = (x - WH) & 1;
      const int q = lane >> 4, j = lane & 15;
      const int r0 = 8 * (q >> 1) + (j >> 2);
      const int cw = (wv * WV + vb) * 32 + 16 * (q & 1) + 4 * (j & 3);
      const int at = g * G::WG + (r0 + 4 * hi) * BV + (((cw >> 3) ^ wswz(r0)) << 3) + (cw & 7);  // row r0 + 4: same swizzle
      const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((KB_LDS s16x4*)(buf + at));
      if (hi)
        f.hi[g][vb] = v;
      else
        f.lo[g][vb] = v;
    }
  };

  f32x16 acc[WV][WH];
  constexpr int NB = WV * WH, M = G::KS * T::PRODS * NB;  // products of a stage
  auto product = [&](const Frag& f, int i) __attribute__((always_inline)) {
    const int ks = i / NB / T::PRODS, p = i / NB % T::PRODS, vb = i % NB / WH, hb = i % NB % WH;
    const int gw = ks * PIECES + (F32 ? prod_w(p) : 0), gh = ks * PIECES + (F32 ? prod_h(p) : 0);
    const bf16x8 fa =
        __builtin_bit_cast(bf16x8, __builtin_shufflevector(f.lo[gw][vb], f.hi[gw][vb], 0, 1, 2, 3, 4, 5, 6, 7));
    acc[vb][hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, f.b[gh][hb], acc[vb][hb], 0, 0, 0);
  };

  // ---- one stage: the products of F[B], with the reads of the next stage's
  // fragments (from the other buffer), the writes of the stage after it (into
  // this stage's buffer) and the loads that follow them spread between them.
  // r: the registers of the stage after next; k2: its number in its tile
  auto stage = [&](auto bc, stage16 (&r)[G::OPS], int k2) __attribute__((always_inline)) {
    constexpr int B = decltype(bc)::value;
    zero_tail(r, k2);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      product(F[B], i);
      // the reads over the first half of the products, the units over all
#pragma unroll
      for (int u = min(2 * i * READS / M, READS); u < min(2 * (i + 1) * READS / M, READS); ++u)
        read(S[B ^ 1], u, F[B ^ 1]);
#pragma unroll
      for (int u = i * UNITS / M; u < (i + 1) * UNITS / M; ++u) unit(r, S[B], u);
      __builtin_amdgcn_sched_barrier(0);
    }
    next_stage();
    lds_barrier();
  };

  // ---- prologue: stages 0 and 1 in LDS, the next NSET in registers
#pragma unroll
  for (int s = 0; s < NSET; ++s) {
#pragma unroll
    for (int i = 0; i < G::OPS; ++i) load(R[s], i);
    next_stage();
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    zero_tail(R[s], s);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) unit(R[s], S[s], u);
    next_stage();
  }
  lds_barrier();
#pragma unroll
  for (int u = 0; u < READS; ++u) read(S[0], u, F[0]);
  lds_barrier();  // every wave has read buffer 0

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  for (int vt = split; vt < a.n_vtiles; vt += a.P) {
    const int v0 = tile_v0(vt);
    // the tile's bias and shared thresholds: asked for now, used after its products
    uint32_t tg[WH];
    epi.load_shared_thr(a, h0, tg);
    constexpr int NBIAS = (BV + 255) / 256;
    float bz[NBIAS];
#pragma unroll
    for (int i = 0; i < NBIAS; ++i) bz[i] = Bg[min(v0 + (tid + 256 * i) % BV, V - 1)];
#pragma unroll
    for (int vb = 0; vb < WV; ++vb)
#pragma unroll
      for (int hb = 0; hb < WH; ++hb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[vb][hb][r] = 0.f;

    for (int kt = 0; kt < nkp; kt += NSET) {
#pragma unroll
      for (int s = 0; s < NSET; s += 2) {
        // stage kt + s writes stage kt + s + 2, of this tile or the next
        const int k2 = kt + s + 2 < nkp ? kt + s + 2 : 0;
        stage(I0{}, R[(s + 2) % NSET], k2);
        stage(I1{}, R[(s + 3) % NSET], k2 + 1);
      }
    }
#pragma unroll
    for (int i = 0; i < NBIAS; ++i) ep.bias[0][(tid + 256 * i) % BV] = bz[i];
    lds_barrier();
    epi.tile(acc, ep, a, h0, v0, vt * BV, vt == split, tg, ep.bias[0]);
    // the next tile's first fragments again, so that the epilogue need not hold them
#pragma unroll
    for (int u = 0; u < READS; ++u) read(S[0], u, F[0]);
    lds_barrier();  // every wave has read buffer 0
  }

  // An infinite operand (in float32 also one whose first piece is) leaves NaN
  // among these products where its own is an infinity or a number: its pieces
  // are inf and inf - inf, and states and pieces of zero meet it.  A NaN stays
  // in its row's sum, so a cell that ends with one is done again as the direct
  // kernel does it, whose infinities are the operands' own.  Without the shared
  // thresholds: those that this pass has published are its own words', whose
  // scores may come out an ulp lower.  (Again tile by tile, inside the loop, it
  // cost every step 300 to 660 spilled registers.)
  bool nan = false;
#pragma unroll
  for (int hb = 0; hb < WH; ++hb) nan |= epi.st_s[hb] != epi.st_s[hb];
  // (a word of its own: a slower wave may still be at its last look at a
  // round's flag, past the round's last barrier)
  if (nan) ep.flag[2] = 1;
  lds_barrier();
  const bool again = ep.flag[2] != 0;
  lds_barrier();  // every wave has read it before the cell starts anew
  if (!again) {
    epi.finish(ep, a, h0, split);
  } else {
    K1Args d = a;
    d.share = 0;
    direct_cell<L, KC, F32, false>(ep, d, h0, split);
  }
}

template <class L, bool F32>
hipError_t launch_k1_stage(int kc, dim3 grid, const K1Args& a, hipStream_t st) {
  if (direct_shape(a.H, a.V) || a.V < L::BV) return hipErrorInvalidValue;
  const dim3 block(256);
  switch (kc) {
    case 4: k1_stage<L, 4, F32><<<grid, block, 0, st>>>(a); break;
    case 8: k1_stage<L, 8, F32><<<grid, block, 0, st>>>(a); break;
    case 12: k1_stage<L, 12, F32><<<grid, block, 0, st>>>(a); break;
    case 16: k1_stage<L, 16, F32><<<grid, block, 0, st>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace kb
