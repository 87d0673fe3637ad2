// Parts shared by both projection kernels: tile layouts, the sorted k-list,
// and the fused epilogue that turns a tile of logits into softmax statistics
// and k-best candidates without writing the logits anywhere.
#pragma once

#include "kb_common.hpp"

namespace kb {

#define KB_LDS __attribute__((address_space(3)))
typedef short s16x4 __attribute__((ext_vector_type(4)));

// XOR swizzle of the 16-byte chunks of W row r: rows r..r+3 read together by
// one transpose read land on distinct banks.
__device__ __forceinline__ int wswz(int r) { return 4 * (r & 3) + 2 * ((r >> 1) & 1); }

// XOR swizzle of the four 16-byte chunks of an h row: the 16 rows read by a
// 16-lane group at one logical chunk fall on 16 distinct 16-byte bank slots.
__device__ __forceinline__ int hswz(int n) { return (n >> 2) & 3; }

// s_waitcnt vmcnt(n) with expcnt / lgkmcnt left alone (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <int WV_, int WH_, int NWV_, int NWH_>
struct Lay {
  static constexpr int WV = WV_;    // 32-wide vocabulary blocks per wave
  static constexpr int WH = WH_;    // 32-wide hypothesis blocks per wave
  static constexpr int NWV = NWV_;  // waves along the vocabulary
  static constexpr int NWH = NWH_;  // waves along the hypotheses
  static_assert(NWV * NWH == 4, "four waves per workgroup");
  static constexpr int BV = 32 * WV * NWV;
  static constexpr int BH = 32 * WH * NWH;
  static constexpr int HOLD = 2 * NWV;  // lanes holding one row's scores of a tile
};

// Layouts: (WV, WH, NWV, NWH)
using LayL256 = Lay<4, 2, 1, 4>;  // 128 words x 256 rows per tile
using LayL128 = Lay<4, 2, 2, 2>;  // 256 words x 128 rows
using LayL32 = Lay<4, 1, 4, 1>;   // 512 words x 32 rows (few live rows)
using LayL32M = Lay<2, 1, 4, 1>;  // 256 words x 32 rows (few rows, more vocabulary tiles)
using LayL32S = Lay<1, 1, 4, 1>;  // 128 words x 32 rows (few rows, small vocabulary)
using LayL64 = Lay<2, 1, 2, 2>;   // 128 words x 64 rows (two workgroups per CU)
using LayL64M = Lay<4, 1, 2, 2>;  // 256 words x 64 rows

// Sizes of the candidate selection.  SEEDS: group maxima per row that give a
// split's first threshold; the k-th largest of 32 lets about k + k^2 / 64
// scores through (5.4 at k = 5, 15 at k = 12, 22 at k = 16).  PC: candidates
// of a row per round (a row with more takes another round): with these a first
// tile rarely needs a second one.  256 rows have room for fewer.
template <class L, int KC>
struct Sel {
  static constexpr int SEEDS = (L::BH == 256 && KC == 16) ? 16 : 32;
  static constexpr int PC = L::BH == 256 ? (KC == 16 ? 8 : (KC == 12 ? 14 : 16)) : (KC <= 8 ? 16 : 32);
  static constexpr int RS = SEEDS + (L::BH == 256 && KC >= 12 ? 0 : 4);  // floats from a row's seeds to the next
  static constexpr int GL = SEEDS / L::HOLD;      // groups per lane and row
  static constexpr int GS = L::WV * 16 / GL;      // scores per group
  static constexpr int TPR = 256 / L::BH;         // threads that merge one row
  static_assert(GL >= 4 && GL * GS == L::WV * 16 && GS >= 4, "whole groups");
};

// Rows of lists and pools are an odd number of 8-byte slots apart, so that
// threads on consecutive rows meet distinct banks, rows of seeds 36 floats where
// there is room.
template <class L, int KC>
struct alignas(16) SmemEpi {
  using X = Sel<L, KC>;
  float bias[2][L::BV];     // bias of the current / next vocabulary tile
  uint32_t tgk[2][L::BH];   // shared-threshold keys read at the tile's first stage
  float thr[L::BH];         // row's local threshold: k-th best score so far, or the seed
  int cnt[L::BH];           // candidates of the row this round (may exceed PC: the rest waits)
  int flag[4];              // "some lane has candidates left" of this and the next round; [2]: k1_stage's vote
  uint64_t lst[L::BH][KC + 1];  // the row's best keys of the split so far, best first; 0: none
  union {
    uint64_t pool[L::BH][X::PC + 1];  // this round's candidates
    float red[L::BH][X::RS];   // seeds, then the per-holder statistics
  } u;
};

// Order-preserving map of floats to unsigned ints for the shared per-row
// threshold (atomicMax).  0 means "no threshold yet".
__device__ __forceinline__ uint32_t f2key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key2f(uint32_t k) {
  if (k == 0u) return kNoThr;
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// 64-bit order key of a (score, word) candidate: higher score first, then
// lower word (the strict-'>' scans of the paper).  -0 is folded into +0 so
// that equal scores compare equal, and a NaN into -inf, which no score that
// passes the filter has (leaving NaNs out where they are picked, by a test of
// every candidate, took 1% of a step).  0 is no candidate's key.
__device__ __forceinline__ uint64_t cand_key(float x, int word) {
  return ((uint64_t)f2key(fmaxf(x, -INFINITY) + 0.0f) << 32) | (uint32_t)~(uint32_t)word;
}
constexpr uint32_t kNegInfKey = 0x007FFFFFu;  // f2key(-inf)

// ------------------------------------------------------------ candidates of a lane
// A lane holds NV (16 or 32) scores of a row in registers, and few of them
// reach the row's threshold.  Looking at every score under a branch cost 380
// cycles a score (some lane of the wave has a candidate at nearly every one);
// instead the lane's passing scores become one bit mask (a subtraction and a
// shift-in of its sign, two instructions a score) and each candidate is
// picked out by its position with a tree of selects, NV - 1 instructions, as
// often as the wave's busiest lane has candidates.

// The threshold t as pass_mask compares with it, so that the sign of x - t is
// that of x >= t for every x but NaN: +0 becomes -0 (-0 - +0 is -0, though the
// two are equal), +inf the largest number (inf - inf is NaN; a threshold may
// be lower than it need be, and what passes is ranked by its key).
__device__ __forceinline__ float pass_floor(float t) { return t == 0.f ? -0.f : fminf(t, FLT_MAX); }

// Bit 31 - i set: x[i] >= t, t a pass_floor.  A NaN's bit may be either (its
// key is that of -inf).
template <int NV>
__device__ __forceinline__ uint32_t pass_mask(const float (&x)[NV], float t) {
  uint32_t below = 0;
#pragma unroll
  for (int i = 0; i < NV; ++i) below = __builtin_amdgcn_alignbit(below, __float_as_uint(x[i] - t), 31);
  if constexpr (NV < 32) below = (below << (32 - NV)) | ((1u << (32 - NV)) - 1);
  return ~below;
}

// x[pos], by bitwise selects: as conditional selects the compiler takes them
// for indexing of an array and compares with every index, at every level.
template <int NV>
__device__ __forceinline__ float pick(const float (&x)[NV], int pos) {
  uint32_t y[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) y[i] = __float_as_uint(x[i]);
#pragma unroll
  for (int w = 1, b = 0; w < NV; w *= 2, ++b) {
    uint32_t m = (uint32_t)__builtin_amdgcn_sbfe(pos, b, 1);  // all ones where bit b of pos is set
    asm("" : "+v"(m));
#pragma unroll
    for (int i = 0; i < NV; i += 2 * w) y[i] = (y[i + w] & m) | (y[i] & ~m);
  }
  return __uint_as_float(y[0]);
}

// Word offset of position p of a lane's 32 scores (two 32-word blocks of an
// accumulator: register 16 b + 4 i + j is word 32 b + 8 i + j).
__device__ __forceinline__ int pos_word(int p) { return p + (p & 28); }

// The k-th largest of a row's N seeds, N / TPR of them in this thread's x, the
// row's others in the TPR - 1 lanes beside it; all of them in row[0 .. N).
template <int N, int TPR, int KC>
__device__ __forceinline__ float kth_seed(const float* row, int t, int k) {
  if constexpr (TPR >= 4) {
    // the largest seed that at least k seeds reach
    float x[N / TPR];
    int ge[N / TPR];
#pragma unroll
    for (int i = 0; i < N / TPR; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(row + t * (N / TPR) + i);
      x[i] = v.x;
      x[i + 1] = v.y;
      x[i + 2] = v.z;
      x[i + 3] = v.w;
    }
#pragma unroll
    for (int i = 0; i < N / TPR; ++i) ge[i] = 0;
#pragma unroll
    for (int j = 0; j < N; j += 4) {
      const float4 v = *reinterpret_cast<const float4*>(row + j);
#pragma unroll
      for (int i = 0; i < N / TPR; ++i)
        ge[i] += (v.x >= x[i] ? 1 : 0) + (v.y >= x[i] ? 1 : 0) + (v.z >= x[i] ? 1 : 0) + (v.w >= x[i] ? 1 : 0);
    }
    float best = -INFINITY;
#pragma unroll
    for (int i = 0; i < N / TPR; ++i) best = fmaxf(best, ge[i] >= k ? x[i] : -INFINITY);
#pragma unroll
    for (int m = 1; m < TPR; m *= 2) best = fmaxf(best, __shfl_xor(best, m));
    return best;
  } else {
    // insertion by median of three into a right-aligned descending list (+inf
    // sentinels first), one thread per row
    float v[KC];
#pragma unroll
    for (int j = 0; j < KC; ++j) v[j] = (j < KC - k) ? INFINITY : -INFINITY;
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      const float4 q = *reinterpret_cast<const float4*>(row + i);
      const float x[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int j = KC - 1; j > 0; --j) v[j] = __builtin_amdgcn_fmed3f(v[j - 1], v[j], x[e]);
        v[0] = fmaxf(v[0], x[e]);
      }
    }
    return v[KC - 1];
  }
}

// ------------------------------------------------------------ the epilogue
// Per lane: running (max, sum) of its scores of each of its WH rows.  In LDS:
// each row's sorted best keys of this split.
template <class L, int KC>
struct Epilogue {
  static constexpr int WV = L::WV, WH = L::WH, NWV = L::NWV;
  using X = Sel<L, KC>;
  using Smem = SmemEpi<L, KC>;
  // the seeds are written and read 16 bytes at a time
  static_assert(offsetof(Smem, u) % 16 == 0 && X::RS % 4 == 0, "aligned seeds");
  static constexpr int NV = WV >= 2 ? 32 : 16;   // scores per mask
  static constexpr int NW = WV * 16 / NV;        // masks per row and lane
  float st_m[WH], st_s[WH];
  float published;  // owner (a row's first merging thread): last value pushed to the shared threshold

  __device__ __forceinline__ void init(Smem& ep, int k) {
    const int tid = threadIdx.x;
    if (tid < L::BH) {
      ep.thr[tid] = kNoThr;
      ep.cnt[tid] = 0;
    }
    for (int i = tid; i < L::BH * (KC + 1); i += 256) (&ep.lst[0][0])[i] = 0ull;
    if (tid < 4) ep.flag[tid] = 0;
#pragma unroll
    for (int hb = 0; hb < WH; ++hb) {
      st_m[hb] = kStatInit;
      st_s[hb] = 0.f;
    }
    published = kNoThr;
  }

  // Shared threshold of this lane's rows (valid lower bounds of each row's
  // k-th best: k scores of the row are >= it).  Issued early, used in tile().
  // (Raw keys: decoding is deferred to the epilogue so that nothing waits on
  // these loads, which would drain the DMA ring issued before them.)
  __device__ __forceinline__ void load_shared_thr(const K1Args& a, int h0, uint32_t (&tg)[WH]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wh = wave / NWV, col = lane & 31;
#pragma unroll
    for (int hb = 0; hb < WH; ++hb) {
      const int row = min(h0 + (wh * WH + hb) * 32 + col, a.N - 1);
      tg[hb] = a.share ? __hip_atomic_load(&a.gthr[row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    }
  }

  __device__ __forceinline__ void owner_publish(const K1Args& a, int row, float v) {
    if (a.share && row < a.N && v > published) {
      atomicMax(&a.gthr[row], f2key(v));
      published = v;
    }
  }

  // One BV x BH tile of logits in acc (MFMA 32x32 layout: lane holds row
  // (hypothesis) col of each 32-block and 16 vocabulary entries).  The tile
  // starts at word v0; its words below vlo belong to the tile before.
  __device__ __forceinline__ void tile(f32x16 (&acc)[WV][WH], Smem& ep, const K1Args& a, int h0, int v0,
                                       int vlo, bool first, const uint32_t (&tg)[WH], const float* bias) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = wave % NWV, wh = wave / NWV;
    const int half = lane >> 5, col = lane & 31;
    const int holder = wv * 2 + half;
    const int k = a.k;

    // ---- bias (Algorithm 3 AddBias, fused) and masking of words >= V or < vlo
    const bool ragged = v0 > a.V - L::BV || v0 < vlo;
#pragma unroll
    for (int vb = 0; vb < WV; ++vb) {
      const int vl = (wv * WV + vb) * 32 + 4 * half;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 bb = *reinterpret_cast<const float4*>(&bias[vl + 8 * i]);
#pragma unroll
        for (int hb = 0; hb < WH; ++hb) {
          acc[vb][hb][4 * i + 0] += bb.x;
          acc[vb][hb][4 * i + 1] += bb.y;
          acc[vb][hb][4 * i + 2] += bb.z;
          acc[vb][hb][4 * i + 3] += bb.w;
        }
      }
      if (ragged) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int v = v0 + vl + 8 * (r >> 2) + (r & 3);
#pragma unroll
          for (int hb = 0; hb < WH; ++hb)
            if ((uint32_t)v >= (uint32_t)a.V || v < vlo) acc[vb][hb][r] = -INFINITY;
        }
      }
    }
    // ---- running softmax statistics: one rescale per tile (Algorithm 4's
    // sum <- e^(max_old - max_new) * sum, then the new terms)
    float tmax[WH][NW];  // the lane's largest score per mask
#pragma unroll
    for (int hb = 0; hb < WH; ++hb) {
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        float m0 = acc[w * NV / 16][hb][0], m1 = acc[w * NV / 16][hb][1];
#pragma unroll
        for (int i = 2; i < NV; i += 2) {
          m0 = fmaxf(m0, acc[(w * NV + i) / 16][hb][i % 16]);
          m1 = fmaxf(m1, acc[(w * NV + i) / 16][hb][i % 16 + 1]);
        }
        tmax[hb][w] = fmaxf(m0, m1);
        mx = fmaxf(mx, tmax[hb][w]);
      }
      const float mnew = fmaxf(st_m[hb], mx);
      const float ml2 = mnew * kL2E;
      float sum = st_s[hb] * exp2_fast((st_m[hb] - mnew) * kL2E);
#pragma unroll
      for (int vb = 0; vb < WV; ++vb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += exp2_fast(fmaf(acc[vb][hb][r], kL2E, -ml2));
      st_s[hb] = sum;
      st_m[hb] = mnew;
    }

    const int row = tid / X::TPR, rt = tid % X::TPR;  // the row this thread helps to merge
    // ---- first tile of the split: seed each row's threshold with the k-th
    // largest group maximum (k distinct scores are >= it)
    if (first) {
#pragma unroll
      for (int hb = 0; hb < WH; ++hb) {
        const int hl = (wh * WH + hb) * 32 + col;
        float gm[X::GL];
#pragma unroll
        for (int g = 0; g < X::GL; ++g) {
#pragma unroll
          for (int i = 0; i < X::GS; ++i) {
            const int q = g * X::GS + i;
            gm[g] = i == 0 ? acc[q / 16][hb][q % 16] : fmaxf(gm[g], acc[q / 16][hb][q % 16]);
          }
        }
#pragma unroll
        for (int g = 0; g < X::GL; g += 4)
          *reinterpret_cast<float4*>(&ep.u.red[hl][holder * X::GL + g]) =
              make_float4(gm[g], gm[g + 1], gm[g + 2], gm[g + 3]);
      }
      lds_barrier();
      if (X::TPR >= 4 || rt == 0) {
        const float kth = kth_seed<X::SEEDS, X::TPR, KC>(&ep.u.red[row][0], rt, k);
        if (rt == 0 && kth > ep.thr[row]) {
          ep.thr[row] = kth;
          owner_publish(a, h0 + row, kth);
        }
      }
      lds_barrier();
    }

    // ---- candidate rounds.  Every score >= max(row's local threshold, shared
    // threshold) goes to the row's pool (ties are kept; the keys settle them by
    // word index).  Scores that find the pool full wait for another round,
    // against the raised threshold.
    uint32_t left[WH][NW];  // scores not yet in a pool
#pragma unroll
    for (int hb = 0; hb < WH; ++hb)
#pragma unroll
      for (int w = 0; w < NW; ++w) left[hb][w] = ~0u;
    for (int round = 0;; ++round) {
      uint32_t any = 0;
#pragma unroll
      for (int hb = 0; hb < WH; ++hb) {
        const int hl = (wh * WH + hb) * 32 + col;
        const float t = pass_floor(fmaxf(ep.thr[hl], key2f(tg[hb])));
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          if (__builtin_amdgcn_ballot_w64(tmax[hb][w] >= t) == 0ull) {
            left[hb][w] = 0;
            continue;
          }
          float x[NV];
#pragma unroll
          for (int i = 0; i < NV; ++i) x[i] = acc[(w * NV + i) / 16][hb][i % 16];
          uint32_t m = pass_mask<NV>(x, t) & left[hb][w], kept = 0;
          const int vbase = v0 + (wv * WV + w * (NV / 16)) * 32 + 4 * half;
          while (__builtin_amdgcn_ballot_w64(m != 0) != 0ull) {
            const int p = __builtin_clz(m | 1u);
            const uint32_t bit = 0x80000000u >> p;
            const float cx = pick<NV>(x, p);
            if (m != 0) {
              const int at = __hip_atomic_fetch_add(&ep.cnt[hl], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              const uint64_t key = cand_key(cx, vbase + pos_word(p));  // while the slot is on its way
              ep.u.pool[hl][min(at, X::PC)] = key;                    // slot PC is nobody's
              kept |= at < X::PC ? 0u : bit;
              m &= ~bit;
            }
          }
          left[hb][w] = kept;
          any |= kept;
        }
      }
      if (any) ep.flag[round & 1] = 1;
      lds_barrier();
      if (tid == 0) ep.flag[(round + 1) & 1] = 0;  // read only after the next barrier
      merge_pool(ep, a, h0, row, rt, k);
      lds_barrier();
      if (ep.flag[round & 1] == 0) break;
    }
  }

  // One row's threads (lanes of one wave, so all reads come before the
  // writes): thread rt takes the list's entries rt, rt + TPR, ... and the
  // pool's, NQ of those, counts the larger keys and puts each in its place.
  // List entries past the k-th are 0.
  template <int NQ>
  __device__ __forceinline__ void rank_pool(Smem& ep, int row, int rt, int c, int k) {
    constexpr int OQ = (KC + X::TPR - 1) / X::TPR;
    uint64_t ok[OQ], nk[NQ], old[KC];
    int orank[OQ], nrank[NQ];
#pragma unroll
    for (int j = 0; j < KC; ++j) old[j] = ep.lst[row][j];
#pragma unroll
    for (int q = 0; q < OQ; ++q) {
      const int e = rt + X::TPR * q;
      ok[q] = ep.lst[row][min(e, KC)];
      orank[q] = e < k ? e : KC;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = rt + X::TPR * q;
      nk[q] = ep.u.pool[row][min(e, X::PC)];
      nrank[q] = e < c ? 0 : KC;
    }
    for (int j0 = 0; __builtin_amdgcn_ballot_w64(j0 < c) != 0ull; j0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + u;
        const uint64_t v = ep.u.pool[row][min(j, X::PC)];
        const uint64_t o = j < c ? v : 0ull;
#pragma unroll
        for (int q = 0; q < OQ; ++q) orank[q] += o > ok[q] ? 1 : 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) nrank[q] += o > nk[q] ? 1 : 0;
      }
    }
#pragma unroll
    for (int j = 0; j < KC; ++j)
#pragma unroll
      for (int q = 0; q < NQ; ++q) nrank[q] += old[j] > nk[q] ? 1 : 0;
#pragma unroll
    for (int q = 0; q < OQ; ++q)
      if (orank[q] < k) ep.lst[row][orank[q]] = ok[q];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      if (nrank[q] < k) ep.lst[row][nrank[q]] = nk[q];
  }

  // The row's pool into its sorted list, and the row's threshold after it.
  // Up to 64 rows: every key's place is the number of larger ones, counted by
  // the row's 4 or 8 threads.  More rows: one thread per row inserts key after
  // key (counting with 2 threads a row took 6% longer on a 1,152-row step).
  __device__ __forceinline__ void merge_pool(Smem& ep, const K1Args& a, int h0, int row, int rt, int k) {
    const int c = min(ep.cnt[row], X::PC);
    if (__builtin_amdgcn_ballot_w64(c > 0) == 0ull) return;
    uint64_t kth = 0;
    if constexpr (X::TPR >= 4) {
      // most rows have few candidates: one per thread then
      if (__builtin_amdgcn_ballot_w64(c > X::TPR) == 0ull)
        rank_pool<1>(ep, row, rt, c, k);
      else
        rank_pool<(X::PC + X::TPR - 1) / X::TPR>(ep, row, rt, c, k);
      kth = ep.lst[row][k - 1];
    } else if (rt == 0) {
      uint64_t l[KC];
#pragma unroll
      for (int j = 0; j < KC; ++j) l[j] = ep.lst[row][j];
      for (int i = 0; i < c; ++i) {
        const uint64_t key = ep.u.pool[row][i];
        // the keys are descending, so gt[] is false then true and the key lands at the first true
        bool gt[KC];
#pragma unroll
        for (int j = 0; j < KC; ++j) gt[j] = key > l[j];
#pragma unroll
        for (int j = KC - 1; j > 0; --j) l[j] = gt[j] ? (gt[j - 1] ? l[j - 1] : key) : l[j];
        l[0] = gt[0] ? key : l[0];
      }
#pragma unroll
      for (int j = 0; j < KC; ++j) ep.lst[row][j] = l[j];
      kth = ep.lst[row][k - 1];
    }
    if (rt == 0) {
      ep.cnt[row] = 0;
      const float v = key2f((uint32_t)(kth >> 32));
      if (kth != 0ull && v > ep.thr[row]) {
        ep.thr[row] = v;
        owner_publish(a, h0 + row, v);
      }
    }
  }

  // Merge the holders' statistics and write this split's partial of each row.
  __device__ __forceinline__ void finish(Smem& ep, const K1Args& a, int h0, int split) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wv = wave % NWV, wh = wave / NWV;
    const int half = lane >> 5, col = lane & 31;
    const int holder = wv * 2 + half;
    const int k = a.k;
    __syncthreads();
#pragma unroll
    for (int hb = 0; hb < WH; ++hb) {
      const int hl = (wh * WH + hb) * 32 + col;
      ep.u.red[hl][2 * holder + 0] = st_m[hb];
      ep.u.red[hl][2 * holder + 1] = st_s[hb];
    }
    __syncthreads();
    if (tid < L::BH && h0 + tid < a.N) {
      float M = kStatInit;
#pragma unroll
      for (int i = 0; i < L::HOLD; ++i) M = fmaxf(M, ep.u.red[tid][2 * i]);
      float S = 0.f;
#pragma unroll
      for (int i = 0; i < L::HOLD; ++i)
        S += ep.u.red[tid][2 * i + 1] * exp2_fast((ep.u.red[tid][2 * i] - M) * kL2E);
      a.stats[(size_t)split * a.N + h0 + tid] = make_float2(M, S);
    }
    // the lists, consecutive entries by consecutive threads
    int2* const out = a.lists + ((size_t)split * a.N + h0) * k;
    const int n = min(L::BH, a.N - h0) * k;
    for (int i = tid; i < n; i += 256) {
      const uint64_t key = ep.lst[i / k][i % k];
      const uint32_t score = (uint32_t)(key >> 32);  // (0: no candidate)
      out[i] = score > kNegInfKey ? make_int2(__float_as_int(key2f(score)), (int)~(uint32_t)key)
                                  : make_int2(__float_as_int(-INFINITY), INT_MAX);
    }
  }
};

}  // namespace kb
