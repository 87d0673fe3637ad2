// K2: merge the vocabulary splits of every row, then the rows of every sentence.
//
// One workgroup per sentence, W waves (one per row of an average sentence, two
// past 128 splits, W <= 16, and no more than the staged lists fit in LDS); the
// sentence's rows are taken as many at a time as there are waves.  With two
// waves a row each takes half of its splits (one wave with four lists a lane
// spent twice the time of two in the rounds: 8.7 us against 6.9 at 5 rows and
// 196 splits):
//   * the row's split lists are staged in LDS, sixteen loads in flight per
//     lane, while its split statistics are reduced in registers;
//   * LSE = M + ln(sum_p s_p * exp(m_p - M)) over the P split partials -- the
//     rescaling identity of Algorithm 4 applied between shards, the reduction
//     step of Algorithm 6 extended from (max, best) to softmax statistics;
//   * the row's best words: rounds of a wave-wide maximum of the scores'
//     ordered bits, then of the words where heads share a score (wave_keys.hpp),
//     over the heads of the P sorted split lists (strict total order).  5 rows of
//     125 splits: k = 10 17.9 -> 16.6 us a step against maxima of both every
//     round.  Each lane keeps its lists' heads and the entries after them in
//     registers, so a round reads no LDS on its critical path.
//     The rounds stop once a score (prev + x - LSE) falls below the sentence's
//     k-th best so far: the row's later entries are worse still;
//   * the running k best of the sentence and the chunk's candidates are ranked
//     by (score desc, flat index asc), flat index being
//     (row - first row) * V + word, one thread per candidate, and the first k
//     kept.  Because the score adds a per-row constant to x, a sentence's k
//     best lie in the union of its rows' k best, so nothing outside these
//     candidates can be selected.
#include "kb_launch.hpp"
#include "wave_keys.hpp"

namespace kb {

constexpr int K2_MAXW = 16;                  // waves per workgroup: rows merged at once
constexpr int K2_MAXP = 256;                 // splits: up to two lists per lane of two waves
constexpr int K2_LS = 16;                    // LDS slots per staged split list (k <= 16)
constexpr int K2_PAD = 2;                    // slots after the last list: a spent list's next entry is read, never used
constexpr int K2_C = K2_MAXW * 16 + 16 + 2;  // running best + one chunk (+ pad to pairs)
constexpr int kNegInfBits = (int)0xff800000;  // -inf: the score of an empty entry (word INT_MAX)
static_assert(K2_C % 2 == 0, "candidate keys are read in pairs");

// Wave-wide reductions from DPP moves within each row of 16 lanes (quad
// xor 1, quad xor 2, half-row mirror, row mirror), then the four row results
// read out (v_readlane): no LDS permutes on the merge's critical path.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
__device__ __forceinline__ float lane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f<kDppXor1>(v));
  v = fmaxf(v, dpp_f<kDppXor2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_f<kDppMirror>(v));
  return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<kDppXor1>(v);
  v += dpp_f<kDppXor2>(v);
  v += dpp_f<kDppHalfMirror>(v);
  v += dpp_f<kDppMirror>(v);
  return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}
// M + ln S with S = m 2^e, m in [1/2, 1): the hardware logarithm of S itself
// (log2 S is 15 or so) is off by up to half a unit of 2^-20, the largest error
// in a row's log-sum-exp; of m it is within 2^-24, and e ln 2 is added in two
// parts, the first exact.
__device__ __forceinline__ float log_plus(float M, float S) {
  const float e = (float)__builtin_amdgcn_frexp_expf(S), l = __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(S));
  constexpr float kLn2Hi = 0.693115234375f, kLn2Lo = 3.194618494e-5f;  // their sum is ln 2 to float32
  return fmaf(e, kLn2Hi, M) + fmaf(l, 0.69314718056f, e * kLn2Lo);
}
// A candidate of the sentence merge as one 64-bit key (key_of) of its score
// and flat index: a higher score, then a lower flat index, gives the larger key.
__device__ __forceinline__ uint64_t cand_key(float score, int flat) { return key_of(score, flat); }

// NQ: split lists per lane (at most 64 * NQ per wave); HW: waves per row.  Up
// to 16 waves, so 128 VGPRs: a form for 8 waves and 256 VGPRs staged longer
// lists in one batch, but two waves a row do so too, without its spilled SGPRs.
template <int NQ, int HW>
__global__ __launch_bounds__(64 * K2_MAXW) void k2_merge(K2Args a) {
  __shared__ __align__(16) uint64_t key[K2_C];  // read two at a time when ranked
  __shared__ int c_t[K2_C];
  __shared__ int c_p[K2_C];
  __shared__ uint64_t n_key[16];
  __shared__ int n_t[16], n_p[16];
  __shared__ float2 half_st[K2_MAXW];  // each wave's (max, sum) of its share of a row's splits
  // one list of empty entries, then per wave one row's P lists of K2_LS slots
  extern __shared__ int2 lists_dyn[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int RW = (blockDim.x >> 6) / HW;  // rows at a time
  const int s = blockIdx.x;
  const int k = a.k;
  // this wave's splits p_lo .. p_lo + P - 1
  const int share = (a.P + HW - 1) / HW, p_lo = (wave % HW) * share, P = min(share, a.P - p_lo);
  const int r0 = a.off[s], r1 = a.off[s + 1];

  if (tid < K2_LS) lists_dyn[tid] = make_int2(kNegInfBits, INT_MAX);
  // running best k of the sentence lives in slots [0, k); empty slots hold
  // distinct keys below every real candidate
  if (tid < k) {
    key[tid] = cand_key(-INFINITY, INT_MAX - tid);
    c_t[tid] = -1;
    c_p[tid] = -1;
  }
  const int wbase = K2_LS + wave * share * K2_LS;  // this wave's lists in lists_dyn
  int lidx[NQ];  // each lane's lists, or the empty list where it has none
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int p = lane + 64 * q;
    lidx[q] = p < P ? wbase + p * K2_LS : 0;
  }

  for (int cr0 = r0; cr0 < r1; cr0 += RW) {
    const int nrows = min(RW, r1 - cr0);
    const int ri = wave / HW;
    const bool active = ri < nrows;
    const int r = cr0 + ri;
    float2 st[NQ];
    float prev_r = 0.f;
    if (active) {
      // the row's split statistics and previous score first, so that their
      // loads are in flight with the lists' (one memory round trip for a
      // row whose lists take one batch)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int p = lane + 64 * q;
        st[q] = p < P ? a.stats[(size_t)(p_lo + p) * a.N + r] : make_float2(kStatInit, 0.f);
      }
      prev_r = a.prev[r];
      // lane = kp * g + j (kp: k rounded up to a power of two) stages entry j
      // of lists p0 + g, p0 + gpl + g, ... (gpl = 64 / kp lists per load;
      // slots k .. kp - 1 get empty entries): LB loads in flight per lane
      // before the first LDS write, as many as the registers allow.  Slots past
      // kp are never read before a list has given up all k entries, so they
      // stay unwritten.
      constexpr int LB = 16;
      const int lgk = k <= 1 ? 0 : (k <= 2 ? 1 : (k <= 4 ? 2 : (k <= 8 ? 3 : 4)));
      const int j = lane & ((1 << lgk) - 1), g = lane >> lgk, gpl = 64 >> lgk;
      for (int p0 = 0; p0 < P; p0 += LB * gpl) {
        int2 v[LB];
#pragma unroll
        for (int u = 0; u < LB; ++u) {
          const int p = p0 + u * gpl + g;
          v[u] = make_int2(kNegInfBits, INT_MAX);
          if (p < P && j < k) v[u] = a.lists[((size_t)(p_lo + p) * a.N + r) * k + j];
        }
#pragma unroll
        for (int u = 0; u < LB; ++u) {
          const int p = p0 + u * gpl + g;
          if (p < P) lists_dyn[wbase + p * K2_LS + j] = v[u];
        }
      }
    }
    float M = kStatInit, S = 0.f;
    if (active) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) M = fmaxf(M, st[q].x);
      M = wave_max(M);
#pragma unroll
      for (int q = 0; q < NQ; ++q) S += st[q].y * __expf(st[q].x - M);
      S = wave_sum(S);
      if (HW > 1 && lane == 0) half_st[wave] = make_float2(M, S);
    }
    __syncthreads();  // the staged lists are visible; the running best is settled
    uint64_t my_key = cand_key(-INFINITY, INT_MAX - (k + wave * k + lane));
    int my_t = -1;
    if (active) {
      if constexpr (HW > 1) {
        const float2 o = half_st[wave ^ 1];
        const float m = fmaxf(M, o.x);
        S = S * __expf(M - m) + o.y * __expf(o.x - m);
        M = m;
      }
      const float lse = log_plus(M, S);
      if (a.row_lse != nullptr && lane == 0 && wave % HW == 0) a.row_lse[r] = lse;
      const float base = prev_r - lse;
      const float kth = key_score(key[k - 1]);  // running k-th best (-inf before the first chunk)

      // per list of this lane: its head's key in two halves, and the entry after it
      uint32_t hi[NQ], lo[NQ];
      int2 nx[NQ];
      int at[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int2 h = lists_dyn[lidx[q]];
        at[q] = lidx[q] + 1;
        nx[q] = lists_dyn[at[q]];
        const uint64_t hk = key_of(__int_as_float(h.x), h.y);
        hi[q] = (uint32_t)(hk >> 32);
        lo[q] = (uint32_t)hk;
      }
      // A round is one chain of dependent instructions, some 8 cycles each, so
      // it has as few as there can be: one maximum over the high words (the low
      // ones only where two heads share it), the winner out of its lane as two
      // scalars, no branch but that and the cut-off.
      uint32_t my_hi = (uint32_t)(kEmptyKey >> 32), my_lo = (uint32_t)kEmptyKey;  // lane jr: the row's jr-th best
      for (int jr = 0; jr < k; ++jr) {
        uint32_t m = hi[0];
#pragma unroll
        for (int q = 1; q < NQ; ++q) m = max(m, hi[q]);
        const uint32_t top = wave_umax(m);
        uint64_t won[NQ];  // the lanes whose head it is
        int heads = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          won[q] = __ballot(hi[q] == top);
          heads += __builtin_popcountll(won[q]);
        }
        uint32_t low;
        if (heads == 1) {
          low = __builtin_amdgcn_readlane((int)lo[0], __builtin_ctzll(won[0] | 1ull << 63));
#pragma unroll
          for (int q = 1; q < NQ; ++q) {
            const uint32_t l = __builtin_amdgcn_readlane((int)lo[q], __builtin_ctzll(won[q] | 1ull << 63));
            low = won[q] != 0 ? l : low;
          }
        } else {
          // equal scores: the lowest word (empty heads are all alike and advance together)
          uint32_t l = 0;
#pragma unroll
          for (int q = 0; q < NQ; ++q) l = max(l, hi[q] == top ? lo[q] : 0u);
          low = wave_umax(l);
#pragma unroll
          for (int q = 0; q < NQ; ++q) won[q] = __ballot(hi[q] == top && lo[q] == low);
        }
        // the row's later entries are worse still: once this one scores below
        // the sentence's k-th best of the rows ranked so far, none can enter
        if (cr0 != r0 && key_score((uint64_t)top << 32) + base < kth) break;
        my_hi = lane == jr ? top : my_hi;
        my_lo = lane == jr ? low : my_lo;
        // The list whose head won advances; every lane then reloads the
        // entry after its heads, so the read is waited for only at the next
        // round.  A list advances at most once a round, k rounds in all, and
        // its head is compared only while rounds remain, so what is read past
        // its k entries (within the staged lists and their pad) is never used.
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const bool adv = __builtin_amdgcn_inverse_ballot_w64(won[q]);
          const uint64_t nk = key_of(__int_as_float(nx[q].x), nx[q].y);
          hi[q] = adv ? (uint32_t)(nk >> 32) : hi[q];
          lo[q] = adv ? (uint32_t)nk : lo[q];
          at[q] += adv ? 1 : 0;
          nx[q] = lists_dyn[at[q]];
        }
      }
      const uint64_t mine = ((uint64_t)my_hi << 32) | my_lo;
      if (lane < k && key_score(mine) > -INFINITY) {
        my_t = key_index(mine);
        my_key = cand_key(key_score(mine) + base, (r - r0) * a.V + my_t);
      }
    }
    const int C = k + nrows * HW * k;
    if (active && lane < k) {
      const int slot = k + wave * k + lane;
      key[slot] = my_key;
      c_t[slot] = my_t;
      c_p[slot] = r;
    }
    if (tid == 0 && (C & 1)) key[C] = 0;  // pairs: a pad below every key
    __syncthreads();
    // rank every candidate (running best + this chunk) and keep the first k
    if (tid < C) {
      const uint64_t me = key[tid];
      const ulonglong2* kp = reinterpret_cast<const ulonglong2*>(key);
      int rank = 0;
      const int C2 = (C + 1) >> 1;
#pragma unroll 4
      for (int o = 0; o < C2; ++o) {
        const ulonglong2 q = kp[o];
        rank += (q.x > me ? 1 : 0) + (q.y > me ? 1 : 0);
      }
      if (rank < k) {
        n_key[rank] = me;
        n_t[rank] = c_t[tid];
        n_p[rank] = c_p[tid];
      }
    }
    __syncthreads();
    if (tid < k) {
      key[tid] = n_key[tid];
      c_t[tid] = n_t[tid];
      c_p[tid] = n_p[tid];
    }
    __syncthreads();
  }
  if (tid < k) {
    a.tok[s * k + tid] = c_t[tid];
    a.par[s * k + tid] = c_p[tid];
    a.score[s * k + tid] = key_score(key[tid]);
  }
}

__global__ __launch_bounds__(256) void zero_u32(uint32_t* p, int n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = 0u;
}

hipError_t launch_zero_u32(uint32_t* p, int n, hipStream_t st) {
  const int blocks = n > 0 ? min((n + 255) / 256, 1024) : 1;
  zero_u32<<<dim3(blocks), dim3(256), 0, st>>>(p, n);
  return hipGetLastError();
}

// Greedy (beam 1) merge, the reduction of Algorithm 6: per row, the best
// (score, word) over the P split lists of length 1, in the strict order
// higher score, then lower word.  One wave per row: each lane scans the
// splits lane, lane + 64, ..., then the wave-wide largest key.  Empty list slots
// hold scores below every real one, and the split holding the row's maximum
// always lists it.
__global__ __launch_bounds__(256) void k2_argmax(const int2* __restrict__ lists, int P, int N,
                                                 int32_t* __restrict__ tok, float* __restrict__ val) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= N) return;  // whole waves leave together
  uint64_t best = kEmptyKey;
  for (int p = lane; p < P; p += 64) {
    const int2 e = lists[(size_t)p * N + r];
    const uint64_t key = key_of(__int_as_float(e.x), e.y);
    best = key > best ? key : best;
  }
  best = wave_max64(best);
  if (lane == 0) {
    tok[r] = key_index(best);
    val[r] = key_score(best);
  }
}

hipError_t launch_k2_argmax(const int2* lists, int P, int N, int32_t* tok, float* val, hipStream_t st) {
  if (N <= 0) return hipSuccess;
  k2_argmax<<<dim3((N + 3) / 4), dim3(256), 0, st>>>(lists, P, N, tok, val);
  return hipGetLastError();
}

template <int NQ, int HW>
static hipError_t launch_k2_nq(const K2Args& a, hipStream_t st) {
  // HW waves per row of a sentence of average length (longer sentences take
  // their rows in chunks), as many as the staged lists fit in 144 KB of LDS
  // (the kernel's static LDS is under 5 KB): at most 16 up to P = 72, 8 (4 rows) at P = 256
  const int share = (a.P + HW - 1) / HW;
  const size_t per_wave = (size_t)share * K2_LS * sizeof(int2);
  const int rows_per = (a.N + a.S - 1) / a.S;
  const int fit = (int)std::min<size_t>(K2_MAXW, (144 * 1024) / per_wave) / HW;  // rows at once
  const int W = std::min(fit, std::max(1, rows_per)) * HW;
  const size_t lds = (size_t)(K2_LS + K2_PAD) * sizeof(int2) + (size_t)W * per_wave;
  static bool attr_set = false;  // the kernel's LDS ceiling (at most 144 KB + one list), raised once per process
  if (lds > 48 * 1024 && !attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k2_merge<NQ, HW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)((K2_LS + K2_PAD) * sizeof(int2) + 144 * 1024));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  k2_merge<NQ, HW><<<dim3(a.S), dim3(64 * W), lds, st>>>(a);
  return hipGetLastError();
}

// A vocabulary shard's partial lists hold shard-local words; this moves them
// to the shard's place in the whole vocabulary.  Empty entries (word -1 or
// INT_MAX, score below every real one) keep their word.
__global__ __launch_bounds__(256) void add_word_base(int2* __restrict__ lists, size_t n, int base, int v_shard) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const int w = lists[i].y;
    if ((unsigned)w < (unsigned)v_shard) lists[i].y = w + base;
  }
}

hipError_t launch_add_word_base(int2* lists, size_t n, int base, int v_shard, hipStream_t st) {
  if (n == 0 || base == 0) return hipSuccess;
  const int blocks = (int)std::min<size_t>((n + 255) / 256, 2048);
  add_word_base<<<dim3(blocks), dim3(256), 0, st>>>(lists, n, base, v_shard);
  return hipGetLastError();
}

hipError_t launch_k2(const K2Args& a, hipStream_t st) {
  if (a.P < 1 || a.P > K2_MAXP || a.k < 1 || a.k > K2_LS) return hipErrorInvalidValue;
  if (a.S <= 0) return hipSuccess;
  // two waves a row past 128 splits, and for lists of more than 8 past 64 (a
  // wave's lists then take one staging batch) where a sentence's rows still
  // fit in one go
  if (a.P > 128) return launch_k2_nq<2, 2>(a, st);
  if (a.P > 64) return a.k > 8 && a.N <= 8 * a.S ? launch_k2_nq<1, 2>(a, st) : launch_k2_nq<2, 1>(a, st);
  return launch_k2_nq<1, 1>(a, st);
}

}  // namespace kb
