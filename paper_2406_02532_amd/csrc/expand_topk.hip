// Draft-side expansion step (Alg. 2: probs -> selectBest by cumulative log-probability).
//
// Kernel 1, row_topk_kernel: one workgroup per expanded node.  The row of V fp32 logits is read
// from HBM exactly once into registers (float4 per lane, fully coalesced), and everything else
// -- max, sum of exponentials, the k best entries -- is computed from those registers.  This is
// the HBM-bound part: 4*V bytes per row in, 8*k bytes out.
// Selection: the k-th largest of the per-thread maxima is a lower bound t0 of the k-th largest
// entry of the row (k distinct threads hold a value >= t0), so only entries >= t0 can be among
// the k best.  For k << V that leaves a few dozen candidates, which are sorted in LDS by
// (value descending, index ascending).  Rows where the bound is useless (massive ties) fall back
// to an exact bitwise threshold search over the same registers.
//
// Vocabularies above 32768 do not fit the registers of such a workgroup: several share the row and
// merge_shares_kernel puts their lists together, or, for few rows and for large k, row_topk_stream_kernel
// streams the row instead (running maximum and rescaled sum per lane) and takes the candidates
// from a second sweep that L2 serves.
//
// Kernel 2, select_kernel: the B best of the N*k candidates by score = cum_logp[row] + logp, ties to the lower flat index,
// in that order.
#include "kernels.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kCandCap = 1024;  // LDS slots for row candidates before the exact fallback is taken

// An entry's place among the others of its row: NaN behind every number (a comparison with the bound passes it by as well).
__device__ __forceinline__ unsigned row_order_key(float x) { return x == x ? f32_order_key(x) : 0u; }

// The first entries equal to t0, in the order of their indices, behind the C entries in cand[] until there are k (fewer if the
// row has no more).  The row comes from L2, from its beginning on: where this is needed ties are the many.
template <int THREADS>
__device__ __noinline__ int append_ties(const float* __restrict__ x, int V, int k, float t0, int C, int* redi,
                                        unsigned long long* cand) {
  constexpr int NW = THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i0 = 0; i0 < V && C < k; i0 += THREADS) {
    const int i = i0 + tid;
    const bool tie = i < V && x[i] == t0;
    const unsigned long long b = __builtin_amdgcn_ballot_w64(tie);
    if (lane == 0) redi[wave] = __builtin_popcountll(b);
    __syncthreads();
    int pos = C + __builtin_popcountll(b & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) pos += redi[w];
      C += redi[w];
    }
    if (tie && pos < k) cand[pos] = ((unsigned long long)(~f32_order_key(t0)) << 32) | (unsigned)i;
    __syncthreads();
    C = min(C, k);
  }
  return C;
}

// Exact selection for rows the cheap bound t0 (at most the k-th largest entry) cannot handle, from L2: the row was just read.
// Mostly the entries equal to t0 are the many (a masked row, or a masked share of one: -inf or one low value almost
// everywhere): one sweep takes those above it, and if there are fewer than k the first equal ones follow.  Otherwise bitwise search for the k-th largest order key, then for the index below which
// ties are taken, each probe being one pass over the row.  (By the search alone 128 rows of 128256 with all but 300 entries
// masked took 2177 us, now 66.)  Returns the number of entries left in cand[], at least k.
template <int THREADS>
__device__ __noinline__ int exact_topk_from_memory(const float* __restrict__ x, int V, int k, float t0, int* redi, int* s_cnt,
                                                   unsigned long long* cand) {
  constexpr int NW = THREADS / 64;
  const int tid = threadIdx.x;
  __syncthreads();  // (everybody has read the count that led here)
  if (tid == 0) *s_cnt = 0;
  __syncthreads();
  constexpr int U = 8;  // loads in flight per lane
  for (int i0 = 0; i0 < V; i0 += U * THREADS) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = i0 + u * THREADS + tid < V ? x[i0 + u * THREADS + tid] : t0;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v[u] > t0) {
        const int pos = atomicAdd(s_cnt, 1);
        if (pos < kCandCap)
          cand[pos] = ((unsigned long long)(~f32_order_key(v[u])) << 32) | (unsigned)(i0 + u * THREADS + tid);
      }
  }
  __syncthreads();
  int C = *s_cnt;
  if (C <= kCandCap) {
    C = append_ties<THREADS>(x, V, k, t0, C, redi, cand);
    if (C >= k) return C;
  }
  unsigned K = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const unsigned trial = K | (1u << bit);
    int c = 0;
    for (int i = tid; i < V; i += THREADS) c += (row_order_key(x[i]) >= trial) ? 1 : 0;
    if (block_sum_i<NW>(c, redi) >= k) K = trial;
  }
  int cg = 0;
  for (int i = tid; i < V; i += THREADS) cg += (row_order_key(x[i]) > K) ? 1 : 0;
  const int need = k - block_sum_i<NW>(cg, redi);  // ties to take, >= 1
  unsigned Y = 0;                                 // largest Y with #(tie, idx < Y) <= need
  for (int bit = 17; bit >= 0; --bit) {
    const unsigned trial = Y | (1u << bit);
    int c = 0;
    for (int i = tid; i < V && (unsigned)i < trial; i += THREADS) c += (row_order_key(x[i]) == K) ? 1 : 0;
    if (block_sum_i<NW>(c, redi) <= need) Y = trial;
  }
  if (tid == 0) *s_cnt = 0;
  __syncthreads();
  for (int i = tid; i < V; i += THREADS) {
    const unsigned key = row_order_key(x[i]);
    if (key > K || (key == K && (unsigned)i < Y)) {
      const int pos = atomicAdd(s_cnt, 1);
      if (pos < kCandCap) cand[pos] = ((unsigned long long)(~key) << 32) | (unsigned)i;
    }
  }
  __syncthreads();
  C = min(*s_cnt, kCandCap);
  __syncthreads();
  return C;
}

// Long rows shared out among several workgroups: each takes `len` entries of a row (a multiple of four) and leaves its k
// best as sort keys, in order, and its maximum and sum of exponentials; merge_shares_kernel puts a row's shares together.
struct RowShares {
  int parts, len;
  unsigned long long* keys;  // [N][parts][k]: (~order key of the value) << 32 | index in the row, ascending
  float2* ms;                // [N][parts]
};

// THREADS lanes, each holding IPT4 float4 of the row.  Element (j, c) of a lane is index
// (j*THREADS + tid)*4 + c.  SHARE: of this workgroup's share of the row.
template <int THREADS, int IPT4, bool VEC, bool SHARE>
__global__ __launch_bounds__(THREADS) void row_topk_kernel(const float* __restrict__ logits,
                                                           const float* __restrict__ cum_logp, int V_row, int k,
                                                           float* __restrict__ topk_logp,
                                                           int* __restrict__ topk_idx,
                                                           float* __restrict__ score, RowShares sh) {
  constexpr int NW = THREADS / 64;
  __shared__ float smax[THREADS];
  __shared__ float redf[32];
  __shared__ float s_gmax[64];
  __shared__ int redi[16];
  __shared__ float s_t0;
  __shared__ int s_cnt;
  __shared__ int s_part[NW][64];  // partial ranks / places, one row per wave
  __shared__ unsigned long long cand[kCandCap];

  const int tid = threadIdx.x;
  const size_t row = SHARE ? blockIdx.x / sh.parts : blockIdx.x;
  const int first = SHARE ? (int)(blockIdx.x % sh.parts) * sh.len : 0;
  const int V = SHARE ? min(sh.len, V_row - first) : V_row;
  const float* x = logits + row * (size_t)V_row + first;
  const float NEG_INF = -__builtin_huge_valf();

  float v[IPT4 * 4];
#pragma unroll
  for (int j = 0; j < IPT4; ++j) {
    const int base = (j * THREADS + tid) * 4;
    if (VEC) {
      if (base < V) {
        const float4 t = *reinterpret_cast<const float4*>(x + base);
        v[4 * j + 0] = t.x; v[4 * j + 1] = t.y; v[4 * j + 2] = t.z; v[4 * j + 3] = t.w;
      } else {
        v[4 * j + 0] = v[4 * j + 1] = v[4 * j + 2] = v[4 * j + 3] = NEG_INF;
      }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[4 * j + c] = (base + c < V) ? x[base + c] : NEG_INF;
    }
  }

  // ---- maxima: per lane, per group of GS lanes (64 groups), per wave -----------------------------
  constexpr int GS = THREADS / 64;
  float tm = NEG_INF;
#pragma unroll
  for (int e = 0; e < IPT4 * 4; ++e) tm = fmaxf(tm, v[e]);
  float gm = tm;
#pragma unroll
  for (int o = 1; o < GS; o <<= 1) gm = fmaxf(gm, __shfl_xor(gm, o, 64));
  const float wmx = wave_max(gm);
  const bool small_k = k <= 64;  // uniform
  if ((tid & 63) == 0) redf[tid >> 6] = wmx;
  if ((tid & (GS - 1)) == 0) s_gmax[tid / GS] = gm;
  if (!small_k) smax[tid] = tm;
  if (tid == 0) s_cnt = 0;
  __syncthreads();  // (1)
  float M = redf[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmaxf(M, redf[w]);

  // ---- sum of exponentials, and the ranks of the group maxima ------------------------------------------
  // t0 = k-th largest of a set of group maxima (rank by value, then group id) is a lower bound of
  // the k-th largest entry.  k <= 64: 64 groups (hardly looser than per-lane maxima and far cheaper),
  // ranked with lane broadcasts by all waves together, each comparing the 64 maxima with its share of
  // 64 / NW of them (all 64 broadcasts on one wave were the longest single-wave stretch of the kernel);
  // the partial ranks meet in LDS at the next barrier.  Larger k: every lane is a group.
  const int lane = tid & 63, wave = tid >> 6;
  float gmine = 0.f;
  if (small_k) {
    gmine = s_gmax[lane];
    int prank = 0;
#pragma unroll
    for (int jj = 0; jj < 64 / NW; ++jj) {
      const int j = __builtin_amdgcn_readfirstlane(wave) * (64 / NW) + jj;
      const float o = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gmine), j));
      prank += (o > gmine || (o == gmine && j < lane)) ? 1 : 0;
    }
    s_part[wave][lane] = prank;
  }
  float se = 0.f;
  const float mshift = -M * kLog2e;
#pragma unroll
  for (int e = 0; e < IPT4 * 4; ++e) se += __builtin_amdgcn_exp2f(fmaf(v[e], kLog2e, mshift));
  se = wave_sum(se);
  if ((tid & 63) == 0) redf[NW + (tid >> 6)] = se;
  if (!small_k) {
    int rank = 0;
    for (int j = 0; j < THREADS; ++j) {
      const float o = smax[j];
      rank += (o > tm || (o == tm && j < tid)) ? 1 : 0;
    }
    if (rank == k - 1) s_t0 = tm;
  }
  __syncthreads();  // (2)
  float S = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) S += redf[NW + w];
  // The shift overflows for a share masked with the lowest number, and is none for one of -inf alone (whose sum is 0,
  // or NaN with a NaN): anew, with the difference to M first.  (As a branch around the loop above 200 rows of 128256 took 34.3 us
  // for 33.5.)
  if (SHARE && !(fabsf(M) < 1e37f)) {
    const float ref = M == NEG_INF ? 0.f : M;
    se = 0.f;
#pragma unroll
    for (int e = 0; e < IPT4 * 4; ++e) se += __builtin_amdgcn_exp2f((v[e] - ref) * kLog2e);
    se = wave_sum(se);
    __syncthreads();
    if ((tid & 63) == 0) redf[NW + (tid >> 6)] = se;
    __syncthreads();
    S = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) S += redf[NW + w];
  }
  const float lse = M + logf(S);
  if (SHARE && tid == 0) sh.ms[blockIdx.x] = make_float2(M, S);
  float t0;
  if (small_k) {  // exactly one group has rank k - 1 (ranks are a permutation of 0..63)
    int rank = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) rank += s_part[w][lane];
    const unsigned long long who = __builtin_amdgcn_ballot_w64(rank == k - 1);
    t0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gmine), __builtin_ctzll(who)));
  } else {
    t0 = s_t0;
  }
  // A share may lie in the masked part of its row while others do not: with many groups at the bound only what is above it is
  // gathered, and ties follow below.  (600 rows of 128256, k = 32, a third masked: 3680 us with the bitwise search, 141 with the
  // sweep from memory, 76 so and without a mask.)
  const bool above = SHARE && __builtin_popcountll(__builtin_amdgcn_ballot_w64(gmine == t0)) > 16;
  const float bound = above ? f32_from_order_key(f32_order_key(t0) + 1u) : t0;  // (above +inf: NaN, which nothing reaches)

  // ---- gather candidates >= t0 ---------------------------------------------------------------
  // Hits are rare (a few dozen per row): the four values of a register quad are looked at only where the
  // quad's maximum of some lane of the wave reaches t0 -- two instructions and one scalar branch per quad.
#pragma unroll
  for (int j = 0; j < IPT4; ++j) {
    const float m4 = fmaxf(fmaxf(v[4 * j + 0], v[4 * j + 1]), fmaxf(v[4 * j + 2], v[4 * j + 3]));
    if (__builtin_amdgcn_ballot_w64(m4 >= bound) != 0ull) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int idx = (j * THREADS + tid) * 4 + c;
        if (v[4 * j + c] >= bound && idx < V) {
          const int pos = atomicAdd(&s_cnt, 1);
          if (pos < kCandCap)
            cand[pos] = ((unsigned long long)(~f32_order_key(v[4 * j + c])) << 32) | (unsigned)idx;
        }
      }
    }
  }
  __syncthreads();  // (3)
  int C = s_cnt;
  const float cl = cum_logp ? cum_logp[row] : 0.f;
  if (SHARE && above && C < k) C = append_ties<THREADS>(x, V, k, t0, C, redi, cand);
  // the bound was useless (massive ties), or the row has fewer than k numbers: exact search, re-reading the row from L2
  if (C > kCandCap || C < k) C = exact_topk_from_memory<THREADS>(x, V, k, t0, redi, &s_cnt, cand);

  if (small_k && C <= 64) {
    // ---- the usual case: a few dozen candidates, ordered in registers ------------------------------------
    // Keys are distinct (the index is part of them), so a candidate's place is the number of smaller keys:
    // scalar broadcasts and compares, no sorting network and no cross-lane latency chain.  Every wave holds
    // all candidates (lane = candidate) and counts against its share of 64 / NW of them.
    const unsigned long long x64 = lane < C ? cand[lane] : ~0ull;
    const unsigned xlo = (unsigned)x64, xhi = (unsigned)(x64 >> 32);
    int pplace = 0;
#pragma unroll
    for (int jj = 0; jj < 64 / NW; ++jj) {
      const int j = __builtin_amdgcn_readfirstlane(wave) * (64 / NW) + jj;
      const unsigned olo = __builtin_amdgcn_readlane(xlo, j), ohi = __builtin_amdgcn_readlane(xhi, j);
      pplace += (ohi < xhi || (ohi == xhi && olo < xlo)) ? 1 : 0;
    }
    s_part[wave][lane] = pplace;  // (the ranks in there were read before barrier (3))
    __syncthreads();  // (4)
    if (tid >= 64) return;
    int place = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) place += s_part[w][lane];
    if (SHARE) {
      if (tid < C && place < k) sh.keys[blockIdx.x * (size_t)k + place] = x64 + (unsigned)first;
    } else if (tid < C && place < k) {
      const float val = f32_from_order_key(~xhi);
      const float lp = val - lse;
      const size_t o = row * (size_t)k + place;
      topk_idx[o] = (int)xlo;
      topk_logp[o] = lp;
      if (score) score[o] = cl + lp;
    }
    return;
  }
  __syncthreads();

  // ---- general case: order the candidates in LDS and emit the first k --------------------------------
  const int n = next_pow2(C < 2 ? 2 : C);
  for (int i = C + tid; i < n; i += THREADS) cand[i] = ~0ull;
  block_bitonic_sort_u64<THREADS>(cand, n);
  for (int c = tid; c < k; c += THREADS) {
    const unsigned long long e = cand[c];
    if (SHARE) {
      sh.keys[blockIdx.x * (size_t)k + c] = e + (unsigned)first;
      continue;
    }
    const float val = f32_from_order_key(~(unsigned)(e >> 32));
    const float lp = val - lse;
    const size_t o = row * (size_t)k + c;
    topk_idx[o] = (int)(unsigned)(e & 0xFFFFFFFFull);
    topk_logp[o] = lp;
    if (score) score[o] = cl + lp;
  }
}

// Lane `tid` owns the float4 slots tid, tid + THREADS, ... of the row (element index 4 * slot + c).
// Pass 1 streams the row from HBM four slots at a time, keeping only a running maximum and a sum of
// exponentials relative to it; pass 2 streams it again, now from L2, and keeps the few entries >= t0.
// Few registers whatever V is: used for vocabularies too large for the register-resident kernel above and not shared out.
template <int THREADS, bool VEC>
__global__ __launch_bounds__(THREADS) void row_topk_stream_kernel(const float* __restrict__ logits,
                                                           const float* __restrict__ cum_logp, int V, int k,
                                                           float* __restrict__ topk_logp,
                                                           int* __restrict__ topk_idx,
                                                           float* __restrict__ score) {
  constexpr int NW = THREADS / 64;
  constexpr int U = 4;  // float4 slots in flight per lane
  __shared__ float smax[THREADS];
  __shared__ float redf[32];
  __shared__ float s_gmax[64];
  __shared__ int redi[16];
  __shared__ float s_t0;
  __shared__ int s_cnt;
  __shared__ unsigned long long cand[kCandCap];

  const int tid = threadIdx.x;
  const size_t row = blockIdx.x;
  const float* x = logits + row * (size_t)V;
  const float NEG_INF = -__builtin_huge_valf();
  const int nslot = (V + 3) / 4;

  // slots [s0, s0 + U * THREADS) of the row into c[U * 4]; out-of-range elements read as -inf
  auto load_chunk = [&](int s0, float (&c)[U * 4]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int slot = s0 + u * THREADS + tid;
      if (VEC) {
        if (slot < nslot) {
          const float4 t = *reinterpret_cast<const float4*>(x + 4 * (size_t)slot);
          c[4 * u + 0] = t.x; c[4 * u + 1] = t.y; c[4 * u + 2] = t.z; c[4 * u + 3] = t.w;
        } else {
          c[4 * u + 0] = c[4 * u + 1] = c[4 * u + 2] = c[4 * u + 3] = NEG_INF;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[4 * u + e] = (4 * slot + e < V) ? x[4 * (size_t)slot + e] : NEG_INF;
      }
    }
  };

  // ---- pass 1: lane maximum tm and lane sum se of exp(x - tm), rescaled whenever tm rises ----------------
  float tm = NEG_INF, se = 0.f;
  for (int s0 = 0; s0 < nslot; s0 += U * THREADS) {
    float c[U * 4];
    load_chunk(s0, c);
    float cm = c[0];
#pragma unroll
    for (int e = 1; e < U * 4; ++e) cm = fmaxf(cm, c[e]);
    if (cm > tm) {  // also the first finite chunk: exp2(-inf) = 0 clears the (empty) sum
      se *= __builtin_amdgcn_exp2f((tm - cm) * kLog2e);
      tm = cm;
    }
    if (tm > NEG_INF) {
#pragma unroll
      for (int e = 0; e < U * 4; ++e) se += __builtin_amdgcn_exp2f((c[e] - tm) * kLog2e);
    } else {  // nothing above -inf yet: adds 0, or NaN
#pragma unroll
      for (int e = 0; e < U * 4; e += 2) se = __builtin_isunordered(c[e], c[e + 1]) ? __builtin_nanf("") : se;
    }
  }

  // ---- maxima: per group of GS lanes (64 groups), per wave ---------------------------------------------
  constexpr int GS = THREADS / 64;
  float gm = tm;
#pragma unroll
  for (int o = 1; o < GS; o <<= 1) gm = fmaxf(gm, __shfl_xor(gm, o, 64));
  const float wmx = wave_max(gm);
  const bool small_k = k <= 64;  // uniform
  if ((tid & 63) == 0) redf[tid >> 6] = wmx;
  if ((tid & (GS - 1)) == 0) s_gmax[tid / GS] = gm;
  if (!small_k) smax[tid] = tm;
  if (tid == 0) s_cnt = 0;
  __syncthreads();  // (1)
  float M = redf[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) M = fmaxf(M, redf[w]);

  // ---- lane sums brought to the row maximum; meanwhile wave 0 ranks the group maxima -----------------------
  // t0 = k-th largest of a set of group maxima (rank by value, then group id) is a lower bound of
  // the k-th largest entry.  k <= 64: 64 groups ranked by one wave with lane broadcasts (hardly
  // looser than per-lane maxima and far cheaper); else every lane is a group.
  se = tm > NEG_INF ? se * __builtin_amdgcn_exp2f((tm - M) * kLog2e) : se;
  se = wave_sum(se);
  if ((tid & 63) == 0) redf[NW + (tid >> 6)] = se;
  if (small_k) {
    if (tid < 64) {
      const float g = s_gmax[tid];
      int rank = 0;
#pragma unroll
      for (int j = 0; j < 64; ++j) {
        const float o = __shfl(g, j, 64);
        rank += (o > g || (o == g && j < tid)) ? 1 : 0;
      }
      if (rank == k - 1) s_t0 = g;
    }
  } else {
    int rank = 0;
    for (int j = 0; j < THREADS; ++j) {
      const float o = smax[j];
      rank += (o > tm || (o == tm && j < tid)) ? 1 : 0;
    }
    if (rank == k - 1) s_t0 = tm;
  }
  __syncthreads();  // (2)
  float S = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) S += redf[NW + w];
  const float lse = M + logf(S);
  const float t0 = s_t0;

  // ---- pass 2: gather candidates >= t0 (the row comes from L2 this time) -------------------------------
  // Hits are rare (a few dozen per row): one compare and one scalar branch per value, and the divergent
  // code only where some lane of the wave has one.  A lane whose maximum is below t0 holds none, and a
  // wave of such lanes skips its share of the row altogether.
  if (__builtin_amdgcn_ballot_w64(tm >= t0) != 0ull) {
    for (int s0 = 0; s0 < nslot; s0 += U * THREADS) {
      float c[U * 4];
      load_chunk(s0, c);
#pragma unroll
      for (int e = 0; e < U * 4; ++e) {
        const bool hit = c[e] >= t0;
        if (__builtin_amdgcn_ballot_w64(hit) != 0ull) {
          const int idx = 4 * (s0 + (e >> 2) * THREADS + tid) + (e & 3);
          if (hit && idx < V) {
            const int pos = atomicAdd(&s_cnt, 1);
            if (pos < kCandCap) cand[pos] = ((unsigned long long)(~f32_order_key(c[e])) << 32) | (unsigned)idx;
          }
        }
      }
    }
  }
  __syncthreads();  // (3)
  int C = s_cnt;
  const float cl = cum_logp ? cum_logp[row] : 0.f;
  if (C > kCandCap || C < k) C = exact_topk_from_memory<THREADS>(x, V, k, t0, redi, &s_cnt, cand);  // as above

  if (small_k && C <= 64) {
    // ---- the usual case: a few dozen candidates, placed by one wave in registers --------------------
    // keys are distinct (the index is part of them), so a candidate's place is the number of smaller
    // keys: 64 scalar broadcasts and compares, no sorting network and no cross-lane latency chain
    if (tid >= 64) return;
    const unsigned long long x64 = tid < C ? cand[tid] : ~0ull;
    const unsigned xlo = (unsigned)x64, xhi = (unsigned)(x64 >> 32);
    int place = 0;
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      const unsigned olo = __builtin_amdgcn_readlane(xlo, j), ohi = __builtin_amdgcn_readlane(xhi, j);
      place += (ohi < xhi || (ohi == xhi && olo < xlo)) ? 1 : 0;
    }
    if (tid < C && place < k) {
      const float val = f32_from_order_key(~xhi);
      const float lp = val - lse;
      const size_t o = row * (size_t)k + place;
      topk_idx[o] = (int)xlo;
      topk_logp[o] = lp;
      if (score) score[o] = cl + lp;
    }
    return;
  }
  __syncthreads();

  // ---- general case: order the candidates in LDS and emit the first k --------------------------------
  const int n = next_pow2(C < 2 ? 2 : C);
  for (int i = C + tid; i < n; i += THREADS) cand[i] = ~0ull;
  block_bitonic_sort_u64<THREADS>(cand, n);
  for (int c = tid; c < k; c += THREADS) {
    const unsigned long long e = cand[c];
    const float val = f32_from_order_key(~(unsigned)(e >> 32));
    const float lp = val - lse;
    const size_t o = row * (size_t)k + c;
    topk_idx[o] = (int)(unsigned)(e & 0xFFFFFFFFull);
    topk_logp[o] = lp;
    if (score) score[o] = cl + lp;
  }
}

// A row's shares put together: a key's place is its place in its own list and the number of smaller keys in the others, by
// binary search.  Dynamic LDS: the parts * k keys.
constexpr int kMergeThreads = 256;
__global__ __launch_bounds__(kMergeThreads) void merge_shares_kernel(RowShares sh, const float* __restrict__ cum_logp, int k,
                                                                     float* __restrict__ topk_logp, int* __restrict__ topk_idx,
                                                                     float* __restrict__ score) {
  extern __shared__ unsigned long long lists[];
  const size_t row = blockIdx.x;
  const int n = sh.parts * k;
  for (int i = threadIdx.x; i < n; i += kMergeThreads) lists[i] = sh.keys[row * n + i];
  float M = -__builtin_huge_valf(), S = 0.f;
  for (int p = 0; p < sh.parts; ++p) M = fmaxf(M, sh.ms[row * sh.parts + p].x);
  for (int p = 0; p < sh.parts; ++p) {  // (a share of -inf alone adds 0, one with a NaN makes the row's sum NaN)
    const float2 t = sh.ms[row * sh.parts + p];
    // The share's exponents were shifted by t.x log2(e) rounded, all of them by the same error, which is taken back here (left
    // in, the scores of 256 rows of 50000 around 5000 were off by up to 0.75 units in the log-sum-exp's last place; streamed 0.5).
    const float r = fabsf(t.x) < 1e37f ? fmaf(-t.x, kLog2e, t.x * kLog2e) : 0.f;
    S += t.y * __builtin_amdgcn_exp2f((t.x == M ? 0.f : (t.x - M) * kLog2e) + r);
  }
  const float lse = M + logf(S), cl = cum_logp ? cum_logp[row] : 0.f;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kMergeThreads) {
    const unsigned long long e = lists[i];
    const int p = i / k;
    int place = i - p * k;
    for (int q = 0; q < sh.parts; ++q) {
      if (q == p) continue;
      int lo = 0, hi = k;  // smaller keys of list q
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (lists[q * k + mid] < e) lo = mid + 1;
        else hi = mid;
      }
      place += lo;
    }
    if (place < k) {
      const float lp = f32_from_order_key(~(unsigned)(e >> 32)) - lse;
      const size_t o = row * (size_t)k + place;
      topk_idx[o] = (int)(unsigned)e;
      topk_logp[o] = lp;
      if (score) score[o] = cl + lp;
    }
  }
}

// The Bsel best of n candidates, in order.  What bounds it is a chain of block-wide steps, so it is short: select_kernel
// below, in many workgroups, counts places; only where very many scores are equal or close does one workgroup of 1024 lanes
// do it by histograms:
//   threshold   with d = (largest order key) - (order key), the smallest D with #(d <= D) >= Bsel, by histograms of d in
//               LDS: 4096 bins of 2^14 keys (512 per octave of the scores, 8 octaves below the best; bins of an eighth of
//               an octave made a row's candidates meet in one bin, and their atomics queue), then bins of 4, then single
//               keys, as far as needed.  Scores further apart (-inf among the winners) take bins over all 32 bits.  Equal
//               scores need no threshold, and ties are ranked 4096 at a time until enough are found;
//   order       the winners fall into 4096 buckets of equal key range (two per bucket at most on average), are placed
//               by a scan of the bucket counts and ranked inside their bucket by counting smaller entries.  Where one
//               bucket holds more than kBucketMax (many equal scores) they go through a sorting network instead.
constexpr int kSelThreads = 1024;
constexpr int kSelBins = 4096;
constexpr unsigned kBucketMax = 32;
constexpr int kPlaceCap = 8192;     // candidates whose places are counted: beyond that, counting takes longer than histograms
constexpr int kSelBlocks = 256;     // workgroups at most
constexpr int kSamplesPerLane = 6;  // at most
constexpr unsigned kShareHash = 2654435761u;  // bits 16 and up of flat index * this: whose entry it is
// order key of a candidate: never 0, which marks the slots past the end (only one NaN pattern would map there)
__device__ __forceinline__ unsigned select_key(float v) { return max(f32_order_key(v), 1u); }

// Exclusive sum over the lanes of `mine`, every lane of the workgroup calling.
__device__ __forceinline__ int block_exclusive_scan(int mine, int* s_wave) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += s_wave[w];
  return before + incl - mine;
}

// The `keep` smallest of L <= 8192 distinct entries (distance from the best score << 32 | flat index), in order, to the
// outputs; distances are at most `range`.  `placed` has room for L entries, or for the padding to a power of two of
// sbuf's; hist is clear, *s_big zero.
__device__ __forceinline__ void order_and_emit(unsigned long long* sbuf, unsigned long long* placed, int L, int keep,
                                               unsigned range, unsigned* hist, int* s_wave, unsigned* s_big,
                                               const float* __restrict__ score, const int* __restrict__ topk_idx, int k,
                                               int* __restrict__ out_row, int* __restrict__ out_token,
                                               float* __restrict__ out_score) {
  constexpr int E = 8192 / kSelThreads, BPT = kSelBins / kSelThreads;
  const int tid = threadIdx.x;
  auto emit = [&](int place, unsigned flat) {
    if (place >= keep) return;
    out_row[place] = (int)(flat / (unsigned)k);
    out_token[place] = topk_idx[flat];
    out_score[place] = score[flat];
  };
  const int shift = range < (unsigned)kSelBins ? 0 : 32 - 12 - __builtin_clz(range);  // range >> shift < 4096
  unsigned bucket[E], slot[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = e * kSelThreads + tid;
    bucket[e] = slot[e] = 0;
    if (i < L) {
      bucket[e] = min((unsigned)(sbuf[i] >> 32) >> shift, (unsigned)(kSelBins - 1));
      slot[e] = atomicAdd(&hist[bucket[e]], 1u);
      if (slot[e] >= kBucketMax) *s_big = 1;
    }
  }
  __syncthreads();
  if (*s_big == 0) {
    int mine = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) mine += (int)hist[tid * BPT + i];
    int start = block_exclusive_scan(mine, s_wave);
#pragma unroll
    for (int i = 0; i < BPT; ++i) {  // each lane turns its own four counts into first place << 8 | count
      const unsigned h = hist[tid * BPT + i];
      hist[tid * BPT + i] = ((unsigned)start << 8) | h;
      start += (int)h;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = e * kSelThreads + tid;
      if (i < L) placed[(hist[bucket[e]] >> 8) + slot[e]] = sbuf[i];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = e * kSelThreads + tid;
      if (i < L) {
        const unsigned h = hist[bucket[e]], first = h >> 8, cnt = h & 255u;
        const unsigned long long me = sbuf[i];
        int place = (int)first;
        for (unsigned j = 0; j < cnt; ++j) place += placed[first + j] < me ? 1 : 0;
        emit(place, (unsigned)me);
      }
    }
  } else {
    const int nsort = next_pow2(L < 2 ? 2 : L);
    for (int i = L + tid; i < nsort; i += kSelThreads) sbuf[i] = ~0ull;
    block_bitonic_sort_u64<kSelThreads>(sbuf, nsort);
    for (int i = tid; i < keep; i += kSelThreads) emit(i, (unsigned)(sbuf[i] & 0xFFFFFFFFull));
  }
}

// sbuf: winners, then room to place them: 2 x next_pow2(Bsel).  QUADS > 0 (n <= 4096 QUADS): lane t holds the keys of the
// candidates 4 (j 1024 + t) .. + 3, j < QUADS, in registers; 0: every pass re-reads them, which beyond 16384 candidates costs
// less than the code it takes to hold them (8192 of 16200: 33 us with four, 37 re-read).
template <int QUADS>
__device__ __forceinline__ void select_by_one(const float* __restrict__ score, const int* __restrict__ topk_idx, int n, int k,
                                              int B, int* __restrict__ out_row, int* __restrict__ out_token,
                                              float* __restrict__ out_score, int* __restrict__ n_out,
                                              unsigned long long* sbuf, unsigned* hist, int* s_wave) {
  constexpr int BPT = kSelBins / kSelThreads, R = QUADS > 0 ? QUADS * 4 : 1;
  __shared__ unsigned s_max, s_min, s_big;
  __shared__ int s_pos, s_bin, s_above;

  const int tid = threadIdx.x, lane = tid & 63;
  const int Bsel = min(B, n);

  // f(four order keys, flat index of the first) over the candidates in memory, U quads in flight per lane.  (A rolled
  // loop on purpose: with 64 keys a lane in registers every pass is 64 copies of its body, and a workgroup that runs
  // through them once waits for instructions: 63 us against 48.)
  auto stream = [&](auto f) {
    constexpr int U = 4;
    for (int i0 = 0; i0 < n; i0 += U * 4 * kSelThreads) {
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + (u * kSelThreads + tid) * 4;
        if (i + 4 <= n) {
          v[u] = *reinterpret_cast<const f32x4*>(score + i);
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) v[u][c] = i + c < n ? score[i + c] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + (u * kSelThreads + tid) * 4;
        unsigned t[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = i + c < n ? select_key(v[u][c]) : 0u;
        f(t[0], t[1], t[2], t[3], i);
      }
    }
  };
  unsigned d[R];  // first the order key (slots past n: 0, below every real key), then its distance from the largest
  if constexpr (QUADS > 0) {
    f32x4 v[QUADS];
#pragma unroll
    for (int j = 0; j < QUADS; ++j) {
      const int i = (j * kSelThreads + tid) * 4;
      if (i + 4 <= n) {
        v[j] = *reinterpret_cast<const f32x4*>(score + i);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[j][c] = i + c < n ? score[i + c] : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < R; ++e) d[e] = ((e / 4) * kSelThreads + tid) * 4 + e % 4 < n ? select_key(v[e / 4][e % 4]) : 0u;
  }
  unsigned top = 0;
  auto clear = [&]() {
    *reinterpret_cast<u32x4*>(hist + 4 * tid) = u32x4{0u, 0u, 0u, 0u};
  };
  // sum of hist over the bins that come before this lane's four
  auto scan = [&]() -> int {
    int mine = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) mine += (int)hist[tid * BPT + i];
    return block_exclusive_scan(mine, s_wave);
  };

  clear();
  if (tid == 0) {
    s_pos = 0;
    s_max = 0;
    s_min = 0xFFFFFFFFu;
    s_big = 0;
    s_bin = 0;
    s_above = n;
  }
  __syncthreads();
  unsigned low = 0xFFFFFFFFu;  // one less than the smallest key (a slot past n: the largest number)
  if constexpr (QUADS > 0) {
#pragma unroll
    for (int e = 0; e < R; ++e) top = max(top, d[e]);
  } else {
    stream([&](unsigned a, unsigned b, unsigned c, unsigned e, int) {
      top = max(top, max(max(a, b), max(c, e)));
      low = min(low, min(min(a - 1u, b - 1u), min(c - 1u, e - 1u)));
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) low = min(low, (unsigned)__shfl_xor((int)low, o, 64));
    if (lane == 0) atomicMin(&s_min, low);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, o, 64));
  if (lane == 0) atomicMax(&s_max, top);
  __syncthreads();
  const unsigned kmax = s_max;  // slots past n end up at d == kmax, beyond every real key
  // f(four d, flat index of the first) over all candidates of this lane, in the same number of calls for every lane
  if constexpr (QUADS > 0) {
    unsigned differ = 0;
#pragma unroll
    for (int e = 0; e < R; ++e) {
      d[e] = kmax - d[e];
      differ |= ((e / 4) * kSelThreads + tid) * 4 + e % 4 < n ? d[e] : 0u;
    }
    if (differ) s_min = 0;
    __syncthreads();
  }
  const bool equal = QUADS > 0 ? s_min != 0 : s_min + 1u == kmax;
  auto each4 = [&](auto f) {
    if constexpr (QUADS > 0) {
#pragma unroll
      for (int j = 0; j < QUADS; ++j) f(d[4 * j], d[4 * j + 1], d[4 * j + 2], d[4 * j + 3], (j * kSelThreads + tid) * 4);
      return;
    }
    stream([&](unsigned a, unsigned b, unsigned c, unsigned e, int i) { f(kmax - a, kmax - b, kmax - c, kmax - e, i); });
  };

  // ---- threshold ---------------------------------------------------------------------------------------
  unsigned D = 0xFFFFFFFFu;
  int need = Bsel, ties = Bsel;  // of the candidates in the threshold's last bin: how many are taken, how many there are
  if (n > Bsel && equal) {  // all scores equal: the first ones are taken
    D = 0;
    ties = n;
  } else if (n > Bsel) {
    unsigned prefix = 0;
    int above = 0, shift = 14, bits = 12;
    bool first = true, wide = false;
    while (true) {
      if (first) {
        each4([&](unsigned a, unsigned b, unsigned c, unsigned e, int) {
          const unsigned t[4] = {a, b, c, e};
#pragma unroll
          for (int i = 0; i < 4; ++i) atomicAdd(&hist[min(t[i] >> shift, (unsigned)(kSelBins - 1))], 1u);
        });
      } else {
        each4([&](unsigned a, unsigned b, unsigned c, unsigned e, int) {
          const unsigned t[4] = {a, b, c, e};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((t[i] >> (shift + bits)) == prefix && t[i] != kmax) atomicAdd(&hist[(t[i] >> shift) & ((1u << bits) - 1u)], 1u);
        });
      }
      __syncthreads();
      int start = above + scan();
#pragma unroll
      for (int i = 0; i < BPT; ++i) {
        const int h = (int)hist[tid * BPT + i];
        if (start < Bsel && start + h >= Bsel) {
          s_bin = tid * BPT + i;
          s_above = start;
        }
        start += h;
      }
      __syncthreads();
      const unsigned b = (unsigned)s_bin;
      const int at = s_above, h = (int)hist[b];
      __syncthreads();
      clear();
      __syncthreads();
      if (first && !wide && b == (unsigned)(kSelBins - 1)) {  // beyond 8 octaves: again, over all 32 bits
        wide = true;
        shift = 20;
        continue;
      }
      first = false;
      above = at;
      prefix = (prefix << bits) | b;
      need = Bsel - above;
      ties = h;
      D = shift ? ((prefix + 1u) << shift) - 1u : prefix;
      if (ties == need || shift == 0) break;
      bits = min(shift, 12);  // 14 -> 2 -> 0, or 20 -> 8 -> 0
      shift -= bits;
    }
  }

  // ---- winners: every d <= D where they are Bsel; else every d < D and of the d == D the `need` lowest flat indices
  const bool all_ties = ties == need;
  const unsigned take = all_ties ? D : D - 1u;  // (not all ties: some are better than D, or D = 0 and take wraps)
  const bool none = !all_ties && D == 0;
  if (!none) each4([&](unsigned a, unsigned b, unsigned c, unsigned e, int flat) {
    if (__builtin_amdgcn_ballot_w64(min(min(a, b), min(c, e)) <= take) == 0ull) return;
    const unsigned t[4] = {a, b, c, e};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool hit = t[i] <= take && flat + i < n;
      const unsigned long long who = __builtin_amdgcn_ballot_w64(hit);
      if (who == 0ull) continue;
      const int leader = __builtin_ctzll(who);
      int pos = 0;
      if (lane == leader) pos = atomicAdd(&s_pos, __builtin_popcountll(who));
      pos = __builtin_amdgcn_readlane(pos, leader) + __builtin_popcountll(who & ((1ull << lane) - 1ull));
      if (hit && pos < Bsel) sbuf[pos] = ((unsigned long long)t[i] << 32) | (unsigned)(flat + i);
    }
  });
  if (__builtin_expect(!all_ties, 0)) {
    // More candidates at D than fit: the `need` lowest flat indices, 4096 candidates at a time, a scan over the lanes' quads
    // giving each its rank, until enough are found.
    int found = 0;
#pragma unroll 1
    for (int i0 = 0; i0 < n && found < need; i0 += 4 * kSelThreads) {
      const int i = i0 + 4 * tid;
      unsigned tie = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (i + c < n && kmax - select_key(score[i + c]) == D) tie |= 1u << c;
      int rank = found + block_exclusive_scan(__builtin_popcount(tie), s_wave);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (tie >> c & 1) {
          if (rank < need) sbuf[Bsel - need + rank] = ((unsigned long long)D << 32) | (unsigned)(i + c);
          ++rank;
        }
      if (tid == kSelThreads - 1) s_above = rank;
      __syncthreads();
      found = s_above;
      __syncthreads();
    }
  }
  __syncthreads();

  order_and_emit(sbuf, sbuf + next_pow2(Bsel < 2 ? 2 : Bsel), Bsel, Bsel, min(D, kmax), hist, s_wave, &s_big, score, topk_idx, k,
                 out_row, out_token, out_score);
  if (tid == 0) n_out[0] = Bsel;
}

// In many workgroups: each of them gathers, in LDS, a set of at most kPlaceCap candidates that holds the Bsel best -- all of
// them, or those from a threshold up that the order keys of one candidate out of every few set a few deviations beyond Bsel --
// and its waves count, for their share of the set, the better ones: a ballot and a bit count per 64 entries.  Candidates that
// tie at the threshold (equal scores; the -inf of dead rows) are not gathered: they fill the places that the set leaves, in
// index order.  All workgroups gather the same set (read 256 times, by 256 compute units at once, 256 KB of scores take them
// 4 us) and write disjoint places, so nobody waits for anybody, and the order in which LDS atomics fill a set does not show.
// 65536 candidates, 2048 picks: 19 us, by histograms in one workgroup 31; where the scores lie close together 24 and 175; with
// -inf among the picks 22 and 286; all equal 17 and 60.  3200 candidates, 100 picks: 6.3 and 7.8; 8192 candidates, 64
// picks 4.3 (all of them counted: 11.3) and 10.3.  From 6144 picks on, where counting would take longer, one
// workgroup does it: 8192 of 16000 33 us.
template <int QUADS>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float* __restrict__ score, const int* __restrict__ topk_idx,
                                                             int n, int k, int B, bool count, int* __restrict__ out_row,
                                                             int* __restrict__ out_token, float* __restrict__ out_score,
                                                             int* __restrict__ n_out) {
  typedef unsigned long long u64;
  extern __shared__ __attribute__((aligned(16))) u64 keys[];  // [kPlaceCap] the set: ~order key << 32 | flat index
  __shared__ __attribute__((aligned(16))) unsigned hist[kSelBins];
  __shared__ int s_wave[kSelThreads / 64];
  __shared__ int s_cnt, s_bad, s_own, s_bin, s_above, s_in;
  __shared__ unsigned s_tied, s_first, s_mixed;
  // [kSelBins]: this workgroup's entries, by a hash of the flat index (select_blocks() keeps a workgroup's share of all flat
  // indices below that)
  u64* const own = keys + kPlaceCap;
  const int tid = threadIdx.x, lane = tid & 63;
  const int Bsel = min(B, n);
  auto entry = [](unsigned key, int flat) { return ((u64)~key << 32) | (unsigned)flat; };
  auto claim = [&](u64 e) {
    if (((unsigned)e * kShareHash >> 16 & (gridDim.x - 1u)) != blockIdx.x) return;
    const int at = atomicAdd(&s_own, 1);
    if (at < kSelBins) own[at] = e;  // always
  };
  int W = n, bad = 0;  // size of the set, entries that are none
  unsigned tied = 0;   // key of the score that fills the places which the set leaves
  if (tid == 0) s_own = s_cnt = s_bad = s_mixed = 0;
  *reinterpret_cast<u32x4*>(hist + 4 * tid) = u32x4{0u, 0u, 0u, 0u};  // the places so far of `own`
  __syncthreads();
  auto pad = [&](int i) {  // the set ends with entries worse than any, in whole steps of the count
    for (; i < (W + 4095 & ~4095); i += kSelThreads) keys[i] = ~0ull;
  };
  if (!count) {
    W = -1;
  } else if (n <= kPlaceCap / 2 || (n <= kPlaceCap && 4 * Bsel > n)) {
    for (int i = tid; i < n; i += kSelThreads) {
      const u64 e = entry(select_key(score[i]), i);
      keys[i] = e;
      claim(e);
    }
    pad(n + tid);
    __syncthreads();
  } else {
    // ---- the threshold: the want-th best of the samples, from the upper 14 bits of their keys (32 bins per octave of the
    // scores), and from the next 14 where that bin holds too much ------------------------------------------------------
    constexpr int E = kSamplesPerLane, kBins = 16384, BPT = kBins / kSelThreads;
    // A sample per lane takes 0.6 us; fewer of them make a larger set, to be on the safe side, or a set that is missed.  16384
    // candidates, 256 picks: 10.4 us with one, 11.9 with four; 65536, 2048 picks: 24.3 with one, 19.5 with three, 20.1 with
    // four, 21.3 with six; 524288, 2048 picks: 59.1, 59.0 and 66.6 with three, six and sixteen, but 6000 picks leave a deviation
    // to either side with three.  (Fewer samples than candidates: every range below has one.)
    const int per_lane = n <= 24576 ? 1 : n <= 131072 ? 3 : E, samples = per_lane * kSelThreads;
    unsigned* const bins = reinterpret_cast<unsigned*>(keys);
    unsigned sample[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      sample[e] = 0;
      if (e >= per_lane) continue;
      const unsigned i = e * kSelThreads + tid;
      const unsigned lo = (unsigned)((u64)i * (unsigned)n / samples), hi = (unsigned)((u64)(i + 1) * (unsigned)n / samples);
      sample[e] = select_key(score[lo + (i * kShareHash >> 8) % (hi - lo)]);  // (rows are sorted: not always the same rank)
    }
    // four deviations beyond Bsel, or midway to what the set holds
    const float per_sample = (float)n / samples, mean = (float)Bsel / per_sample;
    const int want = min((int)min(mean + 4.0f * sqrtf(mean) + 8.0f, 0.5f * (mean + kPlaceCap / per_sample)), samples);
    unsigned thr = 0;
    int above = 0;
    if (tid == 0) s_first = sample[0];
#pragma unroll 1
    for (int shift = 18; shift >= 4; shift -= 14) {
#pragma unroll
      for (int i = 0; i < BPT / 4; ++i) *reinterpret_cast<u32x4*>(bins + 4 * (i * kSelThreads + tid)) = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
      bool mixed = false;
#pragma unroll
      for (int e = 0; e < E; ++e) mixed |= e < per_lane && sample[e] != s_first;
      if (mixed) s_mixed = 1;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e < per_lane && (shift == 18 || (sample[e] ^ thr) >> 18 == 0)) {
          // (many equal scores: one add for the lanes that are here; 64 to one address are 64 adds, one after the other)
          const unsigned bin = (sample[e] >> shift) & (kBins - 1), one = (unsigned)__builtin_amdgcn_readfirstlane((int)bin);
          const u64 same = __builtin_amdgcn_ballot_w64(bin == one);
          if (bin != one) atomicAdd(&bins[bin], 1u);
          else if (lane == __builtin_ctzll(same)) atomicAdd(&bins[bin], (unsigned)__builtin_popcountll(same));
        }
      __syncthreads();
      if (s_mixed == 0) {  // all samples equal
        tied = s_first;
        break;
      }
      u32x4 h[BPT / 4];  // this lane's bins, the highest first
      int mine = 0;
#pragma unroll
      for (int i = 0; i < BPT / 4; ++i) {
        h[i] = *reinterpret_cast<const u32x4*>(bins + kBins - BPT * (tid + 1) + 4 * (BPT / 4 - 1 - i));
        mine += (int)((h[i][0] + h[i][1]) + (h[i][2] + h[i][3]));
      }
      int start = above + block_exclusive_scan(mine, s_wave);
      if (start < want && start + mine >= want) {
#pragma unroll
        for (int i = 0; i < BPT; ++i) {
          const int c = (int)h[i / 4][3 - i % 4];
          if (start < want && start + c >= want) {
            s_bin = kBins - 1 - BPT * tid - i;
            s_above = start;
            s_in = start + c;
          }
          start += c;
        }
      }
      __syncthreads();
      thr |= (unsigned)s_bin << shift;
      above = s_above;
      if ((float)s_in * per_sample <= 0.8f * kPlaceCap && s_in <= 2 * want) break;  // (the same answer in every lane: s_in is read between barriers)
      __syncthreads();
    }
    // Where the threshold is -inf, or one score is so frequent that the bin is too large all the same, the set is what is
    // above that score, and its first candidates in index order fill the places that the set leaves.
    constexpr float kInf = __builtin_huge_valf();
    if (!tied && thr <= f32_order_key(-kInf)) {
      tied = f32_order_key(-kInf);
    } else if (!tied && (float)s_in * per_sample > 0.95f * kPlaceCap) {
      if (tid == 0) s_tied = 0;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < E; ++e) tied = e < per_lane && (sample[e] ^ thr) >> 4 == 0 ? max(tied, sample[e]) : tied;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) tied = max(tied, (unsigned)__shfl_xor((int)tied, o, 64));
      if (lane == 0) atomicMax(&s_tied, tied);
      __syncthreads();
      tied = s_tied;
    }
    if (tied) thr = tied + 1u;
    // The set is all keys from thr up, gathered by comparing floats: not less than `least`, its score (the key is monotonic,
    // and -0 counts as +0 in both).  That takes every NaN too, of which those with the sign (keys below -inf's) do not belong
    // to the set and are sorted out where the few hits are stored.  `least` itself cannot be a NaN: not below the key of
    // -inf + 1, and where it is above that of +inf (many equal NaN) the set is given up.
    const float least = f32_from_order_key(thr);
    // ---- the set ---------------------------------------------------------------------------------------------------------
    W = -1;
    if (least <= kInf) {
      __syncthreads();  // the bins have been read
      // 64 scores a lane (16 where that is all), all on their way together; a lane's hits go behind those of the lanes before it, and a wave asks for
      // room once (a ballot and an atomic per element held the waves up for 20 us: every fourth has a hit)
      constexpr int U = QUADS > 0 ? QUADS : 16;
      for (int i0 = 0; i0 < n; i0 += U * 4 * kSelThreads) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + (u * kSelThreads + tid) * 4;
          if (i + 4 <= n) {
            v[u] = *reinterpret_cast<const f32x4*>(score + i);
          } else {  // (no score: below every threshold)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[u][c] = i + c < n ? score[i + c] : -__builtin_huge_valf();
          }
        }
        int hits = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c) hits += v[u][c] < least ? 0 : 1;
        int incl = hits;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int t = __shfl_up(incl, o, 64);
          if (lane >= o) incl += t;
        }
        int at = 0;
        if (lane == 63 && incl) at = atomicAdd(&s_cnt, incl);
        at = __builtin_amdgcn_readlane(at, 63) + incl - hits;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (!(v[u][c] < least)) {  // (as little as possible here: 64 copies of it)
              if (at < kPlaceCap) keys[at] = (u64)__float_as_uint(v[u][c]) << 32 | (unsigned)(i0 + (u * kSelThreads + tid) * 4 + c);
              ++at;
            }
      }
      __syncthreads();
      W = s_cnt;
      for (int i = tid; i < min(W, kPlaceCap); i += kSelThreads) {
        const unsigned key = select_key(__uint_as_float((unsigned)(keys[i] >> 32)));
        const u64 e = key >= thr ? entry(key, (int)(unsigned)keys[i]) : ~0ull;
        keys[i] = e;
        if (key >= thr) claim(e);
        else atomicAdd(&s_bad, 1);
      }
      if (W <= kPlaceCap) pad(W + tid);
      __syncthreads();
      bad = s_bad;
    }
  }
  const int rest = max(Bsel - (W - bad), 0);
  bool alone = W < 0 || (rest > 0 && !tied) || W > kPlaceCap;  // (too few: the samples were off by four deviations)
  if (!alone) {
    // ---- places: a wave holds 1/16 of the set, four entries a lane at a time, and counts for every entry of the workgroup's
    // list (entry e in lane e % 64) how many of them are better ---------------------------------------------------------------
    const int m = s_own;
    for (int j0 = 0; j0 < W; j0 += 4 * kSelThreads) {
      u32x2 other[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) other[r] = *reinterpret_cast<const u32x2*>(keys + j0 + r * kSelThreads + tid);
      for (int e0 = 0; e0 < m; e0 += 64) {
        const u64 mine = own[min(e0 + lane, m - 1)];
        int place = 0;
        for (int e = 0; e < min(64, m - e0); ++e) {
          const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(mine >> 32), e);
          int c = 0;
          u64 equal = 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(other[r][1] < hi));
            equal |= __builtin_amdgcn_ballot_w64(other[r][1] == hi);
          }
          if (equal) {
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)mine, e);
#pragma unroll
            for (int r = 0; r < 4; ++r)
              c += __builtin_popcountll(__builtin_amdgcn_ballot_w64(other[r][1] == hi && other[r][0] < lo));
          }
          place = lane == e ? c : place;
        }
        if (e0 + lane < m && place) atomicAdd(&hist[e0 + lane], (unsigned)place);
      }
    }
    __syncthreads();
    for (int e = tid; e < m; e += kSelThreads) {
      const int p = (int)hist[e];
      if (p < Bsel) {
        const unsigned flat = (unsigned)own[e];
        out_row[p] = (int)(flat / (unsigned)k);
        out_token[p] = topk_idx[flat];
        out_score[p] = score[flat];
      }
    }
    if (blockIdx.x != gridDim.x - 1) return;
    // ---- the last workgroup: the first `rest` candidates of key `tied`, 16384 candidates at a time ---------------------------
    int found = 0;
    for (int i0 = 0; i0 < n && found < rest; i0 += 16 * kSelThreads) {
      const int i = i0 + 16 * tid;
      f32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i + 4 * u + 4 <= n) {
          v[u] = *reinterpret_cast<const f32x4*>(score + i + 4 * u);
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) v[u][c] = i + 4 * u + c < n ? score[i + 4 * u + c] : 0.f;
        }
      }
      unsigned tie = 0;
#pragma unroll
      for (int c = 0; c < 16; ++c)
        if (i + c < n && select_key(v[c / 4][c % 4]) == tied) tie |= 1u << c;
      int rank = found + block_exclusive_scan(__builtin_popcount(tie), s_wave);
      if (tid == kSelThreads - 1) s_cnt = rank + __builtin_popcount(tie);
      for (; tie && rank < rest; tie &= tie - 1, ++rank) {
        const int flat = i + __builtin_ctz(tie), p = Bsel - rest + rank;
        out_row[p] = flat / k;
        out_token[p] = topk_idx[flat];
        out_score[p] = score[flat];
      }
      __syncthreads();
      found = s_cnt;
      __syncthreads();
    }
    alone = found < rest;  // NaN with the sign are among the picks (the others' places are the same)
  }
  if (blockIdx.x != gridDim.x - 1) return;
  __syncthreads();
  if (alone) select_by_one<QUADS>(score, topk_idx, n, k, B, out_row, out_token, out_score, n_out, keys, hist, s_wave);
  else if (tid == 0) n_out[0] = Bsel;
}

// The same for few candidates in one workgroup (64 candidates: 2.4 us, 6.3 by histograms).  Counting one key per lane grows
// with the square: 1024 candidates would take 54 us, select_kernel takes less from some 300 on.
constexpr int kSmallSelect = 256;
__global__ __launch_bounds__(kSelThreads) void small_select_kernel(const float* __restrict__ score,
                                                                   const int* __restrict__ topk_idx, int n, int k, int B,
                                                                   int* __restrict__ out_row, int* __restrict__ out_token,
                                                                   float* __restrict__ out_score, int* __restrict__ n_out) {
  __shared__ unsigned long long keys[kSelThreads];
  const int tid = threadIdx.x;
  float s = 0.f;
  if (tid < n) {
    s = score[tid];
    keys[tid] = ((unsigned long long)(~select_key(s)) << 32) | (unsigned)tid;
  }
  __syncthreads();
  int shift;
  const int place = block_place_u64<kSelThreads>(keys, n, &shift), i = tid >> shift;
  if (i < n && (tid & ((1 << shift) - 1)) == 0 && place < B) {
    out_row[place] = i / k;
    out_token[place] = topk_idx[i];
    out_score[place] = score[i];
  }
  if (tid == 0) n_out[0] = min(B, n);
}

template <int THREADS, int IPT4>
void launch_row(const float* logits, const float* cum, int N, int V, int k, float* lp, int* idx, float* score,
                hipStream_t st) {
  const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(logits) & 15) == 0);
  if (vec)
    row_topk_kernel<THREADS, IPT4, true, false><<<N, THREADS, 0, st>>>(logits, cum, V, k, lp, idx, score, RowShares{});
  else
    row_topk_kernel<THREADS, IPT4, false, false><<<N, THREADS, 0, st>>>(logits, cum, V, k, lp, idx, score, RowShares{});
}

// Workgroups that share a row too long for the registers of one; 1: none.  A row streamed by one workgroup is read twice: with
// the selection, k = 32, 2048 rows of 128256 357 -> 194 us (5.4 TB/s), of 50000 140 -> 100, 256 rows of 128256 51 -> 42.  Not
// for at most 128 rows: alone 100 of 128256 gain too (30.2 -> 25.8), but right after the head that made them the two
// together took 235.9 us for 226.8, the head being slower by more than that.  Shares find k from 33 on too often by
// sorting: their 64 group maxima bound it loosely (600 rows of 80000, k = 56, 88 -> 108 us).
// Rows whose entries are loaded one by one (V not a multiple of 4) gain from lanes instead, up to 128 rows and k = 56 (16 rows of
// 100003, k = 32, 56 -> 22 us), and lose beyond: 2048 rows of 40001 167 -> 179.
constexpr int kShareMaxK = 56;
int row_parts(int N, int V, int k, bool vec) {
  if (V <= 32768 || (vec ? N <= 128 || k > 32 : N > 128 || k > kShareMaxK)) return 1;
  return V <= 65536 ? (N <= 8 ? 4 : 2) : (N <= 16 ? 8 : 4);
}
size_t shares_bytes(size_t shares, int k) { return sx_align_up(shares * 8, 256) + sx_align_up(shares * k * 8, 256); }
// for every call of at most N rows, V entries and k picks, so that a workspace made for the largest serves the others as well
size_t shares_bytes_up_to(int N, int V, int k) {
  return V <= 32768 ? 0 : shares_bytes(N <= 16 ? 8 * (size_t)N : N <= 32 ? 128 : 4 * (size_t)N, k < kShareMaxK ? k : kShareMaxK);
}
template <bool VEC>
void launch_shares(const float* logits, const float* cum, int N, int V, int k, float* lp, int* idx, float* score, void* scratch,
                   hipStream_t st) {
  RowShares sh;
  sh.parts = row_parts(N, V, k, V % 4 == 0);
  sh.len = ((V + sh.parts - 1) / sh.parts + 3) & ~3;
  sh.ms = static_cast<float2*>(scratch);
  sh.keys = reinterpret_cast<unsigned long long*>(static_cast<char*>(scratch) + sx_align_up((size_t)N * sh.parts * 8, 256));
  if (sh.len <= 16384) row_topk_kernel<256, 16, VEC, true><<<N * sh.parts, 256, 0, st>>>(logits, cum, V, k, lp, idx, score, sh);
  else row_topk_kernel<512, 16, VEC, true><<<N * sh.parts, 512, 0, st>>>(logits, cum, V, k, lp, idx, score, sh);
  merge_shares_kernel<<<N, kMergeThreads, (size_t)sh.parts * k * 8, st>>>(sh, cum, k, lp, idx, score);
}

int row_topk_dispatch(const float* logits, const float* cum, int N, int V, int k, float* lp, int* idx, float* score,
                      void* scratch, hipStream_t st) {
  // lanes x float4-per-lane sized so that a row fits in registers with >= 2 workgroups per CU
  if (V <= 1024) launch_row<256, 1>(logits, cum, N, V, k, lp, idx, score, st);
  else if (V <= 4096) launch_row<256, 4>(logits, cum, N, V, k, lp, idx, score, st);
  else if (V <= 16384) launch_row<256, 16>(logits, cum, N, V, k, lp, idx, score, st);
  else if (V <= 32768) launch_row<512, 16>(logits, cum, N, V, k, lp, idx, score, st);
  else {  // the row no longer fits the registers of a workgroup that leaves room for a second one
    const bool vec = (V % 4 == 0) && ((reinterpret_cast<uintptr_t>(logits) & 15) == 0);
    if (scratch && (vec || V % 4 != 0) && row_parts(N, V, k, vec) > 1) {
      if (vec) launch_shares<true>(logits, cum, N, V, k, lp, idx, score, scratch, st);
      else launch_shares<false>(logits, cum, N, V, k, lp, idx, score, scratch, st);
      SX_LAUNCH_CHECK();
      return SX_OK;
    }
    // No more rows than compute units: a row has one to itself, and what it can keep in flight is the bound (64 bytes per
    // lane), so twice the lanes: 100 rows of 128256 36 -> 28.7 us.  Not for k > 64, where every lane ranks its maximum
    // among those of all lanes, which then takes longer than the row (k = 200: 57.7 us with 512 lanes, 68 with 1024).
    if (N <= sx_compute_units() && k <= 64) {
      if (vec) row_topk_stream_kernel<1024, true><<<N, 1024, 0, st>>>(logits, cum, V, k, lp, idx, score);
      else row_topk_stream_kernel<1024, false><<<N, 1024, 0, st>>>(logits, cum, V, k, lp, idx, score);
    } else if (vec) row_topk_stream_kernel<512, true><<<N, 512, 0, st>>>(logits, cum, V, k, lp, idx, score);
    else row_topk_stream_kernel<512, false><<<N, 512, 0, st>>>(logits, cum, V, k, lp, idx, score);
  }
  SX_LAUNCH_CHECK();
  return SX_OK;
}

bool row_shape_ok(int N, int V, int k) {
  return N >= 1 && V >= 1 && V <= 131072 && k >= 1 && k <= 256 && k <= V && (long long)N * k < (1ll << 31);
}

}  // namespace

int sx_launch_row_scores(const float* logits, const float* cum_logp, int N, int V, int k, float* lp, int32_t* idx, float* score,
                         hipStream_t st) {
  if (!row_shape_ok(N, V, k)) return SX_ERR_SHAPE;
  sx_prof_begin(SX_K_ROW_TOPK, st);
  const int rc = row_topk_dispatch(logits, cum_logp, N, V, k, lp, idx, score, nullptr, st);
  sx_prof_end(st);
  return rc;
}

extern "C" int sx_row_logsoftmax_topk(const float* logits, int32_t N, int32_t V, int32_t k, float* topk_logp,
                                      int32_t* topk_idx, void* stream) {
  if (!logits || !topk_logp || !topk_idx) return SX_ERR_NULL;
  if (!row_shape_ok(N, V, k)) return SX_ERR_SHAPE;
  return row_topk_dispatch(logits, nullptr, N, V, k, topk_logp, topk_idx, nullptr, nullptr, (hipStream_t)stream);
}

// workspace: header | score f32[N*k] | topk_logp f32[N*k] | topk_idx i32[N*k] | shares of long rows (used if there)
size_t sx_expand_topk_min_workspace(int N, int k) { return SX_WS_HEADER + 3 * sx_align_up((size_t)N * (size_t)k * 4, 256); }
extern "C" size_t sx_expand_topk_workspace(int32_t N, int32_t V, int32_t k, int32_t B) {
  (void)B;
  if (N < 1 || k < 1) return 0;
  return sx_expand_topk_min_workspace(N, k) + shares_bytes_up_to(N, V, k);
}

namespace {

// dynamic LDS of the select kernel: the set, or by histograms winners and room to place them (B = 8192); more than a launch
// gets by default: allowed once per device
constexpr size_t kSelectLds = 131072;
static_assert(kSelectLds >= (kPlaceCap + kSelBins) * 8, "the set and the list of a workgroup");
int configure_select_once() {
  static bool configured[64] = {};
  int dev = 0;
  SX_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return SX_ERR_HIP;
  if (configured[dev]) return SX_OK;
  const void* forms[] = {reinterpret_cast<const void*>(&select_kernel<0>), reinterpret_cast<const void*>(&select_kernel<4>)};
  for (const void* f : forms) SX_HIP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSelectLds));
  configured[dev] = true;
  return SX_OK;
}

// both kernels of the expansion step on `st`; score / lp / idx hold N*k entries each (every one of them is
// written by the first kernel before the second reads it: nothing has to be cleared)
// Workgroups of the selection of Bsel out of n > kSmallSelect candidates: some 20 to 60 entries of the set for each; one
// alone, by histograms, where the set would be too large.  The set is not known here, but a workgroup's share of all flat
// indices is: n / blocks and, counted out up to the largest n, 8 more at most -- 2060 of the kSelBins that its list holds.
int select_blocks(int n, int Bsel) {
  if (n > kPlaceCap && (Bsel > kPlaceCap * 3 / 4 || n > kSelBlocks * kSelBins / 2)) return 1;
  return n <= 2048 ? 64 : kSelBlocks;
}

int expand_topk_run(const float* logits, const float* cum_logp, int N, int V, int k, int B, int* out_row,
                    int* out_token, float* out_cum_logp, int* n_out, float* score, float* lp, int* idx, void* scratch,
                    hipStream_t st) {
  SX_TRY(configure_select_once());
  sx_prof_begin(SX_K_ROW_TOPK, st);
  const int rc = row_topk_dispatch(logits, cum_logp, N, V, k, lp, idx, score, scratch, st);
  sx_prof_end(st);
  if (rc != SX_OK) return rc;
  const int n = N * k;
  sx_prof_begin(SX_K_SELECT, st);
  if (n <= kSmallSelect) {
    small_select_kernel<<<1, kSelThreads, 0, st>>>(score, idx, n, k, B, out_row, out_token, out_cum_logp, n_out);
  } else {
    const int blocks = select_blocks(n, B < n ? B : n);
    const bool count = blocks > 1;
    const auto form = n <= 4 * 4 * kSelThreads ? select_kernel<4> : select_kernel<0>;
    form<<<blocks, kSelThreads, kSelectLds, st>>>(score, idx, n, k, B, count, out_row, out_token, out_cum_logp, n_out);
  }
  sx_prof_end(st);
  SX_LAUNCH_CHECK();
  return SX_OK;
}

}  // namespace

extern "C" int sx_expand_topk(const float* logits, const float* cum_logp, int32_t N, int32_t V, int32_t k, int32_t B,
                              int32_t* out_row, int32_t* out_token, float* out_cum_logp, int32_t* n_out,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (!logits || !cum_logp || !out_row || !out_token || !out_cum_logp || !n_out) return SX_ERR_NULL;
  if (!row_shape_ok(N, V, k) || B < 1 || B > 8192) return SX_ERR_SHAPE;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) ||
      workspace_bytes < sx_expand_topk_min_workspace(N, k))
    return SX_ERR_WORKSPACE;
  const int parts = row_parts(N, V, k, V % 4 == 0);
  const bool shares = parts > 1 && workspace_bytes - sx_expand_topk_min_workspace(N, k) >= shares_bytes((size_t)N * parts, k);
  const size_t nk = sx_align_up((size_t)N * (size_t)k * 4, 256);
  char* ws = static_cast<char*>(workspace);
  return expand_topk_run(logits, cum_logp, N, V, k, B, out_row, out_token, out_cum_logp, n_out,
                         reinterpret_cast<float*>(ws + SX_WS_HEADER), reinterpret_cast<float*>(ws + SX_WS_HEADER + nk),
                         reinterpret_cast<int*>(ws + SX_WS_HEADER + 2 * nk), shares ? ws + SX_WS_HEADER + 3 * nk : nullptr,
                         (hipStream_t)stream);
}

// ---- the same step for callers that cannot allocate ----------------------------------------------------
// The three candidate arrays (score, log-probability, token id; N*k entries each) live in a file-scope
// device array instead of a caller's workspace.  Every GPU holds its own copy of the array at its own
// address; the name below is only a host-side handle for hipGetSymbolAddress, never a kernel argument.
namespace {
constexpr int kStaticMaxCand = SX_EXPAND_STATIC_MAX_CANDIDATES;
static __device__ __align__(256) unsigned char scratch[3 * (size_t)kStaticMaxCand * 4];
void* g_scratch_ptr[64] = {};  // per device: address of that device's copy of `scratch`
}  // namespace

extern "C" int sx_expand_topk_static(const float* logits, const float* cum_logp, int32_t N, int32_t V, int32_t k,
                                     int32_t B, int32_t* out_row, int32_t* out_token, float* out_cum_logp,
                                     int32_t* n_out, void* stream) {
  if (!logits || !cum_logp || !out_row || !out_token || !out_cum_logp || !n_out) return SX_ERR_NULL;
  if (!row_shape_ok(N, V, k) || B < 1 || B > 8192) return SX_ERR_SHAPE;
  if ((long long)N * k > kStaticMaxCand) return SX_ERR_SHAPE;  // beyond the fixed scratch: use sx_expand_topk
  int dev = 0;
  SX_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return SX_ERR_HIP;
  if (!g_scratch_ptr[dev]) {  // first call on this device (with it current): look its copy of the array up
    void* p = nullptr;
    SX_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return SX_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  char* base = static_cast<char*>(g_scratch_ptr[dev]);
  const size_t nk = (size_t)kStaticMaxCand * 4;
  return expand_topk_run(logits, cum_logp, N, V, k, B, out_row, out_token, out_cum_logp, n_out,
                         reinterpret_cast<float*>(base), reinterpret_cast<float*>(base + nk),
                         reinterpret_cast<int*>(base + 2 * nk), nullptr, (hipStream_t)stream);
}
