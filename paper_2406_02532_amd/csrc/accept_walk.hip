// Acceptance walk (Alg. 1, main loop): sequential sampling from the target model, served from the
// tree of precomputed distributions for as long as the sampled tokens stay on a tree path.
//
// A step, data-parallel over the V logits of its node, is one workgroup's; the steps of a walk are taken by many
// workgroups at once where that pays (kNodes below), otherwise by one, one after the other.
// What bounds it: the chain of a step -- a row (128 KB at V = 32000) through one compute unit, barriers, the search for
// the child -- times the number of steps.  So a step makes two passes over the row and works on little after that:
//   1. the row maximum M;
//   2. with e = exp((x - M)/t): elements below (1 - top_p)/2V are less than half of what the nucleus may leave out, even
//      all of them together (the sum Z is at least 1); they only count towards Z.  The others are listed, with peaked
//      rows a few out of V;
//   3. at most 64 of them are finished by one wave in registers: the nucleus threshold, the largest bit pattern K with
//      sum{e >= K} >= top_p * Z, ties, nucleus mass, and the draw, the largest id Y with  sum{nucleus, id < Y} <= u * mass
//      (inverse CDF in id order).  Longer lists are cut by histograms over the bits of e.  Where the list overflows (flat
//      rows, top_p = 1) e of every element is computed once and kept -- over the row in LDS, or in the scratch row -- for
//      the same histograms over the row, and the draw takes a wave's 256 consecutive ids per sum.
// All sums but that of the small elements are integers: e in units of 2^-44 (at most 2^17 elements of at most 1, so 61
// bits; what an element loses to truncation is below 2^-44, 7e-9 of Z in all, an order below what fp32 partial sums
// lose).  Integer sums do not depend on the order in which LDS atomics arrive, so a given input always gives the same path.
// The form before this one searched threshold and draw bit by bit, 48 block-wide sums per step of about 1 us each (at
// V > 32768 each a pass over 512 KB in L2).  Per step, that form -> this one: peaked rows of 32000 60 -> 6.3 us (2.4 the
// row, 1.2 the candidates, 0.9 the child); rows of 32000 independent N(0, 1) logits at top_p = 0.9 60 -> 42, at top_p = 1
// 60 -> 24 (with e computed again in each of seven sweeps and every element through LDS atomics: 70 and 79); of 128256:
// peaked 805 -> 14, N(0, 1) 813 -> 127 and 784 -> 80.
//
// With draft probabilities (SI = true) the same kernel runs the comparison system of Sect. 4.1 instead:
// a drafted child with token x is accepted with probability P_target(x) / P_draft(x), capped at one.  The
// warped target distribution p of the current node is then kept normalised -- the nucleus in order of id, in the
// registers of one wave (at most 64 elements), as a list in LDS, or as a whole scratch row where it is larger; the
// children are tried in index order, child j of the position accepted when r_j q[x] < p[x]; a rejection replaces p by
// the renormalised positive part of p - q; after the last rejection the token is drawn from what p has become and the
// walk ends.
#include "kernels.h"

namespace {

typedef unsigned long long u64;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

constexpr int kBins = 1024;      // histogram bins: bits 20.. of the pattern of e <= 1, then bits 10..19 and 0..9; ids by blocks of 128
constexpr int kListCap = 1024;   // elements kept in LDS
constexpr int kStageNodes = 4096;  // the parents of trees up to this size are read once, into LDS

// The walk by many workgroups.  What a step draws depends on its node alone (the uniforms are keyed by position, that is
// by depth), so the steps need not wait for each other: one launch, in which workgroup i takes the step at node i, i < kNodes,
// at once, and records token and child.  The first one (the walker) goes on from node 0 along the records; where they end it
// takes the step itself, and the others, who have followed them to the same node, the steps at the nodes below, in index
// order; and so on.  Nobody waits but for a bounded time: the walker can take every step itself, and the others leave when the
// walk has ended or does not come on.  Draft trees come in the order of a best-first search, so the path is mostly among the
// first nodes, and the subtree below a node late in the order is small.  More than 64 workgroups make the rows wait for each
// other in memory: 2048 nodes, V = 128256 50.5 us with 64, 61.8 with 256.
// us, means over walks of 3 to 19 steps: by one workgroup | in two launches, the second at the nodes below the first record
// missing after the first | in one.  V = 32000: 64 nodes 54 | 14.0 | 13.3, 2048 nodes 95 | 30.7 | 24.6; V = 128256: 384 nodes
// 188 | 34.6 | 35.7, by ratio 232 | 45.8 | 45.5, 2048 nodes by ratio 295 | 71.6 | 50.8.  Flat rows, where the walk ends at its
// first node: V = 32000 43.4 | 46.8 | 46.1, t = 1, top_p = 1 25.3 | 28.5 | 26.6; V = 128256 133 | 144 | 134.6.  (What is left
// of that is code: the walker without the others takes as long.)  Rows not quite as flat, which the others take: N(0, 1.8)
// logits, t = 0.6 35 or 44, by seed | 49 | 47.5 or 52.
constexpr int kNodes = 64;
constexpr int kSmallVocab = 4096;  // up to here four waves walk alone: a step takes them 1 us
constexpr int kSpecDepth = 32;   // nodes further below node 0, or the walker's, are not taken ahead of the walk
// Words of the workspace.  [0]: the board, where the walker posts its own steps; [i]: the record of node i; [kNodes + i - 1]: of
// the node that workgroup i has taken since.  Fields: state, token (board: depth of the child), child or none + 1, node, tag.
// The tag makes words of this launch known from what was in the workspace before: the walker begins by reading them all and
// posts a tag that none of them has.  Who publishes uses the tag on the board; a tag from before the walker's post is on no
// word that the walker would believe, since the one it posts differs from it.
constexpr unsigned kDone = 0, kDoneError = 1, kPending = 2, kDeclined = 3;  // records
constexpr unsigned kBegun = 0, kWalking = 1, kEnded = 2;                    // the board
constexpr int kWords = 2 * kNodes;
constexpr unsigned kTokenMax = 0x3FFFF;
__device__ __forceinline__ unsigned long long pack_word(unsigned tag, int node, int child, unsigned token, unsigned state) {
  return (unsigned long long)tag << 48 | (unsigned long long)node << 33 | (unsigned long long)(child + 1) << 20 | token << 2 | state;
}
// the same value in every lane, told to the compiler: what depends on it stays in scalar registers and branches
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned long long uniform(unsigned long long v) {
  return (unsigned long long)(unsigned)uniform((int)(v >> 32)) << 32 | (unsigned)uniform((int)v);
}
struct Word {
  unsigned tag, state, token;
  int node, child;
  __device__ __forceinline__ explicit Word(unsigned long long w)
      : tag((unsigned)(w >> 48)), state((unsigned)w & 3u), token((unsigned)(w >> 2) & kTokenMax), node((int)(w >> 33) & 0xFFF),
        child((int)((unsigned)(w >> 20) & 0x1FFFu) - 1) {}
};
// A row of more candidates than the list holds and Z above this is so flat that the walk hardly goes on behind it.  Such
// rows, the slow ones, are not taken ahead.
constexpr float kFlat = 8.0f;

__device__ __forceinline__ u64 mix24(u64 seed, long long position) {  // the uniform of a position, in units of 2^-24
  u64 z = seed + (u64)(position + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = z ^ (z >> 31);
  return z >> 40;
}
// the uniform of the trial-th decision at one position (the ratio test needs several per position)
__device__ __forceinline__ u64 trial24(u64 seed, long long position, int trial) {
  return mix24(seed + (u64)(trial + 1) * 0xD6E8FEB86659FD93ull, position);
}
// floor(mass * u), u in units of 2^-24
__device__ __forceinline__ u64 scaled(u64 mass, u64 u24) {
  return (__umul64hi(mass, u24) << 40) | ((mass * u24) >> 24);
}
// a float in [0, 1], given by its bits, in units of 2^-44 (rounded down; anything else, a NaN included, counts nothing)
__device__ __forceinline__ u64 fix44(unsigned bits) {
  if (bits > 0x3F800000u) return 0;
  const int s = (int)(bits >> 23) - 106;
  const unsigned m = (bits & 0x7FFFFFu) | 0x800000u;
  return s >= 0 ? (u64)m << s : (u64)(s > -24 ? m >> -s : 0u);
}
__device__ __forceinline__ u64 wave_sum_u64(u64 v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ unsigned lane_u32(unsigned v, int j) { return __builtin_amdgcn_readlane(v, j); }
__device__ __forceinline__ u64 lane_u64(u64 v, int j) {
  return ((u64)lane_u32((unsigned)(v >> 32), j) << 32) | lane_u32((unsigned)v, j);
}

// max / min over the wave inside the vector unit (row shifts, then two row broadcasts; lane 63 ends up with the result):
// six instructions, where exchanges through LDS cost a round trip each
#define SX_WAVE_REDUCE(NAME, OP, NEUTRAL)                                                                    \
  __device__ __forceinline__ unsigned NAME(unsigned v) {                                                    \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x111, 0xf, 0xf, false));          \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x112, 0xf, 0xf, false));          \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x114, 0xf, 0xf, false));          \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x118, 0xf, 0xf, false));          \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x142, 0xa, 0xf, false));          \
    v = OP(v, (unsigned)__builtin_amdgcn_update_dpp((int)NEUTRAL, (int)v, 0x143, 0xc, 0xf, false));          \
    return lane_u32(v, 63);                                                                                  \
  }
SX_WAVE_REDUCE(wave_max_u32, max, 0u)
SX_WAVE_REDUCE(wave_min_u32, min, 0xFFFFFFFFu)
#undef SX_WAVE_REDUCE
__device__ __forceinline__ float wave_max_f32(float v) {
#define SX_STEP(CTRL, ROWS) \
  v = fmaxf(v, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp((int)0xFF800000, (int)__float_as_uint(v), CTRL, ROWS, 0xf, false)));
  SX_STEP(0x111, 0xf)
  SX_STEP(0x112, 0xf)
  SX_STEP(0x114, 0xf)
  SX_STEP(0x118, 0xf)
  SX_STEP(0x142, 0xa)
  SX_STEP(0x143, 0xc)
#undef SX_STEP
  return __uint_as_float(lane_u32(__float_as_uint(v), 63));
}
// sum over the lanes up to and with this one, the same way
__device__ __forceinline__ u64 wave_scan_u64(u64 v) {
#define SX_STEP(CTRL, ROWS)                                                                                              \
  v += ((u64)(unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xf, false) << 32) |                   \
       (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
  SX_STEP(0x111, 0xf)
  SX_STEP(0x112, 0xf)
  SX_STEP(0x114, 0xf)
  SX_STEP(0x118, 0xf)
  SX_STEP(0x142, 0xa)
  SX_STEP(0x143, 0xc)
#undef SX_STEP
  return v;
}

template <int N>
struct Const {
  static constexpr int value = N;
};

// INLDS: the row fits the LDS (V <= 32768) and is copied there by loads that write LDS; otherwise every pass reads it
// from memory, after the first one from L2.  (Held in registers the row cost more than it saved: 32 unrolled copies of
// every pass's body outgrew the instruction cache, and the rest of the kernel spilled.)  SI: acceptance by the ratio of
// target and draft probability.
// MANY: the walk by many workgroups.
// AHEAD: the workgroup is one of the others, not the walker.
template <int NT, bool SI>
struct Shared {
  u64 hist[kBins];
  u64 list[kListCap];  // id << 32 | bits of e
  u64 wsum[NT / 64], low, above;
  float plist[SI ? kListCap : 1], redf[16], px;
  int redi[16], n, nl, bin, token, child, err, pick, hops;
  unsigned tag;
  short par[kStageNodes];
};
template <int NT, bool INLDS, bool SI, bool MANY, bool AHEAD>
__device__ __forceinline__ void walk_steps(const float* __restrict__ logits, const float* __restrict__ draft_probs,
                                           const int* __restrict__ tokens, const int* __restrict__ parent, int T, int V,
                                           float temperature, float top_p, u64 seed, int pos0, int* __restrict__ path_out,
                                           int* __restrict__ tokens_out, int* __restrict__ n_out, float* __restrict__ scratch,
                                           u64* __restrict__ rec, int* __restrict__ status, Shared<NT, SI>& sh,
                                           float* const row) {
  constexpr int NW = NT / 64;
  constexpr int BPT = kBins / NT;  // bins per lane in a scan
  constexpr bool ahead = AHEAD;
  u64(&hist)[kBins] = sh.hist;
  u64(&list)[kListCap] = sh.list;
  auto& plist = sh.plist;
  auto& redf = sh.redf;
  auto& redi = sh.redi;
  auto& s_par = sh.par;
  auto& s_wsum = sh.wsum;
  u64 &s_low = sh.low, &s_above = sh.above;
  int &s_n = sh.n, &s_nl = sh.nl, &s_bin = sh.bin, &s_token = sh.token, &s_child = sh.child, &s_err = sh.err, &s_pick = sh.pick,
      &s_hops = sh.hops;
  unsigned& s_tag = sh.tag;
  float& s_px = sh.px;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float NEG_INF = -__builtin_huge_valf();

  const int who = AHEAD ? (int)(blockIdx.x - (blockIdx.x >> 3)) : 0;
  const int words = min(T, kWords);
  // the scratch row: of the walker at `scratch`, of the others behind the words (all pieces on 256 bytes)
  float* const ebuf =
      ahead ? reinterpret_cast<float*>(rec) + ((words * 2 + 63) & ~63) + (size_t)(who - 1) * (size_t)((V + 63) & ~63) : scratch;
  const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
  auto copy_row = [&](const float* x) {  // copies past the end of the row write zeros
    const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, V * 4, 0x00020000);
    if (vec) {
      for (int b0 = 0; b0 < V; b0 += 4 * NT)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(res, (lds_void_ptr)(row + b0 + wave * 256), 16, (b0 + tid * 4) * 4, 0, 0, 0);
    } else {
      for (int b0 = 0; b0 < V; b0 += 4 * NT)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(res, (lds_void_ptr)(row + b0 + wave * 256 + c * 64), 4,
                                                   (b0 + wave * 256 + c * 64 + lane) * 4, 0, 0, 0);
    }
  };
  auto word = [&](int i) { return __hip_atomic_load(rec + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto post = [&](int i, u64 w) { __hip_atomic_store(rec + i, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  int cur = who, depth = 0, n = 0;
  bool copied = false;  // the row of `cur` is on its way already
  if (MANY && INLDS) {
    copy_row(logits + (size_t)cur * (size_t)V);
    copied = true;
  }
  if (tid == 0) {
    if (!ahead) status[0] = (parent[0] != -1) ? SX_ERR_TREE : SX_OK;  // node 0 must be the root
    s_err = 0;
  }
  const bool staged = MANY || T <= kStageNodes;
  if (staged)
    for (int j = tid; j < T; j += NT) s_par[j] = (short)max(min(parent[j], T), -1);  // (a parent past the end is nobody's)
  auto par_of = [&](int j) { return staged ? (int)s_par[j] : parent[j]; };

  // sum of hist over the bins before this lane's first (ascending order of r; bin = r or kBins - 1 - r), and over all
  auto scan = [&](bool desc, u64& total) -> u64 {
    u64 mine = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int r = tid * BPT + i;
      mine += hist[desc ? kBins - 1 - r : r];
    }
    u64 incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const u64 t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) s_wsum[wave] = incl;
    __syncthreads();
    u64 before = 0, all = 0;
#pragma unroll 4
    for (int w = 0; w < NW; ++w) {
      if (w < wave) before += s_wsum[w];
      all += s_wsum[w];
    }
    total = all;
    return before + incl - mine;
  };
  // the first r whose running sum (from `start`) reaches `need`: its bin to s_bin, the sum before it to s_above
  auto find = [&](bool desc, u64 start, u64 need) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int r = tid * BPT + i, b = desc ? kBins - 1 - r : r;
      const u64 h = hist[b];
      if (start < need && start + h >= need) {
        s_bin = b;
        s_above = start;
      }
      start += h;
    }
    __syncthreads();
  };
  auto clear_hist = [&]() {
#pragma unroll
    for (int i = 0; i < BPT; ++i) hist[i * NT + tid] = 0;
    if (tid == 0) {
      s_bin = 0;
      s_above = 0;
    }
    __syncthreads();
  };
  // id of the first element, in id order, at which the running sum of weight(bits, id) over `each` exceeds `target`
  auto first_beyond = [&](auto each, auto weight, u64 target) -> int {
    __syncthreads();
    clear_hist();
    each([&](unsigned b, int id) {
      const u64 f = weight(b, id);
      if (f) atomicAdd(&hist[(unsigned)id >> 7], f);
    });
    __syncthreads();
    u64 total;
    u64 start = scan(false, total);
    find(false, start, target + 1);
    const int block = s_bin;
    const u64 base = s_above;
    __syncthreads();
    clear_hist();
    each([&](unsigned b, int id) {
      if ((id >> 7) == block) {
        const u64 f = weight(b, id);
        if (f) atomicAdd(&hist[id & 127], f);
      }
    });
    __syncthreads();
    start = base + scan(false, total);
    find(false, start, target + 1);
    return min(block * 128 + s_bin, V - 1);
  };

  // ---- many workgroups ------------------------------------------------------------------------------------------------
  // One wave, all words in two registers of it: along the records from node `at`, its depth beside it, to the first node that
  // has none (-1: the walk ends); true if the step there is in progress.  found(node, record) for every record passed.
  auto chase = [&](u64 w0, u64 w1, unsigned tag, int& at, int& dep, auto found) -> bool {
    while (at >= 0) {
      u64 w;
      if (at < kNodes) {
        w = lane_u64(w0, at);
      } else {
        const u64 who_has = __builtin_amdgcn_ballot_w64(kNodes + lane < words && Word(w1).tag == tag && Word(w1).node == at);
        if (who_has == 0) return false;
        w = lane_u64(w1, __builtin_ctzll(who_has));
      }
      const Word r(w);
      if (r.tag != tag || r.node != at) return true;  // (of the first kNodes: not there yet)
      if (r.state > kDoneError) return r.state == kPending;
      found(at, r);
      ++dep;
      at = r.child > at ? r.child : -1;
    }
    return false;
  };
  // One of the others: its step's result, and the next node if it finds where the walker is; false: nothing more to do.
  // They look for that (some 1.3 us a time) about as long as a peaked row's step takes: flat rows take several times as long,
  // a walk that has come to one is nearly over, and they have left before it ends.
  const int polls = who <= T - kNodes ? 12 + V / 4096 : 0;
  int slot = who, seen = 0;
  unsigned slot_tag = 0;  // of the words that led to the step's node; in the first step what is on the board near its end
  auto publish_and_next = [&](int child, int tok, unsigned state) -> bool {
    __syncthreads();
    if (wave == 0) {
      if ((unsigned)tok > kTokenMax) state = kDeclined;  // (a row of NaN: left to the walker)
      if (state == kDone && s_err) state = kDoneError;
      auto record = [&](unsigned with) {
        if (lane == 0) post(slot, pack_word(with, cur, child, (unsigned)tok & kTokenMax, state));
      };
      record(slot_tag);
      int at = -1, dep = 0;
      unsigned tag = slot_tag;
      for (int p = 0; p <= polls; ++p) {
        const u64 w0 = word(min(lane, words - 1)), w1 = word(min(kNodes + lane, words - 1));
        const Word b(lane_u64(w0, 0));
        if (p == 0 && slot == who && b.tag != tag) record(b.tag);
        at = -1;
        if (b.state == kEnded || p == polls) break;
        if (b.state == kWalking) {
          at = b.child < T ? b.child : -1;
          dep = (int)b.token;
          tag = b.tag;
          const bool wait = chase(w0, w1, tag, at, dep, [](int, const Word&) {});
          if (at < 0 || (!wait && at > seen)) break;
        }
        __builtin_amdgcn_s_sleep(4);
      }
      if (lane == 0) {
        s_err = 0;
        s_pick = at;
        s_hops = dep;
        s_tag = tag;
      }
    }
    __syncthreads();
    seen = uniform(s_pick);
    if (seen < 0) return false;
    const int seen_depth = uniform(s_hops);
    slot_tag = (unsigned)uniform((int)s_tag);
    // the who-th of the nodes below `seen`, in index order, the first kNodes left out
    constexpr int E = kStageNodes / NT;
    const int per = (T + NT - 1) / NT;
    int p[E], hops[E], hits = 0;
    bool on[E], hit[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      p[i] = tid * per + i;
      hops[i] = 0;
      hit[i] = false;
      on[i] = i < per && p[i] > seen && p[i] >= kNodes && p[i] < T;
    }
    for (int h = 0; h < kSpecDepth; ++h) {
      bool any = false;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        if (!on[i]) continue;
        const int q = s_par[p[i]];
        ++hops[i];
        hit[i] = q == seen;
        on[i] = q > seen && q < p[i];
        p[i] = q;
        any |= on[i];
      }
      if (__builtin_amdgcn_ballot_w64(any) == 0) break;
    }
#pragma unroll
    for (int i = 0; i < E; ++i) hits += hit[i];
    int incl = hits;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    if (lane == 63) redi[wave] = incl;
    __syncthreads();
    if (tid == 0) s_pick = -1;
    __syncthreads();
    int rank = incl - hits;
    for (int w = 0; w < wave; ++w) rank += redi[w];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      if (hit[i] && rank == who - 1) {
        s_pick = tid * per + i;
        s_hops = hops[i];
      }
      rank += hit[i];
    }
    __syncthreads();
    if (uniform(s_pick) < 0) return false;
    cur = uniform(s_pick);
    depth = seen_depth + uniform(s_hops);
    slot = kNodes + who - 1;
    if (tid == 0) post(slot, pack_word(slot_tag, cur, -1, 0, kPending));
    return true;
  };
  auto walk_ended = [&]() -> bool {
    if (tid == 0) s_pick = Word(word(0)).state == kEnded ? 1 : 0;
    __syncthreads();
    const bool e = uniform(s_pick) != 0;
    __syncthreads();
    return e;
  };
  // The same at the end of each sweep of a slow step: one lane asks, and behind the barrier that is there anyway everybody
  // knows.  (V = 32000, N(0, 1.8) logits at t = 0.6: the walk ends at node 0 after 37 or 46 us, half of the others are at steps
  // of up to 50.  The call takes 47.5 or 52, and 52 in either case when they only ask once.  Asked in every round of a sweep,
  // with the rest of it skipped, the others get slower: 44.5 or 53.5.)
  auto ask = [&]() {
    if (ahead && tid == 0) s_pick = Word(word(0)).state == kEnded ? 1 : 0;
  };
  auto told = [&]() -> bool { return ahead && uniform(s_pick) != 0; };
  // the result of a step: child or -1, token, and for the others the state of the record
  int r_child = -1, r_token = 0;
  unsigned r_state = kDone;
  bool declined = false;  // there is none: the node is not taken
  u64 begun = __builtin_amdgcn_s_memtime();
  if (ahead) {
    __syncthreads();
    int j = cur, hops = 0;  // nodes deeper than kSpecDepth, and those that do not hang from node 0, are left alone
    while (j > 0 && hops < kSpecDepth) {
      const int p = uniform(s_par[j]);
      if (p < 0 || p >= j) break;
      j = p;
      ++hops;
    }
    depth = hops;
    if (j != 0) {
      __builtin_amdgcn_s_waitcnt(0x0070);  // the row's copy: this workgroup may end
      copied = false;
      declined = true;
      r_state = kDeclined;
    }
  }

  __syncthreads();
  bool first = true;
  // The step at `cur`.  False (the others only): the walk has ended meanwhile.
  auto take_step = [&]() -> bool {
    const float* x = logits + (size_t)cur * (size_t)V;
    // f(four consecutive elements, id of the first) over the row, in the same number of rounds for every lane; past the
    // end x reads as -inf.  A lane always takes the same quads, so in LDS it reads what its own wave has copied.
    auto edge = [&](float v, int id) { return id < V ? v : NEG_INF; };
    auto sweep_by = [&](auto quads, auto f) {
      if constexpr (INLDS) {
        int id = tid * 4;
        for (; id - tid * 4 + 4 * NT <= V; id += 4 * NT) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(row + id);
          f(v[0], v[1], v[2], v[3], id);
        }
        if (id - tid * 4 < V) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(row + id);
          f(edge(v[0], id), edge(v[1], id + 1), edge(v[2], id + 2), edge(v[3], id + 3), id);
        }
      } else {
        constexpr int U = decltype(quads)::value;  // quads in flight per lane
        if (vec) {  // quads lie inside the row or past its end
          for (int b0 = 0; b0 < V; b0 += U * 4 * NT) {
            f32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
              v[u] = *reinterpret_cast<const f32x4*>(x + min(b0 + (u * NT + tid) * 4, V - 4));
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int id = b0 + (u * NT + tid) * 4;
              const bool in = id < V;
              f(in ? v[u][0] : NEG_INF, in ? v[u][1] : NEG_INF, in ? v[u][2] : NEG_INF, in ? v[u][3] : NEG_INF, id);
            }
          }
          return;
        }
        for (int b0 = 0; b0 < V; b0 += U * 4 * NT) {
          float v[U][4];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[u][c] = x[(unsigned)min(b0 + (u * NT + tid) * 4 + c, V - 1)];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int id = b0 + (u * NT + tid) * 4;
            f(edge(v[u][0], id), edge(v[u][1], id + 1), edge(v[u][2], id + 2), edge(v[u][3], id + 3), id);
          }
        }
      }
    };
    auto sweep = [&](auto f) { sweep_by(Const<4>{}, f); };
    if constexpr (INLDS) {
      if (!copied) copy_row(x);
      copied = false;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0070);  // all of this wave's copies are in
      asm volatile("" ::: "memory");
    }
    const long long pos = (long long)pos0 + depth + 1;
    // the first step's last wave of the walker: what the words were, asked for behind the row
    const bool tags = MANY && !ahead && first && wave == NW - 1;
    u64 old0 = 0, old1 = 0;
    if (tags) {
      old0 = word(min(lane, words - 1));
      old1 = word(min(kNodes + lane, words - 1));
    }
    // ---- row maximum (and the greedy answer) ------------------------------------------------------
    float tm = NEG_INF;
    sweep_by(Const<8>{}, [&](float v0, float v1, float v2, float v3, int) { tm = fmaxf(tm, fmaxf(fmaxf(v0, v1), fmaxf(v2, v3))); });
#pragma unroll
    for (int i = 0; i < BPT; ++i) hist[i * NT + tid] = 0;
    if (tid == 0) {
      s_low = 0;
      s_n = 0;
      s_bin = 0;
      s_above = 0;
      s_token = 0;
      s_child = 0x7FFFFFFF;
    }
    tm = wave_max_f32(tm);
    if (lane == 0) redf[wave] = tm;
    if (tags) {  // a tag that no word has: 128 words, 65536 tags
      const unsigned t0 = Word(old0).tag, t1 = Word(old1).tag;
      unsigned tag = lane_u32(t0, 0);
      do tag = (tag + 1) & 0xFFFFu;
      while (__builtin_amdgcn_ballot_w64(t0 == tag || t1 == tag));
      if (lane == 0) {
        post(0, pack_word(tag, 0, -1, 0, kBegun));
        s_tag = tag;
      }
    }
    __syncthreads();
    float M = redf[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, redf[w]);
    int token;
    int nl = -1;          // SI: entries of the nucleus list; -1: the distribution is in ebuf
    if (temperature == 0.f) {
      int best = 0x7FFFFFFF;
      sweep([&](float v0, float v1, float v2, float v3, int id) {
        const float v[4] = {v0, v1, v2, v3};
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (v[c] == M && id + c < V) best = min(best, id + c);
      });
      token = block_min_i<NW>(best, redi);
      if constexpr (SI) {  // p = all mass on the argmax
        if (tid == 0) {
          list[0] = (u64)(unsigned)min(token, V - 1) << 32;
          plist[0] = 1.0f;
        }
        nl = 1;
        __syncthreads();
      }
    } else {
      // ---- the elements that can be in the nucleus, and the sum of the others ---------------------------------
      const float inv_t = 1.0f / temperature;
      auto e_bits = [&](float v) { return __float_as_uint(expf((v - M) * inv_t)); };
      // the x below which e is certainly under `e` (the slack covers the roundings of this line and of e_bits)
      auto x_below = [&](float e) {
        const float l = logf(e);
        return M + temperature * (l - 1e-4f * (1.0f - l)) - 1e-6f * fabsf(M);
      };
      // appends (id, payload) of the lanes that hit; entries past the end of the list are counted only, and a wave that has
      // found it full stops counting
      bool full = false;
      auto append = [&](bool hit, int id, unsigned payload) {
        const u64 who = __builtin_amdgcn_ballot_w64(hit);
        if (who == 0 || full) return;
        const int leader = __builtin_ctzll(who);
        int slot = 0;
        if (lane == leader) slot = atomicAdd(&s_n, __builtin_popcountll(who));
        slot = __builtin_amdgcn_readlane(slot, leader);
        full = slot >= kListCap;
        slot += __builtin_popcountll(who & ((1ull << lane) - 1ull));
        if (hit && slot < kListCap) list[slot] = ((u64)(unsigned)id << 32) | payload;
      };
      // e below 2^-46 counts nothing, as in fix44: with peaked rows that skips most exponentials
      const float x_zero = x_below(1.4210854715202004e-14f);
      const float x_cut = fmaxf(x_zero, x_below(0.4f * (1.0f - top_p) / (float)V));
      // e of the small ones: from v - M, which is exact or nearly so (with v c2 - M c2 the rounding of the product, a row's
      // offset over t times 2^-24, would be an error of every term)
      const float c2 = inv_t * 1.4426950408889634f;
      auto small_e = [&](float v) { return __builtin_amdgcn_exp2f((v - M) * c2); };
      float lowf = 0.f;
      sweep([&](float v0, float v1, float v2, float v3, int id) {
        const float m4 = fmaxf(fmaxf(v0, v1), fmaxf(v2, v3));
        if (__builtin_amdgcn_ballot_w64(m4 >= x_zero) == 0) return;
        const float v[4] = {v0, v1, v2, v3};
        if (__builtin_amdgcn_ballot_w64(m4 >= x_cut) == 0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) lowf += small_e(v[c]);  // exp2(-inf) = 0 past the end
          return;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const bool hit = v[c] >= x_cut;
          if (!hit) lowf += small_e(v[c]);
          append(hit && id + c < V, id + c, __float_as_uint(v[c]));
        }
      });
      // (at top_p = 1 the threshold is the sum of the candidates: the rest, below 2^-46 each, is not to raise it)
      const u64 low = top_p < 1.0f ? wave_scan_u64(fix44(__float_as_uint(lowf))) : 0;
      if (lane == 63 && low) atomicAdd(&s_low, low);
      __syncthreads();
      const u64 u24 = mix24(seed, pos);
      int nc = s_n;
      const bool overflow = nc > kListCap;
      if (ahead && (first || overflow) && tid == 0) {
        const Word b(word(0));
        if (first) slot_tag = b.tag;
        s_pick = b.state == kEnded ? 1 : 0;
      }
      if (ahead && overflow) {
        // Z from a quad per lane, those of the peak left out
        const float* at = (INLDS ? row : x) + (V >> 2) / NT * 4 * tid;
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float e = __uint_as_float(e_bits(at[c]));
          z += e < 0.0625f ? e : 0.f;
        }
        const bool flat = block_sum<NW>(z, redf) * (float)V > kFlat * (float)(4 * NT);
        if (told()) return false;  // the slow steps end with the walk
        if (flat) {
          r_child = -1;
          r_state = kDeclined;
          return true;
        }
      }
      u64 thr = 0;
      unsigned K = 0, Ytie = 0xFFFFFFFFu;  // the nucleus: e > K, or e == K and id < Ytie
      u64 mass = 0;
      token = 0;
      auto threshold = [&](u64 Z) -> u64 {
        const u64 t = (u64)ceil((double)top_p * (double)Z);
        return t > Z ? Z : (t < 1 ? 1 : t);
      };
      auto in_nucleus = [&](unsigned b, unsigned id) { return b > K || (b == K && id < Ytie); };
      auto weight_of = [&](unsigned b, int id) { return in_nucleus(b, (unsigned)id) ? fix44(b) : 0; };
      auto is_tie = [&](unsigned b, int) { return (u64)(b == K ? 1 : 0); };
      // the flat row's e, four at a time: what a lane wrote in one sweep it reads in the next
      float* const es = INLDS ? row : ebuf;
      auto row_bits = [&](float v0, float v1, float v2, float v3) -> u32x4 {
        const float v[4] = {v0, v1, v2, v3};
        u32x4 b = {0u, 0u, 0u, 0u};
        if (__builtin_amdgcn_ballot_w64(fmaxf(fmaxf(v0, v1), fmaxf(v2, v3)) >= x_cut) == 0) return b;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          b[c] = v[c] >= x_cut ? e_bits(v[c]) : 0u;
          if (b[c] > 0x3F800000u) b[c] = 0u;  // a NaN
        }
        return b;
      };
      auto keep_e = [&](int id, u32x4 b) {
        if (id < V) *reinterpret_cast<u32x4*>(es + id) = b;  // (either array ends on 16 bytes)
      };
      auto sweep_e = [&](auto f) {
        for (int id = tid * 4; id < V; id += 4 * NT) f(*reinterpret_cast<const u32x4*>(es + id), id);
      };
      // as first_beyond, over the row: a wave's 64 quads are 256 consecutive ids, whose sum needs no atomics.  (The others: -1,
      // the walk has ended meanwhile.)
      auto first_beyond_e = [&](auto weight, u64 target) -> int {
        __syncthreads();
        clear_hist();
        sweep_e([&](u32x4 b, int id) {
          const u64 f = (weight(b[0], id) + weight(b[1], id + 1)) + (weight(b[2], id + 2) + weight(b[3], id + 3));
          const u64 incl = wave_scan_u64(f);
          if (lane == 63 || id + 4 >= V) hist[id >> 8] = incl;  // (the last lane that has a quad)
        });
        ask();
        __syncthreads();
        if (told()) return -1;
        u64 sum;
        const u64 start = scan(false, sum);
        find(false, start, target + 1);
        if (wave == 0) {
          const int id = s_bin * 256 + lane * 4;
          u32x4 b = {0u, 0u, 0u, 0u};
          if (id < V) b = *reinterpret_cast<const u32x4*>(es + id);
          u64 f[4], all = 0;
#pragma unroll
          for (int c = 0; c < 4; ++c) all += f[c] = weight(b[c], id + c);
          u64 before = s_above + wave_scan_u64(all) - all;
          unsigned hit = 0x7FFFFFFFu;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            before += f[c];
            if (before > target) hit = min(hit, (unsigned)(id + c));
          }
          hit = wave_min_u32(hit);
          if (lane == 0) s_token = hit < (unsigned)V ? (int)hit : min(s_bin * 256, V - 1);
        }
        __syncthreads();
        return s_token;
      };
      // K from its top bits (`prefix`, the sum `above` that bin): the lower ones by two more histograms; then the nucleus mass
      // and how many of the elements equal to K are in it
      bool ties_left = false;  // not all of them
      u64 ties_taken = 0;
      auto refine = [&](auto each, unsigned prefix, u64 above) -> bool {  // false: the walk has ended meanwhile
        for (int shift = 10; shift >= 0; shift -= 10) {
          __syncthreads();
          clear_hist();
          each([&](unsigned b, int) {
            if (b <= 0x3F800000u && (b >> (shift + 10)) == prefix) {
              const u64 f = fix44(b);
              if (f) atomicAdd(&hist[(b >> shift) & (kBins - 1)], f);
            }
          });
          ask();
          __syncthreads();
          if (told()) return false;
          u64 t2;
          const u64 st = above + scan(true, t2);
          find(true, st, thr);
          prefix = (prefix << 10) | (unsigned)s_bin;
          above = s_above;
        }
        K = prefix;
        const u64 fk = fix44(K);
        const u64 tie_sum = hist[K & (kBins - 1)];  // the last histogram's bin holds the elements equal to K alone
        mass = above;
        if (fk > 0) {
          const u64 n_tie = tie_sum / fk;
          u64 m = thr > above ? (thr - above + fk - 1) / fk : 1;
          m = m < 1 ? 1 : (m > n_tie ? n_tie : m);
          mass = above + m * fk;
          ties_left = m < n_tie;
          ties_taken = m;
        }
        return true;
      };
      // at most 64 candidates in `list` (payload: bits of e), one per lane of one wave; `thr` known (have_thr) or made
      // from their sum and the small elements'
      auto few = [&](int cnt, bool have_thr) {
        const u64 entry = lane < cnt ? list[lane] : 0xFFFFFFFF00000000ull;
        const unsigned b = (unsigned)entry, id = (unsigned)(entry >> 32);
        const u64 f = fix44(b);
        u64 ge = 0;       // sum over elements at least as large
        u64 all = 0;
        int earlier = 0;  // equal ones with a lower id
        for (int j = 0; j < cnt; ++j) {
          const unsigned bj = lane_u32(b, j), idj = lane_u32(id, j);
          const u64 fj = lane_u64(f, j);
          all += fj;
          ge += bj >= b ? fj : 0;
          earlier += (bj == b && idj < id) ? 1 : 0;
        }
        const u64 need = have_thr ? thr : threshold(s_low + all);
        unsigned k = lane < cnt && ge >= need ? b : 0u;
        k = wave_max_u32(k);
        const u64 ties = __builtin_amdgcn_ballot_w64(lane < cnt && b == k);
        int m = 1;  // ties (equal probabilities) enter in id order until the mass reaches the threshold
        u64 sum = 0;
        if (ties) {
          const int tl0 = __builtin_ctzll(ties), n_tie = __builtin_popcountll(ties);
          const u64 fk = lane_u64(f, tl0), gt = lane_u64(ge, tl0) - (u64)n_tie * fk;
          while (m < n_tie && gt + (u64)m * fk < need) ++m;
          sum = gt + (u64)m * fk;
        }
        const bool member = lane < cnt && (b > k || (b == k && earlier < m));
        const u64 fm = member ? f : 0;
        u64 cum = 0;    // sum over members up to this one, in id order
        int place = 0;  // members with a lower id
        for (int j = 0; j < cnt; ++j) {
          const u64 fj = lane_u64(fm, j);
          const unsigned idj = lane_u32(id, j);
          cum += idj <= id ? fj : 0;
          place += (fj != 0 && idj < id) ? 1 : 0;
        }
        if constexpr (SI) {  // the nucleus in order of id, normalised (a member of weight 0 is one that p rounds to 0)
          const float inv_mass = (float)(17592186044416.0 / (double)sum);  // 2^44 / mass
          if (fm != 0) {
            list[place] = entry;
            plist[place] = __uint_as_float(b) * inv_mass;
          }
          const u64 kept = __builtin_amdgcn_ballot_w64(fm != 0);
          if (lane == 0) s_nl = __builtin_popcountll(kept);
        } else {
          const u64 target = scaled(sum, u24);
          unsigned t = member && cum > target ? id : 0x7FFFFFFFu;
          t = wave_min_u32(t);
          if (lane == 0) s_token = t < (unsigned)V ? (int)t : 0;
        }
      };
      bool done = false, in_list = true;  // finished by one wave; the nucleus is among the entries of the list
      if (nc <= 64) {
        if (wave == 0) {
          if (lane < nc) list[lane] = (list[lane] & 0xFFFFFFFF00000000ull) | e_bits(__uint_as_float((unsigned)list[lane]));
          few(nc, false);
        }
        done = true;
      } else if (overflow && top_p >= 1.0f) {
        // ---- a flat row of which every element is in the nucleus ---------------------------------------------
        u64 part = 0;
        sweep([&](float v0, float v1, float v2, float v3, int id) {
          const u32x4 b = row_bits(v0, v1, v2, v3);
          keep_e(id, b);
          part += (fix44(b[0]) + fix44(b[1])) + (fix44(b[2]) + fix44(b[3]));
        });
        part = wave_scan_u64(part);
        if (lane == 63) atomicAdd(&s_low, part);
        ask();
        __syncthreads();
        if (told()) return false;
        mass = s_low;
        Ytie = 0;
        in_list = false;
      } else {
        // ---- more: bin of the threshold by a histogram over the top bits of e (8 bins per octave) ---------------
        if (!overflow) {
          for (int i = tid; i < nc; i += NT) {
            const unsigned b = e_bits(__uint_as_float((unsigned)list[i]));
            const u64 f = fix44(b);
            if (f) atomicAdd(&hist[min(b >> 20, (unsigned)(kBins - 1))], f);
          }
        } else {
          sweep([&](float v0, float v1, float v2, float v3, int id) {
            const u32x4 b = row_bits(v0, v1, v2, v3);
            keep_e(id, b);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const u64 f = fix44(b[c]);
              if (f) atomicAdd(&hist[b[c] >> 20], f);
            }
          });
          ask();
        }
        __syncthreads();
        if (overflow && told()) return false;
        u64 total;
        const u64 start = scan(true, total);
        thr = threshold(total + s_low);
        find(true, start, thr);
        const unsigned floor_bits = (unsigned)s_bin << 20;
        u64 above = s_above;
        // ---- the elements of that bin and above as a list, if they fit ------------------------------------------
        full = false;
        if (!overflow) {  // in place: every lane takes its entries before anyone writes
          u64 mine[kListCap / NT];
#pragma unroll
          for (int i = 0; i < kListCap / NT; ++i) mine[i] = i * NT + tid < nc ? list[i * NT + tid] : 0;
          __syncthreads();
          if (tid == 0) s_n = 0;
          __syncthreads();
#pragma unroll
          for (int i = 0; i < kListCap / NT; ++i) {
            const unsigned b = e_bits(__uint_as_float((unsigned)mine[i]));
            append(i * NT + tid < nc && b >= floor_bits && b <= 0x3F800000u, (int)(mine[i] >> 32), b);
          }
        } else {
          __syncthreads();
          if (tid == 0) s_n = 0;
          __syncthreads();
          sweep_e([&](u32x4 b, int id) {
            if (__builtin_amdgcn_ballot_w64(max(max(b[0], b[1]), max(b[2], b[3])) >= floor_bits) == 0) return;
#pragma unroll
            for (int c = 0; c < 4; ++c) append(b[c] >= floor_bits && id + c < V, id + c, b[c]);
          });
          ask();
        }
        __syncthreads();
        if (overflow && told()) return false;
        nc = s_n;
        in_list = nc <= kListCap;
        if (nc <= 64) {
          if (wave == 0) few(nc, true);
          done = true;
        } else {  // still many: the lower bits of the threshold by two more histograms, the draw by blocks of ids
          if (in_list) {
            auto each = [&](auto f) {
              for (int i = tid; i < nc; i += NT) f((unsigned)list[i], (int)(list[i] >> 32));
            };
            if (!refine(each, floor_bits >> 20, above)) return false;
            if (ties_left) Ytie = (unsigned)first_beyond(each, is_tie, ties_taken);
            if constexpr (!SI) token = first_beyond(each, weight_of, scaled(mass, u24));
          } else {
            if (!refine([&](auto f) { sweep_e([&](u32x4 b, int id) {
#pragma unroll
                                        for (int c = 0; c < 4; ++c) f(b[c], id + c);
                                      }); },
                        floor_bits >> 20, above))
              return false;
            if (ties_left) {
              const int y = first_beyond_e(is_tie, ties_taken);
              if (ahead && y < 0) return false;
              Ytie = (unsigned)y;
            }
          }
        }
      }
      if (!in_list) {
        if constexpr (!SI) {
          token = first_beyond_e(weight_of, scaled(mass, u24));
          if (ahead && token < 0) return false;
        } else {  // the nucleus as a list, if it is short enough for one
          __syncthreads();
          if (tid == 0) s_n = 0;
          __syncthreads();
          full = false;
          sweep_e([&](u32x4 b, int id) {
#pragma unroll
            for (int c = 0; c < 4; ++c) append(in_nucleus(b[c], (unsigned)(id + c)), id + c, b[c]);
          });
          ask();
          __syncthreads();
          if (told()) return false;
          nc = s_n;
        }
      }
      if (done) {
        __syncthreads();
        if constexpr (SI) nl = s_nl;
        else token = s_token;
      }
      if (SI && !done) {  // p = the nucleus, normalised
        const float inv_mass = (float)(17592186044416.0 / (double)mass);  // 2^44 / mass
        __syncthreads();
        if (nc <= kListCap) {
          // in order of id: sums over the list then have one order, whatever order the atomics filled it in.  By buckets of 128
          // ids, a scan of their counts and the place inside the bucket (a sorting network over 1024 entries, 55 stages with
          // a barrier each, was half of such a step: 32 -> 19 us at V = 1000)
          constexpr int E = kListCap / NT;
          u64 mine[E];
          unsigned slot[E], place[E];
          bool in[E];
#pragma unroll
          for (int i = 0; i < E; ++i) {
            mine[i] = i * NT + tid < nc ? list[i * NT + tid] : 0;
            in[i] = i * NT + tid < nc && in_nucleus((unsigned)mine[i], (unsigned)(mine[i] >> 32));
          }
          __syncthreads();
          clear_hist();
#pragma unroll
          for (int i = 0; i < E; ++i) slot[i] = in[i] ? (unsigned)atomicAdd(&hist[mine[i] >> 39], 1ull) : 0u;
          __syncthreads();
          u64 members;
          u64 first = scan(false, members);
          nl = (int)members;
#pragma unroll
          for (int i = 0; i < BPT; ++i) {  // count -> first place << 32 | count
            const u64 h = hist[tid * BPT + i];
            hist[tid * BPT + i] = first << 32 | h;
            first += h;
          }
          __syncthreads();
#pragma unroll
          for (int i = 0; i < E; ++i)
            if (in[i]) list[(unsigned)(hist[mine[i] >> 39] >> 32) + slot[i]] = mine[i];
          __syncthreads();
#pragma unroll
          for (int i = 0; i < E; ++i) {
            const u64 h = in[i] ? hist[mine[i] >> 39] : 0;
            place[i] = (unsigned)(h >> 32);
            for (unsigned j = 0; j < (unsigned)h; ++j) place[i] += list[(unsigned)(h >> 32) + j] < mine[i] ? 1 : 0;
          }
          __syncthreads();
#pragma unroll
          for (int i = 0; i < E; ++i)
            if (in[i]) {
              list[place[i]] = mine[i];
              plist[place[i]] = __uint_as_float((unsigned)mine[i]) * inv_mass;
            }
        } else {
          for (int id = tid; id < V; id += NT) {
            const float e = es[id];
            ebuf[id] = in_nucleus(__float_as_uint(e), (unsigned)id) ? e * inv_mass : 0.f;
          }
        }
        __syncthreads();
      }
    }
    if constexpr (SI) {
      // ---- ratio test over the children of cur, in index order ------------------------------------------
      const float* q = draft_probs + (size_t)cur * (size_t)V;
      if (nl >= 0 && nl <= 64 && staged) {
        // one wave holds the distribution: p and q of an element per lane, in order of id.  (A token that p gives no mass is
        // rejected whatever q is.)
        if (wave == 0) {
          const unsigned id = lane < nl ? (unsigned)(list[lane] >> 32) : 0xFFFFFFFFu;
          float pv = lane < nl ? plist[lane] : 0.f;
          const float qv = lane < nl ? q[id] : 0.f;
          int trial = 0, found = -1;
          for (int j0 = cur + 1; j0 < T && found < 0; j0 += 64) {
            const int j = j0 + lane;
            const bool kid = j < T && s_par[min(j, T - 1)] == cur;
            u64 kids = __builtin_amdgcn_ballot_w64(kid);
            const int tj = kid ? tokens[j] : 0;
            while (kids) {
              const int l = __builtin_ctzll(kids);
              kids &= kids - 1;
              const int xt = __builtin_amdgcn_readlane(tj, l);
              const u64 here = __builtin_amdgcn_ballot_w64(lane < nl && (int)id == xt);
              if (xt < 0 || xt >= V) {  // not a token: nothing to accept, nothing the draft could have covered
                if (lane == 0) s_err = 1;
                ++trial;
                continue;
              }
              const float r = (float)trial24(seed, pos, trial) * 5.9604644775390625e-08f;  // 2^-24
              if (__builtin_amdgcn_ballot_w64((here >> lane & 1) && r * qv < pv)) {
                found = j0 + l;
                break;
              }
              ++trial;
              const float d = fmaxf(pv - qv, 0.f);
              const float Zr = wave_sum(d);
              if (Zr > 0.f) pv = d * (1.0f / Zr);
            }
          }
          int last = 0;
          if (found < 0) {  // every child rejected: draw from what p has become
            const u64 f = fix44(min(__float_as_uint(pv), 0x3F800000u));
            u64 incl = f;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
              const u64 t = __shfl_up(incl, o, 64);
              if (lane >= o) incl += t;
            }
            const u64 target = scaled(lane_u64(incl, 63), trial24(seed, pos, trial));
            const u64 beyond = __builtin_amdgcn_ballot_w64(lane < nl && incl > target);
            if (beyond) last = (int)lane_u32(id, __builtin_ctzll(beyond));
          }
          if (lane == 0) {
            s_child = found;
            s_token = last;
          }
        }
        __syncthreads();
        r_child = s_child;
        r_token = r_child >= 0 ? tokens[r_child] : s_token;
        return true;
      }
      int after = cur, trial = 0, accepted = -1;
      bool ended = false;
      while (true) {
        if (ahead && trial > 0 && (ended = walk_ended())) break;
        int c = 0x7FFFFFFF;
        // (trees whose parents stay in memory: four loads in flight; 6000 nodes, V = 4000 149 us a walk, 173 one by one)
#pragma unroll 4
        for (int j = after + 1 + tid; j < T; j += NT)
          if (par_of(j) == cur) c = min(c, j);
        c = block_min_i<NW>(c, redi);
        if (c == 0x7FFFFFFF) break;
        const int xt = tokens[c];
        after = c;
        if (xt < 0 || xt >= V) {  // not a token: nothing to accept, nothing the draft could have covered
          if (tid == 0) s_err = 1;
          ++trial;
          continue;
        }
        float px;
        if (nl >= 0) {
          if (tid == 0) s_px = 0.f;
          __syncthreads();
          for (int i = tid; i < nl; i += NT)
            if ((int)(list[i] >> 32) == xt) s_px = plist[i];
          __syncthreads();
          px = s_px;
        } else {
          px = ebuf[xt];
        }
        const float r = (float)trial24(seed, pos, trial) * 5.9604644775390625e-08f;  // 2^-24
        if (r * q[xt] < px) {
          accepted = c;
          break;
        }
        ++trial;
        float z = 0.f;
        if (nl >= 0) {
          for (int i = tid; i < nl; i += NT) z += fmaxf(plist[i] - q[list[i] >> 32], 0.f);
        } else {
          for (int id = tid; id < V; id += NT) z += fmaxf(ebuf[id] - q[id], 0.f);
        }
        const float Zr = block_sum<NW>(z, redf);  // its barriers also order the reads of p[x] above before the writes
        if (Zr > 0.f) {
          const float inv = 1.0f / Zr;
          if (nl >= 0) {
            for (int i = tid; i < nl; i += NT) plist[i] = fmaxf(plist[i] - q[list[i] >> 32], 0.f) * inv;
          } else {
            for (int id = tid; id < V; id += NT) ebuf[id] = fmaxf(ebuf[id] - q[id], 0.f) * inv;
          }
        }
        __syncthreads();
      }
      if (ended) return false;
      if (accepted >= 0) {
        r_child = accepted;
        r_token = tokens[accepted];
        return true;
      }
      // ---- every child rejected: draw from what p has become, then stop ----------------------------------
      // (p is at most 1 up to the rounding of its normalisation; a value above 1 counts as 1)
      auto weight = [&](unsigned b, int) { return fix44(min(b, 0x3F800000u)); };
      auto each = [&](auto f) {
        if (nl >= 0) {
          for (int i = tid; i < nl; i += NT) f(__float_as_uint(plist[i]), (int)(list[i] >> 32));
        } else {
          for (int id = tid; id < V; id += NT) f(__float_as_uint(ebuf[id]), id);
        }
      };
      u64 part = 0;
      each([&](unsigned b, int id) { part += weight(b, id); });
      part = wave_sum_u64(part);
      __syncthreads();
      if (tid == 0) s_low = 0;
      __syncthreads();
      if (lane == 0 && part) atomicAdd(&s_low, part);
      __syncthreads();
      token = first_beyond(each, weight, scaled(s_low, trial24(seed, pos, trial)));
      r_child = -1;
      r_token = token;
      return true;
    }
    // ---- cache lookup: lowest-index child of cur carrying the sampled token -------------------------
    int child = 0x7FFFFFFF;
    for (int j = cur + 1 + tid; j < T; j += NT)
      if (par_of(j) == cur && tokens[j] == token) child = min(child, j);
    if (child != 0x7FFFFFFF) atomicMin(&s_child, child);
    __syncthreads();
    r_child = s_child == 0x7FFFFFFF ? -1 : s_child;
    r_token = token;
    return true;
  };
  while (true) {
    if (!declined && !take_step()) break;
    first = declined = false;
    // the step's result, and where to go from there
    if (ahead) {
      if (!publish_and_next(r_child, r_token, r_state)) break;
      r_state = kDone;
      continue;
    }
    if (tid == 0) {
      path_out[n] = cur;
      tokens_out[n] = r_token;
    }
    __syncthreads();  // everybody has read child and token before the next step clears them
    ++n;
    ++depth;
    const int stepped = cur;
    cur = uniform(r_child);
    if constexpr (MANY) {
      // What the others have found.  A node one of them is at is waited for as long as the walker's own last step took, and
      // some 4 us for their way there: they have begun earlier, if they have begun.
      if (__builtin_expect(cur >= 0, 0)) {  // (out of the way of the steps: with it inside, a flat one is 0.2 to 0.8 us longer)
        if (wave == 0) {
          const unsigned tag = (unsigned)uniform((int)s_tag);
          if (lane == 0) post(0, pack_word(tag, stepped, cur, (unsigned)depth, kWalking));
          const u64 now = __builtin_amdgcn_s_memtime(), until = now + (now - begun) + 8192;
          int at = cur, dep = depth;
          while (true) {
            const u64 w0 = word(min(lane, words - 1)), w1 = word(min(kNodes + lane, words - 1));
            const bool wait = chase(w0, w1, tag, at, dep, [&](int node, const Word& r) {
              if (lane != 0) return;
              path_out[n + dep - depth] = node;
              tokens_out[n + dep - depth] = (int)r.token;
              if (r.state == kDoneError) s_err = 1;
            });
            if (!wait || __builtin_amdgcn_s_memtime() >= until) break;
          }
          if (lane == 0) {
            s_pick = at;
            s_hops = dep;
          }
        }
        __syncthreads();
        cur = uniform(s_pick);
        n += uniform(s_hops) - depth;
        depth = uniform(s_hops);
        __syncthreads();
        begun = __builtin_amdgcn_s_memtime();
      }
    }
    if (cur < 0) break;
  }
  if (!ahead && tid == 0) {
    n_out[0] = n;
    if (s_err) status[0] = SX_ERR_TREE;
    if (MANY) post(0, pack_word(s_tag, 0, -1, 0, kEnded));
  }
}

template <int NT, bool INLDS, bool SI, bool MANY>
__global__ __launch_bounds__(NT) void accept_walk_kernel(const float* __restrict__ logits,
                                                         const float* __restrict__ draft_probs,
                                                         const int* __restrict__ tokens,
                                                         const int* __restrict__ parent, int T, int V,
                                                         float temperature, float top_p, u64 seed,
                                                         int pos0, int* __restrict__ path_out,
                                                         int* __restrict__ tokens_out, int* __restrict__ n_out,
                                                         float* __restrict__ scratch, u64* __restrict__ rec,
                                                         int* __restrict__ status) {
  __shared__ Shared<NT, SI> sh;
  extern __shared__ __attribute__((aligned(1024))) float row[];  // INLDS: V rounded up to 4 NT
  if (!MANY || blockIdx.x == 0) {
    walk_steps<NT, INLDS, SI, MANY, false>(logits, draft_probs, tokens, parent, T, V, temperature, top_p, seed, pos0, path_out,
                                           tokens_out, n_out, scratch, rec, status, sh, row);
    return;
  }
  // Workgroups go round the eight XCDs; those that would share the walker's, and its L2, stay away.  (A flat row of 128256
  // is read again and again from there: 139.7 us for the step with seven others' rows beside it, 135.2 without; a peaked walk
  // over 64 such nodes 23.3 and 24.3.)
  if constexpr (MANY)
    if (blockIdx.x & 7)
      walk_steps<NT, INLDS, SI, MANY, true>(logits, draft_probs, tokens, parent, T, V, temperature, top_p, seed, pos0, path_out,
                                            tokens_out, n_out, scratch, rec, status, sh, row);
}

}  // namespace

namespace {

struct WalkArgs {
  const float *logits, *draft_probs;
  const int *tokens, *parent;
  int T, V;
  float temperature, top_p;
  u64 seed;
  int pos0;
  int *path_out, *tokens_out, *n_out;
  float* ebuf;
  u64* rec;  // null: one workgroup
  int* status;
};

template <int NT, bool INLDS, bool SI, bool MANY>
int launch_walk(const WalkArgs& a, hipStream_t st) {
  const size_t row_bytes = INLDS ? sx_align_up((size_t)a.V * 4, (size_t)NT * 16) : 0;
  if (INLDS) {  // above the default limit of dynamic LDS: allowed once per device
    static bool configured[64] = {};
    int dev = 0;
    SX_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64) return SX_ERR_HIP;
    if (!configured[dev]) {
      SX_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&accept_walk_kernel<NT, INLDS, SI, MANY>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)sx_align_up((NT == 256 ? 4096 : 32768) * 4, (size_t)NT * 16)));
      configured[dev] = true;
    }
  }
  int blocks = 1;
  if (MANY) {  // a walker and up to 63 others, who number without the multiples of 8
    const int others = (a.T < kNodes ? a.T : kNodes) - 1;
    blocks += others + (others - 1) / 7;
  }
  accept_walk_kernel<NT, INLDS, SI, MANY><<<blocks, NT, row_bytes, st>>>(
      a.logits, a.draft_probs, a.tokens, a.parent, a.T, a.V, a.temperature, a.top_p, a.seed, a.pos0, a.path_out, a.tokens_out,
      a.n_out, a.ebuf, a.rec, a.status);
  SX_LAUNCH_CHECK();
  return SX_OK;
}
template <bool INLDS, bool SI>
int launch_walks(const WalkArgs& a, hipStream_t st) {
  return a.rec ? launch_walk<1024, INLDS, SI, true>(a, st) : launch_walk<1024, INLDS, SI, false>(a, st);
}

// Many workgroups where the parents fit the LDS and the steps saved outweigh what their code costs a flat row that ends the
// walk at once, 2.5 us up to V = 32768 and 1 above (us, peaked walk to the last node, by one workgroup -> by many | flat):
// 4 nodes, V = 5000 17.8 -> 9.3 | 21.0 -> 23.7, V = 32000 26.5 -> 11.6 | 42.9 -> 45.2; 2 nodes, V = 5000 10.0 -> 9.5 |
// 21.0 -> 23.9, V = 32000 14.3 -> 10.5 | 42.9 -> 45.3, V = 33000 by ratio 17.2 -> 11.7 | 84.8 -> 86.0.
bool walk_by_many(int32_t T, int32_t V) { return V > kSmallVocab && T <= kStageNodes && (T > 3 || (T > 1 && V > 32768)); }
size_t scratch_bytes(int32_t V) { return sx_align_up((size_t)V * 4, 256); }

}  // namespace

extern "C" size_t sx_accept_walk_workspace(int32_t T, int32_t V) {
  if (V < 1) return 0;
  // (one workgroup walks a larger tree, but a buffer sized for it is to serve the smaller ones too)
  if (T > kStageNodes) T = kStageNodes;
  // many workgroups: the words, and a scratch row for every other workgroup
  const size_t many = walk_by_many(T, V)
                          ? sx_align_up((size_t)(T < kWords ? T : kWords) * 8, 256) + (size_t)((T < kNodes ? T : kNodes) - 1) * scratch_bytes(V)
                          : 0;
  return sx_accept_walk_min_workspace(V) + many;
}
size_t sx_accept_walk_min_workspace(int32_t V) { return SX_WS_HEADER + scratch_bytes(V); }

extern "C" int sx_accept_walk(const float* logits, const float* draft_probs, const int32_t* tree_tokens,
                              const int32_t* parent_idx, int32_t T, int32_t V, float temperature, float top_p,
                              uint64_t seed, int32_t pos0, int32_t* path_out, int32_t* tokens_out, int32_t* n_out,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (!logits || !tree_tokens || !parent_idx || !path_out || !tokens_out || !n_out) return SX_ERR_NULL;
  if (T < 1 || V < 1 || V > 131072 || !(top_p > 0.f) || top_p > 1.f || !(temperature >= 0.f)) return SX_ERR_SHAPE;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) || workspace_bytes < sx_accept_walk_min_workspace(V))
    return SX_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  int* status = reinterpret_cast<int*>(workspace);
  float* ebuf = reinterpret_cast<float*>(static_cast<char*>(workspace) + SX_WS_HEADER);
  // (a workspace of the size that one workgroup needs is one workgroup's)
  u64* rec = nullptr;
  if (walk_by_many(T, V) && workspace_bytes >= sx_accept_walk_workspace(T, V)) {
    rec = reinterpret_cast<u64*>(static_cast<char*>(workspace) + sx_accept_walk_min_workspace(V));
  }
  const WalkArgs a = {logits, draft_probs, tree_tokens, parent_idx, T, V, temperature, top_p, (u64)seed, pos0, path_out,
                      tokens_out, n_out, ebuf, rec, status};
  sx_prof_begin(SX_K_WALK, st);
  int rc;
  // the row in LDS while it fits; small rows with fewer waves to meet at the barriers
  if (V <= kSmallVocab)
    rc = draft_probs ? launch_walk<256, true, true, false>(a, st) : launch_walk<256, true, false, false>(a, st);
  else if (V <= 32768)
    rc = draft_probs ? launch_walks<true, true>(a, st) : launch_walks<true, false>(a, st);
  else
    rc = draft_probs ? launch_walks<false, true>(a, st) : launch_walks<false, false>(a, st);
  sx_prof_end(st);
  return rc;
}
