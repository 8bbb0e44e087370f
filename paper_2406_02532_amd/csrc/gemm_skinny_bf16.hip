// Y = X W^T for few rows (M <= 128): the linear layers of the draft model's forward over one batch of tree
// nodes (Alg. 2, forward(batch, theta_draft)).  At this M the product is bound by streaming the weights once
// from HBM, so the tile is narrow in N (all rows x 64, 96 or 128 columns: many workgroups, each a different slice of W)
// and, where even that leaves compute units idle, K is cut as well and the partial sums are added up by the
// last workgroup to arrive, in a fixed order.  Same building blocks as the wide kernel: operands go global ->
// LDS by buffer loads that write LDS (whole 128-byte lines, chunk swizzle applied on the global side), slabs of K = 64
// in as many stages as fit, one barrier per slab, v_mfma_f32_16x16x32_bf16 with the product formed transposed so that
// a lane holds 4 consecutive output columns.
//
// What bounds it: HBM up to some 32 rows (5.5 to 6.6 TB/s of weights where the chip is full); beyond that the copies into LDS
// as a whole, weights and X together, at 10 to 11 TB/s: every column tile copies all of X again, at 100 rows and 128 columns
// as many bytes as of W.  Hence:
//   the tile has as many blocks of 16 rows as M asks for (1, 2, 4, 5, 7 or 8), whose room goes to further stages (up to five);
//   96 columns where 128 leave a third of the chip idle (gate|up of 2 x 11008: 172 tiles or 230);
//   of 96 columns on, W goes past the caches' other contents (nontemporal), which leaves X there (without it, at 100 rows: head
//   of 32000 51.4 us for 47.4, 7B gate|up 38.4 for 36.4, 70B down 99 for 89).  With 64 columns, cut, that was 2 to 7 % slower, and
//   so it is with a single matrix that the last-level cache still holds from the call before: 7B gate|up over and over, 100 rows,
//   35.8 us for 33.2, and 31 with the kernel before; a model's layers do not meet that.
// Weights from memory, us, the kernel before (128 rows of X always, 64 or 128 columns, three or four stages) -> now, at 16,
// 64, 100 and 128 rows: 7B QKV 33.4 -> 23.2, 34.5 -> 26.4, 35.8 -> 29.2, 37.1 -> 31.1; O 14.0 -> 10.5, 14.8 -> 12.1, 15.5 -> 14.6,
// 16.1 -> 15.7; gate|up 34.7 -> 30.0, 38.1 -> 31.8, 41.6 -> 36.0, 45.1 -> 38.5; down 25.1 -> 19.0, 26.2 -> 22.4, 27.8 -> 27.4, 30.1
// -> 29.4; head of 32000 45.2 -> 43.1, 47.5 -> 42.2, 50.1 -> 47.0, 52.8 -> 49.3; 70B O 33.1 -> 25.9, 35.1 -> 28.9, 37.0 -> 34.8,
// 38.9 -> 38.8; down 89.5 -> 71.8, 94.7 -> 79.4, 102.0 -> 89.6, 107.2 -> 97.2.  Nineteen shapes at 13 row counts: 0.85 of the time.
// Measured and not kept: W straight into registers in the layout of the MFMA operand (a load then touches 16 rows, 64 bytes
// each, and the address unit bounds it: head at 100 rows 59 us); 32 columns (7B O at 16 rows 9.2, no better from 64 rows on); a
// walk that starts at the same slab everywhere (see the rotation below).
#include "kernels.h"

namespace {

constexpr int BK = 64;  // K of a slab

struct SkinnyArgs {
  const unsigned short* X;
  const void* W[3];  // bf16 [n][K]
  int n0, n1, n2;    // rows of the stacked matrices
  void* Y;
  int M, N, K;       // N: columns of Y (SwiGLU: of one matrix)
  int tiles, split;
  int rounds;        // of workgroups, one per compute unit
  float* part;
  int* part_cnt;
  const float2* cs;  // QKV: rows of 64 (cos, sin)
  unsigned short *q, *k, *v;
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// (bytes 0: reads nothing)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int bytes = -1) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// all LDS reads of this wave done, at most N of its vector-memory operations outstanding
constexpr int wait_vm(int n) { return 0x0070 | (n & 15) | ((n >> 4) << 14); }

// Copy instructions (1 KB each) of a slab: RB blocks of 16 rows of X, then BN rows of W; the same number to every wave, and a KB
// of its own in the stage for those that are over.
constexpr int copies(int rb, int bn) { return rb * 2 + bn / 8; }
constexpr int stage_kb(int rb, int bn, int waves) { return copies(rb, bn) + (copies(rb, bn) % waves != 0); }
// stages of a tile: as many as fit the 160 KB of LDS, up to 5 (eight were no faster: 0.856 of the time of the kernel before over
// 14 shapes at 1 to 128 rows, five 0.849, four 0.850, three 0.889)
constexpr int stages(int rb, int bn, int waves) {
  const int s = (160 * 1024 - 1024) / (stage_kb(rb, bn, waves) * 1024);
  return s < 5 ? s : 5;
}

// CG column groups of WB blocks of 16 columns, times RG groups of rows: a wave each; RB blocks of 16 rows.
template <int MODE, int CG, int RG, int WB, int RB>
__global__ __launch_bounds__(64 * CG * RG) void gemm_skinny_bf16_kernel(SkinnyArgs a) {
  constexpr int NW = CG * RG;
  constexpr int S = stages(RB, 16 * CG * WB, NW);
  constexpr int NCB = CG * WB, BN = 16 * NCB;   // columns of the workgroup, in blocks and singly
  constexpr int RW = (RB + RG - 1) / RG;        // row blocks per wave
  constexpr int BLOCKS = RB * NCB;              // 16 x 16 blocks of the tile
  constexpr int kPartFloats = BLOCKS * 256;     // partial sums of one K part of one tile
  // CP copy instructions to every wave; what is over reads nothing.  (Behind a branch by wave, the compiler would wait for more
  // of them than needed before each LDS read.)
  constexpr int COPIES = copies(RB, BN), CP = (COPIES + NW - 1) / NW;
  constexpr int kXBytes = RB * 2048, kStage = stage_kb(RB, BN, NW) * 1024;
  constexpr bool kStream = BN >= 96;            // W past the caches' other contents, where an instruction is all W
  constexpr int kNt = 2;
  constexpr bool kPairs = MODE == SX_GEMM_SWIGLU || MODE == SX_GEMM_QKV_ROPE;
  static_assert(CP <= 8 && S >= 3 && S <= 5, "");
  // one array per stage: X rows then W rows, 128 bytes each, 16-byte chunk c of row r at position c ^ ((r >> 1) & 7)
  __shared__ __attribute__((aligned(1024))) unsigned char st0[kStage];
  __shared__ __attribute__((aligned(1024))) unsigned char st1[kStage];
  __shared__ __attribute__((aligned(1024))) unsigned char st2[kStage];
  __shared__ __attribute__((aligned(S > 3 ? 1024 : 16))) unsigned char st3[S > 3 ? kStage : 16];
  __shared__ __attribute__((aligned(S > 4 ? 1024 : 16))) unsigned char st4[S > 4 ? kStage : 16];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int wc = wave % CG, wr = wave / CG;
  const int tile_n = blockIdx.x / a.split, kpart = blockIdx.x % a.split;
  // Where columns go in pairs (gate and up, the two halves of a head), the tile's blocks of 16 alternate between the first
  // and the second of them.
  auto stacked_row = [&](int col) {  // column of the tile -> row of the stacked matrices
    const int p = tile_n * (BN / 2) + (col >> 5) * 16 + (col & 15), second = (col >> 4) & 1;
    return MODE == SX_GEMM_SWIGLU    ? min(p, a.n0 - 1) + (second ? a.n0 : 0)
           : MODE == SX_GEMM_QKV_ROPE ? min((p >> 6) * 128 + second * 64 + (p & 63), a.N - 1)
                                      : min(tile_n * BN + col, a.N - 1);
  };

  // ---- copies: instruction c fills rows 8 c .. 8 c + 7 of the stage; wave w issues w, w + NW, ...
  const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.X);
  __amdgpu_buffer_rsrc_t res[8];
  int off[8];  // [CP] (of sizes that the template does not give the host pass drops the kernel)
#pragma unroll
  for (int t = 0; t < CP; ++t) {
    const int c = wave + t * NW, r = 8 * (c < RB * 2 ? c : c - RB * 2) + (lane >> 3);
    const int chunk = (lane & 7) ^ ((r >> 1) & 7);
    if (c < RB * 2) {
      res[t] = xres;
      off[t] = (int)(((unsigned)min(r, a.M - 1) * (unsigned)a.K + chunk * 8) * 2u);
    } else if (c < COPIES) {
      const int b0 = stacked_row((c - RB * 2) * 8);  // (eight rows belong to one of the stacked matrices)
      const int which = b0 >= a.n0 + a.n1 ? 2 : b0 >= a.n0 ? 1 : 0;
      const int n = stacked_row(r) - (which == 2 ? a.n0 + a.n1 : which == 1 ? a.n0 : 0);
      res[t] = make_rsrc(which == 2 ? a.W[2] : which == 1 ? a.W[1] : a.W[0]);
      off[t] = (int)(((unsigned)n * (unsigned)a.K + chunk * 8) * 2u);
    } else {
      res[t] = make_rsrc(a.X, 0);
      off[t] = 0;
    }
  }
  // Slabs [first, first + NB) of K from slab first + rot on and round.  Past the end of the walk the copies read nothing (with
  // the last slab again, a part of 16 slabs in five stages copied a quarter as much once more).
  const int nb_all = a.K / BK;
  const int first = kpart * nb_all / a.split;
  const int NB = (kpart + 1) * nb_all / a.split - first;
  // Every workgroup walks its slabs from another one on.  Started all at their first, hundreds of workgroups ask for the
  // same 128 bytes of rows that lie a power of two apart, step after step, and the memory channels take turns.  By
  // neighbours on an XCD in a launch of one round, by all neighbours where later rounds drift apart anyway: in this kernel's
  // predecessor 7B gate|up at 100 rows 46.8 -> 41.5 us, head of 32000 rows 61.3 -> 50.7, of 128256 rows 236 -> 204.
  const int rot = (int)((a.rounds > 1 ? 5u * blockIdx.x : blockIdx.x >> 3) % (unsigned)NB);
  const int so_begin = first * (BK * 2), so_end = so_begin + NB * (BK * 2);
  int so = so_begin + rot * (BK * 2), left = NB;  // the next slab to copy; slabs to copy
  const __amdgpu_buffer_rsrc_t nothing = make_rsrc(a.X, 0);
#define SX_COPY(STG_)                                                                                            \
  {                                                                                                              \
    const bool some = __builtin_amdgcn_readfirstlane(left) > 0;                                                  \
    _Pragma("unroll") for (int t = 0; t < CP; ++t) {                                                             \
      const lds_void_ptr to = (lds_void_ptr)(STG_ + min(wave + t * NW, COPIES) * 1024);                          \
      const __amdgpu_buffer_rsrc_t from = some ? res[t] : nothing;                                               \
      if (kStream && t * NW >= RB * 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(from, to, 16, off[t], so, 0, kNt); \
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(from, to, 16, off[t], so, 0, 0);                             \
    }                                                                                                            \
    so = so + BK * 2 == so_end ? so_begin : so + BK * 2;                                                         \
    --left;                                                                                                      \
    asm volatile("" ::: "memory"); /* (the waits count copies, which must go out slab by slab) */                \
  }
// this wave's copies but those of the N_ youngest slabs are in; then everybody's
#define SX_WAIT(N_)                                                                                              \
  asm volatile("" ::: "memory");                                                                                 \
  __builtin_amdgcn_s_waitcnt(wait_vm((N_) * CP));                                                                \
  __builtin_amdgcn_s_barrier();                                                                                  \
  asm volatile("" ::: "memory");

  // acc[i][j]: W rows (output columns) 16 (WB wc + i) .. + 15 of the tile, X rows (output rows) 16 (RW wr + j) .. + 15
  f32x4 acc[WB][RW];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < RW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fsw = (l16 >> 1) & 7;
  const int wrow = kXBytes + (WB * wc * 16 + l16) * 128;
#define SX_SLAB(STG_)                                                                                            \
  _Pragma("unroll") for (int s = 0; s < 2; ++s) {                                                                \
    bf16x8 fw[WB], fx[RW];                                                                                       \
    const int kc = ((4 * s + lq) ^ fsw) << 4;                                                                    \
    _Pragma("unroll") for (int i = 0; i < WB; ++i)                                                               \
        fw[i] = *reinterpret_cast<const bf16x8*>(STG_ + wrow + i * 2048 + kc);                                   \
    _Pragma("unroll") for (int j = 0; j < RW; ++j)                                                               \
        fx[j] = *reinterpret_cast<const bf16x8*>(STG_ + (min(RW * wr + j, RB - 1) * 16 + l16) * 128 + kc);       \
    _Pragma("unroll") for (int i = 0; i < WB; ++i) _Pragma("unroll") for (int j = 0; j < RW; ++j)                \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i], fx[j], acc[i][j], 0, 0, 0);                   \
  }

  // Slab t of the walk sits in stage t % S.  Per slab: wait for its copies (those of the next S - 2 stay in flight) and for
  // everybody to be done with the slab before it, start the copies of slab t + S - 1 into that stage, multiply.
  SX_COPY(st0)
  SX_COPY(st1)
  if constexpr (S > 3) SX_COPY(st2)
  if constexpr (S > 4) SX_COPY(st3)
#define SX_STEP(STG_, PREV_)             \
  {                                      \
    SX_WAIT(S - 2)                       \
    SX_COPY(PREV_)                       \
    SX_SLAB(STG_)                        \
  }
#define SX_STEP0()                                   \
  if constexpr (S == 3) SX_STEP(st0, st2)            \
  if constexpr (S == 4) SX_STEP(st0, st3)            \
  if constexpr (S == 5) SX_STEP(st0, st4)
  int s = 0;
  for (; s + S <= NB; s += S) {
    SX_STEP0()
    SX_STEP(st1, st0)
    SX_STEP(st2, st1)
    if constexpr (S > 3) SX_STEP(st3, st2)
    if constexpr (S > 4) SX_STEP(st4, st3)
  }
  s = NB - s;  // slabs left, fewer than S
  if (s > 0) {
    SX_STEP0()
    if (s > 1) {
      SX_STEP(st1, st0)
      if (S > 3 && s > 2) {
        SX_STEP(st2, st1)
        if constexpr (S > 4) if (s > 3) SX_STEP(st3, st2)
      }
    }
  }
  SX_WAIT(0)  // every copy is in and every stage is read: the LDS is free
#undef SX_STEP0
#undef SX_STEP
#undef SX_SLAB
#undef SX_COPY
#undef SX_WAIT

  // ---- which 16 x 16 blocks of the tile are this wave's from here on; block b = row block * NCB + column block.  Columns in pairs
  // go by unit, two blocks side by side.  A wave of two column blocks keeps its own (row blocks past the last one are the last
  // again, with the same sums, and store nothing), unless the waves' row blocks are too uneven; otherwise the waves leave theirs
  // in LDS, as the lanes hold them, and take every NW-th unit.  (All dealt out anew, head of 32000 x 768 at 100 rows 15.8 us, 768
  // x 3072 of gate|up 3 % more; none, 2048 x 2048 at 32 rows 7.8 us for 7.5, four row groups sharing two blocks.)
  constexpr int PER = kPairs ? 2 : 1;                        // blocks of a unit
  constexpr int UNITS = BLOCKS / PER;
  constexpr bool kDeal = WB != 2 || RW * RG * 5 > RB * 6;
  constexpr int NU = kDeal ? (UNITS + NW - 1) / NW : RW * WB / PER;  // per wave
  auto unit_ok = [&](int u) { return kDeal ? wave + u * NW < UNITS : RW * wr + u * PER / WB < RB; };
  auto unit = [&](int u) {
    return kDeal ? min(wave + u * NW, UNITS - 1)
                 : min(RW * wr + u * PER / WB, RB - 1) * (NCB / PER) + wc * (WB / PER) + u % (WB / PER);
  };
  f32x4 v[NU][PER];
  if constexpr (kDeal) {
    auto slot = [&](int b) -> unsigned char* {
      constexpr int PER_STAGE = kStage / 1024;
      const int stage = b / PER_STAGE;
      return (stage == 0 ? st0 : stage == 1 ? st1 : stage == 2 ? st2 : stage == 3 ? st3 : st4) +
             (b - stage * PER_STAGE) * 1024 + lane * 16;
    };
    static_assert(BLOCKS <= S * (kStage / 1024), "a block lies in one stage");
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < RW; ++j)
        if (RB % RG == 0 || RW * wr + j < RB) *reinterpret_cast<f32x4*>(slot((RW * wr + j) * NCB + WB * wc + i)) = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int e = 0; e < PER; ++e) v[u][e] = *reinterpret_cast<const f32x4*>(slot(unit(u) * PER + e));
  } else {
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int e = 0; e < PER; ++e) v[u][e] = acc[(u * PER + e) % WB][u * PER / WB];
  }

  // ---- K split: partial sums meet in memory, the last workgroup to arrive adds them in part order
  // (device-scope stores and loads, stores complete before the counter's device-scope atomic is issued)
  if (a.split > 1) {
    constexpr int kScopeDevice = 16;
    __shared__ int s_last;
    const __amdgpu_buffer_rsrc_t pres = make_rsrc(a.part);
    const unsigned all = (unsigned)(tile_n * a.split * kPartFloats + lane * 4) * 4u;  // bytes
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int b = unit(u) * PER + e;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[u][e]), pres,
                                               all + (unsigned)kpart * (kPartFloats * 4u) + b * 1024, 0, kScopeDevice);
      }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __syncthreads();
    if (tid == 0) {
      const int before = atomicAdd(a.part_cnt + tile_n, 1);
      s_last = before == a.split - 1;
      if (s_last) a.part_cnt[tile_n] = 0;  // ready for the next launch
    }
    __syncthreads();
    if (!s_last) return;
    // all blocks of a part are requested together (one memory round trip per part, not one per block); the workgroup's own
    // part comes from its registers (the same bits that it stored)
    f32x4 sum[NU][PER];
    for (int p = 0; p < a.split; ++p) {
      f32x4 x[NU][PER];
      if (p == kpart) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int e = 0; e < PER; ++e) x[u][e] = v[u][e];
      } else {
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int e = 0; e < PER; ++e)
            x[u][e] = __builtin_bit_cast(
                f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                           pres, all + (unsigned)p * (kPartFloats * 4u) + (unit(u) * PER + e) * 1024, 0,
                           kScopeDevice));
      }
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < PER; ++e) sum[u][e] = p == 0 ? x[u][e] : sum[u][e] + x[u][e];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int e = 0; e < PER; ++e) v[u][e] = sum[u][e];
  }
  // ---- epilogue.  v[u][.][e]: output row 16 j + l16, column 4 lq + e of its block
  if constexpr (MODE == SX_GEMM_SWIGLU) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = unit(u), m = b / (NCB / 2) * 16 + l16, f = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      if (!unit_ok(u) || m >= a.M || f >= a.N) continue;
      float h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = silu_mul_bf16_bound(v[u][0][e], v[u][PER - 1][e]);
      unsigned short* y = static_cast<unsigned short*>(a.Y) + (size_t)m * a.N + f;
      u32x2 o;
      o[0] = pack_bf16x2(h[0], h[1]);
      o[1] = pack_bf16x2(h[2], h[3]);
      if ((a.N & 3) == 0) {
        *reinterpret_cast<u32x2*>(y) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (f + e < a.N) y[e] = (unsigned short)(o[e >> 1] >> (16 * (e & 1)));
      }
    }
  } else if constexpr (MODE == SX_GEMM_QKV_ROPE) {
    // a unit's blocks hold the pairs that the rotary embedding turns by the row's angle; rounded once, after it
    const int hq = a.n0 >> 7, hkv = a.n1 >> 7;
    f32x4 t[NU][2];
#pragma unroll
    for (int u = 0; u < NU; ++u) {  // all rows' angles are requested before the first is used
      const int b = unit(u), p = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      const f32x4* c = reinterpret_cast<const f32x4*>(a.cs + (size_t)min(b / (NCB / 2) * 16 + l16, a.M - 1) * 64 + (p & 63));
      t[u][0] = c[0];
      t[u][1] = c[1];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = unit(u), m = b / (NCB / 2) * 16 + l16, p = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      if (!unit_ok(u) || m >= a.M || 2 * p >= a.N) continue;
      const int head = p >> 6;
      const bool is_v = head >= hq + hkv;
      const int nheads = head < hq ? hq : hkv, first_head = is_v ? hq + hkv : head >= hq ? hq : 0;
      unsigned short* y = (head < hq ? a.q : is_v ? a.v : a.k) + ((size_t)m * nheads + head - first_head) * 128 + (p & 63);
      float lo[4], hi[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x0 = v[u][0][e], x1 = v[u][PER - 1][e];
        rope_turn(x0, x1, t[u][e >> 1][2 * (e & 1)], t[u][e >> 1][2 * (e & 1) + 1], lo[e], hi[e]);
        if (is_v) lo[e] = x0, hi[e] = x1;
      }
      u32x2 o;
      o[0] = pack_bf16x2(lo[0], lo[1]);
      o[1] = pack_bf16x2(lo[2], lo[3]);
      *reinterpret_cast<u32x2*>(y) = o;
      o[0] = pack_bf16x2(hi[0], hi[1]);
      o[1] = pack_bf16x2(hi[2], hi[3]);
      *reinterpret_cast<u32x2*>(y + 64) = o;
    }
  } else if ((a.N & 3) == 0) {
    // the residual of all blocks is requested before the first add (rows and columns past the end read the last ones and
    // store nothing); block by block the epilogue was a chain of memory round trips
    float* Y = static_cast<float*>(a.Y);
    f32x4 r[NU];
    if (MODE == SX_GEMM_RESIDUAL) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int b = unit(u), m = min(b / NCB * 16 + l16, a.M - 1);
        r[u] = *reinterpret_cast<const f32x4*>(Y + (size_t)m * a.N + min(tile_n * BN + b % NCB * 16 + 4 * lq, a.N - 4));
      }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = unit(u), m = b / NCB * 16 + l16, n = tile_n * BN + b % NCB * 16 + 4 * lq;
      if (!unit_ok(u)) continue;
      if (m >= a.M || n >= a.N) continue;
      f32x4 x = v[u][0];
      if (MODE == SX_GEMM_RESIDUAL) x += r[u];
      *reinterpret_cast<f32x4*>(Y + (size_t)m * a.N + n) = x;
    }
  } else {
    float* Y = static_cast<float*>(a.Y);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = unit(u), m = b / NCB * 16 + l16, n = tile_n * BN + b % NCB * 16 + 4 * lq;
      if (!unit_ok(u) || m >= a.M) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) {
          float* y = Y + (size_t)m * a.N + n + e;
          if (MODE == SX_GEMM_RESIDUAL) *y += v[u][0][e];
          else *y = v[u][0][e];
        }
    }
  }
}

// Tiles of 128, 96 or 64 columns and cut of K.  The figures are fitted to 5100 launches at 1 to 128 rows, 40 products of 1024 to
// 57000 columns and K of 2048 to 28672, in all these forms, weights from memory: 2.1 us a round; a compute unit's copies at
// 63 GB/s and the weights from memory at 5.2 TB/s, which hinder each other (root of the sum of squares); and, cut, what the
// last arriver does.  The choice is within 0.6 % of the best launch on average, 8 % at worst.
// 96 columns only where columns come in pairs: they are for gate|up of 2 x 11008 rows (128 columns 41.6 us at 100 rows, 96 38.0)
// and QKV of 12288 (cut in two 29.4 and 25.8); none of the plain products of the models' layers is best with them.
struct SkinnyPlan {
  int columns, split;
};
SkinnyPlan plan_skinny(int M, int cols, int K, bool pairs, bool have_ws, size_t split_ws_bytes) {
  const int cus = sx_compute_units(), nb = K / BK, rb = M <= 16 ? 1 : M <= 32 ? 2 : M <= 64 ? 4 : M <= 80 ? 5 : M <= 112 ? 7 : 8;
  SkinnyPlan p = {64, 1};
  float best = 1e30f;
  for (int bn = 128; bn >= 64; bn -= 32) {
    if (bn == 96 && !pairs) continue;
    const int tiles = (cols + bn - 1) / bn;
    for (int split = 1; split <= 16; ++split) {
      const double part = split > 1 ? (double)split * rb * 16 * bn * sizeof(float) : 0.;  // bytes per tile
      if (split > 1 && (!have_ws || tiles > 256 || tiles * split > cus || nb / split < 6 || split_ws_bytes < 1024 + tiles * part))
        break;
      const int rounds = (tiles * split + cus - 1) / cus;
      const float unit = rounds * ((nb + split - 1) / split) * (rb * 2048 + bn * 128) / 63e3f;
      const float weights = (float)tiles * nb * bn * 128 / 5.2e6f;
      float cost = 2.1f * rounds + sqrtf(unit * unit + weights * weights) +
                   (split > 1 ? 1.3f + 0.07f * split + 2.5e-5f * (float)part : 0.f);
      if (split > 1 && bn == 128 && rb == 8) cost *= 1.01f;  // four stages instead of five: 8192 x 8192 at 128 rows 39.9 us, 64 columns 38.6
      if (cost < best) best = cost, p = {bn, split};
    }
  }
  return p;
}

template <int MODE, int CG, int RG, int WB>
void launch_rows(const SkinnyArgs& a, hipStream_t st) {
  // (fewer blocks of rows than row groups: the groups that are over multiply along, since all are wanted for the copies)
  const int grid = a.tiles * a.split;
  if (a.M <= 16) gemm_skinny_bf16_kernel<MODE, CG, 2, WB, 1><<<grid, 64 * CG * 2, 0, st>>>(a);
  else if (a.M <= 32) gemm_skinny_bf16_kernel<MODE, CG, RG, WB, 2><<<grid, 64 * CG * RG, 0, st>>>(a);
  else if (a.M <= 64) gemm_skinny_bf16_kernel<MODE, CG, RG, WB, 4><<<grid, 64 * CG * RG, 0, st>>>(a);
  else if (a.M <= 80) gemm_skinny_bf16_kernel<MODE, CG, RG, WB, 5><<<grid, 64 * CG * RG, 0, st>>>(a);
  else if (a.M <= 112) gemm_skinny_bf16_kernel<MODE, CG, RG, WB, 7><<<grid, 64 * CG * RG, 0, st>>>(a);
  else gemm_skinny_bf16_kernel<MODE, CG, RG, WB, 8><<<grid, 64 * CG * RG, 0, st>>>(a);
}

// cols: rows of W that the launch walks
template <int MODE>
int launch(SkinnyArgs& a, int cols, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  constexpr bool pairs = MODE == SX_GEMM_SWIGLU || MODE == SX_GEMM_QKV_ROPE;
  const SkinnyPlan p = plan_skinny(a.M, cols, a.K, pairs, split_ws != nullptr, split_ws_bytes);
  a.tiles = (cols + p.columns - 1) / p.columns;
  a.split = p.split;
  a.rounds = (a.tiles * a.split + sx_compute_units() - 1) / sx_compute_units();
  if (a.split > 1) {
    a.part_cnt = static_cast<int*>(split_ws);
    a.part = reinterpret_cast<float*>(static_cast<char*>(split_ws) + 1024);
  }
  if (p.columns == 128) {
    launch_rows<MODE, 4, 2, 2>(a, st);
  } else if (p.columns == 64) {
    launch_rows<MODE, 2, 4, 2>(a, st);
  } else if constexpr (pairs) {
    launch_rows<MODE, 2, 4, 3>(a, st);
  }
  SX_LAUNCH_CHECK();
  return SX_OK;
}

}  // namespace

// M <= 128.  Arguments as sx_launch_gemm_bf16 (modes store, residual, SwiGLU).
int sx_launch_gemm_skinny_bf16(const void* X, const void* W0, const void* W1, const void* W2, int n0, int n1, int n2,
                               void* Y, int M, int K, int mode, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || M > 128 || K < BK || K % BK != 0 || n0 < 1 || n1 < 0 || n2 < 0) return SX_ERR_SHAPE;
  if (!sx_operand_fits_u32(M, 2ll * K) || !sx_operand_fits_u32(n0, 2ll * K) || !sx_operand_fits_u32(n1, 2ll * K) ||
      !sx_operand_fits_u32(n2, 2ll * K))
    return SX_ERR_SHAPE;
  if (mode != SX_GEMM_SWIGLU && ((n1 > 0 && n0 % 8 != 0) || (n2 > 0 && n1 % 8 != 0))) return SX_ERR_SHAPE;
  SkinnyArgs a = {};
  a.X = static_cast<const unsigned short*>(X);
  a.W[0] = W0;
  a.W[1] = W1 ? W1 : W0;
  a.W[2] = W2 ? W2 : W0;
  a.n0 = n0;
  a.n1 = n1;
  a.n2 = n2;
  a.Y = Y;
  a.M = M;
  a.K = K;
  int cols;  // rows of W that a launch walks (gate and up both count)
  if (mode == SX_GEMM_SWIGLU) {
    if (n1 != n0 || n2 != 0 || !W1) return SX_ERR_SHAPE;
    a.N = n0;
    cols = 2 * n0;
  } else {
    a.N = n0 + n1 + n2;
    cols = a.N;
  }
  switch (mode) {
    case SX_GEMM_STORE: return launch<SX_GEMM_STORE>(a, cols, split_ws, split_ws_bytes, st);
    case SX_GEMM_RESIDUAL: return launch<SX_GEMM_RESIDUAL>(a, cols, split_ws, split_ws_bytes, st);
    case SX_GEMM_SWIGLU: return launch<SX_GEMM_SWIGLU>(a, cols, split_ws, split_ws_bytes, st);
  }
  return SX_ERR_SHAPE;
}

// The QKV projection with the rotation and the split into heads in the epilogue: sx_launch_gemm_qkv_rope_bf16, M <= 128.
int sx_launch_gemm_skinny_qkv_rope_bf16(const void* X, const void* Wq, const void* Wk, const void* Wv, int hq, int hkv,
                                        const float2* rope_cs, void* q, void* k, void* v, int M, int K, void* split_ws,
                                        size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || M > 128 || K < BK || K % BK != 0 || hq < 1 || hkv < 1) return SX_ERR_SHAPE;
  if (!sx_operand_fits_u32(M, 2ll * K) || !sx_operand_fits_u32(128ll * hq, 2ll * K) ||
      !sx_operand_fits_u32(128ll * hkv, 2ll * K))
    return SX_ERR_SHAPE;
  SkinnyArgs a = {};
  a.X = static_cast<const unsigned short*>(X);
  a.W[0] = Wq;
  a.W[1] = Wk;
  a.W[2] = Wv;
  a.n0 = hq * 128;
  a.n1 = a.n2 = hkv * 128;
  a.M = M;
  a.N = a.n0 + a.n1 + a.n2;
  a.K = K;
  a.cs = rope_cs;
  a.q = static_cast<unsigned short*>(q);
  a.k = static_cast<unsigned short*>(k);
  a.v = static_cast<unsigned short*>(v);
  return launch<SX_GEMM_QKV_ROPE>(a, a.N, split_ws, split_ws_bytes, st);
}

extern "C" int sx_gemm_bf16_narrow_plan_rows(int32_t M, int32_t N, int32_t K, int32_t mode, size_t workspace_bytes,
                                             int32_t* tile_columns, int32_t* k_parts) {
  if (!tile_columns || !k_parts) return SX_ERR_NULL;
  if (M < 1 || M > 128 || mode < 0 || mode > SX_GEMM_QKV_ROPE || N < 1 || K < BK || K % BK != 0) return SX_ERR_SHAPE;
  const SkinnyPlan p = plan_skinny(M, mode == SX_GEMM_SWIGLU ? 2 * N : N, K, mode == SX_GEMM_SWIGLU || mode == SX_GEMM_QKV_ROPE,
                                   workspace_bytes != 0, workspace_bytes);
  *tile_columns = p.columns;
  *k_parts = p.split;
  return SX_OK;
}

extern "C" int sx_gemm_bf16_narrow_plan(int32_t N, int32_t K, int32_t mode, size_t workspace_bytes, int32_t* tile_columns,
                                        int32_t* k_parts) {
  if (tile_columns && k_parts && (mode < 0 || mode > 2)) return SX_ERR_SHAPE;
  return sx_gemm_bf16_narrow_plan_rows(128, N, K, mode, workspace_bytes, tile_columns, k_parts);
}
