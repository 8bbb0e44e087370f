// Y = X W^T for few rows (M <= 128) with 4-bit group-quantised weights, second form (Sect. 5: the paper's fastest
// setting runs its models quantised to 4 bits; for the draft model's small batches the product is bound by
// streaming the weights, and these are a quarter of the bytes).
//
// The weights never pass through LDS.  The A operand of v_mfma_f32_16x16x32_bf16 wants, per lane, eight
// consecutive k of one W row -- exactly one 32-bit word of eight 4-bit codes.  So a lane fetches the words of
// its own fragments straight from global memory (16 bytes = four fragments per load), dequantises them in
// registers (w = bf16(scale * (code - zero)): one byte-to-float conversion and one fma per weight, exact in
// fp32, rounded once) and feeds the matrix core.  Only X goes through LDS (copied by buffer loads that write
// LDS), where the 128 rows are shared by the eight waves.
//
// Tiling: a workgroup owns all rows, in 1, 2, 4, 5, 7 or 8 blocks of 16 as M asks for, x 128, 96 or 64 columns.  K is walked in
// slabs of 128 (four k-steps), and its eight waves (96 columns: twelve) are four (six) column groups times the two halves of
// every slab's k-steps, whose sums meet in LDS at the end: two waves per SIMD without a second copy of X or a second
// partial tile.  The contraction index may be permuted as long as both operands agree: in k-step s of a slab a
// lane of quarter lq takes the 16-byte chunk 4 lq + s of its row, so its two fragments of the slab are one
// contiguous 8-byte load (64 contiguous bytes per W row).
// What bounds it: up to some 16 rows the stream of words (128 columns at 8192 x 28672 cut in four: 2.4 TB/s, 16 rows of a load
// at 32 bytes each); beyond that a compute unit's own slab, 0.58 us plus 0.08 per block of rows at 128 columns: X read from LDS
// by every column group, the dequantisation and the MFMAs, which hardly overlap.  So: no more row blocks than M asks for; X
// three slabs ahead in four stages (a barrier waits only for its own slab's operations, by count), whose swizzle keeps the
// fragment reads off each other's banks (conflicts half of the cycles in which the LDS is busy with row & 15, 5 to 14 % now); codes
// converted from their bytes in place (the compiler extracted each one first, 6 more instructions a word); scales and zero
// points of up to 48 groups fetched into LDS at a time, side by side; the words of two slabs, which share their lines, fetched
// together.  Weights from memory, us, the kernel before (128 rows always, 128 or 64 columns) -> now, at 16, 64, 100 and 128
// rows: 4096 x 4096 16.9 -> 11.8, 17.1 -> 13.7, 17.5 -> 17.0, 17.5 -> 17.6; 4096 x 11008 26.8 -> 16.7, 27.6 -> 21.0, 28.0 ->
// 27.4, 28.2 -> 28.3; 12288 x 4096 28.6 -> 16.8, 29.2 -> 21.4, 30.1 -> 26.1, 31.0 -> 28.5; 22016 x 4096 42.3 -> 22.9, 44.9 ->
// 30.2, 46.0 -> 36.3, 46.6 -> 40.2; 57344 x 8192 158 -> 88, 161 -> 122, 161 -> 151, 163 -> 160; 8192 x 28672 76.5 -> 48.2, 81.3
// -> 61.0, 82.5 -> 77.7, 82.1 -> 82.0.
// (The two k-steps software-pipelined by hand with the MFMAs, reads and dequantisation dealt out evenly, and codes made floats
// by their exponent bits instead of conversions, were measured: within 2 % either way.)
// Where column tiles are fewer than compute units the K range is cut among workgroups (grid.y); partial sums meet in
// memory and the last workgroup to arrive adds them in part order (deterministic, nobody waits).
//
// Up to three weight matrices may be stacked along N (the QKV projections, or gate and up) as long as each
// holds a multiple of 64 rows: a block of 16 columns then belongs to one matrix.
#include "kernels.h"

namespace {

constexpr int BK = 128;             // K of a slab
constexpr int kParGroups = 48;      // groups whose scales and zero points are in LDS at a time

struct W4Mat {
  const uint32_t* q;          // [n][K/8]
  const unsigned short* s;    // bf16 [n][K/group]
  const unsigned char* z;     // [n][K/group]
};

struct W4RegArgs {
  const unsigned short* X;
  W4Mat m[3];
  int n0, n1, n2;
  int group_log2;
  float* Y;
  int ldy;
  int M, N, K;
  int split;
  float* part;
  int* part_cnt;
  const float2* cs;                // QKV: rows of 64 (cos, sin)
  unsigned short *q, *k, *v;
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// (bytes 0: reads nothing)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, int bytes = -1) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// eight codes of one word -> eight bf16 in k order; sc = scale, nzs = -zero * scale (both exact in fp32, and so is
// code * sc + nzs = sc * (code - zero): 8 significant bits times at most 4)
__device__ __forceinline__ bf16x8 dequant8(uint32_t q, float sc, float nzs) {
  uint32_t lo = q & 0x0F0F0F0Fu, hi = (q >> 4) & 0x0F0F0F0Fu;  // codes 0,2,4,6 and 1,3,5,7, one per byte
  // (hidden from the compiler, which would extract each code's four bits first instead of converting its byte)
  asm("" : "+v"(lo), "+v"(hi));
  u32x4 o;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float e = fmaf((float)((lo >> (8 * b)) & 0xFFu), sc, nzs);
    const float f = fmaf((float)((hi >> (8 * b)) & 0xFFu), sc, nzs);
    o[b] = pack_bf16x2(e, f);
  }
  return __builtin_bit_cast(bf16x8, o);
}

// all LDS reads of this wave done, at most N of its vector-memory operations outstanding, then meet the other waves
constexpr int wait_vm(int n) { return 0x0070 | (n & 15) | ((n >> 4) << 14); }
#define SX_WAIT_BARRIER(IMM)               \
  asm volatile("" ::: "memory");           \
  __builtin_amdgcn_s_waitcnt(IMM);         \
  __builtin_amdgcn_s_barrier();            \
  asm volatile("" ::: "memory");

// CG column groups of WB blocks of 16 columns, times two halves of every slab's k-steps: a wave each; RB blocks of 16 rows.
template <int MODE, int CG, int WB, int RB>
__global__ __launch_bounds__(128 * CG) void gemm_w4_regs_kernel(W4RegArgs a) {
  constexpr int NW = 2 * CG, NT = 64 * NW;
  constexpr int NCB = CG * WB, BN = 16 * NCB;   // columns of the workgroup, in blocks and singly
  constexpr int BLOCKS = RB * NCB;              // 16 x 16 blocks of the tile
  constexpr int kPartFloats = BLOCKS * 256;     // partial sums of one K part of one tile
  // copy instructions (1 KB each) of a slab, CP to every wave; what is over reads nothing, into a KB of its own
  constexpr int CP = (RB * 4 + NW - 1) / NW;
  constexpr int kXBytes = RB * 4096 + (CP * NW > RB * 4 ? 1024 : 0);
  constexpr bool kPairs = MODE == SX_GEMM_SWIGLU || MODE == SX_GEMM_QKV_ROPE;
  static_assert(NCB <= 8, "the sums of a half fit two stages");
  __shared__ __attribute__((aligned(1024))) unsigned char sx0[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx1[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx2[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx3[kXBytes];
  __shared__ unsigned s_par[kParGroups * BN];  // [group][column]: the scale's bits, above the zero point
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int wc = wave % CG, half = wave / CG;  // columns; k-steps 2 half and 2 half + 1 of every slab
  const int tile_n = blockIdx.x, kpart = blockIdx.y;
  // Where columns go in pairs (gate and up, the two halves of a head), the tile's blocks of 16 alternate between the first
  // and the second of them.
  auto stacked_row = [&](int col) {  // column of the tile -> row of the stacked matrices, for pairs
    const int p = tile_n * (BN / 2) + (col >> 5) * 16 + (col & 15), second = (col >> 4) & 1;
    return MODE == SX_GEMM_SWIGLU ? min(p, a.n0 - 1) + (second ? a.n0 : 0)
                                  : min((p >> 6) * 128 + second * 64 + (p & 63), a.N - 1);
  };

  // ---- X copies.  A slab's row r is 256 bytes at 256 r, its 16-byte chunk c at position c ^ f(r): a fragment read takes
  // 16 lanes at a time -- eight rows 0..3 and 12..15 of one chunk with rows 4..11 of the next lane quarter's, or the other
  // eight of each -- and with f those fall on 16 different groups of banks.
  auto swizzle = [](int r) { return (r & 15) ^ (((r >> 2) ^ (r >> 3)) & 1) << 2; };
  const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.X), nothing = make_rsrc(a.X, 0);
  __amdgpu_buffer_rsrc_t xr[4];
  int xoff[4];  // [CP] (of sizes that the template does not give the host pass drops the kernel)
#pragma unroll
  for (int t = 0; t < CP; ++t) {
    const int id = wave + t * NW, r = 4 * id + (lane >> 4);
    xr[t] = id < RB * 4 ? xres : nothing;
    xoff[t] = (int)(((unsigned)min(r, a.M - 1) * (unsigned)a.K + ((lane & 15) ^ swizzle(r)) * 8) * 2u);
  }

  // ---- W: a block of 16 columns belongs to one of the stacked matrices
  int woff[WB];
  __amdgpu_buffer_rsrc_t wres[WB];
#pragma unroll
  for (int i = 0; i < WB; ++i) {
    const int col = 16 * (WB * wc + i);
    const int b0 = kPairs ? stacked_row(col) : min(tile_n * BN + col, a.N - 1);
    int n = kPairs ? stacked_row(col + l16) : min(tile_n * BN + col + l16, a.N - 1);  // past the end: the last row again
    const int which = b0 >= a.n0 + a.n1 ? 2 : b0 >= a.n0 ? 1 : 0;
    n -= which == 2 ? a.n0 + a.n1 : which == 1 ? a.n0 : 0;
    woff[i] = (int)(((unsigned)n * (unsigned)(a.K / 8) + 4u * lq + 2u * half) * 4u);  // + 64 bytes per slab
    wres[i] = make_rsrc(which == 2 ? a.m[2].q : which == 1 ? a.m[1].q : a.m[0].q);
  }
  struct WRegs {
    u32x2 q[WB];
  };
  WRegs w0, w1, w2, w3;

  // Slabs [first_slab, first_slab + NB) of K.  Past the end the copies of X read nothing, the words are those of the last slab.
  const int nb_all = a.K / BK;
  const int first_slab = kpart * nb_all / a.split;
  const int NB = (kpart + 1) * nb_all / a.split - first_slab;
#define SX_SLAB_AT(i) (first_slab + min((i), NB - 1))
#define SX_COPY(STG_, T_)                                                                                        \
  {                                                                                                              \
    const int so = (first_slab + (T_)) * (BK * 2);                                                               \
    const bool some = __builtin_amdgcn_readfirstlane(T_) < NB;                                                   \
    _Pragma("unroll") for (int t = 0; t < CP; ++t) __builtin_amdgcn_raw_ptr_buffer_load_lds(                     \
        some ? xr[t] : nothing, (lds_void_ptr)(STG_ + min(wave + t * NW, RB * 4) * 1024), 16, xoff[t], so, 0, 0); \
    asm volatile("" ::: "memory"); /* (the waits count operations: in this order) */                             \
  }
  // the words of slabs A_ and B_, which share their 128-byte lines
#define SX_PAIR(WA_, WB_, T_)                                                                                    \
  {                                                                                                              \
    const int sa = SX_SLAB_AT(T_) * 64, sb = SX_SLAB_AT((T_) + 1) * 64;                                          \
    asm volatile("" ::: "memory");                                                                               \
    _Pragma("unroll") for (int i = 0; i < WB; ++i) {                                                             \
      WA_.q[i] = __builtin_amdgcn_raw_buffer_load_b64(wres[i], woff[i], sa, 0);                                  \
      WB_.q[i] = __builtin_amdgcn_raw_buffer_load_b64(wres[i], woff[i], sb, 0);                                  \
    }                                                                                                            \
    asm volatile("" ::: "memory");                                                                               \
  }
  // Scales and zero points of the slabs [S0_, S1_) into LDS; par0 becomes the first of their groups.  A thread takes
  // four (column, group) pairs at a time, the groups of a column side by side in memory.
  int par0 = 0;
  const int ngroups = a.K >> a.group_log2;
  auto fill = [&](int s0, int s1) {
    par0 = (s0 * BK) >> a.group_log2;
    const int ng = ((s1 * BK - 1) >> a.group_log2) - par0 + 1, total = ng * BN;
    for (int b = 0; b < total; b += 4 * NT) {
      unsigned ps[4], pz[4];
      int at[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int idx = min(b + u * NT + tid, total - 1);
        const int col = idx / ng, g = idx - col * ng;
        int n = kPairs ? stacked_row(col) : min(tile_n * BN + col, a.N - 1);
        const int wm = n >= a.n0 + a.n1 ? 2 : n >= a.n0 ? 1 : 0;
        n -= wm == 2 ? a.n0 + a.n1 : wm == 1 ? a.n0 : 0;
        const size_t e = (size_t)n * ngroups + par0 + g;
        ps[u] = (wm == 2 ? a.m[2].s : wm == 1 ? a.m[1].s : a.m[0].s)[e];
        pz[u] = (wm == 2 ? a.m[2].z : wm == 1 ? a.m[1].z : a.m[0].z)[e];
        at[u] = g * BN + col;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) s_par[at[u]] = ps[u] << 16 | pz[u];
    }
  };

  // acc[i][j]: W rows (output columns) 16 (WB wc + i) .. + 15 of the tile, X rows (output rows) 16 j .. + 15
  f32x4 acc[WB][RB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // X fragment of block j in k-step s: row 16 j + l16, chunk 4 lq + 2 half + s
  const int xrow = l16 * 256;
#define SX_SLAB(XS_, W_, T_)                                                                                     \
  {                                                                                                              \
    /* group of this lane's k range, k = 128 slab + 32 lq + (0..31) (groups are powers of two >= 64) */          \
    const int g = (((first_slab + (T_)) * BK + 32 * lq) >> a.group_log2) - par0;                                 \
    float sc[WB], nzs[WB];                                                                                       \
    _Pragma("unroll") for (int i = 0; i < WB; ++i) {                                                             \
      const unsigned pr = s_par[g * BN + 16 * (WB * wc + i) + l16];                                              \
      sc[i] = __uint_as_float(pr & 0xFFFF0000u);                                                                 \
      nzs[i] = -(float)(pr & 0xFFu) * sc[i];                                                                     \
    }                                                                                                            \
    _Pragma("unroll") for (int s = 0; s < 2; ++s) {                                                              \
      bf16x8 fw[WB], fx[RB];                                                                                     \
      const int xc = xrow + (((4 * lq + 2 * half + s) ^ swizzle(l16)) << 4);                                     \
      _Pragma("unroll") for (int j = 0; j < RB; ++j)                                                             \
          fx[j] = *reinterpret_cast<const bf16x8*>(XS_ + j * 4096 + xc);                                         \
      _Pragma("unroll") for (int i = 0; i < WB; ++i) fw[i] = dequant8(W_.q[i][s], sc[i], nzs[i]);                \
      _Pragma("unroll") for (int i = 0; i < WB; ++i) _Pragma("unroll") for (int j = 0; j < RB; ++j)              \
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i], fx[j], acc[i][j], 0, 0, 0);                 \
    }                                                                                                            \
  }

  // Slab t sits in stage t % 4 and its W words in register set t % 4.  Per slab: wait for its own copies and words (the two
  // younger slabs' copies and the younger pair of words stay in flight) and for everybody to be done with the slab before it,
  // start the copies of slab t + 3 into that stage, multiply; after every second slab fetch the words of slabs t + 3 and
  // t + 4 together.
  constexpr int kFly = 2 * CP + 2 * WB;
#define SX_STEP(XS_, W_, XN_, T_)          \
  SX_WAIT_BARRIER(wait_vm(kFly))           \
  SX_COPY(XN_, (T_) + 3)                   \
  SX_SLAB(XS_, W_, T_)
  const int par_slabs = a.group_log2 > 6 ? kParGroups : kParGroups / 2;  // slabs whose groups fit s_par
  SX_COPY(sx0, 0)
  SX_PAIR(w0, w1, 0)
  SX_COPY(sx1, 1)
  SX_COPY(sx2, 2)
  SX_PAIR(w2, w3, 2)
  fill(first_slab, first_slab + min(NB, par_slabs));
  int t = 0, refill = par_slabs;
  for (; t + 4 <= NB; t += 4) {
    if (t == refill) {  // everybody is done with the last groups' parameters; the next barrier shows the new ones
      __syncthreads();
      fill(first_slab + t, first_slab + min(NB, t + par_slabs));
      refill += par_slabs;
    }
    SX_STEP(sx0, w0, sx3, t)
    SX_STEP(sx1, w1, sx0, t + 1)
    SX_PAIR(w0, w1, t + 4)
    SX_STEP(sx2, w2, sx1, t + 2)
    SX_STEP(sx3, w3, sx2, t + 3)
    SX_PAIR(w2, w3, t + 6)
  }
  // Up to three slabs are left, all on their way.  (They start no others: words nobody uses would be dropped by the
  // compiler, and the counts of operations in flight would not hold.)
  if (t < NB) {
    if (t == refill) {
      __syncthreads();
      fill(first_slab + t, first_slab + NB);
    }
    SX_WAIT_BARRIER(wait_vm(kFly))
    SX_SLAB(sx0, w0, t)
    if (t + 1 < NB) {
      SX_WAIT_BARRIER(wait_vm(CP + 2 * WB))
      SX_SLAB(sx1, w1, t + 1)
    }
    if (t + 2 < NB) {
      SX_WAIT_BARRIER(wait_vm(0))
      SX_SLAB(sx2, w2, t + 2)
    }
  }
  SX_WAIT_BARRIER(wait_vm(0))  // every copy is in and every stage is read: the LDS is free
#undef SX_STEP
#undef SX_SLAB
#undef SX_PAIR
#undef SX_COPY
#undef SX_SLAB_AT

  // ---- the sums meet in LDS, block after block of 16 x 16 as the lanes hold them; from here on block b = j NCB + column
  // block belongs to wave b % NW (pairs: their number, likewise)
  auto sums = [&](int k, int b) -> unsigned char* {
    const bool second = b >= RB * 4;
    return (k == 0 ? (second ? sx1 : sx0) : (second ? sx3 : sx2)) + (b - (second ? RB * 4 : 0)) * 1024 + lane * 16;
  };
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j) *reinterpret_cast<f32x4*>(sums(half, j * NCB + WB * wc + i)) = acc[i][j];
  __syncthreads();
  constexpr int PER = kPairs ? 2 : 1;                        // blocks of a unit, side by side in a row of blocks
  constexpr int UNITS = BLOCKS / PER, NU = (UNITS + NW - 1) / NW;  // per wave
  f32x4 v[NU][PER];
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int b = min(wave + u * NW, UNITS - 1) * PER + e;
      v[u][e] = *reinterpret_cast<const f32x4*>(sums(0, b)) + *reinterpret_cast<const f32x4*>(sums(1, b));
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
        const int b = min(wave + u * NW, UNITS - 1) * PER + e;
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
                           pres, all + (unsigned)p * (kPartFloats * 4u) + (min(wave + u * NW, UNITS - 1) * PER + e) * 1024, 0,
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
      const int b = wave + u * NW, m = b / (NCB / 2) * 16 + l16, f = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      if (b >= UNITS || m >= a.M || f >= a.n0) continue;
      float h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = silu_mul_bf16_bound(v[u][0][e], v[u][PER - 1][e]);
      u32x2 o;
      o[0] = pack_bf16x2(h[0], h[1]);
      o[1] = pack_bf16x2(h[2], h[3]);
      *reinterpret_cast<u32x2*>(reinterpret_cast<unsigned short*>(a.Y) + (size_t)m * a.n0 + f) = o;  // (n0 a multiple of 64)
    }
  } else if constexpr (MODE == SX_GEMM_QKV_ROPE) {
    // a unit's blocks hold the pairs that the rotary embedding turns by the row's angle; rounded once, after it
    const int hq = a.n0 >> 7, hkv = a.n1 >> 7;
    f32x4 t[NU][2];
#pragma unroll
    for (int u = 0; u < NU; ++u) {  // all rows' angles are requested before the first is used
      const int b = min(wave + u * NW, UNITS - 1), p = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      const f32x4* c = reinterpret_cast<const f32x4*>(a.cs + (size_t)min(b / (NCB / 2) * 16 + l16, a.M - 1) * 64 + (p & 63));
      t[u][0] = c[0];
      t[u][1] = c[1];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = wave + u * NW, m = b / (NCB / 2) * 16 + l16, p = tile_n * (BN / 2) + b % (NCB / 2) * 16 + 4 * lq;
      if (b >= UNITS || m >= a.M || 2 * p >= a.N) continue;
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
  } else if ((a.N & 3) == 0 && (a.ldy & 3) == 0) {
    // the residual of all blocks is requested before the first add (rows and columns past the end read the last ones and
    // store nothing); block by block the epilogue was a chain of memory round trips
    float* Y = a.Y;
    f32x4 r[NU];
    if (MODE == SX_GEMM_RESIDUAL) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int b = min(wave + u * NW, UNITS - 1), m = min(b / NCB * 16 + l16, a.M - 1);
        r[u] = *reinterpret_cast<const f32x4*>(Y + (size_t)m * a.ldy + min(tile_n * BN + b % NCB * 16 + 4 * lq, a.N - 4));
      }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = wave + u * NW, m = b / NCB * 16 + l16, n = tile_n * BN + b % NCB * 16 + 4 * lq;
      if (b >= UNITS) continue;
      if (m >= a.M || n >= a.N) continue;
      f32x4 x = v[u][0];
      if (MODE == SX_GEMM_RESIDUAL) x += r[u];
      *reinterpret_cast<f32x4*>(Y + (size_t)m * a.ldy + n) = x;
    }
  } else {
    float* Y = a.Y;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int b = wave + u * NW, m = b / NCB * 16 + l16, n = tile_n * BN + b % NCB * 16 + 4 * lq;
      if (b >= UNITS || m >= a.M) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < a.N) {
          float* y = Y + (size_t)m * a.ldy + n + e;
          if (MODE == SX_GEMM_RESIDUAL) *y += v[u][0][e];
          else *y = v[u][0][e];
        }
    }
  }
}
#undef SX_WAIT_BARRIER

template <int MODE, int CG, int WB>
void launch_rows(const W4RegArgs& a, dim3 grid, hipStream_t st) {
  if (a.M <= 16) gemm_w4_regs_kernel<MODE, CG, WB, 1><<<grid, 128 * CG, 0, st>>>(a);
  else if (a.M <= 32) gemm_w4_regs_kernel<MODE, CG, WB, 2><<<grid, 128 * CG, 0, st>>>(a);
  else if (a.M <= 64) gemm_w4_regs_kernel<MODE, CG, WB, 4><<<grid, 128 * CG, 0, st>>>(a);
  else if (a.M <= 80) gemm_w4_regs_kernel<MODE, CG, WB, 5><<<grid, 128 * CG, 0, st>>>(a);
  else if (a.M <= 112) gemm_w4_regs_kernel<MODE, CG, WB, 7><<<grid, 128 * CG, 0, st>>>(a);
  else gemm_w4_regs_kernel<MODE, CG, WB, 8><<<grid, 128 * CG, 0, st>>>(a);
}
template <int MODE>
void launch_form(const W4RegArgs& a, int columns, dim3 grid, hipStream_t st) {
  if (columns == 128) launch_rows<MODE, 4, 2>(a, grid, st);
  else if (columns == 96) launch_rows<MODE, 6, 1>(a, grid, st);
  else launch_rows<MODE, 4, 1>(a, grid, st);
}

// Columns per workgroup and cut of K, one workgroup to a compute unit, parts of at least 3 slabs.  The figures are fitted to
// 1600 launches of 12 shapes (2048 to 57344 columns, K of 2048 to 28672) at 1 to 128 rows, weights from memory: a slab's
// time grows with columns, rows and both; a cut costs what the last arriver does, at 96 columns with its twelve waves 0.4 us
// more a part (without that 11264 x 2048 at 128 rows took 22.8 us cut in two for 19.2 with 64 columns uncut).  Within 0.4 % of the best launch on average, 5 % at worst, over 17 shapes at six row counts.
struct W4Plan {
  int columns, split;
};
W4Plan plan_w4(int M, int N, int K, bool have_ws, size_t split_ws_bytes) {
  const int cus = sx_compute_units(), nb = K / BK;
  const int rb = M <= 16 ? 1 : M <= 32 ? 2 : M <= 64 ? 4 : M <= 80 ? 5 : M <= 112 ? 7 : 8;
  W4Plan p = {64, 1};
  float best = 1e30f;
  for (int bn = 128; bn >= 64; bn -= 32) {
    const int tiles = (N + bn - 1) / bn;
    const float c = bn / 128.f, r = rb / 8.f, slab = 0.045f + 0.531f * c + 0.316f * r + 0.331f * c * r;
    for (int split = 1; split <= 16; ++split) {
      const size_t part = split > 1 ? (size_t)split * rb * 16 * bn * sizeof(float) : 0;  // bytes per tile
      if (split > 1 && (!have_ws || tiles > 256 || tiles * split > cus || nb / split < 3 || split_ws_bytes < 1024 + tiles * part))
        break;
      const int rounds = (tiles * split + cus - 1) / cus;
      const float cost = rounds * (0.42f + (nb + split - 1) / split * slab) +
                         (split > 1 ? 1.8f + (bn == 96 ? 0.75f : 0.33f) * split + 1.8e-5f * (float)part : 0.f);
      if (cost < best) best = cost, p = {bn, split};
    }
  }
  return p;
}

// Stacked 4-bit matrices (n1, n2 may be 0; every non-final segment a multiple of 64 rows), M <= 128, K a multiple of 128,
// group a power of two >= 64 dividing K.  Y fp32 [M][ldy] (ldy >= n0 + n1 + n2), mode store or residual.
// split_ws: 1 KB of counters (zero before the first launch; the kernel leaves them zero) followed by room for the
// partial sums; null = no K split.  Returns SX_ERR_SHAPE for shapes outside this form (the caller then takes the
// LDS-dequantising kernel).
int launch_w4(W4RegArgs& a, const void* X, const sx_w4_matrix* mats, const int* ns, int n_mats, int group, float* Y, int ldy,
              int M, int K, int mode, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || M > 128 || K < BK || K % BK != 0 || n_mats < 1 || n_mats > 3) return SX_ERR_SHAPE;
  if (group < 64 || (group & (group - 1)) != 0 || K % group != 0) return SX_ERR_SHAPE;
  int N = 0;
  for (int i = 0; i < 3; ++i) {
    const int n = i < n_mats ? ns[i] : 0;
    if (i < n_mats && (n < 1 || !mats[i].qweight || !mats[i].scales || !mats[i].zeros)) return SX_ERR_SHAPE;
    if (i + 1 < n_mats && n % 64 != 0) return SX_ERR_SHAPE;
    if (!sx_operand_fits_u32(n, K / 2)) return SX_ERR_SHAPE;
    const sx_w4_matrix& src = mats[i < n_mats ? i : 0];
    a.m[i].q = static_cast<const uint32_t*>(src.qweight);
    a.m[i].s = static_cast<const unsigned short*>(src.scales);
    a.m[i].z = static_cast<const unsigned char*>(src.zeros);
    N += n;
  }
  if (!sx_operand_fits_u32(M, 2ll * K) || ldy < N) return SX_ERR_SHAPE;
  a.X = static_cast<const unsigned short*>(X);
  a.n0 = ns[0];
  a.n1 = n_mats > 1 ? ns[1] : 0;
  a.n2 = n_mats > 2 ? ns[2] : 0;
  a.group_log2 = __builtin_ctz((unsigned)group);
  a.Y = Y;
  a.ldy = ldy;
  a.M = M;
  a.N = N;
  a.K = K;
  const W4Plan p = plan_w4(M, N, K, split_ws != nullptr, split_ws_bytes);
  const int columns = p.columns;
  a.split = p.split;
  a.part = nullptr;
  a.part_cnt = nullptr;
  const dim3 grid((N + columns - 1) / columns, a.split);
  if (a.split > 1) {
    a.part_cnt = static_cast<int*>(split_ws);
    a.part = reinterpret_cast<float*>(static_cast<char*>(split_ws) + 1024);
  }
  switch (mode) {
    case SX_GEMM_STORE: launch_form<SX_GEMM_STORE>(a, columns, grid, st); break;
    case SX_GEMM_RESIDUAL: launch_form<SX_GEMM_RESIDUAL>(a, columns, grid, st); break;
    case SX_GEMM_SWIGLU: launch_form<SX_GEMM_SWIGLU>(a, columns, grid, st); break;
    case SX_GEMM_QKV_ROPE: launch_form<SX_GEMM_QKV_ROPE>(a, columns, grid, st); break;
  }
  SX_LAUNCH_CHECK();
  return SX_OK;
}

}  // namespace

int sx_launch_gemm_w4_regs(const void* X, const sx_w4_matrix* mats, const int* ns, int n_mats, int group, float* Y, int ldy,
                           int M, int K, int mode, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (mode != SX_GEMM_STORE && mode != SX_GEMM_RESIDUAL) return SX_ERR_SHAPE;
  W4RegArgs a = {};
  return launch_w4(a, X, mats, ns, n_mats, group, Y, ldy, M, K, mode, split_ws, split_ws_bytes, st);
}

// gate | up: act bf16 [M][F] = silu(X Wg^T) * (X Wu^T), F a multiple of 64.  The products stay in registers: through
// memory in fp32 the SwiGLU was a launch of its own, 4.2 us and a gap; with it and the rotation in the epilogues a forward of
// two 7B-shaped layers over 100 rows takes 352 us, 373 before.
int sx_launch_gemm_w4_swiglu(const void* X, const sx_w4_matrix* gate_up, int F, int group, void* act, int M, int K,
                             void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (F < 1 || F % 64 != 0) return SX_ERR_SHAPE;
  const int ns[2] = {F, F};
  W4RegArgs a = {};
  return launch_w4(a, X, gate_up, ns, 2, group, static_cast<float*>(act), 2 * F, M, K, SX_GEMM_SWIGLU, split_ws, split_ws_bytes,
                   st);
}

// q | k | v, rotated and split into heads of 128: sx_launch_gemm_qkv_rope_bf16 with 4-bit matrices, M <= 128
int sx_launch_gemm_w4_qkv_rope(const void* X, const sx_w4_matrix* qkv, int hq, int hkv, int group, const float2* rope_cs, void* q,
                               void* k, void* v, int M, int K, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (hq < 1 || hkv < 1) return SX_ERR_SHAPE;
  const int ns[3] = {hq * 128, hkv * 128, hkv * 128};
  W4RegArgs a = {};
  a.cs = rope_cs;
  a.q = static_cast<unsigned short*>(q);
  a.k = static_cast<unsigned short*>(k);
  a.v = static_cast<unsigned short*>(v);
  return launch_w4(a, X, qkv, ns, 3, group, nullptr, ns[0] + ns[1] + ns[2], M, K, SX_GEMM_QKV_ROPE, split_ws, split_ws_bytes, st);
}

extern "C" int sx_gemm_w4a16_plan(int32_t M, int32_t N, int32_t K, size_t workspace_bytes, int32_t* tile_columns, int32_t* k_parts) {
  if (!tile_columns || !k_parts) return SX_ERR_NULL;
  if (M < 1 || M > 128 || N < 1 || K < BK || K % BK != 0) return SX_ERR_SHAPE;
  const W4Plan p = plan_w4(M, N, K, workspace_bytes != 0, workspace_bytes);
  *tile_columns = p.columns;
  *k_parts = p.split;
  return SX_OK;
}
