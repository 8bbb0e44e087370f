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
// Tiling: a workgroup owns all M <= 128 rows x 128 or 64 columns.  K is walked in slabs of 128 (four k-steps), and its
// eight waves are four column groups (2 or 1 blocks of 16 W rows each, x 8 blocks of 16 X rows) times the two halves of
// every slab's k-steps, whose sums meet in LDS at the end: two waves per SIMD without a second copy of X or a second
// partial tile.  The contraction index may be permuted as long as both operands agree: in k-step s of a slab a
// lane of quarter lq takes the 16-byte chunk 4 lq + s of its row, so its two fragments of the slab are one
// contiguous 8-byte load (64 contiguous bytes per W row).
// What bounds it: not HBM (23 MB in 31 us) but a compute unit's own slab, 1.35 us for 128 columns whether 32 or 172
// workgroups run: X copied into LDS and read by every wave, the dequantisation, 64 MFMAs per SIMD.  So: X three slabs
// ahead in four stages (a barrier waits only for its own slab's operations, by count); scales and zero points of up
// to 48 groups fetched into LDS at a time, side by side, instead of two loads per lane, block and slab that each touch
// 16 lines; the words of two slabs, which share their lines, fetched together.  Measured at 128 rows, before (4 waves, two
// stages, loads of scales per slab) -> with eight waves and four stages -> now, 4096 x 4096: 28.4 -> 22.0 -> 19.0 us;
// 4096 x 11008: 44.4 -> 34.7 -> 31.3; 12288 x 4096: 33.0 -> 42.1 -> 31.3; 22016 x 4096: 52.3 -> 64.4 -> 45.6; 10240 x
// 8192: 49.8 -> 51.9 -> 40.2; 8192 x 28672: 95 -> 124 -> 89.  (The two k-steps software-pipelined by hand with the
// MFMAs, reads and dequantisation dealt out evenly, and codes made floats by their exponent bits instead of
// conversions, were measured: within 2 % either way.)
// Where column tiles are fewer than compute units the K range is cut among workgroups (grid.y); partial sums meet in
// memory and the last workgroup to arrive adds them in part order (deterministic, nobody waits).
//
// Up to three weight matrices may be stacked along N (the QKV projections, or gate and up) as long as each
// holds a multiple of 64 rows: a block of 16 columns then belongs to one matrix.
#include "kernels.h"

namespace {

constexpr int BM = 128, BK = 128;   // rows, K of a slab; columns: 4 groups x WB blocks of 16 (template parameter)
constexpr int kThreads = 512;
constexpr int kXBytes = BM * BK * 2;   // 32 KB: one slab of X
constexpr int kParGroups = 48;         // groups whose scales and zero points are in LDS at a time

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
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00020000);
}
__device__ __forceinline__ unsigned cvt_pk_bf16(float lo, float hi) {  // one v_cvt_pk_bf16_f32
  f32x2 t = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(t, bf16x2));
}

// eight codes of one word -> eight bf16 in k order; sc = scale, nzs = -zero * scale (both exact in fp32, and so is
// code * sc + nzs = sc * (code - zero): 8 significant bits times at most 4)
__device__ __forceinline__ bf16x8 dequant8(uint32_t q, float sc, float nzs) {
  const uint32_t lo = q & 0x0F0F0F0Fu, hi = (q >> 4) & 0x0F0F0F0Fu;  // codes 0,2,4,6 and 1,3,5,7, one per byte
  u32x4 o;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float e = fmaf((float)((lo >> (8 * b)) & 0xFFu), sc, nzs);
    const float f = fmaf((float)((hi >> (8 * b)) & 0xFFu), sc, nzs);
    o[b] = cvt_pk_bf16(e, f);
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

template <int MODE, int WB>
__global__ __launch_bounds__(kThreads) void gemm_w4_regs_kernel(W4RegArgs a) {
  constexpr int BN = 64 * WB;             // columns of the workgroup
  constexpr int kPartFloats = BM * BN;    // partial sums of one K part of one tile
  // X slab: row r is 256 bytes at r * 256, its 16-byte chunk c at position c ^ (r & 15): the 16 rows a fragment
  // read touches for one chunk index fall on 16 different bank groups.  Four stages.
  __shared__ __attribute__((aligned(1024))) unsigned char sx0[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx1[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx2[kXBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char sx3[kXBytes];
  __shared__ unsigned s_par[kParGroups * BN];  // [group][column]: the scale's bits, above the zero point
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int wc = wave & 3, half = wave >> 2;  // columns; k-steps 2 half and 2 half + 1 of every slab
  // Where columns go in pairs (gate and up, the two halves of a head), the tile's blocks of 16 alternate between the first
  // and the second of them.
  constexpr bool kPairs = MODE == SX_GEMM_SWIGLU || MODE == SX_GEMM_QKV_ROPE;
  auto stacked_row = [&](int col) {  // column of the tile -> row of the stacked matrices, for pairs
    const int p = blockIdx.x * (BN / 2) + (col >> 5) * 16 + (col & 15), second = (col >> 4) & 1;
    return MODE == SX_GEMM_SWIGLU ? p + (second ? a.n0 : 0) : (p >> 6) * 128 + second * 64 + (p & 63);
  };
  const int tile_n = blockIdx.x, kpart = blockIdx.y;

  // ---- X copies: instruction t (0..3) of wave w fills rows 16 w + 4 t .. + 3 (1 KB of LDS): lane l supplies row
  // + l / 16, position l % 16, i.e. chunk (l % 16) ^ (row & 15) of that row's 256 bytes of the slab
  const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.X);
  int xoff[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = 16 * wave + 4 * t + (lane >> 4);
    const int c = (lane & 15) ^ (r & 15);
    const int m = r < a.M ? r : a.M - 1;
    xoff[t] = (int)(((unsigned)m * (unsigned)a.K + c * 8) * 2u);
  }
#define SX_COPY(STG_, SLAB_)                                                                                     \
  {                                                                                                              \
    const int so = (SLAB_) * (BK * 2);                                                                           \
    _Pragma("unroll") for (int t = 0; t < 4; ++t) __builtin_amdgcn_raw_ptr_buffer_load_lds(                      \
        xres, (lds_void_ptr)(STG_ + wave * 4096 + t * 1024), 16, xoff[t], so, 0, 0);                             \
  }

  // ---- W: a block of 16 columns belongs to one of the stacked matrices ------------------------------------------
  const int c0 = tile_n * BN + 16 * WB * wc;  // first column of the wave (uniform)
  const bool wave_has_cols = c0 < a.N;
  const int ngroups = a.K >> a.group_log2;
  int qoff[WB];
  __amdgpu_buffer_rsrc_t qres[WB];
#pragma unroll
  for (int i = 0; i < WB; ++i) {
    const int b0 = kPairs ? stacked_row(16 * (WB * wc + i)) : c0;
    const int which = b0 >= a.n0 + a.n1 ? 2 : b0 >= a.n0 ? 1 : 0;
    const int first = which == 2 ? a.n0 + a.n1 : which == 1 ? a.n0 : 0;
    const int rows = which == 2 ? a.n2 : which == 1 ? a.n1 : a.n0;
    int n = b0 - first + (kPairs ? 0 : 16 * i) + l16;  // row of the matrix; columns past the end re-read the last row
    n = n < rows ? n : rows - 1;
    n = n < 0 ? 0 : n;
    qoff[i] = (int)(((unsigned)n * (unsigned)(a.K / 8) + 4u * lq + 2u * half) * 4u);   // + 64 bytes per slab
    qres[i] = make_rsrc(which == 2 ? a.m[2].q : which == 1 ? a.m[1].q : a.m[0].q);
  }
  struct WRaw {
    u32x2 q[2];
  };
  // the words of slabs A_ and B_, which share their 128-byte lines
#define SX_LOAD_W2(WA_, WB_, A_, B_)                                                                             \
  _Pragma("unroll") for (int i = 0; i < WB; ++i) {                                                               \
    WA_.q[i] = __builtin_amdgcn_raw_buffer_load_b64(qres[i], qoff[i], (A_) * 64, 0);                              \
    WB_.q[i] = __builtin_amdgcn_raw_buffer_load_b64(qres[i], qoff[i], (B_) * 64, 0);                              \
  }
  // Scales and zero points of the slabs [S0_, S1_) into LDS; par0 becomes the first of their groups.  A thread takes
  // four (column, group) pairs at a time, the groups of a column side by side in memory.
#define SX_FILL(S0_, S1_)                                                                                        \
  {                                                                                                              \
    par0 = ((S0_) * BK) >> a.group_log2;                                                                         \
    const int ng = (((S1_) * BK - 1) >> a.group_log2) - par0 + 1, total = ng * BN;                               \
    for (int b = 0; b < total; b += 4 * kThreads) {                                                              \
      unsigned ps[4], pz[4];                                                                                     \
      int at[4];                                                                                                 \
      _Pragma("unroll") for (int u = 0; u < 4; ++u) {                                                            \
        const int idx = min(b + u * kThreads + tid, total - 1);                                                  \
        const int col = idx / ng, g = idx - col * ng;                                                            \
        int n = kPairs ? stacked_row(col) : min(tile_n * BN + col, a.N - 1);                                     \
        const int wm = n >= a.n0 + a.n1 ? 2 : n >= a.n0 ? 1 : 0;                                                 \
        n -= wm == 2 ? a.n0 + a.n1 : wm == 1 ? a.n0 : 0;                                                         \
        const size_t e = (size_t)n * ngroups + par0 + g;                                                         \
        ps[u] = (wm == 2 ? a.m[2].s : wm == 1 ? a.m[1].s : a.m[0].s)[e];                                         \
        pz[u] = (wm == 2 ? a.m[2].z : wm == 1 ? a.m[1].z : a.m[0].z)[e];                                         \
        at[u] = g * BN + col;                                                                                    \
      }                                                                                                          \
      _Pragma("unroll") for (int u = 0; u < 4; ++u) s_par[at[u]] = ps[u] << 16 | pz[u];                          \
    }                                                                                                            \
  }

  // acc[i][j]: W rows (output columns) c0 + 16 i .. + 15, X rows (output rows) 16 j .. + 15
  f32x4 acc[WB][8];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // X fragment of block j in k-step s: row 16 j + l16, chunk 4 lq + s, at position chunk ^ (row & 15) = chunk ^ l16
  const int xrow = l16 * (BK * 2);
#define SX_SLAB(XS_, W_, T_)                                                                                     \
  {                                                                                                              \
    /* group of this lane's k range, k = 128 slab + 32 lq + (0..31) (groups are powers of two >= 64) */          \
    const int g = (((first_slab + (T_)) * BK + 32 * lq) >> a.group_log2) - par0;                                 \
    float sc[WB], nzs[WB];                                                                                       \
    _Pragma("unroll") for (int i = 0; i < WB; ++i) {                                                             \
      const unsigned pr = s_par[g * BN + 16 * WB * wc + 16 * i + l16];                                           \
      sc[i] = __uint_as_float(pr & 0xFFFF0000u);                                                                 \
      nzs[i] = -(float)(pr & 0xFFu) * sc[i];                                                                     \
    }                                                                                                            \
    _Pragma("unroll") for (int s = 0; s < 2; ++s) {                                                              \
      bf16x8 fw[WB], fx[8];                                                                                      \
      const int xc = xrow + (((4 * lq + 2 * half + s) ^ l16) << 4);                                              \
      _Pragma("unroll") for (int j = 0; j < 8; ++j)                                                              \
          fx[j] = *reinterpret_cast<const bf16x8*>(XS_ + j * (16 * BK * 2) + xc);                                \
      _Pragma("unroll") for (int i = 0; i < WB; ++i) fw[i] = dequant8(W_.q[i][s], sc[i], nzs[i]);                \
      _Pragma("unroll") for (int i = 0; i < WB; ++i) _Pragma("unroll") for (int j = 0; j < 8; ++j)               \
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[i], fx[j], acc[i][j], 0, 0, 0);                 \
    }                                                                                                            \
  }

  // Slabs [first_slab, first_slab + NB) of K; slab t sits in stage t % 4 and its W words in register set t % 4.  Per
  // slab: wait for its own copies and words (the two younger slabs' copies and the younger pair of words stay in
  // flight) and for everybody to be done with the slab before it, start the copies of slab t + 3 into that stage,
  // multiply; after every second slab fetch the words of slabs t + 3 and t + 4 together.  Past the end of K the last
  // slab is fetched again.
  constexpr int kFly = 8 + 2 * WB;  // two slabs' copies, one pair's words
#define SX_SLAB_AT(i) (first_slab + min((i), NB - 1))
#define SX_STEP(XS_, W_, XN_, T_)                                                                                \
  SX_WAIT_BARRIER(wait_vm(kFly))                                                                                 \
  SX_COPY(XN_, SX_SLAB_AT((T_) + 3))                                                                             \
  asm volatile("" ::: "memory");                                                                                 \
  SX_SLAB(XS_, W_, T_)
#define SX_PAIR(WA_, WB_, T_)                                                                                    \
  asm volatile("" ::: "memory");                                                                                 \
  SX_LOAD_W2(WA_, WB_, SX_SLAB_AT(T_), SX_SLAB_AT((T_) + 1))                                                     \
  asm volatile("" ::: "memory");
  const int nb_all = a.K / BK;
  const int first_slab = kpart * nb_all / a.split;
  const int NB = (kpart + 1) * nb_all / a.split - first_slab;
  const int par_slabs = a.group_log2 > 6 ? kParGroups : kParGroups / 2;  // slabs whose groups fit s_par
  int par0;
  WRaw w0, w1, w2, w3;
  SX_COPY(sx0, first_slab)
  SX_PAIR(w0, w1, 0)
  SX_COPY(sx1, SX_SLAB_AT(1))
  asm volatile("" ::: "memory");  // (the waits count operations: in this order)
  SX_COPY(sx2, SX_SLAB_AT(2))
  SX_PAIR(w2, w3, 2)
  SX_FILL(first_slab, first_slab + min(NB, par_slabs))
  int t = 0, refill = par_slabs;
  for (; t + 4 <= NB; t += 4) {
    if (t == refill) {  // everybody is done with the last groups' parameters; the next barrier shows the new ones
      __syncthreads();
      SX_FILL(first_slab + t, first_slab + min(NB, t + par_slabs))
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
      SX_FILL(first_slab + t, first_slab + NB)
    }
    SX_WAIT_BARRIER(wait_vm(kFly))
    SX_SLAB(sx0, w0, t)
    if (t + 1 < NB) {
      SX_WAIT_BARRIER(wait_vm(4 + 2 * WB))
      SX_SLAB(sx1, w1, t + 1)
    }
    if (t + 2 < NB) {
      SX_WAIT_BARRIER(wait_vm(0))
      SX_SLAB(sx2, w2, t + 2)
    }
  }
  SX_WAIT_BARRIER(wait_vm(0))  // every copy is in and every stage is read: the LDS is free
#undef SX_STEP
#undef SX_PAIR
#undef SX_SLAB_AT
#undef SX_SLAB
#undef SX_FILL
#undef SX_LOAD_W2
#undef SX_COPY

  // ---- the two halves of the k-steps: the upper half's waves leave their sums in LDS, the lower half's add them ----
  {
    unsigned char* ob = (WB == 2 && (wc & 2) ? sx1 : sx0) + (WB == 2 ? wc & 1 : wc) * (8192 * WB) + lane * 16;
    if (half == 1) {
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) *reinterpret_cast<f32x4*>(ob + (i * 8 + j) * 1024) = acc[i][j];
    }
    __syncthreads();
    if (half == 0) {
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] += *reinterpret_cast<const f32x4*>(ob + (i * 8 + j) * 1024);
    }
  }

  // ---- K split: partial sums meet in memory, the last workgroup to arrive adds them in part order -------------
  // (device-scope stores and loads, stores complete before the counter's device-scope atomic is issued)
  if (a.split > 1) {
    constexpr int kScopeDevice = 16;
    __shared__ int s_last;
    const __amdgpu_buffer_rsrc_t pres = make_rsrc(a.part);
    const unsigned mine =
        (unsigned)((tile_n * a.split + kpart) * kPartFloats + wc * (8 * WB * 256) + lane * 4) * 4u;  // bytes
    if (half == 0) {
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), pres, mine + (i * 8 + j) * 1024, 0,
                                                 kScopeDevice);
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
    // batches of 8 blocks per part, all loads of a batch in flight together (one memory round trip per batch
    // and part, not one per block); parts are added in part order, this workgroup's own out of its registers
    const unsigned all = (unsigned)(tile_n * a.split * kPartFloats + wc * (8 * WB * 256) + lane * 4) * 4u;
    if (half == 0) {
#pragma unroll
      for (int i = 0; i < WB; ++i) {
        f32x4 sum[8];
        for (int p = 0; p < a.split; ++p) {
          f32x4 part[8];
          if (p == kpart) {
#pragma unroll
            for (int j = 0; j < 8; ++j) part[j] = acc[i][j];
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              part[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                      pres, all + (unsigned)p * (kPartFloats * 4u) + (i * 8 + j) * 1024, 0,
                                                      kScopeDevice));
          }
#pragma unroll
          for (int j = 0; j < 8; ++j) sum[j] = p == 0 ? part[j] : sum[j] + part[j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = sum[j];
      }
    }
  }

  // ---- epilogue of pairs: the first of them in lo, the second in hi, 4 consecutive ones of row 16 (j0 + j) + l16 -----
  if constexpr (kPairs) {
    constexpr int NJ = WB == 2 ? 8 : 4;
    f32x4 lo[NJ], hi[NJ];
    if constexpr (WB == 2) {
      if (half == 1) return;
#pragma unroll
      for (int j = 0; j < 8; ++j) lo[j] = acc[0][j], hi[j] = acc[1][j];
    } else {
      // one block per wave: the wave of the firsts keeps rows 0 .. 63 and hands on the others, that of the seconds the
      // other way round, through a stage the sums above do not use
      unsigned char* xb = sx2 + lane * 16;
      const bool second = wc & 1;  // (branches, not selections: those put the accumulators into scratch memory)
      if (half == 0 && second) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4*>(xb + (wc * 4 + j) * 1024) = acc[0][j];
      } else if (half == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4*>(xb + (wc * 4 + j) * 1024) = acc[0][j + 4];
      }
      __syncthreads();
      if (half == 1) return;
      if (second) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lo[j] = *reinterpret_cast<const f32x4*>(xb + ((wc - 1) * 4 + j) * 1024);
          hi[j] = acc[0][j + 4];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lo[j] = acc[0][j];
          hi[j] = *reinterpret_cast<const f32x4*>(xb + ((wc + 1) * 4 + j) * 1024);
        }
      }
    }
    const int row0 = (WB == 1 && (wc & 1) ? 64 : 0) + l16;
    const int p = tile_n * (BN / 2) + (WB == 2 ? wc : wc >> 1) * 16 + 4 * lq;
    if constexpr (MODE == SX_GEMM_SWIGLU) {
      unsigned short* Y = reinterpret_cast<unsigned short*>(a.Y) + p;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int m = row0 + 16 * j;
        if (m >= a.M) continue;
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_mul_bf16_bound(lo[j][e], hi[j][e]);
        u32x2 o;
        o[0] = pack_bf16x2(h[0], h[1]);
        o[1] = pack_bf16x2(h[2], h[3]);
        *reinterpret_cast<u32x2*>(Y + (size_t)m * a.n0) = o;
      }
    } else {
      const int head = p >> 6, w = p & 63, hq = a.n0 >> 7, hkv = a.n1 >> 7;
      const bool is_v = head >= hq + hkv;
      const int nheads = head < hq ? hq : hkv, first = is_v ? hq + hkv : head >= hq ? hq : 0;
      unsigned short* Y = (head < hq ? a.q : is_v ? a.v : a.k) + (size_t)(head - first) * 128 + w;
      f32x4 t[NJ][2];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const f32x4* c = reinterpret_cast<const f32x4*>(a.cs + (size_t)min(row0 + 16 * j, a.M - 1) * 64 + w);
        t[j][0] = c[0];
        t[j][1] = c[1];
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int m = row0 + 16 * j;
        if (m >= a.M) continue;
        float x[4], y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x0 = lo[j][e], x1 = hi[j][e];
          const float c = t[j][e >> 1][2 * (e & 1)], s = t[j][e >> 1][2 * (e & 1) + 1];
          rope_turn(x0, x1, c, s, x[e], y[e]);
          if (is_v) x[e] = x0, y[e] = x1;
        }
        unsigned short* to = Y + (size_t)m * nheads * 128;
        u32x2 o;
        o[0] = pack_bf16x2(x[0], x[1]);
        o[1] = pack_bf16x2(x[2], x[3]);
        *reinterpret_cast<u32x2*>(to) = o;
        o[0] = pack_bf16x2(y[0], y[1]);
        o[1] = pack_bf16x2(y[2], y[3]);
        *reinterpret_cast<u32x2*>(to + 64) = o;
      }
    }
    return;
  }
  if (half == 1) return;

  // ---- epilogue.  acc[i][j][e]: output row 16 j + l16, column c0 + 16 i + 4 lq + e --------------------------------
  if (!wave_has_cols) return;
  const bool vec = (a.N & 3) == 0 && (a.ldy & 3) == 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int m = 16 * j + l16;
#pragma unroll
    for (int i = 0; i < WB; ++i) {
      const int n = c0 + 16 * i + 4 * lq;
      if (m >= a.M || n >= a.N) continue;
      float* y = a.Y + (size_t)m * a.ldy + n;
      if (vec) {
        f32x4 v = acc[i][j];
        if (MODE == SX_GEMM_RESIDUAL) v += *reinterpret_cast<const f32x4*>(y);
        *reinterpret_cast<f32x4*>(y) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < a.N) {
            if (MODE == SX_GEMM_RESIDUAL) y[e] += acc[i][j][e];
            else y[e] = acc[i][j][e];
          }
      }
    }
  }
}
#undef SX_WAIT_BARRIER

// Stacked 4-bit matrices (n1, n2 may be 0; every non-final segment a multiple of 64 rows), M <= 128, K a multiple of 128,
// group a power of two >= 64 dividing K.  Y fp32 [M][ldy] (ldy >= n0 + n1 + n2), mode store or residual.
// split_ws: 1 KB of counters (zero before the first launch; the kernel leaves them zero) followed by room for the
// partial sums; null = no K split.  Returns SX_ERR_SHAPE for shapes outside this form (the caller then takes the
// LDS-dequantising kernel).
int launch_w4(W4RegArgs& a, const void* X, const sx_w4_matrix* mats, const int* ns, int n_mats, int group, float* Y, int ldy,
              int M, int K, int mode, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || M > BM || K < BK || K % BK != 0 || n_mats < 1 || n_mats > 3) return SX_ERR_SHAPE;
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
  // Columns per workgroup and K cut, by expected slab times of the 128-column form (1.35 us): a 64-column slab costs
  // 0.63, and every part's partial tile, written and read back by the last arriver, 1.25 per 64 columns.  One workgroup
  // fits a compute unit; parts of at least 4 slabs.  (4096 x 4096: 64 columns cut 4 ways 19.0 us, uncut 29.7, 128
  // columns cut 4 ways 24.8; 8192 x 28672: 128 columns cut 4 ways 89, 64 cut 2 ways 102.)
  const int cus = sx_compute_units(), nb = K / BK;
  a.part = nullptr;
  a.part_cnt = nullptr;
  int wb = 2;
  float best = 1e30f;
  for (int w = 1; w <= 2; ++w) {
    const int tiles = (N + 64 * w - 1) / (64 * w);
    for (int sp = 1; sp <= 16; ++sp) {
      if (sp > 1 && (!split_ws || tiles > 256 || tiles * sp > cus || nb / sp < 4 ||
                     split_ws_bytes < 1024 + (size_t)tiles * sp * BM * 64 * w * sizeof(float)))
        break;
      const float cost = (float)((tiles * sp + cus - 1) / cus) * ((nb + sp - 1) / sp) * (w == 1 ? 0.63f : 1.f) +
                         (sp > 1 ? 1.25f * w * sp : 0.f);
      if (cost < best) best = cost, wb = w, a.split = sp;
    }
  }
  const dim3 grid((N + 64 * wb - 1) / (64 * wb), a.split);
  if (a.split > 1) {
    a.part_cnt = static_cast<int*>(split_ws);
    a.part = reinterpret_cast<float*>(static_cast<char*>(split_ws) + 1024);
  }
#define SX_GO(MODE_)                                                            \
  if (wb == 1) gemm_w4_regs_kernel<MODE_, 1><<<grid, kThreads, 0, st>>>(a);     \
  else gemm_w4_regs_kernel<MODE_, 2><<<grid, kThreads, 0, st>>>(a);
  switch (mode) {
    case SX_GEMM_STORE: SX_GO(SX_GEMM_STORE) break;
    case SX_GEMM_RESIDUAL: SX_GO(SX_GEMM_RESIDUAL) break;
    case SX_GEMM_SWIGLU: SX_GO(SX_GEMM_SWIGLU) break;
    case SX_GEMM_QKV_ROPE: SX_GO(SX_GEMM_QKV_ROPE) break;
  }
#undef SX_GO
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
