// Y = X W^T on the gfx950 matrix cores: the linear layers of the decoder forward (Alg. 1, FORWARD) at
// M = number of tree tokens.  bf16 operands, fp32 accumulation.
//
// Tiling.  A workgroup of 4 waves (2 x 2) owns a 32 JB x 256 output tile; each wave a 16 JB x 128
// quadrant = JB x 8 blocks of v_mfma_f32_16x16x32_bf16, 4 * 8 * JB fp32 accumulators per lane.  The tile height is
// a template parameter, JB = 8 (256 rows) down to 4 (128): the most arithmetic per operand byte where the rows and the
// compute units come out even, lower where 256-row tiles would multiply padding or leave compute units without a tile
// (pick_plan() below has the rule and the figures).  With real
// operand data the chip is power-limited long before the MFMA issue rate is: in a pure register loop
// the 16x16x32 shape sustains ~1.95 PFLOP/s against ~1.75 for 32x32x16 (it holds a ~10% higher
// clock), which is why the smaller block is used.  The product is formed transposed (W rows feed
// the A operand, X rows the B operand), so a lane ends up with 4 consecutive output columns of one
// row: 16-byte stores.
//
// K is walked in slabs of 64 (two MFMA k-steps, 16 JB MFMAs per wave) held in LDS stages of 4 JB KB of X and 32 KB of W.
// With two stages a copy has one slab's MFMAs to arrive, 0.6 us at 160 rows, and weights from HBM take longer: a slab took
// 1.3 to 1.5 us whatever the height.  With three it has two slabs': 0.95 to 1.1 us (0.6 with the operands in L2).  Three of
// both fit the 160 KB at JB = 4 and 5.  From JB = 6 on W has three and X two (160 KB to the byte at JB = 8): X is small
// and comes from L2, it is the weights that are late.  As two stages of both, now three of W: a slab of 192 rows 1.40 -> 1.04 us, of 224 1.48 -> 1.16
// and of 256 1.50 -> 1.30; 70B gate|up at 512 rows 417 -> 361 us, 7B gate|up at 396 rows 99 -> 74, 32000 columns, K = 4096,
// at 337 rows 109 -> 84; 850 products of the 1B to 70B shapes at 129 to 2400 rows take 0.95 of the time on average.
//
// Global -> LDS without registers.  Operand slabs are copied by buffer loads that write LDS
// directly (16 bytes per lane, a wave fills 1 KB of consecutive LDS per instruction), so the K loop
// spends no vector registers and no LDS-write instructions on staging.  Both operands are
// K-contiguous in memory, which is the per-lane layout the MFMA wants (8 consecutive k per lane),
// so an LDS row is a plain 128-byte row segment; the XOR swizzle of its 16-byte chunks that makes
// fragment reads conflict-free on the 64-bank LDS is applied on the global side (each lane picks
// the chunk whose swizzled position is the lane's slot in the wave's 1 KB).  Eight lanes fetch
// one whole 128-byte line.  That matters: the copy stream of this kernel alone (no math) runs at
// 17 TB/s L2 -> LDS with whole-line requests and at 11.5 TB/s with half-line ones, which would make
// the copies, not the MFMAs, the bound.  Whole lines are why a stage holds 64 K-elements.
// Each stage of each operand is its own __shared__ array: the compiler tracks outstanding loads-to-LDS per array,
// so a fragment read of one stage does not wait for the copies in flight to the other.
//
// Schedule of a slab, with two stages (S, the other S'; with three a copy may take a slab longer): phase 1 runs the MFMAs of k-step 0 and reads the
// fragments of k-step 1; then one barrier, before which every wave waits for its own copies of the
// next slab (now S' is complete and S is read out); phase 2 runs the MFMAs of k-step 1, starts the
// copies of the slab after next into S and reads the next slab's k-step 0 from S'.  One barrier
// per 16 JB MFMAs; a copy has about a slab's worth of MFMAs to arrive.  Copies and fragment reads
// are dealt out evenly between the MFMAs: bursts of copies fill the memory pipeline's queues and
// stall the wave that issues them.
//
// XCD-aware tile order.  Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.
// Tile index = xcd * chunk + id / 8 with tiles ordered M-fastest, so the workgroups resident on
// one XCD at a time share the same few W column tiles (fetched from HBM once per XCD) and sweep
// all of X's row tiles.
//
// Epilogues: store fp32, add into an fp32 residual, or SwiGLU.  For SwiGLU the W slab interleaves
// 16-row groups of W_gate and W_up, so gate and up of one output column sit in the same lane and
// register of neighbouring accumulator blocks and silu(g)*u needs no data movement.
#include "kernels.h"

namespace {

constexpr int BN = 256;                   // tile columns; tile rows are 32 JB
constexpr int BK = 64;                    // K elements per LDS stage ("slab"): two MFMA k-steps, whole 128-byte lines
constexpr int kThreads = 256;
constexpr int kWBytes = BN * BK * 2;                  // 32 KB: W's part of a slab
constexpr int kPfDist = 3;                            // slabs between an L2 prefetch and the copy of the same lines

constexpr int kLds = 160 * 1024;
// LDS stages of X's and of W's slabs of a tile of 32 jb rows: three where they fit the 160 KB (jb <= 5), W's alone up to 8
constexpr int stages(int jb) { return 3 * (jb * 4096 + kWBytes) <= kLds - 2048 ? 3 : 2; }
constexpr int w_stages(int jb, bool pf) { return stages(jb) == 3 || (!pf && 2 * jb * 4096 + 3 * kWBytes <= kLds) ? 3 : 2; }

struct GemmArgs {
  const unsigned short* X;
  const unsigned short* W0;
  const unsigned short* W1;
  const unsigned short* W2;
  int n0, n1, n2;
  void* Y;
  int M, N, K;  // N = logical output columns
  int tilesM, tilesN, chunk;
  int rotate;  // the XCDs walk K from different eighths on
  // SX_GEMM_QKV_ROPE only: rotary table [M][64] (cos, sin), outputs bf16 [M][hq][128], [M][hkv][128] x 2
  const float2* cs;
  unsigned short *q, *k, *v;
  int hq, hkv;
  // K split of the tail tiles (split > 1): partial sums [tail tile][split][wave][block][lane] f32x4, counters
  float* part;
  int* part_cnt;
  int split, full_tiles, tail_items, full_per_xcd, tail_per_xcd;
};

typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Raw buffer resource over a whole matrix (no bounds: rows are clamped by the caller; < 4 GB).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00020000);
}

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]):
// all LDS reads done, at most N vector-memory operations outstanding.
constexpr int wait_vm(int n) { return 0x0070 | (n & 15) | ((n >> 4) << 14); }
constexpr int kWaitVm0 = wait_vm(0), kWaitVm2 = wait_vm(2);

// Wait until this wave's LDS reads are done and at most the given number of copies are in flight, then
// meet the other waves.  The barrier intrinsic alone does not order memory operations for the compiler,
// and a workgroup fence makes it wait for every copy in flight, so empty asm statements that claim to
// touch memory pin the LDS reads and the copies to their side of the barrier instead.
#define SX_WAIT_BARRIER(IMM)              \
  asm volatile("" ::: "memory");          \
  __builtin_amdgcn_s_waitcnt(IMM);        \
  __builtin_amdgcn_s_barrier();           \
  asm volatile("" ::: "memory");

template <int MODE, int JB, bool PF>
__global__ __launch_bounds__(kThreads) void gemm_bf16_kernel(GemmArgs a) {
#ifdef __HIP_DEVICE_COMPILE__  // the host pass has no use for the body and drops the launch stub over its asm constraints
  // One array per stage (see the header).  Row r of an operand's slab is 128 bytes at r * 128; 16-byte
  // chunk c of the row sits at position c ^ ((r >> 1) & 7).  The LDS serves 16 lanes x 16 bytes per
  // cycle (64 banks): 16 consecutive rows reading the same k chunk fall on 16 different bank groups.
  constexpr int BM = 32 * JB, kXBytes = BM * BK * 2;
  constexpr int NS = stages(JB), NW = w_stages(JB, PF), kCopies = 8 + JB;  // copies of a slab per wave
  __shared__ __attribute__((aligned(1024))) unsigned char xA[kXBytes], xB[kXBytes], wA[kWBytes], wB[kWBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char xC[NS == 3 ? kXBytes : 16], wC[NW == 3 ? kWBytes : 16];
  constexpr int kAhead = 4;
  constexpr bool TOUCH = PF && NS == 3, SHARE = PF && NS == 2;
  __shared__ __attribute__((aligned(256))) unsigned char dump[TOUCH ? 1024 : 16];  // where touched lines end up
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lq = lane >> 4;

  // ---- which tile ----------------------------------------------------------------------------
  // Without a K split: tile lin = xcd * chunk + slot.  With one (a.split > 1) the first full_per_xcd
  // slots of an XCD are whole tiles and the rest are the tail: the last few tiles, which would
  // otherwise occupy a fraction of the chip for a whole round, each cut into a.split K ranges.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int lin, kpart = 0, ksplit = 1;
  if (a.split > 1) {
    if (slot < a.full_per_xcd) {
      lin = xcd * a.full_per_xcd + slot;
      if (lin >= a.full_tiles) return;
    } else {
      const int idx = xcd * a.tail_per_xcd + (slot - a.full_per_xcd);
      if (slot - a.full_per_xcd >= a.tail_per_xcd || idx >= a.tail_items) return;
      lin = a.full_tiles + idx / a.split;
      kpart = idx % a.split;
      ksplit = a.split;
    }
  } else {
    lin = xcd * a.chunk + slot;
    if (slot >= a.chunk || lin >= a.tilesM * a.tilesN) return;
  }
  const int tile_m = lin % a.tilesM, tile_n = lin / a.tilesM;

  // ---- global sources of this lane's copies ---------------------------------------------------------
  // Copy instruction t of wave w fills rows 64 w + 8 t .. + 7 of W's slab (t < 8) or rows 8 (JB w + t) .. + 7 of X's
  // (t < JB), 1 KB of LDS: lane l supplies row .. + l / 8, LDS chunk position l % 8, i.e. k chunk
  // (l % 8) ^ ((row >> 1) & 7) with (row >> 1) & 7 = (4 t + l / 16) & 7 for W and (4 (JB w + t) + l / 16) & 7 for X.  Eight lanes read one whole
  // 128-byte line: the L2 serves whole-line requests half again as fast as half-line ones.  An 8-row
  // group never straddles two weight matrices (segment sizes are multiples of 16).
  const int crow = 64 * wave + (lane >> 3);
  const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.X);
  const __amdgpu_buffer_rsrc_t wres0 = make_rsrc(a.W0), wres1 = make_rsrc(a.W1), wres2 = make_rsrc(a.W2);
  __amdgpu_buffer_rsrc_t wres[8];
  int xoff[JB], woff[8];
#pragma unroll
  for (int t = 0; t < JB; ++t) {
    const int g = JB * wave + t;
    int m = tile_m * BM + 8 * g + (lane >> 3);
    m = m < a.M ? m : a.M - 1;
    xoff[t] = (int)(((unsigned)m * (unsigned)a.K + ((lane & 7) ^ ((4 * (g & 1) + (lane >> 4)) & 7)) * 8) * 2u);
  }
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int r = crow + 8 * t;
    const int cchunk = (lane & 7) ^ ((4 * (t & 1) + (lane >> 4)) & 7);
    if (MODE == SX_GEMM_SWIGLU) {
      // slab rows in 16-row groups: even group = gate, odd = up; rows 64 w + 8 t are in group 4 w + t / 2
      int f = tile_n * (BN / 2) + (2 * wave + (t >> 2)) * 16 + (t & 1) * 8 + (lane >> 3);
      f = f < a.N ? f : a.N - 1;
      wres[t] = (t & 2) ? wres1 : wres0;
      woff[t] = (int)(((unsigned)f * (unsigned)a.K + cchunk * 8) * 2u);
    } else {
      const int g0 = min(tile_n * BN + 64 * wave + 8 * t, a.N - 1);  // first row of the group decides the matrix
      int n = tile_n * BN + r;
      n = n < a.N ? n : a.N - 1;
      int first = 0;
      wres[t] = wres0;
      if (g0 >= a.n0 + a.n1) {
        wres[t] = wres2;
        first = a.n0 + a.n1;
      } else if (g0 >= a.n0) {
        wres[t] = wres1;
        first = a.n0;
      }
      woff[t] = (int)(((unsigned)(n - first) * (unsigned)a.K + cchunk * 8) * 2u);
    }
  }
  const int xdst = wave * (JB * 1024), wdst = wave * 8192;  // this wave's share of X's and of W's slab

  // ---- L2 prefetch (PF kernels: 8 row tiles, column tiles a multiple of 4) ---------------------------
  // The 32 workgroups that run side by side on an XCD are then 8 row tiles x 4 column tiles: an X tile
  // is read by 4 of them and a W tile by 8, at about the same time, so all of them wait for the one
  // fabric access.  Instead each touches its share of the lines (X: 64 rows = 16 per wave; W: 32 rows
  // = 8 per wave; one dword per 128-byte line) kPfDist slabs ahead, and the copies of all of them find
  // the lines in L2.  Measured at the 70B shapes: QKV +12%, gate/up +4%, down +6%, O -3%.
  int pfx = 0, pfw = 0, pfxoff = 0, pfwoff = 0;
  __amdgpu_buffer_rsrc_t pfwres = wres0;
  if (SHARE) {
    int m = tile_m * BM + 64 * (tile_n & 3) + 16 * wave + (lane & 15);
    m = m < a.M ? m : a.M - 1;
    pfxoff = (int)((unsigned)m * (unsigned)a.K * 2u);
    const int r = 32 * tile_m + 8 * wave;  // slab row of this wave's 8 W rows (uniform)
    if (MODE == SX_GEMM_SWIGLU) {
      int f = tile_n * (BN / 2) + (r >> 5) * 16 + (r & 15) + (lane & 7);
      f = f < a.N ? f : a.N - 1;
      pfwres = ((r >> 4) & 1) ? wres1 : wres0;
      pfwoff = (int)((unsigned)f * (unsigned)a.K * 2u);
    } else {
      const int g0 = min(tile_n * BN + r, a.N - 1);
      int n = min(tile_n * BN + r + (lane & 7), a.N - 1);
      int first = 0;
      if (g0 >= a.n0 + a.n1) {
        pfwres = wres2;
        first = a.n0 + a.n1;
      } else if (g0 >= a.n0) {
        pfwres = wres1;
        first = a.n0;
      }
      pfwoff = (int)((unsigned)(n - first) * (unsigned)a.K * 2u);
    }
  }

  // With three stages (TOUCH): the row tiles of a column tile, neighbours on an XCD, share its 256 W rows out among them,
  // and each touches a dword of the line of its rows kAhead slabs ahead of the copies, by a load that writes LDS nobody reads:
  // memory operations retire in order, and a load into a register would be waited for a slab later.  (Lanes whose row is
  // another tile's touch the start of W0: every wave issues the same number of operations.)
  const unsigned char* touch = reinterpret_cast<const unsigned char*>(a.W0);
  if (TOUCH) {
    const int r = 64 * wave + lane;
    if (r % a.tilesM == tile_m) {
      if (MODE == SX_GEMM_SWIGLU) {
        const int f = min(tile_n * (BN / 2) + (r >> 5) * 16 + (r & 15), a.N - 1);
        touch = reinterpret_cast<const unsigned char*>(((r >> 4) & 1) ? a.W1 : a.W0) + (size_t)f * a.K * 2;
      } else {
        int n = min(tile_n * BN + r, a.N - 1);
        const unsigned short* w = a.W0;
        if (n >= a.n0 + a.n1) w = a.W2, n -= a.n0 + a.n1;
        else if (n >= a.n0) w = a.W1, n -= a.n0;
        touch = reinterpret_cast<const unsigned char*>(w) + (size_t)n * a.K * 2;
      }
    }
  }
#define SX_TOUCH(i) \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(touch + SX_OFFSET(i)), (lds_void_ptr)(dump + wave * 256), 4, 0, 0);

  // acc[i][j]: W rows (output columns) 16 i .. + 15 of the quadrant, X rows (output rows) 16 j .. + 15
  f32x4 acc[8][JB];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // fragment addresses: row (quadrant base + 16 i + l16), k chunk 4 ks + lq at position ^ ((row >> 1) & 7)
  const int fsw = (l16 >> 1) & 7;
  const int xrow = (wm * (16 * JB) + l16) * (BK * 2);
  const int wrow = (wn * 128 + l16) * (BK * 2);
  const int kc0 = ((lq ^ fsw) << 4), kc1 = (((4 + lq) ^ fsw) << 4);
  bf16x8 fx0[JB], fw0[8], fx1[JB], fw1[8];   // k-step 0 and k-step 1 of a slab

// One copy instruction: rows 8 t .. + 7 of this wave's share of X (OP_ 0) or W (OP_ 1) at byte offset SO_
// along K into stage STG_.  The K offset travels in the scalar offset: the instruction's immediate
// offset would be added to the LDS address as well.
#define SX_COPY1(STG_, SO_, OP_, t)                                                                            \
  if (OP_)                                                                                                     \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(wres[t], (lds_void_ptr)(STG_ + wdst + (t) * 1024), 16, woff[t], SO_, 0, 0); \
  else if ((t) < JB)                                                                                           \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_void_ptr)(STG_ + xdst + (t) * 1024), 16, xoff[(t) % JB], SO_, 0, 0);
#define SX_COPY(XSTG_, WSTG_, SO_)                                                                            \
  _Pragma("unroll") for (int t = 0; t < 8; ++t) {                                                             \
    SX_COPY1(XSTG_, SO_, 0, t)                                                                                 \
    SX_COPY1(WSTG_, SO_, 1, t)                                                                                 \
  }
#define SX_READW(STG_, FW, i, KC) FW[i] = *reinterpret_cast<const bf16x8*>(STG_ + wrow + (i) * (16 * BK * 2) + KC);
#define SX_READX(STG_, FX, i, KC) if ((i) < JB) FX[(i) % JB] = *reinterpret_cast<const bf16x8*>(STG_ + xrow + (i) * (16 * BK * 2) + KC);
// The MFMA is written out: left to itself the compiler gives an accumulator that is updated more than
// once per loop body a new destination register each time and shuffles hundreds of registers per
// iteration to undo it.  "+a" keeps every accumulator in place in the accumulation registers.  The
// statements are volatile, so the issue order below is the one written here.
#define SX_MFMA(ACC, A, B) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(ACC) : "v"(A), "v"(B));
// byte offset along K of this workgroup's i-th slab (past the last one: the last one's)
#define SX_OFFSET(i) ((first + min((i), NB - 1) + rot - (min((i), NB - 1) + rot < NB ? 0 : NB)) * (BK * 2))
// The 8 + JB fragment reads of a k-step, dealt over the 8 row blocks of the phase before it in the order
// the next phase needs them: W block 0 and all X blocks first, then W blocks 1..7.
#define SX_READS_A(XSTG_, WSTG_, FX, FW, KC, r)                                                                \
  if (r == 0) { SX_READW(WSTG_, FW, 0, KC) SX_READX(XSTG_, FX, 0, KC) }                                        \
  if (r == 1) { SX_READX(XSTG_, FX, 2, KC) SX_READX(XSTG_, FX, 3, KC) }                                        \
  if (r == 2) { SX_READX(XSTG_, FX, 5, KC) SX_READX(XSTG_, FX, 6, KC) }                                        \
  if (r == 3) { SX_READW(WSTG_, FW, 1, KC) }                                                                   \
  if (r == 4) { SX_READW(WSTG_, FW, 3, KC) }                                                                   \
  if (r == 5) { SX_READW(WSTG_, FW, 5, KC) }                                                                   \
  if (r == 6) { SX_READW(WSTG_, FW, 7, KC) }
#define SX_READS_B(XSTG_, WSTG_, FX, FW, KC, r)                                                                \
  if (r == 0) { SX_READX(XSTG_, FX, 1, KC) }                                                                   \
  if (r == 1) { SX_READX(XSTG_, FX, 4, KC) }                                                                   \
  if (r == 2) { SX_READX(XSTG_, FX, 7, KC) }                                                                   \
  if (r == 3) { SX_READW(WSTG_, FW, 2, KC) }                                                                   \
  if (r == 4) { SX_READW(WSTG_, FW, 4, KC) }                                                                   \
  if (r == 5) { SX_READW(WSTG_, FW, 6, KC) }
// The copies of a slab, dealt over the 16 half row blocks of a phase: X's before W's where W has a stage more, since then
// the barrier waits for X's and leaves W's in flight, by their number (the empty statement keeps the compiler from issuing one
// of W's among X's: they write arrays of their own); one of each in turn otherwise.
#define SX_COPIES(XSTG_, WSTG_, XSO_, WSO_, h)                                                                 \
  if (NW > NS) {                                                                                               \
    if ((h) < JB) { SX_COPY1(XSTG_, XSO_, 0, h) }                                                              \
    else if ((h) < JB + 8) {                                                                                   \
      if ((h) == JB) asm volatile("" ::: "memory");                                                            \
      SX_COPY1(WSTG_, WSO_, 1, ((h) - JB) & 7)                                                                 \
    }                                                                                                          \
  } else {                                                                                                     \
    if ((h) & 1) { SX_COPY1(WSTG_, WSO_, 1, (h) / 2) } else { SX_COPY1(XSTG_, XSO_, 0, (h) / 2) }              \
  }
// One slab from stages XSTG_ and WSTG_ (its k-step 0 already in fx0/fw0):
//   phase 1: the 8 JB MFMAs of k-step 0, with the fragment reads of k-step 1 between them;
//   barrier: everybody has read all of both stages, and everybody's copies of the next slab (stages XSTG_N, WSTG_N) are in
//   (three stages: those of the slab after it may be in flight, three of W alone: its W copies);
//   phase 2: the 8 JB MFMAs of k-step 1, with the copies of the slabs that take these stages (XNEXT_, WNEXT_)
//   and the reads of the next slab's k-step 0 between them.  The copies have until the next barrier, a slab's
//   worth of MFMAs away, or until the one after it.
#define SX_SLAB(XSTG_, XSTG_N, XNEXT_, WSTG_, WSTG_N, WNEXT_)                                                  \
  const int xso = SX_OFFSET(XNEXT_), wso = SX_OFFSET(WNEXT_);                                                  \
  _Pragma("unroll") for (int r = 0; r < 8; ++r) {                                                             \
    _Pragma("unroll") for (int j = 0; j < JB / 2; ++j) SX_MFMA(acc[r][j], fw0[r], fx0[j])                  \
    SX_READS_A(XSTG_, WSTG_, fx1, fw1, kc1, r)                                                                 \
    _Pragma("unroll") for (int j = JB / 2; j < JB; ++j) SX_MFMA(acc[r][j], fw0[r], fx0[j])                 \
    SX_READS_B(XSTG_, WSTG_, fx1, fw1, kc1, r)                                                                 \
  }                                                                                                            \
  SX_WAIT_BARRIER(NS == 3 ? wait_vm(kCopies + (TOUCH ? 1 : 0)) : NW == 3 ? wait_vm(8) : SHARE ? kWaitVm2 : kWaitVm0) \
  _Pragma("unroll") for (int r = 0; r < 8; ++r) {                                                             \
    _Pragma("unroll") for (int j = 0; j < JB / 2; ++j) SX_MFMA(acc[r][j], fw1[r], fx1[j])                  \
    SX_COPIES(XSTG_, WSTG_, xso, wso, 2 * r)                                                                   \
    SX_READS_A(XSTG_N, WSTG_N, fx0, fw0, kc0, r)                                                               \
    _Pragma("unroll") for (int j = JB / 2; j < JB; ++j) SX_MFMA(acc[r][j], fw1[r], fx1[j])                 \
    SX_COPIES(XSTG_, WSTG_, xso, wso, 2 * r + 1)                                                               \
    SX_READS_B(XSTG_N, WSTG_N, fx0, fw0, kc0, r)                                                               \
  }                                                                                                            \
  if (TOUCH) { asm volatile("" ::: "memory"); SX_TOUCH((WNEXT_) + kAhead) asm volatile("" ::: "memory"); }    \
  if (SHARE) { /* youngest in the queue: the barrier's wait lets these two loads stay in flight */             \
    asm volatile("" ::"v"(pfx), "v"(pfw) : "memory"); /* and they stay behind the copies issued above */       \
    const int pso = SX_OFFSET((WNEXT_) + kPfDist);                                                             \
    pfx = __builtin_amdgcn_raw_buffer_load_b32(xres, pfxoff, pso, 0);                                          \
    pfw = __builtin_amdgcn_raw_buffer_load_b32(pfwres, pfwoff, pso, 0);                                        \
  }

  // The loop body is branch-free: past the end of K it copies the last slab again, into a stage nobody
  // reads any more, and reads fragments nobody uses.
  const int nb_all = a.K / BK;
  const int first = kpart * nb_all / ksplit;                      // slabs of this workgroup: [first, first + NB)
  const int NB = (kpart + 1) * nb_all / ksplit - first;
  // Each XCD walks K from another eighth on (pick_plan() has the rule): started all at the first slab, 256 workgroups ask for
  // the same 128 bytes of rows that lie a power of two apart, and the memory channels take turns.  The workgroups of an
  // XCD stay in step with each other, since they share the operand lines in its L2 (rotated against each other they are
  // up to 8 % slower at 2048 rows).
  const int rot = SHARE || !a.rotate ? 0 : xcd * NB / 8;
  // (The waits count operations, so the slabs' copies have to go out in this order; they write arrays of their own, and
  // nothing else keeps the compiler from mixing them.)
  SX_COPY(xA, wA, SX_OFFSET(0))
  asm volatile("" ::: "memory");
  SX_COPY(xB, wB, SX_OFFSET(1))
  if (SHARE) {
    // The in-loop barriers let the two youngest operations stay in flight, taking them to be a slab's two
    // prefetch loads.  Before the first slab has issued any, the two youngest would be the last copies into the
    // second stage (X and W rows 56..63 of each wave's share), read by the first slab's second phase: so the
    // prologue issues a pair of prefetch loads of its own.  (Without them those rows were occasionally stale.)
    asm volatile("" ::: "memory");
    const int pso = SX_OFFSET(2);
    pfx = __builtin_amdgcn_raw_buffer_load_b32(xres, pfxoff, pso, 0);
    pfw = __builtin_amdgcn_raw_buffer_load_b32(pfwres, pfwoff, pso, 0);
  }
  if constexpr (NS == 3) { asm volatile("" ::: "memory"); SX_COPY(xC, wC, SX_OFFSET(2)) }
  else if constexpr (NW == 3) {
    asm volatile("" ::: "memory");
    _Pragma("unroll") for (int t = 0; t < 8; ++t) SX_COPY1(wC, SX_OFFSET(2), 1, t)
  }
  if (TOUCH) { asm volatile("" ::: "memory"); SX_TOUCH(2 + kAhead) asm volatile("" ::: "memory"); }
  SX_WAIT_BARRIER(wait_vm((NS - 1) * JB + (NW - 1) * 8 + (SHARE ? 2 : TOUCH ? 1 : 0)))
  _Pragma("unroll") for (int i = 0; i < 8; ++i) { SX_READW(wA, fw0, i, kc0) }
  _Pragma("unroll") for (int i = 0; i < JB; ++i) { SX_READX(xA, fx0, i, kc0) }
  int s = 0;
  if constexpr (NS == 3) {
    for (; s + 3 <= NB; s += 3) {
      { SX_SLAB(xA, xB, s + 3, wA, wB, s + 3) }
      { SX_SLAB(xB, xC, s + 4, wB, wC, s + 4) }
      { SX_SLAB(xC, xA, s + 5, wC, wA, s + 5) }
    }
    if (s < NB) {
      SX_SLAB(xA, xB, NB, wA, wB, NB)
    }
    if (s + 1 < NB) {
      SX_SLAB(xB, xC, NB, wB, wC, NB)
    }
  } else if constexpr (NW == 3) {
    for (; s + 6 <= NB; s += 6) {
      { SX_SLAB(xA, xB, s + 2, wA, wB, s + 3) }
      { SX_SLAB(xB, xA, s + 3, wB, wC, s + 4) }
      { SX_SLAB(xA, xB, s + 4, wC, wA, s + 5) }
      { SX_SLAB(xB, xA, s + 5, wA, wB, s + 6) }
      { SX_SLAB(xA, xB, s + 6, wB, wC, s + 7) }
      { SX_SLAB(xB, xA, s + 7, wC, wA, s + 8) }
    }
    if (s < NB) {
      SX_SLAB(xA, xB, s + 2, wA, wB, s + 3)
    }
    if (s + 1 < NB) {
      SX_SLAB(xB, xA, s + 3, wB, wC, s + 4)
    }
    if (s + 2 < NB) {
      SX_SLAB(xA, xB, s + 4, wC, wA, NB)
    }
    if (s + 3 < NB) {
      SX_SLAB(xB, xA, NB, wA, wB, NB)
    }
    if (s + 4 < NB) {
      SX_SLAB(xA, xB, NB, wB, wC, NB)
    }
  } else {
    for (; s + 2 <= NB; s += 2) {
      { SX_SLAB(xA, xB, s + 2, wA, wB, s + 2) }
      { SX_SLAB(xB, xA, s + 3, wB, wA, s + 3) }
    }
    if (s < NB) {  // one slab left, in stage A
      SX_SLAB(xA, xB, NB, wA, wB, NB)
    }
  }
  // Copies past the end of K may still be in flight: they must land before this workgroup's LDS is released.
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  asm volatile("" ::"v"(pfx), "v"(pfw));
  // the matrix pipe's last results must be written back before ordinary instructions read them; the
  // compiler cannot see the hand-written MFMAs, so the wait states are spelled out
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#undef SX_TOUCH
#undef SX_COPY1
#undef SX_OFFSET
#undef SX_COPY
#undef SX_READW
#undef SX_READX
#undef SX_MFMA
#undef SX_SLAB
#undef SX_READS_A
#undef SX_READS_B
#undef SX_COPIES

  // ---- K-split tail: the partial sums meet in memory, the last workgroup to arrive adds them up ---------
  // Every part writes its accumulators (register layout, 1 KB per wave and block: coalesced) and
  // bumps the tile's counter; whoever finds the others' bumps already there reads all parts back in
  // part order, so the sum does not depend on who came last.  Nobody waits for anybody.
  // Coherence without flushing caches: the partial sums are stored and loaded with device scope
  // (sc1: the stores write through the XCD's L2, the loads do not trust it), the stores are
  // complete (vmcnt 0) before the counter's device-scope atomic is issued, and the loads are issued
  // after it has returned.  A release/acquire fence pair would do the same by writing back and
  // invalidating the whole L2 under the feet of the workgroups still computing (measured: +40 us).
  if (ksplit > 1) {
    constexpr int kScopeDevice = 16;  // cache-policy bit sc1
    int& s_last = *reinterpret_cast<int*>(xA);  // the stages are read out, and may fill the LDS
    const int tail_tile = lin - a.full_tiles;
    const __amdgpu_buffer_rsrc_t pres = make_rsrc(a.part);
    const unsigned mine = (unsigned)(((tail_tile * ksplit + kpart) * 4 + wave) * (JB * 8 * 256) + lane * 4) * 4u;  // bytes
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < JB; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), pres, mine + (i * JB + j) * 1024, 0,
                                               kScopeDevice);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (tid == 0) {
      const int before = atomicAdd(a.part_cnt + tail_tile, 1);
      s_last = before == ksplit - 1;
      if (s_last) a.part_cnt[tail_tile] = 0;  // ready for the next launch
    }
    __syncthreads();
    if (!s_last) return;
    constexpr int kBatch = 2 * JB;
    // Read back in batches of kBatch blocks per part, all loads of a batch in flight together: one memory round
    // trip per batch and part instead of one per block (a block at a time, the 64 dependent round trips were
    // most of what the split cost).  Parts are added in part order whatever the batch size.
    const unsigned all = (unsigned)((tail_tile * ksplit * 4 + wave) * (JB * 8 * 256) + lane * 4) * 4u;
#pragma unroll
    for (int b0 = 0; b0 < 8 * JB; b0 += kBatch) {
      f32x4 sum[kBatch];
      for (int p = 0; p < ksplit; ++p) {
        f32x4 t[kBatch];
        if (p == kpart) {  // this workgroup's own part is still in its registers (the same bits it stored)
#pragma unroll
          for (int b = 0; b < kBatch; ++b) t[b] = acc[(b0 + b) / JB][(b0 + b) % JB];
        } else {
#pragma unroll
          for (int b = 0; b < kBatch; ++b)
            t[b] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                 pres, all + (unsigned)p * (4u * JB * 8 * 256 * 4) + (b0 + b) * 1024, 0,
                                                 kScopeDevice));
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) sum[b] = p == 0 ? t[b] : sum[b] + t[b];
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) acc[(b0 + b) / JB][(b0 + b) % JB] = sum[b];
    }
  }

  // ---- epilogue.  acc[i][j][e]: output row 16 j + l16 of the quadrant, W row 16 i + 4 lq + e ---------
  const int mbase = tile_m * BM + wm * (16 * JB);
  const bool vec = (a.N & 3) == 0;  // then every group of 4 columns is whole and 16-byte (8-byte) aligned
  if (MODE == SX_GEMM_QKV_ROPE) {
    // The quadrant's 128 columns are one head (head_dim 128): query head, key head or value head,
    // the same for the whole wave.  Column 16 i + 4 lq + e and column + 64 (block i + 4, same lane and
    // register) are the pair the rotary embedding turns by the row's angle (Alg. 1: node at position
    // P + depth); the values are rounded to bf16 once, after the rotation.
    // The tile's rows of the cos/sin table (512 bytes each) are first copied into the LDS the K loop has
    // left free -- 64 to a slab's stage -- and read from there:
    // loaded from memory row block by row block, every load waited behind the stores of the block before (one
    // counter covers both on this chip), 32 memory round trips per tile.  16-byte chunk c of table row r sits at
    // chunk position (c & 16) | ((c ^ r) & 15) of its 512 bytes: the 16 rows a read instruction covers fall on 16
    // bank groups.
    auto table = [&](int r64) -> unsigned char* { return r64 == 0 ? wA : r64 == 1 ? wB : NW == 3 ? (r64 == 2 ? wC : xA) : r64 == 2 ? xA : xB; };
    const int head = tile_n * 2 + wn;
    const bool is_v = head >= a.hq + a.hkv;
    unsigned short* dst = head < a.hq ? a.q : is_v ? a.v : a.k;
    const int hh = head < a.hq ? head : is_v ? head - a.hq - a.hkv : head - a.hq;
    const int nh = head < a.hq ? a.hq : a.hkv;
    if (tile_n * 2 < a.hq + a.hkv) {  // the tile holds a query or key head (same answer in all four waves)
      __syncthreads();  // every wave is past its last fragment reads of the stages
      const __amdgpu_buffer_rsrc_t cres = make_rsrc(a.cs);
#pragma unroll
      for (int t = 0; t < 4 * JB; ++t) {  // copy t of wave w: table rows 2 blk and 2 blk + 1
        const int blk = 4 * t + wave, r = 2 * blk + (lane >> 5);
        int m = tile_m * BM + r;
        m = m < a.M ? m : a.M - 1;
        const int pch = lane & 31, c = (pch & 16) | ((pch ^ r) & 15);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(cres, (lds_void_ptr)(table(t / 8) + blk % 32 * 1024), 16,
                                                 (int)((unsigned)m * 512u + (unsigned)c * 16u), 0, 0, 0);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    if (head < a.hq + 2 * a.hkv) {
#pragma unroll
      for (int j = 0; j < JB; ++j) {
        const int m = mbase + 16 * j + l16;
        if (m >= a.M) continue;
        unsigned short* y = dst + ((size_t)m * nh + hh) * 128 + 4 * lq;
        if (is_v) {
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            u32x2 o;
            o[0] = pack_bf16x2(acc[i][j][0], acc[i][j][1]);
            o[1] = pack_bf16x2(acc[i][j][2], acc[i][j][3]);
            *reinterpret_cast<u32x2*>(y + 16 * i) = o;
          }
        } else {
          const int r = wm * (16 * JB) + 16 * j + l16;
          const unsigned char* trow = table((wm * JB + j) / 4) + r % 64 * 512;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // (cos, sin) of pairs 16 i + 4 lq + 0..3: chunks 8 i + 2 lq and + 1 of the row
            const int c0 = 8 * i + 2 * lq;
            const f32x4 c01 = *reinterpret_cast<const f32x4*>(trow + (((c0 & 16) | ((c0 ^ r) & 15)) << 4));
            const f32x4 c23 = *reinterpret_cast<const f32x4*>(trow + ((((c0 + 1) & 16) | (((c0 + 1) ^ r) & 15)) << 4));
            const float cs_[4] = {c01[0], c01[2], c23[0], c23[2]}, sn_[4] = {c01[1], c01[3], c23[1], c23[3]};
            float lo[4], hi[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x0 = acc[i][j][e], x1 = acc[i + 4][j][e];
              rope_turn(x0, x1, cs_[e], sn_[e], lo[e], hi[e]);
            }
            u32x2 o;
            o[0] = pack_bf16x2(lo[0], lo[1]);
            o[1] = pack_bf16x2(lo[2], lo[3]);
            *reinterpret_cast<u32x2*>(y + 16 * i) = o;
            o[0] = pack_bf16x2(hi[0], hi[1]);
            o[1] = pack_bf16x2(hi[2], hi[3]);
            *reinterpret_cast<u32x2*>(y + 64 + 16 * i) = o;
          }
        }
      }
    }
  } else if (MODE == SX_GEMM_SWIGLU && vec && tile_m * BM + BM <= a.M && tile_n * (BN / 2) + BN / 2 <= a.N) {
    // a whole tile: no edge tests between the stores
    unsigned short* Yb = static_cast<unsigned short*>(a.Y) + (size_t)(mbase + l16) * a.N + (tile_n * (BN / 2) + wn * 64 + 4 * lq);
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) {
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_mul_bf16_bound(acc[2 * ii][j][e], acc[2 * ii + 1][j][e]);
        u32x2 v;
        v[0] = pack_bf16x2(h[0], h[1]);
        v[1] = pack_bf16x2(h[2], h[3]);
        *reinterpret_cast<u32x2*>(Yb + (size_t)(16 * j) * a.N + 16 * ii) = v;
      }
  } else if (MODE == SX_GEMM_SWIGLU) {
    unsigned short* Y = static_cast<unsigned short*>(a.Y);
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int m = mbase + 16 * j + l16;
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) {
        const int f = tile_n * (BN / 2) + wn * 64 + ii * 16 + 4 * lq;
        if (m >= a.M || f >= a.N) continue;
        unsigned short h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[2 * ii][j][e], u = acc[2 * ii + 1][j][e];
          h[e] = (unsigned short)f32_to_bf16_bits(silu_mul_bf16_bound(g, u));
        }
        unsigned short* y = Y + (size_t)m * a.N + f;
        if (vec) {
          u32x2 v;
          v[0] = h[0] | ((uint32_t)h[1] << 16);
          v[1] = h[2] | ((uint32_t)h[3] << 16);
          *reinterpret_cast<u32x2*>(y) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (f + e < a.N) y[e] = h[e];
        }
      }
    }
  } else if (vec && tile_m * BM + BM <= a.M && tile_n * BN + BN <= a.N) {
    // A whole tile: no edge tests, and the residual comes in 16 loads at a time (two row blocks) before the first
    // add -- a load, an add and a store per block, each waiting for its own load, made the epilogue 64 memory
    // round trips long.
    float* Yb = static_cast<float*>(a.Y) + (size_t)(mbase + l16) * a.N + (tile_n * BN + wn * 128 + 4 * lq);
#pragma unroll
    for (int j0 = 0; j0 < JB; j0 += 2) {
      f32x4 r[2][8];
      if (MODE == SX_GEMM_RESIDUAL) {
#pragma unroll
        for (int jj = 0; jj < 2 && j0 + jj < JB; ++jj)
#pragma unroll
          for (int i = 0; i < 8; ++i)
            r[jj][i] = *reinterpret_cast<const f32x4*>(Yb + (size_t)(16 * (j0 + jj)) * a.N + 16 * i);
      }
#pragma unroll
      for (int jj = 0; jj < 2 && j0 + jj < JB; ++jj)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          f32x4 v = acc[i][j0 + jj];
          if (MODE == SX_GEMM_RESIDUAL) v += r[jj][i];
          *reinterpret_cast<f32x4*>(Yb + (size_t)(16 * (j0 + jj)) * a.N + 16 * i) = v;
        }
    }
  } else {
    float* Y = static_cast<float*>(a.Y);
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int m = mbase + 16 * j + l16;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int n = tile_n * BN + wn * 128 + 16 * i + 4 * lq;
        if (m >= a.M || n >= a.N) continue;
        float* y = Y + (size_t)m * a.N + n;
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
#endif
}
#undef SX_WAIT_BARRIER


// Decides which tiles of 32 jb rows are cut along K, given memory for the partial sums, and returns what the launch is
// expected to take, in us.  Fewer tiles than half the compute units: all of them, in as many ways as keeps the parts in one
// round.  More tiles than compute units with a remainder that would fill at most half of the chip for a whole round: the
// remainder, in up to 6 ways.  Parts are at least 8 slabs long, and a cut has to pay: what it saves are slabs, what it costs
// are the partial tiles, written by all parts at once and read back by the last to arrive.  (Batches of at most 128 rows
// mostly take the narrow-tile kernel instead: for them a partial tile outweighs the weights a part streams.)
// The figures are fitted to 7100 launches: tiles of 128 to 256 rows, with and without the prefetch, uncut and cut in all
// these ways, the layer shapes of widths 2048 to 8192 (1B to 70B) at 25 row counts from 129 to 3000, weights from memory.  A
// slab's time is a stage's copies and MFMAs; those from 192 rows on are of 1120 launches with three stages of W (10 shapes, 16
// row counts).  (256 rows are bound by power where they fill the chip for many rounds, 1.4 to 1.5; the choice does not change.)
constexpr int kMaxRows = 256;
constexpr float slab_us(int jb) { return jb == 4 ? 0.815f : jb == 5 ? 0.975f : jb == 6 ? 1.04f : jb == 7 ? 1.16f : 1.30f; }
constexpr float kRoundUs = 4.1f;   // a round's beginning and end: first copies, epilogue
constexpr float kCutUs = 2.5f, kWayUs = 5.2f, kPartsUs = 16.f;  // 256-row tiles: a cut, per way, per chip full of parts
constexpr int kCutMaxWays = 16, kTailMaxWays = 6;
float plan_split(GemmArgs& a, int jb, void* split_ws, size_t split_ws_bytes) {
  a.tilesM = (a.M + 32 * jb - 1) / (32 * jb);
  a.chunk = (a.tilesM * a.tilesN + 7) / 8;
  a.split = 1;
  a.part = nullptr;
  a.part_cnt = nullptr;
  a.full_tiles = a.tail_items = a.full_per_xcd = a.tail_per_xcd = 0;
  const int cus = sx_compute_units(), tiles = a.tilesM * a.tilesN, nb = a.K / BK;
  const float walk = nb * slab_us(jb);
  const size_t part_bytes = (size_t)jb * 32 * BN * sizeof(float);
  const float uncut = (tiles + cus - 1) / cus * (walk + kRoundUs);
  const int rest = tiles % cus;
  const bool all = 2 * tiles <= cus;
  if (!split_ws || (!all && (tiles <= cus || rest == 0 || 2 * rest > cus))) return uncut;
  const int cut = all ? tiles : rest;
  if (cut > 256) return uncut;  // counters
  float best = uncut;
  for (int s = 2; s * cut <= cus && s <= (all ? kCutMaxWays : kTailMaxWays) && nb / s >= 8; ++s) {
    if (split_ws_bytes < 1024 + (size_t)cut * s * part_bytes) break;
    const float cost = uncut - walk + walk / s + jb / 8.f * (kCutUs + kWayUs * s + kPartsUs * cut * s / cus);
    if (cost < best) {
      best = cost;
      a.split = s;
    }
  }
  if (a.split > 1) {
    a.full_tiles = tiles - cut;
    a.tail_items = cut * a.split;
    a.full_per_xcd = (a.full_tiles + 7) / 8;
    a.tail_per_xcd = (a.tail_items + 7) / 8;
    a.part_cnt = static_cast<int*>(split_ws);
    a.part = reinterpret_cast<float*>(static_cast<char*>(split_ws) + 1024);
  }
  return best;
}

// What a launch looks like: tile height 32 jb, the prefetching form or not, and a's split and rotation.
//
// The height: the one that plan_split's figures expect to be fastest.  Over the 160 products of the second fit the choice is
// within 0.3 % of the best launch on average, 6 % at worst.
// Four things the figures do not know:
//   the prefetching form of 256 rows (8 row tiles, whole groups of 4 column tiles), unless every tile is cut, streams the
//   weights better than they say: a tenth;
//   so does that of 128 and 160 rows over several rounds, none of them cut (8192 x 8192 at 2500 rows, two rounds of 160 rows
//   278 us, 256 rows with 64 tiles cut 309): a twentieth;
//   short parts of K gain less from W's third stage: two stages of X and all tiles cut, 6 % (7B down at 670 rows, 64 tiles
//   of 192 rows in four parts 81 us, 80 of 160 rows in three 76);
//   a last row tile of several that is mostly padding takes less, which shows at 128 and 160 rows: without the discount 7B
//   gate|up at 525 rows took 103.6 us with 192 rows for 100.8 with 128, 70B down at 165 rows 141.0 for 136.6, 13824 -> 5120 at
//   525 rows 90.7 for 89.0.  (Not under a cut tail, where 70B down at 1040 rows would go from 419 to 438, nor with all tiles
//   cut in two, 7B QKV at 145 rows 41.1 to 41.9; with 192 rows 13824-wide gate|up at 2497 rows would go from 513 to 537.)
// (224 rows in as many row tiles as of 256 only drop padding, and are still faster: 7B QKV at 1100 rows 84 us for 93, gate|up 153
// for 169, 32000 columns, K = 4096, at 1300 rows 260 for 295.)
//
// The prefetch at 128 and 160 rows: from three row tiles on, where they share the touched lines, and only where they are all
// but full: 4 % on average, up to 18 (70B down, 640 rows in five tiles, 397 -> 336 us).  A row tile that is mostly padding
// copies less, runs ahead of the others and is their prefetch by itself; touching costs up to 8 % there, and up to 30 % where
// one row tile streams the weights for itself (70B gate|up at 150 rows).  Nor where rounds of uncut tiles follow each other with
// the last one nine tenths full but not whole: 32000 columns, K = 4096, at 600 rows (1.95 rounds) 142 us and 161 with it, at
// 740 (2.93) 190 and 199, at 1280 (3.91) 293 and 318; all ten products measured there are slower with it, those of whole
// rounds (70B O at 2048 rows, 2.0) up to 11 % faster.
//
// The rotation: at 128 and 160 rows always (150 rows, 70B gate|up 214 -> 173 us, never more than 2 % slower).  At 224 and 256:
// 2 to 3 %, at best 15 %, for one or two row tiles, where a launch is bound by the weight stream, 1 % and
// at best 6 up to 8 row tiles (70B O at 1000 rows, two parts of K: 142.7 -> 138.2 us).  Beyond that, and under a last round
// that is cut from four row tiles on, it gives and takes up to 3 %; parts of less than 20 slabs start apart by themselves
// and lose up to 5 % (7B O at 320 rows, four parts of 16).
struct Plan {
  int jb;
  bool prefetch;
};
Plan pick_plan(GemmArgs& a, void* split_ws, size_t split_ws_bytes) {
  Plan p = {8, false};
  const float tall = plan_split(a, 8, split_ws, split_ws_bytes);
  const int cus = sx_compute_units();
  const bool can_prefetch = a.tilesM == 8 && a.tilesN % 4 == 0;
  auto touch = [&](int jb) {  // the prefetching form of three stages, for the plan that a holds
    const int tiles = a.tilesM * a.tilesN;
    const bool nearly_whole = a.split == 1 && tiles > cus && tiles % cus * 10 >= 9 * cus;
    return stages(jb) == 3 && a.tilesM >= 3 && a.M * 25ll >= 23ll * 32 * jb * a.tilesM && !nearly_whole;
  };
  auto padding = [&](int jb) {  // of the plan that a holds: less for a mostly empty last row tile
    const float empty = a.tilesM - a.M / (32.f * jb);
    const bool counts = stages(jb) == 3 && a.tilesM > 1 && (a.split == 1 || (a.full_tiles == 0 && a.split > 2));
    return counts && empty > 0.6f ? 1.f - 0.12f * (empty - 0.6f) : 1.f;
  };
  const bool all_cut8 = a.split > 1 && a.full_tiles == 0;
  float best = (all_cut8 ? 1.06f : can_prefetch ? 0.9f : 1.f) * tall;
  for (int t = 7; t >= 4; --t) {
    float cost = plan_split(a, t, split_ws, split_ws_bytes);
    if (a.split == 1 && a.tilesM * a.tilesN > cus && touch(t)) cost *= 0.95f;
    if (a.split > 1 && a.full_tiles == 0 && stages(t) == 2) cost *= 1.06f;
    cost *= padding(t);
    if (cost < best) best = cost, p.jb = t;
  }
  plan_split(a, p.jb, split_ws, split_ws_bytes);
  if (stages(p.jb) == 3) {
    p.prefetch = touch(p.jb);
    a.rotate = 1;
  } else {
    p.prefetch = p.jb == 8 && can_prefetch;
    a.rotate = a.tilesM <= (a.split > 1 && a.full_tiles > 0 ? 3 : 8) && a.K / BK / a.split >= 20;
  }
  return p;
}

template <int MODE>
int launch(GemmArgs& a, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  const Plan p = pick_plan(a, split_ws, split_ws_bytes);
  const int grid = a.split > 1 ? 8 * (a.full_per_xcd + a.tail_per_xcd) : 8 * a.chunk;
  if (p.jb == 4 && p.prefetch) gemm_bf16_kernel<MODE, 4, true><<<grid, kThreads, 0, st>>>(a);
  else if (p.jb == 4) gemm_bf16_kernel<MODE, 4, false><<<grid, kThreads, 0, st>>>(a);
  else if (p.jb == 5 && p.prefetch) gemm_bf16_kernel<MODE, 5, true><<<grid, kThreads, 0, st>>>(a);
  else if (p.jb == 5) gemm_bf16_kernel<MODE, 5, false><<<grid, kThreads, 0, st>>>(a);
  else if (p.jb == 6) gemm_bf16_kernel<MODE, 6, false><<<grid, kThreads, 0, st>>>(a);
  else if (p.jb == 7) gemm_bf16_kernel<MODE, 7, false><<<grid, kThreads, 0, st>>>(a);
  else if (p.prefetch) gemm_bf16_kernel<MODE, 8, true><<<grid, kThreads, 0, st>>>(a);
  else gemm_bf16_kernel<MODE, 8, false><<<grid, kThreads, 0, st>>>(a);
  SX_LAUNCH_CHECK();
  return SX_OK;
}

}  // namespace

int sx_launch_gemm_bf16(const void* X, const void* W0, const void* W1, const void* W2, int n0, int n1, int n2,
                        void* Y, int M, int K, int mode, void* split_ws, size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || K < BK || K % BK != 0 || n0 < 1 || n1 < 0 || n2 < 0) return SX_ERR_SHAPE;
  if (!sx_operand_fits_u32(M, 2ll * K) || !sx_operand_fits_u32(n0, 2ll * K) || !sx_operand_fits_u32(n1, 2ll * K) ||
      !sx_operand_fits_u32(n2, 2ll * K))
    return SX_ERR_SHAPE;
  // At most 128 rows, the weight-streaming regime: narrow tiles, whose X is half as large a share of the copies and whose
  // partial sums are a quarter.  But where the 128-column ones take two rounds for what 256-column tiles do in one (20 %
  // faster on average: 100 rows, 28672 columns of gate|up, K = 8192 181 -> 165 us; 40000 columns, K = 4096 92.5 -> 77), and
  // beyond one round where the rows are nearly 128 (120000 columns 214 -> 200; at 64 rows 2 % slower on average), these.
  if (M <= 128) {
    const int cus = sx_compute_units(), wide = mode == SX_GEMM_SWIGLU ? (n0 + BN / 2 - 1) / (BN / 2) : (n0 + BN - 1) / BN;
    const bool one_matrix = mode == SX_GEMM_SWIGLU || (n1 == 0 && n2 == 0);
    if (!one_matrix || 2 * wide <= cus || (wide > cus && M <= 112))
      return sx_launch_gemm_skinny_bf16(X, W0, W1, W2, n0, n1, n2, Y, M, K, mode, split_ws, split_ws_bytes, st);
  }
  // a 16-row copy group must not straddle two stacked weight matrices
  if (mode != SX_GEMM_SWIGLU && ((n1 > 0 && n0 % 16 != 0) || (n2 > 0 && n1 % 16 != 0))) return SX_ERR_SHAPE;
  GemmArgs a;
  a.X = static_cast<const unsigned short*>(X);
  a.W0 = static_cast<const unsigned short*>(W0);
  a.W1 = static_cast<const unsigned short*>(W1 ? W1 : W0);
  a.W2 = static_cast<const unsigned short*>(W2 ? W2 : W0);
  a.n0 = n0;
  a.n1 = n1;
  a.n2 = n2;
  a.Y = Y;
  a.M = M;
  a.K = K;
  if (mode == SX_GEMM_SWIGLU) {
    if (n1 != n0 || n2 != 0 || !W1) return SX_ERR_SHAPE;
    a.N = n0;
    a.tilesN = (n0 + BN / 2 - 1) / (BN / 2);
  } else {
    a.N = n0 + n1 + n2;
    a.tilesN = (a.N + BN - 1) / BN;
  }
  switch (mode) {
    case SX_GEMM_STORE: return launch<SX_GEMM_STORE>(a, split_ws, split_ws_bytes, st);
    case SX_GEMM_RESIDUAL: return launch<SX_GEMM_RESIDUAL>(a, split_ws, split_ws_bytes, st);
    case SX_GEMM_SWIGLU: return launch<SX_GEMM_SWIGLU>(a, split_ws, split_ws_bytes, st);
  }
  return SX_ERR_SHAPE;
}

// 1 KB of counters (at most 256 split tiles, zero before the first launch) and one partial tile per compute unit
size_t sx_gemm_split_workspace() { return 1024 + (size_t)sx_compute_units() * kMaxRows * BN * sizeof(float); }

int sx_launch_gemm_qkv_rope_bf16(const void* X, const void* Wq, const void* Wk, const void* Wv, int hq, int hkv,
                                 const float2* rope_cs, void* q, void* k, void* v, int M, int K, void* split_ws,
                                 size_t split_ws_bytes, hipStream_t st) {
  if (M < 1 || K < BK || K % BK != 0 || hq < 1 || hkv < 1) return SX_ERR_SHAPE;
  if (!sx_operand_fits_u32(M, 2ll * K) || !sx_operand_fits_u32(128ll * hq, 2ll * K) ||
      !sx_operand_fits_u32(128ll * hkv, 2ll * K) || !sx_operand_fits_u32(M, 512))  // the table: 512 bytes per row
    return SX_ERR_SHAPE;
  if (M <= 128)
    return sx_launch_gemm_skinny_qkv_rope_bf16(X, Wq, Wk, Wv, hq, hkv, rope_cs, q, k, v, M, K, split_ws, split_ws_bytes, st);
  GemmArgs a;
  a.X = static_cast<const unsigned short*>(X);
  a.W0 = static_cast<const unsigned short*>(Wq);
  a.W1 = static_cast<const unsigned short*>(Wk);
  a.W2 = static_cast<const unsigned short*>(Wv);
  a.n0 = hq * 128;
  a.n1 = a.n2 = hkv * 128;
  a.Y = nullptr;
  a.M = M;
  a.K = K;
  a.N = a.n0 + a.n1 + a.n2;
  a.tilesN = (a.N + BN - 1) / BN;
  a.cs = rope_cs;
  a.q = static_cast<unsigned short*>(q);
  a.k = static_cast<unsigned short*>(k);
  a.v = static_cast<unsigned short*>(v);
  a.hq = hq;
  a.hkv = hkv;
  return launch<SX_GEMM_QKV_ROPE>(a, split_ws, split_ws_bytes, st);
}

extern "C" size_t sx_gemm_bf16_workspace(void) { return sx_gemm_split_workspace(); }

extern "C" int sx_gemm_bf16_wide_plan(int32_t M, int32_t N, int32_t K, int32_t mode, size_t workspace_bytes, int32_t* tile_rows,
                                      int32_t* k_parts, int32_t* cut_tiles, int32_t* prefetch) {
  if (!tile_rows || !k_parts || !cut_tiles || !prefetch) return SX_ERR_NULL;
  if (mode < 0 || mode > 2 || M < 1 || N < 1 || K < BK || K % BK != 0) return SX_ERR_SHAPE;
  GemmArgs a;
  a.M = M;
  a.K = K;
  a.tilesN = mode == SX_GEMM_SWIGLU ? (N + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
  int32_t somewhere = 0;  // (only whether there is memory is asked)
  const Plan p = pick_plan(a, workspace_bytes ? &somewhere : nullptr, workspace_bytes);
  *tile_rows = 32 * p.jb;
  *k_parts = a.split;
  *cut_tiles = a.split > 1 ? a.tilesM * a.tilesN - a.full_tiles : 0;
  *prefetch = p.prefetch;
  return SX_OK;
}

extern "C" int sx_gemm_bf16_ws(const void* X, const void* W, const void* W2, void* Y, int32_t M, int32_t N, int32_t K,
                               int32_t mode, void* workspace, size_t workspace_bytes, void* stream) {
  if (!X || !W || !Y || (mode == SX_GEMM_SWIGLU && !W2)) return SX_ERR_NULL;
  if (mode < 0 || mode > 2 || N < 1) return SX_ERR_SHAPE;
  if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 255)) return SX_ERR_WORKSPACE;
  if (mode == SX_GEMM_SWIGLU)
    return sx_launch_gemm_bf16(X, W, W2, nullptr, N, N, 0, Y, M, K, mode, workspace, workspace_bytes, (hipStream_t)stream);
  return sx_launch_gemm_bf16(X, W, nullptr, nullptr, N, 0, 0, Y, M, K, mode, workspace, workspace_bytes,
                             (hipStream_t)stream);
}

extern "C" int sx_gemm_bf16(const void* X, const void* W, const void* W2, void* Y, int32_t M, int32_t N, int32_t K,
                            int32_t mode, void* stream) {
  return sx_gemm_bf16_ws(X, W, W2, Y, M, N, K, mode, nullptr, 0, stream);
}
