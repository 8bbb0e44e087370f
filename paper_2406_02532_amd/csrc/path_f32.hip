// fp32 variants of the two heavy pieces of the forward (Alg. 1, FORWARD; App. D tree mask), used when
// the model dtype is fp32 (the tiny configuration that is compared with the oracle to 1e-4): every product and sum is
// an fp32 one.
#include "kernels.h"

namespace {

// ---- Y[M][N] = f(X)[M][K] [W0; W1; W2]^T on v_mfma_f32_16x16x4_f32 ----------------------------------------------------
// What bounds it at the sizes of such models (64 x 1024 x 256): latency -- a few memory round trips and the launch.  So a
// workgroup is small in output (16 MB rows x 16 NB columns, MB = NB = 1 where that gives too few workgroups otherwise),
// its waves share K between them (chunks of 16, the partial sums meet in LDS and are added in wave order), operands go
// straight from memory to registers with all loads of a batch in flight, and whatever else would be a launch of its own
// happens here: the projections that read the same X are one launch, the RMSNorm before a product is its prologue (NORM)
// and the rotary embedding and the split into heads are the epilogue of the QKV product.  16 rows of the tiny configuration
// (d 256, FFN 688), as launches of a trace: norm 2.8 + QKV 3.9 + rotation 2.6 us -> 4.4; norm 2.8 + gate|up 5.5 -> 5.0;
// O 3.8 -> 3.5 and down 7.5 -> 4.4 (eight and sixteen waves instead of four share K).
// A lane (l16 = lane % 16, lq = lane / 16) holds X[row l16] and W[row l16] at k = 16 c + 4 lq .. + 3: one 16-byte load each
// feeds four MFMAs, whose k index may be permuted as long as both operands agree.  The product is formed transposed (W
// rows as A), so a lane ends up with 4 consecutive output columns of one row.
// NORM: X is h g / sqrt(mean(h^2) + eps).  The row's factor is one for all of K: the product is formed over h g, the sum of
// squares on the side, and the factor multiplies the result -- fp32 either way, the factor rounded in once at the end
// instead of once per element.
struct F32Args {
  const float* X;
  const float *W0, *W1, *W2;
  int n0, n1, n2;
  float* Y;
  int M, N, K, ldy;  // N: output columns
  const float* gain;  // NORM
  float eps;
  const float2* cs;  // QKV: [M][Dh / 2]
  float *q, *k, *v;  //      [M][n0], [M][n1], [M][n2]
  int Dh;
};

// VEC: K is a multiple of 4 and all rows are 16-byte aligned.
// NW: waves; U: chunks of K in flight per wave.
template <int MODE, int MB, int NB, int NW, int U, bool NORM, bool VEC>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(F32Args a) {
  constexpr bool SWIGLU = MODE == SX_GEMM_SWIGLU, QKV = MODE == SX_GEMM_QKV_ROPE;
  constexpr int WB = SWIGLU ? 2 * NB : NB;        // blocks of W rows: gate and up of the same columns
  __shared__ __attribute__((aligned(16))) float red[NW][MB * WB][64][4];
  __shared__ float s_ss[NW][MB][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * 16 * MB, n0 = blockIdx.x * 16 * NB;
  const float *xp[MB], *wp[WB];
#pragma unroll
  for (int j = 0; j < MB; ++j) xp[j] = a.X + (size_t)min(m0 + 16 * j + l16, a.M - 1) * a.K;
#pragma unroll
  for (int i = 0; i < WB; ++i) {
    if (SWIGLU) {
      wp[i] = (i < NB ? a.W0 : a.W1) + (size_t)min(n0 + 16 * (i % NB) + l16, a.N - 1) * a.K;
    } else {
      int n = n0 + 16 * i + l16;
      if (QKV) {  // a block is eight pairs (j, j + Dh/2) of one head: the first eight rows are the j
        const int block = n >> 4, per = a.Dh >> 4;
        n = block / per * a.Dh + block % per * 8 + (l16 & 7) + (l16 >> 3) * (a.Dh >> 1);
      }
      n = min(n, a.N - 1);
      const float* w = a.W0;
      if (n >= a.n0 + a.n1) {
        w = a.W2;
        n -= a.n0 + a.n1;
      } else if (n >= a.n0) {
        w = a.W1;
        n -= a.n0;
      }
      wp[i] = w + (size_t)n * a.K;
    }
  }
  const bool ragged = a.K % 16 != 0;
  auto load = [&](const float* p, int k) -> f32x4 {
    f32x4 v;
    if (VEC) {
      v = *reinterpret_cast<const f32x4*>(p + min(k, a.K - 4));
      if (ragged) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = k < a.K ? v[e] : 0.f;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = p[min(k + e, a.K - 1)];
        v[e] = k + e < a.K ? t : 0.f;
      }
    }
    return v;
  };
  f32x4 acc[WB][MB];
  float ss[MB];
#pragma unroll
  for (int j = 0; j < MB; ++j) {
    ss[j] = 0.f;
#pragma unroll
    for (int i = 0; i < WB; ++i) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int k0 = 16 * wave; k0 < a.K; k0 += 16 * NW * U) {
    f32x4 x[U][MB], w[U][WB], g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && k0 + 16 * NW * u >= a.K) break;
      const int k = k0 + 16 * NW * u + 4 * lq;  // past the end both operands are zero
#pragma unroll
      for (int j = 0; j < MB; ++j) x[u][j] = load(xp[j], k);
      if (NORM) g[u] = load(a.gain, k);
#pragma unroll
      for (int i = 0; i < WB; ++i) w[u][i] = load(wp[i], k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u > 0 && k0 + 16 * NW * u >= a.K) break;
      if (NORM) {
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ss[j] += x[u][j][e] * x[u][j][e];
            x[u][j][e] *= g[u][e];
          }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
          for (int j = 0; j < MB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][s], x[u][j][s], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < MB; ++j) {
#pragma unroll
    for (int i = 0; i < WB; ++i) *reinterpret_cast<f32x4*>(red[wave][i * MB + j][lane]) = acc[i][j];
    if (NORM) {
      ss[j] += __shfl_xor(ss[j], 16, 64);
      ss[j] += __shfl_xor(ss[j], 32, 64);
      if (lq == 0) s_ss[wave][j][l16] = ss[j];
    }
  }
  __syncthreads();
  // Entry o of a block (i, j), as the lanes have left it: row 16 j + (o >> 2) % 16, column 16 i + 4 (o >> 6) + o % 4.  A lane
  // takes one at a time.
  for (int all = tid; all < 256 * NB * MB; all += 64 * NW) {
    const int b = all >> 8, o = all & 255, i = b / MB, j = b % MB, row = (o >> 2) & 15;
    const int m = m0 + 16 * j + row, n = n0 + 16 * i + 4 * (o >> 6) + (o & 3);
    if (m >= a.M || n >= a.N) continue;
    float r = 1.f;
    if (NORM) {
      float t = s_ss[0][j][row];
#pragma unroll
      for (int w = 1; w < NW; ++w) t += s_ss[w][j][row];
      r = 1.0f / sqrtf(t / (float)a.K + a.eps);
    }
    auto total = [&](int blk, int entry) {
      float v = (&red[0][blk][0][0])[entry];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += (&red[w][blk][0][0])[entry];
      return NORM ? v * r : v;
    };
    float v = total(b, o);
    if (SWIGLU) v = v / (1.0f + expf(-v)) * total(b + NB * MB, o);
    float* y = a.Y + (size_t)m * a.ldy + n;
    if (QKV) {
      const int half = a.Dh >> 1, per = a.Dh >> 4, block = n >> 4;
      const int j0 = block % per * 8 + (n & 7);  // the pair's first element
      const int second = (n >> 3) & 1, col = block / per * a.Dh + j0 + second * half;
      if (col < a.n0 + a.n1) {
        const float2 t = a.cs[(size_t)m * half + j0];
        const float other = total(b, o ^ 128);
        v = second ? other * t.y + v * t.x : v * t.x - other * t.y;
      }
      y = col < a.n0            ? a.q + (size_t)m * a.n0 + col
          : col < a.n0 + a.n1 ? a.k + (size_t)m * a.n1 + (col - a.n0)
                              : a.v + (size_t)m * a.n2 + (col - a.n0 - a.n1);
    }
    *y = MODE == SX_GEMM_RESIDUAL ? *y + v : v;
  }
}

template <int MODE, int MB, int NB, int NW, int U, bool NORM>
void go(const F32Args& a, bool vec, hipStream_t st) {
  const dim3 grid((a.N + 16 * NB - 1) / (16 * NB), (a.M + 16 * MB - 1) / (16 * MB));
  if (vec) gemm_f32_kernel<MODE, MB, NB, NW, U, NORM, true><<<grid, NW * 64, 0, st>>>(a);
  else gemm_f32_kernel<MODE, MB, NB, NW, U, NORM, false><<<grid, NW * 64, 0, st>>>(a);
}

// ---- tree attention ---------------------------------------------------------------------------------------------
// One workgroup per (node, query head).  Keys = the P prefix rows, then the node's ancestors and itself: from the list that
// the bookkeeping launch has made (anc, [n][anc_stride], self first), or found by walking parent pointers.
// What bounds it: the chain of its memory round trips.  So the softmax is a running one: K and V rows are fetched together,
// a batch of prefix keys while the ancestors are looked up, and each group of 16 lanes keeps maximum, sum and output of its
// own keys; they are merged once at the end.  16 nodes, 4 heads, 128 prefix keys: 8.0 -> 5.7 us (with the scores of all keys
// in LDS, a maximum, a sum and a second pass for V, and the parents walked in every workgroup), of which an empty launch is 2.
// Sixteen lanes share a key row, W consecutive elements per lane and load (W = 4 where rows are 16-byte aligned), so rows
// are read coalesced and the 16 groups of the workgroup work on 16 keys at a time.
constexpr int kAttnThreads = 256;
constexpr int kAttnWalkLds = 2048;  // nodes up to this number walk their parents in LDS
// sum over the 16 lanes of a row, inside the vector unit; every lane gets it
__device__ __forceinline__ float row16_sum(float v) {
#define SX_STEP(CTRL) v += __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
  SX_STEP(0x128)  // rotations by 8, 4, 2 and 1
  SX_STEP(0x124)
  SX_STEP(0x122)
  SX_STEP(0x121)
#undef SX_STEP
  return v;
}

// exp(x), x <= 0 or NaN, to 2 ulp: 2^h of the hardware, h the rounding of x log2(e); what h has lost, to the product and to
// the constant (whose second part it takes: without it 5 ulp at -20 and 20 at -85), comes back as a factor.  (A tenth of the
// code of expf.)
__device__ __forceinline__ float exp_neg(float x) {
  constexpr float l2e = 1.4426950408889634f, l2e_low = (float)(1.4426950408889634 - (double)l2e), ln2 = 0.6931471805599453f;
  x = x < -200.f ? -200.f : x;
  const float h = x * l2e, e = __builtin_amdgcn_exp2f(h);
  return __builtin_fmaf(e, __builtin_fmaf(x, l2e_low, __builtin_fmaf(x, l2e, -h)) * ln2, e);
}

template <int W, int NI>  // element (i, e) of a lane: (i * 16 + lane % 16) * W + e, i < NI
__global__ __launch_bounds__(kAttnThreads) void tree_attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_tree, const float* __restrict__ v_tree,
    const float* __restrict__ k_prefix, const float* __restrict__ v_prefix, const int* __restrict__ anc_list, int anc_stride,
    const int* __restrict__ par_s, const int* __restrict__ depth, int first, int T, int P, int Hq, int Hkv, int Dh,
    float* __restrict__ out) {
  typedef float vec __attribute__((ext_vector_type(W == 1 ? 1 : 4)));
  constexpr int NG = kAttnThreads / 16;
  constexpr int U = W * NI <= 8 ? 4 : 2;  // keys in flight per group, and as many ahead
  extern __shared__ float lds[];
  __shared__ float s_m[kAttnThreads / 64], s_l[kAttnThreads / 64];
  const int node = first + blockIdx.x, h = blockIdx.y;
  const int kv = h / (Hq / Hkv);
  const int tid = threadIdx.x, l16 = tid & 15, grp = tid >> 4;
  int* anc = reinterpret_cast<int*>(lds);         // [na]
  int* sp = anc + T;                              // [node + 1]
  // (the list's first entries are requested before their number is known)
  const int near = anc_list ? anc_list[(size_t)blockIdx.x * anc_stride + min(tid, T - 1)] : 0;
  const int na = depth[node] + 1, nk = P + na;
  const float* qp = q + ((size_t)blockIdx.x * Hq + h) * Dh;
  // the scale goes into q: as a factor of the score it would be contracted into the difference to the maximum, which is
  // then not zero for the maximum itself (1e22 for a score of 1e30)
  const float scale = 1.0f / sqrtf((float)Dh);
  vec qv[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = (i * 16 + l16) * W;
#pragma unroll
    for (int e = 0; e < W; ++e) qv[i][e] = c + e < Dh ? qp[c + e] * scale : 0.f;
  }
  // (the lowest finite value instead of -inf: the difference of two -inf scores must not become a NaN)
  float mx = -3.4028234663852886e38f, sum = 0.f;
  vec o[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < W; ++e) o[i][e] = 0.f;
  // this lane's elements of a row; past Dh it re-reads the row's last ones, which nobody may multiply by a zero: an
  // infinity there is another lane's
  auto row = [&](const float* p, vec (&r)[NI]) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = min((i * 16 + l16) * W, Dh - W);
      r[i] = *reinterpret_cast<const vec*>(p + c);
    }
  };
  vec kr[U][NI], vr[U][NI], kn[U][NI], vn[U][NI];
  auto fetch = [&](vec (&k)[U][NI], vec (&v)[U][NI], int j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * NG, nk - 1);
      const bool pre = j < P;
      const size_t at = ((size_t)(pre ? j : anc[max(j - P, 0)]) * Hkv + kv) * Dh;
      row((pre ? k_prefix : k_tree) + at, k[u]);
      row((pre ? v_prefix : v_tree) + at, v[u]);
    }
  };
  if (anc_list) {
    if (tid < na) anc[tid] = near;
    for (int s = tid + kAttnThreads; s < na; s += kAttnThreads) anc[s] = anc_list[(size_t)blockIdx.x * anc_stride + s];
  } else {
    const bool in_lds = node < kAttnWalkLds;  // the walk's loads depend on each other: from LDS they are short
    if (in_lds)
      for (int j = tid; j <= node; j += kAttnThreads) sp[j] = par_s[j];
    __syncthreads();
    if (tid == 0) {
      int j = node;
      for (int s = 0; s < na; ++s) {
        anc[s] = j;
        j = in_lds ? sp[j] : par_s[j];
      }
    }
  }
  __syncthreads();
  fetch(kr, vr, grp);
  for (int j0 = grp; j0 < nk; j0 += NG * U) {
    if (j0 + NG * U < nk) fetch(kn, vn, j0 + NG * U);
    float s[U], top = mx;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < W; ++e) s[u] += (i * 16 + l16) * W < Dh ? qv[i][e] * kr[u][i][e] : 0.f;
      s[u] = row16_sum(s[u]);
      if (j0 + u * NG < nk) top = fmaxf(top, s[u]);
    }
    const float f = exp_neg(mx - top);
    mx = top;
    sum *= f;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < W; ++e) o[i][e] *= f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * NG < nk) {  // (past the end the last key is read again)
        const float p = exp_neg(s[u] - top);
        sum += p;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < W; ++e) o[i][e] += p * vr[u][i][e];
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        kr[u][i] = kn[u][i];
        vr[u][i] = vn[u][i];
      }
  }
  // the four groups of a wave, then the four waves
  auto merge = [&](int lanes) {
    const float m2 = __shfl_xor(mx, lanes, 64), top = fmaxf(mx, m2);
    const float f = exp_neg(mx - top), f2 = exp_neg(m2 - top);
    sum = sum * f + __shfl_xor(sum, lanes, 64) * f2;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < W; ++e) o[i][e] = o[i][e] * f + __shfl_xor(o[i][e], lanes, 64) * f2;
    mx = top;
  };
  merge(16);
  merge(32);
  __syncthreads();  // the list has been read: the waves' outputs take its place
  if ((tid & 63) < 16) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int e = 0; e < W; ++e) {
        const int c = (i * 16 + l16) * W + e;
        if (c < Dh) lds[(tid >> 6) * Dh + c] = o[i][e];
      }
    if (l16 == 0) {
      s_m[tid >> 6] = mx;
      s_l[tid >> 6] = sum;
    }
  }
  __syncthreads();
  const float top = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
  float f[4], all = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    f[w] = exp_neg(s_m[w] - top);
    all += s_l[w] * f[w];
  }
  const float inv = 1.0f / all;
  for (int c = tid; c < Dh; c += kAttnThreads)
    out[((size_t)blockIdx.x * Hq + h) * Dh + c] =
        (((lds[c] * f[0] + lds[Dh + c] * f[1]) + lds[2 * Dh + c] * f[2]) + lds[3 * Dh + c] * f[3]) * inv;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

int sx_launch_gemm_f32(const SxF32Gemm& g, hipStream_t st) {
  F32Args a;
  a.X = g.X;
  a.W0 = g.W0;
  a.W1 = g.W1 ? g.W1 : g.W0;
  a.W2 = g.W2 ? g.W2 : g.W0;
  a.n0 = g.n0;
  a.n1 = g.n1;
  a.n2 = g.n2;
  a.Y = g.Y;
  a.M = g.M;
  a.N = g.mode == SX_GEMM_SWIGLU ? g.n0 : g.n0 + g.n1 + g.n2;
  a.K = g.K;
  a.ldy = g.ldy;
  a.gain = g.gain;
  a.eps = g.eps;
  a.cs = g.cs;
  a.q = g.q;
  a.k = g.k;
  a.v = g.v;
  a.Dh = g.Dh;
  const bool vec = g.K % 4 == 0 && aligned16(g.X) && aligned16(a.W0) && aligned16(a.W1) && aligned16(a.W2) &&
                   (!g.gain || aligned16(g.gain));
  // 16 x 16 outputs per workgroup until that makes more workgroups than the chip can hold several of per compute unit;
  // 64 x 64 (a quarter of the operand traffic per output) from there on
  const bool small = (long long)((a.N + 15) / 16) * ((g.M + 15) / 16) <= 8ll * sx_compute_units();
  // (two chunks per wave are all there is up to K = 256; past K a chunk costs its multiplications all the same)
#define SX_GO(MODE_, NORM_)                                                   \
  if (small && g.K <= 256) go<MODE_, 1, 1, 8, 2, NORM_>(a, vec, st);          \
  else if (small) go<MODE_, 1, 1, 16, 3, NORM_>(a, vec, st);                  \
  else go<MODE_, 4, MODE_ == SX_GEMM_SWIGLU ? 2 : 4, 4, 1, NORM_>(a, vec, st)
  switch (g.mode) {
    case SX_GEMM_STORE: SX_GO(SX_GEMM_STORE, true); break;
    case SX_GEMM_RESIDUAL: SX_GO(SX_GEMM_RESIDUAL, false); break;
    case SX_GEMM_SWIGLU: SX_GO(SX_GEMM_SWIGLU, true); break;
    case SX_GEMM_QKV_ROPE: SX_GO(SX_GEMM_QKV_ROPE, true); break;
    default: return SX_ERR_SHAPE;
  }
#undef SX_GO
  SX_LAUNCH_CHECK();
  return SX_OK;
}

int sx_launch_tree_attn_f32(const float* q, const float* k_tree, const float* v_tree, const float* k_prefix,
                            const float* v_prefix, const int32_t* anc, int anc_stride, const int32_t* par_s,
                            const int32_t* depth, int T, int first, int P, int Hq, int Hkv, int Dh, float* out, hipStream_t st) {
  if ((size_t)(P + 2 * T) * sizeof(float) > 60 * 1024) return SX_ERR_SHAPE;
  // ancestors (worst case: a chain, depth T - 1) and, where it is walked here, the parents; the four waves' outputs at the end
  size_t shmem = (size_t)(anc ? T : 2 * T) * sizeof(float);
  if (shmem < 4 * (size_t)Dh * sizeof(float)) shmem = 4 * (size_t)Dh * sizeof(float);
  dim3 grid(T - first, Hq);
  const bool vec = Dh % 4 == 0 && aligned16(k_tree) && aligned16(v_tree) && aligned16(k_prefix) && aligned16(v_prefix);
#define SX_GO(W, NI)                                                                                                   \
  tree_attn_f32_kernel<W, NI><<<grid, kAttnThreads, shmem, st>>>(q, k_tree, v_tree, k_prefix, v_prefix, anc, anc_stride, \
                                                                 par_s, depth, first, T, P, Hq, Hkv, Dh, out)
  // as few loads per key row and lane as cover it (1024 nodes, 1024 prefix keys, 32 heads of width 2, a whole layer: 2390 us
  // with sixteen, 667 with one; a thread per key took 1975)
  if (vec && Dh <= 64) SX_GO(4, 1);
  else if (vec && Dh <= 128) SX_GO(4, 2);
  else if (vec) SX_GO(4, 4);
  else if (Dh <= 16) SX_GO(1, 1);
  else if (Dh <= 64) SX_GO(1, 4);
  else if (Dh <= 128) SX_GO(1, 8);
  else SX_GO(1, 16);
#undef SX_GO
  SX_LAUNCH_CHECK();
  return SX_OK;
}
