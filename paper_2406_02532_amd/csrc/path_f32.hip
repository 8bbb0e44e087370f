// fp32 variants of the two heavy pieces of the forward (Alg. 1, FORWARD; App. D tree mask), used when
// the model dtype is fp32 (the tiny configuration that is compared with the oracle to 1e-4): every product and sum is
// an fp32 one.
#include "kernels.h"

namespace {

// ---- Y[M][N] = X[M][K] [W0; W1; W2]^T on v_mfma_f32_16x16x4_f32 -------------------------------------------------------
// What bounds it at the sizes of such models (64 x 1024 x 256): latency -- a few memory round trips and the launch.  So a
// workgroup is small in output (16 MB rows x 16 NB columns, MB = NB = 1 where that gives too few workgroups otherwise),
// its four waves share K between them (chunks of 16, the partial sums meet in LDS and are added in wave order), operands
// go straight from memory to registers with all loads of a batch in flight, and the projections that read the same X are
// one launch.  The tiled form before it (64 x 64 outputs, slabs of 16 through LDS, two barriers and a round trip each) took
// 62 us per product at 64 rows and 44 at 16; this one 4 to 6.
// A lane (l16 = lane % 16, lq = lane / 16) holds X[row l16] and W[row l16] at k = 16 c + 4 lq .. + 3: one 16-byte load each
// feeds four MFMAs, whose k index may be permuted as long as both operands agree.  The product is formed transposed (W
// rows as A), so a lane ends up with 4 consecutive output columns of one row.
struct F32Args {
  const float* X;
  const float *W0, *W1, *W2;
  int n0, n1, n2;
  float* Y;
  int M, N, K, ldy;  // N: output columns
};

// VEC: K is a multiple of 4 and all rows are 16-byte aligned.
template <int MODE, int MB, int NB, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Args a) {
  constexpr bool SWIGLU = MODE == SX_GEMM_SWIGLU;
  constexpr int WB = SWIGLU ? 2 * NB : NB;        // blocks of W rows: gate and up of the same columns
  constexpr int U = MB * WB >= 8 ? 1 : MB * WB >= 4 ? 2 : 4;  // chunks of K in flight per wave
  __shared__ __attribute__((aligned(16))) float red[4][MB * WB][64][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
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
      int n = min(n0 + 16 * i + l16, a.N - 1);
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
  auto load = [&](const float* p, int k) -> f32x4 {
    f32x4 v;
    if (VEC) {
      v = *reinterpret_cast<const f32x4*>(p + min(k, a.K - 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = k < a.K ? v[e] : 0.f;
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
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 16 * wave; k0 < a.K; k0 += 64 * U) {
    f32x4 x[U][MB], w[U][WB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u + 4 * lq;  // past the end both operands are zero
#pragma unroll
      for (int j = 0; j < MB; ++j) x[u][j] = load(xp[j], k);
#pragma unroll
      for (int i = 0; i < WB; ++i) w[u][i] = load(wp[i], k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < WB; ++i)
#pragma unroll
          for (int j = 0; j < MB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][s], x[u][j][s], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) *reinterpret_cast<f32x4*>(red[wave][i * MB + j][lane]) = acc[i][j];
  __syncthreads();
  auto total = [&](int b) {
    f32x4 v = *reinterpret_cast<const f32x4*>(red[0][b][lane]);
#pragma unroll
    for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const f32x4*>(red[w][b][lane]);
    return v;
  };
  // block (i, j): row 16 j + l16, columns 16 i + 4 lq .. + 3
  for (int b = wave; b < NB * MB; b += 4) {
    const int i = b / MB, j = b % MB;
    const int m = m0 + 16 * j + l16, n = n0 + 16 * i + 4 * lq;
    f32x4 v = total(b);
    if (SWIGLU) {
      const f32x4 u = total(b + NB * MB);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * u[e];
    }
    if (m >= a.M) continue;
    float* y = a.Y + (size_t)m * a.ldy + n;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < a.N) y[e] = MODE == SX_GEMM_RESIDUAL ? y[e] + v[e] : v[e];
  }
}

template <int MODE, int MB, int NB>
void go(const F32Args& a, bool vec, hipStream_t st) {
  const dim3 grid((a.N + 16 * NB - 1) / (16 * NB), (a.M + 16 * MB - 1) / (16 * MB));
  if (vec) gemm_f32_kernel<MODE, MB, NB, true><<<grid, 256, 0, st>>>(a);
  else gemm_f32_kernel<MODE, MB, NB, false><<<grid, 256, 0, st>>>(a);
}

// ---- tree attention ---------------------------------------------------------------------------------------------
// One workgroup per (node, query head).  Keys = the P prefix rows, then the node's ancestors and
// itself (found by walking parent pointers).  LDS: scores for all keys, then the ancestor list; at the
// end the waves' partial outputs.
// Sixteen lanes share a key row, W consecutive elements per lane and load (W = 4 where rows are 16-byte aligned), so rows
// are read coalesced and the 16 groups of the workgroup work on 16 keys at a time -- a lane per key with its row to
// itself, and in the second product a lane per output element walking all keys, took 37 us at 190 keys, this 9.
constexpr int kAttnThreads = 256;
constexpr int kAttnWalkLds = 2048;  // nodes up to this number walk their parents in LDS
template <int W, int NI>  // element (i, e) of a lane: (i * 16 + lane % 16) * W + e, i < NI
__global__ __launch_bounds__(kAttnThreads) void tree_attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_tree, const float* __restrict__ v_tree,
    const float* __restrict__ k_prefix, const float* __restrict__ v_prefix, const int* __restrict__ par_s,
    const int* __restrict__ depth, int first, int T, int P, int Hq, int Hkv, int Dh, float* __restrict__ out) {
  typedef float vec __attribute__((ext_vector_type(W == 1 ? 1 : 4)));
  constexpr int NG = kAttnThreads / 16;
  extern __shared__ float lds[];
  __shared__ float red[kAttnThreads / 64];
  const int node = first + blockIdx.x, h = blockIdx.y;
  const int kv = h / (Hq / Hkv);
  const int na = depth[node] + 1;
  const int nk = P + na;
  float* sc = lds;                                    // [nk], nk <= P + T
  int* anc = reinterpret_cast<int*>(lds + P + T);     // [na]
  const int tid = threadIdx.x, l16 = tid & 15, grp = tid >> 4;
  const bool in_lds = node < kAttnWalkLds;            // the walk's loads depend on each other: from LDS they are short
  int* sp = reinterpret_cast<int*>(lds);              // [node + 1], before the scores take the place
  if (in_lds) {
    for (int j = tid; j <= node; j += kAttnThreads) sp[j] = par_s[j];
    __syncthreads();
  }
  if (tid == 0) {
    int j = node;
    for (int s = na - 1; s >= 0; --s) {
      anc[s] = j;
      j = in_lds ? sp[j] : par_s[j];
    }
  }
  __syncthreads();
  const float* qp = q + ((size_t)blockIdx.x * Hq + h) * Dh;
  vec qv[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = (i * 16 + l16) * W;
#pragma unroll
    for (int e = 0; e < W; ++e) qv[i][e] = c + e < Dh ? qp[c + e] : 0.f;
  }
  // this lane's elements of a row; past Dh it re-reads the row's last ones, which nobody may multiply by a zero: an
  // infinity there is another lane's
  auto row = [&](const float* prefix, const float* tree, int j, vec (&r)[NI]) {
    const float* p = j < P ? prefix + ((size_t)j * Hkv + kv) * Dh : tree + ((size_t)anc[j - P] * Hkv + kv) * Dh;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = min((i * 16 + l16) * W, Dh - W);
      r[i] = *reinterpret_cast<const vec*>(p + c);
    }
  };
  const float scale = 1.0f / sqrtf((float)Dh);
  float mx = -__builtin_huge_valf();
  constexpr int U = 4;  // keys in flight per group
  for (int j0 = grp; j0 < nk; j0 += NG * U) {
    vec r[U][NI];
#pragma unroll
    for (int u = 0; u < U; ++u) row(k_prefix, k_tree, min(j0 + u * NG, nk - 1), r[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < W; ++e) s += (i * 16 + l16) * W < Dh ? qv[i][e] * r[u][i][e] : 0.f;
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o, 64);
      s *= scale;
      if (j0 + u * NG < nk) {
        if (l16 == 0) sc[j0 + u * NG] = s;
        mx = fmaxf(mx, s);
      }
    }
  }
  mx = block_max<kAttnThreads / 64>(mx, red);  // includes the barriers that publish sc[]
  float sum = 0.f;
  for (int j = tid; j < nk; j += kAttnThreads) {
    const float p = expf(sc[j] - mx);
    sc[j] = p;
    sum += p;
  }
  sum = block_sum<kAttnThreads / 64>(sum, red);
  const float inv = 1.0f / sum;
  vec o[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < W; ++e) o[i][e] = 0.f;
  for (int j0 = grp; j0 < nk; j0 += NG * U) {
    vec r[U][NI];
    float p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * NG, nk - 1);
      row(v_prefix, v_tree, j, r[u]);
      p[u] = sc[j];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j0 + u * NG < nk) {  // (past the end the last key is read again)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < W; ++e) o[i][e] += p[u] * r[u][i][e];
      }
  }
  // the four groups of a wave, then the four waves
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < W; ++e) {
      float t = o[i][e];
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      o[i][e] = t;
    }
  __syncthreads();  // the scores have been read: the waves' sums take their place
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const int c = (i * 16 + l16) * W + e;
      if ((tid & 63) < 16 && c < Dh) lds[(tid >> 6) * Dh + c] = o[i][e];
    }
  __syncthreads();
  for (int c = tid; c < Dh; c += kAttnThreads)
    out[((size_t)blockIdx.x * Hq + h) * Dh + c] = (((lds[c] + lds[Dh + c]) + lds[2 * Dh + c]) + lds[3 * Dh + c]) * inv;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

int sx_launch_gemm_f32(const float* X, const float* W0, const float* W1, const float* W2, int n0, int n1, int n2, float* Y,
                       int M, int K, int ldy, int mode, hipStream_t st) {
  F32Args a;
  a.X = X;
  a.W0 = W0;
  a.W1 = W1 ? W1 : W0;
  a.W2 = W2 ? W2 : W0;
  a.n0 = n0;
  a.n1 = n1;
  a.n2 = n2;
  a.Y = Y;
  a.M = M;
  a.N = mode == SX_GEMM_SWIGLU ? n0 : n0 + n1 + n2;
  a.K = K;
  a.ldy = ldy;
  const bool vec = K % 4 == 0 && aligned16(X) && aligned16(a.W0) && aligned16(a.W1) && aligned16(a.W2);
  // 16 x 16 outputs per workgroup until that makes more workgroups than the chip can hold several of per compute unit;
  // 64 x 64 (a quarter of the operand traffic per output) from there on
  const bool small = (long long)((a.N + 15) / 16) * ((M + 15) / 16) <= 8ll * sx_compute_units();
#define SX_GO(MODE_)                                       \
  if (small) go<MODE_, 1, 1>(a, vec, st);                  \
  else go<MODE_, 4, MODE_ == SX_GEMM_SWIGLU ? 2 : 4>(a, vec, st)
  switch (mode) {
    case SX_GEMM_STORE: SX_GO(SX_GEMM_STORE); break;
    case SX_GEMM_RESIDUAL: SX_GO(SX_GEMM_RESIDUAL); break;
    case SX_GEMM_SWIGLU: SX_GO(SX_GEMM_SWIGLU); break;
    default: return SX_ERR_SHAPE;
  }
#undef SX_GO
  SX_LAUNCH_CHECK();
  return SX_OK;
}

int sx_launch_tree_attn_f32(const float* q, const float* k_tree, const float* v_tree, const float* k_prefix,
                            const float* v_prefix, const int32_t* par_s, const int32_t* depth, int T, int first, int P,
                            int Hq, int Hkv, int Dh, float* out, hipStream_t st) {
  // worst case: a chain, depth T-1
  size_t shmem = (size_t)(P + 2 * T) * sizeof(float);
  if (shmem > 60 * 1024) return SX_ERR_SHAPE;
  if (shmem < 4 * (size_t)Dh * sizeof(float)) shmem = 4 * (size_t)Dh * sizeof(float);  // the four waves' outputs at the end
  dim3 grid(T - first, Hq);
  const bool vec = Dh % 4 == 0 && aligned16(k_tree) && aligned16(v_tree) && aligned16(k_prefix) && aligned16(v_prefix);
#define SX_GO(W, NI)                                                                                                   \
  tree_attn_f32_kernel<W, NI><<<grid, kAttnThreads, shmem, st>>>(q, k_tree, v_tree, k_prefix, v_prefix, par_s, depth,  \
                                                                 first, T, P, Hq, Hkv, Dh, out)
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
