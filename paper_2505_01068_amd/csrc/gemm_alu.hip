// fp32-ALU GEMM with strided operands for bf16 tensors whose widths the matrix-core kernels do not take (rows that are
// not whole 16-byte chunks); fp32 tensors go to gemm_split.hip.  Also: deterministic column sums and LayerNorm.
#include <type_traits>
#include "common.hpp"

namespace imattn {

constexpr int GA_BM = 64, GA_BN = 64, GA_BK = 16, GA_THREADS = 256;

struct GemmDev {
  const void* A;
  long sam, sak;
  const void* B[3];
  long sbk, sbn;
  int b_split, n_per, k_per;
  const void* bias[3];
  void* C[3];
  int c_split, bias_split;
  long ldc;
  const void* res;
  int M, N, K, gelu, split_k;
  float* partial;
  int kb, kt;
  long sab, sbb;
};

__device__ __forceinline__ float gelu_exact(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752440f)); }

template <typename TA, typename TB, typename TC>
__global__ __launch_bounds__(GA_THREADS) void gemm_alu_kernel(GemmDev g) {
  __shared__ __attribute__((aligned(16))) float As[GA_BK][GA_BM + 4];
  __shared__ __attribute__((aligned(16))) float Bs[GA_BK][GA_BN + 4];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * GA_BM, n0 = blockIdx.x * GA_BN;
  const int tx = tid % 16, ty = tid / 16;
  const TA* A = (const TA*)g.A;

  // K range of this split
  const int ktiles = (g.K + GA_BK - 1) / GA_BK;
  const int per_split = (ktiles + g.split_k - 1) / g.split_k;
  const int kt_begin = blockIdx.z * per_split;
  const int kt_end = min(ktiles, kt_begin + per_split);

  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  const bool a_kfast = (g.sak == 1);
  const bool b_nfast = (g.sbn == 1);
  // The next k-tile is fetched into registers while the current one is multiplied (the global round
  // trip would otherwise be exposed once per 16-deep tile).
  float ra[4], rb[4];
  auto fetch = [&](int kt) {
    const int kbase = kt * GA_BK;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = tid + u * GA_THREADS;
      int m, k;
      if (a_kfast) { k = idx % GA_BK; m = idx / GA_BK; } else { m = idx % GA_BM; k = idx / GA_BM; }
      const int gm = m0 + m, gk = kbase + k;
      float v = 0.f;
      if (gm < g.M && gk < g.K) {
        long off;
        if (g.kb > 1) { const int bb = gk / g.kt, kk = gk % g.kt; off = bb * g.sab + (long)kk * g.sak; }
        else off = (long)gk * g.sak;
        v = ldf(A + (long)gm * g.sam + off);
      }
      ra[u] = v;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = tid + u * GA_THREADS;
      int n, k;
      if (b_nfast) { n = idx % GA_BN; k = idx / GA_BN; } else { k = idx % GA_BK; n = idx / GA_BK; }
      const int gn = n0 + n, gk = kbase + k;
      float v = 0.f;
      if (gn < g.N && gk < g.K) {
        int sel = 0, kk = gk, nn = gn;
        long boff = 0;
        if (g.b_split == 1) { sel = gn / g.n_per; nn = gn % g.n_per; }
        else if (g.b_split == 2) { sel = gk / g.k_per; kk = gk % g.k_per; }
        if (g.kb > 1) { const int bb = gk / g.kt; kk = gk % g.kt; boff = bb * g.sbb; }
        v = ldf((const TB*)g.B[sel] + boff + (long)kk * g.sbk + (long)nn * g.sbn);
      }
      rb[u] = v;
    }
  };
  if (kt_begin < kt_end) fetch(kt_begin);
  for (int kt = kt_begin; kt < kt_end; ++kt) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int idx = tid + u * GA_THREADS;
      if (a_kfast) As[idx % GA_BK][idx / GA_BK] = ra[u]; else As[idx / GA_BM][idx % GA_BM] = ra[u];
      if (b_nfast) Bs[idx / GA_BN][idx % GA_BN] = rb[u]; else Bs[idx % GA_BK][idx / GA_BK] = rb[u];
    }
    __syncthreads();
    if (kt + 1 < kt_end) fetch(kt + 1);
#pragma unroll
    for (int k = 0; k < GA_BK; ++k) {
      const float4 a = *(const float4*)&As[k][ty * 4];
      const float4 b = *(const float4*)&Bs[k][tx * 4];
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
  }

#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int gm = m0 + ty * 4 + i;
    if (gm >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int gn = n0 + tx * 4 + j;
      if (gn >= g.N) continue;
      float v = acc[i][j];
      if (g.split_k > 1) {
        g.partial[((long)blockIdx.z * g.M + gm) * g.N + gn] = v;
        continue;
      }
      int sel = 0, nn = gn;
      if (g.n_per > 0) { sel = gn / g.n_per; nn = gn % g.n_per; }
      const int bsel = g.bias_split ? sel : 0;
      if (g.bias[bsel]) v += ldf((const TC*)g.bias[bsel] + (g.bias_split ? nn : gn));
      if (g.gelu) v = gelu_exact(v);
      if (g.c_split) {
        stf((TC*)g.C[sel] + (long)gm * g.ldc + nn, v);
      } else {
        if (g.res) v += ldf((const TC*)g.res + (long)gm * g.ldc + gn);
        stf((TC*)g.C[0] + (long)gm * g.ldc + gn, v);
      }
    }
  }
}

// Sum split-K partials in a fixed order and write fp32 outputs (weight gradients).  A block of 256
// threads owns 64 consecutive outputs; thread (zz, o) sums partials z = zz, zz+4, ... and the four
// sub-sums are added in a fixed order, so the result does not depend on scheduling.
__global__ __launch_bounds__(256) void gemm_splitk_reduce_kernel(GemmDev g) {
  __shared__ float part[4][64];
  const long n_out = (long)g.M * g.N;
  const int o = threadIdx.x & 63, zz = threadIdx.x >> 6;
  const long i = (long)blockIdx.x * 64 + o;
  float s = 0.f;
  if (i < n_out)
    for (int z = zz; z < g.split_k; z += 4) s += g.partial[z * n_out + i];
  part[zz][o] = s;
  __syncthreads();
  if (zz == 0 && i < n_out) {
    s = (part[0][o] + part[1][o]) + (part[2][o] + part[3][o]);
    const int gm = i / g.N, gn = i % g.N;
    int sel = 0, nn = gn;
    if (g.n_per > 0) { sel = gn / g.n_per; nn = gn % g.n_per; }
    if (g.c_split) ((float*)g.C[sel])[(long)gm * g.ldc + nn] = s;
    else ((float*)g.C[0])[(long)gm * g.ldc + gn] = s;
  }
}

size_t gemm_alu_partial_bytes(int M, int N, int K, int* split_k) {
  // Split only reductions that are much longer than the output is wide (weight gradients).
  int s = 1;
  const long tiles = (long)((M + GA_BM - 1) / GA_BM) * ((N + GA_BN - 1) / GA_BN);
  if (K >= 2048 && tiles < 256) {
    s = (int)((512 + tiles - 1) / tiles);
    const int ktiles = (K + GA_BK - 1) / GA_BK;
    if (s > ktiles / 8) s = ktiles / 8;
    if (s > 128) s = 128;
    if (s < 1) s = 1;
  }
  if (split_k) *split_k = s;
  return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

int launch_gemm_alu(const GemmDesc& d, int a_bf16, int b_bf16, int c_bf16, hipStream_t st) {
  GemmDev g;
  g.A = d.A; g.sam = d.sam; g.sak = d.sak;
  for (int i = 0; i < 3; ++i) { g.B[i] = d.B[i]; g.bias[i] = d.bias[i]; g.C[i] = d.C[i]; }
  g.sbk = d.sbk; g.sbn = d.sbn; g.b_split = d.b_split; g.n_per = d.n_per; g.k_per = d.k_per; g.c_split = d.c_split;
  g.bias_split = d.bias_split; g.ldc = d.ldc;
  g.res = d.res; g.M = d.M; g.N = d.N; g.K = d.K; g.gelu = d.gelu;
  g.split_k = d.split_k > 1 ? d.split_k : 1; g.partial = d.partial;
  g.kb = d.kb > 1 ? d.kb : 1; g.kt = d.kb > 1 ? d.kt : d.K; g.sab = d.sab; g.sbb = d.sbb;
  if (g.M <= 0 || g.N <= 0) return IM_OK;
  if (!a_bf16 && !b_bf16 && !c_bf16 && gemm_split_ok(d)) {
    launch_gemm_split(d, st);
    return IM_OK;
  }
  dim3 grid((g.N + GA_BN - 1) / GA_BN, (g.M + GA_BM - 1) / GA_BM, g.split_k), block(GA_THREADS);
  const int key = (a_bf16 ? 4 : 0) | (b_bf16 ? 2 : 0) | (c_bf16 ? 1 : 0);
  switch (key) {
    case 7: hipLaunchKernelGGL((gemm_alu_kernel<bf16_t, bf16_t, bf16_t>), grid, block, 0, st, g); break;
    case 6: hipLaunchKernelGGL((gemm_alu_kernel<bf16_t, bf16_t, float>), grid, block, 0, st, g); break;
    default: set_error("gemm_alu: unsupported operand type combination %d", key); return IM_ERR_UNSUPPORTED;
  }
  if (g.split_k > 1)
    hipLaunchKernelGGL(gemm_splitk_reduce_kernel, dim3((unsigned)(((long)g.M * g.N + 63) / 64)), dim3(256), 0, st, g);
  return IM_OK;
}

// ---- column sums (bias gradients): stage 1 sums blocks of rows, stage 2 sums the blocks in order ----
// ---- weight gradient of a narrow bf16 layer: C[M, N] = A[R, M]^T G[R, N], M <= 64, N <= 256, R long ----
// The general GEMM above spends its time in a latency-bound loop of R / split 16-deep k-tiles.  Here a
// block stages WS_RB rows of A and G in LDS with all loads in flight at once and every thread keeps a
// TM x TN patch of the output in registers (thread (ty, tx): rows ty + 8 i, columns tx + 32 j, so the
// LDS reads are broadcasts / consecutive words).  Each block writes one partial [M, N]; the caller
// reduces the partials in a fixed order.
constexpr int WS_RB = 32;
constexpr int WS_MAX_BLOCKS = 1024;
template <int TM, int TN>
__global__ __launch_bounds__(256) void wgrad_small_kernel(const bf16_t* __restrict__ A, long lda, const bf16_t* __restrict__ G,
                                                          long ldg, int R, int M, int N, float* __restrict__ partial) {
  __shared__ float sm[WS_RB * (64 + 256)];
  float* sA = sm;
  float* sG = sm + WS_RB * M;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  float acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;
  int mi[TM], nj[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) mi[i] = min(ty + 8 * i, M - 1);
#pragma unroll
  for (int j = 0; j < TN; ++j) nj[j] = min(tx + 32 * j, N - 1);
  const int nchunks = (R + WS_RB - 1) / WS_RB;
  for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const long row0 = (long)ch * WS_RB;
    __syncthreads();
    for (int e = threadIdx.x; e < WS_RB * M; e += 256) {
      const int r = e / M, m = e - r * M;
      sA[e] = row0 + r < R ? ldf(A + (row0 + r) * lda + m) : 0.f;
    }
    for (int e = threadIdx.x; e < WS_RB * N; e += 256) {
      const int r = e / N, n = e - r * N;
      sG[e] = row0 + r < R ? ldf(G + (row0 + r) * ldg + n) : 0.f;
    }
    __syncthreads();
#pragma unroll 4
    for (int r = 0; r < WS_RB; ++r) {
      float a[TM], g[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = sA[r * M + mi[i]];
#pragma unroll
      for (int j = 0; j < TN; ++j) g[j] = sG[r * N + nj[j]];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = fmaf(a[i], g[j], acc[i][j]);
    }
  }
  float* out = partial + (long)blockIdx.x * M * N;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = ty + 8 * i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = tx + 32 * j;
      if (n < N) out[(long)m * N + n] = acc[i][j];
    }
  }
}

// out[m, n] = sum_z partial[z][m][n], z in a fixed order; column block s of n_per columns goes to the [M, n_per]
// matrix o<s> (NULL = dropped) when n_per > 0, else everything to o0.  A block of 256 threads owns 16
// consecutive outputs: thread (g, o) sums z = g, g + 16, ... with four running sums (independent loads in
// flight), then the 16 groups are added in a fixed order.
__global__ __launch_bounds__(256) void wgrad_small_reduce_kernel(const float* __restrict__ partial, int nz, int M, int N,
                                                                 float* o0, float* o1, float* o2, int n_per) {
  __shared__ float red[16][16];
  const int o = threadIdx.x & 15, g = threadIdx.x >> 4;
  const long n_out = (long)M * N;
  const long i = (long)blockIdx.x * 16 + o;
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  if (i < n_out) {
    int z = g;
    for (; z + 48 < nz; z += 64) {
      s0 += partial[(long)z * n_out + i];
      s1 += partial[(long)(z + 16) * n_out + i];
      s2 += partial[(long)(z + 32) * n_out + i];
      s3 += partial[(long)(z + 48) * n_out + i];
    }
    for (; z < nz; z += 16) s0 += partial[(long)z * n_out + i];
  }
  red[g][o] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (g == 0 && i < n_out) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) v += red[k][o];
    const int m = (int)(i / N), n = (int)(i - (long)m * N);
    if (n_per > 0) {
      float* dst = (n / n_per == 0) ? o0 : (n / n_per == 1) ? o1 : o2;
      if (dst) dst[(long)m * n_per + n % n_per] = v;
    } else {
      o0[i] = v;
    }
  }
}
void launch_wgrad_small_reduce(const float* partial, int nz, int M, int N, float* o0, float* o1, float* o2, int n_per,
                               hipStream_t st) {
  const long n_out = (long)M * N;
  hipLaunchKernelGGL(wgrad_small_reduce_kernel, dim3((unsigned)((n_out + 15) / 16)), dim3(256), 0, st, partial, nz, M, N, o0,
                     o1, o2, n_per);
}

bool wgrad_small_ok(int M, int N, int n_per) {
  (void)n_per;
  return M >= 1 && M <= 64 && N >= 1 && N <= 256;
}
int wgrad_small_blocks(int R) {
  const int nchunks = (R + WS_RB - 1) / WS_RB;
  return nchunks < WS_MAX_BLOCKS ? nchunks : WS_MAX_BLOCKS;
}
size_t wgrad_small_partial_bytes(int M, int N, int R) { return (size_t)wgrad_small_blocks(R) * M * N * sizeof(float); }

template <int TM>
static void launch_wgrad_small_tn(const bf16_t* A, long lda, const bf16_t* G, long ldg, int R, int M, int N, float* partial,
                                  int blocks, hipStream_t st) {
  const int tn = (N + 31) / 32;
  if (tn <= 2) hipLaunchKernelGGL((wgrad_small_kernel<TM, 2>), dim3(blocks), dim3(256), 0, st, A, lda, G, ldg, R, M, N, partial);
  else if (tn <= 4) hipLaunchKernelGGL((wgrad_small_kernel<TM, 4>), dim3(blocks), dim3(256), 0, st, A, lda, G, ldg, R, M, N, partial);
  else if (tn <= 6) hipLaunchKernelGGL((wgrad_small_kernel<TM, 6>), dim3(blocks), dim3(256), 0, st, A, lda, G, ldg, R, M, N, partial);
  else hipLaunchKernelGGL((wgrad_small_kernel<TM, 8>), dim3(blocks), dim3(256), 0, st, A, lda, G, ldg, R, M, N, partial);
}
// Writes wgrad_small_blocks(R) partial [M, N] matrices; returns that count (the number of partials to reduce).
int launch_wgrad_small(const void* A, long lda, const void* G, long ldg, int R, int M, int N, float* partial, hipStream_t st) {
  const int blocks = wgrad_small_blocks(R), tm = (M + 7) / 8;
  const bf16_t *a = (const bf16_t*)A, *g = (const bf16_t*)G;
  if (tm <= 4) launch_wgrad_small_tn<4>(a, lda, g, ldg, R, M, N, partial, blocks, st);
  else if (tm <= 5) launch_wgrad_small_tn<5>(a, lda, g, ldg, R, M, N, partial, blocks, st);
  else launch_wgrad_small_tn<8>(a, lda, g, ldg, R, M, N, partial, blocks, st);
  return blocks;
}

// Column sums of up to four [R, n] matrices in two deterministic stages (one launch each for all of
// them: blockIdx.z selects the matrix).  Stage 1: a block of 256 threads = 4 row groups x 64 columns
// sums CS_ROWS rows (thread (g, c): rows r0 + g, r0 + g + 4, ..., with four independent running sums so
// loads overlap), then the 4 groups are added in a fixed order through LDS.  Stage 2 adds the
// per-block partials ([matrix][row block][n]) the same way with 16 groups x 16 columns.
constexpr int CS_ROWS = 256;
struct ColsumArgs {
  const void* a[4];
  long lda[4];
  float* out[4];   // nullptr: this matrix is skipped
};

template <typename T>
__global__ __launch_bounds__(256) void colsum_stage1(ColsumArgs q, int R, int n, float* __restrict__ partial) {
  __shared__ float red[4][64];
  const int z = blockIdx.z;
  if (!q.out[z]) return;
  const T* __restrict__ a = (const T*)q.a[z];
  const long lda = q.lda[z];
  const int tx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + tx;
  const int r0 = blockIdx.y * CS_ROWS, r1 = min(R, r0 + CS_ROWS);
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  if (c < n) {
    int r = r0 + g;
    for (; r + 12 < r1; r += 16) {
      s0 += ldf(a + (long)r * lda + c);
      s1 += ldf(a + (long)(r + 4) * lda + c);
      s2 += ldf(a + (long)(r + 8) * lda + c);
      s3 += ldf(a + (long)(r + 12) * lda + c);
    }
    for (; r < r1; r += 4) s0 += ldf(a + (long)r * lda + c);
  }
  red[g][tx] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (g == 0 && c < n)
    partial[((long)z * gridDim.y + blockIdx.y) * n + c] = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
}
// Stage 1 with 16-byte loads, for matrices whose rows allow them (n and lda multiples of the vector width, base
// aligned, n <= 256 vectors): a block covers all n columns of its CS_ROWS rows as (n / VW column groups) x (row
// groups); a thread requests eight rows at a time.  The element-per-thread kernel above walks 64 rows per thread
// with four loads in flight, which at 30 000 rows is sixteen exposed round trips per launch.
template <typename T>
__global__ __launch_bounds__(256) void colsum_stage1_vec(ColsumArgs q, int R, int n, float* __restrict__ partial) {
  constexpr int VW = 16 / sizeof(T);
  __shared__ float red[256 * VW];
  const int z = blockIdx.z;
  if (!q.out[z]) return;
  const T* __restrict__ a = (const T*)q.a[z];
  const long lda = q.lda[z];
  const int CG = n / VW, RG = 256 / CG;
  const int cg = threadIdx.x % CG, rg = threadIdx.x / CG;
  const int r0 = blockIdx.y * CS_ROWS, r1 = min(R, r0 + CS_ROWS);
  float s[VW];
#pragma unroll
  for (int e = 0; e < VW; ++e) s[e] = 0.f;
  if (rg < RG) {
    for (int r = r0 + rg; r < r1; r += 8 * RG) {
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int rr = min(r + u * RG, r1 - 1);   // every load is issued (no branch, no wait per row); rows past the
        v[u] = *(const uint4*)(a + (long)rr * lda + cg * VW);   // block are read again and dropped below
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (r + u * RG >= r1) v[u] = make_uint4(0u, 0u, 0u, 0u);
        const unsigned w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (sizeof(T) == 2) { s[2 * e] += __uint_as_float(w[e] << 16); s[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u); }
          else s[e] += __uint_as_float(w[e]);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < VW; ++e) red[rg * n + cg * VW + e] = s[e];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < n; c += 256) {
    float t = red[c];
    for (int g = 1; g < RG; ++g) t += red[g * n + c];
    partial[((long)z * gridDim.y + blockIdx.y) * n + c] = t;
  }
}
__global__ __launch_bounds__(256) void colsum_stage2(const float* __restrict__ partial, int nblk, int n, ColsumArgs q) {
  // 16 groups x 16 columns: group g adds row blocks g, g + 16, ... in ascending order, then the 16 group sums are
  // added in a fixed order (a block of 4 groups x 64 columns left one workgroup walking through all the partials)
  __shared__ float red[16][16];
  const int z = blockIdx.z;
  if (!q.out[z]) return;
  const int tx = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int c = blockIdx.x * 16 + tx;
  float s = 0.f;
  if (c < n)
    for (int b = g; b < nblk; b += 16) s += partial[((long)z * nblk + b) * n + c];
  red[g][tx] = s;
  __syncthreads();
  if (g != 0 || c >= n) return;
  for (int k = 1; k < 16; ++k) s += red[k][tx];
  q.out[z][c] = s;
}
// bytes of `partial` for ONE matrix; launch_colsum_multi needs count times as much
size_t colsum_partial_bytes(int R, int n) { return (size_t)((R + CS_ROWS - 1) / CS_ROWS) * n * sizeof(float); }

// One launch for a list of second-stage sums.  A block is 16 output quads x 16 lanes over the
// partials: lane zl adds partials zl, zl + 16, ... in ascending order, then the 16 lane sums are added in a fixed
// order through LDS -- the same order as colsum_stage2 and the parallel split-K reduction use on their own.  Fewer lanes share
// a quad (8, 4 or 2, with as many times the quads per block) where no lane would have a second partial otherwise, or where the
// output alone fills the chip: 786 432 sums of 10 partials took 19 us with 16 lanes, six of them idle.  More than 256
// partials are shared by 32 or 64 lanes: 925 of them are 15 trips to memory, one after the other, for 16 lanes.
// ODD: some job's rows or column blocks are not whole quads.
template <bool ODD>
__global__ __launch_bounds__(256) void reduce_list_kernel(ReduceList l) {
  __shared__ float4 red[256];
  int ji = 0;   // the blocks of a job follow those of the one before it
  for (int k = 1; k < l.n; ++k) ji += (int)blockIdx.x >= l.first[k];
  const ReduceJob& j = l.job[ji];
  const long n_out = (long)j.M * j.N;
  const int lanes = l.lanes[ji], quads = 256 / lanes;   // powers of two
  const int ql = threadIdx.x & (quads - 1), zl = threadIdx.x / quads;
  const long i = ((long)((int)blockIdx.x - l.first[ji]) * quads + ql) * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n_out) {
    const int np = j.nparts;
    for (int z = zl; z < np; z += 4 * lanes) {   // four requests in flight; added in ascending order
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *(const float4*)(j.partial + min(z + u * lanes, np - 1) * j.stride + i);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (z + u * lanes < np) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (zl != 0 || i >= n_out) return;
  for (int k = 1; k < lanes; ++k) {
    const float4 v = red[k * quads + ql];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  if (!ODD) {   // the quad lies in one row of one output
    const int m = (int)(i / j.N), n = (int)(i % j.N);
    float* o = j.o[0];
    long at = i;
    if (j.n_per > 0) {
      const int sel = n / j.n_per;
      o = sel == 0 ? j.o[0] : sel == 1 ? j.o[1] : j.o[2];
      at = (long)m * j.n_per + n % j.n_per;
    }
    if (!o) return;
    o[at] = s.x; o[at + 1] = s.y; o[at + 2] = s.z; o[at + 3] = s.w;   // caller pointers: no alignment assumed
    return;
  }
  const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (i + u >= n_out) break;
    const int m = (int)((i + u) / j.N), n = (int)((i + u) % j.N), sel = j.n_per > 0 ? n / j.n_per : 0;
    float* const o = sel == 0 ? j.o[0] : sel == 1 ? j.o[1] : j.o[2];
    if (o) o[j.n_per > 0 ? (long)m * j.n_per + n % j.n_per : i + u] = v[u];
  }
}
bool reduce_deferrable(int M, int N, int nparts) {
  return N % 4 == 0 && (long)M * N <= 4L * 65536 && (long)M * N * nparts * 4 <= (8L << 20);
}
void reduce_push(ReduceList* l, const float* partial, int nparts, int M, int N, float* o0, float* o1, float* o2, int n_per,
                 long stride) {
  ReduceJob& j = l->job[l->n++];
  j.stride = stride ? stride : (long)M * N;
  j.partial = partial; j.nparts = nparts; j.M = M; j.N = N; j.n_per = n_per;
  j.o[0] = o0; j.o[1] = o1; j.o[2] = o2;
}
void launch_reduce_list(ReduceList& l, hipStream_t st) {
  if (l.n == 0) return;
  int blocks = 0;
  bool odd = false;
  for (int i = 0; i < l.n; ++i) {
    const int np = l.job[i].nparts;
    const long quads = ((long)l.job[i].M * l.job[i].N + 3) / 4;
    int lanes = 16;
    while (lanes < 64 && np > 16 * lanes) lanes *= 2;
    while (lanes > 2 && (lanes / 2 >= np || quads * lanes > 131072)) lanes /= 2;   // 131 072 threads: eight waves per CU
    l.lanes[i] = lanes;
    l.first[i] = blocks;
    const long per = 4 * 256 / l.lanes[i];
    blocks += (int)(((long)l.job[i].M * l.job[i].N + per - 1) / per);
    odd = odd || l.job[i].N % 4 != 0 || l.job[i].n_per % 4 != 0;
  }
  if (odd) hipLaunchKernelGGL(reduce_list_kernel<true>, dim3(blocks), dim3(256), 0, st, l);
  else hipLaunchKernelGGL(reduce_list_kernel<false>, dim3(blocks), dim3(256), 0, st, l);
}

int launch_colsum_multi(const void* const* a, const long* lda, float* const* out, int count, int R, int n, int a_bf16,
                        float* partial, hipStream_t st, ReduceList* defer) {
  ColsumArgs q;
  bool any = false;
  for (int i = 0; i < 4; ++i) {   // count <= 4
    q.a[i] = i < count ? a[i] : nullptr;
    q.lda[i] = i < count ? lda[i] : 0;
    q.out[i] = i < count ? out[i] : nullptr;
    any = any || q.out[i];
  }
  if (!any) return IM_OK;
  const int nblk = (R + CS_ROWS - 1) / CS_ROWS;
  dim3 grid((n + 63) / 64, nblk, count), block(256);
  const int vw = a_bf16 ? 8 : 4;
  bool vec = n % vw == 0 && n / vw <= 256;
  for (int i = 0; i < count; ++i)
    if (q.out[i]) vec = vec && q.lda[i] % vw == 0 && (reinterpret_cast<uintptr_t>(q.a[i]) & 15) == 0;
  if (vec && a_bf16) hipLaunchKernelGGL((colsum_stage1_vec<bf16_t>), dim3(1, nblk, count), block, 0, st, q, R, n, partial);
  else if (vec) hipLaunchKernelGGL((colsum_stage1_vec<float>), dim3(1, nblk, count), block, 0, st, q, R, n, partial);
  else if (a_bf16) hipLaunchKernelGGL((colsum_stage1<bf16_t>), grid, block, 0, st, q, R, n, partial);
  else hipLaunchKernelGGL((colsum_stage1<float>), grid, block, 0, st, q, R, n, partial);
  if (defer && reduce_deferrable(1, n, nblk) && defer->n + count <= 16) {
    for (int i = 0; i < count; ++i)
      if (q.out[i]) reduce_push(defer, partial + (long)i * nblk * n, nblk, 1, n, q.out[i], nullptr, nullptr, 0);
    return IM_OK;
  }
  hipLaunchKernelGGL(colsum_stage2, dim3((n + 15) / 16, 1, count), dim3(256), 0, st, partial, nblk, n, q);
  return IM_OK;
}

// ---- LayerNorm over the feature axis: one wavefront per row, two-pass (mean, then variance) in fp32 ----
template <typename T>
__global__ __launch_bounds__(256) void layernorm_kernel(const T* __restrict__ x, const T* __restrict__ gamma,
                                                        const T* __restrict__ beta, T* __restrict__ y, int R, int d,
                                                        float eps) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const long r = (long)blockIdx.x * 4 + wave;
  if (r >= R) return;
  const T* xr = x + r * d;
  float s = 0.f;
  for (int e = lane; e < d; e += 64) s += ldf(xr + e);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const float mu = s / d;
  float v = 0.f;
  for (int e = lane; e < d; e += 64) { const float t = ldf(xr + e) - mu; v = fmaf(t, t, v); }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const float rstd = rsqrtf(v / d + eps);
  for (int e = lane; e < d; e += 64) stf(y + r * d + e, (ldf(xr + e) - mu) * rstd * ldf(gamma + e) + ldf(beta + e));
}

// eight bf16 (16 bytes) as fp32 and back
__device__ __forceinline__ void unpack8(const uint4& r, float (&v)[8]) {
  const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) { v[2 * j] = __uint_as_float(w[j] << 16); v[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u); }
}
__device__ __forceinline__ uint4 pack8_rne(const float (&v)[8]) {
  unsigned w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j] = (unsigned)f2bf(v[2 * j]) | ((unsigned)f2bf(v[2 * j + 1]) << 16);
  return make_uint4(w[0], w[1], w[2], w[3]);
}
// Rows as 16-byte pieces: LPR lanes (a power of two) share a row, lane i < d / VW holds elements VW i .. VW i + VW - 1, and a
// wave normalises 64 / LPR rows at once (d a multiple of VW = 4 fp32 or 8 bf16 elements, 16-byte aligned rows).  One row per
// wave and one element per lane, the form above, left 24 of 64 lanes idle at d = 40 and asked for a memory round trip per
// row: 33 600 x 40 fp32 9.8 us, 4.0 like this.
template <typename T> struct LnVec { static constexpr int VW = 16 / sizeof(T); };
__device__ __forceinline__ void ln_load(const float* p, float (&v)[4]) {
  const float4 r = *(const float4*)p;
  v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
}
__device__ __forceinline__ void ln_store(float* p, const float (&v)[4]) { *(float4*)p = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void ln_load(const bf16_t* p, float (&v)[8]) { unpack8(*(const uint4*)p, v); }
__device__ __forceinline__ void ln_store(bf16_t* p, const float (&v)[8]) { *(uint4*)p = pack8_rne(v); }
template <int LPR>
__device__ __forceinline__ float ln_rowsum(float v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <typename T, int LPR>
__global__ __launch_bounds__(256) void layernorm_rows_kernel(const T* __restrict__ x, const T* __restrict__ gamma,
                                                             const T* __restrict__ beta, T* __restrict__ y, int R, int d, float eps) {
  constexpr int VW = LnVec<T>::VW, RPW = 64 / LPR;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const long r = ((long)blockIdx.x * 4 + wave) * RPW + lane / LPR;
  const bool in = (lane % LPR) * VW < d;
  const int c = in ? (lane % LPR) * VW : 0;
  const long at = min(r, (long)R - 1) * d + c;
  float v[VW], gm[VW], bt[VW];
  ln_load(x + at, v);
  ln_load(gamma + c, gm);
  ln_load(beta + c, bt);
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < VW; ++j) s += v[j];
  const float mu = ln_rowsum<LPR>(in ? s : 0.f) / d;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < VW; ++j) { const float t = v[j] - mu; q = fmaf(t, t, q); }
  const float rstd = rsqrtf(ln_rowsum<LPR>(in ? q : 0.f) / d + eps);
  if (r >= R || !in) return;
#pragma unroll
  for (int j = 0; j < VW; ++j) v[j] = (v[j] - mu) * rstd * gm[j] + bt[j];
  ln_store(y + at, v);
}
// lanes per row for rows of n 16-byte pieces (0: more than a wave)
static int ln_lanes(int n) { return n <= 8 ? 8 : n <= 16 ? 16 : n <= 32 ? 32 : n <= 64 ? 64 : 0; }
#define LN_LANES(LPR, CALL) \
  do { if (LPR == 8) { CALL(8); } else if (LPR == 16) { CALL(16); } else if (LPR == 32) { CALL(32); } else { CALL(64); } } while (0)

// ---- pieces of the encoder-layer backward ----
__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752440f)); }
// d/dz [z Phi(z)] = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.f + erff(z * 0.70710678118654752440f)) + z * __expf(-0.5f * z * z) * 0.39894228040143267794f;
}
template <typename T>
__global__ void gelu_fwd_kernel(const T* __restrict__ z, T* __restrict__ a, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) stf(a + i, gelu_f(ldf(z + i)));
}
template <typename T>
__global__ void gelu_bwd_kernel(const T* __restrict__ z, T* __restrict__ g, long n) {  // g: da in, dz out
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    stf(g + i, ldf(g + i) * gelu_grad_f(ldf(z + i)));
}
// Phi(x), the standard normal CDF, with erf from Abramowitz & Stegun 7.1.26 (|error| <= 1.5e-7, far below the
// bf16 rounding of the results): a reciprocal, an exp2 and six multiply-adds instead of the library erff.
__device__ __forceinline__ float phi_as_f(float x) {
  const float u = fabsf(x) * 0.70710678118654752440f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, u, 1.f));
  float pl = fmaf(1.061405429f, t, -1.453152027f);
  pl = fmaf(pl, t, 1.421413741f);
  pl = fmaf(pl, t, -0.284496736f);
  pl = fmaf(pl, t, 0.254829592f);
  const float e = pl * t * __builtin_amdgcn_exp2f(-1.44269504088896340736f * u * u);  // 1 - erf(u)
  return x >= 0.f ? 1.f - 0.5f * e : 0.5f * e;
}
__global__ void gelu_fwd8_kernel(const bf16_t* __restrict__ z, bf16_t* __restrict__ a, long n8) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n8; i += (long)gridDim.x * blockDim.x) {
    float v[8];
    unpack8(*(const uint4*)(z + 8 * i), v);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= phi_as_f(v[j]);
    *(uint4*)(a + 8 * i) = pack8_rne(v);
  }
}
__global__ void gelu_bwd8_kernel(const bf16_t* __restrict__ z, bf16_t* __restrict__ g, long n8) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n8; i += (long)gridDim.x * blockDim.x) {
    float v[8], w[8];
    unpack8(*(const uint4*)(z + 8 * i), v);
    unpack8(*(const uint4*)(g + 8 * i), w);
#pragma unroll
    for (int j = 0; j < 8; ++j)   // d/dz [z Phi(z)] = Phi(z) + z phi(z)
      w[j] *= phi_as_f(v[j]) + v[j] * __expf(-0.5f * v[j] * v[j]) * 0.39894228040143267794f;
    *(uint4*)(g + 8 * i) = pack8_rne(w);
  }
}
static bool vec8_ok(const void* a, const void* b, long n) { return n % 8 == 0 && (((uintptr_t)a | (uintptr_t)b) & 15) == 0; }
int launch_gelu_fwd(const void* z, void* a, long n, int bf16, hipStream_t st) {
  if (bf16 && vec8_ok(z, a, n)) {
    const long n8 = n / 8;
    const int blocks8 = (int)((n8 + 255) / 256 < 8192 ? (n8 + 255) / 256 : 8192);
    hipLaunchKernelGGL(gelu_fwd8_kernel, dim3(blocks8), dim3(256), 0, st, (const bf16_t*)z, (bf16_t*)a, n8);
    return IM_OK;
  }
  const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  if (bf16) hipLaunchKernelGGL((gelu_fwd_kernel<bf16_t>), dim3(blocks), dim3(256), 0, st, (const bf16_t*)z, (bf16_t*)a, n);
  else hipLaunchKernelGGL((gelu_fwd_kernel<float>), dim3(blocks), dim3(256), 0, st, (const float*)z, (float*)a, n);
  return IM_OK;
}
int launch_gelu_bwd(const void* z, void* g, long n, int bf16, hipStream_t st) {
  if (bf16 && vec8_ok(z, g, n)) {
    const long n8 = n / 8;
    const int blocks8 = (int)((n8 + 255) / 256 < 8192 ? (n8 + 255) / 256 : 8192);
    hipLaunchKernelGGL(gelu_bwd8_kernel, dim3(blocks8), dim3(256), 0, st, (const bf16_t*)z, (bf16_t*)g, n8);
    return IM_OK;
  }
  const int blocks = (int)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  if (bf16) hipLaunchKernelGGL((gelu_bwd_kernel<bf16_t>), dim3(blocks), dim3(256), 0, st, (const bf16_t*)z, (bf16_t*)g, n);
  else hipLaunchKernelGGL((gelu_bwd_kernel<float>), dim3(blocks), dim3(256), 0, st, (const float*)z, (float*)g, n);
  return IM_OK;
}

// LayerNorm backward of one row per wave: with xhat = (x - mean) * rstd and a = gamma * dy,
//   dx = rstd * (a - mean(a) - xhat * mean(a * xhat)) + res,      t = dy * xhat
// (the column sums of t and dy over all rows are the gradients of gamma and beta).
template <typename T>
__global__ __launch_bounds__(256) void layernorm_bwd_kernel(const T* __restrict__ x, const T* __restrict__ gamma,
                                                            const T* __restrict__ dy, const T* __restrict__ res,
                                                            T* __restrict__ dx, T* __restrict__ t, int R, int d,
                                                            float eps) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const long r = (long)blockIdx.x * 4 + wave;
  if (r >= R) return;
  const T* xr = x + r * d;
  const T* gr = dy + r * d;
  float s = 0.f;
  for (int e = lane; e < d; e += 64) s += ldf(xr + e);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const float mu = s / d;
  float v = 0.f;
  for (int e = lane; e < d; e += 64) { const float c = ldf(xr + e) - mu; v = fmaf(c, c, v); }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const float rstd = rsqrtf(v / d + eps);
  float m1 = 0.f, m2 = 0.f;
  for (int e = lane; e < d; e += 64) {
    const float a = ldf(gamma + e) * ldf(gr + e), xh = (ldf(xr + e) - mu) * rstd;
    m1 += a;
    m2 = fmaf(a, xh, m2);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { m1 += __shfl_xor(m1, o, 64); m2 += __shfl_xor(m2, o, 64); }
  m1 /= d;
  m2 /= d;
  for (int e = lane; e < d; e += 64) {
    const float g = ldf(gr + e), a = ldf(gamma + e) * g, xh = (ldf(xr + e) - mu) * rstd;
    stf(dx + r * d + e, rstd * (a - m1 - xh * m2) + (res ? ldf(res + r * d + e) : 0.f));
    stf(t + r * d + e, g * xh);
  }
}
// The same in 16-byte pieces (see layernorm_rows_kernel), and the column sums with it: a workgroup takes `rows` rows, a
// lane adds g xhat and g of its columns over its rows in fp32, and the block's sums leave as one partial result
// [2][d] (gain, bias).  The next rows are requested before the present ones are used.  Without it the gain's products went
// to memory, rounded to the tensor type, and were read back with dy by two more launches: 33 600 x 40 fp32 15.5 + 4.8 us, 8.0 like this.
template <typename T, int LPR>
__global__ __launch_bounds__(256) void layernorm_bwd_rows_kernel(const T* __restrict__ x, const T* __restrict__ gamma,
                                                                 const T* __restrict__ dy, const T* __restrict__ res,
                                                                 T* __restrict__ dx, float* __restrict__ partial, int R, int d,
                                                                 float eps, int rows) {
  constexpr int VW = LnVec<T>::VW, RPW = 64 / LPR, STEP = 4 * RPW;
  __shared__ float red[4][2][LPR * VW];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const bool in = (lane % LPR) * VW < d;
  const int c = in ? (lane % LPR) * VW : 0;
  const long r0 = (long)blockIdx.x * rows + wave * RPW + lane / LPR;   // rows % STEP == 0
  float gm[VW], sg[VW], sb[VW], xn[VW], gn[VW], rn[VW];
  ln_load(gamma + c, gm);
#pragma unroll
  for (int j = 0; j < VW; ++j) sg[j] = sb[j] = rn[j] = 0.f;
  auto request = [&](long r) {
    const long at = min(r, (long)R - 1) * d + c;
    ln_load(x + at, xn);
    ln_load(dy + at, gn);
    if (res) ln_load(res + at, rn);
  };
  request(r0);
  for (int k = 0; k < rows; k += STEP) {
    const long r = r0 + k;
    float xv[VW], g[VW], rs[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      xv[j] = xn[j];
      g[j] = gn[j];
      rs[j] = rn[j];
    }
    if (k + STEP < rows) request(r + STEP);
    float s = 0.f, q = 0.f, m1 = 0.f, m2 = 0.f, a[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) s += xv[j];
    const float mu = ln_rowsum<LPR>(in ? s : 0.f) / d;
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      xv[j] -= mu;
      q = fmaf(xv[j], xv[j], q);
    }
    const float rstd = rsqrtf(ln_rowsum<LPR>(in ? q : 0.f) / d + eps);
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      xv[j] *= rstd;   // xhat
      a[j] = gm[j] * g[j];
      m1 += a[j];
      m2 = fmaf(a[j], xv[j], m2);
    }
    m1 = ln_rowsum<LPR>(in ? m1 : 0.f) / d;
    m2 = ln_rowsum<LPR>(in ? m2 : 0.f) / d;
    if (r >= R || !in) continue;
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      sg[j] += g[j] * xv[j];
      sb[j] += g[j];
      a[j] = rstd * (a[j] - m1 - xv[j] * m2) + rs[j];
    }
    ln_store(dx + r * d + c, a);
  }
#pragma unroll
  for (int j = 0; j < VW; ++j)
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      sg[j] += __shfl_xor(sg[j], o, 64);
      sb[j] += __shfl_xor(sb[j], o, 64);
    }
  if (lane < LPR)
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      red[wave][0][lane * VW + j] = sg[j];
      red[wave][1][lane * VW + j] = sb[j];
    }
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * d; i += 256) {
    const int w = i >= d, e = i - (w ? d : 0);
    partial[(long)blockIdx.x * 2 * d + i] = (red[0][w][e] + red[1][w][e]) + (red[2][w][e] + red[3][w][e]);
  }
}
// Rows per workgroup: two workgroups per CU, one to sixteen passes of its waves each (layer step at 8 400 x 256 bf16: 245 us
// with 132 workgroups of 64 rows, 227 with 525 of 16).
static int lnb_rows(int R, int lpr) {
  const int step = 4 * (64 / lpr);
  return step * std::max(1, std::min(16, R / (512 * step)));
}
size_t layernorm_bwd_partial_bytes(int R, int d, int bf16) {
  const int vw = bf16 ? 8 : 4, lpr = d % vw == 0 ? ln_lanes(d / vw) : 0;
  size_t n = 2 * colsum_partial_bytes(R, d);   // where the kernel above does not serve the call
  if (lpr) n = std::max(n, (size_t)((R + lnb_rows(R, lpr) - 1) / lnb_rows(R, lpr)) * 2 * d * sizeof(float));
  return n;
}
int launch_layernorm_bwd(const void* x, const void* gamma, const void* dy, const void* res, void* dx, void* t, int R,
                         int d, float eps, int bf16, float* dgamma, float* dbeta, float* partial, ReduceList* red, hipStream_t st) {
  dim3 grid((R + 3) / 4), block(256);
  const uintptr_t al = (uintptr_t)x | (uintptr_t)gamma | (uintptr_t)dy | (uintptr_t)res | (uintptr_t)dx;
  const int vw = bf16 ? 8 : 4, lpr = d % vw == 0 ? ln_lanes(d / vw) : 0;
  if (lpr && (al & 15) == 0) {
    const int rows = lnb_rows(R, lpr), blocks = (R + rows - 1) / rows;
#define LNB_BF16(N) hipLaunchKernelGGL((layernorm_bwd_rows_kernel<bf16_t, N>), dim3(blocks), block, 0, st, (const bf16_t*)x, \
                    (const bf16_t*)gamma, (const bf16_t*)dy, (const bf16_t*)res, (bf16_t*)dx, partial, R, d, eps, rows)
#define LNB_F32(N) hipLaunchKernelGGL((layernorm_bwd_rows_kernel<float, N>), dim3(blocks), block, 0, st, (const float*)x, \
                   (const float*)gamma, (const float*)dy, (const float*)res, (float*)dx, partial, R, d, eps, rows)
    if (bf16) LN_LANES(lpr, LNB_BF16); else LN_LANES(lpr, LNB_F32);
#undef LNB_BF16
#undef LNB_F32
    ReduceList own;
    own.n = 0;
    ReduceList* l = red && red->n + 2 <= 16 ? red : &own;
    if (dgamma) reduce_push(l, partial, blocks, 1, d, dgamma, nullptr, nullptr, 0, 2 * d);
    if (dbeta) reduce_push(l, partial + d, blocks, 1, d, dbeta, nullptr, nullptr, 0, 2 * d);
    launch_reduce_list(own, st);
    return IM_OK;
  }
  if (bf16)
    hipLaunchKernelGGL((layernorm_bwd_kernel<bf16_t>), grid, block, 0, st, (const bf16_t*)x, (const bf16_t*)gamma,
                       (const bf16_t*)dy, (const bf16_t*)res, (bf16_t*)dx, (bf16_t*)t, R, d, eps);
  else
    hipLaunchKernelGGL((layernorm_bwd_kernel<float>), grid, block, 0, st, (const float*)x, (const float*)gamma,
                       (const float*)dy, (const float*)res, (float*)dx, (float*)t, R, d, eps);
  const void* src[2] = {t, dy};
  const long ld2[2] = {d, d};
  float* out[2] = {dgamma, dbeta};
  return launch_colsum_multi(src, ld2, out, 2, R, d, bf16, partial, st, red);
}

int launch_layernorm(const void* x, const void* gamma, const void* beta, void* y, int R, int d, float eps, int bf16,
                     hipStream_t st) {
  dim3 grid((R + 3) / 4), block(256);
  const bool aligned = (((uintptr_t)x | (uintptr_t)y | (uintptr_t)gamma | (uintptr_t)beta) & 15) == 0;
  const int vw = bf16 ? 8 : 4, lpr = d % vw == 0 ? ln_lanes(d / vw) : 0;
  if (lpr && aligned) {
    const int rows_per_block = 4 * (64 / lpr);
    const dim3 g2((R + rows_per_block - 1) / rows_per_block);
#define LN_BF16(N) hipLaunchKernelGGL((layernorm_rows_kernel<bf16_t, N>), g2, block, 0, st, (const bf16_t*)x, (const bf16_t*)gamma, \
                                      (const bf16_t*)beta, (bf16_t*)y, R, d, eps)
#define LN_F32(N) hipLaunchKernelGGL((layernorm_rows_kernel<float, N>), g2, block, 0, st, (const float*)x, (const float*)gamma, \
                                     (const float*)beta, (float*)y, R, d, eps)
    if (bf16) LN_LANES(lpr, LN_BF16); else LN_LANES(lpr, LN_F32);
#undef LN_BF16
#undef LN_F32
    return IM_OK;
  }
  if (bf16)
    hipLaunchKernelGGL((layernorm_kernel<bf16_t>), grid, block, 0, st, (const bf16_t*)x, (const bf16_t*)gamma,
                       (const bf16_t*)beta, (bf16_t*)y, R, d, eps);
  else
    hipLaunchKernelGGL((layernorm_kernel<float>), grid, block, 0, st, (const float*)x, (const float*)gamma,
                       (const float*)beta, (float*)y, R, d, eps);
  return IM_OK;
}

}  // namespace imattn
