// IM attention inference for the smallest fp32 calls, projections included, in ONE launch.
//
// A sample of a few dozen rows is three dependent launches of 4 to 5 us (Q|K|V projection, attention, output projection), each of
// them launch latency, a memory round trip and a barrier on a handful of workgroups; the arithmetic is some 10^5 multiply-adds.
// Here a workgroup owns 8 query rows of a sample.  It projects the K and V rows of ALL keys its segment reads (up to 40) for
// itself -- the redundant products cost less than a launch -- then its own Q rows, takes the softmax with eight lanes per (row,
// head), and projects the output: one round trip to memory in front, one store behind, everything between in LDS and registers.
// 2 x 8/8/8 rows, d = 32, 4 heads: 14.5 -> 9 us, of which the launch is about a third.
//
// The projections sum in 64 bits (a multiply-add costs what it costs in 32, and plain fp32 sums are less exact than the three
// launches' matrix-core ones: relative error at d = 32, 16 keys 1.46e-7 with fp32 sums, 0.97e-7 so, 1.17e-7 in three launches); the
// rest is fp32.  The score is (scale log2(e) q) . k in the exponent of 2, the softmax subtracts the row's maximum.  Masked and dead
// keys are not read into any sum.
#include "common.hpp"

namespace imattn {

constexpr int TINY_ROWS = 8, TINY_KEYS = 40, TINY_D = 32, TINY_THREADS = 512;   // of a workgroup: query rows, keys at most,
                                                                                   // padded width, threads

// the weights' columns a thread multiplies by: all requests of a column before its first use; zeros from the width on (the last
// row again would do for finite weights, but its infinity times the operand's 0 is NaN)
__device__ __forceinline__ void load_col(const float* w, int d, int c, float (&out)[TINY_D]) {
#pragma unroll
  for (int k = 0; k < TINY_D; ++k) out[k] = w[(long)min(k, d - 1) * d + c];
#pragma unroll
  for (int k = 0; k < TINY_D; ++k) out[k] = k < d ? out[k] : 0.f;
}
// x . w + b in 64 bits, rounded once (x holds zeros from the width on)
template <typename W>
__device__ __forceinline__ float dot_row(const double* x, const W (&w)[TINY_D], float b) {
  double a[4] = {b, 0., 0., 0.};
#pragma unroll
  for (int k = 0; k < TINY_D; k += 4)
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = fma(x[k + e], (double)w[k + e], a[e]);
  return (float)((a[0] + a[1]) + (a[2] + a[3]));
}

struct TinyArgs {
  const float *x, *w[4], *b[4], *res;
  float* y;
  const int32_t* valid_len;
  const uint8_t* key_pad;
  int tile0[IM_MAX_SEG + 1];   // first tile of a segment
};

// DHP: the head dimension, padded to 4, 8 or 16
template <int DHP>
__global__ __launch_bounds__(TINY_THREADS) void tiny_fwd_kernel(Geo g, TinyArgs p) {
  constexpr int DP = TINY_D, LD = DP + 4, NT = TINY_THREADS;
  __shared__ __attribute__((aligned(16))) double sX[TINY_KEYS][DP], sQX[TINY_ROWS][DP], sO[TINY_ROWS][DP];   // (fp32 values)
  __shared__ float sK[TINY_KEYS][LD], sV[TINY_KEYS][LD], sQ[TINY_ROWS][LD];
  __shared__ int sRow[TINY_KEYS];   // the key's row in the tensor, or -1 - row if it is masked
  const int tid = threadIdx.x, b = blockIdx.y, tile = blockIdx.x, d = g.d, dh = g.dh;
  int seg = 0;
#pragma unroll
  for (int s = 1; s < IM_MAX_SEG; ++s)
    if ((s < g.n_seg) & (tile >= p.tile0[s])) seg = s;
  const int q0 = (tile - p.tile0[seg]) * TINY_ROWS, qlen = seg_rows(g, b, seg);
  if (q0 >= qlen) return;   // packed rows: the batch element's segment ends before the tile
  const long qrow0 = seg_row0(g, b, seg) + q0;
  // the keys: the valid rows of the live segments, one after the other
  int nk = 0;
  for (int j = 0; j < g.n_seg; ++j) {
    if (!((g.q_live[seg] >> j) & 1u)) continue;
    int n = seg_rows(g, b, j);
    if (p.valid_len) n = min(n, max(0, p.valid_len[b * g.n_seg + j]));
    n = min(n, TINY_KEYS - nk);   // (the launcher has checked the lengths)
    const long r0 = seg_row0(g, b, j);
    if (tid < n) sRow[nk + tid] = (int)(p.key_pad && p.key_pad[r0 + tid] != 0 ? -1 - (r0 + tid) : r0 + tid);
    nk += n;
  }
  // columns of this thread: K|V (2 d of them), Q and the output
  constexpr int CKV = 2 * DP, GKV = NT / CKV, GQ = NT / DP;   // groups of threads that have all columns
  const int ckv = tid % CKV, c1 = tid % DP;
  const bool is_v = ckv >= DP;
  const int ck = min(is_v ? ckv - DP : ckv, d - 1), cq = min(c1, d - 1);
  float wkv[DP], wq[DP], wo[DP];
  load_col(is_v ? p.w[2] : p.w[1], d, ck, wkv);
  load_col(p.w[0], d, cq, wq);
  load_col(p.w[3], d, cq, wo);
  const float* const bkv_p = is_v ? p.b[2] : p.b[1];
  const float bkv = bkv_p ? bkv_p[ck] : 0.f, bq = p.b[0] ? p.b[0][cq] : 0.f, bo = p.b[3] ? p.b[3][cq] : 0.f;
  double wkv64[DP];   // used for several rows
#pragma unroll
  for (int k = 0; k < DP; ++k) wkv64[k] = wkv[k];
  __syncthreads();   // sRow
  for (int i = tid; i < (nk + TINY_ROWS) * DP; i += NT) {
    const int r = i / DP, c = i % DP;
    const bool key = r < nk;
    const int kr = key ? sRow[r] : 0;
    const long row = key ? (long)(kr < 0 ? -1 - kr : kr) : qrow0 + min(r - nk, qlen - 1 - q0);
    const float v = p.x[row * d + min(c, d - 1)];
    (key ? &sX[r][0] : &sQX[r - nk][0])[c] = c < d ? (double)v : 0.;
  }
  __syncthreads();
  if (tid < GKV * CKV)
    for (int r = tid / CKV; r < nk; r += GKV) (is_v ? sV : sK)[r][is_v ? ckv - DP : ckv] = dot_row(sX[r], wkv64, bkv);
  if (tid < GQ * DP)
    for (int r = tid / DP; r < TINY_ROWS; r += GQ) sQ[r][c1] = dot_row(sQX[r], wq, bq) * g.scale_log2e;
  for (int i = tid; i < TINY_ROWS * DP; i += NT) sO[i / DP][i % DP] = 0.;
  __syncthreads();
  // softmax: eight lanes per (row, head), every eighth key each
  const int l8 = tid & 7;
  for (int pair = tid >> 3; pair < TINY_ROWS * g.H; pair += NT / 8) {
    const int r = pair & (TINY_ROWS - 1), hc = (pair / TINY_ROWS) * dh;
    float q[DHP], acc[DHP], s[TINY_KEYS / 8];
#pragma unroll
    for (int e = 0; e < DHP; ++e) {
      q[e] = e < dh ? sQ[r][hc + e] : 0.f;
      acc[e] = 0.f;
    }
    float m = IM_NEG_INF, l = 0.f;
#pragma unroll
    for (int u = 0; u < TINY_KEYS / 8; ++u) {
      const int k = l8 + 8 * u;
      s[u] = IM_NEG_INF;
      if (k < nk && sRow[k] >= 0) {
        float v = 0.f;
#pragma unroll
        for (int e = 0; e < DHP; ++e) v = fmaf(q[e], e < dh ? sK[k][hc + e] : 0.f, v);
        s[u] = v;
        m = fmaxf(m, v);
      }
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
    const float ms = m == IM_NEG_INF ? 0.f : m;
#pragma unroll
    for (int u = 0; u < TINY_KEYS / 8; ++u) {
      const int k = l8 + 8 * u;
      if (k < nk && sRow[k] >= 0) {
        const float pk = __builtin_amdgcn_exp2f(s[u] - ms);
        l += pk;
#pragma unroll
        for (int e = 0; e < DHP; ++e) acc[e] = fmaf(pk, e < dh ? sV[k][hc + e] : 0.f, acc[e]);
      }
    }
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      l += __shfl_xor(l, o);
#pragma unroll
      for (int e = 0; e < DHP; ++e) acc[e] += __shfl_xor(acc[e], o);
    }
    const float inv = l > 0.f ? 1.f / l : l != l ? l : 0.f;   // no key: 0; a NaN stays one
    if (l8 == 0)
#pragma unroll
      for (int e = 0; e < DHP; ++e)
        if (e < dh) sO[r][hc + e] = acc[e] * inv;
  }
  __syncthreads();
  if (tid >= GQ * DP) return;
  for (int r = tid / DP; r < TINY_ROWS && q0 + r < qlen; r += GQ) {
    const float v = dot_row(sO[r], wo, bo);
    const long at = (qrow0 + r) * d + c1;
    if (c1 < d) p.y[at] = v + (p.res ? p.res[at] : 0.f);
  }
}

// Whether the call goes to the kernel above: fp32, width up to 32, head dimension up to 16, every query segment reads at most 40
// rows, and the workgroups have a CU each.  Every workgroup repeats the projections of its keys, whose cost grows with their number
// and the square of the width: us of a call, three launches / one, at d = 32 with 16 keys 16.3 / 9.9 (2 to 80 samples alike),
// 40 keys 15.7 / 11.9, 64 keys 16.4 / 14.8 with 4 heads but 15.9 / 19.0 with 32; in a form of 64 columns, at d = 40 with 40 keys
// 16.1 / 16.8 and at d = 48 with 60 keys 16.3 / 21.4.  The line at width 32 is that of the one form there is, not of the method: a
// form of 40 columns takes 11.4 at d = 40 with 16 keys and 14.5 with 40 (16.3 and 17.2 in three launches), but 253 registers, and
// 10 to 15 % more at d = 32.
// y must not overlap x: a workgroup reads rows of x that another one has finished.
bool tiny_fwd_ok(const Geo& g, const void* x, const void* y) {
  if (g.d > TINY_D || g.dh > 16) return false;
  long tiles = 0;
  for (int i = 0; i < g.n_seg; ++i) {
    long keys = 0;
    for (int j = 0; j < g.n_seg; ++j)
      if ((g.q_live[i] >> j) & 1u) keys += g.seg_len[j];
    if (keys > TINY_KEYS) return false;
    tiles += (g.seg_len[i] + TINY_ROWS - 1) / TINY_ROWS;
  }
  const size_t bytes = (size_t)g.R * g.d * sizeof(float);
  const uintptr_t a = (uintptr_t)x, c = (uintptr_t)y;
  return tiles * g.B <= cu_count() && g.R < (1L << 30) && (a + bytes <= c || c + bytes <= a);
}
void launch_tiny_fwd(const Geo& g, const void* x, const void* const (&w)[4], const void* const (&b)[4], const int32_t* valid_len,
                     const uint8_t* key_pad, void* y, const void* res, hipStream_t st) {
  TinyArgs p;
  p.x = (const float*)x; p.y = (float*)y; p.res = (const float*)res;
  p.valid_len = valid_len; p.key_pad = key_pad;
  for (int i = 0; i < 4; ++i) { p.w[i] = (const float*)w[i]; p.b[i] = (const float*)b[i]; }
  p.tile0[0] = 0;
  for (int i = 0; i < g.n_seg; ++i) p.tile0[i + 1] = p.tile0[i] + (g.seg_len[i] + TINY_ROWS - 1) / TINY_ROWS;
  const dim3 grid(p.tile0[g.n_seg], g.B);
  ProfScope ps(PF_ATTN_FWD, st);
  if (g.dh <= 4) hipLaunchKernelGGL((tiny_fwd_kernel<4>), grid, dim3(TINY_THREADS), 0, st, g, p);
  else if (g.dh <= 8) hipLaunchKernelGGL((tiny_fwd_kernel<8>), grid, dim3(TINY_THREADS), 0, st, g, p);
  else hipLaunchKernelGGL((tiny_fwd_kernel<16>), grid, dim3(TINY_THREADS), 0, st, g, p);
}

}  // namespace imattn
