// bf16 weight gradients C[M,N] = A[R,M]^T G[R,N] (fp32) of a whole backward pass in one launch, with the column sums of G
// (bias gradients) beside them.
//
// A layer has four such products over the same R token rows; each alone is one launch of a few dozen tiles, plus a launch
// for its bias gradient, plus a reduction.  Here a workgroup is one T x T tile of one product over one range of rows: the
// tiles of all products for a range are neighbours on one XCD (they share operand rows in its L2), and all partial results
// are summed by one reduction.  Both operands are k-major (rows = contraction), copied to LDS asynchronously 64 rows at a
// time into two stages, one in flight while the other is multiplied, and read with the transpose read.
// T = 64 while a product's larger side is at most 256 (a width-64 model: 12 tiles, four workgroups per CU), else 128 (two):
// what bounds both is the L2 -> LDS copy of the operands, 2 T columns for T^2 products per row.
// One gradient after the other, each with a bias gradient and its reductions, took (four products of a layer, or the two of
// an attention) 79 us at d = 64, d_ff = 256, 29 600 rows and takes 17; 124 -> 37 at d = 256, d_ff = 1024, 8 400 rows;
// 58 -> 21 at d = 256, 9 372 rows, attention; 170 (without biases 121) -> 109 at d = 512, 36 864 rows.
#include <algorithm>

#include "mfma_common.hpp"
#include "mfma_path.hpp"

namespace imattn {

constexpr int WK = 64;   // rows of a stage
// Stages that one accumulator sums: it rounds once per 16 rows, and a longer range adds up several of them (dWo of d = 512
// over 1 200 000 rows: 1.4e-6 with ranges of 782 stages in one accumulator, 4.5e-7 like this, 8.8e-7 in the split-K products).
constexpr int WSUM = 80;
template <int T> constexpr int wgrad_lds_bytes() { return 2 * 2 * WK * T * 2; }
// byte offset of chunk c (8 columns) of row k in a [64][T] operand tile
template <int T>
__device__ __forceinline__ int wg_swz(int k, int c) { return (k * (T / 8) + (c ^ (T == 128 ? (k & 3) << 2 : sw_f(k)))) * 16; }

template <int T>
__global__ __launch_bounds__(256, T == 64 ? 4 : 2) void wgrad_ring_kernel(WgradRing l) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int MB = T / 64, CH = T / 32, CPR = T / 8;   // 32-column blocks per wave and side; chunks per thread / per row
  constexpr int OPB = WK * T * 2, STB = 2 * OPB;
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  int bx, by, bz;
  xcd_block_index(bx, by, bz);      // grid (tiles, row ranges)
  int tile = bx, pi = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i) pi += i < l.n && tile >= l.first[i];
  WgradRingItem it = l.item[0];
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (pi == i) it = l.item[i];
  tile -= pi == 0 ? 0 : pi == 1 ? l.first[1] : pi == 2 ? l.first[2] : l.first[3];
  const int tm = tile / it.tiles_n, tn = tile - tm * it.tiles_n;
  const int m0 = tm * T, n0 = tn * T;
  const int kt = (l.R + WK - 1) / WK;
  const int k_begin = by * l.per, n_it = min(kt, k_begin + l.per) - k_begin;   // the launcher makes every range non-empty

  const bf16_t *pa[CH], *pg[CH];
  int krow[CH];
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int slot = (wave * CH + j) * 64 + lane, k = slot / CPR, c = (slot % CPR) ^ (T == 128 ? (k & 3) << 2 : sw_f(k));
    krow[j] = k;
    pa[j] = it.A + min(m0 + c * 8, it.M - 8);
    pg[j] = it.G + min(n0 + c * 8, it.N - 8);
  }
  auto issue = [&](int i) {
    char* base = smem + (i & 1) * STB;
    const int r0 = (k_begin + i) * WK;
#pragma unroll
    for (int j = 0; j < CH; ++j) dma16(pa[j] + (long)min(r0 + krow[j], l.R - 1) * it.lda, base + (wave * CH + j) * 1024);
#pragma unroll
    for (int j = 0; j < CH; ++j) dma16(pg[j] + (long)min(r0 + krow[j], l.R - 1) * it.ldg, base + OPB + (wave * CH + j) * 1024);
  };
  // the lane's transpose-read offsets in an operand tile at k = 0 (first four rows; a k-step of 16 rows and the second four
  // rows are constants on top, except for the swizzle of T = 64, which changes by one bit)
  const int tj = lane & 15, tg = lane >> 4, tkr = 8 * (tg >> 1) + (tj >> 2), tcol = 16 * (tg & 1) + 4 * (tj & 3);
  auto frag = [&](const char* op, int s, int col0) -> bf16x8 {
    const int col = col0 + tcol, k = tkr;
    typedef v4i16 __attribute__((address_space(3))) * lds_v4_ptr;
    union { v4i16 h[2]; bf16x8 v; } f;
    f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(op + s * 16 * T * 2 + wg_swz<T>(k, col >> 3) + (col & 7) * 2));
    f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(op + s * 16 * T * 2 + wg_swz<T>(k + 4, col >> 3) + (col & 7) * 2));
    return f.v;
  };

  issue(0);
  f32x16 acc[MB][MB];   // [n block][m block]
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
  f32x16 total[MB][MB];   // of whole runs of WSUM stages
  auto fold = [&](bool first) {
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < MB; ++b) {
        total[a][b] = first ? acc[a][b] : total[a][b] + acc[a][b];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
      }
  };
  // column sums of G: a thread adds one column pair over its share of a stage's rows, in fp32 on the vector ALU
  constexpr int PAIRS = T / 2, RG = 256 / PAIRS, RPG = WK / RG;
  const bool sums = it.sums && tm == 0;
  const int cp = tid % PAIRS, rg = tid / PAIRS;
  float s0 = 0.f, s1 = 0.f;

  for (int i = 0; i < n_it; ++i) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (i + 1 < n_it) issue(i + 1);
    char* st = smem + (i & 1) * STB;
    const int left = l.R - (k_begin + i) * WK;
    if (left < WK) {   // the last stage of the last range: its rows past the end are copies, both operands' become zero
      for (int c = tid; c < 2 * WK * CPR; c += 256)
        if (c / CPR % WK >= left) *(u32x4*)(st + c * 16) = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      bf16x8 fa[MB], fg[MB];
#pragma unroll
      for (int x = 0; x < MB; ++x) {
        fa[x] = frag(st, s, (wm * MB + x) * 32);
        fg[x] = frag(st + OPB, s, (wn * MB + x) * 32);
      }
#pragma unroll
      for (int nb = 0; nb < MB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = mfma32(fg[nb], fa[mb], acc[nb][mb]);
    }
    if (i % WSUM == WSUM - 1 && i + 1 < n_it) fold(i < WSUM);
    if (sums) {
      const char* g = st + OPB;
#pragma unroll
      for (int r = 0; r < RPG; ++r) {
        const int k = rg * RPG + r;
        const unsigned v = *(const unsigned*)(g + wg_swz<T>(k, cp >> 2) + (cp & 3) * 4);
        s0 += __uint_as_float(v << 16);
        s1 += __uint_as_float(v & 0xffff0000u);
      }
    }
  }
  if (n_it > WSUM)
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < MB; ++b) acc[a][b] += total[a][b];
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();   // every wave has finished reading the last stage
  asm volatile("" ::: "memory");

  float* const out = it.partial + (long)by * it.stride;
  // 32 rows at a time through the wave's share of the ring, 16 bytes per lane and whole row segments of the wave
  constexpr int WC = 32 * MB, EP_LD = WC + 4, LPR = WC / 4;
  static_assert(4 * 32 * EP_LD * 4 <= wgrad_lds_bytes<T>(), "the staging areas lie in the ring");
  float* stg = (float*)smem + wave * (32 * EP_LD);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int nb = 0; nb < MB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(float4*)(stg + lo * EP_LD + nb * 32 + 8 * i + 4 * hi) =
            make_float4(acc[nb][mb][4 * i], acc[nb][mb][4 * i + 1], acc[nb][mb][4 * i + 2], acc[nb][mb][4 * i + 3]);
    asm volatile("" ::: "memory");   // the wave's LDS accesses execute in order; the compiler must keep them so across lanes
    const int n = n0 + wn * WC + lane % LPR * 4;
#pragma unroll
    for (int t = 0; t < 32 * LPR / 64; ++t) {
      const int r = lane / LPR + t * (64 / LPR), m = m0 + (wm * MB + mb) * 32 + r;
      const float4 v = *(const float4*)(stg + r * EP_LD + lane % LPR * 4);
      if (m < it.M && n < it.N) *(float4*)(out + (long)m * it.N + n) = v;   // M % 8 == N % 8 == 0
    }
    asm volatile("" ::: "memory");
  }
  if (sums) {
    __syncthreads();
    float* red = (float*)smem;   // [RG][T]
    red[rg * T + 2 * cp] = s0;
    red[rg * T + 2 * cp + 1] = s1;
    __syncthreads();
    if (tid < T && n0 + tid < it.N) {
      float s = red[tid];
      for (int k = 1; k < RG; ++k) s += red[k * T + tid];
      out[(long)it.M * it.N + n0 + tid] = s;
    }
  }
}

static int wg_tile(const int (&mn)[4][2], int n) {
  int side = 0;
  for (int i = 0; i < n; ++i) side = std::max(side, std::max(mn[i][0], mn[i][1]));
  return side <= 256 ? 64 : 128;
}
// Row ranges: as many workgroups as are resident at once (512 at T = 128; 512 of 1024 at T = 64, where twice as many ranges
// double the partial results), at least 4 stages each, and of tall inputs as many whole rounds of workgroups as ranges of 80
// stages make, but no more partial results than the split-K products of the same gradients would take (attention of d = 512
// at 1 075 200 rows: 4.54 GB of workspace, 5.32 with ranges of 80 stages throughout; step at 300 000 rows 3 940 -> 3 830 us).
static WgradPlan wgrad_ring_plan(const int (&mn)[4][2], int n, int R) {
  WgradPlan p;
  p.T = wg_tile(mn, n);
  p.tiles = 0;
  for (int i = 0; i < n; ++i) p.tiles += ((mn[i][0] + p.T - 1) / p.T) * ((mn[i][1] + p.T - 1) / p.T);
  const int kt = (R + WK - 1) / WK;
  const int want = std::max(1, 512 / p.tiles);
  p.per = std::min(WSUM, std::max(std::min(4, kt), (kt + want - 1) / want));
  double split = 0, all = 0;
  for (int i = 0; i < n; ++i) {
    split += (double)mfma_gemm_split(mn[i][0], mn[i][1], R) * mn[i][0] * mn[i][1];
    all += (double)(mn[i][0] + 1) * mn[i][1];
  }
  const int most = want * std::max(1, (int)(split / all) / want);
  p.per = std::max(p.per, (kt + most - 1) / most);
  p.z = (kt + p.per - 1) / p.per;
  return p;
}
WgradPlan wgrad_ring_plan_attention(int d, int R) {
  const int mn[4][2] = {{d, d}, {d, 3 * d}};
  return wgrad_ring_plan(mn, 2, R);
}
WgradPlan wgrad_ring_plan_layer(int d, int d_ff, int R) {
  const int mn[4][2] = {{d, d}, {d, 3 * d}, {d, d_ff}, {d_ff, d}};
  return wgrad_ring_plan(mn, 4, R);
}
size_t wgrad_ring_bytes(const WgradPlan& p, int M, int N) { return (size_t)p.z * ((size_t)M * N + N) * sizeof(float); }

void wgrad_ring_push(WgradRing* l, const WgradPlan& p, ReduceList* red, const void* A, long lda, const void* G, long ldg, int M, int N,
                     float* partial, int n_per, float* w0, float* w1, float* w2, float* b0, float* b1, float* b2) {
  const bool w = w0 || w1 || w2, b = b0 || b1 || b2;
  if (!w && !b) return;
  WgradRingItem& it = l->item[l->n];
  it.A = (const bf16_t*)A; it.G = (const bf16_t*)G; it.lda = lda; it.ldg = ldg; it.M = M; it.N = N;
  it.tiles_n = (N + p.T - 1) / p.T;
  it.partial = partial; it.stride = (long)M * N + N; it.sums = b;
  l->first[l->n++] = l->tiles;
  l->tiles += (M + p.T - 1) / p.T * it.tiles_n;
  if (w) reduce_push(red, partial, p.z, M, N, w0, w1, w2, n_per, it.stride);
  if (b) reduce_push(red, partial + (long)M * N, p.z, 1, N, b0, b1, b2, n_per, it.stride);
}
void launch_wgrad_ring(WgradRing& l, const WgradPlan& p, int R, hipStream_t st) {
  if (l.n == 0) return;
  l.R = R; l.per = p.per;
  const dim3 grid(l.tiles, p.z);
  if (p.T == 64) hipLaunchKernelGGL((wgrad_ring_kernel<64>), grid, dim3(256), wgrad_lds_bytes<64>(), st, l);
  else hipLaunchKernelGGL((wgrad_ring_kernel<128>), grid, dim3(256), wgrad_lds_bytes<128>(), st, l);
}

}  // namespace imattn
