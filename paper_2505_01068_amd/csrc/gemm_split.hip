// fp32 GEMMs of the narrow models on the bf16 matrix cores.
//
// An fp32 number is the sum of three bf16 numbers (8 + 8 + 8 significand bits, rounded to nearest; from 2^-110 up: below,
// the last part ends at bf16's smallest number, 2^-133); a product of two of them is taken as x1 y1 + x1 y2 + x2 y1 + x2 y2 +
// x1 y3 + x3 y1, each exact in fp32 and accumulated in fp32.  The dropped terms are below 2^-26 of the product, a quarter of
// an fp32 rounding.  Six 32x32x16 bf16 instructions (15.5 ns
// each) replace eight 32x32x2 fp32 ones (27 ns each, and those take the vector ALU's issue slots).
#include <algorithm>

#include "mfma_common.hpp"

namespace imattn {

// eight fp32 values -> the operands of their three parts
__device__ __forceinline__ void split_parts8(const float (&x)[8], bf16x8 (&out)[3]) {
  float r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = x[i];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[i] = pack_bf16(r[2 * i], r[2 * i + 1]);
      if (k < 2) {
        r[2 * i] -= __uint_as_float(w[i] << 16);
        r[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
      }
    }
    out[k] = as_bf16x8(w);
  }
}
// The large term into `big`, the five small ones into `rest`.  The instruction's rounding is 0.4 to 0.9 units in the last place
// of its largest addend (rms over random sums) and not quite without a sign: its mean is -0.05 units where accumulator and
// products are of one size, -0.01 and less where the accumulator is ten times as large.  All six terms in one accumulator would
// be rounded six times at full size, and a column sum over the rows of the result (a LayerNorm or bias gradient) adds the mean up -- 1.4e-6 instead of 4e-7 relative over 8400 rows.
__device__ __forceinline__ void mfma32_split(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x16& big, f32x16& rest) {
  rest = mfma32(a[2], b[0], rest);
  big = mfma32(a[0], b[0], big);
  rest = mfma32(a[0], b[2], rest);
  rest = mfma32(a[1], b[1], rest);
  rest = mfma32(a[1], b[0], rest);
  rest = mfma32(a[0], b[1], rest);
}

// An infinity, or a finite value beyond bf16's largest (3.39e38), has infinities and NaN among its parts, and NaN is every
// sum that it reaches.  A lane whose sums are not all finite takes those that are not again from memory with fp32
// multiply-adds and stores them over the first ones (one instruction per element for the check; no lane of any ordinary call).
__device__ __forceinline__ unsigned not_finite(const f32x16& a, const f32x16& b) {   // one bit each
  unsigned bad = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = a[r] + b[r];
    bad |= v - v != 0.f ? 1u << r : 0u;
  }
  return bad;
}

// C[M, N] = A[M, K] B[K, N] (+ bias) (GELU) (+ res).  A row-major; B element (k, n) at k sbk + n sbn with one of the two
// strides 1 (BT: sbk == 1), possibly in up to three buffers by columns or by rows of B.
// A workgroup of 4 waves owns 64 rows x 64 columns, a wave 32 x 32.  K is walked in chunks of KS 16-deep k-steps: the
// weight's parts go to LDS in operand order (each wave splits its share), the wave's own 32 rows are read straight into
// the operand layout (lane = row, eight consecutive k) and split in registers.  At 30 000 rows and K = 40 the whole
// kernel is one chunk: one memory round trip, one barrier, 18 matrix instructions per wave; it is bound by that chain
// (a wave waits half of its life) and by launch latency.  64 columns per wave halve the splitting of A but leave fewer
// waves to overlap the chain: QKV projection 12.3 instead of 10.4 us at 29 600 x 40 x 120, out 12.3 instead of 6.6.
// The result has lane = column: a store is 128 contiguous bytes per row, and no alignment or width is required.
// Measured against the kernels it replaced (fp32 matrix instruction with the weight in LDS up to N = K = 128, a 64 x 64
// vector-ALU tile for the rest): QKV 11.8 -> 10.4 us, output projection 8.0 -> 6.6 (29 600 rows, d = 40); MLP products
// at 33 600 x 40 x 160 and 33 600 x 160 x 40: 38 -> 14 .. 16 us; 48 x 32 x 96: 11 -> 4.5 us.
// The weight's column nn (and, with row blocks, row kk) -> its buffer and the index inside it.
__device__ __forceinline__ const float* gs_buffer(const float* b0, const float* b1, const float* b2, int& i, int per) {
  const int sel = (i >= per) + (i >= 2 * per);
  i -= sel * per;
  return sel == 0 ? b0 : sel == 1 ? b1 : b2;
}
constexpr int gs_lds(int ks) { return ks * 2 * 3 * 64; }   // of u32x4
template <int KS, bool BT, bool OCT, bool GELU>
__device__ __forceinline__ void gemm_split_tile(const GemmDesc& g, unsigned bx, unsigned by, u32x4* sB) {
  constexpr int UNITS = KS * 2, UPW = (UNITS + 3) / 4;   // (k-step, 32-column block) units of the weight; per wave
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = lane & 31, h = lane >> 5, wr = wave & 1, wc = wave >> 1;
  const int m0 = bx * 64 + wr * 32, n0 = by * 64;
  const int K = g.K, N = g.N;
  const float* const arow = (const float*)g.A + (long)min(m0 + lo, g.M - 1) * g.sam;
  const int ldw = (int)(BT ? g.sbn : g.sbk);
  const float *const b0 = (const float*)g.B[0], *const b1 = (const float*)g.B[1], *const b2 = (const float*)g.B[2];

  float a[KS][8], w[UPW][8];
  // Requests a chunk.  Nothing here reads what it requests (elements past K are zeroed when the chunk is split): a
  // select on a loaded value between two requests would be a memory round trip.
  auto load = [&](int k0) {
    if (OCT) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const float* const p = arow + min(k0 + 16 * s + 8 * h, K - 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[s][e] = p[e];
      }
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) a[s][e] = arow[min(k0 + 16 * s + 8 * h + e, K - 1)];
    }
#pragma unroll
    for (int i = 0; i < UPW; ++i) {
      const int u = min(4 * i + wave, UNITS - 1);
      const int s = u >> 1, nb = u & 1, k = k0 + 16 * s + 8 * h;
      int nn = min(n0 + nb * 32 + lo, N - 1);
      const float* bp = g.b_split == 1 ? gs_buffer(b0, b1, b2, nn, g.n_per) : b0;
      if (OCT) {
        int kk = min(k, K - 8);
        if (g.b_split == 2) bp = gs_buffer(b0, b1, b2, kk, g.k_per);
        const float* const p = bp + (unsigned)(BT ? nn * ldw + kk : kk * ldw + nn);
#pragma unroll
        for (int e = 0; e < 8; ++e) w[i][e] = p[BT ? e : e * ldw];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          int kk = min(k + e, K - 1);
          const float* const q = g.b_split == 2 ? gs_buffer(b0, b1, b2, kk, g.k_per) : bp;
          w[i][e] = q[BT ? nn * ldw + kk : kk * ldw + nn];
        }
      }
    }
  };
  auto mask = [&](float (&v)[8], int ku) {   // zeros past K (ku: the k-step's first k)
    if (ku + 16 > K)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = ku + 8 * h + e < K ? v[e] : 0.f;
  };
  const int c0 = n0 + wc * 32;
  load(0);
  f32x16 acc, rest;
  {
    int nn = min(c0 + lo, N - 1);
    const float* const bp = g.bias_split ? gs_buffer((const float*)g.bias[0], (const float*)g.bias[1], (const float*)g.bias[2], nn, g.n_per)
                                         : (const float*)g.bias[0];
    const float bv = bp ? bp[nn] : 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[r] = bv;
      rest[r] = 0.f;
    }
  }
  for (int k0 = 0; k0 < K; k0 += 16 * KS) {
    if (k0 > 0) __syncthreads();
#pragma unroll
    for (int i = 0; i < UPW; ++i) {
      const int u = 4 * i + wave;
      if (UNITS % 4 != 0 && u >= UNITS) break;
      bf16x8 p[3];
      mask(w[i], k0 + 16 * (u >> 1));
      split_parts8(w[i], p);
#pragma unroll
      for (int q = 0; q < 3; ++q) sB[(u * 3 + q) * 64 + lane] = __builtin_bit_cast(u32x4, p[q]);
    }
    bf16x8 pa[KS][3];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      mask(a[s], k0 + 16 * s);
      split_parts8(a[s], pa[s]);
    }
    if (k0 + 16 * KS < K) load(k0 + 16 * KS);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bf16x8 b[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) b[q] = as_bf16x8(sB[((s * 2 + wc) * 3 + q) * 64 + lane]);
      mfma32_split(pa[s], b, acc, rest);
    }
  }
  // rows m0 + 8 q + j (+ 4 for the upper lanes): the row's address is scalar, the lane adds its column
  const int n = c0 + lo;
  if (n >= N) return;
  const unsigned off = 4 * h * (unsigned)g.ldc + n;
  const bool all = m0 + 32 <= g.M;
  float rv[16];
  if (g.res)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + 8 * (r >> 2) + (r & 3);
      rv[r] = all || m + 4 * h < g.M ? ((const float*)g.res + m * g.ldc)[off] : 0.f;
    }
  float check = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + 8 * (r >> 2) + (r & 3);
    float v = acc[r] + rest[r];
    check = fmaf(0.f, v, check);
    if (GELU) v = 0.5f * v * (1.f + erff(v * 0.70710678118654752440f));
    if (g.res) v += rv[r];
    if (all || m + 4 * h < g.M) ((float*)g.C[0] + m * g.ldc)[off] = v;
  }
  if (__builtin_expect(check != check, 0)) {
    int nn = n;
    const float* bp = g.bias_split ? gs_buffer((const float*)g.bias[0], (const float*)g.bias[1], (const float*)g.bias[2], nn, g.n_per)
                                   : (const float*)g.bias[0];
    const float bv = bp ? bp[nn] : 0.f;
    nn = n;
    bp = g.b_split == 1 ? gs_buffer(b0, b1, b2, nn, g.n_per) : b0;
    for (unsigned bad = not_finite(acc, rest); bad; bad &= bad - 1) {
      const int r = __builtin_ctz(bad), m = m0 + 8 * (r >> 2) + 4 * h + (r & 3);
      if (m >= g.M) break;
      float v = bv;
      for (int k = 0; k < K && v == v; ++k) {   // (a NaN stays one)
        int kk = k;
        const float* const q = g.b_split == 2 ? gs_buffer(b0, b1, b2, kk, g.k_per) : bp;
        v = fmaf(((const float*)g.A + (long)m * g.sam)[k], q[BT ? nn * ldw + kk : kk * ldw + nn], v);
      }
      if (GELU) v = 0.5f * v * (1.f + erff(v * 0.70710678118654752440f));
      if (g.res) v += ((const float*)g.res + m * g.ldc)[n];
      ((float*)g.C[0] + m * g.ldc)[n] = v;
    }
  }
}

template <int KS, bool BT, bool OCT, bool GELU>
__global__ __launch_bounds__(256, 3) void gemm_split_kernel(GemmDesc g) {
  __shared__ u32x4 sB[gs_lds(KS)];
  gemm_split_tile<KS, BT, OCT, GELU>(g, blockIdx.x, blockIdx.y, sB);
}

bool gemm_split_ok(const GemmDesc& g) {
  return g.split_k <= 1 && g.kb <= 1 && !g.c_split && g.sak == 1 && (g.sbn == 1 || g.sbk == 1);
}
// Octets of k are inside or outside K, and inside one row block of the weight, as a whole: all widths that are
// multiples of 8 (one address and two 16-byte loads per octet).  Both forms in one kernel cost every width the 16-byte
// loads: the compiler merges the two branches' requests into one list of 4-byte loads at computed addresses (QKV
// projection at 29 600 x 40 x 120: 18.4 us instead of 10.4).
static bool gs_oct(const GemmDesc& g) { return g.K % 8 == 0 && (g.b_split != 2 || g.k_per % 8 == 0); }
// k-steps per chunk: one chunk up to K = 64, two up to K = 128 (33 600 x 120 x 40: 10.6 us with two chunks of four
// k-steps, 11.5 with four of two), beyond that short ones (33 600 x 160 x 40: 16 us with chunks of two, 20 with chunks
// of four or five, whose next chunk waits in registers that cost resident waves)
static int gs_ksteps(const GemmDesc& g) {
  const int nk = (g.K + 15) / 16;
  return nk <= 4 ? nk : nk <= 8 ? (nk + 1) / 2 : 2;
}
void launch_gemm_split(const GemmDesc& g, hipStream_t st) {
  const bool bt = g.sbn != 1;
  const bool oct = gs_oct(g);
  const int ks = gs_ksteps(g);
  const dim3 grid((g.M + 63) / 64, (g.N + 63) / 64);
#define GS_LAUNCH(KS, OCT)                                                                                          \
  do {                                                                                                              \
    if (bt && g.gelu) hipLaunchKernelGGL((gemm_split_kernel<KS, true, OCT, true>), grid, dim3(256), 0, st, g);      \
    else if (bt) hipLaunchKernelGGL((gemm_split_kernel<KS, true, OCT, false>), grid, dim3(256), 0, st, g);          \
    else if (g.gelu) hipLaunchKernelGGL((gemm_split_kernel<KS, false, OCT, true>), grid, dim3(256), 0, st, g);      \
    else hipLaunchKernelGGL((gemm_split_kernel<KS, false, OCT, false>), grid, dim3(256), 0, st, g);                 \
  } while (0)
  if (!oct) GS_LAUNCH(4, false);
  else if (ks <= 2) GS_LAUNCH(2, true);
  else if (ks == 3) GS_LAUNCH(3, true);
  else GS_LAUNCH(4, true);
#undef GS_LAUNCH
}

// ---- weight gradients: C[M, N] = A[R, M]^T G[R, N], and the column sums of G (the bias gradient beside it) ----
// The contraction runs over the rows and the operands are read as they lie in memory: lane (c = lane % 32, h) takes
// column c of rows 8 h .. 8 h + 7 of a 16-row step, 128 contiguous bytes per half wave and request.  A workgroup owns a
// 64 x 64 tile of C (blockIdx.y) over its rows (blockIdx.x): each wave requests and splits one 32-column block of A or
// G, the parts meet in LDS in operand order, and a wave multiplies one 32 x 32 block of C.  Partial results leave in
// row-major order and are summed in a fixed order by the reduction list.  Several gradients over the same rows share a
// launch (blockIdx.z).
// Bound: memory for the tall inputs (29 600 rows, [dWq|dWk|dWv] and dWo of d = 40: 28 MB read, 6 MB of partial results
// written, 12.9 us at 4.8 TB/s of copy rate plus a launch; fp32 matrix instructions: 16.5 us.  33 600 rows, all four
// gradients of an encoder layer of 40 x 160: 28 us, the vector-ALU kernel took 38 us each for the two of the MLP; the
// bias gradients cost nothing).  At a few thousand rows a workgroup's chain of steps, 0.5 us each, and the launch: 2850
// rows 5 us (8.2), 9600 rows 7.5 us (6.3, with 75 longer workgroups whose bias gradients were another pair of launches).
// More steps in flight did not help: the chain is splitting, LDS and matrix instructions, not the requests.
typedef u32x4 WgradFrag[2][4][3][64];   // [step parity][A block 0, 1, G block 0, 1][part][lane]
__device__ __forceinline__ void wgrad_split_tile(const WgradSplitList& l, unsigned bx, unsigned by, unsigned bz, WgradFrag& frag) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = lane & 31, h = lane >> 5;
  const WgradSplit& p = l.p[bz];
  const int tm = p.tn_magic ? __umulhi(by, p.tn_magic) : by, tn = by - tm * ((p.N + 63) >> 6);
  if (tm * 64 >= p.M) return;
  // this wave's share of the operands: a 32-column block of A (waves 0, 1) or G (2, 3); and its block of C
  const bool is_g = wave >= 2;
  const int ld = (int)(is_g ? p.ldg : p.lda), width = is_g ? p.N : p.M, x0 = (is_g ? tn : tm) * 64 + (wave & 1) * 32;
  const int m0 = tm * 64 + (wave & 1) * 32, n0 = tn * 64 + (wave >> 1) * 32;
  const bool stage = x0 < width, mine = m0 < p.M && n0 < p.N;
  const int r0 = bx * l.rows, nrows = min(l.rows, l.R - r0), nst = (nrows + 15) >> 4;
  const float* const X = (is_g ? p.G : p.A) + (long)r0 * ld;
  const int col = min(x0 + lo, width - 1);
  const unsigned off = 8 * h * ld + col;
  f32x16 big, rest;
#pragma unroll
  for (int r = 0; r < 16; ++r) big[r] = rest[r] = 0.f;
  float cs = 0.f, v[8];
  auto load = [&](int s) {
    if (16 * s + 16 <= nrows) {   // a whole step: row addresses are scalar, the lane adds a fixed offset
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (X + (long)(16 * s + e) * ld)[off];
    } else {   // the matrix's last rows: rows past the end are read again (and dropped when split)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = X[(long)min(16 * s + 8 * h + e, nrows - 1) * ld + col];
    }
  };
  if (stage) load(0);
  for (int s = 0; s < nst; ++s) {
    if (stage) {
      if (16 * s + 16 > nrows)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 16 * s + 8 * h + e < nrows ? v[e] : 0.f;
      bf16x8 q[3];
      cs += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
      split_parts8(v, q);
#pragma unroll
      for (int k = 0; k < 3; ++k) frag[s & 1][wave][k][lane] = __builtin_bit_cast(u32x4, q[k]);
      if (s + 1 < nst) load(s + 1);
    }
    __syncthreads();   // one per step: the other parity's readers have passed it
    if (mine) {
      bf16x8 pa[3], pg[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        pa[k] = as_bf16x8(frag[s & 1][wave & 1][k][lane]);
        pg[k] = as_bf16x8(frag[s & 1][2 + (wave >> 1)][k][lane]);
      }
      mfma32_split(pa, pg, big, rest);
    }
  }
  if (p.csum && is_g && tm == 0 && x0 + lo < p.N) {
    cs += __shfl_xor(cs, 32);
    if (h == 0) p.csum[(long)bx * ((p.N + 3) & ~3) + x0 + lo] = cs;
  }
  const int n = n0 + lo;
  if (!p.partial || m0 >= p.M || n >= p.N) return;
  float* const out = p.partial + (long)bx * p.stride + n;
  float check = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + 8 * (r >> 2) + 4 * h + (r & 3);
    const float v = big[r] + rest[r];
    check = fmaf(0.f, v, check);
    if (m < p.M) out[m * p.N] = v;
  }
  if (__builtin_expect(check != check, 0)) {
    const float *const A = p.A + (long)r0 * p.lda, *const G = p.G + (long)r0 * p.ldg;
    for (unsigned bad = not_finite(big, rest); bad; bad &= bad - 1) {
      const int r = __builtin_ctz(bad), m = m0 + 8 * (r >> 2) + 4 * h + (r & 3);
      if (m >= p.M) break;
      float v = 0.f;
      for (int i = 0; i < nrows && v == v; ++i) v = fmaf(A[(long)i * p.lda + m], G[(long)i * p.ldg + n], v);
      out[m * p.N] = v;
    }
  }
}

__global__ __launch_bounds__(256, 4) void wgrad_split_kernel(WgradSplitList l) {
  __shared__ WgradFrag frag;
  wgrad_split_tile(l, blockIdx.x, blockIdx.y, blockIdx.z, frag);
}

// The weight gradients and the input gradient dx = G W^T beside them (both read what the attention backward wrote, neither reads
// what the other writes): one launch.  Alone each of them is a chain of memory round trips on workgroups that leave most of the
// chip's issue slots idle; together the launch takes what the longer one takes.  The gradients' workgroups come first, their
// chains are the longer ones.  The product takes chunks of two k-steps at every width (107 registers: four resident workgroups).
// Training step of 9600 x 40 67 -> 62.5 us, 2850 x 40 57.7 -> 53.6, 29 600 x 40 145.2 -> 142.5, layer of 33 600 x 40 x 160 305 -> 297
// (with the product's own chunks and three resident workgroups 62.4, 53.3, 144.5, 303).
__global__ __launch_bounds__(256, 4) void wgrad_dx_split_kernel(WgradSplitList l, GemmDesc g, unsigned ranges, unsigned nw) {
  __shared__ union {
    WgradFrag frag;
    u32x4 sB[gs_lds(2)];
  } lds;
  unsigned id = blockIdx.x, q, r;
  if (id < nw) {
    udivmod(id, ranges, q, r);
    unsigned z, t;
    udivmod(q, l.tiles, z, t);
    wgrad_split_tile(l, __builtin_amdgcn_readfirstlane(r), __builtin_amdgcn_readfirstlane(t), __builtin_amdgcn_readfirstlane(z), lds.frag);
  } else {
    udivmod(id - nw, (g.M + 63) / 64, q, r);
    gemm_split_tile<2, true, true, false>(g, __builtin_amdgcn_readfirstlane(r), __builtin_amdgcn_readfirstlane(q), lds.sB);
  }
}

// Rows per workgroup.  At most 224 row ranges, so that a reduction reads what a few hundred workgroups wrote, and at most
// 2048 workgroups over all the products of the pass, eight per CU: what they write and the reduction reads back is then 34 MB
// at every width (224 ranges alone: 1 GB at d = 256, d_ff = 1024, 33 600 rows, 12 GB at d = 1024; layer step of 29 600 rows at
// d = 256 2540 us with 224, 2310 like this, at d = 512 8500 / 7070, 3 700 rows at d = 1024 5420 / 3320).
// Ranges of at most 2048 rows up to 12 tiles (d = 64, d_ff = 256; below 2 per cent of the tensors of those rows): a sum's
// roundings, one per 16 rows, grow with the square root of its length, dWo of d = 8 over 1 048 560 rows 4.2e-7 with 224 ranges
// of 4 688 rows, 3.0e-7 like this.  (The matrix instruction's rounding has no preferred sign here: with the sums of every
// second range negated every error stays what it was.)
static int wgrad_split_rows(int R, long tiles) {
  const int ranges = (int)std::max(1L, std::min(224L, 2048 / tiles));
  const int rows = std::max(32, ((R + ranges - 1) / ranges + 15) & ~15);
  return tiles <= 12 ? std::min(rows, 2048) : rows;
}
static long wgrad_split_tiles(int M, int N) { return (long)((M + 63) / 64) * ((N + 63) / 64); }
int wgrad_split_rows_attention(int d, int R) { return wgrad_split_rows(R, wgrad_split_tiles(d, d) + wgrad_split_tiles(d, 3 * d)); }
int wgrad_split_rows_layer(int d, int d_ff, int R) {
  return wgrad_split_rows(R, wgrad_split_tiles(d, d) + wgrad_split_tiles(d, 3 * d) + wgrad_split_tiles(d, d_ff) + wgrad_split_tiles(d_ff, d));
}
size_t wgrad_split_bytes(int M, int N, int R, int rows) {
  return (size_t)((R + rows - 1) / rows) * (((long)M * N + 3) / 4 * 4 + (N + 3) / 4 * 4) * sizeof(float);
}
void wgrad_split_push(WgradSplitList* l, int rows, ReduceList* red, const float* A, long lda, const float* G, long ldg, int R, int M,
                      int N, float* partial, int n_per, float* w0, float* w1, float* w2, float* b0, float* b1, float* b2) {
  const bool w = w0 || w1 || w2, b = b0 || b1 || b2;
  if (!w && !b) return;
  WgradSplit& p = l->p[l->n++];
  const int parts = (R + rows - 1) / rows;
  p.A = A; p.G = G; p.lda = lda; p.ldg = ldg; p.M = M; p.N = N;
  p.stride = (int)(((long)M * N + 3) / 4 * 4);
  p.partial = w ? partial : nullptr;
  p.csum = b ? partial + (long)parts * p.stride : nullptr;
  const unsigned tn = (N + 63) / 64, tiles = (M + 63) / 64 * tn;
  p.tn_magic = tn == 1 ? 0u : (unsigned)(((1ull << 32) + tn - 1) / tn);   // t / tn = mulhi(t, magic) for t tn < 2^32; 0: tn is 1
  l->tiles = l->tiles > (int)tiles ? l->tiles : (int)tiles;
  l->R = R;
  l->rows = rows;
  if (w) reduce_push(red, p.partial, parts, M, N, w0, w1, w2, n_per, p.stride);
  if (b) reduce_push(red, p.csum, parts, 1, N, b0, b1, b2, n_per, (N + 3) / 4 * 4);
}
void launch_wgrad_split(const WgradSplitList& l, hipStream_t st) {
  if (l.n == 0) return;
  hipLaunchKernelGGL(wgrad_split_kernel, dim3((l.R + l.rows - 1) / l.rows, l.tiles, l.n), dim3(256), 0, st, l);
}
static bool overlap(const void* a, long na, const void* b, long nb) {   // of fp32 elements
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + 4 * (size_t)nb && y < x + 4 * (size_t)na;
}
// The two launches stay two where dx lies over one of the gradients' operands (dx in place of x or dy: the second launch alone
// writes it), where there is nothing on the list, and at widths that are not multiples of 8: the element-wise form of the product
// needs 154 registers, and three resident workgroups instead of four cost the gradients more than a launch (training step of
// 17 600 x 44 166.6 us in one launch, 159.8 in two; 17 600 x 52 204 / 196).
void launch_wgrad_dx_split(const WgradSplitList& l, const GemmDesc& g, hipStream_t st) {
  bool two = l.n == 0 || !gs_oct(g);
  for (int i = 0; i < l.n; ++i)
    two |= overlap(g.C[0], (long)g.M * g.ldc, l.p[i].A, (long)l.R * l.p[i].lda) || overlap(g.C[0], (long)g.M * g.ldc, l.p[i].G, (long)l.R * l.p[i].ldg);
  const long ranges = l.n ? (l.R + l.rows - 1) / l.rows : 0, nw = ranges * l.tiles * l.n;
  const long wgs = nw + (long)((g.M + 63) / 64) * ((g.N + 63) / 64);
  if (two || wgs >= 1L << 31) {
    launch_wgrad_split(l, st);
    launch_gemm_split(g, st);
    return;
  }
  hipLaunchKernelGGL(wgrad_dx_split_kernel, dim3((unsigned)wgs), dim3(256), 0, st, l, g, (unsigned)ranges, (unsigned)nw);
}

}  // namespace imattn
