// IM attention for small head dimensions (dh <= 16) in fp32 arithmetic on the bf16 matrix cores.
//
// The multimodal-sentiment shapes have head dimension 5..8 and fp32 tensors.  gfx950's fp32 matrix instructions run at
// the vector ALU's rate and do not overlap with it (measured: 16x16x4 f32 13.5 ns, plus 1.25 ns for every vector
// instruction beside it), so fp32 products gain nothing there; the bf16 instruction 16x16x32 takes 7.8 ns for 32 times
// the products per k and runs beside the vector ALU.  Every operand is therefore written as the sum of THREE bf16
// numbers, which holds all 24 bits of an fp32 significand exactly (from 2^-110 up), and a product x y is the sum of the products of
// parts, each exact in fp32, accumulated in fp32:
//   scores:  x y = x1 y1 + x1 y2 + x1 y3 + x2 y1 + x2 y2 + x3 y1.  With round-to-nearest parts |x2| <= 2^-9 |x|,
//            |x3| <= 2^-18 |x|: the three dropped terms are below 2^-26 |x y|, a quarter of an fp32 rounding.  The
//            contraction over dh is so short that the six terms of all dh columns lie side by side in the 32 k-slots of
//            ONE instruction (dh <= 5; two for dh <= 10).
//   P V:     the three parts of V's columns are rows of the A operand (3 dh <= 16 rows: one instruction for all three),
//            and the probabilities' three parts are three B operands.
// One slot of the score product is left for the key mask (1 on the query side, 0 or -inf on the key side), one row of
// the P V product is all ones (the row sum).  The score has the same bits in all three kernels: the product starts from zero
// (the reference or lse is subtracted from its result) and has the same terms in the same slots, whichever side is the A
// operand.  So exp2(score - lse) is the forward's probability to a rounding of lse.  With -m and -lse as the accumulator's
// start (eight subtractions less per step) each kernel rounded the score in its own way: at scores around 300 the
// probability of a row's only key was off by 1e-5 and dWv with it (3.0e-6 like this, 1.1e-5 so), at 1e6 dWv by 20 %.
//
// Bound: vector-instruction issue.  Per score the forward has one subtraction, one exp2, half a max and 5.5 instructions that
// split the probability (71 per 32 x 16 step and wave, five matrix instructions beside them), dQ two and dK/dV eight more;
// at 32 x 50/500/375 rows, 8 heads of 5, the counters showed the vector ALUs two thirds busy, the rest is the latency of a
// workgroup's own prologue.  The kernels before these (one query or key row per lane, fused multiply-adds, the other
// operand broadcast from LDS) needed 10 to 20 multiply-adds and four LDS broadcasts per score: forward / dQ / dK/dV
// 42 / 49 / 61 us at that shape against 28 / 32 / 41, 13 / 16 / 16 us at 64 x 50/50/50 rows against 8 / 9 / 12.
//
// Lane layout of v_mfma_f32_16x16x32_bf16, lane l, g = l / 16: A row l % 16 / B column l % 16, k = 8 g .. 8 g + 7;
// C/D column l % 16, register r = row 4 g + r.  A step is 32 rows of the streamed operand: row u of a step is row
// m = 4 (u / 8) + u % 4 of score block (u / 4) % 2, so that a lane's eight scores of the two blocks are rows
// 8 g .. 8 g + 7 of the step -- exactly the k-slots it supplies to the next product.  No score leaves its lane.
//
// A workgroup (4 waves) owns a tile of 64 rows of one modality segment, 16 per wave; it streams the rows of the
// segments that the Interlaced Mask leaves live (Sec. 6 "Decomposition"), trimmed to the valid length, in chunks that
// all four waves share, with one running reference and sum per row across all of them (joint row softmax, Sec.
// "Information Disorder").
#include <limits.h>

#include <type_traits>

#include "mfma_common.hpp"

namespace imattn {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Kernels are instantiated for head dimensions 4, 5, 6, 8, 10, 12, 16; a smaller one is padded with zero columns.
template <int DH>
struct SplitCfg {
  static constexpr int NS = (6 * DH + 1 + 31) / 32;     // k-steps of a score product (six terms per column, mask slot)
  static constexpr int NT = (3 * DH + 15) / 16;         // 16-row blocks of the transposed operand's parts
  static constexpr int NT1 = (3 * DH + 1 + 15) / 16;    // the same with the row of ones
  static constexpr int BLK = NS * 64 + 8;               // 16-byte units of a 16-row score-operand block; the 8 spread
                                                        // the two blocks of a step over the banks (writer's side)
};
constexpr float SPLIT_MASKED = -__builtin_inff();   // mask slot of a key that must not be attended: whatever the key's row holds
constexpr float SPLIT_LAZY = 8.f;         // the softmax reference moves when a score exceeds it by 2^8

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// the upper halves of two floats as a pair of bf16 (lo in the low half)
__device__ __forceinline__ unsigned top_pair(float lo, float hi) {
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ float top_of(float x) { return __uint_as_float(__float_as_uint(x) & 0xffff0000u); }

// x = p[0] + p[1] + p[2], each a bf16 value (low half zero) rounded to nearest
template <int DH>
__device__ __forceinline__ void split_rows(const float (&x)[DH], float (&p)[3][DH]) {
  float r[DH];
#pragma unroll
  for (int e = 0; e < DH; ++e) r[e] = x[e];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < DH; e += 2) {
      const unsigned u = pack_bf16(r[e], e + 1 < DH ? r[e + 1] : 0.f);
      p[k][e] = __uint_as_float(u << 16);
      r[e] -= p[k][e];
      if (e + 1 < DH) {
        p[k][e + 1] = __uint_as_float(u & 0xffff0000u);
        r[e + 1] -= p[k][e + 1];
      }
    }
}

// The query row as the score product takes it: one fp32 value per column in every kernel.  (Contracted with the subtraction
// in split_rows, the product's own rounding error would enter the second part, in some kernels and not in others.)
template <int DH>
__device__ __forceinline__ void scale_row(float (&x)[DH], float by) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < DH; ++e) x[e] = x[e] * by;
}

// position of streamed row t of a chunk: 16-row score block, row inside it
__device__ __forceinline__ void step_pos(int t, int& blk, int& m) {
  blk = 2 * (t >> 5) + ((t >> 2) & 1);
  m = 4 * ((t & 31) >> 3) + (t & 3);
}

// Score operand of one row: slot s = DH term + column holds part {0,0,0,1,1,2}[term] on the query side and
// {0,1,2,0,1,0}[term] on the key side; slot 6 DH holds `mask`.  neg: the row enters with the other sign.
template <int DH, bool QSIDE>
__device__ __forceinline__ void store_score_row(u32x4* S, int blk, int m, const float (&p)[3][DH], float mask, bool neg = false) {
  using C = SplitCfg<DH>;
  constexpr int QP[6] = {0, 0, 0, 1, 1, 2}, KP[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
  for (int q = 0; q < 4 * C::NS; ++q) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int s = 8 * q + 2 * i + k;
        v[k] = s < 6 * DH ? p[QSIDE ? QP[s / DH] : KP[s / DH]][s % DH] : s == 6 * DH ? mask : 0.f;
      }
      w[i] = top_pair(v[0], v[1]) ^ (neg ? 0x80008000u : 0u);
    }
    S[blk * C::BLK + (q >> 2) * 64 + (q & 3) * 16 + m] = w;
  }
}
template <int DH>
__device__ __forceinline__ bf16x8 score_frag(const u32x4* S, int blk, int s, int lane) {
  return as_bf16x8(S[blk * SplitCfg<DH>::BLK + s * 64 + lane]);
}

// Transposed operand of one row: column r of the row's 16 NTB columns holds part r / DH of head column r % DH, column
// 3 DH the value one (ONES).  Stored [step][16-column block][32 rows][16]; read back transposed.  The rows of odd steps
// are stored with the other sign (see accumulate_tr), those with neg once more.
template <int DH, int NTB, bool ONES>
__device__ __forceinline__ void store_tr_row(bf16_t* Tr, int blk, int m, const float (&p)[3][DH], bool neg = false) {
  const unsigned flip = neg != ((blk & 2) != 0) ? 0x80008000u : 0u;
#pragma unroll
  for (int q = 0; q < 2 * NTB; ++q) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int r = 8 * q + 2 * i + k;
        v[k] = r < 3 * DH ? p[r / DH][r % DH] : (ONES && r == 3 * DH) ? 1.f : 0.f;
      }
      w[i] = top_pair(v[0], v[1]) ^ flip;
    }
    *(u32x4*)(Tr + ((((blk >> 1) * NTB + (q >> 1)) * 32 + (blk & 1) * 16 + m) << 4) + (q & 1) * 8) = w;
  }
}
// A operand: row lane % 16 of column block rb, k = the lane's eight rows of step st (ds_read_b64_tr_b16: see
// lds_frag_tr for the exchange inside a group of 16 lanes)
template <int NTB>
__device__ __forceinline__ bf16x8 tr_frag(const bf16_t* Tr, int st, int rb, int lane) {
  const int j = lane & 15, g = lane >> 4;
  const bf16_t* p = Tr + (((st * NTB + rb) * 32 + 4 * g + (j >> 2)) << 4) + 4 * (j & 3);
  typedef v4i16 __attribute__((address_space(3))) * lds_v4_ptr;
  union { v4i16 h[2]; bf16x8 v; } x;
  x.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p));
  x.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_ptr)(p + 256));
  return x.v;
}

// eight fp32 values as three B operands whose sum is exact: 8 + 8 + 8 bits by truncation
__device__ __forceinline__ void split8(const float (&v)[8], bf16x8 (&out)[3]) {
  float r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = v[i];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = top_pair(r[2 * i], r[2 * i + 1]);
    out[k] = as_bf16x8(w);
    if (k < 2)
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] -= top_of(r[i]);
  }
}
// part k of the streamed side against column block rb of the transposed operand: not needed where it would only
// multiply that operand's third parts by a second or third part (below 2^-24 of the product)
template <int DH>
__host__ __device__ constexpr bool tr_needed(int k, int rb, bool ones) {
  return k == 0 || ones || rb * 16 < 2 * DH;
}
// acc += the step's product.  The three parts' instructions start from zero and the step's sum is added with a rounding to
// nearest: the instruction's own rounding, 0.6 to 0.9 units of its largest addend (rms), would be three per step at the
// accumulator's size, and its mean is below zero (0.05 units where accumulator and products are of one size).  What the step's own products lose that way has
// one sign too, and the bias gradients add it over all rows: odd steps multiply the operand with the other sign and are
// subtracted, which turns the rounding around (the dQ and dK/dV kernels do the same to dP between odd and even query
// rows).  Without, dbq was off by 2.4e-6 at 20 x 39/480/461 rows.  Segments of up to 32 rows have one step each: the dK/dV
// kernel, whose results no other sign turns around, sums them with the other sign in every second batch element and tile;
// without, dbv was off by 3.2e-7 at 200 x 10/30/25 rows (1.9e-7 with, fp32 multiply-adds 2.4e-7).
template <int DH, int NTB, bool ONES>
__device__ __forceinline__ void accumulate_tr(const bf16_t* Tr, int st, const bf16x8 (&b)[3], f32x4 (&acc)[NTB], int lane) {
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb) {
    const bf16x8 a = tr_frag<NTB>(Tr, st, rb, lane);
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 2; k >= 0; --k)
      if (tr_needed<DH>(k, rb, ONES && rb == NTB - 1)) x = mfma16(a, b[k], x);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[rb][i] = fmaf(x[i], (st & 1) ? -1.f : 1.f, acc[rb][i]);
  }
}

// The head's dh values of one row (p = the row's first column of the head), zero beyond dh.  Every load is issued, none
// sits behind a branch per element; with EXACT (dh == DH) they merge into 16-byte loads.
template <typename T, int DH, bool EXACT>
__device__ __forceinline__ void load_head_row(const T* p, int dh, float (&out)[DH]) {
  if (EXACT) {
#pragma unroll
    for (int e = 0; e < DH; ++e) out[e] = ldf(p + e);
  } else {
    float v[DH];
#pragma unroll
    for (int e = 0; e < DH; ++e) v[e] = ldf(p + (e < dh ? e : 0));
#pragma unroll
    for (int e = 0; e < DH; ++e) out[e] = e < dh ? v[e] : 0.f;
  }
}

// One side (query tiles or key tiles) of a problem, by value.  Kept small and indexed statically: an array of kernel
// arguments indexed at run time is one scalar-memory round trip per access, and the short workgroups of these shapes
// would spend most of their life in them.
struct SplitGeo {
  int H, dh, n_seg, T, pair0, pairs;   // the launch's (batch element, head) pairs: first one, number
  unsigned h_magic;                    // pair / H = mulhi(pair, h_magic); 0: divide
  int tile0[IM_MAX_SEG], seg[IM_MAX_SEG];   // k-th segment of the tile order: its first tile (INT_MAX: none), its index
  unsigned live[IM_MAX_SEG];           // ... and the segments of the other side that it meets
  int len[IM_MAX_SEG], off[IM_MAX_SEG];     // by segment
  float scale, scale_log2e;
  long R;
  const int32_t* cu;                   // packed rows (see Geo)
};
__device__ __forceinline__ int pick(const int (&a)[IM_MAX_SEG], int i) {
  int v = a[0];
#pragma unroll
  for (int k = 1; k < IM_MAX_SEG; ++k) v = i == k ? a[k] : v;
  return v;
}
// Rows of segment s of batch element b: number, first row of the [rows, .] tensors, first element of the per-row
// statistics of head h.
struct SplitRows { int n; long row0, stat0; };
__device__ __forceinline__ SplitRows split_rows_of(const SplitGeo& g, int b, int h, int s) {
  SplitRows r;
  if (g.cu) {
    const int c0 = __builtin_amdgcn_readfirstlane(g.cu[b * g.n_seg + s]), c1 = __builtin_amdgcn_readfirstlane(g.cu[b * g.n_seg + s + 1]);
    r.n = c1 - c0;
    r.row0 = c0;
    r.stat0 = (long)h * g.R + c0;
  } else {
    const int off = pick(g.off, s);
    r.n = pick(g.len, s);
    r.row0 = (long)b * g.T + off;
    r.stat0 = ((long)b * g.H + h) * g.T + off;
  }
  return r;
}
// Workgroup -> tile: grid (8 ceil(pairs / 8), tiles).  x % 8 is the XCD: each takes a contiguous range of (batch
// element, head) pairs, so that the heads of a batch element, whose columns share cache lines, meet in one L2; tiles
// run in the order of decreasing work.  false: no such rows.
constexpr int SPLIT_ROWS = 64;    // rows of a tile, and streamed rows of a chunk
struct SplitTile { int b, h, nrows, vlen; unsigned live; long row0, stat0; };   // vlen: valid rows from the tile's first one
__device__ __forceinline__ bool find_tile(const SplitGeo& g, int tile_base, const int32_t* valid_len, SplitTile& t) {
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3, per = g.pairs >> 3, rem = g.pairs & 7;
  const unsigned pair = g.pair0 + xcd * per + min(xcd, rem) + idx;
  t.b = g.h_magic ? __umulhi(pair, g.h_magic) : pair / g.H;
  t.h = pair - t.b * g.H;
  const int tile = blockIdx.y + tile_base;
  int first = 0, s = g.seg[0];
  t.live = g.live[0];
#pragma unroll
  for (int k = 1; k < IM_MAX_SEG; ++k)
    if (tile >= g.tile0[k]) {
      first = g.tile0[k];
      s = g.seg[k];
      t.live = g.live[k];
    }
  if (idx >= per + (xcd < rem)) return false;
  const SplitRows r = split_rows_of(g, t.b, t.h, s);
  const int r0 = (tile - first) * SPLIT_ROWS;
  t.nrows = min(SPLIT_ROWS, r.n - r0);
  t.vlen = valid_len ? __builtin_amdgcn_readfirstlane(valid_len[t.b * g.n_seg + s]) - r0 : t.nrows;
  t.row0 = r.row0 + r0;
  t.stat0 = r.stat0 + r0;
  return t.nrows > 0;   // packed rows: the batch element's segment may end before the tile
}

// Walks the chunks of the live segments: rows row0 .. row0 + n - 1 (valid_len: of the streamed side, or null).
struct SplitWalk {
  unsigned live;
  int left, n;        // rows of the segment from the chunk's first one; rows of the chunk
  long row0, stat0;
  __device__ __forceinline__ SplitWalk(unsigned lv) : live(lv), left(0), n(0), row0(0), stat0(0) {}
  __device__ __forceinline__ bool next(const SplitGeo& g, int b, int h, const int32_t* valid_len) {
    left -= n;
    row0 += n;
    stat0 += n;
    while (left <= 0) {
      if (!live) return false;
      const int j = __builtin_ctz(live);
      live &= live - 1;
      const SplitRows r = split_rows_of(g, b, h, j);
      left = valid_len ? min(r.n, __builtin_amdgcn_readfirstlane(valid_len[b * g.n_seg + j])) : r.n;
      row0 = r.row0;
      stat0 = r.stat0;
    }
    n = min(SPLIT_ROWS, left);
    return true;
  }
};

// Per wave, the 16 x (16 NTB) result block of a transposed product through LDS: lane (column n = lane % 16, first head
// column lane / 16) reads the parts' sums.  X: 16 (16 NTB + 4) floats of the wave.
template <int NTB>
__device__ __forceinline__ void spill_acc(float* X, const f32x4 (&acc)[NTB], int lane) {
  const int n = lane & 15, g = lane >> 4;
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb) *(f32x4*)(X + n * (16 * NTB + 4) + 16 * rb + 4 * g) = acc[rb];
}
template <int DH, int NTB>
__device__ __forceinline__ float part_sum(const float* X, int n, int e) {
  const float* x = X + n * (16 * NTB + 4);
  return (x[2 * DH + e] + x[DH + e]) + x[e];
}
template <int NTB>
__host__ __device__ constexpr int spill_units() { return 16 * (16 * NTB + 4); }   // 16-byte units, four waves

constexpr int cmax(int a, int b) { return a > b ? a : b; }

// ---- rows that the three-part products cannot give ----
// An infinity, or a finite value beyond bf16's largest (3.39e38), has NaN among its parts, and NaN is every result that it
// reaches.  A row whose result is NaN or infinite is computed again from memory in plain fp32 multiply-adds, one row per wave
// and one row of the streamed operand per lane (no row of any ordinary call).  Rows whose own operands hold a NaN that makes
// every term NaN (padding rows of NaN, a diverged training step) get NaN at once, all of them together (a training step of
// 29 600 rows of NaN: 197 us, 2555 us with every row by itself).
// Such rows of the wave (row = lane % 16), one bit each.  check: the sum of zero times every value of the lane's accumulators.
__device__ __forceinline__ unsigned not_finite(float check, bool in) {
  unsigned long long b = __builtin_amdgcn_ballot_w64(check != check && in);
  if (__builtin_expect(b == 0, 1)) return 0u;
  b |= b >> 32;
  return (unsigned)((b | b >> 16) & 0xffffu);
}
template <int NTB>
__device__ __forceinline__ float check_acc(const f32x4 (&acc)[NTB], float check) {
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) check = fmaf(0.f, acc[rb][i], check);
  return check;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
template <int DH>
__device__ __forceinline__ float dot_from(float s, const float (&a)[DH], const float (&b)[DH]) {
#pragma unroll
  for (int e = 0; e < DH; ++e) s = fmaf(a[e], b[e], s);
  return s;
}

// The wave's rows of X (first row of the tile, first column of the head) that hold a NaN, one bit each; and their result.
template <typename T, int DH, bool EXACT>
__device__ __forceinline__ unsigned nan_rows(const T* X, long ld, int row0, int nrows, int dh) {
  const int lane = threadIdx.x & 63;
  bool nan = false;
  if (lane < 16 && row0 + lane < nrows) {
    float x[DH];
    load_head_row<T, DH, EXACT>(X + (row0 + lane) * ld, dh, x);
#pragma unroll
    for (int e = 0; e < DH; ++e) nan = nan || x[e] != x[e];
  }
  return (unsigned)__builtin_amdgcn_ballot_w64(nan);
}
template <typename T>
__device__ __forceinline__ void put_rows(unsigned rows, T* X, long ld, int row0, int dh, float v) {
  const int lane = threadIdx.x & 63;
  if (lane < 16 && ((rows >> lane) & 1))
    for (int e = 0; e < dh; ++e) stf(X + (row0 + lane) * ld + e, v);
}

// Output row `row` of the tile (wave-uniform).
template <typename T, int DH, bool EXACT>
__device__ __forceinline__ void plain_fwd_row(const SplitGeo& g, const SplitTile& t, int row, int dh, const T* Q, const T* K, const T* V,
                                              long ld, const int32_t* valid_len, const uint8_t* key_pad, T* O, long ldo,
                                              float* lse2) {
  const int lane = threadIdx.x & 63, hc = t.h * dh;
  float q[DH], acc[DH], m = IM_NEG_INF, l = 0.f;
  load_head_row<T, DH, EXACT>(Q + (t.row0 + row) * ld + hc, dh, q);
  scale_row<DH>(q, g.scale_log2e);
#pragma unroll
  for (int e = 0; e < DH; ++e) acc[e] = 0.f;
  SplitWalk walk(t.live);
  while (walk.next(g, t.b, t.h, valid_len)) {
    if (lane >= walk.n) continue;
    const long r = walk.row0 + lane;
    float k[DH], v[DH];
    load_head_row<T, DH, EXACT>(K + r * ld + hc, dh, k);
    load_head_row<T, DH, EXACT>(V + r * ld + hc, dh, v);
    const float s = dot_from<DH>(key_pad && key_pad[r] != 0 ? IM_NEG_INF : 0.f, q, k);
    const float mn = fmaxf(s, m), ms = mn == IM_NEG_INF ? 0.f : mn;
    const float alpha = __builtin_amdgcn_exp2f(m - ms), p = __builtin_amdgcn_exp2f(s - ms);
    l = l * alpha + p;
#pragma unroll
    for (int e = 0; e < DH; ++e) acc[e] = fmaf(p, v[e], acc[e] * alpha);
    m = mn;
  }
  float mw = m;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mw = fmaxf(mw, __shfl_xor(mw, o));
  const float ms = mw == IM_NEG_INF ? 0.f : mw, alpha = __builtin_amdgcn_exp2f(m - ms);
  l = wave_sum(l * alpha);
  const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
  for (int e = 0; e < DH; ++e) {
    const float v = wave_sum(acc[e] * alpha) * inv;
    if (lane == 0 && e < dh) stf(O + (t.row0 + row) * ldo + hc + e, v);
  }
  if (lse2 && lane == 0) lse2[t.stat0 + row] = l > 0.f ? mw + log2f(l) : IM_NEG_INF;
}

// A wave owns 16 rows of the tile.  Waves 0 and 1 stage a chunk (one matrix each), the others the tile's own rows, which
// go to LDS beside the first chunk: one memory round trip and one barrier before the first product.  Two 16-row blocks
// per wave (128-row tiles, 128-row chunks: half the staging per score) measured the same at 500-row segments and a
// quarter slower at 50-row ones.
template <typename T, int DH, bool EXACT>
__global__ __launch_bounds__(256, DH > 5 ? 2 : 5)
void split_fwd_kernel(SplitGeo g, int tile_base, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                      long ld, const int32_t* __restrict__ valid_len, const uint8_t* __restrict__ key_pad,
                      T* __restrict__ O, long ldo, float* __restrict__ lse2) {
  using F = SplitCfg<DH>;
  constexpr int NS = F::NS, NTB = F::NT1;
  constexpr int S_UNITS = 4 * F::BLK, T_UNITS = 2 * NTB * 64;
  constexpr int CH = S_UNITS + T_UNITS;   // one chunk; two of them, the second one first holds the own rows
  __shared__ u32x4 smem[cmax(2 * CH, spill_units<NTB>())];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SplitTile t;
  if (!find_tile(g, tile_base, nullptr, t)) return;
  const int dh = EXACT ? DH : g.dh, hc = t.h * dh;

  float raw[DH], part[3][DH];
  unsigned char pad = 0;
  SplitWalk walk(t.live);
  auto request = [&]() {
    if (wave < 2 && lane < ((walk.n + 31) & ~31)) {
      const int r = min(lane, walk.n - 1);
      load_head_row<T, DH, EXACT>((wave ? V : K) + walk.row0 * ld + hc + r * (int)ld, dh, raw);
      pad = key_pad && !wave ? key_pad[walk.row0 + r] : (unsigned char)0;
    }
  };
  auto store = [&](u32x4* buf, int n) {
    if (wave < 2 && lane < ((n + 31) & ~31)) {
      const bool in = lane < n;
#pragma unroll
      for (int e = 0; e < DH; ++e) raw[e] = in ? raw[e] : 0.f;
      split_rows<DH>(raw, part);
      int blk, mm;
      step_pos(lane, blk, mm);
      if (wave) store_tr_row<DH, NTB, true>((bf16_t*)(buf + S_UNITS), blk, mm, part);
      else store_score_row<DH, false>(buf, blk, mm, part, in && pad == 0 ? 0.f : SPLIT_MASKED);
    }
  };
  if (wave == 3) load_head_row<T, DH, EXACT>(Q + t.row0 * ld + hc + min(lane, t.nrows - 1) * (int)ld, dh, raw);
  bool more = walk.next(g, t.b, t.h, valid_len);
  if (more) request();
  if (wave == 3) {
    scale_row<DH>(raw, g.scale_log2e);
    split_rows<DH>(raw, part);
    store_score_row<DH, true>(smem + CH, lane >> 4, lane & 15, part, 1.f);
  }
  if (more) store(smem, walk.n);
  __syncthreads();
  bf16x8 bq[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) bq[s] = score_frag<DH>(smem + CH, wave, s, lane);
  const bool active = wave * 16 < t.nrows;

  f32x4 acc[NTB];
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb) acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = 0.f;
  int thr = INT_MIN;   // bits of the exponent from which the reference moves; INT_MIN: the row has no reference yet
  auto steps = [&](const u32x4* sS, int nst) {
    const bf16_t* const sT = (const bf16_t*)(sS + S_UNITS);
    for (int st = 0; st < nst; ++st) {
      f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        x0 = mfma16(score_frag<DH>(sS, 2 * st, s, lane), bq[s], x0);
        x1 = mfma16(score_frag<DH>(sS, 2 * st + 1, s, lane), bq[s], x1);
      }
      float e[8];   // score - m
      int big = INT_MIN;   // as integers: exact above 0, where the threshold lies, and no NaN canonicalisation
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        e[i] = x0[i] - m;
        e[4 + i] = x1[i] - m;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) big = max(big, __float_as_int(e[i]));
      // rare: no reference yet (>=: a score of -0.0 has the bits of INT_MIN), or a score 2^8 above it
      if (__builtin_amdgcn_ballot_w64(big >= thr)) {
        float mx = x0[0];
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, fmaxf(x0[i], x1[i]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const bool unset = thr == INT_MIN, move = unset ? mx > IM_NEG_INF : mx - m > SPLIT_LAZY;
        const float to = move ? mx : m;
        const float alpha = __builtin_amdgcn_exp2f(unset ? 0.f : m - to);
#pragma unroll
        for (int rb = 0; rb < NTB; ++rb) acc[rb] *= alpha;
        m = to;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[i] = x0[i] - m;
          e[4 + i] = x1[i] - m;
        }
        thr = move ? __float_as_int(SPLIT_LAZY) : thr;
      }
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(e[i]);
      bf16x8 bp[3];
      split8(p, bp);
      accumulate_tr<DH, NTB, true>(sT, st, bp, acc, lane);
    }
  };
  if (!more) __syncthreads();   // no key at all: the own rows have been read before the results take their place
  for (int cur = 0; more; ++cur) {
    const int nst = (walk.n + 31) >> 5;
    more = walk.next(g, t.b, t.h, valid_len);
    if (more) request();
    if (active) steps(smem + (cur & 1) * CH, nst);
    if (more) {
      if (cur == 0) __syncthreads();   // the own rows have been read (afterwards: the buffer was, before the last barrier)
      store(smem + (~cur & 1) * CH, walk.n);
    }
    __syncthreads();
  }
  if (!active) return;
  float* X = (float*)(smem + wave * (spill_units<NTB>() / 4));
  const int n = lane & 15, e0 = lane >> 4, row = wave * 16 + n;
  spill_acc<NTB>(X, acc, lane);
  unsigned bad = not_finite(check_acc<NTB>(acc, 0.f), row < t.nrows);
  __builtin_amdgcn_wave_barrier();
  const float l = X[n * (16 * NTB + 4) + 3 * DH];
  const float inv = l > 0.f ? 1.f / l : 0.f;
  if (row < t.nrows && !((bad >> n) & 1)) {
    T* const o = O + t.row0 * ldo + hc + row * (int)ldo;
#pragma unroll
    for (int i = 0; i < (DH + 3) / 4; ++i) {
      const int e = e0 + 4 * i;
      if (e < dh) stf(o + e, part_sum<DH, NTB>(X, n, e) * inv);
    }
    if (lse2 && e0 == 0) lse2[t.stat0 + row] = l > 0.f ? m + __log2f(l) : IM_NEG_INF;
  }
  if (__builtin_expect(bad == 0, 1)) return;
  const unsigned nan = bad & nan_rows<T, DH, EXACT>(Q + t.row0 * ld + hc, ld, wave * 16, t.nrows, dh);
  put_rows(nan, O + t.row0 * ldo + hc, ldo, wave * 16, dh, __builtin_nanf(""));
  if (lse2 && lane < 16 && ((nan >> lane) & 1)) lse2[t.stat0 + row] = IM_NEG_INF;
  for (bad &= ~nan; bad; bad &= bad - 1)
    plain_fwd_row<T, DH, EXACT>(g, t, wave * 16 + __builtin_ctz(bad), dh, Q, K, V, ld, valid_len, key_pad, O, ldo, lse2);
}

template <typename T, int DH, bool EXACT>
__device__ __forceinline__ void plain_dq_row(const SplitGeo& g, const SplitTile& t, int row, int dh, const T* Q, const T* K, const T* V,
                                             long ld, const T* O, const T* dO, long ldo, const float* lse2,
                                             const int32_t* valid_len, const uint8_t* key_pad, float* delta, T* dQ, long ldg) {
  const int lane = threadIdx.x & 63, hc = t.h * dh;
  float q[DH], go[DH], acc[DH];
  load_head_row<T, DH, EXACT>(O + (t.row0 + row) * ldo + hc, dh, q);
  load_head_row<T, DH, EXACT>(dO + (t.row0 + row) * ldo + hc, dh, go);
  const float dl = dot_from<DH>(0.f, go, q);
  load_head_row<T, DH, EXACT>(Q + (t.row0 + row) * ld + hc, dh, q);
  scale_row<DH>(q, g.scale_log2e);
#pragma unroll
  for (int e = 0; e < DH; ++e) acc[e] = 0.f;
  float ls = lse2[t.stat0 + row];
  if (ls == IM_NEG_INF) ls = -IM_NEG_INF;
  SplitWalk walk(t.live);
  while (walk.next(g, t.b, t.h, valid_len)) {
    if (lane >= walk.n) continue;
    const long r = walk.row0 + lane;
    float k[DH], v[DH];
    load_head_row<T, DH, EXACT>(K + r * ld + hc, dh, k);
    load_head_row<T, DH, EXACT>(V + r * ld + hc, dh, v);
    const float s = dot_from<DH>(key_pad && key_pad[r] != 0 ? IM_NEG_INF : 0.f, q, k);
    const float ds = __builtin_amdgcn_exp2f(s - ls) * (dot_from<DH>(0.f, go, v) - dl);
#pragma unroll
    for (int e = 0; e < DH; ++e) acc[e] = fmaf(ds, k[e], acc[e]);
  }
#pragma unroll
  for (int e = 0; e < DH; ++e) {
    const float v = wave_sum(acc[e]) * g.scale;
    if (lane == 0 && e < dh) stf(dQ + (t.row0 + row) * ldg + hc + e, v);
  }
  if (lane == (row & 15)) delta[t.stat0 + row] = (row & 1) ? -dl : dl;   // the lane that has stored it before
}

// dQ (and delta = rowsum(dO * O)): own rows are queries, keys are streamed.
// delta comes from the matrix cores with the operand order of dP = dO V^T, so that a row with a single key (O = V bit
// for bit) has dP - delta = 0 exactly.  Odd query rows carry -dO: their dP, delta (stored so) and dS have the other sign.
template <typename T, int DH, bool EXACT>
__global__ __launch_bounds__(256, DH > 5 ? 2 : 4)
void split_dq_kernel(SplitGeo g, int tile_base, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                     long ld, const T* __restrict__ O, const T* __restrict__ dO, long ldo, const float* __restrict__ lse2,
                     const int32_t* __restrict__ valid_len, const uint8_t* __restrict__ key_pad, float* __restrict__ delta,
                     T* __restrict__ dQ, long ldg) {
  using F = SplitCfg<DH>;
  constexpr int NS = F::NS, NTB = F::NT;
  constexpr int S_UNITS = 4 * F::BLK, T_UNITS = 2 * NTB * 64;
  // Two chunks (K, V, K transposed); the second one first holds the own rows: Q, dO, O.  At the largest head dimension
  // O takes Q's place once Q has been read, so that two workgroups fit a CU.
  constexpr bool O_LATE = DH > 12;
  constexpr int CH = 2 * S_UNITS + T_UNITS, O_AT = O_LATE ? 0 : 2 * S_UNITS;
  __shared__ u32x4 smem[cmax(CH + cmax(CH, (O_LATE ? 2 : 3) * S_UNITS), spill_units<NTB>())];
  u32x4* const sOwn = smem + CH;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SplitTile t;
  if (!find_tile(g, tile_base, nullptr, t)) return;
  const int dh = EXACT ? DH : g.dh, hc = t.h * dh;

  float raw[DH], raw2[DH], part[3][DH];
  unsigned char pad = 0;
  SplitWalk walk(t.live);
  auto request = [&]() {
    if (wave < 2 && lane < ((walk.n + 31) & ~31)) {
      const int r = min(lane, walk.n - 1);
      load_head_row<T, DH, EXACT>((wave ? V : K) + walk.row0 * ld + hc + r * (int)ld, dh, raw);
      pad = key_pad && !wave ? key_pad[walk.row0 + r] : (unsigned char)0;
    }
  };
  auto store = [&](u32x4* buf, int n) {
    if (wave < 2 && lane < ((n + 31) & ~31)) {
      const bool in = lane < n;
#pragma unroll
      for (int e = 0; e < DH; ++e) raw[e] = in ? raw[e] : 0.f;
      split_rows<DH>(raw, part);
      int blk, mm;
      step_pos(lane, blk, mm);
      store_score_row<DH, false>(buf + (wave ? S_UNITS : 0), blk, mm, part, wave || (in && pad == 0) ? 0.f : SPLIT_MASKED);
      if (!wave) store_tr_row<DH, NTB, false>((bf16_t*)(buf + 2 * S_UNITS), blk, mm, part);
    }
  };
  {
    const int r = min(lane, t.nrows - 1);
    if (wave == 2) load_head_row<T, DH, EXACT>(dO + t.row0 * ldo + hc + r * (int)ldo, dh, raw);
    if (wave == 3) {
      load_head_row<T, DH, EXACT>(Q + t.row0 * ld + hc + r * (int)ld, dh, raw);
      load_head_row<T, DH, EXACT>(O + t.row0 * ldo + hc + r * (int)ldo, dh, raw2);
    }
  }
  float ls = lse2[t.stat0 + min(wave * 16 + (lane & 15), t.nrows - 1)];
  bool more = walk.next(g, t.b, t.h, valid_len);
  const bool keys = more;
  if (more) request();
  if (wave >= 2) {
    if (wave == 3) scale_row<DH>(raw, g.scale_log2e);
    split_rows<DH>(raw, part);
    store_score_row<DH, true>(sOwn + (wave == 2 ? S_UNITS : 0), lane >> 4, lane & 15, part, wave == 2 ? 0.f : 1.f,
                              wave == 2 && (lane & 1));
    if (wave == 3 && !O_LATE) {
      split_rows<DH>(raw2, part);
      store_score_row<DH, false>(sOwn + O_AT, lane >> 4, lane & 15, part, 0.f);
    }
  }
  if (more) store(smem, walk.n);
  __syncthreads();
  const bool active = wave * 16 < t.nrows;
  const int n = lane & 15, row = wave * 16 + n;
  bf16x8 bq[NS], bg[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    bq[s] = score_frag<DH>(sOwn, wave, s, lane);
    bg[s] = score_frag<DH>(sOwn + S_UNITS, wave, s, lane);
  }
  if (O_LATE) {
    __syncthreads();
    if (wave == 3) {
      split_rows<DH>(raw2, part);
      store_score_row<DH, false>(sOwn + O_AT, lane >> 4, lane & 15, part, 0.f);
    }
    __syncthreads();
  }
  f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) x = mfma16(score_frag<DH>(sOwn + O_AT, wave, s, lane), bg[s], x);
  // the diagonal: row n of column n sits in register n % 4 of lane group n / 4
  const float diag = (n & 2) ? ((n & 1) ? x[3] : x[2]) : ((n & 1) ? x[1] : x[0]);
  const float dl = __shfl(diag, 16 * (n >> 2) + n);
  if (lane < 16 && row < t.nrows) delta[t.stat0 + row] = dl;
  ls = ls == IM_NEG_INF ? -IM_NEG_INF : ls;   // row with no live valid key: every p becomes 0
  f32x4 acc[NTB];
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb) acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto steps = [&](const u32x4* sK, int nst) {
    const u32x4* const sV = sK + S_UNITS;
    const bf16_t* const sT = (const bf16_t*)(sK + 2 * S_UNITS);
    for (int st = 0; st < nst; ++st) {
      f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0, y0 = x0, y1 = x0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        x0 = mfma16(score_frag<DH>(sK, 2 * st, s, lane), bq[s], x0);
        x1 = mfma16(score_frag<DH>(sK, 2 * st + 1, s, lane), bq[s], x1);
        y0 = mfma16(score_frag<DH>(sV, 2 * st, s, lane), bg[s], y0);
        y1 = mfma16(score_frag<DH>(sV, 2 * st + 1, s, lane), bg[s], y1);
      }
      float ds[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ds[i] = __builtin_amdgcn_exp2f(x0[i] - ls) * (y0[i] - dl);
        ds[4 + i] = __builtin_amdgcn_exp2f(x1[i] - ls) * (y1[i] - dl);
      }
      bf16x8 bd[3];
      split8(ds, bd);
      accumulate_tr<DH, NTB, false>(sT, st, bd, acc, lane);
    }
  };
  if (!more) __syncthreads();   // no key at all: the own rows have been read before the results take their place
  for (int cur = 0; more; ++cur) {
    const int nst = (walk.n + 31) >> 5;
    more = walk.next(g, t.b, t.h, valid_len);
    if (more) request();
    if (active) steps(smem + (cur & 1) * CH, nst);
    if (more) {
      if (cur == 0) __syncthreads();   // the own rows have been read (afterwards: the buffer was, before the last barrier)
      store(smem + (~cur & 1) * CH, walk.n);
    }
    __syncthreads();
  }
  if (!active) return;
  float* X = (float*)(smem + wave * (spill_units<NTB>() / 4));
  spill_acc<NTB>(X, acc, lane);
  unsigned bad = not_finite(check_acc<NTB>(acc, 0.f * dl), row < t.nrows);
  __builtin_amdgcn_wave_barrier();
  if (row < t.nrows && !((bad >> n) & 1)) {
    T* const o = dQ + t.row0 * ldg + hc + row * (int)ldg;
#pragma unroll
    for (int i = 0; i < (DH + 3) / 4; ++i) {
      const int e = (lane >> 4) + 4 * i;
      if (e < dh) stf(o + e, part_sum<DH, NTB>(X, n, e) * ((row & 1) ? -g.scale : g.scale));
    }
  }
  if (__builtin_expect(bad == 0, 1)) return;
  const unsigned nan = bad & (nan_rows<T, DH, EXACT>(Q + t.row0 * ld + hc, ld, wave * 16, t.nrows, dh) |
                              nan_rows<T, DH, EXACT>(dO + t.row0 * ldo + hc, ldo, wave * 16, t.nrows, dh) |
                              nan_rows<T, DH, EXACT>(O + t.row0 * ldo + hc, ldo, wave * 16, t.nrows, dh));
  put_rows(nan, dQ + t.row0 * ldg + hc, ldg, wave * 16, dh, keys ? __builtin_nanf("") : 0.f);   // (delta stands)
  for (bad &= ~nan; bad; bad &= bad - 1)
    plain_dq_row<T, DH, EXACT>(g, t, wave * 16 + __builtin_ctz(bad), dh, Q, K, V, ld, O, dO, ldo, lse2, valid_len, key_pad, delta, dQ,
                               ldg);
}

template <typename T, int DH, bool EXACT>
__device__ __forceinline__ void plain_dkv_row(const SplitGeo& g, const SplitTile& t, int row, int dh, const T* Q, const T* K,
                                              const T* V, long ld, const T* dO, long ldo, const float* lse2, const float* delta,
                                              const uint8_t* key_pad, T* dK, T* dV, long ldg) {
  const int lane = threadIdx.x & 63, hc = t.h * dh;
  float k[DH], v[DH], ak[DH], av[DH];
  load_head_row<T, DH, EXACT>(K + (t.row0 + row) * ld + hc, dh, k);
  load_head_row<T, DH, EXACT>(V + (t.row0 + row) * ld + hc, dh, v);
#pragma unroll
  for (int e = 0; e < DH; ++e) ak[e] = av[e] = 0.f;
  // a masked key's gradients are zero, whatever its row holds
  if (row < t.vlen && !(key_pad && key_pad[t.row0 + row] != 0)) {
    SplitWalk walk(t.live);
    while (walk.next(g, t.b, t.h, nullptr)) {
      if (lane >= walk.n) continue;
      const long r = walk.row0 + lane;
      float q[DH], go[DH];
      load_head_row<T, DH, EXACT>(Q + r * ld + hc, dh, q);
      load_head_row<T, DH, EXACT>(dO + r * ldo + hc, dh, go);
      const float ls = lse2[walk.stat0 + lane], dl = (lane & 1) ? -delta[walk.stat0 + lane] : delta[walk.stat0 + lane];
      scale_row<DH>(q, g.scale_log2e);
      const float p = __builtin_amdgcn_exp2f(dot_from<DH>(0.f, q, k) - (ls == IM_NEG_INF ? -IM_NEG_INF : ls));
      const float ds = p * (dot_from<DH>(0.f, go, v) - dl);
#pragma unroll
      for (int e = 0; e < DH; ++e) {
        av[e] = fmaf(p, go[e], av[e]);
        ak[e] = fmaf(ds, q[e], ak[e]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < DH; ++e) {
    const float a = wave_sum(ak[e]) * 0.69314718055994530942f, b = wave_sum(av[e]);
    if (lane == 0 && e < dh) {
      stf(dK + (t.row0 + row) * ldg + hc + e, a);
      stf(dV + (t.row0 + row) * ldg + hc + e, b);
    }
  }
}

// dK, dV: own rows are keys; query rows (Q, dO, lse, delta) are streamed.  Each key tile has a single producer
// workgroup, so no atomics.
template <typename T, int DH, bool EXACT>
__global__ __launch_bounds__(256, DH > 5 ? 2 : 4)
void split_dkv_kernel(SplitGeo g, int tile_base, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                      long ld, const T* __restrict__ dO, long ldo, const float* __restrict__ lse2,
                      const float* __restrict__ delta, const int32_t* __restrict__ valid_len,
                      const uint8_t* __restrict__ key_pad, T* __restrict__ dK, T* __restrict__ dV, long ldg) {
  using F = SplitCfg<DH>;
  constexpr int NS = F::NS, NTB = F::NT;
  constexpr int S_UNITS = 4 * F::BLK, T_UNITS = 2 * NTB * 64;
  // One chunk (Q, dO, both transposed, lse, delta) and the own rows (K, V): with two chunk buffers, one barrier less
  // per chunk, the kernel took 44 instead of 41 us (101 registers).
  constexpr int CH = 2 * S_UNITS + 2 * T_UNITS + 2 * SPLIT_ROWS / 4, STAT_AT = 2 * S_UNITS + 2 * T_UNITS;
  __shared__ u32x4 smem[cmax(CH + 2 * S_UNITS, 2 * spill_units<NTB>())];
  u32x4* const sOwn = smem + CH;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  SplitTile t;
  if (!find_tile(g, tile_base, valid_len, t)) return;
  const int dh = EXACT ? DH : g.dh, hc = t.h * dh;
  if (t.vlen <= 0) {   // a tile behind the segment's valid length has no key that any query attends: zeros
    for (int i = tid; i < t.nrows * dh; i += 256) {
      const int r = i / dh, e = i - r * dh;
      stf(dK + (t.row0 + r) * ldg + hc + e, 0.f);
      stf(dV + (t.row0 + r) * ldg + hc + e, 0.f);
    }
    return;
  }

  float raw[DH], part[3][DH], stat = 0.f;
  const bool turn = (t.b + blockIdx.y) & 1;   // the sums have the other sign
  SplitWalk walk(t.live);
  auto request = [&]() {
    if (wave < 2 && lane < ((walk.n + 31) & ~31)) {
      const int r = min(lane, walk.n - 1);
      load_head_row<T, DH, EXACT>(wave ? dO + walk.row0 * ldo + hc + r * (int)ldo : Q + walk.row0 * ld + hc + r * (int)ld, dh, raw);
      stat = (wave ? delta : lse2)[walk.stat0 + r];
    }
  };
  auto store = [&](u32x4* buf, int n) {
    if (wave < 2 && lane < ((n + 31) & ~31)) {
      const bool in = lane < n;
#pragma unroll
      for (int e = 0; e < DH; ++e) raw[e] = in ? raw[e] : 0.f;
      if (!wave) scale_row<DH>(raw, g.scale_log2e);
      split_rows<DH>(raw, part);
      int blk, mm;
      step_pos(lane, blk, mm);
      // odd query rows: -dO (and -delta from the dQ kernel) give -dS, which meets -Q; dV takes dO as it is
      store_score_row<DH, true>(buf + (wave ? S_UNITS : 0), blk, mm, part, wave ? 0.f : 1.f, wave && (lane & 1));
      store_tr_row<DH, NTB, false>((bf16_t*)(buf + 2 * S_UNITS + (wave ? T_UNITS : 0)), blk, mm, part, (!wave && (lane & 1)) != turn);
      ((float*)(buf + STAT_AT))[(wave ? SPLIT_ROWS : 0) + blk * 16 + mm] =
          wave ? (in ? stat : 0.f) : (in && stat != IM_NEG_INF) ? stat : -IM_NEG_INF;
    }
  };
  bool ok = true;
  if (wave >= 2) {
    const int r = min(lane, t.nrows - 1);
    load_head_row<T, DH, EXACT>((wave == 3 ? V : K) + t.row0 * ld + hc + r * (int)ld, dh, raw);
    ok = wave == 3 || (lane < min(t.vlen, t.nrows) && !(key_pad && key_pad[t.row0 + r] != 0));
  }
  bool more = walk.next(g, t.b, t.h, nullptr);
  if (more) request();
  if (wave >= 2) {
    split_rows<DH>(raw, part);
    store_score_row<DH, false>(sOwn + (wave - 2) * S_UNITS, lane >> 4, lane & 15, part, ok ? 0.f : SPLIT_MASKED);
  }
  if (more) store(smem, walk.n);
  __syncthreads();
  bf16x8 bk[NS], bv[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    bk[s] = score_frag<DH>(sOwn, wave, s, lane);
    bv[s] = score_frag<DH>(sOwn + S_UNITS, wave, s, lane);
  }
  const bool active = wave * 16 < min(t.vlen, t.nrows);
  f32x4 ak[NTB], av[NTB];
#pragma unroll
  for (int rb = 0; rb < NTB; ++rb) ak[rb] = av[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int g4 = lane >> 4;
  auto steps = [&](const u32x4* sQ, int nst) {
    const u32x4* const sG = sQ + S_UNITS;
    const bf16_t *const sQT = (const bf16_t*)(sQ + 2 * S_UNITS), *const sGT = (const bf16_t*)(sQ + 2 * S_UNITS + T_UNITS);
    const f32x4 *const sL = (const f32x4*)(sQ + STAT_AT), *const sD = sL + SPLIT_ROWS / 4;
    for (int st = 0; st < nst; ++st) {
      f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0, y0 = x0, y1 = x0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        x0 = mfma16(score_frag<DH>(sQ, 2 * st, s, lane), bk[s], x0);
        x1 = mfma16(score_frag<DH>(sQ, 2 * st + 1, s, lane), bk[s], x1);
        y0 = mfma16(score_frag<DH>(sG, 2 * st, s, lane), bv[s], y0);
        y1 = mfma16(score_frag<DH>(sG, 2 * st + 1, s, lane), bv[s], y1);
      }
      const f32x4 l0 = sL[8 * st + g4], l1 = sL[8 * st + 4 + g4], d0 = sD[8 * st + g4], d1 = sD[8 * st + 4 + g4];
      float p[8], ds[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[i] = __builtin_amdgcn_exp2f(x0[i] - l0[i]);
        p[4 + i] = __builtin_amdgcn_exp2f(x1[i] - l1[i]);
        ds[i] = p[i] * (y0[i] - d0[i]);
        ds[4 + i] = p[4 + i] * (y1[i] - d1[i]);
      }
      bf16x8 bp[3];
      split8(p, bp);
      accumulate_tr<DH, NTB, false>(sGT, st, bp, av, lane);
      split8(ds, bp);
      accumulate_tr<DH, NTB, false>(sQT, st, bp, ak, lane);
    }
  };
  if (!more) __syncthreads();   // no query at all: the own rows have been read before the results take their place
  while (more) {
    const int nst = (walk.n + 31) >> 5;
    more = walk.next(g, t.b, t.h, nullptr);
    if (more) request();
    if (active) steps(smem, nst);
    __syncthreads();
    if (more) {
      store(smem, walk.n);
      __syncthreads();
    }
  }
  if (wave * 16 >= t.nrows) return;
  float* X = (float*)(smem + wave * (2 * spill_units<NTB>() / 4));
  float* X2 = X + 16 * (16 * NTB + 4);
  const int n = lane & 15, row = wave * 16 + n;
  const float ln2 = 0.69314718055994530942f;   // the staged Q carries scale * log2(e); dK = scale * dS^T q
  spill_acc<NTB>(X, ak, lane);
  spill_acc<NTB>(X2, av, lane);
  unsigned bad = not_finite(check_acc<NTB>(av, check_acc<NTB>(ak, 0.f)), row < t.nrows);
  __builtin_amdgcn_wave_barrier();
  if (row < t.nrows && !((bad >> n) & 1)) {
    T *const pk = dK + t.row0 * ldg + hc + row * (int)ldg, *const pv = dV + t.row0 * ldg + hc + row * (int)ldg;
#pragma unroll
    for (int i = 0; i < (DH + 3) / 4; ++i) {
      const int e = g4 + 4 * i;
      if (e < dh) {
        stf(pk + e, part_sum<DH, NTB>(X, n, e) * (turn ? -ln2 : ln2));
        stf(pv + e, part_sum<DH, NTB>(X2, n, e) * (turn ? -1.f : 1.f));
      }
    }
  }
  if (__builtin_expect(bad == 0, 1)) return;
  const unsigned nan = bad & nan_rows<T, DH, EXACT>(K + t.row0 * ld + hc, ld, wave * 16, t.nrows, dh);
  const float v = row < t.vlen && !(key_pad && row < t.nrows && key_pad[t.row0 + row] != 0) ? __builtin_nanf("") : 0.f;
  put_rows(nan, dK + t.row0 * ldg + hc, ldg, wave * 16, dh, v);
  put_rows(nan, dV + t.row0 * ldg + hc, ldg, wave * 16, dh, v);
  for (bad &= ~nan; bad; bad &= bad - 1)
    plain_dkv_row<T, DH, EXACT>(g, t, wave * 16 + __builtin_ctz(bad), dh, Q, K, V, ld, dO, ldo, lse2, delta, key_pad, dK, dV, ldg);
}

// Zero columns col0 .. col0+ncols-1 of the rows of segment s (all batch elements): outputs of query
// segments with no live key segment, gradients of segments that no live block reads.
template <typename T>
__global__ void zero_seg_rows_kernel(Geo g, int s, T* p, long ld, int col0, int ncols) {
  const int nrows = g.seg_len[s];
  const long n = (long)g.B * nrows * ncols;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int e = i % ncols;
    const long r = i / ncols;
    const int b = r / nrows, rr = r % nrows;
    if (rr < seg_rows(g, b, s)) stf(p + (seg_row0(g, b, s) + rr) * ld + col0 + e, 0.f);
  }
}
// per-row statistic (lse) of segment s, all batch elements and heads := value
__global__ void fill_seg_stat_kernel(Geo g, int s, float* stat, float value) {
  const int nrows = g.seg_len[s];
  const long n = (long)g.B * g.H * nrows;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int rr = i % nrows;
    const long bh = i / nrows;
    const int b = bh / g.H, h = bh % g.H;
    if (rr < seg_rows(g, b, s)) stat[seg_stat0(g, b, h, s) + rr] = value;
  }
}
void launch_zero_seg_rows(const Geo& g, int s, int bf16, void* p, long ld, int col0, int ncols, hipStream_t st) {
  if (bf16) hipLaunchKernelGGL((zero_seg_rows_kernel<bf16_t>), dim3(64), dim3(256), 0, st, g, s, (bf16_t*)p, ld, col0, ncols);
  else hipLaunchKernelGGL((zero_seg_rows_kernel<float>), dim3(64), dim3(256), 0, st, g, s, (float*)p, ld, col0, ncols);
}
void launch_fill_seg_stat(const Geo& g, int s, float* stat, float value, hipStream_t st) {
  hipLaunchKernelGGL(fill_seg_stat_kernel, dim3(16), dim3(256), 0, st, g, s, stat, value);
}

bool smallhead_supports(int dh) { return dh >= 1 && dh <= 16; }

static SplitGeo split_geo(const Geo& g, bool query_side) {
  SplitGeo s;
  s.H = g.H; s.dh = g.dh; s.n_seg = g.n_seg; s.T = g.T; s.R = g.R; s.cu = g.cu;
  s.scale = g.scale; s.scale_log2e = g.scale_log2e;
  s.pair0 = s.pairs = 0;   // set per launch
  s.h_magic = g.H > 1 && (uint64_t)g.B * g.H * g.H < (1ull << 32) ? (unsigned)((1ull << 32) / g.H + ((1ull << 32) % g.H != 0)) : 0u;
  const int nord = query_side ? g.q_nord : g.k_nord;
  for (int k = 0; k < IM_MAX_SEG; ++k) {
    const int seg = k < nord ? (query_side ? g.q_order[k] : g.k_order[k]) : 0;
    s.tile0[k] = k < nord ? (query_side ? g.q_tile_prefix[k] : g.k_tile_prefix[k]) : INT_MAX;
    s.seg[k] = seg;
    s.live[k] = query_side ? g.q_live[seg] : g.k_live[seg];
    s.len[k] = k < g.n_seg ? g.seg_len[k] : 0;
    s.off[k] = k < g.n_seg ? g.seg_off[k] : 0;
  }
  return s;
}

// KERNEL for head dimension dh: exact instantiations, or the next larger of 4 / 8 / 12 / 16 with columns beyond dh zeroed.
#define SPLIT_DISPATCH(dh, KERNEL, ...)                               \
  do {                                                                \
    if ((dh) == 4) SPLIT_LAUNCH(KERNEL, 4, true, __VA_ARGS__);        \
    else if ((dh) == 5) SPLIT_LAUNCH(KERNEL, 5, true, __VA_ARGS__);   \
    else if ((dh) == 6) SPLIT_LAUNCH(KERNEL, 6, true, __VA_ARGS__);   \
    else if ((dh) == 8) SPLIT_LAUNCH(KERNEL, 8, true, __VA_ARGS__);   \
    else if ((dh) == 10) SPLIT_LAUNCH(KERNEL, 10, true, __VA_ARGS__); \
    else if ((dh) == 12) SPLIT_LAUNCH(KERNEL, 12, true, __VA_ARGS__); \
    else if ((dh) == 16) SPLIT_LAUNCH(KERNEL, 16, true, __VA_ARGS__); \
    else if ((dh) < 4) SPLIT_LAUNCH(KERNEL, 4, false, __VA_ARGS__);   \
    else if ((dh) < 8) SPLIT_LAUNCH(KERNEL, 8, false, __VA_ARGS__);   \
    else if ((dh) < 12) SPLIT_LAUNCH(KERNEL, 12, false, __VA_ARGS__); \
    else SPLIT_LAUNCH(KERNEL, 16, false, __VA_ARGS__);                \
  } while (0)
// grid (8 ceil(pairs / 8), tiles); a launch takes at most 2^22 pairs (a grid's x holds 2^32 - 1 threads) and 65535 tiles
constexpr unsigned SPLIT_MAX_PAIRS = 1u << 22;
#define SPLIT_LAUNCH(KERNEL, DHV, EX, ...)                                                                                  \
  do {                                                                                                                      \
    const unsigned npairs = (unsigned)g.B * g.H;                                                                            \
    for (unsigned p0 = 0; p0 < npairs; p0 += SPLIT_MAX_PAIRS) {                                                             \
      sg.pair0 = (int)p0;                                                                                                   \
      sg.pairs = (int)(npairs - p0 < SPLIT_MAX_PAIRS ? npairs - p0 : SPLIT_MAX_PAIRS);                                      \
      for (int t0 = 0; t0 < ntiles; t0 += 65535)                                                                            \
        hipLaunchKernelGGL((KERNEL<T, DHV, EX>), dim3((sg.pairs + 7) / 8 * 8, ntiles - t0 < 65535 ? ntiles - t0 : 65535),   \
                           dim3(256), 0, st, sg, t0, __VA_ARGS__);                                                          \
    }                                                                                                                       \
  } while (0)

template <typename T>
static int fwd_dispatch(const Geo& g, const T* q, const T* k, const T* v, long ld, const int32_t* vl,
                        const uint8_t* kp, T* o, long ldo, float* lse2, hipStream_t st) {
  const int ntiles = g.q_tile_prefix[g.q_nord];
  SplitGeo sg = split_geo(g, true);
  SPLIT_DISPATCH(g.dh, split_fwd_kernel, q, k, v, ld, vl, kp, o, ldo, lse2);
  return IM_OK;
}

// Rows of query segments with no live block never get written by the kernels: the
// host zero-fills them (output 0, lse -inf) before launching.
template <typename T>
static void zero_dead_rows(const Geo& g, bool query_side, T* p, long ld, hipStream_t st) {
  for (int s = 0; s < g.n_seg; ++s) {
    const unsigned live = query_side ? g.q_live[s] : g.k_live[s];
    if (live) continue;
    launch_zero_seg_rows(g, s, sizeof(T) == 2, p, ld, 0, g.d, st);
  }
}

int launch_smallhead_fwd(const Geo& g, int bf16, const void* q, const void* k, const void* v, long ld,
                       const int32_t* valid_len, const uint8_t* key_pad, void* o, long ldo, float* lse2,
                       hipStream_t st) {
  if (!smallhead_supports(g.dh)) return IM_ERR_UNSUPPORTED;
  for (int s = 0; s < g.n_seg; ++s)
    if (!g.q_live[s] && lse2)
      launch_fill_seg_stat(g, s, lse2, IM_NEG_INF, st);
  if (bf16) {
    zero_dead_rows<bf16_t>(g, true, (bf16_t*)o, ldo, st);
    return fwd_dispatch<bf16_t>(g, (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, ld, valid_len, key_pad,
                                (bf16_t*)o, ldo, lse2, st);
  }
  zero_dead_rows<float>(g, true, (float*)o, ldo, st);
  return fwd_dispatch<float>(g, (const float*)q, (const float*)k, (const float*)v, ld, valid_len, key_pad, (float*)o,
                             ldo, lse2, st);
}

template <typename T>
static int bwd_dispatch(const Geo& g, const T* q, const T* k, const T* v, long ld, const T* o, const T* d_o,
                        long ldo, const float* lse2, const int32_t* vl, const uint8_t* kp, float* delta, T* dq, T* dk, T* dv,
                        long ldg, hipStream_t st) {
  zero_dead_rows<T>(g, true, dq, ldg, st);
  zero_dead_rows<T>(g, false, dk, ldg, st);
  zero_dead_rows<T>(g, false, dv, ldg, st);
  {
    ProfScope ps(PF_ATTN_DQ, st);
    const int ntiles = g.q_tile_prefix[g.q_nord];
    SplitGeo sg = split_geo(g, true);
    SPLIT_DISPATCH(g.dh, split_dq_kernel, q, k, v, ld, o, d_o, ldo, lse2, vl, kp, delta, dq, ldg);
  }
  {
    ProfScope ps(PF_ATTN_DKV, st);
    const int ntiles = g.k_tile_prefix[g.k_nord];
    SplitGeo sg = split_geo(g, false);
    SPLIT_DISPATCH(g.dh, split_dkv_kernel, q, k, v, ld, d_o, ldo, lse2, delta, vl, kp, dk, dv, ldg);
  }
  return IM_OK;
}

int launch_smallhead_bwd(const Geo& g, int bf16, const void* q, const void* k, const void* v, long ld, const void* o,
                       const void* d_o, long ldo, const float* lse2, const int32_t* valid_len, const uint8_t* key_pad,
                       float* delta, void* dq, void* dk, void* dv, long ldg, hipStream_t st) {
  if (!smallhead_supports(g.dh)) return IM_ERR_UNSUPPORTED;
  if (bf16)
    return bwd_dispatch<bf16_t>(g, (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, ld, (const bf16_t*)o,
                                (const bf16_t*)d_o, ldo, lse2, valid_len, key_pad, delta, (bf16_t*)dq, (bf16_t*)dk,
                                (bf16_t*)dv, ldg, st);
  return bwd_dispatch<float>(g, (const float*)q, (const float*)k, (const float*)v, ld, (const float*)o,
                             (const float*)d_o, ldo, lse2, valid_len, key_pad, delta, (float*)dq, (float*)dk,
                             (float*)dv, ldg, st);
}

}  // namespace imattn
