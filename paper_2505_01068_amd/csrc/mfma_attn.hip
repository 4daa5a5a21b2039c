// Flash-style IM attention on the CDNA4 matrix cores: bf16 operands, fp32
// accumulation, head dimension 64 (forward also head dimensions 8 / 16 in its
// sub-head mode; their backward is in mfma_attn_sub.hip).
//
// All three kernels compute "transposed" products so that every per-row
// quantity of the softmax lives on the lane that owns the row:
//   forward / dQ : lane <-> query row.  S^T = K Q^T  (rows = keys, cols = queries);
//                  O^T = V^T P^T and dQ^T = K^T dS^T take P^T / dS^T straight from
//                  the accumulator registers (see perm32 in mfma_common.hpp).
//   dK / dV      : lane <-> key row.    S = Q K^T (rows = queries), dP = dO V^T;
//                  dV^T = dO^T P and dK^T = Q^T dS take P / dS from registers.
// K/V (or Q/dO) tiles of 64 rows go through a ring of LDS stages, row-major
// (swizzled, filled by asynchronous global->LDS copies); products
// that need the tile transposed (V^T, K^T, Q^T, dO^T as the MFMA "A" operand)
// read it with the gfx950 LDS transpose read (ds_read_b64_tr_b16), so no
// transposed copy of any tensor exists in HBM.
//
// Conventions between the kernels: the Q rows arrive multiplied by scale * log2(e) (the QKV projection's
// epilogue does it before its one rounding to bf16), so Q K^T is the score in the exponent domain of
// exp2 and no kernel multiplies scores; the per-row statistic saved by the forward is the NEGATED
// log2-sum-exp (-inf for a row without any valid key), which the backward kernels add to the score --
// by starting their score accumulators from it, as the dP accumulators start from -delta: the MFMA
// chains end as S - lse and dP - delta and the softmax needs no add per element.  The forward's start from the negated reference of
// the row, the largest score of its first 32 keys.
//
// Only live (query segment, key segment) blocks of the Interlaced Mask are
// visited (Sec. 6 "Decomposition"); a row with several live segments carries
// one running sum across all of them (Sec. "Information Disorder").
#include <algorithm>
#include <type_traits>
#include "mfma_attn_common.hpp"
#include "mfma_path.hpp"

namespace imattn {

// ------------------------------------------------------------------------------------------
// Forward.  Workgroup = 4 waves; each wave owns QB blocks of 32 query rows.
//
// DH = 64: one head = one 64-column group of the activation rows.
// DH = 8 or 16 ("sub-head" mode, d % 64 == 0): a head is a slice of a 64-column group.  The K/V
// tiles of the whole group are streamed as before; S^T needs only the one 16-deep k-step that
// holds the head's columns (for DH = 8 the Q operand of the other lane half is zero), and
// O^T only the one 32-row block of V^T that holds them.  Per 64-key tile that is 2 + 4 MFMAs per
// query block instead of 8 + 8, and the softmax stays on 32 x 32 accumulator tiles -- about a
// quarter of the VALU instructions of the row-per-lane kernel at these head sizes.
// KS = 2: tiles of half the height, see split_rows.
// PAIR: two problems of the same shape in one launch (two encoders side by side; see Geo::pair_B): grid z = 2 B.
constexpr float BF16_MAX = 3.3895313892515355e38f;
constexpr int FWD_NST = 2;                  // stages of its ring
template <int QB, int DH, int WGS, bool PAIR, int KS = 1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WGS, WGS))) void mfma_fwd_kernel(Geo g, const bf16_t* __restrict__ QKV, long ld,
                                                       const int32_t* __restrict__ valid_len,
                                                       const uint8_t* __restrict__ key_pad, bf16_t* __restrict__ O,
                                                       long ldo, float* __restrict__ lse2) {
  __shared__ __attribute__((aligned(1024))) bf16_t sT[FWD_NST * RING_STAGE];  // per stage: K tile, V tile
  __shared__ __attribute__((aligned(256))) unsigned sKP[FWD_NST * KT];        // per stage: key_pad bytes of the 64 keys, one per dword
  __shared__ __attribute__((aligned(16))) unsigned sPM[4][KT / 2];            // key masks of the wave's tile
  __shared__ SegTable sSeg[4];
  // Sub-head mode: ones, four to each of the 16-key steps of a tile, where the step's V^T fragment has its rows in the tile.
  // The lanes whose four rows of the fragment are not the head's read them: those rows of O^T are then the row sum of P,
  // which the matrix cores take beside the product (a dot product per pair of probabilities otherwise, 8 of 40 vector
  // instructions per 32 x 32 scores).  Between them, at head dimension 8, the ones that the reference's parts meet.
  constexpr bool ONES = DH != 64;
  __shared__ __attribute__((aligned(16))) bf16_t sOnes[ONES ? 3 * 16 * SW_LD + 4 : 4];
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: branches on it are wave-uniform
  int tile, h, b;
  xcd_tile_index(g.q_tile_prefix, g.q_nord, g.cu != nullptr, g.even_cus, tile, h, b);
  constexpr bool HEADW = DH != 64;
  // HEADW (sub-head mode, where the head count is a multiple of 4): the four waves of a workgroup are four heads of one 64-column group over the SAME 32 QB
  // query rows (grid.y counts groups of four heads) -- the K/V stream is shared as before, but a tile is 64 rows instead of
  // 256, which at segment lengths like 50 / 500 / 375 leaves 4 % of the rows of the tiles empty instead of 28 %.
  if (HEADW) h = h * 4 + wave;
  const bool second = PAIR && b >= g.pair_B;
  const int bm = second ? b - g.pair_B : b;   // batch element of the masks (valid_len, key_pad)
  constexpr int WG_ROWS = HEADW ? 32 * QB : 128 * QB / KS;
  static_assert(KS == 1 || (DH == 64 && QB == 1 && !PAIR && !HEADW), "");
  const int rb = wave / KS, kg = wave % KS;   // row block of the tile, key block of a stage (KS = 2)
  // HALF: the launch may give the query segment with the longest key range tiles of half the height (one query
  // block per wave instead of two), see launch_mfma_fwd; such a workgroup runs the loop below for one block.
  constexpr bool HALF = HEADW && !PAIR && QB == 2;
  int qs, q0, ord;
  if (second) tile_segment(g.q_order2, g.q_tile_prefix2, g.q_nord2, tile, qs, q0, ord);
  else tile_segment(g.q_order, g.q_tile_prefix, g.q_nord, tile, qs, q0, ord);
  const bool half_tile = HALF && ((g.q_half >> ord) & 1u);
  q0 *= half_tile ? WG_ROWS / 2 : WG_ROWS;
  const unsigned live = second ? g.q_live2[qs] : g.q_live[qs];   // live key segments of the tile's query segment
  int qoff, qlen;
  SegTable& sg = sSeg[wave];
  const unsigned row_set = seg_rows_table(sg, g, b, live, lane, qs, qoff, qlen);
  if (q0 >= qlen) return;  // packed rows: this batch element's segment ends before the tile
  const int d = g.d;
  const long row_b = g.cu ? 0 : (long)b * g.T, qrow0 = row_b + qoff;   // rows of the batch element, of segment qs

  constexpr int NS = DH == 64 ? 4 : 1;    // k-steps of S^T
  constexpr int NDB = DH == 64 ? 2 : 1;   // 32-row blocks of O^T
  const int cg = (h * DH) >> 6;           // 64-column group of this head
  const int wo = (h * DH) & 63;           // first column of the head inside the group
  const int s0 = DH == 64 ? 0 : wo >> 4;  // k-step and O^T block that hold the head (sub-head mode)
  const int db0 = DH == 64 ? 0 : wo >> 5;

  KvStream<FWD_NST> ring(sg, sT, sKP, QKV + row_b * ld + d, key_pad ? key_pad + (g.cu ? 0 : (long)bm * g.T) : nullptr, ld, d, wave, lane, cg);
  const int seg1 = row_set ? __builtin_ctz(row_set) : 0;   // its first tile goes ahead of everything
  if (row_set) ring.first(seg1);
  const int valid = valid_len ? valid_len[bm * g.n_seg + min(lane, g.n_seg - 1)] : 0;

  // Q operand (B of S^T = K Q^T): lane holds query row lo of each block, 8 consecutive dh per k-step
  bf16x8 qreg[QB][NS];
  int qrow[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    qrow[qb] = q0 + ((HEADW ? 0 : rb * QB) + qb) * 32 + lo;
    if (HALF && half_tile && qb > 0) qrow[qb] = qlen;   // the next tile's rows: not computed, not stored
    const int rc = min(qrow[qb], qlen - 1);
    const bf16_t* p = QKV + (qrow0 + rc) * ld + cg * 64 + hi * 8;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      u32x4 v = *(const u32x4*)(p + (s0 + s) * 16);
      if (DH == 8 && hi != ((wo >> 3) & 1)) v = u32x4{0u, 0u, 0u, 0u};  // the other head of this k-step
      qreg[qb][s] = as_bf16x8(v);
    }
  }

  f32x16 oacc[NDB][QB];
  float m[QB], l[QB];

  // V^T fragments in sub-head mode: the lane's two addresses (lds_frag_tr_sw) from the V tile on, or the ones
  unsigned vt0 = 0, vt1 = 0, vt_tile = 0;   // vt_tile: all bits set where the tile's address is to be added
  if (ONES) {
    const int j = lane & 15, gg = lane >> 4, lrow = 8 * (gg >> 1) + (j >> 2), lchunk = 2 * (gg & 1) + ((j & 3) >> 1);
    const int chunk = (db0 * 4) | lchunk, f = sw_f(lrow);
    const unsigned ones = (unsigned)(uintptr_t)sOnes;
    const bool own = chunk >= (wo >> 3) && chunk < (wo + DH) >> 3;
    vt0 = own ? (unsigned)(lrow * SW_LD + ((chunk ^ f) << 3) + 4 * (j & 1)) * 2u : ones;
    vt1 = own ? (unsigned)((lrow + 4) * SW_LD + ((chunk ^ f ^ 1) << 3) + 4 * (j & 1)) * 2u : ones;
    vt_tile = own ? ~0u : 0u;
    if (lane < 16) sOnes[(lane >> 2) * 16 * SW_LD + (lane & 3)] = 0x3f80;   // every wave, so that none waits for another
    else if (lane < 24) sOnes[8 + (lane & 7)] = (lane & 7) < 3 ? 0x3f80 : 0;   // three ones and zeros: what the reference's parts meet
  }

  const int prow = perm32(lo);
  // The negated reference of the query rows enters S^T through the matrix cores: as the seed of the accumulators (head dimension
  // 64), or as three bf16 parts that meet ones (bf16_parts) -- in the lane half of the k-step that is not the head's (8), or in an
  // 8-deep k-step of their own (16), where the seeds of two row blocks have no room in 128 registers.  (At 64 such a k-step takes
  // 16 x 2048 rows, 2 heads, from 78 to 81 us.)
  u32x2 nmp[DH == 16 ? QB : 1];
  f32x16 nm;
  const bool spare = DH == 8 && hi != ((wo >> 3) & 1);
  const unsigned kf = spare ? (unsigned)(uintptr_t)(sOnes + 8) : (unsigned)(prow * SW_LD + (((2 * s0 + hi) ^ sw_f(prow)) << 3)) * 2u;
  const unsigned kf_tile = spare ? 0u : ~0u;
  auto set_reference = [&](int qb, float v) __attribute__((always_inline)) {   // v: negated
    if (DH == 64) {
#pragma unroll
      for (int r = 0; r < 16; ++r) nm[r] = v;
      return;
    }
    const u32x2 pt = bf16_parts(v);
    if (DH == 8) qreg[qb][0] = spare ? as_bf16x8(u32x4{pt[0], pt[1], 0u, 0u}) : qreg[qb][0];
    else nmp[DH == 16 ? qb : 0] = hi == 0 ? pt : u32x2{0u, 0u};
  };
  // The compiler does not see the asynchronous copies in its vmcnt bookkeeping: consuming the Q
  // registers here makes it wait for their (ordinary) loads now, not inside the ring loop.
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" :: "v"(qreg[qb][s]));

  const unsigned key_set = valid_len ? seg_lens_table(sg, valid, row_set, lane) : row_set;

  // A row's reference is its largest score in the first 32-key block that has a valid key.  fp32 and bf16 share their exponent range,
  // so probabilities above 1 lose nothing, and the reference moves only where one would exceed 2^24 (sub-head mode; at head dimension
  // 64 a lane's part of a block's sum): almost every block is exponentiated as it leaves the matrix cores, no maximum is taken.
  //
  // In sub-head mode, where row sums come out of the matrix cores too late for that, references are 23 larger than the score.  A
  // probability of 2^24 is 2 then and sets bit 14 of its bf16, and eight three-way ORs and a compare find it for 32 x 64 scores.
  // (Probabilities below 2^-103 of the largest vanish, and values of V below 1e-31.)
  //
  // Without any reference the largest probability of the first block is rounded to bf16 like the others instead of being exactly 1, and
  // with it the log-sum-exp that the backward takes all probabilities from.  Errors against fp64, rms of 6 seeds, 40 shapes of 8
  // to 1000 keys, ordinary and peaked scores, times those with a reference that moves in every block that needs it: y up to 1.03,
  // dWo 1.04, dWv 1.05, dWq and dWk 1.04; as here 0.99 to 1.00.
  // Time, us:                                            4 encoder layers of     16 x 2048 rows, 8 heads of 8, scores with a standard
  //                                                      32 x 50/500/375 rows    deviation of 1.4 / 10 / 20 bits
  //   row sums by dot products, first references in the
  //     loop, three workgroups per CU                      147                     123 / 129 / 142
  //   row sums by dot products                             137                     110 / 116 / 132
  //   here                                                 131                      97 / 111 / 133
  //   one check behind the loop, a second pass             129                      94 / 198 / 202
  //   no reference                                         126                      92 / 127 / 202
  auto row_max = [&](const f32x16& s) __attribute__((always_inline)) {   // of the lane's column of S^T, both lane halves
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
  };
  auto clamp_ref = [](float v) __attribute__((always_inline)) { return fminf(fmaxf(v, -BF16_MAX), BF16_MAX); };   // has a bf16
  constexpr float REF_OFF = ONES ? 23.f : 0.f;
  // One pass over the live key tiles, for NQB of the wave's QB query blocks (NQB < QB: a tile of half the height).
  auto stream = [&](auto nqb_tag) __attribute__((always_inline)) {
    constexpr int NQB = decltype(nqb_tag)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      m[qb] = IM_NEG_INF;
      l[qb] = 0.f;
      set_reference(qb, 0.f);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][qb][r] = 0.f;
    }
    static_assert(FWD_NST == 2, "the slot refilled while a tile is consumed is that of the tile before");
    int cslot = 0, keys = 0, keys1 = row_set ? ring.begin(seg1, key_set) : -1;   // valid keys of the present tile, of the one
                                                                                 // requested after it (-1: there is none)
    const bf16_t *sK = sT, *sV = sT;
    bool need_mask = false;   // tail tile or key_pad present (wave-uniform)
    auto advance = [&]() __attribute__((always_inline)) {   // to the next tile
      ring_wait(false);
      keys = keys1;
      keys1 = ring.issue();
      sK = sT + cslot * RING_STAGE;
      sV = sK + KT * SW_LD;
      need_mask = keys < KT || key_pad != nullptr;
      if (need_mask) tile_masks(sPM[wave], key_pad ? sKP + cslot * KT : nullptr, keys);
      cslot ^= 1;
    };
    // S^T = K Q^T, less the reference
    auto scores = [&](f32x16 (&sacc)[QB], int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bf16x8 a = DH == 8 ? lds_b128((kf_tile & ((unsigned)(uintptr_t)sK + kb * 32 * SW_LD * 2)) + kf)
                                 : lds_frag_sw(sK, kb * 32, prow, 2 * (s0 + s) + hi);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) {
          if (s == 0) sacc[qb] = DH == 8 ? f32x16{} : DH == 64 ? nm : mfma32_k8(u32x2{ONES01, ONES2}, nmp[DH == 16 ? qb : 0], f32x16{});
          sacc[qb] = mfma32(a, qreg[qb][s], sacc[qb]);
        }
      }
    };
    // The references, from the first block with a valid key (wave-uniform); the tiles before it contribute nothing.
    bool seen = false;
    while (!seen && keys1 >= 0) {
      advance();
#pragma unroll 1
      for (int kk = 0; kk < 2 / KS && !seen; ++kk) {
        const int kb = KS == 1 ? kk : kg;
        if (kb == 1 && keys <= 32) break;
        f32x16 sacc[QB];
        scores(sacc, kb);
        seen = true;
        if (need_mask) {
          unsigned pmask[8], some = 0u;
          block_masks(sPM[wave], kb, hi, pmask);
#pragma unroll
          for (int e = 0; e < 8; ++e) some |= pmask[e];
          seen = __any(some != 0u);
#pragma unroll
          for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb) sacc[qb][r] = (pmask[r >> 1] >> (16 * (r & 1)) & 1u) ? sacc[qb][r] : IM_NEG_INF;
        }
        if (!seen) continue;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) m[qb] = clamp_ref(row_max(sacc[qb]) + REF_OFF);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) set_reference(qb, -m[qb]);
      }
    }
    while (seen && keys > 0) {
      const unsigned vta = (vt_tile & (unsigned)(uintptr_t)sV) + vt0, vtb = (vt_tile & (unsigned)(uintptr_t)sV) + vt1;
      // The tile is processed as two blocks of 32 keys, each S^T -> softmax -> O^T (KS = 2: one by each of two waves).
      auto block = [&](int kb) __attribute__((always_inline)) {
        f32x16 sacc[QB];
        scores(sacc, kb);
        // ---- softmax ----
        bf16x8 pb[QB][2];
        float rs[QB];
        unsigned pmask[8];   // the validity of the keys of a packed pair of probabilities
        if (need_mask) block_masks(sPM[wave], kb, hi, pmask);
        // P^T operands of a query block from its scores, 0 for a masked key whatever its row holds.  Not 0 on a lane whose row is to
        // move its reference: by a bit of the packed probabilities, or by the lane's part of the row sum, which is taken over
        // the bf16-rounded probabilities (the values that multiply V) with two-element dot products against (1, 1).
        auto exponentiate = [&](int qb) __attribute__((always_inline)) {
          float p[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) p[r] = fast_exp2(sacc[qb][r]);
          pb[qb][0] = pack8(p);
          pb[qb][1] = pack8(p + 8);
          if (need_mask) {
            pb[qb][0] = and_bf16x8(pb[qb][0], pmask);
            pb[qb][1] = and_bf16x8(pb[qb][1], pmask + 4);
          }
          if (ONES) return (or_bf16x8(pb[qb][0]) | or_bf16x8(pb[qb][1])) & 0x40004000u;
          rs[qb] = sum_bf16x8(pb[qb][1], sum_bf16x8(pb[qb][0], 0.f));
          return rs[qb] > 0x1p24f ? 1u : 0u;
        };
        unsigned over = 0u;
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) over |= exponentiate(qb);
        if (__builtin_expect(__any(over != 0u), 0)) {
          asm volatile("" ::: "memory");  // a real branch: nothing of it is to be executed speculatively
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb)
            if (m[qb] == -BF16_MAX) set_reference(qb, 0.f);
          scores(sacc, kb);   // again, so that the registers of these are free above
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) {
            if (need_mask)
#pragma unroll
              for (int r = 0; r < 16; ++r) sacc[qb][r] = (pmask[r >> 1] >> (16 * (r & 1)) & 1u) ? sacc[qb][r] : IM_NEG_INF;
            // Rows that move: without a reference so far, or with a maximum 2^8 above the one that theirs was taken from.  The others
            // get the same probabilities again.
            const bool first = m[qb] == -BF16_MAX;
            const float mx = row_max(sacc[qb]), from = first ? 0.f : m[qb];
            const bool upd = first ? mx > IM_NEG_INF : mx > 8.f - REF_OFF;
            const float to = clamp_ref(from + mx + REF_OFF), shift = upd ? to - from : 0.f, alpha = first ? 0.f : fast_exp2(-shift);
            if (upd) m[qb] = to;
            set_reference(qb, -m[qb]);
            if (QB > 1 && !__any(upd)) continue;
            l[qb] *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
              for (int r = 0; r < 16; ++r) oacc[db][qb][r] *= alpha;
#pragma unroll
            for (int r = 0; r < 16; ++r) sacc[qb][r] -= shift;
            exponentiate(qb);
          }
        }
        if (!ONES)
#pragma unroll
          for (int qb = 0; qb < NQB; ++qb) l[qb] += rs[qb];
        // ---- O^T += V^T P^T over the 32 keys of the block ----
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const bf16x8 a = ONES ? lds_frag_tr_at(vta, vtb, (kb * 32 + half * 16) * SW_LD * 2)
                                  : lds_frag_tr_sw(sV, kb * 32 + half * 16, (db0 + db) * 32, lane);
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb) oacc[db][qb] = mfma32(a, pb[qb][half], oacc[db][qb]);
          }
      };
      if (KS == 2) {
        if (kg == 0 || keys > 32) block(kg);
      } else {
        block(0);
        if (keys > 32) block(1);
      }
      if (keys1 < 0) break;
      advance();
    }
    if (ONES) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) l[qb] = (wo & 31) == 0 ? oacc[0][qb][8] : oacc[0][qb][0];   // rows 16.. / 0.. of O^T: not the head's
    }
  };

  if (HALF && half_tile) stream(std::integral_constant<int, 1>{});
  else stream(std::integral_constant<int, QB>{});

  // ---- epilogue: normalise, write O rows, O^T columns and the log-sum-exp ----
  if (KS == 2) {
    // The two waves of a row block have every other key block each: a wave gives the other one 32 of the 64 columns,
    // and both sums go together with their references (without one both are 0).
    __syncthreads();   // the ring is read no more
    float* ex = (float*)sT;   // per wave: 16 x 64 of the accumulator, then l and m
    constexpr int EX = 18 * 64;
#pragma unroll
    for (int r = 0; r < 16; ++r) ex[wave * EX + r * 64 + lane] = kg ? oacc[0][0][r] : oacc[NDB - 1][0][r];
    ex[wave * EX + 16 * 64 + lane] = l[0];
    ex[wave * EX + 17 * 64 + lane] = m[0];
    __syncthreads();
    const float* in = ex + (wave ^ 1) * EX;
    const float m1 = in[17 * 64 + lane], l1 = in[16 * 64 + lane], mm = fmaxf(m[0], m1);
    const float a0 = m[0] == IM_NEG_INF ? 0.f : fast_exp2(m[0] - mm), a1 = m1 == IM_NEG_INF ? 0.f : fast_exp2(m1 - mm);
    m[0] = mm;
    l[0] = a0 * l[0] + a1 * l1;
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[0][0][r] = a0 * (kg ? oacc[NDB - 1][0][r] : oacc[0][0][r]) + a1 * in[r * 64 + lane];
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float lt = ONES ? l[qb] : l[qb] + __shfl_xor(l[qb], 32, 64);
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const int row = qrow[qb];
    if (row >= qlen) continue;
    const long t = qrow0 + row;
    if (hi == 0 && kg == 0 && lse2) lse2[(g.cu ? (long)h * g.R : ((long)b * g.H + h) * g.T) + qoff + row] = lt > 0.f ? -(m[qb] + log2f(lt)) : IM_NEG_INF;  // negated
#pragma unroll
    for (int db = 0; db < NDB / KS; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int dh0 = (KS == 2 ? kg : db0 + db) * 32 + 8 * i + 4 * hi;  // column inside the 64-column group
        if (DH < 64 && (dh0 < wo || dh0 >= wo + DH)) continue;
        float v[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) v[jj] = oacc[db][qb][4 * i + jj] * inv;
        const u32x2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *(u32x2*)(O + t * ldo + cg * 64 + dh0) = pk;
      }
  }
}

// ------------------------------------------------------------------------------------------
// dQ (and delta = rowsum(dO * O)).  Same ownership as the forward: lane <-> query row.
// With the two constant accumulator seeds (negated lse, -delta: 32 registers; 167 in all, three workgroups per CU) the softmax is exp2,
// one multiply and the bf16 pack per score; without them the kernel is 7 % slower.
template <int QB, int NST, int WGS, int KS = 1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WGS, WGS))) void mfma_dq_kernel(Geo g, const bf16_t* __restrict__ QKV, long ld,
                                                      const bf16_t* __restrict__ O,
                                                      const bf16_t* __restrict__ dO, long ldo,
                                                      const float* __restrict__ lse2,
                                                      const int32_t* __restrict__ valid_len,
                                                      const uint8_t* __restrict__ key_pad, float* __restrict__ delta,
                                                      bf16_t* __restrict__ dQKV, long ldg) {
  __shared__ __attribute__((aligned(1024))) bf16_t sT[NST * RING_STAGE];  // per stage: K tile, V tile
  __shared__ __attribute__((aligned(256))) unsigned sKP[NST * KT];        // per stage: key_pad bytes of the 64 keys, one per dword
  __shared__ __attribute__((aligned(16))) unsigned sPM[4][KT / 2];        // key masks of the wave's tile
  __shared__ SegTable sSeg[4];
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: branches on it are wave-uniform
  int tile, h, b;
  xcd_tile_index(g.q_tile_prefix, g.q_nord, g.cu != nullptr, g.even_cus, tile, h, b);
  constexpr int WG_ROWS = 128 * QB / KS;
  static_assert(KS == 1 || QB == 1, "");
  const int rb = wave / KS, kg = wave % KS;   // row block of the tile, key block of a stage (KS = 2)
  int qs, q0, ord;
  tile_segment(g.q_order, g.q_tile_prefix, g.q_nord, tile, qs, q0, ord);
  q0 *= WG_ROWS;
  int qoff, qlen;
  SegTable& sg = sSeg[wave];
  const unsigned row_set = seg_rows_table(sg, g, b, g.q_live[qs], lane, qs, qoff, qlen);
  if (q0 >= qlen) return;  // packed rows: this batch element's segment ends before the tile
  const int d = g.d;
  const long row_b = g.cu ? 0 : (long)b * g.T, qrow0 = row_b + qoff;   // rows of the batch element, of segment qs
  const long stat0 = (g.cu ? (long)h * g.R : ((long)b * g.H + h) * g.T) + qoff;

  constexpr int NS = 4, NDB = 2;   // k-steps of the scores, 32-column blocks of the gradients

  KvStream<NST> ring(sg, sT, sKP, QKV + row_b * ld + d, key_pad ? key_pad + row_b : nullptr, ld, d, wave, lane, h);
  const int seg1 = row_set ? __builtin_ctz(row_set) : 0;   // its first tile goes ahead of everything
  if (row_set) ring.first(seg1);
  const int valid = valid_len ? valid_len[b * g.n_seg + min(lane, g.n_seg - 1)] : 0;

  bf16x8 qreg[QB][NS], greg[QB][NS];
  int qrow[QB];
  float ls[QB], dl[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    qrow[qb] = q0 + (rb * QB + qb) * 32 + lo;
    const int rc = min(qrow[qb], qlen - 1);
    const long t = qrow0 + rc;
    const bf16_t* p = QKV + t * ld + h * 64 + hi * 8;
    const bf16_t* pg = dO + t * ldo + h * 64 + hi * 8;
    const bf16_t* po = O + t * ldo + h * 64 + hi * 8;
    float acc = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      u32x4 qv = *(const u32x4*)(p + s * 16);
      u32x4 gv = *(const u32x4*)(pg + s * 16);
      const u32x4 ov = *(const u32x4*)(po + s * 16);
      qreg[qb][s] = as_bf16x8(qv);
      greg[qb][s] = as_bf16x8(gv);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc = fmaf(__uint_as_float(gv[e] << 16), __uint_as_float(ov[e] << 16), acc);
        acc = fmaf(__uint_as_float(gv[e] & 0xffff0000u), __uint_as_float(ov[e] & 0xffff0000u), acc);
      }
    }
    acc += __shfl_xor(acc, 32, 64);
    dl[qb] = acc;
    const long li = stat0 + rc;
    const float lv = lse2[li];
    ls[qb] = lv;  // negated log2-sum-exp; -inf for a row without valid keys: every probability is exactly zero
    if (hi == 0 && kg == 0 && qrow[qb] < qlen) delta[li] = -acc;  // see the dK/dV kernel
  }

  f32x16 dqacc[NDB][QB], nlb[QB], ndb[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dqacc[db][qb][r] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { nlb[qb][r] = ls[qb]; ndb[qb][r] = -dl[qb]; }
  }

  const int prow = perm32(lo);
  // The compiler does not see the asynchronous copies in its vmcnt bookkeeping: consuming the
  // loaded registers here makes it wait for their (ordinary) loads now, not inside the ring loop.
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" :: "v"(qreg[qb][s]), "v"(greg[qb][s]));
    asm volatile("" :: "v"(ls[qb]), "v"(dl[qb]));
  }

  const unsigned key_set = valid_len ? seg_lens_table(sg, valid, row_set, lane) : row_set;
  int cslot = 0, keys1 = -1;
  if (row_set) {   // the first stage is under way
    keys1 = ring.begin(seg1, key_set);
    if (keys1 == 0) {   // the segment has no valid key: what its rows hold must not meet a dS of 0
      cslot = 1;
      keys1 = ring.issue();
      if (keys1 < 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copy ends before its stage is used otherwise
    }
  }
  int keys2 = NST > 2 ? ring.issue() : -1;
  while (keys1 >= 0) {
    ring_wait(keys2 >= 0, ring.kp_copy);
    const int keys = keys1;
    keys1 = keys2;
    (NST > 2 ? keys2 : keys1) = ring.issue();
    const bf16_t* sK = sT + cslot * RING_STAGE;
    const bf16_t* sV = sK + KT * SW_LD;
    cslot = (cslot + 1 == NST) ? 0 : cslot + 1;
    const unsigned* kp = sKP + (sK - sT) / RING_STAGE * KT;
    {
      const bool need_mask = keys < KT || key_pad != nullptr;
      if (need_mask) tile_masks(sPM[wave], key_pad ? kp : nullptr, keys);
      // two blocks of 32 keys, each S^T, dP^T -> dS^T -> dQ^T, so that one block of dS^T is live at a time
#pragma unroll
      for (int kk = 0; kk < 2 / KS; ++kk) {
        const int kb = KS == 1 ? kk : kg;
        if (kb == 1 && keys <= 32) break;
        bf16x8 dsb[QB][2];
        // The chains start from the row's negated lse resp. -delta (nlb, ndb: the lane's value in all 16
        // registers), so they end as S^T - lse and dP^T - delta.
        f32x16 sacc[QB], pacc[QB];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 ak = lds_frag_sw(sK, kb * 32, prow, 2 * s + hi);
          const bf16x8 av = lds_frag_sw(sV, kb * 32, prow, 2 * s + hi);
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            sacc[qb] = mfma32(ak, qreg[qb][s], s == 0 ? nlb[qb] : sacc[qb]);   // S^T  = K Q^T
            pacc[qb] = mfma32(av, greg[qb][s], s == 0 ? ndb[qb] : pacc[qb]);   // dP^T = V dO^T
          }
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          float ds[16];
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float p = fast_exp2(sacc[qb][r]);
            ds[r] = p * pacc[qb][r];
          }
          dsb[qb][0] = pack8(ds);
          dsb[qb][1] = pack8(ds + 8);
          if (need_mask) {  // wave-uniform: tail tile or key_pad present; a masked key's dS is 0 whatever its row holds
            unsigned pmask[8];
            block_masks(sPM[wave], kb, hi, pmask);
            dsb[qb][0] = and_bf16x8(dsb[qb][0], pmask);
            dsb[qb][1] = and_bf16x8(dsb[qb][1], pmask + 4);
          }
        }
        // dQ^T += K^T dS^T over the 32 keys of the block
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const bf16x8 a = lds_frag_tr_sw(sK, kb * 32 + half * 16, db * 32, lane);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) dqacc[db][qb] = mfma32(a, dsb[qb][half], dqacc[db][qb]);
          }
      }
    }
  }

  if (KS == 2) {   // as in the forward: a wave gives the other one of its row block 32 of the 64 columns
    __syncthreads();
    float* ex = (float*)sT;
#pragma unroll
    for (int r = 0; r < 16; ++r) ex[wave * 1024 + r * 64 + lane] = kg ? dqacc[0][0][r] : dqacc[NDB - 1][0][r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r)
      dqacc[0][0][r] = (kg ? dqacc[NDB - 1][0][r] : dqacc[0][0][r]) + ex[(wave ^ 1) * 1024 + r * 64 + lane];
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int row = qrow[qb];
    if (row >= qlen) continue;
    const long t = qrow0 + row;
#pragma unroll
    for (int db = 0; db < NDB / KS; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int dh0 = (KS == 2 ? kg : db) * 32 + 8 * i + 4 * hi;  // column inside the 64-column group
        float v[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) v[jj] = dqacc[db][qb][4 * i + jj] * g.scale;
        const u32x2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        *(u32x2*)(dQKV + t * ldg + h * 64 + dh0) = pk;
      }
  }
}

// ------------------------------------------------------------------------------------------
// dK, dV.  Each wave owns KB blocks of 32 key rows (lane <-> key row) and streams
// the query rows of every query segment that reads this key segment.  A key tile
// has exactly one producer, so the result is deterministic without atomics.
//
// Ring stage = Q tile, dO tile (see RING_STAGE) plus the 64 lse and 64 delta values of the rows.
// The delta buffer holds -delta (the dQ kernel writes it so): the dP accumulator
// starts from it, so the MFMA chain ends as dP - delta and no separate subtraction is needed.
__device__ const float k_neg_inf = -__builtin_inff();

template <int KB, int KS = 1>
__global__ __launch_bounds__(256, 3) void mfma_dkv_kernel(Geo g, const bf16_t* __restrict__ QKV, long ld,
                                                       const bf16_t* __restrict__ dO, long ldo,
                                                       const float* __restrict__ lse2, const float* __restrict__ delta,
                                                       const int32_t* __restrict__ valid_len,
                                                       const uint8_t* __restrict__ key_pad, bf16_t* __restrict__ dQKV,
                                                       long ldg) {
  __shared__ __attribute__((aligned(1024))) bf16_t sT[RING_NST * RING_STAGE];
  __shared__ __attribute__((aligned(256))) float sLD[RING_NST * 2 * KT];  // per stage: lse[64], delta[64]
  __shared__ SegTable sSeg[4];
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: branches on it are wave-uniform
  int tile, h, b;
  xcd_tile_index(g.k_tile_prefix, g.k_nord, g.cu != nullptr, g.even_cus, tile, h, b);
  constexpr int WG_ROWS = 128 * KB / KS;
  static_assert(KS == 1 || KB == 1, "");
  const int rb = wave / KS, rg = wave % KS;   // key block of the tile, row block of a stage (KS = 2)
  int ks, k0, ord;
  tile_segment(g.k_order, g.k_tile_prefix, g.k_nord, tile, ks, k0, ord);
  k0 *= WG_ROWS;
  int koff, klen_seg;
  SegTable& sg = sSeg[wave];
  const unsigned row_set = seg_rows_table(sg, g, b, g.k_live[ks], lane, ks, koff, klen_seg);
  if (k0 >= klen_seg) return;  // packed rows: this batch element's segment ends before the tile
  const int d = g.d;
  const long row_b = g.cu ? 0 : (long)b * g.T, krow0 = row_b + koff;   // rows of the batch element, of segment ks
  const long stat_b = g.cu ? (long)h * g.R : ((long)b * g.H + h) * g.T;

  constexpr int NS = 4, NDB = 2;   // k-steps of the scores, 32-column blocks of the gradients

  const RingLane rl = ring_lane(wave, lane, h);
  const unsigned ldb = (unsigned)ld * 2u, ldob = (unsigned)ldo * 2u;  // row pitches in bytes
  const RingLaneOff rlo = ring_lane_off(rl, ldb, ldob);
  TileCursor ic = {row_set, 0, 0};
  int islot = 0, cslot = 0;
  RingFeed feed = {nullptr, nullptr, 0};
  const float* feed_l = nullptr;  // lse and delta of the next tile's first row
  const float* feed_d = nullptr;
  auto next_seg = [&]() {  // Q and dO rows, lse and delta of the next segment
    if (!cursor_next_seg(ic, sg)) return;
    const int off = seg_get(sg.off, ic.seg);
    feed.a = (const char*)(QKV + (row_b + off) * ld);
    feed.b = (const char*)(dO + (row_b + off) * ldo);
    feed.rows = ic.left;
    feed_l = lse2 + stat_b + off;
    feed_d = delta + stat_b + off;
  };
  next_seg();
  auto issue = [&]() {   // requests the next stage; returns the rows left of its segment, -1 if there is none
    if (ic.left <= 0) return -1;
    const int rows = ic.left;
    // negated lse (wave 0) and delta (wave 1), one float per lane.  Rows past the segment read -inf
    // as negated lse, so their probabilities are exactly zero.
    if (wave < 2) {
      float* dst = sLD + islot * 2 * KT + wave * KT;
      if (feed.rows >= KT) {
        dma4_off(wave == 0 ? feed_l : feed_d, (unsigned)lane * 4u, dst);
      } else {
        const float* src = (wave == 0) ? (lane < feed.rows ? feed_l + lane : &k_neg_inf) : feed_d + min(lane, feed.rows - 1);
        dma4(src, dst);
      }
    }
    feed_l += KT;
    feed_d += KT;
    ring_feed_issue(rl, rlo, feed, ldb, ldob, wave, sT + islot * RING_STAGE);
    islot = (islot + 1 == RING_NST) ? 0 : islot + 1;
    ic.left -= KT;
    if (ic.left <= 0) next_seg();
    return rows;
  };
  int rows1 = issue();   // the first stage, ahead of everything

  bf16x8 kreg[KB][NS], vreg[KB][NS];
  int krow[KB];
  bool kvalid[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    krow[kb] = k0 + (rb * KB + kb) * 32 + lo;
    const int rc = min(krow[kb], klen_seg - 1);
    const long t = krow0 + rc;
    const bf16_t* p = QKV + t * ld + d + h * 64 + hi * 8;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      u32x4 kv = *(const u32x4*)(p + s * 16), vv = *(const u32x4*)(p + d + s * 16);
      kreg[kb][s] = as_bf16x8(kv);
      vreg[kb][s] = as_bf16x8(vv);
    }
    bool ok = krow[kb] < klen_seg;
    if (ok && valid_len) ok = krow[kb] < valid_len[b * g.n_seg + ks];
    if (ok && key_pad) ok = key_pad[t] == 0;
    kvalid[kb] = ok;
  }

  f32x16 dkacc[NDB][KB], dvacc[NDB][KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) { dkacc[db][kb][r] = 0.f; dvacc[db][kb][r] = 0.f; }

  // The compiler does not see the asynchronous copies in its vmcnt bookkeeping.  Consuming the
  // K / V registers here makes it wait for their (ordinary) loads now, before the ring starts,
  // instead of draining the ring with a vmcnt(0) at their first use inside the loop.
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" :: "v"(kreg[kb][s]), "v"(vreg[kb][s]));

  int rows2 = issue();
  const int prow = perm32(lo);
  while (rows1 >= 0) {
    // Copies complete in issue order.  The wanted stage is complete once at most the copies of the
    // stage requested after it (4 tile chunks, plus 1 on the waves that fetch lse / delta) are
    // outstanding.  Behind the barrier the stage is visible to all waves, and everyone is done with the one before.
    ring_wait(rows2 >= 0, wave < 2);
    const int rows = rows1;
    rows1 = rows2;
    rows2 = issue();  // refills the slot of the stage consumed before
    const bf16_t* sQ = sT + cslot * RING_STAGE;
    const bf16_t* sG = sQ + KT * SW_LD;
    const float* sL = sLD + cslot * 2 * KT;
    const float* sD = sL + KT;
    cslot = (cslot + 1 == RING_NST) ? 0 : cslot + 1;
#pragma unroll
    for (int qq = 0; qq < 2 / KS; ++qq) {
      const int qb = KS == 1 ? qq : rg;
      if (qb == 1 && rows <= 32) break;
      // negated lse / -delta of the query rows of the block: register r of an accumulator holds row
      // (r / 8) * 16 + hi * 8 + r % 8.  Both go straight into the accumulators: the MFMA chains then end as S - lse and
      // dP - delta, and neither needs a vector instruction per element.
      auto rows4 = [&](const float* base, int r4) {   // values of registers 4 r4 .. 4 r4 + 3
        return *(const float4*)&base[qb * 32 + (r4 >> 1) * 16 + hi * 8 + (r4 & 1) * 4];
      };
      bf16x8 pb[KB][2], dsb[KB][2];
      f32x16 sacc[KB], pacc[KB];
      float D[16], NL[16];
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const float4 d4 = rows4(sD, r4);
        D[4 * r4] = d4.x; D[4 * r4 + 1] = d4.y; D[4 * r4 + 2] = d4.z; D[4 * r4 + 3] = d4.w;
        const float4 l4 = rows4(sL, r4);
        NL[4 * r4] = l4.x; NL[4 * r4 + 1] = l4.y; NL[4 * r4 + 2] = l4.z; NL[4 * r4 + 3] = l4.w;
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[kb][r] = NL[r]; pacc[kb][r] = D[r]; }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const bf16x8 aq = lds_frag_sw(sQ, qb * 32, prow, 2 * s + hi);
        const bf16x8 ag = lds_frag_sw(sG, qb * 32, prow, 2 * s + hi);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
          sacc[kb] = mfma32(aq, kreg[kb][s], sacc[kb]);   // S  = Q K^T
          pacc[kb] = mfma32(ag, vreg[kb][s], pacc[kb]);   // dP = dO V^T
        }
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        float p[16], ds[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          p[r] = fast_exp2(sacc[kb][r]);
          ds[r] = p[r] * pacc[kb][r];
        }
        pb[kb][0] = pack8(p); pb[kb][1] = pack8(p + 8);
        dsb[kb][0] = pack8(ds); dsb[kb][1] = pack8(ds + 8);
      }
      // dV^T += dO^T P ; dK^T += Q^T dS   (contraction over the 32 query rows of this block)
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const bf16x8 agt = lds_frag_tr_sw(sG, qb * 32 + half * 16, db * 32, lane);
          const bf16x8 aqt = lds_frag_tr_sw(sQ, qb * 32 + half * 16, db * 32, lane);
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) {
            dvacc[db][kb] = mfma32(agt, pb[kb][half], dvacc[db][kb]);
            dkacc[db][kb] = mfma32(aqt, dsb[kb][half], dkacc[db][kb]);
          }
        }
    }
  }

  const int lane_e = lane_id(), hi_e = lane_e >> 5;
  if (KS == 2) {   // the two waves of a key block have every other row block each: one finishes dK, the other dV
    __syncthreads();
    float* ex = (float*)sT;
    f32x16 sum[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) ex[(wave * NDB + db) * 1024 + r * 64 + lane_e] = rg ? dkacc[db][0][r] : dvacc[db][0][r];
    __syncthreads();
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sum[db][r] = (rg ? dvacc[db][0][r] : dkacc[db][0][r]) + ex[((wave ^ 1) * NDB + db) * 1024 + r * 64 + lane_e];
    const int krow_e = k0 + rb * 32 + (lane_e & 31);
    if (krow_e >= klen_seg) return;
    const bool ok = kvalid[0];   // see below
    const float z = rg ? 1.f : 0.69314718055994530942f;
    bf16_t* p = dQKV + (krow0 + krow_e) * ldg + (rg ? 2 * d : d) + h * 64;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(u32x2*)(p + db * 32 + 8 * i + 4 * hi_e) = ok ? u32x2{pack_bf16(sum[db][4 * i] * z, sum[db][4 * i + 1] * z),
                                                             pack_bf16(sum[db][4 * i + 2] * z, sum[db][4 * i + 3] * z)} : u32x2{0u, 0u};
    return;
  }
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int row = k0 + (rb * KB + kb) * 32 + (lane_e & 31);
    if (row >= klen_seg) continue;
    const long t = krow0 + row;
    // dK = scale dS^T Q, and the staged Q rows are scale log2(e) Q: the accumulator needs a factor ln 2.  A masked key's accumulators
    // are dropped, not multiplied by 0: no log-sum-exp bounds its scores, and 2^(S - lse) may have been infinite.
    constexpr float zk = 0.69314718055994530942f;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int dh0 = db * 32 + 8 * i + 4 * hi_e;  // column inside the 64-column group
        const u32x2 pk = {pack_bf16(dkacc[db][kb][4 * i] * zk, dkacc[db][kb][4 * i + 1] * zk),
                          pack_bf16(dkacc[db][kb][4 * i + 2] * zk, dkacc[db][kb][4 * i + 3] * zk)};
        const u32x2 pv = {pack_bf16(dvacc[db][kb][4 * i], dvacc[db][kb][4 * i + 1]), pack_bf16(dvacc[db][kb][4 * i + 2], dvacc[db][kb][4 * i + 3])};
        *(u32x2*)(dQKV + t * ldg + d + h * 64 + dh0) = kvalid[kb] ? pk : u32x2{0u, 0u};
        *(u32x2*)(dQKV + t * ldg + 2 * d + h * 64 + dh0) = kvalid[kb] ? pv : u32x2{0u, 0u};
      }
  }
}

// ---- host launchers ----
// Launch shapes, each chosen by measurement at B = 8, segments 512 / 2048 / 2048, d = 512, 8 heads:
//   forward, head dim 64: 1 query block per wave, 4 waves, a 2-stage ring and 128 registers, so that four
//     workgroups (16 waves) share a CU -- 10 % faster than 3 stages at three workgroups; 8-wave workgroups
//     (256 query rows) were slower;
//   forward, sub-head mode: 2 query blocks per wave (half the K/V tile traffic per score), 2 stages, 4 workgroups (128
//     registers; four layers of 32 x 50/500/375 rows, no padding, intra-modal mask, before the rows had references: 169 us with 3
//     stages and 3 workgroups, 160 with 2 and 4, 150 with the row sums on the matrix cores);
//   dQ, head dim 64: 3 stages, 3 workgroups per CU, accumulators seeded with -lse and -delta (unseeded: 7 % slower;
//     4 workgroups need spills);
//   dK/dV: 1 key block per wave, 3 workgroups per CU.  (Sub-head backward: mfma_attn_sub.hip.)
constexpr int FWD_QB = 1, FWD_QB_SUB = 2, DQ_QB = 1, DKV_KB = 1;
constexpr int FWD_WGS = 4, FWD_SUB_WGS = 4;           // workgroups per CU, head dimension 64 and sub-head mode
constexpr int DQ_NST = 3, DQ_WGS = 3;                 // dQ at head dim 64
// CUs per XCD if a launch of `wgs` workgroups is dealt out evenly (see xcd_tile_index), else 0: all resident with `per_cu`
// workgroups on a CU, of different lengths.  Lengths of packed rows are not known here.
static unsigned even_cus(const Geo& g, int nord, long wgs, int per_cu) {
  const int cus = cu_count();
  return !g.cu && nord > 1 && cus % 8 == 0 && wgs > cus && wgs <= (long)per_cu * cus ? (unsigned)cus / 8u : 0u;
}
// Head dimension 64, few workgroups: tiles of 64 rows instead of 128, the two 32-row blocks of a stage going to two waves of
// a row block, which add their accumulators at the end (KS = 2).  With about one workgroup per CU a stage is a chain of
// latencies (barrier, LDS reads, dependent matrix instructions, exponentials) with one wave per SIMD: 1.1 us for a forward
// stage, 1.4 for dK/dV, 0.8 and 0.9 for half of it.  The copies per score double, and so the line is where the chip is full
// without it; us for a training step, 128 / 64 rows, at 256 CUs:
//   workgroups of 128 rows   104 (333/1501/1290 x 4 heads)  204 / 155      288 (512/2048/2048 x 8)  193 / 178
//                            312                            227 / 192      320 (40/120/300 x 4)      85 / 82
//                            416                            238 / 239      432 (50/500/500 x 4, layer) 255 / 257
//                            624                            286 / 319      576 (512/2048/2048 x 8)  269 / 264
static bool split_rows(const Geo& g, const int* prefix, int nord) {
  return g.dh == 64 && 2 * (long)prefix[nord] * g.H * g.B <= 3L * cu_count();
}
// Tables of a schedule for tiles of `rows` rows (build_geo's for another height)
static void retile(const Geo& g, const int* order, int nord, int rows, int* prefix) {
  for (int k = 0; k < nord; ++k) prefix[k + 1] = prefix[k] + (g.seg_len[order[k]] + rows - 1) / rows;
}
// sub-head mode: four heads of a 64-column group per workgroup, 64-row tiles
int mfma_fwd_tile_rows(int dh) { return dh == 64 ? 128 * FWD_QB : 32 * FWD_QB_SUB; }
int mfma_dq_tile_rows() { return 128 * DQ_QB; }
int mfma_dkv_tile_rows() { return 128 * DKV_KB; }

// Sub-head forward, padded rows.  The workgroups of the query segment with the longest
// key range finish last; when they are few (at most a quarter of the workgroup slots -- segments 50 / 500 / 375 under
// the forward inter-modal mask: the one tile of the 50 text rows reads 500 keys, the eight tiles of the vision rows
// 375) and clearly the longest, their tiles become 32 rows tall: twice the workgroups, one query block per wave,
// a shorter tail of the launch (measured: -3 % at that shape).  A half-height workgroup does more work per score (the
// K/V fragments are read per block), so a launch whose long workgroups are many -- it is bound by the CUs'
// instruction issue, not by its last workgroup -- keeps the full tiles (halving them there measured +3 %).
static void fwd_half_tiles(Geo& g) {
  g.q_half = 0;
  if (g.cu || g.q_nord < 2) return;
  const int rows = 32 * FWD_QB_SUB;
  const long units = (long)g.B * (g.H / 4), slots = (long)FWD_SUB_WGS * cu_count();
  long len[IM_MAX_SEG], tiles[IM_MAX_SEG];
  int longest = 0;
  for (int k = 0; k < g.q_nord; ++k) {
    const int sgm = g.q_order[k];
    len[k] = 0;
    for (int j = 0; j < g.n_seg; ++j)
      if ((g.q_live[sgm] >> j) & 1u) len[k] += (g.seg_len[j] + KT - 1) / KT;
    tiles[k] = (g.seg_len[sgm] + rows - 1) / rows;
    if (len[k] > len[longest]) longest = k;
  }
  long second = 0;
  for (int k = 0; k < g.q_nord; ++k)
    if (k != longest && len[k] > second) second = len[k];
  if (4 * len[longest] < 5 * second || 4 * tiles[longest] * units > slots) return;
  const long half_tiles = (g.seg_len[g.q_order[longest]] + rows / 2 - 1) / (rows / 2);
  g.q_half = 1u << longest;
  for (int k = 0; k < g.q_nord; ++k)
    g.q_tile_prefix[k + 1] = g.q_tile_prefix[k] + (int)(k == longest ? half_tiles : tiles[k]);
}

void launch_mfma_fwd(const Geo& g_in, const bf16_t* qkv, long ld, const int32_t* valid_len, const uint8_t* key_pad,
                     bf16_t* o, long ldo, float* lse2, hipStream_t st) {
  Geo g = g_in;
  g.q_half = 0;
  if (g.dh != 64) fwd_half_tiles(g);
  const bool split = split_rows(g, g.q_tile_prefix, g.q_nord);
  if (split) retile(g, g.q_order, g.q_nord, 64 * FWD_QB, g.q_tile_prefix);
  // query segments with no live block: output 0, lse -inf
  for (int s = 0; s < g.n_seg; ++s) {
    if (g.q_live[s]) continue;
    launch_zero_seg_rows(g, s, 1, o, ldo, 0, g.d, st);
    if (lse2) launch_fill_seg_stat(g, s, lse2, -__builtin_inff(), st);
  }
  const int nt = g.q_tile_prefix[g.q_nord];
  if (nt == 0) return;
  g.even_cus = g.dh == 64 ? even_cus(g, g.q_nord, (long)nt * g.H * g.B, FWD_WGS) : 0u;
  ProfScope ps(PF_ATTN_FWD, st);
  const dim3 grid(nt, g.H, g.B), gridw(nt, g.H / 4, g.B);
  if (split) hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB, 64, FWD_WGS, false, 2>), grid, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
  else if (g.dh == 64) hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB, 64, FWD_WGS, false>), grid, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
  else if (g.dh == 16) hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB_SUB, 16, FWD_SUB_WGS, false>), gridw, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
  else hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB_SUB, 8, FWD_SUB_WGS, false>), gridw, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
}

// Forward of two problems of the same shape (masks g0 / g1) in one launch; their rows follow each other in
// qkv, o and lse2 (2 B batch elements).  Sub-head mode and padded rows only; both masks must give every query
// segment a live block (same tile count), which the caller checks with mfma_fwd_pair_ok.
bool mfma_fwd_pair_ok(const Geo& g0, const Geo& g1) {
  if (g0.dh == 64 || g0.cu || g1.cu || g0.q_tile_prefix[g0.q_nord] != g1.q_tile_prefix[g1.q_nord]) return false;
  for (int s = 0; s < g0.n_seg; ++s)
    if (!g0.q_live[s] || !g1.q_live[s]) return false;
  return 2L * g0.B <= 65535;
}
void launch_mfma_fwd_pair(const Geo& g0, const Geo& g1, const bf16_t* qkv, long ld, const int32_t* valid_len,
                          const uint8_t* key_pad, bf16_t* o, long ldo, float* lse2, hipStream_t st) {
  Geo g = g0;
  g.pair_B = g0.B;
  g.q_nord2 = g1.q_nord;
  for (int i = 0; i < IM_MAX_SEG; ++i) { g.q_live2[i] = g1.q_live[i]; g.q_order2[i] = g1.q_order[i]; }
  for (int i = 0; i <= IM_MAX_SEG; ++i) g.q_tile_prefix2[i] = g1.q_tile_prefix[i];
  ProfScope ps(PF_ATTN_FWD, st);
  const dim3 gridw(g.q_tile_prefix[g.q_nord], g.H / 4, 2 * g.B);
  if (g.dh == 16) hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB_SUB, 16, FWD_SUB_WGS, true>), gridw, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
  else hipLaunchKernelGGL((mfma_fwd_kernel<FWD_QB_SUB, 8, FWD_SUB_WGS, true>), gridw, dim3(256), 0, st, g, qkv, ld, valid_len, key_pad, o, ldo, lse2);
}

void launch_mfma_bwd(const Geo& g_in, const bf16_t* qkv, long ld, const bf16_t* o, const bf16_t* d_o, long ldo,
                     const float* lse2, const int32_t* valid_len, const uint8_t* key_pad, float* delta, bf16_t* dqkv,
                     long ldg, hipStream_t st) {
  Geo g = g_in;
  if (g.dh != 64) {
    retile(g, g.q_order, g.q_nord, mfma_sub_dq_tile_rows(), g.q_tile_prefix);
    retile(g, g.k_order, g.k_nord, mfma_sub_dkv_tile_rows(g.dh), g.k_tile_prefix);
  }
  const bool split_q = split_rows(g, g.q_tile_prefix, g.q_nord), split_k = split_rows(g, g.k_tile_prefix, g.k_nord);
  if (split_q) retile(g, g.q_order, g.q_nord, 64 * DQ_QB, g.q_tile_prefix);
  if (split_k) retile(g, g.k_order, g.k_nord, 64 * DKV_KB, g.k_tile_prefix);
  for (int s = 0; s < g.n_seg; ++s) {
    if (!g.q_live[s])
      launch_zero_seg_rows(g, s, 1, dqkv, ldg, 0, g.d, st);
    if (!g.k_live[s])
      launch_zero_seg_rows(g, s, 1, dqkv, ldg, g.d, 2 * g.d, st);
  }
  const int nq = g.q_tile_prefix[g.q_nord], nk = g.k_tile_prefix[g.k_nord];
  if (nq == 0) return;
  if (g.dh != 64) {
    launch_mfma_sub_bwd(g, qkv, ld, o, d_o, ldo, lse2, valid_len, key_pad, delta, dqkv, ldg, st);
    return;
  }
  { ProfScope ps(PF_ATTN_DQ, st);
    const dim3 grid(nq, g.H, g.B);
    g.even_cus = even_cus(g, g.q_nord, (long)nq * g.H * g.B, DQ_WGS);
    if (split_q) hipLaunchKernelGGL((mfma_dq_kernel<DQ_QB, DQ_NST, DQ_WGS, 2>), grid, dim3(256), 0, st, g, qkv, ld, o, d_o, ldo, lse2, valid_len, key_pad, delta, dqkv, ldg);
    else hipLaunchKernelGGL((mfma_dq_kernel<DQ_QB, DQ_NST, DQ_WGS>), grid, dim3(256), 0, st, g, qkv, ld, o, d_o, ldo, lse2, valid_len, key_pad, delta, dqkv, ldg); }
  { ProfScope ps(PF_ATTN_DKV, st);
    const dim3 grid(nk, g.H, g.B);
    g.even_cus = even_cus(g, g.k_nord, (long)nk * g.H * g.B, 3);
    if (split_k) hipLaunchKernelGGL((mfma_dkv_kernel<DKV_KB, 2>), grid, dim3(256), 0, st, g, qkv, ld, d_o, ldo, lse2, delta, valid_len, key_pad, dqkv, ldg);
    else hipLaunchKernelGGL((mfma_dkv_kernel<DKV_KB>), grid, dim3(256), 0, st, g, qkv, ld, d_o, ldo, lse2, delta, valid_len, key_pad, dqkv, ldg); }
}

}  // namespace imattn
