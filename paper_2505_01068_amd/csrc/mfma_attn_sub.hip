// Backward of the bf16 matrix-core attention at head dimensions 8 and 16 ("sub-head": d % 64 == 0, a head is a slice of a
// 64-column group).  The products and their layout are those of mfma_attn.hip; what differs is what bounds them.  A score
// needs few matrix instructions (one 16-deep k-step for S and dP, one 32-row block for the gradients), so vector-instruction
// issue is the limit: exp2, one multiply and half a pack per gradient operand are what a score cannot do without, and
// everything else is taken off the vector ALU:
//  - The four waves of a workgroup are four heads of one 64-column group over the same rows, so that the streamed tiles serve
//    all four and tiles are 32 or 64 rows tall (segments like 50 / 500 / 375 leave 128-row tiles up to 60 % empty).
//  - The rows' statistics go through the matrix cores.  S - lse and dP - delta come out of the products: a statistic is the sum
//    of three bf16 numbers (exact to 2^-24 of it) that meet ones on the other side.  At head dimension 8 a k-step has eight slots
//    to spare, and the lane half that holds them supplies the parts and the ones; at 16 they are a matrix instruction of their
//    own.  Subtracting per score took 32 of dK/dV's 80 vector instructions per 32 x 32 scores, and in dQ the seed registers
//    that a third workgroup per CU had no room for.
//  - Key masks are an AND on packed gradients (tile_masks).
// One layer's training step at 32 x 50/500/375 rows, 8 heads of 8: dQ 25.9 -> 22.4 us, dK/dV 29.4 -> 23.4 us against 128-row tiles
// of one head per workgroup; what is left beside the scores is a prologue of some 300 vector instructions per wave of 4 to 8 stages.
#include <type_traits>
#include "mfma_attn_common.hpp"
#include "mfma_path.hpp"

namespace imattn {

__device__ const u32x4 k_ones_chunk = {ONES01, ONES2, 0u, 0u};

// Head of wave `wave` in unit hw of four heads, and where its columns lie: 64-column group, first column in it, k-step (16
// columns), 32-column block, the lane half of the k-step (head dimension 8)
struct SubHead { int h, cg, wo, s0, db0, half; };
template <int DH>
__device__ __forceinline__ SubHead sub_head(int hw, int wave) {
  const int h = hw * 4 + wave, wo = (h * DH) & 63;
  return {h, (h * DH) >> 6, wo, wo >> 4, wo >> 5, (wo >> 3) & 1};
}

// ------------------------------------------------------------------------------------------
// dQ and -delta = -rowsum(dO * O).  lane <-> query row; a wave owns 32 rows of its head.
//
// Four workgroups per CU (78 registers at head dimension 8, 100 at 16).  Two row blocks per wave and three workgroups: 21.8 against 22.4 us at 32 x 50/500/375 rows,
// 8 heads of 8, but 26.7 against 21.7 at 8 heads of 16.
constexpr int SUB_DQ_NST = 2, SUB_DQ_WGS = 4;
template <int DH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SUB_DQ_WGS, SUB_DQ_WGS))) void sub_dq_kernel(
    Geo g, const bf16_t* __restrict__ QKV, long ld, const bf16_t* __restrict__ O, const bf16_t* __restrict__ dO, long ldo,
    const float* __restrict__ lse2, const int32_t* __restrict__ valid_len, const uint8_t* __restrict__ key_pad,
    float* __restrict__ delta, bf16_t* __restrict__ dQKV, long ldg) {
  __shared__ __attribute__((aligned(1024))) bf16_t sT[SUB_DQ_NST * RING_STAGE];  // per stage: K tile, V tile
  __shared__ __attribute__((aligned(256))) unsigned sKP[SUB_DQ_NST * KT];        // per stage: key_pad bytes of the 64 keys, one per dword
  __shared__ __attribute__((aligned(16))) unsigned sPM[4][KT / 2];        // key masks of the wave's tile
  __shared__ __attribute__((aligned(16))) unsigned sOne[4];               // ones chunk: what the spare slots of K and V hold
  __shared__ SegTable sSeg[4];
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile, hw, b;
  xcd_tile_index(g.q_tile_prefix, g.q_nord, g.cu != nullptr, 0u, tile, hw, b);
  const SubHead sh = sub_head<DH>(hw, wave);
  int qs, q0, ord;
  tile_segment(g.q_order, g.q_tile_prefix, g.q_nord, tile, qs, q0, ord);
  q0 *= 32;
  int qoff, qlen;
  SegTable& sg = sSeg[wave];
  const unsigned row_set = seg_rows_table(sg, g, b, g.q_live[qs], lane, qs, qoff, qlen);
  if (q0 >= qlen) return;  // packed rows: this batch element's segment ends before the tile
  const int d = g.d;
  const long row_b = g.cu ? 0 : (long)b * g.T, qrow0 = row_b + qoff;   // rows of the batch element, of segment qs
  const long stat0 = (g.cu ? (long)sh.h * g.R : ((long)b * g.H + sh.h) * g.T) + qoff;
  const bool spare = DH == 8 && hi != sh.half;   // this lane half's slots of the k-step are not the head's

  KvStream<SUB_DQ_NST> ring(sg, sT, sKP, QKV + row_b * ld + d, key_pad ? key_pad + row_b : nullptr, ld, d, wave, lane, sh.cg);
  const int seg1 = row_set ? __builtin_ctz(row_set) : 0;   // its first tile goes ahead of everything
  if (row_set) ring.first(seg1);
  const int valid = valid_len ? valid_len[b * g.n_seg + min(lane, g.n_seg - 1)] : 0;

  // B operands: Q and dO rows, and the parts of -lse and -delta (in the spare slots, or a k-step of their own)
  const int row = q0 + lo, rc = min(row, qlen - 1);
  const long t = qrow0 + rc;
  const int col = sh.cg * 64 + sh.s0 * 16 + hi * 8;
  const u32x4 qv = *(const u32x4*)(QKV + t * ld + col), gv = *(const u32x4*)(dO + t * ldo + col);
  const u32x4 ov = *(const u32x4*)(O + t * ldo + col);
  const float lv = lse2[stat0 + rc];
  float acc = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc = fmaf(__uint_as_float(gv[e] << 16), __uint_as_float(ov[e] << 16), acc);
    acc = fmaf(__uint_as_float(gv[e] & 0xffff0000u), __uint_as_float(ov[e] & 0xffff0000u), acc);
  }
  if (spare) acc = 0.f;
  acc += __shfl_xor(acc, 32, 64);
  if (hi == 0 && row < qlen) delta[stat0 + rc] = -acc;
  const u32x2 lp = bf16_parts(lv), dp = bf16_parts(-acc);
  const u32x4 l4 = {lp[0], lp[1], 0u, 0u}, d4 = {dp[0], dp[1], 0u, 0u}, z = {0u, 0u, 0u, 0u};
  const bf16x8 qreg = as_bf16x8(spare ? l4 : qv), greg = as_bf16x8(spare ? d4 : gv);
  const bf16x8 ls = as_bf16x8(hi == 0 ? l4 : z), dl = as_bf16x8(hi == 0 ? d4 : z);
  const bf16x8 ones = as_bf16x8(u32x4{ONES01, ONES2, 0u, 0u});

  f32x16 dqacc;
#pragma unroll
  for (int r = 0; r < 16; ++r) dqacc[r] = 0.f;

  // Row fragments of K and V: byte offset in a tile of the lane's 16 bytes, or the ones
  const int prow = perm32(lo);
  const unsigned kf = spare ? (unsigned)(uintptr_t)sOne : (unsigned)(prow * SW_LD + (((2 * sh.s0 + hi) ^ sw_f(prow)) << 3)) * 2u;
  const unsigned kf_tile = spare ? 0u : ~0u;
  if (lane < 4) sOne[lane] = k_ones_chunk[lane];   // every wave, so that none waits for another

  // The compiler does not see the asynchronous copies in its vmcnt bookkeeping: consuming the loaded registers here makes it
  // wait for their (ordinary) loads now, not inside the ring loop.
  asm volatile("" :: "v"(qreg), "v"(greg), "v"(ls), "v"(dl));

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
  while (keys1 >= 0) {
    ring_wait(false);
    const int keys = keys1;
    keys1 = ring.issue();
    const bf16_t* sK = sT + cslot * RING_STAGE;
    const unsigned* kp = sKP + cslot * KT;
    cslot ^= 1;
    const bool need_mask = keys < KT || key_pad != nullptr;
    if (need_mask) tile_masks(sPM[wave], key_pad ? kp : nullptr, keys);
    const unsigned tile_at = (unsigned)(uintptr_t)sK;
    // two blocks of 32 keys, each S^T - lse, dP^T - delta -> dS^T -> dQ^T
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      if (kb == 1 && keys <= 32) break;
      const bf16x8 ak = lds_b128((kf_tile & (tile_at + kb * 32 * SW_LD * 2)) + kf);
      const bf16x8 av = lds_b128((kf_tile & (tile_at + (KT + kb * 32) * SW_LD * 2)) + kf);
      f32x16 sacc = DH == 8 ? f32x16{} : mfma32(ones, ls, f32x16{}), pacc = DH == 8 ? f32x16{} : mfma32(ones, dl, f32x16{});
      sacc = mfma32(ak, qreg, sacc);   // S^T  = K Q^T - lse
      pacc = mfma32(av, greg, pacc);   // dP^T = V dO^T - delta
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = fast_exp2(sacc[r]) * pacc[r];
      bf16x8 dsb[2] = {pack8(ds), pack8(ds + 8)};
      if (need_mask) {  // a masked key's dS is 0 whatever its row holds
        unsigned pmask[8];
        block_masks(sPM[wave], kb, hi, pmask);
        dsb[0] = and_bf16x8(dsb[0], pmask);
        dsb[1] = and_bf16x8(dsb[1], pmask + 4);
      }
#pragma unroll
      for (int half = 0; half < 2; ++half)   // dQ^T += K^T dS^T
        dqacc = mfma32(lds_frag_tr_sw(sK, kb * 32 + half * 16, sh.db0 * 32, lane), dsb[half], dqacc);
    }
  }

  if (row >= qlen) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int dh0 = sh.db0 * 32 + 8 * i + 4 * hi;  // column inside the 64-column group
    if (dh0 < sh.wo || dh0 >= sh.wo + DH) continue;
    *(u32x2*)(dQKV + (qrow0 + row) * ldg + sh.cg * 64 + dh0) =
        u32x2{pack_bf16(dqacc[4 * i] * g.scale, dqacc[4 * i + 1] * g.scale), pack_bf16(dqacc[4 * i + 2] * g.scale, dqacc[4 * i + 3] * g.scale)};
  }
}

// ------------------------------------------------------------------------------------------
// dK, dV.  lane <-> key row; a wave owns KB blocks of 32 key rows of its head and streams the query rows of every segment that
// reads them.  Two ring stages (Q tile, dO tile); the 64 rows' negated lse and -delta of a stage are the wave's own ordinary
// loads, one row per lane, requested with the stage and turned into parts when it is there.
template <int DH, int KB, int WGS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WGS, WGS))) void sub_dkv_kernel(
    Geo g, const bf16_t* __restrict__ QKV, long ld, const bf16_t* __restrict__ dO, long ldo, const float* __restrict__ lse2,
    const float* __restrict__ delta, const int32_t* __restrict__ valid_len, const uint8_t* __restrict__ key_pad,
    bf16_t* __restrict__ dQKV, long ldg) {
  __shared__ __attribute__((aligned(1024))) bf16_t sT[2 * RING_STAGE];
  __shared__ __attribute__((aligned(16))) u32x4 sSt[4][2 * KT];           // per head: parts of lse and of delta of a row, 16 bytes each
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tile, hw, b;
  xcd_tile_index(g.k_tile_prefix, g.k_nord, g.cu != nullptr, 0u, tile, hw, b);
  const SubHead sh = sub_head<DH>(hw, wave);
  int ks, k0, ord;
  tile_segment(g.k_order, g.k_tile_prefix, g.k_nord, tile, ks, k0, ord);
  k0 *= 32 * KB;
  // the segments of the batch element (seg_rows_table), in registers: four workgroups fill the LDS to the byte
  int soff = 0, srows = 0;
  if (g.cu) {
    const int32_t* c = g.cu + b * g.n_seg + min(lane, g.n_seg - 1);
    soff = c[0];
    srows = c[1] - c[0];
  } else {
#pragma unroll
    for (int s = 0; s < IM_MAX_SEG; ++s)
      if (lane == s) { soff = g.seg_off[s]; srows = g.seg_len[s]; }
  }
  const int koff = __builtin_amdgcn_readlane(soff, ks), klen_seg = __builtin_amdgcn_readlane(srows, ks);
  if (k0 >= klen_seg) return;  // packed rows: this batch element's segment ends before the tile
  unsigned rest = (unsigned)__ballot(lane < g.n_seg && ((g.k_live[ks] >> (lane & 31)) & 1u) && srows > 0);
  const int d = g.d;
  const long row_b = g.cu ? 0 : (long)b * g.T, krow0 = row_b + koff;   // rows of the batch element, of segment ks
  const long stat_b = g.cu ? (long)sh.h * g.R : ((long)b * g.H + sh.h) * g.T;
  const bool spare = DH == 8 && hi != sh.half;   // this lane half's slots of the k-step are not the head's

  const RingLane rl = ring_lane(wave, lane, sh.cg);
  const unsigned ldb = (unsigned)ld * 2u, ldob = (unsigned)ldo * 2u;
  const RingLaneOff rlo = ring_lane_off(rl, ldb, ldob);
  int slot = 0;
  RingFeed feed = {nullptr, nullptr, 0};
  const float *feed_l = nullptr, *feed_d = nullptr;  // lse and delta of the next tile's first row
  float lv = 0.f, dv = 0.f;                          // of the requested stage's row `lane`
  auto issue = [&]() __attribute__((always_inline)) {   // requests the next stage; returns the rows left of its segment, -1 if there is none
    if (feed.rows <= 0) {
      if (!rest) return -1;
      const int seg = __builtin_ctz(rest), off = __builtin_amdgcn_readlane(soff, seg);
      rest &= rest - 1;
      feed.a = (const char*)(QKV + (row_b + off) * ld);
      feed.b = (const char*)(dO + (row_b + off) * ldo);
      feed.rows = __builtin_amdgcn_readlane(srows, seg);
      feed_l = lse2 + stat_b + off;
      feed_d = delta + stat_b + off;
    }
    const int rows = feed.rows, r = min(lane_id(), rows - 1);
    ring_feed_issue(rl, rlo, feed, ldb, ldob, wave, sT + slot * RING_STAGE);
    lv = feed_l[r];
    dv = feed_d[r];
    feed_l += KT;
    feed_d += KT;
    slot ^= 1;
    return rows;
  };
  int rows1 = issue();   // ahead of everything

  // B operands: K and V rows, with the ones that the statistics' parts meet in the spare slots (or in a k-step of their own)
  const u32x4 one4 = {ONES01, ONES2, 0u, 0u}, z4 = {0u, 0u, 0u, 0u};
  bf16x8 kreg[KB], vreg[KB];
  const bf16x8 ones = as_bf16x8(hi == 0 ? one4 : z4);
  bool kvalid[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int krow = k0 + kb * 32 + lo, rc = min(krow, klen_seg - 1);
    const long t = krow0 + rc;
    const bf16_t* p = QKV + t * ld + d + sh.cg * 64 + sh.s0 * 16 + hi * 8;
    const u32x4 kv = *(const u32x4*)p, vv = *(const u32x4*)(p + d);
    kreg[kb] = as_bf16x8(spare ? one4 : kv);
    vreg[kb] = as_bf16x8(spare ? one4 : vv);
    bool ok = krow < klen_seg;
    if (ok && valid_len) ok = krow < valid_len[b * g.n_seg + ks];
    if (ok && key_pad) ok = key_pad[t] == 0;
    kvalid[kb] = ok;
  }
  f32x16 dkacc[KB], dvacc[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dkacc[kb][r] = 0.f; dvacc[kb][r] = 0.f; }

  // Row fragments of Q and dO: byte offset in a tile of the lane's 16 bytes; the spare lanes read the row's statistics
  const int prow = perm32(lo);
  const unsigned tf = (unsigned)(prow * SW_LD + (((2 * sh.s0 + hi) ^ sw_f(prow)) << 3)) * 2u;
  const unsigned sf = (unsigned)(uintptr_t)sSt[wave] + (unsigned)prow * 32u;

#pragma unroll
  for (int kb = 0; kb < KB; ++kb) asm volatile("" :: "v"(kreg[kb]), "v"(vreg[kb]));   // their wait here, not inside the loop

  int cslot = 0;
  while (rows1 >= 0) {
    ring_wait(false);   // all copies and loads: the stage is there
    asm volatile("" : "+v"(lv), "+v"(dv));   // the compiler's own wait for the two loads, before the next stage is requested
    const int rows = rows1;
    {
      // the statistics of row `lane`; a row past the segment's end gets probability 0
      const u32x2 lp = bf16_parts(lane < rows ? lv : IM_NEG_INF), dp = bf16_parts(dv);
      sSt[wave][2 * lane] = u32x4{lp[0], lp[1], 0u, 0u};
      sSt[wave][2 * lane + 1] = u32x4{dp[0], dp[1], 0u, 0u};
    }
    rows1 = issue();
    const bf16_t* sQ = sT + cslot * RING_STAGE;
    const bf16_t* sG = sQ + KT * SW_LD;
    const unsigned tile_at = (unsigned)(uintptr_t)sQ;
    cslot ^= 1;
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      if (qb == 1 && rows <= 32) break;
      const unsigned q_at = tile_at + qb * 32 * SW_LD * 2 + tf, s_at = sf + qb * 32 * 32;
      const bf16x8 aq = lds_b128(spare ? s_at : q_at), ag = lds_b128(spare ? s_at + 16 : q_at + KT * SW_LD * 2);
      bf16x8 as = aq, ad = ag;
      if (DH == 16) { as = lds_b128(s_at); ad = lds_b128(s_at + 16); }
      bf16x8 agt[2], aqt[2];
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        agt[half] = lds_frag_tr_sw(sG, qb * 32 + half * 16, sh.db0 * 32, lane);
        aqt[half] = lds_frag_tr_sw(sQ, qb * 32 + half * 16, sh.db0 * 32, lane);
      }
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        f32x16 sacc = f32x16{}, pacc = f32x16{};
        if (DH == 16) {
          sacc = mfma32(as, ones, sacc);
          pacc = mfma32(ad, ones, pacc);
        }
        sacc = mfma32(aq, kreg[kb], sacc);    // S  = Q K^T - lse
        pacc = mfma32(ag, vreg[kb], pacc);    // dP = dO V^T - delta
        float p[16], ds[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          p[r] = fast_exp2(sacc[r]);
          ds[r] = p[r] * pacc[r];
        }
        const bf16x8 pb[2] = {pack8(p), pack8(p + 8)}, dsb[2] = {pack8(ds), pack8(ds + 8)};
#pragma unroll
        for (int half = 0; half < 2; ++half) {   // dV^T += dO^T P ; dK^T += Q^T dS
          dvacc[kb] = mfma32(agt[half], pb[half], dvacc[kb]);
          dkacc[kb] = mfma32(aqt[half], dsb[half], dkacc[kb]);
        }
      }
    }
  }

  const int lane_e = lane_id();
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int row = k0 + kb * 32 + (lane_e & 31);
    if (row >= klen_seg) continue;
    // dK = scale dS^T Q, and the staged Q rows are scale log2(e) Q: the accumulator needs a factor ln 2.  A masked key's accumulators
    // are dropped, not multiplied by 0: no log-sum-exp bounds its scores, and 2^(S - lse) may have been infinite.
    constexpr float zk = 0.69314718055994530942f;
    const bool ok = kvalid[kb];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int dh0 = sh.db0 * 32 + 8 * i + 4 * (lane_e >> 5);  // column inside the 64-column group
      if (dh0 < sh.wo || dh0 >= sh.wo + DH) continue;
      bf16_t* o = dQKV + (krow0 + row) * ldg + d + sh.cg * 64 + dh0;
      const u32x2 pk = {pack_bf16(dkacc[kb][4 * i] * zk, dkacc[kb][4 * i + 1] * zk), pack_bf16(dkacc[kb][4 * i + 2] * zk, dkacc[kb][4 * i + 3] * zk)};
      const u32x2 pv = {pack_bf16(dvacc[kb][4 * i], dvacc[kb][4 * i + 1]), pack_bf16(dvacc[kb][4 * i + 2], dvacc[kb][4 * i + 3])};
      *(u32x2*)o = ok ? pk : u32x2{0u, 0u};
      *(u32x2*)(o + d) = ok ? pv : u32x2{0u, 0u};
    }
  }
}

// dK/dV: two key blocks per wave halve the streamed rows and the statistics per score and take head dimension 8 from 24.3 to 23.4 us
// at 32 x 50/500/375 rows, 8 heads, with three workgroups per CU; at 16 they spill, and one key block and four workgroups remain.
int mfma_sub_dq_tile_rows() { return 32; }
int mfma_sub_dkv_tile_rows(int dh) { return dh == 8 ? 64 : 32; }

// g's tiles have the heights above; live segments only (the caller zero-fills the others)
void launch_mfma_sub_bwd(const Geo& g, const bf16_t* qkv, long ld, const bf16_t* o, const bf16_t* d_o, long ldo, const float* lse2,
                         const int32_t* valid_len, const uint8_t* key_pad, float* delta, bf16_t* dqkv, long ldg, hipStream_t st) {
  const dim3 gq(g.q_tile_prefix[g.q_nord], g.H / 4, g.B), gk(g.k_tile_prefix[g.k_nord], g.H / 4, g.B);
  { ProfScope ps(PF_ATTN_DQ, st);
    if (g.dh == 8) hipLaunchKernelGGL((sub_dq_kernel<8>), gq, dim3(256), 0, st, g, qkv, ld, o, d_o, ldo, lse2, valid_len, key_pad, delta, dqkv, ldg);
    else hipLaunchKernelGGL((sub_dq_kernel<16>), gq, dim3(256), 0, st, g, qkv, ld, o, d_o, ldo, lse2, valid_len, key_pad, delta, dqkv, ldg); }
  { ProfScope ps(PF_ATTN_DKV, st);
    if (g.dh == 8) hipLaunchKernelGGL((sub_dkv_kernel<8, 2, 3>), gk, dim3(256), 0, st, g, qkv, ld, d_o, ldo, lse2, delta, valid_len, key_pad, dqkv, ldg);
    else hipLaunchKernelGGL((sub_dkv_kernel<16, 1, 4>), gk, dim3(256), 0, st, g, qkv, ld, d_o, ldo, lse2, delta, valid_len, key_pad, dqkv, ldg); }
}

}  // namespace imattn
