// Pieces shared by the bf16 matrix-core attention kernels (mfma_attn.hip, mfma_attn_sub.hip): the order of the workgroups, the
// segment table of a batch element, key masks, and the ring of LDS stages that the streamed tiles go through.
#pragma once
#include "mfma_common.hpp"

namespace imattn {

constexpr int KT = 64;  // keys (or query rows) per staged tile

// the lane's index from the hardware, where keeping it over a loop would cost a register that the loop does not have
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// Workgroup -> (tile, head, batch element).  As with xcd_block_index every XCD owns a contiguous range of (batch element,
// head, tile), but inside that range the workgroups are ordered by segment first (the tile order lists the segments by
// decreasing work per tile), then pair, then tile.  A workgroup of a long live range runs several times longer than one of
// a short range; started pair by pair, the long workgroups of the last pairs begin late and the XCD drains with most of its
// CUs idle.  Started first, they leave the short ones to fill the tail.
//
// cus != 0: the whole launch is resident at once and its tiles differ in length, so that nothing is left to fill a tail.  The
// dispatcher deals the workgroups of an XCD to its `cus` CUs in turn (measured: workgroups i, i + cus, i + 2 cus share
// a CU), and in plain order the CUs that get one workgroup more are those with the longest ones.  Here the CUs with one less
// take the longest, and each group of CUs is dealt to and fro.  3 x 333/1501/1290 rows, 4 heads of 64 (12 pairs), forward + dQ +
// dK/dV: in pair order 52 + 59 + 61 us, segment first and dealt like this 44 + 51 + 52.
__device__ __forceinline__ unsigned even_rank(unsigned pos, unsigned n, unsigned cus) {
  const unsigned full = n / cus, more = n % cus, round = pos / cus, cu = pos % cus;
  const bool a = cu >= more;
  const unsigned w = a ? cus - more : more, c = a ? cu - more : cu;
  return (a ? 0u : (cus - more) * full) + round * w + ((round & 1u) ? w - 1u - c : c);
}
__device__ __forceinline__ void xcd_tile_index(const int (&prefix)[IM_MAX_SEG + 1], int nord, bool tile_first, unsigned cus, int& tile, int& h,
                                               int& b) {
  const unsigned gx = gridDim.x, gy = gridDim.y, npair = gy * gridDim.z, total = gx * npair;
  const unsigned lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const unsigned xcd = lin & 7u, q = total >> 3, r = total & 7u, n = q + (xcd < r ? 1u : 0u);
  unsigned idx = lin >> 3, pair, t;
  if (cus) idx = even_rank(idx, n, cus);
  if ((npair & 7u) == 0u) {   // whole pairs
    const unsigned per = npair >> 3;  // pairs per XCD
    int first = 0, last = prefix[1];
#pragma unroll
    for (int k = 1; k < IM_MAX_SEG; ++k)
      if ((k < nord) & (idx >= per * (unsigned)prefix[k])) { first = prefix[k]; last = prefix[k + 1]; }
    const unsigned nt = (unsigned)(last - first), j = idx - per * (unsigned)first;
    if (tile_first) udivmod(j, per, t, pair);  // packed rows: the later tiles of most pairs find no rows
    else udivmod(j, nt, pair, t);
    pair += xcd * per;
    t += (unsigned)first;
  } else {
    // tiles a .. of pair p0, all tiles of the pairs between, tiles .. c - 1 of pair p1
    const unsigned start = xcd * q + (xcd < r ? xcd : r);
    unsigned p0, a, p1, c;
    udivmod(start, gx, p0, a);
    udivmod(start + n, gx, p1, c);
    const bool one = p0 == p1;
    const unsigned e0 = one ? c : gx, mid = one ? 0u : p1 - p0 - 1u, e1 = one ? 0u : c;
    pair = p0;
    t = a;
#pragma unroll 1
    for (int k = 0; k < nord; ++k) {
      const unsigned lo = (unsigned)prefix[k], nt = (unsigned)prefix[k + 1] - lo;
      const unsigned f0 = max(lo, a), f1 = min(lo + nt, e0), nf = f1 > f0 ? f1 - f0 : 0u;
      const unsigned l1 = min(lo + nt, e1), nl = l1 > lo ? l1 - lo : 0u;
      if (idx < nf) { t = f0 + idx; break; }
      idx -= nf;
      if (idx < mid * nt) {
        unsigned pl;
        udivmod(idx, nt, pl, t);
        pair = p0 + 1u + pl;
        t += lo;
        break;
      }
      idx -= mid * nt;
      if (idx < nl) { pair = p1; t = lo + idx; break; }
      idx -= nl;
    }
  }
  unsigned bb, hh;
  udivmod(pair, gy, bb, hh);
  tile = (int)t;
  h = (int)hh;
  b = (int)bb;
}

// Segment of a tile and the tile's position in it, with constant indexes: the tables come in one scalar load each, where a loop over
// them is a chain of loads.
// k: position of the segment in `order`.
__device__ __forceinline__ void tile_segment(const int (&order)[IM_MAX_SEG], const int (&prefix)[IM_MAX_SEG + 1], int nord,
                                             int tile, int& seg, int& in_seg, int& k) {
  int first = 0;
  k = 0;
  seg = order[0];
#pragma unroll
  for (int i = 1; i < IM_MAX_SEG; ++i)
    if ((i < nord) & (tile >= prefix[i])) { k = i; seg = order[i]; first = prefix[i]; }
  in_seg = tile - first;
}

// The segments of one batch element: first row inside the batch element (packed rows: in the tensor), rows, and the rows
// that are streamed (rows, or a key segment's valid length if that is less).  Read by lane s for segment s and kept in LDS,
// a copy per wave; reading valid_len segment by segment put a chain of loads in front of the first tile and one into the
// loop at every segment's end.  Padded rows need no memory for off and rows, so that a kernel requests the first tile of the
// first live segment before it waits for anything: the valid lengths, its own rows and that tile come in one round trip
// where they were two or three (workgroups of the small shapes live for 4 to 8 stages).  If the segment turns out to have no valid
// key its tile is not consumed.
struct SegTable { int off[IM_MAX_SEG], rows[IM_MAX_SEG], len[IM_MAX_SEG]; };
__device__ __forceinline__ int seg_get(const int (&v)[IM_MAX_SEG], int s) { return __builtin_amdgcn_readfirstlane(v[s]); }
// off and rows (len = rows) of the wave's table; qs_off, qs_rows: of segment qs; returns the segments of `live` that have rows
__device__ __forceinline__ unsigned seg_rows_table(SegTable& t, const Geo& g, int b, unsigned live, int lane, int qs, int& qs_off, int& qs_rows) {
  int off = 0, rows = 0;
  if (g.cu) {
    const int32_t* c = g.cu + b * g.n_seg + min(lane, g.n_seg - 1);
    off = c[0];
    rows = c[1] - c[0];
  } else {
#pragma unroll
    for (int s = 0; s < IM_MAX_SEG; ++s)
      if (lane == s) { off = g.seg_off[s]; rows = g.seg_len[s]; }
  }
  if (lane < IM_MAX_SEG) { t.off[lane] = off; t.rows[lane] = rows; t.len[lane] = rows; }
  qs_off = __builtin_amdgcn_readlane(off, qs);
  qs_rows = __builtin_amdgcn_readlane(rows, qs);
  return (unsigned)__ballot(lane < g.n_seg && ((live >> (lane & 31)) & 1u) && rows > 0);
}
// len from the lane's valid length (lane s: of segment s); returns the segments of `set` that have keys
__device__ __forceinline__ unsigned seg_lens_table(SegTable& t, int valid, unsigned set, int lane) {
  const int len = min(t.rows[lane & (IM_MAX_SEG - 1)], max(0, valid));
  if (lane < IM_MAX_SEG) t.len[lane] = len;
  return (unsigned)__ballot(lane < IM_MAX_SEG && ((set >> (lane & 31)) & 1u) && len > 0);
}

// Validity of the 64 keys of a staged tile as masks for packed bf16 pairs, 0xffff per valid key: keys from `keys` on and
// those with a key_pad byte (kp: one per dword, or NULL) are not valid.  A lane makes one pair's mask and reads the eight of
// its registers of a 32-key block back (block_masks): 10 vector instructions for a block where testing a bit per register
// took 32 (forward) and 48 (dQ).  The table is the wave's own, so no barrier stands between.
__device__ __forceinline__ void tile_masks(unsigned* pm, const unsigned* kp, int keys) {
  const int i = lane_id() & 31;
  u32x2 pad = {0u, 0u};
  if (kp) pad = *(const u32x2*)(kp + 2 * i);
  pm[i] = (2 * i < keys && pad[0] == 0u ? 0xffffu : 0u) | (2 * i + 1 < keys && pad[1] == 0u ? 0xffff0000u : 0u);
}
// register r of block kb on lane half hi is key kb*32 + 16*(r/8) + 8*hi + r%8
__device__ __forceinline__ void block_masks(const unsigned* pm, int kb, int hi, unsigned (&m)[8]) {
  const u32x4 a = *(const u32x4*)(pm + 16 * kb + 4 * hi), b = *(const u32x4*)(pm + 16 * kb + 8 + 4 * hi);
#pragma unroll
  for (int e = 0; e < 4; ++e) { m[e] = a[e]; m[4 + e] = b[e]; }
}

// x as a sum of three bf16 numbers, packed {p0 | p1 << 16, p2}.  -inf (the log-sum-exp of a row without a valid key) becomes
// bf16's lowest value, which has the same effect on a finite score and may meet a zero; NaN and +inf stay as they are.
__device__ __forceinline__ u32x2 bf16_parts(float x) {
  x = x == IM_NEG_INF ? -3.3895313892515355e38f : x;
  const unsigned a = pack_bf16(x, 0.f) & 0xffffu;
  const float ra = x - __uint_as_float(a << 16);
  const bool fin = (a & 0x7f80u) != 0x7f80u;
  const unsigned b = fin ? pack_bf16(ra, 0.f) & 0xffffu : 0u;
  const float rb = ra - __uint_as_float(b << 16);
  const unsigned c = fin ? pack_bf16(rb, 0.f) & 0xffffu : 0u;
  return u32x2{a | (b << 16), c};
}
constexpr unsigned ONES01 = 0x3f803f80u, ONES2 = 0x00003f80u;   // the three ones that the parts meet

// Streamed operands (K and V tiles in the forward and dQ kernels, Q and dO tiles in the dK/dV
// kernel) go from global memory straight into a ring of RING_NST LDS stages with asynchronous
// global->LDS copies (no staging registers, no LDS store instructions): stage t+2 is requested
// while stage t is consumed, with one workgroup barrier per stage.  Each lane fetches the 16-byte
// chunk that belongs at ITS position of the swizzled tile (see sw_f), so the copy produces the
// conflict-free layout directly.  The tiles of all live segments form one sequence, so the ring
// does not drain between segments.
constexpr int RING_NST = 3;
constexpr int RING_STAGE = 2 * KT * SW_LD;  // bf16 elements per stage: two 64 x 64 tiles

// Cursor over the 64-row tiles of the live segments, ascending segment order; segments of length <= 0 are not in `rest`.
// left: rows from the next tile's first one to the end of its segment; <= 0 <=> exhausted.  All scalar.
struct TileCursor {
  unsigned rest;  // live segments not started yet
  int seg, left;
};
__device__ __forceinline__ bool cursor_next_seg(TileCursor& c, const SegTable& t) {
  if (!c.rest) { c.left = 0; return false; }
  c.seg = __builtin_ctz(c.rest);
  c.rest &= c.rest - 1;
  c.left = seg_get(t.len, c.seg);
  return true;
}

// Per-lane constants of the ring copies: the two tile rows (32 apart) whose chunk positions this lane fills in each streamed matrix,
// and the byte offset of the logical chunk inside a row of head h.  Workgroups have four waves.
struct RingLane {
  int trow0, trow1;
  unsigned col0, col1;
};
__device__ __forceinline__ RingLane ring_lane(int wave, int lane, int h) {
  RingLane r;
  r.trow0 = wave * 8 + (lane >> 3);
  r.trow1 = r.trow0 + 32;
  r.col0 = (unsigned)(h * 64 + (((lane & 7) ^ sw_f(r.trow0)) << 3)) * 2u;
  r.col1 = (unsigned)(h * 64 + (((lane & 7) ^ sw_f(r.trow1)) << 3)) * 2u;
  return r;
}
// Scalar state of the ring copies inside the current segment: byte pointers to the first row of the
// next tile of the two streamed matrices, and the rows the segment has from there on (> 0).  Kept in
// scalar registers and advanced by one tile per request, so a request costs a handful of scalar adds.
struct RingFeed {
  const char* a;
  const char* b;
  int rows;
};
// per-lane byte offsets of this lane's four chunks in a tile that lies wholly inside the segment
struct RingLaneOff { unsigned a0, b0, a1, b1; };
__device__ __forceinline__ RingLaneOff ring_lane_off(const RingLane& rl, unsigned pitch_a, unsigned pitch_b) {
  return {__umul24((unsigned)rl.trow0, pitch_a) + rl.col0, __umul24((unsigned)rl.trow0, pitch_b) + rl.col0,
          __umul24((unsigned)rl.trow1, pitch_a) + rl.col1, __umul24((unsigned)rl.trow1, pitch_b) + rl.col1};
}
// Request the next 64-row tile pair of the segment into LDS stage `stage` (4 copies per wave; row pitches in bytes) and advance the
// feed.  Only the last tile of a segment can be ragged; its missing rows repeat the segment's last row.
__device__ __forceinline__ void ring_feed_issue(const RingLane& rl, const RingLaneOff& lo, RingFeed& f, unsigned pitch_a,
                                                unsigned pitch_b, int wave, bf16_t* stage) {
  if (f.rows >= KT) {
    dma16_off(f.a, lo.a0, stage + wave * 512);
    dma16_off(f.b, lo.b0, stage + KT * SW_LD + wave * 512);
    dma16_off(f.a, lo.a1, stage + (4 + wave) * 512);
    dma16_off(f.b, lo.b1, stage + KT * SW_LD + (4 + wave) * 512);
  } else {
    const unsigned r0c = (unsigned)min(rl.trow0, f.rows - 1), r1c = (unsigned)min(rl.trow1, f.rows - 1);
    dma16_off(f.a, __umul24(r0c, pitch_a) + rl.col0, stage + wave * 512);
    dma16_off(f.b, __umul24(r0c, pitch_b) + rl.col0, stage + KT * SW_LD + wave * 512);
    dma16_off(f.a, __umul24(r1c, pitch_a) + rl.col1, stage + (4 + wave) * 512);
    dma16_off(f.b, __umul24(r1c, pitch_b) + rl.col1, stage + KT * SW_LD + (4 + wave) * 512);
  }
  f.a += (size_t)KT * pitch_a;
  f.b += (size_t)KT * pitch_b;
  f.rows -= KT;
}
// wait for the oldest stage requested (later: one more stage has been requested after it; 4 copies per wave and stage), then meet
// the other waves: the wanted stage is visible to all, and every wave has finished reading the stage consumed before it.
// `extra`: this wave issues one more copy per stage, ahead of the others.
__device__ __forceinline__ void ring_wait(bool later, bool extra = false) {
  if (later) {
    if (extra) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __builtin_amdgcn_s_barrier();
}

// The K and V tiles of the live segments that a workgroup's query rows read, through a ring of NST stages (forward and dQ).
template <int NST>
struct KvStream {
  const SegTable& sg;
  bf16_t* sT;               // the stages: K tile, V tile
  unsigned* sKP;            // per stage: key_pad bytes of the 64 keys, one per dword
  const bf16_t* k;          // K columns of the batch element's first row; V is d columns further on
  const uint8_t* key_pad;   // of that row, or NULL
  long ld, d;
  int wave;
  RingLane rl;
  RingLaneOff rlo;
  bool kp_copy;             // this wave fetches a stage's key_pad bytes
  TileCursor at = {0u, 0, 0};
  int slot = 0;
  RingFeed feed = {nullptr, nullptr, 0};
  const uint8_t* feed_kp = nullptr;

  __device__ __forceinline__ KvStream(const SegTable& t, bf16_t* st, unsigned* skp, const bf16_t* kcols, const uint8_t* kpad, long pitch,
                                      long width, int w, int lane, int group)
      : sg(t), sT(st), sKP(skp), k(kcols), key_pad(kpad), ld(pitch), d(width), wave(w), rl(ring_lane(w, lane, group)),
        rlo(ring_lane_off(rl, (unsigned)pitch * 2u, (unsigned)pitch * 2u)), kp_copy(w == 0 && kpad != nullptr) {}
  // K and V rows of a segment; rows past the valid length but inside the segment are fetched and masked
  __device__ __forceinline__ void seg_begin(int seg) {
    const int off = seg_get(sg.off, seg);
    feed.a = (const char*)(k + off * ld);
    feed.b = feed.a + (size_t)d * 2;
    feed.rows = seg_get(sg.rows, seg);
    if (key_pad) feed_kp = key_pad + off;
  }
  __device__ __forceinline__ void copy() {   // requests the feed's next tile
    // The key_pad bytes travel with the stage: an ordinary load inside the loop would wait for every copy before it.
    if (kp_copy) dma1_off(feed_kp, (unsigned)min(lane_id(), feed.rows - 1), sKP + slot * KT);
    feed_kp += KT;
    ring_feed_issue(rl, rlo, feed, (unsigned)ld * 2u, (unsigned)ld * 2u, wave, sT + slot * RING_STAGE);
    slot = (slot + 1 == NST) ? 0 : slot + 1;
  }
  __device__ __forceinline__ void next_seg() {
    if (cursor_next_seg(at, sg)) seg_begin(at.seg);
  }
  // requests the next stage; returns its number of valid keys (key_pad aside), -1 if there is none
  __device__ __forceinline__ int issue() {
    if (at.left <= 0) return -1;
    const int keys = at.left;
    copy();
    at.left -= KT;
    if (at.left <= 0) next_seg();
    return keys;
  }
  // The first tile of segment seg, ahead of everything; begin(): its valid keys, once the lengths are in the table, and the cursor
  // behind it (set: the segments with valid keys).
  __device__ __forceinline__ void first(int seg) {
    seg_begin(seg);
    copy();
  }
  __device__ __forceinline__ int begin(int seg, unsigned set) {
    at.rest = set & ~(1u << seg);
    const int keys = seg_get(sg.len, seg);
    at.left = keys - KT;
    if (at.left <= 0) next_seg();
    return keys;
  }
};

}  // namespace imattn
