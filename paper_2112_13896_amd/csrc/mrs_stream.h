// One fp32 layer in one kernel, as mrs_blocks.h, for tables too large to stay in
// LDS and rows of up to 256 channels in power-of-two sets: Multiply, Route and
// Sum (Section 3.2 steps 3-5) with the packed table streamed through LDS, k-WTA
// (Section 3.3.3), lists or a dense output.  The sums are formed in the same
// order as there (bias first, taps in order, a list in ascending channel order,
// one fused multiply-add a product), so both give the same bits.
//
// What bounds such a layer is the instructions of one wavefront: a pixel's sums
// are a serial chain, and at the sizes these layers have (a few dozen pixels a
// compute unit) there are few wavefronts to hide it behind.  Hence:
//  * one workgroup per compute unit, of as many wavefronts as share the pixels
//    evenly over all compute units (at most sixteen), 4 to 16 pixels a wavefront,
//    the U = 4, 8 or 16 lanes of a pixel holding GB sets (KP = GB n channels) each;
//  * the table blocks are copied to LDS as they are, by loads that write LDS
//    directly (no registers, no instructions per entry), into the other of two
//    buffers while one is used: one barrier a block.  A Kernel ID becomes an
//    accumulator address with the shift-and-add that adds the lane's column;
//  * the first 32 entries of the next tap's list are loaded a tap ahead, so no
//    load of a list waits behind the table's;
//  * the k-WTA searches bit planes (as many keys a word as the lane has
//    channels) on the lane's own columns.
// Measured against the table-block kernel (256 threads, two sets a lane, table
// blocks staged through registers into one buffer between two barriers; 1.5
// workgroups of four wavefronts a compute unit): 14x14x256 3x3, 64 images, 26 of
// 256 in and out 41.7 -> 36.2 us; 1x1 1024 -> 256, 102 in 33.0 -> 27.1 us; 56x56x128
// 3x3/2, 13 images, 16 of 128 28.4 -> 20.8 us.  The 3x3 layer's 9.8 M vector
// instructions are four cycles each on the 968 SIMDs it runs on, 47 % of its time;
// reading a chunk's table entries a chunk ahead, or four entries' accumulators
// together, changed nothing (36.0, 37.1 us).
//
// The sums alone of a 1x1 layer of more than 256 channels whose table fits a block in
// slices of 256 channels take the same kernel (WIDE), a slice a workgroup (grid y).  The
// sums are added as the table-slice or fused kernel, which such a layer runs on
// otherwise, adds them: in S parts, part s taking the list's chunks of four entries
// s, s + S, ... from zero, the parts added in order (or in pairs), then the bias.  A
// part is one group of U lanes on a list of its own - the entry at place 4 k + e of
// part s is the pixel's entry 4 (s + S k) + e - so both kernels give the same bits.
// Against those kernels, 32 images: 28x28x128 -> 512, 12 in, 138.4 -> 52.4 us (four
// parts); 14x14x256 -> 1024, 25 in, 38.4 -> 20.9 (two); 14x14x64 -> 512, 25 in, 44.1 ->
// 18.2 (four).  In list order the three took 25.4, 18.9 and 10.7: a part is a few
// entries, and each group of lanes pays for its pixel's start and end.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastdiv.h"
#include "kwta_kernels.h"
#include "mrs_blocks.h"
#include "mrs_kernels.h"
#include "wave_ops.h"

namespace cs {

constexpr int STREAM_BD = 1024;          // threads per workgroup at most; accumulator row stride
constexpr int STREAM_SHIFT = 12;         // log2 bytes of an accumulator row
constexpr int STREAM_BLOCK = 32 * 1024;  // bytes of a table block at most
constexpr int STREAM_PIECE = 1024;       // bytes a wavefront copies at once
constexpr int STREAM_PRE = 2;            // groups of sixteen list entries loaded ahead
static_assert(STREAM_BD * 4 == 1 << STREAM_SHIFT, "an accumulator row is one float a thread");

struct StreamArgs {
  int log2U;          // lanes per pixel
  int P;              // pixels per tile = threads / U
  int items;          // output pixels
  int RB;             // table rows per block
  int nblocks;        // ceil(R / RB)
  int tpb;            // taps per block, or 0: a block is a channel range of one tap
  int cblocks;        // channel blocks per tap (C / RB) when tpb == 0
  int log2n, log2G;   // kernels per set; sets of a slice
  int k;              // k-WTA winners per unit; -1: sums only
  int write_sums;
  int log2Us;         // lanes per k-WTA unit
  uint32_t off_t0, off_t1;   // LDS byte offsets of the table buffers
  int row_stride;     // bytes of a table row in memory, all G sets
  int log2S;          // WIDE: parts of a pixel's list, at most 4; P = threads / (U S)
  int pairs;          // WIDE: the parts are added in pairs, not in order
  FastDiv fd_wo, fd_ho, fd_kw;
};

// Sum over the aligned groups of 2^LU lanes: LU DPP adds.
template <int LU>
__device__ __forceinline__ uint32_t group_sum_c(uint32_t c) {
  if (LU >= 1) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xF, 0xF, false);
  if (LU >= 2) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x4E, 0xF, 0xF, false);
  if (LU >= 3) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x141, 0xF, 0xF, false);
  if (LU >= 4) c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x140, 0xF, 0xF, false);
  return c;
}

// Transpose, in place, of the 32 / N blocks of N x N bits that N words hold side
// by side (N = 4, 8 or 16): afterwards bit N q + j of a[i] is bit N q + i of the
// original a[j] (log2 N stages of block swaps, each row pair by two shifts and
// two bit-field selects).
template <int N>
__device__ __forceinline__ void bit_transpose_n(uint32_t (&a)[N]) {
  constexpr uint32_t M[4] = {0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const int w = 8 >> st;
    if (w >= N) continue;
    const uint32_t m = M[st];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (j & w) continue;
      const uint32_t x = a[j], y = a[j + w];
      a[j] = (x & m) | ((y << w) & ~m);
      a[j + w] = ((x >> w) & m) | (y & ~m);
    }
  }
}

// The search of stream_kwta: the k-th largest key of every unit, bit by bit
// on the lane's bit planes sl (plane of bit N q + i: bits N q .. N q + N - 1 of
// sl[i]).  A step's count is the keys already above the prefix plus one bit
// count of the plane's AND with the keys still matching it, summed over the
// unit; each step is branch-free: a unit still searching takes the bit when at
// least k keys are at or above the candidate, else the matching keys with the
// bit set are above the prefix from now on; a unit whose keys at or above the
// prefix are exactly k is done.  Leaves the winners as masks: gtm, the keys
// above the prefix, and eqm, the keys that match it.  LU: log2 of the lanes
// per unit, or -1 (taken from mk).
template <int N, int LU>
__device__ __forceinline__ void stream_search(const uint32_t (&sl)[N], const uint32_t (&mk)[4], int k,
                                           int c_unit, bool done, uint32_t& gtm, uint32_t& eqm) {
  uint32_t match = N == 32 ? 0xFFFFFFFFu : (1u << (N & 31)) - 1u, above = 0u, above_m = 0u;
  int cntp = c_unit;
  for (int q = 32 / N - 1; q >= 0; --q) {                // uniform
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
      if (__ballot(!done) == 0ull) break;                // every unit of the wavefront found
      const uint32_t plane = __builtin_amdgcn_ubfe(sl[i], (uint32_t)(N * q), (uint32_t)N);
      const uint32_t hit = match & plane;
      const uint32_t nh = (uint32_t)__popc(hit);
      const uint32_t c = LU >= 0 ? group_sum_c<LU < 0 ? 0 : LU>(above + nh)
                                 : group_sum_nb(above + nh, mk);
      const bool take = !done && (int)c >= k;
      const bool drop = !done && (int)c < k;
      cntp = take ? (int)c : cntp;
      match = take ? hit : (drop ? (match & ~plane) : match);
      above = drop ? above + nh : above;
      above_m = drop ? (above_m | hit) : above_m;
      done = done || cntp == k;
    }
  }
  gtm = above_m;
  eqm = match;
}

// k-WTA over the U lanes of each pixel, the lanes that computed its sums: lane
// u holds channels u*KP .. u*KP+KP-1 (KP = GB * n) in its own accumulator
// column, bias included, so no other lane's data is read and no barrier is
// needed.  The row is split into units of Us = 1 << log2Us lanes (KP * Us
// channels; Us = U: the whole row), each keeping its own k winners (the k-WTA
// in units of Section 5's channel partitioning).  The k-th largest key of a
// unit is found on bit planes (stream_search), which leaves the winners as
// masks; ties go to the lower index; the winners of the whole row are written
// as one list (non-zero values, ascending index) or densely.
template <typename TO, int KP, int BD>
__device__ __forceinline__ void stream_kwta(const float* acc, int log2U, int log2Us,
                                             int64_t row, bool live, int c_out, int k,
                                             int write_sums, float* __restrict__ y,
                                             TO* __restrict__ out, const ListOut& lo) {
  const int tid = threadIdx.x;
  const int p = tid & ((1 << log2U) - 1);                // lane position in the group
  const int ps = p & ((1 << log2Us) - 1);                // lane position in its unit
  const int c_unit = KP << log2Us;                       // channels per k-WTA unit
  const int o0 = p * KP;                                 // first channel of the lane
  constexpr uint32_t kAll = (1u << KP) - 1u;
  if (write_sums && live) {
    float* yr = y + row * c_out + o0;                    // 16-byte aligned (host)
#pragma unroll
    for (int j = 0; j < KP; j += 4)
      *reinterpret_cast<float4*>(yr + j) =
          make_float4(acc[j * BD + tid], acc[(j + 1) * BD + tid], acc[(j + 2) * BD + tid],
                      acc[(j + 3) * BD + tid]);
  }
  if (k < 0) return;
  uint32_t mk[4];
  group_masks(log2Us, mk);
  uint32_t gtm = 0u, eqm = 0u;
  if (k > 0 && k < c_unit) {
    uint32_t sl[KP];
#pragma unroll
    for (int j = 0; j < KP; ++j) sl[j] = order_key(acc[j * BD + tid]);
    bit_transpose_n<KP>(sl);
    // (k as a vector value: the scalar one is a spilled argument, reloaded
    // every step)
    int kv = k;
    asm volatile("" : "+v"(kv));
    if (log2Us == 4) stream_search<KP, 4>(sl, mk, kv, c_unit, !live, gtm, eqm);
    else if (log2Us == 3) stream_search<KP, 3>(sl, mk, kv, c_unit, !live, gtm, eqm);
    else if (log2Us == 2) stream_search<KP, 2>(sl, mk, kv, c_unit, !live, gtm, eqm);
    else stream_search<KP, -1>(sl, mk, kv, c_unit, !live, gtm, eqm);
  }
  CS_STAMP(19);
  // need = k minus the unit's keys above; the first `need` matching keys of
  // the unit in index order win (every lane takes part in the sums)
  const int nabove = (int)group_sum_nb((uint32_t)__popc(gtm), mk);
  const int eq_l = __popc(eqm);
  const int tie0 = group_incl_sum(eq_l, log2Us, ps) - eq_l;
  int m = k - nabove - tie0;
  m = m < 0 ? 0 : (m > eq_l ? eq_l : m);
  uint32_t tm = m >= eq_l ? eqm : 0u;
  if (m > 0 && m < eq_l) {                              // a tie split at this lane (rare)
    for (uint32_t e2 = eqm; m > 0; --m) {
      const uint32_t lb = e2 & (0u - e2);
      tm |= lb;
      e2 ^= lb;
    }
  }
  const uint32_t winm = (!live || k == 0) ? 0u : (k >= c_unit ? kAll : (gtm | tm));
  uint32_t putm = winm;                                 // bit j: channel o0 + j is listed
  if (lo.idx) {
    // winners whose value is exactly zero are left out of the list
    for (uint32_t w = winm; w != 0u; w &= w - 1u) {
      const int j = __builtin_ctz(w);
      if (acc[j * BD + tid] == 0.f) putm &= ~(1u << j);
    }
  }
  CS_STAMP(20);
  if (lo.idx) {
    const int wcount = __popc(putm);
    const int incl = group_incl_sum(wcount, log2U, p);
    int pos = incl - wcount;
    if (live) {
      uint16_t* oi = lo.idx + row * lo.cap;
      TO* ov = static_cast<TO*>(lo.val) + row * lo.cap;
      // one pass per winner of the lane (a few), the value read back from
      // the lane's own column, instead of KP predicated slots
      for (uint32_t w = putm; w != 0u; w &= w - 1u) {
        const int j = __builtin_ctz(w);
        oi[pos] = (uint16_t)(o0 + j);
        ov[pos] = (TO)acc[j * BD + tid];
        ++pos;
      }
      if (p == (1 << log2U) - 1) lo.cnt[row] = incl;
    }
  } else if (live) {
    TO* orow = out + row * c_out + o0;
#pragma unroll
    for (int j = 0; j < KP; j += 4) {
      float w4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w4[e] = (winm >> (j + e)) & 1u ? acc[(j + e) * BD + tid] : 0.f;
      *reinterpret_cast<float4*>(orow + j) = make_float4(w4[0], w4[1], w4[2], w4[3]);
    }
  }
}

// Where a lane's window starts, worked out once per tile: a tap is then one
// uniform addition and two unsigned comparisons away.
struct TapPlace {
  int hy, wx;              // input row and column of tap (0, 0); hy a large negative: no pixel
  uint32_t q;              // its list row (modulo 2^32)
  uint32_t off;            // its list row's first entry, q * cap (modulo 2^32)
};

// The part of a pixel's list that a group of lanes takes: all of it unless WIDE.
template <bool WIDE>
struct ListPart {
  int log2S;               // parts
  int s4;                  // 4 * this part
  // place in the list of the part's chunk at pos (a multiple of four)
  __device__ __forceinline__ int at(int pos) const { return WIDE ? (pos << log2S) + s4 : pos; }
  // entries of this part among the first m of the list
  __device__ __forceinline__ int count(int m) const {
    if (!WIDE) return m;
    const int rounds = m >> (log2S + 2), rest = m - (rounds << (log2S + 2));
    return 4 * rounds + max(0, min(rest - s4, 4));
  }
};

// A tap's list, its first STREAM_PRE groups of sixteen entries already loaded:
// lane p of a quad holds entries g0 + 16 i + 4p .. + 3 in ch[i].
struct StreamPre {
  int off;                 // list row offset, or -1: the tap is outside the image
  int cnt;
  BChunk ch[STREAM_PRE];
};

template <bool WIDE>
__device__ __forceinline__ void stream_load(BChunk& c, const uint16_t* __restrict__ lidx,
                                            const float* __restrict__ lval, uint32_t base, int pos,
                                            int cap, ListPart<WIDE> part) {
  const size_t e = (size_t)(base + (uint32_t)min(part.at(pos), cap - 4));    // inside the row
  c.idx = *reinterpret_cast<const uint2*>(lidx + e);
  c.val = *reinterpret_cast<const float4*>(lval + e);
}

template <bool WIDE>
__device__ __forceinline__ void stream_prefetch(StreamPre& tp, const uint16_t* __restrict__ lidx,
                                                const float* __restrict__ lval,
                                                const int32_t* __restrict__ lcnt,
                                                const ConvGeom& geo, const TapPlace& pl, int t,
                                                int j0, const FastDiv& fd_kw, ListPart<WIDE> part) {
  const int ky = (int)fdiv((uint32_t)t, fd_kw), kx = t - ky * geo.KW;         // uniform
  const bool in = t < geo.KH * geo.KW;
  const uint32_t dq = in ? (uint32_t)(ky * geo.W + kx) : 0u;
  const bool ok = in && (uint32_t)(pl.hy + ky) < (uint32_t)geo.H &&
                  (uint32_t)(pl.wx + kx) < (uint32_t)geo.W;
  const uint32_t q = ok ? pl.q + dq : 0u;
  const uint32_t base = ok ? pl.off + dq * (uint32_t)geo.cap : 0u;
  tp.off = ok ? (int)base : -1;
  tp.cnt = lcnt[(size_t)q];
  const int p = (j0 & ~3) + 4 * (int)(threadIdx.x & 3);
#pragma unroll
  for (int i = 0; i < STREAM_PRE; ++i)
    if (16 * i < geo.cap)                                                     // uniform
      stream_load(tp.ch[i], lidx, lval, base, p + 16 * i, geo.cap, part);
}

// Route + Sum of four entries into the lane's GB accumulators, in pairs as
// blk_chunk: both reads, then the writes in entry order, the second entry of a pair
// adding onto the first's new value when their Kernel IDs are equal; an ID
// becomes the address of its row of the lane's column.
template <int GB>
__device__ __forceinline__ void stream_route(const float (&x)[4], const uint2 (&te)[4][GB],
                                             const unsigned char* smem,
                                             const uint32_t (&col)[GB]) {
  unsigned char* lds = const_cast<unsigned char*>(smem);
#pragma unroll
  for (int pr = 0; pr < 4; pr += 2) {
    float* p0[GB];
    float* p1[GB];
    float a0[GB], a1[GB];
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      p0[j] = reinterpret_cast<float*>(lds + ((te[pr][j].y << STREAM_SHIFT) + col[j]));
      p1[j] = reinterpret_cast<float*>(lds + ((te[pr + 1][j].y << STREAM_SHIFT) + col[j]));
      a0[j] = *p0[j];
      a1[j] = *p1[j];
    }
#pragma unroll
    for (int j = 0; j < GB; ++j) {
      const float v0 = __builtin_fmaf(x[pr], __uint_as_float(te[pr][j].x), a0[j]);
      const float b1 = te[pr + 1][j].y == te[pr][j].y ? v0 : a1[j];
      const float v1 = __builtin_fmaf(x[pr + 1], __uint_as_float(te[pr + 1][j].x), b1);
      *p0[j] = v0;
      *p1[j] = v1;
    }
  }
}

// The entries of one tap's list from position j0 on (and, in channel mode,
// below channel c_hi) against the staged block.  A lane turns the four entries it
// loaded into what the quad needs - the LDS address of each one's table row and
// its value, a dead entry (past the list, before j0 or from channel c_hi on)
// reading the block's first row with value 0 - and the quad then takes the
// sixteen entries chunk by chunk: masking, index unpacking and the row address
// are so done once per entry and quad, and the broadcasts fold into the
// instruction that uses them (a DPP operand of the address add).  Returns the
// list position where the quad stopped.
template <int GB, bool CH, bool WIDE>
__device__ __forceinline__ int stream_tap(const StreamPre& tp, const uint16_t* __restrict__ lidx,
                                          const float* __restrict__ lval, int cap, int j0, int c_hi,
                                          int row_add, const unsigned char* smem, uint32_t tab,
                                          int log2row, uint32_t lane_tab,
                                          const uint32_t (&col)[GB], ListPart<WIDE> part) {
  if (tp.off < 0) return j0;
  const int m = part.count(min(tp.cnt, cap));
  const uint32_t row0 = tab + ((uint32_t)row_add << log2row);
  int end = m;
  // sixteen entries from list position g0 on; true: the list goes on after them
  auto group = [&](const BChunk& mine, int g0) {
    const int p4 = g0 + 4 * (int)(threadIdx.x & 3);
    uint32_t rb[4];
    float xv[4];
    int nl = 0;                                          // this lane's live entries
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t i = (uint32_t)bchunk_idx(mine.idx, e);
      bool ok = p4 + e < m;
      if constexpr (CH) ok = ok && p4 + e >= j0 && (int)i < c_hi;   // the list ascends
      rb[e] = ok ? (i << log2row) + row0 : tab;
      xv[e] = ok ? bchunk_val(mine.val, e) : 0.f;
      nl += ok ? 1 : 0;
    }
    if constexpr (CH) {
      uint32_t n4 = (uint32_t)nl;
      n4 += quad_xor1(n4);
      n4 += quad_xor2(n4);
      end = (j0 > g0 ? j0 : g0) + (int)n4;
    }
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
      if (g0 + 4 * s2 < end && (!CH || g0 + 4 * s2 + 4 > j0)) {      // the same in the quad
        CS_COUNT_PRODUCTS_ADD((int)quad_bcast((uint32_t)nl, s2) * GB);
        uint2 te[4][GB];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned char* q = smem + (quad_bcast(rb[e], s2) + lane_tab);
          if constexpr (GB == 1) {
            te[e][0] = *reinterpret_cast<const uint2*>(q);
          } else {
            const uint4 w = *reinterpret_cast<const uint4*>(q);
            te[e][0] = make_uint2(w.x, w.y);
            te[e][1] = make_uint2(w.z, w.w);
          }
        }
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(quad_bcast(__float_as_uint(xv[e]), s2));
        stream_route<GB>(x, te, smem, col);
      }
    }
    return end >= g0 + 16 && g0 + 16 < m;
  };
  int g0 = j0 & ~3;
#pragma unroll
  for (int i = 0; i < STREAM_PRE; ++i) {
    if (!group(tp.ch[i], g0)) return CH ? end : m;
    g0 += 16;
  }
  while (true) {
    BChunk c;
    stream_load(c, lidx, lval, (uint32_t)tp.off, g0 + 4 * (int)(threadIdx.x & 3), cap, part);
    if (!group(c, g0)) return CH ? end : m;
    g0 += 16;
  }
}

// The sums of a pixel's 256 channels of a slice from its S parts' accumulators, and the
// bias: of the sixteen channels of the S lanes' columns each lane finishes 16 / S, from
// s * 16 / S on (s: its part; bv: their bias, yr: their place).  The groups of lanes read
// different parts at a time - the same part of different rows would be one bank - and
// turn the values back into part order in registers.
template <int KP>
__device__ __forceinline__ void stream_sum_parts(const float* acc, int log2S, int pairs, int s,
                                                 const float (&bv)[KP], float* __restrict__ yr) {
  static_assert(KP == 16, "sixteen lanes of sixteen channels a pixel");
  const int tid = threadIdx.x, per = 16 >> log2S;
  const float* col = acc + (tid & ~((16 << log2S) - 1)) + (tid & 15);   // part 0's column
#pragma unroll
  for (int j0 = 0; j0 < KP; j0 += 4) {
    if (j0 >= per) break;                                // uniform
    float v[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const float* cj = col + (s * per + j0 + jj) * STREAM_BD;
      float a = 0.f;
      if (log2S == 0) {
        a += cj[0];
      } else if (log2S == 1) {
        const float r0 = cj[16 * s], r1 = cj[16 * (1 - s)];
        a = (a + (s ? r1 : r0)) + (s ? r0 : r1);
      } else {
        float r[4], q[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) r[t] = cj[16 * ((t + s) & 3)];
#pragma unroll
        for (int t = 0; t < 4; ++t) q[t] = (s & 1) ? r[(t + 3) & 3] : r[t];
#pragma unroll
        for (int t = 0; t < 4; ++t) r[t] = (s & 2) ? q[(t + 2) & 3] : q[t];
        a = pairs ? (r[0] + r[1]) + (r[2] + r[3]) : (((a + r[0]) + r[1]) + r[2]) + r[3];
      }
      v[jj] = a + bv[j0 + jj];
    }
    *reinterpret_cast<float4*>(yr + j0) = make_float4(v[0], v[1], v[2], v[3]);
  }
}

template <typename TO, int GB, bool CH, int KP, bool WIDE>
__global__ __launch_bounds__(STREAM_BD, 4) void mrs_stream_f32(
    const uint16_t* __restrict__ lidx, const float* __restrict__ lval,
    const int32_t* __restrict__ lcnt, const uint2* __restrict__ aug,
    const float* __restrict__ bias, float* __restrict__ y, TO* __restrict__ out, ListOut lo,
    ConvGeom geo, StreamArgs sa) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), nwv = (int)blockDim.x >> 6;
  const int C = geo.C, T_ = geo.KH * geo.KW, R = T_ * C;
  const int u = tid & ((1 << sa.log2U) - 1);             // the lane's sets u*GB .. u*GB+GB-1
  // sums of rows of more than 256 channels: a slice of the sets a workgroup, and a
  // part of its pixel's list a group of U lanes
  const int set0 = WIDE ? (int)blockIdx.y << sa.log2G : 0, ch0 = set0 << sa.log2n;
  const int log2S = WIDE ? sa.log2S : 0;
  const ListPart<WIDE> part{log2S, WIDE ? 4 * ((tid >> sa.log2U) & ((1 << log2S) - 1)) : 0};
  float* acc = reinterpret_cast<float*>(smem);           // [KP][STREAM_BD]
  const int log2row = sa.log2G + 3;                      // bytes of a table row
  const uint32_t lane_tab = (uint32_t)(u * GB * 8);
  uint32_t col[GB];
#pragma unroll
  for (int j = 0; j < GB; ++j) col[j] = (uint32_t)tid * 4u + ((uint32_t)(j << sa.log2n) << STREAM_SHIFT);

  // rows [r0, r0 + RB) of the slice's table (the last block's end) to LDS offset
  // off, STREAM_PIECE bytes a wavefront and instruction; a lane past the table
  // reads its last row (the buffers are whole pieces)
  auto copy_block = [&](int r0, uint32_t off) {
    const int rows = R - r0 < sa.RB ? R - r0 : sa.RB;
    const int bytes = rows << log2row;
    for (int p = wv; p * STREAM_PIECE < bytes; p += nwv) {           // uniform
      const int at = p * STREAM_PIECE + 16 * (tid & 63);
      const int row = min(at >> log2row, rows - 1);
      const int64_t g = (int64_t)(r0 + row) * sa.row_stride + set0 * 8 + (at & ((1 << log2row) - 1));
      __builtin_amdgcn_global_load_lds(
          reinterpret_cast<const __attribute__((address_space(1))) void*>(
              reinterpret_cast<uintptr_t>(aug) + (uintptr_t)g),
          (__attribute__((address_space(3))) void*)(smem + off + p * STREAM_PIECE),
          16, 0, 0);
    }
  };
  // every wavefront's copies are in LDS, and no one reads the buffer before
  auto block_done = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  CS_STAMP_COUNT(31);
  CS_STAMP(16);
  const int item0 = (int)blockIdx.x * sa.P;
  const int item = item0 + (tid >> (sa.log2U + log2S));
  const bool live = item < sa.items;
  int bb = 0, ho = 0, wo = 0;
  if (live) {
    const uint32_t t1 = fdiv((uint32_t)item, sa.fd_wo);
    wo = item - (int)(t1 * sa.fd_wo.d);
    const uint32_t t2 = fdiv(t1, sa.fd_ho);
    ho = (int)(t1 - t2 * sa.fd_ho.d);
    bb = (int)t2;
  }
  TapPlace place;
  place.hy = live ? ho * geo.S - geo.P : -(1 << 30);
  place.wx = wo * geo.S - geo.P;
  place.q = (uint32_t)((bb * geo.H + ho * geo.S - geo.P) * geo.W + place.wx);
  place.off = place.q * (uint32_t)geo.cap;
  // accumulators start at the bias of their channels (its loads together, then
  // the first lists' and the table's)
  float bv[KP];
#pragma unroll
  for (int j = 0; j < KP; ++j) bv[j] = 0.f;
  // (WIDE: of the channels it finishes, added last)
  const int per = KP >> log2S, bias0 = ch0 + u * KP + (part.s4 >> 2) * per;
  if (bias != nullptr) {                                 // uniform
#pragma unroll
    for (int j = 0; j < KP; ++j)
      if (!WIDE || j < per) bv[j] = bias[bias0 + j];
  }
  StreamPre q;
  stream_prefetch(q, lidx, lval, lcnt, geo, place, 0, 0, sa.fd_kw, part);
  copy_block(0, sa.off_t0);
#pragma unroll
  for (int j = 0; j < KP; ++j) acc[j * STREAM_BD + tid] = WIDE ? 0.f : bv[j];
  block_done();

  int cursor = 0;                                        // place in the current tap's list
  unsigned long long blk_time = 0;                       // stamping build: the blocks' products
  for (int blk = 0; blk < sa.nblocks; ++blk) {           // uniform
    const bool has_next = blk + 1 < sa.nblocks;
    const uint32_t toff = (blk & 1) ? sa.off_t1 : sa.off_t0;
    const uint32_t tnext = (blk & 1) ? sa.off_t0 : sa.off_t1;
    const unsigned long long blk_t0 = CS_CLOCK();
    if constexpr (!CH) {
      const int t0 = blk * sa.tpb, t1 = min(T_, t0 + sa.tpb);
      for (int t = t0; t < t1; ++t) {
        StreamPre nxt;
        stream_prefetch(nxt, lidx, lval, lcnt, geo, place, t + 1, 0, sa.fd_kw, part);
        if (t == t0 && has_next) copy_block((blk + 1) * sa.RB, tnext);
        stream_tap<GB, false, WIDE>(q, lidx, lval, geo.cap, 0, C, (t - t0) * C, smem, toff,
                                    log2row, lane_tab, col, part);
        q = nxt;
      }
    } else {
      // one tap, the channels [c_lo, c_lo + RB): the quad goes on in the tap's
      // list where the previous block stopped
      const int t0 = blk / sa.cblocks;
      const int c_lo = (blk - t0 * sa.cblocks) * sa.RB;
      if (c_lo == 0) cursor = 0;
      if (has_next) copy_block((blk + 1) * sa.RB, tnext);
      cursor = stream_tap<GB, true, WIDE>(q, lidx, lval, geo.cap, cursor, c_lo + sa.RB, -c_lo, smem,
                                          toff, log2row, lane_tab, col, part);
      const int tn = (blk + 1) / sa.cblocks;
      stream_prefetch(q, lidx, lval, lcnt, geo, place, has_next ? tn : T_, tn == t0 ? cursor : 0,
                      sa.fd_kw, part);
    }
    blk_time += CS_CLOCK() - blk_t0;
    if (has_next) block_done();
  }
  CS_STAMP(17);
  CS_STAMP_ADD(21, blk_time);
  if constexpr (WIDE) {
    wave_lds_order();                                    // a pixel's parts: one wavefront's lanes
    if (live)
      stream_sum_parts<KP>(acc, log2S, sa.pairs, part.s4 >> 2, bv,
                           y + (int64_t)item * geo.c_out + bias0);
  } else {
    stream_kwta<TO, KP, STREAM_BD>(acc, sa.log2U, sa.log2Us, (int64_t)item, live, geo.c_out, sa.k,
                                   sa.write_sums, y, out, lo);
  }
  CS_STAMP(18);
}

}  // namespace cs
