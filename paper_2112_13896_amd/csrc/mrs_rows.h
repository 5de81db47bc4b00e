// One wavefront per item: Multiply, Route and Sum (Section 3.2 steps 3-5)
// and k-WTA (Section 3.3.3) for an int8 layer whose window is one tap (a 1x1
// convolution with stride 1) with many items, each with a short list and a row of
// 129-2048 outputs or a k over 32, or the sums alone.
//
//  * the workgroup stages the packed table (value and Kernel ID per slot, the
//    ID already turned into the byte offset of its accumulator within the
//    set) in LDS once; after that its wavefronts work without workgroup
//    barriers, each on its own items;
//  * a wavefront's accumulator row is in output-channel order and starts at
//    the bias; lane j holds entries j and j + 64 of the item's list (table row
//    offset and value); sets in groups of 64 take the entries one after
//    another (broadcast from their lanes), a rest of at most 32 sets as 64 /
//    rest slices, a slice taking every (64 / rest)-th entry; a lane reads the
//    table entry of (entry, set g), multiplies and adds the product to channel
//    g*n + kid with an LDS integer add (exact in any order, so lanes may meet
//    on one channel): three vector instructions a product, the multiply and
//    the address add each selecting their byte of the entry;
//  * k-WTA: lane l holds channels l, l + 64, ... of the row in registers, as
//    differences from the row minimum, and the row's memory becomes a 512-bin
//    histogram of their top nine bits; a scan from the top bin finds the bin of
//    the k-th largest.  With a row's sums spread over the bins that bin holds a
//    key or two: if all of it wins the threshold lies just below it, else a few
//    keys are picked out one by one; only a crowded bin takes another
//    histogram pass over nine more bits.  Ties go to the lower channel;
//  * the winners' list positions are ballot ranks (channel order is column
//    order, lane order within a column): a compare and a count of mask bits a
//    column, no scans; the list is staged in the row's memory and copied out
//    with consecutive lanes on consecutive entries, then the row is put back to
//    the bias for the next item.
//
// What bounds it: the issue of a wavefront's serial chain (990 instructions an
// item, 480 of them vector, its share of the wavefront's set-up included; six to
// eight wavefronts a SIMD) and, behind it, the LDS adds.  25,088 items, 96 -> 576 in sets of eight, 12 entries,
// 72 winners as int8 lists: 46.1 -> 32.5 us (740 vector instructions an item
// before: a full histogram pass per nine bits, list positions by scans over
// strided lanes, an item loop compiled as divergent); the 576 -> 96 sums of the
// same items 22.7 -> 17.2 us (72 entries in one piece instead of two).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastdiv.h"
#include "kwta_kernels.h"
#include "mrs_kernels.h"
#include "wave_ops.h"

namespace cs {

constexpr int ROWS_BD = 1024;             // most threads per workgroup (16 wavefronts)
constexpr int ROWS_BATCH = 4;             // table entries a lane reads before it adds
constexpr int ROWS_ENTS = 128;            // list entries held by a wavefront at a time
constexpr int ROWS_ENT_STRIDE = ROWS_ENTS + 2;   // int2 slots per wavefront entry copy (+ zero + pad)
constexpr int ROWS_DIGIT = 9;             // bits per histogram pass
constexpr int ROWS_BINS = 1 << ROWS_DIGIT;
constexpr int ROWS_HIST = ROWS_BINS + 64; // bins + one spare bin per lane
constexpr int ROWS_STAGE = 4;             // 16-byte table loads of a thread in flight
constexpr int ROWS_FEW = 16;              // list entries up to which a rest of sets runs as a group
constexpr int ROWS_EXTRACT = 4;           // most winners of a bin picked out one by one
constexpr int ROWS_BIN_KEYS = 16;         // ... from at most so many keys of the bin

struct RowsArgs {
  int k;
  int shift;
  int write_sums;
  int qf;             // groups of 64 sets with wavefront-uniform entries (the last may be partial)
  int S;              // slices of the remaining Gs sets (0: none)
  int gbase;          // first of the remaining sets (64 qf)
  uint32_t off_acc;    // LDS byte offset of the wavefronts' rows (table at 0)
  uint32_t acc_words;  // words per wavefront row (whole columns, >= ROWS_HIST for a k-WTA)
  uint32_t off_bias;   // LDS byte offset of the bias (whole 64-channel columns)
  uint32_t off_ent;    // LDS byte offset of the wavefronts' entry copies (S > 0 only)
  int64_t per_wg;      // items per workgroup
  FastDiv fd_g;        // / Gs
};

// A staged table entry: the value in byte 0, the accumulator's byte offset
// within its set (4 * kid <= 124) in byte 1.
__device__ __forceinline__ uint32_t rows_entry2(uint32_t w) {       // two entries
  return (w & 0x00FF00FFu) | ((w & 0x1F001F00u) << 2);
}

// What the kernel writes: the sums, the winners as lists, or densely.
constexpr int ROWS_SUMS = 0, ROWS_LISTS = 1, ROWS_DENSE = 2;

// M: 64-channel columns held by a lane (64 M >= c_out; 0, sums only: any number, looped
// over).  FULL: c_out == 64 M.  H: 64-entry halves of ROWS_ENTS a list can reach into.
// Short rows of short lists are all overhead per item, and the loops' count: 25,088
// items 32 -> 192, 4 entries, sums 11.8 us with M = 0 and both halves, 10.8 with M = 3,
// 10.5 with H = 1 too; 16 -> 96, 3 entries, 10.6, 10.0 and 9.5.
// Registers held to eight wavefronts per SIMD up to nine columns.
template <typename TO, int MODE, int M, bool FULL, int H = 2>
__global__ __launch_bounds__(ROWS_BD, M <= 9 ? 8 : 4) void mrs_rows(const uint16_t* __restrict__ lidx,
                                                    const int8_t* __restrict__ lval,
                                                    const int32_t* __restrict__ lcnt,
                                                    const uint16_t* __restrict__ aug,
                                                    const int32_t* __restrict__ bias,
                                                    int32_t* __restrict__ y, TO* __restrict__ out,
                                                    ListOut lo, ConvGeom geo, RowsArgs ra,
                                                    int64_t items) {
  typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  // the wavefront's number as a scalar: with it in a vector register the whole
  // item loop is compiled as divergent (masks for branches, 64-bit addresses
  // in vector registers)
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nthr = (int)blockDim.x, nwv = nthr >> 6;
  const int G = geo.G, n = geo.n, c = geo.c_out, cap = geo.cap;
  // the packed table [C][G] is at LDS offset 0
  int32_t* acc = reinterpret_cast<int32_t*>(smem + ra.off_acc) + wv * ra.acc_words;
  unsigned char* accb = reinterpret_cast<unsigned char*>(acc);
  uint32_t* hist = reinterpret_cast<uint32_t*>(acc);                // the same words
  int32_t* bias_s = reinterpret_cast<int32_t*>(smem + ra.off_bias); // [64 cols]
  // (row offset, value) of up to ROWS_ENTS entries, then a (0, 0) entry for slots past the list
  int2* ent = reinterpret_cast<int2*>(smem + ra.off_ent) + wv * ROWS_ENT_STRIDE;

  // ---- the table into LDS (16-byte pieces), once per workgroup
  {
    const int nb = geo.C * G * 2;                                   // R = C (one tap)
    const int n16 = nb / 16;
    const uint4* src = reinterpret_cast<const uint4*>(aug);
    uint4* dst = reinterpret_cast<uint4*>(smem);
    for (int b0 = 0; b0 < n16; b0 += nthr * ROWS_STAGE) {
      uint4 v[ROWS_STAGE];
#pragma unroll
      for (int u = 0; u < ROWS_STAGE; ++u) {
        const int e = b0 + u * nthr + tid;
        v[u] = src[e < n16 ? e : n16 - 1];
      }
#pragma unroll
      for (int u = 0; u < ROWS_STAGE; ++u) {
        const int e = b0 + u * nthr + tid;
        if (e < n16)
          dst[e] = make_uint4(rows_entry2(v[u].x), rows_entry2(v[u].y), rows_entry2(v[u].z),
                              rows_entry2(v[u].w));
      }
    }
    for (int e = n16 * 8 + tid; e < nb / 2; e += nthr)              // the tail entries
      reinterpret_cast<uint16_t*>(smem)[e] = (uint16_t)rows_entry2(aug[e]);
  }
  const int cols = (c + 63) >> 6;
  for (int o = tid; o < 64 * cols; o += nthr) bias_s[o] = bias != nullptr && o < c ? bias[o] : 0;
  if (ra.S > 0 && lane == 0) ent[ROWS_ENTS] = make_int2(0, 0);
  __syncthreads();
  // columns past c_out are skipped (uniform); the last column's lanes past
  // c_out are pads: words of their own, never in the histogram, never winners
  // (c_out is made unknown again at each loop, or the comparisons would all be
  // held in scalar registers across the item loop and spilled)
  int cc = c;
  auto has = [&](int j) { return FULL || 64 * j < cc; };
  auto valid = [&](int j, int ln) { return FULL || 64 * j + ln < cc; };
  auto reset_row = [&](int ln) {
    if constexpr (M == 0) {
      for (int j = 0; j < cols; ++j) acc[64 * j + ln] = bias_s[64 * j + ln];
    } else {
      cc = opaque_uniform(c);
#pragma unroll
      for (int j = 0; j < M; ++j)
        if (has(j)) acc[64 * j + ln] = bias_s[64 * j + ln];
    }
  };
  reset_row(lane);

  const int64_t ib = (int64_t)blockIdx.x * ra.per_wg;
  const int nit = (int)(items - ib < ra.per_wg ? items - ib : ra.per_wg);
  // the remaining sets as slices: this lane's slice s and set gbase + g0
  // (lanes past S * Gs idle)
  const int s = (int)fdiv((uint32_t)lane, ra.fd_g);
  const int g0 = lane - s * (int)ra.fd_g.d;
  const bool job = s < ra.S;

  // the next item's count and first 128 list entries (two per lane) are loaded
  // while the current item is processed
  int cnt_n = 0;
  uint16_t pi_n[2] = {0, 0};
  int8_t pv_n[2] = {0, 0};
  auto prefetch = [&](int li) {
    if (li < nit) {
      const int64_t it = ib + li;
      cnt_n = lcnt[it];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        if (64 * h < cap) {                                         // uniform
          const int j = lane + 64 * h < cap ? lane + 64 * h : cap - 1;
          pi_n[h] = lidx[it * cap + j];
          pv_n[h] = lval[it * cap + j];
        }
      }
    }
  };
  auto add = [&](unsigned char* ag, uint32_t w, int x) {
    __hip_atomic_fetch_add(reinterpret_cast<int32_t*>(ag + ((w >> 8) & 0xFFu)),
                           __mul24(x, (int)(int8_t)(w & 0xFFu)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  int li = wv;                                                      // uniform
  prefetch(li);
  while (li < nit) {
    const int lnext = li + nwv;
    // (the lane's places are worked out per item, not held for every column)
    const int lane = opaque_int(tid) & 63;
    const int64_t it = ib + li;
    int cnt = __builtin_amdgcn_readfirstlane(cnt_n);
    cnt = cnt < 0 ? 0 : (cnt > cap ? cap : cnt);
    uint16_t pi[2] = {pi_n[0], pi_n[1]};
    int8_t pv[2] = {pv_n[0], pv_n[1]};
    prefetch(lnext);

    // ---- Multiply, Route, Sum
    const int64_t lb = it * cap;
    // a rest of sets runs as one more (partial) group when the list is short:
    // a product in a group costs three instructions, the entry copy and the
    // slices' reads of it about forty once and nine an entry slot
    const bool group = ra.S > 0 && ra.qf > 0 && cnt <= ROWS_FEW;
    const int qf = group ? ra.qf + 1 : ra.qf;
    for (int j0 = 0; j0 < cnt; j0 += ROWS_ENTS) {                   // uniform
      const int nb = cnt - j0 < ROWS_ENTS ? cnt - j0 : ROWS_ENTS;
      // lane l holds entries j0 + l and j0 + l + 64: their table rows' byte
      // offsets and their values (zero past the list)
      int pre[2], xv[2];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int j = lane + 64 * h;
        pre[h] = xv[h] = 0;
        if (64 * h < nb) {                                          // uniform
          if (j0 > 0) {
            const int jc = j < nb ? j : nb - 1;
            pi[h] = lidx[lb + j0 + jc];
            pv[h] = lval[lb + j0 + jc];
          }
          pre[h] = j < nb ? (int)pi[h] * G * 2 : 0;
          xv[h] = j < nb ? (int)pv[h] : 0;
        }
      }
      // groups of 64 sets: lane l takes set 64 q + l, the entries one after
      // another (wavefront-uniform, read from their lanes)
      if (qf > 0) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const int nh = nb - 64 * h < 64 ? nb - 64 * h : 64;
          for (int e = 0; e < nh; e += ROWS_BATCH) {                // uniform
            int sp[ROWS_BATCH], sx[ROWS_BATCH];
#pragma unroll
            for (int u = 0; u < ROWS_BATCH; ++u) {                  // lanes past nh hold (0, 0)
              sp[u] = __builtin_amdgcn_readlane(pre[h], e + u);
              sx[u] = __builtin_amdgcn_readlane(xv[h], e + u);
            }
            auto group_add = [&](int g) {                           // this lane's set g
              CS_COUNT_PRODUCTS_ADD(min(ROWS_BATCH, nh - e));
              uint32_t w[ROWS_BATCH];
#pragma unroll
              for (int u = 0; u < ROWS_BATCH; ++u)
                w[u] = *reinterpret_cast<const uint16_t*>(smem + sp[u] + 2 * g);
              unsigned char* ag = accb + g * n * 4;
#pragma unroll
              for (int u = 0; u < ROWS_BATCH; ++u) add(ag, w[u], sx[u]);
            };
            // all lanes but in a last partial group
            if (lane < G) group_add(lane);
            for (int q = 1; q < qf; ++q)                            // uniform
              if (lane + 64 * q < G) group_add(lane + 64 * q);
          }
        }
      }
      // the remaining Gs sets (from gbase on) as S slices: lane (s, g0) takes
      // set gbase + g0 and the entries s, s + S, ..., read from a
      // wavefront-private copy of the entries in LDS
      if (ra.S > 0 && !group) {
        ent[lane] = make_int2(pre[0], xv[0]);
        if (H > 1 && nb > 64) ent[lane + 64] = make_int2(pre[1], xv[1]);
        wave_lds_order();
        if (job) {
          const int S = ra.S;
          const int g = ra.gbase + g0;
          unsigned char* ag = accb + g * n * 4;
          for (int e = 0; e < nb; e += S * ROWS_BATCH) {            // uniform
            int2 en[ROWS_BATCH];
#pragma unroll
            for (int u = 0; u < ROWS_BATCH; ++u) {
              const int el = e + s + S * u;
              en[u] = ent[el < nb ? el : ROWS_ENTS];
            }
            CS_COUNT_PRODUCTS_ADD(min(ROWS_BATCH, (nb - e - s + S - 1) / S));
            uint32_t w[ROWS_BATCH];
#pragma unroll
            for (int u = 0; u < ROWS_BATCH; ++u)
              w[u] = *reinterpret_cast<const uint16_t*>(smem + en[u].x + 2 * g);
#pragma unroll
            for (int u = 0; u < ROWS_BATCH; ++u) add(ag, w[u], en[u].y);
          }
        }
        wave_lds_order();                                           // before the buffer is rewritten
      }
    }
    wave_lds_order();

    if constexpr (MODE == ROWS_SUMS) {
      // ---- sums only: the row to HBM (16-byte stores when c_out allows),
      // then back to the bias
      if ((c & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0) {
        typedef int32_t i4_t __attribute__((ext_vector_type(4)));
        i4_t* y4 = reinterpret_cast<i4_t*>(y + it * c);
        for (int o = lane; o < (c >> 2); o += 64) y4[o] = reinterpret_cast<const i4_t*>(acc)[o];
      } else {
        for (int o = lane; o < c; o += 64) y[it * c + o] = acc[o];
      }
      wave_lds_order();
      reset_row(lane);
      li = lnext;
      continue;
    } else {

    // ---- the row into registers (key: the difference from the row's
    // minimum); its memory becomes the histogram
    uint32_t key[M];
    int32_t vmin = INT32_MAX, vmax = INT32_MIN;
    cc = opaque_uniform(c);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if (has(j)) {
        const int32_t v = acc[64 * j + lane];
        key[j] = (uint32_t)v;
        if (valid(j, lane)) {
          if (ra.write_sums) y[it * c + 64 * j + lane] = v;
          vmin = v < vmin ? v : vmin;
          vmax = v > vmax ? v : vmax;
        }
      }
    }
    // (order keys: the unsigned reductions of the wavefront)
    const uint32_t kmn = wave_min_u32(order_key(vmin)), kmx = wave_max_u32(order_key(vmax));
    const uint32_t range = kmx - kmn;
    const uint32_t vbase = kmn ^ 0x80000000u;                       // the minimum's bits
    cc = opaque_uniform(c);
#pragma unroll
    for (int j = 0; j < M; ++j)
      if (has(j)) key[j] -= vbase;
    const int k = ra.k;
    // winners: key > thr, and the first `need` keys (lowest channels) == thr
    uint32_t thr = 0u;
    int need = 0;
    if (k <= 0) {
      thr = 0xFFFFFFFFu;
    } else if (k >= c) {
      need = c;                                                     // every key >= 0 wins
    } else if (range == 0u) {
      need = k;
    } else {
      int rem = 32 - __builtin_clz(range);                          // bits not yet resolved
      uint32_t prefix = 0u;                                         // the bits above them
      int nd = k;                                                   // winners among the prefix's keys
      const u4_t z = {0u, 0u, 0u, 0u};
      for (bool first = true;; first = false) {                     // uniform
        const int width = rem < ROWS_DIGIT ? rem : ROWS_DIGIT;
        const int sh = rem - width;
        wave_lds_order();                                           // the row (or bins) read
        reinterpret_cast<u4_t*>(hist)[lane] = z;
        reinterpret_cast<u4_t*>(hist)[64 + lane] = z;
        wave_lds_order();
        const int spare = ROWS_BINS + lane;
        const uint32_t dmask = (1u << width) - 1u;
        cc = opaque_uniform(c);
#pragma unroll
        for (int j = 0; j < M; ++j) {
          if (has(j)) {
            int bin;
            if (first) {
              bin = valid(j, lane) ? (int)(key[j] >> sh) : spare;
            } else {
              const bool in = valid(j, lane) && (key[j] >> rem) == prefix;   // rem < 32 here
              bin = in ? (int)((key[j] >> sh) & dmask) : spare;
            }
            __hip_atomic_fetch_add(hist + bin, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
        wave_lds_order();
        // lane l holds bins 8(63 - l) .. 8(63 - l) + 7: an inclusive scan over
        // lanes counts the keys in a lane's bins and above
        const int b0 = 8 * (63 - lane);
        const u4_t h0 = reinterpret_cast<const u4_t*>(hist + b0)[0];
        const u4_t h1 = reinterpret_cast<const u4_t*>(hist + b0)[1];
        const int ls = (int)((h0.x + h0.y) + (h0.z + h0.w) + (h1.x + h1.y) + (h1.z + h1.w));
        const int incl = (int)wave_incl_scan((uint32_t)ls, 0u, OpAdd{});
        const uint64_t fb = __ballot(incl >= nd);                   // not empty: nd <= the prefix's keys
        const int f = __ffsll((unsigned long long)fb) - 1;
        const int above = __builtin_amdgcn_readlane(incl - ls, f);
        // the eight bins of that lane, highest first, in lanes 0..7
        const int bl = 8 * (63 - f) + 7 - (lane & 7);
        const int hb = (int)hist[bl];
        int run = hb;
        run += __builtin_amdgcn_update_dpp(0, run, 0x111, 0xF, 0xF, false);
        run += __builtin_amdgcn_update_dpp(0, run, 0x112, 0xF, 0xF, false);
        run += __builtin_amdgcn_update_dpp(0, run, 0x114, 0xF, 0xF, false);
        const uint64_t gb = __ballot(above + run >= nd);            // lanes 0..7: not empty
        const int p = __ffsll((unsigned long long)gb) - 1;
        const int m = __builtin_amdgcn_readlane(hb, p);             // keys of the bin
        nd -= above + __builtin_amdgcn_readlane(run, p) - m;        // of them that win, 1 .. m
        prefix = (prefix << width) | (uint32_t)(8 * (63 - f) + 7 - p);
        rem = sh;
        if (m == nd) {                  // the whole bin wins (not the lowest bin: k < c)
          thr = (prefix << rem) - 1u;
          break;
        }
        if (rem == 0) {                                             // one value, some of its copies win
          thr = prefix;
          need = nd;
          break;
        }
        if (nd <= ROWS_EXTRACT && m <= ROWS_BIN_KEYS) {
          // the bin's keys one after another into a sorted list of its largest
          // (scalars; key - base + 1, so 0 is no key)
          const uint32_t base = prefix << rem;
          uint32_t top[ROWS_EXTRACT + 1] = {0u};
          cc = opaque_uniform(c);
#pragma unroll
          for (int j = 0; j < M; ++j) {
            if (has(j)) {
              const uint32_t d = key[j] - base;                     // below the bin: wraps high
              uint64_t in = __ballot(valid(j, lane) && d < (1u << rem));
              while (in != 0ull) {                                  // uniform, m rounds in all
                const int l = __ffsll((unsigned long long)in) - 1;
                in &= in - 1ull;
                uint32_t x = 1u + (uint32_t)__builtin_amdgcn_readlane((int)d, l);
#pragma unroll
                for (int t = 0; t <= ROWS_EXTRACT; ++t) {
                  const uint32_t hi = top[t] > x ? top[t] : x;
                  x = top[t] > x ? x : top[t];
                  top[t] = hi;
                }
              }
            }
          }
          uint32_t val = top[0], next = top[1];                     // the nd-th and the one after
          int gt = 0;
#pragma unroll
          for (int t = 1; t < ROWS_EXTRACT; ++t) {
            val = t < nd ? top[t] : val;
            next = t < nd ? top[t + 1] : next;
          }
#pragma unroll
          for (int t = 0; t < ROWS_EXTRACT; ++t) gt += top[t] > val ? 1 : 0;
          const bool split = next == val;                           // copies of it that lose
          thr = base + val - (split ? 1u : 2u);                     // (not below 0: k < c)
          need = split ? nd - gt : 0;
          break;
        }
      }
    }
    // ---- winners in channel order, at list positions counted by ballots
    int total = 0;
    wave_lds_order();                                               // after the histogram reads
    uint16_t* gx = nullptr;
    TO* gv = nullptr;
    if constexpr (MODE == ROWS_LISTS) {
      gx = lo.idx + it * lo.cap;
      gv = static_cast<TO*>(lo.val) + it * lo.cap;
    }
    // list position of a column's winner: the winners of the columns before
    // and of the lanes before
    auto rank = [&](uint64_t mask, int before) {
      return (int)__builtin_amdgcn_mbcnt_hi(
          (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)before));
    };
    // the keys and channels of the winners staged in the row's memory, then
    // requantised and written with consecutive lanes on consecutive entries:
    // when they fit there, no tie is split and no winner's output can be zero
    // (the least winner, thr + 1, is at least 2^shift)
    const uint32_t off_ch = ((uint32_t)k * 4 + 15) & ~15u;
    bool fast = false;
    if constexpr (MODE == ROWS_LISTS) {
      const int64_t least = (int64_t)(int32_t)vbase + (int64_t)thr + 1;
      fast = need == 0 && least >= (sizeof(TO) == 1 ? (int64_t)1 << ra.shift : (int64_t)1) &&
             off_ch + 2u * (uint32_t)k <= 4u * ra.acc_words;
    }
    if (fast) {                                                     // uniform
      uint16_t* sch = reinterpret_cast<uint16_t*>(accb + off_ch);
      cc = opaque_uniform(c);
#pragma unroll
      for (int j = 0; j < M; ++j) {
        if (has(j)) {
          const bool win = valid(j, lane) && key[j] > thr;
          const uint64_t wb = __ballot(win);
          const int pos = rank(wb, total);
          if (win) {
            hist[pos] = key[j];
            sch[pos] = (uint16_t)(64 * j + lane);
          }
          total += __popcll(wb);
        }
      }
      wave_lds_order();
      for (int q = lane; q < total; q += 64) {
        gx[q] = sch[q];
        gv[q] = kwta_out<int32_t, TO>((int32_t)(hist[q] + vbase), ra.shift);
      }
    } else {
      int ties = 0;
      cc = opaque_uniform(c);
#pragma unroll
      for (int j = 0; j < M; ++j) {
        if (has(j)) {
          const bool eq = need > 0 && valid(j, lane) && key[j] == thr;
          const uint64_t eb = __ballot(eq);
          const bool win = (valid(j, lane) && key[j] > thr) || (eq && rank(eb, ties) < need);
          ties += __popcll(eb);
          const TO ov = kwta_out<int32_t, TO>((int32_t)(key[j] + vbase), ra.shift);
          if constexpr (MODE == ROWS_LISTS) {
            const bool put = win && ov != TO(0);
            const uint64_t pb = __ballot(put);
            const int pos = rank(pb, total);
            if (put) {
              gx[pos] = (uint16_t)(64 * j + lane);
              gv[pos] = ov;
            }
            total += __popcll(pb);
          } else {
            if (valid(j, lane)) out[it * c + 64 * j + lane] = win ? ov : TO(0);
          }
        }
      }
    }
    if constexpr (MODE == ROWS_LISTS) {
      if (lane == 0) lo.cnt[it] = total;
    }
    // ---- the row back to the bias for the next item
    wave_lds_order();
    reset_row(lane);
    li = lnext;
    }
  }
}

}  // namespace cs
