// Sparse-dense convolution with block Complementary Sparsity (the layer of
// conv_dense_blocks.h: dense int8 input, a block = one tap's c_in <= 4
// channels with one Kernel ID) on the matrix cores.
//
// The input is dense, so the layer is a contraction of length kh*kw*c_in and
// the only data-dependent step is where a (tap, set) block's weights belong:
// the Kernel ID routes the block once, when the workgroup builds its weight
// operand, instead of routing one product per (output pixel, tap, set).  The
// products with the zeros of the other kernels cost nothing here: at 7x7x3
// -> 64 the int8 tiles of a 224x224 image take a few percent of the time its
// int32 output takes to write, which is what bounds the kernel.
//
//  * contraction order: a tap is one 32-bit word (its channels in the low
//    bytes, zeros above), a tap row is padded to whole chunks of four taps
//    (16 bytes), KS steps of four chunks (one 16x16x64 MFMA each);
//  * A operand = weights, 16 output channels x 64 bytes a tile, CT tiles held
//    in registers for the whole workgroup (persistent over tiles); B operand
//    = 16 output pixels' windows, read from the staged pixel words; a lane
//    then holds four consecutive channels of one pixel per tile and stores
//    them with 16 bytes (64 contiguous bytes a pixel and instruction);
//  * tile: RO output rows x up to 16*gseg columns; the input rows under it are
//    staged one word per pixel, zero outside the image, each pixel read with
//    one (unaligned) 4-byte load kept inside x.
//
// Measured, 32 images of 224x224x3, 7x7/2, 64 outputs in sets of four (103 MB
// of int32 output, 21 us at the 4.9 TB/s of a large copy): 31 us a call, against
// 104 us for the routed kernel (one LDS add per pixel, tap and set).  Tiles of one
// or two output rows take 38 and 36 us of kernel time against 31 us for four: the
// input rows under a tile are staged less often.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastdiv.h"
#include "mrs_kernels.h"
#include "wave_ops.h"

namespace cs {

constexpr int MB_BD = 256;            // threads per workgroup
constexpr int MB_PRE = 8;             // staged pixels a thread loads together
constexpr int MB_STAGE = 4096;        // staged pixels per tile at most (16 KB)

struct BlocksMfmaArgs {
  int RO;             // output rows per tile
  int gseg;           // groups of 16 output columns per tile row
  int nseg;           // tiles across an output row
  int nrb;            // tiles down an image, ceil(Ho / RO)
  int ntiles;         // B * nrb * nseg
  int SW;             // staged words per input row (even)
  int rows_in;        // staged input rows, (RO - 1) * S + KH
  int cpr;            // chunks per tap row, ceil(KW / 4)
  int nchunk;         // KH * cpr <= 4 * KS
  int64_t xbytes;     // bytes of x
  int img_bytes;      // H * W * C
  FastDiv fd_nseg, fd_nrb, fd_sw, fd_gseg;
};

// A2: the windows of all chunks start at even words (even stride): 8-byte reads.
template <int KS, int CT, bool A2>
__global__ __launch_bounds__(MB_BD, 4) void conv_blocks_mfma(
    const int8_t* __restrict__ x, const uint16_t* __restrict__ aug,
    const uint8_t* __restrict__ kidb, const int32_t* __restrict__ bias, int32_t* __restrict__ y,
    ConvGeom geo, BlocksMfmaArgs ma) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  constexpr int CH = 16 * CT;                            // channels of this workgroup
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int C = geo.C, G = geo.G, n = geo.n, T = geo.KH * geo.KW, S = geo.S;
  const int c0 = (int)blockIdx.y * CH;
  const int q = lane >> 4;                               // chunk within a step, channel quad
  int32_t* bias_s = reinterpret_cast<int32_t*>(smem);    // [CH]
  uint32_t* xs = reinterpret_cast<uint32_t*>(smem + CH * 4);

  // ---- weights: [chunk][channel] 16 bytes in LDS, zero, then every block of
  // (tap, set) at its kernel's channel (four blocks' loads at a time)
  uint32_t* wt = xs;                                     // over the staged pixels
  for (int e = tid; e < 4 * KS * CH * 4; e += MB_BD) wt[e] = 0u;
  for (int e = tid; e < CH; e += MB_BD) bias_s[e] = bias ? bias[c0 + e] : 0;
  __syncthreads();
  for (int e0 = tid; e0 < T * G; e0 += 4 * MB_BD) {
    uint32_t w4[4];
    int kid[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * MB_BD < T * G ? e0 + u * MB_BD : T * G - 1;
      const int t = e / G, g = e - t * G;
      kid[u] = kidb[e];
      w4[u] = 0u;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t a = aug[(size_t)(t * C + (c < C ? c : 0)) * G + g] & 0xFFu;
        w4[u] |= (c < C ? a : 0u) << (8 * c);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * MB_BD;
      const int t = e / G, g = e - t * G;
      // kid < n for cs_pack_blocks output
      const int ch = g * n + (kid[u] < n ? kid[u] : n - 1) - c0;
      if (e >= T * G || ch < 0 || ch >= CH) continue;
      const int ky = t / geo.KW, kx = t - ky * geo.KW;
      wt[((ky * ma.cpr + (kx >> 2)) * CH + ch) * 4 + (kx & 3)] = w4[u];
    }
  }
  __syncthreads();
  v4i wf[KS][CT];
  int off[KS];                                           // the lane's chunk of step s: word offset
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int ck = 4 * s + q;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      wf[s][ct] = *reinterpret_cast<const v4i*>(wt + ((ck * CH) + ct * 16 + (lane & 15)) * 4);
    // chunks past the window meet zero weights: any staged word will do
    const int ky = ck < ma.nchunk ? ck / ma.cpr : 0;
    const int kc = ck < ma.nchunk ? ck - ky * ma.cpr : 0;
    off[s] = ky * ma.SW + 4 * kc + (lane & 15) * S;
  }

  const int nst = ma.rows_in * ma.SW;
  const uint32_t cmask = C == 4 ? 0xFFFFFFFFu : (1u << (8 * C)) - 1u;
  const int groups = ma.RO * ma.gseg;
  for (int tile = blockIdx.x; tile < ma.ntiles; tile += gridDim.x) {
    const uint32_t r = fdiv((uint32_t)tile, ma.fd_nseg);
    const int seg = tile - (int)r * ma.nseg;
    const uint32_t bb = fdiv(r, ma.fd_nrb);
    const int oy0 = ((int)r - (int)bb * ma.nrb) * ma.RO;
    const int ox0 = seg * ma.gseg * 16;
    const int iy0 = oy0 * S - geo.P, ix0 = ox0 * S - geo.P;
    // the image's first byte, and the last place in it that four bytes can be
    // read at (host: an image has 4 .. 2^31 - 1 bytes)
    const int64_t img = (int64_t)bb * ma.img_bytes;
    const unsigned char* xi = reinterpret_cast<const unsigned char*>(x) + img;
    const int64_t left = ma.xbytes - 4 - img;
    const uint32_t olast = left < INT32_MAX ? (uint32_t)left : (uint32_t)INT32_MAX;
    // (the staged places are worked out per tile: held across tiles they would
    // take the registers of the weight tiles)
    const int tv = opaque_int(tid);
    __syncthreads();                                     // xs: weights or the last tile are read
    for (int b0 = 0; b0 < nst; b0 += MB_BD * MB_PRE) {
      uint32_t v[MB_PRE];
#pragma unroll
      for (int u = 0; u < MB_PRE; ++u) {
        const int e = b0 + u * MB_BD + tv;
        const int ry = (int)fdiv((uint32_t)e, ma.fd_sw), col = e - ry * ma.SW;
        const int iy = iy0 + ry, ix = ix0 + col;
        uint32_t w = 0u;
        if (e < nst && iy >= 0 && iy < geo.H && ix >= 0 && ix < geo.W) {
          // four bytes at the pixel, or the last four of x shifted down
          const uint32_t o = (uint32_t)((iy * geo.W + ix) * C);
          const uint32_t a = o < olast ? o : olast;
          __builtin_memcpy(&w, xi + a, 4);
          w = (w >> (8 * (o - a))) & cmask;
        }
        v[u] = w;
      }
#pragma unroll
      for (int u = 0; u < MB_PRE; ++u) {
        const int e = b0 + u * MB_BD + tv;
        if (e < nst) xs[e] = v[u];
      }
    }
    __syncthreads();
    for (int gi = wv; gi < groups; gi += MB_BD / 64) {
      const int ro = (int)fdiv((uint32_t)gi, ma.fd_gseg), gx = gi - ro * ma.gseg;
      const uint32_t* xw = xs + ro * S * ma.SW + gx * 16 * S;
      v4i b[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const uint32_t* p = xw + off[s];
        if constexpr (A2) {
          const uint2 lo2 = *reinterpret_cast<const uint2*>(p);
          const uint2 hi2 = *reinterpret_cast<const uint2*>(p + 2);
          b[s] = v4i{(int)lo2.x, (int)lo2.y, (int)hi2.x, (int)hi2.y};
        } else {
          b[s] = v4i{(int)p[0], (int)p[1], (int)p[2], (int)p[3]};
        }
      }
      v4i acc[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        acc[ct] = *reinterpret_cast<const v4i*>(bias_s + ct * 16 + 4 * q);
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          acc[ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[s][ct], b[s], acc[ct], 0, 0, 0);
      // column = the lane's pixel, rows 4q .. 4q+3 = its channels of each tile
      const int oy = oy0 + ro, ox = ox0 + gx * 16 + (lane & 15);
      if (oy < geo.Ho && ox < geo.Wo) {
        int32_t* yr = y + (((int64_t)bb * geo.Ho + oy) * geo.Wo + ox) * geo.c_out + c0 + 4 * q;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) *reinterpret_cast<v4i*>(yr + ct * 16) = acc[ct];
      }
    }
  }
}

}  // namespace cs
