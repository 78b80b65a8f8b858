// Operand words of an implicitly lowered convolution input.  Index arithmetic
// and loads only (no HIP types), so that a host compiler can check the two
// forms against each other.
#pragma once

#include <stdint.h>

namespace fp8t {

// Implicit lowering of a convolution (Sec. 2.2: a convolution is computed by
// lowering its input and then a GEMM): the lowered matrix Xcol, M = N * OH *
// OW rows (output pixels, row-major n, oh, ow) by KH * KW * C columns (order
// kh, kw, c), is read straight from the NHWC input X:
//   Xcol(p, (kh, kw, c)) = X[n, oh * stride - pad + kh, ow * stride - pad + kw, c]
// (0 outside the image).
struct ConvGeom {
    int H, W, C;        // input height, width, channels
    int KW, KWC;        // kernel width, KW * C
    int OW, OHW;        // output width, OH * OW
    int pad, stride;
    int vec;            // C % 4 == 0 and X 4-byte aligned: 4 channels per load
};

namespace valu_impl {

// One thread's operand words (4 codes each) of a slab of R rows x BK k: the
// operand is Xcol (KC: element (r, k) = Xcol(r, k), rows are output pixels)
// or Xcol^T (element (r, k) = Xcol(k, r)).  A word holds 4 consecutive Xcol
// columns of one pixel: 4 consecutive channels of one input position when
// C % 4 == 0 (one 4-byte load), otherwise gathered byte by byte.
__device__ __forceinline__ uint32_t xcol_byte(const uint8_t* __restrict__ X, const ConvGeom& cg,
                                              int pix, int col) {
    const int n = pix / cg.OHW, rem = pix - n * cg.OHW;
    const int oh = rem / cg.OW, ow = rem - oh * cg.OW;
    const int kh = col / cg.KWC, r2 = col - kh * cg.KWC;
    const int kw = r2 / cg.C, c = r2 - kw * cg.C;
    const int ih = oh * cg.stride - cg.pad + kh, iw = ow * cg.stride - cg.pad + kw;
    if ((unsigned)ih >= (unsigned)cg.H || (unsigned)iw >= (unsigned)cg.W) return 0u;
    return X[(((int64_t)n * cg.H + ih) * cg.W + iw) * cg.C + c];
}

template <bool KC, int R, int BK, int NT, int W>
__device__ __forceinline__ void slab_load_conv(const uint8_t* __restrict__ X, const ConvGeom& cg,
                                               int r0, int rows, int k0, int kend, int tid,
                                               uint32_t (&reg)[W]) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int d = tid + NT * w;
        int r, k;
        if (KC) { r = d / (BK / 4); k = (d % (BK / 4)) * 4; }
        else    { k = d / (R / 4);  r = (d % (R / 4)) * 4; }
        const int gr = r0 + r, gk = k0 + k;
        // pixel and first column of the word; valid columns [col, col + nb)
        const int pix = KC ? gr : gk, col = KC ? gk : gr;
        const bool in = gr < rows && gk < kend;
        const int lim = KC ? kend - gk : rows - gr;
        const int nb = lim < 4 ? lim : 4;
        uint32_t v = 0;
        if (in) {
            // one 4-byte load when the word is 4 aligned channels of one input
            // position (chunk ranges need not start at a multiple of 4)
            if (cg.vec && (col & 3) == 0) {
                const int n = pix / cg.OHW, rem = pix - n * cg.OHW;
                const int oh = rem / cg.OW, ow = rem - oh * cg.OW;
                const int kh = col / cg.KWC, r2 = col - kh * cg.KWC;
                const int kw = r2 / cg.C, c = r2 - kw * cg.C;
                const int ih = oh * cg.stride - cg.pad + kh, iw = ow * cg.stride - cg.pad + kw;
                if ((unsigned)ih < (unsigned)cg.H && (unsigned)iw < (unsigned)cg.W)
                    v = *reinterpret_cast<const uint32_t*>(
                        X + (((int64_t)n * cg.H + ih) * cg.W + iw) * cg.C + c);
                if (nb < 4) v &= (1u << (8 * nb)) - 1u;
            } else {
                for (int b = 0; b < nb; ++b) v |= xcol_byte(X, cg, pix, col + b) << (8 * b);
            }
        }
        reg[w] = v;
    }
}

// The same walk with the index arithmetic carried along, for words of 4 aligned
// channels (ConvGeom::vec, first k a multiple of 4): a piece's slabs follow
// each other in k, so each thread keeps its words' positions in the input and
// its column's (kh, kw, c) and advances them by BK instead of dividing the
// pixel and column of every word (8 divisions per slab and thread; Forward and
// Gradient kernels of a 32 x 14 x 14 x 256 -> 256 3 x 3 convolution 243 / 240
// -> 233 / 234 us).
template <bool KC, int R, int BK, int NT, int W>
struct ConvWalk {
    static_assert(KC ? NT % (BK / 4) == 0 : NT % (R / 4) == 0, "a thread's words share a column");
    int at;                     // first k of the slab the walk stands at
    int kh, kw, c;              // the thread's column: KC that of the slab, else fixed
    int n[W], y[W], x[W];       // KC: image and input origin of the word's pixel (a row of
                                // the operand); else its pixel (n, oh, ow)
    __device__ __forceinline__ void column(const ConvGeom& cg, int col) {
        kh = col / cg.KWC;
        const int r2 = col - kh * cg.KWC;
        kw = r2 / cg.C;
        c = r2 - kw * cg.C;
    }
    __device__ __forceinline__ void start(const ConvGeom& cg, int r0, int k0, int tid) {
        at = k0;
        column(cg, KC ? k0 + (tid % (BK / 4)) * 4 : r0 + (tid % (R / 4)) * 4);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int d = tid + NT * w;
            const int pix = KC ? r0 + d / (BK / 4) : k0 + d / (R / 4);
            n[w] = pix / cg.OHW;
            const int rem = pix - n[w] * cg.OHW;
            const int oh = rem / cg.OW, ow = rem - oh * cg.OW;
            y[w] = KC ? oh * cg.stride - cg.pad : oh;
            x[w] = KC ? ow * cg.stride - cg.pad : ow;
        }
    }
    // on to the slab at k0 = at + BK
    __device__ __forceinline__ void next(const ConvGeom& cg, int k0, int tid) {
        at = k0;
        if (KC) {
            if (2 * cg.C >= BK) {
                c += BK;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if (c >= cg.C) {
                        c -= cg.C;
                        if (++kw == cg.KW) { kw = 0; ++kh; }
                    }
                }
            } else {
                column(cg, k0 + (tid % (BK / 4)) * 4);
            }
        } else {
            // BK pixels on: whole images, rows and columns, with carries
            const int OH = cg.OHW / cg.OW;
            const int dn = BK / cg.OHW, dr = BK - dn * cg.OHW;
            const int dy = dr / cg.OW, dx = dr - dy * cg.OW;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                x[w] += dx;
                y[w] += dy;
                if (x[w] >= cg.OW) { x[w] -= cg.OW; ++y[w]; }
                n[w] += dn;
                if (y[w] >= OH) { y[w] -= OH; ++n[w]; }
            }
        }
    }
    // The slab at k0: the one the walk stands at, or the next one.  Moved on
    // here and not after a load, so that a piece of one slab does not pay for a
    // step it never takes, and in at most two carries or by division, not in a
    // loop over few channels (8 turns for C = 4: Forward of 14 x 14 x 14 x 4,
    // 3 x 3, to 32 channels 15.1 us, now 14.1, words divided out 13.6).
    __device__ __forceinline__ void load(const uint8_t* __restrict__ X, const ConvGeom& cg, int r0,
                                         int rows, int k0, int kend, int tid, uint32_t (&reg)[W]) {
        if (k0 != at) next(cg, k0, tid);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int d = tid + NT * w;
            const int gr = r0 + (KC ? d / (BK / 4) : (d % (R / 4)) * 4);
            const int gk = k0 + (KC ? (d % (BK / 4)) * 4 : d / (R / 4));
            const int ih = (KC ? y[w] : y[w] * cg.stride - cg.pad) + kh;
            const int iw = (KC ? x[w] : x[w] * cg.stride - cg.pad) + kw;
            uint32_t v = 0;
            if (gr < rows && gk < kend && (unsigned)ih < (unsigned)cg.H &&
                (unsigned)iw < (unsigned)cg.W) {
                v = *reinterpret_cast<const uint32_t*>(
                    X + (((int64_t)n[w] * cg.H + ih) * cg.W + iw) * cg.C + c);
                const int lim = KC ? kend - gk : rows - gr;
                if (lim < 4) v &= (1u << (8 * lim)) - 1u;
            }
            reg[w] = v;
        }
    }
};

}  // namespace valu_impl
}  // namespace fp8t
