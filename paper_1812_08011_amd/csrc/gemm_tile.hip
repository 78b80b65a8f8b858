// chunk_gemm_sr: the chunk-based GEMM of Sec. 2.3 / Fig. 3(a) with FP8
// operands and every FP16 addition rounded stochastically (Eq. (1)) instead
// of to nearest -- the paper's second rounding mode after FP16 additions,
// whose behaviour on long accumulations Fig. 3(b) compares with nearest
// rounding.  A vector-ALU tile kernel.
//
// Each addition first forms the FP32 sum of the running value and the next
// product (a product of two FP8 values is exact in FP32) and then rounds it
// into FP16.  As in chunk_gemm's exact mode, FP16 quantities are held scaled
// by 2^96 (fp8t_device.h), so FP16 overflow is FP32 overflow and FP16
// subnormals are FP32 normals: operands enter as a(k) 2^96 and b(k).
// Stochastic rounding of the 14 discarded mantissa bits D with uniform u
// rounds the magnitude up iff D > (u >> 2); adding (2^14 - 1 - (u >> 2)) to
// the raw bits and clearing the low 14 bits does exactly that, with the carry
// running into the exponent (and to the Inf encoding past the largest FP16
// value).  Sums below 2^-30 are multiples of 2^-39 with at most 9 significant
// bits, so their discarded bits are zero and the rounding leaves them
// unchanged, as the fixed subnormal step requires.
//
// Random bits: Philox4x32-10, key = seed, eight 16-bit uniforms per block
// (word halves, low half first).  The addition of product k into output
// (i, j) takes uniform 4 (k mod 2) + (j mod 4) of block (i, j / 4, k / 2,
// 2 offset): a thread owning 4 x 4 outputs (four rows of four aligned
// columns) draws four blocks per two k.  The addition of chunk c into the
// running sum takes uniform j mod 8 of block (i, j / 8, c, 2 offset + 1).
//
// The work decomposition is the persistent plan of gemm_plan.h: whole tiles,
// then the chunks of the remaining tiles shared out as ranges; a piece that
// does not start at chunk 0 leaves each chunk's FP16 sum in the workspace and
// chunk_fold_sr continues the running sum over them in ascending order, with
// the same random bits -- the result does not depend on the plan.
#include "fp8t_device.h"
#include "fp8train.h"
#include "fp8t_host.h"
#include "gemm_plan.h"

#include <stdio.h>

#include <type_traits>

namespace fp8t {
namespace {

constexpr int kT = 4;                 // outputs per thread in each direction
constexpr int kTiles = 16;            // threads per tile edge
constexpr int kBM = kT * kTiles, kBN = kT * kTiles;
constexpr int kNT = kTiles * kTiles;  // 256 threads
constexpr int kBK = 32;               // k per LDS slab (a multiple of 8)
constexpr int kPitch = kBM + 4;       // floats per LDS row
constexpr size_t kWsAlign = 256;

struct TileArgs {
    const uint8_t* A;
    const uint8_t* B;
    uint16_t* C;
    uint16_t* ws;                     // chunk sums of the shared tiles
    int64_t lda, ldb, ldc;
    int M, N, K, CL;
    uint32_t k0, k1;                  // Philox key (stochastic rounding)
    uint32_t w3;                      // 2 * offset
    int c_vec;                        // C rows allow 8-byte stores of 4 codes
    int a_vec, b_vec;                 // A / B rows allow 8-element loads
};

// Uniform-derived addend: (2^14 - 1) - (u >> 2) for the 16-bit uniform in
// bits [16 h, 16 h + 16) of word w, taken from the complemented word.
__device__ __forceinline__ uint32_t sr_addend(uint32_t nw, int h) {
    return __builtin_amdgcn_ubfe(nw, 16 * h + 2, 14);
}

// Stochastic rounding of a scaled-domain float given its addend.
__device__ __forceinline__ float sr16s(float x, uint32_t add) {
    return __uint_as_float((__float_as_uint(x) + add) & 0xFFFFC000u);
}

__device__ __forceinline__ u32x4 block_of(uint32_t i, uint32_t j, uint32_t q, uint32_t w3,
                                          const TileArgs& g) {
    const u32x4 c = {i, j, q, w3};
    return philox4x32_10(c, g.k0, g.k1);
}

// The uniforms of a thread's 4 x 4 outputs for products k = 2 kq, 2 kq + 1:
// Philox blocks (i + r, j4, kq, w3), r = 0 .. 3, complemented.  The first
// three rounds share most of their work between the blocks of a thread and
// between its k: with round q's products p0 = M0 x, p1 = M1 z,
//   round 1: p0 = M0 (i + r) does not depend on k, p1 = M1 kq is wave-uniform;
//   round 2: p0 = M0 x is the same for the four rows (x = hi(M1 kq) ^ j4 ^ key),
//            p1 = M1 z does not depend on k (z = hi(M0 (i + r)) ^ w3 ^ key);
//   round 3 xors with values of the row or of k alone.
// What depends on the row alone is computed once per tile (RowBits), so four
// blocks take 65 multiplications instead of 80.  The keys of rounds 4 .. 10
// are held in vector registers: the three-input xor issues at half rate with
// a scalar operand.  Bound by the vector ALUs: about 5.8 full-rate slots of
// Philox per multiply-accumulate and 4.5 for the sum.  Measured, 512 x 512
// outputs, K 4096: 346 -> 278 us, most of it from four waves per SIMD (the
// chunk end outside the loop over k) instead of two.
struct LateKeys {
    uint32_t a[7], b[7];              // keys of rounds 4 .. 10
    __device__ __forceinline__ explicit LateKeys(const TileArgs& g) {
#pragma unroll
        for (uint32_t r = 0; r < 7; ++r) {
            a[r] = in_vgpr(g.k0 + (r + 3) * kPhiloxW0);
            b[r] = in_vgpr(g.k1 + (r + 3) * kPhiloxW1);
        }
    }
};

struct RowBits {
    uint32_t jk;                      // j4 ^ key of round 1
    uint32_t hz[kT];                  // hi(M1 z) of round 2
    uint32_t lz[kT];                  // lo(M1 z) of round 2 ^ round 3's first key
    uint32_t lx[kT];                  // lo(M0 (i + r)) of round 1 ^ round 2's second key
    __device__ __forceinline__ RowBits(uint32_t i, uint32_t j4, const TileArgs& g) {
        jk = j4 ^ g.k0;
#pragma unroll
        for (uint32_t r = 0; r < kT; ++r) {
            const uint64_t p0 = (uint64_t)kPhiloxM0 * (i + r);
            const uint32_t z = (uint32_t)(p0 >> 32) ^ g.w3 ^ g.k1;
            const uint64_t p1 = (uint64_t)kPhiloxM1 * z;
            hz[r] = (uint32_t)(p1 >> 32);
            lz[r] = (uint32_t)p1 ^ (g.k0 + 2u * kPhiloxW0);
            lx[r] = (uint32_t)p0 ^ (g.k1 + kPhiloxW1);
        }
    }
    // kq wave-uniform
    __device__ __forceinline__ void blocks(uint32_t kq, const LateKeys& key, const TileArgs& g,
                                           uint32_t (&nw)[kT][4]) const {
        const uint64_t u = (uint64_t)kPhiloxM1 * kq;                    // round 1, uniform
        const uint32_t yk = in_vgpr((uint32_t)u ^ (g.k0 + kPhiloxW0));
        const uint64_t s = (uint64_t)kPhiloxM0 * (jk ^ (uint32_t)(u >> 32));   // round 2, shared
        const uint32_t sh = (uint32_t)(s >> 32);
        const uint32_t sl = (uint32_t)s ^ (g.k1 + 2u * kPhiloxW1);
#pragma unroll
        for (int r = 0; r < kT; ++r) {
            uint64_t p0 = (uint64_t)kPhiloxM0 * (hz[r] ^ yk);           // round 3
            uint64_t p1 = (uint64_t)kPhiloxM1 * (sh ^ lx[r]);
            uint32_t x = (uint32_t)(p1 >> 32) ^ lz[r], y = (uint32_t)p1;
            uint32_t z = (uint32_t)(p0 >> 32) ^ sl, w = (uint32_t)p0;
#pragma unroll
            for (int q = 0; q < 6; ++q) {                               // rounds 4 .. 9
                p0 = (uint64_t)kPhiloxM0 * x;
                p1 = (uint64_t)kPhiloxM1 * z;
                x = xor3_vvv((uint32_t)(p1 >> 32), y, key.a[q]);
                y = (uint32_t)p1;
                z = xor3_vvv((uint32_t)(p0 >> 32), w, key.b[q]);
                w = (uint32_t)p0;
            }
            p0 = (uint64_t)kPhiloxM0 * x;                               // round 10
            p1 = (uint64_t)kPhiloxM1 * z;
            nw[r][0] = xnor3_vvv((uint32_t)(p1 >> 32), y, key.a[6]);
            nw[r][1] = ~(uint32_t)p1;
            nw[r][2] = xnor3_vvv((uint32_t)(p0 >> 32), w, key.b[6]);
            nw[r][3] = ~(uint32_t)p0;
        }
    }
};

// Stage a whole slab (64 rows x 32 k, all inside the matrix, aligned rows)
// with one 8-byte load per thread, A scaled by 2^96, B plain.  KC: k is
// contiguous in memory (element (r, k) at p[r * ld + k]); otherwise the row
// index is.
template <bool IS_A, bool KC>
__device__ __forceinline__ void stage_fast(const uint8_t* __restrict__ p, int64_t ld, int r0,
                                           int k0, float (*X)[kPitch], int tid) {
    uint32_t w[2];
    float f[8];
    int r, kq, k, rq;
    if (KC) {
        r = tid / (kBK / 8), kq = (tid % (kBK / 8)) * 8;
        const uint2 v = *reinterpret_cast<const uint2*>(p + (int64_t)(r0 + r) * ld + k0 + kq);
        w[0] = v.x, w[1] = v.y;
    } else {
        k = tid / (kBM / 8), rq = (tid % (kBM / 8)) * 8;
        const uint2 v = *reinterpret_cast<const uint2*>(p + (int64_t)(k0 + k) * ld + r0 + rq);
        w[0] = v.x, w[1] = v.y;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t c = (w[e / 4] >> (8 * (e % 4))) & 0xFFu;
        f[e] = IS_A ? fp8_to_f32<96>(c) : fp8_to_f32<0>(c);
    }
    if (KC) {
#pragma unroll
        for (int e = 0; e < 8; ++e) X[kq + e][r] = f[e];
    } else {
        *reinterpret_cast<float4*>(&X[k][rq]) = make_float4(f[0], f[1], f[2], f[3]);
        *reinterpret_cast<float4*>(&X[k][rq + 4]) = make_float4(f[4], f[5], f[6], f[7]);
    }
}

// One launch of the persistent plan: workgroup w takes whole tiles w, w + G,
// ..., then its range of the shared tile-chunks.
template <bool TA, bool TB, int WPE>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(WPE)))
void chunk_gemm_sr_kernel(TileArgs g, Plan p) {
    const uint8_t* __restrict__ A = g.A;
    const uint8_t* __restrict__ B = g.B;
    __shared__ __attribute__((aligned(16))) float As[kBK][kPitch];
    __shared__ __attribute__((aligned(16))) float Bs[kBK][kPitch];
    const int tid = threadIdx.x;
    const int tx = tid % kTiles, ty = tid / kTiles;
    const LateKeys keys(g);

    // chunks [c0, c1) of tile; lt >= 0 for a shared tile
    auto piece = [&](int64_t tile, int c0, int c1, int64_t lt) __attribute__((always_inline)) {
        int tr, tc;
        tile_rc(p, tile, tr, tc);
        const int m0 = tr * kBM;
        const int n0 = tc * kBN;
        const int kbeg = (int)((int64_t)c0 * g.CL);
        const int64_t kend64 = (int64_t)c1 * g.CL;
        const int kend = kend64 < g.K ? (int)kend64 : g.K;
        const bool to_ws = c0 > 0;
        const uint32_t gi = (uint32_t)(m0 + ty * kT), gj = (uint32_t)(n0 + tx * kT);
        const RowBits bits(gi, gj >> 2, g);
        float P[kT][kT], S[kT][kT];
#pragma unroll
        for (int r = 0; r < kT; ++r)
#pragma unroll
            for (int c = 0; c < kT; ++c) P[r][c] = S[r][c] = 0.0f;
        int chunk = c0;
        int64_t cend = (int64_t)(c0 + 1) * g.CL;
        if (cend > g.K) cend = g.K;

        auto chunk_end = [&]() __attribute__((always_inline)) {
            if (to_ws) {
                uint16_t* dst = g.ws + (lt * p.nch + chunk) * (int64_t)(kBM * kBN) +
                                (ty * kT) * kBN + tx * kT;
#pragma unroll
                for (int r = 0; r < kT; ++r) {
                    uint2 v;
                    v.x = (uint32_t)f32s_to_fp16(P[r][0]) | ((uint32_t)f32s_to_fp16(P[r][1]) << 16);
                    v.y = (uint32_t)f32s_to_fp16(P[r][2]) | ((uint32_t)f32s_to_fp16(P[r][3]) << 16);
                    *reinterpret_cast<uint2*>(dst + r * kBN) = v;
                }
            } else {
                // uniforms 4 (tx mod 2) + c of block (i, j / 8, chunk)
                const bool odd = tx & 1;
#pragma unroll
                for (int r = 0; r < kT; ++r) {
                    const u32x4 b = block_of(gi + r, gj >> 3, (uint32_t)chunk, g.w3 + 1u, g);
                    const uint32_t w0 = ~(odd ? b.z : b.x), w1 = ~(odd ? b.w : b.y);
#pragma unroll
                    for (int c = 0; c < kT; ++c)
                        S[r][c] = sr16s(S[r][c] + P[r][c], sr_addend(c < 2 ? w0 : w1, c % 2));
                }
            }
#pragma unroll
            for (int r = 0; r < kT; ++r)
#pragma unroll
                for (int c = 0; c < kT; ++c) P[r][c] = 0.0f;
            ++chunk;
            cend += g.CL;
            if (cend > g.K) cend = g.K;
        };

        for (int sb = kbeg & ~(kBK - 1); sb < kend; sb += kBK) {
            const int lo = sb > kbeg ? sb : kbeg;
            const int hi = sb + kBK < kend ? sb + kBK : kend;
            __syncthreads();               // the previous slab is consumed
            // stage op(A)[m0.., lo..hi) and op(B)[lo..hi), n0..) as floats;
            // rows, columns and k outside are zero (two codes at a time: with
            // all eight in flight four waves per SIMD spilled up to 96
            // registers, 832 x 3488 x 16: 29.9 us against 21.4)
            if (lo == sb && hi == sb + kBK && m0 + kBM <= g.M && g.a_vec) {
                stage_fast<true, !TA>(A, g.lda, m0, sb, As, tid);
            } else {
#pragma unroll 2
                for (int q = 0; q < kBM * kBK / kNT; ++q) {
                    const int e = tid + kNT * q;
                    int mm, kk;
                    if (TA) { kk = e / kBM; mm = e % kBM; } else { mm = e / kBK; kk = e % kBK; }
                    const int m = m0 + mm, k = sb + kk;
                    uint32_t code = 0;
                    if (m < g.M && k >= lo && k < hi)
                        code = TA ? A[(int64_t)k * g.lda + m] : A[(int64_t)m * g.lda + k];
                    As[kk][mm] = fp8_to_f32<96>(code);
                }
            }
            if (lo == sb && hi == sb + kBK && n0 + kBN <= g.N && g.b_vec) {
                stage_fast<false, TB>(B, g.ldb, n0, sb, Bs, tid);
            } else {
#pragma unroll 2
                for (int q = 0; q < kBN * kBK / kNT; ++q) {
                    const int e = tid + kNT * q;
                    int nn, kk;
                    if (TB) { nn = e / kBK; kk = e % kBK; } else { kk = e / kBN; nn = e % kBN; }
                    const int n = n0 + nn, k = sb + kk;
                    uint32_t code = 0;
                    if (n < g.N && k >= lo && k < hi)
                        code = TB ? B[(int64_t)n * g.ldb + k] : B[(int64_t)k * g.ldb + n];
                    Bs[kk][nn] = fp8_to_f32<0>(code);
                }
            }
            __syncthreads();
            // up to the chunk's end or the slab's: two k per set of blocks (the
            // chunk end outside that loop: inside it, its registers kept the
            // kernel at two waves per SIMD)
            for (int kseg = lo; kseg < hi;) {
                const int kstop = cend < hi ? (int)cend : hi;
                auto product = [&](int k, auto round) __attribute__((always_inline)) {
                    const float4 a4 = *reinterpret_cast<const float4*>(&As[k - sb][ty * kT]);
                    const float4 b4 = *reinterpret_cast<const float4*>(&Bs[k - sb][tx * kT]);
                    const float av[4] = {a4.x, a4.y, a4.z, a4.w};
                    const float bv[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                    for (int r = 0; r < kT; ++r)
#pragma unroll
                        for (int c = 0; c < kT; ++c)
                            P[r][c] = round(__builtin_fmaf(av[r], bv[c], P[r][c]), r, c);
                };
                // A chunk's first product goes into +0: an FP16 value, which no
                // uniform changes.  On an odd k, or as the whole chunk, it is
                // taken without blocks, so that a pair of k cut by a chunk's end
                // draws them once (otherwise twice: 203 x 1065 x 2674, CL 1,
                // 3089 us against 2065).
                if (kseg == (int64_t)chunk * g.CL && ((kseg & 1) || kstop == kseg + 1)) {
                    product(kseg, [](float x, int, int) __attribute__((always_inline)) { return x; });
                    ++kseg;
                }
#pragma unroll 1
                for (int gq = kseg; gq < kstop; gq += 2) {
                    // rows' blocks for k = gq (even), gq + 1 (complemented words)
                    uint32_t nw[kT][4];
                    bits.blocks((uint32_t)(gq >> 1), keys, g, nw);
                    product(gq, [&](float x, int r, int c) __attribute__((always_inline)) {
                        return sr16s(x, sr_addend(nw[r][c / 2], c % 2));
                    });
                    if (gq + 1 < kstop)
                        product(gq + 1, [&](float x, int r, int c) __attribute__((always_inline)) {
                            return sr16s(x, sr_addend(nw[r][2 + c / 2], c % 2));
                        });
                }
                kseg = kstop;
                if (kstop == cend) chunk_end();
            }
        }
        if (to_ws) return;
        // the running sum: the result of a whole tile, or the start of a
        // shared tile's chain (continued by chunk_fold_sr)
#pragma unroll
        for (int r = 0; r < kT; ++r) {
            const int m = m0 + ty * kT + r, n = n0 + tx * kT;
            if (m >= g.M) continue;
            uint16_t* cp = g.C + (int64_t)m * g.ldc + n;
            if (g.c_vec && n + kT <= g.N) {
                uint2 v;
                v.x = (uint32_t)f32s_to_fp16(S[r][0]) | ((uint32_t)f32s_to_fp16(S[r][1]) << 16);
                v.y = (uint32_t)f32s_to_fp16(S[r][2]) | ((uint32_t)f32s_to_fp16(S[r][3]) << 16);
                *reinterpret_cast<uint2*>(cp) = v;
            } else {
#pragma unroll
                for (int c = 0; c < kT; ++c)
                    if (n + c < g.N) cp[c] = f32s_to_fp16(S[r][c]);
            }
        }
    };

    const int w = blockIdx.x;
    for (int64_t t = w; t < p.t_whole; t += p.G) piece(whole_tile(p, t), 0, p.nch, -1);
    if (p.L > 0) {
        int64_t s = (int64_t)w * p.L / p.G;
        const int64_t e = (int64_t)(w + 1) * p.L / p.G;
        while (s < e) {
            const int64_t lt = s / p.nch;
            const int c0 = (int)(s - lt * p.nch);
            const int64_t c1l = e - lt * p.nch;
            const int c1 = c1l < p.nch ? (int)c1l : p.nch;
            piece(p.t_whole + lt, c0, c1, lt);
            s = lt * p.nch + c1;
        }
    }
}

// Continue the running sums of the shared tiles (in C, from their first
// pieces) over the chunk sums in the workspace, in ascending chunk order --
// the additions a whole-tile pass makes, with the same inter-chunk uniforms.
// A thread takes 4 consecutive outputs of a row: one 8-byte load of chunk
// sums and half of a block of uniforms per chunk (with the block's 8 outputs a
// thread, 512 x 512 outputs are half a wave per SIMD and the blocks' latency
// stands alone).
constexpr int kFoldV = 4, kFoldTU = 8, kFoldT = 64;

__global__ __launch_bounds__(kFoldT) void chunk_fold_sr(TileArgs g, Plan p) {
    const int64_t per = (int64_t)kBM * kBN;
    const int64_t idx = ((int64_t)blockIdx.x * kFoldT + threadIdx.x) * kFoldV;
    const int64_t lt = idx / per;
    if (lt * p.nch >= p.L) return;
    const int local = (int)(idx - lt * per);
    const int64_t tile = p.t_whole + lt;
    int tr, tc;
    tile_rc(p, tile, tr, tc);
    const int m = tr * kBM + local / kBN;
    const int n0 = tc * kBN + local % kBN;
    if (m >= g.M || n0 >= g.N) return;
    const int a = first_piece_end(p, lt);
    if (a >= p.nch) return;
    const int nv = min(kFoldV, g.N - n0);
    uint16_t* cp = g.C + (int64_t)m * g.ldc + n0;
    float S[kFoldV];
#pragma unroll
    for (int v = 0; v < kFoldV; ++v) S[v] = v < nv ? fp16_to_f32s(cp[v]) : 0.0f;
    const uint2* src = reinterpret_cast<const uint2*>(g.ws + lt * p.nch * per + local);
    const int64_t step = per / kFoldV;
    const PhiloxKeys keys(g.k0, g.k1);
    const bool odd = (n0 >> 2) & 1;               // the block's second four uniforms
    auto add = [&](const uint2& q, int c) __attribute__((always_inline)) {
        const uint32_t cw[2] = {q.x, q.y};
        const u32x4 b = philox4x32_10(
            {(uint32_t)m, (uint32_t)(n0 >> 3), (uint32_t)c, g.w3 + 1u}, keys);
        const uint32_t nw[2] = {~(odd ? b.z : b.x), ~(odd ? b.w : b.y)};
#pragma unroll
        for (int v = 0; v < kFoldV; ++v) {
            const float x = S[v] + fp16_to_f32s((cw[v / 2] >> (16 * (v % 2))) & 0xFFFFu);
            S[v] = sr16s(x, sr_addend(nw[v / 2], v % 2));
        }
    };
    // Batches of kFoldTU chunk loads, the next batch in flight while one is
    // added; every batch load is unconditional (indices clamped to the last
    // chunk, the extra values never added) so the compiler waits for the
    // older batch only.
    const int last = p.nch - 1;
    auto load = [&](uint2 (&q)[kFoldTU], int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kFoldTU; ++u) q[u] = src[(int64_t)min(c0 + u, last) * step];
    };
    auto fold = [&](const uint2 (&q)[kFoldTU], int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kFoldTU; ++u)
            if (c0 + u < p.nch) add(q[u], c0 + u);
    };
    uint2 q0[kFoldTU], q1[kFoldTU];
    int c = a;
    load(q0, c);
    for (;;) {
        if (c + kFoldTU >= p.nch) {
            fold(q0, c);
            break;
        }
        load(q1, c + kFoldTU);
        fold(q0, c);
        c += kFoldTU;
        if (c + kFoldTU >= p.nch) {
            fold(q1, c);
            break;
        }
        load(q0, c + kFoldTU);
        fold(q1, c);
        c += kFoldTU;
    }
#pragma unroll
    for (int v = 0; v < kFoldV; ++v)
        if (v < nv) cp[v] = f32s_to_fp16(S[v]);
}

__global__ void fill_zero16(uint16_t* __restrict__ C, int64_t ldc, int M, int N) {
    const int64_t total = (int64_t)M * N;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += step)
        C[(i / N) * ldc + i % N] = 0;
}

template <int WPE>
const void* tile_kernel(int ta, int tb) {
    if (!ta && !tb) return reinterpret_cast<const void*>(&chunk_gemm_sr_kernel<false, false, WPE>);
    if (!ta && tb) return reinterpret_cast<const void*>(&chunk_gemm_sr_kernel<false, true, WPE>);
    if (ta && !tb) return reinterpret_cast<const void*>(&chunk_gemm_sr_kernel<true, false, WPE>);
    return reinterpret_cast<const void*>(&chunk_gemm_sr_kernel<true, true, WPE>);
}

struct TilePlan {
    Plan plan{};
    size_t ws_bytes = 0;
    bool ok = false;
};

// Time of a plan's parts in microseconds, fitted to calls of 1 .. 2060 tiles, K
// 16 .. 16000 and CL 1 .. 500, as whole tiles and shared out over two and four
// workgroups per CU (8% root mean square): one k of a tile with r workgroups on
// its CU, a chunk's end, and the fold pass (launch, each chunk of an output's
// chain, and a million chunk sums).
constexpr double kTileUsPerK[5] = {0.0, 0.365, 0.51, 0.72, 0.895};
constexpr double kTileUsPerChunk = 0.23;
constexpr double kTileFoldUs = 7.0, kTileFoldUsPerChunk = 0.36, kTileFoldUsPerMillion = 0.52;

// r workgroups per CU, each `chunks` chunks of CL (one after the other)
double tile_us(int64_t r, double chunks, int64_t CL) {
    if (r > 4) r = 4;
    return chunks * ((double)CL * kTileUsPerK[r] + (double)r * kTileUsPerChunk);
}

// Whole tiles, or (with a workspace allowed) the chunks of the tiles that do
// not divide evenly over the slots shared out, every workgroup then ending
// with the same number of chunks: over four workgroups per CU, or over two,
// the kernel's two register budgets.  Four resident waves per SIMD round about
// 10% more products a second than two (1000 tiles of K 512: 503 us against 553),
// but a call of few chunks loses more to the fold pass and to workgroups with a
// chunk each (K 65, CL 64: 512 tiles whole 43 us, shared over four 80; 468 tiles
// 44 / 79, over two 57), hence the estimate.
TilePlan plan_tile(const void* fn, int64_t M, int64_t N, int64_t K, int64_t CL, bool allow_ws) {
    TilePlan r;
    const int cus = device_cus();
    int occ = kernel_occupancy(fn, kNT, current_device());
    if (cus <= 0 || occ <= 0) return r;
    if (occ > 4) occ = 4;
    const int force_g = env_int("FP8T_GEMM_WGS", 0);
    const int force_split = env_int("FP8T_GEMM_SPLIT", -1);
    const int64_t tiles_m = (M + kBM - 1) / kBM, tiles_n = (N + kBN - 1) / kBN;
    const int64_t T = tiles_m * tiles_n;
    const int64_t nch = (K + CL - 1) / CL;
    auto slots = [&](int per_cu) {
        const int64_t g = (int64_t)cus * per_cu;
        return force_g > 0 && force_g < g ? (int64_t)force_g : g;
    };
    Plan& p = r.plan;
    p.tiles_n = tiles_n;
    p.nch = (int)nch;
    p.t_whole = T;
    p.L = 0;
    p.G = (int)(T < slots(occ) ? T : slots(occ));
    // rounds of `occ` tiles per CU, then the rest
    const int64_t per_cu = (T + cus - 1) / cus;
    const double tile_chunks = (double)K / (double)CL;
    double est = (double)(per_cu / occ) * tile_us(occ, tile_chunks, CL) +
                 (per_cu % occ ? tile_us(per_cu % occ, tile_chunks, CL) : 0.0);
    for (int wgs : {occ, 2}) {
        const int64_t g = slots(wgs), q = T / g;
        // with many rounds the last, partly idle one costs little
        if (!allow_ws || force_split == 0 || nch == 1 || T % g == 0 ||
            (q >= 4 && force_split != 1))
            continue;
        Plan c{};
        c.tiles_n = tiles_n;
        c.nch = (int)nch;
        c.G = (int)(g < T * nch ? g : T * nch);
        c.t_whole = (T / c.G) * c.G;
        c.L = (T - c.t_whole) * nch;
        if (c.L == 0) continue;
        const double sums = (double)c.L * kBM * kBN;
        const double e = tile_us((c.G + cus - 1) / cus,
                                 (double)(T / c.G) * tile_chunks + (double)((c.L + c.G - 1) / c.G),
                                 CL) + kTileFoldUs + kTileFoldUsPerChunk * (double)nch +
                         kTileFoldUsPerMillion * sums * 1e-6;
        if (e >= est && !(force_split == 1 && p.L == 0)) continue;
        est = e;
        p = c;
        r.ws_bytes = (size_t)c.L * kBM * kBN * sizeof(uint16_t) + kWsAlign;
    }
    p.xcd_remap = p.t_whole % 8 == 0 && p.G % 8 == 0;
    if (env_int("FP8T_GEMM_VERBOSE", 0))
        fprintf(stderr, "[fp8t tile plan] occ %d G %d T %lld t_whole %lld L %lld ws %zu est %.1f us\n",
                occ, p.G, (long long)T, (long long)p.t_whole, (long long)p.L, r.ws_bytes, est);
    r.ok = true;
    return r;
}

bool tile_args_ok(int ta, int tb, int64_t M, int64_t N, int64_t K, int64_t CL) {
    if (M < 0 || N < 0 || K < 0 || CL < 1) return false;
    if ((ta != 0 && ta != 1) || (tb != 0 && tb != 1)) return false;
    // 32-bit indices inside the kernel (k also runs one slab past K)
    return M <= kMaxGemmDim && N <= kMaxGemmDim && K <= kMaxGemmDim;
}

// Validation, K = 0, planning and launch.
int tile_call(int ta, int tb, int64_t M, int64_t N, int64_t K, int64_t CL, const uint8_t* A,
              int64_t lda, const uint8_t* B, int64_t ldb, uint16_t* C, int64_t ldc, uint64_t seed,
              uint64_t offset, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (!tile_args_ok(ta, tb, M, N, K, CL)) return FP8T_EINVAL;
    if (M == 0 || N == 0) return FP8T_OK;
    if (!C || ldc < N) return FP8T_EINVAL;
    if (K > 0) {
        if (!A || !B) return FP8T_EINVAL;
        if (lda < (ta ? M : K) || ldb < (tb ? K : N)) return FP8T_EINVAL;
    }
    if (workspace_bytes > 0 && !workspace) return FP8T_EINVAL;
    if (K == 0) {
        const int64_t total = M * N;
        hipLaunchKernelGGL(fill_zero16, dim3(stride_blocks(total, 256)), dim3(256), 0,
                           stream, C, ldc, (int)M, (int)N);
        return launch_status();
    }
    if (CL > K) CL = K;
    const void* fn = tile_kernel<4>(ta, tb);
    const TilePlan tp = plan_tile(fn, M, N, K, CL, workspace_bytes > 0);
    if (!tp.ok) return FP8T_EHIP;
    if (tp.ws_bytes > workspace_bytes) return FP8T_EWORKSPACE;
    TileArgs g{};
    g.A = A;
    g.B = B;
    g.C = C;
    if (tp.plan.L > 0)
        g.ws = reinterpret_cast<uint16_t*>(((uintptr_t)workspace + kWsAlign - 1) &
                                           ~(uintptr_t)(kWsAlign - 1));
    g.lda = lda;
    g.ldb = ldb;
    g.ldc = ldc;
    g.M = (int)M;
    g.N = (int)N;
    g.K = (int)K;
    g.CL = (int)CL;
    g.k0 = (uint32_t)seed;
    g.k1 = (uint32_t)(seed >> 32);
    g.w3 = 2u * (uint32_t)offset;
    g.c_vec = aligned(C, 8) && ldc % 4 == 0;
    g.a_vec = aligned(A, 8) && lda % 8 == 0;
    g.b_vec = aligned(B, 8) && ldb % 8 == 0;
    Plan plan = tp.plan;
    // two workgroups per CU or fewer: the registers of four waves per SIMD are
    // not needed, and with twice as many nothing is spilled and the blocks of a
    // thread's rows overlap more (93 x 2043 x 2781: 1270 -> 1105 us; 16 x 16 x
    // 16: 13.4 -> 11.4)
    if (plan.G <= 2 * device_cus()) fn = tile_kernel<2>(ta, tb);
    void* args[] = {&g, &plan};
    if (hipLaunchKernel(fn, dim3(plan.G), dim3(kNT), args, 0, stream) != hipSuccess)
        return FP8T_EHIP;
    if (plan.L > 0) {
        const int64_t threads = (plan.L / plan.nch) * kBM * kBN / kFoldV;
        hipLaunchKernelGGL(chunk_fold_sr, dim3((unsigned)((threads + kFoldT - 1) / kFoldT)),
                           dim3(kFoldT), 0, stream, g, plan);
    }
    return launch_status();
}

size_t tile_workspace(int ta, int tb, int64_t M, int64_t N, int64_t K, int64_t CL) {
    if (!tile_args_ok(ta, tb, M, N, K, CL)) return 0;
    if (M == 0 || N == 0 || K == 0) return 0;
    const TilePlan tp = plan_tile(tile_kernel<4>(ta, tb), M, N, K, CL > K ? K : CL, true);
    return tp.ok ? tp.ws_bytes : 0;
}

}  // namespace
}  // namespace fp8t

using namespace fp8t;

extern "C" size_t chunk_gemm_sr_workspace_size(int trans_a, int trans_b, int64_t M, int64_t N,
                                               int64_t K, int64_t CL) {
    return tile_workspace(trans_a, trans_b, M, N, K, CL);
}

extern "C" int chunk_gemm_sr(int trans_a, int trans_b, int64_t M, int64_t N, int64_t K,
                             int64_t CL, const uint8_t* A, int64_t lda, const uint8_t* B,
                             int64_t ldb, uint16_t* C, int64_t ldc, uint64_t seed,
                             uint64_t offset, void* workspace, size_t workspace_bytes,
                             hipStream_t stream) {
    if (offset >= 0x80000000ull) return FP8T_EINVAL;
    return tile_call(trans_a, trans_b, M, N, K, CL, A, lda, B, ldb, C, ldc, seed, offset,
                     workspace, workspace_bytes, stream);
}
