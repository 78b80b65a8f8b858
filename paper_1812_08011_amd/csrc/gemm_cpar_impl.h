// chunk_gemm on the vector ALUs, a chunk per wave: the exact mode for GEMMs
// whose outputs alone do not fill the chip evenly.
//
// The arithmetic and its two paths (guarded, safe) are those of
// chunk_gemm_valu (gemm_valu_impl.h).  What differs is who does what.  The
// chunks of a dot product are independent until their sums are added, in
// order, into the running sum (Sec. 2.3), so
//   * a workgroup owns a small tile (8 T x 8 T outputs) and its NW waves take
//     NW consecutive chunks of it at a time: each wave stages its own chunk's
//     operands in LDS of its own (decoded to FP32, no workgroup barrier) and
//     forms the chunk's sums of the whole tile, T x T per lane;
//   * the waves leave their chunk sums in LDS, and after a barrier every
//     thread adds the NW sums of its outputs into their running sums in
//     ascending chunk order -- the additions of a whole-tile pass, so the
//     same bits.
// So a GEMM of few outputs fills the chip without writing its chunk sums to
// memory and without a second kernel: 512 x 512 outputs are 256 tiles of 32 x
// 32, one per CU, with 16 waves each.  The exchange costs a barrier pair and NW
// three-instruction additions per thread against 3 CL T^2 instructions of a
// wave's chunk.
// Operands are read 8 codes per lane and load at any alignment; a wave's two
// LDS buffers let it stage the next slab before it computes on the current one
// (with one buffer and slabs twice as long the staging latency stood between
// them: 512 x 512 x 16384 262 us against 249).
// Bound by the vector ALUs (3 instructions per multiply-accumulate); the
// staging of a 32 x 32 tile adds about 5% to them, LDS reads take a third of
// the LDS's cycles, the exchange about 4% of a round of 16 waves.  Measured
// against the kernels before it (microseconds): 128 x 128 x 1024 13.1 -> 9.7,
// 256 x 1024 x 1024 26.2 -> 20.0, 1024 x 1024 x 256 24.1 -> 20.0, 2304 x 256 x
// 50176 1727 -> 1680; for GEMMs with many outputs the 64 x 128 tiles, which
// stage less per product, stay faster (50176 x 256 x 2304: 1461 against 1676).
#pragma once

#include "gemm_valu_impl.h"

namespace fp8t {
namespace cpar {

using valu_impl::wave_reduce;

constexpr int kCodes = 8;                  // codes per lane and operand slab

// Orders a wave's LDS accesses across its lanes (the LDS executes one wave's
// instructions in order; the fences keep the compiler from moving accesses).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Position of a lane's 8 codes in a slab of R rows x BK k: KC (k contiguous
// in memory): 8 k of one row; else 8 rows at one k.
template <bool KC, int R, int BK>
__device__ __forceinline__ void slab_pos(int lane, int& r, int& k) {
    static_assert(R * BK == 64 * kCodes, "one 8-byte load per lane");
    if (KC) { r = lane / (BK / kCodes); k = (lane % (BK / kCodes)) * kCodes; }
    else    { k = lane / (R / kCodes);  r = (lane % (R / kCodes)) * kCodes; }
}

// A lane's 8 codes as loaded: 8 bytes (FP8) or 16 (FP16).
typedef unsigned __int128 codes16_t;
template <bool P16> using codes_of = typename std::conditional<P16, codes16_t, uint64_t>::type;

// Codes pos .. pos + 7 of a contiguous run of `lim` (>= 8) codes at `base`:
// one load at any alignment (global memory takes unaligned vector
// loads here, so odd leading dimensions are read as wide as aligned ones).  A
// piece that reaches past the run's end is loaded from the run's last 8 codes
// and moved down by `drop` codes when it is staged (8: nothing is left).
template <typename Codes>
__device__ __forceinline__ void load_codes(const uint8_t* __restrict__ base, int pos, int lim,
                                           bool valid, Codes& v, int& drop) {
    constexpr int EB = sizeof(Codes) / kCodes;
    const int start = min(pos, lim - kCodes);
    __builtin_memcpy(&v, base + (int64_t)start * EB, sizeof(Codes));
    drop = valid ? min(pos - start, kCodes) : kCodes;
}
// The 8 codes moved down by `drop` codes, zeros after them.
template <typename Codes>
__device__ __forceinline__ Codes drop_codes(Codes v, int drop) {
    return drop >= kCodes ? (Codes)0 : v >> (int)(sizeof(Codes) * drop);
}

// Decode a lane's 8 codes into the wave's slab [k][row] (pitch floats per
// k), values times 2^SH; TRACK keeps the largest magnitude, NaN and Inf
// included (the maximum propagates NaN).
template <bool KC, int R, int BK, int SH, bool TRACK>
__device__ __forceinline__ void stage(float* lds, int pitch, int lane, uint64_t codes,
                                      float& amax) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    int r, k;
    slab_pos<KC, R, BK>(lane, r, k);
    const uint32_t v[2] = {(uint32_t)codes, (uint32_t)(codes >> 32)};
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const v2f lo = __builtin_amdgcn_cvt_pk_f32_bf8((int)v[w], false);
        const v2f hi = __builtin_amdgcn_cvt_pk_f32_bf8((int)v[w], true);
        float f[4] = {lo.x, lo.y, hi.x, hi.y};
        if (TRACK) {
            amax = maximum3_abs(amax, f[0], f[1]);
            amax = maximum3_abs(amax, f[2], f[3]);
        }
        if (SH != 0) {
#pragma unroll
            for (int b = 0; b < 4; ++b) f[b] *= __builtin_ldexpf(1.0f, SH);   // exact
        }
        if (KC) {
#pragma unroll
            for (int b = 0; b < 4; ++b) lds[(k + 4 * w + b) * pitch + r] = f[b];
        } else {
            *reinterpret_cast<float4*>(&lds[k * pitch + r + 4 * w]) =
                make_float4(f[0], f[1], f[2], f[3]);
        }
    }
}

// ---- FP16 operands (chunk_gemm_p16): products rounded to FP16 -----------------
//
// The guarded path holds FP16 quantities scaled by 2^-110 (kP16Dom): FP16's
// smallest step 2^-39 is then FP32's 2^-149 and FP16's smallest normal 2^-30
// the point where x (2^14 - 1) leaves FP32's normal range, so gradual
// underflow comes with the FP32 operations.  With a scaled by 2^-55 and b by
// 2^14 2^-55 (b14), bs = b14 (2^-14 - 1) -- exact, b having at most 10
// significant bits --, a product x = a b is rounded to FP16 by
//   s = RN(a bs) = RN(x (1 - 2^14)),  hi = fma(a, b14, s),
// the two-step rounding of rn16v with the product's multiplication folded in:
// x (1 - 2^14) is rounded once from its exact value, to FP32's 24 bits or, where
// |x| < 2^-30, to multiples of 2^-149, the fixed step of FP16's subnormals.
// hi is exact as long as 2^14 x is a multiple of 2^-39, which holds for every
// |x| >= 2^-34 (its last bit is at least 2^-53).  A slab that may hold a
// smaller nonzero product -- the smallest |a| times the smallest |b| of the
// wave's slab tells -- rounds its products by the clamped magic-number add
// (rn16_product) instead.  Five instructions per multiply-accumulate against
// seven with Veltkamp splitting and a per-k bound on the products from 2^-30.
// Measured, last layer of a 1024 -> 6000 network at batch 256: Forward 248 ->
// 164 us, Backward 250 -> 181, Gradient 211 -> 182 (128 x 64 tiles with shared
// chunks before).
constexpr int kP16Dom = -110;

// Value times 2^-96 of a finite code in bits 16-31 / 0-15 of w (an Inf or NaN
// code comes out as 2^32 2^-96 or more, which fails the guard): the code's
// fields moved into FP32's, its subnormals onto FP32's.
__device__ __forceinline__ float code_hi(uint32_t w) {
    return __uint_as_float((uint32_t)((int32_t)w >> 2) & 0x9FFFC000u);
}
__device__ __forceinline__ float code_lo(uint32_t w) { return code_hi(w << 16); }

// Decode a lane's 8 FP16 codes into the wave's slab, values times 2^SH (SAFE:
// Inf and NaN kept); TRACK keeps the largest magnitude (of the scaled values)
// and returns the wave's smallest nonzero magnitude code less one (65535:
// none).
template <bool KC, int R, int BK, int SH, bool TRACK>
__device__ __forceinline__ uint32_t stage16(float* lds, int pitch, int lane, codes16_t codes,
                                            float& amax) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    int r, k;
    slab_pos<KC, R, BK>(lane, r, k);
    us2 key = {0xFFFFu, 0xFFFFu};
    float f[kCodes];
#pragma unroll
    for (int w = 0; w < kCodes / 2; ++w) {
        const uint32_t v = (uint32_t)(codes >> (32 * w));
        if (TRACK) {
            f[2 * w] = code_lo(v) * __builtin_ldexpf(1.0f, 96 + SH);
            f[2 * w + 1] = code_hi(v) * __builtin_ldexpf(1.0f, 96 + SH);
            amax = max3_abs(amax, f[2 * w], f[2 * w + 1]);
            const uint32_t m = v & 0x7FFF7FFFu;
            us2 c;
            __builtin_memcpy(&c, &m, 4);
            key = __builtin_elementwise_min(key, (us2)(c - (us2){1, 1}));
        } else {
            f[2 * w] = fp16_to_f32_pow2<SH>(v & 0xFFFFu);
            f[2 * w + 1] = fp16_to_f32_pow2<SH>(v >> 16);
        }
    }
    if (KC) {
#pragma unroll
        for (int b = 0; b < kCodes; ++b) lds[(k + b) * pitch + r] = f[b];
    } else {
#pragma unroll
        for (int b = 0; b < kCodes; b += 4)
            *reinterpret_cast<float4*>(&lds[k * pitch + r + b]) =
                make_float4(f[b], f[b + 1], f[b + 2], f[b + 3]);
    }
    if (!TRACK) return 0;
    auto umin = [](uint32_t x, uint32_t y) __attribute__((always_inline)) { return min(x, y); };
    return wave_reduce(min((uint32_t)key.x, (uint32_t)key.y), umin);
}

// Whether every nonzero product of magnitudes with these smallest keys is at
// least 2^-34.
__device__ __forceinline__ bool products_ok(uint32_t ka, uint32_t kb) {
    const float a = __uint_as_float((ka + 1) << 14), b = __uint_as_float((kb + 1) << 14);
    return ka == 0xFFFFu || kb == 0xFFFFu || (a * 0x1p96f) * (b * 0x1p96f) >= 0x1p-34f;
}

template <int T> struct Tile {
    static constexpr int B = 8 * T;                       // tile edge
    static constexpr int BK = 64 * kCodes / B;            // k per slab
    // padded pitches (floats) keep the transposing stores of a k-contiguous
    // operand off each other's banks
    static constexpr int PKC = B + T, PRC = B;
};

template <int T, int NW, bool TA, bool TB, bool P16>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4)))
void chunk_gemm_cpar(GemmArgs g, Plan p) {
    constexpr int B = Tile<T>::B, BK = Tile<T>::BK;
    constexpr bool KCA = !TA, KCB = TB;
    constexpr int PA = KCA ? Tile<T>::PKC : Tile<T>::PRC;
    constexpr int PB = KCB ? Tile<T>::PKC : Tile<T>::PRC;
    // floats of one of a wave's two LDS buffers: a slab of both operands, or
    // (in the buffer of a chunk's last slab) the chunk's sums
    constexpr int RS = BK * (PA + PB) > B * B ? BK * (PA + PB) : B * B;
    constexpr int NT = 64 * NW;
    // outputs whose running sums a thread owns
    constexpr int OPT = B * B > NT ? B * B / NT : 1;

    __shared__ __attribute__((aligned(16))) float region[NW][2][RS];
    // |a| max, |b| max, |S| max of the guarded pieces, three slots in turn:
    // a piece clears the slot of the next one, whose last readers (two pieces
    // ago) have since passed a check's barrier
    __shared__ uint32_t s_track[3][3];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ly = lane >> 3, lx = lane & 7;
    int ra, ka, rb, kb;
    slab_pos<KCA, B, BK>(lane, ra, ka);
    slab_pos<KCB, B, BK>(lane, rb, kb);
    int gslot = 0;
    if (tid < 9) (&s_track[0][0])[tid] = 0;
    __syncthreads();

    typedef codes_of<P16> Codes;
    constexpr int EB = P16 ? 2 : 1;      // bytes per code
    Codes va = 0, vb = 0;                // codes of the slab fetched last
    float P[T][T];

    // One piece: chunks [c0, c1) of tile `tile` (see gemm_valu_impl.h).
    auto piece = [&](auto safe_tag, int64_t tile, int c0, int c1, int64_t lt)
                     __attribute__((always_inline)) -> bool {
        constexpr bool SAFE = decltype(safe_tag)::value;
        // value scale of the path, and of A's staged values
        constexpr int DOM = SAFE ? 96 : P16 ? kP16Dom : 0;
        constexpr bool TRACK = !SAFE;
        int tr, tc;
        tile_rc(p, tile, tr, tc);
        const int m0 = tr * B;
        const int n0 = tc * B;
        const bool to_ws = c0 > 0;
        float amax_a = 0.0f, amax_b = 0.0f, smax = 0.0f;
        auto rnd = [&](float x) __attribute__((always_inline)) -> float {
            return SAFE ? rn16s(x) : rn16v(x);
        };
        auto code = [&](float x) __attribute__((always_inline)) -> uint32_t {
            // on the FP16 grid and below 2^32 on the guarded path
            if constexpr (DOM == kP16Dom) return f32g_to_fp16(x * 0x1p110f);
            else return fp16_code<DOM>(x);
        };
        // a slab's codes at k0, 8 per lane and operand (k beyond K and rows
        // beyond the matrix read as zero; the k beyond a chunk's end are not
        // used).  A slab inside both matrices is loaded without a look at
        // their edges.
        const bool inner = m0 + B <= g.M && n0 + B <= g.N;
        bool edge = false;               // the fetched slab touches an edge
        int da = 0, db = 0;
        auto fetch = [&](int k0) __attribute__((always_inline)) {
            const int ga = k0 + ka, gb = k0 + kb;
            edge = !(inner && k0 + BK <= g.K);
            if (!edge) {
                __builtin_memcpy(&va, g.A + EB * (KCA ? (int64_t)(m0 + ra) * g.lda + ga
                                                      : (int64_t)ga * g.lda + m0 + ra),
                                 sizeof(Codes));
                __builtin_memcpy(&vb, g.B + EB * (KCB ? (int64_t)(n0 + rb) * g.ldb + gb
                                                      : (int64_t)gb * g.ldb + n0 + rb),
                                 sizeof(Codes));
            } else {
                const int ma = m0 + ra, nb = n0 + rb;
                if (KCA)
                    load_codes(g.A + EB * ((int64_t)min(ma, g.M - 1) * g.lda), ga, g.K, ma < g.M, va, da);
                else
                    load_codes(g.A + EB * ((int64_t)min(ga, g.K - 1) * g.lda), ma, g.M, ga < g.K, va, da);
                if (KCB)
                    load_codes(g.B + EB * ((int64_t)min(nb, g.N - 1) * g.ldb), gb, g.K, nb < g.N, vb, db);
                else
                    load_codes(g.B + EB * ((int64_t)min(gb, g.K - 1) * g.ldb), nb, g.N, gb < g.K, vb, db);
            }
        };
        auto read = [&](float (&a)[T], float (&b)[T], const float* buf, int q)
                        __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < T; ++i) a[i] = buf[q * PA + ly * T + i];
#pragma unroll
            for (int j = 0; j < T; ++j) b[j] = buf[BK * PA + q * PB + lx * T + j];
        };
        bool staged_ok = true;           // FP16 operands: products_ok of the slab staged last
        auto stage_slab = [&](float* buf) __attribute__((always_inline)) {
            if (edge) {
                va = drop_codes(va, da);
                vb = drop_codes(vb, db);
            }
            if constexpr (P16) {
                const uint32_t kma = stage16<KCA, B, BK, SAFE ? 48 : kP16Dom / 2, TRACK>(
                    buf, PA, lane, va, amax_a);
                const uint32_t kmb = stage16<KCB, B, BK, SAFE ? 16 : kP16Dom / 2 + 14, TRACK>(
                    buf + BK * PA, PB, lane, vb, amax_b);
                if (TRACK)
                    staged_ok = __builtin_amdgcn_readfirstlane((int)products_ok(kma, kmb)) != 0;
            } else {
                stage<KCA, B, BK, DOM, TRACK>(buf, PA, lane, va, amax_a);
                stage<KCB, B, BK, 0, TRACK>(buf + BK * PA, PB, lane, vb, amax_b);
            }
        };
        // FP16 operands: a product rounded to FP16 (see above; SPLIT: every
        // nonzero one is at least 2^-34)
        auto product = [&](auto split, float a, float b, float bs) __attribute__((always_inline)) {
            if constexpr (SAFE) return rn16_product_s(a * b) + 0.0f;
            else if constexpr (decltype(split)::value) return __builtin_fmaf(a, b, a * bs);
            else return rn16_product((a * 0x1p55f) * (b * 0x1p41f)) * 0x1p-110f + 0.0f;
        };
        auto fma_step = [&](auto split, const float (&a)[T], const float (&b)[T])
                            __attribute__((always_inline)) {
            float bs[T];
#pragma unroll
            for (int j = 0; j < T; ++j) bs[j] = P16 ? b[j] * (0x1p-14f - 1.0f) : 0.0f;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    if constexpr (P16) P[i][j] = rnd(P[i][j] + product(split, a[i], b[j], bs[j]));
                    else P[i][j] = rnd(__builtin_fmaf(a[i], b[j], P[i][j]));
                }
        };
        // a chunk's first product, rounded to FP16 if its operands are (an FP8
        // product is an FP16 value), is the chunk's sum so far
        auto first_step = [&](auto split, const float (&a)[T], const float (&b)[T])
                              __attribute__((always_inline)) {
            float bs[T];
#pragma unroll
            for (int j = 0; j < T; ++j) bs[j] = P16 ? b[j] * (0x1p-14f - 1.0f) : 0.0f;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    if constexpr (P16) P[i][j] = product(split, a[i], b[j], bs[j]);
                    else P[i][j] = __builtin_fmaf(a[i], b[j], 0.0f);
                }
        };

        float S[OPT];                      // the thread's running sums
#pragma unroll
        for (int o = 0; o < OPT; ++o) S[o] = 0.0f;

        // The wave's slabs, of its chunks c0 + wave, c0 + wave + NW, ... in
        // turn: while one is computed on, the next is staged into the other
        // buffer and the one after it is on its way from memory.
        int fc = c0 + wave;                              // chunk and k of the fetched slab
        int fk = 0, fend = 0;                            // (a chunk past the last has no k in range)
        bool more = fc < c1;
        auto chunk_end = [&](int c) __attribute__((always_inline)) {
            const int kbeg = c * g.CL;
            return g.CL < g.K - kbeg ? kbeg + g.CL : g.K;
        };
        auto fetch_next = [&]() __attribute__((always_inline)) {
            fk += BK;
            if (fk >= fend) {
                fc += NW;
                more = fc < c1;
                if (!more) return;
                fk = fc * g.CL;
                fend = chunk_end(fc);
            }
            fetch(fk);
        };
        const int ns = (g.CL + BK - 1) / BK;             // slabs of a chunk, and of the last one
        const int ns_last = (g.K - (p.nch - 1) * g.CL + BK - 1) / BK;
        int done_slabs = 0;
        int buf = 0;
        if (more) {
            fk = fc * g.CL;
            fend = chunk_end(fc);
            fetch(fk);
            stage_slab(region[wave][0]);
            fetch_next();
        }
        for (int cr = c0; cr < c1; cr += NW) {
            const int c = cr + wave;
            if (c < c1) {
                const int kbeg = c * g.CL, kend = chunk_end(c);
                for (int ks = kbeg; ks < kend; ks += BK) {
                    wave_sync();
                    const bool ok = staged_ok;
                    // a wave that stages goes before those that compute, so
                    // that it has its next slab under way while they do
                    // (1000 x 777 x 3001: 165 -> 160 us)
                    if (more) {
                        __builtin_amdgcn_s_setprio(1);
                        stage_slab(region[wave][buf ^ 1]);
                        fetch_next();
                        __builtin_amdgcn_s_setprio(0);
                    }
                    const float* const cur = region[wave][buf];
                    const int kmax = kend - ks;
                    if (kmax >= BK && (!P16 || ok)) {
                        constexpr std::true_type split{};
                        float a0[T], b0[T], a1[T], b1[T];
                        read(a0, b0, cur, 0);
#pragma unroll
                        for (int q = 0; q < BK; q += 2) {
                            read(a1, b1, cur, q + 1);
                            if (q == 0 && ks == kbeg) first_step(split, a0, b0);
                            else fma_step(split, a0, b0);
                            if (q + 2 < BK) read(a0, b0, cur, q + 2);
                            fma_step(split, a1, b1);
                        }
                    } else {
                        // a chunk's last, shorter slab, or tiny products
                        const int qn = kmax < BK ? kmax : BK;
                        for (int q = 0; q < qn; ++q) {
                            float a[T], b[T];
                            read(a, b, cur, q);
                            if (q == 0 && ks == kbeg) first_step(std::false_type{}, a, b);
                            else fma_step(std::false_type{}, a, b);
                        }
                    }
                    buf ^= 1;
                }
                wave_sync();
                if (to_ws) {
                    // chunk sums read once, by the fold pass (ws_index)
                    typedef uint32_t codes_t __attribute__((ext_vector_type(T / 2)));
#pragma unroll
                    for (int i = 0; i < T; ++i) {
                        codes_t q;
#pragma unroll
                        for (int j = 0; j < T / 2; ++j)
                            q[j] = code(P[i][2 * j]) | (code(P[i][2 * j + 1]) << 16);
                        __builtin_nontemporal_store(
                            q, reinterpret_cast<codes_t*>(
                                   g.ws + ws_index(p, B, B, lt, c, ly * T + i, lx * T)));
                    }
                } else {
                    // the chunk's sums, row-major in the buffer of its last slab
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
                            region[wave][buf ^ 1][(ly * T + i) * B + lx * T + j] = P[i][j];
                }
            }
            if (!to_ws) {
                __syncthreads();
                // a wave's buffers alternate slab by slab: its sums are in the
                // buffer of parity (slabs so far) - 1; every chunk has the same
                // slabs but the last one of the dot product
                const int n = c1 - cr < NW ? c1 - cr : NW;
                const int slot = (done_slabs + ns - 1) & 1;
                const int last = cr + n == p.nch ? (done_slabs + ns_last - 1) & 1 : slot;
                if (tid * OPT < B * B) {
                    auto add = [&](const float (&q)[OPT]) __attribute__((always_inline)) {
#pragma unroll
                        for (int o = 0; o < OPT; ++o) S[o] = rnd(S[o] + q[o]);
                        if (TRACK) {
#pragma unroll
                            for (int o = 0; o < OPT; ++o) smax = max3_abs(smax, S[o], S[o]);
                        }
                    };
                    if (n == NW) {
                        float q[NW][OPT];
#pragma unroll
                        for (int w = 0; w < NW; ++w)
#pragma unroll
                            for (int o = 0; o < OPT; ++o) q[w][o] = region[w][w == NW - 1 ? last : slot][tid * OPT + o];
#pragma unroll
                        for (int w = 0; w < NW; ++w) add(q[w]);
                    } else {
                        for (int w = 0; w < n; ++w) {
                            float q[OPT];
#pragma unroll
                            for (int o = 0; o < OPT; ++o) q[o] = region[w][w == n - 1 ? last : slot][tid * OPT + o];
                            add(q);
                        }
                    }
                }
                __syncthreads();           // the buffers are staged into next
            }
            done_slabs += ns;
        }

        if (!SAFE) {
            // the overflow guard of chunk_gemm_valu: no Inf/NaN operand, chunk
            // partial sums at most 3 CL max|a| max|b| < 2^31, running sums
            // below 2^31 at every chunk end.  Non-negative floats (and NaN,
            // above them all) order as their bits.
            auto umax = [](uint32_t x, uint32_t y) __attribute__((always_inline)) { return max(x, y); };
            uint32_t ua = wave_reduce(__float_as_uint(amax_a) & 0x7FFFFFFFu, umax);
            uint32_t ub = wave_reduce(__float_as_uint(amax_b) & 0x7FFFFFFFu, umax);
            uint32_t uS = wave_reduce(__float_as_uint(smax) & 0x7FFFFFFFu, umax);
            uint32_t* st = s_track[gslot];
            if (lane == 0) {
                atomicMax(&st[0], ua);
                atomicMax(&st[1], ub);
                atomicMax(&st[2], uS);
            }
            gslot = gslot == 2 ? 0 : gslot + 1;
            if (tid < 3) s_track[gslot][tid] = 0;
            __syncthreads();
            ua = st[0], ub = st[1], uS = st[2];
            float ma = __uint_as_float(ua), mb = __uint_as_float(ub), sm = __uint_as_float(uS);
            if (P16) {
                // unscaled; an Inf or NaN code decodes to 2^32 or more
                ma *= 0x1p55f, mb *= 0x1p41f, sm *= 0x1p110f;
                if (!(ma < 0x1p32f && mb < 0x1p32f)) return false;
            } else if (max(ua, ub) >= kF32Inf) {
                return false;
            }
            // a product rounded to FP16 is at most (1 + 2^-10) |a b|, or 2^-39
            // in the subnormal range
            const double bound = P16 ? 3.01 * (double)g.CL * (double)ma * (double)mb + 1.0
                                     : 3.0 * (double)g.CL * (double)ma * (double)mb;
            if (!(bound < 2147483648.0)) return false;
            if (!(sm < 2147483648.0f)) return false;
        }
        if (to_ws) return true;

        // results: OPT consecutive codes of the row-major tile per thread
        if (tid * OPT >= B * B) return true;
        const int row = tid * OPT / B, col = tid * OPT % B;
        if (lt >= 0 && !g.C) {
            // the first piece of a shared tile, only the FP8 result wanted
            uint16_t* dst = g.s_ws + (lt * B + row) * B + col;
#pragma unroll
            for (int o = 0; o < OPT; ++o) dst[o] = (uint16_t)code(S[o]);
            return true;
        }
        const int m = m0 + row, n = n0 + col;
        if (m >= g.M) return true;
        if (g.C) {
            uint16_t* crow = g.C + (int64_t)m * g.ldc + n;
            if constexpr (OPT == 4) {
                if (g.c_vec8 && n + OPT <= g.N) {
                    *reinterpret_cast<uint2*>(crow) = make_uint2(code(S[0]) | (code(S[1]) << 16),
                                                                 code(S[2]) | (code(S[3]) << 16));
                } else {
#pragma unroll
                    for (int o = 0; o < OPT; ++o)
                        if (n + o < g.N) crow[o] = (uint16_t)code(S[o]);
                }
            } else if constexpr (OPT == 2) {
                if (g.c_vec && n + OPT <= g.N) {
                    *reinterpret_cast<uint32_t*>(crow) = code(S[0]) | (code(S[1]) << 16);
                } else {
                    if (n < g.N) crow[0] = (uint16_t)code(S[0]);
                    if (n + 1 < g.N) crow[1] = (uint16_t)code(S[1]);
                }
            } else {
                if (n < g.N) crow[0] = (uint16_t)code(S[0]);
            }
        }
        if (!P16 && g.C8 && lt < 0) {
            uint8_t* qrow = g.C8 + (int64_t)m * g.ldc8 + n;
#pragma unroll
            for (int o = 0; o < OPT; ++o)
                if (n + o < g.N) qrow[o] = (uint8_t)f32d_to_fp8_scaled<P16 ? 0 : DOM>(S[o], g.q_scale);
        }
        return true;
    };

    // work items of this workgroup: whole tiles, then its range of the shared
    // tile-chunks (gemm_plan.h)
    const int w = blockIdx.x;
    int64_t t = w;
    int64_t s = p.L > 0 ? (int64_t)w * p.L / p.G : 0;
    const int64_t e = p.L > 0 ? (int64_t)(w + 1) * p.L / p.G : 0;
    for (;;) {
        int64_t tile, lt;
        int c0, c1;
        if (t < p.t_whole) {
            tile = whole_tile(p, t);
            lt = -1;
            c0 = 0;
            c1 = p.nch;
            t += p.G;
        } else if (s < e) {
            lt = s / p.nch;
            c0 = (int)(s - lt * p.nch);
            const int64_t c1l = e - lt * p.nch;
            c1 = c1l < p.nch ? (int)c1l : p.nch;
            tile = p.t_whole + lt;
            s = lt * p.nch + c1;
        } else {
            break;
        }
        bool done = false;
        if (g.guarded) done = piece(std::integral_constant<bool, false>{}, tile, c0, c1, lt);
        if (!done) piece(std::integral_constant<bool, true>{}, tile, c0, c1, lt);
    }
}

// Entry addresses (configurations 0 .. 5 of this family).
template <bool TA, bool TB, bool P16>
const void* table(int i) {
    switch (i) {
        case 0: return reinterpret_cast<const void*>(&chunk_gemm_cpar<4, 4, TA, TB, P16>);
        case 1: return reinterpret_cast<const void*>(&chunk_gemm_cpar<4, 8, TA, TB, P16>);
        case 2: return reinterpret_cast<const void*>(&chunk_gemm_cpar<4, 16, TA, TB, P16>);
        case 3: return reinterpret_cast<const void*>(&chunk_gemm_cpar<2, 4, TA, TB, P16>);
        case 4: return reinterpret_cast<const void*>(&chunk_gemm_cpar<2, 8, TA, TB, P16>);
        case 5: return reinterpret_cast<const void*>(&chunk_gemm_cpar<2, 16, TA, TB, P16>);
        default: return nullptr;
    }
}

}  // namespace cpar
}  // namespace fp8t
