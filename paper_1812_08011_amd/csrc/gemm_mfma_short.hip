// chunk_gemm fast mode on the matrix cores for short K: K a multiple of 64, at
// most 256 (the Backward GEMM of a layer, whose K is its output channels).
//
// Same arithmetic, instruction and lane layout as chunk_gemm_mfma_wave
// (gemm_mfma_wave.hip), so the same bits.  There every wave streams its own
// operands 128 k at a time through one LDS tile, which at such K is one or two
// rounds, each waited for alone (a last half round through registers), and
// each of a workgroup's four waves loads the same rows of A.  Here a workgroup
// owns 32 RB x 128 outputs and
//   * starts all its loads at once -- both operands' whole K straight into
//     LDS (global_load_lds), every row once for the four waves -- and waits
//     once;
//   * each wave forms 32 x 32 RB outputs, A's operands in registers (8 per 64-k
//     slab), B's read per slab, a block's matrix instructions independent of
//     the epilogue of the block before;
//   * with RB = 2 the finished codes leave as whole 128-byte lines.
// LDS rows are the K bytes (KP: 64, 128 or 256), their 16-byte pieces
// XOR-swizzled by the row through the lanes' fetch addresses.  A wave whose
// block fails the guard (running sums at 2^31 or NaN) forms it again from the
// same operands with the 2^96-scaled epilogue.
// Bound by the result stores and the epilogue on the vector ALUs (about 44 and
// 32 us of the first shape below), which workgroups of different age overlap
// in part.  Measured (us, chunk_gemm_mfma_wave / RB = 1 / RB = 2), M x N x K,
// CL 64: 50176 x 2304 x 256 114 / 102 / 94 (2.5 TB/s of results), 50176 x 576
// x 64 55 / 14.9 / 14.0, 25088 x 1728 x 192 83 / 36.9 / 33.4, 12544 x 1152 x
// 128 13.7 / 11.0 / 11.1; few tiles: 3136 x 4608 x 256 (CL 256) 16.2 / 13.7 /
// 14.5, 50176 x 256 x 256 20.6 / 18.1 / 18.8.  128 rows per workgroup (two
// resident on a CU): 105 on the first; non-temporal stores: 95.
#include "fp8t_device.h"
#include "gemm_mfma.h"

namespace fp8t {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int kWaves = 4;
constexpr int kNT = 64 * kWaves;
constexpr int kBN = 32 * kWaves;

// Result register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
__device__ __forceinline__ int out_row(int l, int r) { return 8 * (r / 4) + 4 * (l / 32) + r % 4; }

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// XOR of a row's 16-byte piece index: rows whose equal pieces share LDS banks
// (256 bytes apart) get different ones.
template <int KP> __device__ __forceinline__ int swz(int r) {
    return KP == 256 ? r & 15 : KP == 128 ? (r >> 1) & 7 : (r >> 2) & 3;
}

// NS: 64-k slabs (K = 64 NS); RB: 1 or 2; ONE: every slab is a chunk of its own
// (CL = 64).
template <int NS, int RB, bool ONE>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(RB == 2 ? 3 : 4)))
void chunk_gemm_mfma_short(GemmArgs g, Plan p) {
    constexpr int KP = NS == 1 ? 64 : NS == 2 ? 128 : 256;
    constexpr int NSEG = KP / 16;          // 16-byte pieces of a row
    constexpr int RPI = 64 / NSEG;         // rows of one load instruction
    constexpr int NA = 32 * RB / RPI, NB = 32 / RPI;
    constexpr int CB = RB;                 // 32-column blocks of a wave
    constexpr int OP = 64 * CB;            // LDS row pitch (bytes) of the staged codes
    constexpr int SA = 32 * RB * KP;
    constexpr int SC = RB == 2 ? kWaves * 32 * OP : 0;     // the codes' tiles, in place of A
    __shared__ __attribute__((aligned(16))) uint8_t sa[SA > SC ? SA : SC];
    __shared__ __attribute__((aligned(16))) uint8_t sb[kWaves][32 * KP];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rl = lane & 31, h = lane >> 5;       // operand row, k half
    const int lr = lane / NSEG, ls = lane % NSEG;  // row and LDS piece of a load
    int tr, tc;
    tile_rc(p, whole_tile(p, blockIdx.x), tr, tc);
    const int wr = wave / (kWaves / RB), wc = wave % (kWaves / RB);
    const int t0 = tr * (32 * RB), u0 = tc * kBN;  // the tile
    const int m0 = t0 + 32 * wr, n0 = u0 + 32 * CB * wc;   // the wave's part of it

    // Load instruction i of a 32-row group: lane l lands at i KB + 16 l, row
    // RPI i + l / NSEG, piece l % NSEG, so it fetches piece (l % NSEG) ^ swz(row)
    // (rows beyond the matrix read as its last; a piece beyond K, of NS = 3
    // only, as the last one before it: never used).
    auto load = [&](const uint8_t* base, int64_t ld, int r0, int rows, int i, uint8_t* dst)
                    __attribute__((always_inline)) {
        const int row = RPI * i + lr;
        int piece = ls ^ swz<KP>(row);
        if (NS == 3) piece = min(piece, 4 * NS - 1);
        const int rb = min(r0, rows - 1);
        const uint8_t* const b = base + (int64_t)rb * ld;
        const uint32_t off = (uint32_t)((min(r0 + row, rows - 1) - rb) * (int)ld + 16 * piece);
        __builtin_amdgcn_global_load_lds((gptr_t)(b + off), (lptr_t)(dst + i * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < NB; ++i) load(g.B, g.ldb, u0 + 32 * wave, g.N, i, sb[wave]);
#pragma unroll
    for (int j = 0; j < (NA + kWaves - 1) / kWaves; ++j) {
        const int i = wave + kWaves * j;
        if (i < NA) {
            const int grp = i / NB;
            load(g.A, g.lda, t0 + 32 * grp, g.M, i % NB, sa + grp * 32 * KP);
        }
    }
    // direct loads count in vmcnt; the compiler does not see their LDS writes
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    auto operand = [&](const uint8_t* rows, int sl) __attribute__((always_inline)) {
        const int s0 = 4 * sl + 2 * h;
        const vu4 x = *reinterpret_cast<const vu4*>(rows + rl * KP + 16 * (s0 ^ swz<KP>(rl)));
        const vu4 y = *reinterpret_cast<const vu4*>(rows + rl * KP + 16 * ((s0 + 1) ^ swz<KP>(rl)));
        v8i o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            o[q] = (int)x[q];
            o[4 + q] = (int)y[q];
        }
        return o;
    };
    v8i a8[NS];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) a8[sl] = operand(sa + wr * 32 * KP, sl);
    // the codes' tile of the wave: with RB = 2 in place of A, which every wave
    // holds in registers behind this barrier; else in the wave's own rows of
    // B, written when its only block is formed
    if (RB == 2) __syncthreads();
    if (m0 >= g.M || n0 >= g.N) return;    // no barrier after this
    uint8_t* const lco = RB == 2 ? sa + wave * 32 * OP : sb[wave];
    // byte offset of 16-byte piece q of the tile's row r: 4 rows on, where the
    // lanes' other half writes, the 64-byte halves change places
    auto code_off = [&](int r, int q) __attribute__((always_inline)) {
        return r * OP + 16 * (RB == 2 ? q ^ (r & 4) : q);
    };

    // The wave's block of columns n0 + 32 cb ..: its codes to the tile; false: it
    // failed the guard.
    auto block = [&](auto safe_tag, int cb) __attribute__((always_inline)) -> bool {
        constexpr bool SAFE = decltype(safe_tag)::value;
        const uint8_t* const rows = sb[wc * CB + cb];
        const v16f zero = {};
        float S[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = 0.0f;
        float vmax = 0.0f;                 // largest |S| at chunk ends (NaN stays)
        v16f acc = zero;
        int crem = g.CL;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            // format selectors 1, 1: both operands bf8 (= the FP8 codes); no
            // scaling; a chunk's first slab starts from zero
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                a8[sl], operand(rows, sl), ONE || crem == g.CL ? zero : acc, 1, 1, 0, 0, 0, 0);
            if (!ONE) {
                crem -= 64;
                if (crem != 0 && sl + 1 < NS) continue;
                crem = g.CL;
            }
            if (SAFE) {
#pragma unroll
                for (int r = 0; r < 16; ++r) S[r] = rn16s(S[r] + rn16s(acc[r] * 0x1p96f));
            } else {
                // S = rn16v(S + rn16v(acc)), step by step over the 16 outputs
                float c[16], x[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) c[r] = acc[r] * -16383.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = __builtin_fmaf(acc[r], 16384.0f, c[r]);
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = S[r] + x[r];
#pragma unroll
                for (int r = 0; r < 16; ++r) c[r] = x[r] * -16383.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) S[r] = __builtin_fmaf(x[r], 16384.0f, c[r]);
#pragma unroll
                for (int r = 0; r < 16; r += 2) vmax = maximum3_abs(vmax, S[r], S[r + 1]);
            }
        }
        if (!SAFE && __any(!(vmax < 2147483648.0f))) return false;
        if (RB == 1) wave_lds_sync();      // the codes go over the rows of B just read
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = out_row(lane, r), col = 32 * cb + rl;
            *reinterpret_cast<uint16_t*>(lco + code_off(row, col / 8) + 2 * (col % 8)) =
                (uint16_t)fp16_code<SAFE ? 96 : 0>(S[r]);
        }
        return true;
    };
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
        if (!g.guarded || !block(std::false_type{}, cb)) block(std::true_type{}, cb);

    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 2 * CB; ++q) {
        const int u = lane + 64 * q;
        const int row = u / (4 * CB), piece = u % (4 * CB);
        const vu4 v = *reinterpret_cast<const vu4*>(lco + code_off(row, piece));
        const int m = m0 + row, n = n0 + 8 * piece;
        if (m >= g.M || n >= g.N) continue;
        if (g.C) {
            uint16_t* cp = g.C + (int64_t)m * g.ldc + n;
            if (g.c_vec16 && n + 8 <= g.N) {
                *reinterpret_cast<vu4*>(cp) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (n + e < g.N) cp[e] = (uint16_t)(v[e / 2] >> (16 * (e % 2)));
            }
        }
        if (g.C8) {
            auto val = [&](int e) __attribute__((always_inline)) {
                return fp16_to_f32((v[e / 2] >> (16 * (e % 2))) & 0xFFFFu) * g.q_scale;
            };
            uint2 v8;
            v8.x = f32x2_to_fp8x2<true>(val(2), val(3), f32x2_to_fp8x2<false>(val(0), val(1), 0u));
            v8.y = f32x2_to_fp8x2<true>(val(6), val(7), f32x2_to_fp8x2<false>(val(4), val(5), 0u));
            uint8_t* qp = g.C8 + (int64_t)m * g.ldc8 + n;
            if (g.c8_vec8 && n + 8 <= g.N) {
                *reinterpret_cast<uint2*>(qp) = v8;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (n + e < g.N) qp[e] = (uint8_t)((e < 4 ? v8.x : v8.y) >> (8 * (e % 4)));
            }
        }
    }
}

template <int RB, bool ONE>
const void* entry(int ns) {
    switch (ns) {
        case 1: return reinterpret_cast<const void*>(&chunk_gemm_mfma_short<1, RB, ONE>);
        case 2: return reinterpret_cast<const void*>(&chunk_gemm_mfma_short<2, RB, ONE>);
        case 3: return reinterpret_cast<const void*>(&chunk_gemm_mfma_short<3, RB, ONE>);
        case 4: return reinterpret_cast<const void*>(&chunk_gemm_mfma_short<4, RB, ONE>);
        default: return nullptr;
    }
}

}  // namespace

const void* mfma_short_kernel(int rb, int ns, int one) {
    if (rb == 1) return one ? entry<1, true>(ns) : entry<1, false>(ns);
    return one ? entry<2, true>(ns) : entry<2, false>(ns);
}

}  // namespace fp8t
