// Fused transform + quantization with row tiles of 16 (MFMA 16x16x32): n2 a multiple of 32, n1 padded to a multiple of 16 only.
//
// Same method as the other activation kernels (Eq. (2) left factor, fused as in Sec. 3.3): one wave per 32-column slab of n2;
// Z = X~ P2[:, slab], Y^T = Z^T P1 with Z split into fp16 hi + lo, per-token absmax, clip, round, pack, store; INT4 codes with a step per
// token, or MXFP4; the same bytes as tq_fast_kernel, whose order of sums it keeps (an MFMA adds its operands' groups of eight k, one per lane
// group, one after the other: v_mfma_f32_16x16x32_f16 gives the bits of two v_mfma_f32_32x32x16_f16).  Large launches are bound by the power that fp16
// MFMAs draw (112 x 256 at 16384 tokens, tq_fast_kernel: 490 us, 361 on all-zero rows) and small ones by the prologue's chain of latencies, so
// what counts is work not done:
//   * 112 rows are seven tiles of 16, not four of 32, in both contractions (112 x 256 at 16384 tokens 490 -> 425 us).  With an odd number of row
//     tiles the first one goes by MFMAs of 16 rows, and Z's accumulators (four rows of a column per lane) become the second one's operand by
//     exchanges between lane groups (v_permlane16_swap, v_permlane32_swap).  Even numbers go by tiles of 32.
//   * Two tiles of LDS per workgroup, filled by global-to-LDS loads with the 16-byte chunks swizzled: no registers and no LDS writes by the
//     waves, and one barrier per token (the absmax exchange, which also hands the tiles over), so that a wave rounds and stores its codes
//     while others are in the next token's MFMAs (64 x 128 at 2048 tokens 14.6 -> 13.2, 96 x 256 55 -> 52).
//   * The factors' staging takes global-to-LDS loads as well, P2 in one piece (86 x 128 at 64 tokens 6.0 -> 4.9 us, 112 x 128 7.8 -> 6.0), and P1's
//     fragments stay in registers where they fit beside P2's (up to 96 rows; 112 with four slabs).
#include "fq_internal.h"
#include "fq_device.h"

namespace fq {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Tokens' tiles in pairs, P1's fragment table behind them, then the absmax exchange and MXFP4's exponents (both twice); the factors'
// staging lies over all of it.
template <int R, int B, bool MX>
struct RowsLds {
    static constexpr int N2 = 32 * B, PW = 16 * R;
    // Odd numbers of row tiles: all of Y by tiles of 16 columns, whose hi and lo parts share an MFMA: fewer exchanges, less power, twice the
    // fragments of P1.  us with tiles of 32 and a last one of 16 / of 16: 72 x 128 at 16384 tokens 122 / 111, 48 x 128 77 / 68, 48 x 64 32 / 29, 112 x 256 at 8192
    // 246 / 231.  Not where only the former's fragments fit in registers (112 x 128 187 / 212), nor for even numbers (86 x 128 136 / 144).
    static constexpr bool T16 = R % 2 == 1 && (R <= 5 || B > 4);
    static constexpr int E = T16 ? 0 : R / 2, NT16 = R - 2 * E, EN = E + NT16, NF = R * EN;   // tiles of 32 and of 16 columns of Y, fragments of P1
    static constexpr int FRAG = T16 ? 512 : 1024;                  // both half-waves have the same fragment for tiles of 16
    static constexpr bool P1REG = T16 ? R <= 5 : R <= 6 || (R == 7 && B <= 4);    // P1's fragments beside P2's in registers
    static constexpr int TILE = 16 * R * N2 * 2;
    static constexpr int P1FLAT_BYTES = PW * PW * 2, STG_BYTES = P1FLAT_BYTES + N2 * N2 * 2;
    // the second tile lies behind the staging area, where that leaves room for two waves per SIMD (two slabs: four): its token is requested at once
    static constexpr bool EARLY = P1REG && STG_BYTES + TILE + 64 + (MX ? 32 * R * B : 0) <= 160 * 1024 / (B >= 5 ? 1 : B >= 3 ? 2 : 8);
    static constexpr int TILE1 = EARLY ? STG_BYTES : TILE;
    static constexpr int P1S = TILE1 + TILE, P1S_BYTES = P1REG ? 0 : NF * FRAG;
    static constexpr int RED = P1S + P1S_BYTES, EXPS = RED + 64, EXPS_BYTES = 16 * R * B;
    static constexpr int TOTAL = (cmax(EXPS + (MX ? 2 * EXPS_BYTES : 0), STG_BYTES) + 15) & ~15;
};

template <int R, int B, bool MX>
__global__ __launch_bounds__(64 * B) __attribute__((amdgpu_waves_per_eu(2))) void tq_rows_kernel(TqDev p, const float* __restrict__ clip) {
    using L = RowsLds<R, B, MX>;
    constexpr int N2 = L::N2, PW = L::PW, NF = L::NF, NT = 64 * B, E = L::E, NT16 = L::NT16, EN = L::EN;
    constexpr bool ODD = NT16 > 0;             // MFMAs of 16 rows in the first contraction
    constexpr bool P1REG = L::P1REG;
    constexpr int SW = B % 4 == 0 ? 15 : B % 2 == 0 ? 7 : 3, SWS = B % 4 == 0 ? 0 : B % 2 == 0 ? 1 : 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* red = reinterpret_cast<float*>(smem + L::RED);
    _Float16* P1flat = reinterpret_cast<_Float16*>(smem);
    _Float16* P2flat = reinterpret_cast<_Float16*>(smem + L::P1FLAT_BYTES);
    typedef __attribute__((address_space(3))) void* lptr;

    const int tid = threadIdx.x, l = tid & 63, c = l & 15, q = l >> 4, c32 = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n1 = p.n1;
    const int64_t G = gridDim.x;
    int64_t t = blockIdx.x;

    // ---- token rows: instruction k of a wave brings 1 KB, rows 16 k .. of which this lane has one 16-byte chunk.  The chunk of slot s of
    // row r is s ^ ((r >> SWS) & SW): 16 rows at the same chunk are 16 different slots of the banks.  Rows past n1 read as zeros.
    const int xrow = (64 * w + l) / (4 * B), xslot = (64 * w + l) % (4 * B);
    const int xoff = xrow * (64 * B) + 16 * (xslot ^ ((xrow >> SWS) & SW));
    auto row_buffer = [&](int64_t tok) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.x) + tok * p.x_stride, 0, n1 * N2 * 2, 0x00020000);
    };
    auto fetch = [&](int64_t tok, int buf) {              // straight into the tile
        const __amdgpu_buffer_rsrc_t xb = row_buffer(tok);
#pragma unroll
        for (int k = 0; k < R; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xb, (lptr)(smem + buf * L::TILE1 + (w + B * k) * 1024), 16, xoff, k * 1024 * B, 0, 2);
    };

    // ---- the factors: P2 as it is, P1's rows at the pitch of whole tiles (the padding zero); the first token behind them, in registers
    {
        const __amdgpu_buffer_rsrc_t pb = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.P2), 0, N2 * N2 * 2, 0x00020000);
#pragma unroll
        for (int k = 0; k < 2 * B; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(pb, (lptr)(smem + L::P1FLAT_BYTES + (w + B * k) * 1024), 16, 16 * l, (w + B * k) * 1024, 0, 0);
    }
    // P1: a wave takes whole rows, a lane a pair of columns.  Rows of an even length go straight into LDS (lanes past them and rows past the
    // last read as zeros); odd ones start on odd halves and go through registers, their last pair loaded one half early.
    constexpr int RPW = (PW + B - 1) / B;
    u32x4 pre[R];
    auto fetch_first = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        const __amdgpu_buffer_rsrc_t xb = row_buffer(t);
#pragma unroll
        for (int k = 0; k < R; ++k) pre[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xb, xoff, k * 1024 * B, 2));
        __builtin_amdgcn_sched_barrier(0);
    };
    if (n1 == PW && (reinterpret_cast<uintptr_t>(p.P1) & 15) == 0) {   // whole tiles: as it is
        const __amdgpu_buffer_rsrc_t pb = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.P1), 0, PW * PW * 2, 0x00020000);
        constexpr int CH = PW * PW / 8;
#pragma unroll
        for (int k = 0; k < (CH + NT - 1) / NT; ++k)
            if (NT * (k + 1) <= CH || tid + NT * k < CH)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(pb, (lptr)(smem + (w + B * k) * 1024), 16, 16 * l, (w + B * k) * 1024, 0, 0);
        fetch_first();
    } else if ((n1 & 1) == 0) {
        const __amdgpu_buffer_rsrc_t pb = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.P1), 0, n1 * n1 * 2, 0x00020000);
        const int off = 2 * l < n1 ? 4 * l : 0x40000000;
        if (l < PW / 2) {
#pragma unroll
            for (int k = 0; k < RPW; ++k)
                if (B * (k + 1) <= PW || w + B * k < PW)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(pb, (lptr)(smem + (w + B * k) * (2 * PW)), 4, off, (w + B * k) * (2 * n1), 0, 0);
        }
        fetch_first();
    } else {
        typedef uint32_t __attribute__((aligned(2))) pair_t;
        const int nq = (n1 + 1) >> 1;
        const bool half = l >= nq - 1;
        const int off = half ? n1 - 2 : 2 * l;
        uint32_t v[RPW];
#pragma unroll
        for (int k = 0; k < RPW; ++k) {
            const int row = w + k * B;
            v[k] = *reinterpret_cast<const pair_t*>(p.P1 + (row < n1 ? row : n1 - 1) * n1 + off);
        }
        fetch_first();
        uint32_t* dst = reinterpret_cast<uint32_t*>(P1flat);
#pragma unroll
        for (int k = 0; k < RPW; ++k) {
            const int row = w + k * B;
            if (row < PW && l < PW / 2) dst[row * (PW / 2) + l] = row < n1 && l < nq ? (half ? v[k] >> 16 : v[k]) : 0u;
        }
    }
    if (L::EARLY && t + G < p.T) {
        fetch(t + G, 1);
        wait_vm_pending<2 * R>();                                  // all but the tokens' rows
    } else {
        wait_vm_pending<R>();
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // P2 as the second operand: of the MFMAs of 32 rows, P2[16 k + 8 h + j][slab + c32], or, with an odd number of row tiles, of those of 16,
    // P2[32 m + 8 q + j][slab + 16 ct + c] for k = 2 m + ct
    half8 p2f[2 * B];
#pragma unroll
    for (int k = 0; k < 2 * B; ++k)
        p2f[k] = ODD ? lds_column8(P2flat, N2, 16 * (k & ~1) + 8 * q, 4, 32 * w + 16 * (k & 1), c) : lds_column8(P2flat, N2, 16 * k + 8 * h, 4, 32 * w + (c32 & 16), c);
    // P1, fragment kk EN + It: the eight rows of row tile kk that Z's operand has, and columns 32 It + c32, or the last 16 of an odd number of row
    // tiles, where the upper half-wave's rows are the lower one's again (hi and lo parts in one MFMA)
    constexpr int NP1 = P1REG ? NF : (NF + B - 1) / B;
    half8 p1f[NP1];
#pragma unroll
    for (int k = 0; k < NP1; ++k) {
        const int e = P1REG ? k : w + B * k < NF ? w + B * k : 0, kk = e / EN, It = e % EN;
        const bool last = It >= E;
        p1f[k] = lds_column8(P1flat, PW, 16 * kk + 4 * (last ? q & 1 : h), 8, last ? 32 * E + 16 * (It - E) : 32 * It + (c32 & 16), c);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the staging area is free
    if constexpr (!P1REG) {
#pragma unroll
        for (int k = 0; k < NP1; ++k)
            if (w + B * k < NF && (L::FRAG == 1024 || h == 0)) *reinterpret_cast<half8*>(smem + L::P1S + (w + B * k) * L::FRAG + 16 * (L::FRAG == 1024 ? l : c32)) = p1f[k];
    }
#pragma unroll
    for (int k = 0; k < R; ++k) *reinterpret_cast<u32x4*>(smem + (w + B * k) * 1024 + 16 * l) = pre[k];
    if (!L::EARLY && t + G < p.T) fetch(t + G, 1);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // 16-byte chunk j of a row is in slot j ^ swizzle.  An operand's chunks: 2 k + h of row c32, or 4 m + q of row c
    const int swz = (c >> SWS) & SW;          // (of c32 as well)
    const int u = (ODD ? q : h) ^ swz, row_bytes = (ODD ? c : c32) * (64 * B);
    constexpr float kadd = 2047.5f / 32767.0f;
    uint8_t* exps = reinterpret_cast<uint8_t*>(p.out_scales);
    auto copy_exponents = [&](int64_t tok, int buf) {              // n1 * B bytes, a multiple of 4 (checked on the host)
        const uint8_t* src = smem + L::EXPS + buf * L::EXPS_BYTES;
        if (p.mx_tiled) {   // tile order of the MXFP4 product: byte (((t / 128) KI + j) 128 + t % 128) 8 + b
            const int ki = n1 * B / 8;
            uint2* dst = reinterpret_cast<uint2*>(exps) + (tok >> 7) * ((int64_t)ki * 128) + (tok & 127);
            for (int j = tid; j < ki; j += NT) dst[(int64_t)j * 128] = reinterpret_cast<const uint2*>(src)[j];
        } else {
            uint32_t* dst = reinterpret_cast<uint32_t*>(exps + tok * ((int64_t)n1 * B));
            for (int i = tid; i < n1 * B / 4; i += NT) dst[i] = reinterpret_cast<const uint32_t*>(src)[i];
        }
    };

#pragma unroll 1
    for (int buf = 0;; buf ^= 1, t += G) {
        const float clipv = clip[p.clip_mode ? t : 0];
        f32x16 acc[E > 0 ? E : 1];
        f32x4 tail[NT16 > 0 ? NT16 : 1][2];                        // columns 32 E + 16 j .. of Y, 16 channels each
#pragma unroll
        for (int It = 0; It < E; ++It)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[It][r] = 0.0f;
#pragma unroll
        for (int j = 0; j < NT16; ++j)
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) tail[j][ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        constexpr int NX = ODD ? 4 : 8, STEP = ODD ? 4 : 2;        // operands of 256 bytes of a row, chunks from one to the next
        const unsigned char* xb[NX];
#pragma unroll
        for (int m = 0; m < NX; ++m) xb[m] = smem + buf * L::TILE1 + row_bytes + 16 * ((STEP * m) ^ u);
        auto operand = [&](int m, int tile) {                      // tile: of 32 rows, ODD: 16
            return *reinterpret_cast<const half8*>(xb[m % NX] + (m / NX) * 256 + tile * (ODD ? 16 : 32) * 64 * B);
        };
        auto p1 = [&](int e) { return P1REG ? p1f[P1REG ? e : 0] : *reinterpret_cast<const half8*>(smem + L::P1S + e * L::FRAG + 16 * (L::FRAG == 1024 ? l : c32)); };
        auto second = [&](int kk, half8 zh, half8 zl) {            // Y^T += Z^T P1 over row tile kk
            half8 b[E > 0 ? E : 1];
#pragma unroll
            for (int It = 0; It < E; ++It) b[It] = p1(kk * EN + It);
#pragma unroll
            for (int It = 0; It < E; ++It) acc[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zh, b[It], acc[It], 0, 0, 0);
#pragma unroll
            for (int It = 0; It < E; ++It) acc[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zl, b[It], acc[It], 0, 0, 0);
        };
        if constexpr (!ODD) {
            // row tiles of 32 in pairs, so that consecutive MFMAs are independent
#pragma unroll
            for (int I0 = 0; I0 < E; I0 += 2) {
                const bool two = I0 + 1 < E;
                f32x16 z[2];
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) z[d][r] = 0.0f;
                half8 next[2];
                next[0] = operand(0, I0);
                if (two) next[1] = operand(0, I0 + 1);
#pragma unroll
                for (int k = 0; k < 2 * B; ++k) {
                    const half8 a0 = next[0], a1 = next[1];
                    if (k + 1 < 2 * B) {
                        next[0] = operand(k + 1, I0);
                        if (two) next[1] = operand(k + 1, I0 + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    z[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, p2f[k], z[0], 0, 0, 0);
                    if (two) z[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, p2f[k], z[1], 0, 0, 0);
                }
#pragma unroll
                for (int kq = 0; kq < 4; ++kq)
                    if (kq < 2 || two) {
                        half8 zh, zl;
                        split_hi_lo(z[kq / 2], 8 * (kq % 2), zh, zl);
                        second(2 * I0 + kq, zh, zl);
                    }
            }
        } else {
#pragma unroll
            for (int s = 0; s < (R + 1) / 2; ++s) {                // row tiles of 16 in pairs
                const bool two = 2 * s + 1 < R;
                f32x4 z[2][2];
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) z[d][ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                half8 next[2];
                next[0] = operand(0, 2 * s);
                if (two) next[1] = operand(0, 2 * s + 1);
#pragma unroll
                for (int m = 0; m < B; ++m) {
                    const half8 a0 = next[0], a1 = next[1];
                    if (m + 1 < B) {
                        next[0] = operand(m + 1, 2 * s);
                        if (two) next[1] = operand(m + 1, 2 * s + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) {
                        z[0][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, p2f[2 * m + ct], z[0][ct], 0, 0, 0);
                        if (two) z[1][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, p2f[2 * m + ct], z[1][ct], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int d = 0; d < 2; ++d)
                    if (d == 0 || two) {
                        // a lane has rows 4 q .. of columns c and 16 + c.  For the MFMAs of 32 columns it takes rows 4 h .. and 8 + 4 h .. of
                        // column c32; for those of 16, rows 4 (q & 1) .. and 8 + 4 (q & 1) .. of a column, hi parts in the lower half-wave, lo in the upper
                        uint32_t hi[2][2], lo[2][2];
#pragma unroll
                        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const float z0 = z[d][ct][2 * k], z1 = z[d][ct][2 * k + 1];
                                hi[ct][k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(z0, z1));
                                lo[ct][k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(sub_half<0>(z0, hi[ct][k]), sub_half<1>(z1, hi[ct][k])));
                            }
                        auto columns32 = [&](const uint32_t (&v)[2][2]) {
                            u32x4 o;
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const auto s16 = __builtin_amdgcn_permlane16_swap(v[0][k], v[1][k], false, false);
                                const auto s32 = __builtin_amdgcn_permlane32_swap(s16[0], s16[1], false, false);
                                o[k] = s32[0];
                                o[2 + k] = s32[1];
                            }
                            return __builtin_bit_cast(half8, o);
                        };
                        const int kk = 2 * s + d;
                        if constexpr (E > 0) second(kk, columns32(hi), columns32(lo));
                        half8 z16[2];
#pragma unroll
                        for (int ct = 0; ct < 2; ++ct) {
                            u32x4 o;
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const auto s32 = __builtin_amdgcn_permlane32_swap(hi[ct][k], lo[ct][k], false, false);
                                o[k] = s32[0];
                                o[2 + k] = s32[1];
                            }
                            z16[ct] = __builtin_bit_cast(half8, o);
                        }
#pragma unroll
                        for (int j = 0; j < NT16; ++j) {
                            const half8 b = p1(kk * EN + E + j);
#pragma unroll
                            for (int ct = 0; ct < 2; ++ct) tail[j][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(z16[ct], b, tail[j][ct], 0, 0, 0);
                        }
                    }
            }
        }
        if constexpr (!MX) {
            float m = 0.0f;
#pragma unroll
            for (int It = 0; It < E; ++It)
#pragma unroll
                for (int r = 0; r < 16; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(acc[It][r]));
#pragma unroll
            for (int j = 0; j < NT16; ++j)
#pragma unroll
                for (int r = 0; r < 8; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(tail[j][r >> 2][r & 3]));
            m = wave_max(m);
            if (l == 0) red[buf * 8 + w] = m;
        }
        // One barrier per token: every wave is done with this tile, the next one has arrived, this token's absmax parts (the last one's
        // exponents) are visible.
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 2 * G < p.T) fetch(t + 2 * G, buf);
        float kmul = 0.0f;
        if constexpr (!MX) {
            float m = 0.0f;
#pragma unroll
            for (int b = 0; b < B; ++b) m = __builtin_fmaxf(m, red[buf * 8 + b]);
            const _Float16 sh = (_Float16)(clipv * m * 0.142857149f);   // step = alpha * max / 7, round-to-nearest-even to fp16
            const float st = (float)sh;
            const float inv = (st > 0.0f && st <= 65504.0f) ? __builtin_amdgcn_rcpf(st) : 0.0f;
            kmul = inv * (4096.0f / 32767.0f);
            if (w == 0) p.out_scales[t] = sh;
        } else if (t != blockIdx.x) {
            copy_exponents(t - G, buf ^ 1);
        }
        uint8_t* dst = p.out_codes + t * (int64_t)(n1 * (N2 / 2)) + 16 * w;
        // codes of values a .. of a lane, b .. behind them
        auto codes8 = [&](const auto& a, int ai, const auto& b, int bi, float scale) {
            if constexpr (MX) {
                uint32_t pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, a[ai], a[ai + 1], scale, 0);
                pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, a[ai + 2], a[ai + 3], scale, 1);
                pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, b[bi], b[bi + 1], scale, 2);
                return (uint32_t)__builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, b[bi + 2], b[bi + 3], scale, 3);
            } else {
                uint32_t D[4];
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    D[r] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pknorm_i16(__builtin_fmaf(a[ai + r], kmul, kadd), __builtin_fmaf(b[bi + r], kmul, kadd)));
                // bytes 1 and 3 of D[r] carry nibbles r and r + 4 on top: even nibbles -> E, odd ones -> F
                const uint32_t ev = __builtin_amdgcn_perm(D[2], D[0], 0x07030501u);
                const uint32_t od = __builtin_amdgcn_perm(D[3], D[1], 0x07030501u);
                return (od & 0xF0F0F0F0u) | ((ev >> 4) & 0x0F0F0F0Fu);
            }
        };
        // MXFP4: the shared exponent of a block whose largest magnitude in this lane's part is m, lane pairs (c32, h) or all four lane groups
        auto exponent = [&](float m, bool four) {
            const uint32_t mb = __builtin_bit_cast(uint32_t, m);
            const auto s32 = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
            m = __builtin_fmaxf(__builtin_bit_cast(float, (uint32_t)s32[0]), __builtin_bit_cast(float, (uint32_t)s32[1]));
            if (four) {
                const uint32_t m2 = __builtin_bit_cast(uint32_t, m);
                const auto s16 = __builtin_amdgcn_permlane16_swap(m2, m2, false, false);
                m = __builtin_fmaxf(__builtin_bit_cast(float, (uint32_t)s16[0]), __builtin_bit_cast(float, (uint32_t)s16[1]));
            }
            m *= clipv;
            const int be = (int)((__builtin_bit_cast(uint32_t, m) >> 23) & 0xffu);   // biased exponent of alpha * max
            return be > 2 ? be - 2 : 0;
        };
        uint2 first8 = {0u, 0u};
#pragma unroll
        for (int It = 0; It < E; ++It) {
            const int row = 32 * It + c32;
            float scale = 0.0f;
            if constexpr (MX) {
                float m = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(acc[It][r]));
                const int e = exponent(m, false);
                scale = __builtin_bit_cast(float, (uint32_t)e << 23);
                if (h == 0) smem[L::EXPS + buf * L::EXPS_BYTES + row * B + w] = (uint8_t)e;
            }
            // channels 8 g + 4 h .. of the slab in registers 4 g ..: afterwards half-wave 0 has the groups g = 0, 1 of both, half-wave 1 the others
            const auto sw = __builtin_amdgcn_permlane32_swap(codes8(acc[It], 0, acc[It], 4, scale), codes8(acc[It], 8, acc[It], 12, scale), false, false);
            const uint2 o = {__builtin_amdgcn_perm(sw[1], sw[0], 0x05040100u), __builtin_amdgcn_perm(sw[1], sw[0], 0x07060302u)};
            if (It % 2 == 0 && It + 1 < E) {                       // with the next row tile: half-wave h stores 16 bytes of row tile It + h
                first8 = o;
            } else if (It % 2 == 0) {
                if (row < n1) *reinterpret_cast<uint2*>(dst + row * (N2 / 2) + 8 * h) = o;
            } else {
                const auto x = __builtin_amdgcn_permlane32_swap(first8.x, o.x, false, false);
                const auto y = __builtin_amdgcn_permlane32_swap(first8.y, o.y, false, false);
                const int row2 = 32 * (It - 1 + h) + c32;
                if (row2 < n1) *reinterpret_cast<u32x4*>(dst + row2 * (N2 / 2)) = u32x4{x[0], y[0], x[1], y[1]};
            }
        }
#pragma unroll
        for (int g = 0; g < (NT16 + 3) / 4; ++g) {                 // tiles of 16, four at a time
            uint32_t d[4];                                         // of tile 4 g + k: channels 4 q .. and 16 + 4 q .. of row c
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = 4 * g + k;
                d[k] = 0;
                if (j >= NT16) continue;
                float scale = 0.0f;
                if constexpr (MX) {
                    float m = 0.0f;
#pragma unroll
                    for (int r = 0; r < 8; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(tail[j][r >> 2][r & 3]));
                    const int e = exponent(m, true);
                    scale = __builtin_bit_cast(float, (uint32_t)e << 23);
                    if (q == 0) smem[L::EXPS + buf * L::EXPS_BYTES + (32 * E + 16 * j + c) * B + w] = (uint8_t)e;
                }
                d[k] = codes8(tail[j][0], 0, tail[j][1], 0, scale);
            }
            // 4 x 4 between the lane groups and the tiles: afterwards lane group q has all 32 channels of tile 4 g + q
            const auto e0 = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
            const auto e1 = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
            const auto f0 = __builtin_amdgcn_permlane16_swap(e0[0], e1[0], false, false);
            const auto f1 = __builtin_amdgcn_permlane16_swap(e0[1], e1[1], false, false);
            const u32x4 o = {__builtin_amdgcn_perm(f0[1], f0[0], 0x05040100u), __builtin_amdgcn_perm(f1[1], f1[0], 0x05040100u),
                             __builtin_amdgcn_perm(f0[1], f0[0], 0x07060302u), __builtin_amdgcn_perm(f1[1], f1[0], 0x07060302u)};
            const int j = 4 * g + q, row = 32 * E + 16 * j + c;
            if (j < NT16 && row < n1) *reinterpret_cast<u32x4*>(dst + row * (N2 / 2)) = o;
        }
        if (t + G >= p.T) {
            if constexpr (MX) {
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                copy_exponents(t, buf);
            }
            break;
        }
    }
}

using RowsFn = void (*)(TqDev, const float*);
struct RowsVariant {
    RowsFn fn;
    int lds;
};
// an instance, if any left factor of these row tiles gets here
template <int R, int B, bool MX>
static RowsVariant rows_instance() {
    if constexpr (rows_kernel_reached(R, B, MX)) return {&tq_rows_kernel<R, B, MX>, RowsLds<R, B, MX>::TOTAL};
    else return {nullptr, 0};
}
template <int R>
static RowsVariant rows_variant_a(int B, bool mx) {
    switch (B) {
        case 2: return mx ? rows_instance<R, 2, true>() : rows_instance<R, 2, false>();
        case 3: return mx ? rows_instance<R, 3, true>() : rows_instance<R, 3, false>();
        case 4: return mx ? rows_instance<R, 4, true>() : rows_instance<R, 4, false>();
        case 5: return mx ? rows_instance<R, 5, true>() : rows_instance<R, 5, false>();
        case 6: return mx ? rows_instance<R, 6, true>() : rows_instance<R, 6, false>();
        case 7: return mx ? rows_instance<R, 7, true>() : rows_instance<R, 7, false>();
        default: return mx ? rows_instance<R, 8, true>() : rows_instance<R, 8, false>();
    }
}
static RowsVariant rows_variant(int R, int B, bool mx) {
    switch (R) {
        case 2: return rows_variant_a<2>(B, mx);
        case 3: return rows_variant_a<3>(B, mx);
        case 4: return rows_variant_a<4>(B, mx);
        case 5: return rows_variant_a<5>(B, mx);
        case 6: return rows_variant_a<6>(B, mx);
        case 7: return rows_variant_a<7>(B, mx);
        default: return rows_variant_a<8>(B, mx);
    }
}

int64_t tq_rows_lds_bytes(int n1, int n2) { return rows_variant((n1 + 15) / 16, n2 / 32, false).lds; }

hipError_t tq_rows_launch(const TqDev& d, hipStream_t stream, bool mx) {
    const int R = (d.n1 + 15) / 16, B = d.n2 / 32;
    const RowsVariant v = rows_variant(R, B, mx);
    static OccCache occ_cache[9][9][2];
    int occ = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(v.fn), 64 * B, v.lds, occ_cache[R][B][mx], occ);
    if (e != hipSuccess) return e;
    const int cap = tuned(Knob::WG_PER_CU, 0);
    if (cap > 0 && cap < occ) occ = cap;
    const int64_t resident = (int64_t)cu_count() * occ, rounds = (d.T + resident - 1) / resident;
    return launch(v.fn, dim3((unsigned)((d.T + rounds - 1) / rounds)), dim3(64 * B), v.lds, stream, d, d.clip);
}

}  // namespace fq
