// Fused per-token Kronecker transform + symmetric INT4 quantization for gfx950.
//
// Computes, for every token row, Q(P1^T X~ P2) (Eq. (2), left factor; the fused
// design of Sec. 3.3 / App. "Detailed Design of Kernel Fusion": both small
// contractions and the quantizer in one launch, intermediates never leave the
// chip).  The mapping to CDNA4 differs from the paper's one-thread-block-per-
// token Triton design:
//
//   * A workgroup has one wavefront per 32-column slab of n2.  Wave w owns
//     output columns j' in [32w, 32w+32).
//   * Contraction over axis 2, Z = X~ P2[:, slab]: MFMA 32x32x16 f16 with the
//     token tile read from LDS as the A operand (rows i, 8 consecutive j per
//     lane = one 16-byte LDS read) and the wave's P2 slab resident in VGPRs as
//     the B operand.  Result: lanes <-> j', registers <-> i.
//   * Contraction over axis 1, Y^T = Z^T P1: the fp32 accumulators of Z are
//     split into fp16 hi + lo parts (so the fp64 oracle's codes are reproduced)
//     and fed straight back as the A operand -- the accumulator layout of one
//     MFMA is a valid A/B operand layout for the next as long as the constant
//     operand (P1) is gathered with the same k-permutation, so there is no LDS
//     round trip.  Result: lanes <-> i', registers <-> j' with 4 consecutive j'
//     per register quad, i.e. 4 consecutive channels = 2 packed bytes per lane.
//   * absmax: in-lane over registers, wave butterfly, one float per wave in LDS.
//   * Codes are staged in LDS in channel order and written with 16-byte stores.
//   * Workgroups are persistent over tokens; the next token row is prefetched
//     into registers while the current one is in the MFMA pipe.
//
// tq_kernel is that kernel for n2 < 8, for INT4 rows that are only quantized, for MXFP4 rows whose staged values only fit in LDS
// without padding and where any_is_faster() says so; tq_any_kernel, further down, takes every other call that the specialised
// kernels (fq_tq_fast.hip) do not.
#include <type_traits>

#include "fq_internal.h"
#include "fq_device.h"

namespace fq {

__device__ __forceinline__ half8 split_hi(const float* z, float* resid) {
    // hi = fp16(z) rounded toward zero (never overflows to inf), resid = z - hi exactly
    half8 h;
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        auto pk = __builtin_amdgcn_cvt_pkrtz(z[k], z[k + 1]);
        h[k] = (_Float16)pk[0];
        h[k + 1] = (_Float16)pk[1];
        resid[k] = z[k] - (float)h[k];
        resid[k + 1] = z[k + 1] - (float)h[k + 1];
    }
    return h;
}

__device__ __forceinline__ half8 to_half8_rtz(const float* z) {
    half8 h;
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        auto pk = __builtin_amdgcn_cvt_pkrtz(z[k], z[k + 1]);
        h[k] = (_Float16)pk[0];
        h[k + 1] = (_Float16)pk[1];
    }
    return h;
}

// round-half-even of a value already clamped to [-8, 7], as a 4-bit two's complement nibble
__device__ __forceinline__ uint32_t nibble(float y, float inv) {
    float u = __builtin_fminf(__builtin_fmaxf(y * inv, -8.0f), 7.0f);
    return (uint32_t)(int)__builtin_rintf(u) & 0xFu;
}

// nibble() of eight values, the first in the lowest bits.  1.5 * 2^23 is added to the clamped quotient: the sum is rounded to whole
// numbers, ties to even, and its low bits hold 0x4B400000 + q, so the eight chain with shift-adds; the constant comes off and 8 goes on
// in every field at once (q + 8 = 0 .. 15: nothing borrows), and q + 8 is q's two's-complement nibble with the top bit turned.
// The clamp stands between product and sum, so that the quotient is rounded to fp32 like nibble()'s: the same code for every value.
template <typename F>
__device__ __forceinline__ uint32_t nibbles8(F&& y, float inv) {
    constexpr uint32_t kFix = 0x88888888u - 0x4B400000u * 0x11111111u;
    uint32_t b[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(y(k) * inv, -8.0f, 7.0f) + 12582912.0f);
    const uint32_t lo = lshl_add(lshl_add(b[3], 4, b[2]), 8, lshl_add(b[1], 4, b[0]));
    const uint32_t hi = lshl_add(lshl_add(b[7], 4, b[6]), 8, lshl_add(b[5], 4, b[4]));
    return (lshl_add(hi, 16, lo) + kFix) ^ 0x88888888u;
}

// exponent of an MXFP4 block from alpha max = m: floor(log2(m)) - 2, 0 for an all-zero block
__device__ __forceinline__ uint32_t mx_exponent(float m) {
    const uint32_t be = (__builtin_bit_cast(uint32_t, m) >> 23) & 0xffu;
    return be > 2 ? be - 2 : 0;
}
// eight elements, converted with the stored exponent (the conversion reads the exponent field of its scale operand only, and field 0
// means 2^-127)
__device__ __forceinline__ uint32_t mx_codes8(float4 a, float4 b, float scale) {
    uint32_t pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, a.x, a.y, scale, 0);
    pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, a.z, a.w, scale, 1);
    pk = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, b.x, b.y, scale, 2);
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(pk, b.z, b.w, scale, 3);
}

// MX: MXFP4 output for the shapes the specialised kernels do not take (n2 not a multiple of 32, where a block of 32
// consecutive channels straddles rows of X~ and column slabs): the token's Y is staged in LDS as fp32 in channel order,
// then one thread per block takes its 32 values, forms the shared exponent and converts.
// Up to 64 rows two waves per SIMD are asked for: in workgroups of up to four waves the compiler otherwise takes the registers
// of the second one (accumulation registers beside 256 others), and a CU holds half as many tokens.  Without / with the
// request, us: 60 x 88 4096 tokens 53.0 / 30.5, 60 x 120 57.4 / 33.6, 56 x 92 MXFP4 54.4 / 33.0, 60 x 24 at one to 4096 tokens
// 5 - 9 % (up to 32 rows -7 .. +18 %, larger workgroups the same code).  With more than 64 rows one wave per SIMD has to do.
template <int A, int B, bool P1LDS, bool MX = false>
__global__ __launch_bounds__(64 * B) __attribute__((amdgpu_waves_per_eu(A <= 2 ? 2 : 1))) void tq_kernel(TqDev p) {
    constexpr int NT = 64 * B;
    constexpr int PITCH = 32 * B + kLdsPad;      // halves per LDS row of the token tile
    constexpr int XS_HALVES = 32 * A * PITCH;
    constexpr int STAGE_BYTES = (MX ? 4096 : 512) * A * B;     // >= n / 2 bytes of codes, or 4 n bytes of fp32 values
    constexpr int NPRE = 2 * A;                  // 16-byte chunks per thread per token (upper bound)
    constexpr int KB2 = 2 * B;                   // K blocks (of 16) over j
    constexpr int KB1 = 2 * A;                   // K blocks (of 16) over i

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    _Float16* Xs = reinterpret_cast<_Float16*>(smem);
    uint8_t* stage = smem + XS_HALVES * 2;
    float* red = reinterpret_cast<float*>(stage + STAGE_BYTES);
    u32x4* P1s = reinterpret_cast<u32x4*>(red + 8);

    const int tid = threadIdx.x;
    const int l = tid & 63, w = tid >> 6, c = l & 31, h = l >> 5;
    const int n1 = p.n1, n2 = p.n2;
    const int n = n1 * n2;

    // ---- one-off: zero the tile (pad rows/columns stay zero for the whole kernel)
    for (int q = tid; q < XS_HALVES / 8; q += NT) reinterpret_cast<u32x4*>(Xs)[q] = u32x4{0u, 0u, 0u, 0u};

    // ---- one-off: the constant factors.  Every element is a 2-byte load of its own (any n1, n2 and alignment), and all of
    // them are requested before the first one is used: bounds are the buffer descriptor's (rows past the end, and columns
    // past it through an offset that is out of range, read as zero, and so does all of a left-out factor), so nothing branches
    // around a load.  (With a test around each load, and around each request of a token's chunks, every one of them cost its
    // own latency.  Before / now, us: 64 x 80 one token 12.9 / 6.2, 777 tokens 28.9 / 11.6, 16384 tokens 328 / 98, the last two
    // with the second wave per SIMD above; 64 x 172 14.8 / 9.3, 31.4 / 25.6, 389 / 319; 30 x 34 6.1 / 4.6, 7.3 / 6.2, 30.8 /
    // 26.6; 128 x 250 27.4 / 19.8, 148 / 112, 8192 tokens 1186 / 934.)
    constexpr int kOut = 0x40000000;             // byte offset past any factor
    const __amdgpu_buffer_rsrc_t p1buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.P1), 0, p.P1 ? n1 * n1 * 2 : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t p2buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(p.P2), 0, p.P2 ? n2 * n2 * 2 : 0, 0x00020000);
    auto element = [](__amdgpu_buffer_rsrc_t buf, int off) -> _Float16 {
        return __builtin_bit_cast(_Float16, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(buf, off, 0, 0));
    };

    // ---- this wave's P2 slab as B-operand fragments (lane <-> j', 8 k-values <-> j)
    half8 p2f[KB2];
    {
        const int jp = 32 * w + c;
        const int base = jp < n2 ? 2 * (8 * h * n2 + jp) : kOut;
#pragma unroll
        for (int kb = 0; kb < KB2; ++kb)
#pragma unroll
            for (int s = 0; s < 8; ++s) p2f[kb][s] = element(p2buf, base + 2 * (16 * kb + s) * n2);
        if (!p.P2) {                             // a left-out factor: identity
#pragma unroll
            for (int kb = 0; kb < KB2; ++kb)
#pragma unroll
                for (int s = 0; s < 8; ++s) p2f[kb][s] = (_Float16)(16 * kb + 8 * h + s == jp && jp < n2 ? 1.0f : 0.0f);
        }
    }
    // ---- P1 as B-operand fragments of the second contraction (lane <-> i'),
    // gathered with the k-permutation that the accumulator layout of the first one imposes:
    // K block kk, slot s of half-wave h  <->  i = 32(kk/2) + 8(2(kk%2) + s/4) + 4h + s%4.
    half8 p1f[P1LDS ? 1 : A][P1LDS ? 1 : KB1];
    if constexpr (P1LDS) {
#pragma unroll
        for (int e0 = 0; e0 < A * KB1 * 64; e0 += NT) {
            const int e = e0 + tid;
            if (A * KB1 % B != 0 && e >= A * KB1 * 64) break;
            const int ln = e & 63, kk = (e >> 6) % KB1, It = (e >> 6) / KB1;
            const int cc = ln & 31, hh = ln >> 5;
            const int ip = 32 * It + cc;
            const int i0 = 16 * kk + 4 * hh, base = ip < n1 ? 2 * (i0 * n1 + ip) : kOut;
            half8 f;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int i = 8 * (s >> 2) + (s & 3);
                const _Float16 v = element(p1buf, base + 2 * i * n1);
                f[s] = !p.P1 && i0 + i == ip && ip < n1 ? (_Float16)1.0f : v;
            }
            *reinterpret_cast<half8*>(&P1s[e]) = f;
        }
    } else {
#pragma unroll
        for (int It = 0; It < A; ++It)
#pragma unroll
            for (int kk = 0; kk < KB1; ++kk) {
                const int ip = 32 * It + c;
                const int i0 = 16 * kk + 4 * h, base = ip < n1 ? 2 * (i0 * n1 + ip) : kOut;
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int i = 8 * (s >> 2) + (s & 3);
                    const _Float16 v = element(p1buf, base + 2 * i * n1);
                    p1f[It][kk][s] = !p.P1 && i0 + i == ip && ip < n1 ? (_Float16)1.0f : v;
                }
            }
    }

    // ---- per-thread LDS destinations of the 16-byte chunks of a token row (fixed for all tokens)
    const int nchunks = n >> 3;
    int xoff[NPRE];
#pragma unroll
    for (int k = 0; k < NPRE; ++k) {
        const int q = tid + k * NT;
        const int e = q * 8;
        const int i = e / n2;
        xoff[k] = (p.vec8 && q < nchunks) ? i * PITCH + (e - i * n2) : -1;
    }

    auto issue = [&](int64_t t, u32x4 (&pre)[NPRE]) {
        const u32x4* src = reinterpret_cast<const u32x4*>(p.x + t * p.x_stride);
#pragma unroll
        for (int k = 0; k < NPRE; ++k)
            pre[k] = __builtin_nontemporal_load(src + (tid + k * NT < nchunks ? tid + k * NT : nchunks - 1));   // past the end the last chunk again: no branch
    };
    auto commit = [&](const u32x4 (&pre)[NPRE]) {
#pragma unroll
        for (int k = 0; k < NPRE; ++k)
            if (xoff[k] >= 0) *reinterpret_cast<u32x4*>(Xs + xoff[k]) = pre[k];
    };
    // rows that cannot move in 16-byte chunks (n2 not a multiple of 8, or an unaligned x): pairs of halves, requested
    // into registers before the MFMA work like the chunks above (n / 2 pairs over the workgroup: at most 8 A per thread);
    // a pair never straddles a row (n2 is even), and its row is umulhi(2 u, magic) with the magic divisor from the host
    constexpr int NPS = 8 * A;
    static_assert(NPS == 4 * NPRE, "the pairs use the registers of the chunks");
    auto issue_slow = [&](int64_t t, u32x4 (&pre)[NPRE]) {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(p.x + t * p.x_stride);
#pragma unroll
        for (int k = 0; k < NPS; ++k) {
            const int u = tid + k * NT;
            pre[k >> 2][k & 3] = src[u < (n >> 1) ? u : (n >> 1) - 1];
        }
    };
    auto commit_slow = [&](const u32x4 (&pre)[NPRE]) {
#pragma unroll
        for (int k = 0; k < NPS; ++k) {
            const int u = tid + k * NT;
            if (u < (n >> 1)) {
                const int e = 2 * u, i = (int)__umulhi((uint32_t)e, p.n2_magic);
                *reinterpret_cast<uint32_t*>(Xs + i * PITCH + (e - i * n2)) = pre[k >> 2][k & 3];
            }
        }
    };

    __syncthreads();   // zero fill (and P1s) complete before the first tile lands
    u32x4 pre[NPRE];
    int64_t t = blockIdx.x;
    if (t < p.T) {
        if (p.vec8) { issue(t, pre); commit(pre); } else { issue_slow(t, pre); commit_slow(pre); }
    }
    __syncthreads();

    for (; t < p.T; t += gridDim.x) {
        const int64_t tn = t + gridDim.x;
        const bool have_next = tn < p.T;
        if (have_next) {
            if (p.vec8) issue(tn, pre); else issue_slow(tn, pre);
        }

        f32x16 acc2[A];
#pragma unroll
        for (int It = 0; It < A; ++It)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc2[It][r] = 0.0f;

#pragma unroll
        for (int I = 0; I < A; ++I) {
            // Z[32I .. 32I+31, slab] = X~[32I.., :] P2[:, slab]
            f32x16 acc1;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc1[r] = 0.0f;
            const _Float16* arow = Xs + (32 * I + c) * PITCH + 8 * h;
#pragma unroll
            for (int kb = 0; kb < KB2; ++kb) {
                if (16 * kb < n2) {
                    const half8 a = *reinterpret_cast<const half8*>(arow + 16 * kb);
                    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, p2f[kb], acc1, 0, 0, 0);
                }
            }
            // Y^T[slab, :] += Z^T[slab, K block] P1[K block, :], hi and lo parts of Z
#pragma unroll
            for (int kq = 0; kq < 2; ++kq) {
                const int kk = 2 * I + kq;
                if (16 * kk < n1) {
                    float z[8], resid[8];
#pragma unroll
                    for (int s = 0; s < 8; ++s) z[s] = acc1[8 * kq + s];
                    const half8 zh = split_hi(z, resid);
                    const half8 zl = to_half8_rtz(resid);
#pragma unroll
                    for (int It = 0; It < A; ++It) {
                        half8 b;
                        if constexpr (P1LDS) b = *reinterpret_cast<const half8*>(&P1s[(It * KB1 + kk) * 64 + l]);
                        else b = p1f[It][kk];
                        acc2[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zh, b, acc2[It], 0, 0, 0);
                        acc2[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zl, b, acc2[It], 0, 0, 0);
                    }
                }
            }
        }

        const float clipv = p.clip[p.clip_mode ? t : 0];
        _Float16 sh = (_Float16)0.0f;
        if constexpr (MX) {
            __syncthreads();   // (A) all waves are done reading the token tile
            float* stagef = reinterpret_cast<float*>(stage);
#pragma unroll
            for (int It = 0; It < A; ++It) {
                const int ip = 32 * It + c;
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int jp = 32 * w + 8 * g + 4 * h + k;
                        if (ip < n1 && jp < n2) stagef[ip * n2 + jp] = acc2[It][4 * g + k];
                    }
            }
        } else {
        // ---- per-token absmax (padded rows/columns are exact zeros)
        float m = 0.0f;
#pragma unroll
        for (int It = 0; It < A; ++It)
#pragma unroll
            for (int r = 0; r < 16; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(acc2[It][r]));
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off));
        if (l == 0) red[w] = m;
        __syncthreads();   // (A) all waves are also done reading the token tile
#pragma unroll
        for (int b = 0; b < B; ++b) m = __builtin_fmaxf(m, red[b]);

        sh = (_Float16)(clipv * m / 7.0f);   // round-to-nearest-even to fp16
        const float s = (float)sh;
        const float inv = (s > 0.0f && s <= 65504.0f) ? 1.0f / s : 0.0f;

        // ---- round, clamp, pack 4 consecutive channels per register quad, stage in channel order
#pragma unroll
        for (int It = 0; It < A; ++It) {
            const int ip = 32 * It + c;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int jp = 32 * w + 8 * g + 4 * h;
                if (ip < n1 && jp < n2) {
                    const uint32_t pk = nibble(acc2[It][4 * g + 0], inv) | (nibble(acc2[It][4 * g + 1], inv) << 4) |
                                        (nibble(acc2[It][4 * g + 2], inv) << 8) | (nibble(acc2[It][4 * g + 3], inv) << 12);
                    const int byte = (ip * n2 + jp) >> 1;
                    if ((n2 & 3) == 0) {
                        *reinterpret_cast<uint16_t*>(stage + byte) = (uint16_t)pk;
                    } else {
                        stage[byte] = (uint8_t)pk;
                        if (jp + 2 < n2) stage[byte + 1] = (uint8_t)(pk >> 8);
                    }
                }
            }
        }
        }
        // ---- next token tile into LDS (its loads were issued before the MFMA work)
        if (have_next) {
            if (p.vec8) commit(pre); else commit_slow(pre);
        }
        __syncthreads();   // (B) staged codes and next tile visible

        uint8_t* dst = p.out_codes + t * (int64_t)(n >> 1);
        if constexpr (MX) {
            // Block b = channels 32 b .. 32 b + 31: exponent floor(log2(alpha max)) - 2 (0 for an all-zero block), elements
            // converted with the stored exponent (the conversion reads the exponent field of its scale operand only,
            // and field 0 means 2^-127); 16 bytes of codes per block, exponents row-major or in the product's tile order
            const float* stagef = reinterpret_cast<const float*>(stage);
            uint8_t* exps = reinterpret_cast<uint8_t*>(p.out_scales);
            const int nblk = n >> 5;
            for (int b = tid; b < nblk; b += NT) {
                float y[32];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float4 v = reinterpret_cast<const float4*>(stagef + 32 * b)[k];
                    y[4 * k] = v.x; y[4 * k + 1] = v.y; y[4 * k + 2] = v.z; y[4 * k + 3] = v.w;
                }
                float bm = 0.0f;
#pragma unroll
                for (int k = 0; k < 32; ++k) bm = __builtin_fmaxf(bm, __builtin_fabsf(y[k]));
                const uint32_t e = mx_exponent(bm * clipv);
                const float scale = __builtin_bit_cast(float, e << 23);
                u32x4 o;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    o[d] = mx_codes8(float4{y[8 * d], y[8 * d + 1], y[8 * d + 2], y[8 * d + 3]}, float4{y[8 * d + 4], y[8 * d + 5], y[8 * d + 6], y[8 * d + 7]}, scale);
                reinterpret_cast<u32x4*>(dst)[b] = o;
                if (p.mx_tiled) exps[((((t >> 7) * (int64_t)(n >> 8) + (b >> 3)) * 128 + (t & 127)) << 3) + (b & 7)] = (uint8_t)e;
                else exps[t * (int64_t)nblk + b] = (uint8_t)e;
            }
        } else {
            if (p.out_vec16) {
                for (int q = tid; q < (n >> 5); q += NT)
                    __builtin_nontemporal_store(reinterpret_cast<const u32x4*>(stage)[q], reinterpret_cast<u32x4*>(dst) + q);
            } else {
                for (int q = tid; q < (n >> 1); q += NT) dst[q] = stage[q];
            }
            if (tid == 0) p.out_scales[t] = sh;
        }
    }
}

// where P1's fragment table starts behind a token tile and the staged values of MXFP4, and the bytes in all (the factors' may be more)
template <int A, int B>
__host__ __device__ constexpr int any_mx_r0(int n) {
    return (FastLds<A, B>::XS_BYTES + 64 + n / 32 * 144 + 15) & ~15;
}
template <int A, int B>
constexpr int any_mx_lds(int n) {
    return (cmax(any_mx_r0<A, B>(n) + FastLds<A, B>::P1S_BYTES, FastLds<A, B>::STG_BYTES) + 15) & ~15;
}

// Any pair of factors (n2 >= 8; INT4: either may be left out: identity): the plain loop of the specialised kernels (fq_tq_fast.hip:
// same wave mapping and contractions) for right factors that are not a multiple of 32 and rows that do not
// start on 16 bytes.  What is different: the factors' LDS copies are padded with zeros to whole tiles; a token's row is requested in
// flat 16-byte chunks wherever they start (dword-aligned), and a chunk that straddles two rows of X~ goes into LDS in pieces of 8
// or 4 bytes, whichever divides n2; the codes are rounded as in the kernel above (the same bytes: which of the two runs must not show)
// and a lane's 8 bytes of them are stored as far as the row goes.  Against the kernel above (2-byte loads of the factors, rounding and
// packing in 8 instructions per value, here 4, codes staged in LDS), us:
// 64 x 80 at 64 tokens 6.8 / 5.1, 777 11.2 / 8.6, 2048 17.3 / 13.0, 16384 97 / 74; 64 x 172 10.2 / 7.7 (64), 45 / 30 (2048), 318 / 181
// (16384); 45 x 90 21.6 / 13.9 (2048); 97 x 98 60.9 / 36.8 (2048); 128 x 250 939 / 337 (8192); 16 x 18 7.2 / 6.1 (4096).  (Rounding by
// v_cvt_pknorm_i16, 2 instructions per value as in the specialised kernels, moves ties and what lies within 2e-6 of one:
// 64 x 80 12.4 at 2048, 68 at 16384.)
// MX: MXFP4 output for the same shapes: Y is staged in LDS in channel order, as fp32 with 4 words of padding per block of 32 (reads of
// consecutive blocks spread over the banks), then one thread per block forms the exponent and converts.  Same bytes as the kernel
// above; against it, us: 64 x 80 at 64 tokens 7.6 / 5.8, 777 14.6 / 9.8, 2048 23.7 / 14.7, 16384 142 / 80; 64 x 172 10.3 / 8.6 (64), 41.5 / 29.8 (2048),
// 142 / 96 (8192); 48 x 112 26.4 / 17.3 (2048); 96 x 90 41.6 / 25.6; 128 x 100 61.3 / 45.5; 32 x 18 5.6 / 5.3.
template <int A, int B, bool MX>
__global__ __launch_bounds__(64 * B) __attribute__((amdgpu_waves_per_eu(2))) void tq_any_kernel(TqDev p) {
    using L = FastLds<A, B>;
    constexpr int NT = 64 * B, N2 = 32 * B, PITCH = L::PITCH, PW = 32 * A;
    constexpr int KB1 = 2 * A, KB2 = 2 * B, NPRE = 2 * A;
    constexpr bool P1LDS = L::P1LDS, DEEP = NPRE <= 4;
    typedef u32x4 __attribute__((aligned(4))) chunk_t;               // token rows start on dwords,
    typedef u32x4 __attribute__((aligned(2))) chunk2_t;              // factors on halves
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    _Float16* Xs = reinterpret_cast<_Float16*>(smem);
    float* red = reinterpret_cast<float*>(smem + L::XS_BYTES);
    u32x4* P1s = reinterpret_cast<u32x4*>(smem + (MX ? any_mx_r0<A, B>(p.n1 * p.n2) : L::R0));
    float* stagef = reinterpret_cast<float*>(smem + L::XS_BYTES + 64);      // MX, behind the token tile
    _Float16* P1flat = reinterpret_cast<_Float16*>(smem);
    _Float16* P2flat = reinterpret_cast<_Float16*>(smem + L::P1FLAT_BYTES);
    const int tid = threadIdx.x, l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n1 = p.n1, n2 = p.n2, n = n1 * n2;
    const int piece = (n2 & 7) == 0 ? 8 : (n2 & 3) == 0 ? 4 : 2;     // halves that never straddle a row

    // ---- token rows: chunk k of this thread starts at half e, the last one early enough to end with the row; chunks past it are
    // the last one again (same bytes to the same place), so that nothing branches
    auto first_half = [&](int k) { return 8 * (tid + k * NT) < n - 8 ? 8 * (tid + k * NT) : n - 8; };
    uint32_t xput[NPRE];                         // LDS offset in halves (below 2^16), halves left in its row of X~ (16 bits up)
#pragma unroll
    for (int k = 0; k < NPRE; ++k) {
        const int e = first_half(k), i = (int)__umulhi((uint32_t)e, p.n2_magic), col = e - i * n2;
        xput[k] = (uint32_t)(i * PITCH + col) | (uint32_t)(n2 - col) << 16;
    }
    auto issue = [&](int64_t t, u32x4 (&pre)[NPRE]) {
        const _Float16* row = p.x + t * p.x_stride;
#pragma unroll
        for (int k = 0; k < NPRE; ++k) pre[k] = __builtin_nontemporal_load(reinterpret_cast<const chunk_t*>(row + first_half(k)));
    };
    // chunks to where `where` (as above) says in a matrix of `pitch`
    auto put = [&](_Float16* dst, int pitch, auto& where, auto& v, auto cnt) {
        constexpr int N = decltype(cnt)::value;
        if (piece == 8) {
#pragma unroll
            for (int k = 0; k < N; ++k) *reinterpret_cast<u32x4*>(dst + (where[k] & 0xFFFFu)) = v[k];
        } else if (piece == 4) {
#pragma unroll
            for (int k = 0; k < N; ++k)
#pragma unroll
                for (int d = 0; d < 2; ++d)
                    *reinterpret_cast<uint2*>(dst + (int)(where[k] & 0xFFFFu) + 4 * d + (4 * d >= (int)(where[k] >> 16) ? pitch - n2 : 0)) = uint2{v[k][2 * d], v[k][2 * d + 1]};
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k)
#pragma unroll
                for (int d = 0; d < 4; ++d) *reinterpret_cast<uint32_t*>(dst + (int)(where[k] & 0xFFFFu) + 2 * d + (2 * d >= (int)(where[k] >> 16) ? pitch - n2 : 0)) = v[k][d];
        }
    };
    auto commit = [&](const u32x4 (&pre)[NPRE]) { put(Xs, PITCH, xput, pre, std::integral_constant<int, NPRE>{}); };
    u32x4 pre0[NPRE], pre1[DEEP ? NPRE : 1];
    int64_t t = blockIdx.x;
    const int64_t G = gridDim.x;
    issue(t, pre0);

    // ---- the factors: requested, then their LDS image zeroed, then put into it; fragments by transposing reads
    half8 p2f[KB2];
    half8 p1f[P1LDS ? 1 : A][P1LDS ? 1 : KB1];
    constexpr int NP1S = P1LDS ? (A * KB1 * 64 + NT - 1) / NT : 1;
    half8 p1s[NP1S];                             // on their way from the staging area into the table
    constexpr int N1P = (PW * PW / 2 + NT - 1) / NT, B1 = N1P < 16 ? N1P : 16;          // pairs of P1 per thread, and in flight
    constexpr int N2C = (L::P2ROWS * N2 / 8 + NT - 1) / NT;                            // chunks of P2 per thread and pass
#pragma unroll
    for (int pass = 0; pass < L::P2PASSES; ++pass) {
        const int r0 = pass * L::P2ROWS, rows = n2 - r0 < L::P2ROWS ? n2 - r0 : L::P2ROWS;    // rows of this pass (at least one)
        const int last2 = rows * n2 - 8;                              // a left-out factor reads the first bytes of x, for nothing
        const _Float16* s2 = p.P2 ? p.P2 + r0 * n2 : p.x;
        u32x4 v2[N2C];
        int e2[N2C];
#pragma unroll
        for (int k = 0; k < N2C; ++k) {
            const int q = 8 * (tid + k * NT);
            e2[k] = q < last2 ? q : last2;
            v2[k] = *reinterpret_cast<const chunk2_t*>(s2 + (p.P2 ? e2[k] : 0));
        }
        const int n1sq = n1 * n1, last1 = p.P1 && n1 > 1 ? (n1sq >> 1) - 1 : 0;
        const _Float16* s1 = p.P1 && n1 > 1 ? p.P1 : p.x;
        auto load1 = [&](int base, uint32_t (&v)[B1]) {
            typedef uint32_t __attribute__((aligned(2))) pair_t;
#pragma unroll
            for (int k = 0; k < B1; ++k) {
                const int u = tid + (base + k) * NT;
                v[k] = *reinterpret_cast<const pair_t*>(s1 + 2 * (u < last1 ? u : last1));
            }
        };
        uint32_t v1[B1];
        if (pass == 0) {
            load1(0, v1);
            if constexpr (DEEP) issue(t + G < p.T ? t + G : p.T - 1, pre1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (pass > 0) __syncthreads();                                // previous pass fully consumed
        for (int q = tid + (pass > 0 ? L::P1FLAT_BYTES / 16 : 0); q < L::STG_BYTES / 16; q += NT) reinterpret_cast<u32x4*>(smem)[q] = u32x4{0u, 0u, 0u, 0u};
        __syncthreads();
        if (p.P2) {
            uint32_t put2[N2C];
#pragma unroll
            for (int k = 0; k < N2C; ++k) {
                const int i = (int)__umulhi((uint32_t)e2[k], p.n2_magic), col = e2[k] - i * n2;
                put2[k] = (uint32_t)(i * N2 + col) | (uint32_t)(n2 - col) << 16;
            }
            put(P2flat, N2, put2, v2, std::integral_constant<int, N2C>{});
        } else {
            for (int r = tid; r < rows; r += NT) P2flat[r * N2 + r0 + r] = (_Float16)1.0f;
        }
        if (pass == 0) {
            uint16_t* d1 = reinterpret_cast<uint16_t*>(P1flat);
            if (!p.P1) {
                for (int r = tid; r < n1; r += NT) P1flat[r * PW + r] = (_Float16)1.0f;
            } else {
                if (n1 > 1) {
#pragma unroll 1
                    for (int base = 0; base < N1P; base += B1) {
                        if (base > 0) load1(base, v1);
#pragma unroll
                        for (int k = 0; k < B1; ++k) {                // each half on its own: a pair straddles two rows when n1 is odd
                            const int u = tid + (base + k) * NT, f = 2 * (u < last1 ? u : last1);
                            const int row = (int)__umulhi((uint32_t)f, p.n1_magic), col = f - row * n1, a0 = row * PW + col;
                            d1[a0] = (uint16_t)v1[k];
                            d1[a0 + 1 + (col + 1 == n1 ? PW - n1 : 0)] = (uint16_t)(v1[k] >> 16);
                        }
                    }
                }
                if ((n1 & 1) && tid == 0) d1[(n1 - 1) * PW + n1 - 1] = reinterpret_cast<const uint16_t*>(p.P1)[n1sq - 1];
            }
        }
        __syncthreads();
#pragma unroll
        for (int kb = pass * (L::P2ROWS / 16); kb < (pass + 1) * (L::P2ROWS / 16); ++kb)
            p2f[kb] = lds_column8(P2flat, N2, 16 * kb - r0 + 8 * h, 4, 32 * w + (c & 16), l & 15);
        if (pass == 0) {
            if constexpr (P1LDS) {
#pragma unroll
                for (int k = 0; k < NP1S; ++k) {
                    const int e = tid + k * NT < A * KB1 * 64 ? tid + k * NT : 0;
                    const int kk = (e >> 6) % KB1, It = (e >> 6) / KB1;
                    p1s[k] = lds_column8(P1flat, PW, 32 * (kk >> 1) + 16 * (kk & 1) + 4 * h, 8, 32 * It + (c & 16), l & 15);
                }
            } else {
#pragma unroll
                for (int It = 0; It < A; ++It)
#pragma unroll
                    for (int kk = 0; kk < KB1; ++kk) p1f[It][kk] = lds_column8(P1flat, PW, 32 * (kk >> 1) + 16 * (kk & 1) + 4 * h, 8, 32 * It + (c & 16), l & 15);
            }
        }
    }
    __syncthreads();   // the staging area becomes the token tile; what no token's row covers stays zero
    for (int q = tid; q < L::XS_BYTES / 16; q += NT) reinterpret_cast<u32x4*>(smem)[q] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (P1LDS) {
#pragma unroll
        for (int k = 0; k < NP1S; ++k)
            if (tid + k * NT < A * KB1 * 64) *reinterpret_cast<half8*>(&P1s[tid + k * NT]) = p1s[k];
    }
    __syncthreads();
    commit(pre0);
    __syncthreads();

    auto body = [&](int64_t t, u32x4 (&pre_next)[NPRE], u32x4 (&pre_far)[NPRE]) __attribute__((always_inline)) {
        const int64_t tf = t + (DEEP ? 2 : 1) * G;
        issue(tf < p.T ? tf : p.T - 1, pre_far);
        __builtin_amdgcn_sched_barrier(0);
        const float clipv = p.clip[p.clip_mode ? t : 0];
        f32x16 acc2[A];
#pragma unroll
        for (int It = 0; It < A; ++It)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc2[It][r] = 0.0f;
#pragma unroll
        for (int I0 = 0; I0 < A; I0 += 2) {      // row tiles in pairs, so that consecutive MFMAs are independent
            constexpr int NI_MAX = 2;
            const int ni = A - I0 < NI_MAX ? A - I0 : NI_MAX;
            f32x16 acc1[NI_MAX];
#pragma unroll
            for (int d = 0; d < NI_MAX; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc1[d][r] = 0.0f;
            const _Float16* arow = Xs + (32 * I0 + c) * PITCH + 8 * h;
#pragma unroll
            for (int kb = 0; kb < KB2; ++kb)
#pragma unroll
                for (int d = 0; d < NI_MAX; ++d)
                    if (d < ni) {
                        const half8 a = *reinterpret_cast<const half8*>(arow + d * 32 * PITCH + 16 * kb);
                        acc1[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, p2f[kb], acc1[d], 0, 0, 0);
                    }
#pragma unroll
            for (int d = 0; d < NI_MAX; ++d)
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    const int kk = 2 * (I0 + d) + kq;
                    if (d < ni && (A < 4 || 16 * kk < n1)) {
                        half8 zh, zl, b[A];
                        split_hi_lo(acc1[d], 8 * kq, zh, zl);
#pragma unroll
                        for (int It = 0; It < A; ++It) {
                            if constexpr (P1LDS) b[It] = *reinterpret_cast<const half8*>(&P1s[(It * KB1 + kk) * 64 + l]);
                            else b[It] = p1f[It][kk];
                        }
#pragma unroll
                        for (int It = 0; It < A; ++It) acc2[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zh, b[It], acc2[It], 0, 0, 0);
#pragma unroll
                        for (int It = 0; It < A; ++It) acc2[It] = __builtin_amdgcn_mfma_f32_32x32x16_f16(zl, b[It], acc2[It], 0, 0, 0);
                    }
                }
        }
        if constexpr (MX) {
            __syncthreads();                     // (A) every wave is done reading the token tile, and the values staged before
            const int pair = n2 & 2;             // runs of 4 channels stay inside a block if n2 is a multiple of 4, else runs of 2
            int ro = c * n2 + 32 * w + 4 * h;
            asm volatile("" : "+v"(ro));         // opaque: the 8 A offsets below are formed here, not held across the tokens (they spill)
#pragma unroll
            for (int It = 0; It < A; ++It) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int jp = 32 * w + 8 * g + 4 * h, e = ro + 32 * It * n2 + 8 * g;
                    if (32 * It + c < n1 && jp < n2) {
                        if (pair == 0) {
                            *reinterpret_cast<float4*>(stagef + e + 4 * (e >> 5)) = float4{acc2[It][4 * g], acc2[It][4 * g + 1], acc2[It][4 * g + 2], acc2[It][4 * g + 3]};
                        } else {
                            *reinterpret_cast<float2*>(stagef + e + 4 * (e >> 5)) = float2{acc2[It][4 * g], acc2[It][4 * g + 1]};
                            if (jp + 2 < n2) *reinterpret_cast<float2*>(stagef + e + 2 + 4 * ((e + 2) >> 5)) = float2{acc2[It][4 * g + 2], acc2[It][4 * g + 3]};
                        }
                    }
                }
            }
            if (t + G < p.T) commit(pre_next);   // (the last token does not wait for its re-read)
            __syncthreads();                     // (B) staged values and the next tile are visible
            uint8_t* exps = reinterpret_cast<uint8_t*>(p.out_scales);
            const int nblk = n >> 5;
            for (int b = tid; b < nblk; b += NT) {
                const float4* src = reinterpret_cast<const float4*>(stagef + 36 * b);
                float bm = 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float4 v = src[k];
                    bm = __builtin_fmaxf(__builtin_fmaxf(bm, __builtin_fabsf(v.x)), __builtin_fabsf(v.y));
                    bm = __builtin_fmaxf(__builtin_fmaxf(bm, __builtin_fabsf(v.z)), __builtin_fabsf(v.w));
                }
                asm volatile("" ::: "memory");   // read again rather than held: 32 registers beside the factors' fragments spill
                const uint32_t e = mx_exponent(bm * clipv);
                const float scale = __builtin_bit_cast(float, e << 23);
                u32x4 o;
#pragma unroll
                for (int d = 0; d < 4; ++d) o[d] = mx_codes8(src[2 * d], src[2 * d + 1], scale);
                reinterpret_cast<u32x4*>(p.out_codes + t * (int64_t)(n >> 1))[b] = o;
                if (p.mx_tiled) exps[((((t >> 7) * (int64_t)(n >> 8) + (b >> 3)) * 128 + (t & 127)) << 3) + (b & 7)] = (uint8_t)e;
                else exps[t * (int64_t)nblk + b] = (uint8_t)e;
            }
            return;
        }
        float m = 0.0f;                          // padded rows and columns are exact zeros
#pragma unroll
        for (int It = 0; It < A; ++It)
#pragma unroll
            for (int r = 0; r < 16; ++r) m = __builtin_fmaxf(m, __builtin_fabsf(acc2[It][r]));
        m = wave_max(m);
        if (l == 0) red[w] = m;
        __syncthreads();                         // (A) every wave is also done reading the token tile
#pragma unroll
        for (int b = 0; b < B; ++b) m = __builtin_fmaxf(m, red[b]);
        const _Float16 sh = (_Float16)(clipv * m / 7.0f);             // round-to-nearest-even to fp16
        const float s = (float)sh;
        const float inv = (s > 0.0f && s <= 65504.0f) ? 1.0f / s : 0.0f;
        uint8_t* row_out = p.out_codes + t * (int64_t)(n >> 1);
        const int left = n2 - 32 * w - 16 * h;   // channels of this lane's 16 that exist
#pragma unroll
        for (int It = 0; It < A; ++It) {
            uint32_t Wq[2];
#pragma unroll
            for (int mm = 0; mm < 2; ++mm) Wq[mm] = nibbles8([&](int k) { return acc2[It][8 * mm + k]; }, inv);
            const auto sw = __builtin_amdgcn_permlane32_swap(Wq[0], Wq[1], false, false);
            uint2 o;
            o.x = __builtin_amdgcn_perm(sw[1], sw[0], 0x05040100u);
            o.y = __builtin_amdgcn_perm(sw[1], sw[0], 0x07060302u);
            const int ip = 32 * It + c;
            if (ip < n1 && left > 0) {
                typedef unsigned int __attribute__((ext_vector_type(2), aligned(1))) codes8_t;
                typedef uint32_t __attribute__((aligned(1))) codes4_t;
                uint8_t* dst = row_out + ((ip * n2 + 32 * w + 16 * h) >> 1);
                if (left >= 16) {
                    *reinterpret_cast<codes8_t*>(dst) = codes8_t{o.x, o.y};
                } else {                          // 1 .. 7 bytes
                    uint32_t r = o.x;
                    if (left >= 8) {
                        *reinterpret_cast<codes4_t*>(dst) = o.x;
                        dst += 4;
                        r = o.y;
                    }
                    for (int b = 0; b < (left & 7) >> 1; ++b) dst[b] = (uint8_t)(r >> (8 * b));
                }
            }
        }
        p.out_scales[t] = sh;                    // every lane writes the same two bytes
        if (t + G >= p.T) return;                // (not waiting for the re-read last row)
        commit(pre_next);
        __syncthreads();                         // (B) the next tile is visible
    };
    if constexpr (DEEP) {
        while (true) {
            body(t, pre1, pre0);
            t += G;
            if (t >= p.T) break;
            body(t, pre0, pre1);
            t += G;
            if (t >= p.T) break;
        }
    } else {
        for (; t < p.T; t += G) body(t, pre0, pre0);
    }
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------
using KernelFn = void (*)(TqDev);
constexpr int kLdsMax = 160 * 1024;

template <int A, int B>
static constexpr KernelFn kernel_for() { return &tq_kernel<A, B, (A >= 3)>; }

static KernelFn kernel_table(int A, int B) {
    static const KernelFn tab[4][8] = {
        {kernel_for<1, 1>(), kernel_for<1, 2>(), kernel_for<1, 3>(), kernel_for<1, 4>(), kernel_for<1, 5>(), kernel_for<1, 6>(), kernel_for<1, 7>(), kernel_for<1, 8>()},
        {kernel_for<2, 1>(), kernel_for<2, 2>(), kernel_for<2, 3>(), kernel_for<2, 4>(), kernel_for<2, 5>(), kernel_for<2, 6>(), kernel_for<2, 7>(), kernel_for<2, 8>()},
        {kernel_for<3, 1>(), kernel_for<3, 2>(), kernel_for<3, 3>(), kernel_for<3, 4>(), kernel_for<3, 5>(), kernel_for<3, 6>(), kernel_for<3, 7>(), kernel_for<3, 8>()},
        {kernel_for<4, 1>(), kernel_for<4, 2>(), kernel_for<4, 3>(), kernel_for<4, 4>(), kernel_for<4, 5>(), kernel_for<4, 6>(), kernel_for<4, 7>(), kernel_for<4, 8>()},
    };
    return tab[A - 1][B - 1];
}

// LDS of tq_kernel with A row tiles and B slabs, and with MXFP4 output; what that does not leave room for is not supported
__host__ __device__ constexpr int generic_lds(int A, int B) { return 32 * A * (32 * B + kLdsPad) * 2 + 512 * A * B + 32 + (A >= 3 ? A * 2 * A * 64 * 16 : 0); }
__host__ __device__ constexpr int mx_staged_lds(int A, int B) { return generic_lds(A, B) + (4096 - 512) * A * B; }

struct AnyVariant {
    KernelFn fn;                                 // null: MXFP4 rows that neither kernel has room for
    int lds;
};
template <int A, int B>
static AnyVariant any_variant_ab(bool mx, int n) {
    if (mx) {
        if constexpr (mx_staged_lds(A, B) > kLdsMax) return {nullptr, kLdsMax + 1};
        else return {&tq_any_kernel<A, B, true>, any_mx_lds<A, B>(n)};
    }
    return {&tq_any_kernel<A, B, false>, FastLds<A, B>::TOTAL};
}
template <int A>
static AnyVariant any_variant_a(int B, bool mx, int n) {
    switch (B) {
        case 1: return any_variant_ab<A, 1>(mx, n);
        case 2: return any_variant_ab<A, 2>(mx, n);
        case 3: return any_variant_ab<A, 3>(mx, n);
        case 4: return any_variant_ab<A, 4>(mx, n);
        case 5: return any_variant_ab<A, 5>(mx, n);
        case 6: return any_variant_ab<A, 6>(mx, n);
        case 7: return any_variant_ab<A, 7>(mx, n);
        default: return any_variant_ab<A, 8>(mx, n);
    }
}
static AnyVariant any_variant(int n1, int n2, bool mx) {
    const int A = (n1 + 31) / 32, B = (n2 + 31) / 32;
    switch (A) {
        case 1: return any_variant_a<1>(B, mx, n1 * n2);
        case 2: return any_variant_a<2>(B, mx, n1 * n2);
        case 3: return any_variant_a<3>(B, mx, n1 * n2);
        default: return any_variant_a<4>(B, mx, n1 * n2);
    }
}
// Whether tq_any_kernel is the faster one of the two general kernels, which give the same bytes.  tq_kernel / tq_any_kernel in us, tokens in
// parentheses (CUs: 256); the lines are where two thousand launches per format over all (A, B) crossed, and no launch measured is more
// than 5 % slower than with tq_kernel alone.  From two row tiles and two slabs on it is (0.5 .. 0.97 of the time), but for launches that tq_kernel, whose
// tiles are smaller in LDS, finishes in one round of workgroups and tq_any_kernel in two:
//   four row tiles x two slabs INT4, three x two MXFP4, two workgroups of tq_kernel per CU: 128 x 36 12.8 / 11.3 (256), 13.1 / 14.0 (512), 18.4 / 18.2 (640);
//     96 x 34 MXFP4 9.2 / 8.5 (256), 9.6 / 10.3 (512), 13.2 / 10.9 (640);
//   one slab x four row tiles, three workgroups (MXFP4 two): 128 x 20 15.8 / 15.9 (512), 15.9 / 18.6 (640), 20.6 / 18.7 (900); MXFP4 16.0 / 16.5 (384), 21.1 / 19.8 (640).
// One slab x two row tiles: a row has few values, and the prologue (two staging passes through LDS) is made up for by many tokens (not with
// n2 = 8) or, in INT4, by rows that tq_kernel loads in pairs of halves: 64 x 28 5.9 / 5.7 (64), 6.6 / 6.2 (1024); 64 x 16 5.2 / 5.5 (64), 7.1 / 7.5 (2048),
// 23.1 / 20.7 (16384); 33 x 16 10.1 / 10.4 (4311); 48 x 8 19.1 / 19.7 (16384); MXFP4 64 x 16 4.8 / 5.4 (64), 48 x 12 9.4 / 10.3 (4192), 50 x 16 23.7 / 18.7 (13869).
// One row tile, INT4: but for the longest prologue with one token per CU (16 x 250 8.0 / 8.3 (64), 10.5 / 10.1 (512)).
// One row tile, MXFP4: tq_kernel has more workgroups per CU up to four slabs, and one from there on.
//   Up to four slabs, n2 % 8 != 0 (values move in pieces of 8 or 16 bytes): 16 x 66 4.3 / 4.4 (64), 11.5 / 14.1 (4096).
//   n2 % 8 == 0: tq_any_kernel moves and stages whole tiles, so it gains where they are filled: 32 x 80 (0.83) 5.8 / 4.7 (300), 60 / 44 (16384);
//     24 x 80 (0.63) 48 / 41, 12 x 72 (0.28) 5.3 / 5.7 (600), 28 / 40 (16384); one slab 32 x 16 (0.5) 14.9 / 12.3; fewer tokens 24 x 72 (0.56) 8.4 / 8.2 (2048), 36 / 41 (16384),
//     two slabs 12 x 40 6.5 / 5.6 (2048), 17 / 22 (16384).
//   Five slabs on: 16 x 134 5.7 / 6.2 (256), 9.5 / 7.3 (300); 16 x 136 5.3 / 5.1 (64), 9.1 / 6.4 (300); 16 x 250 7.6 / 8.8 (256), 13.6 / 14.1 (1024), 17.7 / 17.5 (1500); 16 x 248 7.5 / 7.7 (256),
//     9.4 / 9.1 (512); 8 x 248 8.6 / 8.9 (512), 12.0 / 11.8 (1024).
static bool any_is_faster(const TqDev& d, bool mx) {
    const int A = (d.n1 + 31) / 32, B = (d.n2 + 31) / 32;
    const int64_t cu = cu_count();
    if (A >= 2 && B >= 2) return !(B == 2 && A == (mx ? 3 : 4)) || d.T <= cu || d.T > 2 * cu;
    if (A == 3) return true;
    if (A == 4) return mx ? d.T > 2 * cu : d.n2 > 8 && d.T > 3 * cu;
    if (A == 2) return (d.n2 > 8 && d.T > (mx ? 32 : 16) * cu) || (!mx && d.n2 > 16);
    if (!mx) return B < 8 || d.T > cu;
    const bool chunks = d.n2 % 8 == 0;
    if (B >= 5) {
        if (B == 8 || !chunks) return d.T > (B <= 6 || (chunks && d.n1 > 8) ? 1 : 4) * cu;
        return true;
    }
    const int filled = 100 * d.n1 * d.n2 / (32 * 32 * B);                     // percent of the tiles
    return chunks && (filled >= (B == 1 ? 50 : 60) || (d.T <= 8 * cu && (B == 2 || filled >= 45)));
}

static hipError_t any_launch(const TqDev& d, hipStream_t stream, bool mx) {
    const int A = (d.n1 + 31) / 32, B = (d.n2 + 31) / 32;
    const AnyVariant v = any_variant(d.n1, d.n2, mx);
    static OccCache occ_cache[4][8];
    int occ = 0;
    if (!mx) {
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(v.fn), 64 * B, v.lds, occ_cache[A - 1][B - 1], occ);
        if (e != hipSuccess) return e;
    } else {                                     // the LDS depends on n: occupancy for the most it takes, then what this launch takes
        static OccCache occ_mx[4][8];
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(v.fn), 64 * B, kLdsMax, occ_mx[A - 1][B - 1], occ);
        if (e != hipSuccess) return e;
        occ = kLdsMax / v.lds;
        if (occ * B > 8) occ = 8 / B;            // two waves per SIMD
        if (occ < 1) occ = 1;
    }
    const int cap = tuned(Knob::WG_PER_CU, 0);
    if (cap > 0 && cap < occ) occ = cap;
    const int64_t cu = cu_count();
    return launch(v.fn, dim3(token_loop_grid(d.T, cu, occ, any_loop_alone(d.T, cu, A, B))), dim3(64 * B), v.lds, stream, d);
}

// MXFP4 instances of tq_kernel: where any_is_faster() can say no, and four row tiles x five slabs, whose longest rows (n > 19555) tq_any_kernel's
// padded staging has no room for.  Everywhere else there is none (null).
template <int A, int B>
static constexpr KernelFn mx_kernel_for() {
    if constexpr (A == 1 || B == 1 || (A == 3 && B == 2) || (A == 4 && B == 5)) {
        return &tq_kernel<A, B, (A >= 3), true>;
    } else {
        static_assert(mx_staged_lds(A, B) > kLdsMax || any_mx_lds<A, B>(1024 * A * B) <= kLdsMax, "tq_any_kernel takes all of these rows");
        return nullptr;
    }
}

static KernelFn mx_kernel_table(int A, int B) {
    static const KernelFn tab[4][8] = {
        {mx_kernel_for<1, 1>(), mx_kernel_for<1, 2>(), mx_kernel_for<1, 3>(), mx_kernel_for<1, 4>(), mx_kernel_for<1, 5>(), mx_kernel_for<1, 6>(), mx_kernel_for<1, 7>(), mx_kernel_for<1, 8>()},
        {mx_kernel_for<2, 1>(), mx_kernel_for<2, 2>(), mx_kernel_for<2, 3>(), mx_kernel_for<2, 4>(), mx_kernel_for<2, 5>(), mx_kernel_for<2, 6>(), mx_kernel_for<2, 7>(), mx_kernel_for<2, 8>()},
        {mx_kernel_for<3, 1>(), mx_kernel_for<3, 2>(), mx_kernel_for<3, 3>(), mx_kernel_for<3, 4>(), mx_kernel_for<3, 5>(), mx_kernel_for<3, 6>(), mx_kernel_for<3, 7>(), mx_kernel_for<3, 8>()},
        {mx_kernel_for<4, 1>(), mx_kernel_for<4, 2>(), mx_kernel_for<4, 3>(), mx_kernel_for<4, 4>(), mx_kernel_for<4, 5>(), mx_kernel_for<4, 6>(), mx_kernel_for<4, 7>(), mx_kernel_for<4, 8>()},
    };
    return tab[A - 1][B - 1];
}

bool tq_supported(int n1, int n2) {
    return n1 >= 1 && n1 <= kMaxN1 && n2 >= 2 && n2 <= kMaxN2 && (n2 % 2) == 0;
}

static int64_t generic_lds_bytes(int n1, int n2) { return generic_lds((n1 + 31) / 32, (n2 + 31) / 32); }

int64_t tq_lds_bytes(int n1, int n2) {
    if (!tq_supported(n1, n2)) return 0;
    const int64_t b = generic_lds_bytes(n1, n2), a = any_variant(n1, n2, false).lds;
    const int64_t f = tq_fast_lds_bytes(n1, n2);   // the specialised kernels stage P1/P2 in LDS as well
    return f > b && f > a ? f : a > b ? a : b;
}

static int64_t generic_mx_lds_bytes(int n1, int n2) { return mx_staged_lds((n1 + 31) / 32, (n2 + 31) / 32); }

// MXFP4 output through the general kernel: any supported (n1, n2) with whole blocks of 32 channels per row whose
// fp32 staging fits in LDS beside the token tile (64 x 172: 74 KB), 16-byte aligned code rows.
bool tq_mx_generic_applicable(const TqDev& d) {
    const int64_t n = (int64_t)d.n1 * d.n2;
    return tq_supported(d.n1, d.n2) && n % 32 == 0 && d.out_vec16 && d.P1 && d.P2 && generic_mx_lds_bytes(d.n1, d.n2) <= kLdsMax;
}

hipError_t tq_mx_generic_launch(const TqDev& d, hipStream_t stream) {
    const int A = (d.n1 + 31) / 32, B = (d.n2 + 31) / 32;
    // FLATQUANT_FORCE_GENERIC = 3 / 2 forces tq_any_kernel / tq_kernel, an error where there is none; 1 tq_any_kernel where it can
    const int force = tuned(Knob::FORCE_GENERIC, 0);
    if (d.n2 >= 8 && any_variant(d.n1, d.n2, true).lds <= kLdsMax && (force == 1 || force == 3 || (force != 2 && any_is_faster(d, true)))) return any_launch(d, stream, true);
    KernelFn fn = mx_kernel_table(A, B);
    if (!fn || force == 3) return hipErrorInvalidValue;
    const int lds = (int)generic_mx_lds_bytes(d.n1, d.n2);
    static OccCache occ_cache[4][8];
    int occ = 0;
    {
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(fn), 64 * B, lds, occ_cache[A - 1][B - 1], occ);
        if (e != hipSuccess) return e;
    }
    int64_t grid = (int64_t)cu_count() * occ;
    if (grid > d.T) grid = d.T;
    return launch(fn, dim3((unsigned)grid), dim3(64 * B), lds, stream, d);
}

TqDev tq_dev_args(const TqArgs& a) {
    TqDev d;
    d.x = a.x; d.P1 = a.P1; d.P2 = a.P2; d.clip = a.clip;
    d.out_codes = a.out_codes; d.out_scales = a.out_scales;
    d.x_stride = a.x_stride; d.T = a.T; d.n1 = a.n1; d.n2 = a.n2; d.clip_mode = a.clip_mode;
    d.mx_tiled = a.mx_tiled;
    d.n1_magic = a.n1 >= 2 ? (uint32_t)(0x100000000ull / (uint64_t)a.n1) + 1u : 0u;
    d.n2_magic = a.n2 >= 2 ? (uint32_t)(0x100000000ull / (uint64_t)a.n2) + 1u : 0u;
    d.vec8 = (a.n2 % 8 == 0) && (a.x_stride % 8 == 0) && ((reinterpret_cast<uintptr_t>(a.x) & 15) == 0);
    const int64_t n = (int64_t)a.n1 * a.n2;
    d.out_vec16 = (n % 32 == 0) && ((reinterpret_cast<uintptr_t>(a.out_codes) & 15) == 0);
    return d;
}

hipError_t tq_launch(const TqArgs& a, hipStream_t stream) {
    const int A = (a.n1 + 31) / 32, B = (a.n2 + 31) / 32;
    KernelFn fn = kernel_table(A, B);
    const int lds = (int)generic_lds_bytes(a.n1, a.n2);
    const int nt = 64 * B;

    const TqDev d = tq_dev_args(a);
    // FLATQUANT_FORCE_GENERIC=1 keeps the general kernel testable on shapes the specialised ones would take
    if (tq_fast_applicable(d) && tuned(Knob::FORCE_GENERIC, 0) == 0) return tq_fast_launch(d, stream);

    // Right factors of fewer than 8 columns stay with tq_kernel (a chunk of a row could straddle three rows of X~), and so do rows that
    // are only quantized (both factors left out), which have not been moved: there the other one gives the same bytes in less time (64 x 80
    // at 2048 tokens 17.9 / 12.4 us, 64 x 128 at 16384 110 / 78).  FLATQUANT_FORCE_GENERIC as for MXFP4.
    const int force = tuned(Knob::FORCE_GENERIC, 0);
    if (a.n2 >= 8 && (a.P1 || a.P2) && force != 2 && (force == 1 || force == 3 || any_is_faster(d, false))) return any_launch(d, stream, false);
    if (force == 3) return hipErrorInvalidValue;
    static OccCache occ_cache[4][8];   // per variant and device
    int occ = 0;
    {
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(fn), nt, (int)lds, occ_cache[A - 1][B - 1], occ);
        if (e != hipSuccess) return e;
    }
    const int cap = tuned(Knob::WG_PER_CU, 0);
    if (cap > 0 && cap < occ) occ = cap;
    int64_t grid = (int64_t)cu_count() * occ;
    if (grid > a.T) grid = a.T;

    return launch(fn, dim3((unsigned)grid), dim3(nt), lds, stream, d);
}

}  // namespace fq
