// W4A4 matrix product for gfx950: out[t, o] = fp16( s_x[t] s_w[o] sum_k q_x[t, k] q_w[o, k] ), the low-bit matrix
// multiplication that consumes the two quantized factors of Eq. (2) (Sec. 3.2: low-bit matrix multiplications for all
// linear layers; Sec. 3.3: the transform + quantization kernel feeds an INT4 GEMM).
//
// Both operands arrive as packed 4-bit two's-complement codes, K contiguous (activations [T, n/2], weights [m, n/2]),
// which is the operand order of an MFMA for C = A B^T.  The codes are widened to int8 on the fly without a sign
// extension: for a packed dword w, (w << 4) & 0xF0F0F0F0 holds 16 q of the even channels and w & 0xF0F0F0F0 holds 16 q
// of the odd channels, as signed bytes.  Both operands are widened the same way, so the K order inside an MFMA is
// the same permutation for both and every product carries a factor 256 that the epilogue divides out exactly.
// v_mfma_i32_32x32x32_i8 accumulates in int32 (|sum| <= 128 * 128 * n < 2^31 for n <= 65536).  Large launches widen to FP6
// instead (w4a4_fp6_kernel, further down).
//
// Workgroup: 4 waves, C tile 128 tokens x 128 output channels (or 8 waves, 256 x 128, when the launch has enough such
// tiles for every CU), each wave 64 x 64 (2 x 2 MFMA tiles; the weights are
// the MFMA's first operand so that a lane ends up with runs of 4 consecutive output channels of one token).  K advances by
// 256 codes (128 bytes = one cache line per row) per iteration through double-buffered LDS tiles, one barrier per
// iteration; the tiles go from global memory straight into LDS, a whole iteration before they are read.
// Launches whose 128 x 128 tiles would reach at most half of the CUs (decode, short prefill chunks) take the few-token
// kernel further down instead.
#include "fq_internal.h"

namespace fq {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int GT = 128;               // tile edge, tokens and output channels
constexpr int GKB = 128;              // packed bytes of K per row and iteration (256 codes)
constexpr int GPITCH = GKB;           // LDS row pitch: rows are written by global-to-LDS loads, 8 whole rows per wave and
                                      // instruction, so there is no padding; the 16-byte chunks of a row are swizzled instead
constexpr int G_NT = 256;
constexpr int G_TILE_BYTES = GT * GPITCH;
constexpr int G_LDS_BYTES = 4 * G_TILE_BYTES + GT * 4;   // A and B, two buffers each, + the weight steps of the tile
constexpr int G_LDS_BYTES_WIDE = 6 * G_TILE_BYTES + GT * 4;   // 256-token tile: A twice the size

struct GemmDev {
    const uint8_t* xc;
    const _Float16* xs;
    const uint8_t* wc;
    const _Float16* ws;
    _Float16* out;
    int64_t T;
    int64_t out_stride;
    int m, n;
};

// two k-steps of MFMA operands from 16 packed bytes
__device__ __forceinline__ void widen(const u32x4 w, i32x4& s0, i32x4& s1) {
    constexpr unsigned M = 0xF0F0F0F0u;
    s0 = i32x4{(int)((w[0] << 4) & M), (int)(w[0] & M), (int)((w[1] << 4) & M), (int)(w[1] & M)};
    s1 = i32x4{(int)((w[2] << 4) & M), (int)(w[2] & M), (int)((w[3] << 4) & M), (int)(w[3] & M)};
}

// TW = waves along the token axis: 2 -> C tile 128 tokens x 128 channels (4 waves), 4 -> 256 x 128 (8 waves): a quarter
// less operand traffic from L2 per product term, for launches with enough 256-token tiles to fill the chip.
template <int TW>
__global__ __launch_bounds__(128 * TW) __attribute__((amdgpu_waves_per_eu(2))) void w4a4_kernel(GemmDev p) {
    constexpr int GTM = 64 * TW;                       // tokens per tile
    constexpr int NW = 2 * TW;                         // waves
    constexpr int A_TILE = GTM * GPITCH, B_TILE = GT * GPITCH, STAGE = A_TILE + B_TILE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w % TW, wn = w / TW;
    const int64_t t0 = (int64_t)blockIdx.x * GTM;
    const int o0 = blockIdx.y * GT;
    const int64_t kbytes = p.n / 2;
    const int nk = p.n / (2 * GKB);

    // Tile loads go from global memory straight into LDS (global_load_lds_dwordx4: lane i of a wave writes 16 bytes at
    // the wave's LDS base + 16 i, from any global address).  One instruction fills 8 rows of 128 bytes; wave w owns rows
    // 32 w .. 32 w + 31 of both tiles (4 instructions per operand and iteration).  LDS slot j of row r holds the row's
    // chunk j ^ ((r >> 1) & 7): with that swizzle the 16-byte operand reads of 32 consecutive rows (same chunk) spread
    // over all banks although the pitch is a multiple of the bank width.  Rows past the end re-read the last row.
    static_assert(GKB == 128 && GT == 128, "load mapping below");
    constexpr int NLA = GTM / 8 / NW, NLB = GT / 8 / NW;   // 8-row instructions per wave: 4 and 4 (4 waves), 4 and 2 (8 waves)
    const unsigned char* asrc[NLA];
    const unsigned char* bsrc[NLB];
#pragma unroll
    for (int k = 0; k < NLA; ++k) {
        const int row = 8 * (NLA * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        int64_t tr = t0 + row;
        if (tr >= p.T) tr = p.T - 1;
        asrc[k] = p.xc + tr * kbytes + 16 * ch;
    }
#pragma unroll
    for (int k = 0; k < NLB; ++k) {
        const int row = 8 * (NLB * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        int orow = o0 + row;
        if (orow >= p.m) orow = p.m - 1;
        bsrc[k] = p.wc + (int64_t)orow * kbytes + 16 * ch;
    }
    typedef const __attribute__((address_space(1))) void* gptr;
    typedef __attribute__((address_space(3))) void* lptr;
    auto issue = [&](int it, int buf) {   // past the last tile the last one is re-read (nobody uses it): no branch in the loop body
        const int itc = it < nk ? it : nk - 1;
        unsigned char* A = smem + buf * STAGE + w * (8 * NLA * GPITCH);
        unsigned char* B = smem + buf * STAGE + A_TILE + w * (8 * NLB * GPITCH);
#pragma unroll
        for (int k = 0; k < NLA; ++k) __builtin_amdgcn_global_load_lds((gptr)(asrc[k] + (int64_t)itc * GKB), (lptr)(A + k * 8 * GPITCH), 16, 0, 0);
#pragma unroll
        for (int k = 0; k < NLB; ++k) __builtin_amdgcn_global_load_lds((gptr)(bsrc[k] + (int64_t)itc * GKB), (lptr)(B + k * 8 * GPITCH), 16, 0, 0);
    };
    // the tile requested last has arrived in LDS (this wave's part), then every wave's part has
    auto tile_ready = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    i32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    if (tid < GT) {
        const int o = o0 + tid;
        reinterpret_cast<float*>(smem + 2 * STAGE)[tid] = (o < p.m) ? (float)p.ws[o] : 0.0f;
    }
    const int aoff = (64 * wm + c) * GPITCH;
    const int boff = (64 * wn + c) * GPITCH;
    const int hs = h ^ ((c >> 1) & 7);   // chunk 2 kp + h of row 32 x + c sits in slot (2 kp) ^ hs (the row's swizzle is that of c)
    constexpr int NKP = GKB / 32;   // K step pairs (64 codes) per tile
    static_assert(NKP >= 4 && NKP % 2 == 0, "the pipeline below reads two step pairs ahead and alternates two register stages");
    // packed operands of one K step pair: x = 0, 1: tokens 32 x + c (A); x = 2, 3: output channels 32 (x - 2) + c (B)
    auto lds_chunk = [&](int buf, int kp, int x) -> u32x4 {
        const unsigned char* base = smem + buf * STAGE + ((x >> 1) ? A_TILE + boff : aoff);
        return *reinterpret_cast<const u32x4*>(base + 32 * (x & 1) * GPITCH + 16 * ((2 * kp) ^ hs));
    };
    // Software pipeline over K step pairs g = it * NKP + kp, three stages deep: while the MFMAs of pair g run on the
    // widened operands W[g & 1], pair g + 1 is widened from its packed registers P[(g + 1) & 1] into W[(g + 1) & 1] and
    // pair g + 2 is read from LDS into P[g & 1].  The work is cut into 8 slices per pair, one MFMA followed by one
    // slice of widening (6 vector instructions, shorter than the MFMA) and at most one LDS read, in this order in
    // the instruction stream: a wave issues in order, so only vector work that sits between two MFMAs can run in
    // the shadow of the first.
    u32x4 P[2][4];
    i32x4 W[2][4][2];   // [stage][operand x][K step s]
    issue(0, 0);
    tile_ready();
    issue(1, 1);
#pragma unroll
    for (int x = 0; x < 4; ++x) { P[0][x] = lds_chunk(0, 0, x); P[1][x] = lds_chunk(0, 1, x); }
    constexpr unsigned M = 0xF0F0F0F0u;
    auto widen_slice = [&](const u32x4& w, int s) -> i32x4 {
        return i32x4{(int)((w[2 * s] << 4) & M), (int)(w[2 * s] & M), (int)((w[2 * s + 1] << 4) & M), (int)(w[2 * s + 1] & M)};
    };
#pragma unroll
    for (int x = 0; x < 4; ++x) { W[0][x][0] = widen_slice(P[0][x], 0); W[0][x][1] = widen_slice(P[0][x], 1); }
    // one iteration: tile `it` (LDS buffer `buf`) through the MFMAs.  After pair NKP - 3 nobody reads that buffer any
    // more (the later pairs were read ahead), so behind the barrier that publishes tile it + 1 it takes tile it + 2.
    auto iteration = [&](int it, int buf) {
#pragma unroll
        for (int kp = 0; kp < NKP; ++kp) {
            const int cur = kp & 1, nxt = cur ^ 1;           // NKP is even: the stage parity of pair g is that of kp
            const int fkp = (kp + 2) % NKP;                   // pair g + 2: in this tile, or the first pairs of the next one
            const int fbuf = (kp + 2 < NKP) ? buf : buf ^ 1;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int s = m >> 2, i = (m >> 1) & 1, j = m & 1;
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(W[cur][2 + j][s], W[cur][i][s], acc[i][j], 0, 0, 0);
                W[nxt][m >> 1][m & 1] = widen_slice(P[nxt][m >> 1], m & 1);
                // P[cur] was widened during the previous pair: its registers take pair g + 2
                if (m >= 4) P[cur][m - 4] = lds_chunk(fbuf, fkp, m - 4);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (kp == NKP - 3) {
                tile_ready();
                issue(it + 2, buf);
            }
        }
    };
    for (int it = 0; it < nk; it += 2) {
        iteration(it, 0);
        if (it + 1 < nk) iteration(it + 1, 1);
    }
    tile_ready();   // no load is still writing, every wave is done with the K tiles: the epilogue reuses their space

    // epilogue.  The weights are the MFMA's first operand, so in acc[i][j] a lane holds, for token 64 wm + 32 i + c,
    // the output channels 64 wn + 32 j + 8 (r / 4) + 4 h + r % 4: runs of 4 consecutive channels.  They are scaled,
    // rounded to fp16 and staged in LDS (the K tiles are dead by now) as a [128 tokens][128 channels] tile, which then
    // leaves in whole 16-byte pieces.  Every sum is a multiple of 256 (both operands carry a factor 16).
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    constexpr int OPITCH = 2 * GT + 16;
    unsigned char* otile = smem;
    float* sws = reinterpret_cast<float*>(smem + 2 * STAGE);          // [128] weight steps of this tile
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t t = t0 + 64 * wm + 32 * i + c;
        const float sx = (float)p.xs[t < p.T ? t : p.T - 1];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int oc = 64 * wn + 32 * j + 8 * g + 4 * h;
                const float4 sw = *reinterpret_cast<const float4*>(sws + oc);
                const half4 v = {(_Float16)((float)(acc[i][j][4 * g] >> 8) * sx * sw.x), (_Float16)((float)(acc[i][j][4 * g + 1] >> 8) * sx * sw.y),
                                 (_Float16)((float)(acc[i][j][4 * g + 2] >> 8) * sx * sw.z), (_Float16)((float)(acc[i][j][4 * g + 3] >> 8) * sx * sw.w)};
                *reinterpret_cast<half4*>(otile + (64 * wm + 32 * i + c) * OPITCH + 2 * oc) = v;
            }
    }
    __syncthreads();
    const bool wide = ((reinterpret_cast<uintptr_t>(p.out) & 15) == 0) && (p.out_stride % 8 == 0);
#pragma unroll
    for (int k = 0; k < GTM * 16 / (64 * NW); ++k) {
        const int q = tid + 64 * NW * k, row = q >> 4, ch = q & 15;
        const int64_t t = t0 + row;
        const int o = o0 + 8 * ch;
        if (t < p.T && o < p.m) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(otile + row * OPITCH + 16 * ch);
            _Float16* dst = p.out + t * p.out_stride + o;
            if (wide && o + 8 <= p.m) {
                *reinterpret_cast<u32x4*>(dst) = v;
            } else {
                const _Float16* e = reinterpret_cast<const _Float16*>(&v);
                for (int x = 0; x < 8; ++x)
                    if (o + x < p.m) dst[x] = e[x];
            }
        }
    }
}

// ---- many tokens.  A chunk of 32 codes becomes an FP6 operand (E2M3) in registers: the code q offset to q + 8 = 0 .. 15 IS
// the E2M3 bit pattern of (q + 8) / 8 (subnormal up to 7 / 8, the first binade up to 15 / 8), so the codes need only be
// spread from 4-bit to 6-bit fields, 8 vector instructions per 16 codes.  Their order inside a lane is free as long as both
// operands share it.  The sums are exact: every product is an integer / 64 and the total at most 225 n / 64 with
// n <= 65536, which fits 24 bits.  The offset leaves in the epilogue,
//   sum q_x q_w = sum (q_x + 8)(q_w + 8) - 8 sum q_x - 8 sum q_w - 64 n,
// with the row sums of the codes (one v_dot8 per dword) taken on the way.
// FP6 MFMAs have twice the rate of int8 ones and are held back less by the power limit: alone, for the 2.2e12 operations of
// 16384 x 8192 x 8192 on random codes, they take 303 us (328 with sign and magnitude in place of the offset), int8 ones 531.
// What bounds the kernel there (613 - 672 us from box to box; 835 - 888 with the int8 kernel above): one wave per SIMD issues in
// order, and it issues in 68 % of its cycles (12.0 vector instructions per MFMA, the MFMA among them: spreading and row
// sums); waits for the tiles take 13 %, the MFMA pipe is busy 37 % of the time, at 2.0 GHz.  Without the row sums 554, without
// loads as well 483.  Two waves per SIMD (eight of 128 x 64) spread every weight row four times: 697.  Row sums by one of
// the two waves that share a row: the same time, twice the code.
constexpr unsigned kSpreadA0 = 0x0F00F00Fu, kSpreadA1 = 0xF00F00F0u, kSpreadA2 = 0x00F00F00u;   // fields that do not move
constexpr unsigned kSpreadM0 = 0xCF3CF3CFu, kSpreadM1 = 0xF3CF3CF3u, kSpreadM2 = 0x3CF3CF3Cu;   // the low 4 bits of all fields
constexpr unsigned kSpreadX0 = 0x08208208u, kSpreadX1 = 0x82082082u, kSpreadX2 = 0x20820820u;   // bit 3 of all fields
__device__ __forceinline__ unsigned pick_bits(unsigned mask, unsigned a, unsigned b) { return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA); }   // mask ? a : b
__device__ __forceinline__ unsigned and_xor(unsigned v, unsigned m, unsigned x) { return __builtin_amdgcn_bitop3_b32(v, m, x, 0x6A); }           // (v & m) ^ x
// 16 codes -> 16 fields of 6 bits in three dwords.  Every nibble stays or moves up by 2 bits, into the next dword where it
// straddles the end (fields in order: nibbles 0 1 3 4 6 7 of lo, 1 2 4 5 7 0 of hi, 2 of lo, 3 of hi, 5 of lo, 6 of hi).
__device__ __forceinline__ void spread16(unsigned lo, unsigned hi, unsigned* o) {
    const unsigned t = lo << 2, u = __builtin_amdgcn_alignbit(hi, lo, 30);      // u = hi << 2 | lo >> 30
    o[0] = and_xor(pick_bits(kSpreadA0, lo, t), kSpreadM0, kSpreadX0);
    o[1] = and_xor(pick_bits(kSpreadA1, hi, u), kSpreadM1, kSpreadX1);
    o[2] = and_xor(pick_bits(kSpreadA2, lo, u), kSpreadM2, kSpreadX2);
}

struct Fp6Tile {
    // MFMA tiles of 32 x 32 per wave (tokens x channels), waves, LDS stages: 256 x 256 with a wave on each SIMD, as large as
    // the register file allows, so that every code is spread by two waves only and crosses LDS and L2 least often
    static constexpr int TI = 4, TJ = 4, WM = 2, WN = 2, NST = 2;
    static constexpr int NW = WM * WN;
    static constexpr int TOK = 32 * TI * WM, CH = 32 * TJ * WN, ROWS = TOK + CH;
    static constexpr int STAGE = ROWS * GKB;                        // code tiles of one K iteration
    static constexpr int OPITCH = 64 * TJ + 16;                     // output staging: 32 tokens of a wave's channels
    static constexpr int WCOL = 32 * TJ * 8;                        // step and row sum of a wave's channels
    static constexpr int LDS = NST * STAGE + NW * WCOL;
    static_assert(NW * 32 * OPITCH <= STAGE && LDS <= 160 * 1024 && NST >= 2, "LDS budget");
};

// Every operand byte goes from global memory straight into LDS (global-to-LDS loads, unpadded 128-byte rows, 16-byte chunks
// swizzled), NST iterations of 256 codes deep, one barrier per iteration; persistent workgroups whose loads run on from one
// output tile into the next.  ODD: the output's rows are not all dword-aligned and leave in halves, by a loop that only such
// launches carry (6486 x 5705 x 256 82 us with the halves of 16-byte pieces stored one by one, now 69; int8 78; 2733 x 3333 x
// 2048 41.0, now 39.1; int8 48.1).
template <bool ODD>
__global__ __launch_bounds__(64 * Fp6Tile::NW) __attribute__((amdgpu_waves_per_eu(1, 1))) void w4a4_fp6_kernel(GemmDev p) {
    using L = Fp6Tile;
    constexpr int TI = L::TI, TJ = L::TJ, WM = L::WM, NST = L::NST;
    constexpr int NW = L::NW, TOK = L::TOK, CH = L::CH, STAGE = L::STAGE, A_TILE = TOK * GKB, NOP = TI + TJ;
    constexpr int NLA = TOK / 8 / NW, NLB = CH / 8 / NW, NL = NLA + NLB;   // load instructions per wave and iteration
    constexpr int NKP = GKB / 32;                                   // K steps (64 codes) per iteration
    constexpr int LA = 2, KB = NKP - LA;                            // operands are read LA steps ahead; the steps before the barrier
    constexpr int NQ = TI * TJ;                                     // MFMAs per step
    constexpr int LSTEPS = 2;                                       // steps over which an iteration's loads are spread
    static_assert(NKP == 4, "register stages below");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w % WM, wn = w / WM;
    const int64_t kbytes = p.n / 2;
    const int nk = p.n / (2 * GKB);
    const int ntx = (int)((p.T + TOK - 1) / TOK), nty = (p.m + CH - 1) / CH;
    const int64_t ntiles = (int64_t)ntx * nty;

    // Tiles of this workgroup.  Workgroup b runs on XCD b % 8: every XCD takes a contiguous eighth of a tile order that
    // goes through panels of PW token tiles, so that the tiles in flight on an XCD share rows of both operands in its L2.
    constexpr int PW = 4;
    const int64_t per_xcd = (ntiles + 7) / 8;
    const int xcd = blockIdx.x & 7;
    const int64_t first = xcd * per_xcd, left = ntiles - first;
    const int64_t mine = left < per_xcd ? left : per_xcd;           // tiles of this XCD (<= 0: none)
    const int64_t qstep = gridDim.x >> 3;
    int64_t q = blockIdx.x >> 3;
    if (q >= mine) return;
    struct Pos { int64_t t0; int o0; };
    auto tile_pos = [&](int64_t qq) -> Pos {
        const int64_t pos = first + qq, panel = pos / ((int64_t)PW * nty);
        const int r = (int)(pos - panel * ((int64_t)PW * nty));
        const int width = ntx - panel * PW < PW ? (int)(ntx - panel * PW) : PW;
        const int ty = r / width;
        return Pos{(panel * PW + r - ty * width) * TOK, ty * CH};
    };

    // ---- loads: one instruction fills 8 rows of 128 bytes; LDS slot j of row r holds the row's chunk j ^ ((r >> 1) & 7).
    // Rows past the end re-read the last row.
    __amdgpu_buffer_rsrc_t abuf, bbuf;
    uint32_t aoff[NLA], boff[NLB];
    auto set_source = [&](const Pos& t) {
        const int arows = (int)(p.T - t.t0 < TOK ? p.T - t.t0 : TOK), brows = p.m - t.o0 < CH ? p.m - t.o0 : CH;
        abuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.xc) + t.t0 * kbytes, 0, arows * (int)kbytes, 0x00020000);
        bbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wc) + (int64_t)t.o0 * kbytes, 0, brows * (int)kbytes, 0x00020000);
#pragma unroll
        for (int k = 0; k < NLA; ++k) {
            const int row = 8 * (NLA * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
            aoff[k] = (uint32_t)(row < arows ? row : arows - 1) * (uint32_t)kbytes + 16 * ch;
        }
#pragma unroll
        for (int k = 0; k < NLB; ++k) {
            const int row = 8 * (NLB * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
            boff[k] = (uint32_t)(row < brows ? row : brows - 1) * (uint32_t)kbytes + 16 * ch;
        }
    };
    typedef __attribute__((address_space(3))) void* lptr;
    // loads k0 .. k1 - 1 of the NL that bring iteration `it` (past the last one it is re-read; nobody uses it)
    auto issue = [&](int it, int stage, int k0, int k1) {
        const int itc = it < nk ? it : nk - 1;
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            if (k < NLA) __builtin_amdgcn_raw_ptr_buffer_load_lds(abuf, (lptr)(smem + stage + (NLA * w + k) * 8 * GKB), 16, (int)aoff[k], itc * GKB, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(bbuf, (lptr)(smem + stage + A_TILE + (NLB * w + k - NLA) * 8 * GKB), 16, (int)boff[k - NLA], itc * GKB, 0, 0);
        }
    };

    // ---- operands.  x < TI: tokens 32 (TI wm + x) + c; else channels 32 (TJ wn + x - TI) + c
    const int hs = h ^ ((c >> 1) & 7);   // chunk 2 kp + h of row 32 x + c sits in slot (2 kp) ^ hs
    const int abyte = (32 * TI * wm + c) * GKB, bbyte = A_TILE + (32 * TJ * wn + c) * GKB;
    auto lds_chunk = [&](int stage, int kp, int x) -> u32x4 {
        const int a = stage + (x < TI ? abyte + 32 * x * GKB : bbyte + 32 * (x - TI) * GKB) + 16 * ((2 * kp) ^ hs);
        return *reinterpret_cast<const u32x4*>(smem + a);
    };
    // Three register stages: while the MFMAs of step kp run on the FP6 operands W[kp & 1], the packed codes P of step kp + 1
    // are spread into W[(kp + 1) & 1], and as each operand has been spread its registers take the codes of step kp + 2 from
    // LDS.  A wave issues in order, so the vector work stands between the MFMAs, a share behind each.
    f32x16 acc[TI][TJ];
    u32x4 P[NOP];
    unsigned W[2][NOP][6];
    int rsum[NOP];                       // sums of this lane's codes, per operand row
    auto mfma = [&](int i, int j, int st) {
        const unsigned *wv = W[st][TI + j], *xv = W[st][i];
        const i32x8 a = {(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3], (int)wv[4], (int)wv[5], 0, 0};
        const i32x8 b = {(int)xv[0], (int)xv[1], (int)xv[2], (int)xv[3], (int)xv[4], (int)xv[5], 0, 0};
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 2, 2, 0, 0, 0, 0);   // FP6 E2M3 for both, no scale
    };
    auto spread = [&](int st, int u) {   // half u & 1 of operand u / 2: 16 codes
        const int x = u >> 1, s = u & 1;
        const unsigned lo = P[x][2 * s], hi = P[x][2 * s + 1];
        spread16(lo, hi, &W[st][x][3 * s]);
        rsum[x] = __builtin_amdgcn_sdot8((int)hi, 0x11111111, __builtin_amdgcn_sdot8((int)lo, 0x11111111, rsum[x], false), false);
    };
    // K step kp and a share of the loads of iteration `lit` into `stage_load`.  Steps KB .. NKP - 1 of an iteration, then
    // 0 .. KB - 1 of the next one, lie between two barriers: s is the step's place in that sequence, which the loads are
    // spread over.  `next`: there is a next step in this tile.
    auto step = [&](int kp, int stage_ahead, int lit, int stage_load, int s, int s0, int nsteps, bool next) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
            mfma(m / TJ, m % TJ, kp & 1);
#pragma unroll
            for (int u = m * 2 * NOP / NQ; next && u < (m + 1) * 2 * NOP / NQ; ++u) {
                spread((kp + 1) & 1, u);
                if (u & 1) P[u >> 1] = lds_chunk(stage_ahead, (kp + LA) % NKP, u >> 1);
            }
            if (s >= s0 && s < s0 + nsteps) issue(lit, stage_load, ((s - s0) * NQ + m) * NL / (nsteps * NQ), ((s - s0) * NQ + m + 1) * NL / (nsteps * NQ));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the next iteration has arrived (this wave's part, then everybody's) and nobody reads the current one's stage any more
    auto arrive = [&]() {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * NL) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto read_step = [&](int stage, int kp) {
#pragma unroll
        for (int x = 0; x < NOP; ++x) P[x] = lds_chunk(stage, kp, x);
    };

    Pos cur = tile_pos(q);
    set_source(cur);
#pragma unroll
    for (int s = 0; s + 1 < NST; ++s) issue(s, s * STAGE, 0, NL);
    arrive();
    int st = 0, stl = (NST - 1) * STAGE;     // stage of the current iteration, and the one to be loaded next
    auto advance = [&](int stage) { return stage + STAGE == NST * STAGE ? 0 : stage + STAGE; };
    read_step(0, 0);

    // Loads run NST - 1 iterations ahead of the steps 0 .. KB - 1 and go on into the next tile: the last NST - 1 iterations
    // of a tile load the first ones of the next.
    const bool flow = nk >= NST;
    while (true) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
#pragma unroll
        for (int x = 0; x < NOP; ++x) rsum[x] = 0;
#pragma unroll
        for (int u = 0; u < 2 * NOP; ++u) spread(0, u);
        read_step(st, 1);
        // steps 0 .. KB - 1 of iteration 0; loads of iteration NST - 1
#pragma unroll
        for (int kp = 0; kp < KB; ++kp) step(kp, st, NST - 1, stl, kp, 0, LSTEPS, true);
        arrive();
        int lit = NST;                       // iteration to be loaded next
        auto body = [&]() {
            const int stn = advance(st);
            stl = advance(stl);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, lit, stl, kp - KB, 0, LSTEPS, true);
#pragma unroll
            for (int kp = 0; kp < KB; ++kp) step(kp, stn, lit, stl, kp + LA, 0, LSTEPS, true);
            arrive();
            st = stn;
            ++lit;
        };
        int it = 0;
        for (; it < nk - 1 && lit < nk; ++it) body();
        const int64_t qn = q + qstep;
        const bool more = qn < mine;
        Pos nxt = cur;
        if (more) nxt = tile_pos(qn);
        if (more && flow) { set_source(nxt); lit = 0; }
        for (; it < nk - 1; ++it) body();
        // the quantization steps of this tile's rows and channels, requested ahead of the epilogue (raw bits: nothing waits here)
        const uint16_t* xs_bits = reinterpret_cast<const uint16_t*>(p.xs);
        const uint16_t* ws_bits = reinterpret_cast<const uint16_t*>(p.ws);
        unsigned esx[TI], esw[TJ];
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const int64_t t = cur.t0 + 32 * (TI * wm + i) + c;
            esx[i] = xs_bits[t < p.T ? t : p.T - 1];
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int o = cur.o0 + 32 * (TJ * wn + j) + c;
            esw[j] = ws_bits[o < p.m ? o : p.m - 1];
        }
        // the last steps of the tile: nothing is loaded, the current stage takes the output tile
        {
            const int stn = advance(st);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, 0, 0, 0, 1, 0, kp + 1 < NKP);
        }
        __builtin_amdgcn_sched_barrier(0);

        // epilogue: in acc[i][j] a lane holds, for token 32 (TI wm + i) + c, the output channels 32 (TJ wn + j) + 8 (r / 4) +
        // 4 h + r % 4.  Rounded to fp16 and turned, 32 tokens at a time, through a part of LDS that belongs to the wave
        // alone (no barrier), from where they leave in 16-byte pieces of whole rows.  All corrections are integers below
        // 2^24, so their fp32 sums are exact.
        typedef _Float16 half4 __attribute__((ext_vector_type(4)));
        constexpr int OPITCH = L::OPITCH, CPR = 4 * TJ;              // 16-byte pieces per token
        unsigned char* ot = smem + st + w * (32 * OPITCH);
        float* wcol = reinterpret_cast<float*>(smem + NST * STAGE + w * L::WCOL);   // [32 TJ] steps, [32 TJ] corrections
#pragma unroll
        for (int x = 0; x < NOP; ++x) rsum[x] += __shfl_xor(rsum[x], 32);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            wcol[32 * j + c] = (float)__builtin_bit_cast(_Float16, (uint16_t)esw[j]);   // both halves of the wave store the same
            wcol[32 * TJ + 32 * j + c] = (float)(-8 * rsum[TI + j]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uintptr_t pitch_bits = reinterpret_cast<uintptr_t>(p.out) | (uintptr_t)(2 * p.out_stride);
        const bool wide = (pitch_bits & 15) == 0, pairs = (pitch_bits & 3) == 0;   // whole pieces, dwords, or halves
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            const float sx = (float)__builtin_bit_cast(_Float16, (uint16_t)esx[i]);
            const float cx = (float)(-8 * rsum[i] - 64 * p.n);
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 sw = *reinterpret_cast<const float4*>(wcol + 32 * j + 8 * g + 4 * h);
                    const float4 cw = *reinterpret_cast<const float4*>(wcol + 32 * TJ + 32 * j + 8 * g + 4 * h);
                    const half4 v = {(_Float16)(fmaf(acc[i][j][4 * g], 64.0f, cx + cw.x) * sx * sw.x),
                                     (_Float16)(fmaf(acc[i][j][4 * g + 1], 64.0f, cx + cw.y) * sx * sw.y),
                                     (_Float16)(fmaf(acc[i][j][4 * g + 2], 64.0f, cx + cw.z) * sx * sw.z),
                                     (_Float16)(fmaf(acc[i][j][4 * g + 3], 64.0f, cx + cw.w) * sx * sw.w)};
                    *reinterpret_cast<half4*>(ot + c * OPITCH + 64 * j + 16 * g + 8 * h) = v;
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if constexpr (ODD) {             // 64 consecutive halves per instruction: whole lines as far as they go
                const int64_t t = cur.t0 + 32 * (TI * wm + i);
                const int o = cur.o0 + 32 * TJ * wn + l, rows = (int)(p.T - t < 32 ? p.T - t : 32);
                _Float16* dst = p.out + t * p.out_stride + o;
#pragma unroll 4
                for (int row = 0; row < rows; ++row, dst += p.out_stride)
#pragma unroll
                    for (int x = 0; x < TJ / 2; ++x) {
                        const _Float16 v = *reinterpret_cast<const _Float16*>(ot + row * OPITCH + 2 * (l + 64 * x));
                        if (o + 64 * x < p.m) dst[64 * x] = v;
                    }
            } else {                         // `pairs` holds (the same loop without the test measured 1 - 2 % slower)
#pragma unroll
                for (int k = 0; k < 32 * CPR / 64; ++k) {
                    const int e = l + 64 * k, row = e / CPR, ch = e % CPR;
                    const int64_t t = cur.t0 + 32 * (TI * wm + i) + row;
                    const int o = cur.o0 + 32 * TJ * wn + 8 * ch;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(ot + row * OPITCH + 16 * ch);
                    if (t < p.T && o < p.m) {
                        _Float16* dst = p.out + t * p.out_stride + o;
                        if (wide && o + 8 <= p.m) {
                            *reinterpret_cast<u32x4*>(dst) = v;
                        } else if (pairs && o + 8 <= p.m) {
                            for (int x = 0; x < 4; ++x) reinterpret_cast<uint32_t*>(dst)[x] = v[x];
                        } else {
                            const _Float16* ev = reinterpret_cast<const _Float16*>(&v);
                            for (int x = 0; x < 8; ++x)
                                if (o + x < p.m) dst[x] = ev[x];
                        }
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (!more) break;
        q = qn;
        cur = nxt;
        if (flow) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();    // every wave is done with the output stage: it takes the next loads
            stl = st;
            st = advance(st);
        } else {                             // fewer iterations than stages: start over
            wait_vm_pending<0>();
            __syncthreads();
            set_source(cur);
#pragma unroll
            for (int s = 0; s + 1 < NST; ++s) issue(s, s * STAGE, 0, NL);
            arrive();
            st = 0;
            stl = (NST - 1) * STAGE;
            read_step(0, 0);
        }
    }
    wait_vm_pending<0>();                    // nothing may still be on its way into LDS when the workgroup ends
}

// ---- few tokens (decode, short prefill chunks): the weights are read once (per tile of 64 tokens), and what bounds the kernel is how fast the CUs take
// them in.  A workgroup owns 32 (or 16) output channels for all tokens.  Every operand byte goes from global memory
// straight into LDS, a whole cache line per row at a time: a wave owns every nwv-th 128-byte line of K (256 codes) of
// the workgroup's weight rows and of the token rows, with a ring of `depth` line slots of its own in LDS.  One
// global-to-LDS instruction moves 8 whole rows; the wave waits only for its own oldest slot (no barrier in the loop),
// multiplies it and requests the line `depth` steps ahead into the same slot.  The slots use the swizzle of the tiled
// kernel (slot chunk j of row r holds the row's chunk j ^ ((r >> 1) & 7)).  The partial sums of the waves are added
// through LDS at the end.  (Feeding the MFMA from registers instead, 32 bytes of 32 rows per load, costs four
// instructions and tag look-ups per cache line and holds far less in flight: 1.5 to 3 times slower.)
// ROWS = 16: the workgroup owns 16 output channels only (twice as many workgroups, for layers with too few channels
// to give every CU one of 32); the MFMA's upper 16 rows repeat the lower ones and are dropped.
template <int NTD, int ROWS>   // token rows in groups of 8 (one load instruction each): 1, 2, 4, 8 for T <= 8, 16, 32, 64
__global__ __launch_bounds__(NTD >= 8 ? 512 : 1024) void w4a4_skinny_kernel(GemmDev p, int depth) {
    static_assert(ROWS == 16 || ROWS == 32, "weight rows per workgroup");
    constexpr int NWI = ROWS / 8;                        // load instructions per line of the weight rows
    constexpr int NG = ROWS / 8;                         // groups of 8 output channels
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int NTT = NTD > 4 ? NTD / 4 : 1;           // MFMA token tiles of 32
    constexpr int XROWS = 8 * NTD;
    constexpr int XOFF = ROWS * 128;
    constexpr int SLOT = (ROWS + XROWS) * 128;           // weight rows, then token rows, one line each
    constexpr int NI = NWI + NTD;                        // load instructions per step
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int o0 = blockIdx.x * ROWS;
    const int64_t t0 = (int64_t)blockIdx.y * XROWS;      // more than one token tile: launches past 64 tokens (tiles of 64)
    const int64_t kbytes = p.n / 2;
    const int nl = p.n / 256;                            // lines per row
    const int nwv = blockDim.x >> 6;                     // waves: 4, 8 or 16
    const int ns = (nl - w + nwv - 1) / nwv;             // this wave's steps: lines w, w + nwv, ...
    unsigned char* ring = smem + w * depth * SLOT;

    const unsigned char* wsrc[NWI];
    const unsigned char* xsrc[NTD];
#pragma unroll
    for (int k = 0; k < NWI; ++k) {
        const int row = 8 * k + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        int orow = o0 + row;
        if (orow >= p.m) orow = p.m - 1;
        wsrc[k] = p.wc + (int64_t)orow * kbytes + 128 * w + 16 * ch;
    }
#pragma unroll
    for (int k = 0; k < NTD; ++k) {
        const int row = 8 * k + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        int64_t t = t0 + row;
        if (t >= p.T) t = p.T - 1;
        xsrc[k] = p.xc + t * kbytes + 128 * w + 16 * ch;
    }
    typedef const __attribute__((address_space(1))) void* gptr;
    typedef __attribute__((address_space(3))) void* lptr;
    auto issue = [&](int s, int slot) {
        unsigned char* base = ring + slot * SLOT;
        const int64_t off = (int64_t)s * (128 * nwv);
#pragma unroll
        for (int k = 0; k < NWI; ++k) __builtin_amdgcn_global_load_lds((gptr)(wsrc[k] + off), (lptr)(base + k * 1024), 16, 0, 0);
#pragma unroll
        for (int k = 0; k < NTD; ++k) __builtin_amdgcn_global_load_lds((gptr)(xsrc[k] + off), (lptr)(base + XOFF + k * 1024), 16, 0, 0);
    };
    i32x16 acc[NTT];
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;
    const int woff = (c & (ROWS - 1)) * 128;
    const int whs = h ^ (((c & (ROWS - 1)) >> 1) & 7);
    int xoff[NTT], xhs[NTT];
#pragma unroll
    for (int i = 0; i < NTT; ++i) {
        const int row = (32 * i + c) & (XROWS - 1);       // fewer than 32 token rows: the lanes past them repeat rows
        xoff[i] = XOFF + row * 128;
        xhs[i] = h ^ ((row >> 1) & 7);
    }
    // The epilogue's element e = tid + k blockDim is 4 output channels of one token: their steps are requested now, so
    // that the kernel's tail does not wait for them (at least 256 threads: k < NK).
    constexpr int NE = NTT * NG * 64;
    constexpr int NK = (NE + 255) / 256;
    unsigned esx[NK] = {}, esw[NK][4] = {};              // raw fp16 bits, converted in the epilogue: nothing waits for them here
    const uint16_t* xs_bits = reinterpret_cast<const uint16_t*>(p.xs);
    const uint16_t* ws_bits = reinterpret_cast<const uint16_t*>(p.ws);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int e = tid + k * (int)blockDim.x;
        const int el = e & 63, g = (e >> 6) % NG, i = (e >> 6) / NG;
        const int64_t t = t0 + 32 * i + (el & 31);
        const int o = o0 + 8 * g + 4 * (el >> 5);
        if (e < NE) {
            esx[k] = xs_bits[t < p.T ? t : p.T - 1];
#pragma unroll
            for (int x = 0; x < 4; ++x) esw[k][x] = ws_bits[o + x < p.m ? o + x : p.m - 1];
        }
    }
    const int npre = ns < depth ? ns : depth;
    for (int s = 0; s < npre; ++s) issue(s, s);
    int slot = 0;
    for (int s = 0; s < ns; ++s) {
        const int left = ns - 1 - s;
        wait_ring_step<NI>(left < depth - 1 ? left : depth - 1);
        const unsigned char* base = ring + slot * SLOT;
        u32x4 wv[4], xv[4][NTT];
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) {
            wv[kp] = *reinterpret_cast<const u32x4*>(base + woff + 16 * ((2 * kp) ^ whs));
#pragma unroll
            for (int i = 0; i < NTT; ++i) xv[kp][i] = *reinterpret_cast<const u32x4*>(base + xoff[i] + 16 * ((2 * kp) ^ xhs[i]));
        }
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) {
            i32x4 ws0, ws1;
            widen(wv[kp], ws0, ws1);
#pragma unroll
            for (int i = 0; i < NTT; ++i) {
                i32x4 xs0, xs1;
                widen(xv[kp][i], xs0, xs1);
                acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ws0, xs0, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ws1, xs1, acc[i], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read: it may take the next line
        if (s + depth < ns) issue(s + depth, slot);
        slot = (slot + 1 == depth) ? 0 : slot + 1;
    }
    wait_vm_pending<0>();
    __syncthreads();                                     // every wave is done with its ring: the partial sums go there
    i32x4* part = reinterpret_cast<i32x4*>(smem);
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g)
            part[((w * NTT + i) * NG + g) * 64 + l] = i32x4{acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
    __syncthreads();
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    const bool wide = ((reinterpret_cast<uintptr_t>(p.out) & 7) == 0) && (p.out_stride % 4 == 0);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int e = tid + k * (int)blockDim.x;
        if (e >= NE) break;
        const int el = e & 63, g = (e >> 6) % NG, i = (e >> 6) / NG;
        i32x4 sum = part[e];
        for (int ww = 1; ww < nwv; ++ww) sum += part[ww * NE + e];
        const int64_t t = t0 + 32 * i + (el & 31);
        const int o = o0 + 8 * g + 4 * (el >> 5);
        if (t < p.T && o < p.m) {
            // (the empty statement pins the conversions here: hoisted to the loads, they would stall the kernel's start)
            asm volatile("" : "+v"(esx[k]), "+v"(esw[k][0]), "+v"(esw[k][1]), "+v"(esw[k][2]), "+v"(esw[k][3]));
            const float sx = (float)__builtin_bit_cast(_Float16, (uint16_t)esx[k]);
            _Float16 v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) v[x] = (_Float16)((float)(sum[x] >> 8) * sx * (float)__builtin_bit_cast(_Float16, (uint16_t)esw[k][x]));
            _Float16* dst = p.out + t * p.out_stride + o;
            if (wide && o + 4 <= p.m) {
                *reinterpret_cast<half4*>(dst) = half4{v[0], v[1], v[2], v[3]};
            } else {
                for (int x = 0; x < 4; ++x)
                    if (o + x < p.m) dst[x] = v[x];
            }
        }
    }
}

template <int NTD, int ROWS>
static hipError_t skinny_launch_rows(const GemmDev& d, hipStream_t stream, int token_tiles) {
    if (token_tiles < 1 || (token_tiles > 1 && NTD < 4)) return hipErrorInvalidValue;   // tiles of 32 tokens or more keep their exponents inside one 128-row tile
    static OccCache oc;
    int unused = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_skinny_kernel<NTD, ROWS>), NTD >= 8 ? 512 : 1024, kRingLdsMax, oc, unused);
    if (e != hipSuccess) return e;
    constexpr int SLOT = (ROWS + 8 * NTD) * 128, NI = ROWS / 8 + NTD;
    const unsigned wgx = (unsigned)((d.m + ROWS - 1) / ROWS);
    const int64_t wgs = (int64_t)wgx * token_tiles;
    const int nl = d.n / 256;
    // One workgroup per CU (or fewer): 8 waves, so that every SIMD has two to overlap, and two slots each.  More than
    // one per CU: small workgroups (4 waves, one slot) that are all resident at once; what the second slot or the
    // other four waves would hide, the neighbouring workgroup hides.  (Measured on 4096 / 11008-wide layers.)
    const bool crowded = wgs > cu_count();
    int nwv = env_int("FLATQUANT_GEMM_WAVES", crowded ? 4 : 8);
    int depth = env_int("FLATQUANT_GEMM_DEPTH", crowded ? 1 : 2);
    if ((nwv != 4 && nwv != 8 && nwv != 16) || depth < 1 || depth > kRingMaxDepth) return hipErrorInvalidValue;
    if (NTD >= 8 && nwv > 8) nwv = 8;                                      // two token tiles of accumulators: compiled for at most 8 waves
    while (nwv > 4 && nwv * SLOT > kRingLdsMax) nwv >>= 1;
    const int steps = (nl + nwv - 1) / nwv;                               // of the wave with the most lines
    if (depth > steps) depth = steps;
    while (depth > 1 && (nwv * depth * SLOT > kRingLdsMax || (depth - 1) * NI > 63)) --depth;
    const int bytes = nwv * depth * SLOT;                                 // the partial sums (at most 4 KB per wave and token tile) reuse the rings
    return launch((w4a4_skinny_kernel<NTD, ROWS>), dim3(wgx, (unsigned)token_tiles), dim3(64 * nwv), bytes, stream, d, depth);
}
// 16 channels per workgroup while that still leaves at most one workgroup per CU (FLATQUANT_GEMM_ROWS forces 16 or 32):
// the kernel is bound by what one CU takes in, so the channels go to as many CUs as there are.
template <int NTD>
static hipError_t skinny_launch(const GemmDev& d, hipStream_t stream, int token_tiles = 1) {
    const int rows = env_int("FLATQUANT_GEMM_ROWS", (int64_t)((d.m + 15) / 16) * token_tiles <= cu_count() ? 16 : 32);
    if (rows == 16) return skinny_launch_rows<NTD, 16>(d, stream, token_tiles);
    if (rows == 32) return skinny_launch_rows<NTD, 32>(d, stream, token_tiles);
    return hipErrorInvalidValue;
}

template <bool ODD>
static hipError_t fp6_launch_rows(const GemmDev& d, hipStream_t stream) {
    using L = Fp6Tile;
    static OccCache cache;
    int occ = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_fp6_kernel<ODD>), 64 * L::NW, L::LDS, cache, occ);
    if (e != hipSuccess) return e;
    // persistent: every XCD (eight of them) gets as many workgroups as it holds at once, or as it has tiles
    const int64_t tiles = ((d.T + L::TOK - 1) / L::TOK) * ((d.m + L::CH - 1) / L::CH);
    const int64_t per_xcd = (tiles + 7) / 8, resident = (int64_t)occ * cu_count() / 8;
    const unsigned grid = 8 * (unsigned)(per_xcd < resident ? per_xcd : resident);
    return launch(w4a4_fp6_kernel<ODD>, dim3(grid), dim3(64 * L::NW), L::LDS, stream, d);
}

static hipError_t fp6_launch(const GemmDev& d, hipStream_t stream) {
    const bool odd = (reinterpret_cast<uintptr_t>(d.out) | (uintptr_t)(2 * d.out_stride)) & 3;
    return odd ? fp6_launch_rows<true>(d, stream) : fp6_launch_rows<false>(d, stream);
}

hipError_t w4a4_launch(const GemmArgs& a, hipStream_t stream) {
    int unused = 0;
    GemmDev d;
    d.xc = a.x_codes; d.xs = a.x_scales; d.wc = a.w_codes; d.ws = a.w_scales; d.out = a.out;
    d.T = a.T; d.out_stride = a.out_stride; d.m = a.m; d.n = a.n;
    if (env_int("FLATQUANT_GEMM_TILED", 0) == 0) {
        // decode and short prefill chunks: one pass over the weights, K split inside a workgroup (the ring kernel)
        if (a.T <= 8) return skinny_launch<1>(d, stream);
        if (a.T <= 16) return skinny_launch<2>(d, stream);
        if (a.T <= 32) return skinny_launch<4>(d, stream);
        if (a.T <= 64) return skinny_launch<8>(d, stream);
        // More tokens: the ring kernel on tiles of 64 tokens, as long as the 128 x 128 tiles of the kernel below would
        // reach at most half of the CUs (measured cross-over on 1024 .. 11008 channels; FLATQUANT_GEMM_RING_MAX_T
        // replaces the rule by a token count).
        const int64_t tiled_wgs = ((a.T + GT - 1) / GT) * ((a.m + GT - 1) / GT);
        const int ring_max = env_int("FLATQUANT_GEMM_RING_MAX_T", -1);
        if (ring_max >= 0 ? a.T <= ring_max : (2 * tiled_wgs <= cu_count() && a.T <= 4096))
            return skinny_launch<8>(d, stream, (int)((a.T + 63) / 64));
    }
    static OccCache ct, ctw;
    // Tile form (FLATQUANT_GEMM_WIDE forces one): int8 with 128 x 128 tiles, with 256 x 128 tiles when these still give every
    // CU a workgroup (1), or FP6 with 256 x 256 tiles (2).  A launch takes rounds of one tile per CU, measured at n = 4096: 5 + 29
    // us per round of 256 x 128 int8 tiles, 9 + 43 us per round of FP6 tiles of twice the size, whose first pass over its
    // code costs more.  Both parts grow with n, so their order holds from n = 1024 on.  (int8 / FP6, us: 2048 x 4096 x 4096 33.5 /
    // 46.4, 3000 x 4096 x 4096 58.7 / 49.3, 4096 x 4096 x 4096 64.1 / 52.6, 1024 x 11008 x 4096 57.1 / 48.9, 2048 x 11008 x 4096
    // 91.0 / 93.5, 2048 x 8192 x 14336 193 / 147, 8192 x 8192 x 1024 87.4 / 73.1, 777 x 5120 x 5120 33.2 / 49.8, 16384 x 8192 x
    // 8192 835 - 857 / 613 - 646.  FP6 with 256 x 128 and 128 x 128 tiles is bound by the vector work and gains nothing over
    // int8: 30.0 and 32.9 at 2048 x 4096 x 4096 with everything in the caches, but 41 against 39 for the whole layer on
    // fresh data.)
    // Shorter rows are one or two iterations, and output more than product: a round of FP6 tiles takes 11 us at n = 256 and 13 at
    // n = 512, one of int8 tiles 6 and 7.5, and an int8 round on a part x of the CUs takes 0.6 + 0.4 x of that.  FP6 stays
    // where its last round is nearly full (there the formula is not sharp enough) or comes out shorter all the same.  (int8 /
    // FP6: 4230 x 8320 x 256, 2.2 rounds of FP6, 32.6 / 36.7; 10622 x 8576 x 256, 5.6, 64.1 / 69.1; 13407 x 8192 x 256, 6.6, 84.7 /
    // 80.1; 4096 x 4096 x 256, 1, 16.2 / 15.2; 1429 x 8000 x 512, 0.75, 16.2 / 16.9; 9882 x 2496 x 512, 1.5, 32.3 / 29.5; 5144 x
    // 5440 x 512, 1.8, 33.3 / 29.5.)  This is for rows of whole 128-byte lines; into others the int8 kernel's output costs
    // more (1659 x 5716 x 256 29.7 / 20.0).
    const int64_t cu = cu_count();
    const int64_t wide_wgs = ((a.T + 255) / 256) * ((a.m + GT - 1) / GT), fp6_wgs = ((a.T + 255) / 256) * ((a.m + 255) / 256);
    const int64_t int8_rounds = (wide_wgs + cu - 1) / cu, fp6_rounds = (fp6_wgs + cu - 1) / cu;
    bool fp6 = wide_wgs >= cu && 9 + fp6_rounds * 43 < 5 + int8_rounds * 29;
    if (fp6 && a.n <= 512 && ((reinterpret_cast<uintptr_t>(a.out) | (uintptr_t)(2 * a.out_stride)) & 127) == 0) {
        const int64_t part = wide_wgs % cu;
        const double int8_us = 3.2 + (wide_wgs / cu + (part ? 0.6 + 0.4 * part / cu : 0.0)) * (4.4 + 0.0061 * a.n);
        const double fp6_us = 3.7 + fp6_rounds * (8.6 + 0.009 * a.n);
        const bool full = 16 * fp6_wgs >= (a.n <= 256 ? 15 : 13) * fp6_rounds * cu;
        fp6 = full || fp6_us < int8_us;
    }
    const int rule = fp6 ? 2 : wide_wgs >= cu ? 1 : 0, asked = env_int("FLATQUANT_GEMM_WIDE", rule);
    const int wide = asked >= 0 && asked <= 2 ? asked : rule;
    if (wide == 2) return fp6_launch(d, stream);
    if (wide) {
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_kernel<4>), 512, G_LDS_BYTES_WIDE, ctw, unused);
        if (e != hipSuccess) return e;
        const dim3 grid((unsigned)((a.T + 255) / 256), (unsigned)((a.m + GT - 1) / GT));
        return launch(w4a4_kernel<4>, grid, dim3(512), G_LDS_BYTES_WIDE, stream, d);
    }
    {
        hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_kernel<2>), G_NT, G_LDS_BYTES, ct, unused);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((a.T + GT - 1) / GT), (unsigned)((a.m + GT - 1) / GT));
    return launch(w4a4_kernel<2>, grid, dim3(G_NT), G_LDS_BYTES, stream, d);
}

}  // namespace fq
