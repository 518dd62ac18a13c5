// W4A4 matrix product for gfx950: out[t, o] = fp16( s_x[t] s_w[o] sum_k q_x[t, k] q_w[o, k] ), the low-bit matrix
// multiplication that consumes the two quantized factors of Eq. (2) (Sec. 3.2: low-bit matrix multiplications for all
// linear layers; Sec. 3.3: the transform + quantization kernel feeds an INT4 GEMM).
//
// Both operands arrive as packed 4-bit two's-complement codes, K contiguous (activations [T, n/2], weights [m, n/2]),
// which is the operand order of an MFMA for C = A B^T.  The codes become MFMA operands in registers, both sides in the same way,
// so that the K order inside an MFMA is the same permutation for both:
//  * int8: for a packed dword w, (w << 4) & 0xF0F0F0F0 holds 16 q of the even channels and w & 0xF0F0F0F0 holds 16 q of the odd
//    channels, as signed bytes; every product carries a factor 256.  v_mfma_i32_32x32x32_i8 accumulates in int32 (|sum| <= 128 *
//    128 * n < 2^31 for n <= 65536).
//  * FP6 (E2M3): the code offset to q + 8 = 0 .. 15 IS the bit pattern of (q + 8) / 8 (subnormal up to 7 / 8, the first binade up to
//    15 / 8), so the codes need only be spread from 4-bit to 6-bit fields.  The sums are exact: every product is an integer / 64
//    and the total at most 225 n / 64, which fits 24 bits.  The offset leaves in the epilogue, with the row sums of the codes (one
//    v_dot8 per dword) taken on the way.
// The weights are the MFMA's first operand, so that a lane ends up with runs of 4 consecutive output channels of one token.
// Many tokens take the tiled kernel, up to 64 (decode) the few-token kernel further down, and in between the one that w4a4_launch estimates to
// be faster (short prefill chunks, few output channels).
#include <cmath>
#include <type_traits>

#include "fq_internal.h"

namespace fq {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int GKB = 128;              // packed bytes of K per row and iteration (256 codes)

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

// ---- many tokens.  What bounds this kernel: a SIMD issues one instruction per 4 clocks (an MFMA takes two such slots), whether it
// holds one wave or two, so that behind a 32-clock MFMA there is room for 6 others; and the power limit, which holds the chip at
// 1.7 GHz under a full load of MFMAs (2.2 and more with half of the CUs busy).  FP6 MFMAs do twice the work of int8 ones in the same 32
// clocks, and for less power: alone, for the 2.2e12 operations of 16384 x 8192 x 8192 on random codes, 303 us, int8 531.
// Spreading the codes costs 7 instructions per 16 codes and is what an FP6 tile must save on: a wave that owns 128 x 128
// (16 MFMAs per 8 operands of 32 rows and 64 codes) spreads 7 instructions per MFMA, a 64 x 64 one 14, where int8, 6 per MFMA, is
// the faster one.  So the FP6 forms have waves of 128 x 128, one per SIMD, as large as the register file allows: 2 x 2 waves
// (256 x 256), and 2 x 1 waves with K in two parts (256 x 128, every weight row spread twice instead of the four times of 64 x 64 tiles),
// whose partial sums meet in LDS.  A row that two waves read is summed by one of them, half of the rows each: a dot product
// does not overlap with the MFMA before it (measured: two of them behind an MFMA, 54 clocks instead of 33), so those of a step stand
// together.
// 16384 x 8192 x 8192 650 -> 568 us, 4096 x 4096 x 4096 47.7 -> 41.3, 16384 x 8192 x 1024 142 -> 112 (one box; before: 8 instructions per 16
// codes, row sums by both waves and between the MFMAs, and an epilogue whose hoisted offsets went through scratch); 2048 x 4096 x 8192
// 55.5 -> 43.8 in 256 x 128 tiles.
constexpr unsigned kSpreadA0 = 0x0F00F00Fu, kSpreadA1 = 0xF00F00F0u, kSpreadA2 = 0x00F00F00u;   // fields that do not move
constexpr unsigned kSpreadM0 = 0xCF3CF3CFu, kSpreadM1 = 0xF3CF3CF3u, kSpreadM2 = 0x3CF3CF3Cu;   // the low 4 bits of all fields
constexpr unsigned kSpreadX0 = 0x08208208u, kSpreadX1 = 0x82082082u, kSpreadX2 = 0x20820820u;   // bit 3 of all fields
// 16 codes -> 16 fields of 6 bits in three dwords.  Every nibble stays or moves up by 2 bits, into the next dword where it
// straddles the end (fields in order: nibbles 0 1 3 4 6 7 of lo, 1 2 4 5 7 0 of hi, 2 of lo, 3 of hi, 5 of lo, 6 of hi).  One 64-bit
// shift serves all that move; then mask ? stay : moved (0xca) and (v & fields) ^ bit 3 (0x6a) per dword: 7 instructions of 4
// clocks.  One block, because the compiler takes the shift apart into five.
__device__ __forceinline__ void spread16(unsigned lo, unsigned hi, unsigned* o) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    asm("v_lshlrev_b64 v[254:255], 2, %3\n\t"
        "v_bitop3_b32 %0, %6, %4, v254 bitop3:0xca\n\t"
        "v_bitop3_b32 %1, %7, %5, v255 bitop3:0xca\n\t"
        "v_bitop3_b32 %2, %8, %4, v255 bitop3:0xca\n\t"
        "v_bitop3_b32 %0, %0, %9, %12 bitop3:0x6a\n\t"
        "v_bitop3_b32 %1, %1, %10, %13 bitop3:0x6a\n\t"
        "v_bitop3_b32 %2, %2, %11, %14 bitop3:0x6a"
        : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2])
        : "v"(u32x2{lo, hi}), "v"(lo), "v"(hi), "s"(kSpreadA0), "s"(kSpreadA1), "s"(kSpreadA2), "s"(kSpreadM0), "s"(kSpreadM1), "s"(kSpreadM2),
          "v"(kSpreadX0), "v"(kSpreadX1), "v"(kSpreadX2)
        : "v254", "v255");
}

// A tile form: MFMA tiles of 32 x 32 per wave (tokens x channels), waves (tokens x channels x parts of K), LDS stages, waves
// per SIMD.
template <bool FP6_, int TI_, int TJ_, int WM_, int WN_, int KS_, int NST_, int WPE_>
struct Tile {
    static constexpr bool FP6 = FP6_;
    static constexpr int TI = TI_, TJ = TJ_, WM = WM_, WN = WN_, KS = KS_, NST = NST_, WPE = WPE_;
    static constexpr int NW = WM * WN * KS;
    static constexpr int TOK = 32 * TI * WM, CH = 32 * TJ * WN, ROWS = TOK + CH;
    static constexpr int STAGE = ROWS * GKB;                        // code tiles of one K iteration
    static constexpr int OPITCH = 64 * TJ + 16;                     // output staging: 32 tokens of a wave's channels
    static constexpr int WCOL = 32 * TJ * 4;                        // steps of a wave's channels
    static constexpr int SUMS = NST * STAGE + NW * WCOL;            // row sums of the tile, for each part of K
    static constexpr int LDS = SUMS + (FP6 ? 4 * KS * ROWS : 0);
    static_assert(NW * 32 * OPITCH <= STAGE && LDS <= 160 * 1024 && NST >= 2, "LDS budget");
    static_assert(TOK / 8 % NW == 0 && CH / 8 % NW == 0, "loads are whole groups of 8 rows per wave");
    static_assert(!FP6 || (TI == 4 && TJ == 4), "a spread block and the MFMA that reads it: see the steps");
    static_assert(KS == 1 || (KS == 2 && FP6 && TI % 2 == 0 && WN == 1 && NST >= 3), "the two waves that share a tile finish half of its tokens each");
};

// Every operand byte goes from global memory straight into LDS (global-to-LDS loads, unpadded 128-byte rows, 16-byte chunks
// swizzled), NST iterations of 256 codes deep, one barrier per iteration; persistent workgroups whose loads run on from one
// output tile into the next.  The output leaves through LDS in 16-byte pieces, by buffer stores without branches where all rows
// are made of such pieces.  OUT: how it leaves (tiled_output).  odd: the output's rows are not all dword-aligned and leave in
// halves, by a loop that only such launches carry (6486 x 5705 x 256 61 us, 82 with the halves of 16-byte pieces stored one by one).
template <class L, Out OUT>
__global__ __launch_bounds__(64 * L::NW) __attribute__((amdgpu_waves_per_eu(L::WPE, L::WPE))) void w4a4_tiled_kernel(GemmDev p) {
    constexpr bool FP6 = L::FP6, ODD = OUT == Out::odd;
    constexpr int TI = L::TI, TJ = L::TJ, WM = L::WM, WN = L::WN, NST = L::NST;
    constexpr int NW = L::NW, TOK = L::TOK, CH = L::CH, STAGE = L::STAGE, A_TILE = TOK * GKB, NOP = TI + TJ;
    constexpr int NLA = TOK / 8 / NW, NLB = CH / 8 / NW, NL = NLA + NLB;   // load instructions per wave and iteration
    constexpr int KS = L::KS, NKP = GKB / 32 / KS;                  // K steps (64 codes) per wave and iteration
    constexpr int LA = 2, KB = NKP - LA;                            // operands are read LA steps ahead; the steps before the barrier
    constexpr int NQ = TI * TJ * (FP6 ? 1 : 2);                     // MFMAs per step
    constexpr int WD = FP6 ? 3 : 4;                                 // dwords of an operand register per 16 codes
    constexpr int LSTEPS = NST == 2 || NKP == 2 ? 2 : NKP;                                       // steps over which an iteration's loads are spread
    static_assert(NKP == 4 || NKP == 2, "register stages below");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w % WM, wn = w / WM % WN, ks = w / (WM * WN);
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
    // Rows past the end are out of the buffer's range and read as zeros.
    __amdgpu_buffer_rsrc_t abuf, bbuf;
    uint32_t aoff[NLA], boff[NLB];
#pragma unroll
    for (int k = 0; k < NLA; ++k) {
        const int row = 8 * (NLA * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        aoff[k] = (uint32_t)row * (uint32_t)kbytes + 16 * ch;
    }
#pragma unroll
    for (int k = 0; k < NLB; ++k) {
        const int row = 8 * (NLB * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
        boff[k] = (uint32_t)row * (uint32_t)kbytes + 16 * ch;
    }
    auto set_source = [&](const Pos& t) {
        const int arows = (int)(p.T - t.t0 < TOK ? p.T - t.t0 : TOK), brows = p.m - t.o0 < CH ? p.m - t.o0 : CH;
        abuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.xc) + t.t0 * kbytes, 0, arows * (int)kbytes, 0x00020000);
        bbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p.wc) + (int64_t)t.o0 * kbytes, 0, brows * (int)kbytes, 0x00020000);
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

    // ---- operands.  x < TI: tokens 32 tok_tile(x) + c; else channels 32 ch_tile(x - TI) + c
    const int hs = h ^ ((c >> 1) & 7);   // chunk 2 kp + h of row 32 x + c sits in slot (2 kp) ^ hs
    const int atile = TI * wm, btile = TJ * wn;                     // first 32-row tiles of this wave
    // A wave takes the tiles of its rows in an order of its own.  FP6: of the waves that read the same codes each sums a part of the
    // rows, its first HA token and HB channel tiles; with K in two parts each wave finishes its first half of the tokens.
    constexpr int HA = FP6 && L::WN == 2 ? (TI + 1) / 2 : TI, HB = FP6 && WM == 2 ? (TJ + 1) / 2 : TJ, IH = TI / KS;
    const int arot = KS == 2 ? IH * ks : (TI - HA) * wn, brot = (TJ - HB) * wm;
    constexpr int AH = KS == 2 ? IH : HA;
    auto tok_tile = [&](int i) { return atile + (i < AH ? i + arot : i - (KS == 2 ? AH * ks : AH * wn)); };
    auto ch_tile = [&](int j) { return btile + (j < HB ? j + brot : j - HB * wm); };
    int lane_byte[NKP];                  // this lane's chunk of K step kp in a 32-row tile
#pragma unroll
    for (int kp = 0; kp < NKP; ++kp) lane_byte[kp] = c * GKB + 16 * ((2 * (NKP * ks + kp)) ^ hs);
    auto lds_chunk = [&](int stage, int kp, int x) -> u32x4 {
        const int a = stage + (x < TI ? 32 * GKB * tok_tile(x) : A_TILE + 32 * GKB * ch_tile(x - TI));   // scalar
        return *reinterpret_cast<const u32x4*>(smem + a + lane_byte[kp]);
    };
    // Three register stages: while the MFMAs of step kp run on the FP6 operands W[kp & 1], the packed codes P of step kp + 1
    // are spread into W[(kp + 1) & 1], and as each operand has been spread its registers take the codes of step kp + 2 from
    // LDS.  A wave issues in order, so the vector work stands between the MFMAs, a share behind each.
    typedef typename std::conditional<FP6, f32x16, i32x16>::type acc_t;
    acc_t acc[TI][TJ];
    u32x4 P[NOP];
    unsigned W[2][NOP][2 * WD];
    int rsum[NOP];                       // FP6: sums of this lane's codes, of the rows that this wave sums
    auto mfma = [&](int m, int st, bool first) {     // m-th MFMA of a step; the first step of a tile starts from zero
        const int i = m / TJ % TI, j = m % TJ;
        const unsigned *wv = W[st][TI + j], *xv = W[st][i];
        acc_t from = acc[i][j];
        if (first && m < TI * TJ)
#pragma unroll
            for (int r = 0; r < 16; ++r) from[r] = 0;
        if constexpr (FP6) {             // FP6 E2M3 for both, no scale
            const i32x8 a = {(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3], (int)wv[4], (int)wv[5], 0, 0};
            const i32x8 b = {(int)xv[0], (int)xv[1], (int)xv[2], (int)xv[3], (int)xv[4], (int)xv[5], 0, 0};
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, from, 2, 2, 0, 0, 0, 0);
        } else {
            const int s = 4 * (m / (TI * TJ));
            const i32x4 a = {(int)wv[s], (int)wv[s + 1], (int)wv[s + 2], (int)wv[s + 3]};
            const i32x4 b = {(int)xv[s], (int)xv[s + 1], (int)xv[s + 2], (int)xv[s + 3]};
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, from, 0, 0, 0);
        }
    };
    // operands are spread in the order in which the MFMAs of a step ask for them: channels, then tokens
    auto operand = [&](int u) { return (u >> 1) < TJ ? TI + (u >> 1) : (u >> 1) - TJ; };
    auto spread = [&](int st, int u) {   // half u & 1 of operand(u): 16 codes
        const int x = operand(u), s = u & 1;
        const unsigned lo = P[x][2 * s], hi = P[x][2 * s + 1];
        unsigned* o = &W[st][x][WD * s];
        if constexpr (FP6) {
            spread16(lo, hi, o);
        } else {
            constexpr unsigned M = 0xF0F0F0F0u;
            o[0] = (lo << 4) & M; o[1] = lo & M; o[2] = (hi << 4) & M; o[3] = hi & M;
        }
    };
    // Row sums of the codes in P.  A dot product waits for the matrix pipe to drain (measured: 22 clocks longer than its own 4 when
    // it follows an MFMA), so all of a step's stand in one place.
    auto row_sums = [&]() {
#pragma unroll
        for (int x = 0; x < NOP; ++x)
            if (x < TI ? x < HA : x - TI < HB)
#pragma unroll
                for (int k = 0; k < 4; ++k) rsum[x] = __builtin_amdgcn_sdot8((int)P[x][k], 0x11111111, rsum[x], false);
    };
    // K step kp and a share of the loads of iteration `lit` into `stage_load`.  Steps KB .. NKP - 1 of an iteration, then
    // 0 .. KB - 1 of the next one, lie between two barriers: s is the step's place in that sequence, which the loads are
    // spread over.  `next`: there is a next step in this tile.
    auto step = [&](int kp, int stage_ahead, int lit, int stage_load, int s, int s0, int nsteps, bool next, bool first) __attribute__((always_inline)) {
        if constexpr (FP6)
            if (next) row_sums();
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
            mfma(m, kp & 1, first);
#pragma unroll
            for (int u = m * 2 * NOP / NQ; next && u < (m + 1) * 2 * NOP / NQ; ++u) {
                spread((kp + 1) & 1, u);
                if (u & 1) P[operand(u)] = lds_chunk(stage_ahead, (kp + LA) % NKP, operand(u));
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
        for (int x = 0; x < NOP; ++x) rsum[x] = 0;
        if constexpr (FP6) row_sums();
#pragma unroll
        for (int u = 0; u < 2 * NOP; ++u) spread(0, u);
        if constexpr (FP6) {
            // An MFMA needs wait states after the vector instructions that wrote its operands, and the compiler does not see those
            // in spread16's block.  Inside the steps other MFMAs stand between: the operand spread last is the one read last.
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 7" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        read_step(st, 1);
        // steps 0 .. KB - 1 of iteration 0; loads of iteration NST - 1
        if constexpr (KB == 0) issue(NST - 1, stl, 0, NL);
#pragma unroll
        for (int kp = 0; kp < KB; ++kp) step(kp, st, NST - 1, stl, kp, 0, LSTEPS < KB ? LSTEPS : KB, true, kp == 0);
        arrive();
        int lit = NST;                       // iteration to be loaded next
        auto body = [&](bool first) __attribute__((always_inline)) {
            const int stn = advance(st);
            stl = advance(stl);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, lit, stl, kp - KB, 0, LSTEPS, true, first && kp == 0);
#pragma unroll
            for (int kp = 0; kp < KB; ++kp) step(kp, stn, lit, stl, kp + LA, 0, LSTEPS, true, false);
            arrive();
            st = stn;
            ++lit;
        };
        int it = 0;
        if constexpr (KB == 0) {
            if (nk > NST) {
                body(true);
                ++it;
            } else {
#pragma unroll
                for (int i = 0; i < TI; ++i)
#pragma unroll
                    for (int j = 0; j < TJ; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
            }
        }
        for (; it < nk - 1 && lit < nk; ++it) body(false);
        const int64_t qn = q + qstep;
        const bool more = qn < mine;
        Pos nxt = cur;
        if (more) nxt = tile_pos(qn);
        if (more && flow) { set_source(nxt); lit = 0; }
        for (; it < nk - 1; ++it) body(false);
        // the quantization steps of this tile's rows and channels, requested ahead of the epilogue (raw bits: nothing waits here)
        const uint16_t* xs_bits = reinterpret_cast<const uint16_t*>(p.xs);
        const uint16_t* ws_bits = reinterpret_cast<const uint16_t*>(p.ws);
        unsigned esx[IH], esw[TJ];
#pragma unroll
        for (int i = 0; i < IH; ++i) {
            const int64_t t = cur.t0 + 32 * tok_tile(i) + c;
            esx[i] = xs_bits[t < p.T ? t : p.T - 1];
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int o = cur.o0 + 32 * ch_tile(j) + c;
            esw[j] = ws_bits[o < p.m ? o : p.m - 1];
        }
        // the last steps of the tile: nothing is loaded, the current stage takes the output tile
        {
            const int stn = advance(st);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, 0, 0, 0, 1, 0, kp + 1 < NKP, false);
        }
        __builtin_amdgcn_sched_barrier(0);

        // epilogue: in acc[i][j] a lane holds, for token 32 tok_tile(i) + c, the output channels 32 ch_tile(j) + 8 (r / 4) +
        // 4 h + r % 4.  Rounded to fp16 and turned, 32 tokens at a time, through a part of LDS that belongs to the wave
        // alone (no barrier), from where they leave in 16-byte pieces of whole rows.  FP6: all corrections are integers
        // below 2^24, so their fp32 sums are exact.  int8: every sum is a multiple of 256 (both operands carry a factor 16).
        typedef _Float16 half4 __attribute__((ext_vector_type(4)));
        constexpr int OPITCH = L::OPITCH, CPR = 4 * TJ;              // 16-byte pieces per token
        unsigned char* ot = smem + st + w * (32 * OPITCH);
        float* wcol = reinterpret_cast<float*>(smem + NST * STAGE + w * L::WCOL);   // [32 TJ] steps of this wave's channels
        int* sums = reinterpret_cast<int*>(smem + L::SUMS);      // FP6: sums of q + 8 of the tile's tokens, then channels, for each part of K
#pragma unroll
        for (int j = 0; j < TJ; ++j) wcol[32 * j + c] = (float)__builtin_bit_cast(_Float16, (uint16_t)esw[j]); // both halves of the wave store the same
        if constexpr (FP6) {
#pragma unroll
            for (int x = 0; x < HA; ++x) sums[ks * L::ROWS + 32 * tok_tile(x) + c] = rsum[x] + __shfl_xor(rsum[x], 32) + 8 / KS * p.n;
#pragma unroll
            for (int x = 0; x < HB; ++x) sums[ks * L::ROWS + TOK + 32 * ch_tile(x) + c] = rsum[TI + x] + __shfl_xor(rsum[TI + x], 32) + 8 / KS * p.n;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        if constexpr (KS == 2) {
            // The other part of K: this wave's second half of the tokens goes to its partner, whose second half is this wave's first;
            // through the free stage, a few tiles at a time.  The sums stay exact.
            constexpr int UPP = STAGE / NW / 4096, US = IH * TJ;     // tiles per turn, and in all
            static_assert(UPP >= 1, "room for a tile per wave");
            f32x4* mine_x = reinterpret_cast<f32x4*>(smem + st + w * (UPP * 4096)) + l;
            const f32x4* theirs = reinterpret_cast<const f32x4*>(smem + st + (w ^ (WM * L::WN)) * (UPP * 4096)) + l;
#pragma unroll
            for (int u0 = 0; u0 < US; u0 += UPP) {
#pragma unroll
                for (int u = u0; u < u0 + UPP && u < US; ++u)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const acc_t& a = acc[IH + u / TJ][u % TJ];
                        mine_x[(u - u0) * 256 + q4 * 64] = f32x4{(float)a[4 * q4], (float)a[4 * q4 + 1], (float)a[4 * q4 + 2], (float)a[4 * q4 + 3]};
                    }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int u = u0; u < u0 + UPP && u < US; ++u)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x4 v = theirs[(u - u0) * 256 + q4 * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[u / TJ][u % TJ][4 * q4 + e] += v[e];
                    }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
        }
        if constexpr (FP6) {
            // sum q_x q_w = 64 (sum of products of (q + 8) / 8 - row sum of tokens - row sum of channels + n): one more MFMA per
            // tile adds the last three, each sum as 64 s1 + s0 (s1 < 2^11, s0 a multiple of 1 / 8 below 64).  All partial sums are
            // multiples of 1 / 64 below 2^18: exact.
            half8 ax[IH], bw[TJ];
            auto pieces = [&](int row, _Float16& s1, _Float16& s0) {
                const int sum = sums[row] + (KS == 2 ? sums[L::ROWS + row] : 0);
                s1 = (_Float16)(float)(sum >> 9);
                s0 = (_Float16)((float)(sum & 511) * 0.125f);
            };
            const half8 none = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < IH; ++i) {
                half8 v = {-64, -1, 0, 0, 256, 0, 0, 0};
                _Float16 s1, s0;
                pieces(32 * tok_tile(i) + c, s1, s0);
                v[2] = s1; v[3] = s0;
                ax[i] = h ? none : v;
            }
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                half8 v = {0, 0, -64, -1, 0, 0, 0, 0};
                _Float16 s1, s0;
                pieces(TOK + 32 * ch_tile(j) + c, s1, s0);
                v[0] = s1; v[1] = s0; v[4] = (_Float16)(float)(p.n / 256);
                bw[j] = h ? none : v;
            }
#pragma unroll
            for (int i = 0; i < IH; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bw[j], ax[i], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float4 sw[TJ][4];                                            // steps of this lane's channels
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) sw[j][g] = *reinterpret_cast<const float4*>(wcol + 32 * j + 8 * g + 4 * h);
        const uintptr_t pitch_bits = reinterpret_cast<uintptr_t>(p.out) | (uintptr_t)(2 * p.out_stride);
        const bool wide = (pitch_bits & 15) == 0, pairs = (pitch_bits & 3) == 0;   // whole pieces, dwords, or halves
        // Whole pieces only: buffer stores from one scalar base, with an offset out of range for pieces outside the output.
        const bool whole = !ODD && wide && p.m % 8 == 0 && p.out_stride < (1 << 20);
        int64_t stride = p.out_stride;
        int lane = l;
        asm volatile("" : "+s"(stride), "+v"(lane));                 // offsets are made here, not kept (and spilled) through the main loop
        const int pitch = (int)(2 * stride);
        const int rows_left = (int)(p.T - cur.t0 < TOK ? p.T - cur.t0 : TOK);
        const __amdgpu_buffer_rsrc_t obuf = __builtin_amdgcn_make_buffer_rsrc(p.out + cur.t0 * stride + cur.o0, 0, 0x40000000, 0x00020000);
        auto scaled = [&](int i, int j, int r, float sx) {
            float v = (float)acc[i][j][r] * sx * reinterpret_cast<const float*>(&sw[j][r >> 2])[r & 3];
            asm("" : "+v"(v));               // rounded to fp32 as it stands, not inside a mixed-precision fma: the same bits in every form
            return (_Float16)v;
        };
#pragma unroll
        for (int i = 0; i < IH; ++i) {
            const float sx = (float)__builtin_bit_cast(_Float16, (uint16_t)esx[i]) * (FP6 ? 64.0f : 1.0f / 256);   // the sums' unit
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<half4*>(ot + c * OPITCH + 64 * j + 16 * g + 8 * h) =
                        half4{scaled(i, j, 4 * g, sx), scaled(i, j, 4 * g + 1, sx), scaled(i, j, 4 * g + 2, sx), scaled(i, j, 4 * g + 3, sx)};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if constexpr (ODD) {             // 64 consecutive halves per instruction: whole lines as far as they go
                const int64_t t = cur.t0 + 32 * tok_tile(i);
                const int rows = (int)(p.T - t < 32 ? p.T - t : 32);
                _Float16* dst = p.out + t * stride + cur.o0;
#pragma unroll 4
                for (int row = 0; row < rows; ++row, dst += stride)
#pragma unroll
                    for (int x = 0; x < (TJ + 1) / 2; ++x) {
                        const int e = lane + 64 * x, j = 2 * x + h;                    // column of the staged row, and its tile
                        if (TJ % 2 && j >= TJ) continue;
                        const int o = 32 * ch_tile(j) + c;
                        const _Float16 v = *reinterpret_cast<const _Float16*>(ot + row * OPITCH + 2 * e);
                        if (cur.o0 + o < p.m) dst[o] = v;
                    }
            } else if (whole) {
#pragma unroll
                for (int k = 0; k < 32 * CPR / 64; ++k) {
                    const int e = lane + 64 * k, ch = e % CPR, r = e / CPR;
                    const int o = 32 * ch_tile(ch >> 2) + 8 * (ch & 3), row = 32 * tok_tile(i) + r;
                    const int col = cur.o0 + o < p.m ? 2 * o : 0x40000000;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(ot + r * OPITCH + 16 * ch);
                    __builtin_amdgcn_raw_buffer_store_b128(v, obuf, row < rows_left ? row * pitch + col : 0x40000000, 0, OUT == Out::through ? 16 : 0);   // 16: sc1
                }
            } else {                         // `pairs` holds (the same loop without the test measured 1 - 2 % slower)
#pragma unroll
                for (int k = 0; k < 32 * CPR / 64; ++k) {
                    const int e = lane + 64 * k, row = e / CPR, ch = e % CPR, j = ch >> 2;
                    const int64_t t = cur.t0 + 32 * tok_tile(i) + row;
                    const int o = cur.o0 + 32 * ch_tile(j) + 8 * (ch & 3);
                    const u32x4 v = *reinterpret_cast<const u32x4*>(ot + row * OPITCH + 16 * ch);
                    if (t < p.T && o < p.m) {
                        _Float16* dst = p.out + t * stride + o;
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

// ---- few tokens (decode, short prefill chunks): the weights are read once per tile of up to 64 tokens, and what bounds the kernel is
// memory (the weights at 5 TB/s behind 2.4 us of launch and first latency) or how fast the CUs take in their rows (45 KB per us each).  A
// workgroup owns 16 to 64 output channels for 8 to 64 tokens, whatever spreads the rows best (ring_shape).  Every operand byte goes from global memory
// straight into LDS, a whole cache line per row at a time: a wave owns every nwv-th 128-byte line of K (256 codes) of
// the workgroup's weight rows and of the token rows, with a ring of `depth` line slots of its own in LDS.  One
// global-to-LDS instruction moves 8 whole rows; the wave waits only for its own oldest slot (no barrier in the loop),
// multiplies it and requests the line `depth` steps ahead into the same slot.  The slots use the swizzle of the tiled
// kernel (slot chunk j of row r holds the row's chunk j ^ ((r >> 1) & 7)).  The partial sums of the waves are added
// through LDS at the end.  (Arguments are plain and in the order they are needed: they arrive in registers at wave start.  One
// token, 4096 x 4096: MXFP4 4.25 -> 4.02 us, 23 x 11008 x 4096 7.7 -> 7.4.  Touching the later lines at the start, to have them in L2
// in time, is slower: 8 x 4096 x 11008 7.4 -> 9.0 us, as is a deeper ring, 8.4.  Feeding the MFMA from registers instead, 32 bytes of 32 rows per load, costs four
// instructions and tag look-ups per cache line and holds far less in flight: 1.5 to 3 times slower.)
// NTD: token rows in groups of 8 (one load instruction each): 1, 2, 4, 8 for tiles of 8, 16, 32, 64 tokens.  ROWS output channels;
// where the last MFMA tile has 16 of them, its upper 16 rows repeat the lower ones and are dropped.
template <int NTD, int ROWS>
__global__ __launch_bounds__(ring_max_waves(NTD, ROWS) * 64) void w4a4_skinny_kernel(const uint8_t* wc, const uint8_t* xc, const _Float16* ws, const _Float16* xs, _Float16* out,
                                                                             int n, int m, int T, RingConfig cfg, int64_t out_stride) {
    static_assert(ROWS == 16 || ROWS == 32 || ROWS == 48 || ROWS == 64, "weight rows per workgroup");
    constexpr int NWI = ROWS / 8;                        // load instructions per line of the weight rows
    constexpr int NG = ROWS / 8;                         // groups of 8 output channels
    constexpr int NCT = (ROWS + 31) / 32;                // MFMA channel tiles of 32
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int NTT = NTD > 4 ? NTD / 4 : 1;           // MFMA token tiles of 32
    constexpr int XROWS = 8 * NTD;
    constexpr int XOFF = ROWS * 128;
    constexpr int SLOT = (ROWS + XROWS) * 128;           // weight rows, then token rows, one line each
    constexpr int NI = NWI + NTD;                        // load instructions per step
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RingTile wg = ring_tile(blockIdx.x, (m + ROWS - 1) / ROWS, cfg, T / 2 > m);
    if (wg.channels < 0) return;
    const int o0 = wg.channels * ROWS;
    const int t0 = wg.tokens * XROWS;
    const uint32_t kbytes = (uint32_t)(n / 2);
    const int nl = n / 256;                              // lines per row
    const int nwv = cfg.waves(), depth = cfg.depth();
    const int ns = (nl - w + nwv - 1) >> cfg.log2_waves();   // this wave's steps: lines w, w + nwv, ...
    unsigned char* ring = smem + w * depth * SLOT;

    // Row 8 k + l / 8, the chunk that belongs into slot l % 8 of it: one offset per k for both operands, from a scalar base each.
    // Rows past the end are out of the buffers' range and read as zeros.  (With 64-bit addresses and clamped rows the first
    // request left after some 500 instructions, 1 us.)
    const int mrows = m - o0 < ROWS ? m - o0 : ROWS, trows = T - t0 < XROWS ? T - t0 : XROWS;
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wc) + (int64_t)o0 * kbytes, 0, mrows * (int)kbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(xc) + (int64_t)t0 * kbytes, 0, trows * (int)kbytes, 0x00020000);
    constexpr int NV = NWI > NTD ? NWI : NTD;
    uint32_t voff[NV];
    {
        const uint32_t r = l >> 3, first = r * kbytes + 128 * w, ch = (l & 7) ^ (r >> 1);
#pragma unroll
        for (int k = 0; k < NV; ++k) voff[k] = first + 16 * (k & 1 ? ch ^ 4 : ch) + 8 * k * kbytes;
    }
    typedef __attribute__((address_space(3))) void* lptr;
    auto issue = [&](int s, int slot) {
        unsigned char* base = ring + slot * SLOT;
        const int off = s * (128 * nwv);
#pragma unroll
        for (int k = 0; k < NWI; ++k) __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (lptr)(base + k * 1024), 16, (int)voff[k], off, 0, 0);
#pragma unroll
        for (int k = 0; k < NTD; ++k) __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (lptr)(base + XOFF + k * 1024), 16, (int)voff[k], off, 0, 0);
    };
    const int npre = ns < depth ? ns : depth;
#pragma unroll 1
    for (int s = 0; s < npre; ++s) issue(s, s);
    // The epilogue's element e = tid + k blockDim is 4 output channels of one token: their steps are requested now, behind the
    // first lines, so that the kernel's tail does not wait for them (at least 256 threads: k < NK; elements past the last one
    // are out of the tokens' range).
    constexpr int NE = NTT * NG * 64;
    constexpr int NK = (NE + 255) / 256;
    _Float16 esx[NK], esw[NK][4];                        // converted in the epilogue: nothing waits for them here
    const __amdgpu_buffer_rsrc_t sxbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(xs) + t0, 0, 2 * (T - t0 < 32 * NTT ? T - t0 : 32 * NTT), 0x00020000);
    const __amdgpu_buffer_rsrc_t swbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(ws) + o0, 0, 2 * mrows, 0x00020000);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int e = tid + (k << (6 + cfg.log2_waves()));
        const int el = e & 63, g = (e >> 6) % NG, i = (e >> 6) / NG;
        esx[k] = __builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(sxbuf, 2 * (32 * i + (el & 31)), 0, 0));
#pragma unroll
        for (int x = 0; x < 4; ++x) esw[k][x] = __builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(swbuf, 2 * (8 * g + 4 * (el >> 5) + x), 0, 0));
    }
    i32x16 acc[NTT][NCT];
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int j = 0; j < NCT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    int woff[NCT], whs[NCT];
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
        const int row = 32 * j + (c & (ROWS - 32 * j >= 32 ? 31 : 15));
        woff[j] = row * 128;
        whs[j] = h ^ ((row >> 1) & 7);
    }
    int xoff[NTT], xhs[NTT];
#pragma unroll
    for (int i = 0; i < NTT; ++i) {
        const int row = (32 * i + c) & (XROWS - 1);       // fewer than 32 token rows: the lanes past them repeat rows
        xoff[i] = XOFF + row * 128;
        xhs[i] = h ^ ((row >> 1) & 7);
    }
    int slot = 0;
    for (int s = 0; s < ns; ++s) {
        const int left = ns - 1 - s;
        wait_ring_step<NI>(left < depth - 1 ? left : depth - 1);   // (the first time the quantization steps as well: they are younger, and not counted)
        const unsigned char* base = ring + slot * SLOT;
        u32x4 wv[4][NCT], xv[4][NTT];
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) {
#pragma unroll
            for (int j = 0; j < NCT; ++j) wv[kp][j] = *reinterpret_cast<const u32x4*>(base + woff[j] + 16 * ((2 * kp) ^ whs[j]));
#pragma unroll
            for (int i = 0; i < NTT; ++i) xv[kp][i] = *reinterpret_cast<const u32x4*>(base + xoff[i] + 16 * ((2 * kp) ^ xhs[i]));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read: it may take the next line
        if (s + depth < ns) issue(s + depth, slot);
#pragma unroll
        for (int kp = 0; kp < 4; ++kp) {
            i32x4 ws0[NCT], ws1[NCT];
#pragma unroll
            for (int j = 0; j < NCT; ++j) widen(wv[kp][j], ws0[j], ws1[j]);
#pragma unroll
            for (int i = 0; i < NTT; ++i) {
                i32x4 xs0, xs1;
                widen(xv[kp][i], xs0, xs1);
#pragma unroll
                for (int j = 0; j < NCT; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ws0[j], xs0, acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < NCT; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ws1[j], xs1, acc[i][j], 0, 0, 0);
            }
        }
        slot = (slot + 1 == depth) ? 0 : slot + 1;
    }
    wait_vm_pending<0>();
    __syncthreads();                                     // every wave is done with its ring: the partial sums go there
    i32x4* part = reinterpret_cast<i32x4*>(smem);
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g)
            part[((w * NTT + i) * NG + g) * 64 + l] = i32x4{acc[i][g / 4][4 * (g % 4)], acc[i][g / 4][4 * (g % 4) + 1], acc[i][g / 4][4 * (g % 4) + 2], acc[i][g / 4][4 * (g % 4) + 3]};
    __syncthreads();
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    const bool wide = ((reinterpret_cast<uintptr_t>(out) & 7) == 0) && (out_stride % 4 == 0);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int e = tid + (k << (6 + cfg.log2_waves()));
        if (e >= NE) break;
        const int el = e & 63, g = (e >> 6) % NG, i = (e >> 6) / NG;
        i32x4 sum = part[e];
        for (int ww = 1; ww < nwv; ++ww) sum += part[ww * NE + e];
        const int t = t0 + 32 * i + (el & 31);
        const int o = o0 + 8 * g + 4 * (el >> 5);
        if (t < T && o < m) {
            // (the empty statement pins the conversions here: hoisted to the loads, they would stall the kernel's start)
            asm volatile("" : "+v"(esx[k]), "+v"(esw[k][0]), "+v"(esw[k][1]), "+v"(esw[k][2]), "+v"(esw[k][3]));
            const float sx = (float)esx[k];
            _Float16 v[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                float y = __builtin_fmaf((float)(sum[x] >> 8) * sx, (float)esw[k][x], 0.0f);
                asm("" : "+v"(y));           // rounded to fp32 as it stands, as in the tiled kernel: the same bits whichever of the two runs (the fma takes the step as fp16)
                v[x] = (_Float16)y;
            }
            _Float16* dst = out + t * out_stride + o;
            if (wide && o + 4 <= m) {
                *reinterpret_cast<half4*>(dst) = half4{v[0], v[1], v[2], v[3]};
            } else {
                for (int x = 0; x < 4; ++x)
                    if (o + x < m) dst[x] = v[x];
            }
        }
    }
}

// What a launch of the few-token kernels takes, for a workgroup of `tokens` x `rows`: a fixed part, the lines of 256 codes that a wave
// works on one after the other, the operand rows that the fullest CU and that all CUs take in per line, the products of all CUs and
// of one wave, the partial sums that meet in LDS, and the weights.  Fits to about 500 launches per format of 1 <= T <= 4000,
// 256 <= m <= 14336, 256 <= n <= 28672, 8 to 24 shapes each, with the weights in memory and in the last-level cache (so the weights' term is no
// memory rate: 16 to 39 TB/s).  Against a single shape per T and one rule on workgroups (64 tokens from 33 on; 32 channels, or 16 while no
// CU has more than one workgroup of those; 8 waves while none has more than one, else 4), us: INT4 64 x 4096 x 11008 12.0, here 9.6 in 32 x 32;
// 45 x 1408 x 12288 9.8 / 7.0 in 32 x 16; 45 x 8666 x 11008 20.0 / 16.5 in 64 x 48; 230 x 7936 x 14336 44 / 33 in 64 x 64; MXFP4 42 x 1664 x 28672 20.6 / 13.3.
// The estimates are off by 6 % (more than two workgroups per CU: 10 to 30 % too low), so up to 32 tokens, where that rule's tokens and channels
// are rarely far from the best, other channels have to promise 5 % (INT4 2 x 14336 x 2048 4.9 -> 4.1, 13824 x 3072 6.1 -> 4.7); and 16 channels in 4
// waves are not taken for more tokens and workgroups than CUs (INT4 213 x 4096 x 256 4.6 -> 3.7, 1638 x 512 x 1280 6.4 -> 5.1).  4000 launches per
// format against that rule: 5 % faster up to 32 tokens (MXFP4 6), 16 up to 64, 11 up to 256, 7 beyond (MXFP4 9); 3 % of them more than 3 % slower
// up to 32 tokens, 5 % beyond (MXFP4 none and 3).
// Waves and slots: 8 waves give every SIMD two to overlap where CUs have one workgroup; where they have more, small ones (4 waves)
// that are all resident overlap each other.  A second slot per wave helps MXFP4 (T = 2, 1792 x 28672: 9.4 us, 12.6 with one), whose
// steps are shorter; INT4 is faster without (53 x 2960 x 11008 8.1 / 7.6: memory does better with fewer lines asked for) unless few tokens leave
// it 16 lines per wave or more (1 x 2250 x 65536 26.6 / 23.8, 4 x 14336 x 65536 107 / 89).
struct RingForm {
    int waves, depth;
    double fixed, line, rows_fullest, rows_all, product, sums_fullest, sums_all, weights, product_wave;
};
static const RingForm kRingInt4[] = {{8, 1, 2.4295, 0.2834, 0.7443e-3, 0.0503e-3, 3.2499e-5, 4.7473e-4, 1.6524e-4, 0.0258e-6, 0.0639e-5},
                                     {4, 1, 2.4459, 0.3433, 0.3771e-3, 0.1285e-3, 2.4934e-5, 3.0777e-4, 0.0010e-4, 0.0300e-6, 8.2138e-5}};
static const RingForm kRingMx[] = {{8, 2, 2.5729, 0.0215, 1.0573e-3, 0.0366e-3, 2.0803e-5, 2.1883e-4, 2.3732e-4, 0.0607e-6, 0.0128e-5},
                                   {4, 1, 2.8166, 0.1582, 0.5245e-3, 0.4159e-3, 0.2941e-5, 0.3131e-4, 0.0438e-4, 0.0330e-6, 13.6616e-5},
                                   {4, 2, 2.2628, 0.1485, 0.7724e-3, 0.0967e-3, 2.4500e-5, 4.8268e-4, 0.7322e-4, 0.0376e-6, 0.2875e-5}};

RingShape ring_shape(int64_t T, int m, int n, bool mx) {
    const RingForm* forms = mx ? kRingMx : kRingInt4;
    const int nforms = mx ? 3 : 2;
    const double cu = cu_count(), nl = n / 256, weights = 0.5 * m * (double)n;
    const int want_tokens = tuned(Knob::GEMM_TOKENS, 0), want_rows = tuned(Knob::GEMM_ROWS, 0);
    RingShape best{};
    double limit = 1e300;
    auto consider = [&](int tokens, int rows) {
        const int64_t groups = ((m + rows - 1) / rows) * ((T + tokens - 1) / tokens);
        const double all = groups / cu, fullest = std::ceil(all), sums = rows * (tokens < 32 ? 32 : tokens), lines = nl * (rows + tokens);
        for (int f = 0; f < nforms; ++f) {
            const RingForm& r = forms[f];
            if (T > 32 && rows == 16 && r.waves == 4 && all > 1 && !want_rows) continue;
            const double steps = std::ceil(nl / r.waves);
            const double us = r.fixed + r.line * steps + lines * (r.rows_fullest * fullest + r.rows_all * all) + r.weights * weights +
                              sums * (r.product * nl * all + r.product_wave * steps + r.sums_fullest * fullest + r.sums_all * all);
            if (us >= limit) continue;
            best = RingShape{tokens, rows, r.waves, !mx && T <= 32 && r.waves == 8 && steps >= 16 ? 2 : r.depth, us};
            limit = us;
        }
    };
    auto over_rows = [&](int tokens) {
        if (want_rows) return consider(tokens, want_rows);
        const int plain = T > 32 ? 0 : (m + 15) / 16 <= cu ? 16 : 32;
        if (plain) {
            consider(tokens, plain);
            limit *= 0.95;
        }
        for (int rows = 16; rows <= 64; rows += 16)
            if (rows != plain) consider(tokens, rows);
    };
    if (want_tokens) {
        over_rows(want_tokens);
    } else if (T <= 32) {
        over_rows(T <= 8 ? 8 : T <= 16 ? 16 : 32);
    } else {
        over_rows(64);      // first: of two shapes of the same cost the one with fewer token tiles
        over_rows(32);
    }
    best.waves = tuned(Knob::GEMM_WAVES, best.waves);
    best.depth = tuned(Knob::GEMM_DEPTH, best.depth);
    return best;
}

bool ring_launch(const RingShape& s, int64_t T, int m, int n, int slot, int loads, RingLaunch& r) {
    const int64_t groups = (m + s.rows - 1) / s.rows, tiles = (T + s.tokens - 1) / s.tokens;
    const int64_t grid = tiles == 1 ? groups : (groups * tiles + 7) / 8 * 8;   // whole rounds of the eight XCDs (see ring_tile)
    if (grid > 0x7fffffff || tiles > RingConfig::kMaxTokenTiles) return false;
    if (tiles > 1 && s.tokens < 32) return false;                         // the lanes past a smaller tile repeat its rows: only tokens past T are dropped
    int nwv = s.waves, depth = s.depth;
    if ((nwv != 4 && nwv != 8 && nwv != 16) || depth < 1 || depth > kRingMaxDepth) return false;
    if (nwv > ring_max_waves(s.tokens / 8, s.rows)) nwv = ring_max_waves(s.tokens / 8, s.rows);
    while (nwv > 4 && nwv * slot > kRingLdsMax) nwv >>= 1;
    const int steps = (n / 256 + nwv - 1) / nwv;                          // of the wave with the most lines
    if (depth > steps) depth = steps;
    while (depth > 1 && (nwv * depth * slot > kRingLdsMax || (depth - 1) * loads > 63)) --depth;
    r.grid = (unsigned)grid;
    // More than a workgroup per CU, a whole number of groups per XCD, and their weights fit in its L2 or are less than the tokens: the weights stay
    // there while the tokens pass.  us contiguous / channels first, tokens x channels x n, 4 waves: INT4 2048 x 1024 x 12288 (64 x 32) 52.8 / 35.2;
    // 256 x 5120 x 1792 (32 x 32) 8.6 / 7.4; MXFP4 241 x 4096 x 5120 (32 x 64) 12.2 / 10.9; 1300 forms of 900 such launches 0.975 on average.  Otherwise the
    // weights would come again for every token tile: 254 x 13824 x 11008 (32 x 64) 1.5 times as long.  Not groups of 16, of which INT4 takes 2 % longer.
    const bool channels_first = tiles > 1 && groups % 8 == 0 && s.rows > 16 && T / 2 <= m && ((int64_t)m * n <= 8LL * 2 * (4 << 20) || 8 * T > m) &&
                                groups * tiles > cu_count();
    r.cfg = RingConfig(depth, nwv, channels_first, (int)tiles);
    r.lds = nwv * depth * slot;                                           // the partial sums (128 bytes per channel and 32 tokens, per wave) reuse the rings
    return true;
}

template <int NTD, int ROWS>
static hipError_t skinny_launch_shape(const GemmDev& d, hipStream_t stream, const RingShape& s) {
    static OccCache oc;
    int unused = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_skinny_kernel<NTD, ROWS>), 64 * ring_max_waves(NTD, ROWS), kRingLdsMax, oc, unused);
    if (e != hipSuccess) return e;
    RingLaunch r;
    if (!ring_launch(s, d.T, d.m, d.n, (ROWS + 8 * NTD) * 128, ROWS / 8 + NTD, r)) return hipErrorInvalidValue;
    return launch((w4a4_skinny_kernel<NTD, ROWS>), dim3(r.grid), dim3(64 * r.cfg.waves()), r.lds, stream, d.wc, d.xc, d.ws, d.xs, d.out, d.n, d.m, (int)d.T, r.cfg, d.out_stride);
}
template <int NTD>
static hipError_t skinny_launch_tokens(const GemmDev& d, hipStream_t stream, const RingShape& s) {
    switch (s.rows) {
        case 16: return skinny_launch_shape<NTD, 16>(d, stream, s);
        case 32: return skinny_launch_shape<NTD, 32>(d, stream, s);
        case 48: return skinny_launch_shape<NTD, 48>(d, stream, s);
        case 64: return skinny_launch_shape<NTD, 64>(d, stream, s);
        default: return hipErrorInvalidValue;
    }
}
static hipError_t skinny_launch(const GemmDev& d, hipStream_t stream, const RingShape& s) {
    switch (s.tokens) {
        case 8: return skinny_launch_tokens<1>(d, stream, s);
        case 16: return skinny_launch_tokens<2>(d, stream, s);
        case 32: return skinny_launch_tokens<4>(d, stream, s);
        case 64: return skinny_launch_tokens<8>(d, stream, s);
        default: return hipErrorInvalidValue;
    }
}

// What is dirty in L2 when a kernel ends is written back before the next one starts, about 1.5 us for a whole tile per CU.  So rows of
// whole cache lines are written through, while the other tiles are still at work: us cached / through, INT4 2048 x 4096 x 4096 27.5 / 26.8,
// 777 x 5120 x 5120 24.0 / 22.8, 16384 x 8192 x 1024 115.3 / 110.6; MXFP4 2048 x 4096 x 11008 51.8 / 49.4, 1139 x 7296 x 4096 30.7 / 29.7,
// 2508 x 2944 x 4096 21.8 / 20.2; 46 such launches of 7 to 268 MB 0.976 on average, 0.976 also together with a kernel that reads the output.
// (Non-temporal stores save more, 0.94, but the reader pays it back: 0.99 together.)  The ends of other rows are merged in L2, written through
// they are writes of their own: 8192 x 8200 x 512 50 / 64, MXFP4 2580 x 10328 x 2048 37.5 / 39.3.
Out tiled_output(const void* out, int64_t out_stride) {
    const uintptr_t rows = reinterpret_cast<uintptr_t>(out) | (uintptr_t)(2 * out_stride);
    return rows & 3 ? Out::odd : rows & 127 ? Out::cached : Out::through;
}

template <class L, Out OUT>
static hipError_t tiled_launch_rows(const GemmDev& d, hipStream_t stream) {
    static OccCache cache;
    int occ = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(w4a4_tiled_kernel<L, OUT>), 64 * L::NW, L::LDS, cache, occ);
    if (e != hipSuccess) return e;
    // persistent: every XCD (eight of them) gets as many workgroups as it holds at once, or as it has tiles
    const int64_t tiles = ((d.T + L::TOK - 1) / L::TOK) * ((d.m + L::CH - 1) / L::CH);
    const int64_t per_xcd = (tiles + 7) / 8, resident = (int64_t)occ * cu_count() / 8;
    const unsigned grid = 8 * (unsigned)(per_xcd < resident ? per_xcd : resident);
    return launch(w4a4_tiled_kernel<L, OUT>, dim3(grid), dim3(64 * L::NW), L::LDS, stream, d);
}

template <class L>
static hipError_t tiled_launch(const GemmDev& d, hipStream_t stream) {
    switch (tiled_output(d.out, d.out_stride)) {
        case Out::odd: return tiled_launch_rows<L, Out::odd>(d, stream);
        case Out::through: return tiled_launch_rows<L, Out::through>(d, stream);
        default: return tiled_launch_rows<L, Out::cached>(d, stream);
    }
}

// Tile form (FLATQUANT_GEMM_WIDE forces one): int8 with 128 x 128 tiles, two workgroups per CU (0) or 160 x 128, one (4); FP6 with
// 256 x 128 tiles, K in two parts (1), or 256 x 256 (2).  A launch takes rounds of one tile per slot, and a round a fixed part
// and one per K iteration that grows with the share of the slots in use (the clock falls).  The constants are a fit to 110
// launches of 100 <= T <= 16384, 512 <= m <= 14336, 256 <= n <= 28672 (rms 5 - 6 %); what they choose is 0.2 % slower than the best
// form on average, 10 % at worst.  (Forms 0 / 1 / 2 / 4, us: 2048 x 4096 x 1024 11.4 / 14.3 / 16.3 / 15.5, 2048 x 4096 x 4096 28.4 / 26.7 /
// 36.2 / 38.5, 2048 x 4096 x 8192 52.7 / 43.7 / 62.2 / 68.8, 777 x 5120 x 5120 28.8 / 27.5 / 40.8 / 23.3, 768 x 5120 x 5120 20.6 / 27.6 / 41.7 /
// 24.1, 3000 x 4096 x 4096 40.9 / 44.8 / 37.0 / 54.8, 6000 x 4096 x 11008 203 / 159 / 170 / 233.)
static double w4a4_tiled_us(const GemmArgs& a, int& form) {
    const int64_t cu = cu_count();
    const double nk = a.n / 256;
    auto round_us = [&](int tok, int ch, int64_t slots, double& part) {   // full rounds; part: how full the last one is
        const int64_t tiles = ((a.T + tok - 1) / tok) * ((a.m + ch - 1) / ch);
        part = (double)(tiles % slots) / (double)slots;
        return (double)(tiles / slots);
    };
    double x;
    double us[5];
    us[0] = 3.5 + round_us(128, 128, 2 * cu, x) * (2.7 + 1.43 * nk);
    if (x > 0.5) us[0] += 2.7 + (0.84 + 0.59 * x) * nk;              // CUs with one and with two tiles
    else if (x > 0) us[0] += 0.5 + (0.63 + 0.28 * x) * nk;
    us[1] = 2.8 + round_us(256, 128, cu, x) * (5.9 + 1.08 * nk);
    if (x > 0) us[1] += 5.9 + (0.88 + 0.20 * x) * nk;
    us[2] = 0.8 + round_us(256, 256, cu, x) * (7.7 + 1.89 * nk);
    if (x > 0) us[2] += 7.7 + (1.57 + 0.32 * x) * nk;
    us[4] = 1.5 + round_us(160, 128, cu, x) * (3.3 + 1.0 * nk);
    if (x > 0) us[4] += 3.3 + (0.86 + 0.14 * x) * nk;
    int best = 0;
    for (int f : {1, 2, 4})
        if (us[f] < us[best]) best = f;
    form = best;
    return us[best];
}

hipError_t w4a4_launch(const GemmArgs& a, hipStream_t stream) {
    GemmDev d;
    d.xc = a.x_codes; d.xs = a.x_scales; d.wc = a.w_codes; d.ws = a.w_scales; d.out = a.out;
    d.T = a.T; d.out_stride = a.out_stride; d.m = a.m; d.n = a.n;
    // Decode and short prefill chunks: one pass over the weights per tile of up to 64 tokens, K split inside a workgroup (the ring
    // kernel), for as long as it is the cheaper one (FLATQUANT_GEMM_RING_MAX_T replaces the comparison by a token count).  Beyond one
    // 128 x 128 tile per CU it has to promise a quarter less: the tiled kernel's estimate holds there (3 % too low), the ring kernel's is 10 to 30 %
    // too low (tiled / ring, us: 2048 x 8200 x 11008 164 / 227, 384 x 11008 x 8192 39 / 49, 777 x 5120 x 28672 113 / 148; 192 x 8200 x 65536 232 / 125).
    const bool ring = tuned(Knob::GEMM_TILED, 0) == 0;
    if (ring && a.T <= 64) return skinny_launch(d, stream, ring_shape(a.T, a.m, a.n, false));
    int form = 0;
    const double tiled_us = w4a4_tiled_us(a, form);
    const int ring_max = tuned(Knob::GEMM_RING_MAX_T, -1);
    if (ring && a.T <= (ring_max >= 0 ? ring_max : 4096)) {
        const RingShape s = ring_shape(a.T, a.m, a.n, false);
        const bool tile_per_cu = ((a.T + 127) / 128) * ((a.m + 127) / 128) <= cu_count();
        if (ring_max >= 0 || s.us * (tile_per_cu ? 1.0 : 1.25) < tiled_us) return skinny_launch(d, stream, s);
    }
    const int asked = tuned(Knob::GEMM_WIDE, form);
    if (asked == 0 || asked == 1 || asked == 2 || asked == 4) form = asked;
    switch (form) {
        case 1: return tiled_launch<Tile<true, 4, 4, 2, 1, 2, 3, 1>>(d, stream);
        case 2: return tiled_launch<Tile<true, 4, 4, 2, 2, 1, 2, 1>>(d, stream);
        case 4: return tiled_launch<Tile<false, 5, 1, 1, 4, 1, 3, 1>>(d, stream);
        default: return tiled_launch<Tile<false, 2, 2, 2, 2, 1, 2, 2>>(d, stream);
    }
}

}  // namespace fq
