// Product of two MXFP4 factors on gfx950's scaled FP4 MFMA: out[t, o] = fp16( sum_k x^[t, k] w^[o, k] ), the low-bit
// matrix multiplication of Sec. 3.2 for the data type the paper's "Limitations" name next.  x^ and w^ are the
// de-quantized outputs of flatquant_transform_mxfp4_tiled (activations [T, n/2] codes + n/32 exponents per token in
// tile order, weights likewise): E2M1 elements times one power of two per block of 32 consecutive channels.
//
// v_mfma_scale_f32_32x32x64_f8f6f4 with both formats FP4 takes, per lane, 32 consecutive K elements (16 bytes of
// packed nibbles: lane (c, h) <-> row c, K half h) and one E8M0 exponent for exactly those 32 elements, so the stored
// layout is the operand layout: no unpacking, no widening, the block scales are applied inside the MFMA (measured on
// the device: the result equals the fp64 sum for random operands whose partial sums fit fp32).
//
// Tiled kernel (many tokens): every operand byte goes from global memory straight into LDS (global-to-LDS loads, unpadded
// 128-byte rows, 16-byte chunks swizzled), NST iterations of 256 codes deep, one barrier per iteration, persistent
// workgroups whose loads run on from one output tile into the next.  What bounds it, measured at 16384 x 8192 x 8192 (zero
// codes in brackets): MFMAs and barriers alone 381 us (269: the chip keeps 1.5 GHz under FP4 MFMAs on random operands,
// 22 ns per 32x32x64 instead of 13.5), with the output tiles 396 (289), with the operand reads from LDS 421 (306), with
// the loads 504 (408).  Beside the power limit it is the operand traffic, so the tile per wave is as large as the register
// file allows: 128 x 128 (4 waves, one per SIMD, 256 accumulators) moves half as many bytes per product term through LDS
// and L2 as the 64 x 64 wave tiles of 128 x 128 workgroups.  Against the two-stage kernel that was here (128 x 128, exponents
// one iteration ahead, MFMAs bunched behind the barrier; same box): 16384 x 8192 x 8192 678 -> 505 us, 2048 x 4096 x
// 11008 56.8 -> 49.6, 4096 x 4096 x 4096 45.9 -> 37.0, 777 x 5120 x 5120 25.4 -> 20.5.
#include "fq_internal.h"

namespace fq {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int XT = 128;               // tile edge, tokens and output channels
constexpr int XKB = 128;              // packed bytes of K per row and iteration (256 codes, 8 blocks)
struct MxGemmDev {
    const uint8_t* xc;
    const uint8_t* xe;
    const uint8_t* wc;
    const uint8_t* we;
    _Float16* out;
    int64_t T;
    int64_t out_stride;
    int m, n;
};

// TI x TJ: MFMA tiles per wave (tokens x channels), WM x WN: waves, NST: LDS stages, LA: K steps that an operand is read
// from LDS ahead of its MFMAs.  Off: offsets of a tile's rows from its first one.  32 bits hold 256 rows of n / 2 bytes up
// to n = 2^25 (kOff32MaxN); longer rows take 64.  OUT: how the output leaves (tiled_output); odd: its rows are not
// all dword-aligned and leave in halves, by a loop that only such launches carry (beside the other one it costs the aligned rows
// 1 - 2 %).  With the halves of 16-byte pieces stored one by one, eight rows to an instruction, 520 x 12609 x 2048 took 25.5 us, now 16.6; 1538 x 10027 x 4096 77.9,
// now 66.9; 1223 x 1819 x 2048 13.4, now 12.3 with two stages.
constexpr int kOff32MaxN = 1 << 25;
template <int TI, int TJ, int WM, int WN, int NST>
struct MxTile {
    static constexpr int NW = WM * WN;
    static constexpr int TOK = 32 * TI * WM, CH = 32 * TJ * WN, ROWS = TOK + CH;
    static constexpr int CODES = ROWS * XKB;                        // code tiles of one K iteration, then its exponents
    static constexpr int STAGE = CODES + 8 * ROWS;
    static constexpr int OPITCH = 64 * TJ + 16;                     // output staging: 32 tokens of a wave's channels
    static constexpr int LDS = NST * STAGE;
    static_assert(NW * 32 * OPITCH <= STAGE && LDS <= 160 * 1024 && NST >= 2, "LDS budget");
};

template <int TI, int TJ, int WM, int WN, int NST, int LA, typename Off, Out OUT>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(TI * TJ > 4 ? 1 : 2, TI * TJ > 4 ? 1 : 2))) void mxfp4_gemm_kernel(MxGemmDev p) {
    using L = MxTile<TI, TJ, WM, WN, NST>;
    constexpr bool ODD = OUT == Out::odd;
    constexpr int NW = L::NW, TOK = L::TOK, CH = L::CH, STAGE = L::STAGE, A_TILE = TOK * XKB, NOP = TI + TJ;
    constexpr int NLA = TOK / 8 / NW, NLB = CH / 8 / NW, NL = 1 + NLA + NLB;   // load instructions per wave and iteration
    constexpr int NPC = L::ROWS / 128;                              // 1 KB pieces of exponents per iteration
    constexpr int NKP = XKB / 32;                                   // K steps (64 codes) per iteration
    static_assert(NKP == 4 && (LA == 1 || LA == 2), "exponent bytes and the operand ring below");
    static_assert(TOK <= 256 && CH <= 256, "kOff32MaxN");
    constexpr int KB = NKP - LA;                                    // the steps before the iteration's barrier
    constexpr int RING = LA == 1 ? 2 : 4;
    constexpr int NQ = TI * TJ, RPS = NQ > 4 ? 2 : 1;               // MFMAs per step; LDS reads behind each of the first ones
    constexpr int LSTEPS = NST == 2 ? 2 : NKP;                      // steps over which an iteration's loads are spread
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int l = tid & 63, c = l & 31, h = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w % WM, wn = w / WM;
    const int64_t kbytes = p.n / 2;
    const int nk = p.n / (2 * XKB);
    const int64_t tile_e = (int64_t)nk * 1024;                      // bytes of exponents per tile of 128 rows
    const int ntx = (int)((p.T + TOK - 1) / TOK), nty = (p.m + CH - 1) / CH;
    const int64_t ntiles = (int64_t)ntx * nty;

    // Tiles of this workgroup.  Workgroup b runs on XCD b % 8: every XCD takes a contiguous eighth of a tile order that
    // goes through panels of PW token tiles, so that the tiles in flight on an XCD share rows of both operands in its L2
    // (32 workgroups that stream 256 + 256 rows each: 100 KB per us and CU arrive in LDS with 4 x 8 tiles per XCD, 55 with
    // a token tile per XCD and all the channels).
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
        const int pos = (int)(first + qq), panel = pos / (PW * nty), r = pos - panel * (PW * nty);
        const int width = ntx - panel * PW < PW ? ntx - panel * PW : PW;
        const int ty = r / width;
        return Pos{(int64_t)(panel * PW + r - ty * width) * TOK, ty * CH};
    };

    // ---- loads: one instruction fills 8 rows of 128 bytes of codes; LDS slot j of row r holds the row's chunk
    // j ^ ((r >> 1) & 7).  Rows past the end re-read the last row.  The exponents (8 bytes per row and iteration, in tile
    // order: per 128-row tile and iteration 1 KB in one piece) take one instruction per 128 rows; wave w brings piece w,
    // waves past the last piece repeat it, so that every wave counts the same number of loads.
    const unsigned char *abase, *bbase, *ebase;
    Off aoff[NLA], boff[NLB];
    const int pc = w < NPC ? w : NPC - 1;
    auto set_source = [&](const Pos& t) {
        abase = p.xc + t.t0 * kbytes;
        bbase = p.wc + (int64_t)t.o0 * kbytes;
        const int arows = (int)(p.T - t.t0 < TOK ? p.T - t.t0 : TOK), brows = p.m - t.o0 < CH ? p.m - t.o0 : CH;
#pragma unroll
        for (int k = 0; k < NLA; ++k) {
            const int row = 8 * (NLA * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
            aoff[k] = (Off)(row < arows ? row : arows - 1) * (Off)kbytes + 16 * ch;
        }
#pragma unroll
        for (int k = 0; k < NLB; ++k) {
            const int row = 8 * (NLB * w + k) + (l >> 3), ch = (l & 7) ^ ((row >> 1) & 7);
            boff[k] = (Off)(row < brows ? row : brows - 1) * (Off)kbytes + 16 * ch;
        }
        const bool tok = pc < TOK / 128;
        const int64_t tile = tok ? (t.t0 >> 7) + pc : (int64_t)(t.o0 >> 7) + pc - TOK / 128;
        const int64_t last = tok ? (p.T - 1) >> 7 : (int64_t)(p.m - 1) >> 7;   // tiles past the end do not exist
        ebase = (tok ? p.xe : p.we) + (tile < last ? tile : last) * tile_e + 16 * l;
    };
    typedef const __attribute__((address_space(1))) void* gptr;
    typedef __attribute__((address_space(3))) void* lptr;
    // loads k0 .. k1 - 1 of the NL that bring iteration `it` (past the last one it is re-read; nobody uses it)
    auto issue = [&](int it, int stage, int k0, int k1) {
        const int itc = it < nk ? it : nk - 1;
#pragma unroll
        for (int k = k0; k < k1; ++k) {
            if (k == 0) __builtin_amdgcn_global_load_lds((gptr)(ebase + (int64_t)itc * 1024), (lptr)(smem + stage + L::CODES + pc * 1024), 16, 0, 0);
            else if (k <= NLA) __builtin_amdgcn_global_load_lds((gptr)(abase + (int64_t)itc * XKB + aoff[k - 1]), (lptr)(smem + stage + (NLA * w + k - 1) * 8 * XKB), 16, 0, 0);
            else __builtin_amdgcn_global_load_lds((gptr)(bbase + (int64_t)itc * XKB + boff[k - 1 - NLA]), (lptr)(smem + stage + A_TILE + (NLB * w + k - 1 - NLA) * 8 * XKB), 16, 0, 0);
        }
    };

    // ---- operands.  x < TI: tokens 32 (TI wm + x) + c; else channels 32 (TJ wn + x - TI) + c
    const int hs = h ^ ((c >> 1) & 7);   // chunk 2 kp + h of row 32 x + c sits in slot (2 kp) ^ hs
    const int abyte = (32 * TI * wm + c) * XKB, bbyte = A_TILE + (32 * TJ * wn + c) * XKB;
    auto lds_chunk = [&](int stage, int kp, int x) -> u32x4 {
        const int a = stage + (x < TI ? abyte + 32 * x * XKB : bbyte + 32 * (x - TI) * XKB) + 16 * ((2 * kp) ^ hs);
        return *reinterpret_cast<const u32x4*>(smem + a);
    };
    // K step kp (64 codes) uses block 2 kp + h; the MFMA picks a byte of a register by an immediate, the same for every
    // lane, so the half-wave h = 1 shifts its bytes down by one: byte 2 (kp & 1) of dword kp / 2 then is the block of
    // this lane.
    auto lds_exps = [&](int stage, int x) -> u32x2 {
        const int row = (x < TI ? 32 * (TI * wm + x) : TOK + 32 * (TJ * wn + x - TI)) + c;
        return *reinterpret_cast<const u32x2*>(smem + stage + L::CODES + 8 * row);
    };
    f32x16 acc[TI][TJ];
    u32x4 P[RING][NOP];
    u32x2 ec[NOP], en[NOP];              // exponents of the current iteration, and of the next one as they are stored
    auto mfma = [&](int i, int j, int kp) {
        const u32x4 &wv = P[kp % RING][TI + j], &xv = P[kp % RING][i];
        const i32x8 a = {(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3], 0, 0, 0, 0};
        const i32x8 b = {(int)xv[0], (int)xv[1], (int)xv[2], (int)xv[3], 0, 0, 0, 0};
        // formats: 4 = FP4 (E2M1) for both operands; byte 2 (kp & 1) of the exponent registers
        if (kp & 1) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 4, 4, 2, (int)ec[TI + j][kp >> 1], 2, (int)ec[i][kp >> 1]);
        else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 4, 4, 0, (int)ec[TI + j][kp >> 1], 0, (int)ec[i][kp >> 1]);
    };
    // K step kp: its MFMAs, between them the operands of the step LA further on (of `stage_ahead`) and a share of the
    // loads of iteration `lit` into `stage_load`.  Steps KB .. NKP - 1 of an iteration, then 0 .. KB - 1 of the next one, lie
    // between two barriers: s is the step's place in that sequence, which the loads are spread over.
    auto step = [&](int kp, int stage_ahead, int lit, int stage_load, int s, int s0, int nsteps) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
            mfma(m / TJ, m % TJ, kp);
#pragma unroll
            for (int x = m * RPS; x < (m + 1) * RPS && x < NOP; ++x) P[(kp + LA) % RING][x] = lds_chunk(stage_ahead, (kp + LA) % NKP, x);
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
    auto read_exps = [&](int stage) {
#pragma unroll
        for (int x = 0; x < NOP; ++x) en[x] = lds_exps(stage, x);
    };
    auto next_exps = [&]() {
#pragma unroll
        for (int x = 0; x < NOP; ++x) ec[x] = u32x2{en[x][0] >> (8 * h), en[x][1] >> (8 * h)};
    };

    Pos cur = tile_pos(q);
    set_source(cur);
#pragma unroll
    for (int s = 0; s + 1 < NST; ++s) issue(s, s * STAGE, 0, NL);
    arrive();
    int st = 0, stl = (NST - 1) * STAGE;     // stage of the current iteration, and the one to be loaded next
    auto advance = [&](int stage) { return stage + STAGE == NST * STAGE ? 0 : stage + STAGE; };
    read_exps(0);
#pragma unroll
    for (int d = 0; d < LA; ++d)
#pragma unroll
        for (int x = 0; x < NOP; ++x) P[d][x] = lds_chunk(0, d, x);

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
        next_exps();
        // steps 0 .. KB - 1 of iteration 0; loads of iteration NST - 1
#pragma unroll
        for (int kp = 0; kp < KB; ++kp) step(kp, st, NST - 1, stl, kp, 0, LSTEPS < KB ? LSTEPS : KB);
        arrive();
        int lit = NST;                       // iteration to be loaded next
        auto body = [&]() {
            const int stn = advance(st);
            read_exps(stn);
            stl = advance(stl);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, lit, stl, kp - KB, 0, LSTEPS);
            next_exps();
#pragma unroll
            for (int kp = 0; kp < KB; ++kp) step(kp, stn, lit, stl, kp + LA, 0, LSTEPS);
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
        // the last steps of the tile: nothing is loaded, the current stage takes the output tile
        {
            const int stn = advance(st);
            read_exps(stn);
#pragma unroll
            for (int kp = KB; kp < NKP; ++kp) step(kp, stn, 0, 0, 0, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);

        // epilogue: in acc[i][j] a lane holds, for token 32 (TI wm + i) + c, the output channels 32 (TJ wn + j) + 8 (r / 4) +
        // 4 h + r % 4.  Rounded to fp16 and turned, 32 tokens at a time, through a part of LDS that belongs to the wave
        // alone (no barrier), from where they leave in 16-byte pieces of whole rows.
        typedef _Float16 half4 __attribute__((ext_vector_type(4)));
        constexpr int OPITCH = L::OPITCH, CPR = 4 * TJ;              // 16-byte pieces per token
        unsigned char* ot = smem + st + w * (32 * OPITCH);
        const uintptr_t pitch_bits = reinterpret_cast<uintptr_t>(p.out) | (uintptr_t)(2 * p.out_stride);
        const bool wide = (pitch_bits & 15) == 0, pairs = (pitch_bits & 3) == 0;   // whole pieces, dwords, or halves
#pragma unroll
        for (int i = 0; i < TI; ++i) {
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const half4 v = {(_Float16)acc[i][j][4 * g], (_Float16)acc[i][j][4 * g + 1], (_Float16)acc[i][j][4 * g + 2], (_Float16)acc[i][j][4 * g + 3]};
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
                            // (in asm: there is no builtin for it with a 64-bit address.  The s_nop is what a store of more than 8 bytes needs before its
                            // data registers are written again)
                            if constexpr (OUT == Out::through) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
                            else *reinterpret_cast<u32x4*>(dst) = v;
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
            read_exps(0);
#pragma unroll
            for (int d = 0; d < LA; ++d)
#pragma unroll
                for (int x = 0; x < NOP; ++x) P[d][x] = lds_chunk(0, d, x);
        }
    }
    wait_vm_pending<0>();                    // nothing may still be on its way into LDS when the workgroup ends
}

// ---- few tokens (decode, short prefill chunks; tiles of up to 64 tokens): the weights are read once per tile and the kernel is bound by how fast a CU takes them in.  A
// workgroup owns 16 to 64 output channels for 8 to 64 tokens (ring_shape); its waves split K by 128-byte lines (256 codes: wave w takes
// lines w, w + waves, ...) and each keeps a ring of line slots of its own in LDS: four global-to-LDS instructions
// bring 32 weight rows of a line (8 whole rows each), one per 8 token rows the tokens, one the 256 bytes of weight
// exponents of 32 channels (the tile order keeps them contiguous) and one per 32 tokens theirs.  A wave waits only for its own
// oldest slot (no barrier in the loop).  The partial sums of the waves are added in fp32 through LDS at the end.
// NTD and ROWS as for the INT4 product.
template <int NTD, int ROWS>
__global__ __launch_bounds__(ring_max_waves(NTD, ROWS) * 64) void mxfp4_skinny_kernel(const uint8_t* wc, const uint8_t* xc, const uint8_t* we, const uint8_t* xe, _Float16* out,
                                                                              int n, int m, int T, RingConfig cfg, int64_t out_stride) {
    static_assert(ROWS == 16 || ROWS == 32 || ROWS == 48 || ROWS == 64, "weight rows per workgroup");
    constexpr int NWI = ROWS / 8;                        // load instructions per line of the weight rows
    constexpr int NG = ROWS / 8;                         // groups of 8 output channels
    constexpr int NCT = (ROWS + 31) / 32;                // MFMA channel tiles of 32, and 256-byte pieces of their exponents
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int NTT = NTD > 4 ? NTD / 4 : 1;           // MFMA token tiles of 32
    constexpr int XROWS = 8 * NTD;
    constexpr int XOFF = ROWS * 128, WEOFF = XOFF + 1024 * NTD, XEOFF = WEOFF + 256 * NCT;
    constexpr int SLOT = XEOFF + 256 * NTT;
    constexpr int NI = NWI + NTD + NCT + NTT;            // load instructions per step
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
    const int ns = (nl - w + nwv - 1) >> cfg.log2_waves();   // this wave's steps
    unsigned char* ring = smem + w * depth * SLOT;

    // Row 8 k + l / 8, the chunk that belongs into slot l % 8 of it: one offset per k for both operands, from a scalar base each.
    // Rows past the end are out of the buffers' range and read as zeros.
    const int mrows = m - o0 < ROWS ? m - o0 : ROWS, trows = T - t0 < XROWS ? T - t0 : XROWS;
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wc) + (int64_t)o0 * kbytes, 0, mrows * (int)kbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(xc) + (int64_t)t0 * kbytes, 0, trows * (int)kbytes, 0x00020000);
    // exponents of line j: 1 KB per tile of 128 rows, 8 bytes per row.  The workgroup's channels are 256 bytes of a tile for every 32
    // of them (48 channels may begin in one tile and end in the next); the tokens are 32 or 64 consecutive rows of one tile
    // (the tensor is padded to whole tiles, so rows past T exist).  Rows past the last tile are out of the buffer's range.
    const int wt = o0 >> 7, wtiles = ((m + 127) >> 7) - wt;
    const __amdgpu_buffer_rsrc_t webuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(we) + (int64_t)wt * nl * 1024, 0, __builtin_amdgcn_readfirstlane(nl * 1024 * (wtiles < 2 ? 1 : 2)), 0x00020000);
    const __amdgpu_buffer_rsrc_t xebuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(xe) + (int64_t)(t0 >> 7) * nl * 1024 + 8 * (t0 & 127), 0, nl * 1024 - 8 * (t0 & 127), 0x00020000);
    constexpr int NV = NWI > NTD ? NWI : NTD;
    uint32_t voff[NV];
    {
        const uint32_t r = l >> 3, first = r * kbytes + 128 * w, ch = (l & 7) ^ (r >> 1);
#pragma unroll
        for (int k = 0; k < NV; ++k) voff[k] = first + 16 * (k & 1 ? ch ^ 4 : ch) + 8 * k * kbytes;
    }
    int wev[NCT];                                        // lanes 2 r, 2 r + 1: the 8 bytes of channel r of a piece
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
        const int row = (o0 & 127) + 32 * j + ((l >> 1) & (ROWS - 32 * j >= 32 ? 31 : 15));
        wev[j] = 1024 * w + (row >> 7) * nl * 1024 + 8 * (row & 127) + 4 * (l & 1);
    }
    const int xev = 1024 * w + 4 * l;
    typedef __attribute__((address_space(3))) void* lptr;
    auto issue = [&](int s, int slot) {
        unsigned char* base = ring + slot * SLOT;
        const int off = s * (128 * nwv), eoff = 8 * off;
#pragma unroll
        for (int k = 0; k < NWI; ++k) __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (lptr)(base + k * 1024), 16, (int)voff[k], off, 0, 0);
#pragma unroll
        for (int k = 0; k < NTD; ++k) __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (lptr)(base + XOFF + k * 1024), 16, (int)voff[k], off, 0, 0);
#pragma unroll
        for (int j = 0; j < NCT; ++j) __builtin_amdgcn_raw_ptr_buffer_load_lds(webuf, (lptr)(base + WEOFF + 256 * j), 4, wev[j], eoff, 0, 0);
#pragma unroll
        for (int i = 0; i < NTT; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(xebuf, (lptr)(base + XEOFF + 256 * i), 4, xev + 256 * i, eoff, 0, 0);
    };
    const int npre = ns < depth ? ns : depth;
#pragma unroll 1
    for (int s = 0; s < npre; ++s) issue(s, s);

    f32x16 acc[NTT][NCT];
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int j = 0; j < NCT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    int woff[NCT], whs[NCT], wexp[NCT];
#pragma unroll
    for (int j = 0; j < NCT; ++j) {
        const int row = 32 * j + (c & (ROWS - 32 * j >= 32 ? 31 : 15));
        woff[j] = row * 128;
        whs[j] = h ^ ((row >> 1) & 7);
        wexp[j] = WEOFF + 8 * row;
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
        wait_ring_step<NI>(left < depth - 1 ? left : depth - 1);
        const unsigned char* base = ring + slot * SLOT;
        // block 2 kp + h of this lane's row: after the shift by 8 h, byte 2 (kp & 1) of dword kp / 2
        u32x2 ew[NCT];
#pragma unroll
        for (int j = 0; j < NCT; ++j) {
            const u32x2 v = *reinterpret_cast<const u32x2*>(base + wexp[j]);
            ew[j] = u32x2{v[0] >> (8 * h), v[1] >> (8 * h)};
        }
        u32x2 ex[NTT];
#pragma unroll
        for (int i = 0; i < NTT; ++i) {
            const u32x2 v = *reinterpret_cast<const u32x2*>(base + XEOFF + 256 * i + 8 * c);
            ex[i] = u32x2{v[0] >> (8 * h), v[1] >> (8 * h)};
        }
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
#pragma unroll
            for (int i = 0; i < NTT; ++i) {
                const i32x8 b = {(int)xv[kp][i][0], (int)xv[kp][i][1], (int)xv[kp][i][2], (int)xv[kp][i][3], 0, 0, 0, 0};
#pragma unroll
                for (int j = 0; j < NCT; ++j) {
                    const i32x8 a = {(int)wv[kp][j][0], (int)wv[kp][j][1], (int)wv[kp][j][2], (int)wv[kp][j][3], 0, 0, 0, 0};
                    if (kp & 1) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 4, 4, 2, (int)ew[j][kp >> 1], 2, (int)ex[i][kp >> 1]);
                    else acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 4, 4, 0, (int)ew[j][kp >> 1], 0, (int)ex[i][kp >> 1]);
                }
            }
        }
        slot = (slot + 1 == depth) ? 0 : slot + 1;
    }
    wait_vm_pending<0>();
    __syncthreads();                                     // every wave is done with its ring: the partial sums go there
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    f32x4* part = reinterpret_cast<f32x4*>(smem);        // [wave][tile][quad g][lane] x 4 floats
#pragma unroll
    for (int i = 0; i < NTT; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g)
            part[((w * NTT + i) * NG + g) * 64 + l] = f32x4{acc[i][g / 4][4 * (g % 4)], acc[i][g / 4][4 * (g % 4) + 1], acc[i][g / 4][4 * (g % 4) + 2], acc[i][g / 4][4 * (g % 4) + 3]};
    __syncthreads();
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    const bool wide = ((reinterpret_cast<uintptr_t>(out) & 7) == 0) && (out_stride % 4 == 0);
    for (int e = tid; e < NTT * NG * 64; e += 64 * nwv) {
        const int el = e & 63, g = (e >> 6) % NG, i = (e >> 6) / NG;
        f32x4 sum = part[e];
        for (int ww = 1; ww < nwv; ++ww) sum += part[ww * NTT * NG * 64 + e];
        const int t = t0 + 32 * i + (el & 31);
        const int o = o0 + 8 * g + 4 * (el >> 5);
        if (t < T && o < m) {
            const _Float16 v[4] = {(_Float16)sum[0], (_Float16)sum[1], (_Float16)sum[2], (_Float16)sum[3]};
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

template <int NTD, int ROWS>
static hipError_t mx_skinny_launch_shape(const MxGemmDev& d, hipStream_t stream, const RingShape& s) {
    static OccCache oc;
    int unused = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(mxfp4_skinny_kernel<NTD, ROWS>), 64 * ring_max_waves(NTD, ROWS), kRingLdsMax, oc, unused);
    if (e != hipSuccess) return e;
    constexpr int NTT = NTD > 4 ? NTD / 4 : 1, NCT = (ROWS + 31) / 32;
    RingLaunch r;
    if (!ring_launch(s, d.T, d.m, d.n, ROWS * 128 + 1024 * NTD + 256 * (NCT + NTT), ROWS / 8 + NTD + NCT + NTT, r)) return hipErrorInvalidValue;
    return launch((mxfp4_skinny_kernel<NTD, ROWS>), dim3(r.grid), dim3(64 * r.cfg.waves()), r.lds, stream, d.wc, d.xc, d.we, d.xe, d.out, d.n, d.m, (int)d.T, r.cfg, d.out_stride);
}
template <int NTD>
static hipError_t mx_skinny_launch_tokens(const MxGemmDev& d, hipStream_t stream, const RingShape& s) {
    switch (s.rows) {
        case 16: return mx_skinny_launch_shape<NTD, 16>(d, stream, s);
        case 32: return mx_skinny_launch_shape<NTD, 32>(d, stream, s);
        case 48: return mx_skinny_launch_shape<NTD, 48>(d, stream, s);
        case 64: return mx_skinny_launch_shape<NTD, 64>(d, stream, s);
        default: return hipErrorInvalidValue;
    }
}
static hipError_t mx_skinny_launch(const MxGemmDev& d, hipStream_t stream) {
    const RingShape s = ring_shape(d.T, d.m, d.n, true);
    switch (s.tokens) {
        case 8: return mx_skinny_launch_tokens<1>(d, stream, s);
        case 16: return mx_skinny_launch_tokens<2>(d, stream, s);
        case 32: return mx_skinny_launch_tokens<4>(d, stream, s);
        case 64: return mx_skinny_launch_tokens<8>(d, stream, s);
        default: return hipErrorInvalidValue;
    }
}

template <int TI, int TJ, int WM, int WN, int NST, int LA, typename Off, Out OUT>
static hipError_t mx_tile_launch_rows(const MxGemmDev& d, hipStream_t stream) {
    using L = MxTile<TI, TJ, WM, WN, NST>;
    static OccCache cache;
    int occ = 0;
    hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(mxfp4_gemm_kernel<TI, TJ, WM, WN, NST, LA, Off, OUT>), 64 * L::NW, L::LDS, cache, occ);
    if (e != hipSuccess) return e;
    // persistent: every XCD (eight of them) gets as many workgroups as it holds at once, or as it has tiles
    const int64_t tiles = ((d.T + L::TOK - 1) / L::TOK) * ((d.m + L::CH - 1) / L::CH);
    const int64_t per_xcd = (tiles + 7) / 8, resident = (int64_t)occ * cu_count() / 8;
    const unsigned grid = 8 * (unsigned)(per_xcd < resident ? per_xcd : resident);
    return launch((mxfp4_gemm_kernel<TI, TJ, WM, WN, NST, LA, Off, OUT>), dim3(grid), dim3(64 * L::NW), L::LDS, stream, d);
}

template <int TI, int TJ, int WM, int WN, int NST, int LA, typename Off = uint32_t>
static hipError_t mx_tile_launch(const MxGemmDev& d, hipStream_t stream) {
    switch (tiled_output(d.out, d.out_stride)) {
        case Out::odd: return mx_tile_launch_rows<TI, TJ, WM, WN, NST, LA, Off, Out::odd>(d, stream);
        case Out::through: return mx_tile_launch_rows<TI, TJ, WM, WN, NST, LA, Off, Out::through>(d, stream);
        default: return mx_tile_launch_rows<TI, TJ, WM, WN, NST, LA, Off, Out::cached>(d, stream);
    }
}

// Tile form: 0 = 128 x 128 (two workgroups per CU, or one with three stages), 1 = 256 x 128, 2 = 256 x 256 (one per CU).  The
// time of a launch goes in rounds of what is resident at once; the cost of a round, full / at most half full, is what 8192
// channels take in us: 39 / 23, 35 / 26 and 64 / 45.  (Measured, us for forms 0 / 1 / 2: 1024 x 4096 x 4096 13.9 / 17.0 / 26.5,
// 2048 x 4096 x 4096 23.5 / 22.7 / 29.9, 3000 x 4096 x 4096 35.2 / 35.6 / 32.4, 4096 x 4096 x 4096 43.3 / 40.8 / 37.1, 2048 x
// 4096 x 11008 53.2 / 49.6 / 60.3, 1024 x 11008 x 4096 34.4 / 35.2 / 31.3, 16384 x 8192 x 8192 635 / 567 / 510.)
// Form 1 has three LDS stages: with fewer iterations than that (n < 768) its loads cannot run on into the next tile and it
// is behind form 0 at every size (forms 0 / 1: 777 x 5120 x 256 5.6 / 6.4, 2048 x 4096 x 512 8.1 / 8.5, 4096 x 14336 x 512
// 31.2 / 39.2, 15069 x 2510 x 256 22.3 / 27.0; at n = 768 2048 x 4096 12.1 / 10.0).
static int mx_tile_form(const MxGemmDev& d) {
    const int64_t cu = cu_count();
    auto cost = [&](int64_t tok, int64_t ch, int64_t slots, int64_t full, int64_t half) {
        const int64_t tiles = ((d.T + tok - 1) / tok) * ((d.m + ch - 1) / ch);
        return 2 * tiles <= slots ? half : (tiles + slots - 1) / slots * full;
    };
    const int64_t c0 = cost(128, 128, 2 * cu, 39, 23), c1 = cost(256, 128, cu, 35, 26), c2 = cost(256, 256, cu, 64, 45);
    return c2 <= c0 && c2 <= c1 ? 2 : c1 <= c0 && d.n >= 3 * 2 * XKB ? 1 : 0;
}

hipError_t mxfp4_gemm_launch(const MxGemmArgs& a, hipStream_t stream) {
    MxGemmDev d;
    d.xc = a.x_codes; d.xe = a.x_exps; d.wc = a.w_codes; d.we = a.w_exps; d.out = a.out;
    d.T = a.T; d.out_stride = a.out_stride; d.m = a.m; d.n = a.n;
    if (tuned(Knob::GEMM_TILED, 0) == 0 && d.n <= kOff32MaxN) {
        // decode and short prefill chunks: one pass over the weights, K split inside a workgroup (the ring kernel)
        if (a.T <= 64) return mx_skinny_launch(d, stream);
        // More tokens: the ring kernel on tiles of 32 or 64 tokens, as long as the 128 x 128 tiles of the kernel below would
        // reach at most half of the CUs (FLATQUANT_GEMM_RING_MAX_T replaces the rule by a token count).  Tiled / ring, us, weights from
        // memory, the number of those tiles in front: 32 128 x 4096 x 4096 13.5 / 6.8, 32 512 x 1024 x 4096 10.8 / 5.9, 64 256 x 4096 x 11008
        // 29.9 / 16.5, 64 1024 x 1024 x 4096 10.9 / 8.0, 80 640 x 2048 x 8192 21.1 / 17.7, 112 128 x 14336 x 4096 14.5 / 15.1, 128 512 x 4096 x 4096 13.1 / 12.6,
        // 128 256 x 8192 x 8192 23.3 / 23.0, 128 2048 x 1024 x 4096 11.3 / 12.9, 172 256 x 11008 x 4096 13.8 / 19.2, 192 768 x 4096 x 4096 13.1 / 17.9.
        const int64_t tiled_wgs = ((a.T + XT - 1) / XT) * ((a.m + XT - 1) / XT);
        const int ring_max = tuned(Knob::GEMM_RING_MAX_T, -1);
        if (ring_max >= 0 ? a.T <= ring_max : (2 * tiled_wgs <= cu_count() && a.T <= 4096))
            return mx_skinny_launch(d, stream);
    }
    // Rows whose offsets inside a tile need 64 bits: the smallest tile, whatever the form asked for.  They are far beyond
    // what the transform produces (n <= 32768), so there is one instance for them (1024 x 2304 x 33686272: 142.8 ms; 143.8
    // with the two-stage kernel mentioned at the top, all 64-bit addresses).
    if (d.n > kOff32MaxN) return mx_tile_launch<2, 2, 2, 2, 2, 1, uint64_t>(d, stream);
    const int rule = mx_tile_form(d), asked = tuned(Knob::GEMM_WIDE, rule);
    switch (asked >= 0 && asked <= 2 ? asked : rule) {
        case 1: return mx_tile_launch<4, 2, 2, 2, 3, 2>(d, stream);
        case 2: return mx_tile_launch<4, 4, 2, 2, 2, 1>(d, stream);
        default:
            // At most one 128 x 128 tile per CU: nobody else covers a workgroup's wait for its tiles, so a third stage takes the
            // place of the second workgroup (us with two / three stages: 160 x 8896 x 2048 9.1 / 7.5, 4060 x 632 x 7168 22.7 /
            // 16.3, 1024 x 4096 x 4096 15.6 / 12.7, 1024 x 4096 x 28672 85.6 / 63.9; a fourth one gains nothing: 7.7, 16.6,
            // 12.9, 63.8).
            if (((d.T + XT - 1) / XT) * ((d.m + XT - 1) / XT) <= cu_count()) return mx_tile_launch<2, 2, 2, 2, 3, 2>(d, stream);
            return mx_tile_launch<2, 2, 2, 2, 2, 1>(d, stream);
    }
}

}  // namespace fq
