// Internal declarations shared by the translation units of libflatquant.
// Nothing here is part of the public ABI (see include/flatquant.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace fq {

constexpr int kTile = 32;          // MFMA tile edge (v_mfma_f32_32x32x16_f16)
constexpr int kMaxN1 = 128;        // up to 4 row tiles
constexpr int kMaxN2 = 256;        // up to 8 column slabs (one wavefront each)
constexpr int kLdsPad = 8;         // halves of padding per LDS row (keeps 16-byte reads off one bank group)

struct TqArgs {
    const _Float16* x;
    const _Float16* P1;
    const _Float16* P2;
    const float* clip;
    int clip_mode;
    int64_t T;
    int n1, n2;
    int64_t x_stride;
    uint8_t* out_codes;
    _Float16* out_scales;
    int mx_tiled = 0;
};

// Kernel-side argument block of the activation kernels.
struct TqDev {
    const _Float16* x;
    const _Float16* P1;
    const _Float16* P2;
    const float* clip;
    uint8_t* out_codes;
    _Float16* out_scales;
    int64_t x_stride;
    int64_t T;
    int n1, n2;
    int clip_mode;
    int vec8;       // rows can be moved in 16-byte chunks that never straddle a row of X~
    int out_vec16;  // code rows are whole 16-byte units at 16-byte aligned addresses
    int mx_tiled = 0;   // MXFP4 output only: exponents in the tile order the MXFP4 product reads (see flatquant.h)
    uint32_t n1_magic = 0;   // floor(2^32 / n1) + 1 (n1 >= 2): floor(f / n1) = umulhi(f, n1_magic) for f < 2^16
    uint32_t n2_magic = 0;   // the same for n2
};

// Specialised kernels for n2 a multiple of 32 and 16-byte aligned buffers (fq_tq_fast.hip).
bool tq_fast_applicable(const TqDev& d);
int64_t tq_fast_lds_bytes(int n1, int n2);
hipError_t tq_fast_launch(const TqDev& d, hipStream_t stream);
// One wavefront per token, rows through a wave-private LDS tile (fq_tq_wave.hip; n2 = 64, n1 = 32 or 64; INT4 or MXFP4).
bool tq_wave_applicable(const TqDev& d);
hipError_t tq_wave_launch(const TqDev& d, hipStream_t stream, int tpw, bool loop, bool mx);
// ... and its left-factor-only sibling for 128-wide rows (P2 == nullptr, n1 = 32 or 64; loop-free).
bool po_wave_applicable(const TqDev& d);
hipError_t po_wave_launch(const TqDev& d, hipStream_t stream);
// Row tiles of 16, one barrier per token (fq_tq_rows.hip): for the factors that rows_kernel_takes() names.
int64_t tq_rows_lds_bytes(int n1, int n2);
hipError_t tq_rows_launch(const TqDev& d, hipStream_t stream, bool mx);
// Grid of a persistent loop over the tokens with room for occ workgroups per CU: every workgroup gets the same number of tokens (+-1).
// Four row tiles with three or four slabs have room for two.  Both stage the factors, and a round of tokens takes the two 1.6 times as long as
// one alone (tq_any_kernel 1.35 times), so few tokens per CU, and numbers of them that leave the second workgroup a round short, are faster with one:
// r1 and r2 are the rounds with one and with two.  us with one / two: 128 x 128 9.8 / 10.8 (300 tokens), 13.2 / 15.4 (640), 18.3 / 19.0 (1024), 20.6 / 21.8
// (1100), 25.8 / 25.6 (1536), 33.0 / 31.9 (2048), 114 / 100 (8192); 113 x 96 10.5 / 11.0, 13.5 / 15.3, 16.7 / 16.3, 19.0 / 19.6, 21.4 (1300) / 20.0; MXFP4 128 x 96 12.8 / 14.4 (640),
// 16.2 / 15.5 (1024); tq_any_kernel 112 x 80 13.0 / 13.4 (300), 16.7 / 18.4 (768), 22.9 / 22.6 (1100).
inline unsigned token_loop_grid(int64_t T, int64_t cu, int occ, bool one) {
    if (one && occ == 2) occ = 1;
    const int64_t rounds = (T + cu * occ - 1) / (cu * occ);
    return (unsigned)((T + rounds - 1) / rounds);
}
inline bool slab_loop_alone(int64_t T, int64_t cu, int A, int B, bool full) {
    if (A != 4 || (B != 3 && B != 4)) return false;
    const int64_t r1 = (T + cu - 1) / cu, r2 = (r1 + 1) / 2;
    // (four slabs, two tokens for nearly every CU: as fast or slower alone, 128 x 128 at 512 tokens 11.0 / 11.9 on one machine and 15.8 / 13.1 on another)
    if (B == 4 && r1 == 2 && 4 * T > 7 * cu) return false;
    return 5 * r1 <= 8 * r2 + (full && B == 4 ? 4 : 2);
}
inline bool any_loop_alone(int64_t T, int64_t cu, int A, int B) {
    if (A != 4 || (B != 3 && B != 4)) return false;
    const int64_t r1 = (T + cu - 1) / cu, r2 = (r1 + 1) / 2;
    return 3 * r1 <= 4 * r2 + 2;
}
// Whether a left factor of n1 rows and a right factor of 32 B columns go to tq_rows_kernel rather than to tq_fast_kernel; both give the same
// bytes.  tq_fast_kernel / tq_rows_kernel in us, tokens in parentheses: row tiles that are not full gain most, by the 16 rows that are no longer
// padding and by the prologue: 48 x 64 4.2 / 3.3 (64), 44 / 29 (16384); 72 x 128 5.9 / 5.0, 135 / 111; 86 x 128 6.0 / 4.9, 142 / 136; 104 x 64 8.5 / 5.2,
// 127 / 89; 112 x 128 7.8 / 6.0, 122 / 99 (8192); 112 x 256 11.7 / 10.7, 490 / 425 (16384); MXFP4 112 x 224 13.5 / 8.6, 302 / 203 (8192).  Full ones gain by one
// barrier less per token and by tokens that arrive straight in LDS: 32 x 160 7.8 / 4.8 (512), 87 / 68 (16384); 64 x 96 5.5 / 4.5, 71 / 67; 64 x 128 4.2 / 4.0 (64),
// 14.6 / 13.2 (2048); 96 x 256 9.6 / 8.2 (64), 55 / 52 (2048); 128 x 224 10.3 / 9.2, 69 / 66, MXFP4 13.2 / 9.1, 87 / 64.
// Not taken: 32- and 64-wide rows of full tiles (wave-per-token kernel); five slabs of 49 .. 64 rows, which tq_fast_kernel has two workgroups
// per CU for (12.4 / 14.0 at 1024); eight slabs of 64 rows; 113 rows on with up to four slabs (128 x 128 113 / 124 at 8192) and with eight, whose two
// tiles LDS has no room for; MXFP4 at 32 rows with an even number of slabs (32 x 128 39 / 43 at 16384) and long launches of 49 .. 63 x 64 (56 x 64
// 8.4 / 7.4 at 2048, 37 / 38 at 16384); 64-wide rows of an odd P1, whose staging goes through registers, before the loop has made up for it (49 x 64
// 3.8 / 4.1 (1), 4.8 / 5.4 (300), 14.3 / 14.8 (4096), 25.1 / 22.8 (8192); 33 x 64 4.5 / 4.8 (300), 7.9 / 8.1 (2048), 9.7 / 8.5 (2500)).
constexpr bool rows_kernel_takes(int n1, int B, bool mx, int64_t T) {
    if (B < 2 || B > 8) return false;
    if (B == 2 && n1 % 2 == 1 && n1 > 32 && n1 < 64 && T <= (n1 < 48 ? 2048 : 5632)) return false;
    switch ((n1 + 15) / 16) {
        case 2: return n1 == 32 && B >= 3 && (!mx || B % 2 == 1);
        case 4: return n1 == 64 ? B >= 3 && B != 5 && B != 8 : B != 5 && !(B == 2 && mx && T > 8192);
        case 8: return B >= 5 && B <= 7;
        default: return n1 > 16;
    }
}
// whether any left factor of R row tiles of 16 goes to tq_rows_kernel, by few tokens or many
constexpr bool rows_kernel_reached(int R, int B, bool mx) {
    for (int n1 = 16 * R - 15; n1 <= 16 * R; ++n1)
        if (rows_kernel_takes(n1, B, mx, 1) || rows_kernel_takes(n1, B, mx, INT64_MAX)) return true;
    return false;
}
// whether any left factor of A row tiles of 32, full or not, is left to tq_fast_kernel, by few tokens or many
constexpr bool slab_kernel_reached(int A, int B, bool full, bool mx) {
    for (int n1 = full ? 32 * A : 32 * A - 31; n1 < 32 * A + full; ++n1)
        if (!rows_kernel_takes(n1, B, mx, 1) || !rows_kernel_takes(n1, B, mx, INT64_MAX)) return true;
    return false;
}
// MXFP4 output variant of the specialised kernels (d.out_scales points at the u8 [T, n/32] shared exponents).
bool tq_mx_applicable(const TqDev& d);
hipError_t tq_mx_launch(const TqDev& d, hipStream_t stream);
// ... and of the general kernel, for the shapes those do not take (fq_transform_quant.hip).
bool tq_mx_generic_applicable(const TqDev& d);
hipError_t tq_mx_generic_launch(const TqDev& d, hipStream_t stream);
// Fills the kernel-side block from the checked arguments (alignment facts included).
TqDev tq_dev_args(const TqArgs& a);

// LDS bytes of the fused activation kernel for (n1, n2); 0 if unsupported.
int64_t tq_lds_bytes(int n1, int n2);
bool tq_supported(int n1, int n2);
// Enqueue the fused kernel; returns hipSuccess or the launch error.
hipError_t tq_launch(const TqArgs& a, hipStream_t stream);

struct KvArgs {
    const _Float16* kv;
    const _Float16* P;
    int Hp;
    float clip;
    int64_t T;
    int H, D;
    uint8_t* out_codes;
    _Float16* out_scales;
    _Float16* out_zeros;
    bool fp16_out = false;   // transform only: out_codes points at an fp16 [T, H, D] tensor, no steps / zero points
    int bits = 4;            // code width of the quantizing mode: 2, 3 or 4
};
hipError_t kv_launch(const KvArgs& a, hipStream_t stream);

hipError_t dequant_mxfp4_launch(const uint8_t* codes, const uint8_t* exps, int64_t rows, int n, float* out, hipStream_t stream);
hipError_t dequant_bits_launch(const uint8_t* codes, const _Float16* scales, const _Float16* zeros,
                               int64_t rows, int n, int bits, float* out, hipStream_t stream);
hipError_t dequant_launch(const uint8_t* codes, const _Float16* scales, const _Float16* zeros,
                          int64_t rows, int n, float* out, hipStream_t stream);

struct GemmArgs {
    const uint8_t* x_codes;
    const _Float16* x_scales;
    const uint8_t* w_codes;
    const _Float16* w_scales;
    _Float16* out;
    int64_t T;
    int64_t out_stride;
    int m, n;
};
// W4A4 matrix product of the two quantized factors (fq_gemm.hip).
hipError_t w4a4_launch(const GemmArgs& a, hipStream_t stream);

struct MxGemmArgs {
    const uint8_t* x_codes;
    const uint8_t* x_exps;
    const uint8_t* w_codes;
    const uint8_t* w_exps;
    _Float16* out;
    int64_t T;
    int64_t out_stride;
    int m, n;
};
hipError_t mxfp4_gemm_launch(const MxGemmArgs& a, hipStream_t stream);

// How the tiled products' output leaves: in halves (rows that are not all dword-aligned), or in 16-byte pieces where it can, which
// stay in L2 or are written through it.
enum class Out { odd, cached, through };
Out tiled_output(const void* out, int64_t out_stride);
// Few-token products (fq_gemm.hip, fq_gemm_mx.hip): per wave a ring of LDS slots filled by global-to-LDS loads.
constexpr int kRingMaxDepth = 8;
constexpr int kRingLdsMax = 160 * 1024;
// waves that a workgroup of 8 ntd tokens and `rows` channels is compiled for: more than 32 of either need the registers of two waves per SIMD
constexpr int ring_max_waves(int ntd, int rows) { return ntd >= 8 || rows > 32 ? 8 : 16; }
// Tokens (8, 16, 32, 64) and output channels (16, 32, 48, 64) of a workgroup, its waves and line slots per wave, and what the launch is
// expected to take.
struct RingShape {
    int tokens, rows, waves, depth;
    double us;
};
RingShape ring_shape(int64_t T, int m, int n, bool mx);
// Ring depth, waves, order and number of the token tiles of a launch in one dword (the kernels' arguments arrive in registers, as many as there is room for).
struct RingConfig {
    static constexpr int kMaxTokenTiles = (1 << 24) - 1;
    uint32_t bits;
    RingConfig() = default;
    RingConfig(int depth, int waves, bool channels_first, int token_tiles)
        : bits((uint32_t)depth | (uint32_t)__builtin_ctz(waves) << 4 | (uint32_t)channels_first << 7 | (uint32_t)token_tiles << 8) {}
    __host__ __device__ int depth() const { return bits & 15; }
    __host__ __device__ int log2_waves() const { return bits >> 4 & 7; }
    __host__ __device__ int waves() const { return 1 << log2_waves(); }
    __host__ __device__ bool channels_first() const { return bits >> 7 & 1; }
    __host__ __device__ int token_tiles() const { return (int)(bits >> 8); }
};
struct RingLaunch {
    unsigned grid;
    RingConfig cfg;
    int lds;
};
// Waves, ring depth and grid for slots of `slot` bytes that `loads` instructions fill; false for overrides that no launch can honour.
bool ring_launch(const RingShape& s, int64_t T, int m, int n, int slot, int loads, RingLaunch& r);
#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)
// Channel group and token tile of a workgroup.  Workgroup b runs on XCD b % 8: an XCD takes a contiguous eighth of an order in which the
// tiles that share the larger operand follow each other, so that its rows come from memory once and are in that L2 for the others
// (1025 x 842 x 11008 20.8 -> 16.7 us; 4000 x 512 x 4096, with the smaller one, 16 -> 21).  channels < 0: nothing to do (the grid
// is a whole number of rounds of the XCDs).  RingConfig::channels_first (ring_launch says when): channel groups in their own order, one
// token tile after the other; every XCD has the same eighth of the groups in each.
struct RingTile {
    int channels, tokens;
};
__device__ __forceinline__ RingTile ring_tile(int b, int groups, RingConfig cfg, bool more_tokens) {
    const int token_tiles = cfg.token_tiles();
    if (__builtin_expect(token_tiles == 1, true)) return RingTile{b, 0};   // decode: the rest is out of its way
    const int all = groups * token_tiles, per_xcd = (all + 7) >> 3, q = cfg.channels_first() ? b : (b & 7) * per_xcd + (b >> 3);
    if (q >= all) return RingTile{-1, 0};
    more_tokens |= cfg.channels_first();
    const int inner = more_tokens ? groups : token_tiles, outer = q / inner, r = q - outer * inner;
    return more_tokens ? RingTile{r, outer} : RingTile{outer, r};
}
// Every kernel launch of the library goes through here.  The runtime keeps the last error of any earlier call on the
// thread (the caller's own, unrelated ones included) until somebody reads it: it is read and dropped first, so that
// what is returned belongs to this launch.
template <typename... KArgs, typename... Args>
inline hipError_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, int lds, hipStream_t stream, Args&&... args) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, static_cast<KArgs>(args)...);
    return hipGetLastError();
}
// until at most N of this wave's vector-memory loads are outstanding (they complete in order)
template <int N>
__device__ __forceinline__ void wait_vm_pending() {
    static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// until the ring step with `pend` later steps of NI load instructions each in flight has landed
template <int NI>
__device__ __forceinline__ void wait_ring_step(int pend) {
    switch (pend) {
        case 0: wait_vm_pending<0>(); break;
        case 1: if constexpr (NI <= 63) wait_vm_pending<NI>(); else wait_vm_pending<0>(); break;
        case 2: if constexpr (2 * NI <= 63) wait_vm_pending<2 * NI>(); else wait_vm_pending<0>(); break;
        case 3: if constexpr (3 * NI <= 63) wait_vm_pending<3 * NI>(); else wait_vm_pending<0>(); break;
        case 4: if constexpr (4 * NI <= 63) wait_vm_pending<4 * NI>(); else wait_vm_pending<0>(); break;
        case 5: if constexpr (5 * NI <= 63) wait_vm_pending<5 * NI>(); else wait_vm_pending<0>(); break;
        case 6: if constexpr (6 * NI <= 63) wait_vm_pending<6 * NI>(); else wait_vm_pending<0>(); break;
        case 7: if constexpr (7 * NI <= 63) wait_vm_pending<7 * NI>(); else wait_vm_pending<0>(); break;
        default: wait_vm_pending<0>(); break;
    }
}
#endif

// Copy-like probe with the activation kernel's traffic (fq_probe.hip).
hipError_t stream_probe_launch(const void* x, int64_t T, int n, int64_t x_stride, uint8_t* out, hipStream_t stream);

// Launch facts of one kernel, cached per device: the first call on a device raises the kernel's dynamic-LDS limit to
// `lds` bytes and asks the runtime how many workgroups of `threads` threads fit on a CU.  Concurrent first calls
// compute the same value; devices past the table are served without caching.
constexpr int kMaxDevices = 64;
struct OccCache {
    std::atomic<int> per_device[kMaxDevices];
};
hipError_t kernel_occupancy(const void* fn, int threads, int lds, OccCache& cache, int& wg_per_cu);

// Number of compute units of the current device (cached per device).
int cu_count();
// Tuning overrides (kernel flavour, workgroups per CU, ...), for measurements and for the tests that must reach every code
// path; kKnobNames (fq_api.hip) has their names in the same order.  Each starts from the environment variable of that name, read
// once per process, and can be changed with fq_set_tuning.
enum class Knob { MODE, WG_PER_CU, FORCE_GENERIC, KV_WG_PER_CU, GEMM_TILED, GEMM_WIDE, GEMM_DEPTH, GEMM_WAVES, GEMM_ROWS, GEMM_TOKENS, GEMM_RING_MAX_T, KV_FOLD_HEADS, KV_FEW, WAVE_TPW, PROBE_SHAPE, COUNT };
struct KnobState {
    std::atomic<int> state{0};   // 0: environment not read yet, 1: unset (callers use their default), 2: set
    std::atomic<int> value{0};
};
extern KnobState g_knobs[(int)Knob::COUNT];
int tuned_slow(Knob k, int dflt);
// The override's value, or `dflt`: on the launch path one load (by index: comparing names there took 0.3 us of a product's launch).
inline int tuned(Knob k, int dflt) { return g_knobs[(int)k].state.load(std::memory_order_acquire) == 1 ? dflt : tuned_slow(k, dflt); }

}  // namespace fq
