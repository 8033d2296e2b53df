// Internal declarations shared by the host API and the gfx950 kernels of libdeepgemm_hip.
// Nothing here is part of the public ABI (that is include/deepgemm_hip.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "deepgemm_hip.h"

// A 3- or 4-bit table as the sum of two 2-bit lookups of the activation code, if it is one whose parts fit int8
// (dg_onehot_kernel.hip): T[w][4 i + j] = low[w][j] + high[w][i], a row of four entries to a word.
struct DgTwoLookups {
    bool splits;
    uint32_t low[16], high[16];
    int32_t lo, hi;              // range of all their entries
};

// A table whose entries are sums of what the activation code's bits add, as dg_planes_kernel.hip takes it.
struct DgBitSums {
    bool sums;
    uint32_t bytes;              // 2-bit codes: byte w, u[w]
    int32_t low, high, both;     // 2-bit codes: what the sums of its three planes count for; others: T[w][1] = low w + high
    int32_t most;                // the largest number on the weights' side times the largest on the other
};

// A 2-bit table that is a product of levels which dg_twopower_kernel.hip takes.
struct DgTwoPowers {
    bool levels;
    uint32_t bytes[6];           // of four FP6 numbers' three bytes: code w's share in byte w
    uint32_t powers;             // byte a: the two signed powers of activation code a, as FP4
    int32_t factor, reach;       // reach: the largest magnitude that a position adds, over the factor, its two powers taken apart
};

// The opaque table object: levels, the 16 products, and what the kernels need to know about them.
struct dg_lut {
    int32_t bits;        // code width: 2 (the paper's kernels), 3 or 4 (Sec. 3.3); 2^bits levels per side
    int8_t levels_w[16];
    int8_t levels_a[16];
    int16_t entry[256];  // entry[(w << bits) | a] = levels_w[w] * levels_a[a]; 2^(2*bits) entries are used
    dg_lut_dtype dtype;
    bool separable;      // built from level vectors (the matrix-core comparison kernel needs them)
    float fentry[16];    // DG_LUT_F32 tables only: binary32 products of floating-point levels
    int32_t min_entry;   // smallest product
    int32_t max_entry;   // largest product
    int32_t max_abs;     // max |product|
    DgTwoLookups two[2]; // of the table, and of the transposed one (found when the table is built)
    DgBitSums bit_sums;  // (found when the table is built)
    DgTwoPowers two_powers;      // (the same)
};

// 16 table entries passed to kernels by value (no device allocation is needed for a table).
struct DgTable16 {
    int16_t e[16];
};

// One implicit-GEMM problem.  A plain GEMM is the convolution with B = N, H = W = 1, a 1x1 filter
// and Cin = K: "pixel" n is activation row n.
//   M = Cout, N = B*OH*OW, K = KH*KW*Cin, reduction index k = (kh*KW + kw)*Cin + ci.
struct DgProblem {
    int32_t M, N, K;
    int32_t H, W, Cin, KH, KW, sh, sw, ph, pw, OH, OW;
    const uint8_t *Wp;    // packed weights, [M][K/4]
    const uint8_t *Xp;    // packed activations, [B*H*W][Cin/4]
    int32_t *C;           // int32 output (used when scale == nullptr)
    float *Cf;            // fp32 output (used when scale != nullptr)
    const float *scale;   // per-m scale or nullptr
    int64_t stride_cm, stride_cn;   // element strides of the output
    // Re-quantising epilogue (the packed activations of the next layer instead of C / Cf), used when Qp != nullptr:
    // code = clip(rint(q_scale * (float(sum) * scale[m]) + q_zero), q_lo, q_lo + 3) - q_lo, four channels per byte.
    uint8_t *Qp;          // [N][M/4]; requires scale, M % 4 == 0 and the NHWC output order (stride_cm == 1)
    float q_scale, q_zero;
    int32_t q_lo;
    int32_t cached;       // the output goes through the caches (dg_output_cached; set by the kernels' launchers)
};

// Whether an output is better written through the caches than past them: a tile's rows are 128-byte pieces of the output's, and where those
// are no whole multiples of 64 bytes a memory line's parts come from different wavefronts and tiles; streamed they are written one by
// one, through L2 together.  Same kernels, us, streamed and through the caches: 5942 x 6830 x 320 (direct-load tiles) 108, 51; 3648 x 7425 x 256
// (stationary weights) 52.8, 29.7; 1986 x 7254 x 1280 (staged) 56.5, 42.2; 28x28x512 -> 264 at batch 32 15.5, 14.1; 28x28x128 -> 104 3x3 at batch
// 16, 4-bit, 12.6, 12.0; 1000 x 1001 x 2048 8.1, 8.0; and one-bit tables (dg_onebit_kernel.hip) 3569 x 7478 x 704 55, 28.  Whole pieces: 56x56x256 -> 64 at
// batch 32 8.6, 9.9; one-bit tables 112x112x64 -> 96 3x3 at batch 12 20.4, 22.5.  Of 400 drawn layers and products with such rows, 0.1 to 400 MB, two were more than 2 % longer
// through the caches (112x112x64 -> 24 at batch 21, stationary weights, 7.8, 8.3; one-bit tables 7079 x 1548 x 2112 29.1, 31.3); two planes 15x15x448 -> 1000 3x3
// at batch 14 56.4, 56.6.
inline int32_t dg_output_cached(const DgProblem &p)
{
    if (p.Qp) return 0;                                     // (packed codes, bytes)
    const int64_t row = p.stride_cm == 1 ? p.stride_cn : p.stride_cm;
    return row % 16 != 0 || (p.scale ? (uintptr_t)p.Cf : (uintptr_t)p.C) % 64 != 0;
}

// n / d for 0 <= n < 2^31 by multiply-high and shift, d fixed per launch and prepared on the host:
// n / d == umulhi(2 n, mul) >> shift with shift = ceil(log2 d) and mul = ceil(2^(31+shift) / d) < 2^32
// (the error mul * d - 2^(31+shift) is below d <= 2^shift = 2^((31+shift) - 31)).  d = 1 is no case of its own (mul = 2^31, shift = 0):
// a branch around it cost a kernel's start, which works out four to eight pixels' places, 10 to 30 instructions.
struct DgFastDiv {
    uint32_t mul, shift, d;
};

__device__ __forceinline__ uint32_t dg_fdiv(uint32_t n, const DgFastDiv &f)
{
    return __umulhi(2u * n, f.mul) >> f.shift;
}

inline DgFastDiv dg_make_div(uint32_t d)
{
    DgFastDiv f = {0x80000000u, 0u, d};
    if (d < 2) return f;
    while ((1ull << f.shift) < d) ++f.shift;
    f.mul = (uint32_t)(((1ull << (31 + f.shift)) + d - 1) / d);
    return f;
}

// The kernel's arguments, BYTES of them, asked for at once: one word of every 64-byte line, all before the first is waited for.  A
// line's first reader waits 0.2 - 0.4 us for it (500 - 900 cycles measured, launches with new arguments), and a structure of 300 to
// 550 bytes read where its fields are needed pays for that two or three times in a row before a kernel's first load.  The staged kernel
// with it: 28x28x128 -> 128 3x3 at batch 8 with 4-bit codes (packing kernel included) 11.4 -> 10.9 us, 28x28x256 -> 256 in two planes
// 20.8 -> 20.4.  The split-K, stationary-weight, few-columns and ragged kernels, whose argument loads the compiler puts together by
// itself, gained nothing.
template <size_t BYTES>
__device__ __forceinline__ void dg_fetch_arguments()
{
    constexpr int LINES = (int)((BYTES + 63) / 64);
    static_assert(LINES <= 10, "one operand of the statement below per line");
    typedef const uint32_t __attribute__((address_space(4))) *Segment;
    const Segment s = (Segment)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t v[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) v[i] = s[16 * (i < LINES ? i : LINES - 1)];
    asm volatile("" ::"s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]), "s"(v[4]), "s"(v[5]), "s"(v[6]), "s"(v[7]), "s"(v[8]), "s"(v[9]));
}

// Value of a test / measurement override (an environment variable), or nullptr.  Overrides are looked at only when
// DG_TEST_OVERRIDES=1 was set when the library was first called; otherwise this returns nullptr without reading anything.
const char *dg_override(const char *name);
bool dg_overrides_enabled();
// Number of SIMD units of the current device (compute units x 4), asked from the runtime once.
int dg_simd_count();
// Record the calling thread's error detail and return `s`.
dg_status dg_fail(dg_status s, const char *fmt, ...);
// Turn the launch status of the last kernel into a dg_status.
dg_status dg_check_launch(const char *what);

// Kernel launchers (each validates nothing: the API layer has done that).
dg_status dg_launch_pack(const uint8_t *codes, int64_t rows, int64_t K, int bits, uint8_t *packed,
                         hipStream_t stream);
// 2-bit codes of the pixels (b, oh * sh, ow * sw) only, [B][H][W][Cin] -> [B][OH][OW][Cin / 4]; Cin % 16 == 0, codes
// 16-byte and packed 4-byte aligned (the caller checks)
dg_status dg_launch_pack_strided_pixels(const uint8_t *codes, int64_t B, int32_t H, int32_t W, int32_t OH, int32_t OW, int32_t sh,
                                        int32_t sw, int32_t Cin, uint8_t *packed, hipStream_t stream);
dg_status dg_launch_quantize_pack(const float *x, int64_t rows, int64_t K, float scale, float zero_point,
                                  int32_t lo, uint8_t *packed, hipStream_t stream);
dg_status dg_launch_dequantize(const int32_t *acc, int64_t rows, int64_t C, const float *scale, float *out,
                               hipStream_t stream);
dg_status dg_launch_lds(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
dg_status dg_launch_lds_f32(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_onehot_f32_preferred(const dg_lut *lut, const DgProblem &p);   // binary32 tables on the matrix cores
dg_status dg_launch_onehot_f32(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_perm_supports(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_perm(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_perm_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_decode_supports(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_decode(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_decode_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_lut65k_supports(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_lut65k(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_onehot_supports(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_onehot(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_onehot_config_name(const dg_lut *lut, const DgProblem &p);
// the one-hot split-K kernel reading activations one code per byte (p.Xp = those bytes) and packing them as it loads
bool dg_onehot_codes_supports(const dg_lut *lut, const DgProblem &p);
bool dg_onehot_codes_pays(const DgProblem &p);      // AUTO: the repeated packing costs less than the saved launch
// (`sparse_tiles`: the tiled form on the sparse instruction, where dg_onehot_codes_tiled_sparse says it applies)
dg_status dg_launch_onehot_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream, bool sparse_tiles = false);
const char *dg_onehot_codes_config_name(const dg_lut *lut, const DgProblem &p, bool sparse_tiles = false);
// the one-hot tiled kernel (64 x 32 and 64 x 64 tiles) doing the same on layers of a few microseconds
bool dg_onehot_codes_tiled_supports(const dg_lut *lut, const DgProblem &p);
bool dg_onehot_codes_tiled_sparse(const dg_lut *lut, const DgProblem &p);  // on the sparse instruction (channel axis contiguous)
bool dg_onehot_codes_tiled_pays(const dg_lut *lut, const DgProblem &p, bool sparse_tiles);   // AUTO: shorter than packing kernel + AUTO's kernel
bool dg_sparse_supports(const dg_lut *lut, const DgProblem &p);
bool dg_sparse_preferred(const dg_lut *lut, const DgProblem &p);     // AUTO's choice between the two one-hot kernels
dg_status dg_launch_sparse(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
// What AUTO's plan on the one-hot kernels is: K split over a workgroup, or tiles on the dense or the sparse instruction, from direct loads or staged.
enum class DgOneHotForm { SplitK, Dense, Sparse, Staged, Staged32x128 };
// *busiest: what its tiles give the busiest SIMD, in blocks of 32 x 32 by thousands of positions.
DgOneHotForm dg_onehot_auto_form(const dg_lut *lut, const DgProblem &p, double *busiest = nullptr);
const char *dg_sparse_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_onebit_preferred(const dg_lut *lut, const DgProblem &p);       // tables that are two one-bit lookups, on the FP4 instruction
dg_status dg_launch_onebit(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_onebit_config_name(const DgProblem &p);
bool dg_twopower_preferred(const dg_lut *lut, const DgProblem &p);     // products of levels, on the FP6 / FP4 instruction
dg_status dg_launch_twopower(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_twopower_config_name(const DgProblem &p);
// A 2-bit table as factor * u[w] * v[a], u and v whole numbers without a common factor each; false if it is no such product.
bool dg_find_levels(const dg_lut *lut, int (&u)[4], int (&v)[4], int *factor);
void dg_find_bit_sums(dg_lut *lut);
void dg_find_two_powers(dg_lut *lut);
bool dg_planes_codes_preferred(const dg_lut *lut, const DgProblem &p);    // p.Xp: codes one per byte, by their bits on the int8 instruction
dg_status dg_launch_planes_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_planes_codes_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_planes_preferred(const dg_lut *lut, const DgProblem &p);          // the same on packed 2-bit codes
dg_status dg_launch_planes(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
// About how long AUTO's kernels take, us: 3- and 4-bit codes as two lookups, from `codes` MB of unpacked codes, packing included; 2-bit tables with
// entries beyond int8, on packed codes.  0 where that was not measured.
double dg_onehot_nibble_time(const dg_lut *lut, const DgProblem &p, double codes);
double dg_onehot_two_plane_time(const dg_lut *lut, const DgProblem &p);
bool dg_onebit_codes_preferred(const dg_lut *lut, const DgProblem &p, bool stationary);    // p.Xp: codes one per byte
bool dg_onebit_codes_spare_packing(const dg_lut *lut, const DgProblem &p);                 // in place of packing first, where AUTO then runs the one-bit kernel
dg_status dg_launch_onebit_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_ragged_preferred(const dg_lut *lut, const DgProblem &p, bool codes);      // taps of no whole 32-position groups; `codes`: p.Xp one per byte
const char *dg_ragged_config_name(const dg_lut *lut, const DgProblem &p, bool codes);
dg_status dg_launch_ragged(const dg_lut *lut, const DgProblem &p, bool codes, hipStream_t stream);
void dg_find_two_lookups(dg_lut *lut);
bool dg_nibble_preferred(const dg_lut *lut, const DgProblem &p);      // 3- and 4-bit codes as two 2-bit ones each
dg_status dg_launch_nibble(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_nibble_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_sparse4_supports(const dg_lut *lut, const DgProblem &p);      // 4-bit codes on the sparse instruction
bool dg_sparse4_preferred(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_sparse4(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_sparse2p_supports(const dg_lut *lut, const DgProblem &p);     // two-plane 2-bit tables on the sparse instruction
bool dg_sparse2p_preferred(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_sparse2p(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_staged2p_preferred(const dg_lut *lut, const DgProblem &p);    // the same with staged operands, in any of their tiles
dg_status dg_launch_staged2p(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
const char *dg_staged2p_config_name(const dg_lut *lut, const DgProblem &p);
bool dg_sparse_ws_supports(const dg_lut *lut, const DgProblem &p);    // short K: weight operands stationary in registers
bool dg_sparse_ws_preferred(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_sparse_ws(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_sparse_ws_codes_supports(const dg_lut *lut, const DgProblem &p);                       // p.Xp: codes one per byte
dg_status dg_launch_sparse_ws_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_fewn_supports(const dg_lut *lut, const DgProblem &p);         // few activation rows: weights as the sparse operand
bool dg_fewn_preferred(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_fewn(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
bool dg_smalln_supports(const dg_lut *lut, const DgProblem &p);
dg_status dg_launch_smalln(const dg_lut *lut, const DgProblem &p, hipStream_t stream);
dg_status dg_launch_smalln_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream);   // p.Xp: codes one per byte
