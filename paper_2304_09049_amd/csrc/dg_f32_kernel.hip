// Binary32 tables on the matrix cores.  The sum is one binary32 addition per reduction position, in ascending k, from +0
// (dg_lds_kernel.hip is the plain form); it cannot be split or reordered, so the parallel axis is the outputs alone.
//
//   acc[n][m] <- acc[n][m] + T[w(m,k)][a(n,k)]  =  fma chain over v = 0..3 of  [a(n,k) == v] * T[w(m,k)][v]
//
// v_mfma_f32_16x16x4_f32 does that for a 16 x 16 block and one position: its four products per output are the four codes v,
// three of them by zero.  A product by zero is +-0 and leaves the sum as it is (a sum that starts at +0 never becomes -0), the
// fourth is the entry itself, so whatever the order of the four, the result is the one rounded addition.  That needs finite
// entries (0 * inf is not 0), and no subnormal numbers, which this kernel does not want to depend on: every entry 0 or at least
// 2^-100, hence every partial sum a multiple of 2^-123 (the host checks; other tables stay with the plain kernel).
//
// Operands: lane (i = lane % 16, v = lane / 16) supplies [a(n0 + i, k) == v] and T[w(m0 + i, k)][v].  Two positions' worth comes from
// one 8-byte LDS read at a 4-bit index, the two codes: 16 pairs per v, for either operand; a pixel whose tap lies outside the
// image reads pairs of zeros instead.
//
// Bound by the matrix pipe: 32 cycles of it per position and block of 256 outputs, a quarter of it useful -- 8 table additions per SIMD and
// cycle at best.  Binary32 matrix instructions do not overlap with vector instructions at all, whosever they are: a group of n between two of
// them costs 4.4 + 2 n cycles at two wavefronts per SIMD (measured, registers only), while LDS reads between them are free.  So a word's 16
// matrix instructions are issued in one piece, only the next word's table reads between them, and the next word's 28 vector
// instructions before or behind them in another: 40 cycles per position instead of 51 with the vector instructions
// spread three at a time.  A sum cannot be split along K, so blocks are small and wavefronts many.  The plain kernel spends 5 vector instructions
// and an LDS read per addition (3 additions per SIMD and cycle).  Packed codes, graph replays, the plain kernel, this one: 28x28x128 -> 128 3x3
// at batch 4 (1568 blocks) 61.1, 42.3 us (spread: 48.8), at batch 8 118.7, 81.2; 56x56x64 -> 64 3x3 at batch 8 109.2, 72.7; 14x14x36 -> 100 3x3 at
// batch 8 (686) 18.4, 13.1.  Layers of one load per pixel, K = 32, with ten or more blocks per SIMD were 2 - 4 % shorter spread (56x56x32 -> 152 1x1
// at batch 6 13.7, 14.0), other two-word loads 2 - 30 % longer.
// Reading the pairs one at a time, just before their instructions, instead of a word ahead: 57.1 us on the first, 48.3 then.
#include "dg_common.h"

#include <cmath>
#include <cstdlib>

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct F32Args {
    DgProblem p;
    float e[16];
    DgFastDiv div_ow, div_oh;
    int32_t tiles_m;
    int64_t tiles;
};

template <int CHW>
struct __attribute__((packed, aligned(1))) RawWords {
    uint32_t v[CHW];
};

// CHW: words per load, 4 or 2 where a tap is whole groups of so many.  WHOLE: Cin % 16 == 0, every
// word of a tap is 16 codes; otherwise the last word of a tap is read so that it ends with the tap, and shifted.
// One software pipeline over all of K: a word's pairs are read from LDS between the matrix instructions of the word before.
template <int CHW, bool WHOLE>
__global__ void __launch_bounds__(256)
onehot_f32_kernel(F32Args a)
{
    static_assert(WHOLE || CHW == 1, "taps that are no whole words are loaded word by word");
    constexpr int RING = CHW == 1 ? 4 : 2;                  // loads in flight
    __shared__ float s_table[2 * 4 * 32 + 32];              // pairs of entries [v][pair], pairs of one-hot values, pairs of zeros
    const DgProblem &p = a.p;
    for (int i = threadIdx.x; i < 2 * 4 * 32 + 32; i += 256) {
        const int v = (i >> 5) & 3, code = (i & 1) ? (i >> 3) & 3 : (i >> 1) & 3;
        s_table[i] = i < 128 ? a.e[4 * code + v] : (i < 256 && code == v ? 1.0f : 0.0f);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, i16 = lane & 15, v = lane >> 4;
    const int64_t tile = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= a.tiles) return;                            // (whole wavefronts; no barrier follows)
    const int m0 = (int)(tile % a.tiles_m) * 16, n0 = (int)(tile / a.tiles_m) * 16;
    const int L = p.Cin / 4, loads = (L + 4 * CHW - 1) / (4 * CHW), total = p.KH * p.KW * loads;

    const uint8_t *w_next = p.Wp + (int64_t)min(m0 + i16, p.M - 1) * (p.K / 4);
    // this lane's pixel (32-bit offsets: the host sends inputs below 2^31 bytes; unsigned, as what a pixel's and a tap's offset
    // are by themselves may be more where the padding is large, and their sum is the one of a byte inside)
    const bool live = n0 + i16 < p.N;
    const int nn = min(n0 + i16, p.N - 1);
    const int line = (int)dg_fdiv((uint32_t)nn, a.div_ow), ow = nn - line * p.OW;
    const int img = (int)dg_fdiv((uint32_t)line, a.div_oh), oh = line - img * p.OH;
    const int ih0 = oh * p.sh - p.ph, iw0 = ow * p.sw - p.pw;
    const uint32_t off0 = ((uint32_t)(img * p.H + ih0) * (uint32_t)p.W + (uint32_t)iw0) * (uint32_t)L;

    struct Load {
        RawWords<CHW> w, x;
        uint32_t base;                                      // where this pixel's pairs are read
        int shift, codes;                                   // (the same in every lane)
    };
    const uint32_t w_base = 128 * v, x_base = 512 + 128 * v, zeros = 1024;
    int kh = 0, kw = 0, j = 0, fetched = 0;
    uint32_t x_at;                                          // the tap's bytes of the pixel (outside the image: the first pixel's)
    uint32_t tap_base;
    auto enter_tap = [&]() {
        const uint32_t tap_off = ((uint32_t)kh * (uint32_t)p.W + (uint32_t)kw) * (uint32_t)L;
        const bool ok = live & ((uint32_t)(ih0 + kh) < (uint32_t)p.H) & ((uint32_t)(iw0 + kw) < (uint32_t)p.W);
        x_at = ok ? off0 + tap_off : 0u;
        tap_base = ok ? x_base : zeros;
    };
    enter_tap();
    auto fetch = [&](Load &t) {                              // past the end: the last words again, as pairs of zeros
        const int start = WHOLE ? 4 * CHW * j : min(4 * j, L - 4);
        t.shift = 8 * (4 * j - start);
        t.codes = min(16, 4 * (L - 4 * j));
        t.w = *(const RawWords<CHW> *)(w_next + start);
        t.x = *(const RawWords<CHW> *)(p.Xp + x_at + start);
        t.base = fetched < total ? tap_base : zeros;
        if (++fetched < total && ++j == loads) {             // (uniform)
            j = 0;
            if (++kw == p.KW) kw = 0, ++kh;
            w_next += L;
            enter_tap();
        }
    };

    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const char *table = (const char *)s_table;
    struct Pairs {
        float2 e[8], o[8];
    };
    // Pair q = bits 4q ... 4q + 3 of the word, as a byte offset into a table of pairs: the even q in the bytes of one word, the odd
    // ones in another's (kept as they are: a byte of them plus the base is one instruction).
    auto read_pairs = [&](const Load &t, int c, Pairs &d) {
        auto split = [&](uint32_t word, uint32_t (&s)[2]) {
            if (!WHOLE) word >>= t.shift;
            s[0] = (word & 0x0F0F0F0Fu) << 3, s[1] = (word >> 1) & 0x78787878u;
            asm("" : "+v"(s[0]), "+v"(s[1]));
        };
        uint32_t w[2], x[2];
        split(t.w.v[c], w);
        split(t.x.v[c], x);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            d.e[q] = *(const float2 *)(table + (w_base + ((w[q & 1] >> (8 * (q / 2))) & 255u)));
            d.o[q] = *(const float2 *)(table + (t.base + ((x[q & 1] >> (8 * (q / 2))) & 255u)));
        }
    };
    auto multiply = [&](const Pairs &d, int q0, int q1) {
#pragma unroll
        for (int q = q0; q < q1; ++q) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.o[q].x, d.e[q].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d.o[q].y, d.e[q].y, acc, 0, 0, 0);
        }
    };

    Load ring[RING];
    Pairs pairs[2];
#pragma unroll
    for (int i = 0; i < RING; ++i) fetch(ring[i]);
    read_pairs(ring[0], 0, pairs[0]);
    for (int done = 0; done < total; done += RING)
#pragma unroll
        for (int i = 0; i < RING; ++i) {
            if (done + i >= total) break;                   // (uniform)
            const int codes = ring[i].codes;
#pragma unroll
            for (int c = 0; c < CHW; ++c) {
                const int cur = (i * CHW + c) & 1;
                read_pairs(c + 1 < CHW ? ring[i] : ring[(i + 1) % RING], c + 1 < CHW ? c + 1 : 0, pairs[cur ^ 1]);
                if constexpr (WHOLE) {
                    multiply(pairs[cur], 0, 8);
                    __builtin_amdgcn_sched_group_barrier(0x002, 64, 0);      // (all the vector instructions there are, then none)
#pragma unroll
                    for (int k = 0; k < 16; ++k) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                } else {
                    multiply(pairs[cur], 0, 2);
                    if (codes > 4) multiply(pairs[cur], 2, 4);       // (uniform)
                    if (codes > 8) multiply(pairs[cur], 4, 6);
                    if (codes > 12) multiply(pairs[cur], 6, 8);
                }
            }
            fetch(ring[i]);
        }

    const int m = m0 + i16;
    if (m >= p.M) return;
    const float scale = p.scale ? p.scale[m] : 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int n = n0 + 4 * v + e;
        if (n >= p.N) continue;
        const int64_t o = (int64_t)m * p.stride_cm + (int64_t)n * p.stride_cn;
        p.Cf[o] = p.scale ? __fmul_rn(acc[e], scale) : acc[e];
    }
}

}   // namespace

// AUTO compares what the two kernels take per position of K.  This one: 2 + 16.7 w ns, w the wavefronts on the busiest SIMD (a
// workgroup of four blocks per compute unit at a time; w = 1: 17.5 - 21 ns measured, 2: 37, 3: 52, 4: 68), and a start 0.2 us longer than the
// plain one's; with less than 64 positions, or a second word per tap that is mostly empty (Cin = 20 ... 28), 7 + 19.5 w in all.  The plain one: the
// outputs at 5.8 thousand per ns -- 5.4 to 7.9 measured, half of that where it reads bytes (Cin % 16 != 0) -- and 21 at least where K is long, below
// which its own chain of additions does not get (50 to 100 thousand outputs: 21.2 - 22.6; one word per load here, Cin % 32 == 16, is no
// faster).  Of 215 layers of 40 to 400 thousand outputs the choice costs 1.1 % over the better one on average, 4 % at most against 7 + 19.5 w for all
// and no chain, 5 % less than it on average: 14x14x256 -> 256 3x3 at batch 2 (400 blocks) goes over (52.1 -> 43.8 us), 28x28x32 -> 72 3x3 at
// batch 2 9.4 -> 8.4, 28x28x100 -> 48 3x3 at batch 2 40.5 -> 28.0; 7x7x16 -> 576 1x1 at batch 4 stays (2.9 against 3.1), 28x28x20 -> 16 1x1 at
// batch 5 (2.9 against 3.5), 14x14x48 -> 320 5x5 (28.8 against 30.4) and 28x28x32 -> 72 1x1 at batch 2 (3.2 against 3.3) too.
// DG_F32_MFMA: 0 never, 1 whatever the size.
bool dg_onehot_f32_preferred(const dg_lut *lut, const DgProblem &p)
{
    if (lut->dtype != DG_LUT_F32 || p.Cin < 16) return false;
    for (int i = 0; i < 16; ++i) {
        const float e = lut->fentry[i];
        if (!std::isfinite(e) || (e != 0.0f && std::fabs(e) < 0x1p-100f)) return false;
    }
    const int64_t blocks = ((int64_t)(p.M + 15) / 16) * (((int64_t)p.N + 15) / 16);
    if (blocks > INT32_MAX) return false;
    if ((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * (p.Cin / 4) >= ((int64_t)1 << 31)) return false;      // (32-bit byte offsets)
    if (const char *f = dg_override("DG_F32_MFMA")) return atoi(f) != 0;
    const int64_t groups = (blocks + 3) / 4, units = dg_simd_count() / 4;
    const double w = (double)((groups + units - 1) / units), few = 5.0 + 2.8 * w, start = 200.0 / p.K;
    const double here = 2.0 + 16.7 * w + (p.K < 64 || (p.Cin < 32 && p.Cin % 16 != 0) ? few : start);
    const double plain = (double)p.M * p.N / (p.Cin % 16 == 0 ? 5800.0 : 2900.0);
    const double chain = blocks >= 256 && p.K > 256 && p.Cin % 32 == 0 ? 21.0 : 0.0;
    return here < (plain > chain ? plain : chain);
}

dg_status dg_launch_onehot_f32(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    F32Args a;
    a.p = p;
    for (int i = 0; i < 16; ++i) a.e[i] = lut->fentry[i];
    a.div_ow = dg_make_div((uint32_t)p.OW), a.div_oh = dg_make_div((uint32_t)p.OH);
    a.tiles_m = (p.M + 15) / 16;
    a.tiles = (int64_t)a.tiles_m * (((int64_t)p.N + 15) / 16);
    const dim3 grid((unsigned)((a.tiles + 3) / 4));
    if (p.Cin % 64 == 0) hipLaunchKernelGGL((onehot_f32_kernel<4, true>), grid, dim3(256), 0, stream, a);
    else if (p.Cin % 32 == 0) hipLaunchKernelGGL((onehot_f32_kernel<2, true>), grid, dim3(256), 0, stream, a);
    else if (p.Cin % 16 == 0) hipLaunchKernelGGL((onehot_f32_kernel<1, true>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((onehot_f32_kernel<1, false>), grid, dim3(256), 0, stream, a);
    return dg_check_launch("onehot_f32_kernel");
}
