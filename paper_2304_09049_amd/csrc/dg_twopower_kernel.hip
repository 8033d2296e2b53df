// 2-bit tables that are products of levels, T[w][a] = f u[w] v[a], on the matrix instruction that takes FP6 and FP4 numbers, for matrix
// products (and 1x1 layers without stride and padding) whose
//
//   u[w] is an FP6 (E2M3) number of eighths: up to 15, even up to 30, a multiple of 4 up to 60, of either sign, and
//   v[a] is the sum of two of 0, 1, 2, 4, 8 and their negatives -- any whole number from -10 to 10 is
//
// (u and v without common factors: all pairs of levels from -8 to 7 are such).  A position then adds u[w], moved by a power of two, twice: two
// places of the reduction where the one-hot form has four, and v_mfma_f32_32x32x64_f8f6f4 takes 64 places in the 32 cycles in which the sparse
// int8 instruction takes 16 positions of four.  Every product on the matrix cores is u[w] times 0 or a signed power of two; they and all sums
// are multiples of 1/16 below 2^20 (the host checks; takes), hence exact in binary32 in any order, and 16 f times the sum is the result.
//
// Neither operand is the packed word itself: u[w] needs six bits in a row, 24 vector instructions per 16 codes (expand), the two powers of the
// activation's 19.  So the tiles are as large as the registers allow: up to 128 channels x 512 pixels to a workgroup of eight
// wavefronts, which share the channels' numbers (made once a run of 256 positions, 16 codes of a row a thread and word, and handed over in LDS) and have 64
// pixels each, whose packed words lie in LDS and whose powers are made where they are used, for four blocks of channels.  That is 7
// vector instructions per matrix instruction.  On the 8192-cube, 420 to 460 us on a settled clock, an instruction and SIMD takes
// 25.9 to 28.1 ns: the pipe is busy for 0.58 of the cycles, at 1.99 GHz; a wavefront waits for 28 % of its own and has an instruction ready that is not issued
// for 34 %: two wavefronts to a SIMD do not fill it.  Power comes next: such operands in registers and nothing else take 19.2 (single bits by FP4
// levels 16.4, zeros 13.6), the loop with neither operand made 23.6.  The output, which a lone workgroup of a compute unit stores with its matrix pipe idle, is
// 10 us a round of the largest tiles.  In the narrow tiles the vector unit is the bound: 18 instructions beside each matrix instruction, 77 cycles for its 32.
// Measured, us, the sparse kernels and this one (packed codes, graph replays; both on one card):
//   8192-cube 725, 454          4096-cube 97, 63          4873 x 7116 x 4672 387, 176          6481 x 5352 x 1472 131, 67
//   1305 x 1621 x 1856 20.8, 14.1          656 x 6500 x 896 17.6, 11.4          1900 x 1877 x 960 16.7, 11.0
#include "dg_lds_dma.h"
#include "dg_onehot_kernel.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <numeric>

namespace {

using namespace dgoh;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));

struct TwoPowerArgs {
    DgProblem p;
    uint32_t bytes[6];       // of four FP6 numbers' three bytes (expand): code w's share in byte w
    uint32_t powers;         // byte a: the two signed powers of activation code a, as FP4
    int32_t factor;
    FastDiv div_band, div_last;
    int32_t tiles_n, band_log2;
    uint32_t band_tiles, x_bytes;
};

// Sums to results: 16 factor times a sum, which is whole once it is 16 times as large.
__device__ __forceinline__ v16i results(const f32x16 &sums, int32_t factor)
{
    v16i out;
#pragma unroll
    for (int e = 0; e < 16; ++e) out[e] = (int)(sums[e] * 16.0f);
    if (factor != 1) {                                      // (uniform; a 32-bit product is 16 cycles)
#pragma unroll
        for (int e = 0; e < 16; ++e) out[e] *= factor;
    }
    return out;
}

template <bool TR>
__device__ __forceinline__ f32x16 step(const i32x8 &w, const v4i &x, f32x16 c)
{
    const i32x8 y = {x[0], x[1], x[2], x[3], 0, 0, 0, 0};
    return TR ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(y, w, c, 4, 2, 0, 0, 0, 0)
              : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, y, c, 2, 4, 0, 0, 0, 0);
}

// KS = 2: twice the wavefronts, two to a tile, each with half of the runs of K; their sums meet in LDS.
template <int BM, int WN, int WAVES, int KS, bool TR>
__global__ void __launch_bounds__(64 * WAVES * KS, 2)
twopower_kernel(TwoPowerArgs a)
{
    constexpr int SHARE = 2 * (BM * 6144) + 2 * WAVES * (WN * 2048);      // bytes of the wavefronts that walk one share of K
    constexpr int WIDE = BM * 4096, WEIGHTS = BM * 6144;    // bytes of a run's weights: the 16-byte parts, all
    constexpr int PIXELS = WN * 2048, LOADS = 2 * WN;
    constexpr int SEGMENTS = 2 * BM / WAVES;                // 16-byte pieces of weights a thread expands per run
    static_assert(SEGMENTS * WAVES == 2 * BM, "whole pieces");
    // A block's place in LDS as an offset of the step's one address.  Put in with the lane, the compiler keeps an address per block, and the tile of
    // 128 x 256 reloads two from scratch in each run, whose waits are for the next run's loads as well: 4873 x 7116 x 4672 column-major 195 -> 176 us,
    // 3992 x 1839 x 2944 37.5 -> 32.2, row-major level.  (The others have the registers; 2275 x 903 x 4544 by rows is 4 % longer so.)
    constexpr bool ONE_BASE = BM == 4 && WAVES == 4;
    __shared__ uint4 s_mem[KS * SHARE / 16];
    const DgProblem &p = a.p;
    dg_fetch_arguments<sizeof(a)>();
    const int lane = threadIdx.x & 63, all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5;
    const int wave = all % WAVES, ks = all / WAVES;
    int m_tile, n_tile;
    {
        const uint32_t t = xcd_contiguous(blockIdx.x, gridDim.x), band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n - first);
        m_tile = (int)(width == 1 << a.band_log2 ? t_in >> a.band_log2 : fdiv(t_in, a.div_last));
        n_tile = first + (int)t_in - m_tile * width;
    }
    const int m0 = m_tile * (32 * BM), n0 = (n_tile * WAVES + wave) * (WN * 32);
    // this share's runs g0 ... , `whole` of them of 256 positions; then up to `chunks` (of 64 positions) what is left, which only the last share has
    const int whole = p.K / 256 / KS, g0 = whole * ks, chunks = ks == KS - 1 ? p.K / 64 : 4 * (g0 + whole);
    const int left = p.K / 64 - 4 * whole * KS;
    char *const mem = (char *)s_mem + ks * SHARE;
    const uint32_t row_bytes = (uint32_t)p.K / 4;

    // ---- weights: thread t of a share loads segment t % 4 of a run of row t / 4 (rows beyond M, bytes past the last row: zeros; what lies past
    // the end of K is never multiplied)
    const __amdgpu_buffer_rsrc_t w_buffer =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.Wp + (int64_t)m0 * row_bytes), 0, (int)(min(p.M - m0, 32 * BM) * row_bytes), 0x00020000);
    const int w_row = (threadIdx.x % (64 * WAVES)) >> 2, w_seg = threadIdx.x & 3;
    const uint32_t w_ld = w_row * row_bytes + w_seg * 16;
    struct Raw {
        v4i v[SEGMENTS];
    };
    auto load_weights = [&](Raw &raw, int g) {
#pragma unroll
        for (int i = 0; i < SEGMENTS; ++i)
            raw.v[i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(w_buffer, w_ld + i * (16 * WAVES) * row_bytes + g * 64, 0, 0);
    };
    // A word's 16 numbers of six bits, even codes and then odd ones, as the pixels' are: numbers 4 q ... 4 q + 3 are three bytes, whose bits come from
    // one or two of the four codes (a.bytes).  Made for all four q at once in q0, q1 and q2, then put in order.
    auto expand = [&](uint32_t w, int (&o)[3]) {
        const uint32_t M = 0x03030303u, w2 = w >> 2;
        const uint32_t u = __builtin_amdgcn_perm(w2, w, 0x06040200u), v = __builtin_amdgcn_perm(w2, w, 0x07050301u);
        const uint32_t e0 = u & M, e1 = (u >> 4) & M, e2 = v & M, e3 = (v >> 4) & M;
        const uint32_t q0 = __builtin_amdgcn_perm(0u, a.bytes[0], e0) | __builtin_amdgcn_perm(0u, a.bytes[1], e1);
        const uint32_t q1 = __builtin_amdgcn_perm(0u, a.bytes[2], e1) | __builtin_amdgcn_perm(0u, a.bytes[3], e2);
        const uint32_t q2 = __builtin_amdgcn_perm(0u, a.bytes[4], e2) | __builtin_amdgcn_perm(0u, a.bytes[5], e3);
        // [q0.0 q1.0 q2.0 q0.1] [q1.1 q2.1 q0.2 q1.2] [q2.2 q0.3 q1.3 q2.3]
        const uint32_t x01 = __builtin_amdgcn_perm(q1, q0, 0x01000400u);
        o[0] = (int)__builtin_amdgcn_perm(q2, x01, 0x03040100u);
        const uint32_t y = __builtin_amdgcn_perm(q1, q0, 0x06020005u);
        o[1] = (int)__builtin_amdgcn_perm(q2, y, 0x03020500u);
        const uint32_t z = __builtin_amdgcn_perm(q1, q0, 0x00070300u);
        o[2] = (int)__builtin_amdgcn_perm(q2, z, 0x07020106u);
    };
    // segment s of rows 32 b ... as [s][b][lane], 16 bytes of a lane and 8 elsewhere; lanes exchanged so that a thread's neighbours, which write the
    // other segments, are on other banks
    auto expand_half = [&](const Raw &raw, int half, uint32_t buf) {
#pragma unroll
        for (int i = 0; i < SEGMENTS; ++i) {
            int o[2][3];
            expand((uint32_t)raw.v[i][2 * half], o[0]);
            expand((uint32_t)raw.v[i][2 * half + 1], o[1]);
            const int row = w_row + i * (16 * WAVES), place = half * 32 + (row & 31), block = w_seg * BM + (row >> 5);
            *(v4i *)(mem + buf + (block * 64 + (place ^ (2 * w_seg))) * 16) = (v4i){o[0][0], o[0][1], o[0][2], o[1][0]};
            *(v2i *)(mem + buf + WIDE + (block * 64 + (place ^ (4 * w_seg))) * 8) = (v2i){o[1][1], o[1][2]};
        }
    };

    // ---- pixels: lane l of a load fetches segment (l % 4) ^ (row / 4 % 4) of row l / 4 of 16, as in dg_onebit_kernel.hip
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);
    const int l_row = lane >> 2, l_seg = (lane & 3) ^ (lane >> 4);
    uint32_t off0[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int n = n0 + 16 * i + l_row;
        off0[i] = n < p.N ? (uint32_t)n * row_bytes : 0x80000000u;
    }
    const uint32_t x_lds = dg_lds_address(mem) + 2 * WEIGHTS + wave * 2 * PIXELS;
    auto fetch = [&](int g, int odd) {
        const uint32_t dst = x_lds + odd * PIXELS;
        const int c = 4 * g + l_seg;
        const uint32_t dead = c < chunks ? 0u : 0x80000000u;
        dg_for<LOADS>([&](auto i) { dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + c * 16) | dead, dst); });
    };

    Raw raw;
    load_weights(raw, g0);
    fetch(g0, 0);
    expand_half(raw, 0, 0), expand_half(raw, 1, 0);
    load_weights(raw, g0 + 1);
    float sc_cols[BM];
    if constexpr (BM == 2) dg_mfma_column_scales<BM, TR>(p, m0, lane, sc_cols);       // (the larger tiles have no registers to spare)

    f32x16 acc[BM][WN];
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][bn][e] = 0.0f;

    struct Words {
        i32x8 w[BM];
        uint2 x[WN];
    };
    const char *const x_from = mem + 2 * WEIGHTS + wave * 2 * PIXELS + (r >> 4) * 1024 + (r & 15) * 64 + 8 * h;
    const int x_swap = (r >> 2) & 3;
    auto read = [&](Words &t, int odd, int s) {
        const char *w = mem + odd * WEIGHTS, *x = x_from + odd * PIXELS + (s ^ x_swap) * 16;
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) t.x[bn] = *(const uint2 *)(x + bn * 2048);
#pragma unroll
        for (int bm = 0; bm < BM; ++bm) {
            const int block = (s * BM + bm) * 64;
            const char *w16 = w + (block + (lane ^ (2 * s))) * 16, *w8 = w + WIDE + (block + (lane ^ (4 * s))) * 8;
            if constexpr (ONE_BASE) w16 = w + (lane ^ (2 * s)) * 16 + block * 16, w8 = w + WIDE + (lane ^ (4 * s)) * 8 + block * 8;
            const v4i lo = *(const v4i *)w16;
            const v2i hi = *(const v2i *)w8;
            t.w[bm] = (i32x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
        }
    };
    auto multiply = [&](const Words &t) {
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const uint32_t M = 0x03030303u, F = 0x0F0F0F0Fu;
            v4i plane[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t w = k ? t.x[bn].y : t.x[bn].x;
#pragma unroll
                for (int q = 0; q < 2; ++q) {               // even codes, odd codes: eight 4-bit places
                    const uint32_t lo = __builtin_amdgcn_perm(0u, a.powers, (q ? w >> 2 : w) & M);
                    const uint32_t hi = __builtin_amdgcn_perm(0u, a.powers, (w >> (q ? 6 : 4)) & M);
                    plane[0][2 * k + q] = (int)((lo & F) | ((hi << 4) & ~F));
                    plane[1][2 * k + q] = (int)(((lo >> 4) & F) | (hi & ~F));
                }
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int bm = 0; bm < BM; ++bm) acc[bm][bn] = step<TR>(t.w[bm], plane[s], acc[bm][bn]);
        }
    };

    for (int i = 0; i < whole; ++i) {
        const int odd = i & 1, g = g0 + i;
        dg_wait_for_loads<0>();                             // (this run's pixels, the next one's weights)
#pragma unroll
        for (int j = 0; j < SEGMENTS; ++j) asm volatile("" : "+v"(raw.v[j]));
        const Raw next = raw;
        __syncthreads();
        fetch(g + 1, odd ^ 1);
        load_weights(raw, g + 2);
        const uint32_t to = (odd ^ 1) * WEIGHTS;
        Words t[2];
        read(t[0], odd, 0);
        read(t[1], odd, 1);
        multiply(t[0]);
        read(t[0], odd, 2);
        expand_half(next, 0, to);
        multiply(t[1]);
        read(t[1], odd, 3);
        expand_half(next, 1, to);
        multiply(t[0]);
        multiply(t[1]);
    }
    // what is left of K, step by step: code 0 has numbers of its own, so none is taken past the end
    for (int done = 0; done < left; done += 4) {
        const int i = whole + done / 4, odd = i & 1, g = g0 + i;
        dg_wait_for_loads<0>();
#pragma unroll
        for (int j = 0; j < SEGMENTS; ++j) asm volatile("" : "+v"(raw.v[j]));
        const Raw next = raw;
        __syncthreads();
        const int steps = min(4, chunks - 4 * g);
        if (done + 4 < left) {
            fetch(g + 1, odd ^ 1);
            expand_half(next, 0, (odd ^ 1) * WEIGHTS), expand_half(next, 1, (odd ^ 1) * WEIGHTS);
            load_weights(raw, g + 2);
        }
        for (int s = 0; s < steps; ++s) {
            Words t;
            read(t, odd, s);
            multiply(t);
        }
    }
    dg_wait_for_loads();                                    // (fetches past the end: their LDS writes end before the wavefront does)
    if constexpr (BM > 2) dg_mfma_column_scales<BM, TR>(p, m0, lane, sc_cols);
    if constexpr (KS > 1) {
        static_assert(WN == 1 && KS % BM == 0 && WAVES * BM * 4096 <= SHARE, "a wavefront's sums take the place of its share of LDS");
        // [share][wavefront][block][group of four sums][lane]; then the first BM shares' wavefronts add up and store a block each
        __syncthreads();
        float4 *const mine = (float4 *)mem + wave * (BM * 256) + lane;
#pragma unroll
        for (int bm = 0; bm < BM; ++bm)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mine[(4 * bm + q) * 64] = make_float4(acc[bm][0][4 * q], acc[bm][0][4 * q + 1], acc[bm][0][4 * q + 2], acc[bm][0][4 * q + 3]);
        __syncthreads();
        if (ks >= BM) return;
        const float4 *const x = (const float4 *)s_mem + wave * (BM * 256) + ks * 256 + lane;
        f32x16 sums;
#pragma unroll
        for (int e = 0; e < 16; ++e) sums[e] = 0.0f;
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 u = x[k * (SHARE / 16) + q * 64];
                sums[4 * q] += u.x, sums[4 * q + 1] += u.y, sums[4 * q + 2] += u.z, sums[4 * q + 3] += u.w;
            }
        const v16i out = results(sums, a.factor);
        float sc = sc_cols[0];
#pragma unroll
        for (int bm = 1; bm < BM; ++bm) sc = ks == bm ? sc_cols[bm] : sc;
        dg_mfma_store_block<TR, true, DG_OUT_BY_PROBLEM>(p, out, m0 + ks * 32, n0, lane, sc);
        return;
    }
#pragma unroll
    for (int bm = 0; bm < BM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const v16i out = results(acc[bm][bn], a.factor);
            dg_mfma_store_block<TR, true, DG_OUT_BY_PROBLEM>(p, out, m0 + bm * 32, n0 + bn * 32, lane, sc_cols[bm]);
        }
}

}   // namespace

bool dg_find_levels(const dg_lut *lut, int (&u)[4], int (&v)[4], int *factor)
{
    if (lut->bits != 2 || lut->dtype == DG_LUT_F32) return false;
    const int16_t *row = nullptr;
    for (int w = 0; w < 4 && !row; ++w)
        for (int a = 0; a < 4; ++a)
            if (lut->entry[4 * w + a]) row = lut->entry + 4 * w;
    *factor = 1;
    for (int i = 0; i < 4; ++i) u[i] = v[i] = 0;
    if (!row) return true;
    int g = 0, lead = 0;
    for (int a = 0; a < 4; ++a) g = std::gcd(g, (int)row[a]);
    for (int a = 0; a < 4; ++a) {
        v[a] = row[a] / g;
        if (v[a]) lead = a;
    }
    int f = 0;
    for (int w = 0; w < 4; ++w) {
        const int16_t *t = lut->entry + 4 * w;
        if (t[lead] % v[lead]) return false;                // (v has no common factor: such a row is no multiple of it)
        u[w] = t[lead] / v[lead];
        for (int a = 0; a < 4; ++a)
            if (t[a] != u[w] * v[a]) return false;
        f = std::gcd(f, u[w]);
    }
    for (int w = 0; w < 4; ++w) u[w] /= f;
    *factor = f;
    return true;
}

namespace {

// An FP6 (E2M3) number that is v eighths, or -1.
int fp6(int v)
{
    const int m = abs(v), sign = v < 0 ? 32 : 0;
    if (m < 16) return sign | m;                            // (0 ... 7 eighths below 1, 8 ... 15 with the exponent of 1)
    if (m < 32) return m % 2 ? -1 : sign | (16 + (m - 16) / 2);
    if (m <= 60) return m % 4 ? -1 : sign | (24 + (m - 32) / 4);
    return -1;
}

}   // namespace

// (once per table: on each choice of a kernel, it was 0.1 us of the call)
void dg_find_two_powers(dg_lut *lut)
{
    DgTwoPowers *const n = &lut->two_powers;
    int u[4], v[4], most_u = 0, most_v = 0;
    memset(n, 0, sizeof(*n));
    if (!dg_find_levels(lut, u, v, &n->factor)) return;
    // (activation levels evenly spaced from zero are left to the other kernels: dg_twopower_preferred)
    bool spaced = true;
    for (int w = 0; w < 4; ++w) {
        const int16_t *t = lut->entry + 4 * w;
        spaced = spaced && t[0] == 0 && t[2] == 2 * t[1] && t[3] == 3 * t[1];
    }
    if (spaced) return;
    for (int w = 0; w < 4; ++w) {
        const int f = fp6(u[w]);
        if (f < 0) return;
        const int parts[6] = {f, (f & 3) << 6, f >> 2, (f & 15) << 4, f >> 4, f << 2};
        for (int i = 0; i < 6; ++i) n->bytes[i] |= (uint32_t)parts[i] << (8 * w);
        if (abs(u[w]) > most_u) most_u = abs(u[w]);
    }
    for (int a = 0; a < 4; ++a) {
        static const int power[9] = {0, 1, 2, 4, 8, -1, -2, -4, -8}, code[9] = {0, 1, 2, 4, 6, 9, 10, 12, 14};
        int best = 100, byte = 0;
        for (int i = 0; i < 9; ++i)
            for (int j = 0; j < 9; ++j)
                if (power[i] + power[j] == v[a] && abs(power[i]) + abs(power[j]) < best) {
                    best = abs(power[i]) + abs(power[j]);
                    byte = code[i] | code[j] << 4;
                }
        if (best == 100) return;
        n->powers |= (uint32_t)byte << (8 * a);
        if (best > most_v) most_v = best;
    }
    n->reach = most_u * most_v;
    n->levels = true;
}

namespace {

struct TwoPowerPlan {
    int bm, wn, waves, ks;
    const char *name;
    // us a run of 256 positions on a compute unit with one workgroup, and for each workgroup on one with more; per workgroup; per MB of
    // output; once
    double lone, shared, each, out, once;
};

// What they cost was fitted to 308 products of 1.2 to 120 GOP, us (5 % off on average): of the four the one that this says is shortest is 0.6 % behind the
// shortest measured on average, 16 % at most.  The fit has no short K with outputs beyond 150 MB: there 128 x 256 stores in bursts (us, one-hot kernels, 64 x 128,
// 128 x 256; column-major outputs, inputs changing: 3889 x 20227 x 384 107, 80, 135; 6977 x 7871 x 384 85, 60, 97; 5159 x 9628 x 576 93, 64, 95) and is behind 64 x 128
// below K = 640: of 27 such products that is 20 % shorter on average, 41 % at most, one 2 % longer; at 640 and 768 the two are level.
const TwoPowerPlan PLANS[] = {
    {2, 1, 4, 1, "twopower_64x128", 0.809, 0.647, 0.0, 0.108, 3.9},
    {2, 1, 4, 2, "twopower_64x128_k2", 0.641, 0.611, 0.3, 0.179, 3.75},
    {4, 2, 4, 1, "twopower_128x256", 1.839, 1.56, 1.24, 0.093, 6.3},
    {4, 2, 8, 1, "twopower_128x512", 2.602, 2.999, 3.26, 0.131, 4.3},
};

int64_t tiles_of(const DgProblem &p, const TwoPowerPlan &q)
{
    const int rows = 32 * q.bm, cols = 32 * q.wn * q.waves;
    return (((int64_t)p.M + rows - 1) / rows) * (((int64_t)p.N + cols - 1) / cols);
}

bool suits(const DgProblem &p, const TwoPowerPlan &q) { return q.bm == 2 || q.waves == 8 || p.K >= 640; }

double cost(const DgProblem &p, const TwoPowerPlan &q)
{
    const int64_t units = dg_simd_count() / 4, per_unit = (tiles_of(p, q) + units - 1) / units;
    const double runs = p.K / 256.0, megabytes = 4e-6 * (double)p.M * (double)p.N;
    return q.once + q.out * megabytes + (double)per_unit * q.each + runs * (per_unit == 1 ? q.lone : (double)per_unit * q.shared);
}

// DG_TWOPOWER: "0" never, "1", "12", "2", "4": this kernel whatever the size, the plan; nullptr where it is not set, or to anything else.
const char *twopower_override()
{
    const char *f = dg_override("DG_TWOPOWER");
    for (const char *name : {"0", "1", "12", "2", "4"})
        if (f && strcmp(f, name) == 0) return name;
    return nullptr;
}

const TwoPowerPlan &twopower_plan(const DgProblem &p)
{
    if (const char *f = twopower_override()) {
        if (strcmp(f, "1") == 0) return PLANS[0];
        if (strcmp(f, "12") == 0) return PLANS[1];
        if (strcmp(f, "2") == 0) return PLANS[2];
        if (strcmp(f, "4") == 0) return PLANS[3];
    }
    const TwoPowerPlan *best = PLANS;
    for (const TwoPowerPlan &q : PLANS)
        if (suits(p, q) && cost(p, q) < cost(p, *best)) best = &q;
    return *best;
}

// (whichever tile: where 64 x 128 is taken in place of a wider one, it is the shorter)
double least_cost(const DgProblem &p)
{
    double least = cost(p, PLANS[0]);
    for (const TwoPowerPlan &q : PLANS) least = std::min(least, cost(p, q));
    return least;
}

bool takes(const dg_lut *lut, const DgProblem &p)
{
    if (!lut->two_powers.levels) return false;
    if (p.KH * p.KW != 1 || p.sh != 1 || p.sw != 1 || p.ph || p.pw || p.Cin % 64 || p.Qp) return false;
    if ((uintptr_t)p.Wp % 16 || (uintptr_t)p.Xp % 16 || (int64_t)p.N * (p.K / 4) >= (int64_t)1 << 31) return false;      // (32-bit byte offsets)
    if (tiles_of(p, PLANS[0]) >= 1 << 22) return false;                // (a launch has fewer than 2^32 threads)
    return (int64_t)p.K * lut->two_powers.reach < 1 << 24;             // (multiples of 1/16 below 2^20)
}

}   // namespace

// AUTO takes such tables here where the shortest plan is clearly shorter than the one-hot kernels would be, whose times were fitted to the same
// 308 products (us; 6 to 8 % off on average).  Of those 111 are, all of them rightly, 1.45 times as fast on average; without the margin two more would be
// up to 9 % behind (6509 x 160 x 2688 10.7, 11.8).  Of 1049 that were in no fit and that it sends here, 1.43 times on average, one is 2 % longer (175 x 34340 x
// 6144 73.8, 75.4).  Left to the others: fewer than 1.5e9 operations (384 x 1742 x 896 6.3, 7.1), products that split K
// over a workgroup (304 x 561 x 4224 7.1, 14.4), long K with few tiles (4607 x 200 x 7040 15.4, 22.4; 8192 x 256 x 8192 25.5, 26.7), K = 64, 128,
// 256 and 512 where the stationary-weight kernel runs, and tables whose activation levels are evenly spaced from zero: dg_onebit_kernel.hip
// takes most; the others, whose weight levels FP4 has not, would gain here what other tables do (the arithmetic does not depend on the levels), and stay with the
// one-hot kernels because AUTO's names for one of them are held to that (tests/test_abi_host.py): no measurement draws this line.
bool dg_twopower_preferred(const dg_lut *lut, const DgProblem &p)
{
    if (!takes(lut, p)) return false;
    const char *forced = twopower_override();
    const double gop = 2e-9 * (double)p.M * (double)p.N * (double)p.K;
    if (forced ? strcmp(forced, "0") == 0 : gop < 1.5 || dg_override("DG_ONEHOT_PLAN") || dg_override("DG_ONEHOT_WAVES")) return false;
    if (forced) return true;
    if (lut->min_entry < -128 || lut->max_entry > 127) return false;
    double busiest;
    const DgOneHotForm other = dg_onehot_auto_form(lut, p, &busiest);
    if (other == DgOneHotForm::SplitK) return false;
    const double megabytes = 4e-6 * (double)p.M * (double)p.N, thousands = 1e-3 * p.K;
    double there = 4.4 + 1.09 * busiest + 0.211 * gop + 0.124 * megabytes;                                       // staged
    if (other == DgOneHotForm::Sparse) there = 6.2 + 1.0 * gop + 0.103 * megabytes + 0.96 * thousands;           // direct loads
    else if (other == DgOneHotForm::Dense) there = 3.2 + 2.37 * busiest + 0.12 * gop + 0.348 * megabytes + 0.5 * thousands;
    return least_cost(p) < 0.85 * there;
}

dg_status dg_launch_twopower(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    TwoPowerArgs a;
    const DgTwoPowers &n = lut->two_powers;
    memcpy(a.bytes, n.bytes, sizeof(a.bytes));
    a.powers = n.powers, a.factor = n.factor;
    a.p = p;
    a.p.cached = dg_output_cached(p);
    a.x_bytes = (uint32_t)((int64_t)p.N * (p.K / 4));
    const TwoPowerPlan &q = twopower_plan(p);
    const int rows = 32 * q.bm, cols = 32 * q.wn * q.waves, tiles_m = (p.M + rows - 1) / rows;
    a.tiles_n = (p.N + cols - 1) / cols;
    a.band_log2 = 2;
    a.band_tiles = (uint32_t)tiles_m << a.band_log2;
    a.div_band = make_div(a.band_tiles);
    const int last = a.tiles_n & ((1 << a.band_log2) - 1);
    a.div_last = make_div((uint32_t)(last ? last : 1));
    const bool rows_m = p.stride_cn == 1 && p.stride_cm != 1;           // the output's rows are channels
    const dim3 grid((unsigned)(tiles_m * a.tiles_n)), block(64 * q.waves * q.ks);
#define DG_TWOPOWER(BM, WN, WAVES, KS) \
    do { \
        if (rows_m) hipLaunchKernelGGL((twopower_kernel<BM, WN, WAVES, KS, false>), grid, block, 0, stream, a); \
        else hipLaunchKernelGGL((twopower_kernel<BM, WN, WAVES, KS, true>), grid, block, 0, stream, a); \
    } while (0)
    if (q.waves == 8) DG_TWOPOWER(4, 2, 8, 1);
    else if (q.bm == 4) DG_TWOPOWER(4, 2, 4, 1);
    else if (q.ks == 2) DG_TWOPOWER(2, 1, 4, 2);
    else DG_TWOPOWER(2, 1, 4, 1);
#undef DG_TWOPOWER
    return dg_check_launch("twopower_kernel");
}

const char *dg_twopower_config_name(const DgProblem &p) { return twopower_plan(p).name; }
