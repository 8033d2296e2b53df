// Layers by the codes' BITS, on the int8 matrix instruction, from unpacked codes (planes_packed_kernel: packed 2-bit ones), for tables whose entries
// are sums of what single bits add:
//
//   3- and 4-bit codes, T[w][a] = a T[w][1] (evenly spaced activation levels from zero): bit b of the code adds T[w][1] 2^b
//   2-bit codes, T[w][a] = f u[w] v[a] with v[0] = 0 and entries beyond int8: the low bit adds f u[w] v[1], the high bit f u[w] v[2], and
//   both together f u[w] (v[3] - v[1] - v[2]), three sums per output, each of the u[w] whose bits are set, put together at the end
//
// A code per byte is the operand as it is: masked with 0x01010101 << b it holds bit b's 0 or 2^b, one vector instruction per four codes
// and bit.  The other operand is a byte per weight code, T[w][1] or u[w].  Three or four products per position on the int8 instruction, 32
// positions of it in 32 cycles, are as many cycles as (3-bit codes and entries beyond int8: three quarters of) what the packed codes take on the
// sparse instruction as two lookups or in two planes; every product is by 0 or a power of two.  What is saved is the launch of the
// packing kernel, the rows of tables read per position, and their fill.
//
// Eight wavefronts: 64 channels, PXW blocks of 32 pixels, K in KS = 8 / PXW shares.  The wavefronts of a share take its runs of 128 positions
// together, as in dg_onebit_kernel.hip: pixels' pieces straight to LDS, one run ahead, each lane working out its own piece's filter tap
// and reading zeros outside the image (code 0 adds nothing); the channels' bytes made once for the share's wavefronts, one barrier a run.
#include "dg_lds_dma.h"
#include "dg_onehot_kernel.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>

namespace {

using namespace dgoh;

struct PlanesArgs {
    DgProblem p;
    uint32_t bytes;          // 2-bit codes: byte w, u[w]
    int32_t low, high, both; // 2-bit codes: what the three sums count for; others: T[w][1] = low w + high
    FastDiv div_ow, div_oh, div_kw, div_cpt, div_band, div_last;      // (div_cpt: by the 16-position pieces of a filter tap)
    int32_t tiles_n, band_log2;
    uint32_t band_tiles, x_bytes;
};

// Where the rows of bytes of pixels n, n + 8, n + 16 and n + 24 begin, and which of their taps lie outside the image (bit t, tap t): all, beyond the
// last pixel.
__device__ __forceinline__ void place_pixels(const PlanesArgs &a, int n, uint32_t (&off0)[4], uint32_t (&outside)[4])
{
    const DgProblem &p = a.p;
    uint32_t columns[4];
    int h0[4], h1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const Column c = make_column(p, a.div_ow, a.div_oh, n + 8 * i, p.Cin, 0);
        const int c0 = max(0, -c.iw0), c1 = min(p.KW, p.W - c.iw0);
        h0[i] = -c.ih0, h1[i] = c.ok ? p.H - c.ih0 : 0;
        off0[i] = (uint32_t)c.off0;
        columns[i] = c1 > c0 ? (~0u >> (32 - (c1 - c0))) << c0 : 0u;
        outside[i] = ~0u;
    }
    for (int kh = 0; kh < p.KH; ++kh)
#pragma unroll
        for (int i = 0; i < 4; ++i) outside[i] &= ~(kh >= h0[i] && kh < h1[i] ? columns[i] << (kh * p.KW) : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) asm("" : "+v"(off0[i]));    // (kept, not worked out again for each load)
}

template <int BITS, int PXW>
__global__ void __launch_bounds__(512, 2)
planes_kernel(PlanesArgs a)
{
    constexpr int KS = 8 / PXW, SUMS = BITS == 2 ? 3 : 1;
    constexpr int WEIGHTS = 8192, PIXELS = 4096;            // bytes of a run: a share's weights, a wavefront's pixels
    constexpr int SHARE = 2 * WEIGHTS + 2 * PXW * PIXELS;
    constexpr int UNITS = 4 / PXW, WORDS = BITS == 2 ? 2 : 4;          // quarters of a row's run that a thread expands, their packed words
    __shared__ uint4 s_mem[KS * SHARE / 16];
    __shared__ alignas(16) int32_t s_codes[BITS == 2 ? 4 : 256];       // [share][wavefront][pixel]: sums of codes
    const DgProblem &p = a.p;
    dg_fetch_arguments<sizeof(a)>();
    const int lane = threadIdx.x & 63, all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5;
    const int wave = all % PXW, ks = all / PXW;
    int m_tile, n_tile;                                     // numbered in bands of 2^band_log2 pixel tiles, as in dg_sparse_staged_kernel.h
    {
        const uint32_t t = xcd_contiguous(blockIdx.x, gridDim.x), band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n - first);
        m_tile = (int)(width == 1 << a.band_log2 ? t_in >> a.band_log2 : fdiv(t_in, a.div_last));
        n_tile = first + (int)t_in - m_tile * width;
    }
    const int m0 = m_tile * 64, n0 = (n_tile * PXW + wave) * 32;
    // this share's runs g0 ... g1 - 1 of K; the shares walk equally many, past their ends as zeros
    const int all_runs = (p.K + 127) / 128, g0 = all_runs * ks / KS, g1 = all_runs * (ks + 1) / KS, runs = (all_runs + KS - 1) / KS;
    const int pieces = min(p.K / 16, 8 * g1);
    char *const mem = (char *)s_mem + ks * SHARE;

    // ---- weights: quarter q of a run's positions of a row is a thread's unit (rows beyond M, bytes past the last row: zeros; past the end of K:
    // the next row's, which meet pixels of zero)
    constexpr int RUN_BYTES = BITS == 2 ? 32 : 64;
    const uint32_t row_bytes = (uint32_t)p.K / (BITS == 2 ? 4 : 2);
    const __amdgpu_buffer_rsrc_t w_buffer =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.Wp + (int64_t)m0 * row_bytes), 0, (int)(min(p.M - m0, 64) * row_bytes), 0x00020000);
    const int w_row = (threadIdx.x % (64 * PXW)) >> 2, quarter = threadIdx.x & 3;
    const uint32_t w_ld = w_row * row_bytes + quarter * (RUN_BYTES / 4);
    typedef int v2i __attribute__((ext_vector_type(2)));
    struct Raw {
        uint32_t v[UNITS][WORDS];
    };
    auto load_weights = [&](Raw &raw, int g) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const uint32_t at = w_ld + i * (16 * PXW) * row_bytes + g * RUN_BYTES;
            if constexpr (BITS == 2) {
                const v2i t = (v2i)__builtin_amdgcn_raw_buffer_load_b64(w_buffer, at, 0, 0);
                raw.v[i][0] = (uint32_t)t[0], raw.v[i][1] = (uint32_t)t[1];
            } else {
                const v4i t = (v4i)__builtin_amdgcn_raw_buffer_load_b128(w_buffer, at, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) raw.v[i][j] = (uint32_t)t[j];
            }
        }
    };
    // step i's bytes of rows 32 b ... as [i][b][lane], lane (r, half) with positions 64 half + 16 i ... of the run; lanes exchanged so that a
    // thread's neighbours, which write the other quarters, are on other banks
    auto expand = [&](const Raw &raw, uint32_t buf) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int row = w_row + i * (16 * PXW);
            char *const to = mem + buf + ((2 * (quarter & 1)) * 2 + (row >> 5)) * 1024 + ((quarter >> 1) * 32 + ((row & 31) ^ (2 * quarter))) * 16;
#pragma unroll
            for (int s = 0; s < 2; ++s) {                   // 16 positions each
                v4i o;
                if constexpr (BITS == 2) {
                    const uint32_t w = raw.v[i][s];
#pragma unroll
                    for (int d = 0; d < 4; ++d) {           // (four codes of a byte, one to a byte)
                        const uint32_t pairs = (((w >> (8 * d)) & 255u) * 0x1001u) & 0x000F000Fu;
                        o[d] = (int)__builtin_amdgcn_perm(0u, a.bytes, (pairs << 6 | pairs) & 0x03030303u);
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const uint32_t w = raw.v[i][2 * s + d], even = w & 0x0F0F0F0Fu, odd = (w >> 4) & 0x0F0F0F0Fu;
                        o[2 * d] = (int)__builtin_amdgcn_perm(odd, even, 0x05010400u), o[2 * d + 1] = (int)__builtin_amdgcn_perm(odd, even, 0x07030602u);
                    }
                }
                *(v4i *)(to + s * 2048) = o;
            }
        }
    };

    Raw raw;
    load_weights(raw, g0);                                  // (before the pixels' places are worked out)

    // ---- pixels: lane l of a load fetches piece (l % 8) ^ (row % 8) of row l / 8 of eight
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);
    const int l_row = lane >> 3, l_piece = (lane & 7) ^ l_row;
    uint32_t off0[4], outside[4];
    place_pixels(a, n0 + l_row, off0, outside);
    const uint32_t x_lds = dg_lds_address(mem) + 2 * WEIGHTS + wave * 2 * PIXELS;
    auto fetch = [&](int g, int odd) {
        const uint32_t dst = x_lds + odd * PIXELS;
        const int c = 8 * g + l_piece;
        const uint32_t dead = c < pieces ? 0u : 0x80000000u;
        const int tap = (int)fdiv((uint32_t)c, a.div_cpt), kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
        const uint32_t tap_off = (uint32_t)((kh * p.W + kw) * p.Cin + (c - tap * (p.Cin >> 4)) * 16);
        dg_for<4>([&](auto i) {
            const uint32_t out = (outside[i] << ((31 - tap) & 31)) | dead;
            dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + tap_off) | (out & 0x80000000u), dst);
        });
    };

    fetch(g0, 0);
    expand(raw, 0);
    load_weights(raw, g0 + 1);
    float sc_cols[2];
    dg_mfma_column_scales<2, true>(p, m0, lane, sc_cols);
    v16i acc[2][SUMS];
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int k = 0; k < SUMS; ++k)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][k][e] = 0;

    int codes_sum = 0;                                      // BITS > 2: of the codes that this lane has multiplied
    const char *const x_from = mem + 2 * WEIGHTS + wave * 2 * PIXELS + r * 128;
    for (int i = 0; i < runs; ++i) {
        const int odd = i & 1, g = g0 + i;
        dg_wait_for_loads<0>();                             // (this run's pixels, the next one's weights)
#pragma unroll
        for (int j = 0; j < UNITS; ++j)
#pragma unroll
            for (int k = 0; k < WORDS; ++k) asm volatile("" : "+v"(raw.v[j][k]));
        const Raw next = raw;
        __syncthreads();
        v4i xs[4], ws[4][2];
        auto read = [&](int s) {
            xs[s] = *(const v4i *)(x_from + odd * PIXELS + ((4 * h + s) ^ (r & 7)) * 16);
#pragma unroll
            for (int bm = 0; bm < 2; ++bm)
                ws[s][bm] = *(const v4i *)(mem + odd * WEIGHTS + (2 * s + bm) * 1024 + (h * 32 + (r ^ (2 * (2 * h + (s >> 1))))) * 16);
        };
        read(0), read(1), read(2), read(3);                 // (before the next run's addresses are worked out: 28x28x256 -> 256 3x3 at batch 8
        fetch(g + 1, odd ^ 1);                              // beyond int8 15.0 -> 14.1 us, 28x28x128 -> 128 3-bit 8.22 -> 8.13)
        load_weights(raw, g + 2);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const v4i x = xs[s], (&w)[2] = ws[s];
#pragma unroll
            for (int d = 0; d < (BITS == 2 ? 0 : 4); ++d)
                codes_sum = (int)__builtin_amdgcn_udot4((uint32_t)x[d] & ((1u << BITS) - 1) * 0x01010101u, 0x01010101u, (uint32_t)codes_sum, false);
#pragma unroll
            for (int k = 0; k < (BITS == 2 ? 3 : BITS); ++k) {
                v4i plane;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t c = (uint32_t)x[d];
                    plane[d] = (int)(BITS == 2 && k == 2 ? c & (c >> 1) & 0x01010101u : c & (0x01010101u << k));
                }
#pragma unroll
                for (int bm = 0; bm < 2; ++bm)
                    acc[bm][SUMS == 3 ? k : 0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(plane, w[bm], acc[bm][SUMS == 3 ? k : 0], 0, 0, 0);
            }
            if (s == 1) expand(next, (odd ^ 1) * WEIGHTS);
        }
    }
    dg_wait_for_loads();                                    // (fetches past the end: their LDS writes end before the wavefront does)

    if constexpr (BITS == 2) {                              // (sums below 2^23: takes; what they count for below 2^17, three entries of 16 bits)
#pragma unroll
        for (int bm = 0; bm < 2; ++bm)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc[bm][0][e] = __mul24(acc[bm][0][e], a.low) + __mul24(acc[bm][1][e] >> 1, a.high) + __mul24(acc[bm][2][e], a.both);
    }
    if constexpr (BITS != 2) {
        codes_sum += __shfl_xor(codes_sum, 32);
        if (h == 0) s_codes[all * 32 + r] = codes_sum;
    }
    // [share][wavefront][block][group of four sums][lane]; then each wavefront adds up and stores 1 / KS of its pixels' two blocks
    __syncthreads();
    int4 *const mine = (int4 *)s_mem + all * 512 + lane;
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v16i &t = acc[bm][0];
            mine[(4 * bm + q) * 64] = make_int4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
        }
    __syncthreads();
    constexpr int NQ = 8 / KS;
    const int first = ks * NQ, bm = first >> 2, q0 = first & 3;
    const int4 *const from = (const int4 *)s_mem + wave * 512 + first * 64 + lane;
    dg_v4i sums[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        sums[q] = (dg_v4i){0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int4 t = from[k * (PXW * 512) + q * 64];
            sums[q][0] += t.x, sums[q][1] += t.y, sums[q][2] += t.z, sums[q][3] += t.w;
        }
        if constexpr (BITS != 2) {
            dg_v4i codes = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KS; ++k) codes += *(const dg_v4i *)(s_codes + (k * PXW + wave) * 32 + 8 * (q0 + q) + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) sums[q][e] = __mul24(sums[q][e], a.low) + __mul24(codes[e], a.high);
        }
    }
    dg_mfma_store_quads<NQ>(p, sums, q0, m0 + bm * 32, n0, lane, bm ? sc_cols[1] : sc_cols[0]);
}

// 2-bit codes that are packed already, for larger layers: four wavefronts, 64 channels and 32 pixels each, K in runs of 128 positions.  A lane's
// half of a run is four words, the bits of whose codes are 20 vector instructions per 16 codes and three planes: 5 beside each matrix instruction, three
// wavefronts to a SIMD.  Three matrix instructions per 32 positions and block where two planes on the sparse one take four, and no rows of a
// table: 56x56x256 -> 256 3x3 at batch 16 94 -> 70 us, 2646 instructions on every SIMD at 26 ns (20 with random bytes in registers and nothing else).
__global__ void __launch_bounds__(256, 3)
planes_packed_kernel(PlanesArgs a)
{
    constexpr int WEIGHTS = 8192, PIXELS = 1024;            // bytes of a run: the weights, a wavefront's pixels
    __shared__ uint4 s_mem[(2 * WEIGHTS + 8 * PIXELS) / 16];
    const DgProblem &p = a.p;
    dg_fetch_arguments<sizeof(a)>();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5;
    int m_tile, n_tile;
    {
        const uint32_t t = xcd_contiguous(blockIdx.x, gridDim.x), band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n - first);
        m_tile = (int)(width == 1 << a.band_log2 ? t_in >> a.band_log2 : fdiv(t_in, a.div_last));
        n_tile = first + (int)t_in - m_tile * width;
    }
    const int m0 = m_tile * 64, n0 = (n_tile * 4 + wave) * 32;
    const int runs = (p.K + 127) / 128, pieces = p.K / 64;  // (a piece: 64 positions, a lane's 16 bytes)
    char *const mem = (char *)s_mem;

    // ---- weights, as above
    const uint32_t row_bytes = (uint32_t)p.K / 4;
    const __amdgpu_buffer_rsrc_t w_buffer =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.Wp + (int64_t)m0 * row_bytes), 0, (int)(min(p.M - m0, 64) * row_bytes), 0x00020000);
    const int w_row = threadIdx.x >> 2, quarter = threadIdx.x & 3;
    const uint32_t w_ld = w_row * row_bytes + quarter * 8;
    typedef int v2i __attribute__((ext_vector_type(2)));
    auto load_weights = [&](int g) { return (v2i)__builtin_amdgcn_raw_buffer_load_b64(w_buffer, w_ld + g * 32, 0, 0); };
    char *const w_to = mem + ((2 * (quarter & 1)) * 2 + (w_row >> 5)) * 1024 + ((quarter >> 1) * 32 + ((w_row & 31) ^ (2 * quarter))) * 16;
    auto expand = [&](const v2i &raw, int s, uint32_t buf) {
        v4i o;
#pragma unroll
        for (int d = 0; d < 4; ++d) o[d] = (int)__builtin_amdgcn_perm(0u, a.bytes, ((uint32_t)raw[s] >> (2 * d)) & 0x03030303u);
        *(v4i *)(w_to + buf + s * 2048) = o;
    };

    // ---- pixels: lane l of the load fetches piece l % 2 of row l / 2
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);
    uint32_t off0, outside;
    {
        const Column c = make_column(p, a.div_ow, a.div_oh, n0 + (lane >> 1), p.Cin / 4, 0);
        const int h0 = -c.ih0, h1 = c.ok ? p.H - c.ih0 : 0, c0 = max(0, -c.iw0), c1 = min(p.KW, p.W - c.iw0);
        const uint32_t columns = c1 > c0 ? (~0u >> (32 - (c1 - c0))) << c0 : 0u;
        off0 = (uint32_t)c.off0, outside = ~0u;
        for (int kh = 0; kh < p.KH; ++kh) outside &= ~(kh >= h0 && kh < h1 ? columns << (kh * p.KW) : 0u);
        asm("" : "+v"(off0));
    }
    const uint32_t x_lds = dg_lds_address(mem) + 2 * WEIGHTS + wave * 2 * PIXELS;
    auto fetch = [&](int g, int odd) {
        const int c = 2 * g + (lane & 1);
        const int tap = (int)fdiv((uint32_t)c, a.div_cpt), kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
        const uint32_t tap_off = (uint32_t)((kh * p.W + kw) * (p.Cin >> 2) + (c - tap * (p.Cin >> 6)) * 16);
        const uint32_t out = (outside << ((31 - tap) & 31)) | (c < pieces ? 0u : 0x80000000u);
        dg_load16_to_lds<0>(x_buffer, (off0 + tap_off) | (out & 0x80000000u), x_lds + odd * PIXELS);
    };

    v2i raw = load_weights(0);
    fetch(0, 0);
    expand(raw, 0, 0), expand(raw, 1, 0);
    raw = load_weights(1);
    float sc_cols[2];
    dg_mfma_column_scales<2, true>(p, m0, lane, sc_cols);
    v16i acc[2][3];
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][k][e] = 0;
    for (int g = 0; g < runs; ++g) {
        const int odd = g & 1;
        dg_wait_for_loads<0>();                             // (this run's pixels, the next one's weights)
        asm volatile("" : "+v"(raw));
        const v2i next = raw;
        __syncthreads();
        const v4i x = *(const v4i *)(mem + 2 * WEIGHTS + wave * 2 * PIXELS + odd * PIXELS + (2 * r + h) * 16);
        v4i ws[4][2];
        auto read = [&](int s) {
#pragma unroll
            for (int bm = 0; bm < 2; ++bm)
                ws[s][bm] = *(const v4i *)(mem + odd * WEIGHTS + (2 * s + bm) * 1024 + (h * 32 + (r ^ (2 * (2 * h + (s >> 1))))) * 16);
        };
        read(0), read(1);
        fetch(g + 1, odd ^ 1);
        raw = load_weights(g + 2);
        read(2), read(3);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const v4i (&w)[2] = ws[s];
            const uint32_t c = (uint32_t)x[s], both = c & (c >> 1);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                v4i plane;
#pragma unroll
                for (int d = 0; d < 4; ++d) plane[d] = (int)(((k == 2 ? both : c) >> (2 * d)) & (k == 1 ? 0x02020202u : 0x01010101u));
#pragma unroll
                for (int bm = 0; bm < 2; ++bm) acc[bm][k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(plane, w[bm], acc[bm][k], 0, 0, 0);
            }
            if (s & 1) expand(next, s >> 1, (odd ^ 1) * WEIGHTS);
        }
    }
    dg_wait_for_loads();                                    // (fetches past the end: their LDS writes end before the wavefront does)
#pragma unroll
    for (int bm = 0; bm < 2; ++bm) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            acc[bm][0][e] = __mul24(acc[bm][0][e], a.low) + __mul24(acc[bm][1][e] >> 1, a.high) + __mul24(acc[bm][2][e], a.both);
        dg_mfma_store_block<true, true, DG_OUT_BY_PROBLEM>(p, acc[bm][0], m0 + bm * 32, n0, lane, sc_cols[bm]);
    }
}

template <int PXW>
int64_t tiles_of(const DgProblem &p) { return (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 32 * PXW - 1) / (32 * PXW)); }

// Codes of the activations.
int64_t codes_of(const DgProblem &p) { return (int64_t)(p.N / (p.OH * p.OW)) * p.H * p.W * p.Cin; }

// DG_PLANES: 0 never, 2, 4 this kernel with so many pixel blocks whatever the size; -1 where it is not set, or to anything else.
int planes_override()
{
    const char *f = dg_override("DG_PLANES");
    if (f && (strcmp(f, "0") == 0 || strcmp(f, "2") == 0 || strcmp(f, "4") == 0)) return f[0] - '0';
    return -1;
}

// us: once, a round of workgroups (one to a compute unit), a run of one, an MB of output.  Fitted to 222 layers for 2-bit codes, to 700 whichever kernel is the
// shorter for 3- and 4-bit ones (3 to 4 % off on average, 19 % at most).
template <int PXW>
double cost(const DgProblem &p, int bits)
{
    static const double fits[3][2][4] = {{{1.6, 3.2, 1.28, 0.165}, {2.0, 2.7, 1.06, 0.18}},
                                         {{1.97, 2.28, 1.22, 0.24}, {2.17, 2.22, 1.04, 0.21}},
                                         {{2.04, 2.15, 1.39, 0.25}, {2.32, 2.04, 1.25, 0.22}}};
    const double *const f = fits[bits - 2][PXW == 4];
    const int64_t units = dg_simd_count() / 4, rounds = (tiles_of<PXW>(p) + units - 1) / units;
    const int runs = ((p.K + 127) / 128 + 8 / PXW - 1) / (8 / PXW);
    return f[0] + (double)rounds * (f[1] + f[2] * runs) + f[3] * 4e-6 * (double)p.M * (double)p.N;
}

int pixel_blocks(const DgProblem &p, int bits)
{
    const int forced = planes_override();
    return forced > 0 ? forced : (cost<2>(p, bits) < cost<4>(p, bits) ? 2 : 4);
}

// (what most calls fail by first)
bool takes(const dg_lut *lut, const DgProblem &p)
{
    if (!lut->bit_sums.sums || p.stride_cm != 1 || p.Cin % 64 != 0 || p.Qp) return false;
    if (p.KH * p.KW > 32 || (uintptr_t)p.Wp % 16 != 0 || (uintptr_t)p.Xp % 16 != 0) return false;
    if ((int64_t)p.K * lut->bit_sums.most >= 1 << 23) return false;    // (24-bit products)
    if (codes_of(p) >= (int64_t)1 << 31) return false;                 // (32-bit byte offsets)
    return tiles_of<2>(p) < 1 << 22;                                   // (a launch has fewer than 2^32 threads)
}

}   // namespace

// The kernel on packed codes, us, fitted to 240 layers of 0.15 to 90 GOP (6 % off on average): once, a run of one, two or more workgroups of a compute
// unit, a workgroup, an MB of output.
static double packed_cost(const DgProblem &p)
{
    const int64_t units = dg_simd_count() / 4, n = (tiles_of<4>(p) + units - 1) / units;
    const double runs = (double)(((int64_t)p.K + 127) / 128), per_run = n == 1 ? 0.611 : (n == 2 ? 0.439 : 0.465);
    return 3.3 + (double)n * (0.575 + per_run * runs) + 0.065 * 4e-6 * (double)p.M * (double)p.N;
}

// (K = 64 is half of a run, and beyond 64 MB its output's stores are all: us, two planes and this one, 56x56x64 -> 1480 stride 2 at batch 26 27.0, 27.9; 28x27x64 ->
// 1968 at batch 23 34.9, 35.9; with less 56x56x64 -> 804 at batch 4 14.8, 12.7; of 27 such layers 4 % shorter on average, seven up to 3 % longer, all of those with more)
static bool packed_pays(const DgProblem &p, double two_planes)
{
    return packed_cost(p) < 0.87 * two_planes && (p.K > 64 || 4e-6 * (double)p.M * (double)p.N <= 64.0);
}

static bool beyond_int8(const dg_lut *lut) { return lut->min_entry < -128 || lut->max_entry > 127; }

static bool other_overrides()
{
    if (!dg_overrides_enabled()) return false;
    for (const char *name : {"DG_ONEHOT_PLAN", "DG_ONEHOT_WAVES", "DG_NIBBLES", "DG_STAGED_2P", "DG_STAGED_2P_PLAN"})
        if (dg_override(name)) return true;
    return false;
}

// (once per table)
void dg_find_bit_sums(dg_lut *lut)
{
    DgBitSums &n = lut->bit_sums;
    memset(&n, 0, sizeof(n));
    if (lut->bits == 2) {
        int v[4], u[4], factor;
        if (!dg_find_levels(lut, u, v, &factor) || v[0] != 0) return;
        n.low = factor * v[1], n.high = factor * v[2], n.both = factor * (v[3] - v[1] - v[2]);
        for (int w = 0; w < 4; ++w) {
            if (u[w] < -128 || u[w] > 127) return;
            n.bytes |= (uint32_t)(uint8_t)u[w] << (8 * w);
            if (abs(u[w]) > n.most) n.most = abs(u[w]);
        }
    } else {
        const int codes = 1 << lut->bits;
        n.high = lut->entry[1], n.low = lut->entry[codes + 1] - n.high, n.most = (codes - 1) * (codes - 1);
        for (int w = 0; w < codes; ++w)
            for (int c = 0; c < codes; ++c)
                if (lut->entry[codes * w + c] != c * (n.high + n.low * w)) return;
    }
    n.sums = true;
}

// AUTO, where a layer would be packed first: 3- and 4-bit codes that run as two lookups, 2-bit tables with entries beyond int8.  From codes, us, the two
// kernels and this one (graph replays): 28x28x128 -> 128 3x3 at batch 8, 4-bit 10.1, 8.8, 3-bit 10.1, 8.2; 28x28x256 -> 256 3x3 at batch 8, entries
// beyond int8 18.4, 14.1; 112x112x128 -> 112 3x3 stride 2 at batch 5, 3-bit 16.2, 10.4.  It is behind with many rounds of tiles, whose codes are read
// again for every 64 channels (112x112x64 -> 112 3x3 at batch 4, 4-bit 19.9, 29.9; with more than four rounds the fit is not asked:
// 116x116x64 -> 104 3x3 at batch 13, beyond int8, 72, 79), on long K with few tiles (14x14x384 -> 360 3x3 at batch 2, beyond int8, 10.1, 14.2), and with 3-
// and 4-bit codes where the split-K kernel has few blocks to a compute unit and a share here one run (315 x 128 -> 1564, 4-bit, 5.8, 6.7; 36x36x64 -> 352
// stride 2 at batch 17, 4-bit, 8.2, 10.0; 715 x 384 -> 252, 4-bit, 5.7, 6.0): the fit has to say more there.  Of the 1400 layers of 3- and 4-bit codes to which it was
// fitted, inputs changing from pass to pass, it sends 305 here, 1.28 times as fast on average, none longer; of 1427 others that it sends here, 1.27 times on
// average, two are 3 % longer; of 602 of entries beyond int8, 1.37 times, none.
bool dg_planes_codes_preferred(const dg_lut *lut, const DgProblem &p)
{
    if (!takes(lut, p)) return false;
    const int forced = planes_override();
    if (forced >= 0) return forced > 0;
    if (tiles_of<4>(p) > dg_simd_count() || other_overrides()) return false;
    const double here = std::min(cost<2>(p, lut->bits), cost<4>(p, lut->bits)), codes = 1e-6 * (double)codes_of(p);
    if (lut->bits != 2) {
        const double margin = p.K > 512 ? 0.95 : (p.K > 256 || p.sh * p.sw == 1 ? 0.92 : 0.88);
        return here < margin * dg_onehot_nibble_time(lut, p, codes);
    }
    if (!beyond_int8(lut)) return false;
    const double packing = 1.9 + 0.08 * codes, two_planes = dg_onehot_two_plane_time(lut, p);
    if (here >= 0.94 * (two_planes + packing)) return false;
    if (packed_pays(p, two_planes) && here >= 0.94 * (packed_cost(p) + packing)) return false;
    return !dg_onebit_preferred(lut, p);
}

// AUTO, 2-bit tables with entries beyond int8 on packed codes, where the fit says a seventh less than the kernels in two planes (6 to 12 % off on average): us, those
// and this one, 56x56x256 -> 256 3x3 at batch 16 94, 70; 116x116x64 -> 104 3x3 at batch 13 66, 41; 28x28x256 -> 256 3x3 at batch 16 26.9, 21.0;
// 112x112x128 -> 40 3x3 at batch 4 16.5, 12.6; not 28x28x128 -> 128 3x3 at batch 8 8.3, 9.2; 14x14x384 -> 360 3x3 at batch 2 8.2, 20.4; 34x34x128 -> 352 at batch
// 4 4.9, 5.5.  Of the 240 layers to which it was fitted 70 go here, 1.38 times as fast on average, none slower; 230 others that it sent here were 1.41 times as fast,
// two of them 3 % longer, with K = 64 (packed_pays).
// DG_PLANES_PACKED: "0" never, "1" whatever the size.
bool dg_planes_preferred(const dg_lut *lut, const DgProblem &p)
{
    if (lut->bits != 2 || !beyond_int8(lut) || !takes(lut, p)) return false;
    const char *f = dg_override("DG_PLANES_PACKED");
    if (f && strcmp(f, "0") == 0) return false;
    if (f && strcmp(f, "1") == 0) return true;
    return !other_overrides() && packed_pays(p, dg_onehot_two_plane_time(lut, p));
}

namespace {

void fill(const dg_lut *lut, const DgProblem &p, int pxw, int piece, int bytes_per_pixel, PlanesArgs *args)
{
    PlanesArgs &a = *args;
    const DgBitSums &n = lut->bit_sums;
    a.bytes = n.bytes, a.low = n.low, a.high = n.high, a.both = n.both;
    a.p = p;
    a.p.cached = dg_output_cached(p);
    a.div_ow = make_div((uint32_t)p.OW), a.div_oh = make_div((uint32_t)p.OH), a.div_kw = make_div((uint32_t)p.KW);
    a.div_cpt = make_div((uint32_t)(p.Cin / piece));
    a.tiles_n = (p.N + 32 * pxw - 1) / (32 * pxw);
    a.band_log2 = 2;
    a.band_tiles = (uint32_t)((p.M + 63) / 64) << a.band_log2;
    a.div_band = make_div(a.band_tiles);
    const int last = a.tiles_n & ((1 << a.band_log2) - 1);
    a.div_last = make_div((uint32_t)(last ? last : 1));
    a.x_bytes = (uint32_t)((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * bytes_per_pixel);
}

}   // namespace

dg_status dg_launch_planes(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    PlanesArgs a;
    fill(lut, p, 4, 64, p.Cin / 4, &a);
    hipLaunchKernelGGL(planes_packed_kernel, dim3((unsigned)(((p.M + 63) / 64) * a.tiles_n)), dim3(256), 0, stream, a);
    return dg_check_launch("planes_packed_kernel");
}

dg_status dg_launch_planes_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    PlanesArgs a;
    const int pxw = pixel_blocks(p, lut->bits);
    fill(lut, p, pxw, 16, p.Cin, &a);
    const dim3 grid((unsigned)(((p.M + 63) / 64) * a.tiles_n));
#define DG_PLANES(BITS) \
    do { \
        if (pxw == 4) hipLaunchKernelGGL((planes_kernel<BITS, 4>), grid, dim3(512), 0, stream, a); \
        else hipLaunchKernelGGL((planes_kernel<BITS, 2>), grid, dim3(512), 0, stream, a); \
    } while (0)
    if (lut->bits == 2) DG_PLANES(2);
    else if (lut->bits == 3) DG_PLANES(3);
    else DG_PLANES(4);
#undef DG_PLANES
    return dg_check_launch("planes_kernel");
}

const char *dg_planes_codes_config_name(const dg_lut *lut, const DgProblem &p)
{
    return pixel_blocks(p, lut->bits) == 4 ? "codes_planes_64x128_k2" : "codes_planes_64x64_k4";
}
