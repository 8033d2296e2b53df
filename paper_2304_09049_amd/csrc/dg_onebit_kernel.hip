// 2-bit tables that are two ONE-BIT lookups, on the FP4 matrix instruction.  Where
//
//   T[w][0] = 0,  T[w][2] = 2 T[w][1],  T[w][3] = T[w][1] + T[w][2]       (evenly spaced activation levels from zero)
//
// and the entries T[w][1], over a common factor, are among 0, 1, 2, 3, 4, 6, 8, 12 and their negatives (find_numbers; not -2, 5, 0, 1),
//
// a position adds the entry T[w][1] if bit 0 of its activation code is set, and the entry T[w][2] if bit 1 is.  As a contraction that is
// two places of the reduction per position, the entries on one side and single bits on the other, where the one-hot form of any table
// needs four (dg_onehot_kernel.h); and v_mfma_f32_32x32x64_f8f6f4 takes 64 places of 4-bit numbers in the 32 cycles in which the sparse int8
// instruction takes 16 positions of four.  So the matrix work is half of that kernel's, and no row of a table is read per position.
//
// Numbers: FP4 (E2M1) is 0, 0.5, 1, 1.5, 2, 3, 4, 6 and their negatives.  A code's bits are masked out where they lie in the packed word:
// the low bit at the bottom of a 4-bit place is 0.5, the high bit next to it is 1, of even codes as loaded, of odd ones after a shift by
// two -- five vector instructions for the operands of two instructions.  Weight code w is the number N[w] = T[w][1] / (2 f), the same for
// both bits, f the entries' common factor.  All products and sums are multiples of 1/4 below 2^22, hence exact in binary32 in any order
// (the host checks; takes), and 4 f times the sum is the integer result.
//
// A workgroup's four wavefronts share 64 channels, each with 32 WN pixels of its own.  A run is 256 positions of K, 64 bytes of a row: four
// neighbouring lanes fetch a row's, the pixels' straight to LDS (dg_lds_dma.h), one run ahead.  A 16-byte segment lies in one filter tap
// (Cin % 64 == 0); each lane works out its own segment's, and fetches zeros where the tap lies outside the image: nothing is masked later.
// The weights' 4-bit numbers are made once for the four wavefronts, 13 vector instructions per word of 16 codes, 16 bytes a thread, and
// handed over in LDS: one barrier per run.
//
// Bound by the matrix pipe at the clock it runs at on large layers (8192-cube: 22 ns per instruction and SIMD, where registers alone with
// random operands take 18.4 at 1.77 GHz, constant ones 13.5 at 2.4), by the start, the end and lone wavefronts' issue slots on those of a few
// microseconds: a run of the 64 x 128 tile takes 0.5 us then.  The staged sparse kernel, this one (packed codes, graph replays, us):
//   8192-cube 648, 356          56x56x256 -> 256 3x3 at batch 16 47.1, 30.6          28x28x512 -> 512 3x3 at batch 16 46.1, 29.9
//   28x28x128 -> 128 3x3 at batch 32 12.2, 8.6          28x28x256 -> 256 3x3 at batch 8 10.9, 7.9          3569 x 7478 x 704 81.5, 28.3
// (the last by its stores too: dg_output_cached).
#include "dg_lds_dma.h"
#include "dg_onehot_kernel.h"

#include <cstdlib>
#include <cstring>
#include <numeric>

namespace {

using namespace dgoh;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Sums to results: 4 f times a sum, which is whole once it is four times as large.
__device__ __forceinline__ v16i results(const f32x16 &sums, int32_t factor)
{
    v16i out;
#pragma unroll
    for (int e = 0; e < 16; ++e) out[e] = (int)(sums[e] * 4.0f);
    if (factor != 1) {                                      // (uniform; a 32-bit product is 16 cycles)
#pragma unroll
        for (int e = 0; e < 16; ++e) out[e] *= factor;
    }
    return out;
}

struct OneBitArgs {
    DgProblem p;
    uint32_t numbers;        // byte w: N[w] as FP4
    int32_t factor;          // f
    FastDiv div_ow, div_oh, div_kw, div_cpt, div_band;      // (div_cpt: by the 64-position segments of a filter tap)
    int32_t band_log2;
    uint32_t band_tiles, x_bytes;
    // the pixels before n_narrow in tiles of the kernel's width, `wide` workgroups, the rest in narrow ones
    uint32_t wide;
    int32_t tiles_n[2], n_narrow;
    FastDiv div_last[2];
};

__device__ __forceinline__ f32x16 fp4_step(const v4i &a, const v4i &b, f32x16 c)
{
    const i32x8 x = {a[0], a[1], a[2], a[3], 0, 0, 0, 0}, y = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, c, 4, 4, 0, 0, 0, 0);
}

// Where pixel n's row of bytes begins, and, with a filter window, which of its taps lie outside the image (bit t, tap t).  Without a window a
// pixel outside begins at byte 2^31, beyond any buffer taken here and still beyond it a row of K on.  (Its own offset with the top bit set is not:
// from just under 2^31 such a row wraps to the buffer's first bytes.)
template <bool TAPS>
__device__ __forceinline__ void place_pixel(const OneBitArgs &a, int n, int bytes_per_pixel, uint32_t &off0, uint32_t &outside)
{
    const DgProblem &p = a.p;
    const Column c = make_column(p, a.div_ow, a.div_oh, n, bytes_per_pixel, 0);
    const int h0 = max(0, -c.ih0), h1 = c.ok ? min(p.KH, p.H - c.ih0) : 0, c0 = max(0, -c.iw0), c1 = min(p.KW, p.W - c.iw0);
    off0 = (uint32_t)c.off0;
    if constexpr (TAPS) {
        const uint32_t columns = c1 > c0 ? (~0u >> (32 - (c1 - c0))) << c0 : 0u;
        uint32_t in = 0;
        for (int kh = 0; kh < p.KH; ++kh) in |= kh >= h0 && kh < h1 ? columns << (kh * p.KW) : 0u;
        outside = ~in;
    } else if (!(h1 > h0 && c1 > c0)) {
        off0 = 0x80000000u;
    }
    asm("" : "+v"(off0));                                   // (kept, not worked out again for each load)
}

// One tile: 64 channels, 4 x 32 WN pixels.
//
// KS = 2: eight wavefronts, two to a tile, each with half of K; their sums meet in LDS.  TAPS: a filter window.  TR: channels on the
// matrix instruction's columns (dg_mfma_tile.h).
// FIRST: a run's words are read from LDS before the next run's loads start, whose addresses are vector instructions in which the matrix pipe would wait.
// The loads then start later, which is the longer where they come from beyond the L2 caches or are the only thing to wait for (reads_first).
template <int WN, int KS, bool TAPS, bool TR, bool FIRST>
__device__ __forceinline__ void onebit_tile(const OneBitArgs &a, uint4 *s_mem, uint32_t block, uint32_t blocks, int part)
{
    constexpr int WEIGHTS = 8192;                           // bytes of a run's weight operands: 64 rows, 256 positions
    constexpr int PIXELS = WN * 2048;                       // bytes of a wavefront's pixels of a run
    constexpr int LOADS = 2 * WN;                           // loads of 16 rows each
    constexpr int BESIDE = WN > 1 ? 6 : 0;                  // other instructions between two matrix instructions (8192-cube 372 -> 356 us; 0: the compiler's order)
    constexpr int SHARE = 2 * WEIGHTS + 8 * PIXELS;         // bytes of the four wavefronts that walk one share of K
    const DgProblem &p = a.p;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5;
    const int w4 = wave & 3, ks = KS == 1 ? 0 : wave >> 2;
    int m_tile, n_tile;                                     // numbered in bands of 2^band_log2 pixel tiles, as in dg_sparse_staged_kernel.h
    {
        const uint32_t t = xcd_contiguous(block, blocks), band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n[part] - first);
        m_tile = (int)(width == 1 << a.band_log2 ? t_in >> a.band_log2 : fdiv(t_in, a.div_last[part]));
        n_tile = first + (int)t_in - m_tile * width;
    }
    const int m0 = m_tile * 64, n0 = (part ? a.n_narrow : 0) + (n_tile * 4 + w4) * (WN * 32);
    const int cq = p.Cin / 4, all_runs = (p.K + 255) / 256;
    // this share's runs g0 ... g1 - 1 of K and its chunks (64 positions); the shares walk equally many runs, past their ends as zeros
    const int g0 = KS == 1 ? 0 : all_runs * ks / KS, g1 = KS == 1 ? all_runs : all_runs * (ks + 1) / KS;
    const int runs = (all_runs + KS - 1) / KS, chunks = min(p.K / 64, 4 * g1);
    char *const mem = (char *)s_mem + ks * SHARE;

    // ---- weights: thread t of a share loads segment t % 4 of a run of row t / 4 (rows beyond M, bytes past the last row: zeros; past the end of
    // K: the next row's, which meet pixels of zero)
    const uint32_t row_bytes = (uint32_t)p.K / 4;
    const __amdgpu_buffer_rsrc_t w_buffer =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.Wp + (int64_t)m0 * row_bytes), 0, (int)(min(p.M - m0, 64) * row_bytes), 0x00020000);
    const int w_row = (threadIdx.x >> 2) & 63, w_seg = threadIdx.x & 3;
    const uint32_t w_ld = w_row * row_bytes + w_seg * 16;
    auto load_weights = [&](int g) { return (v4i)__builtin_amdgcn_raw_buffer_load_b128(w_buffer, w_ld + g * 64, 0, 0); };
    const uint32_t low = a.numbers, high = a.numbers << 4;
    // segment s of rows 32 b ... as [s][b][lane], lane (r, half) with its two words' numbers of even and odd codes; lanes exchanged so that a
    // thread's neighbours, which write the other segments, are on other banks
    char *const w_to = mem + ((2 * w_seg + (w_row >> 5)) * 64 + ((w_row & 31) ^ (2 * w_seg))) * 16;
    auto expand = [&](uint32_t word, int &even, int &odd) {
        even = (int)(__builtin_amdgcn_perm(0u, low, word & 0x03030303u) | __builtin_amdgcn_perm(0u, high, (word >> 4) & 0x03030303u));
        odd = (int)(__builtin_amdgcn_perm(0u, low, (word >> 2) & 0x03030303u) | __builtin_amdgcn_perm(0u, high, (word >> 6) & 0x03030303u));
    };
    auto expand_half = [&](const v4i &raw, int half, uint32_t buf) {
        v4i o;
        int e0, o0, e1, o1;
        expand((uint32_t)raw[2 * half], e0, o0);
        expand((uint32_t)raw[2 * half + 1], e1, o1);
        o[0] = e0, o[1] = o0, o[2] = e1, o[3] = o1;
        *(v4i *)(w_to + buf + half * 512) = o;
    };

    // ---- pixels: lane l of a load fetches segment (l % 4) ^ (row / 4 % 4) of row l / 4 of 16: a segment's 16 rows lie on 16 places of the banks
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);
    const int l_row = lane >> 2, l_seg = (lane & 3) ^ (lane >> 4);
    uint32_t off0[LOADS], outside[TAPS ? LOADS : 1];       // (place_pixel)
#pragma unroll
    for (int i = 0; i < LOADS; ++i) place_pixel<TAPS>(a, n0 + 16 * i + l_row, cq, off0[i], outside[TAPS ? i : 0]);
    const uint32_t x_lds = dg_lds_address(mem) + 2 * WEIGHTS + w4 * 2 * PIXELS;
    auto fetch = [&](int g, int odd) {
        const uint32_t dst = x_lds + odd * PIXELS;
        const int c = 4 * g + l_seg;
        const uint32_t dead = c < chunks ? 0u : 0x80000000u;
        if constexpr (TAPS) {
            const int tap = (int)fdiv((uint32_t)c, a.div_cpt), kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
            const uint32_t tap_off = (uint32_t)((kh * p.W + kw) * cq + (c - tap * (cq >> 4)) * 16);
            dg_for<LOADS>([&](auto i) {
                const uint32_t out = (outside[i] << ((31 - tap) & 31)) | dead;
                dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + tap_off) | (out & 0x80000000u), dst);
            });
        } else {
            dg_for<LOADS>([&](auto i) { dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + c * 16) | dead, dst); });
        }
    };

    v4i raw = load_weights(g0);
    fetch(g0, 0);
    expand_half(raw, 0, 0), expand_half(raw, 1, 0);
    raw = load_weights(g0 + 1);
    float sc_cols[2];
    dg_mfma_column_scales<2, TR>(p, m0, lane, sc_cols);

    f32x16 acc[2][WN];
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][bn][e] = 0.0f;

    struct Words {
        v4i w[2];
        uint2 x[WN];
    };
    const char *const x_from = mem + 2 * WEIGHTS + w4 * 2 * PIXELS + (r >> 4) * 1024 + (r & 15) * 64 + 8 * h;
    const int x_swap = (r >> 2) & 3;
    auto read = [&](Words &t, int odd, int s) {
        const char *w = mem + odd * WEIGHTS + (lane ^ (2 * s)) * 16, *x = x_from + odd * PIXELS + (s ^ x_swap) * 16;
#pragma unroll
        for (int bm = 0; bm < 2; ++bm) t.w[bm] = *(const v4i *)(w + (2 * s + bm) * 1024);
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) t.x[bn] = *(const uint2 *)(x + bn * 2048);
    };
    auto multiply = [&](const Words &t) {
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const uint32_t x0 = t.x[bn].x, x1 = t.x[bn].y, y0 = x0 >> 2, y1 = x1 >> 2;
#pragma unroll
            for (int bit = 0; bit < 2; ++bit) {
                const uint32_t M = bit ? 0x22222222u : 0x11111111u;
                const v4i x = {(int)(x0 & M), (int)(y0 & M), (int)(x1 & M), (int)(y1 & M)};
#pragma unroll
                for (int bm = 0; bm < 2; ++bm) {
                    acc[bm][bn] = TR ? fp4_step(x, t.w[bm], acc[bm][bn]) : fp4_step(t.w[bm], x, acc[bm][bn]);
                    if constexpr (BESIDE > 0) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x302, BESIDE, 0);
                    }
                }
            }
        }
    };

    for (int i = 0; i < runs; ++i) {
        const int odd = i & 1, g = g0 + i;
        dg_wait_for_loads<0>();                             // (this run's pixels, the next one's weights)
        asm volatile("" : "+v"(raw));
        const v4i next = raw;
        __syncthreads();
        Words t[2];
        if constexpr (FIRST) read(t[0], odd, 0), read(t[1], odd, 1);
        fetch(g + 1, odd ^ 1);
        raw = load_weights(g + 2);
        if constexpr (!FIRST) read(t[0], odd, 0), read(t[1], odd, 1);
        const uint32_t to = (odd ^ 1) * WEIGHTS;
        multiply(t[0]);
        read(t[0], odd, 2);
        expand_half(next, 0, to);
        multiply(t[1]);
        read(t[1], odd, 3);
        expand_half(next, 1, to);
        multiply(t[0]);
        multiply(t[1]);
    }
    dg_wait_for_loads();                                    // (fetches past the end: their LDS writes end before the wavefront does)

    if constexpr (KS > 1) {
        static_assert(KS == 2 && WN == 1, "a wavefront's sums take the place of its share of LDS");
        // [share][wavefront][block][group of four sums][lane]; then each wavefront of a pair adds up and stores one of their two blocks
        __syncthreads();
        float4 *const mine = (float4 *)s_mem + wave * 512 + lane;
#pragma unroll
        for (int bm = 0; bm < 2; ++bm)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mine[(4 * bm + q) * 64] = make_float4(acc[bm][0][4 * q], acc[bm][0][4 * q + 1], acc[bm][0][4 * q + 2], acc[bm][0][4 * q + 3]);
        __syncthreads();
        const float4 *const theirs = (const float4 *)s_mem + w4 * 512 + ks * 256 + lane;
        f32x16 sums;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = theirs[q * 64], y = theirs[2048 + q * 64];
            sums[4 * q] = x.x + y.x, sums[4 * q + 1] = x.y + y.y, sums[4 * q + 2] = x.z + y.z, sums[4 * q + 3] = x.w + y.w;
        }
        const v16i out = results(sums, a.factor);
        dg_mfma_store_block<TR, true, DG_OUT_BY_PROBLEM>(p, out, m0 + ks * 32, n0, lane, ks ? sc_cols[1] : sc_cols[0]);
        return;
    }
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const v16i out = results(acc[bm][bn], a.factor);
            dg_mfma_store_block<TR, true, DG_OUT_BY_PROBLEM>(p, out, m0 + bm * 32, n0 + bn * 32, lane, sc_cols[bm]);
        }
}

// WN = 2: the last workgroups may take narrow tiles (onebit_plan).
template <int WN, int KS, bool TAPS, bool TR, bool FIRST = (WN > 1 || !TR)>
__global__ void __launch_bounds__(256 * KS, 2)
onebit_kernel(OneBitArgs a)
{
    __shared__ uint4 s_mem[KS * (16384 + WN * 16384) / 16];
    dg_fetch_arguments<sizeof(a)>();
    if (WN == 2 && blockIdx.x >= a.wide) onebit_tile<1, 1, TAPS, TR, !TR>(a, s_mem, blockIdx.x - a.wide, gridDim.x - a.wide, 1);
    else onebit_tile<WN, KS, TAPS, TR, FIRST>(a, s_mem, blockIdx.x, WN == 2 ? a.wide : gridDim.x, 0);
}

// The same from activations that are still one code per byte (p.Xp = those bytes): 64 channels x 4 x 32 pixels, runs of 128 positions.  Nothing is
// packed: eight codes' bytes become an operand's word of 4-bit places by one shift and one bit-field insert, position i of the first
// four at the bottom of byte i, of the second four at its top, and the weights' numbers are made in that order.  Bound by its start and by
// lone wavefronts' issue slots, as the narrow tile on packed codes is: 112x112x64 -> 48 3x3 at batch 7 17.1 (sparse instruction, codes packed in
// registers) -> 10.8 us, 22 MB of codes and sums in 9 us.
template <bool TAPS>
__global__ void __launch_bounds__(256, 4)
onebit_codes_kernel(OneBitArgs a)
{
    constexpr int WEIGHTS = 4096, PIXELS = 4096;            // bytes of a run: the weights' numbers, a wavefront's pixels
    __shared__ uint4 s_mem[(2 * WEIGHTS + 8 * PIXELS) / 16];
    const DgProblem &p = a.p;
    dg_fetch_arguments<sizeof(a)>();
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 31, h = lane >> 5;
    int m_tile, n_tile;
    {
        const uint32_t t = xcd_contiguous(blockIdx.x, gridDim.x), band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n[0] - first);
        m_tile = (int)(width == 1 << a.band_log2 ? t_in >> a.band_log2 : fdiv(t_in, a.div_last[0]));
        n_tile = first + (int)t_in - m_tile * width;
    }
    const int m0 = m_tile * 64, n0 = (n_tile * 4 + w4) * 32;
    const int runs = (p.K + 127) / 128, pieces = p.K / 16;  // (a piece: 16 positions, a lane's 16 bytes)

    // ---- weights: thread t loads quarter t % 4 of a run's 32 bytes of row t / 4: word pair `half` of segment `seg`
    const uint32_t row_bytes = (uint32_t)p.K / 4;
    const __amdgpu_buffer_rsrc_t w_buffer =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.Wp + (int64_t)m0 * row_bytes), 0, (int)(min(p.M - m0, 64) * row_bytes), 0x00020000);
    const int w_row = threadIdx.x >> 2, w_quarter = threadIdx.x & 3;
    const uint32_t w_ld = w_row * row_bytes + w_quarter * 8;
    typedef int v2i __attribute__((ext_vector_type(2)));
    auto load_weights = [&](int g) { return (v2i)__builtin_amdgcn_raw_buffer_load_b64(w_buffer, w_ld + g * 32, 0, 0); };
    const uint32_t low = a.numbers, high = a.numbers << 4;
    char *const w_to = (char *)s_mem + (((w_quarter >> 1) * 2 + (w_row >> 5)) * 64 + (w_quarter & 1) * 32 + ((w_row & 31) ^ (2 * w_quarter))) * 16;
    auto spread = [](uint32_t word, int byte) {             // its four codes, one to a byte
        const uint32_t pairs = (((word >> (8 * byte)) & 255u) * 0x1001u) & 0x000F000Fu;
        return (pairs << 6 | pairs) & 0x03030303u;
    };
    auto expand = [&](const v2i &raw, uint32_t buf) {
        v4i o;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t word = (uint32_t)raw[q / 2];
            o[q] = (int)(__builtin_amdgcn_perm(0u, low, spread(word, 2 * (q & 1))) | __builtin_amdgcn_perm(0u, high, spread(word, 2 * (q & 1) + 1)));
        }
        *(v4i *)(w_to + buf) = o;
    };

    // ---- pixels: lane l of a load fetches piece (l % 8) ^ (row % 8) of row l / 8 of eight
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);
    const int l_row = lane >> 3, l_piece = (lane & 7) ^ l_row;
    uint32_t off0[4], outside[TAPS ? 4 : 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) place_pixel<TAPS>(a, n0 + 8 * i + l_row, p.Cin, off0[i], outside[TAPS ? i : 0]);
    const uint32_t x_lds = dg_lds_address(s_mem) + 2 * WEIGHTS + w4 * 2 * PIXELS;
    auto fetch = [&](int g, int odd) {
        const uint32_t dst = x_lds + odd * PIXELS;
        const int c = 8 * g + l_piece;
        const uint32_t dead = c < pieces ? 0u : 0x80000000u;
        if constexpr (TAPS) {
            const int tap = (int)fdiv((uint32_t)c, a.div_cpt), kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
            const uint32_t tap_off = (uint32_t)((kh * p.W + kw) * p.Cin + (c - tap * (p.Cin >> 4)) * 16);
            dg_for<4>([&](auto i) {
                const uint32_t out = (outside[i] << ((31 - tap) & 31)) | dead;
                dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + tap_off) | (out & 0x80000000u), dst);
            });
        } else {
            dg_for<4>([&](auto i) { dg_load16_to_lds<i * 1024>(x_buffer, (off0[i] + c * 16) | dead, dst); });
        }
    };

    v2i raw = load_weights(0);
    fetch(0, 0);
    expand(raw, 0);
    raw = load_weights(1);
    float sc_cols[2];
    dg_mfma_column_scales<2, true>(p, m0, lane, sc_cols);
    f32x16 acc[2];
#pragma unroll
    for (int bm = 0; bm < 2; ++bm)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[bm][e] = 0.0f;

    const char *const x_from = (const char *)s_mem + 2 * WEIGHTS + w4 * 2 * PIXELS + r * 128;
    for (int g = 0; g < runs; ++g) {
        const int odd = g & 1;
        dg_wait_for_loads<0>();                             // (this run's pixels, the next one's weights)
        asm volatile("" : "+v"(raw));
        const v2i next = raw;
        __syncthreads();
        fetch(g + 1, odd ^ 1);
        raw = load_weights(g + 2);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            v4i w[2];
            uint4 x[2];
#pragma unroll
            for (int bm = 0; bm < 2; ++bm)
                w[bm] = *(const v4i *)((const char *)s_mem + odd * WEIGHTS + ((2 * s + bm) * 64 + h * 32 + (r ^ (2 * (2 * s + h)))) * 16);
#pragma unroll
            for (int e = 0; e < 2; ++e) x[e] = *(const uint4 *)(x_from + odd * PIXELS + ((4 * s + 2 * h + e) ^ (r & 7)) * 16);
            uint32_t t[4];
            auto merge = [](uint32_t first, uint32_t second) { return (first & 0x0F0F0F0Fu) | ((second << 4) & 0xF0F0F0F0u); };
            t[0] = merge(x[0].x, x[0].y), t[1] = merge(x[0].z, x[0].w), t[2] = merge(x[1].x, x[1].y), t[3] = merge(x[1].z, x[1].w);
#pragma unroll
            for (int bit = 0; bit < 2; ++bit) {
                const uint32_t M = bit ? 0x22222222u : 0x11111111u;
                const v4i o = {(int)(t[0] & M), (int)(t[1] & M), (int)(t[2] & M), (int)(t[3] & M)};
#pragma unroll
                for (int bm = 0; bm < 2; ++bm) acc[bm] = fp4_step(o, w[bm], acc[bm]);
            }
            if (s == 0) expand(next, (odd ^ 1) * WEIGHTS);
        }
    }
    dg_wait_for_loads();                                    // (fetches past the end: their LDS writes end before the wavefront does)
#pragma unroll
    for (int bm = 0; bm < 2; ++bm) {
        const v16i out = results(acc[bm], a.factor);
        dg_mfma_store_block<true, true, DG_OUT_BY_PROBLEM>(p, out, m0 + bm * 32, n0, lane, sc_cols[bm]);
    }
}

// N[w] and f of a table of the form above, if its N are FP4 numbers; *largest: the largest |T[w][1]| / f.
bool find_numbers(const dg_lut *lut, uint32_t *numbers, int32_t *factor, int32_t *largest)
{
    if (lut->bits != 2 || lut->dtype == DG_LUT_F32) return false;
    int f = 0;
    for (int w = 0; w < 4; ++w) {
        const int16_t *row = lut->entry + 4 * w;
        if (row[0] != 0 || row[2] != 2 * row[1] || row[3] != row[1] + row[2]) return false;
        f = std::gcd(f, (int)row[1]);
    }
    if (f == 0) f = 1;
    *numbers = 0, *factor = f, *largest = 0;
    for (int w = 0; w < 4; ++w) {
        static const int doubled[8] = {0, 1, 2, 3, 4, 6, 8, 12};
        const int t = lut->entry[4 * w + 1] / f, magnitude = abs(t);
        int code = 0;
        while (code < 8 && doubled[code] != magnitude) ++code;
        if (code == 8) return false;
        *numbers |= (uint32_t)(code | (t < 0 ? 8 : 0)) << (8 * w);
        if (magnitude > *largest) *largest = magnitude;
    }
    return true;
}

bool takes(const dg_lut *lut, const DgProblem &p)
{
    uint32_t numbers;
    int32_t factor, largest;
    if (!find_numbers(lut, &numbers, &factor, &largest)) return false;
    if ((int64_t)p.K * 3 * largest >= 1 << 24) return false;           // (multiples of 1/4 below 2^22)
    if (p.Cin % 64 != 0 || p.KH * p.KW > 32 || (uintptr_t)p.Wp % 16 != 0 || (uintptr_t)p.Xp % 16 != 0) return false;
    if ((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * (p.Cin / 4) >= (int64_t)1 << 31) return false;      // (32-bit byte offsets)
    return (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 127) / 128) < 1 << 24;           // (a launch has fewer than 2^32 threads)
}

struct OneBitPlan {
    int wn, ks;
    int64_t columns;         // of wide tiles, the pixel tiles; what is left takes narrow ones
};

// The output's rows are channels: a GEMM with n contiguous.
bool rows_are_channels(const DgProblem &p) { return p.stride_cn == 1 && p.stride_cm != 1 && p.KH * p.KW == 1 && !p.Qp; }
// (they are pixels, of 32-bit sums)
bool rows_are_pixels(const DgProblem &p) { return !rows_are_channels(p) && !p.Qp; }

int64_t tiles_of(const DgProblem &p, int wn) { return (((int64_t)p.M + 63) / 64) * (((int64_t)p.N + 128 * wn - 1) / (128 * wn)); }

bool large_output(const DgProblem &p) { return tiles_of(p, 1) >= 13 * (dg_simd_count() / 4); }

// DG_ONEBIT: 0 never, 1, 2, 4 this kernel with WN so large, 12 with WN = 1 and KS = 2, 21 with WN = 2 and half of the pixels in narrow tiles, whatever the
// size; -1 where it is not set, or to anything else.
int onebit_override()
{
    static const char *const names[] = {"0", "1", "2", "4", "12", "21"};
    if (const char *f = dg_override("DG_ONEBIT"))
        for (const char *name : names)
            if (strcmp(f, name) == 0) return atoi(name);
    return -1;
}

OneBitPlan onebit_plan(const DgProblem &p)
{
    const int64_t units = dg_simd_count() / 4, runs = ((int64_t)p.K + 255) / 256, t1 = tiles_of(p, 1), tm = ((int64_t)p.M + 63) / 64;
    auto columns = [&](int wn) { return ((int64_t)p.N + 128 * wn - 1) / (128 * wn); };
    const int forced = onebit_override();
    if (forced == 21) return OneBitPlan{2, 1, columns(2) / 2};
    if (forced == 12) return OneBitPlan{1, 2, columns(1)};
    if (forced > 0) return OneBitPlan{forced, 1, columns(forced)};
    // A tile twice (four times) as wide costs 1.82 (3.55) times as much per run on a busy compute unit, so the plan is the one that
    // leaves the busiest the least: 112x112x128 -> 128 3x3 at batch 10 (1960, 980, 490 tiles) 24.2, 22.7, 25.0 us; 56x56x128 -> 112 3x3 at batch 26
    // (1274, 638) 16.7, 18.1; 56x56x256 -> 112 3x3 at batch 28 (1372, 686) 28.3, 25.2.  Few runs do not pay for a wide tile's longer end:
    // 6648 x 2359 x 832 22.1, 25.2, but on large outputs (8192 x 8192 x 320 by rows 58.0, 51.3; 224x224x64 -> 64 3x3 at batch 16 re-quantising 48.5, 47.2), if
    // they are not short rows, pixel by pixel, after one or two runs: 1000 x 200000 x 192 174, 255; 2048 x 16384 x 192 27.1, 34.0, x 384 28.9, 36.9.
    // The widest wants nine: 1986 x 7254 x 6272 83.7, 78.3, 74.9, 8192-cube 402, 367, 356, 112x112x128 -> 120 3x3 at batch 25 60.2, 54.7,
    // 59.4.  Rounds of wide tiles that would leave compute units idle in the last one end in narrow tiles: 56x56x256 -> 256 3x3 at batch 16
    // (784 tiles on 256 compute units) 35.1, as 768 and 32 narrow ones 31.1; 112x112x128 -> 112 3x3 at batch 18 42.4, 39.4; 3200 x 6400 x 2304
    // 42.9, 40.4.  Not the widest: the first as 256 of 512 pixels and 544 narrow ones was 3 us longer than that.
    if (t1 <= units) return OneBitPlan{1, runs >= 8 ? 2 : 1, columns(1)};
    OneBitPlan q = {1, 1, columns(1)};
    double best = (double)((t1 + units - 1) / units);
    auto consider = [&](int wn, double cost) {
        const int64_t all = tm * columns(wn), whole = all / units * units / tm;          // columns that fill whole rounds
        const double c = all <= units ? 4.1 : cost * ((all + units - 1) / units);          // (a lone wavefront per SIMD is slower: WN = 4)
        if (c < best) best = c, q = OneBitPlan{wn, 1, columns(wn)};
        const int64_t rest = p.N - whole * 128 * wn;
        if (wn == 2 && whole > 0 && rest > 0) {
            const double mixed = cost * (all / units) + (double)((tm * ((rest + 127) / 128) + units - 1) / units);
            if (mixed < best) best = mixed, q = OneBitPlan{wn, 1, whole};
        }
    };
    if (t1 > 2 * units && (runs >= 5 || (large_output(p) && !(runs <= 2 && rows_are_pixels(p) && p.M < 4000)))) {
        consider(2, 1.82);
        if (runs >= 9) consider(4, 3.55);
    }
    return q;
}

}   // namespace

// AUTO takes such tables here where the tiles are many and full enough.  In us on packed codes, the one-hot kernels and this one:
//  - from 130 tiles of 64 x 128 in place of the staged kernel: 14x14x256 -> 744 3x3 at batch 7 (132 tiles) 11.4, 9.2.  With fewer, long K is walked by
//    too few wavefronts, 7x7x1152 -> 1680 3x3 at batch 10 (108 tiles, 41 runs) 18.5, 20.8, and short K is level, 28x28x128 -> 128 3x3 at batch
//    8 (98, 5 runs) 6.1, 6.2, re-quantising between other layers 0.4 longer here; some between are shorter here and not taken, 28x28x256 -> 64 3x3
//    at batch 8 (98, 9 runs) 8.3, 7.9, 134 x 4171 x 4480 (99) 15.3, 11.3: the line counts tiles, not time.
//  - from 35 in place of direct loads: 738 x 360 x 5568 (36) 15.3, 12.2; 28x28x320 -> 512 3x3 (56) 8.9, 8.9; from 60 in place of the split-K kernel, which
//    makes one round of long K there: 28x28x512 -> 144 3x3 at batch 2 (39) 7.6, 10.7, 1416 x 135 x 6912 (46) 12.1, 13.5, but 80 x 4112 x 2880 (66) 9.7, 8.1,
//    85 x 4336 x 5184 (68) 17.5, 11.6 (entries beyond int8 from 35: 2240 x 65 x 5568 13.0, 12.0).
//  - from 1.5e9 operations: smaller products were not measured.
//  - from 65 columns, half of the tile: 4096 x 64 x 5568 (64) 9.3, 12.0, x 65 columns 15.1, 12.1; 8192 x 32 x 8192 (128) 11.4, 15.9; 11008 x 64 x 4096 (172) 9.9,
//    10.2, x 65 13.9, 10.4.  (Entries beyond int8 cost the others twice as much: 8192 x 32 x 8192 13.8, 15.7, but 11008 x 32 x 4096 13.8, 9.9.)
//  - from 33 rows, half of the tile, in place of staged tiles of 32 x 128: 56x56x128 -> 28 3x3 at batch 32 12.0, 13.0, -> 36 17.8, 14.5; 56x56x384 -> 16 at
//    batch 16 13.0, 14.6.  The other tiles are behind there too: 112x112x64 -> 16 3x3 at batch 16 26.4, 14.5, 32 x 30000 x 2048 10.2, 7.2 -- but for direct
//    loads of one or two runs where the output's rows are channels: 32 x 262144 x 320 11.1, 12.0 (x 448 13.7, 12.8), 24 x 262144 x 192 9.1, 10.7.
//  - not with one run of K and long rows, pixel by pixel, of a large output: 4096 x 20480 x 192 60.1, 65.2 (1000 x 100000 x 192 113, 89).
bool dg_onebit_preferred(const dg_lut *lut, const DgProblem &p)
{
    const int forced = onebit_override();
    const int64_t t1 = tiles_of(p, 1);
    if (forced >= 0 ? forced == 0 : t1 < 35 || 2.0 * (double)p.M * (double)p.N * (double)p.K < 1.5e9) return false;
    if (!takes(lut, p)) return false;
    if (forced > 0) return true;
    if (dg_override("DG_ONEHOT_PLAN") || dg_override("DG_ONEHOT_WAVES")) return false;
    const DgOneHotForm other = dg_onehot_auto_form(lut, p);
    const bool int8 = lut->min_entry >= -128 && lut->max_entry <= 127;
    if (p.N <= 64 && (int8 || t1 < 130)) return false;
    if (p.M <= 32 && (other == DgOneHotForm::Staged32x128 || (other == DgOneHotForm::Sparse && p.K <= 320 && rows_are_channels(p)))) return false;
    if (p.M >= 4000 && p.K <= 256 && int8 && rows_are_pixels(p) && large_output(p)) return false;
    if (other == DgOneHotForm::SplitK && int8) return t1 >= 60;
    return t1 >= 130 || other < DgOneHotForm::Staged;
}

namespace {

void fill(const dg_lut *lut, const DgProblem &p, const OneBitPlan &q, OneBitArgs *args)
{
    OneBitArgs &a = *args;
    int32_t largest;
    a.p = p;
    a.p.cached = dg_output_cached(p);
    find_numbers(lut, &a.numbers, &a.factor, &largest);
    a.div_ow = make_div((uint32_t)p.OW), a.div_oh = make_div((uint32_t)p.OH), a.div_kw = make_div((uint32_t)p.KW);
    a.div_cpt = make_div((uint32_t)(p.Cin / 64));
    const int64_t tiles_m = ((int64_t)p.M + 63) / 64, rest = p.N - q.columns * 128 * q.wn;
    a.n_narrow = (int32_t)(rest > 0 ? q.columns * 128 * q.wn : 0);
    a.tiles_n[0] = (int32_t)q.columns, a.tiles_n[1] = (int32_t)(rest > 0 ? (rest + 127) / 128 : 0);
    a.wide = (uint32_t)(tiles_m * a.tiles_n[0]);
    a.band_log2 = 2;
    a.band_tiles = (uint32_t)tiles_m << a.band_log2;
    a.div_band = make_div(a.band_tiles);
    for (int i = 0; i < 2; ++i) {
        const int last = a.tiles_n[i] & ((1 << a.band_log2) - 1);
        a.div_last[i] = make_div((uint32_t)(last ? last : 1));
    }
    a.x_bytes = (uint32_t)((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * (p.Cin / 4));
}

}   // namespace

// Which forms read a run's words first (FIRST), us, loads first and words first, inputs changing (780 calls, each form's mean in brackets):
//  - wide tiles, a little (0.992)
//  - 64 x 128: where the output's rows are channels (0.993); else the loads go first, 1201 x 7199 x 384 column-major 12.8, 13.9, 14x16x448 -> 1120 5x5 at
//    batch 9 37.1, 38.5 (1.007)
//  - with K shared by two: where there is a filter window, 28x28x256 -> 256 3x3 at batch 8 8.2, 7.9 (0.964); without one the loads are all that a run waits
//    for, 729 x 486 x 7488 15.9, 17.5 (1.029).  Nor with more weights and activations than an XCD's L2 cache holds: of 400 such layers the 298 with less than
//    4 MB are 0.961, one 4 % longer; those from 7 MB 1.034, 28x28x2496 -> 896 5x5 at batch 2 100, 117.
static bool reads_first(const DgProblem &p)
{
    const int64_t codes = (int64_t)p.M * p.K + (int64_t)(p.N / (p.OH * p.OW)) * p.H * p.W * p.Cin;
    return codes <= (int64_t)1 << 24;
}

dg_status dg_launch_onebit(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    const OneBitPlan q = onebit_plan(p);
    OneBitArgs a;
    fill(lut, p, q, &a);
    const dim3 grid(a.wide + (unsigned)((((int64_t)p.M + 63) / 64) * a.tiles_n[1]));
    const bool taps = p.KH * p.KW > 1, rows_m = rows_are_channels(p);
#define DG_ONEBIT_FORM(WN, KS, ...) hipLaunchKernelGGL((onebit_kernel<WN, KS, __VA_ARGS__>), grid, dim3(256 * KS), 0, stream, a)
#define DG_ONEBIT(WN) \
    do { \
        if (rows_m) DG_ONEBIT_FORM(WN, 1, false, false); \
        else if (taps) DG_ONEBIT_FORM(WN, 1, true, true); \
        else DG_ONEBIT_FORM(WN, 1, false, true); \
    } while (0)
    if (q.wn == 4) DG_ONEBIT(4);
    else if (q.wn == 2) DG_ONEBIT(2);
    else if (q.ks == 1) DG_ONEBIT(1);
    else if (rows_m) DG_ONEBIT_FORM(1, 2, false, false, false);
    else if (!taps) DG_ONEBIT_FORM(1, 2, false, true, false);
    else if (reads_first(p)) DG_ONEBIT_FORM(1, 2, true, true, true);
    else DG_ONEBIT_FORM(1, 2, true, true, false);
#undef DG_ONEBIT
#undef DG_ONEBIT_FORM
    return dg_check_launch("onebit_kernel");
}

const char *dg_onebit_config_name(const DgProblem &p)
{
    const OneBitPlan q = onebit_plan(p);
    if (q.wn == 4) return "onebit_64x512";
    if (q.wn == 2) return p.N > q.columns * 256 ? "onebit_64x256_64x128" : "onebit_64x256";
    return q.ks == 2 ? "onebit_64x128_k2" : "onebit_64x128";
}

// p.Xp: codes one per byte.  AUTO, where it would run a one-hot kernel that packs while loading: from 140 tiles of 64 x 128 up, us, that kernel, this one
// (inputs changing from pass to pass): 56x56x64 -> 40 3x3 stride 2 at batch 25 (154 tiles) 10.8, 8.7; 112x112x64 -> 48 3x3 at batch 7 (686) 17.1, 10.8;
// 14x14x192 -> 280 3x3 at batch 23 (180) 14.6, 13.5; of 290 such calls one layer behind, 56x56x192 -> 64 at batch 32 10.5, 10.8; below, 112x112x128 -> 64
// 3x3 (98) 8.3, 9.3; 28x28x320 -> 88 3x3 stride 2 at batch 31 (96) 15.2, 17.9.  Not for 64 columns or fewer, half of the tile: 9000 x 17 x 192 (141)
// 3.9, 5.6, 9000 x 32 x 1024 6.5, 7.9, 12000 x 64 x 576 6.2, 6.6, x 65 8.6, 6.6.
// Nor in place of the kernel with stationary weights, whose loads run ahead of its stores.  It is behind that on 56x56x256 -> 64 at batch 32, 8.6, 8.2 with the
// input in L2, but 9.4, 10.4 from the last-level cache, on 56x56x128 -> 40 at batch 16 6.1, 7.3, 56x56x256 -> 64 at batch 8 5.5, 5.8; of 17 such
// layers 13 are shorter here, 28x28x256 -> 256 at batch 16 7.0, 6.1, 56x56x256 -> 200 at batch 16 20.5, 18.1: a rule between them is not made yet.
// DG_ONEBIT_CODES: 0 never, 1 wherever a kernel packs while loading.
bool dg_onebit_codes_preferred(const dg_lut *lut, const DgProblem &p, bool stationary)
{
    const char *f = dg_override("DG_ONEBIT_CODES");
    if (f ? atoi(f) == 0 : stationary || tiles_of(p, 1) < 140 || p.N <= 64) return false;
    if (!f && (dg_override("DG_ONEHOT_PLAN") || dg_override("DG_ONEHOT_WAVES") || dg_override("DG_ONEHOT_CODES_TILED"))) return false;
    if (!takes(lut, p) || p.stride_cm != 1 || p.Qp) return false;
    return (int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * p.Cin < (int64_t)1 << 31;                   // (32-bit byte offsets)
}

// The same in place of the packing kernel and this one on packed codes.  A tile of 64 x 128 reads a pixel's codes once per filter tap and 64 channels, four
// times the bytes of packed ones: where that is five times or less (1x1 layers of up to 320 channels, 3x3 ones of stride 2 and up to 128) the spared
// launch and pass are more.  us, both kernels, this one, inputs changing from pass to pass: 28x28x512 -> 208 at batch 32 13.6, 10.9; 112x112x128 -> 96 3x3
// stride 2 at batch 14 18.1, 14.6; 56x56x128 -> 120 3x3 stride 2 at batch 15 (184 tiles) 13.0, 11.9.  Not 56x56x128 -> 64 3x3 at batch 12 (nine times) 9.3, 9.7;
// nor with fewer tiles (12 at stride 2, 148, 9.1, 9.4), with more than 1152 positions (56x56x256 -> 96 3x3 stride 2 at batch 23 16.2, 18.5) or K that two
// halves of a workgroup share (54x64x256 -> 88 3x3 stride 2 at batch 6 10.3, 14.3).
// Nor where several tiles of channels read the codes in many rounds of tiles, which wide tiles of packed codes make fewer of and whose codes fall out of the
// caches: two such tiles of channels read them up to six rounds, more up to four (56x56x512 -> 296 at batch 10, 1225 tiles, 18.5, 20.8; 112x112x384 -> 260 at
// batch 14, 6860, 62, 86; 112x112x576 -> 112 at batch 19, 3724, 59, 65; one tile of channels is ahead whatever the rounds).  Of 852 layers within
// the other lines 319 are within these, 1.35 times as fast on average, none longer; 84 of the others were 2 to 39 % longer.
// DG_ONEBIT_CODES: 2 wherever this kernel would be run on packed codes.
bool dg_onebit_codes_spare_packing(const dg_lut *lut, const DgProblem &p)
{
    if (lut->bits != 2 || p.stride_cm != 1 || p.Qp) return false;
    const char *f = dg_override("DG_ONEBIT_CODES");
    if (f || onebit_override() >= 0) {
        if (!f || strcmp(f, "2") != 0) return false;
    } else {
        if (p.K > 1152) return false;
        const int64_t t1 = tiles_of(p, 1), tm = ((int64_t)p.M + 63) / 64, units = dg_simd_count() / 4, reads = p.KH * p.KW * tm, strides = (int64_t)p.sh * p.sw;
        if (t1 < 150 || reads > 5 * strides || (tm > 1 && t1 > (reads <= 2 * strides ? 6 : 4) * units) || onebit_plan(p).ks != 1) return false;
    }
    return takes(lut, p) && (int64_t)(p.N / (p.OH * p.OW)) * p.H * p.W * p.Cin < (int64_t)1 << 31;
}

dg_status dg_launch_onebit_codes(const dg_lut *lut, const DgProblem &p, hipStream_t stream)
{
    OneBitArgs a;
    fill(lut, p, OneBitPlan{1, 1, ((int64_t)p.N + 127) / 128}, &a);
    a.div_cpt = make_div((uint32_t)(p.Cin / 16));
    a.x_bytes = (uint32_t)((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * p.Cin);
    const dim3 grid(a.wide);
    if (p.KH * p.KW > 1) hipLaunchKernelGGL((onebit_codes_kernel<true>), grid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((onebit_codes_kernel<false>), grid, dim3(256), 0, stream, a);
    return dg_check_launch("onebit_codes_kernel");
}
