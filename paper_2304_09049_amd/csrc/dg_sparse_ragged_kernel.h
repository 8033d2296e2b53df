// 2-bit table kernel on the sparse matrix instruction (operand layout, index register and row-pair table as in
// dg_onehot_kernel.h, BITS = 20) for layers whose filter taps are NOT whole 32-position groups: Cin % 32 != 0, Cin >= 16.
//
// A lane half's operand words must come from one filter tap each, and a tap is L = Cin / 4 packed bytes, which need be no
// multiple of anything.  A lane half therefore walks SEGMENTS, each inside one tap, in WINDOWS of CH words that never leave
// the segment: the last window of a segment ends where the segment ends and overlaps the one before it, and what the
// overlap would count twice is taken out by kept bytes of zero.  (A packed byte is four codes and four codes are one dword
// of kept bytes, so every byte count can be masked.)  Nothing is read beyond a tap, hence nothing beyond the tensors, and
// no load needs padding, clamping or shifting; loads may be unaligned, which the hardware allows.
//   in pairs:  half h walks tap 2i + h as one segment (an odd tap count leaves half 1 of the last pair without a tap)
//   in halves: half 0 walks the first, half 1 the last Ls = 4 ceil(L / 8) bytes of tap i (in the 2 Ls - L bytes that both
//              hold, half 1's are masked)
// whichever takes fewer words.  (Words that are masked in both halves are multiplied all the same: a branch around them cost
// more than the words, since it kept the loads of the next window from being issued between this one's instructions.)
//
// Bound by issue slots and by how few wavefronts such small layers have, not by the matrix pipe.  So S wavefronts
// of a workgroup share one tile and split the windows of K among them, their sums meeting in LDS (exact in any order).  Registers are
// kept to 128: with 134 the second workgroup of a compute unit, of five wavefronts, did not fit beside the first and ran after it (11.6 us
// for the 9.3 below).  29x27x48 -> 120 5x5 at batch 8 from codes, timestamps: start to first loads 1.1 us, the windows 3.0 (3.6 packed as they
// were loaded), the end 0.9 (2.0 with a bounds test, an address and a load of the scale for every element).  With the last window fetching no other
// (it made a tile's wavefronts, of three windows or so each, wait for loads that nobody used): 28x28x48 -> 120 11.7 -> 10.2, 28x28x208 -> 256 1x1 at
// batch 4 10.1 -> 6.6, 14x14x100 -> 100 3x3 at batch 8 packed 6.4 -> 5.8, 56x56x20 -> 128 at batch 4 10.6 -> 8.1, 7x7x500 -> 200 at batch 16 12.1 -> 10.5
// (unshared tiles with many windows, 57x57x36 -> 128 at batch 4: 8.65 -> 8.75; one loop for them, the last window fetching another, 9.15).
// Measured against the permute kernel (Cin % 16 == 0) and the LDS kernel that ran these layers before, packed codes, graph replays:
// 8x29x27x48 -> 120 5x5 43.1 -> 8.6 us (0.2 of the rate at which the instruction can select: 1.8 us), 28x28x112 -> 224 3x3 at batch
// 16 76.5 -> 16.3, 57x57x36 -> 128 3x3 at batch 4 142 -> 8.9, 56x56x16 -> 32 for one image 6.2 -> 3.8 (a launch: 1.6).
// RAW: the activations are codes one per byte and are packed in registers as they are loaded, which spares the packing
// kernel's launch.
#pragma once

#include "dg_onehot_kernel.h"

#include <type_traits>

namespace dgoh {

struct RaggedArgs {
    DgProblem p;                 // as the kernel runs it: activations on the matrix rows, p.M on its columns
    Pools pools;
    FastDiv div_ow, div_oh, div_kw, div_win;
    int32_t tiles_m;
    int32_t pair_taps;           // 1: in pairs of taps, 0: each tap in halves
    int32_t seg;                 // bytes of a segment
    int32_t base1, lead1;        // half 1: its segment's first byte within the tap, masked bytes at its start
    int32_t windows;             // windows per segment
    int32_t chunks, cpw;         // windows in all, and per wavefront
    int32_t scale_rows;          // the scale goes with p's n, not its m (a row-major GEMM, run transposed)
    int32_t n_first;             // the output is contiguous in n: consecutive threads store consecutive n
};

template <int CH>
struct __attribute__((packed, aligned(1))) RawWords {
    uint32_t v[CH];
};

template <int CH>
__device__ __forceinline__ Words<CH> load_unaligned(const uint8_t *ptr)
{
    const RawWords<CH> t = *(const RawWords<CH> *)ptr;
    Words<CH> w;
#pragma unroll
    for (int i = 0; i < CH; ++i) w.v[i] = t.v[i];
    return w;
}

template <int WM, int WN, int CH, bool RAW>
__global__ void __launch_bounds__(WM * WN == 1 ? 1024 : 512, WM * WN <= 2 ? 4 : 2)
smfmac_ragged_kernel(RaggedArgs a)
{
    constexpr int NB = WM * WN, XB = RAW ? 4 : 1;           // activation bytes per packed byte
    __shared__ uint2 s_rows[16];
    __shared__ int32_t s_sum[NB * 1024];                    // [block][accumulator register][lane]
    const DgProblem &p = a.p;
    const int lane = threadIdx.x & 63, S = blockDim.x >> 6;
    int ws = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int tile = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    int m0 = (tile % a.tiles_m) * (WM * 32), n0 = (tile / a.tiles_m) * (WN * 32);
    // (these as they are: the compiler keeps what they were made from beside them, and with more than 80 scalar registers a SIMD holds seven
    // wavefronts instead of eight: 29x29x24 -> 64 5x5 at batch 6, 316 tiles of 13 wavefronts, 6.8 us at 82, 5.4 at 79)
    asm("" : "+s"(ws), "+s"(m0), "+s"(n0));
    const int L = p.Cin / 4, taps = p.KH * p.KW;
    // this wavefront's windows (the host leaves none without one; the max only keeps an odd launch harmless)
    const int c0 = ws * a.cpw, c1 = max(c0, min(c0 + a.cpw, a.chunks));
    const bool through_lds = S > 1 || a.scale_rows || a.n_first;

    float sc_cols[WM];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) sc_cols[bm] = 0.0f;
    if (!a.scale_rows) dg_mfma_column_scales<WM, true>(p, m0, lane, sc_cols);
    const uint8_t *w_ptr[WM];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) w_ptr[bm] = p.Wp + (int64_t)min(m0 + bm * 32 + r, p.M - 1) * (p.K / 4);
    Column col[WN];
#pragma unroll
    for (int bn = 0; bn < WN; ++bn) col[bn] = make_column(p, a.div_ow, a.div_oh, n0 + bn * 32 + r, L * XB, 0);

    const int base = h ? a.base1 : 0, lead = h ? a.lead1 : 0;
    // the window fetched next
    int pair = (int)fdiv((uint32_t)min(c0, a.chunks - 1), a.div_win), win = min(c0, a.chunks - 1) - pair * a.windows;
    // A window as it is loaded -- codes one per byte are packed when their turn comes, not before: packed at once, as they
    // were, every window waited for the next one's loads in the middle of its own matrix instructions.  (Two windows in flight: slower, the
    // compiler moves them between registers at the loop's end and waits for them there.)
    struct Window {
        Words<CH> wa[WM][2];
        Words<RAW ? 4 : CH> x[WN][RAW ? CH : 1];
        bool vb[WN];
        int dead;                                           // bytes, from its start, that an earlier window or the other half counts
    };
    auto fetch = [&](Window &w) {
        const int start = min(4 * CH * win, a.seg - 4 * CH), overlap = 4 * CH * win - start;
        w.dead = max(overlap, lead - (4 * CH * win - overlap));
        // weights: both halves' words; (an odd tap count: the last pair's second tap is any tap, its kept bytes are zero)
        const int tap0 = a.pair_taps ? 2 * pair : pair, tap1 = a.pair_taps ? min(tap0 + 1, taps - 1) : tap0;
        const int w0 = tap0 * L + start, w1 = tap1 * L + a.base1 + start;
#pragma unroll
        for (int bm = 0; bm < WM; ++bm) {
            w.wa[bm][0] = load_unaligned<CH>(w_ptr[bm] + w0);
            w.wa[bm][1] = load_unaligned<CH>(w_ptr[bm] + w1);
        }
        const int tap = a.pair_taps ? 2 * pair + h : pair;
        const int kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
        const int inside = base + start;
        const int64_t tap_off = ((int64_t)kh * p.W + kw) * L + inside;
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const int ih = col[bn].ih0 + kh, iw = col[bn].iw0 + kw;
            w.vb[bn] = col[bn].ok & (tap < taps) & ((uint32_t)ih < (uint32_t)p.H) & ((uint32_t)iw < (uint32_t)p.W);
            // (outside the image: the same bytes of the first pixel, multiplied by kept bytes of zero)
            const uint8_t *ptr = w.vb[bn] ? p.Xp + col[bn].off0 + tap_off * XB : p.Xp + inside * XB;
#pragma unroll
            for (int i = 0; i < (RAW ? CH : 1); ++i) w.x[bn][i] = load_unaligned<RAW ? 4 : CH>(ptr + 16 * i);
        }
        if (++win == a.windows) win = 0, ++pair;            // (uniform)
    };

    // The table's rows come with the other scalar arguments, before the first loads: as two loads per lane at the kernel's start, written
    // while the first window's were on their way, they made 59 of 105 layers 2 - 15 % slower (31x28x88 -> 316 1x1 at batch 7 5.6 ->
    // 6.5 us, 14x14x100 -> 100 3x3 at batch 8 4.4 -> 4.6), and none faster by more than 2 %.
    sparse_fill_table(s_rows, a.pools, threadIdx.x);
    Window w;
    fetch(w);
    // every wavefront's zeroes go to LDS while the loads are on their way
    if (through_lds)
        for (int i = threadIdx.x; i < NB * 1024; i += blockDim.x) s_sum[i] = 0;
    v16i acc[WM][WN];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][bn][e] = 0;
    // (the scales, asked for first, are in: said once, or they are waited for, and every store before with them, at each group of stores)
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) asm volatile("" : "+v"(sc_cols[bm]));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t pick = sparse_pick(h);
    // (the last window by itself: it has none to fetch, which a branch in the loop would keep from being fetched among the matrix instructions)
    auto window = [&](auto more) {
        Words<CH> ca[WM][2], cb[WN];
        bool valid[WN];
        const int dead = w.dead;
#pragma unroll
        for (int bm = 0; bm < WM; ++bm) ca[bm][0] = w.wa[bm][0], ca[bm][1] = w.wa[bm][1];
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            valid[bn] = w.vb[bn];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                if constexpr (RAW) {
                    const Words<4> &t = w.x[bn][i];
                    cb[bn].v[i] = dg_pack_codes16(make_uint4(t.v[0], t.v[1], t.v[2], t.v[3]));
                } else {
                    cb[bn].v[i] = w.x[bn][0].v[i];
                }
            }
        }
        if constexpr (more) fetch(w);
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            v4i kept, ones[WN];
#pragma unroll
            for (int b = 0; b < 4; ++b) kept[b] = 4 * t + b >= dead ? 0x00010001 : 0;
#pragma unroll
            for (int bn = 0; bn < WN; ++bn)
#pragma unroll
                for (int b = 0; b < 4; ++b) ones[bn][b] = valid[bn] ? kept[b] : 0;
            // (one block of channels after the other: the operands of both at once are registers that a fourth wavefront per SIMD needs)
#pragma unroll
            for (int bm = 0; bm < WM; ++bm) {
                v8i dn[2];
                sparse_dense_rows_shared(s_rows, ca[bm][0].v[t], ca[bm][1].v[t], pick, dn[0], dn[1]);
#pragma unroll
                for (int bn = 0; bn < WN; ++bn) {
                    acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones[bn], dn[0], acc[bm][bn], (int)cb[bn].v[t], 0, 0);
                    acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones[bn], dn[1], acc[bm][bn], (int)(cb[bn].v[t] >> 2), 0, 0);
                }
            }
        }
    };
    for (int c = c0; c + 1 < c1; ++c) window(std::true_type());
    if (c0 < c1) window(std::false_type());

    // (Every load is in: said once.  A wavefront without windows has its first one's under way, and the compiler would wait for them -- and
    // with them for the stores -- wherever a store's address takes one of their registers.)
    __builtin_amdgcn_s_waitcnt(0x0F70);                     // vmcnt(0)
    // (this lane's number once more, which takes no register of the walk's)
    const int lane_out = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), r_out = lane_out & 31, h_out = lane_out >> 5;
    // (streamed whatever the rows (dg_output_cached): through the caches 80 layers of up to 22 MB of output were the same within 4 %, of 22 to 110 MB
    // three 2 % behind and six ahead, 56x56x60 -> 252 at batch 27 37.5, 17.5 us; not made yet)
    if (!through_lds) {
        dg_mfma_store_tile<WM, WN, true>(p, acc, m0, n0, lane_out, sc_cols);
        return;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            __hip_atomic_fetch_add(&s_sum[(i * 16 + e) * 64 + lane_out], acc[i / WN][i % WN][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
    if (!a.n_first && !a.scale_rows && p.stride_cm == 1) {  // (uniform: the channels contiguous, their scales at hand)
        if (S <= NB * 4) {
            for (int u = ws; u < NB * 4; u += S) {          // groups of four registers: 8 pixels x 32 channels each
                const int i = u >> 2;
                v4i sum[1];
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[0][e] = s_sum[(4 * u + e) * 64 + lane_out];
                dg_mfma_store_quads<1>(p, sum, u & 3, m0 + (i / WN) * 32, n0 + (i % WN) * 32, lane_out, WM == 1 || i / WN == 0 ? sc_cols[0] : sc_cols[WM - 1]);
            }
            return;
        }
        for (int u = ws; u < NB * 16; u += S) {             // more wavefronts than groups: a register at a time
            const int i = u >> 4, e = u & 15, m = m0 + (i / WN) * 32 + r_out, n = n0 + (i % WN) * 32 + 8 * (e >> 2) + 4 * h_out + (e & 3);
            if (m >= p.M || n >= p.N) continue;
            const int32_t sum = s_sum[u * 64 + lane_out];
            const int64_t o = m + (int64_t)n * p.stride_cn;
            if (p.scale) p.Cf[o] = (float)sum * (WM == 1 || i / WN == 0 ? sc_cols[0] : sc_cols[WM - 1]);
            else p.C[o] = sum;
        }
        return;
    }
    for (int idx = threadIdx.x; idx < NB * 1024; idx += blockDim.x) {
        const int i = idx >> 10;
        int e = (idx >> 6) & 15, l = idx & 63;
        if (a.n_first) {                                      // (uniform: element (idx / 32) of the channels, idx % 32 of the pixels)
            const int x = idx & 31, y = (idx >> 5) & 31;
            e = 4 * (x >> 3) + (x & 3), l = ((x >> 2) & 1) * 32 + y;
        }
        const int m = m0 + (i / WN) * 32 + (l & 31), n = n0 + (i % WN) * 32 + 8 * (e / 4) + 4 * (l >> 5) + (e % 4);
        if (m >= p.M || n >= p.N) continue;
        const int64_t o = (int64_t)m * p.stride_cm + (int64_t)n * p.stride_cn;
        const int32_t sum = s_sum[(i * 16 + e) * 64 + l];
        if (p.scale)
            p.Cf[o] = (float)sum * p.scale[a.scale_rows ? n : m];
        else
            p.C[o] = sum;
    }
}

// `raw`: p.Xp holds codes one per byte.  The activations' offsets fit 31 bits (the caller checks).
inline void launch_ragged(const DgProblem &p, const Pools &pools, const RaggedPlan &q, bool scale_rows, bool n_first, bool raw, hipStream_t stream)
{
    RaggedArgs a;
    a.p = p;
    a.pools = pools;
    a.div_ow = make_div((uint32_t)p.OW), a.div_oh = make_div((uint32_t)p.OH), a.div_kw = make_div((uint32_t)p.KW);
    a.div_win = make_div((uint32_t)q.windows);
    a.tiles_m = (p.M + 32 * q.wm - 1) / (32 * q.wm);
    a.pair_taps = q.pair_taps, a.seg = q.seg, a.base1 = q.base1, a.lead1 = q.lead1, a.windows = q.windows;
    a.chunks = q.chunks, a.cpw = q.cpw;
    a.scale_rows = scale_rows, a.n_first = n_first;
    const int64_t tiles = (int64_t)a.tiles_m * (((int64_t)p.N + 32 * q.wn - 1) / (32 * q.wn));
    const dim3 grid((unsigned)tiles), block(64 * q.S);
#define DG_RAGGED(WM, WN, CH) \
    if (raw) hipLaunchKernelGGL((smfmac_ragged_kernel<WM, WN, CH, true>), grid, block, 0, stream, a); \
    else hipLaunchKernelGGL((smfmac_ragged_kernel<WM, WN, CH, false>), grid, block, 0, stream, a)
#define DG_RAGGED_TILES(CH) \
    if (q.wm == 2 && q.wn == 2) { DG_RAGGED(2, 2, CH); } \
    else if (q.wm == 2) { DG_RAGGED(2, 1, CH); } \
    else { DG_RAGGED(1, 1, CH); }
    if (q.ch == 4) { DG_RAGGED_TILES(4) }
    else if (q.ch == 3) { DG_RAGGED_TILES(3) }
    else if (q.ch == 2) { DG_RAGGED_TILES(2) }
    else { DG_RAGGED_TILES(1) }
#undef DG_RAGGED_TILES
#undef DG_RAGGED
}

}   // namespace dgoh
