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
// Bound by issue slots and by how few wavefronts such small layers have, not by the matrix pipe (8x29x27x48 -> 120 5x5 from codes:
// 36 VALU instructions per matrix instruction, VALU issue 0.35 of the cycles, the pipe 0.08, 1.4 wavefronts per SIMD).  So S wavefronts
// of a workgroup share one tile and split the windows of K among them, their sums meeting in LDS (exact in any order).
// Measured against the permute kernel (Cin % 16 == 0) and the LDS kernel that ran these layers, packed codes, graph replays:
// 8x29x27x48 -> 120 5x5 43.1 -> 8.6 us (0.2 of the rate at which the instruction can select: 1.8 us), 28x28x112 -> 224 3x3 at batch
// 16 76.5 -> 16.3, 57x57x36 -> 128 3x3 at batch 4 142 -> 8.9, 56x56x16 -> 32 for one image 6.2 -> 3.8 (a launch: 1.6).
// RAW: the activations are codes one per byte and are packed in registers as they are loaded, which spares the packing
// kernel's launch.
#pragma once

#include "dg_onehot_kernel.h"

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
__global__ void __launch_bounds__(WM * WN == 1 ? 1024 : 512, WM * WN == 1 ? 4 : 2)
smfmac_ragged_kernel(RaggedArgs a)
{
    constexpr int NB = WM * WN, XB = RAW ? 4 : 1;           // activation bytes per packed byte
    __shared__ uint2 s_rows[16];
    __shared__ int32_t s_sum[NB * 1024];                    // [block][accumulator register][lane]
    const DgProblem &p = a.p;
    const int lane = threadIdx.x & 63, ws = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), S = blockDim.x >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int tile = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int m0 = (tile % a.tiles_m) * (WM * 32), n0 = (tile / a.tiles_m) * (WN * 32);
    const int L = p.Cin / 4, taps = p.KH * p.KW;
    // this wavefront's windows (the host leaves none without one; the max only keeps an odd launch harmless)
    const int c0 = ws * a.cpw, c1 = max(c0, min(c0 + a.cpw, a.chunks));
    const bool through_lds = S > 1 || a.scale_rows || a.n_first;

    sparse_fill_table(s_rows, a.pools, threadIdx.x);
    if (through_lds)
        for (int i = threadIdx.x; i < NB * 1024; i += blockDim.x) s_sum[i] = 0;
    const uint8_t *w_ptr[WM];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) w_ptr[bm] = p.Wp + (int64_t)min(m0 + bm * 32 + r, p.M - 1) * (p.K / 4);
    Column col[WN];
#pragma unroll
    for (int bn = 0; bn < WN; ++bn) col[bn] = make_column(p, a.div_ow, a.div_oh, n0 + bn * 32 + r, L * XB, 0);
    float sc_cols[WM];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) sc_cols[bm] = 0.0f;
    if (!a.scale_rows) dg_mfma_column_scales<WM, true>(p, m0, lane, sc_cols);

    v16i acc[WM][WN];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][bn][e] = 0;

    const int base = h ? a.base1 : 0, lead = h ? a.lead1 : 0;
    // the window fetched next
    int pair = (int)fdiv((uint32_t)min(c0, a.chunks - 1), a.div_win), win = min(c0, a.chunks - 1) - pair * a.windows;
    Words<CH> wa[WM][2], wb[WN];
    bool vb[WN];
    auto fetch = [&]() {
        const int start = min(4 * CH * win, a.seg - 4 * CH);
        // weights: both halves' words; (an odd tap count: the last pair's second tap is any tap, its kept bytes are zero)
        const int tap0 = a.pair_taps ? 2 * pair : pair, tap1 = a.pair_taps ? min(tap0 + 1, taps - 1) : tap0;
        const int w0 = tap0 * L + start, w1 = tap1 * L + a.base1 + start;
#pragma unroll
        for (int bm = 0; bm < WM; ++bm) {
            wa[bm][0] = load_unaligned<CH>(w_ptr[bm] + w0);
            wa[bm][1] = load_unaligned<CH>(w_ptr[bm] + w1);
        }
        const int tap = a.pair_taps ? 2 * pair + h : pair;
        const int kh = (int)fdiv((uint32_t)tap, a.div_kw), kw = tap - kh * p.KW;
        const int inside = base + start;
        const int64_t tap_off = ((int64_t)kh * p.W + kw) * L + inside;
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const int ih = col[bn].ih0 + kh, iw = col[bn].iw0 + kw;
            vb[bn] = col[bn].ok & (tap < taps) & ((uint32_t)ih < (uint32_t)p.H) & ((uint32_t)iw < (uint32_t)p.W);
            // (outside the image: the same bytes of the first pixel, multiplied by kept bytes of zero)
            const uint8_t *ptr = vb[bn] ? p.Xp + col[bn].off0 + tap_off * XB : p.Xp + inside * XB;
            if constexpr (RAW) {
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const Words<4> t = load_unaligned<4>(ptr + 16 * i);
                    wb[bn].v[i] = dg_pack_codes16(make_uint4(t.v[0], t.v[1], t.v[2], t.v[3]));
                }
            } else {
                wb[bn] = load_unaligned<CH>(ptr);
            }
        }
    };

    fetch();
    // the table and every wavefront's zeroes are in LDS; the loads above stay in flight across this barrier
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t pick = sparse_pick(h);
    for (int c = c0; c < c1; ++c) {
        Words<CH> ca[WM][2], cb[WN];
        bool valid[WN];
#pragma unroll
        for (int bm = 0; bm < WM; ++bm) ca[bm][0] = wa[bm][0], ca[bm][1] = wa[bm][1];
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) cb[bn] = wb[bn], valid[bn] = vb[bn];
        // bytes of this window, from its start, that an earlier window or the other half counts
        const int overlap = 4 * CH * win - min(4 * CH * win, a.seg - 4 * CH);
        const int dead = max(overlap, lead - (4 * CH * win - overlap));
        if (c + 1 < c1) {                                    // (uniform; the last one re-reads in bounds and is unused)
            if (++win == a.windows) win = 0, ++pair;
        }
        fetch();
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            v8i dn[WM][2];
#pragma unroll
            for (int bm = 0; bm < WM; ++bm)
                sparse_dense_rows_shared(s_rows, ca[bm][0].v[t], ca[bm][1].v[t], pick, dn[bm][0], dn[bm][1]);
            v4i kept;
#pragma unroll
            for (int b = 0; b < 4; ++b) kept[b] = 4 * t + b >= dead ? 0x00010001 : 0;
#pragma unroll
            for (int bn = 0; bn < WN; ++bn) {
                v4i ones;
#pragma unroll
                for (int b = 0; b < 4; ++b) ones[b] = valid[bn] ? kept[b] : 0;
                const int even = (int)cb[bn].v[t], odd = (int)(cb[bn].v[t] >> 2);
#pragma unroll
                for (int bm = 0; bm < WM; ++bm) acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones, dn[bm][0], acc[bm][bn], even, 0, 0);
#pragma unroll
                for (int bm = 0; bm < WM; ++bm) acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones, dn[bm][1], acc[bm][bn], odd, 0, 0);
            }
        }
    }

    if (!through_lds) {
        dg_mfma_store_tile<WM, WN, true>(p, acc, m0, n0, lane, sc_cols);
        return;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            __hip_atomic_fetch_add(&s_sum[(i * 16 + e) * 64 + lane], acc[i / WN][i % WN][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
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
