// Accumulator tiles of v_mfma_i32_32x32x32_i8 and their way to memory, shared by the two matrix-core kernels.
//
// A 32x32 accumulator block lives in 16 registers per lane: the lane holds MFMA column (lane % 32) and MFMA rows
// 8*(e/4) + 4*(lane/32) + e%4, e = 0..15.  Which problem axis sits on the MFMA columns is the kernel's choice (the two
// operands have the same lane layout, so swapping them transposes the block): the axis whose output stride is 1
// goes on the columns, so that the 32 lanes of a half wavefront store 128 contiguous bytes.
//   TR == false: MFMA rows = m, columns = n  (acc = mfma(weights, activations)) -- row-major GEMM output, n contiguous
//   TR == true : MFMA rows = n, columns = m  (acc = mfma(activations, weights)) -- NHWC convolution output, m contiguous
#pragma once

#include "dg_common.h"
#include "dg_quant.h"

typedef int dg_v4i __attribute__((ext_vector_type(4)));
typedef int dg_v16i __attribute__((ext_vector_type(16)));

template <bool TR>
__device__ __forceinline__ dg_v16i dg_mfma_step(dg_v4i w, dg_v4i x, dg_v16i acc)
{
    return TR ? __builtin_amdgcn_mfma_i32_32x32x32_i8(x, w, acc, 0, 0, 0)
              : __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, acc, 0, 0, 0);
}

// With TR a lane stores one channel m per row block whatever the element, so its scales can be fetched long before the
// stores: dg_mfma_column_scales at the start of the kernel, handed to dg_mfma_store_tile at the end.
template <int WM, bool TR>
__device__ __forceinline__ void dg_mfma_column_scales(const DgProblem &p, int m0, int lane, float (&sc)[WM])
{
#pragma unroll
    for (int bm = 0; bm < WM; ++bm) {
        const int m = min(m0 + bm * 32 + (lane & 31), p.M - 1);
        sc[bm] = (TR && p.scale) ? p.scale[m] : 0.0f;
    }
}

// Store one 32x32 block whose first row / column sit at (mb, nb): int32 as it is, or float(acc) * scale[m] (one
// conversion, one multiply); `sc` is the lane's prefetched scale (TR only).
// OR of `v` over the four lanes of a quad (two DPP quad permutes); every lane gets the result.
__device__ __forceinline__ uint32_t dg_quad_or(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);    // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    return v;
}

// Re-quantising store of one block (TR layout only: the lanes of a quad hold four consecutive channels of one output
// pixel).  Each lane turns its 16 sums into 2-bit codes.  For four consecutive pixels (accumulator registers 4q .. 4q+3)
// a lane places its four codes in the four bytes of a word, at the bit position of its channel within the packed byte;
// one OR across the quad (two DPP permutes) completes the four packed bytes in every lane, and lane i of the quad
// stores the byte of pixel i -- so all lanes store.  Call with all 64 lanes active.
__device__ __forceinline__ void dg_mfma_requant_quad(const DgProblem &p, const dg_v4i &acc, int e4, int mb, int nb, int lane, float sc)
{
    const int r = lane & 31, h = lane >> 5, q = r & 3;
    const bool live = mb + r < p.M;                       // (M % 4 == 0: a quad is inside M or outside as a whole)
    const float lo_f = (float)p.q_lo, hi_f = (float)(p.q_lo + 3);
    uint32_t word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float y = __fmul_rn((float)acc[i], sc);
        word |= dg_quantize_code_clamped(y, p.q_scale, p.q_zero, lo_f, hi_f) << (8 * i);
    }
    word = dg_quad_or(live ? word << (2 * q) : 0u);       // byte i = the packed byte of pixel i
    const int n = nb + 8 * e4 + 4 * h + q;                // the pixel whose byte this lane stores
    if (live && n < p.N) p.Qp[(int64_t)n * (p.M / 4) + (mb + r) / 4] = (uint8_t)(word >> (8 * q));
}
__device__ __forceinline__ void dg_mfma_requant_block(const DgProblem &p, const dg_v16i &acc, int mb, int nb, int lane,
                                                      float sc)
{
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4)
        dg_mfma_requant_quad(p, (dg_v4i){acc[4 * e4], acc[4 * e4 + 1], acc[4 * e4 + 2], acc[4 * e4 + 3]}, e4, mb, nb, lane, sc);
}

// Whether a block's rows all lie inside the output and its 32 x 32 footprint spans less than 2^30 elements (strides may be
// negative): what the stores without a test per element need, besides the columns.
__device__ __forceinline__ bool dg_mfma_rows_whole(int64_t row_stride, int64_t col_stride, int rowb, int row_limit)
{
    const int64_t span = 32 * ((row_stride < 0 ? -row_stride : row_stride) + (col_stride < 0 ? -col_stride : col_stride));
    return rowb + 32 <= row_limit && span < ((int64_t)1 << 30);
}

// How a block's stores go: past the caches, through them, or as the problem says (DgProblem::cached: dg_output_cached).
enum DgOut { DG_OUT_STREAM, DG_OUT_CACHED, DG_OUT_BY_PROBLEM };
template <DgOut OUT, class T>
__device__ __forceinline__ void dg_put(T v, T *to)
{
    static_assert(OUT != DG_OUT_BY_PROBLEM, "decided before");
    if constexpr (OUT == DG_OUT_STREAM) __builtin_nontemporal_store(v, to);
    else *to = v;
}

// EDGE_COLUMNS: blocks whose columns are not all inside take the stores without a test per element too, the lanes of columns
// beyond the last sitting them out.  For kernels whose wavefronts have one column block each, all of which would be stored
// element by element where it is partial: dg_sparse_ws_kernel.h, and dg_sparse_staged_kernel.h, where (packed codes, graph
// replays) 28x28x256 -> 200 at batch 32 went from 17.4 to 14.5 us with 3-bit codes, 56x56x256 -> 72 from 28.6 to 23.3, 56x56x128 ->
// 72 3x3 at batch 16 from 21.7 to 17.9 with 2-bit ones, and layers of whole blocks stayed (56x56x128 -> 128 3x3 17.0, 17.2).
template <bool TR, bool EDGE_COLUMNS, DgOut OUT>
__device__ __forceinline__ void dg_mfma_store_sums(const DgProblem &p, const dg_v16i &acc, int mb, int nb, int lane, float sc)
{
    const int r = lane & 31, h = lane >> 5;
    // (mb and nb are the same in every lane of the wavefront: say so, and the block's base address is scalar arithmetic)
    const int colb = __builtin_amdgcn_readfirstlane(TR ? mb : nb), rowb = __builtin_amdgcn_readfirstlane(TR ? nb : mb);
    const int col_limit = TR ? p.M : p.N, row_limit = TR ? p.N : p.M;
    const int64_t row_stride = TR ? p.stride_cn : p.stride_cm, col_stride = TR ? p.stride_cm : p.stride_cn;
    // A block wholly inside the output: one uniform base address, a 32-bit offset per lane, then steps of the row stride
    // -- no bounds test and no 64-bit arithmetic per element.  The stores are streaming (non-temporal) stores, the output
    // being written once and read by a later kernel, where its rows are whole 64-byte pieces (dg_output_cached).
    if ((EDGE_COLUMNS || colb + 32 <= col_limit) && dg_mfma_rows_whole(row_stride, col_stride, rowb, row_limit)) {
        if (EDGE_COLUMNS && colb + r >= col_limit) return;
        const int64_t base = (int64_t)colb * col_stride + (int64_t)rowb * row_stride;
        const int rs = (int)row_stride, off0 = r * (int)col_stride + 4 * h * rs;
        if (p.scale) {
            float *out = p.Cf + base;
            const float *scale_rows = p.scale + rowb + 4 * h;          // (row-major GEMM output: the scale goes with the row)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = 8 * (e / 4) + (e % 4);
                dg_put<OUT>((float)acc[e] * (TR ? sc : scale_rows[k]), out + (off0 + k * rs));
            }
        } else {
            int32_t *out = p.C + base;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = 8 * (e / 4) + (e % 4);
                dg_put<OUT>(acc[e], out + (off0 + k * rs));
            }
        }
        return;
    }
    // a block on the output's edge: every element tested
    const int col = colb + r;
    if (col >= col_limit) return;
    const int row0 = rowb + 4 * h;
    const int64_t first = (int64_t)col * col_stride + (int64_t)row0 * row_stride;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int k = 8 * (e / 4) + (e % 4);
        if (row0 + k >= row_limit) continue;
        const int64_t o = first + k * row_stride;
        if (p.scale)
            dg_put<OUT>((float)acc[e] * (TR ? sc : p.scale[row0 + k]), p.Cf + o);
        else
            dg_put<OUT>(acc[e], p.C + o);
    }
}
template <bool TR, bool EDGE_COLUMNS = false, DgOut OUT = DG_OUT_STREAM>
__device__ __forceinline__ void dg_mfma_store_block(const DgProblem &p, const dg_v16i &acc, int mb, int nb, int lane,
                                                    float sc)
{
    if (TR && p.Qp) dg_mfma_requant_block(p, acc, mb, nb, lane, sc);
    else if (OUT == DG_OUT_CACHED || (OUT == DG_OUT_BY_PROBLEM && p.cached))           // (uniform)
        dg_mfma_store_sums<TR, EDGE_COLUMNS, DG_OUT_CACHED>(p, acc, mb, nb, lane, sc);
    else dg_mfma_store_sums<TR, EDGE_COLUMNS, DG_OUT_STREAM>(p, acc, mb, nb, lane, sc);
}

// Store NQ groups of four registers of a block, the first one group q0 (TR layout; a partial last block of channels as with EDGE_COLUMNS
// above; always past the caches, whatever dg_output_cached says: shared tiles belong to layers of a few microseconds, whose outputs gain 4 % at most the other
// way; the kernel by the codes' bits has up to four rounds of tiles, 32 MB, for which the other way was not measured).
template <int NQ>
__device__ __forceinline__ void dg_mfma_store_quads(const DgProblem &p, const dg_v4i (&acc)[NQ], int q0, int mb, int nb, int lane, float sc)
{
    if (p.Qp) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) dg_mfma_requant_quad(p, acc[q], q0 + q, mb, nb, lane, sc);
        return;
    }
    const int r = lane & 31, h = lane >> 5;
    const int colb = __builtin_amdgcn_readfirstlane(mb), rowb = __builtin_amdgcn_readfirstlane(nb), row0 = rowb + 8 * q0;
    if (colb + r >= p.M) return;                          // (group q: rows 8 q + 4 h ... + 3 of the block, this lane's)
    if (dg_mfma_rows_whole(p.stride_cn, p.stride_cm, rowb, p.N)) {
        const int64_t base = (int64_t)colb * p.stride_cm + (int64_t)row0 * p.stride_cn;
        const int rs = (int)p.stride_cn, off0 = r * (int)p.stride_cm + 4 * h * rs;
        if (p.scale) {
            float *out = p.Cf + base;
#pragma unroll
            for (int e = 0; e < 4 * NQ; ++e) dg_put<DG_OUT_STREAM>((float)acc[e / 4][e % 4] * sc, out + (off0 + (8 * (e / 4) + e % 4) * rs));
        } else {
            int32_t *out = p.C + base;
#pragma unroll
            for (int e = 0; e < 4 * NQ; ++e) dg_put<DG_OUT_STREAM>(acc[e / 4][e % 4], out + (off0 + (8 * (e / 4) + e % 4) * rs));
        }
        return;
    }
    const int64_t first = (int64_t)(colb + r) * p.stride_cm + (int64_t)(row0 + 4 * h) * p.stride_cn;
#pragma unroll
    for (int e = 0; e < 4 * NQ; ++e) {
        const int k = 8 * (e / 4) + e % 4;
        if (row0 + 4 * h + k >= p.N) continue;
        const int64_t o = first + k * p.stride_cn;
        if (p.scale) dg_put<DG_OUT_STREAM>((float)acc[e / 4][e % 4] * sc, p.Cf + o);
        else dg_put<DG_OUT_STREAM>(acc[e / 4][e % 4], p.C + o);
    }
}

// Store the (WM*32) x (WN*32) tile at (m0, n0).  (How, decided once for the tile: a branch in each of 14 blocks is more than the compiler unrolls.)
template <int WM, int WN, bool TR, bool EDGE_COLUMNS = false, DgOut OUT = DG_OUT_STREAM>
__device__ __forceinline__ void dg_mfma_store_tile(const DgProblem &p, const dg_v16i (&acc)[WM][WN], int m0, int n0,
                                                   int lane, const float (&sc_cols)[WM])
{
    if (OUT == DG_OUT_BY_PROBLEM && p.cached) {             // (uniform)
#pragma unroll
        for (int bm = 0; bm < WM; ++bm)
#pragma unroll
            for (int bn = 0; bn < WN; ++bn)
                dg_mfma_store_sums<TR, EDGE_COLUMNS, DG_OUT_CACHED>(p, acc[bm][bn], m0 + bm * 32, n0 + bn * 32, lane, sc_cols[bm]);
        return;
    }
#pragma unroll
    for (int bm = 0; bm < WM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
            dg_mfma_store_block<TR, EDGE_COLUMNS, OUT == DG_OUT_CACHED ? DG_OUT_CACHED : DG_OUT_STREAM>(p, acc[bm][bn], m0 + bm * 32, n0 + bn * 32,
                                                                                                          lane, sc_cols[bm]);
}
