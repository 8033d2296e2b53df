// 2-bit table kernel on the sparse matrix instruction (operand layout, index register and row-pair table as in
// dg_onehot_kernel.h, BITS = 20), with the packed operands fetched in WHOLE 32-BYTE RUNS and handed to their lanes
// through LDS.  A wavefront owns a tile of 32 (or 64) channels x 64 ... 224 pixels and walks all of K, or a share of it.
//
// Why: the matrix instruction wants lane (r, half) to hold words of row r, so a direct load has 32 lanes reading 8
// bytes each from 32 different rows.  The address unit of a compute unit takes such a load one cache line per cycle
// (dg_lds_dma.h): 64 cycles and more for 512 or 1024 bytes, and on a GEMM with K = 8192 it was busy 93 % of the
// kernel's time (counters TA_TA_BUSY / TCP_GATE_EN) while the matrix pipe idled -- the loads, not the arithmetic, set
// the time.  Here two neighbouring lanes read the two 16-byte halves of one row's run, so a load instruction covers 32
// rows x 32 bytes, at half the address cycles per byte (26 % busy on the same GEMM).  The loads write LDS directly
// (lane l's 16 bytes land at the instruction's LDS base + 16 l; no registers are held while they are in flight), into
// staging rows of the wavefront's own, from which lane (r, half) reads its 8 bytes per 64 positions of K.  Staging
// rows belong to one wavefront, so no barrier is involved: a wavefront waits for its own loads (vmcnt) before it reads
// a run, and runs go round in two or three buffers.
// The multiplication is one software pipeline over all of K: the dense operands of a step are made between the matrix
// instructions of the step before (or the one before that), and the words they are made from are read from LDS a step or more earlier still, across
// chunks, runs and filter taps alike.
//
// A run is 128 positions of K inside one filter tap (Cin % 128 == 0; Cin % 128 == 64: HALF below).  A tap outside the image is fetched from
// wherever it would lie (outside the tensor: as zeros) and contributes nothing because the kept bytes of its lanes are zero.
//
// Where the time goes (timestamps per wavefront at 100 MHz, us; before: the words read a step later, every operand from pairs, the table
// filled before the first load, sums met by atomic additions, two wavefronts of four storing):
//   28x28x256 -> 256 3x3 at batch 8, two planes, 32 x 128 by four   start to first words 3.0 -> 2.4, the walk over K 10.3 -> 9.1,
//                                                                   the end 2.3 -> 2.3; kernel 18.1 -> 16.1, the call 20.9 -> 18.4
//   8192 x 256 x 8192, 32 x 128 by four                             the walk 20.0 -> 17.5; kernel 27.8 -> 25.9 - 26.8
// The second's matrix instructions are 32.8 thousand cycles per SIMD, 16.8 us at the 1.95 GHz that the kernel runs at (50.4 thousand cycles in
// 25.9 us): its walk is the matrix pipe's, and the pipe is busy 0.65 of the kernel.  A lone wavefront, whose other instructions do not all hide
// behind its own matrix instructions, spends about 0.48 us per run beside them.
#pragma once

#include "dg_lds_dma.h"
#include "dg_onehot_kernel.h"

#include <type_traits>

namespace dgoh {

// The table of rows in LDS, one for the workgroup, in one of two forms.
//
// PairTable: 16 entries of two rows (NIB: 16 low rows, 16 high rows), as in dg_onehot_kernel.h.  A step's operands are 16 vector instructions
// (NIB 13) and 8 reads (16) at 4-bit indices, without bank conflicts: little for LDS, much for the vector units.
template <bool NIB, bool TWO>
struct PairTable {
    static constexpr int HIGH = NIB ? 1040 : 128;           // the high rows (the high plane's pairs) begin here
    static constexpr int BYTES = NIB ? HIGH + 64 + 16 : (TWO ? 256 : 128);
    // entry i as thread i of 16 reads it from the kernel's arguments (vector loads, asked for at the kernel's start), and as it writes it
    struct Entry {
        uint32_t q[4];
    };
    static __device__ __forceinline__ Entry load(const Pools &pl, int i)
    {
        Entry e;
        i &= 15;
        e.q[0] = pl.w[NIB ? i : i & 3], e.q[1] = pl.w[NIB ? 16 + i : i >> 2];
        e.q[2] = TWO ? pl.w[4 + (i & 3)] : 0, e.q[3] = TWO ? pl.w[4 + (i >> 2)] : 0;
        return e;
    }
    static __device__ __forceinline__ void wait(Entry &e) { asm volatile("" : "+v"(e.q[0]), "+v"(e.q[1]), "+v"(e.q[2]), "+v"(e.q[3])); }
    static __device__ __forceinline__ void store(char *table, const Entry &e, int i)
    {
        if (i >= 16) return;
        if constexpr (NIB) {
            *(uint32_t *)(table + 4 * i) = e.q[0], *(uint32_t *)(table + HIGH + 4 * i) = e.q[1];
        } else {
            *(uint2 *)(table + 8 * i) = make_uint2(e.q[0], e.q[1]);
            if (TWO) *(uint2 *)(table + HIGH + 8 * i) = make_uint2(e.q[2], e.q[3]);
        }
    }
    static __device__ __forceinline__ uint32_t copy(int) { return 0; }
    static __device__ __forceinline__ void read(const char *table, uint32_t, uint32_t w0, uint32_t w1, uint32_t pick, v8i (&lo)[2], v8i (&hi)[2])
    {
        uint32_t e, o;
        sparse_row_offsets<NIB>(__builtin_amdgcn_perm(w1, w0, pick), e, o);
        asm("" : "+v"(e), "+v"(o));                         // (kept pre-multiplied, a byte each, and movable between matrix instructions)
        sparse_read_rows<NIB, HIGH>((const uint2 *)table, e, o, lo[0], lo[1]);
        if constexpr (TWO) sparse_read_rows<false>((const uint2 *)(table + HIGH), e, o, hi[0], hi[1]);
    }
    static constexpr int BESIDE = NIB ? 30 : (TWO ? 34 : 26);      // instructions of a step's operands
};

// QuadTable: 256 entries.  2-bit codes: entry i, 16 bytes, holds the rows of FOUR codes -- those of bits 0-1,
// 4-5, 2-3, 6-7 of i -- so that one 16-byte read fills half an operand; TWO: the high plane's entries PLANE bytes behind.  NIB: entry
// i, 8 bytes, the low rows of two 4-bit slots (a packed byte), their high rows PLANE bytes behind.  A step's operands are 12 vector
// instructions (NIB 9) and 4 reads (8): beside a matrix instruction (32 cycles) four vector instructions are free, six make it 36.5
// and eight 44, with any number of wavefronts (measured, registers only).  The reads' indices are random, so an entry is held COPIES times, lane l
// reading copy l % COPIES: 16 lanes are served at a time, and with one copy the fullest of the 16 places in the banks gets three of them
// on average, with four two.
template <bool NIB, bool TWO, int COPIES>
struct QuadTable {
    static constexpr int ENTRY = NIB ? 8 : 16;
    static constexpr int SHIFT = (NIB ? 3 : 4) + (COPIES == 8 ? 3 : (COPIES == 4 ? 2 : (COPIES == 2 ? 1 : 0)));      // log2 of an entry's copies
    static constexpr int PLANE = 256 << SHIFT;
    static constexpr int BYTES = PLANE * (NIB || TWO ? 2 : 1);
    static_assert((ENTRY * COPIES) == (1 << SHIFT), "COPIES: 1, 2, 4 or 8");

    // Entry i as thread i of 256 reads it from the kernel's arguments (vector loads: asked for at the kernel's start, they come with the
    // other arguments; `wait` before any load that is not waited for by the compiler), and as it writes it.
    struct Entry {
        uint32_t q[NIB || TWO ? 2 : 1][4];
    };
    static __device__ __forceinline__ Entry load(const Pools &pl, int i)
    {
        Entry e;
#pragma unroll
        for (int plane = 0; plane < (NIB || TWO ? 2 : 1); ++plane) {
            if constexpr (NIB) {
                e.q[plane][0] = pl.w[16 * plane + (i & 15)], e.q[plane][1] = pl.w[16 * plane + (i >> 4)];
                e.q[plane][2] = e.q[plane][3] = 0;
            } else {
                e.q[plane][0] = pl.w[4 * plane + (i & 3)], e.q[plane][1] = pl.w[4 * plane + ((i >> 4) & 3)];
                e.q[plane][2] = pl.w[4 * plane + ((i >> 2) & 3)], e.q[plane][3] = pl.w[4 * plane + (i >> 6)];
            }
        }
        return e;
    }
    static __device__ __forceinline__ void wait(Entry &e)
    {
#pragma unroll
        for (int plane = 0; plane < (NIB || TWO ? 2 : 1); ++plane)
            asm volatile("" : "+v"(e.q[plane][0]), "+v"(e.q[plane][1]), "+v"(e.q[plane][2]), "+v"(e.q[plane][3]));
    }
    static __device__ __forceinline__ void store(char *table, const Entry &e, int i)
    {
        const int turn = (i & 63) / (NIB ? 32 / COPIES : 16 / COPIES);        // (neighbouring threads on different banks)
#pragma unroll
        for (int plane = 0; plane < (NIB || TWO ? 2 : 1); ++plane) {
            char *entry = table + plane * PLANE + (i << SHIFT);
#pragma unroll
            for (int c = 0; c < COPIES; ++c) {
                if constexpr (NIB) *(uint2 *)(entry + ((c + turn) & (COPIES - 1)) * 8) = make_uint2(e.q[plane][0], e.q[plane][1]);
                else *(uint4 *)(entry + ((c + turn) & (COPIES - 1)) * 16) = make_uint4(e.q[plane][0], e.q[plane][1], e.q[plane][2], e.q[plane][3]);
            }
        }
    }

    static __device__ __forceinline__ uint32_t shifted(uint32_t v, int by) { return by >= 0 ? v << by : v >> -by; }

    // The dense operands of the two instructions that consume one packed word per lane half (w0, w1, pick: sparse_dense_rows in
    // dg_onehot_kernel.h); `copy`: this lane's copy, as a byte offset.
    static __device__ __forceinline__ void read(const char *table, uint32_t copy, uint32_t w0, uint32_t w1, uint32_t pick, v8i (&lo)[2], v8i (&hi)[2])
    {
        constexpr uint32_t INDEX = 255u << SHIFT;
        const uint32_t v = __builtin_amdgcn_perm(w1, w0, pick);
        if constexpr (NIB) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const char *x = table + ((shifted(v, SHIFT - 8 * b) & INDEX) | copy);
                const uint2 l = *(const uint2 *)x, h = *(const uint2 *)(x + PLANE);
                lo[0][2 * b] = (int)l.x, lo[0][2 * b + 1] = (int)l.y;
                lo[1][2 * b] = (int)h.x, lo[1][2 * b + 1] = (int)h.y;
            }
        } else {
            // the even (odd) codes of a lane's two 16-bit halves, each half's four brought together as an index: codes 0, 2 (1, 3) stay
            // 4 bits apart and codes 4, 6 (5, 7) go between them
            constexpr uint32_t M = (uint32_t)(0x33333333ull << SHIFT);
            uint32_t e = (shifted(v, SHIFT) & M) | (shifted(v, SHIFT - 6) & ~M);
            uint32_t o = (shifted(v, SHIFT - 2) & M) | (shifted(v, SHIFT - 8) & ~M);
            asm("" : "+v"(e), "+v"(o));                     // (kept as they are: an index in its place, for both halves)
            const uint32_t at[4] = {(e & INDEX) | copy, ((e >> 16) & INDEX) | copy, (o & INDEX) | copy, ((o >> 16) & INDEX) | copy};
#pragma unroll
            for (int plane = 0; plane < (TWO ? 2 : 1); ++plane) {
                v8i(&out)[2] = plane ? hi : lo;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint4 q = *(const uint4 *)(table + at[i] + plane * PLANE);
                    const int d = 4 * (i & 1);
                    out[i / 2][d] = (int)q.x, out[i / 2][d + 1] = (int)q.y, out[i / 2][d + 2] = (int)q.z, out[i / 2][d + 3] = (int)q.w;
                }
            }
        }
    }
    static __device__ __forceinline__ uint32_t copy(int lane) { return (lane & (COPIES - 1)) * ENTRY; }
    static constexpr int BESIDE = NIB ? 17 : (TWO ? 20 : 16);      // instructions of a step's operands
};

// SKW = 1: a wavefront walks all of K.  SKW = 2 or 4 (layers whose tiles alone would leave SIMDs idle): SKW wavefronts
// of the workgroup share a tile and split K between them (run by run, or in contiguous shares); their sums meet in LDS and each of them
// adds up and stores a share of the tile.
//
// HALF (unshared tiles, Cin % 128 == 64): a filter tap is an odd number of
// 64-position chunks, so the two chunks of a run may lie in different taps -- two different pixels for the loader's two
// lanes of a row, two sets of kept bytes for the run's two halves -- and the last run of K may be half a run, whose
// second chunk is fetched from the first's place and multiplied by kept bytes of zero.
//
// NIB: 3- and 4-bit codes as two 2-bit ones each (dg_onehot_kernel.h, BITS = 24); K and Cin count the 2-bit codes.
//
// TWO: entries beyond int8, T = 256 * hi + lo (dg_onehot_kernel.h).  The planes take the places of two weight row blocks: a
// tile is ONE block of 32 rows, whose words are staged once and whose table indices are worked out once for both planes'
// dense operands; pool words 4 ... 7 are the high plane's rows.
// Registers: the narrow tiles are held to 128 (with two planes and wavefronts taking turns to 168), so that four (three) wavefronts share a SIMD
// and up to 1024 (768) shared tiles are all resident at once.  At 132 - 136 (180) they ran in two rounds: 56x56x128 -> 160 3x3 at batch 4 (980
// tiles) 10.6 us against 9.2, 28x28x1024 -> 160 1x1 at batch 16 8.3 against 7.6, two planes 28x28x1024 -> 256 1x1 at batch 6 (592) 10.1 against
// 8.5.  A spill is no way there: its scratch memory alone costs a launch 0.3 us.
template <int WM, int WN, int SKW, bool TURNS, bool HALF, bool NIB, bool TWO, bool SHORT = false>
__global__ void __launch_bounds__(256, WN > 2 ? 2 : (TWO ? (TURNS ? 3 : 2) : 4))
smfmac_staged_kernel(Args a)
{
    static_assert(!HALF || SKW == 1, "taps of half runs: unshared tiles only");
    static_assert(!SHORT || (WM == 1 && WN == 4 && SKW == 1), "a form of its own for short K: the unshared 32 x 128 tile");
    static_assert(!TWO || (WM == 2 && !NIB), "two planes stand in for two weight row blocks");
    constexpr int RB = TWO ? 1 : WM;                       // weight row blocks of the tile
    constexpr int ROWS = (RB + WN) * 32;                    // staged rows of a wavefront: its weight rows, then its pixels
    constexpr int BUF = ROWS * 32;                          // bytes of one wavefront's buffer
    constexpr int TPW = 4 / SKW;                           // tiles per workgroup
    constexpr int NB = RB * WN;                            // 32x32 output blocks per tile
    constexpr int MN = WM * WN;                            // matrix instructions per parity of a step
    // how many steps ahead the dense operands are made, and how many buffers the runs go round in (three on the wider tiles too: 1 % slower)
    constexpr int AHEAD = MN <= 2 ? 2 : 1, SETS = AHEAD == 2 ? 4 : 2;
    constexpr int BUFS = WN <= 2 ? 3 : 2;
    constexpr bool LATE = WM == 2 && !TWO;                   // (that tile has no registers for a chunk's words beside the next one's)
    // Which table: on narrow tiles, whose operands serve few pixels, its random reads keep LDS busier than the vector instructions they
    // spare are worth (28x28x128 -> 128 3x3 at batch 8, 4-bit codes, 32 x 64 by four: 9.9 us with quads, 9.2 with pairs); with 4-bit slots on
    // the 32 x 128 and 64 x 128 tiles too (28x28x256 -> 256 3x3 at batch 8, 32 x 128 by four: 21.5, 19.5; 28x28x512 -> 256 1x1 at batch 32, unshared:
    // 22.0, 19.3).  SHORT: unshared 32 x 128 tiles where K is short (launch_sparse_staged) pay for filling 16 KB of quads, and beside these a
    // compute unit has room for two workgroups instead of three.  On the others quads are ahead: 8192-cube 740 us with pairs,
    // 706 with quads; 56x56x256 ->
    // 256 3x3 at batch 16, 4-bit, 32 x 224: 98.2, 96.8.
    constexpr bool QUADS = WN >= 4 && !(WN == 4 && NIB) && !SHORT;
    constexpr int LOADS = RB + WN;                          // a run's loads
    constexpr int REGION = SKW > 1 && NB * 4096 > BUFS * BUF ? NB * 4096 : BUFS * BUF;      // a wavefront's: its buffers, then its sums
    typedef std::conditional_t<QUADS, QuadTable<NIB, TWO, (TWO && SKW > 1 ? 2 : 4)>, PairTable<NIB, TWO>> Table;
    // A wavefront's staging rows [buffer][block * 64 + slot] which the sums of a
    // wavefront that shares its tile replace, [block][group of four sum registers][lane]; then the table of rows.
    // A block of 32 rows is 64 slots of 16 bytes, slot j = what loader lane j fetched: row j / 2, segment
    // (j % 2) ^ (j / 16 % 2) of the row's 32 bytes -- the exchange puts rows r and r + 8 of a segment on different
    // LDS banks, which leaves the consumers' reads (32 rows of one segment) two to a bank instead of four.
    static_assert(4 * REGION + Table::BYTES <= 80 * 1024, "two workgroups per compute unit (160 KB of LDS)");
    __shared__ uint4 s_mem[(4 * REGION + Table::BYTES) / 16];
    char *s_table = (char *)s_mem + 4 * REGION;
    // the narrower tiles have the registers for a second set of kept bytes, (0, 1), which spares the odd codes' shift (with two planes: where
    // two wavefronts per SIMD are enough)
    constexpr bool SHIFT_ODD = MN >= 7 || (TWO && WN <= 2 && TURNS);
    const DgProblem &p = a.p;
    typename Table::Entry entry = Table::load(a.pools, threadIdx.x);
    dg_fetch_arguments<sizeof(a)>();
    Table::wait(entry);
    const int lane = threadIdx.x & 63, w4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = w4 % SKW, tw = w4 / SKW;                 // this wavefront's share of K, and its tile within the workgroup
    const int64_t my_tile = (int64_t)xcd_contiguous(blockIdx.x, gridDim.x) * TPW + tw;
    const bool active = my_tile < a.wave_tiles;             // (a wavefront without a tile only joins the barriers)
    const int64_t wave_tile = active ? my_tile : 0;
    const int r = lane & 31, h = lane >> 5;
    // Tiles are numbered in bands of 2^band_log2 pixel tiles; inside a band groups of 2^m_log2 channel tiles (the four
    // wavefronts of a workgroup, which then share their pixels' loads) follow each other along the pixels first.  The
    // tiles in flight on an XCD at one time (consecutive numbers, see xcd_contiguous) then form a patch about as high
    // as it is wide, whose weight rows and pixels that XCD's L2 fetches once (numbered along the channels first, every
    // column of tiles streamed all of the weights through the L2 again: 4.3 times the operands' bytes on an 8192-cube).
    int m_tile, n_tile;
    {
        const uint32_t t = (uint32_t)wave_tile, band = fdiv(t, a.div_band), t_in = t - band * a.band_tiles;
        const uint32_t g = t_in >> a.m_log2, mi = t_in & ((1u << a.m_log2) - 1u);
        const int first = (int)band << a.band_log2, width = min(1 << a.band_log2, a.tiles_n - first);
        uint32_t mg;
        if (width == 1 << a.band_log2)
            mg = g >> a.band_log2;
        else
            mg = fdiv(g, a.div_last);                       // (the last band, narrower)
        n_tile = first + (int)(g - mg * (uint32_t)width);
        m_tile = (int)((mg << a.m_log2) + mi);
    }
    const int m0 = m_tile * (RB * 32), n0 = n_tile * (WN * 32);
    const int cq = p.Cin / 4;                               // packed bytes per pixel
    // This wavefront's runs of K: g0, g0 + stride, ... below g1.  TURNS (layers without a filter window): wavefronts sharing
    // a tile take turns run by run (stride SKW), so that at any time the four of them read the four 32-byte runs of the SAME
    // cache lines -- one fetch into the compute unit's cache serves all; with a contiguous quarter of K each, every
    // wavefront streamed lines of its own, which the cache lost before their next run came up (66 address cycles per
    // load against 34; 8192 x 256 x 8192: 28.7 -> 24.4 us).  With a window they keep contiguous shares: taking turns
    // puts every run of a wavefront in another filter tap, and the kept bytes made anew per run cost more than the
    // cache gives (3x3 layers 7 - 14 % slower).
    static_assert(!TURNS || SKW > 1, "taking turns is for wavefronts that share a tile");
    constexpr int stride = TURNS ? SKW : 1;
    const int runs = HALF ? (p.K + 127) / 128 : p.K / 128;
    const int chunks = p.K / 64, cpt = p.Cin / 64;          // HALF: 64-position chunks in all, and per filter tap
    const int g0 = TURNS ? min(ks, runs) : runs * ks / SKW, g1 = !active ? g0 : (TURNS ? runs : runs * (ks + 1) / SKW);
    const int runs_per_tap = cq / 32;
    const int tap0 = (int)fdiv((uint32_t)g0, a.div_runs), rt0 = g0 - tap0 * runs_per_tap;

    // ---- the loader's side: as a loader, this lane fetches 16-byte segment lseg of row lrow of every 32-row block.  Both operands are
    // read as buffers, whose bounds the hardware checks: rows beyond M, a tap outside the tensor and runs past the end read as zeros
    // without a clamp (a tap outside its image, but inside the tensor, reads whatever lies there: its kept bytes are zero).
    const int lrow = lane >> 1, lseg = (lane & 1) ^ ((lane >> 4) & 1);
    const uint32_t row_bytes = (uint32_t)p.K / 4;
    const v4i w_buffer = dg_buffer(p.Wp + (int64_t)m0 * row_bytes, (uint32_t)min(p.M - m0, RB * 32) * row_bytes);
    const v4i x_buffer = dg_buffer(p.Xp, a.x_bytes);        // (the host sends inputs below 2^31 bytes)
    uint32_t w_ld[RB], x_ld[WN];
#pragma unroll
    for (int bm = 0; bm < RB; ++bm) w_ld[bm] = (uint32_t)(bm * 32 + lrow) * row_bytes + (HALF ? 0 : lseg * 16);
#pragma unroll
    for (int bn = 0; bn < WN; ++bn)
        x_ld[bn] = (uint32_t)make_column(p, a.div_ow, a.div_oh, n0 + bn * 32 + lrow, cq, HALF ? 0 : lseg * 16).off0;
    const uint32_t stage_lds = dg_lds_address(s_mem) + w4 * REGION;
    // filter tap and byte within the pixel of the run fetched next, and its buffer
    int kh = (int)fdiv((uint32_t)tap0, a.div_kw), kw = tap0 - kh * p.KW, cib = rt0 * 32, fetched = g0;
    uint32_t fetch_to = 0;
    auto next_buffer = [](uint32_t b) { return BUFS == 2 ? BUF - b : (b == (BUFS - 1) * BUF ? 0u : b + BUF); };
    auto fetch = [&]() {                                    // this wavefront's next run, into the buffer whose turn it is
        const uint32_t dst = stage_lds + fetch_to;
        fetch_to = next_buffer(fetch_to);
        const bool live = fetched < g1;                     // (uniform; past the end: outside both buffers)
        if constexpr (HALF) {
            // this lane's chunk of the run: 2 g + lseg (past the end of K: the chunk before), its tap and place in it
            const int c0 = 2 * fetched, c1 = min(2 * fetched + 1, chunks - 1);
            auto pixel_offset = [&](int c) {
                const int tap = (int)fdiv((uint32_t)c, a.div_cpt), th = (int)fdiv((uint32_t)tap, a.div_kw);
                return live ? (uint32_t)((th * p.W + (tap - th * p.KW)) * cq + (c - tap * cpt) * 16) : 0x80000000u;
            };
            const uint32_t off0 = pixel_offset(c0), off1 = pixel_offset(c1);
            const uint32_t w_off = live ? (uint32_t)(lseg ? c1 : c0) * 16 : 0x80000000u, x_off = lseg ? off1 : off0;
            dg_for<RB>([&](auto bm) { dg_load16_to_lds<bm * 1024>(w_buffer, w_ld[bm] + w_off, dst); });
            dg_for<WN>([&](auto bn) { dg_load16_to_lds<(RB + bn) * 1024>(x_buffer, x_ld[bn] + x_off, dst); });
            ++fetched;
            return;
        }
        const uint32_t w_off = live ? (uint32_t)fetched * 32 : 0x80000000u;
        dg_for<RB>([&](auto bm) { dg_load16_to_lds<bm * 1024>(w_buffer, w_ld[bm] + w_off, dst); });
        const uint32_t tap_off = live ? (uint32_t)((kh * p.W + kw) * cq + cib) : 0x80000000u;
        // (a tap above the first image is "negative": beyond the buffer's size like what lies past its end)
        dg_for<WN>([&](auto bn) { dg_load16_to_lds<(RB + bn) * 1024>(x_buffer, x_ld[bn] + tap_off, dst); });
        fetched += stride;
        cib += 32 * stride;
        if constexpr (TURNS) {
            while (cib >= cq) cib -= cq;                    // (uniform; no filter window: the tap stays)
        } else if (cib == cq) {                             // (uniform)
            cib = 0;
            if (++kw == p.KW) {
                kw = 0;
                ++kh;
            }
        }
    };
    if (g0 < g1) {                                          // (uniform; the first runs are asked for before anything else is made ready)
        fetch();
        fetch();
    }
    Table::store(s_table, entry, threadIdx.x);
    if (BUFS > 2 && g0 < g1) {                              // (uniform)
#pragma unroll
        for (int i = 2; i < BUFS; ++i) fetch();
    }

    // ---- the consumer's side: row / pixel r (lane half h) of every block; its slot of segment s is slot0 ^ s
    const int slot0 = 2 * r + ((r >> 3) & 1);
    const uint32_t copy = Table::copy(lane);
    // Which rows h0 ... h1 - 1 and columns w0 ... w1 - 1 of the filter window lie inside the image for pixel r of a block (beyond N: none,
    // h1 = h0), as the bytes h0, 128 - h1, w0, 128 - w1: kept_bytes asks for all four bounds with one subtraction.
    uint32_t window[WN];
    int taps_in[WN];
#pragma unroll
    for (int bn = 0; bn < WN; ++bn) {
        const Column c = make_column(p, a.div_ow, a.div_oh, n0 + bn * 32 + r, cq, 0);
        const int h0 = min(max(0, -c.ih0), 127), h1 = c.ok ? max(h0, min(p.KH, p.H - c.ih0)) : h0;
        const int w0 = min(max(0, -c.iw0), 127), w1 = max(w0, min(p.KW, p.W - c.iw0));
        window[bn] = 0x80008000u + (uint32_t)(h0 - (h1 << 8)) + ((uint32_t)(w0 - (w1 << 8)) << 16);
        taps_in[bn] = (h1 - h0) * (w1 - w0);
    }

    v16i acc[WM][WN];
#pragma unroll
    for (int bm = 0; bm < WM; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[bm][bn][e] = 0;
    float sc_cols[RB];
    dg_mfma_column_scales<RB, true>(p, m0, lane, sc_cols);

    // Words of a chunk (64 positions): of weight row r both halves' 8 bytes, of pixel r its own half's.  Lane offsets into a buffer
    // for a run's first chunk; its second chunk's differ in bit 4 (worked out with the buffer's place in one instruction: kept beside
    // the first's, which the compiler would do, they are registers that the narrow tiles do not have).
    const uint32_t w_at = slot0 * 16, x_at = slot0 * 16 + h * 8;
    auto place = [&](uint32_t at, uint32_t buf, int s) -> const char * {
        const uint32_t base = w4 * REGION + buf;            // (a multiple of 1024)
        if (s == 0) return (const char *)s_mem + (at + base);
        uint32_t second;
        asm("v_xad_u32 %0, %1, 16, %2" : "=v"(second) : "v"(at), "s"(base));
        return (const char *)s_mem + second;
    };
    struct Weights {
        uint2 ca[RB], ca1[RB];
    };
    struct Pixels {
        uint2 cb[WN];
    };
    auto read_weights = [&](Weights &w, uint32_t buf, int s) {
        const char *src = place(w_at, buf, s);
#pragma unroll
        for (int bm = 0; bm < RB; ++bm) {
            const uint4 q = *(const uint4 *)(src + bm * 1024);
            w.ca[bm] = make_uint2(q.x, q.y), w.ca1[bm] = make_uint2(q.z, q.w);
        }
    };
    auto read_pixels = [&](Pixels &x, uint32_t buf, int s) {
        const char *src = place(x_at, buf, s);
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) x.cb[bn] = *(const uint2 *)(src + (RB + bn) * 1024);
    };
    const uint32_t pick = sparse_pick(h);
    auto word = [](const uint2 &v, int t) { return t ? v.y : v.x; };
    // the dense operands of all weight blocks (TWO: of both planes) for word t
    auto dense_rows = [&](v8i (&out)[WM][2], const Weights &w, int t) {
#pragma unroll
        for (int u = 0; u < RB; ++u) Table::read(s_table, copy, word(w.ca[u], t), word(w.ca1[u], t), pick, out[u], out[TWO ? 1 : u]);
    };
    v4i ones[WN], ones_odd[SHIFT_ODD ? 1 : WN];
    // which of this lane's pixels see a filter tap: the kept bytes, (1, 0) per position (and (0, 1) for the odd codes),
    // or zeros outside the image (or for a chunk past the end of K)
    auto kept_bytes = [&](int tap, bool live) {
        const int khc = (int)fdiv((uint32_t)tap, a.div_kw), kwc = tap - khc * p.KW;
        // bytes 128 + khc, 255 - khc, 128 + kwc, 255 - kwc: none borrows from the next, and 128 stays of each whose bound holds
        const uint32_t at = 0xFF80FF80u + (uint32_t)khc * 0xFFFFFF01u + ((uint32_t)kwc << 16) - ((uint32_t)kwc << 24);
#pragma unroll
        for (int bn = 0; bn < WN; ++bn) {
            const int x = live && ((at - window[bn]) & 0x80808080u) == 0x80808080u ? 0x00010001 : 0;
            ones[bn] = (v4i){x, x, x, x};
            if constexpr (!SHIFT_ODD) {
                const int y = x << 8;
                ones_odd[bn] = (v4i){y, y, y, y};
            }
        }
    };
    // One step = one word of the chunk: two instructions (even codes, odd codes) per block of the tile, with the dense operands of
    // the next step (or the one after) and the reads of later words -- `beside` -- made between them.
    // (see dg_onehot_kernel.h for the index register and the kept bytes)
    auto step = [&](const v8i (&dn)[WM][2], const Pixels &x, int t, auto &&beside) {
        beside();
        int odd_ix[SHIFT_ODD ? WN : 1];
        if constexpr (SHIFT_ODD) {
#pragma unroll
            for (int bn = 0; bn < WN; ++bn) odd_ix[bn] = (int)(word(x.cb[bn], t) >> 2);
        }
        constexpr int OTHERS = Table::BESIDE * RB + (SHIFT_ODD ? WN : 0) + (WN + 3) / 2;
        constexpr int PER = (OTHERS + 2 * MN - 1) / (2 * MN);      // other instructions per matrix instruction
#pragma unroll
        for (int i = 0; i < 2 * MN; ++i) {
            const int par = i / MN, bm = (i % MN) / WN, bn = i % WN;
            if (par && !SHIFT_ODD)
                acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones_odd[SHIFT_ODD ? 0 : bn], dn[bm][1], acc[bm][bn], (int)word(x.cb[bn], t), 0, 0);
            else
                acc[bm][bn] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(ones[bn], dn[bm][par], acc[bm][bn],
                                                                      par ? odd_ix[SHIFT_ODD ? bn : 0] : (int)word(x.cb[bn], t), 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x102, PER, 0);
        }
    };
    __syncthreads();                                       // (the table)

    if (g0 < g1) {                                          // (uniform; a wavefront without a share of K only joins the barriers)
        // The sums start at zero, or -- the table's entries having been raised by a.bias to make them all small and
        // non-negative (launch_sparse_staged says why) -- at minus the bias for every position of K the pixel really
        // sees: Cin per filter tap inside the image.  Lane (r, .) works that out for pixel r of a block; sum register
        // e of a lane belongs to pixel 8 (e / 4) + 4 h + e % 4 and takes it from that lane.  Of the wavefronts sharing
        // a tile one that surely has a share of K does this.  Done here, while the first runs are on their way.
        if (a.bias != 0 && ks == (TURNS ? 0 : SKW - 1)) {                       // (uniform)
#pragma unroll
            for (int bn = 0; bn < WN; ++bn) {
                const int start = -a.bias * p.Cin * taps_in[bn];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int v = __builtin_amdgcn_ds_bpermute(4 * (8 * (e / 4) + 4 * h + e % 4), start);
#pragma unroll
                    for (int bm = 0; bm < WM; ++bm) acc[bm][bn][e] = v;
                }
            }
        }
        Weights w0, w1;                                     // of the run's first and second chunk
        Pixels x0, x1;
        v8i dn[SETS][WM][2];
        uint32_t cur = 0, nxt = BUFS > 1 ? BUF : 0;         // the buffers of this run and the next
        dg_wait_for_loads<(BUFS - 1) * LOADS>();
        read_weights(w0, cur, 0);
        if constexpr (AHEAD == 2) read_weights(w1, cur, 1);
        read_pixels(x0, cur, 0);
        dense_rows(dn[0], w0, 0);
        if constexpr (AHEAD == 2) dense_rows(dn[1], w0, 1);
        // run g, whose first chunk's words and operands (both steps' where they are made two ahead) are at hand
        auto run = [&](int g) {
            if constexpr (AHEAD == 2) {
                step(dn[0], x0, 0, [&]() { read_pixels(x1, cur, 1), dense_rows(dn[2], w1, 0); });
                dg_wait_for_loads<(BUFS - 2) * LOADS>();       // the next run is in
                step(dn[1], x0, 1, [&]() { read_weights(w0, nxt, 0), dense_rows(dn[SETS - 1], w1, 1); });
            } else {
                step(dn[0], x0, 0, [&]() {
                    if (LATE) dense_rows(dn[1], w0, 1);
                    read_weights(w1, cur, 1);
                    if (!LATE) read_pixels(x1, cur, 1), dense_rows(dn[1], w0, 1);
                });
                step(dn[1], x0, 1, [&]() {
                    dense_rows(dn[0], w1, 0);
                    if (LATE) read_pixels(x1, cur, 1);
                });
                dg_wait_for_loads<(BUFS - 2) * LOADS>();
            }
            // (the second chunk's kept bytes take the first's registers)
            if constexpr (HALF) kept_bytes((int)fdiv((uint32_t)min(2 * g + 1, chunks - 1), a.div_cpt), 2 * g + 1 < chunks);
            if constexpr (AHEAD == 2)
                step(dn[SETS - 2], x1, 0, [&]() { read_pixels(x0, nxt, 0), read_weights(w1, nxt, 1), dense_rows(dn[0], w0, 0); });
            else
                step(dn[0], x1, 0, [&]() {
                    if (LATE) dense_rows(dn[1], w1, 1);
                    read_weights(w0, nxt, 0);
                    if (!LATE) read_pixels(x0, nxt, 0), dense_rows(dn[1], w1, 1);
                });
            // This run's words have all been read and used: its buffer takes the run BUFS after it.
#pragma unroll
            for (int bn = 0; bn < WN; ++bn) asm volatile("" ::"v"(x1.cb[bn].x), "v"(x1.cb[bn].y));
            if constexpr (AHEAD == 1 && !LATE) {             // (LATE: those words' operands are made first of all in the step above)
#pragma unroll
                for (int bm = 0; bm < RB; ++bm) asm volatile("" ::"v"(w1.ca[bm].x), "v"(w1.ca1[bm].y));
            }
            fetch();
            step(dn[SETS - 1], x1, 1, [&]() {
                dense_rows(dn[AHEAD - 1], w0, AHEAD - 1);
                if (LATE) read_pixels(x0, nxt, 0);
            });
            cur = nxt;
            nxt = next_buffer(nxt);
        };
        if constexpr (HALF) {
            for (int g = g0; g < g1; ++g) {
                kept_bytes((int)fdiv((uint32_t)(2 * g), a.div_cpt), true);
                run(g);
            }
        } else if constexpr (TURNS) {
            kept_bytes(tap0, true);
            for (int g = g0; g < g1; g += stride) run(g);
        } else {
            int g = g0, first = rt0;
            for (int tap = tap0; g < g1; ++tap, first = 0) {
                kept_bytes(tap, true);
                const int end = min(g + runs_per_tap - first, g1);
                for (; g < end; ++g) run(g);
            }
        }
        dg_wait_for_loads();                                   // (unused fetches past the end: their LDS writes end before the wavefront does)
    }
    if (SKW == 1 && !active) return;                       // (whole wavefronts; no barrier follows on this path)
    // (this lane's number once more, which takes no register of the walk's)
    const int lane_out = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    // (The scales are in: said here, or the compiler, which cannot tell across the stores' branches, waits for them -- and with them for
    // every store before -- again at each group of stores.)
#pragma unroll
    for (int bm = 0; bm < RB; ++bm) asm volatile("" : "+v"(sc_cols[bm]));
    // the tile's blocks as they go to memory: two planes merge into one block row, 256 * hi + lo
    v16i out[RB][WN];
#pragma unroll
    for (int bm = 0; bm < RB; ++bm)
#pragma unroll
        for (int bn = 0; bn < WN; ++bn)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                out[bm][bn][e] = TWO ? (int)((uint32_t)acc[0][bn][e] + ((uint32_t)acc[WM - 1][bn][e] << 8)) : acc[bm][bn][e];
    if (SKW == 1) {
        dg_mfma_store_tile<RB, WN, true, true, DG_OUT_BY_PROBLEM>(p, out, m0, n0, lane_out, sc_cols);
        return;
    }
    // Every wavefront's sums take the place of its own staging rows (its last loads have landed), 16 bytes per lane and group of four
    // sum registers; once all are there, each wavefront of the tile adds up and stores a share of the groups: 8 rows of
    // 32 channels each.  (The sums met by atomic additions before, with two barriers more, and with two blocks two of four wavefronts stored.)
    uint4 *const mine = s_mem + w4 * (REGION / 16) + lane_out;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v16i &b = out[i / WN][i % WN];
            mine[(4 * i + q) * 64] = make_uint4(b[4 * q], b[4 * q + 1], b[4 * q + 2], b[4 * q + 3]);
        }
    __syncthreads();
    if (!active) return;
    const uint4 *const theirs = s_mem + (w4 - ks) * (REGION / 16) + lane_out;
    static_assert(SKW == 1 || RB == 1, "a share's blocks are one row of blocks");
    constexpr int GROUPS = NB * 4 / SKW, NQ = GROUPS < 4 ? GROUPS : 4;        // this wavefront's, and those of a block among them
#pragma unroll
    for (int j = 0; j < GROUPS / NQ; ++j) {
        const int first = ks * GROUPS + j * NQ, i = first / 4, q0 = first % 4;
        v4i sum[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            sum[q] = (v4i){0, 0, 0, 0};
#pragma unroll
            for (int w = 0; w < SKW; ++w) {
                const uint4 t = theirs[w * (REGION / 16) + (first + q) * 64];
                sum[q] += (v4i){(int)t.x, (int)t.y, (int)t.z, (int)t.w};
            }
        }
        dg_mfma_store_quads<NQ>(p, sum, q0, m0, n0 + i * 32, lane_out, sc_cols[0]);
    }
}

// `wave_tiles` tiles of q.wm x q.wn blocks, 4 / q.skw of them per workgroup
//
// `bias`: the caller added it to every entry of the table in `pools` (0: the table as it is).  The matrix pipe's power
// draw, and with it the clock the chip sustains, follows the bits that toggle in its operands and sums: the same
// 8192-cube takes 550 us with an all-zero table, 640 us with entries 0 ... 9, 700 us with -6 ... 3 and 800 us with
// -64 ... 64.  A table raised to 0 ... max - min keeps the high bits of the dense operand and of the growing sums
// quiet; the kernel starts each sum at minus the bias times the pixel's positions of K, so the result is the same.
template <bool NIB, bool TWO>
void launch_sparse_staged(const DgProblem &p, const Pools &pools, int32_t bias, const Plan &q, int64_t wave_tiles, hipStream_t stream)
{
    Args a;
    a.p = p;
    a.p.cached = dg_output_cached(p);
    a.pools = pools;
    a.bias = bias;
    a.x_bytes = (uint32_t)((int64_t)p.N / ((int64_t)p.OH * p.OW) * p.H * p.W * (p.Cin / 4));
    const int rows = TWO ? 32 : q.wm * 32;                 // (two planes: q.wm = 2 blocks of the same 32 rows)
    a.tiles_m = (p.M + rows - 1) / rows;
    a.wave_tiles = wave_tiles;
    a.div_ow = make_div((uint32_t)p.OW), a.div_oh = make_div((uint32_t)p.OH);
    a.div_cin = make_div((uint32_t)p.Cin), a.div_kw = make_div((uint32_t)p.KW);
    const bool half = p.Cin % 128 != 0;                    // (see the kernel: taps of an odd number of 64-position chunks)
    a.div_runs = make_div((uint32_t)(half ? 1 : p.Cin / 128));
    a.div_cpt = make_div((uint32_t)(p.Cin / 64));
    a.tiles_n = (int32_t)((p.N + q.wn * 32 - 1) / (q.wn * 32));
    a.band_log2 = 3;                                       // bands of 8 pixel tiles
    a.m_log2 = a.tiles_m % 4 == 0 ? 2 : 0;                 // (unshared tiles: a workgroup's four wavefronts)
    a.band_tiles = (uint32_t)a.tiles_m << a.band_log2;
    a.div_band = make_div(a.band_tiles);
    const int last = a.tiles_n & ((1 << a.band_log2) - 1);
    a.div_last = make_div((uint32_t)(last ? last : 1));
    const int tpw = 4 / q.skw;
    const dim3 grid((unsigned)((wave_tiles + tpw - 1) / tpw));
    const bool turns = p.KH * p.KW == 1;                   // (see the kernel: run by run without a filter window)
#define DG_STAGED(WM, WN, SKW, TURNS) hipLaunchKernelGGL((smfmac_staged_kernel<WM, WN, SKW, TURNS, false, NIB, TWO>), grid, dim3(256), 0, stream, a)
    if constexpr (TWO) {
        if (half) hipLaunchKernelGGL((smfmac_staged_kernel<2, 2, 1, false, true, NIB, TWO>), grid, dim3(256), 0, stream, a);
        else if (q.wn == 4 && q.skw == 1) DG_STAGED(2, 4, 1, false);
        else if (q.wn == 4 && q.skw == 2 && turns) DG_STAGED(2, 4, 2, true);
        else if (q.wn == 4 && q.skw == 2) DG_STAGED(2, 4, 2, false);
        else if (q.wn == 4 && turns) DG_STAGED(2, 4, 4, true);
        else if (q.wn == 4) DG_STAGED(2, 4, 4, false);
        else if (q.skw == 1) DG_STAGED(2, 2, 1, false);
        else if (turns) DG_STAGED(2, 2, 4, true);
        else DG_STAGED(2, 2, 4, false);
    } else {
        if (half && q.wn == 4) hipLaunchKernelGGL((smfmac_staged_kernel<1, 4, 1, false, true, NIB, false>), grid, dim3(256), 0, stream, a);
        else if (half) hipLaunchKernelGGL((smfmac_staged_kernel<1, 2, 1, false, true, NIB, false>), grid, dim3(256), 0, stream, a);
        else if (q.wm == 2) DG_STAGED(2, 4, 1, false);
        else if (q.wn == 7) DG_STAGED(1, 7, 1, false);
        else if (q.wn == 6) DG_STAGED(1, 6, 1, false);
        else if (q.wn == 4 && q.skw == 4 && turns) DG_STAGED(1, 4, 4, true);
        else if (q.wn == 4 && q.skw == 4) DG_STAGED(1, 4, 4, false);
        else if (q.wn == 4 && q.skw == 2 && turns) DG_STAGED(1, 4, 2, true);
        else if (q.wn == 4 && q.skw == 2) DG_STAGED(1, 4, 2, false);
        else if (q.wn == 4) {
            // K below 2304 and output rows of whole cache lines: the table of pairs (the kernel's SHORT form).  With quads, with pairs: 56x56x128 -> 128
            // 3x3 at batch 16 16.6 us, 16.2; 128x96000x512 17.5, 16.1; 8192x4096x384 41.5, 38.3; 1920x5856x640 19.7, 18.3; 96x43936x1152 16.0, 15.4.
            // Other rows: 1919x5832x640 26.4, 27.4, 56x56x128 -> 100 3x3 at batch 20 20.4, 21.6, eight more within 1 %.  K from 2304 up:
            // 1611x4573x2816 43.3, 45.6; 14x14x512 -> 512 3x3 at batch 50 34.7, 35.3; 1536x4480x4096 44.7, 44.9.
            if (!NIB && p.K < 2304 && p.stride_cn % 32 == 0)
                hipLaunchKernelGGL((smfmac_staged_kernel<1, 4, 1, false, false, NIB, false, !NIB>), grid, dim3(256), 0, stream, a);
            else DG_STAGED(1, 4, 1, false);
        } else if (q.skw == 4 && turns) DG_STAGED(1, 2, 4, true);
        else if (q.skw == 4) DG_STAGED(1, 2, 4, false);
        else if (q.skw == 2 && turns) DG_STAGED(1, 2, 2, true);
        else if (q.skw == 2) DG_STAGED(1, 2, 2, false);
        else DG_STAGED(1, 2, 1, false);
    }
#undef DG_STAGED
}

}   // namespace dgoh
