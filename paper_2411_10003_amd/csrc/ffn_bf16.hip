// Grouped expert FFN in bf16 with fp32 accumulation on the gfx950 matrix cores (Section 4.2 of
// the paper: forward and backward expert computation over the inputs a device hosts).
//
// Every contraction of the forward and backward pass is one launch of the same tiled kernel:
//   fwd1  Z(,U) = Xp W1(,W3)        epilogue: Z, U, Act = act(Z)(*U)
//   fwd2  Yp    = Act W2
//   bwd1  dA    = dYp W2^T          epilogue: dZ (,dU), Act recomputed from the saved Z (,U)
//   bwd2  dXp   = dZ W1^T (+ dU W3^T)
//   wgrad dW1 = Xp^T dZ, dW3 = Xp^T dU, dW2 = Act^T dYp over the rows of each group
// Groups are ragged and may be empty; row tiles start at the group's first row and the last one
// is masked, so nothing is padded to the largest load.  The kernel is persistent: one block per
// CU (two of the small geometry) walks its share of the tiles, which it derives on the device from
// the group offsets (the host never reads the counts).
//
// Tiling: 256 x 256 output tile per block (128 x 128 where those leave the chip idle, see GeometryCost), 32-deep
// contraction slices moved from HBM/L2 straight into a 5-deep ring of LDS buffers by buffer loads (no
// register staging; rows outside a ragged group arrive as zeros because they lie past the end of the buffer resource), 16x16x32 bf16 MFMA
// with the accumulators in AGPRs.  An operand whose contraction index is contiguous in memory is
// kept row-major in LDS and read with 16-byte loads; one whose contraction index is the slow one
// is kept as it is and read with the transposing LDS load, so no operand is ever transposed in
// HBM.  Both layouts are XOR-swizzled so that fragment reads are free of bank conflicts.  Every
// request to L2 is a whole 128-byte line: a K-contiguous operand is therefore fetched two slices
// at a time for half of the tile's rows (128 rows x 64 steps per ring buffer), a K-major one a
// slice at a time (32 steps x 256 columns); the L2 channels, not HBM, are what the loop queues at
// when the same bytes are asked for in 64-byte pieces.  The MFMA
// is issued with the operands swapped, which leaves every lane with four consecutive output
// columns of one row.  The two rows of waves of a block alternate between fetching fragments and
// multiplying, half an iteration apart.
#include "internal.h"
#include <type_traits>
#include <algorithm>
#include <cmath>
#include <numeric>

// Where the main loop starts relative to a 256-byte boundary of the code, in 4-byte steps (LOOP_OFF: the weight gradients, LOOP_OFF_P: the
// others).  The loop is one basic block that every wave runs tens of thousands of times, and how its two phases fall into the
// instruction fetch windows changes its time, so the placement is fixed instead of being left to what precedes the loop.  With
// 32x32x16 instructions the weight gradients changed by 6 % from the best to the worst placement (period: 32 bytes) and 4 was the best.
// With the 16x16x32 loop 0 .. 7 change forward and backward together, against 4, by -0.55, -0.50, -0.61, -0.32, 0, -0.41, -0.49, -0.50 %
// (d = 4096, h = 14336, SwiGLU; d = 2048, h = 8192, GELU: -0.20, -0.02, -0.31, -0.16, 0, -0.20, -0.24, -0.14), a third of which is weight
// gradients; LOOP_OFF_P by less than 0.25 either way.
#ifndef LOOP_OFF
#define LOOP_OFF 4
#endif
#define LOOP_OFF_STR2(x) #x
#define LOOP_OFF_STR1(x) LOOP_OFF_STR2(x)
#define LOOP_OFF_STR LOOP_OFF_STR1(LOOP_OFF)
#ifndef LOOP_OFF_P
#define LOOP_OFF_P 4
#endif
#define LOOP_OFF_P_STR LOOP_OFF_STR1(LOOP_OFF_P)

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
#define LDS_PTR(T) __attribute__((address_space(3))) T*

enum Kind { KIND_NN = 0, KIND_NT = 1, KIND_TN = 2 };
enum Epi { EPI_BF16 = 0, EPI_F32 = 1, EPI_FWD1_GELU = 2, EPI_FWD1_SWIGLU = 3, EPI_BWD1_GELU = 4, EPI_BWD1_SWIGLU = 5 };

struct GemmParams {
    // contraction segments (bwd2 of SwiGLU has two: dZ W1^T + dU W3^T)
    const bf16_t* A[2];
    const bf16_t* B[2];
    const bf16_t* B_dual;        // fwd1 SwiGLU: second weight matrix read beside B[0]
    long lda, ldb;               // leading dimensions in elements
    long b_group_stride;         // elements between the weight matrices of consecutive groups (0 for TN)
    int n_seg, Kseg;             // NN/NT: contraction length per segment
    int Mout, N;                 // TN: output rows; all kinds: output columns
    const int32_t *slot_offsets, *dest_slots;
    int self, Gcap;
    int row_tiles, col_tiles;    // tile counts (row_tiles is an upper bound for NN/NT)
    int band;                    // row tiles per band of the tile walk (a round of 32 tiles is band x 32/band)
    int n_tiles;
    // outputs
    bf16_t *O0, *O1, *O2;        // EPI_BF16: O0.  FWD1: Z, U, Act.  BWD1: dZ, dU, Act
    float* OF;                   // EPI_F32
    int accumulate;              // EPI_F32: add to the output instead of overwriting it
    long ldo, o_group_stride;
    const bf16_t *Zin, *Uin;     // BWD1: saved pre-activations
    int write_act;               // BWD1: recompute the activation into O2 (0: the forward pass's copy is still there)
    float* split_ws;             // partial tiles of split contractions, [unit][wave][registers][64 lanes]; null: none is split
    int split_cap;               // units that fit there
    int tn_over;                 // TN: what a tile costs beside its slices, in slices
    int split_max, split_slices; // parts of a tile at most, slices of a part at least
    int uneven_cap;              // units an uneven cut may use (0: none is made)
    int* arrived;                // uneven cut: parts of a tile that have been stored, a counter per tile; all zero between two launches
    int clear_arrived;           // the first launch of a call: make them so
};

// Row contractions whose tiles may be cut unevenly, the part that is done last finishing its tile.  The counters that takes are
// cleared by the first launch of a call (fwd1, bwd1), which therefore has no such tiles itself.
constexpr bool last_finishes(int epi) { return epi == EPI_BF16; }

// How contractions are cut, for the kernel (which alone knows the rows) and for moe_ffn_tiling (which is told them).
// NN/NT: parts of each of the `rem` tiles left over after the last full round of `nblk` blocks.
__host__ __device__ inline int row_parts(int rem, int nblk, int slices, int split_max, int split_slices, int split_cap)
{
    if (rem <= 0) return 1;
    const int fill = nblk / rem, worth = slices / split_slices;    // a part has to be worth its round trip
    int S = fill < split_max ? fill : split_max;
    if (S > worth) S = worth > 1 ? worth : 1;
    return rem * S > split_cap ? 1 : S;
}
// NN/NT, epilogues of last_finishes: where the tiles left over are more than half of the blocks (and stay whole by the rule
// above), each keeps a block for its first slices and the other blocks share the rest, `turns` remainders each.  Returns the
// first slices (0: the tiles stay whole).  A remainder costs its block about UNEVEN_OVER slices beside its own (ring filled,
// 256 KB stored), and the block that finishes a tile about as much again to add it, so a remainder has to be worth twice that.
constexpr int UNEVEN_OVER = 14, UNEVEN_SLICES = 28;
__host__ __device__ inline int uneven_cut(int rem, int nblk, int slices, int cap, int& turns)
{
    const int others = nblk - rem;
    turns = 0;
    if (rem <= others || others <= 0 || 2 * rem > cap) return 0;
    turns = (rem + others - 1) / others;
    const int rest = (slices - turns * UNEVEN_OVER) / (turns + 1) & ~1;
    return rest >= UNEVEN_SLICES ? slices - rest : 0;
}
// TN: parts of a group of k slices.  Its rounds (a round: as many tiles as an XCD has blocks, or what there are) run on one
// XCD each, so cutting it shortens the whole only where it is longer than an XCD's share of all rounds; the parts are then
// about as long as a block's share of all tiles, and no shorter than split_slices.  tiles, rounds: of a group; slices: of all.
// n_cut groups are cut into at most what the workspace holds and, where all parts would be more than the 64 lanes that keep
// them, an equal number of the lanes left beside one for each group.
__host__ __device__ inline int tn_parts(int k, int tiles, int rounds, int slices, int groups, int nblk, int tn_over, int split_max, int split_slices)
{
    const long all = slices + (long)groups * tn_over;
    const int xcd_share = (int)(rounds * all / 8), share = (int)(tiles * all / nblk);
    if (k == 0 || k + tn_over <= xcd_share + xcd_share / 4) return 1;      // an empty group is one part: its zeros
    const int len = share - tn_over > split_slices ? share - tn_over : split_slices;
    const int n = (k + len - 1) / len;
    return n < split_max ? n : split_max;
}
__host__ __device__ inline int tn_most_units(int split_cap, int tiles, int n_cut) { const int n = split_cap / (tiles * n_cut); return n > 1 ? n : 1; }
__host__ __device__ inline int tn_most_lanes(int groups, int n_cut) { return 1 + (64 - groups) / n_cut; }
// Whether the cut is worth its finishing launch (about what a tile costs beside its slices): the longest chain, or the rounds
// of the busiest XCD at the mean length, with n groups whole (the longest of k slices) and as `parts` of at most `len`.
__host__ __device__ inline bool tn_pays(int k, int len, int slices, int n, int parts, int rounds, int tn_over)
{
    const int whole = (n * rounds + 7) / 8 * (slices / n + tn_over), cut = (parts * rounds + 7) / 8 * (slices / parts + tn_over);
    return (cut > len + tn_over ? cut : len + tn_over) + tn_over < (whole > k + tn_over ? whole : k + tn_over);
}

// GELU (Eq. 2 with the Gaussian CDF) and its derivative from one exponential and one reciprocal: erf by the
// five-term rational approximation of Abramowitz & Stegun 7.1.26 (absolute error below 1.5e-7, two orders under
// what a bf16 output resolves), whose exp(-x^2) at x = z / sqrt(2) is also the density the derivative needs.  The
// library erff is some thirty instructions with branches, per element of an epilogue that the matrix cores wait for.
// Relative to GELU the error is 0.35 % at z = -6 and 2.0 % at -10 (the derivative's 2e-4).  exp2 of a polynomial in |z| takes 11 vector
// instructions for these 18 (a forward layer of d = 1024, h = 4096, 9279 rows 225 us for 232, training of d = 2048, h = 8192, 29112 rows
// 4650 for 4667), but fitted on [0, 5] it is off by 4 % at -6 and 78 % at -8; fitted up to -10 it is not, and either leaves the gate's
// bias gradient 1 to 2 % further from 64 bits than this (T = 16384, 64 experts, k = 1) and the other results where they are.
struct gelu_parts { float cdf, pdf; };                     // Phi(z) and phi(z)
__device__ __forceinline__ gelu_parts gelu_terms(float z)
{
    const float x = z * 0.70710678118654752f, ax = __builtin_fabsf(x);
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, ax, 1.0f));
    const float e = __expf(-(ax * ax));                    // exp(-z^2 / 2)
    float y = __builtin_fmaf(1.061405429f, t, -1.453152027f);
    y = __builtin_fmaf(y, t, 1.421413741f);
    y = __builtin_fmaf(y, t, -0.284496736f);
    y = __builtin_fmaf(y, t, 0.254829592f);
    const float half_erfc = 0.5f * (y * t) * e;            // (1 - erf|x|) / 2
    gelu_parts r;
    r.cdf = z < 0.0f ? half_erfc : 1.0f - half_erfc;
    r.pdf = 0.3989422804014327f * e;
    return r;
}
__device__ __forceinline__ float gelu_f(float z) { return z * gelu_terms(z).cdf; }
__device__ __forceinline__ float gelu_grad_f(float z) { const gelu_parts g = gelu_terms(z); return __builtin_fmaf(z, g.pdf, g.cdf); }
// exp and reciprocal are one instruction each (1 ulp); a full-precision division would be a dozen per element of an
// epilogue whose vector instructions are what the matrix cores wait for between two tiles
__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// Tile geometries.  Contraction slices of 32 are staged through a ring of LDS buffers.
//   Large: 256 x 256 outputs per block of 8 waves of 128 x 64, one block per CU (a 5-deep ring of 32 KB: all of LDS).
//   Small: 128 x 128 outputs per block of 4 waves of 64 x 64, two blocks per CU (5-deep rings of 16 KB).
constexpr int BK = 32;
template <int WGM_, int WGN_, int TM_, int TN_, int STAGES_, int BLOCKS_> struct Geometry {
    static constexpr int WGM = WGM_, WGN = WGN_, TM = TM_, TN = TN_, STAGES = STAGES_, BLOCKS = BLOCKS_;
    static constexpr int NWAVES = WGM * WGN, THREADS = NWAVES * 64;
    static constexpr int WM = 32 * TM, WN = 32 * TN, BM = WM * WGM, BN = WN * WGN;
    static constexpr uint32_t A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int PA = A_BYTES / 1024 / NWAVES, PB = B_BYTES / 1024 / NWAVES;   // 1-KB DMA pieces per wave and slice
    static constexpr int EP_PITCH = WN * 4 + 16;           // epilogue patch: bytes per staged row of WN floats (padded against bank conflicts)
    static constexpr int EP_ROWS = 32;                     // rows a wave stages at a time: two rows of fragments
    static constexpr int EP_WAVE = EP_ROWS * EP_PITCH;
    static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE_BYTES;
    static constexpr bool TWO_PHASE = BLOCKS == 1;         // the rows of waves of a block alternate; else the blocks of a CU do
    static constexpr int UNIT_BYTES = BM * BN * 4;         // a partial tile of a K-split round
    static_assert(LDS_BYTES >= (size_t)NWAVES * EP_WAVE && BLOCKS * LDS_BYTES <= 160 * 1024, "patches inside the ring, rings inside LDS");
    static_assert(WGM == 2 && WGN % 2 == 0, "the two halves of a K-contiguous operand's rows belong to one row of waves or half the columns");
};
typedef Geometry<2, 4, 4, 2, 5, 1> Large;
typedef Geometry<2, 2, 2, 2, 5, 2> Small;

// Row tiles per band of the tile walk, per contraction.  Measured, us, 3 | 5 | 6 | 7 | 8 | 16 row tiles: fwd1 at d = 4096, h = 14336,
// SwiGLU 7990 | 8020 | 7950 | 7920 | 8125 | 8245 (and fwd2 after it 3670 | 3645 | 3640 | 3685 | 3600 | 3590), bwd1 4245 | 4295 | 4315 |
// 4265 | 4350 | 4494; forward and backward against 7 there, 8 for both +0.39 %, 16 and 8 +0.58; d = 2048, h = 8192, GELU +0.15 and +0.22, the
// size of the spread, fwd1 883 | 879 | 875 | 871 | 873 | 872 (GELU as a polynomial), bwd1 893 | 888 | 890 | 889 | 903 | 909; the others
// are best at 8, which is what the L2 of an XCD needs least fills for (4: weight gradients +0.8 %, 16: +1 % and more).
#ifndef BAND_FWD1
#define BAND_FWD1 7
#endif
#ifndef BAND_FWD2
#define BAND_FWD2 8
#endif
#ifndef BAND_BWD1
#define BAND_BWD1 7
#endif
#ifndef BAND_BWD2
#define BAND_BWD2 8
#endif
#ifndef BAND_WGRAD
#define BAND_WGRAD 8
#endif
// ---- LDS layouts (byte offsets inside one operand buffer) --------------------------------------
// K-contiguous operand (NN and NT fetch it in whole 128-byte lines): a buffer holds 128 rows x 64 steps (two
// slices of 32), 128 bytes per row, its eight 16-byte pieces XOR-swizzled by the row so that 16 consecutive rows of
// one piece cover all banks.
__device__ __forceinline__ uint32_t halfpair_off(int row, int piece8) { return row * 128 + ((piece8 ^ ((row >> 1) & 7)) << 4); }
// K-major operand, 32 steps x COLS columns: two steps beside each other, 64 columns (a 128-byte line of memory) of one and of
// the other in turn, the four 16-column chunks of a line XOR-swizzled by bits 1 and 3 of the step.  A transposing load takes
// four steps of every lane block, and its lane blocks are eight steps apart: the eight steps that 32 lanes touch differ in
// bits 0, 1 and 3, and their chunks of one column group cover all banks.
__device__ __forceinline__ int kmajor_swizzle(int krow) { return ((krow >> 1) & 1) | ((krow >> 2) & 2); }
template <int COLS>
__device__ __forceinline__ uint32_t kmajor_off(int krow, int col)
{
    return (krow >> 1) * (COLS * 4) + (col >> 6) * 256 + (krow & 1) * 128 + ((((col >> 4) & 3) ^ kmajor_swizzle(krow)) << 5) + (col & 15) * 2;
}
// The inverse for the DMA: byte offset in memory of the 16-byte piece that belongs at slot L of such a buffer.
template <int COLS>
__device__ __forceinline__ uint32_t kmajor_source(int L, long ld)
{
    constexpr int PER_PAIR = COLS / 4;                     // slots of two steps
    const int in_pair = L % PER_PAIR, part = L & 7, krow = L / PER_PAIR * 2 + ((in_pair >> 3) & 1);
    const int col = (in_pair >> 4) * 64 + (((part >> 1) ^ kmajor_swizzle(krow)) << 4) + (part & 1) * 8;
    return (uint32_t)((krow * ld + col) * 2);
}

// Fragment = 16 rows (or columns) x 32 contraction steps; lane l holds row l%16, steps 8*(l/16)..+7.
// Fragment reads are issued as assembly and waited for by hand (WAIT_FRAGS below): the compiler's
// own wait insertion cannot express "the set loaded one iteration ago is complete" and would stall
// every MFMA group on the fragments that were only just requested for the next iteration.
template <int IMM>
__device__ __forceinline__ void lds_frag_kcontig_at(bf16x8& f, uint32_t addr)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f) : "v"(addr), "n"(IMM));
}
// The transposing load works on blocks of 16 lanes: lane s of a block points at 4 consecutive columns
// of step s/4; lane i of the block receives column i of steps 0..3.  Two loads give the 8 steps of a
// lane in the same order as the K-contiguous fragment.  IMM: a constant distance added to the address.
template <int STEP4_BYTES, int IMM>
__device__ __forceinline__ void lds_frag_kmajor_at(bf16x8& f, uint32_t addr)
{
    s16x4 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                 : "=&v"(lo), "=&v"(hi) : "v"(addr), "n"(IMM), "n"(IMM + STEP4_BYTES));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    f = __builtin_bit_cast(bf16x8, v);
}

typedef __attribute__((ext_vector_type(4))) int rsrc_t;     // raw buffer resource (4 scalar registers)
typedef __amdgpu_buffer_rsrc_t buf_rsrc_t;                   // the same thing as the store builtin wants it
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, long long bytes)
{
    if (bytes < 0) bytes = 0;
    if (bytes > 0xffffffffll) bytes = 0xffffffffll;
    const unsigned long long b = (unsigned long long)base;
    rsrc_t r;
    r[0] = (int)(unsigned)(b & 0xffffffffull);
    r[1] = (int)(unsigned)((b >> 32) & 0xffffull);         // stride 0: raw buffer, byte offsets
    r[2] = (int)(unsigned)bytes;                           // bytes past this limit read as zero
    r[3] = 0x00020000;
    return r;
}

// 16 bytes per lane from a buffer straight into LDS at lds_base + lane*16 (lds_base is uniform and
// goes through M0); bytes past the end of the buffer arrive as zeros.  Issued as assembly so that
// the compiler does not serialise later LDS reads of other ring slots behind it; completion is
// tracked by hand with WAIT_VMCNT before the barrier that publishes the slot.
template <bool NT = false>
__device__ __forceinline__ void dma16(rsrc_t r, uint32_t lds_base, uint32_t voff, uint32_t soff)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                     :: "s"(lds_base), "v"(voff), "s"(r), "s"(soff) : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds_base), "v"(voff), "s"(r), "s"(soff) : "memory");
}

#define WAIT_VMCNT(n) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(n) : "memory")
#define BLOCK_BARRIER() asm volatile("s_barrier" ::: "memory")


// ---- the kernel ---------------------------------------------------------------------------------
// LAST: tiles may be cut unevenly.  Contractions that are too short for it run without that code (d = 256, h = 896, 80 rows: 0.5 and
// 0.8 us of 14 and 12 more with it).
// ONCE: the weights are read by one block and not again while the caches keep them (read_once): nontemporal requests.
template <int KIND, int EPI, bool FIN, class GEO, bool LAST, bool ONCE>
__global__ __launch_bounds__(GEO::THREADS, GEO::BLOCKS * GEO::NWAVES / 4) void grouped_gemm_kernel(const GemmParams p)
{
    constexpr int WGN = GEO::WGN, NWAVES = GEO::NWAVES, WM = GEO::WM, WN = GEO::WN, BM = GEO::BM, BN = GEO::BN, TM = GEO::TM, TN = GEO::TN;
    constexpr int STAGES = GEO::STAGES, PA = GEO::PA, PB = GEO::PB, EP_PITCH = GEO::EP_PITCH, EP_ROWS = GEO::EP_ROWS, EP_WAVE = GEO::EP_WAVE;
    constexpr uint32_t A_BYTES = GEO::A_BYTES, STAGE_BYTES = GEO::STAGE_BYTES;
    constexpr size_t LDS_BYTES = GEO::LDS_BYTES;
    constexpr bool A_KMAJOR = (KIND == KIND_TN);
    constexpr bool B_KMAJOR = (KIND != KIND_NT);
    constexpr bool DUAL = (EPI == EPI_FWD1_SWIGLU);
    static_assert(!LAST || (last_finishes(EPI) && !FIN), "counters are there, and parts are left to no other launch");
    static_assert(!DUAL || (TN % 2 == 0), "dual-B needs an even number of column fragments per wave");

    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_PTR(unsigned char))smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    if (!FIN && p.clear_arrived)
        for (int i = blockIdx.x * GEO::THREADS + tid; i < SPLIT_COUNTERS; i += gridDim.x * GEO::THREADS) p.arrived[i] = 0;

    // ---- group table, once per block: lane i of every wave holds hosted group i (at most 64 groups)
    int first_slot, n_groups;
    hosted_range(p.dest_slots, p.self, p.Gcap, first_slot, n_groups);
    int g_row0 = 0, g_rows = 0;
    if (lane < n_groups) {
        g_row0 = p.slot_offsets[first_slot + lane];
        g_rows = p.slot_offsets[first_slot + lane + 1] - g_row0;
    }
    const int g_nt = (g_rows + BM - 1) / BM;               // row tiles of the group (NN/NT)
    int g_incl = g_nt;                                     // inclusive prefix over groups
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(g_incl, off, 64);
        if (lane >= off) g_incl += up;
    }
    const int total_rt = __builtin_amdgcn_readlane(g_incl, 63);
    const int g_excl = g_incl - g_nt;

    // ---- which tiles.  The kernel is persistent: one block per CU walks its share of the tiles, so a
    // tile's stores drain under the next tile's loads and nothing is relaunched.  Blocks go round-robin
    // over the 8 XCDs (block b runs on XCD b % 8), each with its own L2.  The tiles that actually exist
    // (the counts are only known here) are cut into rounds of as many tiles as an XCD has blocks, walked
    // column by column inside a band of p.band row tiles (7 or 8 by 4 to 5 column tiles), so that the tiles in
    // flight on an XCD share operand slices in its L2; consecutive rounds go to the 8 XCDs in turn, so
    // that at any time the XCDs work on neighbouring rounds and what one of them has fetched from HBM
    // the others find in the memory-side cache.
    const int xcd = blockIdx.x & 7, q0 = blockIdx.x >> 3, q_stride = gridDim.x >> 3;
    const int BAND = p.band;
    const int tiles_g = p.row_tiles * p.col_tiles;         // TN: tiles of one group
    const int n_act = total_rt * p.col_tiles;              // NN/NT: tiles that exist
    const int rpg = (tiles_g + q_stride - 1) / q_stride;   // TN: rounds per group
    // NN/NT: the tiles left over after the last full round of the chip (fewer than there are blocks) are cut
    // along the contraction into S parts, each an item of its own, so that the last round keeps S times as
    // many blocks busy for 1/S of a tile's time.  A part leaves its accumulators in the workspace; a second
    // launch (FIN) adds the parts of a tile in a fixed order and runs the tile's epilogue.
    const int nblk = gridDim.x;
    const int n_full = (KIND == KIND_TN) ? 0 : (n_act / nblk) * nblk, rem = n_act - n_full;
    int S = 1;
    if (KIND != KIND_TN && p.split_ws != nullptr)
        S = row_parts(rem, nblk, p.n_seg * (p.Kseg / BK), p.split_max, p.split_slices, p.split_cap);
    if (KIND != KIND_TN && FIN && S == 1) return;
    int turns = 0, first_slices = 0;                       // uneven cut: remainders per block, slices of a tile's first part
    if (LAST && S == 1) first_slices = uneven_cut(rem, nblk, p.n_seg * (p.Kseg / BK), p.uneven_cap, turns);
    const int n_items = LAST && first_slices ? n_full + nblk : n_full + rem * S;
    const int n_rounds = (n_items + q_stride - 1) / q_stride;

    // TN: the contraction of a group is as long as its rows are many, and a group may have fewer tiles than there are
    // blocks.  A group whose contraction is longer than a block's share of all the work is cut along it into parts of about
    // that share; lane v holds part v (of some group; a whole group is its only part).  The parts' tiles go through the
    // workspace and the finishing launch like those of a split last round.
    // Parts differ in length, so their rounds are dealt to the XCDs by load: the longest first, a part's rounds spread
    // evenly, the odd ones to the XCDs with the least to do so far (every block keeps the loads of all eight, lane x that
    // of XCD x, and so comes to the same dealing).  Measured, us
    // per product, whole groups dealt in turn (256 x 256 tiles, 128 x 128) -> now, with the finishing launch: d = 3136,
    // h = 576, 20623 rows in 8 uneven groups 310, 266 -> 142; d = 3968, h = 704, 12532 rows in 2 216, 179 -> 112 to 144;
    // d = 2944, h = 576, one group of 3002 71, 47 -> 35; d = 1024, h = 4096, 9279 rows in 4 150, 126 -> 118.  Where nothing is
    // cut: d = 512, h = 14272, 2522 rows 93 -> 80; the largest configuration the same (4.12 ms).  Cut where whole groups fill
    // the XCDs: d = 256, h = 512, eight groups of 3276 rows, the backward pass 178, whole 117; d = 384, h = 512, eight of 1866
    // 119, whole 86; d = 64, h = 512, 37605 rows in 16 329, whole 246; or nearly, and the parts would not: d = 1728, h = 64, six
    // of 2128 192, whole 137; d = 1280, h = 1792, three of 1982 261, whole 217.
    int n_parts = 0, v_group = 0, v_row0 = 0, v_rows = 0, v_of = 1, v_unit = 0;     // unit of the part's tile 0
    int tn_split = 1, tn_unit = 0;                         // lane g: parts of group g, unit of its first part's tile 0
    unsigned long long tn_split_mask = 0ull;
    if (KIND == KIND_TN) {
        n_parts = p.Gcap; v_group = lane; v_row0 = g_row0; v_rows = g_rows;
    }
    if (KIND == KIND_TN && p.split_ws != nullptr) {
        const int k = lane < p.Gcap ? (g_rows + BK - 1) / BK : 0;
        int all = k;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) all += __shfl_xor(all, off, 64);
        tn_split = tn_parts(k, tiles_g, rpg, all, p.Gcap, nblk, p.tn_over, p.split_max, p.split_slices);
        tn_split_mask = __ballot(tn_split > 1);
        if (tn_split_mask) {
            tn_split = min(tn_split, tn_most_units(p.split_cap, tiles_g, __popcll(tn_split_mask)));
            tn_split_mask = __ballot(tn_split > 1);
        }
        int incl, units, own_units;
        while (true) {
            incl = lane < p.Gcap ? tn_split : 0;
            own_units = units = tn_split > 1 ? tn_split : 0;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int up = __shfl_up(incl, off, 64), uu = __shfl_up(units, off, 64);
                if (lane >= off) { incl += up; units += uu; }
            }
            if (__builtin_amdgcn_readlane(incl, 63) <= 64) break;
            tn_split = min(tn_split, tn_most_lanes(p.Gcap, __popcll(tn_split_mask)));      // then they do fit
            tn_split_mask = __ballot(tn_split > 1);
        }
        tn_unit = (units - own_units) * tiles_g;
        if (tn_split_mask != 0ull) {
            int longest = k, len = (k + tn_split - 1) / tn_split;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) { longest = max(longest, __shfl_xor(longest, off, 64)); len = max(len, __shfl_xor(len, off, 64)); }
            const int n = __popcll(__ballot(k > 0)), total = __builtin_amdgcn_readlane(incl, 63) - (p.Gcap - n);
            if (!__builtin_amdgcn_readfirstlane(tn_pays(longest, len, all, n, total, rpg, p.tn_over))) tn_split_mask = 0ull;
        }
        if (tn_split_mask != 0ull) {
            n_parts = __builtin_amdgcn_readlane(incl, 63);
            const int first = incl - tn_split;
            for (int i = 0; i < p.Gcap; ++i) {
                const int f = __builtin_amdgcn_readlane(first, i), n = __builtin_amdgcn_readlane(tn_split, i);
                const int part = lane - f, kk = __builtin_amdgcn_readlane(k, i), rows = __builtin_amdgcn_readlane(g_rows, i);
                const int r0 = __builtin_amdgcn_readlane(g_row0, i), u = __builtin_amdgcn_readlane(tn_unit, i);
                if (part >= 0 && part < n) {
                    const int lo = (int)((long)part * kk / n) * BK, hi = part + 1 == n ? rows : (int)((long)(part + 1) * kk / n) * BK;
                    v_group = i; v_row0 = r0 + lo; v_rows = hi - lo; v_of = n; v_unit = u + part;
                }
            }
        }
    }
    if (KIND == KIND_TN && FIN && tn_split_mask == 0ull) return;
    int tn_left = n_parts;                                 // parts not taken yet
    unsigned long long tn_taken = 0ull;
    int tn_v = 0, tn_n = 0, tn_i = 0, tn_extra = 0;        // current part, its rounds for this XCD, the next one, its odd round
    int tn_load = 0;                                       // lane x: slices and tile boundaries dealt to XCD x
    auto tn_next_part = [&]() {
        const bool mine = lane < n_parts && !((tn_taken >> lane) & 1ull);
        int best = mine ? v_rows : -1;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) best = max(best, __shfl_xor(best, off, 64));
        tn_v = __ffsll((unsigned long long)__ballot(mine && v_rows == best)) - 1;
        tn_taken |= 1ull << tn_v;
        --tn_left;
        const int cost = (best + BK - 1) / BK + p.tn_over, even = rpg >> 3, odd = rpg & 7;
        int rank = 0;                                      // of XCD `lane` by load, then number
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const int o = __builtin_amdgcn_readlane(tn_load, x);
            rank += (o < tn_load || (o == tn_load && x < (lane & 7))) ? 1 : 0;
        }
        tn_load += (even + (rank < odd ? 1 : 0)) * cost;   // lanes past 7 hold nothing that is read
        const int my_rank = __builtin_amdgcn_readlane(rank, xcd);
        tn_n = even + (my_rank < odd ? 1 : 0);
        tn_extra = 8 * even + my_rank;
        tn_i = 0;
    };
    // few rounds: one each, in turn
    const bool tn_simple = n_parts * rpg <= 8;
    if (KIND == KIND_TN && tn_simple) {
        tn_left = 0;
        tn_v = xcd / rpg;
        tn_n = tn_v < n_parts ? 1 : 0;
    }
    const int q_first = FIN ? (int)blockIdx.x : q0;
    const int q_step = FIN ? nblk : q_stride;
    const int q_end = FIN ? (KIND == KIND_TN ? __popcll(tn_split_mask) * tiles_g : rem) * TM       // FIN: two rows of fragments (32 rows) of a tile's upper and lower waves are an item
                          : (KIND == KIND_TN ? 0x7fffffff : ((n_rounds + 7) >> 3) * q_stride);

  int turn = 0, next = q_step;
  for (int q = q_first; q < q_end; q += next) {
    int g, rt, ct;
    int part = 0, parts = 1, unit = 0;                     // K-split: which part of how many, and where it is kept
    long a_row0, a_row_end;      // valid rows of the A tile (NN/NT) or of the contraction (TN)
    int k_tiles;
    int m0;                      // first output row of the tile (global row for NN/NT, row of dW for TN)
    if (KIND == KIND_TN) {
        // every group has the same tile grid but its own contraction length: a round never mixes
        // groups, so the blocks of an XCD stay on the same contraction slices of shared operands
        int t;
        long row0 = 0;
        int rows = 0;
        if (FIN) {
            const int i = q / TM;
            unsigned long long m = tn_split_mask;
            for (int n = i / tiles_g; n > 0; --n) m &= m - 1;              // the n-th group that was split
            g = __ffsll(m) - 1;
            t = i % tiles_g;
            parts = __builtin_amdgcn_readlane(tn_split, g);
            unit = __builtin_amdgcn_readlane(tn_unit, g) + t * parts;
        } else {
            while (tn_i == tn_n && tn_left > 0) tn_next_part();
            if (tn_i == tn_n) break;
            const int in_part = tn_simple ? xcd % rpg : ((tn_i + 1 == tn_n && tn_n > (rpg >> 3)) ? tn_extra : tn_i * 8 + xcd);
            ++tn_i;
            t = in_part * q_stride + q0;
            if (t >= tiles_g) continue;
            g = __builtin_amdgcn_readlane(v_group, tn_v);
            row0 = __builtin_amdgcn_readlane(v_row0, tn_v);
            rows = __builtin_amdgcn_readlane(v_rows, tn_v);
            parts = __builtin_amdgcn_readlane(v_of, tn_v);
            unit = __builtin_amdgcn_readlane(v_unit, tn_v) + t * parts;
        }
        const int band = t / (BAND * p.col_tiles);
        const int in_band = t - band * BAND * p.col_tiles;
        const int band_rows = min(BAND, p.row_tiles - band * BAND);
        rt = band * BAND + in_band % band_rows;
        ct = in_band / band_rows;
        a_row0 = row0; a_row_end = row0 + rows;                            // none for unused groups
        k_tiles = (rows + BK - 1) / BK;
        m0 = rt * BM;
    } else {
        int t;
        if (FIN) {
            t = n_full + q / TM; parts = S; unit = (q / TM) * S;
        } else {
            const int item = (((q - q0) / q_stride) * 8 + xcd) * q_stride + q0;
            if (item >= n_items) break;
            t = item;
            if (item >= n_full) {
                int i = item - n_full;
                if (LAST && first_slices) {
                    if (i >= rem) {                        // the remainders of tiles i, i + others, ..: one iteration each
                        const int others = nblk - rem;
                        i += turn * others - rem;
                        if (i >= rem) break;
                        ++turn;
                        next = turn < turns ? 0 : q_step;
                        part = 1;
                    }
                    t = n_full + i; parts = 2; unit = 2 * i + part;
                } else {
                    t = n_full + i / S; part = i % S; parts = S; unit = i;
                }
            }
        }
        const int band = t / (BAND * p.col_tiles);
        const int in_band = t - band * BAND * p.col_tiles;
        const int band_rows = min(BAND, total_rt - band * BAND);
        rt = band * BAND + in_band % band_rows;
        ct = in_band / band_rows;
        g = __popcll(__ballot(g_incl <= rt)) & 63;                         // first group whose tiles reach past rt
        const int gr0 = __builtin_amdgcn_readlane(g_row0, g);
        const int row0 = gr0 + (rt - __builtin_amdgcn_readlane(g_excl, g)) * BM;
        const int row_end = gr0 + __builtin_amdgcn_readlane(g_rows, g);
        a_row0 = row0; a_row_end = row_end;
        k_tiles = p.n_seg * (p.Kseg / BK);
        m0 = row0;
    }
    const int n0 = ct * (DUAL ? BN / 2 : BN);             // first output column (hidden unit for dual)
    const int k_per_seg = (KIND == KIND_TN) ? k_tiles : p.Kseg / BK;
    // slices of this item: all of them, or one part of a split tile; none in the finishing launch
    // (a K-contiguous operand is fetched two slices at a time: parts begin at even slices)
    // (TN: the rows are those of the part)
    auto part_begin = [&](int i) { return LAST && first_slices ? first_slices * i : ((int)((long)i * k_tiles / parts) & ~1); };
    const int k_lo = (KIND == KIND_TN) ? 0 : part_begin(part);
    const int k_hi = (KIND == KIND_TN || part + 1 == parts) ? k_tiles : part_begin(part + 1);
    const int k_cnt = FIN ? 0 : k_hi - k_lo;

    // ---- buffer resources: everything outside the valid rows of an operand reads as zero --------
    // Each wave moves two 1-KB pieces of the A slice and two of the B slice per contraction slice.
    rsrc_t rA[2], rB[2];                   // per segment (A), per segment or per dual half (B)
    uint32_t voffA[PA], voffB[PB];                         // per-lane byte offsets of this wave's pieces
    uint32_t ldsA[PA], ldsB[PB];                           // LDS byte offsets of the pieces inside a stage
    uint32_t stepA, stepB;                                 // byte advance of the source per slice
    const bf16_t *tn_baseA = nullptr, *tn_baseB = nullptr; // TN: where the current resources start, and how many
    long tn_bytesA = 0, tn_bytesB = 0;                     // bytes of the group's rows lie behind that point
    {
        const long a_rows = a_row_end - a_row0;
        if (KIND == KIND_TN) {
            tn_baseA = p.A[0] + a_row0 * p.lda + m0; tn_bytesA = (a_rows * p.lda - m0) * 2;
            tn_baseB = p.B[0] + a_row0 * p.ldb + n0; tn_bytesB = (a_rows * p.ldb - n0) * 2;
            rA[0] = rA[1] = make_rsrc(tn_baseA, tn_bytesA);
            rB[0] = rB[1] = make_rsrc(tn_baseB, tn_bytesB);
            stepA = (uint32_t)(BK * p.lda * 2);
            stepB = (uint32_t)(BK * p.ldb * 2);
        } else {
            for (int s = 0; s < 2; ++s) {
                const int ss = s < p.n_seg ? s : 0;
                rA[s] = make_rsrc(p.A[ss] + a_row0 * p.lda, a_rows * p.lda * 2);
            }
            stepA = BK * 2;
            const long gofs = (long)g * p.b_group_stride;
            if (KIND == KIND_NN) {
                rB[0] = make_rsrc(p.B[0] + gofs + n0, ((long)p.Kseg * p.ldb - n0) * 2);
                rB[1] = DUAL ? make_rsrc(p.B_dual + gofs + n0, ((long)p.Kseg * p.ldb - n0) * 2) : rB[0];
                stepB = (uint32_t)(BK * p.ldb * 2);
            } else {
                for (int s = 0; s < 2; ++s) {
                    const int ss = s < p.n_seg ? s : 0;
                    rB[s] = make_rsrc(p.B[ss] + gofs + (long)n0 * p.ldb, (long)(p.N - n0) * p.ldb * 2);
                }
                stepB = BK * 2;
            }
        }
        // a 1-KB piece of a K-contiguous operand is 8 rows x 128 bytes of half the tile's rows: lane l reads piece l%8 of
        // row l/8, where the swizzle of the buffer puts it
        auto line_source = [&](int blk, long ld) {
            const int row = blk * 8 + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
            return (uint32_t)((row * ld + piece * 8) * 2);
        };
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int blk = wave + NWAVES * i;             // piece index inside an operand buffer
            ldsA[i] = blk * 1024;
            voffA[i] = A_KMAJOR ? kmajor_source<BM>(blk * 64 + lane, p.lda) : line_source(blk, p.lda);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int blk = wave + NWAVES * i;
            if (DUAL) {
                // two sub-buffers of [32][BN / 2]; this wave's pieces alternate between them
                const int half = i & 1, blk2 = wave + NWAVES * (i >> 1);
                ldsB[i] = half * (GEO::B_BYTES / 2) + blk2 * 1024;
                voffB[i] = kmajor_source<BN / 2>(blk2 * 64 + lane, p.ldb);
            } else {
                ldsB[i] = blk * 1024;
                voffB[i] = B_KMAJOR ? kmajor_source<BN>(blk * 64 + lane, p.ldb) : line_source(blk, p.ldb);
            }
        }
    }

    // Slices are requested strictly in order; the source offsets advance with the stream.
    int iss_stage = 0;
    int iss_seg = (KIND == KIND_TN) ? 0 : k_lo / k_per_seg, iss_in_seg = (KIND == KIND_TN) ? 0 : k_lo - iss_seg * k_per_seg;
    uint32_t soffA = (uint32_t)iss_in_seg * stepA, soffB = (uint32_t)iss_in_seg * stepB;
    // The requests of one slice (or, NN and NT, of one group, below) into stage iss_stage, with the resources the caller has
    // picked: no decision in it.  The caller says when each of them goes out.
    constexpr int SLICE_OPS = PA + PB;                     // of one wave
    auto request_piece = [&](int n, uint32_t st, const rsrc_t ra, const rsrc_t rb0, const rsrc_t rb1, uint32_t oa, uint32_t ob) {
        if (n < PA) dma16(ra, st + ldsA[n], voffA[n], oa);
        else dma16<ONCE>((DUAL && ((n - PA) & 1)) ? rb1 : rb0, st + A_BYTES + ldsB[n - PA], voffB[n - PA], ob);
    };
    auto next_stage = [&]() { iss_stage = (iss_stage + 1 == STAGES) ? 0 : iss_stage + 1; };
    auto slice_done = [&]() { next_stage(); ++iss_in_seg; soffA += stepA; soffB += stepB; };
    auto issue_with = [&](const rsrc_t ra, const rsrc_t rb0, const rsrc_t rb1) {
        const uint32_t st = lds0 + (uint32_t)iss_stage * STAGE_BYTES;
#pragma unroll
        for (int n = 0; n < SLICE_OPS; ++n) request_piece(n, st, ra, rb0, rb1, soffA, soffB);
        slice_done();
    };
    // What may have to change between two slices: the next contraction segment (NN/NT), or, for TN, whose offset
    // runs over all rows of the group, the base of the resources: buffer offsets are 32 bits, so the resources are
    // moved up to the current slice long before that overflows (a group of 2^31 bytes and more).
    auto issue_fixups = [&]() {
        if (KIND != KIND_TN && iss_in_seg == k_per_seg) { iss_in_seg = 0; ++iss_seg; soffA = 0; soffB = 0; }
        if (KIND == KIND_TN && ((soffA | soffB) & 0xc0000000u)) {
            tn_baseA += soffA / 2; tn_bytesA -= soffA; soffA = 0;
            tn_baseB += soffB / 2; tn_bytesB -= soffB; soffB = 0;
            rA[0] = rA[1] = make_rsrc(tn_baseA, tn_bytesA);
            rB[0] = rB[1] = make_rsrc(tn_baseB, tn_bytesB);
        }
    };
    auto issue_next = [&]() {                              // one slice, strictly in order
        issue_with(iss_seg ? rA[1] : rA[0], (KIND == KIND_NT && iss_seg) ? rB[1] : rB[0], rB[1]);
        issue_fixups();
    };
    // how many slices can be requested from here without a fixup in between (at least one)
    auto issue_run = [&]() -> int {
        if (KIND != KIND_TN) return k_per_seg - iss_in_seg;
        const uint32_t hi = soffA > soffB ? soffA : soffB, st = stepA > stepB ? stepA : stepB;
        return (int)((0x3fffffffu - hi) / st) + 1;
    };

    // NN and NT fetch their K-contiguous operands in whole 128-byte lines: a request group carries, for such an
    // operand, 128 rows x 64 steps (two slices) instead of 256 rows x 32 steps: group n holds the upper (n even) or
    // lower (n odd) 128 rows of the tile for slices 2 (n / 2) and 2 (n / 2) + 1.  Same bytes and same number of
    // instructions per group as a slice, half as many requests to L2.  A K-major operand (the weights of NN) keeps
    // one slice per group.  PAR: the parity of the group, known where the loop is written out.
    constexpr bool A_PAIR = !A_KMAJOR, B_PAIR = !B_KMAJOR;
    const uint32_t halfA = (uint32_t)(BM / 2 * p.lda * 2), halfB = (uint32_t)(BN / 2 * p.ldb * 2);   // to the lower half
    auto group_offsets = [&](auto PAR, uint32_t& oa, uint32_t& ob) {
        constexpr int par = decltype(PAR)::value;
        oa = (A_PAIR && par) ? soffA + halfA : soffA;
        ob = (B_PAIR && par) ? soffB + halfB : soffB;
    };
    auto group_done = [&](auto PAR) {
        constexpr int par = decltype(PAR)::value;
        next_stage();
        ++iss_in_seg;
        if (!A_PAIR || par) soffA += A_PAIR ? 2 * stepA : stepA;
        if (!B_PAIR || par) soffB += B_PAIR ? 2 * stepB : stepB;
    };
    auto issue_group = [&](auto PAR, const rsrc_t ra, const rsrc_t rb0, const rsrc_t rb1) {
        const uint32_t st = lds0 + (uint32_t)iss_stage * STAGE_BYTES;
        uint32_t oa, ob;
        group_offsets(PAR, oa, ob);
#pragma unroll
        for (int n = 0; n < SLICE_OPS; ++n) request_piece(n, st, ra, rb0, rb1, oa, ob);
        group_done(PAR);
    };
    // after an odd group (segments hold an even number of slices): the next contraction segment
    auto group_fixups = [&]() {
        if (iss_in_seg == k_per_seg) { iss_in_seg = 0; ++iss_seg; soffA = 0; soffB = 0; }
    };

    // ---- per-lane fragment addresses inside a ring buffer.  The buffer's base is the only part of a fragment
    // address that changes from slice to slice, and every vector instruction of the fetching wave takes an issue
    // slot from the matrix instructions of its partner: fragments that lie a constant distance apart share one
    // address register and differ in the instruction's immediate offset.
    constexpr int FM = 2 * TM, FN = 2 * TN;                // fragments of 16 rows, of 16 columns
    static_assert((FM == 8 || FM == 4) && FN == 4 && WN == 64, "the fragment reads below are written out for 8 x 4 or 4 x 4 fragments");
    // K-major operands: one address per 16-column chunk of 64 columns; 64 columns lie a constant distance apart.
    constexpr int BCOLS = DUAL ? BN / 2 : BN;
    constexpr int STEP4_A = BM * 8, STEP4_B = BCOLS * 8;         // four steps further on
    static_assert(KIND != KIND_TN || BM == BN, "one set of addresses for both operands");
    uint32_t fk_addr[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int b = lane >> 4, s = lane & 15;
        fk_addr[c] = kmajor_off<BCOLS>(8 * b + (s >> 2), c * 16 + 4 * (s & 3));
    }
    const uint32_t a_cols = wm * (WM / 64) * 256;        // this wave's columns inside a buffer
    const uint32_t b_cols = A_BYTES + (DUAL ? wn >> 1 : wn) * 256;
    // DUAL: 32 columns of either weight matrix, two chunks of a line
    const uint32_t fd_addr[2] = {(wn & 1) ? fk_addr[2] : fk_addr[0], (wn & 1) ? fk_addr[3] : fk_addr[1]};
    // `after(n)`: what goes out between the reads, after the n-th fragment's
    auto load_kmajor_b = [&](bf16x8 (&fb)[FN], uint32_t st, auto after) {
        if constexpr (DUAL) {                              // fragments 0, 1 from the W1 sub-buffer, 2, 3 from the W3 sub-buffer
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t a = st + b_cols + fd_addr[j];
                lds_frag_kmajor_at<STEP4_B, 0>(fb[j], a);
                after(FM + 2 * j);
                lds_frag_kmajor_at<STEP4_B, (int)GEO::B_BYTES / 2>(fb[2 + j], a);
                after(FM + 2 * j + 1);
            }
        } else {
#pragma unroll
            for (int j = 0; j < FN; ++j) { lds_frag_kmajor_at<STEP4_B, 0>(fb[j], st + b_cols + fk_addr[j]); after(FM + j); }
        }
    };
    // TN: both operands K-major, a slice per ring buffer
    auto load_frags = [&](bf16x8 (&fa)[FM], bf16x8 (&fb)[FN], int stage, auto after) {
        const uint32_t st = lds0 + (uint32_t)stage * STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t a = st + a_cols + fk_addr[i];
            lds_frag_kmajor_at<STEP4_A, 0>(fa[i], a);
            after(FM / 4 * i);
            if constexpr (FM == 8) { lds_frag_kmajor_at<STEP4_A, 256>(fa[4 + i], a); after(2 * i + 1); }
        }
        load_kmajor_b(fb, st, after);
    };
    // Operands fetched in 128-byte lines: fragment 0 of this wave in a 128-row buffer, at the buffer's two slices; the
    // wave's other fragments lie 16 rows = 2 KB further on.  The upper row of waves (A) and the waves of the two left
    // columns (B) read the buffer of an even group, the others that of the odd group after it.
    uint32_t fpa[2], fpb[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        fpa[v] = halfpair_off(lane & 15, lane >> 4) ^ (uint32_t)(v << 6);
        fpb[v] = A_BYTES + (halfpair_off((wn % (WGN / 2)) * WN + (lane & 15), lane >> 4) ^ (uint32_t)(v << 6));
    }
    auto load_group_frags = [&](bf16x8 (&fa)[FM], bf16x8 (&fb)[FN], uint32_t stA, uint32_t stB, auto PAR, auto after) {
        constexpr int par = decltype(PAR)::value;          // which slice of the pair
        const uint32_t a = stA + fpa[par];
        auto frag_a = [&](auto I) { lds_frag_kcontig_at<decltype(I)::value * 2048>(fa[decltype(I)::value], a); after(decltype(I)::value); };
        frag_a(std::integral_constant<int, 0>{}); frag_a(std::integral_constant<int, 1>{});
        frag_a(std::integral_constant<int, 2>{}); frag_a(std::integral_constant<int, 3>{});
        if constexpr (FM == 8) {
            frag_a(std::integral_constant<int, 4>{}); frag_a(std::integral_constant<int, 5>{});
            frag_a(std::integral_constant<int, 6>{}); frag_a(std::integral_constant<int, 7>{});
        }
        if constexpr (B_KMAJOR) {                          // stB: the buffer of the slice
            load_kmajor_b(fb, stB, after);
        } else {
            const uint32_t bb = stB + fpb[par];
            auto frag_b = [&](auto J) { lds_frag_kcontig_at<decltype(J)::value * 2048>(fb[decltype(J)::value], bb); after(FM + decltype(J)::value); };
            frag_b(std::integral_constant<int, 0>{}); frag_b(std::integral_constant<int, 1>{});
            frag_b(std::integral_constant<int, 2>{}); frag_b(std::integral_constant<int, 3>{});
        }
    };
    // Which request follows the n-th fragment of a slice: one after every quarter of them.  LDS takes the reads of the four
    // waves of a row and the vector memory path their requests side by side; one after the other they make the fetch phase of a
    // K-major operand longer than the multiply phase it hides behind.  In turn, against all requests after the last read (us):
    // fwd2 3957 -> 3784, weight gradients 4428 -> 4125, fwd1 8702 -> 8645, bwd2 7612 -> 7556 (d = 4096, h = 14336, 46695 rows);
    // d = 1024, h = 4096, 9279 rows: fwd1 121 -> 116, fwd2 92 -> 88.
    auto goes_out = [](int n) { return (n + 1) % ((FM + FN) / SLICE_OPS) == 0 ? (n + 1) / ((FM + FN) / SLICE_OPS) - 1 : -1; };
    auto wait_frags = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);                 // no MFMA moves above the wait
    };

    // NN and NT start their accumulators with the first products of slice 0 (a matrix instruction that takes zero
    // as its addend) instead of clearing 128 registers per tile; TN, whose groups may be empty, clears them.
    f32x4 acc[FM][FN];
    if (KIND == KIND_TN || FIN) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.0f;
    }

    // The FM*FN products of a slice.  The accumulators are pinned to AGPRs, which leaves the VGPRs of the wave to fragments
    // and addresses.  These kernels run at the package's power cap, and 16x16x32 takes less energy per flop than 32x32x16,
    // least in an order in which two instructions in a row share an operand: this loop with LDS reads and products alone
    // sustains 1660 TFLOP/s with 32x32x16, 1850 with 16x16x32 row by row and 1880 with every other row backwards.  In the
    // kernels, with the requests between the reads (goes_out): clock 1.47 -> 1.62 GHz, and d = 4096, h = 14336, SwiGLU, forward
    // and backward 38.9 -> 36.9 ms; d = 2048, h = 8192, GELU 5.39 -> 5.11; d = 1024, h = 4096, forward 264 -> 250 us.
    auto mma = [&](const bf16x8 (&fa)[FM], const bf16x8 (&fb)[FN]) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int jj = 0; jj < FN; ++jj) {
                const int j = (i & 1) ? FN - 1 - jj : jj;
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j]) : "v"(fb[j]), "v"(fa[i]));
            }
    };

    // ---- main loop, two phases per slice.  In its fetch phase a wave reads the fragments of slice t
    // from LDS and requests its share of what lies three or four slices ahead; one barrier later, in its multiply phase, it issues
    // the 32 MFMAs of the slice back to back.  The upper row of waves runs one barrier interval behind
    // the lower one; waves w and w+4 share a SIMD, so while one of them feeds the matrix pipe the other
    // collects its operands.  With LDS reads and MFMAs alone this loop runs at the MFMA rate; what it
    // waits for in practice is the delivery of the slices from L2/HBM.  (A request placed between MFMAs stalls the matrix pipe
    // for several MFMA slots.)
    // Two blocks on a CU (Small) need no such order: a wave of each shares a SIMD, and while one block collects operands,
    // waits or runs an epilogue, the other multiplies.  One barrier per slice then: the waits before it cover this wave's
    // pieces of the next slice and its reads of the current one, and what a request overwrites was last read before the
    // barrier of the slice before.
    if (!FIN && k_cnt > 0) {
      if constexpr (KIND == KIND_TN) {
        bf16x8 fa[FM], fb[FN];
        constexpr int L = STAGES - 1;                      // slices requested ahead
        // Every slice t is preceded by exactly t + L request groups of this wave (the prologue issues L of them,
        // every slice one more), so "my pieces of slice t + 1 have landed" is always "at most L - 1 groups are still
        // on their way": one fixed wait count for the whole contraction.  Where there is no slice left to request
        // (a contraction shorter than the lookahead, and the last L slices of any contraction) the group goes to a
        // resource of zero length: nothing is read, zeros land in a ring slot that nobody reads again.
        const rsrc_t rnull = make_rsrc(p.A[0], 0);
#pragma unroll
        for (int i = 0; i < L; ++i) {
            if (i < k_cnt) issue_next(); else issue_with(rnull, rnull, rnull);
        }
        WAIT_VMCNT((L - 1) * SLICE_OPS);                   // slice 0 has landed
        BLOCK_BARRIER();
        if (GEO::TWO_PHASE && wm == 1) BLOCK_BARRIER();
        int cur = 0;
        asm volatile(".p2align 8\n\t.rept " LOOP_OFF_STR "\n\ts_nop 0\n\t.endr" ::: "memory");
        // One slice: fetch phase (fragments of slice t, then the requests for slice t + L, then the wait for this
        // wave's pieces of slice t + 1), barrier, multiply phase, barrier.  Ring slot (t+4) % 5 held slice t-1,
        // which every wave finished reading at least one barrier ago.  The loop has no decision in it: it runs
        // over stretches of slices that need no fixup between their requests (a whole contraction segment, or
        // all of a group's rows short of 2^30 bytes) with the resources of the stretch.
        int t = 0;
        while (t < k_cnt) {
            const bool more = t + L < k_cnt;               // slices left to request
            const int n = more ? min(k_cnt - L - t, issue_run()) : k_cnt - t;
            const rsrc_t ra = more ? (iss_seg ? rA[1] : rA[0]) : rnull;
            const rsrc_t rb0 = more ? ((KIND == KIND_NT && iss_seg) ? rB[1] : rB[0]) : rnull;
            const rsrc_t rb1 = more ? rB[1] : rnull;
            for (int i = 0; i < n; ++i) {
                const uint32_t to = lds0 + (uint32_t)iss_stage * STAGE_BYTES;
                load_frags(fa, fb, cur, [&](int n) { if (goes_out(n) >= 0) { __builtin_amdgcn_sched_barrier(0); request_piece(goes_out(n), to, ra, rb0, rb1, soffA, soffB); __builtin_amdgcn_sched_barrier(0); } });
                slice_done();
                WAIT_VMCNT((L - 1) * SLICE_OPS);
                wait_frags();
                BLOCK_BARRIER();
                __builtin_amdgcn_s_setprio(1);
                mma(fa, fb);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);
                if (GEO::TWO_PHASE) BLOCK_BARRIER();
                cur = (cur + 1 == STAGES) ? 0 : cur + 1;
            }
            t += n;
            if (more) issue_fixups();
        }
        WAIT_VMCNT(0);                                     // the zero-length requests too: the epilogue reuses the ring
        if (GEO::TWO_PHASE && wm == 0) BLOCK_BARRIER();    // both rows have passed the same number of barriers
        BLOCK_BARRIER();                                   // and everybody's requests have landed
      } else {
        bf16x8 fa[FM], fb[FN];
        // NN and NT.  One request group per slice, three ahead: before slice t come the groups 0 .. t + 2, slice t adds
        // group t + 3 into ring slot (t + 3) % 5, which held group t - 2, last read in slice t - 1.  Slice 2p and 2p + 1
        // read the K-contiguous operands from the buffers of the groups 2p (upper 128 rows) and 2p + 1 (lower 128
        // rows), a K-major operand from the buffer of the slice's own group.  What a slice waits for before its
        // barrier is the data of the next slice: after an even slice the K-major operand's group t + 1 (two groups
        // may still be on their way), after an odd slice the groups t + 1 and t + 2 of the next pair (one group may).
        // Contractions have an even number of slices (d and h are multiples of 64; split parts begin at even slices),
        // so the loop is written out for pairs: slice 0, then pairs of an odd and an even slice, whose two groups are
        // the two halves of one later pair of slices and need no fixup between them, then the last slice.
        constexpr int L = 3;
        const rsrc_t rnull = make_rsrc(p.A[0], 0);
        auto real_a = [&]() { return iss_seg ? rA[1] : rA[0]; };
        auto real_b0 = [&]() { return (KIND == KIND_NT && iss_seg) ? rB[1] : rB[0]; };
        // groups 0, 1, 2: a contraction has at least two slices
        issue_group(std::integral_constant<int, 0>{}, real_a(), real_b0(), rB[1]);
        issue_group(std::integral_constant<int, 1>{}, real_a(), real_b0(), rB[1]);
        group_fixups();
        if (k_cnt > 2) issue_group(std::integral_constant<int, 0>{}, real_a(), real_b0(), rB[1]);
        else issue_group(std::integral_constant<int, 0>{}, rnull, rnull, rnull);
        WAIT_VMCNT(SLICE_OPS);                             // groups 0 and 1 have landed: slices 0 and 1
        BLOCK_BARRIER();
        if (GEO::TWO_PHASE && wm == 1) BLOCK_BARRIER();
        int cur = 0;                                       // ring slot of the slice's own group
        int pair0 = 0;                                     // ring slot of the even group of the slice's pair
        const int hA = wm, hB = wn / (WGN / 2);                   // which group of a pair holds this wave's rows of A and B
        auto slot_base = [&](int slot) { return lds0 + (uint32_t)(slot >= STAGES ? slot - STAGES : slot) * STAGE_BYTES; };
        // One slice of parity PAR; ra .. rb1: the resources of the group it requests (of the opposite parity).
        auto mma_first = [&](const bf16x8 (&fa)[FM], const bf16x8 (&fb)[FN]) {      // acc = products (+ 0)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int jj = 0; jj < FN; ++jj) {
                    const int j = (i & 1) ? FN - 1 - jj : jj;
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc[i][j]) : "v"(fb[j]), "v"(fa[i]));
                }
        };
        auto slice = [&](auto PAR, auto FIRST, const rsrc_t ra, const rsrc_t rb0, const rsrc_t rb1) {
            constexpr int par = decltype(PAR)::value;
            const uint32_t stA = slot_base(pair0 + hA);
            const uint32_t stB = B_KMAJOR ? slot_base(cur) : slot_base(pair0 + hB);
            const uint32_t to = lds0 + (uint32_t)iss_stage * STAGE_BYTES;
            uint32_t oa, ob;
            group_offsets(std::integral_constant<int, 1 - par>{}, oa, ob);
            load_group_frags(fa, fb, stA, stB, PAR, [&](int n) { if (goes_out(n) >= 0) { __builtin_amdgcn_sched_barrier(0); request_piece(goes_out(n), to, ra, rb0, rb1, oa, ob); __builtin_amdgcn_sched_barrier(0); } });
            group_done(std::integral_constant<int, 1 - par>{});
            WAIT_VMCNT(par ? SLICE_OPS : 2 * SLICE_OPS);
            wait_frags();
            BLOCK_BARRIER();
            __builtin_amdgcn_s_setprio(1);
            if constexpr (decltype(FIRST)::value) mma_first(fa, fb); else mma(fa, fb);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            if (GEO::TWO_PHASE) BLOCK_BARRIER();
            cur = (cur + 1 == STAGES) ? 0 : cur + 1;
            if (par) pair0 = (pair0 + 2 >= STAGES) ? pair0 + 2 - STAGES : pair0 + 2;
        };
        // slice 0 requests group 3, the lower rows of slices 2 and 3
        if (k_cnt > 2) { slice(std::integral_constant<int, 0>{}, std::true_type{}, real_a(), real_b0(), rB[1]); group_fixups(); }
        else slice(std::integral_constant<int, 0>{}, std::true_type{}, rnull, rnull, rnull);
        asm volatile(".p2align 8\n\t.rept " LOOP_OFF_P_STR "\n\ts_nop 0\n\t.endr" ::: "memory");
        // slices 2i + 1 and 2i + 2 request the groups 2i + 4 and 2i + 5: slices 2i + 4 and 2i + 5, if there are any
        int t = 1;
        while (t < k_cnt - 1) {
            const bool more = t + L < k_cnt;               // the pair of slices t + 3, t + 4 exists
            const int n = more ? min((k_cnt - L - t + 1) / 2, (k_per_seg - iss_in_seg) / 2) : (k_cnt - 1 - t) / 2;
            const rsrc_t ra = more ? real_a() : rnull;
            const rsrc_t rb0 = more ? real_b0() : rnull;
            const rsrc_t rb1 = more ? rB[1] : rnull;
            for (int i = 0; i < n; ++i) {
                slice(std::integral_constant<int, 1>{}, std::false_type{}, ra, rb0, rb1);
                slice(std::integral_constant<int, 0>{}, std::false_type{}, ra, rb0, rb1);
            }
            t += 2 * n;
            if (more) group_fixups();
        }
        slice(std::integral_constant<int, 1>{}, std::false_type{}, rnull, rnull, rnull);      // the last slice
        WAIT_VMCNT(0);                                     // the zero-length requests too: the epilogue reuses the ring
        if (GEO::TWO_PHASE && wm == 0) BLOCK_BARRIER();    // both rows have passed the same number of barriers
        BLOCK_BARRIER();                                   // and everybody's requests have landed
      }
    }

    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");     // the last MFMAs have written back before the accumulators are read
    // partial tiles of a finishing launch: [unit][wave][register / 4][lane] as float4, every instruction moves 1 KB
    const bool uneven = LAST && first_slices && parts > 1;
    if (!FIN && parts > 1 && !uneven) {
        float4* ws4 = reinterpret_cast<float4*>(p.split_ws) + ((size_t)unit * NWAVES + wave) * (FM * FN) * 64 + lane;
        // fragments past the group's last row (TN: the last row of the gradient) are not kept
        const long rows_left = (KIND == KIND_TN ? p.Mout - m0 : a_row_end - a_row0) - wm * WM;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            if (i / 2 * 32 >= rows_left) continue;
#pragma unroll
            for (int j = 0; j < FN; ++j) ws4[(i * FN + j) * 64] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        continue;
    }
    // ---- epilogue.  A lane holds, per fragment, row l%16 and columns (l/16)*4 + 0..3: storing
    // from there would touch 8-byte pieces of 16 different rows per instruction.  Instead every wave
    // passes its 128 x 64 accumulators through its own LDS patch (two rows of fragments, 32 rows, at a time,
    // fp32) and reads them back row-major, 8 consecutive columns per lane, so that global loads and stores
    // move whole 128/256-byte row segments.  The patches lie at the top of LDS, above ring slots 0 and 1.
    unsigned char* patch = smem + (LDS_BYTES - (size_t)NWAVES * EP_WAVE) + wave * EP_WAVE;
    const int lrow = lane & 15, lcol = (lane >> 4) * 4;
    const long row_limit = (KIND == KIND_TN) ? (long)p.Mout : a_row_end;
    constexpr int CG = DUAL ? WN / 16 : WN / 8;            // 8-column groups per staged row that carry outputs
    const int erow = lane / CG, ecg = lane % CG;
    constexpr int ROWS_PER_PASS = 64 / CG;
    constexpr bool BWD1 = (EPI == EPI_BWD1_GELU || EPI == EPI_BWD1_SWIGLU);
    constexpr int N_PASS = EP_ROWS / ROWS_PER_PASS;        // passes per 32 staged rows
    // NN/NT: every store of the epilogue is issued whatever the tile looks like, as a buffer store whose resource
    // ends with the tile's last valid row (or has no length at all, for an output that is not written): no predicate
    // per row.  TN keeps ordinary predicated stores.
    constexpr bool UNCOND = (KIND != KIND_TN);
    const int wcol0 = n0 + (DUAL ? wn * (WN / 2) : wn * WN);           // first column of this wave: all of its columns exist or none
    buf_rsrc_t rO0 = buf_rsrc_t(), rO1 = buf_rsrc_t(), rO2 = buf_rsrc_t();
    if (UNCOND) {
        const bool cols = wcol0 < p.N;
        const long vrows = row_limit - m0 < BM ? row_limit - m0 : BM;       // the group may go on for millions of rows
        const int bytes = (int)(vrows * p.ldo * 2);
        auto out_rsrc = [&](bf16_t* base, bool on) {
            return __builtin_amdgcn_make_buffer_rsrc((void*)(base ? base + (long)m0 * p.ldo : p.O2), 0, (on && base && cols) ? bytes : 0, 0x00020000);
        };
        rO0 = out_rsrc(p.O0, true);
        rO1 = out_rsrc(p.O1, EPI == EPI_FWD1_SWIGLU || EPI == EPI_BWD1_SWIGLU);
        rO2 = out_rsrc(p.O2, BWD1 ? p.write_act != 0 : (EPI == EPI_FWD1_GELU || EPI == EPI_FWD1_SWIGLU));
    }
    // The saved pre-activations of the backward epilogue are requested a batch of passes ahead, into the second
    // of two register sets: a batch's loads are in flight while the batch before it is computed and stored, and,
    // memory operations completing in the order of issue, no load ever waits for a store issued before it.
#ifndef BWD1_BATCH
#define BWD1_BATCH 2
#endif
    constexpr int BATCH = BWD1 ? BWD1_BATCH : N_PASS;
    constexpr int NB = N_PASS / BATCH;                     // batches per 32 staged rows
    static_assert(N_PASS % BATCH == 0, "batches tile the passes of 32 staged rows");
    uint4 zin[BWD1 ? 2 : 1][BWD1 ? BATCH : 1], uin[EPI == EPI_BWD1_SWIGLU ? 2 : 1][EPI == EPI_BWD1_SWIGLU ? BATCH : 1];
    auto request = [&](int fr, int pb, uint4* zi, uint4* ui) {
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            // rows and columns past the end read the last valid ones (their results are not stored): no
            // predicate, no zero fill
            long row = (long)m0 + wm * WM + fr * EP_ROWS + (pb + k) * ROWS_PER_PASS + erow;
            row = row < row_limit ? row : row_limit - 1;
            const int col = min(n0 + wn * WN + ecg * 8, p.N - 8);
            zi[k] = *reinterpret_cast<const uint4*>(p.Zin + row * p.ldo + col);
            if (EPI == EPI_BWD1_SWIGLU) ui[k] = *reinterpret_cast<const uint4*>(p.Uin + row * p.ldo + col);
        }
    };
    // WHOLE: the tile's results.  Of a tile cut unevenly (LAST): KEEP leaves what this part holds in the workspace as it comes
    // out of the patches, [unit][wave][32 rows][pass][half][lane] as float4; SUM adds the other part from there to this
    // one's and goes on with the sum (of two terms: the same whichever part comes last).
    // Both go past the L2 of the XCD (sc1: coherent on the device, where every XCD has an L2 of its own), so that no L2 has to be
    // written back or invalidated for them: with plain accesses between agent-scope fences d = 1024, h = 4096, 152 tiles of 128
    // slices took 114 us where this takes 90 and whole tiles 108.
    constexpr int WHOLE = 0, SUM = 1, KEEP = 2, AT_DEVICE = 16;
    static_assert(!LAST || GEO::UNIT_BYTES == NWAVES * TM * N_PASS * 2 * 1024, "a part fills its unit");
    const long rows_left = row_limit - m0 - wm * WM;           // 32 rows past the last one are not kept
    auto part_rsrc = [&](int u) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)((char*)p.split_ws + (size_t)u * GEO::UNIT_BYTES), 0, GEO::UNIT_BYTES, 0x00020000);
    };
    int* counter = LAST ? p.arrived + unit / 2 : nullptr;
    auto tell = [&](int v) {                                   // what thread 0 knows, to all
        int* word = reinterpret_cast<int*>(smem);              // ring slot 0: below the patches
        if (tid == 0) *word = v;
        __syncthreads();
        const int r = __builtin_amdgcn_readfirstlane(*word);
        __syncthreads();
        return r;
    };
    // the other part is there already: this one need not be kept
    int before = 0;
    if (LAST && uneven) before = tell(tid == 0 ? __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0);
    // A loop, unrolled, and not a function called per mode: in the kernels without LAST it is no loop at all.  (As a lambda the
    // 256 x 256 bwd1 kernels, which have no mode but WHOLE, spilled 2 and 12 vector registers.)
#pragma unroll
    for (int mode = LAST ? KEEP : WHOLE; mode >= WHOLE; --mode) {
    if (LAST) {
        if (mode == WHOLE ? uneven : !uneven) continue;
        if (mode == KEEP && before != 0) continue;
        if (mode == SUM) {
            if (before != 1) continue;
            if (tid == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (BWD1 && !FIN) request(0, 0, zin[0], uin[0]);
#pragma unroll
    for (int fr = 0; fr < TM; ++fr) {
        if (mode != WHOLE && fr * 32 >= rows_left) continue;
        const int part_ofs = ((wave * TM + fr) * (N_PASS * 2 * 64) + lane) * 16;
        float4 other[LAST ? N_PASS : 1][2];
        if (LAST && mode == SUM) {
            const buf_rsrc_t from = part_rsrc(unit ^ 1);
#pragma unroll
            for (int i = 0; i < N_PASS; ++i)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    other[i][k] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(from, part_ofs + (i * 2 + k) * 1024, 0, AT_DEVICE));
        }
        if (FIN && fr != q % TM) continue;                     // the tile's other rows are items of other blocks
        if (BWD1 && FIN) request(fr, 0, zin[(fr * NB) & 1], uin[EPI == EPI_BWD1_SWIGLU ? (fr * NB) & 1 : 0]);
        float4 fsum[FIN ? 2 * FN : 1];
        if (FIN) {                                             // the parts of a split tile, added in ascending order
#pragma unroll
            for (int i = 0; i < 2 * FN; ++i) fsum[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (fr * 32 < row_limit - m0 - wm * WM) {
                constexpr long PART = (long)NWAVES * (FM * FN) * 64;
                const float4* ws4 = reinterpret_cast<const float4*>(p.split_ws) + unit * PART + (wave * (FM * FN) + fr * 2 * FN) * 64 + lane;
                // All loads of up to four parts, 32 KB of a wave, are on their way before the first is added (the compiler left to
                // itself waits for each: 13 us instead of 8 for 96 tiles in five parts).
                auto add_parts = [&](auto N, int s0) {
                    constexpr int n = decltype(N)::value;
                    float4 x[n][2 * FN];
#pragma unroll
                    for (int s = 0; s < n; ++s)
#pragma unroll
                        for (int i = 0; i < 2 * FN; ++i) x[s][i] = ws4[(s0 + s) * PART + i * 64];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int s = 0; s < n; ++s)
#pragma unroll
                        for (int i = 0; i < 2 * FN; ++i) {
                            fsum[i].x += x[s][i].x; fsum[i].y += x[s][i].y;
                            fsum[i].z += x[s][i].z; fsum[i].w += x[s][i].w;
                        }
                };
                constexpr int AT_ONCE = BWD1 ? 2 : 4;          // BWD1 holds saved pre-activations as well
                int s = 0;                                     // and no load for a part that is not there (five parts 9.1 -> 8.2 us)
#pragma unroll 1
                for (; s + AT_ONCE <= parts; s += AT_ONCE) add_parts(std::integral_constant<int, AT_ONCE>{}, s);
                if (AT_ONCE == 4 && parts - s == 3) add_parts(std::integral_constant<int, 3>{}, s);
                else if (AT_ONCE == 4 && parts - s == 2) add_parts(std::integral_constant<int, 2>{}, s);
                else if (parts - s == 1) add_parts(std::integral_constant<int, 1>{}, s);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4& a = acc[2 * fr + i][j];
                float4 val = make_float4(a[0], a[1], a[2], a[3]);
                if (FIN) val = fsum[i * FN + j];
                *reinterpret_cast<float4*>(patch + (i * 16 + lrow) * EP_PITCH + (j * 16 + lcol) * 4) = val;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int b = 0; b < NB; ++b) {
        const int pb = b * BATCH, cur = (fr * NB + b) & 1;
        if (BWD1) {
            const int nxt = fr * NB + b + 1;
            if (nxt < (FIN ? (fr + 1) * NB : TM * NB)) request(nxt / NB, (nxt % NB) * BATCH, zin[cur ^ 1], uin[cur ^ 1]);
        }
#pragma unroll
        for (int pass = pb; pass < pb + BATCH; ++pass) {
            const int r = pass * ROWS_PER_PASS + erow;                     // row inside the patch
            const int trow = wm * WM + fr * EP_ROWS + r;                   // row inside the tile
            const long row = (long)m0 + trow;
            const int col = wcol0 + ecg * 8;
            if (!UNCOND && (row >= row_limit || col >= p.N)) continue;
            float v[8], u[8];
            {
                // dual: fragments alternate x W1 / x W3, 32 columns each; group ecg sits in pair ecg/4
                const int c0 = DUAL ? ((ecg >> 2) * 64 + (ecg & 3) * 8) * 4 : ecg * 32;
                const float4 x0 = *reinterpret_cast<const float4*>(patch + r * EP_PITCH + c0);
                const float4 x1 = *reinterpret_cast<const float4*>(patch + r * EP_PITCH + c0 + 16);
                v[0] = x0.x; v[1] = x0.y; v[2] = x0.z; v[3] = x0.w; v[4] = x1.x; v[5] = x1.y; v[6] = x1.z; v[7] = x1.w;
            }
            if (DUAL) {                                                    // the next 32 columns of the patch hold x W3
                const int c1 = ((ecg >> 2) * 64 + 32 + (ecg & 3) * 8) * 4;
                const float4 x0 = *reinterpret_cast<const float4*>(patch + r * EP_PITCH + c1);
                const float4 x1 = *reinterpret_cast<const float4*>(patch + r * EP_PITCH + c1 + 16);
                u[0] = x0.x; u[1] = x0.y; u[2] = x0.z; u[3] = x0.w; u[4] = x1.x; u[5] = x1.y; u[6] = x1.z; u[7] = x1.w;
            }
            if (mode == KEEP) {
                const buf_rsrc_t to = part_rsrc(unit);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_float4(v[0], v[1], v[2], v[3])), to, part_ofs + pass * 2048, 0, AT_DEVICE);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_float4(v[4], v[5], v[6], v[7])), to, part_ofs + pass * 2048 + 1024, 0, AT_DEVICE);
                continue;
            }
            if (LAST && mode == SUM) {
                const float4 x0 = other[pass][0], x1 = other[pass][1];
                v[0] += x0.x; v[1] += x0.y; v[2] += x0.z; v[3] += x0.w; v[4] += x1.x; v[5] += x1.y; v[6] += x1.z; v[7] += x1.w;
            }
            const long o = row * p.ldo + col;
            const int bo = (int)(((long)trow * p.ldo + col) * 2);          // byte offset from the tile's first row
            auto pack8 = [](const float* f) {
                return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
            };
            auto unpack8 = [](const uint4 w, float* f) {
                f[0] = __uint_as_float(w.x << 16); f[1] = __uint_as_float(w.x & 0xffff0000u);
                f[2] = __uint_as_float(w.y << 16); f[3] = __uint_as_float(w.y & 0xffff0000u);
                f[4] = __uint_as_float(w.z << 16); f[5] = __uint_as_float(w.z & 0xffff0000u);
                f[6] = __uint_as_float(w.w << 16); f[7] = __uint_as_float(w.w & 0xffff0000u);
            };
            auto put = [&](buf_rsrc_t r, const uint4 w) {      // rows past the tile's last one fall outside the resource
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), r, bo, 0, 0);
            };
            if (EPI == EPI_BF16) {
                put(rO0, pack8(v));
            } else if (EPI == EPI_F32) {
                float* dst = p.OF + (long)g * p.o_group_stride + o;
                if (p.accumulate) {
                    const float4 o0 = *reinterpret_cast<const float4*>(dst), o1 = *reinterpret_cast<const float4*>(dst + 4);
                    v[0] += o0.x; v[1] += o0.y; v[2] += o0.z; v[3] += o0.w;
                    v[4] += o1.x; v[5] += o1.y; v[6] += o1.z; v[7] += o1.w;
                }
                *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
            } else if (EPI == EPI_FWD1_GELU) {
                float a[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) a[e] = gelu_f(v[e]);
                put(rO0, pack8(v));                            // no length in a forward-only pass: Z is not kept
                put(rO2, pack8(a));
            } else if (EPI == EPI_FWD1_SWIGLU) {
                float a[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) a[e] = v[e] * sigmoid_f(v[e]) * u[e];
                put(rO0, pack8(v));                            // no length in a forward-only pass: Z and U are not kept
                put(rO1, pack8(u));
                put(rO2, pack8(a));
            } else if (EPI == EPI_BWD1_GELU) {
                float z[8], dz[8];
                unpack8(zin[cur][pass - pb], z);
#pragma unroll
                for (int e = 0; e < 8; ++e) dz[e] = v[e] * gelu_grad_f(z[e]);
                uint4 aw = make_uint4(0, 0, 0, 0);
                if (p.write_act) {
                    float a[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) a[e] = gelu_f(z[e]);
                    aw = pack8(a);
                }
                put(rO0, pack8(dz));
                put(rO2, aw);                                  // no length when the forward pass's activation is still there
            } else if (EPI == EPI_BWD1_SWIGLU) {
                // silu(z) = z s and silu'(z) = s + z s (1 - s) with s = sigmoid(z): eight vector instructions and
                // two transcendentals per element (this epilogue is bound by its vector instructions)
                float z[8], uu[8], dz[8], du[8], zs[8];
                unpack8(zin[cur][pass - pb], z);
                unpack8(uin[cur][pass - pb], uu);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float sg = sigmoid_f(z[e]);
                    zs[e] = z[e] * sg;
                    du[e] = v[e] * zs[e];
                    dz[e] = (v[e] * uu[e]) * __builtin_fmaf(zs[e], 1.0f - sg, sg);
                }
                uint4 aw = make_uint4(0, 0, 0, 0);
                if (p.write_act) {
                    float a[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) a[e] = zs[e] * uu[e];
                    aw = pack8(a);
                }
                put(rO0, pack8(dz));
                put(rO1, pack8(du));
                put(rO2, aw);                                  // no length when the forward pass's activation is still there
            }
        }
        }
    }
    if (mode == KEEP) {
        // Every wave's stores are complete before the barrier, and thread 0 counts this part after it.  Nobody waits for the
        // other part: whichever is counted last goes on with the tile.
        WAIT_VMCNT(0);
        __syncthreads();
        if (tid == 0) before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = tell(before);
    }
    }
    __syncthreads();             // every wave is done with its patch before the next tile's DMA lands there
  }
}

// ---- host side ----------------------------------------------------------------------------------
// ---- which geometry ------------------------------------------------------------------------------
// Large multiplies a quarter faster once its tiles fill the chip several times over (train-size contractions: 0.72 us per
// slice and round of 256 tiles, where Small takes 0.55 per round of 512 tiles a quarter as large), Small wins where Large
// leaves CUs idle, rounds up to a round it does not need, or spends its time in prologues and epilogues that nothing hides:
// there one of Small's two blocks per CU multiplies while the other stores, and its tiles and parts are four times finer.
// Measured, us, Large | Small (with the finishing launch):  d = 768, h = 3072, 1987 rows in 5 groups: forward 48 + 68 | 41 +
// 33, backward 35 + 74 + 2 x 57 | 24 + 45 + 2 x 36;  d = 1024, h = 1024, 1262 rows: 36 + 27 | 25 + 27;  d = 2944, h = 576,
// 3002 rows: 76 + 25 | 36 + 22;  d = 1024, h = 4096, 9279 rows: 123 + 111 | 134 + 118, weight gradients 156 | 126 each;
// d = 2048, h = 8192, 11742 rows: 444 + 405 | 560 + 478, 420 | 560 each;  29112 rows: 980 + 800 | 1237 + 1050, 850 | 1440.
// The host knows T k and how many of the experts are hosted here, not how many rows they got: it estimates 0.8 T k
// sqrt(G / E) (more than the share of an even load, G / E, while that is below 0.64: hosted experts are the popular ones; a
// fifth less than all rows where all experts are hosted, which chose no worse than all of them) and compares the two by the
// times above, which are those of 256 CUs, of 32x32x16 matrix instructions, and know nothing of uneven cuts.  With those of
// now, over 160 drawn shapes, a contraction takes 3.0 % more than in the better geometry in the mean and up
// to 1.5 times (d = 768, h = 3072, 16 experts of which 5 are hosted, 1999 tokens: fwd1 42 in Large, 34 in Small).  With those of then, over 250 drawn shapes (200 to 40000 rows, d 256 to
// 3072, h 1792 to 12800, 1 to 16 groups of any evenness) the forward pass is within 2.1 % of the best of the four choices for
// its two contractions in the mean, at worst 1.32 times as long (2333 tokens, k = 2, d = 1536, h = 3136, GELU, 8 groups: Large twice 156,
// Small 118); the weight gradients, over 660 shapes (to 60000 rows, 32 groups), within 0.6 % of the better one.
struct GeometryCost { double slice, over_bf16, over_fwd1, over_bwd1, finish, hbm; int tiles_at_once, split_max; };   // us, us, TB/s
constexpr GeometryCost LARGE_COST{0.70, 11.0, 15.0, 18.0, 14.0, 4.2, 256, 4}, SMALL_COST{0.55, 6.5, 9.0, 10.0, 10.0, 5.0, 512, 8};

inline double estimated_rows(const moe_shape_t& s)
{
    const double A = (double)s.T * s.k;
    return std::max(1.0, std::min(A, 0.8 * A * std::sqrt((double)s.G / s.E)));
}
inline double tiles_of(const moe_shape_t& s, int bm, int cols, int bn)
{
    const double rows = estimated_rows(s), groups = std::min((double)s.G, rows);      // as if spread evenly
    return groups * std::ceil(rows / s.G < 1.0 ? 1.0 / bm : rows / s.G / bm) * ((cols + bn - 1) / bn);
}
double row_contraction_cost(const GeometryCost& c, double tiles, int slices, int epi, int split_slices, double weight_mb)
{
    const double over = epi == EPI_BF16 ? c.over_bf16 : ((epi == EPI_FWD1_GELU || epi == EPI_FWD1_SWIGLU) ? c.over_fwd1 : c.over_bwd1);
    const double x = tiles / c.tiles_at_once;
    const bool split = slices >= 2 * split_slices;
    double t;
    if (x <= 1.0) {
        const int S = std::max(1, std::min(std::min(c.split_max, (int)(1.0 / x)), slices / split_slices));
        t = c.slice * slices / S + over + (S > 1 ? c.finish : (split ? 5.0 : 0.0));
    } else {
        t = split ? (x + 0.3) * (c.slice * slices + over) + c.finish : (x + 0.5) * (c.slice * slices + over);
    }
    return std::max(t, weight_mb / c.hbm);
}
constexpr int SMALL_SPLIT_SLICES = 16;
constexpr int SMALL_BAND = 8;                              // 64 tiles in flight on an XCD: 8 x 8 of 128 x 128
// weight gradients: what a tile costs beside its slices, in slices, and the least slices of a part
template <class GEO> constexpr int TN_OVER = GEO::BLOCKS == 1 ? 24 : 16;
template <class GEO> constexpr int TN_SPLIT_SLICES = GEO::BLOCKS == 1 ? 48 : 32;
template <class GEO> constexpr int SPLIT_MAX = GEO::BLOCKS == 1 ? LARGE_COST.split_max : SMALL_COST.split_max;
template <class GEO> constexpr int SPLIT_CAP = (int)((size_t)SPLIT_UNITS * Large::UNIT_BYTES / GEO::UNIT_BYTES);
template <class GEO> constexpr int UNEVEN_CAP = (int)((size_t)UNEVEN_UNITS * Large::UNIT_BYTES / GEO::UNIT_BYTES);
// Large: a part of a split tile has to be worth its 256-KB round trip, 64 slices where the split only shortens the last of
// several rounds, 24 where it is what fills the chip (d = 768, h = 3072, 33 tiles of 96 slices: 69 us whole, 45 in four parts).
inline int large_split_slices(double tiles) { return tiles <= 2.0 * LARGE_COST.tiles_at_once ? 24 : 64; }

bool small_wins_rows(const moe_shape_t& s, int N, int slices, int n_seg, int epi)
{
    const bool dual = epi == EPI_FWD1_SWIGLU;
    const double tl = tiles_of(s, Large::BM, N, dual ? Large::BN / 2 : Large::BN), ts = tiles_of(s, Small::BM, N, dual ? Small::BN / 2 : Small::BN);
    const double mb = std::min((double)s.G, estimated_rows(s)) * s.d * s.h * 2.0 * (dual ? 2 : n_seg) / 1e6;
    GeometryCost sc = SMALL_COST;
    if (dual) sc.hbm = 3.0;                                // 128-byte pieces of two weight matrices
    return row_contraction_cost(sc, ts, slices, epi, SMALL_SPLIT_SLICES, mb) < row_contraction_cost(LARGE_COST, tl, slices, epi, large_split_slices(tl), mb);
}
// Weight gradients.  Whole groups: a round of an XCD's blocks per 32 (64) tiles of a group, dealt to the 8 XCDs, 17 (9) us
// per tile beside the slices (the fp32 tile is stored), and no less than the chain of a group with twice its even share of
// the rows.  Cut groups: every block its share, and a finishing launch of about 20 (12) us.  A cut pays where a group has
// fewer tiles than there are blocks and is longer than an XCD's share of all rounds, and the kernel, which alone knows, only
// makes one where it finds such a group; it is offered wherever four times a group's even share is longer than a block's.
struct WgradPlan { double us; bool cut; };
template <class GEO>
WgradPlan wgrad_plan(const moe_shape_t& s, int Mout, int N)
{
    constexpr bool large = GEO::BLOCKS == 1;
    constexpr double slice = large ? 0.70 : 0.55, over = large ? 17.0 : 9.0, finish = large ? 20.0 : 12.0;
    constexpr int blocks = large ? 256 : 512, over_slices = TN_OVER<GEO>, least = TN_SPLIT_SLICES<GEO>;
    const double tiles = (double)((Mout + GEO::BM - 1) / GEO::BM) * ((N + GEO::BN - 1) / GEO::BN);
    const double even = std::ceil(estimated_rows(s) / s.G / BK), all = std::ceil(estimated_rows(s) / BK);
    const double whole = std::max(std::max(s.G * std::ceil(tiles / (blocks / 8)) / 8.0, 1.0) * (even * slice + over),
                                  std::min(2.0 * even, all) * slice + over);
    const double share = tiles * s.G * (even + over_slices) / blocks, longest = std::min(4.0 * even, all);
    if (tiles >= blocks || longest < 2 * least || longest + over_slices < 1.25 * share) return WgradPlan{whole, false};
    const double cut = std::max(share, (double)least) * slice + over + finish;
    return cut < whole ? WgradPlan{cut, true} : WgradPlan{whole, false};
}

// Whether the forward pass requests its weights past the caches.  A group has one row tile at most (a decoding step), so no two blocks
// share a weight (where several row tiles do, in L2, such requests take 1.8 times as long), and the layer's weights are more than the
// 256 MB on the memory side keep for its next call.  One layer called again, us with plain | nontemporal requests (8 tokens; 64): GELU of
// 235 MB 80.2 | 80.8; 88.5 | 91.1, of 268 MB 91.4 | 91.7; 93.8 | 97.9, of 285 MB 88.9 | 86.8; 107.8 | 103.9, of 403 MB 111.7 | 106.5; 127.9 |
// 117.9; SwiGLU of 252 MB 81.3 | 85.9; 111.9 | 116.2, of 302 MB 98.5 | 97.4; 106.9 | 102.6, of 1.4 GB 131 | 126; 308 | 287.  Layers of less that are
// more than that together gain as well (four of 101 MB 67.8 | 63.6), but a layer does not know of the others, and those that fit lose (eight
// of 25 MB 48.5 | 50.2).
constexpr size_t MEMORY_SIDE_CACHE = (size_t)256 << 20;
inline bool read_once(const moe_shape_t& s, int BM)
{
    return (long)s.T * s.k <= BM && (size_t)s.G * s.d * s.h * (s.act == MOE_ACT_SWIGLU ? 3 : 2) * sizeof(bf16_t) > MEMORY_SIDE_CACHE;
}
// Kernels with such requests: Large only for both weight matrices of SwiGLU.  (The cost rule takes it for nothing else of so few rows; it
// would run with plain requests.)
template <int KIND, int EPI, class GEO> constexpr bool HAS_ONCE = KIND == KIND_NN && (GEO::BM == Small::BM || EPI == EPI_FWD1_SWIGLU);

template <int KIND, int EPI, class GEO>
hipError_t launch_geo(GemmParams p, int rows_upper, int n_groups_cap, bool once_read, bool finish, hipStream_t st)
{
    constexpr bool DUAL = (EPI == EPI_FWD1_SWIGLU);
    constexpr int BM = GEO::BM;
    constexpr size_t LDS_BYTES = GEO::LDS_BYTES;
    const int bn = DUAL ? GEO::BN / 2 : GEO::BN;
    p.col_tiles = (p.N + bn - 1) / bn;
    if (KIND == KIND_TN) {
        p.row_tiles = (p.Mout + BM - 1) / BM;
        p.n_tiles = n_groups_cap * p.row_tiles * p.col_tiles;
    } else {
        p.row_tiles = (rows_upper + BM - 1) / BM + n_groups_cap;      // upper bound; the kernel counts the real ones
        p.n_tiles = p.row_tiles * p.col_tiles;
    }
    if (p.n_tiles == 0) return hipSuccess;
    // persistent: as many blocks as fit the CUs (their LDS allows no more), a multiple of 8.  The CU count and the kernels' dynamic
    // LDS limit are looked up / set once per device (per instantiation).
    static PerDeviceOnce once;
    static std::atomic<int> cus_of[64];
    const int dev = current_device();
    int cus = (dev >= 0 && dev < 64) ? cus_of[dev].load(std::memory_order_acquire) : 0;
    auto kern = grouped_gemm_kernel<KIND, EPI, false, GEO, false, false>;
    auto kern_last = grouped_gemm_kernel<KIND, EPI, false, GEO, last_finishes(EPI), false>;
    auto kern_once = grouped_gemm_kernel<KIND, EPI, false, GEO, false, HAS_ONCE<KIND, EPI, GEO>>;
    auto kern_last_once = grouped_gemm_kernel<KIND, EPI, false, GEO, last_finishes(EPI), HAS_ONCE<KIND, EPI, GEO>>;
    auto kern_fin = grouped_gemm_kernel<KIND, EPI, true, GEO, false, false>;
    if (!once.is_done(dev) || cus == 0) {
        int n = 0;
        if (dev < 0 || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
        cus = n / 8 * 8;
        for (auto k : {kern, kern_last, kern_once, kern_last_once, kern_fin}) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
            if (e != hipSuccess) return e;
        }
        if (dev >= 0 && dev < 64) cus_of[dev].store(cus, std::memory_order_release);
        once.mark(dev);
    }
    const int grid = cus * GEO::BLOCKS;
    p.tn_over = TN_OVER<GEO>;
    p.split_max = SPLIT_MAX<GEO>;
    p.split_cap = SPLIT_CAP<GEO>;
    hipLaunchKernelGGL(once_read ? (p.uneven_cap > 0 ? kern_last_once : kern_once) : (p.uneven_cap > 0 ? kern_last : kern), dim3(grid), dim3(GEO::THREADS), LDS_BYTES, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !finish) return e;
    // the tiles of split contractions: add their parts, run their epilogues
    hipLaunchKernelGGL(kern_fin, dim3(grid), dim3(GEO::THREADS), LDS_BYTES, st, p);
    return hipGetLastError();
}

// Two remainders a block at least.
inline bool long_enough_for_uneven(int slices) { return slices >= 3 * UNEVEN_SLICES + 2 * UNEVEN_OVER; }

// The geometry of a contraction and whether it may be cut (then a finishing launch follows).
// uneven: the tiles of a last round may be cut unevenly.
struct Tiling { bool small, cut; int split_slices; bool uneven; };
Tiling row_tiling(const moe_shape_t& s, int N, int slices, int n_seg, int epi)
{
    Tiling t;
    t.small = small_wins_rows(s, N, slices, n_seg, epi);
    t.split_slices = t.small ? SMALL_SPLIT_SLICES : large_split_slices(tiles_of(s, Large::BM, N, epi == EPI_FWD1_SWIGLU ? Large::BN / 2 : Large::BN));
    t.cut = slices >= 2 * t.split_slices;                  // else too short
    t.uneven = last_finishes(epi) && long_enough_for_uneven(slices);
    return t;
}
Tiling wgrad_tiling(const moe_shape_t& s, int Mout, int N)
{
    const WgradPlan l = wgrad_plan<Large>(s, Mout, N), m = wgrad_plan<Small>(s, Mout, N);
    const bool small = m.us < l.us;
    return Tiling{small, small ? m.cut : l.cut, small ? TN_SPLIT_SLICES<Small> : TN_SPLIT_SLICES<Large>, false};
}

template <int KIND, int EPI>
hipError_t launch(GemmParams p, const moe_shape_t& s, hipStream_t st)
{
    const Tiling t = KIND == KIND_TN ? wgrad_tiling(s, p.Mout, p.N) : row_tiling(s, p.N, p.n_seg * (p.Kseg / BK), p.n_seg, EPI);
    if (!t.cut && !t.uneven) p.split_ws = nullptr;
    p.split_slices = t.cut ? t.split_slices : 0x7fffffff;  // none is worth it
    p.uneven_cap = t.uneven ? (t.small ? UNEVEN_CAP<Small> : UNEVEN_CAP<Large>) : 0;
    if (KIND != KIND_TN && t.small) p.band = SMALL_BAND;
    return t.small ? launch_geo<KIND, EPI, Small>(p, s.T * s.k, s.G, KIND == KIND_NN && read_once(s, Small::BM), t.cut, st)
                   : launch_geo<KIND, EPI, Large>(p, s.T * s.k, s.G, KIND == KIND_NN && read_once(s, Large::BM), t.cut, st);
}

GemmParams base_params(const moe_shape_t& s, const ffn_args& a)
{
    GemmParams p{};
    p.slot_offsets = a.slot_offsets; p.dest_slots = a.dest_slots;
    p.self = s.self; p.Gcap = s.G;
    p.n_seg = 1;
    p.split_ws = a.split_ws;
    p.arrived = a.arrived;
    return p;
}

}  // namespace

// The longest contractions that may be cut unevenly are those over h, of dZ and dU together where there are two.
int ffn_split_units(const moe_shape_t& s)
{
    return long_enough_for_uneven((s.act == MOE_ACT_SWIGLU ? 2 : 1) * (s.h / BK)) ? UNEVEN_UNITS : SPLIT_UNITS;
}

hipError_t launch_ffn_fwd_bf16(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const int A = s.T * s.k;
    if (A == 0) return hipSuccess;
    const long d = s.d, h = s.h;
    hipError_t e;
    {   // fwd1: [rows, d] x W1[g] (d x h)
        GemmParams p = base_params(s, a);
        p.band = BAND_FWD1;
        p.clear_arrived = 1;
        p.A[0] = (const bf16_t*)a.Xp; p.B[0] = (const bf16_t*)a.W1; p.B_dual = (const bf16_t*)a.W3;
        p.lda = d; p.ldb = h; p.b_group_stride = d * h; p.Kseg = s.d; p.N = s.h;
        p.O0 = (bf16_t*)a.Z; p.O1 = (bf16_t*)a.U; p.O2 = (bf16_t*)a.Act; p.ldo = h;
        e = (s.act == MOE_ACT_SWIGLU) ? launch<KIND_NN, EPI_FWD1_SWIGLU>(p, s, st)
                                      : launch<KIND_NN, EPI_FWD1_GELU>(p, s, st);
        if (e != hipSuccess) return e;
    }
    {   // fwd2: Act [rows, h] x W2[g] (h x d)
        GemmParams p = base_params(s, a);
        p.band = BAND_FWD2;
        p.A[0] = (const bf16_t*)a.Act; p.B[0] = (const bf16_t*)a.W2;
        p.lda = h; p.ldb = d; p.b_group_stride = d * h; p.Kseg = s.h; p.N = s.d;
        p.O0 = (bf16_t*)a.Yp; p.ldo = d;
        e = launch<KIND_NN, EPI_BF16>(p, s, st);
    }
    return e;
}

hipError_t launch_ffn_bwd_bf16(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const int A = s.T * s.k;
    const long d = s.d, h = s.h;
    const bool swiglu = s.act == MOE_ACT_SWIGLU;
    hipError_t e = hipSuccess;
    if (A > 0) {
        {   // bwd1: dA = dYp [rows, d] x W2[g]^T (W2 is h x d: contraction index contiguous)
            GemmParams p = base_params(s, a);
            p.band = BAND_BWD1;
            p.clear_arrived = 1;
            p.A[0] = (const bf16_t*)a.dYp; p.B[0] = (const bf16_t*)a.W2;
            p.lda = d; p.ldb = d; p.b_group_stride = d * h; p.Kseg = s.d; p.N = s.h;
            p.O0 = (bf16_t*)a.dZ; p.O1 = (bf16_t*)a.dU; p.O2 = (bf16_t*)a.Act; p.ldo = h;
            p.Zin = (const bf16_t*)a.Z; p.Uin = (const bf16_t*)a.U;
            p.write_act = a.act_saved ? 0 : 1;
            e = swiglu ? launch<KIND_NT, EPI_BWD1_SWIGLU>(p, s, st)
                       : launch<KIND_NT, EPI_BWD1_GELU>(p, s, st);
            if (e != hipSuccess) return e;
        }
        {   // bwd2: dXp = dZ [rows, h] x W1[g]^T (+ dU x W3[g]^T)
            GemmParams p = base_params(s, a);
            p.band = BAND_BWD2;
            p.A[0] = (const bf16_t*)a.dZ; p.B[0] = (const bf16_t*)a.W1;
            p.A[1] = (const bf16_t*)a.dU; p.B[1] = (const bf16_t*)a.W3;
            p.n_seg = swiglu ? 2 : 1;
            p.lda = h; p.ldb = h; p.b_group_stride = d * h; p.Kseg = s.h; p.N = s.d;
            p.O0 = (bf16_t*)a.dXp; p.ldo = d;
            e = launch<KIND_NT, EPI_BF16>(p, s, st);
            if (e != hipSuccess) return e;
        }
    }
    // weight gradients: contraction over the rows of each group
    auto wgrad = [&](const void* L, long ldl, int Mout, const void* R, long ldr, int N, float* out) {
        GemmParams p = base_params(s, a);
        p.band = BAND_WGRAD;
        p.A[0] = (const bf16_t*)L; p.B[0] = (const bf16_t*)R;
        p.lda = ldl; p.ldb = ldr; p.b_group_stride = 0; p.Mout = Mout; p.N = N;
        p.OF = out; p.ldo = N; p.o_group_stride = d * h; p.accumulate = a.accumulate ? 1 : 0;
        return launch<KIND_TN, EPI_F32>(p, s, st);
    };
    e = wgrad(a.Xp, d, s.d, a.dZ, h, s.h, a.dW1);
    if (e != hipSuccess) return e;
    if (swiglu) {
        e = wgrad(a.Xp, d, s.d, a.dU, h, s.h, a.dW3);
        if (e != hipSuccess) return e;
    }
    return wgrad(a.Act, h, s.h, a.dYp, d, s.d, a.dW2);
}

int moe_ffn_reads_once(moe_handle_t hd, int contraction)
{
    if (!hd) return MOE_ERR_NULL;
    const moe_shape_t& s = hd->s;
    if (s.dtype != MOE_BF16) return MOE_ERR_DTYPE;
    if (contraction < 0 || contraction > 1) return MOE_ERR_SHAPE;
    const bool wide = contraction == 0, dual = wide && s.act == MOE_ACT_SWIGLU;
    const Tiling t = row_tiling(s, wide ? s.h : s.d, (wide ? s.d : s.h) / BK, 1, wide ? (dual ? EPI_FWD1_SWIGLU : EPI_FWD1_GELU) : EPI_BF16);
    return t.small ? read_once(s, Small::BM) : dual && read_once(s, Large::BM);
}

int moe_ffn_tiling(moe_handle_t hd, int contraction, int cus, int n_groups, const int32_t* rows, int32_t* out)
{
    if (!hd || !rows || !out) return MOE_ERR_NULL;
    const moe_shape_t& s = hd->s;
    if (s.dtype != MOE_BF16) return MOE_ERR_DTYPE;
    if (contraction < 0 || contraction > 5 || cus < 8 || n_groups < 0 || n_groups > s.G) return MOE_ERR_SHAPE;
    const bool swiglu = s.act == MOE_ACT_SWIGLU, wgrad = contraction >= 4, wide = contraction == 0 || contraction == 2;
    const int epi = contraction == 0 ? (swiglu ? EPI_FWD1_SWIGLU : EPI_FWD1_GELU)
                  : contraction == 2 ? (swiglu ? EPI_BWD1_SWIGLU : EPI_BWD1_GELU) : EPI_BF16;
    const int Mout = contraction == 5 ? s.h : s.d, N = wgrad ? (contraction == 5 ? s.d : s.h) : (wide ? s.h : s.d);
    const int n_seg = contraction == 3 && swiglu ? 2 : 1, slices = n_seg * ((wide ? s.d : s.h) / BK);
    const Tiling t = wgrad ? wgrad_tiling(s, Mout, N) : row_tiling(s, N, slices, n_seg, epi);
    const int side = t.small ? Small::BM : Large::BM, bn = epi == EPI_FWD1_SWIGLU ? side / 2 : side;
    const int nblk = cus / 8 * 8 * (t.small ? Small::BLOCKS : Large::BLOCKS);
    const int split_max = t.small ? SPLIT_MAX<Small> : SPLIT_MAX<Large>, cap = t.small ? SPLIT_CAP<Small> : SPLIT_CAP<Large>;
    const int band[5] = {BAND_FWD1, BAND_FWD2, BAND_BWD1, BAND_BWD2, BAND_WGRAD};
    int row_tiles = 0, all = 0;
    for (int g = 0; g < n_groups; ++g) { row_tiles += (rows[g] + side - 1) / side; all += (rows[g] + BK - 1) / BK; }
    if (wgrad) row_tiles = (Mout + side - 1) / side;
    const int col_tiles = (N + bn - 1) / bn, tiles = row_tiles * col_tiles, n_full = wgrad ? tiles : tiles / nblk * nblk;
    out[0] = side; out[1] = nblk; out[2] = row_tiles; out[3] = col_tiles; out[4] = n_full;
    out[5] = !wgrad && t.cut ? row_parts(tiles - n_full, nblk, slices, split_max, t.split_slices, cap) : 1;
    out[6] = t.small && !wgrad ? SMALL_BAND : band[wgrad ? 4 : contraction];
    out[7] = t.cut; out[8] = wgrad ? all : slices; out[9] = (int32_t)estimated_rows(s);
    if (!wgrad) {
        int turns;
        out[10] = t.uneven && out[5] == 1 ? uneven_cut(tiles - n_full, nblk, slices, t.small ? UNEVEN_CAP<Small> : UNEVEN_CAP<Large>, turns) : 0;
        return MOE_OK;
    }
    const int over = t.small ? TN_OVER<Small> : TN_OVER<Large>, rounds = (tiles + nblk / 8 - 1) / (nblk / 8);
    int* parts = out + 10;
    auto limit = [&](int most) { for (int g = 0; g < s.G; ++g) parts[g] = std::min<int>(parts[g], most); };
    auto n_cut = [&] { return (int)std::count_if(parts, parts + s.G, [](int32_t n) { return n > 1; }); };
    for (int g = 0; g < s.G; ++g)
        parts[g] = t.cut && g < n_groups ? tn_parts((rows[g] + BK - 1) / BK, tiles, rounds, all, s.G, nblk, over, split_max, t.split_slices) : 1;
    if (n_cut()) limit(tn_most_units(cap, tiles, n_cut()));
    if (std::accumulate(parts, parts + s.G, 0) > 64) limit(tn_most_lanes(s.G, n_cut()));
    if (n_cut()) {
        int longest = 0, len = 0, n = 0, total = 0;        // of the groups with rows
        for (int g = 0; g < n_groups; ++g) {
            const int k = (rows[g] + BK - 1) / BK;
            longest = std::max(longest, k); len = std::max(len, (k + parts[g] - 1) / parts[g]);
            n += k > 0; total += k > 0 ? parts[g] : 0;
        }
        if (!tn_pays(longest, len, all, n, total, rounds, over)) limit(1);
    }
    out[5] = *std::max_element(parts, parts + s.G);
    return MOE_OK;
}
