// Gate logits in a fixed fp32 summation order, top-k routing and gate weights (Section 2.1 of
// the paper: the gate relates every input to all experts and routes it to the top-k), and the
// gradient of the gate weights with respect to the logits.
//
// Summation order of logit[t,e] (what makes routing reproducible bit for bit): two partial sums; the
// columns are taken in blocks of 32 and block B belongs to partial B mod 2; inside a block the columns
// are visited as c = 32B + 8q + j with j = 0..7 outer and q = 0..3 inner, one fused multiply-add each;
// logit = (s0 + s1) + bias.  This is the order in which the 16x16x4 fp32 matrix instruction accumulates
// (four fused multiply-adds in ascending k, denormals kept) when a lane feeds it the 8 consecutive
// columns it loaded with one 16-byte request, so the whole contraction runs on the matrix cores.
#include "internal.h"
#include <type_traits>

namespace {

constexpr int GATE_WAVES = 4;                 // waves per block, 16 tokens each
constexpr int GATE_THREADS = GATE_WAVES * 64;
constexpr int GATE_TOK = GATE_WAVES * 16;     // tokens per block

typedef float gate_f4 __attribute__((ext_vector_type(4)));
typedef unsigned gate_u4 __attribute__((ext_vector_type(4)));

// Eight consecutive columns of one token, as loaded.
template <typename XT> struct XPiece;
template <> struct XPiece<bf16_t> { uint4 v; };
template <> struct XPiece<float> { float4 a, b; };

// Loads.  FULL (d % 64 == 0, every staged expert exists): a request is either inside the matrix or belongs to a
// chunk past the end that is never multiplied, so its address is clamped and nothing is selected; the request stays
// unconditional, which matters: a load under a condition makes the compiler drain all outstanding requests at the
// join.  Otherwise columns at or past d and experts at or past E are replaced by zeros.
template <bool VEC, bool FULL>
__device__ __forceinline__ void load_piece(XPiece<bf16_t>& p, const bf16_t* row, int c, int d)
{
    // bf16 shapes have d % 64 == 0: a piece is inside the row or past it
    const uint4 v = *reinterpret_cast<const uint4*>(row + (c < d ? c : 0));
    if (FULL) p.v = v;
    else p.v = (c < d) ? v : make_uint4(0u, 0u, 0u, 0u);
}
template <bool VEC, bool FULL>
__device__ __forceinline__ void load_piece(XPiece<float>& p, const float* row, int c, int d)
{
    if (FULL) {
        p.a = *reinterpret_cast<const float4*>(row + (c < d ? c : 0));
        p.b = *reinterpret_cast<const float4*>(row + (c < d ? c + 4 : 0));
    } else if (VEC) {                           // d % 4 == 0: each half is inside the row or past it
        const float4 a = *reinterpret_cast<const float4*>(row + (c < d ? c : 0));
        const float4 b = *reinterpret_cast<const float4*>(row + (c + 4 < d ? c + 4 : 0));
        p.a = (c < d) ? a : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        p.b = (c + 4 < d) ? b : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float x = row[c + j < d ? c + j : 0];
            v[j] = (c + j < d) ? x : 0.0f;
        }
        p.a = make_float4(v[0], v[1], v[2], v[3]);
        p.b = make_float4(v[4], v[5], v[6], v[7]);
    }
}
template <int J> __device__ __forceinline__ float piece_get(const XPiece<bf16_t>& p)
{
    const uint32_t w = (J / 2 == 0) ? p.v.x : (J / 2 == 1) ? p.v.y : (J / 2 == 2) ? p.v.z : p.v.w;
    return __uint_as_float((J & 1) ? (w & 0xffff0000u) : (w << 16));
}
template <int J> __device__ __forceinline__ float piece_get(const XPiece<float>& p)
{
    const float4& h = (J < 4) ? p.a : p.b;
    return (J % 4 == 0) ? h.x : (J % 4 == 1) ? h.y : (J % 4 == 2) ? h.z : h.w;
}

// Top-k, softmax and gate weights of a token by L lanes (lane = L * token + part; part holds the logits of the experts
// part, part + L, ... in registers): every lane proposes its best remaining logit, log2(L) exchange steps pick the winner
// by (value descending, index ascending), which is the order of a serial scan with NaN ranked as -inf; the softmax sum
// is folded the same way.  All 64 lanes take part in the exchanges; `store` says whether the token exists.
template <int L, int EPL>
__device__ __forceinline__ void route_lanes(const float* lg, int part, int t, bool store, int E, int k, int renorm,
                                            int32_t* __restrict__ idx, float* __restrict__ wout)
{
    constexpr int MAXK = 8;
    float v[EPL];
    unsigned long long left = 0ull;                        // logits of this lane not chosen yet
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = part + L * i;
        const float x = lg[e < E ? e : 0];
        v[i] = (x != x) ? -INFINITY : x;
        if (e < E) left |= 1ull << i;
    }
    const unsigned long long all = left;
    int sel[MAXK];
    float selv[MAXK];
#pragma unroll
    for (int j = 0; j < MAXK; ++j) {
        if (j >= k) break;
        int bi = -1;
        float bv = -INFINITY;
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (((left >> i) & 1ull) && (bi < 0 || v[i] > bv)) { bi = i; bv = v[i]; }
        int best = bi < 0 ? 0x7fffffff : part + L * bi;
#pragma unroll
        for (int off = 1; off < L; off <<= 1) {
            const float ov = __shfl_xor(bv, off, 64);
            const int oi = __shfl_xor(best, off, 64);
            if (oi != 0x7fffffff && (best == 0x7fffffff || ov > bv || (ov == bv && oi < best))) { bv = ov; best = oi; }
        }
        if (best % L == part) left &= ~(1ull << (best / L));
        sel[j] = best;
        selv[j] = bv;
    }
    const float m = selv[0];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < EPL; ++i)
        if ((all >> i) & 1ull) sum += expf(v[i] - m);
#pragma unroll
    for (int off = 1; off < L; off <<= 1) sum += __shfl_xor(sum, off, 64);
    float psum = 0.0f;
#pragma unroll
    for (int j = 0; j < MAXK; ++j) {
        if (j >= k) break;
        selv[j] = expf(selv[j] - m) / sum;
        psum += selv[j];
    }
    if (store && part == 0)
#pragma unroll
        for (int j = 0; j < MAXK; ++j) {
            if (j >= k) break;
            idx[(size_t)t * k + j] = sel[j];
            wout[(size_t)t * k + j] = renorm ? selv[j] / psum : selv[j];
        }
}

// One block = 64 tokens, wave w = tokens 16w..16w+15 over the whole contraction; NT tiles of 16 experts per
// pass.  MFMA roles: rows = experts (A operand: the gate matrix, staged through LDS in chunks of 64 columns
// shared by the four waves), columns = tokens (B operand: the lane's own 16-byte pieces of X, NXP chunks
// requested ahead).  Lane l = (q = l / 16, i = l % 16) feeds expert 16*tile + i and token i with column
// 32B + 8q + j in the j-th instruction of block B; the two blocks of a chunk go to the two partial sums.
// ROUTE: E <= 16 NT, one pass, routing fused; otherwise passes of 16 NT experts write logits only.
template <typename XT, int NT, int NXP, bool ROUTE, bool VEC, bool FULL, bool EVEN>
__global__ __launch_bounds__(GATE_THREADS) void gate_mfma_kernel(
    const XT* __restrict__ X, const float* __restrict__ Wg, const float* __restrict__ bg,
    float* __restrict__ logits, int32_t* __restrict__ idx, float* __restrict__ wout,
    int T, int d, int E, int k, int renorm, int e_pitch)
{
    constexpr int CHF = 1024 * NT;             // floats of one staged chunk: 64 columns x 16 NT experts
    __shared__ float w_lds[2 * CHF];           // [buffer][block s][q][tile][j / 4][i][j % 4]
    extern __shared__ float logit_lds[];       // ROUTE: [GATE_TOK][e_pitch]

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int q = lane >> 4, i16 = lane & 15;
    const int tok0w = blockIdx.x * GATE_TOK + wave * 16;
    const int tok = tok0w + i16;
    const XT* xrow = X + (size_t)(tok < T ? tok : T - 1) * d;     // rows past the end recompute the last token; never stored
    const int npairs = (d + 63) / 64;

    for (int ec0 = 0; ec0 < E; ec0 += 16 * NT) {
        gate_f4 acc[2][NT];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int tl = 0; tl < NT; ++tl) acc[s][tl] = gate_f4{0.0f, 0.0f, 0.0f, 0.0f};

        XPiece<XT> xb[NXP][2];
        auto load_pair = [&](int p, XPiece<XT> (&dst)[2]) {
            load_piece<VEC, FULL>(dst[0], xrow, p * 64 + 8 * q, d);
            load_piece<VEC, FULL>(dst[1], xrow, p * 64 + 32 + 8 * q, d);
        };
        // gate-matrix chunk p: item n of a thread = 4 consecutive experts of one column
        auto load_w = [&](int p, float4 (&wr)[NT]) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int it = n * GATE_THREADS + threadIdx.x;
                const int c = p * 64 + it / (4 * NT), e = ec0 + 4 * (it % (4 * NT));
                const bool in_c = c < d;
                const float* src = Wg + (size_t)(in_c ? c : 0) * E;
                float4 v;
                if (FULL) {
                    v = *reinterpret_cast<const float4*>(src + e);
                } else if (VEC) {                       // E % 4 == 0: the four experts are inside the row or past it
                    v = *reinterpret_cast<const float4*>(src + (e < E ? e : 0));
                    if (!(in_c && e < E)) v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                } else {
                    const float x0 = src[e + 0 < E ? e + 0 : 0], x1 = src[e + 1 < E ? e + 1 : 0];
                    const float x2 = src[e + 2 < E ? e + 2 : 0], x3 = src[e + 3 < E ? e + 3 : 0];
                    v.x = (in_c && e + 0 < E) ? x0 : 0.0f;
                    v.y = (in_c && e + 1 < E) ? x1 : 0.0f;
                    v.z = (in_c && e + 2 < E) ? x2 : 0.0f;
                    v.w = (in_c && e + 3 < E) ? x3 : 0.0f;
                }
                wr[n] = v;
            }
        };
        auto store_w = [&](int buf, const float4 (&wr)[NT]) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int it = n * GATE_THREADS + threadIdx.x;
                const int cc = it / (4 * NT), e4 = it % (4 * NT);
                const int s = cc >> 5, qq = (cc >> 3) & 3, jh = (cc >> 2) & 1, j4 = cc & 3;
                const int tl = e4 >> 2, i0 = (e4 & 3) * 4;
                float* dst = w_lds + buf * CHF + (((((s * 4 + qq) * NT + tl) * 2 + jh) * 16 + i0) * 4 + j4);
                dst[0] = wr[n].x;
                dst[4] = wr[n].y;
                dst[8] = wr[n].z;
                dst[12] = wr[n].w;
            }
        };
        // Ring slot u holds the tokens' columns of chunk p and the gate-matrix chunk p + 1, requested together
        // NXP chunks ahead: the memory counter retires in order, so whatever is needed soon must not have been
        // requested after something that is needed late.
        float4 wreg[NXP][NT];
        load_w(0, wreg[0]);
        store_w(0, wreg[0]);
#pragma unroll
        for (int u = 0; u < NXP; ++u) {
            load_pair(u, xb[u]);                                  // past the row: zeros, no access
            load_w(u + 1, wreg[u]);
        }
        __syncthreads();

        for (int p0 = 0; p0 < npairs; p0 += NXP) {
#pragma unroll
            for (int u = 0; u < NXP; ++u) {
                const int p = p0 + u;
                if (EVEN || p < npairs) {       // EVEN: the chunk count is a multiple of NXP (no branch in the ring)
                    const float* wb = w_lds + (p & 1) * CHF;
                    gate_f4 wf[2][NT][2];
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int tl = 0; tl < NT; ++tl)
#pragma unroll
                            for (int jh = 0; jh < 2; ++jh)
                                wf[s][tl][jh] = *reinterpret_cast<const gate_f4*>(
                                    wb + (((((s * 4 + q) * NT + tl) * 2 + jh) * 16 + i16) * 4));
                    auto step = [&](auto J) {
                        constexpr int j = decltype(J)::value;
                        const float x0 = piece_get<j>(xb[u][0]), x1 = piece_get<j>(xb[u][1]);
#pragma unroll
                        for (int tl = 0; tl < NT; ++tl) {
                            acc[0][tl] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[0][tl][j / 4][j % 4], x0, acc[0][tl], 0, 0, 0);
                            acc[1][tl] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[1][tl][j / 4][j % 4], x1, acc[1][tl], 0, 0, 0);
                        }
                    };
                    step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{});
                    step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{});
                    step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
                    step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 7>{});
                    if (p + 1 < npairs) store_w((p + 1) & 1, wreg[u]);
                    load_pair(p + NXP, xb[u]);
                    load_w(p + NXP + 1, wreg[u]);
                    __syncthreads();
                }
            }
        }

        // lane l, register r of tile tl: expert ec0 + 16 tl + 4q + r, token i16
#pragma unroll
        for (int tl = 0; tl < NT; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = ec0 + 16 * tl + 4 * q + r;
                if (e < E) {
                    const float v = (acc[0][tl][r] + acc[1][tl][r]) + bg[e];
                    if (ROUTE) logit_lds[(wave * 16 + i16) * e_pitch + e] = v;
                    else if (tok < T) logits[(size_t)tok * E + e] = v;
                }
            }
    }
    if (ROUTE) {
        __syncthreads();
        for (int i = lane; i < 16 * E; i += 64) {                 // the wave's 16 rows of logits are contiguous
            const int tk = i / E, e = i - tk * E;
            if (tok0w + tk < T) logits[(size_t)tok0w * E + i] = logit_lds[(wave * 16 + tk) * e_pitch + e];
        }
        route_lanes<4, 4 * NT>(logit_lds + (wave * 16 + (lane >> 2)) * e_pitch, lane & 3, tok0w + (lane >> 2), tok0w + (lane >> 2) < T, E, k, renorm, idx, wout);
    }
}

// ---- E % 4 == 0, bf16 tokens (d % 64 == 0) or fp32 (d % 4 == 0): the same contraction with both operands delivered by buffer loads that write
// LDS directly, so that nothing asynchronous ever targets a register and the waits can be written by hand (the compiler's
// own counts allow a third of the requests that may be outstanding).
// A tile of 16 tokens belongs to two waves, one per partial sum: wave s visits the 32-column blocks s, s + 2, s + 4, ..
// in order, which is the order the interface fixes, and the two sums meet in LDS at the end.  That halves the serial chain
// of a tile (512 matrix instructions of 32 cycles at d = 4096, E = 16) and gives a CU twice the waves.  A step is two of a
// wave's blocks (128 columns of the rows).
// A ring of RING steps of a tile's tokens (4 KB each, 8 in fp32, shared by its two waves: each requests 8 of the 16 rows, so that
// a request is whole 128-byte lines; 64-byte halves, a wave its own columns, asked L2 for every line twice); per partial
// sum a ring of RING steps of the gate matrix (64 columns x 16 NT experts), fetched in equal shares by the waves that
// use it.  A gate-matrix piece (4 consecutive experts of one column) lands where the instruction that uses it finds the 64
// values of its lanes side by side: piece (block of the step, j, tile, q, i / 4) at 16 * ((((8 b + j) NT + tile) 4 + q) 4 +
// i / 4), so the A operand of instruction (b, j, tile) is one `ds_read_b32` at lane * 4 plus a constant.  Experts past the
// last one multiply whatever lies there (the next column's, or zeros past the matrix) into rows that are not stored.
typedef __attribute__((ext_vector_type(4))) int gate_rsrc_t;
#define GATE_LDS_PTR(T) __attribute__((address_space(3))) T*

__device__ __forceinline__ gate_rsrc_t gate_make_rsrc(const void* base, unsigned long long bytes)
{
    if (bytes > 0xffffffffull) bytes = 0xffffffffull;
    const unsigned long long b = (unsigned long long)base;
    gate_rsrc_t r;
    r[0] = (int)(unsigned)(b & 0xffffffffull);
    r[1] = (int)(unsigned)((b >> 32) & 0xffffull);
    r[2] = (int)(unsigned)bytes;                           // reads at or past this limit return zero
    r[3] = 0x00020000;
    return r;
}
__device__ __forceinline__ void gate_dma16(gate_rsrc_t r, uint32_t lds_base, uint32_t voff, uint32_t soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds_base), "v"(voff), "s"(r), "s"(soff) : "memory");
}

template <typename XT, int NT, int TILES, int RING> constexpr int gate_split_lds() { return RING * (2048 * (int)sizeof(XT) * TILES + 2 * 4096 * NT); }

// TILES: token tiles of a block (2 TILES waves).  blockIdx.y: pass of 16 NT experts.  ROUTE: one pass, routing fused.
// What bounds it: few tokens, the chain of dependent matrix instructions of a partial sum, whose order is fixed (0.45 us per
// step; rings of 3, 5 and 10 steps take the same); many, the rows from HBM.  So the chain is kept going: the LDS reads of a
// block go out between the products of the block before it, the requests between those of the odd block.  The call, us,
// back to back and with the caches swept before it, separate reads, products and requests and half lines -> now: T = 64,
// d = 4096, E = 16 20.4, 23 -> 18.6, 21.4; T = 8192, d = 1024 10.8, 15.3 -> 10.3, 14.1; T = 8001, d = 2048, E = 128 55, 62 ->
// 52, 55; T = 16384, E = 64 48, 58 -> 45, 50; T = 32768, d = 4096, E = 16 64, 113 -> 60, 112.
// fp32 tokens, from the general kernel, whose loads wait for each other: T = 512, d = 64, E = 8 8.1 -> 4.4; T = 3291, d = 364, E = 8
// 11.9 -> 5.5; T = 67, d = 640, E = 16 13.4 -> 6.6; with the routing T = 1500, d = 512, E = 64 23 -> 9.5.
// ET: the block's waves share one token tile but not its experts: ET units of two waves, 16 experts each, with rings of their own
// (few tokens: the chain of a wave is as short as with a block per 16 experts, and the routing needs no launch of its own).
template <typename XT, int NT, int TILES, int RING, bool ROUTE, int ET>
__global__ __launch_bounds__(TILES * ET * 128) void gate_split_kernel(
    const XT* __restrict__ X, const float* __restrict__ Wg, const float* __restrict__ bg,
    float* __restrict__ logits, int32_t* __restrict__ idx, float* __restrict__ wout,
    int T, int d, int E, int k, int renorm)
{
    constexpr bool F32 = sizeof(XT) == 4;
    constexpr int XSTEP = 2048 * (int)sizeof(XT), WSTEP = 4096 * NT, XRING = TILES * RING * XSTEP;
    constexpr int XOPS = XSTEP / 2048, WOPS = 4 * NT / TILES, OPS = XOPS + WOPS;   // requests of one wave per step
    static_assert(4 * NT % TILES == 0 && OPS <= 8, "equal shares of the gate matrix, a request per column of a block");
    static_assert(RING >= 2, "a step is requested while the one before it is multiplied");
    constexpr int PITCH = 16 * NT * ET + 1;                // logits of a token in LDS
    static_assert(TILES * 16 * PITCH * 4 + TILES * ET * NT * 1024 <= ET * gate_split_lds<XT, NT, TILES, RING>(), "logits and sums fit the rings");
    static_assert(ET == 1 || (TILES == 1 && NT == 1 && ROUTE), "units of experts share one tile of tokens and all experts");
    extern __shared__ __attribute__((aligned(1024))) unsigned char all_lds[];   // token rings | gate-matrix rings, per unit; then sums | logits
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = wave & 1, tile = ET == 1 ? wave >> 1 : 0, unit = ET == 1 ? 0 : wave >> 1;      // partial sum, token tile, unit
    unsigned char* gsm = all_lds + unit * gate_split_lds<XT, NT, TILES, RING>();
    const uint32_t lds0 = (uint32_t)(uintptr_t)(GATE_LDS_PTR(unsigned char))gsm;
    const int q = lane >> 4, i16 = lane & 15;
    const int blk_tok0 = blockIdx.x * (16 * TILES), tok0w = blk_tok0 + tile * 16, tok = tok0w + i16;
    const int ec0 = (ET == 1 ? (int)blockIdx.y : unit) * (16 * NT);
    const int nb = (d + 63) / 64, steps = (nb + 1) / 2;    // 32-column blocks of each partial sum

    // tokens: rows of this block onwards; a token past the end reads the last one (never stored); a block past the
    // end of a row reads into the next rows or, after the last row, zeros: never multiplied.  The two waves of a tile
    // share its ring: a wave requests 8 of the 16 rows, whole 128-byte lines (64 columns, 32 of either sum); in LDS a
    // row's eight 16-byte pieces are XOR-swizzled by the row, so that the 16 rows of a piece cover all banks.
    // fp32: a line is the 32 columns of one sum; rows end inside a block, and pieces past the end are asked for nowhere (zeros).
    constexpr uint32_t NOWHERE = 0x80000000u;              // past the rows of a block, also with a step's offset added
    const gate_rsrc_t rX = gate_make_rsrc(X + (size_t)blk_tok0 * d, (unsigned long long)(F32 ? min(T - blk_tok0, 16 * TILES) : T - blk_tok0) * d * sizeof(XT));
    const int xrow = 8 * s + (lane >> 3);                  // row of the tile this lane requests a piece of
    const int rowrel = (tok0w + xrow < T ? tok0w + xrow : T - 1) - blk_tok0;
    const int xpiece = (lane & 7) ^ ((xrow >> 1) & 7);
    const uint32_t xv = (uint32_t)(rowrel * d * (int)sizeof(XT) + (xpiece << 4));
    const uint32_t xl = lds0 + (uint32_t)(tile * RING * XSTEP + s * 1024);
    // gate matrix: this wave's share of a step
    const gate_rsrc_t rW = gate_make_rsrc(Wg + ec0, ((unsigned long long)d * E - ec0) * 4);     // past the last column: zeros
    uint32_t wv[WOPS];
#pragma unroll
    for (int n = 0; n < WOPS; ++n) {
        const int L = (tile * WOPS + n) * 64 + lane;       // 16-byte slot of the step
        const int e4 = L & 3, qq = (L >> 2) & 3, tl = (L >> 4) % NT, bj = L / (16 * NT);
        wv[n] = (uint32_t)(((64 * (bj >> 3) + 32 * s + 8 * qq + (bj & 7)) * E + 16 * tl + 4 * e4) * 4);
    }
    const uint32_t wl = lds0 + (uint32_t)(XRING + s * RING * WSTEP + tile * WOPS * 1024);
    auto request = [&](int n, int P, int slot) {           // request n of this wave for step P
        if (n < XOPS) {
            const bool there = !F32 || P * 128 + n * 32 + xpiece * 4 < d;
            gate_dma16(rX, xl + (uint32_t)(slot * XSTEP + n * 2048), there ? xv + 128u * n : NOWHERE, (uint32_t)P * (128u * sizeof(XT)));
        } else gate_dma16(rW, wl + (uint32_t)(slot * WSTEP + (n - XOPS) * 1024), wv[n - XOPS], (uint32_t)P * (uint32_t)(128 * E * 4));
    };
    gate_f4 acc[NT];
#pragma unroll
    for (int tl = 0; tl < NT; ++tl) acc[tl] = gate_f4{0.0f, 0.0f, 0.0f, 0.0f};
    // operands of a block: 8 columns of a token per lane (as loaded), 8 x NT elements of the gate matrix
    struct Block { gate_u4 x[F32 ? 2 : 1]; float w[8][NT]; };
    const uint32_t xr = (uint32_t)(tile * RING * XSTEP + i16 * 128 + (F32 ? s * 2048 : 0) + (((F32 ? 2 * q : 4 * s + q) ^ ((i16 >> 1) & 7)) << 4));
    const uint32_t wr = (uint32_t)(XRING + s * RING * WSTEP + lane * 4);
    auto read_x = [&](Block& o, int slot, int b) {
        o.x[0] = *reinterpret_cast<const gate_u4*>(gsm + xr + slot * XSTEP + b * (XSTEP / 2));
        if constexpr (F32) o.x[1] = *reinterpret_cast<const gate_u4*>(gsm + (xr ^ 16u) + slot * XSTEP + b * (XSTEP / 2));
    };
    auto read_w = [&](Block& o, int slot, int b, int j) {
#pragma unroll
        for (int tl = 0; tl < NT; ++tl) o.w[j][tl] = *reinterpret_cast<const float*>(gsm + wr + slot * WSTEP + ((b * 8 + j) * NT + tl) * 256);
    };
    auto multiply = [&](const Block& o, int j) {
        float a;
        if constexpr (F32) a = __uint_as_float(o.x[j / 4][j % 4]);
        else a = __uint_as_float((j & 1) ? (o.x[0][j / 2] & 0xffff0000u) : (o.x[0][j / 2] << 16));
#pragma unroll
        for (int tl = 0; tl < NT; ++tl) acc[tl] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.w[j][tl], a, acc[tl], 0, 0, 0);
    };
    Block b0, b1;                                          // the even and the odd block of a step
#pragma unroll
    for (int P = 0; P < RING; ++P)
#pragma unroll
        for (int n = 0; n < OPS; ++n) request(n, P, P);
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((RING - 1) * OPS) : "memory");
    asm volatile("s_barrier" ::: "memory");
    read_x(b0, 0, 0);
#pragma unroll
    for (int j = 0; j < 8; ++j) read_w(b0, 0, 0, j);
    int slot = 0;
    for (int P = 0; P < steps; ++P) {
        const int next = (slot + 1 == RING) ? 0 : slot + 1;
        // the odd block's operands come in under the even block's products
        read_x(b1, slot, 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            read_w(b1, slot, 1, j);
            multiply(b0, j);
            __builtin_amdgcn_sched_barrier(0);
        }
        // this wave has read all of step P and its requests for step P + 1 have landed (RING - 2 younger steps may be
        // pending); after the barrier that is true of every wave: step P's slot is free, step P + 1 can be read
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((RING - 2) * OPS) : "memory");
        asm volatile("s_barrier" ::: "memory");
        // under the odd block's products: the requests for step P + RING, the operands of the next even block
        const bool odd = 2 * P + 1 < nb;                   // an odd number of blocks ends with half a step
        read_x(b0, next, 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j < OPS) request(j, P + RING, slot);
            read_w(b0, next, 0, j);
            if (odd) multiply(b1, j);
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = next;
    }
    // requests past the end are still on their way into the rings: nothing may reuse LDS before they land
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float* sums = reinterpret_cast<float*>(all_lds) + (tile + unit) * NT * 256 + lane;
    float* logit_lds = reinterpret_cast<float*>(all_lds) + TILES * ET * NT * 256 + tile * 16 * PITCH;
    if (s == 1)
#pragma unroll
        for (int tl = 0; tl < NT; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) sums[(tl * 4 + r) * 64] = acc[tl][r];
    __syncthreads();
    // lane l, register r of tile tl: expert ec0 + 16 tl + 4q + r, token i16
    if (s == 0)
#pragma unroll
        for (int tl = 0; tl < NT; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = ec0 + 16 * tl + 4 * q + r;
                if (e < E) {
                    const float v = (acc[tl][r] + sums[(tl * 4 + r) * 64]) + bg[e];
                    if (ROUTE) logit_lds[i16 * PITCH + e] = v;
                    else if (tok < T) logits[(size_t)tok * E + e] = v;
                }
            }
    if (ROUTE) {
        __syncthreads();
        if (unit > 0) return;
        if (s == 1) {
            for (int i = lane; i < 16 * E; i += 64) {             // the tile's 16 rows of logits are contiguous
                const int tk = i / E, e = i - tk * E;
                if (tok0w + tk < T) logits[(size_t)tok0w * E + i] = logit_lds[tk * PITCH + e];
            }
        } else {
            route_lanes<4, 4 * NT * ET>(logit_lds + (lane >> 2) * PITCH, lane & 3, tok0w + (lane >> 2), tok0w + (lane >> 2) < T, E, k, renorm, idx, wout);
        }
    }
}

// Routing from logits in global memory (E > 64: the logits were written in passes), 16 lanes per token: a wave reads four
// tokens' rows in whole 64-byte pieces, once.  One lane per token read them k + 1 times an element at a time: 149 us at
// T = 8001, E = 128, k = 4; the whole call 250 -> 95 us, at T = 20000, k = 8 513 -> 107.
constexpr int ROUTE_THREADS = 256, ROUTE_TOK = ROUTE_THREADS / 16;
template <int EPL>
__global__ __launch_bounds__(ROUTE_THREADS) void gate_route_kernel(const float* __restrict__ logits, int32_t* __restrict__ idx,
                                                                   float* __restrict__ wout, int T, int E, int k, int renorm)
{
    const int t = blockIdx.x * ROUTE_TOK + threadIdx.x / 16;
    const bool on = t < T;
    route_lanes<16, EPL>(logits + (size_t)(on ? t : T - 1) * E, threadIdx.x & 15, t, on, E, k, renorm, idx, wout);
}

hipError_t run_gate_route(const moe_shape_t& s, const float* logits, int32_t* idx, float* w, hipStream_t st)
{
    const dim3 grid((s.T + ROUTE_TOK - 1) / ROUTE_TOK), block(ROUTE_THREADS);
    if (s.E <= 128) hipLaunchKernelGGL(gate_route_kernel<8>, grid, block, 0, st, logits, idx, w, s.T, s.E, s.k, s.renorm);
    else if (s.E <= 256) hipLaunchKernelGGL(gate_route_kernel<16>, grid, block, 0, st, logits, idx, w, s.T, s.E, s.k, s.renorm);
    else hipLaunchKernelGGL(gate_route_kernel<64>, grid, block, 0, st, logits, idx, w, s.T, s.E, s.k, s.renorm);
    return hipGetLastError();
}

// Gradient of the gate weights: 16 lanes per token, each with every 16th logit, so that a wave reads and writes whole
// 64-byte pieces of four tokens' rows (one lane per token touched a line per element: 45 us at T = 16384, E = 64, k = 1,
// where the rows are 8 MB; 57 at T = 8001, E = 128; now 10 and under, launch included).
constexpr int GBW_LANES = 16, GBW_THREADS = 256;
__device__ __forceinline__ float gbw_sum(float v)
{
#pragma unroll
    for (int off = GBW_LANES / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__global__ __launch_bounds__(GBW_THREADS) void gate_bwd_kernel(
    const float* __restrict__ dw, const float* __restrict__ logits, const int32_t* __restrict__ idx,
    float* __restrict__ dlogits, int T, int E, int k, int renorm)
{
    constexpr int MAXK = 8;
    const int sub = threadIdx.x % GBW_LANES;
    const int t = blockIdx.x * (GBW_THREADS / GBW_LANES) + threadIdx.x / GBW_LANES;
    if (t >= T) return;                         // all lanes of a token leave together
    const float* lg = logits + (size_t)t * E;
    float* dl = dlogits + (size_t)t * E;
    int s[MAXK];
    float g[MAXK], ps[MAXK];
#pragma unroll
    for (int j = 0; j < MAXK; ++j) {
        s[j] = j < k ? idx[(size_t)t * k + j] : -1;
        g[j] = j < k ? dw[(size_t)t * k + j] : 0.0f;
        ps[j] = j < k ? lg[s[j]] : 0.0f;        // the selected logits for now
    }
    float m = -INFINITY;
    for (int e = sub; e < E; e += GBW_LANES) m = fmaxf(m, lg[e]);
#pragma unroll
    for (int off = GBW_LANES / 2; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    float sum = 0.0f;
    for (int e = sub; e < E; e += GBW_LANES) sum += expf(lg[e] - m);
    const float inv = 1.0f / gbw_sum(sum);
    float psel = 0.0f, gp = 0.0f;               // sum_j p[s_j], sum_j dw_j p[s_j]
#pragma unroll
    for (int j = 0; j < MAXK; ++j)
        if (j < k) {
            ps[j] = expf(ps[j] - m) * inv;
            psel += ps[j];
            gp += g[j] * ps[j];
        }
    if (renorm) {
        float dot = 0.0f;
#pragma unroll
        for (int j = 0; j < MAXK; ++j) if (j < k) dot += (ps[j] / psel) * g[j];
#pragma unroll
        for (int j = 0; j < MAXK; ++j) if (j < k) g[j] = (ps[j] / psel) * (g[j] - dot);
        for (int e = sub; e < E; e += GBW_LANES) {
            float v = 0.0f;
#pragma unroll
            for (int j = 0; j < MAXK; ++j) if (s[j] == e) v = g[j];
            dl[e] = v;
        }
    } else {
        for (int e = sub; e < E; e += GBW_LANES) {
            float v = -gp * (expf(lg[e] - m) * inv);
#pragma unroll
            for (int j = 0; j < MAXK; ++j) if (s[j] == e) v += g[j] * ps[j];
            dl[e] = v;
        }
    }
}

template <typename XT, int NT, int NXP, bool VEC, bool FULL, bool EVEN>
hipError_t run_gate(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                    float* logits, int32_t* idx, float* w, hipStream_t st)
{
    const int grid = (s.T + GATE_TOK - 1) / GATE_TOK;
    if (s.E <= 16 * NT) {
        const int e_pitch = s.E | 1;
        const size_t dyn = (size_t)GATE_TOK * e_pitch * sizeof(float);
        hipLaunchKernelGGL((gate_mfma_kernel<XT, NT, NXP, true, VEC, FULL, EVEN>), dim3(grid), dim3(GATE_THREADS), dyn, st,
                           (const XT*)X, Wg, bg, logits, idx, w, s.T, s.d, s.E, s.k, s.renorm, e_pitch);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((gate_mfma_kernel<XT, NT, NXP, false, VEC, FULL, EVEN>), dim3(grid), dim3(GATE_THREADS), 0, st,
                       (const XT*)X, Wg, bg, logits, idx, w, s.T, s.d, s.E, s.k, s.renorm, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return run_gate_route(s, logits, idx, w, st);
}

template <typename XT, int NT, int TILES, int RING, bool ROUTE, int ET = 1>
hipError_t run_gate_split(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                          float* logits, int32_t* idx, float* w, hipStream_t st)
{
    constexpr int lds = ET * gate_split_lds<XT, NT, TILES, RING>();
    auto kern = gate_split_kernel<XT, NT, TILES, RING, ROUTE, ET>;
    static PerDeviceOnce once;                             // per instantiation
    const int dev = current_device();
    if (!once.is_done(dev)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        once.mark(dev);
    }
    const dim3 grid((s.T + 16 * TILES - 1) / (16 * TILES), ET > 1 ? 1 : (s.E + 16 * NT - 1) / (16 * NT));
    hipLaunchKernelGGL(kern, grid, dim3(TILES * ET * 128), lds, st, (const XT*)X, Wg, bg, logits, idx, w, s.T, s.d, s.E, s.k, s.renorm);
    const hipError_t e = hipGetLastError();
    return (e != hipSuccess || ROUTE) ? e : run_gate_route(s, logits, idx, w, st);
}

template <typename XT, int NT, int NXP>
hipError_t run_gate_n(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                      float* logits, int32_t* idx, float* w, hipStream_t st)
{
    // 16-byte requests need whole pieces inside the rows: E % 4 == 0 for the gate matrix, d % 4 == 0 for fp32
    // tokens (bf16 shapes have d % 64 == 0); other shapes take the same kernel with 4-byte requests.
    if (s.d % (64 * NXP) == 0 && s.E % (16 * NT) == 0) return run_gate<XT, NT, NXP, true, true, true>(s, X, Wg, bg, logits, idx, w, st);
    if (s.d % 64 == 0 && s.E % (16 * NT) == 0) return run_gate<XT, NT, NXP, true, true, false>(s, X, Wg, bg, logits, idx, w, st);
    if (s.E % 4 == 0 && s.d % 4 == 0) return run_gate<XT, NT, NXP, true, false, false>(s, X, Wg, bg, logits, idx, w, st);
    return run_gate<XT, NT, NXP, false, false, false>(s, X, Wg, bg, logits, idx, w, st);
}

template <typename XT>
hipError_t run_gate_t(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                      float* logits, int32_t* idx, float* w, hipStream_t st)
{
    if (s.E <= 16) return run_gate_n<XT, 1, 8>(s, X, Wg, bg, logits, idx, w, st);
    if (s.E <= 32) return run_gate_n<XT, 2, 4>(s, X, Wg, bg, logits, idx, w, st);
    return run_gate_n<XT, 4, 4>(s, X, Wg, bg, logits, idx, w, st);
}

}  // namespace

// A launch has fewer than 2^32 threads along x.  The gate spends up to 16 threads on a token (routing of more than 64
// experts), T may be just short of 2^30: tokens are taken 2^26 at a time.
constexpr int GATE_LAUNCH_TOK = 1 << 26;
static_assert(GATE_LAUNCH_TOK % GATE_TOK == 0 && GATE_LAUNCH_TOK <= (1ll << 32) / 32, "whole blocks, within a launch");

// Few tokens and 17 to 64 experts: whether a block takes all experts of its tokens and routes them (a launch of 4 us fewer), or
// every 16 experts are a block of their own.  In one block the operands of two or more units come in through one CU, which
// delivers those of two units in the time a step takes, of four in twice that: kernels, us, blocks of 16 experts + routing | one
// block, bf16: T = 1999, d = 768, E = 32 6.2 + 4.5 | 7.9; T = 1075, d = 2304, E = 24 12.5 + 4.1 | 13.9; T = 2040, d = 1024, E = 64
// 9.5 + 4.2 | 12.7; T = 600, d = 4096, E = 64 18.7 + 4.1 | 29.2; fp32: T = 1931, d = 700, E = 32 5.8 + 4.8 | 8.1.
// Where the blocks of 16 experts have a CU each (tiles of 16 tokens x 16 experts: up to 256), three units win up to 512 columns, four
// up to 256.  The call, us: bf16 T = 241, d = 512, E = 48 8.1 | 7.8; T = 136, d = 960, E = 36 9.4 | 9.8; T = 187, d = 64, E = 64 6.9 |
// 6.6; T = 13, d = 320, E = 64 7.4 | 7.7; T = 6, d = 960, E = 64 9.1 | 10.4; fp32 T = 94, d = 1400, E = 48 13.1 | 14.0; T = 19, d = 236, E
// = 64 6.6 | 6.5; T = 1, d = 332, E = 52 6.9 | 7.2.  Where they share CUs: bf16 T = 1272, d = 320, E = 52 8.2 | 7.3; fp32 T = 1799, d = 192,
// E = 52 10.3 | 8.7.
static bool one_block(const moe_shape_t& s, long tiles)
{
    const long row = (long)s.d * (s.dtype == MOE_BF16 ? 2 : 4);
    if (s.E <= 32) return row <= 8192;
    return s.E <= 64 && row <= 2048 && (tiles > 256 || s.d <= (s.E <= 48 ? 512 : 256));
}

static hipError_t launch_gate_part(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                                   float* logits, int32_t* idx, float* w, hipStream_t st)
{
    const long tiles = (long)((s.T + 15) / 16) * ((s.E + 15) / 16);
    if (s.dtype == MOE_F32) {
        // the same choice for fp32, whose tokens take twice the LDS
        if (s.E % 4 == 0 && (long long)s.d * 4 * (GATE_TOK + 1) < (1ll << 31) && (long long)s.d * s.E * 4 < (1ll << 31)) {
            if (tiles <= 512) {
                if (s.E <= 16) return run_gate_split<float, 1, 1, 3, true>(s, X, Wg, bg, logits, idx, w, st);
                if (one_block(s, tiles) && s.E <= 32) return run_gate_split<float, 1, 1, 3, true, 2>(s, X, Wg, bg, logits, idx, w, st);
                if (one_block(s, tiles) && s.E <= 48) return run_gate_split<float, 1, 1, 3, true, 3>(s, X, Wg, bg, logits, idx, w, st);
                if (one_block(s, tiles)) return run_gate_split<float, 1, 1, 2, true, 4>(s, X, Wg, bg, logits, idx, w, st);
                return run_gate_split<float, 1, 1, 3, false>(s, X, Wg, bg, logits, idx, w, st);
            }
            if (s.E <= 16) return run_gate_split<float, 1, 4, 3, true>(s, X, Wg, bg, logits, idx, w, st);
            // 17 to 32 experts: 144 KB of rings, one block per CU.  A second round of such blocks does little but fill them where rows
            // are short; the general kernel has several per CU (us, general | split: T = 50676, d = 8, E = 20 17.7 | 27.9; T = 21561, d
            // = 56, E = 24 10.3 | 15.0; T = 24527, d = 152, E = 32 12.9 | 15.1; T = 16628, d = 372, E = 24 17.1 | 17.8; T = 42692, d = 348, E
            // = 20 36.7 | 33.3; one round, T = 15276, d = 36, E = 20 8.8 | 8.4)
            if (s.E <= 32 && s.T > 64 * 256 && s.d <= 256) return run_gate_t<float>(s, X, Wg, bg, logits, idx, w, st);
            if (s.E <= 32) return run_gate_split<float, 2, 4, 3, true>(s, X, Wg, bg, logits, idx, w, st);
            if (s.E <= 64) return run_gate_split<float, 4, 4, 2, true>(s, X, Wg, bg, logits, idx, w, st);
            return run_gate_split<float, 4, 4, 2, false>(s, X, Wg, bg, logits, idx, w, st);
        }
        return run_gate_t<float>(s, X, Wg, bg, logits, idx, w, st);
    }
    // rows of 64 tokens must stay inside the 32-bit offsets of a buffer load; a load that writes LDS moves whole aligned
    // words, so tokens that begin at an odd bf16 take the general kernel (ordinary loads need no alignment)
    if (s.E % 4 == 0 && (reinterpret_cast<uintptr_t>(X) & 3) == 0 && (long long)s.d * 2 * (GATE_TOK + 1) < (1ll << 31) && (long long)s.d * s.E * 4 < (1ll << 31)) {
        // Few tokens: a block per 16 tokens and 16 experts (more experts: as one_block says), so that the
        // gate matrix comes in through as many CUs as there are.  Up to 512 such blocks; beyond, 64 tokens share a block's
        // gate matrix.  The call, us, before -> now: T = 64, d = 4096, E = 16 34 -> 20; T = 1, d = 2048 19 -> 13; T = 3000,
        // d = 1024, E = 48 45 -> 21; T = 2000, E = 100, k = 8 85 -> 34; T = 8001, d = 2048, E = 128 95 -> 56; T = 4000, E = 24
        // 30 -> 15; T = 16384, E = 32 32 -> 29, E = 64 52 -> 49; T = 32768, d = 4096, E = 16 70 -> 66 (the kernel has gained a
        // few percent more since, see there).
        // Rings: three steps, or two where that puts a second block on a CU that has one to run: T = 30000, d = 1984, E = 48
        // 68 -> 61 us; T = 40000, d = 2048, E = 32 76 -> 67 (but T = 16384, one block per CU anyway, caches swept, 37 -> 39).
        if (tiles <= 512) {
            if (s.E <= 16) return run_gate_split<bf16_t, 1, 1, 3, true>(s, X, Wg, bg, logits, idx, w, st);
            if (one_block(s, tiles) && s.E <= 32) return run_gate_split<bf16_t, 1, 1, 3, true, 2>(s, X, Wg, bg, logits, idx, w, st);
            if (one_block(s, tiles) && s.E <= 48) return run_gate_split<bf16_t, 1, 1, 3, true, 3>(s, X, Wg, bg, logits, idx, w, st);
            if (one_block(s, tiles)) return run_gate_split<bf16_t, 1, 1, 3, true, 4>(s, X, Wg, bg, logits, idx, w, st);
            return run_gate_split<bf16_t, 1, 1, 3, false>(s, X, Wg, bg, logits, idx, w, st);
        }
        if (s.E <= 16) return run_gate_split<bf16_t, 1, 4, 3, true>(s, X, Wg, bg, logits, idx, w, st);
        if (s.E <= 32 && s.T <= 64 * 256) return run_gate_split<bf16_t, 2, 4, 3, true>(s, X, Wg, bg, logits, idx, w, st);
        if (s.E <= 32) return run_gate_split<bf16_t, 2, 4, 2, true>(s, X, Wg, bg, logits, idx, w, st);
        if (s.E <= 48) return run_gate_split<bf16_t, 3, 4, 2, true>(s, X, Wg, bg, logits, idx, w, st);
        if (s.E <= 64) return run_gate_split<bf16_t, 4, 4, 3, true>(s, X, Wg, bg, logits, idx, w, st);
        return run_gate_split<bf16_t, 4, 4, 3, false>(s, X, Wg, bg, logits, idx, w, st);
    }
    return run_gate_t<bf16_t>(s, X, Wg, bg, logits, idx, w, st);
}

hipError_t launch_gate_topk(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                            float* logits, int32_t* idx, float* w, hipStream_t st)
{
    const size_t row = (size_t)s.d * (s.dtype == MOE_BF16 ? 2 : 4);
    moe_shape_t part = s;
    hipError_t e = hipSuccess;
    for (int t0 = 0; t0 < s.T && e == hipSuccess; t0 += part.T) {
        part.T = s.T - t0 < GATE_LAUNCH_TOK ? s.T - t0 : GATE_LAUNCH_TOK;
        e = launch_gate_part(part, (const char*)X + t0 * row, Wg, bg, logits + (size_t)t0 * s.E, idx + (size_t)t0 * s.k, w + (size_t)t0 * s.k, st);
    }
    return e;
}

hipError_t launch_gate_bwd(const moe_shape_t& s, const float* dw, const float* logits, const int32_t* idx,
                           float* dlogits, hipStream_t st)
{
    const int tokens = GBW_THREADS / GBW_LANES;
    hipError_t e = hipSuccess;
    for (int t0 = 0; t0 < s.T && e == hipSuccess; t0 += GATE_LAUNCH_TOK) {
        const int n = s.T - t0 < GATE_LAUNCH_TOK ? s.T - t0 : GATE_LAUNCH_TOK;
        const size_t a = (size_t)t0 * s.k, l = (size_t)t0 * s.E;
        hipLaunchKernelGGL(gate_bwd_kernel, dim3((n + tokens - 1) / tokens), dim3(GBW_THREADS), 0, st,
                           dw + a, logits + l, idx + a, dlogits + l, n, s.E, s.k, s.renorm);
        e = hipGetLastError();
    }
    return e;
}
