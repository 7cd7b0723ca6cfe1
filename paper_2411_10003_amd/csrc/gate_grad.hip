// Backward of the gate's linear map logit[t,e] = b[e] + sum_c X[t,c] Wg[c,e] (the gate network of
// Section 2.1 of the paper) and the complete gradient of the layer input:
//   dWg[c,e] = sum_t X[t,c] dlogits[t,e]      dbg[e] = sum_t dlogits[t,e]
//   dX[t,c]  = sum_j dXp[pos[t*k+j],c]  +  sum_e dlogits[t,e] Wg[c,e]
// The first sum of dX is the backward of the send (the fourth all-to-all of the performance model,
// Section 4.2); fusing the gate path into it saves a pass over dX.  Both kernels stream X or dXp once, with E fp32
// multiply-adds per element beside it on the fp32 MFMA; fp32 throughout.  Where the experts no longer fit (32 of them in
// the accumulators of the parameter gradients, 128 in the LDS of the input gradient) they are taken by further blocks or
// in chunks.
#include "internal.h"

#include <algorithm>
#include <type_traits>

namespace {

__device__ __forceinline__ void unpack_bf16x8(const uint4& v, float* f)
{
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
}

// ---- dX = backward of the send + dlogits Wg^T ---------------------------------------------------
// dlogits Wg^T is a dense product with the experts as its short contraction, on the fp32 16x16x4 MFMA.  A wave owns a
// strip of 16 VN columns and takes 16 tokens at a time.  Tile j of the strip holds the columns strip0 + n * VN + j
// (n = 0..15), so that lane l ends up with VN consecutive columns (n = l % 16) of the tokens 4 (l / 16) + r, r = 0..3:
// exactly one 16-byte piece per token, which is what the gather of the dXp rows and the store of dX move.  The A
// operand is dlogits[token l % 16][expert], the B operand the strip of Wg: instruction (i, jj) contracts the experts
// 16 i + 4 q + jj, q = l / 16, so that a lane reads its logit gradients 16 bytes at a time.
// What bounds it: HBM for E <= 32 (dXp and dX), the matrix rate beyond.  The strip of Wg lies in LDS in the order in
// which the instructions read it (two 16-byte reads per eight instructions), staged once per block for up to 128
// experts, in chunks of 128 per 64 tokens beyond.  In registers (what E <= 32 did before) it took 64 and 128 of them per
// lane and left two waves per SIMD; on the vector ALUs with a readlane per expert (what E > 32 did) the LDS reads bound
// it.  All row pieces of a group are requested before its matrix instructions, unconditionally (rows and columns past
// the end read the last valid ones and are not stored): a load under a condition makes the compiler drain them early.  An
// assignment without a row (a negative position, what an expert id out of range leaves where the caller put it) reads row 0
// and adds zeros.
// Measured, us before -> after (bf16): T = 16384, d = 2048, k = 2, E = 32: 81 -> 52 (2.1 GFLOP beside 201 MB); k = 1, E = 64:
// 377 -> 61; T = 8001, k = 4, E = 128: 524 -> 94; T = 1000, d = 512, E = 16: 43 -> 10 (16 blocks before); T = 32768,
// d = 4096, E = 16: 172 -> 172 (807 MB, 4.7 TB/s).  Requesting the next group's rows before the matrix instructions of the current
// one pays with 33 to 64 experts (T = 16384, d = 2048, k = 1, E = 64 61 -> 58; T = 20000, d = 1024, k = 2, E = 48 58 -> 53), where
// those take long enough; with fewer it costs a wave per SIMD and bandwidth (E = 32 54 -> 60, E = 16 159 -> 204).
typedef __attribute__((ext_vector_type(4))) float ig_f32x4_t;

// waves per SIMD the compiler is held to: 4, 3 with two row pieces requested ahead, 2 where the row pieces (16 KMAX registers) or the LDS leave no room for that
template <typename ET, int NE, int KMAX, bool NT>
__global__ __launch_bounds__(256, KMAX <= 2 && NE < 8 ? (NE == 4 && KMAX == 2 ? 3 : 4) : 2) void input_grad_kernel(
    const ET* __restrict__ dXp, const int32_t* __restrict__ pos, const float* __restrict__ dlogits,
    const float* __restrict__ Wg, ET* __restrict__ dX, int T, int d, int E, int k, int groups_per_wave, int vec)
{
    constexpr int VN = 16 / sizeof(ET), SW = 16 * VN, VH = VN / 4, EC = 16 * NE;
    constexpr bool MANY = NE > 2, CHUNKS = NE == 8;                // more than 32 experts; perhaps more than fit LDS at once
    typedef typename std::conditional<sizeof(ET) == 2, uint4, float4>::type raw_t;
    extern __shared__ __attribute__((aligned(16))) float wl[];      // [4 NE steps][VH][64 lanes][4]
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = blockIdx.x * SW;
    const int c = c0 + ln * VN, cc = c < d ? c : 0;

    // the strip's weights for the experts ec0 .. ec0 + EC - 1 (zeros past E and d); whether any of them is not finite
    auto stage = [&](int ec0) -> bool {
        bool odd = false;
        for (int i = tid; i < SW * EC / 4; i += 256) {
            const int cl = i % SW, e4 = i / SW, e = ec0 + 4 * e4, col = c0 + cl;
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (col < d) {
                const float* src = Wg + (size_t)col * E + e;
                if (vec) { if (e < E) v = *reinterpret_cast<const float4*>(src); }
                else {
                    if (e + 0 < E) v.x = src[0];
                    if (e + 1 < E) v.y = src[1];
                    if (e + 2 < E) v.z = src[2];
                    if (e + 3 < E) v.w = src[3];
                }
            }
            float* dst = wl + ((4 * (e4 >> 2)) * VH + (cl % VN) / 4) * 256 + ((e4 & 3) * 16 + cl / VN) * 4 + cl % 4;
            dst[0] = v.x; dst[VH * 256] = v.y; dst[2 * VH * 256] = v.z; dst[3 * VH * 256] = v.w;
            odd |= !(fabsf(v.x) < INFINITY && fabsf(v.y) < INFINITY && fabsf(v.z) < INFINITY && fabsf(v.w) < INFINITY);
        }
        return odd;
    };
    bool skip_zeros = false;
    if (!CHUNKS || E <= EC) skip_zeros = __syncthreads_or(stage(0));

    // rows of a group of 16 tokens; PREFETCH: the next group's are requested before the current one's matrix instructions
    constexpr bool PREFETCH = KMAX <= 2 && NE == 4;
    raw_t raw[4][KMAX], ahead[PREFETCH ? 4 : 1][KMAX];
    auto first_token = [&](int gi) { return (blockIdx.y * groups_per_wave + gi) * 64 + wave * 16; };
    auto request_rows = [&](int gi, raw_t (&to)[4][KMAX]) {
        const int tg = first_token(gi);
        int lowest = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = min(tg + 4 * lq + r, T - 1);
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                const int row = pos[(size_t)t * k + (j < k ? j : 0)];
                lowest = min(lowest, row);
                to[r][j] = load_piece_of<NT>(reinterpret_cast<const raw_t*>(dXp + (size_t)max(row, 0) * d + cc));
            }
        }
        if (__any(lowest < 0))
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < KMAX; ++j)
                    if (j < k && pos[(size_t)min(tg + 4 * lq + r, T - 1) * k + j] < 0) to[r][j] = raw_t{};
    };
    if (PREFETCH) request_rows(0, raw);
    for (int gi = 0; gi < groups_per_wave; ++gi) {
        const int tg = first_token(gi);
        if (!PREFETCH) request_rows(gi, raw);
        ig_f32x4_t acc[VN];
#pragma unroll
        for (int j = 0; j < VN; ++j) acc[j] = ig_f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        const float* dl = dlogits + (size_t)min(tg + ln, T - 1) * E;
        for (int ec0 = 0; ec0 < (CHUNKS ? E : 1); ec0 += EC) {
            if (CHUNKS && E > EC) {
                __syncthreads();                                   // everyone is done with the chunk before
                skip_zeros = __syncthreads_or(stage(ec0));
            }
            float a[4 * NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int e = ec0 + 16 * i + 4 * lq;
                if (vec) {                                         // E is a multiple of 4
                    const float4 v = *reinterpret_cast<const float4*>(dl + (e < E ? e : 0));
                    a[4 * i] = e < E ? v.x : 0.0f; a[4 * i + 1] = e < E ? v.y : 0.0f;
                    a[4 * i + 2] = e < E ? v.z : 0.0f; a[4 * i + 3] = e < E ? v.w : 0.0f;
                } else {
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const float v = dl[e + jj < E ? e + jj : 0];
                        a[4 * i + jj] = e + jj < E ? v : 0.0f;
                    }
                }
            }
            if constexpr (PREFETCH) if (gi + 1 < groups_per_wave) request_rows(gi + 1, ahead);
            // the weights are read from LDS again for every group: hoisted out of the loop over the groups they would spill
            if (NE > 1) asm volatile("" ::: "memory");
            if (!MANY || !skip_zeros) {
#pragma unroll
                for (int m = 0; m < 4 * NE; ++m) {
                    float w[VN];
#pragma unroll
                    for (int v = 0; v < VH; ++v) {
                        const float4 f = *reinterpret_cast<const float4*>(wl + (m * VH + v) * 256 + lane * 4);
                        w[4 * v] = f.x; w[4 * v + 1] = f.y; w[4 * v + 2] = f.z; w[4 * v + 3] = f.w;
                    }
#pragma unroll
                    for (int j = 0; j < VN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], w[j], acc[j], 0, 0, 0);
                }
            } else {
                // A weight that is not finite and more than 32 experts: an expert without a gradient is left out instead
                // of contributing 0 * inf (the routing of a token may well exclude that expert).
#pragma unroll
                for (int m = 0; m < 4 * NE; ++m)
#pragma unroll 1
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float g = __shfl(a[m], q * 16 + 4 * lq + r, 64);
#pragma unroll
                            for (int j = 0; j < VN; ++j) {
                                const float w = wl[(m * VH + j / 4) * 256 + (q * 16 + ln) * 4 + j % 4];
                                if (g != 0.0f) acc[j][r] = fmaf(g, w, acc[j][r]);
                            }
                        }
            }
        }
        // add the k rows of every token (j ascending, as the plain send backward adds them) and store
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = tg + 4 * lq + r;
            float sum[VN];
#pragma unroll
            for (int i = 0; i < VN; ++i) sum[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                if (j >= k) break;
                float x[VN];
                if constexpr (sizeof(ET) == 2) {
                    unpack_bf16x8(raw[r][j], x);
                } else {
                    x[0] = raw[r][j].x; x[1] = raw[r][j].y; x[2] = raw[r][j].z; x[3] = raw[r][j].w;
                }
#pragma unroll
                for (int i = 0; i < VN; ++i) sum[i] += x[i];
            }
#pragma unroll
            for (int i = 0; i < VN; ++i) sum[i] += acc[i][r];
            if (t >= T || c >= d) continue;
            if constexpr (sizeof(ET) == 2) {
                store_piece_of<NT>(reinterpret_cast<uint4*>(dX + (size_t)t * d + c),
                    make_uint4(pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3]),
                               pack_bf16x2(sum[4 % VN], sum[5 % VN]), pack_bf16x2(sum[6 % VN], sum[7 % VN])));
            } else {
                store_piece_of<NT>(reinterpret_cast<float4*>(dX + (size_t)t * d + c), make_float4(sum[0], sum[1], sum[2], sum[3]));
            }
        }
        if constexpr (PREFETCH)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < KMAX; ++j) raw[r][j] = ahead[r][j];
    }
}

// ---- dWg, dbg ---------------------------------------------------------------------------------------
// dWg = X^T dlogits is a dense contraction over the tokens.  In fp32 on the 16x16x4 MFMA, one instruction
// multiplies 16 columns of X by 16 experts over 4 tokens.  Lane l supplies X[token l/16][its column l%16] as
// the A operand and dlogits[token l/16][expert l%16] as the B operand, so both come straight from coalesced
// loads with no exchange between lanes: a lane loads VN consecutive columns of one token (16 bytes) and the VN
// values go to VN instructions, each with its own 16 x 16 accumulator.
// Accumulator j of a strip holds columns strip0 + i * VN + j (i = 0..15) against the 16 experts of a tile:
// lane l, register r is column index i = 4 (l / 16) + r, expert l % 16.
// A block's four waves take every fourth group of 4 tokens of the partition; their sums are folded through
// LDS in a fixed order and written as one partial per token partition (the reduce kernel adds those).
// What bounds it: HBM (X once) beside the matrix rate from E = 32 on, and before either the latency of a wave's loads: a
// wave requests its next 16 tokens before it multiplies the current ones, four waves per SIMD.  More than 32 experts are
// further blocks of the same launch: X comes from cache for them.  Product | sum of the partials, us, with two waves per SIMD,
// loads under selects, 32 partitions of 256 tokens and more, and waves folded one after the other -> now: T = 16384, d = 2048, E
// = 32: 30 | 12 -> 28 | 5, E = 64: 57 | 12 -> 45 | 5; T = 8001, d = 2048, E = 128: 61 | 13 -> 47 | 7; T = 9000, d = 3072, E = 100:
// 102 | 14 -> 76 | 7; T = 32768, d = 4096, E = 16: 79 | 8 -> 79 | 5; T = 4000, d = 1024, E = 16: 14 | 4 -> 7 | 4; T = 584, d =
// 1984, E = 8: 13.5 | 4 -> 5.7 | 2.8.  (The sum's bias took its partitions one by one and was what the launch waited for.)
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <typename ET, int VN, int NE, int CS, bool NT>
__global__ __launch_bounds__(256, sizeof(ET) == 2 ? 4 : 2) void gate_wgrad_mfma_kernel(
    const ET* __restrict__ X, const float* __restrict__ dlogits, float* __restrict__ partial,
    float* __restrict__ partial_b, int T, int d, int E, int tok_per_part)
{
    const int e0 = blockIdx.z * 16 * NE;                           // first expert of the block
    constexpr int SW = 16 * VN;                                    // columns of one strip
    constexpr int NACC = CS * VN * NE;                             // 16 x 16 accumulators of a wave
    typedef typename std::conditional<sizeof(ET) == 2, uint4, float4>::type raw_t;
    static_assert(sizeof(ET) * VN == 16, "a lane loads 16 bytes of a row");
    __shared__ __attribute__((aligned(16))) float fold[4 * NACC / 2 * 4 * 64];
    __shared__ float fold_b[4 * NE * 16];
    static_assert(NACC % 8 == 0, "a quarter of half of the accumulators per wave");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;                      // column / expert of the lane, token of the lane
    const int c0 = blockIdx.x * (CS * SW);
    const int part = blockIdx.y;
    const int t_begin = part * tok_per_part, t_end = min(T, t_begin + tok_per_part);

    f32x4_t acc[CS][VN][NE];
#pragma unroll
    for (int s = 0; s < CS; ++s)
#pragma unroll
        for (int j = 0; j < VN; ++j)
#pragma unroll
            for (int n = 0; n < NE; ++n) acc[s][j][n] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float accb[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) accb[n] = 0.0f;

    constexpr int U = 4;                                           // groups of 4 tokens requested together: one trip
    // bf16: buffer loads from the trip's first token on, whose resource ends with the partition: tokens past it, columns past d
    // and experts past E arrive as zeros, and a trip has no vector instruction beside the conversions (each takes about 8
    // cycles from the matrix units).  fp32, whose rows may be too long for an offset: unconditional loads (tokens past the
    // partition and columns past d read valid ones, replaced by zeros when used).
    constexpr bool BUF = sizeof(ET) == 2;
    constexpr int NOWHERE = (int)0x80000000u;
    int voff_x[CS], voff_dl[NE];
    if (BUF) {
#pragma unroll
        for (int s = 0; s < CS; ++s) voff_x[s] = c0 + s * SW + li * VN < d ? (lk * d + c0 + s * SW + li * VN) * 2 : NOWHERE;
#pragma unroll
        for (int n = 0; n < NE; ++n) voff_dl[n] = e0 + n * 16 + li < E ? (lk * E + e0 + n * 16 + li) * 4 : NOWHERE;
    }
    auto load_trip = [&](int tg, raw_t (&raw)[U][CS], float (&dl)[U][NE]) {
        if constexpr (BUF) {
            auto rsrc = [&](const void* base, long bytes) {
                return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes < 0 ? 0 : (bytes > 0x7fffffffl ? 0x7fffffffl : bytes)), 0x00020000);
            };
            const auto rx = rsrc(X + (size_t)tg * d, (long)(t_end - tg) * d * 2), rd = rsrc(dlogits + (size_t)tg * E, (long)(t_end - tg) * E * 4);
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int n = 0; n < NE; ++n) dl[u][n] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, voff_dl[n], 16 * u * E * 4, 0));
#pragma unroll
                for (int s = 0; s < CS; ++s) raw[u][s] = __builtin_bit_cast(raw_t, __builtin_amdgcn_raw_buffer_load_b128(rx, voff_x[s], 16 * u * d * 2, NT ? 2 : 0));
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = min(tg + 16 * u + lk, T - 1);
#pragma unroll
                for (int n = 0; n < NE; ++n) {
                    const int e = e0 + n * 16 + li;
                    dl[u][n] = dlogits[(size_t)t * E + (e < E ? e : 0)];
                }
#pragma unroll
                for (int s = 0; s < CS; ++s) {
                    const int c = c0 + s * SW + li * VN;
                    raw[u][s] = load_piece_of<NT>(reinterpret_cast<const raw_t*>(X + (size_t)t * d + (c < d ? c : 0)));
                }
            }
        }
    };
    auto use_trip = [&](int tg, const raw_t (&raw)[U][CS], const float (&dl)[U][NE]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool tv = BUF || tg + 16 * u + lk < t_end;
            float g[NE];
#pragma unroll
            for (int n = 0; n < NE; ++n) g[n] = (BUF || (tv && e0 + n * 16 + li < E)) ? dl[u][n] : 0.0f;
#pragma unroll
            for (int s = 0; s < CS; ++s) {
                const raw_t w = (BUF || (tv && c0 + s * SW + li * VN < d)) ? raw[u][s] : raw_t{};
                float x[VN];
                if constexpr (sizeof(ET) == 2) {
                    unpack_bf16x8(w, x);
                } else {
                    x[0] = w.x; x[1] = w.y; x[2] = w.z; x[3] = w.w;
                }
#pragma unroll
                for (int j = 0; j < VN; ++j)
#pragma unroll
                    for (int n = 0; n < NE; ++n)
                        acc[s][j][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], g[n], acc[s][j][n], 0, 0, 0);
            }
#pragma unroll
            for (int n = 0; n < NE; ++n) accb[n] += g[n];
        }
    };
    // the next trip of a wave is on its way while the current one is multiplied (two register sets)
    constexpr int TRIP = 16 * U;
    raw_t raw0[U][CS], raw1[U][CS];
    float dl0[U][NE], dl1[U][NE];
    int tg = t_begin + 4 * wave;
    load_trip(tg, raw0, dl0);
    while (tg < t_end) {
        load_trip(tg + TRIP, raw1, dl1);
        use_trip(tg, raw0, dl0);
        tg += TRIP;
        if (tg >= t_end) break;
        load_trip(tg + TRIP, raw0, dl0);
        use_trip(tg, raw1, dl1);
        tg += TRIP;
    }
    // lanes with the same l % 16 hold pieces of the same bias gradient
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        accb[n] += __shfl_xor(accb[n], 16, 64);
        accb[n] += __shfl_xor(accb[n], 32, 64);
    }
    // fold the four waves, in wave order: every wave leaves its sums in LDS, half of them at a time, and adds up and writes a
    // quarter of those
    if (lane < 16)
#pragma unroll
        for (int n = 0; n < NE; ++n) fold_b[(wave * NE + n) * 16 + lane] = accb[n];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        if (half) __syncthreads();
#pragma unroll
        for (int i = 0; i < NACC / 2; ++i) {
            const int a = half * (NACC / 2) + i;
            *reinterpret_cast<f32x4_t*>(fold + ((wave * (NACC / 2) + i) * 64 + lane) * 4) = acc[a / NE / VN][a / NE % VN][a % NE];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NACC / 8; ++i) {
            const int h = wave * (NACC / 8) + i, a = half * (NACC / 2) + h, n = a % NE, j = a / NE % VN, s = a / NE / VN;
            f32x4_t sum = *reinterpret_cast<const f32x4_t*>(fold + (h * 64 + lane) * 4);
#pragma unroll
            for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const f32x4_t*>(fold + ((w * (NACC / 2) + h) * 64 + lane) * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = c0 + s * SW + (4 * lk + r) * VN + j, e = e0 + n * 16 + li;
                if (c < d && e < E) partial[((size_t)part * d + c) * E + e] = sum[r];
            }
        }
    }
    if (blockIdx.x == 0 && tid < NE * 16 && e0 + tid < E) {
        float sum = fold_b[tid];
#pragma unroll
        for (int w = 1; w < 4; ++w) sum += fold_b[w * NE * 16 + tid];
        partial_b[(size_t)part * E + e0 + tid] = sum;
    }
}


// Columns and experts of a block of gate_wgrad_mfma_kernel.
inline int wgrad_columns(const moe_shape_t& s) { return s.dtype == MOE_BF16 ? (s.E <= 16 ? 256 : 128) : 128; }
inline int wgrad_experts(const moe_shape_t& s) { return s.E <= 16 ? 16 : 32; }

template <typename ET, int VN, int NE, int CS>
hipError_t launch_wgrad_mfma_t(const moe_shape_t& s, const void* X, const float* dlogits, float* partial, float* partial_b,
                               int n_part, int tok_per_part, hipStream_t st)
{
    const int cw = CS * 16 * VN;
    if (cw != wgrad_columns(s) || 16 * NE != wgrad_experts(s)) return hipErrorInvalidValue;
    const dim3 grid((s.d + cw - 1) / cw, n_part, (s.E + 16 * NE - 1) / (16 * NE));
    // X for the last time, and once: further blocks of experts find it in the caches
    auto launch = [&](auto NT) {
        hipLaunchKernelGGL((gate_wgrad_mfma_kernel<ET, VN, NE, CS, decltype(NT)::value>), grid, dim3(256), 0, st, (const ET*)X, dlogits, partial,
                           partial_b, s.T, s.d, s.E, tok_per_part);
        return hipGetLastError();
    };
    return grid.z == 1 && streams((size_t)s.T * s.d * sizeof(ET)) ? launch(std::true_type{}) : launch(std::false_type{});
}

// N partials (FULL) or the n < N that are left, all loads on their way at once, added to four sums: one after the other, 64 partials
// would cost the bias as much precision as the chains that made them.  An addition per load: with the address of each computed
// from its number they went out slowly.
template <int N, bool FULL>
__device__ __forceinline__ void add_partials(float (&sum)[4], const float* __restrict__ p, int i, size_t stride, int n)
{
    float v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) { v[q] = p[i]; if (FULL || q + 1 < n) p += stride; }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < N; ++q) if (FULL || q < n) sum[q % 4] += v[q];
}
// As few loads as there are partials: 32 of them for one or two were most of the launch (T = 17, d = 3584, E = 256, with the product
// 14.7 us, now 9.9; T = 130, d = 3520, three partials 19.9, two now 14.4).
__device__ __forceinline__ float sum_partials(const float* __restrict__ p, int i, size_t stride, int n_part)
{
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (; n_part >= 32; n_part -= 32, p += 32 * stride) add_partials<32, true>(sum, p, i, stride, 32);
    if (n_part > 16) add_partials<32, false>(sum, p, i, stride, n_part);
    else if (n_part > 4) add_partials<16, false>(sum, p, i, stride, n_part);
    else if (n_part > 0) add_partials<4, false>(sum, p, i, stride, n_part);
    return (sum[0] + sum[1]) + (sum[2] + sum[3]);
}
// The last block adds up the bias.
__global__ __launch_bounds__(256) void gate_wgrad_reduce_kernel(const float* __restrict__ partial, const float* __restrict__ partial_b,
                                                                float* __restrict__ dWg, float* __restrict__ dbg, int n_part, int dE, int E)
{
    if (blockIdx.x + 1 == gridDim.x) {
        for (int e = threadIdx.x; e < E; e += 256) dbg[e] = sum_partials(partial_b, e, E, n_part);
        return;
    }
    const size_t first = (size_t)blockIdx.x * 256;
    if (first + threadIdx.x < (size_t)dE) dWg[first + threadIdx.x] = sum_partials(partial + first, threadIdx.x, dE, n_part);
}

}  // namespace

// Token partitions: as many as give the blocks that run at once, at most 64, of whole trips of the four waves (64 tokens; a trip
// that is nearly empty takes as long as a full one, and every partition is a partial to write and to add: fp32, T = 4894, d = 1180,
// E = 16, 64 partitions of two trips, the second of 13 tokens, 18.1 us, 39 partitions 13.4).  At once: four per CU (128
// registers, 33 KB of LDS), three of fp32 with more than 16 experts (168 registers).  More than 128 experts: no more than have 8 MB
// of partials (T = 199, d = 3648, E = 256, 14.9 MB 18.5, 7.5 MB 15.3; fewer experts have not been slower than with 256
// tokens a partition).
// Where the experts are several blocks, a multiple of eight if one is near, so that those which read the same tokens run on one
// XCD and share its L2 (blocks are dealt to the XCDs in turn; fp32, T = 28001, d = 468, E = 64 63 partitions 33.3, 64 30.4).
// But never fewer than 32, or one per 256 tokens: a wave adds up T / (4 partitions) products one after the other, and longer
// chains lose precision.  Error against 64 bits and time with that many | with the blocks that run at once alone: T = 9000, d =
// 3072, E = 100 1.9e-7, 81 us | 2.8e-7, 69 us; T = 16384, d = 4096, E = 128 2.3e-7, 161 us | 4.1e-7, 144 us; T = 8192, d = 2176,
// E = 1024 (one partition) 1.8e-7, 375 us | 8.1e-7, 425 us.
int gate_grad_partitions(const moe_shape_t& s)
{
    const long blocks = (long)((s.d + wgrad_columns(s) - 1) / wgrad_columns(s)) * ((s.E + wgrad_experts(s) - 1) / wgrad_experts(s));
    const long at_once = s.dtype == MOE_F32 && s.E > 16 ? 768 : 1024;
    const long trips = (s.T + 63) / 64, least = std::min<long>(32, (s.T + 255) / 256);
    long want = std::min<long>(64, at_once / blocks);
    if (s.E > 128) want = std::min<long>(want, (8l << 20) / ((long)s.d * s.E * 4));
    want = std::min(trips, std::max(least, want));
    const long each = (trips + want - 1) / want, n = std::max(least, (trips + each - 1) / each), eights = (n + 7) / 8 * 8;
    return (int)(s.E > wgrad_experts(s) && eights * 8 <= n * 9 && eights <= trips && eights * blocks <= at_once ? eights : n);
}

template <typename ET, int NE, int KMAX>
hipError_t launch_input_grad_t(const moe_shape_t& s, const void* dXp, const int32_t* pos, const float* dlogits,
                               const float* Wg, void* dX, hipStream_t st)
{
    constexpr int VN = 16 / sizeof(ET), SW = 16 * VN;
    constexpr size_t lds = (size_t)4 * NE * 64 * VN * sizeof(float);               // 64 KB for 128 experts and bf16
    const int strips = (s.d + SW - 1) / SW, t64 = (s.T + 63) / 64;
    // groups of tokens per wave: as many as leave four blocks per CU, up to 8 (the staging of Wg is 1/8 of a group's
    // traffic by then)
    long gpw = (long)strips * t64 / 1024;
    gpw = gpw < 1 ? 1 : (gpw > 8 ? 8 : gpw);
    const dim3 grid(strips, (unsigned)((t64 + gpw - 1) / gpw));
    const int vec = s.E % 4 == 0 && ((reinterpret_cast<uintptr_t>(Wg) | reinterpret_cast<uintptr_t>(dlogits)) & 15) == 0;
    auto launch = [&](auto NT) {
        hipLaunchKernelGGL((input_grad_kernel<ET, NE, KMAX, decltype(NT)::value>), grid, dim3(256), lds, st, (const ET*)dXp, pos, dlogits, Wg,
                           (ET*)dX, s.T, s.d, s.E, s.k, (int)gpw, vec);
        return hipGetLastError();
    };
    return streams((size_t)s.T * s.d * sizeof(ET)) ? launch(std::true_type{}) : launch(std::false_type{});
}

template <typename ET, int NE>
hipError_t launch_input_grad_k(const moe_shape_t& s, const void* dXp, const int32_t* pos, const float* dlogits,
                               const float* Wg, void* dX, hipStream_t st)
{
    if (s.k == 1) return launch_input_grad_t<ET, NE, 1>(s, dXp, pos, dlogits, Wg, dX, st);
    if (s.k == 2) return launch_input_grad_t<ET, NE, 2>(s, dXp, pos, dlogits, Wg, dX, st);
    if (s.k <= 4) return launch_input_grad_t<ET, NE, 4>(s, dXp, pos, dlogits, Wg, dX, st);
    return launch_input_grad_t<ET, NE, 8>(s, dXp, pos, dlogits, Wg, dX, st);
}

template <typename ET>
hipError_t launch_input_grad_e(const moe_shape_t& s, const void* dXp, const int32_t* pos, const float* dlogits,
                               const float* Wg, void* dX, hipStream_t st)
{
    if (s.E <= 16) return launch_input_grad_k<ET, 1>(s, dXp, pos, dlogits, Wg, dX, st);
    if (s.E <= 32) return launch_input_grad_k<ET, 2>(s, dXp, pos, dlogits, Wg, dX, st);
    if (s.E <= 64) return launch_input_grad_k<ET, 4>(s, dXp, pos, dlogits, Wg, dX, st);
    return launch_input_grad_k<ET, 8>(s, dXp, pos, dlogits, Wg, dX, st);
}

hipError_t launch_input_grad(const moe_shape_t& s, const void* dXp, const int32_t* pos, const float* dlogits,
                             const float* Wg, void* dX, hipStream_t st)
{
    return s.dtype == MOE_BF16 ? launch_input_grad_e<bf16_t>(s, dXp, pos, dlogits, Wg, dX, st)
                               : launch_input_grad_e<float>(s, dXp, pos, dlogits, Wg, dX, st);
}

hipError_t launch_gate_wgrad(const moe_shape_t& s, const void* X, const float* dlogits, float* partial, float* partial_b,
                             float* dWg, float* dbg, hipStream_t st)
{
    const int n_part = gate_grad_partitions(s);
    const int tok_per_part = (s.T + n_part - 1) / n_part;
    hipError_t e;
    const bool bf = s.dtype == MOE_BF16;
    if (s.E <= 16)      e = bf ? launch_wgrad_mfma_t<bf16_t, 8, 1, 2>(s, X, dlogits, partial, partial_b, n_part, tok_per_part, st)
                               : launch_wgrad_mfma_t<float, 4, 1, 2>(s, X, dlogits, partial, partial_b, n_part, tok_per_part, st);
    else                e = bf ? launch_wgrad_mfma_t<bf16_t, 8, 2, 1>(s, X, dlogits, partial, partial_b, n_part, tok_per_part, st)
                               : launch_wgrad_mfma_t<float, 4, 2, 2>(s, X, dlogits, partial, partial_b, n_part, tok_per_part, st);
    if (e != hipSuccess) return e;
    const int dE = s.d * s.E;
    hipLaunchKernelGGL(gate_wgrad_reduce_kernel, dim3((dE + 255) / 256 + 1), dim3(256), 0, st, partial, partial_b, dWg, dbg, n_part, dE, s.E);
    return hipGetLastError();
}
