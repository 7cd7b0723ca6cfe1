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
// d = 4096, E = 16: 172 -> 172 (807 MB, 4.7 TB/s).
typedef __attribute__((ext_vector_type(4))) float ig_f32x4_t;

// waves per SIMD the compiler is held to: 4, or 2 where the row pieces (16 KMAX registers) or the LDS leave no room for that
template <typename ET, int NE, int KMAX>
__global__ __launch_bounds__(256, KMAX <= 2 && NE < 8 ? 4 : 2) void input_grad_kernel(
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

    for (int gi = 0; gi < groups_per_wave; ++gi) {
        const int tg = (blockIdx.y * groups_per_wave + gi) * 64 + wave * 16;
        raw_t raw[4][KMAX];
        int lowest = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = min(tg + 4 * lq + r, T - 1);
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                const int row = pos[(size_t)t * k + (j < k ? j : 0)];
                lowest = min(lowest, row);
                raw[r][j] = *reinterpret_cast<const raw_t*>(dXp + (size_t)max(row, 0) * d + cc);
            }
        }
        if (__any(lowest < 0))
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < KMAX; ++j)
                    if (j < k && pos[(size_t)min(tg + 4 * lq + r, T - 1) * k + j] < 0) raw[r][j] = raw_t{};
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
                *reinterpret_cast<uint4*>(dX + (size_t)t * d + c) =
                    make_uint4(pack_bf16x2(sum[0], sum[1]), pack_bf16x2(sum[2], sum[3]),
                               pack_bf16x2(sum[4 % VN], sum[5 % VN]), pack_bf16x2(sum[6 % VN], sum[7 % VN]));
            } else {
                *reinterpret_cast<float4*>(dX + (size_t)t * d + c) = make_float4(sum[0], sum[1], sum[2], sum[3]);
            }
        }
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
// What bounds it: HBM (X once) beside the matrix rate from E = 32 on, and before either the latency of a wave's loads:
// with the accumulators of 32 experts there are two waves per SIMD, so a wave requests its next 16 tokens before it
// multiplies the current ones (held to 256 registers; without the bound the compiler takes a whole SIMD for one wave,
// 52 us).  More than 32 experts are further blocks of the same launch: X comes from cache for them, and twice the blocks
// with half the accumulators (64 experts in one wave) fill the chip.  Both kernels, us, before -> after: T = 16384,
// d = 2048, E = 32: 45 -> 40, E = 64: 85 -> 65; T = 32768, d = 4096, E = 16: 79 -> 68; T = 8001, d = 2048, E = 128:
// 109 -> 72; T = 4000, d = 1024, E = 100: 52 -> 24.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <typename ET, int VN, int NE, int CS>
__global__ __launch_bounds__(256, 2) void gate_wgrad_mfma_kernel(
    const ET* __restrict__ X, const float* __restrict__ dlogits, float* __restrict__ partial,
    float* __restrict__ partial_b, int T, int d, int E, int tok_per_part)
{
    const int e0 = blockIdx.z * 16 * NE;                           // first expert of the block
    constexpr int SW = 16 * VN;                                    // columns of one strip
    constexpr int NACC = CS * VN * NE;                             // 16 x 16 accumulators of a wave
    typedef typename std::conditional<sizeof(ET) == 2, uint4, float4>::type raw_t;
    static_assert(sizeof(ET) * VN == 16, "a lane loads 16 bytes of a row");
    __shared__ float fold[NACC * 4 * 64];
    __shared__ float fold_b[NE * 16];
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
    // unconditional loads (tokens past the partition and columns past d read valid ones, replaced by zeros when used)
    auto load_trip = [&](int tg, raw_t (&raw)[U][CS], float (&dl)[U][NE]) {
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
                raw[u][s] = *reinterpret_cast<const raw_t*>(X + (size_t)t * d + (c < d ? c : 0));
            }
        }
    };
    auto use_trip = [&](int tg, const raw_t (&raw)[U][CS], const float (&dl)[U][NE]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool tv = tg + 16 * u + lk < t_end;
            float g[NE];
#pragma unroll
            for (int n = 0; n < NE; ++n) g[n] = (tv && e0 + n * 16 + li < E) ? dl[u][n] : 0.0f;
#pragma unroll
            for (int s = 0; s < CS; ++s) {
                const raw_t w = (tv && c0 + s * SW + li * VN < d) ? raw[u][s] : raw_t{};
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
    // fold the four waves: waves 1, 2, 3 hand their sums to wave 0 one after the other
    for (int w = 1; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int s = 0; s < CS; ++s)
#pragma unroll
                for (int j = 0; j < VN; ++j)
#pragma unroll
                    for (int n = 0; n < NE; ++n)
#pragma unroll
                        for (int r = 0; r < 4; ++r) fold[((((s * VN + j) * NE + n) * 4) + r) * 64 + lane] = acc[s][j][n][r];
            if (lane < 16)
#pragma unroll
                for (int n = 0; n < NE; ++n) fold_b[n * 16 + lane] = accb[n];
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int s = 0; s < CS; ++s)
#pragma unroll
                for (int j = 0; j < VN; ++j)
#pragma unroll
                    for (int n = 0; n < NE; ++n)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[s][j][n][r] += fold[((((s * VN + j) * NE + n) * 4) + r) * 64 + lane];
            if (lane < 16)
#pragma unroll
                for (int n = 0; n < NE; ++n) accb[n] += fold_b[n * 16 + lane];
        }
        __syncthreads();
    }
    if (wave == 0) {
#pragma unroll
        for (int s = 0; s < CS; ++s)
#pragma unroll
            for (int j = 0; j < VN; ++j)
#pragma unroll
                for (int n = 0; n < NE; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int c = c0 + s * SW + (4 * lk + r) * VN + j, e = e0 + n * 16 + li;
                        if (c < d && e < E) partial[((size_t)part * d + c) * E + e] = acc[s][j][n][r];
                    }
        if (blockIdx.x == 0 && lane < 16)
#pragma unroll
            for (int n = 0; n < NE; ++n)
                if (e0 + n * 16 + lane < E) partial_b[(size_t)part * E + e0 + n * 16 + lane] = accb[n];
    }
}

template <typename ET, int VN, int NE, int CS>
hipError_t launch_wgrad_mfma_t(const moe_shape_t& s, const void* X, const float* dlogits, float* partial, float* partial_b,
                               int n_part, int tok_per_part, hipStream_t st)
{
    const int cw = CS * 16 * VN;
    const dim3 grid((s.d + cw - 1) / cw, n_part, (s.E + 16 * NE - 1) / (16 * NE));
    hipLaunchKernelGGL((gate_wgrad_mfma_kernel<ET, VN, NE, CS>), grid, dim3(256), 0, st, (const ET*)X, dlogits, partial,
                       partial_b, s.T, s.d, s.E, tok_per_part);
    return hipGetLastError();
}

__global__ void gate_wgrad_reduce_kernel(const float* __restrict__ partial, const float* __restrict__ partial_b,
                                         float* __restrict__ dWg, float* __restrict__ dbg, int n_part, int dE, int E)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < dE) {
        float s = 0.0f;
        int p = 0;
        for (; p + 16 <= n_part; p += 16) {                        // sixteen loads in flight, added in partition order
            float v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = partial[(size_t)(p + q) * dE + i];
#pragma unroll
            for (int q = 0; q < 16; ++q) s += v[q];
        }
        for (; p < n_part; ++p) s += partial[(size_t)p * dE + i];
        dWg[i] = s;
    }
    if (i < E) {
        float s = 0.0f;
        for (int p = 0; p < n_part; ++p) s += partial_b[(size_t)p * E + i];
        dbg[i] = s;
    }
}

}  // namespace

int gate_grad_partitions(const moe_shape_t& s) { return s.T < 32 * 256 ? (s.T + 255) / 256 : 32; }

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
    hipLaunchKernelGGL((input_grad_kernel<ET, NE, KMAX>), grid, dim3(256), lds, st, (const ET*)dXp, pos, dlogits, Wg,
                       (ET*)dX, s.T, s.d, s.E, s.k, (int)gpw, vec);
    return hipGetLastError();
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
    hipLaunchKernelGGL(gate_wgrad_reduce_kernel, dim3((dE + 255) / 256), dim3(256), 0, st, partial, partial_b, dWg, dbg, n_part, dE, s.E);
    return hipGetLastError();
}
