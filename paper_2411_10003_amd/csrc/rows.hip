// Row movers bound by HBM bandwidth: the send buffer of the first all-to-all (dispatch), the
// weighted return after the second one (combine), and their gradients (Fig. 2 of the paper and
// the two backward all-to-alls of its performance model, Section 4.2).
//
// One wavefront owns one token.  A token's row is read once and written to its k send rows
// (scatter form of Xp[r] = X[perm[r]/k]), so traffic is the algorithmic minimum
// (1 + k) * T * d elements.  Lanes move 16 bytes per access.
#include "internal.h"

#include <type_traits>

namespace {

constexpr int ROW_WAVES = 4;   // tokens per block
constexpr int MAXK = 8;

template <typename ET> struct Vec;                      // 16-byte vector of elements
template <> struct Vec<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void unpack(const uint4& v, float* f) {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
    static __device__ __forceinline__ uint4 pack(const float* f) {
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    }
};
template <> struct Vec<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void unpack(const uint4& v, float* f) {
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
        f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
        f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
    }
    static __device__ __forceinline__ uint4 pack(const float* f) {
        return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
    }
};

__device__ __forceinline__ float wave_sum(float v) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Xp[pos[t*k+j], :] = X[t, :]
template <typename ET, bool NT>
__global__ __launch_bounds__(ROW_WAVES * 64) void scatter_rows_kernel(
    const ET* __restrict__ X, const int32_t* __restrict__ pos, ET* __restrict__ Xp, int T, int d, int k)
{
    constexpr int VN = Vec<ET>::N;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROW_WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const uint4* src = reinterpret_cast<const uint4*>(X + (size_t)t * d);
    const int nv = d / VN;
    for (int j = 0; j < k; ++j) {
        // the row is re-read from cache for j > 0; HBM sees it once
        uint4* dst = reinterpret_cast<uint4*>(Xp + (size_t)pos[(size_t)t * k + j] * d);
#pragma unroll 4
        for (int v = lane; v < nv; v += 64) store_piece_of<NT>(dst + v, src[v]);
    }
}

// K-specialised variant: every 16-byte piece is loaded once and stored K times.
template <typename ET, int K, bool NT>
__global__ __launch_bounds__(ROW_WAVES * 64) void scatter_rows_k_kernel(
    const ET* __restrict__ X, const int32_t* __restrict__ pos, ET* __restrict__ Xp, int T, int d)
{
    constexpr int VN = Vec<ET>::N;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROW_WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const uint4* src = reinterpret_cast<const uint4*>(X + (size_t)t * d);
    uint4* dst[K];
#pragma unroll
    for (int j = 0; j < K; ++j) dst[j] = reinterpret_cast<uint4*>(Xp + (size_t)pos[(size_t)t * K + j] * d);
    const int nv = d / VN;
#pragma unroll 4
    for (int v = lane; v < nv; v += 64) {
        const uint4 x = src[v];
#pragma unroll
        for (int j = 0; j < K; ++j) store_piece_of<NT>(dst[j] + v, x);
    }
}

// out[t,:] = sum_j w[t,j] * Yp[pos[t*k+j],:]   (fp32, ascending j, one rounding)
// Bound by HBM: what counts is how many pieces of a token's rows are on their way.  KT is k where it is 1, 2 or 4 (bf16);
// with any k in one loop every row is a branch and one piece of each row is out at a time: k = 4, T = 8000, d = 4096 83 -> 62 us
// (caches swept 125 -> 110), T = 8001, d = 2048 27 -> 25 (71 -> 61).  The scatter gains nothing from more registers: k = 8 97 -> 100.
template <typename ET, int KT, bool NT>
__global__ __launch_bounds__(ROW_WAVES * 64) void combine_kernel(
    const ET* __restrict__ Yp, const int32_t* __restrict__ pos, const float* __restrict__ w,
    ET* __restrict__ out, int T, int d, int k_rt)
{
    constexpr int VN = Vec<ET>::N;
    constexpr int KMAX = KT ? KT : MAXK;
    const int k = KT ? KT : k_rt;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROW_WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const uint4* src[KMAX];
    float wj[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        if (j < k) {
            src[j] = reinterpret_cast<const uint4*>(Yp + (size_t)pos[(size_t)t * k + j] * d);
            wj[j] = w[(size_t)t * k + j];
        }
    }
    uint4* dst = reinterpret_cast<uint4*>(out + (size_t)t * d);
    const int nv = d / VN;
    constexpr int U = (KT == 1 || KT == 2) ? 4 : (KT == 4 ? 2 : 1);      // 16-byte pieces per row and lane requested before any is used
    for (int v0 = lane; v0 < nv; v0 += 64 * U) {
        uint4 raw[U][KMAX];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if (j < k && v0 + 64 * u < nv) raw[u][j] = src[j][v0 + 64 * u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (v0 + 64 * u >= nv) break;
            float acc[VN];
#pragma unroll
            for (int i = 0; i < VN; ++i) acc[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                if (j < k) {
                    float y[VN];
                    Vec<ET>::unpack(raw[u][j], y);
#pragma unroll
                    for (int i = 0; i < VN; ++i) acc[i] = fmaf(wj[j], y[i], acc[i]);
                }
            }
            store_piece_of<NT>(dst + v0 + 64 * u, Vec<ET>::pack(acc));
        }
    }
}

// dYp[pos[a],:] = w[a] * dOut[t,:] ;  dw[t,j] = <dOut[t,:], Yp[pos[a],:]>
template <typename ET, int KT, bool NT>
__global__ __launch_bounds__(ROW_WAVES * 64) void combine_bwd_kernel(
    const ET* __restrict__ dOut, const ET* __restrict__ Yp, const int32_t* __restrict__ pos,
    const float* __restrict__ w, ET* __restrict__ dYp, float* __restrict__ dw, int T, int d, int k_rt)
{
    constexpr int VN = Vec<ET>::N;
    constexpr int KMAX = KT ? KT : MAXK;
    const int k = KT ? KT : k_rt;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROW_WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const uint4* ysrc[KMAX];
    uint4* gdst[KMAX];
    float wj[KMAX], dot[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        dot[j] = 0.0f;
        if (j < k) {
            const size_t row = (size_t)pos[(size_t)t * k + j];
            ysrc[j] = reinterpret_cast<const uint4*>(Yp + row * d);
            gdst[j] = reinterpret_cast<uint4*>(dYp + row * d);
            wj[j] = w[(size_t)t * k + j];
        }
    }
    const uint4* gsrc = reinterpret_cast<const uint4*>(dOut + (size_t)t * d);
    const int nv = d / VN;
    constexpr int U = KT ? 2 : 1;
    for (int v0 = lane; v0 < nv; v0 += 64 * U) {
        uint4 graw[U], yraw[U][KMAX];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (v0 + 64 * u < nv) {
                graw[u] = load_piece_of<NT>(gsrc + v0 + 64 * u);
#pragma unroll
                for (int j = 0; j < KMAX; ++j)
                    if (j < k) yraw[u][j] = load_piece_of<NT>(ysrc[j] + v0 + 64 * u);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (v0 + 64 * u >= nv) break;
            float g[VN];
            Vec<ET>::unpack(graw[u], g);
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                if (j < k) {
                    float y[VN], o[VN];
                    Vec<ET>::unpack(yraw[u][j], y);
#pragma unroll
                    for (int i = 0; i < VN; ++i) { dot[j] = fmaf(g[i], y[i], dot[j]); o[i] = wj[j] * g[i]; }
                    store_piece_of<NT>(gdst[j] + v0 + 64 * u, Vec<ET>::pack(o));
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        if (j < k) {
            const float s = wave_sum(dot[j]);
            if (lane == 0) dw[(size_t)t * k + j] = s;
        }
    }
}

// dX[t,:] = sum_j dXp[pos[t*k+j],:].  Its rows stay in the caches at any size (T = 32768, d = 4096, k = 2: 155 us, past them
// 175, and the step that goes on with them takes as long or longer: STREAM_BYTES).
template <typename ET, int KT>
__global__ __launch_bounds__(ROW_WAVES * 64) void dispatch_bwd_kernel(
    const ET* __restrict__ dXp, const int32_t* __restrict__ pos, ET* __restrict__ dX, int T, int d, int k_rt)
{
    constexpr int VN = Vec<ET>::N;
    constexpr int KMAX = KT ? KT : MAXK;
    const int k = KT ? KT : k_rt;
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * ROW_WAVES + (threadIdx.x >> 6);
    if (t >= T) return;
    const uint4* src[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
        if (j < k) src[j] = reinterpret_cast<const uint4*>(dXp + (size_t)pos[(size_t)t * k + j] * d);
    uint4* dst = reinterpret_cast<uint4*>(dX + (size_t)t * d);
    const int nv = d / VN;
    constexpr int U = (KT == 1 || KT == 2) ? 4 : 1;
    for (int v0 = lane; v0 < nv; v0 += 64 * U) {
        uint4 raw[U][KMAX];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
                if (j < k && v0 + 64 * u < nv) raw[u][j] = src[j][v0 + 64 * u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (v0 + 64 * u >= nv) break;
            float acc[VN];
#pragma unroll
            for (int i = 0; i < VN; ++i) acc[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {
                if (j < k) {
                    float y[VN];
                    Vec<ET>::unpack(raw[u][j], y);
#pragma unroll
                    for (int i = 0; i < VN; ++i) acc[i] += y[i];
                }
            }
            dst[v0 + 64 * u] = Vec<ET>::pack(acc);
        }
    }
}

inline dim3 row_grid(int T) { return dim3((T + ROW_WAVES - 1) / ROW_WAVES); }

// A launch has fewer than 2^32 threads, a token takes 64 of them, T may be just short of 2^30: tokens are taken 2^25 at a
// time (one launch for all but the largest batches).
constexpr int ROW_LAUNCH_TOK = 1 << 25;
template <typename LAUNCH>                               // launch(first token, shape of the part)
hipError_t for_token_parts(const moe_shape_t& s, LAUNCH launch)
{
    moe_shape_t part = s;
    hipError_t e = hipSuccess;
    for (int t0 = 0; t0 < s.T && e == hipSuccess; t0 += part.T) {
        part.T = s.T - t0 < ROW_LAUNCH_TOK ? s.T - t0 : ROW_LAUNCH_TOK;
        launch((size_t)t0, part);
        e = hipGetLastError();
    }
    return e;
}
inline size_t row_bytes(const moe_shape_t& s) { return (size_t)s.d * (s.dtype == MOE_BF16 ? 2 : 4); }
// bytes: those written
template <typename F> hipError_t by_size(size_t bytes, F launch) { return streams(bytes) ? launch(std::true_type{}) : launch(std::false_type{}); }
inline const void* at(const void* p, size_t bytes) { return (const char*)p + bytes; }
inline void* at(void* p, size_t bytes) { return (char*)p + bytes; }

}  // namespace

hipError_t launch_scatter_rows(const moe_shape_t& all, const void* X0, const int32_t* pos0, void* Xp, hipStream_t st)
{
    return by_size((size_t)all.T * all.k * row_bytes(all), [&](auto NT) {
    return for_token_parts(all, [&](size_t t0, const moe_shape_t& s) {
        constexpr bool nt = decltype(NT)::value;
        const dim3 g = row_grid(s.T), b(ROW_WAVES * 64);
        const void* X = at(X0, t0 * row_bytes(s));
        const int32_t* pos = pos0 + t0 * s.k;
        if (s.dtype == MOE_F32)
            hipLaunchKernelGGL((scatter_rows_kernel<float, nt>), g, b, 0, st, (const float*)X, pos, (float*)Xp, s.T, s.d, s.k);
        else if (s.k == 1)
            hipLaunchKernelGGL((scatter_rows_k_kernel<bf16_t, 1, nt>), g, b, 0, st, (const bf16_t*)X, pos, (bf16_t*)Xp, s.T, s.d);
        else if (s.k == 2)
            hipLaunchKernelGGL((scatter_rows_k_kernel<bf16_t, 2, nt>), g, b, 0, st, (const bf16_t*)X, pos, (bf16_t*)Xp, s.T, s.d);
        else
            hipLaunchKernelGGL((scatter_rows_kernel<bf16_t, nt>), g, b, 0, st, (const bf16_t*)X, pos, (bf16_t*)Xp, s.T, s.d, s.k);
    });
    });
}

hipError_t launch_combine(const moe_shape_t& all, const void* Yp, const int32_t* pos0, const float* w0, void* out0, hipStream_t st)
{
    return by_size((size_t)all.T * row_bytes(all), [&](auto NT) {
    return for_token_parts(all, [&](size_t t0, const moe_shape_t& s) {
        constexpr bool nt = decltype(NT)::value;
        const dim3 g = row_grid(s.T), b(ROW_WAVES * 64);
        const int32_t* pos = pos0 + t0 * s.k;
        const float* w = w0 + t0 * s.k;
        void* out = at(out0, t0 * row_bytes(s));
        if (s.dtype == MOE_F32)
            hipLaunchKernelGGL((combine_kernel<float, 0, nt>), g, b, 0, st, (const float*)Yp, pos, w, (float*)out, s.T, s.d, s.k);
        else if (s.k == 1)
            hipLaunchKernelGGL((combine_kernel<bf16_t, 1, nt>), g, b, 0, st, (const bf16_t*)Yp, pos, w, (bf16_t*)out, s.T, s.d, s.k);
        else if (s.k == 2)
            hipLaunchKernelGGL((combine_kernel<bf16_t, 2, nt>), g, b, 0, st, (const bf16_t*)Yp, pos, w, (bf16_t*)out, s.T, s.d, s.k);
        else if (s.k == 4)
            hipLaunchKernelGGL((combine_kernel<bf16_t, 4, nt>), g, b, 0, st, (const bf16_t*)Yp, pos, w, (bf16_t*)out, s.T, s.d, s.k);
        else
            hipLaunchKernelGGL((combine_kernel<bf16_t, 0, nt>), g, b, 0, st, (const bf16_t*)Yp, pos, w, (bf16_t*)out, s.T, s.d, s.k);
    });
    });
}

hipError_t launch_combine_bwd(const moe_shape_t& all, const void* dOut0, const void* Yp, const int32_t* pos0,
                              const float* w0, void* dYp, float* dw0, hipStream_t st)
{
    return by_size((size_t)all.T * all.k * row_bytes(all), [&](auto NT) {
    return for_token_parts(all, [&](size_t t0, const moe_shape_t& s) {
        constexpr bool nt = decltype(NT)::value;
        const dim3 g = row_grid(s.T), b(ROW_WAVES * 64);
        const void* dOut = at(dOut0, t0 * row_bytes(s));
        const int32_t* pos = pos0 + t0 * s.k;
        const float* w = w0 + t0 * s.k;
        float* dw = dw0 + t0 * s.k;
        if (s.dtype == MOE_F32)
            hipLaunchKernelGGL((combine_bwd_kernel<float, 0, nt>), g, b, 0, st, (const float*)dOut, (const float*)Yp, pos, w,
                               (float*)dYp, dw, s.T, s.d, s.k);
        else if (s.k == 1)
            hipLaunchKernelGGL((combine_bwd_kernel<bf16_t, 1, nt>), g, b, 0, st, (const bf16_t*)dOut, (const bf16_t*)Yp, pos, w,
                               (bf16_t*)dYp, dw, s.T, s.d, s.k);
        else if (s.k == 2)
            hipLaunchKernelGGL((combine_bwd_kernel<bf16_t, 2, nt>), g, b, 0, st, (const bf16_t*)dOut, (const bf16_t*)Yp, pos, w,
                               (bf16_t*)dYp, dw, s.T, s.d, s.k);
        else if (s.k == 4)
            hipLaunchKernelGGL((combine_bwd_kernel<bf16_t, 4, nt>), g, b, 0, st, (const bf16_t*)dOut, (const bf16_t*)Yp, pos, w,
                               (bf16_t*)dYp, dw, s.T, s.d, s.k);
        else
            hipLaunchKernelGGL((combine_bwd_kernel<bf16_t, 0, nt>), g, b, 0, st, (const bf16_t*)dOut, (const bf16_t*)Yp, pos, w,
                               (bf16_t*)dYp, dw, s.T, s.d, s.k);
    });
    });
}

hipError_t launch_dispatch_bwd(const moe_shape_t& all, const void* dXp, const int32_t* pos0, void* dX0, hipStream_t st)
{
    return for_token_parts(all, [&](size_t t0, const moe_shape_t& s) {
        const dim3 g = row_grid(s.T), b(ROW_WAVES * 64);
        const int32_t* pos = pos0 + t0 * s.k;
        void* dX = at(dX0, t0 * row_bytes(s));
        if (s.dtype == MOE_F32)
            hipLaunchKernelGGL((dispatch_bwd_kernel<float, 0>), g, b, 0, st, (const float*)dXp, pos, (float*)dX, s.T, s.d, s.k);
        else if (s.k == 1)
            hipLaunchKernelGGL((dispatch_bwd_kernel<bf16_t, 1>), g, b, 0, st, (const bf16_t*)dXp, pos, (bf16_t*)dX, s.T, s.d, s.k);
        else if (s.k == 2)
            hipLaunchKernelGGL((dispatch_bwd_kernel<bf16_t, 2>), g, b, 0, st, (const bf16_t*)dXp, pos, (bf16_t*)dX, s.T, s.d, s.k);
        else
            hipLaunchKernelGGL((dispatch_bwd_kernel<bf16_t, 0>), g, b, 0, st, (const bf16_t*)dXp, pos, (bf16_t*)dX, s.T, s.d, s.k);
    });
}

// ---- Trans on one GPU (Section 4.1: the parameters of a selected expert are transferred to the devices
// that will compute its inputs).  With every expert's parameters in one pool in this GPU's memory, the
// transfer is a gather of the hosted experts into the group slots the grouped FFN reads, driven by the
// plan as it lies in device memory: group g is the g-th expert e (ascending) with expert_dest[e] == self.
// A slot that already holds the right expert in its current version is left alone (placements change little
// from one iteration to the next, Section 3), which slot_expert[G] and slot_version[G] keep track of: an
// expert's parameters are updated before every transfer (Section 5.1), so the pool carries a version per
// expert that the caller bumps with every update, and a replica of an older version is copied again.
namespace {

// The g-th expert (ascending) that is hosted here, -1 if there are fewer.  All 64 lanes of the wave take part: one load and
// one ballot per 64 experts (a scalar walk over the experts waited for one load per expert, 5 us for 16 of them).
__device__ __forceinline__ int hosted_expert_of_group(const int32_t* __restrict__ expert_dest, int E, int self, int g)
{
    const int lane = threadIdx.x & 63;
    for (int e0 = 0; e0 < E; e0 += 64) {
        const unsigned long long m = __ballot(e0 + lane < E && expert_dest[min(e0 + lane, E - 1)] == self);
        const int n = __popcll(m);
        if (g < n) {
            const bool mine = ((m >> lane) & 1ull) && __popcll(m & ((1ull << lane) - 1ull)) == g;
            return e0 + __ffsll((unsigned long long)__ballot(mine)) - 1;
        }
        g -= n;
    }
    return -1;
}

// All tensors of a call in one launch: grid z is the tensor.
constexpr int MAX_TENSORS = 8, MOVE_UNROLL = 4;
struct MoveArgs { const uint4* src[MAX_TENSORS]; uint4* dst[MAX_TENSORS]; long vec[MAX_TENSORS]; };

// The pieces of 16 bytes of one slot and tensor, MOVE_UNROLL per lane and trip: load(u, i) requests piece i into register set u,
// store(u, i) uses it.  Bound by HBM and by how many loads are on their way: under a condition each they went out one by
// one (trans of 67 MB 33.8 -> 24.4 us, 5.5 TB/s).  The last trip's loads past the end read the last piece.
template <typename Load, typename Store>
__device__ __forceinline__ void move_pieces(long n, long lanes, Load load, Store store)
{
    long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
    for (; v + (MOVE_UNROLL - 1) * lanes < n; v += lanes * MOVE_UNROLL) {
#pragma unroll
        for (int u = 0; u < MOVE_UNROLL; ++u) load(u, v + u * lanes);
#pragma unroll
        for (int u = 0; u < MOVE_UNROLL; ++u) store(u, v + u * lanes);
    }
    if (v >= n) return;
#pragma unroll
    for (int u = 0; u < MOVE_UNROLL - 1; ++u) load(u, v + u * lanes < n ? v + u * lanes : n - 1);
#pragma unroll
    for (int u = 0; u < MOVE_UNROLL - 1; ++u)
        if (v + u * lanes < n) store(u, v + u * lanes);
}
// What is read once does not have to stay in the caches; what is written, and read next by others, does unless it is more than
// they keep (NT).  plan, trans of 67 MB and agg of 134 MB into as much, buffers that change from pass to pass | the same buffers
// every time: plain 118.5 | 113 us, sources past the caches 113 | 97.5, all of it 104 | 105.
typedef moe_piece_t piece_t;
typedef float fpiece_t __attribute__((ext_vector_type(4)));

// commit: the slot's expert, written here where no versions are kept (nobody reads it then); with versions other blocks of the
// slot still compare it, and a launch of its own writes both afterwards.  (Over 300 drawn moves of up to 67 MB
// it was a seventh of the call; in a pass that moves 134 MB its 4.8 us of 126 are within the spread.)
template <bool NT>
__global__ __launch_bounds__(256) void trans_gather_kernel(
    const int32_t* __restrict__ expert_dest, const int32_t* __restrict__ pool_version,
    const int32_t* slot_expert, const int32_t* __restrict__ slot_version, int32_t* commit, const MoveArgs a, int E, int self)
{
    const int g = blockIdx.y;
    const int e = hosted_expert_of_group(expert_dest, E, self, g);
    if (e < 0) return;                                     // unused slot: it keeps what it holds
    if (commit != nullptr && blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) commit[g] = e;
    // the expert is already there, in the version the pool holds now (no versions given: always copied)
    if (pool_version != nullptr && e == slot_expert[g] && slot_version[g] == pool_version[e]) return;
    const long vec_per_expert = a.vec[blockIdx.z], lanes = (long)gridDim.x * blockDim.x;
    const piece_t* __restrict__ src = reinterpret_cast<const piece_t*>(a.src[blockIdx.z]) + (long)e * vec_per_expert;
    piece_t* __restrict__ dst = reinterpret_cast<piece_t*>(a.dst[blockIdx.z]) + (long)g * vec_per_expert;
    piece_t r[MOVE_UNROLL];
    move_pieces(vec_per_expert, lanes, [&](int u, long i) { r[u] = load_piece_of<true>(src + i); }, [&](int u, long i) { store_piece_of<NT>(dst + i, r[u]); });
}

// one wave per slot
__global__ __launch_bounds__(64) void trans_commit_kernel(const int32_t* __restrict__ expert_dest, const int32_t* __restrict__ pool_version,
                                    int32_t* __restrict__ slot_expert, int32_t* __restrict__ slot_version, int E, int self)
{
    const int g = blockIdx.x;
    const int e = hosted_expert_of_group(expert_dest, E, self, g);
    if (e >= 0 && threadIdx.x == 0) {                      // an unused slot keeps what it holds
        slot_expert[g] = e;
        slot_version[g] = pool_version[e];
    }
}

// Agg on one GPU (Section 4.1: the gradients a replica computed are added to the expert's gradient where its
// parameters live).  The inverse walk of the gather above: the fp32 gradient of hosted group g is added to the
// pool entry of the expert the plan puts there.  Every element is touched by one thread: same bits every run.
template <bool NT>
__global__ __launch_bounds__(256) void agg_add_kernel(const int32_t* __restrict__ expert_dest, const MoveArgs a, int E, int self)
{
    const int g = blockIdx.y;
    const int e = hosted_expert_of_group(expert_dest, E, self, g);
    if (e < 0) return;
    const long vec_per_expert = a.vec[blockIdx.z], lanes = (long)gridDim.x * blockDim.x;
    const fpiece_t* __restrict__ src = reinterpret_cast<const fpiece_t*>(a.src[blockIdx.z]) + (long)g * vec_per_expert;
    fpiece_t* __restrict__ dst = reinterpret_cast<fpiece_t*>(a.dst[blockIdx.z]) + (long)e * vec_per_expert;
    fpiece_t x[MOVE_UNROLL], y[MOVE_UNROLL];
    move_pieces(vec_per_expert, lanes, [&](int u, long i) { x[u] = load_piece_of<true>(src + i); y[u] = load_piece_of<NT>(dst + i); },
                [&](int u, long i) { store_piece_of<NT>(dst + i, y[u] + x[u]); });
}

// Blocks per slot and tensor: one trip of four pieces per lane up to 512 blocks (8 MB), then a longer walk.
inline unsigned move_blocks(const MoveArgs& a, int n)
{
    long most = 1;
    for (int i = 0; i < n; ++i) most = a.vec[i] > most ? a.vec[i] : most;
    const long bx = (most + 256 * MOVE_UNROLL - 1) / (256 * MOVE_UNROLL);
    return (unsigned)(bx > 512 ? 512 : bx);
}

// Bytes written if every slot moves.
inline size_t move_bytes(const MoveArgs& a, int n, int G)
{
    size_t pieces = 0;
    for (int i = 0; i < n; ++i) pieces += (size_t)a.vec[i];
    return pieces * 16 * G;
}

}  // namespace

hipError_t launch_agg_add(const moe_shape_t& s, const int32_t* expert_dest, int n, const float* const* groups, float* const* pools,
                          const size_t* floats_per_expert, hipStream_t st)
{
    MoveArgs a{};
    for (int i = 0; i < n; ++i) { a.src[i] = (const uint4*)groups[i]; a.dst[i] = (uint4*)pools[i]; a.vec[i] = (long)(floats_per_expert[i] / 4); }
    return by_size(move_bytes(a, n, s.G), [&](auto NT) {
        hipLaunchKernelGGL(agg_add_kernel<decltype(NT)::value>, dim3(move_blocks(a, n), s.G, n), dim3(256), 0, st, expert_dest, a, s.E, s.self);
        return hipGetLastError();
    });
}

hipError_t launch_trans_gather(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* pool_version,
                               int32_t* slot_expert, const int32_t* slot_version,
                               int n, const void* const* pools, void* const* groups, const size_t* bytes_per_expert, hipStream_t st)
{
    MoveArgs a{};
    for (int i = 0; i < n; ++i) { a.src[i] = (const uint4*)pools[i]; a.dst[i] = (uint4*)groups[i]; a.vec[i] = (long)(bytes_per_expert[i] / 16); }
    return by_size(move_bytes(a, n, s.G), [&](auto NT) {
        hipLaunchKernelGGL(trans_gather_kernel<decltype(NT)::value>, dim3(move_blocks(a, n), s.G, n), dim3(256), 0, st, expert_dest, pool_version, slot_expert,
                           slot_version, pool_version == nullptr ? slot_expert : nullptr, a, s.E, s.self);
        return hipGetLastError();
    });
}

hipError_t launch_trans_commit(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* pool_version,
                               int32_t* slot_expert, int32_t* slot_version, hipStream_t st)
{
    if (pool_version == nullptr) return hipSuccess;        // the gather has
    hipLaunchKernelGGL(trans_commit_kernel, dim3(s.G), dim3(64), 0, st, expert_dest, pool_version, slot_expert,
                       slot_version, s.E, s.self);
    return hipGetLastError();
}
