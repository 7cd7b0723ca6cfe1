// Expert FFN forward and backward in fp32 (Section 4.2 of the paper, FEC / BEC) on the fp32 matrix cores, for the
// single-precision workloads and their 1e-5 tolerance.  Groups are ragged and may be empty; any h, d a multiple of 4.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s at the nominal clock).  Every contraction is v_mfma_f32_32x32x2_f32
// on operands staged through LDS, 32 or 64 steps deep, the next slice requested into registers while the current one
// is multiplied (one barrier per slice, two LDS buffers).  An operand whose contraction index is contiguous in memory
// (token rows, the weights of the backward contractions) lies row-major in LDS and is read four steps at a time; one
// whose contraction index is the slow one (the weights of the forward contractions, both operands of the weight
// gradients) lies as it does in memory and is read a step at a time, 32 consecutive columns per read.  The half of a
// wave that holds step 8 s + j of an instruction's pair holds 8 s + 4 + j in the other half, so that both layouts feed
// the same order.
// Tiles: 64 x 64 per block of four waves, or 32 x 32 with the four waves sharing the contraction where those are too
// few to fill the chip (small configurations, whose time is the length of the serial chain; see medium_tiles).
// Measured at T = 3000, d = 512, h = 2048, k = 2, GELU, 4900 hosted rows: forward and backward 4255 us with one output
// per thread on the vector ALUs, 680 us now (91 TFLOP/s); the tiny configuration (T = 512, d = 64, h = 256): forward 18 us,
// 12 us now.
#include "internal.h"
#include <initializer_list>

namespace {

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.3989422804014327f * expf(-0.5f * z * z);
}
__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + expf(-z)); }

typedef __attribute__((ext_vector_type(16))) float f32x16;

enum Mode { FWD1 = 0, FWD2 = 1, BWD1 = 2, BWD2 = 3, WGRAD = 4 };

struct F32Args {
    const int32_t *slot_offsets, *dest_slots;
    int self, Gcap, act, d, h;
    const float *Xp, *W1, *W2, *W3, *dYp, *Zc, *Uc, *Actc, *dZc, *dUc;
    float *Yp, *Z, *U, *Act, *dZ, *dU, *dXp, *dW1, *dW2, *dW3;
    int accumulate;
};

constexpr int F32_THREADS = 256;

// The four waves of a block cover WM x WN x WK (rows, columns, contraction) with 32 x 32 outputs each.
template <int WM_, int WN_, int WK_, int BK_> struct Tile {
    static constexpr int WM = WM_, WN = WN_, WK = WK_, BK = BK_;
    static constexpr int BM = 32 * WM, BN = 32 * WN;
    static constexpr int KW = BK / WK;                     // contraction steps of a slice one wave multiplies
    static_assert(WM * WN * WK == 4 && KW % 8 == 0, "four waves, whole groups of eight steps");
};
typedef Tile<2, 2, 1, 32> TileM;
typedef Tile<1, 1, 4, 64> TileS;

// One operand slice: ROWS rows (or columns of the output) by BK steps.  KC: the contraction index is contiguous.
// LDS pitches: 16-byte reads of 8 consecutive rows (KC) and 4-byte reads of steps 4 apart (not KC) meet all banks.
template <int ROWS, int BK, bool KC> struct Slice {
    static constexpr int PITCH = KC ? BK + 4 : ROWS + 8;
    static constexpr int FLOATS = KC ? ROWS * PITCH : BK * PITCH;
    static constexpr int N4 = ROWS * BK / 4 / F32_THREADS;
    static_assert(ROWS * BK % (4 * F32_THREADS) == 0, "whole 16-byte pieces per thread");
    // p: element (row 0, step 0); ld: leading dimension; n_rows, n_k: what exists from there (the rest is zero)
    template <bool VEC>
    static __device__ __forceinline__ void load(float4 (&r)[N4], const float* p, long ld, int n_rows, int n_k)
    {
#pragma unroll
        for (int i = 0; i < N4; ++i) {
            const int it = i * F32_THREADS + (int)threadIdx.x;
            const int major = it / (KC ? BK / 4 : ROWS / 4), minor = it % (KC ? BK / 4 : ROWS / 4) * 4;
            const int nmaj = KC ? n_rows : n_k, nmin = KC ? n_k : n_rows;
            const float* q = p + (long)major * ld + minor;
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (VEC) {                                     // nmin is a multiple of 4: a piece exists or does not
                if (major < nmaj && minor < nmin) v = *reinterpret_cast<const float4*>(q);
            } else if (major < nmaj) {
                if (minor + 0 < nmin) v.x = q[0];
                if (minor + 1 < nmin) v.y = q[1];
                if (minor + 2 < nmin) v.z = q[2];
                if (minor + 3 < nmin) v.w = q[3];
            }
            r[i] = v;
        }
    }
    static __device__ __forceinline__ void store(float* s, const float4 (&r)[N4])
    {
#pragma unroll
        for (int i = 0; i < N4; ++i) {
            const int it = i * F32_THREADS + (int)threadIdx.x;
            const int major = it / (KC ? BK / 4 : ROWS / 4), minor = it % (KC ? BK / 4 : ROWS / 4) * 4;
            *reinterpret_cast<float4*>(s + major * PITCH + minor) = r[i];
        }
    }
    // four steps k8 + 4 (lane / 32) .. + 3 of row `row`
    static __device__ __forceinline__ void frag(float (&f)[4], const float* s, int row, int k)
    {
        if (KC) {
            const float4 v = *reinterpret_cast<const float4*>(s + row * PITCH + k);
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = s[(k + j) * PITCH + row];
        }
    }
};

// An operand of a contraction: element (0, 0), leading dimension, rows that exist.
struct Operand { const float* p; long ld; int n; };

// acc = sum over K of A(m, k) B(k, n), acc2 the same with B2 (DUAL), or, without DUAL, acc over a second segment of
// the contraction (n_seg = 2: A2, B2 over another K steps).
template <class TL, bool AKC, bool BKC, bool DUAL, bool VEC>
__device__ __forceinline__ void contract(f32x16& acc, f32x16& acc2, float* lds, Operand A, Operand B,
                                         Operand A2, Operand B2, int n_seg, int K)
{
    typedef Slice<TL::BM, TL::BK, AKC> SA;
    typedef Slice<TL::BN, TL::BK, BKC> SB;
    constexpr int BUF = SA::FLOATS + (DUAL ? 2 : 1) * SB::FLOATS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wk = wave % TL::WK, wn = (wave / TL::WK) % TL::WN, wm = wave / (TL::WK * TL::WN);
    const int l32 = lane & 31, kh = 4 * (lane >> 5);
#pragma unroll
    for (int e = 0; e < 16; ++e) { acc[e] = 0.0f; acc2[e] = 0.0f; }
    const int per = (K + TL::BK - 1) / TL::BK, ns = n_seg * per;
    if (ns == 0) return;
    float4 ra[SA::N4], rb[SB::N4], rb2[DUAL ? SB::N4 : 1];
    auto request = [&](int s) {
        const bool second = s >= per;
        const int k0 = (second ? s - per : s) * TL::BK;
        const Operand a = second ? A2 : A, b = second ? B2 : B;
        SA::template load<VEC>(ra, a.p + (AKC ? (long)k0 : (long)k0 * a.ld), a.ld, a.n, K - k0);
        SB::template load<VEC>(rb, b.p + (BKC ? (long)k0 : (long)k0 * b.ld), b.ld, b.n, K - k0);
        if constexpr (DUAL) SB::template load<VEC>(rb2, B2.p + (BKC ? (long)k0 : (long)k0 * B2.ld), B2.ld, B2.n, K - k0);
    };
    auto keep = [&](float* buf) {
        SA::store(buf, ra);
        SB::store(buf + SA::FLOATS, rb);
        if constexpr (DUAL) SB::store(buf + SA::FLOATS + SB::FLOATS, rb2);
    };
    request(0);
    keep(lds);
    __syncthreads();
    for (int s = 0; s < ns; ++s) {
        if (s + 1 < ns) request(s + 1);
        const float* sa = lds + (s & 1) * BUF;
        const float* sb = sa + SA::FLOATS;
#pragma unroll
        for (int k8 = 0; k8 < TL::KW; k8 += 8) {
            const int k = wk * TL::KW + k8 + kh;
            float a[4], b[4], b2[4];
            SA::frag(a, sa, wm * 32 + l32, k);
            SB::frag(b, sb, wn * 32 + l32, k);
            if constexpr (DUAL) SB::frag(b2, sb + SB::FLOATS, wn * 32 + l32, k);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], acc, 0, 0, 0);
                if constexpr (DUAL) acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b2[q], acc2, 0, 0, 0);
            }
        }
        if (s + 1 < ns) keep(lds + ((s + 1) & 1) * BUF);   // the buffer of slice s - 1, which everybody has left
        __syncthreads();
    }
}

// Calls out(m, n, acc, acc2) for every element of the tile (m, n inside the tile).  Waves that shared the contraction
// hand their sums over through LDS, added in wave order.
template <class TL, bool DUAL, typename OUT>
__device__ __forceinline__ void for_each_output(f32x16& acc, f32x16& acc2, float* lds, OUT out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wn = (wave / TL::WK) % TL::WN, wm = wave / (TL::WK * TL::WN);
    const int l32 = lane & 31, kh = 4 * (lane >> 5);
    if constexpr (TL::WK == 1) {
#pragma unroll
        for (int e = 0; e < 16; ++e) out(wm * 32 + 8 * (e >> 2) + kh + (e & 3), wn * 32 + l32, acc[e], acc2[e]);
    } else {
        static_assert(TL::WK == 1 || TL::WK == 4, "one tile, four parts of its contraction");
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            lds[(wave * 16 + e) * 64 + lane] = acc[e];
            if constexpr (DUAL) lds[4096 + (wave * 16 + e) * 64 + lane] = acc2[e];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = wave * 4 + q;
            float v = 0.0f, v2 = 0.0f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                v += lds[(w * 16 + e) * 64 + lane];
                if constexpr (DUAL) v2 += lds[4096 + (w * 16 + e) * 64 + lane];
            }
            out(8 * wave + kh + q, l32, v, v2);
        }
    }
}

template <class TL, bool AKC, bool BKC, bool DUAL> constexpr int lds_floats()
{
    constexpr int ring = 2 * (Slice<TL::BM, TL::BK, AKC>::FLOATS + (DUAL ? 2 : 1) * Slice<TL::BN, TL::BK, BKC>::FLOATS);
    constexpr int fold = TL::WK == 1 ? 0 : (DUAL ? 8192 : 4096);
    return ring > fold ? ring : fold;
}

// Row tile `rt` of the hosted rows: its group and first row inside the group; false past the last one.  G <= E <= 1024.
__device__ __forceinline__ bool find_row_tile(const F32Args& a, int rt, int bm, int& g, int& first_row, int& row0, int& rows)
{
    int first, ng;
    hosted_range(a.dest_slots, a.self, a.Gcap, first, ng);
    const int lane = threadIdx.x & 63;
    int before = 0;
    for (int g0 = 0; g0 < ng; g0 += 64) {
        int r0 = 0, n = 0;
        if (g0 + lane < ng) {
            r0 = a.slot_offsets[first + g0 + lane];
            n = a.slot_offsets[first + g0 + lane + 1] - r0;
        }
        const int nt = (n + bm - 1) / bm;
        int incl = nt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        const unsigned long long past = __ballot(before + incl > rt);
        if (past) {
            const int l = __ffsll((long long)past) - 1;
            g = g0 + l;
            row0 = __shfl(r0, l, 64);
            rows = __shfl(n, l, 64);
            first_row = (rt - before - (__shfl(incl, l, 64) - __shfl(nt, l, 64))) * bm;
            return true;
        }
        before += __shfl(incl, 63, 64);
    }
    return false;
}

// grid: column tiles x row tiles (an upper bound), so that the columns of a row tile run next to each other.  (Two axes: a
// grid has fewer than 2^32 threads along each, and wide layers of many groups need more in all.)
template <int MODE, class TL, bool DUAL, bool VEC>
__global__ __launch_bounds__(F32_THREADS) void ffn_f32_kernel(F32Args a)
{
    constexpr bool BKC = (MODE == BWD1 || MODE == BWD2);
    __shared__ __attribute__((aligned(16))) float lds[lds_floats<TL, true, BKC, DUAL>()];
    int g, first_row, row0, rows;
    if (!find_row_tile(a, blockIdx.y, TL::BM, g, first_row, row0, rows)) return;
    const int d = a.d, h = a.h, n0 = blockIdx.x * TL::BN, nr = rows - first_row;
    const bool swiglu = a.act == MOE_ACT_SWIGLU;
    const long r0 = (long)row0 + first_row, wdh = (long)g * d * h;
    f32x16 acc, acc2;
    if (MODE == FWD1) {
        const Operand A{a.Xp + r0 * d, d, nr}, B{a.W1 + wdh + n0, h, h - n0}, B2{DUAL ? a.W3 + wdh + n0 : nullptr, h, h - n0};
        contract<TL, true, BKC, DUAL, VEC>(acc, acc2, lds, A, B, A, B2, 1, d);
        for_each_output<TL, DUAL>(acc, acc2, lds, [&](int m, int n, float z, float u) {
            if (m >= nr || n0 + n >= h) return;
            const long o = (r0 + m) * h + n0 + n;
            if (a.Z) a.Z[o] = z;                            // forward only: the pre-activations are not kept
            if (DUAL) { if (a.U) a.U[o] = u; a.Act[o] = z * sigmoid_f(z) * u; }
            else a.Act[o] = gelu_f(z);
        });
    } else if (MODE == FWD2) {
        const Operand A{a.Actc + r0 * h, h, nr}, B{a.W2 + wdh + n0, d, d - n0};
        contract<TL, true, BKC, false, VEC>(acc, acc2, lds, A, B, A, B, 1, h);
        for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float y, float) {
            if (m < nr && n0 + n < d) a.Yp[(r0 + m) * d + n0 + n] = y;
        });
    } else if (MODE == BWD1) {                              // dA[m, n] = sum_c dYp[m, c] W2[n, c]
        const Operand A{a.dYp + r0 * d, d, nr}, B{a.W2 + wdh + (long)n0 * d, d, h - n0};
        contract<TL, true, BKC, false, VEC>(acc, acc2, lds, A, B, A, B, 1, d);
        for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float v, float) {
            if (m >= nr || n0 + n >= h) return;
            const long o = (r0 + m) * h + n0 + n;
            const float z = a.Zc[o];
            if (swiglu) {
                const float u = a.Uc[o], s = sigmoid_f(z);
                a.dU[o] = v * z * s;
                a.dZ[o] = v * u * s * (1.0f + z * (1.0f - s));
                a.Act[o] = z * s * u;
            } else {
                a.dZ[o] = v * gelu_grad_f(z);
                a.Act[o] = gelu_f(z);
            }
        });
    } else {                                                // dXp[m, n] = sum_j dZ[m, j] W1[n, j] (+ dU[m, j] W3[n, j])
        const Operand A{a.dZc + r0 * h, h, nr}, B{a.W1 + wdh + (long)n0 * h, h, d - n0};
        const Operand A2 = swiglu ? Operand{a.dUc + r0 * h, h, nr} : A, B2 = swiglu ? Operand{a.W3 + wdh + (long)n0 * h, h, d - n0} : B;
        contract<TL, true, BKC, false, VEC>(acc, acc2, lds, A, B, A2, B2, swiglu ? 2 : 1, h);
        for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float v, float) {
            if (m < nr && n0 + n < d) a.dXp[(r0 + m) * d + n0 + n] = v;
        });
    }
}

// Weight gradients, all products of all groups in one launch: out[m, n] = sum over the group's rows r of L[r, m] R[r, n]
// (dW1 = Xp^T dZ, dW2 = Act^T dYp, dW3 = Xp^T dU).  grid: tiles of a product x (products of group 0, of group 1, ...).
template <class TL, bool VEC>
__global__ __launch_bounds__(F32_THREADS) void ffn_f32_wgrad_kernel(F32Args a, int n_products)
{
    __shared__ __attribute__((aligned(16))) float lds[lds_floats<TL, false, false, false>()];
    const int g = blockIdx.y / n_products, which = blockIdx.y % n_products, tile = blockIdx.x;
    int first, ng;
    hosted_range(a.dest_slots, a.self, a.Gcap, first, ng);
    int row0 = 0, rows = 0;
    if (g < ng) { row0 = a.slot_offsets[first + g]; rows = a.slot_offsets[first + g + 1] - row0; }
    const int Mo = which == 1 ? a.h : a.d, No = which == 1 ? a.d : a.h;
    // the tile counts of d x h and h x d are the same; walk the product's own grid
    const int ctiles = (No + TL::BN - 1) / TL::BN;
    const int m0 = tile / ctiles * TL::BM, n0 = tile % ctiles * TL::BN;
    const float* L = which == 1 ? a.Actc : a.Xp;
    const float* R = which == 0 ? a.dZc : (which == 1 ? a.dYp : a.dUc);
    const Operand A{L + (long)row0 * Mo + m0, Mo, Mo - m0}, B{R + (long)row0 * No + n0, No, No - n0};
    f32x16 acc, acc2;
    contract<TL, false, false, false, VEC>(acc, acc2, lds, A, B, A, B, 1, rows);
    float* dst = (which == 0 ? a.dW1 : (which == 1 ? a.dW2 : a.dW3)) + (long)g * a.d * a.h;
    for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float v, float) {
        if (m0 + m >= Mo || n0 + n >= No) return;
        float* p = dst + (long)(m0 + m) * No + n0 + n;
        *p = a.accumulate ? *p + v : v;
    });
}

F32Args make_args(const moe_shape_t& s, const ffn_args& a)
{
    F32Args f{};
    f.slot_offsets = a.slot_offsets; f.dest_slots = a.dest_slots;
    f.self = s.self; f.Gcap = s.G; f.act = (int)s.act; f.d = s.d; f.h = s.h;
    f.Xp = (const float*)a.Xp; f.W1 = (const float*)a.W1; f.W2 = (const float*)a.W2; f.W3 = (const float*)a.W3;
    f.dYp = (const float*)a.dYp;
    f.Zc = (const float*)a.Z; f.Uc = (const float*)a.U; f.Actc = (const float*)a.Act;
    f.dZc = (const float*)a.dZ; f.dUc = (const float*)a.dU;
    f.Yp = (float*)a.Yp; f.Z = (float*)a.Z; f.U = (float*)a.U; f.Act = (float*)a.Act;
    f.dZ = (float*)a.dZ; f.dU = (float*)a.dU; f.dXp = (float*)a.dXp;
    f.dW1 = a.dW1; f.dW2 = a.dW2; f.dW3 = a.dW3;
    f.accumulate = a.accumulate ? 1 : 0;
    return f;
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// 16-byte loads need every row of every operand 16-byte aligned: d is a multiple of 4 (moe_create), h and the pointers
// are looked at here; anything else takes 4-byte loads.
bool vec_ok(const moe_shape_t& s, std::initializer_list<const void*> ps)
{
    uintptr_t bits = 0;
    for (const void* p : ps) bits |= reinterpret_cast<uintptr_t>(p);
    return s.h % 4 == 0 && (bits & 15) == 0;
}

// 64 x 64 tiles where there are enough of them (rows: all T * k of them, of which a part is hosted here).  Forward and
// backward of the two contractions, us, 32 x 32 against 64 x 64: 512 and 128 tiles (T = 1000, d = 256, h = 1024, k = 2)
// 38 + 67 against 48 + 82; 3008 and 752 tiles (T = 3000, d = 512, h = 2048) 245 + 471 against 229 + 447; 6000 and 2000
// tiles (T = 4000, d = 1024, h = 3072) 877 + 1732 against 768 + 1513.  128 x 128 was the slower one everywhere (287 + 545,
// 799 + 1626 on the latter two: fewer blocks to hide a load behind, a longer last round).
bool medium_tiles(long rows, long cols) { return ((rows + 63) / 64) * ((cols + 63) / 64) >= 700; }

template <int MODE, class TL, bool DUAL>
void launch_rows_t(const moe_shape_t& s, const F32Args& f, int N, bool vec, hipStream_t st)
{
    const int ct = cdiv(N, TL::BN), rt = cdiv(s.T * s.k, TL::BM) + s.G;
    if (vec) hipLaunchKernelGGL((ffn_f32_kernel<MODE, TL, DUAL, true>), dim3(ct, rt), dim3(F32_THREADS), 0, st, f);
    else hipLaunchKernelGGL((ffn_f32_kernel<MODE, TL, DUAL, false>), dim3(ct, rt), dim3(F32_THREADS), 0, st, f);
}

template <int MODE, bool DUAL>
hipError_t launch_rows(const moe_shape_t& s, const F32Args& f, int N, bool vec, hipStream_t st)
{
    if (medium_tiles((long)s.T * s.k, N)) launch_rows_t<MODE, TileM, DUAL>(s, f, N, vec, st);
    else launch_rows_t<MODE, TileS, DUAL>(s, f, N, vec, st);
    return hipGetLastError();
}

template <class TL>
hipError_t launch_wgrad(const moe_shape_t& s, const F32Args& f, bool vec, hipStream_t st)
{
    const int tiles = cdiv(s.d, TL::BM) * cdiv(s.h, TL::BN), np = s.act == MOE_ACT_SWIGLU ? 3 : 2;
    static_assert(TL::BM == TL::BN, "d x h and h x d have the same number of tiles");
    const dim3 grid(tiles, np * s.G);
    if (vec) hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, true>), grid, dim3(F32_THREADS), 0, st, f, np);
    else hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, false>), grid, dim3(F32_THREADS), 0, st, f, np);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_fwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const F32Args f = make_args(s, a);
    const bool vec = vec_ok(s, {a.Xp, a.W1, a.W2, a.W3, a.Act});
    hipError_t e = s.act == MOE_ACT_SWIGLU ? launch_rows<FWD1, true>(s, f, s.h, vec, st) : launch_rows<FWD1, false>(s, f, s.h, vec, st);
    if (e == hipSuccess) e = launch_rows<FWD2, false>(s, f, s.d, vec, st);
    return e;
}

hipError_t launch_ffn_bwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const F32Args f = make_args(s, a);
    const bool vec = vec_ok(s, {a.dYp, a.Xp, a.W1, a.W2, a.W3, a.Act, a.dZ, a.dU});
    hipError_t e = launch_rows<BWD1, false>(s, f, s.h, vec, st);
    if (e == hipSuccess) e = launch_rows<BWD2, false>(s, f, s.d, vec, st);
    if (e != hipSuccess) return e;
    const int np = s.act == MOE_ACT_SWIGLU ? 3 : 2;
    return medium_tiles((long)s.d * np, (long)s.h * s.G) ? launch_wgrad<TileM>(s, f, vec, st) : launch_wgrad<TileS>(s, f, vec, st);
}
