// Expert FFN forward and backward in fp32 (Section 4.2 of the paper, FEC / BEC) on the fp32 matrix cores, for the
// single-precision workloads and their 1e-5 tolerance.  Groups are ragged and may be empty; any h, d a multiple of 4.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s at the nominal clock).  Every contraction is v_mfma_f32_32x32x2_f32
// on operands staged through LDS, 32 or 64 steps deep, the next slice requested while the current one is multiplied (one
// barrier per slice); requests go straight into LDS.  An operand whose contraction index is contiguous in memory
// (token rows, the weights of the backward contractions) lies row-major in LDS and is read four steps at a time; one
// whose contraction index is the slow one (the weights of the forward contractions, both operands of the weight
// gradients) lies as it does in memory and is read a step at a time, 32 consecutive columns per read.  The half of a
// wave that holds step 8 s + j of an instruction's pair holds 8 s + 4 + j in the other half, so that both layouts feed
// the same order.
// Tiles: 64 x 64 per block of four waves, 64 x 32 or 32 x 32 with two or four waves sharing the contraction where those are
// too few to fill the chip (see MEDIUM_TILES).
// Measured at T = 3000, d = 512, h = 2048, k = 2, GELU, 4900 hosted rows, forward and backward: 4255 us with one output
// per thread on the vector ALUs, 703 us staged through registers, 578 us now (107 TFLOP/s); the weight gradients of it 249,
// 212 with the requests straight into LDS, 193 with the longest groups first.
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
template <int WM_, int WN_, int WK_, int BK_, int STAGES_ = 2> struct Tile {
    static constexpr int WM = WM_, WN = WN_, WK = WK_, BK = BK_;
    static constexpr int BM = 32 * WM, BN = 32 * WN;
    static constexpr int KW = BK / WK;                     // contraction steps of a slice one wave multiplies
    static constexpr int STAGES = STAGES_;                 // LDS buffers of a block
    static_assert(WM * WN * WK == 4 && KW % 8 == 0, "four waves, whole groups of eight steps");
};
typedef Tile<2, 2, 1, 32> TileM;
typedef Tile<2, 1, 2, 64> TileH;                          // half a TileM: slices of 32 steps took 10 us more of its 110
typedef Tile<1, 1, 4, 64> TileS;
typedef Tile<1, 1, 4, 64, 4> TileF;                       // few of them

typedef __attribute__((ext_vector_type(4))) int rsrc_t;     // raw buffer resource (4 scalar registers)
constexpr uint32_t NOWHERE = 0xfffffffcu;                   // an offset past the end of every resource
__device__ __forceinline__ rsrc_t make_rsrc(const float* base, long bytes)
{
    const unsigned long long b = (unsigned long long)base;
    const unsigned n = bytes < 0 ? 0u : (bytes > 0xfffffff0l ? 0xfffffff0u : (unsigned)bytes);
    rsrc_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)b);
    r[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(b >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)n);          // bytes past this limit read as zero
    r[3] = 0x00020000;
    return r;
}
// V floats per lane straight into LDS at lds_base + 4 V lane (lds_base is uniform).  As assembly, so that the compiler
// does not wait for the request before it reads another buffer; complete after WAIT_REQUESTS.
template <int V> __device__ __forceinline__ void request_lds(rsrc_t r, uint32_t lds_base, uint32_t voff)
{
    if (V == 4) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds_base), "v"(voff), "s"(r) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" :: "s"(lds_base), "v"(voff), "s"(r) : "memory");
}
#define WAIT_REQUESTS(n) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(n) : "memory")

// An operand slice as buffer loads leave it in LDS, ROWS rows (or columns of the output) by BK steps without padding.  KC:
// the contraction index is contiguous.  V: floats per lane and request, 4 where rows of the operand begin at multiples of 16
// bytes, else 1.  KC: 16-byte piece p of a row is kept at p ^ swizzle(row), 16 consecutive rows of one piece cover all banks.
// Not KC: the two halves of a wave read steps 4 apart of the same 32 columns; the upper half's columns are swapped (64
// columns: a row is all banks), or its steps lie between those of the lower half (32 columns: a row is half of them).
template <int ROWS, int BK, bool KC, int V_> struct Slice {
    static constexpr int V = V_ ? V_ : 1;
    static constexpr int BYTES = ROWS * BK * 4;
    static constexpr int REQUEST = 256 * V;                // bytes of a request
    static constexpr int N = BYTES / REQUEST / 4;          // requests per wave
    static constexpr int ROW = KC ? BK : ROWS;             // floats per row of the buffer
    static constexpr int N_ADDR = KC ? BK / 8 : 1;         // address registers of the fragments of a slice
    static_assert(BYTES % (4 * REQUEST) == 0 && (ROWS == 32 || ROWS == 64) && (BK == 32 || BK == 64) && (V == 1 || V == 4), "whole requests");
    static __device__ __forceinline__ int swizzle(int row) { return ROW == 32 ? (row >> 1) & 7 : row & 15; }
    // what lane `lane` of request i of wave w delivers: its row (not KC: step) and its place in it
    static __device__ __forceinline__ void place(int i, int w, int lane, int& major, int& minor)
    {
        const int f = ((i * 4 + w) * 64 + lane) * V, r = f / ROW, c = f % ROW;
        if (KC) { major = r; minor = c ^ (swizzle(r) << 2); }
        else if (ROWS == 64) { major = r; minor = c ^ (32 * ((r >> 2) & 1)); }
        else { major = (r & ~7) + 4 * (r & 1) + ((r >> 1) & 3); minor = c; }
    }
    // its byte offset from element (row 0, step 0) of the slice
    static __device__ __forceinline__ uint32_t source(int i, int w, int lane, int ld)
    {
        int major, minor;
        place(i, w, lane, major, minor);
        return ((uint32_t)major * (uint32_t)ld + (uint32_t)minor) * 4u;
    }
    // and whether it lies past the n steps that are left of the contraction (not KC: those lie past the resource's end)
    static __device__ __forceinline__ bool past(int i, int w, int lane, int n)
    {
        int major, minor;
        place(i, w, lane, major, minor);
        return KC && minor >= n;
    }
    // V_ = 0: requests of a wave for a slice whose rows are too far apart for an offset, from element (row 0, step 0) on (n_rows
    // rows or columns, n_k steps exist).  A row of the buffer is 64 or 32 floats, so a request is one row with a resource of its
    // own, or two, 4 apart, half a wave each: from one resource where an offset reaches 4 rows, else asked for one after the other.
    // (Few scalar instructions per request: a wave of a long contraction has nothing else to hide them behind.)
    static __device__ __forceinline__ void request_far(uint32_t dst, const float* p, long ld, int n_rows, int n_k, int w, int lane)
    {
        static_assert(ROW == 64 || !KC, "a row of 32 floats lies as in memory");
        constexpr int HALVES = 64 / ROW;
        const int n_major = KC ? n_rows : n_k, bytes = min(KC ? n_k : n_rows, ROW) * 4;
        const bool all = n_major >= 4 * HALVES * N;
        if (HALVES == 1 || ld < (1l << 28) - 64) {
            if (all) far_rows<true, HALVES, HALVES == 2>(dst, p, ld, 0, n_major, bytes, w, lane);
            else far_rows<false, HALVES, HALVES == 2>(dst, p, ld, 0, n_major, bytes, w, lane);
        } else {
            if (lane < 32) far_rows<false, HALVES, false>(dst, p, ld, 0, n_major, bytes, w, lane);
            else far_rows<false, HALVES, false>(dst, p, ld, 4, n_major, bytes, w, lane);
        }
    }
    // place(): request i brings the rows (steps) 4 HALVES i + w + from and, for two, the one 4 further
    template <bool ALL, int HALVES, bool TWO>
    static __device__ __forceinline__ void far_rows(uint32_t dst, const float* p, long ld, int from, int n_major, int bytes, int w, int lane)
    {
        const uint32_t two = TWO ? (uint32_t)(16 * ld) : 0;
        rsrc_t row = make_rsrc(p + (w + from) * ld, (long)two + bytes);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            int major, minor;
            place(i, w, lane, major, minor);
            const int r = 4 * HALVES * i + w + from;
            if (!ALL) row[2] = r < n_major ? (int)(r + 4 < n_major ? two + bytes : bytes) : 0;
            request_lds<1>(row, dst + i * 1024, minor * 4 + (TWO && lane >= 32 ? two : 0));
            const unsigned long long next = ((unsigned long long)(unsigned)row[1] << 32 | (unsigned)row[0]) + 16ull * HALVES * ld;
            row[0] = (int)(unsigned)next;
            row[1] = (int)(unsigned)(next >> 32);
        }
    }
    // byte addresses in a buffer of row `row`, steps k0 + 4 hi (k0 a multiple of 8, the wave's first): KC one for each 8
    // steps from there, else one, the others at a constant distance
    static __device__ __forceinline__ uint32_t address(int row, int k0, int hi, int n)
    {
        if (KC) return row * (BK * 4) + (((k0 / 4 + 2 * n + hi) ^ swizzle(row)) << 4);
        if (ROWS == 64) return k0 * 256 + hi * 1024 + ((row ^ (32 * hi)) * 4);
        return k0 * 128 + hi * 128 + row * 4;
    }
    // four steps of the fragments at 8 n steps past the wave's first
    static __device__ __forceinline__ void frag(float (&f)[4], const unsigned char* buf, const uint32_t (&addr)[N_ADDR], int n)
    {
        if (KC) {
            const float4 v = *reinterpret_cast<const float4*>(buf + addr[n]);
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                f[j] = *reinterpret_cast<const float*>(buf + addr[0] + (ROWS == 64 ? n * 2048 + j * 256 : n * 1024 + j * 256));
        }
    }
};

// An operand of a contraction: element (0, 0), leading dimension, rows that exist.
struct Operand { const float* p; long ld; int n; };

// acc = sum over K of A(m, k) B(k, n), acc2 the same with B2 (DUAL), or, without DUAL, acc over a second segment of
// the contraction (n_seg = 2: A2, B2 over another K steps).  VA, VB: floats per request, 4 where the operand's pointer, its
// leading dimension and, if its contraction index is contiguous, K are whole 16-byte pieces; 0 (requests of one float) where the
// rows of a slice are too far apart for a 32-bit offset.
// Slices go from memory straight into a ring of LDS buffers while an earlier one is multiplied (two; four of the 32 x 32
// tile where there are few of them, whose products don't cover a request).  On a SIMD a vector instruction of any wave takes about 8 cycles
// from its matrix instructions, so the loop has next to none: the addresses of requests and fragments are fixed, what
// moves is the resource's base, and what does not exist lies past the resource's end and arrives as zeros.  With the slices
// staged through registers (predicated loads, LDS stores, 64 vector instructions per 16 products) the five launches of T =
// 3000, d = 512, h = 2048, k = 2 took 131, 138, 154, 134 and 249 us, now 117, 121, 135, 124 and 212 in the same tiles and order.
template <class TL, bool AKC, bool BKC, bool DUAL, int VA, int VB>
__device__ __forceinline__ void contract(f32x16& acc, f32x16& acc2, float* lds_f, Operand A, Operand B, Operand A2, Operand B2, int n_seg, int K)
{
    typedef Slice<TL::BM, TL::BK, AKC, VA> SA;
    typedef Slice<TL::BN, TL::BK, BKC, VB> SB;
    static_assert((VA == 0) == (VB == 0), "both operands");
    constexpr bool FAR = VA == 0;
    constexpr int BUF = SA::BYTES + (DUAL ? 2 : 1) * SB::BYTES, BK = TL::BK;
    unsigned char* lds = reinterpret_cast<unsigned char*>(lds_f);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave % TL::WK, wn = (wave / TL::WK) % TL::WN, wm = wave / (TL::WK * TL::WN);
    const int l32 = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int e = 0; e < 16; ++e) { acc[e] = 0.0f; acc2[e] = 0.0f; }
    // Where two waves share a contraction, every second group of eight steps goes into sums of its own: chains as long as with
    // four waves (error of a contraction of 3000 steps against 64 bits 6.9e-7 without, 4.9e-7 with them; no time).
    constexpr bool TWICE = TL::WK == 2;
    f32x16 odd{}, odd2{};
    const int per = (K + BK - 1) / BK, ns = n_seg * per;
    if (ns == 0) return;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)lds_f;
    uint32_t va[SA::N], vb[SB::N];                         // A2 and B2 have the leading dimensions of A and B
#pragma unroll
    for (int i = 0; i < SA::N; ++i) va[i] = SA::source(i, wave, lane, A.ld);
#pragma unroll
    for (int i = 0; i < SB::N; ++i) vb[i] = SB::source(i, wave, lane, B.ld);
    uint32_t fa[SA::N_ADDR], fb[SB::N_ADDR];
#pragma unroll
    for (int n = 0; n < SA::N_ADDR; ++n) fa[n] = SA::address(wm * 32 + l32, wk * TL::KW, hi, n);
#pragma unroll
    for (int n = 0; n < SB::N_ADDR; ++n) fb[n] = SA::BYTES + SB::address(wn * 32 + l32, wk * TL::KW, hi, n);
    // KC: the tile's rows, from step k0 on; else the steps from k0 on, all columns
    auto rsrc = [&](bool kc, int rows, const Operand& o, int k0) {
        const long n = kc ? (long)(o.n < rows ? o.n : rows) * o.ld - k0 : (long)(K - k0) * o.ld - (o.ld - o.n);
        return make_rsrc(o.p + (kc ? (long)k0 : (long)k0 * o.ld), n * 4);
    };
    auto request = [&](int s) {
        const bool second = s >= per;
        const int k0 = (second ? s - per : s) * BK, left = K - k0;
        const Operand a = second ? A2 : A, b = second ? B2 : B;
        if constexpr (FAR) {
            const uint32_t to = lds0 + s % TL::STAGES * BUF + wave * 256;
            SA::request_far(to, a.p + (AKC ? (long)k0 : (long)k0 * a.ld), a.ld, a.n, left, wave, lane);
            SB::request_far(to + SA::BYTES, b.p + (BKC ? (long)k0 : (long)k0 * b.ld), b.ld, b.n, left, wave, lane);
            if constexpr (DUAL) SB::request_far(to + SA::BYTES + SB::BYTES, B2.p + (BKC ? (long)k0 : (long)k0 * B2.ld), B2.ld, B2.n, left, wave, lane);
            return;
        }
        const rsrc_t ra = rsrc(AKC, TL::BM, a, k0), rb = rsrc(BKC, TL::BN, b, k0);
        const uint32_t dst = lds0 + s % TL::STAGES * BUF, da = dst + wave * SA::REQUEST, db = dst + SA::BYTES + wave * SB::REQUEST;
        if ((AKC || BKC) && left < BK) {                   // past the contraction lies the next row, not the end
#pragma unroll
            for (int i = 0; i < SA::N; ++i) request_lds<VA>(ra, da + i * 4 * SA::REQUEST, SA::past(i, wave, lane, left) ? NOWHERE : va[i]);
#pragma unroll
            for (int i = 0; i < SB::N; ++i) request_lds<VB>(rb, db + i * 4 * SB::REQUEST, SB::past(i, wave, lane, left) ? NOWHERE : vb[i]);
        } else {
#pragma unroll
            for (int i = 0; i < SA::N; ++i) request_lds<VA>(ra, da + i * 4 * SA::REQUEST, va[i]);
#pragma unroll
            for (int i = 0; i < SB::N; ++i) request_lds<VB>(rb, db + i * 4 * SB::REQUEST, vb[i]);
        }
        if constexpr (DUAL) {
            static_assert(!DUAL || !BKC, "the second matrix ends with its steps");
            const rsrc_t rb2 = rsrc(BKC, TL::BN, B2, k0);
#pragma unroll
            for (int i = 0; i < SB::N; ++i) request_lds<VB>(rb2, db + SB::BYTES + i * 4 * SB::REQUEST, vb[i]);
        }
    };
    // Slice s + AHEAD is requested into the buffer of slice s - 1, which everybody has left at the barrier of slice s.
    constexpr int AHEAD = TL::STAGES - 1, OPS = SA::N + (DUAL ? 2 : 1) * SB::N;      // (FAR: or more)
    static_assert((AHEAD - 1) * OPS < 64, "what the counter of requests can say");
    for (int s = 0; s < AHEAD && s < ns; ++s) request(s);
    for (int s = 0, cur = 0; s < ns; ++s) {
        if (s + AHEAD <= ns) WAIT_REQUESTS((AHEAD - 1) * OPS);     // slice s has landed, AHEAD - 1 later ones are on their way
        else WAIT_REQUESTS(0);
        __syncthreads();
        if (s + AHEAD < ns) request(s + AHEAD);
        const unsigned char* buf = lds + cur * BUF;
        cur = cur + 1 == TL::STAGES ? 0 : cur + 1;
#pragma unroll
        for (int n = 0; n < TL::KW / 8; ++n) {
            float a[4], b[4], b2[4];
            SA::frag(a, buf, fa, n);
            SB::frag(b, buf, fb, n);
            if constexpr (DUAL) SB::frag(b2, buf + SB::BYTES, fb, n);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x16 &sum = TWICE && n % 2 ? odd : acc, &sum2 = TWICE && n % 2 ? odd2 : acc2;
                sum = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], sum, 0, 0, 0);
                if constexpr (DUAL) sum2 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b2[q], sum2, 0, 0, 0);
            }
        }
    }
    if (TWICE) { acc += odd; acc2 += odd2; }
    __syncthreads();                                       // the buffers are free
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
        constexpr int OWN = 16 / TL::WK;                   // registers a wave adds up and hands out
        const int wk = wave % TL::WK;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            lds[(wave * 16 + e) * 64 + lane] = acc[e];
            if constexpr (DUAL) lds[4096 + (wave * 16 + e) * 64 + lane] = acc2[e];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < OWN; ++q) {
            const int e = wk * OWN + q;
            float v = 0.0f, v2 = 0.0f;
#pragma unroll
            for (int w = 0; w < TL::WK; ++w) {
                v += lds[((wave - wk + w) * 16 + e) * 64 + lane];
                if constexpr (DUAL) v2 += lds[4096 + ((wave - wk + w) * 16 + e) * 64 + lane];
            }
            out(wm * 32 + 8 * (e >> 2) + kh + (e & 3), wn * 32 + l32, v, v2);
        }
    }
}

template <class TL, bool DUAL> constexpr int lds_floats()
{
    constexpr int ring = TL::STAGES * (TL::BM + (DUAL ? 2 : 1) * TL::BN) * TL::BK;
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
            row0 = __builtin_amdgcn_readlane(r0, l);
            rows = __builtin_amdgcn_readlane(n, l);
            first_row = (rt - before - (__builtin_amdgcn_readlane(incl, l) - __builtin_amdgcn_readlane(nt, l))) * bm;
            return true;
        }
        before += __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}

// grid: column tiles x row tiles (an upper bound), so that the columns of a row tile run next to each other.  (Two axes: a
// grid has fewer than 2^32 threads along each, and wide layers of many groups need more in all.)
template <int MODE, class TL, bool DUAL, int VD, int VH>
__global__ __launch_bounds__(F32_THREADS) void ffn_f32_kernel(F32Args a)
{
    constexpr bool BKC = (MODE == BWD1 || MODE == BWD2);
    __shared__ __attribute__((aligned(1024))) float lds[lds_floats<TL, DUAL>()];
    int g, first_row, row0, rows;
    if (!find_row_tile(a, blockIdx.y, TL::BM, g, first_row, row0, rows)) return;
    const int d = a.d, h = a.h, n0 = blockIdx.x * TL::BN, nr = rows - first_row;
    const bool swiglu = a.act == MOE_ACT_SWIGLU;
    const long r0 = (long)row0 + first_row, wdh = (long)g * d * h;
    f32x16 acc, acc2;
    if (MODE == FWD1) {
        const Operand A{a.Xp + r0 * d, d, nr}, B{a.W1 + wdh + n0, h, h - n0}, B2{DUAL ? a.W3 + wdh + n0 : nullptr, h, h - n0};
        contract<TL, true, BKC, DUAL, VD, VH>(acc, acc2, lds, A, B, A, B2, 1, d);
        for_each_output<TL, DUAL>(acc, acc2, lds, [&](int m, int n, float z, float u) {
            if (m >= nr || n0 + n >= h) return;
            const long o = (r0 + m) * h + n0 + n;
            if (a.Z) a.Z[o] = z;                            // forward only: the pre-activations are not kept
            if (DUAL) { if (a.U) a.U[o] = u; a.Act[o] = z * sigmoid_f(z) * u; }
            else a.Act[o] = gelu_f(z);
        });
    } else if (MODE == FWD2) {
        const Operand A{a.Actc + r0 * h, h, nr}, B{a.W2 + wdh + n0, d, d - n0};
        contract<TL, true, BKC, false, VH, VD>(acc, acc2, lds, A, B, A, B, 1, h);
        for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float y, float) {
            if (m < nr && n0 + n < d) a.Yp[(r0 + m) * d + n0 + n] = y;
        });
    } else if (MODE == BWD1) {                              // dA[m, n] = sum_c dYp[m, c] W2[n, c]
        const Operand A{a.dYp + r0 * d, d, nr}, B{a.W2 + wdh + (long)n0 * d, d, h - n0};
        contract<TL, true, BKC, false, VD, VD>(acc, acc2, lds, A, B, A, B, 1, d);
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
        contract<TL, true, BKC, false, VH, VH>(acc, acc2, lds, A, B, A2, B2, swiglu ? 2 : 1, h);
        for_each_output<TL, false>(acc, acc2, lds, [&](int m, int n, float v, float) {
            if (m < nr && n0 + n < d) a.dXp[(r0 + m) * d + n0 + n] = v;
        });
    }
}

// The group with the nth most rows (ties: the lower group first; groups past the hosted ones have none), so that the blocks
// with the longest contraction start first and the short ones fill the chip while they end.  More than 64 groups: as they come.
__device__ __forceinline__ int nth_longest(const F32Args& a, int nth, int first, int ng)
{
    if (a.Gcap > 64) return nth;
    const int lane = threadIdx.x & 63;
    int n = lane < a.Gcap ? 0 : -1;
    if (lane < ng) n = a.slot_offsets[first + lane + 1] - a.slot_offsets[first + lane];
    int rank = 0;
    for (int i = 0; i < a.Gcap; ++i) {
        const int o = __builtin_amdgcn_readlane(n, i);
        rank += (o > n || (o == n && i < lane)) ? 1 : 0;
    }
    return __ffsll((long long)__ballot(lane < a.Gcap && rank == nth)) - 1;
}

// Weight gradients, all products of all groups in one launch: out[m, n] = sum over the group's rows r of L[r, m] R[r, n]
// (dW1 = Xp^T dZ, dW2 = Act^T dYp, dW3 = Xp^T dU).  grid: tiles of a product x (products of group 0, of group 1, ...).
template <class TL, int VD, int VH>
__global__ __launch_bounds__(F32_THREADS) void ffn_f32_wgrad_kernel(F32Args a, int n_products)
{
    __shared__ __attribute__((aligned(1024))) float lds[lds_floats<TL, false>()];
    const int which = blockIdx.y % n_products, tile = blockIdx.x;
    int first, ng;
    hosted_range(a.dest_slots, a.self, a.Gcap, first, ng);
    // (32 x 32 tiles: too little work for the order to pay for itself, 0.6 us of 34)
    const int g = TL::WK == 1 ? nth_longest(a, blockIdx.y / n_products, first, ng) : blockIdx.y / n_products;
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
    if (VD == VH || which != 1) contract<TL, false, false, false, VD, VH>(acc, acc2, lds, A, B, A, B, 1, rows);
    else contract<TL, false, false, false, VH, VD>(acc, acc2, lds, A, B, A, B, 1, rows);
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

// How operands are requested.  d is a multiple of 4 (moe_create), so rows of d floats begin at multiples of 16 bytes where
// their tensors do; rows of h floats also need h to be a multiple of 4.  A 32-bit offset reaches the 64 rows or steps of a
// slice; in wider layers (2^24 and more) every row has a resource of its own: h = 2^24, d = 4, five rows, GELU, forward 178 ms
// with predicated loads and 64-bit addresses, 157 now, backward 178 and 176; d = 2^24, h = 8, 40 rows, SwiGLU, 246 and 256, 195
// and 169.  Requests of 4 bytes instead of 16 cost little: T = 3000, d = 512, k = 2, forward and backward, h = 2048 578 us, 2047
// 602 (1023 with predicated 4-byte loads into registers).
enum Requests { ALL_16 = 0, ROWS_OF_D_16 = 1, ALL_4 = 2, FAR_APART = 3 };
Requests requests_of(const moe_shape_t& s, std::initializer_list<const void*> rows_of_d, std::initializer_list<const void*> rows_of_h)
{
    constexpr int FAR = (1 << 24) - 64;
    if (s.d > FAR || s.h > FAR) return FAR_APART;
    uintptr_t bits_d = 0, bits_h = s.h % 4;
    for (const void* p : rows_of_d) bits_d |= reinterpret_cast<uintptr_t>(p);
    for (const void* p : rows_of_h) bits_h |= reinterpret_cast<uintptr_t>(p);
    return (bits_d & 15) ? ALL_4 : ((bits_h & 15) ? ROWS_OF_D_16 : ALL_16);
}

// Which tile, by the number of 64 x 64 tiles of all T k rows (a part of them is hosted here).  Few: 32 x 32, the serial chain
// is what counts, and many small tiles are spread evenly.  More: 64 x 64, which requests and reads least per product.  Between
// them, for long contractions, 64 x 32 with two waves along the contraction, because a CU that gets three 64 x 64 tiles where
// others get two is what the launch waits for (of short ones it is the fourth 64 x 32 tile, which has to wait for room).
// Measured, us, one row contraction, 32 x 32 | 64 x 32 | 64 x 64 (T, k = 2, contraction, width; tiles): 600, 1024, 512 (152) 19.7 |
// 23.5 | 26.0;  1200, 512, 512 (304) 17.2 | 20.7 | 24.8, backward 18.7 | 24.6 | 31;  1500, 2048, 512 (376) 61 | 62 | 80;  4000, 1024, 256
// (500) 38.7 | 35.9 | 42.8;  1000, 256, 1024 (512) 19.6 | 22.4 | 19.2, backward 21.6 | 27.9 | 25.3;  3000, 2048, 512 (752) 112 | 107 |
// 117;  1500, 3000, 1000 (752) 159 | 151 | 167;  2500, 292, 612 (790) - | 32.7 | 28.0;  3000, 1020, 640 (940), SwiGLU - | 144 | 150;  700,
// 128, 2800 (968) - | 23.7 | 20.0, backward - | 33.1 | 27.2;  1000, 700, 2000 (1024) - | 67 | 61;  4000, 200, 640 (1250) 32.6 | 32.5 | 27.8;
// 1500, 512, 2048 (1504) 71 | 71 | 67;  4000, 3000, 1000 (2000) 389 | 372 | 365;  3000, 512, 2048 (3008) 134 | 129 | 113.  128 x 128 was the
// slower one everywhere (fewer blocks to hide a request behind, a longer last round).  The weight gradients, whose tiles are
// all of one launch, take 64 x 64 from 700 tiles on.
// 32 x 32 tiles that all find room at once with four buffers (two blocks per CU, one of two weight matrices; the weight
// gradients: one per CU) have four, which hide a request that two don't: T = 512, d = 64, h = 256 fwd2 5.4 | 5.0; 144 tiles of K =
// 1500 15.8 | 14.1.  Others have two, and four or five blocks per CU: 640 tiles of K = 512 14.2 | 17.1, backward 15.7 | 19.9, SwiGLU
// 20.5 | 27.3; weight gradients of d = 300, h = 900, four groups of 100 rows 14.4 | 18.3.
constexpr long MEDIUM_TILES = 700, LONG = 1000, HALF_TILES_LONG = 400, MEDIUM_TILES_LONG = 1100, CUS = 256;
long tiles64(long rows, long cols) { return ((rows + 63) / 64) * ((cols + 63) / 64); }

template <int MODE, class TL, bool DUAL>
void launch_rows_t(const moe_shape_t& s, const F32Args& f, int N, Requests r, hipStream_t st)
{
    const dim3 grid(cdiv(N, TL::BN), cdiv(s.T * s.k, TL::BM) + s.G);
    if (r == ALL_16) hipLaunchKernelGGL((ffn_f32_kernel<MODE, TL, DUAL, 4, 4>), grid, dim3(F32_THREADS), 0, st, f);
    else if (r == ROWS_OF_D_16) hipLaunchKernelGGL((ffn_f32_kernel<MODE, TL, DUAL, 4, 1>), grid, dim3(F32_THREADS), 0, st, f);
    else hipLaunchKernelGGL((ffn_f32_kernel<MODE, TL, DUAL, 1, 1>), grid, dim3(F32_THREADS), 0, st, f);
}

template <int MODE, bool DUAL>
hipError_t launch_rows(const moe_shape_t& s, const F32Args& f, int N, long K, Requests r, hipStream_t st)
{
    const long tiles = tiles64((long)s.T * s.k, N);
    if (r == FAR_APART)
        hipLaunchKernelGGL((ffn_f32_kernel<MODE, TileF, DUAL, 0, 0>), dim3(cdiv(N, TileF::BN), cdiv(s.T * s.k, TileF::BM) + s.G), dim3(F32_THREADS), 0, st, f);
    else if (tiles >= (K >= LONG ? MEDIUM_TILES_LONG : MEDIUM_TILES)) launch_rows_t<MODE, TileM, DUAL>(s, f, N, r, st);
    else if (K >= LONG && tiles >= HALF_TILES_LONG) launch_rows_t<MODE, TileH, DUAL>(s, f, N, r, st);
    else if ((cdiv(s.T * s.k, TileF::BM) + s.G) * (long)cdiv(N, TileF::BN) <= (DUAL ? 1 : 2) * CUS) launch_rows_t<MODE, TileF, DUAL>(s, f, N, r, st);
    else launch_rows_t<MODE, TileS, DUAL>(s, f, N, r, st);
    return hipGetLastError();
}

template <class TL>
hipError_t launch_wgrad(const moe_shape_t& s, const F32Args& f, Requests r, hipStream_t st)
{
    const int tiles = cdiv(s.d, TL::BM) * cdiv(s.h, TL::BN), np = s.act == MOE_ACT_SWIGLU ? 3 : 2;
    static_assert(TL::BM == TL::BN, "d x h and h x d have the same number of tiles");
    const dim3 grid(tiles, np * s.G);
    if (r == ALL_16) hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, 4, 4>), grid, dim3(F32_THREADS), 0, st, f, np);
    else if (r == ROWS_OF_D_16) hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, 4, 1>), grid, dim3(F32_THREADS), 0, st, f, np);
    else if (r == ALL_4) hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, 1, 1>), grid, dim3(F32_THREADS), 0, st, f, np);
    else if constexpr (TL::WK == 1) hipLaunchKernelGGL((ffn_f32_wgrad_kernel<TL, 0, 0>), grid, dim3(F32_THREADS), 0, st, f, np);
    else return hipErrorInvalidValue;                      // layers that wide have more than MEDIUM_TILES tiles
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_fwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const F32Args f = make_args(s, a);
    const Requests r = requests_of(s, {a.Xp, a.W2}, {a.W1, a.W3, a.Act});
    hipError_t e = s.act == MOE_ACT_SWIGLU ? launch_rows<FWD1, true>(s, f, s.h, s.d, r, st) : launch_rows<FWD1, false>(s, f, s.h, s.d, r, st);
    if (e == hipSuccess) e = launch_rows<FWD2, false>(s, f, s.d, s.h, r, st);
    return e;
}

hipError_t launch_ffn_bwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st)
{
    const F32Args f = make_args(s, a);
    const Requests r = requests_of(s, {a.dYp, a.Xp, a.W2}, {a.W1, a.W3, a.Act, a.dZ, a.dU});
    hipError_t e = launch_rows<BWD1, false>(s, f, s.h, s.d, r, st);
    if (e == hipSuccess) e = launch_rows<BWD2, false>(s, f, s.d, s.act == MOE_ACT_SWIGLU ? 2l * s.h : s.h, r, st);
    if (e != hipSuccess) return e;
    const int np = s.act == MOE_ACT_SWIGLU ? 3 : 2;
    if (tiles64((long)s.d * np, (long)s.h * s.G) >= MEDIUM_TILES) return launch_wgrad<TileM>(s, f, r, st);
    if (cdiv(s.d, TileF::BM) * cdiv(s.h, TileF::BN) * np * s.G <= CUS) return launch_wgrad<TileF>(s, f, r, st);
    return launch_wgrad<TileS>(s, f, r, st);
}
