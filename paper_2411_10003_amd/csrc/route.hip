// Input distribution (Section 3 of the paper: inputs per expert), the send layout of a placement
// (Section 4.1) and the stable positions of the assignments inside it.  Integer work only.
//
// Assignments are cut into chunks of ROUTE_CHUNK consecutive ids, one wavefront per chunk.
//   chunk_hist[c][e]  assignments of expert e in chunk c (LDS counters; sums of ones, the same in any order)
//   chunk_base[c][e]  the same summed over all earlier chunks
//   pos[a] = slot_offsets[slot(e)] + chunk_base[c][e] + (rank of a among the chunk's earlier e's)
// What bounds all of it is latency: a few hundred KB at most, so launches, dependent loads and serial loops are what
// counts.  The lanes of a wave that hold the same expert find each other with one ballot per bit of the expert id.
#include "internal.h"

namespace {

constexpr int ROUTE_WAVES = 4;
constexpr int ROUNDS = ROUTE_CHUNK / 64;

__device__ __forceinline__ unsigned long long lanemask_lt(int lane) {
    return (lane == 0) ? 0ull : (~0ull >> (64 - lane));
}

// The expert of assignment a, -1 past the end and for a corrupt index (not counted, gets no row).
__device__ __forceinline__ int expert_of(const int32_t* __restrict__ idx, int a, int A, int E)
{
    const int e = a < A ? idx[a] : -1;
    return (e < 0 || e >= E) ? -1 : e;
}

// Lanes of the wave that hold the same expert as this one (nothing for -1).  bits: of the largest expert id.
__device__ __forceinline__ unsigned long long same_expert(int e, int bits)
{
    unsigned long long m = __ballot(e >= 0);
    for (int b = 0; b < bits; ++b) {
        const bool one = (e >> b) & 1;
        const unsigned long long v = __ballot(one);
        m &= one ? v : ~v;
    }
    return e >= 0 ? m : 0ull;
}
__device__ __forceinline__ int id_bits(int E) { return 32 - __clz(E - 1 > 0 ? E - 1 : 1); }

// One wave: histogram of a chunk in its LDS row.
__device__ __forceinline__ void chunk_histogram(int32_t* hist, const int (&e_of)[ROUNDS], int E, int lane)
{
    for (int e = lane; e < E; e += 64) hist[e] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
        if (e_of[r] >= 0) atomicAdd(&hist[e_of[r]], 1);
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(ROUTE_WAVES * 64) void chunk_hist_kernel(
    const int32_t* __restrict__ idx, int32_t* __restrict__ chunk_hist, int A, int E, int n_chunks)
{
    extern __shared__ int32_t hist_lds[];          // [ROUTE_WAVES][E]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunk = blockIdx.x * ROUTE_WAVES + wave;
    if (chunk >= n_chunks) return;
    int32_t* hist = hist_lds + wave * E;
    int e_of[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) e_of[r] = expert_of(idx, chunk * ROUTE_CHUNK + r * 64 + lane, A, E);
    chunk_histogram(hist, e_of, E, lane);
    for (int e = lane; e < E; e += 64) chunk_hist[(size_t)chunk * E + e] = hist[e];
}

// Histograms and counts of up to COUNT_CHUNKS chunks in one block: one launch instead of two where the second would
// wait for a handful of waves.
constexpr int COUNT_WAVES = 16, COUNT_CHUNKS = 64;
__global__ __launch_bounds__(COUNT_WAVES * 64) void small_counts_kernel(
    const int32_t* __restrict__ idx, int32_t* __restrict__ chunk_hist, int32_t* __restrict__ counts, int A, int E, int n_chunks)
{
    extern __shared__ int32_t hist_lds[];          // [COUNT_WAVES][E] and [E]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t* hist = hist_lds + wave * E;
    int32_t* total = hist_lds + COUNT_WAVES * E;
    for (int e = threadIdx.x; e < E; e += COUNT_WAVES * 64) total[e] = 0;
    int e_of[COUNT_CHUNKS / COUNT_WAVES][ROUNDS];
#pragma unroll
    for (int i = 0; i < COUNT_CHUNKS / COUNT_WAVES; ++i)
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            e_of[i][r] = expert_of(idx, (i * COUNT_WAVES + wave) * ROUTE_CHUNK + r * 64 + lane, A, E);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < COUNT_CHUNKS / COUNT_WAVES; ++i) {
        const int chunk = i * COUNT_WAVES + wave;
        if (chunk >= n_chunks) break;
        chunk_histogram(hist, e_of[i], E, lane);
        for (int e = lane; e < E; e += 64) {
            const int n = hist[e];
            chunk_hist[(size_t)chunk * E + e] = n;
            if (n) atomicAdd(&total[e], n);
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += COUNT_WAVES * 64) counts[e] = total[e];
}

__global__ void counts_from_hist_kernel(const int32_t* __restrict__ chunk_hist, int n_chunks, int E,
                                        int32_t* __restrict__ counts)
{
    // one wavefront per expert: lanes stride over the chunks, then a butterfly sum
    const int lane = threadIdx.x & 63;
    const int e = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (e >= E) return;
    int s = 0;
    for (int c = lane; c < n_chunks; c += 64) s += chunk_hist[(size_t)c * E + e];
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) counts[e] = s;
}

// One wave: the rows of a chunk's assignments.  next: the wave's LDS row with the next free row of every expert.
template <typename PUT>
__device__ __forceinline__ void chunk_positions(int32_t* next, const int (&e_of)[ROUNDS], int E, int lane, PUT put)
{
    const int bits = id_bits(E);
    volatile int32_t* nx = next;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int e = e_of[r];
        const unsigned long long peers = same_expert(e, bits);
        const int rank = __popcll(peers & lanemask_lt(lane));
        int base = 0;
        if (e >= 0) base = nx[e];
        __builtin_amdgcn_wave_barrier();
        if (e >= 0) {
            put(r, base + rank);
            if (rank == 0) nx[e] = base + __popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ __launch_bounds__(ROUTE_WAVES * 64) void positions_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ chunk_base,
    const int32_t* __restrict__ slot_of_expert, const int32_t* __restrict__ slot_offsets,
    int32_t* __restrict__ pos, int32_t* __restrict__ perm, int A, int E, int n_chunks)
{
    extern __shared__ int32_t next_lds[];          // [ROUTE_WAVES][E] next free row per expert
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunk = blockIdx.x * ROUTE_WAVES + wave;
    if (chunk >= n_chunks) return;
    int32_t* next = next_lds + wave * E;
    for (int e = lane; e < E; e += 64)
        next[e] = slot_offsets[slot_of_expert[e]] + chunk_base[(size_t)chunk * E + e];
    int e_of[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) e_of[r] = expert_of(idx, chunk * ROUTE_CHUNK + r * 64 + lane, A, E);
    chunk_positions(next, e_of, E, lane, [&](int r, int row) {
        const int a = chunk * ROUTE_CHUNK + r * 64 + lane;
        pos[a] = row;
        perm[row] = a;
    });
}

// The layout from the counts and the placement, rebuilt by a whole block in LDS.  lds: 5 E + 3 words: dest, slot of each expert,
// count and first row of each slot (E + 1), first slot of each destination (P + 1, P <= E), a flag.
// Slots are ranks by (destination, id).  Up to WALK_EXPERTS experts every expert walks over all of them.  Beyond, one wave finds
// the ranks 64 experts at a time, like the rows of a chunk: the lanes with the same destination find each other by ballots,
// and a counter per destination carries over.  The launch that finds layout and positions, us, walk | wave: E = 16, 65536
// assignments 9.4 | 10.2; E = 32, 32768 6.3 | 6.9; E = 40, 6000 7.7 | 7.0; E = 64, 10000 9.2 | 7.4; E = 128, 32004 11.5 | 8.7,
// 24000 11.4 | 8.1.  Instantiations of their own (WALK): one kernel with both ways in it took the walk longer (counts and
// dispatch of up to 32 experts, 96 drawn shapes: 1 to 3 % in the mean).
constexpr int WALK_EXPERTS = 32;
struct BlockLayout { int32_t *dest, *slot_of, *slot_cnt, *slot_off, *first, *flag; };
__device__ __forceinline__ BlockLayout block_layout_lds(int32_t* lds, int E)
{
    return BlockLayout{lds, lds + E, lds + 2 * E, lds + 3 * E, lds + 4 * E + 1, lds + 5 * E + 2};
}
__host__ __device__ __forceinline__ constexpr int block_layout_words(int E) { return 5 * E + 3; }

// One wave: v[0 .. n) replaced by the sums before them, v[n] by the sum of all.
__device__ __forceinline__ void wave_exclusive_scan(const int32_t* v, int32_t* out, int n, int lane)
{
    int carry = 0;
    for (int s0 = 0; s0 < n; s0 += 64) {
        const int x = s0 + lane < n ? v[s0 + lane] : 0;
        int incl = x;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        if (s0 + lane < n) out[s0 + lane] = carry + incl - x;
        carry += __shfl(incl, 63, 64);
    }
    if (lane == 0) out[n] = carry;
    __builtin_amdgcn_wave_barrier();
}

template <bool WALK>
__device__ __forceinline__ void build_layout(const BlockLayout& L, const int32_t* __restrict__ expert_dest,
                                             const int32_t* __restrict__ counts, int E, int P)
{
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid == 0) *L.flag = 0;
    if (!WALK) for (int p = tid; p <= P; p += blockDim.x) L.first[p] = 0;
    __syncthreads();
    for (int e = tid; e < E; e += blockDim.x) {
        int p = expert_dest[e];
        if (!WALK) L.slot_off[e] = counts[e];               // for now
        if (p < 0 || p >= P) { atomicOr(L.flag, 1); p = p < 0 ? 0 : P - 1; }
        L.dest[e] = p;
    }
    __syncthreads();
    if (WALK) {
        for (int e = tid; e < E; e += blockDim.x) {
            const int p = L.dest[e], n = counts[e];
            int sl = 0;
#pragma unroll 4
            for (int f = 0; f < E; ++f) sl += (L.dest[f] < p) || (L.dest[f] == p && f < e);
            L.slot_of[e] = sl;
            L.slot_cnt[sl] = n;
        }
        __syncthreads();
    } else if (tid < 64) {
        const int bits = id_bits(P);
        volatile int32_t* in_dest = L.first;                // experts of each destination so far
        for (int s0 = 0; s0 < E; s0 += 64) {
            const int e = s0 + lane, p = e < E ? L.dest[e] : -1;
            const unsigned long long peers = same_expert(p, bits);
            const int rank = __popcll(peers & lanemask_lt(lane));
            int base = 0;
            if (p >= 0) base = in_dest[p];
            __builtin_amdgcn_wave_barrier();
            if (p >= 0) {
                L.slot_of[e] = base + rank;
                if (rank == 0) in_dest[p] = base + __popcll(peers);
            }
            __builtin_amdgcn_wave_barrier();
        }
        wave_exclusive_scan(L.first, L.first, P, lane);
        for (int e = lane; e < E; e += 64) {
            const int sl = L.first[L.dest[e]] + L.slot_of[e];
            L.slot_of[e] = sl;
            L.slot_cnt[sl] = L.slot_off[e];
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (tid < 64) wave_exclusive_scan(L.slot_cnt, L.slot_off, E, lane);
    __syncthreads();
}

// One block publishes the layout.
template <bool WALK>
__device__ __forceinline__ void publish_layout(const BlockLayout& L, const moe_layout_t& out, int32_t* __restrict__ status,
                                               int E, int P, int self, int Gcap)
{
    const int tid = threadIdx.x;
    for (int e = tid; e < E; e += blockDim.x) out.slot_of_expert[e] = L.slot_of[e];
    for (int s = tid; s <= E; s += blockDim.x) out.slot_offsets[s] = L.slot_off[s];
    for (int p = tid; p <= P; p += blockDim.x) {
        int first = 0, mine = 0;                            // slots of destinations below p, of p
        if (WALK) {
            for (int f = 0; f < E; ++f) { first += (L.dest[f] < p); mine += (L.dest[f] == p); }
        } else {
            first = L.first[p];
            mine = p < P ? L.first[p + 1] - first : 0;
        }
        out.dest_slots[p] = first;
        out.dest_offsets[p] = L.slot_off[first];
        if (p == self) *status = (*L.flag || mine > Gcap) ? (int32_t)MOE_ERR_PLAN : (int32_t)MOE_OK;
    }
}

// The layout and the per-chunk bases, for more chunks than layout_positions_kernel adds up: one block per 64 experts scans
// their histograms over the chunks, block 0 publishes the layout.
constexpr int SCAN_WAVES = 16;
template <bool WALK>
__global__ __launch_bounds__(SCAN_WAVES * 64) void layout_scan_kernel(
    const int32_t* __restrict__ expert_dest, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ chunk_hist, int32_t* __restrict__ chunk_base, int n_chunks,
    const moe_layout_t out, int32_t* __restrict__ status, int E, int P, int self, int Gcap)
{
    extern __shared__ int32_t lds[];
    __shared__ int32_t part[SCAN_WAVES][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, e = blockIdx.x * 64 + lane;
    if (blockIdx.x == 0) {
        const BlockLayout L = block_layout_lds(lds, E);
        build_layout<WALK>(L, expert_dest, counts, E, P);
        publish_layout<WALK>(L, out, status, E, P, self, Gcap);
    }
    // wave w owns a run of chunks: their sum, the sums of the runs before, then the bases of its chunks
    const int per = (n_chunks + SCAN_WAVES - 1) / SCAN_WAVES, c0 = min(wave * per, n_chunks), c1 = min(c0 + per, n_chunks);
    int sum = 0;
#pragma unroll 8
    for (int c = c0; c < c1; ++c) sum += e < E ? chunk_hist[(size_t)c * E + e] : 0;
    part[wave][lane] = sum;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += part[w][lane];
#pragma unroll 8
    for (int c = c0; c < c1; ++c) {
        const int v = e < E ? chunk_hist[(size_t)c * E + e] : 0;
        if (e < E) chunk_base[(size_t)c * E + e] = base;
        base += v;
    }
}

// Layout and positions in one launch: every block rebuilds the (small) layout in LDS, block 0 publishes it, and the
// base of a block's first chunk is summed from the histograms of all chunks before it (its waves share them; whole rows,
// all loads independent) instead of being read from a prefix table that a launch of a single block would have to write
// first.
template <bool WALK>
__global__ __launch_bounds__(ROUTE_WAVES * 64) void layout_positions_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ expert_dest, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ chunk_hist, const moe_layout_t out, int32_t* __restrict__ status,
    int A, int E, int P, int self, int Gcap, int n_chunks)
{
    extern __shared__ int32_t lds[];               // layout, [ROUTE_WAVES][E] next free rows
    const BlockLayout L = block_layout_lds(lds, E);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunk0 = blockIdx.x * ROUTE_WAVES, chunk = chunk0 + wave;
    int32_t* next = lds + block_layout_words(E);
    int e_of[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) e_of[r] = expert_of(idx, chunk * ROUTE_CHUNK + r * 64 + lane, A, E);
    for (int i = tid; i < ROUTE_WAVES * E; i += blockDim.x) next[i] = 0;
    build_layout<WALK>(L, expert_dest, counts, E, P);
    // wave w adds up every ROUTE_WAVES-th chunk before this block, for everybody, and the block's chunks w .. 2 for the
    // waves behind them; lane l takes the experts l, l + 64, ...
    for (int s0 = 0; s0 < E; s0 += 64) {
        const int e = s0 + lane;
        const bool on = e < E;
        const int32_t* col = chunk_hist + (on ? e : 0);     // unconditional loads
        int sum = 0;
#pragma unroll 8
        for (int c = wave; c < chunk0; c += ROUTE_WAVES) sum += col[(size_t)c * E];
        const int mine = chunk < n_chunks ? col[(size_t)chunk * E] : 0;
        if (on) {
            if (wave == 0) sum += L.slot_off[L.slot_of[e]];
#pragma unroll
            for (int w = 0; w < ROUTE_WAVES; ++w) {
                const int add = sum + (w > wave ? mine : 0);
                if (add) atomicAdd(&next[w * E + e], add);
            }
        }
    }
    __syncthreads();
    if (blockIdx.x == 0) publish_layout<WALK>(L, out, status, E, P, self, Gcap);
    if (chunk >= n_chunks) return;
    chunk_positions(next + wave * E, e_of, E, lane, [&](int r, int row) {
        const int a = chunk * ROUTE_CHUNK + r * 64 + lane;
        out.pos[a] = row;
        out.perm[row] = a;
    });
}

// The whole dispatch of a small batch (up to SMALL_CHUNKS chunks) in one launch: every block finds all positions for itself
// (a chunk per wave, in LDS) and copies its share of the rows; block 0 publishes layout and positions.  No histogram is
// read.  What bounds it is latency: the two launches this replaces took 8 + 5 us of the GPU in a row at T = 64 and 3 us each
// of the host.  Gate, counts and dispatch in a row: T = 1999, d = 768, E = 16, k = 2 30 -> 20 us; T = 512, d = 64, E = 8
// 29 -> 18.
constexpr int SMALL_CHUNKS = 16, SMALL_EXPERTS = 256, PIECE_VECS = 256;
template <bool WALK>
__global__ __launch_bounds__(SMALL_CHUNKS * 64) void small_dispatch_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ expert_dest, const int32_t* __restrict__ counts,
    const uint4* __restrict__ X, uint4* __restrict__ Xp, const moe_layout_t out, int32_t* __restrict__ status,
    int T, int k, int row_vecs, int E, int P, int self, int Gcap, int n_chunks)
{
    extern __shared__ int32_t lds[];               // layout, [SMALL_CHUNKS][E] next free rows, positions
    const BlockLayout L = block_layout_lds(lds, E);
    int32_t* next = lds + block_layout_words(E);
    int32_t* pos = next + SMALL_CHUNKS * E;
    const int tid = threadIdx.x, lane = tid & 63, chunk = tid >> 6, A = T * k;
    int e_of[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int a = chunk * ROUTE_CHUNK + r * 64 + lane;
        e_of[r] = expert_of(idx, a, A, E);
        if (a < A) pos[a] = -1;                    // a corrupt index gets no row
    }
    if (chunk < n_chunks) chunk_histogram(next + chunk * E, e_of, E, lane);
    build_layout<WALK>(L, expert_dest, counts, E, P);    // ends with a barrier
    for (int e = tid; e < E; e += blockDim.x) {    // counts of the chunks -> first rows
        int row = L.slot_off[L.slot_of[e]];
        for (int c = 0; c < n_chunks; ++c) {
            const int n = next[c * E + e];
            next[c * E + e] = row;
            row += n;
        }
    }
    __syncthreads();
    if (chunk < n_chunks)
        chunk_positions(next + chunk * E, e_of, E, lane, [&](int r, int row) {
            const int a = chunk * ROUTE_CHUNK + r * 64 + lane;
            pos[a] = row;
            if (blockIdx.x == 0) { out.pos[a] = row; out.perm[row] = a; }
        });
    __syncthreads();
    if (blockIdx.x == 0) publish_layout<WALK>(L, out, status, E, P, self, Gcap);
    // pieces of 4 KB of a token's row, dealt to the blocks in turn
    const int pieces = (row_vecs + PIECE_VECS - 1) / PIECE_VECS;
    for (int u = chunk * gridDim.x + blockIdx.x; u < T * pieces; u += SMALL_CHUNKS * gridDim.x) {
        const int t = u / pieces, v0 = (u - t * pieces) * PIECE_VECS + lane;
        const uint4* src = X + (size_t)t * row_vecs;
        uint4 x[PIECE_VECS / 64];
#pragma unroll
        for (int i = 0; i < PIECE_VECS / 64; ++i) x[i] = src[min(v0 + 64 * i, row_vecs - 1)];
        for (int j = 0; j < k; ++j) {
            const int row = pos[t * k + j];
            if (row < 0) continue;
            uint4* dst = Xp + (size_t)row * row_vecs;
#pragma unroll
            for (int i = 0; i < PIECE_VECS / 64; ++i) if (v0 + 64 * i < row_vecs) dst[v0 + 64 * i] = x[i];
        }
    }
}

// Layout of the rows a device receives for the experts it hosts: the same slots as the local layout, the row
// offsets of the receive buffer instead of those of the send buffer.
__global__ void recv_layout_kernel(const int32_t* __restrict__ local_dest_slots, const int32_t* __restrict__ recv_offsets,
                                   int32_t* __restrict__ slot_offsets, int32_t* __restrict__ dest_slots, int E, int P, int self, int G)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int first = local_dest_slots[self];
    if (i <= E) {
        int g = i - first;
        g = g < 0 ? 0 : (g > G ? G : g);
        slot_offsets[i] = recv_offsets[g];
    }
    if (i <= P) dest_slots[i] = local_dest_slots[i];
}

}  // namespace

hipError_t launch_chunk_hist(const moe_shape_t& s, const int32_t* idx, int32_t* chunk_hist, int n_chunks, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const int grid = (n_chunks + ROUTE_WAVES - 1) / ROUTE_WAVES;
    hipLaunchKernelGGL(chunk_hist_kernel, dim3(grid), dim3(ROUTE_WAVES * 64), (size_t)ROUTE_WAVES * s.E * sizeof(int32_t), st,
                       idx, chunk_hist, s.T * s.k, s.E, n_chunks);
    return hipGetLastError();
}

// Histograms into chunk_hist and the counts.  Up to COUNT_CHUNKS chunks (and 256 experts: 17 LDS rows) in one launch:
// expert_counts alone 12 -> 8 us, of which the host takes most, the two launches took 6 + 5 us of the GPU in a row.
hipError_t launch_counts(const moe_shape_t& s, const int32_t* idx, int32_t* chunk_hist, int n_chunks, int32_t* counts, hipStream_t st)
{
    if (n_chunks <= COUNT_CHUNKS && s.E <= 256) {
        hipLaunchKernelGGL(small_counts_kernel, dim3(1), dim3(COUNT_WAVES * 64), (size_t)(COUNT_WAVES + 1) * s.E * sizeof(int32_t), st,
                           idx, chunk_hist, counts, s.T * s.k, s.E, n_chunks);
        return hipGetLastError();
    }
    const hipError_t e = launch_chunk_hist(s, idx, chunk_hist, n_chunks, st);
    if (e != hipSuccess) return e;
    const int waves = 4;
    hipLaunchKernelGGL(counts_from_hist_kernel, dim3((s.E + waves - 1) / waves), dim3(waves * 64), 0, st,
                       chunk_hist, n_chunks, s.E, counts);
    return hipGetLastError();
}

hipError_t launch_layout_scan(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* counts,
                              const int32_t* chunk_hist, int32_t* chunk_base, int n_chunks,
                              const moe_layout_t& L, int32_t* status, hipStream_t st)
{
    auto kern = s.E <= WALK_EXPERTS ? layout_scan_kernel<true> : layout_scan_kernel<false>;
    hipLaunchKernelGGL(kern, dim3((s.E + 63) / 64), dim3(SCAN_WAVES * 64), (size_t)block_layout_words(s.E) * sizeof(int32_t), st,
                       expert_dest, counts, chunk_hist, chunk_base, n_chunks, L, status, s.E, s.P, s.self, s.G);
    return hipGetLastError();
}

hipError_t launch_positions(const moe_shape_t& s, const int32_t* idx, const int32_t* chunk_base, int n_chunks,
                            const moe_layout_t& L, hipStream_t st)
{
    if (n_chunks == 0) return hipSuccess;
    const int grid = (n_chunks + ROUTE_WAVES - 1) / ROUTE_WAVES;
    hipLaunchKernelGGL(positions_kernel, dim3(grid), dim3(ROUTE_WAVES * 64), (size_t)ROUTE_WAVES * s.E * sizeof(int32_t), st,
                       idx, chunk_base, L.slot_of_expert, L.slot_offsets, L.pos, L.perm, s.T * s.k, s.E, n_chunks);
    return hipGetLastError();
}

// The fused launch reads n_chunks^2 E / (2 ROUTE_WAVES) histogram words through L2 in all: up to 2^26 / 8 of them (33 MB,
// 1024 chunks of 64 experts) that is less than the launch of a scan costs.
bool layout_positions_fusable(const moe_shape_t& s, int n_chunks)
{
    return n_chunks >= 1 && (long long)n_chunks * n_chunks * s.E <= (1ll << 26);
}

hipError_t launch_layout_positions(const moe_shape_t& s, const int32_t* idx, const int32_t* expert_dest, const int32_t* counts,
                                   const int32_t* chunk_hist, int n_chunks, const moe_layout_t& L, int32_t* status, hipStream_t st)
{
    const int grid = (n_chunks + ROUTE_WAVES - 1) / ROUTE_WAVES;
    const size_t lds = (size_t)(block_layout_words(s.E) + ROUTE_WAVES * s.E) * sizeof(int32_t);
    auto kern = s.E <= WALK_EXPERTS ? layout_positions_kernel<true> : layout_positions_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(ROUTE_WAVES * 64), lds, st, idx, expert_dest, counts, chunk_hist,
                       L, status, s.T * s.k, s.E, s.P, s.self, s.G, n_chunks);
    return hipGetLastError();
}

bool small_dispatch_fits(const moe_shape_t& s, int n_chunks) { return n_chunks >= 1 && n_chunks <= SMALL_CHUNKS && s.E <= SMALL_EXPERTS; }

hipError_t launch_small_dispatch(const moe_shape_t& s, const int32_t* idx, const int32_t* expert_dest, const int32_t* counts,
                                 const void* X, void* Xp, int n_chunks, const moe_layout_t& L, int32_t* status, hipStream_t st)
{
    const int row_vecs = (int)((size_t)s.d * (s.dtype == MOE_BF16 ? 2 : 4) / 16);      // rows are multiples of 16 bytes (moe_create)
    const size_t lds = (size_t)(block_layout_words(s.E) + SMALL_CHUNKS * s.E + n_chunks * ROUTE_CHUNK) * sizeof(int32_t);
    const long pieces = (long)s.T * ((row_vecs + PIECE_VECS - 1) / PIECE_VECS);
    const int grid = pieces < 256 ? (int)pieces : 256;                                 // a block per piece while there are CUs
    auto kern = s.E <= WALK_EXPERTS ? small_dispatch_kernel<true> : small_dispatch_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(SMALL_CHUNKS * 64), lds, st, idx, expert_dest, counts,
                       (const uint4*)X, (uint4*)Xp, L, status, s.T, s.k, row_vecs, s.E, s.P, s.self, s.G, n_chunks);
    return hipGetLastError();
}

hipError_t launch_recv_layout(const moe_shape_t& s, const int32_t* local_dest_slots, const int32_t* recv_offsets,
                              int32_t* slot_offsets, int32_t* dest_slots, hipStream_t st)
{
    const int n = (s.E > s.P ? s.E : s.P) + 1;
    hipLaunchKernelGGL(recv_layout_kernel, dim3((n + 255) / 256), dim3(256), 0, st, local_dest_slots, recv_offsets,
                       slot_offsets, dest_slots, s.E, s.P, s.self, s.G);
    return hipGetLastError();
}

