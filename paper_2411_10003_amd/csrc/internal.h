// Internal declarations shared by the translation units of libmoehot (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <atomic>

#include "../../include/moehot.h"

struct moe_ctx {
    moe_shape_t s;
    // workspace layout (byte offsets, all multiples of 256)
    size_t off_status;     // int32 status word(s)
    size_t off_chunk_hist; // int32 [n_chunks][E] per-chunk expert histograms
    size_t off_chunk_base; // int32 [n_chunks][E] exclusive prefix over chunks
    size_t off_act;        // elt [A,h]  activation output A (forward) / recomputed A (backward)
    size_t off_dz;         // elt [A,h]  dZ
    size_t off_du;         // elt [A,h]  dU (SwiGLU)
    size_t off_gate_part;  // float [partitions][d*E + E] partial sums of the gate parameter gradients
    size_t off_split;      // float [ffn_split_units][256*256] partial tiles of the grouped GEMM's last, K-split round (bf16 path)
    size_t off_arrived;    // int32 [SPLIT_COUNTERS] which of those of an uneven cut are there
    size_t ws_bytes;
    int n_chunks;          // ceil(A / ROUTE_CHUNK)
    // apart from this setting (moe_set_act_saved) a handle is immutable: every call is a function of its arguments
    int act_saved = 0;     // backward may read the activation the forward pass left in the workspace
};

// One-time set-up of a kernel per device (its dynamic LDS limit, the device's CU count).  The set-up
// calls are idempotent, so threads that race simply both make them; devices past 63 are set up on every call.
struct PerDeviceOnce {
    std::atomic<uint64_t> done{0};
    bool is_done(int dev) const { return dev >= 0 && dev < 64 && ((done.load(std::memory_order_acquire) >> dev) & 1u); }
    void mark(int dev) { if (dev >= 0 && dev < 64) done.fetch_or(1ull << dev, std::memory_order_release); }
};
inline int current_device() { int d = 0; if (hipGetDevice(&d) != hipSuccess) d = -1; return d; }

// Assignments handled by one wave of the routing kernels.
constexpr int ROUTE_CHUNK = 256;

typedef uint16_t bf16_t;  // storage only

// Rows that are written once and are many more than the caches between here and HBM can keep until they are read (256 MB on the
// memory side, shared with everything else that passes) go out by nontemporal stores, and with them what is read for the last time:
// left dirty in those caches they are written back under the next kernels' reads, so what counts is the step and not the call.
// Forward and backward of two layers, one after the other (bf16, h = 512), us with plain accesses in one kernel against all of them as
// they are; rows of T x d elements:
//                           34 MB    67 MB   98 MB  134 MB  268 MB | 67 MB, d = 2048 | one expert per token, d = 2048: 134 MB  268 MB
//   scatter                 +10.7    +13.9   +33.8   +43.4   +66.3 | +20.2           |                                  +4.6   +25.2
//   combine                  +2.3     +6.5   +11.0   +11.1    +7.0 |  +1.0           |                                  +1.0   +11.9
//   combine's gradient      +14.0     +9.5   +19.4   +34.9   +46.5 | +10.1           |                                  +6.3   +16.1
//   input gradient           +3.7     +3.7    -1.4    +1.8   +10.9 |  -0.3           |                                  +0.6    +2.2
//   gate's gradients         +1.9     +4.3    +4.5    +6.3   +18.2 |  -1.2           |                                  -3.3    -6.0
//   all plain               +31      +31     +86     +96    +148   | +35             |                                 +28     +61
//   of a step of            668     1098    1436    1733    3022   | 930             |                                1128    2044
// In its own time combine loses (T = 32768, d = 4096, k = 2: 141 -> 150 us) and the step gains all the same; moe_dispatch_bwd in the input
// gradient's place loses in the step as well (+5.6, +15.5, +12.0, -2.8 | +0.4 | +13.2, +18.0 from 67 MB on if streamed): it writes as
// ever.  The line: at 17 MB no kernel gains or loses; at 34 MB this step gains, and a prefill whose experts read their rows at once
// lost 0.8 % (T = 8192, d = 1024, k = 2: 230.5 us a pass, 232.4); from 64 MB on no step measured has been slower.
constexpr size_t STREAM_BYTES = (size_t)64 << 20;
inline bool streams(size_t bytes) { return bytes >= STREAM_BYTES; }
typedef unsigned moe_piece_t __attribute__((ext_vector_type(4)));
// 16 bytes, by a plain or a nontemporal access
template <bool NT, typename V> __device__ __forceinline__ V load_piece_of(const V* p)
{
    static_assert(sizeof(V) == 16, "16 bytes");
    if constexpr (NT) return __builtin_bit_cast(V, __builtin_nontemporal_load(reinterpret_cast<const moe_piece_t*>(p)));
    else return *p;
}
template <bool NT, typename V> __device__ __forceinline__ void store_piece_of(V* p, const V& v)
{
    static_assert(sizeof(V) == 16, "16 bytes");
    if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(moe_piece_t, v), reinterpret_cast<moe_piece_t*>(p));
    else *p = v;
}

// MOE_OK, or MOE_ERR_HIP with the error remembered for moe_last_hip_error() (per thread).
int moe_hip_status(hipError_t e);

// ---- launchers (each returns a hipError_t; they enqueue on `st`) ----------------------------
hipError_t launch_gate_topk(const moe_shape_t& s, const void* X, const float* Wg, const float* bg,
                            float* logits, int32_t* idx, float* w, hipStream_t st);
hipError_t launch_gate_bwd(const moe_shape_t& s, const float* dw, const float* logits, const int32_t* idx,
                           float* dlogits, hipStream_t st);

hipError_t launch_chunk_hist(const moe_shape_t& s, const int32_t* idx, int32_t* chunk_hist, int n_chunks, hipStream_t st);
hipError_t launch_counts(const moe_shape_t& s, const int32_t* idx, int32_t* chunk_hist, int n_chunks, int32_t* counts, hipStream_t st);
hipError_t launch_layout_scan(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* counts,
                              const int32_t* chunk_hist, int32_t* chunk_base, int n_chunks,
                              const moe_layout_t& L, int32_t* status, hipStream_t st);
hipError_t launch_positions(const moe_shape_t& s, const int32_t* idx, const int32_t* chunk_base, int n_chunks,
                            const moe_layout_t& L, hipStream_t st);

hipError_t launch_scatter_rows(const moe_shape_t& s, const void* X, const int32_t* pos, void* Xp, hipStream_t st);
hipError_t launch_combine(const moe_shape_t& s, const void* Yp, const int32_t* pos, const float* w, void* out, hipStream_t st);
hipError_t launch_combine_bwd(const moe_shape_t& s, const void* dOut, const void* Yp, const int32_t* pos,
                              const float* w, void* dYp, float* dw, hipStream_t st);
bool small_dispatch_fits(const moe_shape_t& s, int n_chunks);
hipError_t launch_small_dispatch(const moe_shape_t& s, const int32_t* idx, const int32_t* expert_dest, const int32_t* counts,
                                 const void* X, void* Xp, int n_chunks, const moe_layout_t& L, int32_t* status, hipStream_t st);
bool layout_positions_fusable(const moe_shape_t& s, int n_chunks);
hipError_t launch_layout_positions(const moe_shape_t& s, const int32_t* idx, const int32_t* expert_dest, const int32_t* counts,
                                   const int32_t* chunk_hist, int n_chunks, const moe_layout_t& L, int32_t* status, hipStream_t st);
int gate_grad_partitions(const moe_shape_t& s);
hipError_t launch_input_grad(const moe_shape_t& s, const void* dXp, const int32_t* pos, const float* dlogits,
                             const float* Wg, void* dX, hipStream_t st);
hipError_t launch_gate_wgrad(const moe_shape_t& s, const void* X, const float* dlogits, float* partial, float* partial_b,
                             float* dWg, float* dbg, hipStream_t st);
hipError_t launch_trans_gather(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* pool_version,
                               int32_t* slot_expert, const int32_t* slot_version,
                               int n, const void* const* pools, void* const* groups, const size_t* bytes_per_expert, hipStream_t st);
hipError_t launch_trans_commit(const moe_shape_t& s, const int32_t* expert_dest, const int32_t* pool_version,
                               int32_t* slot_expert, int32_t* slot_version, hipStream_t st);
hipError_t launch_agg_add(const moe_shape_t& s, const int32_t* expert_dest, int n, const float* const* groups, float* const* pools,
                          const size_t* floats_per_expert, hipStream_t st);
hipError_t launch_recv_layout(const moe_shape_t& s, const int32_t* local_dest_slots, const int32_t* recv_offsets,
                              int32_t* slot_offsets, int32_t* dest_slots, hipStream_t st);
hipError_t launch_plan(const moe_planner_t& cfg, const int32_t* gating, const moe_plan_out_t& out, hipStream_t st);
hipError_t launch_dispatch_bwd(const moe_shape_t& s, const void* dXp, const int32_t* pos, void* dX, hipStream_t st);

constexpr int SPLIT_UNITS = 320;       // partial tiles the K-split of a last round may need: at most one per block
constexpr int UNEVEN_UNITS = 512;      // and an uneven cut: two for each of fewer tiles than there are blocks
constexpr int SPLIT_COUNTERS = 1024;   // a counter for each of them, in the smaller tiles
struct ffn_args {
    const void *Xp, *W1, *W2, *W3;
    const int32_t *slot_offsets, *dest_slots;
    void *Yp, *Z, *U, *Act;            // forward outputs (Act in workspace)
    const void* dYp;                   // backward
    void *dXp, *dZ, *dU;               // dZ, dU in workspace
    float *dW1, *dW2, *dW3;
    bool accumulate = false;           // weight gradients are added to what dW holds instead of overwriting it
    bool act_saved = false;            // backward: Act still holds the forward pass's activation (not recomputed)
    float* split_ws = nullptr;         // workspace for K-split partial tiles (ffn_split_units tiles of 256 x 256 floats)
    int32_t* arrived = nullptr;        // workspace, SPLIT_COUNTERS: cleared by the first launch of a pass, zero after every launch
};
int ffn_split_units(const moe_shape_t& s);     // partial tiles the bf16 FFN of these sizes may keep
hipError_t launch_ffn_fwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st);
hipError_t launch_ffn_bwd_f32(const moe_shape_t& s, const ffn_args& a, hipStream_t st);
hipError_t launch_ffn_fwd_bf16(const moe_shape_t& s, const ffn_args& a, hipStream_t st);
hipError_t launch_ffn_bwd_bf16(const moe_shape_t& s, const ffn_args& a, hipStream_t st);

// For the tests, not part of the interface: how the bf16 FFN lays out one of its contractions (0 fwd1, 1 fwd2, 2 bwd1, 3 bwd2,
// 4 dW1 and dW3, 5 dW2) for hosted groups of rows[0 .. n_groups) rows on a GPU of `cus` CUs.  Host only, launches nothing.
//   out[0..9]: side of a tile, blocks, row tiles, column tiles, tiles in full rounds, parts of the others (4, 5: of the
//   group cut into most), row tiles per band, whether a finishing launch follows, slices of the contraction (4, 5: of all
//   groups), rows the choice is made for.  4, 5: out[10 .. 10 + G) are the parts of each group.  0 .. 3: out[10] is 0, or the
//   slices of the first part of each of the other tiles where those are cut unevenly in two.
extern "C" int moe_ffn_tiling(moe_handle_t h, int contraction, int cus, int n_groups, const int32_t* rows, int32_t* out);
// Likewise: 1 if a contraction of the forward pass (0 fwd1, 1 fwd2) requests its weights past the caches, else 0.
extern "C" int moe_ffn_reads_once(moe_handle_t h, int contraction);

// ---- small device helpers ----------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
// Two floats to a pair of bf16, round-to-nearest-even, NaN stays NaN: the hardware conversion of gfx950
// (v_cvt_pk_bf16_f32), one instruction per pair instead of a dozen with a branch for the NaN case.
typedef __attribute__((ext_vector_type(2))) float moe_f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 moe_bf16x2_t;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const moe_f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, moe_bf16x2_t));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.0f) & 0xffffu); }

// Group table of the hosted slots, rebuilt by every FFN block from the layout (G is small).
__device__ __forceinline__ void hosted_range(const int32_t* dest_slots, int self, int Gcap, int& first_slot, int& n_groups) {
    first_slot = dest_slots[self];
    int n = dest_slots[self + 1] - first_slot;
    n_groups = n < Gcap ? n : Gcap;
    if (n_groups < 0) n_groups = 0;
}
