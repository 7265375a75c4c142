// Internal launcher interface between the C-ABI layer (api.hip) and the kernel files.
// Everything here takes device pointers that the API layer has already validated.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "etr.h"

namespace etr {

constexpr int kWave = 64;

// ---- select workspace ------------------------------------------------------
// Column-major copy of the per-expert selection keys plus the per-chunk prefix
// counts of the two-level scan.  All offsets are multiples of 256 bytes.
struct SelectWs {
    uint64_t* cmask;     // [T]          bit e set: token listed expert e (Eq. 5)
    uint32_t* keyT;      // [E][Tpad]    order-preserving key of score[t][e]; 0 = not a candidate
    uint32_t* tau;       // [E]          threshold key of expert e
    int32_t*  need_eq;   // [E]          how many candidates with key == tau are kept (lowest token first)
    int32_t*  pre_gt;    // [E][kMaxChunks] kept-for-sure (key > tau) tokens before the chunk
    int32_t*  pre_eq;    // [E][kMaxChunks] key == tau tokens before the chunk
    int32_t*  pre_kept;  // [E][kMaxChunks] strict-intersection variant: surviving tokens before the chunk
    uint32_t* hist1;     // [E][n_slices][2048] first radix digit counted per slice of the column (long columns only)
    int       n_slices;  // 0: no such pre-pass
    int       slice;     // tokens per slice (multiple of 4)
    int       Tpad;      // row stride of keyT
    int       ipt;       // tokens per chunk (= per thread of the per-expert kernel): 4 ... 64 a power of two, else 4 n
};
constexpr int kSelThreads = 1024;       // threads of the per-expert kernel = max chunks
size_t select_ws_bytes(int T, int E);
SelectWs select_ws_carve(void* ws, int T, int E);
// the allocation-free variant keeps this much scratch in a static device array (select.hip)
constexpr size_t kStaticSelectBytes = 8u << 20;
hipError_t static_select_scratch(void** out);    // its device address on the current device

// ---- launchers ---------------------------------------------------------------
// route.hip
hipError_t launch_route(const etr_config& c, const void* x, const float* w_emb, float* score, float* gate,
                        hipStream_t st);
// select.hip
hipError_t launch_select(const etr_config& c, const float* score, int32_t* topk_expert, int32_t* slot_of,
                         int32_t* slot_token, int32_t* counts, const SelectWs& w, hipStream_t st,
                         const int32_t* capacity_dev = nullptr,   // optional device-side bound <= c.capacity
                         long long sum_need = 0);   // > 0: affinity-sum threshold in 2^-30 units (adaptive token count)
// permute.hip
hipError_t launch_dispatch(const etr_config& c, const void* x, const int32_t* slot_token, const int32_t* counts,
                           void* xp, hipStream_t st);
hipError_t launch_combine(const etr_config& c, const void* yp, const float* gate, const int32_t* slot_of,
                          void* out, hipStream_t st);
// ffn.hip
size_t ffn_ws_bytes(const etr_config& c);
hipError_t launch_expert_ffn(const etr_config& c, const void* xp, const int32_t* counts, const void* w_gate,
                             const void* w_up, const void* w_down, void* yp, void* hidden, hipStream_t st,
                             hipEvent_t between = nullptr,    // optional event recorded between the two GEMMs
                             const int32_t* gather_rows = nullptr,    // see ffn_can_gather
                             void* a_save = nullptr, void* b_save = nullptr);   // optional [E][capacity][H]: W_gate x, W_up x
// True when GEMM-1 can read its rows straight from the token matrix through slot_token
// (then xp is never materialised by the fused forward).
bool ffn_can_gather(const etr_config& c);
int rows_expected(const etr_config& c);      // rows per expert that a batch can be expected to fill
long long rows_total(const etr_config& c);   // rows of all experts together that the selection can keep

// General grouped product of ffn.hip, used by the backward pass:
//   C[g][m][n] = sum_k A[g][m][k] * B[g][n][k]   (both operands contiguous along k)
// A is [G][M][lda] (or, with row_index[G][M], row row_index[g][m] of one [a_rows][lda] matrix),
// B0/B1 are [G][N][ldb], C/C2 are [G][M][N], all of the layer's dtype.  m_counts (optional) bounds the
// rows of each group, k_counts (optional) its contraction length: it is rounded up to a multiple of
// 64, at least 128 (at most K), and the operands must hold zeros in that padding (fp32 with ta: exactly k_counts).
// GEMM_MIDDLE (bf16, tb, rows through row_index): the element-wise middle of the backward on the product u, which is not stored.
enum GemmEpilogue { GEMM_PLAIN = 0, GEMM_SWIGLU = 1, GEMM_DUAL = 2, GEMM_MIDDLE = 3 };   // C = A B0^T | SiLU(A B0^T) .* (A B1^T) | both products | dab, h
struct GroupedGemm {
    const void* A; const void* B0; const void* B1;
    void* C; void* C2;
    const int32_t* m_counts; const int32_t* k_counts; const int32_t* row_index;
    int G, M, N, K, lda, ldb, a_rows;
    int epilogue;
    int dtype;
    // Operands with the contraction index slow (plain epilogue only; bf16: see grouped_gemm_transposed_ok):
    // ta: A is [G][K][lda] holding A[g][m][k] at (k, m); tb: B0 is [G][K][ldb] holding B[g][n][k] at (k, n).
    // With tb and B1 the contraction is split in the middle: B0 and B1 are [G][K/2][ldb] each.
    bool ta = false, tb = false;
    // With ta and tb, the contraction rows of one operand may come through an index (k_gather 1: A, 2: B0): that
    // operand is then one [k_rows][ld] matrix for all groups and row k of group g is its row
    // k_index[g * k_index_stride + k], clamped into [0, k_rows).  Per-group contraction lengths are then rounded up to at
    // least 256 (bf16); in that padding, where the other operand must hold zeros, the group's last row is fetched again.
    const int32_t* k_index = nullptr;
    int k_index_stride = 0, k_rows = 0, k_gather = 0;
    // With ta and the plain epilogue: output rows m < split_m go to C, the others (as rows m - split_m) to C2, both
    // [G][split_m][N]; M = 2 split_m, split_m a multiple of 32.  (Two products that share B in one launch.)
    int split_m = 0;
    // rows per group that the caller expects (0: unknown); picks the kernel for few rows (row-major bf16 operands)
    int rows_expected = 0;
    // rows of all groups together that the batch can fill (0: unknown); sizes the grid of the kernel for few rows, which
    // still covers every row that m_counts names
    long long rows_total = 0;
    // input gradient in launch_backward_products, bf16: the contraction in this many parts; C is float [pieces][G][M][N]
    int pieces = 1;
    // GEMM_MIDDLE: a = W_g x and b = W_u x are [G][M][N]; gate is [a_rows][G], read at the rows' tokens.  Out come C = (da | db)
    // [G][mid_rows][2 N], C2 = h [G][mid_rows][N] (mid_scale_h: gate * h) and mid_part [ceil(N / 64)][G][M], the share of
    // <u, h> of each 64 columns, the group's rows of each.
    const void* mid_a = nullptr; const void* mid_b = nullptr;
    const float* mid_gate = nullptr;
    float* mid_part = nullptr;
    int mid_rows = 0;
    bool mid_scale_h = false;
};
hipError_t launch_grouped_gemm(const GroupedGemm& g, hipStream_t st);
bool grouped_gemm_transposed_ok(const GroupedGemm& g);
// The input gradient (tb) and the weight gradients (ta and tb) in one launch; down with k_gather 1 and one or two gates with
// k_gather 2, only the gates, or none of them (fp32: any).
hipError_t launch_backward_products(const GroupedGemm& dx, const GroupedGemm& down, const GroupedGemm* gates, int n_gates, hipStream_t st);

// backward.hip
size_t backward_ws_bytes(const etr_config& c);
hipError_t launch_moe_backward(const etr_config& c, const void* x, const float* w_emb, const void* w_gate,
                               const void* w_up, const void* w_down, const float* score, const float* gate,
                               const int32_t* slot_of, const int32_t* slot_token, const int32_t* counts,
                               const void* dout, void* dx, void* dw_gate, void* dw_up, void* dw_down,
                               float* dgate, float* dscore, void* ws, hipStream_t st,
                               const void* a_saved = nullptr, const void* b_saved = nullptr);   // from a training-mode forward

// stats.hip
size_t stats_ws_bytes(int T, int E);
hipError_t launch_route_stats(const etr_config& c, const float* gate, const int32_t* slot_of, const int32_t* counts,
                              const float* target, float* load, float* mean_gate, float* kl, int32_t* n_unrouted,
                              void* ws, hipStream_t st);
hipError_t launch_capacity_lower_bound(const etr_config& c, const float* score, float* dmax, int32_t* capacity,
                                       void* ws, hipStream_t st);

// Host-side launch helpers (api.hip).  Both remember their answer per device, so a steady-state call issues no
// runtime call besides its launches.
//   cu_count            compute units of the current device (256 if the query fails)
//   ensure_dynamic_lds  raises a kernel's dynamic-LDS limit to `bytes` unless a limit at least that large has
//                       already been set for this (device, kernel); limits up to 64 KiB need no call at all
int cu_count();
hipError_t ensure_dynamic_lds(const void* kernel, size_t bytes);

// For the tests, which have to know that a size reaches the kernel they are about: the kernel of a product of the expert
// networks (product 0: gate/up, 1: down; gathered: rows read through slot_token, as the fused call does) and its number
// of workgroups.  Host only; `c` must be valid.
// 0 register-staged, 1 few rows, 2 persistent, 3 persistent with a zero-filled last k-tile, 4 ring, 5 / 6 fp32 with
// 64 x 64 / 32 x 32 tiles.
extern "C" int etr_ffn_plan(const etr_config* c, int product, int gathered, long long* workgroups);

// ---- device helpers -----------------------------------------------------------
// Inclusive prefix sum over the 64 lanes of a wave, lane 0 first, by data-parallel-primitive moves: shifts by
// 1, 2, 4, 8 inside each row of 16 lanes (a lane whose source lies outside its row adds nothing), then lane 15 of
// row 0 / 2 is added to all of row 1 / 3 and lane 31 to all of rows 2 and 3.  Call with all lanes active.
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 -> rows 2, 3
    return v;
}

// The same for 64-bit sums.
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_from(long long v) {
    const uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(static_cast<unsigned long long>(v) >> 32);
    const uint32_t l = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(lo), CTRL, ROWS, 0xF, false));
    const uint32_t h = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(hi), CTRL, ROWS, 0xF, false));
    return static_cast<long long>((static_cast<unsigned long long>(h) << 32) | l);
}
__device__ __forceinline__ long long wave_scan_incl(long long v) {
    v += dpp_from<0x111, 0xF>(v);
    v += dpp_from<0x112, 0xF>(v);
    v += dpp_from<0x114, 0xF>(v);
    v += dpp_from<0x118, 0xF>(v);
    v += dpp_from<0x142, 0xA>(v);
    v += dpp_from<0x143, 0xC>(v);
    return v;
}

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }
inline size_t elt_bytes(int dtype) { return dtype == ETR_F32 ? 4 : 2; }

}  // namespace etr
