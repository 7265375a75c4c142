// Expert networks on the kept rows: yp = W_down (SiLU(W_gate x) .* (W_up x)), one SwiGLU
// feed-forward block per expert (Sec. Locality Loss: experts are FFN layers; Sec.
// Experimental Setup: Mixtral experts).  This is the one dense contraction of the layer
// and the operator the paper reports as dominant ("FFN MatMul").
//
// bf16: two grouped "NT" GEMMs on the MFMA units (v_mfma_f32_16x16x32_bf16 in the two kernels
// most layers run on, v_mfma_f32_32x32x16_bf16 in the other forms), fp32 accumulation.  Both
// operands are K-contiguous, staged through LDS in 16-byte chunks with an XOR swizzle.
// GEMM-1 computes the gate and the up projection of the same output tile so that SiLU(g)*u is
// its epilogue and the hidden activation crosses HBM once, in bf16.  choose_bf16 picks the
// kernel: the persistent one for many rows per expert (gemm_bf16_persistent_kernel: one
// workgroup per CU walks the live tiles, the copies run on across tile boundaries), the
// few-rows one for few (gemm_bf16_rows_kernel, whose weights go straight to the fragments), and
// two per-tile kernels, whose grid is that of `capacity` and where a workgroup whose row tile
// starts past counts[e] exits at once.  In all of them counts never leave the device.
// fp32: the same product on v_mfma_f32_16x16x4_f32, one workgroup per tile.

#include <algorithm>
#include <cmath>
#include <numeric>
#include <type_traits>

#include "etr_internal.h"

namespace etr {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct GemmParams {
    const void* A;        // [E][capacity][K]
    const void* B0;       // [E][N][K]
    const void* B1;       // [E][N][K] (GLU only)
    void* C;              // [E][capacity][N]
    const int32_t* counts;
    int E, capacity, N, K;
    int MT, NT;           // row tiles per expert, column tiles
    int SM, SN;           // super-tile shape (see decode_tile)
    const int32_t* row_index;   // optional [E][capacity]: A row m of expert e is row row_index[e][m] of A
    int a_rows;                 // rows of A that row_index may name (indices are clamped into [0, a_rows))
    int lda = 0, ldb = 0;       // row strides of A and B in elements (0: K)
    const int32_t* k_counts = nullptr;   // optional per-group contraction length; it is rounded up to a multiple
                                         // of 64, at least 128 (at most K), and the operands must hold zeros in
                                         // that padding
    void* C2 = nullptr;         // DUAL epilogue: the B1 product goes here, the B0 product to C, no activation
    void* C3 = nullptr;         // SwiGLU epilogue that also keeps the two products: B0 product to C2, B1 product to C3
    // Contraction rows fetched through an index (transposing and fp32 kernels; k_gather 1: A, 2: B0): row k of group g of
    // that operand is row k_index[g * k_index_stride + k] of a [k_rows][ld] matrix, clamped into [0, k_rows); k in the padding:
    // the group's last row again.  The per-group contraction length is then at least 256 (bf16).
    const int32_t* k_index = nullptr;
    int k_index_stride = 0, k_rows = 0, k_gather = 0;
    // Plain epilogue of the transposing kernel with the output rows split between two arrays: rows below split_m go
    // to C, the others (as rows m - split_m) to C2, both [E][split_m][N] (a multiple of 32, capacity = 2 split_m).
    int split_m = 0;
    long long rows_total = 0;   // host only: rows of all groups together that the batch can fill (0: unknown)
    // Input gradient only (transposing kernel, row-major A): the contraction in `pieces` parts, each a tile of its own whose
    // fp32 sums go to C as [pieces][E][capacity][N] (NT counts the column tiles of all parts)
    int pieces = 1;
    // Product of the backward's middle (gemm_bf16_transposing_kernel<.., MID>): see GEMM_MIDDLE
    const void* mid_a = nullptr;
    const void* mid_b = nullptr;
    const float* mid_gate = nullptr;
    float* mid_part = nullptr;
    int mid_rows = 0, mid_scale_h = 0;
};

// rows of group e (counts may be absent: every group has `capacity` rows) and its contraction length
__device__ __forceinline__ int group_rows(const GemmParams& p, int e) {
    return p.counts ? min(p.counts[e], p.capacity) : p.capacity;
}
__device__ __forceinline__ int group_k(const GemmParams& p, int e) {
    return p.k_counts ? min(max((max(p.k_counts[e], 0) + 63) & ~63, p.k_gather ? 256 : 128), p.K) : p.K;
}

// Two fp32 values -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    return make_uint2(pack_bf16(a, b), pack_bf16(c, d));
}

// SiLU(a) = a / (1 + exp(-a)) with the hardware exponential and reciprocal (about 1 ulp each; the result
// is rounded to bf16 right after)
__device__ __forceinline__ float silu(float a) {
    return a * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * a));
}

// Epilogue shared by the MFMA kernels.  acc[i][j] is the 32 x 32 block at rows m_base + 32 i, staged weight rows
// 32 j of this wave (GLU: the first TB/2 blocks are gate rows, the others the up rows of the same output columns).
// A lane holds, per block, row m = lane % 32 and the columns (v / 4) * 8 + (lane / 32) * 4 + v % 4, so every store is
// four consecutive bf16 of one row.
// KEEP (SwiGLU epilogue only): the two products are stored as well (C2, C3), for the training-mode forward.
template <bool GLU, bool DUAL, int TI, int TB, bool KEEP = false>
__device__ __forceinline__ void store_blocks(const GemmParams& p, const f32x16 (&acc)[TI][TB], int e, int m_base,
                                             int n_base, int count, int r32, int half) {
    constexpr int TO = GLU ? TB / 2 : TB;
    uint16_t* Cg = reinterpret_cast<uint16_t*>(p.C) + static_cast<size_t>(e) * p.capacity * p.N;
    uint16_t* C2g = (GLU && (DUAL || KEEP)) ? reinterpret_cast<uint16_t*>(p.C2) + static_cast<size_t>(e) * p.capacity * p.N : nullptr;
    uint16_t* C3g = (GLU && !DUAL && KEEP) ? reinterpret_cast<uint16_t*>(p.C3) + static_cast<size_t>(e) * p.capacity * p.N : nullptr;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int m = m_base + i * 32 + r32;
        if (m >= count) continue;
#pragma unroll
        for (int j = 0; j < TO; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n_base + j * 32 + q * 8 + half * 4;
                if (n >= p.N) continue;
                const size_t o = static_cast<size_t>(m) * p.N + n;
                const f32x16& g0 = acc[i][j];
                if constexpr (GLU) {
                    const f32x16& g1 = acc[i][TO + j];
                    if constexpr (DUAL) {                           // both products, no activation
                        *reinterpret_cast<uint2*>(Cg + o) = pack_bf16x4(g0[q * 4], g0[q * 4 + 1], g0[q * 4 + 2], g0[q * 4 + 3]);
                        *reinterpret_cast<uint2*>(C2g + o) = pack_bf16x4(g1[q * 4], g1[q * 4 + 1], g1[q * 4 + 2], g1[q * 4 + 3]);
                    } else {
                        *reinterpret_cast<uint2*>(Cg + o) =
                            pack_bf16x4(silu(g0[q * 4]) * g1[q * 4], silu(g0[q * 4 + 1]) * g1[q * 4 + 1],
                                        silu(g0[q * 4 + 2]) * g1[q * 4 + 2], silu(g0[q * 4 + 3]) * g1[q * 4 + 3]);
                        if constexpr (KEEP) {                       // keep the pre-activations (training-mode forward)
                            *reinterpret_cast<uint2*>(C2g + o) = pack_bf16x4(g0[q * 4], g0[q * 4 + 1], g0[q * 4 + 2], g0[q * 4 + 3]);
                            *reinterpret_cast<uint2*>(C3g + o) = pack_bf16x4(g1[q * 4], g1[q * 4 + 1], g1[q * 4 + 2], g1[q * 4 + 3]);
                        }
                    }
                } else {
                    *reinterpret_cast<uint2*>(Cg + o) = pack_bf16x4(g0[q * 4], g0[q * 4 + 1], g0[q * 4 + 2], g0[q * 4 + 3]);
                }
            }
        __builtin_amdgcn_sched_barrier(0);               // one row of blocks at a time: keeps the live set small
    }
}

// Workgroup -> (expert, row tile, column tile).  Hardware deals consecutive workgroups round-robin
// to the 8 XCDs, each with its own 4 MiB L2 and 32 CUs.  Tiles are grouped into "super-tiles" of
// SM row tiles x SN column tiles (SM*SN = 32 = the workgroups that run together on one XCD); a whole
// super-tile goes to one XCD, so while its 32 workgroups stream along K together every token-row
// slice is shared by SN of them and every weight slice by SM of them through that XCD's L2.
__device__ __forceinline__ bool decode_tile(const GemmParams& p, int& e, int& mt, int& nt) {
    const int pid = blockIdx.x;
    const int xcd = pid & 7, j = pid >> 3;
    const int per = p.SM * p.SN;
    const int sidx = (j / per) * 8 + xcd, l = j % per;
    const int MG = (p.MT + p.SM - 1) / p.SM, NG = (p.NT + p.SN - 1) / p.SN;
    if (sidx >= p.E * MG * NG) return false;
    e = sidx / (MG * NG);
    const int r = sidx - e * (MG * NG);
    mt = (r % MG) * p.SM + l % p.SM;
    nt = (r / MG) * p.SN + l / p.SM;
    return mt < p.MT && nt < p.NT;
}

// The same for kernels with small tiles: only tiles that hold rows are counted (a scan over the groups, one lane each;
// G <= 64), and each XCD gets an equal, contiguous share of that list, row tiles fastest, so the tiles of one weight
// slice share an L2.  Dealing super-tiles of the capacity instead left XCDs with half-dead ones: 8 fp32 experts of
// 66-640 rows, gate/up product: 127 us against 92.
// by_chunks: groups of very unequal cost per tile (their own contraction lengths): chunks of 8 tiles go round the XCDs, so
// that each has its part of every group (weight gradients of 8 fp32 experts of 66-640 rows, one expert to an XCD: the training
// step 502 us, 486 so).  The grid is then whole 64s.
// What a small tile pays before its first load is latency, so the group's row count is handed back too, and the scan is in the vector
// unit (through LDS, and the count loaded again, 8 fp32 experts of 64 rows, 256 x 512: 10.6 and 8.2 us, now 9.5 and 7.4).
// j: place in the XCD's share, whose length is handed back.  With a workgroup for every tile of the capacity it is
// blockIdx.x / 8 and done; a smaller grid (whole rounds of 8 all the same) goes on in steps of gridDim.x / 8 to the end.
__device__ __forceinline__ bool decode_live_tile(const GemmParams& p, int BM, int j, int& share, int& e, int& mt, int& nt, int& count,
                                                 bool by_chunks = false) {
    const int lane = threadIdx.x & 63;
    const int rows_here = lane < p.E ? group_rows(p, lane) : 0;
    const int mine = max((rows_here + BM - 1) / BM, 0);  // this group's row tiles
    const int incl = wave_scan_incl(mine);
    const int total = __builtin_amdgcn_readlane(incl, 63) * p.NT;
    share = (total + 7) >> 3;
    if (by_chunks) share = (share + 7) & ~7;
    const int q = by_chunks ? ((j >> 3) * 8 + (blockIdx.x & 7)) * 8 + (j & 7) : (blockIdx.x & 7) * share + j;
    if (j >= share || q >= total) return false;
    const uint64_t in = __ballot(incl * p.NT > q);
    e = __builtin_ctzll(in);
    count = __builtin_amdgcn_readlane(rows_here, e);
    const int rows = __builtin_amdgcn_readlane(mine, e);
    const int u = q - (__builtin_amdgcn_readlane(incl, e) - rows) * p.NT;
    nt = u / rows;
    mt = u - nt * rows;
    return true;
}

// Fills MT, NT and the super-tile shape; returns the number of workgroups to launch.
// `wide`: the persistent kernel with 64-wide k-tiles, where a group has many row tiles (the 8-expert workload: 141):
// 8 row tiles x 4 column tiles, except where a row of column tiles is short and not a multiple of 4 (the 11 column
// tiles of that workload's gate/up product): then all of them in one super-tile, 2 x 11, so that no column group
// is left ragged.  Same box, whole layer: 7.42 -> 7.36 ms.  1 x 32 and 16 x 2 lose 3-8 % everywhere.
// With 5 to 8 row tiles per group a super-tile takes them all (5 x 6 ... 8 x 4): the weights are then fetched once, where 4 x 8
// leaves a second row of super-tiles with a tile or two to a weight slice.  5 row tiles, 16 experts, 4096 x 11008: 4277 -> 4243 us
// for the layer, 7.7-7.8 -> 6.0-6.8 GB fetched by the gate/up product, 3.61 -> 2.98 by the down product; 6, 32 experts, 4096 x 2816:
// 2731 -> 2720 us.
inline long long plan_tiles(GemmParams& p, int BM, int BN, bool wide = false) {
    p.MT = (p.capacity + BM - 1) / BM;
    p.NT = (p.N + BN - 1) / BN;
    if (wide && p.MT >= 16) {
        if (p.NT % 4 != 0 && p.NT <= 16) { p.SN = p.NT; p.SM = 32 / p.NT > 0 ? 32 / p.NT : 1; }
        else { p.SM = 8; p.SN = 4; }
        if (p.SM > p.MT) p.SM = p.MT;
    } else if (wide && p.MT > 4 && p.MT <= 8) {
        p.SM = p.MT;
        p.SN = 32 / p.SM;
    } else {
        p.SM = p.MT < 4 ? p.MT : 4;
        p.SN = 32 / p.SM;
    }
    if (p.SN > p.NT) p.SN = p.NT;
    const long long MG = (p.MT + p.SM - 1) / p.SM, NG = (p.NT + p.SN - 1) / p.SN;
    const long long supers = static_cast<long long>(p.E) * MG * NG;
    return (supers + 7) / 8 * 8 * (p.SM * p.SN);
}

// ---------------------------------------------------------------------------------------
// bf16 MFMA grouped GEMM:  C[e][m][n] = sum_k A[e][m][k] * B[e][n][k]   (+ SwiGLU epilogue)
// ---------------------------------------------------------------------------------------
template <int BM, int BN, int BK, int WGM, int WGN, bool GLU, int SWZ, bool DUAL = false>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_bf16_kernel(GemmParams p) {
    constexpr int NTH = WGM * WGN * 64;
    constexpr int BROWS = GLU ? 2 * BN : BN;       // weight rows staged per tile
    constexpr int CPR = BK / 8;                    // 16-byte chunks per tile row
    constexpr int WTM = BM / WGM, WTN = BN / WGN;  // per-wave output tile
    constexpr int TM = WTM / 32, TN = WTN / 32;    // 32x32 MFMA blocks per wave
    constexpr int NB = GLU ? 2 : 1;
    constexpr int A_CH = BM * CPR / NTH, B_CH = BROWS * CPR / NTH;
    static_assert(BM * CPR % NTH == 0 && BROWS * CPR % NTH == 0, "tile must divide over the threads");
    static_assert(WTM % 32 == 0 && WTN % 32 == 0 && BK % 16 == 0, "MFMA shape");

    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4* As = reinterpret_cast<uint4*>(lds_raw);                  // [2][BM][CPR]
    uint4* Bs = As + 2 * BM * CPR;                                  // [2][BROWS][CPR]

    int e, mt, nt;
    if (!decode_tile(p, e, mt, nt)) return;
    const int count = group_rows(p, e);
    const int m0 = mt * BM, n0 = nt * BN;
    if (m0 >= count) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave / WGN) * WTM, wn0 = (wave % WGN) * WTN;
    const int K = group_k(p, e);
    const int LA = (p.lda ? p.lda : p.K) / 8, LB = (p.ldb ? p.ldb : p.K) / 8;     // 16-byte chunks per operand row
    const uint4* Ag = reinterpret_cast<const uint4*>(p.A) + (p.row_index ? 0 : static_cast<size_t>(e) * p.capacity * LA);
    const uint4* B0g = reinterpret_cast<const uint4*>(p.B0) + static_cast<size_t>(e) * p.N * LB;
    const uint4* B1g = GLU ? reinterpret_cast<const uint4*>(p.B1) + static_cast<size_t>(e) * p.N * LB : nullptr;

    // per-thread staging slots: chunk q -> (row, ck)
    const uint4* a_src[A_CH];
    const uint4* b_src[B_CH];
    int a_dst[A_CH], b_dst[B_CH], a_ck[A_CH], b_ck[B_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        const int q = tid + i * NTH, row = q / CPR, ck = q % CPR;
        int m = m0 + row;
        m = m < p.capacity ? m : p.capacity - 1;                   // stay inside the buffer; such rows are never stored
        if (p.row_index) m = min(max(p.row_index[static_cast<size_t>(e) * p.capacity + m], 0), p.a_rows - 1);
        a_src[i] = Ag + static_cast<size_t>(m) * LA + ck;
        a_dst[i] = row * CPR + (ck ^ ((row >> SWZ) & (CPR - 1)));
        a_ck[i] = ck;
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        const int q = tid + i * NTH, row = q / CPR, ck = q % CPR;
        const bool up = GLU && row >= BN;
        int n = n0 + (up ? row - BN : row);
        n = n < p.N ? n : p.N - 1;
        b_src[i] = (up ? B1g : B0g) + static_cast<size_t>(n) * LB + ck;
        b_dst[i] = row * CPR + (ck ^ ((row >> SWZ) & (CPR - 1)));
        b_ck[i] = ck;
    }

    f32x16 acc[NB][TM][TN];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][i][j][v] = 0.f;

    uint4 ra[A_CH], rb[B_CH];
    const int KC = K / 8;                          // chunks per full row
    auto load_global = [&](int kt) {
        const int kc0 = kt * CPR;
#pragma unroll
        for (int i = 0; i < A_CH; ++i)
            ra[i] = (kc0 + a_ck[i] < KC) ? a_src[i][kc0] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int i = 0; i < B_CH; ++i)
            rb[i] = (kc0 + b_ck[i] < KC) ? b_src[i][kc0] : make_uint4(0u, 0u, 0u, 0u);
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) As[buf * BM * CPR + a_dst[i]] = ra[i];
#pragma unroll
        for (int i = 0; i < B_CH; ++i) Bs[buf * BROWS * CPR + b_dst[i]] = rb[i];
    };

    const int KT = (K + BK - 1) / BK;
    load_global(0);                                 // (all zeros when K == 0)
    store_lds(0);
    __syncthreads();

    const int r32 = lane & 31, half = lane >> 5;
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < KT) load_global(kt + 1);
        const uint4* Ab = As + cur * BM * CPR;
        const uint4* Bb = Bs + cur * BROWS * CPR;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int ck = ks * 2 + half;
            bf16x8 af[TM], bfr[NB][TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm0 + i * 32 + r32;
                af[i] = __builtin_bit_cast(bf16x8, Ab[row * CPR + (ck ^ ((row >> SWZ) & (CPR - 1)))]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int row = b * BN + wn0 + j * 32 + r32;
                    bfr[b][j] = __builtin_bit_cast(bf16x8, Bb[row * CPR + (ck ^ ((row >> SWZ) & (CPR - 1)))]);
                }
            // D[n][m] += W[n][k] * X[m][k]: the weight fragment is the row operand, so a lane
            // ends up with 4 consecutive output columns n of one row m (8-byte stores).
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[b][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[b][j], af[i], acc[b][i][j], 0, 0, 0);
        }
        if (kt + 1 < KT) store_lds(cur ^ 1);
        __syncthreads();
    }

    // epilogue: lane holds, per 32x32 block, row m = lane%32 and columns (v/4)*8 + (lane/32)*4 + v%4
    uint16_t* Cg = reinterpret_cast<uint16_t*>(p.C) + static_cast<size_t>(e) * p.capacity * p.N;
    uint16_t* C2g = DUAL ? reinterpret_cast<uint16_t*>(p.C2) + static_cast<size_t>(e) * p.capacity * p.N : nullptr;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm0 + i * 32 + r32;
        if (m >= count) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wn0 + j * 32 + q * 8 + half * 4;
                if (n >= p.N) continue;
                const f32x16& g0 = acc[0][i][j];
                const f32x16& g1 = acc[NB - 1][i][j];
                float o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if constexpr (GLU && !DUAL) o[v] = silu(g0[q * 4 + v]) * g1[q * 4 + v];
                    else o[v] = g0[q * 4 + v];
                }
                *reinterpret_cast<uint2*>(Cg + static_cast<size_t>(m) * p.N + n) = pack_bf16x4(o[0], o[1], o[2], o[3]);
                if constexpr (GLU && DUAL)
                    *reinterpret_cast<uint2*>(C2g + static_cast<size_t>(m) * p.N + n) =
                        pack_bf16x4(g1[q * 4], g1[q * 4 + 1], g1[q * 4 + 2], g1[q * 4 + 3]);
                if constexpr (GLU && !DUAL) {
                    if (p.C3) {                                     // keep the pre-activations (training-mode forward)
                        const size_t o3 = (static_cast<size_t>(e) * p.capacity + m) * p.N + n;
                        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.C2) + o3) =
                            pack_bf16x4(g0[q * 4], g0[q * 4 + 1], g0[q * 4 + 2], g0[q * 4 + 3]);
                        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.C3) + o3) =
                            pack_bf16x4(g1[q * 4], g1[q * 4 + 1], g1[q * 4 + 2], g1[q * 4 + 3]);
                    }
                }
            }
    }
}

// The epilogue of the persistent 64-wide kernel: the output passes through a small per-wave LDS patch, so that
// memory sees whole or half lines of a row instead of 8-byte pieces.  In the accumulator layout a lane owns four
// consecutive columns of one row, so a direct store instruction writes 16 rows x 32 bytes (32 x 16 with the
// 32x32x16 accumulators this was first built for): for a 256 x 256 tile that is thousands of write requests next to
// the 512 read requests of each k-step, a third of all requests of a product with a short contraction.  Here a
// 32 x 32 block is written to LDS as it lies in the registers (row stride 80 bytes), read back with four lanes per
// row (16 bytes each) and stored as 16 rows x 64 bytes per instruction (measured when it went in: the down
// projection of the 8-expert workload, whose contraction is 22 k-steps, 1009 -> 1119 TFLOP/s; 1-4 % elsewhere).
// The patch belongs to the wave (LDS instructions of one wave execute in order), so there is no barrier.  Requires
// whole column tiles (no column mask).
constexpr int kStageStride = 80;                         // bytes per staged row: 64 of data + 16 so that rows spread over the banks
constexpr int kStageBytes = 32 * kStageStride;           // per wave

// The patch is written and read back in assembly.  Through ordinary LDS accesses the compiler puts a vmcnt(0) in
// front of every one of them while asynchronous copies into LDS are in flight (it cannot tell that the next tile's
// k-tiles land elsewhere), and that wait also covers the stores this epilogue has just issued: every block then
// waited for the previous block's stores to reach memory, 4-7 thousand cycles per tile.  LDS instructions of one
// wave execute in order, so a write followed by a read needs no wait in between; each statement ends with its
// own lgkmcnt(0), so its outputs are ordinary, fully written registers.
typedef int epi_v2i __attribute__((ext_vector_type(2)));
typedef int epi_v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}
__device__ __forceinline__ epi_v2i as_v2i(const uint2& v) { return epi_v2i{static_cast<int>(v.x), static_cast<int>(v.y)}; }
__device__ __forceinline__ uint4 as_uint4(const epi_v4i& v) {
    return make_uint4(static_cast<uint32_t>(v.x), static_cast<uint32_t>(v.y), static_cast<uint32_t>(v.z), static_cast<uint32_t>(v.w));
}

// One 32 x 32 output block = four 16 x 16 accumulators (bi, bj) of v_mfma_f32_16x16x32_bf16; in each, lane l holds
// row 16 bi + l % 16 and the four columns 16 bj + 4 (l / 16) .. + 3: pk[2 bi + bj] is that group packed.
// dst = the block's first element.
__device__ __forceinline__ void store_block_staged16(const uint2 (&pk)[4], uint16_t* dst, int ldc, int rows_live,
                                                     unsigned char* stage, int lane) {
    const int l16 = lane & 15, kq = lane >> 4;
    const uint32_t wa = lds_address(stage) + l16 * kStageStride + kq * 8;          // + 32 bj + 16 rows * bi
    const uint32_t ra = lds_address(stage) + (lane >> 2) * kStageStride + (lane & 3) * 16;
    epi_v4i v0, v1;
    static_assert(16 * kStageStride == 1280, "offsets in the statement below");
    asm volatile(
        "ds_write_b64 %2, %4\n\t"
        "ds_write_b64 %2, %5 offset:32\n\t"
        "ds_write_b64 %2, %6 offset:1280\n\t"
        "ds_write_b64 %2, %7 offset:1312\n\t"
        "ds_read_b128 %0, %3\n\t"
        "ds_read_b128 %1, %3 offset:1280\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v0), "=&v"(v1)
        : "v"(wa), "v"(ra), "v"(as_v2i(pk[0])), "v"(as_v2i(pk[1])), "v"(as_v2i(pk[2])), "v"(as_v2i(pk[3]))
        : "memory");
    const int row = lane >> 2, ch = lane & 3;
    if (row < rows_live) *reinterpret_cast<uint4*>(dst + static_cast<size_t>(row) * ldc + ch * 8) = as_uint4(v0);
    if (row + 16 < rows_live) *reinterpret_cast<uint4*>(dst + static_cast<size_t>(row + 16) * ldc + ch * 8) = as_uint4(v1);
}

// Two horizontally adjacent 32 x 32 blocks (64 columns = one 128-byte line per row), 16 rows at a time (row stride
// 144 bytes): eight lanes read one row back and a store instruction writes 8 rows x 128 bytes, whole lines (down
// projection of the 8-expert workload another 1.5 % over the 64-byte pieces).
constexpr int kPairStride = 144;
static_assert(16 * kPairStride <= kStageBytes, "the pair patch must fit the per-wave patch");
__device__ __forceinline__ void store_block_pair_staged16(const uint2 (&pk0)[4], const uint2 (&pk1)[4], uint16_t* dst, int ldc,
                                                          int rows_live, unsigned char* stage, int lane) {
    const int l16 = lane & 15, kq = lane >> 4;
    const uint32_t wa = lds_address(stage) + l16 * kPairStride + kq * 8;
    const uint32_t ra = lds_address(stage) + (lane >> 3) * kPairStride + (lane & 7) * 16;
    static_assert(8 * kPairStride == 1152, "offset in the statement below");
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {                // rows 16 pass .. + 15: every lane owns a piece of them
        epi_v4i v0, v1;
        asm volatile(
            "ds_write_b64 %2, %4\n\t"
            "ds_write_b64 %2, %5 offset:32\n\t"
            "ds_write_b64 %2, %6 offset:64\n\t"
            "ds_write_b64 %2, %7 offset:96\n\t"
            "ds_read_b128 %0, %3\n\t"
            "ds_read_b128 %1, %3 offset:1152\n\t"
            "s_waitcnt lgkmcnt(0)"
            : "=&v"(v0), "=&v"(v1)
            : "v"(wa), "v"(ra), "v"(as_v2i(pk0[pass * 2])), "v"(as_v2i(pk0[pass * 2 + 1])), "v"(as_v2i(pk1[pass * 2])),
              "v"(as_v2i(pk1[pass * 2 + 1]))
            : "memory");
        const int r = pass * 16 + (lane >> 3), ch = lane & 7;
        if (r < rows_live) *reinterpret_cast<uint4*>(dst + static_cast<size_t>(r) * ldc + ch * 8) = as_uint4(v0);
        if (r + 8 < rows_live) *reinterpret_cast<uint4*>(dst + static_cast<size_t>(r + 8) * ldc + ch * 8) = as_uint4(v1);
    }
}
// acc[i][j]: token block i (16 rows) x weight block j (16 rows of the staged weights; SwiGLU: 0, 1 gate and 2, 3 up
// rows of the same 32 columns; plain: 64 columns)
template <bool GLU, bool DUAL, bool KEEP = false>
__device__ __forceinline__ void store_blocks_staged16(const GemmParams& p, const f32x4 (&acc)[8][4], int e, int m_base,
                                                      int n_base, int count, int lane, unsigned char* stage) {
    const size_t eoff = static_cast<size_t>(e) * p.capacity * p.N;
    uint16_t* Cg = reinterpret_cast<uint16_t*>(p.C) + eoff;
    uint16_t* C2g = (GLU && (DUAL || KEEP)) ? reinterpret_cast<uint16_t*>(p.C2) + eoff : nullptr;
    uint16_t* C3g = (GLU && !DUAL && KEEP) ? reinterpret_cast<uint16_t*>(p.C3) + eoff : nullptr;
    auto pack4 = [](const f32x4& v) { return pack_bf16x4(v[0], v[1], v[2], v[3]); };
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
        const int mb = m_base + ib * 32;
        const int live = count - mb;
        if (live <= 0) continue;                         // wave-uniform
        const size_t o = static_cast<size_t>(mb) * p.N + n_base;
        uint2 pk[4], pk1[4];
        if constexpr (!GLU) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                pk[b] = pack4(acc[2 * ib + (b >> 1)][b & 1]);
                pk1[b] = pack4(acc[2 * ib + (b >> 1)][2 + (b & 1)]);
            }
            store_block_pair_staged16(pk, pk1, Cg + o, p.N, live, stage, lane);
        } else {
            if constexpr (!DUAL) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const f32x4& g0 = acc[2 * ib + (b >> 1)][b & 1];
                    const f32x4& g1 = acc[2 * ib + (b >> 1)][2 + (b & 1)];
                    pk[b] = pack_bf16x4(silu(g0[0]) * g1[0], silu(g0[1]) * g1[1], silu(g0[2]) * g1[2], silu(g0[3]) * g1[3]);
                }
            } else {
#pragma unroll
                for (int b = 0; b < 4; ++b) pk[b] = pack4(acc[2 * ib + (b >> 1)][b & 1]);
            }
            store_block_staged16(pk, Cg + o, p.N, live, stage, lane);
            if constexpr (DUAL || KEEP) {                    // the two products themselves
                if constexpr (KEEP) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) pk[b] = pack4(acc[2 * ib + (b >> 1)][b & 1]);
                    store_block_staged16(pk, C2g + o, p.N, live, stage, lane);
                }
#pragma unroll
                for (int b = 0; b < 4; ++b) pk[b] = pack4(acc[2 * ib + (b >> 1)][2 + (b & 1)]);
                store_block_staged16(pk, (KEEP ? C3g : C2g) + o, p.N, live, stage, lane);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The epilogue of the transposing persistent kernel: 32 rows x 64 columns of a wave (pk[bi][bj]: its 16 x 16 accumulators
// packed, lane: row 16 bi + l % 16 and the four columns 16 bj + 4 (l / 16) .. + 3) pass through LDS and leave as whole
// 128-byte lines, 8 rows per instruction.  Stored directly an instruction would write 32 bytes of 16 rows; a weight
// gradient, whose contraction is an expert's few hundred rows, then spends as long storing its tile as multiplying it.
// The patch is four pieces of 1 KiB, 8 KiB apart (8 rows x 128 bytes each): the wave's own copy target, see the kernel.  The
// 16-byte pieces of a row are XORed with the row (no padding fits): two-way bank conflicts on the writes, none on the
// reads.  In assembly for the reason given above.  N % 8 == 0: a 16-byte piece is all in or all out.
// v[u]: row 8 u + lane / 8, columns 8 (lane % 8) .. + 7
__device__ __forceinline__ void rows_through_patch(const uint2 (&pk)[2][4], uint32_t patch, int lane, epi_v4i (&v)[4]) {
    const int l16 = lane & 15, kq = lane >> 4;
    const uint32_t wbase = patch + (l16 >> 3) * 8192 + (l16 & 7) * 128 + (kq & 1) * 8;
    uint32_t wa[4];
#pragma unroll
    for (int bj = 0; bj < 4; ++bj) wa[bj] = wbase + (((2 * bj + (kq >> 1)) ^ (l16 & 7)) * 16);
    const int rr = lane >> 3, ch = lane & 7;
    const uint32_t ra = patch + rr * 128 + ((ch ^ rr) * 16);
    asm volatile(
        "ds_write_b64 %4, %9\n\t"
        "ds_write_b64 %5, %10\n\t"
        "ds_write_b64 %6, %11\n\t"
        "ds_write_b64 %7, %12\n\t"
        "ds_write_b64 %4, %13 offset:16384\n\t"
        "ds_write_b64 %5, %14 offset:16384\n\t"
        "ds_write_b64 %6, %15 offset:16384\n\t"
        "ds_write_b64 %7, %16 offset:16384\n\t"
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:8192\n\t"
        "ds_read_b128 %2, %8 offset:16384\n\t"
        "ds_read_b128 %3, %8 offset:24576\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
        : "v"(wa[0]), "v"(wa[1]), "v"(wa[2]), "v"(wa[3]), "v"(ra), "v"(as_v2i(pk[0][0])), "v"(as_v2i(pk[0][1])),
          "v"(as_v2i(pk[0][2])), "v"(as_v2i(pk[0][3])), "v"(as_v2i(pk[1][0])), "v"(as_v2i(pk[1][1])), "v"(as_v2i(pk[1][2])),
          "v"(as_v2i(pk[1][3]))
        : "memory");
}
__device__ __forceinline__ void store_rows_staged_lines(const uint2 (&pk)[2][4], uint16_t* dst, int ldc, int rows_live, int cols_live,
                                                        uint32_t patch, int lane) {
    epi_v4i v[4];
    rows_through_patch(pk, patch, lane, v);
    const int rr = lane >> 3, ch = lane & 7;
    const bool col = ch * 8 < cols_live;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = 8 * u + rr;
        if (col && r < rows_live) *reinterpret_cast<uint4*>(dst + static_cast<size_t>(r) * ldc + ch * 8) = as_uint4(v[u]);
    }
}

// s_waitcnt immediate: vmcnt(n) (6 bits, split 3:0 and 15:14), expcnt untouched, lgkmcnt(0) or untouched
constexpr int waitcnt_imm(int vm, bool lgkm0) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lgkm0 ? 0 : 0x0F00); }

// Buffer descriptors: the range of one that bounds nothing that exists, and an offset past any range (see buffer_copy_to_lds)
constexpr uint32_t kBufferRange = 0xFFFFFF00u, kPastRange = 0xFFFFFF80u;

// v of the lane whose number differs in bit M (1, 2 or 4), in the vector unit; all lanes active
template <int M>
__device__ __forceinline__ float lane_xor(float v) {
    const int u = __builtin_bit_cast(int, v);
    int o;
    if constexpr (M == 4) o = __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, u, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else o = __builtin_amdgcn_update_dpp(0, u, M == 2 ? 0x4E : 0xB1, 0xF, 0xF, true);
    return __builtin_bit_cast(float, o);
}

// The epilogue of the product u = dOut_p Wd in the backward: the element-wise middle (see backward.hip) on the wave's 128 rows x
// 64 columns while they are in registers.  u, rounded to bf16, passes through the patch into whole lines as above; a and b of the
// same piece are loaded beside it, a block of 32 rows ahead, and da, db and h leave as whole lines.  gates: LDS address of the
// weights of the wave's rows.
// Bound by the vector unit (25 issue slots an element, 8 of them the exponential and the reciprocal) and by the 640 KiB that a tile
// moves, with the matrix pipe idle: some 20 us a tile.  A pass of its own, which also writes and reads u, took longer.  Training
// step, pass / this: 16 experts of 166-1024 rows, 2048 x 5632: 2634 / 2575 us; 12 of 677, 1080 x 2744: 910 / 877; 8 of 32 000,
// 4096 x 1408: 23525 / 23120; 8 of 512, 896 x 5248: 560 / 557.  Where its tiles leave CUs idle see middle_in_product.
// Not kept: waits counted by hand instead of the compiler's (the same); workgroups with a tile less than others half a tile behind
// them, so that not all epilogues meet in memory (0-2 % of the product).
__device__ __forceinline__ void store_middle(const GemmParams& p, const f32x4 (&acc)[8][4], int e, int m_base, int nb, int count, uint32_t gates,
                                             uint32_t patch, int lane) {
    if (nb >= p.N || m_base >= count) return;            // wave-uniform
    asm volatile("" : "+v"(lane));                       // (what depends on it is not worth registers of the loop over k-tiles)
    const int rr = lane >> 3, ch = lane & 7, N = p.N;
    const bool col = nb + ch * 8 < N;
    typedef __attribute__((address_space(1))) char* global_bytes;
    typedef const __attribute__((address_space(1))) epi_v4i* global_piece;
    auto uniform = [](const void* base, size_t bytes) -> uint64_t {
        const uint64_t b = reinterpret_cast<uint64_t>(base) + bytes;
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32));
        return (static_cast<uint64_t>(hi) << 32) | lo;
    };
    // Stores through a descriptor of each of the group's outputs: a lane that has nothing to store asks for an offset past it.
    // (Byte offsets inside a group fit 32 bits: a launch condition.)
    auto output = [&](const void* base, size_t before, size_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform(base, before)), 0, static_cast<int>(bytes), 0x00027000);
    };
    const size_t in_bytes = static_cast<size_t>(p.capacity) * N * 2, out_bytes = static_cast<size_t>(p.mid_rows) * N * 2;
    const global_bytes a_base = (global_bytes)uniform(p.mid_a, e * in_bytes), b_base = (global_bytes)uniform(p.mid_b, e * in_bytes);
    const __amdgpu_buffer_rsrc_t dab = output(p.C, 2 * e * out_bytes, 2 * out_bytes), hid = output(p.C2, e * out_bytes, out_bytes);
    const __amdgpu_buffer_rsrc_t part = output(p.mid_part, (static_cast<size_t>(nb >> 6) * p.E + e) * p.capacity * 4, static_cast<size_t>(p.capacity) * 4);
    // byte offsets of this lane's row m_base + rr and of its piece (a lane past the row repeats the first one; never stored)
    const uint32_t lane_row = static_cast<uint32_t>(m_base + rr) * N * 2u, piece = (nb + (col ? ch * 8 : 0)) * 2u;
    const uint32_t last_row = static_cast<uint32_t>(count - 1) * N * 2u;
    epi_v4i av[4], bv[4];
    auto request = [&](int ib, int u) {
        const uint32_t off = min(lane_row + (ib * 32 + 8 * u) * 2u * N, last_row) + piece;
        av[u] = *(global_piece)(a_base + off);
        bv[u] = *(global_piece)(b_base + off);
    };
#pragma unroll
    for (int u = 0; u < 4; ++u) request(0, u);
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
        const int mb = m_base + ib * 32;
        if (mb >= count) break;                          // wave-uniform
        uint2 pk[2][4];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 4; ++bj) {
                const f32x4& v = acc[2 * ib + bi][bj];
                pk[bi][bj] = pack_bf16x4(v[0], v[1], v[2], v[3]);
            }
        epi_v4i uv[4];
        rows_through_patch(pk, patch, lane, uv);
        float gv[4];
        asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:32\n\tds_read_b32 %2, %4 offset:64\n\tds_read_b32 %3, %4 offset:96\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(gv[0]), "=&v"(gv[1]), "=&v"(gv[2]), "=&v"(gv[3]) : "v"(gates + (ib * 32 + rr) * 4) : "memory");
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int m = mb + 8 * u + rr;
            const float gate = gv[u], h_scale = p.mid_scale_h ? gate : 1.0f;
            float dot = 0.f;
            uint32_t da[4], db[4], hh[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                float fda[2], fdb[2], fh[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    auto half = [&](int word) { return __uint_as_float(j ? static_cast<uint32_t>(word) & 0xFFFF0000u : static_cast<uint32_t>(word) << 16); };
                    const float uf = half(uv[u][w]), af = half(av[u][w]), bf = half(bv[u][w]);
                    const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504088896341f * af));
                    const float sl = af * sg, h = sl * bf, dh = gate * uf;
                    fda[j] = dh * bf * (sg * (1.0f + af * (1.0f - sg)));
                    fdb[j] = dh * sl;
                    dot += uf * h;
                    fh[j] = h * h_scale;
                }
                da[w] = pack_bf16(fda[0], fda[1]);
                db[w] = pack_bf16(fdb[0], fdb[1]);
                hh[w] = pack_bf16(fh[0], fh[1]);
            }
            if (ib < 3) request(ib + 1, u);              // (in front of this piece's stores)
            dot = col ? dot : 0.f;                       // added up over the eight lanes of a row
            dot += lane_xor<4>(dot);
            dot += lane_xor<2>(dot);
            dot += lane_xor<1>(dot);
            const uint32_t row = lane_row + (ib * 32 + 8 * u) * 2u * N;
            auto put = [&](const __amdgpu_buffer_rsrc_t& rsrc, uint32_t off, const uint32_t (&v)[4]) {
                typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0], v[1], v[2], v[3]}, rsrc, static_cast<int>(col && m < count ? off : kPastRange), 0, 0);
            };
            put(dab, 2 * row + piece, da);
            put(dab, 2 * row + piece + 2u * N, db);
            put(hid, row + piece, hh);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dot), part, static_cast<int>(m < count && ch == 0 ? m * 4u : kPastRange), 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

typedef const __attribute__((address_space(1))) void* global_cptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

__device__ __align__(16) const float kZeroPiece[4] = {0.f, 0.f, 0.f, 0.f};

// A copy into LDS through a buffer descriptor: a scalar base and a 32-bit offset per lane, no 64-bit address in vector
// registers (and not the flat form, behind which the compiler cannot count its waits).  In a ragged contraction a copy
// cannot be masked per lane without leaving stale data behind, so the lanes whose 16-byte piece lies past the end ask for an
// offset past the descriptor's range: such a lane reads nothing and zeros land in its LDS slot.  The descriptor spans all but
// the last 256 bytes of 4 GiB from the tile's base; real offsets stay below it (a launch condition), so the check never
// touches a piece that exists.
__device__ __forceinline__ void buffer_copy_to_lds(uint32_t base_lo, uint32_t base_hi, uint32_t off, uint4* dst) {
    void* base = reinterpret_cast<void*>((static_cast<uint64_t>(base_hi) << 32) | base_lo);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, static_cast<int>(kBufferRange), 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)dst, 16, static_cast<int>(off), 0, 0, 0);
}

// ---------------------------------------------------------------------------------------
// Pipelined bf16 MFMA grouped GEMM (launched for K % 64 == 0; one workgroup per tile; the fall-back of the
// persistent kernels below): 256 x 256 staged rows, BK = 32, a ring of four 32 KiB LDS buffers.
//   * global -> LDS copies bypass the registers (global_load_lds_dwordx4); the XOR swizzle is
//     applied on the source side (lane l fetches the chunk that belongs in LDS slot l);
//   * the copies of tile kt+3 are spread one by one between the MFMAs of iteration kt (a copy
//     issued in a burst blocks the wave's MFMA issue for about 25 cycles each), and they have two
//     full iterations to land: before barrier(kt) a wave waits only until at most 12 copies are
//     outstanding (s_waitcnt vmcnt(12)), i.e. until its share of tile kt+1 is in LDS;
//   * MFMA operands are double-buffered in registers: the ds_reads of k-substep s+1 are issued
//     before the MFMAs of substep s; one barrier per iteration.
// With GLU the 256 staged weight rows are 128 gate rows + 128 up rows of the same output columns
// and the epilogue is SiLU(gate)*up.  With row_index the A rows are gathered straight from the
// token matrix (dispatch folded into the load).
// ---------------------------------------------------------------------------------------

template <bool GLU, int WN = 2, bool DUAL = false, int NBUF = 4>
__global__ __launch_bounds__(128 * WN) void gemm_bf16_ring_kernel(GemmParams p) {
    constexpr int BM = 256, BR = 256, CPR = 4;
    constexpr int BN = GLU ? 128 : 256;
    constexpr int STAGE = (BM + BR) * CPR;              // uint4 per LDS buffer (32 KiB)
    constexpr int NW = 2 * WN;                          // waves: 2 row groups x WN column groups
    constexpr int TB = 4 / (WN / 2);                    // weight fragments per wave and k-substep (4 or 2)
    constexpr int NCP = 16 / NW;                        // row groups (of 16 rows) each wave copies per operand
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4* lds = reinterpret_cast<uint4*>(lds_raw);

    int e, mt, nt;
    if (!decode_tile(p, e, mt, nt)) return;
    const int count = group_rows(p, e);
    const int m0 = mt * BM, n0 = nt * BN;
    if (m0 >= count) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r32 = lane & 31, half = lane >> 5;
    const int KCA = (p.lda ? p.lda : p.K) / 8, KCB = (p.ldb ? p.ldb : p.K) / 8;   // 16-byte chunks per operand row
    const int KT = group_k(p, e) / 32;

    // ---- copy sources: wave w fills row groups w*NCP .. (16 rows x 4 chunks = 1 KiB each)
    // Addresses are a wave-uniform 64-bit base (scalar registers, advanced by 64 bytes per tile)
    // plus a per-lane 32-bit byte offset that never changes (the host checks that it fits).
    const char* Abase = reinterpret_cast<const char*>(p.A) +
                        (p.row_index ? 0 : static_cast<size_t>(e) * p.capacity * KCA * 16);
    const char* Bbase = reinterpret_cast<const char*>((GLU && wave >= NW / 2) ? p.B1 : p.B0) +
                        static_cast<size_t>(e) * p.N * KCB * 16;
    uint32_t off[2 * NCP];                              // first NCP: A groups, then B groups
#pragma unroll
    for (int i = 0; i < NCP; ++i) {
        const int r = (wave * NCP + i) * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((r >> 2) & 3);
        int m = m0 + r;
        m = m < count ? m : count - 1;                   // rows past the count replay a valid row; never stored
        const int row = p.row_index ? min(max(p.row_index[static_cast<size_t>(e) * p.capacity + m], 0), p.a_rows - 1) : m;
        off[i] = (static_cast<uint32_t>(row) * KCA + c) * 16u;
        int n = n0 + (GLU ? (r & 127) : r);
        n = n < p.N ? n : p.N - 1;
        off[NCP + i] = (static_cast<uint32_t>(n) * KCB + c) * 16u;
    }
    auto issue_copy = [&](int kt, int j) {
        uint4* dst = lds + (kt % NBUF) * STAGE + (j / NCP) * (BM * CPR) + (wave * NCP + (j % NCP)) * 64;
        // re-materialise the tile base as a scalar every time, so that the address stays
        // "scalar base + 32-bit lane offset" instead of a per-lane 64-bit pointer
        const uint64_t b64 = reinterpret_cast<uint64_t>(j < NCP ? Abase : Bbase) + static_cast<uint64_t>(kt) * (CPR * 16);
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32));
        const char* base = reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
        __builtin_amdgcn_global_load_lds((global_cptr)(base + off[j]), (lds_ptr)dst, 16, 0, 0);
    };

    const int sw = (r32 >> 2) & 3;
    int a_row[4], b_row[TB];
#pragma unroll
    for (int i = 0; i < 4; ++i) a_row[i] = (wm * 128 + i * 32 + r32) * CPR;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
        const int br = GLU ? ((j / (TB / 2)) * 128 + wn * (16 * TB) + (j % (TB / 2)) * 32) : (wn * (32 * TB) + j * 32);
        b_row[j] = BM * CPR + (br + r32) * CPR;
    }
    const int ck0 = half ^ sw, ck1 = (2 + half) ^ sw;

    f32x16 acc[4][TB];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    bf16x8 fa[2][4], fb[2][TB];
    auto load_frags = [&](int set, int kt, int ck) {
        const uint4* base = lds + (kt % NBUF) * STAGE + ck;
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[set][i] = __builtin_bit_cast(bf16x8, base[a_row[i]]);
#pragma unroll
        for (int j = 0; j < TB; ++j) fb[set][j] = __builtin_bit_cast(bf16x8, base[b_row[j]]);
    };
    // the MFMAs of one k-substep; with `copy`, NCP copies of tile kt_copy go in between, one per 4 MFMAs
    auto mfma_step = [&](int set, bool copy, int kt_copy, int j0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < TB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
            if (copy && (i + 1) % (4 / NCP) == 0) issue_copy(kt_copy, j0 + i / (4 / NCP));
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- prologue: NBUF - 1 tiles in flight, wait for the first
    constexpr int AHEAD = NBUF - 1;
    const int pre = KT < AHEAD ? KT : AHEAD;
    for (int t = 0; t < pre; ++t)
#pragma unroll
        for (int j = 0; j < 2 * NCP; ++j) issue_copy(t, j);
    if (pre == AHEAD) __builtin_amdgcn_s_waitcnt(waitcnt_imm((AHEAD - 1) * 2 * NCP, false));
    else if (pre == 3) __builtin_amdgcn_s_waitcnt(waitcnt_imm(4 * NCP, false));
    else if (pre == 2) __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * NCP, false));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
    __builtin_amdgcn_s_barrier();
    load_frags(0, 0, ck0);

    int kt = 0;
    for (; kt + AHEAD < KT; ++kt) {                          // steady state: tile kt+AHEAD is being fetched
        __builtin_amdgcn_sched_barrier(0);
        load_frags(1, kt, ck1);
        mfma_step(0, true, kt + AHEAD, 0);
        // tile kt+1 is in LDS once at most tiles kt+2 .. kt+AHEAD-1 and half of kt+AHEAD are outstanding
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((2 * (AHEAD - 2) + 1) * NCP, true));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        load_frags(0, kt + 1, ck0);
        mfma_step(1, true, kt + AHEAD, NCP);
    }
    for (; kt < KT; ++kt) {                                  // drain: nothing left to fetch
        __builtin_amdgcn_sched_barrier(0);
        load_frags(1, kt, ck1);
        mfma_step(0, false, 0, 0);
        __builtin_amdgcn_s_waitcnt(0x0070);                  // vmcnt(0) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 1 < KT) load_frags(0, kt + 1, ck0);
        mfma_step(1, false, 0, 0);
    }

    constexpr int TO = GLU ? TB / 2 : TB;
    if (GLU && !DUAL && p.C3) store_blocks<GLU, DUAL, 4, TB, GLU && !DUAL>(p, acc, e, m0 + wm * 128, n0 + wn * (32 * TO), count, r32, half);
    else store_blocks<GLU, DUAL, 4, TB>(p, acc, e, m0 + wm * 128, n0 + wn * (32 * TO), count, r32, half);
}

// ---------------------------------------------------------------------------------------
// Persistent kernels: one workgroup per CU walks a list of tiles, and the copies run on across tile boundaries: while the
// last k-tiles of one tile are multiplied the first k-tiles of the next are already being fetched, and the stores of the
// epilogue overlap with them.  (A workgroup per tile pays launch, address set-up, the first-tile latency and the epilogue
// with the matrix pipe idle: about 5 us per tile, 5-10 % at K = 2048.)
//
// Tile list: only tiles that hold rows (m0 < counts[e]) are enumerated, super-tile by super-tile
// (see decode_tile), from an exclusive prefix over the super-tiles that every workgroup builds in
// LDS at start.  Consecutive groups of gridDim.x / 8 tiles go round-robin to the 8 XCDs, so the
// tiles that run together on one XCD are still (pieces of) one super-tile and share operand
// slices through its L2, and every workgroup gets the same number of tiles +- 1.
// No atomics, no flags: the schedule is a pure function of counts[].
// ---------------------------------------------------------------------------------------
constexpr int kMaxSuper = 4096;          // super-tiles the LDS prefix of the transposing kernel can hold (16 KiB)
constexpr int kMaxSuperWide = 2048;      // the same for the row-major kernel, whose epilogue patches leave less room

// a / d for 0 <= a < 2^20, d >= 1: (a + 1/2) / d is at least 1 / (2 d) away from a whole number, more than the reciprocal and
// the product round off.  For wave-uniform operands.  (The empty statements keep the reciprocal out of loops and the result
// in a scalar register; either would hold a vector register of the kernels' 256.)
__device__ __forceinline__ int small_div(int a, int d) {
    d = __builtin_amdgcn_readfirstlane(d);
    asm volatile("" : "+s"(d));
    int q = static_cast<int>((static_cast<float>(a) + 0.5f) * __builtin_amdgcn_rcpf(static_cast<float>(d)));
    asm volatile("" : "+v"(q));
    return __builtin_amdgcn_readfirstlane(q);
}

// The list of live tiles.  Nothing here touches global memory once the list is built: a load in the tile set-up would wait
// for every copy in flight and for the stores of the epilogue before it.  The rows and k-tiles of the groups (E <= 64) lie in LDS
// beside the prefix; the super-tile of the next tile is found by one ballot over 64 entries, as a workgroup's tiles ascend.
struct LiveTiles {
    const int* pre;              // pre[s] = number of live tiles in the super-tiles before s (s <= S)
    const int* rows;             // rows of each group, then its k-tiles
    int BM, MG, NG, S, total;
    int s = 0, first = 0;        // super-tile of the tile found last, and its first tile's place in the list

    __device__ __forceinline__ static int live_rows(const GemmParams& p, int count, int mg, int BM) {
        return min(max((count + BM - 1) / BM - mg * p.SM, 0), p.SM);
    }
    // by NTH threads, with LDS for S + 1, NTH / 64 and 128 numbers
    template <int NTH>
    __device__ __forceinline__ void build(const GemmParams& p, int tile_rows, int* lds_pre, int* wave_tot, int* lds_rows) {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        pre = lds_pre;
        BM = tile_rows;
        MG = __builtin_amdgcn_readfirstlane((p.MT + p.SM - 1) / p.SM);
        NG = __builtin_amdgcn_readfirstlane((p.NT + p.SN - 1) / p.SN);
        S = p.E * MG * NG;
        rows = lds_rows;
        if (tid < p.E) {
            lds_rows[tid] = group_rows(p, tid);
            lds_rows[64 + tid] = group_k(p, tid) / 64;
        }
        __syncthreads();
        const int CH = (S + NTH - 1) / NTH;
        auto tiles_of = [&](int at) {
            const int e = at / (MG * NG), r = at - e * (MG * NG);
            return live_rows(p, lds_rows[e], r % MG, BM) * min(p.NT - (r / MG) * p.SN, p.SN);
        };
        int sum = 0;
        for (int i = 0; i < CH; ++i) {
            const int at = tid * CH + i;
            if (at < S) sum += tiles_of(at);
        }
        int inc = sum;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int o = __shfl_up(inc, m, 64);
            if (lane >= m) inc += o;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        int run = inc - sum;
        for (int w = 0; w < wave; ++w) run += wave_tot[w];
        for (int i = 0; i < CH; ++i) {
            const int at = tid * CH + i;
            if (at < S) {
                lds_pre[at] = run;
                run += tiles_of(at);
            }
        }
        if (tid == NTH - 1) lds_pre[S] = run;            // the last thread owns the last chunk (or nothing): run = total
        __syncthreads();
        total = __builtin_amdgcn_readfirstlane(lds_pre[S]);
    }
    struct Place { int e, mt, nt; };
    // the tile with list index q (q < total, not below the q of the call before); all lanes active
    __device__ __forceinline__ Place find(const GemmParams& p, int q) {
        const int lane = threadIdx.x & 63;
        for (;;) {
            const int v = pre[min(s + 1 + lane, S)];     // ascending; the last entry is above every q
            const int n = __popcll(__ballot(v <= q));
            if (n > 0) first = __builtin_amdgcn_readlane(v, n - 1);
            s += n;
            if (n < 64) break;
        }
        const int e = small_div(s, MG * NG);
        const int r = s - e * (MG * NG), ng = small_div(r, MG), mg = r - ng * MG;
        const int vm = live_rows(p, count(e), mg, BM);
        const int c = small_div(q - first, vm);
        return {e, mg * p.SM + (q - first) - c * vm, ng * p.SN + c};
    }
    __device__ __forceinline__ int count(int e) const { return __builtin_amdgcn_readfirstlane(rows[e]); }
    __device__ __forceinline__ int k_tiles(int e) const { return __builtin_amdgcn_readfirstlane(rows[64 + e]); }
};

// Which tiles of a list this workgroup takes, in ascending order: in rounds over all workgroups, starting at place `turn`, and
// before that `extra` rounds over the workgroups from place `idle` on, which have nothing else to do (see
// gemm_bf16_backward_kernel).
struct Deal {
    int W, v;                    // workgroups, this one's place: the workgroups of an XCD are neighbours
    int idle, extra = 0, turn = 0;
    __device__ __forceinline__ Deal() {
        W = gridDim.x;
        v = (blockIdx.x & 7) * (W >> 3) + (blockIdx.x >> 3);
        idle = W;
    }
    // list index of this workgroup's i-th tile; at or past the end of the list: none
    __device__ __forceinline__ int tile(int i) const {
        const int own = v >= idle ? extra : 0;
        if (i < own) return i * (W - idle) + v - idle;
        const int w = v >= turn ? v - turn : v - turn + W;
        return extra * (W - idle) + (i - own) * W + w;
    }
};

// Row indices of a tile of 256 rows, on their way through LDS (see the kernels): asynchronous copy by waves 0..3, 64 rows each
__device__ __forceinline__ void request_row_ids(const GemmParams& p, int e, int m0, int count, int wave, int lane, int* dst) {
    if (wave < 4) {
        const int m = min(m0 + wave * 64 + lane, count - 1);             // rows past the count replay a valid row; never stored
        const int32_t* src = p.row_index + static_cast<size_t>(e) * p.capacity + m;
        __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)(dst + wave * 64), 4, 0, 0);
    }
}

// ---------------------------------------------------------------------------------------
// Persistent kernel for row-major operands (the one the forward pass and every row-major product of the backward pass
// run).  k-tiles of 64, and every copy instruction fetches whole 128-byte lines (8 rows x 128 bytes instead of the 16
// rows x 64 bytes of a 32-wide k-tile): on a copy-only loop over L2-resident data the line-sized pieces move 1.6 times the
// bytes per cycle of the half-line ones, and with 32-wide k-tiles the copies, not the matrix pipe, set the cycle count.
//
// Matrix instruction: v_mfma_f32_16x16x32_bf16.  The part is power-limited under this kernel, and a register-
// resident loop on random operands sustains 2.0 PFLOP/s with this shape against 1.77 with 32x32x16 (a fifth fewer
// register operands per flop).  Eight waves, two per SIMD; a wave's 128 x 64 slice of the 256 x 256 tile is 8 x 4
// accumulators of 16 x 16 (128 registers).  In an accumulator lane l holds token row l % 16 and the four output
// columns 4 (l / 16) .. + 3 (the weight fragment is the row operand).
//
// Two LDS buffers of 64 KiB (256 token rows + 256 weight rows x 128 bytes).  Step g multiplies buffer g & 1: two
// k-steps of 32 (ks), each split into the token blocks 0..3 and 4..7 (h), four substeps u = 2 ks + h of 16 MFMAs.
// Fragments: lane l reads row l % 16 of a 16-row block and the 16-byte chunk 4 ks + l / 16 of the k-tile (the
// chunk index is XORed with bits of the row on the copy's source side, which keeps each group of 16 lanes on 64
// distinct banks).  Token fragments are double-buffered by h, weight fragments by ks; every fragment read sits
// behind one MFMA of the substep before the one that needs it.  When the fourth substep's fragments have been asked
// for nobody reads that buffer any more: behind one wait (all copies landed, all own LDS reads done) and one
// barrier it is released.
//
// Copies (into LDS, no registers).  A wave's copies of k-tile g + 2 go out in two bursts, each behind the first MFMA
// of a substep: its groups of token rows in the fourth substep of step g (right behind the barrier), its groups of weight
// rows in the first substep of step g + 1.  They are bound by the time they take to land, before the barrier of step
// g + 1: spread behind every other MFMA of half a substep they cost 1-2 % more (gate/up and down product, 16 experts of 1280,
// 4096 x 11008: 4177 / 4110 us; 8 of 32 000, 4096 x 1408: 6601 / 6525; 16 of 600-1024, 2048 x 5632: 871 / 852), half a substep
// later another 1-4 %.  All eight in one substep is twice what a CU's address unit takes in that time (4-7 %).  The weight rows of a
// tile are whole column tiles (a launch condition), so their addresses are a wave-uniform base plus one of two
// per-lane offsets that never change; only the token rows carry per-tile lane offsets.  There is always something
// to copy: past the end of a workgroup's list the last k-tile is fetched again into a buffer nobody reads any
// more, which keeps the unrolled MFMA sequences free of branches.
//
// Gathered token rows (row_index).  The 256 row indices of a tile travel through LDS as well: 4-byte
// asynchronous copies by waves 0..3, requested two tiles ahead, so no wave ever waits for a global load while it
// sets up a tile.  Three slots rotate; a slot is read one tile after it was requested (at least two barriers with
// vmcnt(0) lie in between) and rewritten two tiles after it was read.
//
// Measured and not kept in this kernel (per-wave cycle stamps around the barrier, 16-expert 11008-wide workload):
// a step of the 32x32x16 form took 2900 cycles for 2048 cycles of MFMA work at 1.67 GHz, 320 of them waiting for
// copies.  Staging the operands through registers (plain loads issued a whole step ahead and evenly spread, LDS
// writes behind the barrier) removed that wait and brought the step to 2540 cycles, and the clock fell to
// 1.49 GHz: the same time.  One wave per SIMD with 128 x 128 slices (a third fewer LDS bytes per flop) needs
// 2700-2900 cycles of issue alone.  One memory instruction behind each MFMA instead of groups: the same time.
// ---------------------------------------------------------------------------------------
//
// TAIL: the contraction need not be whole k-tiles (K % 8 == 0 suffices); the 16-byte pieces of the last k-tile that
// lie past its end are zero-filled by the copy (buffer_copy_to_lds).  An instantiation of its own, so that the plain
// one keeps its scalar registers.
template <bool GLU, bool DUAL = false, bool KEEP = false, bool TAIL = false>
__global__ __launch_bounds__(512) void gemm_bf16_persistent_kernel(GemmParams p) {
    static_assert(!KEEP || (GLU && !DUAL), "the pre-activations are kept by the SwiGLU epilogue only");
    constexpr int NW = 8;                                // waves: 2 (token halves) x 4 (weight quarters)
    constexpr int BM = 256, BR = 256, CPR = 8, SWZ = 1;
    constexpr int BN = GLU ? 128 : 256;
    constexpr int STAGE = (BM + BR) * CPR;               // uint4 per LDS buffer (64 KiB)
    constexpr int NCP = 32 / NW;                         // groups of 8 rows each wave copies per operand
    constexpr int WROWS = 8 * NCP;                       // staged rows of each operand a wave copies
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4* lds = reinterpret_cast<uint4*>(lds_raw);
    __shared__ int pre[kMaxSuperWide + 1];
    __shared__ int wave_tot[NW], rows_of_group[128];
    __shared__ int row_ids[3][BM];                       // gathered rows of a tile: this, the next, the one after
    __shared__ __attribute__((aligned(16))) unsigned char stage_all[NW * kStageBytes];   // epilogue patches, one per wave

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int KCA = (p.lda ? p.lda : p.K) / 8, KCB = (p.ldb ? p.ldb : p.K) / 8;
    const bool gather = p.row_index != nullptr;

    LiveTiles tiles;
    tiles.build<NW * 64>(p, BM, pre, wave_tot, rows_of_group);
    const int total = tiles.total;
    const Deal deal;

    struct Tile {
        int e, m0, n0, count, KT;
        uint64_t Abase, Bbase;                           // wave-uniform; Bbase includes the wave's first weight row
        uint32_t offA[NCP];                              // per-lane byte offsets of the wave's token-row groups
    };
    // row group i of this wave: rows rr0 + 8 i, chunk c0 ^ 4 (i & 1) of the swizzle (8 rows further on flips bit 2)
    const int rr0 = wave * WROWS + (lane >> 3);
    const int c0 = (lane & 7) ^ ((rr0 >> SWZ) & 7);
    const uint32_t laneB[2] = {(static_cast<uint32_t>(lane >> 3) * KCB + ((lane & 7) ^ ((lane >> 4) & 7))) * 16u,
                               (static_cast<uint32_t>(lane >> 3) * KCB + ((lane & 7) ^ ((lane >> 4) & 7) ^ 4)) * 16u};
    const uint64_t strideB8 = static_cast<uint64_t>(8) * KCB * 16;      // 8 weight rows further on
    // TAIL: whether this lane's piece of the last k-tile lies past the contraction, for row groups of even / odd index
    // (the swizzle term of a lane is the same for both operands: a wave's rows start at a multiple of 32)
    const bool over[2] = {TAIL && 8 * c0 >= (p.K & 63), TAIL && 8 * (c0 ^ 4) >= (p.K & 63)};

    auto fill = [&](const LiveTiles::Place& at, Tile& t) {              // scalar part of a tile
        const int e = at.e;
        // (a ragged last column tile is moved back to end on the last column: it computes some columns of its left
        // neighbour once more and stores the same values, and no weight-row address or store needs a bound)
        t.e = e; t.m0 = at.mt * BM; t.n0 = min(at.nt * BN, p.N - BN);
        t.count = tiles.count(e);
        t.KT = TAIL ? (p.K + 63) / 64 : tiles.k_tiles(e);
        t.Abase = reinterpret_cast<uint64_t>(p.A) + (gather ? 0 : static_cast<uint64_t>(e) * p.capacity * KCA * 16);
        // this wave's staged weight rows: GLU stages 128 gate rows, then the 128 up rows of the same columns
        const int nrow = t.n0 + (GLU ? (wave % (NW / 2)) * WROWS : wave * WROWS);
        t.Bbase = reinterpret_cast<uint64_t>((GLU && wave >= NW / 2) ? p.B1 : p.B0) +
                  (static_cast<uint64_t>(e) * p.N + nrow) * KCB * 16;
    };
    // per-lane offsets of the token rows; with `gather` the indices have landed in slot `slot`
    auto finish = [&](Tile& t, int slot) {
        int row[NCP];
        if (gather) {                                    // one uniform branch around straight-line code
#pragma unroll
            for (int i = 0; i < NCP; ++i) row[i] = min(max(row_ids[slot][rr0 + 8 * i], 0), p.a_rows - 1);
        } else {
#pragma unroll
            for (int i = 0; i < NCP; ++i) row[i] = min(t.m0 + rr0 + 8 * i, t.count - 1);
        }
#pragma unroll
        for (int i = 0; i < NCP; ++i) t.offA[i] = (static_cast<uint32_t>(row[i]) * KCA + (c0 ^ (4 * (i & 1)))) * 16u;
    };
    auto copy_to = [&](uint64_t b64, uint32_t off, uint4* dst) {
        buffer_copy_to_lds(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64)),
                           __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32)), off, dst);
    };
    // token-row group i / weight-row group i of the k-tile at abase / bbase into buffer buf; `last`: the short k-tile
    auto copy_a = [&](uint64_t abase, uint32_t off, int buf, int i) {
        copy_to(abase, off, lds + buf * STAGE + (wave * NCP + i) * 64);
    };
    auto copy_b = [&](uint64_t bbase, int buf, int i, bool last) {
        const uint32_t off = TAIL && last && over[i & 1] ? kPastRange : laneB[i & 1];
        copy_to(bbase + i * strideB8, off, lds + buf * STAGE + BM * CPR + (wave * NCP + i) * 64);
    };

    // fragments: fah[h][i] = token block 4 h + i, fbk[ks][j] = weight block j of k-step ks
    f32x4 acc[8][4];
    bf16x8 fah[2][4], fbk[2][4];
    const int l16 = lane & 15, kq = lane >> 4;
    const int a_row = (wm * 128 + l16) * CPR;
    int b_row[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // SwiGLU: blocks 0, 1 are gate rows and 2, 3 the up rows of the same 32 output columns; plain: 64 columns
        const int br = GLU ? ((j >> 1) * 128 + wn * 32 + (j & 1) * 16) : (wn * 64 + j * 16);
        b_row[j] = BM * CPR + (br + l16) * CPR;
    }
    const int ck[2] = {kq ^ ((l16 >> SWZ) & 7), (4 + kq) ^ ((l16 >> SWZ) & 7)};
    auto read_a = [&](int buf, int ks, int h, int idx) {
        fah[h][idx] = __builtin_bit_cast(bf16x8, lds[buf * STAGE + a_row + (4 * h + idx) * 16 * CPR + ck[ks]]);
    };
    auto read_b = [&](int buf, int ks, int idx) {
        fbk[ks][idx] = __builtin_bit_cast(bf16x8, lds[buf * STAGE + b_row[idx] + ck[ks]]);
    };
    // substep u = 2 ks + h; `mem(m)` is the memory work behind its m-th MFMA.  Consecutive MFMAs share one operand (back and
    // forth over the token blocks): registers that do not change cost no power, and power is the limit.  FFN of 16 experts of
    // 1280 rows, 4096 x 11008, the layer, weight blocks restarted at each token block / this: 4346 / 4303 us; 8 of 32 000,
    // 4096 x 1408: 7451 / 7389; back and forth over the weight blocks 4337 and 7397.
    // (Without the barrier in front of mem(m) the compiler moves a substep's first reads before its first MFMA, where the wait
    // for the fragments then waits for these reads as well: 4128 / 4085 us and 7128 / 6972, 16 of 1024 bidirectional 2666 / 2627.)
    auto substep = [&](int u, auto&& mem) {
        const int ks = u >> 1, h = u & 1;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const int j = m >> 2, i = (j & 1) ? 3 - (m & 3) : (m & 3);
            acc[4 * h + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fbk[ks][j], fah[h][i], acc[4 * h + i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            mem(m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (deal.tile(0) >= total) return;                   // uniform: nothing for this workgroup
    Tile cur, nxt;
    LiveTiles::Place next_at{}, after{};
    fill(tiles.find(p, deal.tile(0)), cur);
    int seq = 0;                                         // tiles this workgroup has started; tile n uses slot n % 3
    bool has_next = deal.tile(1) < total;
    if (has_next) next_at = tiles.find(p, deal.tile(1));
    if (gather) {
        request_row_ids(p, cur.e, cur.m0, cur.count, wave, lane, row_ids[0]);
        if (has_next) request_row_ids(p, next_at.e, next_at.mt * BM, tiles.count(next_at.e), wave, lane, row_ids[1]);
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
        __builtin_amdgcn_s_barrier();                    // the indices were fetched by other waves
    }
    finish(cur, 0);
    int g = 0;                                           // global step: buffer g & 1
    for (int t = 0; t < 2; ++t) {                        // KT >= 2 is a launch condition
#pragma unroll
        for (int i = 0; i < NCP; ++i) copy_a(cur.Abase + t * 128, cur.offA[i], t, i);
#pragma unroll
        for (int i = 0; i < NCP; ++i) copy_b(cur.Bbase + t * 128, t, i, false);   // (TAIL: KT >= 3)
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * NCP, false));             // the first k-tile (copies retire in order)
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) { read_a(0, 0, 0, i); read_b(0, 0, i); }
    uint64_t lateB = cur.Bbase + 128;                    // weight rows still owed to the other buffer (none yet:
                                                         // the second k-tile's own once more)
    bool late_last = false;                              // they belong to a short k-tile
    for (;;) {
        if (has_next) {
            fill(next_at, nxt);
            finish(nxt, (seq + 1) % 3);
        }
        const bool has_after = deal.tile(seq + 2) < total;               // its row indices are requested two tiles ahead
        if (has_after) {
            after = tiles.find(p, deal.tile(seq + 2));
            if (gather) request_row_ids(p, after.e, after.mt * BM, tiles.count(after.e), wave, lane, row_ids[(seq + 2) % 3]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
        const int KT = cur.KT;
        for (int kt = 0; kt < KT; ++kt, ++g) {
            // k-tile g + 2: of this tile, else of the next one, else (nothing left) this tile's last one again
            const bool in_cur = kt + 2 < KT;
            const bool from_next = !in_cur && has_next;
            const int kf = in_cur ? kt + 2 : (from_next ? kt + 2 - KT : KT - 1);
            const uint64_t baseA = (from_next ? nxt.Abase : cur.Abase) + kf * 128;
            const uint64_t baseB = (from_next ? nxt.Bbase : cur.Bbase) + kf * 128;
            uint32_t offs[NCP];
#pragma unroll
            for (int i = 0; i < NCP; ++i) offs[i] = from_next ? nxt.offA[i] : cur.offA[i];
            const bool last = TAIL && kf == KT - 1;      // (every tile has the same KT here)
            if constexpr (TAIL) {
#pragma unroll
                for (int i = 0; i < NCP; ++i) offs[i] = last && over[i & 1] ? kPastRange : offs[i];
            }
            const int buf = g & 1;
            __builtin_amdgcn_sched_barrier(0);
            substep(0, [&](int m) {                      // token blocks 4..7 of this k-step, half of the next k-step's weights,
                if (m < 4) read_a(buf, 0, 1, m);         // and the weight rows of k-tile g + 1 into the other buffer
                else if (m < 6) read_b(buf, 1, m - 4);
                if (m == 0) {
#pragma unroll
                    for (int i = 0; i < NCP; ++i) copy_b(lateB, buf ^ 1, i, late_last);
                }
            });
            substep(1, [&](int m) {
                if (m < 4) read_a(buf, 1, 0, m);
                else if (m < 6) read_b(buf, 1, m - 2);
            });
            substep(2, [&](int m) {
                if (m < 4) read_a(buf, 1, 1, m);
            });
            // k-tile g + 1 has landed and this wave's reads of buffer buf are done; past the barrier that holds for all
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            substep(3, [&](int m) {                      // the next k-tile's first fragments, and the token rows of k-tile
                if (m < 4) read_a(buf ^ 1, 0, 0, m);     // g + 2 into the buffer just released
                else if (m < 8) read_b(buf ^ 1, 0, m - 4);
                if (m == 0) {
#pragma unroll
                    for (int i = 0; i < NCP; ++i) copy_a(baseA, offs[i], buf, i);
                }
            });
            lateB = baseB;
            late_last = last;
        }
        // ---- epilogue of cur (the copies of the next tile are in flight)
        store_blocks_staged16<GLU, DUAL, KEEP>(p, acc, cur.e, cur.m0 + wm * 128, cur.n0 + wn * (GLU ? 32 : 64), cur.count, lane,
                                               stage_all + wave * kStageBytes);
        if (!has_next) break;
        cur = nxt;
        next_at = after;
        has_next = has_after;
        ++seq;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));   // the re-fetched k-tiles of the last two steps
}

// ---------------------------------------------------------------------------------------
// Persistent kernel for operands whose contraction index is the slow one (backward pass): B is [K][N], and A is row-major
// [M][K] or, with TRA, [K][M] (row strides lda / ldb, group stride K * ld).  With B1 the contraction is split in the
// middle: first half from B0, second half from B1, each [K/2][N].  Plain products only: row-major operands with an
// epilogue take the kernel above, whose tile list, k-tiles of 64, two LDS buffers and substeps this one shares.
//
// Staging.  A k-tile of such an operand is 64 k x 256 rows; a copy instruction takes 8 k x 128 bytes (whole lines), and LDS
// holds it as [4 groups of 64 rows][64 k][128 bytes].  Wave w copies the k rows 8 w .. 8 w + 7 of all four groups.
// Fragments come out through the transposing read ds_read_b64_tr_b16: inside a group of 16 lanes, lane i supplies the
// address of 4 consecutive elements and receives element i % 4 of lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.  With lane
// (q = i % 4, j = i / 4) pointing at (k0 + j, r0 + 4 q) lane i receives rows r0 + i at k0 .. k0 + 3: two reads give the 8
// consecutive k of one row that the MFMA operand layout wants.  Half a wave reads 32 bytes of each of the k rows 8 kq + j (kq =
// 0, 1 or 2, 3; j = 0..3), which lie on two half sets of banks: the 32-byte piece o of a k row is stored at o ^ f(k), f(k) =
// bit 1 of k, bit 3 of k, so that the eight pieces cover all 64 banks (applied on the source side of the copy).
//
// KG (1: A, 2: B): the contraction rows of that operand are fetched through p.k_index (a gather along the slow index).  The
// four copies of a lane share one k row, so a lane needs one row number per k-tile, loaded three k-tiles ahead.  Row
// numbers are clamped into [0, k_rows).  In the padding of a group's contraction, where the other operand is zero, its own last
// row is fetched again: any other row's infinities or NaNs would turn those zeros into NaNs of a group that never had the row.
// A group without rows has none to repeat, and nobody has written its padding: its tiles are stored as zeros whatever was
// multiplied (TRA).
//
// TAIL (row-major A): the contraction, or each half of a split one, need not be whole k-tiles.  The last k-tile of it is
// short: pieces of a token row and whole weight rows past its end are zero-filled (buffer_copy_to_lds).
//
// Bound as the kernel above is.  Measured against the form it replaces (32-wide k-tiles in a ring of four, v_mfma_f32_32x32x16,
// the wait of every fragment read in the open): weight gradients of 8 experts x 32 000 gathered rows, 4096 x 1408: 2864 ->
// 2452 us and, both gate and up, 5561 -> 4603 us (1.06 -> 1.28 PFLOP/s); 16 experts of 166-1024 rows, 2048 x 5632: 281 -> 268 us
// each, input gradient 603 -> 586 us.
// ---------------------------------------------------------------------------------------
struct TransposingLds {                                  // beside the two buffers
    int pre[kMaxSuper + 1];
    int wave_tot[8], rows_of_group[128];
    int row_ids[3][256];                                 // gathered rows of a tile: this, the next, the one after
    float gates[3][256];                                 // MID: weights of a tile's rows, in the same three slots
    int k_last[64];                                      // TRA: last row of each group's contraction (-1: it has none)
};
// What a product leaves to the ones behind it in the same launch: the workgroups from place `idle` on are `ahead` k-tiles
// ahead of the others (a tile counts kTileSteps more than it has); the next list's rounds begin at place `turn`.
constexpr int kTileSteps = 2;
struct DealState {
    int idle, ahead = 0, turn = 0;
    // uniform: k-tiles of every tile (0: the groups' own)
    __device__ __forceinline__ void deal(const GemmParams& p, const LiveTiles& tiles, int uniform, Deal& d) {
        int steps = uniform;                             // of a tile on average: every group has the same number of tiles here
        if (uniform == 0) {
            const int lane = threadIdx.x & 63;
            steps = lane < p.E ? tiles.rows[64 + lane] : 0;
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) steps += __shfl_xor(steps, m, 64);
            steps = small_div(__builtin_amdgcn_readfirstlane(steps), p.E);
        }
        steps += kTileSteps;
        const int free = d.W - idle;
        if (free > 0 && ahead >= steps) {
            const int most = small_div(tiles.total, free), wanted = small_div(ahead, steps);
            d.idle = idle;
            d.extra = wanted < most ? wanted : most;
            ahead -= d.extra * steps;
        }
        d.turn = turn;
        const int rest = tiles.total - d.extra * free, late = rest - small_div(rest, d.W) * d.W;
        if (uniform != 0 && turn == 0 && ahead == 0) {   // the long product in front: a partly filled last round
            idle = late > 0 ? late : d.W;
            ahead = late > 0 ? steps : 0;
        }
        turn = turn + late < d.W ? turn + late : turn + late - d.W;
    }
};
template <bool TRA, int KG, bool TAIL, bool MID = false>
__device__ __forceinline__ void transposing_tiles(const GemmParams& p, TransposingLds& sh, DealState& state) {
    static_assert(KG == 0 || TRA, "gathered contraction rows: both operands transposed");
    static_assert(!TAIL || (!TRA && KG == 0), "short k-tiles: row-major A");
    static_assert(!MID || !TRA, "the middle of the backward: row-major A");
    constexpr int NW = 8, BM = 256, BN = 256, CPR = 8, SWZ = 1;
    constexpr int HALF = 256 * CPR;                      // uint4 per operand and LDS buffer (32 KiB)
    constexpr int STAGE = 2 * HALF;
    constexpr int NCP = 4;                               // copies per wave, operand and k-tile
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    uint4* lds = reinterpret_cast<uint4*>(lds_raw);
    int (&row_ids)[3][BM] = sh.row_ids;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const bool gather = !TRA && p.row_index != nullptr;
    const int lda = p.lda ? p.lda : p.K, ldb = p.ldb ? p.ldb : p.K;
    const bool splitB = p.B1 != nullptr;
    const int Kh = splitB ? p.K / 2 : p.K, KTh = (Kh + 63) / 64;         // of the whole product, or of each half of a split one
    const int k_rem = (Kh & 63) ? (Kh & 63) : 64;        // valid k of the last k-tile

    if (TRA && tid < p.E) {
        const int n = min(p.k_counts ? max(p.k_counts[tid], 0) : p.K, p.K);
        sh.k_last[tid] = (KG != 0 ? min(n, p.k_index_stride) : n) - 1;
    }
    LiveTiles tiles;
    tiles.build<NW * 64>(p, BM, sh.pre, sh.wave_tot, sh.rows_of_group);          // (its barriers cover k_last)
    const int total = tiles.total;
    Deal deal;
    const int k_all = splitB ? 2 * KTh : KTh, k_piece = (k_all + p.pieces - 1) / p.pieces;      // k-tiles of the product, of a part
    state.deal(p, tiles, TRA ? 0 : k_piece, deal);

    struct Tile {
        int e, m0, n0, count, KT;
        int k0, piece;                                   // first k-tile, part of the contraction
        int k_last;                                      // TRA: last row of the contraction
        uint64_t Abase, Bbase, Bbase1;                   // wave-uniform; Bbase1: second half of a split B
        uint32_t offA[TRA ? 1 : NCP];                    // row-major A: byte offsets of this lane's row groups
    };
    // row-major A: this lane's copies are rows rr0 + 8 i, chunk c0 ^ 4 (i & 1) of the swizzle
    const int rr0 = wave * 32 + (lane >> 3);
    const int c0 = (lane & 7) ^ ((rr0 >> SWZ) & 7);
    const bool over_a[2] = {TAIL && 8 * c0 >= k_rem, TAIL && 8 * (c0 ^ 4) >= k_rem};
    // transposed operands: k row of this lane's copies, and its first row inside a group of 64 rows
    const int k_row = wave * 8 + (lane >> 3);
    const int lane_r = 16 * (((lane & 7) >> 1) ^ (((k_row >> 1) & 1) | ((k_row >> 2) & 2))) + 8 * (lane & 1);
    const bool over_b = TAIL && k_row >= k_rem;
    const uint32_t fixedA = KG == 1 ? 0u : static_cast<uint32_t>(k_row) * lda * 2u;      // (a gathered row comes from the index)
    const uint32_t fixedB = KG == 2 ? 0u : static_cast<uint32_t>(k_row) * ldb * 2u;
    const int limitA = p.capacity - 8, limitB = p.N - 8; // copies stay inside the k row; what they repeat is never stored

    auto fill = [&](const LiveTiles::Place& at, Tile& t) {              // scalar part of a tile
        const int e = at.e;
        const int columns = (p.N + BN - 1) / BN;
        t.piece = !TRA && p.pieces > 1 ? small_div(at.nt, columns) : 0;
        t.e = e; t.m0 = at.mt * BM; t.n0 = (at.nt - t.piece * columns) * BN;
        t.count = tiles.count(e);
        t.k0 = t.piece * k_piece;
        t.KT = TRA ? tiles.k_tiles(e) : min(k_piece, k_all - t.k0);
        t.k_last = TRA ? __builtin_amdgcn_readfirstlane(sh.k_last[e]) : 0;
        t.Abase = reinterpret_cast<uint64_t>(p.A);
        if (KG != 1) t.Abase += TRA ? static_cast<uint64_t>(e) * p.K * lda * 2
                                    : (p.row_index ? 0 : static_cast<uint64_t>(e) * p.capacity * lda * 2);
        const uint64_t group = KG == 2 ? 0 : static_cast<uint64_t>(e) * Kh * ldb * 2;
        t.Bbase = reinterpret_cast<uint64_t>(p.B0) + group;
        t.Bbase1 = splitB ? reinterpret_cast<uint64_t>(p.B1) + group : t.Bbase;
    };
    // row-major A: per-lane offsets of the token rows; with `gather` the indices have landed in slot `slot`
    auto finish = [&](Tile& t, int slot) {
        if constexpr (!TRA) {
            int row[NCP];
            if (gather) {                                // one uniform branch around straight-line code
#pragma unroll
                for (int i = 0; i < NCP; ++i) row[i] = min(max(row_ids[slot][rr0 + 8 * i], 0), p.a_rows - 1);
            } else {
#pragma unroll
                for (int i = 0; i < NCP; ++i) row[i] = min(t.m0 + rr0 + 8 * i, t.count - 1);
            }
#pragma unroll
            for (int i = 0; i < NCP; ++i) t.offA[i] = (static_cast<uint32_t>(row[i]) * lda + (c0 ^ (4 * (i & 1))) * 8) * 2u;
        }
    };
    auto a_ktile = [&](uint64_t a, int k) -> uint64_t {
        if constexpr (TRA) return KG == 1 ? a : a + static_cast<uint64_t>(k) * (static_cast<uint64_t>(lda) * 128);
        const bool second = splitB && k >= KTh;
        return a + (second ? static_cast<uint64_t>(Kh) * 2 + static_cast<uint64_t>(k - KTh) * 128 : static_cast<uint64_t>(k) * 128);
    };
    auto b_ktile = [&](uint64_t b0, uint64_t b1, int k) -> uint64_t {
        if constexpr (KG == 2) return b0;
        const bool second = splitB && k >= KTh;
        return (second ? b1 : b0) + static_cast<uint64_t>(second ? k - KTh : k) * (static_cast<uint64_t>(ldb) * 128);
    };
    auto is_short = [&](int k) { return TAIL && (k == KTh - 1 || k == 2 * KTh - 1); };
    auto copy_to = [&](uint64_t b64, uint32_t off, uint4* dst) {
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32));
        if constexpr (TAIL) {
            buffer_copy_to_lds(lo, hi, off, dst);
        } else {
            const char* base = reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
            __builtin_amdgcn_global_load_lds((global_cptr)(base + off), (lds_ptr)dst, 16, 0, 0);
        }
    };
    // copy i of the A / B operand of one k-tile into buffer buf (off_row: row-major A's offset, or the k row's)
    auto copy_a = [&](uint64_t base, uint32_t off_row, int m0, int buf, int i) {
        if constexpr (TRA)
            copy_to(base, off_row + 2u * min(m0 + 64 * i + lane_r, limitA), lds + buf * STAGE + i * (HALF / 4) + wave * 64);
        else
            copy_to(base, off_row, lds + buf * STAGE + (wave * NCP + i) * 64);
    };
    auto copy_b = [&](uint64_t base, uint32_t off_row, int n0, bool last, int buf, int i) {
        uint32_t off = off_row + 2u * min(n0 + 64 * i + lane_r, limitB);
        if (TAIL) off = last && over_b ? kPastRange : off;
        copy_to(base, off, lds + buf * STAGE + HALF + i * (HALF / 4) + wave * 64);
    };
    // KG: this lane's row number in k-tile kl of group e, whose last row is k_last, and the byte offset of that row
    auto load_index = [&](int e, int k_last, int kl) -> int {
        return p.k_index[static_cast<size_t>(e) * p.k_index_stride + max(min(kl * 64 + k_row, k_last), 0)];
    };
    auto row_offset = [&](int index) -> uint32_t {
        return static_cast<uint32_t>(min(max(index, 0), p.k_rows - 1)) * static_cast<uint32_t>(KG == 1 ? lda : ldb) * 2u;
    };

    const int l16 = lane & 15, kq = lane >> 4;
    // row-major A: as in the kernel above
    const int a_row = (wm * 128 + l16) * CPR;
    const int ck[2] = {kq ^ ((l16 >> SWZ) & 7), (4 + kq) ^ ((l16 >> SWZ) & 7)};
    // transposing reads: LDS byte address (buffer 0) of this lane's 4 elements of the 16-row blocks 0..3 of a group of 64
    // rows, first k-step; + 512: the k four further on, + 4096: the second k-step, + 8192: the next group
    typedef int v2i __attribute__((ext_vector_type(2)));
    typedef int v4i __attribute__((ext_vector_type(4)));
    const uint32_t lds_base = lds_address(lds_raw);
    uint32_t a_tr[4], b_tr[4];
    {
        const int q = l16 & 3, j = l16 >> 2, f = ((j >> 1) & 1) | ((kq & 1) << 1);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const uint32_t at = lds_base + (8 * kq + j) * 128 + ((o ^ f) * 32) + q * 8;
            a_tr[o] = at + wm * 2 * 8192;
            b_tr[o] = at + HALF * 16 + wn * 8192;
        }
    }
    f32x4 acc[8][4];
    bf16x8 fah[2][4], fbk[2][4];
    auto tr_pack = [](v2i lo, v2i hi) -> bf16x8 {        // k .. k + 3 and k + 4 .. k + 7 of one row
        const v4i r = {lo.x, lo.y, hi.x, hi.y};
        return __builtin_bit_cast(bf16x8, r);
    };
    // The transposing reads are assembly: through the compiler's builtin every such read waits for ALL outstanding copies
    // (vmcnt(0)), because it is taken to alias the asynchronous LDS writes.  A statement holds eight MFMAs (two token blocks,
    // four weight blocks, back and forth as in the kernel above: training step of 16 experts of 166-1024 rows, 2048 x 5632, 2637 ->
    // 2620 us) with the reads of up to four fragments behind the first of them and its own wait at the end: the
    // reads land under the remaining MFMAs, and the outputs are ordinary, fully written registers when it ends.  (The reads
    // in statements of their own, with the wait right behind them: 5 % slower over 32 000 rows.)  What the compiler
    // cannot see inside: two wait states between an ordinary write of an operand and its use (the s_nop in front); it must
    // not touch an accumulator right behind a statement (settle() before the epilogue).
#define ETR_MF(C, B, A) "v_mfma_f32_16x16x32_bf16 %[c" #C "], %[b" #B "], %[a" #A "], %[c" #C "]\n\t"
#define ETR_TR(N) "ds_read_b64_tr_b16 %[x" #N "], %[p" #N "] offset:%c[o" #N "]\n\tds_read_b64_tr_b16 %[y" #N "], %[p" #N "] offset:%c[q" #N "]\n\t"
#define ETR_ACC(i) [c0] "+v"(acc[i][0]), [c1] "+v"(acc[i][1]), [c2] "+v"(acc[i][2]), [c3] "+v"(acc[i][3]), \
                   [c4] "+v"(acc[i + 1][0]), [c5] "+v"(acc[i + 1][1]), [c6] "+v"(acc[i + 1][2]), [c7] "+v"(acc[i + 1][3])
#define ETR_FRAGS [a0] "v"(fa[0]), [a1] "v"(fa[1]), [b0] "v"(fb[0]), [b1] "v"(fb[1]), [b2] "v"(fb[2]), [b3] "v"(fb[3])
#define ETR_OUT(N) [x##N] "=&v"(x[N]), [y##N] "=&v"(y[N])
#define ETR_AT(N, OFF) [p##N] "v"(at##N + slot), [o##N] "n"(OFF), [q##N] "n"(OFF + 512)
    // MFMAs of token blocks I, I + 1 (accumulators) = fa[0], fa[1] with fb[0..3]; reads fragments 0 .. R - 1 from at0.. at the
    // constant offsets O0..
    auto mfma8 = [&](auto reads, auto block, const bf16x8* fa, const bf16x8* fb, uint32_t slot, bf16x8* f0, uint32_t at0, auto o0,
                     bf16x8* f1, uint32_t at1, auto o1, bf16x8* f2, uint32_t at2, auto o2, bf16x8* f3, uint32_t at3, auto o3) {
        constexpr int R = decltype(reads)::value, I = decltype(block)::value;
        constexpr int O0 = decltype(o0)::value, O1 = decltype(o1)::value, O2 = decltype(o2)::value, O3 = decltype(o3)::value;
        v2i x[4], y[4];
        if constexpr (R == 1)
            asm volatile("s_nop 1\n\t" ETR_MF(0, 0, 0) ETR_TR(0) ETR_MF(1, 1, 0) ETR_MF(2, 2, 0) ETR_MF(3, 3, 0)
                         ETR_MF(7, 3, 1) ETR_MF(6, 2, 1) ETR_MF(5, 1, 1) ETR_MF(4, 0, 1) "s_waitcnt lgkmcnt(0)"
                         : ETR_ACC(I), ETR_OUT(0) : ETR_FRAGS, ETR_AT(0, O0));
        if constexpr (R == 2)
            asm volatile("s_nop 1\n\t" ETR_MF(0, 0, 0) ETR_TR(0) ETR_MF(1, 1, 0) ETR_TR(1) ETR_MF(2, 2, 0) ETR_MF(3, 3, 0)
                         ETR_MF(7, 3, 1) ETR_MF(6, 2, 1) ETR_MF(5, 1, 1) ETR_MF(4, 0, 1) "s_waitcnt lgkmcnt(0)"
                         : ETR_ACC(I), ETR_OUT(0), ETR_OUT(1) : ETR_FRAGS, ETR_AT(0, O0), ETR_AT(1, O1));
        if constexpr (R == 3)
            asm volatile("s_nop 1\n\t" ETR_MF(0, 0, 0) ETR_TR(0) ETR_MF(1, 1, 0) ETR_TR(1) ETR_MF(2, 2, 0) ETR_TR(2) ETR_MF(3, 3, 0)
                         ETR_MF(7, 3, 1) ETR_MF(6, 2, 1) ETR_MF(5, 1, 1) ETR_MF(4, 0, 1) "s_waitcnt lgkmcnt(0)"
                         : ETR_ACC(I), ETR_OUT(0), ETR_OUT(1), ETR_OUT(2) : ETR_FRAGS, ETR_AT(0, O0), ETR_AT(1, O1), ETR_AT(2, O2));
        if constexpr (R == 4)
            asm volatile("s_nop 1\n\t" ETR_MF(0, 0, 0) ETR_TR(0) ETR_MF(1, 1, 0) ETR_TR(1) ETR_MF(2, 2, 0) ETR_TR(2) ETR_MF(3, 3, 0)
                         ETR_TR(3) ETR_MF(7, 3, 1) ETR_MF(6, 2, 1) ETR_MF(5, 1, 1) ETR_MF(4, 0, 1) "s_waitcnt lgkmcnt(0)"
                         : ETR_ACC(I), ETR_OUT(0), ETR_OUT(1), ETR_OUT(2), ETR_OUT(3)
                         : ETR_FRAGS, ETR_AT(0, O0), ETR_AT(1, O1), ETR_AT(2, O2), ETR_AT(3, O3));
        if constexpr (R == 0) {
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int i = m >> 2, j = i ? 7 - m : m;
                acc[I + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[I + i][j], 0, 0, 0);
            }
        }
        if constexpr (R > 0) *f0 = tr_pack(x[0], y[0]);
        if constexpr (R > 1) *f1 = tr_pack(x[1], y[1]);
        if constexpr (R > 2) *f2 = tr_pack(x[2], y[2]);
        if constexpr (R > 3) *f3 = tr_pack(x[3], y[3]);
    };
#define ETR_OFF(x) std::integral_constant<int, (x)>{}
    auto read_a_rows = [&](int buf, int ks, int h, int idx) {           // row-major A, one block
        fah[h][idx] = __builtin_bit_cast(bf16x8, lds[buf * STAGE + a_row + (4 * h + idx) * 16 * CPR + ck[ks]]);
    };
    // substep u = 2 ks + h: 16 MFMAs, and the reads of what substep u + 1 needs (from buffer `buf`; u = 3: of the next k-tile);
    // mem(0), mem(1), mem(2): memory work in front of the first eight MFMAs, between the two eights, behind them
    auto substep = [&](auto u, int buf, auto&& mem) {
        constexpr int U = decltype(u)::value, ks = U >> 1, h = U & 1;
        const uint32_t slot = static_cast<uint32_t>(buf) * (STAGE * 16);
        bf16x8* const na = fah[h ^ 1];                   // fragments of substep u + 1
        bf16x8* const nb = fbk[U == 3 ? 0 : 1];
        constexpr int OA = U == 0 ? 8192 : (U == 1 ? 4096 : (U == 2 ? 8192 + 4096 : 0)), OB = U == 3 ? 0 : 4096;
        constexpr int J = U == 1 ? 2 : 0;                // weight blocks read in substeps 0 and 1: two each
        const auto oa = ETR_OFF(OA);
        const auto ob = ETR_OFF(OB);
        if constexpr (!TRA) {
#pragma unroll
            for (int i = 0; i < 4; ++i) read_a_rows(buf, U == 3 ? 0 : (U + 1) >> 1, h ^ 1, i);
        }
        mem(0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TRA && U < 2)
            mfma8(ETR_OFF(3), ETR_OFF(4 * h), fah[h], fbk[ks], slot, na, a_tr[0], oa, na + 1, a_tr[1], oa, na + 2, a_tr[2], oa, na, 0u, oa);
        else if constexpr (TRA && U == 2)
            mfma8(ETR_OFF(2), ETR_OFF(4 * h), fah[h], fbk[ks], slot, na, a_tr[0], oa, na + 1, a_tr[1], oa, na, 0u, oa, na, 0u, oa);
        else if constexpr (TRA)
            mfma8(ETR_OFF(4), ETR_OFF(4 * h), fah[h], fbk[ks], slot, na, a_tr[0], oa, na + 1, a_tr[1], oa, na + 2, a_tr[2], oa, na + 3, a_tr[3], oa);
        else if constexpr (U < 2)
            mfma8(ETR_OFF(1), ETR_OFF(4 * h), fah[h], fbk[ks], slot, nb + J, b_tr[J], ob, na, 0u, oa, na, 0u, oa, na, 0u, oa);
        else if constexpr (U == 2)
            mfma8(ETR_OFF(0), ETR_OFF(4 * h), fah[h], fbk[ks], slot, na, 0u, oa, na, 0u, oa, na, 0u, oa, na, 0u, oa);
        else
            mfma8(ETR_OFF(2), ETR_OFF(4 * h), fah[h], fbk[ks], slot, nb, b_tr[0], ob, nb + 1, b_tr[1], ob, na, 0u, oa, na, 0u, oa);
        __builtin_amdgcn_sched_barrier(0);
        mem(1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TRA && U < 2)
            mfma8(ETR_OFF(3), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, na + 3, a_tr[3], oa, nb + J, b_tr[J], ob, nb + J + 1, b_tr[J + 1], ob, na, 0u, oa);
        else if constexpr (TRA && U == 2)
            mfma8(ETR_OFF(2), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, na + 2, a_tr[2], oa, na + 3, a_tr[3], oa, na, 0u, oa, na, 0u, oa);
        else if constexpr (TRA)
            mfma8(ETR_OFF(4), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, nb, b_tr[0], ob, nb + 1, b_tr[1], ob, nb + 2, b_tr[2], ob, nb + 3, b_tr[3], ob);
        else if constexpr (U < 2)
            mfma8(ETR_OFF(1), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, nb + J + 1, b_tr[J + 1], ob, na, 0u, oa, na, 0u, oa, na, 0u, oa);
        else if constexpr (U == 2)
            mfma8(ETR_OFF(0), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, na, 0u, oa, na, 0u, oa, na, 0u, oa, na, 0u, oa);
        else
            mfma8(ETR_OFF(2), ETR_OFF(4 * h + 2), fah[h] + 2, fbk[ks], slot, nb + 2, b_tr[2], ob, nb + 3, b_tr[3], ob, na, 0u, oa, na, 0u, oa);
        __builtin_amdgcn_sched_barrier(0);
        mem(2);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the first fragments of a workgroup (buffer 0), read and waited for on their own
    auto read_first = [&]() {
        auto tr = [&](uint32_t at) {
            v2i x, y;
            asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:512\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(x), "=&v"(y) : "v"(at));
            return tr_pack(x, y);
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (TRA) fah[0][i] = tr(a_tr[i]);
            else read_a_rows(0, 0, 0, i);
            fbk[0][i] = tr(b_tr[i]);
        }
    };
    // nothing the compiler places behind this reads an accumulator sooner than its MFMA has written it
    auto settle = [&]() {
#pragma unroll
        for (int i = 0; i < 8; i += 2)
            asm volatile("s_nop 15\n\ts_nop 3" : ETR_ACC(i));
    };

    // MID: the weights of the rows whose token numbers lie in a slot, beside them (zero for a number that is none)
    auto request_gates = [&](int e, int slot) {
        if (wave < 4) {
            const int token = row_ids[slot][wave * 64 + lane];
            const bool in = token >= 0 && token < p.a_rows;
            const float* src = in ? p.mid_gate + static_cast<size_t>(token) * p.E + e : kZeroPiece;
            __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)(sh.gates[slot] + wave * 64), 4, 0, 0);
        }
    };

    if (deal.tile(0) >= total) return;                   // uniform: nothing for this workgroup
    Tile cur, nxt;
    LiveTiles::Place next_at{}, after{};
    fill(tiles.find(p, deal.tile(0)), cur);
    int seq = 0;                                         // tiles this workgroup has started; tile n uses slot n % 3
    bool has_next = deal.tile(1) < total;
    if (has_next) next_at = tiles.find(p, deal.tile(1));
    if (gather) {
        request_row_ids(p, cur.e, cur.m0, cur.count, wave, lane, row_ids[0]);
        if (has_next) request_row_ids(p, next_at.e, next_at.mt * BM, tiles.count(next_at.e), wave, lane, row_ids[TRA ? 0 : 1]);
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
        __builtin_amdgcn_s_barrier();                    // the indices were fetched by other waves
    }
    finish(cur, 0);
    if constexpr (MID) request_gates(cur.e, 0);
    int g = 0;                                           // global step: buffer g & 1
    int index = 0;                                       // KG: this lane's row number in k-tile g + 2
    if constexpr (KG != 0) index = load_index(cur.e, cur.k_last, 2); // (KT >= 4)
    uint32_t row_a = fixedA, row_b = fixedB;             // byte offset of this lane's k row in the k-tile to copy next
    for (int t = 0; t < 2; ++t) {                        // KT >= 2 is a launch condition
        if constexpr (KG == 1) row_a = row_offset(load_index(cur.e, cur.k_last, t));
        if constexpr (KG == 2) row_b = row_offset(load_index(cur.e, cur.k_last, t));
        const uint64_t baseA = a_ktile(cur.Abase, cur.k0 + t), baseB = b_ktile(cur.Bbase, cur.Bbase1, cur.k0 + t);
#pragma unroll
        for (int i = 0; i < NCP; ++i) {
            uint32_t off = row_a;
            if constexpr (!TRA) off = is_short(cur.k0 + t) && over_a[i & 1] ? kPastRange : cur.offA[i];
            copy_a(baseA, off, cur.m0, t, i);
        }
#pragma unroll
        for (int i = 0; i < NCP; ++i) copy_b(baseB, row_b, cur.n0, is_short(cur.k0 + t), t, i);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * NCP, false));             // the first k-tile (copies retire in order)
    __builtin_amdgcn_s_barrier();
    read_first();
    // B rows still owed to the other buffer (none yet: the second k-tile's own once more)
    uint64_t late_base = b_ktile(cur.Bbase, cur.Bbase1, cur.k0 + 1);
    int late_n0 = cur.n0;
    bool late_last = is_short(cur.k0 + 1);
    for (;;) {
        if (has_next) {
            fill(next_at, nxt);
            finish(nxt, (seq + 1) % 3);
            if constexpr (MID) request_gates(nxt.e, (seq + 1) % 3);
        }
        const bool has_after = deal.tile(seq + 2) < total;               // its row indices are requested two tiles ahead
        if (has_after) {
            after = tiles.find(p, deal.tile(seq + 2));
            if (gather) request_row_ids(p, after.e, after.mt * BM, tiles.count(after.e), wave, lane, row_ids[TRA ? 0 : (seq + 2) % 3]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
        const int KT = cur.KT;
        for (int kt = 0; kt < KT; ++kt, ++g) {
            // k-tile g + 2: of this tile, else of the next one, else (nothing left) this tile's last one again
            const bool in_cur = kt + 2 < KT;
            const bool from_next = !in_cur && has_next;
            const int kf = in_cur ? cur.k0 + kt + 2 : (from_next ? nxt.k0 + kt + 2 - KT : cur.k0 + KT - 1);
            const uint64_t baseA = a_ktile(from_next ? nxt.Abase : cur.Abase, kf);
            const uint64_t baseB = b_ktile(from_next ? nxt.Bbase : cur.Bbase, from_next ? nxt.Bbase1 : cur.Bbase1, kf);
            const int m0 = from_next ? nxt.m0 : cur.m0, n0 = from_next ? nxt.n0 : cur.n0;
            const bool last = is_short(kf);
            uint32_t offs[NCP] = {};
            if constexpr (!TRA) {
#pragma unroll
                for (int i = 0; i < NCP; ++i) {
                    offs[i] = from_next ? nxt.offA[i] : cur.offA[i];
                    if (TAIL) offs[i] = last && over_a[i & 1] ? kPastRange : offs[i];
                }
            }
            const int buf = g & 1;
            __builtin_amdgcn_sched_barrier(0);
            substep(ETR_OFF(0), buf, [&](int m) {        // and the B rows of k-tile g + 1 into the other buffer
                if (m == 2) return;
                copy_b(late_base, row_b, late_n0, late_last, buf ^ 1, 2 * m);
                copy_b(late_base, row_b, late_n0, late_last, buf ^ 1, 2 * m + 1);
            });
            if constexpr (KG == 1) row_a = row_offset(index);
            if constexpr (KG == 2) row_b = row_offset(index);
            substep(ETR_OFF(1), buf, [&](int m) {        // and the row number in k-tile g + 3, wanted one step from now
                if constexpr (KG != 0) {
                    const bool stay = kt + 3 < KT || !has_next;
                    if (m == 0) index = load_index(stay ? cur.e : nxt.e, stay ? cur.k_last : nxt.k_last, stay ? kt + 3 : kt + 3 - KT);
                }
            });
            substep(ETR_OFF(2), buf, [&](int) {});
            // k-tile g + 1 has landed and this wave's reads of buffer buf are done; past the barrier that holds for all
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            substep(ETR_OFF(3), buf ^ 1, [&](int m) {    // the next k-tile's first fragments, and the A rows of k-tile
                if (m == 2) return;                      // g + 2 into the buffer just released
                copy_a(baseA, TRA ? row_a : offs[2 * m], m0, buf, 2 * m);
                copy_a(baseA, TRA ? row_a : offs[2 * m + 1], m0, buf, 2 * m + 1);
            });
            late_base = baseB;
            late_n0 = n0;
            late_last = last;
        }
        settle();
        if (TRA && cur.k_last < 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // ---- epilogue of cur (the copies of the next tile are in flight).  The patch is the wave's own copy target in the
        // B half of the buffer just multiplied: behind the last barrier nobody reads it any more, and the next copies into
        // it are the wave's own, in its next substep 0.
        const uint32_t patch = lds_base + static_cast<uint32_t>((g - 1) & 1) * (STAGE * 16) + HALF * 16 + wave * 1024;
        if constexpr (MID) {
            store_middle(p, acc, cur.e, cur.m0 + wm * 128, cur.n0 + wn * 64, cur.count, lds_address(sh.gates[seq % 3] + wm * 128), patch, lane);
        } else if (!TRA && p.pieces > 1) {               // few rows: fp32 sums, 16 rows x 64 bytes an instruction
            float* out = static_cast<float*>(p.C) + (static_cast<size_t>(cur.piece) * p.E + cur.e) * p.capacity * p.N;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int m = cur.m0 + wm * 128 + i * 16 + l16;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int n = cur.n0 + wn * 64 + j * 16 + kq * 4;
                    if (m < cur.count && n < p.N) *reinterpret_cast<f32x4*>(out + static_cast<size_t>(m) * p.N + n) = acc[i][j];
                }
            }
        } else {
            const int nb = cur.n0 + wn * 64;
            auto pack4 = [](const f32x4& v) { return pack_bf16x4(v[0], v[1], v[2], v[3]); };
#pragma unroll
            for (int ib = 0; ib < 4; ++ib) {
                const int mb = cur.m0 + wm * 128 + ib * 32;
                uint2 pk[2][4];
#pragma unroll
                for (int bi = 0; bi < 2; ++bi)
#pragma unroll
                    for (int bj = 0; bj < 4; ++bj) pk[bi][bj] = pack4(acc[2 * ib + bi][bj]);
                uint16_t* out = reinterpret_cast<uint16_t*>(p.C) + (static_cast<size_t>(cur.e) * p.capacity + mb) * p.N + nb;
                if (p.split_m) {                         // a block of 32 rows lies on one side of the split
                    const bool second = mb >= p.split_m;
                    out = reinterpret_cast<uint16_t*>(second ? p.C2 : p.C) +
                          (static_cast<size_t>(cur.e) * p.split_m + (second ? mb - p.split_m : mb)) * p.N + nb;
                }
                if (mb < cur.count && nb < p.N) store_rows_staged_lines(pk, out, p.N, cur.count - mb, p.N - nb, patch, lane);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!has_next) break;
        cur = nxt;
        next_at = after;
        has_next = has_after;
        ++seq;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));   // the re-fetched k-tiles of the last two steps
}
template <bool TRA, int KG, bool TAIL, bool MID>
__global__ __launch_bounds__(512) void gemm_bf16_transposing_kernel(GemmParams p) {
    __shared__ TransposingLds sh;
    DealState state;
    state.idle = gridDim.x;
    transposing_tiles<TRA, KG, TAIL, MID>(p, sh, state);
}

// The last products of the backward in one launch: the input gradient (p[0]: row-major A, TAIL as above), then the weight
// gradients (p[1]: down; p[2] and, with two, p[3]: gate and up), their rows through an index or not (Fetch).  They do
// not depend on each other, and the input gradient is few tiles with a long contraction (2 H): its last round leaves
// workgroups idle, which here start on the weight gradients' many short tiles, as many rounds of them as its k-tiles stand
// for.  Where even so a tile of the input gradient is longer than all the rest (few rows), its contraction comes in parts
// (p[0].pieces, see dx_pieces in backward.hip).  Bound as the kernels above are.  Training step, a launch for each product /
// this, in one part: 12 experts of 677 rows, 1080 x 2744 (180 tiles of 86 k-tiles): 994 / 898 us; 4 of 300, 2048 x 5632: 719 / 639;
// 8 of 512, 1024 x 2816: 482 / 428; 16 of 166-1024, 2048 x 5632 (1.6 rounds, at the power limit): 2678 / 2580; 8 of 64, 2048 x
// 5632: 753 / 646, 32 of 32, 512 x 1024: 186 / 156.
// All instantiations spill: 4 to 7 vector registers in the set-up of a product and of a tile, none in the loop over k-tiles.
struct BackwardProducts { GemmParams p[4]; int n_gates; };
enum class Fetch { NONE, GATES, ALL };                   // contraction rows through an index: B of the gate and up products, A of down too
template <bool TAIL, Fetch FETCH>
__global__ __launch_bounds__(512) void gemm_bf16_backward_kernel(BackwardProducts b) {
    __shared__ TransposingLds sh;
    DealState state;
    state.idle = gridDim.x;
    transposing_tiles<false, 0, TAIL>(b.p[0], sh, state);
    __syncthreads();                                     // the tile list and the buffers are free
    transposing_tiles<true, FETCH == Fetch::ALL ? 1 : 0, false>(b.p[1], sh, state);
    for (int i = 0; i < b.n_gates; ++i) {
        __syncthreads();
        transposing_tiles<true, FETCH == Fetch::NONE ? 0 : 2, false>(b.p[2 + i], sh, state);
    }
}
#undef ETR_OFF
#undef ETR_AT
#undef ETR_OUT
#undef ETR_FRAGS
#undef ETR_ACC
#undef ETR_TR
#undef ETR_MF

// ---------------------------------------------------------------------------------------
// Grouped bf16 GEMM for few rows per group (decode steps, short prompts): the weights are read once and that is all the
// time there is, so a 256-row tile would multiply padding for longer than the weights take to arrive.
//
// A workgroup takes 64 weight rows (GLU: 32 gate and the 32 up rows of the same columns) and up to 64 token rows of one
// expert; wave w has 16 of the weight rows (GLU: 8 and 8) over the whole contraction.  Weights go from memory straight into
// the MFMA fragments (lane l: row l % 16, 16-byte piece l / 16 of a k-step); the token rows, which all four waves need,
// come once per workgroup through LDS.  Both are requested in chunks of two 64-wide k-tiles, two chunks ahead: 8 KiB of
// weights in flight per wave, 64 KiB per CU at two workgroups, and one barrier per chunk.  Pieces past the contraction, in
// the last chunk, come from a zero page.
// LDS rows are 256 bytes; piece j of row r lies at j ^ (r % 16) (applied on the source side of the copy), so that the 16
// lanes of a fragment read touch all banks once.
// Row blocks of 16 that hold no row are skipped (MB = 1, 2 or 4 blocks).
// The products are added in ascending k, 32 at a time, as on the 64-wide persistent kernel, so few rows give the same bits
// as many (a form whose waves split the contraction instead did not, and took 8 % longer at 32 rows and 6-22 % at 64).
// Measured, both products, 256-row tiles / this: 16 experts, 2048 x 5632, 2, 32, 64 rows each: 316 / 187, 328 / 209,
// 331 / 252 us; 32 experts, 4096 x 2816: 507 / 364, 536 / 411, 543 / 483; 8 experts, 512 x 1024: 39 / 12, 40 / 13, 41 / 15.
// (1.11 GB of weights in 187 us: 5.9 TB/s.)
// ---------------------------------------------------------------------------------------
constexpr int kRowsBM = 64;                             // token rows per workgroup
constexpr int kRowsBuffers = 3, kRowsPieces = 16;       // LDS buffers; 16-byte pieces of a staged token row (128 k)

template <int MB, bool GLU, bool DUAL, bool KEEP>
__device__ __forceinline__ void rows_tile(const GemmParams& p, int e, int m0, int n0, int count, uint4* lds) {
    constexpr int BK = 128, KS = BK / 32;               // k per chunk, MFMA k-steps
    constexpr int STAGE = 16 * MB * kRowsPieces;        // pieces per LDS buffer
    constexpr int NCP = MB, LOADS = NCP + KS;           // per wave and chunk: copies (4 rows each), all requests
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kq = lane >> 4;
    const int K = p.K, n_chunks = (K + BK - 1) / BK, n_whole = K / BK;
    const int LA = p.lda ? p.lda : p.K, LB = p.ldb ? p.ldb : p.K;
    typedef const __attribute__((address_space(1))) char* global_bytes;
    typedef const __attribute__((address_space(1))) bf16x8* global_piece;
    const char* zero = reinterpret_cast<const char*>(kZeroPiece);

    // copy i of this wave: rows 4 (wave * NCP + i) .. + 3; this lane's row and piece
    const char* Ab = static_cast<const char*>(p.A) + (p.row_index ? 0 : static_cast<size_t>(e) * p.capacity * LA * 2);
    auto copy_row = [&](int i) { return (wave * NCP + i) * 4 + (lane >> 4); };
    auto copy_piece = [&](int i) { return (lane & 15) ^ (copy_row(i) & 15); };
    uint32_t aoff[NCP];
#pragma unroll
    for (int i = 0; i < NCP; ++i) {
        int m = min(m0 + copy_row(i), count - 1);       // rows past the count replay a valid row; never stored
        if (p.row_index) m = min(max(p.row_index[static_cast<size_t>(e) * p.capacity + m], 0), p.a_rows - 1);
        aoff[i] = (static_cast<uint32_t>(m) * LA + copy_piece(i) * 8) * 2u;
    }
    // this lane's weight row; GLU: 8 gate rows, then the 8 up rows of the same columns
    const int nw = n0 + wave * (GLU ? 8 : 16);
    const int nrow = min(nw + (GLU ? l16 & 7 : l16), p.N - 1);
    const global_bytes wrow = (global_bytes)(static_cast<const char*>(GLU && l16 >= 8 ? p.B1 : p.B0) +
                                             ((static_cast<size_t>(e) * p.N + nrow) * LB + kq * 8) * 2);
    f32x4 acc[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][v] = 0.f;

    struct Weights { bf16x8 w[KS]; };                   // one chunk
    auto request = [&](auto whole, Weights& s, int c, int buf) {        // whole: the chunk does not end past the contraction
        constexpr bool W = decltype(whole)::value;
        const int k0 = c * BK;
        const uint64_t a64 = reinterpret_cast<uint64_t>(Ab) + static_cast<size_t>(k0) * 2;
        const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a64));
        const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a64 >> 32));
        const char* ab = reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
        const global_bytes wp = wrow + static_cast<size_t>(k0) * 2;
#pragma unroll
        for (int q = 0; q < KS; ++q) s.w[q] = *(global_piece)(W || k0 + q * 32 + kq * 8 < K ? wp + q * 64 : (global_bytes)zero);
#pragma unroll
        for (int i = 0; i < NCP; ++i) {
            const char* src = W || k0 + copy_piece(i) * 8 < K ? ab + aoff[i] : zero;
            __builtin_amdgcn_global_load_lds((global_cptr)src, (lds_ptr)(lds + buf * STAGE + (wave * NCP + i) * 64), 16, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // chunk c in buffer buf: this wave's requests for it have landed (those for chunk c + 1 may be in flight); past the
    // barrier that holds for all waves, and the buffer of chunk c - 1 is free for chunk c + 2
    auto step = [&](auto steady, Weights& now, Weights& free, int c, int buf) {         // steady: chunk c + 2 is whole
        constexpr bool S = decltype(steady)::value;
        if (S || c + 1 < n_chunks) __builtin_amdgcn_s_waitcnt(waitcnt_imm(LOADS, true));
        else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (S || c + 2 < n_chunks) request(steady, free, c + 2, buf == 0 ? 2 : buf - 1);
        const uint4* As = lds + buf * STAGE + l16 * kRowsPieces;
        bf16x8 a[KS][MB];
#pragma unroll
        for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int i = 0; i < MB; ++i) a[q][i] = __builtin_bit_cast(bf16x8, As[i * 16 * kRowsPieces + ((4 * q + kq) ^ l16)]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < KS; ++q)
#pragma unroll
            for (int i = 0; i < MB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.w[q], a[q][i], acc[i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr std::integral_constant<bool, true> yes{};
    constexpr std::integral_constant<bool, false> no{};
    static_assert(kRowsBuffers == 3, "step and its callers count three buffers");
    Weights w0, w1, w2;
    int c = 0;
    if (n_whole >= 2) {                                 // (straight into the loop: a wait there must not cover other paths)
        request(yes, w0, 0, 0);
        request(yes, w1, 1, 1);
        for (; c + 5 <= n_whole; c += 3) {
            step(yes, w0, w2, c, 0);
            step(yes, w1, w0, c + 1, 1);
            step(yes, w2, w1, c + 2, 2);
        }
    } else {
        request(no, w0, 0, 0);
        if (n_chunks > 1) request(no, w1, 1, 1);
    }
    for (; c < n_chunks; c += 3) {                      // at most five chunks, the first two of them requested
        step(no, w0, w2, c, 0);
        if (c + 1 < n_chunks) step(no, w1, w0, c + 1, 1);
        if (c + 2 < n_chunks) step(no, w2, w1, c + 2, 2);
    }

    // a lane holds token row l16 of block i and, of the wave's 16 weight rows, 4 kq .. + 3
    const size_t eoff = static_cast<size_t>(e) * p.capacity * p.N;
    auto pack4 = [](const f32x4& v) { return pack_bf16x4(v[0], v[1], v[2], v[3]); };
    const int n = nw + (GLU ? kq & 1 : kq) * 4;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int m = m0 + i * 16 + l16;
        const bool in = m < count && n < p.N;           // N % 4 == 0
        const size_t o = eoff + static_cast<size_t>(m) * p.N + n;
        auto put = [&](void* base, const uint2& v) { *reinterpret_cast<uint2*>(static_cast<uint16_t*>(base) + o) = v; };
        const f32x4 g = acc[i];                         // GLU: the gate product in lanes 0..31, the up product in the others
        if constexpr (!GLU) {
            if (in) put(p.C, pack4(g));
        } else if constexpr (DUAL) {
            if (in) put(kq < 2 ? p.C : p.C2, pack4(g));
        } else {
            f32x4 up;
#pragma unroll
            for (int v = 0; v < 4; ++v) up[v] = __shfl_xor(g[v], 32, kWave);
            if (in && kq < 2) put(p.C, pack_bf16x4(silu(g[0]) * up[0], silu(g[1]) * up[1], silu(g[2]) * up[2], silu(g[3]) * up[3]));
            if constexpr (KEEP) {
                if (in) put(kq < 2 ? p.C2 : p.C3, pack4(g));
            }
        }
    }
}

template <bool GLU, bool DUAL = false, bool KEEP = false>
__global__ __launch_bounds__(256, 2) void gemm_bf16_rows_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(16))) uint4 lds[kRowsBuffers * kRowsBM * kRowsPieces];
    int share, e, mt, nt, count;
    for (int j = blockIdx.x >> 3; decode_live_tile(p, kRowsBM, j, share, e, mt, nt, count);) {
        const int m0 = mt * kRowsBM, n0 = nt * (GLU ? 32 : 64);
        const int rows = count - m0;
        if (rows <= 16) rows_tile<1, GLU, DUAL, KEEP>(p, e, m0, n0, count, lds);
        else if (rows <= 32) rows_tile<2, GLU, DUAL, KEEP>(p, e, m0, n0, count, lds);
        else rows_tile<4, GLU, DUAL, KEEP>(p, e, m0, n0, count, lds);
        j += gridDim.x >> 3;
        if (j >= share) return;
        __syncthreads();                                // every wave has read its last fragments: the buffers are free
    }
}

// ---------------------------------------------------------------------------------------
// fp32 grouped GEMM on v_mfma_f32_16x16x4_f32 (full fp32 products and accumulation).
//
// Bound by the matrix pipe on large layers (157 TFLOP/s dense; plain FMAs, without packed instructions, stop at half of
// that) and by latency on small ones.  One workgroup of four waves (2 x 2) per BM x BN tile; k-tiles of 32 floats, so
// a staged row is 128 bytes and layout, swizzle and fragment addresses are those of the 64-wide bf16 kernel: lane l
// reads row l % 16 and the 16-byte piece 4 ks + l / 16 of a 16-row block, four floats, and MFMA v of the k-step contracts
// component v of both operands (the k order inside a step is permuted alike on both sides).  A ring of NBUF buffers
// is filled by copies that bypass the registers, NBUF - 1 k-tiles ahead; behind the end of the contraction the last
// k-tile is copied again, which keeps the wait count constant.  Copies go through a buffer descriptor whose base moves with the
// k-tile, so a lane carries one 32-bit offset that never changes, and a piece past the contraction, of a row past the group's own or
// of a weight row past the last asks for an offset past the range (see buffer_copy_to_lds).  With the last row in place of those
// it took up to 12 % more where groups end in a nearly empty tile and the widths are ragged, 0.5 % less elsewhere: layer of 32
// experts of 66 rows, 888 x 800: 182 / 162 us; training step of 12 of 500, 1000 x 328 597 / 573, of 8 of 512, 512 x 1024 397 / 398.
// The other form of a copy into LDS is a flat instruction to the compiler, which then waits for every LDS read and every load in
// flight, not for those it needs; with its 64-bit addresses the layer took, 8192 tokens on 8 experts, 1024 x 2048, 1786 us, now 1630;
// 2048 tokens, 512 x 1024 140 / 130; 1024 tokens 108 / 103.  WIDE keeps it, for operands of 4 GiB and more (f32_wide): the zeros
// then come from a zero page, and the last row stands for those past the end.
// Tile: 64 x 64, or 32 x 32 where the capacity gives fewer than two 64 x 64 tiles per CU (see launch_f32).  Measured
// against the plain-FMA kernel this replaces: 8 experts of 66-640 rows, 512 x 1024: gate/up 298 -> 91 us (86 TFLOP/s),
// the plain products 182 -> 60 us on average; 8 experts of 80 rows, 256 x 512: 71 -> 11 us and 55 -> 8 us; 8 x 2048 rows,
// 1024 x 4096: 120 TFLOP/s.  Two waves per SIMD (launch bounds) keep the accumulators out of the accumulation registers,
// whose renaming moves cost 1-4 %.  More buffers, or the barrier between the two k-steps with every fragment read a
// k-step ahead, change nothing (-2 .. +4 % time): what is lost is lost where the waves of two workgroups meet at barriers.
//
// Operands whose contraction index is the slow one (backward; TRB: B is [K][N], TRA: A is [K][M] too): a k-tile is staged as
// [32 k][rows], and lane l takes its elements one by one: row l % 16 of a block at k = 16 ks + 4 (l / 16) + v, 64 bytes of four k
// rows per read.  The 64-byte piece b of k row k is stored at b ^ (k / 4 % 4) (applied on the copy's source side), so that
// the four lie on different banks (32-row tiles have two pieces: two-way conflicts).  With B1 the contraction is split in the
// middle ([K/2][ldb] each; the k-tiles of each half are its own, the last one may be short); with k_gather (1: A, 2: B) the k
// rows of that operand are rows k_index[g * k_index_stride + k] of one [k_rows][ld] matrix.
// ---------------------------------------------------------------------------------------
template <int BM, int BN, int NBUF, bool GLU> constexpr int f32_pieces() { return NBUF * (BM + (GLU ? 2 : 1) * BN) * 8; }
// tile j of this XCD's share of the list; lds: f32_pieces
template <int BM, int BN, int NBUF, bool GLU, bool DUAL, bool TRA, bool TRB, bool WIDE>
__device__ __forceinline__ void gemm_f32_tile(const GemmParams& p, int j, uint4* lds) {
    static_assert(!GLU || !TRB, "epilogues: row-major operands");
    static_assert(!TRA || TRB, "transposed A: both are");
    constexpr int CPR = 8, BK = 32, NB = GLU ? 2 : 1, BROWS = NB * BN;
    constexpr int STAGE = (BM + BROWS) * CPR;           // 16-byte pieces per buffer
    constexpr int NCA = BM / 32, NCB = BROWS / 32;      // copies (1 KiB: 8 rows x 128 bytes, or 4 k rows x 256) per wave and k-tile
    constexpr int TM = BM / 32, TN = BN / 32;           // 16 x 16 blocks per wave and product
    constexpr int AHEAD = NBUF - 1;
    int share, e, mt, nt, count;
    if (!decode_live_tile(p, BM, j, share, e, mt, nt, count, TRA)) return;
    const int m0 = mt * BM, n0 = nt * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // (transposed: zeros stand for the k rows past the group's own, so that no padding is multiplied)
    const int K = TRA ? (p.k_counts ? min(max(p.k_counts[e], 0), p.K) : p.K) : group_k(p, e);
    const bool splitB = TRB && !TRA && p.B1 != nullptr;
    const int Kh = splitB ? K / 2 : K, KTh = max((Kh + BK - 1) / BK, 1), KT = splitB ? 2 * KTh : KTh;   // of a half, of all
    const int k_rem = Kh - (KTh - 1) * BK;               // valid k of the last k-tile of a half
    const int LA = p.lda ? p.lda : p.K, LB = p.ldb ? p.ldb : p.K;

    // copy sources: a wave-uniform base and this lane's offset in bytes: row and 16-byte piece (the swizzle is applied here, on the
    // source side)
    typedef std::conditional_t<WIDE, size_t, uint32_t> Offset;
    Offset off[NCA + NCB];
    const int r8 = lane >> 3;
    bool past[2];                                       // row-major: piece of the last k-tile that lies past the contraction
#pragma unroll
    for (int h = 0; h < 2; ++h) past[h] = 4 * ((lane & 7) ^ ((4 * h + (lane >> 4)) & 7)) >= k_rem;
    // transposed: k row of copy i of a wave's NC and first row of the piece
    constexpr int PA = BM / 4, PB = BN / 4;             // 16-byte pieces of a k row
    auto k_of = [&](int i, int NC, int pieces) { return ((wave * NC + i) * 64 + lane) / pieces; };
    auto r_of = [&](int i, int NC, int pieces) {
        const int slot = ((wave * NC + i) * 64 + lane) % pieces;
        return 16 * ((slot >> 2) ^ ((k_of(i, NC, pieces) >> 2) & (pieces / 4 - 1))) + 4 * (slot & 3);
    };
    const bool gathered_a = TRA && p.k_gather == 1, gathered_b = TRA && p.k_gather == 2;       // (their k rows come from `rows`)
#pragma unroll
    for (int i = 0; i < NCA; ++i) {
        if constexpr (TRA) {                            // (pieces past the row repeat; never stored)
            off[i] = (static_cast<Offset>(gathered_a ? 0 : k_of(i, NCA, PA)) * LA + min(m0 + r_of(i, NCA, PA), p.capacity - 4)) * 4;
        } else {
            const int r = (wave * NCA + i) * 8 + r8;
            int m = min(m0 + r, count - 1);
            if (p.row_index) m = min(max(p.row_index[static_cast<size_t>(e) * p.capacity + m], 0), p.a_rows - 1);
            off[i] = (static_cast<Offset>(m) * LA + 4 * ((lane & 7) ^ ((r >> 1) & 7))) * 4;
            if (!WIDE && m0 + r >= count) off[i] = kPastRange;           // (never stored; WIDE: a valid row again)
        }
    }
#pragma unroll
    for (int i = 0; i < NCB; ++i) {
        if constexpr (TRB) {
            off[NCA + i] = (static_cast<Offset>(gathered_b ? 0 : k_of(i, NCB, PB)) * LB + min(n0 + r_of(i, NCB, PB), p.N - 4)) * 4;
        } else {
            const int r = (wave * NCB + i) * 8 + r8;
            const int n = n0 + (GLU && r >= BN ? r - BN : r);
            off[NCA + i] = (static_cast<Offset>(min(n, p.N - 1)) * LB + 4 * ((lane & 7) ^ ((r >> 1) & 7))) * 4;
            if (!WIDE && n >= p.N) off[NCA + i] = kPastRange;
        }
    }
    const uint64_t a_base = reinterpret_cast<uint64_t>(p.A) +
                            (gathered_a || (!TRA && p.row_index) ? 0 : static_cast<uint64_t>(e) * (TRA ? p.K : p.capacity) * LA * 4);
    const uint64_t b_group = gathered_b ? 0 : static_cast<uint64_t>(e) * (TRB ? (splitB ? p.K / 2 : p.K) : p.N) * LB * 4;
    // row numbers of this lane's gathered k rows in the k-tile requested next
    constexpr int NG = TRA ? (NCA > NCB ? NCA : NCB) : 1;
    int rows[NG], rows_next[NG];
    auto load_rows = [&](int kt, int (&rows)[NG]) {
        if constexpr (TRA) {
            if (p.k_gather) {
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    const int k = min(kt, KT - 1) * BK + (p.k_gather == 1 ? k_of(i < NCA ? i : 0, NCA, PA) : k_of(i < NCB ? i : 0, NCB, PB));
                    rows[i] = min(max(p.k_index[static_cast<size_t>(e) * p.k_index_stride + min(k, p.k_index_stride - 1)], 0), p.k_rows - 1);
                }
            }
        }
    };
    auto copy_tile = [&](int kt, int buf) {
        const bool second = splitB && kt >= KTh;         // half of a split contraction
        const int kh = second ? kt - KTh : kt;
        const bool last = kh == KTh - 1;
        const uint64_t row_step = static_cast<uint64_t>(kh) * (BK * 4);
        const uint64_t a_at = a_base + (TRA ? (gathered_a ? 0 : row_step * LA) : row_step + (second ? static_cast<uint64_t>(Kh) * 4 : 0));
        const uint64_t b_step = TRB ? (gathered_b ? 0 : row_step * LB) : row_step;
#pragma unroll
        for (int i = 0; i < NCA + NCB; ++i) {
            const bool a = i < NCA;
            const int n = a ? i : i - NCA, group = wave * (a ? NCA : NCB) + n;           // of 8 rows; its parity picks the swizzle half
            const bool up = !a && (second || (GLU && group * 8 >= BN));
            const uint64_t at = a ? a_at : reinterpret_cast<uint64_t>(up ? p.B1 : p.B0) + b_group + b_step;
            Offset o = off[i];
            bool over = last && past[group & 1];
            if (a ? TRA : TRB) {
                over = last && (a ? k_of(n, NCA, PA) : k_of(n, NCB, PB)) >= k_rem;
                if (a ? gathered_a : gathered_b) o += static_cast<Offset>(rows[n < NG ? n : 0]) * (a ? LA : LB) * 4;
            }
            uint4* dst = lds + buf * STAGE + (a ? 0 : BM * CPR) + group * 64;
            if constexpr (WIDE) {
                const char* g = over ? reinterpret_cast<const char*>(kZeroPiece) : reinterpret_cast<const char*>(at) + o;
                __builtin_amdgcn_global_load_lds((global_cptr)g, (lds_ptr)dst, 16, 0, 0);
            } else {
                const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at));
                const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(at >> 32));
                buffer_copy_to_lds(lo, hi, over ? kPastRange : o, dst);
            }
        }
    };

    f32x4 acc[NB][TM][TN];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int n = 0; n < TN; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[b][i][n][v] = 0.f;

    for (int t = 0; t < AHEAD; ++t) {
        load_rows(t, rows);
        copy_tile(min(t, KT - 1), t);
    }
    load_rows(AHEAD, rows);
    const int l16 = lane & 15, kq = lane >> 4;
    const int ck[2] = {kq ^ (l16 >> 1), (4 + kq) ^ (l16 >> 1)};
    // fragment of the 16-row block blk of an operand of `pieces` pieces a k row
    auto transposed = [&](const uint4* at, int pieces, int blk, int ks) {
        const float* f = reinterpret_cast<const float*>(at) + (16 * ks + 4 * kq) * pieces * 4 + 16 * (blk ^ (kq & (pieces / 4 - 1))) + l16;
        return f32x4{f[0], f[pieces * 4], f[pieces * 8], f[pieces * 12]};
    };
    int buf = 0;
    for (int kt = 0; kt < KT; ++kt) {
        // this wave's share of k-tile kt has landed and its reads of k-tile kt - 1 are done; past the barrier that
        // holds for all waves, and the buffer of k-tile kt - 1 is free
        __builtin_amdgcn_s_waitcnt(waitcnt_imm((AHEAD - 1) * (NCA + NCB), true));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const uint4* Ab = lds + buf * STAGE;
        const uint4* Bb = Ab + BM * CPR;
        const uint4* As = Ab + (wm * (BM / 2) + l16) * CPR;
        const uint4* Bs = Bb + (wn * (BN / 2) + l16) * CPR;
        f32x4 fas[2][TM], fbs[2][NB][TN];
        auto read = [&](int ks) {
            auto& fa = fas[ks]; auto& fb = fbs[ks];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if constexpr (TRA) fa[i] = transposed(Ab, PA, wm * TM + i, ks);
                else fa[i] = __builtin_bit_cast(f32x4, As[i * 16 * CPR + ck[ks]]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int n = 0; n < TN; ++n) {
                    if constexpr (TRB) fb[b][n] = transposed(Bb, PB, wn * TN + n, ks);
                    else fb[b][n] = __builtin_bit_cast(f32x4, Bs[(b * BN + n * 16) * CPR + ck[ks]]);
                }
        };
        auto multiply = [&](int ks, int v0, int v1) {
            auto& fa = fas[ks]; auto& fb = fbs[ks];
#pragma unroll
            for (int v = v0; v < v1; ++v)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int n = 0; n < TN; ++n)
                            acc[b][i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[b][n][v], fa[i][v], acc[b][i][n], 0, 0, 0);
        };
        // The copies go out behind a quarter of the first k-step's MFMAs, the second one's fragments are asked for behind three:
        // before both, or with the copies in front, LDS and the address unit are busy while the matrix pipe waits.  2048 tokens on 8
        // experts, 512 x 1024, training step: copies, fragments, MFMAs 434 us; first fragments, copies, MFMAs 400; this 395 (copies
        // behind half 396, behind all 407).
        read(0);
        __builtin_amdgcn_sched_barrier(0);
        load_rows(kt + AHEAD + 1, rows_next);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        copy_tile(min(kt + AHEAD, KT - 1), buf == 0 ? NBUF - 1 : buf - 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, 1, 3);
        __builtin_amdgcn_sched_barrier(0);
        read(1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, 3, 4);
        multiply(1, 0, 4);
        buf = buf == NBUF - 1 ? 0 : buf + 1;
#pragma unroll
        for (int i = 0; i < NG; ++i) rows[i] = rows_next[i];
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));    // the copies past the end: nothing may land in LDS after the wave

    // lane l holds row l % 16 and the four columns 4 (l / 16) .. + 3 of each block
    const size_t eoff = static_cast<size_t>(e) * p.capacity * p.N;
    float* Cg = static_cast<float*>(p.C) + eoff;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * (BM / 2) + i * 16 + l16;
        if (m >= count) continue;
#pragma unroll
        for (int c = 0; c < TN; ++c) {
            const int n = n0 + wn * (BN / 2) + c * 16 + kq * 4;
            if (n >= p.N) continue;                               // N % 4 == 0
            const size_t o = static_cast<size_t>(m) * p.N + n;
            f32x4 r = acc[0][i][c];
            if constexpr (GLU) {
                const f32x4 u = acc[1][i][c];
                if constexpr (DUAL) {
                    *reinterpret_cast<f32x4*>(static_cast<float*>(p.C2) + eoff + o) = u;
                } else {
                    if (p.C3) {                                   // keep the pre-activations (training-mode forward)
                        *reinterpret_cast<f32x4*>(static_cast<float*>(p.C2) + eoff + o) = r;
                        *reinterpret_cast<f32x4*>(static_cast<float*>(p.C3) + eoff + o) = u;
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) r[v] = r[v] / (1.0f + expf(-r[v])) * u[v];
                }
            }
            *reinterpret_cast<f32x4*>(Cg + o) = r;
        }
    }
}
template <int BM, int BN, int NBUF, bool GLU, bool DUAL, bool TRB, bool WIDE>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(16))) uint4 lds[f32_pieces<BM, BN, NBUF, GLU>()];
    gemm_f32_tile<BM, BN, NBUF, GLU, DUAL, false, TRB, WIDE>(p, blockIdx.x >> 3, lds);
}

// The last products of the backward in one launch, as in gemm_bf16_backward_kernel: the workgroups of p[0], the input
// gradient, come first, and the tiles of the weight gradients fill in behind them as CUs fall free.
// Training step, the operands transposed in memory and a launch for each product / this: 8 experts of 66-640 rows, 512 x 1024:
// 499 / 435 us; 8 of 1200, 1024 x 2048: 2754 / 2322; 4 of 64, 256 x 512: 88 / 63.
struct BackwardProductsF32 { GemmParams p[4]; int first[4]; };       // first[i]: workgroup at which product i begins (a multiple of 8)
template <int BM, int BN, int NBUF, bool WIDE>
__global__ __launch_bounds__(256, 2) void gemm_f32_backward_kernel(BackwardProductsF32 b) {
    __shared__ __attribute__((aligned(16))) uint4 lds[f32_pieces<BM, BN, NBUF, false>()];
    const int blk = blockIdx.x;
    if (blk < b.first[1]) {
        gemm_f32_tile<BM, BN, NBUF, false, false, false, true, WIDE>(b.p[0], blk >> 3, lds);
        return;
    }
    const int i = blk >= b.first[3] ? 3 : (blk >= b.first[2] ? 2 : 1);
    gemm_f32_tile<BM, BN, NBUF, false, false, true, true, WIDE>(b.p[i], (blk - b.first[i]) >> 3, lds);
}

template <int BM, int BN, int BK, int WGM, int WGN, bool GLU, int SWZ, bool DUAL = false>
hipError_t launch_bf16(GemmParams p, hipStream_t st) {
    constexpr int BROWS = GLU ? 2 * BN : BN;
    constexpr size_t lds = 2ull * (BM + BROWS) * BK * 2;
    const long long blocks = plan_tiles(p, BM, BN);
    auto kern = gemm_bf16_kernel<BM, BN, BK, WGM, WGN, GLU, SWZ, DUAL>;
    hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(WGM * WGN * 64), lds, st, p);
    return hipGetLastError();
}

template <bool GLU, int WN = 2, bool DUAL = false, int NBUF = 4>
hipError_t launch_bf16_ring(GemmParams p, hipStream_t st) {
    constexpr size_t lds = static_cast<size_t>(NBUF) * 512 * 32 * 2;        // NBUF buffers of 256 + 256 rows x 32 bf16
    const long long blocks = plan_tiles(p, 256, GLU ? 128 : 256);
    auto kern = gemm_bf16_ring_kernel<GLU, WN, DUAL, NBUF>;
    hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(128 * WN), lds, st, p);
    return hipGetLastError();
}

// Transposing kernel: needs every group's contraction length >= 128 (two k-tiles to prefetch; 256 where it fetches rows
// through an index) and the super-tile prefix to fit in LDS.
template <bool TRA, int KG, bool TAIL = false, bool MID = false>
hipError_t launch_bf16_transposing(GemmParams p, hipStream_t st, int n_cu) {
    constexpr size_t lds = 2ull * 512 * 64 * 2;                             // two buffers of 256 + 256 rows x 64 bf16
    plan_tiles(p, 256, 256);
    auto kern = gemm_bf16_transposing_kernel<TRA, KG, TAIL, MID>;
    hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(n_cu / 8 * 8)), dim3(512), lds, st, p);
    return hipGetLastError();
}
template <bool TAIL, Fetch FETCH>
hipError_t launch_bf16_backward_form(BackwardProducts b, hipStream_t st, int n_cu) {
    constexpr size_t lds = 2ull * 512 * 64 * 2;
    for (int i = 0; i < 2 + b.n_gates; ++i) plan_tiles(b.p[i], 256, 256);
    b.p[0].NT *= b.p[0].pieces;
    auto kern = gemm_bf16_backward_kernel<TAIL, FETCH>;
    hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(n_cu / 8 * 8)), dim3(512), lds, st, b);
    return hipGetLastError();
}
template <bool GLU, bool DUAL = false, bool KEEP = false, bool TAIL = false>
hipError_t launch_bf16_persistent_form(GemmParams p, hipStream_t st, int n_cu) {
    constexpr size_t lds = 2ull * 512 * 64 * 2;                             // two buffers of 256 + 256 rows x 64 bf16
    plan_tiles(p, 256, GLU ? 128 : 256, true);
    auto kern = gemm_bf16_persistent_kernel<GLU, DUAL, KEEP, TAIL>;
    hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(n_cu / 8 * 8)), dim3(512), lds, st, p);
    return hipGetLastError();
}
template <bool GLU, bool DUAL = false, bool KEEP = false>
hipError_t launch_bf16_persistent(GemmParams p, hipStream_t st, int n_cu) {
    return p.K % 64 == 0 ? launch_bf16_persistent_form<GLU, DUAL, KEEP, false>(p, st, n_cu)
                         : launch_bf16_persistent_form<GLU, DUAL, KEEP, true>(p, st, n_cu);
}
// the 64-wide persistent kernel bounds no weight-row address: at least one whole column tile, and 16-byte stores
// (its ragged last tile overlaps the one before)
inline bool whole_column_tiles(const GemmParams& g, bool glu) { return g.N >= (glu ? 128 : 256) && g.N % 8 == 0; }
// wide: the row-major kernel's super-tiles (see plan_tiles)
inline bool persist_ok(const GemmParams& g, bool glu, bool wide, int max_super) {
    GemmParams t = g;
    plan_tiles(t, 256, glu ? 128 : 256, wide);
    const long long MG = (t.MT + t.SM - 1) / t.SM, NG = (t.NT + t.SN - 1) / t.SN;
    // (with k_counts the contraction is at least min(128, K) long: two k-tiles)
    return g.K >= 128 && static_cast<long long>(g.E) * MG * NG <= max_super;
}

// Workgroups for decode_live_tile: every tile of the capacity, in whole rounds of the 8 XCDs.
inline long long plan_live_tiles(GemmParams& p, int BM, int BN) {
    p.MT = (p.capacity + BM - 1) / BM;
    p.NT = (p.N + BN - 1) / BN;
    return (static_cast<long long>(p.E) * p.MT * p.NT + 7) / 8 * 8;
}
// Workgroups of the few-rows kernel: one for every tile that rows_total rows in E groups can fill (each group ends in
// one partial row tile at most), never more than the capacity has.  A buffer made once for the largest batch costs
// nothing then: 32 tokens on 16 experts of 2048 x 5632, capacity 32 / 4096: 206 / 214 us for the layer, where a grid of
// the whole capacity took 207 / 429 (256-row tiles: 354 / 369).  Counts beyond rows_total (rows that other processes
// sent) send workgroups round their loop again.
inline long long plan_rows(GemmParams& p, bool glu) {
    const long long all = plan_live_tiles(p, kRowsBM, glu ? 32 : 64);
    constexpr long long kMost = 1 << 23;                 // 2^31 threads: within what one launch may hold
    const long long live = p.rows_total > 0 ? ((p.E + p.rows_total / kRowsBM) * p.NT + 7) / 8 * 8 : all;
    return std::min({all, live, kMost});
}
template <bool GLU, bool DUAL = false, bool KEEP = false>
hipError_t launch_bf16_rows(GemmParams p, hipStream_t st) {
    const long long blocks = plan_rows(p, GLU);
    hipLaunchKernelGGL((gemm_bf16_rows_kernel<GLU, DUAL, KEEP>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, p);
    return hipGetLastError();
}
// Whether a product gets 64 x 64 tiles (two per CU at least) or 32 x 32 ones.  8 experts of 80 rows, 256 x 512 (128 and 64
// tiles of 64 x 64): 11 and 8 us with 32 x 32 tiles, 15 and 14 with 64 x 64
inline bool f32_large_tiles(const GemmParams& p) {
    return static_cast<long long>(p.E) * ((p.capacity + 63) / 64) * ((p.N + 63) / 64) >= 2ll * cu_count();
}
// Whether the byte offsets of a product's copies, which span a group's rows (operands with the contraction slow: a k-tile, or the
// rows that the index may name), need more than the 32 bits of a buffer descriptor's range.
inline bool f32_wide(const GemmParams& p, bool ta, bool tb) {
    const size_t a_row = static_cast<size_t>(p.lda ? p.lda : p.K) * 4, b_row = static_cast<size_t>(p.ldb ? p.ldb : p.K) * 4;
    const size_t a_rows = ta ? (p.k_gather == 1 ? p.k_rows : 32) : (p.row_index ? p.a_rows : p.capacity);
    const size_t b_rows = tb ? (p.k_gather == 2 ? p.k_rows : 32) : p.N;
    return (a_rows + 1) * a_row >= kBufferRange || (b_rows + 1) * b_row >= kBufferRange;
}
template <bool GLU, bool DUAL, bool TRB, bool WIDE>
hipError_t launch_f32_form(GemmParams p, hipStream_t st) {
    if (f32_large_tiles(p)) {
        const long long blocks = plan_live_tiles(p, 64, 64);
        hipLaunchKernelGGL((gemm_f32_kernel<64, 64, 3, GLU, DUAL, TRB, WIDE>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, p);
    } else {
        const long long blocks = plan_live_tiles(p, 32, 32);
        hipLaunchKernelGGL((gemm_f32_kernel<32, 32, 4, GLU, DUAL, TRB, WIDE>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, p);
    }
    return hipGetLastError();
}
template <bool GLU, bool DUAL = false, bool TRB = false>
hipError_t launch_f32(const GemmParams& p, hipStream_t st) {
    return f32_wide(p, false, TRB) ? launch_f32_form<GLU, DUAL, TRB, true>(p, st) : launch_f32_form<GLU, DUAL, TRB, false>(p, st);
}
// Products [from, to) of b in one launch (as many workgroups as one launch may hold, else one by one).
template <int T, int NBUF>
hipError_t launch_f32_backward_tiles(BackwardProductsF32 b, int from, int to, hipStream_t st) {
    long long at = 0;
    bool wide = false;
    for (int i = 0; i < 4; ++i) {
        b.first[i] = static_cast<int>(std::min<long long>(at, 1 << 30));
        if (i >= from && i < to) {
            at += (plan_live_tiles(b.p[i], T, T) + 63) / 64 * 64;
            wide = wide || f32_wide(b.p[i], i > 0, true);
        }
    }
    if (at > (1 << 23) && to - from > 1) {               // 2^31 threads
        for (int i = from; i < to; ++i) {
            const hipError_t err = launch_f32_backward_tiles<T, NBUF>(b, i, i + 1, st);
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    auto kern = wide ? gemm_f32_backward_kernel<T, T, NBUF, true> : gemm_f32_backward_kernel<T, T, NBUF, false>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(at)), dim3(256), 0, st, b);
    return hipGetLastError();
}

}  // namespace

size_t ffn_ws_bytes(const etr_config& c) {
    return align_up(static_cast<size_t>(c.E) * c.capacity * c.H * elt_bytes(c.dtype));
}

// Which kernel a row-major bf16 product takes.  Both pipelined kernels need 32-bit byte offsets inside one operand.
//   PERSISTENT  at least one whole column tile, a contraction of 128 or more, the super-tile prefix in LDS.  A
//               contraction that is not whole 64-wide k-tiles takes its zero-filling instantiation (per-group lengths
//               are always whole k-tiles).
//   RING        whole k-tiles where the persistent kernel does not apply (narrow outputs, short contractions)
//   ROWS        any width; few rows per group, or too few 256-row tiles to fill the chip
//   STAGED      any width; the only one without a limit on sizes
// Without a row count: the first of PERSISTENT, RING, STAGED that applies.  With one, by estimate.
enum class Bf16Kernel { ROWS, PERSISTENT, RING, STAGED };
// Estimated microseconds of a product whose groups have about `rows` rows each: rounds of tiles over the CUs, each a time
// per 64-wide k-tile and a time besides, and at least the weights at the rate that the kernel reads them with.
//   ROWS        tiles of 64 rows x 64 staged weight rows, two on a CU at once: 0.58 us per two k-tiles (0.47 and 0.25 for a
//               lone block of 32 or 16 rows) and 0.95 us; 5.2 TB/s; 2.8 us per launch
//   PERSISTENT  256-row tiles: 1.13 us per k-tile where few CUs have one, 1.69 on a full chip (its power limit), 1.08 times
//               that with zero-filling copies, and 1.65 us; 4.65 TB/s; 5 us
//   RING        the same tiles: 1.03 us per k-tile and 7 us
//   STAGED      128-row tiles: 0.87 us per k-tile in the first round, 0.66 in the others (two run on a CU at once), and 3.3 us
//               for each two rounds; 4.5 TB/s; 0.4 us
// RING and STAGED deal super-tiles of the capacity to the XCDs (decode_tile): their rounds are those of the busiest XCD,
// where a super-tile that is live in part keeps its CUs worse than in proportion, and their dead workgroups take 2 and
// 0.5 us per one of each CU.  4 rows in each of 16 experts, 2048 x 5632, capacity 256 / 1024 / 4096 / 16384: RING 329 / 667 / 2600 /
// 4980 us for both products, ROWS 190 throughout.
// Fitted to 7190 measured products: 2 to 64 groups of 1 to 13 000 rows, even and uneven counts, capacities of 1 to 4 times
// that, widths from 8 to 11008, half of them ragged.  A kernel newer than the ones that took everything once (PERSISTENT and
// RING for whole k-tiles, STAGED for ragged ones) has to be estimated 5 % faster.  Against those the geometric mean is 0.63
// of the time and 69 products are more than 3 % (and 1 us) slower; against the best kernel of each product it is 1.009.
static double estimate_us(Bf16Kernel kernel, const GemmParams& g, bool glu, int rows) {
    const double n_cu = cu_count(), weight_bytes = 2.0 * g.E * g.N * (glu ? 2 : 1) * g.K;
    const int KT = (g.K + 63) / 64;
    auto least = [&](double us, double terabytes_per_s) { return std::max(us, weight_bytes / (terabytes_per_s * 1e6)); };
    // live row tiles of a group: half a tile more than the rows fill, on average, up to the capacity
    auto row_tiles = [&](int BM) {
        return std::min<double>((g.capacity + BM - 1) / BM, std::max<double>((rows + BM - 1) / BM, static_cast<double>(rows) / BM + 0.5));
    };
    auto tiles = [&](int BM, int BN) { return g.E * row_tiles(BM) * ((g.N + BN - 1) / BN); };
    // super-tile dealing: live tiles of the busiest XCD, and dead workgroups per CU
    auto deal = [&](int BM, int BN, double& busiest, double& dead) {
        GemmParams p = g;
        plan_tiles(p, BM, BN);
        const int MG = (p.MT + p.SM - 1) / p.SM, NG = (p.NT + p.SN - 1) / p.SN;
        const double live = row_tiles(BM), live_groups = std::ceil(live / p.SM);
        const double xcds = std::min(8.0, 8 / std::gcd(MG, 8) * live_groups);         // that the live super-tiles fall on
        busiest = std::ceil(g.E * NG * live_groups / xcds) * p.SN * std::sqrt(p.SM * live / live_groups);
        dead = (static_cast<double>(g.E) * MG * NG * p.SM * p.SN - tiles(BM, BN)) / n_cu;
    };
    double busiest, dead;
    switch (kernel) {
        case Bf16Kernel::ROWS: {
            const double step = rows <= 16 ? 0.25 : (rows <= 32 ? 0.47 : 0.58), rounds = tiles(kRowsBM, glu ? 32 : 64) / n_cu;
            return least((rounds <= 1 ? 1.0 : rounds + 0.37) * ((g.K + 127) / 128 * step + 0.95), 5.2) + 2.8;
        }
        case Bf16Kernel::PERSISTENT: {
            const double t = tiles(256, glu ? 128 : 256), step = (1.13 + 0.56 * std::min(1.0, t / n_cu)) * (g.K % 64 ? 1.08 : 1.0);
            return least(std::ceil(t / n_cu) * (KT * step + 1.65), 4.65) + 5.0;
        }
        case Bf16Kernel::RING:
            deal(256, glu ? 128 : 256, busiest, dead);
            return std::ceil(busiest / (n_cu / 8)) * (KT * 1.03 + 7.0) + 2.0 * dead;
        case Bf16Kernel::STAGED:
            deal(128, glu ? 64 : 128, busiest, dead);
            return least(KT * (0.21 + 0.66 * std::ceil(busiest / (n_cu / 8))) + std::ceil(busiest / (n_cu / 4)) * 3.3, 4.5) + 0.4 + 0.5 * dead;
    }
    return 0.0;
}
static Bf16Kernel choose_bf16(const GemmParams& g, bool glu, size_t a_rows, int rows_expected) {
    const size_t a_row_bytes = static_cast<size_t>(g.lda ? g.lda : g.K) * 2, b_row_bytes = static_cast<size_t>(g.ldb ? g.ldb : g.K) * 2;
    const size_t a_bytes = a_rows * a_row_bytes, b_bytes = static_cast<size_t>(g.N) * b_row_bytes;
    if (g.K % 8 != 0 || a_row_bytes % 16 != 0 || b_row_bytes % 16 != 0 || a_bytes >= (1ull << 32) || b_bytes >= (1ull << 32))
        return Bf16Kernel::STAGED;
    const bool whole = g.K % 64 == 0;
    const bool persistent = persist_ok(g, glu, true, kMaxSuperWide) && whole_column_tiles(g, glu) &&
                            a_bytes < kBufferRange && b_bytes < kBufferRange && (whole || !g.k_counts);
    if (rows_expected <= 0 || g.k_counts)
        return persistent ? Bf16Kernel::PERSISTENT : (whole ? Bf16Kernel::RING : Bf16Kernel::STAGED);
    Bf16Kernel best = !whole ? Bf16Kernel::STAGED : (persistent ? Bf16Kernel::PERSISTENT : Bf16Kernel::RING);
    double best_us = 0.95 * estimate_us(best, g, glu, rows_expected);
    auto offer = [&](Bf16Kernel kernel) {
        const double us = estimate_us(kernel, g, glu, rows_expected);
        if (us < best_us) { best = kernel; best_us = us; }
    };
    offer(Bf16Kernel::ROWS);
    if (!whole && persistent) offer(Bf16Kernel::PERSISTENT);
    return best;
}

// General entry for the other stages of the library: grouped "NT" product
//   C[g][m][n] = sum_k A[g][m][k] * B[g][n][k],  g < G, m < m_counts[g] (or M), k < k_counts[g] (or K).
static GemmParams params_of(const GroupedGemm& q) {
    GemmParams g{q.A, q.B0, q.B1, q.C, q.m_counts, q.G, q.M, q.N, q.K, 0, 0, 0, 0, q.row_index, q.a_rows};
    g.lda = q.lda; g.ldb = q.ldb; g.k_counts = q.k_counts; g.C2 = q.C2;
    g.k_index = q.k_index; g.k_index_stride = q.k_index_stride; g.k_rows = q.k_rows; g.k_gather = q.k_gather;
    g.split_m = q.split_m;
    g.rows_total = q.rows_total;
    g.pieces = q.pieces;
    g.mid_a = q.mid_a; g.mid_b = q.mid_b; g.mid_gate = q.mid_gate; g.mid_part = q.mid_part;
    g.mid_rows = q.mid_rows; g.mid_scale_h = q.mid_scale_h ? 1 : 0;
    return g;
}

// bf16 operands stored with the contraction index slow run only on the transposing kernel.
bool grouped_gemm_transposed_ok(const GroupedGemm& q) {
    if (q.dtype != ETR_BF16 || (q.epilogue != GEMM_PLAIN && q.epilogue != GEMM_MIDDLE) || !q.tb) return false;
    if (q.epilogue == GEMM_MIDDLE && (q.ta || q.B1 || !q.row_index || !q.C2 || !q.mid_a || !q.mid_b || !q.mid_gate || !q.mid_part || q.mid_rows < q.M ||
                                          static_cast<size_t>(q.mid_rows) * 4 * q.N >= kBufferRange)) return false;
    // (row-major A and transposed B take any multiple of 8; a contraction over padded rows is whole k-tiles anyway)
    if (q.N % 8 != 0 || q.N < 8) return false;                     // 16-byte stores, and chunks along the rows of a [K][rows] operand
    if (!q.ta && q.k_counts) return false;
    const bool tail_form = !q.ta;
    const int half_k = q.B1 ? q.K / 2 : q.K;
    if (q.K < 128 || half_k % (tail_form ? 8 : 64) != 0) return false;
    if (q.ta && (q.M % 8 != 0 || q.M < 8)) return false;
    const int lda = q.lda ? q.lda : q.K, ldb = q.ldb ? q.ldb : q.K;
    if (lda % 8 != 0 || ldb % 8 != 0) return false;
    if (q.ta && (q.row_index || q.m_counts)) return false;
    if (q.B1 && !(tail_form && q.K % 2 == 0)) return false;                      // split B: two halves of the contraction
    // 32-bit per-lane offsets inside one k-tile / one operand
    const size_t a_span = q.ta ? 64ull * lda * 2 : (q.row_index ? static_cast<size_t>(q.a_rows) : static_cast<size_t>(q.M)) * lda * 2;
    const size_t b_span = 64ull * ldb * 2;
    const size_t limit = half_k % 64 == 0 ? (1ull << 32) : kBufferRange;          // zero-filling copies: see buffer_copy_to_lds
    if (a_span >= limit || b_span >= limit) return false;
    if (q.split_m && (!q.ta || q.split_m % 32 != 0 || q.M != 2 * q.split_m || !q.C2 || q.m_counts)) return false;
    if (q.k_gather) {
        // gathered contraction rows: both operands transposed, four k-tiles per group at least, 32-bit row offsets
        if (!(q.ta && q.tb) || (q.k_gather != 1 && q.k_gather != 2) || !q.k_index || q.k_index_stride < 1 || q.k_rows < 1) return false;
        if (q.K < 256 || q.B1) return false;
        if (static_cast<size_t>(q.k_rows) * (q.k_gather == 1 ? lda : ldb) * 2 >= (1ull << 32)) return false;
    }
    return persist_ok(params_of(q), false, false, kMaxSuper);
}

hipError_t launch_backward_products(const GroupedGemm& dx, const GroupedGemm& down, const GroupedGemm* gates, int n_gates, hipStream_t st) {
    if (dx.dtype == ETR_F32) {
        BackwardProductsF32 f{};
        long long tiles = 0;
        for (int i = 0; i < 2 + n_gates; ++i) {
            const GroupedGemm& q = i == 0 ? dx : (i == 1 ? down : gates[i - 2]);
            if (!q.tb || q.ta != (i > 0) || q.split_m || q.N < 8 || q.M < 4 || (i > 0 && q.M < 8)) return hipErrorInvalidValue;
            f.p[i] = params_of(q);
            tiles += static_cast<long long>(q.G) * ((q.M + 63) / 64) * ((q.N + 63) / 64);
        }
        return tiles >= 2ll * cu_count() ? launch_f32_backward_tiles<64, 3>(f, 0, 2 + n_gates, st)
                                         : launch_f32_backward_tiles<32, 4>(f, 0, 2 + n_gates, st);
    }
    BackwardProducts b{};
    if (n_gates < 1 || n_gates > 2 || dx.ta || !down.ta || down.k_gather == 2) return hipErrorInvalidValue;
    if (down.k_gather && !gates[0].k_gather) return hipErrorInvalidValue;
    const Fetch fetch = down.k_gather ? Fetch::ALL : (gates[0].k_gather ? Fetch::GATES : Fetch::NONE);
    if (dx.pieces > 1) {                                 // parts of two k-tiles at least, and the list of their tiles in LDS
        const int half = dx.B1 ? dx.K / 2 : dx.K, k_all = (half + 63) / 64 * (dx.B1 ? 2 : 1), k_piece = (k_all + dx.pieces - 1) / dx.pieces;
        if (k_all - (dx.pieces - 1) * k_piece < 2 || !persist_ok(params_of(dx), false, false, kMaxSuper / dx.pieces)) return hipErrorInvalidValue;
    }
    b.n_gates = n_gates;
    b.p[0] = params_of(dx);
    b.p[1] = params_of(down);
    if (!grouped_gemm_transposed_ok(dx) || !grouped_gemm_transposed_ok(down)) return hipErrorInvalidValue;
    for (int i = 0; i < n_gates; ++i) {
        if (!grouped_gemm_transposed_ok(gates[i]) || !gates[i].ta || gates[i].k_gather != (fetch == Fetch::NONE ? 0 : 2)) return hipErrorInvalidValue;
        b.p[2 + i] = params_of(gates[i]);
    }
    const int n_cu = cu_count();
    const bool tail = (dx.B1 ? dx.K / 2 : dx.K) % 64 != 0;
    switch (fetch) {
        case Fetch::NONE: return tail ? launch_bf16_backward_form<true, Fetch::NONE>(b, st, n_cu) : launch_bf16_backward_form<false, Fetch::NONE>(b, st, n_cu);
        case Fetch::GATES: return tail ? launch_bf16_backward_form<true, Fetch::GATES>(b, st, n_cu) : launch_bf16_backward_form<false, Fetch::GATES>(b, st, n_cu);
        case Fetch::ALL: return tail ? launch_bf16_backward_form<true, Fetch::ALL>(b, st, n_cu) : launch_bf16_backward_form<false, Fetch::ALL>(b, st, n_cu);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_grouped_gemm(const GroupedGemm& q, hipStream_t st) {
    GemmParams g = params_of(q);
    if (q.N % 4 != 0 || q.K < 0 || q.G < 1 || q.M < 1 || q.pieces != 1) return hipErrorInvalidValue;
    if (q.dtype == ETR_F32 && q.tb) {
        if (q.ta || q.epilogue != GEMM_PLAIN || q.N < 8) return hipErrorInvalidValue;
        return launch_f32<false, false, true>(g, st);
    }
    if (q.ta || q.tb) {
        if (!grouped_gemm_transposed_ok(q)) return hipErrorInvalidValue;
        const int n_cu = cu_count();
        if (q.k_gather == 1) return launch_bf16_transposing<true, 1>(g, st, n_cu);
        if (q.k_gather == 2) return launch_bf16_transposing<true, 2>(g, st, n_cu);
        if (q.ta) return hipErrorInvalidValue;           // (such products come in launch_backward_products)
        // a contraction that is not whole k-tiles: the zero-filling instantiation
        const bool tail = (q.B1 ? q.K / 2 : q.K) % 64 != 0;
        if (q.epilogue == GEMM_MIDDLE)
            return tail ? launch_bf16_transposing<false, 0, true, true>(g, st, n_cu) : launch_bf16_transposing<false, 0, false, true>(g, st, n_cu);
        return tail ? launch_bf16_transposing<false, 0, true>(g, st, n_cu) : launch_bf16_transposing<false, 0>(g, st, n_cu);
    }
    if (q.dtype == ETR_BF16) {
        if (q.K % 8 != 0 || (q.lda ? q.lda : q.K) % 8 != 0 || (q.ldb ? q.ldb : q.K) % 8 != 0) return hipErrorInvalidValue;
        const Bf16Kernel kind = choose_bf16(g, q.epilogue != GEMM_PLAIN, q.row_index ? static_cast<size_t>(q.a_rows) : static_cast<size_t>(q.M), q.rows_expected);
        if (kind == Bf16Kernel::ROWS) {
            switch (q.epilogue) {
                case GEMM_PLAIN: return launch_bf16_rows<false>(g, st);
                case GEMM_SWIGLU: return launch_bf16_rows<true>(g, st);
                case GEMM_DUAL: return launch_bf16_rows<true, true>(g, st);
            }
        }
        const bool ring = kind == Bf16Kernel::RING;
        if (kind == Bf16Kernel::PERSISTENT) {
            const int n_cu = cu_count();
            switch (q.epilogue) {
                case GEMM_PLAIN: return launch_bf16_persistent<false>(g, st, n_cu);
                case GEMM_SWIGLU: return launch_bf16_persistent<true>(g, st, n_cu);
                case GEMM_DUAL: return launch_bf16_persistent<true, true>(g, st, n_cu);
            }
        }
        switch (q.epilogue) {
            case GEMM_PLAIN: return ring ? launch_bf16_ring<false, 4>(g, st) : launch_bf16<128, 128, 64, 2, 2, false, 1>(g, st);
            case GEMM_SWIGLU: return ring ? launch_bf16_ring<true, 4>(g, st) : launch_bf16<128, 64, 64, 2, 2, true, 1>(g, st);
            case GEMM_DUAL: return ring ? launch_bf16_ring<true, 4, true>(g, st) : launch_bf16<128, 64, 64, 2, 2, true, 1, true>(g, st);
        }
        return hipErrorInvalidValue;
    }
    if (q.K % 4 != 0 || (q.lda ? q.lda : q.K) % 4 != 0 || (q.ldb ? q.ldb : q.K) % 4 != 0) return hipErrorInvalidValue;
    switch (q.epilogue) {
        case GEMM_PLAIN: return launch_f32<false>(g, st);
        case GEMM_SWIGLU: return launch_f32<true>(g, st);
        case GEMM_DUAL: return launch_f32<true, true>(g, st);
    }
    return hipErrorInvalidValue;
}

// Rows per expert that a batch can be expected to fill (the counts live on the device): every token on k experts, or,
// where the experts choose, their capacity.
int rows_expected(const etr_config& c) {
    const long long even = c.mode == ETR_MODE_ECR ? c.T : (static_cast<long long>(c.T) * c.k + c.E - 1) / c.E;
    return static_cast<int>(even < c.capacity ? even : c.capacity);
}
// Rows of all experts together that the selection can keep.
long long rows_total(const etr_config& c) {
    const long long full = static_cast<long long>(c.E) * std::min(c.T, c.capacity);
    return c.mode == ETR_MODE_ECR ? full : std::min(full, static_cast<long long>(c.T) * c.k);
}

bool ffn_can_gather(const etr_config& c) {
    if (c.dtype != ETR_BF16) return true;
    GemmParams g1{nullptr, nullptr, nullptr, nullptr, nullptr, c.E, c.capacity, c.H, c.d, 0, 0, 0, 0, nullptr, c.T};
    // every kernel reads its rows through an index if asked; only a token matrix past the 32-bit offsets of the
    // pipelined kernels is better rearranged first, where the per-expert buffers are within them.  Asked without a row
    // count, so that the size query that depends on it needs no estimate and with it no device.
    return choose_bf16(g1, true, static_cast<size_t>(c.T), 0) != Bf16Kernel::STAGED ||
           choose_bf16(g1, true, static_cast<size_t>(c.capacity), 0) == Bf16Kernel::STAGED;
}

hipError_t launch_expert_ffn(const etr_config& c, const void* xp, const int32_t* counts, const void* w_gate,
                             const void* w_up, const void* w_down, void* yp, void* hidden, hipStream_t st,
                             hipEvent_t between, const int32_t* gather_rows, void* a_save, void* b_save) {
    // with gather_rows (= slot_token) xp is the token matrix x itself and GEMM-1 fetches row
    // gather_rows[e][s] of it: the rearrangement is folded into the operand load
    GemmParams g1{xp, w_gate, w_up, hidden, counts, c.E, c.capacity, c.H, c.d, 0, 0, 0, 0, gather_rows, c.T};
    GemmParams g2{hidden, w_down, nullptr, yp, counts, c.E, c.capacity, c.d, c.H, 0, 0, 0, 0, nullptr, c.capacity};
    g1.rows_total = g2.rows_total = rows_total(c);
    if (a_save && b_save) { g1.C2 = a_save; g1.C3 = b_save; }      // training mode: GEMM-1 also keeps W_gate x and W_up x
    hipError_t err;
    if (c.dtype == ETR_BF16) {
        if (gather_rows && !ffn_can_gather(c)) return hipErrorInvalidValue;
        const Bf16Kernel kind1 = choose_bf16(g1, true, gather_rows ? static_cast<size_t>(c.T) : static_cast<size_t>(c.capacity), rows_expected(c));
        const Bf16Kernel kind2 = choose_bf16(g2, false, static_cast<size_t>(c.capacity), rows_expected(c));
        const int n_cu = cu_count();
        if (kind1 == Bf16Kernel::ROWS)
            err = g1.C3 ? launch_bf16_rows<true, false, true>(g1, st) : launch_bf16_rows<true>(g1, st);
        else if (kind1 == Bf16Kernel::PERSISTENT)
            err = g1.C3 ? launch_bf16_persistent<true, false, true>(g1, st, n_cu) : launch_bf16_persistent<true>(g1, st, n_cu);
        else err = (kind1 == Bf16Kernel::RING && !g1.C3) ? launch_bf16_ring<true, 4>(g1, st) : launch_bf16<128, 64, 64, 2, 2, true, 1>(g1, st);
        if (err != hipSuccess) return err;
        if (between && (err = hipEventRecord(between, st)) != hipSuccess) return err;
        if (kind2 == Bf16Kernel::ROWS) return launch_bf16_rows<false>(g2, st);
        if (kind2 == Bf16Kernel::STAGED) return launch_bf16<128, 128, 64, 2, 2, false, 1>(g2, st);
        return kind2 == Bf16Kernel::PERSISTENT ? launch_bf16_persistent<false>(g2, st, n_cu) : launch_bf16_ring<false, 4>(g2, st);
    }
    err = launch_f32<true>(g1, st);
    if (err != hipSuccess) return err;
    if (between && (err = hipEventRecord(between, st)) != hipSuccess) return err;
    return launch_f32<false>(g2, st);
}

}  // namespace etr

extern "C" int etr_ffn_plan(const etr_config* c, int product, int gathered, long long* workgroups) {
    using namespace etr;
    const bool glu = product == 0;
    GemmParams p{nullptr, nullptr, nullptr, nullptr, nullptr, c->E, c->capacity, glu ? c->H : c->d, glu ? c->d : c->H};
    p.rows_total = rows_total(*c);
    if (c->dtype != ETR_BF16) {
        const bool large = f32_large_tiles(p);
        *workgroups = plan_live_tiles(p, large ? 64 : 32, large ? 64 : 32);
        return large ? 5 : 6;
    }
    const Bf16Kernel kind = choose_bf16(p, glu, static_cast<size_t>(glu && gathered ? c->T : c->capacity), rows_expected(*c));
    switch (kind) {
        case Bf16Kernel::ROWS: *workgroups = plan_rows(p, glu); return 1;
        case Bf16Kernel::PERSISTENT: *workgroups = cu_count() / 8 * 8; return p.K % 64 == 0 ? 2 : 3;
        case Bf16Kernel::RING: *workgroups = plan_tiles(p, 256, glu ? 128 : 256); return 4;
        case Bf16Kernel::STAGED: *workgroups = plan_tiles(p, 128, glu ? 64 : 128); return 0;
    }
    return -1;
}
