// Bidirectional selection under the capacity bound (Sec. Routing Strategy, Eqs. 5-6; keep
// rules of the pure phases from the Proof of the Theorem, parts 1 and 2) and the
// prefix-sum permutation tables.
//
// Three launches (four for long columns, one for short batches: small_select_kernel), no global atomics, integer counting only, so the result is
// bit-reproducible:
//   1. token_choice_kernel   one lane per (token, expert): k rounds of arg-max inside a lane group (DPP folds)
//                            give the token's Top-k list (Eq. 5); writes the candidate mask and, through an LDS
//                            tile, a column-major copy of the selection keys
//   2. expert_choice_kernel  one 1024-thread workgroup per expert, keys in registers as whole rows of the
//                            column: the key tau_e of the C-th best candidate (Eq. 6) by a radix search over the
//                            bits in which the candidates' order-preserving keys differ at all (11 bits per
//                            pass, one LDS histogram per pass, the digit picked by every wave for itself), then
//                            the (key > tau, key == tau) counts of each chunk are scanned into exclusive prefixes
//                            (long columns: the first digit is counted beforehand by key_histogram_kernel,
//                            up to 16 workgroups per expert)
//   (where experts keep few of the tokens: choice_lists_kernel, expert_lists_kernel, slot_lists_kernel, see by_lists)
//   3. slot_kernel           one lane per (expert, token): the position inside the chunk comes from a
//                            ballot, so slot_of / slot_token are written without any serial walk; the slots of
//                            64 tokens leave as whole rows of slot_of
// All three phases are one algorithm: in TCR every candidate has the same key, so
// "the C best, lowest token first among equals" is "the first C in token order".
#include <mutex>
#include <type_traits>

#include "etr_internal.h"

// Scratch of the allocation-free entry point (etr_select_noalloc): device memory that belongs to the library, one
// copy per GPU the library runs on, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels and copies are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[etr::kStaticSelectBytes];

namespace etr {
namespace {

// fp32 -> uint32 that preserves order; 0 is reserved for "not a candidate".
__device__ __forceinline__ uint32_t order_key(float s) {
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u) u = 0u;                       // -0.0 ties with +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Key under which expert e ranks token t ("the C best keys, lowest token first among equals"):
//   TCR        1 for every chooser (position priority)
//   ECR/BIDIR  the affinity, for all tokens / for the choosers
//   TCR_RANK   k - (position of e in the token's list): first choices before second choices (variant)
//   STRICT     the affinity for ALL tokens; the chooser set is intersected afterwards (variant)
__device__ __forceinline__ uint32_t selection_key(float s, bool cand, int mode, int k = 0, int rank = 0) {
    if (mode == ETR_MODE_BIDIR_STRICT) return order_key(s);
    if (!cand) return 0u;
    if (mode == ETR_MODE_TCR) return 1u;
    if (mode == ETR_MODE_TCR_RANK) return static_cast<uint32_t>(k - rank);
    return order_key(s);
}

// ---------------------------------------------------------------------------------------
// 1. token choice
// ---------------------------------------------------------------------------------------
// Maximum (MAX) or minimum over aligned groups of G lanes, every lane of a group gets it: swaps inside quads, the
// mirror images of the half row and of the row (16 lanes) as data-parallel-primitive moves, then the row-pair and
// half-wave swaps.  Call with all lanes active.
template <bool MAX> __device__ __forceinline__ uint32_t pick(uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); }
template <bool MAX, int CTRL>
__device__ __forceinline__ uint32_t dpp_fold(uint32_t v) {
    return pick<MAX>(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int>(v), static_cast<int>(v), CTRL, 0xF, 0xF, false)));
}
template <int G, bool MAX>
__device__ __forceinline__ uint32_t lane_group_fold(uint32_t v) {
    if constexpr (G >= 2) v = dpp_fold<MAX, 0xB1>(v);        // quad_perm [1,0,3,2]
    if constexpr (G >= 4) v = dpp_fold<MAX, 0x4E>(v);        // quad_perm [2,3,0,1]
    if constexpr (G >= 8) v = dpp_fold<MAX, 0x141>(v);       // row_half_mirror
    if constexpr (G >= 16) v = dpp_fold<MAX, 0x140>(v);      // row_mirror
    if constexpr (G >= 32) {                                 // odd rows of one copy <-> even rows of the other
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = pick<MAX>(r[0], r[1]);
    }
    if constexpr (G >= 64) {                                 // upper half of one copy <-> lower half of the other
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = pick<MAX>(r[0], r[1]);
    }
    return v;
}

template <int G> constexpr int token_tile() { return G <= 4 ? 256 / G : 64; }       // tokens per workgroup
template <int G> constexpr int token_threads() { return G >= 16 ? 1024 : 256; }       // threads per workgroup

// G = lanes per token, a power of two >= E.  A workgroup takes token_tile<G>() tokens in one to four passes, all of
// whose affinities are requested before the first is used.  Each of the k rounds of Eq. 5 is a maximum over the
// token's lanes of the order-preserving affinities still in the contest, then a minimum over the experts that hold
// it (the lower expert wins among equals; from 32 lanes per token on by a ballot: 65536 tokens x 64 experts, k = 4,
// 28 -> 20 us); the winner leaves the contest.  The keys of the tile go through LDS, so
// that each column of the column-major copy is written in whole stretches.
template <int G>
__global__ __launch_bounds__(token_threads<G>()) void token_choice_kernel(const float* __restrict__ score, int T, int E,
                                                                          int k, int mode, int32_t* __restrict__ topk,
                                                                          uint64_t* __restrict__ cmask,
                                                                          uint32_t* __restrict__ keyT, int Tpad) {
    constexpr int TT = token_tile<G>(), NT = token_threads<G>();
    constexpr int PASSES = TT * G / NT;
    static_assert(PASSES >= 1 && PASSES * NT == TT * G, "whole passes");
    __shared__ uint32_t tile[G][TT + 1];
    const int t_base = blockIdx.x * TT;
    const int e = threadIdx.x % G, tl0 = threadIdx.x / G;      // (NT is a multiple of G: the same expert in every pass)
    float vals[PASSES];
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const int t = t_base + pass * (NT / G) + tl0;
        vals[pass] = (t < T && e < E) ? score[static_cast<size_t>(t) * E + e] : 0.f;
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const int tl = pass * (NT / G) + tl0;
        const int t = t_base + tl;
        const bool valid = t < T && e < E;
        const float val = vals[pass];
        uint64_t mask = 0;
        int my_rank = 0, choice = 0;
        if (mode != ETR_MODE_ECR) {
            // 0 = out of the contest (no such expert, or already chosen)
            uint32_t mine = valid ? max(order_key(val), 1u) : 0u;
            for (int r = 0; r < k; ++r) {
                const uint32_t best = lane_group_fold<G, true>(mine);
                int bi;
                if constexpr (G >= 32) {
                    // half a wave or a wave per token: the holders of the maximum as a ballot, the lowest by a scalar
                    // bit scan.  (k <= E, so somebody is still in the contest.)
                    const uint64_t at = __ballot(mine == best);
                    if constexpr (G == 64) bi = __builtin_ctzll(at | (1ull << 63));
                    else bi = (threadIdx.x & 32) ? __builtin_ctz(static_cast<uint32_t>(at >> 32) | (1u << 31))
                                                 : __builtin_ctz(static_cast<uint32_t>(at) | (1u << 31));
                } else {
                    bi = static_cast<int>(lane_group_fold<G, false>(mine == best && best != 0u ? static_cast<uint32_t>(e) : 255u));
                }
                if (e == bi) { mine = 0u; my_rank = r; }
                if (e == r) choice = bi;
            }
            // the token's candidate set: the lanes of its group that have left the contest (one ballot after the
            // rounds, not a shifted bit per round)
            const uint64_t chosen = __ballot(valid && mine == 0u);
            mask = (chosen >> (threadIdx.x & (kWave - 1) & ~(G - 1))) & (G >= 64 ? ~0ull : ((1ull << G) - 1ull));
            if (topk && e < k && t < T) topk[static_cast<size_t>(t) * k + e] = choice;
        } else {
            mask = E >= 64 ? ~0ull : ((1ull << E) - 1ull);
        }
        tile[e][tl] = valid ? selection_key(val, (mask >> e) & 1ull, mode, k, my_rank) : 0u;
        if (e == 0 && t < T) cmask[t] = mask;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * TT; i += NT) {
        const int ee = i / TT, tl = i % TT;
        const int t = t_base + tl;
        if (ee < E && t < T) keyT[static_cast<size_t>(ee) * Tpad + t] = tile[ee][tl];
    }
}

// ---------------------------------------------------------------------------------------
// 2a. first radix digit, spread over the chip (long columns only): workgroup (slice, expert) counts the top
// kRadixBits bits of the candidate keys of its slice of the column; expert_choice_kernel<IPT, true> adds the
// slices up instead of walking all of its keys once more (its per-key work is what bounds it: one CU per expert).
// Integer counts, so the result does not depend on the split.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void key_histogram_kernel(const uint32_t* __restrict__ keyT, int Tpad, int T,
                                                            int slice, uint32_t* __restrict__ hist1) {
    constexpr int NBINS = 1 << 11;
    __shared__ uint32_t h[NBINS];
    const int b = blockIdx.x, e = blockIdx.y, nb = gridDim.x, tid = threadIdx.x;
    for (int i = tid; i < NBINS; i += 256) h[i] = 0u;
    __syncthreads();
    const uint32_t* col = keyT + static_cast<size_t>(e) * Tpad;
    const int t_end = min(T, (b + 1) * slice);
    for (int t = b * slice + tid * 4; t < t_end; t += 1024) {       // slice and Tpad are multiples of 4
        const uint4 v = *reinterpret_cast<const uint4*>(col + t);
        const uint32_t k4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t + j < T && k4[j] != 0u) atomicAdd(&h[k4[j] >> (32 - 11)], 1u);
    }
    __syncthreads();
    uint32_t* out = hist1 + (static_cast<size_t>(e) * nb + b) * NBINS;
    for (int i = tid; i < NBINS; i += 256) out[i] = h[i];
}

// ---------------------------------------------------------------------------------------
// 2. expert choice: threshold search + chunk prefixes
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
    return v;
}

// Sum over aligned groups of Q lanes (Q = 1, 2, 4, 8, 16), every lane of a group gets the group's total:
// swaps inside quads, then the mirror images of the half row and of the row.  Call with all lanes active.
template <int Q>
__device__ __forceinline__ int lane_group_sum(int v) {
    if constexpr (Q >= 2) v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);    // quad_perm [1,0,3,2]
    if constexpr (Q >= 4) v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm [2,3,0,1]
    if constexpr (Q >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    if constexpr (Q >= 16) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
    return v;
}

// Block-wide sums of three counters (all threads get the totals).
__device__ __forceinline__ void block_sum3(int& a, int& b, int& c, int (*red)[3]) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    a = wave_sum_i(a); b = wave_sum_i(b); c = wave_sum_i(c);
    __syncthreads();                                   // previous readers of red are done
    if (lane == 0) { red[wave][0] = a; red[wave][1] = b; red[wave][2] = c; }
    __syncthreads();
    a = b = c = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) { a += red[w][0]; b += red[w][1]; c += red[w][2]; }
}

// Fixed-point term of a positive affinity (key >= key(+0)): round(min(s, 1) * 2^30).  Scaling by a power of two is exact,
// so the rounding in fp32 is that of the exact product.
__device__ __forceinline__ uint32_t affinity_term(uint32_t key) {
    return static_cast<uint32_t>(__builtin_rintf(fminf(__uint_as_float(key & 0x7FFFFFFFu), 1.0f) * 1073741824.0f));
}

constexpr int kRadixBits = 11;           // digit width of the threshold search
constexpr int kBins = 1 << kRadixBits;   // 2048 bins: 32 per lane of a wave
constexpr int kMaxDigits = 3;            // 32 key bits in digits of at most 11
constexpr int kMaxSlices = 16;           // workgroups per expert that count the first digit of a long column

// A wave's view of one histogram of kBins counters in LDS (narrower digits leave the upper bins zero), walked
// from the largest digit down: lane g owns the 32 bins [kBins - 32 (g + 1), kBins - 32 g).  Every wave of the
// workgroup takes the same view by itself, so no barrier is needed between the histogram and its use.
struct DigitView {
    int own;       // candidates in this lane's 32 bins
    int upto;      // candidates in the bins of lanes 0..g (inclusive scan)
    int total;     // candidates in all bins
};

__device__ __forceinline__ DigitView digit_view(const uint32_t* hist) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint4* q4 = reinterpret_cast<const uint4*>(hist) + 8 * (kWave - 1 - lane);
    int s = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {                       // the lane's eight quads, rotated by the lane: no bank conflicts
        const uint4 v = q4[(q + lane) & 7];
        s += static_cast<int>(v.x + v.y + v.z + v.w);
    }
    DigitView d;
    d.own = s;
    d.upto = wave_scan_incl(s);
    d.total = __builtin_amdgcn_readlane(d.upto, kWave - 1);
    return d;
}

// The digit that holds the need-th largest candidate (1 <= need <= total) and the number of candidates with a
// larger digit.
__device__ __forceinline__ void digit_pick(const uint32_t* hist, const DigitView& d, int need, int& digit, int& above) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t m1 = __ballot(d.upto >= need);
    const int g = m1 ? __builtin_ctzll(m1) : kWave - 1;                       // the lane whose bins hold it
    const int before = __builtin_amdgcn_readlane(d.upto - d.own, g);
    const int h = lane < 32 ? static_cast<int>(hist[kBins - 1 - 32 * g - lane]) : 0;   // its bins, largest first
    const int upto = wave_scan_incl(h);
    const uint64_t m2 = __ballot(before + upto >= need);
    const int j = m2 ? __builtin_ctzll(m2) : 31;
    digit = kBins - 1 - 32 * g - j;
    above = before + __builtin_amdgcn_readlane(upto - h, j);
}

// The key at which the sum of the affinities' terms, walked from the highest down, reaches sum_need, digit by digit: an LDS
// histogram of the terms (64-bit sums) over up to 11 bits at a time of the low `shift` ones, walked from the top; the positive keys
// agree with th above those.  True where that happens within n_keep candidates, which then is their number.  By a whole
// workgroup; for_keys(f) calls f on this thread's keys.
template <typename Keys>
__device__ __forceinline__ bool sum_threshold(Keys&& for_keys, long long sum_need, uint32_t th, int shift, unsigned long long* sums, int& n_keep,
                                              uint32_t& theta) {
    __shared__ int red_cnt[kSelThreads / kWave], picked_digit;
    __shared__ long long wave_sums[kSelThreads / kWave], picked_above;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    long long above_sum = 0;                             // sum over the candidates above th, the settled bits of theta
    while (shift > 0) {
        const int w = shift < kRadixBits ? shift : kRadixBits;
        shift -= w;
        const uint32_t span = (1u << (shift + w)) - 1u, dmask = (1u << w) - 1u;
        __syncthreads();                                 // the histogram's previous readers are done
        sums[2 * tid] = 0ull; sums[2 * tid + 1] = 0ull;
        __syncthreads();
        for_keys([&](uint32_t key) {
            if (key - th <= span) atomicAdd(&sums[(key >> shift) & dmask], static_cast<unsigned long long>(affinity_term(key)));
        });
        __syncthreads();
        // the highest bin at which the sum from the top reaches the threshold: two bins to a thread, the highest to thread 0
        const long long need = sum_need - above_sum;     // > 0
        const int low = kBins - 2 - 2 * tid;
        const long long high_bin = static_cast<long long>(sums[low + 1]), both = high_bin + static_cast<long long>(sums[low]);
        const long long upto = wave_scan_incl(both);
        if (lane == kWave - 1) wave_sums[wave] = upto;
        __syncthreads();
        long long before = upto - both, total = 0;
#pragma unroll
        for (int w = 0; w < kSelThreads / kWave; ++w) {
            if (w < wave) before += wave_sums[w];
            total += wave_sums[w];
        }
        if (total < need) return false;                  // (uniform; from the second digit on never) the positive affinities never get there: take all
        if (before < need && need <= before + both) {    // one thread
            const bool high = before + high_bin >= need;
            picked_digit = high ? low + 1 : low;
            picked_above = high ? before : before + high_bin;
        }
        __syncthreads();
        above_sum += picked_above;
        th |= static_cast<uint32_t>(picked_digit) << shift;
    }
    // th is settled: above_sum is the sum over the keys above it; count them
    int n_gt = 0;
    for_keys([&](uint32_t key) { n_gt += key > th; });
    n_gt = wave_sum_i(n_gt);
    if (lane == 0) red_cnt[wave] = n_gt;
    __syncthreads();
    n_gt = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) n_gt += red_cnt[w];
    const long long q_th = affinity_term(th);
    if (q_th == 0) return false;                         // (only where all positive keys are the same)
    const long long ell = n_gt + (sum_need - above_sum + q_th - 1) / q_th;       // q_th > 0: its bin reached the sum
    if (ell > n_keep) return false;
    n_keep = static_cast<int>(ell);
    theta = th;
    return true;
}

// The n_keep-th largest key, by radix search from the top; the bits above the low `shift` ones are those of prefix.  The first
// `counted` digits (0 or 1) have been counted, the first one's view is `first`.  hist: kMaxDigits histograms of zeros.
// wide (or null): room for 4 kBins words, in which four copies of each word are counted, a lane in that of its number.  A column in
// which many candidates lie close together, or are one key, would add to few words all at once, and one wave's adds to a word are
// done one after the other.
template <typename Keys>
__device__ __forceinline__ uint32_t count_threshold(Keys&& for_keys, int n_keep, int shift, uint32_t prefix, uint32_t (*hist)[kBins], int counted,
                                                    const DigitView& first, uint32_t* wide = nullptr) {
    int need = n_keep;
    for (int p = 0; p < kMaxDigits && shift > 0; ++p) {
        const int w = shift < kRadixBits ? shift : kRadixBits;
        const int top = shift;                           // bits [31:top] are settled
        shift -= w;
        int digit, above;
        if (p < counted) {
            digit_pick(hist[0], first, need, digit, above);
        } else {
            // candidates whose settled bits equal the prefix: lo <= key <= lo + span
            const uint32_t lo = prefix > 1u ? prefix : 1u;
            const uint32_t span = (top >= 32 ? 0xFFFFFFFFu : prefix + ((1u << top) - 1u)) - lo;
            const uint32_t dmask = (1u << w) - 1u;
            uint32_t* h = hist[p];
            if (wide) {
                uint4* own = reinterpret_cast<uint4*>(wide) + 2 * threadIdx.x;           // of two words
                own[0] = own[1] = make_uint4(0u, 0u, 0u, 0u);
                __syncthreads();
                for_keys([&](uint32_t key) {
                    if (key - lo <= span) atomicAdd(&wide[4 * ((key >> shift) & dmask) + (threadIdx.x & 3)], 1u);
                });
                __syncthreads();
                const uint4 x = own[0], y = own[1];
                h[2 * threadIdx.x] = x.x + x.y + x.z + x.w;
                h[2 * threadIdx.x + 1] = y.x + y.y + y.z + y.w;
            } else {
                for_keys([&](uint32_t key) {
                    if (key - lo <= span) atomicAdd(&h[(key >> shift) & dmask], 1u);     // LDS; integer adds, so order-free
                });
            }
            __syncthreads();
            const DigitView d = digit_view(h);
            digit_pick(h, d, need, digit, above);
        }
        prefix |= static_cast<uint32_t>(digit) << shift;
        need -= above;
        if (static_cast<int>(hist[p][digit]) == need) break;         // all of the digit's keys are kept: its first value will do
    }
    return prefix;
}

// One 1024-thread workgroup per expert.
// IPT > 0 (4, 8, 16, 32, 64; equal to ipt): the column's keys live in registers.  Wave w holds the 64 chunks
//   [64 w, 64 w + 64) of IPT tokens each, as IPT/4 rows of 64 pieces of four keys: row r, lane l is piece
//   64 r + l of the wave's stretch of the column, so every load instruction reads 1 KiB in one piece.  The search
//   does not care which lane holds which key; only the last step, the per-chunk counts, puts the pieces of a
//   chunk (IPT/4 neighbouring lanes of one row) together.
// IPT == 0: keys streamed from memory, thread t owns chunk t (columns longer than 64 keys per thread).
// PRE: the histogram of the first digit (the top kRadixBits bits) comes from key_histogram_kernel (hist1, n_slices).
// ADAPT: with the adaptive token count (an instantiation of its own: its sums over the keys in registers would otherwise
//   cost the plain search of the long columns registers and 16 KiB of LDS).
template <int IPT, bool PRE = false, bool ADAPT = false>
__global__ __launch_bounds__(kSelThreads) void expert_choice_kernel(const uint32_t* __restrict__ keyT, int Tpad, int T,
                                                                    int ipt, int capacity_host, int mode,
                                                                    const int32_t* __restrict__ capacity_dev,
                                                                    long long sum_need,
                                                                    uint32_t* __restrict__ tau_out,
                                                                    int32_t* __restrict__ need_eq_out,
                                                                    int32_t* __restrict__ pre_gt,
                                                                    int32_t* __restrict__ pre_eq,
                                                                    int32_t* __restrict__ counts,
                                                                    const uint32_t* __restrict__ hist1, int n_slices) {
    constexpr int Q = IPT > 0 ? IPT / 4 : 1;            // rows of a wave = pieces of a chunk
    static_assert(IPT == 0 || (IPT >= 4 && IPT <= 64 && (IPT & (IPT - 1)) == 0), "chunk lengths held in registers");
    __shared__ int red[kSelThreads / kWave][3];
    __shared__ int wave_tot[kSelThreads / kWave][2];
    __shared__ uint32_t range[kSelThreads / kWave][2];
    __shared__ __attribute__((aligned(16))) uint32_t hist[kMaxDigits][kBins];
    __shared__ int chunk_cnt[kSelThreads / kWave][kWave];
    const int e = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    // a capacity computed on the device (e.g. the lower bound of the Remark) may tighten the host one
    const int capacity = capacity_dev ? min(capacity_host, max(1, *capacity_dev)) : capacity_host;
    const uint32_t* col = keyT + static_cast<size_t>(e) * Tpad;

    uint32_t keys[IPT > 0 ? IPT : 1];
    if constexpr (IPT > 0) {
        const int seg = wave * kWave * IPT;             // first token of the wave's stretch
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            const int idx = seg + (r * kWave + lane) * 4;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (idx < Tpad) v = *reinterpret_cast<const uint4*>(col + idx);     // Tpad is a multiple of 4
            keys[4 * r + 0] = idx + 0 < T ? v.x : 0u;
            keys[4 * r + 1] = idx + 1 < T ? v.y : 0u;
            keys[4 * r + 2] = idx + 2 < T ? v.z : 0u;
            keys[4 * r + 3] = idx + 3 < T ? v.w : 0u;
        }
    }
    // The histograms of all digits start at zero; the first barrier below lies between this and their first use.
    if constexpr (PRE) {
        // first digit: the slices' counts of this thread's two bins, added up (integer sums, any order)
        static_assert(kSelThreads * 2 == kBins, "two bins of the first digit per thread");
        const uint32_t* hp = hist1 + static_cast<size_t>(e) * n_slices * kBins + 2 * tid;
        uint32_t s0 = 0u, s1 = 0u;
#pragma unroll
        for (int b = 0; b < kMaxSlices; ++b) {          // all loads in flight at once; slices past the last count as zero
            const uint2 v = *reinterpret_cast<const uint2*>(hp + static_cast<size_t>(b < n_slices ? b : 0) * kBins);
            const uint32_t on = b < n_slices ? 0xFFFFFFFFu : 0u;
            s0 += v.x & on; s1 += v.y & on;
        }
        hist[0][2 * tid] = s0; hist[0][2 * tid + 1] = s1;
    } else {
        hist[0][2 * tid] = 0u; hist[0][2 * tid + 1] = 0u;
    }
#pragma unroll
    for (int p = 1; p < kMaxDigits; ++p) { hist[p][2 * tid] = 0u; hist[p][2 * tid + 1] = 0u; }

    int ncand;
    DigitView first{0, 0, 0};                           // PRE: the view of the first digit
    if constexpr (PRE) {
        __syncthreads();
        first = digit_view(hist[0]);
        ncand = first.total;
    } else {
        int d1 = 0, d2 = 0;
        ncand = 0;
        if constexpr (IPT > 0) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) ncand += keys[j] != 0u;
        } else {
            for (int idx = tid; idx < T; idx += kSelThreads) ncand += col[idx] != 0u;
        }
        block_sum3(ncand, d1, d2, red);
    }
    int n_keep = ncand < capacity ? ncand : capacity;

    // Adaptive token count (Sec. Routing Strategy: "l is determined by a threshold of the sum of
    // affinity scores"): walking the candidates from the highest affinity down, stop at the first
    // prefix whose affinity sum reaches the threshold.  Affinities are summed as fixed-point
    // integers round(clamp(s,-1,1) * 2^30), so the sum of "all candidates with key >= theta" is exact and order-free.
    // The key theta at which that sum reaches the threshold is found digit by digit, as the capacity threshold below
    // is: an LDS histogram of the terms (64-bit sums) over 11, 11 and 9 bits below the sign, walked from the top.  (A
    // bisection over the 31 bits sums all keys up to 33 times: 64 experts x 65536 tokens, 378 us for the kernel; with
    // the histograms 38 us.)  Where the sum binds before the capacity, theta is the threshold the search below would look
    // for: the n_keep candidates end among the keys equal to it.
    bool settled = false;
    uint32_t theta = 0u;
    auto for_keys = [&](auto&& f) {
        if constexpr (IPT > 0) {
#pragma unroll
            for (int j = 0; j < IPT; ++j) f(keys[j]);
        } else {
            for (int idx = tid; idx < T; idx += kSelThreads) f(col[idx]);
        }
    };
    if constexpr (ADAPT) if (sum_need > 0 && (mode == ETR_MODE_ECR || mode == ETR_MODE_BIDIR) && n_keep > 0) {
        __shared__ __attribute__((aligned(16))) unsigned long long sums[kBins];
        settled = sum_threshold([&](auto&& f) {
            for_keys([&](uint32_t key) {
                asm volatile("" : "+v"(key));           // computed anew for each digit: kept terms would spill
                f(key);
            });
        }, sum_need, 0x80000000u, 31, sums, n_keep, theta);
    }

    uint32_t tau;
    if (n_keep == 0) {
        tau = 0xFFFFFFFFu;
    } else if (mode == ETR_MODE_TCR) {
        tau = 1u;                                       // every candidate carries key 1
    } else if (ADAPT && settled) {
        tau = theta;
    } else {
        // The n_keep-th largest key, by radix search from the top.  Only the bits in which the candidates differ
        // have to be resolved (affinities of one expert share sign, exponent and often leading mantissa bits), so
        // the search starts below the common prefix of the largest and the smallest candidate key.
        int shift = 32;                                              // low bits still to resolve
        uint32_t prefix = 0u;
        if constexpr (!PRE) {
            uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
            auto fold = [&](uint32_t key) { if (key != 0u) { kmax = max(kmax, key); kmin = min(kmin, key); } };
            if constexpr (IPT > 0) {
#pragma unroll
                for (int j = 0; j < IPT; ++j) fold(keys[j]);
            } else {
                for (int idx = tid; idx < T; idx += kSelThreads) fold(col[idx]);
            }
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                kmax = max(kmax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmax), m, kWave)));
                kmin = min(kmin, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmin), m, kWave)));
            }
            if (lane == 0) { range[wave][0] = kmax; range[wave][1] = kmin; }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kSelThreads / kWave; ++w) { kmax = max(kmax, range[w][0]); kmin = min(kmin, range[w][1]); }
            const uint32_t diff = kmax ^ kmin;
            shift = diff ? 32 - __builtin_clz(diff) : 0;             // low bits that vary among the candidates
            prefix = shift >= 32 ? 0u : (kmax >> shift) << shift;
        }
        tau = count_threshold(for_keys, n_keep, shift, prefix, hist, PRE ? 1 : 0, first);
    }

    // per-chunk counts of (key > tau, key == tau) in token order, then an exclusive block scan
    int gt = 0, eq = 0;
    if constexpr (IPT > 0) {
        const bool some = tau != 0u;                    // (a key of 0 is no candidate)
        int cnt[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            int g = 0, q = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { g += keys[4 * r + j] > tau; q += (keys[4 * r + j] == tau) && some; }
            cnt[r] = lane_group_sum<Q>(g | (q << 16));  // at most 64 each: the halves do not meet
        }
        if constexpr (Q > 1) {
            // row r, lanes [Q c', Q c' + Q) hold chunk r (64 / Q) + c' of the wave; lane c takes chunk c
            if ((lane & (Q - 1)) == 0) {
#pragma unroll
                for (int r = 0; r < Q; ++r) chunk_cnt[wave][r * (kWave / Q) + lane / Q] = cnt[r];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int mine = chunk_cnt[wave][lane];
            gt = mine & 0xFFFF; eq = mine >> 16;
        } else {
            gt = cnt[0] & 0xFFFF; eq = cnt[0] >> 16;
        }
    } else {
        const int base = tid * ipt;
        for (int j = 0; j < ipt; ++j) {
            const int idx = base + j;
            uint32_t key = idx < T ? col[idx] : 0u;
            gt += key > tau; eq += (key == tau) && key != 0u;
        }
    }
    const int igt = wave_scan_incl(gt), ieq = wave_scan_incl(eq);
    if (lane == kWave - 1) { wave_tot[wave][0] = igt; wave_tot[wave][1] = ieq; }
    __syncthreads();
    int off_gt = 0, off_eq = 0, tot_gt = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) {
        if (w < wave) { off_gt += wave_tot[w][0]; off_eq += wave_tot[w][1]; }
        tot_gt += wave_tot[w][0];
    }
    pre_gt[e * kSelThreads + tid] = off_gt + igt - gt;
    pre_eq[e * kSelThreads + tid] = off_eq + ieq - eq;
    if (tid == 0) {
        tau_out[e] = tau;
        need_eq_out[e] = n_keep - tot_gt;
        counts[e] = n_keep;
    }
}

// ---------------------------------------------------------------------------------------
// 2b. strict intersection (variant): expert_choice_kernel has ranked ALL tokens; a pair survives
// only if the token also lists the expert.  One workgroup per expert, thread = chunk: count the
// survivors of the chunk, scan, and replace counts[e] by the number of survivors.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelThreads) void strict_filter_kernel(const uint32_t* __restrict__ keyT, int Tpad, int T,
                                                                    int ipt, const uint64_t* __restrict__ cmask,
                                                                    const uint32_t* __restrict__ tau_in,
                                                                    const int32_t* __restrict__ need_eq_in,
                                                                    const int32_t* __restrict__ pre_eq,
                                                                    int32_t* __restrict__ pre_kept,
                                                                    int32_t* __restrict__ counts) {
    __shared__ int wave_tot[kSelThreads / kWave];
    const int e = blockIdx.x, tid = threadIdx.x;
    const uint32_t tau = tau_in[e];
    const int need = need_eq_in[e];
    int eq = pre_eq[e * kSelThreads + tid], n = 0;
    const int t_end = min(T, (tid + 1) * ipt);
    for (int t = tid * ipt; t < t_end; ++t) {
        const uint32_t key = keyT[static_cast<size_t>(e) * Tpad + t];
        bool member = key > tau;
        if (key == tau && key != 0u) { member = eq < need; ++eq; }
        n += member && ((cmask[t] >> e) & 1ull);
    }
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    int inc = n;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        int a = __shfl_up(inc, m, kWave);
        if (lane >= m) inc += a;
    }
    if (lane == kWave - 1) wave_tot[wave] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) {
        if (w < wave) off += wave_tot[w];
        tot += wave_tot[w];
    }
    pre_kept[e * kSelThreads + tid] = off + inc - n;
    if (tid == 0) counts[e] = tot;
}

// ---------------------------------------------------------------------------------------
// 3. slots
// ---------------------------------------------------------------------------------------
// A workgroup takes a tile of max(64, ipt) tokens (whole chunks) and all experts, 64 tokens at a time: wave w of W
// does experts w, w + W, ...  Lane = token, so the keys are read in whole stretches of the column-major copy and the
// number of kept tokens in front of a token inside its chunk is a popcount of a ballot (chunks longer than 64
// tokens carry their running counts from one stretch of 64 to the next).  The slots of the 64 x E tile are
// gathered in LDS and leave as whole rows of slot_of.
__global__ __launch_bounds__(kSelThreads) void slot_kernel(const uint64_t* __restrict__ cmask, int T, int E, int capacity,
                                                   int mode, int ipt,
                                                   const uint32_t* __restrict__ tau_in,
                                                   const int32_t* __restrict__ need_eq_in,
                                                   const int32_t* __restrict__ pre_gt,
                                                   const int32_t* __restrict__ pre_eq,
                                                   const int32_t* __restrict__ counts, int32_t* __restrict__ slot_of,
                                                   int32_t* __restrict__ slot_token,
                                                   const uint32_t* __restrict__ keyT, int Tpad,
                                                   const int32_t* __restrict__ pre_kept) {          // STRICT: see strict_filter_kernel
    __shared__ int32_t tile[kWave * (kWave + 1)];       // [token][E + 1]
    __shared__ int carry[kWave][3];                     // per expert: kept-before counts of a long chunk so far
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, nthreads = blockDim.x;
    const bool long_chunk = ipt > kWave;
    const int TT = long_chunk ? ipt : kWave;
    const int t_tile = blockIdx.x * TT;
    const int G = long_chunk ? kWave : ipt;             // lanes per chunk inside a stretch (a power of two)
    const uint64_t group_mask = (G >= 64 ? ~0ull : ((1ull << G) - 1ull)) << (lane & ~(G - 1));
    const uint64_t below = (1ull << lane) - 1ull;
    const int ld = E + 1;
    if (tid < kWave) { carry[tid][0] = 0; carry[tid][1] = 0; carry[tid][2] = 0; }
    __syncthreads();
    for (int j0 = 0; j0 < TT; j0 += kWave) {
        const int t = t_tile + j0 + lane;
        const bool on = t < T && j0 + lane < TT;
        const int c = long_chunk ? static_cast<int>(blockIdx.x) : t / ipt;
        for (int e = wave; e < E; e += nthreads / kWave) {
            const uint32_t tau = tau_in[e];
            const int need = need_eq_in[e];
            const int gt = (on ? pre_gt[e * kSelThreads + c] : 0) + carry[e][0];
            const int eq = (on ? pre_eq[e * kSelThreads + c] : 0) + carry[e][1];
            const uint32_t key = on ? keyT[static_cast<size_t>(e) * Tpad + t] : 0u;
            const bool is_gt = key > tau, is_eq = key == tau && key != 0u;
            const uint64_t w_gt = __ballot(is_gt), w_eq = __ballot(is_eq);
            const int gt_before = gt + __popcll(w_gt & group_mask & below), eq_before = eq + __popcll(w_eq & group_mask & below);
            int slot = -1;
            if (is_gt) slot = gt_before + min(eq_before, need);
            else if (is_eq && eq_before < need) slot = gt_before + eq_before;
            uint64_t w_k = 0ull;
            if (mode == ETR_MODE_BIDIR_STRICT) {        // renumber inside the chooser set
                const int kept = (on ? pre_kept[e * kSelThreads + c] : 0) + carry[e][2];
                const bool keep = slot >= 0 && on && ((cmask[t] >> e) & 1ull);
                w_k = __ballot(keep);
                slot = keep ? kept + __popcll(w_k & group_mask & below) : -1;
            }
            tile[lane * ld + e] = slot;
            if (on && slot >= 0) slot_token[static_cast<size_t>(e) * capacity + slot] = t;
            if (long_chunk && lane == 0) {              // (the whole wave is one chunk here)
                carry[e][0] += __popcll(w_gt); carry[e][1] += __popcll(w_eq); carry[e][2] += __popcll(w_k);
            }
        }
        __syncthreads();
        int rows = T - (t_tile + j0);
        rows = rows < TT - j0 ? rows : TT - j0;
        rows = rows < kWave ? rows : kWave;
        int32_t* out = slot_of + static_cast<size_t>(t_tile + j0) * E;
        for (int i = tid; i < rows * E; i += nthreads) out[i] = tile[(i / E) * ld + i % E];
        __syncthreads();
    }
    // empty slots
    const long long gid = static_cast<long long>(blockIdx.x) * nthreads + tid;
    const long long total = static_cast<long long>(gridDim.x) * nthreads;
    for (long long i = gid; i < static_cast<long long>(E) * capacity; i += total) {
        const int ee = static_cast<int>(i / capacity), sl = static_cast<int>(i - static_cast<long long>(ee) * capacity);
        if (sl >= counts[ee]) slot_token[i] = -1;
    }
}

// ---------------------------------------------------------------------------------------
// Selection by lists, where experts keep few of the tokens (see by_lists): three launches that pass on the chosen pairs only, where
// the ones above write, read and read again a key for every (token, expert).
//   1. choice_lists_kernel   a workgroup per tile of 64 tokens, a lane per token: the k best experts by insertion while the row is
//                            walked; then the tile's pairs, sorted by expert and token, and where each expert's begin
//   2. expert_lists_kernel   a workgroup per expert: its pairs of all tiles brought together in LDS or, where they are many, in
//                            registers, the threshold search on them, and the (key > tau, key == tau) counts in front of each tile
//   3. slot_lists_kernel     a workgroup per tile, a thread per pair: its place among the tile's pairs of the expert from
//                            ballots; the slots leave as whole rows of slot_of
// Bound by launches and latency and by the tables themselves; with a crowded column by its search on one CU.  65536 tokens x 64
// experts, k = 4, even: the choice 20 -> 9.3 us, the threshold with the affinity sum 6 + 31 -> 16, the slots 15 -> 7.6.
// ---------------------------------------------------------------------------------------
constexpr int kListK = 4;                                // experts of a token, at most
constexpr int kTileTokens = 64;
struct ChoiceLists {
    uint32_t* keys;      // [tiles][64 k]   selection keys of the tile's pairs by (expert, token)
    uint16_t* pairs;     // [tiles][64 k]   token of the tile | expert << 6
    uint16_t* begin;     // [tiles][E + 1]  where each expert's pairs begin
    int tiles;
};
// They lie where the column-major keys would: 6 k + (E + 1) / 32 bytes a token, and k <= E / 4.
inline ChoiceLists carve_lists(const SelectWs& w, int T, int E, int k) {
    ChoiceLists l;
    l.tiles = (T + kTileTokens - 1) / kTileTokens;
    l.keys = w.keyT;
    l.pairs = reinterpret_cast<uint16_t*>(l.keys + static_cast<size_t>(l.tiles) * kTileTokens * k);
    l.begin = l.pairs + static_cast<size_t>(l.tiles) * kTileTokens * k;
    return l;
}

__global__ __launch_bounds__(256) void choice_lists_kernel(const float* __restrict__ score, int T, int E, int k, int mode,
                                                           int32_t* __restrict__ topk, ChoiceLists lists) {
    __shared__ float tile[kTileTokens * (kWave + 1)];
    __shared__ uint32_t part_key[4][kListK][kTileTokens];
    __shared__ int part_e[4][kListK][kTileTokens];
    __shared__ uint32_t chosen[kWave][2];                // tokens that chose the expert
    __shared__ int begin[kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int t0 = blockIdx.x * kTileTokens, rows = min(kTileTokens, T - t0), ld = E | 1;       // (odd: no bank conflicts)
    const float* in = score + static_cast<size_t>(t0) * E;
    const int width = (E & 3) == 0 ? 4 : 1, step = 256 * width, dr = step / E, dc = step - dr * E;
    int r = tid * width / E, c = tid * width - r * E;
    for (int i = tid * width; i < rows * E; i += step) {
        float* at = tile + r * ld + c;
        if (width == 4) {
            const float4 v = *reinterpret_cast<const float4*>(in + i);
            at[0] = v.x; at[1] = v.y; at[2] = v.z; at[3] = v.w;
        } else {
            at[0] = in[i];
        }
        r += dr; c += dc;
        if (c >= E) { c -= E; ++r; }
    }
    if (tid < kWave) chosen[tid][0] = chosen[tid][1] = 0u;
    __syncthreads();
    // the best of this wave's quarter of the experts, largest key first, the lower expert first among equals: they come in
    // ascending order and move up only past smaller keys
    uint32_t best[kListK] = {0u, 0u, 0u, 0u};
    int who[kListK] = {0, 0, 0, 0};
    auto insert = [&](uint32_t key, int e) {
        bool up[kListK];
#pragma unroll
        for (int i = 0; i < kListK; ++i) up[i] = key > best[i];
#pragma unroll
        for (int i = kListK - 1; i > 0; --i) {
            best[i] = up[i - 1] ? best[i - 1] : (up[i] ? key : best[i]);
            who[i] = up[i - 1] ? who[i - 1] : (up[i] ? e : who[i]);
        }
        best[0] = up[0] ? key : best[0];
        who[0] = up[0] ? e : who[0];
    };
    const int quarter = (E + 3) / 4, e_end = min(E, (wave + 1) * quarter);
    const int mine = min(lane, rows - 1) * ld;
#pragma unroll 4
    for (int e = wave * quarter; e < e_end; ++e) insert(max(order_key(tile[mine + e]), 1u), e);
#pragma unroll
    for (int i = 0; i < kListK; ++i) { part_key[wave][i][lane] = best[i]; part_e[wave][i][lane] = who[i]; }
    __syncthreads();
    if (wave != 0) return;                               // (no barrier below)
#pragma unroll
    for (int w = 1; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < kListK; ++i) insert(part_key[w][i][lane], part_e[w][i][lane]);
    const bool live = lane < rows;
    uint32_t pair_key[kListK];                           // (a key of 0 is no candidate: not listed)
#pragma unroll
    for (int i = 0; i < kListK; ++i) pair_key[i] = i < k && live ? selection_key(tile[mine + who[i]], true, mode, k, i) : 0u;
#pragma unroll
    for (int i = 0; i < kListK; ++i)
        if (pair_key[i] != 0u) atomicOr(&chosen[who[i]][lane >> 5], 1u << (lane & 31));
    auto in_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    in_order();
    const int n = __popc(chosen[lane][0]) + __popc(chosen[lane][1]);    // (experts past E: none)
    const int upto = wave_scan_incl(n);
    begin[lane] = upto - n;
    uint16_t* out = lists.begin + static_cast<size_t>(blockIdx.x) * (E + 1);
    if (lane < E) out[lane] = static_cast<uint16_t>(upto - n);
    if (lane == E - 1) out[E] = static_cast<uint16_t>(upto);
    in_order();
    const size_t first = static_cast<size_t>(blockIdx.x) * kTileTokens * k;
#pragma unroll
    for (int i = 0; i < kListK; ++i) {
        const int e = who[i];
        if (i < k && live && topk) topk[static_cast<size_t>(t0 + lane) * k + i] = e;
        if (pair_key[i] != 0u) {
            const uint64_t all = chosen[e][0] | (static_cast<uint64_t>(chosen[e][1]) << 32);
            const size_t at = first + begin[e] + __popcll(all & ((1ull << lane) - 1ull));
            lists.keys[at] = pair_key[i];
            lists.pairs[at] = static_cast<uint16_t>(lane | (e << 6));
        }
    }
}

// A column of up to list_keys lies in LDS.  Where an expert is chosen by more tokens than that, as happens before training has
// spread the load, and where there are few tiles, its keys stay in registers: R per thread, a wave to a tile (a tile holds up to 64
// pairs of an expert, which 16 lanes would load one load behind the other).  The digits of a long such column are counted in four
// copies (see count_threshold).  Selection: 65536 tokens, k = 2, all on the first of 16 experts, the column read again for each
// digit 74 us, in registers 33; half of a column the same key, 64 experts, k = 4: 150, in registers 117, with four copies 65.  The
// room: 24 keys for each tile that R stands for, 12: routing read-outs of 51822 tokens, 24 experts, k = 2, skewed 94 / 105 us, of 40829,
// 384 wide, k = 4 87 / 93; 8, selection of 16384 tokens, loads of 1 to 6, 16 experts: 14.5 / 16.7.
// The room is static: a dynamic one of this size would need an attribute of the kernel first, and a selection may be captured
// without a first call at its shape.
template <int R> constexpr int list_keys() { return R <= 8 ? 0 : 24 * R * (kSelThreads / kWave); }
template <bool ADAPT, int R>
__global__ __launch_bounds__(kSelThreads) void expert_lists_kernel(ChoiceLists lists, int E, int k, int capacity_host, int mode,
                                                                   const int32_t* __restrict__ capacity_dev, long long sum_need,
                                                                   uint32_t* __restrict__ tau_out, int32_t* __restrict__ need_eq_out,
                                                                   int32_t* __restrict__ pre_gt, int32_t* __restrict__ pre_eq,
                                                                   int32_t* __restrict__ counts) {
    constexpr int kWaves = kSelThreads / kWave, kKeys = list_keys<R>();
    __shared__ __attribute__((aligned(16))) uint32_t keys[kKeys == 0 ? 4 : (kKeys > 4 * kBins ? kKeys : 4 * kBins)];       // or the four copies
    __shared__ __attribute__((aligned(16))) uint32_t hist[kMaxDigits][kBins];
    __shared__ __attribute__((aligned(16))) unsigned long long sums[ADAPT ? kBins : 2];
    __shared__ int place[kSelThreads], from[kSelThreads], many[kSelThreads];             // of each tile's pairs
    __shared__ int wave_tot[kSelThreads / kWave][2];
    __shared__ uint32_t range[kWaves][2];
    __shared__ int by_rank[kWaves][kListK];
    const int e = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int capacity = capacity_dev ? min(capacity_host, max(1, *capacity_dev)) : capacity_host;
    int own = 0, src = 0;
    if (tid < lists.tiles) {
        const uint16_t* b = lists.begin + static_cast<size_t>(tid) * (E + 1) + e;
        own = b[1] - b[0];
        src = tid * kTileTokens * k + b[0];
    }
#pragma unroll
    for (int p = 0; p < kMaxDigits; ++p) { hist[p][2 * tid] = 0u; hist[p][2 * tid + 1] = 0u; }
    const int upto = wave_scan_incl(own);
    if (lane == kWave - 1) wave_tot[wave][0] = upto;
    __syncthreads();
    int n = 0, first = upto - own;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) {
        if (w < wave) first += wave_tot[w][0];
        n += wave_tot[w][0];
    }
    int n_keep = min(n, capacity), gt = 0, eq = 0;       // gt, eq: this tile's pairs with key > tau, key == tau
    uint32_t tau;
    const bool by_sum = ADAPT && sum_need > 0 && mode == ETR_MODE_BIDIR && n_keep > 0;
    if (mode == ETR_MODE_TCR) {                          // every candidate carries key 1
        tau = n_keep > 0 ? 1u : 0xFFFFFFFFu;
        eq = own;
    } else if (!by_sum && n <= capacity) {               // nobody is turned away: all are above 0
        tau = 0u;
        gt = own;
    } else {
        place[tid] = first; from[tid] = src; many[tid] = own;
        __syncthreads();
        const bool crowded = n > kKeys;
        const int uwave = __builtin_amdgcn_readfirstlane(wave);
        uint32_t held[R];                                // crowded: tile uwave + 16 r, pair `lane` of it (0: none)
        uint32_t kmax = 0u, kmin = 0xFFFFFFFFu;
        if (crowded) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int c = uwave + r * kWaves;        // (< kSelThreads; tiles past the last have no pairs)
                held[r] = lane < many[c] ? lists.keys[from[c] + lane] : 0u;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                kmax = max(kmax, held[r]);
                kmin = min(kmin, held[r] - 1u);          // (0 wraps past all)
            }
            kmin += kmin != 0xFFFFFFFFu;
        } else {
            // every pair of the column, 16 lanes to a tile (a tile has k / E of its 64 tokens on average), kAtOnce tiles at a time
            constexpr int kAtOnce = 8, kApart = kSelThreads / 16;
            const int sub = tid & 15;
            for (int c0 = tid >> 4; c0 < lists.tiles; c0 += kAtOnce * kApart) {
                int m[kAtOnce], at[kAtOnce], g[kAtOnce];
                uint32_t v[kAtOnce], v2[kAtOnce];
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    const int c = min(c0 + i * kApart, kSelThreads - 1);         // (tiles past the last have no pairs)
                    m[i] = many[c]; at[i] = place[c]; g[i] = from[c];
                }
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    v[i] = sub < m[i] ? lists.keys[g[i] + sub] : 0u;
                    v2[i] = sub + 16 < m[i] ? lists.keys[g[i] + sub + 16] : 0u;
                }
                auto take = [&](int to, uint32_t key) {
                    keys[to] = key;
                    kmax = max(kmax, key); kmin = min(kmin, key);
                };
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    if (sub < m[i]) take(at[i] + sub, v[i]);
                    if (sub + 16 < m[i]) take(at[i] + sub + 16, v2[i]);
                    for (int j = sub + 32; j < m[i]; j += 16) take(at[i] + j, lists.keys[g[i] + j]);
                }
            }
        }
        kmax = lane_group_fold<kWave, true>(kmax);
        kmin = lane_group_fold<kWave, false>(kmin);
        if (lane == 0) { range[wave][0] = kmax; range[wave][1] = kmin; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { kmax = max(kmax, range[w][0]); kmin = min(kmin, range[w][1]); }
        // Only the low bits in which the keys differ have to be resolved.  (The affinities of one expert crowd into few values
        // of the bits above, and adds to one word of LDS wait for each other.)
        auto varying = [](uint32_t diff) { return diff ? 32 - __builtin_clz(diff) : 0; };
        auto settled = [](uint32_t key, int shift) { return shift >= 32 ? 0u : (key >> shift) << shift; };
        auto search = [&](auto&& for_keys) {
            if constexpr (ADAPT) {
                if (by_sum && kmax >= 0x80000000u) {
                    const int shift = varying(kmax ^ max(kmin, 0x80000000u));
                    if (sum_threshold(for_keys, sum_need, settled(kmax, shift), shift, sums, n_keep, tau)) return;
                }
            }
            const int shift = varying(kmax ^ kmin);
            if (n_keep == n) {
                tau = 0u;
            } else if (mode == ETR_MODE_TCR_RANK && shift > 0) {      // keys 1 to kListK: a count of each, no histogram of so few words
                uint32_t mine = 0u;                      // (a thread has at most 64 keys)
                for_keys([&](uint32_t key) { mine += key ? 1u << (8 * (key - 1)) : 0u; });
                const int odd = wave_scan_incl(static_cast<int>(mine & 0x00FF00FFu)), even = wave_scan_incl(static_cast<int>((mine >> 8) & 0x00FF00FFu));
                if (lane == kWave - 1) {
                    by_rank[wave][0] = odd & 0xFFFF; by_rank[wave][1] = even & 0xFFFF;
                    by_rank[wave][2] = odd >> 16; by_rank[wave][3] = even >> 16;
                }
                __syncthreads();
                int above = 0;
                for (int v = kListK; v >= 1; --v) {
#pragma unroll
                    for (int w = 0; w < kWaves; ++w) above += by_rank[w][v - 1];
                    if (above >= n_keep) { tau = static_cast<uint32_t>(v); break; }
                }
            } else {
                tau = count_threshold(for_keys, n_keep, shift, settled(kmax, shift), hist, 0, DigitView{0, 0, 0},
                                      kKeys > 0 && crowded ? keys : nullptr);
            }
        };
        if (crowded) {
            search([&](auto&& f) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint32_t key = held[r];
                    asm volatile("" : "+v"(key));       // what is computed from it is not kept from one digit to the next: it would spill
                    f(key);
                }
            });
            // a tile's counts from ballots, left in place of its number of pairs
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int c = uwave + r * kWaves;
                const uint64_t w_gt = __ballot(held[r] > tau), w_eq = __ballot(held[r] == tau && held[r] != 0u);
                if (lane == 0) many[c] = __popcll(w_gt) | (__popcll(w_eq) << 16);
            }
            __syncthreads();
            if (tid < lists.tiles) { gt = many[tid] & 0xFFFF; eq = many[tid] >> 16; }
        } else {
            search([&](auto&& f) { for (int i = tid; i < n; i += kSelThreads) f(keys[i]); });
            for (int j0 = 0; j0 < own; j0 += 4) {
                uint32_t v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = keys[first + min(j0 + i, own - 1)];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    gt += j0 + i < own && v[i] > tau;
                    eq += j0 + i < own && v[i] == tau;
                }
            }
        }
    }
    const int igt = wave_scan_incl(gt), ieq = wave_scan_incl(eq);
    __syncthreads();                                     // (wave_tot has been read)
    if (lane == kWave - 1) { wave_tot[wave][0] = igt; wave_tot[wave][1] = ieq; }
    __syncthreads();
    int off_gt = 0, off_eq = 0, tot_gt = 0;
#pragma unroll
    for (int w = 0; w < kSelThreads / kWave; ++w) {
        if (w < wave) { off_gt += wave_tot[w][0]; off_eq += wave_tot[w][1]; }
        tot_gt += wave_tot[w][0];
    }
    if (tid < lists.tiles) {
        pre_gt[e * kSelThreads + tid] = off_gt + igt - gt;
        pre_eq[e * kSelThreads + tid] = off_eq + ieq - eq;
    }
    if (tid == 0) {
        tau_out[e] = tau;
        need_eq_out[e] = n_keep - tot_gt;
        counts[e] = n_keep;
    }
}

__global__ __launch_bounds__(kTileTokens * kListK) void slot_lists_kernel(ChoiceLists lists, int T, int E, int k, int capacity,
                                                                          const uint32_t* __restrict__ tau_in,
                                                                          const int32_t* __restrict__ need_eq_in,
                                                                          const int32_t* __restrict__ pre_gt,
                                                                          const int32_t* __restrict__ pre_eq,
                                                                          const int32_t* __restrict__ counts,
                                                                          int32_t* __restrict__ slot_of,
                                                                          int32_t* __restrict__ slot_token) {
    constexpr int NT = kTileTokens * kListK;
    __shared__ __attribute__((aligned(16))) int32_t tile[kTileTokens * kWave];           // [token][E]
    __shared__ uint64_t above[kListK], equal[kListK];    // of the tile's pairs, 64 to a word
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int t0 = blockIdx.x * kTileTokens, rows = min(kTileTokens, T - t0);
    const uint16_t* begins = lists.begin + static_cast<size_t>(blockIdx.x) * (E + 1);
    const bool on = tid < begins[E];
    uint32_t key = 0u;
    int e = 0, token = 0;
    if (on) {
        const size_t at = static_cast<size_t>(blockIdx.x) * kTileTokens * k + tid;
        const int pair = lists.pairs[at];
        key = lists.keys[at];
        e = pair >> 6;
        token = pair & (kTileTokens - 1);
    }
    const uint32_t tau = tau_in[e];
    const int need = need_eq_in[e], gt = pre_gt[e * kSelThreads + blockIdx.x], eq = pre_eq[e * kSelThreads + blockIdx.x];
    const int begin = begins[e];
    const int4 none = make_int4(-1, -1, -1, -1);
    for (int i = 4 * tid; i < rows * E; i += 4 * NT) *reinterpret_cast<int4*>(tile + i) = none;          // (the tile ends at a multiple of 4)
    const bool is_gt = on && key > tau, is_eq = on && key == tau && key != 0u;
    const uint64_t w_gt = __ballot(is_gt), w_eq = __ballot(is_eq);
    if (lane == 0) { above[wave] = w_gt; equal[wave] = w_eq; }
    __syncthreads();
    // set bits of places [begin, tid): an expert has at most 64 pairs here, so they lie in two words
    auto before = [&](const uint64_t* words) {
        const int w0 = begin >> 6;
        const uint64_t upto = (1ull << lane) - 1ull, from = ~0ull << (begin & 63);
        return w0 == wave ? __popcll(words[wave] & upto & from) : __popcll(words[wave] & upto) + __popcll(words[w0] & from);
    };
    if (on) {
        const int gt_before = gt + before(above), eq_before = eq + before(equal);
        int slot = -1;
        if (is_gt) slot = gt_before + min(eq_before, need);
        else if (is_eq && eq_before < need) slot = gt_before + eq_before;
        tile[token * E + e] = slot;
        if (slot >= 0) slot_token[static_cast<size_t>(e) * capacity + slot] = t0 + token;
    }
    __syncthreads();
    int32_t* out = slot_of + static_cast<size_t>(t0) * E;
    const int whole = rows * E & ~3;
    for (int i = 4 * tid; i < whole; i += 4 * NT) *reinterpret_cast<int4*>(out + i) = *reinterpret_cast<const int4*>(tile + i);
    if (tid < rows * E - whole) out[whole + tid] = tile[whole + tid];
    // empty slots
    const unsigned total = static_cast<unsigned>(E) * capacity, stride = gridDim.x * NT;
    for (unsigned i = blockIdx.x * NT + tid; i < total; i += stride) {
        const unsigned ee = i / static_cast<unsigned>(capacity);
        if (static_cast<int>(i - ee * capacity) >= counts[ee]) slot_token[i] = -1;
    }
}

// ---------------------------------------------------------------------------------------
// Everything in one launch for short batches (T <= kSmallTokens, no strict intersection):
// one workgroup per expert, one thread per token.  What a small call pays for is launches and dependent latencies, so
// each workgroup reads all scores (they are in the caches) and finds its expert's place in every token's list by
// counting the better experts of the row; the candidates of its column are brought together in LDS, and one is kept if
// fewer than `capacity` precede it (a larger key, or the same key and a lower token), again by counting: a quarter of them
// in broadcast reads per thread instead of a radix search, and none where all fit (as in decode steps).  The slot is the number
// of kept tokens in front, from ballots.  Counting grows with the square of the candidates.  One call against the three
// launches, T x E: 32 x 16 3.4 / 12.3 us, 256 x 32 5.2 / 14.5, 512 x 8 3.5 / 12.3, 512 x 64 11 / 20.7 (with every token of the
// column in the count, candidate or not: 5.6, 9.2, 10.3 and 15.7); where experts choose, 512 x 8: 9.5; from 1024 tokens on
// that would be the slower one.
// ---------------------------------------------------------------------------------------
// ADAPT: with the affinity-sum threshold (ECR and BIDIR).  The walk from the highest affinity down stops at the first
// prefix whose sum of positive affinities reaches it, so a candidate is kept if the terms of those that precede it do
// not: one more sum in the same pass (82 tokens x 8 experts: 57 us in three launches by bisection, 24 with the
// digit histograms, 9 here).
constexpr int kSmallTokens = 512;
template <bool ADAPT>
__global__ __launch_bounds__(kSmallTokens) void small_select_kernel(const float* __restrict__ score, int T, int E, int k,
                                                                    int capacity_host, int mode,
                                                                    const int32_t* __restrict__ capacity_dev, long long sum_need,
                                                                    int32_t* __restrict__ topk, int32_t* __restrict__ slot_of,
                                                                    int32_t* __restrict__ slot_token, int32_t* __restrict__ counts) {
    __shared__ __attribute__((aligned(16))) uint32_t keys[kSmallTokens];
    __shared__ __attribute__((aligned(16))) uint32_t terms[ADAPT ? kSmallTokens : 4];
    __shared__ int tokens[kSmallTokens], wave_count[kSmallTokens / kWave], wave_kept[kSmallTokens / kWave];
    const int e = blockIdx.x, t = threadIdx.x, nthreads = blockDim.x;       // nthreads: T rounded up to whole waves
    const int lane = t & (kWave - 1), wave = t / kWave;
    const int capacity = capacity_dev ? min(capacity_host, max(1, *capacity_dev)) : capacity_host;
    uint32_t key = 0u;
    if (t < T) {
        const float* row = score + static_cast<size_t>(t) * E;
        const float own_score = row[e];
        int rank = 0;
        if (mode != ETR_MODE_ECR) {
            const uint32_t own = max(order_key(own_score), 1u);
            if ((E & 3) == 0) {
#pragma unroll 4
                for (int q = 0; q < E; q += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(row + q);
                    const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t other = max(order_key(f[j]), 1u);
                        rank += other > own || (other == own && q + j < e);
                    }
                }
            } else {
#pragma unroll 4
                for (int q = 0; q < E; ++q) {
                    const uint32_t other = max(order_key(row[q]), 1u);
                    rank += other > own || (other == own && q < e);
                }
            }
            if (topk && rank < k) topk[static_cast<size_t>(t) * k + rank] = e;
        }
        key = selection_key(own_score, mode == ETR_MODE_ECR || rank < k, mode, k, rank);
    }
    int32_t* mine = slot_token + static_cast<size_t>(e) * capacity_host;
    int n = T, token = t;                                // candidates (a key of 0 is none); whose this thread's is
    // Where nearly every token is a candidate and some are turned away there is little to bring together.  Counted all / brought
    // together, 0.9 of the even share: 512 x 8, k = 5 10.7 / 9.5 us, k = 7 10.6 / 10.9; 512 x 64, k = 40 16.4 / 15.3, k = 60 16.4 / 16.9.
    // With a quarter more than the even share there may be none to count: k = 5 10.8 / 4.0.
    if (mode == ETR_MODE_TCR || capacity >= T || (mode != ETR_MODE_ECR && (4 * k <= 3 * E || 4ll * E * capacity >= 5ll * T * k))) {
        // place among the column's candidates, in token order
        const uint64_t in_column = __ballot(key != 0u);
        if (lane == 0) wave_count[wave] = __popcll(in_column);
        __syncthreads();
        int place = __popcll(in_column & ((1ull << lane) - 1ull));
        n = 0;
        for (int w = 0; w < nthreads / kWave; ++w) {
            if (w < wave) place += wave_count[w];
            n += wave_count[w];
        }
        if (mode == ETR_MODE_TCR || (!ADAPT && n <= capacity)) {   // uniform: the first ones, or all, in their own order
            const bool kept = key != 0u && place < capacity;
            const int total = min(n, capacity);
            if (t < T) slot_of[static_cast<size_t>(t) * E + e] = kept ? place : -1;
            if (kept) mine[place] = t;
            for (int i = total + t; i < capacity_host; i += nthreads) mine[i] = -1;
            if (t == 0) counts[e] = total;
            return;
        }
        // side by side; from here on a thread has the candidate of its own number
        if (t < T && key == 0u) slot_of[static_cast<size_t>(t) * E + e] = -1;
        if (key != 0u) {
            keys[place] = key;
            tokens[place] = t;
            if constexpr (ADAPT) terms[place] = key >= 0x80000000u ? affinity_term(key) : 0u;
        }
        if (t >= n) keys[t] = 0u;
        __syncthreads();
        key = keys[t];
        token = tokens[t];
    } else {
        keys[t] = key;
        if constexpr (ADAPT) terms[t] = key >= 0x80000000u ? affinity_term(key) : 0u;
        __syncthreads();
    }
    // candidates that precede this one: of the waves before, >=; of the waves behind, >; inside the wave by lane
    int before = 0;
    unsigned long long before_sum = 0ull;
    const uint4* k4 = reinterpret_cast<const uint4*>(keys);
    const uint4* t4 = reinterpret_cast<const uint4*>(terms);
    const int uwave = __builtin_amdgcn_readfirstlane(wave), waves = (n + kWave - 1) / kWave;
    for (int w = 0; w < waves && uwave < waves; ++w) {
        if (w == uwave) continue;
        uint4 v[kWave / 4];                             // a wave's 64 keys requested together
#pragma unroll
        for (int i = 0; i < kWave / 4; ++i) v[i] = k4[w * (kWave / 4) + i];
        const uint32_t edge = w < uwave ? key - 1u : key;              // >= key as > key - 1 (candidates: key >= 1)
#pragma unroll
        for (int i = 0; i < kWave / 4; ++i) {
            before += (v[i].x > edge) + (v[i].y > edge) + (v[i].z > edge) + (v[i].w > edge);
            if constexpr (ADAPT) {
                const uint4 q = t4[w * (kWave / 4) + i];
                before_sum += (v[i].x > edge ? q.x : 0u);
                before_sum += (v[i].y > edge ? q.y : 0u);
                before_sum += (v[i].z > edge ? q.z : 0u);
                before_sum += (v[i].w > edge ? q.w : 0u);
            }
        }
    }
    if (uwave < waves) {
#pragma unroll 4
        for (int i = 0; i < kWave / 4; ++i) {
            const uint4 v = k4[uwave * (kWave / 4) + i];
            const uint32_t f[4] = {v.x, v.y, v.z, v.w};
            uint32_t term[4];
            if constexpr (ADAPT) {
                const uint4 q = t4[uwave * (kWave / 4) + i];
                term[0] = q.x; term[1] = q.y; term[2] = q.z; term[3] = q.w;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool first = f[j] > key || (f[j] == key && 4 * i + j < lane);
                before += first;
                if constexpr (ADAPT) before_sum += first ? term[j] : 0u;
            }
        }
    }
    bool kept = key != 0u && before < capacity;
    if constexpr (ADAPT) kept = kept && before_sum < static_cast<unsigned long long>(sum_need);
    const uint64_t in_wave = __ballot(kept);
    if (lane == 0) wave_kept[wave] = __popcll(in_wave);
    __syncthreads();
    int slot = __popcll(in_wave & ((1ull << lane) - 1ull)), total = 0;
    for (int w = 0; w < nthreads / kWave; ++w) {
        if (w < wave) slot += wave_kept[w];
        total += wave_kept[w];
    }
    if (t < n) {
        slot_of[static_cast<size_t>(token) * E + e] = kept ? slot : -1;
        if (kept) mine[slot] = token;
    }
    for (int i = total + t; i < capacity_host; i += nthreads) mine[i] = -1;
    if (t == 0) counts[e] = total;
}

}  // namespace

// Tokens per chunk (= per thread of the per-expert kernel): a power of two from 4 to 64 while the column fits
// that kernel's registers, else a multiple of 4.
static int chunk_tokens(int T) {
    const int ipt = (T + kSelThreads - 1) / kSelThreads;
    for (int p = 4; p <= 64; p <<= 1)
        if (ipt <= p) return p;
    return (ipt + 3) / 4 * 4;
}

// Long columns (more than 32 keys per thread of the per-expert kernel) get their first radix digit counted by
// up to 16 workgroups per expert.
static int select_slices(int T) {
    if (chunk_tokens(T) <= 32) return 0;
    const int n = (T + 4095) / 4096;
    return n > kMaxSlices ? kMaxSlices : n;
}

size_t select_ws_bytes(int T, int E) {
    const size_t Tpad = align_up(static_cast<size_t>(T), 64);
    return align_up(sizeof(uint64_t) * T) + align_up(sizeof(uint32_t) * E * Tpad) + 2 * align_up(sizeof(int32_t) * E) +
           3 * align_up(sizeof(int32_t) * E * kSelThreads) +
           align_up(sizeof(uint32_t) * E * select_slices(T) * 2048);
}

SelectWs select_ws_carve(void* ws, int T, int E) {
    SelectWs w;
    char* p = static_cast<char*>(ws);
    w.Tpad = static_cast<int>(align_up(static_cast<size_t>(T), 64));
    w.cmask = reinterpret_cast<uint64_t*>(p);  p += align_up(sizeof(uint64_t) * T);
    w.keyT = reinterpret_cast<uint32_t*>(p);   p += align_up(sizeof(uint32_t) * E * w.Tpad);
    w.tau = reinterpret_cast<uint32_t*>(p);    p += align_up(sizeof(int32_t) * E);
    w.need_eq = reinterpret_cast<int32_t*>(p); p += align_up(sizeof(int32_t) * E);
    w.pre_gt = reinterpret_cast<int32_t*>(p);  p += align_up(sizeof(int32_t) * E * kSelThreads);
    w.pre_eq = reinterpret_cast<int32_t*>(p);  p += align_up(sizeof(int32_t) * E * kSelThreads);
    w.pre_kept = reinterpret_cast<int32_t*>(p); p += align_up(sizeof(int32_t) * E * kSelThreads);
    w.hist1 = reinterpret_cast<uint32_t*>(p);
    w.ipt = chunk_tokens(T);
    w.n_slices = select_slices(T);
    w.slice = w.n_slices ? ((T + w.n_slices - 1) / w.n_slices + 3) / 4 * 4 : 0;
    return w;
}

hipError_t static_select_scratch(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (!p) return hipErrorInvalidSymbol;
        ptrs[dev] = p;
    }
    *out = ptrs[dev];
    return hipSuccess;
}

// Lists of the chosen pairs instead of a key for every (token, expert): where experts are chosen by an eighth of the tokens on
// average, and by a quarter where the capacity has room for the even share and a quarter more.  How many tokens choose one expert the
// host does not know, so both forms were measured with loads that are even, skewed (affinities to expert e ahead by 0.1 / e), halved
// (half of all tokens on one expert, a quarter on the next) and with all tokens on one.  Selection in us, keys / lists, T x E, k, capacity over the even share:
//   65536 x 64, 4, 1.25: even 58 / 21, halved 58 / 40, one 59 / 42      65536 x 16, 2, 1.25: even 37 / 12, halved 37 / 32, one 37 / 33
//   8192 x 16, 2, 1.0: even 14.8 / 14.0, one 14.8 / 14.0              position priority, 65536 x 16, 2, 1.0: one 143 / 24
//   a quarter: 2048 x 8, 2, 1.25: even 13.2 / 9.1, skewed 13.2 / 12.5, halved 13.3 / 13.7; 65536 x 16, 4, 1.25: even 39 / 13, halved 39 / 39
//   a quarter without room: 2048 x 8, 2, 1.0: even 12.1 / 12.4; 16384 x 16, 4, 0.9: 16.2 / 17.8; 65536 x 8, 2, 0.9: 31 / 34, halved 31 / 37
//   a half, 65536 x 8, 4, 0.9: 31 / 54.  Up to 1024 tokens, 1000 x 16, 2: 13.0 / 13.8
// With room lists gain much where the load is even and lose 4 % (one figure 8 %) where it is not.  A capacity that is read on the device
// may leave no room: up to 32768 tokens that costs little (above), beyond it only a search that the affinity sum asks for anyway is
// worth it (65536 x 8, 2, 1.25 with a sum: 45 / 32, halved 51 / 45).  A tile is a thread of the per-expert kernel.
static bool by_lists(const etr_config& c, bool capacity_on_device, bool by_sum) {
    if (c.mode != ETR_MODE_TCR && c.mode != ETR_MODE_TCR_RANK && c.mode != ETR_MODE_BIDIR) return false;
    if (c.k > kListK || c.T <= 1024 || c.T > kTileTokens * kSelThreads) return false;
    const bool room = c.mode == ETR_MODE_TCR ||
                      (4ll * c.E * c.capacity >= 5ll * c.T * c.k && (!capacity_on_device || by_sum || c.T <= 32768));
    return 8 * c.k <= c.E || (4 * c.k <= c.E && room);
}

hipError_t launch_select(const etr_config& c, const float* score, int32_t* topk_expert, int32_t* slot_of,
                         int32_t* slot_token, int32_t* counts, const SelectWs& w, hipStream_t st,
                         const int32_t* capacity_dev, long long sum_need) {
    if (c.T <= kSmallTokens && c.mode != ETR_MODE_BIDIR_STRICT) {
        const bool by_sum = sum_need > 0 && (c.mode == ETR_MODE_ECR || c.mode == ETR_MODE_BIDIR);
        hipLaunchKernelGGL(by_sum ? small_select_kernel<true> : small_select_kernel<false>, dim3(c.E),
                           dim3((c.T + kWave - 1) / kWave * kWave), 0, st, score, c.T, c.E, c.k, c.capacity, c.mode, capacity_dev,
                           sum_need, topk_expert, slot_of, slot_token, counts);
        return hipGetLastError();
    }
    if (by_lists(c, capacity_dev != nullptr, sum_need > 0)) {
        const ChoiceLists lists = carve_lists(w, c.T, c.E, c.k);
        hipLaunchKernelGGL(choice_lists_kernel, dim3(lists.tiles), dim3(256), 0, st, score, c.T, c.E, c.k, c.mode, topk_expert, lists);
        auto kern = [&](auto adapted) {
            constexpr bool A = decltype(adapted)::value;
            const int per_wave = (lists.tiles + kSelThreads / kWave - 1) / (kSelThreads / kWave);
            return per_wave <= 4 ? expert_lists_kernel<A, 4> : per_wave <= 8 ? expert_lists_kernel<A, 8> : per_wave <= 16 ? expert_lists_kernel<A, 16>
                 : per_wave <= 32 ? expert_lists_kernel<A, 32> : expert_lists_kernel<A, 64>;
        };
        hipLaunchKernelGGL(sum_need > 0 ? kern(std::true_type{}) : kern(std::false_type{}), dim3(c.E), dim3(kSelThreads), 0, st, lists,
                           c.E, c.k, c.capacity, c.mode, capacity_dev, sum_need, w.tau, w.need_eq, w.pre_gt, w.pre_eq, counts);
        hipLaunchKernelGGL(slot_lists_kernel, dim3(lists.tiles), dim3(kTileTokens * kListK), 0, st, lists, c.T, c.E, c.k, c.capacity, w.tau,
                           w.need_eq, w.pre_gt, w.pre_eq, counts, slot_of, slot_token);
        return hipGetLastError();
    }
    int G = 1;
    while (G < c.E) G <<= 1;
#define ETR_TC(GG)                                                                                              \
    hipLaunchKernelGGL(token_choice_kernel<GG>, dim3((c.T + token_tile<GG>() - 1) / token_tile<GG>()),         \
                       dim3(token_threads<GG>()), 0, st,                                                        \
                       score, c.T, c.E, c.k, c.mode, topk_expert, w.cmask, w.keyT, w.Tpad)
    switch (G) {
        case 1: ETR_TC(1); break;
        case 2: ETR_TC(2); break;
        case 4: ETR_TC(4); break;
        case 8: ETR_TC(8); break;
        case 16: ETR_TC(16); break;
        case 32: ETR_TC(32); break;
        default: ETR_TC(64); break;
    }
#undef ETR_TC
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;

    // TCR keeps by position and searches nothing, so it skips the pre-pass
    const bool pre = w.n_slices > 0 && c.mode != ETR_MODE_TCR;
    if (pre) {
        hipLaunchKernelGGL(key_histogram_kernel, dim3(w.n_slices, c.E), dim3(256), 0, st, w.keyT, w.Tpad, c.T, w.slice,
                           w.hist1);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    const bool adapt = sum_need > 0;
#define ETR_EC1(II, PP, AA)                                                                                           \
    hipLaunchKernelGGL((expert_choice_kernel<II, PP, AA>), dim3(c.E), dim3(kSelThreads), 0, st, w.keyT, w.Tpad, c.T, w.ipt, \
                       c.capacity, c.mode, capacity_dev, sum_need, w.tau, w.need_eq, w.pre_gt, w.pre_eq, counts, w.hist1, \
                       w.n_slices)
#define ETR_EC(II, PP) do { if (adapt) ETR_EC1(II, PP, true); else ETR_EC1(II, PP, false); } while (0)
    if (w.ipt == 4) ETR_EC(4, false);                       // (the register variants take exactly their chunk length)
    else if (w.ipt == 8) ETR_EC(8, false);
    else if (w.ipt == 16) ETR_EC(16, false);
    else if (w.ipt == 32) ETR_EC(32, false);                // (no pre-pass up to here, see select_slices)
    else if (w.ipt == 64) { if (pre) ETR_EC(64, true); else ETR_EC(64, false); }
    else { if (pre) ETR_EC(0, true); else ETR_EC(0, false); }
#undef ETR_EC
#undef ETR_EC1
    err = hipGetLastError();
    if (err != hipSuccess) return err;

    if (c.mode == ETR_MODE_BIDIR_STRICT) {
        hipLaunchKernelGGL(strict_filter_kernel, dim3(c.E), dim3(kSelThreads), 0, st, w.keyT, w.Tpad, c.T, w.ipt, w.cmask,
                           w.tau, w.need_eq, w.pre_eq, w.pre_kept, counts);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    const int tile3 = w.ipt > kWave ? w.ipt : kWave;     // tokens per workgroup of slot_kernel
    const int blocks3 = (c.T + tile3 - 1) / tile3;
    const int waves3 = c.E < 4 ? 4 : (c.E > 16 ? 16 : c.E);   // one expert per wave up to 16 waves
    hipLaunchKernelGGL(slot_kernel, dim3(blocks3), dim3(waves3 * kWave), 0, st, w.cmask, c.T, c.E, c.capacity, c.mode, w.ipt,
                       w.tau, w.need_eq, w.pre_gt, w.pre_eq, counts, slot_of, slot_token, w.keyT, w.Tpad, w.pre_kept);
    return hipGetLastError();
}

}  // namespace etr
