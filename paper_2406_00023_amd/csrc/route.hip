// GrAP pooling, cosine affinity and gate (Sec. Cost-Efficient Sparse Expert-Token
// Affinity, Eqs. 2-4; gate = row softmax of Eq. 1's text).
//
// HBM-bound: every token row is read exactly once with 16-byte loads; one
// wavefront owns one token.  The pooled vector g (P floats) is reduced inside
// the wave (vector-unit permutes) and staged in LDS; the expert embeddings sit in
// LDS with a padded row stride so that the E x L lane grid of the dot-product
// stage reads conflict-free.  Scores and gates leave as fp32.
#include <algorithm>
#include <type_traits>

#include "etr_internal.h"

namespace etr {
namespace {

constexpr int kUnroll = 8;
// Waves resident per SIMD.  Measured on the 32-expert workload (48 us at 4): 5 need at most 96 registers, spill, and take
// 59 us; keeping a lane's share of its embedding row in registers (172 registers, two waves
// per SIMD) takes 83 us.  The kernel lives on loads in flight, but not at the price of spills.
constexpr int kRouteWavesPerSimd = 4;

// g lives in a per-wave LDS region: a wave's LDS instructions execute in issue order, so ordering
// them in the instruction stream is all that is needed (no workgroup barrier, no waiting)
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f(value of this lane, value of lane ^ M) in the vector unit, in either order (f commutes); all lanes active.  Through LDS
// (__shfl_xor), some 40 a token, 32768 tokens x 32 experts x 128 features took 51.5 us, 48.5 so; 512 x 8 x 32 (fp32) 5.6, 4.6.
template <int CTRL>
__device__ __forceinline__ uint32_t permuted(uint32_t u) { return __builtin_amdgcn_update_dpp(0, u, CTRL, 0xF, 0xF, true); }
template <int M, typename F>
__device__ __forceinline__ float with_lane_xor(float v, F f) {
    const uint32_t u = __float_as_uint(v);
    if constexpr (M >= 16) {                             // rows, halves of the wave swapped between two copies
        const auto r = [&] {
            if constexpr (M == 32) return __builtin_amdgcn_permlane32_swap(u, u, false, false);
            else return __builtin_amdgcn_permlane16_swap(u, u, false, false);
        }();
        return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    } else {
        uint32_t o;
        if constexpr (M == 8) o = permuted<0x128>(u);                                // row_ror:8
        else if constexpr (M == 4) o = permuted<0x1B>(permuted<0x141>(u));           // ^ 7 (row_half_mirror), ^ 3 (quad_perm 3210)
        else if constexpr (M == 2) o = permuted<0x4E>(u);                            // quad_perm 2301
        else o = permuted<0xB1>(u);                                                  // quad_perm 1032
        return f(v, __uint_as_float(o));
    }
}
struct Add { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct Max { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Butterfly steps from, 2 from, ... below to (powers of two, wave-uniform), N values at a time.
template <int N, typename F>
__device__ __forceinline__ void butterflies(float (&v)[N], int from, int to, F f) {
    auto step = [&](auto m) {
        constexpr int M = decltype(m)::value;
        if (from <= M && M < to) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = with_lane_xor<M>(v[i], f);
        }
    };
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 8>{});
    step(std::integral_constant<int, 16>{});
    step(std::integral_constant<int, 32>{});
}
template <typename F>
__device__ __forceinline__ float butterflies(float v, int from, int to, F f) {
    float one[1] = {v};
    butterflies(one, from, to, f);
    return one[0];
}
template <int M = 32>
__device__ __forceinline__ float wave_sum(float v) {     // widest step first
    v = with_lane_xor<M>(v, Add{});
    if constexpr (M > 1) v = wave_sum<M / 2>(v);
    return v;
}

template <bool BF16>
struct Chunk;   // one 16-byte piece of a token row

__device__ __forceinline__ uint4 load_chunk(const void* row, int c, bool ok) {
    return ok ? reinterpret_cast<const uint4*>(row)[c] : make_uint4(0u, 0u, 0u, 0u);
}

template <>
struct Chunk<false> {
    static constexpr int kVec = 4;
    __device__ static void unpack(const uint4& v, float* f) {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
    __device__ static float scalar(const void* row, int i) { return reinterpret_cast<const float*>(row)[i]; }
    // s += sum of the chunk, xx += sum of squares
    __device__ static void accumulate(const uint4& v, float& s, float& xx) {
        float f[4];
        unpack(v, f);
#pragma unroll
        for (int j = 0; j < 4; ++j) { s += f[j]; xx = fmaf(f[j], f[j], xx); }
    }
};

template <>
struct Chunk<true> {
    static constexpr int kVec = 8;
    __device__ static void unpack(const uint4& v, float* f) {
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
        f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xFFFF0000u);
        f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xFFFF0000u);
    }
    __device__ static float scalar(const void* row, int i) {
        return __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t*>(row)[i]) << 16);
    }
    // s += sum of the chunk, xx += sum of squares: two-element bf16 dot products with fp32 accumulation
    // (v_dot2c_f32_bf16), one instruction per pair instead of unpack + add + fma
    __device__ static void accumulate(const uint4& v, float& s, float& xx) {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const bf16x2 one = __builtin_bit_cast(bf16x2, 0x3F803F80u);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bf16x2 p2 = __builtin_bit_cast(bf16x2, w[j]);
            s = __builtin_amdgcn_fdot2_f32_bf16(p2, one, s, false);
            xx = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, xx, false);
        }
    }
};

struct RouteParams {
    int T, d, E, D, P;
    int cos_mode;
    int L;          // lanes cooperating on one expert in the dot-product stage (power of two, E*L <= 64)
    int w_stride;   // padded LDS row stride of the embeddings (floats)
    int R;          // 16-byte chunks per pooling group when that is a power of two <= 64, else 0
};

// FAST: the whole row fits one pass of kUnroll loads per lane and pools with lane shuffles;
// otherwise the general walk (several passes, or one lane per pooled feature).
// W: waves of a workgroup, which share one copy of the embeddings in LDS.
template <bool BF16, bool FAST, int W>
__global__ __launch_bounds__(W * kWave, kRouteWavesPerSimd) void route_kernel(RouteParams p, const void* __restrict__ x,
                                                              const float* __restrict__ w_emb,
                                                              float* __restrict__ score, float* __restrict__ gate) {
    using C = Chunk<BF16>;
    constexpr int V = C::kVec;
    extern __shared__ float smem[];
    float* Ws = smem;                                  // [E][w_stride]
    float* wn = Ws + p.E * p.w_stride;                 // [64] embedding norms
    float* gs = wn + 64;                               // [waves][P]

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int nchunks = p.d / V;
    const size_t row_bytes = static_cast<size_t>(p.d) * (BF16 ? 2 : 4);
    // one pass of kUnroll 16-byte loads per lane covers d <= 64 * kUnroll * V elements (4096 bf16):
    // then the row of the NEXT token is fetched while the current one is reduced
    constexpr bool one_pass = FAST;
    uint4 raw[FAST ? kUnroll : 1];                                 // the row stays packed until it is reduced
    auto fetch = [&](int t) {
        if constexpr (FAST) {
            const bool live = t < p.T;
            const char* row = reinterpret_cast<const char*>(x) + static_cast<size_t>(live ? t : 0) * row_bytes;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                int c = u * kWave + lane;
                raw[u] = load_chunk(row, c, live && c < nchunks);
            }
        }
    };
    // the first row is requested before the embeddings are staged, so both latencies overlap
    if (one_pass) fetch(blockIdx.x * W + wave);

    // Embeddings and their norms: a wave takes R rows at a time, so that as many loads and then as many butterflies are
    // in flight.  Row after row, with a division per element, this prologue was half of a small call: 256 tokens x 32
    // experts, 128 pooled features, 19.6 -> 10.8 us; 2 x 64 experts 29 -> 16 us; 32768 x 32 experts 74 -> 66 us.
    auto stage = [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        for (int e0 = wave; e0 < p.E; e0 += W * R) {
            float s[R];
#pragma unroll
            for (int r = 0; r < R; ++r) s[r] = 0.f;
            for (int q = lane; q < p.P; q += kWave) {
                float w[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = e0 + r * W;
                    w[r] = e < p.E ? w_emb[static_cast<size_t>(e) * p.P + q] : 0.f;
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = e0 + r * W;
                    if (e < p.E) Ws[e * p.w_stride + q] = w[r];
                    s[r] += w[r] * w[r];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) s[r] = wave_sum(s[r]);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (lane == 0 && e0 + r * W < p.E) wn[e0 + r * W] = sqrtf(s[r]);
        }
    };
    if (p.E <= 2 * W) stage(std::integral_constant<int, 2>{});
    else stage(std::integral_constant<int, 8>{});
    __syncthreads();

    float* g = gs + wave * p.P;
    const float invD = 1.0f / static_cast<float>(p.D);
    const float sqrtD = sqrtf(static_cast<float>(p.D));
    const int e_lane = lane / p.L, sub = lane & (p.L - 1);

    for (int t0 = blockIdx.x * W; t0 < p.T; t0 += gridDim.x * W) {
        const int t = t0 + wave;
        const bool live = t < p.T;
        const char* row = reinterpret_cast<const char*>(x) + static_cast<size_t>(live ? t : 0) * row_bytes;
        float xx = 0.f;
        if constexpr (one_pass) {
            float s[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                s[u] = 0.f;
                C::accumulate(raw[u], s[u], xx);
            }
            fetch(t + gridDim.x * W);          // next token of this wave (masked past T)
            butterflies(s, 1, p.R, Add{});
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int c = u * kWave + lane;
                if ((lane & (p.R - 1)) == 0 && c < nchunks) g[c / p.R] = s[u] * invD;
            }
        } else if (p.R > 0) {
            for (int c0 = 0; c0 < nchunks; c0 += kWave * kUnroll) {
                uint4 rr[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    int c = c0 + u * kWave + lane;
                    rr[u] = load_chunk(row, c, live && c < nchunks);
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    int c = c0 + u * kWave + lane;
                    float ff[V];
                    C::unpack(rr[u], ff);
                    float s = 0.f;
#pragma unroll
                    for (int j = 0; j < V; ++j) { s += ff[j]; xx += ff[j] * ff[j]; }
                    s = butterflies(s, 1, p.R, Add{});
                    if ((lane & (p.R - 1)) == 0 && c < nchunks) g[c / p.R] = s * invD;
                }
            }
        } else if (p.D % V == 0) {
            // whole 16-byte pieces per group, but not a power of two of them (D = 24): one lane per pooled feature walks
            // its pieces, four requested at a time, adding element after element as the scalar walk does
            // (21342 tokens, 3840 wide: 155 -> 48 us; 36292 tokens, 2496 wide: 164 -> 52 us).
            const int n = p.D / V;
            for (int q = lane; q < p.P; q += kWave) {
                float s = 0.f;
                for (int j0 = 0; j0 < n; j0 += 4) {
                    uint4 rr[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) rr[j] = load_chunk(row, q * n + j0 + j, live && j0 + j < n);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float ff[V];
                        C::unpack(rr[j], ff);
                        if (j0 + j < n) {
#pragma unroll
                            for (int i = 0; i < V; ++i) { s += ff[i]; xx += ff[i] * ff[i]; }
                        }
                    }
                }
                g[q] = s * invD;
            }
        } else {
            // group size not a multiple of the 16-byte vector: scalar walk, one lane per pooled feature
            for (int q = lane; q < p.P; q += kWave) {
                float s = 0.f;
                for (int j = 0; j < p.D; ++j) {
                    float v = live ? C::scalar(row, q * p.D + j) : 0.f;
                    s += v; xx += v * v;
                }
                g[q] = s * invD;
            }
        }
        xx = wave_sum(xx);
        wave_lds_fence();                               // g was written by other lanes of this wave

        float acc = 0.f, gg = 0.f;
        if (e_lane < p.E) {
            const float* wr = Ws + e_lane * p.w_stride;
            if ((p.P & 3) == 0) {
                // four pooled features per LDS access and four independent accumulators: the loop is bound by
                // LDS latency, not bandwidth (the row stride makes the 16-byte reads conflict-free, see launch_route)
                const float4* g4 = reinterpret_cast<const float4*>(g);
                const float4* w4 = reinterpret_cast<const float4*>(wr);
                float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
                auto add = [&](const float4& gv, const float4& wv) {
                    a0 = fmaf(gv.x, wv.x, a0); a1 = fmaf(gv.y, wv.y, a1);
                    a2 = fmaf(gv.z, wv.z, a2); a3 = fmaf(gv.w, wv.w, a3);
                };
                const int n = p.P >> 2;
                int q = sub;
                for (; q + 3 * p.L < n; q += 4 * p.L) {
                    float4 gv[4], wv[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) { gv[i] = g4[q + i * p.L]; wv[i] = w4[q + i * p.L]; }
                    __builtin_amdgcn_sched_barrier(0);   // (or each pair is waited for before the next is requested: 388 / 551 us)
#pragma unroll
                    for (int i = 0; i < 4; ++i) add(gv[i], wv[i]);
                }
                for (; q < n; q += p.L) add(g4[q], w4[q]);
                acc = (a0 + a1) + (a2 + a3);
            } else {
                for (int q = sub; q < p.P; q += p.L) acc += g[q] * wr[q];
            }
        }
        acc = butterflies(acc, 1, p.L, Add{});
        float den;
        if (p.cos_mode == ETR_COS_POOLED) {
            for (int q = lane; q < p.P; q += kWave) gg += g[q] * g[q];
            gg = wave_sum(gg);
            den = sqrtf(gg);
        } else {
            den = sqrtf(xx);
            acc *= sqrtD;
        }
        const bool is_e = e_lane < p.E;
        den *= is_e ? wn[e_lane] : 0.f;
        const float sc = (is_e && den > 0.f) ? acc / den : 0.f;
        const float mx = butterflies(is_e ? sc : -INFINITY, p.L, kWave, Max{});
        const float ex = is_e ? expf(sc - mx) : 0.f;
        const float z = butterflies(ex, p.L, kWave, Add{});
        if (live && is_e && sub == 0) {
            score[static_cast<size_t>(t) * p.E + e_lane] = sc;
            gate[static_cast<size_t>(t) * p.E + e_lane] = ex / z;
        }
        wave_lds_fence();                               // g is rewritten by the next iteration
    }
}

}  // namespace

hipError_t launch_route(const etr_config& c, const void* x, const float* w_emb, float* score, float* gate,
                        hipStream_t st) {
    RouteParams p;
    p.T = c.T; p.d = c.d; p.E = c.E; p.D = c.D; p.P = c.d / c.D; p.cos_mode = c.cos;
    int e2 = 1;
    while (e2 < c.E) e2 <<= 1;
    p.L = kWave / e2;
    // LDS row stride of the embeddings.  Scalar walk (P % 4 != 0): stride = L (mod 64 banks), so the E x L lane grid
    // reads distinct banks.  Vector walk: a 16-byte read is served 16 lanes at a time = 16/L experts x L lanes x 4
    // banks, conflict-free when consecutive rows start 4L banks apart.
    const int step = (p.P % 4 == 0) ? 4 * p.L : p.L;
    p.w_stride = p.P + ((step - p.P % 64) % 64 + 64) % 64;
    const int V = c.dtype == ETR_BF16 ? 8 : 4;
    p.R = 0;
    if (c.D % V == 0) {
        int r = c.D / V;
        if (r <= 64 && (r & (r - 1)) == 0) p.R = r;
    }
    // Waves of a workgroup: the fewest that leave the most waves on a CU, between the embeddings' copies in its 160 KiB and the
    // registers (a call that is resident as a whole with 4 stays there: more workgroups share the staging).  64 experts x 512
    // pooled features (131 KiB) with 4 / 8 waves, 65536 tokens: 388 / 223 us; 32 x 512 (73 KiB), 4 / 16: 156 / 126; 64 x 256 (74
    // KiB), 4 / 8: 159 / 133; 48 x 240 (53 KiB), 40000 tokens, 4 / 8: 102 / 74.
    auto lds_of = [&](int waves) { return sizeof(float) * (static_cast<size_t>(p.E) * p.w_stride + 64 + static_cast<size_t>(waves) * p.P); };
    auto resident_waves = [&](int waves) {
        const size_t fit = 160 * 1024 / lds_of(waves);
        return waves * static_cast<int>(std::min<size_t>(fit, 4 * kRouteWavesPerSimd / waves));
    };
    if (lds_of(4) > 160 * 1024) return hipErrorInvalidValue;
    int waves = 4;
    for (int w = 8; w <= 16; w *= 2)
        if (c.T > cu_count() * resident_waves(4) && resident_waves(w) > resident_waves(waves)) waves = w;
    const size_t lds = lds_of(waves);
    int blocks = (c.T + waves - 1) / waves;
    // What is resident at once, so that a CU stages the embeddings once per place (64 x 512, two workgroups for each place / one:
    // 65536 tokens 211 / 203 us, 6000 tokens 37 / 29).
    const int resident = cu_count() * (resident_waves(waves) / waves);
    if (blocks > resident) blocks = resident;
    if (blocks < 1) blocks = 1;
    const bool fast = p.R > 0 && p.d / V <= kWave * kUnroll;
    auto of_waves = [&](auto w) {
        constexpr int W = decltype(w)::value;
        return c.dtype == ETR_BF16 ? (fast ? route_kernel<true, true, W> : route_kernel<true, false, W>)
                                   : (fast ? route_kernel<false, true, W> : route_kernel<false, false, W>);
    };
    auto kern = waves == 4 ? of_waves(std::integral_constant<int, 4>{})
                           : (waves == 8 ? of_waves(std::integral_constant<int, 8>{}) : of_waves(std::integral_constant<int, 16>{}));
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(waves * kWave), lds, st, p, x, w_emb, score, gate);
    return hipGetLastError();
}

}  // namespace etr
