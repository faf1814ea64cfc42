// Router kernels: gate GEMM (fp32 logits), then per-token top-k with renormalised softmax
// weights.  Follows the paper's description of the MoE router (Sec. 2.1, Sec. 2.2): each token is
// assigned to its k most relevant experts.
//
// bf16: logits come from 16x16x32 bf16 MFMA tiles (16 tokens x 16 experts per tile), fp32
// accumulation.  Wg is [H,E] with E contiguous, the wrong majorness for MFMA operands, so a
// small kernel first writes it transposed (and padded to a multiple of 16 experts) into scratch.
// A workgroup owns 16 tokens; its 8 waves split the hidden dimension into 8 contiguous ranges and
// add their partial tiles through LDS in wave order, so the summation order is fixed; the same
// workgroup then selects the experts (fused, no second launch).
// fp32: one wave per token, lanes stride the hidden dimension, butterfly reduction, then the same selection.
// top-k: k rounds of a wave-wide maximum in the order (logit desc, index asc), or, where the bf16 router chooses
// many of at most 64 experts, the rank of every expert in that order.
//
// These kernels are chains of latencies, 6 to 12 us of a layer of 40 to 500: what counts is their length, and in how many CUs
// the weights are taken in (gate_in_parts).
#include <hip/hip_runtime.h>

#include <climits>
#include <mutex>
#include <type_traits>

#include "qmoe_internal.h"

// Scratch of moe_route_noalloc: the router weight transposed and padded, bf16 [ceil16(E)][H].  One
// copy per GPU the library runs on, held until the process ends.  In host code this name is only a
// handle for hipGetSymbolAddress; kernels get the device address that call returns.
constexpr size_t kRouteScratchBytes = 2u << 20;
static __device__ __align__(256) unsigned char scratch[kRouteScratchBytes];

namespace qmoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void wg_transpose_bf16(const uint16_t *__restrict__ Wg, uint16_t *__restrict__ WgT,
                                                         int H, int E, int E16) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= (long)E16 * H) return;
    const int e = (int)(i / H), h = (int)(i % H);
    WgT[i] = e < E ? Wg[(long)h * E + e] : (uint16_t)0;
}

// Largest value of the wave's 64 lanes, in every lane (v_max_f32 over DPP row shifts and broadcasts; a NaN
// loses against a number).
__device__ __forceinline__ float wave_max(float v) {
    auto step = [&](auto ctrl) {
        const int old = __builtin_bit_cast(int, v);
        v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(old, old, decltype(ctrl)::value, 0xf, 0xf, false)));
    };
    step(std::integral_constant<int, 0x111>{});      // row_shr 1, 2, 4, 8: lane 15 of a row holds the row's maximum
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{});      // row_bcast 15 and 31: lane 63 holds the wave's
    step(std::integral_constant<int, 0x143>{});
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Lane j < k holds the logit and the expert of slot j: the weights are the softmax over the k logits.
// idx_out[h] == nullptr: nothing is stored for token h.
template <int NT>
__device__ __forceinline__ void store_slots(const float (&my_v)[NT], const int (&my_e)[NT], int l, int k,
                                            int32_t *const (&idx_out)[NT], float *const (&w_out)[NT]) {
    float p[NT], s[NT];
#pragma unroll
    for (int h = 0; h < NT; ++h) {
        const float top = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_v[h]), 0));
        p[h] = l < k ? expf(my_v[h] - top) : 0.f;
        s[h] = p[h];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int h = 0; h < NT; ++h) s[h] += __shfl_xor(s[h], o, 64);
#pragma unroll
    for (int h = 0; h < NT; ++h)
        if (l < k && idx_out[h] != nullptr) {
            idx_out[h][l] = my_e[h];
            w_out[h][l] = p[h] / s[h];
        }
}

// Top-k of NT tokens by one wave, side by side.  Lane l holds the logits of experts l, l+64, ... (NS of
// them) in v[h][].  k rounds in the order (logit descending, expert index ascending): the wave's maximum,
// one ballot per slot for the lanes that hold it, the first of them is taken.  What is left is kept as
// one bit mask per slot, so that a logit of -inf is chosen like any other; if only NaNs are left the
// lowest index is taken.  Lane j ends up with slot j; weights = softmax over the k selected logits.
// Bound by the latency of a round, k rounds.  Comparing every expert with every other one (the tokens'
// logits in LDS) took 15000 cycles for 64 experts, top-8, 16 tokens in 8 waves: of the router's 17.8 us on
// 32 tokens x 64 experts it left 13.9, and 11.4 -> 9.6 on 64 x 8.
// idx_out[h] == nullptr: nothing is stored for token h.
constexpr int kSlots = kMaxExperts / 64;
template <int NT, int NS>
__device__ __forceinline__ void wave_topk(const float (&v)[NT][NS], int l, int E, int k, int32_t *const (&idx_out)[NT],
                                          float *const (&w_out)[NT]) {
    unsigned long long left[NT][NS];
    float cur[NT][NS], my_v[NT];                     // cur: v with what has been taken set to -inf
    int my_e[NT];
#pragma unroll
    for (int h = 0; h < NT; ++h) {
        my_v[h] = 0.f;
        my_e[h] = 0;
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            left[h][c] = __ballot(l + 64 * c < E);
            cur[h][c] = l + 64 * c < E ? v[h][c] : -INFINITY;
        }
    }
    for (int j = 0; j < k; ++j) {
#pragma unroll
        for (int h = 0; h < NT; ++h) {
            float best = -INFINITY;
#pragma unroll
            for (int c = 0; c < NS; ++c) best = fmaxf(best, cur[h][c]);
            best = wave_max(best);
            int e = -1, any = 0;
#pragma unroll
            for (int c = NS - 1; c >= 0; --c) {
                const unsigned long long m = __ballot(v[h][c] == best) & left[h][c];
                if (m) e = 64 * c + __builtin_ctzll(m);
                if (left[h][c]) any = 64 * c + __builtin_ctzll(left[h][c]);
            }
            if (e < 0) e = any;
            float ev = v[h][0];
#pragma unroll
            for (int c = 0; c < NS; ++c)
                if (c == e >> 6) {
                    left[h][c] &= ~(1ull << (e & 63));
                    cur[h][c] = l == (e & 63) ? -INFINITY : cur[h][c];
                    ev = v[h][c];
                }
            ev = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ev), e & 63));
            if (l == j) { my_v[h] = ev; my_e[h] = e; }
        }
    }
    store_slots<NT>(my_v, my_e, l, k, idx_out, w_out);
}

// The same by ranks, for E <= 64: lane l counts the experts that precede its own (a NaN is less than any number,
// as above) and hands its logit to lane `rank`.  It costs E comparisons whatever k is, where wave_topk costs k
// rounds.
__device__ __forceinline__ int order_key(float v) {
    const int b = __builtin_bit_cast(int, v + 0.f);          // -0 and 0 are equal
    return v != v ? INT_MIN : b ^ ((b >> 31) & INT_MAX);
}
template <int NT>
__device__ __forceinline__ void wave_topk_rank(const float (&v)[NT][1], int l, int E, int k, int32_t *const (&idx_out)[NT],
                                               float *const (&w_out)[NT]) {
    int key[NT], rank[NT], my_e[NT];
    float my_v[NT];
#pragma unroll
    for (int h = 0; h < NT; ++h) {
        key[h] = l < E ? order_key(v[h][0]) : INT_MIN;
        rank[h] = 0;
    }
    for (int o0 = 0; o0 < E; o0 += 8) {                      // lanes from E on precede no expert
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                const int other = __builtin_amdgcn_readlane(key[h], o0 + i);
                rank[h] += other > key[h] || (other == key[h] && o0 + i < l) ? 1 : 0;
            }
    }
#pragma unroll
    for (int h = 0; h < NT; ++h) {                           // lanes from E on have ranks from E on: lanes of no slot
        my_v[h] = __builtin_bit_cast(float, __builtin_amdgcn_ds_permute(4 * rank[h], __builtin_bit_cast(int, v[h][0])));
        my_e[h] = __builtin_amdgcn_ds_permute(4 * rank[h], l);
    }
    store_slots<NT>(my_v, my_e, l, k, idx_out, w_out);
}

// Gate GEMM and top-k of 16 tokens per workgroup.  NB = number of 16-expert blocks held in
// registers (E16 <= 16*NB).  The 8 waves split the hidden dimension into 8 contiguous ranges (loads
// issued 8, 4 or 2 k-steps at a time), add their partial tiles through LDS in wave order, and then
// each wave selects the experts of 2 of the 16 tokens.
// Up to 128 experts (NB <= 8) registers and LDS leave room for at least two workgroups on a CU, which halves
// the time on 8192 tokens x 64 experts.  NB = 8 has to be told: by itself it takes 132 registers, one workgroup
// per CU, 44.6 us for 8192 tokens x 128 experts, top-8, H 2048; 40.1 us with 128 registers, and small batches
// the same.  NB = 16 fills the LDS of a CU alone.
// PARTS: the partial tiles come from gate_parts_bf16 (same ranges, same chains, so the same logits) instead.
template <int NB, bool PARTS>
__device__ __forceinline__ void gate_topk_tile(const uint16_t *__restrict__ x, const uint16_t *__restrict__ WgT, const float *__restrict__ parts,
                                               const float *__restrict__ bias, float *__restrict__ logits, int32_t *__restrict__ topk_idx,
                                               float *__restrict__ topk_w, int N, int H, int E, int nb, int k) {
    __shared__ float red[PARTS ? 1 : 8][NB][4][64];
    __shared__ float lt[16][NB * 16 + 1];
    __shared__ float sbias[NB * 16];
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int t16 = l & 15, q = l >> 4;
    if (tid < NB * 16) sbias[tid] = (bias && tid < E) ? bias[tid] : 0.f;   // read after the first barrier
    if constexpr (!PARTS) {
        int tok = blockIdx.x * 16 + t16;
        if (tok > N - 1) tok = N - 1;
        const int steps = H / 32;
        const int per = (steps + 7) / 8;
        const int s0 = w * per, s1 = min(steps, s0 + per);
        f32x4 acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint16_t *xa = x + (long)tok * H + q * 8;
        // Expert rows from E on are padding: their lanes read the last expert again (no bytes of their own), and
        // nothing uses what they compute.  A CU takes 11 to 20 bytes a clock here: with 8 experts that is half
        // of the weights' time (one token, H 4096: 7.7 -> 5.7 us; all k-steps requested at once gave nothing).
        const uint16_t *wb[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) wb[b] = WgT + (long)min(b * 16 + t16, E - 1) * H + q * 8;
        constexpr int CH = NB == 1 ? 8 : (NB == 2 ? 4 : 2);   // k-steps whose loads are issued together
        for (int s = s0; s < s1; s += CH) {
            bf16x8 a[CH], bv[CH][NB];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int sc = min(s + c, s1 - 1);
                a[c] = *reinterpret_cast<const bf16x8 *>(xa + sc * 32);
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    bv[c][b] = *reinterpret_cast<const bf16x8 *>(wb[b] + sc * 32);
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (s + c < s1) {
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (b < nb) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], bv[c][b], acc[b], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[w][b][r][l] = acc[b][r];
    }
    __syncthreads();
    // The NB*4 (expert block, D register) pairs are dealt to the 8 waves; each sum runs over the waves'
    // partial tiles in wave order.
#pragma unroll
    for (int j = 0; j < (NB * 4 + 7) / 8; ++j) {
        const int pr = w + 8 * j;
        const int b = pr >> 2, r = pr & 3;
        if (pr < NB * 4 && b < nb) {
            float p[8];
#pragma unroll
            for (int ww = 0; ww < 8; ++ww) {
                if constexpr (PARTS) p[ww] = parts[(((long)blockIdx.x * 8 + ww) * nb + b) * 256 + l * 4 + r];
                else p[ww] = red[ww][b][r][l];
            }
            float v = p[0];
#pragma unroll
            for (int ww = 1; ww < 8; ++ww) v += p[ww];
            const int e = b * 16 + t16;                 // D: column = expert
            const int tl = q * 4 + r;                   // D: row = token (within the 16)
            const int t = blockIdx.x * 16 + tl;
            const float lv = v + sbias[e];
            lt[tl][e] = lv;
            if (e < E && t < N) logits[(long)t * E + e] = lv;
        }
    }
    __syncthreads();
    const int t0 = blockIdx.x * 16 + w * 2;             // this wave's two tokens
    if (t0 < N) {
        constexpr int NS = (NB + 3) / 4;
        float v[2][NS];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < NS; ++c) v[h][c] = l + 64 * c < E ? lt[w * 2 + h][l + 64 * c] : -INFINITY;
        int32_t *const io[2] = {topk_idx + (long)t0 * k, t0 + 1 < N ? topk_idx + (long)(t0 + 1) * k : nullptr};
        float *const wo[2] = {topk_w + (long)t0 * k, t0 + 1 < N ? topk_w + (long)(t0 + 1) * k : nullptr};
        // Ranks from a quarter of the experts on: 32 tokens, H 2048 (H 4096 for 8 experts), us by rounds / by ranks:
        // top-2 of 8 8.9 / 8.9, top-8 of 8 10.7 / 8.9; of 16 top-2 6.6 / 7.1, top-4 7.2 / 7.1, top-16 10.5 / 7.1;
        // of 32 top-6 9.6 / 9.8, top-8 10.1 / 9.7, top-32 17.0 / 9.8; of 64 top-8 13.7 / 15.5, top-16 16.2 / 15.4,
        // top-32 20.8 / 15.5.  Above 64 experts the rounds are the faster ones up to the largest k.
        if constexpr (NS == 1) {
            if (4 * k >= E) {
                wave_topk_rank<2>(v, l, E, k, io, wo);
                return;
            }
        }
        wave_topk<2, NS>(v, l, E, k, io, wo);
    }
}

template <int NB>
__global__ __launch_bounds__(512, NB == 8 ? 4 : 2) void gate_topk_bf16(const uint16_t *__restrict__ x, const uint16_t *__restrict__ WgT,
                                                      const float *__restrict__ bias, float *__restrict__ logits,
                                                      int32_t *__restrict__ topk_idx, float *__restrict__ topk_w, int N, int H,
                                                      int E, int nb, int k) {
    gate_topk_tile<NB, false>(x, WgT, nullptr, bias, logits, topk_idx, topk_w, N, H, E, nb, k);
}

template <int NB>
__global__ __launch_bounds__(512) void add_topk_bf16(const float *__restrict__ parts, const float *__restrict__ bias, float *__restrict__ logits,
                                                     int32_t *__restrict__ topk_idx, float *__restrict__ topk_w, int N, int E, int nb, int k) {
    gate_topk_tile<NB, true>(nullptr, nullptr, parts, bias, logits, topk_idx, topk_w, N, 0, E, nb, k);
}

// The gate GEMM alone, for batches whose token tiles are too few to fill the chip: workgroup (token tile, K range), one wave
// per 16-expert block, its partial tile to memory where add_topk_bf16 adds them.  Each CU then
// reads an eighth of the weights.
__global__ __launch_bounds__(1024) void gate_parts_bf16(const uint16_t *__restrict__ x, const uint16_t *__restrict__ WgT, float *__restrict__ parts,
                                                        int N, int H, int E) {
    const int b = threadIdx.x >> 6, l = threadIdx.x & 63, nb = blockDim.x >> 6;
    const int t16 = l & 15, q = l >> 4;
    const uint16_t *xa = x + (long)min((int)blockIdx.x * 16 + t16, N - 1) * H + q * 8;
    const uint16_t *wb = WgT + (long)min(b * 16 + t16, E - 1) * H + q * 8;
    const int steps = H / 32, per = (steps + 7) / 8;
    const int s0 = blockIdx.y * per, s1 = min(steps, s0 + per);
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    constexpr int CH = 8;
    for (int s = s0; s < s1; s += CH) {
        bf16x8 a[CH], w[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int sc = min(s + c, s1 - 1);
            a[c] = *reinterpret_cast<const bf16x8 *>(xa + sc * 32);
            w[c] = *reinterpret_cast<const bf16x8 *>(wb + sc * 32);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (s + c < s1) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], w[c], acc, 0, 0, 0);
    }
    *reinterpret_cast<f32x4 *>(parts + (((long)blockIdx.x * 8 + blockIdx.y) * nb + b) * 256 + l * 4) = acc;
}

// One wave per token: lane l sums the elements h = l, l + 64, ... of EB logits at a time (U of them
// loaded together), a butterfly adds the lanes, and the wave selects its experts.  VEC: E is a multiple of
// EB, so the EB weights of a row are read 16 bytes at a time (rows need only 4-byte alignment).
// 509 tokens x 8 experts, H 1024: 20.6 us with scalar loads one element at a time, and 4.8 us for the
// selection as a launch of its own; 6.2 us here.  The sums are the same, bit for bit.
template <int EB, bool VEC>
__global__ __launch_bounds__(256) void gate_topk_f32(const float *__restrict__ x, const float *__restrict__ Wg,
                                                     const float *__restrict__ bias, float *__restrict__ logits,
                                                     int32_t *__restrict__ topk_idx, float *__restrict__ topk_w, int N, int H,
                                                     int E, int k) {
    constexpr int U = 8;
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int tok = blockIdx.x * 4 + w;
    if (tok >= N) return;
    const float *xr = x + (long)tok * H;
    float v[1][kSlots];
#pragma unroll
    for (int c = 0; c < kSlots; ++c) v[0][c] = -INFINITY;
    for (int e0 = 0; e0 < E; e0 += EB) {
        float acc[EB];
#pragma unroll
        for (int j = 0; j < EB; ++j) acc[j] = 0.f;
        for (int h0 = l; h0 < H; h0 += 64 * U) {
            float xv[U], wv[U][EB];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int h = min(h0 + 64 * u, H - 1);
                xv[u] = xr[h];
                const float *wr = Wg + (long)h * E + e0;
                if constexpr (VEC) {
#pragma unroll
                    for (int j = 0; j < EB; j += 4) {
                        const f32x4u t = *reinterpret_cast<const f32x4u *>(wr + j);
                        wv[u][j] = t[0]; wv[u][j + 1] = t[1]; wv[u][j + 2] = t[2]; wv[u][j + 3] = t[3];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < EB; ++j) wv[u][j] = e0 + j < E ? wr[j] : 0.f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (h0 + 64 * u < H) {
#pragma unroll
                    for (int j = 0; j < EB; ++j) acc[j] = fmaf(xv[u], wv[u][j], acc[j]);
                }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < EB; ++j) acc[j] += __shfl_xor(acc[j], o, 64);
#pragma unroll
        for (int j = 0; j < EB; ++j) {
            const int e = e0 + j;
            if (e < E && (e & 63) == l) {
                const float lg = acc[j] + (bias ? bias[e] : 0.f);
                logits[(long)tok * E + e] = lg;
#pragma unroll
                for (int c = 0; c < kSlots; ++c)
                    if (c == e >> 6) v[0][c] = lg;
            }
        }
    }
    int32_t *const io[1] = {topk_idx + (long)tok * k};
    float *const wo[1] = {topk_w + (long)tok * k};
    wave_topk<1, kSlots>(v, l, E, k, io, wo);
}

}  // namespace

hipError_t launch_pack_gate(const void *Wg, void *WgT, int H, int E, hipStream_t s) {
    const int E16 = (E + 15) / 16 * 16;
    const long tot = (long)E16 * H;
    hipLaunchKernelGGL(wg_transpose_bf16, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, (const uint16_t *)Wg,
                       (uint16_t *)WgT, H, E, E16);
    return hipGetLastError();
}

hipError_t launch_route(const RouteArgs &a, hipStream_t s) {
    if (a.N <= 0) return hipSuccess;
    if (a.dtype == MOE_BF16) {
        const int E16 = (a.E + 15) / 16 * 16, nb = E16 / 16;
        const long tot = (long)E16 * a.H;
        if (!a.packed)
            hipLaunchKernelGGL(wg_transpose_bf16, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s,
                               (const uint16_t *)a.Wg, (uint16_t *)a.WgT, a.H, a.E, E16);
        const dim3 g((a.N + 15) / 16), b(512);
        const uint16_t *x = (const uint16_t *)a.x, *wt = (const uint16_t *)(a.packed ? a.Wg : a.WgT);
        const bool parts = a.parts != nullptr && gate_in_parts(a.N, a.E, a.H);
        if (parts) hipLaunchKernelGGL(gate_parts_bf16, dim3(g.x, 8), dim3(64 * nb), 0, s, x, wt, a.parts, a.N, a.H, a.E);
#define QMOE_GATE(NBV)                                                                                                                       \
    if (parts) hipLaunchKernelGGL(add_topk_bf16<NBV>, g, b, 0, s, a.parts, a.bias, a.logits, a.topk_idx, a.topk_w, a.N, a.E, nb, a.k);      \
    else hipLaunchKernelGGL(gate_topk_bf16<NBV>, g, b, 0, s, x, wt, a.bias, a.logits, a.topk_idx, a.topk_w, a.N, a.H, a.E, nb, a.k)
        if (nb <= 1) { QMOE_GATE(1); }
        else if (nb <= 2) { QMOE_GATE(2); }
        else if (nb <= 4) { QMOE_GATE(4); }
        else if (nb <= 8) { QMOE_GATE(8); }
        else { QMOE_GATE(16); }
#undef QMOE_GATE
    } else {
        const dim3 g((a.N + 3) / 4), b(256);
        const float *x = (const float *)a.x, *wg = (const float *)a.Wg;
        if (a.E % 8 == 0) hipLaunchKernelGGL((gate_topk_f32<8, true>), g, b, 0, s, x, wg, a.bias, a.logits, a.topk_idx, a.topk_w, a.N, a.H, a.E, a.k);
        else if (a.E % 4 == 0) hipLaunchKernelGGL((gate_topk_f32<4, true>), g, b, 0, s, x, wg, a.bias, a.logits, a.topk_idx, a.topk_w, a.N, a.H, a.E, a.k);
        else hipLaunchKernelGGL((gate_topk_f32<8, false>), g, b, 0, s, x, wg, a.bias, a.logits, a.topk_idx, a.topk_w, a.N, a.H, a.E, a.k);
    }
    return hipGetLastError();
}

}  // namespace qmoe

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each device, once looked up
}  // namespace

extern "C" int32_t moe_route_noalloc(const moe_config *cfg, const void *x, int32_t n_tokens, const void *Wg,
                                     const float *logit_bias, float *logits, int32_t *topk_idx, float *topk_w, void *stream) {
    using qmoe::set_error;
    if (!cfg) return set_error(MOE_E_ARG, "moe_route_noalloc: null config");
    if (cfg->E < 1 || cfg->E > qmoe::kMaxExperts || cfg->k < 1 || cfg->k > cfg->E || cfg->k > qmoe::kMaxTopK || cfg->H < 1 ||
        (cfg->dtype != MOE_F32 && cfg->dtype != MOE_BF16) || (cfg->dtype == MOE_BF16 && cfg->H % 64))
        return set_error(MOE_E_ARG, "moe_route_noalloc: bad configuration (E 1..256, k 1..min(E,32), bf16 needs H a multiple of 64)");
    if (n_tokens < 0 || (int64_t)n_tokens * cfg->k >= (int64_t)1 << 31) return set_error(MOE_E_ARG, "moe_route_noalloc: n_tokens out of range");
    if (!Wg || !logits || !topk_idx || !topk_w || (n_tokens > 0 && !x)) return set_error(MOE_E_ARG, "moe_route_noalloc: null pointer");
    const size_t need = cfg->dtype == MOE_BF16 ? (size_t)((cfg->E + 15) / 16 * 16) * (size_t)cfg->H * 2 : 0;
    if (need > kRouteScratchBytes)
        return set_error(MOE_E_ARG, "moe_route_noalloc: ceil16(E)*H*2 = %zu bytes exceed the %zu-byte static scratch", need,
                         (size_t)kRouteScratchBytes);
    if (n_tokens == 0) return MOE_OK;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_error(MOE_E_HIP, "moe_route_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return set_error(MOE_E_ARG, "moe_route_noalloc: device %d out of range", dev);
    void *ptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p)
                return set_error(MOE_E_HIP, "moe_route_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
            g_scratch_ptr[dev] = p;
        }
        ptr = g_scratch_ptr[dev];
    }
    qmoe::RouteArgs a{};
    a.x = x; a.Wg = Wg; a.bias = logit_bias;
    a.WgT = ptr;                  // every element the kernels read is rewritten by this call's transpose first
    a.logits = logits; a.topk_idx = topk_idx; a.topk_w = topk_w;
    a.N = n_tokens; a.H = cfg->H; a.E = cfg->E; a.k = cfg->k; a.dtype = cfg->dtype;
    a.packed = false;
    e = qmoe::launch_route(a, (hipStream_t)stream);
    if (e != hipSuccess) return set_error(MOE_E_HIP, "moe_route_noalloc: launch: %s", hipGetErrorString(e));
    return MOE_OK;
}
