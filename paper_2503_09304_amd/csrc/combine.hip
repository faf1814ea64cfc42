// Gate-weighted combine of complete tokens (Sec. 3.1, "Top-k expert selection": finished expert
// outputs are tracked as state and only fully processed tokens feed the next layer).
//   y[n,:] = sum_j w[n,j] * out[inv[n*k+j], :],  j = 0..k-1 in slot order, fp32 fma chain from 0,
// one rounding to the output type.  A gather-reduce: bound by HBM for large batches (8192 tokens x top-8,
// H 2048: 103 us for 571 MB, 5.6 TB/s), by a chain of dependent reads for small ones.  A workgroup takes a token
// or, in small batches, 1024 columns of one: the token's positions and weights are the same for every lane, so they
// come through scalar loads without LDS or barriers, and the rows of a column are all requested before the first is
// used.  Positions through LDS and one row at a time took 5.8 us for 64 tokens (H 4096, top-2, 4 K ranges), 8.2 for
// 512 tokens (2 K ranges), 28.4 for 2048 x top-8 (H 2048) and 103 for 8192 of these; 3.0, 6.2, 26.3 and 103 here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "qmoe_internal.h"

namespace qmoe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// One 16-byte piece of an expert output row.  KS > 1: the down projection left KS partial planes
// (K ranges); they are added here in the fixed order ((p0 + p1) + p2) + p3, so the value is the one a
// separate reduction pass would have stored.  Read once: non-temporal.
template <int KS>
__device__ __forceinline__ f32x4 load_out(const float *__restrict__ p, long plane) {
    f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    if constexpr (KS > 1) {
#pragma unroll
        for (int q = 1; q < KS; ++q) {
            const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p + q * plane));
            v[0] = v[0] + t[0]; v[1] = v[1] + t[1]; v[2] = v[2] + t[2]; v[3] = v[3] + t[3];
        }
    }
    return v;
}

// acc += w[j] * out[inv[j], h..h+3] for j = j0 .. j0+U-1 in slot order: the loads of all U rows are requested
// before the first is used.
template <int KS, int U>
__device__ __forceinline__ void add_rows(f32x4 &acc, const float *__restrict__ out, long plane, const int32_t *__restrict__ inv,
                                         const float *__restrict__ w, int j0, int H, int h) {
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load_out<KS>(out + (long)inv[j0 + u] * H + h, plane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float wj = w[j0 + u];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = fmaf(wj, v[u][i], acc[i]);
    }
}

// done == nullptr: tokens are selected by class (the host has checked that the class is finished).
// done != nullptr: a token is selected when done[] is set for all k of its sorted positions;
// complete[n] (if given) reports the selection.
template <bool BF16, int KS>
__global__ __launch_bounds__(256) void combine_rows(const float *__restrict__ out, long plane, const float *__restrict__ topk_w,
                                                    const int32_t *__restrict__ inv, const uint8_t *__restrict__ cls,
                                                    const uint8_t *__restrict__ done, uint8_t *__restrict__ complete,
                                                    void *__restrict__ y, int H, int k, int class_mask) {
    const int n = blockIdx.x;
    const int32_t *pos = inv + (long)n * k;             // the same for every lane: scalar loads
    const float *wgt = topk_w + (long)n * k;
    if (done == nullptr) {
        const int bit = cls[n] == 0 ? MOE_CLASS_LS : MOE_CLASS_BE;
        if (!(class_mask & bit)) return;
    } else {
        const int lane = threadIdx.x & 63;              // lane j of every wave looks at row j (k <= 32)
        const bool missing = __any(lane < k && done[pos[lane]] == 0);
        if (complete != nullptr && blockIdx.y == 0 && threadIdx.x == 0) complete[n] = missing ? 0 : 1;
        if (missing) return;
    }
    const int step = (int)gridDim.y * 256;
    if ((H & 3) == 0) {
        constexpr int U = KS == 4 ? 4 : 8;              // at most 16 rows of 16 bytes in flight per lane
        for (int h = ((int)blockIdx.y * 256 + (int)threadIdx.x) * 4; h < H; h += step * 4) {
            f32x4 acc{0.f, 0.f, 0.f, 0.f};
            int j = 0;
            for (; j + U <= k; j += U) add_rows<KS, U>(acc, out, plane, pos, wgt, j, H, h);
            if (U > 4 && (k & 4)) { add_rows<KS, 4>(acc, out, plane, pos, wgt, j, H, h); j += 4; }
            if (k & 2) { add_rows<KS, 2>(acc, out, plane, pos, wgt, j, H, h); j += 2; }
            if (k & 1) add_rows<KS, 1>(acc, out, plane, pos, wgt, j, H, h);
            if (BF16) {
                __bf16 r[4] = {(__bf16)acc[0], (__bf16)acc[1], (__bf16)acc[2], (__bf16)acc[3]};
                *reinterpret_cast<uint2 *>((uint16_t *)y + (long)n * H + h) = *reinterpret_cast<uint2 *>(r);
            } else {
                *reinterpret_cast<f32x4 *>((float *)y + (long)n * H + h) = acc;
            }
        }
    } else {
        for (int h = (int)blockIdx.y * 256 + (int)threadIdx.x; h < H; h += step) {
            float acc = 0.f;
            for (int j = 0; j < k; ++j) {
                const long at = (long)pos[j] * H + h;
                float v = out[at];
#pragma unroll
                for (int q = 1; q < KS; ++q) v = v + out[q * plane + at];
                acc = fmaf(wgt[j], v, acc);
            }
            if (BF16) ((__bf16 *)y)[(long)n * H + h] = (__bf16)acc;
            else ((float *)y)[(long)n * H + h] = acc;
        }
    }
}

// done[row] = 1 for the rows of up to kMaxSegs row ranges: one workgroup per range.
struct MarkArgs {
    int n;
    Seg seg[kMaxSegs];
};

__global__ __launch_bounds__(256) void mark_rows(const MarkArgs m, uint8_t *__restrict__ done) {
    const Seg g = m.seg[blockIdx.x];
    for (int r = threadIdx.x; r < g.rows; r += 256) done[g.row0 + r] = 1;
}

__global__ __launch_bounds__(256) void clear_bytes(uint8_t *__restrict__ p, long n) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) p[i] = 0;
}

__global__ void gate_kernel(const int32_t *__restrict__ stop_host, int32_t *__restrict__ go, int g) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int prev_open = g == 0 ? 1 : go[g - 1];
    const int stop = __hip_atomic_load(stop_host, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    go[g] = (prev_open && stop == 0) ? 1 : 0;
}

struct ReportArgs {
    int n;
    Seg seg[kMaxSegs];
};

__global__ __launch_bounds__(256) void report_ranges(const ReportArgs r, const int32_t *__restrict__ cnt_dn,
                                                     int32_t *__restrict__ ok_host, int dtype, int H, int ksplit) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= r.n) return;
    const Seg g = r.seg[i];
    const int ok = cnt_dn[g.row0] == down_wgs_of_range(dtype, H, ksplit, g.rows) ? 1 : 0;
    __hip_atomic_store(ok_host + i, ok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void clear_words(int32_t *__restrict__ p, long n) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long)gridDim.x * 256) p[i] = 0;
}

}  // namespace

hipError_t launch_gate(const int32_t *stop_host, int32_t *go, int g, hipStream_t s) {
    hipLaunchKernelGGL(gate_kernel, dim3(1), dim3(64), 0, s, stop_host, go, g);
    return hipGetLastError();
}

hipError_t launch_report(const Seg *ranges, int n, const int32_t *cnt_dn, int32_t *ok_host, int dtype, int H, int ksplit,
                         hipStream_t s) {
    for (int i = 0; i < n; i += kMaxSegs) {
        ReportArgs r{};
        r.n = std::min(kMaxSegs, n - i);
        std::copy(ranges + i, ranges + i + r.n, r.seg);
        hipLaunchKernelGGL(report_ranges, dim3((r.n + 255) / 256), dim3(256), 0, s, r, cnt_dn, ok_host + i, dtype, H, ksplit);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_clear_words(int32_t *p, long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<long>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(clear_words, dim3(blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

template <bool BF16, int KS>
static void launch_combine_ks(const CombineArgs &a, hipStream_t s) {
    // A token's chunks go to workgroups of their own only where the tokens alone are too few for the chip: beyond that
    // a workgroup's start costs more than it hides.  Us without / with such a split: 64 tokens x top-2, H 4096,
    // 4 K ranges 5.8 / 3.0; 512 tokens, 2 K ranges 6.3 / 6.2; 1024 tokens, top-1 6.5 / 6.9; 2048 x top-8, H 2048
    // 26.3 / 29.1; 3584 x top-2, H 4096 27.0 / 26.6; 8192 x top-1 38.1 / 44.8; 8192 x top-8, H 2048 102.7 / 106.5.
    const int chunks = a.H % 4 == 0 ? (a.H + 1023) / 1024 : (a.H + 255) / 256;
    hipLaunchKernelGGL((combine_rows<BF16, KS>), dim3(a.N, std::min(chunks, std::max(1, 2048 / a.N))), dim3(256), 0, s, a.out,
                       a.plane, a.topk_w, a.inv, a.cls, a.done, a.complete, a.y, a.H, a.k, a.class_mask);
}

hipError_t launch_combine(const CombineArgs &a, hipStream_t s) {
    if (a.N <= 0) return hipSuccess;
    const bool bf = a.dtype == MOE_BF16;
    if (a.ksplit == 4) { if (bf) launch_combine_ks<true, 4>(a, s); else launch_combine_ks<false, 4>(a, s); }
    else if (a.ksplit == 2) { if (bf) launch_combine_ks<true, 2>(a, s); else launch_combine_ks<false, 2>(a, s); }
    else { if (bf) launch_combine_ks<true, 1>(a, s); else launch_combine_ks<false, 1>(a, s); }
    return hipGetLastError();
}

hipError_t launch_clear_done(uint8_t *done, long n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<long>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(clear_bytes, dim3(blocks), dim3(256), 0, s, done, n);
    return hipGetLastError();
}

hipError_t launch_mark_done(const Seg *segs, int n, uint8_t *done, hipStream_t s) {
    for (int i = 0; i < n; i += kMaxSegs) {
        MarkArgs m{};
        m.n = std::min(kMaxSegs, n - i);
        std::copy(segs + i, segs + i + m.n, m.seg);
        hipLaunchKernelGGL(mark_rows, dim3(m.n), dim3(256), 0, s, m, done);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qmoe
