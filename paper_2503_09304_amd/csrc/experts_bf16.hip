// bf16 expert path: launch dispatch, the plane reduction of the K-split down projection, and the
// weight re-layout kernel.  The GEMM kernels themselves are the templates of experts_bf16_tile.h.
#include "experts_bf16_tile.h"

namespace qmoe {
namespace {

using bf16k::BArgs;
using bf16k::f32x4;

// out[r,:] = ((p0 + p1) + p2) + p3 (or p0 + p1 with two planes) for the rows of the segments.
struct ReduceArgs {
    int nseg;
    Seg seg[kMaxSegs];
};

__global__ __launch_bounds__(256) void reduce_planes(const ReduceArgs b, const float *__restrict__ part, float *__restrict__ out,
                                                     int H, int ksplit, long plane) {
    const Seg g = b.seg[blockIdx.y];
    const int per_row = H >> 2;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < (long)g.rows * per_row; i += (long)gridDim.x * 256) {
        const long off = ((long)g.row0 * H) + i * 4;
        const f32x4 a = *reinterpret_cast<const f32x4 *>(part + off);
        const f32x4 p1 = *reinterpret_cast<const f32x4 *>(part + plane + off);
        f32x4 v;
        if (ksplit == 4) {
            const f32x4 p2 = *reinterpret_cast<const f32x4 *>(part + 2 * plane + off);
            const f32x4 p3 = *reinterpret_cast<const f32x4 *>(part + 3 * plane + off);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = ((a[q] + p1[q]) + p2[q]) + p3[q];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = a[q] + p1[q];
        }
        *reinterpret_cast<f32x4 *>(out + off) = v;
    }
}

// Re-layout of [E][R][K] row-major bf16 into the packed block order: one thread per 16-byte piece.
__global__ __launch_bounds__(256) void pack_weights_bf16(const uint4 *__restrict__ src, uint4 *__restrict__ dst, long pieces,
                                                         int R, int K) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;   // destination piece index
    if (i >= pieces) return;
    const long per_expert = (long)R * K / 8;
    const long e = i / per_expert, q = i - e * per_expert;
    const int lane = (int)(q & 63);
    const long blk = q >> 6;                                // nt * (K/16) + kstep
    const int ksteps = K / 16;
    const long nt = blk / ksteps;
    const int ks = (int)(blk - nt * ksteps);
    const long r = nt * 32 + (lane & 31);
    const int k = ks * 16 + (lane >> 5) * 8;
    dst[i] = src[(e * R + r) * (K / 8) + k / 8];
}

// Re-layout of 4-bit weights: one thread per 16-byte piece of the destination (expert, row tile,
// iteration, lane); lanes of the lower k-half also write their row's two scale bytes.
__global__ __launch_bounds__(256) void pack_weights_mxfp4(const uint8_t *__restrict__ codes, const uint8_t *__restrict__ scales,
                                                          uint4 *__restrict__ dcodes, uint16_t *__restrict__ dscales,
                                                          long pieces, int R, int K) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= pieces) return;
    const int lane = (int)(i & 63);
    const long blk = i >> 6;                                // (e * R/32 + nt) * K/64 + it
    const int kb = K >> 6;
    const int it = (int)(blk % kb);
    const long row_tile = blk / kb;                         // e * R/32 + nt
    const long row = row_tile * 32 + (lane & 31);           // e * R + r
    const int lh = lane >> 5;
    const uint8_t *src = codes + (row * K + it * 64 + lh * 8) / 2;
    uint4 v;
    v.x = *reinterpret_cast<const uint32_t *>(src);
    v.y = *reinterpret_cast<const uint32_t *>(src + 8);
    v.z = *reinterpret_cast<const uint32_t *>(src + 16);
    v.w = *reinterpret_cast<const uint32_t *>(src + 24);
    dcodes[i] = v;
    if (lh == 0) {
        const uint8_t *sp = scales + row * (K >> 5) + it * 2;
        dscales[blk * 32 + lane] = (uint16_t)(sp[0] | (sp[1] << 8));
    }
}

}  // namespace

hipError_t launch_reduce_planes(const Seg *segs, int nseg, const float *partial, float *out, int H, int ksplit, long plane,
                                hipStream_t s) {
    for (int i = 0; i < nseg; i += kMaxSegs) {
        ReduceArgs r{};
        r.nseg = std::min(kMaxSegs, nseg - i);
        int max_rows = 1;
        for (int j = 0; j < r.nseg; ++j) { r.seg[j] = segs[i + j]; max_rows = std::max(max_rows, (int)segs[i + j].rows); }
        const int per_seg = std::max(1, std::min(64, (max_rows * (H / 4) + 255) / 256));
        hipLaunchKernelGGL(reduce_planes, dim3(per_seg, r.nseg), dim3(256), 0, s, r, partial, out, H, ksplit, plane);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_pack_mxfp4(const void *codes, const void *scales, void *dcodes, void *dscales, int E, int R, int K,
                             hipStream_t s) {
    const long pieces = (long)E * (R / 32) * (K / 64) * 64;
    hipLaunchKernelGGL(pack_weights_mxfp4, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, (const uint8_t *)codes,
                       (const uint8_t *)scales, (uint4 *)dcodes, (uint16_t *)dscales, pieces, R, K);
    return hipGetLastError();
}

hipError_t launch_pack(const void *src, void *dst, int E, int R, int K, hipStream_t s) {
    const long pieces = (long)E * R * K / 8;
    hipLaunchKernelGGL(pack_weights_bf16, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, (const uint4 *)src,
                       (uint4 *)dst, pieces, R, K);
    return hipGetLastError();
}

static long cu_count() {
    static const long cus = [] {       // (once, by whichever thread launches first)
        int dev = 0, v = 0;
        return hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1 ? 256 : v;
    }();
    return cus;
}

void launch_experts_bf16(const ExpertArgs &a, const KArgs &gu_in, const KArgs &dn_in, hipStream_t s) {
    BArgs b{};
    b.ksplit = 1;
    b.plane = 0;
    b.nseg = a.segs ? a.nseg : 0;
    const bool stream = b.nseg > 0 && items_stream(a.segs, b.nseg);
    const int tiles = (a.max_rows + 31) / 32;
    const unsigned n = b.nseg > 0 ? (unsigned)b.nseg : a.nu;
    b.k = gu_in;
    b.k.cw = a.wave_cols ? a.wave_cols : gate_up_wave_columns(stream, a.wfmt, tiles, (int)n, a.F, cu_count());
    // A lane's place in a packed row tile is a 32-bit offset from the tile of the wave's first row (64 * H bytes each): rows so
    // long keep waves of 32 columns, which lie in one tile.
    if (a.H >= 1 << 26) b.k.cw = 32;
    b.k.col_tiles = (a.F + 4 * b.k.cw - 1) / (4 * b.k.cw);
    auto launch_one = [&](bool gateup) {
        using namespace bf16k;
        if (a.wfmt == WF_MXFP4) gateup ? launch_expert_kernel<WF_MXFP4, true>(tiles, stream, b, s) : launch_expert_kernel<WF_MXFP4, false>(tiles, stream, b, s);
        else if (a.wfmt == WF_PACKED) gateup ? launch_expert_kernel<WF_PACKED, true>(tiles, stream, b, s) : launch_expert_kernel<WF_PACKED, false>(tiles, stream, b, s);
        else gateup ? launch_expert_kernel<WF_ROWMAJOR, true>(tiles, stream, b, s) : launch_expert_kernel<WF_ROWMAJOR, false>(tiles, stream, b, s);
    };
    bool dealt = false;
    auto launch = [&](bool gateup) {
        // segments in the arguments are one launch, a range of the unit list as many as it takes
        const unsigned cols = (unsigned)(b.k.col_tiles * b.ksplit);
        if (b.nseg > 0 && (gateup || !stream))       // the order of a launch that streams does not depend on its columns
            dealt = plan_items(a.segs, b.nseg, stream, cols, a.wfmt == bf16k::WF_MXFP4, b.seg, b.xcd);
        const unsigned most = b.nseg > 0 ? n : segs_per_launch(cols);
        for (unsigned at = 0; at < n; at += (unsigned)b.k.nu) {
            b.k.u0 = a.u0 + at;
            b.k.nu = (int)std::min(most, n - at);
            b.items = dealt ? 0 : (unsigned)b.k.nu * cols;
            launch_one(gateup);
        }
    };
    { Scope sc(a.prof, MOE_PROF_GATE_UP, s); launch(true); }

    const int gu_col_tiles = b.k.col_tiles;
    b.k = dn_in;
    b.k.need = gu_col_tiles;         // gate-up workgroups per row range
    b.k.cw = 32;
    b.k.col_tiles = (a.H + 255) / 256;
    if (a.ksplit > 1 && a.partial != nullptr) {
        // the planes stay apart: moe_combine adds them in the fixed order ((p0+p1)+p2)+p3 as it reads them
        b.ksplit = a.ksplit;
        b.plane = a.plane;
        b.k.dst = a.partial;
    }
    // Streaming launches of at most 32 rows a segment in 128 columns a workgroup, where the twice as many workgroups take less than twice
    // the whole rounds of the CUs (a round of half the columns takes about half the time).  Us, 256 / 128 columns (workgroups):
    // one token on 8 experts (128 / 256) 46.7 / 39.7, 32 tokens on 64 experts, skewed (304 / 608: 2 rounds / 3) 47.4 / 42.7; not:
    // two tokens on 8 experts (192 / 384) 56.3 / 60.6, 8 on 64 (about 184 / 368) 26.3 / 28.8, 32 on 64 (504 / 1008)
    // 59.1 / 59.7, 16 on 8, 4-bit (512 / 1024) 40.5 / 42.7.  Stoppable launches count workgroups of 256 columns.
    if (stream && tiles == 1 && a.go == nullptr) {
        auto rounds = [&](int cols) { return ((long)n * ((a.H + cols - 1) / cols) * b.ksplit + cu_count() - 1) / cu_count(); };
        b.narrow = rounds(128) < 2 * rounds(256);
        if (b.narrow) b.k.col_tiles = (a.H + 127) / 128;
    }
    { Scope sc(a.prof, MOE_PROF_DOWN, s); launch(false); }
}

}  // namespace qmoe
