// fp32 expert kernels on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation),
// SwiGLU fused into the gate-up epilogue.
//
// Bound: the fp32 MFMA rate (256 FLOP per clock and CU, 157 TFLOP/s on the chip at 2.4 GHz).  A
// workgroup takes 32 token rows x 32 output columns; each of its 4 waves a 16 x 16 tile of them (gate-up:
// one of W1 and the same one of W3, so a gate and its up value meet in one lane).  Tiles this small
// because fp32 MFMAs are slow against LDS and L2 (24 bytes per clock and CU from L2, a third of what it
// gives): they cost no bandwidth, leave 5 and more workgroups on every CU to cover each other's barriers,
// and even out ragged units (64 x 64 tiles: 93 / 76 us where these take 98 / 57).
// Both operands go through LDS in rows of 32 k (128 bytes, 16-byte slots XOR-swizzled by row), two
// stages, global loads D iterations ahead in a register ring.  Rows need only 4-byte alignment (H and F
// are arbitrary here), the loads are 16 bytes wide all the same.
// A K that is no multiple of 32 has its remainder done FIRST, zero-padded, by guarded loads of the
// prologue: the main loop then has no guards and no exposed last load.
// Each output is one accumulation chain over K in an order that K alone fixes: results do not
// depend on the segment or tile a row sits in.
// Measured on 509 tokens x 8 experts, top-2, H 1024, F 2048 (gate-up / down): 409 / 369 us as 64x64 FMA
// tiles with scalar loads, 98 / 56 us here (MFMA pipe 67 % / 53 % busy); 64 tokens x 4 experts, H 128, F 256:
// 26 / 33 us, 5 / 5 us here.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "experts_common.h"

namespace qmoe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte load from a 4-byte aligned row

constexpr int BM = kF32RowTile, BN = kF32ColTile, BK = 32;
static_assert(BM == 32 && BN == 32, "2 x 2 waves of 16 x 16 tiles");

__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

struct FArgs {
    KArgs k;
    int row_tiles;       // row tiles of the longest segment
    int nseg;            // > 0: work on seg[0..nseg); 0: on units[u0 .. u0+nu) of the device list
    Seg seg[kMaxSegs];
};

// The K loop of one workgroup.  TB: 16-column tiles per wave (2 = gate and up, 1 = down); D: iterations
// between a load and its use.
template <int TB, int D>
struct Loop {
    static constexpr int AR = BM / 32, BR = TB * BN / 32;      // staged rows per thread: 256 threads = 32 rows x 8 slots
    static constexpr int STAGE = (BM + TB * BN) * 128;
    const float *ap[AR], *bp[BR];
    char *lds;
    int tid, w, l;
    f32x4 reg[D][AR + BR];
    f32x4 acc[TB];

    template <int S> __device__ __forceinline__ void load(long k) {
#pragma unroll
        for (int j = 0; j < AR; ++j) reg[S][j] = *reinterpret_cast<const f32x4u *>(ap[j] + k);
#pragma unroll
        for (int j = 0; j < BR; ++j) reg[S][AR + j] = *reinterpret_cast<const f32x4u *>(bp[j] + k);
    }
    // elements k .. k+3 of the slot, zero from K on (kl: this thread's first k)
    template <int S> __device__ __forceinline__ void load_tail(int k, int kl, int K) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool ok = k + kl + i < K;
#pragma unroll
            for (int j = 0; j < AR; ++j) reg[S][j][i] = ok ? ap[j][k + i] : 0.f;
#pragma unroll
            for (int j = 0; j < BR; ++j) reg[S][AR + j][i] = ok ? bp[j][k + i] : 0.f;
        }
    }
    template <int S> __device__ __forceinline__ void store(int stage) {
        const int r0 = tid >> 3, slot = tid & 7;
#pragma unroll
        for (int j = 0; j < AR + BR; ++j) {
            const int r = r0 + 32 * j;
            *reinterpret_cast<f32x4 *>(lds + stage * STAGE + (r * 8 + (slot ^ swz(r))) * 16) = reg[S][j];
        }
    }
    __device__ __forceinline__ f32x4 frag(int stage, int r, int slot) const {
        return *reinterpret_cast<const f32x4 *>(lds + stage * STAGE + (r * 8 + (slot ^ swz(r))) * 16);
    }
    // 32 k of one stage.  A lane reads 4 consecutive k of its row at once; MFMA step s takes element s of
    // every lane, i.e. k = {s, 4+s, 8+s, 12+s} of the 16-k group: any order of k does, it is always this one.
    __device__ __forceinline__ void compute(int stage) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int slot = g * 4 + (l >> 4);
            const f32x4 a = frag(stage, (w & 1) * 16 + (l & 15), slot);
            f32x4 b[TB];
#pragma unroll
            for (int n = 0; n < TB; ++n) b[n] = frag(stage, BM + n * BN + (w >> 1) * 16 + (l & 15), slot);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int n = 0; n < TB; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[n][s], acc[n], 0, 0, 0);
        }
    }
    // Tiles 0 .. n-1 of the sequence; the first is the guarded remainder if K % 32.
    __device__ __forceinline__ void run(int K) {
#pragma unroll
        for (int n = 0; n < TB; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int full = K / BK, rem = K - full * BK;
        const int lead = rem ? 1 : 0, n = full + lead;
        const int last = full - 1;
        // k of tile t of the sequence, clamped to the last full tile
        auto koff = [&](int t) { return (long)min(t - lead, last) * BK; };
        if (rem) load_tail<0>(full * BK, (tid & 7) * 4, K);
        else load<0>(0);
        if (full == 0) {
            store<0>(0);
            __syncthreads();
            compute(0);
            return;
        }
        store<0>(0);
        // set S holds tile t with t % D == S; tile 0 is in LDS already
        if constexpr (D > 1) load<1 % D>(koff(1));
        if constexpr (D > 2) load<2 % D>(koff(2));
        if constexpr (D > 3) load<3 % D>(koff(3));
        __syncthreads();
        int t = 0;
        for (; t + D <= n; t += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) body(t + i, i, koff(t + i + D));
        }
#pragma unroll
        for (int i = 0; i < D - 1; ++i)
            if (t + i < n) body(t + i, i, koff(t + i + D));
    }
    // tile t at ring position i: request tile t+D into the set that tile t has left, compute, hand tile
    // t+1 to LDS
    __device__ __forceinline__ void body(int t, int i, long k) {
        static_assert(D == 2 || D == 4, "ring of 2 or 4 sets");
        if (i == 0) load<0>(k);
        if (i == 1) load<1 % D>(k);
        if (i == 2) load<2 % D>(k);
        if (i == 3) load<3 % D>(k);
        compute(t & 1);
        const int st = (t + 1) & 1;
        if (i == 0) store<1 % D>(st);
        if (i == 1) store<2 % D>(st);
        if (i == 2) store<3 % D>(st);
        if (i == 3) store<0>(st);
        __syncthreads();
    }
};

template <bool GATEUP>
__device__ __forceinline__ void expert_rows(const KArgs &p, const moe_unit &un, int r0, int ct, char *lds) {
    constexpr int TB = GATEUP ? 2 : 1;
    Loop<TB, GATEUP ? 2 : 4> L;
    L.lds = lds; L.tid = threadIdx.x; L.w = __builtin_amdgcn_readfirstlane(L.tid >> 6); L.l = L.tid & 63;
    const int wr0 = r0 + (L.w & 1) * 16;                         // first row of this wave
    const float *b0 = (const float *)p.b0 + (long)un.expert * p.b_estride;
    const float *b1 = GATEUP ? (const float *)p.b1 + (long)un.expert * p.b_estride : b0;
    const int srow = L.tid >> 3, sk = (L.tid & 7) * 4;
#pragma unroll
    for (int j = 0; j < L.AR; ++j) {
        const int r = min(r0 + srow + 32 * j, un.rows - 1);      // rows beyond the unit repeat its last one; they are not stored
        const long src = GATEUP ? (long)(p.perm[un.row0 + r] / p.kdiv) : (long)(un.row0 + r);
        L.ap[j] = (const float *)p.a_src + src * p.lda + sk;
    }
    const long c = min(ct * BN + srow, p.ncols - 1);
    L.bp[0] = b0 + c * p.K + sk;
    if (GATEUP) L.bp[TB - 1] = b1 + c * p.K + sk;
    L.run(p.K);
    // D register i of lane l: token row 4*(l/16) + i, column l%16
    const int col = ct * BN + (L.w >> 1) * 16 + (L.l & 15);
    if (col >= p.ncols) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = wr0 + 4 * (L.l >> 4) + i;
        if (r >= un.rows) continue;
        float *d = (float *)p.dst + (long)(un.row0 + r) * p.ldd + col;
        const float g = L.acc[0][i];
        if (GATEUP) *d = (g / (1.f + expf(-g))) * L.acc[TB - 1][i];
        else *d = g;
    }
}

template <bool GATEUP>
__global__ __launch_bounds__(256) void expert_f32(const FArgs f) {
    __shared__ int s_run;
    __shared__ __attribute__((aligned(16))) char lds[2 * (BM + (GATEUP ? 2 : 1) * BN) * 128];
    const KArgs &p = f.k;
    int bid = blockIdx.x;
    const int ct = bid % p.col_tiles; bid /= p.col_tiles;
    const int rt = bid % f.row_tiles;
    const int ui = bid / f.row_tiles;
    moe_unit un;
    if (f.nseg > 0) {
        const Seg g = f.seg[ui];
        un.expert = g.expert; un.cls = 0; un.row0 = (int)g.row0; un.rows = g.rows;
    } else {
        un = p.units[p.u0 + ui];
    }
    const int r0 = rt * BM;
    if (r0 >= un.rows) return;
    if (!wg_may_run(p, un.row0, (un.rows + BM - 1) / BM, &s_run)) return;
    expert_rows<GATEUP>(p, un, r0, ct, lds);
}

}  // namespace

// One kernel over all n segments or units of f, in launches of as many as one can hold.
template <bool GATEUP>
static void launch_f32(FArgs &f, const Seg *segs, unsigned n, hipStream_t s) {
    const unsigned u0 = f.k.u0, wgs = (unsigned)f.row_tiles * (unsigned)f.k.col_tiles, most = segs_per_launch(wgs);
    for (unsigned at = 0; at < n; at += std::min(most, n - at)) {
        const unsigned cnt = std::min(most, n - at);
        if (segs) {
            f.nseg = (int)cnt;
            std::copy(segs + at, segs + at + cnt, f.seg);
        } else {
            f.k.u0 = u0 + at;
        }
        hipLaunchKernelGGL(expert_f32<GATEUP>, dim3(cnt * wgs), dim3(256), 0, s, f);
    }
}

void launch_experts_f32(const ExpertArgs &a, const KArgs &gu_in, const KArgs &dn_in, hipStream_t s) {
    FArgs f{};
    const unsigned n = a.segs ? (unsigned)a.nseg : a.nu;
    f.row_tiles = (a.max_rows + BM - 1) / BM;
    const int gu_cols = (a.F + BN - 1) / BN, dn_cols = (a.H + BN - 1) / BN;
    f.k = gu_in;
    f.k.col_tiles = gu_cols;
    { Scope sc(a.prof, MOE_PROF_GATE_UP, s); launch_f32<true>(f, a.segs, n, s); }
    f.k = dn_in;
    f.k.col_tiles = dn_cols;
    f.k.need = gu_cols;              // gate-up workgroups per row tile
    { Scope sc(a.prof, MOE_PROF_DOWN, s); launch_f32<false>(f, a.segs, n, s); }
}

}  // namespace qmoe
