// bf16 expert kernels (gate-up with fused SwiGLU, and down projection) on MFMA: the templates.
// Included by experts_bf16.hip (dispatch) and by experts_bf16_w<WF>_<kernel>.hip (one instantiation per weight
// format and kernel).
//
// All three weight matrices are [rows_out, K] with K contiguous, and so are the activations, so
// both MFMA operands are read 8 consecutive K-elements (16 bytes) per lane with no transposition.
// v_mfma_f32_16x16x32_bf16: A = 16 weight rows x 32 k, B = 16 tokens x 32 k, D[weight row, token]
// in fp32.  A workgroup has 4 waves.  Each wave owns 64 weight rows (gate-up: 32 rows of W1 and the
// same 32 of W3, so the gate and up value of one (token, f) meet in one lane and register) and every
// 16-token fragment of the unit.  No two waves use the same weight fragment, so weights go straight from
// global memory into MFMA operand registers (with the packed layout a wave load is a contiguous KiB or four runs
// of 256 bytes); only the token tile (gathered x rows, or act rows), which all 4 waves share, is
// staged in LDS, double-buffered, its 16-byte slots XOR-swizzled by row so that the 16 rows read
// by one ds_read_b128 pass fall into distinct banks.
//
// Why 16x16x32.  From about 150 rows an expert on these kernels run at the clock that the power limit leaves
// them, so what counts is energy per flop: on random operands a loop of nothing but MFMAs sustains 2.00-2.06
// PFLOP/s with 16x16x32 and 1.79-1.82 with 32x32x16.  Fragments of 16 tokens also leave less padding than tiles of 32.  Against
// the same kernel on 32x32x16 (us, gate-up / down): 3584 tokens on 8 experts, H 4096, F 14336 1353 / 711 and 1255 / 682,
// with 4-bit weights 1329 / 628 and 1229 / 579; 8192 tokens on 64 experts, H 2048, F 1408 657 / 422 and 613 / 401; 512
// tokens on 8 experts with row-major weights, where a lane's rows now come 64 contiguous bytes at a time, 816 / 382 and 510 / 256.
//
// Pipeline of one K-iteration (64 k), prefetch distance D: issue the global loads of the token
// pieces and weight fragments for it+D (register rings of D+1 sets), run the MFMAs of iteration it,
// write the token tile for it+1 into the other LDS stage, one barrier.  Vector loads complete in
// issue order, so the waits leave about D iterations of weight loads (8 KB per wave each) in flight.
// Loads are unconditional (row and iteration indices are clamped instead) so that the wait counters
// stay exact.
//
// Down projection with K-split (a property of the context's configuration: weight-streaming shapes
// have too few output tiles to fill the chip): K is cut into 2 or 4 contiguous ranges, each computed
// by its own workgroup into a partial plane; a second kernel adds the planes in the fixed order
// ((p0+p1)+p2)+p3.
//
// A launch works on row segments: the host joins the row-adjacent units of one expert in a call (the
// LS and BE part of its queue, consecutive chunks) and cuts each such run into segments of at most 256
// rows, equal within a tile of 32 rows or a fragment of 16 (cut_runs), so that one pass over the weights serves them and workgroups
// that share weight tiles keep the same pace.
//
// Determinism.  Each output element is one chain of MFMA accumulations over K in ascending order
// (K-split: 2 or 4 chains added in a fixed order), the same for every row of the context: it depends on
// neither the tile a row sits in, nor the rows that share it, nor the weight layout.  Results are
// therefore bit-identical however the unit list is split into launches.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "expert_items.h"
#include "experts_common.h"

namespace qmoe {
namespace bf16k {

// Smallest number of 32-row pieces whose variant keeps three LDS stages (see P3 in expert_tile).
constexpr int kP3MinT = 3;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// silu(z) = z / (1 + e^-z) as one exponential and one reciprocal (v_exp_f32, v_rcp_f32: about 1 ulp
// each, far below the bf16 rounding the product gets next).  An IEEE division costs three times the
// instructions, and a workgroup's epilogue applies this to T*32 x 128 values while its MFMA pipes idle.
__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

// LDS layout of the token tile: rows of 128 bytes = 8 slots of 16 bytes; slot s of row r is stored
// at slot s ^ swz(r).  swz is a permutation of 0..7 over any 8 consecutive rows, and over 16
// consecutive rows the pairs (row parity, swz) are all distinct: the 8 or 16 lanes of one
// ds_read_b128 / ds_write_b128 pass hit distinct banks whether a pass spans 128 or 256 bytes.
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>).  Register
// arrays are only ever indexed with these constants, so they stay in registers.
template <int N, class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// acc += weights x tokens (16 weight rows x 16 tokens x 32 k).  In assembly so that an accumulator stays
// in its place: given the builtin, the compiler writes 16 x 16 results to other registers than it read them from and
// moves them back (428 moves per 336 MFMAs with 7 token tiles).  It does not see the matrix unit's hazards here: a vector
// instruction that writes an operand must stand two wait states before (the operands come from loads; swaps are followed by
// such a wait, the conversions of 4-bit weights stand slots before), and after the last MFMA of an iteration eight wait states keep anything else off the accumulators.
template <bool LAST>
__device__ __forceinline__ void mma(f32x4 &c, const bf16x8 &w, const bf16x8 &x) {
    if constexpr (LAST) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 7" : "+a"(c) : "v"(w), "v"(x));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}

// Pointers into global memory, said to be so: the compiler gives up tracing the larger kernels' pointers back to the
// arguments and takes loads that may go to LDS too, which wait for one another (gate-up at half its speed).
typedef const __attribute__((address_space(1))) char *gchar;
template <class V>
__device__ __forceinline__ V gload(gchar p) { return *reinterpret_cast<const __attribute__((address_space(1))) V *>(p); }
template <class V>
__device__ __forceinline__ V gload_nt(gchar p) { return __builtin_nontemporal_load(reinterpret_cast<const __attribute__((address_space(1))) V *>(p)); }
template <class V>
__device__ __forceinline__ void gstore_nt(const V &v, void *p) { __builtin_nontemporal_store(v, (__attribute__((address_space(1))) V *)p); }

// Launch-local arguments of the bf16 kernels.
struct BArgs {
    KArgs k;
    int ksplit;          // 1, or 2 or 4: K ranges, one workgroup each, partial planes in k.dst
    long plane;          // elements between partial planes
    int narrow;          // down projection in the narrow form
    int nseg;            // > 0: work on seg[0..nseg); 0: on units[u0 .. u0+nu) of the device list
    unsigned items;      // (segments or units) x column tiles x K ranges of a list; 0: XCD x works on seg[xcd[x]..xcd[x+1])
    uint32_t xcd[kXcds + 1];
    ItemSeg seg[kMaxSegs];
};

// One (unit, column tile, K range) on a workgroup.
// NM: 32-row matrices per wave (gate-up: W1, W3; down: its 64 rows of W2, or 32 of them in the narrow form).
template <int NF, bool GATEUP, int WF, bool STREAM, int D, int NM = 2>
__device__ __forceinline__ void expert_tile(const KArgs &p, const moe_unit un, const int ct, const int kq, const int ksplit,
                                            const long plane, char *lds) {
    // Stoppable launches: the workgroup leaves behind the prologue's barrier if the stop word is set or
    // (down projection) the gate-up workgroups of its rows did not all run.
    __shared__ int s_run;
    constexpr int T = (NF + 1) / 2;        // 32-row pieces of the token tile that a thread stages
    constexpr int ROWS = T * 32;
    constexpr int STAGE = ROWS * 128;      // bytes of one LDS stage: 64 bf16 per row
    // The variants of more than 64 rows keep three token-tile stages, write tile it+2 during
    // iteration it, and so may read the first fragments of tile it+1 before the iteration's barrier;
    // the LDS latency after the barrier disappears from the MFMA stream.  Gate-up / down us with two stages everywhere, three
    // from 129 rows on, three from 65 on, top-2 of 8 experts, H 4096, F 14336: 3584 tokens 1354 / 706, 1339 / 702, 1332 / 696; 512 tokens
    // 337 / 163, 333 / 161, 331 / 159; 350 tokens all alike.  Below, an iteration is bound by the weight stream alone.
    constexpr bool P3 = T >= kP3MinT;
    // Output columns per wave.  Gate-up: 32, or fewer (p.cw, a multiple of 4) on launches whose
    // workgroup count would otherwise end in a partly filled round of the chip; the wave's MFMA rows
    // beyond p.cw repeat its last weight row and are dropped in the epilogue.
    const int cpw = GATEUP ? p.cw : 32 * NM;
    const int rows = un.rows;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int lr = l & 15, lg = l >> 4;
    const int Kg = p.K / ksplit;           // this workgroup's K range: [kq*Kg, (kq+1)*Kg)
    const int iters = Kg / 64;
    const int col_base = ct * (4 * cpw) + w * cpw;

    // ---- weight rows of this lane ----
    // A wave has two matrices of 32 rows (gate-up: W1, W3; down: the two halves of its 64 rows of W2), each in two row
    // halves of 16 (rt).  Of an iteration's 64 k, eight pieces of 8, MFMA step j (0, 1) takes for lane group lg piece
    // 4j + 2*(lg%2) + lg/2, tokens and weights alike: any order does, and this one is a single swap of lane groups away
    // from the 4-bit blocks (see dequant_piece).
    // A load = uniform base of the matrix + the lane's 32-bit offset + constants.
    // Row-major: 16 bytes of the lane's row, pieces 2j apart 32 bytes.
    // Packed: the 1 KiB block of k-step s of row tile nt starts at (nt*(K/16)+s)*1024 bytes; pieces (s, half) of the
    // 32 rows lie 512 bytes apart: a load is four runs of 256 bytes.
    // MXFP4: per (row tile, iteration) one KiB of codes (lane l: 16 bytes, the words of row l%32's k half l/32 in each of
    // the 4 k-steps) and 64 bytes of scales (row l%32: the two e8m0 bytes of the iteration's two 32-element blocks).
    constexpr bool PACKED = WF == WF_PACKED;
    constexpr bool MX = WF == WF_MXFP4;
    // Gate-up launches that may have waves of fewer than 32 columns read the packed blocks whole (row l%32, half l/32) and
    // swap lane groups into place: a wave's rows then start anywhere in a row tile, and loads of 16 rows would ask for
    // the lines at their edges twice (64 tokens on 8 experts, 28 columns: 302 us with such loads, 293 so).
    constexpr bool SWAP = PACKED && STREAM && GATEUP && NF <= 6;
    constexpr int BJ = PACKED ? 2048 : 64;      // bytes between the two MFMA steps
    constexpr int BIT = PACKED ? 4096 : (MX ? 1024 : 128);   // bytes between iterations (MXFP4: of codes)
    gchar bbase[2], sbase[2];                   // the matrices (MXFP4: codes and scales), at this workgroup's K range
    // Row-major rows lie 2*K bytes apart, and 64 of them pass 4 GiB from K of 34 million on.
    std::conditional_t<WF == WF_ROWMAJOR, unsigned long, unsigned> boff[2][2];      // [matrix][row half]; MXFP4: [matrix][0], one load for both halves
    unsigned soff[2];
    {
        gchar e0 = (gchar)p.b0, e1 = GATEUP ? (gchar)p.b1 : e0;
        const long ebytes = MX ? p.b_estride >> 1 : p.b_estride * 2;
        e0 += un.expert * ebytes; e1 += un.expert * ebytes;
        const int ntiles = p.ncols >> 5;
        const int first = min(col_base, p.ncols - 1);          // rows from p.ncols on repeat the last one
        const int lane_piece = PACKED ? (lg & 1) * 1024 + (lg >> 1) * 512 : (lg & 1) * 32 + (lg >> 1) * 16;
        const long kblocks = p.K >> 6, tile_bytes = kblocks * BIT;                  // packed formats: one row tile
        const long k0 = (long)kq * (Kg >> 6) * BIT;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            gchar e = n ? e1 : e0;
            const int nt = GATEUP ? first >> 5 : min((col_base >> 5) + n, ntiles - 1);
            if constexpr (PACKED || MX) bbase[n] = e + nt * tile_bytes + k0;
            else bbase[n] = e + (long)first * p.K * 2 + k0;
            if constexpr (MX) {
                gchar s = (gchar)(GATEUP && n ? p.s1 : p.s0) + un.expert * (p.b_estride >> 5);
                sbase[n] = s + (nt * kblocks + (long)kq * (Kg >> 6)) * 64;
            } else sbase[n] = nullptr;
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                const int r = MX || SWAP ? l & 31 : rt * 16 + lr;
                const int row = GATEUP ? min(col_base + min(r, cpw - 1), p.ncols - 1) : (PACKED || MX ? r : min(col_base + n * 32 + r, p.ncols - 1));
                const unsigned t = GATEUP ? (unsigned)((row >> 5) - nt) : 0u;      // the row may lie in the next row tile (fewer than 32 columns a wave)
                if constexpr (MX) {
                    boff[n][rt] = t * (unsigned)tile_bytes + (unsigned)(((l >> 5) * 32 + (row & 31)) * 16);
                    soff[n] = t * (unsigned)(kblocks * 64) + (unsigned)((row & 31) * 2);
                } else if constexpr (SWAP) {
                    boff[n][rt] = t * (unsigned)tile_bytes + (unsigned)(rt * 1024 + ((l >> 5) * 32 + (row & 31)) * 16);
                } else if constexpr (PACKED) {
                    boff[n][rt] = t * (unsigned)tile_bytes + (unsigned)(lane_piece + (row & 31) * 16);
                } else {
                    boff[n][rt] = (unsigned long)(row - first) * ((unsigned long)p.K * 2) + (unsigned)lane_piece;
                }
            }
        }
    }
    // ---- token rows this thread stages into LDS (A operand): row tid/8 + 32*j, slot tid%8 ----
    const int srow = tid >> 3, sslot = tid & 7;
    // Addressed as a wave-uniform 64-bit base plus a 32-bit offset per row in units of 16 bytes (the
    // host checks that x and act stay below 64 GiB), which halves the registers the row table costs.
    gchar abase = (gchar)p.a_src + ((long)kq * Kg + sslot * 8) * 2;
    unsigned aoff[T];
    static_for<T>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int r = min(srow + 32 * j, rows - 1);
        unsigned src_row;
        if (GATEUP) src_row = (unsigned)(gload<int>((gchar)p.perm + 4l * (un.row0 + r)) / p.kdiv);
        else src_row = (unsigned)(un.row0 + r);
        aoff[j] = src_row * ((unsigned)p.lda >> 3);        // in 16-byte units: lda is a multiple of 64 elements
    });

    constexpr int NQ = 2 * NM;              // (matrix, row half) pairs
    f32x4 acc[NF * NQ];                     // [fragment][matrix][row half]: 4 consecutive weight rows 4*lg .. of token lr
    static_for<NF * NQ>([&](auto tc) { acc[decltype(tc)::value] = f32x4{0.f, 0.f, 0.f, 0.f}; });

    // Register rings: weight fragments of iterations it .. it+D (NB sets), token pieces of
    // it+1 .. it+D (NA sets).  Ring positions are compile-time constants: the loop is unrolled NA*NB.
    // The token pieces, from L2, need no more than 2, and a loop unrolled less: a small launch
    // meets its code cold (unrolled 12 instead of 4 times, one or two fragments: +1 to 2 %).
    constexpr int DA = P3 || D == 2 ? 1 : 2;
    constexpr int NB = D + 1, NA = DA, U = (NB % NA == 0) ? NB : NA * NB;
    u32x4 a_reg[NA * T];
    bf16x8 b_reg[(MX ? 1 : NB) * 2 * NQ];    // [set][step j][matrix][row half]; MXFP4: the operands of the current iteration
    u32x4 c_reg[NB * NM];                // MXFP4: codes [set][matrix]
    unsigned short s_reg[NB * NM];       // MXFP4: the two scale bytes

    // One load (piece j of T, piece i of BL) of iteration `it`, one LDS write of a token piece.
    auto load_a = [&](int it, auto setc, auto jc) {
        constexpr int S = decltype(setc)::value, j = decltype(jc)::value;
        a_reg[S * T + j] = gload<u32x4>(abase + ((unsigned long)(aoff[j] + (unsigned)min(it, iters - 1) * 8u) << 4));
    };
    auto store_a = [&](int stage, auto setc, auto jc) {
        constexpr int S = decltype(setc)::value, j = decltype(jc)::value;
        const int r = srow + 32 * j;
        *reinterpret_cast<u32x4 *>(lds + stage * STAGE + (r * 8 + (sslot ^ swz(r))) * 16) = a_reg[S * T + j];
    };
    auto load_b = [&](int it, auto setc, auto ic) {
        constexpr int S = decltype(setc)::value, i = decltype(ic)::value, q = i % NQ, n = q >> 1, rt = q & 1;
        const long at = (long)min(it, iters - 1) * BIT;
        if constexpr (MX && i >= NM) {
            s_reg[S * NM + i - NM] = gload<unsigned short>(sbase[i - NM] + (at >> 4) + soff[i - NM]);
        } else if constexpr (MX) {
            const gchar from = bbase[i] + at + boff[i][0];
            c_reg[S * NM + i] = STREAM ? gload_nt<u32x4>(from) : gload<u32x4>(from);
        } else {
            const gchar from = bbase[n] + at + boff[n][rt] + (i / NQ) * BJ;
            b_reg[S * 2 * NQ + i] = STREAM ? gload_nt<bf16x8>(from) : gload<bf16x8>(from);
        }
    };
    auto load_a_all = [&](int it, auto setc) { static_for<T>([&](auto jc) { load_a(it, setc, jc); }); };
    auto store_a_all = [&](int stage, auto setc) { static_for<T>([&](auto jc) { store_a(stage, setc, jc); }); };
    constexpr int BL = MX ? 2 * NM : 2 * NQ;       // weight loads of an iteration
    auto load_b_all = [&](int it, auto setc) { static_for<BL>([&](auto ic) { load_b(it, setc, ic); }); };
    // MXFP4: codes and scales of ring set S -> the bf16 operands of (step j, matrix n), both row halves
    // (v_cvt_scalef32_pk_bf16_fp4: two e2m1 nibbles of one byte times a float scale, exact for a power-of-two scale).
    // Lane groups of 16 hold (rows 0-15, half 0), (16-31, 0), (0-15, 1), (16-31, 1) of the k-steps' words; swapping the odd
    // groups of word 2j with the even ones of word 2j + 1 leaves rows 0-15 in the one and rows 16-31 in the other.
    // In kPieces pieces, so that they can be dealt out among MFMAs (see body): the swaps, then two conversions each.
    constexpr int kPieces = 5;
    u32x2 dq_w[NM], dq_s[NM];            // words and scales of a matrix, by row half
    auto dequant_piece = [&](auto setc, auto jc, auto nc, auto pc) {
        constexpr int S = decltype(setc)::value, j = decltype(jc)::value, n = decltype(nc)::value, p = decltype(pc)::value;
        if constexpr (p == 0) {
            dq_w[n] = __builtin_amdgcn_permlane16_swap(c_reg[S * NM + n][2 * j], c_reg[S * NM + n][2 * j + 1], false, false);
            const unsigned sb = ((unsigned)(s_reg[S * NM + n] >> (8 * j)) << 23) & 0x7f800000u;     // (the other byte's bits go)
            dq_s[n] = __builtin_amdgcn_permlane16_swap(sb, sb, false, false);
        } else {
            constexpr int rt = (p - 1) / 2, h = (p - 1) % 2;
            const unsigned sb = dq_s[n][rt];     // (a bit cast of a vector's element itself takes element 0)
            const float f = __builtin_bit_cast(float, sb);
            const bf16x2 e0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(dq_w[n][rt], f, 2 * h);
            const bf16x2 e1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(dq_w[n][rt], f, 2 * h + 1);
            bf16x8 &v = b_reg[j * NQ + n * 2 + rt];
            v[4 * h] = e0[0]; v[4 * h + 1] = e0[1]; v[4 * h + 2] = e1[0]; v[4 * h + 3] = e1[1];
        }
    };
    auto dequant_all = [&](auto setc, auto jc) {
        static_for<NM * kPieces>([&](auto vc) {
            constexpr int v = decltype(vc)::value;
            dequant_piece(setc, jc, std::integral_constant<int, v / kPieces>{}, std::integral_constant<int, v % kPieces>{});
        });
    };

    // One K-iteration is 2*NF slots, written out in the order in which they shall issue (nothing moves across a slot's
    // end): slot s has the 4 MFMAs of one token fragment (step j = s / NF, fragment s % NF; with CHAIN two slots have the 8 of one; its (matrix, row half) pairs in turn
    // upwards and downwards, so that one operand at a time changes between MFMAs: fewer bits toggle, and the clock of the power-limited
    // launches rises; a loop of nothing but MFMAs on random operands 2.06 -> 2.10 PFLOP/s, gate-up of 3584 tokens on 8 experts 1367 -> 1351 us, with
    // 4-bit weights 1251 -> 1238, 8192 tokens on 64 experts 674 -> 667), one LDS fragment read (LA
    // slots before its use), and its share of the T + 8 global loads and of the T LDS writes of the next token tile (last slots).
    // The loads of the four waves keep the texture path busy for about 16 clocks each, 1024 of an iteration's 2048 clocks of MFMA with
    // 256 rows: dealt out over the first half of the slots they queue, and a wave that cannot issue its load issues no MFMA either.
    // With more than 64 rows and bf16 weights they are dealt out over all slots: down projection us with the first half / all, top-2 of
    // 8 experts, H 4096, F 14336: 3584 tokens 694 / 640, 1531 tokens in 4 K ranges 355 / 335, 700 tokens 188 / 184; 8192 tokens on 64 experts
    // 410 / 394; gate-up, at the clock that the power limit leaves, alike within 1 %.  4-bit weights have 4 loads where bf16 has 8, which makes the
    // token pieces arrive too late for their LDS writes (3584 tokens, down 580 / 611); up to 64 rows the stream of weights is the bound.
    // CHAIN: the two steps of an accumulator stand back to back (fragment by fragment, step innermost), so that the matrix unit hands
    // the sum on instead of writing and reading it: a loop of nothing but MFMAs on random operands 2.12 -> 2.21 PFLOP/s (two steps
    // with another accumulator's in between: no gain; four in a row 2.25, but that takes two iterations' operands at a time).
    // 3584 tokens on 8 experts, layer 1912 -> 1890 us, 8192 tokens on 64 experts 1158 -> 1143.  It wants the operands of step 1 half an
    // iteration earlier, so not where the weight stream is the bound (128 tokens on 8 experts, 4 K ranges 540 -> 544 us), and not for 4-bit
    // weights, whose operands of step 1 are made during step 0.  An accumulator's sums run in the same order either way.
    constexpr bool CHAIN = !MX && P3 && !STREAM;
    constexpr int SL = 2 * NF, RF = P3 ? 6 : (SL < 4 ? SL : 4);
    constexpr int LA = CHAIN ? 4 : RF - 1;     // slots read ahead
    static_assert(!P3 || U * SL % RF == 0, "the ring of fragments goes on from iteration to iteration");
    bf16x8 af[RF];
    const char *a_at[2];                    // this lane's piece of step 0 and 1 in a token row
#pragma unroll
    for (int j = 0; j < 2; ++j) a_at[j] = lds + lr * 128 + ((j * 4 + (lg & 1) * 2 + (lg >> 1)) ^ swz(lr)) * 16;
    auto read_af = [&](int stage, auto pc, auto rc) {         // fragment of slot p into place r of the ring
        constexpr int p = decltype(pc)::value, j = CHAIN ? p % 2 : p / NF, f = CHAIN ? p / 2 : p % NF;
        af[decltype(rc)::value] = *reinterpret_cast<const bf16x8 *>(a_at[j] + stage * STAGE + f * 2048);
    };
    auto read_first = [&](int stage) { static_for<LA>([&](auto pc) { read_af(stage, pc, pc); }); };
    // Iteration `it`, position i = it mod U in the unrolled loop: request the operands of it+D (token
    // pieces first: the wait for them must not cover the weight loads), run the MFMAs of it, move the
    // token pieces of it+1 (requested earlier) into the other LDS stage.  Loads complete in issue
    // order, so neither wait disturbs the iterations of weight loads issued after the data waited for.
    auto body = [&](int it, auto ic) {
        constexpr int i = decltype(ic)::value, S = MX ? 0 : i % NB;
        static_assert(!P3 || (NA == 1 && U % 3 == 0), "three stages: one token register set, loop unrolled by a multiple of 3");
        const int stage = P3 ? i % 3 : it & 1, next = P3 ? (i + 1) % 3 : (it + 1) & 1, put = P3 ? (i + 2) % 3 : next;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!P3) read_first(stage);
        if constexpr (SWAP) {
            // blocks 2j and 2j + 1 of a matrix -> its row halves of step j, as in dequant_piece
            static_for<4>([&](auto pc) {
                constexpr int at = S * 2 * NQ + decltype(pc)::value * 2;
                u32x4 x = __builtin_bit_cast(u32x4, b_reg[at]), y = __builtin_bit_cast(u32x4, b_reg[at + 1]);
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const u32x2 v = __builtin_amdgcn_permlane16_swap(x[d], y[d], false, false);
                    x[d] = v[0]; y[d] = v[1];
                }
                b_reg[at] = __builtin_bit_cast(bf16x8, x); b_reg[at + 1] = __builtin_bit_cast(bf16x8, y);
            });
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 1");               // see mma
        }
        static_for<NQ * SL>([&](auto mc) {
            constexpr int m = decltype(mc)::value, s = m / NQ, q = m % NQ;
            constexpr int j = CHAIN ? m % 2 : s / NF, f = CHAIN ? s / 2 : s % NF, qu = CHAIN ? m % (2 * NQ) / 2 : q, qz = f % 2 ? NQ - 1 - qu : qu;
            constexpr int ring = P3 ? i * SL : 0;              // slots before this iteration
            mma<m == NQ * SL - 1>(acc[f * NQ + qz], b_reg[S * 2 * NQ + j * NQ + qz], af[(ring + (CHAIN ? 2 * f + j : s)) % RF]);
            constexpr bool reads = CHAIN ? m % (2 * NQ) < 2 : q == 0;
            constexpr int p = (CHAIN ? 2 * f + m % 2 : s) + LA;
            if constexpr (reads && p < SL) read_af(stage, std::integral_constant<int, p>{}, std::integral_constant<int, (ring + p) % RF>{});
            else if constexpr (reads && P3) read_af(next, std::integral_constant<int, p - SL>{}, std::integral_constant<int, (ring + p) % RF>{});
            constexpr int NV = T + BL, SPAN = P3 && !MX ? NQ * SL : NQ * SL / 2, V0 = m * NV / SPAN, V1 = (m + 1) * NV / SPAN;
            if constexpr (m < SPAN) {
                static_for<V1 - V0>([&](auto vc) {
                    constexpr int v = V0 + decltype(vc)::value;
                    if constexpr (v < T) load_a(it + (P3 ? 2 : DA), std::integral_constant<int, P3 ? 0 : (i + DA) % NA>{}, std::integral_constant<int, v>{});
                    else load_b(it + D, std::integral_constant<int, (i + D) % NB>{}, std::integral_constant<int, v - T>{});
                });
            }
            if constexpr (MX) {
                // The operands of step 1, then those of the next iteration's step 0, their pieces dealt out behind the step's first SP
                // MFMAs (never its last: see mma).  An MFMA of 16 cycles hides three or four vector instructions; a matrix converted in
                // one go behind one MFMA leaves the matrix unit idle where no other wave has MFMAs to issue.  Us in one go / dealt out:
                // 308 tokens on 64 experts, 16 units a launch, 177 / 166; 60 tokens, top-8 of 16, H 1344, F 10816, down projection
                // 83.4 / 77.7; 500 tokens on 8 experts 359 / 345, 3584 tokens 1854 / 1798.  With 4 fragments a step's second half is
                // better left to the LDS writes: that down projection 78.6 with pieces up to the step's end.
                constexpr int set = j == 0 ? i % NB : (i + 1) % NB, t = m - j * NF * NQ, NP = NM * kPieces;
                constexpr int SP = NF == 4 ? NF * NQ / 2 : NF * NQ - 1;
                if constexpr (t < SP) {
                    constexpr int P0 = t * NP / SP, P1 = (t + 1) * NP / SP;
                    static_for<P1 - P0>([&](auto vc) {
                        constexpr int v = P0 + decltype(vc)::value;
                        dequant_piece(std::integral_constant<int, set>{}, std::integral_constant<int, 1 - j>{}, std::integral_constant<int, v / kPieces>{},
                                      std::integral_constant<int, v % kPieces>{});
                    });
                }
            }
            if constexpr (q == NQ - 2 && s >= SL - T) store_a(put, std::integral_constant<int, P3 ? 0 : (i + 1) % NA>{}, std::integral_constant<int, s - (SL - T)>{});
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };

    // prologue: operands of iterations 0 .. D-1; tile 0 into LDS stage 0
    load_a_all(0, std::integral_constant<int, 0>{});
    load_b_all(0, std::integral_constant<int, 0>{});
    const WgProbe probe = wg_probe(p, un.row0);       // (behind the loads that the first stores to LDS wait for)
    store_a_all(0, std::integral_constant<int, 0>{});
    if constexpr (P3) {                      // three stages: tile 1 goes into stage 1 as well
        load_a_all(1, std::integral_constant<int, 0>{});
        store_a_all(1, std::integral_constant<int, 0>{});
    }
    static_for<D - 1>([&](auto ic) {
        constexpr int j = decltype(ic)::value + 1;
        if constexpr (!P3 && j < DA) load_a_all(j, std::integral_constant<int, j % NA>{});
        load_b_all(j, std::integral_constant<int, j % NB>{});
    });
    if constexpr (MX) dequant_all(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    wg_decide(p, un.row0, 1, probe, &s_run);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if (p.go != nullptr && s_run == 0) return;
    if constexpr (P3) read_first(0);
    int it = 0;
    for (; it + U <= iters; it += U) {
        static_for<U>([&](auto ic) { body(it + decltype(ic)::value, ic); });
    }
    static_for<U - 1>([&](auto ic) {
        if (it + decltype(ic)::value < iters) body(it + decltype(ic)::value, ic);
    });

    // ---- epilogue.  acc[fragment][matrix][row half]: lane (lg, lr) holds weight rows 4*lg .. 4*lg + 3 of token lr ----
    // Before the first store the prefetches past the last iteration are waited for: as long as they may be pending the compiler
    // waits, at every store under a condition, for everything before it, the store before included: about 280 clocks a store.
    // Down projection of 224 rows: epilogue 17 -> 11 to 14 thousand clocks; 8192 tokens on 64 experts 1132 -> 1124 us, 1531 enqueued 983 -> 976.
    // What is left is the fabric: a round of 256 rows a workgroup ends with 8 MB of fp32 to store on each XCD, 400 bytes a clock.
    constexpr int kAllLoaded = 0x0f70;        // vmcnt 0
    if (GATEUP) {
        // SwiGLU in fp32, one rounding to bf16; the wave's [T*32 tokens][32 f] tile goes through LDS
        // (free after the last barrier of the main loop; a wave's LDS accesses are carried out in order) so that it leaves as
        // 16-byte stores, with the non-temporal hint: the next kernel reads it, nothing in this one does.
        __bf16 *st = reinterpret_cast<__bf16 *>(lds) + w * (ROWS * 32);
        static_for<NF>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            static_for<2>([&](auto rc) {
                constexpr int rt = decltype(rc)::value;
                bf16x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (__bf16)(silu_f(acc[f * NQ + rt][r]) * acc[f * NQ + NQ - 2 + rt][r]);
                *reinterpret_cast<bf16x4 *>(st + (f * 16 + lr) * 32 + rt * 16 + lg * 4) = v;
            });
        });
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_s_waitcnt(kAllLoaded);
        if (cpw == 32) {
            const int f0 = col_base + (l & 3) * 8;
#pragma unroll
            for (int j = 0; j < 2 * T; ++j) {
                const int i = (l >> 2) + 16 * j;
                const u32x4 v = *reinterpret_cast<const u32x4 *>(st + i * 32 + (l & 3) * 8);
                if (i < rows && f0 < p.ncols) gstore_nt(v, ((__bf16 *)p.dst + (long)(un.row0 + i) * p.ldd + f0));
            }
        } else {
            // narrower waves start at multiples of 4 columns: 8-byte stores of the first cpw columns
            const int fo = (l & 7) * 4;
#pragma unroll
            for (int j = 0; j < 4 * T; ++j) {
                const int i = (l >> 3) + 8 * j;
                const u32x2 v = *reinterpret_cast<const u32x2 *>(st + i * 32 + fo);
                if (i < rows && fo < cpw && col_base + fo < p.ncols) gstore_nt(v, ((__bf16 *)p.dst + (long)(un.row0 + i) * p.ldd + col_base + fo));
            }
        }
    } else {
        // fp32 tile of 32 tokens x 64 (narrow: 32) columns at a time through this wave's part of LDS (slots of 16 bytes,
        // XORed by token), so that it leaves as 16-byte stores of 256 (128) contiguous bytes per token row.
        constexpr int SR = 8 * NM;              // slots of a token
        char *st = lds + w * (32 * SR * 16);
        float *obase = (float *)p.dst + kq * plane + (long)un.row0 * p.ldd + col_base + (l % SR) * 4;
        const bool col_ok = col_base + (l % SR) * 4 < p.ncols;
        static_for<T>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            if (t * 32 < rows) {
                __builtin_amdgcn_wave_barrier();
                static_for<2 * NQ>([&](auto qc) {
                    constexpr int q = decltype(qc)::value % NQ, h = decltype(qc)::value / NQ;
                    if constexpr (2 * t + h < NF) *reinterpret_cast<f32x4 *>(st + ((h * 16 + lr) * SR + ((q * 4 + lg) ^ (lr % SR))) * 16) = acc[(2 * t + h) * NQ + q];
                });
                __builtin_amdgcn_wave_barrier();
                if constexpr (t == 0) __builtin_amdgcn_s_waitcnt(kAllLoaded);
                f32x4 v[4 * NM];
#pragma unroll
                for (int j = 0; j < 4 * NM; ++j) {
                    const int i = l / SR + 64 / SR * j;
                    v[j] = *reinterpret_cast<const f32x4 *>(st + (i * SR + ((l % SR) ^ (i % SR))) * 16);
                }
#pragma unroll
                for (int j = 0; j < 4 * NM; ++j) {
                    const int i = l / SR + 64 / SR * j;
                    if (t * 32 + i < rows && col_ok) gstore_nt(v[j], (obase + (long)(t * 32 + i) * p.ldd));
                }
            }
        });
    }
}

// Workgroup id -> (unit, column tile, K range): see expert_items.h.  A launch that streams deals nothing to the XCDs.
template <bool STREAM>
__device__ __forceinline__ bool map_block(const BArgs &b, moe_unit &un, int &ct, int &kq) {
    // This stands in front of every workgroup's first load: one round of scalar loads for what tells the three orders
    // apart, one piece of code for the two that go by columns.  With a flag of its own for dealt-out experts and a
    // branch of its own for each order, 3584 tokens on 8 experts took 0.3 % longer with 4-bit weights or fed in fours.
    const unsigned items = b.items, cols = (unsigned)(b.k.col_tiles * b.ksplit);
    unsigned item = blockIdx.x / kXcds, first = 0, n = b.nseg > 0 ? 0 : (unsigned)b.k.nu;     // n segments or units by columns
    if (!STREAM && __builtin_expect(items == 0, 0)) {
        const unsigned x = blockIdx.x % kXcds;
        first = b.xcd[x];
        n = b.xcd[x + 1] - first;
        if (item >= n * cols) return false;
    } else if (!item_of(blockIdx.x, items, item)) {
        return false;
    }
    ItemPos ip;
    if (__builtin_expect(n > 0, 0)) {
        ip = column_item_pos(item, n, cols);
        ip.pos += first;
    } else {
        ip = item_pos(item, cols, [&](unsigned q, unsigned &in, unsigned &size) { in = b.seg[q].grp & 15; size = b.seg[q].grp >> 4; });
    }
    if (b.nseg > 0) {
        const ItemSeg g = b.seg[ip.pos];
        un.expert = g.expert; un.cls = 0; un.row0 = (int)g.row0; un.rows = g.rows;
    } else {
        un = b.k.units[b.k.u0 + ip.pos];
    }
    kq = (int)ip.cq / b.k.col_tiles;
    ct = (int)ip.cq - kq * b.k.col_tiles;
    return true;
}

// TCAP: largest number of 32-row pieces a segment of this launch may have (1, 2, 4, 6 or 8).  A
// workgroup takes the fully unrolled variant for as many 16-token fragments as its unit has (1, 2, 4 to 16).
// STREAM: no two segments of the launch belong to one expert, so every weight element is read by
// exactly one workgroup: the loads carry the non-temporal hint and do not displace the token tiles
// in L2.  Where segments share an expert's weights the hint is left off so that L2 serves the re-reads.
template <int TCAP, bool GATEUP, int WF, bool STREAM>
__global__ __launch_bounds__(256) void expert_bf16(const BArgs b) {
    // two token-tile stages (three from 65 rows on, kP3MinT); at least 8 KiB per wave for the
    // epilogue's store staging
    __shared__ __attribute__((aligned(16))) char lds[((TCAP >= kP3MinT ? 3 : 2) * TCAP * 32 * 128) > 32768 ? ((TCAP >= kP3MinT ? 3 : 2) * TCAP * 32 * 128) : 32768];
    // A closed gate: the sequence was stopped before this launch, or an earlier workgroup of it saw
    // the stop word.  The word may change while the launch runs, so one thread reads it for all.
    if (b.k.go != nullptr) {
        __shared__ int s_go;
        if (threadIdx.x == 0) s_go = __hip_atomic_load(b.k.go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_go == 0) return;
    }
    int ct, kq;
    moe_unit un;
    if (!map_block<STREAM>(b, un, ct, kq)) return;
    const int nf = (un.rows + 15) >> 4;
    // One copy for all variants: the compiler reads the arguments in place only where it finds few enough uses of them,
    // and keeps them in scratch memory otherwise.
    const KArgs k = b.k;
    const int ksplit = b.ksplit;
    const long plane = b.plane;
    // Prefetch distance of the weights: 2 iterations for the three-stage variants (their loop is unrolled by
    // a multiple of 3) and up to 64 rows, 3 up to 32 rows; 4-bit iterations are short and their codes take few registers:
    // 5 (top-2 of 8 experts, H 4096, F 14336, 2 K ranges, down projection with 2 / 3 / 5: 8 tokens 64 / 47 / 42 us, 64 tokens,
    // skewed, 87 / 59 / 56; the layer after 5 ms of idle, its code cold, with 3 / 5: 8 tokens 169 / 165, one token 85 / 80.  K loops
    // of up to 20 iterations gain 2 to 4 % of a launch with 3 where every workgroup has a CU to itself, lose as much where not).
#define QMOE_TILE(n, d) else if (2 * TCAP >= n && nf >= n) expert_tile<(2 * TCAP >= n ? n : 1), GATEUP, WF, STREAM, d>(k, un, ct, kq, ksplit, plane, lds)
    constexpr int D1 = WF == WF_MXFP4 ? 5 : 3, D2 = WF == WF_MXFP4 ? 5 : 2;
    if (false) {}
    QMOE_TILE(16, 2); QMOE_TILE(15, 2); QMOE_TILE(14, 2); QMOE_TILE(13, 2); QMOE_TILE(12, 2); QMOE_TILE(11, 2); QMOE_TILE(10, 2); QMOE_TILE(9, 2);
    QMOE_TILE(8, 2); QMOE_TILE(7, 2); QMOE_TILE(6, 2); QMOE_TILE(5, 2); else if (TCAP >= 2 && nf >= 3) expert_tile<(TCAP >= 2 ? 4 : 1), GATEUP, WF, STREAM, D2>(k, un, ct, kq, ksplit, plane, lds);
    QMOE_TILE(2, D1); QMOE_TILE(1, D1);
#undef QMOE_TILE
}

// The down projection of at most 32 rows in the narrow form: 128 columns a workgroup, for launches of few workgroups.
template <int WF>
__global__ __launch_bounds__(256) void expert_down_narrow(const BArgs b) {
    __shared__ __attribute__((aligned(16))) char lds[16384];
    int ct, kq;
    moe_unit un;
    if (!map_block<true>(b, un, ct, kq)) return;
    const KArgs k = b.k;
    const int ksplit = b.ksplit;
    const long plane = b.plane;
    if (un.rows > 16) expert_tile<2, false, WF, true, 5, 1>(k, un, ct, kq, ksplit, plane, lds);
    else expert_tile<1, false, WF, true, 5, 1>(k, un, ct, kq, ksplit, plane, lds);
}

template <int TCAP, bool GATEUP, int WF, bool STREAM>
void launch1(const BArgs &b, hipStream_t s) {
    const unsigned grid = b.items ? item_grid(b.items) : dealt_grid(b.xcd, (unsigned)(b.k.col_tiles * b.ksplit));
    hipLaunchKernelGGL((expert_bf16<TCAP, GATEUP, WF, STREAM>), dim3(grid), dim3(256), 0, s, b);
}

template <bool GATEUP, int WF, bool STREAM>
void launch_ts(int tiles, const BArgs &b, hipStream_t s) {
    // The kernel for up to 64 rows is of use to 4-bit weights alone (two workgroups of it share a CU); 160 tokens on 8 experts
    // with bf16 weights: gate-up 306 us in one of their own, 296 in the kernel for up to 128 rows.
    if (tiles <= 1) launch1<1, GATEUP, WF, STREAM>(b, s);
    else if (WF == WF_MXFP4 && tiles <= 2) launch1<(WF == WF_MXFP4 ? 2 : 4), GATEUP, WF, STREAM>(b, s);
    else if (tiles <= 4) launch1<4, GATEUP, WF, STREAM>(b, s);
    else if (tiles <= 6) launch1<6, GATEUP, WF, STREAM>(b, s);
    else launch1<8, GATEUP, WF, STREAM>(b, s);
}

// One expert kernel of one weight format, for segments of at most `tiles` 32-row pieces.  Each is instantiated in a
// translation unit of its own (experts_bf16_w<WF>_<kernel>.hip).
template <int WF, bool GATEUP>
void launch_expert_kernel(int tiles, bool stream, const BArgs &b, hipStream_t s) {
    if constexpr (!GATEUP) {
        if (b.narrow) {
            hipLaunchKernelGGL(expert_down_narrow<WF>, dim3(item_grid(b.items)), dim3(256), 0, s, b);
            return;
        }
    }
    if (stream) launch_ts<GATEUP, WF, true>(tiles, b, s);
    else launch_ts<GATEUP, WF, false>(tiles, b, s);
}

extern template void launch_expert_kernel<WF_ROWMAJOR, true>(int, bool, const BArgs &, hipStream_t);
extern template void launch_expert_kernel<WF_ROWMAJOR, false>(int, bool, const BArgs &, hipStream_t);
extern template void launch_expert_kernel<WF_PACKED, true>(int, bool, const BArgs &, hipStream_t);
extern template void launch_expert_kernel<WF_PACKED, false>(int, bool, const BArgs &, hipStream_t);
extern template void launch_expert_kernel<WF_MXFP4, true>(int, bool, const BArgs &, hipStream_t);
extern template void launch_expert_kernel<WF_MXFP4, false>(int, bool, const BArgs &, hipStream_t);

}  // namespace bf16k
}  // namespace qmoe
