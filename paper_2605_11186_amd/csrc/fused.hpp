#pragma once
// Weight-streaming products whose workgroups end with complete sums, so that the step behind the
// product (rotation and cache append for q|k|v, SwiGLU for gate|up) is carried out on them before
// anything is written: no partial tiles, no row kernel.
//
// What bounds it: HBM for the weights up to about 32 rows, beyond that the cache lines that a compute unit can have on
// their way: every workgroup requests all of X (16 M rows x K x 4 bytes) beside its weights.
//
// Split.  A workgroup owns R column groups of 16 for the whole of K; its W waves split K, each one
// streaming its own weight and activation fragments from memory straight into MFMA operand registers
// (a register ring of D steps of 32 k-values).  Nothing is shared between the waves before the end, so
// the stream has no barrier and no LDS staging; X arrives in fragment order (see packed X below), one
// contiguous kilobyte per wave load.  At the end the waves' sums meet in LDS.  A column group is eight rows
// of one place in the weights and eight of another (gate and up rows of the same columns; the two
// halves of a rotation pair), so that whatever the step behind the product combines is inside one group
// and any number of groups makes a workgroup: R is the smallest count with which the chip holds all of them at once.
//
// Measured on the 7B shape, kernel times: gate|up (180 MB of weights) 31 us at 16 rows, 40 at 63, 60 at 128;
// q|k|v (100 MB) 20 / 30 / 46 us.  The growth with the rows is not matrix time (16 and 22 % of the cycles at 64 rows, 30 at
// 128): time = (lines of W x 1000 cycles + lines of X x 240) / (compute units x 58 to 96 lines on their way), by the
// counters of L1 requests and their latency, within 5 % at 64 and 128 rows.
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.hpp"

namespace {

enum { EPI_QKV = 0, EPI_SWIGLU = 1 };

// Packed X: 16-row x 32-column fragments in MFMA 16x16x32 operand order, [row block][k step][hi, lo]
// of 512 elements each; lane l of a fragment holds row l % 16, k-values 8 (l / 16) .. + 7.
// Rows past T inside the last blocks are stale: they only reach accumulator rows that nothing stores.
//
// MFMA 16x16x32 bf16 (wave64): lane l supplies, for A, row l % 16 and k = 8 (l / 16) .. + 7; for B,
// column l % 16 and the same k; its four results are D[4 (l / 16) + r][l % 16].
template <int R, int M, int W, int D, bool PACKED, int EPI>
__global__ __launch_bounds__(64 * W) void cats_gemm_rows(FusedArgs a) {
    constexpr int THREADS = 64 * W;
    constexpr int LD = 16 * R + 4;   // row pitch of the sums in LDS: 4 LD = 16 (mod 64) banks, conflict-free stores
    // row blocks per pass of the final reduction (LDS holds W waves' sums of them)
    constexpr int FIT = 150 * 1024 / (W * 16 * LD * 4);
    constexpr int PM = FIT >= M ? M : (FIT >= (M + 1) / 2 ? (M + 1) / 2 : (FIT >= 2 && M % 2 == 0 ? 2 : 1));
    static_assert(PM <= FIT, "reduction pass exceeds the LDS");
    __shared__ float red[W][PM * 16][LD];
    __shared__ float s_rs[CATS_MAX_TREE];

    // consecutive units on one XCD (block b runs on XCD b % 8): neighbours write parts of the same lines
    const int upx = gridDim.x / 8;
    const int unit = static_cast<int>(blockIdx.x) % 8 * upx + static_cast<int>(blockIdx.x) / 8;
    if (unit * R >= a.groups) return;   // whole workgroup

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, q = lane >> 4;
    const int S = a.K / 32, C = (a.K + GEMM_KC - 1) / GEMM_KC;
    const int s0 = S * wave / W, n = S * (wave + 1) / W - s0;   // this wave's k steps (none if K is tiny)
    const int last = max(n - 1, 0);

    const bf16_t* wp[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int gr = min(unit * R + r, a.groups - 1);
        const bf16_t* base;
        int row;
        if (EPI == EPI_SWIGLU) {
            base = r16 < 8 ? a.w[0] : a.w[1];
            row = 8 * gr + (r16 & 7);
        } else {
            const int per_sec = a.H / 16;
            const int sec = gr >= 2 * per_sec ? 2 : (gr >= per_sec ? 1 : 0);
            const int u = gr - sec * per_sec;
            base = sec == 0 ? a.w[0] : (sec == 1 ? a.w[1] : a.w[2]);
            if (sec < 2) {   // dims 8 jb .. + 7 of a head and the ones half a head further
                const int h = u >> a.hd_shift, jb = u & ((1 << a.hd_shift) - 1);
                row = h * a.d + 8 * jb + (r16 & 7) + (r16 < 8 ? 0 : a.d / 2);
            } else {
                row = 16 * u + r16;
            }
        }
        wp[r] = PACKED ? base + (static_cast<size_t>(row / PACK_ROWS) * C * 8 + 2 * s0 + (q >> 1)) * PACK_FRAG +
                             (row % PACK_ROWS + 32 * (q & 1)) * 8
                       : base + static_cast<size_t>(row) * a.K + 32 * s0 + 8 * q;
    }
    constexpr int W_STEP = PACKED ? 2 * PACK_FRAG : 32;
    const bf16_t* xb = a.xp + static_cast<size_t>(s0) * 1024 + lane * 8;

    u32x4 wr[D][R], xr[D][2 * M];
    f32x4 acc[R][M];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[r][m] = f32x4{0.f, 0.f, 0.f, 0.f};

    // loads are unconditional (indices past the range are clamped: harmless reloads), see gemm.hip
    auto load = [&](int slot, int i) __attribute__((always_inline)) {
        const int ic = min(i, last);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const bf16_t* xs = xb + (static_cast<size_t>(m) * S + ic) * 1024;
            xr[slot][2 * m] = *reinterpret_cast<const u32x4*>(xs);
            xr[slot][2 * m + 1] = *reinterpret_cast<const u32x4*>(xs + 512);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            wr[slot][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wp[r] + static_cast<size_t>(ic) * W_STEP));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mult = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bf16x8 b = as_bf16x8(wr[slot][r]);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xr[slot][2 * m]), b, acc[r][m], 0, 0, 0);
                acc[r][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xr[slot][2 * m + 1]), b, acc[r][m], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load(s, s);
    int c = 0;
    for (; c + D < n; c += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            mult(s);
            load(s, c + s + D);
        }
    }
    // the rows' sums of squares: eight lanes per row, 16 bytes each, requested ahead of the last products
    constexpr int SQ_PASS = THREADS / 8, SQ_N = (16 * M + SQ_PASS - 1) / SQ_PASS;
    f32x4 sq[SQ_N];
#pragma unroll
    for (int p = 0; p < SQ_N; ++p)
        sq[p] = *reinterpret_cast<const f32x4*>(a.ns.ss + min(p * SQ_PASS + (tid >> 3), a.T - 1) * SS_STRIDE + 4 * (tid & 7));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (c + s < n) mult(s);
#pragma unroll
    for (int p = 0; p < SQ_N; ++p) {
        float v = (sq[p][0] + sq[p][1]) + (sq[p][2] + sq[p][3]);
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) v += __shfl_xor(v, o);
        const int t = p * SQ_PASS + (tid >> 3);
        if ((tid & 7) == 0 && t < a.T) s_rs[t] = 1.0f / sqrtf(v / static_cast<float>(a.ns.H) + a.ns.eps);
    }

#pragma unroll
    for (int p0 = 0; p0 < M; p0 += PM) {
        if (p0) __syncthreads();   // the pass before has been read
#pragma unroll
        for (int m = 0; m < PM; ++m)
            if (p0 + m < M)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e) red[wave][m * 16 + 4 * q + e][r * 16 + r16] = acc[r][(p0 + m) < M ? p0 + m : 0][e];
        __syncthreads();
        constexpr int TP = 16 * PM;
        const int t_lim = min(a.T - 16 * p0, TP);
        for (int i = tid; i < TP * R * 2; i += THREADS) {
            // SwiGLU: columns fastest (rows of h are contiguous); q|k|v: nodes fastest (columns of the
            // transposed value cache are)
            const int tl = EPI == EPI_SWIGLU ? i / (2 * R) : i % TP;
            const int rq = EPI == EPI_SWIGLU ? i % (2 * R) : i / TP;
            const int qd = rq & 1, r = rq >> 1;
            const int gr = unit * R + r;
            if (tl >= t_lim || gr >= a.groups) continue;
            const int t = 16 * p0 + tl;
            f32x4 va = *reinterpret_cast<const f32x4*>(&red[0][tl][r * 16 + 4 * qd]);
            f32x4 vb = *reinterpret_cast<const f32x4*>(&red[0][tl][r * 16 + 8 + 4 * qd]);
#pragma unroll
            for (int w = 1; w < W; ++w) {
                va += *reinterpret_cast<const f32x4*>(&red[w][tl][r * 16 + 4 * qd]);
                vb += *reinterpret_cast<const f32x4*>(&red[w][tl][r * 16 + 8 + 4 * qd]);
            }
            const float rs = s_rs[t];
            if (EPI == EPI_SWIGLU) {
                uint2 hi, lo;
                swiglu_split4(va, vb, rs, hi, lo);
                const size_t o = static_cast<size_t>(t) * a.F + 8 * gr + 4 * qd;
                *reinterpret_cast<uint2*>(a.h + o) = hi;
                *reinterpret_cast<uint2*>(a.h_lo + o) = lo;
                continue;
            }
            va *= rs;
            vb *= rs;
            const int per_sec = a.H / 16;
            const int sec = gr >= 2 * per_sec ? 2 : (gr >= per_sec ? 1 : 0);
            const int u = gr - sec * per_sec;
            if (sec == 2) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int col = 16 * u + 4 * qd + (e < 4 ? e : e + 4);   // h * d + dim
                    const float v = e < 4 ? va[e & 3] : vb[e & 3];
                    const bf16_t hi = f2bf(v);
                    a.vt[static_cast<size_t>(col) * a.max_ctx + a.row0 + t] = hi;
                    a.vt_lo[static_cast<size_t>(col) * TREE_WIN + a.win0 + t] = f2bf(v - bf2f(hi));
                }
                continue;
            }
            const int h = u >> a.hd_shift, j = 8 * (u & ((1 << a.hd_shift) - 1)) + 4 * qd, half = a.d / 2;
            float o0[4], o1[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 cs = a.cs[t * half + j + e];
                o0[e] = va[e] * cs.x - vb[e] * cs.y;
                o1[e] = va[e] * cs.y + vb[e] * cs.x;
            }
            uint2 h0, l0, h1, l1;
            split_bf2(o0[0], o0[1], h0.x, l0.x);
            split_bf2(o0[2], o0[3], h0.y, l0.y);
            split_bf2(o1[0], o1[1], h1.x, l1.x);
            split_bf2(o1[2], o1[3], h1.y, l1.y);
            bf16_t *dst, *dst_lo;
            if (sec == 0) {
                const size_t o = static_cast<size_t>(t) * a.H + h * a.d + j;
                dst = a.q + o;
                dst_lo = a.q_lo + o;
            } else {
                dst = a.kc + (static_cast<size_t>(h) * a.max_ctx + a.row0 + t) * a.d + j;
                dst_lo = a.k_lo + (static_cast<size_t>(h) * TREE_WIN + a.win0 + t) * a.d + j;
            }
            *reinterpret_cast<uint2*>(dst) = h0;
            *reinterpret_cast<uint2*>(dst + half) = h1;
            *reinterpret_cast<uint2*>(dst_lo) = l0;
            *reinterpret_cast<uint2*>(dst_lo + half) = l1;
        }
    }
}

// Waves and ring depth: eight waves (two per SIMD, 256 registers each: one multiplies while the other
// waits) with the deepest ring that fits, else four waves with up to 512 registers.  Depths are powers of
// two so that they divide a wave's step count at the usual widths (K = 4096: 16 steps on eight
// waves); a depth of 3 or 5 there costs 4-10 % in reloads at the range's end.  (Beyond 96 rows gate|up with R = 8, and with
// R = 7 on row-major weights, still spills two to five registers.)
template <int R, int M>
struct Shape {
    static constexpr int regs(int depth) { return 4 * R * M + 4 * depth * (R + 2 * M) + 2 * R + 28; }
    static constexpr int D8 = regs(4) <= 256 ? 4 : (regs(2) <= 256 ? 2 : (regs(1) <= 256 ? 1 : 0));
    static constexpr int W = D8 ? 8 : 4;
    static constexpr int D = D8 ? D8 : (regs(4) <= 480 ? 4 : (regs(2) <= 480 ? 2 : 1));
};

template <int R, int M, int EPI>
void launch_rm(const FusedArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    constexpr int W = Shape<R, M>::W, D = Shape<R, M>::D;
    const int units = (a.groups + R - 1) / R;
    const dim3 grid((units + 7) / 8 * 8), block(64 * W);
    if (a.packed)
        hipExtLaunchKernelGGL((cats_gemm_rows<R, M, W, D, true, EPI>), grid, block, 0, st, e0, e1, 0, a);
    else
        hipExtLaunchKernelGGL((cats_gemm_rows<R, M, W, D, false, EPI>), grid, block, 0, st, e0, e1, 0, a);
}

template <int R, int EPI>
void launch_r(const FusedArgs& a, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    switch (fused_row_blocks(a.T)) {
        case 1: return launch_rm<R, 1, EPI>(a, st, e0, e1);
        case 2: return launch_rm<R, 2, EPI>(a, st, e0, e1);
        case 3: return launch_rm<R, 3, EPI>(a, st, e0, e1);
        case 4: return launch_rm<R, 4, EPI>(a, st, e0, e1);
        case 6: return launch_rm<R, 6, EPI>(a, st, e0, e1);
        default: return launch_rm<R, 8, EPI>(a, st, e0, e1);
    }
}

}  // namespace
