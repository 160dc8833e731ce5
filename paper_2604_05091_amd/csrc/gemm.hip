// bf16 x bf16 -> fp32-accumulate GEMM on the gfx950 matrix cores.
//
//   C[M,N] = A[M,K] . B[N,K]^T (+ bias) (+ R)      both operands have the reduction index contiguous
//
// This one entry point serves every projection of a transformer block (Algorithm 1,
// "h_i <- f_i(h_{i-1}; theta_i)" and "LocalBackward"): forward uses the weight as
// stored ([out,in]); the input-gradient and weight-gradient products are brought to
// the same form by transposing one or both operands with transpose_bf16 first.
//
// Here a workgroup owns a 256 x 256 tile of C made of 16x16 MFMA blocks (v_mfma_f32_16x16x32_bf16, 4 fp32 accumulators
// per lane per block): 4 waves x 128x128 quadrants, K walked in steps of 64 through a double-buffered LDS stage,
// software-pipelined inside the wave.  Grids that 256 x 256 tiles fill badly go to the kernels with smaller tiles in
// gemm_ring.hip (choose_tile).
//
// Workgroup -> tile mapping: consecutive workgroup ids are dealt round-robin to the
// 8 XCDs, each with a private L2.  The id is first re-numbered so that every XCD gets
// a contiguous range of tiles, then walked in column-major groups of kGroupMLarge tile rows
// so the 32 tiles resident on one XCD form a 4 x 8 patch that shares A and B panels.
#include <stdlib.h>

#include <algorithm>
#include <cmath>
#include <iterator>
#include <type_traits>

#include "common.h"

namespace mt {

namespace {

constexpr int BK = 64;
constexpr int kXcd = 8;
constexpr int kRound = 256;   // workgroups of one round: a compute unit holds one of these kernels' workgroups
constexpr int W4_BM = 256, W4_BN = 256, W4_NT = 256;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// bf16 results leave through LDS.  Stored straight from the accumulator layout, a store instruction touches 32
// rows with 16 bytes each, and these partial-line writes cost 10-13 us per tile; instead every wave writes its
// 128 x NC block (bf16) into a private LDS region (the k-loop's stages are free after its last barrier) and reads
// it back row-wise, so that a store instruction covers whole 128-byte lines (16 bytes per lane, consecutive lanes
// at consecutive addresses).  Region pitch NC + 8 elements: conflict-free for the 8-byte writes and the 16-byte reads.
constexpr int W4_EP_PITCH = 128 + 8;

// second half: rows of the wave's block from LDS to C, NC columns starting at col0; rows >= M skipped
template <int NC>
__device__ __forceinline__ void w4_flush_rows(bf16_t *C, int64_t ldc, int M, int row0, int col0, const bf16_t *region,
                                              int lane) {
    constexpr int LPR = NC / 8, RPI = 64 / LPR;   // lanes per row, rows per instruction
    const int lr = lane / LPR, lc = (lane % LPR) * 8;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own LDS writes have landed
#pragma unroll 8
    for (int it = 0; it < 128 / RPI; ++it) {
        const int r = it * RPI + lr;
        const int64_t row = row0 + r;
        if (row >= M) continue;
        *reinterpret_cast<uint4 *>(C + row * ldc + col0 + lc) = *reinterpret_cast<const uint4 *>(region + r * W4_EP_PITCH + lc);
    }
}

// Epilogue of the 4-wave kernels.  The MFMAs are issued with the operands swapped (B fragment first), so each
// 16x16 block holds C transposed: the lane owns row l16 of the block and its four consecutive columns
// 4 hq + (0..3): one 16-byte store each in fp32.
__device__ __forceinline__ void w4_store_guarded_f32(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm, int wn,
                                                     int l16, int hq) {
    const int row_l = m0 + wm * 128 + l16, col_l = n0 + wn * 128 + hq * 4;
    const bool vec = m0 + W4_BM <= g.M && n0 + W4_BN <= g.N && !(g.ldc & 3) && !((uintptr_t)g.C & 15);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = row_l + i * 16;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int col = col_l + j * 16;
            f32x4 v = acc[i][j];
            float *cp = reinterpret_cast<float *>(g.C) + (int64_t)row * g.ldc + col;
            if (vec) {
                if (g.accumulate) v += *reinterpret_cast<const f32x4 *>(cp);
                *reinterpret_cast<f32x4 *>(cp) = v;
            } else if (row < g.M) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < g.N) cp[e] = v[e] + (g.accumulate ? cp[e] : 0.f);
            }
        }
    }
}

// bf16 for any columns, pitches and alignment, bias and residual added in fp32 before the one rounding.  Blocks of 16 rows pass through
// the wave's LDS region as fp32 (pitch 132: the 16-byte writes of consecutive rows fall on disjoint banks) and leave row-wise, 8 columns
// per lane.  From the accumulator layout with a test per element -> here, us:
// 16384 x 11000 x 4096 1176 -> 1055, 16384 x 11000 x 512 319 -> 222, 8192 x 4096 x 1024 with a pitch of 4100 110 -> 63 (with residual 170 -> 83).
__device__ __forceinline__ void w4_store_guarded_bf16(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm, int wn,
                                                      int l16, int hq, bf16_t *region) {
    constexpr int P = 132;
    static_assert(16 * P * 4 <= 128 * W4_EP_PITCH * 2, "room in the region");
    float *st = reinterpret_cast<float *>(region);
    const int lr = hq, lc = l16 * 8, col = n0 + wn * 128 + lc;
    const int access = row_access(g.C, g.ldc, col, g.N), access_r = row_access(g.R, g.ldr, col, g.N);
    float bias[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bias[e] = g.bias && col + e < g.N ? bf2f(g.bias[col + e]) : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's reads of the block before
#pragma unroll
        for (int j = 0; j < 8; ++j) *reinterpret_cast<f32x4 *>(st + l16 * P + j * 16 + hq * 4) = acc[i][j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // its writes have landed
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(st + (p * 4 + lr) * P + lc), hi = *reinterpret_cast<const f32x4 *>(st + (p * 4 + lr) * P + lc + 4);
            const int64_t row = m0 + wm * 128 + i * 16 + p * 4 + lr;
            if (row >= g.M || col >= g.N) continue;
            float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += bias[e];
            if (g.R) row_add8(v, g.R + row * g.ldr + col, access_r, col, g.N);
            row_store8(reinterpret_cast<bf16_t *>(g.C) + row * g.ldc + col, v, access, col, g.N);
        }
    }
}

// complete, aligned column tiles (what the host checks before it picks the kernel instantiated with this store;
// a ragged last row tile is handled by row guards).  Bias
// and residual are template parameters as well: tested per element at run time they turned every one of the 64
// loads into a branch with its own wait.  Here a row block's 16 residual loads are in flight together.
template <bool BIAS, bool RES>
__device__ __forceinline__ void w4_store_full_bf16(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm,
                                                   int wn, int l16, int hq, bf16_t *region) {
    const int lane = hq * 16 + l16;
    const int col_l = n0 + wn * 128 + hq * 4;
    uint2 bv[8];
    if constexpr (BIAS) {
#pragma unroll
        for (int j = 0; j < 8; ++j) bv[j] = *reinterpret_cast<const uint2 *>(g.bias + col_l + j * 16);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        bf16_t *lp = region + (i * 16 + l16) * W4_EP_PITCH + hq * 4;
        // bias and residual are added in fp32, before the one rounding to bf16
        uint2 rv[8];
        if constexpr (RES) {
            // rows past M (a ragged last row tile) re-read the last row; the second half never stores them
            const bf16_t *rp = g.R + (int64_t)min(m0 + wm * 128 + i * 16 + l16, g.M - 1) * g.ldr + col_l;
#pragma unroll
            for (int j = 0; j < 8; ++j) rv[j] = *reinterpret_cast<const uint2 *>(rp + j * 16);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f32x4 v = acc[i][j];
            if constexpr (BIAS) {
                v[0] += bflo(bv[j].x); v[1] += bfhi(bv[j].x); v[2] += bflo(bv[j].y); v[3] += bfhi(bv[j].y);
            }
            if constexpr (RES) {
                v[0] += bflo(rv[j].x); v[1] += bfhi(rv[j].x); v[2] += bflo(rv[j].y); v[3] += bfhi(rv[j].y);
            }
            *reinterpret_cast<uint2 *>(lp + j * 16) = uint2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
        }
    }
    w4_flush_rows<128>(reinterpret_cast<bf16_t *>(g.C), g.ldc, g.M, m0 + wm * 128, n0 + wn * 128, region, lane);
}

__device__ __forceinline__ void w4_store_full_f32(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm,
                                                  int wn, int l16, int hq) {
    const int row_l = m0 + wm * 128 + l16, col_l = n0 + wn * 128 + hq * 4;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (row_l + i * 16 >= g.M) continue;   // ragged last row tile
        float *cp = reinterpret_cast<float *>(g.C) + (int64_t)(row_l + i * 16) * g.ldc + col_l;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f32x4 v = acc[i][j];
            if (g.accumulate) v += *reinterpret_cast<const f32x4 *>(cp + j * 16);
            *reinterpret_cast<f32x4 *>(cp + j * 16) = v;
        }
    }
}

// bf16 store with the rotary embedding applied on the way out (g.rope_*): the wave's 128 columns are one head,
// the lane holds both members (j, j + 64) of every pair of its rows: blocks j and j + 4 of acc.  Columns are
// complete (N % 128 == 0, checked on the host); rows are guarded.  Heads at or beyond rope_cols (the value
// projection) are stored unrotated.  Bias, if any, is added before the rotation.  The rows leave through LDS.
template <bool BIAS>
__device__ __forceinline__ void w4_store_rope(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm, int wn,
                                              int l16, int hq, bf16_t *region) {
    const int row_l = m0 + wm * 128 + l16, col_w = n0 + wn * 128;
    if (col_w >= g.N) return;
    const bool rot = col_w < g.rope_cols;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // rows past M compute values nobody stores; their table row is still a valid one
        const int64_t tpos = (int64_t)((row_l + i * 16) % g.rope_T) * 64;
        bf16_t *lp = region + (i * 16 + l16) * W4_EP_PITCH;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int jc = j * 16 + hq * 4;  // pair index inside the head, < 64
            f32x4 a = acc[i][j], b = acc[i][j + 4];
            if constexpr (BIAS) {
                const uint2 ba = *reinterpret_cast<const uint2 *>(g.bias + col_w + jc);
                const uint2 bb = *reinterpret_cast<const uint2 *>(g.bias + col_w + jc + 64);
                a[0] += bflo(ba.x); a[1] += bfhi(ba.x); a[2] += bflo(ba.y); a[3] += bfhi(ba.y);
                b[0] += bflo(bb.x); b[1] += bfhi(bb.x); b[2] += bflo(bb.y); b[3] += bfhi(bb.y);
            }
            if (rot) {
                const f32x4 c = *reinterpret_cast<const f32x4 *>(g.rope_cos + tpos + jc);
                const f32x4 sn = *reinterpret_cast<const f32x4 *>(g.rope_sin + tpos + jc);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ya = a[e] * c[e] - b[e] * sn[e], yb = b[e] * c[e] + a[e] * sn[e];
                    a[e] = ya;
                    b[e] = yb;
                }
            }
            *reinterpret_cast<uint2 *>(lp + jc) = uint2{pack2bf(a[0], a[1]), pack2bf(a[2], a[3])};
            *reinterpret_cast<uint2 *>(lp + jc + 64) = uint2{pack2bf(b[0], b[1]), pack2bf(b[2], b[3])};
        }
    }
    w4_flush_rows<128>(reinterpret_cast<bf16_t *>(g.C), g.ldc, g.M, m0 + wm * 128, col_w, region, hq * 16 + l16);
}

// SwiGLU store (g.glu_*): the tile's 256 B rows are gate columns c .. c+63, up columns c .. c+63, gate c+64 ..,
// up c+64 .. with c = 128 tn, so a wave holds gate (blocks 0..3) and up (blocks 4..7) of the same 64 columns.
// Both go through the wave's LDS region; the row-wise second half computes the activation and stores it (and
// gate | up if asked for) as whole lines.  Rows are guarded; columns are complete (glu_F % 128 == 0).
__device__ __forceinline__ void w4_store_glu(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int tn, int wm, int wn,
                                             int l16, int hq, bf16_t *region) {
    const int lane = hq * 16 + l16;
    // first half: gate (blocks 0..3) to columns 0..63 of the wave's LDS region, up (blocks 4..7) to 64..127
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        bf16_t *lp = region + (i * 16 + l16) * W4_EP_PITCH + hq * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            *reinterpret_cast<uint2 *>(lp + j * 16) = uint2{pack2bf(acc[i][j][0], acc[i][j][1]), pack2bf(acc[i][j][2], acc[i][j][3])};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // second half, row-wise: a lane takes 8 consecutive columns of a row, 8 rows per pass
    const int lr = lane >> 3, lc = (lane & 7) * 8;
    const int col = tn * 128 + wn * 64 + lc;
    bf16_t *cw = reinterpret_cast<bf16_t *>(g.C);
#pragma unroll 4
    for (int it = 0; it < 16; ++it) {
        const int r = it * 8 + lr;
        const int64_t row = m0 + wm * 128 + r;
        if (row >= g.M) continue;
        const uint4 gv = *reinterpret_cast<const uint4 *>(region + r * W4_EP_PITCH + lc);
        const uint4 uv = *reinterpret_cast<const uint4 *>(region + r * W4_EP_PITCH + 64 + lc);
        if (cw) {
            *reinterpret_cast<uint4 *>(cw + row * g.ldc + col) = gv;
            *reinterpret_cast<uint4 *>(cw + row * g.ldc + g.glu_F + col) = uv;
        }
        const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w}, uw[4] = {uv.x, uv.y, uv.z, uv.w};
        uint32_t sw[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float g0 = bflo(gw[k]), g1 = bfhi(gw[k]);
            sw[k] = pack2bf(g0 * sigmoid_rcp(g0) * bflo(uw[k]), g1 * sigmoid_rcp(g1) * bfhi(uw[k]));
        }
        *reinterpret_cast<uint4 *>(g.glu_out + row * g.ld_glu + col) = uint4{sw[0], sw[1], sw[2], sw[3]};
    }
}

// SwiGLU backward store (g.glu_bwd_*): the accumulators are ds; they go to the wave's LDS region as bf16, and the
// row-wise second half reads 8 consecutive ds per lane, loads the forward's gate and up of the same elements
// (16 bytes each) and stores dgate and dup, all as whole lines.  Rows >= M and column chunks >= N are skipped.
__device__ __forceinline__ void w4_store_glu_bwd(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm,
                                                 int wn, int l16, int hq, bf16_t *region) {
    const int lane = hq * 16 + l16;
    const int lr = lane >> 4, lc = (lane & 15) * 8;
    const int col = n0 + wn * 128 + lc;
    const bool col_ok = col < g.N;
    // The forward's gate and up values come from memory, a microsecond or two away.  The loads of the first kDepth
    // row passes are issued before the accumulators are converted (the k-loop's fragment registers are free by now),
    // each later pass is requested when the pass kDepth before it has been consumed, so the second half never waits
    // for a load it has only just issued.  Rows past M re-read row M - 1 (never stored).  Measured at the 7B shape:
    // depth 2: 5.48 ms, 4: 5.43, 6: 5.44, 8: 5.46, 12: 5.51, 16: 5.6, 32: 5.7 (loads issued on demand, 4 at a
    // time: 5.93): beyond a few passes the requests only queue up behind the chip-wide burst of every tile's store.
    constexpr int kDepth = 4;
    uint4 gq[kDepth], uq[kDepth];
    const bf16_t *gu = g.glu_bwd_gu + (col_ok ? col : 0);
    const int64_t row0 = m0 + wm * 128 + lr;
#pragma unroll
    for (int it = 0; it < kDepth; ++it) {
        const int64_t row = min(row0 + it * 4, (int64_t)g.M - 1);
        gq[it] = *reinterpret_cast<const uint4 *>(gu + row * g.ld_glu_bwd);
        uq[it] = *reinterpret_cast<const uint4 *>(gu + row * g.ld_glu_bwd + g.N);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        bf16_t *lp = region + (i * 16 + l16) * W4_EP_PITCH + hq * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            *reinterpret_cast<uint2 *>(lp + j * 16) = uint2{pack2bf(acc[i][j][0], acc[i][j][1]), pack2bf(acc[i][j][2], acc[i][j][3])};
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    bf16_t *C = reinterpret_cast<bf16_t *>(g.C);
#pragma unroll
    for (int it = 0; it < 32; ++it) {
        const int r = it * 4 + lr;
        const int64_t row = m0 + wm * 128 + r;
        const uint4 dv = *reinterpret_cast<const uint4 *>(region + r * W4_EP_PITCH + lc);
        const uint4 gv = gq[it % kDepth], uv = uq[it % kDepth];
        if (it + kDepth < 32) {
            const int64_t nrow = min(row0 + (it + kDepth) * 4, (int64_t)g.M - 1);
            gq[it % kDepth] = *reinterpret_cast<const uint4 *>(gu + nrow * g.ld_glu_bwd);
            uq[it % kDepth] = *reinterpret_cast<const uint4 *>(gu + nrow * g.ld_glu_bwd + g.N);
        }
        const uint32_t dw[4] = {dv.x, dv.y, dv.z, dv.w}, gw[4] = {gv.x, gv.y, gv.z, gv.w}, uw[4] = {uv.x, uv.y, uv.z, uv.w};
        uint32_t og[4], ou[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float a0, b0, a1, b1;
            swiglu_bwd_elem(bflo(dw[k]), bflo(gw[k]), bflo(uw[k]), &a0, &b0);
            swiglu_bwd_elem(bfhi(dw[k]), bfhi(gw[k]), bfhi(uw[k]), &a1, &b1);
            og[k] = pack2bf(a0, a1);
            ou[k] = pack2bf(b0, b1);
        }
        if (col_ok && row < g.M) {
            *reinterpret_cast<uint4 *>(C + row * g.ldc + col) = uint4{og[0], og[1], og[2], og[3]};
            *reinterpret_cast<uint4 *>(C + row * g.ldc + g.N + col) = uint4{ou[0], ou[1], ou[2], ou[3]};
        }
    }
}

// The epilogue is a template parameter: one kernel that carries all of them keeps so much guarded store code alive
// that the compiler moves accumulators through scratch memory on the way out (measured: 13-16 us per tile).
enum { EPI_GUARDED_BF16 = 0, EPI_GUARDED_F32 = 10, EPI_FULL_BF16 = 1, EPI_FULL_F32 = 2, EPI_ROPE = 3, EPI_GLU = 4, EPI_GLU_BWD = 5, EPI_FULL_BF16_RES = 6,
       EPI_FULL_BF16_BIAS = 7, EPI_ROPE_BIAS = 8, EPI_QUADS_F32 = 9 };
// region: the wave's private LDS staging block (128 rows of W4_EP_PITCH bf16), free once the k-loop's last barrier has passed
template <int EPI>
__device__ __forceinline__ void w4_epilogue(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int tn, int wm, int wn,
                                            int l16, int hq, bf16_t *region) {
    if constexpr (EPI == EPI_GLU) w4_store_glu(g, acc, m0, tn, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_ROPE) w4_store_rope<false>(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_ROPE_BIAS) w4_store_rope<true>(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_GLU_BWD) w4_store_glu_bwd(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_FULL_BF16) w4_store_full_bf16<false, false>(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_FULL_BF16_RES) w4_store_full_bf16<false, true>(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_FULL_BF16_BIAS) w4_store_full_bf16<true, false>(g, acc, m0, n0, wm, wn, l16, hq, region);
    else if constexpr (EPI == EPI_FULL_F32) w4_store_full_f32(g, acc, m0, n0, wm, wn, l16, hq);
    else if constexpr (EPI == EPI_GUARDED_BF16) w4_store_guarded_bf16(g, acc, m0, n0, wm, wn, l16, hq, region);
    else w4_store_guarded_f32(g, acc, m0, n0, wm, wn, l16, hq);
}
// ---------------------------------------------------------------------------------------------
// The main loop.  Operands go from memory straight into LDS (no staging registers, no LDS store instructions): full
// k-steps of 64, a wave-load fills 8 rows of 128 bytes (whole cache lines per request), two slots of 64 KB
// (A 256 x 64 | B 256 x 64 bf16), chunk c of row r stored at position c ^ ((r >> 1) & 7).
//   step t:  k-slice 0 (32 indices): 64 MFMAs  ||  the 16 LDS reads of slice 1
//            wait for the loads of step t + 1 (all that are in flight) and for the wave's last reads of the slot; barrier
//            k-slice 1: 64 MFMAs  ||  the 16 LDS reads of slice 0 of step t + 1  ||  the 16 loads of step t + 2 into the
//            slot just freed, one per four MFMAs (64 clocks: the path into LDS takes a wave's 1 KB every 16 clocks and
//            four waves share it), which leaves every load at least the 1024 clocks of the next slice 0 to land
// What bounds it is power: the chip clocks down to what its matrix cores, registers and LDS draw.  The 16x16x32 MFMA
// moves a fifth fewer register bytes per multiplication than 32x32x16 (each accumulator is read and written once per 32
// reduction indices instead of 16), and the 2 x 2 zigzag below changes one operand per MFMA: 8192^3 743 us -> 691 (1480 ->
// 1591 TFLOP/s), 4096^3 100 -> 91, 16384 x 11008 x 4096 1074 -> 1014 (boxes differ by 5 %).  The accumulators are updated in place by assembly (mfma16_acc):
// given the builtin, the register allocator renames them, 500 moves per 256 MFMAs (8192^3: 916 us).
constexpr int WE_HALF = 256 * 64 * 2, WE_SLOT = 2 * WE_HALF, WE_ARRAY = 2 * 128 * W4_EP_PITCH * 2;
static_assert(WE_ARRAY >= WE_SLOT, "a slot must fit into two staging blocks");

// MFMAs 4 U .. 4 U + 3 of a slice's 64: the four blocks (2 x 2) number U, walked in zigzag
template <int U>
__device__ __forceinline__ void w4_mfma_group(f32x4 (&acc)[8][8], const bf16x8 (&fr)[16]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = (U >> 2) * 2 + (e >> 1), j0 = (U & 3) * 2 + ((e & 1) ^ (e >> 1)), j = (U >> 2) & 1 ? 7 - j0 : j0;
        mfma16_acc(acc[i][j], fr[8 + j], fr[i]);
    }
}

// TAIL (K % 64 != 0, K > 64): the last, partial k-step is walked first; it goes through registers, chunks at or beyond K as zeros.
// In 256 x 128 tiles (gemm_ring.hip) -> here, us: 16384 x 4096 x 11024 1798 -> 1351, 14080 x 1024 x 14200 601 -> 459, 22016 x 4096 x 3000
// 552 -> 484, 16384 x 4096 x 1416 232 -> 173.
template <int EPI, bool TAIL>
__global__ __launch_bounds__(W4_NT) void gemm_nt_w4e_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    __shared__ __attribute__((aligned(1024))) char sl0[WE_ARRAY];
    __shared__ __attribute__((aligned(1024))) char sl1[WE_ARRAY];
    typedef __attribute__((address_space(3))) void *lptr;
    const int nb = (int)gridDim.x;   // all tiles, or the first rounds of them
    int pid = blockIdx.x;
    {
        const int q = nb / kXcd, r = nb % kXcd, x = pid % kXcd;
        pid = x * q + (x < r ? x : r) + pid / kXcd;
    }
    int tm, tn;
    gemm_tile_of(pid, tiles_m, tiles_n, g.group_m, &tm, &tn);
    const int m0 = tm * W4_BM, n0 = tn * W4_BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, hq = lane >> 4;

    // loader: wave w fills rows 64 w .. 64 w + 63 of the A half and of the B half of a slot, 8 rows per load;
    // lane l delivers to chunk position l & 7 of row l >> 3 and fetches the chunk that belongs there
    constexpr bool glu = EPI == EPI_GLU;
    const bf16_t *abase = g.A + (int64_t)m0 * g.lda;
    const bf16_t *bbase = g.B + (glu ? 0 : (int64_t)n0 * g.ldb);
    uint32_t off[16];   // byte offsets from abase (0..7) / bbase (8..15)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = wave * 64 + j * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((r >> 1) & 7);
        off[j] = (uint32_t)(min(r, g.M - 1 - m0) * (int)g.lda + chunk * 8) * 2u;
        // SwiGLU pairing: tile rows in blocks of 64 = gate c.., up c.., gate c+64.., up c+64.. (c = 128 tn)
        const int brow = glu ? ((r >> 6) & 1) * g.glu_F + tn * 128 + ((r >> 7) & 1) * 64 + (r & 63) : min(r, g.N - 1 - n0);
        off[8 + j] = (uint32_t)(brow * (int)g.ldb + chunk * 8) * 2u;
    }
    const uint32_t fill_off = (uint32_t)(wave * 64 * 128);
    // fragment reads: k-chunk 4 ks + hq of row l16 + 16 i sits at chunk position (4 ks + hq) ^ ((l16 >> 1) & 7)
    uint32_t rda[2], rdb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const uint32_t pos = (uint32_t)(((4 * ks + hq) ^ ((l16 >> 1) & 7)) * 16);
        rda[ks] = (uint32_t)((wm * 128 + l16) * 128) + pos;
        rdb[ks] = (uint32_t)(WE_HALF + (wn * 128 + l16) * 128) + pos;
    }
    bf16x8 fr[2][16];   // [set][A block 0..7 | B block 0..7]
    f32x4 acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // One load-to-LDS, written out as assembly: the compiler orders every later LDS read after all earlier builtin
    // load-to-LDS instructions it cannot tell apart (a full vmcnt(0) in front of reads of the other slot), which undoes
    // the overlap; ordering is done by hand instead (WE_WAIT).  M0 carries the wave-uniform LDS address, lane i lands
    // at M0 + 16 i; the global address is the uniform base plus the lane's 32-bit byte offset.  (M0 is a reserved
    // register: the compiler keeps no value in it and sets it itself before any instruction of its own that reads it.)
#define WE_LOAD1(SLOT, J, T)                                                                            \
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"                       \
                 :                                                                                      \
                 : "v"(off[J]), "s"(((J) < 8 ? abase : bbase) + (T) * 64),                              \
                   "s"((uint32_t)(uintptr_t)(lptr)(SLOT) + ((J) < 8 ? 0u : (uint32_t)WE_HALF) + fill_off + ((J) & 7) * 1024u) \
                 : "memory")
#define WE_READ1(SET, SLOT, KS, IDX)                                                                    \
    fr[SET][IDX] = *reinterpret_cast<const bf16x8 *>((SLOT) + ((IDX) < 8 ? rda[KS] : rdb[KS]) + ((IDX) & 7) * 2048)
#define WE_WAIT(N) asm volatile("s_waitcnt vmcnt(" #N ") lgkmcnt(0)\n\ts_barrier" ::: "memory")
    // four MFMAs of slice SET with one fragment read of (RSET, RSLOT, KS) and, if LD, load U of step TL into LSLOT in front;
    // pinned in this order.  The B fragments are read first: the next slice's first four MFMAs need B 0, 1 and A 0, 1.
#define WE_GROUP(SET, RSET, RSLOT, KS, U, LD, LSLOT, TL)                                                \
    {                                                                                                   \
        if (LD) WE_LOAD1(LSLOT, U, TL);                                                                 \
        WE_READ1(RSET, RSLOT, KS, ((U) < 8 ? 8 + (U) : (U) - 8));                                       \
        w4_mfma_group<U>(acc, fr[SET]);                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
#define WE_SLICE(SET, RSET, RSLOT, KS, LD, LSLOT, TL)                                                   \
    {                                                                                                   \
        WE_GROUP(SET, RSET, RSLOT, KS, 0, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 1, LD, LSLOT, TL);   \
        WE_GROUP(SET, RSET, RSLOT, KS, 2, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 3, LD, LSLOT, TL);   \
        WE_GROUP(SET, RSET, RSLOT, KS, 4, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 5, LD, LSLOT, TL);   \
        WE_GROUP(SET, RSET, RSLOT, KS, 6, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 7, LD, LSLOT, TL);   \
        WE_GROUP(SET, RSET, RSLOT, KS, 8, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 9, LD, LSLOT, TL);   \
        WE_GROUP(SET, RSET, RSLOT, KS, 10, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 11, LD, LSLOT, TL); \
        WE_GROUP(SET, RSET, RSLOT, KS, 12, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 13, LD, LSLOT, TL); \
        WE_GROUP(SET, RSET, RSLOT, KS, 14, LD, LSLOT, TL); WE_GROUP(SET, RSET, RSLOT, KS, 15, LD, LSLOT, TL); \
    }
    // step T out of CUR.  Past the end of K the last step is requested again (clamped): the same instruction stream for
    // every step, no branches around the MFMAs; the extra data lands in a free slot and is never read.
#define WE_STEP(CUR, NXT, T)                                                                            \
    {                                                                                                   \
        const int t2_ = at(min((T) + 2, nk - 1));                                                       \
        WE_SLICE(0, 1, CUR, 1, false, CUR, 0);                                                          \
        WE_WAIT(0);                                                                                     \
        WE_SLICE(1, 0, NXT, 0, true, CUR, t2_);                                                         \
    }

    const int nk = (g.K + BK - 1) / BK, start = TAIL ? -1 : gemm_walk_start(tm, nk);
    const auto at = [&](int t) { return t + start - (t + start >= nk ? nk : 0); };   // k-step walked as number t
    {
        const int t0_ = at(0), t1_ = at(min(1, nk - 1));
        u32x4 tv[TAIL ? 16 : 1];
        if constexpr (TAIL) {
            const int kt = (nk - 1) * BK;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int r = wave * 64 + (j & 7) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
                const bool ok = kt + chunk * 8 < g.K;   // otherwise column 0 of the row is read (in bounds) and replaced
                const char *p = reinterpret_cast<const char *>(j < 8 ? abase : bbase) + off[j] + (ok ? kt * 2 : -chunk * 16);
                tv[j] = *reinterpret_cast<const u32x4 *>(p);
                if (!ok) tv[j] = u32x4{0u, 0u, 0u, 0u};
            }
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) WE_LOAD1(sl0, j, t0_);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) WE_LOAD1(sl1, j, t1_);
        if constexpr (TAIL) {
#pragma unroll
            for (int j = 0; j < 16; ++j)
                *reinterpret_cast<u32x4 *>(sl0 + (j < 8 ? 0 : WE_HALF) + fill_off + (j & 7) * 1024 + lane * 16) = tv[j];
        }
    }
    WE_WAIT(16);
#pragma unroll
    for (int u = 0; u < 16; ++u) WE_READ1(0, sl0, 0, u);
    int kt = 0;
    if constexpr (TAIL) __builtin_assume(nk >= 2);   // one path less on which the accumulators could be moved about
    for (; kt + 2 <= nk; kt += 2) {
        WE_STEP(sl0, sl1, kt);
        WE_STEP(sl1, sl0, kt + 1);
    }
    if (kt < nk) {
        WE_STEP(sl0, sl1, kt);
        mfma16_drain();
    }
    WE_WAIT(0);   // the loads requested past the end have landed before the store staging reuses the arrays
#undef WE_LOAD1
#undef WE_READ1
#undef WE_WAIT
#undef WE_GROUP
#undef WE_SLICE
#undef WE_STEP
    mfma16_settle(acc);
    // every wave has passed the last step's barrier, i.e. has read its last fragments: the arrays are free
    bf16_t *region = reinterpret_cast<bf16_t *>((wave < 2 ? sl0 : sl1) + (wave & 1) * (128 * W4_EP_PITCH * 2));
    w4_epilogue<EPI>(g, acc, m0, n0, tn, wm, wn, l16, hq, region);
}

// ---------------------------------------------------------------------------------------------
// The same in tiles of 256 x 32 NB, bf16 results, for grids that 256 x 256 tiles fill badly.  NB = 10: 4096 x 5120 is one round of 256 x 320 and 1.25 of 256 x 256;
// NB = 6: 1000 x 11008 fills 0.91 of a round of 256 x 192 and 0.67 of one of 256 x 256.  4 waves x 128 x 16 NB.  NB = 10 has 80 accumulators, of which 64 lie in
// the accumulation registers and 16 (columns 128 .. 159 of the wave) among the vector registers, where the fragments leave room because a column block's
// fragment is given up before the other slice's are all there (the blocks are walked column by column).  Two slots of 72 (56) KB.  Loads, waits and reads as
// above, spread evenly over a slice's MFMAs.  The results leave in two halves of 64 rows; columns are whole groups of 8.
template <int NB>
struct Wide {
    static constexpr int BN = 32 * NB, A = 256 * 64 * 2, SLOT = A + BN * 64 * 2, COLS = 16 * NB, PITCH = COLS + 8, LB = BN / 32, N = 8 + LB;   // N: loads, and reads, of a wave
    static constexpr int GROUPS = 2 * NB;   // of four MFMAs in a slice
    static_assert(2 * 64 * PITCH * 2 <= SLOT, "two staging blocks in a slot");
};

template <int NB, bool BIAS, bool RES>
__global__ __launch_bounds__(W4_NT) void gemm_nt_wide_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    using W = Wide<NB>;
    constexpr int NA = NB < 8 ? NB : 8, NV = NB - NA;   // column blocks with accumulators of either kind
    __shared__ __attribute__((aligned(1024))) char sl0[W::SLOT];
    __shared__ __attribute__((aligned(1024))) char sl1[W::SLOT];
    typedef __attribute__((address_space(3))) void *lptr;
    int pid = blockIdx.x;
    {
        const int nb = (int)gridDim.x, q = nb / kXcd, r = nb % kXcd, x = pid % kXcd;
        pid = x * q + (x < r ? x : r) + pid / kXcd;
    }
    int tm, tn;
    gemm_tile_of(pid, tiles_m, tiles_n, g.group_m, &tm, &tn);
    const int m0 = tm * W4_BM, n0 = tn * W::BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, hq = lane >> 4;

    // loader: wave w fills rows 64 w .. of the A part and 8 LB w .. of the B part of a slot, 8 rows per load; rows past the edge re-read the last one
    const bf16_t *abase = g.A + (int64_t)m0 * g.lda, *bbase = g.B + (int64_t)n0 * g.ldb;
    uint32_t off[W::N];   // byte offsets from abase (0..7) / bbase
#pragma unroll
    for (int j = 0; j < W::N; ++j) {
        const int r = j < 8 ? wave * 64 + j * 8 + (lane >> 3) : wave * (8 * W::LB) + (j - 8) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
        off[j] = (uint32_t)((j < 8 ? min(r, g.M - 1 - m0) * (int)g.lda : min(r, g.N - 1 - n0) * (int)g.ldb) + chunk * 8) * 2u;
    }
    const uint32_t fill_a = (uint32_t)(wave * 64 * 128), fill_b = (uint32_t)(W::A + wave * 8 * W::LB * 128);
    uint32_t rda[2], rdb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const uint32_t pos = (uint32_t)(((4 * ks + hq) ^ ((l16 >> 1) & 7)) * 16);
        rda[ks] = (uint32_t)((wm * 128 + l16) * 128) + pos;
        rdb[ks] = (uint32_t)(W::A + (wn * W::COLS + l16) * 128) + pos;
    }
    bf16x8 fr[2][W::N];   // [set][A block 0..7 | B blocks]
    f32x4 acc[8][NA], accv[8][NV > 0 ? NV : 1];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < NA; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NV; ++j) accv[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const auto load = [&](const char *slot, int j, int t) {   // (as assembly, ordered by hand: see gemm_nt_w4e_kernel)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(off[j]), "s"((j < 8 ? abase : bbase) + t * 64),
                       "s"((uint32_t)(uintptr_t)(lptr)slot + (j < 8 ? fill_a + j * 1024u : fill_b + (j - 8) * 1024u))
                     : "memory");
    };
    const auto read = [&](auto set, const char *slot, int ks, int f) {
        fr[set()][f] = *reinterpret_cast<const bf16x8 *>(slot + (f < 8 ? rda[ks] + f * 2048 : rdb[ks] + (f - 8) * 2048));
    };
#define WX_WAIT(N) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory")
    // the products of the slice in `set`, the reads of the next one (out of rslot) and, with lslot, the loads of step t into it
    const auto slice = [&](auto set, const char *rslot, int ks, auto loads, const char *lslot, int t) {
        constexpr int C = set();
#pragma unroll
        for (int u = 0; u < W::GROUPS; ++u) {
#pragma unroll
            for (int f = u * W::N / W::GROUPS; f < (u + 1) * W::N / W::GROUPS; ++f) {
                if constexpr (loads()) load(lslot, f, t);
                read(std::integral_constant<int, 1 - C>(), rslot, ks, f);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 4 * u + e, j = m / 8, i = j & 1 ? 7 - m % 8 : m % 8;
                if (j < NA) mfma16_acc(acc[i][j < NA ? j : 0], fr[C][8 + j], fr[C][i]);
                else mfma16_acc_v(accv[i][j < NA ? 0 : j - NA], fr[C][8 + j], fr[C][i]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};
    const int nk = g.K / BK, start = gemm_walk_start(tm, nk);
    const auto at = [&](int t) { return t + start - (t + start >= nk ? nk : 0); };   // k-step walked as number t
    const auto step = [&](const char *cur, const char *nxt, int t) {
        slice(first, cur, 1, std::false_type(), cur, 0);
        WX_WAIT(0);
        slice(second, nxt, 0, std::true_type(), cur, at(min(t + 2, nk - 1)));
    };
#pragma unroll
    for (int j = 0; j < W::N; ++j) load(sl0, j, at(0));
#pragma unroll
    for (int j = 0; j < W::N; ++j) load(sl1, j, at(min(1, nk - 1)));
    WX_WAIT(W::N);
#pragma unroll
    for (int f = 0; f < W::N; ++f) read(first, sl0, 0, f);
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
        step(sl0, sl1, kt);
        step(sl1, sl0, kt + 1);
    }
    if (kt < nk) {
        step(sl0, sl1, kt);
        mfma16_drain();
    }
    WX_WAIT(0);   // the loads requested past the end have landed before the store staging reuses the arrays
#undef WX_WAIT
    mfma16_settle(acc);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < NV; ++j) asm volatile("" : "+v"(accv[i][j]));

    bf16_t *region = reinterpret_cast<bf16_t *>((wave < 2 ? sl0 : sl1) + (wave & 1) * (64 * W::PITCH * 2));
    const int col_w = n0 + wn * W::COLS, row_w = m0 + wm * 128, col_l = col_w + hq * 4;
    uint2 bv[BIAS ? NB : 1];   // (columns past the last ones re-read these and are not stored)
    if constexpr (BIAS) {
#pragma unroll
        for (int j = 0; j < NB; ++j) bv[j] = *reinterpret_cast<const uint2 *>(g.bias + min(col_l + j * 16, g.N - 4));
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = half * 4 + k;
            bf16_t *lp = region + (k * 16 + l16) * W::PITCH + hq * 4;
            uint2 rv[RES ? NB : 1];
            if constexpr (RES) {
                const bf16_t *rp = g.R + (int64_t)min(row_w + i * 16 + l16, g.M - 1) * g.ldr;
#pragma unroll
                for (int j = 0; j < NB; ++j) rv[j] = *reinterpret_cast<const uint2 *>(rp + min(col_l + j * 16, g.N - 4));
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                f32x4 v = j < NA ? acc[i][j < NA ? j : 0] : accv[i][j < NA ? 0 : j - NA];
                if constexpr (BIAS) {
                    v[0] += bflo(bv[j].x); v[1] += bfhi(bv[j].x); v[2] += bflo(bv[j].y); v[3] += bfhi(bv[j].y);
                }
                if constexpr (RES) {
                    v[0] += bflo(rv[j].x); v[1] += bfhi(rv[j].x); v[2] += bflo(rv[j].y); v[3] += bfhi(rv[j].y);
                }
                *reinterpret_cast<uint2 *>(lp + j * 16) = uint2{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own LDS writes have landed
        bf16_t *C = reinterpret_cast<bf16_t *>(g.C) + (int64_t)(row_w + half * 64) * g.ldc + col_w;
        constexpr int LPR = 2 * NB;   // lanes of a row
#pragma unroll 5
        for (int it = 0; it < LPR; ++it) {
            const int at16 = it * 64 + lane, r = at16 / LPR, c = at16 % LPR * 8;
            if (row_w + half * 64 + r < g.M && col_w + c < g.N)
                *reinterpret_cast<uint4 *>(C + r * g.ldc + c) = *reinterpret_cast<const uint4 *>(region + r * W::PITCH + c);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // and its reads
    }
}

// MT_GROUP_M (diagnostics): forces the tile-row group of the large-grid kernels
int group_m_override() {
    static const int v = [] {
        const char *e = getenv("MT_GROUP_M");
        return e ? atoi(e) : 0;
    }();
    return v;
}

// every column tile complete and every access of the store aligned: the vector stores (rows are guarded)
bool whole_line_store(const GemmArgs &g) {
    return g.N % W4_BN == 0 && !(g.ldc & 7) && !((uintptr_t)g.C & 15) &&
           (!g.R || (!(g.ldr & 3) && !((uintptr_t)g.R & 7))) && !((uintptr_t)g.bias & 7) && !(g.bias && g.R);
}

// n_tiles > 0: only that many tiles of the tile order
template <int EPI>
hipError_t launch_w4e_epi(const GemmArgs &g, hipStream_t s, int n_tiles = 0) {
    const int tiles_m = (g.M + W4_BM - 1) / W4_BM, tiles_n = EPI == EPI_GLU ? g.glu_F / 128 : (g.N + W4_BN - 1) / W4_BN;
    auto kernel = gemm_nt_w4e_kernel<EPI, false>;
    // (the fused stores take whole k-steps only)
    if constexpr (EPI == EPI_GUARDED_BF16 || EPI == EPI_GUARDED_F32 || EPI == EPI_FULL_BF16 || EPI == EPI_FULL_F32 || EPI == EPI_FULL_BF16_RES || EPI == EPI_FULL_BF16_BIAS)
        if (g.K % BK) kernel = gemm_nt_w4e_kernel<EPI, true>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_tiles > 0 ? n_tiles : tiles_m * tiles_n)), dim3(W4_NT), 0, s, g, tiles_m, tiles_n);
    return hipGetLastError();
}

bool takes_wide(const GemmArgs &g) {
    return g.K % BK == 0 && g.N % 8 == 0 && !g.out_fp32 && !(g.ldc & 7) && !((uintptr_t)g.C & 15) && (!g.R || (!(g.ldr & 3) && !((uintptr_t)g.R & 7))) &&
           !((uintptr_t)g.bias & 7) && !(g.bias && g.R);
}
template <int NB>
hipError_t launch_wide(const GemmArgs &g, hipStream_t s) {
    const int tiles_m = (g.M + W4_BM - 1) / W4_BM, tiles_n = (g.N + 32 * NB - 1) / (32 * NB);
    const auto kernel = g.R ? gemm_nt_wide_kernel<NB, false, true> : g.bias ? gemm_nt_wide_kernel<NB, true, false> : gemm_nt_wide_kernel<NB, false, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(W4_NT), 0, s, g, tiles_m, tiles_n);
    return hipGetLastError();
}

hipError_t launch_w4e(const GemmArgs &g, hipStream_t s, int n_tiles = 0) {
    if (g.glu_F > 0) return launch_w4e_epi<EPI_GLU>(g, s);
    if (g.rope_cos) return g.bias ? launch_w4e_epi<EPI_ROPE_BIAS>(g, s) : launch_w4e_epi<EPI_ROPE>(g, s);
    if (g.glu_bwd_gu) return launch_w4e_epi<EPI_GLU_BWD>(g, s);
    if (!whole_line_store(g)) return g.out_fp32 ? launch_w4e_epi<EPI_GUARDED_F32>(g, s, n_tiles) : launch_w4e_epi<EPI_GUARDED_BF16>(g, s, n_tiles);
    if (g.out_fp32) return launch_w4e_epi<EPI_FULL_F32>(g, s, n_tiles);
    if (g.R) return launch_w4e_epi<EPI_FULL_BF16_RES>(g, s, n_tiles);
    return g.bias ? launch_w4e_epi<EPI_FULL_BF16_BIAS>(g, s, n_tiles) : launch_w4e_epi<EPI_FULL_BF16>(g, s, n_tiles);
}

// ---------------------------------------------------------------------------------------------
// Weight-gradient form: C[M,N] = sum_k At[k][m] Bt[k][n] with both operands token-major ([K, M] and [K, N]),
// i.e. dW = dY^T X straight from the activations as the other kernels produce them.  Same tile, waves, loads and
// schedule as gemm_nt_w4e_kernel; the LDS slots are A [64 k][256 m] | B [64 k][256 n] bf16 (rows of 512 bytes, unpadded), a
// wave-load fills two k rows, and the MFMA operands are read with ds_read_b64_tr_b16, which hands a lane four reduction
// indices of one output row: two reads per fragment.  A read instruction touches rows 8 q + 0..3 (and + 4 in the second
// one), 32 bytes each; the 32-byte column group c of k row r is stored at group position c ^ tn_swz(r), which puts the
// eight rows that half a wave reads together on disjoint banks.  fp32 output only.
constexpr int WT_HALF = 64 * 256 * 2, WT_SLOT = 2 * WT_HALF;
__device__ __forceinline__ int tn_swz(int r) { return ((r & 3) << 1) | ((r >> 3) & 1); }

// fp32 store of a tile with aligned rows.  FULL: complete column tiles, otherwise whole groups of four columns (N is a multiple of
// 8).  What it adds to is requested four row blocks (of 8 loads) ahead; rows and columns past the edge re-read the last ones.  One
// instruction stream with and without accumulation (sums that start at +0 stay what they are when +0 is added): two would
// both keep the accumulators alive, and the compiler then copies all of them out and spills.
template <bool FULL>
__device__ __forceinline__ void tn_store(const GemmArgs &g, const f32x4 (&acc)[8][8], int m0, int n0, int wm, int wn, int l16, int hq) {
    constexpr int AHEAD = 4;
    const int row_l = m0 + wm * 128 + l16, col_l = n0 + wn * 128 + hq * 4;
    float *C = reinterpret_cast<float *>(g.C);
    f32x4 c[AHEAD][8];
    const auto fetch = [&](int i) {
        int row = min(row_l + i * 16, g.M - 1);
        asm volatile("" : "+v"(row));   // addresses are worked out here, not kept in registers during the walk
        const float *cp = C + (int64_t)row * g.ldc;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            c[i % AHEAD][j] = *reinterpret_cast<const f32x4 *>(cp + (FULL ? col_l + j * 16 : min(col_l + j * 16, g.N - 4)));
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (g.accumulate) fetch(i);
        else
#pragma unroll
            for (int j = 0; j < 8; ++j) c[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        int row = row_l + i * 16;
        asm volatile("" : "+v"(row));
        float *cp = C + (int64_t)row * g.ldc + col_l;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            f32x4 v = acc[i][j];
            asm volatile("" : "+a"(v));   // leaves the accumulation registers here, not with all the others in front
            v += c[i % AHEAD][j];
            if (row < g.M && (FULL || col_l + j * 16 < g.N)) *reinterpret_cast<f32x4 *>(cp + j * 16) = v;
        }
        __builtin_amdgcn_sched_barrier(0);
        if (i + AHEAD < 8 && g.accumulate) fetch(i + AHEAD);
    }
}

template <int EPI>
__global__ __launch_bounds__(W4_NT) void gemm_tn_w4e_kernel(GemmArgs g, int tiles_m, int tiles_n, int n_whole, int sums, int sums_tail) {
    __shared__ __attribute__((aligned(1024))) char sl0[WT_SLOT];
    __shared__ __attribute__((aligned(1024))) char sl1[WT_SLOT];
    typedef __attribute__((address_space(3))) void *lptr;
    typedef __attribute__((address_space(3))) s16x4 *trptr;
    constexpr int BM = W4_BM, BN = W4_BN;
    // Split reduction.  The first n_whole tiles walk the whole reduction.  The others (those of the last, partial round, if any)
    // have a workgroup for each of split_k chunks; these units are ordered chunk-major, so the workgroups running together
    // still form tile patches that walk the same K range; chunk 0 owns C, the others a slice of the workspace.  Either kind is
    // summed in pieces (sums of them, sums_tail in a chunk) that are added to C or the slice one after the other.
    const int n_tail = tiles_m * tiles_n - n_whole;
    const bool whole = (int)blockIdx.x < n_whole;
    int pid = blockIdx.x - (whole ? 0 : n_whole), chunk = 0;
    {
        const int nb = whole ? n_whole : n_tail * g.split_k;
        const int q = nb / kXcd, r = nb % kXcd, x = pid % kXcd;
        pid = x * q + (x < r ? x : r) + pid / kXcd;
    }
    if (!whole) {
        chunk = pid / n_tail;
        pid += n_whole - chunk * n_tail;
    }
    const int pieces = whole ? sums : g.split_k * sums_tail;
    int piece = whole ? 0 : chunk * sums_tail;
    const int piece_end = piece + (whole ? sums : sums_tail);
    const int nk_all = g.K / BK;
    if (chunk > 0) {
        g.C = g.split_ws + (int64_t)(chunk - 1) * g.M * g.N;
        g.ldc = g.N;
        g.accumulate = 0;
    }
    int tm, tn;
    gemm_tile_of(pid, tiles_m, tiles_n, g.group_m, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, hq = lane >> 4;

    // loader: wave w fills k rows 16 w .. 16 w + 15 of the A half and of the B half of a slot, two rows per load;
    // lane l delivers to the 16-byte position l & 31 of row l >> 5 and fetches the chunk that belongs there.
    // Chunks past the matrix edge re-read the last chunk; they only feed outputs that are never stored.
    const bf16_t *abase, *bbase;   // first k row of the piece
    uint32_t off[16];   // byte offsets from abase (0..7) / bbase (8..15)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = wave * 16 + j * 2 + (lane >> 5);
        const int c16 = ((((lane & 31) >> 1) ^ tn_swz(r)) << 1) | (lane & 1);
        off[j] = (uint32_t)(r * (int)g.lda + min(m0 + c16 * 8, g.M - 8)) * 2u;
        off[8 + j] = (uint32_t)(r * (int)g.ldb + min(n0 + c16 * 8, g.N - 8)) * 2u;
    }
    const uint32_t fill_off = (uint32_t)(wave * 16 * 512);
    // transposing fragment reads: lane (hq, i = l16) supplies k row 8 hq + (i >> 2) of the slice (and that row + 4), columns
    // (i & 3) * 4 .. + 3 of the block's 16; block b of the wave's quadrant is column group 8 wm + b (A) or 8 wn + b (B)
    uint32_t rd[16];
    {
        const int row = hq * 8 + (l16 >> 2), inner = (l16 & 3) * 8;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            rd[b] = (uint32_t)(row * 512 + ((wm * 8 + b) ^ tn_swz(row)) * 32 + inner);
            rd[8 + b] = (uint32_t)(WT_HALF + row * 512 + ((wn * 8 + b) ^ tn_swz(row)) * 32 + inner);
        }
    }
    bf16x8 fr[2][16];
    f32x4 acc[8][8];

    // one load-to-LDS as assembly, ordered by hand (see gemm_nt_w4e_kernel); a k-step advances both operands by 64 rows
#define WT_LOAD1(SLOT, J, T)                                                                            \
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"                       \
                 :                                                                                      \
                 : "v"(off[J]), "s"((J) < 8 ? abase + (int64_t)(T) * BK * g.lda : bbase + (int64_t)(T) * BK * g.ldb), \
                   "s"((uint32_t)(uintptr_t)(lptr)(SLOT) + ((J) < 8 ? 0u : (uint32_t)WT_HALF) + fill_off + ((J) & 7) * 1024u) \
                 : "memory")
#define WT_READ1(SET, SLOT, KS, IDX)                                                                    \
    {                                                                                                   \
        const s16x4 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)((SLOT) + rd[IDX] + (KS) * 16384));        \
        const s16x4 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)((SLOT) + rd[IDX] + (KS) * 16384 + 2048)); \
        typedef __attribute__((ext_vector_type(8))) short s16x8_;                                       \
        const s16x8_ v_ = {lo_[0], lo_[1], lo_[2], lo_[3], hi_[0], hi_[1], hi_[2], hi_[3]};             \
        fr[SET][IDX] = __builtin_bit_cast(bf16x8, v_);                                                  \
    }
#define WT_WAIT(N) asm volatile("s_waitcnt vmcnt(" #N ") lgkmcnt(0)\n\ts_barrier" ::: "memory")
#define WT_GROUP(SET, RSET, RSLOT, KS, U, LD, LSLOT, TL)                                                \
    {                                                                                                   \
        if (LD) WT_LOAD1(LSLOT, U, TL);                                                                 \
        WT_READ1(RSET, RSLOT, KS, ((U) < 8 ? 8 + (U) : (U) - 8));                                       \
        w4_mfma_group<U>(acc, fr[SET]);                                                                 \
        __builtin_amdgcn_sched_barrier(0);                                                              \
    }
#define WT_SLICE(SET, RSET, RSLOT, KS, LD, LSLOT, TL)                                                   \
    {                                                                                                   \
        WT_GROUP(SET, RSET, RSLOT, KS, 0, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 1, LD, LSLOT, TL);   \
        WT_GROUP(SET, RSET, RSLOT, KS, 2, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 3, LD, LSLOT, TL);   \
        WT_GROUP(SET, RSET, RSLOT, KS, 4, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 5, LD, LSLOT, TL);   \
        WT_GROUP(SET, RSET, RSLOT, KS, 6, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 7, LD, LSLOT, TL);   \
        WT_GROUP(SET, RSET, RSLOT, KS, 8, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 9, LD, LSLOT, TL);   \
        WT_GROUP(SET, RSET, RSLOT, KS, 10, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 11, LD, LSLOT, TL); \
        WT_GROUP(SET, RSET, RSLOT, KS, 12, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 13, LD, LSLOT, TL); \
        WT_GROUP(SET, RSET, RSLOT, KS, 14, LD, LSLOT, TL); WT_GROUP(SET, RSET, RSLOT, KS, 15, LD, LSLOT, TL); \
    }
#define WT_STEP(CUR, NXT, T)                                                                            \
    {                                                                                                   \
        const int t2_ = min((T) + 2, nk - 1);                                                           \
        WT_SLICE(0, 1, CUR, 1, false, CUR, 0);                                                          \
        WT_WAIT(0);                                                                                     \
        WT_SLICE(1, 0, NXT, 0, true, CUR, t2_);                                                         \
    }

    int nk;
    // a piece's first two steps are requested; the slots are free: the barrier that ended the piece before lies behind every read
#define WT_BEGIN()                                                                                      \
    {                                                                                                   \
        const int kb_ = (int)((int64_t)piece * nk_all / pieces);                                        \
        nk = (int)((int64_t)(piece + 1) * nk_all / pieces) - kb_;                                       \
        abase = g.A + (int64_t)kb_ * BK * g.lda;                                                        \
        bbase = g.B + (int64_t)kb_ * BK * g.ldb;                                                        \
        const int t1_ = min(1, nk - 1);                                                                 \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) WT_LOAD1(sl0, j, 0);                             \
        _Pragma("unroll") for (int j = 0; j < 16; ++j) WT_LOAD1(sl1, j, t1_);                           \
    }
    WT_BEGIN();
    for (;;) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        WT_WAIT(16);   // (the stores of the piece before are younger than these loads and may be waited for as well)
#pragma unroll
        for (int u = 0; u < 16; ++u) WT_READ1(0, sl0, 0, u);
        int kt = 0;
        for (; kt + 2 <= nk; kt += 2) {
            WT_STEP(sl0, sl1, kt);
            WT_STEP(sl1, sl0, kt + 1);
        }
        if (kt < nk) {
            WT_STEP(sl0, sl1, kt);
            mfma16_drain();
        }
        WT_WAIT(0);
        mfma16_settle(acc);
        const bool more = EPI != EPI_GUARDED_F32 && ++piece < piece_end;   // (a split has aligned rows)
        if (more) WT_BEGIN();   // their flight covers the store
        if constexpr (EPI == EPI_GUARDED_F32) w4_store_guarded_f32(g, acc, m0, n0, wm, wn, l16, hq);
        else tn_store<EPI == EPI_FULL_F32>(g, acc, m0, n0, wm, wn, l16, hq);
        if (!more) break;
        g.accumulate = 1;
    }
#undef WT_BEGIN
#undef WT_LOAD1
#undef WT_READ1
#undef WT_WAIT
#undef WT_GROUP
#undef WT_SLICE
#undef WT_STEP
}

// C (pitch ldc) += ws[0] + ws[1] + ... (n_ws slices of M x N floats, pitch N), added in that order
__global__ __launch_bounds__(256) void split_reduce_kernel(float *C, int64_t ldc, const float *ws, int n_ws, int M, int N) {
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4, total = (int64_t)M * N;
    if (idx >= total) return;
    const int64_t row = idx / N;
    const int col = (int)(idx % N);
    f32x4 v = *reinterpret_cast<const f32x4 *>(C + row * ldc + col);
    for (int k = 0; k < n_ws; ++k) v += *reinterpret_cast<const f32x4 *>(ws + (int64_t)k * total + idx);
    *reinterpret_cast<f32x4 *>(C + row * ldc + col) = v;
}
// the same for the tiles from position `first` of the tile order on; a block takes 32 rows of a tile (a wave a whole row)
__global__ __launch_bounds__(256) void split_reduce_tiles_kernel(float *C, int64_t ldc, const float *ws, int n_ws, int M, int N,
                                                                 int first, int tiles_m, int tiles_n, int group_m) {
    int tm, tn;
    gemm_tile_of(first + blockIdx.x / 8, tiles_m, tiles_n, group_m, &tm, &tn);
    const int64_t total = (int64_t)M * N;
    const int col = tn * W4_BN + (threadIdx.x & 63) * 4;
    if (col >= N) return;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int64_t row = tm * W4_BM + (blockIdx.x & 7) * 32 + it * 4 + (threadIdx.x >> 6);
        if (row >= M) return;
        f32x4 v = *reinterpret_cast<const f32x4 *>(C + row * ldc + col);
        for (int k = 0; k < n_ws; ++k) v += *reinterpret_cast<const f32x4 *>(ws + k * total + row * N + col);
        *reinterpret_cast<f32x4 *>(C + row * ldc + col) = v;
    }
}

int variant_override() {
    static int v = [] {
        const char *e = getenv("MT_GEMM_VARIANT");
        return e ? atoi(e) : 0;
    }();
    return v;
}

}  // namespace

// The fused stores exist in the 256 x 256 kernel only, for whole k-steps.  They are taken from 192 tiles on: below, the separate pass over a
// small result costs less than the idle compute units.
static bool takes_w4(const GemmArgs &g) {
    const int64_t big_tiles = (int64_t)((g.M + 255) / 256) * ((g.N + 255) / 256);
    const int v = variant_override();
    return g.K % BK == 0 && (v == 6 || (v == 0 && big_tiles >= 192));
}

// Which tile takes a problem: the one with the smallest estimated time.  A kernel with one workgroup per compute unit
// runs rounds of n_cu tiles; a stage of 64 reduction indices costs `part` us when few compute units are busy and
// `full` us when all are (shared bandwidth, lower clock), in between with the square of the share; a tile costs
// `fixed` us on top (first loads, store).  The two smallest tiles share a compute unit (two and three workgroups): per
// tile and compute unit `full` us a stage, but never less than a lone one's `part`.  All figures measured at
// K = 1000 .. 11008 and 16 .. 1600 tiles; the estimates came out within 10 % where rows are whole cache lines.  NT in us,
// this kernel against the 256 x 256 / 128 x 128 register-staged one it replaced:
//   1000 x 2048 x 11008  57 (128 x 64) : 130      1024 x 1024 x 3000  17 (64 x 64) : 47
//   3000 x 1024 x 1024   11 (64 x 64) : 20        4096 x 5120 x 5120  183 (256 x 128) : 201 (256 x 256: 1.25 rounds)
//   1000 x 11008 x 2048  46 (256 x 256, 172 tiles) : 77
struct TileCost {
    RingTile tile;
    int bm, bn, per_cu;
    double part, full, fixed, fixed_shared;
};
static const TileCost kNtCosts[] = {{RingTile::none, 256, 256, 1, 0.95, 1.30, 9.0, 0.0},
                                    {RingTile::t256x128, 256, 128, 1, 0.53, 0.79, 5.0, 0.0},
                                    {RingTile::t128x128, 128, 128, 1, 0.36, 0.43, 3.2, 0.0},
                                    {RingTile::t128x64, 128, 64, 2, 0.33, 0.275, 2.0, 1.2},
                                    {RingTile::t64x64, 64, 64, 3, 0.26, 0.18, 2.0, 0.5}};
static const TileCost kTnCosts[] = {{RingTile::none, 256, 256, 1, 0.90, 1.46, 10.0, 0.0},
                                    {RingTile::t256x128, 256, 128, 1, 0.50, 0.84, 5.0, 0.0},
                                    {RingTile::t128x128, 128, 128, 1, 0.42, 0.47, 3.0, 0.0},
                                    {RingTile::t128x64, 128, 64, 2, 0.34, 0.29, 2.0, 1.2},
                                    {RingTile::t64x64, 64, 64, 3, 0.23, 0.175, 2.0, 0.4}};
constexpr int kComputeUnits = 256;

static double tile_count(const TileCost &c, int64_t M, int64_t N) {
    return (double)((M + c.bm - 1) / c.bm) * (double)((N + c.bn - 1) / c.bn);
}
static double tile_time(const TileCost &c, double tiles, double stages, int n_cu) {
    if (c.per_cu > 1) {
        const double per = std::ceil(tiles / n_cu);
        return std::max(stages * c.part + c.fixed, per * (stages * c.full + c.fixed_shared));
    }
    const double rounds = std::floor(tiles / n_cu), share = (tiles - rounds * n_cu) / n_cu;
    return rounds * (stages * c.full + c.fixed) +
           (share > 0 ? stages * (c.part + (c.full - c.part) * share * share) + c.fixed : 0.0);
}
// How many partial sums every output of a weight gradient is made of at the least.  A long chain of fp32 additions loses
// precision, so this number never falls below that of the plainest split there is, all 256 x 256 tiles into the same number of
// workgroups, where it pays by a model of its own: a k-step 1.65 us, the reduction 3.5 TB/s, a gain of 4 %.  Relative error
// against 64 bits for normal data in that many sums and in one: 2048 x 1024 x 16384 3.2e-7 (6 sums) and 8.2e-7, 7168 x 5120 x 32768
// 5.1e-7 (5) and 1.2e-6.
static int tn_partial_sums(int64_t M, int64_t N, int64_t K, int n_cu) {
    const int64_t tiles = ((M + W4_BM - 1) / W4_BM) * ((N + W4_BN - 1) / W4_BN), nk = K / BK;
    int best = 1;
    double best_t = 0.0;
    for (int sp = 1; sp <= 6 && nk / sp >= 32; ++sp) {
        const double t = (double)((tiles * sp + n_cu - 1) / n_cu) * (double)nk / sp * 1.65e-6 +
                         (sp > 1 ? (sp + 1) * 4.0 * (double)M * (double)N / 3.5e12 : 0.0);
        if (sp == 1) best_t = 0.96 * t;
        else if (t < best_t) {
            best_t = t;
            best = sp;
        }
    }
    return best;
}

// Weight gradient with its reduction split.  The 256 x 256 kernel leaves the tiles of the last round to a workgroup per chunk, or
// walks the whole reduction of every tile in one workgroup; the others have a workgroup per chunk for every tile.  Partial
// results in the workspace are read and added at about 3.5 TB/s, by a launch of its own (3 us).  Every unit makes as many
// partial sums as its precision asks for (an unsplit product of 256 x 256 tiles a single one: its caller chose that).
// A round of 256 x 256 tiles adds a further partial sum to C in 28 us, a single one, which finds C in the memory-side cache, in 16.
constexpr double kPiece = 28.0, kPieceAlone = 16.0;
struct TnRoute { double time; int n_whole, sums, sums_tail; };
static TnRoute tn_big_route(const TileCost &c, int64_t M, int64_t N, double stages, int split, int sums, int n_cu) {
    const double tiles = tile_count(c, M, N), full = std::floor(tiles / kRound) * kRound, cut = tiles - full;
    const int sums_tail = (sums + split - 1) / split;
    const TnRoute whole = {tile_time(c, tiles, stages, n_cu) + (sums - 1) * (tiles == n_cu ? kPieceAlone : std::ceil(tiles / n_cu) * kPiece),
                           (int)tiles, sums, 1};
    if (split == 1 || cut == 0.0) return whole;
    const TnRoute tail = {tile_time(c, full, stages, n_cu) + (sums - 1) * (full == n_cu ? kPieceAlone : full / n_cu * kPiece) +
                              tile_time(c, cut * split, stages / split, n_cu) + (sums_tail - 1) * std::ceil(cut * split / n_cu) * kPieceAlone + 3.0 +
                              (split + 1) * 4.0 * cut * c.bm * c.bn / 3.5e6, (int)full, sums, sums_tail};
    return tail.time < whole.time ? tail : whole;
}
static double tn_time(const TileCost &c, int64_t M, int64_t N, double stages, int split, int n_cu) {
    if (c.tile == RingTile::none)
        return tn_big_route(c, M, N, stages, split, split == 1 ? 1 : tn_partial_sums(M, N, (int64_t)stages * BK, n_cu), n_cu).time;
    const double t = tile_time(c, tile_count(c, M, N) * split, stages / split, n_cu);
    if (split == 1) return t;
    // the tiles that share a compute unit gain nothing from a split: 184 x 4248 x 13312 in five 54 us (256 x 128 tiles in six: 37),
    // 1952 x 200 x 2048 in four 12.3 (unsplit 9.0); their estimate carries the unsplit walk of a tile once more
    return t + 3.0 + (split + 1) * 4.0 * (double)M * (double)N / 3.5e6 + (c.per_cu > 1 ? stages * c.part + c.fixed : 0.0);
}

// The 256 x 256 kernel's guarded stores (ragged columns, unaligned rows) cost this much more per tile: in fp32, and element by element,
// they write partial lines.
constexpr double kGuardedStore = 14.0, kGuardedRows = 2.0;
static double guarded_store(const GemmArgs &g) {
    const bool rows = !g.out_fp32 && !(g.ldc & 3) && !((uintptr_t)g.C & 7) && (!g.R || (!(g.ldr & 3) && !((uintptr_t)g.R & 7)));
    return whole_line_store(g) ? 0.0 : rows ? kGuardedRows : kGuardedStore;
}

template <int N_COSTS>
static const TileCost &choose_tile(const TileCost (&costs)[N_COSTS], int64_t M, int64_t N, int64_t K, int split) {
    const double stages = (double)((K + BK - 1) / BK);
    const int first = K < BK ? 1 : 0;   // the 256 x 256 kernel takes a whole stage at least
    const TileCost *best = &costs[first];
    double best_t = tn_time(*best, M, N, stages, split, kComputeUnits);
    for (int i = first + 1; i < N_COSTS; ++i) {
        const double t = tn_time(costs[i], M, N, stages, split, kComputeUnits);
        if (t < 0.97 * best_t) {
            best = &costs[i];
            best_t = t;
        }
    }
    return *best;
}

bool gemm_nt_fuses_rope(const GemmArgs &g) {
    return g.M > 0 && g.N > 0 && g.K > 0 && takes_w4(g) && !g.out_fp32 && !g.R && g.rope_T > 0 && (g.N % 128) == 0 &&
           (g.rope_cols % 128) == 0 && g.rope_cols <= g.N && !(g.ldc & 7) && !((uintptr_t)g.C & 15) &&
           !((uintptr_t)g.bias & 7) && g.rope_cos && g.rope_sin && !((uintptr_t)g.rope_cos & 15) &&
           !((uintptr_t)g.rope_sin & 15);
}

bool gemm_nt_fuses_glu(const GemmArgs &g) {
    return g.M > 0 && g.K > 0 && g.glu_F > 0 && g.N == 2 * g.glu_F && (g.glu_F % 128) == 0 && takes_w4(g) && !g.out_fp32 &&
           !g.R && !g.bias && !g.rope_cos && !g.rope_sin && g.glu_out && !(g.ld_glu & 7) && g.ld_glu >= g.glu_F &&
           !((uintptr_t)g.glu_out & 15) && (!g.C || (!(g.ldc & 7) && !((uintptr_t)g.C & 15))) &&
           (int64_t)g.N * g.ldb < ((int64_t)1 << 31);
}

bool gemm_nt_fuses_glu_bwd(const GemmArgs &g) {
    return g.M > 0 && g.N > 0 && g.K > 0 && (g.N & 7) == 0 && takes_w4(g) && !g.out_fp32 && !g.R && !g.bias && !g.rope_cos &&
           !g.rope_sin && !g.glu_F && !g.glu_out && g.glu_bwd_gu && g.C && !(g.ldc & 7) && g.ldc >= 2 * (int64_t)g.N &&
           !((uintptr_t)g.C & 15) && !(g.ld_glu_bwd & 7) && g.ld_glu_bwd >= 2 * (int64_t)g.N &&
           !((uintptr_t)g.glu_bwd_gu & 15);
}

// Small grids with a long reduction: the waves of a workgroup share it (share_nt_kernel).  Measured, like the kernels it is compared with, on 600 shapes
// (128 .. 8192 rows and columns, K 512 .. 20 000, up to 900 tiles of 64 x 64) with operands that come from memory; the estimates of the table above, of
// operands in the caches, are 1.4 times too low there (two workgroups of 128 x 64 tiles on a compute unit: 1.7).  Taken from less of that on, 1.3 and 1.6 times
// the other estimate, the choice is within 0.4 % of the best on average and nowhere more than 5 % behind the other kernels (240 x 3232 x 832), 1.34 times
// faster than they over all shapes and up to 2.7 times.  At least a stage for every wave, 128 x 64 tiles with four waves eight: 4040 x 304 x 1152, 18
// stages, 11.0 -> 12.9 us, but 4472 x 336 x 3520 28.9 -> 26.5.
// From operands in the caches it gains less: of 2400 shapes those with estimates of 0.9 to 1 took 0.96 of the other kernels' time from memory and 1.08 from the
// caches (0.8 to 0.9: 0.88 and 0.99; 0.5 to 0.7: 0.72 and 0.92), so the line lies at 0.9; with more than 8192 columns, where those of 0.8 to 1 (325 shapes)
// took 0.99 and 1.03, at 0.8.
// Beyond 8192 rows, where it was not fitted, sharing gains nothing (500 shapes of up to 600 columns: 1.00 on average, up to 1.19 times slower: 41 236 x 8 x 7664
// 177 -> 203 us); beyond 8192 columns it does in one round of tiles (348 shapes 0.95; more than 256 tiles 1.01, 29 x 16 848 x 4608 66 -> 74).  So
// the products that a fused store takes too (192 tiles of 256 x 256 or more, i.e. over 700 here) are one chain of additions by either route.
// fp32 results over whole stages stay one chain of additions: they are what the precision of a split weight gradient is measured against
// (those that need speed, weight gradients of ragged token counts, have a partial stage).
struct ShareCost { TileCost cost; int waves, stages; double from_memory; };
static const ShareCost kShareCosts[] = {{{RingTile::s32x32, 32, 32, 1, 0.122, 0.122, 2.7, 0.0}, 8, 8, 1.3},
                                        {{RingTile::s32x64, 32, 64, 1, 0.176, 0.184, 3.07, 0.0}, 8, 8, 1.3},
                                        {{RingTile::s64x64, 64, 64, 1, 0.242, 0.268, 3.5, 0.0}, 4, 8, 1.3},
                                        {{RingTile::s128x64, 128, 64, 1, 0.371, 0.419, 4.89, 0.0}, 4, 32, 1.6}};
constexpr int kShareTiles = 600, kShareSide = 8192;
static const ShareCost *share_tile(const GemmArgs &g, const TileCost &other) {
    if ((g.out_fp32 && g.K % BK == 0) || g.M > kShareSide) return nullptr;
    const int most = g.N > kShareSide ? kComputeUnits : kShareTiles;
    const double stages = (double)((g.K + BK - 1) / BK), other_t = tn_time(other, g.M, g.N, stages, 1, kComputeUnits);
    double best = g.N > kShareSide ? 0.8 : 0.9;
    const ShareCost *tile = nullptr;
    for (const ShareCost &c : kShareCosts) {
        const double tiles = tile_count(c.cost, g.M, g.N), t = tile_time(c.cost, tiles, stages, kComputeUnits) / (c.from_memory * other_t);
        if (g.K / BK >= c.stages && tiles <= most && t < best) {
            tile = &c;
            best = t;
        }
    }
    return tile;
}
// Some rows of a product whose reduction is shared: tiles with as many waves, the cheapest for these rows, sum them in the same order.
static const TileCost *share_part(const GemmArgs &g, const ShareCost &whole) {
    const double stages = (double)((g.K + BK - 1) / BK);
    const TileCost *tile = &whole.cost;
    for (const ShareCost &c : kShareCosts)
        if (c.waves == whole.waves && g.K / BK >= c.stages &&
            tile_time(c.cost, tile_count(c.cost, g.M, g.N), stages, kComputeUnits) < tile_time(*tile, tile_count(*tile, g.M, g.N), stages, kComputeUnits))
            tile = &c.cost;
    return tile;
}

// Rows that are not whole lines: the kernels above ask for most lines twice, those that fetch whole lines (line_nt_kernel) for each once, with tiles of at
// most 128 x 128.  Share of an operand's rows whose pieces of 128 bytes touch two lines:
static double straddling_rows(const bf16_t *p, int64_t ld) {
    const int q = (int)(ld / 8 & 7);
    return q == 0 ? ((uintptr_t)p & 127 ? 1.0 : 0.0) : q == 4 ? 0.5 : q & 1 ? 0.875 : 0.75;
}
// Such stages take 1 + kStraddle times that share longer (K % 64 = 32: 1.20, 16 and 48: 1.32, odd multiples of 8: 1.38 measured on 2000 x 1024 x 2816 ..
// 4096 x 4096 x 14 976).  Fitted, with the line kernels' figures, to 420 shapes of down and weight-gradient products, heads and their gradients (K 128 ..
// 24 000, operands from memory, compared with the kernels that the rules above choose), so that the choice is nowhere more than 1 % slower than without line
// kernels.  us: 2048 x 2048 x 10 008 138 -> 97, 2000 x 2048 x 5528 66 -> 54, 1024 x 2816 x 3000 32.5 -> 25.7; in a chain of products, where operands come
// from the caches, less: the MLP of 512 tokens, 4160 x 12 400, forward 259 -> 231, a head of 3008 tokens, 640 x 1080 49.8 -> 47.8, most others even.  Products
// that 256 x 256 tiles take keep them: they would gain up to 1.3 times alone (5120 x 2048 x 4008 139 -> 108) and lose 1 % in a chain under the power
// limit (the projections of 2 x 1480 tokens, 3136 wide, 922 -> 931 us).  A shared reduction stays shared.
constexpr double kStraddle = 0.40;
constexpr int kLineStages = 10;   // (they start later: 256 x 256 x 472 4.9 us, 5.2 with them)
static const TileCost kLineCosts[] = {{RingTile::l128x128, 128, 128, 1, 0.40, 0.48, 4.0, 0.0},
                                      {RingTile::l128x64, 128, 64, 1, 0.30, 0.28, 2.7, 0.0},
                                      {RingTile::l64x64, 64, 64, 2, 0.22, 0.175, 3.0, 0.9}};

// Tiles of 256 x 320 (widths that are multiples of 320) and of 256 x 192 (of 64).  Fitted to 263 plain products of MLPs, projections and heads (K 512 .. 15 000,
// half a round to eight): taken from an estimated gain of 3 and 4 % on, 1.013 times faster over all of them.  us, before ->
// here: 4096 x 5120 x 5120 (one round of 256 x 320 instead of 1.25) 155 -> 143, x 7168 210 -> 194, x 27 648 897 -> 774, 8192 x 2560 x 2560 89 -> 80, 65 536 x 5120 x 5120
// (16 rounds instead of 20) 2524 -> 2452, x 13 824 6523 -> 6283 (1477 TFLOP/s); the projections of 5 x 512
// tokens, 3712 wide, forward (of which 2560 x 3712 x 3712 in 0.78 of a round of 256 x 192) 291 -> 269; among products that run at the power limit even;
// 2000 x 5120 x 5120 (half a round) 94, in 256 x 320 115, and 8200 x 2560 x 6400 (1.03 rounds) 213, 301, keep theirs.
// The kernel takes any width of whole groups of 8.  Other widths, by the same estimate but alone, operands from memory: 256 x 320 where N % 64 == 0 1.02 to 1.36 times faster
// (24 products, 1.14 on average: 4152 x 4672 x 2304 93 -> 74 us), any N 1.01 to 1.27 (12, 1.09), 256 x 192 with any N 1.08 to 1.26 (8, 1.15).  They keep their
// tiles: among the other products of a block, at the power limit, that has not been measured.
constexpr int kWideStages = 8;   // (shorter walks were not looked at)
static const TileCost kWideCosts[] = {{RingTile::wide320, 256, 320, 1, 1.03, 1.545, 12.5, 0.0}, {RingTile::wide192, 256, 192, 1, 0.55, 1.09, 9.8, 0.0}};

// What takes an NT product without a fused store: the first `whole` tiles of 256 x 256 in the tile order the kernel above, the others
// that of `tile` (null: there are none).
struct NtRoute { int whole; const TileCost *tile; };
static NtRoute nt_route(const GemmArgs &g, int32_t of_rows = 0) {
    const double stages = (double)((g.K + BK - 1) / BK);
    const double straddle = g.K % BK && g.K >= kLineStages * BK ? 1.0 + kStraddle * 0.5 * (straddling_rows(g.A, g.lda) + straddling_rows(g.B, g.ldb)) : 1.0;
    TileCost costs[sizeof kNtCosts / sizeof kNtCosts[0]];
    std::copy(std::begin(kNtCosts), std::end(kNtCosts), costs);
    costs[0].fixed += guarded_store(g);
    const TileCost &one = choose_tile(costs, g.M, g.N, g.K, 1);
    if (of_rows > g.M) {
        GemmArgs whole = g;
        whole.M = of_rows;
        if (const ShareCost *share = share_tile(whole, choose_tile(costs, whole.M, g.N, g.K, 1))) return {0, share_part(g, *share)};
    } else if (const ShareCost *share = share_tile(g, one)) {
        return {0, &share->cost};
    }
    // Or the full rounds of 256 x 256 tiles, and what is left in smaller ones that fill the chip (a launch of its own: 3 us).
    // 4096 x 5120 x 5120 (1.25 rounds) 204 -> 179 us; x 7168 253 -> 212; 3000 x 5632 x 1024 (1.03)
    // 50 -> 37; 12000 x 3072 x 3072 (2.2) 186 -> 162; 4096 x 7168 x 5120 (1.75) keeps its 208.
    const double tiles = tile_count(costs[0], g.M, g.N);
    const int whole = (int)(std::floor(tiles / kRound) * kRound), rest = (int)tiles - whole;
    NtRoute route = one.tile == RingTile::none ? NtRoute{(int)tiles, nullptr} : NtRoute{0, &kNtCosts[&one - costs]};
    double route_t = tn_time(one, g.M, g.N, stages, 1, kComputeUnits);
    if (g.K >= BK && whole > 0 && rest > 0) {
        double best_t = 0.97 * route_t;
        for (int i = 1; i < (int)std::size(kNtCosts); ++i) {
            const TileCost &c = kNtCosts[i];
            const double t = tile_time(costs[0], whole, stages, kComputeUnits) + 3.0 +
                             tile_time(c, (double)rest * (256 / c.bm) * (256 / c.bn), stages, kComputeUnits);
            if (t < best_t) {
                best_t = route_t = t;
                route = {whole, &c};
            }
        }
    }
    if (takes_wide(g) && stages >= kWideStages) {
        const TileCost *wide = nullptr;
        double best_t = route_t;
        for (const TileCost &c : kWideCosts) {
            const double t = tile_time(c, tile_count(c, g.M, g.N), stages, kComputeUnits);
            if (t < best_t && g.N % (c.bn == 320 ? 320 : 64) == 0 && t < (c.bn == 320 ? 0.97 : 0.96) * route_t) {
                best_t = t;
                wide = &c;
            }
        }
        if (wide) return {0, wide};
    }
    if (straddle > 1.0 && route.whole == 0) {
        double best_t = 0.92 * tn_time(one, g.M, g.N, stages * straddle, 1, kComputeUnits);
        for (const TileCost &c : kLineCosts) {
            const double t = tn_time(c, g.M, g.N, stages, 1, kComputeUnits);
            if (t < best_t) {
                best_t = t;
                route = {0, &c};
            }
        }
    }
    return route;
}

hipError_t gemm_nt(const GemmArgs &g0, hipStream_t s, int32_t of_rows) {
    GemmArgs g = g0;
    if (group_m_override() > 0) g.group_m = group_m_override();
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
    if (g.glu_bwd_gu && !gemm_nt_fuses_glu_bwd(g)) return hipErrorNotSupported;
    if ((g.rope_cos || g.rope_sin) && !gemm_nt_fuses_rope(g)) return hipErrorNotSupported;
    if ((g.glu_F || g.glu_out) && !gemm_nt_fuses_glu(g)) return hipErrorNotSupported;
    if (!g.C && !g.glu_F) return hipErrorInvalidValue;
    if ((g.K & 7) || (g.lda & 7) || (g.ldb & 7)) return hipErrorInvalidValue;
    if (((uintptr_t)g.A & 15) || ((uintptr_t)g.B & 15)) return hipErrorInvalidValue;
    if (g.lda < g.K || g.ldb < g.K || (g.C && g.ldc < g.N)) return hipErrorInvalidValue;
    if (g.R && (g.out_fp32 || g.ldr < g.N)) return hipErrorInvalidValue;
    if (g.bias && g.out_fp32) return hipErrorInvalidValue;
    // offsets inside one tile are 32-bit: 256 rows of A, and the 320 of B that the widest tile has, must stay below 2^31 elements
    if (g.lda >= (1 << 22) || g.ldb >= (1 << 22)) return hipErrorInvalidValue;
    if (g.rope_cos || g.glu_F || g.glu_bwd_gu) return launch_w4e(g, s);
    switch (variant_override()) {   // diagnostic override (MT_GEMM_VARIANT), 0 = the estimate
        case 2: return gemm_nt_ring(g, RingTile::t256x128, -1, s);
        case 3: return gemm_nt_ring(g, RingTile::t128x128, -1, s);
        case 6: if (g.K >= BK) return launch_w4e(g, s); break;          // 256 x 256 kernel on any grid
        case 7: if (takes_wide(g)) return launch_wide<10>(g, s); break;   // 256 x 320
        case 8: if (takes_wide(g)) return launch_wide<6>(g, s); break;    // 256 x 192
        default: break;
    }
    const NtRoute r = nt_route(g, of_rows);
    if (r.whole == 0)
        return r.tile->tile == RingTile::wide320 ? launch_wide<10>(g, s) : r.tile->tile == RingTile::wide192 ? launch_wide<6>(g, s) : gemm_nt_ring(g, r.tile->tile, -1, s);
    const hipError_t e = launch_w4e(g, s, r.whole);
    return e == hipSuccess && r.tile ? gemm_nt_ring(g, r.tile->tile, r.whole, s) : e;
}

void gemm_nt_route(const GemmArgs &g, int *whole, int *tile_m, int *tile_n) {
    const NtRoute r = nt_route(g);
    *whole = r.whole;
    *tile_m = r.tile ? r.tile->bm : 0;
    *tile_n = r.tile ? r.tile->bn : 0;
}
int gemm_nt_sharers(const GemmArgs &g) {
    const NtRoute r = nt_route(g);
    for (const ShareCost &c : kShareCosts)
        if (r.tile && c.cost.tile == r.tile->tile) return c.waves;
    return 1;
}
bool gemm_nt_fetches_lines(const GemmArgs &g) {
    const TileCost *tile = nt_route(g).tile;
    return tile >= std::begin(kLineCosts) && tile < std::end(kLineCosts);
}

int gemm_tn_pick_split(int64_t M, int64_t N, int64_t K, int n_cu) {
    if (M <= 0 || N <= 0 || K < BK || n_cu <= 0) return 1;
    const int64_t nk = K / BK;
    const int sums = tn_partial_sums(M, N, K, n_cu);
    // A split has to win by 1.5 % in the estimate, a finer one by another 1 % (27648 x 5120 x 16384, 8.4 rounds: 1.8 % estimated, 3506 ->
    // 3325 us measured).  22016 x 4096 x 16384 (5.4 rounds of 256 x 256 tiles): unsplit 2301 us, the last round in two 2123 (all tiles
    // in two: 2394); 7168 x 5120 x 4096 (2.2 rounds) 258, in three 228.  With as many partial sums in the full rounds as the size asks
    // for: 7168 x 5120 x 32768 (five) 1902 (a workgroup per chunk everywhere: 2081), 5128 x 4096 x 8192 (three) 300 (374),
    // 11008 x 2048 x 16384 (two) 568 (657).
    int best = 0;
    double best_t = 0.0;
    for (int sp = 1; sp <= 6; ++sp) {
        const TileCost &c = choose_tile(kTnCosts, M, N, K, sp);   // what gemm_tn will take
        const bool big = c.tile == RingTile::none;
        if (sp > 1 ? nk / sp < (big ? 16 : 8) : big && sums > 1) continue;
        const double t = tn_time(c, M, N, (double)nk, sp, n_cu);
        if (best == 0 || t < (best == 1 ? 0.985 : 0.99) * best_t) {
            best_t = t;
            best = sp;
        }
    }
    return std::max(best, 1);
}

template <int EPI>
static hipError_t launch_tn_epi(const GemmArgs &g0, const TnRoute &route, hipStream_t s) {
    GemmArgs g = g0;
    if (group_m_override() > 0) g.group_m = group_m_override();
    const int tiles_m = (g.M + W4_BM - 1) / W4_BM, tiles_n = (g.N + W4_BN - 1) / W4_BN, n_tail = tiles_m * tiles_n - route.n_whole;
    hipLaunchKernelGGL(gemm_tn_w4e_kernel<EPI>, dim3((unsigned)(route.n_whole + n_tail * g.split_k)), dim3(W4_NT), 0, s, g, tiles_m, tiles_n,
                       route.n_whole, route.sums, route.sums_tail);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_tail == 0) return e;
    hipLaunchKernelGGL(split_reduce_tiles_kernel, dim3((unsigned)n_tail * 8), dim3(256), 0, s, reinterpret_cast<float *>(g.C), g.ldc,
                       g.split_ws, g.split_k - 1, g.M, g.N, route.n_whole, tiles_m, tiles_n, g.group_m);
    return hipGetLastError();
}

// A split of the caller's own (any but the one that gemm_tn_pick_split returns) is taken at its word: that many partial sums of
// every output, also of the tiles that have one workgroup.  22016 x 4096 x 16384 in four: relative error against 64 bits 4.0e-7 (one chain in the
// full rounds: 8.0e-7), 2545 us.
static int tn_sums_of_split(const GemmArgs &g) {
    if (g.split_k == 1) return 1;
    const int sums = tn_partial_sums(g.M, g.N, g.K, kComputeUnits);
    return g.split_k == gemm_tn_pick_split(g.M, g.N, g.K, kComputeUnits) ? sums : std::max(sums, g.split_k);
}

static hipError_t launch_tn(const GemmArgs &g, hipStream_t s) {
    const TnRoute route = tn_big_route(kTnCosts[0], g.M, g.N, g.K / BK, g.split_k, tn_sums_of_split(g), kComputeUnits);
    if ((g.ldc & 3) || ((uintptr_t)g.C & 15)) return launch_tn_epi<EPI_GUARDED_F32>(g, route, s);   // (unsplit then)
    return g.N % W4_BN == 0 ? launch_tn_epi<EPI_FULL_F32>(g, route, s) : launch_tn_epi<EPI_QUADS_F32>(g, route, s);
}

hipError_t gemm_tn(const GemmArgs &g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
    if ((g.lda & 7) || (g.ldb & 7) || ((uintptr_t)g.A & 15) || ((uintptr_t)g.B & 15)) return hipErrorInvalidValue;
    if (g.lda < g.M || g.ldb < g.N || g.ldc < g.N || !g.out_fp32 || g.R || g.bias || g.rope_cos || g.rope_sin || g.glu_F ||
        g.glu_out || g.glu_bwd_gu)
        return hipErrorInvalidValue;
    if ((g.K % BK) || (g.M & 7) || (g.N & 7)) return hipErrorNotSupported;
    if (g.split_k < 1 || g.split_k > g.K / BK) return hipErrorInvalidValue;
    // the reduction of a split reads and writes C four floats at a time
    if (g.split_k > 1 && (!g.split_ws || ((uintptr_t)g.split_ws & 15) || (g.ldc & 3) || (g.N & 3) || ((uintptr_t)g.C & 15)))
        return hipErrorInvalidValue;
    const int v = variant_override();
    const RingTile tile = v == 6 ? RingTile::none : v == 2 ? RingTile::t256x128 : v == 3 ? RingTile::t128x128
                                                                                                   : choose_tile(kTnCosts, g.M, g.N, g.K, g.split_k).tile;
    if (tile == RingTile::none) return launch_tn(g, s);
    const hipError_t e = gemm_tn_ring(g, tile, tn_partial_sums(g.M, g.N, g.K, kComputeUnits), s);
    if (e != hipSuccess || g.split_k == 1) return e;
    const int64_t quads = ((int64_t)g.M * g.N + 3) / 4;
    hipLaunchKernelGGL(split_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, reinterpret_cast<float *>(g.C),
                       g.ldc, g.split_ws, g.split_k - 1, g.M, g.N);
    return hipGetLastError();
}

void gemm_tn_route(const GemmArgs &g, int *whole, int *tile_m, int *tile_n) {
    const TileCost &c = choose_tile(kTnCosts, g.M, g.N, g.K, g.split_k);
    *whole = c.tile == RingTile::none ? tn_big_route(c, g.M, g.N, g.K / BK, g.split_k, tn_sums_of_split(g), kComputeUnits).n_whole : 0;
    *tile_m = c.bm;
    *tile_n = c.bn;
}

}  // namespace mt
