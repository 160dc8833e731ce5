// HBM-bound kernels of the transformer block: transpose, RMSNorm, rotary embedding,
// SwiGLU, embedding gather / scatter, cross-entropy and a fixed-order sum.
//
// All of them move 16 bytes per lane per access (8 bf16 or 4 fp32), do their
// arithmetic in fp32 and reduce inside a 64-lane wave with cross-lane shuffles.
// None uses atomics, so every result is bit-reproducible from run to run.
#include <algorithm>
#include <type_traits>
#include <atomic>

#include "common.h"

namespace mt {

namespace {

// four floats of a caller's fp32 array, which need not be aligned to more than a float
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void unpack8(const uint4 &u, float *f) {
    f[0] = bflo(u.x); f[1] = bfhi(u.x); f[2] = bflo(u.y); f[3] = bfhi(u.y);
    f[4] = bflo(u.z); f[5] = bfhi(u.z); f[6] = bflo(u.w); f[7] = bfhi(u.w);
}
__device__ __forceinline__ uint4 pack8(const float *f) {
    uint4 u;
    u.x = pack2bf(f[0], f[1]); u.y = pack2bf(f[2], f[3]); u.z = pack2bf(f[4], f[5]); u.w = pack2bf(f[6], f[7]);
    return u;
}

// ------------------------------------------------------------------ transpose
// HBM-bound.  A block moves 128 rows x 64 columns through LDS and reads them back with the transposing load: two of them give a
// lane eight consecutive rows of its column, so a store instruction writes 64 bytes to each of 16 output rows and a block
// whole 256-byte pieces.  Against 16-bit LDS reads and 16 bytes to each of 64 rows: 4096 x 11008 37.3 -> 28.9 us (6.2 TB/s),
// 2048 x 5504 15.3 -> 8.8, 1000 x 11008 12.1 -> 8.8, 32000 x 4096 125 -> 112.
// LDS rows are 128 bytes; their 32-byte group c of row r sits at group position c ^ transpose_swz(r), which puts the eight rows
// (0 .. 3 and 8 .. 11 of 16) that half a wave reads together on disjoint banks.
constexpr int kTrRows = 128, kTrCols = 64;
__device__ __forceinline__ int transpose_swz(int r) { return (((r >> 1) & 1) << 1) | ((r >> 3) & 1); }
__global__ __launch_bounds__(256) void transpose_kernel(TransposeArgs t) {
    __shared__ __attribute__((aligned(16))) bf16_t tile[kTrRows * kTrCols];
    typedef __attribute__((address_space(3))) s16x4 *trptr;
    const int b0 = blockIdx.z / t.nb1, b1 = blockIdx.z % t.nb1;
    const bf16_t *in = t.in + b0 * t.in_s0 + b1 * t.in_s1;
    bf16_t *out = t.out + b0 * t.out_s0 + b1 * t.out_s1;
    const int r0 = blockIdx.y * kTrRows, c0 = blockIdx.x * kTrCols;
    const int tid = threadIdx.x, c16 = tid & 7, rl = tid >> 3;
    const int cin = min(c0 + c16 * 8, t.cols - 8);   // past the edge: the last chunk or row again, never stored
    uint4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v[j] = *reinterpret_cast<const uint4 *>(in + (int64_t)min(r0 + rl + 32 * j, t.rows - 1) * t.ld_in + cin);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = rl + 32 * j;
        *reinterpret_cast<uint4 *>(tile + r * kTrCols + (((c16 >> 1) ^ transpose_swz(r)) << 4) + (c16 & 1) * 8) = v[j];
    }
    __syncthreads();
    // wave w: columns 16 w .. + 15; lane (g, i) asks for row 8 q + (i >> 2) (and + 4), columns 4 (i & 3) .. + 3, and gets
    // column i of rows 8 q .. + 7, q = g + 4 j
    const int lane = tid & 63, wave = tid >> 6, g = lane >> 4, i = lane & 15;
    bf16_t *op = out + (int64_t)(c0 + wave * 16 + i) * t.ld_out + r0;
    const bool cok = c0 + wave * 16 + i < t.cols;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int q = g + 4 * j, r = 8 * q + (i >> 2);
        const bf16_t *p = tile + r * kTrCols + ((wave ^ transpose_swz(r)) << 4) + (i & 3) * 4;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)(p + 4 * kTrCols));
        if (cok && r0 + 8 * q < t.rows) {
            const uint2 a = __builtin_bit_cast(uint2, lo), b = __builtin_bit_cast(uint2, hi);
            *reinterpret_cast<uint4 *>(op + 8 * q) = uint4{a.x, a.y, b.x, b.y};
        }
    }
}

// NT: past the caches.  For results that the L2 caches (32 MB in all) cannot hold for their reader: the lines written take no place from those read.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
template <bool NT>
__device__ __forceinline__ void norm_store(uint4 *p, const uint4 &v) {
    if constexpr (NT)
        __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
    else
        *p = v;
}

// ------------------------------------------------------------------ RMSNorm forward
// One wave per row; the row is held in registers (NCH chunks of 8 per lane).  PACKED: as it was loaded; otherwise the compiler keeps
// the unpacked row, and fewer waves fit on a SIMD (NCH = 8: five instead of eight).  A launch of few rounds is the faster for more
// waves, one of many for fewer (see rmsnorm_fwd).
template <int NCH, bool PACKED, bool NT>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(bf16_t *y, const bf16_t *x, const bf16_t *gain, int64_t n,
                                                          int d, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // scalar addresses
    if (row >= n) return;
    const int nch = d >> 3;
    const char *xr = reinterpret_cast<const char *>(x + row * d);
    uint4 xv[NCH];
    float ss = 0.f;
    // all loads first and without branches (chunks past the row re-read its last one): under a branch each load would be
    // waited for before the next is issued; 32-bit offsets, or the addresses take as many registers as half the row
#pragma unroll
    for (int i = 0; i < NCH; ++i) xv[i] = *reinterpret_cast<const uint4 *>(xr + 16u * (uint32_t)min(lane + 64 * i, nch - 1));
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        float f[8];
        unpack8(xv[i], f);
        if (lane + 64 * i < nch) {
#pragma unroll
            for (int k = 0; k < 8; ++k) ss += f[k] * f[k];
        }
    }
    ss = wave_sum(ss);
    if constexpr (PACKED) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) asm volatile("" : "+v"(xv[i].x), "+v"(xv[i].y), "+v"(xv[i].z), "+v"(xv[i].w));
    }
    const float r = 1.0f / sqrtf(ss / (float)d + eps);
    const uint4 *gr = reinterpret_cast<const uint4 *>(gain);
    uint4 *yr = reinterpret_cast<uint4 *>(y + row * d);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) {
            float f[8], gf[8];
            unpack8(xv[i], f);
            unpack8(gr[c], gf);
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = f[k] * r * gf[k];
            norm_store<NT>(yr + c, pack8(f));
        }
    }
}

// ------------------------------------------------------------------ RMSNorm backward
// Per row: r and dot = sum_j g_j dy_j x_j, then dx = r g dy - x r^3 dot / d (+ dres).  The gain gradient sum_t dy x r is
// kept in registers per thread and column; every block writes one partial row, a second kernel adds the partial rows.
// HBM-bound: three tensors read, one written, once each.  A row belongs to WPR waves of the block, NCH chunks of 16 bytes
// per thread: one wave up to 1024 elements (with all four waves on a row, half of them would be idle), four beyond, so that
// a row of any width fits the registers next to its gain gradient.  The next row is requested before this one is reduced.
// One wave per row at every width, loads on demand and rows beyond 4096 read twice took (gain-gradient sum included)
// 722 us for 65 536 x 5120, 479 for x 4096, 145 for x 1024; this kernel takes 518, 398 and 102 (5.2 and 5.4 TB/s at the
// first two; a copy reaches 4.9), and since its loads have no branches (selecting zeros for them put the zeros and the
// selected address into scratch memory) 372, 288 and 74 on a box where it took 446, 305 and 79.
// A row of its own per block also makes a thread's chain of additions four times as long: it is cut every 32 rows, so that the
// gain gradient of many rows stays as exact as with a chain per wave (262 144 rows, d = 1032, relative error against 64 bits:
// one chain 4.2e-7, a chain per wave 2.7e-7, cut 1.6e-7).
// The residual's gradient (dres) is requested with its own row where a thread has several chunks, a row ahead like the others where
// it has one: 65 536 x 6144 639 -> 602 us, x 5120 (with dres) 518 -> 488, 45 448 x 6016 427 -> 410; x 2048 stays at 189 (238).
constexpr int kNormBwdBlocks = 512, kNormChain = 32;

template <int NCH, int WPR, bool NT>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(bf16_t *dx, float *partial, const bf16_t *dy, const bf16_t *x,
                                                          const bf16_t *gain, const bf16_t *dres, int64_t n, int d, float eps) {
    static_assert(WPR == 1 || WPR == 4, "a row belongs to one wave or to the whole block");
    constexpr int TPR = 64 * WPR, RPB = 4 / WPR;   // threads per row, rows per block at a time
    __shared__ float red[2][2][4];                 // [parity of the row][sum x^2, dot][wave]
    __shared__ float dgs[8 * TPR * NCH];           // WPR == 1: one set for the four waves; 4: the sums of each thread's ended chains
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tr = threadIdx.x % TPR;
    const int nch = d >> 3;
    float dg[NCH][8];
    uint4 gv[NCH], xn[NCH], yn[NCH], rn[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        gv[i] = reinterpret_cast<const uint4 *>(gain)[min(tr + TPR * i, nch - 1)];
        rn[i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int k = 0; k < 8; ++k) dg[i][k] = 0.f;
    }
    // without branches (chunks past the row re-read its last one and are left out of the sums)
    auto fetch = [&](int64_t row) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int64_t c = row * nch + min(tr + TPR * i, nch - 1);
            xn[i] = reinterpret_cast<const uint4 *>(x)[c];
            yn[i] = reinterpret_cast<const uint4 *>(dy)[c];
        }
    };
    auto fetch_res = [&](int64_t row) {
        if (!dres) return;
#pragma unroll
        for (int i = 0; i < NCH; ++i) rn[i] = reinterpret_cast<const uint4 *>(dres)[row * nch + min(tr + TPR * i, nch - 1)];
    };
    constexpr bool kResAhead = WPR == 1 || NCH == 1;
    const int64_t row0 = (int64_t)blockIdx.x * RPB + (WPR == 1 ? wave : 0), stride = (int64_t)gridDim.x * RPB;
    if (row0 < n) {
        fetch(row0);
        if (kResAhead) fetch_res(row0);
    }
    bool ended = false;
    const auto end_chain = [&]() {   // dg += the chains before
        if (!ended) return;
#pragma unroll
        for (int i = 0; i < NCH; ++i)
#pragma unroll
            for (int k = 0; k < 8; ++k) dg[i][k] = dgs[(i * 8 + k) * TPR + tr] + dg[i][k];
    };
    int par = 0, chain = 0;
    for (int64_t row = row0; row < n; row += stride, par ^= 1) {   // WPR == 4: the same rows in every wave of the block
        if (WPR == 4 && ++chain > kNormChain) {
            end_chain();
#pragma unroll
            for (int i = 0; i < NCH; ++i)
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    dgs[(i * 8 + k) * TPR + tr] = dg[i][k];
                    dg[i][k] = 0.f;
                }
            ended = true;
            chain = 1;
        }
        uint4 xv[NCH], yv[NCH], rv[NCH];
        float ss = 0.f, dot = 0.f;
        if (!kResAhead) fetch_res(row);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            xv[i] = xn[i];
            yv[i] = yn[i];
            if (kResAhead) rv[i] = rn[i];
            float xf[8], yf[8], gf[8];
            unpack8(xv[i], xf);
            unpack8(yv[i], yf);
            unpack8(gv[i], gf);
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                s1 += xf[k] * xf[k];
                s2 += gf[k] * yf[k] * xf[k];
            }
            const bool in_row = tr + TPR * i < nch;
            ss += in_row ? s1 : 0.f;
            dot += in_row ? s2 : 0.f;
        }
        if (row + stride < n) {
            fetch(row + stride);
            if (kResAhead) fetch_res(row + stride);
        }
        ss = wave_sum(ss);
        dot = wave_sum(dot);
        if constexpr (WPR == 4) {
            if (lane == 0) {
                red[par][0][wave] = ss;
                red[par][1][wave] = dot;
            }
            __syncthreads();   // one per row: the other parity's slots are rewritten only after the next row's barrier
            ss = (red[par][0][0] + red[par][0][1]) + (red[par][0][2] + red[par][0][3]);
            dot = (red[par][1][0] + red[par][1][1]) + (red[par][1][2] + red[par][1][3]);
        }
        const float r = 1.0f / sqrtf(ss / (float)d + eps);
        const float cc = r * r * r * dot / (float)d;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = tr + TPR * i;
            float xf[8], yf[8], gf[8], of[8];
            unpack8(xv[i], xf);
            unpack8(yv[i], yf);
            unpack8(gv[i], gf);
            unpack8(kResAhead ? rv[i] : rn[i], of);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                of[k] += r * gf[k] * yf[k] - xf[k] * cc;
                dg[i][k] += yf[k] * xf[k] * r;
            }
            if (c < nch) norm_store<NT>(reinterpret_cast<uint4 *>(dx + row * d) + c, pack8(of));
        }
    }
    if constexpr (WPR == 4) end_chain();
    if constexpr (WPR == 1) {   // the four waves' sums, ((w0 + w1) + w2) + w3
        for (int w = 0; w < 4; ++w) {
            if (wave == w)
#pragma unroll
                for (int i = 0; i < NCH; ++i)
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        float *p = &dgs[(i * 8 + k) * TPR + tr];
                        if (w > 0) dg[i][k] = *p + dg[i][k];
                        *p = dg[i][k];
                    }
            __syncthreads();
        }
        if (wave != 3) return;
    }
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tr + TPR * i;
        if (c < nch) {
            f32x4_a4 *p = reinterpret_cast<f32x4_a4 *>(partial + (int64_t)blockIdx.x * d + c * 8);
            p[0] = f32x4_a4{dg[i][0], dg[i][1], dg[i][2], dg[i][3]};
            p[1] = f32x4_a4{dg[i][4], dg[i][5], dg[i][6], dg[i][7]};
        }
    }
}

// out[j] (+)= sum over rows of partial[r][j].  A block owns 32 columns, four per lane; its RG row groups each add every
// RG-th row in order (at most 4 of the 512 rows that the callers produce: all of them in flight together) and the group
// sums are added in a fixed tree, so the result does not depend on the launch.  Bound by latency, not by the 10 MB:
// 512 x 5120 took 20.6 us with one float per lane and 8 row groups, 5.0 us with 128.  Few rows take fewer groups (the same
// sums: the others would add zeros): less of the chip and fewer barriers.
template <int RG>
__global__ __launch_bounds__(8 * RG) void colsum_kernel(float *out, const float *partial, int nrows, int d, int accumulate) {
    __shared__ f32x4 red[RG][8];
    const int cl = threadIdx.x & 7, rg = threadIdx.x >> 3;
    const int j = blockIdx.x * 32 + cl * 4;   // d is a multiple of 8
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (j < d) {
#pragma unroll 4
        for (int r = rg; r < nrows; r += RG) s += *reinterpret_cast<const f32x4_a4 *>(partial + (int64_t)r * d + j);
    }
    red[rg][cl] = s;
    __syncthreads();
#pragma unroll
    for (int h = RG / 2; h > 0; h >>= 1) {
        if (rg < h) red[rg][cl] += red[rg + h][cl];
        __syncthreads();
    }
    if (rg == 0 && j < d) {
        f32x4_a4 *o = reinterpret_cast<f32x4_a4 *>(out + j);
        *o = accumulate ? *o + red[0][cl] : red[0][cl];
    }
}
void launch_colsum(float *out, const float *partial, int nrows, int d, int accumulate, hipStream_t s) {
    const dim3 grid((unsigned)((d + 31) / 32));
    if (nrows <= 8) hipLaunchKernelGGL(colsum_kernel<8>, grid, dim3(64), 0, s, out, partial, nrows, d, accumulate);
    else if (nrows <= 32) hipLaunchKernelGGL(colsum_kernel<32>, grid, dim3(256), 0, s, out, partial, nrows, d, accumulate);
    else hipLaunchKernelGGL(colsum_kernel<128>, grid, dim3(1024), 0, s, out, partial, nrows, d, accumulate);
}

// ------------------------------------------------------------------ bias gradient (column sums of a bf16 matrix)
// block (bx, by): 16-byte column chunk bx*256 + thread of the rows [by*rpb, (by+1)*rpb) -> partial[by][cols]
constexpr int kBiasGradRowBlocks = 128;
__global__ __launch_bounds__(256) void bias_grad_partial_kernel(float *partial, const bf16_t *x, int64_t ld, int64_t n,
                                                                int cols, int64_t rpb) {
    const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (c >= cols) return;
    const int64_t r0 = (int64_t)blockIdx.y * rpb, r1 = min(n, r0 + rpb);
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int64_t r = r0; r < r1; ++r) {
        const uint4 u = *reinterpret_cast<const uint4 *>(x + r * ld + c);
        a[0] += bflo(u.x); a[1] += bfhi(u.x); a[2] += bflo(u.y); a[3] += bfhi(u.y);
        a[4] += bflo(u.z); a[5] += bfhi(u.z); a[6] += bflo(u.w); a[7] += bfhi(u.w);
    }
    float *p = partial + (int64_t)blockIdx.y * cols + c;
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = a[e];
}

// ------------------------------------------------------------------ rotary embedding
// thread = (row, head, group of 8 pair indices j); pairs (j, j + hd/2)
__global__ __launch_bounds__(256) void rope_kernel(bf16_t *x, int64_t ld, int64_t n, int T, int n_heads, int hd,
                                                   const float *cs, const float *sn, float sign) {
    const int half = hd >> 1, gpr = half >> 3;  // groups per head
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = n * n_heads * gpr;
    if (idx >= total) return;
    const int gi = (int)(idx % gpr);
    const int h = (int)((idx / gpr) % n_heads);
    const int64_t row = idx / ((int64_t)gpr * n_heads);
    const int t = (int)(row % T);
    bf16_t *p = x + row * ld + (int64_t)h * hd + gi * 8;
    uint4 *pa = reinterpret_cast<uint4 *>(p), *pb = reinterpret_cast<uint4 *>(p + half);
    float a[8], b[8];
    unpack8(*pa, a);
    unpack8(*pb, b);
    const float4 *cp = reinterpret_cast<const float4 *>(cs + (int64_t)t * half + gi * 8);
    const float4 *sp = reinterpret_cast<const float4 *>(sn + (int64_t)t * half + gi * 8);
    const float4 c0 = cp[0], c1 = cp[1], s0 = sp[0], s1 = sp[1];
    const float c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    const float s[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    float oa[8], ob[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float sk = sign * s[k];
        oa[k] = a[k] * c[k] - b[k] * sk;
        ob[k] = b[k] * c[k] + a[k] * sk;
    }
    *pa = pack8(oa);
    *pb = pack8(ob);
}

// ------------------------------------------------------------------ SwiGLU
__device__ __forceinline__ float sigmoidf_(float v) { return sigmoid_rcp(v); }

__global__ __launch_bounds__(256) void swiglu_fwd_kernel(bf16_t *sout, const bf16_t *gu, int64_t n, int F) {
    const int cpr = F >> 3;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * cpr) return;
    const int64_t row = idx / cpr;
    const int c = (int)(idx % cpr) * 8;
    float g[8], u[8], o[8];
    unpack8(*reinterpret_cast<const uint4 *>(gu + row * 2 * F + c), g);
    unpack8(*reinterpret_cast<const uint4 *>(gu + row * 2 * F + F + c), u);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = g[k] * sigmoidf_(g[k]) * u[k];
    *reinterpret_cast<uint4 *>(sout + row * F + c) = pack8(o);
}

__global__ __launch_bounds__(256) void swiglu_bwd_kernel(bf16_t *dgu, const bf16_t *ds, const bf16_t *gu, int64_t n,
                                                         int F) {
    const int cpr = F >> 3;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * cpr) return;
    const int64_t row = idx / cpr;
    const int c = (int)(idx % cpr) * 8;
    float g[8], u[8], d[8], og[8], ou[8];
    unpack8(*reinterpret_cast<const uint4 *>(gu + row * 2 * F + c), g);
    unpack8(*reinterpret_cast<const uint4 *>(gu + row * 2 * F + F + c), u);
    unpack8(*reinterpret_cast<const uint4 *>(ds + row * F + c), d);
#pragma unroll
    for (int k = 0; k < 8; ++k) swiglu_bwd_elem(d[k], g[k], u[k], &og[k], &ou[k]);
    *reinterpret_cast<uint4 *>(dgu + row * 2 * F + c) = pack8(og);
    *reinterpret_cast<uint4 *>(dgu + row * 2 * F + F + c) = pack8(ou);
}

// ------------------------------------------------------------------ embedding
__global__ __launch_bounds__(256) void embed_gather_kernel(bf16_t *h, const bf16_t *table, const int32_t *tokens,
                                                           int64_t n, int d) {
    const int cpr = d >> 3;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n * cpr) return;
    const int64_t row = idx / cpr;
    const int c = (int)(idx % cpr);
    reinterpret_cast<uint4 *>(h + row * d)[c] = reinterpret_cast<const uint4 *>(table + (int64_t)tokens[row] * d)[c];
}

// Gradient of the table: row v of dtable = sum of the dh rows listed for token v.  HBM-bound (every dh row read once,
// every table row written once), if the rows of frequent tokens do not become a serial chain: token ids in text follow
// Zipf's law, so at 65 536 tokens one row has some 2000 terms while most have none to three.
// NC blocks of 8 waves share 8 NC rows (x, x + groups, ...: tokenizers give frequent words neighbouring ids) of
// NC x 512 columns.  Rows of up to kScatterShort terms: a wave sums one row in list order over all NC x 512 columns, so
// that the chain row_start -> list -> dh is paid once for 4 KB.  Longer rows: every block sums its own 512 columns with
// all waves, wave w taking the w-th eighth of the list, 16 loads in flight, and the 8 sums are added in wave order.  No
// atomics, a fixed order.
// 65 536 Zipf-distributed tokens, d = 4096, V = 32 000: one block per row with one serial sum 3690 us, this one 239 us with
// scattered ids and 275 us with ids in order of frequency (1.06 GB: 4.45 and 3.86 TB/s; a copy reaches 4.9); uniform tokens
// 219 and 213 us (over three sets of buffers in turn: 326, 327 and 214; with the column ranges side by side and
// whole lines per store ids in order of frequency 269, uniform ones 211; the heaviest rows first 265, 214).  Without sharing (every block its own 512 columns of 8 rows) uniform tokens took 370 us.
constexpr int kScatterWaves = 8, kScatterShort = 32, kScatterHeavy = 256, kScatterLook = 4;

__device__ __forceinline__ void scatter_add(float *a, const uint4 &v) {
    float f[8];
    unpack8(v, f);
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] += f[k];
}
// A lane's 8 sums as fp32.  Lanes 2 k and 2 k + 1 exchange halves, so that the 8 lanes that loaded a line of dh (in the order 0, 4, 1, 5, ..) store a
// whole line each time, past the caches: with 32 bytes per lane every store covered half of each line.  us, before -> here: 16 384 Zipf tokens, 32 000 x
// 4096 193 -> 157, 65 536 tokens, 152 064 x 4096 832 -> 682, 4096 tokens, 16 000 x 768 26 -> 12.5; of these the caches' share 7, 23, 0.
// o: where the lane's first four go, left: columns from there to the end of the row.
template <bool ADD>
__device__ __forceinline__ void scatter_store(float *o, const float *acc, int left) {
    const bool odd = threadIdx.x & 1;
    float a[2][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float give = odd ? acc[k] : acc[4 + k];
        const float got = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(give), 0xb1, 0xf, 0xf, true));   // quad_perm 1, 0, 3, 2
        a[0][k] = odd ? got : acc[k];
        a[1][k] = odd ? acc[4 + k] : got;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (32 * h >= left) return;
        f32x4 *p = reinterpret_cast<f32x4 *>(o + 32 * h), v = {a[h][0], a[h][1], a[h][2], a[h][3]};
        if (ADD) v = *p + v;
        __builtin_nontemporal_store(v, p);
    }
}

// NR terms r[0..NR) of the list, added to acc[j] (columns col + 512 j) in order
template <int NC, int NR>
__device__ __forceinline__ void scatter_terms(float (*acc)[8], const bf16_t *dh, const int32_t *r, int d, int col) {
    uint4 v[NR][NC];
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        const bf16_t *p = dh + (int64_t)r[u] * d + col;
#pragma unroll
        for (int j = 0; j < NC; ++j) v[u][j] = col + 512 * j < d ? *reinterpret_cast<const uint4 *>(p + 512 * j) : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
        for (int j = 0; j < NC; ++j) scatter_add(acc[j], v[u][j]);
}

// ADD: on top of what the table's gradient holds already (rows without a token are then left alone).  SIDE: the blocks come by groups of
// rows, all column ranges of a group side by side; else by column ranges, all groups of one.
template <int NC, bool ADD, bool SIDE>
__global__ __launch_bounds__(64 * kScatterWaves) void embed_scatter_kernel(float *dtable, const bf16_t *dh,
                                                                           const int32_t *row_start, const int32_t *order,
                                                                           int V, int d, int groups, int heavy, int enough) {
    __shared__ float part[kScatterWaves - 1][8][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int bx = SIDE ? blockIdx.z * gridDim.y + blockIdx.y : blockIdx.x / NC, x = bx - heavy, share = blockIdx.x % NC;
    const int gx = groups;
    if (x >= gx) return;
    const int y = SIDE ? (blockIdx.x / NC + bx) % (gridDim.x / NC) : blockIdx.y;   // (turned, so that a narrow last range comes to every XCD)
    const int col0 = y * (512 * NC), col = col0 + (lane >> 3) * 64 + (lane & 1) * 32 + (lane & 6) * 4;   // (what scatter_store wants)
    const int out0 = (lane >> 3) * 64 + (lane & 7) * 4;
    const int c = col + 512 * share;
    // the blocks below heavy sum the longest rows of 64 kScatterLook, before all others, if the list has `enough` terms; the other blocks theirs of a group
    const bool ahead = NC == 4 && heavy > 0 && row_start[V] >= enough;   // (heavy = 0 where NC < 4; unread there, which is 0.1 us of 4)
    if (x < 0 && !ahead) return;
    int first = x >= 0 ? x : bx;
    const int step = x >= 0 ? gx : heavy, n_rows = x >= 0 ? NC * kScatterWaves : 64;
    const int more = x >= 0 ? kScatterShort : kScatterHeavy, most = x >= 0 && ahead ? kScatterHeavy : INT32_MAX;
    // which of these rows are long: one row per lane, so that the usual block does not pay for looking
    int g_beg = 0, g_cnt = 0;
    const auto look = [&]() {
        const int v = first + lane * step;
        g_cnt = 0;
        if (lane < n_rows && v < V) {
            g_beg = row_start[v];
            g_cnt = row_start[v + 1] - g_beg;
        }
    };
    look();
    if (x >= 0) {
        const int v = x + (share * kScatterWaves + wave) * gx;
        if (v < V) {
            const int beg = row_start[v], end = row_start[v + 1];
            if (end - beg <= kScatterShort && (!ADD || beg < end)) {
                float acc[NC][8] = {};
                int i = beg;
                // 8 loads in flight.  16 384 uniform tokens, 1024 x 1024 (NC = 1): two terms at a time whatever NC 10.2 us, here 8.8 (13.5 with stores of half lines)
                for (; i + 8 / NC <= end; i += 8 / NC) scatter_terms<NC, 8 / NC>(acc, dh, order + i, d, col);
                if (NC == 1 && i + 4 <= end) scatter_terms<NC, 4>(acc, dh, order + i, d, col), i += 4;
                if (NC <= 2 && i + 2 <= end) scatter_terms<NC, 2>(acc, dh, order + i, d, col), i += 2;
                if (i < end) scatter_terms<NC, 1>(acc, dh, order + i, d, col);
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    scatter_store<ADD>(dtable + (int64_t)v * d + col0 + out0 + 512 * j, acc[j], d - (col0 + out0 + 512 * j));
            }
        }
    }
    if (col0 + 512 * share >= d) return;   // uniform over the block
    for (int k = 1;; ++k) {
        uint64_t todo = __builtin_amdgcn_ballot_w64(g_cnt > more && g_cnt <= most);
        for (; todo; todo &= todo - 1) {   // the same in every wave
            const int w = __builtin_ctzll(todo), v = first + w * step;
            const int beg = __builtin_amdgcn_readlane(g_beg, w), cnt = __builtin_amdgcn_readlane(g_cnt, w);
            const int i0 = beg + (int)((int64_t)cnt * wave / kScatterWaves), i1 = beg + (int)((int64_t)cnt * (wave + 1) / kScatterWaves);
            float acc[1][8] = {};
            for (int ib = i0; ib < i1; ib += 64) {
                const int idx = order[min(ib + lane, i1 - 1)], m = min(64, i1 - ib);   // the next 64 terms, one per lane
                int i = 0;
                for (; i + 16 <= m; i += 16) {
                    int32_t r[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) r[u] = __builtin_amdgcn_readlane(idx, i + u);
                    scatter_terms<1, 16>(acc, dh, r, d, c);
                }
                for (; i + 4 <= m; i += 4) {
                    int32_t r[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) r[u] = __builtin_amdgcn_readlane(idx, i + u);
                    scatter_terms<1, 4>(acc, dh, r, d, c);
                }
                for (; i < m; ++i) {
                    const int32_t r[1] = {__builtin_amdgcn_readlane(idx, i)};
                    scatter_terms<1, 1>(acc, dh, r, d, c);
                }
            }
            if (wave > 0)
#pragma unroll
                for (int k = 0; k < 8; ++k) part[wave - 1][k][lane] = acc[0][k];
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int q = 0; q < kScatterWaves - 1; ++q)
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc[0][k] += part[q][k][lane];
                scatter_store<ADD>(dtable + (int64_t)v * d + col0 + out0 + 512 * share, acc[0], d - (col0 + out0 + 512 * share));
            }
            __syncthreads();
        }
        if (x >= 0 || k == kScatterLook) return;
        first += 64 * heavy;
        look();
    }
}

// ------------------------------------------------------------------ cross-entropy
// One block per row: maximum and sum of exponentials, then the gradient.  HBM-bound at 6 V bytes per row if the logits are
// read once: up to 4 NR NT of them (32 768) stay in the registers of the block's NT threads between the two passes; wider
// rows (NR = 0) are read twice, the first time with a running maximum.  8192 rows, before (256 threads, two reads) and
// after: V = 32 000 468 -> 282 us (5.6 TB/s), 16 384 208 -> 156, 8000 99 -> 75, 1024 14.1 -> 12.5.

template <int NT>
__device__ __forceinline__ float block_reduce(float v, float *buf, bool is_max) {
    v = is_max ? wave_max(v) : wave_sum(v);
    if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = buf[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r = is_max ? fmaxf(r, buf[w]) : r + buf[w];
    return r;
}

// e: exponentials of the logits relative to the row's maximum, inv: 1 / their sum (relative to the maximum and not to the
// log-sum-exp: the difference of two large numbers is exact, their log-sum-exp is not)
__device__ __forceinline__ uint2 ce_grad(const float4 &e, float inv, int c, int label, float inv_n) {
    float p0 = e.x * inv, p1 = e.y * inv, p2 = e.z * inv, p3 = e.w * inv;
    if (label == c) p0 -= 1.f;
    if (label == c + 1) p1 -= 1.f;
    if (label == c + 2) p2 -= 1.f;
    if (label == c + 3) p3 -= 1.f;
    return make_uint2(pack2bf(p0 * inv_n, p1 * inv_n), pack2bf(p2 * inv_n, p3 * inv_n));
}

template <int NT, int NR>
__global__ __launch_bounds__(NT) void cross_entropy_kernel(float *loss_rows, bf16_t *dlogits, const float *logits,
                                                           const int32_t *labels, int V, float inv_n) {
    __shared__ float smax[NT / 64], ssum[NT / 64];
    const int64_t row = blockIdx.x;
    const int label = labels[row];
    const float4 *z = reinterpret_cast<const float4 *>(logits + row * V);
    uint2 *dz = reinterpret_cast<uint2 *>(dlogits + row * V);
    const int nq = V >> 2;
    if (label < 0) {
        if (threadIdx.x == 0) loss_rows[row] = 0.f;
        for (int i = threadIdx.x; i < nq; i += NT) dz[i] = make_uint2(0u, 0u);
        return;
    }
    if constexpr (NR > 0) {
        float4 v[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = threadIdx.x + NT * k;
            v[k] = i < nq ? z[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < NR; ++k) mx = fmaxf(fmaxf(fmaxf(mx, v[k].x), fmaxf(v[k].y, v[k].z)), v[k].w);
        mx = block_reduce<NT>(mx, smax, true);
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            v[k] = make_float4(__expf(v[k].x - mx), __expf(v[k].y - mx), __expf(v[k].z - mx), __expf(v[k].w - mx));
            sum += (v[k].x + v[k].y) + (v[k].z + v[k].w);
        }
        sum = block_reduce<NT>(sum, ssum, false);
        if (threadIdx.x == 0) loss_rows[row] = __logf(sum) + (mx - logits[row * V + label]);
        const float inv = 1.0f / sum;
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int i = threadIdx.x + NT * k;
            if (i < nq) dz[i] = ce_grad(v[k], inv, i * 4, label, inv_n);
        }
        return;
    }
    float mx = -INFINITY, sum = 0.f;
    for (int i = threadIdx.x; i < nq; i += NT) {
        const float4 v = z[i];
        const float m4 = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
        if (m4 > mx) {
            sum *= __expf(mx - m4);
            mx = m4;
        }
        sum += __expf(v.x - mx) + __expf(v.y - mx) + __expf(v.z - mx) + __expf(v.w - mx);
    }
    const float bmx = block_reduce<NT>(mx, smax, true);
    sum = block_reduce<NT>(mx == -INFINITY ? 0.f : sum * __expf(mx - bmx), ssum, false);
    if (threadIdx.x == 0) loss_rows[row] = __logf(sum) + (bmx - logits[row * V + label]);
    const float inv = 1.0f / sum;
    for (int i = threadIdx.x; i < nq; i += NT) {
        const float4 v = z[i];
        dz[i] = ce_grad(make_float4(__expf(v.x - bmx), __expf(v.y - bmx), __expf(v.z - bmx), __expf(v.w - bmx)), inv, i * 4, label, inv_n);
    }
}

// fixed-order sum with one block of 1024 threads
__global__ __launch_bounds__(1024) void reduce_sum_kernel(float *out, const float *in, int64_t n, float scale,
                                                          int accumulate) {
    __shared__ float part[16];
    float s = 0.f;
    for (int64_t i = threadIdx.x; i < n; i += 1024) s += in[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int i = 0; i < 16; ++i) t += part[i];
        out[0] = (accumulate ? out[0] : 0.f) + scale * t;
    }
}

// delta[b,h,t] = sum_j do[b,t,h,j] o[b,t,h,j]; hd/8 lanes per (token, head)
__global__ __launch_bounds__(256) void attn_delta_kernel(float *delta, const bf16_t *dout, int64_t lddo,
                                                         const bf16_t *o, int64_t ldo, int B, int T, int H, int hd) {
    const int lpg = hd >> 3;  // lanes per group: 8 or 16
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t grp = idx / lpg;
    const int li = (int)(idx % lpg);
    const int64_t total = (int64_t)B * T * H;
    float s = 0.f;
    int64_t row = 0;
    int h = 0;
    if (grp < total) {
        row = grp / H;
        h = (int)(grp % H);
        float a[8], b[8];
        unpack8(*reinterpret_cast<const uint4 *>(dout + row * lddo + (int64_t)h * hd + li * 8), a);
        unpack8(*reinterpret_cast<const uint4 *>(o + row * ldo + (int64_t)h * hd + li * 8), b);
#pragma unroll
        for (int k = 0; k < 8; ++k) s += a[k] * b[k];
    }
    for (int off = lpg >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (grp < total && li == 0) {
        const int64_t b = row / T, t = row % T;
        delta[(b * H + h) * T + t] = s;
    }
}

__global__ __launch_bounds__(256) void fill_kernel(uint32_t *p, uint32_t v, size_t n) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t st = (size_t)gridDim.x * 256;
    for (; i < n; i += st) p[i] = v;
}

inline unsigned blocks_for(int64_t work, int per_block) { return (unsigned)((work + per_block - 1) / per_block); }

}  // namespace

hipError_t transpose_bf16(const TransposeArgs &t, hipStream_t s) {
    if (t.rows <= 0 || t.cols <= 0 || t.nb0 <= 0 || t.nb1 <= 0) return hipErrorInvalidValue;
    if ((t.rows & 7) || (t.cols & 7) || (t.ld_in & 7) || (t.ld_out & 7)) return hipErrorInvalidValue;
    if ((t.in_s0 & 7) || (t.in_s1 & 7) || (t.out_s0 & 7) || (t.out_s1 & 7)) return hipErrorInvalidValue;
    if (((uintptr_t)t.in & 15) || ((uintptr_t)t.out & 15)) return hipErrorInvalidValue;
    if (t.ld_in < t.cols || t.ld_out < t.rows) return hipErrorInvalidValue;
    const int64_t nz = (int64_t)t.nb0 * t.nb1;
    if (nz > 65535) return hipErrorInvalidValue;
    dim3 grid((t.cols + kTrCols - 1) / kTrCols, (t.rows + kTrRows - 1) / kTrRows, (unsigned)nz);
    hipLaunchKernelGGL(transpose_kernel, grid, dim3(256), 0, s, t);
    return hipGetLastError();
}

// (norm_store) forward and backward, us: 65 536 x 5120 738 -> 714, 16 384 x 4096 159 -> 142, 65 536 x 1024 152 -> 134, 8192 x 8192 169 -> 148; results of
// less than twice the caches may be there yet when their reader comes.
static bool past_caches(int64_t n, int32_t d) { return n * d * 2 >= (int64_t)64 << 20; }
hipError_t rmsnorm_fwd(bf16_t *y, const bf16_t *x, const bf16_t *gain, int64_t n, int32_t d, float eps,
                       hipStream_t s) {
    if (n <= 0 || d <= 0 || (d & 7) || d > 8192) return hipErrorInvalidValue;
    const unsigned grid = blocks_for(n, 4);
    // Few rows: by the next multiple of 1024 columns (a kernel for wider rows would load past the end of this one for nothing), rows
    // packed: 5136 x 3904 14.7 -> 13.4 us, 8192 x 5120 25.9 -> 24.1, 3117 x 6144 16.7 -> 13.8, 4026 x 7368 22.0 -> 18.4.  Many: with fewer waves,
    // 24 576 x 5120 98 -> 94, 65 536 x 3072 146 -> 141, x 5120 248 -> 241, x 6144 298 -> 288; 16 384 x 4096 39.5 -> 40.6.
    const int k = (d - 1) / 1024;
    const auto pick = [&](auto nt) {
        constexpr bool NT = decltype(nt)::value;
        decltype(&rmsnorm_fwd_kernel<2, false, NT>) const few[8] = {
            rmsnorm_fwd_kernel<2, false, NT>, rmsnorm_fwd_kernel<4, false, NT>, rmsnorm_fwd_kernel<6, true, NT>, rmsnorm_fwd_kernel<8, true, NT>,
            rmsnorm_fwd_kernel<10, true, NT>, rmsnorm_fwd_kernel<12, true, NT>, rmsnorm_fwd_kernel<14, true, NT>, rmsnorm_fwd_kernel<16, true, NT>};
        const auto many = k <= 1 ? few[k] : k <= 3 ? rmsnorm_fwd_kernel<8, false, NT> : k == 4 ? rmsnorm_fwd_kernel<10, false, NT> : rmsnorm_fwd_kernel<16, false, NT>;
        return n < 20480 ? few[k] : many;
    };
    const auto kernel = past_caches(n, d) ? pick(std::true_type{}) : pick(std::false_type{});
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, y, x, gain, n, d, eps);
    return hipGetLastError();
}

size_t rmsnorm_bwd_ws_floats(int32_t d) { return (size_t)kNormBwdBlocks * (size_t)d; }

hipError_t rmsnorm_bwd(bf16_t *dx_out, float *dgain, const bf16_t *dy, const bf16_t *x, const bf16_t *gain,
                       const bf16_t *dres, float *partial, int64_t n, int32_t d, float eps, hipStream_t s,
                       int accumulate_dgain) {
    if (n <= 0 || d <= 0 || (d & 7) || d > 8192) return hipErrorInvalidValue;
    const int rpb = d <= 1024 ? 4 : 1;   // rows a block has in hand
    const unsigned grid = (unsigned)std::min<int64_t>((n + rpb - 1) / rpb, kNormBwdBlocks);
    const auto pick = [&](auto nt) {
        constexpr bool NT = decltype(nt)::value;
        return d <= 512 ? rmsnorm_bwd_kernel<1, 1, NT> : d <= 1024 ? rmsnorm_bwd_kernel<2, 1, NT> : d <= 2048 ? rmsnorm_bwd_kernel<1, 4, NT>
             : d <= 4096 ? rmsnorm_bwd_kernel<2, 4, NT> : d <= 6144 ? rmsnorm_bwd_kernel<3, 4, NT> : rmsnorm_bwd_kernel<4, 4, NT>;
    };
    const auto kernel = past_caches(n, d) ? pick(std::true_type{}) : pick(std::false_type{});
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, dx_out, partial, dy, x, gain, dres, n, d, eps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_colsum(dgain, partial, (int)grid, d, accumulate_dgain, s);
    return hipGetLastError();
}

// ---- RMSNorm backward for callers that may not allocate: the partial-gain-gradient workspace is a file-scope
// device array instead of a caller buffer.  Its name is only a host-side handle; the device address is looked up
// once per device (each device holds its own copy) and passed to the kernels like any other workspace.
constexpr int kStaticNormMaxD = 8192;
static __device__ __align__(256) float scratch[(size_t)kNormBwdBlocks * kStaticNormMaxD];  // 16 MiB per device
constexpr int kMaxDevices = 64;

hipError_t rmsnorm_bwd_static(bf16_t *dx_out, float *dgain, const bf16_t *dy, const bf16_t *x, const bf16_t *gain,
                              const bf16_t *dres, int64_t n, int32_t d, float eps, hipStream_t s) {
    static std::atomic<float *> scratch_of_device[kMaxDevices];
    if (d <= 0 || d > kStaticNormMaxD) return hipErrorInvalidValue;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    float *ptr = scratch_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        scratch_of_device[dev].store(ptr, std::memory_order_release);  // same value from every thread
    }
    // every partial row that the column sum reads is written by the first kernel of this call: nothing to clear
    return rmsnorm_bwd(dx_out, dgain, dy, x, gain, dres, ptr, n, d, eps, s, 0);
}

size_t bias_grad_ws_floats(int32_t cols) { return (size_t)kBiasGradRowBlocks * (size_t)cols; }

hipError_t bias_grad(float *db, const bf16_t *x, int64_t ld, int64_t n, int32_t cols, float *ws, hipStream_t s) {
    if (n <= 0 || cols <= 0 || (cols & 7) || (ld & 7)) return hipErrorInvalidValue;
    const int64_t rpb = (n + kBiasGradRowBlocks - 1) / kBiasGradRowBlocks;
    hipLaunchKernelGGL(bias_grad_partial_kernel, dim3(blocks_for(cols / 8, 256), kBiasGradRowBlocks), dim3(256), 0, s, ws, x,
                       ld, n, cols, rpb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_colsum(db, ws, kBiasGradRowBlocks, cols, 0, s);
    return hipGetLastError();
}

hipError_t rope_inplace(bf16_t *x, int64_t ld, int64_t n, int32_t T, int32_t n_heads, int32_t hd, const float *cs,
                        const float *sn, int sign, hipStream_t s) {
    if (n <= 0 || T <= 0 || n_heads <= 0 || (hd & 15) || (ld & 7)) return hipErrorInvalidValue;
    const int64_t total = n * n_heads * (hd >> 4);
    hipLaunchKernelGGL(rope_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, s, x, ld, n, T, n_heads, hd, cs, sn,
                       sign >= 0 ? 1.0f : -1.0f);
    return hipGetLastError();
}

hipError_t swiglu_fwd(bf16_t *sout, const bf16_t *gu, int64_t n, int32_t F, hipStream_t s) {
    if (n <= 0 || F <= 0 || (F & 7)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(blocks_for(n * (F >> 3), 256)), dim3(256), 0, s, sout, gu, n, F);
    return hipGetLastError();
}

hipError_t swiglu_bwd(bf16_t *dgu, const bf16_t *ds, const bf16_t *gu, int64_t n, int32_t F, hipStream_t s) {
    if (n <= 0 || F <= 0 || (F & 7)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(swiglu_bwd_kernel, dim3(blocks_for(n * (F >> 3), 256)), dim3(256), 0, s, dgu, ds, gu, n, F);
    return hipGetLastError();
}

hipError_t embed_gather(bf16_t *h, const bf16_t *table, const int32_t *tokens, int64_t n, int32_t d, hipStream_t s) {
    if (n <= 0 || d <= 0 || (d & 7)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(embed_gather_kernel, dim3(blocks_for(n * (d >> 3), 256)), dim3(256), 0, s, h, table, tokens, n,
                       d);
    return hipGetLastError();
}

ScatterRoute embed_scatter_route(int32_t V, int32_t d) {
    ScatterRoute r;
    // wide shares for big tables; smaller ones where the blocks would be too few for the chip (NC = 1 / 2 / 4 / a block per row, us):
    // 4848 uniform tokens, V = 1096, d = 1280 5.4 / 5.4 / 6.3 / 5.6; 4096 tokens, V = 1024, d = 1024 4.5 / 5.4 / 6.0 / 5.1; 65 536, 2000, 5120
    // 173 / 167 / 188 / 207; 4096, 4000, 4096 16.5 / 16.1 / 16.5 / 18.9; 800, 11 704, 1600 17.8 / 16.0 / 15.6 / 15.2; 65 536, 32 000, 4096
    // 297 / 260 / 213 / 217
    const auto blocks = [&](int nc) { return (int64_t)((V + 7) / 8) * ((d + 512 * nc - 1) / (512 * nc)); };
    r.nc = d > 1024 && blocks(4) >= 1200 ? 4 : d > 512 && blocks(2) >= 260 ? 2 : 1;
    r.ranges = (int)blocks_for(d, 512 * r.nc);
    // Rows of more than kScatterHeavy terms first, in blocks of their own that look through 64 kScatterLook rows of a column range: a frequent token's row that
    // comes late is summed alone at the end.  Measured on 288 tables (V 5000 .. 64 000, one to three ranges, 4096 .. 65 536 ids of a Zipf law scattered over the table,
    // or uniform ones), without -> with such blocks.
    // Their number is groups x ranges x 4.  From 46 groups x ranges on, three quarters of a block per compute unit: 47 .. 64 1.06 times faster on average (65 536 ids,
    // 12 000 x 1280 88 -> 78 us, 8000 x 4096 162 -> 149); fewer hold too many long rows each: at 40 from 10 000 x 1280
    // 82 -> 95 to 5000 x 4096 173 -> 166.
    // And from two terms to three rows x ranges on, which only the device knows: what the long rows save grows with the terms, what the looking costs with rows x
    // ranges.  1.04 times faster on average (32 000 x 4096, 65 536 ids 230 -> 218; uniform ids 211 -> 214); below that it costs 2 to 4 % (16 384 ids, 32 000 x 4096 137 -> 142,
    // 64 000 x 4096 235 -> 246), and blocks that leave at once up to 1 % (235 -> 236).
    const int groups = (int)blocks_for(V, 64 * kScatterLook);
    r.heavy = r.nc == 4 && (int64_t)groups * r.ranges >= 46 ? groups : 0;
    r.enough = (int)std::min<int64_t>(INT32_MAX, (int64_t)V * r.ranges * 2 / 3);
    // Several column ranges come side by side: by ranges, the heavy rows of the later ones begin late, and all shares of such a row fall on NC XCDs.
    // Zipf-distributed ids in order of frequency, by ranges -> side by side, us: 65 536 tokens, V = 32 000, d = 4096 328 -> 284 (uniform ids
    // 215 -> 217), d = 5120 418 -> 345, 4096 tokens, V = 1024, d = 4096 30.2 -> 21-23.  Not where narrow blocks come out even or as the better
    // end: with one whole range and a narrower one (65 536, 32 000, 2560) 309 with the lookup, side by side 323; 8192, 4000, 3584 (NC = 2) 60.7,
    // 61.6; nor two ranges of NC = 2 (4096, 1500, 2048: 18.1, 18.7) and NC = 1, tables small enough to be at work all at once.
    r.side = r.nc == 4 ? d >= 2 * 512 * r.nc : r.nc == 2 && d > 2 * 512 * r.nc && d % (512 * r.nc) == 0;
    return r;
}
hipError_t embed_scatter(float *dtable, const bf16_t *dh, const int32_t *row_start, const int32_t *order, int32_t V,
                         int32_t d, bool add, hipStream_t s) {
    if (V <= 0 || d <= 0 || (d & 7)) return hipErrorInvalidValue;
    const ScatterRoute r = embed_scatter_route(V, d);
    const int gx = (int)blocks_for(V, kScatterWaves * r.nc), gy = std::min(gx + r.heavy, 1 << 15);
    const dim3 grid = r.side ? dim3(r.nc * r.ranges, gy, blocks_for(gx + r.heavy, gy)) : dim3(r.nc * (gx + r.heavy), r.ranges), block(64 * kScatterWaves);
    auto kernel = r.nc == 1 ? embed_scatter_kernel<1, false, false> : r.nc == 2 ? embed_scatter_kernel<2, false, false> : embed_scatter_kernel<4, false, false>;
    if (add) kernel = r.nc == 1 ? embed_scatter_kernel<1, true, false> : r.nc == 2 ? embed_scatter_kernel<2, true, false> : embed_scatter_kernel<4, true, false>;
    if (r.side && r.nc == 2) kernel = add ? embed_scatter_kernel<2, true, true> : embed_scatter_kernel<2, false, true>;
    if (r.side && r.nc == 4) kernel = add ? embed_scatter_kernel<4, true, true> : embed_scatter_kernel<4, false, true>;
    hipLaunchKernelGGL(kernel, grid, block, 0, s, dtable, dh, row_start, order, V, d, gx, r.heavy, r.enough);
    return hipGetLastError();
}

hipError_t cross_entropy(float *loss_rows, bf16_t *dlogits, const float *logits, const int32_t *labels, int64_t n,
                         int32_t V, float inv_n, hipStream_t s) {
    if (n <= 0 || V <= 0 || (V & 3)) return hipErrorInvalidValue;
    // the smallest block, and the fewest registers per thread, that hold the row
    const int nt = V <= 8192 ? 256 : V <= 16384 ? 512 : 1024;
    auto kernel = V <= 1024 ? cross_entropy_kernel<256, 1> : V <= 2048 ? cross_entropy_kernel<256, 2>
                : V <= 4096 ? cross_entropy_kernel<256, 4> : V <= 8192 ? cross_entropy_kernel<256, 8>
                : V <= 16384 ? cross_entropy_kernel<512, 8> : V <= 32768 ? cross_entropy_kernel<1024, 8> : cross_entropy_kernel<1024, 0>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(nt), 0, s, loss_rows, dlogits, logits, labels, V, inv_n);
    return hipGetLastError();
}

hipError_t reduce_sum(float *out, const float *in, int64_t n, float scale, int accumulate, hipStream_t s) {
    if (n < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reduce_sum_kernel, dim3(1), dim3(1024), 0, s, out, in, n, scale, accumulate);
    return hipGetLastError();
}

hipError_t attn_delta(float *delta, const bf16_t *dout, int64_t lddo, const bf16_t *o, int64_t ldo, int32_t B,
                      int32_t T, int32_t H, int32_t hd, hipStream_t s) {
    if (hd != 64 && hd != 128) return hipErrorInvalidValue;
    const int64_t total = (int64_t)B * T * H * (hd >> 3);
    hipLaunchKernelGGL(attn_delta_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, s, delta, dout, lddo, o, ldo, B, T,
                       H, hd);
    return hipGetLastError();
}

hipError_t fill_u32(void *p, uint32_t value, size_t n_words, hipStream_t s) {
    if (n_words == 0) return hipSuccess;
    size_t blocks = (n_words + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, s, reinterpret_cast<uint32_t *>(p), value,
                       n_words);
    return hipGetLastError();
}

}  // namespace mt
