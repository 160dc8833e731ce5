// Shared declarations of the gfx950 library: vector types, bf16 helpers, wave
// reductions and the launchers that the engine and the kernel-level C ABI call.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <atomic>

namespace mt {

typedef uint16_t bf16_t;  // raw bfloat16 bits in memory
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kWave = 64;

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ __forceinline__ float bflo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bfhi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
// round-to-nearest-even pack of two floats (hardware v_cvt_pk_bf16_f32); a in the low half
__device__ __forceinline__ uint32_t pack2bf(float a, float b) {
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ bf16_t f2bf(float a) { return __builtin_bit_cast(bf16_t, (__bf16)a); }
// Logistic function with the hardware reciprocal (1 ulp) instead of the IEEE division sequence (about ten
// instructions): the results are rounded to bf16 right after, and inside a GEMM store the arithmetic of a 256 x 256
// tile runs on four waves.  Every SwiGLU path (stand-alone kernels and GEMM stores) uses this one function.
__device__ __forceinline__ float sigmoid_rcp(float v) { return __builtin_amdgcn_rcpf(1.0f + __expf(-v)); }

// SwiGLU backward of one element: s = silu(g) * u, ds given -> dg, du (shared by the stand-alone kernel and the
// GEMM store that applies it, so both round alike)
__device__ __forceinline__ void swiglu_bwd_elem(float d, float g, float u, float *dg, float *du) {
    const float sg = sigmoid_rcp(g);
    *dg = d * u * sg * (1.0f + g * (1.0f - sg));
    *du = d * g * sg;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

#ifdef __HIPCC__
typedef __attribute__((ext_vector_type(4))) short s16x4;

// acc += a b (16 x 16 x 32, bf16): lane l holds of a and of b row l & 15, reduction indices 8 (l >> 4) .. + 7, and of acc
// column l & 15, rows 4 (l >> 4) .. + 3.  In place in the accumulation registers: through the builtin the compiler gives a large
// set of accumulators new registers every time and moves them back.  It neither sees that this is a matrix instruction: whoever
// reads an accumulator calls mfma16_settle first, and operands come from LDS reads (the wait for those is the
// compiler's as usual), not from a vector instruction right in front.
__device__ __forceinline__ void mfma16_acc(f32x4 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// the same with the accumulator among the vector registers (there are 256 of either kind, and a wave that is alone on its SIMD may use all)
__device__ __forceinline__ void mfma16_acc_v(f32x4 &acc, const bf16x8 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// every accumulator has been written (16 wait states, the slowest of these instructions needs 11) and may be read
__device__ __forceinline__ void mfma16_drain() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// The accumulators have been set (before the first of these instructions, where the compiler would set them right in front of it).
template <int I, int J>
__device__ __forceinline__ void mfma16_begin(f32x4 (&acc)[I][J]) {
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) asm volatile("" : "+a"(acc[i][j]));
    mfma16_drain();
}
// The same as mfma16_drain, for the compiler too.  Where two paths with these instructions meet in front of it, the compiler may move accumulators at
// the end of one of them: that path ends with a mfma16_drain of its own (tests/test_matrix_hazards.py looks for such moves).
template <int I, int J>
__device__ __forceinline__ void mfma16_settle(f32x4 (&acc)[I][J]) {
    mfma16_drain();
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// Tile-row group of the 256 x 256 GEMM kernels: the 32 workgroups of an XCD then cover 4 x 8 tiles and a
// group's A rows are left after two patches.  Measured inside the step against 8 (8 x 4 patches): 14B GEMM class
// +0.9 %, 1.3B +0.9 %, 7B +0.2 %; 3 and 6 lose at 14B.  (Stand-alone timings of one GEMM repeated on the same
// operands favour small groups far more, up to 7 % at K = 11008, but there the operands are still in the memory-side
// cache from the previous repetition.)
constexpr int kGroupMLarge = 4;
// position in the tile order of those kernels -> tile
__device__ __forceinline__ void gemm_tile_of(int pid, int tiles_m, int tiles_n, int group_m, int *tm, int *tn) {
    const int gm = group_m > 0 ? group_m : kGroupMLarge;
    const int group = gm * tiles_n;
    const int first_m = (pid / group) * gm;
    const int gsz = min(tiles_m - first_m, gm);
    *tm = first_m + (pid % group) % gsz;
    *tn = (pid % group) / gsz;
}

// From 128 k-steps on (operand rows of 16 KB and more, whose lines at one k crowd onto few memory channels) a group of four
// rows of 256 x 256 tiles starts its walk over K at an eighth of K of its own, so that the XCDs, which work on different
// groups, read different columns: 16384 x 4096 x 11008 1095 -> 1042 us, x 22016 2303 -> 2116; K = 8192, 13824 and 32000 +- 1 %.
// The start depends on the 256-row tile alone and every NT kernel that takes whole k-steps and all of them in turn (share_nt_kernel
// does not) keeps to it, so that a product's sums run in the same order whichever of their tiles and stores compute it.
constexpr int kStaggerSteps = 128;
__device__ __forceinline__ int gemm_walk_start(int tm, int nk) {
    if (nk < kStaggerSteps) return 0;
    int h = tm >> 2;
    h ^= h >> 1; h ^= h >> 2; h ^= h >> 4;   // any eight groups in arithmetic progression by a power of two: distinct low bits
    return (h & 7) * (nk >> 3);
}

// Eight bf16 columns of a row that need not be complete or aligned.  Class of an access of the columns col .. + 7 of [.., n] with row
// pitch ld at p: 16 (bytes at once), 8, or 2 (element by element, columns < n only).
__device__ __forceinline__ int row_access(const void *p, int64_t ld, int col, int n) {
    return col + 8 > n ? 2 : !(ld & 7) && !((uintptr_t)p & 15) ? 16 : !(ld & 3) && !((uintptr_t)p & 7) ? 8 : 2;
}
__device__ __forceinline__ void row_add8(float (&v)[8], const bf16_t *r, int access, int col, int n) {
    if (access >= 8) {
        const uint4 u = access == 16 ? *reinterpret_cast<const uint4 *>(r)
                                     : uint4{reinterpret_cast<const uint2 *>(r)[0].x, reinterpret_cast<const uint2 *>(r)[0].y,
                                             reinterpret_cast<const uint2 *>(r)[1].x, reinterpret_cast<const uint2 *>(r)[1].y};
        v[0] += bflo(u.x); v[1] += bfhi(u.x); v[2] += bflo(u.y); v[3] += bfhi(u.y);
        v[4] += bflo(u.z); v[5] += bfhi(u.z); v[6] += bflo(u.w); v[7] += bfhi(u.w);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (col + e < n) v[e] += bf2f(r[e]);
    }
}
__device__ __forceinline__ void row_store8(bf16_t *c, const float (&v)[8], int access, int col, int n) {
    const uint4 u = {pack2bf(v[0], v[1]), pack2bf(v[2], v[3]), pack2bf(v[4], v[5]), pack2bf(v[6], v[7])};
    if (access == 16) {
        *reinterpret_cast<uint4 *>(c) = u;
    } else if (access == 8) {
        reinterpret_cast<uint2 *>(c)[0] = uint2{u.x, u.y};
        reinterpret_cast<uint2 *>(c)[1] = uint2{u.z, u.w};
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (col + e < n) c[e] = f2bf(v[e]);
    }
}

#endif  // __HIPCC__

// ---------------------------------------------------------------- launchers (host side)
// More than 48 KB of dynamic LDS have to be asked for once per kernel (done: that kernel's own flag; threads that launch
// it for the first time at the same time may both ask).
template <typename K>
inline hipError_t ensure_lds(K kernel, size_t bytes, std::atomic<bool> *done) {
    if (done->load(std::memory_order_relaxed) || bytes <= 48 * 1024) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done->store(true, std::memory_order_relaxed);
    return e;
}

// Every launcher validates nothing: callers (engine, C ABI wrappers) check shapes first.

// C[M,N] = A[M,K] . B[N,K]^T (+ R) ; A, B bf16 with the reduction index contiguous.
//   out_fp32 = 0: C bf16, optional residual R bf16 [M,N] added before rounding
//   out_fp32 = 1: C fp32; accumulate = 1 adds to the existing C
//   bias: optional per-column bf16 vector added before the residual and the rounding (bf16 output only)
struct GemmArgs {
    const bf16_t *A; int64_t lda;
    const bf16_t *B; int64_t ldb;
    void *C; int64_t ldc;
    const bf16_t *R; int64_t ldr;
    int32_t M, N, K;
    int32_t out_fp32, accumulate;
    const bf16_t *bias = nullptr;  // optional bf16 [N], added to every row (bf16 output only)
    // optional rotary embedding fused into the store (gemm_nt only, see gemm_nt_fuses_rope): columns
    // [0, rope_cols) are heads of 128 whose pairs (j, j + 64) are rotated by the angle of position
    // row % rope_T; tables cos/sin [rope_T][64] fp32
    const float *rope_cos = nullptr, *rope_sin = nullptr;
    int32_t rope_T = 0, rope_cols = 0;
    // optional SwiGLU fused into the store (gemm_nt only, see gemm_nt_fuses_glu): B is [2 glu_F, K], gate rows
    // then up rows (N = 2 glu_F); a tile computes the gate and the up columns of the same 128 indices and stores
    // glu_out[M, glu_F] = silu(gate) * up (bf16, from the bf16-rounded gate and up, as a separate pass over C would).
    // C may then be NULL (gate | up themselves are not stored).
    int32_t glu_F = 0;
    bf16_t *glu_out = nullptr; int64_t ld_glu = 0;
    // optional SwiGLU backward fused into the store (gemm_nt only, see gemm_nt_fuses_glu_bwd): the product is
    // ds [M, N] (N = F, the gradient of the activation, rounded to bf16 as a stored ds would be); with the forward's
    // gate | up in glu_bwd_gu [M, 2N] the kernel stores C [M, 2N] = dgate | dup instead of ds
    const bf16_t *glu_bwd_gu = nullptr; int64_t ld_glu_bwd = 0;
    // optional split of the reduction (gemm_tn only) for tile counts that fill the last round of workgroups badly (see
    // gemm_tn_pick_split): the K range is cut into split_k chunks that run as separate workgroups, for the tiles of the last
    // round (256 x 256 kernel) or for all tiles (smaller ones); chunk 0 stores to C, chunk s > 0 to split_ws + (s - 1) M N
    // (fp32, pitch N; where a tile is not split, left as it is), and a second kernel adds them to C in that order.  With
    // split_k > 1, and in the kernels with smaller tiles always, every output is made of as many partial sums as its size
    // asks for (1 to 6), whether they have a workgroup each or share one; with a split that is not gemm_tn_pick_split's own of at
    // least split_k.
    int32_t split_k = 1;
    float *split_ws = nullptr;
    // tile order of the large-grid kernels: tile rows per group (a group is walked column by column); 0 = kGroupMLarge
    int32_t group_m = 0;
};
// of_rows: the product's rows are some of a larger one's, of that many, and are to be summed in the same order as there (they then equal its rows
// bit for bit; K < 8192, see gemm_walk_start); 0: a product of its own.
hipError_t gemm_nt(const GemmArgs &g, hipStream_t s, int32_t of_rows = 0);
// The kernels with smaller tiles behind gemm_nt and gemm_tn (same arguments, no fused rotary / SwiGLU stores; the caller
// has checked the operands).  gemm_nt_ring takes any K % 8 == 0; gemm_tn_ring leaves the chunks of a split unreduced; every
// output is the sum of at least partial_sums partial sums.
// l...: rows that are not whole lines, s...: reductions shared among waves (both NT only, first < 0); wide...: gemm_nt's own 256 x 320, 256 x 192.
enum class RingTile { none, t256x128, t128x128, t128x64, t64x64, l128x128, l128x64, l64x64, wide320, wide192, s128x64, s64x64, s32x64, s32x32 };
// first >= 0: only the 256 x 256 tiles from position `first` of that kernel's tile order on (gemm_nt has covered the others).
hipError_t gemm_nt_ring(const GemmArgs &g, RingTile tile, int first, hipStream_t s);
hipError_t gemm_tn_ring(const GemmArgs &g, RingTile tile, int partial_sums, hipStream_t s);
// true when gemm_nt would apply g.rope_* in its epilogue for this problem (large grid, K % 64 == 0, head-aligned
// columns); otherwise a call with rope_cos set fails with hipErrorNotSupported and the caller rotates separately
bool gemm_nt_fuses_rope(const GemmArgs &g);
// the same for g.glu_*: large grid, K % 64 == 0, glu_F % 128 == 0, bf16 output without residual or bias
bool gemm_nt_fuses_glu(const GemmArgs &g);
// and for g.glu_bwd_*: large grid, K % 64 == 0, N % 8 == 0, bf16 output without residual or bias
bool gemm_nt_fuses_glu_bwd(const GemmArgs &g);
// C[M,N] = A^T . B with A given as [K, M] and B as [K, N] (lda, ldb their row pitches): the weight-gradient
// form dW = dY^T X taken straight from token-major activations.  fp32 output (accumulate optional);
// needs K % 64 == 0, M % 8 == 0, N % 8 == 0; returns hipErrorNotSupported otherwise (callers then transpose
// the operands and use gemm_nt).
hipError_t gemm_tn(const GemmArgs &g, hipStream_t s);
// Reduction split for gemm_tn that minimises the estimated time of an M x N x K weight-gradient product on n_cu
// compute units without summing it in longer chains than its size allows, 1 = none; the workspace is (split - 1) * M * N floats.
int gemm_tn_pick_split(int64_t M, int64_t N, int64_t K, int n_cu);
// What gemm_nt (without a fused store) and gemm_tn take for a product, for tests and tools (no launch; a diagnostic override is left
// out).  nt: the first `whole` tiles of 256 x 256 go to that kernel, the others to tiles of tile_m x tile_n (0: there are none).
// tn: tiles of tile_m x tile_n, `whole` of which a workgroup walks alone in the 256 x 256 kernel.
void gemm_nt_route(const GemmArgs &g, int *whole, int *tile_m, int *tile_n);
int gemm_nt_sharers(const GemmArgs &g);   // waves that share the reduction of such a tile
// its tile fetches whole lines of rows that are not whole lines (line_nt_kernel)
bool gemm_nt_fetches_lines(const GemmArgs &g);
void gemm_tn_route(const GemmArgs &g, int *whole, int *tile_m, int *tile_n);

// out[b][c][r] = in[b][r][c] for r < rows, c < cols (bf16); leading dimensions in elements.
// Two batch levels (b0 < nb0, b1 < nb1) with independent strides on each side.
struct TransposeArgs {
    const bf16_t *in; bf16_t *out;
    int32_t rows, cols;
    int64_t ld_in, ld_out;
    int32_t nb0, nb1;
    int64_t in_s0, in_s1, out_s0, out_s1;
};
hipError_t transpose_bf16(const TransposeArgs &t, hipStream_t s);

hipError_t rmsnorm_fwd(bf16_t *y, const bf16_t *x, const bf16_t *gain, int64_t n, int32_t d, float eps, hipStream_t s);
// dx_out = dres + rmsnorm_backward(dy; x, gain); dgain[d] fp32 (written, or added to when accumulate_dgain:
// rows processed in several calls). partial: >= rmsnorm_bwd_ws_floats(d) floats.
size_t rmsnorm_bwd_ws_floats(int32_t d);
hipError_t rmsnorm_bwd(bf16_t *dx_out, float *dgain, const bf16_t *dy, const bf16_t *x, const bf16_t *gain,
                       const bf16_t *dres, float *partial, int64_t n, int32_t d, float eps, hipStream_t s,
                       int accumulate_dgain = 0);

// The same with the workspace in a file-scope device array of the library (d <= 8192): no allocation, but calls that
// overlap on one device share that array and race.
hipError_t rmsnorm_bwd_static(bf16_t *dx_out, float *dgain, const bf16_t *dy, const bf16_t *x, const bf16_t *gain,
                              const bf16_t *dres, int64_t n, int32_t d, float eps, hipStream_t s);

// In-place rotation of the first n_heads heads of each row of x [n, ld]; cos/sin tables [T, hd/2] fp32;
// position of row r is r % T; sign +1 forward, -1 inverse.
hipError_t rope_inplace(bf16_t *x, int64_t ld, int64_t n, int32_t T, int32_t n_heads, int32_t hd, const float *cs,
                        const float *sn, int sign, hipStream_t s);

// gu [n, 2F] (gate | up) -> s [n, F]
hipError_t swiglu_fwd(bf16_t *sout, const bf16_t *gu, int64_t n, int32_t F, hipStream_t s);
// dgu [n, 2F] from ds [n, F] and gu
hipError_t swiglu_bwd(bf16_t *dgu, const bf16_t *ds, const bf16_t *gu, int64_t n, int32_t F, hipStream_t s);

hipError_t embed_gather(bf16_t *h, const bf16_t *table, const int32_t *tokens, int64_t n, int32_t d, hipStream_t s);
// dtable[V,d] fp32: row v = sum of dh rows listed in order[start[v] .. start[v+1]), added to what it holds or (fully) written
hipError_t embed_scatter(float *dtable, const bf16_t *dh, const int32_t *row_start, const int32_t *order, int32_t V,
                         int32_t d, bool add, hipStream_t s);
// Its kernel: blocks of 512 nc columns in so many ranges, side by side or one after the other; blocks in front (a range's) for the longest rows, if the lists
// have `enough` terms
struct ScatterRoute {
    int nc, ranges;
    bool side;
    int heavy, enough;
};
ScatterRoute embed_scatter_route(int32_t V, int32_t d);

// Per row: loss_rows[r] = logsumexp(z_r) - z_r[label] (0 for ignored rows); dlogits bf16 = (softmax - onehot) * inv_n
hipError_t cross_entropy(float *loss_rows, bf16_t *dlogits, const float *logits, const int32_t *labels, int64_t n,
                         int32_t V, float inv_n, hipStream_t s);
// out[0] = (accumulate ? out[0] : 0) + scale * sum(in[0..n)) , one block, fixed order
hipError_t reduce_sum(float *out, const float *in, int64_t n, float scale, int accumulate, hipStream_t s);
// db[cols] fp32 (written) = sum over the n rows of x [n, ld] bf16; ws: >= bias_grad_ws_floats(cols) floats
size_t bias_grad_ws_floats(int32_t cols);
hipError_t bias_grad(float *db, const bf16_t *x, int64_t ld, int64_t n, int32_t cols, float *ws, hipStream_t s);

// Flash attention (causal, grouped KV heads).  q/k/v/o rows are tokens (b*T + t); head h occupies
// columns [h*hd, (h+1)*hd) from the given base pointer with the given leading dimension.
// lse [B, Hq, T] fp32 = log sum_u exp(s_tu) of the scaled scores.
struct AttnArgs {
    int32_t B, T, Hq, Hkv, hd;
    float scale;
    const bf16_t *q; int64_t ldq;
    const bf16_t *k; int64_t ldk;
    const bf16_t *v; int64_t ldv;
    bf16_t *o; int64_t ldo;
    float *lse;
    // backward only
    const bf16_t *dout; int64_t lddo;
    float *delta;  // [B,Hq,T] rowsum(do * o), written
    bf16_t *dq; int64_t lddq;
    bf16_t *dk; int64_t lddk;
    bf16_t *dv; int64_t lddv;
    // optional, backward only: q and k had a rotary embedding applied before the attention (pairs (j, j + hd/2),
    // tables cos/sin [T][hd/2] fp32); dq and dk are then rotated back by the row's angle as they are stored
    const float *rope_cos = nullptr, *rope_sin = nullptr;
};
hipError_t flash_fwd(const AttnArgs &a, hipStream_t s);
// delta[b,h,t] = sum_j do[b,t,h,j] * o[b,t,h,j]
hipError_t attn_delta(float *delta, const bf16_t *dout, int64_t lddo, const bf16_t *o, int64_t ldo, int32_t B, int32_t T,
                      int32_t H, int32_t hd, hipStream_t s);
hipError_t flash_bwd(const AttnArgs &a, hipStream_t s);   // delta, dq, dk, dv
// What the forward, dQ and dK/dV launch for this problem: rows of a block (queries; keys of dK/dV), sets of waves that share it, and whether one
// workgroup per compute unit goes through a list of them (group: see chain_map).  For tests and tools, no launch.
struct AttnKernel {
    int rows, sets;
    bool list;
    int group;
};
void flash_kernels(const AttnArgs &a, AttnKernel (&k)[3]);
// dQ and dK/dV share a launch (where dK and dV are apart from the inputs)
bool flash_bwd_together(const AttnArgs &a);

hipError_t fill_u32(void *p, uint32_t value, size_t n_words, hipStream_t s);

}  // namespace mt
